// The head of the time-parallel gated stacks with 256 classes (gfx950; bf16 with R = 64, S = H = 512, or
// float32 with R = 32, S = H = 256): skip sum over all layers, relu, first 1x1, relu, output 1x1, one
// kernel from the z rows to the logits (v_mfma_f32_16x16x32_bf16 or 16x16x4_f32, fp32 accumulation).
//
// As three GEMM launches (fwg_parallel.hip, 128 x 128 tiles) the head read the z rows four times (once
// per column tile), wrote and re-read the skip sums and hidden rows, and staged both operands through
// LDS: 390 us per 65,536 rows of a 30-layer model (~500 TFLOP/s).  Here a block takes BM rows through
// all three products at full width:
//  - the products are transposed, D[channel][row] = W[channel][k] X[row][k]; wave w of 8 owns an
//    eighth of the channels (32 of the 256 classes) for all BM rows, so no weight is loaded twice in a block and
//    weights go straight from the L2 into registers as pre-packed 1 KB fragments, each slot refilled
//    one k-tile (128 bytes of k) ahead as soon as its products are issued;
//  - only the rows go through LDS (the z rows in double-buffered k-tiles, one barrier each; then the
//    whole skip-sum and hidden rows, 1 KB per row): 8 B operands feed 32 products per wave and k-step;
//  - nothing but the logits goes back to memory.
// Measured (30 layers): 65,536 rows 178 us (1,015 TFLOP/s; the three launches 390 us), 32,768 rows 75 us
// (1,204 TFLOP/s; a large library product reaches ~1,130 on this card): the matrix cores bound it.
// float32, 20 layers: 64 x 3,001 steps 2.05 -> 1.75 ms for the whole call.
// BM = 128 halves the weight traffic per row; BM = 64 fits two blocks per compute unit and splits small
// row counts over more of them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fwg_internal.h"
#include "fwg_mfma_dev.h"
#include "fwg_par.h"

namespace fwg {
namespace phd {

using namespace mfd;

// Everything below counts 16-byte pieces, and the two operand types come to the same numbers: a z row of
// one layer is 128 bytes (R = 64 bf16, 32 float32), a skip-sum or hidden row 1 KB (512 and 256), a k-step
// 64 bytes of a row (32 bf16: one product; 16 float32: four products of 4, element j of lane group g
// standing for k = 4g + j on both sides).
constexpr int Q = 256, NW = 8, NT = 64 * NW;
constexpr int ZB = 128, XB = 1024;            // bytes of a z row (one layer) and of a skip-sum or hidden row
constexpr int PZ = ZB + 16, PS = XB + 16;     // LDS row strides: rows spread over the banks

template <typename OT> struct Op;
template <> struct Op<uint16_t> {
  static constexpr int NC = 4;  // channel tiles per wave: 512 channels over 8 waves
  __device__ static __forceinline__ f32x4 mma(const u32x4 &a, const u32x4 &b, f32x4 c) { return mfma(a, b, c); }
  __device__ static __forceinline__ void put4(unsigned char *p, const f32x4 &v) { *(u32x2 *)p = pack4(v); }
};
template <> struct Op<float> {
  static constexpr int NC = 2;  // 256 channels over 8 waves
  __device__ static __forceinline__ f32x4 mma(const u32x4 &a, const u32x4 &b, f32x4 c) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[j]), __uint_as_float(b[j]), c, 0, 0, 0);
    return c;
  }
  __device__ static __forceinline__ void put4(unsigned char *p, const f32x4 &v) { stf4((float *)p, v); }
};

// Four logits at an address that is a float's (the caller's array may start anywhere).
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// One product over k-tiles of 128 bytes: NC channel tiles x NM row tiles per wave.  src: the wave's
// fragment stream (k-tile, k-step, channel tile); the first k-tile's fragments are in w already.
template <int NC>
__device__ __forceinline__ void load_tile(u32x4 (&w)[2][NC], const u32x4 *src, int kt, int lane) {
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int c = 0; c < NC; ++c) w[ks][c] = src[((kt * 2 + ks) * NC + c) * 64 + lane];
}
// Products of one k-tile from rows at `x` (row stride `px`), refilling each fragment from k-tile `next`.
template <typename OT, int NC, int NM>
__device__ __forceinline__ void tile(f32x4 (&acc)[NC][NM], u32x4 (&w)[2][NC], const unsigned char *x, int px,
                                     const u32x4 *src, int next, int lane) {
  const int n = lane & 15, q = lane >> 4;
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    u32x4 b[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) b[m] = *(const u32x4 *)(x + (16 * m + n) * px + 64 * ks + 16 * q);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int m = 0; m < NM; ++m) acc[c][m] = Op<OT>::mma(w[ks][c], b[m], acc[c][m]);
      __builtin_amdgcn_sched_barrier(0);
      w[ks][c] = src[((next * 2 + ks) * NC + c) * 64 + lane];
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Sums start from zero and the bias joins the finished sum (the order with the smaller error against 64 bits,
// and the GEMM kernels').
template <int NC, int NM>
__device__ __forceinline__ void zero(f32x4 (&acc)[NC][NM]) {
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[c][m] = f32x4{0.f, 0.f, 0.f, 0.f};
}
template <int NC, int NM>
__device__ __forceinline__ void add_bias(f32x4 (&acc)[NC][NM], const float *bias, int ch, int q) {
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const float4 b = *(const float4 *)(bias + ch + 16 * c + 4 * q);
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[c][m] += f32x4{b.x, b.y, b.z, b.w};
  }
}

template <typename OT, int BM>
__global__ void __launch_bounds__(NT, BM == 64 ? 4 : 2) head_kernel(ParHead g) {
  constexpr int NM = BM / 16, NC = Op<OT>::NC, E = sizeof(OT), KX = XB / ZB;  // KX: k-tiles of a 1x1
  constexpr int UX = E == 4 ? KX : 1;  // (bf16 unrolled spills its accumulators)
  extern __shared__ float4 lds_raw[];
  unsigned char *sm = (unsigned char *)lds_raw;  // z k-tiles [2][BM][PZ], then rows [BM][PS]
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, q = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.x * BM, L = g.L;
  const u32x4 *ws = (const u32x4 *)g.packed + (size_t)w * L * (2 * NC) * 64;
  const u32x4 *wh = (const u32x4 *)g.packed + (NW * (size_t)L + (size_t)w * KX) * (2 * NC) * 64;
  const u32x4 *wo = (const u32x4 *)g.packed + ((NW * (size_t)L + NW * KX) * (2 * NC) + (size_t)w * KX * 4) * 64;

  // z rows: thread -> row tid / 8 (+ 64), 16-byte piece tid % 8 of a k-tile (= one layer)
  constexpr int NZ = BM / 64;
  // byte offsets from the block's first row (a chunk of many streams x layers may hold more than 4 GB of z rows)
  const char *const zb = (const char *)g.z + (size_t)m0 * (size_t)(g.ldz * E);
  uint32_t zo[NZ];
#pragma unroll
  for (int i = 0; i < NZ; ++i) {
    const int r = min((tid >> 3) + 64 * i, g.M - 1 - m0);  // rows past the end repeat the last one
    zo[i] = (uint32_t)r * (uint32_t)(g.ldz * E) + 16 * (tid & 7);
  }
  u32x4 zr[NZ];
  f32x4 acc[NC][NM];
  u32x4 wf[2][NC];
  load_tile(wf, ws, 0, lane);
#pragma unroll
  for (int i = 0; i < NZ; ++i) zr[i] = *(const u32x4 *)(zb + zo[i]);
  zero(acc);
#pragma unroll
  for (int i = 0; i < NZ; ++i) *(u32x4 *)(sm + ((tid >> 3) + 64 * i) * PZ + 16 * (tid & 7)) = zr[i];
  __syncthreads();
  for (int kt = 0; kt < L; ++kt) {
    const int nx = kt + 1 < L ? kt + 1 : kt;
#pragma unroll
    for (int i = 0; i < NZ; ++i) zr[i] = *(const u32x4 *)(zb + (zo[i] + (uint32_t)nx * ZB));
    tile<OT>(acc, wf, sm + (kt & 1) * BM * PZ, PZ, ws, nx, lane);
    unsigned char *dst = sm + ((kt + 1) & 1) * BM * PZ;
#pragma unroll
    for (int i = 0; i < NZ; ++i) *(u32x4 *)(dst + ((tid >> 3) + 64 * i) * PZ + 16 * (tid & 7)) = zr[i];
    __syncthreads();
  }
  // relu(skip sum) rows, over the z k-tiles (no wave reads those any more)
  auto rows_out = [&]() {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int m = 0; m < NM; ++m)
        Op<OT>::put4(sm + (16 * m + n) * PS + (16 * (NC * w + c) + 4 * q) * E, relu4(acc[c][m]));
  };
  load_tile(wf, wh, 0, lane);
  add_bias(acc, g.skip_b, 16 * NC * w, q);
  rows_out();
  zero(acc);
  __syncthreads();
#pragma unroll (UX)
  for (int kt = 0; kt < KX; ++kt) tile<OT>(acc, wf, sm + ZB * kt, PS, wh, kt + 1 < KX ? kt + 1 : kt, lane);
  __syncthreads();
  // relu(hidden) rows over them
  u32x4 wq[2][2];
  load_tile(wq, wo, 0, lane);
  add_bias(acc, g.head_b, 16 * NC * w, q);
  rows_out();
  f32x4 lg[2][NM];
  zero(lg);
  __syncthreads();
#pragma unroll (UX)
  for (int kt = 0; kt < KX; ++kt) tile<OT>(lg, wq, sm + ZB * kt, PS, wo, kt + 1 < KX ? kt + 1 : kt, lane);
  add_bias(lg, g.out_b, 32 * w, q);
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    const int row = m0 + 16 * m + n;
    if (row >= g.M) continue;
    const int b = row / g.Tcur, j = row - b * g.Tcur;
    float *dst = g.logits + ((long long)b * g.n_steps + g.s0 + j) * Q + 32 * w + 4 * q;
#pragma unroll
    for (int c = 0; c < 2; ++c) *(f32x4_any *)(dst + 16 * c) = lg[c][m];
  }
}

// Fragment (channel tile, k-step) of M[out][k] gives lane i the 16 bytes of row 16 tile + i % 16 at piece
// 4 ks + i / 16.  One matrix with rows of `row` bytes into a wave's streams of nc channel tiles: fragment
// (k-tile kt, k-step ks, tile c) of wave w at (((w * nkt + kt) * 2 + ks) * nc + c); this call fills k-tiles kt0 ..
// kt0 + row / 128 - 1 of nkt.
__global__ void pack_kernel(const unsigned char *src, uint4 *dst, int row, int nc, int nkt, int kt0) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x, kts = row / ZB;
  if (e >= NW * kts * 2 * nc * 64) return;
  const int i = e % 64, f = e / 64, c = f % nc, ks = f / nc % 2, kt = f / (2 * nc) % kts, w = f / (2 * nc * kts);
  // 16 bits at a time: the caller's bf16 arrays may start at any element
  const uint16_t *p = (const uint16_t *)(src + (long long)(16 * (nc * w + c) + i % 16) * row + ZB * kt + 64 * ks + 16 * (i / 16));
  uint32_t v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = p[2 * j] | ((uint32_t)p[2 * j + 1] << 16);
  dst[((((size_t)w * nkt + kt0 + kt) * 2 + ks) * nc + c) * 64 + i] = make_uint4(v[0], v[1], v[2], v[3]);
}

static void pack(const void *src, void *dst, int row, int nc, int nkt, int kt0, hipStream_t s) {
  const int n = NW * (row / ZB) * 2 * nc * 64;
  hipLaunchKernelGGL(pack_kernel, dim3((n + 255) / 256), dim3(256), 0, s, (const unsigned char *)src, (uint4 *)dst, row,
                     nc, nkt, kt0);
}

static size_t lds_bytes(int BM) {
  const size_t z = (size_t)2 * BM * PZ, r = (size_t)BM * PS;
  return z > r ? z : r;
}

template <typename OT, int BM>
static hipError_t set_lds() {
  return hipFuncSetAttribute((const void *)head_kernel<OT, BM>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)lds_bytes(BM));
}
template <typename OT>
static void launch(const ParHead &g, int bm, hipStream_t s) {
  if (bm == 128) hipLaunchKernelGGL((head_kernel<OT, 128>), dim3((g.M + 127) / 128), dim3(NT), lds_bytes(128), s, g);
  else hipLaunchKernelGGL((head_kernel<OT, 64>), dim3((g.M + 63) / 64), dim3(NT), lds_bytes(64), s, g);
}
static int tiles_of(int dtype) { return dtype == 1 ? Op<uint16_t>::NC : Op<float>::NC; }

}  // namespace phd

bool par_head_ok(int kind, int dtype, int C, int S, int H, int Q) {
  const int es = dtype == 1 ? 2 : 4;
  return kind == 2 && C * es == phd::ZB && S * es == phd::XB && H * es == phd::XB && Q == phd::Q;
}

size_t par_head_bytes(int dtype, int L) {
  const size_t kx = phd::XB / phd::ZB;
  return ((L + kx) * 2 * phd::tiles_of(dtype) + kx * 4) * phd::NW * 1024;
}

hipError_t set_par_head_lds_limit() {
  hipError_t e;
  if ((e = phd::set_lds<uint16_t, 64>()) != hipSuccess) return e;
  if ((e = phd::set_lds<uint16_t, 128>()) != hipSuccess) return e;
  if ((e = phd::set_lds<float, 64>()) != hipSuccess) return e;
  return phd::set_lds<float, 128>();
}

hipError_t launch_par_head(const ParHead &g, int dtype, int rows_per_block, hipStream_t s) {
  if (g.M <= 0) return hipSuccess;
  if (dtype == 1) phd::launch<uint16_t>(g, rows_per_block, s);
  else phd::launch<float>(g, rows_per_block, s);
  return hipGetLastError();
}

hipError_t launch_par_head_pack_skip(const void *skip, int dtype, int l, int L, void *packed, hipStream_t s) {
  phd::pack(skip, packed, phd::ZB, phd::tiles_of(dtype), L, l, s);
  return hipGetLastError();
}

hipError_t launch_par_head_pack(const void *head, const void *out, int dtype, int L, void *packed, hipStream_t s) {
  const int nc = phd::tiles_of(dtype), kx = phd::XB / phd::ZB;
  char *p = (char *)packed + (size_t)phd::NW * L * 2 * nc * 1024;
  phd::pack(head, p, phd::XB, nc, kx, 0, s);
  phd::pack(out, p + (size_t)phd::NW * kx * 2 * nc * 1024, phd::XB, 2, kx, 0, s);
  return hipGetLastError();
}

}  // namespace fwg
