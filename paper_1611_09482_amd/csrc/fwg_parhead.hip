// The head of the time-parallel gated bf16 stacks with S = H = 512 and 256 classes (gfx950): skip sum
// over all layers, relu, first 1x1, relu, output 1x1, one kernel from the z rows to the logits
// (v_mfma_f32_16x16x32_bf16, fp32 accumulation).
//
// As three GEMM launches (fwg_parallel.hip, 128 x 128 tiles) the head read the z rows four times (once
// per column tile), wrote and re-read the skip sums and hidden rows, and staged both operands through
// LDS: 390 us per 65,536 rows of a 30-layer model (~500 TFLOP/s).  Here a block takes BM rows through
// all three products at full width:
//  - the products are transposed, D[channel][row] = W[channel][k] X[row][k]; wave w of 8 owns 64 of the
//    512 channels (32 of the 256 classes) for all BM rows, so no weight is loaded twice in a block and
//    weights go straight from the L2 into registers as pre-packed 1 KB fragments, each slot refilled
//    one k-tile (64 k) ahead as soon as its products are issued;
//  - only the rows go through LDS (the z rows in double-buffered k-tiles, one barrier each; then the
//    whole skip-sum and hidden rows, 1 KB per row): 8 B operands feed 32 products per wave and k-step;
//  - nothing but the logits goes back to memory.
// Measured (30 layers): 65,536 rows 178 us (1,015 TFLOP/s; the three launches 390 us), 32,768 rows 75 us
// (1,204 TFLOP/s; a large library product reaches ~1,130 on this card): the matrix cores bound it.
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

constexpr int R = 64, S = 512, H = 512, Q = 256, NW = 8, NT = 64 * NW;
constexpr int PZ = R + 8, PS = S + 8;  // LDS row strides (bf16): rows spread over the banks

// One product over KT k-tiles of 64: NC channel tiles x NM row tiles per wave.  W: the wave's fragment
// stream (k-tile, k-step, channel tile); the first k-tile's fragments are in w already.
template <int NC>
__device__ __forceinline__ void load_tile(u32x4 (&w)[2][NC], const u32x4 *src, int kt, int lane) {
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int c = 0; c < NC; ++c) w[ks][c] = src[((kt * 2 + ks) * NC + c) * 64 + lane];
}
// Products of one k-tile from rows at `x` (row stride `px`), refilling each fragment from k-tile `next`.
template <int NC, int NM>
__device__ __forceinline__ void tile(f32x4 (&acc)[NC][NM], u32x4 (&w)[2][NC], const uint16_t *x, int px, const u32x4 *src,
                                     int next, int lane) {
  const int n = lane & 15, q = lane >> 4;
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    u32x4 b[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) b[m] = lds16(x + (16 * m + n) * px + 32 * ks + 8 * q);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int m = 0; m < NM; ++m) acc[c][m] = mfma(w[ks][c], b[m], acc[c][m]);
      __builtin_amdgcn_sched_barrier(0);
      w[ks][c] = src[((next * 2 + ks) * NC + c) * 64 + lane];
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int NC, int NM>
__device__ __forceinline__ void start(f32x4 (&acc)[NC][NM], const float *bias, int ch, int q) {
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const float4 b = *(const float4 *)(bias + ch + 16 * c + 4 * q);
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[c][m] = f32x4{b.x, b.y, b.z, b.w};
  }
}

template <int BM>
__global__ void __launch_bounds__(NT, BM == 64 ? 4 : 2) head_kernel(ParHead g) {
  constexpr int NM = BM / 16;
  extern __shared__ float4 lds_raw[];
  uint16_t *sm = (uint16_t *)lds_raw;  // z k-tiles [2][BM][PZ], then rows [BM][PS]
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, q = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.x * BM, L = g.L;
  const u32x4 *ws = (const u32x4 *)g.packed + (size_t)w * L * 8 * 64;
  const u32x4 *wh = (const u32x4 *)g.packed + ((size_t)NW * L * 8 + (size_t)w * 64) * 64;
  const u32x4 *wo = (const u32x4 *)g.packed + ((size_t)NW * L * 8 + NW * 64 + (size_t)w * 32) * 64;

  // z rows: thread -> row tid / 8 (+ 64), 16-byte piece tid % 8 of a k-tile (= one layer)
  constexpr int NZ = BM / 64;
  const uint16_t *zp[NZ];
#pragma unroll
  for (int i = 0; i < NZ; ++i) {
    const int m = min(m0 + (tid >> 3) + 64 * i, g.M - 1);  // rows past the end repeat the last one
    zp[i] = (const uint16_t *)g.z + (long long)m * g.ldz + 8 * (tid & 7);
  }
  u32x4 zr[NZ];
  f32x4 acc[4][NM];
  u32x4 wf[2][4];
  load_tile(wf, ws, 0, lane);
#pragma unroll
  for (int i = 0; i < NZ; ++i) zr[i] = *(const u32x4 *)zp[i];
  start(acc, g.skip_b, 64 * w, q);
#pragma unroll
  for (int i = 0; i < NZ; ++i) *(u32x4 *)(sm + ((tid >> 3) + 64 * i) * PZ + 8 * (tid & 7)) = zr[i];
  __syncthreads();
  for (int kt = 0; kt < L; ++kt) {
    const int nx = kt + 1 < L ? kt + 1 : kt;
#pragma unroll
    for (int i = 0; i < NZ; ++i) zr[i] = *(const u32x4 *)(zp[i] + (long long)nx * R);
    tile(acc, wf, sm + (kt & 1) * BM * PZ, PZ, ws, nx, lane);
    uint16_t *dst = sm + ((kt + 1) & 1) * BM * PZ;
#pragma unroll
    for (int i = 0; i < NZ; ++i) *(u32x4 *)(dst + ((tid >> 3) + 64 * i) * PZ + 8 * (tid & 7)) = zr[i];
    __syncthreads();
  }
  // relu(skip sum) rows, over the z k-tiles (no wave reads those any more)
  load_tile(wf, wh, 0, lane);
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int m = 0; m < NM; ++m) lds8(sm + (16 * m + n) * PS + 64 * w + 16 * c + 4 * q, pack4(relu4(acc[c][m])));
  start(acc, g.head_b, 64 * w, q);
  __syncthreads();
  for (int kt = 0; kt < S / 64; ++kt) tile(acc, wf, sm + 64 * kt, PS, wh, kt + 1 < S / 64 ? kt + 1 : kt, lane);
  __syncthreads();
  // relu(hidden) rows over them
  u32x4 wq[2][2];
  load_tile(wq, wo, 0, lane);
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int m = 0; m < NM; ++m) lds8(sm + (16 * m + n) * PS + 64 * w + 16 * c + 4 * q, pack4(relu4(acc[c][m])));
  f32x4 lg[2][NM];
  start(lg, g.out_b, 32 * w, q);
  __syncthreads();
  for (int kt = 0; kt < H / 64; ++kt) tile(lg, wq, sm + 64 * kt, PS, wo, kt + 1 < H / 64 ? kt + 1 : kt, lane);
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    const int row = m0 + 16 * m + n;
    if (row >= g.M) continue;
    const int b = row / g.Tcur, j = row - b * g.Tcur;
    float *dst = g.logits + ((long long)b * g.n_steps + g.s0 + j) * Q + 32 * w + 4 * q;
#pragma unroll
    for (int c = 0; c < 2; ++c) *(float4 *)(dst + 16 * c) = make_float4(lg[c][m][0], lg[c][m][1], lg[c][m][2], lg[c][m][3]);
  }
}

// Fragment (channel tile, k-step) of M[out][k] gives lane i the 8 values M[16 tile + i % 16][32 ks + 8 (i / 16)
// + j].  One matrix of K columns into a wave's streams of nc channel tiles: fragment (k-tile kt, k-step ks, tile
// c) of wave w at (((w * nkt + kt) * 2 + ks) * nc + c); this call fills k-tiles kt0 .. kt0 + K / 64 - 1 of nkt.
__global__ void pack_kernel(const uint16_t *src, uint4 *dst, int K, int nc, int nkt, int kt0) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x, kts = K / 64;
  if (e >= NW * kts * 2 * nc * 64) return;
  const int i = e % 64, f = e / 64, c = f % nc, ks = f / nc % 2, kt = f / (2 * nc) % kts, w = f / (2 * nc * kts);
  const uint16_t *p = src + (long long)(16 * (nc * w + c) + i % 16) * K + 64 * kt + 32 * ks + 8 * (i / 16);
  dst[((((size_t)w * nkt + kt0 + kt) * 2 + ks) * nc + c) * 64 + i] =
      make_uint4(p[0] | (p[1] << 16), p[2] | (p[3] << 16), p[4] | (p[5] << 16), p[6] | (p[7] << 16));
}

static void pack(const void *src, void *dst, int K, int nc, int nkt, int kt0, hipStream_t s) {
  const int n = NW * (K / 64) * 2 * nc * 64;
  hipLaunchKernelGGL(pack_kernel, dim3((n + 255) / 256), dim3(256), 0, s, (const uint16_t *)src, (uint4 *)dst, K, nc, nkt,
                     kt0);
}

static size_t lds_bytes(int BM) {
  const size_t z = (size_t)2 * BM * PZ * 2, r = (size_t)BM * PS * 2;
  return z > r ? z : r;
}

}  // namespace phd

bool par_head_ok(int kind, int dtype, int C, int S, int H, int Q) {
  return kind == 2 && dtype == 1 && C == phd::R && S == phd::S && H == phd::H && Q == phd::Q;
}

size_t par_head_bytes(int L) { return ((size_t)phd::NW * L * 8 + phd::NW * 64 + phd::NW * 32) * 1024; }

hipError_t set_par_head_lds_limit() {
  hipError_t e = hipFuncSetAttribute((const void *)phd::head_kernel<128>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)phd::lds_bytes(128));
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void *)phd::head_kernel<64>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)phd::lds_bytes(64));
}

hipError_t launch_par_head(const ParHead &g, int rows_per_block, hipStream_t s) {
  if (g.M <= 0) return hipSuccess;
  if (rows_per_block == 128)
    hipLaunchKernelGGL(phd::head_kernel<128>, dim3((g.M + 127) / 128), dim3(phd::NT), phd::lds_bytes(128), s, g);
  else
    hipLaunchKernelGGL(phd::head_kernel<64>, dim3((g.M + 63) / 64), dim3(phd::NT), phd::lds_bytes(64), s, g);
  return hipGetLastError();
}

hipError_t launch_par_head_pack_skip(const void *skip, int l, int L, void *packed, hipStream_t s) {
  phd::pack(skip, packed, phd::R, 4, L, l, s);
  return hipGetLastError();
}

hipError_t launch_par_head_pack(const void *head, const void *out, int L, void *packed, hipStream_t s) {
  char *p = (char *)packed + (size_t)phd::NW * L * 8 * 1024;
  phd::pack(head, p, phd::S, 4, phd::S / 64, 0, s);
  phd::pack(out, p + (size_t)phd::NW * 64 * 1024, phd::H, 2, phd::H / 64, 0, s);
  return hipGetLastError();
}

}  // namespace fwg
