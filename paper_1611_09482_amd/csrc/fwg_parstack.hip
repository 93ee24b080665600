// Time-parallel evaluation of a whole gated bf16 stack (R = 64, width 2) with the rows kept on the
// compute unit (gfx950, v_mfma_f32_16x16x32_bf16, fp32 accumulation).
//
// A layer's launch of the per-layer kernel (fwg_parallel.hip) moves ~1.1 KB per row through memory
// (tap rows, the fp32 residual stream in and out, its operand copy, z) for 41 kFLOP and is bound by
// that: 20 us per 65,536 rows and layer.  Here one block takes one stream and runs every layer over
// 256 consecutive steps at a time: the layer inputs stay in LDS (bf16 rows, the operands of the next
// dilated product), the residual stream in registers (fp32, in the accumulator layout), and only z
// (the skip GEMM's rows) and the queues touch memory.  States from before the 256 steps come from
// the layer's queue, which the block itself refreshed at the previous 256 steps, so blocks never wait
// for each other.  Weights (40 KB per layer) are double-buffered in LDS.
//
// Measured: 30 layers over 256 streams x 256 steps 254 us (8.5 us per layer; 24 us with a launch per layer),
// 7.0 us per layer when few blocks run.  What bounds it is the gate: 32 of tanhf, exp and a full division per
// lane and layer, two waves per SIMD, of which the products (1,280 cycles per layer and SIMD) hide behind
// little.  (With the hardware's exps and reciprocals alone it took 5.0 us, but lost bits of z, see gate.)  What
// helped: accesses without branches around them (see Rsrc), and the next layer's loads spread over the layer
// instead of issued right after the barrier (-8%).
//
// Wave w owns rows 32w .. 32w + 31.  Products are transposed, D[channel][row] = W[channel][k]
// X[row][k]: each lane's result is 4 consecutive channels of one row, so z and x go back to LDS as
// 8-byte pieces of operand rows and the residual 1x1 needs only the wave's own rows.  Per layer:
//   1. the layer input's newest rows into its queue; the next layer's weights and queue rows in flight
//   2. per pair p of 4: tanh tile p and sigmoid tile p over both taps (K = 128), gate, z into the
//      wave's rows of the next input buffer
//   3. residual 1x1 from those rows (added into the residual stream), z rows out to memory, the new
//      x over them
//   4. the next layer's weights into the other LDS buffer; one barrier
// The next layer's queue rows have landed in registers before that barrier, so any wave may refresh
// that queue after it.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fwg_internal.h"
#include "fwg_mfma_dev.h"
#include "fwg_par.h"

namespace fwg {
namespace pst {

using namespace mfd;

constexpr int R = 64, NW = 8, NT = 64 * NW, NR = kStackRows;
constexpr int PX = R + 8;           // LDS row stride of a layer input (bf16): rows spread over the banks
constexpr int NF = 40;              // weight fragments per layer: conv 8 tiles x 4 k-steps, residual 4 x 2
constexpr int NB = 3 * R;           // biases per layer: conv 2R, residual R
constexpr int LB = kStackLayerBytes;  // one layer's fragments and biases
static_assert(NF / NW == 5 && LB == NF * 1024 + NB * 4 && NF % NW == 0 && NR == 32 * NW, "layer block and row split");

struct Lds {
  uint16_t x[2][NR * PX];           // layer inputs, by running layer parity
  __attribute__((aligned(16))) unsigned char w[2][LB];  // weights and biases, by running layer parity
  // followed by the per-layer tables: queue offset in rows of R values (32 bits of them reach 512 GB) [L],
  // dilation [L], slot of the first row [L], slot of the first row that is kept [L]
};

// Queue rows and z rows go through raw buffer accesses whose offset is put past the end where a lane
// has nothing to move (such loads return 0 and such stores are dropped): a branch around them would
// make the compiler wait for every access in flight where the paths meet.
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ __forceinline__ Rsrc rsrc(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00020000);
}
constexpr uint32_t NOWHERE = 0xF0000000u;
__device__ __forceinline__ u32x4 load16(Rsrc r, uint32_t off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ void store16(Rsrc r, uint32_t off, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, 0);
}
// The loads behind v have landed: other waves may overwrite their source after the next barrier.
__device__ __forceinline__ void landed(const u32x4 &v) { asm volatile("" ::"v"(v)); }
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The per-layer kernel's gate, bit by bit: 1 - 2 / (exp(2a) + 1) loses the relative bits of small a.
__device__ __forceinline__ float gate(float a, float g) { return tanhf(a) * (1.f / (1.f + __expf(-g))); }

__global__ void __launch_bounds__(NT) stack_kernel(ParStack g) {
  extern __shared__ float4 lds_raw[];
  Lds &s = *(Lds *)lds_raw;
  const int L = g.L, tid = threadIdx.x, lane = tid & 63, n = lane & 15, q = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x;
  uint32_t *roff = (uint32_t *)((char *)lds_raw + sizeof(Lds));
  int *dil = (int *)(roff + L), *first = dil + L, *keep = first + L;
  for (int l = tid; l < L; l += NT) {
    roff[l] = (uint32_t)(g.layers[l].ring_off / R);
    dil[l] = g.layers[l].dil;
    first[l] = (int)(g.t0 % (long long)g.layers[l].dil);
  }
  const uint32_t slotb = (uint32_t)g.brows * (R * 2), rowb = (uint32_t)b * (R * 2);  // bytes
  auto queue = [&](int l) {
    const uint32_t off = __builtin_amdgcn_readfirstlane(roff[l]), d = __builtin_amdgcn_readfirstlane(dil[l]);
    return rsrc((const char *)g.ring + (size_t)off * (R * 2), d * slotb);
  };
  // the first layer's weights
  {
    const u32x4 *src = (const u32x4 *)g.packed;
    for (int i = tid; i < LB / 16; i += NT) ((u32x4 *)s.w[0])[i] = src[i];
  }
  __syncthreads();

  // queue rows of layer l for the wave's rows (n-tile t, k-step ks) at rows of this part: rows j < d
  u32x4 pop[2][2];
  auto pops = [&](int l, int rows) {
    const int d = __builtin_amdgcn_readfirstlane(dil[l]), f = first[l];
    if (32 * w >= d) return;  // every tap of the wave's rows lies in the part (the registers go unread)
    const Rsrc r = queue(l);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int j = 32 * w + 16 * t + n;
      int slot = f + j;
      slot = slot >= d ? slot - d : slot;
      const uint32_t off = j < d && j < rows ? (uint32_t)slot * slotb + rowb + 16 * q : NOWHERE;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) pop[t][ks] = load16(r, off + 64 * ks);
    }
  };
  auto pops_landed = [&]() {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) landed(pop[t][ks]);
  };

  int par = 0;  // running layer parity
  for (int j0 = 0; j0 < g.Tcur; j0 += g.part) {
    const int rows = min(g.part, g.Tcur - j0);
    // slots of this part's first kept row: the newest min(d, rows) rows go into the queue
    for (int l = tid; l < L; l += NT) {
      const int skip = rows > dil[l] ? rows - dil[l] : 0;
      keep[l] = (first[l] + skip) % dil[l];
    }
    if (j0 == 0) pops(0, rows);
    // x^0: embedding rows plus bias, fp32 in the accumulator layout and bf16 in LDS
    f32x4 xr[4][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int j = 32 * w + 16 * t + n;
      const long long st = g.s0 + j0 + j;
      int tok = 0;
      if (j < rows) {
        if (g.mode == MODE_TEACHER) tok = g.inputs[(long long)b * g.n_steps + st];
        else tok = st == 0 ? g.last[b] : g.inputs[(long long)b * g.n_steps + st - 1];
      }
      const uint16_t *e = (const uint16_t *)g.embed + (long long)tok * R;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int ch = 16 * c + 4 * q;
        const u32x2 raw = *(const u32x2 *)(e + ch);
        const float4 eb = *(const float4 *)(g.embed_b + ch);
        xr[c][t] = f32x4{bf_lo(raw.x) + eb.x, bf_hi(raw.x) + eb.y, bf_lo(raw.y) + eb.z, bf_hi(raw.y) + eb.w};
        lds8(s.x[par] + j * PX + ch, pack4(xr[c][t]));
      }
    }
    pops_landed();
    __syncthreads();

    for (int l = 0; l < L; ++l) {
      const uint16_t *xc = s.x[par];
      uint16_t *xn = s.x[par ^ 1];
      const unsigned char *wl = s.w[par];
      const float *bias = (const float *)(wl + NF * 1024);
      const int d = dil[l];
      // ---- 2a. operands: current rows, and the rows d steps back from LDS or the queue
      u32x4 xb[2][4];  // [n-tile][k-step]: recurrent tap 0,1, current tap 2,3
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int j = 32 * w + 16 * t + n;
        const bool in = j >= d;
        const uint16_t *xo = xc + (in ? j - d : 0) * PX + 8 * q, *xk = xc + j * PX + 8 * q;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const u32x4 v = lds16(xo + 32 * ks);
#pragma unroll
          for (int i = 0; i < 4; ++i) xb[t][ks][i] = in ? v[i] : pop[t][ks][i];
          xb[t][2 + ks] = lds16(xk + 32 * ks);
        }
      }
      // ---- 1. moved between the products below: next layer's weights and queue rows in flight, this
      // layer's queue refreshed (all issued at once they held every wave for ~1,600 cycles)
      const int ln = l + 1 < L ? l + 1 : 0;
      const u32x4 *wsrc = (const u32x4 *)((const char *)g.packed + (size_t)ln * LB);
      u32x4 wr[NF / NW], br;
      auto refresh = [&]() {
        const int lo = rows > d ? rows - d : 0, kb = keep[l];
        if (32 * w + 32 <= __builtin_amdgcn_readfirstlane(lo)) return;
        const Rsrc r = queue(l);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int j = 32 * w + 8 * i + (lane >> 3);
          int slot = kb + (j - lo);
          slot = slot >= d ? slot - d : slot;
          const uint32_t off = j >= lo && j < rows ? (uint32_t)slot * slotb + rowb + 16 * (lane & 7) : NOWHERE;
          store16(r, off, lds16(xc + j * PX + 8 * (lane & 7)));
        }
      };
      // ---- 2b. dilated product and gate, one pair of tiles at a time: the products of pair p + 1 are
      // issued before the gate of pair p, and the fragments of pair p + 2 read.  Sums start from zero and the
      // biases join the finished sums, as in the per-layer kernel (the same bits, and the smaller error).
      u32x4 wf[2][8];
      f32x4 at[2][2], ag[2][2];
      auto frags = [&](int p) {
#pragma unroll
        for (int f = 0; f < 8; ++f) wf[p & 1][f] = *(const u32x4 *)(wl + ((p * 8 + f) * 64 + lane) * 16);
      };
      auto product = [&](int p) {
#pragma unroll
        for (int t = 0; t < 2; ++t) at[p & 1][t] = ag[p & 1][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            at[p & 1][t] = mfma(wf[p & 1][2 * ks], xb[t][ks], at[p & 1][t]);
            ag[p & 1][t] = mfma(wf[p & 1][2 * ks + 1], xb[t][ks], ag[p & 1][t]);
          }
      };
      frags(0);
      frags(1);
      product(0);
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        __builtin_amdgcn_sched_barrier(0);
        if (p == 0) {
          if (l + 1 < L) pops(l + 1, rows);
          wr[0] = wsrc[tid];
          wr[1] = wsrc[NT + tid];
        }
        if (p == 1) {
          wr[2] = wsrc[2 * NT + tid];
          wr[3] = wsrc[3 * NT + tid];
          refresh();
        }
        if (p == 2) {
          wr[4] = wsrc[4 * NT + tid];
          br = wsrc[NF * 64 + min(tid, NB / 4 - 1)];
        }
        if (p < 3) product(p + 1);
        if (p < 3) frags(p + 2);  // p = 2: the residual fragments
        const f32x4 bt = ldsf4(bias + 16 * p + 4 * q), bg = ldsf4(bias + R + 16 * p + 4 * q);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          f32x4 z;
#pragma unroll
          for (int i = 0; i < 4; ++i) z[i] = gate(at[p & 1][t][i] + bt[i], ag[p & 1][t][i] + bg[i]);
          lds8(xn + (32 * w + 16 * t + n) * PX + 16 * p + 4 * q, pack4(z));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      wave_order();
      // ---- 3. residual 1x1, z rows out
      u32x4 zb[2][2], zo[4];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) zb[t][ks] = lds16(xn + (32 * w + 16 * t + n) * PX + 32 * ks + 8 * q);
#pragma unroll
      for (int i = 0; i < 4; ++i) zo[i] = lds16(xn + (32 * w + 8 * i + (lane >> 3)) * PX + 8 * (lane & 7));
      wave_order();
      {  // (the last layer's residual output feeds nothing)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const f32x4 rb = ldsf4(bias + 2 * R + 16 * c + 4 * q);
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            f32x4 r = mfma(wf[0][2 * c], zb[t][0], f32x4{0.f, 0.f, 0.f, 0.f});
            r = mfma(wf[0][2 * c + 1], zb[t][1], r);
            xr[c][t] += r + rb;
          }
#pragma unroll
          for (int t = 0; t < 2; ++t)
            lds8(xn + (32 * w + 16 * t + n) * PX + 16 * c + 4 * q, pack4(xr[c][t]));
        }
      }
      {
        const uint32_t zrow = (uint32_t)g.ldz * 2;
        const Rsrc r = rsrc((uint16_t *)g.zout + ((long long)b * g.Tcur + j0) * g.ldz, (uint32_t)rows * zrow);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int j = 32 * w + 8 * i + (lane >> 3);
          store16(r, j < rows && g.zout ? (uint32_t)j * zrow + (uint32_t)(l * R * 2) + 16 * (lane & 7) : NOWHERE, zo[i]);
        }
      }
      // ---- 4. next layer's weights into the other buffer (its last readers passed the last barrier)
      {
        u32x4 *dst = (u32x4 *)s.w[par ^ 1];
#pragma unroll
        for (int i = 0; i < NF / NW; ++i) dst[i * NT + tid] = wr[i];
        if (tid < NB / 4) dst[NF * 64 + tid] = br;
      }
      pops_landed();
      __syncthreads();
      par ^= 1;
    }
    // the next part's times: its first rows' slots, then layer 0's queue rows
    if (j0 + g.part < g.Tcur) {
      for (int l = tid; l < L; l += NT) first[l] = (first[l] + rows) % dil[l];
      __syncthreads();
      pops(0, min(g.part, g.Tcur - j0 - g.part));
    }
  }
}

// One layer's block: conv fragment (pair p, k-step ks, half h: tanh, sigmoid) at (p * 4 + ks) * 2 + h,
// residual fragment (tile c, k-step ks) at 32 + 2 c + ks; fragment (tile, k-step) of M[out][k] gives
// lane i the 8 values M[16 tile + i % 16][32 ks + 8 (i / 16) + j]; then the biases.
__global__ void pack_kernel(const uint16_t *conv, const uint16_t *res, const float *conv_b, const float *res_b, uint4 *dst) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < NB) ((float *)dst)[NF * 256 + e] = e < 2 * R ? (conv_b ? conv_b[e] : 0.f) : (res_b ? res_b[e - 2 * R] : 0.f);
  if (e >= NF * 64) return;
  const int i = e % 64, f = e / 64, m = i % 16, kq = 8 * (i / 16);
  uint16_t v[8];
  for (int j = 0; j < 8; ++j) {
    if (f < 32) {
      const int p = f / 8, ks = (f / 2) % 4, o = (f & 1) * R + 16 * p + m, k = 32 * ks + kq + j;
      v[j] = conv[(o * R + (k % R)) * 2 + k / R];
    } else {
      const int c = (f - 32) / 2, ks = f & 1;
      v[j] = res[(16 * c + m) * R + 32 * ks + kq + j];
    }
  }
  dst[e] = make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
}

}  // namespace pst

static size_t stack_lds_bytes(int L) { return sizeof(pst::Lds) + 16 * (size_t)L; }

bool par_stack_ok(int kind, int dtype, int C, int w, int L) {
  return kind == 2 && dtype == 1 && C == pst::R && w == 2 && L >= 2 && stack_lds_bytes(L) <= 160 * 1024;
}

hipError_t set_par_stack_lds_limit(int L) {
  return hipFuncSetAttribute((const void *)pst::stack_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)stack_lds_bytes(L));
}

hipError_t launch_par_stack(const ParStack &g, int batch, hipStream_t s) {
  hipLaunchKernelGGL(pst::stack_kernel, dim3(batch), dim3(pst::NT), stack_lds_bytes(g.L), s, g);
  return hipGetLastError();
}

hipError_t launch_par_stack_pack(const void *conv, const void *res, const float *conv_b, const float *res_b, void *dst,
                                 hipStream_t s) {
  hipLaunchKernelGGL(pst::pack_kernel, dim3((pst::NF * 64 + 255) / 256), dim3(256), 0, s, (const uint16_t *)conv,
                     (const uint16_t *)res, conv_b, res_b, (uint4 *)dst);
  return hipGetLastError();
}

}  // namespace fwg
