// HIP kernels of the Fast Wavenet generation library, written for gfx950.
//
// This file holds the general ("VALU") step kernel and the small utility kernels (weight repacking,
// fills).  One launch runs n_steps whole generation steps, one block per stream: every step pops
// each layer's queue, runs the generation model (one step of a multi-layer RNN, paper Section 2.2,
// Fig. 4), pushes the new states, computes the output distribution and samples the next input (fed
// back, Section 1).
//
// Layout decisions:
//   * queues: one ring buffer per layer, ring_l[slot][stream][channel] with the
//     channel index contiguous, slot = t mod d_l (Section 2.1: depth = dilation);
//     popping reads the slot written d_l steps earlier, pushing overwrites it
//     after every lane has read it (pop before push, Section 2.2);
//   * weights: streamed from L2 in a 16-byte K-blocked layout, so consecutive
//     lanes read consecutive 16-byte chunks;
//   * activations of the block's stream: LDS, float32.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fwg_bf16.h"
#include "fwg_internal.h"
#include "fwg_valu.h"
#include "fwg_sample.h"


namespace fwg {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <typename WT> struct WTraits;
template <> struct WTraits<float> {
  static constexpr int KB = 4;
  __device__ static __forceinline__ void unpack(u32x4 v, float *w) {
    w[0] = __uint_as_float(v.x); w[1] = __uint_as_float(v.y);
    w[2] = __uint_as_float(v.z); w[3] = __uint_as_float(v.w);
  }
  __device__ static __forceinline__ float load1(const void *p, long long i) { return ((const float *)p)[i]; }
  __device__ static __forceinline__ void store1(void *p, long long i, float v) { ((float *)p)[i] = v; }
  __device__ static __forceinline__ float opnd(float x) { return x; }
};
template <> struct WTraits<uint16_t> {
  static constexpr int KB = 8;
  __device__ static __forceinline__ void unpack(u32x4 v, float *w) {
    w[0] = bf16_lo(v.x); w[1] = bf16_hi(v.x); w[2] = bf16_lo(v.y); w[3] = bf16_hi(v.y);
    w[4] = bf16_lo(v.z); w[5] = bf16_hi(v.z); w[6] = bf16_lo(v.w); w[7] = bf16_hi(v.w);
  }
  __device__ static __forceinline__ float load1(const void *p, long long i) {
    return __uint_as_float(((uint32_t)((const uint16_t *)p)[i]) << 16);
  }
  __device__ static __forceinline__ void store1(void *p, long long i, float v) { ((uint16_t *)p)[i] = bf16_bits(v); }
  __device__ static __forceinline__ float opnd(float x) { return round_bf16(x); }
};

// ---------------------------------------------------------------------------
// Products of one stream: part[kg][n] = sum over K-group kg of W^T[k][n] A[k] (+ bias[n] in group 0), A in
// LDS.  With NT threads:
// N >= NT: each thread owns columns tid, tid + NT, ... over all of K (one group); N < NT (N divides NT):
// NT / N K-groups of N threads each.
// A thread's weights are chunks of U 16-byte pieces (consecutive k-blocks of a column); the first chunk and the bias are
// loaded by `head` before the barrier that makes A ready (weights depend on no activation), every later
// chunk while the one before is multiplied.  Weights come through raw buffer
// loads: one VGPR offset per thread and product, kept for the launch, and a scalar offset per piece
// (with 64-bit addresses the index arithmetic of runtime shapes cost more than the products).
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ __forceinline__ Rsrc rsrc(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00020000);
}
// A uniform value that the compiler takes as new here: what follows from it is computed where it is used
// (hoisted out of the layer loop, the scalar offsets of every piece overflowed the scalar registers).
__device__ __forceinline__ int fresh(int v) {
  v = __builtin_amdgcn_readfirstlane(v);
  asm volatile("" : "+s"(v));
  return v;
}
template <typename T> __device__ __forceinline__ T *uniform_ptr(T *p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (T *)(((uint64_t)hi << 32) | lo);
}

template <typename WT, int NT, int U_>
struct Product {
  static constexpr int KB = WTraits<WT>::KB, U = U_;
  // the thread's share: first piece and first column, first k, K-group; k-blocks per column
  int piece, n, k0, kg, per, N;
  __device__ __forceinline__ void init(int K, int N_) {
    const int nkb = K / KB, tid = threadIdx.x;
    N = N_;
    if (N >= NT) {
      n = tid;
      kg = 0;
      per = nkb;
    } else {
      const int sh = __builtin_ctz(N);
      n = tid & (N - 1);
      kg = tid >> sh;
      per = nkb >> (__builtin_ctz(NT) - sh);
    }
    k0 = kg * per * KB;
    piece = kg * per * N + n;
  }
  // byte offset of the thread's first piece in its c-th column (threads past the last column repeat it)
  __device__ __forceinline__ uint32_t at(int c) const {
    return (uint32_t)(piece + min(NT * c, N - 1 - n)) * 16u;
  }
};

// One product in flight: a ring of U pieces, refilled four at a time as they are multiplied.
template <typename WT, int NT, int U>
struct Flight {
  static constexpr int KB = WTraits<WT>::KB;
  u32x4 w[U];
  float bias;
  __device__ __forceinline__ void load4(int N, int per, Rsrc r, uint32_t base, uint32_t voff, int kb, int g) {
#pragma unroll
    for (int u = g; u < g + 4; ++u)  // past the end: the last piece again, not multiplied
      w[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                           r, voff, base + (uint32_t)(min(kb + u, per - 1) * N) * 16u, 0));
  }
  __device__ __forceinline__ void load_bias(const Product<WT, NT, U> &p, Rsrc rb, uint32_t bias_at, int c) {
    bias = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, 4 * min(p.n + NT * c, p.N - 1), bias_at, 0));
  }
  // base: byte offset of the product's weights in r; bias_at: byte offset of its biases in rb
  __device__ __forceinline__ void head(const Product<WT, NT, U> &p, Rsrc r, uint32_t base, Rsrc rb, uint32_t bias_at) {
    load_bias(p, rb, bias_at, 0);
    const uint32_t voff = p.at(0);
    const int N = fresh(p.N), per = fresh(p.per);
#pragma unroll
    for (int g = 0; g < U; g += 4)
      if (g < per) load4(N, per, r, base, voff, 0, g);
  }
  // R streams: operand rows `lda` apart, partial sums valu_part_cols(N, NT) apart
  template <int R = 1>
  __device__ __forceinline__ void run(const Product<WT, NT, U> &p, Rsrc r, uint32_t base, Rsrc rb, uint32_t bias_at,
                                      const float *A, float *part, int lda = 0) {
    const int N = fresh(p.N), per = fresh(p.per), cols = (N + NT - 1) / NT;
    A += p.k0;
    float *out = part + p.kg * p.N + p.n;
    for (int c = 0; c < cols; ++c) {
      const float b = p.kg == 0 ? bias : 0.f;
      float acc[R];  // the bias joins the finished sum
#pragma unroll
      for (int i = 0; i < R; ++i) acc[i] = 0.f;
      if (c + 1 < cols) load_bias(p, rb, bias_at, c + 1);
      for (int kb = 0; kb < per; kb += U) {
        // the chunk after this one: of this column, or the first of the next
        const bool here = kb + U < per, next = here || c + 1 < cols;
        const int nkb = here ? kb + U : 0;
        const uint32_t nvoff = p.at(here ? c : c + 1);
        const float *x = A + kb * KB;
        constexpr int XU = R == 1 ? U : 4;  // pieces whose operands are held at a time
        float4 xv[R][XU * KB / 4];
        auto operands = [&](int g) {  // past the end: not multiplied
#pragma unroll
          for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < XU * KB / 4; ++j) xv[i][j] = *(const float4 *)(x + i * lda + g * KB + 4 * j);
        };
        if (R == 1) operands(0);
        auto piece = [&](int u) {
          float wv[KB];
          WTraits<WT>::unpack(w[u], wv);
#pragma unroll
          for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < KB; j += 4) {
              const float4 xx = xv[i][(u % XU * KB + j) / 4];
              acc[i] = fmaf(wv[j], xx.x, acc[i]);
              acc[i] = fmaf(wv[j + 1], xx.y, acc[i]);
              acc[i] = fmaf(wv[j + 2], xx.z, acc[i]);
              acc[i] = fmaf(wv[j + 3], xx.w, acc[i]);
            }
        };
        const int left = per - kb;
#pragma unroll
        for (int g = 0; g < U; g += 4) {
          if (R > 1) operands(g);
          if (left >= g + 4) {
#pragma unroll
            for (int u = g; u < g + 4; ++u) piece(u);
          } else {
#pragma unroll
            for (int u = g; u < g + 3; ++u)
              if (u < left) piece(u);
          }
          if (next && nkb + g < per) load4(N, per, r, base, nvoff, nkb, g);
        }
      }
      if (p.n + NT * c < p.N) {
#pragma unroll
        for (int i = 0; i < R; ++i) out[i * valu_part_cols(p.N, NT) + NT * c] = acc[i] + b;
      }
    }
  }
};

// Sum of the K-group partials of output n.
template <int NT>
__device__ __forceinline__ float part_sum(const float *part, int N, int n) {
  float s = part[n];
  if (N < NT)
    for (int i = n + N; i < NT; i += N) s += part[i];
  return s;
}

__device__ __forceinline__ float bias_or0(const float *b, int i) { return b ? b[i] : 0.f; }

// ---------------------------------------------------------------------------
// The general step kernel: one block of NT threads per stream (ROWS = 2: per two streams).
//
// What bounds it is the compute unit's load path: a step streams every weight from the L2 at up to 64
// bytes per cycle (a layer of R = 64, S = 256 float32 channels, 147 KB, ~1 us).  So a stream gets a
// compute unit of its own for as long as there are any: with up to 8 streams on a block, to share its
// weights, most of the chip was idle (16 streams of that 20-layer model: 562 us per step on 2 blocks,
// 74 now; 512 streams 568 and 96).  Blocks of 256 threads share a compute unit from 257 streams on.
// At ~3.5 us per layer the chain of barriers, LDS reads and partial sums is still what bounds it.
// MANY: past two streams per compute unit throughput counts, so half the registers (and pieces in flight) let
// four blocks share one.  ROWS = 2 (ReLU stacks of large layers, with MANY): there the weight stream itself is the
// bound, and two streams of a block share it.  2,048 streams, us per step, with 8 streams on a block / one
// stream, two blocks per compute unit / now: gated R = 32, S = 64 float32, 10 layers 86 / 138 / 75; ReLU C = 512
// float32, 6 layers 814 / 1,060 / 718; ReLU C = 1024 bf16, 3 layers 830 / 1,438 / 841.
// Latency hiding: the states a layer pops do not depend on the current step (they were pushed
// at least d steps earlier), so the pops of layer l + 1 -- or of layer 0 of the next step -- are
// loaded into registers while layer l computes and land in the second of two LDS buffers at the
// end of the layer; each product's first weights are in registers before its operands are ready.
// GATED and W2 (filter width 2) are compile-time: fewer shape values stay live.
template <typename WT, int NT, bool GATED, bool W2, bool MANY, int ROWS>
__global__ void __launch_bounds__(NT, MANY && ROWS == 1 ? 4 : 2) valu_step_kernel(StepArgs a) {
  static_assert(ROWS == 1 || !GATED, "several streams per block: ReLU stacks");
  constexpr int U = MANY && ROWS == 1 ? 4 : 8;  // pieces in flight per product
  extern __shared__ float4 lds_raw[];
  float *lds = (float *)lds_raw;
  const int kind = GATED ? 2 : a.kind, C = a.C, S = a.S, H = a.H, Q = 256, w = W2 ? 2 : a.w, L = a.L;
  const ValuLds lay = valu_lds_layout(kind, C, S, H, Q, L, w, NT, ROWS);
  // the two buffers of operand rows (the w - 1 popped states, oldest first, then the current input)
  auto vbuf = [&](int p) { return lds + (p ? lay.vx2 : lay.vx); };
  float *xf = lds + lay.xf, *zo = lds + lay.zo, *so = lds + lay.so, *h2 = lds + lay.h2;
  float *lg = lds + lay.lg, *partA = lds + lay.partA, *partB = lds + lay.partB;
  int *slots = (int *)(lds + lay.slots);
  int *ins = (int *)(lds + lay.ins);
  ValuLayer *ltab = (ValuLayer *)(lds + lay.ltab);

  const int tid = threadIdx.x, b = blockIdx.x * ROWS;  // the block's first stream
  const int nrows = ROWS == 1 ? 1 : min(ROWS, a.batch - b);
  const int Co = GATED ? 2 * C : C;
  const int K = w * C, XO = (w - 1) * C;  // row length of the operands; where the current input starts
  const uint32_t es = sizeof(WT);
  // offsets inside a layer's block: conv | res | skip weights, then conv_b | res_b | skip_b
  const uint32_t o_res = (uint32_t)K * Co * es, o_skip = o_res + (uint32_t)C * C * es;
  const uint32_t o_cb = GATED ? o_skip + (uint32_t)S * C * es : o_res;
  const uint32_t o_rb = o_cb + (uint32_t)Co * 4, o_sb = o_rb + (uint32_t)C * 4, o_end = GATED ? o_sb + S * 4 : o_rb;

  for (int l = tid; l < L; l += NT) {
    const LayerDev ld = a.layers[l];
    ValuLayer v;
    v.block = ld.conv;
    v.ring_off = ld.ring_off;
    v.dil = ld.dil;
    v.depth = ld.depth;
    v.pad_[0] = v.pad_[1] = 0;
    ltab[l] = v;
    slots[l] = (int)(a.t0 % (long long)ld.depth);
  }
  // the thread that handles a stream's input: thread r for stream r
  const bool owner = ROWS == 1 ? tid == 0 : tid < nrows;
  const int own = ROWS == 1 ? 0 : tid;
  if (owner) ins[own] = a.mode == MODE_TEACHER ? a.inputs[(long long)(b + own) * a.n_steps] : a.last[b + own];
  __syncthreads();

  // prefetch registers of the next layer's popped states: element i of a stream is tap i / C, channel i % C
  // (streams past the last one repeat it)
  float pp[kValuPrefPops];
  auto fetch = [&](int l, int slot_) {
    const ValuLayer ld = ltab[l];
    const int slot = fresh(slot_), depth = fresh(ld.depth), dil = fresh(ld.dil);
    const char *row = uniform_ptr((const char *)a.ring + (ld.ring_off + (long long)b * C) * es);
    const long long slot_bytes = (long long)fresh(a.bmax) * C * es;
#pragma unroll
    for (int j = 0; j < kValuPrefPops; ++j) {
      if (j * NT >= ROWS * XO) break;
      const int e = tid + j * NT, r = ROWS == 1 ? 0 : e / XO, i = e - r * XO;
      float v = 0.f;
      if (e < ROWS * XO) {
        int k = 0, c = i;
        if (!W2) {
          k = i / C;
          c = i - k * C;
        }
        int sk = slot + (W2 ? 0 : k * dil);  // k dilations after the oldest state
        if (!W2 && sk >= depth) sk -= depth;
        v = WTraits<WT>::load1(row + sk * slot_bytes, min(r, nrows - 1) * C + c);
      }
      pp[j] = v;
    }
  };
  auto land = [&](int par) {
    float *vb = vbuf(par);
#pragma unroll
    for (int j = 0; j < kValuPrefPops; ++j) {
      if (j * NT >= ROWS * XO) break;
      const int e = tid + j * NT;
      if (e < ROWS * XO) vb[ROWS == 1 ? e : e / XO * K + e % XO] = pp[j];
    }
  };
  auto layer_rsrc = [&](int l) { return rsrc(uniform_ptr((const char *)ltab[l].block), o_end); };

  Product<WT, NT, U> pconv, pres, pskip, phead, pout;
  const int Ktop = GATED ? H : C;
  pconv.init(K, Co);
  pout.init(Ktop, Q);
  if constexpr (GATED) {
    pres.init(C, C);
    pskip.init(C, S);
    phead.init(S, H);
  }
  Flight<WT, NT, U> conv;

  fetch(0, slots[0]);
  land(0);
  Rsrc rl = layer_rsrc(0);
  conv.head(pconv, rl, 0, rl, o_cb);
  int par = 0;  // buffer holding the current layer's operands

  for (int s = 0; s < a.n_steps; ++s) {
    // ---- current input (h^0_e): a row gather of the transposed 1x1 convolution
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      const int tok = ins[min(r, nrows - 1)];
      for (int c = tid; c < C; c += NT) {
        const float v = WTraits<WT>::load1(a.embed, (long long)tok * C + c) + bias_or0(a.embed_b, c);
        xf[r * C + c] = v;
        vbuf(par)[r * K + XO + c] = WTraits<WT>::opnd(v);
      }
    }
    if constexpr (GATED)
      for (int i = tid; i < S; i += NT) so[i] = 0.f;
    __syncthreads();

    for (int l = 0; l < L; ++l) {
      const ValuLayer ld = ltab[l];
      // the layer that runs next: layer l + 1 now, or layer 0 at the next step (its slot one on)
      const bool more = l + 1 < L || s + 1 < a.n_steps;
      const int nl = l + 1 < L ? l + 1 : 0;
      int nslot = slots[nl];
      if (l + 1 == L) nslot = nslot + 1 == ltab[0].depth ? 0 : nslot + 1;
      const float *vo = vbuf(par);
      float *xn = vbuf(par ^ 1) + XO;  // the layer's output: the current input of the next one
      // with one layer, the next step's pops include the state this layer pushes now: fetch after it
      if (more && L > 1) fetch(nl, nslot);
      // ---- push phase for this queue: the layer's input x^{l-1}_t replaces the oldest state,
      // whose pop has landed in LDS already
      char *qrow = uniform_ptr((char *)a.ring + (ld.ring_off + ((long long)slots[l] * a.bmax + b) * C) * es);
#pragma unroll
      for (int r = 0; r < ROWS; ++r)
        if (r < nrows)
          for (int c = tid; c < C; c += NT) WTraits<WT>::store1(qrow, r * C + c, vo[r * K + XO + c]);
      if (more && L == 1) {
        __syncthreads();
        fetch(nl, nslot);
      }
      // ---- dilated convolution of width w: [v_0 .. v_{w-2} x] . [W_0 ; .. ; W_{w-1}]
      conv.template run<ROWS>(pconv, rl, 0, rl, o_cb, vo, partA, K);
      if constexpr (GATED) {
        Flight<WT, NT, U> res, skip;
        res.head(pres, rl, o_res, rl, o_rb);
        skip.head(pskip, rl, o_skip, rl, o_sb);
        __syncthreads();
        // gate: z = tanh(a[0:R]) * sigmoid(a[R:2R])
        for (int c = tid; c < C; c += NT) {
          const float af = part_sum<NT>(partA, Co, c), ag = part_sum<NT>(partA, Co, C + c);
          // tanh(a) = 1 - 2 / (e^{2a} + 1) and sigmoid(g) = 1 / (1 + e^{-g}), one exp and one
          // reciprocal each (absolute error ~1e-7, saturating correctly at both ends)
          const float z = (1.f - 2.f * __builtin_amdgcn_rcpf(__expf(2.f * af) + 1.f)) *
                          __builtin_amdgcn_rcpf(1.f + __expf(-ag));
          zo[c] = WTraits<WT>::opnd(z);
        }
        __syncthreads();
        // residual and skip 1x1 products
        res.run(pres, rl, o_res, rl, o_rb, zo, partB);
        skip.run(pskip, rl, o_skip, rl, o_sb, zo, partA);
        if (more) {
          rl = layer_rsrc(nl);
          conv.head(pconv, rl, 0, rl, o_cb);
        }
        __syncthreads();
        for (int c = tid; c < C; c += NT) {
          const float v = xf[c] + part_sum<NT>(partB, C, c);
          xf[c] = v;
          xn[c] = WTraits<WT>::opnd(v);
        }
        for (int k = tid; k < S; k += NT) so[k] += part_sum<NT>(partA, S, k);
      } else {
        if (more) {
          rl = layer_rsrc(nl);
          conv.head(pconv, rl, 0, rl, o_cb);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
          for (int c = tid; c < C; c += NT) {
            const float pre = part_sum<NT>(partA + r * valu_part_cols(Co, NT), Co, c);
            const float v = (kind == 1 ? xf[r * C + c] : 0.f) + fmaxf(pre, 0.f);
            xf[r * C + c] = v;
            xn[r * K + c] = WTraits<WT>::opnd(v);
          }
      }
      if (more) land(par ^ 1);
      __syncthreads();
      par ^= 1;
    }

    // ---- output head (the top layer's output sits where layer 0's next input will)
    Flight<WT, NT, U> top;
    const float *x = vbuf(par) + XO;
    const Rsrc ro = rsrc(a.out, (uint32_t)Ktop * Q * es), rob = rsrc(a.out_b, Q * 4);
    if constexpr (GATED) {
      const Rsrc rh = rsrc(a.head, (uint32_t)S * H * es), rhb = rsrc(a.head_b, H * 4);
      top.head(phead, rh, 0, rhb, 0);
      for (int i = tid; i < S; i += NT) so[i] = WTraits<WT>::opnd(fmaxf(so[i], 0.f));
      __syncthreads();
      top.run(phead, rh, 0, rhb, 0, so, partA);
      top.head(pout, ro, 0, rob, 0);
      __syncthreads();
      for (int n = tid; n < H; n += NT) h2[n] = WTraits<WT>::opnd(fmaxf(part_sum<NT>(partA, H, n), 0.f));
      __syncthreads();
      x = h2;
    } else {
      top.head(pout, ro, 0, rob, 0);
    }
    top.template run<ROWS>(pout, ro, 0, rob, 0, x, partA, K);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
      if (tid < Q) lg[r * Q + tid] = part_sum<NT>(partA + r * valu_part_cols(Q, NT), Q, tid);
    __syncthreads();

    if (a.mode != MODE_GENERATE) {
#pragma unroll
      for (int r = 0; r < ROWS; ++r)
        if (a.logits && r < nrows && tid < Q) a.logits[((long long)(b + r) * a.n_steps + s) * Q + tid] = lg[r * Q + tid];
      // the next input: the following element of the forced sequence (teacher forcing), or this
      // step's observed sample (online prediction)
      const int nx = s + forced_shift(a.mode);
      if (owner && nx < a.n_steps) ins[own] = a.inputs[(long long)(b + own) * a.n_steps + nx];
    } else if (tid < 64 * nrows) {
      // ---- sample and feed back: one wavefront per stream
      const int r = ROWS == 1 ? 0 : tid / 64;
      const float u = a.uniforms[(long long)(b + r) * a.n_steps + s];
      const int k = sample_row_256(lg + r * Q, u);
      if (ROWS == 1 ? tid == 0 : tid == 64 * r) {
        a.samples[(long long)(b + r) * a.n_steps + s] = k;
        ins[r] = k;
      }
    }
    // ---- advance every queue's slot
    for (int l = tid; l < L; l += NT) {
      const int nx = slots[l] + 1;
      slots[l] = nx == ltab[l].depth ? 0 : nx;
    }
    __syncthreads();
  }
  if (a.mode != MODE_TEACHER && owner) a.last[b + own] = ins[own];
}

typedef void (*ValuKernel)(StepArgs);
template <typename WT, int NT, bool MANY>
static ValuKernel valu_kernel_of(int kind, int w) {
  if (kind == 2) return w == 2 ? valu_step_kernel<WT, NT, true, true, MANY, 1> : valu_step_kernel<WT, NT, true, false, MANY, 1>;
  return w == 2 ? valu_step_kernel<WT, NT, false, true, MANY, 1> : valu_step_kernel<WT, NT, false, false, MANY, 1>;
}
template <typename WT>
static ValuKernel valu_kernel_of(const ValuVariant &v, int kind, int w) {
  if (v.rows == 2) return w == 2 ? valu_step_kernel<WT, 256, false, true, true, 2> : valu_step_kernel<WT, 256, false, false, true, 2>;
  if (v.many) return valu_kernel_of<WT, 256, true>(kind, w);
  return v.threads == 512 ? valu_kernel_of<WT, 512, false>(kind, w) : valu_kernel_of<WT, 256, false>(kind, w);
}
static ValuKernel valu_kernel_of(const ValuVariant &v, int dtype, int kind, int w) {
  return dtype == 1 ? valu_kernel_of<uint16_t>(v, kind, w) : valu_kernel_of<float>(v, kind, w);
}

hipError_t launch_valu_step(const StepArgs &a, const ValuVariant &v, size_t lds, hipStream_t s) {
  hipLaunchKernelGGL(valu_kernel_of(v, a.dtype, a.kind, a.w), dim3((a.batch + v.rows - 1) / v.rows), dim3(v.threads), lds, s, a);
  return hipGetLastError();
}

hipError_t set_valu_lds_limit(const ValuVariant &v, int dtype, int kind, int w, size_t bytes) {
  return hipFuncSetAttribute((const void *)valu_kernel_of(v, dtype, kind, w), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

// ---------------------------------------------------------------------------
// Weight repacking (once, at create): dst in the VALU K-blocked layout
// Wp[kb][n][j] = W^T[kb*KB + j][n], or the embedding's row-gather table.
template <typename T>
__global__ void repack_kernel(const T *__restrict__ src, T *__restrict__ dst, int mode, int K, int N, int C, int KB) {
  const long long total = (long long)K * N;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
    if (mode == REPACK_EMBED) {
      // dst [Q][C] from src [C][Q]; here K = Q, N = C
      const long long q = i / N, c = i % N;
      dst[i] = src[c * K + q];
      continue;
    }
    const long long j = i % KB, rest = i / KB;
    const long long n = rest % N, kb = rest / N;
    const long long k = kb * KB + j;
    long long si;
    if (mode == REPACK_CONV) si = (n * C + (k % C)) * (K / C) + k / C;  // tap k / C of K / C
    else si = n * K + k;
    dst[i] = src[si];
  }
}

hipError_t launch_repack(const void *src, void *dst, int mode, int dtype, int K, int N, int C, hipStream_t s) {
  const long long total = (long long)K * N;
  const int blocks = (int)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
  if (dtype == 1)
    hipLaunchKernelGGL(repack_kernel<uint16_t>, dim3(blocks), dim3(256), 0, s, (const uint16_t *)src,
                       (uint16_t *)dst, mode, K, N, C, valu_kb_elems(1));
  else
    hipLaunchKernelGGL(repack_kernel<float>, dim3(blocks), dim3(256), 0, s, (const float *)src, (float *)dst,
                       mode, K, N, C, valu_kb_elems(0));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fills (used instead of memset nodes so the calls stay safe under stream capture).
// Zero `bytes` bytes at dst (16-byte aligned): whole 16-byte units, then the tail byte by byte.
__global__ void fill_zero_kernel(uint4 *dst, size_t bytes) {
  const size_t n16 = bytes / 16;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = make_uint4(0, 0, 0, 0);
  if (blockIdx.x == 0 && threadIdx.x < bytes % 16) ((unsigned char *)dst)[n16 * 16 + threadIdx.x] = 0;
}
__global__ void fill_i32_kernel(int32_t *dst, int32_t v, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) dst[i] = v;
}
__global__ void copy_bias_kernel(const float *src, float *dst, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) dst[i] = src ? src[i] : 0.f;
}

hipError_t launch_fill_zero(void *dst, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  const size_t n16 = bytes / 16;  // regions start 256-byte aligned
  const int blocks = (int)(n16 / 256 + 1 < 8192 ? n16 / 256 + 1 : 8192);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, s, (uint4 *)dst, bytes);
  return hipGetLastError();
}
hipError_t launch_fill_i32(int32_t *dst, int32_t v, int n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((n + 255) / 256), dim3(256), 0, s, dst, v, n);
  return hipGetLastError();
}
hipError_t launch_copy_bias(const float *src, float *dst, int n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(copy_bias_kernel, dim3((n + 255) / 256), dim3(256), 0, s, src, dst, n);
  return hipGetLastError();
}

}  // namespace fwg
