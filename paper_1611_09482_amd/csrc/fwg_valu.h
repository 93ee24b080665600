// General step-kernel family (fwg_kernels.hip): packed-weight layout, layer table and LDS layout.
#pragma once

#include "fwg_internal.h"

namespace fwg {

// Packed-weight layout of the VALU family: W^T blocked by 16 bytes along K,
// Wp[kb][n][kb_elems], with W^T[k][n] the weight from input k to output n.
inline int valu_kb_elems(int dtype) { return dtype == 1 ? 8 : 4; }

// The layer fields the general step kernel reads in its loop, copied to LDS at launch.
struct ValuLayer {
  const void *block;    // the layer's weight + bias block
  long long ring_off;   // element offset of the layer's queue
  int dil, depth;
  int pad_[2];
};
static_assert(sizeof(ValuLayer) == 32, "eight floats per layer in the LDS table");

// LDS layout (in floats) of the VALU step kernel: two buffers of layer operand rows (the w - 1 popped
// states, oldest first, then the current input).
struct ValuLds {
  int xf, vx, vx2, zo, so, h2, lg, partA, partB, ltab, slots, ins, total_floats;
};
constexpr int kValuPrefPops = 8;   // popped elements per thread and layer held in registers
__host__ __device__ inline int valu_part_cols(int N, int threads) { return N >= threads ? N : threads; }
__host__ __device__ inline ValuLds valu_lds_layout(int kind, int C, int S, int H, int Q, int L, int w,
                                                   int threads, int rows) {
  ValuLds o;
  int p = 0;
  auto take = [&](int n) { int at = p; p += (n + 3) & ~3; return at; };
  const int Co = kind == 2 ? 2 * C : C;
  o.xf = take(rows * C);
  o.vx = take(rows * w * C);
  o.vx2 = take(rows * w * C);
  o.zo = take(kind == 2 ? C : 0);
  o.so = take(kind == 2 ? S : 0);
  o.h2 = take(kind == 2 ? H : 0);
  o.lg = take(rows * Q);
  int partN = valu_part_cols(Co, threads);
  if (kind == 2) {
    partN = partN > valu_part_cols(S, threads) ? partN : valu_part_cols(S, threads);
    partN = partN > valu_part_cols(H, threads) ? partN : valu_part_cols(H, threads);
  }
  o.partA = take(rows * partN);
  o.partB = take(kind == 2 ? valu_part_cols(C, threads) : 0);
  o.ltab = take(8 * L);  // per layer: weight block address, queue offset, dilation, depth (ValuLayer)
  o.slots = take(L);   // int
  o.ins = take(rows);  // int
  o.total_floats = p;
  return o;
}

// The general step kernel's variant: threads per block; whether up to four blocks share a compute unit (256
// threads, half the registers); streams per block (2: `many`, ReLU stacks).
struct ValuVariant {
  int threads;
  bool many;
  int rows;
};
hipError_t launch_valu_step(const StepArgs &a, const ValuVariant &v, size_t lds_bytes, hipStream_t s);
hipError_t set_valu_lds_limit(const ValuVariant &v, int dtype, int kind, int w, size_t bytes);

}  // namespace fwg
