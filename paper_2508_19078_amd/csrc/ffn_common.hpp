// What the grouped FFN's kernels share: a slot's rows, the layer's pointer
// tables, the tile order inside a slot, and the logistic function.
#pragma once

#include "common.hpp"

namespace fm {
namespace {

constexpr int N_XCD = 8;

struct SlotRows {
  int nrows;    // rows of the slot
  long orow0;   // first row of the slot in the per-row buffers
  long xrow0;   // first row of the slot's input in X_perm (routed) or X (shared)
  bool shared;
};

__device__ __forceinline__ SlotRows slot_rows(int s, const int32_t* offsets, int S_r, int Tn, int k) {
  SlotRows r;
  if (s < S_r) {
    const int b = ld_scalar(offsets + s);
    r.nrows = ld_scalar(offsets + s + 1) - b;
    r.orow0 = b;
    r.xrow0 = b;
    r.shared = false;
  } else {
    r.nrows = Tn;
    r.orow0 = (long)Tn * k + (long)(s - S_r) * Tn;
    r.xrow0 = 0;
    r.shared = true;
  }
  return r;
}

struct RowArgs {
  const int32_t* offsets;
  const int32_t* mbase;
  int S_r, S, Tn, k, d, I;
  int ldA;   // row stride (elements) of the backward's dA_g, dA_u in the workspace
};

template <typename T> struct LayerPtrs {
  const T* const* wg;
  const T* const* wu;
  const T* const* wd;
  float* const* dwg;
  float* const* dwu;
  float* const* dwd;
};

template <typename T> LayerPtrs<T> layer_ptrs(const moe_layer* L) {
  return LayerPtrs<T>{(const T* const*)L->w_gate, (const T* const*)L->w_up, (const T* const*)L->w_down,
                      L->dw_gate, L->dw_up, L->dw_down};
}

// Codes and row scales of the int8 forward.
struct Q8Ptrs {
  const int8_t* const* qg;
  const int8_t* const* qu;
  const int8_t* const* qd;
  const float* const* sg;
  const float* const* su;
  const float* const* sd;
};

// Four consecutive row scales from col (clamped so that the four stay inside
// the row count n, n >= 4; columns past n are never stored).
__device__ __forceinline__ f32x4_t scale4(const float* s, int col, int n) {
  const int c = min(col, n - 4);
  return f32x4_t{s[c], s[c + 1], s[c + 2], s[c + 3]};
}

__device__ __forceinline__ float sigm(float z) { return 1.0f / (1.0f + expf(-z)); }
// Logistic function with the hardware exp2 and reciprocal (about 1 ulp each),
// for epilogues whose results are rounded to bf16.
__device__ __forceinline__ float sigm_fast(float z) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}

// Order of the (row tile, column tile) pairs of one slot: bands of GM row
// tiles; inside a band column tiles advance slowest and row tiles fastest.  The
// blocks of an XCD working on one band share its GM activation tiles and a few
// weight tiles, a working set that fits the XCD's L2.
__device__ __forceinline__ void band_order(int loc, int mt, int NT, int GM, int& m, int& n) {
  const int band = loc / (GM * NT);
  const int h = min(GM, mt - band * GM);
  const int rem = loc - band * GM * NT;
  n = rem / h;
  m = band * GM + rem % h;
}

// x moved between lanes by a DPP control within each 16-lane row.
template <int CTRL> __device__ __forceinline__ float dpp_f(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}

// Sum of x over aligned groups of N = 8, 16 or 32 lanes, in every lane of the
// group: quad permutes (lane ^ 1, lane ^ 2), the half-row mirror (quad pairs)
// and the row mirror (half-row pairs) inside each row of 16, then one exchange
// across the two rows for N = 32.  Each step adds a lane's value to a partner
// holding a sum over the other, equally sized part, so every lane of the group
// ends with the same bits.
template <int N> __device__ __forceinline__ float row_lanes_sum(float x) {
  static_assert(N == 8 || N == 16 || N == 32, "half a DPP row, or one or two");
  x += dpp_f<0xB1>(x);    // quad_perm [1, 0, 3, 2]
  x += dpp_f<0x4E>(x);    // quad_perm [2, 3, 0, 1]
  x += dpp_f<0x141>(x);   // row_half_mirror
  if (N >= 16) x += dpp_f<0x140>(x);   // row_mirror
  if (N == 32) x += __shfl_xor(x, 16);
  return x;
}

}  // namespace
}  // namespace fm
