// Grouped SwiGLU expert FFN on small tiles: fp32 layers, and bf16 layers whose
// slots hold few rows (see tile_plan).  Same rows, outputs and rounding points
// as the large-tile kernels of ffn.hip.
//
// A kernel needs no schedule from an earlier launch: every block turns the
// offsets into its own prefix of row tiles per slot in LDS (a block scan, about
// a microsecond, against a launch of its own for a schedule kernel) and finds a
// tile's slot with a ballot over that prefix.  Blocks are dealt to the 8 XCDs
// round-robin; each XCD walks its own contiguous range of a row product's
// tiles, so that the row tiles of a slot that share a weight tile meet in one
// L2.  Weight-gradient tiles are dealt over all blocks, the slots with most rows
// first, since a tile's cost is its slot's rows.
//
// What bounds them.  fp32: the matrix pipe (157 TFLOP/s), 77 % busy at 24000
// rows, d = 1024, I = 768 (forward + backward 2.87 ms); a step of T = 1023, d =
// 1000, I = 616, 16 + 1 experts takes 0.68 ms (1.14 with a 128 x 128 tile per
// compute unit, register-staged, one slab ahead), one of 256 tokens, d = 128, I =
// 256, 8 experts 73 us (213; 14 launches, the products 48 us of them).  bf16 with few rows per slot: the weights' bytes; at T = 64,
// d = 2048, I = 1408, 64 slots gate-up streams 738 MB in 97 us (126 on 256-row
// tiles, which leave one block per compute unit and 9 of 10 rows empty), down 50
// (75), dH 51 (94), dX 145 (183: k-major rows 4 KB apart share L2 channels).
#include "ffn_common.hpp"
#include "ffn_tile.hpp"
#include "gemm_tile.hpp"

namespace fm {
namespace {

constexpr int MAX_S = 1023;   // slots of a layer (512 routed + 511 shared)

// Block prefix of row tiles: pre[s] = tiles of the slots before s, s in [0, S].
__device__ __forceinline__ void tile_sched(int* pre, int* wsum, const RowArgs& ra, int tile_rows) {
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  int carry = 0;
  for (int b = 0; b < ra.S; b += 256) {
    const int s = b + tid;
    int n = 0;
    if (s < ra.S) {
      const int rows = s < ra.S_r ? ra.offsets[s + 1] - ra.offsets[s] : ra.Tn;
      n = (rows + tile_rows - 1) / tile_rows;
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(n, o);
      if (lane >= o) n += v;
    }
    if (lane == 63) wsum[wave] = n;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int v = wsum[w];
      if (w < wave) n += v;
    }
    if (s < ra.S) pre[s + 1] = carry + n;
    carry += wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
  }
  if (tid == 0) pre[0] = 0;
  __syncthreads();
}

// The slot of row tile m: the number of slots whose tiles all lie before it.
__device__ __forceinline__ int tile_slot(const int* pre, int S, int m) {
  int c = 0;
  for (int b = 0; b < S; b += 64) {
    const int s = b + lane_id();
    c += __builtin_popcountll(__ballot(s < S && pre[s + 1] <= m));
  }
  return __builtin_amdgcn_readfirstlane(c);
}

// One row tile: its slot's rows from the tile's first on, and its column tile.
struct RowTile {
  SlotRows sr;
  int s, m0, n;
  int rows;     // rows of the slot from m0 on
  size_t ob;    // first row in the per-row buffers
};
__device__ __forceinline__ RowTile row_tile_at(const int* pre, const RowArgs& ra, int t, int NT, int RA) {
  RowTile r;
  r.s = tile_slot(pre, ra.S, t / NT);
  const int mb = __builtin_amdgcn_readfirstlane(pre[r.s]);
  const int mt = __builtin_amdgcn_readfirstlane(pre[r.s + 1]) - mb;
  int m;
  band_order(t - mb * NT, mt, NT, 8, m, r.n);
  r.sr = slot_rows(r.s, ra.offsets, ra.S_r, ra.Tn, ra.k);
  r.m0 = m * RA;
  r.rows = r.sr.nrows - r.m0;
  r.ob = (size_t)(r.sr.orow0 + r.m0);
  return r;
}

// This block's tiles of a row product: [lo, hi) by step, the XCD's own range.
struct Span {
  int lo, hi, step;
};
__device__ __forceinline__ Span row_span(const int* pre, const RowArgs& ra, int NT) {
  const long long total = (long long)pre[ra.S] * NT;
  const int x = blockIdx.x % N_XCD;
  return Span{__builtin_amdgcn_readfirstlane((int)(total * x / N_XCD)) + (int)(blockIdx.x / N_XCD),
              __builtin_amdgcn_readfirstlane((int)(total * (x + 1) / N_XCD)), (int)(gridDim.x / N_XCD)};
}

template <typename T> __device__ __forceinline__ float tile_sigm(float z) { return sigm(z); }
template <> __device__ __forceinline__ float tile_sigm<bf16>(float z) { return sigm_fast(z); }

template <class C> __device__ __forceinline__ AccCoord tile_coord(int i, int j, int q) {
  const int lane = lane_id(), wave = tile_wave<C>();
  return AccCoord{tile_row0<C>(wave) + i * 32 + (lane & 31),
                  tile_col0<C>(wave) + j * 32 + 8 * q + 4 * (lane >> 5)};
}

// Whether this wave holds sums after tile_gemm (of the waves that split k, those with wk = 0).
template <class C> __device__ __forceinline__ bool tile_holds() {
  return C::WM * C::WN == 4 || tile_wave<C>() < C::WM * C::WN;
}

// Puts a block's accumulators into LDS as an RA x RB tile of TO.
template <class C, typename TO>
__device__ __forceinline__ void tile_stage(const B16Acc<C::MI, C::NJ>& acc, FM_LDS char* lds) {
  static_assert(C::RA * C::RB * (int)sizeof(TO) <= C::LDS, "staged tile");
  using S = Stage<TO, C::RB>;
  if (tile_holds<C>()) {
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
#pragma unroll
      for (int j = 0; j < C::NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const AccCoord c = tile_coord<C>(i, j, q);
          S::put4(lds, c.row, c.col4, acc.quad(i, j, q));
        }
  }
  barrier_lds_writes();
}

// [A_g | A_u] = X_s [W_gate | W_up]^T, H = silu(A_g) A_u from A_g, A_u as
// stored.  The B tile interleaves 32-row blocks of W_gate and W_up: RB / 2
// intermediate columns per tile.
template <class C>
__global__ __launch_bounds__(256, C::BPC) void kt_gate_up(LayerPtrs<typename C::T> W,
                                                          const typename C::T* __restrict__ X,
                                                          const typename C::T* __restrict__ Xp, RowArgs ra,
                                                          typename C::T* __restrict__ Ag,
                                                          typename C::T* __restrict__ Au,
                                                          typename C::T* __restrict__ H) {
  typedef typename C::T T;
  __shared__ __align__(16) char lds_[C::LDS];
  __shared__ int pre[MAX_S + 1];
  __shared__ int wsum[4];
  FM_LDS char* const lds = (FM_LDS char*)lds_;
  constexpr int CI = C::RB / 2;
  using SG = Stage<T, CI>;
  const int d = ra.d, I = ra.I, NT = (I + CI - 1) / CI;
  tile_sched(pre, wsum, ra, C::RA);
  const Span sp = row_span(pre, ra, NT);
  for (int t = sp.lo; t < sp.hi; t += sp.step) {
    const RowTile r = row_tile_at(pre, ra, t, NT, C::RA);
    const int n0 = r.n * CI, cols = I - n0;
    const TileSrc<T> A{(r.sr.shared ? X : Xp) + (size_t)(r.sr.xrow0 + r.m0) * d, nullptr, nullptr, d, r.rows};
    const TileSrc<T> B{ld_scalar(W.wg + r.s) + (size_t)n0 * d, ld_scalar(W.wu + r.s) + (size_t)n0 * d, nullptr, d, cols};
    B16Acc<C::MI, C::NJ> acc;
    acc.zero();
    tile_gemm<C, true, true, false, true>(A, B, d, lds, acc);
    FM_LDS char* const sg = lds;
    FM_LDS char* const su = lds + C::RA * CI * (int)sizeof(T);
    if (tile_holds<C>()) {
#pragma unroll
      for (int i = 0; i < C::MI; ++i)
#pragma unroll
        for (int j = 0; j < C::NJ; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const AccCoord c = tile_coord<C>(i, j, q);
            SG::put4((c.col4 >> 5) & 1 ? su : sg, c.row, 32 * (c.col4 >> 6) + (c.col4 & 31), acc.quad(i, j, q));
          }
    }
    barrier_lds_writes();
    const int tid = wave_id() * 64 + lane_id_here();
#pragma unroll 2
    for (int idx = tid; idx < C::RA * SG::CPR; idx += 256) {
      const int row = idx / SG::CPR, c = idx % SG::CPR;
      const uint32_t off = row * SG::ROW_BYTES + ((c ^ (row & (SG::CPR - 1))) << 4);
      const u32x4_t g = *(const FM_LDS u32x4_t*)(sg + off);
      const u32x4_t u = *(const FM_LDS u32x4_t*)(su + off);
      if (row < r.rows && c * SG::EPC < cols) {
        const size_t o = (r.ob + row) * I + n0 + c * SG::EPC;
        float a[SG::EPC], v[SG::EPC], h[SG::EPC];
        unpack16(g, a, (T*)nullptr);
        unpack16(u, v, (T*)nullptr);
#pragma unroll
        for (int e = 0; e < SG::EPC; ++e) h[e] = a[e] * tile_sigm<T>(a[e]) * v[e];
        st16(Ag + o, g);
        st16(Au + o, u);
        st16(H + o, pack16(h, (T*)nullptr));
      }
    }
    barrier_lds();
  }
}

// O = H W_down^T.
template <class C>
__global__ __launch_bounds__(256, C::BPC) void kt_down(LayerPtrs<typename C::T> W,
                                                       const typename C::T* __restrict__ H, RowArgs ra,
                                                       typename C::T* __restrict__ O) {
  typedef typename C::T T;
  __shared__ __align__(16) char lds_[C::LDS];
  __shared__ int pre[MAX_S + 1];
  __shared__ int wsum[4];
  FM_LDS char* const lds = (FM_LDS char*)lds_;
  const int d = ra.d, I = ra.I, NT = (d + C::RB - 1) / C::RB;
  tile_sched(pre, wsum, ra, C::RA);
  const Span sp = row_span(pre, ra, NT);
  for (int t = sp.lo; t < sp.hi; t += sp.step) {
    const RowTile r = row_tile_at(pre, ra, t, NT, C::RA);
    const int n0 = r.n * C::RB;
    const TileSrc<T> A{H + r.ob * I, nullptr, nullptr, I, r.rows};
    const TileSrc<T> B{ld_scalar(W.wd + r.s) + (size_t)n0 * I, nullptr, nullptr, I, d - n0};
    B16Acc<C::MI, C::NJ> acc;
    acc.zero();
    tile_gemm<C, true, true>(A, B, I, lds, acc);
    tile_stage<C, T>(acc, lds);
    Stage<T, C::RB>::template copy_out<C::RA, 256>(lds, O + r.ob * d + n0, d, r.rows, d - n0);
    barrier_lds();
  }
}

// dH = dO W_down (B = W_down read k-major), rounded to T, then the SwiGLU
// backward in 16-byte row chunks; per row and column tile the sums of
// dA_g^2 + dA_u^2 and h^2 go to norms[row * NT + n] (the expert utility).
template <class C>
__global__ __launch_bounds__(256, C::BPC) void kt_dh(LayerPtrs<typename C::T> W,
                                                     const typename C::T* __restrict__ dO,
                                                     const typename C::T* __restrict__ Ag,
                                                     const typename C::T* __restrict__ Au, RowArgs ra,
                                                     typename C::T* __restrict__ dAg,
                                                     typename C::T* __restrict__ dAu, float2* __restrict__ norms) {
  typedef typename C::T T;
  __shared__ __align__(16) char lds_[C::LDS];
  __shared__ int pre[MAX_S + 1];
  __shared__ int wsum[4];
  FM_LDS char* const lds = (FM_LDS char*)lds_;
  using S = Stage<T, C::RB>;
  constexpr int V = C::V, CH = S::CPR, PER = C::RA * CH / 256, G = PER < 4 ? PER : 4;
  static_assert(C::RA * CH % 256 == 0 && PER % G == 0, "whole chunks per lane");
  static_assert(C::RB >= NORM_COLS_MIN, "the norm partials' place in the workspace");
  const int d = ra.d, I = ra.I, NT = (I + C::RB - 1) / C::RB;
  tile_sched(pre, wsum, ra, C::RA);
  const Span sp = row_span(pre, ra, NT);
  for (int t = sp.lo; t < sp.hi; t += sp.step) {
    const RowTile r = row_tile_at(pre, ra, t, NT, C::RA);
    const int n0 = r.n * C::RB, cols = I - n0;
    const TileSrc<T> A{dO + r.ob * d, nullptr, nullptr, d, r.rows};
    const TileSrc<T> B{ld_scalar(W.wd + r.s) + n0, nullptr, nullptr, I, cols};
    B16Acc<C::MI, C::NJ> acc;
    acc.zero();
    tile_gemm<C, true, false>(A, B, d, lds, acc);
    // A_g, A_u of the first chunks are on their way while the tile is staged
    const int tid = wave_id() * 64 + lane_id_here();
    u32x4_t ga[G], ua[G];
    auto load = [&](int g) {
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int idx = tid + (g * G + u) * 256, row = idx / CH, c = (idx % CH) * V;
        if (row < r.rows && c < cols) {
          const size_t o = (r.ob + row) * I + n0 + c;
          ga[u] = ld16(Ag + o);
          ua[u] = ld16(Au + o);
        }
      }
    };
    load(0);
    tile_stage<C, T>(acc, lds);
#pragma unroll
    for (int g = 0; g < PER / G; ++g) {
      if (g > 0) load(g);
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int idx = tid + (g * G + u) * 256, row = idx / CH, c = (idx % CH) * V;
        float sa = 0.f, sh = 0.f;
        if (row < r.rows && c < cols) {
          const size_t oo = (r.ob + row) * ra.ldA + n0 + c;
          float dh[V], a[V], up[V], dg[V], du[V];
          const u32x4_t hv = *(const FM_LDS u32x4_t*)(lds + S::at(row, c));
          unpack16(hv, dh, (T*)nullptr);
          unpack16(ga[u], a, (T*)nullptr);
          unpack16(ua[u], up, (T*)nullptr);
#pragma unroll
          for (int e = 0; e < V; ++e) {
            const float sg = tile_sigm<T>(a[e]);
            const float silu = a[e] * sg;
            du[e] = dh[e] * silu;
            dg[e] = dh[e] * up[e] * sg * (1.0f + a[e] * (1.0f - sg));
            const float h = silu * up[e];
            sa = fmaf(dg[e], dg[e], fmaf(du[e], du[e], sa));
            sh = fmaf(h, h, sh);
          }
          st16(dAg + oo, pack16(dg, (T*)nullptr));
          st16(dAu + oo, pack16(du, (T*)nullptr));
        }
        sa = row_lanes_sum<CH>(sa);
        sh = row_lanes_sum<CH>(sh);
        if ((tid & (CH - 1)) == 0 && row < r.rows) norms[(r.ob + row) * NT + r.n] = make_float2(sa, sh);
      }
    }
    barrier_lds();
  }
}

// dX_s = dA_g W_gate + dA_u W_up (B read k-major) as one k loop.
template <class C>
__global__ __launch_bounds__(256, C::BPC) void kt_dx(LayerPtrs<typename C::T> W,
                                                     const typename C::T* __restrict__ dAg,
                                                     const typename C::T* __restrict__ dAu, RowArgs ra,
                                                     typename C::T* __restrict__ dXp) {
  typedef typename C::T T;
  __shared__ __align__(16) char lds_[C::LDS];
  __shared__ int pre[MAX_S + 1];
  __shared__ int wsum[4];
  FM_LDS char* const lds = (FM_LDS char*)lds_;
  const int d = ra.d, I = ra.I, NT = (d + C::RB - 1) / C::RB;
  tile_sched(pre, wsum, ra, C::RA);
  const Span sp = row_span(pre, ra, NT);
  for (int t = sp.lo; t < sp.hi; t += sp.step) {
    const RowTile r = row_tile_at(pre, ra, t, NT, C::RA);
    const int n0 = r.n * C::RB;
    const TileSrc<T> A{dAg + r.ob * ra.ldA, nullptr, dAu + r.ob * ra.ldA, ra.ldA, r.rows};
    const TileSrc<T> B{ld_scalar(W.wg + r.s) + n0, nullptr, ld_scalar(W.wu + r.s) + n0, d, d - n0};
    B16Acc<C::MI, C::NJ> acc;
    acc.zero();
    tile_gemm<C, true, false, false, false, true>(A, B, I, lds, acc);
    tile_stage<C, T>(acc, lds);
    Stage<T, C::RB>::template copy_out<C::RA, 256>(lds, dXp + r.ob * d + n0, d, r.rows, d - n0);
    barrier_lds();
  }
}

// The tuning slots, most rows first (ties: lower index), in order[0 .. n);
// key: S ints of LDS, free again on return.
__device__ __forceinline__ int tile_dw_order(FM_LDS int* key, short* order, const RowArgs& ra,
                                             float* const* dw_tab) {
  int n = 0;
  for (int b = 0; b < ra.S; b += 256) {
    const int s = b + threadIdx.x;
    bool tune = false;
    if (s < ra.S) {
      tune = dw_tab[s] != nullptr;
      key[s] = !tune ? -1 : s < ra.S_r ? ra.offsets[s + 1] - ra.offsets[s] : ra.Tn;
    }
    n += __syncthreads_count(tune);
  }
  for (int s = threadIdx.x; s < ra.S; s += 256) {
    const int rows = key[s];
    if (rows < 0) continue;
    int rank = 0;
    for (int u = 0; u < ra.S; ++u) rank += key[u] > rows || (key[u] == rows && u < s);
    order[rank] = (short)s;
  }
  __syncthreads();
  return n;
}

// Zeros part i of n of a weight gradient of `count` floats, as one contiguous run
// (the gradient of a slot without rows; one that accumulates has nothing to add
// and is skipped).  Written tile by tile, rows that are not whole 128-byte lines
// were stored at half the rate.
__device__ __forceinline__ void zero_part(float* p, long long count, int i, int n) {
  const long long c4 = count / 4, hi = c4 * (i + 1) / n;
  for (long long c = c4 * i / n + threadIdx.x; c < hi; c += 256) st16(p + 4 * c, u32x4_t{0, 0, 0, 0});
}

// dW_gate = dA_g^T X_s and dW_up = dA_u^T X_s in one product: the A tile
// interleaves 32-column blocks of dA_g and dA_u (RA / 2 intermediate rows of
// both per tile); both operands read k-major, k = the slot's rows.
template <class C>
__global__ __launch_bounds__(256, C::BPC) void kt_dw_gu(LayerPtrs<typename C::T> W,
                                                        const typename C::T* __restrict__ X,
                                                        const typename C::T* __restrict__ Xp,
                                                        const typename C::T* __restrict__ dAg,
                                                        const typename C::T* __restrict__ dAu, RowArgs ra,
                                                        int accumulate) {
  typedef typename C::T T;
  __shared__ __align__(16) char lds_[C::LDS];
  __shared__ short order[MAX_S + 1];
  FM_LDS char* const lds = (FM_LDS char*)lds_;
  constexpr int CI = C::RA / 2;
  const int d = ra.d, I = ra.I, ld = ra.ldA;
  const int MT = (I + CI - 1) / CI, NT = (d + C::RB - 1) / C::RB, tps = MT * NT;
  const int total = __builtin_amdgcn_readfirstlane(tile_dw_order((FM_LDS int*)lds, order, ra, W.dwg)) * tps;
  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    const int s = __builtin_amdgcn_readfirstlane(order[t / tps]);
    float* const dwg = ld_scalar(W.dwg + s);
    float* const dwu = ld_scalar(W.dwu + s);
    if (!dwu) continue;
    int m, n;
    band_order(t % tps, MT, NT, 8, m, n);
    const SlotRows sr = slot_rows(s, ra.offsets, ra.S_r, ra.Tn, ra.k);
    const int m0 = m * CI, n0 = n * C::RB;
    auto row_ptr = [=](int r) {
      const int mm = m0 + 32 * (r >> 6) + (r & 31);
      return mm < I ? ((r >> 5) & 1 ? dwu : dwg) + (size_t)mm * d + n0 : (float*)nullptr;
    };
    if (sr.nrows == 0) {
      if (!accumulate) {
        zero_part(dwg, (long long)I * d, t % tps, tps);
        zero_part(dwu, (long long)I * d, t % tps, tps);
      }
      continue;
    }
    const TileSrc<T> A{dAg + (size_t)sr.orow0 * ld + m0, dAu + (size_t)sr.orow0 * ld + m0, nullptr, ld, I - m0};
    const TileSrc<T> B{(sr.shared ? X : Xp) + (size_t)sr.xrow0 * d + n0, nullptr, nullptr, d, d - n0};
    B16Acc<C::MI, C::NJ> acc;
    acc.zero();
    tile_gemm<C, false, false, true, false>(A, B, sr.nrows, lds, acc);
    tile_stage<C, float>(acc, lds);
    Stage<float, C::RB>::template copy_rows<C::RA, 256>(lds, row_ptr, d - n0, accumulate);
    barrier_lds();
  }
}

// dW_down = dO^T H, both operands read k-major.
template <class C>
__global__ __launch_bounds__(256, C::BPC) void kt_dw_d(LayerPtrs<typename C::T> W,
                                                       const typename C::T* __restrict__ dO,
                                                       const typename C::T* __restrict__ H, RowArgs ra,
                                                       int accumulate) {
  typedef typename C::T T;
  __shared__ __align__(16) char lds_[C::LDS];
  __shared__ short order[MAX_S + 1];
  FM_LDS char* const lds = (FM_LDS char*)lds_;
  const int d = ra.d, I = ra.I;
  const int MT = (d + C::RA - 1) / C::RA, NT = (I + C::RB - 1) / C::RB, tps = MT * NT;
  const int total = __builtin_amdgcn_readfirstlane(tile_dw_order((FM_LDS int*)lds, order, ra, W.dwg)) * tps;
  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    const int s = __builtin_amdgcn_readfirstlane(order[t / tps]);
    float* const dwd = ld_scalar(W.dwd + s);
    if (!dwd) continue;
    int m, n;
    band_order(t % tps, MT, NT, 8, m, n);
    const SlotRows sr = slot_rows(s, ra.offsets, ra.S_r, ra.Tn, ra.k);
    const int m0 = m * C::RA, n0 = n * C::RB;
    auto row_ptr = [=](int r) { return m0 + r < d ? dwd + (size_t)(m0 + r) * I + n0 : (float*)nullptr; };
    if (sr.nrows == 0) {
      if (!accumulate) zero_part(dwd, (long long)I * d, t % tps, tps);
      continue;
    }
    const TileSrc<T> A{dO + (size_t)sr.orow0 * d + m0, nullptr, nullptr, d, d - m0};
    const TileSrc<T> B{H + (size_t)sr.orow0 * I + n0, nullptr, nullptr, I, I - n0};
    B16Acc<C::MI, C::NJ> acc;
    acc.zero();
    tile_gemm<C, false, false>(A, B, sr.nrows, lds, acc);
    tile_stage<C, float>(acc, lds);
    Stage<float, C::RB>::template copy_rows<C::RA, 256>(lds, row_ptr, I - n0, accumulate);
    barrier_lds();
  }
}

// The int8 forward: H = silu(s_g (X_s Q_g^T)) (s_u (X_s Q_u^T)) with the codes
// interleaved as in kt_gate_up.  Where a wave's columns are whole gate / up pairs
// of 32-blocks, H is formed from its fp32 sums in registers; a wave of one
// 32-block puts its scaled sums into LDS as fp32 and H is formed on the way out
// (same values, same operations).
template <class C>
__global__ __launch_bounds__(256, C::BPC) void kt_q8_gate_up(Q8Ptrs W, const bf16* __restrict__ X,
                                                             const bf16* __restrict__ Xp, RowArgs ra,
                                                             bf16* __restrict__ H) {
  __shared__ __align__(16) char lds_[C::LDS];
  __shared__ int pre[MAX_S + 1];
  __shared__ int wsum[4];
  static_assert(C::WK == 1 && (C::NJ == 1 || C::NJ % 2 == 0), "one 32-block or gate / up pairs per wave");
  FM_LDS char* const lds = (FM_LDS char*)lds_;
  constexpr int CI = C::RB / 2;
  using SG = Stage<bf16, CI>;
  using SF = Stage<float, C::RB>;
  static_assert(C::NJ > 1 || C::RA * SF::ROW_BYTES <= C::LDS, "staged sums");
  const int d = ra.d, I = ra.I, NT = (I + CI - 1) / CI;
  tile_sched(pre, wsum, ra, C::RA);
  const Span sp = row_span(pre, ra, NT);
  for (int t = sp.lo; t < sp.hi; t += sp.step) {
    const RowTile r = row_tile_at(pre, ra, t, NT, C::RA);
    const int n0 = r.n * CI, cols = I - n0;
    const TileSrc<bf16> A{(r.sr.shared ? X : Xp) + (size_t)(r.sr.xrow0 + r.m0) * d, nullptr, nullptr, d, r.rows};
    const TileSrc<int8_t> B{ld_scalar(W.qg + r.s) + (size_t)n0 * d, ld_scalar(W.qu + r.s) + (size_t)n0 * d, nullptr, d,
                            cols};
    B16Acc<C::MI, C::NJ> acc;
    acc.zero();
    tile_gemm<C, true, true, false, true>(A, B, d, lds, acc);
    const float* const sg = ld_scalar(W.sg + r.s) + n0;
    const float* const su = ld_scalar(W.su + r.s) + n0;
    auto form = [](float a, float u) { return a * sigm_fast(a) * u; };
    if constexpr (C::NJ == 1) {
      // rows of RB fp32 values, 32 gate and 32 up columns in turn
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c4 = tile_coord<C>(0, 0, q).col4;
        const f32x4_t sc = scale4((c4 >> 5) & 1 ? su : sg, 32 * (c4 >> 6) + (c4 & 31), cols);
#pragma unroll
        for (int i = 0; i < C::MI; ++i) {
          const f32x4_t v = acc.quad(i, 0, q);
          SF::put4(lds, tile_coord<C>(i, 0, q).row, c4, f32x4_t{v[0] * sc[0], v[1] * sc[1], v[2] * sc[2], v[3] * sc[3]});
        }
      }
      barrier_lds_writes();
      const int tid = wave_id() * 64 + lane_id_here();
#pragma unroll 2
      for (int idx = tid; idx < C::RA * SG::CPR; idx += 256) {
        const int row = idx / SG::CPR, col = idx % SG::CPR * 8, c = 64 * (col >> 5) + (col & 31);
        float h[8];
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
          const f32x4_t g = *(const FM_LDS f32x4_t*)(lds + SF::at(row, c + e));
          const f32x4_t u = *(const FM_LDS f32x4_t*)(lds + SF::at(row, c + 32 + e));
#pragma unroll
          for (int x = 0; x < 4; ++x) h[e + x] = form(g[x], u[x]);
        }
        if (row < r.rows && col < cols) st16(H + (r.ob + row) * I + n0 + col, pack16(h, (bf16*)nullptr));
      }
    } else {
#pragma unroll
      for (int jj = 0; jj < C::NJ / 2; ++jj)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c4 = tile_coord<C>(0, 2 * jj, q).col4, col = 32 * (c4 >> 6) + (c4 & 31);
          const f32x4_t cg = scale4(sg, col, cols), cu = scale4(su, col, cols);
#pragma unroll
          for (int i = 0; i < C::MI; ++i) {
            const f32x4_t g = acc.quad(i, 2 * jj, q), u = acc.quad(i, 2 * jj + 1, q);
            f32x4_t h;
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = form(g[e] * cg[e], u[e] * cu[e]);
            SG::put4(lds, tile_coord<C>(i, 2 * jj, q).row, col, h);
          }
        }
      barrier_lds_writes();
      SG::template copy_out<C::RA, 256>(lds, H + r.ob * I + n0, I, r.rows, cols);
    }
    barrier_lds();
  }
}

// O = s_d (H Q_d^T).
template <class C>
__global__ __launch_bounds__(256, C::BPC) void kt_q8_down(Q8Ptrs W, const bf16* __restrict__ H, RowArgs ra,
                                                          bf16* __restrict__ O) {
  __shared__ __align__(16) char lds_[C::LDS];
  __shared__ int pre[MAX_S + 1];
  __shared__ int wsum[4];
  FM_LDS char* const lds = (FM_LDS char*)lds_;
  const int d = ra.d, I = ra.I, NT = (d + C::RB - 1) / C::RB;
  tile_sched(pre, wsum, ra, C::RA);
  const Span sp = row_span(pre, ra, NT);
  for (int t = sp.lo; t < sp.hi; t += sp.step) {
    const RowTile r = row_tile_at(pre, ra, t, NT, C::RA);
    const int n0 = r.n * C::RB, cols = d - n0;
    const TileSrc<bf16> A{H + r.ob * I, nullptr, nullptr, I, r.rows};
    const TileSrc<int8_t> B{ld_scalar(W.qd + r.s) + (size_t)n0 * I, nullptr, nullptr, I, cols};
    B16Acc<C::MI, C::NJ> acc;
    acc.zero();
    tile_gemm<C, true, true>(A, B, I, lds, acc);
    const float* const sd = ld_scalar(W.sd + r.s) + n0;
#pragma unroll
    for (int j = 0; j < C::NJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4_t c4 = scale4(sd, tile_coord<C>(0, j, q).col4, cols);
#pragma unroll
        for (int i = 0; i < C::MI; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc.v[i][j][4 * q + e] *= c4[e];
      }
    tile_stage<C, bf16>(acc, lds);
    Stage<bf16, C::RB>::template copy_out<C::RA, 256>(lds, O + r.ob * d + n0, d, r.rows, cols);
    barrier_lds();
  }
}

// ------------------------------------------------------------------ host ----

// (Tile indices fit in 32 bits.  A row product has at most rows / RA + slots row tiles:
// the full ones write 4 KB or more per column tile, so 2^31 would not fit in memory,
// and the partial ones, one per slot, come to no more than the 32-column blocks of the
// slots' weights.  A weight-gradient tile writes at least 8 x 8 values of 4 bytes.)
// Blocks for at most `tiles` tiles, BPC per compute unit, a multiple of the XCDs.
template <class C> dim3 tile_grid(long long tiles) {
  const long long most = (long long)persistent_blocks() * C::BPC;
  const long long g = (tiles + N_XCD - 1) / N_XCD * N_XCD;
  return dim3((unsigned)(g < N_XCD ? N_XCD : g < most ? g : most));
}
// Upper bound of the row tiles of a layer (the bucket sizes are on the device).
template <class C> long long max_row_tiles(const RowArgs& ra) {
  const long long R = (long long)ra.Tn * ra.k;
  const long long routed = R / C::RA + (R < ra.S_r ? R : ra.S_r);
  return routed + (long long)(ra.S - ra.S_r) * ((ra.Tn + C::RA - 1) / C::RA);
}

using F64 = TileCfg<float, 64, 64, 2, 2, 1, 2, 4>;
using F32 = TileCfg<float, 32, 64, 1, 2, 2, 4, 3>;
using FD32 = TileCfg<float, 64, 32, 2, 1, 2, 4, 3>;   // weight gradients, few tiles
// Two of its waves multiply and all four move data: what such a tile waits for is
// its weights.  (k split over two pairs of waves, whose sums met in LDS, gave the same
// 28 and 15 us for gate-up and down at T = 8, d = 4096, I = 688, 16 slots.)
using B32 = TileCfg<bf16, 32, 64, 1, 2, 1, 4, 3>;
using B64 = TileCfg<bf16, 64, 128, 2, 2, 1, 3, 2>;
using B128 = TileCfg<bf16, 128, 128, 2, 2, 1, 2, 2>;
using D128 = TileCfg<bf16, 128, 128, 2, 2, 1, 4, 2, 2, 64>;   // weight gradients: half slabs, three in flight

// int8 weights.  Widening a fragment costs 12 vector instructions, so a wave
// covers all of the tile's rows (each code is widened once per block, not once
// per row of waves): 1, 2 or 4 MFMAs per widened fragment on the 32, 64 and
// 128-row tiles.  The first two give every wave one 32-column block; pairs of
// waves splitting k over two such blocks were 1-5 % slower (gate-up + down at T =
// 512, d = 2048, I = 1408, 64 slots, top-6 165 us, now 161; T = 900, d = 768, I =
// 512, 32 slots, top-5 33.1, now 31.5) and added their sums in another order.
using Q32 = TileCfg<bf16, 32, 128, 1, 4, 1, 4, 3, 1>;
using Q64 = TileCfg<bf16, 64, 128, 1, 4, 1, 3, 3, 1>;
using Q128 = TileCfg<bf16, 128, 256, 1, 4, 1, 2, 2, 1>;

// Calls fn(C{}) with the tile of the plan's row products.
template <class Fn> void with_rows(const TilePlan& p, int dtype, Fn fn) {
  if (dtype == MOE_F32) {
    if (p.rows == TilePlan::ROWS_32) fn(F32{});
    else fn(F64{});
  } else if (p.rows == TilePlan::ROWS_32) {
    fn(B32{});
  } else if (p.rows == TilePlan::ROWS_64) {
    fn(B64{});
  } else {
    fn(B128{});
  }
}
// fp32 products with fewer than two 64 x 64 tiles per compute unit split k over
// two waves on 64 x 32 tiles (backward at T = 2000, d = 256, I = 128, 8 slots: 83
// -> 63 us).
// bf16 weight gradients, each product by its 128 x 128 tiles (every slot counted as
// tuning): 64 x 128 tiles with whole slabs where those would be fewer than five
// per compute unit.  us on 64 x 128, 128 x 128: I = 512, d = 768, 32 slots, r =
// 512: dW_down (768 tiles) 50, 59, dW_gate/up (1536) 80, 77; r = 128 22, 24 and
// 40, 34; I = 256, d = 512, 16 slots, r = 2048 (128, 256 tiles) 66, 112 and 79,
// 123; I = 376, d = 712, 32 slots, r = 375 (576, 1152) 35, 40 and 52, 55; I =
// 1408, d = 2048, 64 slots, r = 96 114, 99 and 250, 187.
// Above 512 rows per slot that holds only where a slot has few tiles, so that the
// rows of a popular slot make a tail (48 of 128 x 128; us of the whole backward): I =
// 2376, d = 984, 3 slots (152, 304 tiles per slot) r = 1000 211, 186; r = 16000 3130,
// 2130; I = 256, d = 4096, 8 slots (64, 128) r = 2000 419, 365; I = 512, d = 1024, 16
// slots (32, 64) r = 1000 232, 229; r = 8000 1657, 1342; I = d = 256, 64 slots (4, 8) r
// = 2000 474, 520, Zipf 692, 857.
DwTile dw_tile_of(int dtype, long long tiles128, int S, double r) {
  if (dtype == MOE_F32) return 4 * tiles128 < 512 ? DW_SPLIT_K : DW_64;
  return tiles128 >= 1280 || (r > 512 && tiles128 >= 48LL * S) ? DW_128 : DW_64;
}
template <class Fn> void with_dw(DwTile t, int dtype, Fn fn) {
  if (dtype == MOE_F32) {
    if (t == DW_SPLIT_K) fn(FD32{});
    else fn(F64{});
  } else {
    if (t == DW_64) fn(B64{});
    else fn(D128{});
  }
}

RowArgs row_args(const moe_layer* L, const int32_t* offsets, int T, int k, int ldA) {
  return RowArgs{offsets, nullptr, L->S_routed, L->S_routed + L->S_shared, T, k, L->d, L->I, ldA};
}

}  // namespace

// Persistent grid unit: one block per compute unit, a multiple of the XCD count.
int persistent_blocks() {
  const int n = device_cus() / N_XCD * N_XCD;
  return n < N_XCD ? N_XCD : n;
}

TilePlan tile_plan(const moe_layer* L, int T, int k) {
  // r = average rows per slot; tiles estimated for average slots
  const int S = L->S_routed + L->S_shared, n_sh = L->S_shared;
  const double r = (double)T * (k + n_sh) / S;
  const double active = (double)((long long)T * k < L->S_routed ? (long long)T * k : L->S_routed) + n_sh;
  const long long wide = (2LL * L->I > L->d ? 2LL * L->I : L->d);
  TilePlan p;
  // Few rows: 32-row tiles make twice the blocks of the 64 x 128 tile and waste
  // less on absent rows, which counts while those would not fill the chip twice.
  // fwd at T = 8: I = 688, d = 4096, 16 slots 36 against 49 us; I = 1408, d = 2048,
  // 64 slots 83 against 93; at T = 64 (1408 tiles) 165 against 169, at r = 31 with
  // 1452 tiles 283 against 249.
  const bool few = r <= 32 && active * ((wide + 127) / 128) < 1024;
  if (L->dtype == MOE_F32) {
    // r = 7.5 (60 tokens, d = 712, I = 376, 32 slots): fwd 36 against 51 us.  Also
    // where the 64 x 64 tiles are fewer than two per compute unit: a tile's k loop is
    // then a chain of MFMAs that the 32-row tile's waves share two ways.  Forward
    // and backward us on 64, 32 rows: T = 256, d = 768, I = 600, 16 slots, k = 4 (456
    // tiles) 62, 47 and 120, 90; T = 500, d = I = 512, 8 slots, k = 2 (314) 40, 37 and
    // 84, 82; T = 256, d = 128, I = 256, 6 slots (90) 18, 18 and 42, 36.
    const bool idle = S * (r / 64 + 0.5) * ((wide + 63) / 64) < 512;
    p.rows = few || idle ? TilePlan::ROWS_32 : TilePlan::ROWS_64;
    p.dw = TilePlan::SMALL_DW;
    return p;
  }
  // Row products.  A large tile pays where its slots have the rows to fill it, its
  // layer the tiles to fill the chip and its k loops the length to hide a tile's ends
  // (one block per compute unit): the line follows r sqrt(S d I).  Below it the 64 x
  // 128 tile serves short buckets, and layers whose 128-row tiles would leave half of
  // the 512 blocks of the narrower of gate-up and down idle; 128 x 128 the rest.
  // Above 288 rows per slot only layers with idle chips lost on the large tiles.
  // us of forward + backward (the same weight-gradient tiles) on 64 x 128, 128 x 128
  // and the large tiles, buckets of a skewed router (even: equal popularity):
  //   S, d, I             r    64    128   large      r    64    128   large
  //   8, 1024, 2816      160  242    303    278      240  293    319    327
  //   16, 4096, 688      128  398    441    471      272  601    542    563
  //   64, 4096, 256       88  505    543    581      240  860    828    805
  //   32, 4096, 1024      88  931    962   1009      208  1334  1299   1198
  //   24, 3072, 1536      72  722    746    822      176  1014  1022    958
  //   64, 2048, 1408      72  1120  1108   1153      144  1377  1297   1289
  //     even              64  1072  1054   1081      144  1462  1447   1337
  //   128, 4096, 1408     72  4091  3868   3863      144  4952  4554   4276
  // The line lies at r^2 S d I = 2.5e12; the one between 64 and 128 at 0.7e12, or at
  // 0.9e12 while a 128-row tile would be a third empty (r <= 88).
  const double work = r * r * S * L->d * L->I;
  const double mt128 = S * (r / 128 + 0.5);
  const int nt128 = (L->d + 127) / 128 < (L->I + 63) / 64 ? (L->d + 127) / 128 : (L->I + 63) / 64;
  if (few) p.rows = TilePlan::ROWS_32;
  else if (r > 288 || work >= 2.5e12) p.rows = TilePlan::LARGE_ROWS;
  else if (work < (r <= 88 ? 0.9e12 : 0.7e12) || mt128 * nt128 <= 288) p.rows = TilePlan::ROWS_64;
  else p.rows = TilePlan::ROWS_128;
  // Weight gradients, us of the backward on the tiles of with_dw and on the large
  // ones.  The large ones need four tiles per compute unit (every slot counted as
  // tuning), and slots of about 288 rows: I = 1408, d = 2048, 64 slots r = 176 1065,
  // 1095; r = 272 1266, 1272; r = 340 1408, 1352; I = 688, d = 4096, 16 slots r = 176
  // 376, 380; r = 304 427, 424.  About 100 rows are enough where I is a multiple of 256
  // and d >= 3072 (the small tiles read half lines, here of rows a multiple of 512
  // bytes apart): I = 1024, 32 slots r = 112 760, 730, r = 240 967, 868; I = 256, d =
  // 4096, 64 slots r = 240 592, 542; I = 1536, d = 3072, 24 slots r = 112 648, 657, r =
  // 240 779, 751; and in the widest layers (d = 4096, I = 1408, 128 slots: r = 112
  // 3362, 3372; r = 240 4592, 4276).
  // Two tiles per compute unit are enough once a tile is long and a slot has 32 of them
  // (with fewer a popular slot's tiles make a tail: I = 280, d = 712, 98 slots, 882
  // tiles, r = 2315, Zipf 1734, 1981): I = 1408, d = 2048, 8 slots (704 tiles) r = 1000
  // 413, 408; r = 4000 1387, 1170; I = 688, d = 2048, 12 slots (576) r = 1000 377, 376; r
  // = 4000 1180, 1065; I = 768, d = 1536, 16 slots (576) r = 2000 648, 688; r = 8000
  // 2373, 2207; I = d = 1024, 16 slots (512) r = 1500 496, 486; r = 4000 1137, 1102.
  // Fewer never gained: I = 1408, d = 2048, 4 slots (352) r = 4000 740, 796; I = 512, d =
  // 768, 32 slots (384) r = 4000 1135, 1280; I = 512, d = 1024, 16 slots (256) r = 4000
  // 725, 853.  Except where the tokens' choices fill every slot alike (k >= S_routed, no
  // popular slot): I = 2376, d = 984, 3 slots (228) r = 2000 294, 287; r = 20000 2377,
  // 2026; I = 1408, d = 2048, 2 slots (176) r = 2000 195, 202; r = 8000 676, 598; I =
  // 2048, d = 768, 3 slots (144) r = 4000 374, 354; not I = d = 1024, 3 slots (96) r =
  // 20000 1087, 1231.
  const double dw256 = (double)S * ((L->I + 127) / 128) * ((L->d + 255) / 256);
  const bool dw_early = dw256 >= 8192 || (L->I % 256 == 0 && L->d >= 3072);
  const bool full = k >= L->S_routed;
  const bool dw_large = dw256 >= 1024 ? r > (dw_early ? 100 : 288)
                              : full ? dw256 >= 128 && r * dw256 >= 5e5
                                     : dw256 >= 512 && dw256 >= 32 * S && r * dw256 >= 1e6;
  p.dw = dw_large ? TilePlan::LARGE_DW : TilePlan::SMALL_DW;
  return p;
}

DwTile dw_tile(const moe_layer* L, int T, int k, bool gate_up) {
  const int S = L->S_routed + L->S_shared;
  return dw_tile_of(L->dtype, (long long)S * cdiv(L->d, 128) * cdiv(L->I, gate_up ? 64 : 128), S,
                    (double)T * (k + L->S_shared) / S);
}

int tile_norm_cols(const moe_layer* L, const TilePlan& p) {
  int n = 0;
  with_rows(p, L->dtype, [&](auto c) { n = decltype(c)::RB; });
  return n;
}

void tile_fwd(const TilePlan& p, const moe_layer* L, const void* X, const void* Xp, const int32_t* offsets, int Tn,
              int k, void* Ag, void* Au, void* H, void* O, hipStream_t st) {
  const RowArgs ra = row_args(L, offsets, Tn, k, L->I);
  with_rows(p, L->dtype, [&](auto c) {
    typedef decltype(c) C;
    typedef typename C::T T;
    const long long mt = max_row_tiles<C>(ra);
    hipLaunchKernelGGL(kt_gate_up<C>, tile_grid<C>(mt * cdiv(ra.I, C::RB / 2)), dim3(256), 0, st, layer_ptrs<T>(L),
                       (const T*)X, (const T*)Xp, ra, (T*)Ag, (T*)Au, (T*)H);
    hipLaunchKernelGGL(kt_down<C>, tile_grid<C>(mt * cdiv(ra.d, C::RB)), dim3(256), 0, st, layer_ptrs<T>(L),
                       (const T*)H, ra, (T*)O);
  });
}

void tile_dh(const TilePlan& p, const moe_layer* L, const int32_t* offsets, int Tn, int k, const void* Ag,
             const void* Au, const void* dO, void* dAg, void* dAu, int ldA, float2* norms, hipStream_t st) {
  const RowArgs ra = row_args(L, offsets, Tn, k, ldA);
  with_rows(p, L->dtype, [&](auto c) {
    typedef decltype(c) C;
    typedef typename C::T T;
    hipLaunchKernelGGL(kt_dh<C>, tile_grid<C>(max_row_tiles<C>(ra) * cdiv(ra.I, C::RB)), dim3(256), 0, st,
                       layer_ptrs<T>(L), (const T*)dO, (const T*)Ag, (const T*)Au, ra, (T*)dAg, (T*)dAu, norms);
  });
}

void tile_dx(const TilePlan& p, const moe_layer* L, const int32_t* offsets, int Tn, int k, const void* dAg,
             const void* dAu, int ldA, void* dXp, hipStream_t st) {
  const RowArgs ra = row_args(L, offsets, Tn, k, ldA);
  with_rows(p, L->dtype, [&](auto c) {
    typedef decltype(c) C;
    typedef typename C::T T;
    hipLaunchKernelGGL(kt_dx<C>, tile_grid<C>(max_row_tiles<C>(ra) * cdiv(ra.d, C::RB)), dim3(256), 0, st,
                       layer_ptrs<T>(L), (const T*)dAg, (const T*)dAu, ra, (T*)dXp);
  });
}

void tile_dw(const moe_layer* L, const void* X, const void* Xp, const int32_t* offsets, int Tn, int k, const void* H,
             const void* dO, const void* dAg, const void* dAu, int ldA, int accumulate, hipStream_t st) {
  const RowArgs ra = row_args(L, offsets, Tn, k, ldA);
  with_dw(dw_tile(L, Tn, k, false), L->dtype, [&](auto c) {
    typedef decltype(c) C;
    typedef typename C::T T;
    hipLaunchKernelGGL(kt_dw_d<C>, tile_grid<C>((long long)ra.S * cdiv(ra.d, C::RA) * cdiv(ra.I, C::RB)), dim3(256), 0,
                       st, layer_ptrs<T>(L), (const T*)dO, (const T*)H, ra, accumulate);
  });
  with_dw(dw_tile(L, Tn, k, true), L->dtype, [&](auto c) {
    typedef decltype(c) C;
    typedef typename C::T T;
    hipLaunchKernelGGL(kt_dw_gu<C>, tile_grid<C>((long long)ra.S * cdiv(ra.I, C::RA / 2) * cdiv(ra.d, C::RB)),
                       dim3(256), 0, st, layer_ptrs<T>(L), (const T*)X, (const T*)Xp, (const T*)dAg, (const T*)dAu, ra,
                       accumulate);
  });
}

// Rows of the int8 forward's row tile, from the average rows per slot r and the tiles:
// 32, 64 and 128 on the core of this file, 256 on the 8-wave tile of ffn.hip.  us of
// gate-up + down on each.  d = 2048, I = 1408, 64 slots: r = 6 94, 92, 120, 186; r = 24
// 144, 132, 155, 241; r = 48 191, 161, 184, 257; r = 96 283, 223, 211, 329; r = 384 930,
// 633, 523, 567.  d = 4096, I = 688, 16 slots: r = 2 45, 50, 89, 101; r = 64 64, 67, 98,
// 111; r = 194 (192 128-row tiles) 134, 101, 118, 151; r = 375 (330 tiles) 249, 167,
// 164, 191; r = 1024 622, 432, 357, 359.  d = 768, I = 512, 32 slots: r = 2 17, 19, 33,
// 38; r = 128 37, 29, 37, 57; r = 512 100, 72, 67, 90.
// The 256-row tile moves 3/4 of the bytes per product and holds one block per compute
// unit, so it needs many rows and large layers (r^2 S d I, as the bf16 row products),
// us on 128, 256 rows: 64 slots, d = 2048, I = 1408 r = 512 615, 645; r = 1024 1174,
// 1146; r = 4096 4665, 4278; d = 4096, I = 1024 r = 4096 6945, 6203; d = 1024, I = 2816 r
// = 768 944, 971; r = 2048 2395, 2363; 8 slots, d = 4096, I = 2816 r = 512 290, 305; r =
// 2048 1034, 996; r = 8192 4286, 3822; 4 slots r = 2000 569, 552; r = 10000 2621, 2436.
// Smaller layers need more rows: 16 slots, d = 4096, I = 688 r = 2048 638, 690; r = 4096
// 1228, 1272; r = 8192 2457, 2448; 8 slots, d = 2048, I = 1408 r = 2000 300, 310; r =
// 10000 1395, 1324; 16 slots, d = I = 1024 r = 5000 566, 596; r = 10000 1114, 1072; 32
// slots, d = 1024, I = 512 r = 8192 936, 981; the smallest never gained: 3 slots, d =
// 976, I = 2368 r = 5000 242, 276; r = 20000 952, 954.
int q8_tile(const moe_layer_q8* L, int T, int k) {
  const int S = L->S_routed + L->S_shared;
  const double r = (double)T * (k + L->S_shared) / S;
  const double active = (double)((long long)T * k < L->S_routed ? (long long)T * k : L->S_routed) + L->S_shared;
  if (r <= 64 && active * ((2LL * L->I + 127) / 128) < 768) return 32;
  const double layer = (double)S * L->d * L->I;
  if (r * r * layer >= (layer >= 4.6e7 ? 1.5e14 : 1.2e15) && layer >= 1e7) return 256;
  return r >= 72 && S * (r / 128 + 0.5) * ((L->I + 127) / 128) >= 288 ? 128 : 64;
}

void tile_fwd_q8(const moe_layer_q8* L, const void* X, const void* Xp, const int32_t* offsets, int Tn, int k, void* H,
                 void* O, hipStream_t st) {
  const RowArgs ra{offsets, nullptr, L->S_routed, L->S_routed + L->S_shared, Tn, k, L->d, L->I, L->I};
  const Q8Ptrs W{L->q_gate, L->q_up, L->q_down, L->s_gate, L->s_up, L->s_down};
  auto run = [&](auto c) {
    typedef decltype(c) C;
    const long long mt = max_row_tiles<C>(ra);
    hipLaunchKernelGGL(kt_q8_gate_up<C>, tile_grid<C>(mt * cdiv(ra.I, C::RB / 2)), dim3(256), 0, st, W, (const bf16*)X,
                       (const bf16*)Xp, ra, (bf16*)H);
    hipLaunchKernelGGL(kt_q8_down<C>, tile_grid<C>(mt * cdiv(ra.d, C::RB)), dim3(256), 0, st, W, (const bf16*)H, ra,
                       (bf16*)O);
  };
  switch (q8_tile(L, Tn, k)) {
    case 32: run(Q32{}); break;
    case 64: run(Q64{}); break;
    default: run(Q128{}); break;   // q8_tile(L, Tn, k) < 256
  }
}

}  // namespace fm
