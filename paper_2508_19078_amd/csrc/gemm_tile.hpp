// Small-tile MFMA core for the grouped expert FFN (gfx950, wave64): blocks of
// 4 waves, several per compute unit, fp32 or bf16.
//
// A block computes an RA x RB tile of C = sum_k A(r, k) B(n, k); its waves
// form a WM x WN (x WK) grid and each owns MI x NJ 32 x 32 MFMA tiles
// (v_mfma_f32_32x32x16_bf16, or 4 x v_mfma_f32_32x32x2_f32 per 8 k), operands
// swapped so that a lane holds groups of four consecutive output columns.  On a
// tile with fewer than four 32 x 32 tiles the waves past the grid only move data.
//
// bf16 tiles never split k (WK = 1): every output element is one chain of MFMAs
// over ascending k, as in the large-tile core, so a row's results do not depend
// on the tile that its call takes.
//
// * Slabs of 128 bytes of k per row (64 bf16 or 32 fp32) go global -> LDS with
//   global_load_lds_dwordx4 into a ring of NS slabs of both operands, NS - 1 of
//   them in flight; one block barrier per slab.  The other blocks of the
//   compute unit fill the matrix pipe over a block's barriers, its first slabs
//   and its epilogue, so nothing is pipelined across tiles.
// * K-contiguous operands (element (r, k) at p[r * ld + k]) are stored as
//   [R][128 B], the 16-byte chunk index XOR-swizzled by (r >> 1) & 7: sixteen
//   consecutive rows read at one logical chunk cover the 64 banks once.  A DMA
//   instruction moves whole 128-byte lines of 8 rows.
// * MN-contiguous operands (element (r, k) at p[k * ld + r]) are stored as
//   R / 32 column blocks of k-rows.  bf16: [64 k][32 r], read with
//   ds_read_b64_tr_b16.  fp32: [32 k][32 r], k-rows of each group of 8 in the
//   order 0 4 1 5 2 6 3 7, so that the two halves of a wave (k and k + 4) read
//   the two halves of the banks.
// * An operand may interleave two matrices in 32-row blocks (gate and up), and
//   two products may be summed as one k loop (the slabs of the second pair
//   follow those of the first: dX = dA_g W_gate + dA_u W_up).
// * Rows past the operand's extent read a clamped (valid) address and feed
//   outputs that are never stored; k past K is clamped too and both operands'
//   slabs are zeroed there before they are read.
#pragma once

#include "gemm_bf16.hpp"

namespace fm {

// WM x WN x WK waves that multiply (WK: the waves that split each slab's k;
// where they are fewer than four, the others only move data), NS slabs in the
// ring, BPC blocks per compute unit (what the ring leaves room for).
// BE: bytes per B element, sizeof(T) or 1 (int8 codes widened exactly to bf16 as
// fragments are read; K-contiguous, 64-byte slab rows).
// KR: bytes of k per slab row, 128 or 64.
template <typename T_, int RA_, int RB_, int WM_, int WN_, int WK_, int NS_, int BPC_, int BE_ = (int)sizeof(T_),
          int KR_ = 128>
struct TileCfg {
  typedef T_ T;
  typedef std::conditional_t<BE_ == 1, int8_t, T_> TB;
  static constexpr int RA = RA_, RB = RB_, WM = WM_, WN = WN_, WK = WK_, NS = NS_, BPC = BPC_, BE = BE_, KR = KR_;
  static constexpr int THREADS = 256;
  static constexpr int V = 16 / (int)sizeof(T);       // elements per 16 bytes
  static constexpr int BK = KR / (int)sizeof(T);      // k per slab
  static constexpr int KS = KR / 32;                  // MFMA steps per slab
  static constexpr int TM = RA / WM, TN = RB / WN;    // wave sub-tile
  static constexpr int MI = TM / 32, NJ = TN / 32;    // MFMA tiles per wave
  static constexpr int A_BYTES = RA * KR, SLAB = A_BYTES + RB * BK * BE;
  static constexpr int A_INS = A_BYTES / 4096, B_INS = RB * BK * BE / 4096;   // DMA instructions per wave and slab
  static constexpr int INS = A_INS + B_INS;
  static constexpr int LDS = NS * SLAB;
  static constexpr int MW = WM * WN * WK;             // waves that multiply
  static_assert((MW == 4 || (MW == 2 && WK == 1)) && TM % 32 == 0 && TN % 32 == 0, "4 waves of 32-multiples");
  static_assert(WK == 1 || sizeof(T) == 4, "bf16 sums run over ascending k");
  static_assert(NS >= 2 && BPC * (LDS + 6 * 1024) <= 160 * 1024 + 5 * 1024 && (NS - 2) * INS < 64, "ring");
  static_assert(KR == 128 || (KR == 64 && sizeof(T) == 2 && BE == 2), "slab rows");
  static_assert(WK == 1 || (WK - 1) * RA * RB * 4 <= LDS, "partial sums");
};

// One operand, relative to the tile origin.  p2: the second matrix of an
// interleaved pair (blocks of 32 logical rows alternate); pk: the matrix of the
// second product of a two-product loop.  rows = valid physical rows.
template <typename T> struct TileSrc {
  const T* p;
  const T* p2;
  const T* pk;
  int ld;
  int rows;
};

template <typename T, bool KC, int R, bool INTER, int KR> struct TileDma {
  static constexpr int V = 16 / (int)sizeof(T), BK = KR / (int)sizeof(T);
  static constexpr int NI = R * KR / 4096;   // instructions per wave and slab
  static constexpr int RPI = 1024 / KR;      // rows per instruction (KC)
  static constexpr int CPR = KR / 16;        // chunks per row (KC)
  static constexpr int CB = R / 32;      // column blocks (MN)
  static constexpr int NB = INTER ? NI : 1;
  uint32_t off[NI];
  uintptr_t base[NB];   // uniform: the matrix of each instruction at the next slab
  uintptr_t step;
  int ins0;             // this wave's first instruction

  __device__ __forceinline__ static int block_of(int ins) { return KC ? ins * RPI / 32 : ins % CB; }   // 32-row block
  __device__ __forceinline__ static int lds_at(int ins) {
    return KC ? ins * 1024 : (ins % CB) * (32 * KR) + (ins / CB) * 1024;
  }
  // Chunk swizzle of a K-contiguous row.
  __device__ __forceinline__ static int swz(int r) { return KR == 128 ? (r >> 1) & 7 : (r >> 2) & 3; }
  // Byte offset (from the matrix of the instruction's block at the slab's first
  // k) of this lane's 16 bytes; kv = valid k from there on.
  __device__ __forceinline__ static uint32_t lane_off(const TileSrc<T>& s, int ins, int lane, int kv) {
    if (KC) {
      const int r = RPI * ins + lane / CPR;
      const int k = V * (lane % CPR ^ swz(r));
      const int pr = INTER ? 32 * (r >> 6) + (r & 31) : r;
      return (uint32_t)(((size_t)min(pr, s.rows - 1) * s.ld + min(k, kv - V)) * sizeof(T));
    }
    const int blk = ins % CB, kg = ins / CB;
    const int r0 = 32 * (INTER ? blk >> 1 : blk);
    int k, r;
    if (sizeof(T) == 2) {
      k = 16 * kg + (lane >> 2);
      r = r0 + 8 * (lane & 3);
    } else {
      k = 8 * kg + ((lane >> 4) & 3) + 4 * ((lane >> 3) & 1);
      r = r0 + 4 * (lane & 7);
    }
    return (uint32_t)(((size_t)min(k, kv - 1) * s.ld + min(r, s.rows - V)) * sizeof(T));
  }
  __device__ __forceinline__ void rebase(const TileSrc<T>& s, bool second) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      base[u] = (uintptr_t)(second ? s.pk : s.p);
      if (INTER) base[u] += (block_of(ins0 + u) & 1) ? (uintptr_t)s.p2 - (uintptr_t)s.p : 0;
    }
  }
  __device__ __forceinline__ void init(const TileSrc<T>& s) {
    const int lane = lane_id();
    ins0 = wave_id() * NI;
    step = KC ? KR : (uintptr_t)BK * s.ld * sizeof(T);
#pragma unroll
    for (int u = 0; u < NI; ++u) off[u] = lane_off(s, ins0 + u, lane, BK);
    rebase(s, false);
  }
  // Issues the next slab, kv valid k, and advances.
  __device__ __forceinline__ void issue(const TileSrc<T>& s, int kv, FM_LDS char* tile) {
    if (kv >= BK) {
#pragma unroll
      for (int u = 0; u < NI; ++u) dma16s((const void*)base[INTER ? u : 0], off[u], tile + lds_at(ins0 + u));
    } else {
      const int lane = lane_id_here();
#pragma unroll
      for (int u = 0; u < NI; ++u)
        dma16s((const void*)base[INTER ? u : 0], lane_off(s, ins0 + u, lane, kv), tile + lds_at(ins0 + u));
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) base[u] += step;
  }
  // Zeroes the slab's k >= kv in LDS (the block's 256 threads; after the slab has landed).
  __device__ __forceinline__ static void zero_tail(int kv, FM_LDS char* tile) {
    for (int c = threadIdx.x; c < R * CPR; c += 256) {   // 16-byte chunks
      int k;
      if (KC) k = V * (c % CPR ^ swz(c / CPR));
      else if (sizeof(T) == 2) k = (c >> 2) % BK;      // 64-byte k-rows
      else k = 8 * ((c >> 6) & 3) + ((c >> 4) & 3) + 4 * ((c >> 3) & 1);   // 128-byte k-rows, permuted in groups of 8
      if (k >= kv) *(FM_LDS u32x4_t*)(tile + 16 * c) = u32x4_t{0, 0, 0, 0};
    }
  }
};

// The same for int8 codes, K-contiguous: slab rows of 64 bytes, the 16-byte chunk
// index XOR-swizzled by (r >> 2) & 3 (as I8Frag reads them), an instruction 16
// rows.  The pointers and ld of the operand count bytes.
template <int R, bool INTER> struct TileDmaI8 {
  static constexpr int BK = 64;
  static constexpr int NI = R / 64;      // instructions per wave and slab
  static constexpr int NB = INTER ? NI : 1;
  uint32_t off[NI];
  uintptr_t base[NB];
  int ins0;

  __device__ __forceinline__ static uint32_t lane_off(const TileSrc<int8_t>& s, int ins, int lane, int kv) {
    const int r = 16 * ins + (lane >> 2);
    const int k = 16 * ((lane & 3) ^ swz_kc(r));
    const int pr = INTER ? 32 * (r >> 6) + (r & 31) : r;
    return (uint32_t)((size_t)min(pr, s.rows - 1) * s.ld + min(k, kv - 16));   // kv is a multiple of 16
  }
  __device__ __forceinline__ void rebase(const TileSrc<int8_t>& s, bool) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      base[u] = (uintptr_t)s.p;
      if (INTER) base[u] += ((ins0 + u) >> 1) & 1 ? (uintptr_t)s.p2 - (uintptr_t)s.p : 0;
    }
  }
  __device__ __forceinline__ void init(const TileSrc<int8_t>& s) {
    const int lane = lane_id();
    ins0 = wave_id() * NI;
#pragma unroll
    for (int u = 0; u < NI; ++u) off[u] = lane_off(s, ins0 + u, lane, BK);
    rebase(s, false);
  }
  __device__ __forceinline__ void issue(const TileSrc<int8_t>& s, int kv, FM_LDS char* tile) {
    const int lane = lane_id_here();
#pragma unroll
    for (int u = 0; u < NI; ++u)
      dma16s((const void*)base[INTER ? u : 0], kv >= BK ? off[u] : lane_off(s, ins0 + u, lane, kv),
             tile + (ins0 + u) * 1024);
#pragma unroll
    for (int u = 0; u < NB; ++u) base[u] += 64;
  }
  __device__ __forceinline__ static void zero_tail(int kv, FM_LDS char* tile) {
    for (int c = threadIdx.x; c < R * 4; c += 256)
      if (16 * ((c & 3) ^ swz_kc(c >> 2)) >= kv) *(FM_LDS u32x4_t*)(tile + 16 * c) = u32x4_t{0, 0, 0, 0};
  }
};

template <typename T> struct tile_frag;
template <> struct tile_frag<bf16> { typedef bf16x8_t type; };
template <> struct tile_frag<float> { typedef f32x4_t type; };

// MFMA fragments: lane l holds row r0 + l % 32 and k KST * step +
// (KST / 2) (l / 32) + 0 .. KST / 2 - 1 (16 bytes) of each 32-row block.
template <typename T, bool KC, int R, int NB, int KR> struct TileFrag {
  typedef typename tile_frag<T>::type frag;
  uint32_t off[NB];

  __device__ __forceinline__ void init(int row0) {
    const int lane = lane_id();
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int r0 = row0 + 32 * i;
      if (KC) {
        const int r = r0 + (lane & 31);
        off[i] = (uint32_t)(r * KR + (((lane >> 5) ^ TileDma<T, KC, R, false, KR>::swz(r)) << 4));
      } else if (sizeof(T) == 2) {
        // as B16Frag: output lane i, element j of a 16-lane group comes from
        // the address of lane 4 j + i / 4, offset i % 4
        const int g = lane >> 4, L = lane & 15;
        off[i] = (uint32_t)((r0 >> 5) * (32 * KR) + (8 * (g >> 1) + (L >> 2)) * 64 + (16 * (g & 1) + 4 * (L & 3)) * 2);
      } else {
        off[i] = (uint32_t)((r0 >> 5) * 4096 + (lane >> 5) * 128 + (lane & 31) * 4);
      }
    }
  }
  __device__ __forceinline__ frag read(const FM_LDS char* tile, int i, int st) const {
    if constexpr (KC) {
      return __builtin_bit_cast(frag, *(const FM_LDS u32x4_t*)(tile + (off[i] ^ (uint32_t)(st << 5))));
    } else if constexpr (sizeof(T) == 2) {
      const FM_LDS char* p = tile + off[i] + st * 1024;
      const i16x4_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FM_LDS i16x4_t*)p);
      const i16x4_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FM_LDS i16x4_t*)(p + 4 * 64));
      const u32x2_t w0 = __builtin_bit_cast(u32x2_t, v0), w1 = __builtin_bit_cast(u32x2_t, v1);
      return __builtin_bit_cast(frag, u32x4_t{w0[0], w0[1], w1[0], w1[1]});
    } else {
      const FM_LDS char* p = tile + off[i] + st * 1024;
      frag f;
#pragma unroll
      for (int e = 0; e < 4; ++e) f[e] = *(const FM_LDS float*)(p + 256 * e);
      return f;
    }
  }
};

__device__ __forceinline__ f32x16_t tile_mma(bf16x8_t b, bf16x8_t a, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16_t tile_mma(f32x4_t b, f32x4_t a, f32x16_t c) {
#pragma unroll
  for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_32x32x2f32(b[i], a[i], c, 0, 0, 0);
  return c;
}

// The wave's LDS reads are done and the block meets.
__device__ __forceinline__ void tile_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// This wave's place among the waves that multiply, those with a place below MW.
// Blocks that share a compute unit (256 apart) take opposite pairs of waves, and so
// of SIMDs, when only two multiply.
template <class C> __device__ __forceinline__ int tile_wave() {
  return C::MW == 2 ? wave_id() ^ (2 * ((blockIdx.x >> 8) & 1)) : wave_id();
}
// First row / column of a wave's sub-tile.  With two waves along a side, blocks
// that share a compute unit (256 apart) swap them, so that the waves left idle
// by partial tiles are not all on the same SIMDs.
template <class C> __device__ __forceinline__ int tile_row0(int wave) {
  const int w = wave % C::WM;
  return (C::WM == 2 ? w ^ ((blockIdx.x >> 8) & 1) : w) * C::TM;
}
template <class C> __device__ __forceinline__ int tile_col0(int wave) {
  const int w = wave / C::WM % C::WN;
  return (C::WN == 2 ? w ^ ((blockIdx.x >> 9) & 1) : w) * C::TN;
}

// Waits until at most min(after, N) slabs of INS instructions are in flight.
template <int N, int INS> __device__ __forceinline__ void tile_wait(int after) {
  if constexpr (N == 0) {
    wait_vmcnt<0>();
  } else {
    if (after >= N) wait_vmcnt<N * INS>();
    else tile_wait<N - 1, INS>(after);
  }
}

// acc += A B^T over [0, K), K >= 1 (and over [0, K) of the second pair with TWO).
// The LDS must be free on entry and is free on return (a barrier ends the call).
// Slab kt has landed once at most the NS - 2 slabs issued after it are in
// flight; the barrier at the top of slab kt says that every wave has read slab
// kt - 1, whose buffer then takes slab kt + NS - 1.  A wave issues a slab's
// fragment reads, then the DMA of the coming slab (its address work
// covers the first reads' latency), then the MFMAs.  The partial last slab is
// zero-filled in LDS, so that one copy of the MFMA code serves all slabs.
template <class C, bool AKC, bool BKC, bool AI = false, bool BI = false, bool TWO = false>
__device__ __forceinline__ void tile_gemm(const TileSrc<typename C::T>& A, const TileSrc<typename C::TB>& B, int K,
                                          FM_LDS char* lds, B16Acc<C::MI, C::NJ>& acc) {
  typedef typename C::T T;
  constexpr bool I8 = C::BE == 1;
  static_assert(!I8 || (BKC && !TWO), "int8 B is K-contiguous, one product");
  typedef typename tile_frag<T>::type frag;
  const int n1 = (K + C::BK - 1) / C::BK;
  const int nk = TWO ? 2 * n1 : n1;
  const int wave = tile_wave<C>();
  TileDma<T, AKC, C::RA, AI, C::KR> da;
  std::conditional_t<I8, TileDmaI8<C::RB, BI>, TileDma<T, BKC, C::RB, BI, C::KR>> db;
  da.init(A);
  db.init(B);
  TileFrag<T, AKC, C::RA, C::MI, C::KR> fa;
  std::conditional_t<I8, I8Frag<C::RB, C::NJ>, TileFrag<T, BKC, C::RB, C::NJ, C::KR>> fb;
  const int row0 = tile_row0<C>(wave), col0 = tile_col0<C>(wave);
  fa.init(row0);
  fb.init(col0);
  // a wave whose rows or columns all lie past the operand multiplies nothing: it
  // runs the loop's DMA and barriers and leaves the matrix pipe to other blocks
  // (fp32, 75 rows per slot, d = 3480, I = 712: forward 1990 -> 1860 us, backward
  // 2655 -> 2555; a branch inside the slab loop instead cost full tiles 5-15 %)
  auto phys = [](int r, bool inter) { return inter ? 32 * (r >> 6) + (r & 31) : r; };
  const bool works = (C::MW == 4 || wave < C::MW) && phys(row0, AI) < A.rows && phys(col0, BI) < B.rows;
  constexpr int KW = C::KS / C::WK;   // steps per wave and slab
  // steps whose fragments are read ahead (all, where the registers allow)
  constexpr int SB = C::MI * C::NJ >= 8 && KW > 2 ? 2 : KW;
  const int st0 = wave / (C::WM * C::WN) * KW;
  auto issue = [&](int s, int buf) {
    if (TWO && s == n1) {
      da.rebase(A, true);
      db.rebase(B, true);
    }
    const int kv = K - (TWO && s >= n1 ? s - n1 : s) * C::BK;
    FM_LDS char* t = lds + buf * C::SLAB;
    da.issue(A, kv, t);
    db.issue(B, kv, t + C::A_BYTES);
  };
#pragma nounroll
  for (int s = 0; s < C::NS - 1 && s < nk; ++s) issue(s, s);
  auto loop = [&](auto mul) {
    constexpr bool MUL = decltype(mul)::value;
    int cur = 0, nxt = C::NS - 1;   // buffers of slab kt and of slab kt + NS - 1
#pragma nounroll
    for (int kt = 0; kt < nk; ++kt) {
      const int after = nk - 1 - kt;   // slabs after kt
      tile_wait<C::NS - 2, C::INS>(after);
      tile_barrier();
      FM_LDS char* const ta = lds + cur * C::SLAB;
      FM_LDS char* const tb = ta + C::A_BYTES;
      const int kv = K - (TWO && kt >= n1 ? kt - n1 : kt) * C::BK;
      if (kv < C::BK) {
        da.zero_tail(kv, ta);
        db.zero_tail(kv, tb);
        tile_barrier();
      }
      // int8 codes are widened next to their MFMAs
      typedef std::conditional_t<I8, u32x2_t, frag> bfrag;
      frag xa[SB][C::MI];
      bfrag xb[SB][C::NJ];
      auto read = [&](int st) {
#pragma unroll
        for (int i = 0; i < C::MI; ++i) xa[st % SB][i] = fa.read(ta, i, st0 + st);
#pragma unroll
        for (int j = 0; j < C::NJ; ++j) {
          if constexpr (I8) xb[st % SB][j] = fb.codes(tb, j, st0 + st);
          else xb[st % SB][j] = fb.read(tb, j, st0 + st);
        }
      };
      if constexpr (MUL) {
#pragma unroll
        for (int st = 0; st < SB; ++st) read(st);
      }
      sched_fence();
      if (kt + C::NS - 1 < nk) issue(kt + C::NS - 1, nxt);
      sched_fence();
      if constexpr (MUL) {
#pragma unroll
        for (int st = 0; st < KW; ++st) {
#pragma unroll
          for (int j = 0; j < C::NJ; ++j) {
            frag b;
            if constexpr (I8) b = widen_i8x8(xb[st % SB][j]);
            else b = xb[st % SB][j];
#pragma unroll
            for (int i = 0; i < C::MI; ++i) acc.v[i][j] = tile_mma(b, xa[st % SB][i], acc.v[i][j]);
          }
          if (st + SB < KW) read(st + SB);
        }
      }
      cur = cur + 1 == C::NS ? 0 : cur + 1;
      nxt = nxt + 1 == C::NS ? 0 : nxt + 1;
    }
  };
  if (works) loop(std::true_type{});
  else loop(std::false_type{});
  tile_barrier();
  if (C::WK > 1) {
    // wave wk > 0 leaves its sums at [wk - 1][wave of the WM x WN grid][tile][quad][lane]
    const int w = wave % (C::WM * C::WN), wk = wave / (C::WM * C::WN);
    const int lane = lane_id_here();
    auto at = [&](int k, int i, int j, int q) {
      return lds + (((((k - 1) * C::WM * C::WN + w) * C::MI + i) * C::NJ + j) * 4 + q) * 1024 + lane * 16;
    };
    if (wk > 0) {
#pragma unroll
      for (int i = 0; i < C::MI; ++i)
#pragma unroll
        for (int j = 0; j < C::NJ; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) *(FM_LDS f32x4_t*)at(wk, i, j, q) = acc.quad(i, j, q);
    }
    tile_barrier();
    if (wk == 0) {
      for (int k = 1; k < C::WK; ++k)
#pragma unroll
        for (int i = 0; i < C::MI; ++i)
#pragma unroll
          for (int j = 0; j < C::NJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const f32x4_t v = *(const FM_LDS f32x4_t*)at(k, i, j, q);
#pragma unroll
              for (int e = 0; e < 4; ++e) acc.v[i][j][4 * q + e] += v[e];
            }
    }
    tile_barrier();
  }
}

}  // namespace fm
