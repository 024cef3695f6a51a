// Batched strided GEMM on CDNA4 matrix cores (FP64 and FP32 MFMA).
//
// Every contraction of the density-fitted sigma product (first-order Coulomb and
// exchange terms, the second-order amplitude strips and the amplitude-weighted
// ladder/ring contractions) and of the subspace solver is expressed as one
// GemmDesc; this file owns the only dense-contraction kernel of the library.
//
// Design (gfx950):
//  * 256 threads = 4 wave64, arranged 2x2; each wave owns a (BM/2)x(BN/2) block of
//    C made of 16x16 MFMA tiles (v_mfma_f64_16x16x4f64 / v_mfma_f32_16x16x4f32).
//  * A and B tiles (BK deep) go through two LDS buffers, with one barrier per BK step
//    that stands before the step's last quarter.  FP64 operands contiguous along k (and
//    split-BF16 ones) are loaded straight into LDS, the other layouts through registers
//    that hold the next tile; either way a load has a whole tile's time to arrive.
//  * Workgroup ids are remapped so that the tiles an XCD runs are contiguous in a
//    grouped (row-band) order: tiles sharing A rows or B columns hit the same L2.
//  * Split-K (over the flattened outer x inner reduction) writes per-split partial
//    tiles to a caller workspace; a second kernel sums them in split order, so the
//    result is deterministic and independent of the launch shape of other work.
#include "common.h"

#include <algorithm>
#include <type_traits>
#include <vector>

namespace ppw {
namespace {

template <typename T>
struct Mfma;

// Operand layout (both types): lane l supplies A[l%16][l/16] and B[l/16][l%16].
// Result layout (measured on gfx950): FP64 lane l, register r holds D[l/16 + 4r][l%16];
// FP32 lane l, register r holds D[4(l/16) + r][l%16].
template <>
struct Mfma<double> {
  typedef double acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};

template <>
struct Mfma<float> {
  typedef float acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

constexpr int kThreads = 256;

// XCD-aware remap of a flattened workgroup id: the hardware dispatches consecutive
// ids round-robin over the 8 XCDs, so id -> (id % 8) * per + id / 8 gives each XCD a
// contiguous range of (batch, tile) work that shares operands in its own L2.
__device__ __forceinline__ long xcd_remap(long bid, long total) {
  const long per = total / 8;
  if (per > 0 && bid < per * 8) return (bid % 8) * per + bid / 8;
  return bid;
}

__device__ __forceinline__ void tile_coords(int id, int tiles_m, int tiles_n, int& tm, int& tn) {
  // grouped ordering: bands of GROUP tile-rows walked column by column
  constexpr int GROUP = 8;
  const int in_group = GROUP * tiles_n;
  const int g = id / in_group;
  const int first_m = g * GROUP;
  const int gsize = min(tiles_m - first_m, GROUP);
  const int r = id % in_group;
  tm = first_m + r % gsize;
  tn = r / gsize;
}

// Tiles of a product whose columns d.sym .. d.sym + M - 1 form a symmetric block with its rows
// (GemmDesc): in the grouped order, without the columns of a band of 8 tile rows that lie below
// the block's diagonal for all of them.  Works for host and device.
constexpr int kBand = 8;
__host__ __device__ inline int sym_excluded(const GemmDesc& d, int m0, int BN, int& lo) {
  lo = (int)((d.sym + BN - 1) / BN);
  const int hi = (int)((d.sym + m0) / BN);
  return hi > lo ? hi - lo : 0;
}
__device__ __forceinline__ bool sym_tile_coords(const GemmDesc& d, long id, int BM, int BN, int tiles_m, int tiles_n,
                                                int& tm, int& tn) {
  for (int first = 0; first < tiles_m; first += kBand) {
    const int gsize = min(tiles_m - first, kBand);
    int lo;
    const int ex = sym_excluded(d, first * BM, BN, lo);
    const long cnt = (long)gsize * (tiles_n - ex);
    if (id < cnt) {
      tm = first + (int)(id % gsize);
      tn = (int)(id / gsize);
      if (tn >= lo) tn += ex;
      // a tile of the band that is below the diagonal for its own rows
      return !((long)tn * BN >= d.sym && (long)tn * BN + BN <= d.sym + (long)tm * BM);
    }
    id -= cnt;
  }
  return false;
}
template <int BM, int BN>
long sym_tiles(const GemmDesc& d) {
  const int tiles_m = (d.M + BM - 1) / BM, tiles_n = (d.N + BN - 1) / BN;
  long n = 0;
  for (int first = 0; first < tiles_m; first += kBand) {
    int lo;
    n += (long)std::min(tiles_m - first, kBand) * (tiles_n - sym_excluded(d, first * BM, BN, lo));
  }
  return n;
}

// ---------------------------------------------------------------------------
// FP64 tiles with both operands contiguous along k (the amplitude contraction and its
// grouped launches): operand tiles go from global memory straight into LDS
// (global_load_lds_dwordx4: lane l of a wave writes 16 B at the wave's LDS base + 16 l),
// so no registers hold the next tile and no LDS stores are issued.  A tile row of BK = 16
// doubles is 8 slots of 16 B; (row r, pair kp) lives in slot r * 8 + (kp ^ ((r >> 1) & 7)),
// which puts the 16 rows of an MFMA fragment read in 16 different 16-byte bank groups.
// Lanes choose their source element so that each wave's 64 slots (8 rows) are filled in
// one instruction.  Rows past an edge in m or n repeat the last one (their results are not
// stored); in a ragged k tile the pairs past K repeat the last one and are overwritten by zeros
// once they have landed.  Operands whose rows are not all 16-byte aligned, or of an odd K, go
// through registers into the same layout.  Measured, with element-wise guarded loads of every k
// tile as soon as M, N or K was not a multiple of 8, 8 or 16 | here: 672 x 499100 over 434 8107 |
// 5351 us, 2250 x 1320 over 2250 463 | 289, 5889 x 3760 over 5889 (odd rows) 7381 | 4611; a launch
// of whole tiles is as fast as before (6400 x 7200 over 6400 9.3 ms).  The two LDS buffers are separate
// arrays and the loop is unrolled by two, so a buffer being filled and the buffer being
// read are distinct objects to the compiler.  MFMA operands and their order are those of
// the register-staged path, so results are bit-identical to it.
// x, as a value that the compiler cannot know: what depends on it is worked out where it is used and
// not held in registers through the loops before
__device__ __forceinline__ int hidden(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ int swz16(int r, int kp) { return r * 8 + (kp ^ ((r >> 1) & 7)); }

// Offset of index x along a C dimension that may be a pair (x / R, x % R) with strides
// (S, unit); R = 0 gives x * unit.  The quotient comes from a double product and one
// correction, exact for every int x.
__device__ __forceinline__ long c_index(int x, int R, long S, long unit) {
  if (R == 0) return (long)x * unit;
  int q = (int)((double)x * (1.0 / (double)R));
  int r = x - q * R;
  if (r < 0) {
    --q;
    r += R;
  } else if (r >= R) {
    ++q;
    r -= R;
  }
  return (long)q * S + (long)r * unit;
}

// Epilogue of a tile whose C rows or columns are mapped (no split-K workspace): column
// offsets once per thread, row offsets once per accumulator row.
template <typename T, typename Acc, int TM, int TN, int WTM, int WTN>
__device__ __forceinline__ void store_mapped(const GemmDesc& d, T alpha, T beta, T* __restrict__ Cb, int m0, int n0,
                                             int wm, int wn, int lane, const Acc (&acc)[TM][TN]) {
  long coff[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = n0 + wn * WTN + j * 16 + (lane & 15);
    coff[j] = col < d.N ? c_index(col + d.cBn, d.cRn, d.cSn, 1) : -1;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = m0 + wm * WTM + i * 16 + Mfma<T>::row(lane, r);
      if (row >= d.M) continue;
      const long ro = c_index(row, d.cRm, d.cSm, d.ldc);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (coff[j] < 0) continue;
        T* cp = Cb + ro + coff[j];
        T out = alpha * acc[i][j][r];
        if (beta != T(0)) out += beta * (*cp);
        *cp = out;
      }
    }
}

// STREAM (whole tiles in m, n in steps of 8 and in k in steps of 32, one batch, no splits): the
// workgroup computes 'count' tiles, flat, flat + stride, ..., and loads the first k tiles of the
// next one during the last ones of the present.
constexpr long kDmaRow = 1L << 26;  // 7 rows of it and a k tile lie within 4 GiB
template <int BM, int BN, bool STREAM = false>
__device__ __forceinline__ void gemm_tile_dma(const GemmDesc& d, double alpha, const double* __restrict__ A,
                                              const double* __restrict__ B, double beta, double* __restrict__ C,
                                              double* __restrict__ W, int splitk, long flat, int split,
                                              int count = 1, int stride = 0) {
  constexpr int BK = 16;
  using acc_t = Mfma<double>::acc_t;
  constexpr int WTM = BM / 2, WTN = BN / 2;
  constexpr int TM = WTM / 16, TN = WTN / 16;
  constexpr int SA = BM * BK, SB = BN * BK;
  constexpr int CA = BM / 32, CB = BN / 32;  // 1 KB chunks per wave (4 waves, 8 rows a chunk)
  __shared__ __attribute__((aligned(16))) double As0[SA];
  __shared__ __attribute__((aligned(16))) double As1[SA];
  __shared__ __attribute__((aligned(16))) double Bs0[SB];
  __shared__ __attribute__((aligned(16))) double Bs1[SB];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int tiles_m = (d.M + BM - 1) / BM;
  const int tiles_n = (d.N + BN - 1) / BN;
  const long ntiles = (long)tiles_m * tiles_n;
  const int batch = (int)(flat / ntiles);
  int tm, tn;
  tile_coords((int)(flat % ntiles), tiles_m, tiles_n, tm, tn);
  int m0 = tm * BM, n0 = tn * BN;
  const int b1 = batch / d.nb2, b2 = batch % d.nb2;
  const double* Atile = A + b1 * d.sA1 + b2 * d.sA2 + (long)m0 * d.lda;
  const double* Btile = B + b1 * d.sB1 + b2 * d.sB2 + (long)n0 * d.ldb;
  const int nkt = (d.K + BK - 1) / BK;
  const long total = (long)d.KB * nkt;
  const long chunk = (total + splitk - 1) / splitk;
  const long it0 = (long)split * chunk;
  const long it1 = min(total, it0 + chunk);
  const int lda32 = (int)d.lda, ldb32 = (int)d.ldb;
  const int mrem = d.M - m0, nrem = d.N - n0;
  // A chunk is 8 rows, (wave + 4 c) 8 on; chunks past the edge repeat the last one and rows past it
  // within a chunk the last row.  The first row of a chunk is the same for the whole wave, and the
  // lanes' offsets from it are those of every chunk but the one at an edge, so that a load takes its
  // address from scalar registers and one vector register (32-bit byte offsets: longer rows go through
  // registers).
  const bool dma = (d.lda % 2) == 0 && (d.ldb % 2) == 0 && (d.sAk % 2) == 0 && (d.sBk % 2) == 0 &&
                   ((uintptr_t)Atile % 16) == 0 && ((uintptr_t)Btile % 16) == 0 && d.K % 2 == 0 &&
                   d.lda < kDmaRow && d.ldb < kDmaRow;
  const int kpl = (lane & 7) ^ (4 * (wave & 1) + (lane >> 4));
  long rowA[CA], rowB[CB];
  unsigned laneA[CA], laneB[CB];
  auto chunk_rows = [&](int mr, int nr) {
    // (a stream's edges lie between chunks)
    const int ma = (mr - 1) & ~7, nb = (nr - 1) & ~7;
    const int la = lane >> 3, ea = STREAM ? la : min(la, (mr - 1) & 7), eb = STREAM ? la : min(la, (nr - 1) & 7);
#pragma unroll
    for (int c = 0; c < CA; ++c) {
      const int r = (wave + 4 * c) * 8;
      rowA[c] = (long)min(r, ma) * d.lda;
      laneA[c] = 8u * ((unsigned)(r < ma ? la : ea) * (unsigned)lda32 + 2u * kpl);
    }
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int r = (wave + 4 * c) * 8;
      rowB[c] = (long)min(r, nb) * d.ldb;
      laneB[c] = 8u * ((unsigned)(r < nb ? la : eb) * (unsigned)ldb32 + 2u * kpl);
    }
  };
  chunk_rows(mrem, nrem);
  // the pairs of the ragged k tile that lie past K: how far back (bytes) the last one is from this lane's
  const int kpast = kpl - ((d.K % BK) / 2 - 1);
  const unsigned back = kpast > 0 ? 16u * kpast : 0u;
  // k tile (kb, kt) straight into buffer (Ab, Bb)
  auto fill = [&](double* Ab, double* Bb, int kb, int kt, auto rag) {
    const double* Ak = Atile + kb * d.sAk + kt * BK;
    const double* Bk = Btile + kb * d.sBk + kt * BK;
    const unsigned off = decltype(rag)::value && kt + 1 == nkt ? back : 0u;
#pragma unroll
    for (int c = 0; c < CA; ++c)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)((const char*)(Ak + rowA[c]) + (laneA[c] - off)),
          (__attribute__((address_space(3))) void*)(Ab + (wave + 4 * c) * 128), 16, 0, 0);
#pragma unroll
    for (int c = 0; c < CB; ++c)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)((const char*)(Bk + rowB[c]) + (laneB[c] - off)),
          (__attribute__((address_space(3))) void*)(Bb + (wave + 4 * c) * 128), 16, 0, 0);
  };
  // zeros past K in a ragged tile: the slots that this lane's own loads (landed) filled
  typedef double pair_t __attribute__((ext_vector_type(2)));
  auto cut = [&](double* Ab, double* Bb) {
    if (kpast <= 0) return;
#pragma unroll
    for (int c = 0; c < CA; ++c) *reinterpret_cast<pair_t*>(Ab + (wave + 4 * c) * 128 + 2 * lane) = pair_t{0.0, 0.0};
#pragma unroll
    for (int c = 0; c < CB; ++c) *reinterpret_cast<pair_t*>(Bb + (wave + 4 * c) * 128 + 2 * lane) = pair_t{0.0, 0.0};
  };
  // k tile (kb, kt) through registers: pairs of row r0 + 32 i from element 2 kp on.  A pair past the
  // end of K is read from the last two values of its row (never past them; K is 2 at least) and put
  // right, with zeros past K, when it is stored.  Offsets are worked out anew for every tile: the
  // accumulators need the registers.
  typedef double pair8_t __attribute__((ext_vector_type(2), aligned(8)));
  pair_t sa[CA], sb[CB];
  auto load_regs = [&](int kb, int kt) {
    const double* Ak = Atile + kb * d.sAk + kt * BK;
    const double* Bk = Btile + kb * d.sBk + kt * BK;
    const int id = hidden(tid), r0 = id >> 3, kc = min(2 * (id & 7), d.K - kt * BK - 2);
#pragma unroll
    for (int i = 0; i < CA; ++i)
      sa[i] = *reinterpret_cast<const pair8_t*>(Ak + (min(r0 + 32 * i, mrem - 1) * lda32 + kc));
#pragma unroll
    for (int i = 0; i < CB; ++i)
      sb[i] = *reinterpret_cast<const pair8_t*>(Bk + (min(r0 + 32 * i, nrem - 1) * ldb32 + kc));
  };
  auto store_regs = [&](double* Ab, double* Bb, int kt) {
    const int id = hidden(tid), r0 = id >> 3, kp = id & 7;
    const int left = d.K - kt * BK - 2 * kp;  // values of K from the pair's first on
    auto put = [&](double* p, pair_t v) {
      *reinterpret_cast<pair_t*>(p) = pair_t{left >= 2 ? v[0] : (left == 1 ? v[1] : 0.0), left >= 2 ? v[1] : 0.0};
    };
#pragma unroll
    for (int i = 0; i < CA; ++i) put(Ab + 2 * swz16(r0 + 32 * i, kp), sa[i]);
#pragma unroll
    for (int i = 0; i < CB; ++i) put(Bb + 2 * swz16(r0 + 32 * i, kp), sb[i]);
  };

  acc_t acc[TM][TN];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
  };
  clear();
  auto frag = [&](const double* Ab, const double* Bb, int kk, double (&a)[TM], double (&b)[TN]) {
    const int kr = kk + (lane >> 4);
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = Ab[2 * swz16(wm * WTM + i * 16 + (lane & 15), kr >> 1) + (kr & 1)];
#pragma unroll
    for (int j = 0; j < TN; ++j) b[j] = Bb[2 * swz16(wn * WTN + j * 16 + (lane & 15), kr >> 1) + (kr & 1)];
  };
  auto mma = [&](const double (&a)[TM], const double (&b)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = Mfma<double>::mma(a[i], b[j], acc[i][j]);
  };

  auto finish = [&]() {
    const long nbatch = (long)d.nb1 * d.nb2;
    if (!W && (d.cRm | d.cRn)) {
      store_mapped<double, acc_t, TM, TN, WTM, WTN>(d, alpha, beta, C + b1 * d.sC1 + b2 * d.sC2, m0, n0, wm, wn, lane,
                                                   acc);
      return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = m0 + wm * WTM + i * 16 + Mfma<double>::row(lane, r);
          const int col = n0 + wn * WTN + j * 16 + (lane & 15);
          if (row < d.M && col < d.N) {
            const double v = acc[i][j][r];
            if (W) {
              W[((long)split * nbatch + batch) * ((long)d.M * d.N) + (long)row * d.N + col] = v;
            } else {
              double* cp = C + b1 * d.sC1 + b2 * d.sC2 + (long)row * d.ldc + col;
              double out = alpha * v;
              if (beta != 0.0) out += beta * (*cp);
              *cp = out;
            }
          }
        }
  };
  // issue order pinned: one k group's MFMAs with the next group's fragment reads, and the loads of
  // a tile where there are any, between them
  auto interleave = [&](auto loads) {
    constexpr int R = TM + TN, L = decltype(loads)::value ? CA + CB : 0;
    static_assert(TM * TN >= R && TM * TN >= L, "one read and one load per MFMA");
#pragma unroll
    for (int r = 0; r < TM * TN; ++r) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (r < R) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (r < L) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
    }
  };
  // The one barrier of a k tile stands before its last k group, whose fragments are in registers
  // by then: the next tile has landed (its loads were issued a whole tile earlier), the buffer
  // just read is refilled, and the next tile's first fragments are read during that group's
  // MFMAs.  The loads go out one per MFMA and take their addresses from scalar registers: eight in
  // a row, with 64-bit vector adds before each, hold a wave up for 500 cycles with the matrix
  // core idle (the same loop with both operands in LDS runs at 77 TF/s).  Measured at
  // 6400 x 14336 x 6400: 68.5 TF/s with the barrier at the end of the tile, 69.7 with it here,
  // 72.4 with the loads spread (the library's product: 71.1); matrix units busy 88 -> 93 %.
  constexpr int kWaitAll = 0x0F70;  // vmcnt(0): this wave's loads into LDS have landed
  const int steps = (int)(it1 - it0);
  // the k tile to load next; past the end the last one again, so that no load stands behind a branch,
  // which would keep the MFMAs from hiding its issue (what it brings is not used)
  int kb = (int)(it0 / nkt), kt = (int)(it0 % nkt);
  int ahead = 0;  // tile last loaded (STREAM: output tile whose operands are loaded)
  auto advance = [&]() {
    if constexpr (STREAM) {
      if (kt + 1 < nkt) {
        ++kt;
      } else if (ahead + 1 < count) {
        ++ahead;
        kt = 0;
        tile_coords((int)flat + ahead * stride, tiles_m, tiles_n, tm, tn);
        Atile = A + (long)tm * BM * d.lda;
        Btile = B + (long)tn * BN * d.ldb;
        chunk_rows(d.M - tm * BM, d.N - tn * BN);
      }
    } else {
      const bool more = ahead + 1 < steps, wrap = more && kt + 1 == nkt;
      ahead += more ? 1 : 0;
      kt = wrap ? 0 : kt + (more ? 1 : 0);
      kb += wrap ? 1 : 0;
    }
  };
  double a0[TM], b0[TN], a1[TM], b1v[TN];
  // straight into LDS (rag: the last k tile of each outer block is ragged)
  auto reduce = [&](auto rag) {
    // a tile that has landed, behind the barrier: ragged, it is cut, and the barrier waited for again
    auto landed = [&](double* Ab, double* Bb) {
      if constexpr (decltype(rag)::value) {
        if (kt + 1 == nkt) {
          cut(Ab, Bb);
          __syncthreads();
        }
      }
    };
    fill(As0, Bs0, kb, kt, rag);
    __builtin_amdgcn_s_waitcnt(kWaitAll);
    __syncthreads();
    landed(As0, Bs0);
    advance();
    if (STREAM || steps > 1) fill(As1, Bs1, kb, kt, rag);
    frag(As0, Bs0, 0, a0, b0);
    auto step = [&](double* Ac, double* Bc, double* An, double* Bn) {
      frag(Ac, Bc, 4, a1, b1v);
      mma(a0, b0);
      interleave(std::false_type{});
      frag(Ac, Bc, 8, a0, b0);
      mma(a1, b1v);
      interleave(std::false_type{});
      frag(Ac, Bc, 12, a1, b1v);
      mma(a0, b0);
      interleave(std::false_type{});
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(kWaitAll);
      __syncthreads();
      landed(An, Bn);
      advance();
      fill(Ac, Bc, kb, kt, rag);
      frag(An, Bn, 0, a0, b0);
      mma(a1, b1v);
      interleave(std::true_type{});
      __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (STREAM) {
      for (int i = 0;;) {
        for (int t = 0; t < nkt; t += 2) {
          step(As0, Bs0, As1, Bs1);
          step(As1, Bs1, As0, Bs0);
        }
        if (++i == count) break;
        finish();
        m0 = tm * BM;
        n0 = tn * BN;
        clear();
      }
    } else {
      for (int t = 0; t < steps; t += 2) {
        step(As0, Bs0, As1, Bs1);
        if (t + 1 < steps) step(As1, Bs1, As0, Bs0);
      }
    }
    __builtin_amdgcn_s_waitcnt(kWaitAll);  // no load may outlive the workgroup's LDS
  };
  // through registers, which go to the free buffer during the first k group and take the next tile
  // during the second
  auto reduce_regs = [&]() {
    load_regs(kb, kt);
    store_regs(As0, Bs0, kt);
    if (steps > 1) {
      advance();
      load_regs(kb, kt);
    }
    __syncthreads();
    frag(As0, Bs0, 0, a0, b0);
    auto step = [&](const double* Ac, const double* Bc, double* An, double* Bn) {
      frag(Ac, Bc, 4, a1, b1v);
      store_regs(An, Bn, kt);
      mma(a0, b0);
      __builtin_amdgcn_sched_barrier(0);
      advance();
      frag(Ac, Bc, 8, a0, b0);
      load_regs(kb, kt);
      mma(a1, b1v);
      __builtin_amdgcn_sched_barrier(0);
      frag(Ac, Bc, 12, a1, b1v);
      mma(a0, b0);
      interleave(std::false_type{});
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
      frag(An, Bn, 0, a0, b0);
      mma(a1, b1v);
      interleave(std::false_type{});
      __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = 0; t < steps; t += 2) {
      step(As0, Bs0, As1, Bs1);
      if (t + 1 < steps) step(As1, Bs1, As0, Bs0);
    }
  };
  if constexpr (STREAM) {
    reduce(std::false_type{});
  } else if (steps > 0) {
    if (!dma)
      reduce_regs();
    else if (d.K % BK == 0)
      reduce(std::false_type{});
    else
      reduce(std::true_type{});
  }
  finish();
}

// LDS layouts (chosen per operand at compile time, FP64 64 banks x 4 B):
//  * operand contiguous along k in global memory (A: transA = 0, B: transB = 1):
//    tile stored [m][BK + 2]; a 16-lane group reads 16 rows at one k: bank offsets
//    36 i (+2 for the next k group) are distinct, and the global->LDS writes are
//    consecutive addresses.
//  * operand contiguous along m (or n): tile stored [k][BM + 16]; rows of 16 lanes
//    sit 32 banks apart, writes are consecutive.
// TAG only distinguishes kernel symbols (the amplitude contraction gets its own,
// so that profiles can attribute its time); the code is identical.
// One workgroup's tile of C (or, with W, of split 'split' of its reduction) for the
// flattened (batch, tile) index 'flat' of GEMM d.
// CPF (C prefetch): the C elements an accumulating tile (beta != 0, no split-K, plain
// C) will update are loaded before the reduction instead of after it, so their latency
// hides behind a short reduction; the arithmetic of the update is unchanged.
template <typename T, int BM, int BN, int BK, bool AK, bool BKC, bool CPF = false>
__device__ __forceinline__ void gemm_tile(const GemmDesc& d, T alpha, const T* __restrict__ A,
                                          const T* __restrict__ B, T beta, T* __restrict__ C, T* __restrict__ W,
                                          int splitk, long flat, int split) {
  if constexpr (std::is_same<T, double>::value && AK && BKC && BK == 16) {
    gemm_tile_dma<BM, BN>(d, alpha, A, B, beta, C, W, splitk, flat, split);
    return;
  }
  using acc_t = typename Mfma<T>::acc_t;
  constexpr bool SYM = !AK && !BKC && BM == 128;  // the strips' integrals (B^ov)^T B^ov
  constexpr int PK = 2;   // pad of k-contiguous tiles
  constexpr int PM = 16;  // pad of m/n-contiguous tiles
  constexpr int WTM = BM / 2, WTN = BN / 2;
  constexpr int TM = WTM / 16, TN = WTN / 16;
  constexpr int LA = BM * BK / kThreads, LB = BN * BK / kThreads;
  static_assert(LA * kThreads == BM * BK && LB * kThreads == BN * BK, "tile/thread mismatch");
  constexpr int SA = AK ? BM * (BK + PK) : BK * (BM + PM);
  constexpr int SB = BKC ? BN * (BK + PK) : BK * (BN + PM);
  __shared__ __attribute__((aligned(16))) T As[2][SA];
  __shared__ __attribute__((aligned(16))) T Bs[2][SB];
  typedef T pair_t __attribute__((ext_vector_type(2)));
  // element (m, k) of an LDS tile
  auto aidx = [](int m, int k) { return AK ? m * (BK + PK) + k : k * (BM + PM) + m; };
  auto bidx = [](int n, int k) { return BKC ? n * (BK + PK) + k : k * (BN + PM) + n; };

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  const int tiles_m = (d.M + BM - 1) / BM;
  const int tiles_n = (d.N + BN - 1) / BN;
  const long ntiles = (long)tiles_m * tiles_n;
  int batch = (int)(flat / ntiles);
  int tm, tn;
  if (SYM && d.sym >= 0) {
    batch = 0;
    if (!sym_tile_coords(d, flat, BM, BN, tiles_m, tiles_n, tm, tn)) return;
  } else {
    tile_coords((int)(flat % ntiles), tiles_m, tiles_n, tm, tn);
  }
  const int m0 = tm * BM, n0 = tn * BN;
  const int b1 = batch / d.nb2, b2 = batch % d.nb2;

  const T* Ab = A + b1 * d.sA1 + b2 * d.sA2;
  const T* Bb = B + b1 * d.sB1 + b2 * d.sB2;
  const int nkt = (d.K + BK - 1) / BK;
  const long total = (long)d.KB * nkt;
  const long chunk = (total + splitk - 1) / splitk;
  const long it0 = (long)split * chunk;
  const long it1 = min(total, it0 + chunk);

  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

  // Each thread moves pairs of elements that are adjacent along the contiguous
  // dimension of the operand: pair p = i * 256 + tid covers (m, k), (m, k + 1) of a
  // k-contiguous tile or (m, k), (m + 1, k) of an m-contiguous one.
  constexpr int PA = LA / 2, PB = LB / 2;
  static_assert(PA * 2 == LA && PB * 2 == LB, "pairs");
  auto a_pair = [](int p, int& m, int& k) {
    if (AK) { m = p / (BK / 2); k = 2 * (p % (BK / 2)); }
    else { m = 2 * (p % (BM / 2)); k = p / (BM / 2); }
  };
  auto b_pair = [](int p, int& n, int& k) {
    if (BKC) { n = p / (BK / 2); k = 2 * (p % (BK / 2)); }
    else { n = 2 * (p % (BN / 2)); k = p / (BN / 2); }
  };
  pair_t ra[PA], rb[PB];
  T cpre[CPF ? TM : 1][CPF ? TN : 1][4];
  if constexpr (CPF) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = m0 + wm * WTM + i * 16 + Mfma<T>::row(lane, r);
          const int col = n0 + wn * WTN + j * 16 + (lane & 15);
          cpre[i][j][r] = (row < d.M && col < d.N) ? C[b1 * d.sC1 + b2 * d.sC2 + (long)row * d.ldc + col] : T(0);
        }
  }
  // Tile base pointers are advanced per iteration (wave-uniform 64-bit); per-element
  // offsets inside a tile are 32-bit (row * ld + k stays below 2^31 for every shape
  // the library issues), which keeps register pressure low enough for 2 waves/SIMD.
  const T* Atile = Ab + (AK ? (long)m0 * d.lda : (long)m0);
  const T* Btile = Bb + (BKC ? (long)n0 * d.ldb : (long)n0);
  const int lda32 = (int)d.lda, ldb32 = (int)d.ldb;
  // Pair loads are whole-vector loads when no pair of this tile crosses the edge of its operand
  // and all are 2-element aligned (decided once per tile; wave-uniform).  Pairs past the edge in
  // m or n repeat the last one (their results are not stored), pairs past the end of K are zero.
  const int mrem = d.M - m0, nrem = d.N - n0;
  const bool vec_ok = (AK || mrem % 2 == 0) && (BKC || nrem % 2 == 0) && (d.lda % 2) == 0 && (d.ldb % 2) == 0 &&
                      (d.sAk % 2) == 0 && (d.sBk % 2) == 0 && ((uintptr_t)Atile % (2 * sizeof(T))) == 0 &&
                      ((uintptr_t)Btile % (2 * sizeof(T))) == 0;
  const int mlast = AK ? mrem - 1 : mrem - 2, nlast = BKC ? nrem - 1 : nrem - 2;
  // MODE 0: whole k tiles on the vector path, 1: the vector path with a ragged last one (pairs past K
  // repeat one of the tile, and 'cut' makes them zero on their way to LDS: at the load it would wait for
  // it), 2: guarded
  auto load = [&](int kb, int kt, auto mode) {
    constexpr int MODE = decltype(mode)::value;
    const int k0 = kt * BK;
    const T* Ak = Atile + kb * d.sAk + (AK ? (long)k0 : (long)k0 * d.lda);
    const T* Bk = Btile + kb * d.sBk + (BKC ? (long)k0 : (long)k0 * d.ldb);
    const int krem = d.K - k0;
    if constexpr (MODE == 0) {
#pragma unroll
      for (int i = 0; i < PA; ++i) {
        int m, k;
        a_pair(i * kThreads + tid, m, k);
        m = min(m, mlast);
        ra[i] = *reinterpret_cast<const pair_t*>(Ak + (AK ? (m * lda32 + k) : (k * lda32 + m)));
      }
#pragma unroll
      for (int i = 0; i < PB; ++i) {
        int n, k;
        b_pair(i * kThreads + tid, n, k);
        n = min(n, nlast);
        rb[i] = *reinterpret_cast<const pair_t*>(Bk + (BKC ? (n * ldb32 + k) : (k * ldb32 + n)));
      }
    } else if constexpr (MODE == 1) {
#pragma unroll
      for (int i = 0; i < PA; ++i) {
        int m, k;
        a_pair(i * kThreads + tid, m, k);
        m = min(m, mlast);
        const int kc = k < krem ? k : 0;
        ra[i] = *reinterpret_cast<const pair_t*>(Ak + (AK ? (m * lda32 + kc) : (kc * lda32 + m)));
      }
#pragma unroll
      for (int i = 0; i < PB; ++i) {
        int n, k;
        b_pair(i * kThreads + tid, n, k);
        n = min(n, nlast);
        const int kc = k < krem ? k : 0;
        rb[i] = *reinterpret_cast<const pair_t*>(Bk + (BKC ? (n * ldb32 + kc) : (kc * ldb32 + n)));
      }
    } else {
#pragma unroll
      for (int i = 0; i < PA; ++i) {
        int m, k;
        a_pair(i * kThreads + tid, m, k);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int mh = AK ? m : m + h, kh = AK ? k + h : k;
          T v = T(0);
          if (mh < mrem && kh < krem) v = Ak[AK ? (mh * lda32 + kh) : (kh * lda32 + mh)];
          ra[i][h] = v;
        }
      }
#pragma unroll
      for (int i = 0; i < PB; ++i) {
        int n, k;
        b_pair(i * kThreads + tid, n, k);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int nh = BKC ? n : n + h, kh = BKC ? k + h : k;
          T v = T(0);
          if (nh < nrem && kh < krem) v = Bk[BKC ? (nh * ldb32 + kh) : (kh * ldb32 + nh)];
          rb[i][h] = v;
        }
      }
    }
  };
  auto cut = [&](int kt) {
    const int krem = d.K - kt * BK;
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      int m, k;
      a_pair(i * kThreads + tid, m, k);
      ra[i] = k < krem ? ra[i] : pair_t{T(0), T(0)};
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      int n, k;
      b_pair(i * kThreads + tid, n, k);
      rb[i] = k < krem ? rb[i] : pair_t{T(0), T(0)};
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      int m, k;
      a_pair(i * kThreads + tid, m, k);
      *reinterpret_cast<pair_t*>(&As[buf][aidx(m, k)]) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      int n, k;
      b_pair(i * kThreads + tid, n, k);
      *reinterpret_cast<pair_t*>(&Bs[buf][bidx(n, k)]) = rb[i];
    }
  };
  // MFMA operand fragments of k group kk (4 deep) from LDS buffer buf
  auto frag = [&](int buf, int kk, T (&a)[TM], T (&b)[TN]) {
    const int kr = kk + (lane >> 4);
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = As[buf][aidx(wm * WTM + i * 16 + (lane & 15), kr)];
#pragma unroll
    for (int j = 0; j < TN; ++j) b[j] = Bs[buf][bidx(wn * WTN + j * 16 + (lane & 15), kr)];
  };
  auto mma = [&](const T (&a)[TM], const T (&b)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = Mfma<T>::mma(a[i], b[j], acc[i][j]);
  };

  // issue order pinned: one k group's MFMAs with the next group's fragment reads, and the stores or
  // the loads of a tile where there are any, between them
  auto interleave = [&](auto stores, auto loads) {
    constexpr int R = TM + TN, S = decltype(stores)::value ? PA + PB : 0, L = decltype(loads)::value ? PA + PB : 0;
    static_assert(TM * TN >= R && TM * TN >= PA + PB, "one read, store or load per MFMA");
#pragma unroll
    for (int r = 0; r < TM * TN; ++r) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (r < R) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (r < S) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      if (r < L) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
  };
  // As in the kernel above, the one barrier of a k tile stands before its last k group, whose
  // fragments are in registers by then.  The registers that hold the next tile go to the other
  // buffer during the first k group (the previous tile's barrier has freed it) and take the tile
  // after it during the second, so that a load has a whole tile's time to arrive.  Measured against
  // loads, reads and stores in a row and a barrier at the end of the tile: integrals of the strips
  // at 96/384/1152 25.1 -> 23.4 ms (59 -> 67 TF/s), K_A and U R of the RPA product there 3.08 ->
  // 2.82 and 2.30 -> 1.96 ms, ladder term at 128/512/1536 in FP32 24.4 -> 18.6 ms.
  auto reduce = [&](auto mode) {
    int kb = (int)(it0 / nkt), kt = (int)(it0 % nkt);
    const int steps = (int)(it1 - it0);
    int ahead = 0;  // tile last loaded
    // the next tile; past the end the last one again (not used), so that no load stands behind a
    // branch
    auto advance = [&]() {
      const bool more = ahead + 1 < steps, wrap = more && kt + 1 == nkt;
      ahead += more ? 1 : 0;
      kt = wrap ? 0 : kt + (more ? 1 : 0);
      kb += wrap ? 1 : 0;
    };
    T a0[TM], b0[TN], a1[TM], b1v[TN];
    load(kb, kt, mode);
    if constexpr (decltype(mode)::value == 1) cut(kt);
    store(0);
    if (steps > 1) {
      advance();
      load(kb, kt, mode);
    }
    __syncthreads();
    frag(0, 0, a0, b0);
    auto step = [&](auto cur) {
      constexpr int c = decltype(cur)::value;
      frag(c, 4, a1, b1v);
      if constexpr (decltype(mode)::value == 1) cut(kt);
      store(c ^ 1);
      mma(a0, b0);
      interleave(std::true_type{}, std::false_type{});
      advance();
      frag(c, 8, a0, b0);
      load(kb, kt, mode);
      mma(a1, b1v);
      if constexpr (decltype(mode)::value < 2) interleave(std::false_type{}, std::true_type{});
      frag(c, 12, a1, b1v);
      mma(a0, b0);
      interleave(std::false_type{}, std::false_type{});
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
      frag(c ^ 1, 0, a0, b0);
      mma(a1, b1v);
      interleave(std::false_type{}, std::false_type{});
      __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = 0; t < steps; t += 2) {
      step(std::integral_constant<int, 0>{});
      if (t + 1 < steps) step(std::integral_constant<int, 1>{});
    }
  };
  if (it0 < it1) {
    if (vec_ok && d.K % BK == 0)
      reduce(std::integral_constant<int, 0>{});
    else if (vec_ok && (!(AK || BKC) || d.K % 2 == 0))
      reduce(std::integral_constant<int, 1>{});
    else
      reduce(std::integral_constant<int, 2>{});
  }

  const long nbatch = (long)d.nb1 * d.nb2;
  if (!W && (d.cRm | d.cRn)) {
    store_mapped<T, acc_t, TM, TN, WTM, WTN>(d, alpha, beta, C + b1 * d.sC1 + b2 * d.sC2, m0, n0, wm, wn, lane, acc);
    return;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm * WTM + i * 16 + Mfma<T>::row(lane, r);
        const int col = n0 + wn * WTN + j * 16 + (lane & 15);
        if (row < d.M && col < d.N) {
          const T v = acc[i][j][r];
          if (W) {
            W[((long)split * nbatch + batch) * ((long)d.M * d.N) + (long)row * d.N + col] = v;
          } else {
            T* cp = C + b1 * d.sC1 + b2 * d.sC2 + (long)row * d.ldc + col;
            T out = alpha * v;
            if constexpr (CPF) {
              out += beta * cpre[i][j][r];
            } else {
              if (beta != T(0)) out += beta * (*cp);
            }
            *cp = out;
          }
        }
      }
}

// TAG 4: the C-prefetch variant of the register-staged tile (see gemm_tile).
template <typename T, int BM, int BN, int BK, bool AK, bool BKC, int TAG>
__global__ __launch_bounds__(kThreads, 2) void gemm_kernel(GemmDesc d, T alpha, const T* __restrict__ A,
                                                        const T* __restrict__ B, T beta, T* __restrict__ C,
                                                        T* __restrict__ W, int splitk) {
  // workgroups of all splits in one flat order, so that the tiles of a split, which read the same
  // part of both operands, meet in one XCD's L2.  Measured with the vector loads of edge tiles, at
  // 40/160/600 in FP64: ladder term 823 -> 723 us, ring exchange 519 -> 305, U R 428 -> 370.
  const int per = (int)gridDim.x;
  const int flat = (int)xcd_remap((long)blockIdx.y * per + blockIdx.x, (long)per * gridDim.y);
  const int split = __builtin_amdgcn_readfirstlane(flat / per);
  gemm_tile<T, BM, BN, BK, AK, BKC, TAG == 4>(d, alpha, A, B, beta, C, W, splitk, flat - split * per, split);
}

// The k-contiguous FP64 tiles of a short reduction: 512 workgroups that stay, each XCD with its
// contiguous range of tiles (see gemm_tile_dma).  A workgroup per tile starts with the latency of
// its first loads and ends with the stores of C, while the one wave per SIMD of its neighbour does
// not fill the matrix core.  Measured, a workgroup per tile | here, with the share of the cycles
// that the matrix units are busy: 1536 x 442368 over 384 8080 | 7843 us (85 | 89 %), 1536 x 110592
// over 384 2012 | 1922 us, 960 x 96000 over 160 567 | 524 us (71 | 77 %).
template <int TAG>
__global__ __launch_bounds__(kThreads, 2) void gemm_stream_kernel(GemmDesc d, double alpha, const double* __restrict__ A,
                                                                  const double* __restrict__ B, double beta,
                                                                  double* __restrict__ C) {
  const int ntiles = ((d.M + 127) / 128) * ((d.N + 127) / 128);
  const int x = (int)blockIdx.x % 8, j = (int)blockIdx.x / 8, per = (int)gridDim.x / 8;
  const int t0 = (int)((long)ntiles * x / 8), t1 = (int)((long)ntiles * (x + 1) / 8);
  if (t0 + j >= t1) return;
  gemm_tile_dma<128, 128, true>(d, alpha, A, B, beta, C, nullptr, 1, t0 + j, 0, (t1 - t0 - j + per - 1) / per, per);
}

// Batched updates C_(b1,b2) = alpha A_b2 B_b1 + beta C_(b1,b2) with small A (M, K <= 48): the
// k-space term of G, one o x o by o x v product for each auxiliary function and vector.  They are
// bound by the bytes of C; tiles of 64 x 64 spend a workgroup's start, the staging of A and a
// barrier per k tile on each 16 KB of it.  Here a wave keeps A in registers, in the MFMA layout,
// and walks blocks of 16 (FP64) or 32 columns over all b1, with B and C straight from the caches:
// no LDS, no barrier.  The k steps and their order are those of the tiles.  Measured at 24 x 600
// products of 40 x 160 over 40: FP64 600 -> 400 us (3.7 TB/s), FP32 423 -> 268 us; at 16 x 64 over 16
// in four windows 50 -> 22 us.
template <typename T, int MT>
__global__ __launch_bounds__(256, 2) void gemm_update_kernel(GemmDesc d, T alpha, const T* __restrict__ A,
                                                             const T* __restrict__ B, T beta, T* __restrict__ C) {
  using acc_t = typename Mfma<T>::acc_t;
  constexpr int KS = 4 * MT, CT = sizeof(T) == 8 ? 1 : 2;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int l16 = lane & 15, l4 = lane >> 4;
  const int b2 = blockIdx.x;
  const T* Ab = A + b2 * d.sA2;
  // rows and columns past the edge repeat the last one (their results are not stored), k values
  // past the end are zero
  T a[MT][KS];
  int krow[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int k = 4 * s + l4, kc = min(k, d.K - 1);
    krow[s] = kc * (int)d.ldb;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const T v = Ab[(long)min(16 * i + l16, d.M - 1) * d.lda + kc];
      a[i][s] = k < d.K ? v : T(0);
    }
  }
  const int cols = (d.N + 16 * CT - 1) / (16 * CT), blocks = d.nb1 * cols;
  for (int blk = (int)blockIdx.y * 4 + wave; blk < blocks; blk += 4 * (int)gridDim.y) {
    const int b1 = blk / cols, n0 = (blk - b1 * cols) * 16 * CT;
    const T* Bb = B + b1 * d.sB1;
    T* Cb = C + b1 * d.sC1 + b2 * d.sC2;
    T b[KS][CT], c[MT][CT][4];
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      const int n = min(n0 + 16 * j + l16, d.N - 1);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) c[i][j][r] = Cb[(long)min(16 * i + Mfma<T>::row(lane, r), d.M - 1) * d.ldc + n];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const T v = Bb[krow[s] + n];
        b[s][j] = 4 * s + l4 < d.K ? v : T(0);
      }
    }
    acc_t acc[MT][CT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = Mfma<T>::mma(a[i][s], b[s][j], acc[i][j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * i + Mfma<T>::row(lane, r);
#pragma unroll
        for (int j = 0; j < CT; ++j) {
          const int n = n0 + 16 * j + l16;
          if (m < d.M && n < d.N) {
            T out = alpha * acc[i][j][r];
            out += beta * c[i][j][r];
            Cb[(long)m * d.ldc + n] = out;
          }
        }
      }
  }
}

// ---------------------------------------------------------------------------
// Small FP64 products: the projected matrices and coefficient products of the window solver
// (M, N <= 512, reductions of 40 .. N) and the contractions of small systems.  They are bound by
// latency: a tiled launch of a few workgroups takes 7-20 us (its pipeline fill, one k tile in
// flight, 20-40 KB of unrolled code through a cold instruction cache), and a reduction split
// over workgroups adds a second launch of 3-8 us.  Here a wave computes one 16 x 16 tile with
// operands loaded from the caches straight into the MFMA layout, 4 steps of 8 in flight while
// the last 4 are multiplied, and where the output has few tiles the reduction is shared by WK
// waves of one workgroup (16 at most) and summed through LDS in wave order: one launch, a
// compact loop.  Neither edges nor short reductions are padded beyond 16 rows and 8 values.
// Measured, tiled with its reduction launch | here: 240 square 23.5 | 6.4 us, 40 x 1024 over 240
// 13.4 | 6.2, 960 x 160 over 160 23.6 | 9.6.
template <int WK>
__device__ __forceinline__ void gemm_small_tile(const GemmDesc& d, double alpha, const double* __restrict__ A,
                                                const double* __restrict__ B, double beta, double* __restrict__ C,
                                                int id) {
  using acc_t = Mfma<double>::acc_t;
  constexpr int U = 4;
  __shared__ acc_t part[WK > 1 ? WK : 1][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int tiles_m = (d.M + 15) / 16, tiles_n = (d.N + 15) / 16;
  int tm, tn, batch;
  if constexpr (WK == 1) {  // 2 x 2 tiles, one per wave
    const int gm = (tiles_m + 1) / 2, gn = (tiles_n + 1) / 2;
    batch = id / (gm * gn);
    tm = 2 * (id % (gm * gn) / gn) + (wave >> 1);
    tn = 2 * (id % gn) + (wave & 1);
  } else {
    batch = id / (tiles_m * tiles_n);
    tm = id % (tiles_m * tiles_n) / tiles_n;
    tn = id % tiles_n;
  }
  const int m0 = tm * 16, n0 = tn * 16, kq = lane >> 4;
  const int b1 = batch / d.nb2, b2 = batch % d.nb2;
  const long am = d.transA ? 1 : d.lda, ak = d.transA ? d.lda : 1;
  const long bn = d.transB ? d.ldb : 1, bk = d.transB ? 1 : d.ldb;
  // rows and columns past the edge repeat the last one (their results are not stored)
  const double* a = A + b1 * d.sA1 + b2 * d.sA2 + min(m0 + (lane & 15), d.M - 1) * am + 2 * kq * ak;
  const double* b = B + b1 * d.sB1 + b2 * d.sB2 + min(n0 + (lane & 15), d.N - 1) * bn + 2 * kq * bk;
  // steps of 8 values, the K values of each outer block padded to whole steps; lane group kq takes
  // values 2 kq and 2 kq + 1 of a step (any order of the reduction will do, as long as A and B
  // share it), so that an operand contiguous along k comes in 16-byte loads: of the 16 rows of a
  // load each gives a whole 64-byte line, and the loads per MFMA, which bound this kernel, halve
  const int S = (d.K + 7) / 8, total = d.KB * S;
  const int kw = WK == 1 ? 0 : wave;
  const int s0 = (int)((long)total * kw / WK), s1 = (int)((long)total * (kw + 1) / WK);
  const bool pa = ak == 1 && (d.lda % 2) == 0 && (d.sAk % 2) == 0 && (d.sA1 % 2) == 0 && (d.sA2 % 2) == 0 &&
                  (d.K % 2) == 0 && ((uintptr_t)A % 16) == 0;
  const bool pb = bk == 1 && (d.ldb % 2) == 0 && (d.sBk % 2) == 0 && (d.sB1 % 2) == 0 && (d.sB2 % 2) == 0 &&
                  (d.K % 2) == 0 && ((uintptr_t)B % 16) == 0;
  typedef double pair_t __attribute__((ext_vector_type(2)));
  auto one = [&](const double* p, long k1, bool pairs, int k, bool in) {
    pair_t v = pair_t{0.0, 0.0};
    if (pairs) {
      if (in && k < d.K) v = *reinterpret_cast<const pair_t*>(p);
    } else {
      if (in && k < d.K) v[0] = p[0];
      if (in && k + 1 < d.K) v[1] = p[k1];
    }
    return v;
  };
  int kb = s0 / S, ks = s0 % S;
  auto load = [&](int first, pair_t (&x)[U], pair_t (&y)[U]) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const bool in = first + i < s1;
      const int k = 8 * ks + 2 * kq;
      x[i] = one(a + (kb * d.sAk + 8 * ks * ak), ak, pa, k, in);
      y[i] = one(b + (kb * d.sBk + 8 * ks * bk), bk, pb, k, in);
      if (++ks == S) {
        ks = 0;
        ++kb;
      }
    }
  };
  acc_t acc = acc_t{0, 0, 0, 0};
  auto mul = [&](const pair_t (&x)[U], const pair_t (&y)[U]) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      acc = Mfma<double>::mma(x[i][0], y[i][0], acc);
      acc = Mfma<double>::mma(x[i][1], y[i][1], acc);
    }
  };
  pair_t x0[U], y0[U], x1[U], y1[U];
  load(s0, x0, y0);
  for (int st = s0; st < s1; st += 2 * U) {
    load(st + U, x1, y1);
    mul(x0, y0);
    load(st + 2 * U, x0, y0);
    mul(x1, y1);
  }
  if constexpr (WK > 1) {
    part[wave][lane] = acc;
    __syncthreads();
    if (wave != 0) return;
#pragma unroll 3
    for (int q = 1; q < WK; ++q) acc += part[q][lane];
  }
  const int col = n0 + (lane & 15);
  if (col >= d.N) return;
  const bool mapped = (d.cRm | d.cRn) != 0;
  const long co = b1 * d.sC1 + b2 * d.sC2 + (mapped ? c_index(d.cRn ? col + d.cBn : col, d.cRn, d.cSn, 1) : (long)col);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = m0 + Mfma<double>::row(lane, r);
    if (row >= d.M) continue;
    double* cp = C + co + (mapped ? c_index(row, d.cRm, d.cSm, d.ldc) : (long)row * d.ldc);
    double out = alpha * acc[r];
    if (beta != 0.0) out += beta * (*cp);
    *cp = out;
  }
}

template <int WK>
__global__ __launch_bounds__(WK == 16 ? 1024 : 256) void gemm_small_kernel(GemmDesc d, double alpha,
                                                                          const double* __restrict__ A,
                                                                          const double* __restrict__ B, double beta,
                                                                          double* __restrict__ C) {
  gemm_small_tile<WK>(d, alpha, A, B, beta, C, (int)xcd_remap(blockIdx.x, gridDim.x));
}

// Up to kGroupMax independent GEMMs of one tile shape in one grid: member g owns the
// flattened workgroup ids [start_g, start_{g+1}).  The member is found by a
// wave-uniform scan of the start table, so every member keeps the single-GEMM tile
// schedule (and the XCD remap applies over the whole grid).
constexpr int kGroupMax = 8;
template <typename T>
struct GroupMember {
  GemmDesc d;
  const T* A;
  const T* B;
  T* C;
  T alpha, beta;
  long start;
};
template <typename T>
struct GroupArgs {
  GroupMember<T> m[kGroupMax];
  int n;
};

template <typename T, int BM, int BN, int BK, bool AK, bool BKC, int TAG>
__global__ __launch_bounds__(kThreads, 2) void gemm_group_kernel(GroupArgs<T> g) {
  const long flat = xcd_remap(blockIdx.x, (long)gridDim.x);
  int j = 0;
  for (int q = 1; q < g.n; ++q)
    if (flat >= g.m[q].start) j = q;
  const GroupMember<T>& mb = g.m[__builtin_amdgcn_readfirstlane(j)];
  gemm_tile<T, BM, BN, BK, AK, BKC>(mb.d, mb.alpha, mb.A, mb.B, mb.beta, mb.C, nullptr, 1, flat - mb.start, 0);
}

template <int WK>
__global__ __launch_bounds__(WK == 16 ? 1024 : 256) void gemm_small_group_kernel(GroupArgs<double> g) {
  const long flat = xcd_remap(blockIdx.x, (long)gridDim.x);
  int j = 0;
  for (int q = 1; q < g.n; ++q)
    if (flat >= g.m[q].start) j = q;
  const GroupMember<double>& mb = g.m[__builtin_amdgcn_readfirstlane(j)];
  gemm_small_tile<WK>(mb.d, mb.alpha, mb.A, mb.B, mb.beta, mb.C, (int)(flat - mb.start));
}

// The line between the small products and the tiled ones, from both measured (us, tiled with its
// reduction launch | small): at most 2048 tiles (two waves per SIMD of the chip; a larger output
// fills it with 64 x 64 tiles, which read each operand element once per 64 outputs and can share
// grouped launches) and 6e4 steps of 8 values in all: 480 x 480 x 480 26.9 | 18.0,
// 481 x 660 x 481 38.1 | 42.8; and 512 steps in a reduction, as the 16 waves of a tile share one
// CU's loads: 240 x 40 over 1024 15.7 | 12.4, 78 x 37 over 4070 26.6 | 26.4, 24 x 24 over 6400
// 33 | 50.  Depends on the shape alone, so a product rounds the same way in every launch that it
// is part of.
inline long small_tiles(const GemmDesc& d) {
  return (long)((d.M + 15) / 16) * ((d.N + 15) / 16) * d.nb1 * d.nb2;
}
inline long small_steps(const GemmDesc& d) { return (long)d.KB * ((d.K + 7) / 8); }
inline int small_waves(const GemmDesc& d) {
  const long tiles = small_tiles(d), steps = small_steps(d);
  if (tiles >= 1024 || steps <= 8) return 1;
  return tiles >= 256 || steps <= 64 ? 4 : 16;
}
inline bool small_gemm(const GemmDesc& d) {
  if (d.K == 1 && d.transA == 0 && d.transB != 0) return true;  // rows of one value have no pairs to load
  const long tiles = small_tiles(d), steps = small_steps(d);
  return tiles <= 2048 && steps <= 512 && tiles * steps <= 60000;
}
inline long small_workgroups(const GemmDesc& d) {
  return small_waves(d) == 1 ? (long)((d.M + 31) / 32) * ((d.N + 31) / 32) * d.nb1 * d.nb2 : small_tiles(d);
}
void launch_small(const GemmDesc& d, double alpha, const double* A, const double* B, double beta, double* C,
                  hipStream_t s) {
  if (d.cRm < 0 || d.cRn < 0) throw InvalidArg("gemm: negative C index split");
  const int wk = small_waves(d);
  const long t = small_workgroups(d);
  if (wk == 1)
    gemm_small_kernel<1><<<(unsigned)t, 256, 0, s>>>(d, alpha, A, B, beta, C);
  else if (wk == 4)
    gemm_small_kernel<4><<<(unsigned)t, 256, 0, s>>>(d, alpha, A, B, beta, C);
  else
    gemm_small_kernel<16><<<(unsigned)t, 1024, 0, s>>>(d, alpha, A, B, beta, C);
  PPW_LAUNCH_CHECK();
}

// n <= kGroupMax small products of the same waves per tile in one launch.
void launch_small_group(const GemmCall<double>* const* calls, int n, hipStream_t s) {
  GroupArgs<double> g{};
  long total = 0;
  for (int i = 0; i < n; ++i) {
    const GemmCall<double>& c = *calls[i];
    if (c.d.cRm < 0 || c.d.cRn < 0) throw InvalidArg("gemm: negative C index split");
    g.m[i] = GroupMember<double>{c.d, c.A, c.B, c.C, c.alpha, c.beta, total};
    total += small_workgroups(c.d);
  }
  g.n = n;
  const int wk = small_waves(calls[0]->d);
  if (wk == 1)
    gemm_small_group_kernel<1><<<(unsigned)total, 256, 0, s>>>(g);
  else if (wk == 4)
    gemm_small_group_kernel<4><<<(unsigned)total, 256, 0, s>>>(g);
  else
    gemm_small_group_kernel<16><<<(unsigned)total, 1024, 0, s>>>(g);
  PPW_LAUNCH_CHECK();
}

template <typename T>
__global__ void splitk_reduce_kernel(GemmDesc d, T alpha, T beta, const T* __restrict__ W, T* __restrict__ C,
                                     int splitk) {
  const long per = (long)d.M * d.N;
  const long nbatch = (long)d.nb1 * d.nb2;
  const long total = per * nbatch;
  for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < total; idx += (long)gridDim.x * blockDim.x) {
    const long batch = idx / per;
    const long rc = idx % per;
    const int row = (int)(rc / d.N), col = (int)(rc % d.N);
    T s = T(0);
    // (the order of the sum is that of the splits; the loads of eight go out together: one at a time,
    // 64 splits of a 13 x 37 product over four vectors took 18 us)
    const T* w = W + batch * per + rc;
    const long step = nbatch * per;
    int k = 0;
    for (; k + 8 <= splitk; k += 8) {
      T v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = w[(k + u) * step];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; k < splitk; ++k) s += w[k * step];
    const int b1 = (int)(batch / d.nb2), b2 = (int)(batch % d.nb2);
    T* cp = C + b1 * d.sC1 + b2 * d.sC2 + c_index(row, d.cRm, d.cSm, d.ldc) + c_index(d.cRn ? col + d.cBn : col, d.cRn, d.cSn, 1);
    T out = alpha * s;
    if (beta != T(0)) out += beta * (*cp);
    *cp = out;
  }
}

inline bool ntiles_total_exceeds(long n) { return n <= 0 || n > 2147483647L; }

// Workgroups of one GEMM at tile shape BM x BN (before split-K); checks the limits
// the kernel relies on.
// Reduction splits when the grid is too small to fill 256 CUs: enough for about 1024
// workgroups, at least 4 k tiles per split, within the workspace, at most 256.
int auto_splitk(long wgs, long total, size_t per, size_t ws_bytes) {
  if (wgs >= 512 || total < 8) return 1;
  long want = (1024 + wgs - 1) / wgs;
  want = std::min<long>(want, total / 4);
  if (per > 0) want = std::min<long>(want, (long)(ws_bytes / per));
  want = std::min<long>(want, 256);
  return want >= 2 ? (int)want : 1;
}

template <int BM, int BN, int BK>
long checked_workgroups(const GemmDesc& d) {
  const long nbatch = (long)d.nb1 * d.nb2;
  const long wgs = (long)((d.M + BM - 1) / BM) * ((d.N + BN - 1) / BN) * nbatch;
  if (ntiles_total_exceeds(wgs)) throw InvalidArg("gemm: too many workgroups");
  // per-tile element offsets are 32-bit inside the kernel: rows of a tile that lie
  // outside the operand are never addressed, so a k-contiguous operand needs
  // min(M, BM) rows of lda, an m-contiguous one BK rows
  const double ra = d.transA == 0 ? (double)std::min(d.M, BM) * d.lda + BK : (double)BK * d.lda + BM;
  const double rb = d.transB != 0 ? (double)std::min(d.N, BN) * d.ldb + BK : (double)BK * d.ldb + BN;
  if (ra >= 2147483647.0 || rb >= 2147483647.0 || d.lda >= 2147483647L || d.ldb >= 2147483647L)
    throw InvalidArg("gemm: leading dimension too large for 32-bit tile offsets");
  if (d.cRm < 0 || d.cRn < 0) throw InvalidArg("gemm: negative C index split");
  return wgs;
}

constexpr long kCUs = 256;
constexpr long kResident = 512;  // workgroups resident at once: 256 CUs x 2

// Reductions up to 1024, where starts and ends are 3 % of a tile's time or more (beyond, the one-tile
// kernel's rounds need no whole pairs of k tiles), and two rounds of tiles at least, so that a
// workgroup has a next tile.
inline bool stream_gemm(const GemmDesc& d, const double* A, const double* B) {
  const long ntiles = (long)((d.M + 127) / 128) * ((d.N + 127) / 128);
  return d.nb1 == 1 && d.nb2 == 1 && d.KB == 1 && d.sym < 0 && d.M % 8 == 0 && d.N % 8 == 0 && d.K % 32 == 0 &&
         d.K <= 1024 && ntiles >= 2 * kResident && d.lda % 2 == 0 && d.ldb % 2 == 0 && (uintptr_t)A % 16 == 0 &&
         (uintptr_t)B % 16 == 0;
}

template <typename T, int BM, int BN, int BK, bool AK, bool BKC, int TAG>
void launch(const GemmDesc& d, T alpha, const T* A, const T* B, T beta, T* C, hipStream_t s, Workspace ws) {
  const int tiles_m = (d.M + BM - 1) / BM, tiles_n = (d.N + BN - 1) / BN;
  const long nbatch = (long)d.nb1 * d.nb2;
  checked_workgroups<BM, BN, BK>(d);
  const long ntiles = (long)tiles_m * tiles_n;
  // Wave quantisation: when the last of several waves of 128 x 128 tiles would run at
  // most half full, the trailing tile columns or tile rows that make up that wave (whichever are
  // fewer tiles) are peeled off and computed with 64 x 64 tiles (four times the workgroups, a
  // quarter of the work each), so the tail takes about a quarter of a tile's time.  Every output
  // element is accumulated over the same sequence of MFMA k steps in both tile shapes, so the
  // result is bit-identical to the unpeeled GEMM.  The peeled part has its own kernel symbol
  // (TAG + 2) so that traces tell the two apart.  Measured at 36864 x 2304 x 36864 (288 x 18 tiles,
  // 64 over ten waves): 1 of 18 columns peeled 87.3 + 7.2 ms, 4 of 288 rows 88.1 + 2.5 ms.
  if constexpr (TAG < 2 && BM == 128 && BN == 128) {
   if (nbatch == 1 && ntiles >= 2 * kResident && d.splitk <= 1 && d.sym < 0) {
    const long rem = ntiles % kResident;
    const int cols = (int)((rem + tiles_m - 1) / tiles_m), rows = (int)((rem + tiles_n - 1) / tiles_n);
    if (rem > 0 && rem <= kResident / 2 && d.cRm == 0 && rows < tiles_m && (long)rows * tiles_n < (long)cols * tiles_m) {
      const long nmain = (long)(tiles_m - rows) * BM;
      GemmDesc dm = d, dr = d;
      dm.M = (int)nmain;
      dr.M = d.M - (int)nmain;
      launch<T, BM, BN, BK, AK, BKC, TAG>(dm, alpha, A, B, beta, C, s, Workspace{});
      launch<T, BM / 2, BN / 2, BK, AK, BKC, TAG + 2>(dr, alpha, A + nmain * (AK ? d.lda : 1), B, beta,
                                                      C + nmain * d.ldc, s, Workspace{});
      return;
    }
    if (rem > 0 && rem <= kResident / 2 && cols < tiles_n) {
      const int nmain = (tiles_n - cols) * BN;
      GemmDesc dm = d, dr = d;
      dm.N = nmain;
      dr.N = d.N - nmain;
      launch<T, BM, BN, BK, AK, BKC, TAG>(dm, alpha, A, B, beta, C, s, Workspace{});
      const T* Br = B + (BKC ? (long)nmain * d.ldb : (long)nmain);
      T* Cr = C + nmain;
      if (d.cRn) {  // mapped columns: the tail maps its columns from nmain on
        dr.cBn = d.cBn + nmain;
        Cr = C;
      }
      launch<T, BM / 2, BN / 2, BK, AK, BKC, TAG + 2>(dr, alpha, A, Br, beta, Cr, s, Workspace{});
      return;
    }
   }
  }
  const int nkt = (d.K + BK - 1) / BK;
  const long total = (long)d.KB * nkt;
  const size_t per = (size_t)d.M * d.N * nbatch * sizeof(T);
  int splitk = auto_splitk(ntiles * nbatch, total, per, ws.bytes);
  if (d.splitk > 0) {
    splitk = d.splitk;
    if (splitk > 1 && (splitk > 256 || ws.bytes / per < (size_t)splitk))
      throw InvalidArg("gemm: workspace too small for the requested reduction splits");
  }
  dim3 grid((unsigned)(ntiles * nbatch), (unsigned)splitk, 1);
  if (d.sym >= 0) {
    // tiles left out only in the plain launch of the strips' integrals; elsewhere (64 x 64
    // tiles, reduction splits) the whole product
    constexpr bool SYM = !AK && !BKC && BM == 128 && TAG == 0;
    GemmDesc f = d;
    if (!SYM || splitk != 1 || nbatch != 1) {
      f.sym = -1;
      f.splitk = splitk;
      launch<T, BM, BN, BK, AK, BKC, TAG>(f, alpha, A, B, beta, C, s, ws);
      return;
    }
    grid.x = (unsigned)sym_tiles<BM, BN>(d);
  }
  if constexpr (TAG == 0 && BM == 64 && !(std::is_same<T, double>::value && AK && BKC)) {
    // short accumulating reductions: load C before the reduction (same arithmetic)
    if (splitk == 1 && beta != T(0) && total <= 4 && !(d.cRm | d.cRn)) {
      gemm_kernel<T, BM, BN, BK, AK, BKC, 4><<<grid, kThreads, 0, s>>>(d, alpha, A, B, beta, C, nullptr, 1);
      PPW_LAUNCH_CHECK();
      return;
    }
  }
  // whole rounds of short reductions on workgroups that stay
  if constexpr (std::is_same<T, double>::value && AK && BKC && BM == 128 && TAG < 2) {
    if (splitk == 1 && stream_gemm(d, A, B)) {
      gemm_stream_kernel<TAG><<<(unsigned)kResident, kThreads, 0, s>>>(d, alpha, A, B, beta, C);
      PPW_LAUNCH_CHECK();
      return;
    }
  }
  if (splitk == 1) {
    gemm_kernel<T, BM, BN, BK, AK, BKC, TAG><<<grid, kThreads, 0, s>>>(d, alpha, A, B, beta, C, nullptr, 1);
    PPW_LAUNCH_CHECK();
  } else {
    T* W = static_cast<T*>(ws.ptr);
    gemm_kernel<T, BM, BN, BK, AK, BKC, TAG><<<grid, kThreads, 0, s>>>(d, alpha, A, B, beta, C, W, splitk);
    PPW_LAUNCH_CHECK();
    const long n = (long)d.M * d.N * nbatch;
    const int blocks = (int)std::min<long>((n + 255) / 256, 8192);
    splitk_reduce_kernel<T><<<blocks, 256, 0, s>>>(d, alpha, beta, W, C, splitk);
    PPW_LAUNCH_CHECK();
  }
}

// The tiled kernels' limits hold for small products too.
inline void check_small(const GemmDesc& d) {
  if (d.M >= 96 && d.N >= 96 && d.tile != 64)
    checked_workgroups<128, 128, 16>(d);
  else
    checked_workgroups<64, 64, 16>(d);
}

// A alike for all b1 and B for all b2, and enough 64 x 64 tiles to leave no reduction split.
inline bool update_gemm(const GemmDesc& d, bool accumulates) {
  return accumulates && d.M <= 48 && d.K <= 48 && d.KB == 1 && d.transA == 0 && d.transB == 0 && d.sA1 == 0 &&
         d.sB2 == 0 && d.nb2 > 1 && 48 * d.ldb < 2147483647L && d.splitk <= 1 && d.sym < 0 && !(d.cRm | d.cRn) &&
         (long)((d.N + 63) / 64) * d.nb1 * d.nb2 >= kResident;
}
template <typename T>
void launch_update(const GemmDesc& d, T alpha, const T* A, const T* B, T beta, T* C, hipStream_t s) {
  checked_workgroups<64, 64, 16>(d);  // the tiled kernel's limits
  const int cols = sizeof(T) == 8 ? 16 : 32;
  const long blocks = (long)d.nb1 * ((d.N + cols - 1) / cols);
  // about 2048 workgroups, each wave with some blocks for the one load of A
  const dim3 grid((unsigned)d.nb2, (unsigned)std::max(1L, std::min((2048L + d.nb2 - 1) / d.nb2, blocks / 16)));
  if (d.M <= 16 && d.K <= 16)
    gemm_update_kernel<T, 1><<<grid, 256, 0, s>>>(d, alpha, A, B, beta, C);
  else if (d.M <= 32 && d.K <= 32)
    gemm_update_kernel<T, 2><<<grid, 256, 0, s>>>(d, alpha, A, B, beta, C);
  else
    gemm_update_kernel<T, 3><<<grid, 256, 0, s>>>(d, alpha, A, B, beta, C);
  PPW_LAUNCH_CHECK();
}

template <typename T, int TAG = 0>
void gemm_dispatch(const GemmDesc& d, T alpha, const T* A, const T* B, T beta, T* C, hipStream_t s,
                   Workspace ws) {
  if (d.M <= 0 || d.N <= 0 || d.nb1 <= 0 || d.nb2 <= 0) return;
  if (d.K <= 0 || d.KB <= 0) throw InvalidArg("gemm: empty reduction");
  if constexpr (std::is_same<T, double>::value) {
    if (small_gemm(d)) {
      check_small(d);
      launch_small(d, alpha, A, B, beta, C, s);
      return;
    }
  }
  if constexpr (TAG == 0) {
    if (update_gemm(d, beta != T(0))) {
      launch_update<T>(d, alpha, A, B, beta, C, s);
      return;
    }
  }
  const bool big = d.M >= 96 && d.N >= 96 && d.tile != 64;
  const bool ak = d.transA == 0, bk = d.transB != 0;
#define PPW_GEMM_CASE(BMv, BNv, AKv, BKv)                                           \
  if (ak == AKv && bk == BKv) {                                                     \
    launch<T, BMv, BNv, 16, AKv, BKv, TAG>(d, alpha, A, B, beta, C, s, ws);         \
    return;                                                                         \
  }
  if constexpr (TAG == 0) {
    // Rows of tiles of 96 where as many of them do as of 128 (96 rows in one, 129 .. 192 in two,
    // 257 .. 288 in three): a quarter less work for the same workgroups and reduction splits.  128
    // rows | 96, FP64: 96 x 512 over 96 x 1500, 8 vectors, 2.70 | 2.21 ms, 130 (130 x 1500) 7.10 | 5.49,
    // 192 (192 x 1500) 10.3 | 8.7, 288 (288 x 1500) 21.9 | 18.8; between 1.16 and 1.42 times as fast at
    // 96, 130, 160, 192, 260 and 288 rows, in FP64 and FP32, over operands of all layouts.
    if (big && d.sym < 0 && (d.M + 95) / 96 == (d.M + 127) / 128) {
      checked_workgroups<128, 128, 16>(d);
      PPW_GEMM_CASE(96, 128, true, true)
      PPW_GEMM_CASE(96, 128, true, false)
      PPW_GEMM_CASE(96, 128, false, true)
      PPW_GEMM_CASE(96, 128, false, false)
    }
  }
  if (big) {
    PPW_GEMM_CASE(128, 128, true, true)
    PPW_GEMM_CASE(128, 128, true, false)
    PPW_GEMM_CASE(128, 128, false, true)
    PPW_GEMM_CASE(128, 128, false, false)
  } else {
    PPW_GEMM_CASE(64, 64, true, true)
    PPW_GEMM_CASE(64, 64, true, false)
    PPW_GEMM_CASE(64, 64, false, true)
    PPW_GEMM_CASE(64, 64, false, false)
  }
#undef PPW_GEMM_CASE
}

// One grouped launch of n <= kGroupMax members sharing the tile shape.
template <typename T, int BM, int BN, int BK, bool AK, bool BKC, int TAG>
void launch_group(const GemmCall<T>* const* calls, int n, hipStream_t s) {
  GroupArgs<T> g{};
  long total = 0;
  for (int i = 0; i < n; ++i) {
    const GemmCall<T>& c = *calls[i];
    g.m[i] = GroupMember<T>{c.d, c.A, c.B, c.C, c.alpha, c.beta, total};
    g.m[i].d.sym = -1;
    total += checked_workgroups<BM, BN, BK>(c.d);
  }
  g.n = n;
  if (ntiles_total_exceeds(total)) throw InvalidArg("gemm: too many workgroups in a group");
  gemm_group_kernel<T, BM, BN, BK, AK, BKC, TAG><<<dim3((unsigned)total), kThreads, 0, s>>>(g);
  PPW_LAUNCH_CHECK();
}

template <typename T, int TAG>
void group_dispatch(bool big, bool ak, bool bk, const GemmCall<T>* const* calls, int n, hipStream_t s) {
#define PPW_GROUP_CASE(BMv, BNv, AKv, BKv)                              \
  if (ak == AKv && bk == BKv) {                                         \
    launch_group<T, BMv, BNv, 16, AKv, BKv, TAG>(calls, n, s);          \
    return;                                                             \
  }
  if (big) {
    PPW_GROUP_CASE(128, 128, true, true)
    PPW_GROUP_CASE(128, 128, true, false)
    PPW_GROUP_CASE(128, 128, false, true)
    PPW_GROUP_CASE(128, 128, false, false)
  } else {
    PPW_GROUP_CASE(64, 64, true, true)
    PPW_GROUP_CASE(64, 64, true, false)
    PPW_GROUP_CASE(64, 64, false, true)
    PPW_GROUP_CASE(64, 64, false, false)
  }
#undef PPW_GROUP_CASE
}

template <typename T>
void single_dispatch(const GemmCall<T>& c, hipStream_t s) {
  if (c.tag >= 2) {
    if constexpr (std::is_same<T, float>::value)
      gemm_sbf16(c.d, c.alpha, c.A, c.B, c.beta, c.C, s, c.tag == 3);
    else
      throw InvalidArg("split-BF16 products take FP32 operands");
    return;
  }
  if (c.tag == 1)
    gemm_dispatch<T, 1>(c.d, c.alpha, c.A, c.B, c.beta, c.C, s, c.ws);
  else
    gemm_dispatch<T, 0>(c.d, c.alpha, c.A, c.B, c.beta, c.C, s, c.ws);
}

// Independent GEMMs issued together: members with the same tile shape (and symbol
// tag) go into grouped launches when together they fill the chip without split-K;
// the rest (a lone member, or a set too small to fill 256 CUs) are launched one by
// one, where split-K applies.
template <typename T>
int gemm_group_impl(const std::vector<GemmCall<T>>& calls, hipStream_t s) {
  int grouped = 0;
  struct Key {
    bool big, ak, bk;
    int tag;
    bool operator==(const Key& o) const { return big == o.big && ak == o.ak && bk == o.bk && tag == o.tag; }
  };
  std::vector<Key> keys;
  std::vector<std::vector<const GemmCall<T>*>> sets;
  std::vector<const GemmCall<T>*> small[3];  // small products by waves per tile
  for (const auto& c : calls) {
    const GemmDesc& d = c.d;
    if (d.M <= 0 || d.N <= 0 || d.nb1 <= 0 || d.nb2 <= 0) continue;
    if (d.K <= 0 || d.KB <= 0) throw InvalidArg("gemm: empty reduction");
    if constexpr (std::is_same<T, double>::value) {
      if (small_gemm(d)) {
        check_small(d);
        const int wk = small_waves(d);
        small[wk == 1 ? 0 : (wk == 4 ? 1 : 2)].push_back(&c);
        continue;
      }
    }
    if (d.splitk > 1 || c.tag >= 2) {
      // fixed reduction splits need the split-K launch; split-BF16 has its own kernel
      single_dispatch(c, s);
      continue;
    }
    const Key k{d.M >= 96 && d.N >= 96 && d.tile != 64, d.transA == 0, d.transB != 0, c.tag};
    size_t i = 0;
    while (i < keys.size() && !(keys[i] == k)) ++i;
    if (i == keys.size()) {
      keys.push_back(k);
      sets.emplace_back();
    }
    sets[i].push_back(&c);
  }
  if constexpr (std::is_same<T, double>::value) {
    for (auto& set : small)
      for (size_t j = 0; j < set.size(); j += kGroupMax) {
        const int n = (int)std::min<size_t>(kGroupMax, set.size() - j);
        if (n == 1) {
          single_dispatch(*set[j], s);
        } else {
          launch_small_group(set.data() + j, n, s);
          ++grouped;
        }
      }
  }
  for (size_t i = 0; i < keys.size(); ++i) {
    const Key& k = keys[i];
    auto& set = sets[i];
    long wgs = 0;
    for (auto* c : set)
      wgs += k.big ? checked_workgroups<128, 128, 16>(c->d) : checked_workgroups<64, 64, 16>(c->d);
    if (set.size() == 1 || wgs < 512) {
      for (auto* c : set) single_dispatch(*c, s);
      continue;
    }
    for (size_t j = 0; j < set.size(); j += kGroupMax) {
      const int n = (int)std::min<size_t>(kGroupMax, set.size() - j);
      if (k.tag == 1)
        group_dispatch<T, 1>(k.big, k.ak, k.bk, set.data() + j, n, s);
      else
        group_dispatch<T, 0>(k.big, k.ak, k.bk, set.data() + j, n, s);
      ++grouped;
    }
  }
  return grouped;
}

// ---------------------------------------------------------------------------
// Split-BF16 products.  An FP32 value x is carried as hi = bf16(x) (round to nearest
// even) and lo = bf16(x - hi); a b is taken as hi_a lo_b + lo_a hi_b + hi_a hi_b with FP32
// accumulation (the dropped lo_a lo_b and the rounding of lo leave about 2^-16 of |a b|
// per product).  Operands are split once, in memory, before the product (split_sbf16):
// a row of values is a sequence of 32-byte chunks, chunk c holding the bf16 hi parts of
// values 8c .. 8c+7 and then their 8 lo parts.  A value still occupies 4 bytes, so rows
// keep their FP32 strides (a multiple of 8 values) and an FP32 array is split in place.
//
// Kernel: WM x WN wave64s on BM x BN tiles (4 x 2 on 256 x 256 at one workgroup per CU,
// 2 x 2 on 128 x 128 or 64 x 64 at two), two LDS buffers; a k tile is 32 values = 4 chunks
// = 128 B per row, loaded straight into LDS (global_load_lds_dwordx4) in the swizzled
// slot layout of the FP64 kernel (16-byte slot s of row r at 8r + (s ^ ((r >> 1) & 7)),
// logical slot 2c holding chunk c's hi parts and 2c + 1 its lo parts), so a fragment
// read of 16 rows x 16 B touches every bank once and no conversion happens in the loop.
// Each wave computes 32 x 32 blocks with v_mfma_f32_32x32x16_bf16 (on gfx950 it issues
// at twice the rate of the 16x16x32 form: 2.0 against 1.1 PFLOP/s measured with
// register-only chains), three MFMAs per block and 16-value k step: lane l supplies row
// l % 32 and chunk l / 32 of the step; block results: lane l, register r holds row
// 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.  Values past K inside the last chunk of a row
// must be zero (split_sbf16 of a zero-padded row leaves them so).
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
constexpr int kSbBK = 32;

__device__ __forceinline__ int row32(int lane, int r) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// WM x WN waves (64 WM WN threads), each owning a (BM / WM) x (BN / WN) block of the tile;
// two LDS buffers; OCC workgroups per CU (register budget).  TAG only distinguishes kernel symbols (1: the
// amplitude contraction, so that profiles can attribute its time); the code is identical.
template <int BM, int BN, int WM, int WN, int OCC, int TAG = 0>
__global__ __launch_bounds__(64 * WM * WN, OCC) void gemm_sbf16_kernel(
    GemmDesc d, float alpha, const float* __restrict__ A, const float* __restrict__ B, float beta,
    float* __restrict__ C) {
  constexpr int BK = kSbBK, NW = WM * WN, NT = 64 * NW;
  constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  constexpr int SA = BM * BK, SB = BN * BK;       // storage floats per buffer
  constexpr int CA = BM / (8 * NW), CB = BN / (8 * NW);  // 1 KB wave loads (8 rows each) per operand tile
  static_assert(CA * 8 * NW == BM && CB * 8 * NW == BN && TM * 32 == WTM && TN * 32 == WTN, "tile shape");
  // separate arrays, and a loop unrolled by two: a buffer being filled and the buffer being
  // read are distinct objects to the compiler, which otherwise waits for the loads in flight
  // before every fragment read
  __shared__ __attribute__((aligned(16))) float As0[SA];
  __shared__ __attribute__((aligned(16))) float As1[SA];
  __shared__ __attribute__((aligned(16))) float Bs0[SB];
  __shared__ __attribute__((aligned(16))) float Bs1[SB];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int tiles_m = (d.M + BM - 1) / BM, tiles_n = (d.N + BN - 1) / BN;
  int tm, tn;
  if (d.sym >= 0) {
    if (!sym_tile_coords(d, xcd_remap(blockIdx.x, (long)gridDim.x), BM, BN, tiles_m, tiles_n, tm, tn)) return;
  } else {
    tile_coords((int)xcd_remap(blockIdx.x, (long)gridDim.x), tiles_m, tiles_n, tm, tn);
  }
  const int m0 = tm * BM, n0 = tn * BN;
  const float* At = A + (long)m0 * d.lda;
  const float* Bt = B + (long)n0 * d.ldb;
  const int lda32 = (int)d.lda, ldb32 = (int)d.ldb;
  const int mrem = d.M - m0, nrem = d.N - n0;
  // Every k tile is loaded straight into LDS.  Rows past an edge in m or n repeat the last one (their
  // results are not stored).  A ragged last k tile is the 4 chunks that end with K, so its own chunks
  // come 'back' places late in it (without 4 chunks in a row: the last one is repeated); it is read and
  // cut by tail() below.  Measured, with ragged tiles and edges
  // through registers, in a loop that spilled | here: 6400 x 7200 over 6400 1916 | 1680 us, 6795 x 5500
  // over 6795 2130 | 1557, 13115 x 5600 over 13115 6920 | 5382, 3024 x 1512 over 3024 284 | 126.
  const int nkt = (d.K + BK - 1) / BK, nch = (d.K + 7) / 8;
  const int left = nch - 4 * (nkt - 1), back = nkt > 1 ? 4 - left : 0;
  // A wave's load is 8 rows: its first row is scalar, the lanes' offsets from it are those of every
  // load but the one at an edge.  In a tile without an edge they are 32-bit byte offsets (BM rows of lda
  // lie within 2^31 values), so that a load takes its address from scalar registers and one vector
  // register; at an edge they are worked out for every tile.
  const int sg = (lane & 7) ^ ((4 * wave + (lane >> 4)) & 7), slot = 8 * min(sg >> 1, nch - 1) + 4 * (sg & 1);
  const unsigned inA = 4u * ((lane >> 3) * lda32 + slot), inB = 4u * ((lane >> 3) * ldb32 + slot);
  auto fill = [&](float* Ab, float* Bb, int kt, auto whole) {
    const int k0 = kt * BK - (kt + 1 == nkt ? 8 * back : 0);
    auto rows = [&](const float* X, long ld, int rem, unsigned in, int i) {
      if constexpr (decltype(whole)::value)
        return (const char*)(X + k0 + (long)i * ld) + in;
      else
        return (const char*)(X + k0 + (min(i + (hidden(lane) >> 3), rem - 1) * (int)ld + slot));
    };
#pragma unroll
    for (int c = 0; c < CA; ++c)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)rows(At, d.lda, mrem, inA, (wave + NW * c) * 8),
          (__attribute__((address_space(3))) void*)(Ab + (wave + NW * c) * 256), 16, 0, 0);
#pragma unroll
    for (int c = 0; c < CB; ++c)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)rows(Bt, d.ldb, nrem, inB, (wave + NW * c) * 8),
          (__attribute__((address_space(3))) void*)(Bb + (wave + NW * c) * 256), 16, 0, 0);
  };
  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const int rl = lane & 31, hl = lane >> 5;
  // fragments of 16-value step st of the k tile in buffer (Ab, Bb)
  struct Frags {
    bf16x8_t ah[TM], al[TM], bh[TN], bl[TN];
  };
  auto frags = [&](const float* Ab, const float* Bb, int st, Frags& f) {
    const int ch = 2 * st + hl;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int r = wm * WTM + i * 32 + rl;
      f.ah[i] = *reinterpret_cast<const bf16x8_t*>(Ab + 4 * swz16(r, 2 * ch));
      f.al[i] = *reinterpret_cast<const bf16x8_t*>(Ab + 4 * swz16(r, 2 * ch + 1));
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int r = wn * WTN + j * 32 + rl;
      f.bh[j] = *reinterpret_cast<const bf16x8_t*>(Bb + 4 * swz16(r, 2 * ch));
      f.bl[j] = *reinterpret_cast<const bf16x8_t*>(Bb + 4 * swz16(r, 2 * ch + 1));
    }
  };
  // the same of the last k tile, whose chunks lie 'back' places on; zeros past K (its addresses are
  // worked out there, not kept through the loop)
  auto tail = [&](const float* Ab, const float* Bb, int st, Frags& f) {
    const int id = hidden(tid), rl = id & 31, wm = (id >> 6) / WN, wn = (id >> 6) % WN;
    const int ch = 2 * st + ((id >> 5) & 1), at = min(ch + back, 3);
    const bool in = ch < left;
    const bf16x8_t none = {};
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int r = wm * WTM + i * 32 + rl;
      const bf16x8_t h = *reinterpret_cast<const bf16x8_t*>(Ab + 4 * swz16(r, 2 * at));
      const bf16x8_t l = *reinterpret_cast<const bf16x8_t*>(Ab + 4 * swz16(r, 2 * at + 1));
      f.ah[i] = in ? h : none;
      f.al[i] = in ? l : none;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int r = wn * WTN + j * 32 + rl;
      const bf16x8_t h = *reinterpret_cast<const bf16x8_t*>(Bb + 4 * swz16(r, 2 * at));
      const bf16x8_t l = *reinterpret_cast<const bf16x8_t*>(Bb + 4 * swz16(r, 2 * at + 1));
      f.bh[j] = in ? h : none;
      f.bl[j] = in ? l : none;
    }
  };
  // per column block: the hi-lo products of its row blocks, then lo-hi, then hi-hi
  // (consecutive MFMAs accumulate into different blocks, each element still sums hl, lh, hh
  // in that order, and a column block's B fragments die once it is done)
  auto mma = [&](const Frags& f) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[i], f.bl[j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.al[i], f.bh[j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[i], f.bh[j], acc[i][j], 0, 0, 0);
    }
  };
  // issue order pinned: one step's MFMAs with the next step's fragment reads between them
  auto interleave = [&]() {
    constexpr int R = 2 * (TM + TN), Mf = 3 * TM * TN, P = R < Mf ? R : Mf;
#pragma unroll
    for (int n = 0; n < P; ++n) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    if constexpr (Mf > P) __builtin_amdgcn_sched_group_barrier(0x008, Mf - P, 0);
    if constexpr (R > P) __builtin_amdgcn_sched_group_barrier(0x100, R - P, 0);
  };
  // A k tile is two 16-value steps, and its one barrier stands between them: the fragments of a
  // tile's second step are read during the MFMAs of its first, those of the next tile's first
  // step during the MFMAs of its second (its loads into LDS, issued a whole tile earlier, are
  // waited for at the barrier), and the buffer that the barrier frees is refilled at once.  So
  // no MFMA waits for a read that was not issued a step earlier: with the barrier at the end of
  // the tile, both waves of a SIMD read 12 fragments each with the matrix cores idle (768 cycles
  // of LDS time in every 3100 of MFMA time).  Measured on the amplitude contraction at
  // 128/512/1536 (33792 x 24576 x 65536): matrix units busy 60 -> 80 % of the active cycles and
  // 259 -> 236 ms a launch (420 -> 461 TF/s).  The clock falls from 1.97 to 1.65 GHz as they fill
  // (2.4 nominal): the launch is bound by power, as the library's bf16 product is (1323 TF/s at
  // 16384^3, 441 per three products).
  constexpr int kWaitAll = 0x0F70;  // vmcnt(0), other counters left alone (gfx9 s_waitcnt encoding)
  auto reduce = [&](auto whole) {
    Frags f0, f1;
    fill(As0, Bs0, 0, whole);
    __builtin_amdgcn_s_waitcnt(kWaitAll);
    __syncthreads();
    if (nkt > 1) fill(As1, Bs1, 1, whole);
    frags(As0, Bs0, 0, f0);
    auto step = [&](float* Ac, float* Bc, const float* An, const float* Bn, int kt) {
      frags(Ac, Bc, 1, f1);
      mma(f0);
      interleave();
      __builtin_amdgcn_s_waitcnt(kWaitAll);
      __syncthreads();
      if (kt + 2 < nkt) fill(Ac, Bc, kt + 2, whole);
      frags(An, Bn, 0, f0);
      mma(f1);
      interleave();
    };
    for (int kt = 0; kt + 1 < nkt; kt += 2) {
      step(As0, Bs0, As1, Bs1, kt);
      if (kt + 2 < nkt) step(As1, Bs1, As0, Bs0, kt + 1);
    }
  };
  if (mrem >= BM && nrem >= BN)
    reduce(std::true_type{});
  else
    reduce(std::false_type{});
  {
    const float *Al = (nkt & 1) ? As0 : As1, *Bl = (nkt & 1) ? Bs0 : Bs1;
    Frags f0, f1;
    tail(Al, Bl, 0, f0);
    tail(Al, Bl, 1, f1);
    mma(f0);
    mma(f1);
  }
  // epilogue: column offsets once per thread, row offsets once per accumulator row
  const bool mapped = (d.cRm | d.cRn) != 0;
  long coff[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = n0 + wn * WTN + j * 32 + rl;
    coff[j] = col < d.N ? (mapped ? c_index(col + d.cBn, d.cRn, d.cSn, 1) : (long)col) : -1;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = m0 + wm * WTM + i * 32 + row32(lane, r);
      if (row >= d.M) continue;
      const long ro = mapped ? c_index(row, d.cRm, d.cSm, d.ldc) : (long)row * d.ldc;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (coff[j] < 0) continue;
        float* cp = C + ro + coff[j];
        float out = alpha * acc[i][j][r];
        if (beta != 0.0f) out += beta * (*cp);
        *cp = out;
      }
    }
}

// In-place split of n / 8 chunks of 8 FP32 values into the chunk layout above.
__global__ void split_sbf16_kernel(long nchunks, float* __restrict__ x) {
  for (long c = blockIdx.x * (long)blockDim.x + threadIdx.x; c < nchunks; c += (long)gridDim.x * blockDim.x) {
    const f32x4_t* p = reinterpret_cast<const f32x4_t*>(x + 8 * c);
    const f32x4_t a = p[0], b = p[1];
    const float w[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    store_sbf16_chunk(w, x + 8 * c);
  }
}

}  // namespace

int gemm_auto_splitk(const GemmDesc& d, size_t ws_bytes, bool fp32) {
  if (d.splitk > 0) return d.splitk;
  const bool big = d.M >= 96 && d.N >= 96 && d.tile != 64;
  const int BM = big ? 128 : 64, BN = BM;
  const long ntiles = (long)((d.M + BM - 1) / BM) * ((d.N + BN - 1) / BN);
  const long nbatch = (long)d.nb1 * d.nb2;
  const long total = (long)d.KB * ((d.K + 15) / 16);
  const size_t per = (size_t)d.M * d.N * nbatch * (fp32 ? sizeof(float) : sizeof(double));
  return auto_splitk(ntiles * nbatch, total, per, ws_bytes);
}

void gemm_sbf16(const GemmDesc& d, float alpha, const float* A, const float* B, float beta, float* C, hipStream_t s,
                bool amplitude) {
  if (d.M <= 0 || d.N <= 0) return;
  if (d.K <= 0) throw InvalidArg("gemm: empty reduction");
  if (d.transA != 0 || d.transB == 0 || d.KB != 1 || d.nb1 != 1 || d.nb2 != 1)
    throw InvalidArg("split-BF16 GEMM: operands contiguous along k, no batch or outer reduction");
  if (d.lda % 8 || d.ldb % 8 || d.lda < d.K || d.ldb < d.K || (uintptr_t)A % 16 || (uintptr_t)B % 16)
    throw InvalidArg("split-BF16 GEMM: operand rows must start on 32-byte chunks (leading dimensions a multiple "
                     "of 8 values and at least K, 16-byte aligned operands)");
  if (d.M >= 96 && d.N >= 96) {
    // 256 x 256 tiles (8 waves of 64 x 128, one workgroup per CU: 453 TF/s measured on a
    // 8192 x 65536 x 32768 product) against 128 x 128 (4 waves of 64 x 64, two per CU:
    // 386 TF/s): each round of resident 256-tiles holds twice the work of a round of
    // 128-tiles and runs about 1.05 times faster per flop, so the larger tile is taken
    // when its whole rounds finish first
    const long t256 = d.sym >= 0 ? sym_tiles<256, 256>(d) : (long)((d.M + 255) / 256) * ((d.N + 255) / 256);
    const long t128 = d.sym >= 0 ? sym_tiles<128, 128>(d) : (long)((d.M + 127) / 128) * ((d.N + 127) / 128);
    const double r256 = (double)((t256 + kCUs - 1) / kCUs), r128 = (double)((t128 + 2 * kCUs - 1) / (2 * kCUs));
    if (d.tile == 256 || (d.tile != 128 && r256 * 2.0 / 1.05 < r128)) {
      checked_workgroups<256, 256, kSbBK>(d);
      const long wgs = t256;
      if (amplitude)
        gemm_sbf16_kernel<256, 256, 4, 2, 1, 1><<<dim3((unsigned)wgs), 512, 0, s>>>(d, alpha, A, B, beta, C);
      else
        gemm_sbf16_kernel<256, 256, 4, 2, 1><<<dim3((unsigned)wgs), 512, 0, s>>>(d, alpha, A, B, beta, C);
    } else {
      checked_workgroups<128, 128, kSbBK>(d);
      const long wgs = t128;
      if (amplitude)
        gemm_sbf16_kernel<128, 128, 2, 2, 2, 1><<<dim3((unsigned)wgs), kThreads, 0, s>>>(d, alpha, A, B, beta, C);
      else
        gemm_sbf16_kernel<128, 128, 2, 2, 2><<<dim3((unsigned)wgs), kThreads, 0, s>>>(d, alpha, A, B, beta, C);
    }
  } else {
    const long wgs = checked_workgroups<64, 64, kSbBK>(d);
    GemmDesc f = d;
    f.sym = -1;  // too small to be worth leaving tiles out
    gemm_sbf16_kernel<64, 64, 2, 2, 2><<<dim3((unsigned)wgs), kThreads, 0, s>>>(f, alpha, A, B, beta, C);
  }
  PPW_LAUNCH_CHECK();
}

void split_sbf16(long n, float* x, hipStream_t s) {
  if (n <= 0) return;
  if (n % 8 || (uintptr_t)x % 16) throw InvalidArg("split_sbf16: a whole number of 8-value chunks, 16-byte aligned");
  const long chunks = n / 8;
  const int blocks = (int)std::max<long>(1, std::min<long>((chunks + 255) / 256, 65536));
  split_sbf16_kernel<<<blocks, 256, 0, s>>>(chunks, x);
  PPW_LAUNCH_CHECK();
}

int gemm_group_f64(const std::vector<GemmCall<double>>& calls, hipStream_t s) { return gemm_group_impl(calls, s); }
int gemm_group_f32(const std::vector<GemmCall<float>>& calls, hipStream_t s) { return gemm_group_impl(calls, s); }

void gemm_f64(const GemmDesc& d, double alpha, const double* A, const double* B, double beta, double* C,
              hipStream_t s, Workspace ws) {
  gemm_dispatch<double>(d, alpha, A, B, beta, C, s, ws);
}

void gemm_f64_hhat(const GemmDesc& d, double alpha, const double* A, const double* B, double beta, double* C,
                   hipStream_t s, Workspace ws) {
  gemm_dispatch<double, 1>(d, alpha, A, B, beta, C, s, ws);
}

void gemm_f32_hhat(const GemmDesc& d, float alpha, const float* A, const float* B, float beta, float* C,
                   hipStream_t s, Workspace ws) {
  gemm_dispatch<float, 1>(d, alpha, A, B, beta, C, s, ws);
}

void gemm_f32(const GemmDesc& d, float alpha, const float* A, const float* B, float beta, float* C,
              hipStream_t s, Workspace ws) {
  gemm_dispatch<float>(d, alpha, A, B, beta, C, s, ws);
}

}  // namespace ppw
