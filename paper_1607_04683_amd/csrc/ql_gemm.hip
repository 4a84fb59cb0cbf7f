// ql_gemm.hip -- 8-bit matrix products of Section 3.1 (eq. 1) on gfx950 MFMA.
//
// C[m][n] = sum_k X'[m][k] W'[n][k] with both operands K-contiguous.  Codes
// are stored as signed bytes s = V' - 128 so the signed int8 MFMA
// (v_mfma_i32_32x32x32_i8) applies directly; the exact zero-point terms of
// eq. 1 are added in the epilogue from per-row / per-column code sums, and the
// product is recovered to fp32 there (Fig. 1: R(Mult(.)) + B).
//
// Tiling: a workgroup of WM x WN wavefronts computes a BM x BN tile; each
// wavefront owns a (BM/WM) x (BN/WN) sub-tile built from 32x32 MFMA blocks.
// K advances in steps of BK bytes through two LDS stages (global -> VGPR ->
// LDS, one barrier per step); LDS rows are padded by 16 bytes so the 16-byte
// fragment reads of 32 consecutive rows spread over all banks.
#include "ql_device.h"
#include "ql_launch.h"
#include "ql_quant_rows.h"

namespace ql {

typedef float v4f __attribute__((ext_vector_type(4)));

enum { EPI_RECOVER = 0, EPI_RAW = 1, EPI_SMAX_STATS = 2, EPI_SMAX_OUT = 3 };

struct EpiArgs {
  // row (X) side
  const int32_t *x_zero;
  const float *x_inv_q;
  const int32_t *x_sums;
  // column (W) side
  const int32_t *w_zero;
  const float *w_inv_q;
  const int32_t *w_sums;
  int64_t w_rpb;
  const float *bias;
  // outputs
  float *Y;
  int32_t *acc;
  float *logits;
  float2 *stats;  // [M][ntn] (max, sum exp) per column tile
  int ntn;
  const float2 *rowstat;  // [M] (max, 1 / sum exp) per row
  bool past;              // Y is stored past the caches (see stored_past)
};

template <int BM, int BN, int BK, int WM, int WN>
struct Cfg {
  static constexpr int NT = 64 * WM * WN;
  static constexpr int TM = BM / WM, TN = BN / WN;
  static constexpr int FM = TM / 32, FN = TN / 32;
  static constexpr int LDSS = BK + 16;  // padded LDS row stride in bytes
  static constexpr int STAGE = (BM + BN) * LDSS;
  static constexpr int LDS = 2 * STAGE;
  static constexpr int CPR = BK / 16;   // 16-byte chunks per row
  static constexpr int LA = BM * CPR / NT, LB = BN * CPR / NT;
  static_assert(BM * CPR % NT == 0 && BN * CPR % NT == 0, "tile/threads mismatch");
  static_assert(TM % 32 == 0 && TN % 32 == 0, "wave tile must be a multiple of 32");
};

template <int BM, int BN, int BK, int WM, int WN>
__device__ __forceinline__ void gemm_tile(const int8_t *__restrict__ A, int64_t lda,
                                          const int8_t *__restrict__ B, int64_t ldb, int64_t M,
                                          int64_t N, int64_t Kp, int64_t m0, int64_t n0,
                                          char *smem, v16i (&acc)[Cfg<BM, BN, BK, WM, WN>::FM]
                                                                 [Cfg<BM, BN, BK, WM, WN>::FN]) {
  using C = Cfg<BM, BN, BK, WM, WN>;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j) acc[i][j] = v16i{};

  // global source offsets and LDS destinations of this thread's 16-byte chunks
  int64_t oa[C::LA], ob[C::LB];
  int sa[C::LA], sb[C::LB];
#pragma unroll
  for (int i = 0; i < C::LA; ++i) {
    const int c = tid + i * C::NT, r = c / C::CPR, kc = c % C::CPR;
    int64_t gr = m0 + r;
    gr = gr < M ? gr : M - 1;
    oa[i] = gr * lda + kc * 16;
    sa[i] = r * C::LDSS + kc * 16;
  }
#pragma unroll
  for (int i = 0; i < C::LB; ++i) {
    const int c = tid + i * C::NT, r = c / C::CPR, kc = c % C::CPR;
    int64_t gr = n0 + r;
    gr = gr < N ? gr : N - 1;
    ob[i] = gr * ldb + kc * 16;
    sb[i] = BM * C::LDSS + r * C::LDSS + kc * 16;
  }
  const int nk = (int)(Kp / BK);
  v4i ra[C::LA], rb[C::LB];
  if (nk > 0) {
#pragma unroll
    for (int i = 0; i < C::LA; ++i) ra[i] = *reinterpret_cast<const v4i *>(A + oa[i]);
#pragma unroll
    for (int i = 0; i < C::LB; ++i) rb[i] = *reinterpret_cast<const v4i *>(B + ob[i]);
#pragma unroll
    for (int i = 0; i < C::LA; ++i) *reinterpret_cast<v4i *>(smem + sa[i]) = ra[i];
#pragma unroll
    for (int i = 0; i < C::LB; ++i) *reinterpret_cast<v4i *>(smem + sb[i]) = rb[i];
  }
  __syncthreads();
  const int frow = lane & 31, fk = (lane >> 5) * 16;
  for (int kt = 0; kt < nk; ++kt) {
    const bool more = kt + 1 < nk;
    if (more) {
      const int64_t ko = (int64_t)(kt + 1) * BK;
#pragma unroll
      for (int i = 0; i < C::LA; ++i) ra[i] = *reinterpret_cast<const v4i *>(A + oa[i] + ko);
#pragma unroll
      for (int i = 0; i < C::LB; ++i) rb[i] = *reinterpret_cast<const v4i *>(B + ob[i] + ko);
    }
    const char *base = smem + (kt & 1) * C::STAGE;
#pragma unroll
    for (int ks = 0; ks < BK / 32; ++ks) {
      v4i af[C::FM], bf[C::FN];
#pragma unroll
      for (int i = 0; i < C::FM; ++i)
        af[i] = *reinterpret_cast<const v4i *>(base + (wm * C::TM + i * 32 + frow) * C::LDSS +
                                               ks * 32 + fk);
#pragma unroll
      for (int j = 0; j < C::FN; ++j)
        bf[j] = *reinterpret_cast<const v4i *>(base + BM * C::LDSS +
                                               (wn * C::TN + j * 32 + frow) * C::LDSS + ks * 32 +
                                               fk);
#pragma unroll
      for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[i], bf[j], acc[i][j], 0, 0, 0);
    }
    if (more) {
      char *nb = smem + ((kt + 1) & 1) * C::STAGE;
#pragma unroll
      for (int i = 0; i < C::LA; ++i) *reinterpret_cast<v4i *>(nb + sa[i]) = ra[i];
#pragma unroll
      for (int i = 0; i < C::LB; ++i) *reinterpret_cast<v4i *>(nb + sb[i]) = rb[i];
    }
    __syncthreads();
  }
}

// Deeper pipeline for large tiles: K advances ROW bytes (64 or 128) per step
// through NS LDS stages filled by direct global->LDS loads (no VGPR
// staging).  Chunk c (16 bytes) of row r of a stage sits in slot
// c ^ swz(r), which keeps the 16-byte fragment reads of 32 consecutive rows
// free of bank conflicts (any 8 aligned rows, and the even and the odd rows
// of any 16 aligned rows, take distinct slots).  swz uses only bits 0..4 of
// the row, so a fragment's swizzle follows from lane & 31 alone.
typedef __attribute__((address_space(3))) void lds_void;

// One 16-byte direct global->LDS load (each lane's 16 bytes land at
// consecutive 16-byte slots from the wave's LDS base).  A plain function so
// that every kernel instantiation shares one declaration of the builtin call.
__device__ __forceinline__ void load_lds16(const int8_t *g, char *l) {
  __builtin_amdgcn_global_load_lds(g, (lds_void *)l, 16, 0, 0);
}

template <int ROW>
__device__ __forceinline__ int swz(int r) {
  if constexpr (ROW == 64) return ((r >> 1) ^ (r >> 2)) & 3;
  else return (r & 7) ^ ((r >> 3) & 1);
}

// s_waitcnt with only the vector-memory count limited (gfx9 encoding:
// vmcnt in bits 3:0 and 15:14, expcnt 6:4 and lgkmcnt 11:8 left at maximum)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

__device__ __forceinline__ void wait_lgkmcnt0() {
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));
}

template <int BM, int BN, int WM, int WN, int ROW, int NS>
struct CfgDma {
  static constexpr int NT = 64 * WM * WN;
  static constexpr int TBM = BM, TBN = BN;
  static constexpr int TM = BM / WM, TN = BN / WN;
  static constexpr int FM = TM / 32, FN = TN / 32;
  static constexpr int CPR = ROW / 16;           // 16-byte chunks per row
  static constexpr int STAGE = (BM + BN) * ROW;
  static constexpr int LDS = NS * STAGE;
  static constexpr int LA = BM * CPR / NT, LB = BN * CPR / NT;  // loads per thread
  static_assert(ROW == 64 || ROW == 128, "row of 64 or 128 bytes");
  static_assert(BM * CPR % NT == 0 && BN * CPR % NT == 0, "tile/threads mismatch");
  static_assert(NS >= 2, "pipeline needs two stages");
};

template <int BM, int BN, int WM, int WN, int ROW, int NS>
__device__ __forceinline__ void gemm_tile_dma(
    const int8_t *__restrict__ A, int64_t lda, const int8_t *__restrict__ B, int64_t ldb, int64_t M,
    int64_t N, int64_t Kp, int64_t m0, int64_t n0, char *smem,
    v16i (&acc)[CfgDma<BM, BN, WM, WN, ROW, NS>::FM][CfgDma<BM, BN, WM, WN, ROW, NS>::FN]) {
  using C = CfgDma<BM, BN, WM, WN, ROW, NS>;
  constexpr int CPR = C::CPR, Q = ROW / 32;  // Q sub-steps of 32 bytes of K
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j) acc[i][j] = v16i{};

  // Load i of this thread fills LDS slot p = i * NT + tid of the A (or B)
  // region: row p / CPR, slot p % CPR, holding global chunk
  // (p % CPR) ^ swz(row).  Each wave's load instruction covers 1 KB of
  // consecutive slots.
  const int8_t *ga[C::LA], *gb[C::LB];
#pragma unroll
  for (int i = 0; i < C::LA; ++i) {
    const int p = i * C::NT + tid, r = p / CPR, c = (p % CPR) ^ swz<ROW>(r);
    int64_t gr = m0 + r;
    gr = gr < M ? gr : M - 1;
    ga[i] = A + gr * lda + c * 16;
  }
#pragma unroll
  for (int i = 0; i < C::LB; ++i) {
    const int p = i * C::NT + tid, r = p / CPR, c = (p % CPR) ^ swz<ROW>(r);
    int64_t gr = n0 + r;
    gr = gr < N ? gr : N - 1;
    gb[i] = B + gr * ldb + c * 16;
  }
  const int nk = (int)(Kp / ROW);
  // Load i (of LA + LB) of step `ks` into its stage; steps past the end
  // reload the last step into a stage that is never read again, so every
  // step has the same number of loads in flight.
  auto load_one = [&](int ks, int i) {
    const int64_t ko = (int64_t)(ks < nk ? ks : nk - 1) * ROW;
    char *st = smem + (ks % NS) * C::STAGE + wave * 1024;
    if (i < C::LA)
      load_lds16(ga[i] + ko, st + i * C::NT * 16);
    else
      load_lds16(gb[i - C::LA] + ko, st + BM * ROW + (i - C::LA) * C::NT * 16);
  };
  if (nk == 0) return;

  // Fragment q of a sub-step: A fragments 0..FM-1, then B fragments.  A
  // fragment i of sub-step h is rows wm*TM + i*32 + (lane & 31), chunk
  // 2*h + (lane >> 5); swz depends only on lane & 31 here.
  const int fr = lane & 31, fsw = swz<ROW>(fr), fhi = lane >> 5;
  const int offa = (wm * C::TM + fr) * ROW, offb = BM * ROW + (wn * C::TN + fr) * ROW;
  constexpr int NMF = C::FM * C::FN, NRD = C::FM + C::FN, NLD = C::LA + C::LB;
  constexpr int SLOTS = NMF - NRD;  // load slots per sub-step
  static_assert(Q % 2 == 0, "sub-steps alternate between two fragment sets");
  static_assert(SLOTS > 0 && NLD <= Q * SLOTS, "not enough MFMAs to cover the memory ops");
  v4i f0[NRD], f1[NRD];
  auto read_one = [&](int ks, int h, int q, v4i &dst) {
    const char *st = smem + (ks % NS) * C::STAGE + ((2 * h + fhi) ^ fsw) * 16;
    dst = *reinterpret_cast<const v4i *>(st + (q < C::FM ? offa + q * 32 * ROW
                                                         : offb + (q - C::FM) * 32 * ROW));
  };
  auto mfma_one = [&](const v4i(&f)[NRD], int q) {
    const int i = q / C::FN, j = q % C::FN;
    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f[i], f[C::FM + j], acc[i][j], 0, 0, 0);
  };
  // One sub-step: the MFMAs on `cur`, with the next sub-step's fragment
  // reads into `nxt` and loads [l0, l0 + SLOTS) of step `lks` threaded one
  // per MFMA; the scheduling barriers hold that order so the matrix pipe
  // never waits on a memory instruction.
  auto substep = [&](const v4i(&cur)[NRD], v4i(&nxt)[NRD], int rks, int rh, int lks, int l0) {
#pragma unroll
    for (int q = 0; q < NMF; ++q) {
      mfma_one(cur, q);
      if (q < NRD) read_one(rks, rh, q, nxt[q]);
      else if (lks >= 0 && l0 + q - NRD < NLD) load_one(lks, l0 + q - NRD);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  for (int ks = 0; ks < NS; ++ks)
#pragma unroll
    for (int i = 0; i < NLD; ++i) load_one(ks, i);
  wait_vmcnt<(NS - 1) * NLD>();
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NRD; ++q) read_one(0, 0, q, f0[q]);
  wait_lgkmcnt0();
  // Step kt+NS-1 is loaded from the last sub-step of step kt-1 on (the
  // prologue loaded steps 0..NS-1).
  for (int kt = 0; kt < nk; ++kt) {
    const int lprev = kt > 0 ? kt + NS - 1 : -1;
#pragma unroll
    for (int h = 0; h < Q - 1; ++h) {
      if (h % 2 == 0) substep(f0, f1, kt, h + 1, lprev, (h + 1) * SLOTS);
      else substep(f1, f0, kt, h + 1, lprev, (h + 1) * SLOTS);
    }
    // Stage kt is fully read into registers and step kt+1 has landed (steps
    // up to kt+NS-1 were issued): after the barrier stage kt's buffer takes
    // step kt+NS.
    wait_vmcnt<(NS - 2) * NLD>();
    __syncthreads();
    substep(f1, f0, kt + 1, 0, kt + NS, 0);
    // the fragments just read landed while the MFMAs above issued; saying so
    // keeps the LDS counter (15 at most) from forcing a full wait on the
    // next sub-step's reads
    wait_lgkmcnt0();
  }
  wait_vmcnt<0>();
  __syncthreads();
}

// Tile of this (1-D) workgroup.  Workgroups are dealt round-robin to the 8
// XCDs; when the tile count allows, XCD x is given the x-th contiguous eighth
// of the tile order, and that order walks groups of 8 tile rows column by
// column, so the workgroups sharing an L2 also share A and B panels.
__device__ __forceinline__ void tile_of_block(int64_t M, int64_t N, int BM, int BN, int *tm, int *tn) {
  const int ntm = (int)((M + BM - 1) / BM), ntn = (int)((N + BN - 1) / BN);
  const int ntiles = ntm * ntn;
  int bid = blockIdx.x;
  if (ntiles % 8 == 0) bid = (bid % 8) * (ntiles / 8) + bid / 8;
  constexpr int kGroup = 8;
  const int group = bid / (kGroup * ntn);
  const int first = group * kGroup;
  const int gsize = ntm - first < kGroup ? ntm - first : kGroup;
  const int in_group = bid % (kGroup * ntn);
  *tm = first + in_group % gsize;
  *tn = in_group / gsize;
}

// Row/column of element r of a 32x32 MFMA block held by `lane`.
__device__ __forceinline__ int frag_row(int r, int lane) { return ((r >> 2) << 3) + ((lane >> 5) << 2) + (r & 3); }
__device__ __forceinline__ int frag_col(int lane) { return lane & 31; }

// Integer accumulators through LDS: each wave turns 32 rows of its
// accumulators at a time into V'-domain sums (eq. 1 with the code sums) and
// parks them row-major in its own LDS slab (row stride 136 words: the two
// half-waves of a store land on disjoint banks), then stores whole rows with
// 16-byte writes.  The tile's row sums are staged once.  The K loop has left
// LDS idle (its last barrier follows the final wait for loads).
template <class C>
__device__ __forceinline__ void raw_epilogue_lds(const EpiArgs &e, int64_t M, int64_t N, int64_t K,
                                                 int64_t m0, int64_t n0, int wm, int wn, int lane,
                                                 char *smem, v16i (&acc)[C::FM][C::FN]) {
  constexpr int TM = C::TM, TN = C::TN, RS = TN + 8;  // row stride in words
  static_assert(TN % 4 == 0 && (RS * 4) % 16 == 0, "16-byte rows");
  static_assert(C::TBM * 4 <= 4096 && 4096 + (C::NT / 64) * 32 * RS * 4 <= C::LDS, "LDS slabs");
  uint32_t *rterm = reinterpret_cast<uint32_t *>(smem);  // [BM]: 128 * sigma_x
  const int wave = threadIdx.x >> 6;
  uint32_t *slab = reinterpret_cast<uint32_t *>(smem + 4096) + wave * 32 * RS;
  for (int r = threadIdx.x; r < C::TBM; r += C::NT) {
    const int64_t m = m0 + r;
    rterm[r] = m < M ? 128u * (uint32_t)(e.x_sums[m] - 128 * (int32_t)K) : 0u;
  }
  uint32_t cterm[C::FN];
#pragma unroll
  for (int j = 0; j < C::FN; ++j) {
    int64_t n = n0 + wn * TN + j * 32 + (lane & 31);
    n = n < N ? n : N - 1;
    cterm[j] = 128u * (uint32_t)(e.w_sums[n] - 128 * (int32_t)K) + 16384u * (uint32_t)K;
  }
  __syncthreads();
  const bool vec = (N & 3) == 0;
#pragma unroll
  for (int i = 0; i < C::FM; ++i) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = frag_row(r, lane);
      const uint32_t rt = rterm[wm * TM + i * 32 + row];
#pragma unroll
      for (int j = 0; j < C::FN; ++j)
        slab[row * RS + j * 32 + (lane & 31)] = (uint32_t)acc[i][j][r] + cterm[j] + rt;
    }
    // the slab is this wave's own: LDS keeps one wave's accesses in order
#pragma unroll
    for (int it = 0; it < 32 * TN / 256; ++it) {
      const int q = it * 64 + lane, row = q / (TN / 4), c4 = (q % (TN / 4)) * 4;
      const v4i v = *reinterpret_cast<const v4i *>(slab + row * RS + c4);
      const int64_t m = m0 + wm * TM + i * 32 + row, n = n0 + wn * TN + c4;
      if (m < M) {
        int32_t *dst = e.acc + m * N + n;
        if (vec && n + 3 < N) {
          *reinterpret_cast<v4i *>(dst) = v;
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (n + t < N) dst[t] = v[t];
        }
      }
    }
  }
}

// Calls f(integral_constant<int, I>) for I in [B, E).
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// N independent reductions (max or sum) over each group of L lanes (32: a
// half-wave, 16: one DPP row): rotations within 16-lane rows, then for 32
// the exchange of the two rows.
template <bool MAX, int L, int N>
__device__ __forceinline__ void row_reduce(float (&v)[N]) {
  static_assert(L == 16 || L == 32, "16 or 32 lanes");
  auto op = [](float a, float b) { return MAX ? fmaxf(a, b) : a + b; };
  auto ror = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value,
                                                      0xf, 0xf, false));
  };
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = op(v[k], ror(v[k], std::integral_constant<int, 0x128>{}));
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = op(v[k], ror(v[k], std::integral_constant<int, 0x124>{}));
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = op(v[k], ror(v[k], std::integral_constant<int, 0x122>{}));
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = op(v[k], ror(v[k], std::integral_constant<int, 0x121>{}));
  if constexpr (L == 32) {
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = op(v[k], __shfl_xor(v[k], 16, 64));
  }
}

// Recovering epilogues (eq. 1 recovery plus bias; softmax statistics or
// output) through LDS: each wave parks 32 rows of raw signed sums at a time in
// its own slab (as above), then walks them row-major with every lane owning
// the same 4 consecutive columns of each row, so the per-column terms stay in
// registers and every store is a 16-byte write.  The tile's per-row terms are
// staged once.  Softmax statistics are reduced per wave over its TN columns
// (max, then sum of exp(y - max)) and the WN partials of a row are merged
// with the usual rescaling.
template <class C, int EPI, bool PAST>
__device__ __forceinline__ void recover_epilogue_lds(const EpiArgs &e, int64_t M, int64_t N,
                                                     int64_t K, int64_t m0, int64_t n0, int tn,
                                                     int wm, int wn, int lane, char *smem,
                                                     const float *rowmax, const float *rowinv,
                                                     v16i (&acc)[C::FM][C::FN]) {
  constexpr int BM = C::TBM, TM = C::TM, TN = C::TN, RS = TN + 8, WN = C::TBN / C::TN;
  // LPR lanes cover one row of the wave's TN columns, 4 columns each; a wave
  // covers RPI rows per iteration, NIT iterations per 32-row chunk
  constexpr int LPR = TN / 4, RPI = 64 / LPR, NIT = 32 / RPI;
  static_assert(TN == 128 || TN == 64, "32 or 16 lanes per row");
  constexpr int kSlab = (3 * BM * 4 + WN * BM * 8 + 4095) / 4096 * 4096;
  static_assert(kSlab + (C::NT / 64) * 32 * RS * 4 <= C::LDS, "LDS slabs");
  int32_t *rsig = reinterpret_cast<int32_t *>(smem);  // [BM] sigma_x
  int32_t *rzt = rsig + BM;                            // [BM] z~x
  float *riq = reinterpret_cast<float *>(rzt + BM);    // [BM] 1/Qx
  float2 *red = reinterpret_cast<float2 *>(smem + 3 * BM * 4);  // [WN][BM] (max, sum)
  const int wave = threadIdx.x >> 6;
  uint32_t *slab = reinterpret_cast<uint32_t *>(smem + kSlab) + wave * 32 * RS;
  bool fast = true;  // every row and column of the tile on recover()'s fast path
  for (int r = threadIdx.x; r < BM; r += C::NT) {
    int64_t m = m0 + r;
    m = m < M ? m : M - 1;
    rsig[r] = e.x_sums[m] - 128 * (int32_t)K;
    rzt[r] = e.x_zero[m] + 128;
    riq[r] = e.x_inv_q[m];
    fast = fast && fast_row(rzt[r]);
  }
  // this lane's columns: n0 + wn*TN + 4*(lane % LPR) + t
  const int64_t nc = n0 + wn * TN + 4 * (lane % LPR);
  int32_t ztw[4], sigw[4];
  int64_t colterm[4];
  float iqw[4], bn[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int64_t nn = nc + t < N ? nc + t : N - 1;
    const int64_t blk = nn / e.w_rpb;
    ztw[t] = e.w_zero[blk] + 128;
    sigw[t] = e.w_sums[nn] - 128 * (int32_t)K;
    colterm[t] = (int64_t)sigw[t] + K * (int64_t)ztw[t];
    iqw[t] = e.w_inv_q[blk];
    bn[t] = e.bias ? e.bias[nn] : 0.0f;
    fast = fast && fast_col(ztw[t], colterm[t]);
  }
  fast = __syncthreads_and(fast);
  int32_t colt32[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) colt32[t] = (int32_t)colterm[t];
  const bool vec = (N & 3) == 0 && nc + 3 < N;
  // chunks expanded at compile time: acc is only ever indexed by constants
  static_for<0, C::FM>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = frag_row(r, lane);
#pragma unroll
      for (int j = 0; j < C::FN; ++j) slab[row * RS + j * 32 + (lane & 31)] = (uint32_t)acc[i][j][r];
    }
    // the slab is this wave's own: LDS keeps one wave's accesses in order
    // row `it` of this half-wave: recover, store, and hand back y
    auto row_step = [&](int it, float (&y)[4]) {
      const int row = RPI * it + lane / LPR, lr = wm * TM + i * 32 + row;
      const int64_t m = m0 + lr;
      const v4i v = *reinterpret_cast<const v4i *>(slab + row * RS + 4 * (lane % LPR));
      const int32_t sigx = rsig[lr], ztx = rzt[lr];
      const float iqx = riq[lr];
      if (fast) {
#pragma unroll
        for (int t = 0; t < 4; ++t) y[t] = recover_fast(v[t], colt32[t], ztw[t], ztx, sigx, iqw[t], iqx) + bn[t];
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) y[t] = recover(v[t], colterm[t], ztw[t], ztx, sigx, iqw[t], iqx) + bn[t];
      }
      const int64_t off = m * N + nc;
      if (EPI == EPI_RECOVER || EPI == EPI_SMAX_OUT) {
        if (EPI == EPI_SMAX_OUT) {
          const float mx = rowmax[lr], inv = rowinv[lr];
#pragma unroll
          for (int t = 0; t < 4; ++t) y[t] = __expf(y[t] - mx) * inv;
        }
        if (m < M) {
          if (vec) {
            const v4f v = {y[0], y[1], y[2], y[3]};
            if constexpr (PAST) __builtin_nontemporal_store(v, reinterpret_cast<v4f *>(e.Y + off));
            else *reinterpret_cast<v4f *>(e.Y + off) = v;
          } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
              if (nc + t < N) e.Y[off + t] = y[t];
          }
        }
      } else if (m < M && e.logits) {  // EPI_SMAX_STATS
        if (vec) {
          *reinterpret_cast<float4 *>(e.logits + off) = make_float4(y[0], y[1], y[2], y[3]);
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (nc + t < N) e.logits[off + t] = y[t];
        }
      }
      if (EPI != EPI_SMAX_OUT && m < M && e.acc) {
        int32_t a[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = acc_u8(v[t], sigw[t], sigx, K);
        if (vec) {
          *reinterpret_cast<v4i *>(e.acc + off) = v4i{a[0], a[1], a[2], a[3]};
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (nc + t < N) e.acc[off + t] = a[t];
        }
      }
    };
    if constexpr (EPI != EPI_SMAX_STATS) {
#pragma unroll 2
      for (int it = 0; it < NIT; ++it) {
        float y[4];
        row_step(it, y);
      }
    } else {
      float ys[NIT][4];
#pragma unroll
      for (int it = 0; it < NIT; ++it) row_step(it, ys[it]);
      // per row (one per LPR lanes and iteration): max over the wave's TN
      // columns, then sum exp(y - max); NIT rows reduced together so the
      // steps overlap
      float mx[NIT], sm[NIT];
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        mx[it] = -INFINITY;
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (nc + t < N) mx[it] = fmaxf(mx[it], ys[it][t]);
      }
      row_reduce<true, LPR>(mx);
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        sm[it] = 0.0f;
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (nc + t < N) sm[it] += __expf(ys[it][t] - mx[it]);
      }
      row_reduce<false, LPR>(sm);
      if (lane % LPR == 0) {
#pragma unroll
        for (int it = 0; it < NIT; ++it)
          red[wn * BM + wm * TM + i * 32 + RPI * it + lane / LPR] = make_float2(mx[it], sm[it]);
      }
    }
  });
  if constexpr (EPI == EPI_SMAX_STATS) {
    __syncthreads();
    for (int r = threadIdx.x; r < BM; r += C::NT) {
      const int64_t m = m0 + r;
      if (m >= M) continue;
      float mx = -INFINITY;
#pragma unroll
      for (int w = 0; w < WN; ++w) mx = fmaxf(mx, red[w * BM + r].x);
      float sm = 0.0f;
#pragma unroll
      for (int w = 0; w < WN; ++w) {
        const float2 p = red[w * BM + r];
        if (p.y > 0.0f) sm += p.y * __expf(p.x - mx);
      }
      e.stats[m * e.ntn + tn] = make_float2(mx, sm);
    }
  }
}

// NS = 0: register-staged two-stage tile; NS >= 2: direct-load pipeline of
// NS stages with BK-byte rows.
template <int BM, int BN, int BK, int WM, int WN, int NS>
using GemmCfg = std::conditional_t<(NS >= 2), CfgDma<BM, BN, WM, WN, BK, (NS >= 2 ? NS : 2)>,
                                   Cfg<BM, BN, BK, WM, WN>>;

template <int BM, int BN, int BK, int WM, int WN, int NS, int EPI>
__global__ __launch_bounds__(64 * WM *WN) void k_gemm(const int8_t *__restrict__ A, int64_t lda,
                                                       const int8_t *__restrict__ B, int64_t ldb,
                                                       int64_t M, int64_t N, int64_t K,
                                                       int64_t Kp, EpiArgs e) {
  using C = GemmCfg<BM, BN, BK, WM, WN, NS>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int tm, tn;
  tile_of_block(M, N, BM, BN, &tm, &tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / WN, wn = wave % WN;

  // softmax output pass: combine the per-tile statistics of this tile's rows
  float *rowmax = reinterpret_cast<float *>(smem + C::LDS);
  float *rowinv = rowmax + BM;
  if (EPI == EPI_SMAX_OUT) {
    for (int r = threadIdx.x; r < BM; r += C::NT) {
      const int64_t m = m0 + r;
      const float2 st = e.rowstat[m < M ? m : M - 1];
      rowmax[r] = st.x;
      rowinv[r] = st.y;
    }
  }

  v16i acc[C::FM][C::FN];
  if constexpr (NS >= 2)
    gemm_tile_dma<BM, BN, WM, WN, BK, NS>(A, lda, B, ldb, M, N, Kp, m0, n0, smem, acc);
  else
    gemm_tile<BM, BN, BK, WM, WN>(A, lda, B, ldb, M, N, Kp, m0, n0, smem, acc);

  if constexpr (NS >= 2) {
    if constexpr (EPI == EPI_RAW)
      raw_epilogue_lds<C>(e, M, N, K, m0, n0, wm, wn, lane, smem, acc);
    else
      if (EPI != EPI_SMAX_STATS && e.past)
        recover_epilogue_lds<C, EPI, EPI != EPI_SMAX_STATS>(e, M, N, K, m0, n0, tn, wm, wn, lane, smem,
                                                            rowmax, rowinv, acc);
      else
        recover_epilogue_lds<C, EPI, false>(e, M, N, K, m0, n0, tn, wm, wn, lane, smem, rowmax, rowinv,
                                            acc);
    return;
  }

  // per-column terms
  int32_t ztw[C::FN], sigw[C::FN];
  int64_t colterm[C::FN];
  float iqw[C::FN], bn[C::FN];
  int64_t ncol[C::FN];
#pragma unroll
  for (int j = 0; j < C::FN; ++j) {
    int64_t n = n0 + wn * C::TN + j * 32 + frag_col(lane);
    ncol[j] = n;
    const int64_t nn = n < N ? n : N - 1;
    if (EPI == EPI_RAW) {
      sigw[j] = e.w_sums[nn] - 128 * (int32_t)K;
      ztw[j] = 0;
      colterm[j] = 0;
      iqw[j] = 0.0f;
      bn[j] = 0.0f;
    } else {
      const int64_t blk = nn / e.w_rpb;
      ztw[j] = e.w_zero[blk] + 128;
      sigw[j] = e.w_sums[nn] - 128 * (int32_t)K;
      colterm[j] = (int64_t)sigw[j] + K * (int64_t)ztw[j];
      iqw[j] = e.w_inv_q[blk];
      bn[j] = e.bias ? e.bias[nn] : 0.0f;
    }
  }

#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int lr = wm * C::TM + i * 32 + frag_row(r, lane);
      const int64_t m = m0 + lr;
      if (m >= M) continue;
      const int32_t sigx = e.x_sums[m] - 128 * (int32_t)K;
      int32_t ztx = 0;
      float iqx = 0.0f;
      if (EPI != EPI_RAW) {
        ztx = e.x_zero[m] + 128;
        iqx = e.x_inv_q[m];
      }
#pragma unroll
      for (int j = 0; j < C::FN; ++j) {
        const int64_t n = ncol[j];
        if (n >= N) continue;
        const int32_t S = acc[i][j][r];
        if (EPI == EPI_RAW) {
          e.acc[m * N + n] = acc_u8(S, sigw[j], sigx, K);
        } else {
          e.Y[m * N + n] = recover(S, colterm[j], ztw[j], ztx, sigx, iqw[j], iqx) + bn[j];
          if (e.acc) e.acc[m * N + n] = acc_u8(S, sigw[j], sigx, K);
        }
      }
    }
}

// The wave's results of few-row products: lane (fr, fq) holds columns nc .. + 3
// (nc = n0 + 4 fq) of rows m0 + 16 b + fr; row(m) gives a row's params.
struct SkinnyRow {
  int32_t zero, sum;
  float inv_q;
};
template <int MB, class RowFn>
__device__ __forceinline__ void skinny_epilogue(const EpiArgs &e, int64_t M, int64_t N, int64_t K,
                                                int64_t m0, int64_t nc, int fr, const v4i (&acc)[MB],
                                                RowFn row) {
  if (nc >= N) return;
  int32_t ztw[4], sigw[4];
  int64_t colterm[4];
  float iqw[4], bn[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int64_t nn = nc + t < N ? nc + t : N - 1;
    const int64_t blk = nn / e.w_rpb;
    ztw[t] = e.w_zero[blk] + 128;
    sigw[t] = e.w_sums[nn] - 128 * (int32_t)K;
    colterm[t] = (int64_t)sigw[t] + K * (int64_t)ztw[t];
    iqw[t] = e.w_inv_q[blk];
    bn[t] = e.bias ? e.bias[nn] : 0.0f;
  }
  const bool vec = (N & 3) == 0;  // rows of Y and acc 16-byte aligned
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const int64_t m = m0 + 16 * b + fr;
    if (m >= M) continue;
    const SkinnyRow r = row(m);
    const int32_t sigx = r.sum - 128 * (int32_t)K, ztx = r.zero + 128;
    const float iqx = r.inv_q;
    float y[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
      y[t] = recover(acc[b][t], colterm[t], ztw[t], ztx, sigx, iqw[t], iqx) + bn[t];
    const int64_t off = m * N + nc;
    if (vec && ((uintptr_t)e.Y & 15) == 0) {
      *reinterpret_cast<float4 *>(e.Y + off) = make_float4(y[0], y[1], y[2], y[3]);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (nc + t < N) e.Y[off + t] = y[t];
    }
    if (e.acc)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (nc + t < N) e.acc[off + t] = acc_u8(acc[b][t], sigw[t], sigx, K);
  }
}

// Products of few rows (or few tiles): W' is what has to be read, so every
// wave takes 16 of its rows, whole, straight into registers as MFMA fragments
// (no LDS, no barrier), against MB 16-row blocks of X, whose codes the waves
// of a CU share through its cache.  Waves, not tiles, fill the chip: N = 8192
// is 512 of them per 16 MB rows, where 128 x 128 tiles are 64 workgroups that
// each wait four times for a 32 KB stage.  The 16 x 16 result leaves a lane
// four neighbouring columns of one row: one 16-byte store.
constexpr int kSkinnyWaves = 2;
template <int MB>
__global__ __launch_bounds__(64 * kSkinnyWaves) void k_gemm_skinny(
    const int8_t *__restrict__ A, int64_t lda, const int8_t *__restrict__ B, int64_t ldb, int64_t M,
    int64_t N, int64_t K, EpiArgs e) {
  const int lane = threadIdx.x & 63, fr = lane & 15, fq = lane >> 4;
  const int64_t n0 = ((int64_t)blockIdx.x * kSkinnyWaves + (threadIdx.x >> 6)) * 16;
  const int64_t m0 = (int64_t)blockIdx.y * 16 * MB;
  if (n0 >= N) return;
  const int64_t wrow = n0 + fr < N ? n0 + fr : N - 1;
  const int8_t *w = B + wrow * ldb + 16 * fq;
  const int8_t *x[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const int64_t m = m0 + 16 * b + fr;
    x[b] = A + (m < M ? m : M - 1) * lda + 16 * fq;
  }
  v4i acc[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) acc[b] = v4i{};
  const int nk = (int)((K + 63) / 64);  // both leading dimensions cover 64 nk
  int c = 0;
  for (; c + 8 <= nk; c += 8) {
    v4i wf[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) wf[k] = *reinterpret_cast<const v4i *>(w + (c + k) * 64);
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int b = 0; b < MB; ++b)
        acc[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
            wf[k], *reinterpret_cast<const v4i *>(x[b] + (c + k) * 64), acc[b], 0, 0, 0);
  }
  for (; c < nk; ++c) {
    const v4i wf = *reinterpret_cast<const v4i *>(w + c * 64);
#pragma unroll
    for (int b = 0; b < MB; ++b)
      acc[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
          wf, *reinterpret_cast<const v4i *>(x[b] + c * 64), acc[b], 0, 0, 0);
  }
  skinny_epilogue<MB>(e, M, N, K, m0, n0 + 4 * fq, fr, acc, [&](int64_t m) {
    return SkinnyRow{e.x_zero[m], e.x_sums[m], e.x_inv_q[m]};
  });
}

// The product of small operands in one launch: every workgroup quantizes X
// itself (per tensor, or per row), into LDS, and multiplies its 64 rows of W'.
// At these sizes a launch costs more than reading X again (16 x 256 x 128 per
// tensor: two launches 14.3 us a call, one 9.7).
constexpr int kSmallValues = 8192;
// Whether one launch is the faster form.  Every workgroup has four waves for the
// rows, one at a time each (per row: range and params too, one after the other), so
// few rows, fewer per row, where rows off the 16-byte boundaries, which come in
// single floats, weigh more; and many rows only while the workgroups, which all
// repeat that, are few.  rows x K x outputs, us in two launches and in one: per row
// 24 x 64 x 8192 12.4 and 9.0, 32 x 64 x 65536 14.4 and 18.4, 64 x 128 x 8192 12.4
// and 18.9, 16 x 511 x 8192 12.0 and 13.4, x 200000 67 and 52; per tensor 64 x 128 x
// 8192 12.4 and 12.8, x 32768 22.3 and 15.0, x 65536 19.1 and 21.1, 32 x 64 x 200000
// 44.8 and 29.7, 48 x 170 x 8192 12.7 and 14.7.
static bool small_product(const float *X, bool per_row, int64_t M, int64_t N, int64_t K) {
  if (M < 1 || N < 1 || M * K > kSmallValues) return false;
  if (K % 4 != 0 || ((uintptr_t)X & 15) != 0) {
    if (!per_row) return M <= 24 || (M <= 32 && M * K <= 4096);
    return M <= 4 || (M <= 24 && M * K <= 4096) || (M <= 16 && N > 32768);
  }
  return M <= (per_row ? 24 : 32) || (M <= (per_row ? 32 : 64) && N <= 32768);
}
template <int MB, bool PER_ROW>
__global__ __launch_bounds__(256) void k_qmm_small(const float *__restrict__ X, int64_t M,
                                                   const int8_t *__restrict__ B, int64_t ldb, int64_t N,
                                                   int64_t K, EpiArgs e) {
  extern __shared__ __attribute__((aligned(16))) int8_t xs[];  // [M][round_up(K, 64) + 16]
  __shared__ SkinnyRow rows[16 * MB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, fr = lane & 15, fq = lane >> 4;
  const int nk = (int)((K + 63) / 64), ldx = 64 * nk + 16;
  QParams p{};
  if (!PER_ROW) {
    float2 mm = range_minmax_block(X, M * K);
    if (K == 0) mm = make_float2(0.0f, 0.0f);
    p = make_qparams(mm.x, mm.y);
  }
  for (int m = wave; m < (int)M; m += 4) {
    const DenseRow x{X + m * K};
    if (PER_ROW) {
      float2 mm = row_minmax_wave(x, K, lane);
      if (K == 0) mm = make_float2(0.0f, 0.0f);
      p = make_qparams(mm.x, mm.y);
    }
    const int sum = encode_row_wave(x, K, xs + m * ldx, 64 * nk, p.q, p.z, lane);
    if (lane == 0) rows[m] = SkinnyRow{p.z, sum, p.inv_q};
  }
  __syncthreads();
  const int64_t n0 = (int64_t)blockIdx.x * 64 + 16 * wave;
  if (n0 >= N) return;
  const int8_t *w = B + (n0 + fr < N ? n0 + fr : N - 1) * ldb + 16 * fq;
  v4i acc[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) acc[b] = v4i{};
#pragma unroll 8
  for (int c = 0; c < nk; ++c) {
    const v4i wf = *reinterpret_cast<const v4i *>(w + c * 64);
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      const int m = 16 * b + fr < (int)M ? 16 * b + fr : (int)M - 1;
      acc[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
          wf, *reinterpret_cast<const v4i *>(xs + m * ldx + c * 64 + 16 * fq), acc[b], 0, 0, 0);
    }
  }
  skinny_epilogue<MB>(e, M, N, K, 0, n0 + 4 * fq, fr, acc, [&](int64_t m) { return rows[m]; });
}

// Softmax of logit rows already in `post`, in place: one workgroup per row.
// Per 128 columns (max, sum exp) by one half-wave, lane c holding columns c,
// c + 32, c + 64 and c + 96; the sums of the two 64-column halves by a
// butterfly each, added; then the tiles' sums, rescaled to the row's max, in
// tile order.  The order is fixed, whatever the number of rows or of threads.
template <int NT>
__global__ __launch_bounds__(NT) void k_smax_rows(float *__restrict__ post, int64_t N, int ntn,
                                                  float2 *__restrict__ stats,
                                                  float *__restrict__ logits) {
  constexpr int HW = NT / 32;
  __shared__ float smax[NT / 64], sp[NT];
  const int64_t m = blockIdx.x;
  float *y = post + m * N;
  float2 *st = stats + m * ntn;
  const int tid = threadIdx.x, c = tid & 31, hw = tid >> 5;
  float rmx = -INFINITY;
  for (int t = hw; t < ntn; t += HW) {
    const int64_t n0 = (int64_t)t * 128 + c;
    float v[4], mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = n0 + 32 * j < N ? y[n0 + 32 * j] : -INFINITY;
      mx = fmaxf(mx, v[j]);
      if (logits && n0 + 32 * j < N) logits[m * N + n0 + 32 * j] = v[j];
    }
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    float s[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      s[h] = 0.0f;
#pragma unroll
      for (int j = 2 * h; j < 2 * h + 2; ++j)
        if (n0 + 32 * j < N) s[h] += __expf(v[j] - mx);
    }
#pragma unroll
    for (int o = 16; o > 0; o >>= 1)
#pragma unroll
      for (int h = 0; h < 2; ++h) s[h] += __shfl_xor(s[h], o, 64);
    if (c == 0) st[t] = make_float2(mx, s[0] + s[1]);
    rmx = fmaxf(rmx, mx);
  }
  rmx = fmaxf(rmx, __shfl_xor(rmx, 32, 64));
  if ((tid & 63) == 0) smax[tid >> 6] = rmx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) rmx = fmaxf(rmx, smax[w]);
  float sm = 0.0f;
  for (int t0 = 0; t0 < ntn; t0 += NT) {
    if (t0 + tid < ntn) {
      const float2 p = st[t0 + tid];
      sp[tid] = p.y * __expf(p.x - rmx);
    }
    __syncthreads();
    const int n = ntn - t0 < NT ? ntn - t0 : NT;
#pragma unroll 8
    for (int k = 0; k < n; ++k) sm += sp[k];
    __syncthreads();
  }
  const float inv = 1.0f / sm;
  for (int t = hw; t < ntn; t += HW) {
    const int64_t n0 = (int64_t)t * 128 + c;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (n0 + 32 * j < N) y[n0 + 32 * j] = __expf(y[n0 + 32 * j] - rmx) * inv;
  }
}

// ------------------------------------------------------------------ launch
template <int BM, int BN, int BK, int WM, int WN, int NS, int EPI>
static hipError_t run(const int8_t *A, int64_t lda, const int8_t *B, int64_t ldb, int64_t M,
                      int64_t N, int64_t K, const EpiArgs &e, hipStream_t s) {
  using C = GemmCfg<BM, BN, BK, WM, WN, NS>;
  const int64_t Kp = round_up(K, BK);
  size_t lds = (size_t)C::LDS;
  if (EPI == EPI_SMAX_OUT) lds += 2 * BM * sizeof(float);
  auto kern = k_gemm<BM, BN, BK, WM, WN, NS, EPI>;
  static bool attr_set = false;  // per instantiation; idempotent
  if (!attr_set) {
    const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (err != hipSuccess) return err;
    attr_set = true;
  }
  dim3 grid((unsigned)(((N + BN - 1) / BN) * ((M + BM - 1) / BM)));
  hipLaunchKernelGGL(kern, grid, dim3(C::NT), lds, s, A, lda, B, ldb, M, N, K, Kp, e);
  return hipGetLastError();
}

// Kp must stay within the padded leading dimensions: with ld a multiple of 64
// and BK = 64 this always holds; BK = 128 is used when both ld allow it.
// Whether a product of M x N takes 256x256 tiles: once there are enough of
// them to fill the chip.
static bool big_tiles(int64_t M, int64_t N) {
  return ((M + 255) / 256) * ((N + 255) / 256) >= 256;
}

static hipError_t run_skinny(const int8_t *A, int64_t lda, const int8_t *B, int64_t ldb, int64_t M,
                             int64_t N, int64_t K, const EpiArgs &e, hipStream_t s) {
  const int mb = M <= 16 ? 1 : M <= 32 ? 2 : 4;
  auto kern = mb == 1 ? k_gemm_skinny<1> : mb == 2 ? k_gemm_skinny<2> : k_gemm_skinny<4>;
  const dim3 grid((unsigned)((N + 16 * kSkinnyWaves - 1) / (16 * kSkinnyWaves)),
                  (unsigned)((M + 16 * mb - 1) / (16 * mb)));
  hipLaunchKernelGGL(kern, grid, dim3(64 * kSkinnyWaves), 0, s, A, lda, B, ldb, M, N, K, e);
  return hipGetLastError();
}

template <int EPI>
static hipError_t dispatch(const int8_t *A, int64_t lda, const int8_t *B, int64_t ldb, int64_t M,
                           int64_t N, int64_t K, const EpiArgs &e, hipStream_t s) {
  if (M == 0 || N == 0) return hipSuccess;
  const bool k128 = round_up(K, 128) <= lda && round_up(K, 128) <= ldb;
  // 256x256 tiles (128x128 per wave) once there are enough of them to fill
  // the chip; otherwise 128x128 tiles (64x64 per wave)
  if (big_tiles(M, N)) {
    if constexpr (EPI != EPI_RAW) {
      // recovering epilogues: 8 waves of 128x64 (two per SIMD, so one wave's
      // epilogue stalls hide behind the other's work)
      if (k128) return run<256, 256, 128, 2, 4, 2, EPI>(A, lda, B, ldb, M, N, K, e, s);
      return run<256, 256, 64, 2, 4, 4, EPI>(A, lda, B, ldb, M, N, K, e, s);
    }
    if (k128) return run<256, 256, 128, 2, 2, 2, EPI>(A, lda, B, ldb, M, N, K, e, s);
    return run<256, 256, 64, 2, 2, 4, EPI>(A, lda, B, ldb, M, N, K, e, s);
  }
  if constexpr (EPI == EPI_RECOVER) {
    // 128x128 tiles for less than every CU leave the chip idle; but the few-row
    // kernel reads X through the caches once per 16 columns, so its time grows
    // with tiles x K and meets the tiles' at about 80 000.  Per-row product,
    // quantization included, us, tiles then few-row: 64 x 8192 x 512 (64
    // tiles) 23.9 and 18.7; 4000 x 500 x 512 (128) 27.4 and 25.9; 8000 x 500 x
    // 320 (252) 30.0 and 29.4; 8000 x 500 x 512 (252) 31.8 and 40.6; 256 x
    // 8192 x 1024 (128) 29.0 and 32.2.
    const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128);
    if (tiles < 256 && tiles * K < 80000) return run_skinny(A, lda, B, ldb, M, N, K, e, s);
  }
  if constexpr (EPI == EPI_RECOVER || EPI == EPI_RAW) {
    if (k128) return run<128, 128, 128, 2, 2, 0, EPI>(A, lda, B, ldb, M, N, K, e, s);
    return run<128, 128, 64, 2, 2, 0, EPI>(A, lda, B, ldb, M, N, K, e, s);
  }
  return hipErrorInvalidValue;  // the softmax passes run on big tiles only
}

static EpiArgs make_epi(const ActRows &X, const WeightMat &W, const float *bias) {
  EpiArgs e{};
  e.x_zero = X.zero;
  e.x_inv_q = X.inv_q;
  e.x_sums = X.sums;
  e.w_zero = W.zero;
  e.w_inv_q = W.inv_q;
  e.w_sums = W.row_sums;
  e.w_rpb = W.rows_per_block;
  e.bias = bias;
  return e;
}

// Whether the fp32 results of a large product go past the caches: more of them than
// the memory-side cache (256 MB) holds would only push out the operands' panels,
// fewer are still there for the kernel that reads them next.  us through the
// caches and past them: 2048 cells with 512 projected units, 256 rows, product and
// recurrence, 24 frames (201 MB) 450 and 467, 48 frames (403 MB) 858 and 853, 200
// frames 3318 and 3270; product 4096 x 8192 x 512 (134 MB) 46 and 55, 16384 rows
// (537 MB) 206 and 178; a forward with 8192 posteriors of 8192 frames (268 MB) 731
// and 742, 64000 frames 5200 and 5140.
static bool stored_past(int64_t M, int64_t N) { return M * N * 4 > (int64_t)256 << 20; }

hipError_t launch_gemm_recover(const ActRows &X, const WeightMat &W, int64_t M, int64_t N,
                               int64_t K, const float *bias, float *Y, int32_t *acc,
                               hipStream_t s) {
  EpiArgs e = make_epi(X, W, bias);
  e.Y = Y;
  e.acc = acc;
  e.past = stored_past(M, N);
  return dispatch<EPI_RECOVER>(X.codes, X.ld, W.codes, W.ld, M, N, K, e, s);
}

hipError_t launch_qmm_small(const float *X, bool per_row, const WeightMat &W, int64_t M, int64_t N,
                            int64_t K, const float *bias, float *Y, int32_t *acc, hipStream_t s,
                            bool *done) {
  *done = small_product(X, per_row, M, N, K);
  if (!*done) return hipSuccess;
  EpiArgs e = make_epi(ActRows{}, W, bias);
  e.Y = Y;
  e.acc = acc;
  auto kern = per_row    ? (M <= 16 ? k_qmm_small<1, true> : k_qmm_small<2, true>)
              : M <= 16 ? k_qmm_small<1, false>
              : M <= 32 ? k_qmm_small<2, false>
                        : k_qmm_small<4, false>;
  const size_t lds = (size_t)M * (size_t)(round_up(K, 64) + 16);
  hipLaunchKernelGGL(kern, dim3((unsigned)((N + 63) / 64)), dim3(256), lds, s, X, M, W.codes, W.ld, N, K, e);
  return hipGetLastError();
}

hipError_t launch_gemm_raw(const int8_t *A, int64_t lda, const int8_t *B, int64_t ldb,
                           int32_t *C, int64_t M, int64_t N, int64_t K, const int32_t *a_sums,
                           const int32_t *b_sums, hipStream_t s) {
  EpiArgs e{};
  e.x_sums = a_sums;
  e.w_sums = b_sums;
  e.acc = C;
  return dispatch<EPI_RAW>(A, lda, B, ldb, M, N, K, e, s);
}

// Per-tile statistics [M][ntn] (ntn of 128-column tiles is the most any
// launch uses), then the per-row (max, 1 / sum) [M].
static size_t smax_stats_bytes(int64_t M, int64_t N) {
  return align_up((size_t)M * (size_t)((N + 127) / 128) * sizeof(float2), 256);
}
size_t softmax_ws(int64_t M, int64_t N) {
  return smax_stats_bytes(M, N) + align_up((size_t)M * sizeof(float2), 256);
}

// Softmax normaliser of each row from its column tiles' (max, sum exp):
// max over the tiles, sum of sum_t exp(max_t - max), stored as (max, 1/sum).
__global__ __launch_bounds__(256) void k_smax_combine(const float2 *__restrict__ stats, int ntn,
                                                      int64_t M, float2 *__restrict__ rowstat) {
  const int64_t m = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (m >= M) return;
  const float2 *s = stats + m * ntn;
  float mx = -INFINITY;
  for (int t = 0; t < ntn; ++t) mx = fmaxf(mx, s[t].x);
  float sm = 0.0f;
  for (int t = 0; t < ntn; ++t) {
    const float2 st = s[t];
    sm += st.y * __expf(st.x - mx);
  }
  rowstat[m] = make_float2(mx, 1.0f / sm);
}

hipError_t launch_softmax_layer(const ActRows &X, const WeightMat &W, int64_t M, int64_t N,
                                int64_t K, const float *bias, float *post, int32_t *acc,
                                float *logits, void *ws, hipStream_t s) {
  EpiArgs e = make_epi(X, W, bias);
  e.stats = static_cast<float2 *>(ws);
  if (!big_tiles(M, N)) {
    // fewer tiles: the product once, into post, and the rows normalised there
    // (a whole forward with 8192 states, us, as the two passes below on 128x128
    // tiles with a combining launch between them, and now: 1 row 95 and 57, 64
    // rows 123 and 66, 500 rows 134 and 88, 1900 rows 138 and 127)
    e.Y = post;
    e.acc = acc;
    const hipError_t err = dispatch<EPI_RECOVER>(X.codes, X.ld, W.codes, W.ld, M, N, K, e, s);
    if (err != hipSuccess || M == 0 || N == 0) return err;
    const int ntn = (int)((N + 127) / 128);
    // threads a row: half a wave per tile where the tiles are few, so that many
    // rows are in flight; few rows of many tiles take more (product and softmax,
    // us, with 64, 256, 1024 threads and in the two passes below: 32000 rows x 42
    // states 27, 44, 142, 52; 2000 x 2000 42, 33, 39, 56; 400 x 4000 34, 19, 16, 57)
    const int nt = ntn <= 4 ? 64 : ntn <= 32 && M >= 1024 ? 256 : 1024;
    auto kern = nt == 64 ? k_smax_rows<64> : nt == 256 ? k_smax_rows<256> : k_smax_rows<1024>;
    hipLaunchKernelGGL(kern, dim3((unsigned)M), dim3(nt), 0, s, post, N, ntn, e.stats, logits);
    return hipGetLastError();
  }
  // many rows: post is written once; two passes of the product instead of
  // three over M x N floats
  e.ntn = (int)((N + 255) / 256);
  e.acc = acc;
  e.logits = logits;
  hipError_t err = dispatch<EPI_SMAX_STATS>(X.codes, X.ld, W.codes, W.ld, M, N, K, e, s);
  if (err != hipSuccess || M == 0) return err;
  float2 *rowstat = reinterpret_cast<float2 *>(static_cast<char *>(ws) + smax_stats_bytes(M, N));
  hipLaunchKernelGGL(k_smax_combine, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, s,
                     e.stats, e.ntn, M, rowstat);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  e.rowstat = rowstat;
  e.acc = nullptr;
  e.logits = nullptr;
  e.Y = post;
  e.past = stored_past(M, N);
  return dispatch<EPI_SMAX_OUT>(X.codes, X.ld, W.codes, W.ld, M, N, K, e, s);
}

}  // namespace ql
