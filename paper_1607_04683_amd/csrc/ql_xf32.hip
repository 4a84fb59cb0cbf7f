// ql_xf32.hip -- the fp32 recurrence of a layer without a projection on the
// whole chip: the batch rows of a layer never meet, so each XCD runs an eighth
// of them for the whole sequence, and every hand-off stays in its own L2.
//
// The 32 workgroups of an XCD (each reads its XCC_ID and takes the next free
// slot) own 16 cells each.  A workgroup's 64 gate rows of W_h stay in
// registers for the launch, K split over its eight waves (64 floats of each of
// the 64 rows, one register per k), so a step reads nothing but h_{t-1}.
// Products are v_mfma_f32_4x4x1_16b_f32: its 16 blocks are the 16 cells, a
// block's four rows batch rows, its four columns the cell's gates i f g o.
// With at most 8 rows per XCD at batch 64, the 16-row shapes would multiply
// as much padding as data; here 4 rows are the unit.  The row operand is
// broadcast from one block to all, so one register holds h for 16 steps of k.
// A step:
//   1. h_{t-1} of the XCD's rows, 64-bit words (step tag << 32 | fp32) that
//      every tile polls from the L2, to LDS;
//   2. the partial products of each wave's slice of K, to LDS;
//   3. one thread per (cell, row, gate): the eight partial sums in wave order,
//      + (W_x x + b), the gate; the four gates of a pair meet by DPP; c and
//      h_t, published.  W_x x + b of step t + 1 is loaded while step t runs.
// The words of a step parity are rewritten only after every tile of the XCD
// has read them, since a tile publishes h_t only after it has read all of
// h_{t-1}.  Bound by the latency of that chain: one hand-off through L2 (about
// 1 us) and 128 dependent-issue MFMAs a wave (0.85 us at 8 rows).
// Five 500-cell layers at batch 64: 13.7 us a step of one layer in the layout
// with a tile of the batch per workgroup and device-coherent counters, 3.25 us
// here.
#include "ql_device.h"
#include "ql_exchange.h"
#include "ql_launch.h"
#include "ql_xcd.h"

#include <algorithm>

namespace ql {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kXfThreads = 512;
constexpr int kXfWaves = kXfThreads / 64;
constexpr int kXfXcds = 8, kXfSlots = 32;  // XCDs of the MI355X, CUs of one
constexpr int kXfCells = 16;               // cells of a tile: one MFMA block each
constexpr int kXfMaxH = kXfSlots * kXfCells;
constexpr int kXfLdx = kXfMaxH + 4;        // row stride of h in LDS: four rows, four bank groups
constexpr int kXfMaxRows = 16;             // batch rows of an XCD

struct XfTiling {
  int64_t r0, r1;  // batch rows [r0, r1) of this launch
  int rows;        // rows per XCD (the last may hold fewer or none)
};

// NG groups of four batch rows per XCD.
template <int NG>
__global__ __launch_bounds__(kXfThreads) void k_xrec_f32(F32RecArgs a, XfTiling tl) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ int s_abort, s_role;
  constexpr int NR = 4 * NG;                         // rows the layout holds
  constexpr int NA = NG == 1 ? 4 : NG == 2 ? 2 : 1;  // accumulators per row group
  constexpr int NQ = (256 * NG + kXfThreads - 1) / kXfThreads;  // gate values per thread
  float *xs = reinterpret_cast<float *>(smem);         // [NR][kXfLdx] h_{t-1}
  float *part = xs + NR * kXfLdx;                      // [waves][NG][16 cells][4 gates][4 rows]

  const int64_t T = a.T, B = a.B, H = a.H;
  if (threadIdx.x == 0) {
    const int xcc = (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & 15);
    unsigned *slots = reinterpret_cast<unsigned *>(static_cast<char *>(a.ws) + kHeaderBytes);
    s_role = -1;
    s_abort = 0;
    if (xcc < kXfXcds) {
      const unsigned k = __hip_atomic_fetch_add(slots + xcc * 16, 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
      if (k < (unsigned)kXfSlots) s_role = xcc * kXfSlots + (int)k;
    }
  }
  __syncthreads();
  const int role = __builtin_amdgcn_readfirstlane(s_role);
  if (role < 0) return;
  const int64_t b0 = tl.r0 + (int64_t)(role / kXfSlots) * tl.rows;
  const int64_t j0 = (int64_t)(role % kXfSlots) * kXfCells;
  const int nb = (int)std::min<int64_t>(tl.rows, tl.r1 - b0);
  if (nb <= 0 || j0 >= H) return;  // no rows for this XCD, or no cells for this tile
  int *flag = reinterpret_cast<int *>(a.ws) + kHdrFlag;
  uint64_t *X = reinterpret_cast<uint64_t *>(static_cast<char *>(a.ws) + kHeaderBytes +
                                             kCounterBytes);  // [2][B][H]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // W_h: lane 4 c + g holds gate g of cell c, its k from kw on
  const int kpw = (int)((H + 4 * kXfWaves - 1) / (4 * kXfWaves)) * 4;  // k per wave, <= 64
  const int kw = wave * kpw;
  // (no load depends on the lane, so that all are in flight at once: loads of
  // single floats behind tests of the lane's k came in 10 us later at 500 cells;
  // what lies past the ends is dropped)
  float w[64];
  {
    const int64_t j = j0 + (lane >> 2);
    const float *src = a.Wh + ((lane & 3) * H + (j < H ? j : H - 1)) * H;
    if (H % 4 == 0 && ((uintptr_t)a.Wh & 15) == 0) {  // rows 16-byte aligned
      v4f v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q)
        v[q] = 4 * q < kpw ? *reinterpret_cast<const v4f *>(src + std::min<int64_t>(kw + 4 * q, H - 4)) : v4f{};
#pragma unroll
      for (int k = 0; k < 64; ++k) w[k] = kw + k < H ? v[k / 4][k % 4] : 0.0f;
    } else {
#pragma unroll
      for (int k = 0; k < 64; ++k) w[k] = k < kpw ? src[std::min<int64_t>(kw + k, H - 1)] : 0.0f;
#pragma unroll
      for (int k = 0; k < 64; ++k) w[k] = kw + k < H ? w[k] : 0.0f;
    }
  }
  for (int i = tid; i < NR * kXfLdx; i += kXfThreads) xs[i] = 0.0f;  // rows and k past the end

  // this thread's gate values q = tid + 512 r: gate q & 3 of pair q >> 2, which
  // is cell (pair & 63) >> 2, row 4 (pair >> 6) + (pair & 3)
  float cst[NQ], gx[NQ], gxn[NQ];
  int64_t brow[NQ];
  bool live[NQ];
  const int gate = tid & 3;
  const int64_t jc = j0 + ((tid >> 4) & 15);
#pragma unroll
  for (int r = 0; r < NQ; ++r) {
    const int pair = (tid + kXfThreads * r) >> 2, lb = 4 * (pair >> 6) + (pair & 3);
    live[r] = pair < 64 * NG && lb < nb && jc < H;
    brow[r] = live[r] ? b0 + lb : b0;
    cst[r] = live[r] && a.c0 ? a.c0[brow[r] * H + jc] : 0.0f;
  }
  auto load_gx = [&](int64_t t, float (&g)[NQ]) {
#pragma unroll
    for (int r = 0; r < NQ; ++r)
      g[r] = live[r] ? a.gx[(t * B + brow[r]) * 4 * H + gate * H + jc] : 0.0f;
  };
  load_gx(0, gx);
  uint32_t need = 0;
  if (tid < H)
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (i < nb) need |= 1u << i;
  if (j0 == 0) straggle_under_wait_bound();
  __syncthreads();

  for (int64_t t = 0; t < T; ++t) {
    // ---- 1. h_{t-1}: word i of a thread is row i, cell tid
    if (t == 0) {
      if (a.h0 && tid < H)
        for (int i = 0; i < nb; ++i) xs[i * kXfLdx + tid] = a.h0[(b0 + i) * H + tid];
    } else {
      const uint64_t *src = X + (((t - 1) & 1) * B + b0) * H;
      if (!poll_to_lds<NR>(
              need, (uint32_t)t, [&](int i, int th) { return src + i * H + th; },
              [&](int i, int th) { return reinterpret_cast<uint32_t *>(xs + i * kXfLdx + th); }, flag))
        s_abort = 1;
    }
    if (t + 1 < T) load_gx(t + 1, gxn);  // lands behind the products and gates of this step
    __syncthreads();
    if (s_abort) return;

    // ---- 2. this wave's slice of K
    v4f acc[NG][NA];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int n = 0; n < NA; ++n) acc[g][n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    // lane 4 b + i holds h of row i at k = b of each 16
    float h[NG][4];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        h[g][c] = xs[(4 * g + (lane & 3)) * kXfLdx + kw + 16 * c + (lane >> 2)];
    auto four = [&](auto qc) __attribute__((always_inline)) {
      static_for<4 * decltype(qc)::value, 4 * decltype(qc)::value + 4>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
#pragma unroll
        for (int g = 0; g < NG; ++g)
          acc[g][k % NA] =
              __builtin_amdgcn_mfma_f32_4x4x1f32(h[g][k / 16], w[k], acc[g][k % NA], 4, k % 16, 0);
      });
    };
    // (kpw is a multiple of 4: one test skips four.  Layers of over 480 cells have
    // nothing to skip, and the tests would cost one row 7% of its step)
    if (kpw == 64)
      static_for<0, 16>(four);
    else
      static_for<0, 16>([&](auto qc) {
        if (4 * decltype(qc)::value < kpw) four(qc);
      });
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      // the results are read by ordinary instructions below: enough wait
      // states after the last pass, which the hardware does not check
#pragma unroll
      for (int n = 0; n < NA; ++n) asm volatile("s_nop 7\n\ts_nop 7" : "+v"(acc[g][n]));
      v4f s = acc[g][0];
#pragma unroll
      for (int n = 1; n < NA; ++n) s += acc[g][n];
      *reinterpret_cast<v4f *>(part + ((wave * NG + g) * 64 + lane) * 4) = s;
    }
    __syncthreads();

    // ---- 3. gates, c, h_t
    const uint32_t tag = (uint32_t)(t + 1);
    uint64_t *dst = X + (t & 1) * B * H;
#pragma unroll
    for (int r = 0; r < NQ; ++r) {
      const int q = tid + kXfThreads * r;
      float sum = 0.0f;
      if (q < 256 * NG) {
#pragma unroll
        for (int v = 0; v < kXfWaves; ++v)
          sum += part[(v * NG + (q >> 8)) * 256 + ((tid >> 4) & 15) * 16 + gate * 4 + ((q >> 2) & 3)];
      }
      const float av = gx[r] + sum;
      const float sg = sigmoid_cw(gate == 2 ? 2.0f * av : av);
      const float act = gate == 2 ? 2.0f * sg - 1.0f : sg;
      const float ig = quad_bcast<0>(act), fg = quad_bcast<1>(act), gv = quad_bcast<2>(act),
                  og = quad_bcast<3>(act);
      const float cn = (fg * cst[r]) + (ig * gv);
      cst[r] = cn;
      const float m = og * tanh_cw(cn);
      if (live[r]) {
        if (gate == 0) put_word(dst + brow[r] * H + jc, tag, __float_as_uint(m));
        if (gate == 1) a.h[(t * B + brow[r]) * H + jc] = m;
        if (t == T - 1) {
          if (gate == 2 && a.hT) a.hT[brow[r] * H + jc] = m;
          if (gate == 3 && a.cT) a.cT[brow[r] * H + jc] = cn;
        }
      }
      gx[r] = gxn[r];
    }
  }
}

// ------------------------------------------------------------------ host side
template <int NG>
static hipError_t run_xf32(const F32RecArgs &a, const XfTiling &tl, int cus, hipStream_t s,
                           bool *done) {
  // more than half of a CU's LDS, so that a CU holds one workgroup
  const size_t used = (size_t)(4 * NG * kXfLdx + kXfWaves * NG * 256) * sizeof(float);
  const size_t lds = std::max<size_t>(used, 84 * 1024);
  auto kern = k_xrec_f32<NG>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kXfThreads, lds);
  if (e != hipSuccess) return e;
  *done = per_cu >= 1;
  if (!*done) return hipSuccess;
  e = clear_exchange(a.ws, kCounterBytes / 8 + 2 * a.B * a.H, s);
  if (e != hipSuccess) return e;
  F32RecArgs args = a;
  XfTiling t = tl;
  void *kargs[] = {&args, &t};
  return hipLaunchCooperativeKernel(reinterpret_cast<void *>(kern), dim3(cus), dim3(kXfThreads),
                                    kargs, (unsigned)lds, s);
}

// Launches the layout takes a in (up to 16 rows per XCD, as few of equal size as
// that allows); 0: a runs as tiles of the batch over the chip, whose sums are in
// another order (so the choice may not depend on T: chunks of a sequence chain
// with the bits of the whole).  A further launch's steps take as long whatever the
// width, where tiles hold more rows of narrow layers.  50 frames, us, in tiles and
// so: 64 cells, 300 rows 329 and 630; 200 cells, 200 rows 616 and 593, 300 rows 646
// and 840; 256 cells, 500 rows 955 and 1148; 280 cells 1992 and 1227; 400 cells,
// 300 rows 1882 and 1005 (5 frames 290 and 273; 280 cells 207 and 253).
static int plan_xf32(const F32RecArgs &a, int cus, int lds_max) {
  if (cus != kXfXcds * kXfSlots || lds_max < 100 * 1024) return 0;
  if (a.P > 0 || a.H < 1 || a.H > kXfMaxH || a.B < 1 || a.T < 1) return 0;
  const int64_t most = kXfXcds * kXfMaxRows, launches = (a.B + most - 1) / most;
  return launches == 1 || a.H > (launches == 2 ? 200 : 256) ? (int)launches : 0;
}

// The exchange words, [2][B][H] of 8 bytes, are what recurrent_f32_ws holds
// for a layer without a projection.
hipError_t launch_xrec_f32(const F32RecArgs &a, int cus, int lds_max, hipStream_t s, bool *done) {
  *done = false;
  const int64_t launches = plan_xf32(a, cus, lds_max);
  if (launches == 0) return hipSuccess;
  const int64_t chunk = (a.B + launches - 1) / launches;
  for (int64_t r0 = 0; r0 < a.B; r0 += chunk) {
    XfTiling tl{r0, std::min(a.B, r0 + chunk), 0};
    tl.rows = (int)((tl.r1 - tl.r0 + kXfXcds - 1) / kXfXcds);
    const hipError_t e = tl.rows <= 4   ? run_xf32<1>(a, tl, cus, s, done)
                         : tl.rows <= 8 ? run_xf32<2>(a, tl, cus, s, done)
                                        : run_xf32<4>(a, tl, cus, s, done);
    if (e != hipSuccess || !*done) return e;
  }
  return hipSuccess;
}

int xrec_f32_launches(int64_t H, int64_t T, int64_t B, int cus, int lds_max) {
  F32RecArgs a{};
  a.H = H, a.T = T, a.B = B;
  return plan_xf32(a, cus, lds_max);
}

hipError_t set_wait_bound_xf32(int polls) { return set_wait_bound_here(polls); }

}  // namespace ql
