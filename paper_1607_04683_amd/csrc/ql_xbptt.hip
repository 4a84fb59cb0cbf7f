// ql_xbptt.hip -- backpropagation through time of one LSTM layer without a
// projection (the recurrence of ql_train.hip) on the whole chip: each XCD
// runs an eighth of the batch for the whole sequence, as the fp32 recurrence
// forward does, and every hand-off stays in its own L2.
//
//   dh_t = dy_t + W_h^T da_{t+1},  da_t = the cell's backward step on dh_t
//
// da has four values a cell where dh has one, so the workgroups do not gather
// da_{t+1} (64 KB a step each at 8 rows, 128 KB with tags); each multiplies
// the da of its own 16 cells, which never leave it, with its 64 rows of W_h,
// and hands every other workgroup the partial sums of that one's 16 cells:
// 32 KB of tagged words written and read a step.  The 64 rows of W_h stay in
// registers (wave w the cells [64 w, 64 w + 64) as outputs, one register per
// k); products are v_mfma_f32_4x4x1_16b_f32, 16 blocks of four batch rows x
// four output cells, the rows broadcast from one block to all (one register
// of da serves 16 steps of k), so 4 rows are the unit of padding and no sum
// crosses waves before it is published.  A step t = T-1 .. 0:
//   1. the partial sums of W_h^T da_{t+1} for this tile's (row, cell) pairs:
//      four threads a pair, each polls and adds the words of eight tiles in
//      tile order, then the four add up;
//   2. the cell's backward step; thread g of a pair keeps and writes gate g;
//   3. da_t of the tile through LDS into the products, whose results are
//      published as the words of step t - 1.
// A slot is rewritten two steps later, which a tile reaches only after every
// tile has published the step between, and each does that only after all of
// its own polls of the first.  Bound by that chain: one hand-off (about 1 us)
// and 128 MFMAs a wave (0.85 us at 8 rows).  A 500-cell layer at batch 64:
// 8.75 us a step gathering da with device-coherent counters; 6.1 with single
// words stored, 5.0 with two a store, 4.7 with the rows broadcast.
#include "ql_device.h"
#include "ql_exchange.h"
#include "ql_launch.h"
#include "ql_xcd.h"

#include <algorithm>

namespace ql {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kXbThreads = 512;
constexpr int kXbXcds = 8, kXbSlots = 32;  // XCDs of the MI355X, CUs of one
constexpr int kXbCells = 16;               // cells of a tile
constexpr int kXbMaxH = kXbSlots * kXbCells;
constexpr int kXbMaxRows = 16;             // batch rows of an XCD
constexpr int kXbLdx = 64 + 4;             // row stride of the tile's da in LDS
constexpr int kXbSlotBytes = kXbXcds * 64;

struct XbTiling {
  int64_t r0, r1;  // batch rows [r0, r1) of this launch
  int rows;        // rows per XCD (the last may hold fewer or none)
};

// Exchange words of one XCD: [2 parities][dst tile][src tile][row pair][16
// cells][2 rows]: the 16-byte stores of 16 lanes, a cell's two rows each, are
// contiguous.
template <int NG>
struct XbLay {
  static constexpr int64_t src = 4 * NG * kXbCells;
  static constexpr int64_t dst = kXbSlots * src;
  static constexpr int64_t par = kXbSlots * dst;
  static constexpr int64_t xcd = 2 * par;
};

// NG groups of four batch rows per XCD.
template <int NG>
__global__ __launch_bounds__(kXbThreads) void k_xbptt(BpttArgs a, XbTiling tl) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  // expired waits, by step parity: the word of a step is read after its one
  // barrier and written again only after the next, so every wave leaves there
  __shared__ int s_abort[2], s_role;
  using L = XbLay<NG>;
  constexpr int NR = 4 * NG;
  constexpr int NA = NG == 1 ? 4 : NG == 2 ? 2 : 1;              // accumulators per row group
  constexpr int NQ = (256 * NG + kXbThreads - 1) / kXbThreads;   // (pair, gate) values per thread
  float *xs = reinterpret_cast<float *>(smem);                   // [2][NR][kXbLdx] da of the tile

  const int64_t T = a.T, B = a.B, H = a.H;
  if (threadIdx.x == 0) {
    const int xcc = (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & 15);
    unsigned *slots = reinterpret_cast<unsigned *>(static_cast<char *>(a.ws) + kHeaderBytes);
    s_role = -1;
    s_abort[0] = s_abort[1] = 0;
    if (xcc < kXbXcds) {
      const unsigned k = __hip_atomic_fetch_add(slots + xcc * 16, 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
      if (k < (unsigned)kXbSlots) s_role = xcc * kXbSlots + (int)k;
    }
  }
  __syncthreads();
  const int role = __builtin_amdgcn_readfirstlane(s_role);
  if (role < 0) return;
  const int xcd = role / kXbSlots, tile = role % kXbSlots;
  const int64_t b0 = tl.r0 + (int64_t)xcd * tl.rows, j0 = (int64_t)tile * kXbCells;
  const int nb = (int)std::min<int64_t>(tl.rows, tl.r1 - b0);
  if (nb <= 0 || j0 >= H) return;  // no rows for this XCD, or no cells for this tile
  int *flag = reinterpret_cast<int *>(a.ws) + kHdrFlag;
  uint64_t *X = reinterpret_cast<uint64_t *>(static_cast<char *>(a.ws) + kHeaderBytes +
                                             kXbSlotBytes) +
                xcd * L::xcd;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // W_h^T: lane l is output cell 64 wave + l; k = 4 cell + gate of the tile
  float w[64];
  {
    const int64_t o = 64 * wave + lane;
#pragma unroll
    for (int k = 0; k < 64; ++k) {
      const int64_t j = j0 + (k >> 2);
      w[k] = o < H && j < H ? a.Wh[((k & 3) * H + j) * H + o] : 0.0f;
    }
  }
  for (int i = tid; i < 2 * NR * kXbLdx; i += kXbThreads) xs[i] = 0.0f;  // rows and cells past the end

  // (pair, gate) values q = tid + 512 r: gate q & 3 (also: the eighth of the
  // tiles whose partial sums the thread adds) of pair q >> 2, in the order of the
  // exchange words: row 2 (pair >> 5) + (pair & 1), cell (pair >> 1) & 15
  const int gate = tid & 3, cell = (tid >> 3) & 15;
  auto row_of = [&](int r) { return 2 * ((tid + kXbThreads * r) >> 7) + ((tid >> 2) & 1); };
  const int64_t jc = j0 + cell;
  int64_t brow[NQ];
  bool live[NQ];
#pragma unroll
  for (int r = 0; r < NQ; ++r) {
    const int lb = row_of(r);
    live[r] = lb < nb && jc < H;
    brow[r] = live[r] ? b0 + lb : b0;
  }
  // operands of a step: the thread's own gate's value, and c_{t-1} (gates 0
  // and 1), dy_t (gates 2 and 3); shared within the pair by DPP
  struct Op {
    float g[NQ], x[NQ];
  };
  auto load_op = [&](int64_t t, Op &o) {
#pragma unroll
    for (int r = 0; r < NQ; ++r) {
      o.g[r] = o.x[r] = 0.0f;
      if (!live[r] || t < 0) continue;
      const int64_t row = t * B + brow[r];
      o.g[r] = a.gates[(row * 4 + gate) * H + jc];
      if (gate >= 2) o.x[r] = a.dy[row * H + jc];
      else if (t > 0) o.x[r] = a.c[(row - B) * H + jc];
    }
  };
  Op op, opn;
  load_op(T - 1, op);
  float ct[NQ], dcn[NQ];  // c_t; dC/dc carried to the step before
#pragma unroll
  for (int r = 0; r < NQ; ++r) {
    ct[r] = live[r] ? a.c[((T - 1) * B + brow[r]) * H + jc] : 0.0f;
    dcn[r] = 0.0f;
  }
  // the tiles whose words this thread adds: 8 gate .. + 7, those with cells
  const int ntile = (int)((H + kXbCells - 1) / kXbCells);
  uint32_t need = 0;
#pragma unroll
  for (int r = 0; r < NQ; ++r)
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (live[r] && 8 * gate + i < ntile) need |= 1u << (8 * r + i);
  uint64_t *Xin = X + tile * L::dst + 8 * gate * L::src;  // + par, + i * src, + pair
  // where the wave's results go: tile 4 wave + (lane >> 4), cell lane & 15
  uint64_t *Xout = X + (4 * wave + (lane >> 4)) * L::dst + tile * L::src + 2 * (lane & 15);
  const bool out_ok = 64 * wave + 16 * (lane >> 4) < H;
  if (tile == 0) straggle_under_wait_bound();
  __syncthreads();

  for (int64_t t = T - 1; t >= 0; --t) {
    // ---- 1. W_h^T da_{t+1}
    float dhr[NQ];
#pragma unroll
    for (int r = 0; r < NQ; ++r) dhr[r] = 0.0f;
    if (t + 1 < T) {
      uint32_t v[8 * NQ];
#pragma unroll
      for (int i = 0; i < 8 * NQ; ++i) v[i] = 0u;
      const uint64_t *src = Xin + (t & 1) * L::par;
      if (!poll_words<8 * NQ>(
              need, (uint32_t)(T - t), v,
              [&](int i) {
                return src + (i & 7) * L::src + ((tid + kXbThreads * (i >> 3)) >> 2);
              },
              flag))
        s_abort[t & 1] = 1;
#pragma unroll
      for (int r = 0; r < NQ; ++r)
#pragma unroll
        for (int i = 0; i < 8; ++i) dhr[r] += __uint_as_float(v[8 * r + i]);
    }
    load_op(t - 1, opn);  // lands behind this step's products and the next hand-off

    // ---- 2. the cell's backward step
    float *xt = xs + (t & 1) * NR * kXbLdx;
#pragma unroll
    for (int r = 0; r < NQ; ++r) {
      const float dh =
          quad_bcast<2>(op.x[r]) + ((quad_bcast<0>(dhr[r]) + quad_bcast<1>(dhr[r])) +
                                    (quad_bcast<2>(dhr[r]) + quad_bcast<3>(dhr[r])));
      const float ig = quad_bcast<0>(op.g[r]), fg = quad_bcast<1>(op.g[r]),
                  gg = quad_bcast<2>(op.g[r]), og = quad_bcast<3>(op.g[r]);
      const float cp = quad_bcast<0>(op.x[r]);
      const float tc = tanh_cw(ct[r]);
      const float d_o = dh * tc;
      const float d_c = dh * og * (1.0f - tc * tc) + dcn[r];
      const float d_i = d_c * gg, d_g = d_c * ig, d_f = d_c * cp;
      dcn[r] = d_c * fg;
      ct[r] = cp;
      const float v = gate == 0   ? d_i * ig * (1.0f - ig)
                      : gate == 1 ? d_f * fg * (1.0f - fg)
                      : gate == 2 ? d_g * (1.0f - gg * gg)
                                  : d_o * og * (1.0f - og);
      if (live[r]) {
        a.da[((t * B + brow[r]) * 4 + gate) * H + jc] = v;
        xt[row_of(r) * kXbLdx + 4 * cell + gate] = v;
      }
    }
#pragma unroll
    for (int r = 0; r < NQ; ++r) op.g[r] = opn.g[r], op.x[r] = opn.x[r];
    __syncthreads();
    if (s_abort[t & 1]) return;
    if (t == 0) break;

    // ---- 3. this tile's part of W_h^T da_t, published for step t - 1
    v4f acc[NG][NA];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int n = 0; n < NA; ++n) acc[g][n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    // lane 4 b + i holds da of row i at k = b of each 16
    float d[NG][4];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int c = 0; c < 4; ++c) d[g][c] = xt[(4 * g + (lane & 3)) * kXbLdx + 16 * c + (lane >> 2)];
    static_for<0, 64>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
#pragma unroll
      for (int g = 0; g < NG; ++g)
        acc[g][k % NA] =
            __builtin_amdgcn_mfma_f32_4x4x1f32(d[g][k / 16], w[k], acc[g][k % NA], 4, k % 16, 0);
    });
    const uint32_t tag = (uint32_t)(T - t + 1);
    uint64_t *dst = Xout + ((t - 1) & 1) * L::par;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      // the results are read by ordinary instructions below: enough wait
      // states after the last pass, which the hardware does not check
#pragma unroll
      for (int n = 0; n < NA; ++n) asm volatile("s_nop 7\n\ts_nop 7" : "+v"(acc[g][n]));
      v4f s = acc[g][0];
#pragma unroll
      for (int n = 1; n < NA; ++n) s += acc[g][n];
      if (out_ok)
#pragma unroll
        for (int i = 0; i < 4; i += 2)
          put_words2(dst + (4 * g + i) * kXbCells, tag, __float_as_uint(s[i]), __float_as_uint(s[i + 1]));
    }
  }
}

// ------------------------------------------------------------------ host side
static int rows_per_xcd(int64_t B, int64_t *chunk) {
  // up to 16 rows per XCD, in as few launches of equal size as that allows
  const int64_t most = kXbXcds * kXbMaxRows;
  const int64_t launches = (B + most - 1) / most;
  *chunk = (B + launches - 1) / launches;
  return (int)((*chunk + kXbXcds - 1) / kXbXcds);
}
static size_t xbptt_words(int rows) {
  return (size_t)kXbXcds * (rows <= 4 ? XbLay<1>::xcd : rows <= 8 ? XbLay<2>::xcd : XbLay<4>::xcd);
}
size_t xbptt_ws(int64_t B) {
  int64_t chunk;
  return kHeaderBytes + kXbSlotBytes + 8 * xbptt_words(rows_per_xcd(std::max<int64_t>(B, 1), &chunk));
}

template <int NG>
static hipError_t run_xbptt(const BpttArgs &a, const XbTiling &tl, int cus, hipStream_t s,
                            bool *done) {
  // more than half of a CU's LDS, so that a CU holds one workgroup
  const size_t lds = 84 * 1024;
  static_assert((size_t)2 * 4 * NG * kXbLdx * sizeof(float) <= 84 * 1024, "da buffers");
  auto kern = k_xbptt<NG>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kXbThreads, lds);
  if (e != hipSuccess) return e;
  *done = per_cu >= 1;
  if (!*done) return hipSuccess;
  e = clear_exchange(a.ws, (int64_t)(kXbSlotBytes / 8 + kXbXcds * XbLay<NG>::xcd), s);
  if (e != hipSuccess) return e;
  BpttArgs args = a;
  XbTiling t = tl;
  void *kargs[] = {&args, &t};
  return hipLaunchCooperativeKernel(reinterpret_cast<void *>(kern), dim3(cus), dim3(kXbThreads),
                                    kargs, (unsigned)lds, s);
}

// Launches the layout takes a in; 0: a runs faster, or only, on k_bptt, which has
// the whole batch in one.  A second launch pays for narrow layers and for few
// steps (where start-up counts), a third never.  A training step of one layer, us,
// k_bptt and so: 64 cells, 200 rows, 100 frames 2310 and 2265; 128 cells the same
// 2448 and 2539, 20 frames 1053 and 1016; 64 cells, 300 rows, 100 frames 2490 and
// 2909, 20 frames 1036 and 1083.
static int plan_xbptt(const BpttArgs &a, int cus, int lds_max) {
  if (cus != kXbXcds * kXbSlots || lds_max < 100 * 1024) return 0;
  if (a.H < 1 || a.H > kXbMaxH || a.B < 1 || a.T < 1) return 0;
  const int64_t most = kXbXcds * kXbMaxRows, launches = (a.B + most - 1) / most;
  return launches == 1 || (launches == 2 && (a.H <= 64 || a.T <= 40)) ? (int)launches : 0;
}

hipError_t launch_xbptt(const BpttArgs &a, int cus, int lds_max, hipStream_t s, bool *done) {
  *done = false;
  if (plan_xbptt(a, cus, lds_max) == 0) return hipSuccess;
  int64_t chunk;
  const int rows = rows_per_xcd(a.B, &chunk);
  for (int64_t r0 = 0; r0 < a.B; r0 += chunk) {
    const XbTiling tl{r0, std::min(a.B, r0 + chunk), rows};
    const hipError_t e = rows <= 4   ? run_xbptt<1>(a, tl, cus, s, done)
                         : rows <= 8 ? run_xbptt<2>(a, tl, cus, s, done)
                                     : run_xbptt<4>(a, tl, cus, s, done);
    if (e != hipSuccess || !*done) return e;
  }
  return hipSuccess;
}

int xbptt_launches(int64_t H, int64_t T, int64_t B, int cus, int lds_max) {
  BpttArgs a{};
  a.H = H, a.T = T, a.B = B;
  return plan_xbptt(a, cus, lds_max);
}

hipError_t set_wait_bound_xbptt(int polls) { return set_wait_bound_here(polls); }

}  // namespace ql
