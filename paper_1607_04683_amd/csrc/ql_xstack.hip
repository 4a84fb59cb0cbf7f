// ql_xstack.hip -- stacked LSTM layers without a projection (Section 4) in
// persistent launches over the whole chip, run as a wavefront: layer l works
// on frame t while layer l-1 is already further on.
//
// The unit of work is a row group of one layer: up to 16 batch rows (one MFMA
// tile) over the whole sequence, on 16 workgroups of one XCD (one per CU; each
// reads its XCC_ID and takes the next free slot of its XCD) of 32 cells each,
// or on 8 workgroups of 64 cells.  The chip holds 16 or 32 units, so n layers
// take floor(16 / n) or floor(32 / n) row groups a launch (5 layers: 48 or 96
// rows), and larger batches several launches where those pay (ql_stack.hip says
// when).  Every hand-off inside a unit stays in that XCD's L2: plain stores,
// device-coherent loads that find them there.  What bounds a step is the latency of two such hand-offs (about 1 us
// each) and of the phases between them; 64-cell tiles add their second cells'
// arithmetic.  A frame through 5 x 500 cells (200 frames, start-up included),
// us: 16 rows 4.3, 48 rows 4.6, 64 rows 5.6, 96 rows 5.9, 150 rows (two
// launches) 11.1.  Before, two groups of 32 rows of one XCD per layer served
// batch 16 to 64 only (5.0 at 16 rows, 7.3 at 64) and k_stack the others
// (6 rows 23.7, 80 rows 16.4, 150 rows 28.8).
//
// A tile keeps the gate rows of its cells of both W_x' and W_h' in registers as
// MFMA fragments, four cells (their gates i f g o adjacent) per 16-row block,
// so an MFMA result gives a lane the four gate sums of one (cell, row) pair,
// and c stays in that lane's registers; one more product, with ones, gives it
// the code sum of its row.  A step t, for the tile's rows:
//   1. the product with W_h' of the codes of h_{t-1}; the tile's part of them
//      goes out, with the rows' params, as the layer's quantized output of
//      step t-1 (which layer l+1 reads, on another XCD, once an arrival counter
//      says that every tile's part is out); the codes of x_{t+1} (the launch's
//      input, or the codes layer l-1 made of its h) go to LDS;
//   2. recovered (eq. 1 / eq. 3), + (W_x x + b), gates, c and h_t;
//   3. E1: the per-row min/max of h_t over the tile's cells, published; the
//      product of x_{t+1} with W_x' while the other tiles' parts arrive; every
//      tile reads all parts and forms the quantizer of each row (eq. 2, fp64
//      params);
//   4. E2: each tile encodes its own cells of h_t and publishes the codes; it
//      recovers W_x x_{t+1} (plus the bias, exactly as the hoisted input
//      product does) and takes the codes of h_t from the unit's tiles.
// The loads of x_{t+2} go out behind the poll for the codes of h_t, so that
// they have most of a step to cross from another XCD and nothing waits behind
// them.  Exchanged words are 64-bit (step tag << 32 | payload) in a double
// buffer by step parity; a tile can only reuse a half after every tile of its
// unit has read it, since each hand-off needs the previous one from all of
// them.  Every wait is bounded: on expiry a flag in the workspace is raised and
// every workgroup leaves at the end of its step.  The arithmetic is that of
// k_stack and the one-layer path, so the results are bit-identical to them.
#include "ql_device.h"
#include "ql_exchange.h"
#include "ql_launch.h"
#include "ql_rec_common.h"
#include "ql_xcd.h"

#include <algorithm>
#include <cstddef>

namespace ql {

constexpr int kXsThreads = 512;
constexpr int kXsWaves = kXsThreads / 64;
constexpr int kXsXcds = 8;      // XCDs of the MI355X, each with its own L2
constexpr int kXsSlots = 32;    // CUs (workgroups) of one XCD
constexpr int kXsMaxW = 512;    // widths (cells, input) the layout is sized for
constexpr int kXsSlotBytes = kXsXcds * 64;
constexpr int kXsCounterBytes = 2048;  // [unit][parity], 32 bytes apart

constexpr int kXsRows = 16;  // batch rows of a unit, at most: one MFMA tile

// Zero point and recovery factor of a row of x.
struct XsRow {
  int32_t z;
  float iq;
};

struct XsTiling {
  int ng;            // row groups per layer
  int rows;          // batch rows per row group (the last may hold fewer)
  int64_t r0, r1;    // batch rows [r0, r1) of this launch
  size_t lds_bytes;  // (host) dynamic LDS of the instance
  int64_t xwords;    // (host) exchange words per unit
  int cb;            // (host) instance
};

// LDS and exchange layout of an instance: CB 4-cell blocks per wave.
template <int CB>
struct XsLay {
  static constexpr int bX = kXsRows, u = 4 * kXsWaves * CB, uw = u / 4;
  static constexpr int tiles = kXsMaxW / u;             // cell tiles (workgroups) of a unit
  static constexpr int units = kXsXcds * kXsSlots / tiles;  // units a launch can hold
  static constexpr int ldsX = kXsMaxW + 16;  // row stride of the codes of x and of h
  static constexpr size_t xx = 0;                                              // [bX][ldsX]
  static constexpr size_t xh = xal16(xx + (size_t)bX * ldsX);                  // [bX][ldsX]
  static constexpr size_t cph = xal16(xh + (size_t)bX * ldsX);                 // [u][4]
  static constexpr size_t cpx = xal16(cph + (size_t)4 * u * sizeof(ColParam)); // [u][4]
  static constexpr size_t cf = xal16(cpx + (size_t)4 * u * sizeof(ColParam));  // 6 x [u] x 16
  static constexpr size_t bias = xal16(cf + (size_t)6 * u * 16);               // [u] float4
  static constexpr size_t rpx = xal16(bias + (size_t)u * 16);                  // [bX]
  static constexpr size_t hp = xal16(rpx + (size_t)bX * sizeof(XsRow));        // [bX]
  static constexpr size_t pm = xal16(hp + (size_t)bX * sizeof(XParam));        // [bX][32][2]
  static constexpr size_t mcs = xal16(pm + (size_t)bX * 32 * 2 * 4);           // [bX][u]
  static constexpr size_t bytes = xal16(mcs + (size_t)bX * u);
  // exchange words of one unit, one parity:
  //   E1  [bX][tiles][2]   min / max keys of h_t
  //   E2  [bX][tiles][uw]  codes of h_t
  static constexpr int64_t e1 = 0;
  static constexpr int64_t e2 = e1 + (int64_t)bX * tiles * 2;
  static constexpr int64_t gwords = (e2 + (int64_t)bX * tiles * uw + 31) / 32 * 32;
  static constexpr int64_t uwords = 2 * gwords;  // a unit: 2 parities
  static_assert(units * 2 * 32 <= kXsCounterBytes, "arrival counters");
};

struct XsKArgs {
  StackArgs a;
  XsTiling tl;
};
typedef const __attribute__((address_space(4))) XsKArgs *XsKArgPtr;

// What a workgroup derives from the launch's scalars and its role: stated
// once for the kernel, and again (through the kernel-argument pointer) on the
// rare output path of the step.  What the step needs on every step (the x
// and output addresses) is held in vector registers instead, so that no
// scalar reload sits on the step's chain.
#define XS_SCALARS(a, tl, role)                                                                 \
  const int unit = (role) / L::tiles, ct = (role) % L::tiles;                                  \
  const int l = unit / tl.ng, g = unit % tl.ng;                                                \
  auto &Ly = a.L[l];                                                                           \
  const int64_t T = a.T, B = a.B, H = a.H, IN = Ly.in;                                         \
  int *flag = reinterpret_cast<int *>(a.ws) + kHdrFlag;                                        \
  const int64_t b0 = tl.r0 + (int64_t)g * tl.rows;                                             \
  const int nb = (int)std::min<int64_t>((int64_t)tl.rows, tl.r1 - b0);                         \
  const int64_t j0 = (int64_t)ct * u;                                                          \
  const int ldX = (int)((IN + 63) / 64 * 64), ldH = (int)((H + 63) / 64 * 64);                 \
  unsigned *cnt0 = reinterpret_cast<unsigned *>(static_cast<char *>(a.ws) + kHeaderBytes +     \
                                                kXsSlotBytes);                                 \
  auto ctr = [&](int layer, int64_t par, int grp) {                                            \
    return cnt0 + ((layer * tl.ng + grp) * 2 + (int)par) * 8;                                  \
  };                                                                                           \
  uint64_t *X = reinterpret_cast<uint64_t *>(static_cast<char *>(a.ws) + kHeaderBytes +        \
                                             kXsSlotBytes + kXsCounterBytes) +                 \
                (int64_t)unit * L::uwords;                                                     \
  auto E = [&](int64_t tt_) { return X + (tt_ & 1) * L::gwords; };                             \
  (void)T, (void)flag, (void)ldX, (void)ldH, (void)ctr, (void)E, (void)IN

template <int CB, bool TP>
__global__ __launch_bounds__(kXsThreads) void k_xstack(StackArgs a, XsTiling tl) {
  static_assert(offsetof(XsKArgs, tl) == sizeof(StackArgs), "argument layout");
  using L = XsLay<CB>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ int s_abort, s_role;
  constexpr int bX = L::bX, u = L::u, uw = L::uw, ldsX = L::ldsX;

  if (threadIdx.x == 0) {
    const int xcc = (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & 15);
    unsigned *slots = reinterpret_cast<unsigned *>(static_cast<char *>(a.ws) + kHeaderBytes);
    s_role = -1;
    s_abort = 0;
    if (xcc < kXsXcds) {
      const unsigned k = __hip_atomic_fetch_add(slots + xcc * 16, 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
      // units 0 .. 7 on an XCD of their own each, then the next share of each
      const int unit = (int)(k / L::tiles) * kXsXcds + xcc;
      if (k < (unsigned)kXsSlots && unit < a.nl * tl.ng)
        s_role = unit * L::tiles + (int)(k % L::tiles);
    }
  }
  __syncthreads();
  const int role = __builtin_amdgcn_readfirstlane(s_role);
  if (role < 0) return;
  int8_t *xx = reinterpret_cast<int8_t *>(smem + L::xx);          // codes of x_{t+1}
  int8_t *xh = reinterpret_cast<int8_t *>(smem + L::xh);          // codes of h_{t-1}
  ColParam *cph = reinterpret_cast<ColParam *>(smem + L::cph);    // [u][4] W_h' rows
  ColParam *cpx = reinterpret_cast<ColParam *>(smem + L::cpx);    // [u][4] W_x' rows
  // the same for the 24-bit recovery, four gates of a cell per vector (low 32
  // bits of colterm, shifted zero point, 1/Q), h side then x side
  int4 *ctmh = reinterpret_cast<int4 *>(smem + L::cf);
  int4 *czth = ctmh + u;
  float4 *ciqh = reinterpret_cast<float4 *>(czth + u);
  int4 *ctmx = reinterpret_cast<int4 *>(ciqh + u);
  int4 *cztx = ctmx + u;
  float4 *ciqx = reinterpret_cast<float4 *>(cztx + u);
  float4 *bias4 = reinterpret_cast<float4 *>(smem + L::bias);      // [u] gates i f g o
  XsRow *rpx = reinterpret_cast<XsRow *>(smem + L::rpx);          // rows of x_t, then x_{t+1}
  XParam *hp = reinterpret_cast<XParam *>(smem + L::hp);          // quantizer of each row of h
  int *pm = reinterpret_cast<int *>(smem + L::pm);                // min/max parts of h_t
  uint8_t *mcs = reinterpret_cast<uint8_t *>(smem + L::mcs);      // own cells' codes of h_t

  XS_SCALARS(a, tl, role);

  // ---- prologue: W_x', W_h' fragments, column params, bias, c_0
  const int tid0 = threadIdx.x, wave0 = tid0 >> 6, fr0 = tid0 & 15, fq0 = (tid0 & 63) >> 4;
  // blocks of wave w: cells 4 (w + 8 cb) .. + 3; lane row fr is gate fr & 3 of cell fr >> 2
  v4i wh[CB][8], wx[CB][8];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int jj = 4 * (wave0 + kXsWaves * cb) + (fr0 >> 2);
    const bool ok = j0 + jj < H;
    const int64_t n = (int64_t)(fr0 & 3) * H + j0 + jj;
    const int8_t *sh = Ly.Wh.codes + n * Ly.Wh.ld + 16 * fq0;
    const int8_t *sx = Ly.Wx.codes + n * Ly.Wx.ld + 16 * fq0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      wh[cb][c] = ok && c * 64 < ldH ? *reinterpret_cast<const v4i *>(sh + c * 64) : v4i{};
      wx[cb][c] = ok && c * 64 < ldX ? *reinterpret_cast<const v4i *>(sx + c * 64) : v4i{};
    }
  }
  for (int r = tid0; r < 4 * u; r += kXsThreads) {
    const int jj = r >> 2, gate = r & 3;
    const int64_t n = (int64_t)gate * H + std::min<int64_t>(j0 + jj, H - 1);
    {
      const int64_t blk = n / Ly.Wh.rows_per_block;
      ColParam c;
      c.ztw = Ly.Wh.zero[blk] + 128;
      c.sigw = Ly.Wh.row_sums[n] - 128 * (int32_t)H;
      c.colterm = (int64_t)c.sigw + H * (int64_t)c.ztw;
      c.iqw = Ly.Wh.inv_q[blk];
      c.pad = 0;
      cph[r] = c;
      reinterpret_cast<int *>(ctmh + jj)[gate] = (int32_t)c.colterm;
      reinterpret_cast<int *>(czth + jj)[gate] = c.ztw;
      reinterpret_cast<float *>(ciqh + jj)[gate] = c.iqw;
    }
    {
      const int64_t blk = n / Ly.Wx.rows_per_block;
      ColParam c;
      c.ztw = Ly.Wx.zero[blk] + 128;
      c.sigw = Ly.Wx.row_sums[n] - 128 * (int32_t)IN;
      c.colterm = (int64_t)c.sigw + IN * (int64_t)c.ztw;
      c.iqw = Ly.Wx.inv_q[blk];
      c.pad = 0;
      cpx[r] = c;
      reinterpret_cast<int *>(ctmx + jj)[gate] = (int32_t)c.colterm;
      reinterpret_cast<int *>(cztx + jj)[gate] = c.ztw;
      reinterpret_cast<float *>(ciqx + jj)[gate] = c.iqw;
    }
    reinterpret_cast<float *>(bias4 + jj)[gate] = Ly.bias[n];
  }
  // the codes' bytes past the padded widths stay zero, so that the products
  // and the code sums may run over all of a row
  for (int i = tid0; i < 2 * bX * ldsX / 4; i += kXsThreads) reinterpret_cast<int *>(xx)[i] = 0;
  // the lane's (cell, row) pairs: cell 4 (wave + 8 cb) + fq, row fr
  float cst[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int64_t j = j0 + 4 * (wave0 + kXsWaves * cb) + fq0;
    cst[cb] = Ly.c0 && j < H && fr0 < nb ? Ly.c0[(b0 + fr0) * H + j] : 0.0f;
  }
  __syncthreads();
  // whether the lane's cells allow the 24-bit recovery on every gate: bit
  // 2 cb the recurrent side, bit 2 cb + 1 the input side
  int cfm = 0;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    bool fh = true, fx = true;
#pragma unroll
    for (int gate = 0; gate < 4; ++gate) {
      const int r = (4 * (wave0 + kXsWaves * cb) + fq0) * 4 + gate;
      const ColParam ch = cph[r], cx = cpx[r];
      fh = fh && fast_col(ch.ztw, ch.colterm);
      fx = fx && fast_col(cx.ztw, cx.colterm);
    }
    cfm |= ((fh ? 1 : 0) | (fx ? 2 : 0)) << (2 * cb);
  }

  XsKArgPtr kp = (XsKArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
  // The codes of x_t (the launch's input, or layer l-1's output, once its
  // arrival counter says step t is complete) and the rows' zero points and
  // recovery factors, in registers: word i of a thread is row 8 i + tid / 64,
  // 8-byte word tid % 64 (a row has at most 64); even waves take the zero
  // points, odd ones the factors.  park_x puts them into LDS.  Every load is
  // issued whatever the rows and width (words past them read some valid word
  // that park_x drops), so that no branch makes the compiler wait for more
  // than a step needs.  What load_x and park_x need is computed once and held
  // in vector registers (no scalar reloads on the step's critical path): bit i
  // of xmask says whether word i of this thread is a real code word.
  uint64_t xv[bX / 8];
  int32_t xm = 0;
  const int xr0 = tid0 >> 6, xwd = tid0 & 63;
  uint32_t xmask = 0;
#pragma unroll
  for (int i = 0; i < bX / 8; ++i)
    if (8 * i + xr0 < nb && xwd < ldX / 8) xmask |= 1u << i;
  const char *xsrc0 = reinterpret_cast<const char *>(
      Ly.xin.codes + (b0 + std::min(xr0, nb - 1)) * Ly.xin.ld + 8 * std::min(xwd, ldX / 8 - 1));
  const int32_t *xmp = (wave0 & 1 ? reinterpret_cast<const int32_t *>(Ly.xin.inv_q) : Ly.xin.zero) +
                       b0 + std::min(tid0 & 63, nb - 1);
  int64_t xrow8 = 8 * Ly.xin.ld, xstep = B * Ly.xin.ld, xB = B;
  asm volatile("" : "+v"(xrow8), "+v"(xstep), "+v"(xB));
  const unsigned *cprev = l > 0 ? ctr(l - 1, 0, g) : nullptr;  // parity 1: + 8
  // Each wave waits for the counter itself (no barrier), starting from a value
  // `seen` it read earlier (0: none), so that a count already reached costs no
  // round trip; if the wait expires it raises the abort, which the next check
  // after a barrier acts on, and its loads read whatever is there.
  auto wait_x = [&](int64_t tx, unsigned seen) {
    if (cprev) {
      const unsigned *c = cprev + (tx & 1) * 8;
      const unsigned target = (unsigned)((tx >> 1) + 1) * L::tiles;
      long it = 0;
      while (seen < target) {
        if (wait_expired(flag, it)) {
          s_abort = 1;
          break;
        }
        seen = __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  };
  auto load_x = [&](int64_t tx) {
    const char *src = xsrc0 + tx * xstep;
#pragma unroll
    for (int i = 0; i < bX / 8; ++i)
      xv[i] = ld_coherent64(reinterpret_cast<const uint64_t *>(src + ((xmask >> i) & 1u ? i * xrow8 : 0)));
    xm = ld_coherent_i(xmp + tx * xB);
  };
  auto park_x = [&]() {
    // (landed for every lane, also those that drop them: otherwise the compiler
    // waits again, for later operations too, where it reuses their registers)
#pragma unroll
    for (int i = 0; i < bX / 8; ++i) asm volatile("" : "+v"(xv[i]));
    asm volatile("" : "+v"(xm));
#pragma unroll
    for (int i = 0; i < bX / 8; ++i)
      if ((xmask >> i) & 1u) *reinterpret_cast<uint64_t *>(xx + (8 * i + xr0) * ldsX + 8 * xwd) = xv[i];
    if ((threadIdx.x & ~64u) < (unsigned)bX)  // lanes 0 .. 15 of waves 0 and 1
      reinterpret_cast<int32_t *>(rpx + (threadIdx.x & 63))[threadIdx.x >> 6] = xm;
  };
  // The products of the codes in LDS with the lane's weight fragments, and the
  // sum of each row's signed codes as one more product, with ones: a lane
  // ends with the four gate sums of its (cell, row) pairs and the code sum of
  // its row, so no sums are handed over, staged or waited for.
  const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
  auto products = [&](const int8_t *codes, const v4i(&w)[CB][8], int fr, int fq, v4i(&acc)[CB],
                      v4i &sum) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[cb] = v4i{};
    sum = v4i{};
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const v4i b = *reinterpret_cast<const v4i *>(codes + fr * ldsX + c * 64 + 16 * fq);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        acc[cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[cb][c], b, acc[cb], 0, 0, 0);
      sum = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, b, sum, 0, 0, 0);
    }
    // the results are read by ordinary instructions: at least 19 wait states
    // after the last pass, which the hardware does not check
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) asm volatile("" : "+v"(acc[cb]));
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(sum), "+v"(acc[0]), "+v"(acc[CB - 1]));
  };
  v4i accx[CB], sumx;
  // This tile's part of the layer's quantized output of step tx (codes of
  // its cells, from the codes of h_tx in LDS; tile 0 also the rows' z, 1/Q
  // and code sums), with device-coherent stores, for layer l+1 on another XCD;
  // taps of the codes.
  // What publish_out needs on every step, held in vector registers like the
  // above: this thread's word of 4 codes (row tid / uw, word tid % uw of the
  // tile's cells) and, in tile 0, its row's params.
  const int orw = tid0 / uw, oww = tid0 % uw;
  const bool ocode = orw < nb && j0 + 4 * oww < ldH;
  const int oxh = orw * ldsX + (int)j0 + 4 * oww;
  uint32_t *ocp = reinterpret_cast<uint32_t *>(Ly.out.codes + (b0 + orw) * Ly.out.ld + j0) + oww;
  int64_t ostep = B * Ly.out.ld / 4;  // 4-byte words from frame t to t + 1
  int hk = (int)H, xk = (int)IN;
  asm volatile("" : "+v"(ostep), "+v"(hk), "+v"(xk));
  const bool ometa = ct == 0 && tid0 < nb;
  int32_t *ozp = Ly.out.zero + b0 + tid0;
  float *oqp = Ly.out.inv_q + b0 + tid0;
  int32_t *osp = Ly.out.sums + b0 + tid0;
  // (the last tile zeroes the rows' padding up to the output's stride; taps)
  const bool orare = (ct == L::tiles - 1 && Ly.out.ld > ldH) || Ly.tap_codes || Ly.tap_zero ||
                     Ly.tap_inv_q;
  auto publish_out = [&](int64_t tx, int sigma) {
    if (ometa) {  // lanes of wave 0 with fq = 0: sigma is the sum of row tid's signed codes
      const int64_t o = tx * xB;
      st_coherent_i(ozp + o, hp[threadIdx.x].z);
      st_coherent(oqp + o, hp[threadIdx.x].inv_q);
      st_coherent_i(osp + o, sigma + 128 * hk);
    }
    if (ocode)
      __hip_atomic_store(ocp + tx * ostep, *reinterpret_cast<const uint32_t *>(xh + oxh),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (orare) {
      auto &a = kp->a;
      auto &tl = kp->tl;
      XS_SCALARS(a, tl, role);
      const int tid = threadIdx.x;
      const int64_t orow0 = tx * B + b0;
      if (ct == 0 && tid < nb) {
        if (Ly.tap_zero) Ly.tap_zero[orow0 + tid] = hp[tid].z;
        if (Ly.tap_inv_q) Ly.tap_inv_q[orow0 + tid] = hp[tid].inv_q;
      }
      if (ct == L::tiles - 1)
        for (int idx = tid; idx < nb * (int)((Ly.out.ld - ldH) / 4); idx += kXsThreads) {
          const int nw = (int)((Ly.out.ld - ldH) / 4), r2 = idx / nw, w2 = idx % nw;
          __hip_atomic_store(reinterpret_cast<uint32_t *>(Ly.out.codes + (orow0 + r2) * Ly.out.ld + ldH) + w2,
                             0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      if (Ly.tap_codes)
        for (int idx = tid; idx < nb * u; idx += kXsThreads) {
          const int r2 = idx / u, k = idx % u;
          if (j0 + k < H) Ly.tap_codes[(orow0 + r2) * H + j0 + k] = xh[r2 * ldsX + j0 + k];
        }
    }
  };
  float *hout = Ly.h;
  asm volatile("" : "+v"(hout));
  // the codes of h_{-1} and x_0 to LDS, x_1 into registers (the weight fragments
  // have landed before the loop: no wait for them in it)
  wait_vmcnt0();
  __syncthreads();
  wait_x(0, 0u);
  load_x(0);
  park_x();
  {
    RowParam *rp = reinterpret_cast<RowParam *>(pm);  // (pm is free before the first step)
    if (!quant_tile<8, 2, kSrcPlain>(nb, bX, H, 0u, (int)H, xh, ldsX, ldH, flag, rp,
                                     [&](int lb) -> const void * {
                                       return Ly.h0 ? Ly.h0 + (b0 + lb) * H : nullptr;
                                     }))
      s_abort = 1;
    __syncthreads();
    if (tid0 < bX) {  // (rows past the unit's too: the products' exact form is never theirs)
      hp[tid0].z = rp[tid0].z;
      hp[tid0].inv_q = rp[tid0].iqx;
    }
  }
  if (T > 1) wait_x(1, 0u);
  load_x(std::min<int64_t>(1, T - 1));
  wait_vmcnt0();  // nothing in flight on the loop's first entry
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(s_abort)) return;
  products(xx, wx, fr0, fq0, accx, sumx);

  // W_x' x recovered (eq. 1 / eq. 3) plus the bias, as the hoisted input product
  // forms it (tx: x's step, for the tap)
  float xb[CB][4];
  auto recover_x = [&](int64_t tx, int wave, int fr, int fq) {
    const int32_t ztx = rpx[fr].z + 128, sigx = sumx[0];
    const float iqx = rpx[fr].iq;
    const bool fast = fast_row(ztx);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const int jjL = 4 * (wave + kXsWaves * cb) + fq;  // the lane's cell (tile-local)
      const int4 ct4 = ctmx[jjL], zt4 = cztx[jjL];
      const float4 iq4 = ciqx[jjL], b4 = bias4[jjL];
      const v4i ax = accx[cb];
      float yx[4];
      yx[0] = recover_fast(ax[0], ct4.x, zt4.x, ztx, sigx, iq4.x, iqx);
      yx[1] = recover_fast(ax[1], ct4.y, zt4.y, ztx, sigx, iq4.y, iqx);
      yx[2] = recover_fast(ax[2], ct4.z, zt4.z, ztx, sigx, iq4.z, iqx);
      yx[3] = recover_fast(ax[3], ct4.w, zt4.w, ztx, sigx, iq4.w, iqx);
      // the exact form where a zero point or column term rules the 24-bit
      // one out (rare), in a branch the wave takes only then
      const bool fastx = fast && ((cfm >> (2 * cb)) & 2);
      if (__any(!fastx) && !fastx)
#pragma unroll
        for (int gate = 0; gate < 4; ++gate) {
          const ColParam c = cpx[jjL * 4 + gate];
          yx[gate] = recover(ax[gate], c.colterm, c.ztw, ztx, sigx, c.iqw, iqx);
        }
      xb[cb][0] = yx[0] + b4.x;
      xb[cb][1] = yx[1] + b4.y;
      xb[cb][2] = yx[2] + b4.z;
      xb[cb][3] = yx[3] + b4.w;
      if (TP && Ly.acc_x && tx < T && j0 + jjL < H && fr < nb)
#pragma unroll
        for (int gate = 0; gate < 4; ++gate)
          Ly.acc_x[((tx * B + b0 + fr) * 4 + gate) * H + j0 + jjL] =
              acc_u8(ax[gate], cpx[jjL * 4 + gate].sigw, sigx, xk);
    }
    
  };
  recover_x(0, wave0, fr0, fq0);
  __syncthreads();  // every wave has read x_0 and its rows' params: step 0 puts x_1 in their place

  // the words of the poll for the codes of h (E2): word i of a thread is row
  // 4 i + tid / 128, word tid % 128 (a row has at most 128)
  constexpr int CW = bX / 4;
  constexpr int rs4 = 4 * L::tiles * uw, ls4 = 4 * ldsX;
  static_assert(L::tiles * uw == 128, "code words of a row");
  uint32_t need2 = 0;
#pragma unroll
  for (int k = 0; k < CW; ++k)
    if (4 * k + (tid0 >> 7) < nb && (tid0 & 127) < ldH / 4) need2 |= 1u << k;
  auto e2src = [&](const uint64_t *e) {
    const uint64_t *e2 = e + L::e2;
    return [=](int i, int th) -> const uint64_t * {
      return e2 + i * rs4 + (th >> 7) * (rs4 / 4) + (th & 127);
    };
  };
  auto e2dst = [&](int i, int th) -> uint32_t * {
    return reinterpret_cast<uint32_t *>(xh + i * ls4 + (th >> 7) * ldsX + 4 * (th & 127));
  };
  uint64_t w2[CW];
  // the codes of h_{tx} (their poll is in flight) into LDS
  auto take_h = [&](int64_t tx) {
    if (!poll_to_lds_finish<CW>(need2, (uint32_t)(tx + 1), w2, e2src(E(tx)), e2dst, flag))
      s_abort = 1;
    __syncthreads();
  };
  // The loop has one exit, its condition, so that the compiler's waits for a
  // step's loads are those of the step alone.  An expired wait therefore ends
  // the loop with its step: what the step still computes is undefined, as are
  // the outputs then, and its further waits end at once.
  int stop = 0;
  int64_t t = 0;
  do {
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6, fr = lane & 15, fq = lane >> 4;

    // ---- 1. W_h' h_{t-1}; x_{t+1} (loaded a step ago) to LDS
    v4i acch[CB], sumh;
    products(xh, wh, fr, fq, acch, sumh);
    park_x();
    // the arrival count of x_{t+2}, read now so that it is in hand when its
    // loads are issued (4)
    unsigned seen = 0;
    if (l > 0 && t + 2 < T)
      seen = __hip_atomic_load(cprev + (t & 1) * 8, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // this tile's part of the layer's quantized output of step t-1, across
    // XCDs: its stores complete while the gates are computed
    if (t > 0) publish_out(t - 1, sumh[0]);

    // ---- 2. recovery of W_h' h_{t-1}, + (W_x x + b), gates, c and h_t
    float hv[CB];
    {
      const int32_t ztx = hp[fr].z + 128, sigx = sumh[0];
      const float iqx = hp[fr].inv_q;
      const bool fast = fast_row(ztx);
      const int64_t brow = b0 + fr;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const int jjL = 4 * (wave + kXsWaves * cb) + fq;
        const int64_t jL = j0 + jjL;
        const int4 ct4 = ctmh[jjL], zt4 = czth[jjL];
        const float4 iq4 = ciqh[jjL];
        const v4i ah = acch[cb];
        float y[4];
        y[0] = recover_fast(ah[0], ct4.x, zt4.x, ztx, sigx, iq4.x, iqx);
        y[1] = recover_fast(ah[1], ct4.y, zt4.y, ztx, sigx, iq4.y, iqx);
        y[2] = recover_fast(ah[2], ct4.z, zt4.z, ztx, sigx, iq4.z, iqx);
        y[3] = recover_fast(ah[3], ct4.w, zt4.w, ztx, sigx, iq4.w, iqx);
        const bool fasth = fast && ((cfm >> (2 * cb)) & 1);
        if (__any(!fasth) && !fasth)
#pragma unroll
          for (int gate = 0; gate < 4; ++gate) {
            const ColParam c = cph[jjL * 4 + gate];
            y[gate] = recover(ah[gate], c.colterm, c.ztw, ztx, sigx, c.iqw, iqx);
          }
        float gv[4];
#pragma unroll
        for (int gate = 0; gate < 4; ++gate) {
          const float av = xb[cb][gate] + y[gate];
          const float sg = sigmoid_cw(gate == 2 ? 2.0f * av : av);
          gv[gate] = gate == 2 ? 2.0f * sg - 1.0f : sg;
        }
        const float cn = (gv[1] * cst[cb]) + (gv[0] * gv[2]);
        cst[cb] = cn;
        const float m = gv[3] * tanh_cw(cn);
        hv[cb] = m;
        if (jL < H && fr < nb) {
          if (hout) hout[(t * B + brow) * H + jL] = m;
          if (TP) {
            if (Ly.acc_h)
#pragma unroll
              for (int gate = 0; gate < 4; ++gate)
                Ly.acc_h[((t * B + brow) * 4 + gate) * H + jL] =
                    acc_u8(ah[gate], cph[jjL * 4 + gate].sigw, sigx, H);
            if (Ly.tap_gates) {
              float *gp = Ly.tap_gates + (t * B + brow) * 4 * H + jL;
              gp[0] = gv[0], gp[H] = gv[1], gp[2 * H] = gv[2], gp[3 * H] = gv[3];
            }
            if (Ly.tap_c) Ly.tap_c[(t * B + brow) * H + jL] = cn;
            if (Ly.tap_m) Ly.tap_m[(t * B + brow) * H + jL] = m;
            if (t == T - 1) {
              if (Ly.hT) Ly.hT[brow * H + jL] = m;
              if (Ly.cT) Ly.cT[brow * H + jL] = cn;
            }
          }
        }
      }
    }

    // ---- 3. E1: min/max of h_t per row over the tile's cells
    {
      int lo = 0x7fffffff, hi = 0x7fffffff;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        if (j0 + 4 * (wave + kXsWaves * cb) + fq < H) {
          const int key = float_key(hv[cb]);
          lo = min(lo, key);
          hi = min(hi, ~key);
        }
      int *d = pm + (fr * 32 + wave * 4 + fq) * 2;
      d[0] = lo;
      d[1] = hi;
    }
    __syncthreads();
    uint64_t *e = E(t);
    const uint32_t tag = (uint32_t)(t + 1);
    {
      // waves 0 .. 3: 16 lanes per row, two of the row's 32 (wave, lane group)
      // parts each; then every row's params from the tiles' parts, one tile's
      // (min, max) words a lane (lanes without a part load some word and drop it)
      const int row = tid >> 4, j = tid & 15;
      const bool part = row < nb && j < L::tiles;
      const uint64_t *e1 = e + L::e1 + (row * L::tiles + min(j, L::tiles - 1)) * 2;
      uint64_t w1[2];
      if (wave < 4) {
        const int4 q = *reinterpret_cast<const int4 *>(pm + (row * 32 + 2 * j) * 2);
        const int lo = red16(min(q.x, q.z), MinI{}), hi = red16(min(q.y, q.w), MinI{});
        if (row < nb && j == 0) {
          put_word(e + L::e1 + (row * L::tiles + ct) * 2, tag, (uint32_t)lo);
          put_word(e + L::e1 + (row * L::tiles + ct) * 2 + 1, tag, (uint32_t)hi);
        }
      }
      // W_x' x_{t+1} while the other tiles' parts arrive: polled at once, 95% of
      // the first rounds came too early, and a second cost more than this
      products(xx, wx, fr, fq, accx, sumx);
      if (wave < 4) {
        w1[0] = ld_tagged(e1);
        w1[1] = ld_tagged(e1 + 1);
        uint32_t v[2] = {0u, 0u};
        uint32_t left = part ? 3u : 0u;
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (((left >> i) & 1u) && (uint32_t)(w1[i] >> 32) == tag) {
            v[i] = (uint32_t)w1[i];
            left &= ~(1u << i);
          }
        bool ok = true;
        if (__any(left != 0))
          ok = poll_words<2>(left, tag, v, [&](int i) -> const uint64_t * { return e1 + i; }, flag);
        if (!ok) s_abort = 1;
        const int lo = red16(part ? (int)v[0] : 0x7fffffff, MinI{});
        const int hi = red16(part ? (int)v[1] : 0x7fffffff, MinI{});
        if (row < nb && j == 0 && ok) {
          const QParams prm = make_qparams(key_float(lo), key_float(~hi));
          XParam xp;
          xp.q = prm.q;
          xp.z = prm.z;
          xp.inv_q = prm.inv_q;
          hp[row] = xp;
        }
      }
    }
    // every memory operation so far has completed (the output stores of step
    // t-1 among them): after the barrier, layer l+1 is told that step t-1 is out
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    stop = __builtin_amdgcn_readfirstlane(s_abort);  // (written on the far sides of this barrier
                                                     // and the next)
    if (t > 0 && tid == 0)
      __hip_atomic_fetch_add(ctr(l, (t - 1) & 1, g), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // ---- 4. E2: the tile's cells of h_t encoded (eq. 2)
    {
      const XParam xp = hp[fr];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const int jjL = 4 * (wave + kXsWaves * cb) + fq;
        int code = 128;  // device byte 0: cells past H add nothing to a product
        if (j0 + jjL < H) code = encode(hv[cb], xp.q, xp.z);
        mcs[fr * u + jjL] = (uint8_t)(code ^ 0x80);
      }
    }
    __syncthreads();
    {
      // one word of four codes per thread
      const int row = tid / uw, wd = tid % uw;
      if (row < nb)
        put_word(e + L::e2 + row * (L::tiles * uw) + ct * uw + wd, tag,
                 *reinterpret_cast<const uint32_t *>(mcs + row * u + 4 * wd));
    }
    // the first round of the poll for the codes of h_t, then the loads of
    // x_{t+2} behind it (past the end: x_{T-1} again, never used); with 64-cell
    // tiles after the recovery below, as half of the first rounds came too
    // early without it
    if (t + 2 < T) wait_x(t + 2, seen);
    if (CB == 2) recover_x(t + 1, wave, fr, fq);
    poll_to_lds_issue_all<CW>(e2src(e), w2);
    load_x(std::min(t + 2, T - 1));
    // W_x' x_{t+1} recovered while the codes of h_t are on their way, then those
    if (CB == 1) recover_x(t + 1, wave, fr, fq);
    take_h(t);
  } while (++t < T && !stop);
  if (stop || s_abort) return;

  // the last step's output, and the arrival once its stores have completed
  {
    v4i acc[CB], sum;
    products(xh, wh, fr0, fq0, acc, sum);
    publish_out(T - 1, sum[0]);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_fetch_add(ctr(l, (T - 1) & 1, g), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------ host side
static size_t unit_bytes(int cb) { return 8 * (size_t)(cb == 1 ? XsLay<1>::uwords : XsLay<2>::uwords); }
static int chip_units(int cb) { return cb == 1 ? XsLay<1>::units : XsLay<2>::units; }
constexpr size_t kXsHead = kHeaderBytes + kXsSlotBytes + kXsCounterBytes;

// (what two row groups of 32 rows in 32-cell tiles per layer take)
size_t xstack_ws(int nl) { return kXsHead + (size_t)nl * 2 * 90112; }

// The rows from r0 on that one launch takes: 32-cell tiles while the chip (and
// the scratch) holds enough units for the whole batch, else 64-cell tiles, and
// then as few launches, of equal size, as the batch needs.
static bool plan_xstack(const StackArgs &a, size_t ws_bytes, int cus, int lds_max, int64_t r0,
                        XsTiling *out) {
  if (cus != kXsXcds * kXsSlots || a.nl < 1 || a.nl > kXsXcds) return false;
  if (a.B < 1 || a.H > kXsMaxW || ws_bytes < kXsHead) return false;
  const int64_t ldH = round_up(a.H, 64);
  for (int l = 0; l < a.nl; ++l) {
    const StackLayer &L = a.L[l];
    if (L.in > kXsMaxW || L.Wx.ld < round_up(L.in, 64) || L.Wh.ld < ldH) return false;
    if (L.out.ld < ldH || L.out.ld % 4) return false;
  }
  auto most_rows = [&](int cb) {
    const size_t fit = (ws_bytes - kXsHead) / (a.nl * unit_bytes(cb));
    return (int64_t)kXsRows * (int64_t)std::min<size_t>(chip_units(cb) / a.nl, fit);
  };
  XsTiling tl{};
  tl.cb = a.B <= most_rows(1) ? 1 : 2;
  const int64_t most = most_rows(tl.cb);
  if (most < 1) return false;
  const int64_t launches = (a.B + most - 1) / most, chunk = (a.B + launches - 1) / launches;
  tl.r0 = r0;
  tl.r1 = std::min(a.B, r0 + chunk);
  const int64_t n = tl.r1 - tl.r0;
  tl.ng = (int)((n + kXsRows - 1) / kXsRows);
  tl.rows = (int)((n + tl.ng - 1) / tl.ng);
  tl.lds_bytes = tl.cb == 2 ? XsLay<2>::bytes : XsLay<1>::bytes;
  tl.xwords = (int64_t)unit_bytes(tl.cb) / 8;
  if (tl.lds_bytes + 64 > (size_t)lds_max) return false;
  *out = tl;
  return true;
}

using XsKernel = void (*)(StackArgs, XsTiling);

bool xstack_applies(const StackArgs &a, size_t ws_bytes, int cus, int lds_max) {
  XsTiling tl;
  return plan_xstack(a, ws_bytes, cus, lds_max, 0, &tl);
}

int xstack_launches(const StackArgs &a, size_t ws_bytes, int cus, int lds_max, int *cells) {
  int n = 0;
  XsTiling tl{};
  for (int64_t r0 = 0; r0 < a.B; r0 = tl.r1, ++n)
    if (!plan_xstack(a, ws_bytes, cus, lds_max, r0, &tl)) return 0;
  *cells = 32 * tl.cb;
  return n;
}

hipError_t launch_xstack(const StackArgs &a, size_t ws_bytes, int cus, int lds_max, bool taps,
                         hipStream_t s, bool *done) {
  *done = false;
  for (int64_t r0 = 0; r0 < a.B;) {
    XsTiling tl;
    if (!plan_xstack(a, ws_bytes, cus, lds_max, r0, &tl)) return hipSuccess;
    XsKernel kern = tl.cb == 2 ? (taps ? k_xstack<2, true> : k_xstack<2, false>)
                               : (taps ? k_xstack<1, true> : k_xstack<1, false>);
    hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)tl.lds_bytes);
    if (e != hipSuccess) return e;
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kXsThreads, tl.lds_bytes);
    if (e != hipSuccess) return e;
    if (per_cu < 1) return hipSuccess;
    e = clear_exchange(a.ws, (kXsSlotBytes + kXsCounterBytes) / 8 + (int64_t)a.nl * tl.ng * tl.xwords,
                       s);
    if (e != hipSuccess) return e;
    StackArgs args = a;
    void *kargs[] = {&args, &tl};
    e = hipLaunchCooperativeKernel(reinterpret_cast<void *>(kern), dim3(cus), dim3(kXsThreads),
                                   kargs, (unsigned)tl.lds_bytes, s);
    if (e != hipSuccess) return e;
    r0 = tl.r1;
  }
  *done = true;
  return hipSuccess;
}

hipError_t set_wait_bound_xstack(int polls) { return set_wait_bound_here(polls); }

}  // namespace ql
