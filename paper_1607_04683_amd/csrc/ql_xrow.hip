// ql_xrow.hip -- stacked LSTM layers (Section 4), all without or all with a
// projection, at one batch row, the live stream: one persistent launch over
// the whole chip, one XCD per layer, run as a wavefront as in ql_xstack.hip.
//
// Up to 32 workgroups of an XCD (each reads its XCC_ID and takes the next free
// slot) own 16 cells of the layer each, and 16 outputs of its projection.
// With one row nothing is bound by arithmetic or bytes, only by the chain from
// h_{t-1} to h_t, so the kernel keeps that chain short: one hand-off a step
// (h_t itself, in tagged words through the XCD's L2, which every tile then
// quantizes whole; with a projection a second, of m_t), two barriers for each,
// and nothing on it that another wave can do.
//   All eight waves, a lane per cell: poll h_{t-1}, wave min/max, barrier, the
//   row's quantizer (eq. 2, fp64 params) in every lane, its code to LDS,
//   barrier.
//   Waves 0-3, four cells each: the 64 gate rows of W_h', as MFMA fragments in
//   registers, times the codes.  Every column of the B operand is the same
//   row, so the result gives every lane of a group the four gate sums of its
//   cell: lane g takes gate g.  Recovery (eq. 1 / eq. 3), + (W_x x + b) from
//   LDS, the gate; the four gates of a cell meet by DPP; c, m_t (h_t without a
//   projection), published at once by each wave.
//   With a projection, m_t is taken as h_{t-1} was, and wave 0 multiplies its
//   codes with the tile's 16 rows of W_r' and publishes h_t.
//   Waves 4-7 meanwhile: the tile's part of the quantized output of step t-1,
//   as tagged words for the next layer; then W_x' x_{t+1} + b for LDS.  Each
//   takes all of x_{t+1} for itself (1 KB of tagged words the layer before
//   wrote, or the launch's input codes), loaded a step and a half ahead, so
//   that crossing from another XCD costs nothing.
// The words of a step parity are rewritten only two steps later, after every
// tile has read them (a tile publishes h_t only after all its waves have read
// h_{t-1}); the codes for the next layer have a slot for every frame.  Every
// wait is bounded: on expiry a flag in the workspace is raised and every
// workgroup leaves.  The arithmetic is that of k_stack, k_pstack and the
// one-layer path, so the results are bit-identical to them.
// 5 x 500 cells, us a frame: 1.9 (k_stack, with its products and gates on the
// whole workgroup between barriers and two waves quantizing: 4.2).
#include "ql_device.h"
#include "ql_exchange.h"
#include "ql_launch.h"
#include "ql_rec_common.h"
#include "ql_xcd.h"

#include <algorithm>
#include <type_traits>

namespace ql {

constexpr int kXwThreads = 512;
constexpr int kXwXcds = 8, kXwSlots = 32;  // XCDs of the MI355X, CUs of one
constexpr int kXwCells = 16;               // cells of a tile
constexpr int kXwMaxW = 512;               // widths (cells, input)
constexpr int kXwSlotBytes = kXwXcds * 64;

// Exchange words of a layer of H cells whose h_t has R values: h [2 parities][R],
// with a projection m [2][H], then per frame the codes of h_t (a word of four
// codes each), z and 1/Q.
__host__ __device__ inline int64_t xrow_frame_words(int64_t R) { return (R + 3) / 4 + 2; }
__host__ __device__ inline int64_t xrow_words(int64_t H, int64_t R, bool proj, int64_t T) {
  return (T < 2 ? T : 2) * (R + (proj ? H : 0)) + T * xrow_frame_words(R);
}

// What a wave of the input side holds of one x_t: two words of four codes (8
// codes from 8 lane on) and the row's z and 1/Q, with their tags.
struct XRowX {
  uint64_t w[2], z, q;
};

// Cells, and values of h, of layer l.
__host__ __device__ inline int64_t xrow_cells(const StackArgs &a, int) { return a.H; }
__host__ __device__ inline int64_t xrow_cells(const PStackArgs &a, int l) { return a.L[l].H; }
__host__ __device__ inline int64_t xrow_width(const StackArgs &a, int) { return a.H; }
__host__ __device__ inline int64_t xrow_width(const PStackArgs &a, int l) { return a.L[l].P; }

template <class Args, bool TP>
__global__ __launch_bounds__(kXwThreads) void k_xrow(Args a) {
  constexpr bool PROJ = std::is_same<Args, PStackArgs>::value;
  __shared__ __attribute__((aligned(16))) int8_t s_xh[kXwMaxW];       // codes of h_{t-1}
  __shared__ __attribute__((aligned(16))) int8_t s_xm[PROJ ? kXwMaxW : 4];  // codes of m_t
  __shared__ __attribute__((aligned(16))) int8_t s_xx[4][kXwMaxW];    // codes of x, a copy per wave
  __shared__ __attribute__((aligned(16))) int s_red[2 * kXwThreads / 64];  // min/max keys per wave
  __shared__ float s_xb[2][4 * kXwCells];                             // W_x x + b, by step parity
  __shared__ int s_abort, s_role;

  if (threadIdx.x == 0) {
    const int xcc = (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & 15);
    unsigned *slots = reinterpret_cast<unsigned *>(static_cast<char *>(a.ws) + kHeaderBytes);
    s_role = -1;
    s_abort = 0;
    if (xcc < a.nl) {
      const unsigned k = __hip_atomic_fetch_add(slots + xcc * 16, 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
      if (k < (unsigned)kXwSlots) s_role = xcc * kXwSlots + (int)k;
    }
  }
  __syncthreads();
  const int role = __builtin_amdgcn_readfirstlane(s_role);
  if (role < 0) return;
  const int l = role / kXwSlots, tile = role % kXwSlots;
  const auto &Ly = a.L[l];
  const int T = (int)a.T, H = (int)xrow_cells(a, l), R = (int)xrow_width(a, l), IN = (int)Ly.in;
  const int j0 = tile * kXwCells;
  if (j0 >= H && j0 >= R) return;
  int *flag = reinterpret_cast<int *>(a.ws) + kHdrFlag;
  const int64_t fw = xrow_frame_words(R);
  uint64_t *hx = reinterpret_cast<uint64_t *>(static_cast<char *>(a.ws) + kHeaderBytes + kXwSlotBytes);
  for (int k = 0; k < l; ++k) hx += xrow_words(xrow_cells(a, k), xrow_width(a, k), PROJ, T);
  uint64_t *mx = hx + (int64_t)std::min(T, 2) * R;
  uint64_t *cx = mx + (PROJ ? (int64_t)std::min(T, 2) * H : 0);
  // the layer before's codes (its h_t has IN values)
  const int64_t fwin = xrow_frame_words(IN);
  const uint64_t *cin = l > 0 ? hx - (int64_t)T * fwin : nullptr;

  const int tid = threadIdx.x, lane = tid & 63, fr = lane & 15, fq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool hside = wave < 4;
  const int bw = wave & 3;

  // ---- prologue: this wave's fragments (block of cells 4 bw .. + 3; row r of a
  // block is gate r & 3 of cell r >> 2) and this lane's gate of its cell
  const WeightMat W = hside ? Ly.Wh : Ly.Wx;
  const int K = hside ? R : IN;
  v4i wf[8];
  {
    const int j = j0 + 4 * bw + (fr >> 2);
    const int8_t *src = W.codes + ((int64_t)(fr & 3) * H + std::min(j, H - 1)) * W.ld + 16 * fq;
#pragma unroll
    for (int c = 0; c < 8; ++c)
      wf[c] = j < H && c * 64 < K ? *reinterpret_cast<const v4i *>(src + c * 64) : v4i{};
  }
  const int gate = fr & 3, cell = j0 + 4 * bw + fq;
  const bool live = cell < H;
  int32_t ztw, sigw;
  int64_t colterm;
  float iqw, bias;
  {
    const int64_t n = (int64_t)gate * H + std::min(cell, H - 1), blk = n / W.rows_per_block;
    ztw = W.zero[blk] + 128;
    sigw = W.row_sums[n] - 128 * K;
    colterm = (int64_t)sigw + (int64_t)K * ztw;
    iqw = W.inv_q[blk];
    bias = Ly.bias[n];
  }
  float cst = hside && live && Ly.c0 ? Ly.c0[cell] : 0.0f;
  // the projection's rows (wave 0): row r of the block is output j0 + r
  v4i wr[PROJ ? 8 : 1];
  int32_t rztw = 0, rsigw = 0;
  int64_t rcolterm = 0;
  float riqw = 0.0f;
  const int out = j0 + 4 * fq + gate;
  if constexpr (PROJ) {
    const int p = j0 + fr;
    const int8_t *src = Ly.Wr.codes + (int64_t)std::min(p, R - 1) * Ly.Wr.ld + 16 * fq;
#pragma unroll
    for (int c = 0; c < 8; ++c)
      wr[c] = p < R && c * 64 < H ? *reinterpret_cast<const v4i *>(src + c * 64) : v4i{};
    const int64_t n = std::min(out, R - 1), blk = n / Ly.Wr.rows_per_block;
    rztw = Ly.Wr.zero[blk] + 128;
    rsigw = Ly.Wr.row_sums[n] - 128 * H;
    rcolterm = (int64_t)rsigw + (int64_t)H * rztw;
    riqw = Ly.Wr.inv_q[blk];
  }
  // padding bytes stay zero, so that products and code sums run over all of a row
  for (int i = tid; i < kXwMaxW / 4; i += kXwThreads) {
    reinterpret_cast<int *>(s_xh)[i] = 0;
    if (PROJ) reinterpret_cast<int *>(s_xm)[i] = 0;
  }
  for (int i = tid; i < kXwMaxW; i += kXwThreads) reinterpret_cast<int *>(s_xx[0])[i] = 0;

  // The product of 512 codes in LDS with a block of fragments, and their sum (as
  // signed codes): the lane's row (gate) of its group's four.
  const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
  auto product = [&](const int8_t *codes, const v4i *w, int32_t &sum) -> int32_t {
    v4i acc[2] = {v4i{}, v4i{}}, sm[2] = {v4i{}, v4i{}};
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const v4i b = *reinterpret_cast<const v4i *>(codes + c * 64 + 16 * fq);
      acc[c & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[c], b, acc[c & 1], 0, 0, 0);
      sm[c & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, b, sm[c & 1], 0, 0, 0);
    }
    // the results are read by ordinary instructions: at least 19 wait states
    // after the last pass, which the hardware does not check
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(acc[0]), "+v"(acc[1]), "+v"(sm[0]), "+v"(sm[1]));
    sum = sm[0][0] + sm[1][0];
    const int32_t s0 = acc[0][0] + acc[1][0], s1 = acc[0][1] + acc[1][1],
                  s2 = acc[0][2] + acc[1][2], s3 = acc[0][3] + acc[1][3];
    return gate < 2 ? (gate == 0 ? s0 : s1) : (gate == 2 ? s2 : s3);
  };

  // ---- the input side
  const int nwx = (IN + 3) / 4;  // words of four codes of a row the layer before writes
  auto issue_x = [&](int t, XRowX &x) {
    if (cin) {
      const uint64_t *src = cin + (int64_t)t * fwin;
      x.w[0] = ld_tagged(src + std::min(2 * lane, nwx - 1));
      x.w[1] = ld_tagged(src + std::min(2 * lane + 1, nwx - 1));
      x.z = ld_tagged(src + nwx);
      x.q = ld_tagged(src + nwx + 1);
    } else {
      const int o = std::min(8 * lane, (IN - 1) / 8 * 8);  // (a row's stride is a multiple of 64)
      x.w[0] = *reinterpret_cast<const uint64_t *>(Ly.xin.codes + (int64_t)t * Ly.xin.ld + o);
      x.w[1] = 0;
      x.z = (uint32_t)Ly.xin.zero[t];
      x.q = __float_as_uint(Ly.xin.inv_q[t]);
    }
  };
  // W_x x_t + b of the tile's cells into s_xb, from x's words
  auto use_x = [&](int t, XRowX &x) {
    uint64_t codes;
    if (cin) {
      const uint32_t tag = (uint32_t)(t + 1);
      long it = 0;
      for (;;) {
        const uint32_t bad = ((uint32_t)(x.w[0] >> 32) ^ tag) | ((uint32_t)(x.w[1] >> 32) ^ tag) |
                             ((uint32_t)(x.z >> 32) ^ tag) | ((uint32_t)(x.q >> 32) ^ tag);
        if (!__any(bad != 0)) break;
        if (wait_expired(flag, it)) {
          s_abort = 1;
          break;
        }
        issue_x(t, x);
      }
      codes = (x.w[0] & 0xffffffffull) | (x.w[1] << 32);
      if (2 * lane + 1 >= nwx) codes &= 0xffffffffull;
      if (2 * lane >= nwx) codes = 0;
    } else {
      codes = 8 * lane < IN ? x.w[0] : 0;
    }
    *reinterpret_cast<uint64_t *>(s_xx[bw] + 8 * lane) = codes;
    const int32_t z = (int32_t)(uint32_t)x.z;
    const float iq = __uint_as_float((uint32_t)x.q);
    int32_t sig;
    const int32_t S = product(s_xx[bw], wf, sig);
    const float y = recover(S, colterm, ztw, z + 128, sig, iqw, iq);
    if (fr < 4) s_xb[t & 1][4 * (4 * bw + fq) + gate] = y + bias;
    if (TP && Ly.acc_x && fr < 4 && live)
      Ly.acc_x[((int64_t)t * 4 + gate) * H + cell] = acc_u8(S, sigw, sig, IN);
  };

  // ---- a row of n values: polled (tag > 0; else from init, null: zeros),
  // quantized, its codes in LDS; z and 1/Q in every lane
  int stop = 0;
  auto take = [&](const uint64_t *words, const float *init, int n, uint32_t tag, int8_t *codes,
                  int32_t &z, float &iq, auto after_poll) {
    float v = 0.0f;
    if (tag == 0) {
      if (init && tid < n) v = init[tid];
    } else {
      const uint64_t *src = words + std::min(tid, n - 1);
      long it = 0;
      for (;;) {
        const uint64_t w = ld_tagged(src);
        v = __uint_as_float((uint32_t)w);
        if (!__any((uint32_t)(w >> 32) != tag)) break;
        if (wait_expired(flag, it)) {
          s_abort = 1;
          break;
        }
      }
    }
    after_poll();
    int mm[2] = {0x7fffffff, 0x7fffffff};
    if (tid < n) {
      const int key = float_key(v);
      mm[0] = key;
      mm[1] = ~key;
    }
    wave_min_n<2>(mm);
    if (lane == 0) *reinterpret_cast<int2 *>(s_red + 2 * wave) = make_int2(mm[0], mm[1]);
    __syncthreads();
    stop |= __builtin_amdgcn_readfirstlane(s_abort);  // (written outside these two barriers only)
    int lo = 0x7fffffff, hi = 0x7fffffff;
#pragma unroll
    for (int w = 0; w < kXwThreads / 128; ++w) {
      const int4 q = reinterpret_cast<const int4 *>(s_red)[w];
      lo = min(lo, min(q.x, q.z));
      hi = min(hi, min(q.y, q.w));
    }
    const QParams p = make_qparams(key_float(lo), key_float(~hi));
    z = p.z;
    iq = p.inv_q;
    if (tid < n) codes[tid] = (int8_t)(encode(v, p.q, p.z) ^ 0x80);
    __syncthreads();
  };
  int32_t hz = 0;
  float hiq = 0.0f;
  XRowX xe{}, xo{};  // x of even and odd steps
  auto take_h = [&](int t, XRowX &xnext) {
    take(hx + ((t - 1) & 1) * R, Ly.h0, R, (uint32_t)t, s_xh, hz, hiq, [&]() {
      // x_{t+2}, for the window after the next barriers but one (past the end:
      // x_{T-1} again, never used)
      if (!hside) issue_x(std::min(t + 2, T - 1), xnext);
    });
  };

  // ---- this tile's part of the layer's quantized output of step t (h's codes
  // are in LDS): waves 4 (codes) and 5 (the row's params, tile 0)
  const int nout = (R + kXwCells - 1) / kXwCells;  // tiles with values of h
  auto put_out = [&](int t) {
    uint64_t *dst = cx + (int64_t)t * fw;
    if (wave == 4 && lane < 4) {
      const int wd = j0 / 4 + lane;  // (cells past H: code byte 0)
      const uint32_t codes = reinterpret_cast<const uint32_t *>(s_xh)[wd];
      if (4 * wd < R) st_coherent64(dst + wd, ((uint64_t)(uint32_t)(t + 1) << 32) | codes);
      if (4 * wd < Ly.out.ld) reinterpret_cast<uint32_t *>(Ly.out.codes + (int64_t)t * Ly.out.ld)[wd] = codes;
    }
    if (wave == 5) {
      if (tile == 0) {
        const int nw = (R + 3) / 4;
        if (lane < 2)
          st_coherent64(dst + nw + lane, ((uint64_t)(uint32_t)(t + 1) << 32) |
                                             (lane ? __float_as_uint(hiq) : (uint32_t)hz));
        int sum = 0;
#pragma unroll
        for (int k = 0; k < 2; ++k)
          sum = __builtin_amdgcn_sdot4(reinterpret_cast<const int *>(s_xh)[2 * lane + k], 0x01010101, sum,
                                       false);
        sum = wave_sum(sum);
        if (lane == 0) {
          Ly.out.zero[t] = hz;
          Ly.out.inv_q[t] = hiq;
          Ly.out.sums[t] = sum + 128 * R;
          if (Ly.tap_zero) Ly.tap_zero[t] = hz;
          if (Ly.tap_inv_q) Ly.tap_inv_q[t] = hiq;
        }
      }
      if (tile == nout - 1)
        for (int64_t i = (int64_t)nout * kXwCells + 4 * lane; i < Ly.out.ld; i += 256)
          *reinterpret_cast<uint32_t *>(Ly.out.codes + (int64_t)t * Ly.out.ld + i) = 0u;
      if (Ly.tap_codes && lane < kXwCells && j0 + lane < R)
        Ly.tap_codes[(int64_t)t * R + j0 + lane] = s_xh[j0 + lane];
    }
  };

  // ---- one step: x (in hand since the step before) is x_{t+1}, xnext's words
  // are loaded for x_{t+2}
  auto step = [&](int t, XRowX &x, XRowX &xnext) {
    take_h(t, xnext);
    if (hside) {
      int32_t sig;
      const int32_t S = product(s_xh, wf, sig);
      const float y = recover(S, colterm, ztw, hz + 128, sig, iqw, hiq);
      const float av = s_xb[t & 1][4 * (4 * bw + fq) + gate] + y;
      const float sg = sigmoid_cw(gate == 2 ? 2.0f * av : av);
      const float act = gate == 2 ? 2.0f * sg - 1.0f : sg;
      const float ig = quad_bcast<0>(act), fg = quad_bcast<1>(act), gv = quad_bcast<2>(act),
                  og = quad_bcast<3>(act);
      const float cn = (fg * cst) + (ig * gv);
      cst = cn;
      const float m = og * tanh_cw(cn);
      if (fr == 0 && live) {
        put_word((PROJ ? mx : hx) + (t & 1) * H + cell, (uint32_t)(t + 1), __float_as_uint(m));
        if (!PROJ && Ly.h) Ly.h[(int64_t)t * H + cell] = m;
        if (TP) {
          if (Ly.tap_c) Ly.tap_c[(int64_t)t * H + cell] = cn;
          if (Ly.tap_m) Ly.tap_m[(int64_t)t * H + cell] = m;
          if (t == T - 1) {
            if (!PROJ && Ly.hT) Ly.hT[cell] = m;
            if (Ly.cT) Ly.cT[cell] = cn;
          }
        }
      }
      if (TP && fr < 4 && live) {
        if (Ly.acc_h) Ly.acc_h[((int64_t)t * 4 + gate) * H + cell] = acc_u8(S, sigw, sig, R);
        if (Ly.tap_gates) Ly.tap_gates[((int64_t)t * 4 + gate) * H + cell] = act;
      }
    } else {
      if (t > 0) put_out(t - 1);
      if (!PROJ && t + 1 < T) use_x(t + 1, x);
    }
    if constexpr (PROJ) {
      int32_t mz;
      float miq;
      take(mx + (t & 1) * H, nullptr, H, (uint32_t)(t + 1), s_xm, mz, miq, []() {});
      if (wave == 0) {
        int32_t sig;
        const int32_t S = product(s_xm, wr, sig);
        const float h = recover(S, rcolterm, rztw, mz + 128, sig, riqw, miq);
        if (fr < 4 && out < R) {
          put_word(hx + (t & 1) * R + out, (uint32_t)(t + 1), __float_as_uint(h));
          if (Ly.h) Ly.h[(int64_t)t * R + out] = h;
          if (TP && Ly.acc_r) Ly.acc_r[(int64_t)t * R + out] = acc_u8(S, rsigw, sig, H);
          if (TP && t == T - 1 && Ly.hT) Ly.hT[out] = h;
        }
      } else if (!hside && t + 1 < T) {
        use_x(t + 1, x);
      }
    }
  };

  if (!hside) {
    issue_x(0, xe);
    issue_x(std::min(1, T - 1), xo);
  }
  __syncthreads();  // LDS is zeroed
  if (!hside) use_x(0, xe);
  int t = 0;
  for (;;) {
    step(t, xo, xe);
    if (stop || ++t == T) break;
    step(t, xe, xo);
    if (stop || ++t == T) break;
  }
  if (stop) return;
  // the last step's output
  take_h(T, xe);
  if (stop) return;
  if (!hside) put_out(T - 1);
}

// ------------------------------------------------------------------ host side
// Whether the layout takes a; its exchange words.
template <class Args>
static bool plan_xrow(const Args &a, size_t ws_bytes, int cus, int64_t *words_out) {
  constexpr bool PROJ = std::is_same<Args, PStackArgs>::value;
  if (cus != kXwXcds * kXwSlots || a.nl < 1 || a.nl > kXwXcds || a.T < 1 || a.T >= (1 << 30))
    return false;
  int64_t words = 0;
  for (int l = 0; l < a.nl; ++l) {
    const auto &L = a.L[l];
    const int64_t H = xrow_cells(a, l), R = xrow_width(a, l);
    if (H < 1 || H > kXwMaxW || R < 1 || R > kXwMaxW || L.in < 1 || L.in > kXwMaxW) return false;
    if (l > 0 && L.in != xrow_width(a, l - 1)) return false;
    if (L.Wx.ld < round_up(L.in, 64) || L.Wh.ld < round_up(R, 64)) return false;
    if constexpr (PROJ)
      if (L.Wr.ld < round_up(H, 64)) return false;
    if (L.out.ld < R || L.out.ld % 4) return false;
    words += xrow_words(H, R, PROJ, a.T);
  }
  if (a.L[0].xin.ld % 8 || a.L[0].xin.ld < a.L[0].in) return false;
  *words_out = words;
  return kHeaderBytes + kXwSlotBytes + (size_t)words * 8 <= ws_bytes;
}

template <class Args>
static hipError_t launch_xrow_any(const Args &a, size_t ws_bytes, int cus, bool taps, hipStream_t s,
                                  bool *done) {
  *done = false;
  int64_t words = 0;
  if (!plan_xrow(a, ws_bytes, cus, &words)) return hipSuccess;
  auto kern = taps ? k_xrow<Args, true> : k_xrow<Args, false>;
  // more than half of a CU's LDS, so that a CU holds one workgroup
  const size_t lds = 84 * 1024;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kXwThreads, lds);
  if (e != hipSuccess) return e;
  if (per_cu < 1) return hipSuccess;
  e = clear_exchange(a.ws, kXwSlotBytes / 8 + words, s);
  if (e != hipSuccess) return e;
  Args args = a;
  void *kargs[] = {&args};
  e = hipLaunchCooperativeKernel(reinterpret_cast<void *>(kern), dim3(cus), dim3(kXwThreads), kargs,
                                 (unsigned)lds, s);
  if (e == hipSuccess) *done = true;
  return e;
}

hipError_t launch_xrow(const StackArgs &a, size_t ws_bytes, int cus, bool taps, hipStream_t s,
                       bool *done) {
  *done = false;
  if (a.B != 1) return hipSuccess;
  return launch_xrow_any(a, ws_bytes, cus, taps, s, done);
}
hipError_t launch_xrow(const PStackArgs &a, size_t ws_bytes, int cus, bool taps, hipStream_t s,
                       bool *done) {
  return launch_xrow_any(a, ws_bytes, cus, taps, s, done);
}

bool xrow_applies(const StackArgs &a, size_t ws_bytes, int cus) {
  int64_t words;
  return a.B == 1 && plan_xrow(a, ws_bytes, cus, &words);
}
bool xrow_applies(const PStackArgs &a, size_t ws_bytes, int cus) {
  int64_t words;
  return plan_xrow(a, ws_bytes, cus, &words);
}

hipError_t set_wait_bound_xrow(int polls) { return set_wait_bound_here(polls); }

}  // namespace ql
