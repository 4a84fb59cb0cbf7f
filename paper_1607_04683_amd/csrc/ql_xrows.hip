// ql_xrows.hip -- stacked LSTM layers (Section 4), all without or all with a
// projection, at a few batch rows per group: the one-row kernel's chain
// (ql_xrow.hip) for up to eight rows, one persistent launch over the whole
// chip, one XCD per layer and row group, run as a wavefront.
//
// A row group is up to NR rows (4, or 8 with a projection); n layers leave room for
// floor(8 / n) groups a launch, and larger batches with projections take several
// launches where those pay.  Up to 32 workgroups of an XCD own 16 cells of the
// layer each, and 16 outputs of its projection.  Waves 0-3 carry the chain from h_{t-1} to h_t: NR / 4 rows each,
// 64 values an instruction, polled in tagged words through the XCD's L2,
// quantized in the wave (eq. 2), the codes to LDS, one barrier; then the 64 gate
// rows of W_h' times the codes, rows in the columns of the MFMA.  The rows
// repeat in its 16 columns, so a lane has the four gate sums of one (cell, row)
// pair and computes NR / 4 of its gates, which meet by lane exchange; c, m_t
// (h_t without a projection), published at once.  With a projection, m_t is
// taken the same way and wave 0 multiplies its codes with the tile's 16 rows of
// W_r'.  Waves 4-7 never touch the chain: the quantized output of step t-1 as
// tagged words for the next layer, W_x' x_{t+1} + b from codes that came to LDS
// a step ago, the codes of x_{t+2} to LDS, the loads of x_{t+3}.  Buffers that
// both halves touch alternate by step parity.  Exchange words, their reuse and
// the bounded waits are those of ql_xrow.hip; the results are bit-identical to
// the one-layer path's.
#include "ql_device.h"
#include "ql_exchange.h"
#include "ql_launch.h"
#include "ql_rec_common.h"
#include "ql_xcd.h"

#include <algorithm>
#include <type_traits>

namespace ql {

constexpr int kXvThreads = 512;
constexpr int kXvXcds = 8, kXvSlots = 32;  // XCDs of the MI355X, CUs of one
constexpr int kXvCells = 16;               // cells of a tile
constexpr int kXvMaxW = 512;               // widths (cells, projection, input)
constexpr int kXvLds = kXvMaxW + 16;       // row stride of codes in LDS
constexpr int kXvSlotBytes = kXvXcds * 64;

struct XvTiling {
  int ng, rows;    // row groups, and batch rows per group (the last may hold fewer)
  int64_t r0, r1;  // batch rows [r0, r1) of this launch
  uint64_t *words; // exchange words
};
struct XvRow {
  int32_t z;
  float iq;
};

// Exchange words of a layer of one group of `rows` rows: h [2 parities][rows][R],
// with a projection m [2][rows][H], then per frame and row the codes of h_t (a
// word of four codes each), z and 1/Q.
__host__ __device__ inline int64_t xv_frame_words(int64_t R) { return (R + 3) / 4 + 2; }
__host__ __device__ inline int64_t xv_words(int64_t H, int64_t R, bool proj, int64_t T, int64_t rows) {
  return rows * ((T < 2 ? T : 2) * (R + (proj ? H : 0)) + T * xv_frame_words(R));
}
// Cells, and values of h, of layer l.
__host__ __device__ inline int64_t xv_cells(const StackArgs &a, int) { return a.H; }
__host__ __device__ inline int64_t xv_cells(const PStackArgs &a, int l) { return a.L[l].H; }
__host__ __device__ inline int64_t xv_width(const StackArgs &a, int) { return a.H; }
__host__ __device__ inline int64_t xv_width(const PStackArgs &a, int l) { return a.L[l].P; }

template <class Args, int NR, bool TP>
__global__ __launch_bounds__(kXvThreads) void k_xrows(Args a, XvTiling tl) {
  constexpr bool PROJ = std::is_same<Args, PStackArgs>::value;
  constexpr int RW = NR / 4;  // rows per quantizing and per input wave; gates per lane
  __shared__ __attribute__((aligned(16))) int8_t s_xh[2][NR][kXvLds];  // codes of h, by parity
  __shared__ __attribute__((aligned(16))) int8_t s_xx[2][NR][kXvLds];  // codes of x, by parity
  __shared__ __attribute__((aligned(16))) int8_t s_xm[PROJ ? NR : 1][kXvLds];  // codes of m_t
  // the projection's fragments: in wave 0's registers, or with eight rows, whose
  // polls take the registers, in LDS
  constexpr bool WRL = PROJ && NR == 8;
  __shared__ __attribute__((aligned(16))) int8_t s_wr[WRL ? 16 : 1][kXvLds];
  __shared__ XvRow s_hp[2][NR], s_xp[2][NR], s_mp[NR];
  __shared__ float s_xb[2][NR][4 * kXvCells];  // W_x x + b, by parity
  // expired waits, by the parity of the barrier that the writer has yet to pass:
  // after a barrier only its own word is read, which nobody writes before the
  // next one, so every wave leaves at the same barrier
  __shared__ int s_abort[2], s_role;

  if (threadIdx.x == 0) {
    const int xcc = (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & 15);
    unsigned *slots = reinterpret_cast<unsigned *>(static_cast<char *>(a.ws) + kHeaderBytes);
    s_role = -1;
    s_abort[0] = s_abort[1] = 0;
    if (xcc < a.nl * tl.ng) {
      const unsigned k = __hip_atomic_fetch_add(slots + xcc * 16, 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
      if (k < (unsigned)kXvSlots) s_role = xcc * kXvSlots + (int)k;
    }
  }
  __syncthreads();
  const int role = __builtin_amdgcn_readfirstlane(s_role);
  if (role < 0) return;
  const int l = (role / kXvSlots) % a.nl, g = (role / kXvSlots) / a.nl, tile = role % kXvSlots;
  const auto &Ly = a.L[l];
  const int T = (int)a.T, H = (int)xv_cells(a, l), R = (int)xv_width(a, l), IN = (int)Ly.in;
  const int64_t B = a.B, b0 = tl.r0 + (int64_t)g * tl.rows;
  const int nb = (int)std::min<int64_t>(tl.rows, tl.r1 - b0), rows = tl.rows;
  const int j0 = tile * kXvCells;
  if ((j0 >= H && j0 >= R) || nb <= 0) return;
  int *flag = reinterpret_cast<int *>(a.ws) + kHdrFlag;
  const int64_t fw = xv_frame_words(R), fwin = xv_frame_words(IN);
  uint64_t *hx = tl.words;
  for (int k = 0; k < a.nl; ++k)
    hx += (int64_t)(k < l ? g + 1 : g) * xv_words(xv_cells(a, k), xv_width(a, k), PROJ, T, rows);
  const int par = std::min(T, 2);
  uint64_t *mx = hx + (int64_t)par * rows * R;
  uint64_t *cx = mx + (PROJ ? (int64_t)par * rows * H : 0);
  // the layer before's codes of the same group: the last words of its area,
  // which lies right before this layer's when areas go group by group
  const uint64_t *cin = l > 0 ? hx - (int64_t)T * rows * fwin : nullptr;

  const int tid = threadIdx.x, lane = tid & 63, fr = lane & 15, fq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool hside = wave < 4;
  const int bw = wave & 3;
  // the lane's (cell, row) pair, and its gates gate0 .. + RW - 1
  const int row = fr & (NR - 1), gate0 = fr / NR * RW;
  const int cl = 4 * bw + fq, cell = j0 + cl;
  const bool live = cell < H && row < nb;
  const int64_t brow = b0 + std::min(row, nb - 1);

  // ---- prologue: this wave's fragments (block of cells 4 bw .. + 3; row r of a
  // block is gate r & 3 of cell r >> 2) and the column params of this lane's gates
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
  struct Col {
    int32_t ztw, sigw;
    int64_t colterm;
    float iqw, bias;
  };
  auto col = [](const WeightMat &M, int64_t n, int Kc) {
    const int64_t blk = n / M.rows_per_block;
    Col c;
    c.ztw = M.zero[blk] + 128;
    c.sigw = M.row_sums[n] - 128 * Kc;
    c.colterm = (int64_t)c.sigw + (int64_t)Kc * c.ztw;
    c.iqw = M.inv_q[blk];
    c.bias = 0.0f;
    return c;
  };
  Col cp[RW];
#pragma unroll
  for (int k = 0; k < RW; ++k) {
    const int64_t n = (int64_t)(gate0 + k) * H + std::min(cell, H - 1);
    cp[k] = col(W, n, K);
    cp[k].bias = Ly.bias[n];
  }
  float cst = hside && live && Ly.c0 ? Ly.c0[brow * H + cell] : 0.0f;
  // the projection's rows (wave 0): row r of the block is output j0 + r; this
  // lane's outputs out0 .. + RW - 1 of its row
  v4i wr[PROJ && !WRL ? 8 : 1];
  Col rp[PROJ ? RW : 1];
  const int out0 = j0 + 4 * fq + gate0;
  if constexpr (PROJ) {
    const int p = j0 + fr;
    const int8_t *src = Ly.Wr.codes + (int64_t)std::min(p, R - 1) * Ly.Wr.ld + 16 * fq;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const v4i w = p < R && c * 64 < H ? *reinterpret_cast<const v4i *>(src + c * 64) : v4i{};
      if constexpr (WRL) {
        if (wave == 0) *reinterpret_cast<v4i *>(s_wr[fr] + c * 64 + 16 * fq) = w;
      } else {
        wr[c] = w;
      }
    }
#pragma unroll
    for (int k = 0; k < RW; ++k) rp[k] = col(Ly.Wr, std::min(out0 + k, R - 1), H);
  }
  // bytes past the widths and rows past the group stay zero
  for (int i = tid; i < 2 * NR * kXvLds / 4; i += kXvThreads) {
    reinterpret_cast<int *>(s_xh)[i] = 0;
    reinterpret_cast<int *>(s_xx)[i] = 0;
  }
  if (PROJ)
    for (int i = tid; i < NR * kXvLds / 4; i += kXvThreads) reinterpret_cast<int *>(s_xm)[i] = 0;
  if (tid < 2 * NR) s_hp[0][tid] = s_xp[0][tid] = XvRow{0, 0.0f};
  if (tid < NR) s_mp[tid] = XvRow{0, 0.0f};

  // The product of the rows' codes in LDS with a block of fragments, and their
  // sums (as signed codes): the lane's gates (outputs) of its pair.
  const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
  auto product = [&](const int8_t *codes, auto frag, int32_t(&S)[RW], int32_t &sum) __attribute__((always_inline)) {
    v4i acc[2] = {v4i{}, v4i{}}, sm[2] = {v4i{}, v4i{}};
    const int8_t *x = codes + row * kXvLds + 16 * fq;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const v4i b = *reinterpret_cast<const v4i *>(x + c * 64);
      acc[c & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(frag(c), b, acc[c & 1], 0, 0, 0);
      sm[c & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, b, sm[c & 1], 0, 0, 0);
    }
    // the results are read by ordinary instructions: at least 19 wait states
    // after the last pass, which the hardware does not check
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(acc[0]), "+v"(acc[1]), "+v"(sm[0]), "+v"(sm[1]));
    sum = sm[0][0] + sm[1][0];
    int32_t s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = acc[0][i] + acc[1][i];
    if constexpr (RW == 1) {
      S[0] = gate0 < 2 ? (gate0 == 0 ? s[0] : s[1]) : (gate0 == 2 ? s[2] : s[3]);
    } else {
      S[0] = gate0 == 0 ? s[0] : s[2];
      S[1] = gate0 == 0 ? s[1] : s[3];
    }
  };

  // ---- the input side: wave 4 + bw takes rows bw RW .. + RW - 1
  const int nwx = (IN + 3) / 4;  // words of four codes of a row the layer before writes
  uint64_t xw[RW][2], xz[RW], xq[RW];
  auto issue_x = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const int lr = std::min(bw * RW + r, nb - 1);
      if (cin) {
        const uint64_t *src = cin + ((int64_t)t * rows + lr) * fwin;
        xw[r][0] = ld_tagged(src + std::min(2 * lane, nwx - 1));
        xw[r][1] = ld_tagged(src + std::min(2 * lane + 1, nwx - 1));
        xz[r] = ld_tagged(src + nwx);
        xq[r] = ld_tagged(src + nwx + 1);
      } else {
        const int64_t o = (int64_t)t * B + b0 + lr;
        // (a row's stride is a multiple of 64)
        xw[r][0] = *reinterpret_cast<const uint64_t *>(Ly.xin.codes + o * Ly.xin.ld +
                                                       std::min(8 * lane, (IN - 1) / 8 * 8));
        xw[r][1] = 0;
        xz[r] = (uint32_t)Ly.xin.zero[o];
        xq[r] = __float_as_uint(Ly.xin.inv_q[o]);
      }
    }
  };
  int turn = 0, stop = 0;  // parity of the next barrier (those of `take`); an expired wait
  // the words of x_t, once they carry its tag, to LDS
  auto land_x = [&](int t) __attribute__((always_inline)) {
    if (cin) {
      const uint32_t tag = (uint32_t)(t + 1);
      long it = 0;
      for (;;) {
        uint32_t bad = 0;
#pragma unroll
        for (int r = 0; r < RW; ++r)
          bad |= ((uint32_t)(xw[r][0] >> 32) ^ tag) | ((uint32_t)(xw[r][1] >> 32) ^ tag) |
                 ((uint32_t)(xz[r] >> 32) ^ tag) | ((uint32_t)(xq[r] >> 32) ^ tag);
        if (!__any(bad != 0)) break;
        if (wait_expired(flag, it)) {
          s_abort[turn] = 1;
          break;
        }
        issue_x(t);
      }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const int lr = bw * RW + r;
      uint64_t codes;
      if (cin) {
        codes = (xw[r][0] & 0xffffffffull) | (xw[r][1] << 32);
        if (2 * lane + 1 >= nwx) codes &= 0xffffffffull;
        if (2 * lane >= nwx) codes = 0;
      } else {
        codes = 8 * lane < IN ? xw[r][0] : 0;
      }
      if (lr < nb) {
        *reinterpret_cast<uint64_t *>(s_xx[t & 1][lr] + 8 * lane) = codes;
        if (lane == 0)
          s_xp[t & 1][lr] = XvRow{(int32_t)(uint32_t)xz[r], __uint_as_float((uint32_t)xq[r])};
      }
    }
  };
  // W_x x_t + b of the tile's cells into s_xb
  auto use_x = [&](int t) __attribute__((always_inline)) {
    int32_t S[RW], sig;
    product(s_xx[t & 1][0], [&](int c) { return wf[c]; }, S, sig);
    const XvRow p = s_xp[t & 1][row];
#pragma unroll
    for (int k = 0; k < RW; ++k) {
      const float y = recover(S[k], cp[k].colterm, cp[k].ztw, p.z + 128, sig, cp[k].iqw, p.iq);
      s_xb[t & 1][row][4 * cl + gate0 + k] = y + cp[k].bias;
      if (TP && Ly.acc_x && live)
        Ly.acc_x[(((int64_t)t * B + brow) * 4 + gate0 + k) * H + cell] =
            acc_u8(S[k], cp[k].sigw, sig, IN);
    }
  };

  // ---- waves 0-3: rows of n values (a row every n words), polled (tag > 0; else
  // from init, null: zeros), quantized, their codes and params in LDS; ends with
  // the workgroup's barrier
  auto take = [&](const uint64_t *words, const float *init, int n, uint32_t tag, int8_t *codes,
                  XvRow *params) __attribute__((always_inline)) {
    if (hside) {
      float v[RW][8];
      if (tag == 0) {
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int k = 64 * i + lane, lr = bw * RW + r;
            v[r][i] = init && lr < nb && k < n ? init[(b0 + lr) * n + k] : 0.0f;
          }
      } else {
        // a round trip's worth of slack before the first read: with four rows most
        // came too early (P = 200: 4.37 us a step at once, 4.26 so; with eight rows
        // their loads take that long themselves)
        if (RW == 1) __builtin_amdgcn_s_sleep(4);
        long it = 0;
        for (;;) {
          uint64_t w[RW][8];
#pragma unroll
          for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int i = 0; i < 8; ++i)
              w[r][i] = ld_tagged(words + (int64_t)std::min(bw * RW + r, nb - 1) * n +
                                  std::min(64 * i + lane, n - 1));
          uint32_t bad = 0;
#pragma unroll
          for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              bad |= (uint32_t)(w[r][i] >> 32) ^ tag;
              v[r][i] = __uint_as_float((uint32_t)w[r][i]);
            }
          if (!__any(bad != 0)) break;
          if (wait_expired(flag, it)) {
            s_abort[turn] = 1;
            break;
          }
        }
      }
      // (values past n repeat value n - 1, which changes no min or max; at tag
      // 0 they are zeros, and only values below n count)
      int mm[2 * RW];
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        int lo = 0x7fffffff, hi = 0x7fffffff;
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (64 * i + lane < n) {
            const int key = float_key(v[r][i]);
            lo = min(lo, key);
            hi = min(hi, ~key);
          }
        mm[r] = lo;
        mm[RW + r] = hi;
      }
      wave_min_n<2 * RW>(mm);
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        const int lr = bw * RW + r;
        if (lr < nb) {
          const QParams p = make_qparams(key_float(mm[r]), key_float(~mm[RW + r]));
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (64 * i + lane < n)
              codes[lr * kXvLds + 64 * i + lane] = (int8_t)(encode(v[r][i], p.q, p.z) ^ 0x80);
          if (lane == 0) params[lr] = XvRow{p.z, p.inv_q};
        }
      }
    }
    __syncthreads();
    stop |= __builtin_amdgcn_readfirstlane(s_abort[turn]);
    turn ^= 1;
  };
  auto take_h = [&](int t) __attribute__((always_inline)) {
    take(hx + (int64_t)((t - 1) & 1) * rows * R, Ly.h0, R, (uint32_t)t, s_xh[t & 1][0], s_hp[t & 1]);
  };

  // ---- waves 4-7: this tile's part of the layer's quantized output of step t
  // (its codes are in the buffer of parity t + 1), rows bw RW .. + RW - 1
  const int nout = (R + kXvCells - 1) / kXvCells;  // tiles with values of h
  auto put_out = [&](int t) __attribute__((always_inline)) {
    const int hb = (t + 1) & 1;
    const uint64_t tag = (uint64_t)(uint32_t)(t + 1) << 32;
    {
      const int lr = bw * RW + (lane >> 2), wd = j0 / 4 + (lane & 3);  // (cells past R: code byte 0)
      if (lane < 4 * RW && lr < nb) {
        const uint32_t codes = reinterpret_cast<const uint32_t *>(s_xh[hb][lr])[wd];
        if (4 * wd < R) st_coherent64(cx + ((int64_t)t * rows + lr) * fw + wd, tag | codes);
        if (Ly.out.codes && 4 * wd < Ly.out.ld)
          reinterpret_cast<uint32_t *>(Ly.out.codes + ((int64_t)t * B + b0 + lr) * Ly.out.ld)[wd] = codes;
      }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const int lr = bw * RW + r;
      if (lr >= nb) break;
      const int64_t o = (int64_t)t * B + b0 + lr;
      if (tile == 0) {
        const XvRow p = s_hp[hb][lr];
        if (lane < 2)
          st_coherent64(cx + ((int64_t)t * rows + lr) * fw + (R + 3) / 4 + lane,
                        tag | (lane ? __float_as_uint(p.iq) : (uint32_t)p.z));
        if (Ly.out.codes) {
          const int *c = reinterpret_cast<const int *>(s_xh[hb][lr]) + 2 * lane;
          const int sum = wave_sum(__builtin_amdgcn_sdot4(
              c[1], 0x01010101, __builtin_amdgcn_sdot4(c[0], 0x01010101, 0, false), false));
          if (lane == 0) {
            Ly.out.zero[o] = p.z;
            Ly.out.inv_q[o] = p.iq;
            Ly.out.sums[o] = sum + 128 * R;
          }
        }
        if (lane == 0 && Ly.tap_zero) Ly.tap_zero[o] = p.z;
        if (lane == 0 && Ly.tap_inv_q) Ly.tap_inv_q[o] = p.iq;
      }
      if (Ly.out.codes && tile == nout - 1)
        for (int64_t i = (int64_t)nout * kXvCells + 4 * lane; i < Ly.out.ld; i += 256)
          *reinterpret_cast<uint32_t *>(Ly.out.codes + o * Ly.out.ld + i) = 0u;
      if (Ly.tap_codes && lane < kXvCells && j0 + lane < R)
        Ly.tap_codes[o * R + j0 + lane] = s_xh[hb][lr][j0 + lane];
    }
  };

  // ---- x_0 to its product, x_1 to LDS, x_2 in flight
  __syncthreads();  // LDS is zeroed
  if (!hside) {
    issue_x(0);
    land_x(0);
  }
  __syncthreads();
  if (!hside) {
    use_x(0);
    issue_x(std::min(1, T - 1));
    if (T > 1) land_x(1);
    issue_x(std::min(2, T - 1));
  }
  for (int t = 0; t < T; ++t) {
    take_h(t);
    if (stop) return;
    if (hside) {
      int32_t S[RW], sig;
      product(s_xh[t & 1][0], [&](int c) { return wf[c]; }, S, sig);
      const XvRow p = s_hp[t & 1][row];
      float act[RW], o[4];
#pragma unroll
      for (int k = 0; k < RW; ++k) {
        const int gate = gate0 + k;
        const float y = recover(S[k], cp[k].colterm, cp[k].ztw, p.z + 128, sig, cp[k].iqw, p.iq);
        const float av = s_xb[t & 1][row][4 * cl + gate] + y;
        const float sg = sigmoid_cw(gate == 2 ? 2.0f * av : av);
        act[k] = gate == 2 ? 2.0f * sg - 1.0f : sg;
      }
      // the pair's other gates: lanes row + NR j of the 16 hold gates RW j .. + RW - 1
#pragma unroll
      for (int gt = 0; gt < 4; ++gt) o[gt] = __shfl(act[gt % RW], (lane & 48) + row + NR * (gt / RW), 64);
      const float cn = (o[1] * cst) + (o[0] * o[2]);
      cst = cn;
      const float m = o[3] * tanh_cw(cn);
      const int64_t fo = (int64_t)t * B + brow;
      if (live && fr < NR) {
        put_word((PROJ ? mx : hx) + ((int64_t)(t & 1) * rows + row) * H + cell, (uint32_t)(t + 1),
                 __float_as_uint(m));
        if (!PROJ && Ly.h) Ly.h[fo * H + cell] = m;
        if (TP) {
          if (Ly.tap_c) Ly.tap_c[fo * H + cell] = cn;
          if (Ly.tap_m) Ly.tap_m[fo * H + cell] = m;
          if (t == T - 1) {
            if (!PROJ && Ly.hT) Ly.hT[brow * H + cell] = m;
            if (Ly.cT) Ly.cT[brow * H + cell] = cn;
          }
        }
      }
      if (TP && live)
#pragma unroll
        for (int k = 0; k < RW; ++k) {
          if (Ly.acc_h) Ly.acc_h[(fo * 4 + gate0 + k) * H + cell] = acc_u8(S[k], cp[k].sigw, sig, R);
          if (Ly.tap_gates) Ly.tap_gates[(fo * 4 + gate0 + k) * H + cell] = act[k];
        }
    } else {
      if (t + 1 < T) use_x(t + 1);
      if (t > 0) put_out(t - 1);
      if (t + 2 < T) land_x(t + 2);
      issue_x(std::min(t + 3, T - 1));
    }
    if constexpr (PROJ) {
      take(mx + (int64_t)(t & 1) * rows * H, nullptr, H, (uint32_t)(t + 1), s_xm[0], s_mp);
      if (wave == 0) {
        int32_t S[RW], sig;
        product(s_xm[0], [&](int c) {
          if constexpr (WRL) return *reinterpret_cast<const v4i *>(s_wr[fr] + c * 64 + 16 * fq);
          else return wr[c];
        }, S, sig);
        const XvRow p = s_mp[row];
        const int64_t fo = (int64_t)t * B + brow;
#pragma unroll
        for (int k = 0; k < RW; ++k) {
          const float h = recover(S[k], rp[k].colterm, rp[k].ztw, p.z + 128, sig, rp[k].iqw, p.iq);
          const int out = out0 + k;
          if (row < nb && out < R) {
            put_word(hx + ((int64_t)(t & 1) * rows + row) * R + out, (uint32_t)(t + 1),
                     __float_as_uint(h));
            if (Ly.h) Ly.h[fo * R + out] = h;
            if (TP && Ly.acc_r) Ly.acc_r[fo * R + out] = acc_u8(S[k], rp[k].sigw, sig, H);
            if (TP && t == T - 1 && Ly.hT) Ly.hT[brow * R + out] = h;
          }
        }
      }
    }
  }
  // the last step's output
  take_h(T);
  if (stop) return;
  if (!hside) put_out(T - 1);
}

// ------------------------------------------------------------------ host side
// How the layout takes a: rows per group it is built for (4 or 8; 0: it does
// not take a), batch rows and exchange words of a launch.
struct XvPlan {
  XvTiling tl;
  int nr;
  int64_t launches, chunk, nwords;
};
template <class Args>
static XvPlan plan_xrows(const Args &a, size_t word_bytes, int cus) {
  constexpr bool PROJ = std::is_same<Args, PStackArgs>::value;
  XvPlan p{};
  if (cus != kXvXcds * kXvSlots || a.nl < 1 || a.nl > kXvXcds || a.T < 1 || a.T >= (1 << 30) || a.B < 1)
    return p;
  const int groups = kXvXcds / a.nl;
  for (int l = 0; l < a.nl; ++l) {
    const auto &L = a.L[l];
    const int64_t H = xv_cells(a, l), R = xv_width(a, l);
    if (H < 1 || H > kXvMaxW || R < 1 || R > kXvMaxW || L.in < 1 || L.in > kXvMaxW) return p;
    if (l > 0 && L.in != xv_width(a, l - 1)) return p;
    if (L.Wx.ld < round_up(L.in, 64) || L.Wh.ld < round_up(R, 64)) return p;
    if constexpr (PROJ)
      if (L.Wr.ld < round_up(H, 64)) return p;
    if (L.out.codes && (L.out.ld < R || L.out.ld % 4)) return p;
  }
  if (a.L[0].xin.ld % 8 || a.L[0].xin.ld < a.L[0].in) return p;
  // Groups of up to four rows while the chip has them, with a projection then of
  // up to eight, over launches of equal size, where that is the faster layout.
  // Through 5 x 500 cells, us a frame (100 frames, start-up included): without a
  // projection 3.5 in fours against 4.7 in k_xstack, in eights no faster than
  // that, so fours in one launch only.  With P = 200, 5.5 in fours and 7.4 a
  // launch in eights, against 39-43 with one launch per layer (31-35 for 4
  // layers).
  const int64_t most = (int64_t)groups * (PROJ ? 8 : 4);
  p.launches = (a.B + most - 1) / most;
  p.chunk = (a.B + p.launches - 1) / p.launches;
  if (p.launches > (PROJ ? a.nl : 1)) return p;
  // Several launches each fill the wavefront anew, 18 us a layer, for 6.2 a frame;
  // a launch per layer (from 16 rows on k_xrec) costs 30 us and 7.2 a frame.
  // 5 x 500, P = 200, 40 rows (5 launches), us so and with a launch per layer: 12
  // frames 1000 and 721, 30 frames 1569 and 1409, 100 frames 3762 and 4061; 32
  // rows (4 launches), 12 frames 817 and 713.
  if (p.launches > 1 && p.launches * (18.0 * a.nl + 6.2 * a.T) > a.nl * (30.0 + 7.2 * a.T)) return p;
  const int nr = p.chunk <= 4 * groups ? 4 : 8;
  const int ng = (int)((p.chunk + nr - 1) / nr);
  p.tl.rows = (int)((p.chunk + ng - 1) / ng);
  for (int l = 0; l < a.nl; ++l)
    p.nwords += ng * xv_words(xv_cells(a, l), xv_width(a, l), PROJ, a.T, p.tl.rows);
  if ((size_t)p.nwords * 8 <= word_bytes) p.nr = nr;
  return p;
}

template <class Args>
static hipError_t launch_xrows_any(const Args &a, void *words, size_t word_bytes, int cus, bool taps,
                                   hipStream_t s, bool *done) {
  constexpr bool PROJ = std::is_same<Args, PStackArgs>::value;
  *done = false;
  const XvPlan p = plan_xrows(a, word_bytes, cus);
  if (!p.nr) return hipSuccess;
  XvTiling tl = p.tl;
  tl.words = static_cast<uint64_t *>(words);
  auto kern = taps ? k_xrows<Args, 4, true> : k_xrows<Args, 4, false>;
  if constexpr (PROJ)
    if (p.nr == 8) kern = taps ? k_xrows<Args, 8, true> : k_xrows<Args, 8, false>;
  // with the static part more than half of a CU's LDS, so that a CU holds one workgroup
  const size_t lds = 84 * 1024;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kXvThreads, lds);
  if (e != hipSuccess) return e;
  if (per_cu < 1) return hipSuccess;
  for (int64_t r0 = 0; r0 < a.B; r0 += p.chunk) {
    tl.r0 = r0;
    tl.r1 = std::min(a.B, r0 + p.chunk);
    tl.ng = (int)((tl.r1 - r0 + tl.rows - 1) / tl.rows);
    e = clear_exchange2(a.ws, kXvSlotBytes / 8, tl.words, p.nwords, s);
    if (e != hipSuccess) return e;
    Args args = a;
    XvTiling t = tl;
    void *kargs[] = {&args, &t};
    e = hipLaunchCooperativeKernel(reinterpret_cast<void *>(kern), dim3(cus), dim3(kXvThreads), kargs,
                                   (unsigned)lds, s);
    if (e != hipSuccess) return e;
  }
  *done = true;
  return hipSuccess;
}

size_t xrows_ws(int64_t H, int64_t T, int64_t B) {
  return kHeaderBytes + kXvSlotBytes + 8 * (size_t)xv_words(H, H, false, T, B + kXvXcds);
}

hipError_t launch_xrows(const StackArgs &a, size_t ws_bytes, int cus, bool taps, hipStream_t s,
                        bool *done) {
  const size_t head = kHeaderBytes + kXvSlotBytes;
  *done = false;
  if (ws_bytes < head) return hipSuccess;
  return launch_xrows_any(a, static_cast<char *>(a.ws) + head, ws_bytes - head, cus, taps, s, done);
}
hipError_t launch_xrows(const PStackArgs &a, void *words, size_t word_bytes, int cus, bool taps,
                        hipStream_t s, bool *done) {
  return launch_xrows_any(a, words, word_bytes, cus, taps, s, done);
}

int xrows_applies(const StackArgs &a, size_t ws_bytes, int cus, int *launches) {
  const size_t head = kHeaderBytes + kXvSlotBytes;
  const XvPlan p = plan_xrows(a, ws_bytes < head ? 0 : ws_bytes - head, cus);
  *launches = (int)p.launches;
  return p.nr;
}
int xrows_applies(const PStackArgs &a, size_t word_bytes, int cus, int *launches) {
  const XvPlan p = plan_xrows(a, word_bytes, cus);
  *launches = (int)p.launches;
  return p.nr;
}

hipError_t set_wait_bound_xrows(int polls) { return set_wait_bound_here(polls); }

}  // namespace ql
