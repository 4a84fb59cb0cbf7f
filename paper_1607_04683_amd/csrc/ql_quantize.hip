// ql_quantize.hip -- the quantizer of Section 3 / eq. 2 on gfx950.
//
//  * k_quantize_rows: the on-the-fly activation quantizer (Section 3.1: inputs
//    are quantized on the fly).  One wavefront per vector: fused min/max
//    wavefront reduction -> (R, Q, round(Q Vmin), Q^-1) -> packed codes and the
//    code sum, in one pass over HBM (4 bytes read + 1 byte written per value).
//  * k_quantize_stacked: the same quantizer reading the network's input straight
//    from the frontend's base frames (Section 4: 8 consecutive frames stacked,
//    every third stacked frame presented), so the stacked copy is never written.
//  * k_set_*: quantization of larger sets (a weight matrix or one of its gate
//    blocks; a whole activation tensor): partial min/max over many blocks,
//    then the row encoder; one block per set for small ones.
//  * k_dequantize: recovery of eq. 3.
#include "ql_device.h"
#include "ql_launch.h"
#include "ql_quant_rows.h"

#include <algorithm>

namespace ql {

// One wave quantizes one vector: min/max, params, codes, code sum.
template <class Row>
__device__ __forceinline__ void quantize_row_wave(const Row &x, int64_t K, int64_t row,
                                                  int8_t *__restrict__ codes, int64_t ld,
                                                  int32_t *__restrict__ zero,
                                                  float *__restrict__ inv_q,
                                                  int32_t *__restrict__ sums, int lane) {
  float2 mm = row_minmax_wave(x, K, lane);
  if (K == 0) mm = make_float2(0.0f, 0.0f);
  const QParams p = make_qparams(mm.x, mm.y);
  const int s = encode_row_wave(x, K, codes + row * ld, ld, p.q, p.z, lane);
  if (lane == 0) {
    if (zero) zero[row] = p.z;
    if (inv_q) inv_q[row] = p.inv_q;
    if (sums) sums[row] = s;
  }
}

__global__ __launch_bounds__(256) void k_quantize_rows(const float *__restrict__ X, int64_t ldx,
                                                       int64_t m, int64_t K,
                                                       int8_t *__restrict__ codes, int64_t ld,
                                                       int32_t *__restrict__ zero,
                                                       float *__restrict__ inv_q,
                                                       int32_t *__restrict__ sums,
                                                       int *__restrict__ flag) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x >> 6);
  if (flag && blockIdx.x == 0 && threadIdx.x == 0) *flag = 0;
  if (row >= m) return;
  quantize_row_wave(DenseRow{X + row * ldx}, K, row, codes, ld, zero, inv_q, sums, lane);
}

// Frontend fused into the input quantizer: presented input t of utterance b
// (row t * B + b of the output) is base frames skip*t .. skip*t + stack - 1 of
// that utterance, frames [nframes][B][dim]; the caller guarantees
// skip * (T - 1) + stack <= nframes.
__global__ __launch_bounds__(256) void k_quantize_stacked(const float *__restrict__ frames,
                                                          int64_t B, int dim, int stack,
                                                          int skip, int64_t m,
                                                          int8_t *__restrict__ codes, int64_t ld,
                                                          int32_t *__restrict__ zero,
                                                          float *__restrict__ inv_q,
                                                          int32_t *__restrict__ sums,
                                                          int *__restrict__ flag) {
  const int lane = threadIdx.x & 63;
  if (flag && blockIdx.x == 0 && threadIdx.x == 0) *flag = 0;
  const int64_t row = (int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x >> 6);
  if (row >= m) return;
  const int64_t t = row / B, b = row - t * B;
  const StackedRow x{frames + ((int64_t)skip * t * B + b) * dim, dim, B * (int64_t)dim};
  quantize_row_wave(x, (int64_t)stack * dim, row, codes, ld, zero, inv_q, sums, lane);
}

// Quantization of larger sets (a weight matrix, one of its gate blocks, an
// activation tensor): set s is rows [s * rps, (s + 1) * rps) of a dense
// [rows][cols] matrix.  Two passes over memory are what it cannot do without
// (the range is needed before the first code), so it is two launches: partial
// min/max over up to kSetParts slices of every set, then the encoder, each of
// whose blocks reduces its set's partials by itself.  16384 x 512 values:
// 116 us as three launches (min/max of 128 scalar-loading blocks 96, a
// one-thread reduction of the partials 13, encoder 9), 18 us now.
__global__ __launch_bounds__(256) void k_set_minmax(const float *__restrict__ X, int64_t setsize,
                                                    int64_t per, float2 *__restrict__ part) {
  const int s = blockIdx.y, p = blockIdx.x;
  const int64_t b = (int64_t)p * per;
  const int64_t n = b >= setsize ? 0 : (per < setsize - b ? per : setsize - b);
  const float2 mm = range_minmax_block(X + (int64_t)s * setsize + b, n);
  if (threadIdx.x == 0) part[(int64_t)s * gridDim.x + p] = mm;
}

// Where a quantized set goes: codes with row sums, per-set params, optional
// per-row copies of the set's zero point and recovery factor.
struct SetOut {
  int8_t *codes;
  int64_t ld;
  double *range;       // per set (nullable, as all below)
  int32_t *zero;
  float *inv_q;
  int32_t *row_sums;   // per row
  int32_t *row_zero;
  float *row_inv_q;
};
// The block's waves encode rows [r0, r1) of set s.
__device__ __forceinline__ void encode_set_rows(const float *__restrict__ X, int64_t r0, int64_t r1,
                                                int64_t cols, const QParams &p, const SetOut &o) {
  const int lane = threadIdx.x & 63;
  for (int64_t row = r0 + (threadIdx.x >> 6); row < r1; row += blockDim.x >> 6) {
    const int sum =
        encode_row_wave(DenseRow{X + row * cols}, cols, o.codes + row * o.ld, o.ld, p.q, p.z, lane);
    if (lane == 0) {
      if (o.row_sums) o.row_sums[row] = sum;
      if (o.row_zero) o.row_zero[row] = p.z;
      if (o.row_inv_q) o.row_inv_q[row] = p.inv_q;
    }
  }
}
__device__ __forceinline__ void put_set_params(const QParams &p, int64_t s, const SetOut &o) {
  if (o.range) o.range[s] = p.range;
  if (o.zero) o.zero[s] = p.z;
  if (o.inv_q) o.inv_q[s] = p.inv_q;
}

__global__ __launch_bounds__(256) void k_set_encode(const float *__restrict__ X, int64_t rps,
                                                    int64_t cols,
                                                    const float2 *__restrict__ part, int nparts,
                                                    int brows, SetOut o) {
  const int64_t s = blockIdx.y;
  float lo = INFINITY, hi = -INFINITY;
  for (int i = threadIdx.x; i < nparts; i += 256) {
    const float2 v = part[s * nparts + i];
    lo = fminf(lo, v.x);
    hi = fmaxf(hi, v.y);
  }
  const float2 mm = block_minmax(lo, hi);
  const QParams p = make_qparams(mm.x, mm.y);
  if (blockIdx.x == 0 && threadIdx.x == 0) put_set_params(p, s, o);
  const int64_t r0 = (int64_t)blockIdx.x * brows;
  encode_set_rows(X, s * rps + r0, s * rps + (r0 + brows < rps ? r0 + brows : rps), cols, p, o);
}

// Small sets, one block each: range, params and codes in one launch (the
// second read hits the CU's cache).
__global__ __launch_bounds__(1024) void k_set_small(const float *__restrict__ X, int64_t rps,
                                                    int64_t cols, SetOut o) {
  const int64_t s = blockIdx.x;
  float2 mm = range_minmax_block(X + s * rps * cols, rps * cols);
  if (cols == 0) mm = make_float2(0.0f, 0.0f);
  const QParams p = make_qparams(mm.x, mm.y);
  if (threadIdx.x == 0) put_set_params(p, s, o);
  encode_set_rows(X, s * rps, (s + 1) * rps, cols, p, o);
}

// Recovery (eq. 3), one wave per row: four codes per lane and load where the
// rows of both sides are aligned for it.
__global__ __launch_bounds__(256) void k_dequantize_rows(const int8_t *__restrict__ codes, int64_t ld,
                                                         int64_t rows, int64_t cols, int64_t rpb,
                                                         const int32_t *__restrict__ zero,
                                                         const float *__restrict__ inv_q,
                                                         float *__restrict__ dst, int vec) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x >> 6);
  if (r >= rows) return;
  const int64_t b = r / rpb;
  const int z = zero[b] + 128;  // V' = code + 128
  const float iq = inv_q[b];
  const int8_t *c = codes + r * ld;
  float *d = dst + r * cols;
  int64_t done = 0;
  if (vec) {
    for (int64_t i = lane; i < cols / 4; i += kWave) {
      const uint32_t w = reinterpret_cast<const uint32_t *>(c)[i];
      float4 v;
      v.x = (float)((int)(int8_t)w + z) * iq;
      v.y = (float)((int)(int8_t)(w >> 8) + z) * iq;
      v.z = (float)((int)(int8_t)(w >> 16) + z) * iq;
      v.w = (float)((int)(int8_t)(w >> 24) + z) * iq;
      reinterpret_cast<float4 *>(d)[i] = v;
    }
    done = cols / 4 * 4;
  }
  for (int64_t i = done + lane; i < cols; i += kWave) d[i] = (float)((int)c[i] + z) * iq;
}

// The same, W values of a row per thread (4 where the rows of both sides are
// aligned for it, else 1), the matrix taken as one run of n of them, so that any
// shape fills the chip.
template <int W>
__global__ __launch_bounds__(256) void k_dequantize(const int8_t *__restrict__ codes, int64_t ld,
                                                    uint32_t n, uint32_t per_row, uint32_t rpb,
                                                    const int32_t *__restrict__ zero,
                                                    const float *__restrict__ inv_q,
                                                    float *__restrict__ dst) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint32_t r = i / per_row, c = i - r * per_row, b = r / rpb;
  const int z = zero[b] + 128;  // V' = code + 128
  const float iq = inv_q[b];
  const int8_t *src = codes + (int64_t)r * ld + (int64_t)W * c;
  if constexpr (W == 4) {
    const uint32_t w = *reinterpret_cast<const uint32_t *>(src);
    float4 v;
    v.x = (float)((int)(int8_t)w + z) * iq;
    v.y = (float)((int)(int8_t)(w >> 8) + z) * iq;
    v.z = (float)((int)(int8_t)(w >> 16) + z) * iq;
    v.w = (float)((int)(int8_t)(w >> 24) + z) * iq;
    reinterpret_cast<float4 *>(dst)[i] = v;
  } else {
    dst[i] = (float)((int)*src + z) * iq;
  }
}

// Row sums of 0..255 codes stored in the signed layout.
__global__ __launch_bounds__(256) void k_code_row_sums(const int8_t *__restrict__ codes,
                                                       int64_t ld, int64_t rows, int64_t K,
                                                       int32_t *__restrict__ sums) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int8_t *c = codes + row * ld;
  int s = 0;
  for (int64_t i = lane; i < K; i += kWave) s += (int)c[i] + 128;
  s = wave_sum(s);
  if (lane == 0) sums[row] = s;
}

__global__ void k_gate_fn(int fn, const float *__restrict__ x, float *__restrict__ y, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float v = x[i];
  y[i] = fn == 0 ? exp_cw(v) : fn == 1 ? sigmoid_cw(v) : fn == 2 ? tanh_cw(v) : recip_ge1(v);
}

// ---------------------------------------------------------------- launchers
static inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

hipError_t launch_quantize_rows(const float *X, int64_t ldx, int64_t m, int64_t K, int8_t *codes,
                                int64_t ld, int32_t *zero, float *inv_q, int32_t *sums,
                                hipStream_t s, int *flag) {
  if (m == 0) return hipSuccess;
  hipLaunchKernelGGL(k_quantize_rows, dim3(blocks_for(m, 4)), dim3(256), 0, s, X, ldx, m, K,
                     codes, ld, zero, inv_q, sums, flag);
  return hipGetLastError();
}

hipError_t launch_quantize_stacked(const float *frames, int64_t B, int dim, int stack, int skip,
                                   int64_t T, int8_t *codes, int64_t ld, int32_t *zero,
                                   float *inv_q, int32_t *sums, hipStream_t s, int *flag) {
  const int64_t m = T * B;
  if (m == 0) return hipSuccess;
  hipLaunchKernelGGL(k_quantize_stacked, dim3(blocks_for(m, 4)), dim3(256), 0, s, frames, B, dim,
                     stack, skip, m, codes, ld, zero, inv_q, sums, flag);
  return hipGetLastError();
}

// Slices of a set's partial min/max: 8192 values a block (eight float4 per
// thread, one round of loads) up to 512 blocks, beyond which a block's further
// rounds cost less than longer reductions of the partials.
static int set_parts(int64_t setsize) {
  return (int)std::min<int64_t>(kSetParts, std::max<int64_t>(1, (setsize + 8191) / 8192));
}
// Threads of the block that takes a set whole; 0: two launches over all CUs beat
// one block's passes.  Up to 8192 values, one round of its loads (more where there
// are many sets to fill the chip with blocks), in at most 16 rows a wave, which
// encodes them one after the other (one set of 4 columns, us, two launches and one
// block: 256 rows 17.5 and 14.7, 512 17.2 and 26.2, 1024 17.5 and 49; 256 sets of
// 256 x 16 18.4 and 31).
static int set_small_threads(int64_t rps, int64_t setsize, int64_t nsets) {
  const int threads = setsize <= 4096 && nsets > 1 ? 256 : 1024;
  const bool few = setsize <= 8192 || (setsize <= 65536 && nsets >= 256);
  return few && rps <= threads / kWave * 16 ? threads : 0;
}

size_t set_quantize_ws(int64_t rows, int64_t cols, int nsets) {
  const int64_t n = nsets > 0 ? rows / nsets * cols : 0;
  return align_up((size_t)nsets * set_parts(n) * sizeof(float2), 256);
}

hipError_t launch_set_quantize(const float *X, int64_t rows, int64_t cols, int nsets, int8_t *codes,
                               int64_t ld, double *range, int32_t *zero, float *inv_q,
                               int32_t *row_sums, int32_t *row_zero, float *row_inv_q, void *ws,
                               hipStream_t s) {
  if (rows == 0) return hipSuccess;
  const SetOut o{codes, ld, range, zero, inv_q, row_sums, row_zero, row_inv_q};
  const int64_t rps = rows / nsets, n = rps * cols;
  const int small = n == 0 ? 1024 : set_small_threads(rps, n, nsets);
  if (small) {
    hipLaunchKernelGGL(k_set_small, dim3(nsets), dim3(small), 0, s, X, rps, cols, o);
    return hipGetLastError();
  }
  float2 *part = static_cast<float2 *>(ws);
  const int parts = set_parts(n);
  const int64_t per = round_up((n + parts - 1) / parts, 4);
  hipLaunchKernelGGL(k_set_minmax, dim3(parts, nsets), dim3(256), 0, s, X, n, per, part);
  // rows of a block of the encoder: 16, so that its reduction of the partials is
  // a small part, or one per wave where that leaves the chip idle (16 x 100000, us:
  // 593 with 16, 123 with 4)
  const int brows = (rps + 15) / 16 * nsets >= 256 ? 16 : 4;
  hipLaunchKernelGGL(k_set_encode, dim3(blocks_for(rps, brows), nsets), dim3(256), 0, s, X, rps, cols,
                     part, parts, brows, o);
  return hipGetLastError();
}

hipError_t launch_dequantize(const int8_t *codes, int64_t ld, int64_t rows, int64_t cols,
                             int nblocks, const int32_t *zero, const float *inv_q, float *dst,
                             hipStream_t s) {
  if (rows * cols == 0) return hipSuccess;
  // every row of codes 4-byte aligned, every row of dst 16-byte aligned
  const bool vec = ld % 4 == 0 && reinterpret_cast<uintptr_t>(codes) % 4 == 0 && cols % 4 == 0 &&
                   reinterpret_cast<uintptr_t>(dst) % 16 == 0;
  // a wave per row where that fills the chip: no division (us, by rows and by
  // threads: 16384 x 8192 134 and 157, 16383 x 8191 237 and 374, 16 x 33024 30 and
  // 6.4, 1 x 1000000 723 and 6.8, 1000000 x 1 107 and 11, 100000 x 40 13 and 6.3,
  // 273607 x 175 57 and 76), and where 32 bits do not count the threads
  const int64_t per_row = vec ? cols / 4 : cols, n = rows * per_row;
  if ((rows >= 1024 && cols >= (vec ? 256 : 128)) || n > (int64_t)UINT32_MAX - 255)
    hipLaunchKernelGGL(k_dequantize_rows, dim3(blocks_for(rows, 4)), dim3(256), 0, s, codes, ld, rows, cols,
                       rows / nblocks, zero, inv_q, dst, (int)vec);
  else
    hipLaunchKernelGGL((vec ? k_dequantize<4> : k_dequantize<1>), dim3(blocks_for(n, 256)), dim3(256), 0, s,
                       codes, ld, (uint32_t)n, (uint32_t)per_row, (uint32_t)(rows / nblocks), zero, inv_q,
                       dst);
  return hipGetLastError();
}

hipError_t launch_code_row_sums(const int8_t *codes, int64_t ld, int64_t rows, int64_t K,
                                int32_t *sums, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  hipLaunchKernelGGL(k_code_row_sums, dim3(blocks_for(rows, 4)), dim3(256), 0, s, codes, ld,
                     rows, K, sums);
  return hipGetLastError();
}

hipError_t launch_gate_fn(int fn, const float *x, float *y, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gate_fn, dim3(blocks_for(n, 256)), dim3(256), 0, s, fn, x, y, n);
  return hipGetLastError();
}

}  // namespace ql
