// ql_quant_rows.h -- range and codes (Section 3 / eq. 2) of rows and of
// contiguous values, by a wave or a workgroup; used by the quantizer's kernels
// and by the product of small operands.
#pragma once
#include "ql_device.h"

namespace ql {

// min and max over the block (up to 16 waves), in every thread.
__device__ __forceinline__ float2 block_minmax(float lo, float hi) {
  __shared__ float slo[16], shi[16];
  const int nw = blockDim.x >> 6;
  lo = wave_min(lo);
  hi = wave_max(hi);
  if ((threadIdx.x & 63) == 0) {
    slo[threadIdx.x >> 6] = lo;
    shi[threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  lo = slo[0], hi = shi[0];
  for (int w = 1; w < nw; ++w) {
    lo = fminf(lo, slo[w]);
    hi = fmaxf(hi, shi[w]);
  }
  return make_float2(lo, hi);
}

// Row accessors of the on-the-fly quantizer: value i of one input vector.
// A row of a dense [m][ldx] matrix.
struct DenseRow {
  const float *x;
  __device__ bool vec4(int64_t K) const { return (K & 3) == 0 && (((uintptr_t)x) & 15) == 0; }
  __device__ float4 load4(int64_t q) const { return reinterpret_cast<const float4 *>(x)[q]; }
  __device__ float load1(int64_t i) const { return x[i]; }
};
// One presented input of the frontend (Section 4): `stack` consecutive base
// frames of one utterance, `dim` values each, laid end to end.  f points at the
// first of them; consecutive base frames of the utterance lie `fstride` floats
// apart (B * dim in a time-major [frames][B][dim] array).  K = stack * dim < 2^31.
struct StackedRow {
  const float *f;
  int dim;
  int64_t fstride;
  __device__ bool vec4(int64_t) const {
    return (dim & 3) == 0 && (fstride & 3) == 0 && (((uintptr_t)f) & 15) == 0;
  }
  __device__ float4 load4(int64_t q) const {  // dim % 4 == 0: a float4 never straddles frames
    const int i = 4 * (int)q, j = i / dim;
    return *reinterpret_cast<const float4 *>(f + j * fstride + (i - j * dim));
  }
  __device__ float load1(int64_t i) const {
    const int j = (int)i / dim;
    return f[j * fstride + ((int)i - j * dim)];
  }
};

// min and max of the K values of row x, reduced over the wave (every lane).
template <class Row>
__device__ __forceinline__ float2 row_minmax_wave(const Row &x, int64_t K, int lane) {
  float lo = INFINITY, hi = -INFINITY;
  if (x.vec4(K)) {
    for (int64_t i = lane; i < K / 4; i += kWave) {
      const float4 v = x.load4(i);
      lo = fminf(fminf(lo, v.x), fminf(v.y, fminf(v.z, v.w)));
      hi = fmaxf(fmaxf(hi, v.x), fmaxf(v.y, fmaxf(v.z, v.w)));
    }
  } else {
    for (int64_t i = lane; i < K; i += kWave) {
      const float v = x.load1(i);
      lo = fminf(lo, v);
      hi = fmaxf(hi, v);
    }
  }
  return make_float2(wave_min(lo), wave_max(hi));
}

// Encode the K values of row x with params (q, z) into out[0, ld);
// returns the code sum (0..255 domain) in every lane of the wave.
template <class Row>
__device__ __forceinline__ int encode_row_wave(const Row &x, int64_t K, int8_t *__restrict__ out,
                                               int64_t ld, double q, int32_t z, int lane) {
  int sum = 0;
  if (x.vec4(K)) {
    uint32_t *o4 = reinterpret_cast<uint32_t *>(out);
    for (int64_t i = lane; i < K / 4; i += kWave) {
      const float4 v = x.load4(i);
      const int c0 = encode(v.x, q, z), c1 = encode(v.y, q, z), c2 = encode(v.z, q, z),
                c3 = encode(v.w, q, z);
      sum += c0 + c1 + c2 + c3;
      o4[i] = pack4_s8(c0, c1, c2, c3);
    }
  } else {
    for (int64_t i = lane; i < K; i += kWave) {
      const int c = encode(x.load1(i), q, z);
      sum += c;
      out[i] = (int8_t)(c ^ 0x80);
    }
  }
  // zero padding [K, ld) in the signed layout (V' - 128 = 0 contributes 0)
  for (int64_t i = K + lane; i < ld; i += kWave) out[i] = 0;
  return wave_sum(sum);
}

// min and max of n contiguous values over the block (every thread); up to
// eight float4 a thread in flight where the values are 16-byte aligned.
__device__ __forceinline__ float2 range_minmax_block(const float *__restrict__ x, int64_t n) {
  float lo = INFINITY, hi = -INFINITY;
  const int64_t T = blockDim.x;
  auto take = [&](const float4 &v) {
    lo = fminf(fminf(lo, v.x), fminf(v.y, fminf(v.z, v.w)));
    hi = fmaxf(fmaxf(hi, v.x), fmaxf(v.y, fmaxf(v.z, v.w)));
  };
  int64_t done = 0;
  if ((((uintptr_t)x) & 15) == 0) {
    const float4 *x4 = reinterpret_cast<const float4 *>(x);
    const int64_t n4 = n / 4;
    int64_t i = threadIdx.x;
    for (; i + 7 * T < n4; i += 8 * T) {
      float4 v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = x4[i + k * T];
#pragma unroll
      for (int k = 0; k < 8; ++k) take(v[k]);
    }
    for (; i < n4; i += T) take(x4[i]);
    done = 4 * n4;
  }
  for (int64_t i = done + threadIdx.x; i < n; i += T) {
    lo = fminf(lo, x[i]);
    hi = fmaxf(hi, x[i]);
  }
  return block_minmax(lo, hi);
}

}  // namespace ql
