// Morton-ordered fixed-point codec of a Gaussian set (Sec. 4.3, "Quantization
// and compression": Gaussians sorted along the Morton curve; positions
// normalised to the bounding box with 14 bits per axis; intensity 12 bits on
// [0, 1]; log-scales 12 bits; quaternions on the positive half-sphere, 12 bits
// per component; intensities normalised to [0, 1] by their maximum).  The
// codes are stored as 11 uint16 planes and decoded in
// registers by the renderer (attribute type GP_QM), 22 bytes per Gaussian.
//
// Every decision that yields a code is a fixed binary32 sequence (contraction
// off): code = floor(((v - lo) / (hi - lo)) * (levels - 1) + 0.5), clamped;
// decoding is lo + code * ((hi - lo) / (levels - 1)).
//
// Encoding: bounds (per-workgroup minima and maxima, added up by one workgroup)
// -> codes and the 42-bit Morton key -> a stable LSD radix sort of (key, index)
// in two stages (the low 27 bits, then the high 15 bits of the keys gathered in
// that order: five passes) -> the codes gathered in Morton order.  Bound by the
// sort's launches.  Minima and maxima by atomics on nine shared words took 0.049
// ms for 500,000 Gaussians (now 0.012 and 0.004), gathers of 2-byte codes from 11 planes
// 0.060 (one record per Gaussian: 0.012), a split at 32 bits six passes.
//
// A record is 16 bytes: the eight 12-bit codes and the low part of the Morton key, from
// which, with the sorted high part, the three position codes are read back.  With the
// sort's five arrays that is 36 bytes of scratch per Gaussian (52 with the codes spelled
// out in 32 bytes, which made the largest set that can be encoded smaller).
#include "gp_internal.h"

#include <algorithm>

namespace gp {
namespace {

constexpr int kLowBits = 27, kHighBits = 42 - kLowBits;   // the sort's two stages: passes of 9 and of 8 bits
constexpr float kPosLevels1 = 16383.0f;   // 2^14 - 1
constexpr float kAttrLevels1 = 4095.0f;   // 2^12 - 1

__device__ __forceinline__ uint32_t ordered(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unordered(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// Parameter row r (0..10) of Gaussian j: rows 0..2 from the means, 3..10 from
// the attributes.
__device__ __forceinline__ float prow(const float* m, const float* at, int64_t stride, int r, int64_t j) {
  return r < 3 ? m[r * stride + j] : at[(r - 3) * stride + j];
}

// part[9 b + i] of workgroup b: i = 0..2 min mu, 3..5 max mu, 6 min l, 7 max l, 8
// max intensity (ordered ints)
constexpr unsigned kBoundsBlocks = 512;

__global__ __launch_bounds__(256) void k_codec_bounds(const float* __restrict__ m, const float* __restrict__ at,
                                                      int64_t n, int64_t stride, uint32_t* __restrict__ part) {
  __shared__ uint32_t smin[4][5], smax[4][5];
  uint32_t mn[5] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, mx[5] = {0u, 0u, 0u, 0u, 0u};
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float v = prow(m, at, stride, a, j);
      if (isfinite(v)) {
        mn[a] = min(mn[a], ordered(v));
        mx[a] = max(mx[a], ordered(v));
      }
    }
#pragma unroll
    for (int a = 3; a < 6; ++a) {
      const float v = prow(m, at, stride, a, j);
      if (isfinite(v)) {
        mn[3] = min(mn[3], ordered(v));
        mx[3] = max(mx[3], ordered(v));
      }
    }
    const float al = prow(m, at, stride, 10, j);
    if (isfinite(al)) mx[4] = max(mx[4], ordered(al));
  }
#pragma unroll
  for (int i = 0; i < 5; ++i)
    for (int o = 32; o > 0; o >>= 1) {
      mn[i] = min(mn[i], (uint32_t)__shfl_xor((int)mn[i], o));
      mx[i] = max(mx[i], (uint32_t)__shfl_xor((int)mx[i], o));
    }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
    for (int i = 0; i < 5; ++i) {
      smin[wave][i] = mn[i];
      smax[wave][i] = mx[i];
    }
  __syncthreads();
  if (threadIdx.x < 5) {
    const int i = threadIdx.x;
    uint32_t a = min(min(smin[0][i], smin[1][i]), min(smin[2][i], smin[3][i]));
    uint32_t b = max(max(smax[0][i], smax[1][i]), max(smax[2][i], smax[3][i]));
    uint32_t* p = part + 9 * (size_t)blockIdx.x;
    if (i < 4) p[i < 3 ? i : 6] = a;
    p[i < 3 ? 3 + i : (i == 3 ? 7 : 8)] = b;
  }
}

// The header from the workgroups' bounds, and the count the sort reads; wavefront i
// takes bound i.
__global__ __launch_bounds__(576) void k_codec_header(const uint32_t* __restrict__ part, int nparts, uint32_t n,
                                                      float* __restrict__ hdr, uint32_t* __restrict__ count) {
  const int i = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const bool is_min = (i < 3) || i == 6;
  uint32_t k = is_min ? 0xFFFFFFFFu : 0u;
  for (int b = lane; b < nparts; b += 64) {
    const uint32_t v = part[9 * (size_t)b + i];
    k = is_min ? min(k, v) : max(k, v);
  }
  for (int o = 32; o > 0; o >>= 1) {
    const uint32_t v = (uint32_t)__shfl_xor((int)k, o, 64);
    k = is_min ? min(k, v) : max(k, v);
  }
  if (threadIdx.x == 0) *count = n;
  if (lane != 0) return;
  // no finite value: the min stays at all-ones, the max at zero
  const bool empty = is_min ? (k == 0xFFFFFFFFu) : (k == 0u);
  float v = empty ? 0.0f : unordered(k);
  if (i == 8) v = fmaxf(v, 0.0f);   // intensities are coded on [0, amax]
  hdr[i] = v;
}

__device__ __forceinline__ uint32_t code_of(float v, float lo, float hi, float levels1) {
#pragma clang fp contract(off)
  if (!(hi > lo)) return 0u;
  const float c = floorf(((v - lo) / (hi - lo)) * levels1 + 0.5f);
  if (!isfinite(c)) return 0u;
  return (uint32_t)fminf(fmaxf(c, 0.0f), levels1);
}

__device__ __forceinline__ uint64_t spread3_64(uint32_t v) {
  uint64_t x = v & 0x3FFFu;
  x = (x | (x << 16)) & 0x0000FF0000FFull;
  x = (x | (x << 8)) & 0x00F00F00F00Full;
  x = (x | (x << 4)) & 0x0C30C30C30C3ull;
  x = (x | (x << 2)) & 0x249249249249ull;
  return x;
}

// The inverse of spread3_64: bits 0, 3, 6, ... of x.
__device__ __forceinline__ uint32_t gather3_64(uint64_t x) {
  x &= 0x249249249249ull;
  x = (x | (x >> 2)) & 0x0C30C30C30C3ull;
  x = (x | (x >> 4)) & 0x00F00F00F00Full;
  x = (x | (x >> 8)) & 0x0000FF0000FFull;
  x = (x | (x >> 16)) & 0x3FFFull;
  return (uint32_t)x;
}

__global__ __launch_bounds__(256) void k_codec_codes(const float* __restrict__ m, const float* __restrict__ at,
                                                     int64_t n, int64_t stride,
                                                     const float* __restrict__ hdr, uint4* __restrict__ codes,
                                                     uint32_t* __restrict__ key_lo, uint32_t* __restrict__ key_hi,
                                                     uint32_t* __restrict__ idx) {
#pragma clang fp contract(off)
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= n) return;
  uint32_t c[11];
#pragma unroll
  for (int a = 0; a < 3; ++a) c[a] = code_of(prow(m, at, stride, a, j), hdr[a], hdr[3 + a], kPosLevels1);
#pragma unroll
  for (int a = 0; a < 3; ++a) c[3 + a] = code_of(prow(m, at, stride, 3 + a, j), hdr[6], hdr[7], kAttrLevels1);
  float q[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) q[r] = prow(m, at, stride, 6 + r, j);
  const float n2 = ((q[0] * q[0] + q[1] * q[1]) + q[2] * q[2]) + q[3] * q[3];
  const float rn = sqrtf(n2);
  float qn[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) qn[r] = q[r] / rn;
  const bool flip = qn[0] < 0.0f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float v = flip ? -qn[r] : qn[r];
    const float cc = floorf(((v + 1.0f) * 0.5f) * kAttrLevels1 + 0.5f);
    c[6 + r] = isfinite(cc) ? (uint32_t)fminf(fmaxf(cc, 0.0f), kAttrLevels1) : 0u;
  }
  c[10] = code_of(fmaxf(prow(m, at, stride, 10, j), 0.0f), 0.0f, hdr[8], kAttrLevels1);
  const uint64_t key = spread3_64(c[0]) | (spread3_64(c[1]) << 1) | (spread3_64(c[2]) << 2);
  const uint32_t lo = (uint32_t)key & ((1u << kLowBits) - 1u);
  codes[j] = make_uint4(c[3] | (c[4] << 12) | (c[5] << 24), (c[5] >> 8) | (c[6] << 4) | (c[7] << 16) | (c[8] << 28),
                        (c[8] >> 4) | (c[9] << 8) | (c[10] << 20), lo);
  key_lo[j] = lo;
  key_hi[j] = (uint32_t)(key >> kLowBits);
  idx[j] = (uint32_t)j;
}

__global__ __launch_bounds__(256) void k_codec_gather_u32(const uint32_t* __restrict__ src,
                                                          const uint32_t* __restrict__ perm, int64_t n,
                                                          uint32_t* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = src[perm[i]];
}

// key_hi: the sorted high parts of the keys (in the order of perm).
__global__ __launch_bounds__(256) void k_codec_gather_codes(const uint4* __restrict__ src,
                                                            const uint32_t* __restrict__ perm,
                                                            const uint32_t* __restrict__ key_hi, int64_t n,
                                                            int64_t stride_out, uint16_t* __restrict__ dst,
                                                            uint32_t* __restrict__ perm_out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint32_t j = perm[i];
  const uint4 v = src[j];
  const uint64_t key = ((uint64_t)key_hi[i] << kLowBits) | v.w;
  const uint32_t c[11] = {gather3_64(key), gather3_64(key >> 1), gather3_64(key >> 2),
                          v.x & 0xFFFu, (v.x >> 12) & 0xFFFu, (v.x >> 24) | ((v.y & 0xFu) << 8),
                          (v.y >> 4) & 0xFFFu, (v.y >> 16) & 0xFFFu, (v.y >> 28) | ((v.z & 0xFFu) << 4),
                          (v.z >> 8) & 0xFFFu, v.z >> 20};
#pragma unroll
  for (int r = 0; r < 11; ++r) dst[r * stride_out + i] = (uint16_t)c[r];
  if (perm_out) perm_out[i] = j;
}

}  // namespace

hipError_t launch_encode(const float* means, const float* attrs, int64_t n, int64_t stride, uint16_t* codes_out,
                         int64_t stride_out, uint32_t* perm_out, float* d_hdr, const CodecScratch& t, hipStream_t s) {
  const unsigned blocks = (unsigned)((n + 255) / 256), parts = std::min(blocks, kBoundsBlocks);
  if (n > 0) k_codec_bounds<<<parts, 256, 0, s>>>(means, attrs, n, stride, t.bounds);
  k_codec_header<<<1, 576, 0, s>>>(t.bounds, (int)parts, (uint32_t)n, d_hdr, t.count);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || n == 0) return e;
  k_codec_codes<<<blocks, 256, 0, s>>>(means, attrs, n, stride, d_hdr, t.codes, t.key_lo, t.key_hi, t.idx);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // stable sort by the low key bits, then by the high ones (keys gathered in that order)
  uint32_t *k_sorted = nullptr, *i_sorted = nullptr;
  e = launch_radix_sort(t.key_lo, t.idx, t.key2, t.val2, t.count, nullptr, n, kLowBits, t.hist, s, &k_sorted, &i_sorted);
  if (e != hipSuccess) return e;
  uint32_t* hi_perm = (k_sorted == t.key_lo) ? t.key2 : t.key_lo;   // the buffer the sort left free
  k_codec_gather_u32<<<blocks, 256, 0, s>>>(t.key_hi, i_sorted, n, hi_perm);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  uint32_t* i_free = (i_sorted == t.idx) ? t.val2 : t.idx;
  uint32_t* v_alt = (hi_perm == t.key_lo) ? t.key2 : t.key_lo;
  uint32_t *k2 = nullptr, *perm = nullptr;
  e = launch_radix_sort(hi_perm, i_sorted, v_alt, i_free, t.count, nullptr, n, kHighBits, t.hist, s, &k2, &perm);
  if (e != hipSuccess) return e;
  k_codec_gather_codes<<<blocks, 256, 0, s>>>(t.codes, perm, k2, n, stride_out, codes_out, perm_out);
  return hipGetLastError();
}

}  // namespace gp

namespace gp {

// The scratch of an encode of n Gaussians, carved from one block (null: only
// its size, in *bytes).
static CodecScratch codec_scratch(void* block, int64_t n, size_t* bytes) {
  const int64_t nn = std::max<int64_t>(n, 1);
  const int64_t hist = std::max(radix_hist_entries(kLowBits, nn), radix_hist_entries(kHighBits, nn));
  char* const b = static_cast<char*>(block);
  size_t at = 0;
  auto take = [&](size_t size) {
    char* const p = b ? b + at : nullptr;
    at += (size + 255) / 256 * 256;
    return p;
  };
  auto u32 = [&](int64_t count) { return reinterpret_cast<uint32_t*>(take(sizeof(uint32_t) * (size_t)count)); };
  CodecScratch t{};
  t.codes = reinterpret_cast<uint4*>(take(sizeof(uint4) * (size_t)nn));
  t.bounds = u32(9 * kBoundsBlocks);
  t.count = u32(1);
  t.key_lo = u32(nn);
  t.key_hi = u32(nn);
  t.idx = u32(nn);
  t.key2 = u32(nn);
  t.val2 = u32(nn);
  t.hist = u32(hist);
  *bytes = at;
  return t;
}

int64_t encode_scratch(int64_t n) {
  size_t bytes = 0;
  codec_scratch(nullptr, n, &bytes);
  return (int64_t)bytes;
}

// Encodes with the caller's scratch (encode_scratch(n) bytes), or, without any,
// with one allocated for the call (one block: ten allocations and releases took a
// quarter of an encode); synchronises, whether it succeeds or not.
gp_status encode_volume(const float* means, const float* attrs, int64_t n, int64_t stride, uint16_t* codes_out,
                        int64_t stride_out, uint32_t* perm_out, float* d_hdr, void* scratch, hipStream_t s) {
  void* own = nullptr;
  if (!scratch) {
    if (hipMalloc(&own, (size_t)encode_scratch(n)) != hipSuccess) {
      set_error("encode: out of device memory");
      return GP_ENOMEM;
    }
  }
  size_t bytes = 0;
  const CodecScratch t = codec_scratch(scratch ? scratch : own, n, &bytes);
  hipError_t e = launch_encode(means, attrs, n, stride, codes_out, stride_out, perm_out, d_hdr, t, s);
  // (also after an error: what was launched before it still writes the scratch)
  const hipError_t waited = hipStreamSynchronize(s);
  if (e == hipSuccess) e = waited;
  const gp_status st = e == hipSuccess ? GP_OK : hip_fail(e, "encode");
  if (own) (void)hipFree(own);
  return st;
}

}  // namespace gp
