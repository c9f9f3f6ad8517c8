// Slice loss L = mean |I - T| + lambda (1 - mean SSIM) and dL/dI (Sec. 4.3, loss
// function: an L1 term plus a D-SSIM term weighted by lambda; lambda = 0.2 in
// Sec. 5.1).  SSIM follows Wang et al. 2004: local means, variances and the
// covariance under an 11 x 11 Gaussian window (sigma 1.5, unit sum; zeros
// outside the slice), C1 = 0.01^2, C2 = 0.03^2.
//
// With A1 = 2 mx my + C1, A2 = 2 sxy + C2, B1 = mx^2 + my^2 + C1,
// B2 = sxx + syy + C2 and S = A1 A2 / (B1 B2), S at pixel q depends on the
// image only through the window sums mx, E[x^2] and E[xy] at q:
//   dS/dmx    = 2 my (A2 - A1) / (B1 B2) - 2 mx S (1/B1 - 1/B2)
//   dS/dE[x2] = -S / B2
//   dS/dE[xy] = 2 A1 / (B1 B2)
// so dL/dI(p) = sign(I - T)/n - lambda/n (W*c_mu + 2 I W*c_x2 + T W*c_xy)(p),
// where W* is the (symmetric) window filter of the three coefficient maps.
//
// Two stencil kernels, each over 32 x 16 output tiles, the 11-tap filter applied
// separably: along columns from global memory (the output rows, over the width of
// the halo), then along rows from LDS.  In both passes a thread takes neighbouring
// outputs and reads (and, in the first pass, converts and multiplies) each of
// their inputs once.
//   k_ssim_stats: five window sums -> S and the three coefficient maps;
//   k_ssim_grad:  window sums of the three maps -> dL/dI (its first workgroup
//                 also adds up the loss terms).
// With one output per thread and the halo staged in LDS, LDS traffic and two more
// barriers bounded them: 16 slices of 1024^2 0.318 -> 0.250 and 0.237 -> 0.232 (now 0.157) ms,
// 8 of 256^2 0.0149 -> 0.0126 and 0.0115 -> 0.0079.  Slower: tiles of 64 x 16
// staged in LDS (0.40 / 0.24: too few wavefronts), 32 x 32 (0.285 / 0.228), two
// outputs along columns (0.286 / 0.314); a contiguous run of tiles per XCD changed
// nothing.  With one float64 division per pixel for four, the first takes 0.231 ms
// (2.3 TB/s of the bytes it cannot do without, the other 3.8).
// Both compute in float64: the moments form of the variances (E[x^2] - mx^2)
// and the sum mx-term + 2 I x2-term cancel to a few bits in smooth regions,
// and the whole loss costs about 300 flops per pixel, far from any bound.
#include <mutex>

#include "gp_internal.h"

namespace gp {
namespace {

constexpr int kSW = 32, kSH = 16, kR = 5, kRW = kSW + 2 * kR;
constexpr int kThreads = 256;
constexpr int kCol = 4, kRow = 2;              // neighbouring outputs per thread of a pass
constexpr int kColItems = kRW * (kSH / kCol);
// The gradient's first pass: a thread takes one of the three maps and eight outputs,
// which fills 252 of the 256 threads with one batch of 18 loads (three batches of 14
// by 168 threads, one per map: 0.237 ms for 0.178, 16 slices of 1024^2).  Maps larger
// than the last-level cache (256 MB) come from HBM, and there whole columns of the tile
// by half the threads, fewer loads in all, are faster still (0.157).  The whole loss on
// slices of 1024^2, by eight rows and by whole columns: 4 (100 MB) 117 and 118 us, 6 158
// and 160, 8 (201 MB) 210 and 205, 9 245 and 235, 11 (277 MB) 293 and 278, 20 510 and
// 486; 12 MB 0.0082 and 0.0085 for the kernel.
constexpr int64_t kTallMinBytes = 1ll << 28;
static_assert(kColItems <= kThreads && 3 * kRW * (kSH / 8) <= kThreads && (kSW / kRow) * kSH == kThreads, "each pass is one round of the workgroup");
// Place of column c in a row of column sums: the even columns, then the odd ones,
// so that threads whose first outputs are kRow apart read neighbouring places.
constexpr int kPlane = (kRW + kRow - 1) / kRow, kRS = kRow * kPlane;
__device__ constexpr int place(int c) { return (c % kRow) * kPlane + c / kRow; }

struct SsimArgs {
  const float* x;       // [S][H][W] rendered slices
  const float* y;       // [S][H][W] targets
  double* maps;         // [3][S][H][W] coefficient maps
  double* part;         // [2][blocks]: per-block sums of the two loss terms
  float* grad;          // [S][H][W] dL/dI (written)
  float* loss;          // [2]: += L1 term, += D-SSIM term
  int W, H;
  int64_t npix;         // S * H * W
  double inv_n, lam;
  double w[2 * kR + 1];
};

__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[wave] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < kThreads / 64; ++i) t += sh[i];
  return t;
}

// Column gx of the slice, rows gy0 .. gy0 + N - 1, zeros outside it: all loads from
// clamped addresses (a branch around each would leave them one after the other; a
// path without clamps for tiles inside the slice was not faster).
template <int N, typename T>
__device__ __forceinline__ void load_column(const T* __restrict__ src, int gx, int gy0, int W, int H, T (&v)[N]) {
  const T* col = src + min(max(gx, 0), W - 1);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = col[(int64_t)min(max(gy0 + i, 0), H - 1) * W];
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (gx < 0 || gx >= W || gy0 + i < 0 || gy0 + i >= H) v[i] = (T)0;
}

__global__ __launch_bounds__(kThreads) void k_ssim_stats(SsimArgs a) {
  __shared__ double vs[5][kSH][kRS];   // column sums
  __shared__ double red[kThreads / 64];
  const int ox = blockIdx.x * kSW, oy = blockIdx.y * kSH;
  const int64_t base = (int64_t)blockIdx.z * a.H * a.W;
  if (threadIdx.x < kColItems) {
    const int c = threadIdx.x % kRW, r0 = threadIdx.x / kRW * kCol;
    float x[kCol + 2 * kR], y[kCol + 2 * kR];
    load_column(a.x + base, ox - kR + c, oy + r0 - kR, a.W, a.H, x);
    load_column(a.y + base, ox - kR + c, oy + r0 - kR, a.W, a.H, y);
    double t[kCol][5];
#pragma unroll
    for (int j = 0; j < kCol; ++j)
#pragma unroll
      for (int q = 0; q < 5; ++q) t[j][q] = 0.0;
#pragma unroll
    for (int i = 0; i < kCol + 2 * kR; ++i) {
      const double u = x[i], v = y[i];
      const double uu = u * u, vv = v * v, uv = u * v;
#pragma unroll
      for (int j = 0; j < kCol; ++j) {
        const int k = i - j;
        if (k < 0 || k > 2 * kR) continue;
        const double wk = a.w[k];
        t[j][0] += wk * u;
        t[j][1] += wk * v;
        t[j][2] += wk * uu;
        t[j][3] += wk * vv;
        t[j][4] += wk * uv;
      }
    }
#pragma unroll
    for (int j = 0; j < kCol; ++j)
#pragma unroll
      for (int q = 0; q < 5; ++q) vs[q][r0 + j][place(c)] = t[j][q];
  }
  __syncthreads();
  double part_l1 = 0.0, part_d = 0.0;
  const int r = threadIdx.x / (kSW / kRow), cg = threadIdx.x % (kSW / kRow);
  const int gx0 = ox + cg * kRow, gy = oy + r;
  if (gy < a.H && gx0 < a.W) {
    const int64_t o = base + (int64_t)gy * a.W + gx0;
    float px[kRow], py[kRow];
#pragma unroll
    for (int j = 0; j < kRow; ++j) {
      const int64_t oj = gx0 + j < a.W ? o + j : o;
      px[j] = a.x[oj];
      py[j] = a.y[oj];
    }
    double m[kRow][5];
#pragma unroll
    for (int q = 0; q < 5; ++q) {
#pragma unroll
      for (int j = 0; j < kRow; ++j) m[j][q] = 0.0;
#pragma unroll
      for (int i = 0; i < kRow + 2 * kR; ++i) {
        const double v = vs[q][r][place(i) + cg];
#pragma unroll
        for (int j = 0; j < kRow; ++j) {
          const int k = i - j;
          if (k >= 0 && k <= 2 * kR) m[j][q] += a.w[k] * v;
        }
      }
    }
    double out[3][kRow];
#pragma unroll
    for (int j = 0; j < kRow; ++j) {
      const double mx = m[j][0], my = m[j][1];
      const double vx = m[j][2] - mx * mx, vy = m[j][3] - my * my, cxy = m[j][4] - mx * my;
      const double A1 = 2.0 * mx * my + 1e-4, A2 = 2.0 * cxy + 9e-4;
      const double B1 = mx * mx + my * my + 1e-4, B2 = vx + vy + 9e-4;
      const double inv = 1.0 / (B1 * B2);
      const double S = A1 * A2 * inv;
      // (1 / B1 - 1 / B2 and 1 / B2 through the one division)
      out[0][j] = 2.0 * my * (A2 - A1) * inv - 2.0 * mx * S * ((B2 - B1) * inv);
      out[1][j] = -S * (B1 * inv);
      out[2][j] = 2.0 * A1 * inv;
      if (gx0 + j < a.W) {
        part_d += 1.0 - S;
        part_l1 += fabs((double)px[j] - (double)py[j]);
      }
    }
    static_assert(kRow == 2, "the maps are stored in pairs");
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      double* dst = a.maps + q * a.npix + o;
      if (gx0 + 1 < a.W && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
        *reinterpret_cast<double2*>(dst) = make_double2(out[q][0], out[q][1]);
      } else {
        dst[0] = out[q][0];
        if (gx0 + 1 < a.W) dst[1] = out[q][1];
      }
    }
  }
  const double t1 = block_sum(part_l1, red);
  __syncthreads();
  const double t2 = block_sum(part_d, red);
  if (threadIdx.x == 0) {
    const int64_t bid = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    a.part[2 * bid] = t1;
    a.part[2 * bid + 1] = t2;
  }
}

// The two loss terms from the per-block sums of k_ssim_stats, in a fixed order
// (one writer: deterministic, and no contended atomics).  Run by the first
// workgroup of k_ssim_grad, which starts after every sum is written.
__device__ void ssim_loss_sum(const double* __restrict__ part, int64_t nblocks, double inv_n,
                              float* __restrict__ loss, double* red) {
  double s1 = 0.0, s2 = 0.0;
  for (int64_t b = threadIdx.x; b < nblocks; b += kThreads) {
    s1 += part[2 * b];
    s2 += part[2 * b + 1];
  }
  const double t1 = block_sum(s1, red);
  __syncthreads();
  const double t2 = block_sum(s2, red);
  if (threadIdx.x == 0) {
    loss[0] += (float)(t1 * inv_n);
    loss[1] += (float)(t2 * inv_n);
  }
}

template <int MAP_COL>
__global__ __launch_bounds__(kThreads) void k_ssim_grad(SsimArgs a) {
  __shared__ double vs[3][kSH][kRS];   // column sums of the maps
  const int ox = blockIdx.x * kSW, oy = blockIdx.y * kSH;
  const int64_t base = (int64_t)blockIdx.z * a.H * a.W;
  constexpr int kMapItems = kRW * (kSH / MAP_COL);
  if (threadIdx.x < 3 * kMapItems) {
    const int q = threadIdx.x / kMapItems, item = threadIdx.x % kMapItems;
    const int c = item % kRW, r0 = item / kRW * MAP_COL;
    double v[MAP_COL + 2 * kR];
    load_column(a.maps + q * a.npix + base, ox - kR + c, oy + r0 - kR, a.W, a.H, v);
#pragma unroll
    for (int j = 0; j < MAP_COL; ++j) {
      double t = 0.0;
#pragma unroll
      for (int k = 0; k <= 2 * kR; ++k) t += a.w[k] * v[j + k];
      vs[q][r0 + j][place(c)] = t;
    }
  }
  __syncthreads();
  const int r = threadIdx.x / (kSW / kRow), cg = threadIdx.x % (kSW / kRow);
  const int gx0 = ox + cg * kRow, gy = oy + r;
  if (gy < a.H && gx0 < a.W) {
    const int64_t o = base + (int64_t)gy * a.W + gx0;
    float px[kRow], py[kRow];
#pragma unroll
    for (int j = 0; j < kRow; ++j) {
      const int64_t oj = gx0 + j < a.W ? o + j : o;
      px[j] = a.x[oj];
      py[j] = a.y[oj];
    }
    double u[kRow][3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
      for (int j = 0; j < kRow; ++j) u[j][q] = 0.0;
#pragma unroll
      for (int i = 0; i < kRow + 2 * kR; ++i) {
        const double v = vs[q][r][place(i) + cg];
#pragma unroll
        for (int j = 0; j < kRow; ++j) {
          const int k = i - j;
          if (k >= 0 && k <= 2 * kR) u[j][q] += a.w[k] * v;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kRow; ++j) {
      if (gx0 + j >= a.W) continue;
      const double xv = px[j], yv = py[j];
      const double sg = xv > yv ? 1.0 : (xv < yv ? -1.0 : 0.0);
      const double dS = u[j][0] + 2.0 * xv * u[j][1] + yv * u[j][2];
      a.grad[o + j] = (float)(a.inv_n * (sg - a.lam * dS));
    }
  }
  if (a.loss && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0) {
    __shared__ double red[kThreads / 64];
    ssim_loss_sum(a.part, (int64_t)gridDim.x * gridDim.y * gridDim.z, a.inv_n, a.loss, red);
  }
}

// Scratch of the allocation-free loss entry point: the coefficient maps of up to
// 2^21 pixels and the per-block sums, held by every GPU the library runs on
// until the process ends.  Host code never passes the array's name to a kernel
// (on the host it is only a stand-in): its device address is looked up once per
// device, with that device current, and that address is used instead.
constexpr int64_t kNoAllocScratchDoubles = 3ll * (1ll << 21) + (1ll << 17);
static __device__ __align__(256) double scratch[kNoAllocScratchDoubles];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_dev[kMaxDevices] = {};

}  // namespace

int64_t ssim_noalloc_capacity() { return kNoAllocScratchDoubles; }

hipError_t ssim_noalloc_scratch(double** out) {
  *out = nullptr;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_dev[dev] = static_cast<double*>(p);
  }
  *out = g_scratch_dev[dev];
  return hipSuccess;
}

int64_t ssim_scratch(int n_slices, int width, int height) {
  const int64_t blocks = (int64_t)((width + kSW - 1) / kSW) * ((height + kSH - 1) / kSH) * n_slices;
  return 3 * (int64_t)n_slices * width * height + 2 * blocks;
}

hipError_t launch_ssim_loss(const float* x, const float* y, int n_slices, int width, int height, double lam,
                            double* maps, float* grad, float* loss, hipStream_t s) {
  SsimArgs a{};
  a.x = x;
  a.y = y;
  a.maps = maps;
  a.part = maps + 3 * (int64_t)n_slices * width * height;
  a.grad = grad;
  a.loss = loss;
  a.W = width;
  a.H = height;
  a.npix = (int64_t)n_slices * width * height;
  a.inv_n = 1.0 / (double)a.npix;
  a.lam = lam;
  double sum = 0.0;
  for (int k = 0; k <= 2 * kR; ++k) {
    const double d = (double)(k - kR);
    a.w[k] = std::exp(-(d * d) / (2.0 * 1.5 * 1.5));
    sum += a.w[k];
  }
  for (int k = 0; k <= 2 * kR; ++k) a.w[k] /= sum;
  const dim3 grid((unsigned)((width + kSW - 1) / kSW), (unsigned)((height + kSH - 1) / kSH), (unsigned)n_slices);
  k_ssim_stats<<<grid, kThreads, 0, s>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (3 * (int64_t)sizeof(double) * a.npix >= kTallMinBytes)
    k_ssim_grad<16><<<grid, kThreads, 0, s>>>(a);
  else
    k_ssim_grad<8><<<grid, kThreads, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace gp
