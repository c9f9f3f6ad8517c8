// Differentiable voxeliser (Sec. 4.3, "Differentiable Voxelization"): the
// intensity volume sigma(x) = sum_i alpha_i exp(-1/2 (x - mu_i)^T Sigma_i^-1
// (x - mu_i)) of the world-space Gaussians (no focus re-parameterisation),
// accumulated over 8 x 8 x 8-voxel tiles that keep the Gaussians whose 3-sigma
// box reaches them, and its adjoint.
//
// Pipeline (one forward, no floating-point atomics anywhere):
//   k_vox_count   per Gaussian: activation, binary32 3-sigma tile box (the same
//                 operation sequence as the slice footprint: r = bbox sqrt(S_aa),
//                 floor(((mu -+ r - origin) / pitch) / 8)), the voxel-space record;
//   scan          instance slots in Gaussian order;
//   k_vox_emit    one (tile, Gaussian) pair per tile of each box;
//   radix sort    stable, by tile: every list ends in Gaussian order;
//   k_vox_fwd     one wavefront per tile; lane (x, y) of the 8 x 8 face owns the
//                 column of 8 voxels along z, so the x-y part of the quadratic
//                 form is shared by 8 voxels.
// Backward:
//   k_vox_bwd     one wavefront per tile, eight lanes per list entry (one z
//                 layer each): ten moments of G e over the tile's 512 voxels
//                 (sum, first and second moments of the offset), written at
//                 the entry's own instance slot;
//   k_vox_chain   per Gaussian: moments summed in a fixed order by eight lanes,
//                 then the chain rule to (mu, l, q, alpha), added into the
//                 gradient.
//
// Voxel-space record: with o the origin, h the pitch and d = (i + 1/2) - (mu -
// o)/h the offset of voxel i from the mean in voxel units, a contribution is
// w exp2(cxx dx^2 + cyy dy^2 + czz dz^2 + cxy dx dy + cxz dx dz + cyz dy dz),
// the coefficients carrying -1/2 log2(e), the precision matrix P = Sigma^-1 =
// R diag(1/s^2) R^T and the pitches.
#include "gp_internal.h"
#include "gp_spec.h"

#include <algorithm>
#include <cmath>

namespace gp {
namespace {

constexpr int kVT = 8;                       // tile edge in voxels
constexpr int kVTVox = kVT * kVT * kVT;      // voxels per tile
constexpr float kLog2e = 1.4426950408889634f;

struct VoxArgs {
  const float* means;
  const void* attrs;
  int64_t stride;
  int n;
  float x0, y0, z0, dx, dy, dz;
  int nx, ny, nz, ntx, nty, ntz, n_tiles;
  float bbox, scale_mod;
  uint32_t flags;
  // [n][4], one 64-byte line per Gaussian (three planes of records and three of
  // boxes cost a gather up to seven lines): (x, y, z, w), (cxx, cyy, czz, cxy),
  // (cxz, cyz, gz, gx), then as bits the tile box, t0 | t1 << 16 per axis
  // (x, y, z), which the emit replaces by (slot, w, h): the entry of tile
  // (tx, ty, tz) has the instance slot `slot` + (tz h + ty) w + tx (mod 2^32)
  float4* rec;
  uint32_t* ninst;        // [n] tiles of the box (0 if culled)
  const uint32_t* ibase;  // [n] first instance slot (scanned)
  uint32_t* inst_key;
  uint32_t* inst_val;
  uint32_t inst_cap;
  uint32_t* tile_lo;
  uint32_t* tile_hi;
  const uint32_t* list;
  const uint32_t* list_key;   // the tile of every list position
  uint32_t pieces, piece;     // the equal pieces the positions are cut into (backward), and a piece's entries
  float* vol;
  const float* gvol;
  float* mom;             // [inst][10]: M0, Mx, My, Mz, Mxx, Myy, Mzz, Mxy, Mxz, Myz
  float* grad;
  int64_t grad_stride;
};

struct VoxGauss {
  float p[11];
  SpecCov c;
  bool ok;
};

template <int DT>
__device__ __forceinline__ void vox_load(const VoxArgs& a, int j, VoxGauss& g) {
  g.p[0] = a.means[j];
  g.p[1] = a.means[a.stride + j];
  g.p[2] = a.means[2 * a.stride + j];
#pragma unroll
  for (int r = 0; r < 8; ++r) g.p[3 + r] = load_attr<DT>(a.attrs, r, a.stride, j);
  bool finite = true;
#pragma unroll
  for (int r = 0; r < 11; ++r) finite = finite && isfinite(g.p[r]);
  spec_cov(g.p[3], g.p[4], g.p[5], g.p[6], g.p[7], g.p[8], g.p[9], a.scale_mod, g.c);
  g.ok = finite && g.c.n2 > 0.0f;
}

// Binary32 tile range of one axis; false if the box misses the grid.
__device__ __forceinline__ bool vox_axis(float mu, float saa, float o, float h, int nt, float bbox, int* t0,
                                         int* t1) {
#pragma clang fp contract(off)
  const float r = bbox * sqrtf(saa);
  const float lo = floorf((((mu - r) - o) / h) * 0.125f);
  const float hi = floorf((((mu + r) - o) / h) * 0.125f);
  const float fn = (float)(nt - 1);
  if (!(hi >= 0.0f) || !(lo <= fn)) return false;
  *t0 = (int)fmaxf(lo, 0.0f);
  *t1 = (int)fminf(hi, fn);
  return true;
}

// Records with a diagonal coefficient >= -4 (sigma >= 0.42 voxel along that
// axis) take the product recurrence along it.
constexpr float kVoxSmooth = -4.0f;

template <int DT>
__global__ __launch_bounds__(256) void k_vox_count(VoxArgs a) {
  // the forward's reset of the tile ranges
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < a.n_tiles; i += (int64_t)gridDim.x * 256) {
    a.tile_lo[i] = 0u;
    a.tile_hi[i] = 0u;
  }
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= a.n) return;
  VoxGauss g;
  vox_load<DT>(a, j, g);
  int tx0 = 0, tx1 = -1, ty0 = 0, ty1 = -1, tz0 = 0, tz1 = -1;
  bool vis = g.ok;
  if (vis && (a.flags & GP_FLAG_EXACT)) {
    tx0 = 0; tx1 = a.ntx - 1; ty0 = 0; ty1 = a.nty - 1; tz0 = 0; tz1 = a.ntz - 1;
  } else if (vis) {
    vis = vox_axis(g.p[0], g.c.sxx, a.x0, a.dx, a.ntx, a.bbox, &tx0, &tx1) &&
          vox_axis(g.p[1], g.c.syy, a.y0, a.dy, a.nty, a.bbox, &ty0, &ty1) &&
          vox_axis(g.p[2], g.c.szz, a.z0, a.dz, a.ntz, a.bbox, &tz0, &tz1);
  }
  uint32_t cnt = 0u;
  if (vis) cnt = (uint32_t)((tx1 - tx0 + 1) * (ty1 - ty0 + 1) * (tz1 - tz0 + 1));
  a.ninst[j] = cnt;
  // voxel-space record (binary32 image arithmetic, not part of the membership)
  float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), r1 = r0, r2 = r0;
  if (vis) {
    const SpecCov& c = g.c;
    const float i0 = 1.0f / (c.s0 * c.s0), i1 = 1.0f / (c.s1 * c.s1), i2 = 1.0f / (c.s2 * c.s2);
    float P[3][3];
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
      for (int v = 0; v < 3; ++v) P[u][v] = c.R[u][0] * c.R[v][0] * i0 + c.R[u][1] * c.R[v][1] * i1 + c.R[u][2] * c.R[v][2] * i2;
    const float k = -0.5f * kLog2e;
    r0 = make_float4((g.p[0] - a.x0) / a.dx - 0.5f, (g.p[1] - a.y0) / a.dy - 0.5f, (g.p[2] - a.z0) / a.dz - 0.5f,
                     g.p[10]);
    r1 = make_float4(k * P[0][0] * a.dx * a.dx, k * P[1][1] * a.dy * a.dy, k * P[2][2] * a.dz * a.dz,
                     2.0f * k * P[0][1] * a.dx * a.dy);
    // the per-voxel ratio's change along z (forward columns) and along x
    // (backward rows) for the product recurrence, -1 where it is not used
    const float czz = r1.z, cxx = r1.x;
    r2 = make_float4(2.0f * k * P[0][2] * a.dx * a.dz, 2.0f * k * P[1][2] * a.dy * a.dz,
                     czz >= kVoxSmooth ? exp2f(2.0f * czz) : -1.0f, cxx >= kVoxSmooth ? exp2f(2.0f * cxx) : -1.0f);
  }
  float4* rec = a.rec + 4 * (size_t)j;
  rec[0] = r0;
  rec[1] = r1;
  rec[2] = r2;
  reinterpret_cast<uint4*>(rec)[3] = make_uint4((uint32_t)tx0 | ((uint32_t)(tx1 & 0xFFFF) << 16),
                                                (uint32_t)ty0 | ((uint32_t)(ty1 & 0xFFFF) << 16),
                                                (uint32_t)tz0 | ((uint32_t)(tz1 & 0xFFFF) << 16), 0u);
}

__global__ __launch_bounds__(256) void k_vox_emit(VoxArgs a) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= a.n) return;
  const uint32_t cnt = a.ninst[j];
  if (cnt == 0u) return;
  uint32_t slot = a.ibase[j];
  if ((uint64_t)slot + cnt > a.inst_cap) return;   // sized from the count: cannot happen
  uint4* box = reinterpret_cast<uint4*>(a.rec + 4 * (size_t)j) + 3;
  const uint32_t bx = box->x, by = box->y, bz = box->z;
  const uint32_t w = (bx >> 16) - (bx & 0xFFFFu) + 1u, h = (by >> 16) - (by & 0xFFFFu) + 1u;
  *box = make_uint4(slot - (((bz & 0xFFFFu) * h + (by & 0xFFFFu)) * w + (bx & 0xFFFFu)), w, h, 0u);
  for (int tz = (int)(bz & 0xFFFFu); tz <= (int)(bz >> 16); ++tz)
    for (int ty = (int)(by & 0xFFFFu); ty <= (int)(by >> 16); ++ty)
      for (int tx = (int)(bx & 0xFFFFu); tx <= (int)(bx >> 16); ++tx, ++slot) {
        a.inst_key[slot] = (uint32_t)((tz * a.nty + ty) * a.ntx + tx);
        a.inst_val[slot] = (uint32_t)j;
      }
}

__global__ __launch_bounds__(256) void k_vox_ranges(const uint32_t* __restrict__ key, uint32_t n, uint32_t n_tiles,
                                                    uint32_t* __restrict__ lo, uint32_t* __restrict__ hi) {
  for (uint32_t p = blockIdx.x * 256 + threadIdx.x; p < n; p += gridDim.x * 256) {
    const uint32_t b = key[p];
    if (b >= n_tiles) continue;
    if (p == 0 || key[p - 1] != b) lo[b] = p;
    if (p + 1 == n || key[p + 1] != b) hi[b] = p + 1;
  }
}

__device__ __forceinline__ void vox_tile_xyz(const VoxArgs& a, int tile, int* tx, int* ty, int* tz) {
  *tx = tile % a.ntx;
  *ty = (tile / a.ntx) % a.nty;
  *tz = tile / (a.ntx * a.nty);
}

// One wavefront (and workgroup) per tile; lane (lx, ly) owns the column of 8
// voxels along z.  The hardware's dispatch is the work queue: a shared
// counter, with one ticket per item, had bounded this kernel and the backward
// (same-address atomics are served at about one per 12 ns, whatever the number
// of wavefronts asking: 0.43 -> 0.32 ms here, 0.68 -> 0.50 ms there, on the 51,200
// tiles of 256 x 256 x 400 voxels).  With it went the pairs of tiles per item
// (now 0.7 % slower than one) and any need to place neighbours on one XCD (no
// change at runs of 1, 16 or 64 tiles).
__global__ __launch_bounds__(64) void k_vox_fwd(VoxArgs a) {
  __shared__ float4 b0[64], b1[64], b2[64];
  const int lane = threadIdx.x;
  const int lx = lane & 7, ly = lane >> 3;
  for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
    int tx, ty, tz;
    vox_tile_xyz(a, tile, &tx, &ty, &tz);
    const float fx = (float)(tx * kVT + lx), fy = (float)(ty * kVT + ly), fz0 = (float)(tz * kVT);
    const uint32_t start = a.tile_lo[tile], end = a.tile_hi[tile];
    float acc[kVT];
#pragma unroll
    for (int k = 0; k < kVT; ++k) acc[k] = 0.f;
    for (uint32_t base = start; base < end; base += 64) {
      if (base + lane < end) {
        const uint32_t j = a.list[base + lane];
        const float4* rec = a.rec + 4 * (size_t)j;
        b0[lane] = rec[0];
        b1[lane] = rec[1];
        b2[lane] = rec[2];
      }
      __syncthreads();
      const int cnt = __builtin_amdgcn_readfirstlane((int)min(64u, end - base));
      for (int e = 0; e < cnt; ++e) {
        const float4 r0 = b0[e], r1 = b1[e], r2 = b2[e];
        const float ddx = fx - r0.x, ddy = fy - r0.y;
        // q = cxx dx^2 + cxy dx dy + cyy dy^2 + dz (cxz dx + cyz dy + czz dz)
        const float pxy = fmaf(fmaf(r1.x, ddx, r1.w * ddy), ddx, r1.y * ddy * ddy);
        const float lz = fmaf(r2.x, ddx, r2.y * ddy);
        const float dz0 = fz0 - r0.z;
        float ev[kVT];
        if (r2.z > 0.0f) {
          // two four-voxel segments, each from an exact exp2 by the product
          // recurrence along z (the raster's reasoning with czz >= -4: a
          // ratio that overflows meets e = 0, and 0 * inf = 0)
#pragma unroll
          for (int h = 0; h < kVT; h += 4) {
            const float dz = dz0 + (float)h;
            ev[h] = __builtin_amdgcn_exp2f(fmaf(fmaf(r1.z, dz, lz), dz, pxy));
            float r = __builtin_amdgcn_exp2f(fmaf(r1.z, fmaf(2.0f, dz, 1.0f), lz));
#pragma unroll
            for (int k = 1; k < 4; ++k) {
              ev[h + k] = mul0(ev[h + k - 1], r);
              r *= r2.z;
            }
          }
        } else {
#pragma unroll
          for (int k = 0; k < kVT; ++k) {
            const float dz = dz0 + (float)k;
            ev[k] = __builtin_amdgcn_exp2f(fmaf(fmaf(r1.z, dz, lz), dz, pxy));
          }
        }
        // (added up after the branch: sums formed inside it cost a move each)
#pragma unroll
        for (int k = 0; k < kVT; ++k) acc[k] = fmaf(r0.w, ev[k], acc[k]);
      }
      __syncthreads();
    }
    const int ix = tx * kVT + lx, iy = ty * kVT + ly;
    if (ix < a.nx && iy < a.ny) {
#pragma unroll
      for (int k = 0; k < kVT; ++k) {
        const int iz = tz * kVT + k;
        if (iz < a.nz) a.vol[((int64_t)iz * a.ny + iy) * a.nx + ix] = acc[k];
      }
    }
  }
}

// One wavefront (and workgroup) per tile, eight lanes per list entry:
// lane z of an entry's eight sweeps the tile's layer z, so the offset along z
// is a constant of the lane and the z-moments follow from its layer's sums.
// Bound by fp32 VALU.  A tile of the 256 x 256 x 400 volume lists about 76
// entries: with one lane per entry and 256 lanes per tile, one wavefront ran 64
// of them, the next 12, and two waited; in eighths of an entry the list is
// ten rounds of one wavefront, nearly all of them full (with the work counter
// gone too: 0.818 -> 0.498 ms).  The layers are kLayer floats apart in LDS, so that the eight
// rows the wavefront reads at a time lie in different banks.
//
// A small volume, or a clump in a large one, has few tiles with long lists.  So the
// positions of the lists, laid end to end, are cut into at most kVoxPieces equal pieces
// of at least kVoxMinPiece entries, and a list longer than a piece is swept up to the
// first cut by its tile's workgroup and from each cut on by the workgroup of that piece
// (at the front of the grid; those whose cut lies in a shorter list leave at once).
// 100,000 Gaussians on 48^3 voxels: 1.38 -> 0.151 ms (four wavefronts per tile 0.366), in
// a corner of that size of 256^3 2.90 -> 0.188 (1.02), 10,000 on 64^3 0.091 -> 0.050
// (0.058); the volume of 51,200 tiles above unchanged.  4,096 pieces: 0.165 and 0.211, and
// 0.383 for 0.314 on 128^3 with 200,000; at least 32 entries 0.030 for 0.038 on 16^3 with
// 1,000, at least 128 0.054.
constexpr int kLayer = kVT * kVT + 4;
constexpr uint32_t kVoxPieces = 8192, kVoxMinPiece = 64;

__global__ __launch_bounds__(64) void k_vox_bwd(VoxArgs a) {
  __shared__ __align__(16) float G[kVT * kLayer];
  const int lane = threadIdx.x;
  const int lz = lane & 7, sub = lane >> 3;
  const int pieces = (int)a.pieces;
  const bool is_piece = (int)blockIdx.x < pieces;
  const uint32_t cut = is_piece ? blockIdx.x * a.piece : 0u;   // a filled position
  int tile = is_piece ? (int)a.list_key[cut] : (int)blockIdx.x - pieces;
  for (; tile < a.n_tiles; tile = is_piece ? a.n_tiles : tile + (int)gridDim.x - pieces) {
    uint32_t start = a.tile_lo[tile], end = a.tile_hi[tile];
    const bool cuts = end - start > a.piece;
    if (is_piece) {
      if (!cuts || start == cut) continue;   // the tile's workgroup does it
      start = cut;
      end = cut + min(end - cut, a.piece);
    } else if (cuts) {
      end = start + min(end - start, a.piece - start % a.piece);   // to the first cut after its start
    }
    if (start != end) {
      int tx, ty, tz;
      vox_tile_xyz(a, tile, &tx, &ty, &tz);
      uint32_t jn = start + sub < end ? a.list[start + sub] : 0u;
      {
        // (clamped addresses: a branch around each load would leave them one
        // after the other)
        const int ix = tx * kVT + (lane & 7), iy = ty * kVT + (lane >> 3);
        const bool in = ix < a.nx && iy < a.ny;
        const float* col = a.gvol + (int64_t)min(iy, a.ny - 1) * a.nx + min(ix, a.nx - 1);
        const int64_t plane = (int64_t)a.ny * a.nx;
        float v[kVT];
#pragma unroll
        for (int k = 0; k < kVT; ++k) v[k] = col[min(tz * kVT + k, a.nz - 1) * plane];
#pragma unroll
        for (int k = 0; k < kVT; ++k) G[k * kLayer + lane] = in && tz * kVT + k < a.nz ? v[k] : 0.f;
      }
      __syncthreads();
      const float fx0 = (float)(tx * kVT), fy0 = (float)(ty * kVT), fz = (float)(tz * kVT + lz);
      const float* layer = G + lz * kLayer;
      for (uint32_t eb = start; eb < end; eb += 8) {
        const uint32_t idx = eb + sub;
        const bool valid = idx < end;
        const uint32_t j = jn;
        if (idx + 8 < end) jn = a.list[idx + 8];
        float V[10];   // M0, Mx, My, Mz, Mxx, Myy, Mzz, Mxy, Mxz, Myz of the lane's layer
#pragma unroll
        for (int i = 0; i < 10; ++i) V[i] = 0.f;
        uint32_t slot = 0u;
        if (valid) {
          const float4* rec = a.rec + 4 * (size_t)j;
          const float4 r0 = rec[0], r1 = rec[1], r2 = rec[2];
          const uint4 r3 = reinterpret_cast<const uint4*>(rec)[3];
          slot = r3.x + ((uint32_t)tz * r3.z + (uint32_t)ty) * r3.y + (uint32_t)tx;
          const float dz = fz - r0.z;
          float dxs[kVT];
#pragma unroll
          for (int c = 0; c < kVT; ++c) dxs[c] = (fx0 - r0.x) + (float)c;
          const float bz = r2.x * dz, cz = r1.z * dz * dz, lz_y = r2.y * dz;
          float M0 = 0.f, Mx = 0.f, My = 0.f, Mxx = 0.f, Myy = 0.f, Mxy = 0.f;
          // (one path for the wavefront: the recurrence only where all of its
          // entries allow it)
          const bool smooth = __builtin_amdgcn_read_exec() == __builtin_amdgcn_ballot_w64(r2.w > 0.0f);
          for (int y = 0; y < kVT; ++y) {
            const float dy = (fy0 + (float)y) - r0.y;
            // q = cxx dx^2 + dx (cxy dy + cxz dz) + (cyy dy^2 + cyz dy dz + czz dz^2)
            const float bx = fmaf(r1.w, dy, bz);
            const float c0 = fmaf(fmaf(r1.y, dy, lz_y), dy, cz);
            const float4 g0 = *reinterpret_cast<const float4*>(layer + y * kVT);
            const float4 g1 = *reinterpret_cast<const float4*>(layer + y * kVT + 4);
            const float grow[kVT] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
            float s0 = 0.f, sx = 0.f, sxx = 0.f;
            float ev[kVT];
            if (smooth) {
              // the product recurrence along x over two four-voxel segments
#pragma unroll
              for (int h = 0; h < kVT; h += 4) {
                const float d = dxs[h];
                ev[h] = __builtin_amdgcn_exp2f(fmaf(fmaf(r1.x, d, bx), d, c0));
                float r = __builtin_amdgcn_exp2f(fmaf(r1.x, fmaf(2.0f, d, 1.0f), bx));
#pragma unroll
                for (int k = 1; k < 4; ++k) {
                  ev[h + k] = mul0(ev[h + k - 1], r);
                  r *= r2.w;
                }
              }
            } else {
#pragma unroll
              for (int c = 0; c < kVT; ++c) {
                const float d = dxs[c];
                ev[c] = __builtin_amdgcn_exp2f(fmaf(fmaf(r1.x, d, bx), d, c0));
              }
            }
#pragma unroll
            for (int c = 0; c < kVT; ++c) {
              const float d = dxs[c];
              const float we = grow[c] * ev[c];
              const float wd = we * d;
              s0 += we;
              sx += wd;
              sxx = fmaf(wd, d, sxx);
            }
            M0 += s0;
            Mx += sx;
            Mxx += sxx;
            My = fmaf(dy, s0, My);
            Myy = fmaf(dy * dy, s0, Myy);
            Mxy = fmaf(dy, sx, Mxy);
          }
          V[0] = M0; V[1] = Mx; V[2] = My; V[3] = dz * M0; V[4] = Mxx;
          V[5] = Myy; V[6] = (dz * dz) * M0; V[7] = Mxy; V[8] = dz * Mx; V[9] = dz * My;
        }
        // the sums over an entry's eight layers, scattered over its lanes (in a
        // fixed order): lane bits 2, 1, 0 choose a half of the values each time
        const bool b2 = (lz & 4) != 0, b1 = (lz & 2) != 0, b0 = (lz & 1) != 0;
        float u[6];
#pragma unroll
        for (int i = 0; i < 5; ++i) u[i] = (b2 ? V[5 + i] : V[i]) + __shfl_xor(b2 ? V[i] : V[5 + i], 4, 64);
        u[5] = 0.f;
        float v[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = (b1 ? u[3 + i] : u[i]) + __shfl_xor(b1 ? u[i] : u[3 + i], 2, 64);
        const float w0 = (b0 ? v[2] : v[0]) + __shfl_xor(b0 ? v[0] : v[2], 1, 64);
        const float w1 = (b0 ? 0.f : v[1]) + __shfl_xor(b0 ? v[1] : 0.f, 1, 64);
        if (valid) {
          float* m = a.mom + 10 * (size_t)slot + (b2 ? 5 : 0) + (b1 ? 3 : 0) + (b0 ? 2 : 0);
          if (!(b1 && b0)) m[0] = w0;
          if (!b0) m[1] = w1;
        }
      }
      __syncthreads();   // G[] is reused by the next tile
    }
  }
}

// Chain rule per Gaussian.  With d_w = h * d_v the world offset (h the pitch),
// e = exp(-1/2 d_w^T P d_w) and P = R diag(1/s^2) R^T:
//   dL/dalpha = sum G e = M0
//   dL/dmu    = alpha P (h * m1)                  (m1 = sum G e d_v)
//   dL/dP     = -1/2 alpha (h h^T) * M2           (M2 = sum G e d_v d_v^T)
//   dL/dl_k   = -2 / s_k^2 r_k^T (dL/dP) r_k      (s_k = exp(l_k) mod)
//   dL/dR_ak  = 2 / s_k^2 (dL/dP r_k)_a
// then through R(q^) and the normalisation q^ = q / |q|.
//
// Bound by the moments it reads (40 B per instance).  A wavefront's 64
// Gaussians own one contiguous run of slots: eight lanes per Gaussian, eight
// Gaussians at a time, read neighbouring slots and add their sums by a
// fixed butterfly; the chain rule then runs with one lane per Gaussian (one
// lane reading all of its own slots took 0.162 ms for the 500,000 Gaussians
// of the 400-slice volume, this 0.047 ms).
template <int DT>
__global__ __launch_bounds__(256) void k_vox_chain(VoxArgs a) {
  __shared__ float sums[4][64][11];   // (ten used; the odd stride spreads the banks)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = blockIdx.x * 256 + threadIdx.x;
  const uint32_t cnt = j < a.n ? a.ninst[j] : 0u;
  const uint32_t first = j < a.n ? a.ibase[j] : 0u;
#pragma unroll 2
  for (int r = 0; r < 8; ++r) {
    const int gi = 8 * r + (lane >> 3);
    const uint32_t c = __shfl(cnt, gi, 64), s0 = __shfl(first, gi, 64);
    float m[10];
#pragma unroll
    for (int i = 0; i < 10; ++i) m[i] = 0.f;
    for (uint32_t s = lane & 7; s < c; s += 8) {
      const float2* src = reinterpret_cast<const float2*>(a.mom + 10 * (size_t)(s0 + s));
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        const float2 v = src[i];
        m[2 * i] += v.x;
        m[2 * i + 1] += v.y;
      }
    }
#pragma unroll
    for (int o = 1; o < 8; o <<= 1)
#pragma unroll
      for (int i = 0; i < 10; ++i) m[i] += __shfl_xor(m[i], o, 64);
    if ((lane & 7) == 0)
#pragma unroll
      for (int i = 0; i < 10; ++i) sums[wave][gi][i] = m[i];
  }
  __syncthreads();
  if (cnt == 0u) return;
  VoxGauss g;
  vox_load<DT>(a, j, g);
  const float* m = sums[wave][lane];
  const float M0 = m[0], m1[3] = {m[1], m[2], m[3]};
  float M2[3][3] = {{m[4], m[7], m[8]}, {0.f, m[5], m[9]}, {0.f, 0.f, m[6]}};
  M2[1][0] = M2[0][1]; M2[2][0] = M2[0][2]; M2[2][1] = M2[1][2];
  const SpecCov& c = g.c;
  const float alpha = g.p[10];
  const float h[3] = {a.dx, a.dy, a.dz};
  const float is[3] = {1.0f / (c.s0 * c.s0), 1.0f / (c.s1 * c.s1), 1.0f / (c.s2 * c.s2)};
  float P[3][3];
#pragma unroll
  for (int u = 0; u < 3; ++u)
#pragma unroll
    for (int v = 0; v < 3; ++v) P[u][v] = c.R[u][0] * c.R[v][0] * is[0] + c.R[u][1] * c.R[v][1] * is[1] + c.R[u][2] * c.R[v][2] * is[2];
  float gmu[3];
#pragma unroll
  for (int u = 0; u < 3; ++u) gmu[u] = alpha * (P[u][0] * h[0] * m1[0] + P[u][1] * h[1] * m1[1] + P[u][2] * h[2] * m1[2]);
  float GP[3][3];
#pragma unroll
  for (int u = 0; u < 3; ++u)
#pragma unroll
    for (int v = 0; v < 3; ++v) GP[u][v] = -0.5f * alpha * h[u] * h[v] * M2[u][v];
  float gl[3], GR[3][3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    float t[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) t[u] = GP[u][0] * c.R[0][k] + GP[u][1] * c.R[1][k] + GP[u][2] * c.R[2][k];
    gl[k] = -2.0f * is[k] * (c.R[0][k] * t[0] + c.R[1][k] * t[1] + c.R[2][k] * t[2]);
#pragma unroll
    for (int u = 0; u < 3; ++u) GR[u][k] = 2.0f * is[k] * t[u];
  }
  const float w = c.w, x = c.x, y = c.y, z = c.z;
  const float gw = 2.0f * (-z * GR[0][1] + y * GR[0][2] + z * GR[1][0] - x * GR[1][2] - y * GR[2][0] + x * GR[2][1]);
  const float gx = 2.0f * (y * GR[0][1] + z * GR[0][2] + y * GR[1][0] - 2.0f * x * GR[1][1] - w * GR[1][2] +
                           z * GR[2][0] + w * GR[2][1] - 2.0f * x * GR[2][2]);
  const float gy = 2.0f * (-2.0f * y * GR[0][0] + x * GR[0][1] + w * GR[0][2] + x * GR[1][0] + z * GR[1][2] -
                           w * GR[2][0] + z * GR[2][1] - 2.0f * y * GR[2][2]);
  const float gz = 2.0f * (-2.0f * z * GR[0][0] - w * GR[0][1] + x * GR[0][2] + w * GR[1][0] - 2.0f * z * GR[1][1] +
                           y * GR[1][2] + x * GR[2][0] + y * GR[2][1]);
  // through q^ = q / |q|
  const float rn = 1.0f / sqrtf(c.n2);
  const float dot = w * gw + x * gx + y * gy + z * gz;
  float* gp = a.grad + j;
  const int64_t gs = a.grad_stride;
  gp[0] += gmu[0];
  gp[gs] += gmu[1];
  gp[2 * gs] += gmu[2];
  gp[3 * gs] += gl[0];
  gp[4 * gs] += gl[1];
  gp[5 * gs] += gl[2];
  gp[6 * gs] += (gw - w * dot) * rn;
  gp[7 * gs] += (gx - x * dot) * rn;
  gp[8 * gs] += (gy - y * dot) * rn;
  gp[9 * gs] += (gz - z * dot) * rn;
  gp[10 * gs] += M0;
}

}  // namespace

VoxLaunch vox_prepare(const gp_gaussians* g, const gp_volume_grid* grid, const gp_render_opts* o) {
  VoxLaunch L{};
  L.n = (int)g->n;
  L.ntx = (grid->nx + kVT - 1) / kVT;
  L.nty = (grid->ny + kVT - 1) / kVT;
  L.ntz = (grid->nz + kVT - 1) / kVT;
  L.n_tiles = (int64_t)L.ntx * L.nty * L.ntz;
  (void)o;
  return L;
}

static VoxArgs vox_args(const Workspace& ws, const gp_gaussians* g, const gp_volume_grid* grid,
                        const gp_render_opts* o, const VoxLaunch& L) {
  VoxArgs a{};
  a.means = static_cast<const float*>(g->means);
  a.attrs = g->attrs;
  a.stride = g->stride;
  a.n = L.n;
  a.x0 = grid->x0; a.y0 = grid->y0; a.z0 = grid->z0;
  a.dx = grid->dx; a.dy = grid->dy; a.dz = grid->dz;
  a.nx = grid->nx; a.ny = grid->ny; a.nz = grid->nz;
  a.ntx = L.ntx; a.nty = L.nty; a.ntz = L.ntz;
  a.n_tiles = (int)L.n_tiles;
  a.bbox = o->bbox_sigmas;
  a.scale_mod = o->scale_mod;
  a.flags = o->flags;
  a.rec = ws.d_vox_rec;
  a.ninst = ws.d_g_ninst;
  a.ibase = ws.d_g_rbase;
  a.inst_key = ws.d_inst_key;
  a.inst_val = ws.d_inst_val;
  a.inst_cap = (uint32_t)ws.inst_cap;
  a.tile_lo = ws.d_bin_lo;
  a.tile_hi = ws.d_bin_hi;
  a.list = ws.d_list;
  a.list_key = ws.d_list_key;
  a.mom = ws.d_vox_mom;
  return a;
}

hipError_t launch_vox_count(const Workspace& ws, const gp_gaussians* g, const gp_volume_grid* grid,
                            const gp_render_opts* o, const VoxLaunch& L, hipStream_t s) {
  if (L.n <= 0) return hipSuccess;
  const VoxArgs a = vox_args(ws, g, grid, o, L);
  // enough workgroups for the reset of the tile ranges too (16 tiles per thread): 64
  // Gaussians on a million tiles 0.465 -> 0.320 ms (65,536 there 0.351)
  const int64_t reset_blocks = std::min<int64_t>((L.n_tiles + 4095) / 4096, 16384);
  const unsigned blocks = (unsigned)std::max<int64_t>(((int64_t)L.n + 255) / 256, reset_blocks);
  switch (g->attr_dtype) {
    case GP_BF16: k_vox_count<GP_BF16><<<blocks, 256, 0, s>>>(a); break;
    case GP_F16: k_vox_count<GP_F16><<<blocks, 256, 0, s>>>(a); break;
    case GP_Q16: k_vox_count<GP_Q16><<<blocks, 256, 0, s>>>(a); break;
    default: k_vox_count<GP_F32><<<blocks, 256, 0, s>>>(a); break;
  }
  return hipGetLastError();
}

hipError_t launch_vox_emit(const Workspace& ws, const gp_gaussians* g, const gp_volume_grid* grid,
                           const gp_render_opts* o, const VoxLaunch& L, hipStream_t s) {
  if (L.n <= 0) return hipSuccess;
  const VoxArgs a = vox_args(ws, g, grid, o, L);
  k_vox_emit<<<(unsigned)((L.n + 255) / 256), 256, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_vox_ranges(const Workspace& ws, const VoxLaunch& L, uint32_t n_inst, hipStream_t s) {
  if (n_inst == 0) return hipSuccess;   // (the count cleared the ranges)
  int64_t blocks = ((int64_t)n_inst + 255) / 256;
  blocks = blocks > 8192 ? 8192 : blocks;
  k_vox_ranges<<<(unsigned)blocks, 256, 0, s>>>(ws.d_list_key, n_inst, (uint32_t)L.n_tiles, ws.d_bin_lo,
                                                ws.d_bin_hi);
  return hipGetLastError();
}

// One workgroup per tile (of larger grids, several tiles per workgroup).
static unsigned vox_grid(int64_t tiles) { return (unsigned)(tiles < (1 << 22) ? tiles : (1 << 22)); }

hipError_t launch_vox_fwd(const Workspace& ws, const gp_gaussians* g, const gp_volume_grid* grid,
                          const gp_render_opts* o, const VoxLaunch& L, float* vol, hipStream_t s) {
  if (L.n_tiles <= 0) return hipSuccess;
  VoxArgs a = vox_args(ws, g, grid, o, L);
  a.vol = vol;
  k_vox_fwd<<<vox_grid(L.n_tiles), 64, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_vox_bwd(const Workspace& ws, const gp_gaussians* g, const gp_volume_grid* grid,
                          const gp_render_opts* o, const VoxLaunch& L, const float* gvol, float* grad,
                          int64_t grad_stride, hipStream_t s) {
  if (L.n_tiles <= 0 || L.n <= 0) return hipSuccess;
  VoxArgs a = vox_args(ws, g, grid, o, L);
  a.gvol = gvol;
  a.grad = grad;
  a.grad_stride = grad_stride;
  const uint32_t n_list = (uint32_t)ws.vox_ninst;
  a.piece = std::max(kVoxMinPiece, n_list / kVoxPieces + 1u);
  a.pieces = n_list / a.piece + (n_list % a.piece != 0u ? 1u : 0u);
  k_vox_bwd<<<vox_grid(L.n_tiles) + a.pieces, 64, 0, s>>>(a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const unsigned gb = (unsigned)((L.n + 255) / 256);
  switch (g->attr_dtype) {
    case GP_BF16: k_vox_chain<GP_BF16><<<gb, 256, 0, s>>>(a); break;
    case GP_F16: k_vox_chain<GP_F16><<<gb, 256, 0, s>>>(a); break;
    case GP_Q16: k_vox_chain<GP_Q16><<<gb, 256, 0, s>>>(a); break;
    default: k_vox_chain<GP_F32><<<gb, 256, 0, s>>>(a); break;
  }
  return hipGetLastError();
}

}  // namespace gp
