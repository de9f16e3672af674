// ring2.hip -- the IFCM step for the two Chebyshev rings of the 5x5x5 cube
// (V = 2, eq (10) weights W_1, W_2), fused like the 3x3x3 step, for C <= 4.
//
// Per voxel i and ring r (the cells at Chebyshev distance r):
//   H_ij = sum_r W_r g_inv_ir sum_{k in r} u_kj g_ik    (eqs (5), (6), (10))
//   F_ij = sum_r W_r q_inv_ir sum_{k in r} u_kj^2 q_ik  (eqs (7), (8), (10))
// with g_inv_ir = 1 / sum_{k in r} g_ik and q_inv_ir = 1 / sum_{k in r} q_ik.
// Both depend on x only and are computed once per call (k_ring2_invariants);
// a ring whose cells all share the voxel's intensity stores -1 / n_r and its
// centre value is shifted by -1 when forming g, so every g_ik of it is 1 and
// the ring contributes the mean of its memberships (the equal-weight limit).
//
// Work decomposition: as in the fused step, a wave owns a tile of 16 x 4
// columns and zc planes and walks it along z.  Each plane of the tile plus a
// two-voxel halo (20 x 8 cells of x and U) is staged once in the wave's LDS
// (four plane buffers), and every lane reads its 5 x 5 in-plane cells once:
// they contribute to the five voxels of its column at planes p-2 .. p+2, kept
// in five register slots that move down by one after each plane (mostly
// in the destination of the last sum).  For F the squared memberships of the 25
// cells are summed per in-plane offset class once per plane and weighted per
// plane distance, which two slots share.  The last cluster's H comes from
// sum_j H_ij = sum_r W_r (rows of U sum to 1).  Voxel p-2 is complete after
// plane p and is finalised: eqs (4), (1), (2), (3) as in the fused step.
//
// Bound by VALU issue: 124 differences, 372 + 100 + 84 multiply-adds for H, the
// squares and F at C = 4, 829 instructions per voxel in all (939 before).  Two
// waves per SIMD: the ring invariants wait in LDS for their voxel instead of in
// the slots, ring 1 has no slot p+2, cells beside the volume are zeroed once per
// tile and their lanes store to a spare cell, so loads need no test and plane
// bases are scalar.  At C = 4 two waves leave 256 registers and 8 to 20 are
// spilled (writes 1.08 x the new memberships); C = 2 and 3 fit.  A step of 8
// particles on 204 x 251 x 104, C = 4: 1659 -> 1065 us.
#include "common.h"
#include "pifcm_kernels.h"

namespace pifcm {

// Ring invariants of one volume: per voxel and ring g_inv (or -1 / n_r, see
// above; 0 for a ring without cells) and q_inv.
//
// A wave owns kInv2Cols x kInv2Rows columns of a run of zc planes and walks it
// along z.  Lane l holds column x0 - 2 + l (the two outer lanes on each side are
// halo), the columns beside it come from the lanes beside it (DPP wave shifts),
// the rows from its own registers, and each plane serves the voxels of five
// planes.  Cells outside the volume are loaded from a clamped address and
// weighted 0.  The eq (7) denominators depend on the position only: products of
// per-axis sums of 1, d^2 and d^4 over the offsets inside the volume (whole
// numbers, exact), formed again only for planes next to a z face.
// Bound by VALU issue (124 differences and sums per voxel): 85 us for 204 x 251 x
// 104 voxels, where one thread per voxel reading its 124 neighbours through the
// caches with a test each took 328 us.
constexpr int kInv2Cols = 60, kInv2Rows = 2;

namespace {
// Sums of 1, d^2 and d^4 over the offsets |d| <= r of one axis that stay inside
// the volume (r = 1, 2).
struct Axis {
  float n[2], a[2], b[2];
};
__device__ __forceinline__ Axis axis_sums(int g, int n) {
  const int e1 = (g > 0) + (g < n - 1), e2 = (g > 1) + (g < n - 2);
  Axis s;
  s.n[0] = (float)(1 + e1);
  s.a[0] = s.b[0] = (float)e1;
  s.n[1] = (float)(1 + e1 + e2);
  s.a[1] = (float)(e1 + 4 * e2);
  s.b[1] = (float)(e1 + 16 * e2);
  return s;
}
// Cells of ring r (0, 1) and the inverse of their eq (7) weights' sum.
__device__ __forceinline__ void ring_sums(const Axis& x, const Axis& y, const Axis& z, int q2_sqdist,
                                          float (&cnt)[2], float (&qinv)[2]) {
  float q[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const float xy = x.n[r] * y.n[r], a = x.a[r] * y.n[r] + y.a[r] * x.n[r];
    cnt[r] = xy * z.n[r] - 1.f;
    if (q2_sqdist)
      q[r] = a * z.n[r] + z.a[r] * xy;
    else
      q[r] = (x.b[r] * y.n[r] + y.b[r] * x.n[r] + 2.f * (x.a[r] * y.a[r])) * z.n[r] + z.b[r] * xy + 2.f * (z.a[r] * a);
  }
  cnt[1] -= cnt[0];
  q[1] -= q[0];
#pragma unroll
  for (int r = 0; r < 2; ++r) qinv[r] = cnt[r] > 0.f ? 1.f / q[r] : 0.f;
}
}  // namespace

__global__ __launch_bounds__(256) void k_ring2_invariants(const float* __restrict__ x, float* __restrict__ rinv,
                                                          int nx, int ny, int nz, int zc, int nitems,
                                                          int q2_sqdist) {
  constexpr int R = kInv2Rows;
  const int lane = threadIdx.x & 63;
  const int item = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (item >= nitems) return;
  const int ntx = (nx + kInv2Cols - 1) / kInv2Cols, nty = (ny + R - 1) / R;
  const int gx = (item % ntx) * kInv2Cols + lane - 2, y0 = (item / ntx) % nty * R;
  const int zlo = item / ntx / nty * zc, zhi = min(zlo + zc, nz);
  const bool own = lane >= 2 && lane < 2 + kInv2Cols && gx < nx;
  const int cx = min(max(gx, 0), nx - 1);
  // Weights (0 or 1) of the cells two left of the lane's column to two right of
  // it, by row: rows y0 - 2 .. y0 + R + 1.
  float w[R + 4][5];
  uint32_t ofs[R + 4];
#pragma unroll
  for (int r = 0; r < R + 4; ++r) {
    const int gy = y0 - 2 + r;
#pragma unroll
    for (int d = 0; d < 5; ++d)
      w[r][d] = gy >= 0 && gy < ny && gx + d - 2 >= 0 && gx + d - 2 < nx ? 1.f : 0.f;
    ofs[r] = ((uint32_t)min(max(gy, 0), ny - 1) * (uint32_t)nx + (uint32_t)cx) * 4u;
  }
  const size_t psz = (size_t)nx * ny;
  auto load = [&](int p, float (&v)[R + 4]) __attribute__((always_inline)) {
    const gfloat* base = opaque_base(as_global(x) + (size_t)min(max(p, 0), nz - 1) * psz);
#pragma unroll
    for (int r = 0; r < R + 4; ++r) v[r] = *at_lane(base, ofs[r]);
  };
  const Axis ax = axis_sums(gx, nx);
  float cnt[R][2], qinv[R][2];
  bool full = false;  // cnt and qinv are those of a plane off the z faces
  // x of the planes p - 2 .. p + 2 (xs[4] and the rows beside the lane's own
  // only as the next planes' cells), and the ring sums of their voxels: ring 1
  // starts a plane later.
  float xs[5][R + 4], ahead[R + 4], s1[R][4], s2[R][5];
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int k = 0; k < 4; ++k) s1[r][k] = 0.f;
#pragma unroll
    for (int k = 0; k < 5; ++k) s2[r][k] = 0.f;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int r = 0; r < R + 4; ++r) xs[k][r] = 0.f;
  load(zlo - 2, xs[2]);
  load(zlo - 1, xs[3]);
  load(zlo, xs[4]);
  for (int p = zlo - 2; p <= zhi + 1; ++p) {
    load(p + 3, ahead);
    if (p >= 0 && p < nz) {
      float c[R + 4][5];
#pragma unroll
      for (int r = 0; r < R + 4; ++r) {
        c[r][2] = xs[2][r];
        c[r][1] = from_left_lane(c[r][2]);
        c[r][0] = from_left_lane(c[r][1]);
        c[r][3] = from_right_lane(c[r][2]);
        c[r][4] = from_right_lane(c[r][3]);
      }
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int dy = 0; dy < 5; ++dy)
#pragma unroll
          for (int dx = 0; dx < 5; ++dx)
#pragma unroll
            for (int k = 0; k < 5; ++k) {  // voxel of plane p - 2 + k
              if (dy == 2 && dx == 2 && k == 2) continue;
              const bool in1 = dy >= 1 && dy <= 3 && dx >= 1 && dx <= 3 && k >= 1 && k <= 3;
              float& s = in1 ? s1[r][k] : s2[r][k];
              s = fmaf(fabsf(xs[k][r + 2] - c[r + dy][dx]), w[r + dy][dx], s);
            }
    }
    const int z = p - 2;
    if (z >= zlo) {
      gfloat* out = opaque_base(as_global(rinv) + (size_t)z * psz * 4);
      const bool inner = z > 1 && z < nz - 2;
      if (!inner || !full) {
        const Axis az = axis_sums(z, nz);
#pragma unroll
        for (int r = 0; r < R; ++r) ring_sums(ax, axis_sums(y0 + r, ny), az, q2_sqdist, cnt[r], qinv[r]);
        full = inner;
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (own && y0 + r < ny) {
          float o[4];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const float g = q == 0 ? s1[r][0] : s2[r][0];
            const float d = (g > 0.f ? 1.f : -1.f) / (g > 0.f ? g : cnt[r][q]);
            o[q] = g > 0.f || cnt[r][q] > 0.f ? d : 0.f;
            o[2 + q] = qinv[r][q];
          }
          uint32_t at = ofs[r + 2] * 4u;
          store_row<4>(at_lane(out, at), o);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int r = 0; r < R + 4; ++r) xs[k][r] = xs[k + 1][r];
#pragma unroll
    for (int r = 0; r < R + 4; ++r) xs[4][r] = ahead[r];
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
      for (int k = 0; k < 3; ++k) s1[r][k] = s1[r][k + 1];
      s1[r][3] = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) s2[r][k] = s2[r][k + 1];
      s2[r][4] = 0.f;
    }
  }
}

hipError_t launch_ring2_invariants(const float* x, float* rinv, int nx, int ny, int nz, int q2_sqdist,
                                   hipStream_t s) {
  // Runs of 32 planes (four more are read for their ends), shorter while the
  // planes give fewer than 3000 waves: three per SIMD of the card.
  const long txy = (long)((nx + kInv2Cols - 1) / kInv2Cols) * ((ny + kInv2Rows - 1) / kInv2Rows);
  int zc = 32;
  while (zc > 4 && txy * ((nz + zc - 1) / zc) < 3000) zc /= 2;
  const long items = txy * ((nz + zc - 1) / zc);
  if (items > 0x7fffffffL - 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_ring2_invariants, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, s, x, rinv, nx, ny, nz, zc,
                     (int)items, q2_sqdist);
  return hipGetLastError();
}

namespace r2 {
constexpr int TX = 16, TY = 4, HX = TX + 4, HY = TY + 4;
constexpr int NCELL = HX * HY;  // 160 cells per staged plane
constexpr int NHALO = NCELL - 64;  // 96 halo cells: one per lane, a second for lanes 0..31
constexpr int NBUF = 4;
// In-plane offset classes (|dx|, |dy|) sorted: (0,0) (0,1) (1,1) (0,2) (1,2) (2,2).
__host__ __device__ constexpr int cls(int a, int b) {
  return (a > b ? cls(b, a) : (b < 2 ? a + b : 3 + a));
}
static_assert(cls(0, 0) == 0 && cls(1, 0) == 1 && cls(1, 1) == 2, "classes");
static_assert(cls(2, 0) == 3 && cls(1, 2) == 4 && cls(2, 2) == 5, "classes");
// Halo cell h (0 .. 95) of the 20 x 8 staged plane: two rows above, two
// below, two columns on each side of the 16 x 4 tile.
__device__ __forceinline__ void halo_cell(int h, int& cx, int& cy) {
  if (h < 2 * HX) {
    cy = h / HX;
    cx = h - cy * HX;
  } else if (h < 4 * HX) {
    const int k = h - 2 * HX;
    cy = TY + 2 + k / HX;
    cx = k % HX;
  } else {
    const int k = h - 4 * HX;  // 0 .. 15
    cy = 2 + ((k & 7) >> 1);
    cx = (k < 8 ? 0 : TX + 2) + (k & 1);
  }
}
// f(integral_constant<int, B>) ... f(integral_constant<int, E - 1>): the
// loop index is a constant expression, so arrays indexed by values derived
// from it stay in registers.
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}
}  // namespace r2

// RUNS: tiles may hold several runs of VolDev::sc planes, whose sums are kept
// apart (as in the fused step).
template <int C, bool M2, bool STEP, bool RUNS>
__global__ __launch_bounds__(64 * kRing2Waves, 2) void k_ifcm_ring2(const LaunchArgs a) {
  static_assert(C >= 2 && C <= 4, "the fused two-ring step holds C <= 4 clusters");
  using namespace r2;
  constexpr int CP = 4, CH = C - 1, NW = kRing2Waves;
  constexpr int NV = STEP ? 2 * C + 1 : 1;
  // One spare cell takes the stores of lanes that have no cell in the volume.
  __shared__ float s_x[NW][NBUF][NCELL + 1];
  __shared__ __align__(16) float s_u[NW][NBUF][(NCELL + 1) * CP];
  // Ring invariants of the lane's voxels p-2 .. p+1.
  __shared__ __align__(16) float s_r[NW][NBUF][64 * 4];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tx = lane & (TX - 1), ty = lane / TX;
  const int own_cell = (ty + 2) * HX + (tx + 2);
  int h0x, h0y, h1x = 0, h1y = 0;
  halo_cell(lane, h0x, h0y);
  const bool has_h1 = lane + 64 < NHALO;
  if (has_h1) halo_cell(lane + 64, h1x, h1y);
  const float W1 = a.W[1], W2 = a.W[2];
  auto qw = [&](int s2) { return a.q2_sqdist ? (float)s2 : (float)(s2 * s2); };

  const int xcd = blockIdx.x & 7;
  const int it_end = a.xcd_begin[xcd + 1];
  const int it_step = (gridDim.x >> 3) * NW;
  for (int it = a.xcd_begin[xcd] + (blockIdx.x >> 3) * NW + wave; it < it_end; it += it_step) {
    const int b = vol_of_item(a, it);
    const VolDev vd = ld_const(a.vols + b);
    const int r = it - a.item_begin[b];
    const int pidx = r / vd.tiles;
    const int tile = r - pidx * vd.tiles;
    const PairDev pr = ld_const(a.pairs + b * a.P + pidx);
    const SolveState* st = pr.st;
    if (STEP && ld_const(&st->stop)) continue;
    const int t = STEP ? ld_const(&st->iter) + 1 : ld_const(&st->iter);
    const gfloat* Uin = as_global(uniform_ptr(STEP ? u_in_of(pr, t) : u_state_of(pr, t)));
    gfloat* Uout = STEP ? as_global(uniform_ptr(u_out_of(pr, t))) : nullptr;
    const gfloat* X = as_global(uniform_ptr(vd.x));
    const gfloat* RI = as_global(uniform_ptr(vd.rinv));
    float cj[C];
#pragma unroll
    for (int j = 0; j < C; ++j) cj[j] = ld_const(&st->c[(STEP ? t - 1 : t) & 1][j]);
    const float lam = ld_const(&st->lam), xi = ld_const(&st->xi);
    const int nx = vd.nx, ny = vd.ny, nz = vd.nz;
    const int txi = tile % vd.ntx;
    const int rest = tile / vd.ntx;
    const int tyi = rest % vd.nty;
    const int tzi = rest / vd.nty;
    const int x0 = txi * TX, y0 = tyi * TY;
    const int zlo = vd.zbeg + tzi * vd.zc, zhi = min(zlo + vd.zc, vd.zend);
    const int gx = x0 + tx, gy = y0 + ty;
    const bool active = gx < nx && gy < ny;
    auto in_xy = [&](int cx, int cy) {
      const int hx = x0 - 2 + cx, hy = y0 - 2 + cy;
      return hx >= 0 && hx < nx && hy >= 0 && hy < ny;
    };
    const bool v0 = in_xy(h0x, h0y), v1 = has_h1 && in_xy(h1x, h1y);
    const size_t psz = (size_t)nx * ny;
    // Lane byte offsets of the three cells within a plane of x (rows of C
    // floats are C times that); the plane's base moves in scalar registers.
    uint32_t own_ofs = active ? ((uint32_t)gy * nx + gx) * 4u : 0u;
    uint32_t h0_ofs = v0 ? ((uint32_t)(y0 - 2 + h0y) * nx + (x0 - 2 + h0x)) * 4u : 0u;
    uint32_t h1_ofs = v1 ? ((uint32_t)(y0 - 2 + h1y) * nx + (x0 - 2 + h1x)) * 4u : 0u;
    uint32_t own_ofs_u = own_ofs * C, h0_ofs_u = h0_ofs * C, h1_ofs_u = h1_ofs * C, own_ofs_r = own_ofs * 4u;
    // A cell beside the volume is 0 in every buffer from here on: its lane
    // loads the plane's first voxel and stores it in the spare cell.
    auto cell_of = [&](int cx, int cy, bool valid) __attribute__((always_inline)) {
      const int cell = cy * HX + cx;
      if (valid) return cell;
      const float zero[CP] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < NBUF; ++q) {
        s_x[wave][q][cell] = 0.f;
        lds_cell_store<CP, CP>(&s_u[wave][q][cell * CP], zero);
      }
      return NCELL;
    };
    __builtin_amdgcn_wave_barrier();
    const int own_dst = cell_of(tx + 2, ty + 2, active);
    const int h0_dst = cell_of(h0x, h0y, v0);
    const int h1_dst = has_h1 ? cell_of(h1x, h1y, v1) : NCELL;
    __builtin_amdgcn_wave_barrier();
    auto bufof = [&](int q) { return (q - zlo + 2) & (NBUF - 1); };

    // Prefetch registers of the next staged plane (own cell, two halo cells)
    // and of the lane's own intensity and ring invariants two planes ahead.
    // Planes outside the volume are read from plane 0 and not used.
    float px, pu[C], qx0, qu0[C], qx1, qu1[C];
    float ox, ri[4];
    auto load_cells = [&](int q) __attribute__((always_inline)) {
      const size_t pofs = q >= 0 && q < nz ? (size_t)q * psz : 0;
      const gfloat* Xq = opaque_base(X + pofs);
      const gfloat* Uq = opaque_base(Uin + pofs * C);
      px = *at_lane(Xq, own_ofs);
      qx0 = *at_lane(Xq, h0_ofs);
      qx1 = *at_lane(Xq, h1_ofs);
      load_row<C>(at_lane(Uq, own_ofs_u), pu);
      load_row<C>(at_lane(Uq, h0_ofs_u), qu0);
      load_row<C>(at_lane(Uq, h1_ofs_u), qu1);
    };
    auto load_own = [&](int q) __attribute__((always_inline)) {
      const size_t pofs = q >= 0 && q < nz ? (size_t)q * psz : 0;
      ox = *at_lane(opaque_base(X + pofs), own_ofs);
      load_row<4>(at_lane(opaque_base(RI + pofs * 4), own_ofs_r), ri);
    };
    auto store_cells = [&](int buf) __attribute__((always_inline)) {
      float* sx = &s_x[wave][buf][0];
      float* su = &s_u[wave][buf][0];
      sx[own_dst] = px;
      lds_cell_store<C, CP>(su + own_dst * CP, pu);
      sx[h0_dst] = qx0;
      lds_cell_store<C, CP>(su + h0_dst * CP, qu0);
      sx[h1_dst] = qx1;
      lds_cell_store<C, CP>(su + h1_dst * CP, qu1);
    };

    // Slots of the voxels p-2 .. p+2 of the lane's column: H numerators (first
    // C - 1 clusters) and F numerators of ring 1 (h1, f1; they start with slot
    // 3) and of ring 2 (h2, f2), and the centre value by ring.
    float h1[4][CH], h2[5][CH], f1[4][C], f2[5][C], xcs[5][2];
    float acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = 0.f;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      xcs[k][0] = xcs[k][1] = 0.f;
#pragma unroll
      for (int j = 0; j < C; ++j) {
        if (j < CH) h2[k][j] = 0.f;
        f2[k][j] = 0.f;
        if (k < 4 && j < CH) h1[k][j] = 0.f;
        if (k < 4) f1[k][j] = 0.f;
      }
    }

    auto finalize = [&](int z, int bz, const float (&inv)[4]) __attribute__((always_inline)) {
      const float xv = s_x[wave][bz][own_cell];
      float uo[C];
      lds_cell_load<C, CP>(&s_u[wave][bz][own_cell * CP], uo);
      const float g1 = W1 * fabsf(inv[0]), g2 = W2 * fabsf(inv[1]);
      const float q1 = W1 * inv[2], q2 = W2 * inv[3];
      float H[C], F[C];
      // A ring's ratios sum to 1 over the clusters (0 for a ring without cells).
      float rest_h = (inv[0] != 0.f ? W1 : 0.f) + (inv[1] != 0.f ? W2 : 0.f);
#pragma unroll
      for (int j = 0; j < CH; ++j) {
        H[j] = fmaf(g2, h2[0][j], g1 * h1[0][j]);
        rest_h -= H[j];
      }
      H[C - 1] = rest_h;
#pragma unroll
      for (int j = 0; j < C; ++j) F[j] = fmaf(q2, f2[0][j], q1 * f1[0][j]);
      float d2[C];
      float Jv = 0.f;
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const float av = 1.f - lam * H[j] - xi * F[j];  // eq (4) factor
        const float dd = xv - cj[j];
        d2[j] = fmaxf(dd * dd * av, kDFloor);
        Jv = fmaf(pow_m<M2>(uo[j], a.m), d2[j], Jv);  // eq (1)
      }
      Jv = active ? Jv : 0.f;
      if constexpr (STEP) {
        float un[C];
        memberships<C, M2>(d2, a.m, un);  // eq (2)
        if (active) store_row<C>(at_lane(opaque_base(Uout + (size_t)z * psz * C), own_ofs_u), un);
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const float w = active ? pow_m<M2>(un[j], a.m) : 0.f;
          acc[j] = fmaf(w, xv, acc[j]);  // eq (3)
          acc[C + j] += w;
        }
        acc[2 * C] += Jv;
      } else {
        acc[0] += Jv;
      }
    };

    // One plane p: its 5 x 5 cells added to the voxels p-2 .. p+2, the slot of
    // p+2 started, plane p+1 staged, p+2 and the own values of p+3 prefetched,
    // voxel p-2 finalised, the slots moved down.  GEN: the tile's first and last
    // planes, with the validity tests.
    auto plane = [&](int p, auto GENc) __attribute__((always_inline)) {
      constexpr bool GEN = decltype(GENc)::value;
      const bool pv = !GEN || (p >= 0 && p < nz);
      // Voxel p+2 starts from its prefetched values; its invariants take the
      // place of those of voxel p-2.
      float inv[4];
      float* const sr = &s_r[wave][bufof(p + 2)][lane * 4];
      lds_cell_load<4, 4>(sr, inv);
      __builtin_amdgcn_wave_barrier();
      lds_cell_store<4, 4>(sr, ri);
      xcs[4][0] = ri[0] < 0.f ? ox - 1.f : ox;
      xcs[4][1] = ri[1] < 0.f ? ox - 1.f : ox;
      if (!GEN || p + 3 <= zhi + 1) load_own(p + 3);
      __builtin_amdgcn_sched_barrier(0);
      if (pv) {
        const int bp = bufof(p);
        const float* sx = &s_x[wave][bp][own_cell];
        const float* su = &s_u[wave][bp][own_cell * CP];
        float cs[6][C];
        static_for<0, 5>([&](auto yc) {
          constexpr int dy = decltype(yc)::value - 2;
          static_for<0, 5>([&](auto xc) {
            constexpr int dx = decltype(xc)::value - 2;
            constexpr int ad = dx < 0 ? -dx : dx, bd = dy < 0 ? -dy : dy;
            const float xk = sx[dy * HX + dx];
            float u[C];
            lds_cell_load<C, CP>(su + (dy * HX + dx) * CP, u);
            // The first cell of a class, and of a slot, starts its sum.
            constexpr int c = cls(ad, bd);
            constexpr bool first = dy == -(ad > bd ? ad : bd) && dx == -(ad < bd ? ad : bd);
#pragma unroll
            for (int j = 0; j < C; ++j) cs[c][j] = first ? u[j] * u[j] : fmaf(u[j], u[j], cs[c][j]);
            static_for<0, 5>([&](auto kc) {
              constexpr int k = decltype(kc)::value;
              constexpr int dz = 2 - k, ed = dz < 0 ? -dz : dz;
              if constexpr (!(dx == 0 && dy == 0 && dz == 0)) {
                constexpr bool ring1 = ad <= 1 && bd <= 1 && ed <= 1;
                const float g = fabsf(xcs[k][ring1 ? 0 : 1] - xk);  // eq (6)
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                  if constexpr (ring1)
                    h1[k][j] = k == 3 && dy == -1 && dx == -1 ? u[j] * g : fmaf(u[j], g, h1[k][j]);
                  else
                    h2[k][j] = k == 4 && dy == -2 && dx == -2 ? u[j] * g : fmaf(u[j], g, h2[k][j]);
                }
              }
            });
          });
          // One row of cells at a time: keeps the row's LDS reads, not the
          // whole window's, in registers.
          __builtin_amdgcn_sched_barrier(0);
        });
        // eq (7): the class sums, weighted by the distance of the slot's plane
        // (the slots on both sides of the plane share theirs).
#pragma unroll
        for (int j = 0; j < C; ++j) {
          f1[2][j] = fmaf(qw(1), cs[1][j], f1[2][j]);
          f1[2][j] = fmaf(qw(2), cs[2][j], f1[2][j]);
          f2[2][j] = fmaf(qw(4), cs[3][j], f2[2][j]);
          f2[2][j] = fmaf(qw(5), cs[4][j], f2[2][j]);
          f2[2][j] = fmaf(qw(8), cs[5][j], f2[2][j]);
          const float n1 = fmaf(qw(3), cs[2][j], fmaf(qw(2), cs[1][j], cs[0][j]));
          const float n2 = fmaf(qw(9), cs[5][j], fmaf(qw(6), cs[4][j], qw(5) * cs[3][j]));
          f1[1][j] += n1;
          f1[3][j] = n1;
          f2[1][j] += n2;
          f2[3][j] += n2;
          float n3 = fmaf(qw(6), cs[2][j], fmaf(qw(5), cs[1][j], qw(4) * cs[0][j]));
          n3 = fmaf(qw(12), cs[5][j], fmaf(qw(9), cs[4][j], fmaf(qw(8), cs[3][j], n3)));
          f2[0][j] += n3;
          f2[4][j] = n3;
        }
      } else {
#pragma unroll
        for (int j = 0; j < C; ++j) {
          if (j < CH) h1[3][j] = h2[4][j] = 0.f;
          f1[3][j] = f2[4][j] = 0.f;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (!GEN || p + 1 <= zhi + 1) {
        store_cells(bufof(p + 1));
        if (!GEN || p + 2 <= zhi + 1) load_cells(p + 2);
      }
      if (!GEN || (p - 2 >= zlo && p - 2 < zhi)) finalize(p - 2, bufof(p - 2), inv);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        xcs[k][0] = xcs[k + 1][0];
        xcs[k][1] = xcs[k + 1][1];
#pragma unroll
        for (int j = 0; j < C; ++j) {
          if (j < CH) h2[k][j] = h2[k + 1][j];
          f2[k][j] = f2[k + 1][j];
          if (k < 3 && j < CH) h1[k][j] = h1[k + 1][j];
          if (k < 3) f1[k][j] = f1[k + 1][j];
        }
      }
    };

    using Gen = std::integral_constant<bool, true>;
    using Steady = std::integral_constant<bool, false>;

    // The sums of a finished run of sc planes go to its slot (slots are
    // numbered like tiles of sc planes); without RUNS a tile is one run.
    const int txy = vd.ntx * vd.nty;
    int slot = RUNS ? tile + tzi * (vd.zc / vd.sc - 1) * txy : tile, left = vd.sc;
    auto finished = [&](int z) __attribute__((always_inline)) {
      if (RUNS && --left > 0 && z + 1 < zhi) return;
      wave_tile_store<NV>(pr.partials, slot, vd.slots, acc);
#pragma unroll
      for (int k = 0; k < NV; ++k) acc[k] = 0.f;
      slot += txy;
      left = vd.sc;
    };

    // Prologue: plane zlo-2 staged, zlo-1 prefetched, the own values of zlo
    // (the voxel that enters at plane zlo-2) prefetched.
    load_cells(zlo - 2);
    store_cells(bufof(zlo - 2));
    load_cells(zlo - 1);
    load_own(zlo);
    int p = zlo - 2;
    for (; p < zlo + 2; ++p) plane(p, Gen{});
    // Interior planes: every per-plane test is true (the loads still clamp
    // the plane).  tests/test_plane_walk.py replays this walk.
    for (; p + 4 <= zhi; ++p) {
      plane(p, Steady{});
      if constexpr (RUNS) finished(p - 2);
    }
    for (; p <= zhi + 1; ++p) {
      plane(p, Gen{});
      if constexpr (RUNS) finished(p - 2);
    }
    if constexpr (!RUNS) finished(zhi - 1);
  }
}

template <int C, bool M2, bool RUNS>
static const void* ring2_kernel(bool step) {
  return step ? reinterpret_cast<const void*>(&k_ifcm_ring2<C, M2, true, RUNS>)
              : reinterpret_cast<const void*>(&k_ifcm_ring2<C, M2, false, RUNS>);
}
template <int C>
static const void* ring2_kernel(bool m2, bool step, bool runs) {
  if (m2) return runs ? ring2_kernel<C, true, true>(step) : ring2_kernel<C, true, false>(step);
  return runs ? ring2_kernel<C, false, true>(step) : ring2_kernel<C, false, false>(step);
}
static const void* ring2_kernel(int C, bool m2, bool step, bool runs) {
  switch (C) {
    case 2: return ring2_kernel<2>(m2, step, runs);
    case 3: return ring2_kernel<3>(m2, step, runs);
    case 4: return ring2_kernel<4>(m2, step, runs);
    default: return nullptr;
  }
}

hipError_t launch_ring2(int C, const LaunchArgs& a, int grid, bool m2, bool step, hipStream_t s) {
  const void* f = ring2_kernel(C, m2, step, a.runs != 0);
  if (!f) return hipErrorInvalidValue;
  void* args[] = {const_cast<LaunchArgs*>(&a)};
  return hipLaunchKernel(f, dim3(grid), dim3(64 * kRing2Waves), args, 0, s);
}

int ring2_occupancy(int C, bool m2, bool step, bool runs) {
  int n = 0;
  const void* f = ring2_kernel(C, m2, step, runs);
  if (!f || hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, 64 * kRing2Waves, 0) != hipSuccess) n = 1;
  return std::max(1, n);
}

}  // namespace pifcm
