// pointwise.hip -- the per-voxel kernels of libpifcm (plain FCM step for
// lambda = xi = 0, initial memberships, iteration invariants, labels,
// normalisation, checks) and the dispatchers over the cluster count.
#include "common.h"
#include "pifcm_kernels.h"

namespace pifcm {

// ------------------------------------------------ pointwise FCM (lambda=xi=0)
// With lambda = xi = 0 the attraction factor of eq (4) is exactly 1, so H and
// F are not needed and the step is plain FCM (eqs (1)-(3)).
//
// Its new memberships are then a function of x and the centres alone, so a
// run needs none of them in memory but the last: k_fcm_x forms U^(t-1) of
// iteration t from the centres it came from (c^(t-2), still in the other half
// of the pair's double buffer; only iteration 1 may read a caller's U^(0)),
// and k_fcm_last forms and stores U^(T).  An iteration reads 4 B per voxel
// where k_fcm_point moves 8 C + 4: 181x217x181 voxels, C = 4, take 14 us
// instead of 31 us, bound by VALU issue (two memberships per voxel).
// k_fcm_point remains for the adjoint, which keeps every state.
template <int C, bool M2>
__device__ __forceinline__ void fcm_memberships(float xv, const float (&c)[C], float m, float (&u)[C]) {
  float d2[C];
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const float dd = xv - c[j];
    d2[j] = fmaxf(dd * dd, kDFloor);
  }
  memberships<C, M2>(d2, m, u);
}

// Voxels in flight per thread (their loads are issued together).
constexpr int kFcmAhead = 4;
static_assert(kRunTerms % kFcmAhead == 0, "a run of sums ends between groups");

// One iteration; WJ: J of its input state is wanted (a stop rule or a
// history); LONG: a thread has more than kRunTerms voxels (the instance without
// has fewer registers: 59 against 93 at C = 16).
template <int C, bool M2, bool WJ, bool LONG>
__global__ __launch_bounds__(256) void k_fcm_x(const LaunchArgs a) {
  constexpr int NT = 256;
  constexpr int NV = 2 * C + 1;
  __shared__ float s_red[(NT / 64) * NV];
  const int xcd = blockIdx.x & 7;
  const int it_end = a.xcd_begin[xcd + 1];
  for (int it = a.xcd_begin[xcd] + (blockIdx.x >> 3); it < it_end; it += gridDim.x >> 3) {
    const int b = vol_of_item(a, it);
    const VolDev vd = ld_const(a.vols + b);
    const int r = it - a.item_begin[b];
    const int pidx = r / vd.tiles1d;
    const int tile = r - pidx * vd.tiles1d;
    const PairDev pr = ld_const(a.pairs + b * a.P + pidx);
    const SolveState* st = pr.st;
    if (ld_const(&st->stop)) continue;
    const int t = ld_const(&st->iter) + 1;
    const gfloat* X = as_global(vd.x);
    const gfloat* U0 = t == 1 && pr.U0 ? as_global(pr.U0) : nullptr;
    float c[C], cp[C];  // c^(t-1), c^(t-2) (both c^(0) at t = 1)
#pragma unroll
    for (int j = 0; j < C; ++j) {
      c[j] = ld_const(&st->c[(t - 1) & 1][j]);
      cp[j] = ld_const(&st->c[t & 1][j]);
    }
    const size_t psz = (size_t)vd.nx * vd.ny;
    const size_t N = (size_t)vd.zend * psz;  // end of the planes iterated
    RunSums<NV, LONG> sums;
    float(&acc)[NV] = sums.run;
    const size_t base = (size_t)vd.zbeg * psz + (size_t)tile * NT * vd.vpt + threadIdx.x;
    for (int k = 0; k < vd.vpt; k += kFcmAhead) {
      sums.before(k);
      float xs[kFcmAhead];
#pragma unroll
      for (int q = 0; q < kFcmAhead; ++q) xs[q] = X[min(base + (size_t)(k + q) * NT, N - 1)];
#pragma unroll
      for (int q = 0; q < kFcmAhead; ++q) {
        const size_t i = base + (size_t)(k + q) * NT;
        if (k + q >= vd.vpt || i >= N) break;
        const float xv = xs[q];
        float d2[C];
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const float dd = xv - c[j];
          d2[j] = fmaxf(dd * dd, kDFloor);
        }
        if constexpr (WJ) {
          float uo[C];
          if (U0) load_row<C>(U0 + i * C, uo);
          else fcm_memberships<C, M2>(xv, cp, a.m, uo);
          float Jv = 0.f;
#pragma unroll
          for (int j = 0; j < C; ++j) Jv = fmaf(pow_m<M2>(uo[j], a.m), d2[j], Jv);
          acc[2 * C] += Jv;
        }
        float un[C];
        memberships<C, M2>(d2, a.m, un);
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const float w = pow_m<M2>(un[j], a.m);
          acc[j] = fmaf(w, xv, acc[j]);
          acc[C + j] += w;
        }
      }
    }
    block_tile_store<NV, NT>(pr.partials, tile, vd.tiles1d, sums.total(), s_red);
  }
}

// The final state: U^(T) into pr.Ua (if not NULL) and its objective.  With
// a.fcm_sorted the columns are stored in the order of their centres (ties by
// index).
template <int C, bool M2>
__global__ __launch_bounds__(256) void k_fcm_last(const LaunchArgs a) {
  constexpr int NT = 256;
  __shared__ float s_red[NT / 64];
  const int xcd = blockIdx.x & 7;
  const int it_end = a.xcd_begin[xcd + 1];
  for (int it = a.xcd_begin[xcd] + (blockIdx.x >> 3); it < it_end; it += gridDim.x >> 3) {
    const int b = vol_of_item(a, it);
    const VolDev vd = ld_const(a.vols + b);
    const int r = it - a.item_begin[b];
    const int pidx = r / vd.tiles1d;
    const int tile = r - pidx * vd.tiles1d;
    const PairDev pr = ld_const(a.pairs + b * a.P + pidx);
    const SolveState* st = pr.st;
    const int T = ld_const(&st->iter);
    const gfloat* X = as_global(vd.x);
    const gfloat* U0 = T == 0 && pr.U0 ? as_global(pr.U0) : nullptr;
    gfloat* out = as_global(pr.Ua);
    float c[C], cp[C];  // c^(T), c^(T-1)
    int col[C];         // column of cluster j in the stored rows
    bool moved = false;
#pragma unroll
    for (int j = 0; j < C; ++j) {
      c[j] = ld_const(&st->c[T & 1][j]);
      cp[j] = ld_const(&st->c[T == 0 ? 0 : (T - 1) & 1][j]);
    }
#pragma unroll
    for (int j = 0; j < C; ++j) {
      col[j] = 0;
#pragma unroll
      for (int k = 0; k < C; ++k) col[j] += c[k] < c[j] || (c[k] == c[j] && k < j) ? 1 : 0;
      moved = moved || (a.fcm_sorted && col[j] != j);
    }
    const size_t psz = (size_t)vd.nx * vd.ny;
    const size_t N = (size_t)vd.zend * psz;
    RunSums<1, true> sums;
    float(&acc)[1] = sums.run;
    const size_t base = (size_t)vd.zbeg * psz + (size_t)tile * NT * vd.vpt + threadIdx.x;
    for (int k = 0; k < vd.vpt; k += kFcmAhead) {
      sums.before(k);
      float xs[kFcmAhead];
#pragma unroll
      for (int q = 0; q < kFcmAhead; ++q) xs[q] = X[min(base + (size_t)(k + q) * NT, N - 1)];
#pragma unroll
      for (int q = 0; q < kFcmAhead; ++q) {
        const size_t i = base + (size_t)(k + q) * NT;
        if (k + q >= vd.vpt || i >= N) break;
        const float xv = xs[q];
        float u[C];
        if (U0) load_row<C>(U0 + i * C, u);
        else fcm_memberships<C, M2>(xv, cp, a.m, u);
        float Jv = 0.f;
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const float dd = xv - c[j];
          Jv = fmaf(pow_m<M2>(u[j], a.m), fmaxf(dd * dd, kDFloor), Jv);
        }
        acc[0] += Jv;
        if (out) {
          if (moved) {
            float v[C];
#pragma unroll
            for (int p = 0; p < C; ++p) {
              v[p] = 0.f;
#pragma unroll
              for (int j = 0; j < C; ++j) v[p] = col[j] == p ? u[j] : v[p];
            }
            store_row<C>(out + i * C, v);
          } else {
            store_row<C>(out + i * C, u);
          }
        }
      }
    }
    block_tile_store<1, NT>(pr.partials, tile, vd.tiles1d, sums.total(), s_red);
  }
}

template <int C, bool M2, bool STEP>
__global__ __launch_bounds__(256) void k_fcm_point(const LaunchArgs a) {
  constexpr int NT = 256;
  constexpr int NV = STEP ? 2 * C + 1 : 1;
  __shared__ float s_red[(NT / 64) * NV];
  const int xcd = blockIdx.x & 7;
  const int it_end = a.xcd_begin[xcd + 1];
  for (int it = a.xcd_begin[xcd] + (blockIdx.x >> 3); it < it_end; it += gridDim.x >> 3) {
    const int b = vol_of_item(a, it);
    const VolDev vd = ld_const(a.vols + b);
    const int r = it - a.item_begin[b];
    const int pidx = r / vd.tiles1d;
    const int tile = r - pidx * vd.tiles1d;
    const PairDev pr = ld_const(a.pairs + b * a.P + pidx);
    const SolveState* st = pr.st;
    if (STEP && ld_const(&st->stop)) continue;
    const int t = STEP ? ld_const(&st->iter) + 1 : ld_const(&st->iter);
    const gfloat* Uin = as_global(STEP ? u_in_of(pr, t) : u_state_of(pr, t));
    gfloat* Uout = STEP ? as_global(u_out_of(pr, t)) : nullptr;
    const gfloat* X = as_global(vd.x);
    float cj[C];
#pragma unroll
    for (int j = 0; j < C; ++j) cj[j] = ld_const(&st->c[(STEP ? t - 1 : t) & 1][j]);
    const size_t psz = (size_t)vd.nx * vd.ny;
    const size_t N = (size_t)vd.zend * psz;  // end of the planes iterated
    RunSums<NV, true> sums;
    float(&acc)[NV] = sums.run;
    const size_t base = (size_t)vd.zbeg * psz + (size_t)tile * NT * vd.vpt;
#pragma unroll 2
    for (int k = 0; k < vd.vpt; ++k) {
      const size_t i = base + (size_t)k * NT + threadIdx.x;
      if (i >= N) break;
      sums.before(k);
      const float xv = X[i];
      float uo[C], d2[C];
      load_row<C>(Uin + i * C, uo);
      float Jv = 0.f;
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const float dd = xv - cj[j];
        d2[j] = fmaxf(dd * dd, kDFloor);
        Jv = fmaf(pow_m<M2>(uo[j], a.m), d2[j], Jv);
      }
      if constexpr (STEP) {
        float un[C];
        memberships<C, M2>(d2, a.m, un);
        store_row<C>(Uout + i * C, un);
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const float w = pow_m<M2>(un[j], a.m);
          acc[j] = fmaf(w, xv, acc[j]);
          acc[C + j] += w;
        }
        acc[2 * C] += Jv;
      } else {
        acc[0] += Jv;
      }
    }
    block_tile_store<NV, NT>(pr.partials, tile, vd.tiles1d, sums.total(), s_red);
  }
}

// ----------------------------------------------------------- small kernels
// Iteration invariants of one volume: g_inv = 1 / sum_k |x_i - x_k| over the
// in-volume 3x3x3 neighbourhood (denominator of eq (5)); for a voxel whose
// neighbours all have its intensity, -1 / (number of neighbours), which the
// fused step turns into the equal-weight mean; 0 for a voxel without
// neighbours.  Also flags non-finite intensities.
//
// A wave owns kInvCols x kInvRows columns of a run of zc planes and walks it
// along z.  Lane l holds column x0 - 1 + l, so the wave's two outer lanes are
// halo and every cell is loaded once per wave row: a lane's left and right
// neighbours come from the lanes beside it (DPP wave shifts), the rows above
// and below from its own registers, and each plane serves the voxels of three
// planes.  Cells outside the volume are loaded from a clamped address and
// weighted 0.  Every voxel's terms are added in the order dz, dy, dx.
// Bound by VALU issue (26 differences and sums per voxel, an IEEE division):
// 29 us for 181x217x181 voxels (57 MB), where one thread per voxel reading its
// 26 neighbours through the caches with a test each took 108 us.
constexpr int kInvCols = 62, kInvRows = 4;

__global__ __launch_bounds__(256) void k_invariants(const float* __restrict__ x, float* __restrict__ invg,
                                                    int nx, int ny, int nz, int zbeg, int zend, int zc,
                                                    int nitems, int* __restrict__ flag) {
  constexpr int R = kInvRows;
  const int lane = threadIdx.x & 63;
  const int item = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (item >= nitems) return;
  const int ntx = (nx + kInvCols - 1) / kInvCols, nty = (ny + R - 1) / R;
  const int gx = (item % ntx) * kInvCols + lane - 1, y0 = (item / ntx) % nty * R;
  const int zlo = zbeg + item / ntx / nty * zc, zhi = min(zlo + zc, zend);
  const bool own = lane >= 1 && lane <= kInvCols && gx < nx;
  const int cx = min(max(gx, 0), nx - 1);
  // Weights (0 or 1) of the cells left of, at and right of the lane's column,
  // by row: rows y0 - 1 .. y0 + R.
  const float mL = gx > 0 ? 1.f : 0.f, mR = gx < nx - 1 ? 1.f : 0.f;
  float wL[R + 2], wC[R + 2], wR[R + 2];
  uint32_t ofs[R + 2];
#pragma unroll
  for (int r = 0; r < R + 2; ++r) {
    const int gy = y0 - 1 + r;
    wC[r] = gy >= 0 && gy < ny ? 1.f : 0.f;
    wL[r] = mL * wC[r];
    wR[r] = mR * wC[r];
    ofs[r] = ((uint32_t)min(max(gy, 0), ny - 1) * (uint32_t)nx + (uint32_t)cx) * 4u;
  }
  const size_t psz = (size_t)nx * ny;
  auto load = [&](int p, float (&v)[R + 2]) __attribute__((always_inline)) {
    const gfloat* base = opaque_base(as_global(x) + (size_t)min(max(p, 0), nz - 1) * psz);
#pragma unroll
    for (int r = 0; r < R + 2; ++r) v[r] = *at_lane(base, ofs[r]);
  };
  const int nxy = 1 + (gx > 0) + (gx < nx - 1);
  bool bad = false;
  float prev[R + 2], cur[R + 2], next[R + 2], ahead[R + 2];
  float sa[R], sb[R], sc[R];  // sums of voxels p - 1, p, p + 1 of each row
#pragma unroll
  for (int r = 0; r < R + 2; ++r) prev[r] = 0.f;
#pragma unroll
  for (int r = 0; r < R; ++r) sa[r] = sb[r] = sc[r] = 0.f;
  load(zlo - 1, cur);
  load(zlo, next);
  for (int p = zlo - 1; p <= zhi; ++p) {
    load(p + 2, ahead);
    if (p >= 0 && p < nz) {
      float le[R + 2], ri[R + 2];
#pragma unroll
      for (int r = 0; r < R + 2; ++r) {
        le[r] = from_left_lane(cur[r]);
        ri[r] = from_right_lane(cur[r]);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float c = 0.f;
#pragma unroll
        for (int d = 0; d < 3; ++d) {  // rows y - 1, y, y + 1
          const float va = prev[r + 1], vb = cur[r + 1], vc = next[r + 1];
          sa[r] = fmaf(fabsf(va - le[r + d]), wL[r + d], sa[r]);
          sa[r] = fmaf(fabsf(va - cur[r + d]), wC[r + d], sa[r]);
          sa[r] = fmaf(fabsf(va - ri[r + d]), wR[r + d], sa[r]);
          sb[r] = fmaf(fabsf(vb - le[r + d]), wL[r + d], sb[r]);
          if (d != 1) sb[r] = fmaf(fabsf(vb - cur[r + d]), wC[r + d], sb[r]);
          sb[r] = fmaf(fabsf(vb - ri[r + d]), wR[r + d], sb[r]);
          c = fmaf(fabsf(vc - le[r + d]), wL[r + d], c);
          c = fmaf(fabsf(vc - cur[r + d]), wC[r + d], c);
          c = fmaf(fabsf(vc - ri[r + d]), wR[r + d], c);
        }
        sc[r] = c;
      }
    }
    const int z = p - 1;
    if (z >= zlo) {
      gfloat* out = opaque_base(as_global(invg) + (size_t)z * psz);
      const int nzv = 1 + (z > 0) + (z < nz - 1);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int gy = y0 + r;
        if (own && gy < ny) {
          bad = bad || !isfinite(prev[r + 1]);
          const int cnt = nxy * (1 + (gy > 0) + (gy < ny - 1)) * nzv - 1;
          *at_lane(out, ofs[r + 1]) = sa[r] > 0.f ? 1.f / sa[r] : (cnt > 0 ? -1.f / (float)cnt : 0.f);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < R + 2; ++r) {
      prev[r] = cur[r];
      cur[r] = next[r];
      next[r] = ahead[r];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      sa[r] = sb[r];
      sb[r] = sc[r];
      sc[r] = 0.f;
    }
  }
  if (bad) atomicOr(flag, 1);
}

// Elements before the first 16-byte boundary of p (at most n).
__device__ __forceinline__ size_t head_of(const float* p, size_t n) {
  return min(n, (size_t)((16 - (reinterpret_cast<uintptr_t>(p) & 15)) & 15) / 4);
}

// U^(0) from centres (eq (2) with the attraction factor 1).
template <int C, bool M2>
__global__ __launch_bounds__(256) void k_init_u(const float* __restrict__ x, size_t N,
                                                const SolveState* __restrict__ st, float m,
                                                float* __restrict__ U) {
  float cj[C];
#pragma unroll
  for (int j = 0; j < C; ++j) cj[j] = st->c[0][j];
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (size_t)gridDim.x * blockDim.x) {
    const float xv = x[i];
    float d2[C], u[C];
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const float dd = xv - cj[j];
      d2[j] = fmaxf(dd * dd, kDFloor);
    }
    memberships<C, M2>(d2, m, u);
    store_row<C>(as_global(U) + i * C, u);
  }
}

// Flags a non-finite intensity (calls that do not need g_inv).  The float4s
// of the 16-byte aligned body, and the few values around it.
__global__ __launch_bounds__(256) void k_check_finite(const float* __restrict__ x, size_t n,
                                                      int* __restrict__ flag) {
  const size_t head = head_of(x, n), n4 = (n - head) / 4;
  const float4* body = reinterpret_cast<const float4*>(x + head);
  const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
  bool bad = false;
#pragma unroll 4
  for (size_t i = tid; i < n4; i += stride) {
    const float4 v = body[i];
    bad = bad || !isfinite(v.x) || !isfinite(v.y) || !isfinite(v.z) || !isfinite(v.w);
  }
  if (tid < head) bad = bad || !isfinite(x[tid]);
  const size_t i = head + 4 * n4 + tid;
  if (i < n) bad = bad || !isfinite(x[i]);
  if (bad) atomicOr(flag, 1);
}

// Rows of a caller's U must be memberships: finite, in [0, 1], sum 1 +- 1e-4.
template <int C>
__device__ __forceinline__ bool row_ok(const float (&u)[C]) {
  float s = 0.f;
  bool ok = true;
#pragma unroll
  for (int j = 0; j < C; ++j) {
    ok = ok && isfinite(u[j]) && u[j] >= 0.f && u[j] <= 1.f + 1e-6f;
    s += u[j];
  }
  return ok && !(fabsf(s - 1.f) > 1e-4f);
}
// argmax_j u_j, ties to the lowest j.
template <int C>
__device__ __forceinline__ uint8_t row_label(const float (&u)[C]) {
  int best = 0;
  float bv = u[0];
#pragma unroll
  for (int j = 1; j < C; ++j) {
    if (u[j] > bv) {
      bv = u[j];
      best = j;
    }
  }
  return (uint8_t)best;
}

// One row per thread, read as wide as its alignment allows.  HBM bound: 7.1 M
// rows of 4 in 19 us (5.9 TB/s), 4.1 M rows of 8 in 25 us; a loop over C
// known at run time, a dword at a time, took 39 and 72 us.
template <int C>
__global__ __launch_bounds__(256) void k_check_rows(const float* __restrict__ U, size_t N,
                                                    int* __restrict__ flag) {
  bool bad = false;
#pragma unroll 2
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (size_t)gridDim.x * blockDim.x) {
    float u[C];
    load_row<C>(as_global(U) + i * C, u);
    bad = bad || !row_ok<C>(u);
  }
  if (bad) atomicOr(flag, 1);
}

// Labels (7.1 M rows of 4 in 30 us, 41 us with a run-time C).
template <int C>
__global__ __launch_bounds__(256) void k_labels(const float* __restrict__ U, size_t N,
                                                uint8_t* __restrict__ out) {
#pragma unroll 2
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (size_t)gridDim.x * blockDim.x) {
    float u[C];
    load_row<C>(as_global(U) + i * C, u);
    out[i] = row_label<C>(u);
  }
}

// The context of a slab solve in one pass over the caller's memberships: the
// row check, the copy into the output and (labels not NULL) the labels; the
// slab's own planes are written again by the solve.  7.1 M rows of 4: 35 us,
// the bytes of the copy alone, instead of 19 + 45 + 30 us in three passes.
template <int C>
__global__ __launch_bounds__(256) void k_context(const float* __restrict__ U, size_t N, float* __restrict__ out,
                                                 uint8_t* __restrict__ labels, int* __restrict__ flag) {
  bool bad = false;
#pragma unroll 2
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (size_t)gridDim.x * blockDim.x) {
    float u[C];
    load_row<C>(as_global(U) + i * C, u);
    bad = bad || !row_ok<C>(u);
    store_row<C>(as_global(out) + i * C, u);
    if (labels) labels[i] = row_label<C>(u);
  }
  if (bad) atomicOr(flag, 1);
}

// Confusion counts of labels (0..C-1) against reference classes (0..K-1):
// counts[j * K + k] += #{i : labels_i = j, truth_i = k}; pairs outside the
// ranges go to counts[C * K].  Per-block LDS histogram, then one atomic add
// per bin (integer sums: the result does not depend on the order).
__global__ __launch_bounds__(256) void k_confusion(const uint8_t* __restrict__ labels,
                                                   const uint8_t* __restrict__ truth, size_t N,
                                                   int C, int K, unsigned long long* counts) {
  __shared__ uint32_t h[kMaxC * kMaxC + 1];
  const int nb = C * K + 1;
  for (int t = threadIdx.x; t < nb; t += blockDim.x) h[t] = 0u;
  __syncthreads();
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (size_t)gridDim.x * blockDim.x) {
    const int j = labels[i], k = truth[i];
    atomicAdd(&h[(j < C && k < K) ? j * K + k : C * K], 1u);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < nb; t += blockDim.x)
    if (h[t]) atomicAdd(&counts[t], (unsigned long long)h[t]);
}

// Min-max normalisation (Algorithm 2 step 1).  Floats are mapped to
// order-preserving unsigned keys so min/max are exact integer atomics.
__device__ __forceinline__ uint32_t fkey(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float kinv(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
// Few, large work groups: each ends in two atomics on the same two words,
// which are served one after the other.  7.1 M values in 12.7 us (28 us with
// 1024 work groups of 256 threads and dword loads).
constexpr int kMinmaxThreads = 1024;
__global__ __launch_bounds__(kMinmaxThreads) void k_minmax(const float* __restrict__ raw, size_t n,
                                                           NormSlot* __restrict__ slot, int* __restrict__ seen) {
  uint32_t lo = 0xffffffffu, hi = 0u;
  bool bad = false;
  auto take = [&](float v) {
    bad = bad || !isfinite(v);
    const uint32_t k = fkey(v);
    lo = min(lo, k);
    hi = max(hi, k);
  };
  // The 16-byte aligned body as float4s, four in flight per thread; the few
  // elements before and after it one each by the first work group.
  const size_t head = head_of(raw, n), n4 = (n - head) / 4;
  const float4* body = reinterpret_cast<const float4*>(raw + head);
  const size_t stride = (size_t)gridDim.x * kMinmaxThreads;
#pragma unroll 4
  for (size_t i = (size_t)blockIdx.x * kMinmaxThreads + threadIdx.x; i < n4; i += stride) {
    const float4 v = body[i];
    take(v.x);
    take(v.y);
    take(v.z);
    take(v.w);
  }
  if (blockIdx.x == 0) {
    if (threadIdx.x < head) take(raw[threadIdx.x]);
    const size_t i = head + 4 * n4 + threadIdx.x;
    if (i < n) take(raw[i]);
  }
  // Wave, then work group, then one atomic per work group and key (min and
  // max of the keys do not depend on the order).
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
  }
  constexpr int NW = kMinmaxThreads / 64;
  __shared__ uint32_t s_lo[NW], s_hi[NW];
  const int any_bad = __syncthreads_or(bad ? 1 : 0);
  if ((threadIdx.x & 63) == 0) {
    s_lo[threadIdx.x >> 6] = lo;
    s_hi[threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NW; ++w) {
      lo = min(lo, s_lo[w]);
      hi = max(hi, s_hi[w]);
    }
    atomicMin(&slot->lo, lo);
    atomicMax(&slot->hi, hi);
    if (any_bad) {
      atomicOr(&slot->bad, 1);
      __hip_atomic_store(seen, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

// One thread scales four elements (float4s where raw and out sit alike on
// 16-byte boundaries); raw and out may be the same array.  HBM bound: 7.1 M
// values in 11 us (5.1 TB/s; 15 us with dwords).  Leaves out alone if a value is
// not finite, and presets the slot of the next call.
__global__ __launch_bounds__(256) void k_normalize(const float* raw, size_t n,
                                                   const NormSlot* __restrict__ slot, NormSlot* __restrict__ next,
                                                   float* out) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *next = NormSlot{0xffffffffu, 0u, 0, 0};
  if (slot->bad) return;
  const double mn = (double)kinv(slot->lo), mx = (double)kinv(slot->hi);
  const bool flat = mx == mn;
  auto scale = [&](float v) { return flat ? 0.f : (float)(((double)v - mn) / (mx - mn)); };
  const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
  if (((reinterpret_cast<uintptr_t>(raw) ^ reinterpret_cast<uintptr_t>(out)) & 15) == 0) {
    const size_t head = head_of(raw, n), n4 = (n - head) / 4;
    const float4* in4 = reinterpret_cast<const float4*>(raw + head);
    float4* out4 = reinterpret_cast<float4*>(out + head);
    for (size_t i = tid; i < n4; i += stride) {
      const float4 v = in4[i];
      out4[i] = make_float4(scale(v.x), scale(v.y), scale(v.z), scale(v.w));
    }
    if (tid < head) out[tid] = scale(raw[tid]);
    const size_t i = head + 4 * n4 + tid;
    if (i < n) out[i] = scale(raw[i]);
  } else {
    for (size_t i = tid; i < n; i += stride) out[i] = scale(raw[i]);
  }
}

// ------------------------------------------------------------- dispatchers
template <int C, bool LONG>
static const void* fcm_x_kernel(bool m2, bool want_j) {
  if (want_j) return m2 ? reinterpret_cast<const void*>(&k_fcm_x<C, true, true, LONG>)
                        : reinterpret_cast<const void*>(&k_fcm_x<C, false, true, LONG>);
  return m2 ? reinterpret_cast<const void*>(&k_fcm_x<C, true, false, LONG>)
            : reinterpret_cast<const void*>(&k_fcm_x<C, false, false, LONG>);
}

template <int C>
static const void* fcm_x_kernel(bool m2, bool step, bool want_j, bool longer) {
  if (!step) return m2 ? reinterpret_cast<const void*>(&k_fcm_last<C, true>)
                       : reinterpret_cast<const void*>(&k_fcm_last<C, false>);
  return longer ? fcm_x_kernel<C, true>(m2, want_j) : fcm_x_kernel<C, false>(m2, want_j);
}

template <int C>
static hipError_t launch_fcm_x_c(const LaunchArgs& a, int grid, bool m2, bool step, hipStream_t s) {
  void* args[] = {const_cast<LaunchArgs*>(&a)};
  return hipLaunchKernel(fcm_x_kernel<C>(m2, step, a.want_j != 0, a.max_vpt > kRunTerms), dim3(grid), dim3(256), args,
                         0, s);
}

template <int C>
static hipError_t launch_fcm_c(const LaunchArgs& a, int grid, bool m2, bool step, hipStream_t s) {
  if (m2) {
    if (step) hipLaunchKernelGGL((k_fcm_point<C, true, true>), dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_fcm_point<C, true, false>), dim3(grid), dim3(256), 0, s, a);
  } else {
    if (step) hipLaunchKernelGGL((k_fcm_point<C, false, true>), dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_fcm_point<C, false, false>), dim3(grid), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

template <int C, int NT>
static hipError_t launch_finalize_ct(const LaunchArgs& a, int npairs, bool step, hipStream_t s) {
  if (step) hipLaunchKernelGGL((k_finalize<C, true, NT>), dim3(npairs), dim3(NT), 0, s, a);
  else hipLaunchKernelGGL((k_finalize<C, false, NT>), dim3(npairs), dim3(NT), 0, s, a);
  return hipGetLastError();
}

template <int C>
static hipError_t launch_finalize_c(const LaunchArgs& a, int npairs, bool step, hipStream_t s) {
  return a.max_slots <= 256 ? launch_finalize_ct<C, 256>(a, npairs, step, s)
                            : launch_finalize_ct<C, 1024>(a, npairs, step, s);
}

template <int C>
static hipError_t launch_init_c(const float* x, size_t N, const SolveState* st, float m, bool m2,
                                float* U, hipStream_t s) {
  const int grid = (int)std::min<size_t>((N + 255) / 256, 65536);
  if (m2) hipLaunchKernelGGL((k_init_u<C, true>), dim3(grid), dim3(256), 0, s, x, N, st, m, U);
  else hipLaunchKernelGGL((k_init_u<C, false>), dim3(grid), dim3(256), 0, s, x, N, st, m, U);
  return hipGetLastError();
}

#define PIFCM_FOR_EACH_C(X) \
  X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

#define DECL(c)                                                                              \
  hipError_t launch_gather_C##c(const LaunchArgs& a, int grid, int ty, bool m2, bool step, \
                                hipStream_t s);                                            \
  int occ_gather_C##c(int ty, int pt, bool m2, bool step, bool runs);
PIFCM_FOR_EACH_C(DECL)
#undef DECL

hipError_t launch_gather(int C, const LaunchArgs& a, int grid, int ty, bool m2, bool step,
                         hipStream_t s) {
  switch (C) {
#define CASE(c) \
  case c: return launch_gather_C##c(a, grid, ty, m2, step, s);
    PIFCM_FOR_EACH_C(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
}

int gather_occupancy(int C, int ty, int pt, bool m2, bool step, bool runs) {
  switch (C) {
#define CASE(c) \
  case c: return occ_gather_C##c(ty, pt, m2, step, runs);
    PIFCM_FOR_EACH_C(CASE)
#undef CASE
    default: return 1;
  }
}

hipError_t launch_fcm(int C, const LaunchArgs& a, int grid, bool m2, bool step, hipStream_t s) {
  switch (C) {
#define CASE(c) \
  case c: return launch_fcm_c<c>(a, grid, m2, step, s);
    PIFCM_FOR_EACH_C(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_fcm_x(int C, const LaunchArgs& a, int grid, bool m2, bool step, hipStream_t s) {
  switch (C) {
#define CASE(c) \
  case c: return launch_fcm_x_c<c>(a, grid, m2, step, s);
    PIFCM_FOR_EACH_C(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_finalize(int C, const LaunchArgs& a, int npairs, bool step, hipStream_t s) {
  switch (C) {
#define CASE(c) \
  case c: return launch_finalize_c<c>(a, npairs, step, s);
    PIFCM_FOR_EACH_C(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_init_u(int C, const float* x, size_t N, const SolveState* st, float m, bool m2,
                         float* U, hipStream_t s) {
  switch (C) {
#define CASE(c) \
  case c: return launch_init_c<c>(x, N, st, m, m2, U, s);
    PIFCM_FOR_EACH_C(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
}

static int small_grid(size_t n) { return (int)std::max<size_t>(1, std::min<size_t>((n + 255) / 256, 65536)); }

hipError_t launch_invariants(const float* x, float* invg, int nx, int ny, int nz, int zbeg, int zend,
                             int* flag, hipStream_t s) {
  // Runs of 16 planes (two more are read for their ends), shorter while the
  // planes give fewer than 3000 waves: three per SIMD of the card.
  const long txy = (long)((nx + kInvCols - 1) / kInvCols) * ((ny + kInvRows - 1) / kInvRows);
  const int np = zend - zbeg;
  int zc = 16;
  while (zc > 2 && txy * ((np + zc - 1) / zc) < 3000) zc /= 2;
  const long items = txy * ((np + zc - 1) / zc);
  if (items > 0x7fffffffL - 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_invariants, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, s, x, invg, nx, ny, nz, zbeg,
                     zend, zc, (int)items, flag);
  return hipGetLastError();
}

// Rows a work group of 256 threads takes: one per thread, two from 2^20 rows on:
// there half the work groups still hold 8 waves for every SIMD, and a thread
// has two loads in flight.
static int row_grid(size_t n) {
  const size_t per = n >= ((size_t)1 << 20) ? 512 : 256;
  return (int)std::max<size_t>(1, std::min<size_t>((n + per - 1) / per, 65536));
}

template <int C>
static hipError_t launch_check_c(const float* U, size_t N, int* flag, hipStream_t s) {
  hipLaunchKernelGGL((k_check_rows<C>), dim3(row_grid(N)), dim3(256), 0, s, U, N, flag);
  return hipGetLastError();
}

hipError_t launch_check_finite(const float* x, size_t n, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_check_finite, dim3(std::min(small_grid((n + 15) / 16), 2048)), dim3(256), 0, s, x, n, flag);
  return hipGetLastError();
}

hipError_t launch_check_rows(const float* U, size_t N, int C, int* flag, hipStream_t s) {
  switch (C) {
#define CASE(c) \
  case c: return launch_check_c<c>(U, N, flag, s);
    PIFCM_FOR_EACH_C(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
}

template <int C>
static hipError_t launch_labels_c(const float* U, size_t N, uint8_t* out, hipStream_t s) {
  hipLaunchKernelGGL((k_labels<C>), dim3(row_grid(N)), dim3(256), 0, s, U, N, out);
  return hipGetLastError();
}

hipError_t launch_labels(const float* U, size_t N, int C, uint8_t* out, hipStream_t s) {
  switch (C) {
#define CASE(c) \
  case c: return launch_labels_c<c>(U, N, out, s);
    PIFCM_FOR_EACH_C(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
}

template <int C>
static hipError_t launch_context_c(const float* U, size_t N, float* out, uint8_t* labels, int* flag,
                                   hipStream_t s) {
  hipLaunchKernelGGL((k_context<C>), dim3(row_grid(N)), dim3(256), 0, s, U, N, out, labels, flag);
  return hipGetLastError();
}

hipError_t launch_context(const float* U, size_t N, int C, float* out, uint8_t* labels, int* flag,
                          hipStream_t s) {
  switch (C) {
#define CASE(c) \
  case c: return launch_context_c<c>(U, N, out, labels, flag, s);
    PIFCM_FOR_EACH_C(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_confusion(const uint8_t* labels, const uint8_t* truth, size_t N, int C, int K,
                            unsigned long long* counts, hipStream_t s) {
  hipLaunchKernelGGL(k_confusion, dim3(small_grid(N)), dim3(256), 0, s, labels, truth, N, C, K, counts);
  return hipGetLastError();
}

hipError_t launch_minmax(const float* raw, size_t n, NormSlot* slot, int* seen, hipStream_t s) {
  // At most one work group per CU (256 on the card), each thread four float4s
  // or more.
  const size_t per = (size_t)kMinmaxThreads * 16;
  const int g = (int)std::max<size_t>(1, std::min<size_t>((n + per - 1) / per, 256));
  hipLaunchKernelGGL(k_minmax, dim3(g), dim3(kMinmaxThreads), 0, s, raw, n, slot, seen);
  return hipGetLastError();
}

hipError_t launch_scale(const float* raw, size_t n, const NormSlot* slot, NormSlot* next, float* out,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_normalize, dim3(small_grid((n + 3) / 4)), dim3(256), 0, s, raw, n, slot, next, out);
  return hipGetLastError();
}

template <int C>
static int occ_fcm_x_c(bool m2, bool step, bool longer) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fcm_x_kernel<C>(m2, step, true, longer), 256,
                                                   0) != hipSuccess) n = 1;
  return std::max(n, 1);
}

int fcm_x_occupancy(int C, bool m2, bool step, bool longer) {
  switch (C) {
#define CASE(c) \
  case c: return occ_fcm_x_c<c>(m2, step, longer);
    PIFCM_FOR_EACH_C(CASE)
#undef CASE
    default: return 1;
  }
}

template <int C>
static int occ_fcm_c(bool m2, bool step) {
  int n = 0;
  const void* f;
  if (m2) f = step ? reinterpret_cast<const void*>(&k_fcm_point<C, true, true>)
                   : reinterpret_cast<const void*>(&k_fcm_point<C, true, false>);
  else f = step ? reinterpret_cast<const void*>(&k_fcm_point<C, false, true>)
                : reinterpret_cast<const void*>(&k_fcm_point<C, false, false>);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, 256, 0) != hipSuccess) n = 1;
  return std::max(n, 1);
}

int fcm_occupancy(int C, bool m2, bool step) {
  switch (C) {
#define CASE(c) \
  case c: return occ_fcm_c<c>(m2, step);
    PIFCM_FOR_EACH_C(CASE)
#undef CASE
    default: return 1;
  }
}

}  // namespace pifcm
