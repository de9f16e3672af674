// common.h -- device helpers shared by the kernels of libpifcm.
#pragma once
#include <algorithm>
#include <type_traits>

#include "pifcm_device.h"

namespace pifcm {

// Global-memory views of pointers read from descriptor tables: loads and
// stores through them are global (not flat) instructions.
typedef __attribute__((address_space(1))) float gfloat;
__device__ __forceinline__ const gfloat* as_global(const float* p) { return (const gfloat*)p; }
__device__ __forceinline__ gfloat* as_global(float* p) { return (gfloat*)p; }

// base + a 32-bit byte offset: with a uniform base this is the scalar-base
// plus vector-offset form of the global instructions (no 64-bit address math).
__device__ __forceinline__ const gfloat* at_byte(const gfloat* base, uint32_t off) {
  return (const gfloat*)((const __attribute__((address_space(1))) char*)base + off);
}
__device__ __forceinline__ gfloat* at_byte(gfloat* base, uint32_t off) {
  return (gfloat*)((__attribute__((address_space(1))) char*)base + off);
}

// Read-only descriptor data (tables, particle state) through the constant
// address space: uniform reads become scalar loads.
template <typename T>
__device__ __forceinline__ T ld_const(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "word-sized descriptors only");
  typedef const __attribute__((address_space(4))) uint32_t CW;
  T out;
  uint32_t* o = reinterpret_cast<uint32_t*>(&out);
  CW* q = (CW*)p;
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; ++i) o[i] = q[i];
  return out;
}

typedef float f4v __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float frcp(float v) { return __builtin_amdgcn_rcpf(v); }

// A pointer that is the same in every lane, pinned to scalar registers (a
// select of descriptor fields can otherwise leave it in vector registers, to
// be read back before every memory instruction that uses it as a base).
template <typename T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<T*>(((uint64_t)hi << 32) | lo);
}

// A uniform base the optimiser may not re-associate with a lane offset: kept
// in scalar registers, so base + 32-bit lane offset stays one memory
// instruction with no vector address arithmetic.
template <typename T>
__device__ __forceinline__ T* opaque_base(T* p) {
  asm("" : "+s"(p));
  return p;
}
// base + a lane offset held in a variable that is redefined (in place, no
// code) at each use: its widening then stays next to the access instead of
// being hoisted out of the loop as a 64-bit vector address.
__device__ __forceinline__ const gfloat* at_lane(const gfloat* base, uint32_t& off) {
  asm("" : "+v"(off));
  return at_byte(base, off);
}
__device__ __forceinline__ gfloat* at_lane(gfloat* base, uint32_t& off) {
  asm("" : "+v"(off));
  return at_byte(base, off);
}

// The value of the lane before / after (0 past the wave's ends).
__device__ __forceinline__ float from_left_lane(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_right_lane(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));
}

__device__ __forceinline__ int vol_of_item(const LaunchArgs& a, int it) {
  int b = 0;
  while (b + 1 < a.nvol && it >= a.item_begin[b + 1]) ++b;
  return b;
}

// Row of C memberships in global memory (16-byte aligned when C % 4 == 0).
template <int C>
__device__ __forceinline__ void load_row(const gfloat* p, float (&u)[C]) {
  typedef __attribute__((address_space(1))) const f4v G4;
  typedef __attribute__((address_space(1))) const f2v G2;
  if constexpr (C % 4 == 0) {
#pragma unroll
    for (int q = 0; q < C / 4; ++q) {
      const f4v v = reinterpret_cast<G4*>(p)[q];
      u[4 * q] = v.x;
      u[4 * q + 1] = v.y;
      u[4 * q + 2] = v.z;
      u[4 * q + 3] = v.w;
    }
  } else if constexpr (C % 2 == 0) {
#pragma unroll
    for (int q = 0; q < C / 2; ++q) {
      const f2v v = reinterpret_cast<G2*>(p)[q];
      u[2 * q] = v.x;
      u[2 * q + 1] = v.y;
    }
  } else {
#pragma unroll
    for (int j = 0; j < C; ++j) u[j] = p[j];
  }
}

template <int C>
__device__ __forceinline__ void store_row(gfloat* p, const float (&u)[C]) {
  typedef __attribute__((address_space(1))) f4v G4;
  typedef __attribute__((address_space(1))) f2v G2;
  if constexpr (C % 4 == 0) {
#pragma unroll
    for (int q = 0; q < C / 4; ++q) {
      f4v v;
      v.x = u[4 * q];
      v.y = u[4 * q + 1];
      v.z = u[4 * q + 2];
      v.w = u[4 * q + 3];
      reinterpret_cast<G4*>(p)[q] = v;
    }
  } else if constexpr (C % 2 == 0) {
#pragma unroll
    for (int q = 0; q < C / 2; ++q) {
      f2v v;
      v.x = u[2 * q];
      v.y = u[2 * q + 1];
      reinterpret_cast<G2*>(p)[q] = v;
    }
  } else {
#pragma unroll
    for (int j = 0; j < C; ++j) p[j] = u[j];
  }
}

// LDS cell of CP floats (C padded to a multiple of 4) read as float4s.
template <int C, int CP>
__device__ __forceinline__ void lds_cell_load(const float* __restrict__ s, float (&u)[C]) {
#pragma unroll
  for (int q = 0; q < CP / 4; ++q) {
    const float4 v = reinterpret_cast<const float4*>(s)[q];
    if (4 * q < C) u[4 * q] = v.x;
    if (4 * q + 1 < C) u[4 * q + 1] = v.y;
    if (4 * q + 2 < C) u[4 * q + 2] = v.z;
    if (4 * q + 3 < C) u[4 * q + 3] = v.w;
  }
}

template <int C, int CP>
__device__ __forceinline__ void lds_cell_store(float* __restrict__ s, const float (&u)[C]) {
#pragma unroll
  for (int q = 0; q < CP / 4; ++q) {
    float4 v;
    v.x = (4 * q < C) ? u[4 * q] : 0.f;
    v.y = (4 * q + 1 < C) ? u[4 * q + 1] : 0.f;
    v.z = (4 * q + 2 < C) ? u[4 * q + 2] : 0.f;
    v.w = (4 * q + 3 < C) ? u[4 * q + 3] : 0.f;
    reinterpret_cast<float4*>(s)[q] = v;
  }
}

// w = u^m for the centre sums of eq (3) and the objective of eq (1).
template <bool M2>
__device__ __forceinline__ float pow_m(float u, float m) {
  if constexpr (M2) return u * u;
  else return u > 0.f ? exp2f(m * log2f(u)) : 0.f;
}

// Memberships of eq (2) from squared distances d2[0..C), d2 > 0, times
// scale (1, or 0 to zero a row).
// m == 2: u_j = (1/d2_j) / sum_k (1/d2_k).  Otherwise u_j is proportional to
// (d2_min / d2_j)^(1/(m-1)), which is eq (2) scaled so no term overflows.
template <int C, bool M2>
__device__ __forceinline__ void memberships(const float (&d2)[C], float m, float (&u)[C],
                                            float scale = 1.f) {
  if constexpr (M2 && C <= 4) {
    // u_j = P_j / sum_k P_k with P_j the product of the other d2: one
    // reciprocal.  d2 lies in [1e-12, 2e3] (|lambda|, |xi| <= 1e3), so the
    // products of at most three stay within float32's normal range.
    float P[C];
    if constexpr (C == 2) {
      P[0] = d2[1];
      P[1] = d2[0];
    } else if constexpr (C == 3) {
      P[0] = d2[1] * d2[2];
      P[1] = d2[0] * d2[2];
      P[2] = d2[0] * d2[1];
    } else {
      const float d01 = d2[0] * d2[1], d23 = d2[2] * d2[3];
      P[0] = d2[1] * d23;
      P[1] = d2[0] * d23;
      P[2] = d2[3] * d01;
      P[3] = d2[2] * d01;
    }
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < C; ++j) s += P[j];
    const float r = frcp(s) * scale;
#pragma unroll
    for (int j = 0; j < C; ++j) u[j] = P[j] * r;
  } else if constexpr (M2) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < C; ++j) {
      u[j] = frcp(d2[j]);
      s += u[j];
    }
    const float r = frcp(s) * scale;
#pragma unroll
    for (int j = 0; j < C; ++j) u[j] *= r;
  } else {
    float dmin = d2[0];
#pragma unroll
    for (int j = 1; j < C; ++j) dmin = fminf(dmin, d2[j]);
    const float e = 1.f / (m - 1.f);
    const float lmin = log2f(dmin);
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < C; ++j) {
      u[j] = exp2f((lmin - log2f(d2[j])) * e);
      s += u[j];
    }
    const float r = scale / s;
#pragma unroll
    for (int j = 0; j < C; ++j) u[j] *= r;
  }
}

// ------------------------------------------------------------ tile sums
// Every tile of a launch leaves NV fp32 sums in its own slot of the pair's
// partials ([NV][slots], so that the slots of one sum are read side by side);
// a per-pair finalise kernel launched right after adds the slots in fp64 in
// tile order.  Both reductions have a fixed order, so the results do not
// depend on scheduling.

// The halves of 32 lanes of a added together in the lower half, those of b in
// the upper half; alike for the rows of 16 within each half; and each row's
// lanes added to those N further on.
__device__ __forceinline__ float swap32_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int N>
__device__ __forceinline__ float ror_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, false));
}
__device__ __forceinline__ double make_f64(uint32_t lo, uint32_t hi) {
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ uint32_t lo_of(double v) { return (uint32_t)__double_as_longlong(v); }
__device__ __forceinline__ uint32_t hi_of(double v) { return (uint32_t)((uint64_t)__double_as_longlong(v) >> 32); }
__device__ __forceinline__ double swap32_add(double a, double b) {
  const auto l = __builtin_amdgcn_permlane32_swap(lo_of(a), lo_of(b), false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(hi_of(a), hi_of(b), false, false);
  return make_f64(l[0], h[0]) + make_f64(l[1], h[1]);
}
__device__ __forceinline__ double swap16_add(double a, double b) {
  const auto l = __builtin_amdgcn_permlane16_swap(lo_of(a), lo_of(b), false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(hi_of(a), hi_of(b), false, false);
  return make_f64(l[0], h[0]) + make_f64(l[1], h[1]);
}
template <int N>
__device__ __forceinline__ double ror_add(double v) {
  const int l = __builtin_amdgcn_update_dpp(0, (int)lo_of(v), 0x120 + N, 0xf, 0xf, false);
  const int h = __builtin_amdgcn_update_dpp(0, (int)hi_of(v), 0x120 + N, 0xf, 0xf, false);
  return v + make_f64((uint32_t)l, (uint32_t)h);
}

// Sums of NV values over the 64 lanes, each by the tree of a butterfly over
// l ^ 32, l ^ 16, ..., l ^ 1.  The first two levels put two and then four
// values into one register, so the rest costs a quarter: about 30
// instructions for 9 values and no LDS, against 108 and 54 LDS permutes for
// one butterfly per value.  On return every lane of row q (lanes 16 q ..
// 16 q + 15) of out[r] holds the sum of value sum_index(r, q), if below NV.
template <int NV>
constexpr int kSumRegs = (NV + 3) / 4;
__device__ __forceinline__ int sum_index(int r, int row) { return 4 * r + ((row & 1) << 1 | row >> 1); }
template <class T, int NV>
__device__ __forceinline__ void wave_sums(const T (&v)[NV], T (&out)[kSumRegs<NV>]) {
#pragma unroll
  for (int r = 0; r < kSumRegs<NV>; ++r) {
    auto at = [&](int k) -> T { return k < NV ? v[k < NV ? k : 0] : T(0); };
    T s = swap16_add(swap32_add(at(4 * r), at(4 * r + 1)), swap32_add(at(4 * r + 2), at(4 * r + 3)));
    s = ror_add<8>(s);
    s = ror_add<4>(s);
    s = ror_add<2>(s);
    out[r] = ror_add<1>(s);
  }
}

// Wave owning a tile: its sums to slot `tile` of `slots`.  Lane r of a row
// stores the row's sum of register r, so one store instruction writes them all.
// The lane number is opaque: kept out of the loops this is called in, the
// addresses derived from it would occupy registers there (170 -> 184 at C = 6).
template <int NV>
__device__ __forceinline__ void wave_tile_store(float* partials, int tile, int slots, const float (&acc)[NV]) {
  float sum[kSumRegs<NV>];
  wave_sums<float, NV>(acc, sum);
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int r = lane & 15;
  float v = sum[0];
#pragma unroll
  for (int q = 1; q < kSumRegs<NV>; ++q) v = r == q ? sum[q] : v;
  const int k = sum_index(r, lane >> 4);
  if (r < kSumRegs<NV> && k < NV) as_global(partials)[(size_t)(uint32_t)k * (uint32_t)slots + (uint32_t)tile] = v;
}

// Work group owning a tile: the sums of its waves, added in order through LDS.
template <int NV, int NT>
__device__ __forceinline__ void block_tile_store(float* partials, int tile, int slots, const float (&acc)[NV],
                                                 float* s_red) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float sum[kSumRegs<NV>];
  wave_sums<float, NV>(acc, sum);
#pragma unroll
  for (int r = 0; r < kSumRegs<NV>; ++r) {
    const int k = sum_index(r, lane >> 4);
    if ((lane & 15) == 0 && k < NV) s_red[wave * NV + k] = sum[r];
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) s += s_red[w * NV + threadIdx.x];
    as_global(partials)[(size_t)threadIdx.x * slots + tile] = s;
  }
  __syncthreads();
}

// A thread's sums over its voxels: in runs of kRunTerms and, where it has more
// than one (LONG), the sum of the runs.  In one chain the roundings of equal
// terms (a region of one intensity) all go the same way: 2e-7 of the sum over 32
// terms, 4e-7 over 64, 1.5e-5 over 4096, against 4e-8 over 8 terms or 8 runs of
// them; a thread never has more (fcm_vpt).
template <int NV, bool LONG>
struct RunSums {
  float run[NV];
  float all[LONG ? NV : 1];
  __device__ __forceinline__ RunSums() {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      run[k] = 0.f;
      if constexpr (LONG) all[k] = 0.f;
    }
  }
  // Before voxel k of the thread's (in steps that divide kRunTerms).
  __device__ __forceinline__ void before(int k) {
    if constexpr (LONG)
      if (k % kRunTerms == 0 && k > 0) fold();
  }
  __device__ __forceinline__ void fold() {
    if constexpr (LONG) {
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        all[k] += run[k];
        run[k] = 0.f;
      }
    }
  }
  // The totals, in run.
  __device__ __forceinline__ const float (&total())[NV] {
    fold();
    if constexpr (LONG) {
#pragma unroll
      for (int k = 0; k < NV; ++k) run[k] = all[k];
    }
    return run;
  }
};

// One work group per pair: add the pair's tile slots in fp64 (thread t takes
// slots t, t + 1024, ...; then the wave's tree and the waves in order) and
// advance its state: new centres (eq (3)), J of the iteration's input state
// (eq (1)) and the stop rule; or, for the objective-only pass, the fitness.
// Pairs that have stopped are left alone.  A short dependent launch, bound by
// latency: the state is read while the slots are, one lane finishes each
// centre.  One step of 16, 2640 and 11556 slots (C = 4): 3.3, 4.9 and 12 us
// (3.9, 7.2 and 18 us with 256 threads reading slots of 2C + 1 floats).
// NT = 256, for launches whose pairs have at most 256 slots, starts 1 us
// sooner than NT = 1024 and gives the same bits (the other threads add zeros).
template <int C, bool STEP, int NT>
__global__ __launch_bounds__(NT) void k_finalize(const LaunchArgs a) {
  constexpr int NV = STEP ? 2 * C + 1 : 1;
  constexpr int NWF = NT / 64;
  __shared__ double s_red[NWF * NV];
  const int pair = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const PairDev pr = ld_const(a.pairs + pair);
  SolveState* st = pr.st;
  if (STEP && ld_const(&st->stop)) return;
  const VolDev* vd = a.vols + pair / a.P;
  const int slots = a.use_1d ? ld_const(&vd->tiles1d) : ld_const(&vd->slots);
  const int t = ld_const(&st->iter) + 1;
  const float c_old = st->c[(t & 1) ^ 1][lane & (kMaxC - 1)];
  const double J1 = st->J_prev1;
  // Without want_j a step leaves no J sums.
  const int nv = STEP && !a.want_j ? 2 * C : NV;
  double d[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) d[k] = 0.0;
  const gfloat* parts = as_global(pr.partials);
  // Four slots in flight per thread (the order of the additions, and so the
  // result, is that of the plain strided loop); with 1024 threads fewer where
  // the 128 registers each then has do not hold more beside the fp64 sums.
  constexpr int kU = NT < 1024 || 6 * NV <= 114 ? 4 : 4 * NV <= 114 ? 2 : 1;
  int s = threadIdx.x;
  for (; s + (kU - 1) * NT < slots; s += kU * NT) {
    float v[kU][NV];
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int k = 0; k < NV; ++k) v[u][k] = k < nv ? parts[(size_t)k * slots + s + u * NT] : 0.f;
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int k = 0; k < NV; ++k) d[k] += (double)v[u][k];
  }
  for (; s < slots; s += NT) {
#pragma unroll
    for (int k = 0; k < NV; ++k) d[k] += k < nv ? (double)parts[(size_t)k * slots + s] : 0.0;
  }
  double sum[kSumRegs<NV>];
  wave_sums<double, NV>(d, sum);
#pragma unroll
  for (int r = 0; r < kSumRegs<NV>; ++r) {
    const int k = sum_index(r, lane >> 4);
    if ((lane & 15) == 0 && k < NV) s_red[wave * NV + k] = sum[r];
  }
  __syncthreads();
  if (wave != 0) return;
  auto total = [&](int k) -> double {
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < NWF; ++w) v += s_red[w * NV + k];
    return v;
  };
  if constexpr (STEP) {
    if (lane < C) {
      const double den = total(C + lane);
      const float c = den > 0.0 ? (float)(total(lane) / den) : c_old;
      st->c[t & 1][lane] = c;
      if (st->B_hist) st->B_hist[(size_t)(t - 1) * C + lane] = den;
      if (st->c_hist) st->c_hist[(size_t)t * C + lane] = c;
    }
    if (lane == 0) {
      const double J = total(2 * C);
      if (st->J_hist) st->J_hist[t - 1] = J;
      int stop = 0;
      if (t >= 2 && st->eps > 0.f && fabs(J - J1) <= (double)st->eps * fabs(J1)) stop = 1;
      if (t >= st->max_iter) stop = 1;
      st->J_prev2 = J1;
      st->J_prev1 = J;
      st->iter = t;
      st->stop = stop;
    }
  } else {
    if (lane == 0) st->J_eval = total(0);
  }
}

}  // namespace pifcm
