// Device pieces shared by the descriptor kernels (descriptors.hip and
// desc_tiles.hip): wave-level LDS ordering, the atom of a block, the cutoff's
// sine and cosine, integer powers and small index arithmetic.
#pragma once

#include <math.h>

#include "common.h"

namespace nnp {

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float fexp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float frcp(float x) { return __builtin_amdgcn_rcpf(x); }
// Orders this wave's LDS accesses: writes before it are seen by reads after
// it in every lane, and the compiler moves no LDS access across it.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
// Keeps this wave's LDS accesses in program order without waiting for them
// to complete: the LDS serves one wave's instructions in the order they are
// issued, so a read issued after a write of the same address by any lane of
// the wave returns the written value.  Only the compiler has to be kept from
// moving or caching accesses across it.
__device__ __forceinline__ void wave_lds_order() { __asm__ volatile("" ::: "memory"); }
__device__ __forceinline__ int nb_species(const float4& f) { return __float_as_int(f.w) & 15; }
__device__ __forceinline__ int nb_entry(const float4& f) { return __float_as_int(f.w) >> 4; }


// The structure of atom i: the largest c < B with atom_ptr[c] <= i.  Each
// round the 64 lanes probe 64 evenly spaced positions of the remaining range
// and one ballot keeps the stretch after the last probe at or below i, so
// 2048 structures take two dependent rounds of loads instead of eleven.
// Every lane of the wave must call it (with the same i).
__device__ __forceinline__ int struct_of_atom(const int64_t* atom_ptr, int32_t B, int64_t i) {
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = B;  // atom_ptr[lo] <= i; the answer lies in [lo, hi)
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) / 64;
    const int p = lo + lane * step;
    const uint64_t le = __ballot(p < hi && atom_ptr[p] <= i);  // a prefix of the lanes: atom_ptr does not decrease
    lo += (__popcll(le) - 1) * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

// The atom a one-atom-per-block descriptor launch works on.  With the
// list's bin order (kept by the list build) the grid is whole rounds of the
// eight XCDs and block b takes slot (b mod 8) * per + b / 8 of that order:
// consecutive blocks go to different XCDs, so each XCD walks one contiguous
// stretch of space and the neighbor positions its atoms gather stay in its
// L2.  Without the order, or while the list is not valid (the order is then
// not a permutation), the slot is the atom.  -1 for slots past the atoms.
__device__ __forceinline__ int64_t atom_of_block(const int32_t* __restrict__ order, int64_t N, bool valid) {
  int64_t slot = blockIdx.x;
  if (order) slot = (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  if (slot >= N) return -1;
  return (order && valid) ? (int64_t)order[slot] : slot;
}

// Blocks of such a launch: whole rounds of the eight XCDs with the order.
static inline unsigned atom_grid(int64_t N, const int32_t* order) {
  return (unsigned)(order ? (N + 7) / 8 * 8 : N);
}

// sin and cos of x in [0, pi/2] by their Taylor series to x^11 and x^12
// (truncation below 6e-8 at pi/2), without range reduction.
__device__ __forceinline__ void sincos_quarter(float x, float& sn, float& cs) {
  const float z = x * x;
  sn = x * fmaf(z, fmaf(z, fmaf(z, fmaf(z, fmaf(z, -2.5052108e-8f, 2.7557319e-6f), -1.9841270e-4f), 8.3333333e-3f),
                        -1.6666667e-1f), 1.0f);
  cs = fmaf(z, fmaf(z, fmaf(z, fmaf(z, fmaf(z, fmaf(z, 2.0876757e-9f, -2.7557319e-7f), 2.4801587e-5f), -1.3888889e-3f),
                        4.1666667e-2f), -0.5f), 1.0f);
}

// x^e for a small positive integer e, on an array (exponent bits outside).
template <int N>
__device__ __forceinline__ void ipow_array(const float (&x)[N], int e, float (&out)[N]) {
  float base[N];
#pragma unroll
  for (int p = 0; p < N; ++p) {
    out[p] = 1.0f;
    base[p] = x[p];
  }
  while (e) {
    if (e & 1) {
#pragma unroll
      for (int p = 0; p < N; ++p) out[p] *= base[p];
    }
    e >>= 1;
    if (e) {
#pragma unroll
      for (int p = 0; p < N; ++p) base[p] *= base[p];
    }
  }
}

// x^E for a compile-time E (fully unrolled); E = 0 selects the runtime loop.
template <int E, int N>
__device__ __forceinline__ void ipow_sel(const float (&x)[N], int e_runtime, float (&out)[N]) {
  if constexpr (E == 0) {
    ipow_array<N>(x, e_runtime, out);
  } else {
    float base[N];
    bool first = true;
#pragma unroll
    for (int p = 0; p < N; ++p) base[p] = x[p];
#pragma unroll
    for (int bit = 0; bit < 11; ++bit) {
      if ((E >> bit) == 0) break;
      if ((E >> bit) & 1) {
#pragma unroll
        for (int p = 0; p < N; ++p) out[p] = first ? base[p] : out[p] * base[p];
        first = false;
      }
      if ((E >> (bit + 1)) != 0) {
#pragma unroll
        for (int p = 0; p < N; ++p) base[p] *= base[p];
      }
    }
  }
}

// q = t / n, r = t mod n for 0 <= t < 2^24 and 0 < n < 2^12, through a
// float reciprocal: the float quotient is off by at most one.
__device__ __forceinline__ void divmod_small(int t, int n, float inv_n, int& q, int& r) {
  q = (int)((float)t * inv_n);
  r = t - q * n;
  if (r < 0) {
    --q;
    r += n;
  } else if (r >= n) {
    ++q;
    r -= n;
  }
}

__device__ __forceinline__ int pair_block(int S, int a, int b) {
  if (a > b) {
    int t = a;
    a = b;
    b = t;
  }
  return a * S - a * (a - 1) / 2 + (b - a);
}

// With one species the descriptor launch also writes the identity grouping.
__device__ __forceinline__ void identity_group(IdentityGroup one, const nn_system& sys, int64_t i, int64_t* meta) {
  one.perm[i] = (int32_t)i;
  if (sys.species[i] != 0) atomicOr((unsigned long long*)&meta[kMetaErr], (unsigned long long)kErrSpecies);
  if (i == 0) {
    one.sp_start[0] = 0;
    one.sp_start[1] = sys.n_atoms;
  }
}

// Floats of the adjoint's radial lambda in LDS: S n_rad rounded up to a
// multiple of 4, so that the angular blocks after it are float4-aligned.
__host__ __device__ constexpr int adj_lam_radial(int S, int n_rad) { return (S * n_rad + 3) / 4 * 4; }

// Packed passes: kPackAtoms atoms per wave, kPackLanes lanes per atom in the
// per-atom phases.  An atom is packed when its row has at most kPackNb
// entries; longer rows go to the one-atom kernels.
constexpr int kPackAtoms = 4;
constexpr int kPackLanes = 16;
constexpr int kPackNb = 32;

// The tile passes of desc_tiles.hip (mBP term): wpa waves per atom, or for
// wpa = 0 only the atoms whose rows the packed passes leave out.
void launch_fwd_tiles(const nn_system& sys, const nn_nlist& nl, const DescConst& P, float* G, IdentityGroup one,
                      int wpa, hipStream_t s);
void launch_adj_tiles(const nn_system& sys, const nn_nlist& nl, const DescConst& P, const float* lam, float4* pg,
                      int wpa, hipStream_t s);

#define NNP_DISPATCH(NT_, NRA_, CALL)                                          \
  do {                                                                         \
    if (nt == 4 && nra == 4) { constexpr int NT_ = 4, NRA_ = 4; CALL; }        \
    else if (nt == 4 && nra == 8) { constexpr int NT_ = 4, NRA_ = 8; CALL; }   \
    else if (nt == 8 && nra == 4) { constexpr int NT_ = 8, NRA_ = 4; CALL; }   \
    else if (nt == 8 && nra == 8) { constexpr int NT_ = 8, NRA_ = 8; CALL; }   \
    else if (nt == 16 && nra == 4) { constexpr int NT_ = 16, NRA_ = 4; CALL; } \
    else if (nt == 16 && nra == 8) { constexpr int NT_ = 16, NRA_ = 8; CALL; } \
  } while (0)

}  // namespace nnp
