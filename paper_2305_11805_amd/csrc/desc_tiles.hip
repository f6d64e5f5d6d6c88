// The mBP descriptor and its adjoint, one atom per block, with the atom's
// neighbors sorted by distance.
//
// What bounds both passes is the FP32 issue rate: a triplet costs its
// geometry, n_theta powers, n_rs_ang Gaussians of the average radius and an
// n_theta x n_rs_ang outer product (or, in the adjoint, two contractions).
// A Gaussian R_q = 2^(-d^2), d = sqrt(eta log2 e) (rbar - Rs'_q), is below
// 2^-50 beyond |d| = kScreen: such a term is under 2^-25 of FP32's
// resolution of one term of ordinary size, and no sum over an atom's
// triplets (at most 18336) can see it.  (A bin that holds no larger term is zero
// here, and below 4e-11 in the passes that form every term.)  A wave therefore takes its triplets
// in strips of neighbors of like distance, so that the rbar of the 64
// triplets it holds at a time lie close together, and leaves out a radius
// term only when all 64 are beyond kScreen of it (one ballot per term, exact
// whatever the grids are and however they are ordered).  With 8 terms 0.64
// to 0.79 A apart and eta = 12 between 4 and 5 of 8 remain.
//
// Measured against passes that take the triplets in index order and every
// radius term (forward on the 4x4x1 FP32 MFMA, adjoint with one LDS
// read-add-write per step of a circular schedule), both directions in us:
//                                      forward         adjoint
//   65536 atoms, 1 species, 52 nb.     590 ->  452     755 ->  680
//   65536 atoms, 2 species, 81 nb.    1268 ->  990    1860 -> 1445
//   32768 atoms, 4 species, 47 nb.     372 ->  331     412 ->  324
// The forward issues 13000 vector instructions for an atom of 81 neighbors
// at 2.9 clocks each, the rate that a plain FMA loop sustains on this chip.
#include <math.h>

#include "common.h"
#include "desc_ops.h"

namespace nnp {

constexpr float kScreen = 7.0710678f;  // sqrt(50): 2^(-kScreen^2) = 2^-50
constexpr float kReach = kScreen + 1e-3f;  // neighbors are sorted to rc / 2^20, about 2e-5 of these units
constexpr int kTileRounds = 2;         // rows of up to 128 entries are staged in one pass
constexpr float kFar = 1e30f;          // distance of lanes and slots that hold no neighbor

typedef unsigned uint2v __attribute__((ext_vector_type(2)));

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppMirror8 = 0x141, kDppRor8 = 0x128;

// a and b become the sums over lane pairs l, l ^ 32: of a in lanes 0-31, of
// b in lanes 32-63.
__device__ __forceinline__ float fold32(float a, float b) {
  const uint2v r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// The same over l, l ^ 16: of a in even rows of 16 lanes, of b in odd rows.
__device__ __forceinline__ float fold16(float a, float b) {
  const uint2v r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Within rows: a where the lane's `bit` is clear, b where it is set, each
// plus the same value of the lane that CTRL pairs it with.
template <int CTRL>
__device__ __forceinline__ float fold_dpp(float a, float b, bool high) {
  const float keep = high ? b : a, send = high ? a : b;
  return keep + dpp_f<CTRL>(send);
}

// Sums of v[0 .. N - 1] over the wave, in a fixed tree: lane l returns the
// sum of v[l mod N] (N = 16, 32 or 64).
template <int N>
__device__ __forceinline__ float wave_sums(const float (&v)[N]) {
  const int lane = threadIdx.x & 63;
  float a[32], b[16], c[8], d[4];
  if constexpr (N == 64) {
#pragma unroll
    for (int i = 0; i < 32; ++i) a[i] = fold32(v[i], v[i + 32]);
  } else if constexpr (N == 32) {
#pragma unroll
    for (int i = 0; i < 32; ++i) a[i] = v[i];
  }
  if constexpr (N >= 32) {
#pragma unroll
    for (int i = 0; i < 16; ++i) b[i] = fold16(a[i], a[i + 16]);
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) b[i] = v[i];
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) c[i] = fold_dpp<kDppRor8>(b[i], b[i + 8], lane & 8);
#pragma unroll
  for (int i = 0; i < 4; ++i) d[i] = fold_dpp<kDppMirror8>(c[i], c[i + 4], lane & 4);
  const float e0 = fold_dpp<kDppXor2>(d[0], d[2], lane & 2), e1 = fold_dpp<kDppXor2>(d[1], d[3], lane & 2);
  float r = fold_dpp<kDppXor1>(e0, e1, lane & 1);
  if constexpr (N == 16) r = fold16(r, r);
  if constexpr (N <= 32) r = fold32(r, r);
  return r;
}

// One level of half_sums: v[i] and v[i + M / 2] folded into M / 2 values.
template <int M, typename Fold>
__device__ __forceinline__ void fold_level(float* v, Fold&& fold) {
#pragma unroll
  for (int i = 0; i < M / 2; ++i) v[i] = fold(v[i], v[i + M / 2]);
}
// Sums of v[0 .. N - 1] over each half of the wave: lane hl of a half
// returns v[E hl + e] in out[e], E = N / 32 (N = 16: v[hl mod 16]).
template <int N>
__device__ __forceinline__ void half_sums(float (&v)[N], float (&out)[N / 32 > 0 ? N / 32 : 1]) {
  const int lane = threadIdx.x & 63;
  constexpr int M = N >= 32 ? N / 2 : N;  // values left after the first level
  if constexpr (N >= 32) fold_level<N>(v, [](float a, float b) { return fold16(a, b); });
  fold_level<M>(v, [&](float a, float b) { return fold_dpp<kDppRor8>(a, b, lane & 8); });
  fold_level<M / 2>(v, [&](float a, float b) { return fold_dpp<kDppMirror8>(a, b, lane & 4); });
  fold_level<M / 4>(v, [&](float a, float b) { return fold_dpp<kDppXor2>(a, b, lane & 2); });
  fold_level<M / 8>(v, [&](float a, float b) { return fold_dpp<kDppXor1>(a, b, lane & 1); });
#pragma unroll
  for (int e = 0; e < (N / 32 > 0 ? N / 32 : 1); ++e) out[e] = N >= 32 ? v[e] : fold16(v[e], v[e]);
}

// ---------------------------------------------------------------------------
// staging
// ---------------------------------------------------------------------------

// One neighbor inside rc from its FP64 displacement: the unit vector, the
// distance scaled for the angular Gaussian (so that the scaled average
// radius of a pair is a sum) and for the radial one, each as hi + lo, the
// cutoff and its derivative (rc - r in FP64, so that they keep their
// relative precision up to rc), and 1/r.
struct PairRec {
  float ux, uy, uz, ra, ra_lo, rr, rr_lo, fc, dfc, ir;
  uint32_t key;  // r in 20 bits, above the low byte
};
// r = sqrt(x) and 1/r in FP64 from the hardware's reciprocal root (about 2^-23)
// by two coupled Newton steps and a last correction of r: both within an
// ulp, in a third of the instructions of a root and a division (Goldschmidt's
// iteration).  For x = 0, atoms in one place, r = 0 and 1/r is NaN, so that the
// radial bins stay finite and only what needs a direction does not.
__device__ __forceinline__ void root64(double x, double& r, double& ir) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  double e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  e = fma(-h, g, 0.5);
  h = fma(h, e, h);
  g = fma(g, e, g);
  r = x > 0.0 ? fma(fma(-g, g, x), h, g) : 0.0;
  ir = h + h;
}
__device__ __forceinline__ PairRec tile_record(const double (&d)[3], double r2, const DescConst& P) {
  PairRec p;
  double r, ir;
  root64(r2, r, ir);
  p.ux = (float)(d[0] * ir);
  p.uy = (float)(d[1] * ir);
  p.uz = (float)(d[2] * ir);
  p.ir = (float)ir;
  const double a = r * P.ra_scale, b = r * P.rr_scale;
  p.ra = (float)a;
  p.ra_lo = (float)(a - (double)p.ra);
  p.rr = (float)b;
  p.rr_lo = (float)(b - (double)p.rr);
  float sn, cs;
  sincos_quarter((float)(P.half_pi_over_rc64 * (P.rc64 - r)), sn, cs);
  p.fc = sn * sn;
  p.dfc = -P.pi_over_rc * (sn * cs);
  p.key = (uint32_t)((float)r * P.key_scale) << 8;
  return p;
}

constexpr int kKeyWords = kMaxNb + 4;
struct TileRow {
  int seg[NN_MAX_SPECIES + 1];
  int n;
  int bad;
  int all;  // adjoint: no term is left out
};

// Stages the neighbors of atom i inside rc, sorted by (species and) distance
// with ties in row order: put(slot, entry - e0, species, record) is called
// by the lane that holds a neighbor, slot being its rank.  Wave 0 works; every
// thread passes the barrier.  Entries at r >= rc get a zero pair gradient if
// pg != nullptr; keys: 16-byte aligned LDS of kKeyWords words, free again
// afterwards.  The rank of a neighbor is the number of smaller keys
// (species, r in 20 bits, position among the valid entries), counted from
// the keys in LDS four at a time: about 5 instructions per key and round of
// 64 entries, 2 to 4 % of a bulk atom's work.
template <bool BY_SPECIES, typename Put>
__device__ __forceinline__ void stage_sorted(TileRow& tr, uint32_t* keys, int64_t i, const nn_system& sys,
                                             const int64_t* __restrict__ offsets, const int32_t* __restrict__ nbr,
                                             const int8_t* __restrict__ shift, const DescConst& P, int64_t* meta,
                                             float4* __restrict__ pg, Put&& put) {
  const int lane = threadIdx.x & 63;
  if (threadIdx.x >= 64) {
    __syncthreads();
    return;
  }
  const double xi[3] = {sys.pos[3 * i], sys.pos[3 * i + 1], sys.pos[3 * i + 2]};
  const int64_t e0 = offsets[i], e1 = offsets[i + 1];
  const double rc2 = P.rc64 * P.rc64;
  const int S = P.S;
  const char4* sh4 = reinterpret_cast<const char4*>(shift);
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  double h[9];
  // the structure's cell: only image shifts need it (with all shifts zero
  // displacement64 gives x_j - x_i exactly whatever the cell)
  auto load_cell = [&](bool need) {
    if (__any(need)) {
      const int c = struct_of_atom(sys.atom_ptr, sys.n_structs, i);
      for (int k = 0; k < 9; ++k) h[k] = sys.cell[9 * (int64_t)c + k];
    } else {
      for (int k = 0; k < 9; ++k) h[k] = 0.0;
    }
  };
  // the number of keys below k0 (and below k1): n keys, padded with ones
  auto rank = [&](int n, uint32_t k0, uint32_t k1, bool two, int& r0, int& r1) {
    const uint4* k4 = reinterpret_cast<const uint4*>(keys);
    r0 = r1 = 0;
    if (two) {
      for (int t = 0; t < n; t += 4) {
        const uint4 k = k4[t >> 2];
        r0 += (k.x < k0 ? 1 : 0) + (k.y < k0 ? 1 : 0) + (k.z < k0 ? 1 : 0) + (k.w < k0 ? 1 : 0);
        r1 += (k.x < k1 ? 1 : 0) + (k.y < k1 ? 1 : 0) + (k.z < k1 ? 1 : 0) + (k.w < k1 ? 1 : 0);
      }
    } else {
      for (int t = 0; t < n; t += 4) {
        const uint4 k = k4[t >> 2];
        r0 += (k.x < k0 ? 1 : 0) + (k.y < k0 ? 1 : 0) + (k.z < k0 ? 1 : 0) + (k.w < k0 ? 1 : 0);
      }
    }
  };
  auto species_key = [&](int sp) { return BY_SPECIES ? (uint32_t)sp << 28 : 0u; };
  bool bad = false;
  if (e1 - e0 <= kTileRounds * kWave) {
    // at most 128 entries, held in registers from the test to the placing
    bool valid[kTileRounds];
    int sp[kTileRounds];
    int32_t jr[kTileRounds];
    char4 s4r[kTileRounds];
    PairRec rec[kTileRounds];
    uint32_t key[kTileRounds];
    bool shifted = false;
#pragma unroll
    for (int r = 0; r < kTileRounds; ++r) {
      const int64_t e = e0 + r * kWave + lane;
      jr[r] = 0;
      s4r[r] = make_char4(0, 0, 0, 0);
      if (e < e1) {
        jr[r] = nbr[e];
        s4r[r] = sh4[e];
        shifted = shifted || (s4r[r].x | s4r[r].y | s4r[r].z) != 0;
      }
    }
    load_cell(shifted);
    int n = 0;
#pragma unroll
    for (int r = 0; r < kTileRounds; ++r) {
      const int64_t e = e0 + r * kWave + lane;
      valid[r] = false;
      sp[r] = 0;
      key[r] = ~0u;
      if (e < e1) {
        double d[3];
        displacement64(xi, sys.pos + 3 * (int64_t)jr[r], h, s4r[r].x, s4r[r].y, s4r[r].z, d);
        const double r2 = norm2_64(d);
        valid[r] = r2 < rc2;
        sp[r] = sys.species[jr[r]];
        if (sp[r] < 0 || sp[r] >= S) {
          bad = bad || valid[r];
          valid[r] = false;
        }
        if (valid[r]) rec[r] = tile_record(d, r2, P);
        else if (pg) pg[e] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
      const uint64_t m = __ballot(valid[r]);
      const int at = n + __popcll(m & lt);
      if (valid[r]) {
        key[r] = species_key(sp[r]) | rec[r].key | (uint32_t)at;
        keys[at] = key[r];
      }
      n += __popcll(m);
    }
    if (lane < 4) keys[n + lane] = ~0u;
    if (BY_SPECIES) {
      int total = 0;
      for (int s2 = 0; s2 < S; ++s2) {
        if (lane == 0) tr.seg[s2] = total;
#pragma unroll
        for (int r = 0; r < kTileRounds; ++r) total += __popcll(__ballot(valid[r] && sp[r] == s2));
      }
      if (lane == 0) tr.seg[S] = total;
    }
    if (lane == 0) {
      tr.n = n;
      tr.bad = 0;
      tr.all = 0;
    }
    wave_lds_sync();
    int slot[kTileRounds];
    rank(n, key[0], key[1], e1 - e0 > kWave, slot[0], slot[1]);
#pragma unroll
    for (int r = 0; r < kTileRounds; ++r)
      if (valid[r]) put(slot[r], r * kWave + lane, sp[r], rec[r]);
  } else {
    // longer rows: a pass that counts and writes the keys, a pass that places
    load_cell(true);
    int n = 0, cnt[NN_MAX_SPECIES];
    for (int s = 0; s < NN_MAX_SPECIES; ++s) cnt[s] = 0;
    auto entry = [&](int64_t e, bool& valid, int& sp, PairRec& rec, bool first) {
      valid = false;
      sp = 0;
      if (e < e1) {
        const int32_t j = nbr[e];
        const char4 s4 = sh4[e];
        double d[3];
        displacement64(xi, sys.pos + 3 * (int64_t)j, h, s4.x, s4.y, s4.z, d);
        const double r2 = norm2_64(d);
        valid = r2 < rc2;
        sp = sys.species[j];
        if (sp < 0 || sp >= S) {
          bad = bad || valid;
          valid = false;
        }
        if (valid) rec = tile_record(d, r2, P);
        else if (pg && first) pg[e] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    };
    for (int64_t base = e0; base < e1; base += kWave) {
      bool valid;
      int sp;
      PairRec rec;
      entry(base + lane, valid, sp, rec, true);
      const uint64_t m = __ballot(valid);
      const int at = n + __popcll(m & lt);
      if (valid && at < kMaxNb) keys[at] = species_key(sp) | rec.key | (uint32_t)at;
      n += __popcll(m);
      for (int s = 0; s < S; ++s) cnt[s] += __popcll(__ballot(valid && sp == s));
    }
    if (n > kMaxNb && lane == 0) atomicOr((unsigned long long*)&meta[kMetaErr], (unsigned long long)kErrTooMany);
    if (n <= kMaxNb && lane < 4) keys[n + lane] = ~0u;
    if (lane == 0) {
      tr.n = n;
      tr.bad = n > kMaxNb;
      tr.all = 0;
      if (BY_SPECIES) {
        int total = 0;
        for (int s = 0; s < S; ++s) {
          tr.seg[s] = total;
          total += cnt[s];
        }
        tr.seg[S] = total;
      }
    }
    wave_lds_sync();
    if (n <= kMaxNb) {
      int seen = 0;
      for (int64_t base = e0; base < e1; base += kWave) {
        bool valid;
        int sp;
        PairRec rec;
        entry(base + lane, valid, sp, rec, false);
        const uint64_t m = __ballot(valid);
        const int at = seen + __popcll(m & lt);
        seen += __popcll(m);
        int slot, none;
        rank(n, valid ? species_key(sp) | rec.key | (uint32_t)at : 0u, 0u, false, slot, none);
        if (valid) put(slot, (int)(base - e0) + lane, sp, rec);
      }
    }
  }
  if (__any(bad) && lane == 0) atomicOr((unsigned long long*)&meta[kMetaErr], (unsigned long long)kErrSpecies);
  __syncthreads();
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------

// sqrt(x), x >= 1e-30: one Newton step on the hardware's reciprocal root,
// within an ulp of the rounded root in 5 instructions instead of 13.
__device__ __forceinline__ float sqrt_near(float x) {
  const float y = __builtin_amdgcn_rsqf(x);
  const float s = x * y;
  return fmaf(fmaf(-s, s, x), 0.5f * y, s);
}

// Triplets of a species-pair block in strips of eight neighbors k.  Two
// species (na of the first, nb of the second): strip c holds the pairs of
// every j with k in [8c, 8c + 8); one species (n): of every j > k.  Odd
// strips run backwards, so that a wave that straddles two strips stays at
// one end of the distances.  Each lane keeps its strip and its place in it
// and moves on by the waves' 64 triplets (no division; strips shorter than a
// wave are few).
struct StripRect {
  int na, n8, full, rem;
  uint32_t inv_rem;  // ceil(2^16 / rem): x * inv_rem >> 16 = x / rem for x < 8 * 192
  int c, x;
  __device__ __forceinline__ void init(int na_, int nb_, int t) {
    na = na_;
    n8 = 8 * na_;
    full = nb_ >> 3;
    rem = nb_ & 7;
    inv_rem = rem ? (65536u + rem - 1) / rem : 0u;
    c = 0;
    x = t;
    wrap();
  }
  __device__ __forceinline__ void wrap() {
    while (n8 > 0 && x >= n8) {
      x -= n8;
      ++c;
    }
  }
  __device__ __forceinline__ void step(int by) {
    x += by;
    wrap();
  }
  __device__ __forceinline__ void at(int& j, int& k) const {
    int row = x >> 3, col = x & 7;
    if (c >= full) {
      row = (int)(__umul24(x, inv_rem) >> 16);
      col = x - __mul24(row, rem);
    }
    j = (c & 1) ? na - 1 - row : row;
    k = 8 * c + col;
  }
};
struct StripTri {
  int n, last;
  int s, x, size;
  __device__ __forceinline__ int size_of(int q) const {
    const int m = n - 8 * q;
    return q < last ? 8 * m - 36 : q == last ? __mul24(m, m - 1) / 2 : 1 << 30;
  }
  __device__ __forceinline__ void init(int n_, int t) {
    n = n_;
    last = n_ >> 3;
    s = 0;
    x = t;
    size = size_of(0);
    wrap();
  }
  __device__ __forceinline__ void wrap() {
    while (x >= size) {
      x -= size;
      ++s;
      size = size_of(s);
    }
  }
  __device__ __forceinline__ void step(int by) {
    x += by;
    wrap();
  }
  __device__ __forceinline__ void at(int& j, int& k) const {
    const int y = (s & 1) ? size - 1 - x : x;
    int row = 8 + ((y - 28) >> 3), col = (y - 28) & 7;
    if (y < 28) {  // the pairs inside the strip's own eight
      row = (int)((1.02f + __builtin_amdgcn_sqrtf(fmaf(8.0f, (float)y, 1.0f))) * 0.5f);
      col = y - (__mul24(row, row - 1) >> 1);
    }
    j = 8 * s + row;
    k = 8 * s + col;
  }
};

// The descriptor row of atom i by the block (WPA waves).  MANY: three or
// more species.  The waves share the triplets (AS = 1), or two waves of 16x8 bins
// the angle terms (AS = 2): each then takes all triplets with eight terms, in 96
// registers and five waves per SIMD where 128 bins take 168 and three, and no
// sums pass between them.  4096 atoms of 52 neighbors 69 -> 63 us, 2048 44 -> 38,
// for the triplets' geometry formed twice: where three waves per SIMD hold all
// atoms (up to 1536) the shared triplets take 30 against 36 us.
template <int NT, int NRA, int WPA, int ZC, bool MANY, int AS = 1>
__device__ __forceinline__ void fwd_tiles_atom(int64_t i, bool list_ok, const nn_system& sys,
                                               const int64_t* __restrict__ offsets, const int32_t* __restrict__ nbr,
                                               const int8_t* __restrict__ shift, const DescConst& P,
                                               float* __restrict__ G, int64_t* meta) {
  constexpr int NB = NT * NRA;
  constexpr int TW = WPA / AS;              // waves that share the triplets
  constexpr int NTW = NT / AS;              // angle terms of a wave
  constexpr int NBW = NTW * NRA;            // and its bins of a species-pair block
  constexpr int NS = NBW > 64 ? 64 : NBW;  // bins summed over the wave at a time
  __shared__ TileRow tr;
  __shared__ float4 nd[kMaxNb];  // unit vector, scaled distance (hi)
  __shared__ float4 nf[kMaxNb];  // fc, scaled distance (lo), distance scaled for the radial bins (hi, lo)
  // per wave: partial sums of the radial bins or of one angular block; while staging, the keys
  __shared__ __align__(16) float xch[WPA][WPA > 1 ? NN_MAX_SPECIES * kMaxRad : kKeyWords];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = WPA > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
  float* Gi = G + i * (int64_t)P.D;
  bool ok = list_ok;
  if (ok) {
    stage_sorted<true>(tr, reinterpret_cast<uint32_t*>(xch), i, sys, offsets, nbr, shift, P, meta, nullptr,
                       [&](int slot, int, int, const PairRec& p) {
                         nd[slot] = make_float4(p.ux, p.uy, p.uz, p.ra);
                         nf[slot] = make_float4(p.fc, p.ra_lo, p.rr, p.rr_lo);
                       });
    ok = !tr.bad;
  }
  if (!ok) {  // no valid list (its entries are never read), or too many neighbors
    for (int d = tid; d < P.D; d += 64 * WPA) Gi[d] = 0.f;
    return;
  }
  const int S = P.S, n_rad = P.n_rad;
  // radial bins: lane (o, k) sums bin k over every NG-th neighbor (NG = 4, 2
  // or 1 for up to 16, 32 or 64 bins), the waves over every WPA-th of those
  {
    const int lg = n_rad <= 16 ? 4 : n_rad <= 32 ? 5 : 6;
    const int ng = kWave >> lg, k = lane & ((1 << lg) - 1), o = lane >> lg;
    const bool in = k < n_rad;
    const float rs = in ? P.rs_rad_sc[k] : 0.f, rs_lo = in ? P.rs_rad_sc_lo[k] : 0.f;
    for (int s = 0; s < S; ++s) {
      float acc = 0.f;
      const int t1 = tr.seg[s + 1];
      auto add = [&](const float4& f, float fc) {
        const float dr = (f.z - rs) + (f.w - rs_lo);
        acc = fmaf(fexp2(-dr * dr), fc, acc);
      };
      if (ng == 1) {
#pragma unroll 4
        for (int t = tr.seg[s] + wv; t < t1; t += WPA) {
          const float4 f = nf[t];
          add(f, f.x);
        }
      } else {
#pragma unroll 2
        for (int t = tr.seg[s] + wv * ng; t < t1; t += ng * WPA) {
          const float4 f = nf[min(t + o, t1 - 1)];
          add(f, t + o < t1 ? f.x : 0.f);
        }
      }
      if (lg <= 5) acc = fold32(acc, acc);
      if (lg == 4) acc = fold16(acc, acc);
      if (in && o == 0) {
        if constexpr (WPA == 1) Gi[s * n_rad + k] = acc;
        else xch[wv][s * n_rad + k] = acc;
      }
    }
    if constexpr (WPA > 1) {
      __syncthreads();
      for (int x = tid; x < S * n_rad; x += 64 * WPA) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < WPA; ++w) v += xch[w][x];
        Gi[x] = v;
      }
      __syncthreads();
    }
  }
  const int tw = AS > 1 ? 0 : wv, p0 = AS > 1 ? NTW * wv : 0;  // its share of the triplets, its first angle term
  auto bin = [&](int x) { return AS > 1 ? x / NTW * NT + p0 + x % NTW : x; };  // place of the wave's bin x in the block
  float x_a[NTW], x_b[NTW];
#pragma unroll
  for (int p = 0; p < NTW; ++p) {
    x_a[p] = AS > 1 && p0 ? P.x_a[(NT - NTW) + p] : P.x_a[p];
    x_b[p] = AS > 1 && p0 ? P.x_b[(NT - NTW) + p] : P.x_b[p];
  }
  float* ang = Gi + n_rad * S;
  // adds the triplet of slots j and k (take: this lane holds one) to acc
  auto triplet = [&](int j, int k, bool take, float (&acc)[NBW]) {
    const float4 u = nd[j], v = nd[k];
    const float4 fu = nf[j], fv = nf[k];
    // cos, the smoothed sine from the cross product, the scaled average
    // radius as hi + lo (TwoSum, plus the low parts), and 2 fc fc
    const float c = fmaf(u.x, v.x, fmaf(u.y, v.y, u.z * v.z));
    const float cx = fmaf(u.y, v.z, -u.z * v.y), cy = fmaf(u.z, v.x, -u.x * v.z), cz = fmaf(u.x, v.y, -u.y * v.x);
    const float ssm = sqrt_near(fmaf(cx, cx, fmaf(cy, cy, fmaf(cz, cz, P.eps_tile))));
    const float sum = u.w + v.w;
    const float bb = sum - u.w;
    const float lo = ((u.w - (sum - bb)) + (v.w - bb)) + (fu.y + fv.y);
    const float rb = take ? sum : kFar;
    const float F2 = take ? 2.0f * fu.x * fv.x : 0.f;
    if constexpr (NTW <= 8) {
      float x[NTW], A[NTW];
#pragma unroll
      for (int p = 0; p < NTW; ++p) x[p] = fmaf(c, x_a[p], fmaf(ssm, x_b[p], P.x_c));
      ipow_sel<(ZC > 0 ? ZC : 0), NTW>(x, P.zeta, A);
#pragma unroll
      for (int q = 0; q < NRA; ++q) {
        const float d0 = rb - P.rs_ang_sc[q];
        if (__any(fabsf(d0) < kScreen)) {
          const float dq = d0 + (lo - P.rs_ang_sc_lo[q]);
          const float R = fexp2(-dq * dq) * F2;
#pragma unroll
          for (int p = 0; p < NTW; ++p) acc[q * NTW + p] = fmaf(A[p], R, acc[q * NTW + p]);
        }
      }
    } else {
      // sixteen angle terms: the radius terms first, then eight powers at a
      // time (16 x 8 bins in 168 registers, three waves per SIMD)
      float R[NRA];
      uint32_t live = 0;
#pragma unroll
      for (int q = 0; q < NRA; ++q) {
        const float d0 = rb - P.rs_ang_sc[q];
        R[q] = 0.f;
        if (__any(fabsf(d0) < kScreen)) {
          const float dq = d0 + (lo - P.rs_ang_sc_lo[q]);
          R[q] = fexp2(-dq * dq) * F2;
          live |= 1u << q;
        }
      }
#pragma unroll
      for (int h = 0; h < NT; h += 8) {
        float x[8], A[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) x[p] = fmaf(c, P.x_a[h + p], fmaf(ssm, P.x_b[h + p], P.x_c));
        ipow_sel<(ZC > 0 ? ZC : 0), 8>(x, P.zeta, A);
#pragma unroll
        for (int q = 0; q < NRA; ++q)
          if (live >> q & 1)
#pragma unroll
            for (int p = 0; p < 8; ++p) acc[q * NT + h + p] = fmaf(A[p], R[q], acc[q * NT + h + p]);
      }
    }
  };
  if constexpr (MANY) {
    // many species-pair blocks of few triplets each: two blocks at a time,
    // one per half of the wave (off-diagonal blocks first, then diagonal
    // ones, so that the two are of like size).  With 4 species and 45
    // neighbors a block holds 66 or 128 triplets: 21 steps of the wave
    // instead of 26, and half as many sums over lanes.
    constexpr int E = NBW / 32 > 0 ? NBW / 32 : 1;
    const int hl = lane & 31, half = lane >> 5;
    const int nblk = S * (S + 1) / 2, noff = S * (S - 1) / 2;
    for (int p0 = 0; p0 < nblk; p0 += 2) {
      const int bi = p0 + half;
      int a = bi - noff, b = a;  // diagonal
      if (bi < noff) {
        a = 0;
        int rest = bi;
        while (rest >= S - 1 - a) {
          rest -= S - 1 - a;
          ++a;
        }
        b = a + 1 + rest;
      }
      const bool has = bi < nblk, same = a == b;
      if (!has) a = b = 0;
      const int sa = tr.seg[a], sb = tr.seg[b];
      const int na = tr.seg[a + 1] - sa, nbb = tr.seg[b + 1] - sb;
      const int T = !has ? 0 : same ? na * (na - 1) / 2 : na * nbb;
      const int Tmax = max(__builtin_amdgcn_readlane(T, 0), __builtin_amdgcn_readlane(T, 32));
      float acc[NBW];
#pragma unroll
      for (int x = 0; x < NBW; ++x) acc[x] = 0.f;
      StripRect rect;
      StripTri tri;
      rect.init(na, nbb, tw * 32 + hl);
      tri.init(na, tw * 32 + hl);
      for (int t0 = tw * 32; t0 < Tmax; t0 += 32 * TW) {
        const bool take = t0 + hl < T;
        int j = 0, k = 0;
        if (take) {
          if (same) {
            tri.at(j, k);
            tri.step(32 * TW);
          } else {
            rect.at(j, k);
            rect.step(32 * TW);
          }
        }
        triplet(take ? sa + j : 0, take ? sb + k : 0, take, acc);
      }
      float sums[E];
      half_sums<NBW>(acc, sums);
      float* out = ang + pair_block(S, a, b) * NB;
      if constexpr (TW == 1) {
        if (has && hl < NBW)
#pragma unroll
          for (int e = 0; e < E; ++e) out[bin(E * hl + e)] = sums[e];
      } else {
        if (hl < NB)
#pragma unroll
          for (int e = 0; e < E; ++e) xch[wv][half * NB + E * hl + e] = sums[e];
        __syncthreads();
        if (wv == 0 && has)
          for (int x = hl; x < NB; x += 32) {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < WPA; ++w) v += xch[w][half * NB + x];
            out[x] = v;
          }
        __syncthreads();
      }
    }
  } else {
    for (int a = 0; a < S; ++a) {
      for (int b = a; b < S; ++b, ang += NB) {
        const int sa = tr.seg[a], sb = tr.seg[b];
        const int na = tr.seg[a + 1] - sa, nbb = tr.seg[b + 1] - sb;
        const bool same = a == b;
        const int T = same ? na * (na - 1) / 2 : na * nbb;
        float acc[NBW];
#pragma unroll
        for (int x = 0; x < NBW; ++x) acc[x] = 0.f;
        StripRect rect;
        StripTri tri;
        if (same) tri.init(na, tw * kWave + lane);
        else rect.init(na, nbb, tw * kWave + lane);
        for (int t0 = tw * kWave; t0 < T; t0 += kWave * TW) {
          const bool take = t0 + lane < T;
          int j = 0, k = 0;
          if (same) {
            if (take) tri.at(j, k);
            tri.step(kWave * TW);
          } else {
            if (take) rect.at(j, k);
            rect.step(kWave * TW);
          }
          triplet(sa + j, sb + k, take, acc);
        }
#pragma unroll
        for (int h = 0; h < NBW / NS; ++h) {
          float part[NS];
#pragma unroll
          for (int x = 0; x < NS; ++x) part[x] = acc[h * NS + x];
          const float sum = wave_sums<NS>(part);
          if (lane < NS) {
            if constexpr (TW == 1) ang[bin(h * NS + lane)] = sum;
            else xch[wv][h * NS + lane] = sum;
          }
        }
        if constexpr (TW > 1) {
          __syncthreads();
          for (int x = tid; x < NB; x += 64 * WPA) {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < WPA; ++w) v += xch[w][x];
            ang[x] = v;
          }
          __syncthreads();
        }
      }
    }
  }
}

// Waves per SIMD that the registers of a wave's bins leave.  At these bounds the
// 8x8 passes keep up to 64 bytes a lane in scratch with three or more species, 20
// with fewer and several waves, and 128 bins 12 to 84: with three or more species
// six to nine accesses for each 64 triplets of a wave's loop, else none to two.
constexpr int fwd_waves(int NT, int NRA, int AS, bool MANY) {
  const int bins = NT * NRA / AS;
  return bins <= 32 ? 6 : bins > 64 ? 3 : NT == 8 || (AS == 2 && !MANY) ? 5 : 4;
}

template <int NT, int NRA, int WPA, int ZC, bool MANY, int AS = 1, int WAVES = fwd_waves(NT, NRA, AS, MANY)>
__global__ void __launch_bounds__(64 * WPA, WAVES) k_fwd_tiles(nn_system sys, const int64_t* __restrict__ offsets,
                                                        const int32_t* __restrict__ nbr,
                                                        const int8_t* __restrict__ shift, DescConst P,
                                                        float* __restrict__ G, int64_t* meta, IdentityGroup one,
                                                        const int32_t* __restrict__ order) {
  const bool list_ok = meta[kMetaValid] == 1;
  const int64_t i = atom_of_block(order, sys.n_atoms, list_ok);
  if (i < 0) return;
  if (one.perm && threadIdx.x == 0) identity_group(one, sys, i, meta);
  fwd_tiles_atom<NT, NRA, WPA, ZC, MANY, AS>(i, list_ok, sys, offsets, nbr, shift, P, G, meta);
}

// The atoms a packed launch leaves out (rows over kPackNb entries), one
// wave per block of 64 atom slots: the lanes test their slots' rows and the
// wave then takes the long ones one after another.  Also writes the
// identity grouping of all atoms.  Nothing else to do while the list is not
// valid (the packed launch zeroes every row then).
template <int NT, int NRA, int ZC, bool MANY>
__global__ void __launch_bounds__(64) k_fwd_tiles_long(nn_system sys, const int64_t* __restrict__ offsets,
                                                       const int32_t* __restrict__ nbr,
                                                       const int8_t* __restrict__ shift, DescConst P,
                                                       float* __restrict__ G, int64_t* meta, IdentityGroup one,
                                                       const int32_t* __restrict__ order) {
  const bool list_ok = meta[kMetaValid] == 1;
  const int64_t slot = (int64_t)blockIdx.x * kWave + threadIdx.x;
  const bool in = slot < sys.n_atoms;
  const int64_t i = !in ? -1 : (order && list_ok) ? (int64_t)order[slot] : slot;
  if (one.perm && in) identity_group(one, sys, i, meta);
  if (!list_ok) return;
  uint64_t m = __ballot(in && offsets[i + 1] - offsets[i] > kPackNb);
  while (m) {
    const int b = __ffsll((unsigned long long)m) - 1;
    m &= m - 1;
    fwd_tiles_atom<NT, NRA, 1, ZC, MANY>(__shfl(i, b), true, sys, offsets, nbr, shift, P, G, meta);
    __syncthreads();  // this atom's LDS reads are done before the next one's staging
  }
}

// ---------------------------------------------------------------------------
// adjoint
// ---------------------------------------------------------------------------

// Per-pair energy gradients dE_i/dd_e (float4 per entry, w unused) of atom i
// from lambda_i = dE_i/dG_i, by the block.
//
// The neighbors are sorted by distance alone (lambda's species-pair block is
// looked up per lane) and cut into blocks of eight.  A tile is the 64 pairs
// of two blocks, lane (row, col) taking neighbor `row` of the farther one
// and `col` of the nearer; the pairs inside a block go two blocks to a tile
// (32 lanes each, 28 pairs: neighbor col with col + s mod 8, s = 1 .. 4).  No
// index arithmetic, no lane idle but for the last block's padding (about
// 8 % of the slots at 81 neighbors), and a tile's gradients reduce within
// rows by DPP and across rows by permlane swaps: one read-add-write of a
// float4 per row neighbor and of a float per column neighbor and component,
// instead of one of each per step of a circular schedule.
//
// E_t = F2 sum_q R_q T_q with T_q = sum_p lambda_qp A_p: one pass over the
// radius terms forms T_q and its derivative along cos, sum_p lambda_qp A'_p,
// together, so a term that is screened out costs neither contraction.
template <int NT, int NRA, bool ONE_SPECIES, int WPA, int ZC>
__device__ __forceinline__ void adj_tiles_atom(int64_t i, const nn_system& sys, const int64_t* __restrict__ offsets,
                                               const int32_t* __restrict__ nbr, const int8_t* __restrict__ shift,
                                               const DescConst& P, const float* __restrict__ lambda,
                                               float4* __restrict__ pg, int64_t* meta) {
  constexpr int NB = NT * NRA;
  constexpr int NBP = NB + 4;  // padded block stride in LDS (bank spread)
  __shared__ TileRow tr;
  constexpr int KQ = NT == 16 || NRA == 4 ? 2 : 4;  // radius terms whose lambda is in flight at once
  __shared__ float4 nd[kMaxNb];       // unit vector, scaled distance
  __shared__ float4 nf[kMaxNb];       // fc, dfc/dr, 1/r, the species' parts of lambda's block offset
  __shared__ uint16_t ent[kMaxNb];    // list entry, from the row's first
  __shared__ float4 g4[WPA][kMaxNb];  // per wave: dE/dd of each slot; first the radial distance (hi, lo) of its octets
  __shared__ float2 rsg[kMaxRad];     // radial centres (hi, lo), scaled; kFar past n_rad
  // [S * n_rad] radial lambda, padded to a multiple of 4 floats, then the
  // angular blocks (16-byte aligned, read as float4); while staging, the keys
  extern __shared__ float4 dyn_lds4[];
  float* lam_r = reinterpret_cast<float*>(dyn_lds4);
  float* lam_a = lam_r + adj_lam_radial(P.S, P.n_rad);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = WPA > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
  const int row = lane >> 3, col = lane & 7;
  const int64_t e0 = offsets[i];
  // this atom's lambda is requested before the neighbor staging (whose
  // loads it then overlaps) and put into LDS after it
  const float* lam = lambda + i * (int64_t)P.D;
  constexpr int kLamPre = 8;
  float lpre[kLamPre];
#pragma unroll
  for (int q = 0; q < kLamPre; ++q) {
    const int d = tid + q * 64 * WPA;
    lpre[q] = d < P.D ? lam[d] : 0.f;
  }
  // block (a, b), a <= b, of lambda starts at f(a) + b blocks, f(a) = a (S - 1)
  // - a (a - 1) / 2; both parts in bytes grow with the species, so the pair's
  // are the minimum's low half and the maximum's high half
  auto species_word = [&](int sp) {
    return (uint32_t)(sp * NBP * 4) << 16 | (uint32_t)((sp * (P.S - 1) - sp * (sp - 1) / 2) * NBP * 4);
  };
  if (tid < kMaxRad)
    rsg[tid] = tid < P.n_rad ? make_float2(P.rs_rad_sc[tid], P.rs_rad_sc_lo[tid]) : make_float2(kFar, 0.f);
  stage_sorted<false>(tr, reinterpret_cast<uint32_t*>(dyn_lds4), i, sys, offsets, nbr, shift, P, meta, pg,
                      [&](int slot, int entry, int sp, const PairRec& p) {
                        nd[slot] = make_float4(p.ux, p.uy, p.uz, p.ra);
                        nf[slot] = make_float4(p.fc, p.dfc, p.ir, __uint_as_float(species_word(sp)));
                        ent[slot] = (uint16_t)entry;
                        g4[(slot >> 3) % WPA][slot] = make_float4(p.rr, p.rr_lo, 0.f, 0.f);
                      });
  if (tr.bad) {
    for (int64_t e = e0 + tid; e < offsets[i + 1]; e += 64 * WPA) pg[e] = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  const int S = P.S;
  const int n = tr.n, nblk = (n + 7) >> 3;
  const int ang0 = P.n_rad * S;
  // An infinite or NaN lambda reaches every neighbor through its term, however
  // small: with one, no term is left out.
  float watch = 0.f;  // NaN once such a lambda was seen
  auto put_lam = [&](int d, float x) {
    watch = fmaf(x, 0.f, watch);
    if (d < ang0) {
      lam_r[d] = x;
    } else {
      const int da = d - ang0;
      lam_a[(da / NB) * NBP + da % NB] = x;
    }
  };
#pragma unroll
  for (int q = 0; q < kLamPre; ++q) {
    const int d = tid + q * 64 * WPA;
    if (d < P.D) put_lam(d, lpre[q]);
  }
  for (int d = tid + kLamPre * 64 * WPA; d < P.D; d += 64 * WPA) put_lam(d, lam[d]);
  // the last block's empty slots: no cutoff, so no gradient, and beyond
  // every radius term
  if (tid < 8 * nblk - n) {
    nd[n + tid] = make_float4(0.f, 0.f, 0.f, kFar);
    nf[n + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (__any(watch != 0.f) && lane == 0) tr.all = 1;
  __syncthreads();
  const bool all = __builtin_amdgcn_readfirstlane(tr.all) != 0;
  // without smoothing the sine has no derivative where two neighbors lie on a
  // line with the atom: 1/r of both becomes NaN, and with it their gradients
  if (P.eps_ang == 0.f) {
    for (int t = tid; t < n * n; t += 64 * WPA) {
      const int j = t / n, k = t % n;
      const float4 u = nd[j], v = nd[k];
      const float cx = fmaf(u.y, v.z, -u.z * v.y), cy = fmaf(u.z, v.x, -u.x * v.z), cz = fmaf(u.x, v.y, -u.y * v.x);
      if (j != k && fmaf(cx, cx, fmaf(cy, cy, cz * cz)) == 0.f && nf[j].x * nf[k].x != 0.f) nf[j].z = __builtin_nanf("");
    }
    __syncthreads();
  }
  // radial: eight neighbors at a time (wave w: octets w, w + WPA, ...),
  // eight lanes each with every eighth bin; dE/dd = (dE/dr) d/r.  The other
  // waves' octets start from zero.
  for (int b = 0; b < nblk; ++b) {
    const int t = 8 * b + row;
    float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
    if (b % WPA == wv) {
      const bool in = t < n;
      const float4 rr = g4[wv][t], fu = nf[t], u = nd[t];
      const float r = in ? rr.x : -kFar, r_lo = in ? rr.y : 0.f;
      const float* lr = lam_r + (int)((__float_as_uint(fu.w) >> 16) / (NBP * 4)) * P.n_rad;
      float gr = 0.f;
      for (int k0 = 0; k0 < P.n_rad; k0 += 8) {
        const int k = k0 + col;
        const float2 rs = rsg[k];
        const float d0 = r - rs.x;
        if (all || __any(fabsf(d0) < kScreen)) {
          const float dr = d0 + (r_lo - rs.y);
          const float gk = (in && k < P.n_rad) ? lr[k] * fexp2(-dr * dr) : 0.f;
          gr = fmaf(gk, fmaf(P.drr * dr, fu.x, fu.y), gr);
        }
      }
      gr += dpp_f<kDppXor1>(gr);
      gr += dpp_f<kDppXor2>(gr);
      gr += dpp_f<kDppMirror8>(gr);
      g = make_float4(gr * u.x, gr * u.y, gr * u.z, 0.f);
    }
    if (col == 0) g4[wv][t] = g;
  }
  wave_lds_order();
  const int zeta1 = P.zeta - 1;
  const float zf = (float)P.zeta;
  const float rsv = lane < NRA ? P.rs_ang_sc[lane < NRA ? lane : 0] : -kFar;  // lane q: centre of radius term q
  // the radius terms within kScreen of [lo, hi]: one bit each
  const uint32_t every = all ? (1u << NRA) - 1 : 0u;
  auto in_reach = [&](float lo, float hi) {
    return (uint32_t)__ballot(hi > rsv - kReach && lo < rsv + kReach) | every;
  };
  // one triplet: the coefficients of its gradients g_j = cu v + au u and
  // g_k = cv u + av v (u, v the unit vectors)
  auto triplet = [&](const float4& u, const float4& fu, const float4& v, const float4& fv, float rb, uint32_t terms,
                     float& cu, float& au, float& cv, float& av) {
    const float* La = lam_a;
    if (!ONE_SPECIES) {
      // first index of the species pair's block: f(min) + max, both in one word
      const uint32_t wa = __float_as_uint(fu.w), wb = __float_as_uint(fv.w);
      La = reinterpret_cast<const float*>(reinterpret_cast<const char*>(lam_a) + (min(wa, wb) & 0xffffu) +
                                          (max(wa, wb) >> 16));
    }
    const int q0 = terms ? min(__builtin_ctz(terms), NRA - KQ) : 0;
    const int q1 = terms ? 31 - __builtin_clz(terms) : -1;
    const float4* La4 = reinterpret_cast<const float4*>(La) + q0 * (NT / 4);  // 16-byte aligned: NBP is a multiple of 4
    // the first KQ radius terms' lambda is requested before the powers
    float4 l4[KQ][NT / 4];
#pragma unroll
    for (int q = 0; q < KQ; ++q)
#pragma unroll
      for (int p = 0; p < NT / 4; ++p) l4[q][p] = La4[q * (NT / 4) + p];
    const float c = fmaf(u.x, v.x, fmaf(u.y, v.y, u.z * v.z));
    const float cx = fmaf(u.y, v.z, -u.z * v.y), cy = fmaf(u.z, v.x, -u.x * v.z), cz = fmaf(u.x, v.y, -u.y * v.x);
    const float ssm = __builtin_amdgcn_sqrtf(fmaf(cx, cx, fmaf(cy, cy, fmaf(cz, cz, P.eps_tile))));
    float x[NT], A[NT], Ad[NT];
#pragma unroll
    for (int p = 0; p < NT; ++p) x[p] = fmaf(c, P.x_a[p], fmaf(ssm, P.x_b[p], P.x_c));
    ipow_sel<(ZC > 0 ? ZC - 1 : 0), NT>(x, zeta1, Ad);
    // sin^2 = 1 - cos^2, so d ssm / d cos = -cos / ssm, and dA/dcos = zeta x^(zeta-1) (x_a + x_b d ssm/d cos)
    const float ds = -c * frcp(ssm);
#pragma unroll
    for (int p = 0; p < NT; ++p) {
      A[p] = Ad[p] * x[p];
      Ad[p] *= fmaf(ds, P.x_b[p], P.x_a[p]);
    }
    float S0 = 0.f, Sr = 0.f, Sc = 0.f;  // sums of R T, R T dq, R T'
    auto term = [&](const float4 (&l)[NT / 4], int q) {
      // the gradient does not need the low parts of the average radius
      const float dq = rb - __int_as_float(__builtin_amdgcn_readlane(__float_as_int(rsv), q));
      const float R = fexp2(-dq * dq);
      float t0 = 0.f, t1 = 0.f;
#pragma unroll
      for (int p = 0; p < NT / 4; ++p) {
        t0 = fmaf(l[p].x, A[4 * p], t0);
        t1 = fmaf(l[p].x, Ad[4 * p], t1);
        t0 = fmaf(l[p].y, A[4 * p + 1], t0);
        t1 = fmaf(l[p].y, Ad[4 * p + 1], t1);
        t0 = fmaf(l[p].z, A[4 * p + 2], t0);
        t1 = fmaf(l[p].z, Ad[4 * p + 2], t1);
        t0 = fmaf(l[p].w, A[4 * p + 3], t0);
        t1 = fmaf(l[p].w, Ad[4 * p + 3], t1);
      }
      const float rt = R * t0;
      S0 += rt;
      Sr = fmaf(rt, dq, Sr);
      Sc = fmaf(R, t1, Sc);
    };
#pragma unroll
    for (int q = 0; q < KQ; ++q) term(l4[q], q0 + q);
    for (int q = q0 + KQ; q <= q1; ++q) {
      float4 l[NT / 4];
#pragma unroll
      for (int p = 0; p < NT / 4; ++p) l[p] = La4[(q - q0) * (NT / 4) + p];
      term(l, q);
    }
    const float F2 = 2.0f * fu.x * fv.x;
    const float half = P.dravg * F2 * Sr;  // half of dE/drbar: drbar/dr = 1/2
    const float coef = Sc * zf * F2;
    // d cos / d d_u = (v^ - cos u^) / r_u
    cu = coef * fu.z;
    cv = coef * fv.z;
    au = fmaf(-cu, c, fmaf(2.0f * S0, fu.y * fv.x, half));
    av = fmaf(-cv, c, fmaf(2.0f * S0, fu.x * fv.y, half));
  };
  // pairs inside a block, two blocks at a time
  const int ndiag = (nblk + 1) >> 1;
  const int step = (row & 3) + 1;
  for (int d = wv; d < ndiag; d += WPA) {
    const int base = 8 * (2 * d + (lane >> 5));
    const int j = base + col, k = base + ((col + step) & 7);
    const bool take = j < n && k < n && (step < 4 || col < 4);
    const int js = take ? j : 0, ks = take ? k : 0;
    const float4 u = nd[js], fu = nf[js], v = nd[ks], fv = nf[ks];
    float cu, au, cv, av;
    // the distances of the two blocks run from the first neighbor of the
    // first to the last of the second
    const float lo = 2.0f * nd[16 * d].w, hi = 2.0f * nd[min(16 * d + 15, n - 1)].w;
    triplet(u, fu, v, fv, u.w + v.w, in_reach(lo, hi), cu, au, cv, av);
    if (!take) cu = au = cv = av = 0.f;
    // k's gradient to the lane of column k, then over the four steps
    const int from = ((lane & 56) | ((col - step) & 7)) << 2;
    const float gk[3] = {fmaf(cv, u.x, av * v.x), fmaf(cv, u.y, av * v.y), fmaf(cv, u.z, av * v.z)};
    const float gj[3] = {fmaf(cu, v.x, au * u.x), fmaf(cu, v.y, au * u.y), fmaf(cu, v.z, au * u.z)};
    float s[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      const float y = gj[x] + __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(gk[x])));
      s[x] = y + dpp_f<kDppRor8>(y);
    }
    const float xy = fold16(s[0], s[1]), z = fold16(s[2], s[2]);  // x in even rows of 16 lanes, y in odd ones
    if (j < n && (lane & 8) == 0) {
      float* g = reinterpret_cast<float*>(&g4[wv][j]);
      if (lane & 16) {
        g[1] += xy;
      } else {
        g[0] += xy;
        g[2] += z;
      }
    }
    wave_lds_order();
  }
  // tiles of two blocks c < m, strip by strip: column neighbor k stays in
  // registers and so does its gradient.  Wave w takes the tiles w, w + WPA,
  // ... of the strips laid end to end.  The next tile's records are requested
  // before this one's gradients are reduced, and its radius terms are known
  // before its powers, behind which lambda's loads then hide.
  // A last block of at most four neighbors is left to the tiles below.
  const int left = n & 7;
  const bool half_last = nblk > 1 && left >= 1 && left <= 4;
  const int nfull = half_last ? nblk - 1 : nblk;
  int c = 0, m = 1 + wv;
  auto settle = [&]() {  // (c, m) past the end of strip c: into the next ones
    while (m >= nfull && c < nfull - 1) {
      m += c + 2 - nfull;
      ++c;
    }
  };
  settle();
  if (c < nfull - 1) {
    float4 u = nd[8 * m + row], fu = nf[8 * m + row], v = nd[8 * c + col], fv = nf[8 * c + col];
    float gk[3] = {0.f, 0.f, 0.f};
    while (true) {
      const float rb = u.w + v.w;
      // sorted: lane 0 has the smallest average radius and the last lane with a neighbor the largest
      const uint32_t terms =
          in_reach(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(rb), 0)),
                   __int_as_float(__builtin_amdgcn_readlane(__float_as_int(rb), min(63, 8 * (n - 1 - 8 * m) + 7))));
      float4* gp = &g4[wv][8 * m + row];
      float4 g = *gp;
      float cu, au, cv, av;
      triplet(u, fu, v, fv, rb, terms, cu, au, cv, av);
      gk[0] = fmaf(cv, u.x, fmaf(av, v.x, gk[0]));
      gk[1] = fmaf(cv, u.y, fmaf(av, v.y, gk[1]));
      gk[2] = fmaf(cv, u.z, fmaf(av, v.z, gk[2]));
      float gj[3] = {fmaf(cu, v.x, au * u.x), fmaf(cu, v.y, au * u.y), fmaf(cu, v.z, au * u.z)};
      const int c0 = c;
      m += WPA;
      settle();
      const bool more = c < nfull - 1;
      if (more) {
        u = nd[8 * m + row];
        fu = nf[8 * m + row];
        if (c != c0) {
          v = nd[8 * c + col];
          fv = nf[8 * c + col];
        }
      }
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        gj[x] += dpp_f<kDppXor1>(gj[x]);
        gj[x] += dpp_f<kDppXor2>(gj[x]);
        gj[x] += dpp_f<kDppMirror8>(gj[x]);
      }
      g.x += gj[0];
      g.y += gj[1];
      g.z += gj[2];
      if (col == 0) *gp = g;
      wave_lds_order();
      if (c != c0) {
        // k's sums: x, y, z of column (lane & 7) in rows 0, 1, 2 of 16 lanes
        float s[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) {
          s[x] = gk[x] + dpp_f<kDppRor8>(gk[x]);
          gk[x] = 0.f;
        }
        const float xyz = fold32(fold16(s[0], s[1]), fold16(s[2], s[2]));
        const int comp = lane >> 4;
        if (comp < 3 && (lane & 8) == 0) reinterpret_cast<float*>(&g4[wv][8 * c0 + col])[comp] += xyz;
        wave_lds_order();
      }
      if (!more) break;
    }
  }
  // the at most four neighbors of the last block against two strips at a
  // time: rows 0-3 of lanes the first strip, 4-7 the second (the tiles of
  // 52 neighbors go from 25 to 22)
  if (half_last)
    for (int p = wv; 2 * p < nfull; p += WPA) {
      const int cc = 2 * p + (row >> 2);
      const bool has = cc < nfull;
      const int j = 8 * nfull + (row & 3), k = has ? 8 * cc + col : 8 * nblk - 1;  // else an empty slot
      const float4 u = nd[j], fu = nf[j], v = nd[k], fv = nf[k];
      const float lo = nd[8 * nfull].w + nd[16 * p].w, hi = nd[n - 1].w + nd[min(16 * p + 15, 8 * nfull - 1)].w;
      float cu, au, cv, av;
      triplet(u, fu, v, fv, u.w + v.w, in_reach(lo, hi), cu, au, cv, av);
      const float gk[3] = {fmaf(cv, u.x, av * v.x), fmaf(cv, u.y, av * v.y), fmaf(cv, u.z, av * v.z)};
      float gj[3] = {fmaf(cu, v.x, au * u.x), fmaf(cu, v.y, au * u.y), fmaf(cu, v.z, au * u.z)};
      float s[3];
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        gj[x] += dpp_f<kDppXor1>(gj[x]);
        gj[x] += dpp_f<kDppXor2>(gj[x]);
        gj[x] += dpp_f<kDppMirror8>(gj[x]);
        gj[x] = fold32(gj[x], gj[x]);
        s[x] = gk[x] + dpp_f<kDppRor8>(gk[x]);
      }
      const float xy = fold16(s[0], s[1]), z = fold16(s[2], s[2]);
      if (col == 0 && row < 4) {
        float4 g = g4[wv][j];
        g.x += gj[0];
        g.y += gj[1];
        g.z += gj[2];
        g4[wv][j] = g;
      }
      if (has && (lane & 8) == 0) {
        float* g = reinterpret_cast<float*>(&g4[wv][k]);
        if (lane & 16) {
          g[1] += xy;
        } else {
          g[0] += xy;
          g[2] += z;
        }
      }
      wave_lds_order();
    }
  __syncthreads();
  for (int t = tid; t < n; t += 64 * WPA) {
    float x = 0.f, y = 0.f, z = 0.f;
#pragma unroll
    for (int w = 0; w < WPA; ++w) {
      const float4 a = g4[w][t];
      x += a.x;
      y += a.y;
      z += a.z;
    }
    pg[e0 + ent[t]] = make_float4(x, y, z, 0.f);
  }
}

// Two or more waves an atom share its records, and the LDS then holds six
// waves per SIMD: 80 registers each (the same loop takes 97 unasked, 5 waves
// per SIMD: 812 against 774 us for 65536 atoms of 52 neighbors).  8x4 bins of one
// species then keep 20 bytes a lane in scratch.
template <int NT, int NRA, bool ONE_SPECIES, int WPA, int ZC>
__global__ void __launch_bounds__(64 * WPA, WPA > 1 && NT <= 8 ? (ZC > 0 ? 6 : 5) : 4) k_adj_tiles(nn_system sys, const int64_t* __restrict__ offsets,
                                                        const int32_t* __restrict__ nbr,
                                                        const int8_t* __restrict__ shift, DescConst P,
                                                        const float* __restrict__ lambda, float4* __restrict__ pg,
                                                        int64_t* meta, const int32_t* __restrict__ order) {
  if (meta[kMetaValid] != 1) return;  // no valid list: the gather writes zero forces
  const int64_t i = atom_of_block(order, sys.n_atoms, true);
  if (i < 0) return;
  adj_tiles_atom<NT, NRA, ONE_SPECIES, WPA, ZC>(i, sys, offsets, nbr, shift, P, lambda, pg, meta);
}

// The atoms a packed adjoint leaves out (rows over kPackNb entries), as in
// k_fwd_tiles_long.
template <int NT, int NRA, bool ONE_SPECIES, int ZC>
__global__ void __launch_bounds__(64) k_adj_tiles_long(nn_system sys, const int64_t* __restrict__ offsets,
                                                       const int32_t* __restrict__ nbr,
                                                       const int8_t* __restrict__ shift, DescConst P,
                                                       const float* __restrict__ lambda, float4* __restrict__ pg,
                                                       int64_t* meta, const int32_t* __restrict__ order) {
  if (meta[kMetaValid] != 1) return;
  const int64_t slot = (int64_t)blockIdx.x * kWave + threadIdx.x;
  const bool in = slot < sys.n_atoms;
  const int64_t i = !in ? -1 : order ? (int64_t)order[slot] : slot;
  uint64_t m = __ballot(in && offsets[i + 1] - offsets[i] > kPackNb);
  while (m) {
    const int b = __ffsll((unsigned long long)m) - 1;
    m &= m - 1;
    adj_tiles_atom<NT, NRA, ONE_SPECIES, 1, ZC>(__shfl(i, b), sys, offsets, nbr, shift, P, lambda, pg, meta);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

template <int NT, int NRA, int WPA, int ZC, bool MANY, int... SHARE>
static void fwd_w(const nn_system& sys, const nn_nlist& nl, const DescConst& P, float* G, IdentityGroup one,
                  hipStream_t s) {
  hipLaunchKernelGGL((k_fwd_tiles<NT, NRA, WPA, ZC, MANY, SHARE...>), dim3(atom_grid(sys.n_atoms, nl.order)),
                     dim3(64 * WPA), 0, s, sys, nl.offsets, nl.nbr, nl.shift, P, G, nl.meta, one, nl.order);
}

// Two waves an atom.  16x8 bins: the triplets shared while three waves for each of
// the 1024 SIMDs hold them all, else the terms; three or more species share the
// terms at every count, since their pair blocks have few triplets to share (four
// species 44 us at 1024 atoms, with one wave 67, before 54).  Up to 2048 atoms four
// waves per SIMD do: where a fifth fits, some SIMDs get five and others
// three (after a list build 42 us at 2048 atoms); where only four do, each gets its
// share (38 us).  More atoms need the fifth: 42 against 47 us at 2064.
template <int NT, int NRA, int ZC, bool MANY>
static void fwd_two(const nn_system& sys, const nn_nlist& nl, const DescConst& P, float* G, IdentityGroup one,
                    hipStream_t s) {
  if constexpr (NT * NRA == 128) {
    if (MANY) fwd_w<NT, NRA, 2, ZC, MANY, 2>(sys, nl, P, G, one, s);
    else if (sys.n_atoms <= 1536) fwd_w<NT, NRA, 2, ZC, MANY, 1>(sys, nl, P, G, one, s);
    else if (sys.n_atoms <= 2048) fwd_w<NT, NRA, 2, ZC, MANY, 2, 4>(sys, nl, P, G, one, s);
    else fwd_w<NT, NRA, 2, ZC, MANY, 2>(sys, nl, P, G, one, s);
  } else {
    fwd_w<NT, NRA, 2, ZC, MANY>(sys, nl, P, G, one, s);
  }
}

template <int NT, int NRA, int ZC, bool MANY>
static void fwd_z(const nn_system& sys, const nn_nlist& nl, const DescConst& P, float* G, IdentityGroup one, int wpa,
                  hipStream_t s) {
  if (wpa == 0)
    hipLaunchKernelGGL((k_fwd_tiles_long<NT, NRA, ZC, MANY>), dim3((unsigned)((sys.n_atoms + kWave - 1) / kWave)), dim3(64),
                       0, s, sys, nl.offsets, nl.nbr, nl.shift, P, G, nl.meta, one, nl.order);
  else if (wpa == 4) fwd_w<NT, NRA, 4, ZC, MANY>(sys, nl, P, G, one, s);
  else if (wpa == 2) fwd_two<NT, NRA, ZC, MANY>(sys, nl, P, G, one, s);
  else fwd_w<NT, NRA, 1, ZC, MANY>(sys, nl, P, G, one, s);
}

static size_t adj_lds(const DescConst& P) {
  const int lam = adj_lam_radial(P.S, P.n_rad) + P.S * (P.S + 1) / 2 * (P.n_theta * P.n_rs_ang + 4);
  return sizeof(float) * (size_t)(lam > kKeyWords ? lam : kKeyWords);
}

template <int NT, int NRA, bool ONE, int WPA, int ZC>
static void adj_w(const nn_system& sys, const nn_nlist& nl, const DescConst& P, const float* lam, float4* pg,
                  hipStream_t s) {
  hipLaunchKernelGGL((k_adj_tiles<NT, NRA, ONE, WPA, ZC>), dim3(atom_grid(sys.n_atoms, nl.order)), dim3(64 * WPA),
                     adj_lds(P), s, sys, nl.offsets, nl.nbr, nl.shift, P, lam, pg, nl.meta, nl.order);
}

template <int NT, int NRA, bool ONE, int ZC>
static void adj_z(const nn_system& sys, const nn_nlist& nl, const DescConst& P, const float* lam, float4* pg, int wpa,
                  hipStream_t s) {
  if (wpa == 0)
    hipLaunchKernelGGL((k_adj_tiles_long<NT, NRA, ONE, ZC>), dim3((unsigned)((sys.n_atoms + kWave - 1) / kWave)),
                       dim3(64), adj_lds(P), s, sys, nl.offsets, nl.nbr, nl.shift, P, lam, pg, nl.meta, nl.order);
  else if (wpa == 4) adj_w<NT, NRA, ONE, 4, ZC>(sys, nl, P, lam, pg, s);
  else if (wpa == 2) adj_w<NT, NRA, ONE, 2, ZC>(sys, nl, P, lam, pg, s);
  else adj_w<NT, NRA, ONE, 1, ZC>(sys, nl, P, lam, pg, s);
}

void launch_fwd_tiles(const nn_system& sys, const nn_nlist& nl, const DescConst& P, float* G, IdentityGroup one,
                      int wpa, hipStream_t s) {
  const int nt = P.n_theta, nra = P.n_rs_ang;
  if (P.S >= 3) {
    if (P.zeta == 50) NNP_DISPATCH(A, B, (fwd_z<A, B, 50, true>(sys, nl, P, G, one, wpa, s)));
    else NNP_DISPATCH(A, B, (fwd_z<A, B, 0, true>(sys, nl, P, G, one, wpa, s)));
  } else {
    if (P.zeta == 50) NNP_DISPATCH(A, B, (fwd_z<A, B, 50, false>(sys, nl, P, G, one, wpa, s)));
    else NNP_DISPATCH(A, B, (fwd_z<A, B, 0, false>(sys, nl, P, G, one, wpa, s)));
  }
}

void launch_adj_tiles(const nn_system& sys, const nn_nlist& nl, const DescConst& P, const float* lam, float4* pg,
                      int wpa, hipStream_t s) {
  const int nt = P.n_theta, nra = P.n_rs_ang;
  if (P.S == 1) {
    if (P.zeta == 50) NNP_DISPATCH(A, B, (adj_z<A, B, true, 50>(sys, nl, P, lam, pg, wpa, s)));
    else NNP_DISPATCH(A, B, (adj_z<A, B, true, 0>(sys, nl, P, lam, pg, wpa, s)));
  } else {
    if (P.zeta == 50) NNP_DISPATCH(A, B, (adj_z<A, B, false, 50>(sys, nl, P, lam, pg, wpa, s)));
    else NNP_DISPATCH(A, B, (adj_z<A, B, false, 0>(sys, nl, P, lam, pg, wpa, s)));
  }
}

}  // namespace nnp
