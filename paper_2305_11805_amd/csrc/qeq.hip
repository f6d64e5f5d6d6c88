// Charge equilibration of Sec. II.B on the device, one structure per wave.
//
// The network gives each atom the coefficients of a second-order expansion of
// its energy in its charge: E0_i, chi_i, J_i.  With Gaussian charges of width
// sigma (per species) the electrostatic energy is a quadratic form, and the
// charges minimise
//   E(q) = sum_i E0_i + chi . q + q^T A q / 2,
//   A_ij = k_e erf(r_ij / (sqrt(2) gamma_ij)) / r_ij  (i != j),
//   A_ii = J_i + k_e / (sigma_i sqrt(pi)),   gamma_ij^2 = sigma_i^2 + sigma_j^2,
// subject to sum_i q_i = Q (the structure's total charge): q = y + mu z with
// A y = -chi, A z = 1 and mu = (Q - sum y) / sum z, every atom at chemical
// potential dE/dq_i = mu, and E = sum E0 + chi . q / 2 + mu Q / 2.
//
// A wave assembles A in LDS in FP64 (lower triangle, packed), factors it by
// Cholesky (A is the Coulomb matrix of Gaussian charges, positive definite,
// plus the hardnesses on the diagonal; a pivot <= 0 is reported) with lane i
// on row i and both right sides in registers, and writes the charges, the
// energy and the output seeds (1, q, q^2 / 2) with which the network's
// backward pass gives the forces at fixed charges (the minimum makes the
// derivative of the solve drop out).  The Coulomb part of the forces follows
// while the positions are at hand.  Every sum has a fixed order, so results
// are the same on every run.
//
// The chain of n pivots bounds it, n^2 / 2 multiply-adds a lane; what it has
// to avoid is waiting at block barriers between them and idle lanes in the
// FP64 erf and exp of the pairs.  A block of 256 threads per structure with
// a barrier per elimination step, and a thread per atom for the Coulomb
// forces, took 121 + 45 us for 4096 structures of 16 and 17 atoms; a wave
// per structure, pairs dealt to all lanes, takes 35 us for both.
#include <math.h>

#include "common.h"

namespace nnp {

// Structures of up to kQeqSmall atoms keep their triangle in 4 KB, and four
// waves per SIMD are resident (one kernel for both, at 17 KB and two waves
// per SIMD, took 57 us); the larger ones are taken by a second launch, whose
// waves leave at once where there are none.
constexpr int kQeqSmall = 32;
constexpr int kQeqPairs = 4;  // pairs per lane whose erf is kept for the forces

__device__ __forceinline__ bool qeq_struct_ok(const QeqArgs& a, int c, int64_t a0, int64_t n) {
  const uint8_t* pb = a.pbc + 3 * (int64_t)c;
  return n <= kQeqMax && pb[0] == 0 && pb[1] == 0 && pb[2] == 0;
}

// This wave's LDS accesses in program order (served in the order issued).
__device__ __forceinline__ void qeq_order() { __asm__ volatile("" ::: "memory"); }

__device__ __forceinline__ double lane_value(double x, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Row of element e of a lower triangle packed row by row (row i starts at
// i (i + 1) / 2).
__device__ __forceinline__ int tri_row(int e) {
  int i = (int)((__builtin_amdgcn_sqrtf(fmaf(8.0f, (float)e, 1.0f)) - 1.0f) * 0.5f);
  if (i * (i + 1) / 2 > e) --i;
  if ((i + 1) * (i + 2) / 2 <= e) ++i;
  return i;
}

template <int NMAX>
struct QeqLds {
  double A[NMAX * (NMAX + 1) / 2];
  double x[NMAX][3];
  double sig[NMAX];
  double h[NMAX];  // hardness, then charge
};

// Fc (may be null): the Coulomb forces [N][3].  It may be a.out: a structure's
// outputs are read before its forces are written.
template <int NMAX, int WAVES>
__global__ void __launch_bounds__(64 * WAVES, NMAX <= 32 ? 4 : 2) k_qeq_solve(QeqArgs a, float* Fc) {
  __shared__ QeqLds<NMAX> lds[WAVES];
  const int lane = threadIdx.x & 63;
  const int c = blockIdx.x * WAVES + (threadIdx.x >> 6);
  if (c >= a.B) return;  // no block barriers below
  QeqLds<NMAX>& m = lds[threadIdx.x >> 6];
  const int64_t a0 = a.atom_ptr[c], a1 = a.atom_ptr[c + 1];
  const int64_t n64 = a1 - a0;
  const bool larger = n64 > kQeqSmall && qeq_struct_ok(a, c, a0, n64);
  if (larger != (NMAX > kQeqSmall)) return;  // the other launch's
  if (n64 <= 0) {
    if (lane == 0) a.E_struct[c] = 0.0;
    return;
  }
  if (!qeq_struct_ok(a, c, a0, n64)) {
    for (int64_t i = a0 + lane; i < a1; i += 64) {
      a.q[i] = 0.0;
      a.seed[3 * i] = 1.f;
      a.seed[3 * i + 1] = 0.f;
      a.seed[3 * i + 2] = 0.f;
      if (Fc) Fc[3 * i] = Fc[3 * i + 1] = Fc[3 * i + 2] = 0.f;
    }
    if (lane == 0) {
      a.E_struct[c] = 0.0;
      atomicOr((unsigned long long*)&a.meta[kMetaErr], (unsigned long long)kErrQeq);
    }
    return;
  }
  const int n = (int)n64;
  const bool in = lane < n;
  const int64_t g = a0 + lane;
  double e0 = 0.0, chi = 0.0;
  if (in) {
    for (int k = 0; k < 3; ++k) m.x[lane][k] = a.pos[3 * g + k];
    m.sig[lane] = a.sigma[a.species[g]];
    e0 = (double)a.out[3 * g];
    chi = (double)a.out[3 * g + 1];
    m.h[lane] = (double)a.out[3 * g + 2];
  }
  qeq_order();
  const double rsqpi = 0.56418958354775628;  // 1 / sqrt(pi)
  // the pairs i > j over the lanes (pair e = i (i - 1) / 2 + j); the first
  // kQeqPairs of a lane keep erf(r / g) for the forces
  const int pairs = n * (n - 1) / 2;
  auto pair_of = [&](int e, int& i, int& j, double& dx, double& dy, double& dz, double& r, double& gw) {
    i = tri_row(e) + 1;
    j = e - i * (i - 1) / 2;
    dx = m.x[i][0] - m.x[j][0];
    dy = m.x[i][1] - m.x[j][1];
    dz = m.x[i][2] - m.x[j][2];
    r = sqrt(dx * dx + dy * dy + dz * dz);
    const double si = m.sig[i], sj = m.sig[j];
    gw = sqrt(2.0 * (si * si + sj * sj));
  };
  auto coupling = [&](int e) {
    int i, j;
    double dx, dy, dz, r, gw;
    pair_of(e, i, j, dx, dy, dz, r, gw);
    const double w = erf(r / gw);
    m.A[i * (i + 1) / 2 + j] = a.ke * w / r;
    return w;
  };
  double kept[kQeqPairs];
#pragma unroll
  for (int q = 0; q < kQeqPairs; ++q) {
    kept[q] = 0.0;
    if (lane + 64 * q < pairs) kept[q] = coupling(lane + 64 * q);
  }
  for (int e = lane + 64 * kQeqPairs; e < pairs; e += 64) coupling(e);
  if (in) m.A[lane * (lane + 1) / 2 + lane] = m.h[lane] + a.ke * rsqpi / m.sig[lane];
  qeq_order();
  // A = L L^T column by column, lane i on row i; L u = b (b = -chi and 1)
  // alongside, u_j being known with column j
  const int row = lane * (lane + 1) / 2;
  double y = -chi, z = 1.0, inv = 1.0;
  bool bad = false;
  for (int j = 0; j < n; ++j) {
    const int rj = j * (j + 1) / 2;
    const bool on = in && lane >= j;
    double s0 = 0.0, s1 = 0.0;
    if (on) {
      s0 = m.A[row + j];
      int k = 0;
      for (; k + 4 <= j; k += 4) {
        s0 = fma(-m.A[row + k], m.A[rj + k], s0);
        s1 = fma(-m.A[row + k + 1], m.A[rj + k + 1], s1);
        s0 = fma(-m.A[row + k + 2], m.A[rj + k + 2], s0);
        s1 = fma(-m.A[row + k + 3], m.A[rj + k + 3], s1);
      }
      for (; k < j; ++k) s0 = fma(-m.A[row + k], m.A[rj + k], s0);
    }
    const double s = s0 + s1;
    const double d = lane_value(s, j);
    if (!(d > 0.0)) bad = true;
    const double piv = d > 0.0 ? sqrt(d) : 1.0;
    const double ip = 1.0 / piv;
    const double l = lane == j ? piv : s * ip;
    if (on) m.A[row + j] = l;
    const double yj = lane_value(y, j) * ip, zj = lane_value(z, j) * ip;
    if (lane == j) {
      y = yj;
      z = zj;
      inv = ip;
    } else if (on) {
      y = fma(-l, yj, y);
      z = fma(-l, zj, z);
    }
    qeq_order();
  }
  // L^T v = u, both right sides at once
  for (int j = n - 1; j >= 0; --j) {
    const double ip = lane_value(inv, j);
    const double yj = lane_value(y, j) * ip, zj = lane_value(z, j) * ip;
    if (lane == j) {
      y = yj;
      z = zj;
    } else if (lane < j) {
      const double l = m.A[j * (j + 1) / 2 + lane];  // (L^T)_ij = L_ji
      y = fma(-l, yj, y);
      z = fma(-l, zj, z);
    }
  }
  const double sy = wave_sum(in ? y : 0.0), sz = wave_sum(in ? z : 0.0);
  const double Q = a.total[c];
  const double mu = (Q - sy) / sz;
  const double qi = bad || !in ? 0.0 : y + mu * z;
  if (in) {
    a.q[g] = qi;
    a.seed[3 * g] = 1.f;
    a.seed[3 * g + 1] = (float)qi;
    a.seed[3 * g + 2] = (float)(0.5 * qi * qi);
    m.h[lane] = qi;
  }
  const double E0 = wave_sum(e0), cq = wave_sum(in ? chi * qi : 0.0);
  if (lane == 0) {
    a.E_struct[c] = bad ? 0.0 : E0 + 0.5 * cq + 0.5 * mu * Q;
    if (bad) atomicOr((unsigned long long*)&a.meta[kMetaErr], (unsigned long long)kErrQeq);
  }
  if (!Fc) return;
  // F_i = -sum_{j != i} k_e q_i q_j f'(r_ij) (x_i - x_j) / r_ij with
  // f(r) = erf(r / g) / r, g = sqrt(2 (sigma_i^2 + sigma_j^2)): each pair's
  // factor once, pairs over the lanes, then lane i sums over j in order
  qeq_order();
  const double tsqpi = 1.1283791670955126;  // 2 / sqrt(pi)
  auto factor = [&](int e, bool known, double w) {
    int i, j;
    double dx, dy, dz, r, gw;
    pair_of(e, i, j, dx, dy, dz, r, gw);
    const double u = r / gw;
    if (!known) w = erf(u);
    const double fp = tsqpi * exp(-u * u) / (gw * r) - w / (r * r);
    m.A[e] = a.ke * m.h[i] * m.h[j] * fp / r;
  };
#pragma unroll
  for (int q = 0; q < kQeqPairs; ++q)
    if (lane + 64 * q < pairs) factor(lane + 64 * q, true, kept[q]);
  for (int e = lane + 64 * kQeqPairs; e < pairs; e += 64) factor(e, false, 0.0);
  qeq_order();
  if (!in) return;
  const double xi = m.x[lane][0], yi = m.x[lane][1], zi = m.x[lane][2];
  const int mine = lane * (lane - 1) / 2;
  double fx = 0.0, fy = 0.0, fz = 0.0;
  for (int j = 0; j < n; ++j) {
    if (j == lane) continue;
    const double s = m.A[j < lane ? mine + j : j * (j - 1) / 2 + lane];
    fx -= s * (xi - m.x[j][0]);
    fy -= s * (yi - m.x[j][1]);
    fz -= s * (zi - m.x[j][2]);
  }
  Fc[3 * g] = (float)fx;
  Fc[3 * g + 1] = (float)fy;
  Fc[3 * g + 2] = (float)fz;
}

void launch_qeq_solve(const QeqArgs& a, float* Fc, hipStream_t s) {
  if (a.B == 0) return;
  hipLaunchKernelGGL((k_qeq_solve<kQeqSmall, 4>), dim3((unsigned)((a.B + 3) / 4)), dim3(256), 0, s, a, Fc);
  if (a.N > kQeqSmall)
    hipLaunchKernelGGL((k_qeq_solve<kQeqMax, 2>), dim3((unsigned)((a.B + 1) / 2)), dim3(128), 0, s, a, Fc);
}

}  // namespace nnp
