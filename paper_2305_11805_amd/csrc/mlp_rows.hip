// Per-species MLP of Eq. (1) (Sec. II.A), FP32, in row blocks: one block
// takes 16 atoms of one species per wave (4 or 8 waves), and each wave carries
// its 16 through the whole network (both hidden layers, the output, and the
// backward pass to lambda = dE/dG).  Every weight block a product needs is
// staged in LDS once per block and read by all waves, so the weights
// are fetched once per 64 or 128 atoms; the tile kernel (mlp.hip) splits the
// hidden units over its waves and fetches them once per 16.
//
// Products (C layout: lane (lm, lk) holds rows 4 lk + j, column lm of a 16x16
// tile):
//   P1  z1 = G W1^T       A: G rows (global), B: W1[:, k0:k0+KC] staged as [n][k]
//   P2  z2 = a1 W2^T      A: a1, B: W2[:, k0:k0+KC] as [n][k]
//   P3  g1 = delta2 W2    A: delta2, B: W2[k0:k0+KC, :] staged transposed as [n][k]
//   P4  lambda = delta1 W1  A: delta1, B: W1[:, c0:c0+NC] staged transposed as [n][k]
// with delta2 = w3 act'(z2), delta1 = g1 act'(z1); E = w3 . a2 + b3.  Sums
// have a fixed order (k in increasing chunks), so results are the same on
// every run.
//
// A product of FP32 values is taken exactly to 2^-23: each operand splits into
// three BF16 parts that hold all its 24 bits, and six of the nine products of
// parts (all above 2^-24 of the whole) go through v_mfma_f32_16x16x32_bf16,
// whose sums are FP32.  The FP32 matrix instruction does 30 multiply-adds a
// clock, six BF16 ones 85, and with 32 k an instruction in place of 4 there are
// fewer roundings: the forces' RMS error against 64 bits, in 1e-6 of their RMS
// over three inputs each, is 1.91 to 2.01 for 2048 molecules (1.93 to 2.03 with
// FP32 instructions), 2.24 to 2.27 for 32768 atoms of 4 species (2.29 to 2.34) and
// 1.60 to 1.89 for 262144 of 2 (1.63 to 1.92); the energies' is smaller too.
//
// What bounds it: 64-32 networks the traffic of G and lambda (2048 molecules,
// D 384, 0.21 GB: 94 -> 65 us), read in P1 and written in P4; the wider ones
// the splitting, the LDS reads and the matrix products of a chunk of 32 k, about
// equal and overlapping only between waves (128-128, D 768, 32768 atoms 158 ->
// 113 us; D 288, 262144 atoms 530 -> 297; 256-128, D 152, 16384 atoms, by
// the tile kernel before, 97 -> 66).  Two chunks in flight instead of one, and
// 32 atoms a wave instead of 16, were slower.  At 128 registers the 128-128 shape
// writes 20 bytes a lane to scratch and reads them once a block, outside the
// loops over chunks.
#include <math.h>

#include <type_traits>

#include "common.h"
#include "mlp_ops.h"

namespace nnp {

constexpr int kRwWaves = 4;
constexpr int kRwAtoms = 16 * kRwWaves;

__device__ __forceinline__ void rw_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// W waves of 16 atoms: 4 for 64-32, where blocks are what fills the chip, and
// for 256-128 (registers); 8 for 128-128, so that a staged block serves 128
// atoms (262144 atoms: 303 us, with 4 waves 332 to 360).
template <int H1T, int H2T, int W>
struct RowsShape {
  static constexpr int H1 = 16 * H1T, H2 = 16 * H2T;
  static constexpr int HM = H1 > H2 ? H1 : H2;
  static constexpr int KC = 32;       // k (P1-P3) or column (P4) chunk of a staged block
  static constexpr int LDA = KC + 4;  // rows of the wave's 16 x KC exchange tile
  static constexpr int U1 = HM * KC / 8, U4 = KC * H1 / 8;
  static constexpr int WSU = U1 > U4 ? U1 : U4;  // 16-byte units (8 values) of one staged part
  static constexpr size_t lds = 3 * 16 * (size_t)WSU + sizeof(float) * (size_t)W * 16 * LDA;
};

// One block's atoms through the network, products by `Part`: Split3, three BF16
// parts an operand, or Whole, FP32 instructions.  Returns whether a sum of this
// lane was not finite.
template <int H1T, int H2T, int W, typename Part>
__device__ __forceinline__ bool rows_block(const MlpArgs& args, int s, int tid, const int32_t* rows, float4* lds4) {
  using Sh = RowsShape<H1T, H2T, W>;
  constexpr int H1 = Sh::H1, H2 = Sh::H2, KC = Sh::KC, LDA = Sh::LDA, WSU = Sh::WSU;
  constexpr bool kSplit = std::is_same<Part, Split3>::value;
  bf16x8* wst = reinterpret_cast<bf16x8*>(lds4);  // Split3: parts h, m, l of WSU units each
  float4* wsf = lds4;                             // Whole: lo, hi of WSU units each
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* xch = reinterpret_cast<float*>(wst + 3 * WSU) + wv * 16 * LDA;  // this wave's exchange tile
  const int lm = lane & 15, lk = lane >> 4;
  // An operand without parts makes NaN of every sum it enters.  From G, W1 and W2
  // that reaches the row's energy (act4 passes NaN on), from delta2 every column
  // of g1, from delta1 every column of lambda: these are looked at.
  bool nan = false;
  auto look = [&](const floatx4& v) {
    if constexpr (kSplit)
#pragma unroll
      for (int j = 0; j < 4; ++j) nan = nan || v[j] != v[j];
  };
  const MlpDev& M = args.model.m[s];
  const int D = args.D;
  const int act1 = M.act[0], act2 = M.act[1];
  // rows past the block's atoms compute on row 0 of G and are never stored
  const int arow = rows[16 * wv + lm];
  const float* Grow = args.G + (int64_t)(arow < 0 ? 0 : arow) * D;
  const float* W1 = M.W[0];
  const float* W2 = M.W[1];
  constexpr int NT = 64 * W;

  // A staged unit is 8 k of one n.  Rows of KC k (P1-P3) hold 4 units, unit u
  // of row n at place u ^ (n / 2 & 3); rows of H1 k (P4) H1 / 8, at
  // u ^ (n & 7): eight lanes on consecutive rows then cover all the banks, in
  // the stores and in the reads, without padding.
  auto at1 = [&](int n, int u) { return 4 * n + (u ^ (n >> 1 & 3)); };
  auto at4 = [&](int n, int u) { return H1 / 8 * n + (u ^ (n & 7)); };
  auto stage = [&](int at, const float (&x)[8]) {
    Part p;
    split_operand(x, p);
    if constexpr (kSplit) {
      wst[at] = p.h;
      wst[WSU + at] = p.m;
      wst[2 * WSU + at] = p.l;
    } else {
      wsf[at] = p.lo;
      wsf[WSU + at] = p.hi;
    }
  };
  // acc[u] += a b_u for the NU column tiles from unit place at(u)
  auto mma = [&](auto NU, floatx4* acc, const Part& a, auto&& at) {
    constexpr int G = kSplit && decltype(NU)::value % 2 == 0 ? 2 : 1;  // independent chains in flight
#pragma unroll
    for (int u0 = 0; u0 < decltype(NU)::value; u0 += G) {
      Part b[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int x = at(u0 + g);
        if constexpr (kSplit) b[g] = Part{wst[x], wst[WSU + x], wst[2 * WSU + x]};
        else b[g] = Part{wsf[x], wsf[WSU + x]};
      }
      mma_parts<G>(acc + u0, a, b);
    }
  };
  // The A fragment of 32 columns held as two tiles in C layout (x[t][j]: row
  // 4 lk + j, column 16 t + lm), by way of the exchange tile: only 32 columns of
  // a wave's rows are ever in LDS, the rest stays in registers, which leaves
  // room for four blocks on a CU instead of two (the LDS serves a wave's
  // accesses in order).
  auto to_a = [&](const float (&x)[2][4]) {
    __asm__ volatile("" ::: "memory");
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int j = 0; j < 4; ++j) xch[(4 * lk + j) * LDA + 16 * t2 + lm] = x[t2][j];
    __asm__ volatile("" ::: "memory");
    const float4 u = *reinterpret_cast<const float4*>(xch + lm * LDA + 8 * lk);
    const float4 v = *reinterpret_cast<const float4*>(xch + lm * LDA + 8 * lk + 4);
    const float y[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
    Part p;
    split_operand(y, p);
    return p;
  };

  // The four products walk chunks of weights: a chunk is requested into
  // registers (w), then split and staged, and the next one (of the next
  // product, at the end of one) requested before this one's products, so the
  // loads overlap them.  The bases are uniform and the lanes' parts 32 bits.
  constexpr int NU = Sh::HM * KC / 8 / NT;
  static_assert(Sh::HM * KC / 8 % NT == 0, "whole units per thread");
  float w[NU][8];
  float ga[8];
  const uint32_t uD = (uint32_t)D;
  auto vec8 = [](const float* p, uint32_t off, float (&x)[8]) {
    const float4 u = *reinterpret_cast<const float4*>(p + off), v = *reinterpret_cast<const float4*>(p + off + 4);
    x[0] = u.x, x[1] = u.y, x[2] = u.z, x[3] = u.w, x[4] = v.x, x[5] = v.y, x[6] = v.z, x[7] = v.w;
  };
  // eight k of a row, zero past D (a multiple of 4)
  auto tail8 = [&](const float* p, int k, float (&x)[8]) {
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = 0.f;
#pragma unroll
    for (int h = 0; h < 8; h += 4)
      if (k + h < D) {
        const float4 u = *reinterpret_cast<const float4*>(p + k + h);
        x[h] = u.x, x[h + 1] = u.y, x[h + 2] = u.z, x[h + 3] = u.w;
      }
  };
  // W1[n][k0 ..]
  auto fetch1 = [&](int k0) {
    if (k0 + KC <= D) {
#pragma unroll
      for (int q = 0; q < H1 * KC / 8 / NT; ++q) {
        const uint32_t c = (uint32_t)(tid + q * NT);
        vec8(W1 + k0, (c >> 2) * uD + 8 * (c & 3), w[q]);
      }
      vec8(Grow + k0, 8 * lk, ga);
    } else {
#pragma unroll
      for (int q = 0; q < H1 * KC / 8 / NT; ++q) {
        const int c = tid + q * NT;
        tail8(W1 + (int64_t)(c >> 2) * D, k0 + 8 * (c & 3), w[q]);
      }
      tail8(Grow, k0 + 8 * lk, ga);
    }
  };
  // W2[n][k0 ..]
  constexpr int N2 = H2 * KC / 8;
  auto fetch2 = [&](int k0) {
#pragma unroll
    for (int q = 0; q < (N2 + NT - 1) / NT; ++q) {
      const uint32_t c = (uint32_t)(tid + q * NT);
      if (N2 % NT == 0 || (int)c < N2) vec8(W2 + k0, (c >> 2) * H1 + 8 * (c & 3), w[q]);
    }
  };
  // W2[k0 ..][n], each of the eight loads coalesced over n
  auto fetch3 = [&](int k0) {
#pragma unroll
    for (int q = 0; q < H1 * KC / 8 / NT; ++q) {
      const uint32_t c = (uint32_t)(tid + q * NT);
#pragma unroll
      for (int k = 0; k < 8; ++k) w[q][k] = (W2 + (k0 + k) * H1)[8 * (c / H1) * H1 + c % H1];
    }
  };
  // W1[k][c0 + n] over all k, coalesced over n
  auto fetch4 = [&](int c0) {
#pragma unroll
    for (int q = 0; q < H1 * KC / 8 / NT; ++q) {
      const uint32_t c = (uint32_t)(tid + q * NT), n = c % KC;
      const bool in = c0 + (int)n < D;
      const uint32_t off = in ? 8 * (c / KC) * uD + n : 0u;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float v = (W1 + (int64_t)k * D + c0)[off];
        w[q][k] = in ? v : 0.f;
      }
    }
  };

  // ---- P1: z1 = G W1^T, staged as [n][k] ----
  floatx4 acc1[H1T];
#pragma unroll
  for (int u = 0; u < H1T; ++u) acc1[u] = floatx4{0.f, 0.f, 0.f, 0.f};
  fetch1(0);
  for (int k0 = 0; k0 < D; k0 += KC) {
#pragma unroll
    for (int q = 0; q < H1 * KC / 8 / NT; ++q) {
      const int c = tid + q * NT;
      stage(at1(c >> 2, c & 3), w[q]);
    }
    Part a;
    split_operand(ga, a);
    __syncthreads();
    if (k0 + KC < D) fetch1(k0 + KC);
    else fetch2(0);
    mma(std::integral_constant<int, H1T>{}, acc1, a, [&](int u) { return at1(16 * u + lm, lk); });
    __syncthreads();
  }
  // ---- P2: z2 = a1 W2^T, 32 columns of a1 = act(z1) at a time ----
  float d1[H1T][4];  // act'(z1) in C layout
  floatx4 acc2[H2T];
#pragma unroll
  for (int u = 0; u < H2T; ++u) acc2[u] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kc = 0; kc < H1 / KC; ++kc) {
#pragma unroll
    for (int q = 0; q < (N2 + NT - 1) / NT; ++q) {
      const int c = tid + q * NT;
      if (N2 % NT == 0 || c < N2) stage(at1(c >> 2, c & 3), w[q]);
    }
    float a1[2][4];
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2) {
      const int u = 2 * kc + t2;
      act4<kSplit>(act1, acc1[u], M.b[0][16 * u + lm], a1[t2], d1[u]);
      if (args.st_a1)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = rows[16 * wv + 4 * lk + j];
          if (r >= 0) args.st_a1[(int64_t)r * H1 + 16 * u + lm] = a1[t2][j];
        }
    }
    const Part a = to_a(a1);
    __syncthreads();
    if (kc + 1 < H1 / KC) fetch2((kc + 1) * KC);
    else fetch3(0);
    mma(std::integral_constant<int, H2T>{}, acc2, a, [&](int u) { return at1(16 * u + lm, lk); });
    __syncthreads();
  }
  // ---- output E = w3 . a2 + b3 and delta2 = w3 act'(z2) ----
  const float* w3 = M.W[2];
  float e[4] = {0.f, 0.f, 0.f, 0.f};
  float d2[H2T][4];
#pragma unroll
  for (int u = 0; u < H2T; ++u) {
    const float wu = w3[16 * u + lm];
    float av[4];
    act4<kSplit>(act2, acc2[u], M.b[1][16 * u + lm], av, d2[u]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      e[j] = fmaf(av[j], wu, e[j]);
      d2[u][j] *= wu;
    }
    if (args.st_a2)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = rows[16 * wv + 4 * lk + j];
        if (r >= 0) {
          args.st_a2[(int64_t)r * H2 + 16 * u + lm] = av[j];
          args.st_d2[(int64_t)r * H2 + 16 * u + lm] = d2[u][j];
        }
      }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float v = e[j];
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    v += __shfl_xor(v, 8);
    e[j] = v;
  }
  if (lm == 0)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = rows[16 * wv + 4 * lk + j];
      if (r >= 0) args.E_atom[r] = e[j] + M.b[2][0];
    }
  look(floatx4{e[0], e[1], e[2], e[3]});
  if (args.lambda == nullptr && args.st_d1 == nullptr) return nan;  // the same for the whole block

  // ---- P3: g1 = delta2 W2 ----
#pragma unroll
  for (int u = 0; u < H1T; ++u) acc1[u] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kc = 0; kc < H2 / KC; ++kc) {
#pragma unroll
    for (int q = 0; q < H1 * KC / 8 / NT; ++q) {
      const int c = tid + q * NT;
      stage(at1(c % H1, c / H1), w[q]);
    }
    const float x[2][4] = {{d2[2 * kc][0], d2[2 * kc][1], d2[2 * kc][2], d2[2 * kc][3]},
                           {d2[2 * kc + 1][0], d2[2 * kc + 1][1], d2[2 * kc + 1][2], d2[2 * kc + 1][3]}};
    const Part a = to_a(x);
    __syncthreads();
    if (kc + 1 < H2 / KC) fetch3((kc + 1) * KC);
    else fetch4(0);
    mma(std::integral_constant<int, H1T>{}, acc1, a, [&](int u) { return at1(16 * u + lm, lk); });
    __syncthreads();
  }
  // ---- P4: lambda = delta1 W1, delta1 = g1 act'(z1), column chunks of KC ----
  Part a4[H1 / 32];  // this wave's delta1 rows as A fragments (k over H1)
#pragma unroll
  for (int kb = 0; kb < H1 / 32; ++kb) {
    float x[2][4];
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2) {
      const int u = 2 * kb + t2;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        x[t2][j] = acc1[u][j] * d1[u][j];
        if (args.st_d1) {
          const int r = rows[16 * wv + 4 * lk + j];
          if (r >= 0) args.st_d1[(int64_t)r * H1 + 16 * u + lm] = x[t2][j];
        }
      }
    }
    a4[kb] = to_a(x);
  }
  if (args.lambda == nullptr) {
    look(acc1[0]);
    return nan;
  }
  float* out[4];  // null for rows past the block's atoms
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = rows[16 * wv + 4 * lk + j];
    out[j] = r < 0 ? nullptr : args.lambda + (int64_t)r * D + lm;
  }
  for (int c0 = 0; c0 < D; c0 += KC) {
#pragma unroll
    for (int q = 0; q < H1 * KC / 8 / NT; ++q) {
      const int c = tid + q * NT;
      stage(at4(c % KC, c / KC), w[q]);
    }
    __syncthreads();
    if (c0 + KC < D) fetch4(c0 + KC);
    floatx4 acc[KC / 16];
#pragma unroll
    for (int ct = 0; ct < KC / 16; ++ct) acc[ct] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < H1 / 32; ++kb)
      mma(std::integral_constant<int, KC / 16>{}, acc, a4[kb], [&](int ct) { return at4(16 * ct + lm, 4 * kb + lk); });
    look(acc[0]);
#pragma unroll
    for (int ct = 0; ct < KC / 16; ++ct) {
      const int col = c0 + 16 * ct;
      if (col + lm < D)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (out[j]) out[j][col] = acc[ct][j];
    }
    __syncthreads();
  }
  return nan;
}

// Blocks whose products of parts gave a sum that is not finite (an infinite or
// NaN operand, a value beyond the largest BF16 one, or a sum beyond FP32) take
// their atoms a second time by FP32 instructions, so that infinities and NaN come
// out as these give them; every product of such an operand is itself not finite,
// so none goes unseen.
template <int H1T, int H2T, int W>
__global__ void __launch_bounds__(64 * W, H1T <= 4 ? 5 : H1T <= 8 ? 4 : 2) k_mlp_rows(MlpArgs args) {
  constexpr int NA = 16 * W;  // atoms of a block
  extern __shared__ float4 rw_lds4[];
  __shared__ int32_t rows[NA];
  __shared__ int again;
  const int tid = threadIdx.x;
  // which species / block of NA atoms
  const int S = args.model.S;
  int64_t t = blockIdx.x;
  int s = 0;
  int64_t ns = 0;
  for (; s < S; ++s) {
    ns = args.sp_start[s + 1] - args.sp_start[s];
    const int64_t nt = (ns + NA - 1) / NA;
    if (t < nt) break;
    t -= nt;
  }
  if (s >= S) return;
  const int64_t r0 = args.sp_start[s] + t * NA;
  const int nrows = (int)min<int64_t>(NA, args.sp_start[s] + ns - r0);
  if (tid < NA) rows[tid] = tid < nrows ? args.perm[r0 + tid] : -1;
  if (tid == 0) again = 0;
  __syncthreads();
  if (__any(rows_block<H1T, H2T, W, Split3>(args, s, tid, rows, rw_lds4)) && (tid & 63) == 0) again = 1;
  __syncthreads();
  if (!again) return;
  int t2 = tid;  // another name, so that no address is kept in registers for this
  __asm__ volatile("" : "+v"(t2));
  (void)rows_block<H1T, H2T, W, Whole>(args, s, t2, rows, rw_lds4);
}

// ---------------------------------------------------------------------------
// BF16 products (MODE kBf16 or kBf16x3, v_mfma_f32_16x16x32_bf16): the same
// row blocks and stages, with every weight block staged from the BF16 hi/lo
// copies of W (rows [n][k]) and W^T (the per-call conversion of both layers),
// so no product transposes while staging.  A wave splits its own rows'
// operands (G, a1, delta2, delta1) once, 8 k per lane per 32-k step; the
// tile kernel instead had every wave of a tile split the whole G tile.
// ---------------------------------------------------------------------------

template <int H1T, int H2T>
struct RowsShapeBf {
  static constexpr int H1 = 16 * H1T, H2 = 16 * H2T;
  static constexpr int HM = H1 > H2 ? H1 : H2;
  static constexpr int KC = 32;                     // k chunk (P1-P3), column chunk (P4)
  static constexpr int LDB = KC + 8;                // staged BF16 [n][k] rows of P1-P3
  static constexpr int LDT = H1 + 8;                // staged BF16 [n][k] rows of P4
  static constexpr int LDA = HM + 4;                // the wave's FP32 rows
  static constexpr int WS1 = HM * LDB, WS4 = KC * LDT;
  static constexpr int WSB = WS1 > WS4 ? WS1 : WS4;  // BF16 values per staged array (hi, lo)
  static constexpr size_t lds = 2 * sizeof(__bf16) * (size_t)WSB + sizeof(float) * (size_t)kRwWaves * 16 * LDA;
};

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

template <int H1T, int H2T, int MODE>
__global__ void __launch_bounds__(64 * kRwWaves) k_mlp_rows_bf(MlpArgs args) {
  using Sh = RowsShapeBf<H1T, H2T>;
  constexpr int H1 = Sh::H1, H2 = Sh::H2, KC = Sh::KC, LDB = Sh::LDB, LDT = Sh::LDT, LDA = Sh::LDA;
  constexpr bool X3 = MODE == kBf16x3;
  constexpr int NT = 64 * kRwWaves;
  extern __shared__ float4 rw_lds4[];
  __bf16* wsh = reinterpret_cast<__bf16*>(rw_lds4);
  __bf16* wsl = wsh + Sh::WSB;
  __shared__ int32_t rows[kRwAtoms];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* abuf = reinterpret_cast<float*>(wsl + Sh::WSB) + wv * 16 * LDA;
  const int lm = lane & 15, lk = lane >> 4;
  const int S = args.model.S;
  int64_t t = blockIdx.x;
  int s = 0;
  int64_t ns = 0;
  for (; s < S; ++s) {
    ns = args.sp_start[s + 1] - args.sp_start[s];
    const int64_t nt = (ns + kRwAtoms - 1) / kRwAtoms;
    if (t < nt) break;
    t -= nt;
  }
  if (s >= S) return;
  const int64_t r0 = args.sp_start[s] + t * kRwAtoms;
  const int nrows = (int)min<int64_t>(kRwAtoms, args.sp_start[s] + ns - r0);
  if (tid < kRwAtoms) rows[tid] = tid < nrows ? args.perm[r0 + tid] : -1;
  __syncthreads();
  const MlpDev& M = args.model.m[s];
  const int D = args.D;
  const int act1 = M.act[0], act2 = M.act[1];
  const int arow = rows[16 * wv + lm];
  const float* Grow = args.G + (int64_t)(arow < 0 ? 0 : arow) * D;
  const u32x4 z4 = {0u, 0u, 0u, 0u};
  // rows [n0, n0 + NR) (of nmax, K columns each), k in [k0, k0 + KCH), into
  // LDS rows 0 .. NR - 1 of stride ld, hi and (split mode) lo; zero outside
  auto stage = [&](const __bf16* hi, const __bf16* lo, int K, int nmax, int n0, int NR, int k0, int KCH, int ld) {
    for (int x = tid; x < NR * KCH / 8; x += NT) {
      const int r = x / (KCH / 8), kk = 8 * (x - r * (KCH / 8));
      const int n = n0 + r, k = k0 + kk;
      const bool in = n < nmax && k < K;
      const int64_t off = (int64_t)n * K + k;
      *reinterpret_cast<u32x4*>(wsh + r * ld + kk) = in ? *reinterpret_cast<const u32x4*>(hi + off) : z4;
      if constexpr (X3) *reinterpret_cast<u32x4*>(wsl + r * ld + kk) = in ? *reinterpret_cast<const u32x4*>(lo + off) : z4;
    }
  };
  // an A fragment (8 k from kb of this lane's row lm) of the wave's FP32 rows,
  // split; every width is a multiple of 32, so kb + 7 stays inside the row
  auto afrag = [&](int kb, bf16x8& ah, bf16x8& al) {
    const float4 u = *reinterpret_cast<const float4*>(abuf + lm * LDA + kb);
    const float4 v = *reinterpret_cast<const float4*>(abuf + lm * LDA + kb + 4);
    const float x[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
    if constexpr (X3) split8(x, ah, al);
    else
#pragma unroll
      for (int q = 0; q < 8; ++q) ah[q] = (__bf16)x[q];
  };
  auto bfrag = [&](int off, bf16x8& bh, bf16x8& bl) {
    bh = *reinterpret_cast<const bf16x8*>(wsh + off);
    if constexpr (X3) bl = *reinterpret_cast<const bf16x8*>(wsl + off);
  };

  // ---- P1: z1 = G W1^T; the next chunk (weights and G) requested during this one ----
  constexpr int NS1 = H1 * KC / 8 / NT;
  static_assert(H1 * KC / 8 % NT == 0, "whole 16-byte units per thread");
  u32x4 ph[NS1], pl[NS1];
  float4 gp[KC / 32][2];
  const __bf16 *W1h = M.Wb[0], *W1l = M.Wl[0];
  auto fetch1 = [&](int k0) {
#pragma unroll
    for (int q = 0; q < NS1; ++q) {
      const int x = tid + q * NT, n = x / (KC / 8), k = k0 + 8 * (x - n * (KC / 8));
      const int64_t off = (int64_t)n * D + k;
      ph[q] = k < D ? *reinterpret_cast<const u32x4*>(W1h + off) : z4;
      if constexpr (X3) pl[q] = k < D ? *reinterpret_cast<const u32x4*>(W1l + off) : z4;
    }
#pragma unroll
    for (int kk = 0; kk < KC / 32; ++kk) {
      const int k = k0 + 32 * kk + 8 * lk;
      gp[kk][0] = k < D ? *reinterpret_cast<const float4*>(Grow + k) : make_float4(0.f, 0.f, 0.f, 0.f);
      gp[kk][1] = k < D ? *reinterpret_cast<const float4*>(Grow + k + 4) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  floatx4 acc1[H1T];
#pragma unroll
  for (int u = 0; u < H1T; ++u) acc1[u] = floatx4{0.f, 0.f, 0.f, 0.f};
  fetch1(0);
  for (int k0 = 0; k0 < D; k0 += KC) {
#pragma unroll
    for (int q = 0; q < NS1; ++q) {
      const int x = tid + q * NT, n = x / (KC / 8), kk = 8 * (x - n * (KC / 8));
      *reinterpret_cast<u32x4*>(wsh + n * LDB + kk) = ph[q];
      if constexpr (X3) *reinterpret_cast<u32x4*>(wsl + n * LDB + kk) = pl[q];
    }
    bf16x8 ah[KC / 32], al[KC / 32];
#pragma unroll
    for (int kk = 0; kk < KC / 32; ++kk) {
      const float x[8] = {gp[kk][0].x, gp[kk][0].y, gp[kk][0].z, gp[kk][0].w,
                          gp[kk][1].x, gp[kk][1].y, gp[kk][1].z, gp[kk][1].w};
      if constexpr (X3) split8(x, ah[kk], al[kk]);
      else
#pragma unroll
        for (int q = 0; q < 8; ++q) ah[kk][q] = (__bf16)x[q];
    }
    __syncthreads();
    if (k0 + KC < D) fetch1(k0 + KC);
#pragma unroll
    for (int kk = 0; kk < KC / 32; ++kk)
#pragma unroll
      for (int u = 0; u < H1T; ++u) {
        bf16x8 bh, bl;
        bfrag((16 * u + lm) * LDB + 32 * kk + 8 * lk, bh, bl);
        acc1[u] = mma_bf16<MODE>(acc1[u], ah[kk], al[kk], bh, bl);
      }
    __syncthreads();
  }
  float d1[H1T][4];
#pragma unroll
  for (int u = 0; u < H1T; ++u) {
    const float bias = M.b[0][16 * u + lm];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float z = acc1[u][j] + bias;
      const float av = act_f(act1, z);
      d1[u][j] = act_d(act1, z, av);
      abuf[(4 * lk + j) * LDA + 16 * u + lm] = av;
      if (args.st_a1) {
        const int r = rows[16 * wv + 4 * lk + j];
        if (r >= 0) args.st_a1[(int64_t)r * H1 + 16 * u + lm] = av;
      }
    }
  }
  rw_wave_sync();

  // ---- P2: z2 = a1 W2^T ----
  floatx4 acc2[H2T];
#pragma unroll
  for (int u = 0; u < H2T; ++u) acc2[u] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < H1; k0 += KC) {
    stage(M.Wb[1], M.Wl[1], H1, H2, 0, H2, k0, KC, LDB);
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < KC / 32; ++kk) {
      if (k0 + 32 * kk >= H1) break;
      bf16x8 ah, al;
      afrag(k0 + 32 * kk + 8 * lk, ah, al);
#pragma unroll
      for (int u = 0; u < H2T; ++u) {
        bf16x8 bh, bl;
        bfrag((16 * u + lm) * LDB + 32 * kk + 8 * lk, bh, bl);
        acc2[u] = mma_bf16<MODE>(acc2[u], ah, al, bh, bl);
      }
    }
    __syncthreads();
  }
  // ---- output E and delta2 (over a1 in abuf: every read of it ended before P2's last barrier) ----
  const float* w3 = M.W[2];
  float e[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < H2T; ++u) {
    const float bias = M.b[1][16 * u + lm];
    const float w = w3[16 * u + lm];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float z = acc2[u][j] + bias;
      const float av = act_f(act2, z);
      e[j] = fmaf(av, w, e[j]);
      const float dl2 = w * act_d(act2, z, av);
      abuf[(4 * lk + j) * LDA + 16 * u + lm] = dl2;
      if (args.st_a2) {
        const int r = rows[16 * wv + 4 * lk + j];
        if (r >= 0) {
          args.st_a2[(int64_t)r * H2 + 16 * u + lm] = av;
          args.st_d2[(int64_t)r * H2 + 16 * u + lm] = dl2;
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float v = e[j];
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    v += __shfl_xor(v, 8);
    e[j] = v;
  }
  if (lm == 0)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = rows[16 * wv + 4 * lk + j];
      if (r >= 0) args.E_atom[r] = e[j] + M.b[2][0];
    }
  if (args.lambda == nullptr && args.st_d1 == nullptr) return;
  rw_wave_sync();

  // ---- P3: g1 = delta2 W2 = delta2 (W2^T)^T, staged from W2^T [H1][H2] ----
#pragma unroll
  for (int u = 0; u < H1T; ++u) acc1[u] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < H2; k0 += KC) {
    stage(M.WbT[1], M.WlT[1], H2, H1, 0, H1, k0, KC, LDB);
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < KC / 32; ++kk) {
      if (k0 + 32 * kk >= H2) break;
      bf16x8 ah, al;
      afrag(k0 + 32 * kk + 8 * lk, ah, al);
#pragma unroll
      for (int u = 0; u < H1T; ++u) {
        bf16x8 bh, bl;
        bfrag((16 * u + lm) * LDB + 32 * kk + 8 * lk, bh, bl);
        acc1[u] = mma_bf16<MODE>(acc1[u], ah, al, bh, bl);
      }
    }
    __syncthreads();
  }
  rw_wave_sync();
#pragma unroll
  for (int u = 0; u < H1T; ++u)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float dd = acc1[u][j] * d1[u][j];
      abuf[(4 * lk + j) * LDA + 16 * u + lm] = dd;
      if (args.st_d1) {
        const int r = rows[16 * wv + 4 * lk + j];
        if (r >= 0) args.st_d1[(int64_t)r * H1 + 16 * u + lm] = dd;
      }
    }
  if (args.lambda == nullptr) return;
  rw_wave_sync();

  // ---- P4: lambda = delta1 W1 = delta1 (W1^T)^T, column chunks staged from W1^T [D][H1] ----
  bf16x8 dh[H1 / 32], dl[H1 / 32];
#pragma unroll
  for (int kb = 0; kb < H1 / 32; ++kb) afrag(32 * kb + 8 * lk, dh[kb], dl[kb]);
  int orow[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) orow[j] = rows[16 * wv + 4 * lk + j];
  constexpr int NS4 = KC * H1 / 8 / NT;
  static_assert(KC * H1 / 8 % NT == 0, "whole 16-byte units per thread");
  u32x4 qh[NS4], ql[NS4];
  const __bf16 *W1Th = M.WbT[0], *W1Tl = M.WlT[0];
  auto fetch4 = [&](int c0) {
#pragma unroll
    for (int q = 0; q < NS4; ++q) {
      const int x = tid + q * NT, r = x / (H1 / 8), k = 8 * (x - r * (H1 / 8));
      const bool in = c0 + r < D;
      const int64_t off = (int64_t)(c0 + r) * H1 + k;
      qh[q] = in ? *reinterpret_cast<const u32x4*>(W1Th + off) : z4;
      if constexpr (X3) ql[q] = in ? *reinterpret_cast<const u32x4*>(W1Tl + off) : z4;
    }
  };
  fetch4(0);
  for (int c0 = 0; c0 < D; c0 += KC) {
#pragma unroll
    for (int q = 0; q < NS4; ++q) {
      const int x = tid + q * NT, r = x / (H1 / 8), k = 8 * (x - r * (H1 / 8));
      *reinterpret_cast<u32x4*>(wsh + r * LDT + k) = qh[q];
      if constexpr (X3) *reinterpret_cast<u32x4*>(wsl + r * LDT + k) = ql[q];
    }
    __syncthreads();
    if (c0 + KC < D) fetch4(c0 + KC);
#pragma unroll
    for (int ct = 0; ct < KC / 16; ++ct) {
      if (c0 + 16 * ct >= D) break;
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < H1 / 32; ++kb) {
        bf16x8 bh, bl;
        bfrag((16 * ct + lm) * LDT + 32 * kb + 8 * lk, bh, bl);
        acc = mma_bf16<MODE>(acc, dh[kb], dl[kb], bh, bl);
      }
      const int col = c0 + 16 * ct + lm;
      if (col < D)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (orow[j] >= 0) args.lambda[(int64_t)orow[j] * D + col] = acc[j];
    }
    __syncthreads();
  }
}

bool mlp_rows_bf_supported(int h1, int h2, int D) {
  return ((h1 == 64 && h2 == 32) || (h1 == 128 && h2 == 128)) && D % 8 == 0;
}

void launch_mlp_rows_bf(const MlpArgs& a, int h1, int h2, int mode, int64_t N, hipStream_t s) {
  if (N == 0) return;
  const unsigned grid = (unsigned)((N + kRwAtoms - 1) / kRwAtoms + a.model.S);
  const dim3 g(grid), b(64 * kRwWaves);
  if (h1 == 64 && h2 == 32) {
    constexpr size_t lds = RowsShapeBf<4, 2>::lds;
    if (mode == kBf16x3) hipLaunchKernelGGL((k_mlp_rows_bf<4, 2, kBf16x3>), g, b, lds, s, a);
    else hipLaunchKernelGGL((k_mlp_rows_bf<4, 2, kBf16>), g, b, lds, s, a);
  } else if (h1 == 128 && h2 == 128) {
    constexpr size_t lds = RowsShapeBf<8, 8>::lds;
    if (mode == kBf16x3) hipLaunchKernelGGL((k_mlp_rows_bf<8, 8, kBf16x3>), g, b, lds, s, a);
    else hipLaunchKernelGGL((k_mlp_rows_bf<8, 8, kBf16>), g, b, lds, s, a);
  }
}

bool mlp_rows_supported(int h1, int h2, int D) {
  return ((h1 == 64 && h2 == 32) || (h1 == 128 && h2 == 128) || (h1 == 256 && h2 == 128)) && D % 4 == 0;
}

// Up to this many atoms plan value 1 means the tile kernel, whose block takes 16
// of them, its waves sharing the columns of each product: the larger blocks
// would leave most CUs without one, and a block's time is then its own chain
// of chunks.  8192 atoms are two tiles for each CU; the next one starts a third
// round, and the row blocks are ahead from there.  MLP time in us, row blocks
// against the tile kernel:
//   64-32, D 384, 4 species    6534 atoms  33 / 29    8571  34 / 36   12213  33 / 36
//   64-32, D 768, 4 species                           9000  57 / 58   11000  57 / 59
//   64-32, D 152, 1 species    8000 atoms  18 / 17   10240  19 / 19   16384  21 / 28
//   128-128, D 96, 1 species   8192 atoms  35 / 25    9000  35 / 35   12000  35 / 37
//   128-128, D 768, 4 species  8192 atoms 102 / 73    9000 102 / 104  12000 102 / 108
//   256-128, D 152, 1 species  8000 atoms  57 / 52   10240  60 / 74   16384  66 / 97
constexpr int64_t kTilesMost = 8192;
bool mlp_rows_pays(int64_t N) { return N > kTilesMost; }

template <int A, int B, int W>
static void launch_rows(const MlpArgs& a, int64_t N, hipStream_t s) {
  const unsigned grid = (unsigned)((N + 16 * W - 1) / (16 * W) + a.model.S);
  constexpr size_t lds = RowsShape<A, B, W>::lds;
  hipLaunchKernelGGL((k_mlp_rows<A, B, W>), dim3(grid), dim3(64 * W), lds, s, a);
}

void launch_mlp_rows(const MlpArgs& a, int h1, int h2, int64_t N, hipStream_t s) {
  if (N == 0) return;
  if (h1 == 64 && h2 == 32) launch_rows<4, 2, 4>(a, N, s);
  else if (h1 == 128 && h2 == 128) launch_rows<8, 8, 8>(a, N, s);
  else if (h1 == 256 && h2 == 128) launch_rows<16, 8, 4>(a, N, s);
}

}  // namespace nnp
