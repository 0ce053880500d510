// HMC with an explicit coupling matrix (Sec. 2: "replace the matrix JK by the
// full coupling matrix"; App. A's infinite-range model is one instance): the
// K~ products of the equations of motion become GEMMs over all chains at once,
//     U = K Psi + C Psi,   F = K W + C W + h'/sqrt(J'),  W = sqrt(J') tanh(sqrt(J') U) - Psi,
// with Psi the N x B matrix of the B chains' fields.
//
// Precision: K (FP64 input) is held as three BF16 limbs K = K0 + K1 + K2 and the
// FP32 operands Psi, W as three BF16 limbs as well (FP32 is exact in three).  A
// GEMM accumulates the limb products K_a X_b with a + b <= 2 (6 products;
// truncation ~2^-24 relative, i.e. FP32-accurate) or a + b <= 1 (3 products on
// two limbs, ~2^-16) in FP32 on the MFMA units.  C Psi and C W are added in FP32
// in the epilogues, so the diagonal never consumes BF16 precision.  The
// Hamiltonian uses an FP64 GEMM of the stored FP32 field with the FP64 K.
//
// Layouts:
//   K limbs   [L] x fragments of (Np x Np), rows = sites i, columns = k
//   X limbs   [L] x fragments of (Bp x Np), rows = chains b, columns = sites k
//   partials  [S][Bp][Np]  FP32 (split-K slices, summed in fixed order)
// "Fragments" stores each 16-row x 32-column block contiguously in the order in
// which the lanes of a 16x16x32 MFMA take it (lane l: row l % 16, columns
// 8 (l / 16) .. + 7, 16 bytes), blocks of a row block in order of k.  A wave then
// loads a fragment with one instruction as 1 KiB in a row and feeds it to the
// matrix unit as it is.  Np is N padded to a multiple of 256, Bp is B padded to a
// multiple of 128; padding is zero.
#include <cfloat>

#include "chain_epilogue.hpp"
#include "dense_kernels.hpp"
#include "device_common.hpp"

namespace ihmc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Offset of element (row, k) of an operand in fragments with Np columns.
__host__ __device__ __forceinline__ int64_t frag(int64_t row, int64_t k, int64_t Np) {
  return (((row >> 4) * (Np >> 5) + (k >> 5)) << 9) + (((k >> 3) & 3) << 7) + ((row & 15) << 3) + (k & 7);
}
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Round-to-nearest-even BF16 limbs of a double: x ~ l0 + l1 + l2.
__device__ __forceinline__ void split3(double x, __bf16& l0, __bf16& l1, __bf16& l2) {
  l0 = (__bf16)(float)x;
  const double r1 = x - (double)(float)l0;
  l1 = (__bf16)(float)r1;
  const double r2 = r1 - (double)(float)l1;
  l2 = (__bf16)(float)r2;
}

// ------------------------------------------------------------ set-up kernels ---

// K (FP64, N x N) into limbs over the padded Np x Np layout; padding = 0.
__global__ void k_dense_split_K(const double* __restrict__ K, int64_t N, int64_t Np, __bf16* __restrict__ Kl) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= Np * Np) return;
  const int64_t i = idx / Np, k = idx % Np;
  const double x = (i < N && k < N) ? K[i * N + k] : 0.0;
  __bf16 a, b, c;
  split3(x, a, b, c);
  const int64_t o = frag(i, k, Np);
  Kl[o] = a;
  Kl[Np * Np + o] = b;
  Kl[2 * Np * Np + o] = c;
}

// Padded FP64 copy of K for the Hamiltonian GEMM and the set-up solvers.
__global__ void k_dense_pad_K(const double* __restrict__ K, int64_t N, int64_t Np, double* __restrict__ K64) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= Np * Np) return;
  const int64_t i = idx / Np, k = idx % Np;
  K64[idx] = (i < N && k < N) ? K[i * N + k] : 0.0;
}

// What the set-up demands of K (N x N): finite entries, symmetric to 1e-12 of the
// largest.  chk[0] counts non-finite entries, chk[1] holds the bits of max |K|
// (finite entries; the bits of non-negative doubles order as integers), chk[2]
// counts pairs that differ; all zero before.  chk[3] sums a mixed word of every
// entry and its place (in any order the same), by which checkpoints tell models
// apart.  On the host the two sweeps took 3.8 ms at N = 1000, half of the set-up.
__global__ __launch_bounds__(256) void k_dense_check(const double* __restrict__ K, int64_t n,
                                                     unsigned long long* __restrict__ chk) {
  double mx = 0.0;
  uint64_t mark = 0;
  bool bad = false;
  for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < n; i += 256ll * gridDim.x) {
    const double k = K[i], v = fabs(k);
    if (v <= DBL_MAX) mx = fmax(mx, v);
    else bad = true;
    uint64_t x = (uint64_t)__double_as_longlong(k + 0.0) + (uint64_t)i * 0x9e3779b97f4a7c15ull;  // -0 as 0
    x = (x ^ (x >> 32)) * 0xd6e8feb86659fd93ull;
    x = (x ^ (x >> 32)) * 0xd6e8feb86659fd93ull;
    mark += x ^ (x >> 32);
  }
  for (int off = 32; off > 0; off >>= 1) {
    mx = fmax(mx, __shfl_xor(mx, off, 64));
    mark += __shfl_xor(mark, off, 64);
  }
  __shared__ double sm[4];
  __shared__ uint64_t sk[4];
  if ((threadIdx.x & 63) == 0) {
    sm[threadIdx.x >> 6] = mx;
    sk[threadIdx.x >> 6] = mark;
  }
  const int any = __syncthreads_or(bad);
  if (threadIdx.x == 0) {  // one atomic per block: they all meet at one address
    atomicMax(chk + 1, (unsigned long long)__double_as_longlong(fmax(fmax(sm[0], sm[1]), fmax(sm[2], sm[3]))));
    if (any) atomicAdd(chk, 1ull);
    atomicAdd(chk + 3, (unsigned long long)(sk[0] + sk[1] + sk[2] + sk[3]));
  }
}

// 32 x 32 tiles above the diagonal (and on it) against their mirror images,
// both read in rows and one turned in LDS
__global__ __launch_bounds__(256) void k_dense_symmetry(const double* __restrict__ K, int64_t N,
                                                        unsigned long long* __restrict__ chk) {
  __shared__ double sm[32][33];
  if (blockIdx.x < blockIdx.y) return;
  const double tol = 1e-12 * __longlong_as_double((long long)chk[1]);
  const int64_t r0 = blockIdx.y * 32ll, c0 = blockIdx.x * 32ll;
  const int x = threadIdx.x & 31, y0 = threadIdx.x >> 5;
  for (int y = y0; y < 32; y += 8) sm[y][x] = (c0 + y < N && r0 + x < N) ? K[(c0 + y) * N + r0 + x] : 0.0;
  __syncthreads();
  bool bad = false;
  for (int y = y0; y < 32; y += 8)
    if (r0 + y < N && c0 + x < N) bad = bad || fabs(K[(r0 + y) * N + c0 + x] - sm[x][y]) > tol;
  if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicAdd(chk + 2, 1ull);
}

// Fixed-order sum over a 1024-thread block, broadcast to every thread.
__device__ double block_sum_1024(double v, double* sh) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < 16; ++w) t += sh[w];
  return t;
}

// Per-site field of a dense model: h' = beta h and h'/sqrt(J') (padding 0).
__global__ void k_dense_field(const double* __restrict__ h, int64_t N, int64_t Np, double beta, double sqJ,
                              double* __restrict__ hp, float* __restrict__ b) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= Np) return;
  const double v = i < N ? beta * h[i] : 0.0;
  hp[i] = v;
  b[i] = (float)(v / sqJ);
}

// ---- Lanczos (lowest eigenvalue of K, for the shift C) ----------------------
//
// Start vector: normals of a fixed Philox stream, normalised (padding 0).
__global__ __launch_bounds__(1024) void k_lanczos_start(double* __restrict__ q0, int64_t N, int64_t Np) {
  __shared__ double sh[16];
  double ss = 0.0;
  for (int64_t i = threadIdx.x; i < Np; i += 1024) {
    double v = 0.0;
    if (i < N) {
      const uint4 r = philox4x32_10(make_uint4((uint32_t)(i >> 1), 0u, 0u, 0x4c414e43u), 0x2545f491u, 0x9e3779b9u);
      const double u1 = unit53(r.x, r.y), u2 = unit53(r.z, r.w);
      const double rad = sqrt(-2.0 * log(u1));
      v = (i & 1) ? rad * sin(2.0 * M_PI * u2) : rad * cos(2.0 * M_PI * u2);
    }
    q0[i] = v;
    ss += v * v;
  }
  ss = block_sum_1024(ss, sh);
  const double inv = 1.0 / sqrt(ss);
  for (int64_t i = threadIdx.x; i < Np; i += 1024) q0[i] *= inv;
}

// Step k of Lanczos with full reorthogonalisation (classical Gram-Schmidt,
// twice): w = K q_k; alpha_k = q_k.w, w is orthogonalised against q_0..q_k,
// beta_k = |w|, q_{k+1} = w / beta_k.  Three launches of lanczos_blocks(Np) blocks,
// each with R = Np / blocks rows of its own; what a launch needs of all rows the
// one before left as one partial sum per block:
//   product  q_k = w / beta_{k-1} from the norm partials, w = K q_k, partials of Q^T w
//   orth     w -= Q c with c from those partials; first time: partials of Q^T w
//            again, second time: partials of |w|^2
// Bound by the latency of three dependent launches (1000 sites: 6.6 + 7.9 + 7.9 us
// a step, 4096: 30.6 + 12.8 + 12.8, means over the run); with the orthogonalisation
// in one block, which read the basis through a single CU four times, a step took
// 53 and 295 us.
constexpr int kLanczosMax = 1024;

__device__ __forceinline__ void lanczos_dots(const double* __restrict__ Q, const double* __restrict__ w, int64_t i0,
                                             int R, int64_t Np, int k, double* __restrict__ P) {
  const int e = threadIdx.x & 15;
  for (int jj = threadIdx.x >> 4; jj <= k; jj += 64) {
    const double* q = Q + (int64_t)jj * Np + i0;
    double s = 0.0;
    for (int i = e; i < R; i += 16) s += q[i] * w[i0 + i];
    for (int off = 8; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (e == 0) P[jj] = s;
  }
}

// u: w of the previous step (k > 0; other blocks read it, so w is another buffer)
__global__ __launch_bounds__(1024) void k_lanczos_product(const double* __restrict__ K64, double* __restrict__ Q, int k,
                                                          const double* __restrict__ u, double* __restrict__ w,
                                                          const double* __restrict__ npart, double* __restrict__ ab,
                                                          double* __restrict__ P, int pstride, int64_t Np, int R) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i0 = (int64_t)blockIdx.x * R;
  double* qk = Q + (int64_t)k * Np;
  double inv = 1.0;
  if (k == 0) {
    u = Q;
  } else {
    double ss = 0.0;
    for (int b = lane; b < (int)gridDim.x; b += 64) ss += npart[b];
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
    const double bk = sqrt(ss);
    inv = bk > 0.0 ? 1.0 / bk : 0.0;
    for (int i = threadIdx.x; i < R; i += 1024) qk[i0 + i] = u[i0 + i] * inv;
    if (blockIdx.x == 0 && threadIdx.x == 0) ab[2 * (k - 1) + 1] = bk;
  }
  for (int r = wave; r < R; r += 16) {
    const double* row = K64 + (i0 + r) * Np;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll 4
    for (int64_t c = 2 * lane; c < Np; c += 128) {
      const double2 kv = *reinterpret_cast<const double2*>(row + c), uv = *reinterpret_cast<const double2*>(u + c);
      s0 += kv.x * (uv.x * inv);
      s1 += kv.y * (uv.y * inv);
    }
    double s = s0 + s1;
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) w[i0 + r] = s;
  }
  __syncthreads();  // the block's rows of w and q_k
  lanczos_dots(Q, w, i0, R, Np, k, P + (int64_t)blockIdx.x * pstride);
}

template <bool FIRST>
__global__ __launch_bounds__(1024) void k_lanczos_orth(const double* __restrict__ Q, int k, double* __restrict__ w,
                                                       const double* __restrict__ P, double* __restrict__ Pnext,
                                                       int pstride, double* __restrict__ npart, double* __restrict__ ab,
                                                       int64_t Np, int R) {
  __shared__ double sc[kLanczosMax], sq[4][256], red[16][16];
  const int t = threadIdx.x, wave = t >> 6, nb4 = (int)gridDim.x >> 2;
  const int64_t i0 = (int64_t)blockIdx.x * R;
  for (int j0 = 0; j0 <= k; j0 += 256) {  // c: a quarter of the blocks' partials per 256 threads
    const int q = t >> 8, jj = j0 + (t & 255);
    double s = 0.0;
    if (jj <= k)
      for (int b = q * nb4; b < (q + 1) * nb4; ++b) s += P[(int64_t)b * pstride + jj];
    sq[q][t & 255] = s;
    __syncthreads();
    if (q == 0 && jj <= k) sc[jj] = (sq[0][t] + sq[1][t]) + (sq[2][t] + sq[3][t]);
    __syncthreads();
  }
  if (blockIdx.x == 0 && t == 0) ab[2 * k] = FIRST ? sc[k] : ab[2 * k] + sc[k];
  const int e = t & 15;
  for (int i = e; i - e < R; i += 16) {  // 64 groups of 16 threads share the basis vectors
    double s = 0.0;
    if (i < R)
      for (int jj = t >> 4; jj <= k; jj += 64) s += sc[jj] * Q[(int64_t)jj * Np + i0 + i];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if ((t & 63) < 16) red[wave][e] = s;
    __syncthreads();
    if (t < 16 && i < R) {
      double d = 0.0;
      for (int g = 0; g < 16; ++g) d += red[g][t];
      w[i0 + i] -= d;
    }
    __syncthreads();
  }
  if (FIRST) {
    lanczos_dots(Q, w, i0, R, Np, k, Pnext + (int64_t)blockIdx.x * pstride);
  } else {
    double ss = 0.0;
    for (int i = t; i < R; i += 1024) ss += w[i0 + i] * w[i0 + i];
    ss = block_sum_1024(ss, red[0]);
    if (t == 0) npart[blockIdx.x] = ss;
  }
}

// Steps k0 .. k1 - 1 of a small matrix (Np = 256) in one workgroup and one launch: the
// sums of the three launches, in their order (16 rows a partial sum, rows past N are
// zero), so the results are the same to the bit.  Three launches a step are what bounds
// the smallest (lowest eigenvalue of 16 sites 0.27 ms, of 64 0.83; in one launch per 16
// steps 0.18 and 0.66); one CU's reads of K and of the basis soon cost more: 100 sites 0.85
// and 0.79 ms, 128 1.16 and 1.22, 160 1.10 and 1.32.
constexpr int kLanczosSmall = 64;       // steps that it takes
constexpr int64_t kLanczosSmallN = 112;  // and sites

__global__ __launch_bounds__(1024) void k_lanczos_small(const double* __restrict__ K64, double* __restrict__ Q, int k0,
                                                        int k1, double* __restrict__ wa, double* __restrict__ wb,
                                                        double* __restrict__ npart, double* __restrict__ ab, int N) {
  constexpr int NP = 256, NB = NP / 16;
  __shared__ double sw[NP], sP[NB][kLanczosSmall], sc[kLanczosSmall], sA[16][NP], sn[NB];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, row = t & (NP - 1), q4 = t >> 8;
  const int nb = (N + 15) / 16;
  if (t < NB) sn[t] = k0 > 0 ? npart[t] : 0.0;
  if (t < NP) sw[t] = 0.0;
  __syncthreads();
  // c = Q^T w: partial sums over 16 rows, then over these
  auto coefficients = [&](int k) {
#pragma unroll 4
    for (int p = t >> 4; p < nb * (k + 1); p += 64) {
      const int b = p % nb, j = p / nb, i = 16 * b + (t & 15);
      double s = Q[(int64_t)j * NP + i] * sw[i];
      for (int off = 8; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
      if ((t & 15) == 0) sP[b][j] = s;
    }
    __syncthreads();
    if (t <= k) {
      double q[4];
      for (int a = 0; a < 4; ++a) {
        q[a] = 0.0;
        for (int b = 4 * a; b < min(4 * a + 4, nb); ++b) q[a] += sP[b][t];
      }
      sc[t] = (q[0] + q[1]) + (q[2] + q[3]);
    }
    __syncthreads();
  };
  // w -= Q c: four terms, then the sixteen sums of four in turn
  auto orthogonalise = [&](int k) {
    double q[16];
#pragma unroll
    for (int a = 0; a < 16; ++a) q[a] = Q[(int64_t)min(16 * q4 + a, k) * NP + row];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double x[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int j = 16 * q4 + 4 * v + a;
        x[a] = j <= k ? 0.0 + sc[j] * q[4 * v + a] : 0.0;
      }
      sA[4 * q4 + v][row] = (x[0] + x[1]) + (x[2] + x[3]);
    }
    __syncthreads();
    if (t < NP) {
      double d = 0.0;
      for (int v = 0; v < 16; ++v) d += sA[v][t];
      sw[t] -= d;
    }
    __syncthreads();
  };
  for (int k = k0; k < k1; ++k) {
    const double* u = k == 0 ? Q : ((k & 1) ? wa : wb);  // w of the step before
    double* w = (k & 1) ? wb : wa;
    double inv = 1.0;
    if (k > 0) {
      double ss = lane < NB ? sn[lane] : 0.0;
      for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
      const double bk = sqrt(ss);
      inv = bk > 0.0 ? 1.0 / bk : 0.0;
      if (t < NP) Q[(int64_t)k * NP + t] = u[t] * inv;
      if (t == 0) ab[2 * (k - 1) + 1] = bk;
    }
    double2 uv[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uv[h] = *reinterpret_cast<const double2*>(u + 2 * lane + 128 * h);
      uv[h].x *= inv;
      uv[h].y *= inv;
    }
#pragma unroll 4
    for (int r = wave; r < N; r += 16) {
      const double* kr = K64 + (int64_t)r * NP + 2 * lane;
      double s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double2 kv = *reinterpret_cast<const double2*>(kr + 128 * h);
        s0 += kv.x * uv[h].x;
        s1 += kv.y * uv[h].y;
      }
      double s = s0 + s1;
      for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
      if (lane == 0) sw[r] = s;
    }
    __syncthreads();  // w and q_k
    coefficients(k);
    const double alpha = sc[k];
    orthogonalise(k);
    coefficients(k);
    if (t == 0) ab[2 * k] = alpha + sc[k];
    orthogonalise(k);
    if (t < NP) {
      w[t] = sw[t];
      double ss = sw[t] * sw[t];
      for (int off = 8; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
      if ((t & 15) == 0) sn[t >> 4] = ss;
    }
    __syncthreads();
  }
  if (t < NB) npart[t] = sn[t];
}

// ---- conjugate gradients (Kt x = rhs, FP64) ---------------------------------
//
// One or two right-hand sides side by side, each with its own vectors and scalars
// (the iteration is bound by launches and latency, not by K: two share them).
// scal[0] = r.r, scal[1] = stopping threshold, scal[2] = r.r at the start;
// it[0] counts iterations, it[1] is the stop flag (1: converged, 2: a direction
// of non-positive curvature, i.e. Kt is not positive definite).
__global__ __launch_bounds__(1024) void k_cg_init(CgPair sys, int64_t Np, double rel_tol) {
  __shared__ double sh[16];
  const CgSystem& c = sys.s[blockIdx.x];
  double ss = 0.0;
  for (int64_t i = threadIdx.x; i < Np; i += 1024) {
    const double v = c.rhs[i];
    c.x[i] = 0.0;
    c.r[i] = v;
    c.d[i] = v;
    ss += v * v;
  }
  ss = block_sum_1024(ss, sh);
  if (threadIdx.x == 0) {
    c.scal[0] = ss;
    c.scal[1] = rel_tol * rel_tol * ss;
    c.scal[2] = ss;
    c.it[0] = 0;
    c.it[1] = (ss == 0.0) ? 1 : 0;
  }
}

// q = K d + C d of the systems that still run: one block of 256 threads per row,
// fixed-order reduction.
template <int NSYS>
__global__ __launch_bounds__(256) void k_cg_product(CgPair sys, const double* __restrict__ K64, int64_t Np, double C) {
  __shared__ double sh[NSYS][4];
  bool run[NSYS], any = false;
#pragma unroll
  for (int y = 0; y < NSYS; ++y) {
    run[y] = sys.s[y].it[1] == 0;
    any = any || run[y];
  }
  if (!any) return;
  const int64_t i = blockIdx.x;
  const double* row = K64 + i * Np;
  double s[NSYS] = {};
  for (int64_t k = threadIdx.x; k < Np; k += 256) {
    const double v = row[k];
#pragma unroll
    for (int y = 0; y < NSYS; ++y) s[y] += v * sys.s[y].d[k];
  }
#pragma unroll
  for (int y = 0; y < NSYS; ++y) {
    for (int off = 32; off > 0; off >>= 1) s[y] += __shfl_xor(s[y], off, 64);
    if ((threadIdx.x & 63) == 0) sh[y][threadIdx.x >> 6] = s[y];
  }
  __syncthreads();
  const int y = threadIdx.x;
  if (y < NSYS && run[y]) {
    const CgSystem& c = sys.s[y];
    c.q[i] = ((sh[y][0] + sh[y][1]) + (sh[y][2] + sh[y][3])) + C * c.d[i];
  }
}

__global__ __launch_bounds__(1024) void k_cg_step(CgPair sys, int64_t Np) {
  __shared__ double sh[16];
  const CgSystem& c = sys.s[blockIdx.x];
  if (c.it[1]) return;
  const double rr = c.scal[0];
  double dq = 0.0;
  for (int64_t i = threadIdx.x; i < Np; i += 1024) dq += c.d[i] * c.q[i];
  dq = block_sum_1024(dq, sh);
  if (!(dq > 0.0)) {  // Kt not positive definite along d (or non-finite)
    if (threadIdx.x == 0) c.it[1] = 2;
    return;
  }
  const double alpha = rr / dq;
  double rn = 0.0;
  for (int64_t i = threadIdx.x; i < Np; i += 1024) {
    c.x[i] += alpha * c.d[i];
    c.r[i] -= alpha * c.q[i];
    rn += c.r[i] * c.r[i];
  }
  rn = block_sum_1024(rn, sh);
  const double bt = rn / rr;
  for (int64_t i = threadIdx.x; i < Np; i += 1024) c.d[i] = c.r[i] + bt * c.d[i];
  if (threadIdx.x == 0) {
    c.scal[0] = rn;
    c.it[0] += 1;
    if (!(rn > c.scal[1])) c.it[1] = 1;
  }
}

// out[0] = a.b (fixed order).
__global__ __launch_bounds__(1024) void k_dense_dot(const double* __restrict__ a, const double* __restrict__ b,
                                                    int64_t Np, double* __restrict__ out) {
  __shared__ double sh[16];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < Np; i += 1024) s += a[i] * b[i];
  s = block_sum_1024(s, sh);
  if (threadIdx.x == 0) out[0] = s;
}

__global__ void k_dense_fill(double* __restrict__ x, int64_t N, int64_t Np, double v) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < Np) x[i] = i < N ? v : 0.0;
}

// ---------------------------------------------------------- split-K MFMA GEMM ---
//
// part[s][b][i] = sum_{k in slice s} sum_{(a, c) in products} Kl[a][i][k] * Xl[c][b][k]
// A workgroup is one wave with 16 RB sites x 16 CB chains (RB x CB MFMA 16x16x32
// blocks), and there is no LDS: operands lie in memory as fragments, so a wave
// loads what it multiplies straight into registers, three or four k-steps in
// turn, the loads of a step issued two or three steps before their use.  Waves
// that share a row or a column of fragments run side by side on one XCD and find
// them in its caches.  Matrix cores bound the large sizes (4096 sites x 256
// chains, six products: 44.0 us, 1170 TFLOP/s; 48.8 us when a 128 x 128 tile went
// through LDS behind a barrier per k-step), reading K the ones with few chains
// (4096 x 20: 16.3 us, 6.2 TB/s; was 42.7), the latency of the chain of k-steps
// the small ones (1024 x 20: 3.8 us, was 12.6; 1024 x 128: 4.8 us, was 12.6).
// Per output the order of the k-steps and of the products within one is that of
// a single accumulator running over the slice, whatever RB and CB are.
template <int NL, int NPROD, int RB, int CB, int D>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, RB * CB >= 16 ? 1 : 2))) void k_dense_gemm_bf16(
    const __bf16* __restrict__ Kl, const __bf16* __restrict__ Xl, float* __restrict__ part, int64_t Np, int64_t Bp,
    int S, int nrow, int ncol) {
  // limb pairs (a, c) with a + c <= 2 (NPROD = 6) or <= 1 (NPROD = 3)
  constexpr int PA[6] = {0, 0, 1, 0, 1, 2};
  constexpr int PC[6] = {0, 1, 0, 2, 1, 0};
  const int lane = threadIdx.x;
  // Blocks go to the 8 XCDs in turn: 8 / S of them take one k slice, each its own
  // run of row tiles, the column tiles of a row tile one after the other.
  const int share = 8 / S, xcd = blockIdx.x & 7, m = blockIdx.x >> 3;
  const int z = xcd / share, ct = m % ncol, rt = m / ncol + (nrow + share - 1) / share * (xcd % share);
  if (rt >= nrow) return;
  const int64_t i0 = (int64_t)rt * (16 * RB), b0 = (int64_t)ct * (16 * CB), k0 = z * (Np / S);
  const int nk = (int)((Np / S) >> 5);
  const int64_t lA = Np * Np, lB = Bp * Np, row16 = Np << 4;
  const __bf16* gA = Kl + frag(i0, k0, Np) + lane * 8;
  const __bf16* gB = Xl + frag(b0, k0, Np) + lane * 8;
  bf16x8 fa[D][NL][RB], fb[D][NL][CB];
  auto load = [&](int buf, int kt) {
    const int64_t o = (int64_t)kt << 9;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
#pragma unroll
      for (int r = 0; r < RB; ++r) fa[buf][l][r] = *reinterpret_cast<const bf16x8*>(gA + l * lA + r * row16 + o);
#pragma unroll
      for (int c = 0; c < CB; ++c) fb[buf][l][c] = *reinterpret_cast<const bf16x8*>(gB + l * lB + c * row16 + o);
    }
  };
  f32x4 acc[RB][CB];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int d = 0; d < D - 1; ++d) load(d, min(d, nk - 1));
  for (int kt = 0; kt < nk; kt += D) {
#pragma unroll
    for (int h = 0; h < D; ++h) {
      if (kt + h < nk) {
        // past the slice's end the last step is loaded again and not used; the
        // scheduling barriers keep the loads ahead of the MFMAs they overlap
        load((h + D - 1) % D, min(kt + h + D - 1, nk - 1));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < NPROD; ++p)
#pragma unroll
          for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int c = 0; c < CB; ++c)
              acc[r][c] =
                  __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[h][PA[p]][r], fb[h][PC[p]][c], acc[r][c], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // D layout of the 16x16 MFMA: lane -> column (chain) lane % 16, rows 4 (lane / 16) + e
  // (stores through the L2: each trajectory of 8 steps on 4096 x 256 1137 -> 1106 us,
  // 1024 x 1024 551 -> 526, 2048 x 64 264 -> 260, 1000 x 40 168 -> 168)
  float* out = part + ((int64_t)z * Bp + b0) * Np;
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int64_t b = 16 * c + (lane & 15);
      const int64_t i = i0 + 16 * r + 4 * (lane >> 4);
      st4_through(out, b * Np + i, acc[r][c]);
    }
}

// ------------------------------------------------------------- FP64 MFMA GEMM ---
//
// U64[b][i] = sum_k K64[i][k] psi[b][k] with psi the stored FP32 fields (exact in
// FP64).  As in the BF16 GEMM a workgroup is one wave with 16 RB sites x 16 CB
// chains (MFMA 16x16x4 FP64 blocks) that loads its operands straight into
// registers, D steps of 16 k in turn: a lane holds 4 consecutive k of its row,
// 32 and 16 bytes, and MFMA e of a step takes the e-th of every lane, so the order
// of k within a step is 4 (lane / 16) + e.  Every output runs over k in this
// order whatever the tile, so a chain's action does not depend on the others.
// Few chains or sites: bound by the chain of MFMAs of an output, 64 cycles each,
// which a wave with one block passes fastest (1024 sites x 40 chains 14.5 us,
// 48.5 with a 64 x 64 tile per workgroup through LDS).  4096 x 256: 184 us against
// 109 at the MFMA rate (196 through LDS); conversions of psi share the FP64 units.
// The field of chain b is read through its state: the accepted field (with its
// sign) for a measurement, else the buffer holding the proposal after pass j.
template <int RB, int CB, int D>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, RB * CB > 1 ? 2 : 4))) void k_dense_gemm_f64(
    const double* __restrict__ K64, const ChainDev* __restrict__ chains, int j, int measure, double* __restrict__ U64,
    int64_t Np, int B, int nrow, int ncol) {
  const int lane = threadIdx.x, kq = lane >> 4;
  // the column tiles of a row tile one after the other on one XCD
  const int m = blockIdx.x >> 3, ct = m % ncol, rt = m / ncol * 8 + (blockIdx.x & 7);
  if (rt >= nrow) return;
  const int64_t i0 = (int64_t)rt * (16 * RB);
  const int b0 = ct * (16 * CB);
  const double* gA = K64 + (i0 + (lane & 15)) * Np + 4 * kq;
  const float* gB[CB];
  float sg[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    const ChainDev& cd = chains[min(b0 + 16 * c + (lane & 15), B - 1)];  // columns past B are not stored
    const ChainState* st = cd.st;
    const int buf = measure ? st->cur : pass_in_buf(st->cur, j);
    gB[c] = (const float*)cd.psi + (int64_t)buf * cd.NP + 4 * kq;
    sg[c] = (measure && st->sign < 0) ? -1.f : 1.f;
  }
  f64x4 fa[D][RB];
  f32x4 fb[D][CB];
  auto load = [&](int s, int kt) {
    const int64_t o = (int64_t)kt << 4;
#pragma unroll
    for (int r = 0; r < RB; ++r) fa[s][r] = *reinterpret_cast<const f64x4*>(gA + (int64_t)(16 * r) * Np + o);
#pragma unroll
    for (int c = 0; c < CB; ++c) fb[s][c] = *reinterpret_cast<const f32x4*>(gB[c] + o);
  };
  f64x4 acc[RB][CB];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[r][c] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int nk = (int)(Np >> 4);
#pragma unroll
  for (int d = 0; d < D - 1; ++d) load(d, min(d, nk - 1));
  for (int kt = 0; kt < nk; kt += D) {
#pragma unroll
    for (int h = 0; h < D; ++h) {
      if (kt + h < nk) {
        load((h + D - 1) % D, min(kt + h + D - 1, nk - 1));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int c = 0; c < CB; ++c)
              acc[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[h][r][e], (double)(sg[c] * fb[h][c][e]),
                                                               acc[r][c], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // D layout of the FP64 16x16 MFMA: lane -> column lane % 16, rows lane / 16 + 4 e
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int b = b0 + 16 * c + (lane & 15);
      if (b >= B) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) U64[(int64_t)b * Np + i0 + 16 * r + kq + 4 * e] = acc[r][c][e];
    }
}

// ---------------------------------------------------------------- epilogues ---

// Sum of the split-K partials in slice order.
// Three BF16 limbs of an FP32 value (exact: 3 x 8 significand bits cover 24).
__device__ __forceinline__ void split_f32(float x, __bf16& l0, __bf16& l1, __bf16& l2) {
  l0 = (__bf16)x;
  const float r1 = x - (float)l0;
  l1 = (__bf16)r1;
  l2 = (__bf16)(r1 - (float)l1);
}

// The per-site kernels below (set-up limbs, both force epilogues, the FP64 action
// terms) run one wave per tile of 256 sites of one chain (grid: tiles x chains,
// so the chain's fields are uniform loads) with four consecutive sites per lane:
// 16-byte loads and stores of the FP32 fields, 8-byte stores of the limbs (four
// consecutive sites are contiguous in a fragment), and one wave per CU
// slot instead of four, so that the whole grid is resident at once.  Sites past
// N (the padding up to Np) carry zeros.
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
constexpr int EPI_SITES = 256, EPI_THREADS = 64;

__device__ __forceinline__ f32x4 ld_f4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ void st_f4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }

__device__ __forceinline__ f32x4 sum_parts4(const float* __restrict__ part, int S, int64_t plane, int64_t off) {
  f32x4 s = ld_f4(part + off);
  for (int q = 1; q < S; ++q) s = s + ld_f4(part + (int64_t)q * plane + off);
  return s;
}

// limbs of four consecutive sites (row b, columns i .. i+3, i % 4 == 0)
__device__ __forceinline__ void store_limbs4(__bf16* __restrict__ X, int64_t limb_stride, int64_t b, int64_t i,
                                             int64_t Np, f32x4 v) {
  bf16x4 l0, l1, l2;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    __bf16 a, c, d;
    split_f32(v[e], a, c, d);
    l0[e] = a;
    l1[e] = c;
    l2[e] = d;
  }
  const int64_t o = frag(b, i, Np);
  *reinterpret_cast<bf16x4*>(X + o) = l0;
  *reinterpret_cast<bf16x4*>(X + limb_stride + o) = l1;
  *reinterpret_cast<bf16x4*>(X + 2 * limb_stride + o) = l2;
}

// Start of a trajectory / set-up: limbs of the accepted fields (sign applied).
__global__ __launch_bounds__(EPI_THREADS) void k_dense_prep(const ChainDev* __restrict__ chains, int64_t Np,
                                                            int64_t Bp, __bf16* __restrict__ Xl) {
  const int b = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * EPI_SITES + 4 * threadIdx.x;
  const ChainDev& cd = chains[b];
  const ChainState* st = cd.st;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (i < cd.N) {
    v = ld_f4((const float*)cd.psi + (int64_t)st->cur * cd.NP + i);
    if (st->sign < 0) v = -v;
  }
  store_limbs4(Xl, Bp * Np, b, i, Np, v);
}

// After U = K Psi: w = sqrt(J') tanh(sqrt(J') (U + C psi) + hw) - psi  -> W (FP32 and
// limbs); hw = h' in the shifted form (per site: sqrt(J') times the stored
// h'/sqrt(J')), else 0.
__global__ __launch_bounds__(EPI_THREADS) void k_dense_epi_w(const ChainDev* __restrict__ chains, int64_t Np,
                                                             int64_t Bp, int S, const float* __restrict__ part, int j,
                                                             float* __restrict__ W32, __bf16* __restrict__ Wl) {
  const int b = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * EPI_SITES + 4 * threadIdx.x;
  const ChainDev& cd = chains[b];
  const ChainState* st = cd.st;
  const int64_t o = (int64_t)b * Np + i;
  const f32x4 ku = sum_parts4(part, S, Bp * Np, o);
  f32x4 w = {0.f, 0.f, 0.f, 0.f};
  if (i < cd.N) {
    const int buf = (j == 0) ? st->cur : pass_in_buf(st->cur, j);
    f32x4 v = ld_f4((const float*)cd.psi + (int64_t)buf * cd.NP + i);
    if (j == 0 && st->sign < 0) v = -v;
    const float a = (float)cd.sqJ, C = (float)cd.C;
    f32x4 hw = {0.f, 0.f, 0.f, 0.f};
    if (cd.form == FORM_SHIFTED) {
      if (cd.h_kind == 2) {
        const f32x4 b4 = ld_f4((const float*)cd.b + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) hw[e] = a * b4[e];
      } else {
        hw = f32x4{(float)cd.hw, (float)cd.hw, (float)cd.hw, (float)cd.hw};
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (i + e < cd.N) {
        const float u = __builtin_fmaf(C, v[e], ku[e]);
        w[e] = __builtin_fmaf(a, tanh_state(__builtin_fmaf(a, u, hw[e])), -v[e]);
      }
    }
  }
  st_f4(W32 + o, w);
  store_limbs4(Wl, Bp * Np, b, i, Np, w);
}

// After F = K W: F += C w + h'/sqrt(J'); kick p, drift psi (not on the last pass),
// new limbs of psi.  The FIRST pass draws the momenta (one Philox draw per pair
// of sites) and sums 1/2 p^2, the LAST pass sums 1/2 p^2 of the final momenta.
template <int MODE>
__global__ __launch_bounds__(EPI_THREADS) void k_dense_epi_f(const ChainDev* __restrict__ chains, int64_t Np,
                                                             int64_t Bp, int S, const float* __restrict__ part,
                                                             const float* __restrict__ W32, int j,
                                                             __bf16* __restrict__ Xl) {
  const int b = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * EPI_SITES + 4 * threadIdx.x;
  const ChainDev& cd = chains[b];
  ChainState* st = cd.st;
  const int64_t o = (int64_t)b * Np + i;
  const int cur = st->cur;
  double kick_d = 0.0, drift_d = 0.0;
  pass_coeffs(cd, j, kick_d, drift_d);
  const float kick = (MODE == PASS_FORCE) ? 1.f : (float)kick_d;
  const float drift = (float)drift_d;
  float* pmom = (float*)cd.p + i;
  const f32x4 kw = sum_parts4(part, S, Bp * Np, o);
  double kin[4] = {0.0, 0.0, 0.0, 0.0};
  f32x4 psi_new = {0.f, 0.f, 0.f, 0.f};
  if (i < cd.N) {
    const int in_buf = (MODE == PASS_FIRST || MODE == PASS_FORCE) ? cur : pass_in_buf(cur, j);
    f32x4 v = ld_f4((const float*)cd.psi + (int64_t)in_buf * cd.NP + i);
    if ((MODE == PASS_FIRST || MODE == PASS_FORCE) && st->sign < 0) v = -v;
    const f32x4 w = ld_f4(W32 + o);
    f32x4 bs = {0.f, 0.f, 0.f, 0.f};  // the shifted form has no linear term
    if (cd.form != FORM_SHIFTED) {
      if (cd.h_kind == 2) bs = ld_f4((const float*)cd.b + i);
      else bs = f32x4{(float)cd.b0, (float)cd.b0, (float)cd.b0, (float)cd.b0};
    }
    f32x4 p = {0.f, 0.f, 0.f, 0.f};
    if (MODE == PASS_FIRST) {
      if (cd.p_given) {
        p = ld_f4(pmom);
      } else {
        float z0, z1, z2, z3;
        normal_pair<float>(cd, (uint32_t)st->traj, TAG_MOM, i >> 1, z0, z1);
        normal_pair<float>(cd, (uint32_t)st->traj, TAG_MOM, (i >> 1) + 1, z2, z3);
        p = f32x4{z0, z1, z2, z3};
      }
    } else if (MODE != PASS_FORCE) {
      p = ld_f4(pmom);
    }
    f32x4 pn = {0.f, 0.f, 0.f, 0.f};
    const float C = (float)cd.C;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (i + e < cd.N) {
        const float F = __builtin_fmaf(C, w[e], kw[e]) + bs[e];
        pn[e] = __builtin_fmaf(kick, F, p[e]);
        if (MODE == PASS_FIRST) kin[e] = 0.5 * (double)p[e] * (double)p[e];
        if (MODE == PASS_LAST) kin[e] = 0.5 * (double)pn[e] * (double)pn[e];
        if (MODE == PASS_FIRST || MODE == PASS_MIDDLE) psi_new[e] = __builtin_fmaf(drift, pn[e], v[e]);
      }
    }
    if (MODE != PASS_LAST || cd.write_p_last) st_f4(pmom, pn);
    if (MODE == PASS_FIRST || MODE == PASS_MIDDLE)
      st_f4((float*)cd.psi + (int64_t)pass_out_buf(cur, j) * cd.NP + i, psi_new);
  }
  if (MODE == PASS_FIRST || MODE == PASS_MIDDLE) store_limbs4(Xl, Bp * Np, b, i, Np, psi_new);
  if (MODE == PASS_FIRST || MODE == PASS_LAST) {
    uint32_t bad = 0u;
    u128 acc[NTERM];
#pragma unroll
    for (int a = 0; a < NTERM; ++a) acc[a] = u128{0ull, 0ull};
    constexpr int a = (MODE == PASS_FIRST) ? T_K0 : T_K1;
    acc[a] = to_fixed(quad_sum(kin[0], kin[1], kin[2], kin[3]), bad);
    block_store_terms<1>(cd, acc, bad, a, a, MODE == PASS_FIRST ? CONTRIB_FIRST : CONTRIB_FINAL_KIN, blockIdx.x);
  }
}

// FP64 action terms of the proposal (LAST) or of the accepted field (MEASURE)
// from U64 = K psi; the block that finishes a chain last closes it (Metropolis
// or measurement).
template <int MODE>
__global__ __launch_bounds__(EPI_THREADS) void k_dense_h(const ChainDev* __restrict__ chains, int64_t Np,
                                                         const double* __restrict__ U64, int j) {
  const int b = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * EPI_SITES + 4 * threadIdx.x;
  const ChainDev& cd = chains[b];
  ChainState* st = cd.st;
  const int cur = st->cur;
  double h[4][4] = {};  // [term - T_S][site]
  if (i < cd.N) {
    const int buf = (MODE == PASS_MEASURE) ? cur : pass_in_buf(cur, j);
    f32x4 v4 = ld_f4((const float*)cd.psi + (int64_t)buf * cd.NP + i);
    if (MODE == PASS_MEASURE && st->sign < 0) v4 = -v4;
    const f64x4 ku = *reinterpret_cast<const f64x4*>(U64 + (int64_t)b * Np + i);
    f64x4 hp4 = {cd.hp0, cd.hp0, cd.hp0, cd.hp0};
    if (cd.h_kind == 2) hp4 = *reinterpret_cast<const f64x4*>(cd.hp + i);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (i + e < cd.N) {
        const double v = (double)v4[e];
        const double u = ku[e] + cd.C * v;
        const double hpx = hp4[e];
        const bool shifted = cd.form == FORM_SHIFTED;
        // shifted form: y = sqrt(J') u + h', no linear term, h[2] = y tanh(y)
        const double y = __builtin_fma(cd.sqJ, u, shifted ? hpx : 0.0);
        double lc, th;
        logcosh_tanh(y, lc, th);
        const double bx = shifted ? 0.0 : ((cd.h_kind == 2) ? hpx / cd.sqJ : cd.b0);
        h[0][e] = 0.5 * v * u - v * bx - lc;
        h[1][e] = v;
        h[2][e] = (shifted ? y : u) * th;
        h[3][e] = v * hpx;
      }
    }
  }
  uint32_t bad = 0u;
  u128 acc[NTERM];
#pragma unroll
  for (int a = 0; a < NTERM; ++a) acc[a] = u128{0ull, 0ull};
#pragma unroll
  for (int a = 0; a < 4; ++a) acc[T_S + a] = to_fixed(quad_sum(h[a][0], h[a][1], h[a][2], h[a][3]), bad);
  // the final kinetic energy was stored by the last force epilogue
  block_store_terms<1>(cd, acc, bad, T_S, T_PSIH, CONTRIB_ACTION, blockIdx.x);
  block_close<MODE == PASS_LAST, 1>(cd, st, MODE == PASS_LAST ? pass_in_buf(cur, j) : cur, blockIdx.x);
}

// ------------------------------------------------------------------ launch ---

hipError_t dense_split_K(const double* K, int64_t N, int64_t Np, __bf16* Kl, hipStream_t s) {
  k_dense_split_K<<<(unsigned)((Np * Np + 255) / 256), 256, 0, s>>>(K, N, Np, Kl);
  return hipGetLastError();
}

hipError_t dense_pad_K(const double* K, int64_t N, int64_t Np, double* K64, hipStream_t s) {
  k_dense_pad_K<<<(unsigned)((Np * Np + 255) / 256), 256, 0, s>>>(K, N, Np, K64);
  return hipGetLastError();
}

hipError_t dense_check(const double* K, int64_t N, unsigned long long* chk, hipStream_t s) {
  const int64_t n = N * N;
  const unsigned tiles = (unsigned)((N + 31) / 32);
  k_dense_check<<<(unsigned)(n / 4096 < 512 ? n / 4096 + 1 : 512), 256, 0, s>>>(K, n, chk);
  k_dense_symmetry<<<dim3(tiles, tiles), 256, 0, s>>>(K, N, chk);
  return hipGetLastError();
}

hipError_t dense_field(const double* h, int64_t N, int64_t Np, double beta, double sqJ, double* hp, float* b,
                       hipStream_t s) {
  k_dense_field<<<(unsigned)((Np + 255) / 256), 256, 0, s>>>(h, N, Np, beta, sqJ, hp, b);
  return hipGetLastError();
}

hipError_t lanczos_start(double* q0, int64_t N, int64_t Np, hipStream_t s) {
  k_lanczos_start<<<1, 1024, 0, s>>>(q0, N, Np);
  return hipGetLastError();
}

// Blocks of a Lanczos step: 16 rows each while that gives no more than 128, whose
// partials every block sums again.
static int lanczos_blocks(int64_t Np) { return (int)(Np / 16 < 128 ? Np / 16 : 128); }

uint64_t lanczos_work_doubles(int64_t Np, int mmax) {
  return 2 * (uint64_t)Np + 128 + 2 * (uint64_t)(mmax + 1) + 2 * (uint64_t)lanczos_blocks(Np) * (uint64_t)(mmax + 1);
}

static hipError_t lanczos_step(const double* K64, double* Q, int k, const LanczosWork& lw, int64_t Np, hipStream_t s) {
  if (k < 0 || k >= kLanczosMax || k >= lw.mmax) return hipErrorInvalidValue;
  const int nb = lanczos_blocks(Np), R = (int)(Np / nb), ps = lw.mmax + 1;
  double *w = lw.w[k & 1], *P2 = lw.P + (int64_t)nb * ps;
  k_lanczos_product<<<nb, 1024, 0, s>>>(K64, Q, k, lw.w[(k & 1) ^ 1], w, lw.npart, lw.ab, lw.P, ps, Np, R);
  k_lanczos_orth<true><<<nb, 1024, 0, s>>>(Q, k, w, lw.P, P2, ps, lw.npart, lw.ab, Np, R);
  k_lanczos_orth<false><<<nb, 1024, 0, s>>>(Q, k, w, P2, lw.P, ps, lw.npart, lw.ab, Np, R);
  return hipGetLastError();
}

hipError_t lanczos_steps(const double* K64, double* Q, int k0, int k1, const LanczosWork& lw, int64_t N, int64_t Np,
                         hipStream_t s) {
  if (k0 < 0 || k1 > lw.mmax) return hipErrorInvalidValue;
  if (Np == 256 && N <= kLanczosSmallN && k1 <= kLanczosSmall) {
    k_lanczos_small<<<1, 1024, 0, s>>>(K64, Q, k0, k1, lw.w[0], lw.w[1], lw.npart, lw.ab, (int)N);
    return hipGetLastError();
  }
  for (int k = k0; k < k1; ++k) {
    const hipError_t e = lanczos_step(K64, Q, k, lw, Np, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

LanczosWork lanczos_work(double* mem, int64_t Np, int mmax) {
  LanczosWork lw;
  lw.npart = mem;
  lw.n_npart = lanczos_blocks(Np);
  lw.ab = lw.npart + 128;
  lw.w[0] = lw.ab + 2 * (int64_t)(mmax + 1);
  lw.w[1] = lw.w[0] + Np;
  lw.P = lw.w[1] + Np;
  lw.mmax = mmax;
  return lw;
}

hipError_t cg_init(const CgPair& sys, int nsys, int64_t Np, double rel_tol, hipStream_t s) {
  k_cg_init<<<nsys, 1024, 0, s>>>(sys, Np, rel_tol);
  return hipGetLastError();
}

hipError_t cg_iterate(const CgPair& sys, int nsys, const double* K64, int64_t Np, double C, hipStream_t s) {
  if (nsys == 2) k_cg_product<2><<<(unsigned)Np, 256, 0, s>>>(sys, K64, Np, C);
  else k_cg_product<1><<<(unsigned)Np, 256, 0, s>>>(sys, K64, Np, C);
  k_cg_step<<<nsys, 1024, 0, s>>>(sys, Np);
  return hipGetLastError();
}

hipError_t dense_dot(const double* a, const double* b, int64_t Np, double* out, hipStream_t s) {
  k_dense_dot<<<1, 1024, 0, s>>>(a, b, Np, out);
  return hipGetLastError();
}

hipError_t dense_fill(double* x, int64_t N, int64_t Np, double v, hipStream_t s) {
  k_dense_fill<<<(unsigned)((Np + 255) / 256), 256, 0, s>>>(x, N, Np, v);
  return hipGetLastError();
}

template <int RB, int CB, int D>
static void launch_gemm_bf16(int nprod, const __bf16* Kl, const __bf16* Xl, float* part, int64_t Np, int64_t Bp, int B,
                             int S, hipStream_t s) {
  const int nrow = (int)(Np / (16 * RB)), ncol = (B + 16 * CB - 1) / (16 * CB), share = 8 / S;
  const unsigned grid = 8u * (unsigned)ncol * (unsigned)((nrow + share - 1) / share);
  if (nprod == 6) k_dense_gemm_bf16<3, 6, RB, CB, D><<<grid, 64, 0, s>>>(Kl, Xl, part, Np, Bp, S, nrow, ncol);
  else k_dense_gemm_bf16<2, 3, RB, CB, D><<<grid, 64, 0, s>>>(Kl, Xl, part, Np, Bp, S, nrow, ncol);
}

// Columns past the last tile that holds a chain are neither computed nor read.
// The tile is the one with the least estimated time per k-step: the rounds its
// waves take on the chip's 1024 SIMDs (one wave each: the two large tiles hold
// more than half the registers) times what one round was measured to take, us:
// 4x4 1.38, 4x2 0.81, 2x2 0.59, 2x1 0.45 (with up to 512 waves: beyond, its loads
// per product make it the slower one).  So a large tile, which reuses fragments
// more often, is taken only where it fills the chip (us: 4096 sites x 256 chains
// 4x4 44.0, 4x2 49.0; x 128 33.4, 26.0, 2x2 31.8; 4352 x 256 71.0, 67.0, 71.1;
// 2048 x 128 4x2 10.9, 2x2 9.5; 1024 x 128 2x2 4.8, 2x1 5.2; x 20 4.4, 3.8).
hipError_t dense_gemm_bf16(int nprod, const __bf16* Kl, const __bf16* Xl, float* part, int64_t Np, int64_t Bp, int B,
                           int S, hipStream_t s) {
  if (Np % 256 != 0 || Bp % 128 != 0 || B < 1 || B > Bp || (S != 1 && S != 2 && S != 4)) return hipErrorInvalidValue;
  auto cost = [&](int rb, int cb, int64_t per_round, double us) {
    const int64_t waves = Np / (16 * rb) * ((B + 16 * cb - 1) / (16 * cb)) * S;
    return us * (double)((waves + per_round - 1) / per_round);
  };
  const double c44 = cost(4, 4, 1024, 1.38), c42 = cost(4, 2, 1024, 0.81), c22 = cost(2, 2, 1024, 0.59),
               c21 = cost(2, 1, 512, 0.45);
  if (c44 <= fmin(c42, fmin(c22, c21))) launch_gemm_bf16<4, 4, 3>(nprod, Kl, Xl, part, Np, Bp, B, S, s);
  else if (c42 <= fmin(c22, c21)) launch_gemm_bf16<4, 2, 3>(nprod, Kl, Xl, part, Np, Bp, B, S, s);
  else if (c22 <= c21) launch_gemm_bf16<2, 2, 3>(nprod, Kl, Xl, part, Np, Bp, B, S, s);
  else launch_gemm_bf16<2, 1, 4>(nprod, Kl, Xl, part, Np, Bp, B, S, s);
  return hipGetLastError();
}

template <int RB, int CB, int D>
static void launch_gemm_f64(const double* K64, const ChainDev* chains, int j, int measure, double* U64, int64_t Np,
                            int B, hipStream_t s) {
  const int nrow = (int)(Np / (16 * RB)), ncol = (B + 16 * CB - 1) / (16 * CB);
  k_dense_gemm_f64<RB, CB, D><<<8u * (unsigned)ncol * (unsigned)((nrow + 7) / 8), 64, 0, s>>>(K64, chains, j, measure,
                                                                                            U64, Np, B, nrow, ncol);
}

// The tile with the least estimated time: rounds of 1024 waves (one per SIMD) times
// what a round was measured to take at 2048 sites, us: 1x1 47, 1x2 64, 2x2 92, and
// with at most half of the SIMDs busy 30, 59, 82.  (2048 x 128: 1x1 47, 1x2 60, 2x2
// 81; x 256: 91, 64, 83; 4096 x 256: 341, 233, 184; 4352 x 128: 213, 188, 173.)
hipError_t dense_gemm_f64(const double* K64, const ChainDev* chains, int j, int measure, double* U64, int64_t Np,
                          int B, hipStream_t s) {
  if (Np % 256 != 0 || B < 1) return hipErrorInvalidValue;
  auto cost = [&](int rb, int cb, double half, double full) {
    const int64_t waves = Np / (16 * rb) * ((B + 16 * cb - 1) / (16 * cb));
    return waves <= 512 ? half : full * (double)((waves + 1023) / 1024);
  };
  const double c11 = cost(1, 1, 30, 47), c12 = cost(1, 2, 59, 64), c22 = cost(2, 2, 82, 92);
  if (c11 <= fmin(c12, c22)) launch_gemm_f64<1, 1, 8>(K64, chains, j, measure, U64, Np, B, s);
  else if (c12 <= c22) launch_gemm_f64<1, 2, 4>(K64, chains, j, measure, U64, Np, B, s);
  else launch_gemm_f64<2, 2, 4>(K64, chains, j, measure, U64, Np, B, s);
  return hipGetLastError();
}

hipError_t dense_prep(const ChainDev* chains, int B, int64_t Np, int64_t Bp, __bf16* Xl, hipStream_t s) {
  if (Np % EPI_SITES != 0) return hipErrorInvalidValue;
  k_dense_prep<<<dim3((unsigned)(Np / EPI_SITES), (unsigned)B), EPI_THREADS, 0, s>>>(chains, Np, Bp, Xl);
  return hipGetLastError();
}

hipError_t dense_epi_w(const ChainDev* chains, int B, int64_t Np, int64_t Bp, int S, const float* part, int j,
                       float* W32, __bf16* Wl, hipStream_t s) {
  if (Np % EPI_SITES != 0) return hipErrorInvalidValue;
  k_dense_epi_w<<<dim3((unsigned)(Np / EPI_SITES), (unsigned)B), EPI_THREADS, 0, s>>>(chains, Np, Bp, S, part, j,
                                                                                      W32, Wl);
  return hipGetLastError();
}

hipError_t dense_epi_f(int mode, const ChainDev* chains, int B, int64_t Np, int64_t Bp, int S, const float* part,
                       const float* W32, int j, __bf16* Xl, hipStream_t s) {
  if (Np % EPI_SITES != 0) return hipErrorInvalidValue;
  dim3 grid((unsigned)(Np / EPI_SITES), (unsigned)B);
  switch (mode) {
    case PASS_FIRST:
      k_dense_epi_f<PASS_FIRST><<<grid, EPI_THREADS, 0, s>>>(chains, Np, Bp, S, part, W32, j, Xl);
      break;
    case PASS_MIDDLE:
      k_dense_epi_f<PASS_MIDDLE><<<grid, EPI_THREADS, 0, s>>>(chains, Np, Bp, S, part, W32, j, Xl);
      break;
    case PASS_LAST:
      k_dense_epi_f<PASS_LAST><<<grid, EPI_THREADS, 0, s>>>(chains, Np, Bp, S, part, W32, j, Xl);
      break;
    case PASS_FORCE:
      k_dense_epi_f<PASS_FORCE><<<grid, EPI_THREADS, 0, s>>>(chains, Np, Bp, S, part, W32, j, Xl);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t dense_h(int mode, const ChainDev* chains, int B, int64_t Np, const double* U64, int j, hipStream_t s) {
  if (Np % EPI_SITES != 0) return hipErrorInvalidValue;
  dim3 grid((unsigned)(Np / EPI_SITES), (unsigned)B);
  if (mode == PASS_LAST) k_dense_h<PASS_LAST><<<grid, EPI_THREADS, 0, s>>>(chains, Np, U64, j);
  else k_dense_h<PASS_MEASURE><<<grid, EPI_THREADS, 0, s>>>(chains, Np, U64, j);
  return hipGetLastError();
}

}  // namespace ihmc
