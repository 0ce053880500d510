// Kt x = h' for chains with a per-site field (set-up; Sec. 2, the remark after
// eq. phi_psi_substitution): the estimator constants h'^T Kt^-1 h' and
// 1^T Kt^-1 h', and x itself for chains that run in translated coordinates.
//
// x enters the starting field of a translated chain, and a trajectory in FP64
// amplifies a last digit of it to 1e-3 in 200 trajectories, so x comes from the
// conjugate gradients that always gave it, operation for operation (k_field_cg),
// and a seed keeps its trajectory.  The constants enter the estimators only; they come
// from a transform, except on lattices too long and thin for it (field_by_transform).
//
// On the periodic lattice Kt is diagonal in the real plane waves
// prod_d cas(2 pi k_d x_d / L_d), cas = cos + sin (the shift operators along an
// axis come in symmetric pairs, which have cos and sin of one frequency as
// eigenvectors of the same eigenvalue), with eigenvalues
//     lambda(k) = C + 2 sum_d cos(2 pi k_d / L_d)
//               = (C - 2 ndim) + sum_d 4 cos^2(pi k_d / L_d),
// the second form exact to rounding also where C barely exceeds 2 ndim.  So they
// take a separable Hartley transform H of h' and a division by lambda:
//     h'^T Kt^-1 h' = sum_k H(k)^2 / (N lambda(k)),   1^T Kt^-1 h' = H(0) / (2 ndim + C).
//
// One axis of all chains is one launch: out[k] = sum_j cas(2 pi j k / L) in[j],
// N L products per chain in FP64, tiles of 64 frequencies x 64 columns, 16
// steps of j staged in LDS at a time.  Bound by FP64 issue for long axes and by
// launches otherwise.  A call of 512 uneven 2D chains of 16 .. 256 sites a row
// went from 180 to 105 ms: the solve took 76.7 ms as conjugate gradients with one
// workgroup per chain (the largest chain's ~160 iterations over 2 MB of vectors
// set it).  Every sum has an
// order of its own chain, so the constants do not depend on which chains share
// the launches.
#include <algorithm>
#include <cmath>

#include "device_common.hpp"
#include "runtime_internal.hpp"

namespace ihmc {

namespace {

constexpr int FT = 64, FJ = 16;     // tile (frequencies, columns), staged steps
constexpr int FTHREADS = 256;
constexpr int CHUNK = 1024;         // modes per partial sum of h' Kt^-1 h'
constexpr unsigned MAX_GRID_X = 4096;

// Work space of one chain (4 N values): two field arrays, then the tables
// cas(2 pi m / L_d) of the axes, then the partial sums.
__device__ __forceinline__ double* cas_table(double* w, const ChainDev& cd, int axis) {
  return w + 2 * cd.N + (axis > 0 ? cd.L0 : 0) + (axis > 1 ? cd.L1 : 0);
}
__device__ __forceinline__ double* partials(double* w, const ChainDev& cd) {
  return w + 2 * cd.N + cd.L0 + cd.L1 + (cd.ndim == 3 ? cd.L2 : 0);
}

// h' in site order into the first array, and the axes' tables.
__global__ __launch_bounds__(FTHREADS) void k_fs_init(const ChainDev* __restrict__ cds, const int* __restrict__ which,
                                                      double* work, const int64_t* __restrict__ woff) {
  const ChainDev& cd = cds[which[blockIdx.y]];
  double* w = work + woff[blockIdx.y];
  const int64_t t0 = blockIdx.x * (int64_t)FTHREADS + threadIdx.x, stride = (int64_t)gridDim.x * FTHREADS;
  for (int64_t i = t0; i < cd.N; i += stride) w[i] = cd.hp[stored_index(cd, i)];
  for (int a = 0; a < cd.ndim; ++a) {
    const int L = a == 0 ? cd.L0 : (a == 1 ? cd.L1 : cd.L2);
    double* tab = cas_table(w, cd, a);
    for (int64_t m = t0; m < L; m += stride) {
      double sn, cs;
      sincos_turn((double)m / (double)L, sn, cs);
      tab[m] = cs + sn;
    }
  }
}

// One axis of every chain, from array `src` to the other.  Columns of axis 0 are
// rows of L0 consecutive values; of axis a > 0, lines of stride prod_{b<a} L_b.
__global__ __launch_bounds__(FTHREADS) void k_fs_axis(const ChainDev* __restrict__ cds, const int* __restrict__ which,
                                                      double* work, const int64_t* __restrict__ woff, int axis,
                                                      int src) {
  __shared__ __align__(16) double sIn[FJ][FT + 2];
  __shared__ __align__(16) double sC[FJ][FT];
  const ChainDev& cd = cds[which[blockIdx.y]];
  if (axis >= cd.ndim) {  // a 2D chain beside 3D ones: the array changes place all the same
    const double* in = work + woff[blockIdx.y] + src * cd.N;
    double* out = work + woff[blockIdx.y] + (1 - src) * cd.N;
    for (int64_t i = blockIdx.x * (int64_t)FTHREADS + threadIdx.x; i < cd.N; i += (int64_t)gridDim.x * FTHREADS)
      out[i] = in[i];
    return;
  }
  double* w = work + woff[blockIdx.y];
  const double* __restrict__ in = w + src * cd.N;
  double* __restrict__ out = w + (1 - src) * cd.N;
  const double* __restrict__ tab = cas_table(w, cd, axis);
  const int L = axis == 0 ? cd.L0 : (axis == 1 ? cd.L1 : cd.L2);
  const int64_t inner = axis == 0 ? 1 : (axis == 1 ? (int64_t)cd.L0 : (int64_t)cd.L0 * cd.L1);
  const int64_t ncol = cd.N / L;
  const int64_t kt = (L + FT - 1) / FT, ntile = kt * ((ncol + FT - 1) / FT);
  const double rL = 1.0 / (double)L;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  auto offset = [&](int64_t c) { return axis == 0 ? c * L : (c / inner) * (L * inner) + c % inner; };
  for (int64_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
    const int k0 = (int)(tile % kt) * FT;
    const int64_t c0 = (tile / kt) * FT;
    double acc[FT / 4];
#pragma unroll
    for (int c = 0; c < FT / 4; ++c) acc[c] = 0.0;
    for (int j0 = 0; j0 < L; j0 += FJ) {
      // values (consecutive threads along the contiguous direction) and the tile of cas
      for (int e = tid; e < FJ * FT; e += FTHREADS) {
        const int jj = axis == 0 ? e % FJ : e / FT, cc = axis == 0 ? e / FJ : e % FT;
        const bool ok = j0 + jj < L && c0 + cc < ncol;
        sIn[jj][cc] = ok ? in[offset(c0 + cc) + (int64_t)(j0 + jj) * inner] : 0.0;
      }
      for (int e = tid; e < FJ * FT; e += FTHREADS) {
        const int jj = e / FT, kk = e % FT;
        double v = 0.0;
        if (j0 + jj < L && k0 + kk < L) {
          const int64_t p = (int64_t)(j0 + jj) * (k0 + kk);  // < 2^40: exact in FP64
          int64_t m = p - (int64_t)((double)p * rL) * L;
          m = m < 0 ? m + L : (m >= L ? m - L : m);
          v = tab[m];
        }
        sC[jj][kk] = v;
      }
      __syncthreads();
#pragma unroll
      for (int jj = 0; jj < FJ; ++jj) {
        const double cs = sC[jj][lane];
#pragma unroll
        for (int c = 0; c < FT / 4; ++c) acc[c] = __builtin_fma(cs, sIn[jj][(FT / 4) * wv + c], acc[c]);
      }
      __syncthreads();
    }
    if (k0 + lane < L)
#pragma unroll
      for (int c = 0; c < FT / 4; ++c) {
        const int64_t col = c0 + (FT / 4) * wv + c;
        if (col < ncol) out[offset(col) + (int64_t)(k0 + lane) * inner] = acc[c];
      }
  }
}

// 4 cos^2(pi k / L): an axis' part of lambda + 2 ndim - C.
__device__ __forceinline__ double axis_eig(int k, int L) {
  double sn, cs;
  sincos_turn((double)k / (2.0 * (double)L), sn, cs);
  return 4.0 * (cs * cs);
}

// Partial sums of H^2 / (N lambda) of the transform in array `src`, over CHUNK modes
// each, one workgroup per chunk, in a fixed order.
__global__ __launch_bounds__(FTHREADS) void k_fs_sums(ChainDev* __restrict__ cds, const int* __restrict__ which,
                                                       double* work, const int64_t* __restrict__ woff, int src) {
  __shared__ double sh[FTHREADS / 64];
  ChainDev& cd = cds[which[blockIdx.y]];
  double* w = work + woff[blockIdx.y];
  const double* H = w + src * cd.N;
  const int64_t nchunk = (cd.N + CHUNK - 1) / CHUNK;
  const double gap = cd.C - 2.0 * cd.ndim, n = (double)cd.N;
  if (blockIdx.x == 0 && threadIdx.x == 0) cd.c_m = H[0] / (2.0 * cd.ndim + cd.C);
  for (int64_t b = blockIdx.x; b < nchunk; b += gridDim.x) {
    double s = 0.0;
    for (int e = threadIdx.x; e < CHUNK; e += FTHREADS) {
      const int64_t i = b * CHUNK + e;
      if (i >= cd.N) continue;
      const int x = (int)(i % cd.L0);
      const int64_t r = i / cd.L0;
      double lam = gap + axis_eig(x, cd.L0) + axis_eig((int)(r % cd.L1), cd.L1);
      if (cd.ndim == 3) lam += axis_eig((int)(r / cd.L1), cd.L2);
      s += H[i] * (H[i] / (n * lam));
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) partials(w, cd)[b] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    __syncthreads();
  }
}

// c_e = the partial sums of a chain, in a fixed order (one wave per chain).
__global__ __launch_bounds__(64) void k_fs_final(ChainDev* __restrict__ cds, const int* __restrict__ which,
                                                 double* work, const int64_t* __restrict__ woff) {
  ChainDev& cd = cds[which[blockIdx.x]];
  const double* p = partials(work + woff[blockIdx.x], cd);
  const int64_t nchunk = (cd.N + CHUNK - 1) / CHUNK;
  double s = 0.0;
  for (int64_t b = threadIdx.x; b < nchunk; b += 64) s += p[b];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (threadIdx.x == 0) cd.c_e = s;
}

// Sum over a block of 256 threads in a fixed order, broadcast to all of them.
__device__ double block_sum(double v, double* sh) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < FTHREADS / 64; ++w) t += sh[w];
  return t;
}

// y = Kt x in site order.
__device__ void apply_kt(const ChainDev& cd, const double* x, double* y) {
  const int L0 = cd.L0, L1 = cd.L1, L2 = cd.L2;
  for (int64_t s = threadIdx.x; s < cd.N; s += FTHREADS) {
    const int gx = (int)(s % L0);
    const int gy = (int)((s / L0) % L1);
    const int gz = (int)(s / ((int64_t)L0 * L1));
    auto at = [&](int a, int b, int c) { return x[a + (int64_t)L0 * (b + (int64_t)L1 * c)]; };
    double acc = (at(gx == 0 ? L0 - 1 : gx - 1, gy, gz) + at(gx == L0 - 1 ? 0 : gx + 1, gy, gz)) +
                 (at(gx, gy == 0 ? L1 - 1 : gy - 1, gz) + at(gx, gy == L1 - 1 ? 0 : gy + 1, gz));
    if (cd.ndim == 3) acc += at(gx, gy, gz == 0 ? L2 - 1 : gz - 1) + at(gx, gy, gz == L2 - 1 ? 0 : gz + 1);
    y[s] = cd.C * x[s] + acc;
  }
}

// x = Kt^-1 h' by conjugate gradients, to a relative residual of 1e-15: one block
// per chain, x in site order at the start of its work space.  With it the constants.
__global__ __launch_bounds__(FTHREADS) void k_field_cg(ChainDev* __restrict__ cds, const int* __restrict__ which,
                                                       double* work, const int64_t* __restrict__ woff) {
  __shared__ double sh[FTHREADS / 64];
  ChainDev& cd = cds[which[blockIdx.x]];
  const int64_t N = cd.N;
  double* x = work + woff[blockIdx.x];
  double* r = x + N;
  double* d = r + N;
  double* q = d + N;
  double hs = 0.0, rr = 0.0;
  for (int64_t i = threadIdx.x; i < N; i += FTHREADS) {
    const double v = cd.hp[stored_index(cd, i)];
    x[i] = 0.0;
    r[i] = v;
    d[i] = v;
    hs += v;
    rr += v * v;
  }
  hs = block_sum(hs, sh);
  rr = block_sum(rr, sh);
  const double stop = 1e-30 * rr;
  for (int it = 0; it < 20000 && rr > stop; ++it) {
    __syncthreads();
    apply_kt(cd, d, q);
    __syncthreads();
    double dq = 0.0;
    for (int64_t i = threadIdx.x; i < N; i += FTHREADS) dq += d[i] * q[i];
    dq = block_sum(dq, sh);
    const double alpha = rr / dq;
    double rn = 0.0;
    for (int64_t i = threadIdx.x; i < N; i += FTHREADS) {
      x[i] += alpha * d[i];
      r[i] -= alpha * q[i];
      rn += r[i] * r[i];
    }
    rn = block_sum(rn, sh);
    const double beta = rn / rr;
    rr = rn;
    for (int64_t i = threadIdx.x; i < N; i += FTHREADS) d[i] = r[i] + beta * d[i];
  }
  __syncthreads();
  double ce = 0.0;
  for (int64_t i = threadIdx.x; i < N; i += FTHREADS) ce += cd.hp[stored_index(cd, i)] * x[i];
  ce = block_sum(ce, sh);
  if (threadIdx.x == 0) {
    cd.c_e = ce;
    cd.c_m = hs / (2.0 * cd.ndim + cd.C);
  }
}

}  // namespace

// Which of the two gives a chain's constants, by the chain alone (so they do not depend on
// the set): the transform fills the GPU but takes L products a site along every axis, on
// tiles of 64 columns; the conjugate gradients take one CU and a number of iterations that
// the extreme eigenvalues set.  The transform while its products stay below 16384 a site
// and iteration: at the line it is 4 to 5 times as fast for one chain (3 x 3 x 60000 23
// against 194 ms, 65536 x 8 at C = 1000 23 against 25), beyond it soon slower (2^20 x 3:
// 9700 ms against 1280 at C = 4.1 and 175 at C = 1000), and slower from the start for
// sets of many such chains, which the conjugate gradients solve side by side.
bool field_by_transform(const ChainDev& c) {
  const int64_t L[3] = {c.L0, c.L1, c.L2};
  double products = 0.0, lo = c.C, hi = c.C;
  for (int a = 0; a < c.ndim; ++a) {
    products += (double)((L[a] + FT - 1) / FT) * (double)((c.N / L[a] + FT - 1) / FT) * (FT * FT) * (double)L[a];
    lo += 2.0 * std::cos(2.0 * M_PI * (double)(L[a] / 2) / (double)L[a]);
    hi += 2.0;
  }
  const double root = std::sqrt(hi / lo);
  const double iterations = std::ceil(std::log(2e15) / std::log((root + 1.0) / (root - 1.0)));
  return products <= 16384.0 * (double)c.N * iterations;
}

hipError_t launch_field_solve(ChainDev* d_cd, const std::vector<const ChainDev*>& host, const int* which, double* work,
                              const int64_t* woff, size_t plain, hipStream_t s) {
  if (plain < host.size())
    k_field_cg<<<(unsigned)(host.size() - plain), FTHREADS, 0, s>>>(d_cd, which + plain, work, woff + plain);
  if (plain == 0) return hipGetLastError();
  // largest number of tiles, sites and dimensions among the chains
  int64_t tiles = 1, sites = 1;
  int nd = 2;
  for (size_t i = 0; i < plain; ++i) {
    const ChainDev* c = host[i];
    const int64_t L[3] = {c->L0, c->L1, c->L2};
    for (int a = 0; a < c->ndim; ++a)
      tiles = std::max(tiles, ((L[a] + FT - 1) / FT) * ((c->N / L[a] + FT - 1) / FT));
    sites = std::max(sites, c->N);
    nd = std::max(nd, c->ndim);
  }
  auto grid_x = [](int64_t n) { return (unsigned)std::min<int64_t>(n, MAX_GRID_X); };
  // the chains fill grid.y, at most 65535 at a time
  for (size_t c0 = 0; c0 < plain; c0 += 65535) {
    const unsigned n = (unsigned)std::min<size_t>(plain - c0, 65535);
    const int* wh = which + c0;
    const int64_t* wo = woff + c0;
    const dim3 gs(grid_x((sites + 4 * FTHREADS - 1) / (4 * FTHREADS)), n), gt(grid_x(tiles), n);
    k_fs_init<<<gs, FTHREADS, 0, s>>>(d_cd, wh, work, wo);
    for (int a = 0; a < nd; ++a) k_fs_axis<<<gt, FTHREADS, 0, s>>>(d_cd, wh, work, wo, a, a & 1);
    const int at = nd & 1;  // the array that holds the transform
    k_fs_sums<<<dim3(grid_x((sites + CHUNK - 1) / CHUNK), n), FTHREADS, 0, s>>>(d_cd, wh, work, wo, at);
    k_fs_final<<<n, 64, 0, s>>>(d_cd, wh, work, wo);
  }
  return hipGetLastError();
}

}  // namespace ihmc
