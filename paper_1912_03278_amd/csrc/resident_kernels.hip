// LDS-resident chains: one workgroup runs whole trajectories of one small chain
// (one Tile entry per chain names it), every pass, the FP64 sums and the
// Metropolis step in one launch, with no partial-sum table and no launch per
// pass.
//
// The chain's sites are dealt to the threads as x-aligned vectors of V sites
// (V = 4 in FP32, 2 in FP64, one 16-byte LDS access each; V = 1 for chains of at
// most one site per thread, where spreading the sites over all four SIMDs is
// what shortens a trajectory).  A thread keeps the field, the momenta, w and the
// per-site field of its NQ vectors in registers for the whole trajectory; LDS
// holds only the two arrays that neighbours read, psi and w, in rows padded to
// whole vectors.  A leap-frog step is then two phases (w; kick and drift) of
// four to six 16-byte LDS reads per vector with a barrier after each.  The
// accepted field stays in registers too, and goes back to its buffer once, at the
// launch's end.
//
// The per-site arithmetic and the grouping of the FP64 sums (in 2D 16 x-aligned
// sites as four quads; in 3D x-aligned quads of columns, each column first
// summed over an aligned 4-plane slab, in z order) are those of the tiled
// passes, so a resident chain's trajectory is bit-identical to the tiled one.
// n_traj = 0 measures S and the estimator sums of the accepted field (the
// set-up pass) instead.
//
// Bound by VALU issue on the chain's one CU: a 64 x 64 FP32 step is 0.83 us on 16
// waves (87 VALU instructions a wave, 79 % of the cycles; the rest of a trajectory
// 94 %; 15 x 15 waits, 24 %) against 6.4 us for the scalar form it replaces (one site per LDS access, five
// LDS arrays, 256 threads, neighbour addresses worked out at every step); momenta,
// FP64 sums and the Metropolis step of a trajectory take 13.4 us there (26 before),
// 4.5 us for 15 x 15 (15.4).  1024 such chains of 64 x 64: 105 us a trajectory of 15 steps (294).
#include <algorithm>
#include <type_traits>

#include "chain_epilogue.hpp"
#include "device_common.hpp"
#include "lattice_common.hpp"
#include "lattice_kernels.hpp"

namespace ihmc {

// Largest resident chain: what four (five with a per-site field) logical
// arrays of a chain may take (5088 FP32 or 2544 FP64 sites, 4070 or 2035 with a
// field).  The two padded LDS arrays take at most 65 088 bytes (FP32 rows of five
// sites are padded most, 8/5: 5 x 1017), the reduction scratch under 2 KiB, of the
// CU's 160 KiB.
constexpr int RES_FIT_BYTES = 81408;

int resident_max_sites(int precision, bool site_field) { return RES_FIT_BYTES / ((site_field ? 5 : 4) * precision); }

// V consecutive LDS values, aligned to V elements.
template <typename T, int V>
__device__ __forceinline__ void ldv(const T* p, T (&v)[V]) {
  if constexpr (V == 4) {
    ld4<T>(p, v);
  } else if constexpr (V == 2 && sizeof(T) == 8) {
    const double2 q = *reinterpret_cast<const double2*>(p);
    v[0] = q.x;
    v[1] = q.y;
  } else {
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = p[e];
  }
}
template <typename T, int V>
__device__ __forceinline__ void stv(T* p, const T (&v)[V]) {
  if constexpr (V == 4) {
    st4<T>(p, v);
  } else if constexpr (V == 2 && sizeof(T) == 8) {
    *reinterpret_cast<double2*>(p) = make_double2(v[0], v[1]);
  } else {
#pragma unroll
    for (int e = 0; e < V; ++e) p[e] = v[e];
  }
}

__device__ __forceinline__ uint32_t pack2(int lo, int hi) { return (uint32_t)lo | ((uint32_t)hi << 16); }

// Ranks of the terms over the lanes that share a sum: K1, S, psi, u tanh, psi h'
// take ranks 0 .. 4 at the trajectory's end, K0 (drawn momenta) rank 5.  psi h' is
// zero without a field and left out then, so that the lanes of a quad convert the
// end's terms in one go.
constexpr int RES_RANKS = 6;

template <typename T, int NDIM, int V, int NT, int NQ>
__global__ __launch_bounds__(NT, 4) void lattice_resident(const ChainDev* __restrict__ chains,
                                                       const Tile* __restrict__ tiles, int n_traj) {
  constexpr int NW = NT / 64;
  // sites a lane evaluates per FP64 sum slot in 2D: its quad, or one site
  constexpr int E = (V == 1) ? 1 : 4;
  // lanes that share one sum and deal its conversions
  constexpr int GL = (NDIM == 2 && E == 1) ? 16 : 4;
  constexpr int NR = (RES_RANKS + GL - 1) / GL;
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ u128 sRed[NW][RES_RANKS];
  __shared__ u128 sSum[RES_RANKS];
  __shared__ uint32_t sBad[NW];
  __shared__ ChainState sSt;
  __shared__ double sAcc[2];  // accept uniforms, by the parity of the trajectory
  __shared__ uint32_t sFlags;
  const ChainDev& cd = chains[tiles[blockIdx.x].chain];
  const int L0 = cd.L0, L1 = cd.L1, L2 = (NDIM == 3) ? cd.L2 : 1;
  const int N = (int)cd.N;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nvr = (L0 + V - 1) / V, PV = nvr * V, rows = L1 * L2;  // vectors per row, LDS row pitch
  T* const sP = reinterpret_cast<T*>(lds);  // field
  T* const sW = sP + PV * rows;             // w; momenta between the phases that use w
  if (tid < (int)(sizeof(ChainState) / 8)) ((uint64_t*)&sSt)[tid] = ((const uint64_t*)cd.st)[tid];
  __syncthreads();
  const int cur = sSt.cur;
  gmem<T>* __restrict__ gpsi = (gmem<T>*)cd.psi + (int64_t)cur * cd.NP;
  const T Ct = (T)cd.C;
  const T at = (T)cd.sqJ, hw = (T)cd.hw;

  // ---- the thread's vectors: LDS offsets of their own sites, of the rows above
  // and below (and planes), and of the sites left of the first and right of the
  // last; `last` = index of the last lattice site of the vector
  // (two 16-bit offsets a register: the arrays hold at most 8 Ki values)
  int own[NQ], last[NQ], gix[NQ];
  uint32_t updn[NQ], zmzp[NQ], lfrt[NQ];
  bool act[NQ];
  T ps[NQ][V], pm[NQ][V], ww[NQ][V], bq[NQ][V], keep[NQ][V];  // keep: the accepted field
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const int q = tid + NT * k;
    act[k] = q < nvr * rows;
    const int row = act[k] ? q / nvr : 0, x = act[k] ? (q - row * nvr) * V : 0;
    const int z = (NDIM == 3) ? row / L1 : 0, y = row - z * L1;
    const int r0 = row * PV;
    own[k] = r0 + x;
    updn[k] = pack2(own[k] + (y == 0 ? (L1 - 1) * PV : -PV), own[k] + (y == L1 - 1 ? -(L1 - 1) * PV : PV));
    const int pl = L1 * PV;
    zmzp[k] = pack2(own[k] + (z == 0 ? (L2 - 1) * pl : -pl), own[k] + (z == L2 - 1 ? -(L2 - 1) * pl : pl));
    lfrt[k] = pack2(r0 + (x == 0 ? L0 - 1 : x - 1), r0 + (x + V >= L0 ? 0 : x + V));
    last[k] = min(V, L0 - x) - 1;
    gix[k] = V == 4 ? own[k] : x + cd.pitch * row;  // stored rows are padded to four values too
#pragma unroll
    for (int e = 0; e < V; ++e) {
      bq[k][e] = (T)cd.b0;
      pm[k][e] = (T)0;
      const bool in = act[k] && e <= last[k];
      if (cd.h_kind == 2 && in) bq[k][e] = ((const gmem<T>*)cd.b)[gix[k] + e];
      keep[k][e] = in ? gpsi[gix[k] + e] : (T)0;
    }
  }
  // right neighbour of element e: the next one, or the site right of the last
  auto right = [&](const T (&c)[V], T r, int k, int e) { return (e == V - 1 || e == last[k]) ? r : c[e + 1 < V ? e + 1 : e]; };

  // ---- FP64 sums into fixed point, grouped as in the tiled passes: slots of E
  // sites of a row (2D; 16 x-aligned sites share a sum) or of one column over an
  // aligned 4-plane slab (3D; an x-aligned quad of columns shares a sum).
  // term(o, gi, xm, xp, ym, yp, zm, zp, v) fills NU terms of the site at LDS
  // offset o and stored index gi.  Every lane takes part in every step.
  u128 accR[NR];
  uint32_t bad = 0u;
  const bool with_h = sums_psih(cd);
  const int n16 = (L0 + 15) / 16, nq4 = (L0 + 3) / 4, nsl = (L2 + 3) / 4;
  const int nslot = (NDIM == 2) ? n16 * (16 / E) * rows : 4 * nq4 * L1 * nsl;
  auto site_sums = [&](auto nu_tag, int rank0, auto term) {
    constexpr int NU = decltype(nu_tag)::value;
    auto left_out = [&](int rank) { return NU > 1 && rank == 4 && !with_h; };  // psi h'
    for (int s0 = 0; s0 < nslot; s0 += NT) {
      const int s = s0 + tid;
      double qv[NU];
#pragma unroll
      for (int a = 0; a < NU; ++a) qv[a] = 0.0;
      if (NDIM == 2) {
        const int g = s / (16 / E), y = g / n16, x = 16 * (g - y * n16) + E * (s & (16 / E - 1));
        // the slot's terms (t0 + t1) + (t2 + t3), two sites at a time
#pragma unroll 1
        for (int h = 0; h < E; h += 2) {
          double t[2][NU];
#pragma unroll
          for (int e = 0; e < (E == 1 ? 1 : 2); ++e) {
#pragma unroll
            for (int a = 0; a < NU; ++a) t[e][a] = 0.0;
            const int xx = x + h + e;
            if (s < nslot && xx < L0) {
              const int r0 = y * PV, o = r0 + xx;
              term(o, xx + (int64_t)cd.pitch * y, r0 + (xx == 0 ? L0 - 1 : xx - 1), r0 + (xx == L0 - 1 ? 0 : xx + 1),
                   o + (y == 0 ? (L1 - 1) * PV : -PV), o + (y == L1 - 1 ? -(L1 - 1) * PV : PV), o, o, t[e]);
            }
          }
#pragma unroll
          for (int a = 0; a < NU; ++a) {
            const double pr = E == 1 ? t[0][a] : t[0][a] + t[1][a];
            qv[a] = h == 0 ? pr : qv[a] + pr;
          }
        }
#pragma unroll
        for (int a = 0; a < NU; ++a) {
          if (left_out(rank0 + a)) continue;
          qv[a] = quad_sum_all(qv[a]);
          if constexpr (E == 1) {
            qv[a] = qv[a] + dpp_f64<DPP_ROW_HALF_MIRROR>(qv[a]);  // q0 + q1, q2 + q3
            qv[a] = qv[a] + dpp_f64<DPP_ROW_MIRROR>(qv[a]);
          }
        }
      } else {
        const int c4 = 4 * nq4, r = s / c4, x = s - r * c4, sl = r / L1, y = r - sl * L1;
        const bool in = s < nslot && x < L0;
        double col[NU];
#pragma unroll
        for (int a = 0; a < NU; ++a) col[a] = 0.0;
        const int z0 = 4 * sl, z1 = min(z0 + 4, L2), pl = L1 * PV;
        if (in) {
#pragma unroll 1
          for (int z = z0; z < z1; ++z) {
            const int row = y + L1 * z, r0 = row * PV, o = r0 + x;
            double v[NU];
            term(o, x + (int64_t)cd.pitch * row, r0 + (x == 0 ? L0 - 1 : x - 1), r0 + (x == L0 - 1 ? 0 : x + 1),
                 o + (y == 0 ? (L1 - 1) * PV : -PV), o + (y == L1 - 1 ? -(L1 - 1) * PV : PV),
                 o + (z == 0 ? (L2 - 1) * pl : -pl), o + (z == L2 - 1 ? -(L2 - 1) * pl : pl), v);
#pragma unroll
            for (int a = 0; a < NU; ++a) col[a] = col[a] + v[a];
          }
        }
#pragma unroll
        for (int a = 0; a < NU; ++a)
          if (!left_out(rank0 + a)) qv[a] = quad_sum_all(col[a]);
      }
      // the sum's lanes convert one term each: rank GL r + l by lane l into accR[r]
      const int gl = lane & (GL - 1);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        if (left_out(GL * r)) continue;  // the one term of its round
        double x = 0.0;
#pragma unroll
        for (int a = 0; a < NU; ++a)
          if ((rank0 + a) / GL == r) x = (gl == (rank0 + a) % GL) ? qv[a] : x;
        accR[r] = add128(accR[r], to_fixed(x, bad));
      }
    }
  };
  auto action_term = [&](int o, int64_t gi, int xm, int xp, int ym, int yp, int zmi, int zpi, double* v) {
    double nb = ((double)sP[xm] + (double)sP[xp]) + ((double)sP[ym] + (double)sP[yp]);
    if (NDIM == 3) nb = nb + ((double)sP[zmi] + (double)sP[zpi]);
    const SiteAction sa = site_action<false>(cd, (double)sP[o], nb, gi);
    v[0] = sa.s;
    v[1] = sa.psi;
    v[2] = sa.ut;
    v[3] = sa.psih;
  };
  // the block's fixed-point totals in sSum (by rank) and flags, for thread 0
  // (the first wave, which thread 0 belongs to, adds the waves' sums)
  auto block_totals = [&]() {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      u128 v = accR[r];
      if constexpr (GL == 4) {
        v = add128(v, dpp_u128<DPP_ROW_ROR4>(v));
        v = add128(v, dpp_u128<DPP_ROW_ROR8>(v));
      }
      v = pair_sum128<false>(v);  // the four rows
      v = pair_sum128<true>(v);
      const int rk = GL * r + lane;
      if (lane < GL && rk < RES_RANKS) sRed[wave][rk] = v;
    }
    const unsigned long long any = __ballot(bad != 0u);
    if (lane == 0) sBad[wave] = any ? 1u : 0u;
    lds_barrier();
    if (tid < RES_RANKS) {
      u128 v = sRed[0][tid];
#pragma unroll
      for (int w = 1; w < NW; ++w) v = add128(v, sRed[w][tid]);
      sSum[tid] = v;
    }
    lds_barrier();
    uint32_t b = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) b |= sBad[w];
    return b;
  };
  auto clear_acc = [&]() {
#pragma unroll
    for (int r = 0; r < NR; ++r) accR[r] = u128{0ull, 0ull};
    bad = 0u;
  };
  // the accepted field, sign applied, into registers and LDS
  auto load_field = [&](int sign) {
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      if (!act[k]) continue;
#pragma unroll
      for (int e = 0; e < V; ++e) ps[k][e] = neg_if(keep[k][e], sign);
      stv<T, V>(sP + own[k], ps[k]);
    }
  };
  using NU1 = std::integral_constant<int, 1>;
  using NU4 = std::integral_constant<int, 4>;
  using NU5 = std::integral_constant<int, 5>;

  if (n_traj == 0) {  // set-up: S and the estimator sums of the accepted field
    load_field(sSt.sign);
    lds_barrier();
    clear_acc();
    site_sums(NU4{}, 1, action_term);
    const uint32_t b = block_totals();
    if (tid == 0) {
      u128 sum[NTERM];
      sum[T_K0] = sum[T_K1] = u128{0ull, 0ull};
#pragma unroll
      for (int a = 0; a < 4; ++a) sum[T_S + a] = sSum[1 + a];
      finalize_measure(cd, cd.st, sum, b);
    }
    return;
  }

  // kick of pass j: kick_end at both ends, else by the parity of j (two kinds of
  // inner kick in the Omelyan scheme); one drift
  const int n_pass = cd.n_pass;
  double kd, dd, unused;
  pass_coeffs(cd, 0, kd, dd);
  const T kick_end = (T)kd, drift = (T)dd;
  pass_coeffs(cd, 1, kd, unused);
  const T kick_odd = (T)kd;
  pass_coeffs(cd, 2, kd, unused);
  const T kick_even = (T)kd;
  const int npair = (N + 1) / 2;

  // Fresh momenta of trajectory `traj` into sW by threads t0, t0 + nt, ..: one
  // Philox draw per site pair; the one past the last pair is the accept uniform.
  // They need nothing of the trajectory before, so all waves but the first draw
  // them while the first makes its Metropolis step (1.4 us of one thread).
  auto draw_momenta = [&](uint32_t traj, int t0, int nt) {
    for (int pr = t0; pr <= npair; pr += nt) {
      const bool mom = pr < npair;
      const uint4 w = draw(cd, mom ? (uint32_t)pr : 0u, traj, mom ? TAG_MOM : TAG_ACC);
      if (!mom) {
        sAcc[traj & 1u] = unit53(w.x, w.y);
        continue;
      }
      double a, b;
      box_muller(w, a, b);
      const int r0 = (2 * pr) / L0, x0 = 2 * pr - r0 * L0;
      const bool wrap = x0 + 1 == L0;
      sW[r0 * PV + x0] = (T)a;
      if (2 * pr + 1 < N) sW[wrap ? (r0 + 1) * PV : r0 * PV + x0 + 1] = (T)b;
    }
  };

  draw_momenta((uint32_t)sSt.traj, tid, NT);
  for (int t = 0; t < n_traj; ++t) {
    const int sign = sSt.sign;
    const uint32_t traj = (uint32_t)sSt.traj;
    load_field(sign);
    lds_barrier();
    clear_acc();
    site_sums(NU1{}, 5, [&](int o, int64_t, int, int, int, int, int, int, double* v) {
      const double pd = (double)sW[o];
      v[0] = 0.5 * pd * pd;
    });
#pragma unroll
    for (int k = 0; k < NQ; ++k)
      if (act[k]) ldv<T, V>(sW + own[k], pm[k]);
    lds_barrier();
    // kick-drift passes; the last one kicks only
#pragma unroll 1
    for (int j = 0; j < n_pass; ++j) {
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        if (!act[k]) continue;
        T u[V], d[V], a[V], b[V];
        ldv<T, V>(sP + (updn[k] & 0xffffu), u);
        ldv<T, V>(sP + (updn[k] >> 16), d);
        if (NDIM == 3) {
          ldv<T, V>(sP + (zmzp[k] & 0xffffu), a);
          ldv<T, V>(sP + (zmzp[k] >> 16), b);
        }
        const T l = sP[lfrt[k] & 0xffffu], r = sP[lfrt[k] >> 16];
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const T xm = (e == 0) ? l : ps[k][e > 0 ? e - 1 : 0];
          const T xp = right(ps[k], r, k, e);
          T s = (xm + xp) + (u[e] + d[e]);
          if (NDIM == 3) s = s + (a[e] + b[e]);
          const T uu = fma_t(Ct, ps[k][e], s);
          ww[k][e] = fma_t(at, tanh_state(fma_t(at, uu, hw)), -ps[k][e]);
        }
        stv<T, V>(sW + own[k], ww[k]);
      }
      lds_barrier();
      const bool fin = (j == n_pass - 1);
      const T kick = (j == 0 || fin) ? kick_end : ((j & 1) ? kick_odd : kick_even);
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        if (!act[k]) continue;
        T u[V], d[V], a[V], b[V];
        ldv<T, V>(sW + (updn[k] & 0xffffu), u);
        ldv<T, V>(sW + (updn[k] >> 16), d);
        if (NDIM == 3) {
          ldv<T, V>(sW + (zmzp[k] & 0xffffu), a);
          ldv<T, V>(sW + (zmzp[k] >> 16), b);
        }
        const T l = sW[lfrt[k] & 0xffffu], r = sW[lfrt[k] >> 16];
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const T wm = (e == 0) ? l : ww[k][e > 0 ? e - 1 : 0];
          const T wp = right(ww[k], r, k, e);
          T sw = (wm + wp) + (u[e] + d[e]);
          if (NDIM == 3) sw = sw + (a[e] + b[e]);
          T F = fma_t(Ct, ww[k][e], sw);
          F = F + bq[k][e];
          pm[k][e] = fma_t(kick, F, pm[k][e]);
        }
        if (!fin) {
#pragma unroll
          for (int e = 0; e < V; ++e) ps[k][e] = fma_t(drift, pm[k][e], ps[k][e]);
          stv<T, V>(sP + own[k], ps[k]);
        }
      }
      lds_barrier();
    }
    // the final momenta take w's place in LDS for the sums
#pragma unroll
    for (int k = 0; k < NQ; ++k)
      if (act[k]) stv<T, V>(sW + own[k], pm[k]);
    lds_barrier();
    site_sums(NU5{}, 0, [&](int o, int64_t gi, int xm, int xp, int ym, int yp, int zmi, int zpi, double* v) {
      const double pd = (double)sW[o];
      v[0] = 0.5 * pd * pd;
      action_term(o, gi, xm, xp, ym, yp, zmi, zpi, v + 1);
    });
    const uint32_t b = block_totals();
    if (tid == 0) {
      u128 sum[NTERM];
      sum[T_K0] = sSum[5];
      sum[T_K1] = sSum[0];
#pragma unroll
      for (int a = 0; a < 4; ++a) sum[T_S + a] = sSum[1 + a];
      sFlags = finalize_trajectory(cd, &sSt, cur, sum, b, 0.0, &sAcc[traj & 1u]);
    }
    if (t + 1 < n_traj) {
      if (NW == 1) draw_momenta(traj + 1u, tid, NT);
      else if (wave > 0) draw_momenta(traj + 1u, tid - 64, NT - 64);
    }
    lds_barrier();
    if (sFlags & REC_ACCEPT) {
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        if (!act[k]) continue;
#pragma unroll
        for (int e = 0; e < V; ++e) keep[k][e] = ps[k][e];
      }
    }
  }
  // the accepted field back to its buffer and the state (finalize kept cur)
#pragma unroll
  for (int k = 0; k < NQ; ++k)
#pragma unroll
    for (int e = 0; e < V; ++e)
      if (act[k] && e <= last[k]) gpsi[gix[k] + e] = keep[k][e];
  if (tid < (int)(sizeof(ChainState) / 8)) ((uint64_t*)cd.st)[tid] = ((const uint64_t*)&sSt)[tid];
}

// ------------------------------------------------------------------ launch ---

static int vectors(const ChainDev& c, int V) { return (c.L0 + V - 1) / V * c.L1 * c.L2; }

void resident_extend(ResidentShape& s, const ChainDev& c) {
  const int V = c.precision == 4 ? 4 : 2;
  s.max_sites = std::max(s.max_sites, (int)c.N);
  s.max_vectors = std::max(s.max_vectors, vectors(c, V));
  s.max_values = std::max(s.max_values, vectors(c, V) * V);
}

template <typename T, int NDIM>
static hipError_t launch_dim(const ResidentShape& r, const ChainDev* chains, const Tile* tiles, int n, int n_traj,
                             hipStream_t s) {
  constexpr int V = sizeof(T) == 4 ? 4 : 2;
  // One site per thread (V = 1) where a launch leaves SIMDs idle anyway: chains
  // of at most 256 sites, at most four per CU (15 x 15 FP32: 0.28 us a step and
  // 4.5 us a trajectory; beyond that the vectors' fewer instructions count).
  if (r.max_sites <= 256 && n <= 4 * 256) {
    lattice_resident<T, NDIM, 1, 256, 1><<<n, 256, 2 * r.max_sites * sizeof(T), s>>>(chains, tiles, n_traj);
    return hipGetLastError();
  }
  const size_t bytes = 2 * (size_t)r.max_values * sizeof(T);
  // The workgroup that gives each thread one vector, up to 1024 threads; two
  // each above (512 threads with two and four vectors spill at the 128 registers
  // that leave four waves a SIMD: 64 x 64 FP32 1.01 against 0.83 us a step, 17^3
  // 3.6 against 1.8; 1024 chains of 64 x 64 gain 13 % that way, 17^3 lose half).
  if (r.max_vectors <= 64) lattice_resident<T, NDIM, V, 64, 1><<<n, 64, bytes, s>>>(chains, tiles, n_traj);
  else if (r.max_vectors <= 256) lattice_resident<T, NDIM, V, 256, 1><<<n, 256, bytes, s>>>(chains, tiles, n_traj);
  else if (r.max_vectors <= 1024) lattice_resident<T, NDIM, V, 1024, 1><<<n, 1024, bytes, s>>>(chains, tiles, n_traj);
  else if (r.max_vectors <= 2048) lattice_resident<T, NDIM, V, 1024, 2><<<n, 1024, bytes, s>>>(chains, tiles, n_traj);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_lattice_resident(int precision, int ndim, const ResidentShape& r, const ChainDev* chains,
                                   const Tile* tiles, int n_chains, int n_traj, hipStream_t s) {
  if (n_chains <= 0) return hipSuccess;
  if (precision == 4)
    return ndim == 2 ? launch_dim<float, 2>(r, chains, tiles, n_chains, n_traj, s)
                     : launch_dim<float, 3>(r, chains, tiles, n_chains, n_traj, s);
  return ndim == 2 ? launch_dim<double, 2>(r, chains, tiles, n_chains, n_traj, s)
                   : launch_dim<double, 3>(r, chains, tiles, n_chains, n_traj, s);
}

}  // namespace ihmc
