// Fused leap-frog passes for HMC on periodic 2D / 3D nearest-neighbour lattices.
//
// One pass = one force evaluation of the equations of motion (Sec. 3):
//     u = Kt psi,  w = sqrt(J') tanh(sqrt(J') u) - psi,  F = Kt w + h'/sqrt(J'),
// followed by the kick p += c_j F and the drift psi' = psi + d_j p.  F at a
// site needs psi on the radius-2 diamond around it, so a workgroup stages psi
// on its tile plus a 2-wide halo in LDS, computes w on the tile plus a 1-wide
// halo, and then F, p and psi' on the tile: every pass reads psi, p (and the
// per-site field) once and writes p and psi' once.
//
// Pass kinds (template MODE):
//   FIRST   - momenta from Philox (Sec. 3, eq. momentum distribution), 1/2 p^2
//             accumulated for H_old, first kick and drift;
//   MIDDLE  - kick and drift;
//   LAST    - final kick, then the FP64 Hamiltonian and estimator sums of the
//             proposal; the block that finishes last takes the Metropolis
//             decision (Sec. 3) and writes the trajectory record;
//   MEASURE - FP64 action and estimator sums of the accepted field (set-up);
//   FORCE   - writes F itself (diagnostic; same arithmetic as the other passes).
// In 2D two or four MIDDLE steps can also run as one launch (lattice_steps2v), with
// the per-site arithmetic of single passes.
//
// Memory layout: rows padded to `pitch` (a multiple of 4 elements), so a thread
// of the 2D kernel moves its four sites with 16-byte vector accesses.  Sums are
// exact 128-bit fixed point (device_common.hpp): results do not depend on the
// tile shape or on which chains share a launch.
#include <algorithm>
#include <utility>
#include <vector>

#include "chain_epilogue.hpp"
#include "device_common.hpp"
#include "lattice_common.hpp"
#include "lattice_kernels.hpp"

namespace ihmc {

__device__ __forceinline__ int wrap_near(int v, int L) { return v < 0 ? v + L : (v >= L ? v - L : v); }
// v mod L in [0, L) for |v| < 2^22 (lattice coordinates plus a halo): the
// quotient from FP32, exact to within one, then corrected in integers.
__device__ __forceinline__ int wrap_any(int v, int L) {
  const int q = (int)floorf((float)v * __builtin_amdgcn_rcpf((float)L));
  int r = v - q * L;
  r = r < 0 ? r + L : r;
  return r >= L ? r - L : r;
}

// The chain-state words a tiled pass reads at its start (accepted buffer,
// sign, trajectory index) do not change during the launch: only the block that
// closes the chain writes them, after every block of the launch has read them.
// They are read through the constant address space, so with scalar loads, and
// the buffer addresses derived from them stay in scalar registers.
__device__ __forceinline__ int32_t state_word(const int32_t* p) {
  return *(const __attribute__((address_space(4))) int32_t*)p;
}

// Where a staging thread finds its 4-element chunk x .. x+3 of every row it
// loads (x a multiple of 4, at least -4 and, when x_near, below 2 L0 - 4;
// x_near says every x + e lies within one period of [0, L0)): one aligned
// vector load at xv, or, for a chunk that straddles the periodic wrap, the
// four wrapped positions xe.  A wrapped chunk is still one vector load when L0
// is a multiple of 4.  Worked out once per thread, used for all its rows.
struct ChunkPos {
  int xv;
  bool vec;
  int xe[4];
};
__device__ __forceinline__ ChunkPos chunk_pos(int x, int L0, bool x_near) {
  ChunkPos cp;
  const int xs = x_near ? wrap_near(x, L0) : x;
  cp.vec = xs >= 0 && xs + 4 <= L0 && (xs & 3) == 0;
  cp.xv = cp.vec ? xs : 0;
  int xe = x_near ? xs : wrap_any(x, L0);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    cp.xe[e] = xe;
    xe = (xe + 1 == L0) ? 0 : xe + 1;
  }
  return cp;
}

// Every lane issues the vector load (a gathering lane from the row start, and
// discards it), so that the compiler keeps it one 16-byte access.
template <typename T>
__device__ __forceinline__ void load_chunk(const gmem<T>* row, const ChunkPos& cp, T (&v)[4]) {
  ld4g<T>(row + cp.xv, v);
  if (!cp.vec) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = row[cp.xe[e]];
  }
}

// Element offset of a row from its index and the row pitch (both non-negative).
__device__ __forceinline__ uint64_t row_offset(int idx, int64_t stride) {
  return (uint64_t)(uint32_t)idx * (uint64_t)stride;
}

// Workgroups are dealt to the eight XCDs round-robin (block b runs on XCD b % 8),
// each XCD with its own L2.  Neighbouring tiles read the same halo cache lines,
// so each XCD takes a contiguous range of the tile table: block b works on tile
// xcd_tile(b, n), a bijection of [0, n).
__device__ __forceinline__ int xcd_tile(int b, int n) {
  const int q = n >> 3, r = n & 7, k = b & 7, m = b >> 3;
  return k * q + (k < r ? k : r) + m;
}

// A LAST launch may cover chains whose trajectories end at different passes
// (j < 0): each block then takes its chain's own last pass j = n_pass - 1 and
// the launch index of that pass under the round's step plan (k != 0: the j - 1
// middle steps ran k per launch, after launch 0; otherwise launch j).
__device__ __forceinline__ void chain_last_pass(const ChainDev& cd, int& j, int& k) {
  j = cd.n_pass - 1;
  k = k ? 1 + (j - 1 + k - 1) / k : j;
}

// --------------------------------------------------------------------- 2D ---
//
// Tile BX x BY, one thread per quad of four consecutive x (NT = BX/4 * BY).
// LDS rows have pitch RP = BX + 8 with lattice x at index x - x0 + 4, so the
// psi halo [x0-2, x0+BX+2) sits inside one 16-byte aligned row and global and
// LDS traffic moves in aligned quads.  p and the per-site field are fetched
// after the staging, so their latency overlaps the barrier and the stencil
// work without holding up the staging.
template <typename T, int BX, int BY, int MODE>
__global__ __launch_bounds__(BX / 4 * BY) void lattice_pass2v(const ChainDev* __restrict__ chains,
                                                              const Tile* __restrict__ tiles, int n_tiles, int j,
                                                              int k) {
  constexpr int QX = BX / 4;
  constexpr int NT = QX * BY;
  constexpr int NWAVE = (NT + 63) / 64;
  constexpr int RP = BX + 8;
  constexpr int PR = BY + 4;
  constexpr int WR = BY + 2;
  constexpr int NWS = (BX + 2) * WR;
  constexpr int NCH = RP / 4;  // 16-byte chunks per staged row
  constexpr bool kHasW = (MODE != PASS_MEASURE);
  constexpr bool kH64 = (MODE == PASS_LAST || MODE == PASS_MEASURE);
  static_assert(BX % 4 == 0 && NT % 64 == 0, "tile shape");
  __shared__ __align__(16) T sP[PR * RP];
  __shared__ __align__(16) T sW[kHasW ? WR * RP : 4];

  const Tile tl = tiles[xcd_tile(blockIdx.x, n_tiles)];
  const ChainDev& cd = chains[tl.chain];
  ChainState* st = cd.st;
  const int L0 = cd.L0, L1 = cd.L1, pitch = cd.pitch;
  const int64_t NP = cd.NP;
  if (MODE == PASS_LAST && j < 0) chain_last_pass(cd, j, k);
  const int cur = state_word(&st->cur);
  const int sign = state_word(&st->sign);
  const int traj = state_word(&st->traj);
  const bool from_cur = (MODE == PASS_FIRST || MODE == PASS_MEASURE || MODE == PASS_FORCE);
  const int in_buf = from_cur ? cur : lat_in_buf(cur, k);
  const int out_buf = lat_out_buf(cur, k);
  const gmem<T>* __restrict__ pin = (const gmem<T>*)cd.psi + (int64_t)in_buf * NP;
  gmem<T>* __restrict__ pout = (gmem<T>*)cd.psi + (int64_t)out_buf * NP;
  // momenta: read from the buffer of launch k - 1, written to that of launch k
  // (the first, last and force passes use buffer 0)
  const gmem<T>* __restrict__ pmi = (const gmem<T>*)cd.p + (int64_t)lat_p_in(k) * NP;
  gmem<T>* __restrict__ pmo = (gmem<T>*)cd.p + (MODE == PASS_MIDDLE ? (int64_t)lat_p_out(k) * NP : 0);
  const bool site_field = (cd.h_kind == 2);

  const int t = threadIdx.x;
  const int qx = t % QX, qy = t / QX;
  const int gx = tl.x0 + 4 * qx, gy = tl.y0 + qy;
  const bool quad_ok = (gx < L0) && (gy < L1);  // the quad's first site is a lattice site
  const int64_t base = gx + (int64_t)pitch * gy;  // gx + 3 < pitch when quad_ok

  T pq[4] = {(T)0, (T)0, (T)0, (T)0};
  T bq[4];
  const T b_uniform = (T)cd.b0;
  bq[0] = bq[1] = bq[2] = bq[3] = b_uniform;

  // ---- stage psi on the tile plus its halo, in aligned 4-element chunks:
  // a chunk inside [0, L0) is one vector load, a chunk crossing the periodic
  // wrap (or the row end) is gathered element by element.
  // Thread t loads chunk column t % NCH of the rows t / NCH + RG k; all its
  // loads are issued before its LDS stores.
  const bool rows_near = (L1 > BY), x_near = (L0 > BX + 2);
  {
    constexpr int RG = NT / NCH;
    constexpr int NRPT = (PR + RG - 1) / RG;
    const int c = t % NCH, rg = t / NCH;
    if (rg < RG) {
      const ChunkPos cp = chunk_pos(tl.x0 - 4 + 4 * c, L0, x_near);
      T v[NRPT][4];
#pragma unroll
      for (int k = 0; k < NRPT; ++k) {
        const int r = rg + RG * k;
        if (r < PR) {
          const int yy = rows_near ? wrap_near(tl.y0 + r - 2, L1) : wrap_any(tl.y0 + r - 2, L1);
          load_chunk<T>(pin + row_offset(yy, pitch), cp, v[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < NRPT; ++k) {
        const int r = rg + RG * k;
        if (r < PR) {
          if (from_cur) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[k][e] = neg_if(v[k][e], sign);
          }
          st4<T>(sP + r * RP + 4 * c, v[k]);
        }
      }
    }
  }
  // p and the field of the quad, issued after the staged rows' LDS stores
  // (loads complete in issue order: issued earlier, they would hold up the
  // wait for the staged values); their latency overlaps the barrier and w
  if (quad_ok) {
    if (MODE == PASS_MIDDLE || MODE == PASS_LAST || (MODE == PASS_FIRST && cd.p_given)) ld4g<T>(pmi + base, pq);
    if (kHasW && site_field) ld4g<T>((const gmem<T>*)cd.b + base, bq);
  }
  lds_barrier();

  const T Ct = (T)cd.C;
  const T at = (T)cd.sqJ, hw = (T)cd.hw;

  // ---- w on the rows y in [-1, BY], in quads over x in [-4, BX+4): the
  // outermost quads hold unused values (their stencil reaches past the staged
  // halo) but keep every LDS access aligned
  if (kHasW) {
    for (int i = t; i < WR * NCH; i += NT) {
      const int wy = i / NCH, c = i % NCH;
      const int pc = (wy + 1) * RP + 4 * c;  // psi at (x = -4 + 4c, y = wy - 1)
      T cv[4], up[4], dn[4], w[4];
      ld4<T>(sP + pc, cv);
      ld4<T>(sP + pc - RP, up);
      ld4<T>(sP + pc + RP, dn);
      const T lft = sP[pc - 1], rgt = sP[pc + 4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const T xm = (e == 0) ? lft : cv[e - 1];
        const T xp = (e == 3) ? rgt : cv[e + 1];
        const T s = (xm + xp) + (up[e] + dn[e]);
        const T u = fma_t(Ct, cv[e], s);
        w[e] = fma_t(at, tanh_state(fma_t(at, u, hw)), -cv[e]);
      }
      st4<T>(sW + wy * RP + 4 * c, w);
    }
    lds_barrier();
  }

  double kick_d = 0.0, drift_d = 0.0;
  pass_coeffs(cd, j, kick_d, drift_d);
  const T kick = (MODE == PASS_FORCE) ? (T)1 : (T)kick_d;
  const T drift = (T)drift_d;

  uint32_t bad = 0u;
  const bool with_h = kH64 && sums_psih(cd);
  double qs[NTERM];  // FP64 sums of the thread's quad (0 without one)
#pragma unroll
  for (int a = 0; a < NTERM; ++a) qs[a] = 0.0;

  if (quad_ok) {
    // momenta of the first pass: one Philox draw per site pair; with an even
    // row length a pair never straddles a row
    if (MODE == PASS_FIRST && !cd.p_given) {
      const int64_t s0 = gx + (int64_t)L0 * gy;  // logical site of the quad's first element
      if ((L0 & 1) == 0) {
        normal_pair<T>(cd, (uint32_t)traj, TAG_MOM, s0 >> 1, pq[0], pq[1]);
        normal_pair<T>(cd, (uint32_t)traj, TAG_MOM, (s0 >> 1) + 1, pq[2], pq[3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          T z0, z1;
          normal_pair<T>(cd, (uint32_t)traj, TAG_MOM, (s0 + e) >> 1, z0, z1);
          pq[e] = ((s0 + e) & 1) ? z1 : z0;
        }
      }
    }
    T pn[4], pv[4];
    const int pc0 = (qy + 2) * RP + 4 * qx + 4;  // psi of the quad's first site
    const int wc0 = (qy + 1) * RP + 4 * qx + 4;  // w of the quad's first site
    T cv[4];
    ld4<T>(sP + pc0, cv);
    T wcv[4], wup[4], wdn[4];
    if (kHasW) {
      ld4<T>(sW + wc0, wcv);
      ld4<T>(sW + wc0 - RP, wup);
      ld4<T>(sW + wc0 + RP, wdn);
    }
    double kin[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool act = (gx + e < L0);
      const T c = cv[e];
      pv[e] = c;
      pn[e] = pq[e];
      kin[e] = 0.0;
      if (kHasW) {
        const T wm = (e == 0) ? sW[wc0 - 1] : wcv[e - 1];
        const T wp = (e == 3) ? sW[wc0 + 4] : wcv[e + 1];
        const T sw = (wm + wp) + (wup[e] + wdn[e]);
        const T F = fma_t(Ct, wcv[e], sw) + bq[e];
        pn[e] = fma_t(kick, F, (MODE == PASS_FORCE) ? (T)0 : pq[e]);
        pv[e] = fma_t(drift, pn[e], c);
        const double pd = (double)((MODE == PASS_FIRST) ? pq[e] : pn[e]);
        kin[e] = act ? 0.5 * pd * pd : 0.0;
      }
    }
    if (MODE == PASS_FIRST) qs[T_K0] = quad_sum(kin[0], kin[1], kin[2], kin[3]);
    if (MODE == PASS_LAST) qs[T_K1] = quad_sum(kin[0], kin[1], kin[2], kin[3]);
    if (MODE == PASS_FIRST || MODE == PASS_MIDDLE) {
      st4g<T>(pmo + base, pn);
      st4g<T>(pout + base, pv);
    } else if (MODE == PASS_FORCE || (MODE == PASS_LAST && cd.write_p_last)) {
      st4g<T>(pmo + base, pn);
    }
    if (kH64) {
      // pair by pair, one site after the other: few registers, more waves
      const bool ragged = (L0 & 3) != 0;
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        SiteAction t[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          const int pc = pc0 + e + f;
          const double nb =
              ((double)sP[pc - 1] + (double)sP[pc + 1]) + ((double)sP[pc - RP] + (double)sP[pc + RP]);
          t[f] = site_action<true>(cd, (double)sP[pc], nb, base + e + f);
          if (ragged && gx + e + f >= L0) t[f] = no_site();
          __builtin_amdgcn_sched_barrier(0);
        }
        const SiteAction q{t[0].s + t[1].s, t[0].psi + t[1].psi, t[0].ut + t[1].ut, t[0].psih + t[1].psih};
        qs[T_S] = e == 0 ? q.s : qs[T_S] + q.s;  // (t0 + t1) + (t2 + t3), as quad_sum
        qs[T_PSI] = e == 0 ? q.psi : qs[T_PSI] + q.psi;
        qs[T_UT] = e == 0 ? q.ut : qs[T_UT] + q.ut;
        if (with_h) qs[T_PSIH] = e == 0 ? q.psih : qs[T_PSIH] + q.psih;
      }
    }
  }

  if (MODE == PASS_MIDDLE || MODE == PASS_FORCE) return;
  // Terms of 16 x-aligned sites: lanes 4m .. 4m+3 hold four consecutive quads
  // of one tile row (tile widths are multiples of 16), summed in FP64 as
  // (q0 + q1) + (q2 + q3) into every lane of the group; the group's lanes then
  // convert different terms to fixed point: the pass's terms T0 .. T0 + NU - 1
  // in rank order, rank 4r + j by lane j into accR[r].  psi h' comes last: without
  // a field LAST has four terms, one conversion and sum instead of two.
  constexpr int T0 = (MODE == PASS_FIRST) ? T_K0 : ((MODE == PASS_MEASURE) ? T_S : T_K1);
  constexpr int NU = (MODE == PASS_FIRST) ? 1 : ((MODE == PASS_MEASURE) ? 4 : 5);
  constexpr int NR = (NU + 3) / 4;
  static_assert(QX % 4 == 0, "rows of whole 16-site groups");
  const int gl = threadIdx.x & 3;
  const int nu = (MODE != PASS_FIRST && !with_h) ? NU - 1 : NU;
  double gv[NU];
#pragma unroll
  for (int r = 0; r < NU; ++r) gv[r] = r < nu ? quad_sum_all(qs[T0 + r]) : 0.0;
  u128 accR[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    accR[r] = u128{0ull, 0ull};
    if (4 * r >= nu) break;
    double x = 0.0;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj)
      if (4 * r + jj < NU) x = (gl == jj) ? gv[4 * r + jj] : x;
    accR[r] = to_fixed(x, bad);
  }
  const int tix = (tl.y0 / BY) * ((L0 + BX - 1) / BX) + tl.x0 / BX;  // tile index within the chain
  block_accumulate_ranks<MODE, NWAVE, NR>(cd, st, accR, bad, lat_in_buf(cur, k), tix);
}

// ------------------------------------------------------ 2D, several steps ---
//
// Up to STEPS (2 or 4) consecutive middle leap-frog steps j, j + 1, .. in one pass
// over a tile.  psi is staged with a halo of 2 STEPS sites; step s evaluates w on
// the tile plus a ring of 2 (STEPS - s) - 1, and its kick and drift on the tile
// plus a ring one narrower (the ring repeats what the neighbouring tiles compute,
// its momenta and field read from their sites), so psi and p move through memory
// once per launch.  Per site the arithmetic is that of single MIDDLE passes,
// operation for operation, so the results are bit-identical.
//
// Positions outside the lattice (the ragged last tile of a row or column, the
// wrap of small lattices) hold periodic images: psi, p and the field are all
// loaded at wrapped coordinates, so every staged position evolves as the
// lattice site it images.  The ring's momenta are read from other tiles; they
// come from the buffer of launch k - 1 while this launch writes that of launch k,
// so no block reads momenta another block of the launch writes.  A chain with
// fewer middle steps left takes those (at most max_steps), on the rows that these
// need (2 steps of halo in y), and stores its tile (2048^2 FP64, one step left on tiles
// for four: 66 us on all rows, 58 on those).  FULL: on all rows whatever is left (their
// number known, FP32 launches take 2 % less: 2048^2 199 -> 195 us a trajectory of 20; a
// body for each number in one kernel costs small launches 1 to 2 %).
//
// A thread owns H consecutive rows of one 4-site chunk column (a strip) and keeps
// their momenta, psi and field in registers for all steps; LDS holds psi and w.
// Marching down a strip each row is read once from LDS (16 bytes) instead of three
// times, every LDS address is a constant offset, and the two sites beside a chunk
// come from the neighbouring lanes (a wave-wide DPP shift; the lanes at the wave's
// ends read theirs from LDS): reading them from LDS conflicts four ways, 45 % of
// the CU's cycles.  The tile's extent is the plan's choice (choose_steps), packed
// into Tile::z0 as bx | by << 16; bx is a multiple of 4.
//
// Bound by VALU issue once launches fill the chip (99 % of the cycles on 8192^2, 80 %
// on 698 chains with a field; 42 VALU instructions a site and step there, 26 of them
// FP32 arithmetic, 3 transcendental, the ring's included), by latency below that
// (1024^2: 5.7 us of issue in 10.0).  Per step, against two steps per launch on 64
// x 16 tiles with one quad a thread: 4096^2 FP32 32.5 -> 23.2 us, 1024^2 3.98 ->
// 2.64, 256^2 2.04 -> 1.30, 600 chains of 64 .. 256 sites a row with a field 36.0 ->
// 22.1; 251 x 130 FP64 4.88 -> 2.61.  Two and three steps a launch measured 30.5 and
// 24.8 us on 4096^2, five and six 26 and 27 on the chains.
// Value of the lane before (wave_left) or after (wave_right) in the wave; the
// first or last lane takes `edge`.
template <int CTRL>
__device__ __forceinline__ uint32_t wave_shift_u32(uint32_t edge, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ float wave_shift(float edge, float v) {
  return __uint_as_float(wave_shift_u32<CTRL>(__float_as_uint(edge), __float_as_uint(v)));
}
template <int CTRL>
__device__ __forceinline__ double wave_shift(double edge, double v) {
  const uint64_t e = (uint64_t)__double_as_longlong(edge), x = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = wave_shift_u32<CTRL>((uint32_t)e, (uint32_t)x);
  const uint32_t hi = wave_shift_u32<CTRL>((uint32_t)(e >> 32), (uint32_t)(x >> 32));
  return __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32)));
}
constexpr int DPP_WAVE_SHR1 = 0x138;  // lane l - 1
constexpr int DPP_WAVE_SHL1 = 0x130;  // lane l + 1

constexpr int MS_BX = 64;  // widest tile

template <typename T, int STEPS, int H, bool THROUGH, bool FULL>
__global__ __launch_bounds__(1024, 4) void lattice_steps2v(const ChainDev* __restrict__ chains,
                                                        const Tile* __restrict__ tiles, int n_tiles, int j, int k,
                                                        int max_steps) {
  constexpr int HALO = 2 * STEPS;             // staged on every side
  constexpr int HCH = HALO / 4;               // the same in chunks
  constexpr int RP = MS_BX + 2 * HALO;        // LDS row pitch
  static_assert(HALO % 4 == 0, "whole chunks of halo");
  extern __shared__ __align__(16) unsigned char lds[];
  const Tile tl = tiles[xcd_tile(blockIdx.x, n_tiles)];
  const ChainDev& cd = chains[tl.chain];
  const ChainState* st = cd.st;
  const int L0 = cd.L0, L1 = cd.L1, pitch = cd.pitch;
  const int64_t NP = cd.NP;
  const int cur = state_word(&st->cur);
  const gmem<T>* __restrict__ pin = (const gmem<T>*)cd.psi + (int64_t)lat_in_buf(cur, k) * NP;
  gmem<T>* __restrict__ pout = (gmem<T>*)cd.psi + (int64_t)lat_out_buf(cur, k) * NP;
  const gmem<T>* __restrict__ pmi = (const gmem<T>*)cd.p + (int64_t)lat_p_in(k) * NP;
  gmem<T>* __restrict__ pmo = (gmem<T>*)cd.p + (int64_t)lat_p_out(k) * NP;
  const gmem<T>* __restrict__ bfield = (const gmem<T>*)cd.b;
  const bool site_field = (cd.h_kind == 2);
  const int bx = tl.z0 & 0xffff, by = tl.z0 >> 16;
  const int nch = bx / 4 + 2 * HCH;             // chunks of a staged row
  const int ns = min(max_steps, cd.n_pass - 1 - j);  // steps taken
  const int hy = FULL ? HALO : 2 * ns;               // rows of halo that they need
  const int prow = by + 2 * hy, wrow = prow - 2;  // staged rows; w rows of the first step
  const int nst = (wrow + H - 1) / H;             // strips of a chunk column
  const bool rows_near = (L1 >= by + HALO), x_near = (L0 >= bx + HALO);
  auto lat_row = [&](int y) { return rows_near ? wrap_near(y, L1) : wrap_any(y, L1); };
  T* const sP = reinterpret_cast<T*>(lds);
  T* const sW = sP + (nst * H + 2) * RP;

  const int t = threadIdx.x;
  const int strip = t / nch, c = t - strip * nch;
  const ChunkPos cp = chunk_pos(tl.x0 - HALO + 4 * c, L0, x_near);
  // ---- stage psi: row r of the staged rows is lattice row y0 + r - hy; each
  // thread loads its chunk column of every nsg-th row, all loads before the stores
  // (nsg >= nst strips, so H + 1 rows a thread cover the prow <= H nst + 2 rows)
  {
    const int nsg = (int)blockDim.x / nch;
    T v[H + 1][4];
    if (strip < nsg) {
#pragma unroll
      for (int q = 0; q < H + 1; ++q) {
        const int r = strip + nsg * q;
        if (r < prow) load_chunk<T>(pin + row_offset(lat_row(tl.y0 + r - hy), pitch), cp, v[q]);
      }
#pragma unroll
      for (int q = 0; q < H + 1; ++q) {
        const int r = strip + nsg * q;
        if (r < prow) st4<T>(sP + r * RP + 4 * c, v[q]);
      }
    }
  }
  // ---- momenta and field of the strip's kick rows r0 .. r0 + H - 1 (row 0 is
  // lattice row y0 - (hy - 2)), issued behind the staging (loads complete in
  // issue order) and first used by the kick
  const bool act = strip < nst;
  const int r0 = strip * H;
  T pm[H][4], bq[H][4], ps[H][4];
  const T b_uniform = (T)cd.b0;
#pragma unroll
  for (int i = 0; i < H; ++i) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      bq[i][e] = b_uniform;
      pm[i][e] = (T)0;
    }
    if (act && r0 + i < wrow - 2) {
      const uint64_t o = row_offset(lat_row(tl.y0 + r0 + i - (hy - 2)), pitch);
      load_chunk<T>(pmi + o, cp, pm[i]);
      if (site_field) load_chunk<T>(bfield + o, cp, bq[i]);
    }
  }
  lds_barrier();

  const T Ct = (T)cd.C, at = (T)cd.sqJ, hw = (T)cd.hw;
  // w row q and kick row q lie one and two rows below psi row q; the edge lanes'
  // neighbours (others read the first lane's: one address, no conflict)
  const int off0 = r0 * RP + 4 * c;
  const int eoff = (t & 63) == 63 ? off0 + 4 : max(0, __builtin_amdgcn_readfirstlane(off0) - 1);
  T* const pc = sP + off0;
  T* const wc = sW + off0;
  const T* const pe = sP + eoff;
  const T* const we = sW + eoff;
  if (act) {
#pragma unroll
    for (int i = 0; i < H; ++i) ld4<T>(pc + (i + 2) * RP, ps[i]);
  }
#pragma unroll 1
  for (int s = 0; s < ns; ++s) {
    // w on the rows the remaining steps need
    if (act && r0 + H > 2 * s && r0 < wrow - 2 * s) {
      T u[4], m[4], d[4];
      ld4<T>(pc, u);
      ld4<T>(pc + RP, m);
#pragma unroll
      for (int i = 0; i < H; ++i) {
        ld4<T>(pc + (i + 2) * RP, d);
        const T edge = pe[(i + 1) * RP];
        const T lft = wave_shift<DPP_WAVE_SHR1>(edge, m[3]), rgt = wave_shift<DPP_WAVE_SHL1>(edge, m[0]);
        T w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const T xm = (e == 0) ? lft : m[e - 1];
          const T xp = (e == 3) ? rgt : m[e + 1];
          const T sum = (xm + xp) + (u[e] + d[e]);
          const T uu = fma_t(Ct, m[e], sum);
          w[e] = fma_t(at, tanh_state(fma_t(at, uu, hw)), -m[e]);
        }
        st4<T>(wc + i * RP, w);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          u[e] = m[e];
          m[e] = d[e];
        }
      }
    }
    lds_barrier();
    if (act && r0 + H > 2 * s && r0 < wrow - 2 - 2 * s) {
      double kick_d = 0.0, drift_d = 0.0;
      pass_coeffs(cd, j + s, kick_d, drift_d);
      const T kick = (T)kick_d, drift = (T)drift_d;
      T u[4], m[4], d[4];
      ld4<T>(wc, u);
      ld4<T>(wc + RP, m);
#pragma unroll
      for (int i = 0; i < H; ++i) {
        ld4<T>(wc + (i + 2) * RP, d);
        const T edge = we[(i + 1) * RP];
        const T lft = wave_shift<DPP_WAVE_SHR1>(edge, m[3]), rgt = wave_shift<DPP_WAVE_SHL1>(edge, m[0]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const T wm = (e == 0) ? lft : m[e - 1];
          const T wp = (e == 3) ? rgt : m[e + 1];
          const T sw = (wm + wp) + (u[e] + d[e]);
          const T F = fma_t(Ct, m[e], sw) + bq[i][e];
          pm[i][e] = fma_t(kick, F, pm[i][e]);
          ps[i][e] = fma_t(drift, pm[i][e], ps[i][e]);
        }
        st4<T>(pc + (i + 2) * RP, ps[i]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          u[e] = m[e];
          m[e] = d[e];
        }
      }
    }
    if (s + 1 < ns) lds_barrier();
  }
  const int gx = tl.x0 - HALO + 4 * c;
  const int64_t base0 = (int64_t)pitch * tl.y0;  // the tile's first row
  if (act && c >= HCH && c < nch - HCH && gx < L0) {
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int ty = r0 + i - (hy - 2), gy = tl.y0 + ty;
      if (ty >= 0 && ty < by && gy < L1) {
        const int64_t base = gx + (int64_t)pitch * gy;  // gx + 3 < pitch
        if constexpr (THROUGH) {
          // at most 64 rows of 2^20 values
          st4_through((float*)(pmo + base0), base - base0, vf4{pm[i][0], pm[i][1], pm[i][2], pm[i][3]});
          st4_through((float*)(pout + base0), base - base0, vf4{ps[i][0], ps[i][1], ps[i][2], ps[i][3]});
        } else {
          st4g<T>(pmo + base, pm[i]);
          st4g<T>(pout + base, ps[i]);
        }
      }
    }
  }
}

enum class StoreKind { plain, through, nontemporal };

template <StoreKind ST, typename T>
__device__ __forceinline__ void store_as(gmem<T>* p, T v) {
  if constexpr (ST == StoreKind::through) st_through(p, v);
  else if constexpr (ST == StoreKind::nontemporal) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// ------------------------------------------------------------ 3D, one phase ---
//
// A block owns a BX x BY x ZR box, one thread per x-y column and aligned
// 4-plane slab (256 threads per slab: the LDS a box stages allows four boxes
// per CU, so an 8-plane box runs eight waves rather than four, to hide the
// latency of a chain too small to fill the GPU).  psi on the box plus its
// 2-wide halo is staged in LDS in one phase, in aligned 4-element chunks (rows
// of RP = BX + 8 values with lattice x at x - x0 + 4, as in 2D), so every load
// of the block is in flight at once; w on the box plus its 1-wide halo follows
// in quads (the outermost quad of a row is unused), then each thread updates
// its column's slab plane by plane.  The momenta and field values of the slab
// are fetched before the staging.  Sums of the FP64 terms follow the same
// order as in every other tiling: per column over each 4-plane slab in z order,
// then per x-aligned quad of columns.
template <typename T, int BX, int BY, int ZR, int MODE, StoreKind ST = StoreKind::plain>
__global__ __launch_bounds__(64 * ZR, 8) void lattice_pass3t(const ChainDev* __restrict__ chains,
                                                          const Tile* __restrict__ tiles, int n_tiles, int j,
                                                          int k) {
  constexpr int NT = 64 * ZR;  // 256 threads per 4-plane slab
  constexpr int RP = BX + 8;
  constexpr int NCH = RP / 4;  // 16-byte chunks per staged row
  constexpr int PR = BY + 4, PZ = ZR + 4;
  constexpr int WR = BY + 2, WZ = ZR + 2;
  constexpr int PPL = PR * RP, WPL = WR * RP;
  constexpr bool kHasW = (MODE != PASS_MEASURE);
  constexpr bool kH64 = (MODE == PASS_LAST || MODE == PASS_MEASURE);
  static_assert(BX * BY == 256 && BX % 4 == 0 && ZR % 4 == 0, "one column and slab per thread");
  __shared__ __align__(16) T sP[PZ * PPL];
  __shared__ __align__(16) T sW[kHasW ? WZ * WPL : 4];

  const Tile tl = tiles[xcd_tile(blockIdx.x, n_tiles)];
  const ChainDev& cd = chains[tl.chain];
  ChainState* st = cd.st;
  if (MODE == PASS_LAST && j < 0) chain_last_pass(cd, j, k);
  const int L0 = cd.L0, L1 = cd.L1, L2 = cd.L2, pitch = cd.pitch;
  const int64_t NP = cd.NP;
  const int64_t plane = (int64_t)pitch * L1;
  const int cur = state_word(&st->cur);
  const int sign = state_word(&st->sign);
  const int traj = state_word(&st->traj);
  const bool from_cur = (MODE == PASS_FIRST || MODE == PASS_MEASURE || MODE == PASS_FORCE);
  const int in_buf = from_cur ? cur : lat_in_buf(cur, k);
  const int out_buf = lat_out_buf(cur, k);
  const gmem<T>* __restrict__ pin = (const gmem<T>*)cd.psi + (int64_t)in_buf * NP;
  gmem<T>* __restrict__ pout = (gmem<T>*)cd.psi + (int64_t)out_buf * NP;
  gmem<T>* __restrict__ pmom = (gmem<T>*)cd.p;
  const int z_end = min(tl.z0 + ZR, L2);
  const T b_uniform = (T)cd.b0;
  const gmem<T>* __restrict__ bsite = (const gmem<T>*)cd.b;
  const bool site_field = (cd.h_kind == 2);

  // ---- the momenta and field values of the thread's column and slab (planes
  // kz0 .. kz0 + 3 of the box)
  const int kz0 = 4 * (threadIdx.x / 256);
  const int lx = threadIdx.x % BX, ly = (threadIdx.x % 256) / BX;
  const int gx = tl.x0 + lx, gy = tl.y0 + ly;
  const bool act = (gx < L0) && (gy < L1);
  const int64_t col = gx + (int64_t)pitch * gy;
  constexpr bool kLoadP = (MODE == PASS_MIDDLE || MODE == PASS_LAST || MODE == PASS_FIRST);
  const bool load_p = kLoadP && act && (MODE != PASS_FIRST || cd.p_given);
  const bool load_b = kHasW && act && site_field;
  T pcol[4], bcol[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    pcol[k] = (T)0;
    bcol[k] = b_uniform;
    if (tl.z0 + kz0 + k < z_end) {
      if (load_p) pcol[k] = pmom[col + plane * (tl.z0 + kz0 + k)];
      if (load_b) bcol[k] = bsite[col + plane * (tl.z0 + kz0 + k)];
    }
  }

  // ---- stage psi on the box plus its halo: thread t owns chunk column c of
  // staged row r (each of the NCH * PR pairs has NH threads) and loads it in a
  // run of consecutive planes, so the row's wrap and offset are worked out
  // once; all its loads are issued before its LDS stores
  const bool rows_near = (L1 > BY), planes_near = (L2 > ZR), x_near = (L0 > BX + 2);
  {
    constexpr int NPAIR = NCH * PR;
    constexpr int NH = NT / NPAIR;
    constexpr int NPP = (PZ + NH - 1) / NH;  // planes per thread
    static_assert(NH >= 1, "box row too long for one block");
    const int pair = threadIdx.x % NPAIR, h = threadIdx.x / NPAIR;
    const int c = pair % NCH, r = pair / NCH;
    const int pz0 = h * NPP;
    T v[NPP][4];
    if (h < NH) {
      const ChunkPos cp = chunk_pos(tl.x0 - 4 + 4 * c, L0, x_near);
      const int yy = rows_near ? wrap_near(tl.y0 + r - 2, L1) : wrap_any(tl.y0 + r - 2, L1);
      const gmem<T>* rowy = pin + row_offset(yy, pitch);
      int zz = planes_near ? wrap_near(tl.z0 + pz0 - 2, L2) : wrap_any(tl.z0 + pz0 - 2, L2);
#pragma unroll
      for (int k = 0; k < NPP; ++k) {
        if (pz0 + k < PZ) load_chunk<T>(rowy + row_offset(zz, plane), cp, v[k]);
        zz = (zz + 1 == L2) ? 0 : zz + 1;
      }
    }
    // momenta of the first pass while the loads are in flight: one Philox draw
    // per site pair.  With an even row length the pair of column x (even) is
    // (x, x + 1), held by the neighbouring lane; over two planes the even lane
    // draws the pair of plane k, the odd lane that of plane k + 1, and each
    // passes its partner the partner's value.
    if (MODE == PASS_FIRST && !cd.p_given && (L0 & 1) == 0) {
      const bool even = (gx & 1) == 0;
#pragma unroll
      for (int k = 0; k < 4; k += 2) {
        const int64_t z = tl.z0 + kz0 + k + (even ? 0 : 1);
        const int64_t site = (gx & ~1) + (int64_t)L0 * (gy + (int64_t)L1 * z);
        T z0, z1;
        normal_pair<T>(cd, (uint32_t)traj, TAG_MOM, site >> 1, z0, z1);
        const T other = __shfl_xor(even ? z1 : z0, 1, 64);
        pcol[k] = even ? z0 : other;
        pcol[k + 1] = even ? other : z1;
      }
    }
    if (h < NH) {
#pragma unroll
      for (int k = 0; k < NPP; ++k) {
        if (pz0 + k < PZ) {
          if (from_cur) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[k][e] = neg_if(v[k][e], sign);
          }
          st4<T>(sP + (pz0 + k) * PPL + r * RP + 4 * c, v[k]);
        }
      }
    }
  }
  lds_barrier();

  const T Ct = (T)cd.C;
  const T at = (T)cd.sqJ, hw = (T)cd.hw;

  // ---- w on the box plus its 1-wide halo, in quads over x in [-4, BX+4):
  // thread t computes chunk column t % NCH of the w rows t / NCH + RG k
  if (kHasW) {
    constexpr int NWROW = WZ * WR;
    constexpr int RG = NT / NCH;
    constexpr int NIT = (NWROW + RG - 1) / RG;
    const int c = threadIdx.x % NCH, rg = threadIdx.x / NCH;
#pragma unroll
    for (int k = 0; k < NIT; ++k) {
      const int R = rg + RG * k;
      if (rg >= RG || R >= NWROW) break;
      const int wz = R / WR, wy = R - wz * WR;
      const int pc = (wz + 1) * PPL + (wy + 1) * RP + 4 * c;  // psi at (x0 - 4 + 4c, y0 - 1 + wy, z0 - 1 + wz)
      T cv[4], up[4], dn[4], zm[4], zp[4], w[4];
      ld4<T>(sP + pc, cv);
      ld4<T>(sP + pc - RP, up);
      ld4<T>(sP + pc + RP, dn);
      ld4<T>(sP + pc - PPL, zm);
      ld4<T>(sP + pc + PPL, zp);
      const T lft = sP[pc - 1], rgt = sP[pc + 4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const T xm = (e == 0) ? lft : cv[e - 1];
        const T xp = (e == 3) ? rgt : cv[e + 1];
        T sum = (xm + xp) + (up[e] + dn[e]);
        sum = sum + (zm[e] + zp[e]);
        const T u = fma_t(Ct, cv[e], sum);
        w[e] = fma_t(at, tanh_state(fma_t(at, u, hw)), -cv[e]);
      }
      st4<T>(sW + wz * WPL + wy * RP + 4 * c, w);
    }
    lds_barrier();
  }

  double kick_d = 0.0, drift_d = 0.0;
  pass_coeffs(cd, j, kick_d, drift_d);
  const T kick = (MODE == PASS_FORCE) ? (T)1 : (T)kick_d;
  const T drift = (T)drift_d;

  // FP64 terms are summed per column over each aligned 4-plane slab (in z
  // order), then per x-aligned quad of columns, and converted to fixed point
  // once per slab and quad: the same grouping for every box depth.  The quad's
  // four lanes hold the same sums and deal the conversions: the pass's terms
  // T0 .. T0 + NU - 1 in rank order, rank 4k + j converted by lane j into accR[k].
  static_assert(ZR % 4 == 0, "boxes are whole 4-plane slabs");
  constexpr bool kAcc = (MODE == PASS_FIRST || MODE == PASS_LAST || MODE == PASS_MEASURE);
  constexpr int T0 = (MODE == PASS_FIRST) ? T_K0 : ((MODE == PASS_MEASURE) ? T_S : T_K1);
  constexpr int NU = (MODE == PASS_FIRST) ? 1 : ((MODE == PASS_MEASURE) ? 4 : 5);
  constexpr int NR = (NU + 3) / 4;
  const int ql = threadIdx.x & 3;
  uint32_t bad = 0u;
  const bool with_h = kH64 && sums_psih(cd);
  const int nu = (MODE != PASS_FIRST && !with_h) ? NU - 1 : NU;
  double hs[NTERM];
  u128 accR[NR];
#pragma unroll
  for (int a = 0; a < NTERM; ++a) hs[a] = 0.0;
#pragma unroll
  for (int r = 0; r < NR; ++r) accR[r] = u128{0ull, 0ull};

#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int k = kz0 + kk;  // plane of the box
    const int z = tl.z0 + k;
    if (z < z_end) {
      const int64_t idx = col + plane * z;
      const int c = (k + 2) * PPL + (ly + 2) * RP + lx + 4;
      const T v = sP[c];
      double kin = 0.0;
      if (kHasW && act) {
        const int q = (k + 1) * WPL + (ly + 1) * RP + lx + 4;
        T sw = (sW[q - 1] + sW[q + 1]) + (sW[q - RP] + sW[q + RP]);
        sw = sw + (sW[q - WPL] + sW[q + WPL]);
        T F = fma_t(Ct, sW[q], sw);
        F = F + bcol[kk];
        T p;
        if (MODE == PASS_FIRST) {
          if (cd.p_given || (L0 & 1) == 0) {
            p = pcol[kk];
          } else {
            const int64_t site = gx + (int64_t)L0 * (gy + (int64_t)L1 * z);
            T z0, z1;
            normal_pair<T>(cd, (uint32_t)traj, TAG_MOM, site >> 1, z0, z1);
            p = (site & 1) ? z1 : z0;
          }
          const double pd = (double)p;
          kin = 0.5 * pd * pd;
        } else if (MODE == PASS_FORCE) {
          p = (T)0;
        } else {
          p = pcol[kk];
        }
        const T pn = fma_t(kick, F, p);
        if (MODE == PASS_FIRST || MODE == PASS_MIDDLE) {
          const T vn = fma_t(drift, pn, v);
          store_as<ST>(pmom + idx, pn);
          store_as<ST>(pout + idx, vn);
        } else if (MODE == PASS_FORCE) {
          pmom[idx] = pn;
        } else if (MODE == PASS_LAST) {
          if (cd.write_p_last) pmom[idx] = pn;
          const double pd = (double)pn;
          kin = 0.5 * pd * pd;
        }
      }
      if (MODE == PASS_FIRST) hs[T_K0] = hs[T_K0] + kin;
      if (MODE == PASS_LAST) hs[T_K1] = hs[T_K1] + kin;
      if (kH64) {
        double nb = ((double)sP[c - 1] + (double)sP[c + 1]) + ((double)sP[c - RP] + (double)sP[c + RP]);
        nb = nb + ((double)sP[c - PPL] + (double)sP[c + PPL]);
        // computed in every lane: as a branch, waves with a few columns in the lattice (rows of
        // 33 or 34 sites) took longer than whole ones (34 x 33 x 24, last pass: 12.2 us, 10.8 so)
        SiteAction sa = site_action<true>(cd, (double)v, nb, act ? idx : 0);
        if (!act) sa = no_site();
        hs[T_S] = hs[T_S] + sa.s;
        hs[T_PSI] = hs[T_PSI] + sa.psi;
        hs[T_UT] = hs[T_UT] + sa.ut;
        if (with_h) hs[T_PSIH] = hs[T_PSIH] + sa.psih;
      }
    }
    // end of a slab: every lane takes part (the quad sums shuffle across the wave)
    if (kAcc && kk == 3) {
      double qv[NU];
#pragma unroll
      for (int r = 0; r < NU; ++r) qv[r] = r < nu ? quad_sum_all(hs[T0 + r]) : 0.0;
#pragma unroll
      for (int kr = 0; kr < NR; ++kr) {
        if (4 * kr >= nu) break;
        double x = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (4 * kr + j < NU) x = (ql == j) ? qv[4 * kr + j] : x;
        accR[kr] = to_fixed(x, bad);
      }
    }
  }

  if (MODE == PASS_MIDDLE || MODE == PASS_FORCE) return;
  const int tix = ((tl.z0 / ZR) * ((L1 + BY - 1) / BY) + tl.y0 / BY) * ((L0 + BX - 1) / BX) + tl.x0 / BX;
  block_accumulate_ranks<MODE, NT / 64, NR>(cd, st, accR, bad, lat_in_buf(cur, k), tix);
}

// ------------------------------------------------------------------ launch ---

// Tile of one chain under a shape: equal tiles of at most bx x by sites, with no
// more rows than `threads` threads can hold in strips of H.
static void steps_tile(const StepShape& g, int L0, int L1, int& bx, int& by, int& threads, int& rows) {
  const int nx = (L0 + g.bx - 1) / g.bx;
  bx = ((L0 + nx - 1) / nx + 3) / 4 * 4;
  const int nch = bx / 4 + g.steps, ring = 4 * g.steps - 2;  // chunks of a staged row; rows a kick adds to a tile's
  const int by_max = std::min(g.by, g.max_threads / nch * g.H - ring);
  const int ny = (L1 + by_max - 1) / by_max;
  by = (L1 + ny - 1) / ny;
  const int nst = (by + ring + g.H - 1) / g.H;
  threads = (nst * nch + 63) / 64 * 64;
  rows = nst * g.H + 2;
}

// What a launch over the lattices takes under a shape; sets the shape's workgroup size
// and LDS rows.
struct StepLoad {
  int64_t tiles = 0, waves = 0;
  int wmax = 0;  // waves of the largest workgroup
};
static StepLoad steps_load(StepShape& g, const std::vector<std::pair<int, int>>& lattices) {
  StepLoad c;
  for (const auto& l : lattices) {
    int bx, by, thr, rows;
    steps_tile(g, l.first, l.second, bx, by, thr, rows);
    const int64_t n = (int64_t)((l.first + bx - 1) / bx) * ((l.second + by - 1) / by);
    c.tiles += n;
    c.waves += n * (thr / 64);
    c.wmax = std::max(c.wmax, thr / 64);
    g.threads = std::max(g.threads, thr);
    g.rows = std::max(g.rows, rows);
  }
  return c;
}

// Shape of the several-steps launches over a set of chains: the one that gives the
// fullest CU the fewest wave-rows (waves x H, four SIMDs at a time).  Tiles of 64
// x 64 repeat the least ring, 16 x 16 spread a small lattice over the CUs (256^2
// FP32, per step: 1.30 us on 16 x 16, 1.41 on 32 x 16, 2.0 on 64 x 64; 1024^2:
// 2.64 on 64 x 64 with H = 2, 2.87 with H = 3, 3.3 on 32 x 32).  Launches of more
// than 1024 tiles keep every CU busy, so the mean counts, and workgroups of 512
// threads at most, three of which share a CU (4096^2: H = 3 at 512 threads 23.2
// us, H = 2 24.8, H = 3 at 768 threads 25.7).
//
// A workgroup alone on its CU waits for LDS and transcendentals, so of equal costs there
// the one with more waves is taken (512^2 FP32: 32 x 32 with H = 3 62.9 us a trajectory
// of 20 steps, with H = 1 53.7).
//
// FP64 launches of more than 1024 tiles of 64 x 50 take two steps: the ring of four costs
// more there than the passes over memory that it saves, and LDS leaves one workgroup a CU
// to 64 x 64 tiles, two to 64 x 50 (us a trajectory of 20 steps, four and two a launch:
// 2048^2 893 and 814, 3000 x 2000 1288 and 1072, 64 chains of 256^2 890 and 800; below the
// line 1024^2 250 and 263, 256 chains of 100 x 90 524 and 557).  Smaller FP64 sets leave
// out shapes of more than 1024 tiles, whose narrow tiles the cost flatters (1128^2 32 x 28
// 510, 64 x 36 375).
//
// Chains of at most two middle steps stage the halo of two (max_middle; 520^2 FP64, n_md =
// 3: 49.6 -> 43.7 us a trajectory, 512^2 FP32 30.2 -> 29.1).
StepShape choose_steps(int precision, const std::vector<std::pair<int, int>>& lattices, int max_middle) {
  if (precision == 8) {
    StepShape g{2, 64, 64, 2, 512};
    if (steps_load(g, lattices).tiles > 1024) return g;
  }
  const int steps = max_middle > 2 ? LAT_STEPS : 2;
  StepShape best;
  StepLoad bl;
  double best_cost = 0.0;
  static const int kExtent[][2] = {{64, 64}, {64, 32}, {32, 32}, {32, 16}, {16, 16}};
  for (const auto& ex : kExtent)
    for (int H = precision == 4 ? 3 : 2; H >= 1; --H)
      for (int cap : {512, 1024}) {
        StepShape g{steps, ex[0], ex[1], H, cap};
        const StepLoad c = steps_load(g, lattices);
        const bool full = c.tiles > 1024;
        if (full && (cap == 1024 || (precision == 8 && (steps == 4 || ex[0] < 64)))) continue;
        const double cost =
            full ? (double)c.waves * H / 1024.0 : (double)(((c.tiles + 255) / 256 * c.wmax + 3) / 4 * H);
        const int64_t rows = c.waves * H, best_rows = bl.waves * best.H;
        const bool tie = cost == best_cost && c.tiles <= 256 && bl.tiles <= 256 &&
                         (steps == 2 && rows != best_rows ? rows < best_rows : H < best.H);
        if (best.H == 0 || cost < best_cost || tie) {
          best = g;
          bl = c;
          best_cost = cost;
        }
      }
  return best;
}

void steps_tiles(const StepShape& g, int chain, int L0, int L1, std::vector<Tile>& out) {
  int bx, by, thr, rows;
  steps_tile(g, L0, L1, bx, by, thr, rows);
  for (int y = 0; y < L1; y += by)
    for (int x = 0; x < L0; x += bx) out.push_back(Tile{chain, x, y, bx | (by << 16)});
}

template <typename T, int STEPS, int H, bool THROUGH, bool FULL>
static void launch_steps(const StepShape& g, const ChainDev* chains, const Tile* tiles, int n_tiles, int j, int k,
                         int max_steps, hipStream_t s) {
  const size_t lds = 2 * (size_t)g.rows * (MS_BX + 4 * STEPS) * sizeof(T);
  lattice_steps2v<T, STEPS, H, THROUGH, FULL>
      <<<(unsigned)n_tiles, (unsigned)g.threads, lds, s>>>(chains, tiles, n_tiles, j, k, max_steps);
}

template <typename T, int STEPS, bool THROUGH, bool FULL>
static void launch_steps_h(const StepShape& g, const ChainDev* chains, const Tile* tiles, int n_tiles, int j, int k,
                           int max_steps, hipStream_t s) {
  if (g.H == 1) return launch_steps<T, STEPS, 1, THROUGH, FULL>(g, chains, tiles, n_tiles, j, k, max_steps, s);
  if (g.H == 2) return launch_steps<T, STEPS, 2, THROUGH, FULL>(g, chains, tiles, n_tiles, j, k, max_steps, s);
  if constexpr (sizeof(T) == 4)
    launch_steps<T, STEPS, 3, THROUGH, FULL>(g, chains, tiles, n_tiles, j, k, max_steps, s);
}

hipError_t launch_lattice_steps(int precision, const StepShape& g, const ChainDev* chains, const Tile* tiles,
                                int n_tiles, int j, int k, int max_steps, bool full, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  if (max_steps < 1 || max_steps > g.steps || g.threads < 64 || g.threads > 1024) return hipErrorInvalidValue;
  if ((g.steps != 2 && g.steps != 4) || g.H < 1 || g.H > (precision == 4 ? 3 : 2)) return hipErrorInvalidValue;
  if (precision == 4) {
    // Stores through the L2 where CUs hold more than one workgroup, so that others run while
    // one stores (us a trajectory: 1024^2 88 -> 84, 1448^2 145 -> 134, 100 x 90 x 256
    // 103 -> 97, 512^2 x 8 88 -> 83; one a CU: 100 x 90 x 64 47.0 -> 47.7, 256^2 43.9 ->
    // 44.3), up to what the L2s hold: sets beyond write back within the launch anyway, and
    // the parts of lines at ragged rows' ends go out twice (a set of 4096 uneven chains
    // 3.64e11 -> 3.55e11 site-MD-steps/s).  Not in FP64, whose two 16-byte stores a chunk
    // each cover half of every 32 bytes (512^2 x 16 566 -> 596, 2048^2 890 -> 932).
    const bool through = n_tiles > 256 && n_tiles <= 2048;
    auto launch = g.steps == 2 ? (through ? launch_steps_h<float, 2, true, false> : launch_steps_h<float, 2, false, false>)
                  : full       ? (through ? launch_steps_h<float, 4, true, true> : launch_steps_h<float, 4, false, true>)
                               : (through ? launch_steps_h<float, 4, true, false> : launch_steps_h<float, 4, false, false>);
    launch(g, chains, tiles, n_tiles, j, k, max_steps, s);
  } else if (g.steps == 4) {
    launch_steps_h<double, 4, false, false>(g, chains, tiles, n_tiles, j, k, max_steps, s);
  } else {
    launch_steps_h<double, 2, false, false>(g, chains, tiles, n_tiles, j, k, max_steps, s);
  }
  return hipGetLastError();
}

template <typename T, int BX, int BY>
static hipError_t launch_mode2v(int mode, const ChainDev* chains, const Tile* tiles, int n_tiles, int j, int k,
                                hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  dim3 grid(n_tiles), block(BX / 4 * BY);
  switch (mode) {
    case PASS_FIRST:
      lattice_pass2v<T, BX, BY, PASS_FIRST><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
      break;
    case PASS_MIDDLE:
      lattice_pass2v<T, BX, BY, PASS_MIDDLE><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
      break;
    case PASS_LAST:
      lattice_pass2v<T, BX, BY, PASS_LAST><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
      break;
    case PASS_MEASURE:
      lattice_pass2v<T, BX, BY, PASS_MEASURE><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
      break;
    case PASS_FORCE:
      lattice_pass2v<T, BX, BY, PASS_FORCE><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Stores of the 3D middle pass by the memory a launch touches (four values a site,
// two read and two written; n_tiles ZR 256 sites), against the L2s' 32 MiB together.
// us a trajectory of 20 steps:
// - up to 32 MiB, where no other 3D group runs beside it (sole), nontemporal: the lines
//   leave the L2s before the launch's end, and the next one finds them in the Infinity
//   Cache (plain, through, nontemporal: 64^3 113, 126, 113; 112^3 199, 197, 191; 128^3
//   224, 222, 205; FP64 96^3 359, 357, 339; beside other groups 30 chains of 16^3 .. 70^3
//   in three classes 224, -, 228).  The lead ends a little above the L2s (128 x 128 x 136,
//   34 MiB, 256, 254, 236; 136 x 136 x 128 290, 291, 286; 140^3, 42 MiB, 332, 338, 351);
// - from 1M sites (two boxes a CU, which hide the longer stores) to 128 MiB through the L2
//   (st4_through), where every row starts at a whole 32 bytes (aligned): 160^3 378, 357,
//   445; 256 chains of 24 x 21 x 30 620, 589, 671; FP64 128^3 680, 641, 709.  Other rows'
//   stores go out in halves of sectors, each twice: 132 x 128 x 128 265, 276, 249; 140^3
//   332, 338, 351; 30 chains of 36^3 264, 274, 260; 50 of 33^3 407, 421, 402;
// - above plainly: most lines are written back within the launch anyway (512 chains of
//   24 x 21 x 30 1108, 1109; FP64 4000, 4040; 256^3 nontemporal 1170 -> 1570).
// Three kernels: a choice inside one costs small launches 1.5 %.
template <typename T, int BX, int BY, int ZR>
static void launch_middle3t(const ChainDev* chains, const Tile* tiles, int n_tiles, int j, int k, bool sole,
                            bool aligned, hipStream_t s) {
  const dim3 grid(n_tiles), block(64 * ZR);
  const int64_t touched = (int64_t)n_tiles * ZR * 256 * 4 * (int)sizeof(T), l2 = 32 << 20;
  if (touched <= l2 && sole)
    lattice_pass3t<T, BX, BY, ZR, PASS_MIDDLE, StoreKind::nontemporal><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
  else if (aligned && (int64_t)n_tiles * ZR > 4096 && touched <= 4 * l2)
    lattice_pass3t<T, BX, BY, ZR, PASS_MIDDLE, StoreKind::through><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
  else
    lattice_pass3t<T, BX, BY, ZR, PASS_MIDDLE><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
}

template <typename T, int BX, int BY, int ZR>
static hipError_t launch_mode3t(int mode, const ChainDev* chains, const Tile* tiles, int n_tiles, int j, int k,
                                bool sole, bool aligned, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  dim3 grid(n_tiles), block(64 * ZR);
  switch (mode) {
    case PASS_FIRST:
      lattice_pass3t<T, BX, BY, ZR, PASS_FIRST><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
      break;
    case PASS_MIDDLE:
      launch_middle3t<T, BX, BY, ZR>(chains, tiles, n_tiles, j, k, sole, aligned, s);
      break;
    case PASS_LAST:
      lattice_pass3t<T, BX, BY, ZR, PASS_LAST><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
      break;
    case PASS_MEASURE:
      lattice_pass3t<T, BX, BY, ZR, PASS_MEASURE><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
      break;
    case PASS_FORCE:
      lattice_pass3t<T, BX, BY, ZR, PASS_FORCE><<<grid, block, 0, s>>>(chains, tiles, n_tiles, j, k);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// 2D tiles: 64 x 16 (256 threads) for rows of 48 sites or more, 32 x 32 (256
// threads) where that wastes less of the last tile of a row, 16 x 16 (64
// threads) for small lattices.  3D boxes: 32 x 8 (or 16 x 16 by the same rule)
// in the plane, 4 planes deep, or 8 where that adds no padding planes (256
// threads per 4-plane slab).
// Tile classes: the narrower tile wherever it leaves fewer idle threads in the
// last tile of a row (row lengths just above a multiple of the wide tile); in
// 3D the 8-plane boxes (fewer halo planes per site) where L2 is a multiple of 8
// and rows are whole vector chunks (L0 a multiple of 4).
int tile_class(int ndim, int L0, int L2) {
  if (ndim == 2) {
    if (L0 < 48) return 1;
    const int r = L0 % 64;
    return (r >= 1 && r <= 32) ? 2 : 0;
  }
  const int r = L0 % 32;
  const int narrow = (r >= 1 && r <= 16) ? 1 : 0;
  const bool deep = (L2 % 8 == 0) && (L0 % 4 == 0);
  return narrow + (deep ? 2 : 0);
}

int tile_class_count(int ndim) { return ndim == 2 ? 3 : 4; }

TileShape tile_shape(int precision, int ndim, int cls) {
  (void)precision;
  if (ndim == 2) {
    if (cls == 1) return TileShape{16, 16, 1};
    if (cls == 2) return TileShape{32, 32, 1};
    return TileShape{64, 16, 1};
  }
  const int bz = cls >= 2 ? 8 : 4;
  return (cls & 1) ? TileShape{16, 16, bz} : TileShape{32, 8, bz};
}

hipError_t launch_lattice_pass(int precision, int ndim, int cls, int mode, const ChainDev* chains,
                               const Tile* tiles, int n_tiles, int j, int k, hipStream_t s, bool sole, bool aligned) {
  if (cls < 0) return hipErrorInvalidValue;  // resident chains run whole trajectories (launch_resident_group)
  if (precision == 4) {
    if (ndim == 2) {
      if (cls == 1) return launch_mode2v<float, 16, 16>(mode, chains, tiles, n_tiles, j, k, s);
      if (cls == 2) return launch_mode2v<float, 32, 32>(mode, chains, tiles, n_tiles, j, k, s);
      return launch_mode2v<float, 64, 16>(mode, chains, tiles, n_tiles, j, k, s);
    }
    switch (cls) {
      case 1: return launch_mode3t<float, 16, 16, 4>(mode, chains, tiles, n_tiles, j, k, sole, aligned, s);
      case 2: return launch_mode3t<float, 32, 8, 8>(mode, chains, tiles, n_tiles, j, k, sole, aligned, s);
      case 3: return launch_mode3t<float, 16, 16, 8>(mode, chains, tiles, n_tiles, j, k, sole, aligned, s);
      default: return launch_mode3t<float, 32, 8, 4>(mode, chains, tiles, n_tiles, j, k, sole, aligned, s);
    }
  }
  if (ndim == 2) {
    if (cls == 1) return launch_mode2v<double, 16, 16>(mode, chains, tiles, n_tiles, j, k, s);
    if (cls == 2) return launch_mode2v<double, 32, 32>(mode, chains, tiles, n_tiles, j, k, s);
    return launch_mode2v<double, 64, 16>(mode, chains, tiles, n_tiles, j, k, s);
  }
  switch (cls) {
    case 1: return launch_mode3t<double, 16, 16, 4>(mode, chains, tiles, n_tiles, j, k, sole, aligned, s);
    case 2: return launch_mode3t<double, 32, 8, 8>(mode, chains, tiles, n_tiles, j, k, sole, aligned, s);
    case 3: return launch_mode3t<double, 16, 16, 8>(mode, chains, tiles, n_tiles, j, k, sole, aligned, s);
    default: return launch_mode3t<double, 32, 8, 4>(mode, chains, tiles, n_tiles, j, k, sole, aligned, s);
  }
}

}  // namespace ihmc
