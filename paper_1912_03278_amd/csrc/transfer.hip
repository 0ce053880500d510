// Set-up and results of many chains in a few launches.
//
// A chain set's set-up resets every chain's state, brings per-site fields to the
// device and draws the starting fields; its results bring every chain's state,
// records and final field to the caller.  Each of these is one launch over all
// chains (grid.y), and host data passes through the context's pinned buffer,
// which the kernels read and write directly: no launch, copy or wait per chain.
// The buffer has two halves, so the host packs or unpacks one while the
// device works on the other.  What does not fit a half (a field of over 122 Ki
// sites) goes by a copy of its own.
//
// Bound by launches and waits when done per chain: results of 128 chains of
// 15 x 15 took 9.2 ms that way, those of 512 uneven chains (48 MB of fields) 40 ms;
// the whole calls went from 11.9 to 4.4 ms (200 trajectories) and from 105 to 67.
#include <algorithm>
#include <cstring>
#include <new>

#include "device_common.hpp"
#include "runtime_internal.hpp"

namespace ihmc {

namespace {

constexpr uint64_t STAGE_HALF = 1ull << 20;

inline uint64_t r64(uint64_t b) { return (b + 63ull) & ~63ull; }

// Workgroups per chain that cover `elems` elements of the largest of n chains
// with a few per thread, without flooding the launch when n is large.
inline unsigned grid_x(int64_t elems, int64_t n) {
  const int64_t want = (elems + 1023) / 1024, lim = std::max<int64_t>(1, 65536 / std::max<int64_t>(n, 1));
  return (unsigned)std::max<int64_t>(1, std::min(want, lim));
}

// One chain's place in a half of the pinned buffer (offsets from its start).
struct StageItem {
  uint64_t state, rec, data;  // data: FP64 field values in site order (~0: none)
  int32_t chain, n_rec;
  double scale;  // uploads: h' = scale h
};

// Fresh state (sign +1, everything else zero), cleared tile counters, and with
// clear_fields the field and momentum buffers of a dense chain.
__global__ __launch_bounds__(256) void k_reset(const ChainDev* __restrict__ cds, int clear_fields) {
  const ChainDev& cd = cds[blockIdx.y];
  if (blockIdx.x == 0) {
    uint64_t* w = (uint64_t*)cd.st;
    for (int i = threadIdx.x; i < (int)(sizeof(ChainState) / 8); i += 256) w[i] = 0ull;
    for (int64_t i = threadIdx.x; i < (int64_t)part_groups(cd.n_tiles); i += 256) cd.gcnt[i] = 0u;
    __syncthreads();
    if (threadIdx.x == 0) cd.st->sign = 1;
  }
  if (clear_fields) {
    float* psi = (float*)cd.psi;
    float* p = (float*)cd.p;
    for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < 3 * cd.NP; i += (int64_t)gridDim.x * 256) {
      psi[i] = 0.f;
      if (i < cd.NP) p[i] = 0.f;
    }
  }
}

// Per-site fields from the pinned buffer: h' = beta h (FP64) and h'/sqrt(J')
// (state precision) at the stored indices.
__global__ __launch_bounds__(256) void k_fields_in(const ChainDev* __restrict__ cds, const StageItem* items,
                                                   const char* half) {
  const StageItem it = items[blockIdx.y];
  const ChainDev& cd = cds[it.chain];
  const double* h = (const double*)(half + it.data);
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < cd.N; i += (int64_t)gridDim.x * 256) {
    const int64_t k = stored_index(cd, i);
    const double hp = it.scale * h[i];
    ((double*)cd.hp)[k] = hp;
    if (cd.precision == 4) ((float*)cd.b)[k] = (float)(hp / cd.sqJ);
    else ((double*)cd.b)[k] = hp / cd.sqJ;
  }
}

// Starting fields: a given one (device, site order) or the TAG_INIT normals, a
// pair of sites per draw, plus the chain's translation, rounded to the state type.
__global__ __launch_bounds__(256) void k_start(const ChainDev* __restrict__ cds, const StartField* __restrict__ from) {
  const StartField f = from[blockIdx.y];
  const ChainDev& cd = cds[f.chain];
  for (int64_t pr = blockIdx.x * 256 + threadIdx.x; 2 * pr < cd.N; pr += (int64_t)gridDim.x * 256) {
    double v[2];
    if (!f.psi0) box_muller(draw(cd, (uint32_t)pr, 0u, TAG_INIT), v[0], v[1]);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int64_t i = 2 * pr + e;
      if (i >= cd.N) continue;
      double x = f.psi0 ? f.psi0[i] : v[e];
      if (f.shift) x += f.shift[i];
      if (cd.precision == 4) ((float*)cd.psi)[stored_index(cd, i)] = (float)x;
      else ((double*)cd.psi)[stored_index(cd, i)] = x;
    }
  }
}

// State, records and accepted field (sign applied, FP64, site order) of the
// items' chains into the pinned buffer.
__global__ __launch_bounds__(256) void k_results_out(const ChainDev* __restrict__ cds, const StageItem* items,
                                                     char* half) {
  const StageItem it = items[blockIdx.y];
  const ChainDev& cd = cds[it.chain];
  const ChainState* st = cd.st;
  const int64_t t0 = blockIdx.x * 256 + threadIdx.x, stride = (int64_t)gridDim.x * 256;
  if (t0 < (int64_t)(sizeof(ChainState) / 8)) ((uint64_t*)(half + it.state))[t0] = ((const uint64_t*)st)[t0];
  const int64_t words = (int64_t)min(st->traj, it.n_rec) * (int64_t)(sizeof(TrajRecord) / 8);
  for (int64_t i = t0; i < words; i += stride) ((uint64_t*)(half + it.rec))[i] = ((const uint64_t*)cd.rec)[i];
  if (it.data != ~0ull) {
    double* out = (double*)(half + it.data);
    const int64_t base = (int64_t)st->cur * cd.NP;
    const bool neg = st->sign < 0;
    for (int64_t i = t0; i < cd.N; i += stride) {
      const int64_t k = base + stored_index(cd, i);
      const double v = cd.precision == 4 ? (double)((const float*)cd.psi)[k] : ((const double*)cd.psi)[k];
      out[i] = neg ? -v : v;
    }
  }
}

void fill_result(const ChainDev& c, const ChainState& st, const TrajRecord* rec, int done, ihmc_result* out) {
  for (int t = 0; t < done; ++t) {
    const TrajRecord& r = rec[t];
    if (out->dH) out->dH[t] = r.dH;
    if (out->H_old) out->H_old[t] = r.H_old;
    if (out->H_new) out->H_new[t] = r.H_new;
    if (out->m) out->m[t] = r.m;
    if (out->abs_m) out->abs_m[t] = r.abs_m;
    if (out->m2c) out->m2c[t] = r.m2c;
    if (out->beta_eps) out->beta_eps[t] = r.beta_eps;
    if (out->accepted) out->accepted[t] = (r.flags & REC_ACCEPT) ? 1 : 0;
    if (out->flipped) out->flipped[t] = (r.flags & REC_FLIP) ? 1 : 0;
  }
  out->n_traj_done = st.traj;
  const int64_t counted = std::max(0, st.traj - c.n_therm);  // trajectories past thermalisation
  out->acceptance = counted ? (double)st.n_acc / (double)counted : 0.0;
  const int64_t nf = counted - st.n_nonfinite;
  out->mean_exp_minus_dH = nf > 0 ? st.sum_exp_mdh / (double)nf : 0.0;
  out->n_nonfinite = st.n_nonfinite;
  out->cg_iterations = st.n_cg;
}

// One chain by copies of its own (it does not fit a half of the buffer).
int result_direct(ihmc_ctx* ctx, const ChainDev& c, const ChainDev* d_cd, int ci, ihmc_result* out) {
  hipStream_t s = ctx->stream;
  HIPCHK(hipStreamSynchronize(s), "sync");
  ChainState st;
  HIPCHK(hipMemcpy(&st, c.st, sizeof st, hipMemcpyDeviceToHost), "state download");
  const int done = std::min(st.traj, c.cap);
  std::vector<TrajRecord> rec((size_t)std::max(done, 1));
  if (done > 0) HIPCHK(hipMemcpy(rec.data(), c.rec, sizeof(TrajRecord) * done, hipMemcpyDeviceToHost), "records");
  fill_result(c, st, rec.data(), done, out);
  if (out->psi_final) {
    double* t = (double*)ctx->arena.alloc(8 * (uint64_t)c.N);
    if (!t) return set_error(IHMC_E_NOMEM, "arena exhausted (export)");
    hipError_t e0 = launch_export_psi(d_cd, ci, t, c.N, c.precision, s);
    hipError_t e = e0 == hipSuccess ? hipMemcpyAsync(out->psi_final, t, 8 * c.N, hipMemcpyDeviceToHost, s) : e0;
    hipError_t e2 = hipStreamSynchronize(s);
    ctx->arena.release(t);
    if (e != hipSuccess) return hip_fail(ctx, e, "psi export");
    if (e2 != hipSuccess) return hip_fail(ctx, e2, "psi export sync");
  }
  return IHMC_OK;
}

// A half of the pinned buffer being filled: items from its start, data behind
// the item table.
struct Half {
  std::vector<StageItem> items;
  uint64_t used = 0;
  int64_t largest = 0;
  bool busy = false;  // its launch has been recorded and not waited for
  void clear() {
    items.clear();
    used = 0;
    largest = 0;
  }
  uint64_t take(uint64_t bytes) {
    const uint64_t at = used;
    used += r64(bytes);
    return at;
  }
};
constexpr size_t MAX_ITEMS = 1024;
constexpr uint64_t ITEM_BYTES = MAX_ITEMS * sizeof(StageItem);
constexpr uint64_t DATA_BYTES = STAGE_HALF - ((ITEM_BYTES + 63) / 64) * 64;

}  // namespace

void stage_destroy(Stage& st) {
  for (hipEvent_t& e : st.ev) {
    if (e) hipEventDestroy(e);
    e = nullptr;
  }
  if (st.host) hipHostFree(st.host);
  st.host = nullptr;
}

// Allocated at the first transfer that uses it; once refused, not asked again.
static void stage_ready(Stage& st) {
  if (st.host || st.tried) return;
  st.tried = true;
  if (hipHostMalloc((void**)&st.host, 2 * STAGE_HALF, 0) != hipSuccess) st.host = nullptr;
  for (hipEvent_t& e : st.ev)
    if (st.host && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
      e = nullptr;
      stage_destroy(st);
    }
  (void)hipGetLastError();
}

hipError_t launch_reset(const ChainDev* d_cd, int n, int64_t clear_values, hipStream_t s) {
  for (int c0 = 0; c0 < n; c0 += 65535) {
    const int m = std::min(n - c0, 65535);
    k_reset<<<dim3(grid_x(clear_values, m), (unsigned)m), 256, 0, s>>>(d_cd + c0, clear_values > 0 ? 1 : 0);
  }
  return hipGetLastError();
}

hipError_t launch_start(const ChainDev* d_cd, const StartField* from, int n, int64_t max_sites, hipStream_t s) {
  for (int c0 = 0; c0 < n; c0 += 65535) {
    const int m = std::min(n - c0, 65535);
    k_start<<<dim3(grid_x(max_sites / 2, m), (unsigned)m), 256, 0, s>>>(d_cd, from + c0);
  }
  return hipGetLastError();
}

int upload_fields(ihmc_ctx* ctx, const std::vector<ChainDev>& cd, const ChainDev* d_cd, const std::vector<int>& idx,
                  const ihmc_lattice* lats, std::vector<void*>& temps) {
  hipStream_t s = ctx->stream;
  Stage& sg = ctx->stage;
  stage_ready(sg);
  Half half[2];
  int cur = 0;
  auto flush = [&](int b) -> hipError_t {
    Half& h = half[b];
    if (h.items.empty()) return hipSuccess;
    char* base = sg.host + b * STAGE_HALF;
    std::memcpy(base, h.items.data(), h.items.size() * sizeof(StageItem));
    k_fields_in<<<dim3(grid_x(h.largest, (int64_t)h.items.size()), (unsigned)h.items.size()), 256, 0, s>>>(
        d_cd, (const StageItem*)base, base + STAGE_HALF - DATA_BYTES);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipEventRecord(sg.ev[b], s);
    h.busy = true;
    h.clear();
    return e;
  };
  for (int i : idx) {
    const int64_t N = cd[i].N;
    const uint64_t bytes = 8 * (uint64_t)N;
    if (!sg.host || r64(bytes) > DATA_BYTES) {
      double* t = (double*)ctx->arena.alloc(bytes);
      if (!t) return set_error(IHMC_E_NOMEM, "arena exhausted (field staging)");
      temps.push_back(t);
      HIPCHK(hipMemcpyAsync(t, lats[i].h, bytes, hipMemcpyHostToDevice, s), "h upload");
      HIPCHK(launch_field_setup(d_cd, i, t, lats[i].beta, N, cd[i].precision, s), "field set-up");
      continue;
    }
    if (half[cur].used + r64(bytes) > DATA_BYTES || half[cur].items.size() == MAX_ITEMS) {
      HIPCHK(flush(cur), "field upload");
      cur ^= 1;
    }
    Half& h = half[cur];
    if (h.busy) {  // the launch that reads this half's earlier contents
      HIPCHK(hipEventSynchronize(sg.ev[cur]), "field upload");
      h.busy = false;
    }
    StageItem it{};
    it.chain = i;
    it.data = h.take(bytes);
    it.scale = lats[i].beta;
    std::memcpy(sg.host + cur * STAGE_HALF + (STAGE_HALF - DATA_BYTES) + it.data, lats[i].h, bytes);
    h.items.push_back(it);
    h.largest = std::max(h.largest, N);
  }
  HIPCHK(flush(cur), "field upload");
  return IHMC_OK;
}

int collect_results(ihmc_ctx* ctx, const std::vector<ChainDev>& cd, const ChainDev* d_cd, int first, int n,
                    const int* done, ihmc_result* outs) {
  hipStream_t s = ctx->stream;
  Stage& sg = ctx->stage;
  stage_ready(sg);
  Half half[2];
  std::vector<StageItem> waiting[2];  // items of a half whose launch runs
  int cur = 0;
  auto flush = [&](int b) -> hipError_t {
    Half& h = half[b];
    if (h.items.empty()) return hipSuccess;
    char* base = sg.host + b * STAGE_HALF;
    std::memcpy(base, h.items.data(), h.items.size() * sizeof(StageItem));
    k_results_out<<<dim3(grid_x(h.largest, (int64_t)h.items.size()), (unsigned)h.items.size()), 256, 0, s>>>(
        d_cd, (const StageItem*)base, base + STAGE_HALF - DATA_BYTES);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipEventRecord(sg.ev[b], s);
    waiting[b].swap(h.items);
    h.clear();
    return e;
  };
  auto drain = [&](int b) -> int {
    if (waiting[b].empty()) return IHMC_OK;
    HIPCHK(hipEventSynchronize(sg.ev[b]), "results");
    const char* base = sg.host + b * STAGE_HALF + (STAGE_HALF - DATA_BYTES);
    for (const StageItem& it : waiting[b]) {
      const ChainDev& c = cd[it.chain];
      ihmc_result* out = &outs[it.chain - first];
      ChainState st;
      std::memcpy(&st, base + it.state, sizeof st);
      if (std::min(st.traj, c.cap) > it.n_rec) {  // more records than the host counted
        const int rc = result_direct(ctx, c, d_cd, it.chain, out);
        if (rc) return rc;
        continue;
      }
      fill_result(c, st, (const TrajRecord*)(base + it.rec), std::min(st.traj, c.cap), out);
      if (it.data != ~0ull) std::memcpy(out->psi_final, base + it.data, 8 * (size_t)c.N);
    }
    waiting[b].clear();
    return IHMC_OK;
  };
  for (int i = first; i < first + n; ++i) {
    const ChainDev& c = cd[i];
    ihmc_result* out = &outs[i - first];
    const int n_rec = std::max(0, std::min(done[i - first], c.cap));
    const uint64_t fb = out->psi_final ? 8 * (uint64_t)c.N : 0;
    const uint64_t need = r64(sizeof(ChainState)) + r64(sizeof(TrajRecord) * (uint64_t)n_rec) + r64(fb);
    if (!sg.host || need > DATA_BYTES) {
      const int rc = result_direct(ctx, c, d_cd, i, out);
      if (rc) return rc;
      continue;
    }
    if (half[cur].used + need > DATA_BYTES || half[cur].items.size() == MAX_ITEMS) {
      HIPCHK(flush(cur), "results");
      cur ^= 1;
      const int rc = drain(cur);  // before this half is written again
      if (rc) return rc;
    }
    Half& h = half[cur];
    StageItem it{};
    it.chain = i;
    it.n_rec = n_rec;
    it.state = h.take(sizeof(ChainState));
    it.rec = h.take(sizeof(TrajRecord) * (uint64_t)n_rec);
    it.data = fb ? h.take(fb) : ~0ull;
    h.items.push_back(it);
    h.largest = std::max({h.largest, (int64_t)(fb / 8), (int64_t)n_rec * 8});
  }
  HIPCHK(flush(cur), "results");
  for (int b : {cur ^ 1, cur}) {
    const int rc = drain(b);
    if (rc) return rc;
  }
  return IHMC_OK;
}

}  // namespace ihmc
