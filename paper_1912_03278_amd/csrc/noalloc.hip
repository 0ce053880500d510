// Allocation-free force evaluation (ihmc_force_noalloc): F = -dS/dpsi (Sec. 3
// equations of motion) on caller-owned device arrays, for callers that cannot
// allocate device memory (code under stream capture, tight serving loops).  One
// launch reads the field and writes the force in the caller's site order.  Where
// the two arrays overlap, blocks would overwrite sites that others still read, so
// the field is staged: the chain descriptor, tile table and padded field then live
// in one file-scope device array; each GPU holds its own copy, whose address is
// looked up once per device when a context is created on it.
#include <hip/hip_runtime.h>

#include <cstring>
#include <mutex>

#include "device_common.hpp"
#include "lattice_common.hpp"
#include "lattice_kernels.hpp"
#include "runtime_internal.hpp"

namespace ihmc {

// Scratch of the allocation-free entry point: 32 MiB per GPU, enough for a
// chain of about 3.9M FP32 or 1.9M FP64 sites (two field arrays plus tiles).
constexpr uint64_t kNoallocBytes = 32ull << 20;
static __device__ __align__(256) unsigned char scratch[kNoallocBytes];

constexpr int kMaxDevices = 64;
static void* g_scratch[kMaxDevices];
static std::mutex g_scratch_mu;

// Device address of this GPU's scratch array; the current device must be
// `device`.  Looked up once per device.
int noalloc_scratch_init(int device, void** out) {
  *out = nullptr;
  if (device < 0 || device >= kMaxDevices) return set_error(IHMC_E_UNSUPPORTED, "device index %d too large", device);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return set_error(IHMC_E_DEVICE, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    g_scratch[device] = p;
  }
  *out = g_scratch[device];
  return IHMC_OK;
}

namespace {
constexpr uint64_t kOffState = 512, kOffTiles = 1024;
static_assert(sizeof(ChainDev) <= kOffState && sizeof(ChainState) <= kOffTiles - kOffState, "scratch header");
inline uint64_t r256(uint64_t b) { return (b + 255ull) & ~255ull; }

struct NoallocLayout {
  uint64_t tiles, psi, p, end;
};
NoallocLayout layout(const ChainDev& c) {
  NoallocLayout l;
  l.tiles = kOffTiles;
  l.psi = l.tiles + r256(sizeof(Tile) * (uint64_t)c.n_tiles);
  l.p = l.psi + r256((uint64_t)c.NP * (uint64_t)c.precision);
  l.end = l.p + r256((uint64_t)c.NP * (uint64_t)c.precision);
  return l;
}

// Descriptor, a fresh state (accepted field in buffer 0, sign +1) and the tile
// table, written into the scratch at `base` (the kernels only ever see it
// through this pointer).  Tiles in the order of the chain sets: x fastest.
__global__ void k_noalloc_setup(ChainDev c, unsigned char* base, uint64_t off_psi, uint64_t off_p, int bx, int by,
                                int bz) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t == 0) {
    c.psi = base + off_psi;
    c.p = base + off_p;
    c.st = (ChainState*)(base + kOffState);
    *(ChainDev*)base = c;
    uint64_t* w = (uint64_t*)(base + kOffState);
    for (int i = 0; i < (int)(sizeof(ChainState) / 8); ++i) w[i] = 0ull;
    c.st->sign = 1;
  }
  if (t < (int64_t)c.n_tiles) {
    const int nx = (c.L0 + bx - 1) / bx, ny = (c.L1 + by - 1) / by;
    Tile tl;
    tl.chain = 0;
    tl.x0 = (int)(t % nx) * bx;
    tl.y0 = (int)((t / nx) % ny) * by;
    tl.z0 = (int)(t / ((int64_t)nx * ny)) * bz;
    ((Tile*)(base + kOffTiles))[t] = tl;
  }
}

// Caller's field (site order) into the padded stored layout; padding zeroed.
template <typename T>
__global__ void k_noalloc_import(const unsigned char* base, const T* __restrict__ src) {
  const ChainDev& c = *(const ChainDev*)base;
  const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (k >= c.NP) return;
  const int64_t x = k % c.pitch, r = k / c.pitch;
  ((T*)c.psi)[k] = x < c.L0 ? src[x + (int64_t)c.L0 * r] : (T)0;
}

// The force (written to momentum buffer 0 by the force pass) back to site order.
template <typename T>
__global__ void k_noalloc_export(const unsigned char* base, T* __restrict__ dst) {
  const ChainDev& c = *(const ChainDev*)base;
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < c.N) dst[i] = ((const T*)c.p)[stored_index(c, i)];
}

// The force straight from and to arrays in site order.  A block takes a tile of
// BX x BY (x BZ) sites: psi with a halo of 2 and w = sqrt(J') tanh(sqrt(J') Kt psi) -
// psi with a halo of 1 go through LDS, positions outside the lattice hold the
// periodic images.  Per site the operations are those of the lattice passes' FORCE
// mode, so the values are the same to the bit.
//
// Small lattices are bound by the call and its launch, so there is one launch, and
// tiles of one site a thread spread the sites over the CUs; large ones, by the
// passes over memory and LDS, take four sites a thread, which halves the halo (2D
// 1.33 loads and 1.16 w a site, 3D 3.1 and 1.9).  Back-to-back calls, against
// descriptor, import, pass and export in four launches: 48 x 40 FP32 13.5 -> 5.0
// us, 1024^2 17.1 -> 5.2, 1900^2 31.1 -> 11.3, 100^3 19.3 -> 12.6, 150^3 34.8 ->
// 28.1, 110^3 FP64 44.9 -> 29.8.  The large ones' stores go through the L2 (plainly 1900^2 12.4,
// 150^3 30.0, 110^3 FP64 30.7).
template <typename T>
struct ForceArgs {
  T C, a, hw, b;
  int L0, L1, L2, nx, ny;
};

__device__ __forceinline__ int wrapped(int g, int L) {
  g = g < 0 ? g + L : g;  // at least -2, and L >= 3
  return g < L ? g : (g - L < L ? g - L : g % L);
}

template <typename T, int NDIM, int BX, int BY, int BZ>
__global__ __launch_bounds__(256) void k_force(ForceArgs<T> q, const T* __restrict__ psi, T* __restrict__ F) {
  constexpr int HZ = NDIM == 3 ? 1 : 0;  // halos along z: 2 HZ and HZ
  constexpr int PX = BX + 4, PY = BY + 4, PZ = BZ + 4 * HZ, WX = BX + 2, WY = BY + 2, WZ = BZ + 2 * HZ;
  __shared__ T sP[PX * PY * PZ];
  __shared__ T sW[WX * WY * WZ];
  const int t = blockIdx.x, tx = t % q.nx, r = t / q.nx, ty = NDIM == 3 ? r % q.ny : r, tz = NDIM == 3 ? r / q.ny : 0;
  const int x0 = tx * BX, y0 = ty * BY, z0 = tz * BZ;
  for (int i = threadIdx.x; i < PX * PY * PZ; i += 256) {
    const int x = i % PX, yz = i / PX, y = yz % PY, z = yz / PY;
    const int gx = wrapped(x0 + x - 2, q.L0), gy = wrapped(y0 + y - 2, q.L1);
    const int gz = NDIM == 3 ? wrapped(z0 + z - 2, q.L2) : 0;
    sP[i] = psi[gx + (int64_t)q.L0 * (gy + (int64_t)q.L1 * gz)];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < WX * WY * WZ; i += 256) {
    const int x = i % WX, yz = i / WX, y = yz % WY, z = yz / WY;
    const T* c = sP + (x + 1) + PX * ((y + 1) + PY * (z + HZ));
    T n = (c[-1] + c[1]) + (c[-PX] + c[PX]);
    if (NDIM == 3) n = n + (c[-PX * PY] + c[PX * PY]);
    const T u = fma_t(q.C, c[0], n);
    sW[i] = fma_t(q.a, tanh_state(fma_t(q.a, u, q.hw)), -c[0]);
  }
  __syncthreads();
#pragma unroll
  for (int i = threadIdx.x; i < BX * BY * BZ; i += 256) {
    const int x = i % BX, yz = i / BX, y = yz % BY, z = yz / BY;
    const T* w = sW + (x + 1) + WX * ((y + 1) + WY * (z + HZ));
    T n = (w[-1] + w[1]) + (w[-WX] + w[WX]);
    if (NDIM == 3) n = n + (w[-WX * WY] + w[WX * WY]);
    const T f = fma_t(q.C, w[0], n) + q.b;
    const int gx = x0 + x, gy = y0 + y, gz = z0 + z;
    if (gx < q.L0 && gy < q.L1 && gz < q.L2) {
      gmem<T>* o = (gmem<T>*)F + (gx + (int64_t)q.L0 * (gy + (int64_t)q.L1 * gz));
      if constexpr (BX * BY * BZ > 256) st_through<T>(o, fma_t((T)1, f, (T)0));
      else *o = fma_t((T)1, f, (T)0);
    }
  }
}

template <typename T, int NDIM, int BX, int BY, int BZ>
hipError_t launch_force_tiles(const ChainDev& c, const void* psi, void* F, hipStream_t s) {
  const int nx = (c.L0 + BX - 1) / BX, ny = (c.L1 + BY - 1) / BY, nz = (c.L2 + BZ - 1) / BZ;
  const ForceArgs<T> q{(T)c.C, (T)c.sqJ, (T)c.hw, (T)c.b0, c.L0, c.L1, c.L2, nx, ny};
  k_force<T, NDIM, BX, BY, BZ><<<(unsigned)((int64_t)nx * ny * nz), 256, 0, s>>>(q, (const T*)psi, (T*)F);
  return hipGetLastError();
}

// Work of a launch on BX x BY x BZ tiles, padding included: staged values and two per
// w, over all tiles; a quarter more where rows of four are loaded.
double force_work(const ChainDev& c, int bx, int by, int bz) {
  const int hz = c.ndim == 3 ? 1 : 0;
  const double tiles = (double)((c.L0 + bx - 1) / bx) * ((c.L1 + by - 1) / by) * ((c.L2 + bz - 1) / bz);
  const double w = tiles * ((bx + 4) * (by + 4) * (bz + 4 * hz) + 2 * (bx + 2) * (by + 2) * (bz + 2 * hz));
  return bx == 4 ? 1.25 * w : w;
}

// The tile with the least work; those of four sites a thread where they still give each
// CU four blocks.  Thin lattices fill little of a wide tile (FP32, on 64 x 16 or 16 x 16 x
// 4 sites, on the tile taken, and in four launches: 4 x 500000 75, 9.7 and 33 us, 3 x 3 x
// 200000 296, 25 and 153, 200000 x 3 x 3 68, 27 and 34, 3 x 200000 x 3 73, 25 and 56).
template <typename T>
hipError_t launch_force(const ChainDev& c, const void* psi, void* F, hipStream_t s) {
  using Launch = hipError_t (*)(const ChainDev&, const void*, void*, hipStream_t);
  struct Tile {
    int ndim, bx, by, bz;
    Launch launch;
  };
  static const Tile kTiles[] = {
      {2, 64, 16, 1, launch_force_tiles<T, 2, 64, 16, 1>}, {2, 32, 8, 1, launch_force_tiles<T, 2, 32, 8, 1>},
      {2, 4, 64, 1, launch_force_tiles<T, 2, 4, 64, 1>},   {3, 16, 16, 4, launch_force_tiles<T, 3, 16, 16, 4>},
      {3, 16, 4, 4, launch_force_tiles<T, 3, 16, 4, 4>},   {3, 4, 16, 4, launch_force_tiles<T, 3, 4, 16, 4>},
      {3, 4, 4, 16, launch_force_tiles<T, 3, 4, 4, 16>}};
  const Tile* best = nullptr;
  double least = 0.0;
  for (const Tile& t : kTiles) {
    if (t.ndim != c.ndim || (t.bx * t.by * t.bz > 256 && c.N < 1024 * 1024)) continue;
    const double w = force_work(c, t.bx, t.by, t.bz);
    if (!best || w < least) {
      best = &t;
      least = w;
    }
  }
  return best->launch(c, psi, F, s);
}
}  // namespace

}  // namespace ihmc

using namespace ihmc;

extern "C" int ihmc_force_noalloc(ihmc_ctx* ctx, const ihmc_lattice* lat, int32_t precision, const void* psi,
                                  void* F, void* stream) {
  CTX_OK(ctx);
  if (!lat || !psi || !F) return set_error(IHMC_E_INVAL, "NULL argument");
  if (!ctx->scratch) return set_error(IHMC_E_DEVICE, "no scratch array on this device");
  ihmc_run r;
  std::memset(&r, 0, sizeof r);
  r.n_md = 1;
  r.n_traj = 1;
  r.traj_len = 1.0;
  r.precision = precision;
  int rc = validate(*lat, r, 0);
  if (rc) return rc;
  if (lat->h_len > 1)
    return set_error(IHMC_E_UNSUPPORTED, "the allocation-free force takes h = 0 or a uniform field only");
  ChainDev c;
  describe_chain(*lat, r, BUILD_TILED, ctx->tune.class_for(tile_key(*lat, precision)), c);
  const NoallocLayout l = layout(c);
  if (l.end > kNoallocBytes)
    return set_error(IHMC_E_INVAL, "lattice of %lld sites needs %llu bytes of scratch, the maximum is %llu",
                     (long long)c.N, (unsigned long long)l.end, (unsigned long long)kNoallocBytes);
  hipStream_t s = stream ? (hipStream_t)stream : ctx->stream;
  const uint64_t bytes = (uint64_t)c.N * (uint64_t)precision;
  const uintptr_t ip = (uintptr_t)psi, iF = (uintptr_t)F;
  if (ip + bytes <= iF || iF + bytes <= ip) {
    const hipError_t e = precision == 4 ? launch_force<float>(c, psi, F, s) : launch_force<double>(c, psi, F, s);
    return e == hipSuccess ? IHMC_OK : hip_fail(ctx, e, "allocation-free force");
  }
  unsigned char* base = (unsigned char*)ctx->scratch;
  const TileShape ts = tile_shape(c.precision, c.ndim, c.tile_cls);
  const unsigned tb = (unsigned)((c.n_tiles + 255) / 256);
  k_noalloc_setup<<<tb, 256, 0, s>>>(c, base, l.psi, l.p, ts.bx, ts.by, ts.bz);
  hipError_t e = hipGetLastError();
  const unsigned nb = (unsigned)((c.NP + 255) / 256), ns = (unsigned)((c.N + 255) / 256);
  if (e == hipSuccess) {
    if (precision == 4) k_noalloc_import<float><<<nb, 256, 0, s>>>(base, (const float*)psi);
    else k_noalloc_import<double><<<nb, 256, 0, s>>>(base, (const double*)psi);
    e = hipGetLastError();
  }
  if (e == hipSuccess)
    e = launch_lattice_pass(c.precision, c.ndim, c.tile_cls, PASS_FORCE, (const ChainDev*)base,
                            (const Tile*)(base + kOffTiles), (int)c.n_tiles, 0, 0, s);
  if (e == hipSuccess) {
    if (precision == 4) k_noalloc_export<float><<<ns, 256, 0, s>>>(base, (float*)F);
    else k_noalloc_export<double><<<ns, 256, 0, s>>>(base, (double*)F);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return hip_fail(ctx, e, "allocation-free force");
  return IHMC_OK;
}
