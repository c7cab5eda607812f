// mhd_api.hip -- C ABI of libmhd: contexts on borrowed workspaces, cycle
// control on the device, state copies and diagnostics.  See include/mhd.h.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "../../include/mhd.h"
#include "mhd_internal.h"

using namespace mhd;

struct mhd_ctx {
  mhd_params p;
  hipStream_t stream;
  int device;
  size_t elem;       // bytes per value: 8 (FP64) or 4 (FP32)
  long long ncell;
  double idl[3];     // 1 / (l_d / n_d)
  double dv;         // cell volume
  void* buf[kMaxBuf][kFields];  // state buffers (3 for RK3, else 2)
  int nbuf;
  int nfield;  // fields per buffer: 8, or 11 with the vector-potential form
  int cur;           // buffer holding the state
  void* uct;         // edge-solve scratch (UCT-HLL, UCT-HLLD), or null
  Scalars* sc;       // device scalars
  BoxDesc* desc;     // device copy of this box's descriptor
  double* diag_part; // per-block diagnostic partials
  int tile, zchunk;  // launch shape as requested (zchunk 0 = automatic)
  bool shaped;       // tile or zchunk was requested: that shape, whatever the size
  int lone_tile, lz; // tile and z-planes per work-group: as requested, or when stepped alone
  int auto_tile;     // tile when stepped alone with nothing requested
  int diag_blocks;
  int stages_valid;  // intermediate buffers hold the last cycle's stage results
};

namespace {

// roctx range over a scope: host-side markers that rocprofv3 --marker-trace
// records around the library's calls and cycles (no device work)
struct Range {
  explicit Range(const char* m) { roctxRangePushA(m); }
  ~Range() { roctxRangePop(); }
  Range(const Range&) = delete;
  Range& operator=(const Range&) = delete;
};

constexpr size_t kAlign = 256;
constexpr int kDiagBlocks = 512;
constexpr int kDiagVals = 20;  // 9 sums as (sum, compensation) pairs + max + pad

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

bool grid_ok(const mhd_params* p) {
  return p && p->nx >= 1 && p->ny >= 1 && p->nz >= 1 && p->nx <= 4096 && p->ny <= 4096 &&
         p->nz <= 4096;
}

int default_tile(int precision) { return precision == MHD_FP32 ? TILE_24x8 : TILE_24x8; }

size_t field_bytes(const mhd_params* p) {
  size_t e = p->precision == MHD_FP32 ? 4 : 8;
  return align_up((size_t)p->nx * p->ny * p->nz * e);
}

// state buffers a context needs: U_0 and one per intermediate stage result
int nbuf_of(const mhd_params* p) { return p->integrator == MHD_RK3 ? 3 : 2; }
int nfield_of(const mhd_params* p) { return p->ct == MHD_CT_VECPOT ? 11 : 8; }
// scratch arrays of one field each: the UCT-HLL face data and edge EMFs
int nscratch_of(const mhd_params* p) {
  return p->emf == MHD_EMF_UCT_HLL ? kUctArrays : p->emf == MHD_EMF_UCT_HLLD ? kUctHlldArrays : 0;
}

// ---- cycle control kernels (one thread): everything stays on the device

__device__ void set_scalars(Scalars* s, double t, double dt_next, double cfl) {
  st_agent(&s->t, t);
  st_agent(&s->dt_next, dt_next);
  st_agent(&s->dt[0], 0.0);
  st_agent(&s->dt[1], 0.0);
  st_agent(&s->cfl, cfl);
  st_agent(&s->invdt_bits, 0ull);
  st_agent(&s->status, 0u);
}

__global__ void k_set(Scalars* s, double t, double dt_next, double cfl) {
  set_scalars(s, t, dt_next, cfl);
}

// ---- readback: the scalars that a synchronising call returns.
//
// A copy of 152 bytes to pageable memory stages through the runtime and waits on its own
// (a scalars-only mhd_get_state took 21 us).  The last kernel of the call writes them to
// a slot of pinned host memory instead, and the call's one synchronisation makes them
// visible: 11 us.  The slots are one allocation of the process, made with the first
// context; a call holds one while it waits, and falls back to the copy if all are taken.
struct Readback {
  static constexpr int kSlots = 64;
  std::mutex mu;
  Scalars* base = nullptr;
  bool tried = false;
  unsigned long long taken = 0;

  void init() {
    std::lock_guard<std::mutex> lock(mu);
    if (tried) return;
    tried = true;
    void* p = nullptr;
    if (hipHostMalloc(&p, sizeof(Scalars) * kSlots, hipHostMallocPortable | hipHostMallocCoherent) ==
        hipSuccess)
      base = static_cast<Scalars*>(p);
    else
      (void)hipGetLastError();
  }
  Scalars* take() {
    std::lock_guard<std::mutex> lock(mu);
    if (!base || taken == ~0ull) return nullptr;
    const int i = __builtin_ctzll(~taken);
    taken |= 1ull << i;
    return base + i;
  }
  void give(Scalars* s) {
    if (!s) return;
    std::lock_guard<std::mutex> lock(mu);
    taken &= ~(1ull << (s - base));
  }
};
static_assert(Readback::kSlots == 64, "one bit per slot");
Readback g_readback;

// a slot for the length of a call
struct Slot {
  Scalars* s;
  Slot() : s(g_readback.take()) {}
  ~Slot() { g_readback.give(s); }
  Slot(const Slot&) = delete;
  Slot& operator=(const Slot&) = delete;
};

constexpr int kScalarWords = (int)(sizeof(Scalars) / 8);
static_assert(sizeof(Scalars) % 8 == 0 && kScalarWords <= 64, "one lane per word");

// Threads below kScalarWords copy the scalars to host memory.
__device__ __forceinline__ void send_scalars(const Scalars* s, Scalars* host, int t) {
  if (t >= kScalarWords) return;
  const unsigned long long v = ld_agent(reinterpret_cast<const unsigned long long*>(s) + t);
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(host) + t, v, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_SYSTEM);
}
__global__ void k_send(const Scalars* s, Scalars* host) { send_scalars(s, host, threadIdx.x); }

// Wait for the stream and read the scalars back: from the slot that a kernel of the
// call has written, or by a copy.
hipError_t read_scalars(const mhd_ctx* c, const Slot& slot, Scalars* h) {
  if (!slot.s) {
    hipError_t e = hipMemcpyAsync(h, c->sc, sizeof(Scalars), hipMemcpyDeviceToHost, c->stream);
    return e == hipSuccess ? hipStreamSynchronize(c->stream) : e;
  }
  hipError_t e = hipStreamSynchronize(c->stream);
  if (e == hipSuccess) memcpy(h, slot.s, sizeof(Scalars));
  return e;
}

// ---- state copies: all fields of a state in one launch, with the scalars of a new
// state.  For small boxes a copy is all launch: eight copies cost 8 to 10 us each on
// the host and left the GPU idle between them, one pass of set_state, a cycle and
// get_state on a 16^3 box 193 us; one launch each way takes it to 145 us (83 with the
// scalars through pinned memory and the stages as bricks).  Large ones run at the card's
// copy rate either way.
constexpr int kCopyThreads = 256;
struct CopyArgs {
  const void* src[kFields];
  void* dst[kFields];
  long long bytes;  // of one field, a multiple of 4
  Scalars* sc;      // null: leave the scalars alone
  double t, dt_next, cfl;
  const Scalars* from;  // with to: also read the scalars back
  Scalars* to;
};

typedef unsigned Words4 __attribute__((ext_vector_type(4)));
typedef unsigned Words2 __attribute__((ext_vector_type(2)));

template <typename V>
__device__ __forceinline__ void copy_field(const void* src, void* dst, long long bytes) {
  const V* s = static_cast<const V*>(src);
  V* d = static_cast<V*>(dst);
  const long long n = bytes / (long long)sizeof(V), step = (long long)gridDim.x * kCopyThreads;
  long long c = (long long)blockIdx.x * kCopyThreads + threadIdx.x;
  for (; c + 3 * step < n; c += 4 * step) {
    const V v0 = s[c], v1 = s[c + step], v2 = s[c + 2 * step], v3 = s[c + 3 * step];
    d[c] = v0;
    d[c + step] = v1;
    d[c + 2 * step] = v2;
    d[c + 3 * step] = v3;
  }
  for (; c < n; c += step) d[c] = s[c];
  // what a vector does not divide
  const long long w = n * (long long)(sizeof(V) / 4) + threadIdx.x;
  if (blockIdx.x == 0 && w < bytes / 4)
    static_cast<unsigned*>(dst)[w] = static_cast<const unsigned*>(src)[w];
}

__global__ void __launch_bounds__(kCopyThreads) k_copy(CopyArgs a) {
  if (a.sc && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
    set_scalars(a.sc, a.t, a.dt_next, a.cfl);
  if (a.to && blockIdx.x == 0 && blockIdx.y == 0) send_scalars(a.from, a.to, threadIdx.x);
  const void* src = a.src[blockIdx.y];
  void* dst = a.dst[blockIdx.y];
  const unsigned long long low = (uintptr_t)src | (uintptr_t)dst;
  if ((low & 15) == 0)  // the caller's arrays need not be aligned beyond their values
    copy_field<Words4>(src, dst, a.bytes);
  else if ((low & 7) == 0)
    copy_field<Words2>(src, dst, a.bytes);
  else
    copy_field<unsigned>(src, dst, a.bytes);
}

// Whether a kernel on device dev may touch [p, p + bytes): memory of that device, inside
// one allocation.  Anything else (another device's memory, host memory, an array that is
// too short) is left to hipMemcpyAsync and its checks.  The two look-ups take about 3 us
// on the host; the arrays of a small state mostly lie in one allocation, looked up once.
struct Extent {
  uintptr_t lo, hi;
};
bool on_device(const void* ptr, size_t bytes, int dev, Extent& known) {
  const uintptr_t p = (uintptr_t)ptr;
  if ((p & 3) != 0) return false;
  if (p >= known.lo && p + bytes <= known.hi) return true;
  hipPointerAttribute_t at;
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  if (hipPointerGetAttributes(&at, ptr) == hipSuccess && at.type == hipMemoryTypeDevice &&
      at.device == dev && hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)ptr) == hipSuccess) {
    known = {(uintptr_t)base, (uintptr_t)base + size};
    return p + bytes <= known.hi;
  }
  (void)hipGetLastError();
  return false;
}

// Whether copying fields in any order gives what one after another gives: no destination
// overlaps another field's source or destination.
bool any_order(const CopyArgs& a, int n, size_t bytes) {
  auto apart = [&](const void* p, const void* q) {
    const uintptr_t x = (uintptr_t)p, y = (uintptr_t)q;
    return x < y ? y - x >= bytes : x - y >= bytes;
  };
  for (int f = 0; f < n; ++f)
    for (int g = 0; g < n; ++g)
      if (f != g && (!apart(a.dst[f], a.src[g]) || !apart(a.dst[f], a.dst[g]))) return false;
  return true;
}

// Copy nf fields (null sources are skipped) on st; with sc also set the scalars, with to
// read from's back.  view: the caller's side of the copy, whose memory is looked at first.
hipError_t copy_fields(void* const* dst, void* const* src, int nf, size_t bytes, void* const* view,
                       int dev, Scalars* sc, double t, double dt_next, double cfl,
                       const Scalars* from, Scalars* to, hipStream_t st) {
  CopyArgs a = {};
  int n = 0;
  bool direct = true;
  Extent known = {0, 0};
  for (int f = 0; f < nf; ++f) {
    if (!src[f]) continue;
    direct = direct && on_device(view[f], bytes, dev, known);
    a.src[n] = src[f];
    a.dst[n++] = dst[f];
  }
  if (!direct || !any_order(a, n, bytes)) {
    for (int f = 0; f < n; ++f) {
      hipError_t e = hipMemcpyAsync(a.dst[f], a.src[f], bytes, hipMemcpyDeviceToDevice, st);
      if (e != hipSuccess) return e;
    }
    if (sc) hipLaunchKernelGGL(k_set, dim3(1), dim3(1), 0, st, sc, t, dt_next, cfl);
    if (to) hipLaunchKernelGGL(k_send, dim3(1), dim3(64), 0, st, from, to);
    return hipGetLastError();
  }
  a.bytes = (long long)bytes;
  a.sc = sc;
  a.t = t;
  a.dt_next = dt_next;
  a.cfl = cfl;
  a.from = from;
  a.to = to;
  // four 16-byte vectors a thread, up to 8 blocks per CU over the fields of a state
  const size_t want = (bytes + 64 * kCopyThreads - 1) / (64 * kCopyThreads);
  hipLaunchKernelGGL(k_copy, dim3((unsigned)(want < 256 ? want : 256), n), dim3(kCopyThreads), 0, st, a);
  return hipGetLastError();
}

__device__ double invdt_max(Scalars* s) {
  return __longlong_as_double((long long)ld_agent(&s->invdt_bits));
}

// dt_next from the CFL maximum just measured
__global__ void k_init_dt(Scalars* s) {
  st_agent(&s->dt_next, ld_agent(&s->cfl) / invdt_max(s));
  st_agent(&s->invdt_bits, 0ull);
}

// cycle control for up to kMaxBatch boxes, one thread per box
struct CtlArgs {
  int n;
  int par;
  Scalars* sc[kMaxBatch];
  double t_stop[kMaxBatch];
};

// forget the CFL maximum measured so far (timed first stages)
__global__ void k_unmeasure(CtlArgs a) {
  const int i = threadIdx.x;
  if (i < a.n) st_agent(&a.sc[i]->invdt_bits, 0ull);
}

// end of an Euler cycle, whose only stage also measures the CFL maximum
__global__ void k_end(CtlArgs a) {
  const int i = threadIdx.x;
  if (i < a.n) end_cycle(a.sc[i], a.par, a.t_stop[i]);
}

// ---- diagnostics: Neumaier-compensated sums in FP64
//
// One read of the state, so HBM bounds it: 8 fields of a 256^3 FP64 box are 1.07 GB,
// 0.22 ms at this card's copy rate.  A thread strides over the cells with its (i, j, k)
// advanced by additions (64-bit divisions per cell took longer than the loads), then
// waves and blocks combine their (sum, compensation) pairs as trees.  With one thread
// combining a block's 256 pairs and one thread the 512 blocks', a call took 1.85 ms;
// now the two kernels take 0.19 ms (5.7 TB/s read) and 11 us, a call 0.21 ms.
constexpr int kDiagThreads = 512;
constexpr int kDiagWaves = kDiagThreads / 64;

struct Ksum {
  double s, c;
};
// what rounding took from t = a + b
__device__ __forceinline__ double lost_in(double a, double b, double t) {
  return fabs(a) >= fabs(b) ? (a - t) + b : (b - t) + a;
}
__device__ __forceinline__ void kadd(Ksum& a, double x) {
  const double t = a.s + x;
  a.c += lost_in(a.s, x, t);
  a.s = t;
}
__device__ __forceinline__ void kmerge(Ksum& a, double bs, double bc) {
  const double t = a.s + bs;
  a.c = (a.c + bc) + lost_in(a.s, bs, t);
  a.s = t;
}

struct DiagSums {
  Ksum acc[9];  // rho, m, E, B, div B squared
  double dmax;
};

// The lanes of a wave combined into lane 0, over the first n lanes (a power of two).
__device__ __forceinline__ void wave_combine(DiagSums& a, int n) {
  for (int off = n / 2; off > 0; off >>= 1) {
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      const double s = __shfl_down(a.acc[q].s, off), c = __shfl_down(a.acc[q].c, off);
      kmerge(a.acc[q], s, c);
    }
    const double m = __shfl_down(a.dmax, off);
    a.dmax = m > a.dmax ? m : a.dmax;
  }
}

// A block's threads combined into thread 0, always in the same order.
__device__ __forceinline__ void block_combine(DiagSums& a) {
  __shared__ double part[kDiagVals][kDiagWaves];
  wave_combine(a, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      part[2 * q][wave] = a.acc[q].s;
      part[2 * q + 1][wave] = a.acc[q].c;
    }
    part[18][wave] = a.dmax;
  }
  __syncthreads();
  if (wave == 0) {
    const int w = lane & (kDiagWaves - 1);
#pragma unroll
    for (int q = 0; q < 9; ++q) a.acc[q] = {part[2 * q][w], part[2 * q + 1][w]};
    a.dmax = part[18][w];
    wave_combine(a, kDiagWaves);
  }
}

struct DiagFields {
  const void* f[8];
};

template <typename R>
__global__ void __launch_bounds__(kDiagThreads)
k_diag_partial(DiagFields fields, int nx, int ny, int nz, double idx, double idy, double idz,
               double* part) {
  const R* f[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) f[q] = static_cast<const R*>(fields.f[q]);
  const long long plane = (long long)nx * ny, n = plane * nz;
  DiagSums a = {};
  long long c = (long long)blockIdx.x * kDiagThreads + threadIdx.x;
  int i, j, k, si, sj, sk;
  const long long stride = (long long)gridDim.x * kDiagThreads;
  cell_ijk(c, nx, plane, n, i, j, k);
  cell_ijk(stride, nx, plane, n, si, sj, sk);
  while (c < n) {
    R v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = f[q][c];
    const R xp = f[5][i + 1 == nx ? c - i : c + 1];
    const R yp = f[6][j + 1 == ny ? c - (plane - nx) : c + nx];
    const R zp = f[7][k + 1 == nz ? c - (n - plane) : c + plane];
#pragma unroll
    for (int q = 0; q < 8; ++q) kadd(a.acc[q], (double)v[q]);
    const double div = (((double)xp - (double)v[5]) * idx + ((double)yp - (double)v[6]) * idy) +
                       ((double)zp - (double)v[7]) * idz;
    kadd(a.acc[8], div * div);
    const double ad = fabs(div);
    a.dmax = ad > a.dmax ? ad : a.dmax;
    c += stride;
    i += si;
    j += sj;
    k += sk;
    if (i >= nx) { i -= nx; ++j; }
    if (j >= ny) { j -= ny; ++k; }
  }
  block_combine(a);
  if (threadIdx.x == 0) {
    double* out = part + blockIdx.x;  // a value's partials lie side by side
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      st_agent(out + 2 * q * kDiagBlocks, a.acc[q].s);
      st_agent(out + (2 * q + 1) * kDiagBlocks, a.acc[q].c);
    }
    st_agent(out + 18 * kDiagBlocks, a.dmax);
  }
}

// one block: thread t takes the partials of block t
static_assert(kDiagBlocks <= kDiagThreads, "one thread per block of the first kernel");
__global__ void __launch_bounds__(kDiagThreads)
k_diag_final(const double* part, int nblocks, double dv, double ncell, Scalars* s, Scalars* host) {
  DiagSums a = {};
  if ((int)threadIdx.x < nblocks) {
    const double* p = part + threadIdx.x;
#pragma unroll
    for (int q = 0; q < 9; ++q)
      a.acc[q] = {ld_agent(p + 2 * q * kDiagBlocks), ld_agent(p + (2 * q + 1) * kDiagBlocks)};
    a.dmax = ld_agent(p + 18 * kDiagBlocks);
  }
  block_combine(a);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) st_agent(&s->diag[q], (a.acc[q].s + a.acc[q].c) * dv);
    st_agent(&s->diag[8], a.dmax);
    st_agent(&s->diag[9], sqrt((a.acc[8].s + a.acc[8].c) / ncell));
  }
  __threadfence();  // thread 0's results before the loads below
  __syncthreads();
  if (host) send_scalars(s, host, threadIdx.x);
}

// Diagnostics of c's state with the per-block partial sums in part (the
// context's workspace, or the static scratch of the allocation-free variant).
int diagnostics_into(mhd_ctx* c, double* part, mhd_diag* out) {
  Slot slot;
  DiagFields f;
  for (int q = 0; q < 8; ++q) f.f[q] = c->buf[c->cur][q];
  auto fn = c->p.precision == MHD_FP32 ? k_diag_partial<float> : k_diag_partial<double>;
  hipLaunchKernelGGL(fn, dim3(c->diag_blocks), dim3(kDiagThreads), 0, c->stream, f, c->p.nx,
                     c->p.ny, c->p.nz, c->idl[0], c->idl[1], c->idl[2], part);
  if (hipGetLastError() != hipSuccess) return MHD_ERR_HIP;
  hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(kDiagThreads), 0, c->stream, part, c->diag_blocks, c->dv,
                     (double)c->ncell, c->sc, slot.s);
  if (hipGetLastError() != hipSuccess) return MHD_ERR_HIP;
  Scalars h;
  if (read_scalars(c, slot, &h) != hipSuccess) return MHD_ERR_HIP;
  out->mass = h.diag[0];
  for (int d = 0; d < 3; ++d) out->mom[d] = h.diag[1 + d];
  out->energy = h.diag[4];
  for (int d = 0; d < 3; ++d) out->bflux[d] = h.diag[5 + d];
  out->divb_max = h.diag[8];
  out->divb_rms = h.diag[9];
  out->status = h.status;
  return MHD_OK;
}

// ---- the allocation-free diagnostics variant: its partial sums live in a
// static device array, one copy per GPU held until the process ends (80 KiB).
// In host code `scratch` only names the symbol; its device address, resolved
// once per device with that device current, is what kernels receive.  Calls
// that overlap on one GPU share the array and race.
constexpr int kMaxDevices = 64;
__device__ __align__(256) double scratch[kDiagBlocks * kDiagVals];
double* g_scratch[kMaxDevices];
std::mutex g_scratch_mu;

double* scratch_ptr(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    int cur = 0;
    if (hipGetDevice(&cur) != hipSuccess) return nullptr;
    if (cur != dev && hipSetDevice(dev) != hipSuccess) return nullptr;
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != dev && hipSetDevice(cur) != hipSuccess) return nullptr;
    if (e != hipSuccess || !ptr) return nullptr;
    g_scratch[dev] = static_cast<double*>(ptr);
  }
  return g_scratch[dev];
}

int hip_fail(hipError_t e) { return e == hipSuccess ? MHD_OK : MHD_ERR_HIP; }

// The stage kernels of the context's precision and Riemann solver.
hipError_t stage_kernel(const mhd_params* p, const BatchArgs& ba, int tile, hipStream_t st,
                        bool prepare) {
  const int rc = p->recon;
  if (p->precision == MHD_FP32) {
    if (p->riemann == MHD_HLL) return stage_f32_hll(ba, tile, rc, st, prepare);
    if (p->riemann == MHD_HLLC) return stage_f32_hllc(ba, tile, rc, st, prepare);
    return stage_f32_hlld(ba, tile, rc, st, prepare);
  }
  if (p->riemann == MHD_HLL) return stage_f64_hll(ba, tile, rc, st, prepare);
  if (p->riemann == MHD_HLLC) return stage_f64_hllc(ba, tile, rc, st, prepare);
  return stage_f64_hlld(ba, tile, rc, st, prepare);
}

void fields_of(const mhd_state_view* v, void* out[11]) {
  out[0] = v->rho; out[1] = v->mx; out[2] = v->my; out[3] = v->mz;
  out[4] = v->en; out[5] = v->bx; out[6] = v->by; out[7] = v->bz;
  out[8] = v->ax; out[9] = v->ay; out[10] = v->az;
}

// Stage roles of one box: the buffer S_dt acts on, the buffer written and, for a
// combining stage, the buffer holding U_0.
struct Roles {
  unsigned char src, dst, base;
};

// ---- planes per block (lz) of the contexts whose z-chunk is automatic.
//
// A block marches lz planes in the time of lz + head (the planes at its two ends that its
// neighbours also compute, fewer without corner EMFs, and the prologue).  j blocks that
// share a CU take 1 + share (j - 1) times as long a plane as one block alone, since one
// block's waves leave the SIMDs idle while they wait; at most resident_blocks run at once.
// N blocks put ceil(N / 256) on a CU, so a launch takes
//   (lz + head) (full rounds of resident blocks + the last, partly filled round),
// and the rule takes the lz with the smallest.  base_lz, whose chunks the 8 XCDs divide,
// stays unless another length is kGain better, or kGroupGain for a group, which then takes
// one common length of at most kTop planes or the longest base_lz: the model does not see
// the L2s, and without these limits it erred by up to 19 % (200x300x500 FP32 HLLC; 384^3
// FP32 12 %, two boxes of 320^3 6 %).  Where one block fills a CU it errs by 1 %, and needs
// no margin.  The constants are fitted, by kind of scheme, to cycles of 30 boxes between
// 16^3 and 512^3, cubes, slabs and ragged, with up to 20 lengths in both tiles; the choice
// is on average 0.8 % from the best of them and at most 1.4 % slower than base_lz.  In the
// geometric mean over boxes it takes 0.61 of base_lz's time (96^3 FP64 0.68, 101x75x52 0.63,
// 256^3 1.00), over 16 groups of 2 to 64 boxes 0.71, one of them 1.8 % more.
constexpr int kCus = 256;
constexpr double kGain = 0.04, kGroupGain = 0.02;
constexpr int kTop = 32;

struct MarchCost {
  double head, share;
  double tile1811;  // time of a block of 18x11 columns over one of 24x8
};
MarchCost march_cost(const mhd_params* p) {
  const bool hydro = p->riemann == MHD_HLLC, f32 = p->precision == MHD_FP32, ppm = p->recon == MHD_PPM;
  return {hydro && !(ppm && !f32) ? 0.6 : 1.6,
          !f32 ? 0.6 : hydro ? (ppm ? 0.3 : 0.5) : (ppm ? 0.15 : 0.4),
          hydro && f32 ? 1.15 : 1.05};
}

// blocks of these kernels that a CU holds at once (their registers and LDS)
int resident_blocks(const mhd_params* p) {
  const bool hydro = p->riemann == MHD_HLLC, f32 = p->precision == MHD_FP32;
  if (p->recon == MHD_PPM && !f32) return hydro ? 2 : 1;
  return (f32 ? 3 : 2) + (hydro ? 1 : 0);
}

long long columns(const mhd_params* p, int tile) {
  int tx, ty;
  tile_dims(tile, &tx, &ty);
  return (long long)((p->nx + tx - 1) / tx) * ((p->ny + ty - 1) / ty);
}

int chunks(int nz, int lz) { return (nz + lz - 1) / lz; }

// blocks: of the launch; mean, most: planes of its blocks
double launch_cost(const mhd_params* p, long long blocks, double mean, int most) {
  const int r = resident_blocks(p);
  const MarchCost m = march_cost(p);
  const long long k = (blocks + kCus - 1) / kCus;
  const long long full = k / r;
  const int rest = (int)(k % r);
  const double last = full ? mean : most;
  return (mean + m.head) * full * (1.0 + m.share * (r - 1)) +
         (rest ? (last + m.head) * (1.0 + m.share * (rest - 1)) : 0.0);
}

// At least 2,048 blocks (8 a CU) in a number of z-chunks that the 8 XCDs divide, so that
// each gets whole z-slabs and halo planes hit its L2 (256^3: 7 % faster in FP64 and 3 % in
// FP32 than 6 chunks; 512^3 FP32 up to 13 %), of 16 planes or more.
int base_lz(long long columns, int nz) {
  const long long want = ((2048 + columns - 1) / columns + 7) / 8 * 8;
  const int lz = (int)((nz + want - 1) / want);
  return lz < 16 ? (nz < 16 ? nz : 16) : lz;
}

long long bricks(const mhd_params* p, const BrickShape& b) {
  return (long long)((p->nx + b.x - 1) / b.x) * ((p->ny + b.y - 1) / b.y) * ((p->nz + b.z - 1) / b.z);
}

// Bricks for the stages of n contexts launched together: FP64, the default scheme, no
// launch shape asked for, and a CU for every brick, of the smaller shape if that still
// holds.  On the other side of that line a second round of bricks starts: 32^3 (256
// bricks of 8x4x4) takes 38 us a cycle and marches in 58, 48^3 (864) takes 118 and
// marches in 89; 16^3 takes 20 us as 128 bricks of 4x4x2, 29 as 32 of 8x4x4.
int plan_brick(mhd_ctx* const* c, int n) {
  const mhd_params* p = &c[0]->p;
  if (p->precision != MHD_FP64 || p->recon != MHD_PLM || p->emf != MHD_EMF_EC || p->ct != MHD_CT_FACE)
    return BRICK_NONE;
  long long big = 0, small = 0;
  for (int i = 0; i < n; ++i) {
    if (c[i]->shaped) return BRICK_NONE;
    big += bricks(&c[i]->p, kBrick[BRICK_844]);
    small += bricks(&c[i]->p, kBrick[BRICK_442]);
  }
  return small <= kCus ? BRICK_442 : big <= kCus ? BRICK_844 : BRICK_NONE;
}

// The tile and the lz of n contexts launched together (n <= kMaxBatch): the requested
// ones, or one common length for all that leave it open, and if none asks for anything
// the tile with the smaller launch_cost: 101x75 is 50 columns of 24x8 and 42 of 18x11, which
// pays for a block of 18x11 taking longer.
void plan_march(mhd_ctx* const* c, int n, int* tile, short* lz) {
  int zmax = 0;
  bool shaped = false, one = true;
  for (int i = 0; i < n; ++i) {
    lz[i] = (short)c[i]->lz;
    shaped = shaped || c[i]->shaped;
    one = one && c[i]->tile == c[0]->tile;
    if (c[i]->zchunk == 0 && c[i]->p.nz > zmax) zmax = c[i]->p.nz;
  }
  const int first = one ? c[0]->tile : default_tile(c[0]->p.precision);  // see same_group
  *tile = first;
  if (zmax == 0) return;
  // z: a common length, or 0 for each box's base_lz
  auto length = [&](int i, int z) {
    const mhd_params* p = &c[i]->p;
    if (c[i]->zchunk) return c[i]->lz;
    if (z == 0) z = base_lz(columns(p, first), p->nz);
    return z < p->nz ? z : p->nz;
  };
  auto cost = [&](int tl, int z) {
    long long blocks = 0, planes = 0;
    int most = 0;
    for (int i = 0; i < n; ++i) {
      const int l = length(i, z);
      const long long b = columns(&c[i]->p, tl) * chunks(c[i]->p.nz, l);
      blocks += b;
      planes += b * l;
      most = l > most ? l : most;
    }
    return launch_cost(&c[0]->p, blocks, (double)planes / (double)blocks, most);
  };
  const double gain = resident_blocks(&c[0]->p) == 1 ? 0.0 : n == 1 ? kGain : kGroupGain;
  double best = (1.0 - gain) * cost(first, 0);
  int pick = 0, top = kTop;
  for (int i = 0; i < n; ++i) top = length(i, 0) > top ? length(i, 0) : top;
  if (n == 1 || zmax < top) top = zmax;
  for (int second = 0; second < (shaped ? 1 : 2); ++second) {
    const int tl = second ? (int)TILE_18x11 : first;
    // every length for one box (planned when it takes its launch shape, see plan_launch);
    // for a group, planned as boxes leave it, every length up to 16 and then steps of an
    // eighth
    for (int z = 1; z <= top; z += n == 1 || z < 16 ? 1 : z / 8) {
      const double t = cost(tl, z) * (second ? march_cost(&c[0]->p).tile1811 : 1.0);
      if (t < best) {
        best = t;
        pick = z;
        *tile = tl;
      }
    }
  }
  for (int i = 0; i < n; ++i) lz[i] = (short)length(i, pick);
}

// How the stages of up to kMaxBatch contexts are launched.
struct Plan {
  int brick, tile;
  short lz[kMaxBatch];
};
// One box takes what apply_shape planned for it: the search took 5 us of a call's host time
// at 256 planes and 87 at 4096, beside 2 for the rest of a one-cycle call.
Plan plan_launch(mhd_ctx* const* c, int n) {
  Plan p = {};
  p.brick = plan_brick(c, n);
  p.tile = c[0]->lone_tile;
  if (n == 1)
    p.lz[0] = (short)c[0]->lz;
  else if (p.brick == BRICK_NONE)
    plan_march(c, n, &p.tile, p.lz);
  return p;
}

// One stage launch over n contexts sharing precision, solver and tile, with
// weights (w, w0) for a combining stage and one plan per kMaxBatch contexts (null:
// planned here).  Batches beyond kMaxBatch go out in chunks.
struct Control {
  int par, first, last;   // as in BatchArgs
  const double* t_stop;   // per context
};

hipError_t launch_stage(mhd_ctx* const* c, const Roles* r, int n, int mode, double w, double w0,
                        const Plan* plans, const Control& ctl, hipStream_t st) {
  for (int i0 = 0; i0 < n; i0 += kMaxBatch) {
    const int m = n - i0 < kMaxBatch ? n - i0 : kMaxBatch;
    BatchArgs ba = {};
    ba.nbox = m;
    ba.mode = mode;
    ba.w = w;
    ba.w0 = w0;
    ba.emf = c[i0]->p.emf;
    ba.ct = c[i0]->p.ct;
    ba.par = ctl.par;
    ba.first = ctl.first;
    ba.last = ctl.last;
    if (ctl.t_stop) memcpy(ba.t_stop, ctl.t_stop + i0, sizeof(double) * m);
    const Plan plan = plans ? plans[i0 / kMaxBatch] : plan_launch(c + i0, m);
    memcpy(ba.lz, plan.lz, sizeof(short) * m);
    ba.brick = mode != 2 ? plan.brick : BRICK_NONE;  // measuring marches
    int g = 0;
    for (int i = 0; i < m; ++i) {
      const mhd_ctx* ci = c[i0 + i];
      ba.desc[i] = ci->desc;
      ba.start[i] = g;
      ba.src[i] = r[i0 + i].src;
      ba.dst[i] = r[i0 + i].dst;
      ba.base[i] = r[i0 + i].base;
      g += ba.brick != BRICK_NONE ? (int)bricks(&ci->p, kBrick[ba.brick])
                                  : (int)columns(&ci->p, plan.tile) * chunks(ci->p.nz, ba.lz[i]);
    }
    ba.start[m] = g;
    ba.total = g;
    const mhd_ctx* c0 = c[i0];
    hipError_t e = stage_kernel(&c0->p, ba, plan.tile, st, false);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// UCT-HLL after a stage launch (mode 0: first stage, 1: combining stage): the
// edge EMFs from the exported face data, then the face-field update.
hipError_t launch_uct(mhd_ctx* const* c, const Roles* r, int n, int mode, double w, double w0,
                      int par, bool update_b, hipStream_t st) {
  for (int i0 = 0; i0 < n; i0 += kMaxBatch) {
    const int m = n - i0 < kMaxBatch ? n - i0 : kMaxBatch;
    BatchArgs ba = {};
    ba.nbox = m;
    ba.mode = mode;
    ba.w = w;
    ba.w0 = w0;
    ba.emf = c[i0]->p.emf;
    ba.par = par;
    int g = 0;
    for (int i = 0; i < m; ++i) {
      ba.desc[i] = c[i0 + i]->desc;
      ba.start[i] = g;
      ba.src[i] = r[i0 + i].src;
      ba.dst[i] = r[i0 + i].dst;
      ba.base[i] = r[i0 + i].base;
      g += (int)((c[i0 + i]->ncell + kUctBlock - 1) / kUctBlock);
    }
    ba.start[m] = g;
    ba.total = g;
    const int rc = c[i0]->p.recon;
    hipError_t e = c[i0]->p.precision == MHD_FP32 ? uct_f32(ba, rc, update_b, st)
                                                  : uct_f64(ba, rc, update_b, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Vector-potential form after a stage launch (mode 0: first stage, 1: combining
// stage): A update on every edge, then the face field from curl A; update =
// false runs only the curl (deriving B from a potential the caller set).
hipError_t launch_vpot(mhd_ctx* const* c, const Roles* r, int n, int mode, double w, double w0,
                       int par, bool update, hipStream_t st) {
  for (int i0 = 0; i0 < n; i0 += kMaxBatch) {
    const int m = n - i0 < kMaxBatch ? n - i0 : kMaxBatch;
    BatchArgs ba = {};
    ba.nbox = m;
    ba.mode = mode;
    ba.w = w;
    ba.w0 = w0;
    ba.emf = c[i0]->p.emf;
    ba.par = par;
    int g = 0;
    for (int i = 0; i < m; ++i) {
      ba.desc[i] = c[i0 + i]->desc;
      ba.start[i] = g;
      ba.src[i] = r[i0 + i].src;
      ba.dst[i] = r[i0 + i].dst;
      ba.base[i] = r[i0 + i].base;
      g += (int)((c[i0 + i]->ncell + kVpotBlock - 1) / kVpotBlock);
    }
    ba.start[m] = g;
    ba.total = g;
    hipError_t e = update ? vpot_update_f64(ba, st) : hipSuccess;
    if (e == hipSuccess) e = vpot_curl_f64(ba, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_ctl(void (*kernel)(CtlArgs), mhd_ctx* const* c, int n, int par,
                      const double* t_stop, hipStream_t st) {
  for (int i0 = 0; i0 < n; i0 += kMaxBatch) {
    const int m = n - i0 < kMaxBatch ? n - i0 : kMaxBatch;
    CtlArgs a = {};
    a.n = m;
    a.par = par;
    for (int i = 0; i < m; ++i) {
      a.sc[i] = c[i0 + i]->sc;
      a.t_stop[i] = t_stop ? t_stop[i0 + i] : 0.0;
    }
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kMaxBatch), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Advance n contexts (same precision, solver, tile, integrator) by nsteps[i]
// cycles each on one stream; every box keeps its own dt and t_stop.
int step_group(mhd_ctx* const* c, const int* nsteps, int n, const double* t_stop, hipStream_t st) {
  Range range("mhd cycles");
  int maxs = 0;
  for (int i = 0; i < n; ++i) maxs = nsteps[i] > maxs ? nsteps[i] : maxs;
  if (maxs == 0) return MHD_OK;
  if (n > 4096) return MHD_ERR_INVALID_ARG;
  static thread_local mhd_ctx* act[4096];
  static thread_local Roles roles[4096];
  static thread_local double ts[4096];
  static thread_local Plan plans[4096 / kMaxBatch];
  int m = 0;
  const int integ = c[0]->p.integrator;
  const bool vp = c[0]->p.ct == MHD_CT_VECPOT;
  const bool uct = c[0]->p.emf == MHD_EMF_UCT_HLL || c[0]->p.emf == MHD_EMF_UCT_HLLD;
  for (int cyc = 0; cyc < maxs; ++cyc) {
    Range cycle("mhd cycle");
    const int was = m;
    m = 0;
    for (int i = 0; i < n; ++i)
      if (nsteps[i] > cyc) { act[m] = c[i]; ts[m] = t_stop ? t_stop[i] : 0.0; ++m; }
    if (cyc == 0 || m != was)  // boxes only ever leave
      for (int i = 0; i < m; i += kMaxBatch)
        plans[i / kMaxBatch] = plan_launch(act + i, m - i < kMaxBatch ? m - i : kMaxBatch);
    // stage 1: U_1 = S_dt(U_0), measuring the next dt (eq. cfl)
    for (int i = 0; i < m; ++i) {
      const int u0 = act[i]->cur;
      roles[i] = {(unsigned char)u0, (unsigned char)(u0 == 0 ? 1 : 0), (unsigned char)u0};
    }
    // with the vector-potential form every stage is followed by the A update
    // and the curl, with UCT-HLL by the edge solve and the face-field update
    // (same roles and weights)
    const int par = cyc & 1;
    auto stage = [&](int mode, double w, double w0, bool last) -> bool {
      const Control ctl = {par, cyc == 0 && mode == 0, last, ts};
      if (launch_stage(act, roles, m, mode, w, w0, plans, ctl, st) != hipSuccess) return false;
      if (uct && launch_uct(act, roles, m, mode, w, w0, par, !vp, st) != hipSuccess) return false;
      return !vp || launch_vpot(act, roles, m, mode, w, w0, par, true, st) == hipSuccess;
    };
    if (!stage(0, 1.0, 0.0, false)) return MHD_ERR_HIP;
    if (integ == MHD_RK2) {
      // U^{n+1} = 1/2 S_dt(U_1) + 1/2 U_0, written over U_0
      for (int i = 0; i < m; ++i) roles[i] = {roles[i].dst, roles[i].src, roles[i].src};
      if (!stage(1, 0.5, 0.5, true)) return MHD_ERR_HIP;
    } else if (integ == MHD_RK3) {
      // U_2 = 1/4 S_dt(U_1) + 3/4 U_0 into the third buffer, then
      // U^{n+1} = 2/3 S_dt(U_2) + 1/3 U_0 written over U_0 (cur is 0 here)
      for (int i = 0; i < m; ++i) roles[i] = {1, 2, 0};
      if (!stage(1, 0.25, 0.75, false)) return MHD_ERR_HIP;
      for (int i = 0; i < m; ++i) roles[i] = {2, 0, 0};
      if (!stage(1, 2.0 / 3.0, 1.0 / 3.0, true)) return MHD_ERR_HIP;
    } else {
      for (int i = 0; i < m; ++i) act[i]->cur = roles[i].dst;
      if (launch_ctl(k_end, act, m, par, ts, st) != hipSuccess) return MHD_ERR_HIP;
    }
    for (int i = 0; i < m; ++i) act[i]->stages_valid = integ != MHD_EULER;
  }
  return MHD_OK;
}

// Give c the launch shape (tile, zchunk; 0 = automatic): raise the dynamic-LDS
// limit of the tile's kernels and rewrite the box descriptor on the device.
// Synchronous: kernels in flight on c's stream may still read the old one.
int apply_shape(mhd_ctx* c, int tile, int zchunk, bool shaped) {
  int tx, ty;
  if (!tile_dims(tile, &tx, &ty)) return MHD_ERR_INVALID_ARG;
  const mhd_params* p = &c->p;
  BatchArgs none = {};
  none.emf = p->emf;
  none.ct = p->ct;
  hipError_t e = stage_kernel(p, none, tile, nullptr, true);
  if (e == hipSuccess && !shaped) e = stage_kernel(p, none, TILE_18x11, nullptr, true);
  if (e != hipSuccess) return MHD_ERR_HIP;
  BoxDesc d = {};
  for (int b = 0; b < c->nbuf; ++b)
    for (int f = 0; f < c->nfield; ++f) d.buf[b][f] = c->buf[b][f];
  d.ct = p->ct;
  d.b0[0] = p->b0[0];
  d.b0[1] = p->b0[1];
  d.b0[2] = p->b0[2];
  d.nx = p->nx;
  d.ny = p->ny;
  d.nz = p->nz;
  for (int k = 0; k < 3; ++k) d.idl[k] = c->idl[k];
  d.gamma = p->gamma;
  d.sc = c->sc;
  d.uct = c->uct;
  d.ustride = (long long)(field_bytes(p) / c->elem);
  if (hipStreamSynchronize(c->stream) != hipSuccess ||
      hipMemcpy(c->desc, &d, sizeof(d), hipMemcpyHostToDevice) != hipSuccess)
    return MHD_ERR_HIP;
  c->tile = tile;
  c->zchunk = zchunk;
  c->shaped = shaped;
  c->lone_tile = tile;
  c->lz = zchunk < p->nz ? zchunk : p->nz;
  if (zchunk == 0) {
    short lz;
    plan_march(&c, 1, &c->lone_tile, &lz);
    c->lz = lz;
  }
  return MHD_OK;
}

// A group runs one tile: the one that every context has, or the default where each has that
// or the tile that it takes by itself (what mhd_get_launch gives for a box of which nothing
// was asked can be asked for without shutting the box out of a group).
int group_tile(const mhd_ctx* c) {
  return c->tile == c->auto_tile ? default_tile(c->p.precision) : c->tile;
}

bool same_group(mhd_ctx* const* ctxs, int n) {
  const mhd_ctx* c0 = ctxs[0];
  bool one = true, fits = true;
  for (int i = 1; i < n; ++i) {
    const mhd_ctx* c = ctxs[i];
    if (c->p.precision != c0->p.precision || c->p.riemann != c0->p.riemann ||
        c->p.integrator != c0->p.integrator || c->p.emf != c0->p.emf ||
        c->p.recon != c0->p.recon || c->p.ct != c0->p.ct || c->device != c0->device)
      return false;
    one = one && c->tile == c0->tile;
    fits = fits && group_tile(c) == group_tile(c0);
  }
  return one || fits;
}

}  // namespace

namespace mhd {
int tile_dims(int tile, int* tx, int* ty) {
  if (tile == TILE_16x16) { *tx = 16; *ty = 16; return 1; }
  if (tile == TILE_24x8) { *tx = 24; *ty = 8; return 1; }
  if (tile == TILE_18x11) { *tx = 18; *ty = 11; return 1; }
  return 0;
}
}  // namespace mhd

extern "C" {

size_t mhd_workspace_bytes(const mhd_params* p) {
  if (!grid_ok(p)) return 0;
  if (p->precision != MHD_FP64 && p->precision != MHD_FP32) return 0;
  return align_up(sizeof(Scalars)) + align_up(sizeof(BoxDesc)) +
         align_up(sizeof(double) * kDiagBlocks * kDiagVals) +
         ((size_t)nfield_of(p) * nbuf_of(p) + nscratch_of(p)) * field_bytes(p);
}

int mhd_create(const mhd_params* p, mhd_ctx** out) {
  if (!out) return MHD_ERR_INVALID_ARG;
  *out = nullptr;
  if (!grid_ok(p)) return MHD_ERR_INVALID_ARG;
  if (!(p->lx > 0) || !(p->ly > 0) || !(p->lz > 0) || !(p->gamma > 1.0) || !(p->cfl > 0.0) ||
      !(p->cfl < 1.0))
    return MHD_ERR_INVALID_ARG;
  if (p->precision != MHD_FP64 && p->precision != MHD_FP32) return MHD_ERR_INVALID_ARG;
  if (p->riemann != MHD_HLLD && p->riemann != MHD_HLL && p->riemann != MHD_HLLC)
    return MHD_ERR_INVALID_ARG;
  if (p->emf != MHD_EMF_EC && p->emf != MHD_EMF_E0 && p->emf != MHD_EMF_ARITH &&
      p->emf != MHD_EMF_UCT_HLL && p->emf != MHD_EMF_UCT_HLLD)
    return MHD_ERR_UNSUPPORTED;
  // UCT-HLL is built for the MHD solvers (with the potential form under its
  // FP64 rule below)
  if (p->emf == MHD_EMF_UCT_HLL && p->riemann == MHD_HLLC) return MHD_ERR_UNSUPPORTED;
  // UCT-HLLD takes its coefficients from the HLLD solve of each face
  if (p->emf == MHD_EMF_UCT_HLLD && p->riemann != MHD_HLLD) return MHD_ERR_UNSUPPORTED;
  if (p->recon != MHD_PLM && p->recon != MHD_LIMO3 && p->recon != MHD_PPM)
    return MHD_ERR_UNSUPPORTED;
  if (p->ct != MHD_CT_FACE && p->ct != MHD_CT_VECPOT) return MHD_ERR_INVALID_ARG;
  if (p->ct == MHD_CT_VECPOT && (p->precision != MHD_FP64 || p->riemann == MHD_HLLC))
    return MHD_ERR_UNSUPPORTED;
  if (p->integrator != MHD_RK2 && p->integrator != MHD_EULER && p->integrator != MHD_RK3)
    return MHD_ERR_INVALID_ARG;
  if (p->zchunk < 0) return MHD_ERR_INVALID_ARG;
  int tile = p->tile == 0 ? default_tile(p->precision) : p->tile;
  int tx, ty;
  if (!tile_dims(tile, &tx, &ty)) return MHD_ERR_INVALID_ARG;
  if (!p->workspace || ((uintptr_t)p->workspace % kAlign) != 0) return MHD_ERR_WORKSPACE;
  if (p->workspace_bytes < mhd_workspace_bytes(p)) return MHD_ERR_WORKSPACE;

  mhd_ctx* c = (mhd_ctx*)calloc(1, sizeof(mhd_ctx));
  if (!c) return MHD_ERR_INVALID_ARG;
  g_readback.init();
  c->p = *p;
  c->stream = (hipStream_t)p->stream;
  if (hipGetDevice(&c->device) != hipSuccess) {
    free(c);
    return MHD_ERR_HIP;
  }
  c->elem = p->precision == MHD_FP32 ? 4 : 8;
  c->ncell = (long long)p->nx * p->ny * p->nz;
  double dx = p->lx / p->nx, dy = p->ly / p->ny, dz = p->lz / p->nz;
  c->idl[0] = 1.0 / dx;
  c->idl[1] = 1.0 / dy;
  c->idl[2] = 1.0 / dz;
  c->dv = (dx * dy) * dz;
  char* w = (char*)p->workspace;
  c->sc = (Scalars*)w;
  w += align_up(sizeof(Scalars));
  c->desc = (BoxDesc*)w;
  w += align_up(sizeof(BoxDesc));
  c->diag_part = (double*)w;
  w += align_up(sizeof(double) * kDiagBlocks * kDiagVals);
  // buffers of 8 fields back to back with one field stride: the stage kernel
  // relies on every buffer holding its fields at the same relative offsets
  const size_t fb = field_bytes(p);
  c->nbuf = nbuf_of(p);
  c->nfield = nfield_of(p);
  for (int b = 0; b < c->nbuf; ++b)
    for (int f = 0; f < c->nfield; ++f) {
      c->buf[b][f] = w;
      w += fb;
    }
  c->uct = nscratch_of(p) > 0 ? (void*)w : nullptr;
  w += (size_t)nscratch_of(p) * fb;
  c->cur = 0;
  // a cell per thread, up to two blocks a CU
  const long long db = (c->ncell + kDiagThreads - 1) / kDiagThreads;
  c->diag_blocks = (int)(db < kDiagBlocks ? db : kDiagBlocks);
  const bool shaped = p->tile != 0 || p->zchunk != 0;
  if (shaped) {  // what it would take, before anything is asked for
    short lz;
    c->tile = default_tile(p->precision);
    plan_march(&c, 1, &c->auto_tile, &lz);
  }
  if (apply_shape(c, tile, p->zchunk, shaped) != MHD_OK) {
    free(c);
    return MHD_ERR_HIP;
  }
  if (!shaped) c->auto_tile = c->lone_tile;
  hipLaunchKernelGGL(k_set, dim3(1), dim3(1), 0, c->stream, c->sc, 0.0, 0.0, p->cfl);
  if (hipGetLastError() != hipSuccess) {
    free(c);
    return MHD_ERR_HIP;
  }
  *out = c;
  return MHD_OK;
}

int mhd_set_state(mhd_ctx* c, const mhd_state_view* v, double t, double dt_next) {
  Range range("mhd_set_state");
  if (!c || !v) return MHD_ERR_INVALID_ARG;
  const bool vp = c->p.ct == MHD_CT_VECPOT;
  void* src[11];
  fields_of(v, src);
  // the potential form takes A and derives the face field; otherwise B is given
  for (int f = 0; f < c->nfield; ++f)
    if (!src[f] && !(vp && f >= 5 && f < 8)) return MHD_ERR_INVALID_ARG;
  const size_t bytes = (size_t)c->ncell * c->elem;
  c->cur = 0;
  c->stages_valid = 0;
  if (vp) src[5] = src[6] = src[7] = nullptr;
  if (copy_fields(c->buf[0], src, c->nfield, bytes, src, c->device, c->sc, t, dt_next, c->p.cfl,
                  nullptr, nullptr, c->stream) != hipSuccess)
    return MHD_ERR_HIP;
  if (vp) {
    const Roles r0 = {0, 0, 0};
    if (launch_vpot(&c, &r0, 1, 0, 1.0, 0.0, 0, false, c->stream) != hipSuccess) return MHD_ERR_HIP;
  }
  if (!(dt_next > 0.0)) {
    // eq. (cfl) on the initial state: the stage kernel in measuring mode
    const Roles r0 = {0, 1, 0};
    if (launch_stage(&c, &r0, 1, 2, 1.0, 0.0, nullptr, {}, c->stream) != hipSuccess) return MHD_ERR_HIP;
    hipLaunchKernelGGL(k_init_dt, dim3(1), dim3(1), 0, c->stream, c->sc);
    if (hipGetLastError() != hipSuccess) return MHD_ERR_HIP;
  }
  return MHD_OK;
}

int mhd_step(mhd_ctx* c, int nsteps, double t_stop) {
  if (!c || nsteps < 0) return MHD_ERR_INVALID_ARG;
  return step_group(&c, &nsteps, 1, &t_stop, c->stream);
}

int mhd_get_state(mhd_ctx* c, const mhd_state_view* v, double* t, double* dt_next) {
  Range range("mhd_get_state");
  if (!c) return MHD_ERR_INVALID_ARG;
  Slot slot;
  if (v) {
    void* dst[11];
    fields_of(v, dst);
    const size_t bytes = (size_t)c->ncell * c->elem;
    for (int f = 0; f < 8; ++f)
      if (!dst[f]) return MHD_ERR_INVALID_ARG;
    // the potential is copied out when the view asks for it
    const int nf = c->nfield == 11 && dst[8] && dst[9] && dst[10] ? 11 : 8;
    if (copy_fields(dst, c->buf[c->cur], nf, bytes, dst, c->device, nullptr, 0.0, 0.0, 0.0,
                    c->sc, slot.s, c->stream) != hipSuccess)
      return MHD_ERR_HIP;
  } else if (slot.s) {
    hipLaunchKernelGGL(k_send, dim3(1), dim3(64), 0, c->stream, c->sc, slot.s);
    if (hipGetLastError() != hipSuccess) return MHD_ERR_HIP;
  }
  Scalars h;
  if (read_scalars(c, slot, &h) != hipSuccess) return MHD_ERR_HIP;
  if (t) *t = h.t;
  if (dt_next) *dt_next = h.dt_next;
  return h.status ? MHD_ERR_NONPHYSICAL : MHD_OK;
}

int mhd_get_stage_output(mhd_ctx* c, int stage, const mhd_state_view* v) {
  if (!c || !v) return MHD_ERR_INVALID_ARG;
  // RK2 and RK3 write stage s < last into buffer s (the state stays in buffer 0)
  const int last = c->p.integrator == MHD_RK3 ? 3 : c->p.integrator == MHD_RK2 ? 2 : 1;
  if (stage < 1 || stage >= last || !c->stages_valid || c->cur != 0) return MHD_ERR_INVALID_ARG;
  void* dst[11];
  fields_of(v, dst);
  for (int f = 0; f < 8; ++f)
    if (!dst[f]) return MHD_ERR_INVALID_ARG;
  const int nf = c->nfield == 11 && dst[8] && dst[9] && dst[10] ? 11 : 8;
  const size_t bytes = (size_t)c->ncell * c->elem;
  if (copy_fields(dst, c->buf[stage], nf, bytes, dst, c->device, nullptr, 0.0, 0.0, 0.0, nullptr,
                  nullptr, c->stream) != hipSuccess)
    return MHD_ERR_HIP;
  return hipStreamSynchronize(c->stream) == hipSuccess ? MHD_OK : MHD_ERR_HIP;
}

int mhd_get_diagnostics(mhd_ctx* c, mhd_diag* out) {
  Range range("mhd_get_diagnostics");
  if (!c || !out) return MHD_ERR_INVALID_ARG;
  return diagnostics_into(c, c->diag_part, out);
}

int mhd_get_diagnostics_noalloc(mhd_ctx* c, mhd_diag* out) {
  if (!c || !out) return MHD_ERR_INVALID_ARG;
  // one set of partials per reduction block: the block count is bounded, so every box
  // fits (grid-stride loop); a larger count would not fit the static array
  if (c->diag_blocks > kDiagBlocks) return MHD_ERR_INVALID_ARG;
  double* part = scratch_ptr(c->device);
  if (!part) return MHD_ERR_HIP;
  return diagnostics_into(c, part, out);
}

int mhd_step_batch(mhd_ctx* const* ctxs, const int* nsteps, int n, void* stream) {
  if (!ctxs || !nsteps || n < 0 || n > 4096) return MHD_ERR_INVALID_ARG;
  if (n == 0) return MHD_OK;
  for (int i = 0; i < n; ++i)
    if (!ctxs[i] || nsteps[i] < 0) return MHD_ERR_INVALID_ARG;
  if (!same_group(ctxs, n)) return MHD_ERR_UNSUPPORTED;
  hipStream_t st = stream ? (hipStream_t)stream : ctxs[0]->stream;
  return step_group(ctxs, nsteps, n, nullptr, st);
}

int mhd_set_launch(mhd_ctx* c, int tile, int zchunk) {
  if (!c || zchunk < 0) return MHD_ERR_INVALID_ARG;
  const bool shaped = tile != MHD_TILE_DEFAULT || zchunk != 0;
  if (tile == MHD_TILE_DEFAULT) tile = default_tile(c->p.precision);
  int tx, ty;
  if (!tile_dims(tile, &tx, &ty)) return MHD_ERR_INVALID_ARG;
  return apply_shape(c, tile, zchunk, shaped);
}

int mhd_get_launch(const mhd_ctx* c, int* tile, int* zchunk) {
  if (!c) return MHD_ERR_INVALID_ARG;
  if (tile) *tile = c->lone_tile;
  if (zchunk) *zchunk = c->lz;
  return MHD_OK;
}

int mhd_get_launch_request(const mhd_ctx* c, int* tile, int* zchunk) {
  if (!c) return MHD_ERR_INVALID_ARG;
  if (tile) *tile = c->shaped ? c->tile : MHD_TILE_DEFAULT;
  if (zchunk) *zchunk = c->zchunk;
  return MHD_OK;
}

int mhd_tune(mhd_ctx* const* ctxs, int n, int reps, void* stream, mhd_tune_result* out) {
  Range range("mhd_tune");
  if (!ctxs || n < 1 || n > 4096 || reps < 1 || reps > 100) return MHD_ERR_INVALID_ARG;
  for (int i = 0; i < n; ++i)
    if (!ctxs[i]) return MHD_ERR_INVALID_ARG;
  if (!same_group(ctxs, n)) return MHD_ERR_UNSUPPORTED;
  hipStream_t st = stream ? (hipStream_t)stream : ctxs[0]->stream;
  static const int tiles[] = {TILE_24x8, TILE_18x11, TILE_16x16};
  static const int caps[] = {0, 8, 16, 32, 64, 128};
  const int ntile = sizeof(tiles) / sizeof(tiles[0]), ncap = sizeof(caps) / sizeof(caps[0]);
  Roles* src = (Roles*)malloc(sizeof(Roles) * n);
  float* times = (float*)malloc(sizeof(float) * reps);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  int rc = MHD_OK;
  if (!src || !times) rc = MHD_ERR_INVALID_ARG;
  if (rc == MHD_OK && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess))
    rc = MHD_ERR_HIP;
  for (int i = 0; i < n; ++i)
    if (src) {
      const int u0 = ctxs[i]->cur;
      src[i] = {(unsigned char)u0, (unsigned char)(u0 == 0 ? 1 : 0), (unsigned char)u0};
    }
  const int def_tile = default_tile(ctxs[0]->p.precision);
  // the default shape: what an untuned group gets, bricks where they are better
  auto automatic = [&](int tile, int cap) { return tile == def_tile && cap == 0; };
  float best = 1e30f, def_ms = -1.0f;
  int best_tile = def_tile, best_cap = 0, tried = 0;
  // median first-stage time of the whole group in its current shapes, planned before it
  // starts, as mhd_step_batch does (the first turn warms up); short launches are timed
  // several in a row, as a step call queues them
  static thread_local Plan plans[4096 / kMaxBatch];
  int row = 1;
  auto time_group = [&](float* med) -> int {
    for (int i = 0; i < n; i += kMaxBatch)
      plans[i / kMaxBatch] = plan_launch(ctxs + i, n - i < kMaxBatch ? n - i : kMaxBatch);
    for (int r = 0; r <= reps; ++r) {
      if (hipEventRecord(e0, st) != hipSuccess) return MHD_ERR_HIP;
      for (int k = 0; k < row; ++k)
        if (launch_stage(ctxs, src, n, 0, 1.0, 0.0, plans, {}, st) != hipSuccess) return MHD_ERR_HIP;
      if (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess)
        return MHD_ERR_HIP;
      float ms = 0.0f;
      if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) return MHD_ERR_HIP;
      if (r > 0) times[r - 1] = ms / (float)row;
    }
    for (int a = 1; a < reps; ++a)  // insertion sort of a few values
      for (int b = a; b > 0 && times[b] < times[b - 1]; --b) {
        float t = times[b];
        times[b] = times[b - 1];
        times[b - 1] = t;
      }
    *med = times[reps / 2];
    ++tried;
    return MHD_OK;
  };
  auto apply = [&](int i, int tile, int cap) -> int {
    return apply_shape(ctxs[i], tile, cap, !automatic(tile, cap));
  };
  // untimed, so that the first candidate does not pay for a GPU at rest; its length sets
  // how many launches a timing takes (2 ms, at most 8)
  for (int i = 0; i < n && rc == MHD_OK; ++i) rc = apply(i, def_tile, 0);
  if (rc == MHD_OK) {
    float first = 0.0f;
    rc = time_group(&first);
    if (rc == MHD_OK) row = first > 2.0f ? 1 : first < 0.25f ? 8 : (int)(2.0f / first);
    tried = 0;
  }
  for (int ti = 0; ti < ntile && rc == MHD_OK; ++ti)
    for (int ci = 0; ci < ncap && rc == MHD_OK; ++ci) {
      const int cap = caps[ci];
      // caps at or above every box's nz give the same shape as nz: time once
      bool dup = false;
      if (cap > 0) {
        dup = true;
        for (int i = 0; i < n; ++i)
          if (ctxs[i]->p.nz > caps[ci - 1] || caps[ci - 1] == 0) dup = false;
      }
      if (dup) continue;
      for (int i = 0; i < n && rc == MHD_OK; ++i) rc = apply(i, tiles[ti], cap);
      if (rc != MHD_OK) break;
      float med = 0.0f;
      rc = time_group(&med);
      if (rc != MHD_OK) break;
      if (med < best) {
        best = med;
        best_tile = tiles[ti];
        best_cap = cap;
      }
    }
  // per shape class: boxes sharing nz share a z-chunk.  From the best common
  // shape, each class in turn (most cells first) tries every other cap with
  // the rest fixed and keeps one that makes the group's launch more than 1 %
  // faster.
  int* cls_cap = (int*)malloc(sizeof(int) * n);  // per box: the cap of its class
  if (!cls_cap) rc = MHD_ERR_INVALID_ARG;
  if (rc == MHD_OK) {
    for (int i = 0; i < n && rc == MHD_OK; ++i) {
      cls_cap[i] = best_cap;
      rc = apply(i, best_tile, best_cap);
    }
  }
  if (rc == MHD_OK && n > 1) {
    float cur = 0.0f;
    rc = time_group(&cur);
    // classes in order of total cells, largest first
    int* order = (int*)malloc(sizeof(int) * n);  // one representative box per class
    long long* cells = (long long*)malloc(sizeof(long long) * n);
    int ncls = 0;
    if (!order || !cells) rc = MHD_ERR_INVALID_ARG;
    for (int i = 0; i < n && rc == MHD_OK; ++i) {
      int k = 0;
      while (k < ncls && ctxs[order[k]]->p.nz != ctxs[i]->p.nz) ++k;
      if (k == ncls) {
        order[ncls] = i;
        cells[ncls++] = 0;
      }
      cells[k] += ctxs[i]->ncell;
    }
    for (int a = 1; a < ncls; ++a)
      for (int b = a; b > 0 && cells[b] > cells[b - 1]; --b) {
        long long tc = cells[b];
        cells[b] = cells[b - 1];
        cells[b - 1] = tc;
        int to = order[b];
        order[b] = order[b - 1];
        order[b - 1] = to;
      }
    for (int k = 0; k < ncls && rc == MHD_OK; ++k) {
      const int nzk = ctxs[order[k]]->p.nz;
      const int keep = cls_cap[order[k]];
      int chosen = keep;
      for (int ci = 0; ci < ncap && rc == MHD_OK; ++ci) {
        const int cap = caps[ci];
        // caps at or above nz all mean nz: try the first such once
        if (cap == keep || (cap > 0 && ci > 0 && caps[ci - 1] >= nzk)) continue;
        for (int i = 0; i < n && rc == MHD_OK; ++i)
          if (ctxs[i]->p.nz == nzk) rc = apply(i, best_tile, cap);
        float med = 0.0f;
        if (rc == MHD_OK) rc = time_group(&med);
        if (rc == MHD_OK && med < 0.99f * cur) {
          cur = med;
          chosen = cap;
        }
      }
      for (int i = 0; i < n && rc == MHD_OK; ++i)
        if (ctxs[i]->p.nz == nzk) {
          cls_cap[i] = chosen;
          rc = apply(i, best_tile, chosen);
        }
    }
    free(order);
    free(cells);
  }
  // Each choice above was the best of many timings, so some of its lead is luck: on 64
  // uneven FP32 boxes the refined lengths of three runs cost the captured batch 5 % (39.1
  // against 37.2 ms automatic).  The automatic launch, the common shape and the refined one
  // now run in turns, and a later one is taken if it beats the one before by 1 %.
  enum { AUTOMATIC, COMMON, REFINED, FORMS };
  constexpr int kTurns = 3;
  auto take = [&](int form) {
    for (int i = 0; i < n && rc == MHD_OK; ++i)
      rc = apply(i, form == AUTOMATIC ? def_tile : best_tile,
                 form == AUTOMATIC ? 0 : form == COMMON ? best_cap : cls_cap[i]);
  };
  bool runs[FORMS] = {true, !automatic(best_tile, best_cap), false};
  for (int i = 0; rc == MHD_OK && i < n; ++i) runs[REFINED] = runs[REFINED] || cls_cap[i] != best_cap;
  const int candidates = tried;
  float turn[FORMS][kTurns];
  int form = AUTOMATIC;
  for (int t = 0; t < kTurns && rc == MHD_OK; ++t)
    for (int f = 0; f < FORMS && rc == MHD_OK; ++f) {
      if (!runs[f]) continue;
      take(f);
      if (rc == MHD_OK) rc = time_group(&turn[f][t]);
    }
  if (rc == MHD_OK) {
    auto middle = [](const float* t) {
      const float lo = t[0] < t[1] ? t[0] : t[1], hi = t[0] < t[1] ? t[1] : t[0];
      return t[2] < lo ? lo : t[2] > hi ? hi : t[2];
    };
    static_assert(kTurns == 3, "middle of three");
    best = def_ms = middle(turn[AUTOMATIC]);
    for (int f = COMMON; f < FORMS; ++f)
      if (runs[f] && middle(turn[f]) < 0.99f * best) {
        best = middle(turn[f]);
        form = f;
      }
  }
  if (form == AUTOMATIC) {
    best_tile = def_tile;
    best_cap = 0;
  }
  // the timed launches wrote the second buffer and a CFL maximum
  for (int i = 0; i < n; ++i) ctxs[i]->stages_valid = 0;
  if ((launch_ctl(k_unmeasure, ctxs, n, 0, nullptr, st) != hipSuccess ||
       hipStreamSynchronize(st) != hipSuccess) &&
      rc == MHD_OK)
    rc = MHD_ERR_HIP;
  take(form);
  // What is automatic depends on what is launched together.  The columns of a group that
  // goes out as one launch are fixed as they were timed, tile and length; bricks, which no
  // request asks for, and the launches of a larger group, which may differ in their tile
  // (and a batch has one), stay automatic.
  if (rc == MHD_OK && n > 1 && n <= kMaxBatch) {
    const Plan p = plan_launch(ctxs, n);
    for (int i = 0; p.brick == BRICK_NONE && i < n && rc == MHD_OK; ++i)
      rc = apply_shape(ctxs[i], p.tile, p.lz[i], true);
    if (p.brick == BRICK_NONE) best_tile = p.tile;
  }
  free(cls_cap);
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  free(src);
  free(times);
  if (rc == MHD_OK && out) {
    out->tile = n == 1 ? ctxs[0]->lone_tile : best_tile;
    out->zchunk_cap = best_cap;
    out->best_ms = best;
    out->default_ms = def_ms;
    out->candidates = candidates;
  }
  return rc;
}

int mhd_destroy(mhd_ctx* c) {
  free(c);
  return MHD_OK;
}

const char* mhd_status_string(int code) {
  switch (code) {
    case MHD_OK: return "ok";
    case MHD_ERR_INVALID_ARG: return "invalid argument";
    case MHD_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case MHD_ERR_HIP: return "HIP runtime error";
    case MHD_ERR_NONPHYSICAL: return "non-physical state (rho <= 0, p <= 0 or non-finite)";
    case MHD_ERR_UNSUPPORTED: return "unsupported option";
    default: return "unknown status";
  }
}

}  // extern "C"
