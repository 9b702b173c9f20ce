// HIP kernels for gfx950 and the C ABI declared in include/acdc.h.
//
// Kernels (one instantiation per supported width):
//   k_real_mq      per-layer quartet coefficients of the layer middle (tiny)
//   k_real_fwd     forward cascade, up to FWD_ROWS rows per workgroup, all K layers
//                  fused, rows kept in registers + one LDS slab per row
//   k_real_bwd     backward cascade with the reduction of dL/da, dL/dd over
//                  the workgroup's rows into one partial per tile, or
//                  (unbiased rows in tiles of at most two rows) persistent
//                  workgroups that add their tiles into one partial each
//   k_real_reduce  fixed-order sum of the partials over workgroups
//   k_real_dct     DCT-II of the batch sums of g (bias gradient, tiny)
// The multi-pass path (acdc_multipass.hip) serves widths beyond the fused
// plans and ACDC_FLAG_MULTIPASS; its host sequence is at the end of this file.
//   k_cplx_*       the same for the complex AFDF layers
#include <hip/hip_runtime.h>

#include <cstdio>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "acdc.h"
#include "acdc_devctx.hpp"
#include "acdc_multipass.hpp"
#include "acdc_registry.hpp"

namespace acdc {

// Number of row syncs (GroupCtx) on this device whose polling budget ran out
// before the row's waves had all arrived; nonzero would mean wrong results.
// acdc_sync_timeouts reads and clears it.
static __device__ unsigned long long sync_timeouts;

// Threads past the K * NSL * T table entries repack perm for the row
// kernels (RealOps::pack_perm_entry), when P16 is given.
template <class PL>
__global__ __launch_bounds__(256) void k_real_mq(const float* __restrict__ D, const float* __restrict__ Bias,
                                                 float4* __restrict__ Mq, int K, const char* __restrict__ tab,
                                                 const int* __restrict__ perm, int4* __restrict__ P16) {
  constexpr int E = PL::NSL * PL::T;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long long)K * E) {
    using O = RealOps<PL>;
    if constexpr (O::kPackedPerm) {
      constexpr int W = O::NIW * PL::T;
      const long long q = i - (long long)K * E;
      if (P16 == nullptr || q >= (long long)K * W) return;
      const int k = int(q / W), r = int(q % W);
      P16[q] = O::pack_perm_entry(perm + (long long)k * PL::N, r / PL::T, unsigned(r % PL::T));
    }
    return;
  }
  const int k = int(i / E), e = int(i % E);
  float4 row[kMqRows];
  real_mq_entry<PL>(D + (long long)k * PL::N, Bias != nullptr ? Bias + (long long)k * PL::N : nullptr, tab, e, row);
  // layout [k][slot][r][t]
  const int slot = e / PL::T, t = e % PL::T;
  float4* out = Mq + (long long)k * E * kMqRows + (long long)slot * kMqRows * PL::T + t;
#pragma unroll
  for (int r = 0; r < kMqRows; ++r) out[r * PL::T] = row[r];
}

// Copy of the FFT twiddle table (the first TW_FLOAT2 float2 of the plan's
// constant table) into LDS; the caller synchronises.
template <class PL>
__device__ __forceinline__ void copy_twiddles(float* dst, const char* tab, int tid, int nthreads) {
  const float2* src = reinterpret_cast<const float2*>(tab);
  float2* d2 = reinterpret_cast<float2*>(dst);
  for (int i = tid; i < PL::TW_FLOAT2; i += nthreads) d2[i] = src[i];
}

// The forward kernel is persistent: workgroup b handles row groups (tiles)
// b, b + gridDim.x, ... of `rpw` rows (fwd_rows).  Rows are independent, so
// results do not depend on the grid size or on rpw.
// ALONE: see fwd_alone.
template <class PL, bool BIAS, bool ALONE>
__global__ __launch_bounds__(ALONE ? kAloneThreads : Launch<PL>::FWD_THREADS)
__attribute__((amdgpu_waves_per_eu(ALONE ? 1 : Launch<PL>::FWD_WPE))) void k_real_fwd(RealArgs a, long long ntiles, int rpw) {
  using L = Launch<PL>;
  constexpr int THREADS = ALONE ? kAloneThreads : L::FWD_THREADS;
  __shared__ float lds[L::TW_FLOATS + THREADS / PL::T * L::FWD_SLAB];
  DevCtx<PL::T> ctx;
  const int tid = threadIdx.x;
  const unsigned t = unsigned(tid) % PL::T;
  int r = tid / PL::T;
  if constexpr (PL::T >= 64) r = __builtin_amdgcn_readfirstlane(r);  // one row per whole wave
  // LDS: [twiddle copy (TW_FLOATS)][row slabs]; the table sits at offset 0
  // so that its loads address it through the instruction's immediate offset
  float* const rows = lds + L::TW_FLOATS;
  float* slab = rows + r * L::FWD_SLAB;
  if constexpr (L::TW_LDS) {
    float* twl = lds;
    copy_twiddles<PL>(twl, a.tab, tid, THREADS);
    ctx.sync_all();
    if (r >= rpw) return;  // whole waves, which have no row: no barrier follows
    const LdsView tw = LdsView::of(twl);
    for (long long tile = blockIdx.x; tile < ntiles; tile += gridDim.x)
      real_forward_row<PL, BIAS, ALONE>(ctx, a, t, tile * rpw, unsigned(r), slab, tw);
  } else {
    const GView tw = GView::of(a.tab);
    for (long long tile = blockIdx.x; tile < ntiles; tile += gridDim.x)
      real_forward_row<PL, BIAS>(ctx, a, t, tile * L::FWD_ROWS, unsigned(r), slab, tw);
  }
}

// Persistent accumulation over tiles: whole tiles of the unbiased plans that
// have it.
template <class PL, bool BIAS, int ROWS>
constexpr bool bwd_acc() {
  return Launch<PL>::BWD_ACC && !BIAS && ROWS == Launch<PL>::BWD_ROWS;
}

// ROWS: rows per workgroup (bwd_rows)
template <class PL, bool BIAS, int ROWS>
__global__ __launch_bounds__(ROWS * PL::T)
__attribute__((amdgpu_waves_per_eu(Launch<PL>::BWD_WPE))) void k_real_bwd(RealArgs a, long long ntiles) {
  using L = Launch<PL>;
  constexpr bool ACC = bwd_acc<PL, BIAS, ROWS>();
  constexpr int LDS_FLOATS = ROWS * L::BWD_SLAB + L::BWD_TW_FLOATS;
  __shared__ float lds[LDS_FLOATS + (ACC ? L::ACC_FLOATS : 0)];
  const int tid = threadIdx.x;
  const unsigned t = unsigned(tid) % PL::T;
  int r = tid / PL::T;
  if constexpr (PL::T >= 64) r = __builtin_amdgcn_readfirstlane(r);  // one row per whole wave
  // LDS: [twiddle copy (TW_FLOATS)][row slabs][previous partial values (ACC)];
  // the table sits at offset 0 so that its loads address it through the
  // instruction's immediate offset
  float* const rows = lds + L::BWD_TW_FLOATS;
  float* slab = rows + r * L::BWD_SLAB;
  auto body = [&](auto& ctx) {
    if constexpr (ACC) {
      // persistent: workgroup w runs tiles w, w + G, ... (G = gridDim.x) and
      // adds them, in that order, into partial slot w
      static_assert(!L::BWD_TW_LDS, "persistent backward reads its twiddles from global memory");
      float* const old = lds + LDS_FLOATS;
      const unsigned w = blockIdx.x, nt = unsigned(ntiles);  // tiles < 2^31: batch <= 2^40 / N rows and N >= 1024
      for (unsigned tile = w; tile < nt; tile += gridDim.x)
        real_backward_row<PL, ROWS, BIAS, true>(ctx, a, t, (long long)tile * ROWS, unsigned(r), tid,
                                                       w, rows, slab, GView::of(a.tab), tile == w ? nullptr : old);
    } else if constexpr (L::BWD_TW_LDS) {
      // one tile per workgroup, one partial slot per tile
      const long long tile = blockIdx.x;
      float* twl = lds;
      copy_twiddles<PL>(twl, a.tab, tid, ROWS * PL::T);
      ctx.sync_all();
      real_backward_row<PL, ROWS, BIAS>(ctx, a, t, tile * ROWS, unsigned(r), tid, tile, rows, slab,
                                               LdsView::of(twl));
    } else {
      const long long tile = blockIdx.x;
      real_backward_row<PL, ROWS, BIAS>(ctx, a, t, tile * ROWS, unsigned(r), tid, tile, rows, slab,
                                               GView::of(a.tab));
    }
  };
  if constexpr (L::group_sync(ROWS)) {
    // rows of several waves meet at their own LDS counter (GroupCtx)
    using G = GroupCtx<PL::T>;
    __shared__ unsigned words[G::kWords * ROWS];
    if (tid < G::kWords * ROWS) words[tid] = 0u;
    DevCtx<PL::T>::lds_barrier();
    G ctx(&words[G::kWords * r]);
    body(ctx);
    G::report(words, ROWS, tid, &sync_timeouts);
  } else {
    DevCtx<PL::T> ctx;
    body(ctx);
  }
}

// Batch reduction: a block of kRedThreads threads owns kRedThreads / PH
// float4 entries of the reduced gradient (over all layers, entry index
// k * PS4 + e4) and sums them over the tiles with one thread per (entry,
// phase); phase sums meet in LDS and are added in phase order
// (tile_phase_sum4 / phases_total4).  128-thread blocks beat 256 and 64
// threads at N = 4096.
constexpr int kRedThreads = 128;

template <class PL, int PH>
__global__ __launch_bounds__(kRedThreads) void k_real_reduce(const float* __restrict__ partial, long long ntiles, int K,
                                                     float* __restrict__ gA, float* __restrict__ gD,
                                                     float* __restrict__ gS, const char* __restrict__ tab,
                                                     int bias, int accumulate) {
  const long long PS4 = partial_entries4<PL>(bias != 0);
  constexpr int E = kRedThreads / PH;
  __shared__ float4 ph[PH][E];
  const int lane = threadIdx.x % E, g = threadIdx.x / E;
  const long long i = (long long)blockIdx.x * E + lane;
  const long long n = (long long)K * PS4;
  ph[g][lane] = i < n ? tile_phase_sum4<PH>(reinterpret_cast<const float4*>(partial), ntiles, n, i, g)
                      : make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();
  if (g == 0 && i < n) {
    float4 all[PH];
#pragma unroll
    for (int q = 0; q < PH; ++q) all[q] = ph[q][lane];
    real_reduce_store4<PL>(phases_total4<PH>(all), int(i / PS4), int(i % PS4), gA, gD, gS, tab, accumulate != 0);
  }
}

// Bias gradient: grad_b[k] (+)= DCT-II of the batch sum of g at layer k.
// One workgroup of T threads per layer.
template <class PL>
__global__ __launch_bounds__(PL::T) void k_real_dct(const float* __restrict__ S, float* __restrict__ gB,
                                                    const float4* __restrict__ Mq, const char* __restrict__ tab,
                                                    int accumulate) {
  __shared__ float lds[Launch<PL>::FWD_SLAB];
  DevCtx<PL::T> ctx;
  const long long k = blockIdx.x;
  real_dct_row<PL>(ctx, S + k * PL::N, gB + k * PL::N, Mq, accumulate != 0, threadIdx.x, lds, GView::of(tab), tab);
}

template <class PL>
__global__ __launch_bounds__(Launch<PL>::FWD_THREADS)
__attribute__((amdgpu_waves_per_eu(Launch<PL>::FWD_WPE))) void k_cplx_fwd(CplxArgs a) {
  using L = Launch<PL>;
  __shared__ float lds[L::FWD_ROWS * L::FWD_SLAB];
  DevCtx<PL::T> ctx;
  const int tid = threadIdx.x;
  const unsigned t = unsigned(tid) % PL::T;
  int r = tid / PL::T;
  if constexpr (PL::T >= 64) r = __builtin_amdgcn_readfirstlane(r);  // one row per whole wave
  cplx_forward_row<PL>(ctx, a, t, (long long)blockIdx.x * L::FWD_ROWS, unsigned(r), lds + r * L::FWD_SLAB);
}

template <class PL, int ROWS>
__global__ __launch_bounds__(ROWS * PL::T)
__attribute__((amdgpu_waves_per_eu(Launch<PL>::BWD_WPE))) void k_cplx_bwd(CplxArgs a) {
  using L = Launch<PL>;
  __shared__ float lds[ROWS * L::BWD_SLAB];
  const int tid = threadIdx.x;
  const unsigned t = unsigned(tid) % PL::T;
  int r = tid / PL::T;
  if constexpr (PL::T >= 64) r = __builtin_amdgcn_readfirstlane(r);  // one row per whole wave
  if constexpr (L::group_sync(ROWS)) {
    using G = GroupCtx<PL::T>;
    __shared__ unsigned words[G::kWords * ROWS];
    if (tid < G::kWords * ROWS) words[tid] = 0u;
    DevCtx<PL::T>::lds_barrier();
    G ctx(&words[G::kWords * r]);
    cplx_backward_row<PL, ROWS>(ctx, a, t, (long long)blockIdx.x * ROWS, unsigned(r), tid,
                                       (long long)blockIdx.x, lds, lds + r * L::BWD_SLAB);
    G::report(words, ROWS, tid, &sync_timeouts);
  } else {
    DevCtx<PL::T> ctx;
    cplx_backward_row<PL, ROWS>(ctx, a, t, (long long)blockIdx.x * ROWS, unsigned(r), tid,
                                       (long long)blockIdx.x, lds, lds + r * L::BWD_SLAB);
  }
}

template <class PL, int PH>
__global__ __launch_bounds__(kRedThreads) void k_cplx_reduce(const float* __restrict__ partial, long long ntiles, int K,
                                                     float* __restrict__ gA, float* __restrict__ gD,
                                                     int accumulate) {
  constexpr long long PS4 = partial_entries4<PL>();
  constexpr int E = kRedThreads / PH;
  __shared__ float4 ph[PH][E];
  const int lane = threadIdx.x % E, g = threadIdx.x / E;
  const long long i = (long long)blockIdx.x * E + lane;
  const long long n = (long long)K * PS4;
  ph[g][lane] = i < n ? tile_phase_sum4<PH>(reinterpret_cast<const float4*>(partial), ntiles, n, i, g)
                      : make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();
  if (g == 0 && i < n) {
    float4 all[PH];
#pragma unroll
    for (int q = 0; q < PH; ++q) all[q] = ph[q][lane];
    cplx_reduce_store4<PL>(phases_total4<PH>(all), int(i / PS4), int(i % PS4), gA, gD, accumulate != 0);
  }
}

// Scratch of the no-allocation forward (acdc_forward_noalloc): the per-layer
// quartet coefficients that acdc_forward keeps in the caller's workspace.
// Each device holds its own copy until the process ends; host code reaches
// it only through the address hipGetSymbolAddress returns on that device.
constexpr size_t kNoAllocScratchBytes = size_t(16) << 20;
static __device__ __align__(256) float4 scratch[kNoAllocScratchBytes / sizeof(float4)];

// ------------------------------------------------------------------ host side

namespace {

thread_local int g_last_hip = 0;
std::mutex g_mu;
std::map<std::tuple<int, int, int>, void*> g_tables;  // (device, N, complex) -> device table

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

int hip_fail(hipError_t e) {
  g_last_hip = int(e);
  return ACDC_ERR_HIP;
}

// ----------------------------------------------------------- kernel timing
// While enabled, every main kernel launch is bracketed by HIP events on its
// stream (kind 0: forward cascade, 1: backward cascade, 2: batch reduction).
struct ProfRec {
  hipEvent_t a, b;
  int kind;
};
bool g_prof_on = false;
std::mutex g_prof_mu;
std::vector<ProfRec> g_prof_recs;
std::vector<hipEvent_t> g_prof_pool;

hipEvent_t prof_event() {
  if (!g_prof_pool.empty()) {
    hipEvent_t e = g_prof_pool.back();
    g_prof_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

struct ProfScope {
  int kind;
  hipStream_t s;
  hipEvent_t a = nullptr, b = nullptr;
  ProfScope(int k, hipStream_t st) : kind(k), s(st) {
    if (!g_prof_on) return;
    std::lock_guard<std::mutex> lock(g_prof_mu);
    a = prof_event();
    b = prof_event();
    if (a && b) (void)hipEventRecord(a, s);
  }
  ~ProfScope() {
    if (!a || !b) return;
    (void)hipEventRecord(b, s);
    std::lock_guard<std::mutex> lock(g_prof_mu);
    g_prof_recs.push_back(ProfRec{a, b, kind});
  }
};

bool fused_supported(int N, unsigned flags) {
  bool ok = false;
  auto probe = [&]<class PL>() { ok = true; };
  if (flags & kFlagComplex) dispatch_complex(N, probe);
  else dispatch_real(N, probe);
  return ok;
}

// Multi-pass path: power-of-two rows, real ones of width 256 ... 2^22 and
// complex ones of 256 ... 2^21 elements (the same M <= 2^21 point FFTs).
bool mp_width(long long N) { return N >= 256 && N <= (1LL << 22) && (N & (N - 1)) == 0; }
bool mp_width(long long N, unsigned flags) {
  return (flags & kFlagComplex) ? N <= (1LL << 21) && mp_width(N) : mp_width(N);
}
bool use_multipass(int N, unsigned flags) {
  return (flags & kFlagMultipass) != 0 || !fused_supported(N, flags);
}
bool supported(int N, unsigned flags) { return use_multipass(N, flags) ? mp_width(N, flags) : true; }

// Constant table of (N, complex) on the current device; built and uploaded
// on first use.
int get_table(int N, bool cplx, const char** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  std::lock_guard<std::mutex> lock(g_mu);
  auto key = std::make_tuple(dev, N, cplx ? 1 : 0);
  auto it = g_tables.find(key);
  if (it != g_tables.end()) {
    *out = static_cast<const char*>(it->second);
    return ACDC_OK;
  }
  std::vector<unsigned char> host;
  bool built = false, ok = false;
  auto build = [&]<class PL>() {
    built = true;
    if constexpr (PL::kComplex) ok = build_complex_tables<PL>(host);
    else ok = build_real_tables<PL>(host);
  };
  if (cplx) dispatch_complex(N, build);
  else dispatch_real(N, build);
  if (!built) return ACDC_ERR_UNSUPPORTED;
  if (!ok) return ACDC_ERR_UNSUPPORTED;
  void* d = nullptr;
  e = hipMalloc(&d, host.size());
  if (e != hipSuccess) return hip_fail(e);
  e = hipMemcpy(d, host.data(), host.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(d);
    return hip_fail(e);
  }
  g_tables[key] = d;
  *out = static_cast<const char*>(d);
  return ACDC_OK;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Workgroups of `kernel` (with `threads` threads) that fit on the current
// device at once (n; the persistent kernels launch min(tiles, n)) and the
// device's CUs.  With `remember` false a value not yet cached is computed
// without caching it (the no-allocation entry point inserts nothing).
struct Resident {
  long long n = 0;
  int cus = 0;
};
std::map<std::pair<const void*, int>, Resident> g_resident;
Resident resident_workgroups(const void* kernel, int threads, bool remember = true) {
  Resident r;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return r;
  std::lock_guard<std::mutex> lock(g_mu);
  auto key = std::make_pair(kernel, dev);
  auto it = g_resident.find(key);
  if (it != g_resident.end()) return it->second;
  int per_cu = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) == hipSuccess &&
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
    r = Resident{(long long)per_cu * cus, cus};
  if (remember) g_resident[key] = r;
  return r;
}

long long persistent_grid(long long resident, long long tiles) {
  return (resident > 0 && resident < tiles) ? resident : tiles;
}

// Per-device address of `scratch`, set by acdc_prepare (the library's set-up
// call) with the device current; null until then.
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};

int scratch_setup() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  if (dev < 0 || dev >= kMaxDevices) return ACDC_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_mu);
  if (g_scratch_ptr[dev] != nullptr) return ACDC_OK;
  void* p = nullptr;
  e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return hip_fail(e);
  g_scratch_ptr[dev] = p;
  return ACDC_OK;
}

// The constant table of (N, complex) on device `dev` if it exists (never
// builds one).
const char* find_table(int dev, int N, bool cplx) {
  std::lock_guard<std::mutex> lock(g_mu);
  auto it = g_tables.find(std::make_tuple(dev, N, cplx ? 1 : 0));
  return it == g_tables.end() ? nullptr : static_cast<const char*>(it->second);
}

constexpr uint32_t kAllFlags = kFlagPerm | kFlagRelu | kFlagComplex | kFlagBias | kFlagAccumulate | kFlagMultipass;

bool flags_supported(uint32_t flags) {
  return !((flags & kFlagComplex) && (flags & (kFlagRelu | kFlagBias)));
}

int check_common(int64_t batch, int32_t N, int32_t K, uint32_t flags) {
  if (flags & ~kAllFlags) return ACDC_ERR_INVALID_ARG;
  if (!flags_supported(flags)) return ACDC_ERR_UNSUPPORTED;
  if (batch < 0 || K < 1 || K > 65535 || N < 1) return ACDC_ERR_INVALID_ARG;
  if (!supported(N, flags)) return ACDC_ERR_UNSUPPORTED;
  if (batch > (int64_t(1) << 40) / N) return ACDC_ERR_INVALID_ARG;
  return ACDC_OK;
}

int check_ptrs(std::initializer_list<const void*> must, std::initializer_list<const void*> may) {
  for (const void* p : must)
    if (p == nullptr || !aligned16(p)) return ACDC_ERR_INVALID_ARG;
  for (const void* p : may)
    if (p != nullptr && !aligned16(p)) return ACDC_ERR_INVALID_ARG;
  return ACDC_OK;
}

bool distinct(std::initializer_list<const void*> outs, std::initializer_list<const void*> all) {
  for (const void* o : outs) {
    if (o == nullptr) continue;
    int seen = 0;
    for (const void* p : all)
      if (p == o) ++seen;
    if (seen != 1) return false;
  }
  return true;
}

template <class PL>
long long fwd_blocks(int64_t batch) {
  return (batch + Launch<PL>::FWD_ROWS - 1) / Launch<PL>::FWD_ROWS;
}
template <class PL>
long long bwd_tiles(int64_t batch) {
  return (batch + bwd_rows<PL>(batch) - 1) / bwd_rows<PL>(batch);
}
// f.template operator()<ROWS>() for the call's rows per backward workgroup.
template <class PL, class F>
void with_bwd_rows(int64_t batch, F&& f) {
  using L = Launch<PL>;
  if (L::BWD_ROWS_FEW != L::BWD_ROWS && bwd_rows<PL>(batch) == L::BWD_ROWS_FEW) f.template operator()<L::BWD_ROWS_FEW>();
  else f.template operator()<L::BWD_ROWS>();
}

size_t elem_floats(uint32_t flags) { return (flags & kFlagComplex) ? 2 : 1; }

// Floats of the `saved` buffer: the layer inputs u_1..u_{K-1}, preceded by
// u_0 (x gathered through perm[0]) with PERM.
size_t saved_layers(int32_t K, uint32_t flags) { return size_t(K - 1) + ((flags & kFlagPerm) ? 1 : 0); }
size_t saved_floats(int64_t batch, int32_t N, int32_t K, uint32_t flags) {
  return saved_layers(K, flags) * size_t(batch) * size_t(N) * elem_floats(flags);
}

struct WsLayout {
  size_t mq = 0, partial = 0, gs = 0, stash = 0, total = 0;
  size_t off_mq = 0, off_partial = 0, off_gs = 0, off_stash = 0;
};

// The quartet table, then for the backward (with PERM, where the plan packs
// it) the packed perm of every layer.
template <class PL>
size_t mq_table_bytes(int32_t K) {
  return align256(size_t(K) * PL::NSL * kMqRows * PL::T * sizeof(float4));
}
template <class PL>
size_t mq_bytes(int32_t K, uint32_t flags, bool backward) {
  using O = RealOps<PL>;
  const bool packed = backward && O::kPackedPerm && (flags & kFlagPerm) != 0;
  return mq_table_bytes<PL>(K) + (packed ? align256(size_t(K) * O::NIW * PL::T * sizeof(int4)) : 0);
}
template <class PL>
int4* perm16_of(float4* Mq, int32_t K, uint32_t flags) {
  if (!RealOps<PL>::kPackedPerm || !(flags & kFlagPerm)) return nullptr;
  return reinterpret_cast<int4*>(reinterpret_cast<char*>(Mq) + mq_table_bytes<PL>(K));
}

WsLayout bwd_layout(int64_t batch, int32_t N, int32_t K, uint32_t flags, bool have_saved) {
  WsLayout w;
  const bool bias = (flags & kFlagBias) != 0;
  auto f = [&]<class PL>() {
    // a buffer sized for one batch also serves the smaller ones, whose tiles
    // may be more (at most kCus, see bwd_rows)
    long long tiles = bwd_tiles<PL>(batch);
    if (Launch<PL>::BWD_ROWS_FEW != Launch<PL>::BWD_ROWS && batch > kCus * Launch<PL>::BWD_ROWS_FEW && tiles < kCus)
      tiles = kCus;
    w.partial = align256(size_t(tiles) * K * partial_entries4<PL>(bias) * sizeof(float4));
    if constexpr (!PL::kComplex) {
      // the bias gradient's DCT reads w, qa, qb' from the quartet table
      if (batch > 0 || bias) w.mq = mq_bytes<PL>(K, flags, true);
      if (bias) w.gs = align256(size_t(K) * PL::N * sizeof(float));
    }
  };
  if (flags & kFlagComplex) dispatch_complex(N, f);
  else dispatch_real(N, f);
  if (!have_saved) w.stash = align256(saved_floats(batch, N, K, flags) * 4);
  w.off_mq = 0;
  w.off_partial = w.off_mq + w.mq;
  w.off_gs = w.off_partial + w.partial;
  w.off_stash = w.off_gs + w.gs;
  w.total = w.off_stash + w.stash;
  return w;
}

size_t fwd_ws(int32_t N, int32_t K, uint32_t flags) {
  size_t b = 0;
  if (!(flags & kFlagComplex))
    dispatch_real(N, [&]<class PL>() { b = mq_bytes<PL>(K, flags, false); });
  return b;
}

// The quartet table into Mq, and the packed perm into P16 (if not null).
template <class PL>
int launch_real_mq(const float* D, const float* Bias, float4* Mq, int K, const char* tab, const int* perm,
                   int4* P16, hipStream_t s) {
  const long long n = (long long)K * PL::NSL * PL::T + (P16 != nullptr ? (long long)K * RealOps<PL>::NIW * PL::T : 0);
  hipLaunchKernelGGL(k_real_mq<PL>, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, D, Bias, Mq, K, tab, perm,
                     P16);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? ACDC_OK : hip_fail(e);
}

template <class PL, bool BIAS>
void launch_real_fwd_k(const RealArgs& a, hipStream_t s, bool remember) {
  using L = Launch<PL>;
  const Resident res = resident_workgroups(reinterpret_cast<const void*>(&k_real_fwd<PL, BIAS, false>),
                                           L::FWD_THREADS, remember);
  const int rpw = fwd_rows<PL>(a.batch, res.cus);
  const long long tiles = (a.batch + rpw - 1) / rpw;
  if constexpr (L::TW_LDS) {
    if (fwd_alone<PL>(a.batch, rpw, res.cus)) {
      hipLaunchKernelGGL((k_real_fwd<PL, BIAS, true>), dim3(unsigned(tiles)), dim3(kAloneThreads), 0, s, a, tiles,
                         rpw);
      return;
    }
  }
  hipLaunchKernelGGL((k_real_fwd<PL, BIAS, false>), dim3(unsigned(persistent_grid(res.n, tiles))),
                     dim3(L::FWD_THREADS), 0, s, a, tiles, rpw);
}

template <class PL>
int launch_real_fwd(const RealArgs& a, hipStream_t s, bool remember = true) {
  ProfScope prof(0, s);
  if (a.flags & kFlagBias) launch_real_fwd_k<PL, true>(a, s, remember);
  else launch_real_fwd_k<PL, false>(a, s, remember);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? ACDC_OK : hip_fail(e);
}

template <class PL>
int launch_cplx_fwd(const CplxArgs& a, hipStream_t s) {
  ProfScope prof(0, s);
  hipLaunchKernelGGL(k_cplx_fwd<PL>, dim3(unsigned(fwd_blocks<PL>(a.batch))), dim3(Launch<PL>::FWD_THREADS), 0,
                     s, a);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? ACDC_OK : hip_fail(e);
}

// ------------------------------------------------------ multi-pass path

struct MpTabs {
  const float2 *tw1 = nullptr, *tw2 = nullptr;
  QuartetTabs q{};
  const char *seg_f = nullptr, *seg = nullptr;  // the segment plans' tables: forward launches, others
};
std::map<std::pair<int, int>, void*> g_mp_tables;  // (device, N) -> device table

// The device copy of a host-built table, made on first use.
template <class Key, class Build>
int device_table(std::map<Key, void*>& tables, const Key& key, Build&& build, void** out) {
  std::lock_guard<std::mutex> lock(g_mu);
  auto it = tables.find(key);
  if (it == tables.end()) {
    std::vector<unsigned char> host;
    if (!build(host)) return ACDC_ERR_UNSUPPORTED;
    void* d = nullptr;
    hipError_t e = hipMalloc(&d, host.size());
    if (e != hipSuccess) return hip_fail(e);
    e = hipMemcpy(d, host.data(), host.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
      (void)hipFree(d);
      return hip_fail(e);
    }
    it = tables.emplace(key, d).first;
  }
  *out = it->second;
  return ACDC_OK;
}

int get_mp_tables(int N, MpTabs* out) {
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  const mp::Geo g = mp::geo(N);
  void *seg[2] = {}, *d = nullptr;
  int rc = ACDC_OK;
  for (int fwd = 0; fwd < 2; ++fwd) {
    // third key values 2 and 3: segment plans (0 real, 1 complex rows)
    rc = device_table(g_tables, std::make_tuple(dev, g.L, 2 + fwd),
                      [&](std::vector<unsigned char>& h) { return mp::build_seg_table(g.L, fwd != 0, h); }, &seg[fwd]);
    if (rc != ACDC_OK) return rc;
  }
  rc = device_table(g_mp_tables, std::make_pair(dev, N),
                    [&](std::vector<unsigned char>& h) { return build_mp_tables(N, g.R1, g.R2, g.L, h); }, &d);
  if (rc != ACDC_OK) return rc;
  const char* base = static_cast<const char*>(d);
  const MpTableLayout l = mp_table_layout(N, g.R1, g.R2, g.L);
  out->seg = static_cast<const char*>(seg[0]);
  out->seg_f = static_cast<const char*>(seg[1]);
  out->tw1 = reinterpret_cast<const float2*>(base + l.tw1);
  out->tw2 = reinterpret_cast<const float2*>(base + l.tw2);
  const double qb = 1.0 / (2.0 * std::sqrt(double(N)));
  out->q = QuartetTabs{reinterpret_cast<const float4*>(base + l.mk0), reinterpret_cast<const float4*>(base + l.mk1),
                       reinterpret_cast<const int4*>(base + l.qidx),
                       float(0.9238795325112867561 * qb), float(0.3826834323650897717 * qb)};
  return ACDC_OK;
}

// Floats per row element (1, or 2 for complex rows), and the geometry of
// rows of N elements.
int mp_ew(uint32_t flags) { return (flags & kFlagComplex) ? 2 : 1; }
mp::Geo mp_geo(int32_t N, uint32_t flags) { return mp::geo((long long)N * mp_ew(flags)); }

// Bytes of the layers' coefficients: the quartet tables (real), d / N in
// storage order (complex).
size_t mp_coef_bytes(long long N, int K, uint32_t flags) {
  return align256((flags & kFlagComplex) ? size_t(K) * N * sizeof(float2)
                                         : size_t(K) * size_t(N / 4) * kMqRows * sizeof(float4));
}
size_t mp_rows_bytes(int64_t batch, long long row_floats) {
  return align256(size_t(batch) * size_t(row_floats) * sizeof(float));
}

// Permutation tables: all K layers' built at once (four launches per call)
// when they take at most 256 MB, else one layer's, rebuilt per layer.
int mp_perm_layers(const mp::Geo& g, int K, int ew) {
  const size_t per = mp::perm_table_ints(g, ew) * sizeof(int);
  return per * size_t(K) <= (size_t(256) << 20) ? K : 1;
}
size_t mp_perm_bytes(const mp::Geo& g, int K, uint32_t flags) {
  if (!(flags & kFlagPerm)) return 0;
  const int ew = mp_ew(flags);
  return align256(mp::perm_table_ints(g, ew) * sizeof(int) * size_t(mp_perm_layers(g, K, ew)));
}

// The permutation tables of one call.
struct MpPerm {
  const int32_t* perm;
  mp::Geo g;
  int ew, K;
  mp::PermTabs base;
  bool all;  // every layer's tables are built
  MpPerm(const int32_t* p, const mp::Geo& geo, int K_, uint32_t flags, char* ws)
      : perm(p), g(geo), ew(mp_ew(flags)), K(K_), all(mp_perm_layers(geo, K_, mp_ew(flags)) == K_) {
    base = mp::perm_tables_at(reinterpret_cast<int*>(ws), g, ew);
  }
  hipError_t prebuild(hipStream_t s) const { return all ? mp::perm_build(perm, g, ew, K, base, s) : hipSuccess; }
  // Layer k's tables.  Not all built: they take the one place there is, so
  // the previous layer's have been used by then.
  hipError_t layer(int k, mp::PermTabs* out, hipStream_t s) const {
    if (all) {
      *out = mp::perm_layer(base, k);
      return hipSuccess;
    }
    *out = base;
    const long long N = 2 * g.M / ew;
    return mp::perm_build(perm + k * N, g, ew, 1, base, s);
  }
};

// Forward workspace: the layers' coefficients, the spectra, and with PERM
// the rows between the two halves of a permutation and the tables.
struct MpFwdWs {
  size_t coef = 0, z = 0, tmp = 0, ptab = 0, total = 0;
};
MpFwdWs mp_fwd_ws(int64_t batch, int32_t N, int32_t K, uint32_t flags) {
  MpFwdWs w;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += align256(bytes);
    return o;
  };
  const mp::Geo g = mp_geo(N, flags);
  const bool perm_on = (flags & kFlagPerm) != 0;
  const size_t rows = mp_rows_bytes(batch, 2 * g.M);
  w.coef = take(mp_coef_bytes(N, K, flags));
  w.z = take(rows);
  w.tmp = take(perm_on ? rows : 0);
  w.ptab = take(mp_perm_bytes(g, K, flags));
  w.total = off;
  return w;
}

// Backward workspace: the coefficients, the h and g spectra (contiguous:
// the second-level passes take both), the rows between the halves of a
// permutation, the row-block sums, with a bias every layer's batch sum of g's
// spectra and their block sums, the recompute stash and the permutation tables.
struct MpBwdWs {
  size_t coef = 0, zhg = 0, tmp = 0, part = 0, zsum = 0, partB = 0, stash = 0, ptab = 0, total = 0;
};
MpBwdWs mp_bwd_ws(int64_t batch, int32_t N, int32_t K, uint32_t flags, bool have_saved) {
  MpBwdWs w;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += align256(bytes);
    return o;
  };
  const mp::Geo g = mp_geo(N, flags);
  const bool perm_on = (flags & kFlagPerm) != 0, bias = (flags & kFlagBias) != 0;
  const size_t rowb = size_t(2 * g.M) * sizeof(float), rows = size_t(batch) * rowb;
  w.coef = take(mp_coef_bytes(N, K, flags));
  w.zhg = take(2 * rows);
  w.tmp = take(perm_on ? rows : 0);
  auto blocks = [&](int rb) { return size_t((batch + rb - 1) / rb); };
  w.part = take(size_t(mp::max_blocks(batch, g, mp_ew(flags))) * rowb);
  w.zsum = take(bias ? size_t(K) * rowb : 0);
  w.partB = take(bias ? blocks(mp::kMaxRows) * rowb : 0);
  w.stash = take(have_saved ? 0 : saved_floats(batch, N, K, flags) * sizeof(float));
  w.ptab = take(mp_perm_bytes(g, K, flags));
  w.total = off;
  return w;
}

#define MP_TRY(call)                          \
  do {                                        \
    const hipError_t e_ = (call);             \
    if (e_ != hipSuccess) return hip_fail(e_); \
  } while (0)

// Stash slot of layer input u_k (the fused path's layout): k - 1, or K - 1
// for u_0 with PERM.
float* mp_slot(float* saved, int k, int K, long long batch, long long row_floats, bool perm_on) {
  if (saved == nullptr) return nullptr;
  if (k > 0) return saved + (long long)(k - 1) * batch * row_floats;
  return perm_on ? saved + (long long)(K - 1) * batch * row_floats : nullptr;
}

// One multi-pass call: geometry, constants, workspace.  The steps are those
// of the fused rows; real and complex layers differ inside the launches.
struct MpCall {
  mp::Geo g;
  MpTabs t;
  bool cplx, perm_on, relu, bias;
  long long B, N, W;  // rows, elements and floats per row
  int K;
  float2* coef;  // quartet tables, or d / N
  hipStream_t s;

  const float4* mq(int k) const { return reinterpret_cast<const float4*>(coef) + (long long)k * (N / 4) * kMqRows; }
  hipError_t coefs(const float* D, const float* Bias) const {
    return cplx ? mp::dn(reinterpret_cast<const float2*>(D), coef, K, g, s)
                : mp::mq(D, Bias, reinterpret_cast<float4*>(coef), K, g, t.q, s);
  }
  hipError_t cols(mp::Src a, mp::Sink b, const mp::Cols& c) const { return mp::cols(a, b, cplx, c, B, g, t.tw1, s); }
  // the segment launch of layer k, between the second-level passes
  hipError_t forward_middle(float2* Z, int k) const {
    hipError_t e = mp::dif2(Z, B, g, t.tw2, s);
    if (e != hipSuccess) return e;
    e = cplx ? mp::cseg_fwd(Z, coef + (long long)k * N, B, g, t.seg_f, s)
             : mp::seg_fwd(Z, mq(k), B, g, bias, t.seg_f, s);
    return e != hipSuccess ? e : mp::dit2(Z, B, g, t.tw2, s);
  }
};

// The K forward layers.  Without y (the backward's recompute) only the layer
// inputs are wanted: they end with u_{K-1}'s store.
int mp_forward_layers(const MpCall& m, const float* x, float* y, const float* A, const MpPerm& pm, float* saved,
                      float2* Z, float* tmp) {
  using mp::Sink;
  using mp::Src;
  mp::PermTabs tk;
  if (m.perm_on) {
    MP_TRY(pm.layer(0, &tk, m.s));
    mp::Cols c;
    c.src = x;
    c.dst = tmp;
    c.pt = &tk;
    MP_TRY(m.cols(Src::rows, Sink::send, c));
  }
  for (int k = 0; k < m.K; ++k) {
    const bool last = k == m.K - 1;
    if (m.perm_on || k == 0) {
      mp::Cols c;  // u_k, its stash, * a, the first DIF pass
      c.src = m.perm_on ? tmp : x;
      c.pt = m.perm_on ? &tk : nullptr;
      c.Z = Z;
      c.a = A + (long long)k * m.W;
      c.stash = mp_slot(saved, k, m.K, m.B, m.W, m.perm_on);
      MP_TRY(m.cols(m.perm_on ? Src::gather : Src::rows, Sink::dif, c));
    }
    if (last && y == nullptr) break;
    MP_TRY(m.forward_middle(Z, k));
    mp::Cols c;
    c.Z = Z;
    c.relu = m.relu && !last ? 1 : 0;
    if (last) {
      c.dst = y;
      MP_TRY(m.cols(Src::dit, Sink::rows, c));
    } else if (m.perm_on) {
      MP_TRY(pm.layer(k + 1, &tk, m.s));
      c.dst = tmp;
      c.pt = &tk;
      MP_TRY(m.cols(Src::dit, Sink::send, c));
    } else {
      c.a = A + (long long)(k + 1) * m.W;
      c.stash = mp_slot(saved, k + 1, m.K, m.B, m.W, false);
      MP_TRY(m.cols(Src::dit, Sink::dif, c));
    }
  }
  return ACDC_OK;
}

int mp_call(MpCall* m, int64_t batch, int32_t N, int32_t K, uint32_t flags, void* coef, hipStream_t s) {
  m->g = mp_geo(N, flags);
  m->cplx = (flags & kFlagComplex) != 0;
  m->perm_on = (flags & kFlagPerm) != 0;
  m->relu = (flags & kFlagRelu) != 0;
  m->bias = (flags & kFlagBias) != 0;
  m->B = batch;
  m->N = N;
  m->W = 2 * m->g.M;
  m->K = K;
  m->coef = static_cast<float2*>(coef);
  m->s = s;
  return get_mp_tables(int(m->W), &m->t);
}

int mp_forward(const float* x, float* y, const float* A, const float* D, const float* bias, const int32_t* perm,
               int64_t batch, int32_t N, int32_t K, uint32_t flags, float* saved, void* workspace, hipStream_t s) {
  const MpFwdWs w = mp_fwd_ws(batch, N, K, flags);
  char* ws = static_cast<char*>(workspace);
  MpCall m;
  const int rc = mp_call(&m, batch, N, K, flags, ws + w.coef, s);
  if (rc != ACDC_OK) return rc;
  const MpPerm pm(perm, m.g, K, flags, ws + w.ptab);
  ProfScope prof(0, s);
  MP_TRY(m.coefs(D, bias));
  if (m.perm_on) MP_TRY(pm.prebuild(s));
  return mp_forward_layers(m, x, y, A, pm, saved, reinterpret_cast<float2*>(ws + w.z),
                           reinterpret_cast<float*>(ws + w.tmp));
}

// Backward, layer by layer from the last: Zg holds the first-level spectrum
// of g (dL/dv_k) at the top of layer k.  Zh = that of u_k * a_k; the segment
// launch sums the dL/dd images and leaves the inverse's segments in Zg; the
// column launch after it sums the dL/da images and takes g * a through the
// adjoint permutation to the next layer's Zg.  dL/db_k is the DCT-II of the
// batch sum of g, taken on its spectrum, for all layers at the end.
int mp_backward(const float* x, const float* grad_y, const float* A, const float* D, const float* bias,
                const int32_t* perm, const float* saved, float* grad_x, float* grad_A, float* grad_D,
                float* grad_bias, int64_t batch, int32_t N, int32_t K, uint32_t flags, bool have_saved,
                void* workspace, hipStream_t s) {
  using mp::Order;
  using mp::Sink;
  using mp::Src;
  const MpBwdWs w = mp_bwd_ws(batch, N, K, flags, have_saved);
  char* ws = static_cast<char*>(workspace);
  MpCall m;
  int rc = mp_call(&m, batch, N, K, flags, ws + w.coef, s);
  if (rc != ACDC_OK) return rc;
  const mp::Geo& g = m.g;
  float2* Zh = reinterpret_cast<float2*>(ws + w.zhg);
  float2* Zg = Zh + batch * g.M;  // the g spectra follow the h spectra
  float* tmp = reinterpret_cast<float*>(ws + w.tmp);
  float* part = reinterpret_cast<float*>(ws + w.part);
  float* zsum = reinterpret_cast<float*>(ws + w.zsum);
  float* partB = reinterpret_cast<float*>(ws + w.partB);
  float* stash = have_saved ? const_cast<float*>(saved) : reinterpret_cast<float*>(ws + w.stash);
  const MpPerm pm(perm, g, K, flags, ws + w.ptab);
  const bool acc = (flags & kFlagAccumulate) != 0;
  const Order order = m.cplx ? Order::spectrum : Order::quartets;
  ProfScope prof(1, s);
  if (batch == 0) {
    // no rows: zero (or unchanged, accumulating) parameter gradients
    for (int k = 0; k < K; ++k)
      for (float* o : {grad_A, grad_D, grad_bias})
        if (o != nullptr)
          MP_TRY(mp::colsum_parts(part, 0, m.W, o + k * m.W, Order::natural, g, nullptr, acc, s));
    return ACDC_OK;
  }
  MP_TRY(m.coefs(D, bias));
  if (m.perm_on) MP_TRY(pm.prebuild(s));
  if (!have_saved) {
    rc = mp_forward_layers(m, x, nullptr, A, pm, stash, Zh, tmp);
    if (rc != ACDC_OK) return rc;
  }
  const long long pseg = (batch + mp::seg_rows(batch, g, m.cplx) - 1) / mp::seg_rows(batch, g, m.cplx);
  const long long pcol = (batch + mp::col_rows(batch, g, mp_ew(flags)) - 1) / mp::col_rows(batch, g, mp_ew(flags));
  {
    mp::Cols c;
    c.src = grad_y;
    c.Z = Zg;
    MP_TRY(m.cols(Src::rows, Sink::dif, c));
  }
  for (int k = K - 1; k >= 0; --k) {
    float* gA = grad_A + (long long)k * m.W;
    float* gD = grad_D + (long long)k * m.W;
    const float* u = k > 0 || m.perm_on ? mp_slot(stash, k, K, batch, m.W, m.perm_on) : x;
    const float* ak = A + (long long)k * m.W;
    {
      mp::Cols c;
      c.src = u;
      c.Z = Zh;
      c.a = ak;
      MP_TRY(m.cols(Src::rows, Sink::dif, c));
    }
    MP_TRY(mp::dif2(Zh, 2 * batch, g, m.t.tw2, s));
    if (m.bias) MP_TRY(mp::colsum(reinterpret_cast<const float*>(Zg), batch, m.W, partB, zsum + k * m.W, s));
    if (m.cplx) MP_TRY(mp::cseg_bwd(Zh, Zg, m.coef + (long long)k * N, batch, g, part, m.t.seg, s));
    else MP_TRY(mp::seg_bwd(Zh, Zg, m.mq(k), batch, g, part, m.t.seg, s));
    MP_TRY(mp::colsum_parts(part, pseg, m.W, gD, order, g, &m.t.q, acc, s));
    MP_TRY(mp::dit2(Zg, batch, g, m.t.tw2, s));
    mp::Cols c;
    c.Z = Zg;
    c.u = u;
    c.a = ak;
    c.part = part;
    c.relu = m.relu && k > 0 ? 1 : 0;
    mp::PermTabs tk;
    if (m.perm_on) {
      MP_TRY(pm.layer(k, &tk, s));
      c.dst = tmp;
      c.pt = &tk;
      MP_TRY(m.cols(Src::dit, Sink::ret, c));
    } else if (k == 0) {
      c.dst = grad_x;
      MP_TRY(m.cols(Src::dit, Sink::rows, c));
    } else {
      MP_TRY(m.cols(Src::dit, Sink::dif, c));
    }
    MP_TRY(mp::colsum_parts(part, pcol, m.W, gA, Order::natural, g, nullptr, acc, s));
    if (m.perm_on) {
      mp::Cols d;
      d.src = tmp;
      d.dst = grad_x;
      d.Z = Zg;
      d.pt = &tk;
      MP_TRY(m.cols(Src::scatter, k == 0 ? Sink::rows : Sink::dif, d));
    }
  }
  if (m.bias) MP_TRY(mp::seg_dct(reinterpret_cast<const float2*>(zsum), m.mq(0), K, g, grad_bias, acc, m.t.seg, s));
  return ACDC_OK;
}

// The fused forward's launches (per-layer quartet coefficients into
// `workspace`, then the cascade).  `remember` false: cache nothing on the host.
int fused_forward(const float* x, float* y, const float* A, const float* D, const float* bias, const int32_t* perm,
                  int64_t batch, int32_t N, int32_t K, uint32_t flags, float* saved, void* workspace,
                  const char* tab, hipStream_t s, bool remember) {
  int rc = ACDC_ERR_UNSUPPORTED;
  if (flags & kFlagComplex) {
    dispatch_complex(N, [&]<class PL>() {
      CplxArgs a{x, y, A, D, perm, saved, nullptr, nullptr, nullptr, tab, batch, K, flags};
      rc = launch_cplx_fwd<PL>(a, s);
    });
  } else {
    dispatch_real(N, [&]<class PL>() {
      float4* Mq = static_cast<float4*>(workspace);
      rc = launch_real_mq<PL>(D, bias, Mq, K, tab, perm, nullptr, s);
      if (rc != ACDC_OK) return;
      RealArgs a{x, y, A, Mq, perm, saved, nullptr, nullptr, nullptr, tab, batch, K, flags};
      rc = launch_real_fwd<PL>(a, s, remember);
    });
  }
  return rc;
}

}  // namespace
}  // namespace acdc

using namespace acdc;

extern "C" int acdc_supported(int32_t N, uint32_t flags) {
  if (flags & ~kAllFlags) return 0;
  if (!flags_supported(flags)) return 0;
  return supported(N, flags) ? 1 : 0;
}

extern "C" int acdc_prepare(int32_t N, uint32_t flags) {
  if (!acdc_supported(N, flags)) return ACDC_ERR_UNSUPPORTED;
  int rc = scratch_setup();
  if (rc != ACDC_OK) return rc;
  if (use_multipass(N, flags)) {
    MpTabs t;
    return get_mp_tables((flags & kFlagComplex) ? 2 * N : N, &t);
  }
  const char* tab = nullptr;
  rc = get_table(N, (flags & kFlagComplex) != 0, &tab);
  if (rc != ACDC_OK || (flags & kFlagComplex)) return rc;
  // cache the persistent grids, so that later calls look them up
  dispatch_real(N, [&]<class PL>() {
    (void)resident_workgroups(reinterpret_cast<const void*>(&k_real_fwd<PL, false, false>), Launch<PL>::FWD_THREADS);
    (void)resident_workgroups(reinterpret_cast<const void*>(&k_real_fwd<PL, true, false>), Launch<PL>::FWD_THREADS);
    if constexpr (Launch<PL>::BWD_ACC)
      (void)resident_workgroups(reinterpret_cast<const void*>(&k_real_bwd<PL, false, Launch<PL>::BWD_ROWS>),
                                Launch<PL>::BWD_THREADS);
  });
  return ACDC_OK;
}

extern "C" size_t acdc_saved_bytes(int64_t batch, int32_t N, int32_t K, uint32_t flags) {
  if (check_common(batch, N, K, flags) != ACDC_OK) return 0;
  return saved_floats(batch, N, K, flags) * sizeof(float);
}

extern "C" size_t acdc_forward_workspace_size(int64_t batch, int32_t N, int32_t K, uint32_t flags) {
  if (check_common(batch, N, K, flags) != ACDC_OK) return 0;
  if (use_multipass(N, flags)) return mp_fwd_ws(batch, N, K, flags).total;
  return fwd_ws(N, K, flags);
}

extern "C" size_t acdc_backward_workspace_size(int64_t batch, int32_t N, int32_t K, uint32_t flags,
                                                int have_saved) {
  if (check_common(batch, N, K, flags) != ACDC_OK) return 0;
  const bool hs = have_saved != 0 || saved_layers(K, flags) == 0;
  if (use_multipass(N, flags)) return mp_bwd_ws(batch, N, K, flags, hs).total;
  return bwd_layout(batch, N, K, flags, hs).total;
}

extern "C" int acdc_forward(const float* x, float* y, const float* A, const float* D, const float* bias,
                            const int32_t* perm, int64_t batch, int32_t N, int32_t K, uint32_t flags, float* saved,
                            size_t saved_bytes, void* workspace, size_t workspace_bytes, acdc_stream_t stream) {
  int rc = check_common(batch, N, K, flags);
  if (rc != ACDC_OK) return rc;
  if (saved != nullptr && saved_bytes < saved_floats(batch, N, K, flags) * sizeof(float)) return ACDC_ERR_WORKSPACE;
  const bool perm_on = (flags & kFlagPerm) != 0;
  const bool bias_on = (flags & kFlagBias) != 0;
  if (batch == 0) return ACDC_OK;
  rc = check_ptrs({x, y, A, D}, {perm_on ? (const void*)perm : nullptr, bias_on ? (const void*)bias : nullptr,
                                 saved, workspace});
  if (rc != ACDC_OK) return rc;
  if ((perm_on && perm == nullptr) || (bias_on && bias == nullptr)) return ACDC_ERR_INVALID_ARG;
  if (!bias_on) bias = nullptr;
  if (!distinct({y, saved}, {x, y, A, D, bias, perm, saved, workspace})) return ACDC_ERR_INVALID_ARG;
  const bool multipass = use_multipass(N, flags);
  const size_t need = multipass ? mp_fwd_ws(batch, N, K, flags).total : fwd_ws(N, K, flags);
  if (need > 0 && (workspace == nullptr || workspace_bytes < need)) return ACDC_ERR_WORKSPACE;
  if (multipass)
    return mp_forward(x, y, A, D, bias, perm, batch, N, K, flags, saved, workspace,
                      reinterpret_cast<hipStream_t>(stream));
  const bool cplx = (flags & kFlagComplex) != 0;
  const char* tab = nullptr;
  rc = get_table(N, cplx, &tab);
  if (rc != ACDC_OK) return rc;
  return fused_forward(x, y, A, D, bias, perm, batch, N, K, flags, saved, workspace, tab,
                       reinterpret_cast<hipStream_t>(stream), true);
}

extern "C" int acdc_forward_noalloc(const float* x, float* y, const float* A, const float* D, const float* bias,
                                    const int32_t* perm, int64_t batch, int32_t N, int32_t K, uint32_t flags,
                                    float* saved, size_t saved_bytes, acdc_stream_t stream) {
  int rc = check_common(batch, N, K, flags);
  if (rc != ACDC_OK) return rc;
  if (use_multipass(N, flags)) return ACDC_ERR_UNSUPPORTED;  // its workspace grows with the batch
  if (saved != nullptr && saved_bytes < saved_floats(batch, N, K, flags) * sizeof(float)) return ACDC_ERR_WORKSPACE;
  const size_t need = fwd_ws(N, K, flags);
  if (need > kNoAllocScratchBytes) return ACDC_ERR_WORKSPACE;
  const bool perm_on = (flags & kFlagPerm) != 0;
  const bool bias_on = (flags & kFlagBias) != 0;
  if (batch == 0) return ACDC_OK;
  rc = check_ptrs({x, y, A, D}, {perm_on ? (const void*)perm : nullptr, bias_on ? (const void*)bias : nullptr, saved});
  if (rc != ACDC_OK) return rc;
  if ((perm_on && perm == nullptr) || (bias_on && bias == nullptr)) return ACDC_ERR_INVALID_ARG;
  if (!bias_on) bias = nullptr;
  if (!distinct({y, saved}, {x, y, A, D, bias, perm, saved})) return ACDC_ERR_INVALID_ARG;
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  if (dev < 0 || dev >= kMaxDevices) return ACDC_ERR_UNSUPPORTED;
  const bool cplx = (flags & kFlagComplex) != 0;
  const char* tab = find_table(dev, N, cplx);
  void* ws = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_mu);
    ws = g_scratch_ptr[dev];
  }
  if (tab == nullptr || ws == nullptr) return ACDC_ERR_NOT_PREPARED;
  return fused_forward(x, y, A, D, bias, perm, batch, N, K, flags, saved, ws, tab,
                       reinterpret_cast<hipStream_t>(stream), false);
}

extern "C" int acdc_backward(const float* x, const float* grad_y, const float* A, const float* D,
                             const float* bias, const int32_t* perm, const float* saved, size_t saved_bytes,
                             float* grad_x, float* grad_A, float* grad_D, float* grad_bias, int64_t batch,
                             int32_t N, int32_t K, uint32_t flags, void* workspace, size_t workspace_bytes,
                             acdc_stream_t stream) {
  int rc = check_common(batch, N, K, flags);
  if (rc != ACDC_OK) return rc;
  if (saved != nullptr && saved_bytes < saved_floats(batch, N, K, flags) * sizeof(float)) return ACDC_ERR_WORKSPACE;
  const bool perm_on = (flags & kFlagPerm) != 0;
  const bool bias_on = (flags & kFlagBias) != 0;
  const int accumulate = (flags & kFlagAccumulate) != 0 ? 1 : 0;
  if (!bias_on) {
    bias = nullptr;
    grad_bias = nullptr;
  }
  rc = check_ptrs({A, D, grad_A, grad_D}, {perm_on ? (const void*)perm : nullptr, bias, grad_bias, saved, workspace});
  if (rc != ACDC_OK) return rc;
  if (bias_on && (bias == nullptr || grad_bias == nullptr)) return ACDC_ERR_INVALID_ARG;
  if (batch > 0) {
    rc = check_ptrs({x, grad_y, grad_x}, {});
    if (rc != ACDC_OK) return rc;
    if (perm_on && perm == nullptr) return ACDC_ERR_INVALID_ARG;
  }
  if (!distinct({grad_x, grad_A, grad_D, grad_bias},
                {x, grad_y, A, D, bias, perm, saved, grad_x, grad_A, grad_D, grad_bias, workspace}))
    return ACDC_ERR_INVALID_ARG;
  // nothing to recompute when no layer input needs storing (K == 1 without PERM)
  const bool have_saved = saved != nullptr || saved_layers(K, flags) == 0;
  if (use_multipass(N, flags)) {
    const size_t need = mp_bwd_ws(batch, N, K, flags, have_saved).total;
    if (workspace == nullptr || workspace_bytes < need) return ACDC_ERR_WORKSPACE;
    return mp_backward(x, grad_y, A, D, bias, perm, saved, grad_x, grad_A, grad_D, grad_bias, batch, N, K, flags,
                       have_saved, workspace, reinterpret_cast<hipStream_t>(stream));
  }
  const WsLayout w = bwd_layout(batch, N, K, flags, have_saved);
  if (w.total > 0 && (workspace == nullptr || workspace_bytes < w.total)) return ACDC_ERR_WORKSPACE;
  const bool cplx = (flags & kFlagComplex) != 0;
  const char* tab = nullptr;
  rc = get_table(N, cplx, &tab);
  if (rc != ACDC_OK) return rc;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  float* partial = reinterpret_cast<float*>(ws + w.off_partial);
  float* stash = have_saved ? const_cast<float*>(saved) : reinterpret_cast<float*>(ws + w.off_stash);
  if (cplx) {
    dispatch_complex(N, [&]<class PL>() {
      using L = Launch<PL>;
      const long long tiles = bwd_tiles<PL>(batch);
      if (batch > 0) {
        if (!have_saved) {
          CplxArgs f{x, nullptr, A, D, perm, stash, nullptr, nullptr, nullptr, tab, batch, K, flags};
          rc = launch_cplx_fwd<PL>(f, s);
          if (rc != ACDC_OK) return;
        }
        CplxArgs a{x, nullptr, A, D, perm, stash, grad_y, grad_x, partial, tab, batch, K, flags};
        hipError_t e;
        {
          ProfScope prof(1, s);
          with_bwd_rows<PL>(batch, [&]<int ROWS>() {
            hipLaunchKernelGGL((k_cplx_bwd<PL, ROWS>), dim3(unsigned(tiles)), dim3(ROWS * PL::T), 0, s, a);
          });
          e = hipGetLastError();
        }
        if (e != hipSuccess) {
          rc = hip_fail(e);
          return;
        }
      }
      const long long n = (long long)K * partial_entries4<PL>();
      hipError_t e;
      {
        ProfScope prof(2, s);
        auto reduce = [&]<int PH>() {
          constexpr int E = kRedThreads / PH;
          hipLaunchKernelGGL((k_cplx_reduce<PL, PH>), dim3(unsigned((n + E - 1) / E)), dim3(kRedThreads), 0, s,
                             partial, tiles, K, grad_A, grad_D, accumulate);
        };
        if (red_phases(n) == 8) reduce.template operator()<8>();
        else reduce.template operator()<4>();
        e = hipGetLastError();
      }
      rc = e == hipSuccess ? ACDC_OK : hip_fail(e);
    });
  } else {
    dispatch_real(N, [&]<class PL>() {
      using L = Launch<PL>;
      const long long tiles = bwd_tiles<PL>(batch);
      // partial slots: one per tile, or one per resident workgroup of the
      // persistent (accumulating) unbiased backward
      const long long slots =
          (L::BWD_ACC && !bias_on && bwd_rows<PL>(batch) == L::BWD_ROWS)
              ? persistent_grid(resident_workgroups(reinterpret_cast<const void*>(&k_real_bwd<PL, false, L::BWD_ROWS>),
                                                    L::BWD_THREADS)
                                    .n,
                                tiles)
              : tiles;
      float4* Mq = reinterpret_cast<float4*>(ws + w.off_mq);
      int4* P16 = batch > 0 ? perm16_of<PL>(Mq, K, flags) : nullptr;
      float* gS = bias_on ? reinterpret_cast<float*>(ws + w.off_gs) : nullptr;
      if (batch > 0 || bias_on) {
        rc = launch_real_mq<PL>(D, bias, Mq, K, tab, perm, P16, s);
        if (rc != ACDC_OK) return;
      }
      if (batch > 0) {
        if (!have_saved) {
          RealArgs f{x, nullptr, A, Mq, perm, stash, nullptr, nullptr, nullptr, tab, batch, K, flags};
          rc = launch_real_fwd<PL>(f, s);
          if (rc != ACDC_OK) return;
        }
        RealArgs a{x, nullptr, A, Mq, perm, stash, grad_y, grad_x, partial, tab, batch, K, flags};
        a.perm16 = P16;
        hipError_t e;
        {
          ProfScope prof(1, s);
          with_bwd_rows<PL>(batch, [&]<int ROWS>() {
            const dim3 block(ROWS * PL::T);
            if (bias_on)
              hipLaunchKernelGGL((k_real_bwd<PL, true, ROWS>), dim3(unsigned(tiles)), block, 0, s, a, tiles);
            else
              hipLaunchKernelGGL((k_real_bwd<PL, false, ROWS>), dim3(unsigned(slots)), block, 0, s, a, tiles);
          });
          e = hipGetLastError();
        }
        if (e != hipSuccess) {
          rc = hip_fail(e);
          return;
        }
      }
      const long long n = (long long)K * partial_entries4<PL>(bias_on);
      hipError_t e;
      {
        ProfScope prof(2, s);
        auto reduce = [&]<int PH>() {
          constexpr int E = kRedThreads / PH;
          hipLaunchKernelGGL((k_real_reduce<PL, PH>), dim3(unsigned((n + E - 1) / E)), dim3(kRedThreads), 0, s,
                             partial, slots, K, grad_A, grad_D, gS, tab, bias_on ? 1 : 0, accumulate);
        };
        if (red_phases(n) == 8) reduce.template operator()<8>();
        else reduce.template operator()<4>();
        e = hipGetLastError();
        if (e == hipSuccess && bias_on) {
          hipLaunchKernelGGL(k_real_dct<PL>, dim3(unsigned(K)), dim3(PL::T), 0, s, gS, grad_bias, Mq, tab,
                             accumulate);
          e = hipGetLastError();
        }
      }
      rc = e == hipSuccess ? ACDC_OK : hip_fail(e);
    });
  }
  return rc;
}

extern "C" int acdc_profile_enable(int enable) {
  std::lock_guard<std::mutex> lock(g_prof_mu);
  g_prof_on = enable != 0;
  return ACDC_OK;
}

extern "C" int acdc_profile_read(double* ms, int64_t* launches) {
  if (ms == nullptr || launches == nullptr) return ACDC_ERR_INVALID_ARG;
  for (int i = 0; i < 3; ++i) {
    ms[i] = 0.0;
    launches[i] = 0;
  }
  std::lock_guard<std::mutex> lock(g_prof_mu);
  int rc = ACDC_OK;
  for (const ProfRec& r : g_prof_recs) {
    float t = 0.f;
    hipError_t e = hipEventSynchronize(r.b);
    if (e == hipSuccess) e = hipEventElapsedTime(&t, r.a, r.b);
    if (e != hipSuccess) rc = hip_fail(e);
    ms[r.kind] += t;
    launches[r.kind] += 1;
    g_prof_pool.push_back(r.a);
    g_prof_pool.push_back(r.b);
  }
  g_prof_recs.clear();
  return rc;
}

extern "C" const char* acdc_status_string(int status) {
  switch (status) {
    case ACDC_OK: return "ok";
    case ACDC_ERR_INVALID_ARG: return "invalid argument";
    case ACDC_ERR_UNSUPPORTED: return "unsupported width or flag combination";
    case ACDC_ERR_WORKSPACE: return "workspace missing or too small";
    case ACDC_ERR_HIP: return "HIP runtime error";
    case ACDC_ERR_NOT_PREPARED: return "width not prepared on this device (call acdc_prepare first)";
    default: return "unknown status";
  }
}

extern "C" int acdc_last_hip_error(void) { return g_last_hip; }

extern "C" int acdc_sync_timeouts(int64_t* count, int clear) {
  if (count == nullptr) return ACDC_ERR_INVALID_ARG;
  *count = 0;
  unsigned long long n = 0;
  hipError_t e = hipMemcpyFromSymbol(&n, HIP_SYMBOL(sync_timeouts), sizeof(n), 0, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return hip_fail(e);
  *count = (int64_t)n;
  if (clear != 0 && n != 0) {
    const unsigned long long zero = 0;
    e = hipMemcpyToSymbol(HIP_SYMBOL(sync_timeouts), &zero, sizeof(zero), 0, hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(e);
  }
  return ACDC_OK;
}
