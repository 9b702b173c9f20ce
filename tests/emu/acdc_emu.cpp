// CPU emulation of the HIP kernels' row bodies (test infrastructure).
//
// The same __host__ __device__ templates that the GPU kernels instantiate are
// run here with one OS thread per GPU thread and a std::barrier standing in
// for every LDS synchronisation, on host memory.  This checks the index
// algebra, the plan tables and the reduction order on the CPU; the GPU tests
// then check the real kernels.  Built by tests/emu/build_emu.py.
#include <barrier>
#include <cstring>
#include <cstdio>
#include <thread>
#include <vector>

#include "../../paper_1511_05946_amd/csrc/acdc_mp_geo.hpp"
#include "../../paper_1511_05946_amd/csrc/acdc_registry.hpp"

using namespace acdc;

namespace {

struct HostCtx {
  std::barrier<>* bar;
  int tid;
  float* xa;  // per-thread exchange slots of the cross-lane swaps
  float* xb;
  void sync_row() { bar->arrive_and_wait(); }
  void sync_all() { bar->arrive_and_wait(); }
  // The GPU's permlane16 / permlane32 swaps (acdc_devctx.hpp), through
  // shared slots between two barriers.
  template <int W>
  void swap(float& a, float& b) {
    xa[tid] = a;
    xb[tid] = b;
    bar->arrive_and_wait();
    const int lane = tid % 64, base = tid - lane;
    const bool upper = (lane / W) % 2 == 1;  // odd row (W = 16) or upper half (W = 32)
    const int partner = base + (upper ? lane - W : lane + W);
    const float na = upper ? xb[partner] : xa[tid];
    const float nb = upper ? xb[tid] : xa[partner];
    bar->arrive_and_wait();
    a = na;
    b = nb;
  }
  void swap16(float& a, float& b) { swap<16>(a, b); }
  void swap32(float& a, float& b) { swap<32>(a, b); }
};

template <class F>
void run_wg(int threads, F&& body) {
  std::barrier<> bar(threads);
  std::vector<float> xa(threads), xb(threads);
  std::vector<std::thread> th;
  th.reserve(threads);
  for (int tid = 0; tid < threads; ++tid)
    th.emplace_back([&, tid] {
      HostCtx ctx{&bar, tid, xa.data(), xb.data()};
      body(ctx, tid);
    });
  for (auto& x : th) x.join();
}

// The batch reduction in the GPU kernel's order: per entry, the phase sums
// in phase order.
template <class PL, class Store>
void reduce_all(const float* partial, long long ntiles, int K, long long PS4, Store&& store) {
  const long long n = (long long)K * PS4;
  auto run = [&]<int PH>() {
    for (long long i = 0; i < n; ++i) {
      float4 ph[PH];
      for (int g = 0; g < PH; ++g)
        ph[g] = tile_phase_sum4<PH>(reinterpret_cast<const float4*>(partial), ntiles, n, i, g);
      store(phases_total4<PH>(ph), int(i / PS4), int(i % PS4));
    }
  };
  if (red_phases(n) == 8) run.template operator()<8>();
  else run.template operator()<4>();
}

// Per-layer quartet coefficients in the kernel's [k][slot][kMqRows][T] layout.
template <class PL>
std::vector<float4> quartet_coefficients(const float* D, const float* B, int K, const std::vector<unsigned char>& tab) {
  constexpr int E = PL::NSL * PL::T;
  std::vector<float4> mq((size_t)K * E * kMqRows);
  for (int k = 0; k < K; ++k)
    for (int e = 0; e < E; ++e) {
      float4 row[kMqRows];
      real_mq_entry<PL>(D + (size_t)k * PL::N, B ? B + (size_t)k * PL::N : nullptr, (const char*)tab.data(), e, row);
      const int slot = e / PL::T, t = e % PL::T;
      for (int r = 0; r < kMqRows; ++r)
        mq[(size_t)k * E * kMqRows + (size_t)(slot * kMqRows + r) * PL::T + t] = row[r];
    }
  return mq;
}

// The packed perm the backward reads where the plan packs it (k_real_mq's
// extra threads on the GPU); empty otherwise.
template <class PL>
std::vector<int4> packed_perm(const int* perm, int K, unsigned flags) {
  using O = RealOps<PL>;
  std::vector<int4> p;
  if (!O::kPackedPerm || !(flags & kFlagPerm) || perm == nullptr) return p;
  p.resize((size_t)K * O::NIW * PL::T);
  for (int k = 0; k < K; ++k)
    for (int j = 0; j < O::NIW; ++j)
      for (int t = 0; t < PL::T; ++t)
        p[((size_t)k * O::NIW + j) * PL::T + t] = O::pack_perm_entry(perm + (size_t)k * PL::N, j, unsigned(t));
  return p;
}

// The launches of small batches on a device of 256 CUs (the forward's fewer
// rows per workgroup and its ALONE form, the backward's BWD_ROWS_FEW) where
// the batch has them; otherwise every batch runs as a large one does.
bool g_small_batch = false;

template <class PL, bool BIAS, bool ALONE>
void real_fwd_rows(const RealArgs& a, const std::vector<unsigned char>& tab, int rpw) {
  using L = Launch<PL>;
  const long long nwg = (a.batch + rpw - 1) / rpw;
  const int wg_rows = (ALONE ? kAloneThreads : L::FWD_THREADS) / PL::T;
  std::vector<float> lds((size_t)L::TW_FLOATS + (size_t)wg_rows * L::FWD_SLAB);
  float* twl = lds.data();
  float* rows = lds.data() + L::TW_FLOATS;
  if (L::TW_LDS) std::memcpy(twl, tab.data(), (size_t)PL::TW_FLOAT2 * 8);
  // the workgroup's waves past rpw rows have nothing to do
  for (long long wg = 0; wg < nwg; ++wg)
    run_wg(rpw * PL::T, [&](HostCtx& ctx, int tid) {
      const int r = tid / PL::T, t = tid % PL::T;
      float* slab = rows + (size_t)r * L::FWD_SLAB;
      if constexpr (L::TW_LDS)
        real_forward_row<PL, BIAS, ALONE>(ctx, a, unsigned(t), wg * rpw, unsigned(r), slab, LdsView::of(twl));
      else
        real_forward_row<PL, BIAS>(ctx, a, unsigned(t), wg * rpw, unsigned(r), slab, GView::of(tab.data()));
    });
}

template <class PL, bool BIAS>
void real_fwd_k(const RealArgs& a, const std::vector<unsigned char>& tab) {
  using L = Launch<PL>;
  const int rpw = g_small_batch ? fwd_rows<PL>(a.batch, int(kCus)) : L::FWD_ROWS;
  if constexpr (L::TW_LDS) {
    if (g_small_batch && fwd_alone<PL>(a.batch, rpw, int(kCus))) return real_fwd_rows<PL, BIAS, true>(a, tab, rpw);
  }
  real_fwd_rows<PL, BIAS, false>(a, tab, rpw);
}

template <class PL>
void real_fwd(const float* x, float* y, const float* A, const float* D, const float* B, const int* perm,
              long long batch, int K, unsigned flags, float* saved, const std::vector<unsigned char>& tab) {
  const std::vector<float4> mq = quartet_coefficients<PL>(D, (flags & kFlagBias) ? B : nullptr, K, tab);
  RealArgs a{x, y, A, mq.data(), perm, saved, nullptr, nullptr, nullptr, (const char*)tab.data(), batch, K, flags};
  if (flags & kFlagBias) real_fwd_k<PL, true>(a, tab);
  else real_fwd_k<PL, false>(a, tab);
}

// Persistent backward workgroups to emulate (0: one workgroup per tile, as
// the GPU runs plans without persistent accumulation or with at least as
// many resident workgroups as tiles).
long long g_bwd_slots = 0;

// f.template operator()<ROWS>() for the rows per backward workgroup.
template <class PL, class F>
void with_rows(long long batch, F&& f) {
  using L = Launch<PL>;
  if (g_small_batch && bwd_rows<PL>(batch) == L::BWD_ROWS_FEW) f.template operator()<L::BWD_ROWS_FEW>();
  else f.template operator()<L::BWD_ROWS>();
}

template <class PL, bool BIAS, int ROWS>
constexpr bool emu_acc() {
  return Launch<PL>::BWD_ACC && !BIAS && ROWS == Launch<PL>::BWD_ROWS;
}

// Partial slots of a backward over ntiles tiles.
template <class PL, bool BIAS, int ROWS>
long long bwd_slots(long long ntiles) {
  return (emu_acc<PL, BIAS, ROWS>() && g_bwd_slots > 0 && g_bwd_slots < ntiles) ? g_bwd_slots : ntiles;
}

template <class PL, bool BIAS, int ROWS>
void real_bwd_k(const RealArgs& a, long long ntiles, float* lds, const std::vector<unsigned char>& tab) {
  using L = Launch<PL>;
  const long long slots = bwd_slots<PL, BIAS, ROWS>(ntiles);
  // workgroup w runs tiles w, w + slots, ... in turn, as the persistent
  // kernel does, adding them into slot w (its LDS kept across its tiles)
  for (long long w = 0; w < slots; ++w)
    for (long long tile = w; tile < ntiles; tile += slots)
      run_wg(ROWS * PL::T, [&](HostCtx& ctx, int tid) {
        const int r = tid / PL::T, t = tid % PL::T;
        float* slab = lds + (size_t)r * L::BWD_SLAB;
        if constexpr (emu_acc<PL, BIAS, ROWS>())
          real_backward_row<PL, ROWS, BIAS, true>(ctx, a, unsigned(t), tile * ROWS, unsigned(r), tid, w, lds, slab,
                                                  GView::of(tab.data()),
                                                  tile == w ? nullptr : lds + L::BWD_LDS_FLOATS);
        else
          real_backward_row<PL, ROWS, BIAS>(ctx, a, unsigned(t), tile * ROWS, unsigned(r), tid, w, lds, slab,
                                            GView::of(tab.data()));
      });
}

template <class PL>
void real_bwd(const float* x, const float* gy, const float* A, const float* D, const float* B, const int* perm,
              const float* saved_in, float* gx, float* gA, float* gD, float* gB, long long batch, int K,
              unsigned flags, const std::vector<unsigned char>& tab) {
  using L = Launch<PL>;
  static_assert(!L::BWD_TW_LDS, "the emulation follows the global-twiddle backward");
  const bool bias = (flags & kFlagBias) != 0;
  const bool acc = (flags & kFlagAccumulate) != 0;
  std::vector<float> saved_buf;
  const float* saved = saved_in;
  const size_t layers = size_t(K - 1) + ((flags & kFlagPerm) ? 1 : 0);  // u_0 too with PERM
  if (saved == nullptr && layers > 0) {
    saved_buf.resize(layers * batch * PL::N);
    real_fwd<PL>(x, nullptr, A, D, B, perm, batch, K, flags, saved_buf.data(), tab);
    saved = saved_buf.data();
  }
  const std::vector<float4> mq = quartet_coefficients<PL>(D, bias ? B : nullptr, K, tab);
  long long ntiles = 0, slots = 0;
  with_rows<PL>(batch, [&]<int ROWS>() {
    ntiles = (batch + ROWS - 1) / ROWS;
    slots = bias ? bwd_slots<PL, true, ROWS>(ntiles) : bwd_slots<PL, false, ROWS>(ntiles);
  });
  const long long PS4 = partial_entries4<PL>(bias);
  std::vector<float> partial((size_t)slots * K * PS4 * 4);
  const std::vector<int4> p16 = packed_perm<PL>(perm, K, flags);
  RealArgs a{x, nullptr, A, mq.data(), perm, const_cast<float*>(saved), gy, gx, partial.data(),
             (const char*)tab.data(), batch, K, flags};
  a.perm16 = p16.empty() ? nullptr : p16.data();
  std::vector<float> lds((size_t)L::BWD_LDS_FLOATS + L::ACC_FLOATS);
  with_rows<PL>(batch, [&]<int ROWS>() {
    if (bias) real_bwd_k<PL, true, ROWS>(a, ntiles, lds.data(), tab);
    else real_bwd_k<PL, false, ROWS>(a, ntiles, lds.data(), tab);
  });
  std::vector<float> gS(bias ? (size_t)K * PL::N : 0);
  reduce_all<PL>(partial.data(), slots, K, PS4, [&](float4 s, int k, int e4) {
    real_reduce_store4<PL>(s, k, e4, gA, gD, gS.data(), (const char*)tab.data(), acc);
  });
  if (bias) {
    std::vector<float> lds1((size_t)L::FWD_SLAB);
    for (int k = 0; k < K; ++k)
      run_wg(PL::T, [&](HostCtx& ctx, int t) {
        real_dct_row<PL>(ctx, gS.data() + (size_t)k * PL::N, gB + (size_t)k * PL::N, mq.data(), acc, unsigned(t),
                         lds1.data(), GView::of(tab.data()), (const char*)tab.data());
      });
  }
}

template <class PL>
void cplx_fwd(const float* x, float* y, const float* A, const float* D, const int* perm, long long batch,
              int K, unsigned flags, float* saved, const std::vector<unsigned char>& tab) {
  using L = Launch<PL>;
  CplxArgs a{x, y, A, D, perm, saved, nullptr, nullptr, nullptr, (const char*)tab.data(), batch, K, flags};
  const long long nwg = (batch + L::FWD_ROWS - 1) / L::FWD_ROWS;
  std::vector<float> lds((size_t)L::FWD_ROWS * L::FWD_SLAB);
  for (long long wg = 0; wg < nwg; ++wg)
    run_wg(L::FWD_THREADS, [&](HostCtx& ctx, int tid) {
      const int r = tid / PL::T, t = tid % PL::T;
      cplx_forward_row<PL>(ctx, a, unsigned(t), wg * L::FWD_ROWS, unsigned(r), lds.data() + (size_t)r * L::FWD_SLAB);
    });
}

template <class PL>
void cplx_bwd(const float* x, const float* gy, const float* A, const float* D, const int* perm,
              const float* saved_in, float* gx, float* gA, float* gD, long long batch, int K, unsigned flags,
              const std::vector<unsigned char>& tab) {
  using L = Launch<PL>;
  std::vector<float> saved_buf;
  const float* saved = saved_in;
  const size_t layers = size_t(K - 1) + ((flags & kFlagPerm) ? 1 : 0);  // u_0 too with PERM
  if (saved == nullptr && layers > 0) {
    saved_buf.resize(layers * batch * 2 * PL::N);
    cplx_fwd<PL>(x, nullptr, A, D, perm, batch, K, flags, saved_buf.data(), tab);
    saved = saved_buf.data();
  }
  long long ntiles = 0;
  with_rows<PL>(batch, [&]<int ROWS>() { ntiles = (batch + ROWS - 1) / ROWS; });
  const long long PS = 4LL * PL::N;
  std::vector<float> partial((size_t)ntiles * K * PS);
  CplxArgs a{x, nullptr, A, D, perm, const_cast<float*>(saved), gy, gx, partial.data(),
             (const char*)tab.data(), batch, K, flags};
  std::vector<float> lds((size_t)L::BWD_ROWS * L::BWD_SLAB);
  with_rows<PL>(batch, [&]<int ROWS>() {
    for (long long wg = 0; wg < ntiles; ++wg)
      run_wg(ROWS * PL::T, [&](HostCtx& ctx, int tid) {
        const int r = tid / PL::T, t = tid % PL::T;
        cplx_backward_row<PL, ROWS>(ctx, a, unsigned(t), wg * ROWS, unsigned(r), tid, wg, lds.data(),
                                    lds.data() + (size_t)r * L::BWD_SLAB);
      });
  });
  reduce_all<PL>(partial.data(), ntiles, K, partial_entries4<PL>(), [&](float4 s, int k, int e4) {
    cplx_reduce_store4<PL>(s, k, e4, gA, gD, (flags & kFlagAccumulate) != 0);
  });
}

}  // namespace

extern "C" int acdc_emu_forward(const float* x, float* y, const float* A, const float* D, const float* B,
                                const int* perm, long long batch, int N, int K, unsigned flags, float* saved) {
  int rc = -2;
  if (flags & kFlagComplex) {
    dispatch_complex(N, [&]<class PL>() {
      std::vector<unsigned char> tab;
      build_complex_tables<PL>(tab);
      cplx_fwd<PL>(x, y, A, D, perm, batch, K, flags, saved, tab);
      rc = 0;
    });
  } else {
    dispatch_real(N, [&]<class PL>() {
      std::vector<unsigned char> tab;
      if (!build_real_tables<PL>(tab)) {
        rc = -5;
        return;
      }
      real_fwd<PL>(x, y, A, D, B, perm, batch, K, flags, saved, tab);
      rc = 0;
    });
  }
  return rc;
}

extern "C" int acdc_emu_backward(const float* x, const float* gy, const float* A, const float* D,
                                 const float* B, const int* perm, const float* saved, float* gx, float* gA,
                                 float* gD, float* gB, long long batch, int N, int K, unsigned flags) {
  int rc = -2;
  if (flags & kFlagComplex) {
    dispatch_complex(N, [&]<class PL>() {
      std::vector<unsigned char> tab;
      build_complex_tables<PL>(tab);
      cplx_bwd<PL>(x, gy, A, D, perm, saved, gx, gA, gD, batch, K, flags, tab);
      rc = 0;
    });
  } else {
    dispatch_real(N, [&]<class PL>() {
      std::vector<unsigned char> tab;
      if (!build_real_tables<PL>(tab)) {
        rc = -5;
        return;
      }
      real_bwd<PL>(x, gy, A, D, B, perm, saved, gx, gA, gD, gB, batch, K, flags, tab);
      rc = 0;
    });
  }
  return rc;
}

// Emulate `slots` persistent backward workgroups where the plan accumulates
// (0: one per tile).  Returns whether the unbiased backward of real rows of
// width N accumulates with the compiled launch settings.
extern "C" int acdc_emu_set_backward_slots(long long slots, int N) {
  g_bwd_slots = slots;
  int acc = 0;
  dispatch_real(N, [&]<class PL>() { acc = Launch<PL>::BWD_ACC ? 1 : 0; });
  return acc;
}

// Run the launches of small batches (see g_small_batch).
extern "C" void acdc_emu_set_small_batch(int on) { g_small_batch = on != 0; }

// Rules of the fused launches on 256 CUs: rows per backward workgroup, rows
// per forward workgroup, and whether the forward runs its ALONE form.
extern "C" int acdc_emu_rows(long long batch, int N, unsigned flags, int* out) {
  int rc = -2;
  auto f = [&]<class PL>() {
    out[0] = bwd_rows<PL>(batch);
    out[1] = Launch<PL>::FWD_ROWS;
    out[2] = 0;
    if constexpr (!PL::kComplex) {
      out[1] = fwd_rows<PL>(batch, int(kCus));
      out[2] = fwd_alone<PL>(batch, out[1], int(kCus)) ? 1 : 0;
    }
    rc = 0;
  };
  if (flags & kFlagComplex) dispatch_complex(N, f);
  else dispatch_real(N, f);
  return rc;
}

// The fixed-order batch reduction alone: out[e] (float4 e < n4) = the sum
// over ntiles tiles of partial[t][e], in the kernels' order (red_phases(n4)
// tile phases, grouped loads, phases added in order).  Returns the number of
// phases used.
extern "C" int acdc_emu_reduce4(const float* partial, long long ntiles, long long n4, float* out) {
  auto run = [&]<int PH>() {
    for (long long e = 0; e < n4; ++e) {
      float4 ph[PH];
      for (int g = 0; g < PH; ++g)
        ph[g] = tile_phase_sum4<PH>(reinterpret_cast<const float4*>(partial), ntiles, n4, e, g);
      reinterpret_cast<float4*>(out)[e] = phases_total4<PH>(ph);
    }
    return PH;
  };
  return red_phases(n4) == 8 ? run.template operator()<8>() : run.template operator()<4>();
}

// Geometry of the multi-pass rows of N elements (ew = 1 real, 2 complex).
// out: rows in turn, threads of a workgroup, workgroups, rows side by side of a
// column launch.
extern "C" void acdc_emu_mp_col_grid(long long batch, int N, int ew, int sums, long long* out) {
  const mp::ColGrid c = mp::col_grid(batch, mp::geo((long long)N * ew), ew, sums != 0);
  out[0] = c.rb;
  out[1] = c.threads;
  out[2] = c.groups;
  out[3] = c.rw;
}

// Quartets of a row's M-point FFT by pair and place: out[p][k2] = the quartet
// there, and back[e] = pair L + place of quartet e.  Returns L.
extern "C" int acdc_emu_mp_quartets(int N, int ew, long long* out, long long* back) {
  const mp::Geo g = mp::geo((long long)N * ew);
  for (int p = 0; p < g.R1 * g.R2 / 2; ++p)
    for (int k2 = 0; k2 < g.L; ++k2) out[(long long)p * g.L + k2] = mp::quartet_of(g, p, k2);
  for (long long e = 0; e < g.M / 2; ++e) {
    int p, k2;
    mp::quartet_place(g, e, p, k2);
    back[e] = (long long)p * g.L + k2;
  }
  return g.L;
}

// Column sets of a row of N elements: set and LDS place of every element
// (part_of), and the element at every local position of every set (elem_of).
// Returns the elements of a set.
extern "C" int acdc_emu_mp_sets(int N, int ew, long long* set, long long* place, long long* elem) {
  const mp::PermGeo p = mp::perm_geo(mp::geo((long long)N * ew), ew);
  for (long long i = 0; i < N; ++i) {
    int d, l;
    mp::part_of(p, i, d, l);
    set[i] = d;
    place[i] = l;
  }
  for (int d = 0; d < p.nC; ++d)
    for (int l = 0; l < (1 << p.lC); ++l) elem[((long long)d << p.lC) + l] = mp::elem_of(p, d, l);
  return 1 << p.lC;
}

// The M-point FFT of such a row: spectrum index of every storage position, the
// segments of every pair ([S/2][2]), and (R1, R2, L).
extern "C" void acdc_emu_mp_spectrum(int N, int ew, long long* spec, int* pairs, int* geo) {
  const mp::Geo g = mp::geo((long long)N * ew);
  for (long long q = 0; q < g.M; ++q) spec[q] = mp::spec_index(g, q);
  for (int p = 0; p < g.R1 * g.R2 / 2; ++p) mp::seg_pair(g, p, pairs[2 * p], pairs[2 * p + 1]);
  geo[0] = g.R1;
  geo[1] = g.R2;
  geo[2] = g.L;
}
