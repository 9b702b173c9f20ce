// Kernels of the multi-pass ACDC layers (declarations and the pass structure
// in acdc_multipass.hpp).
#include <hip/hip_runtime.h>

#include <type_traits>
#include <vector>

#include "acdc_devctx.hpp"
#include "acdc_multipass.hpp"

namespace acdc {
namespace mp {
namespace {

constexpr int kThreads = 256;

// Workgroups go to the 8 XCDs (each with its own L2) in turn: workgroup w
// runs on XCD w mod 8.  Elementwise grids are a multiple of 8 workgroups, and
// gindex() hands XCD x the x-th contiguous eighth of the grid.
constexpr int kXcds = 8;

dim3 grid_for(long long n) {
  long long blocks = (n + kThreads - 1) / kThreads;
  if (blocks > 65536) blocks = 65536;
  blocks = (blocks + kXcds - 1) / kXcds * kXcds;
  if (blocks < kXcds) blocks = kXcds;
  return dim3(unsigned(blocks));
}

__device__ __forceinline__ long long gstride() { return (long long)gridDim.x * blockDim.x; }
__device__ __forceinline__ long long gindex() {
  const unsigned per_xcd = gridDim.x / kXcds;
  const unsigned blk = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  return (long long)blk * blockDim.x + threadIdx.x;
}

// Makhoul packing by float4 chunks: chunk q of a row (floats 4q .. 4q+3)
// holds complex value m = q as (h.x, h.z) and m = M-1-q as (h.w, h.y).
__device__ __forceinline__ float2 chunk_even(float4 h) { return make_float2(h.x, h.z); }
__device__ __forceinline__ float2 chunk_odd(float4 h) { return make_float2(h.w, h.y); }
__device__ __forceinline__ float4 chunk_of(float2 even, float2 odd) { return make_float4(even.x, odd.y, even.y, odd.x); }
__device__ __forceinline__ float4 scale4(float4 h, float4 a) {
  return make_float4(h.x * a.x, h.y * a.y, h.z * a.z, h.w * a.w);
}
__device__ __forceinline__ float4 relu4(float4 h) { return make_float4(relu1(h.x), relu1(h.y), relu1(h.z), relu1(h.w)); }

// ------------------------------------------------------------ permutations

// Table build, a counting sort of the destinations by source set.  Step 1:
// per block of kThreads destinations (all of one set d), the count of each
// source set: cntS[blk][c].  Every step handles layer blockIdx.y (step 3: x).
__global__ __launch_bounds__(kThreads) void k_pt_count(const int* __restrict__ src, long long N, PermGeo pg,
                                                       int* __restrict__ cntS, long long stride) {
  __shared__ int h[kPermMaxChunks];
  src += blockIdx.y * N;
  cntS += blockIdx.y * stride;
  for (int c = threadIdx.x; c < pg.nC; c += kThreads) h[c] = 0;
  __syncthreads();
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  int c, ls;
  part_of(pg, src[elem_of(pg, int(idx >> pg.lC), int(idx & ((1 << pg.lC) - 1)))] & (N - 1), c, ls);
  atomicAdd(&h[c], 1);
  __syncthreads();
  for (int k = threadIdx.x; k < pg.nC; k += kThreads) cntS[(long long)blockIdx.x * pg.nC + k] = h[k];
}

// Step 2, one thread per (d, c): the running count over set d's blocks
// (bpre[blk][c], exclusive) and the total cnt[d][c].
__global__ __launch_bounds__(kThreads) void k_pt_blocks(const int* __restrict__ cntS, PermGeo pg,
                                                        int* __restrict__ bpre, int* __restrict__ cnt,
                                                        long long stride) {
  const int i = blockIdx.x * kThreads + threadIdx.x, nC = pg.nC;
  if (i >= nC * nC) return;
  cntS += blockIdx.y * stride;
  bpre += blockIdx.y * stride;
  cnt += blockIdx.y * stride;
  const int d = i / nC, c = i % nC, per = (1 << pg.lC) / kThreads;
  int run = 0;
  for (int j = 0; j < per; ++j) {
    const long long blk = (long long)d * per + j;
    bpre[blk * nC + c] = run;
    run += cntS[blk * nC + c];
  }
  cnt[i] = run;
}

// Step 3, one workgroup: start[d][c], where the entries bound for d begin in
// set c's list; lst[d][c], where those sourced from c begin in d's values of
// tmp; and delta[c][d] = d C + lst - start.
__global__ __launch_bounds__(kThreads) void k_pt_offsets(const int* __restrict__ cnt, PermGeo pg,
                                                         int* __restrict__ start, int* __restrict__ lst,
                                                         int* __restrict__ delta, long long stride) {
  const int nC = pg.nC;
  cnt += blockIdx.x * stride;
  start += blockIdx.x * stride;
  lst += blockIdx.x * stride;
  delta += blockIdx.x * stride;
  for (int d = threadIdx.x; d < nC; d += kThreads) {
    int run = 0;
    for (int c = 0; c < nC; ++c) {
      lst[d * nC + c] = run;
      run += cnt[d * nC + c];
    }
  }
  __syncthreads();
  for (int c = threadIdx.x; c < nC; c += kThreads) {
    int run = 0;
    for (int d = 0; d < nC; ++d) {
      start[d * nC + c] = run;
      delta[c * nC + d] = (d << pg.lC) + lst[d * nC + c] - run;
      run += cnt[d * nC + c];
    }
  }
}

// Step 4: every destination takes a place in its run (the order inside a
// block's share of a run is whatever the LDS counter hands out; the tables
// stay consistent, and the permuted values do not depend on it).
__global__ __launch_bounds__(kThreads) void k_pt_place(const int* __restrict__ src, long long N, PermGeo pg,
                                                       const int* __restrict__ bpre, const int* __restrict__ start,
                                                       const int* __restrict__ lst, unsigned* __restrict__ item,
                                                       unsigned short* __restrict__ loc, long long stride) {
  __shared__ int h[kPermMaxChunks];
  const long long ls0 = blockIdx.y * stride;
  const int nC = pg.nC, mask = (1 << pg.lC) - 1;
  src += blockIdx.y * N;
  bpre += ls0;
  start += ls0;
  lst += ls0;
  item += ls0;
  loc += 2 * ls0;
  for (int c = threadIdx.x; c < nC; c += kThreads) h[c] = 0;
  __syncthreads();
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  const int d = int(idx >> pg.lC);
  int c, ls;
  part_of(pg, src[elem_of(pg, d, int(idx & mask))] & (N - 1), c, ls);
  const int p = bpre[(long long)blockIdx.x * nC + c] + atomicAdd(&h[c], 1);
  loc[idx] = (unsigned short)((lst[d * nC + c] + p) & mask);
  item[((long long)c << pg.lC) + ((start[d * nC + c] + p) & mask)] = (unsigned(ls) << 8) | unsigned(d);
}

// The tables of rows of one set, in one launch: every destination comes from
// that set, so the list may be in the order of the destinations.  (The four
// steps above took 13 us a call: N = 16384, K = 4, one row, forward 141 us, 132 now.)
__global__ __launch_bounds__(kThreads) void k_pt_one(const int* __restrict__ src, long long N, PermGeo pg,
                                                     unsigned* __restrict__ item, unsigned short* __restrict__ loc,
                                                     int* __restrict__ delta, long long stride) {
  const long long ls0 = blockIdx.y * stride, idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  int c, ls;
  part_of(pg, src[blockIdx.y * N + elem_of(pg, 0, int(idx))] & (N - 1), c, ls);
  item[ls0 + idx] = unsigned(ls) << 8;
  loc[2 * ls0 + idx] = (unsigned short)idx;
  if (idx == 0) delta[ls0] = 0;
}

// A value the compiler takes as new each time: offsets built from it keep the
// loads of per-layer tables inside a loop over rows.  Hoisted out of it, the
// quartet coefficients of a thread alone would be 96 registers.
__device__ __forceinline__ unsigned fresh(unsigned v) {
  asm volatile("" : "+v"(v));
  return v;
}

// ----------------------------------------------------------------- columns

struct ColArgs {
  const float* src;
  float* dst;
  float2* Z;
  const float* a;
  float* stash;
  const float* u;
  float* part;
  const float2* tw;  // [R1-1][Q]: W_M^(n r) at [r-1][n]
  const unsigned* item;
  const unsigned short* loc;
  const int* delta;
  long long B, M;
  int rw, rb, relu;
  PermGeo pg;
};

// The entries i of one set's list that this thread takes, BATCH of them at a
// time: get(i) for all, then put(i, value).  A thread follows a table to HBM,
// so one load at a time would be bound by memory latency.
template <int THREADS, int BATCH, class T, class Get, class Put>
__device__ __forceinline__ void for_entries(int C, Get&& get, Put&& put) {
  if (C % (THREADS * BATCH) == 0) {
    for (int i0 = threadIdx.x; i0 < C; i0 += THREADS * BATCH) {
      T v[BATCH];
#pragma unroll
      for (int q = 0; q < BATCH; ++q) v[q] = get(i0 + q * THREADS);
#pragma unroll
      for (int q = 0; q < BATCH; ++q) put(i0 + q * THREADS, v[q]);
    }
  } else {
    for (int i = threadIdx.x; i < C; i += THREADS) put(i, get(i));
  }
}

// Entry of a set's list with what it refers to.
template <class E>
struct Entry {
  unsigned it;
  E v;
};

// What a column launch does between its source and its sink, and whether it
// needs the LDS chunk.
template <Src SRC, Sink SINK>
constexpr bool needs_lds() {
  return SRC == Src::gather || SRC == Src::scatter || SINK == Sink::send || SINK == Sink::ret;
}

// Row accesses go through views (one 32-bit lane offset, the part that is
// the same for all lanes in a scalar): written as 64-bit addresses per
// access, the addresses alone took the registers of a second workgroup per
// CU.  Fences bound what is in flight at once for the same reason.

// Real rows.  A thread holds CI column pairs, R float4 chunks each: ha[j]
// is chunk n + jQ, hb[j] chunk (Q-1-n) + jQ.
template <int R>
constexpr int col_waves() {
  return R <= 8 ? 4 : 2;
}

// NARROW: A.rw > 1 rows side by side, column col being row col / w's (a
// template of its own: the row arithmetic costs every entry of a list).
// N = 256, K = 4, 40000 rows, forward with permutations and ReLU, segment
// launches as at the time: 1665 us with a row a workgroup, 776 with 64.
template <int R, Src SRC, Sink SINK, bool BWD, bool NARROW>
__global__ __launch_bounds__(col_threads(R, 1))
__attribute__((amdgpu_waves_per_eu(col_waves<R>()))) void k_cols(ColArgs A) {
  constexpr int THREADS = col_threads(R, 1), H = R / 2;
  constexpr int CI = kPermChunk / 4 / (R * THREADS);
  constexpr int W = kPermChunk / 4 / R;  // LDS: chunk js of column col at js W + col
  constexpr unsigned kMask = kPermChunk - 1;
  static_assert(CI >= 1 && CI * THREADS == W, "a set's chunks over the threads");
  __shared__ float4 lds4[needs_lds<SRC, SINK>() ? kPermChunk / 4 : 1];
  __shared__ int dl[kPermMaxChunks];
  float* lds = reinterpret_cast<float*>(lds4);
  const PermGeo pg = A.pg;
  const int C = 1 << pg.lC, w = 1 << pg.lw;
  const long long M = A.M, N = 2 * M;
  const unsigned Q = 1u << pg.lQ;
  const int c = int(blockIdx.x % unsigned(pg.nC));
  const long long p = blockIdx.x / unsigned(pg.nC);
  if constexpr (SRC == Src::scatter || SINK == Sink::send) {
    for (int d = threadIdx.x; d < pg.nC; d += THREADS) dl[d] = A.delta[c * pg.nC + d];
    __syncthreads();
  }
  const unsigned* item = A.item + ((long long)c << pg.lC);
  const GView loc = GView::of(A.loc + ((long long)c << pg.lC)), tw = GView::of(A.tw), av = GView::of(A.a);
  const unsigned sq16 = 16u << pg.lQ, sq8 = 8u << pg.lQ;  // bytes of Q chunks, of Q spectrum values
  float4 ha[CI][H], hb[CI][H], sa[CI][H], sb[CI][H];
  if constexpr (BWD) {
#pragma unroll
    for (int ci = 0; ci < CI; ++ci)
#pragma unroll
      for (int j = 0; j < H; ++j) sa[ci][j] = sb[ci][j] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  // LDS place of entry i of the step's lists whose place in its own row's set
  // is ls: row i / C's columns start at column w i / C.  (For a malformed perm
  // ls is any value.)
  auto at_row = [&](unsigned ls, int i) {
    return (ls + (NARROW ? unsigned(i >> pg.lC) << (pg.lw + 2) : 0u)) & kMask;
  };
  int nr = 1;  // rows side by side in this step
  // f(ci, col, n, nb, o): this thread's column pairs, and the byte offset of
  // its row from the step's first one (the same in rows and spectra)
  auto pairs = [&](auto&& f) {
#pragma unroll
    for (int ci = 0; ci < CI; ++ci) {
      const int col = int(threadIdx.x) + ci * THREADS;
      const int row = NARROW ? col >> pg.lw : 0;
      if (NARROW ? row < nr : col < w) {
        const unsigned n = fresh((unsigned(c) << pg.lw) + unsigned(col - (row << pg.lw)));
        f(ci, col, n, Q - 1 - n, NARROW ? unsigned(row) << (pg.lC + 2) : 0u);
        ACDC_SCHED_FENCE();
      }
    }
  };
  const long long rw = NARROW ? A.rw : 1, b0 = p * A.rb * rw, b1 = b0 + A.rb * rw < A.B ? b0 + A.rb * rw : A.B;
  for (long long b = b0; b < b1; b += rw) {
    if constexpr (NARROW) nr = int(b1 - b < rw ? b1 - b : rw);
    const int total = NARROW ? nr << pg.lC : C;  // elements of this step's (rows of one) set
    const GView z = GView::of(A.Z + b * M);
    if constexpr (SRC == Src::rows) {
      const GView row = GView::of(A.src + b * N);
      pairs([&](int ci, int, unsigned n, unsigned nb, unsigned o) {
#pragma unroll
        for (int j = 0; j < H; ++j) {
          ha[ci][j] = row.ld4(n * 16u + o, j * sq16);
          hb[ci][j] = row.ld4(nb * 16u + o, j * sq16);
        }
      });
    } else if constexpr (SRC == Src::gather) {
      const float4* t4 = reinterpret_cast<const float4*>(A.src + b * N + ((long long)c << pg.lC));
      for_entries<THREADS, 8, float4>(
          total / 4, [&](int i) { return t4[i]; }, [&](int i, float4 v) { lds4[i] = v; });
      __syncthreads();
      pairs([&](int ci, int col, unsigned, unsigned, unsigned o) {
        const unsigned f = o / 4;  // the row's place in LDS
        auto at = [&](int js) {
          const int2 s = loc.ldi2(unsigned(NARROW ? col & (w - 1) : col) * 8u, unsigned(js << pg.lw) * 8u);
          return make_float4(lds[(unsigned(s.x) + f) & kMask], lds[((unsigned(s.x) >> 16) + f) & kMask],
                             lds[(unsigned(s.y) + f) & kMask], lds[((unsigned(s.y) >> 16) + f) & kMask]);
        };
#pragma unroll
        for (int j = 0; j < H; ++j) {
          ha[ci][j] = at(2 * j);
          hb[ci][j] = at(2 * j + 1);
        }
      });
      if (b + rw < b1) __syncthreads();
    } else if constexpr (SRC == Src::scatter) {
      const float* trow = A.src + b * N;
      const unsigned nm = unsigned(N - 1);
      for_entries<THREADS, 16, Entry<float>>(
          total,
          [&](int i) {
            const int r = NARROW ? i >> pg.lC : 0, e = i - (r << pg.lC);
            const unsigned it = item[e];
            return Entry<float>{it, trow[(unsigned(e + dl[it & 255]) & nm) + (unsigned(r) << pg.lC)]};
          },
          [&](int i, const Entry<float>& e) { lds[at_row(e.it >> 8, i)] = e.v; });
      __syncthreads();
      pairs([&](int ci, int col, unsigned, unsigned, unsigned) {
#pragma unroll
        for (int j = 0; j < H; ++j) {
          ha[ci][j] = lds4[(2 * j) * W + col];
          hb[ci][j] = lds4[(2 * j + 1) * W + col];
        }
      });
      if (b + rw < b1) __syncthreads();
    } else {
      pairs([&](int ci, int, unsigned n, unsigned nb, unsigned o) {
        float2 y[R], yb[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          y[r] = z.ld2(n * 8u + o, r * sq8);
          yb[r] = z.ld2(nb * 8u + o, r * sq8);
        }
#pragma unroll
        for (int r = 1; r < R; ++r) y[r] = cmulc(y[r], tw.ld2(n * 8u, (r - 1) * sq8));
        Dft<R, true>::run(y);
        if constexpr (R > 8) ACDC_SCHED_FENCE();
#pragma unroll
        for (int r = 1; r < R; ++r) yb[r] = cmulc(yb[r], tw.ld2(nb * 8u, (r - 1) * sq8));
        Dft<R, true>::run(yb);
#pragma unroll
        for (int j = 0; j < H; ++j) {
          ha[ci][j] = chunk_of(y[j], yb[R - 1 - j]);
          hb[ci][j] = chunk_of(yb[j], y[R - 1 - j]);
        }
      });
      if constexpr (!BWD) {
        if (A.relu) {
          pairs([&](int ci, int, unsigned, unsigned, unsigned) {
#pragma unroll
            for (int j = 0; j < H; ++j) {
              ha[ci][j] = relu4(ha[ci][j]);
              hb[ci][j] = relu4(hb[ci][j]);
            }
          });
        }
      }
    }
    if constexpr (BWD) {
      const GView uv = GView::of(A.u + b * N);
      // u = 0 exactly where the mask is off, so masking g first leaves u * g unchanged
      auto one = [&](float4& g, float4& s, float4 u, float4 a) {
        if (A.relu)
          g = make_float4(u.x > 0.f ? g.x : 0.f, u.y > 0.f ? g.y : 0.f, u.z > 0.f ? g.z : 0.f, u.w > 0.f ? g.w : 0.f);
        s = make_float4(s.x + u.x * g.x, s.y + u.y * g.y, s.z + u.z * g.z, s.w + u.w * g.w);
        g = scale4(g, a);
      };
      pairs([&](int ci, int, unsigned n, unsigned nb, unsigned) {
#pragma unroll
        for (int j = 0; j < H; ++j) one(ha[ci][j], sa[ci][j], uv.ld4(n * 16u, j * sq16), av.ld4(n * 16u, j * sq16));
        ACDC_SCHED_FENCE();
#pragma unroll
        for (int j = 0; j < H; ++j) one(hb[ci][j], sb[ci][j], uv.ld4(nb * 16u, j * sq16), av.ld4(nb * 16u, j * sq16));
      });
    }
    if constexpr (SINK == Sink::dif && !BWD) {
      if (A.stash != nullptr) {
        const GView st = GView::of(A.stash + b * N);
        pairs([&](int ci, int, unsigned n, unsigned nb, unsigned o) {
#pragma unroll
          for (int j = 0; j < H; ++j) {
            st.st4(ha[ci][j], n * 16u + o, j * sq16);
            st.st4(hb[ci][j], nb * 16u + o, j * sq16);
          }
        });
      }
      if (A.a != nullptr) {
        pairs([&](int ci, int, unsigned n, unsigned nb, unsigned) {
#pragma unroll
          for (int j = 0; j < H; ++j) {
            ha[ci][j] = scale4(ha[ci][j], av.ld4(n * 16u, j * sq16));
            hb[ci][j] = scale4(hb[ci][j], av.ld4(nb * 16u, j * sq16));
          }
        });
      }
    }
    if constexpr (SINK == Sink::rows) {
      const GView out = GView::of(A.dst + b * N);
      pairs([&](int ci, int, unsigned n, unsigned nb, unsigned o) {
#pragma unroll
        for (int j = 0; j < H; ++j) {
          out.st4(ha[ci][j], n * 16u + o, j * sq16);
          out.st4(hb[ci][j], nb * 16u + o, j * sq16);
        }
      });
    } else if constexpr (SINK == Sink::send) {
      pairs([&](int ci, int col, unsigned, unsigned, unsigned) {
#pragma unroll
        for (int j = 0; j < H; ++j) {
          lds4[(2 * j) * W + col] = ha[ci][j];
          lds4[(2 * j + 1) * W + col] = hb[ci][j];
        }
      });
      __syncthreads();
      float* trow = A.dst + b * N;
      const unsigned nm = unsigned(N - 1);
      for_entries<THREADS, 8, unsigned>(
          total, [&](int i) { return item[NARROW ? i & (C - 1) : i]; },
          [&](int i, unsigned it) {
            const int r = NARROW ? i >> pg.lC : 0, e = i - (r << pg.lC);
            trow[(unsigned(e + dl[it & 255]) & nm) + (unsigned(r) << pg.lC)] = lds[at_row(it >> 8, i)];
          });
      if (b + rw < b1) __syncthreads();
    } else if constexpr (SINK == Sink::ret) {
      pairs([&](int ci, int col, unsigned, unsigned, unsigned) {
        auto put = [&](int js, float4 h) {
          const int2 s = loc.ldi2(unsigned(col) * 8u, unsigned(js << pg.lw) * 8u);
          lds[unsigned(s.x) & kMask] = h.x;
          lds[(unsigned(s.x) >> 16) & kMask] = h.y;
          lds[unsigned(s.y) & kMask] = h.z;
          lds[(unsigned(s.y) >> 16) & kMask] = h.w;
        };
#pragma unroll
        for (int j = 0; j < H; ++j) {
          put(2 * j, ha[ci][j]);
          put(2 * j + 1, hb[ci][j]);
        }
      });
      __syncthreads();
      float4* t4 = reinterpret_cast<float4*>(A.dst + b * N + ((long long)c << pg.lC));
      for (int i = threadIdx.x; i < C / 4; i += THREADS) t4[i] = lds4[i];
      if (b + rw < b1) __syncthreads();
    } else {
      pairs([&](int ci, int, unsigned n, unsigned nb, unsigned o) {
        float2 x[R];
        // one butterfly of the pair: FIRST the one of column n
        auto bfly = [&](auto first, unsigned at) {
          constexpr bool kFirst = decltype(first)::value;
#pragma unroll
          for (int j = 0; j < H; ++j) {
            x[j] = chunk_even(kFirst ? ha[ci][j] : hb[ci][j]);
            x[R - 1 - j] = chunk_odd(kFirst ? hb[ci][j] : ha[ci][j]);
          }
          Dft<R, false>::run(x);
#pragma unroll
          for (int r = 1; r < R; ++r) x[r] = cmul(x[r], tw.ld2(at * 8u, (r - 1) * sq8));
#pragma unroll
          for (int r = 0; r < R; ++r) z.st2(x[r], at * 8u + o, r * sq8);
        };
        bfly(std::true_type{}, n);
        ACDC_SCHED_FENCE();
        bfly(std::false_type{}, nb);
      });
    }
  }
  if constexpr (BWD) {
    const GView out = GView::of(A.part + p * N);
    pairs([&](int ci, int, unsigned n, unsigned nb, unsigned) {
#pragma unroll
      for (int j = 0; j < H; ++j) {
        out.st4(sa[ci][j], n * 16u, j * sq16);
        out.st4(sb[ci][j], nb * 16u, j * sq16);
      }
    });
  }
}

// Complex rows: columns n, elements n + jQ.  Images gh1 * conj(u), and
// dL/du = gh1 * conj(a).
template <int R, Src SRC, Sink SINK, bool BWD, bool NARROW>
__global__ __launch_bounds__(col_threads(R, 2)) __attribute__((amdgpu_waves_per_eu(4))) void k_ccols(ColArgs A) {
  constexpr int THREADS = col_threads(R, 2), EC = kPermChunk / 2;  // elements of a whole set
  constexpr int CI = EC / (R * THREADS), W = EC / R;
  constexpr unsigned kMask = EC - 1;
  static_assert(CI >= 1 && CI * THREADS == W, "a set's elements over the threads");
  __shared__ float4 lds4[needs_lds<SRC, SINK>() ? kPermChunk / 4 : 1];
  __shared__ int dl[kPermMaxChunks];
  float2* lds = reinterpret_cast<float2*>(lds4);
  const PermGeo pg = A.pg;
  const int C = 1 << pg.lC, w = 1 << pg.lw;
  const long long M = A.M;
  const int c = int(blockIdx.x % unsigned(pg.nC));
  const long long p = blockIdx.x / unsigned(pg.nC);
  if constexpr (SRC == Src::scatter || SINK == Sink::send) {
    for (int d = threadIdx.x; d < pg.nC; d += THREADS) dl[d] = A.delta[c * pg.nC + d];
    __syncthreads();
  }
  const unsigned* item = A.item + ((long long)c << pg.lC);
  const GView loc = GView::of(A.loc + ((long long)c << pg.lC)), tw = GView::of(A.tw), av = GView::of(A.a);
  const unsigned sq8 = 8u << pg.lQ, nm = unsigned(M - 1);
  float2 h[CI][R], s[CI][R];
  if constexpr (BWD) {
#pragma unroll
    for (int ci = 0; ci < CI; ++ci)
#pragma unroll
      for (int j = 0; j < R; ++j) s[ci][j] = make_float2(0.f, 0.f);
  }
  auto at_row = [&](unsigned ls, int i) { return (ls + (NARROW ? unsigned(i >> pg.lC) << pg.lw : 0u)) & kMask; };
  int nr = 1;
  auto columns = [&](auto&& f) {
#pragma unroll
    for (int ci = 0; ci < CI; ++ci) {
      const int col = int(threadIdx.x) + ci * THREADS;
      const int row = NARROW ? col >> pg.lw : 0;
      if (NARROW ? row < nr : col < w) {
        f(ci, col, fresh(((unsigned(c) << pg.lw) + unsigned(col - (row << pg.lw))) * 8u),
          NARROW ? unsigned(row) << (pg.lC + 3) : 0u);
        ACDC_SCHED_FENCE();
      }
    }
  };
  const long long rw = NARROW ? A.rw : 1, b0 = p * A.rb * rw, b1 = b0 + A.rb * rw < A.B ? b0 + A.rb * rw : A.B;
  for (long long b = b0; b < b1; b += rw) {
    if constexpr (NARROW) nr = int(b1 - b < rw ? b1 - b : rw);
    const int total = NARROW ? nr << pg.lC : C;
    const GView z = GView::of(A.Z + b * M);
    if constexpr (SRC == Src::rows) {
      const GView row = GView::of(A.src + 2 * b * M);
      columns([&](int ci, int, unsigned n8, unsigned o) {
#pragma unroll
        for (int j = 0; j < R; ++j) h[ci][j] = row.ld2(n8 + o, j * sq8);
      });
    } else if constexpr (SRC == Src::gather) {
      const float4* t4 = reinterpret_cast<const float4*>(A.src + 2 * (b * M + ((long long)c << pg.lC)));
      for_entries<THREADS, 8, float4>(
          total / 2, [&](int i) { return t4[i]; }, [&](int i, float4 v) { lds4[i] = v; });
      __syncthreads();
      columns([&](int ci, int col, unsigned, unsigned o) {
#pragma unroll
        for (int j = 0; j < R; ++j)
          h[ci][j] = lds[(loc.ldu16(unsigned(NARROW ? col & (w - 1) : col) * 2u, unsigned(j << pg.lw) * 2u) + o / 8) & kMask];
      });
      if (b + rw < b1) __syncthreads();
    } else if constexpr (SRC == Src::scatter) {
      const float2* trow = reinterpret_cast<const float2*>(A.src) + b * M;
      for_entries<THREADS, NARROW ? 8 : 16, Entry<float2>>(
          total,
          [&](int i) {
            const int r = NARROW ? i >> pg.lC : 0, e = i - (r << pg.lC);
            const unsigned it = item[e];
            return Entry<float2>{it, trow[(unsigned(e + dl[it & 255]) & nm) + (unsigned(r) << pg.lC)]};
          },
          [&](int i, const Entry<float2>& e) { lds[at_row(e.it >> 8, i)] = e.v; });
      __syncthreads();
      columns([&](int ci, int col, unsigned, unsigned o) {
#pragma unroll
        for (int j = 0; j < R; ++j) h[ci][j] = lds[j * W + col];
      });
      if (b + rw < b1) __syncthreads();
    } else {
      columns([&](int ci, int, unsigned n8, unsigned o) {
        float2 y[R];
#pragma unroll
        for (int r = 0; r < R; ++r) y[r] = z.ld2(n8 + o, r * sq8);
#pragma unroll
        for (int r = 1; r < R; ++r) y[r] = cmulc(y[r], tw.ld2(n8, (r - 1) * sq8));
        Dft<R, true>::run(y);
#pragma unroll
        for (int j = 0; j < R; ++j) h[ci][j] = y[j];
      });
    }
    if constexpr (BWD) {
      const GView uv = GView::of(A.u + 2 * b * M);
      columns([&](int ci, int, unsigned n8, unsigned o) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
          if (j == R / 2) ACDC_SCHED_FENCE();
          const float2 img = cmulc(h[ci][j], uv.ld2(n8, j * sq8));
          s[ci][j] = make_float2(s[ci][j].x + img.x, s[ci][j].y + img.y);
          h[ci][j] = cmulc(h[ci][j], av.ld2(n8, j * sq8));
        }
      });
    }
    if constexpr (SINK == Sink::dif && !BWD) {
      if (A.stash != nullptr) {
        const GView st = GView::of(A.stash + 2 * b * M);
        columns([&](int ci, int, unsigned n8, unsigned o) {
#pragma unroll
          for (int j = 0; j < R; ++j) st.st2(h[ci][j], n8 + o, j * sq8);
        });
      }
      if (A.a != nullptr) {
        columns([&](int ci, int, unsigned n8, unsigned o) {
#pragma unroll
          for (int j = 0; j < R; ++j) h[ci][j] = cmul(h[ci][j], av.ld2(n8, j * sq8));
        });
      }
    }
    if constexpr (SINK == Sink::rows) {
      const GView out = GView::of(A.dst + 2 * b * M);
      columns([&](int ci, int, unsigned n8, unsigned o) {
#pragma unroll
        for (int j = 0; j < R; ++j) out.st2(h[ci][j], n8 + o, j * sq8);
      });
    } else if constexpr (SINK == Sink::send) {
      columns([&](int ci, int col, unsigned, unsigned o) {
#pragma unroll
        for (int j = 0; j < R; ++j) lds[j * W + col] = h[ci][j];
      });
      __syncthreads();
      float2* trow = reinterpret_cast<float2*>(A.dst) + b * M;
      for_entries<THREADS, 8, unsigned>(
          total, [&](int i) { return item[NARROW ? i & (C - 1) : i]; },
          [&](int i, unsigned it) {
            const int r = NARROW ? i >> pg.lC : 0, e = i - (r << pg.lC);
            trow[(unsigned(e + dl[it & 255]) & nm) + (unsigned(r) << pg.lC)] = lds[at_row(it >> 8, i)];
          });
      if (b + rw < b1) __syncthreads();
    } else if constexpr (SINK == Sink::ret) {
      columns([&](int ci, int col, unsigned, unsigned o) {
#pragma unroll
        for (int j = 0; j < R; ++j) lds[loc.ldu16(unsigned(col) * 2u, unsigned(j << pg.lw) * 2u) & kMask] = h[ci][j];
      });
      __syncthreads();
      float4* t4 = reinterpret_cast<float4*>(A.dst + 2 * (b * M + ((long long)c << pg.lC)));
      for (int i = threadIdx.x; i < C / 2; i += THREADS) t4[i] = lds4[i];
      if (b + rw < b1) __syncthreads();
    } else {
      columns([&](int ci, int, unsigned n8, unsigned o) {
        float2 x[R];
#pragma unroll
        for (int j = 0; j < R; ++j) x[j] = h[ci][j];
        Dft<R, false>::run(x);
#pragma unroll
        for (int r = 1; r < R; ++r) x[r] = cmul(x[r], tw.ld2(n8, (r - 1) * sq8));
#pragma unroll
        for (int r = 0; r < R; ++r) z.st2(x[r], n8 + o, r * sq8);
      });
    }
  }
  if constexpr (BWD) {
    const GView out = GView::of(A.part + 2 * p * M);
    columns([&](int ci, int, unsigned n8, unsigned o) {
#pragma unroll
      for (int j = 0; j < R; ++j) out.st2(s[ci][j], n8, j * sq8);
    });
  }
}

// Second-level radix-R passes on the R1 parts of a row (S = M / R1 = R L):
// butterfly n of a part takes x[n + j L]; tw2 [R-1][L] holds W_S^(n r).
template <int R, bool INV>
__global__ __launch_bounds__(kThreads) void k_part(float2* __restrict__ Z, long long n_bfly, int lL,
                                                   const float2* __restrict__ tw2) {
  for (long long i = gindex(); i < n_bfly; i += gstride()) {
    const long long L = 1LL << lL, n = i & (L - 1);
    float2* z = Z + (i >> lL) * (R * L) + n;
    float2 x[R];
#pragma unroll
    for (int j = 0; j < R; ++j) x[j] = z[j << lL];
    if constexpr (INV) {
#pragma unroll
      for (int r = 1; r < R; ++r) x[r] = cmulc(x[r], tw2[((r - 1) << lL) + n]);
    }
    Dft<R, INV>::run(x);
    if constexpr (!INV) {
#pragma unroll
      for (int r = 1; r < R; ++r) x[r] = cmul(x[r], tw2[((r - 1) << lL) + n]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) z[r << lL] = x[r];
  }
}

// ---------------------------------------------------------------- segments
// Segment plans: one butterfly per thread in the first and last pass, so that
// frequency k2 = t + T s sits in register s of lane t.  8 values per thread;
// at 4096 points the forward takes 16 (one exchange less, a fifth fewer
// operations; complex rows 78 -> 69 us, real ones 102 -> 92 us for 134 MB
// of rows), which in the backward, with several arrays and the image sums
// in registers, spills (real 181 -> 294 us) or gains nothing (complex).
// Slabs are padded by one slot per 16 elements: an LDS access of 8 bytes a
// lane runs 16 lanes at a time over 32 banks, so 16 neighbouring elements
// must not hold a pad (pads of 8, the first radix: 3 % slower in the
// backward).
using SP64 = ComplexPlan<64, 8, 8, 8, 1, 1, 4>;
using SP128 = ComplexPlan<128, 16, 8, 2, 8, 1, 4>;
using SP256 = ComplexPlan<256, 32, 8, 4, 8, 1, 4>;
using SP512 = ComplexPlan<512, 64, 8, 8, 8, 1, 4>;
using SP1024 = ComplexPlan<1024, 128, 8, 4, 4, 8, 4>;
using SP4096 = ComplexPlan<4096, 512, 8, 8, 8, 8, 4>;
using SP4096F = ComplexPlan<4096, 256, 16, 16, 16>;

template <bool FWD, class F>
bool with_seg_plan(int L, F&& f) {
  switch (L) {
    case 64: f.template operator()<SP64>(); return true;
    case 128: f.template operator()<SP128>(); return true;
    case 256: f.template operator()<SP256>(); return true;
    case 512: f.template operator()<SP512>(); return true;
    case 1024: f.template operator()<SP1024>(); return true;
    case 4096:
      if constexpr (FWD) f.template operator()<SP4096F>();
      else f.template operator()<SP4096>();
      return true;
    default: return false;
  }
}
static_assert(SP64::T == seg_fwd_threads(64) && SP1024::T == seg_fwd_threads(1024) &&
                  SP4096F::T == seg_fwd_threads(4096),
              "the forward plans' threads");

// The segment launches loop over rows and are bound by arithmetic and LDS
// about as much as by HBM, so a thread keeps what does not change between
// rows in registers: the twiddles of all passes (the plans' radices are
// palindromes or the inverse loads its own), and for complex rows d / N.
// Several arrays (h and g, the two segments of a pair) run pass by pass
// together, each with its own slab, for two barriers per exchange in all.
template <class PL>
struct Seg {
  using O = CplxOps<PL>;
  static constexpr int T = PL::T, P = PL::P, L = PL::N;
  static_assert(O::B0 == 1 && O::BL == 1 && O::KIND == 0, "register s of lane t holds t + T s at both ends");
  static_assert(PL::palindrome(), "both directions share their twiddles");
  static constexpr int GROUPS = T < 64 ? 64 / T : 1;  // segments (pairs) per workgroup
  static constexpr int THREADS = T < 64 ? 64 : T;
  static constexpr int SLAB = PL::SLAB;
  static constexpr int NP = PL::NPASS;

  // Twiddles of passes 1 .. NP-1 for lane t, and of the last pass for the
  // reversed lane T-1-t.
  struct Tw {
    PassTw<PL, false, 1, 0, 0> w1;
    PassTw<PL, false, 2, 0, 0> w2;
    PassTw<PL, false, 3, 0, 0> w3;
    __device__ __forceinline__ void load(unsigned t, GView tab) {
      w1.load(t, tab);
      if constexpr (NP > 2) w2.load(t, tab);
      if constexpr (NP > 3) w3.load(t, tab);
    }
  };
  template <int PASS, bool INV, int Q>
  __device__ __forceinline__ static void twiddle(float2 (&x)[P], const PassTw<PL, false, Q, 0, 0>& w) {
    constexpr int r = PL::radix(PASS, INV), b = P / r;
#pragma unroll
    for (int beta = 0; beta < b; ++beta)
#pragma unroll
      for (int i = 1; i < r; ++i) x[beta * r + i] = ctw<INV>(x[beta * r + i], w.w[beta * (r - 1) + i - 1]);
  }
  // One pass over NA arrays; with REV the odd arrays' spectra are held with
  // the lanes reversed (their forward last pass and inverse first pass run
  // at lane T-1-t).
  template <bool INV, int PASS, int NA, bool REV, class Ctx>
  __device__ __forceinline__ static void pass(Ctx& ctx, float2 (&x)[NA][P], unsigned t, float2* slab, const Tw& tw,
                                              const Tw& rt) {
    using G = PassGeo<PL, INV, PASS, 0, 0>;
    const G geo(t), rev(T - 1 - t);
    auto geo_of = [&](int a) -> const G& { return REV && (a & 1) && (INV ? PASS == 0 : PASS == NP - 1) ? rev : geo; };
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const bool r = REV && (a & 1) && !INV && PASS == NP - 1;
      if constexpr (PASS > 0) geo_of(a).read(x[a], slab + a * (SLAB / 2));
      if constexpr (PASS == 1) twiddle<PASS, INV>(x[a], r ? rt.w1 : tw.w1);
      if constexpr (PASS == 2) twiddle<PASS, INV>(x[a], r ? rt.w2 : tw.w2);
      if constexpr (PASS == 3) twiddle<PASS, INV>(x[a], r ? rt.w3 : tw.w3);
      G::dft(x[a]);
      if constexpr (NA > 2) ACDC_SCHED_FENCE();
    }
    if constexpr (PASS < NP - 1) {
      ctx.sync_row();
#pragma unroll
      for (int a = 0; a < NA; ++a) geo_of(a).write(x[a], slab + a * (SLAB / 2));
      ctx.sync_row();
    }
  }
  template <bool INV, int NA, bool REV, class Ctx>
  __device__ __forceinline__ static void fft(Ctx& ctx, float2 (&x)[NA][P], unsigned t, float2* slab, const Tw& tw,
                                             const Tw& rt) {
    pass<INV, 0, NA, REV>(ctx, x, t, slab, tw, rt);
    pass<INV, 1, NA, REV>(ctx, x, t, slab, tw, rt);
    if constexpr (NP > 2) pass<INV, 2, NA, REV>(ctx, x, t, slab, tw, rt);
    if constexpr (NP > 3) pass<INV, 3, NA, REV>(ctx, x, t, slab, tw, rt);
  }
  __device__ __forceinline__ static void load(const float2* seg, float2 (&x)[P], unsigned t) {
    O::template ld_row<false>(GView::of(seg), 0u, x, t);
  }
  __device__ __forceinline__ static void store(float2* seg, float2 (&x)[P], unsigned t) {
    O::template st_row<true>(GView::of(seg), 0u, x, t);
  }
};

// The lanes of one pair, x[0] = segment A (lane t), x[1] = segment B, whose
// spectrum is held with the lanes reversed.  Then register s of x[0] and
// register P-1-s of x[1] hold k2 and L-1-k2, Makhoul partners in a generic
// pair.  Slot s has (Z[e], Z[M-e]) = (x[0][s], x[1][P-1-s]) for s < P/2 and
// the other way round from there on, where k > M/2.
template <class PL>
struct PairOps {
  using G = Seg<PL>;
  static constexpr int T = PL::T, P = PL::P, L = PL::N;
  static __device__ __forceinline__ float2& zk(float2 (&v)[P], float2 (&w)[P], int s) {
    return s < P / 2 ? v[s] : w[P - 1 - s];
  }
  static __device__ __forceinline__ float2& zm(float2 (&v)[P], float2 (&w)[P], int s) {
    return s < P / 2 ? w[P - 1 - s] : v[s];
  }
  // Pair 0: the partners lie in other lanes of the same segment.  Through
  // two slabs: segment 0's quartets q = t + T s (k2 = q, L-q; q = 0: 0, L/2)
  // into slots s < P/2, segment B's (q, L-1-q) into the others; and back.
  template <class Ctx>
  __device__ __forceinline__ static void to_quartets(Ctx& ctx, float2 (&v)[P], float2 (&w)[P], unsigned t,
                                                     float2* slab) {
    float2* const slab2 = slab + G::SLAB / 2;
    ctx.sync_row();
#pragma unroll
    for (int s = 0; s < P; ++s) {
      slab[t + T * s] = v[s];
      slab2[T - 1 - t + T * s] = w[s];
    }
    ctx.sync_row();
#pragma unroll
    for (int s = 0; s < P / 2; ++s) {
      const unsigned q = t + T * s;
      zk(v, w, s) = slab[q];
      zm(v, w, s) = slab[q == 0 ? L / 2 : L - q];
      zk(v, w, s + P / 2) = slab2[q];
      zm(v, w, s + P / 2) = slab2[L - 1 - q];
    }
  }
  template <class Ctx>
  __device__ __forceinline__ static void from_quartets(Ctx& ctx, float2 (&v)[P], float2 (&w)[P], unsigned t,
                                                       float2* slab) {
    float2* const slab2 = slab + G::SLAB / 2;
    ctx.sync_row();
#pragma unroll
    for (int s = 0; s < P / 2; ++s) {
      const unsigned q = t + T * s;
      slab[q] = zk(v, w, s);
      slab[q == 0 ? L / 2 : L - q] = zm(v, w, s);
      slab2[q] = zk(v, w, s + P / 2);
      slab2[L - 1 - q] = zm(v, w, s + P / 2);
    }
    ctx.sync_row();
#pragma unroll
    for (int s = 0; s < P; ++s) {
      v[s] = slab[t + T * s];
      w[s] = slab2[T - 1 - t + T * s];
    }
  }
};

// What a workgroup's group of lanes works on: rows b0 .. b1 of unit `unit`
// (a segment or pair; `units` a row), blocks of rb rows.  Groups past the
// end repeat the first unit without storing.
struct SegWork {
  bool valid;
  int unit;
  long long blk, b0, b1;
  __device__ __forceinline__ SegWork(long long id, int units, long long B, int rb) {
    const long long nblk = (B + rb - 1) / rb;
    valid = id < nblk * units;
    unit = valid ? int(id % units) : 0;
    blk = valid ? id / units : 0;
    b0 = blk * rb;
    b1 = b0 + rb < B ? b0 + rb : B;
  }
};

// Waves per SIMD of the forward launches: what the values, the twiddles and
// (complex) d of a thread leave room for.
template <class PL>
constexpr int seg_fwd_waves() {
  return PL::P == 8 ? 4 : 2;
}

// Forward: segment FFTs of a pair, the quartet maps, segment IFFTs.  BIAS: a
// template, since a branch on it per slot kept every slot's c3 load from
// being issued with the others (N = 65536, one row: 15 -> 20 us a launch).
template <class PL, bool BIAS>
__global__ __launch_bounds__(Seg<PL>::THREADS) __attribute__((amdgpu_waves_per_eu(seg_fwd_waves<PL>()))) void k_seg_fwd(
    float2* __restrict__ Z, const float4* __restrict__ Mq, long long B, Geo g, int rb, const char* __restrict__ tab) {
  using G = Seg<PL>;
  using Q = PairOps<PL>;
  constexpr int T = PL::T, P = PL::P;
  __shared__ float lds[G::GROUPS * 2 * G::SLAB];
  const unsigned t = threadIdx.x % T, grp = threadIdx.x / T;
  float2* slab = reinterpret_cast<float2*>(lds + grp * 2 * G::SLAB);
  const SegWork wk((long long)blockIdx.x * G::GROUPS + grp, g.R1 * g.R2 / 2, B, rb);
  const int p = wk.unit;
  int sa, sb;
  seg_pair(g, p, sa, sb);
  DevCtx<T> ctx;
  typename G::Tw tw, rt;
  tw.load(t, GView::of(tab));
  rt.load(T - 1 - t, GView::of(tab));
  const GView mq = GView::of(Mq + (long long)p * PL::N * kMqRows);
  for (long long b = wk.b0; b < wk.b1; ++b) {
    float2* const za = Z + b * g.M + (long long)sa * PL::N;
    float2* const zb = Z + b * g.M + (long long)sb * PL::N;
    const unsigned t16 = fresh(t * 16u);
    float2 x[2][P];
    G::load(za, x[0], t);
    G::load(zb, x[1], t);
    G::template fft<false, 2, true>(ctx, x, t, slab, tw, rt);
    if (p == 0) Q::to_quartets(ctx, x[0], x[1], t, slab);
#pragma unroll
    for (int s = 0; s < P; ++s) {
      if (s % 2 == 0) ACDC_SCHED_FENCE();
      float2& zk = Q::zk(x[0], x[1], s);
      float2& zm = Q::zm(x[0], x[1], s);
      const float4 c0 = mq.ld4(t16, unsigned((0 * PL::N + s * T) * 16));
      const float4 c1 = mq.ld4(t16, unsigned((1 * PL::N + s * T) * 16));
      float4 c3;
      if constexpr (BIAS) c3 = mq.ld4(t16, unsigned((3 * PL::N + s * T) * 16));
      quartet_back(quartet_split(zk, zm, make_float2(c1.z, c1.w)), c0, c1, zk, zm);
      if constexpr (BIAS) {
        zk = make_float2(zk.x + c3.x, zk.y + c3.y);
        zm = make_float2(zm.x + c3.z, zm.y + c3.w);
      }
    }
    if (p == 0) Q::from_quartets(ctx, x[0], x[1], t, slab);
    G::template fft<true, 2, true>(ctx, x, t, slab, tw, rt);
    if (wk.valid) {
      G::store(za, x[0], t);
      G::store(zb, x[1], t);
    }
  }
}

// Backward: rb rows in turn.  Segment FFTs of h and g, the images H*G (dL/dd)
// summed over the rows, g's quartets through the D maps, its segment IFFTs.
template <class PL>
__global__ __launch_bounds__(Seg<PL>::THREADS) __attribute__((amdgpu_waves_per_eu(2))) void k_seg_bwd(
    const float2* __restrict__ Zh, float2* __restrict__ Zg, const float4* __restrict__ Mq, long long B, Geo g, int rb,
    float* __restrict__ part, const char* __restrict__ tab) {
  using G = Seg<PL>;
  using Q = PairOps<PL>;
  constexpr int T = PL::T, P = PL::P;
  __shared__ float lds[G::GROUPS * 2 * G::SLAB];
  const unsigned t = threadIdx.x % T, grp = threadIdx.x / T;
  float2* slab = reinterpret_cast<float2*>(lds + grp * 2 * G::SLAB);
  const SegWork wk((long long)blockIdx.x * G::GROUPS + grp, g.R1 * g.R2 / 2, B, rb);
  const int p = wk.unit;
  int sa, sb;
  seg_pair(g, p, sa, sb);
  DevCtx<T> ctx;
  typename G::Tw tw, rt;
  tw.load(t, GView::of(tab));
  rt.load(T - 1 - t, GView::of(tab));
  const GView mq = GView::of(Mq + (long long)p * PL::N * kMqRows);
  float4 sum[P];
#pragma unroll
  for (int s = 0; s < P; ++s) sum[s] = make_float4(0.f, 0.f, 0.f, 0.f);
  // pair 0 on a path of its own: joined inside the row, its exchanges cost
  // every pair registers (47 spilled at two waves per SIMD)
  auto rows = [&](auto special) {
  for (long long b = wk.b0; b < wk.b1; ++b) {
    const long long oa = b * g.M + (long long)sa * PL::N, ob = b * g.M + (long long)sb * PL::N;
    const unsigned t16 = fresh(t * 16u);
    float2 h[2][P], x[2][P];
    G::load(Zh + oa, h[0], t);
    G::load(Zh + ob, h[1], t);
    G::load(Zg + oa, x[0], t);
    G::load(Zg + ob, x[1], t);
    G::template fft<false, 2, true>(ctx, h, t, slab, tw, rt);
    ACDC_SCHED_FENCE();
    G::template fft<false, 2, true>(ctx, x, t, slab, tw, rt);
    ACDC_SCHED_FENCE();
    if constexpr (special.value) {
      Q::to_quartets(ctx, h[0], h[1], t, slab);
      Q::to_quartets(ctx, x[0], x[1], t, slab);
    }
#pragma unroll
    for (int s = 0; s < P; ++s) {
      if (s % 2 == 0) ACDC_SCHED_FENCE();
      const float4 c0 = mq.ld4(t16, unsigned((0 * PL::N + s * T) * 16));
      const float4 c1 = mq.ld4(t16, unsigned((1 * PL::N + s * T) * 16));
      const float4 c2 = mq.ld4(t16, unsigned((2 * PL::N + s * T) * 16));
      const float2 wt = make_float2(c1.z, c1.w), qa = make_float2(c2.x, c2.y), qbr = make_float2(c2.z, c2.w);
      float2& gk = Q::zk(x[0], x[1], s);
      float2& gm = Q::zm(x[0], x[1], s);
      float H[4], X[4];
      quartet_post(quartet_split(Q::zk(h[0], h[1], s), Q::zm(h[0], h[1], s), wt), qa, qbr, H);
      const Split sg = quartet_split(gk, gm, wt);
      quartet_post(sg, qa, qbr, X);
      sum[s] = make_float4(sum[s].x + H[0] * X[0], sum[s].y + H[1] * X[1], sum[s].z + H[2] * X[2],
                           sum[s].w + H[3] * X[3]);
      quartet_back(sg, c0, c1, gk, gm);
    }
    if constexpr (special.value) Q::from_quartets(ctx, x[0], x[1], t, slab);
    G::template fft<true, 2, true>(ctx, x, t, slab, tw, rt);
    if (wk.valid) {
      G::store(Zg + oa, x[0], t);
      G::store(Zg + ob, x[1], t);
    }
  }
  };
  if (p == 0) rows(std::true_type{});
  else rows(std::false_type{});
  if (!wk.valid) return;
  float4* out = reinterpret_cast<float4*>(part + wk.blk * 2 * g.M) + (long long)p * PL::N;
#pragma unroll
  for (int s = 0; s < P; ++s) out[T * s + t] = sum[s];
}

// DCT-II outputs of one row per layer whose DIF passes are done (the bias
// gradients): out[k] (+)= those of Z[k].  Latency is all there is, so one
// launch takes every layer, all table loads are issued before the FFT, and
// the DCT indices are computed: read per slot between the stores, which the
// compiler cannot move loads across, they took 15 to 20 us, and a launch per
// layer at that.  N = 65536, K = 4, one row with biases, backward 271 -> 190
// us.
template <class PL>
__global__ __launch_bounds__(Seg<PL>::THREADS) void k_seg_dct(const float2* __restrict__ Z,
                                                              const float4* __restrict__ Mq, int K, Geo g,
                                                              float* __restrict__ out, int accumulate,
                                                              const char* __restrict__ tab) {
  using G = Seg<PL>;
  using Q = PairOps<PL>;
  constexpr int T = PL::T, P = PL::P;
  __shared__ float lds[G::GROUPS * 2 * G::SLAB];
  const unsigned t = threadIdx.x % T, grp = threadIdx.x / T;
  float2* slab = reinterpret_cast<float2*>(lds + grp * 2 * G::SLAB);
  const SegWork wk((long long)blockIdx.x * G::GROUPS + grp, g.R1 * g.R2 / 2, K, 1);
  const int p = wk.unit;
  int sa, sb;
  seg_pair(g, p, sa, sb);
  const float2* z = Z + wk.blk * g.M;
  DevCtx<T> ctx;
  typename G::Tw tw, rt;
  float2 x[2][P];
  G::load(z + (long long)sa * PL::N, x[0], t);
  G::load(z + (long long)sb * PL::N, x[1], t);
  tw.load(t, GView::of(tab));
  rt.load(T - 1 - t, GView::of(tab));
  const GView mq = GView::of(Mq + wk.blk * (g.M / 2) * kMqRows + (long long)p * PL::N * kMqRows);
  float4 c1[P], c2[P];
#pragma unroll
  for (int s = 0; s < P; ++s) {
    c1[s] = mq.ld4(t * 16u, unsigned((1 * PL::N + s * T) * 16));
    c2[s] = mq.ld4(t * 16u, unsigned((2 * PL::N + s * T) * 16));
  }
  ACDC_SCHED_FENCE();
  G::template fft<false, 2, true>(ctx, x, t, slab, tw, rt);
  if (p == 0) Q::to_quartets(ctx, x[0], x[1], t, slab);
  if (!wk.valid) return;
  float X[P][4], old[P][4];
  int4 id[P];
  out += wk.blk * 2 * g.M;
#pragma unroll
  for (int s = 0; s < P; ++s) {
    const int e = int(quartet_of(g, p, sa, int(t) + T * s));
    id[s] = quartet_idx(int(2 * g.M), e == 0 ? -2 : e);
    quartet_post(quartet_split(Q::zk(x[0], x[1], s), Q::zm(x[0], x[1], s), make_float2(c1[s].z, c1[s].w)),
                 make_float2(c2[s].x, c2[s].y), make_float2(c2[s].z, c2[s].w), X[s]);
    X[s][1] = -X[s][1];
  }
#pragma unroll
  for (int s = 0; s < P; ++s) {
    const int i4[4] = {id[s].x, id[s].y, id[s].z, id[s].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) old[s][j] = accumulate ? out[i4[j]] : 0.f;
  }
#pragma unroll
  for (int s = 0; s < P; ++s) {
    const int i4[4] = {id[s].x, id[s].y, id[s].z, id[s].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) out[i4[j]] = accumulate ? old[s][j] + X[s][j] : X[s][j];
  }
}

// Complex rows: segment FFT, * d / N (Dn in storage order), segment IFFT.
// The next row is loaded while one is transformed.
template <class PL>
__global__ __launch_bounds__(Seg<PL>::THREADS) __attribute__((amdgpu_waves_per_eu(seg_fwd_waves<PL>()))) void k_cseg_fwd(
    float2* __restrict__ Z, const float2* __restrict__ Dn, long long B, Geo g, int rb, const char* __restrict__ tab) {
  using G = Seg<PL>;
  constexpr int T = PL::T, P = PL::P;
  __shared__ float lds[G::GROUPS * G::SLAB];
  const unsigned t = threadIdx.x % T, grp = threadIdx.x / T;
  float2* slab = reinterpret_cast<float2*>(lds + grp * G::SLAB);
  const SegWork wk((long long)blockIdx.x * G::GROUPS + grp, g.R1 * g.R2, B, rb);
  const GView dn = GView::of(Dn + (long long)wk.unit * PL::N);
  DevCtx<T> ctx;
  typename G::Tw tw;
  tw.load(t, GView::of(tab));
  float2 d[P], n[1][P];
#pragma unroll
  for (int s = 0; s < P; ++s) d[s] = dn.ld2(t * 8u, unsigned(T * s) * 8u);
  float2* z = Z + wk.b0 * g.M + (long long)wk.unit * PL::N;
  G::load(z, n[0], t);
  for (long long b = wk.b0; b < wk.b1; ++b, z += g.M) {
    float2 x[1][P];
#pragma unroll
    for (int s = 0; s < P; ++s) x[0][s] = n[0][s];
    if (b + 1 < wk.b1) G::load(z + g.M, n[0], t);
    ACDC_SCHED_FENCE();
    G::template fft<false, 1, false>(ctx, x, t, slab, tw, tw);
#pragma unroll
    for (int s = 0; s < P; ++s) x[0][s] = cmul(x[0][s], d[s]);
    G::template fft<true, 1, false>(ctx, x, t, slab, tw, tw);
    if (wk.valid) G::store(z, x[0], t);
  }
}

// Backward, rb rows in turn: gh3 = FFT(g) / N, images gh3 * conj(h2) summed
// over the rows (storage order), then gh3 * conj(d) and its segment IFFT.
// N is a power of two, so dividing the sum is exact.
template <class PL>
__global__ __launch_bounds__(Seg<PL>::THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_cseg_bwd(
    const float2* __restrict__ Zh, float2* __restrict__ Zg, const float2* __restrict__ Dn, long long B, Geo g, int rb,
    float2* __restrict__ part, const char* __restrict__ tab) {
  using G = Seg<PL>;
  constexpr int T = PL::T, P = PL::P;
  __shared__ float lds[G::GROUPS * 2 * G::SLAB];
  const unsigned t = threadIdx.x % T, grp = threadIdx.x / T;
  float2* slab = reinterpret_cast<float2*>(lds + grp * 2 * G::SLAB);
  const SegWork wk((long long)blockIdx.x * G::GROUPS + grp, g.R1 * g.R2, B, rb);
  const GView dn = GView::of(Dn + (long long)wk.unit * PL::N);
  DevCtx<T> ctx;
  typename G::Tw tw;
  tw.load(t, GView::of(tab));
  float2 sum[P];
#pragma unroll
  for (int s = 0; s < P; ++s) sum[s] = make_float2(0.f, 0.f);
  for (long long b = wk.b0; b < wk.b1; ++b) {
    const long long at = b * g.M + (long long)wk.unit * PL::N;
    const unsigned t8 = fresh(t * 8u);
    float2 x[2][P];
    G::load(Zh + at, x[0], t);
    G::load(Zg + at, x[1], t);
    G::template fft<false, 2, false>(ctx, x, t, slab, tw, tw);
    float2 y[1][P];
#pragma unroll
    for (int s = 0; s < P; ++s) {
      const float2 img = cmulc(x[1][s], x[0][s]);
      sum[s] = make_float2(sum[s].x + img.x, sum[s].y + img.y);
      y[0][s] = cmulc(x[1][s], dn.ld2(t8, unsigned(T * s) * 8u));
    }
    G::template fft<true, 1, false>(ctx, y, t, slab, tw, tw);
    if (wk.valid) G::store(Zg + at, y[0], t);
  }
  if (!wk.valid) return;
  const float inv = 1.0f / float(g.M);
  float2* out = part + wk.blk * g.M + (long long)wk.unit * PL::N;
#pragma unroll
  for (int s = 0; s < P; ++s) out[T * s + t] = make_float2(sum[s].x * inv, sum[s].y * inv);
}

// Per-layer quartet coefficients, [K][pair][kMqRows][k2].  A pair's quartets
// lie S = R1 R2 apart in the tables and in D, so a workgroup takes a tile of
// cw neighbouring quartets in each of kThreads / cw places k2 and turns it in
// LDS: it reads runs of cw entries and writes runs of neighbouring places.
// N = 2^22 (S = 512), K = 4: 619 us with a thread for each place in order
// (every read a cache line of its own), 112 with the tiles.
constexpr int kMqTile = 16;
__global__ __launch_bounds__(kThreads) void k_mq(const float* __restrict__ D, const float* __restrict__ Bias,
                                                 float4* __restrict__ Mq, int K, Geo g, QuartetTabs q) {
  __shared__ float4 tile[kMqRows][kThreads];
  const int S = g.R1 * g.R2, cw = S < kMqTile ? S : kMqTile, kw = kThreads / cw, places = g.L / 2;
  const int tc = S / cw, tk = (places + kw - 1) / kw;  // tiles of a layer
  const long long NQ = g.M / 2, N = 2 * g.M, total = (long long)K * tc * tk;
  const int tid = threadIdx.x;
  for (long long i = blockIdx.x; i < total; i += gridDim.x) {
    const long long k = i / (tc * tk);
    const int r = int(i % (tc * tk)), c0 = r % tc * cw, k0 = r / tc * kw;
    {
      const int c = tid % cw, kk = tid / cw;
      if (k0 + kk < places) {
        const int e = c0 + c + S * (k0 + kk);
        float4 row[kMqRows];
        quartet_coeffs(D + k * N, Bias ? Bias + k * N : nullptr, q, e, quartet_idx(int(N), e == 0 ? -2 : e), row);
#pragma unroll
        for (int j = 0; j < kMqRows; ++j) tile[j][c * kw + kk] = row[j];
      }
    }
    __syncthreads();
    const int c = tid / kw, kk = tid % kw;
    if (k0 + kk < places) {
      int p, k2;
      quartet_place(g, c0 + c + (long long)S * (k0 + kk), p, k2);
      float4* out = Mq + (k * NQ + (long long)p * g.L) * kMqRows + k2;
#pragma unroll
      for (int j = 0; j < kMqRows; ++j) out[j * g.L] = tile[j][tid];
    }
    __syncthreads();
  }
}

// d / N of every layer in storage order.
__global__ __launch_bounds__(kThreads) void k_dn(const float2* __restrict__ D, float2* __restrict__ Dn, int K, Geo g,
                                                 float inv) {
  const long long total = (long long)K * g.M;
  for (long long i = gindex(); i < total; i += gstride()) {
    const float2 d = D[(i / g.M) * g.M + spec_index(g, i % g.M)];
    Dn[i] = make_float2(d.x * inv, d.y * inv);
  }
}

// -------------------------------------------------------------------- sums

// part[p][w] = sum of rows p*kMaxRows ... of img, in row order, four columns
// per thread.
__global__ __launch_bounds__(kThreads) void k_colsum1(const float* __restrict__ img, long long B, long long W,
                                                      float* __restrict__ part) {
  const long long W4 = W / 4, P = (B + kMaxRows - 1) / kMaxRows, total = P * W4;
  for (long long i = gindex(); i < total; i += gstride()) {
    const long long p = i / W4, w4 = i % W4;
    const long long b0 = p * kMaxRows, b1 = b0 + kMaxRows < B ? b0 + kMaxRows : B;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    const float4* col = reinterpret_cast<const float4*>(img) + w4;
#pragma unroll 4
    for (long long b = b0; b < b1; ++b) s = add4(s, col[b * W4]);
    reinterpret_cast<float4*>(part)[p * W4 + w4] = s;
  }
}

// The block sums in block order: kSumPh phases of consecutive blocks, one
// thread each, added in phase order (a column is a serial chain of P loads;
// W / 4 threads alone would leave the chip idle).
constexpr int kSumPh = 8, kSumCols = kThreads / kSumPh;
template <Order HOW>
__global__ __launch_bounds__(kThreads) void k_colsum2(const float* __restrict__ part, long long P, long long W,
                                                      float* __restrict__ out, Geo g, QuartetTabs q,
                                                      int accumulate) {
  __shared__ float4 ph[kSumPh][kSumCols];
  const int lane = threadIdx.x % kSumCols, f = threadIdx.x / kSumCols;
  const long long w4 = (long long)blockIdx.x * kSumCols + lane, W4 = W / 4;
  const long long per = (P + kSumPh - 1) / kSumPh, p0 = f * per, p1 = p0 + per < P ? p0 + per : P;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (w4 < W4) {
    const float4* col = reinterpret_cast<const float4*>(part) + w4;
#pragma unroll 4
    for (long long p = p0; p < p1; ++p) s = add4(s, col[p * W4]);
  }
  ph[f][lane] = s;
  __syncthreads();
  if (f != 0 || w4 >= W4) return;
#pragma unroll
  for (int r = 1; r < kSumPh; ++r) s = add4(s, ph[r][lane]);
  const bool acc = accumulate != 0;
  if constexpr (HOW == Order::natural) {
    put4(reinterpret_cast<float4*>(out) + w4, s, acc);
  } else if constexpr (HOW == Order::quartets) {
    const long long e = quartet_of(g, int(w4 / g.L), int(w4 % g.L));
    const int4 idx = q.qidx[e];
    put1(out + idx.x, s.x, acc);
    put1(out + idx.y, s.y, acc);
    put1(out + idx.z, s.z, acc);
    put1(out + idx.w, s.w, acc);
  } else {
    float2* o = reinterpret_cast<float2*>(out);
    const long long k0 = spec_index(g, 2 * w4), k1 = spec_index(g, 2 * w4 + 1);
    const float2 z = make_float2(0.f, 0.f);
    const float2 o0 = acc ? o[k0] : z, o1 = acc ? o[k1] : z;
    o[k0] = make_float2(o0.x + s.x, o0.y + s.y);
    o[k1] = make_float2(o1.x + s.z, o1.y + s.w);
  }
}

template <class F>
bool with_r1(int R1, F&& f) {
  switch (R1) {
    case 2: f.template operator()<2>(); return true;
    case 4: f.template operator()<4>(); return true;
    case 8: f.template operator()<8>(); return true;
    case 16: f.template operator()<16>(); return true;
    default: return false;
  }
}

template <Src SRC, Sink SINK, bool BWD>
bool launch_cols(bool cplx, int R1, dim3 grid, const ColArgs& a, hipStream_t s) {
  return with_r1(R1, [&]<int R>() {
    auto launch = [&]<bool NARROW>() {
      if (cplx) hipLaunchKernelGGL((k_ccols<R, SRC, SINK, BWD, NARROW>), grid, dim3(col_threads(R, 2)), 0, s, a);
      else hipLaunchKernelGGL((k_cols<R, SRC, SINK, BWD, NARROW>), grid, dim3(col_threads(R, 1)), 0, s, a);
    };
    if constexpr (narrow(R, BWD)) {
      if (a.rw > 1) return launch.template operator()<true>();
    }
    launch.template operator()<false>();
  });
}

template <bool INV>
hipError_t part_pass(float2* Z, long long B, const Geo& g, const float2* tw2, hipStream_t s) {
  if (g.R2 == 1) return hipSuccess;
  const long long n = B * (g.M / g.R2);
  const dim3 grid = grid_for(n), block(kThreads);
  const int lL = log2_of(g.L);
  switch (g.R2) {
    case 2: hipLaunchKernelGGL((k_part<2, INV>), grid, block, 0, s, Z, n, lL, tw2); break;
    case 4: hipLaunchKernelGGL((k_part<4, INV>), grid, block, 0, s, Z, n, lL, tw2); break;
    case 8: hipLaunchKernelGGL((k_part<8, INV>), grid, block, 0, s, Z, n, lL, tw2); break;
    case 16: hipLaunchKernelGGL((k_part<16, INV>), grid, block, 0, s, Z, n, lL, tw2); break;
    case 32: hipLaunchKernelGGL((k_part<32, INV>), grid, block, 0, s, Z, n, lL, tw2); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Workgroups for `units` segments or pairs of the plan.
template <class PL>
dim3 seg_grid(long long units) {
  return dim3(unsigned((units + Seg<PL>::GROUPS - 1) / Seg<PL>::GROUPS));
}

}  // namespace

size_t perm_table_ints(const Geo& g, int ew) {
  const PermGeo p = perm_geo(g, ew);
  const size_t N = size_t(2 * g.M / ew), nn = size_t(p.nC) * p.nC;
  return N + N / 2 + 2 * (N / kThreads) * p.nC + 4 * nn;
}

PermTabs perm_tables_at(int* base, const Geo& g, int ew) {
  const PermGeo p = perm_geo(g, ew);
  const long long N = 2 * g.M / ew, nb = N / kThreads, nn = (long long)p.nC * p.nC;
  PermTabs t;
  t.stride = (long long)perm_table_ints(g, ew);
  t.item = reinterpret_cast<unsigned*>(base);
  t.loc = reinterpret_cast<unsigned short*>(base + N);
  t.cntS = base + N + N / 2;
  t.bpre = t.cntS + nb * p.nC;
  t.cnt = t.bpre + nb * p.nC;
  t.start = t.cnt + nn;
  t.lst = t.start + nn;
  t.delta = t.lst + nn;
  return t;
}

PermTabs perm_layer(const PermTabs& t, int l) {
  const long long o = l * t.stride;
  PermTabs r = t;
  r.item += o;
  r.loc += 2 * o;
  r.cntS += o;
  r.bpre += o;
  r.cnt += o;
  r.start += o;
  r.lst += o;
  r.delta += o;
  return r;
}

hipError_t perm_build(const int* perm, const Geo& g, int ew, int layers, const PermTabs& t, hipStream_t s) {
  if (layers <= 0) return hipSuccess;
  const PermGeo p = perm_geo(g, ew);
  const long long N = 2 * g.M / ew;
  const unsigned nb = unsigned(N / kThreads), nn = unsigned(p.nC * p.nC), L = unsigned(layers);
  if (p.nC == 1) {
    hipLaunchKernelGGL(k_pt_one, dim3(nb, L), dim3(kThreads), 0, s, perm, N, p, t.item, t.loc, t.delta, t.stride);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_pt_count, dim3(nb, L), dim3(kThreads), 0, s, perm, N, p, t.cntS, t.stride);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_pt_blocks, dim3((nn + kThreads - 1) / kThreads, L), dim3(kThreads), 0, s, t.cntS, p, t.bpre,
                     t.cnt, t.stride);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_pt_offsets, dim3(L), dim3(kThreads), 0, s, t.cnt, p, t.start, t.lst, t.delta, t.stride);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_pt_place, dim3(nb, L), dim3(kThreads), 0, s, perm, N, p, t.bpre, t.start, t.lst, t.item,
                     t.loc, t.stride);
  return hipGetLastError();
}

hipError_t cols(Src src, Sink sink, bool cplx, const Cols& c, long long B, const Geo& g, const float2* tw1,
                hipStream_t s) {
  const PermGeo pg = perm_geo(g, cplx ? 2 : 1);
  const bool bwd = c.u != nullptr;
  const ColGrid cg = col_grid(B, g, pg.ew, bwd);
  if (cg.groups * cg.threads >= 1LL << 32) return hipErrorInvalidValue;
  ColArgs a{c.src,   c.dst, c.Z,  c.a,    c.stash, c.u, c.part, tw1, nullptr, nullptr, nullptr, B, g.M,
            cg.rw, cg.rb, c.relu, pg};
  if (c.pt != nullptr) {
    a.item = c.pt->item;
    a.loc = c.pt->loc;
    a.delta = c.pt->delta;
  }
  const dim3 grid(unsigned(cg.groups));
  auto is = [&](Src x, Sink y, bool w) { return src == x && sink == y && bwd == w; };
  bool ok = false;
  if (is(Src::rows, Sink::send, false)) ok = launch_cols<Src::rows, Sink::send, false>(cplx, g.R1, grid, a, s);
  else if (is(Src::rows, Sink::dif, false)) ok = launch_cols<Src::rows, Sink::dif, false>(cplx, g.R1, grid, a, s);
  else if (is(Src::gather, Sink::dif, false)) ok = launch_cols<Src::gather, Sink::dif, false>(cplx, g.R1, grid, a, s);
  else if (is(Src::dit, Sink::send, false)) ok = launch_cols<Src::dit, Sink::send, false>(cplx, g.R1, grid, a, s);
  else if (is(Src::dit, Sink::rows, false)) ok = launch_cols<Src::dit, Sink::rows, false>(cplx, g.R1, grid, a, s);
  else if (is(Src::dit, Sink::dif, false)) ok = launch_cols<Src::dit, Sink::dif, false>(cplx, g.R1, grid, a, s);
  else if (is(Src::scatter, Sink::dif, false))
    ok = launch_cols<Src::scatter, Sink::dif, false>(cplx, g.R1, grid, a, s);
  else if (is(Src::scatter, Sink::rows, false))
    ok = launch_cols<Src::scatter, Sink::rows, false>(cplx, g.R1, grid, a, s);
  else if (is(Src::dit, Sink::ret, true)) ok = launch_cols<Src::dit, Sink::ret, true>(cplx, g.R1, grid, a, s);
  else if (is(Src::dit, Sink::rows, true)) ok = launch_cols<Src::dit, Sink::rows, true>(cplx, g.R1, grid, a, s);
  else if (is(Src::dit, Sink::dif, true)) ok = launch_cols<Src::dit, Sink::dif, true>(cplx, g.R1, grid, a, s);
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t dif2(float2* Z, long long B, const Geo& g, const float2* tw2, hipStream_t s) {
  return part_pass<false>(Z, B, g, tw2, s);
}
hipError_t dit2(float2* Z, long long B, const Geo& g, const float2* tw2, hipStream_t s) {
  return part_pass<true>(Z, B, g, tw2, s);
}

hipError_t mq(const float* D, const float* Bias, float4* Mq, int K, const Geo& g, const QuartetTabs& q,
              hipStream_t s) {
  // a layer's M / 2 quartets, or one tile's threads where it has fewer
  const long long n = (long long)K * (g.M / 2 > kThreads ? g.M / 2 : kThreads);
  hipLaunchKernelGGL(k_mq, grid_for(n), dim3(kThreads), 0, s, D, Bias, Mq, K, g, q);
  return hipGetLastError();
}

hipError_t seg_fwd(float2* Z, const float4* Mq, long long B, const Geo& g, bool bias, const char* seg_tab,
                   hipStream_t s) {
  const int rb = seg_fwd_rows(B, g, false);
  const bool ok = with_seg_plan<true>(g.L, [&]<class PL>() {
    const dim3 grid = seg_grid<PL>((B + rb - 1) / rb * (g.R1 * g.R2 / 2)), block(Seg<PL>::THREADS);
    if (bias) hipLaunchKernelGGL((k_seg_fwd<PL, true>), grid, block, 0, s, Z, Mq, B, g, rb, seg_tab);
    else hipLaunchKernelGGL((k_seg_fwd<PL, false>), grid, block, 0, s, Z, Mq, B, g, rb, seg_tab);
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t seg_bwd(float2* Zh, float2* Zg, const float4* Mq, long long B, const Geo& g, float* part,
                   const char* seg_tab, hipStream_t s) {
  const int rb = seg_rows(B, g, false);
  const bool ok = with_seg_plan<false>(g.L, [&]<class PL>() {
    hipLaunchKernelGGL(k_seg_bwd<PL>, seg_grid<PL>((B + rb - 1) / rb * (g.R1 * g.R2 / 2)), dim3(Seg<PL>::THREADS), 0,
                       s, Zh, Zg, Mq, B, g, rb, part, seg_tab);
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t seg_dct(const float2* Z, const float4* Mq, int K, const Geo& g, float* gB, bool accumulate,
                   const char* seg_tab, hipStream_t s) {
  const bool ok = with_seg_plan<false>(g.L, [&]<class PL>() {
    hipLaunchKernelGGL(k_seg_dct<PL>, seg_grid<PL>((long long)K * (g.R1 * g.R2 / 2)), dim3(Seg<PL>::THREADS), 0, s, Z,
                       Mq, K, g, gB, accumulate ? 1 : 0, seg_tab);
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t dn(const float2* D, float2* Dn, int K, const Geo& g, hipStream_t s) {
  hipLaunchKernelGGL(k_dn, grid_for((long long)K * g.M), dim3(kThreads), 0, s, D, Dn, K, g, 1.0f / float(g.M));
  return hipGetLastError();
}

hipError_t cseg_fwd(float2* Z, const float2* Dn, long long B, const Geo& g, const char* seg_tab, hipStream_t s) {
  const int rb = seg_fwd_rows(B, g, true);
  const bool ok = with_seg_plan<true>(g.L, [&]<class PL>() {
    hipLaunchKernelGGL(k_cseg_fwd<PL>, seg_grid<PL>((B + rb - 1) / rb * (g.R1 * g.R2)), dim3(Seg<PL>::THREADS), 0, s,
                       Z, Dn, B, g, rb, seg_tab);
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t cseg_bwd(float2* Zh, float2* Zg, const float2* Dn, long long B, const Geo& g, float* part,
                    const char* seg_tab, hipStream_t s) {
  const int rb = seg_rows(B, g, true);
  const bool ok = with_seg_plan<false>(g.L, [&]<class PL>() {
    hipLaunchKernelGGL(k_cseg_bwd<PL>, seg_grid<PL>((B + rb - 1) / rb * (g.R1 * g.R2)), dim3(Seg<PL>::THREADS), 0, s,
                       Zh, Zg, Dn, B, g, rb, reinterpret_cast<float2*>(part), seg_tab);
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t colsum_parts(const float* part, long long P, long long W, float* out, Order how, const Geo& g,
                        const QuartetTabs* q, bool accumulate, hipStream_t s) {
  const QuartetTabs qq = q ? *q : QuartetTabs{};
  const dim3 grid(unsigned((W / 4 + kSumCols - 1) / kSumCols)), block(kThreads);
  const int acc = accumulate ? 1 : 0;
  switch (how) {
    case Order::natural:
      hipLaunchKernelGGL(k_colsum2<Order::natural>, grid, block, 0, s, part, P, W, out, g, qq, acc);
      break;
    case Order::quartets:
      hipLaunchKernelGGL(k_colsum2<Order::quartets>, grid, block, 0, s, part, P, W, out, g, qq, acc);
      break;
    case Order::spectrum:
      hipLaunchKernelGGL(k_colsum2<Order::spectrum>, grid, block, 0, s, part, P, W, out, g, qq, acc);
      break;
  }
  return hipGetLastError();
}

hipError_t colsum(const float* img, long long B, long long W, float* part, float* out, hipStream_t s) {
  Geo g{W / 2, 4096, 2, 1};
  // few rows: one launch, each phase taking the rows of a block
  if (B <= kSumPh * kMaxRows) return colsum_parts(img, B, W, out, Order::natural, g, nullptr, false, s);
  const long long P = (B + kMaxRows - 1) / kMaxRows;
  hipLaunchKernelGGL(k_colsum1, grid_for(P * (W / 4)), dim3(kThreads), 0, s, img, B, W, part);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return colsum_parts(part, P, W, out, Order::natural, g, nullptr, false, s);
}

bool build_seg_table(int L, bool fwd, std::vector<unsigned char>& host) {
  bool ok = false;
  auto build = [&]<class PL>() { ok = build_complex_tables<PL>(host); };
  (void)(fwd ? with_seg_plan<true>(L, build) : with_seg_plan<false>(L, build));
  return ok;
}

}  // namespace mp
}  // namespace acdc
