// Geometry and index algebra of the multi-pass rows: how a row's M-point FFT
// splits, which column set an element belongs to, which segments and values
// pair up, and how many rows and workgroups a launch takes.  Host and device,
// so that the CPU tests run the same code.
#pragma once

#include <initializer_list>

#include "acdc_plans.hpp"

namespace acdc {
namespace mp {

// Geometry of one row's M-point FFT: M = R1 * R2 * L, R1 in {2, 4, 8, 16},
// R2 in {1, 2, ..., 32} (1 = no pass), L the in-LDS segment length: 1024 from M
// = 2048 to 8192, 4096 from 16384 on.  K = 4, forward and backward from the
// stored layer inputs, other lengths against these: M = 4096 in segments of
// 2048 (16 values on each of 128 threads) one row 108 and 210 us, 89 and 134
// so; M = 8192 in segments of 4096 one row 131 and 181 against 98 and 157,
// 1000 rows 479 and 979 against 470 and 963; M = 16384 in segments of 1024 one
// row 130 and 188 against 146 and 199, but 1000 rows 1019 and 1851 against 976
// and 1716.
struct Geo {
  long long M;
  int L, R1, R2;
};
// of real rows of width N (complex rows of N / 2 elements)
inline Geo geo(long long N) {
  Geo g;
  g.M = N / 2;
  g.L = g.M >= 16384 ? 4096 : g.M >= 2048 ? 1024 : int(g.M / 2);
  const long long ratio = g.M / g.L;
  g.R1 = int(ratio <= 16 ? ratio : 16);
  g.R2 = int(ratio / g.R1);
  return g;
}

constexpr int kPermChunk = 16384;                       // floats of a whole column set: 64 KB of LDS
constexpr int kPermMaxChunks = (1 << 22) / kPermChunk;  // the widest row

// Column sets (see "Permutations between column sets", acdc_multipass.hpp).
struct PermGeo {
  int lQ, lw, lC, nC;  // log2 of Q, w, C; sets per row
  int ew;              // floats per element: 1 real, 2 complex
};
inline int log2_of(long long v) {
  int l = 0;
  while ((1LL << (l + 1)) <= v) ++l;
  return l;
}
inline PermGeo perm_geo(const Geo& g, int ew) {
  const long long N = 2 * g.M / ew, cap = kPermChunk / ew;  // elements of a row, of a whole set
  const long long C = N < cap ? N : cap, Q = g.M / g.R1;
  PermGeo p;
  p.ew = ew;
  p.lC = log2_of(C);
  p.nC = int(N / C);
  p.lQ = log2_of(Q);
  p.lw = log2_of(C / (ew == 1 ? 4LL * g.R1 : g.R1));
  return p;
}

// Set of row element i and its place in the LDS image of a column launch
// (chunk or element js of column col at js W + col, W columns for a whole
// set's), and the element at local position l of set d.
__host__ __device__ __forceinline__ void part_of(const PermGeo& p, long long i, int& d, int& l) {
  const int lW = p.lw + (ilog2(kPermChunk) - p.lC) + (p.ew == 1 ? 0 : -1);
  const long long Q = 1LL << p.lQ;
  if (p.ew == 1) {
    const long long q = i >> 2, j = q >> p.lQ, n = q & (Q - 1);
    const int side = n >= Q / 2 ? 1 : 0;
    const long long col = side ? Q - 1 - n : n;
    d = int(col >> p.lw);
    l = int(((((2 * j + side) << lW) + (col & ((1 << p.lw) - 1))) << 2) + (i & 3));
  } else {
    const long long j = i >> p.lQ, n = i & (Q - 1);
    d = int(n >> p.lw);
    l = int((j << lW) + (n & ((1 << p.lw) - 1)));
  }
}
__host__ __device__ __forceinline__ long long elem_of(const PermGeo& p, int d, int l) {
  const long long Q = 1LL << p.lQ;
  if (p.ew == 1) {
    const int l4 = l >> 2, js = l4 >> p.lw;
    const long long col = ((long long)d << p.lw) + (l4 & ((1 << p.lw) - 1));
    const long long n = (js & 1) ? Q - 1 - col : col;
    return ((((long long)(js >> 1) << p.lQ) + n) << 2) + (l & 3);
  }
  return ((long long)(l >> p.lw) << p.lQ) + ((long long)d << p.lw) + (l & ((1 << p.lw) - 1));
}

// Pair p (of S/2) of a real row's segments: Z[k] in one has its Makhoul
// partner Z[M-k] in the other, at L-1-k2.  Pair 0 is the two segments that
// hold their own partners, segment 0 (at L-k2) and one more (at L-1-k2).
__host__ __device__ __forceinline__ void seg_pair(const Geo& g, int p, int& sa, int& sb) {
  if (p == 0) {
    sa = 0;
    sb = g.R2 == 1 ? g.R1 / 2 : g.R2 / 2;
    return;
  }
  int x = p - 1;
  if (x < (g.R1 / 2 - 1) * g.R2) {
    const int r1 = 1 + x / g.R2, r2 = x % g.R2;
    sa = r1 * g.R2 + r2;
    sb = (g.R1 - r1) * g.R2 + (g.R2 - 1 - r2);
    return;
  }
  x -= (g.R1 / 2 - 1) * g.R2;
  if (x < g.R2 / 2) {
    sa = (g.R1 / 2) * g.R2 + x;
    sb = (g.R1 / 2) * g.R2 + (g.R2 - 1 - x);
    return;
  }
  x -= g.R2 / 2;
  sa = 1 + x;
  sb = g.R2 - 1 - x;
}

// Quartet at place k2 of pair p: its number e, where e = 0 is the self-paired
// (Z[0], Z[M/2]) and otherwise Z[e] pairs with Z[M-e].  In a generic pair it
// is the quartet of segment A's k2, in pair 0 those of segment 0 come first
// (k2 < L/2), then the other segment's.
__host__ __device__ __forceinline__ long long quartet_of(const Geo& g, int p, int sa, int k2) {
  const long long S = (long long)g.R1 * g.R2;
  if (p == 0) return k2 < g.L / 2 ? S * k2 : S / 2 + S * (k2 - g.L / 2);
  const long long k = sa / g.R2 + (long long)g.R1 * (sa % g.R2) + S * k2;
  return k < g.M / 2 ? k : g.M - k;
}
__host__ __device__ __forceinline__ long long quartet_of(const Geo& g, int p, int k2) {
  int sa, sb;
  seg_pair(g, p, sa, sb);
  return quartet_of(g, p, sa, k2);
}

// The inverse: pair and place of quartet e.
__host__ __device__ __forceinline__ void quartet_place(const Geo& g, long long e, int& p, int& k2) {
  const int S = g.R1 * g.R2, c = int(e % S), r1 = c % g.R1, r2 = c / g.R1;
  k2 = int(e / S);
  if (c == 0 || c == S / 2) {
    p = 0;
    if (c != 0) k2 += g.L / 2;
    return;
  }
  const int H = 1 + (g.R1 / 2 - 1) * g.R2;  // the first pair inside r1 = R1 / 2
  bool second;                              // e lies in the pair's segment B
  if (r1 == 0) {
    second = r2 > g.R2 / 2;
    p = H + g.R2 / 2 + (second ? g.R2 - 1 - r2 : r2 - 1);
  } else if (r1 == g.R1 / 2) {
    second = r2 >= g.R2 / 2;
    p = H + (second ? g.R2 - 1 - r2 : r2);
  } else {
    second = r1 > g.R1 / 2;
    p = second ? 1 + (g.R1 - r1 - 1) * g.R2 + g.R2 - 1 - r2 : 1 + (r1 - 1) * g.R2 + r2;
  }
  if (second) k2 = g.L - 1 - k2;
}

// Spectrum index of storage position q.
__host__ __device__ __forceinline__ long long spec_index(const Geo& g, long long q) {
  const long long S1 = g.M / g.R1;
  const long long r1 = q / S1, rem = q % S1;
  const long long r2 = rem / g.L, k2 = rem % g.L;
  return r1 + (long long)g.R1 * (r2 + (long long)g.R2 * k2);
}

// Rows per block of the image sums of the segment and column launches: one
// block is one workgroup's loop, so few enough to leave every CU several
// workgroups (kWant in all, two on each of 256 CUs), and at most kMaxRows.
constexpr int kMaxRows = 16;
constexpr long long kWant = 512;
inline int clamp_rows(long long n) { return n < 1 ? 1 : n > kMaxRows ? kMaxRows : int(n); }
inline long long seg_units(const Geo& g, bool cplx) { return g.R1 * g.R2 / (cplx ? 1 : 2); }
inline int seg_rows(long long B, const Geo& g, bool cplx) { return clamp_rows(B * seg_units(g, cplx) / kWant); }
// The forward segment launches keep no sums, so their rows in turn follow the
// threads alone: plans of few threads (8 at L = 64, eight units a workgroup)
// counted by units left most of the chip idle (N = 256, 8000 rows, K = 4: 63
// workgroups of one wave, 150 us a layer).
constexpr int seg_fwd_threads(int L) { return L <= 1024 ? L / 8 : L / 16; }
inline int seg_fwd_rows(long long B, const Geo& g, bool cplx) {
  return clamp_rows(B * seg_units(g, cplx) * seg_fwd_threads(g.L) / (kWant * 256));
}
inline int col_rows(long long B, const Geo& g, int ew) { return clamp_rows(B * perm_geo(g, ew).nC / kWant); }
// An upper bound of the blocks of either for every batch up to B (sizes the
// block sums: a workspace of one batch serves the smaller ones).  With u
// units a row there are at most B blocks, fewer than 2 kWant / u while
// blocks have fewer than kMaxRows rows, and B / kMaxRows from there on.
inline long long max_blocks(long long B, const Geo& g, int ew) {
  long long most = (B + kMaxRows - 1) / kMaxRows;
  for (long long u : {seg_units(g, ew == 2), (long long)perm_geo(g, ew).nC}) {
    const long long few = (2 * kWant + u - 1) / u + 1;
    const long long n = B < few ? B : few;
    most = n > most ? n : most;
  }
  return most;
}

// Threads of a workgroup: 512 at R <= 8 (four waves per SIMD with two
// workgroups a CU); a real row's column pair at R = 16 is 64 values, and a
// set of 16384 floats has 256 pairs.
constexpr int col_threads(int R1, int ew) { return ew == 1 && R1 > 8 ? 256 : 512; }

// Column launch over B rows: a workgroup takes one column set of rw rows side
// by side and rb times as many in turn.
//   rw  Rows of fewer than kPermChunk floats leave columns of a workgroup
//       empty: at N = 256, R1 = 2, a row has 32 column pairs for 512 threads.
//       The launches without image sums fill them with further rows (narrow)
//       while that leaves kWant workgroups.  Forward, K = 4, one row a
//       workgroup and packed: see k_cols.
//   rb  With image sums the rows of their block (col_rows).  The other
//       launches keep nothing from row to row, so one, up to kColGroups
//       workgroups; past that it grows with the batch: HIP takes fewer than
//       2^32 threads a launch, which one workgroup of 512 threads per row
//       reaches at 2^23 rows.
constexpr bool narrow(int R1, bool sums) { return R1 == 2 && !sums; }
constexpr long long kColGroups = 65536;
struct ColGrid {
  int rw, rb, threads;
  long long groups;
};
inline ColGrid col_grid(long long B, const Geo& g, int ew, bool sums) {
  const PermGeo p = perm_geo(g, ew);
  const long long full = narrow(g.R1, sums) ? (kPermChunk / ew) >> p.lC : 1, share = B / kWant;
  const long long rw = share < 1 ? 1 : share < full ? share : full, sets = (B + rw - 1) / rw * p.nC;
  const long long rb = sums ? col_rows(B, g, ew) : (sets + kColGroups - 1) / kColGroups;
  ColGrid c;
  c.rw = int(rw);
  c.rb = int(rb < 1 ? 1 : rb);
  c.threads = col_threads(g.R1, ew);
  c.groups = (B + c.rb * rw - 1) / (c.rb * rw) * p.nC;
  return c;
}

}  // namespace mp
}  // namespace acdc
