// Multi-pass ACDC layers: the M = N/2 point FFT of each row runs through HBM
// in several kernel launches (the multiple-call implementation of Sec. 5.2,
// with hand-written passes in place of a vendor FFT).  Used for widths past
// the fused kernels' on-chip limit, or when ACDC_FLAG_MULTIPASS asks for it.
//
// M = R1 R2 L.  The FFT is a radix-R1 DIF pass over the whole row, a radix-R2
// DIF pass over its R1 parts where R2 > 1, and S = R1 R2 segment FFTs of L
// points; the inverse runs the mirror image.  HBM bandwidth bounds every
// launch, so what counts is how often the batch is read and written:
//   columns   One launch takes a layer from the spectrum of its inverse
//             segment FFTs to the first DIF pass of the next one: DIT pass,
//             ReLU, permutation, stash, * a, DIF pass.  A workgroup holds a
//             set of columns (the same set in the DIT and the DIF), so
//             without a permutation all of it is one launch in registers.  A
//             permutation moves elements between the column sets: the launch
//             is cut in two around it, the first half sending its elements
//             grouped by destination set, the second gathering them in LDS.
//   segments  One launch for the segment FFTs, the layer middle and the
//             segment IFFTs.  The middle of a real row joins Z[k] with
//             Z[M-k]; those lie in two segments (or within two special
//             ones), which one workgroup transforms together (seg_pair).
// A forward layer with a permutation thus takes 3 launches and moves the
// batch 7 times (2 + the stash more than the data needs), a backward layer
// 4 launches and 11 times.  Separate launches for permutation, DIF, segment,
// middle, inverse segment and DIT steps moved it 15 and 24 times.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "acdc_mp_geo.hpp"
#include "acdc_registry.hpp"

namespace acdc {
namespace mp {

// Permutations between column sets.  A set ("chunk") holds the elements of w
// neighbouring columns: for complex rows m = n + j Q (Q = M / R1, j < R1) of
// columns n; for real rows the float4 chunks n + j Q and (Q-1-n) + j Q
// (j < R1/2) of column pairs n, which hold the Makhoul values of butterflies
// n and Q-1-n.  C elements a set, nC sets a row; `local` order is by j (and
// side), then column.
//   send    workgroup (b, c) holds source set c in LDS and writes its values
//           to tmp[b], grouped by destination set d and within it by source
//           set: the C values of set d are tmp[b][dC ...]
//   gather  workgroup (b, d) reads those C values into LDS and picks its
//           elements in local order
// The backward runs the adjoint with the same tables: `ret` (return: the
// elements of set d to their places in tmp[b][dC ...]) and `scatter` (the
// values sourced from set c, back to their places in it).  Every HBM access
// is contiguous, or in runs of C / nC elements.  Table entries are masked
// into range, so a malformed permutation cannot address outside its row.
// Rows of one set (N <= 16384 floats) take the same launches; their list
// follows the destinations.
//
// One layer's tables (layer l's sit stride ints further on):
//   item[cC + i]   entry i of set c's list, ordered by destination set d:
//                  (local source index << 8) | d
//   delta[c][d]    tmp position of entry i bound for set d: i + delta
//   loc[dC + l]    position in d's C values of tmp of the element at local l
struct PermTabs {
  unsigned* item = nullptr;
  unsigned short* loc = nullptr;
  int* delta = nullptr;
  int *cntS = nullptr, *bpre = nullptr;                    // [N / 256][nC]
  int *cnt = nullptr, *start = nullptr, *lst = nullptr;    // [nC][nC]
  long long stride = 0;
};
size_t perm_table_ints(const Geo& g, int ew);  // per layer
PermTabs perm_tables_at(int* base, const Geo& g, int ew);
PermTabs perm_layer(const PermTabs& t, int l);
// Tables of the permutations perm[0 .. layers-1][N] into layers 0 .. layers-1.
hipError_t perm_build(const int* perm, const Geo& g, int ew, int layers, const PermTabs& t, hipStream_t s);

// Column launches.  The source is rows in memory, tmp through a permutation
// table, or the spectrum Z (DIT pass); the sink rows, tmp, or Z (DIF pass).
// Forward: ReLU after the DIT (relu), then stash and * a before the DIF
// (either may be null).  Backward (with u): g is masked where mask (relu)
// and u <= 0, the dL/da images u * g (complex: g * conj(u)) are summed over blocks of rb
// rows into part[ceil(B / rb)][row], and g * conj(a) goes on.
enum class Src { rows, gather, scatter, dit };
enum class Sink { rows, send, ret, dif };
struct Cols {
  const float* src = nullptr;
  float* dst = nullptr;
  float2* Z = nullptr;
  const float* a = nullptr;
  float* stash = nullptr;
  const float* u = nullptr;
  float* part = nullptr;
  const PermTabs* pt = nullptr;
  int relu = 0;
};
hipError_t cols(Src src, Sink sink, bool cplx, const Cols& c, long long B, const Geo& g, const float2* tw1,
                hipStream_t s);

// Second-level DIF / DIT passes, in place (nothing to do when R2 = 1).
hipError_t dif2(float2* Z, long long B, const Geo& g, const float2* tw2, hipStream_t s);
hipError_t dit2(float2* Z, long long B, const Geo& g, const float2* tw2, hipStream_t s);

// Segment launches, in place.
// Real rows: Mq holds the quartet coefficients of all layers in the order
// the segment kernels read them, [K][pair][kMqRows][k2] (mq).
hipError_t mq(const float* D, const float* Bias, float4* Mq, int K, const Geo& g, const QuartetTabs& q,
              hipStream_t s);
hipError_t seg_fwd(float2* Z, const float4* Mq, long long B, const Geo& g, bool bias, const char* seg_tab,
                   hipStream_t s);
// dL/dd images summed over blocks of seg_rows() rows into part[P][N], and
// Zg <- the inverse FFT's segments of DCT-III's input.
hipError_t seg_bwd(float2* Zh, float2* Zg, const float4* Mq, long long B, const Geo& g, float* part,
                   const char* seg_tab, hipStream_t s);
// gB[k] (+)= the DCT-II whose spectrum after the DIF passes is Z[k], one row
// per layer; Mq as above (all K layers).
hipError_t seg_dct(const float2* Z, const float4* Mq, int K, const Geo& g, float* gB, bool accumulate,
                   const char* seg_tab, hipStream_t s);
// Complex rows: Dn holds d / N of all layers in storage order, [K][M] (dn).
hipError_t dn(const float2* D, float2* Dn, int K, const Geo& g, hipStream_t s);
hipError_t cseg_fwd(float2* Z, const float2* Dn, long long B, const Geo& g, const char* seg_tab, hipStream_t s);
hipError_t cseg_bwd(float2* Zh, float2* Zg, const float2* Dn, long long B, const Geo& g, float* part,
                    const char* seg_tab, hipStream_t s);

// Fixed-order sums over row blocks: out[w] (+)= sum over p of part[p][w] in
// block order, column w being in the order of the launch that wrote it.
// `how`: natural (dL/da), real segment order (quartets, to their DCT
// indices) or complex segment order.
enum class Order { natural, quartets, spectrum };
hipError_t colsum_parts(const float* part, long long P, long long W, float* out, Order how, const Geo& g,
                        const QuartetTabs* q, bool accumulate, hipStream_t s);
// out[w] = sum over the B rows of img[b][w]: blocks of kMaxRows rows into
// part, then the block sums (up to 128 rows the rows themselves in their
// place).  W is a multiple of 4.
hipError_t colsum(const float* img, long long B, long long W, float* part, float* out, hipStream_t s);

// Constant table of the segment plan of L points (fill: host bytes): the
// forward launches' (seg_fwd, cseg_fwd), or the other launches'.
bool build_seg_table(int L, bool fwd, std::vector<unsigned char>& host);

}  // namespace mp
}  // namespace acdc
