// One Markov-clustering iteration (a8; paper §5.7) on X = M^T in CSR, FP32,
// in one of two step orders:
//   rpost == 0 (the synthetic workload's order):
//     E = X X;  e <- e^r;  row /= row sum;  drop e < prune;  keep the topk
//     largest (ties to the smaller column);  an emptied row keeps its
//     largest entry;  row /= new row sum.
//   rpost >= 1 (the order the paper describes for its runs):
//     E = X X;  row /= row sum;  drop e < prune;  top-k and emptied rows as
//     above;  e <- e^rpost;  no second normalisation.
// Both are the same kernels with the exponent before the normalisation
// (rpre = r, or 1) and the final step (renormalise, or the power) as
// parameters.
// The unpruned product is never stored.  Row c of Y is written at its final
// column rank into a padded buffer (cap = min(topk, n) slots per row) with
// its length in cnt[c]; a scan of cnt and a compaction copy produce CSR.
//
// Rows whose products fit an LDS table use the numeric kernel's
// order-preserving hash (rank = occupied slots before + inversion counter)
// and run the whole epilogue in LDS; kept entries are flagged by clearing
// the sign of their value slot.  Rows beyond the tables are swept in column
// panels (k_mcl_panel below).
#include <float.h>

#include <vector>

#include "internal.hpp"
#include "rowops.hpp"

namespace spg {

constexpr int kMclUnroll = 4;

__device__ __forceinline__ float ipow(float e, int r) {
  float p = e;
  for (int q = 1; q < r; ++q) p *= e;
  return p;
}

// (value, column) -> orderable key: larger value first, then smaller column
// (values are >= 0, so their bit patterns order like the values).
__device__ __forceinline__ unsigned long long vc_key(float v, int col) {
  return ((unsigned long long)__float_as_uint(v) << 32) | (uint32_t)(~(uint32_t)col);
}

template <int G>
struct MGeom {
  static constexpr bool BLOCK = G > kWave;
  static constexpr int WG = BLOCK ? G : 256;
  static constexpr int R = WG / G;
};

// Batched insert of the expansion products (first probes of all N issued
// together).  Wave groups store the value of a column's first insert and add
// repeats after a wave fence (LDS float atomics are slow), so their value
// table needs no clearing; block groups add atomically into a cleared table.
template <bool PLAIN>
struct MclInsert {
  int *key;
  float *val;
  int *flag;
  uint32_t mul;
  int maxwin;
  template <int N>
  __device__ __forceinline__ void batch(const int (&col)[N], const float (&v)[N]) {
    int h[N], old[N];
    bool ok[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      h[u] = (int)mono_slot((uint32_t)col[u], mul);
      old[u] = col[u] >= 0 ? atomicCAS(&key[h[u]], kEmpty, (int)((uint32_t)col[u] | 0x80000000u))
                           : kEmpty;
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      ok[u] = col[u] >= 0;
      int d = 0;
      while (ok[u] && old[u] != kEmpty && (int)((uint32_t)old[u] & 0xffffffu) != col[u]) {
        if (d == maxwin) {  // the heavy kernel redoes this row
          *flag = 1;
          ok[u] = false;
          break;
        }
        ++d;
        ++h[u];
        old[u] = atomicCAS(&key[h[u]], kEmpty, (int)((uint32_t)col[u] | 0x80000000u));
      }
    }
    if (PLAIN) {
#pragma unroll
      for (int u = 0; u < N; ++u)
        if (ok[u] && old[u] == kEmpty) val[h[u]] = v[u];
      group_sync<false>();
#pragma unroll
      for (int u = 0; u < N; ++u)
        if (ok[u] && old[u] != kEmpty) lds_add_cas(&val[h[u]], v[u]);
    } else {
#pragma unroll
      for (int u = 0; u < N; ++u)
        if (ok[u]) lds_add_cas(&val[h[u]], v[u]);
    }
  }
};

constexpr int32_t kMclPending = -1;  // row length of a row that k_mcl_few gave back

// LDS rows.  Key words pack (col | (128 + counter) << 24), n <= 2^24.
template <int G>
__global__ __launch_bounds__(MGeom<G>::WG) void k_mcl_rows(
    const Problem *__restrict__ pr, const int32_t *__restrict__ rows, WsHeader *__restrict__ hdr,
    int bin, int lS, int TT, uint32_t mul, int maxwin, int r, int rpost, float prune, int topk,
    int cap,
    int32_t *__restrict__ ycol, float *__restrict__ yval, int32_t *__restrict__ ycnt,
    int32_t *__restrict__ fb_rows, const int32_t *__restrict__ failed) {
  using GM = MGeom<G>;
  constexpr bool BLOCK = GM::BLOCK;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ float redf[16];
  __shared__ int redi[16];
  __shared__ unsigned long long redu[16];
  const int rslot = threadIdx.x / G, l = threadIdx.x % G;
  float *vals_all = reinterpret_cast<float *>(smem_raw);
  float *sa_all = vals_all + (size_t)GM::R * TT;
  int *keys_all = reinterpret_cast<int *>(sa_all + (size_t)GM::R * G);
  int *sb_all = keys_all + (size_t)GM::R * TT;
  int *sl_all = sb_all + (size_t)GM::R * G;
  int *rowflag = sl_all + (size_t)GM::R * G;
  float *val = vals_all + (size_t)rslot * TT;
  int *key = keys_all + (size_t)rslot * TT;
  Stage<float> st{sb_all + rslot * G, sl_all + rslot * G, sa_all + rslot * G};
  if (hdr->status) return;
  const int count = hdr->bin_count[bin];
  const int start = hdr->bin_start[bin];
  const int c = TT / G;
  const int s0 = l * c;
  // after k_mcl_few: the rows it did not take, and those it gave back
  const int taken = failed ? min(count, hdr->queue[bin]) : 0;
  const int first = failed && failed[bin] == 0 ? taken : 0;
  for (int ri = first + blockIdx.x * GM::R + rslot; ri < count; ri += gridDim.x * GM::R) {
    int i = rows[start + ri];
    if (ri < taken && ycnt[i] != kMclPending) continue;
    if (G >= kWave) i = __builtin_amdgcn_readfirstlane(i);
    int4 *k4 = reinterpret_cast<int4 *>(key);
    for (int s = l; s < TT / 4; s += G) k4[s] = make_int4(kEmpty, kEmpty, kEmpty, kEmpty);
    if (BLOCK)
      for (int s = l; s < TT; s += G) val[s] = 0.f;
    if (l == 0) rowflag[rslot] = 0;
    group_sync<BLOCK>();
    // 1. expansion E = X X (accumulate row i)
    MclInsert<!BLOCK> fins{key, val, rowflag + rslot, mul, maxwin};
    for_each_product<BLOCK, true, G, kMclUnroll, float>(pr, i, true, l, lS, st, fins);
    group_sync<BLOCK>();
    if (rowflag[rslot]) {  // redone by the heavy kernel
      if (l == 0) fb_rows[atomicAdd(&hdr->fallback_count, 1)] = i;
      group_sync<BLOCK>();
      continue;
    }
    // 2. inflation and row sum
    float part = 0.f;
    for (int j = 0; j < c; ++j) {
      if (key[s0 + j] != kEmpty) {
        const float p = ipow(val[s0 + j], r);
        val[s0 + j] = p;
        part += p;
      }
    }
    const float S = group_sum<BLOCK, G>(part, redf);
    // 3./4. normalise and prune; kept entries have a clear sign bit
    int kept = 0;
    unsigned long long best = 0;
    for (int j = 0; j < c; ++j) {
      const int w = key[s0 + j];
      if (w != kEmpty) {
        const float v = val[s0 + j] / S;
        const unsigned long long kk = vc_key(v, (int)((uint32_t)w & 0xffffffu));
        best = kk > best ? kk : best;
        if (v < prune) {
          val[s0 + j] = -v - 1.f;  // dropped (keeps v recoverable)
        } else {
          val[s0 + j] = v;
          ++kept;
        }
      }
    }
    const int nkept = group_sum<BLOCK, G>(kept, redi);
    if (nkept > topk) {
      // 5. threshold: the largest bit pattern tau with #{kept v >= tau} >= topk
      uint32_t lo = 0, hi = 0x7f800000u;
      while (lo < hi) {
        const uint32_t mid = lo + (hi - lo + 1) / 2;
        int cc = 0;
        for (int j = 0; j < c; ++j) {
          const float v = val[s0 + j];
          cc += (key[s0 + j] != kEmpty && v >= 0.f && __float_as_uint(v) >= mid) ? 1 : 0;
        }
        if (group_sum<BLOCK, G>(cc, redi) >= topk) lo = mid;
        else hi = mid - 1;
      }
      int gt = 0;
      for (int j = 0; j < c; ++j) {
        const float v = val[s0 + j];
        gt += (key[s0 + j] != kEmpty && v >= 0.f && __float_as_uint(v) > lo) ? 1 : 0;
      }
      const int need = topk - group_sum<BLOCK, G>(gt, redi);
      // ties at tau: keep the `need` smallest columns
      for (int j = 0; j < c; ++j) {
        const int w = key[s0 + j];
        const float v = val[s0 + j];
        if (w == kEmpty || v < 0.f) continue;
        const uint32_t b = __float_as_uint(v);
        bool keep = b > lo;
        if (b == lo) {
          const int col = (int)((uint32_t)w & 0xffffffu);
          int before = 0;
          for (int t = 0; t < TT; ++t) {
            const int w2 = key[t];
            const float v2 = val[t];
            if (w2 != kEmpty && v2 >= 0.f && __float_as_uint(v2) == lo &&
                (int)((uint32_t)w2 & 0xffffffu) < col)
              ++before;
          }
          keep = before < need;
        }
        if (!keep) val[s0 + j] = -v - 1.f;
      }
    }
    group_sync<BLOCK>();
    // 6. never empty: keep the largest entry of step 3
    if (nkept == 0) {
      const unsigned long long bb = group_max_u64<BLOCK, G>(best, redu);
      const int bcol = (int)~(uint32_t)(bb & 0xffffffffu);
      for (int j = 0; j < c; ++j) {
        const int w = key[s0 + j];
        if (w != kEmpty && (int)((uint32_t)w & 0xffffffu) == bcol) val[s0 + j] = -val[s0 + j] - 1.f;
      }
    }
    group_sync<BLOCK>();
    // 7. new row sum; counters of the kept entries' order
    float part2 = 0.f;
    for (int j = 0; j < c; ++j) {
      const int w = key[s0 + j];
      if (w != kEmpty) {
        key[s0 + j] = (int)(((uint32_t)w & 0xffffffu) | 0x80000000u);  // counter := 0
        if (val[s0 + j] >= 0.f) part2 += val[s0 + j];
      }
    }
    const float S2 = group_sum<BLOCK, G>(part2, redf);
    group_sync<BLOCK>();
    for (int j = 0; j < c; ++j) {
      const int s = s0 + j;
      const int w = key[s];
      if (w == kEmpty || val[s] < 0.f) continue;
      const int col = (int)((uint32_t)w & 0xffffffu);
      const int home = (int)mono_slot((uint32_t)col, mul);
      int larger = 0;
      for (int t = home; t < s; ++t) {
        const int w2 = key[t];
        if (val[t] >= 0.f && (int)((uint32_t)w2 & 0xffffffu) > col) {
          atomicAdd(&key[t], 1 << 24);
          ++larger;
        }
      }
      if (larger) atomicSub(&key[s], larger << 24);
    }
    group_sync<BLOCK>();
    int mine = 0;
    for (int j = 0; j < c; ++j) mine += (key[s0 + j] != kEmpty && val[s0 + j] >= 0.f) ? 1 : 0;
    int total;
    int rk = group_excl_scan<BLOCK, G>(mine, l, redi, total);
    SPG_GLOBAL int32_t *cb = gpw(ycol) + (size_t)i * cap;
    SPG_GLOBAL float *vb = gpw(yval) + (size_t)i * cap;
    for (int j = 0; j < c; ++j) {
      const int w = key[s0 + j];
      const float v = val[s0 + j];
      if (w != kEmpty && v >= 0.f) {
        int rr = rk + (int)((uint32_t)w >> 24) - 128;
        rr = rr < 0 ? 0 : (rr >= cap ? cap - 1 : rr);
        cb[rr] = (int)((uint32_t)w & 0xffffffu);
        vb[rr] = rpost == 0 ? v / S2 : ipow(v, rpost);
        ++rk;
      }
    }
    if (l == 0) ycnt[i] = total < cap ? total : cap;
    group_sync<BLOCK>();
  }
}

// ---------------------------------------------------------------------------
// Rows of many products on few columns (an iteration that has found its
// clusters: the B rows of a cluster hold the same columns).  One block of 256
// threads per row; at most kFewCols columns in an LDS hash with 64-bit
// fixed-point accumulators (the scale as for the panel kernel below, so sums
// do not depend on the order of the adds), products numbered over the row's
// entries as in k_num_sort, so that every thread has four of them in flight.
// A row with more columns is given back to k_mcl_rows (its length is set to
// kMclPending), and so is one that FP32 sums serve better: an entry's error is
// half a unit (2^-61 of the row's bound at most) per product, so a kept entry
// of less than 2^24 units could lose more than FP32 sums do; and rows whose
// sum is zero or whose products may not be finite.
//
// Which bins are tried: 64 rows spread over a bin's list are looked at
// beforehand (k_row_abs), and where more than a quarter of them have too many
// columns the whole bin is left to k_mcl_rows; so is the rest of a bin when a
// quarter of the rows taken so far came back.  Without the look up to 16384
// rows of a bin (eight a block) are under way before one comes back: on 2^19
// unclustered vertices (MCL iterations 1, 6 and 7, prune 1e-4) 0.3 ms a bin,
// and 7.1 ms for rows of 8193..16384 products while a row with too many
// columns also filled the table and walked it.
//
// k_mcl_rows sizes its table by the products, holds one row per CU, and its
// float compare-and-swap adds collide.  2^16 rows in clusters of 64 (4356
// products, 64 columns a row): 6.60 ms there, 1.06 here
// (2000 vector instructions a wave and row issue 90 % of the time; one row
// per atomic on the queue: 3.93 ms).
constexpr int kFewNT = 256;
constexpr int kFewSlots = 1024;
constexpr int kFewCols = 512;
static_assert(kFewCols + kFewNT < kFewSlots, "a slot stays empty");
constexpr int kFewWords = 256;  // marks of 8192 products at a time
constexpr int kFewBin = 6;      // first bin tried: 257..512 products, which always fit
constexpr int kFewSample = 64;  // rows of a bin looked at beforehand
constexpr int kFewLook = 1024;  // products of such a row
constexpr int kFewTry = 512;    // rows taken before the share given back counts
constexpr int kFewTake = 8;     // rows per atomic on the queue (12 ns each on one word)
constexpr size_t kFewSampleAt = 2048;  // the sample's answers in the workspace, below the row bins
static_assert(kFewSample == kWave, "one answer a lane");
static_assert(kFewSampleAt + (kMaxLdsBin - kFewBin + 1) * kFewSample * 4 <= 4096 &&
                  256 + sizeof(Problem) <= kFewSampleAt,
              "room behind the header and the operand descriptors");

// Whether the table holds more than kFewCols columns.  The number is read anew
// before every column that enters, so at most one per thread enters past it:
// the table never fills, and walks stay short in rows that are given back.
__device__ __forceinline__ bool few_full(const int *ncols) {
  return __hip_atomic_load(ncols, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > kFewCols;
}

// The slot of a column from slot h on, taken if need be.
__device__ __forceinline__ uint32_t few_slot(int col, uint32_t h, int *key, int *ncols) {
  for (int probes = 0; probes < kFewSlots; ++probes) {
    int k = key[h];
    if (k == kEmpty) {
      k = atomicCAS(&key[h], kEmpty, col);
      if (k == kEmpty) atomicAdd(ncols, 1);
    }
    if (k == kEmpty || k == col) break;
    h = (h + 1) & (kFewSlots - 1);
  }
  return h;
}

// Whether row i has more than kFewCols columns (1), by its first products (at
// least kFewLook, or all): one block, its table and counter.
__device__ __forceinline__ int few_look(const Part &P, int i, int *key, int *ncols) {
  const int tid = threadIdx.x, lane = lane_id();
  if (tid == 0) *ncols = 0;
  for (int s = tid; s < kFewSlots; s += kFewNT) key[s] = kEmpty;
  __syncthreads();
  int as, ae;
  a_row(P, i, as, ae);
  const int nA = ae - as;
  int seen = 0;
  for (int e = tid / kWave; e < nA && seen < kFewLook / (kFewNT / kWave);
       e += kFewNT / kWave) {
    const int k = gp(P.acol)[as + e];
    const int b0 = gp(P.brp)[k], len = gp(P.brp)[k + 1] - b0;
    for (int q = lane; q < len; q += kWave) {
      const int col = gp(P.bcol)[b0 + q];
      const uint32_t h = scramble_slot((uint32_t)col, 10);
      if (key[h] != col && !few_full(ncols)) (void)few_slot(col, h, key, ncols);
    }
    seen += len;
  }
  __syncthreads();
  return *ncols > kFewCols ? 1 : 0;
}

struct FewEntry {
  float a;
  int b;  // first B position less the number of its first product
};

__global__ __launch_bounds__(kFewNT, 8) void k_mcl_few(
    const Problem *__restrict__ pr, const int32_t *__restrict__ rows, WsHeader *__restrict__ hdr,
    int bin, int r, int rpost, float prune, int topk, int cap, const double *__restrict__ rabs,
    int32_t *__restrict__ ycol, float *__restrict__ yval, int32_t *__restrict__ ycnt,
    int32_t *__restrict__ failed, const int32_t *__restrict__ sample) {
  __shared__ unsigned long long acc[kFewSlots];
  __shared__ int key[kFewSlots];
  __shared__ FewEntry ent[kFewNT];
  __shared__ uint32_t mark[kFewWords];
  __shared__ int wpre[kFewWords];
  __shared__ int wtot[kFewNT / kWave];
  __shared__ double redd[kFewNT / kWave];
  __shared__ int redi[kFewNT / kWave];
  __shared__ unsigned long long redu[kFewNT / kWave];
  __shared__ __align__(16) int kcol[kFewCols + 4];
  __shared__ int ncols, nlist, item;
  if (hdr->status) return;
  const int count = hdr->bin_count[bin];
  const int start = hdr->bin_start[bin];
  const int tid = threadIdx.x;
  {
    const int looked = min(count, kFewSample), lane = lane_id();
    const int wide = lane < looked ? sample[(bin - kFewBin) * kFewSample + lane] : 0;
    if (__popcll(__ballot(wide)) * 4 > looked) return;  // left to k_mcl_rows
  }
  const Part &P = pr->part[0];
  const SPG_GLOBAL int32_t *brp = gp(P.brp);
  const SPG_GLOBAL int32_t *bcol = gp(P.bcol);
  const SPG_GLOBAL float *bval = gp(static_cast<const float *>(P.bval));
  constexpr int U = 4;
  int it = 0, it1 = 0;  // rows taken from the queue, kFewTake at a time
  while (true) {
    __syncthreads();
    if (tid == 0) {
      if (it == it1) {
        const int bad = __hip_atomic_load(&failed[bin], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        item = bad * 4 > max(kFewTry, it1) ? count : atomicAdd(&hdr->queue[bin], kFewTake);
      }
      ncols = 0;
      nlist = 0;
    }
    for (int s = tid; s < kFewSlots; s += kFewNT) {
      acc[s] = 0ull;
      key[s] = kEmpty;
    }
    __syncthreads();
    if (it == it1) {
      it = item;
      it1 = min(count, it + kFewTake);
    }
    if (it >= count) return;
    const int i = rows[start + it++];
    int row0, row1;
    a_row(P, i, row0, row1);
    const uint32_t as = (uint32_t)row0, ae = (uint32_t)row1;  // a row may end at entry 2^31 - 1
    // the scale: 2^(62 - ex) with the row's bound on sum |a b| below 2^ex
    double sb = 0.0;
    for (uint32_t e = as + tid; e < ae; e += kFewNT)
      sb += fabs((double)gp(static_cast<const float *>(P.aval))[e]) * rabs[gp(P.acol)[e]];
    const double bound = group_sum<true, kFewNT>(sb, redd) * (1.0 + 1.0 / 1048576.0);
    int ex = 0;
    (void)frexp(bound, &ex);
    const double sigma = ldexp(1.0, 62 - ex);
    const double inv_sigma = 1.0 / sigma;  // exact: a power of two
    auto give_back = [&] {
      if (tid == 0) {
        ycnt[i] = kMclPending;
        atomicAdd(&failed[bin], 1);
      }
    };
    if (!(bound > 0.0 && bound < (double)FLT_MAX)) {  // no product overflows below
      give_back();
      continue;
    }
    // 1. expansion, chunks of kFewNT entries, 8192 products at a time
    for (uint32_t c0 = as; c0 < ae && ncols <= kFewCols; c0 += kFewNT) {
      int b0 = 0, len = 0;
      float a = 0.f;
      if (c0 + tid < ae) {
        const int k = gp(P.acol)[c0 + tid];
        a = gp(static_cast<const float *>(P.aval))[c0 + tid];
        b0 = brp[k];
        len = brp[k + 1] - b0;
      }
      int tot, live;
      const int off = group_excl_scan<true, kFewNT>(len, tid, wtot, tot);
      const int rank = group_excl_scan<true, kFewNT>(len > 0 ? 1 : 0, tid, wtot, live);
      if (len > 0) ent[rank] = FewEntry{a, b0 - off};
      for (int w0 = 0; w0 < tot && ncols <= kFewCols; w0 += kFewWords * 32) {
        // bit p - w0: product p is the last of its entry
        mark[tid] = 0u;
        __syncthreads();
        const int last = off + len - 1 - w0;
        if (len > 0 && last >= 0 && last < kFewWords * 32)
          atomicOr(&mark[last >> 5], 1u << (last & 31));
        const int before = __syncthreads_count(len > 0 && last < 0);  // entries done
        int all;
        wpre[tid] = before + group_excl_scan<true, kFewNT>(__popc(mark[tid]), tid, wtot, all);
        __syncthreads();
        const int hi = min(tot - w0, kFewWords * 32);
        for (int p0 = tid; p0 < hi; p0 += U * kFewNT) {
          int col[U];
          float v[U];
          FewEntry en[U];
          bool in[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int p = p0 + u * kFewNT;
            in[u] = p < hi;
            const int pc = in[u] ? p : 0;
            en[u] = ent[wpre[pc >> 5] + __popc(mark[pc >> 5] & ((1u << (pc & 31)) - 1u))];
            en[u].b += w0 + pc;
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            col[u] = bcol[en[u].b];
            v[u] = bval[en[u].b];
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (!in[u]) continue;
            uint32_t h = scramble_slot((uint32_t)col[u], 10);
            if (key[h] != col[u] && !few_full(&ncols)) h = few_slot(col[u], h, key, &ncols);
            const long long q = __double2ll_rn((double)(en[u].a * v[u]) * sigma);
            atomicAdd(&acc[h], (unsigned long long)q);
          }
          if (ncols > kFewCols) break;
        }
        __syncthreads();
      }
    }
    __syncthreads();
    if (ncols > kFewCols) {
      give_back();
      continue;
    }
    // 2.-4. inflation, row sum, prune (thread t: slots t + 256 j)
    constexpr int J = kFewSlots / kFewNT;
    int sc[J];
    float sv[J];
    double part = 0.0;
    bool weak[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int s = tid + j * kFewNT;
      sc[j] = key[s];
      weak[j] = acc[s] + (1ull << 24) < (2ull << 24);  // fewer than 2^24 units either way
      sv[j] = ipow((float)((double)(long long)acc[s] * inv_sigma), r);
      part += sc[j] != kEmpty ? (double)sv[j] : 0.0;
    }
    const float S = (float)group_sum<true, kFewNT>(part, redd);
    unsigned long long best = 0;
    int kept = 0;
    bool keep[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const unsigned long long kk = vc_key(sv[j] / S, sc[j]);
      sv[j] = sv[j] / S;
      keep[j] = sc[j] != kEmpty && !(sv[j] < prune);
      if (sc[j] != kEmpty && kk > best) best = kk;
      kept += keep[j] ? 1 + (weak[j] ? 1 << 16 : 0) : 0;  // weak ones in the upper half
    }
    const int nkept = group_sum<true, kFewNT>(kept, redi);
    if (nkept >> 16 || !(S > 0.f && S <= FLT_MAX)) {
      give_back();
      continue;
    }
    if (nkept > topk) {
      // 5. the largest bit pattern tau with at least topk kept values >= tau;
      //    ties at tau: the smallest columns
      uint32_t lo = 0, hi = 0x7f800000u;
      while (lo < hi) {
        const uint32_t mid = lo + (hi - lo + 1) / 2;
        int cc = 0;
#pragma unroll
        for (int j = 0; j < J; ++j) cc += keep[j] && __float_as_uint(sv[j]) >= mid ? 1 : 0;
        if (group_sum<true, kFewNT>(cc, redi) >= topk) lo = mid;
        else hi = mid - 1;
      }
      int gt = 0;
#pragma unroll
      for (int j = 0; j < J; ++j) gt += keep[j] && __float_as_uint(sv[j]) > lo ? 1 : 0;
      const int need = topk - group_sum<true, kFewNT>(gt, redi);
      // columns at tau, listed
#pragma unroll
      for (int j = 0; j < J; ++j)
        if (keep[j] && __float_as_uint(sv[j]) == lo) kcol[atomicAdd(&nlist, 1)] = sc[j];
      __syncthreads();
      const int nt = nlist;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        if (!keep[j]) continue;
        const uint32_t b = __float_as_uint(sv[j]);
        int before = 0;
        if (b == lo)
          for (int t = 0; t < nt; ++t) before += kcol[t] < sc[j] ? 1 : 0;
        keep[j] = b > lo || (b == lo && before < need);
      }
      __syncthreads();
      if (tid == 0) nlist = 0;
      __syncthreads();
    }
    if (nkept == 0) {  // 6. never empty: the largest entry
      const unsigned long long bb = group_max_u64<true, kFewNT>(best, redu);
      const int bcolm = (int)~(uint32_t)(bb & 0xffffffffu);
#pragma unroll
      for (int j = 0; j < J; ++j) keep[j] = sc[j] != kEmpty && sc[j] == bcolm;
      bool w = false;
#pragma unroll
      for (int j = 0; j < J; ++j) w = w || (keep[j] && weak[j]);
      if (__syncthreads_or(w)) {
        give_back();
        continue;
      }
    }
    // 7. the kept columns' new sum and order: rank = kept columns below
    double part2 = 0.0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if (keep[j]) {
        kcol[atomicAdd(&nlist, 1)] = sc[j];
        part2 += (double)sv[j];
      }
    }
    const float S2 = (float)group_sum<true, kFewNT>(part2, redd);
    const int total = nlist;
    if (tid < 4) kcol[total + tid] = INT32_MAX;
    __syncthreads();
    SPG_GLOBAL int32_t *cb = gpw(ycol) + (size_t)i * cap;
    SPG_GLOBAL float *vb = gpw(yval) + (size_t)i * cap;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if (!keep[j]) continue;
      int rk = 0;
      for (int t = 0; t < total; t += 4) {
        const int4 c4 = *reinterpret_cast<const int4 *>(kcol + t);
        rk += (c4.x < sc[j]) + (c4.y < sc[j]) + (c4.z < sc[j]) + (c4.w < sc[j]);
      }
      if (rk < cap) {
        cb[rk] = sc[j];
        vb[rk] = rpost == 0 ? sv[j] / S2 : ipow(sv[j], rpost);
      }
    }
    if (tid == 0) ycnt[i] = total < cap ? total : cap;
  }
}

// ---------------------------------------------------------------------------
// Heavy rows: column panels with fixed-point accumulators in LDS.
//
// A heavy row (more products than an LDS table holds, or handed over by the
// LDS kernel) is swept in panels of kPanel consecutive columns.  Every entry
// a_ik of X row i keeps a cursor into B row k (sorted, as X is canonical).
// In a panel, S lanes of a wave read S consecutive elements of one entry's B
// row (coalesced), a wave serves several entries at once so that several loads
// are in flight, and a ballot over the S lanes tells how far the entry got
// (elements are ascending, so those inside the panel are a prefix).  S is
// chosen per row from the mean number of elements an entry has per panel.
// A product a_ik * b_kj (exact in FP64) is scaled
// by 2^s and rounded to an int64 that is added into the panel's LDS slot with
// an integer atomic: integer LDS atomics are far cheaper than float ones on
// this chip, and the sum no longer depends on the order of the adds.  The
// scale is chosen per row from sum_k |a_ik| * sum_j |b_kj| (row_abs below) so
// that no partial sum can overflow; the rounding error of an entry is at most
// (terms) * 2^-62 of that bound, far below the FP32 rounding of the result.
//
// After a panel, its columns are inflated (p = v^r) and p is summed into the
// row's running sum.  A column can only survive the prune if p >= prune *
// (final sum) >= prune * (sum of the panels before, or of the first one), so
// only such candidates are appended, in column order, to the row's list in
// the slot scratch (capacity n).  At the end the exact test on p / sum moves
// the kept entries to LDS, the top-k threshold is found there by an eight-way
// search on the float bit patterns, ties go to the smaller columns, and the
// result is renormalised and written in column order.  (More kept entries
// than a panel has columns, or none: the same on the list in place.)
//
// 2^17 rows of 400 entries (160000 products a row), per call: 136 -> 89 ms.
// Of these the accumulation takes 55, bound by its reads (every panel reads
// three lines per entry and array, 336 GB in all; generic pointers to the
// entries' cursors made flat loads there, which waited for each other: 38 ms
// more with them in the loop), the panels' ends 14 (30 with lanes 16 columns
// apart, on two banks, and every value computed twice), the selection 16 (48
// with a block-wide reduction per 1024 entries and bisection step).
constexpr int kPanel = 16384;  // columns per panel: 128 KiB of int64 in LDS
constexpr int kPT = 1024;      // threads of a heavy block
constexpr int kCPT = kPanel / kPT;  // panel columns per thread in the epilogue
// Entry groups a wave serves at once, for rows whose entries have 32 or more
// elements per panel (32 or 64 lanes per entry) and for others (4, 6 and 8
// groups for the first: 1 to 4 % slower).
constexpr int kPUDense = 5, kPUSparse = 4;
constexpr int kPE = 1024;     // entries whose cursors stay in LDS
static_assert(kCPT == 16, "a thread's columns are half a bitmap word");
// Rows with fewer products per panel than this look only at the columns that
// the bitmap marks, two passes over them, instead of at all 16 of a thread:
// 10^5 and 10^4 products a row on 2^19 columns (MCL, iterations 5 and 6, the
// second mostly of such rows) take 704 and 201 ms, 701 and 237 with all rows
// dense; at 3072, with rows of 2500 per panel among them, 710 and 200.
constexpr int kSparse = 1536;

struct PanelRed {
  double s;
  int total, excl, mn;
  unsigned long long best;
};

// Block-wide sum (double), inclusive/exclusive count scan, min and max in one
// barrier.  The caller synchronises before the shared arrays are reused.
__device__ __forceinline__ PanelRed panel_reduce(double s, int c, int mn, unsigned long long best,
                                                 double *rs, int *rc, int *rm,
                                                 unsigned long long *rb) {
  const int lane = lane_id(), w = threadIdx.x / kWave;
  int x = c;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int y = __shfl_up(x, off);
    if (lane >= off) x += y;
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    s += __shfl_xor(s, off);
    const int m2 = __shfl_xor(mn, off);
    mn = m2 < mn ? m2 : mn;
    const unsigned long long b2 = __shfl_xor(best, off);
    best = b2 > best ? b2 : best;
  }
  if (lane == kWave - 1) rc[w] = x;
  if (lane == 0) {
    rs[w] = s;
    rm[w] = mn;
    rb[w] = best;
  }
  __syncthreads();
  // lane l (mod 16) picks up wave l's partials; a butterfly over 16 lanes
  // gives every lane the same totals (IEEE addition is commutative).
  constexpr int NW = kPT / kWave;
  static_assert(NW == 8 || NW == 16, "one partial per lane of a segment");
  const int l16 = lane & (NW - 1);
  double ts = rs[l16];
  int tt = rc[l16];
  int tp = l16 < w ? tt : 0;
  int tm = rm[l16];
  unsigned long long tb = rb[l16];
#pragma unroll
  for (int off = NW / 2; off > 0; off >>= 1) {
    ts += __shfl_xor(ts, off, NW);
    tt += __shfl_xor(tt, off, NW);
    tp += __shfl_xor(tp, off, NW);
    const int m2 = __shfl_xor(tm, off, NW);
    tm = m2 < tm ? m2 : tm;
    const unsigned long long b2 = __shfl_xor(tb, off, NW);
    tb = b2 > tb ? b2 : tb;
  }
  return PanelRed{ts, tt, tp + x - c, tm, tb};
}

// x rounded to the nearest integer (ties to even), |x| < 2^63.
__device__ __forceinline__ unsigned long long round_i64(double x) {
  const double y = rint(x);
  const double hi = floor(y * 0x1p-32);
  const double lo = fma(hi, -0x1p32, y);  // exact, in [0, 2^32)
  return ((unsigned long long)(uint32_t)(int)hi << 32) | (uint32_t)lo;
}

// Adds the products of entries [0, nA) that fall in [plo, plo + width) and
// advances their cursors; returns this lane's smallest next column.  S = 2^LS
// lanes per entry.  TRACK: also marks the columns in the bitmap.  The entry
// arrays come as LDS or as global pointers: generic ones would make flat
// loads, whose waits drain every load in flight.
template <int kPU, int LS, bool TRACK, typename IP, typename EP, typename VP>
__device__ __forceinline__ int panel_accumulate(const SPG_GLOBAL int32_t *bcol,
                                                const SPG_GLOBAL float *bval, IP ecur, EP eend,
                                                VP eval, int nA, double sigma, int plo,
                                                uint32_t width, unsigned long long *pacc,
                                                uint32_t *pbm) {
  constexpr int S = 1 << LS, EPW = kWave >> LS;
  const int lane = lane_id(), w = threadIdx.x / kWave;
  const int sub = lane >> LS, q = lane & (S - 1), base = sub << LS;
  const int phi = plo + kPanel;
  int tmn = INT32_MAX;
  for (int e0 = w * EPW * kPU; e0 < nA; e0 += (kPT / kWave) * EPW * kPU) {
    int c[kPU], en[kPU];
    double a[kPU];
    // Every read below uses an in-range index for every lane (entry 0; B
    // element 0, which exists since a heavy row has products), so the reads
    // of all kPU groups are issued before the first wait.
#pragma unroll
    for (int u = 0; u < kPU; ++u) {
      const int e = e0 + u * EPW + sub;
      const int es = e < nA ? e : 0;
      c[u] = ecur[es];
      en[u] = e < nA ? eend[es] : 0;  // no entry: nothing left to read
      a[u] = (double)eval[es] * sigma;
    }
    bool more;
    do {
      int col[kPU];
      float v[kPU];
#pragma unroll
      for (int u = 0; u < kPU; ++u) {
        const uint32_t idx = (uint32_t)(c[u] + q);  // unsigned: rows may end at 2^31 - 1
        const bool ld = idx < (uint32_t)en[u];
        const uint32_t li = ld ? idx : 0u;
        col[u] = bcol[li];
        v[u] = bval[li];
        col[u] = ld ? col[u] : INT32_MAX;
      }
      more = false;
#pragma unroll
      for (int u = 0; u < kPU; ++u) {
        const bool in = col[u] < phi;
        const uint32_t cl = (uint32_t)(col[u] - plo);
        if (cl < width) {  // columns outside [0, n) are skipped
          atomicAdd(&pacc[cl], round_i64(a[u] * (double)v[u]));
          if (TRACK) atomicOr(&pbm[cl >> 5], 1u << (cl & 31));
        }
        const uint64_t m = __builtin_amdgcn_ballot_w64(in);
        int k;
        if (LS == 6) k = __popcll(m);
        else if (LS == 5) k = lane < 32 ? __popc((uint32_t)m) : __popc((uint32_t)(m >> 32));
        else k = __popc((uint32_t)(m >> base) & ((1u << (S & 31)) - 1u));
        // the columns read past the panel start with the entry's next one
        tmn = min(tmn, in ? INT32_MAX : col[u]);
        c[u] += k;
        if (k < S) en[u] = 0;  // the entry left the panel (or its row ended)
        more = more || k == S;
      }
      more = __any(more);
    } while (more);
#pragma unroll
    for (int u = 0; u < kPU; ++u) {
      const int e = e0 + u * EPW + sub;
      if (e < nA && q == 0) ecur[e] = c[u];
    }
  }
  return tmn;
}

// What a panel leaves behind: every thread owns 16 of its columns (lane l of
// wave w: 1024 w + 64 j + l, so that a wave's reads hit all banks).  Values
// below `low` are no candidates (TRACK: absent columns have none, NaN).  The
// largest value's smallest column is kept; without TRACK only one above zero,
// which is there whatever the bitmap says.
template <bool TRACK>
__device__ __forceinline__ void panel_finish(unsigned long long *pacc, uint32_t *pbm, int plo,
                                             double inv_sigma, int r, bool even, float low,
                                             float (&pw)[kCPT], double &ps, int &cnt,
                                             uint32_t &bbits, int &bcolumn) {
  const int lane = lane_id(), c0 = threadIdx.x / kWave * (kCPT * kWave) + lane;
  ps = 0.0;
  cnt = 0;
  uint32_t top = 0u;
  constexpr int H = kCPT / 2;
#pragma unroll
  for (int j0 = 0; j0 < kCPT; j0 += H) {
    unsigned long long acc[H];
#pragma unroll
    for (int j = 0; j < H; ++j) acc[j] = pacc[c0 + (j0 + j) * kWave];
#pragma unroll
    for (int j = 0; j < H; ++j) pacc[c0 + (j0 + j) * kWave] = 0ull;
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const int jj = j0 + j;
      float p = ipow((float)((double)(long long)acc[j] * inv_sigma), r);
      ps += (double)p;
      if (TRACK) {
        const bool present = pbm[(c0 + jj * kWave) >> 5] >> (lane & 31) & 1u;
        const uint32_t bits = __float_as_uint(p);
        if (present && (bits > bbits || bcolumn < 0)) {  // ties: the smaller column came first
          bbits = bits;
          bcolumn = plo + c0 + jj * kWave;
        }
        if (!present) p = __uint_as_float(0x7fc00000u);
      } else {
        top = max(top, __float_as_uint(p));
        if (!even && acc[j] == 0ull) p = __uint_as_float(0x7fc00000u);
      }
      pw[jj] = p;
      cnt += __popcll(__ballot(p >= low));
    }
  }
  if (!TRACK) {  // the wave's largest value; looked up only when it grows
    const uint32_t wtop =
        (uint32_t)__builtin_amdgcn_readlane(wave_max_last((int)(top ^ 0x80000000u)), kWave - 1) ^
        0x80000000u;
    if (wtop > bbits) {
      bbits = wtop;
      bcolumn = INT32_MAX;  // not in this lane
#pragma unroll
      for (int j = kCPT - 1; j >= 0; --j)
        if (__float_as_uint(pw[j]) == wtop) bcolumn = plo + c0 + j * kWave;
    }
  }
}

__global__ __launch_bounds__(kPT, kPT / 256) void k_mcl_panel(
    const Problem *__restrict__ pr, const int32_t *__restrict__ rows, WsHeader *__restrict__ hdr,
    int blo, int r, int rpost, float prune, int topk, int cap, const double *__restrict__ rabs,
    char *__restrict__ scratch, size_t slot_bytes, const int32_t *__restrict__ fb_rows,
    int32_t *__restrict__ ycol, float *__restrict__ yval, int32_t *__restrict__ ycnt) {
  extern __shared__ __align__(16) unsigned long long pacc[];
  uint32_t *pbm = reinterpret_cast<uint32_t *>(pacc + kPanel);
  __shared__ double rs[kPT / kWave];
  __shared__ int rc[kPT / kWave], rm[kPT / kWave];
  __shared__ unsigned long long rb[kPT / kWave];
  __shared__ int kcnt[2 * 8 * (kPT / kWave)];  // counts of the top-k search
  __shared__ int s_cur[kPE], s_end[kPE];
  __shared__ float s_val[kPE];
  const int n = pr->n;
  const int tid = threadIdx.x;
  char *sp = scratch + (size_t)blockIdx.x * slot_bytes;
  int32_t *lcol = reinterpret_cast<int32_t *>(sp);
  float *lval = reinterpret_cast<float *>(sp + (size_t)4 * n);
  int32_t *ecur = reinterpret_cast<int32_t *>(sp + (size_t)8 * n);
  int32_t *eend = reinterpret_cast<int32_t *>(sp + (size_t)12 * n);
  float *evalg = reinterpret_cast<float *>(sp + (size_t)16 * n);
  __shared__ int stat0;
  if (tid == 0) stat0 = hdr->status;
  __syncthreads();
  if (stat0) return;
  const Part &P = pr->part[0];
  const SPG_GLOBAL int32_t *bcol = gp(P.bcol);
  const SPG_GLOBAL float *bval = gp(static_cast<const float *>(P.bval));
  const int start = hdr->bin_start[blo];
  const int nheavy = hdr->bin_start[kHeavyBin + 1] - start;
  const int count = nheavy + hdr->fallback_count;
  for (int s = tid; s < kPanel; s += kPT) pacc[s] = 0ull;
  for (int s = tid; s < kPanel / 32; s += kPT) pbm[s] = 0u;
  __syncthreads();
  const bool even = (r & 1) == 0;
  __shared__ int item;
  for (int ri = block_next(&hdr->queue[kQueueHeavy], &item); ri < count;
       ri = block_next(&hdr->queue[kQueueHeavy], &item)) {
    const int i = ri < nheavy ? rows[start + ri] : fb_rows[ri - nheavy];
    int as, ae;
    a_row(P, i, as, ae);
    const int nA = ae - as;
    if (nA > n) {  // more entries than columns: a repeated column index
      if (tid == 0) atomicOr(&hdr->status, kStatInvalid);
      break;
    }
    // entries: cursor, end and value, in LDS for rows of at most kPE
    // entries, else in the slot scratch
    const bool lds_state = nA <= kPE;
    int *ccur = lds_state ? s_cur : ecur;
    int *cend = lds_state ? s_end : eend;
    float *cval = lds_state ? s_val : evalg;
    double sb = 0.0;
    int mn = INT32_MAX, plen = 0;
    for (int e = tid; e < nA; e += kPT) {
      const int k = gp(P.acol)[as + e];
      const float av = gp(static_cast<const float *>(P.aval))[as + e];
      const int b0 = gp(P.brp)[k], b1 = gp(P.brp)[k + 1];
      sb += fabs((double)av) * rabs[k];
      ccur[e] = b0;
      cend[e] = b1;
      cval[e] = av;
      plen += b1 - b0;
      if (b0 < b1) mn = min(mn, bcol[b0]);
    }
    PanelRed R = panel_reduce(sb, plen, mn, 0ull, rs, rc, rm, rb);
    __syncthreads();
    // scale 2^s with 2^(62-s) > the row's bound on sum |a b|
    double sigma = 1.0;
    {
      const double bound = R.s * (1.0 + 1.0 / 1048576.0);
      if (bound > 0.0 && bound < 1e300) {
        int ex = 0;
        (void)frexp(bound, &ex);  // bound < 2^ex
        ex = ex < -960 ? -960 : ex;
        sigma = ldexp(1.0, 62 - ex);
      }
    }
    const double inv_sigma = 1.0 / sigma;  // exact: sigma is a power of two
    // lanes per entry: about the mean number of an entry's elements per panel
    int lS = 2;
    {
      const double per = (double)R.total / (double)(nA > 0 ? nA : 1) /
                         (double)((n + kPanel - 1) / kPanel);
      while (lS < 6 && (double)(1 << lS) < per) ++lS;
    }
    // rows of few products per panel: only the marked columns are looked at
    const bool sparse = (double)R.total < (double)kSparse * ((n + kPanel - 1) / kPanel);
    // The bitmap is kept only where it matters: for such rows; with a prune
    // above zero a column whose sum is zero is dropped like an absent one.  A
    // row whose sums are all zero is taken once more, with it.
    const int mfirst = R.mn;
    double scum;
    float S;
    int nc, nk, kept0;
    uint32_t bbits;
    int bcolumn;
    bool track = sparse || !(prune > 0.f);
    while (true) {
      int mnext = mfirst;
      scum = 0.0;
      nc = 0;
      bbits = 0u;
      bcolumn = -1;
#define SPG_ACC(PU, LS, TRACK)                                                              \
  panel_accumulate<PU, LS, TRACK>(bcol, bval, s_cur, s_end, s_val, nA, sigma, plo, width, pacc, \
                                  pbm)
#define SPG_ACC_G(PU, LS)                                                                     \
  panel_accumulate<PU, LS, true>(bcol, bval, gpw(ecur), gpw(eend), gpw(evalg), nA, sigma, plo, \
                                 width, pacc, pbm)
      while (sparse && mnext < n) {
        const int plo = mnext & ~(kPanel - 1);
        const uint32_t width = plo < 0 ? 0u : (uint32_t)min(kPanel, n - plo);
        const int tmn = !lds_state ? SPG_ACC_G(kPUSparse, 3)
                        : lS >= 5  ? SPG_ACC(kPUDense, 5, true)
                                   : SPG_ACC(kPUSparse, 3, true);
        __syncthreads();
        const float low = even ? (float)((double)prune * scum * (1.0 - 1.0 / 1024.0)) : -INFINITY;
        // thread t: the marked ones of columns 16 t .. 16 t + 15
        const uint32_t marked = pbm[tid >> 1] >> ((tid & 1) * 16) & 0xffffu;
        double ps = 0.0;
        int cnt = 0;
        for (uint32_t b = marked; b; b &= b - 1) {
          const int cl = tid * kCPT + __ffs(b) - 1;
          const float p = ipow((float)((double)(long long)pacc[cl] * inv_sigma), r);
          ps += (double)p;
          if (__float_as_uint(p) > bbits || bcolumn < 0) {  // ties: the smaller column came first
            bbits = __float_as_uint(p);
            bcolumn = plo + cl;
          }
          cnt += p >= low ? 1 : 0;
        }
        R = panel_reduce(ps, cnt, tmn, 0ull, rs, rc, rm, rb);
        int o = nc + R.excl;
        for (uint32_t b = marked; b; b &= b - 1) {
          const int cl = tid * kCPT + __ffs(b) - 1;
          const float p = ipow((float)((double)(long long)pacc[cl] * inv_sigma), r);
          pacc[cl] = 0ull;
          if (p >= low) {
            lcol[o] = plo + cl;
            lval[o] = p;
            ++o;
          }
        }
        if ((tid & 1) == 0) pbm[tid >> 1] = 0u;
        scum += R.s;
        nc += R.total;
        mnext = R.mn;
        __syncthreads();
      }
      while (mnext < n) {
        const int plo = mnext & ~(kPanel - 1);
        const uint32_t width = plo < 0 ? 0u : (uint32_t)min(kPanel, n - plo);
        int tmn;
        if (!lds_state) {  // the bitmap does no harm where it is not needed
          tmn = lS >= 5 ? SPG_ACC_G(kPUDense, 5) : SPG_ACC_G(kPUSparse, 3);
        } else if (track) {
          tmn = lS >= 5 ? SPG_ACC(kPUDense, 5, true) : SPG_ACC(kPUSparse, 3, true);
        } else {
          switch (lS) {
            case 6: tmn = SPG_ACC(kPUDense, 6, false); break;
            case 5: tmn = SPG_ACC(kPUDense, 5, false); break;
            case 4: tmn = SPG_ACC(kPUSparse, 4, false); break;
            case 3: tmn = SPG_ACC(kPUSparse, 3, false); break;
            default: tmn = SPG_ACC(kPUSparse, 2, false); break;
          }
        }
        __syncthreads();
        // a product that is zero cannot survive a prune above zero
        const float thr = (float)((double)prune * scum * (1.0 - 1.0 / 1024.0));
        float low = !even ? -INFINITY : track ? thr : fmaxf(thr, 0x1p-149f);
        float pw[kCPT];
        double ps;
        int cnt;
        if (track)
          panel_finish<true>(pacc, pbm, plo, inv_sigma, r, even, low, pw, ps, cnt, bbits, bcolumn);
        else
          panel_finish<false>(pacc, pbm, plo, inv_sigma, r, even, low, pw, ps, cnt, bbits, bcolumn);
        if (even && !track && scum == 0.0) {
          // the first sums: the row's sum is at least theirs
          R = panel_reduce(ps, 0, INT32_MAX, 0ull, rs, rc, rm, rb);
          low = fmaxf((float)((double)prune * R.s * (1.0 - 1.0 / 1024.0)), 0x1p-149f);
          cnt = 0;
#pragma unroll
          for (int j = 0; j < kCPT; ++j) cnt += __popcll(__ballot(pw[j] >= low));
          __syncthreads();
        }
        // the wave's candidates follow those of the waves before it (count 0
        // in all lanes but one)
        R = panel_reduce(ps, lane_id() == kWave - 1 ? cnt : 0, tmn, 0ull, rs, rc, rm, rb);
        if (track || !lds_state)
          for (int wd = tid; wd < kPanel / 32; wd += kPT) pbm[wd] = 0u;
        int o = nc + __shfl(R.excl, 0);
        const int c0 = plo + tid / kWave * (kCPT * kWave) + lane_id();
#pragma unroll
        for (int j = 0; j < kCPT; ++j) {
          const uint64_t m = __ballot(pw[j] >= low);
          if (pw[j] >= low) {
            const int at = o + mbcnt(m);
            lcol[at] = c0 + j * kWave;
            lval[at] = pw[j];
          }
          o += __popcll(m);
        }
        scum += R.s;
        nc += R.total;
        mnext = R.mn;
        // rs, rc, rm are rewritten, and the bitmap marked again, only after
        // the next panel's first barrier, or that of the code below
        if (track || !lds_state) __syncthreads();
      }
#undef SPG_ACC_G
#undef SPG_ACC
      // values that the exact test keeps, per wave (a run of the list each)
      __syncthreads();
      S = (float)scum;
      const int seg = ((nc + kPT - 1) / kPT) * kWave;
      const int l0 = min(nc, tid / kWave * seg), l1 = min(nc, l0 + seg);
      int mine = 0;
      for (int t = l0; t < l1; t += kWave) {
        const int idx = t + lane_id();
        const bool keep = idx < l1 && !(lval[idx < l1 ? idx : l0] / S < prune);
        mine += __popcll(__ballot(keep));
      }
      R = panel_reduce(0.0, lane_id() == kWave - 1 ? mine : 0, INT32_MAX, bbits, rs, rc, rm, rb);
      nk = R.total;
      kept0 = __shfl(R.excl, 0);
      if (track || (scum != 0.0 && (nk > 0 || R.best != 0ull))) break;
      // sums that are all zero: the largest entry is wanted, and which columns
      // are present matters
      track = true;
      __syncthreads();
      for (int e = tid; e < nA; e += kPT) ccur[e] = gp(P.brp)[gp(P.acol)[as + e]];
      __syncthreads();
    }
    __syncthreads();
    SPG_GLOBAL int32_t *cb = gpw(ycol) + (size_t)i * cap;
    SPG_GLOBAL float *vb = gpw(yval) + (size_t)i * cap;
    if (nk > 0 && nk <= kPanel) {
      // the kept entries in LDS (column and value, in the panel's place)
      {
        const int seg = ((nc + kPT - 1) / kPT) * kWave;
        const int l0 = min(nc, tid / kWave * seg), l1 = min(nc, l0 + seg);
        int o = kept0;
        for (int t = l0; t < l1; t += kWave) {
          const int idx = t + lane_id();
          const float q = idx < l1 ? lval[idx] / S + 0.f : 0.f;
          const bool keep = idx < l1 && !(q < prune);
          const uint64_t m = __ballot(keep);
          if (keep)
            pacc[o + mbcnt(m)] = (unsigned long long)(uint32_t)lcol[idx] |
                                 ((unsigned long long)__float_as_uint(q) << 32);
          o += __popcll(m);
        }
      }
      __syncthreads();
      // wave w: entries w seg .. w seg + seg - 1, 64 at a time
      const int seg = ((nk + kPT - 1) / kPT) * kWave;
      const int k0 = min(nk, tid / kWave * seg), k1 = min(nk, k0 + seg);
      const uint32_t *bits_at = reinterpret_cast<const uint32_t *>(pacc) + 1;  // value of entry t: [2 t]
      uint32_t tau = 0u;
      int ties = 0, need = nk;  // ties at tau before this wave's; how many are kept
      if (nk > topk) {
        // the largest tau with at least topk values >= tau, by an eight-way
        // search on the bit patterns (the values are >= 0): seven counts per
        // step and wave, summed over the waves by every wave; two arrays in
        // turn, so that a step needs one barrier
        int step = 0;
        auto count = [&](const uint32_t (&mid)[7], int (&total)[7]) {
          int *slot = kcnt + (step++ & 1) * 8 * (kPT / kWave);
          int cc[7] = {0, 0, 0, 0, 0, 0, 0};
          for (int t = k0; t < k1; t += kWave) {
            const int idx = t + lane_id();
            const uint32_t v = idx < k1 ? bits_at[2 * idx] : 0u;
#pragma unroll
            for (int q = 0; q < 7; ++q) cc[q] += __popcll(__ballot(v >= mid[q]));
          }
          if (lane_id() == 0) {
#pragma unroll
            for (int q = 0; q < 7; ++q) slot[q * (kPT / kWave) + tid / kWave] = cc[q];
          }
          __syncthreads();
          // lane l: counts of threshold l / 16 (two rounds), wave l % 16
          const int x = group_incl_scan<16>(slot[lane_id()]);
          const int y = group_incl_scan<16>(lane_id() < 48 ? slot[64 + lane_id()] : 0);
#pragma unroll
          for (int t = 0; t < 7; ++t)
            total[t] = __builtin_amdgcn_readlane(t < 4 ? x : y, (t & 3) * 16 + 15);
        };
        static_assert(kPT / kWave == 16, "a row of 16 lanes holds the waves' counts");
        uint32_t mid[7];
        int total[7];
        uint32_t lo = prune > 0.f ? __float_as_uint(prune) : 0u;
        uint32_t hi = 0x7f800000u;
        mid[0] = __float_as_uint(1.0625f) + 1u;  // a value is at most its row's sum
#pragma unroll
        for (int t = 1; t < 7; ++t) mid[t] = hi;
        count(mid, total);
        if (total[0] == 0) hi = mid[0] - 1u;
        while (lo < hi) {  // tau in [lo, hi]
          const uint32_t width8 = (hi - lo) / 8 + 1;
#pragma unroll
          for (int t = 0; t < 7; ++t) mid[t] = min(lo + (t + 1) * width8, hi + 1u);
          count(mid, total);
          uint32_t nhi = hi;
#pragma unroll
          for (int t = 6; t >= 0; --t)
            if (total[t] < topk) nhi = mid[t] - 1u;
          uint32_t nlo = lo;
#pragma unroll
          for (int t = 0; t < 7; ++t)
            if (total[t] >= topk) nlo = mid[t];
          lo = nlo;
          hi = max(nhi, nlo);
        }
        tau = lo;
        mid[0] = tau + 1u;
        count(mid, total);
        need = topk - total[0];  // ties at tau to keep, in column order
        int tc = 0;
        for (int t = k0; t < k1; t += kWave) {
          const int idx = t + lane_id();
          tc += __popcll(__ballot(idx < k1 && bits_at[2 * idx] == tau));
        }
        __syncthreads();
        R = panel_reduce(0.0, lane_id() == kWave - 1 ? tc : 0, INT32_MAX, 0ull, rs, rc, rm, rb);
        ties = __shfl(R.excl, 0);
        __syncthreads();
      }
      // the selected entries: their sum, their number per wave
      double s2 = 0.0;
      int ns = 0;
      auto selected = [&](int idx, uint32_t v, int &before) {
        bool on = idx < k1;
        if (nk > topk) {
          const bool tie = on && v == tau;
          const uint64_t m = __ballot(tie);
          on = on && (v > tau || (tie && before + mbcnt(m) < need));
          before += __popcll(m);
        }
        return on;
      };
      int before = ties;
      for (int t = k0; t < k1; t += kWave) {
        const int idx = t + lane_id();
        const uint32_t v = idx < k1 ? bits_at[2 * idx] : 0u;
        const bool on = selected(idx, v, before);
        s2 += on ? (double)__uint_as_float(v) : 0.0;
        ns += __popcll(__ballot(on));
      }
      R = panel_reduce(s2, lane_id() == kWave - 1 ? ns : 0, INT32_MAX, 0ull, rs, rc, rm, rb);
      const float S2 = (float)R.s;
      int o = __shfl(R.excl, 0);
      before = ties;
      for (int t = k0; t < k1; t += kWave) {
        const int idx = t + lane_id();
        const unsigned long long e = idx < k1 ? pacc[idx] : 0ull;
        const bool on = selected(idx, (uint32_t)(e >> 32), before);
        const uint64_t m = __ballot(on);
        const int at = o + mbcnt(m);
        if (on && at < cap) {
          const float q = __uint_as_float((uint32_t)(e >> 32));
          cb[at] = (int)(uint32_t)e;
          vb[at] = rpost == 0 ? q / S2 : ipow(q, rpost);
        }
        o += __popcll(m);
        if (idx < k1) pacc[idx] = 0ull;  // the panel starts clear
      }
      if (tid == 0) ycnt[i] = R.total < cap ? R.total : cap;
      continue;
    }
    // none kept, or more than the panel holds (no prune): the list in place
    const unsigned long long best = bcolumn < 0 ? 0ull
                                                : ((unsigned long long)bbits << 32) |
                                                      (uint32_t)(~(uint32_t)bcolumn);
    const int nlist = nk > 0 ? nc : 0;
    nk = 0;
    for (int c0 = 0; c0 < nlist; c0 += kPT) {
      const int idx = c0 + tid;
      int col = 0;
      float q = 0.f;
      bool keep = false;
      if (idx < nlist) {
        col = lcol[idx];
        q = lval[idx] / S;
        keep = !(q < prune);
      }
      R = panel_reduce(0.0, keep ? 1 : 0, INT32_MAX, best, rs, rc, rm, rb);
      if (keep) {
        lcol[nk + R.excl] = col;
        lval[nk + R.excl] = q + 0.f;
      }
      nk += R.total;
      __syncthreads();
    }
    R = panel_reduce(0.0, 0, INT32_MAX, best, rs, rc, rm, rb);
    const unsigned long long rowbest = R.best;
    __syncthreads();
    // top-k: largest threshold tau with at least topk kept values >= tau
    uint32_t tau = 0u;
    int need = nk;
    if (nk > topk) {
      uint32_t lo = 0u, hi = 0x7f800000u;
      while (lo < hi) {
        const uint32_t mid = lo + (hi - lo + 1) / 2;
        int cc = 0;
        for (int idx = tid; idx < nk; idx += kPT) cc += __float_as_uint(lval[idx]) >= mid ? 1 : 0;
        R = panel_reduce(0.0, cc, INT32_MAX, 0ull, rs, rc, rm, rb);
        __syncthreads();
        if (R.total >= topk) lo = mid;
        else hi = mid - 1;
      }
      tau = lo;
      int gt = 0;
      for (int idx = tid; idx < nk; idx += kPT) gt += __float_as_uint(lval[idx]) > tau ? 1 : 0;
      R = panel_reduce(0.0, gt, INT32_MAX, 0ull, rs, rc, rm, rb);
      __syncthreads();
      need = topk - R.total;  // ties at tau to keep, in column order
    }
    // renormalising sum of the selected entries, then the ordered write
    const bool select_all = nk <= topk;
    double s2 = 0.0;
    {
      int seen = 0;
      for (int c0 = 0; c0 < nk; c0 += kPT) {
        const int idx = c0 + tid;
        float q = 0.f;
        int tie = 0;
        if (idx < nk) {
          q = lval[idx];
          tie = (!select_all && __float_as_uint(q) == tau) ? 1 : 0;
        }
        R = panel_reduce(0.0, tie, INT32_MAX, 0ull, rs, rc, rm, rb);
        bool sel = false;
        if (idx < nk)
          sel = select_all || __float_as_uint(q) > tau || (tie && seen + R.excl < need);
        seen += R.total;
        if (idx < nk && !sel) lval[idx] = -1.f;  // dropped by the top-k
        s2 += sel ? (double)q : 0.0;
        __syncthreads();
      }
    }
    R = panel_reduce(s2, 0, INT32_MAX, 0ull, rs, rc, rm, rb);
    const float S2 = (float)R.s;
    __syncthreads();
    int outn = 0;
    if (nk == 0) {
      if (rowbest != 0ull) {  // emptied row: keep its largest entry
        if (tid == 0) {
          const float q = __uint_as_float((uint32_t)(rowbest >> 32)) / S;
          cb[0] = (int)~(uint32_t)(rowbest & 0xffffffffu);
          vb[0] = rpost == 0 ? q / q : ipow(q, rpost);
        }
        outn = 1;
      }
    } else {
      for (int c0 = 0; c0 < nk; c0 += kPT) {
        const int idx = c0 + tid;
        const bool sel = idx < nk && !(lval[idx] < 0.f);
        R = panel_reduce(0.0, sel ? 1 : 0, INT32_MAX, 0ull, rs, rc, rm, rb);
        const int o = outn + R.excl;
        if (sel && o < cap) {
          cb[o] = lcol[idx];
          vb[o] = rpost == 0 ? lval[idx] / S2 : ipow(lval[idx], rpost);
        }
        outn += R.total;
        __syncthreads();
      }
    }
    if (tid == 0) ycnt[i] = outn < cap ? outn : cap;
    __syncthreads();
  }
}

// Row sums of |x| in FP64 (the bound behind the fixed-point scales); clears
// the counts of rows given back by k_mcl_few.  The first `looks` blocks look at
// rows spread over the lists of the bins from kFewBin on (64 a bin) instead: a
// launch of their own would cost more than they do.
__global__ __launch_bounds__(256) void k_row_abs(const Problem *__restrict__ pr,
                                                 const int32_t *__restrict__ rows,
                                                 const WsHeader *__restrict__ hdr,
                                                 double *__restrict__ rabs,
                                                 int32_t *__restrict__ failed, int looks,
                                                 int32_t *__restrict__ sample) {
  static_assert(kFewNT == 256, "few_look's block");
  __shared__ int key[kFewSlots];
  __shared__ int ncols;
  if (hdr->status) return;
  if ((int)blockIdx.x < looks) {
    const int b = kFewBin + blockIdx.x / kFewSample, s = blockIdx.x % kFewSample;
    const int count = hdr->bin_count[b], looked = min(count, kFewSample);
    if (s >= looked) return;
    const int at = (int)((int64_t)s * count / looked);
    const int wide = few_look(pr->part[0], rows[hdr->bin_start[b] + at], key, &ncols);
    if (threadIdx.x == 0) sample[blockIdx.x] = wide;
    return;
  }
  const int block = blockIdx.x - looks;
  if (block == 0 && threadIdx.x < kNB) failed[threadIdx.x] = 0;
  const Part &P = pr->part[0];
  const int n = P.kdim;
  const int lane = lane_id();
  const int64_t wv = ((int64_t)block * blockDim.x + threadIdx.x) / kWave;
  const int64_t nwv = ((int64_t)(gridDim.x - looks) * blockDim.x) / kWave;
  const SPG_GLOBAL float *bval = gp(static_cast<const float *>(P.bval));
  for (int64_t k = wv; k < n; k += nwv) {
    const int s = gp(P.brp)[k], e = gp(P.brp)[k + 1];
    double t = 0.0;
    for (uint32_t j = (uint32_t)s + lane; j < (uint32_t)e; j += kWave)  // (e up to 2^31 - 1)
      t += fabs((double)bval[j]);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) t += __shfl_xor(t, off);
    if (lane == 0) rabs[k] = t;
  }
}

// Compaction of the padded rows into CSR (row_ptr from the scan of cnt).
__global__ __launch_bounds__(256) void k_mcl_compact(int n, int cap, const int32_t *__restrict__ yrp,
                                                     const int32_t *__restrict__ pcol,
                                                     const float *__restrict__ pval,
                                                     int32_t *__restrict__ ycol,
                                                     float *__restrict__ yval,
                                                     const WsHeader *__restrict__ hdr) {
  if (hdr->status) return;
  const int lane = threadIdx.x & 63;
  const int64_t wv = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwv = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t i = wv; i < n; i += nwv) {
    const int o = yrp[i], len = yrp[i + 1] - o;
    for (int t = lane; t < len; t += 64) {
      ycol[o + t] = pcol[i * cap + t];
      yval[o + t] = pval[i * cap + t];
    }
  }
}

// ---------------------------------------------------------------------------

template <int G>
static void mcl_launch(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int bin, int lS,
                       int TT, uint32_t mul, int maxwin, int r, int rpost, float prune, int topk,
                       int cap,
                       int32_t *ycol, float *yval, int32_t *ycnt, int32_t *fb,
                       const int32_t *failed, int grid, size_t lds, hipStream_t st) {
  hipLaunchKernelGGL(k_mcl_rows<G>, dim3(grid), dim3(MGeom<G>::WG), lds, st, dpr, rows, hdr, bin,
                     lS, TT, mul, maxwin, r, rpost, prune, topk, cap, ycol, yval, ycnt, fb, failed);
}

size_t mcl_lds_bytes(int b, int G) {
  const int WG = G <= kWave ? 256 : G, R = WG / G;
  const size_t TT = (size_t)num_table_slots(b, G);
  return (size_t)R * TT * 8 + (size_t)R * G * 12 + (size_t)R * 4 + 64;
}

hipError_t launch_mcl(const Problem *dpr, const BinPlan &bp, const WsLayout &L, char *ws,
                      int r, int rpost, float prune, int topk, int cap, int32_t *pcol, float *pval,
                      int32_t *ycnt, hipStream_t st) {
  WsHeader *hdr = reinterpret_cast<WsHeader *>(ws);
  const int32_t *rows = reinterpret_cast<const int32_t *>(ws + L.rows);
  int32_t *fb = reinterpret_cast<int32_t *>(ws + L.fbrows);
  const DevInfo &D = dev_info();
  const int maxwin = bp.maxwin < kTail ? bp.maxwin : kTail;
  double *rabs = reinterpret_cast<double *>(ws + L.mcl_rabs);
  // rows given back per bin: the binning's histograms are no longer needed
  int32_t *failed = reinterpret_cast<int32_t *>(ws + L.blockhist);
  int32_t *sample = reinterpret_cast<int32_t *>(ws + kFewSampleAt);
  int looks = 0;
  for (int b = kFewBin; b <= bp.maxbin; ++b)
    if (!bp.known || bp.count[b] >= D.cus) looks = (b - kFewBin + 1) * kFewSample;
  hipLaunchKernelGGL(k_row_abs, dim3(std::max(D.cus * 8, 2 * looks)), dim3(256), 0, st, dpr, rows,
                     hdr, rabs, failed, looks, sample);
  for (int b = 1; b <= bp.maxbin; ++b) {
    if (bp.known && bp.count[b] == 0) continue;
    // a row of this many products may fall on few columns; not worth two
    // launches where every row has a CU (23 rows: 0.06 ms against 0.03)
    const bool few = b >= kFewBin && !(bp.known && bp.count[b] < D.cus);
    if (few) {
      const int grid = bp.known ? std::min(D.cus * 8, bp.count[b]) : D.cus * 8;
      hipLaunchKernelGGL(k_mcl_few, dim3(grid), dim3(kFewNT), 0, st, dpr, rows, hdr, b, r, rpost,
                         prune, topk, cap, rabs, pcol, pval, ycnt, failed, sample);
    }
    int G = bp.lanes[b] < 8 ? 8 : bp.lanes[b];  // no one-thread-per-row MCL kernel
    while (G < 1024 && mcl_lds_bytes(b, G) > D.lds_per_block) G *= 2;
    // a bin past the largest table that fits takes that table (rows whose
    // distinct columns overflow it are handed to the panel kernel)
    int tb = b;
    while (tb > 1 && mcl_lds_bytes(tb, G) > D.lds_per_block) --tb;
    const int WG = G <= kWave ? 256 : G;
    const int R = WG / G;
    const size_t lds = mcl_lds_bytes(tb, G);
    int cap_grid = D.cus * (int)std::max<size_t>(1, std::min<size_t>(D.lds_per_cu / lds, 2048 / WG));
    int grid = cap_grid;
    if (bp.known) grid = std::min(cap_grid, (bp.count[b] + R - 1) / R);
    const int TT = num_table_slots(tb, G);
    const uint32_t mul = mono_mul(bin_slots(tb), bp.n);
    int S = bp.sub[b] > 0 ? bp.sub[b] : 16;
    if (S > G) S = G;
    int lS = 0;
    while ((1 << lS) < S) ++lS;
    switch (G) {
#define SPG_MCL_CASE(g) \
  case g: mcl_launch<g>(dpr, rows, hdr, b, lS, TT, mul, maxwin, r, rpost, prune, topk, cap, pcol, pval, ycnt, fb, few ? failed : nullptr, grid, lds, st); break;
      SPG_MCL_CASE(8)
      SPG_MCL_CASE(16)
      SPG_MCL_CASE(32)
      SPG_MCL_CASE(64)
      SPG_MCL_CASE(128)
      SPG_MCL_CASE(256)
      SPG_MCL_CASE(512)
      default: mcl_launch<1024>(dpr, rows, hdr, b, lS, TT, mul, maxwin, r, rpost, prune, topk, cap, pcol, pval, ycnt, fb, few ? failed : nullptr, grid, lds, st);
#undef SPG_MCL_CASE
    }
  }
  {
    // heavy bins plus rows handed over by the LDS kernels
    // one 1024-thread block per CU (its register use allows no second one)
    const int grid = std::min(mcl_heavy_slots(bp.n), D.cus);
    const size_t lds = (size_t)kPanel * 8 + (size_t)kPanel / 8;
    hipLaunchKernelGGL(k_mcl_panel, dim3(grid), dim3(kPT), lds, st, dpr, rows, hdr, bp.maxbin + 1,
                       r, rpost, prune, topk, cap, rabs, ws + L.mcl_slots, mcl_slot_bytes(bp.n), fb,
                       pcol, pval, ycnt);
  }
  return hipGetLastError();
}

hipError_t launch_mcl_compact(int n, int cap, const int32_t *yrp, const int32_t *pcol,
                              const float *pval, int32_t *ycol, float *yval, const WsHeader *hdr,
                              hipStream_t st) {
  const DevInfo &D = dev_info();
  hipLaunchKernelGGL(k_mcl_compact, dim3(D.cus * 8), dim3(256), 0, st, n, cap, yrp, pcol, pval,
                     ycol, yval, hdr);
  return hipGetLastError();
}

hipError_t configure_mcl_lds(size_t lds_max) {
  const void *ks[] = {
      reinterpret_cast<const void *>(&k_mcl_rows<8>),   reinterpret_cast<const void *>(&k_mcl_rows<16>),
      reinterpret_cast<const void *>(&k_mcl_rows<32>),  reinterpret_cast<const void *>(&k_mcl_rows<64>),
      reinterpret_cast<const void *>(&k_mcl_rows<128>), reinterpret_cast<const void *>(&k_mcl_rows<256>),
      reinterpret_cast<const void *>(&k_mcl_rows<512>), reinterpret_cast<const void *>(&k_mcl_rows<1024>),
      reinterpret_cast<const void *>(&k_mcl_panel),
  };
  for (const void *k : ks) {
    hipError_t e =
        hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_max);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace spg
