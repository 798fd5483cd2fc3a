// Heavy rows shared by many blocks: the symbolic description of a split
// row, the scatter of its products into column ranges, and the merge of
// each segment of ranges (paper §4.4: the level of the row-wise product's
// multi-level accumulator beyond shared memory; here no row is left to a
// single compute unit).
//
// A row of C = sum_k A_k B_k with many products (a power-law hub) used to
// be one block's work from its first product to its last output, so the
// largest row set the length of the whole pass.  Here:
//  - the symbolic kernel (one block per row, column bitmap in LDS) also
//    counts products and distinct columns per range of 8192 columns, cuts
//    the ranges into segments and reserves the row's staging entries;
//  - the scatter kernel takes items of about kSplitItem products of any
//    split row (a window of the row's A entries) and drops each product
//    into its range's run of the row's staging area;
//  - the merge kernel takes one segment at a time and writes it at its output
//    offset: a single range of many products summed in a dense LDS panel of
//    8192 columns; at most kSplitSeg products over a moderate span marked in
//    a bitmap that gives every column its place; over a wider span placed
//    into order-preserving buckets.
//
// What bounds them: the scatter the 8-byte staging stores (a line a lane) and
// the gathers of B; the merge vector instructions (half its time) on segments
// that a row's cuts leave at 1500 products of 4096; the count its two LDS
// atomics a product and, one block a CU, the chain to a row's products.
// R-MAT blocks, 2^20 rows, 8 parts: count 1.29 -> 0.86 ms (products spread
// over all threads at once; the map read, counted and cleared in one sweep by
// range; range counters in copies; a row of 1.6 million products alone on the
// chip 0.33 -> 0.40, its windows one after the other), scatter 1.27 -> 1.12 (one pass: a
// product's place is its counter's old value), merge 1.41 -> 0.84.
// A row the workspace cannot describe or stage stays with the one-block
// heavy kernels, which take the list of such rows.
#include <algorithm>

#include "block_ops.hpp"
#include "internal.hpp"
#include "rowops.hpp"

namespace spg {

// A thread's products of a window loaded together (four at a time: a row of
// 1.6 million products 0.43 ms against 0.40, R-MAT blocks 0.861 against 0.857).
constexpr int kSplitSymUnroll = 8;
constexpr int kScatterNT = 512;         // threads of a scatter block
constexpr int kAccumNT = 512;           // threads of a merge block
constexpr int kRangeWords = (1 << kSplitLog2W) >> 5;  // bitmap words per range
// Segments of one range with at least this many products are summed in the
// dense panel.
constexpr int kDenseMin = 1024;
// Other segments of at most this many columns find their places from a bitmap.
// Against the buckets, R-MAT blocks of 2^20 columns, FP32: 1.17 -> 0.94 ms;
// with at most 2^17 columns (three blocks a CU instead of two) 1.00.  FP64
// keeps to 2^17, two blocks a CU: R-MAT, 2^19 rows on 2^20 / 2^17 rows on 2^22
// columns 0.70 / 0.17 ms, with 2^18 columns and one block 0.92 / 0.24.
template <typename VT>
constexpr int map_cols() { return sizeof(VT) == 4 ? 1 << 18 : 1 << 17; }
static_assert(map_cols<double>() % (64 * kAccumNT) == 0, "whole words per thread");

// ---------------------------------------------------------------------------
// Symbolic: distinct columns of every row from bin blo on (heavy rows, one
// block per row, column bitmap in LDS or in the slot's global bitmap), and
// for rows h < hmax (sa.F > 0) the split description.

template <bool LDSMAP>
__global__ __launch_bounds__(1024) void k_sym_split(const Problem *__restrict__ pr,
                                                    const int32_t *__restrict__ rows,
                                                    WsHeader *__restrict__ hdr, int blo,
                                                    uint32_t *gbitmap, int32_t *cnt,
                                                    SplitArgs sa) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ WinLds<1024, false, float> win;
  __shared__ int pe[kSplitMaxRanges + 1], de[kSplitMaxRanges + 1];
  // products per range in 2^plog copies, so that lanes rarely meet on one
  // counter; later the segments' first ranges
  __shared__ int pcnt[kSplitMaxRanges];
  __shared__ int wtot[16];
  __shared__ int total, item, okflag, segbase, itembase, stagebase;
  __shared__ unsigned long long prod64;  // the row's products (the range counters are 32-bit)
  const int n = pr->n;
  const int nw = (n + 31) >> 5;
  uint32_t *map = LDSMAP ? reinterpret_cast<uint32_t *>(smem_raw) : gbitmap + (size_t)blockIdx.x * nw;
  if (hdr->status) return;
  const int start = hdr->bin_start[blo];
  const int count = hdr->bin_start[kHeavyBin + 1] - start;
  const int tid = threadIdx.x;
  const int F = sa.F;
  const int K = pr->K;
  if (tid < K) win.part[tid] = blk_part<float>(pr->part[tid]);
  const int plog = F > 0 && F <= kSplitMaxRanges / 2 ? 31 - __clz(kSplitMaxRanges / F) : 0;
  const int pcopy = lane_id() & ((1 << plog) - 1);
  for (int w = tid; w < nw; w += 1024) map[w] = 0u;
  for (int ri = block_next(&hdr->queue[kQueueHeavy], &item); ri < count;
       ri = block_next(&hdr->queue[kQueueHeavy], &item)) {
    const int i = rows[start + ri];
    const bool rec = F > 0 && ri < sa.hmax;  // the same in every thread
    static_assert(kSplitMaxRanges <= 1024, "a thread a counter");
    if (rec && tid < kSplitMaxRanges) pcnt[tid] = 0;
    if (tid == 0) {
      total = 0;
      prod64 = 0;
    }
    if (!LDSMAP) __threadfence();
    __syncthreads();
    int mine = 0;  // described rows: products; others: new distinct columns
    BlkHead<float> h;
    h.i = __builtin_amdgcn_readfirstlane(i);
    blk_parts(win.part, K, nullptr, h);
    blk_number(K, h);
    blk_windows<false, kSplitSymUnroll>(
        win, K, h, 0, h.nA, [] {},
        [&](int, int col, float) {
          const uint32_t bit = 1u << (col & 31);
          if (rec) {  // distinct columns come from the popcounts below
            atomicOr(&map[col >> 5], bit);
            atomicAdd(&pcnt[((col >> kSplitLog2W) << plog) | pcopy], 1);
            ++mine;
          } else {
            const uint32_t old = atomicOr(&map[col >> 5], bit);
            mine += (old & bit) ? 0 : 1;
          }
        },
        [] {});
    if (mine) {
      if (rec) atomicAdd(&prod64, (unsigned long long)mine);
      else atomicAdd(&total, mine);
    }
    if (!LDSMAP) __threadfence();
    __syncthreads();
    if (!rec) {
      for (int w = tid; w < nw; w += 1024) map[w] = 0u;  // for the next row
      if (tid == 0) cnt[i] = total;
      continue;
    }
    // distinct columns per range, a wave at a time; the map is clear again
    for (int f = tid / kWave; f < F; f += 1024 / kWave) {
      static_assert(kRangeWords == 4 * kWave, "four words a lane");
      int pop = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int w = f * kRangeWords + q * kWave + lane_id();
        if (w < nw) {
          pop += __popc(map[w]);
          map[w] = 0u;
        }
      }
      pop = group_incl_scan<kWave>(pop);
      if (lane_id() == kWave - 1) de[f] = pop;
    }
    __syncthreads();
    int pc = 0;
    if (tid < F)
      for (int q = 0; q < 1 << plog; ++q) pc += pcnt[(tid << plog) + q];
    const int dc = tid < F ? de[tid] : 0;
    int P, D;
    const int pex = group_excl_scan<true, 1024>(pc, tid, wtot, P);
    const int dex = group_excl_scan<true, 1024>(dc, tid, wtot, D);
    if (tid < F) {
      pe[tid] = pex;
      de[tid] = dex;
    }
    if (tid == 0) {
      pe[F] = P;
      de[F] = D;
    }
    __syncthreads();
    // segment starts: a range holding more than a quarter of a segment stands
    // alone; the others group while their product prefix stays in the same
    // multiple of three quarters (so a group holds fewer than kSplitSeg;
    // halves instead: 10 % more time in the merge, from more segments)
    constexpr int H = kSplitSeg * 3 / 4;
    int flag = 0;
    if (tid < F) {
      const int a = pe[tid];
      if (tid == 0) {
        flag = 1;
      } else {
        const int ap = pe[tid - 1];
        const bool big = pe[tid + 1] - a > kSplitSeg - H, bigp = a - ap > kSplitSeg - H;
        flag = (big || bigp || a / H != ap / H) ? 1 : 0;
      }
    }
    int *sstart = pcnt;
    int nseg;
    const int sidx = group_excl_scan<true, 1024>(flag, tid, wtot, nseg);
    if (flag) sstart[sidx] = tid;
    const int J = (P + kSplitItem - 1) / kSplitItem;
    if (tid == 0) {
      // a row of more products than the staging area holds (then its
      // 32-bit range counters may also have wrapped) is not described
      int ok = prod64 > 0 && prod64 <= (unsigned long long)sa.pcap && nseg > 0;
      long long b = -1;
      int sg = -1, ib = -1;
      if (ok) {
        b = (long long)atomicAdd(&sa.ctl->stage, (unsigned long long)P);
        ok = b + P <= sa.pcap;
      }
      if (ok) {
        sg = atomicAdd(&sa.ctl->segs, nseg);
        ib = atomicAdd(&sa.ctl->items, J);
        ok = sg <= sa.segcap - nseg && ib <= sa.itemcap - J;
      }
      okflag = ok;
      stagebase = ok ? (int)b : -1;
      segbase = sg;
      itembase = ib;
      cnt[i] = D;
      sa.rows[ri] = SplitRow{ok ? (int32_t)b : -1, J, P, i};
    }
    __syncthreads();
    if (okflag) {
      int32_t *fo = sa.fo + (size_t)ri * (F + 1);
      for (int c = tid; c <= F; c += 1024) fo[c] = pe[c];
      for (int s = tid; s < nseg; s += 1024) {
        const int f0 = sstart[s], f1 = s + 1 < nseg ? sstart[s + 1] : F;
        sa.segs[segbase + s] =
            SplitSeg{ri, f0 << kSplitLog2W, min(n, f1 << kSplitLog2W), stagebase + pe[f0],
                     pe[f1] - pe[f0], de[f0], de[f1] - de[f0], -1};
      }
      const int E = h.nA;
      for (int j = tid; j < J; j += 1024)
        sa.items[itembase + j] =
            SplitItem{ri, i, (int)((int64_t)j * E / J), (int)((int64_t)(j + 1) * E / J)};
    } else if (segbase >= 0) {
      // reserved but unusable entries are marked unused
      for (int s = tid; s < nseg && segbase + s < sa.segcap; s += 1024) sa.segs[segbase + s].h = -1;
      for (int j = tid; j < J && itembase + j < sa.itemcap; j += 1024) sa.items[itembase + j].h = -1;
    }
  }
}

// ---------------------------------------------------------------------------
// Numeric, step 0: the scatter cursors of the split rows start at zero, and
// the heavy rows from bin blo on that are not split are listed for the
// one-block kernels.

__global__ void k_split_prepare(const int32_t *__restrict__ rows, WsHeader *__restrict__ hdr,
                                int blo, SplitArgs sa, const int32_t *__restrict__ crp,
                                int32_t *__restrict__ ulist) {
  if (hdr->status) return;
  const int sbin = hdr->bin_start[sa.bin];
  const int nsplit = min(hdr->bin_start[kHeavyBin + 1] - sbin, sa.hmax);
  const int64_t total = (int64_t)nsplit * sa.F;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t = t0; t < total; t += step)
    if (sa.rows[t / sa.F].base >= 0) sa.cur[t] = 0;
  const int start = hdr->bin_start[blo];
  const int count = hdr->bin_start[kHeavyBin + 1] - start;
  for (int64_t t = t0; t < count; t += step) {
    const int h = start + (int)t - sbin;
    if (!(h >= 0 && h < sa.hmax && sa.rows[h].base >= 0))
      ulist[atomicAdd(&sa.ctl->nuns, 1)] = rows[start + t];
  }
  // output positions of the segments
  const int nseg = min(sa.ctl->segs, sa.segcap);
  for (int64_t t = t0; t < nseg; t += step) {
    const SplitSeg sg = sa.segs[t];
    if (sg.h < 0) continue;
    const int i = sa.rows[sg.h].row;
    int out = crp[i] + sg.dstart;
    if (out + sg.dcount > crp[i + 1]) {  // the row_ptr does not match the description
      atomicOr(&hdr->status, kStatInvalid);
      out = -1;
    }
    sa.segs[t].out = out;
  }
}

// The staging area of the split rows: FP32 products as one 8-byte word
// (column in the low half, value bits in the high half: one store in the
// scatter, one load in the merge); FP64 products as a column array and a
// value array.  Global-address-space pointers: global, not flat, memory
// instructions.
template <typename VT>
struct Staging {
  SPG_GLOBAL int32_t *col;
  SPG_GLOBAL VT *val;
  __device__ __forceinline__ void put(int p, int c, VT v) const {
    col[p] = c;
    val[p] = v;
  }
  __device__ __forceinline__ void get(int p, int &c, VT &v) const {
    c = col[p];
    v = val[p];
  }
};
template <>
struct Staging<float> {
  SPG_GLOBAL int32_t *col;  // the area's base, 256-byte aligned: 8-byte words
  SPG_GLOBAL float *val;    // unused
  __device__ __forceinline__ void put(int p, int c, float v) const {
    reinterpret_cast<SPG_GLOBAL unsigned long long *>(col)[p] =
        (unsigned long long)(uint32_t)c | ((unsigned long long)__float_as_uint(v) << 32);
  }
  __device__ __forceinline__ void get(int p, int &c, float &v) const {
    const unsigned long long w = reinterpret_cast<const SPG_GLOBAL unsigned long long *>(col)[p];
    c = (int)(uint32_t)w;
    v = __uint_as_float((uint32_t)(w >> 32));
  }
};

// Numeric, step 1: items of the split rows from bin blo on, in windows of
// eight products a thread.  A product's place among the window's products of
// its range comes from an LDS counter; one atomic per (window, range) on the
// row's range cursor reserves the window's run inside the range.
template <typename VT>
__global__ __launch_bounds__(kScatterNT, sizeof(VT) == 4 ? 6 : 4) void k_split_scatter(
    const Problem *__restrict__ pr, WsHeader *__restrict__ hdr, int blo, SplitArgs sa) {
  __shared__ WinLds<kScatterNT, true, VT> win;
  __shared__ int lc[kSplitMaxRanges];
  __shared__ int item;
  if (hdr->status) return;
  const int sbin = hdr->bin_start[sa.bin];
  const int hlo = hdr->bin_start[blo] - sbin;
  const int nitems = min(sa.ctl->items, sa.itemcap);
  const int tid = threadIdx.x;
  const int F = sa.F;
  const Staging<VT> stg{gpw(sa.scol), gpw(static_cast<VT *>(sa.sval))};
  const int K = pr->K;
  if (tid < K) win.part[tid] = blk_part<VT>(pr->part[tid]);
  for (int t = block_next(&sa.ctl->q_scatter, &item); t < nitems;
       t = block_next(&sa.ctl->q_scatter, &item)) {
    const SplitItem it = sa.items[t];
    // unused, or a row of an LDS bin of this pass
    if (it.h < hlo || it.h >= sa.hmax) continue;
    const int base = sa.rows[it.h].base;
    if (base < 0) continue;
    BlkHead<VT> h;
    h.i = __builtin_amdgcn_readfirstlane(it.i);
    blk_parts(win.part, K, nullptr, h);
    blk_number(K, h);
    const int32_t *fo = sa.fo + (size_t)it.h * (F + 1);
    int32_t *cur = sa.cur + (size_t)it.h * F;
    int col[kBlkE], rk[kBlkE];
    VT val[kBlkE];
    blk_windows<true, kBlkE / 2>(
        win, K, h, it.e0, min(it.e1, h.nA),
        [&] {
          for (int c = tid; c < F; c += kScatterNT) lc[c] = 0;
#pragma unroll
          for (int j = 0; j < kBlkE; ++j) col[j] = -1;
        },
        [&](int j, int c, VT v) {
          col[j] = c;
          val[j] = v;
          rk[j] = atomicAdd(&lc[c >> kSplitLog2W], 1);
        },
        [&] {
          __syncthreads();
          for (int c = tid; c < F; c += kScatterNT) {
            const int k = lc[c];
            if (k) {
              const int p = atomicAdd(&cur[c], k);
              const int lim = fo[c + 1] - fo[c];
              if (p > lim - k) {  // more products than the symbolic pass saw
                atomicOr(&hdr->status, kStatInvalid);
                lc[c] = -1;
              } else {
                lc[c] = base + fo[c] + p;
              }
            }
          }
          __syncthreads();
#pragma unroll
          for (int j = 0; j < kBlkE; ++j) {
            if (col[j] >= 0) {
              const int p = lc[col[j] >> kSplitLog2W];
              if (p >= 0) stg.put(p + rk[j], col[j], val[j]);
            }
          }
        });
  }
}

// ---------------------------------------------------------------------------
// Numeric, step 2: one segment at a time.

// A single range with more products than a sorted segment holds: sums in a
// dense LDS panel of the range's columns, a presence bitmap walked in
// column order.  Returns the distinct columns written.
template <typename VT, typename Next>
__device__ __forceinline__ int merge_dense(const Staging<VT> &stg, int P, int c0, int D, VT *panel,
                                           uint32_t *bm, int *wtot, SPG_GLOBAL int32_t *cb,
                                           SPG_GLOBAL VT *vb, WsHeader *hdr, Next &next) {
  constexpr int W = 1 << kSplitLog2W;
  const int tid = threadIdx.x;
  for (int c = tid; c < W; c += kAccumNT) panel[c] = VT(0);
  for (int w = tid; w < kRangeWords; w += kAccumNT) bm[w] = 0u;
  __syncthreads();
  bool bad = false;
  constexpr int U = 4;
  for (int p0 = tid; p0 < P; p0 += U * kAccumNT) {
    int c[U];
    VT v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = p0 + u * kAccumNT;
      c[u] = -1;
      v[u] = VT(0);
      if (p < P) {
        stg.get(p, c[u], v[u]);
        c[u] -= c0;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (p0 + u * kAccumNT < P) {
        if ((unsigned)c[u] < (unsigned)W) {
          lds_add_cas(&panel[c[u]], v[u]);
          atomicOr(&bm[c[u] >> 5], 1u << (c[u] & 31));
        } else {
          bad = true;
        }
      }
    }
  }
  if (bad) atomicOr(&hdr->status, kStatInvalid);
  next.ticket();
  __syncthreads();
  next.head();
  // columns in order: a wave takes 1024 of them, 64 at a time
  static_assert(kRangeWords == 32 * (kAccumNT / kWave), "32 words a wave");
  const int lane = lane_id(), wv = tid / kWave;
  const uint32_t mine = lane < 32 ? bm[wv * 32 + lane] : 0u;
  const int pop = group_incl_scan<kWave>(__popc(mine));
  if (lane == kWave - 1) wtot[wv] = pop;
  __syncthreads();
  next.load();
  int o = 0, tot = 0;
#pragma unroll
  for (int q = 0; q < kAccumNT / kWave; ++q) {
    o += q < wv ? wtot[q] : 0;
    tot += wtot[q];
  }
#pragma unroll 4
  for (int q = 0; q < 16; ++q) {
    const uint64_t m = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)mine, 2 * q) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)mine, 2 * q + 1) << 32;
    const int c = wv * 1024 + q * kWave + lane, p = o + mbcnt(m);
    if ((m >> lane & 1u) && p < D) {
      cb[p] = c0 + c;
      vb[p] = panel[c];
    }
    o += __popcll(m);
  }
  return tot;
}

// At most kSplitSeg products over the columns [c0, c0 + span): a ticket in
// the bucket floor(c T / span) of each (two 16-bit counters per word), bucket
// starts, then the last steps of rows of one block.
template <typename VT, typename Next>
__device__ __forceinline__ void merge_buckets(int (&kc)[kBlkE], const VT (&kv)[kBlkE], int P,
                                              int c0, int span, int D, uint32_t *cnt, uint32_t *ikey, VT *ival,
                                              int *wtot, int *bigmax, int *ndl, uint32_t *dlist,
                                              SPG_GLOBAL int32_t *cb, SPG_GLOBAL VT *vb,
                                              WsHeader *hdr, Next &next) {
  constexpr int J = kBlkE, T = kSplitSeg;
  static_assert(kSplitSeg == kBlkE * kAccumNT, "eight products a thread");
  const int tid = threadIdx.x;
  const uint32_t mul = T >= span ? 0xffffffffu : (uint32_t)(((uint64_t)T << 32) / (uint64_t)span);
  reinterpret_cast<uint4 *>(cnt)[tid] = make_uint4(0u, 0u, 0u, 0u);
  if (tid == 0) *bigmax = 0;
  bool bad = false;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < J; ++j) {
    if (tid + j * kAccumNT < P) {
      uint32_t c = (uint32_t)(kc[j] - c0);
      if (c >= (uint32_t)span) {  // outside the segment: a changed pattern
        bad = true;
        c = (uint32_t)span - 1;
      }
      const uint32_t b = mono_slot(c, mul), sh = (b & 1u) << 4;
      const uint32_t t = (atomicAdd(&cnt[b >> 1], 1u << sh) >> sh) & 0xffffu;
      kc[j] = (int)(c | min(t, (uint32_t)kBigBucket) << 24);  // column less c0, ticket
    }
  }
  if (bad) atomicOr(&hdr->status, kStatInvalid);
  next.ticket();
  __syncthreads();
  next.head();
  blk_starts<kAccumNT>(cnt, bigmax, wtot);
  __syncthreads();
  const int mx = *bigmax;
  const bool big = mx > kBigBucket;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    if (tid + j * kAccumNT < P) {
      const uint32_t c = (uint32_t)kc[j] & 0xffffffu;
      const int pos = big ? tid + j * kAccumNT : bkt_start(cnt, mono_slot(c, mul)) + (kc[j] >> 24);
      ikey[pos] = c;
      ival[pos] = kv[j];
    }
  }
  if (tid < kBigBucket) ikey[P + tid] = 0x7fffffffu;  // above every column
  __syncthreads();
  next.load();
  blk_finish<kAccumNT, VT>(cnt, ikey, ival, P, D, big, mx, ndl, dlist, wtot, c0, cb, vb, hdr);
}

// Bitmap word w with a gap after every eight: threads that scan runs of eight
// words do not meet on the banks.
__device__ __forceinline__ int map_at(int w) { return w + (w >> 3); }
template <typename VT>
constexpr int map_words() { return map_cols<VT>() / 64 + map_cols<VT>() / 512; }

// At most kSplitSeg products over at most map_cols columns from c0 on: marked
// in a bitmap, whose bits below a column are its place among the D distinct
// ones; values summed and columns written there.
template <typename VT, typename Next>
__device__ __forceinline__ void merge_map(int (&kc)[kBlkE], const VT (&kv)[kBlkE], int P, int c0, int span, int D,
                                          unsigned long long *map, uint16_t *pre, int32_t *okey,
                                          VT *osum, int *wtot, SPG_GLOBAL int32_t *cb,
                                          SPG_GLOBAL VT *vb, WsHeader *hdr, Next &next) {
  constexpr int J = kBlkE;
  const int tid = threadIdx.x;
  const int per = (span + 64 * kAccumNT - 1) / (64 * kAccumNT);  // words a thread, 8 at most
  for (int w = tid; w < map_at(per * kAccumNT); w += kAccumNT) map[w] = 0ull;
  for (int d = tid; d < D; d += kAccumNT) osum[d] = VT(0);
  __syncthreads();
  bool bad = false;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    if (j * kAccumNT >= P) break;
    uint32_t c = (uint32_t)(kc[j] - c0);
    if (c >= (uint32_t)span) {  // outside the segment: a changed pattern
      bad = true;
      c = (uint32_t)span - 1;
    }
    kc[j] = (int)c;
    if (tid + j * kAccumNT < P)
      atomicOr(reinterpret_cast<uint32_t *>(map + map_at(c >> 6)) + (c >> 5 & 1u), 1u << (c & 31));
  }
  next.ticket();
  __syncthreads();
  next.head();
  // places of the words' first columns; thread t scans words t per ...
  int n = 0, tot;
  for (int q = 0; q < per; ++q) n += __popcll(map[map_at(tid * per + q)]);
  int run = blk_scan<kAccumNT>(n, wtot, tot);
  for (int q = 0; q < per; ++q) {
    const int w = map_at(tid * per + q);
    pre[w] = (uint16_t)run;
    run += __popcll(map[w]);
  }
  if (tid == 0) bad = bad || tot != D;
  if (bad) atomicOr(&hdr->status, kStatInvalid);
  __syncthreads();
  next.load();
#pragma unroll
  for (int j = 0; j < J; ++j) {
    if (j * kAccumNT >= P) break;
    if (tid + j * kAccumNT < P) {
      const uint32_t c = (uint32_t)kc[j];
      const int w = map_at(c >> 6);
      const int d = (int)pre[w] + __popcll(map[w] & ((1ull << (c & 63)) - 1ull));
      if (d < D) {
        okey[d] = c0 + (int)c;
        lds_add_cas(&osum[d], kv[j]);
      }
    }
  }
  __syncthreads();
  for (int d = tid; d < D; d += kAccumNT) {
    if (d < tot) {
      cb[d] = okey[d];
      vb[d] = osum[d];
    }
  }
}

// What a merge block holds of its next segment: taken from the queue, read
// and loaded while the current one is worked on.  ticket() goes before a
// barrier, head() behind it, load() where registers allow.
template <typename VT>
struct SegNext {
  const SplitArgs &sa;
  int *item;
  int nseg, hlo, taken, t;
  SplitSeg sg;
  int kc[kBlkE];
  VT kv[kBlkE];

  __device__ __forceinline__ void take() {
    if (threadIdx.x == 0) taken = atomicAdd(&sa.ctl->q_accum, 1);
  }
  __device__ __forceinline__ void ticket() {
    if (threadIdx.x == 0) *item = taken;
  }
  __device__ __forceinline__ void head() {
    t = __builtin_amdgcn_readfirstlane(*item);
    if (t < nseg) sg = sa.segs[t];
  }
  // unused, a row of an LDS bin of this pass, or a row_ptr mismatch
  __device__ __forceinline__ bool live() const { return t < nseg && sg.h >= hlo && sg.out >= 0; }
  __device__ __forceinline__ bool dense() const {
    return sg.pcount > kSplitSeg ||
           (sg.pcount >= kDenseMin && sg.c1 - sg.c0 <= 1 << kSplitLog2W);
  }
  // the segment's part of the staging area (FP32: 8-byte words)
  __device__ __forceinline__ Staging<VT> staging() const {
    return Staging<VT>{gpw(sa.scol + (sizeof(VT) == 4 ? 2 : 1) * (size_t)sg.stage),
                       gpw(static_cast<VT *>(sa.sval) + sg.stage)};
  }
  __device__ __forceinline__ void load() {
    if (!live() || dense() || sg.pcount == 0) return;
    const Staging<VT> stg = staging();
#pragma unroll
    for (int j = 0; j < kBlkE; ++j) {
      if (j * kAccumNT >= sg.pcount) break;
      stg.get(min((int)threadIdx.x + j * kAccumNT, sg.pcount - 1), kc[j], kv[j]);
    }
  }
};

template <typename VT>
__global__ __launch_bounds__(kAccumNT, 4) void k_split_merge(WsHeader *__restrict__ hdr, int blo,
                                                          SplitArgs sa,
                                                          int32_t *__restrict__ ccol,
                                                          VT *__restrict__ cval) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  // bucket merge: values | counters (two per word) | keys; dense merge:
  // panel | bitmap
  VT *ival = reinterpret_cast<VT *>(smem_raw);
  uint32_t *cnt = reinterpret_cast<uint32_t *>(ival + kSplitSeg);
  uint32_t *ikey = cnt + kSplitSeg / 2 + kBigBucket;  // room for a bucket's length either side
  unsigned long long *map = reinterpret_cast<unsigned long long *>(ival + kSplitSeg);
  uint16_t *pre = reinterpret_cast<uint16_t *>(map + map_words<VT>());
  int32_t *okey = reinterpret_cast<int32_t *>(pre + map_words<VT>());
  VT *panel = reinterpret_cast<VT *>(smem_raw);
  uint32_t *bm = reinterpret_cast<uint32_t *>(panel + (1 << kSplitLog2W));
  __shared__ int wtot[kAccumNT / kWave];
  __shared__ int item, bigmax, ndl[2];
  __shared__ uint32_t dlist[kDupList];
  if (hdr->status) return;
  const int sbin = hdr->bin_start[sa.bin];
  const int hlo = hdr->bin_start[blo] - sbin;
  const int nseg = min(sa.ctl->segs, sa.segcap);
  const int tid = threadIdx.x;
  SegNext<VT> next{sa, &item, nseg, hlo, 0, 0, {}, {}, {}};
  if (tid == 0) ndl[0] = ndl[1] = 0;
  next.take();
  next.ticket();
  __syncthreads();
  next.head();
  next.load();
  while (next.t < nseg) {
    const SplitSeg sg = next.sg;
    const Staging<VT> stg = next.staging();
    const bool live = next.live(), dense = next.dense();
    int kc[kBlkE];
    VT kv[kBlkE];
#pragma unroll
    for (int j = 0; j < kBlkE; ++j) {
      kc[j] = next.kc[j];
      kv[j] = next.kv[j];
    }
    __syncthreads();  // the previous segment's last reads
    if (tid == 0) blk_unmoved(ndl, hdr);
    next.take();
    if (!live || sg.pcount == 0) {
      if (live && tid == 0 && sg.dcount != 0) atomicOr(&hdr->status, kStatInvalid);
      next.ticket();
      __syncthreads();
      next.head();
      next.load();
      continue;
    }
    SPG_GLOBAL int32_t *cb = gpw(ccol) + sg.out;
    SPG_GLOBAL VT *vb = gpw(cval) + sg.out;
    if (dense) {
      const int got = merge_dense<VT>(stg, sg.pcount, sg.c0, sg.dcount, panel, bm, wtot, cb, vb,
                                      hdr, next);
      if (tid == 0 && got != sg.dcount) atomicOr(&hdr->status, kStatInvalid);
    } else if (sg.c1 - sg.c0 <= map_cols<VT>() && sg.dcount <= kSplitSeg) {
      merge_map<VT>(kc, kv, sg.pcount, sg.c0, sg.c1 - sg.c0, sg.dcount, map, pre, okey, ival, wtot,
                    cb, vb, hdr, next);
    } else {
      // (the other merges use this memory too)
      if (tid < kBigBucket) ikey[tid - kBigBucket] = 0xffffffffu;  // as an int: below every column
      merge_buckets<VT>(kc, kv, sg.pcount, sg.c0, sg.c1 - sg.c0, sg.dcount, cnt, ikey, ival, wtot,
                        &bigmax, ndl, dlist, cb, vb, hdr, next);
    }
  }
  __syncthreads();
  if (tid == 0) blk_unmoved(ndl, hdr);
}

// ---------------------------------------------------------------------------
// Launchers.

size_t split_sym_static_lds() {
  return sizeof(WinLds<1024, false, float>) + (size_t)2 * (kSplitMaxRanges + 1) * 4 +
         (size_t)kSplitMaxRanges * 4 + 16 * 4 + 64;
}

template <typename VT>
static size_t merge_lds() {
  const size_t buckets = (size_t)kSplitSeg * (6 + sizeof(VT)) + 2 * kBigBucket * 4;
  const size_t dense = ((size_t)sizeof(VT) << kSplitLog2W) + (size_t)kRangeWords * 4;
  const size_t map = (size_t)kSplitSeg * (4 + sizeof(VT)) + (size_t)map_words<VT>() * 10;
  return std::max(map, std::max(buckets, dense));
}

static int per_cu(size_t lds, size_t stat, int threads) {
  const DevInfo &D = dev_info();
  int b = (int)(D.lds_per_cu / (lds + stat));
  const int bt = 2048 / threads;
  b = b < bt ? b : bt;
  return b < 1 ? 1 : b;
}

hipError_t launch_sym_split(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int blo,
                            bool lds_map, uint32_t *gbitmap, int grid, size_t lds,
                            int32_t *cnt, const SplitArgs &sa, hipStream_t st) {
  if (lds_map)
    hipLaunchKernelGGL(k_sym_split<true>, dim3(grid), dim3(1024), lds, st, dpr, rows, hdr, blo,
                       (uint32_t *)nullptr, cnt, sa);
  else
    hipLaunchKernelGGL(k_sym_split<false>, dim3(grid), dim3(1024), 0, st, dpr, rows, hdr, blo,
                       gbitmap, cnt, sa);
  return hipGetLastError();
}

template <typename VT>
static void num_split(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int blo,
                      const SplitArgs &sa, int32_t *ulist, const int32_t *crp, int32_t *ccol,
                      VT *cval, hipStream_t st) {
  const DevInfo &D = dev_info();
  hipLaunchKernelGGL(k_split_prepare, dim3(D.cus * 4), dim3(256), 0, st, rows, hdr, blo, sa,
                     crp, ulist);
  const int sg = D.cus * per_cu(0, sizeof(WinLds<kScatterNT, true, VT>) + kSplitMaxRanges * 4 + 64,
                                kScatterNT);
  hipLaunchKernelGGL(k_split_scatter<VT>, dim3(sg), dim3(kScatterNT), 0, st, dpr, hdr, blo, sa);
  const size_t ml = merge_lds<VT>();
  const int mg = D.cus * per_cu(ml, 256, kAccumNT);
  hipLaunchKernelGGL(k_split_merge<VT>, dim3(mg), dim3(kAccumNT), ml, st, hdr, blo, sa, ccol,
                     cval);
}

hipError_t launch_num_split(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int blo,
                            const SplitArgs &sa, int32_t *ulist, const int32_t *crp,
                            int32_t *ccol, void *cval, bool f64, hipStream_t st) {
  if (sa.F <= 0) return hipSuccess;
  if (f64)
    num_split<double>(dpr, rows, hdr, blo, sa, ulist, crp, ccol, static_cast<double *>(cval), st);
  else
    num_split<float>(dpr, rows, hdr, blo, sa, ulist, crp, ccol, static_cast<float *>(cval), st);
  return hipGetLastError();
}

hipError_t configure_split_lds(size_t lds_max) {
  const void *ks[] = {
      reinterpret_cast<const void *>(&k_sym_split<true>),
      reinterpret_cast<const void *>(&k_split_merge<float>),
      reinterpret_cast<const void *>(&k_split_merge<double>),
  };
  for (const void *k : ks) {
    hipError_t e =
        hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_max);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace spg
