// What the kernels that give one block to a row (or to a piece of one) share:
// the A entries of a row over all block products spread over the block's
// threads, and the last steps of products placed by bucket in LDS.
#pragma once
#include "internal.hpp"
#include "rowops.hpp"

namespace spg {

constexpr int kBlkE = 8;  // products per thread
// Rows with at most this many repeated products (products less distinct
// columns) are ranked inside their buckets; rows with more sort them.
constexpr int kDupList = 32;

// Operand arrays of a block product, in LDS (lanes hold entries of several).
template <typename VT>
struct BlkPart {
  const SPG_GLOBAL int32_t *arp, *acol, *brp, *bcol;
  const SPG_GLOBAL VT *aval, *bval;
};

// An A entry with products: its value, its part, and its first B position
// less the number of its first product.
template <typename VT>
struct BlkEntry {
  VT a;
  int b, k;
};

template <typename VT>
__device__ __forceinline__ BlkPart<VT> blk_part(const Part &P) {
  return BlkPart<VT>{P.a_identity ? nullptr : gp(P.arp), gp(P.acol), gp(P.brp), gp(P.bcol),
                     gp(static_cast<const VT *>(P.aval)), gp(static_cast<const VT *>(P.bval))};
}

// What a thread holds of a row: the row, its place in C, the A entries per
// part (lane k of each wave: part k) and its own entry.
template <typename VT>
struct BlkHead {
  int i = -1, rs = 0, nnz = 0;
  int as = 0, incl = 0, nA = 0;
  int k = 0, r = -1, b0 = 0, len = 0;
  VT a = VT(1);
};

template <typename VT>
__device__ __forceinline__ void blk_parts(const BlkPart<VT> *part, int K, const int32_t *crp,
                                          BlkHead<VT> &h) {
  const int lane = lane_id();
  h.as = 0;
  int n = 0;
  if (h.i >= 0) {
    if (lane < K) {
      const SPG_GLOBAL int32_t *arp = part[lane].arp;
      if (arp) {
        h.as = arp[h.i];
        n = arp[h.i + 1] - h.as;
      } else {  // identity: one entry, (i, 1)
        n = 1;
      }
    }
    if (crp) {
      h.rs = __builtin_amdgcn_readfirstlane(gp(crp)[h.i]);
      h.nnz = __builtin_amdgcn_readfirstlane(gp(crp)[h.i + 1]) - h.rs;
    }
  }
  h.incl = n;
}

// Row `item` of the list (wave-uniform), or -1 past its end.
__device__ __forceinline__ int blk_row(const int32_t *list, int item, int count) {
  item = __builtin_amdgcn_readfirstlane(item);
  return (uint32_t)item < (uint32_t)count ? __builtin_amdgcn_readfirstlane(gp(list)[item]) : -1;
}

// The A entries of the row numbered part by part.
template <typename VT>
__device__ __forceinline__ void blk_number(int K, BlkHead<VT> &h) {
  static_assert(SPG_MAX_PARTS <= 16, "a scan of 16 lanes");
#pragma unroll
  for (int off = 1; off < SPG_MAX_PARTS; off <<= 1) {
    const int y = __shfl_up(h.incl, off);
    if (lane_id() >= off) h.incl += y;
  }
  h.nA = __builtin_amdgcn_readlane(h.incl, K - 1);
}

// Entry e of the row: its part, B row and value.
template <bool VALUES, typename VT>
__device__ __forceinline__ void blk_entry(const BlkPart<VT> *part, int K, int e, BlkHead<VT> &h,
                                          bool first) {
  if (first) blk_number(K, h);
  h.k = 0;
  int before = 0;
  for (int k = 0; k + 1 < K; ++k) {
    const int s = __builtin_amdgcn_readlane(h.incl, k);
    if (e >= s) {
      h.k = k + 1;
      before = s;
    }
  }
  const int as = K == 1 ? __builtin_amdgcn_readfirstlane(h.as) : __shfl(h.as, h.k);
  h.r = -1;
  if (e < h.nA) {
    const BlkPart<VT> &P = part[h.k];
    if (P.arp) {
      h.r = P.acol[as + e - before];
      if (VALUES) h.a = P.aval[as + e - before];
    } else {
      h.r = h.i;
      h.a = VT(1);
    }
  }
}

template <typename VT>
__device__ __forceinline__ void blk_bounds(const BlkPart<VT> *part, BlkHead<VT> &h) {
  h.b0 = h.len = 0;
  if (h.r >= 0) {
    const SPG_GLOBAL int32_t *brp = part[h.k].brp;
    h.b0 = brp[h.r];
    h.len = brp[h.r + 1] - h.b0;
  }
}

// Block-wide exclusive scan of v (one barrier; wt is free again after the
// caller's next one).
template <int NT>
__device__ __forceinline__ int blk_scan(int v, int *wt, int &total) {
  const int x = group_incl_scan<kWave>(v), wv = threadIdx.x / kWave;
  if (lane_id() == kWave - 1) wt[wv] = x;
  __syncthreads();
  int pre = 0;
  total = 0;
#pragma unroll
  for (int q = 0; q < NT / kWave; ++q) {
    pre += q < wv ? wt[q] : 0;
    total += wt[q];
  }
  return pre + x - v;
}

// Products of the A entries of one row in windows of 8 NT, for rows of any
// length: product p of a window goes to element p / NT of thread p % NT.
template <bool VALUES, typename VT>
struct WinEntry {
  VT a;
  int b, k;
};
template <typename VT>
struct WinEntry<false, VT> {
  int b, k;
};

template <int NT, bool VALUES, typename VT>
struct WinLds {
  static constexpr int CAP = kBlkE * NT, W = CAP / 32;
  WinEntry<VALUES, VT> ent[NT];
  uint32_t mark[W];
  int wpre[W];
  int wtot[NT / kWave], wtot2[NT / kWave];
  BlkPart<VT> part[SPG_MAX_PARTS];
};

// Entries [e0, e1) of the row whose A entries per part h holds (lane k: part
// k, as blk_parts left them).  begin() runs before a window's first product,
// between two barriers, take<j>(col, val) on every product (element j of the
// calling thread's eight), done() after the window's last one, with no
// barrier before it.  B rows longer than 2^20 entries take several turns, so
// that a chunk's product numbers fit 31 bits.
template <bool VALUES, int U, int NT, typename VT, typename Begin, typename Take, typename Done>
__device__ __forceinline__ void blk_windows(WinLds<NT, VALUES, VT> &s, int K, const BlkHead<VT> &h0,
                                            int e0, int e1, Begin begin, Take take, Done done) {
  using L = WinLds<NT, VALUES, VT>;
  constexpr int kTurn = 1 << 20;
  const int tid = threadIdx.x;
  for (int c0 = e0; c0 < e1; c0 += NT) {
    BlkHead<VT> h = h0;
    blk_entry<VALUES>(s.part, K, c0 + tid, h, false);
    if (c0 + tid >= e1) h.r = -1;
    blk_bounds(s.part, h);
    h.len = max(0, h.len);
    for (;;) {
      const int len = min(h.len, kTurn);
      // the previous window's reads are done, and long B rows known to all
      const bool more = __syncthreads_or(h.len > kTurn);
      if (tid < L::W) s.mark[tid] = 0u;
      begin();
      // products and entries with products before this thread's, in one scan
      int off, rank, tot = 0;
      {
        const int x = group_incl_scan<kWave>(len), wv = tid / kWave;
        const uint64_t any = __ballot(len > 0);
        if (lane_id() == kWave - 1) {
          s.wtot[wv] = x;
          s.wtot2[wv] = __popcll(any);
        }
        __syncthreads();
        int px = 0, py = 0;
#pragma unroll
        for (int q = 0; q < NT / kWave; ++q) {
          px += q < wv ? s.wtot[q] : 0;
          py += q < wv ? s.wtot2[q] : 0;
          tot += s.wtot[q];
        }
        off = px + x - len;
        rank = py + mbcnt(any);
      }
      const int last = off + len - 1;  // its last product
      if (len > 0) {
        auto &en = s.ent[rank];
        if constexpr (VALUES) en.a = h.a;
        en.b = h.b0 - off;
        en.k = h.k;
      }
      int before = 0;  // marks of earlier windows (wave 0)
      for (int w0 = 0; w0 < tot; w0 += L::CAP) {
        if (w0) {
          __syncthreads();
          if (tid < L::W) s.mark[tid] = 0u;
          begin();
          __syncthreads();
        }
        if (len > 0 && last >= w0 && last < w0 + L::CAP)
          atomicOr(&s.mark[(last - w0) >> 5], 1u << ((last - w0) & 31));
        __syncthreads();
        if (tid < kWave) {  // marks before each word
          constexpr int Q = (L::W + kWave - 1) / kWave;
          int pop[Q], sum = 0;
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            pop[q] = tid * Q + q < L::W ? __popc(s.mark[tid * Q + q]) : 0;
            sum += pop[q];
          }
          const int incl = group_incl_scan<kWave>(sum);
          int pre = before + incl - sum;
          before += __builtin_amdgcn_readlane(incl, kWave - 1);
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            if (tid * Q + q < L::W) s.wpre[tid * Q + q] = pre;
            pre += pop[q];
          }
        }
        __syncthreads();
        const int np = min(tot - w0, L::CAP);
#pragma unroll
        for (int j0 = 0; j0 < kBlkE; j0 += U) {
          if (j0 * NT >= np) break;
          WinEntry<VALUES, VT> en[U];
          int c[U];
          VT bv[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int p = min(tid + (j0 + u) * NT, np - 1);  // past the end: the last product
            const int w = p >> 5;
            en[u] = s.ent[s.wpre[w] + __popc(s.mark[w] & ((1u << (p & 31)) - 1u))];
            en[u].b += w0 + p;
          }
          if (K == 1) {
            const SPG_GLOBAL int32_t *bcol = s.part[0].bcol;
            const SPG_GLOBAL VT *bval = s.part[0].bval;
#pragma unroll
            for (int u = 0; u < U; ++u) {
              c[u] = bcol[en[u].b];
              bv[u] = VALUES ? bval[en[u].b] : VT(0);
            }
          } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const BlkPart<VT> &P = s.part[en[u].k];
              c[u] = P.bcol[en[u].b];
              bv[u] = VALUES ? P.bval[en[u].b] : VT(0);
            }
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (tid + (j0 + u) * NT < np) {
              VT v = VT(0);
              if constexpr (VALUES) v = en[u].a * bv[u];
              take(j0 + u, c[u], v);
            }
          }
        }
        done();
      }
      if (!more) break;
      h.b0 += kTurn;
      h.len = max(0, h.len - kTurn);
    }
  }
}

__device__ __forceinline__ int bkt_start(const uint32_t *cnt, uint32_t b) {
  return (int)((cnt[b >> 1] >> ((b & 1u) << 4)) & 0xffffu);
}

// Bucket starts from the bucket counts (four words of two a thread), in
// place; *bigmax grows to the largest count.
template <int NT>
__device__ __forceinline__ void blk_starts(uint32_t *cnt, int *bigmax, int *wt) {
  const int tid = threadIdx.x;
  const uint4 c4 = reinterpret_cast<const uint4 *>(cnt)[tid];
  uint32_t wv[4] = {c4.x, c4.y, c4.z, c4.w};
  int loc = 0, mx = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    loc += (int)(wv[j] & 0xffffu) + (int)(wv[j] >> 16);
    mx = max(mx, (int)max(wv[j] & 0xffffu, wv[j] >> 16));
  }
  mx = wave_max_last(mx);
  if (lane_id() == kWave - 1) atomicMax(bigmax, mx);
  int total;
  int run = blk_scan<NT>(loc, wt, total);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t lo = (uint32_t)run;
    run += (int)(wv[j] & 0xffffu);
    const uint32_t hi = (uint32_t)run;
    run += (int)(wv[j] >> 16);
    wv[j] = lo | (hi << 16);
  }
  reinterpret_cast<uint4 *>(cnt)[tid] = make_uint4(wv[0], wv[1], wv[2], wv[3]);
}

// By one thread, after a barrier behind blk_finish.
__device__ __forceinline__ void blk_unmoved(int *ndl, WsHeader *hdr) {
  if (ndl[1] != 0) atomicOr(&hdr->status, kStatInvalid);
  ndl[0] = ndl[1] = 0;
}

// The last steps of a row (or a segment of one, of columns from c0 on): P
// products by bucket in ikey and ival (`big`, a bucket of more than
// kBigBucket: in any order), mx the largest bucket, nnz distinct columns by
// the symbolic count.  ikey has kBigBucket words below every column before it
// and above every column behind it.  ndl[0] (the repeats listed) is 0, and so
// is ndl[1], which stays 0 unless the pattern changed: the caller looks at it
// behind its next barrier (blk_unmoved).
template <int NT, typename VT>
__device__ __forceinline__ void blk_finish(uint32_t *cnt, uint32_t *ikey, VT *ival, int P, int nnz,
                                           bool big, int mx, int *ndl, uint32_t *dlist, int *wt,
                                           int c0, SPG_GLOBAL int32_t *cb, SPG_GLOBAL VT *vb,
                                           WsHeader *hdr) {
  constexpr int T = kBlkE * NT;
  const int tid = threadIdx.x;
  const int ndup = P - nnz;  // repeated products, by the symbolic count
  if (!big && ndup >= 0 && ndup <= kDupList) {
    // few repeated columns.  Only products of one bucket can be out of
    // order, so the smaller columns of a product are those placed before
    // it, less the larger ones among its left neighbours, plus the smaller
    // ones among its right neighbours, as far as the largest bucket
    // reaches.  Its output rank is their number less the repeats among
    // them, which are listed; the first product of a column sums the
    // column's products and writes them.  (A repeat's rank is not used, so
    // an equal left neighbour may count as a larger one: every pair out of
    // order moves one rank up and one down, and where no column repeats the
    // moves add up to zero, which they don't in a changed pattern.)
    const int *kk = reinterpret_cast<const int *>(ikey);
    const int reach = __builtin_amdgcn_readfirstlane(mx);
    int c[kBlkE], r[kBlkE];
    uint32_t again = 0u;  // bit j: a repeat of an earlier product's column
#pragma unroll
    for (int j = 0; j < kBlkE; ++j) {
      r[j] = tid + j * NT;
      c[j] = kk[tid + j * NT];  // past the row: unused
    }
    for (int d = 1; d < reach; ++d) {
      const int *lo = kk + (tid - d), *hi = kk + (tid + d);
#pragma unroll
      for (int j = 0; j < kBlkE; ++j) {
        if (j * NT >= P) break;
        r[j] += hi[j * NT] < c[j] ? 1 : 0;
        r[j] -= lo[j * NT] >= c[j] ? 1 : 0;
      }
      if (ndup > 0) {
#pragma unroll
        for (int j = 0; j < kBlkE; ++j) again |= lo[j * NT] == c[j] ? 1u << j : 0u;
      }
    }
    bool bad = false;
    int nd = 0, moved = 0;
    if (ndup > 0) {
#pragma unroll
      for (int j = 0; j < kBlkE; ++j) {
        if (tid + j * NT < P && (again >> j & 1u)) {
          const int e = atomicAdd(ndl, 1);
          if (e < kDupList) dlist[e] = (uint32_t)c[j];
        }
      }
      __syncthreads();
      nd = min(*ndl, kDupList);
      bad = *ndl != ndup;  // a changed pattern
    }
#pragma unroll
    for (int j = 0; j < kBlkE; ++j) {
      const int p = tid + j * NT;
      if (p >= P) break;
      if (again >> j & 1u) continue;
      VT sum = ival[p];
      int o = r[j];
      moved += o - p;
      if (ndup > 0) {
        for (int d = 1; d < reach && p + d < P; ++d)
          if (kk[p + d] == c[j]) sum += ival[p + d];
        for (int e = 0; e < nd; ++e) o -= dlist[e] < (uint32_t)c[j] ? 1 : 0;
      }
      if (o < nnz) {
        cb[o] = c0 + c[j];
        vb[o] = sum;
      } else {
        bad = true;
      }
    }
    if (bad) atomicOr(&hdr->status, kStatInvalid);
    if (ndup == 0) {
      moved = group_incl_scan<kWave>(moved);
      if (lane_id() == kWave - 1) atomicAdd(&ndl[1], moved);
    }
    return;
  }
  // sort every bucket of two or more products by column, or the whole
  //    row when a bucket is large
  if (big) lds_sort_pairs<true, NT, VT>(ikey, ival, P, tid);
  for (int b = big ? T : tid; b < T; b += NT) {
    const int s0 = bkt_start(cnt, (uint32_t)b);
    const int s1 = b + 1 < T ? bkt_start(cnt, (uint32_t)b + 1) : P;
    for (int q = s0 + 1; q < s1; ++q) {
      const uint32_t kq = ikey[q];
      const VT vq = ival[q];
      int r = q - 1;
      while (r >= s0 && ikey[r] > kq) {
        ikey[r + 1] = ikey[r];
        ival[r + 1] = ival[r];
        --r;
      }
      ikey[r + 1] = kq;
      ival[r + 1] = vq;
    }
  }
  __syncthreads();
  // each thread a contiguous range of positions: its run starts, one
  //    block scan, then the first of each run sums the run and writes it
  {
    const int per = (P + NT - 1) / NT;
    const int p0 = tid * per, p1 = min(P, p0 + per);
    int firsts = 0;
    for (int p = p0; p < p1; ++p) firsts += (p == 0 || ikey[p] != ikey[p - 1]) ? 1 : 0;
    int total;
    int d = blk_scan<NT>(firsts, wt, total);
    for (int p = p0; p < p1; ++p) {
      const uint32_t c = ikey[p];
      if (p == 0 || c != ikey[p - 1]) {
        VT sum = ival[p];
        for (int q = p + 1; q < P && ikey[q] == c; ++q) sum += ival[q];
        if (d < nnz) {  // the symbolic count bounds the row (a changed pattern is flagged)
          cb[d] = c0 + (int)c;
          vb[d] = sum;
        }
        ++d;
      }
    }
    if (tid == 0 && total != nnz) atomicOr(&hdr->status, kStatInvalid);
  }
}

}  // namespace spg
