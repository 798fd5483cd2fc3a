// Symbolic count (a3) and numeric pass (a5) of the rows of one block each:
// more products than the register sort takes, at most eight per thread.
//
// All A entries of a row, over all block products, are spread over the
// block's threads (entry e: thread e); a scan of their B row lengths numbers
// the row's products, a bit mask marks the last product of every entry, and
// thread t takes products t, t + NT, ...: it finds the entry of a product
// from the marks below it.  So the loads of all products of a row are issued
// together, whatever the number of parts and the lengths of the B rows, and
// the chain that leads to them (row, A bounds, A entries, B bounds) is walked
// for the next row while the current one is worked on.
//
// The count inserts the columns into an LDS hash set.  In the numeric pass
// each product takes a ticket in the bucket of its order-preserving slot
// floor(col T / n) (T = the bin's edge), a scan gives the bucket starts, and
// the products move from registers to start + ticket in LDS.  Rows with few
// repeated columns rank each product inside its bucket (less the repeats of
// smaller columns, listed first); other rows sort their buckets, rows whose
// columns cluster are sorted as a whole, and the runs of equal columns are
// summed.
//
// Bound by the gathers of B (lines of 128 bytes, at most 56 G/s) and by how
// few rows a CU holds to hide them: three of 512 threads.  Against the
// kernels that walked the row part by part, a wave each: 8 uniform blocks,
// 2^18 rows of 2600 products: numeric 7.20 -> 6.24 ms (4.9 without the ranks,
// 3.9 without ranks and stores, 2.75 without the gathers either), count 3.31
// -> 3.05; 1025..2048 products 0.67 -> 0.51 and 0.33 -> 0.22.  R-MAT blocks:
// numeric 0.72 + 0.60 -> 0.41 + 0.45 ms, count 0.53 + 0.41 + 0.25 -> 0.20 +
// 0.20 + 0.11 ms.
#include <algorithm>

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
  return item < count ? __builtin_amdgcn_readfirstlane(gp(list)[item]) : -1;
}

// Entry e of the row: its part, B row and value.
template <bool VALUES, typename VT>
__device__ __forceinline__ void blk_entry(const BlkPart<VT> *part, int K, int e, BlkHead<VT> &h,
                                          bool first) {
  if (first) {
    static_assert(SPG_MAX_PARTS <= 16, "a scan of 16 lanes");
#pragma unroll
    for (int off = 1; off < SPG_MAX_PARTS; off <<= 1) {
      const int y = __shfl_up(h.incl, off);
      if (lane_id() >= off) h.incl += y;
    }
    h.nA = __builtin_amdgcn_readlane(h.incl, K - 1);
  }
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

template <int NT, typename VT>
struct BlkLds {
  static constexpr int CAP = kBlkE * NT, W = CAP / 32;
  BlkEntry<VT> ent[NT];
  uint32_t mark[W];
  int wpre[W];
  int wtot[NT / kWave], wtot2[NT / kWave];
  BlkPart<VT> part[SPG_MAX_PARTS];
};

template <int NT, typename VT>
__device__ __forceinline__ void blk_load_parts(const Problem *__restrict__ pr, BlkLds<NT, VT> &s) {
  if (threadIdx.x < SPG_MAX_PARTS && (int)threadIdx.x < pr->K) {
    const Part &P = pr->part[threadIdx.x];
    s.part[threadIdx.x] = BlkPart<VT>{P.a_identity ? nullptr : gp(P.arp), gp(P.acol), gp(P.brp),
                                      gp(P.bcol), gp(static_cast<const VT *>(P.aval)),
                                      gp(static_cast<const VT *>(P.bval))};
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

// The products of one chunk of at most NT entries (thread t: entry t), the
// first of them product `base` of the row: product p goes to element p / NT
// of thread p % NT.  Returns the number of products so far.
template <bool VALUES, int NT, typename VT>
__device__ __forceinline__ int blk_chunk(BlkLds<NT, VT> &s, int K, const BlkHead<VT> &h, int base,
                                         int (&col)[kBlkE], VT (&val)[kBlkE]) {
  using L = BlkLds<NT, VT>;
  const int tid = threadIdx.x;
  if (tid < L::W) s.mark[tid] = 0u;
  // a changed pattern may hold more products than CAP: such rows go elsewhere
  const int len = max(0, min(h.len, L::CAP + 1));
  // products and entries with products before this thread's, in one scan
  int tot;
  int off, rank;
  {
    const int x = group_incl_scan<kWave>(len), wv = tid / kWave;
    const uint64_t any = __ballot(len > 0);
    if (lane_id() == kWave - 1) {
      s.wtot[wv] = x;
      s.wtot2[wv] = __popcll(any);
    }
    __syncthreads();
    int px = 0, py = 0;
    tot = 0;
#pragma unroll
    for (int q = 0; q < NT / kWave; ++q) {
      px += q < wv ? s.wtot[q] : 0;
      py += q < wv ? s.wtot2[q] : 0;
      tot += s.wtot[q];
    }
    off = px + x - len;
    rank = py + mbcnt(any);
  }
  const int end = base + off + len;
  if (len > 0) {
    s.ent[rank] = BlkEntry<VT>{h.a, h.b0 - (end - len), h.k};
    if (end <= L::CAP) atomicOr(&s.mark[(end - 1) >> 5], 1u << ((end - 1) & 31));
  }
  __syncthreads();
  if (tid < kWave) {  // marks before each word
    constexpr int Q = (L::W + kWave - 1) / kWave;
    int pop[Q], sum = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      pop[q] = tid * Q + q < L::W ? __popc(s.mark[tid * Q + q]) : 0;
      sum += pop[q];
    }
    int pre = group_incl_scan<kWave>(sum) - sum;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (tid * Q + q < L::W) s.wpre[tid * Q + q] = pre;
      pre += pop[q];
    }
  }
  __syncthreads();
  if (tot > 0 && base < L::CAP) {
    // half of a thread's products at a time: more would cost registers, and
    // with them resident blocks
    constexpr int U = kBlkE / 2;
#pragma unroll
    for (int j0 = 0; j0 < kBlkE; j0 += U) {
      if (j0 * NT >= base + tot) break;
      BlkEntry<VT> en[U];
      bool in[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = tid + (j0 + u) * NT;
        in[u] = p >= base && p < base + tot;
        const int w = p >> 5;
        const int e = in[u] ? s.wpre[w] + __popc(s.mark[w] & ((1u << (p & 31)) - 1u)) : 0;
        en[u] = s.ent[e];
        en[u].b += in[u] ? p : base;  // others read the chunk's first product
      }
      VT bv[U];
      int c[U];
      if (K == 1) {
        const SPG_GLOBAL int32_t *bcol = s.part[0].bcol;
        const SPG_GLOBAL VT *bval = s.part[0].bval;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          c[u] = bcol[en[u].b];
          if (VALUES) bv[u] = bval[en[u].b];
        }
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const BlkPart<VT> &P = s.part[en[u].k];
          c[u] = P.bcol[en[u].b];
          if (VALUES) bv[u] = P.bval[en[u].b];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (in[u]) {
          col[j0 + u] = c[u];
          if (VALUES) val[j0 + u] = en[u].a * bv[u];
        }
      }
    }
  }
  return min(base + tot, L::CAP + 1);
}

__device__ __forceinline__ int bkt_start(const uint32_t *cnt, uint32_t b) {
  return (int)((cnt[b >> 1] >> ((b & 1u) << 4)) & 0xffffu);
}

// Waves per SIMD the kernel is compiled for (bounds its registers): three
// blocks of 512 threads fit a CU's LDS with FP32 values.
template <int NT, typename VT>
constexpr int blk_waves() { return NT == 512 && sizeof(VT) == 4 ? 6 : 4; }

template <int NT, typename VT>
__global__ __launch_bounds__(NT, (blk_waves<NT, VT>())) void k_num_block(
    const Problem *__restrict__ pr, const int32_t *__restrict__ rows, WsHeader *__restrict__ hdr,
    int bin, uint32_t mul, const int32_t *__restrict__ crp, int32_t *__restrict__ ccol,
    VT *__restrict__ cval, int32_t *__restrict__ fb_rows) {
  constexpr int CAP = kBlkE * NT;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ BlkLds<NT, VT> s;
  __shared__ int bigmax, ndl, item;
  __shared__ uint32_t dlist[kDupList];
  const int tid = threadIdx.x;
  constexpr int T = CAP;  // buckets, two 16-bit counters per word: four words a thread
  VT *ival = reinterpret_cast<VT *>(smem_raw);
  uint32_t *cnt = reinterpret_cast<uint32_t *>(ival + CAP);
  uint32_t *ikey = cnt + T / 2 + kBigBucket;  // room for a bucket's length either side
  if (hdr->status) return;
  const int count = hdr->bin_count[bin];
  const int32_t *list = rows + hdr->bin_start[bin];
  const int K = pr->K;
  if (tid < kBigBucket) ikey[tid - kBigBucket] = 0xffffffffu;  // as an int: below every column
  blk_load_parts(pr, s);
  if (tid == 0) item = atomicAdd(&hdr->queue[bin], 1);
  __syncthreads();
  BlkHead<VT> h;
  h.i = blk_row(list, item, count);
  blk_parts(s.part, K, crp, h);
  blk_entry<true>(s.part, K, tid, h, true);
  blk_bounds(s.part, h);
  while (h.i >= 0) {
    // the previous row's last reads of the shared arrays are done
    __syncthreads();
    if (tid == 0) {
      item = atomicAdd(&hdr->queue[bin], 1);
      bigmax = 0;
      ndl = 0;
    }
    reinterpret_cast<uint4 *>(cnt)[tid] = make_uint4(0u, 0u, 0u, 0u);
    int col[kBlkE];
    VT val[kBlkE];
#pragma unroll
    for (int j = 0; j < kBlkE; ++j) {
      col[j] = -1;
      val[j] = VT(0);
    }
    int P = blk_chunk<true, NT, VT>(s, K, h, 0, col, val);
    for (int c0 = NT; c0 < h.nA; c0 += NT) {
      BlkHead<VT> g = h;
      blk_entry<true>(s.part, K, c0 + tid, g, false);
      blk_bounds(s.part, g);
      __syncthreads();
      P = blk_chunk<true, NT, VT>(s, K, g, P, col, val);
    }
    // the next row's head, a link at a time
    BlkHead<VT> nx;
    nx.i = blk_row(list, item, count);
    // tickets
    // (above the column; one too large to fit belongs to a row that is sorted)
#pragma unroll
    for (int j = 0; j < kBlkE; ++j) {
      if (col[j] >= 0) {
        const uint32_t b = mono_slot((uint32_t)col[j], mul), sh = (b & 1u) << 4;
        const uint32_t t = (atomicAdd(&cnt[b >> 1], 1u << sh) >> sh) & 0xffffu;
        col[j] |= (int)(min(t, (uint32_t)kBigBucket) << 24);
      }
    }
    __syncthreads();
    blk_parts(s.part, K, crp, nx);
    // 1. bucket starts: exclusive scan of the 16-bit counters, in place
    {
      const uint4 c4 = reinterpret_cast<const uint4 *>(cnt)[tid];
      uint32_t wv[4] = {c4.x, c4.y, c4.z, c4.w};
      int loc = 0, mx = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        loc += (int)(wv[j] & 0xffffu) + (int)(wv[j] >> 16);
        mx = max(mx, (int)max(wv[j] & 0xffffu, wv[j] >> 16));
      }
      mx = wave_max_last(mx);
      if (lane_id() == kWave - 1) atomicMax(&bigmax, mx);
      int total;
      int run = blk_scan<NT>(loc, s.wtot, total);
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
    __syncthreads();
    blk_entry<true>(s.part, K, tid, nx, true);
    const int i = h.i, rs = h.rs, nnz = h.nnz;
    SPG_GLOBAL int32_t *cb = gpw(ccol) + rs;
    SPG_GLOBAL VT *vb = gpw(cval) + rs;
    if (P > CAP) {  // a changed pattern: the fallback redoes (and flags) the row
      if (tid == 0) fb_rows[atomicAdd(&hdr->fallback_count, 1)] = i;
      blk_bounds(s.part, nx);
      h = nx;
      continue;
    }
    const bool big = bigmax > kBigBucket;
    // 2. every product to start[bucket] + ticket; clustered rows unsorted
#pragma unroll
    for (int j = 0; j < kBlkE; ++j) {
      if (col[j] >= 0) {
        const uint32_t c = (uint32_t)col[j] & 0xffffffu;
        const int pos = big ? tid + j * NT : bkt_start(cnt, mono_slot(c, mul)) + (col[j] >> 24);
        ikey[pos] = c;
        ival[pos] = val[j];
      }
    }
    if (tid < kBigBucket) ikey[P + tid] = 0x7fffffffu;  // above every column
    __syncthreads();
    blk_bounds(s.part, nx);
    h = nx;
    const int ndup = P - nnz;  // repeated products, by the symbolic count
    if (!big && ndup >= 0 && ndup <= kDupList) {
      // few repeated columns.  Only products of one bucket can be out of
      // order, so the smaller columns of a product are those placed before
      // it, less the larger ones among its left neighbours, plus the smaller
      // ones among its right neighbours, as far as the largest bucket
      // reaches.  Its output rank is their number less the repeats among
      // them, which are listed; the first product of a column sums the
      // column's products and writes them.
      const int *k0 = reinterpret_cast<const int *>(ikey);
      const int reach = __builtin_amdgcn_readfirstlane(bigmax);
      int c[kBlkE], r[kBlkE];
      uint32_t again = 0u;  // bit j: a repeat of an earlier product's column
#pragma unroll
      for (int j = 0; j < kBlkE; ++j) {
        r[j] = tid + j * NT;
        c[j] = k0[tid + j * NT];  // past the row: unused
      }
      for (int d = 1; d < reach; ++d) {
        const int *lo = k0 + (tid - d), *hi = k0 + (tid + d);
#pragma unroll
        for (int j = 0; j < kBlkE; ++j) {
          if (j * NT >= P) break;
          r[j] += hi[j * NT] < c[j] ? 1 : 0;
          r[j] -= lo[j * NT] > c[j] ? 1 : 0;
        }
        if (ndup > 0) {
#pragma unroll
          for (int j = 0; j < kBlkE; ++j) again |= lo[j * NT] == c[j] ? 1u << j : 0u;
        }
      }
      bool bad = false;
      int nd = 0;
      if (ndup > 0) {
#pragma unroll
        for (int j = 0; j < kBlkE; ++j) {
          if (tid + j * NT < P && (again >> j & 1u)) {
            const int e = atomicAdd(&ndl, 1);
            if (e < kDupList) dlist[e] = (uint32_t)c[j];
          }
        }
        __syncthreads();
        nd = min(ndl, kDupList);
        bad = ndl != ndup;  // a changed pattern
      }
#pragma unroll
      for (int j = 0; j < kBlkE; ++j) {
        const int p = tid + j * NT;
        if (p >= P) break;
        if (again >> j & 1u) {
          bad = bad || ndup == 0;
          continue;
        }
        VT sum = ival[p];
        int o = r[j];
        if (ndup > 0) {
          for (int d = 1; d < reach && p + d < P; ++d)
            if (k0[p + d] == c[j]) sum += ival[p + d];
          for (int e = 0; e < nd; ++e) o -= dlist[e] < (uint32_t)c[j] ? 1 : 0;
        }
        if (o < nnz) {
          cb[o] = c[j];
          vb[o] = sum;
        } else {
          bad = true;
        }
      }
      if (bad) atomicOr(&hdr->status, kStatInvalid);
      continue;
    }
    // 3. sort every bucket of two or more products by column, or the whole
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
    // 4. each thread a contiguous range of positions: its run starts, one
    //    block scan, then the first of each run sums the run and writes it
    {
      const int per = (P + NT - 1) / NT;
      const int p0 = tid * per, p1 = min(P, p0 + per);
      int firsts = 0;
      for (int p = p0; p < p1; ++p) firsts += (p == 0 || ikey[p] != ikey[p - 1]) ? 1 : 0;
      int total;
      int d = blk_scan<NT>(firsts, s.wtot, total);
      for (int p = p0; p < p1; ++p) {
        const uint32_t c = ikey[p];
        if (p == 0 || c != ikey[p - 1]) {
          VT sum = ival[p];
          for (int q = p + 1; q < P && ikey[q] == c; ++q) sum += ival[q];
          if (d < nnz) {  // the symbolic count bounds the row (a changed pattern is flagged)
            cb[d] = (int)c;
            vb[d] = sum;
          }
          ++d;
        }
      }
      if (tid == 0 && total != nnz) atomicOr(&hdr->status, kStatInvalid);
    }
  }
}

// a3 of the same rows: distinct columns by an LDS hash set with twice as many
// slots as the row may have products.
template <int NT>
__global__ __launch_bounds__(NT, 8) void k_sym_block(const Problem *__restrict__ pr,
                                                  const int32_t *__restrict__ rows,
                                                  WsHeader *__restrict__ hdr, int bin,
                                                  int32_t *__restrict__ cnt) {
  constexpr int CAP = kBlkE * NT, T = 2 * CAP;
  constexpr int LOG2T = 31 - __builtin_clz((unsigned)T);
  extern __shared__ __align__(16) int tab[];
  __shared__ BlkLds<NT, float> s;
  __shared__ int fresh_total, item;
  const int tid = threadIdx.x;
  if (hdr->status) return;
  const int count = hdr->bin_count[bin];
  const int32_t *list = rows + hdr->bin_start[bin];
  const int K = pr->K;
  blk_load_parts(pr, s);
  if (tid == 0) item = blockIdx.x;
  __syncthreads();
  int it = blockIdx.x;
  BlkHead<float> h;
  h.i = blk_row(list, it, count);
  blk_parts(s.part, K, nullptr, h);
  blk_entry<false>(s.part, K, tid, h, true);
  blk_bounds(s.part, h);
  while (h.i >= 0) {
    __syncthreads();  // the previous row's probes are done
    if (tid == 0) fresh_total = 0;
#pragma unroll
    for (int q = 0; q < T / 4 / NT; ++q)
      reinterpret_cast<int4 *>(tab)[tid + q * NT] = make_int4(kEmpty, kEmpty, kEmpty, kEmpty);
    int col[kBlkE];
    float val[kBlkE];
#pragma unroll
    for (int j = 0; j < kBlkE; ++j) col[j] = -1;
    it += gridDim.x;
    BlkHead<float> nx;
    nx.i = blk_row(list, it, count);
    int P = blk_chunk<false, NT, float>(s, K, h, 0, col, val);
    blk_parts(s.part, K, nullptr, nx);
    for (int c0 = NT; c0 < h.nA; c0 += NT) {
      BlkHead<float> g = h;
      blk_entry<false>(s.part, K, c0 + tid, g, false);
      blk_bounds(s.part, g);
      __syncthreads();
      P = blk_chunk<false, NT, float>(s, K, g, P, col, val);
    }
    const int i = h.i;
    blk_entry<false>(s.part, K, tid, nx, true);
    int fresh = 0;
    {
      uint32_t hh[kBlkE];
      int old[kBlkE];
#pragma unroll
      for (int j = 0; j < kBlkE; ++j) {
        hh[j] = scramble_slot((uint32_t)col[j], LOG2T);
        old[j] = col[j] >= 0 ? atomicCAS(&tab[hh[j]], kEmpty, col[j]) : col[j];
      }
#pragma unroll
      for (int j = 0; j < kBlkE; ++j) {
        if (col[j] < 0) continue;
        while (old[j] != kEmpty && old[j] != col[j]) {
          hh[j] = (hh[j] + 1) & (T - 1);
          old[j] = atomicCAS(&tab[hh[j]], kEmpty, col[j]);
        }
        fresh += old[j] == kEmpty ? 1 : 0;
      }
    }
    blk_bounds(s.part, nx);
    fresh = group_incl_scan<kWave>(fresh);
    if (lane_id() == kWave - 1) atomicAdd(&fresh_total, fresh);
    __syncthreads();
    if (tid == 0) cnt[i] = fresh_total;
    h = nx;
  }
}

// Threads of a bin's blocks: the tuned lanes per row, at least an eighth of
// the bin's edge.
int block_rows_threads(int b, int lanes) {
  int nt = std::max(128, std::max(lanes, (8 << b) / kBlkE));
  return std::min(nt, 1024);
}

template <int NT, typename VT>
static size_t num_block_dyn() {
  return (size_t)kBlkE * NT * (6 + sizeof(VT)) + 2 * kBigBucket * 4;
}

template <typename VT>
static size_t num_block_lds(int nt) {
  switch (nt) {
    case 128: return num_block_dyn<128, VT>() + sizeof(BlkLds<128, VT>) + 256;
    case 256: return num_block_dyn<256, VT>() + sizeof(BlkLds<256, VT>) + 256;
    case 512: return num_block_dyn<512, VT>() + sizeof(BlkLds<512, VT>) + 256;
    default: return num_block_dyn<1024, VT>() + sizeof(BlkLds<1024, VT>) + 256;
  }
}

// Bins served: the row fits eight products a thread and one block's LDS, and
// the columns leave the sort's keys positive.
bool block_rows_ok(int b, int lanes, int64_t n, size_t vbytes) {
  const int nt = block_rows_threads(b, lanes);
  if (n > (1 << 24) || (8 << b) > kBlkE * nt) return false;
  const size_t lds = vbytes == 8 ? num_block_lds<double>(nt) : num_block_lds<float>(nt);
  return lds <= dev_info().lds_per_block;
}

template <int NT, typename VT>
static void num_block(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int b, int count,
                      uint32_t mul, const int32_t *crp, int32_t *ccol, VT *cval, int32_t *fb,
                      hipStream_t st) {
  const DevInfo &D = dev_info();
  const size_t lds = num_block_lds<VT>(NT);
  int grid = D.cus * (int)std::max<size_t>(1, std::min<size_t>(D.lds_per_cu / lds, 2048 / NT));
  if (count >= 0) grid = std::min(grid, count);
  hipLaunchKernelGGL((k_num_block<NT, VT>), dim3(grid), dim3(NT), (num_block_dyn<NT, VT>()), st,
                     dpr, rows, hdr, b, mul, crp, ccol, cval, fb);
}

template <int NT>
static constexpr size_t sym_block_dyn() { return (size_t)2 * kBlkE * NT * 4; }

template <int NT>
static void sym_block(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int b, int count,
                      int32_t *cnt, hipStream_t st) {
  const DevInfo &D = dev_info();
  const size_t lds = sym_block_dyn<NT>() + sizeof(BlkLds<NT, float>) + 256;
  int grid = D.cus * (int)std::max<size_t>(1, std::min<size_t>(D.lds_per_cu / lds, 2048 / NT));
  if (count >= 0) grid = std::min(grid, count);
  hipLaunchKernelGGL((k_sym_block<NT>), dim3(grid), dim3(NT), sym_block_dyn<NT>(), st, dpr, rows,
                     hdr, b, cnt);
}

// Rows of bins the symbolic pass hands to k_sym_block.
bool sym_block_ok(int b, int lanes) {
  const int nt = block_rows_threads(b, lanes);
  if ((8 << b) > kBlkE * nt) return false;
  const size_t lds = (size_t)2 * kBlkE * nt * 4 + (size_t)nt * 16 + 4096;
  return lds <= dev_info().lds_per_block;
}

void launch_sym_block(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int bin, int lanes,
                      int count, int32_t *cnt, hipStream_t st) {
  switch (block_rows_threads(bin, lanes)) {
    case 128: sym_block<128>(dpr, rows, hdr, bin, count, cnt, st); break;
    case 256: sym_block<256>(dpr, rows, hdr, bin, count, cnt, st); break;
    case 512: sym_block<512>(dpr, rows, hdr, bin, count, cnt, st); break;
    default: sym_block<1024>(dpr, rows, hdr, bin, count, cnt, st); break;
  }
}

template <typename VT>
static void num_block_bin(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int b, int lanes,
                          int count, int n, const int32_t *crp, int32_t *ccol, VT *cval,
                          int32_t *fb, hipStream_t st) {
  const int nt = block_rows_threads(b, lanes);
  const uint32_t mul = mono_mul(kBlkE * nt, n);
  switch (nt) {
    case 128: num_block<128, VT>(dpr, rows, hdr, b, count, mul, crp, ccol, cval, fb, st); break;
    case 256: num_block<256, VT>(dpr, rows, hdr, b, count, mul, crp, ccol, cval, fb, st); break;
    case 512: num_block<512, VT>(dpr, rows, hdr, b, count, mul, crp, ccol, cval, fb, st); break;
    default: num_block<1024, VT>(dpr, rows, hdr, b, count, mul, crp, ccol, cval, fb, st); break;
  }
}

void launch_num_block(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int bin, int lanes,
                      int count, int n, const int32_t *crp, int32_t *ccol, void *cval, bool f64,
                      int32_t *fb, hipStream_t st) {
  if (f64)
    num_block_bin<double>(dpr, rows, hdr, bin, lanes, count, n, crp, ccol,
                          static_cast<double *>(cval), fb, st);
  else
    num_block_bin<float>(dpr, rows, hdr, bin, lanes, count, n, crp, ccol,
                         static_cast<float *>(cval), fb, st);
}

hipError_t configure_block_lds(size_t lds_max) {
  const void *ks[] = {
#define SPG_BLK_K(nt) reinterpret_cast<const void *>(&k_num_block<nt, float>), \
                      reinterpret_cast<const void *>(&k_num_block<nt, double>),
      SPG_BLK_K(128) SPG_BLK_K(256) SPG_BLK_K(512) SPG_BLK_K(1024)
#undef SPG_BLK_K
      reinterpret_cast<const void *>(&k_sym_block<128>),
      reinterpret_cast<const void *>(&k_sym_block<256>),
      reinterpret_cast<const void *>(&k_sym_block<512>),
      reinterpret_cast<const void *>(&k_sym_block<1024>),
  };
  for (const void *k : ks) {
    hipError_t e =
        hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_max);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace spg
