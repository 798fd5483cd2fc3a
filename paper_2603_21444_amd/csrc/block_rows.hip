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
// -> 2.56; 1025..2048 products 0.67 -> 0.45 and 0.33 -> 0.22.  R-MAT blocks:
// numeric 0.72 + 0.60 -> 0.41 + 0.45 ms, count 0.53 + 0.41 + 0.25 -> 0.18 +
// 0.20 + 0.11 ms.  Where it costs: B rows that stay in the caches leave the
// numbering's barriers to wait for (count of 2^16 rows of 4096 products in
// clusters of 64: 0.44 -> 0.50 ms, their numeric pass 7.21 -> 7.08; 2^15 rows of
// 4000 products of one block product: 0.51 -> 0.54 and 1.16 -> 1.00).
#include <algorithm>

#include "block_ops.hpp"
#include "internal.hpp"
#include "rowops.hpp"

namespace spg {

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
  if (threadIdx.x < SPG_MAX_PARTS && (int)threadIdx.x < pr->K)
    s.part[threadIdx.x] = blk_part<VT>(pr->part[threadIdx.x]);
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

// Waves per SIMD the kernel is compiled for (bounds its registers): three
// blocks of 512 threads fit a CU's LDS with FP32 values, six of 256, of which
// five get by without spills (8 uniform blocks, rows of 1025..2048 products:
// 0.45 ms, 0.47 at six, 0.50 at four; rows of 1300 products in bands, sorted as
// a whole: 5.54, 5.03 and 6.59, 5.35 now).
template <int NT, typename VT>
constexpr int blk_waves() {
  return sizeof(VT) == 8 || NT == 1024 ? 4 : NT == 512 ? 6 : 5;
}

template <int NT, typename VT>
__global__ __launch_bounds__(NT, (blk_waves<NT, VT>())) void k_num_block(
    const Problem *__restrict__ pr, const int32_t *__restrict__ rows, WsHeader *__restrict__ hdr,
    int bin, uint32_t mul, const int32_t *__restrict__ crp, int32_t *__restrict__ ccol,
    VT *__restrict__ cval, int32_t *__restrict__ fb_rows) {
  constexpr int CAP = kBlkE * NT;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ BlkLds<NT, VT> s;
  __shared__ int bigmax, ndl[2], item;
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
  if (tid == 0) {
    item = atomicAdd(&hdr->queue[bin], 1);
    ndl[1] = 0;
  }
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
      blk_unmoved(ndl, hdr);
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
    // (above the column; one too large to fit belongs to a row that is sorted;
    // leaving out half of them once a bucket is large: clustered rows 1 %
    // faster, others 3.5 % slower)
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
    blk_starts<NT>(cnt, &bigmax, s.wtot);
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
    blk_finish<NT, VT>(cnt, ikey, ival, P, nnz, big, bigmax, ndl, dlist, s.wtot, 0, cb, vb, hdr);
  }
  __syncthreads();
  if (tid == 0) blk_unmoved(ndl, hdr);
}

// a3 of the same rows: distinct columns by an LDS hash set with twice as many
// slots as the row may have products.
// Waves per SIMD: 512 threads spill at eight (64 registers) what six keep (80;
// 2049..4096 products: 3.05 -> 2.56 ms, five 3.39); smaller blocks spill
// nothing at eight (98 + 106 us against 104 + 109 at six).
template <int NT>
constexpr int sym_blk_waves() { return NT == 512 ? 6 : 8; }

template <int NT>
__global__ __launch_bounds__(NT, (sym_blk_waves<NT>())) void k_sym_block(const Problem *__restrict__ pr,
                                                  const int32_t *__restrict__ rows,
                                                  WsHeader *__restrict__ hdr, int bin,
                                                  int32_t *__restrict__ cnt) {
  constexpr int CAP = kBlkE * NT, T = 2 * CAP;
  constexpr int LOG2T = 31 - __builtin_clz((unsigned)T);
  extern __shared__ __align__(16) int tab[];
  __shared__ BlkLds<NT, float> s;
  __shared__ int fresh_total;
  const int tid = threadIdx.x;
  if (hdr->status) return;
  const int count = hdr->bin_count[bin];
  const int32_t *list = rows + hdr->bin_start[bin];
  const int K = pr->K;
  blk_load_parts(pr, s);
  __syncthreads();
  uint32_t it = blockIdx.x;
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
    nx.i = blk_row(list, (int)it, count);
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
  int grid = D.cus * (int)std::max<size_t>(1, std::min<size_t>(D.lds_per_cu / lds,
                                                               sym_blk_waves<NT>() * 256 / NT));
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
