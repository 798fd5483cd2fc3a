// Permutation of a CSR matrix: B[prow[i], pcol[j]] = A[i, j] (paper §5.3:
// rows and columns of a structured matrix permuted uniformly at random as a
// light preprocessing step before the product; with prow = pcol it is the
// symmetric permutation P A P^T).
//
// Steps: the inverse permutations by plain stores, and a check that both
// arrays are permutations: every index in range and found again at its own
// place; the new row lengths, their scan into B's row pointer, and lists of
// the old rows by length class; then every old row, in its own order (A is
// read as a stream, and the rows of a band map the same columns one after
// the other), maps its columns and writes them in ascending order at the new
// row's place.  The new columns of a row are distinct, so an element's
// output slot is the number of the row's elements with a smaller new
// column: rows of at most 4096 entries count it over the row's columns
// staged in LDS, longer rows go through column panels (a bitmap of the
// panel's columns, a block scan of its words, then each element writes at
// its rank).
//
// Bound by chains of dependent reads and by the scattered rows of the result.
// 2^20 rows of 16 on diagonal bands, FP32 (0.50 -> 0.22 ms in all): the check
// 23 us instead of 90 (compare-and-swap into a cleared inverse, twice also
// for equal arrays), lengths and lists 23 instead of 191 (one atomic per wave
// and class on one cache line), the rows 141 instead of 197 (203 new row by
// new row, which reads A's rows at random; 172 one row at a time per group;
// 155 with eight blocks a CU instead of four).
#include <algorithm>

#include "internal.hpp"
#include "rowops.hpp"

namespace spg {

constexpr int kPermLong = 4096;    // rows longer than this take the panel kernel
constexpr int kPermPanelBits = 32768;  // columns per panel (one bitmap word per thread)

// inv[p[i]] = i for the indices in range (a repeated one: any of them).
__global__ __launch_bounds__(256) void k_perm_inverse(const int32_t *__restrict__ p, int m,
                                                      int32_t *__restrict__ pinv,
                                                      const int32_t *__restrict__ q, int n,
                                                      int32_t *__restrict__ qinv) {
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  if (p)
    for (int64_t i = t0; i < m; i += step) {
      const int v = p[i];
      if ((unsigned)v < (unsigned)m) pinv[v] = (int)i;
    }
  if (q)
    for (int64_t i = t0; i < n; i += step) {
      const int v = q[i];
      if ((unsigned)v < (unsigned)n) qinv[v] = (int)i;
    }
}

// p is a permutation exactly when all its indices are in range and each is
// the last (only) one stored at its place.
__global__ __launch_bounds__(256) void k_perm_check(const int32_t *__restrict__ p, int m,
                                                    const int32_t *__restrict__ pinv,
                                                    const int32_t *__restrict__ q, int n,
                                                    const int32_t *__restrict__ qinv,
                                                    WsHeader *hdr) {
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  bool bad = false;
  if (p)
    for (int64_t i = t0; i < m; i += step) {
      const int v = p[i];
      bad = bad || (unsigned)v >= (unsigned)m || pinv[v] != (int)i;
    }
  if (q)
    for (int64_t i = t0; i < n; i += step) {
      const int v = q[i];
      bad = bad || (unsigned)v >= (unsigned)n || qinv[v] != (int)i;
    }
  if (bad) atomicOr(&hdr->status, kStatInvalid);
}

// Length classes of the new rows: (0, 16], (16, 64], (64, 256], (256, 1024],
// (1024, 4096] (groups of 16, 16, 64, 256 and 1024 lanes) and longer (in
// panels); empty rows need no work.
constexpr int kPermClasses = 6;
constexpr int kPermLists = 5;  // of m places each

__device__ __forceinline__ int perm_class(int len) {
  return len <= 0     ? -1
         : len <= 16  ? 0
         : len <= 64  ? 1
         : len <= 256 ? 2
         : len <= 1024 ? 3
         : len <= kPermLong ? 4
                            : 5;
}

// Place of row `at` of class c among the lists: one list per class, the last
// two classes share one from both ends.
__device__ __forceinline__ int64_t perm_place(int c, int at, int m) {
  return c < kPermLists ? (int64_t)c * m + at : (int64_t)kPermLists * m - 1 - at;
}

// Length of every new row, and the old row in its class's list (length
// hdr->bin_count[c]).  A block takes a run of consecutive rows, so that one
// atomic per class and block reserves its places; the rows of a list stay in
// runs.
__global__ __launch_bounds__(256) void k_perm_len(const int32_t *__restrict__ arp,
                                                  const int32_t *__restrict__ prow, int m,
                                                  int per, int32_t *__restrict__ cnt,
                                                  int32_t *__restrict__ lists, WsHeader *hdr) {
  __shared__ int have[kPermClasses], next[kPermClasses];
  if (hdr->status) return;
  if (threadIdx.x < kPermClasses) have[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t below = lanes_below();
  const int64_t lo = (int64_t)blockIdx.x * per, hi = min((int64_t)m, lo + per);
  // whole waves step together, so the ballots below see every lane
  for (int64_t i0 = lo; i0 < hi; i0 += 256) {
    const int64_t i = i0 + threadIdx.x;
    int cls = -1;
    if (i < hi) {
      const int len = arp[i + 1] - arp[i];
      cnt[prow ? prow[i] : i] = len;
      cls = perm_class(len);
    }
#pragma unroll
    for (int c = 0; c < kPermClasses; ++c) {
      const uint64_t mk = __ballot(cls == c);
      if (mk && lane_id() == 0) atomicAdd(&have[c], __popcll(mk));
    }
  }
  __syncthreads();
  if (threadIdx.x < kPermClasses)
    next[threadIdx.x] = have[threadIdx.x] ? atomicAdd(&hdr->bin_count[threadIdx.x], have[threadIdx.x]) : 0;
  __syncthreads();
  for (int64_t i0 = lo; i0 < hi; i0 += 256) {
    const int64_t i = i0 + threadIdx.x;
    const int cls = i < hi ? perm_class(arp[i + 1] - arp[i]) : -1;
#pragma unroll
    for (int c = 0; c < kPermClasses; ++c) {
      const uint64_t mk = __ballot(cls == c);
      if (mk == 0) continue;
      int base = 0;
      if (lane_id() == 0) base = atomicAdd(&next[c], __popcll(mk));
      base = __shfl(base, 0);
      if (cls == c) lists[perm_place(c, base + __popcll(mk & below), m)] = (int)i;
    }
  }
}

// Adds to the ranks of a lane's first T elements the row's smaller columns.
template <int T, int E>
__device__ __forceinline__ void perm_ranks(const int *key_s, int len, const int (&key)[E],
                                           int (&rank)[E]) {
  for (int q = 0; q < len; q += 4) {  // places past the row rank last
    const int4 k4 = *reinterpret_cast<const int4 *>(key_s + q);
#pragma unroll
    for (int t = 0; t < T; ++t)
      rank[t] += (k4.x < key[t]) + (k4.y < key[t]) + (k4.z < key[t]) + (k4.w < key[t]);
  }
}

// Rows of a length class (at most E G entries): G lanes per row, elements
// e = l + t G of U rows at a time, so that U rows' chains of dependent reads
// run side by side; the heads of the next rows (old row, its bounds, the new
// row's place) are read while the current ones are written.
template <int G, int E, int U, typename VT>
__device__ __forceinline__ void perm_rows(const int32_t *__restrict__ arp,
                                          const int32_t *__restrict__ acol,
                                          const VT *__restrict__ aval,
                                          const int32_t *__restrict__ prow,
                                          const int32_t *__restrict__ pcol,
                                          const int32_t *__restrict__ list, int count,
                                          const int32_t *__restrict__ brp,
                                          int32_t *__restrict__ bcol, VT *__restrict__ bval,
                                          int *key_s) {
  constexpr int CAP = E * G;  // places of a row in key_s
  constexpr bool BLOCK = G > kWave;
  static_assert(CAP % 4 == 0, "columns are compared four at a time");
  const int R = (int)blockDim.x / G;
  const int l = threadIdx.x % G;
  const int ngroups = gridDim.x * R;
  int idx = blockIdx.x * R + threadIdx.x / G;  // group g takes list entries g U .. g U + U - 1
  // groups of one wave (or block) step together
  int lead = blockIdx.x * R + (BLOCK ? 0 : (int)(threadIdx.x / kWave) * (kWave / G));
  int i1[U], r1[U], i2[U], s[U], len[U], o[U];
  auto rows_at = [&](int g, int (&i)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) i[u] = (int64_t)g * U + u < count ? list[g * U + u] : -1;
  };
  auto new_of = [&](const int (&i)[U], int (&r)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = i[u] < 0 ? -1 : (prow ? prow[i[u]] : i[u]);
  };
  auto bounds = [&](const int (&i)[U], const int (&r)[U], int (&s)[U], int (&len)[U], int (&o)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s[u] = len[u] = o[u] = 0;
      if (i[u] >= 0) {
        s[u] = arp[i[u]];
        len[u] = arp[i[u] + 1] - s[u];
        o[u] = brp[r[u]];
      }
    }
  };
  rows_at(idx, i1);
  new_of(i1, r1);
  bounds(i1, r1, s, len, o);
  rows_at(idx + ngroups, i1);
  new_of(i1, r1);
  rows_at(idx + 2 * ngroups, i2);
  const int nlists = (int)(((int64_t)count + U - 1) / U);
  for (; lead < nlists; lead += ngroups, idx += ngroups) {
    int key[U][E], rank[U][E];
    VT v[U][E];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < E; ++t) {
        const int e = l + t * G;
        key[u][t] = -1;
        v[u][t] = VT(0);
        rank[u][t] = 0;
        if (e < len[u]) {
          key[u][t] = acol[s[u] + e];
          if (aval) v[u][t] = aval[s[u] + e];
        }
      }
    int s1[U], len1[U], o1[U], r2[U], i3[U];
    bounds(i1, r1, s1, len1, o1);
    new_of(i2, r2);
    rows_at(idx + 3 * ngroups, i3);
    if (pcol) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < E; ++t)
          if (key[u][t] >= 0) key[u][t] = pcol[key[u][t]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < E; ++t)
        key_s[u * CAP + l + t * G] = key[u][t] < 0 ? INT32_MAX : key[u][t];
    group_sync<BLOCK>();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // no compares for elements that no lane of the wave holds
      int held = 1;
#pragma unroll
      for (int t = 1; t < E; ++t) held += __any(key[u][t] >= 0) ? 1 : 0;
      switch (held) {
        case 1: perm_ranks<1, E>(key_s + u * CAP, len[u], key[u], rank[u]); break;
        case 2: perm_ranks<E < 2 ? E : 2, E>(key_s + u * CAP, len[u], key[u], rank[u]); break;
        case 3: perm_ranks<E < 3 ? E : 3, E>(key_s + u * CAP, len[u], key[u], rank[u]); break;
        default: perm_ranks<E, E>(key_s + u * CAP, len[u], key[u], rank[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < E; ++t) {
        if (key[u][t] >= 0) {
          bcol[o[u] + rank[u][t]] = key[u][t];
          if (bval) bval[o[u] + rank[u][t]] = v[u][t];
        }
      }
    group_sync<BLOCK>();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s[u] = s1[u];
      len[u] = len1[u];
      o[u] = o1[u];
      i1[u] = i2[u];
      r1[u] = r2[u];
      i2[u] = i3[u];
    }
  }
}

// Rows of at most 1024 entries, but for those of 65..256.
template <typename VT>
__global__ __launch_bounds__(256) void k_perm_short(
    const int32_t *__restrict__ arp, const int32_t *__restrict__ acol,
    const VT *__restrict__ aval, const int32_t *__restrict__ prow,
    const int32_t *__restrict__ pcol, const int32_t *__restrict__ lists, int m,
    const int32_t *__restrict__ brp, int32_t *__restrict__ bcol, VT *__restrict__ bval,
    const WsHeader *hdr) {
  __shared__ __align__(16) int skey[1024];
  if (hdr->status) return;
  const int t = threadIdx.x;
  perm_rows<16, 1, 4, VT>(arp, acol, aval, prow, pcol, lists, hdr->bin_count[0], brp, bcol, bval,
                       skey + t / 16 * 64);
  perm_rows<16, 4, 1, VT>(arp, acol, aval, prow, pcol, lists + m, hdr->bin_count[1], brp, bcol, bval,
                       skey + t / 16 * 64);
  __syncthreads();
  perm_rows<256, 4, 1, VT>(arp, acol, aval, prow, pcol, lists + (size_t)3 * m, hdr->bin_count[3],
                           brp, bcol, bval, skey);
}

// The other rows, two blocks of 1024 threads a CU: 65..256 entries in groups
// of 64 lanes, 1025..kPermLong one block per row, and the longest in panels of
// kPermPanelBits new columns: a bitmap marks the row's columns, a block scan
// of its words gives each word's starting rank, and every element writes at
// that rank plus the marks below it in its word (columns are distinct).
//
// Rows of 257..1024 entries are better off in k_perm_short: their barriers
// then hold up four waves, not sixteen (2^23 entries in rows of 300, in all:
// 0.25 ms against 0.28).  Bound by the compares, so those of elements that a
// wave does not hold are left out (0.25 against 0.55; rows of 1500 0.76
// against 1.87).  One block of 1024 threads a CU for every row of more than
// 256 entries, all compares made: rows of 300 / 700 / 1500 / 4000 took 2.07 /
// 2.02 / 2.01 / 2.18 ms, now 0.25 / 0.43 / 0.76 / 2.02.
template <typename VT>
__global__ __launch_bounds__(1024, 8) void k_perm_long(
    const int32_t *__restrict__ arp, const int32_t *__restrict__ acol,
    const VT *__restrict__ aval, const int32_t *__restrict__ prow,
    const int32_t *__restrict__ pcol, int m, int ncols, const int32_t *__restrict__ lists,
    const int32_t *__restrict__ brp, int32_t *__restrict__ bcol, VT *__restrict__ bval,
    const WsHeader *hdr) {
  static_assert(kPermPanelBits / 32 == 1024, "one bitmap word per thread");
  __shared__ uint32_t bm[kPermPanelBits / 32];
  __shared__ int wpre[kPermPanelBits / 32];
  __shared__ int wtot[1024 / kWave];
  __shared__ __align__(16) int skey[kPermLong];
  if (hdr->status) return;
  const int tid = threadIdx.x;
  perm_rows<64, 4, 1, VT>(arp, acol, aval, prow, pcol, lists + (size_t)2 * m, hdr->bin_count[2],
                          brp, bcol, bval, skey + tid / 64 * 256);
  __syncthreads();  // the groups' parts of skey change
  perm_rows<1024, 4, 1, VT>(arp, acol, aval, prow, pcol, lists + (size_t)4 * m, hdr->bin_count[4],
                            brp, bcol, bval, skey);
  const int count = hdr->bin_count[5];
  for (int li = blockIdx.x; li < count; li += gridDim.x) {
    const int i = lists[perm_place(5, li, m)];
    const int s = arp[i], len = arp[i + 1] - s;
    int base = brp[prow ? prow[i] : i];
    for (int plo = 0; plo < ncols; plo += kPermPanelBits) {
      bm[tid] = 0u;
      __syncthreads();
      for (int e = tid; e < len; e += 1024) {
        const int c0 = acol[s + e];
        const uint32_t c = (uint32_t)((pcol ? pcol[c0] : c0) - plo);
        if (c < (uint32_t)kPermPanelBits) atomicOr(&bm[c >> 5], 1u << (c & 31));
      }
      __syncthreads();
      int total;
      wpre[tid] = group_excl_scan<true, 1024>(__popc(bm[tid]), tid, wtot, total);
      __syncthreads();
      for (int e = tid; e < len; e += 1024) {
        const int c0 = acol[s + e];
        const int cn = pcol ? pcol[c0] : c0;
        const uint32_t c = (uint32_t)(cn - plo);
        if (c < (uint32_t)kPermPanelBits) {
          const int w = (int)(c >> 5);
          const int pos = base + wpre[w] + __popc(bm[w] & ((1u << (c & 31)) - 1u));
          bcol[pos] = cn;
          if (bval) bval[pos] = aval[s + e];
        }
      }
      __syncthreads();
      base += total;
    }
  }
}

size_t perm_workspace_bytes(int64_t m, int64_t n, size_t *rinv_off, size_t *cinv_off,
                            size_t *long_off, size_t *scan_off) {
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  size_t o = 4096;  // header
  *rinv_off = o;
  o = al(o + 4 * (size_t)(m > 0 ? m : 1));
  *cinv_off = o;
  o = al(o + 4 * (size_t)(n > 0 ? n : 1));
  *long_off = o;  // the row lists of the length classes
  o = al(o + 4 * (size_t)kPermLists * (size_t)(m > 0 ? m : 1));
  *scan_off = o;
  o = al(o + 8 * (size_t)((m + 2047) / 2048 + 1));
  return o;
}

template <typename VT>
static hipError_t permute_impl(const int32_t *arp, const int32_t *acol, const void *aval,
                               const int32_t *prow, const int32_t *pcol, int m, int n,
                               const int32_t *brp, int32_t *bcol, void *bval,
                               const int32_t *lists, const WsHeader *hdr, hipStream_t st) {
  const DevInfo &D = dev_info();
  // persistent grids over the classes' lists (their lengths are on the device)
  const int grid = std::max(1, std::min(m, D.cus * 4));
  hipLaunchKernelGGL((k_perm_short<VT>), dim3(grid), dim3(256), 0, st, arp, acol,
                     static_cast<const VT *>(aval), prow, pcol, lists, m, brp, bcol,
                     static_cast<VT *>(bval), hdr);
  hipLaunchKernelGGL((k_perm_long<VT>), dim3(std::max(1, std::min(m, D.cus * 2))), dim3(1024), 0, st,
                     arp, acol, static_cast<const VT *>(aval), prow, pcol, m, n, lists, brp, bcol,
                     static_cast<VT *>(bval), hdr);
  return hipGetLastError();
}

hipError_t launch_permute(const spg_csr &A, const int32_t *prow, const int32_t *pcol,
                          int dtype, int32_t *brp, int32_t *bcol, void *bval, char *ws,
                          hipStream_t st) {
  const int m = A.nrows, n = A.ncols;
  size_t ro, co, lo, so;
  (void)perm_workspace_bytes(m, n, &ro, &co, &lo, &so);
  WsHeader *hdr = reinterpret_cast<WsHeader *>(ws);
  int32_t *rinv = prow ? reinterpret_cast<int32_t *>(ws + ro) : nullptr;
  int32_t *cinv = reinterpret_cast<int32_t *>(ws + co);
  int32_t *longrows = reinterpret_cast<int32_t *>(ws + lo);
  const DevInfo &D = dev_info();
  const int g = D.cus * 4;
  // the column array is checked as well (its inverse is not used); equal
  // arrays of equal length are checked once
  const int32_t *q = pcol == prow && m == n ? nullptr : pcol;
  if (prow || q) {
    hipLaunchKernelGGL(k_perm_inverse, dim3(g), dim3(256), 0, st, prow, m, rinv, q, n, cinv);
    hipLaunchKernelGGL(k_perm_check, dim3(g), dim3(256), 0, st, prow, m, rinv, q, n, cinv, hdr);
  }
  // runs of whole waves, at most g blocks
  const int per = (int)((((int64_t)m + g - 1) / g + 255) / 256 * 256);
  const int runs = m > 0 ? (int)(((int64_t)m + per - 1) / per) : 1;
  hipLaunchKernelGGL(k_perm_len, dim3(runs), dim3(256), 0, st, A.row_ptr, prow, m, per, brp,
                     longrows, hdr);
  WsLayout L{};
  L.scanpart = so;
  hipError_t e = launch_scan(brp, m, -1, L, ws, st);
  if (e != hipSuccess) return e;
  if (dtype == SPG_F64)
    return permute_impl<double>(A.row_ptr, A.col_idx, A.vals, prow, pcol, m, n, brp, bcol, bval,
                                longrows, hdr, st);
  return permute_impl<float>(A.row_ptr, A.col_idx, A.vals, prow, pcol, m, n, brp, bcol, bval,
                             longrows, hdr, st);
}

}  // namespace spg
