// Numeric pass (a5) of rows whose products fit the registers of one group of
// lanes: the products are sorted there by column.
//
// A group of G lanes (16, 32 or 64, inside one wave) holds a row's products,
// E per lane.  Product p of the row (A entry by A entry, in stored order) is
// element p / G of lane p % G: the group scans the lengths of its B rows,
// marks each entry's first product in a bit mask, and every lane finds the
// entry of its products by counting the marks up to them.  So all loads of B
// of a row are issued together, neighbouring lanes read neighbouring
// elements of B, and no lane idles whatever the lengths of the B rows.  The
// keys (column << log2(G E) | p) are sorted by a bitonic network in
// registers; the value of a product stays in LDS at p.  Lane l then holds
// the products of ranks l E .. l E + E - 1 and writes them with one wide
// store.  Where columns repeat (more products than the row of C has
// entries), the sorted keys go to LDS and the first product of a column sums
// the column's products, in stored order.
//
// A step of the network costs two vector instructions per element across
// lanes (a DPP move or half a v_permlane*_swap, and a v_med3 that keeps the
// smaller or the larger key) and one inside a lane; no data-dependent loops,
// and clustered columns cost the same as spread ones.
//
// What bounds it on unstructured rows is the gathers: a random read from
// beyond the L2 fetches a 128-byte line, at most 56 G lines/s, and every A
// entry takes three (bounds, columns and values of its B row).  2^20 rows of
// 256 FP32 products: 1.29 ms against 1.40 for the LDS bucket kernel this
// replaces (1.27 without the comparison of neighbours that flags a changed
// pattern, of which 0.92 with synthetic columns, 0.90 without the stores, 1.22
// without the sort; 414 vector instructions a row against 582).  Rows that
// cluster in bands, which that kernel sorted in LDS: 1.45 against 5.40 ms.
// Rows of 257..512 and 513..1024 products against the block bucket kernel:
// R-MAT blocks 0.32 against 0.84 ms and 0.13 against 0.18 ms (FP32), ragged
// FP64 rows 0.10 against 0.42 and 0.36 against 0.51 ms.  32 elements a lane
// (1025..2048 products) lose to it: 0.91 against 0.61 ms (few waves, spills).
#include <algorithm>

#include "internal.hpp"
#include "rowops.hpp"

namespace spg {

template <int G>
__device__ __forceinline__ int group_uniform(int v) {
  return G == kWave ? __builtin_amdgcn_readfirstlane(v) : v;
}

template <int G>
__device__ __forceinline__ int group_last(int v) {
  return G == kWave ? __builtin_amdgcn_readlane(v, kWave - 1) : __shfl(v, G - 1, G);
}

// lim = 0: the smaller of a and b; lim = ~0: the larger (one v_med3_u32).
__device__ __forceinline__ uint32_t pick(uint32_t a, uint32_t b, uint32_t lim) {
  return max(min(a, b), min(max(a, b), lim));
}

// One step of the network across lanes: lanes l and l ^ D compare element by
// element, the lane with bit D clear keeps the smaller.
template <int D, int E>
__device__ __forceinline__ void clean_lanes(uint32_t (&x)[E], uint32_t lim) {
  if constexpr (D >= 16 && E >= 2) {
    // the swap brings both keys of a pair into one lane, for two elements
#pragma unroll
    for (int t = 0; t < E; t += 2) {
      auto a = D == 16 ? __builtin_amdgcn_permlane16_swap(x[t], x[t + 1], false, false)
                       : __builtin_amdgcn_permlane32_swap(x[t], x[t + 1], false, false);
      const uint32_t lo = min((uint32_t)a[0], (uint32_t)a[1]);
      const uint32_t hi = max((uint32_t)a[0], (uint32_t)a[1]);
      auto b = D == 16 ? __builtin_amdgcn_permlane16_swap(lo, hi, false, false)
                       : __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
      x[t] = b[0];
      x[t + 1] = b[1];
    }
  } else if constexpr (D >= 16) {
    auto a = D == 16 ? __builtin_amdgcn_permlane16_swap(x[0], x[0], false, false)
                     : __builtin_amdgcn_permlane32_swap(x[0], x[0], false, false);
    x[0] = pick(a[0], a[1], lim);
  } else {
#pragma unroll
    for (int t = 0; t < E; ++t) {
      uint32_t y;
      if (D == 1) y = dpp<0xB1>(x[t]);                   // quad_perm [1, 0, 3, 2]
      else if (D == 2) y = dpp<0x4E>(x[t]);              // quad_perm [2, 3, 0, 1]
      else if (D == 4) y = dpp<0x1B>(dpp<0x141>(x[t]));  // mirrored eights, mirrored quads
      else y = dpp<0x128>(x[t]);                         // row_ror 8
      x[t] = pick(x[t], y, lim);
    }
  }
}

// Merge of a bitonic sequence held by one lane.
template <int E>
__device__ __forceinline__ void clean_elements(uint32_t (&x)[E]) {
#pragma unroll
  for (int d = E / 2; d > 0; d >>= 1) {
#pragma unroll
    for (int t = 0; t < E; ++t) {
      if ((t & d) == 0) {
        const uint32_t lo = min(x[t], x[t + d]), hi = max(x[t], x[t + d]);
        x[t] = lo;
        x[t + d] = hi;
      }
    }
  }
}

// Ascending sort of the G E keys of a group, position of element t of lane
// l: l E + t.  Blocks that a bitonic sort holds in descending order are
// complemented instead, so that every step keeps the smaller key at the
// lower position.
template <int G, int E>
__device__ __forceinline__ void group_sort(uint32_t (&x)[E], int l) {
  uint32_t m[6];  // m[b]: all ones where bit b of the lane is set
#pragma unroll
  for (int b = 0; b < 6; ++b) m[b] = (1 << b) < G ? (uint32_t)((l << (31 - b)) >> 31) : 0u;
#pragma unroll
  for (int t = 0; t < E; ++t) x[t] ^= m[0];
  // inside a lane: merges of 2, 4, ..., E elements, mirrored first steps
#pragma unroll
  for (int k = 2; k <= E; k <<= 1) {
#pragma unroll
    for (int t = 0; t < E; ++t) {
      const int u = t ^ (k - 1);
      if (t < u) {
        const uint32_t lo = min(x[t], x[u]), hi = max(x[t], x[u]);
        x[t] = lo;
        x[u] = hi;
      }
    }
#pragma unroll
    for (int d = k / 4; d > 0; d >>= 1) {
#pragma unroll
      for (int t = 0; t < E; ++t) {
        if ((t & d) == 0) {
          const uint32_t lo = min(x[t], x[t + d]), hi = max(x[t], x[t + d]);
          x[t] = lo;
          x[t + d] = hi;
        }
      }
    }
  }
  // merges of 2, 4, ..., G lanes
#pragma unroll
  for (int b = 0; (1 << b) < G; ++b) {
    const uint32_t flip = m[b] ^ ((2 << b) < G ? m[b + 1] : 0u);
#pragma unroll
    for (int t = 0; t < E; ++t) x[t] ^= flip;
    if (b >= 5) clean_lanes<32, E>(x, m[5]);
    if (b >= 4) clean_lanes<16, E>(x, m[4]);
    if (b >= 3) clean_lanes<8, E>(x, m[3]);
    if (b >= 2) clean_lanes<4, E>(x, m[2]);
    if (b >= 1) clean_lanes<2, E>(x, m[1]);
    clean_lanes<1, E>(x, m[0]);
    clean_elements<E>(x);
  }
}

constexpr int ilog2(int v) { return v <= 1 ? 0 : 1 + ilog2(v / 2); }

// An A entry with products: its value, and its first B position less the
// number of its first product.
template <typename VT>
struct SortEntry {
  VT a;
  int b;
};

// LDS of one group.
template <int G, int E, typename VT>
struct SortLds {
  static constexpr int CAP = G * E;
  VT val[CAP];                     // value of product p
  SortEntry<VT> entry[G];
  uint32_t key[CAP];               // sorted keys (rows with repeated columns)
  uint32_t mark[(CAP + 31) / 32];  // bit p: product p is the last of its entry
};

// The products of one chunk of at most G entries (lane l: entry l; length 0:
// none), the first of them product `base` of the row.  Returns the number
// of products so far.
// PAIR: B is read as words of column and FP32 value.  VALUES false: the keys
// are the columns alone.
template <int G, int E, bool PAIR, bool VALUES, typename VT>
__device__ __forceinline__ int sort_chunk(SortLds<G, E, VT> &s, const SPG_GLOBAL int32_t *bcol,
                                          const SPG_GLOBAL VT *bval,
                                          const SPG_GLOBAL unsigned long long *pair, int l, int b0,
                                          int len, VT a, int base, uint32_t (&key)[E]) {
  constexpr int CAP = G * E, W = (CAP + 31) / 32, IB = ilog2(CAP);
  static_assert(W <= G, "one lane clears one word of the marks");
  if (l < W) s.mark[l] = 0u;
  len = max(0, min(len, CAP + 1));  // a changed pattern: more products than CAP go elsewhere
  const int incl = group_incl_scan<G>(len);
  const int tot = group_last<G>(incl);
  const int end = base + incl;
  const uint64_t any = __ballot(len > 0);
  const uint64_t gm = G == kWave ? ~0ull : ((1ull << G) - 1ull) << (lane_id() & ~(G - 1));
  const int rank = mbcnt(any & gm);
  group_sync<false>();
  if (len > 0) {
    s.entry[rank] = SortEntry<VT>{a, b0 - (end - len)};
    if (end <= CAP) atomicOr(&s.mark[(end - 1) >> 5], 1u << ((end - 1) & 31));
  }
  group_sync<false>();
  if (tot > 0 && base < CAP) {
    // entry of product p: the last products below p
    uint32_t w[W];
    int pre[W];
    int c = 0;
#pragma unroll
    for (int j = 0; j < W; ++j) {
      w[j] = s.mark[j];
      pre[j] = c;
      c += __popc(w[j]);
    }
    int e[E];
    bool in[E];
#pragma unroll
    for (int t = 0; t < E; ++t) {
      const int p = t * G + l;
      if constexpr (G == kWave) {
        e[t] = __builtin_amdgcn_mbcnt_hi(w[2 * t + 1],
                                         __builtin_amdgcn_mbcnt_lo(w[2 * t], pre[2 * t]));
      } else {
        const int j = (t * G) >> 5, sh = ((t * G) & 31) + l;
        e[t] = pre[j] + __popc(__builtin_amdgcn_ubfe(w[j], 0, sh));
      }
      in[t] = p >= base && p < base + tot;
      e[t] = in[t] ? e[t] : 0;
    }
    // every lane loads (products outside the chunk: its first one), so that
    // all loads of the row are in flight together
    SortEntry<VT> en[E];
#pragma unroll
    for (int t = 0; t < E; ++t) en[t] = s.entry[e[t]];
    int col[E];
    VT bv[E];
    if constexpr (PAIR) {
#pragma unroll
      for (int t = 0; t < E; ++t) {
        const unsigned long long w = pair[en[t].b + (in[t] ? t * G + l : base)];
        col[t] = (int)(uint32_t)w;
        bv[t] = (VT)__uint_as_float((uint32_t)(w >> 32));
      }
    } else {
#pragma unroll
      for (int t = 0; t < E; ++t) {
        const int q = en[t].b + (in[t] ? t * G + l : base);
        col[t] = bcol[q];
        bv[t] = VALUES ? bval[q] : VT(0);
      }
    }
#pragma unroll
    for (int t = 0; t < E; ++t) {
      const uint32_t p = (uint32_t)(t * G + l);
      if (in[t]) {
        key[t] = VALUES ? ((uint32_t)col[t] << IB) | p : (uint32_t)col[t];
        if (VALUES) s.val[p] = en[t].a * bv[t];
      }
    }
  }
  group_sync<false>();
  return base + tot;
}

// Chain of dependent loads that precedes a row's products, walked for the
// next rows while the current one is worked on: row id, A row bounds, A
// entries, B row bounds.
template <int G, typename VT>
struct SortNext {
  bool has = false;
  int i = 0, as = 0, ae = 0, rs = 0, re = 0;
  int r = -1;
  VT a = VT(1);
  __device__ __forceinline__ void row(const int32_t *rows, uint32_t ri, uint32_t count) {
    has = ri < count;
    i = has ? group_uniform<G>(gp(rows)[ri]) : 0;
  }
  __device__ __forceinline__ void bounds(const Part &P, const int32_t *crp) {
    if (!has) return;
    int s, e;
    a_row(P, i, s, e);
    as = group_uniform<G>(s);
    ae = group_uniform<G>(e);
    if (crp) {
      rs = group_uniform<G>(gp(crp)[i]);
      re = group_uniform<G>(gp(crp)[i + 1]);
    }
  }
  template <bool VALUES = true>
  __device__ __forceinline__ void entry(const Part &P, int l) {
    r = -1;
    if (!has || l >= ae - as) return;
    if (VALUES) a_entry<VT>(P, i, as + l, r, a);
    else r = a_entry_row(P, i, as + l);
  }
};

// Waves per SIMD the kernel is compiled for (bounds its registers).
template <int G, int E>
constexpr int sort_waves() { return E > 4 ? 4 : (E == 4 && G < kWave ? 6 : 8); }

// PAIR: B read as words of column and FP32 value (Part::pair).
template <int G, int E, bool PAIR, typename VT>
__global__ __launch_bounds__(256, (sort_waves<G, E>())) void k_num_sort(
    const Problem *__restrict__ pr, const int32_t *__restrict__ rows, WsHeader *__restrict__ hdr,
    int bin, const int32_t *__restrict__ crp, int32_t *__restrict__ ccol, VT *__restrict__ cval,
    int32_t *__restrict__ fb_rows) {
  constexpr int CAP = G * E, IB = ilog2(CAP), R = 256 / G;
  __shared__ SortLds<G, E, VT> lds[R];
  if (hdr->status) return;
  const int slot = group_uniform<G>(threadIdx.x / G), l = threadIdx.x % G;
  SortLds<G, E, VT> &s = lds[slot];
  // unsigned: a list may hold nearly 2^31 rows
  const uint32_t count = hdr->bin_count[bin];
  const int32_t *list = rows + hdr->bin_start[bin];
  const uint32_t stride = gridDim.x * R;
  const Part &P0 = pr->part[0];
  const SPG_GLOBAL int32_t *bcol0 = gp(P0.bcol);
  const SPG_GLOBAL VT *bval0 = gp(static_cast<const VT *>(P0.bval));
  const SPG_GLOBAL unsigned long long *pair0 = PAIR ? gp(P0.pair) : nullptr;
  const int K = pr->K;
  uint32_t ri = blockIdx.x * R + slot;
  // a wave runs while any of its groups has a row
  uint32_t wri = blockIdx.x * R + (G == kWave ? slot : (int)(threadIdx.x / kWave) * (kWave / G));
  SortNext<G, VT> n0, n1, n2;
  n0.row(list, ri, count);
  n0.bounds(P0, crp);
  n0.entry(P0, l);
  int b0 = 0, len = 0;
  if (n0.r >= 0) {
    b0 = gp(P0.brp)[n0.r];
    len = gp(P0.brp)[n0.r + 1] - b0;
  }
  n1.row(list, ri + stride, count);
  n1.bounds(P0, crp);
  n2.row(list, ri + 2 * stride, count);
  bool again = false;
  for (; wri < count; wri += stride, ri += stride) {
    n1.entry(P0, l);
    uint32_t key[E];
#pragma unroll
    for (int t = 0; t < E; ++t) key[t] = 0xffffffffu;
    int P = sort_chunk<G, E, PAIR, true, VT>(s, bcol0, bval0, pair0, l, b0, len, n0.a, 0, key);
    b0 = len = 0;  // the next row's first entries
    if (n1.r >= 0) {
      b0 = gp(P0.brp)[n1.r];
      len = gp(P0.brp)[n1.r + 1] - b0;
    }
    n2.bounds(P0, crp);
    const bool has = n0.has;
    const int i = n0.i, rs = n0.rs, nnz = n0.re - n0.rs;
    // further entries and parts
    for (int k = 0; k < K; ++k) {
      const Part &Pk = pr->part[k];
      // unsigned: a row may end at entry 2^31 - 1
      uint32_t as = 0, ae = 0;
      if (k == 0) {
        as = (uint32_t)n0.as + G;
        ae = (uint32_t)n0.ae;
      } else if (has) {
        int e0, e1;
        a_row(Pk, i, e0, e1);
        as = (uint32_t)e0;
        ae = (uint32_t)e1;
      }
      while (__any(has && as < ae)) {
        int r = -1, cb = 0, cl = 0;
        VT a = VT(1);
        if (has && as + l < ae) {
          a_entry<VT>(Pk, i, (int)(as + l), r, a);
          cb = gp(Pk.brp)[r];
          cl = gp(Pk.brp)[r + 1] - cb;
        }
        P = min(P, CAP + 1);
        P = sort_chunk<G, E, PAIR, true, VT>(s, gp(Pk.bcol), gp(static_cast<const VT *>(Pk.bval)),
                                       gp(Pk.pair), l, cb, cl, a, P, key);
        if (G == kWave || as < ae) as += G;
      }
    }
    n0 = n1;
    n1 = n2;
    n2.row(list, ri + 3 * stride, count);
    const bool over = P > CAP;  // a changed pattern: the fallback redoes (and flags) the row
    if (over && l == 0) fb_rows[atomicAdd(&hdr->fallback_count, 1)] = i;
    group_sort<G, E>(key, l);
    SPG_GLOBAL int32_t *cb = gpw(ccol) + rs;
    SPG_GLOBAL VT *vb = gpw(cval) + rs;
    const bool live = has && !over;
    const bool plain = live && P == nnz;
    const int p0 = l * E;
    // the column before the lane's first one
    const uint32_t last = G == kWave ? dpp<0x138>(key[E - 1])  // wave_shr 1
                                     : (uint32_t)__shfl_up((int)key[E - 1], 1, G);
    if (plain) {
      int oc[E];
      VT ov[E];
#pragma unroll
      for (int t = 0; t < E; ++t) {
        oc[t] = (int)(key[t] >> IB);
        ov[t] = s.val[key[t] & (uint32_t)(CAP - 1)];
      }
      // as many products as columns by the symbolic count: a column twice
      // means a changed pattern (flagged at the end)
      again = again || (l > 0 && p0 < P && (int)(last >> IB) == oc[0]);
      if (p0 + E <= P) {  // wide stores; the row starts anywhere (4- or 8-byte alignment)
        __builtin_memcpy(cb + p0, oc, sizeof(oc));
        __builtin_memcpy(vb + p0, ov, sizeof(ov));
#pragma unroll
        for (int t = 1; t < E; ++t) again = again || oc[t] == oc[t - 1];
      } else {
#pragma unroll
        for (int t = 0; t < E; ++t) {
          if (p0 + t < P) {
            cb[p0 + t] = oc[t];
            vb[p0 + t] = ov[t];
            again = again || (t > 0 && oc[t] == oc[t > 0 ? t - 1 : 0]);
          }
        }
      }
    }
    if (__any(live && !plain)) {
      // repeated columns
      const bool rep = live && !plain;
      if (rep) {
#pragma unroll
        for (int t = 0; t < E; ++t) s.key[p0 + t] = key[t];
      }
      group_sync<false>();
      bool first[E];
      int firsts = 0;
      uint32_t before = rep && l > 0 ? s.key[p0 - 1] >> IB : 0xffffffffu;
#pragma unroll
      for (int t = 0; t < E; ++t) {
        const uint32_t c = key[t] >> IB;
        first[t] = rep && p0 + t < P && (c != before || p0 + t == 0);
        before = c;
        firsts += first[t] ? 1 : 0;
      }
      const int incl = group_incl_scan<G>(firsts);
      const int total = group_last<G>(incl);
      int d = incl - firsts;
#pragma unroll
      for (int t = 0; t < E; ++t) {
        if (first[t]) {
          const uint32_t c = key[t] >> IB;
          VT sum = s.val[key[t] & (uint32_t)(CAP - 1)];
          for (int u = p0 + t + 1; u < P && s.key[u] >> IB == c; ++u)
            sum += s.val[s.key[u] & (uint32_t)(CAP - 1)];
          if (d < nnz) {  // the symbolic count bounds the row (a changed pattern is flagged)
            cb[d] = (int)c;
            vb[d] = sum;
          }
          ++d;
        }
      }
      if (rep && l == 0 && total != nnz) atomicOr(&hdr->status, kStatInvalid);
    }
    group_sync<false>();
  }
  if (again) atomicOr(&hdr->status, kStatInvalid);
}

// a3 of rows of few products: the columns sorted the same way, distinct ones
// counted between neighbours; no table to clear, no compare-and-swap chains.
// R-MAT blocks, 2^20 rows of up to 128 products: 233 -> 181 us over the four
// bins against the hash set; 4096 rows of 64 products 9.4 -> 4.7; 2^20 rows of
// 16 random entries of one product each 0.32 ms either way (the gathers).
// Up to 256 products the sort's instructions cost more than the hash set's
// waits: 2^20 rows 0.87 ms against 0.59.
template <int G, int E>
__global__ __launch_bounds__(256, 8) void k_sym_sort(const Problem *__restrict__ pr,
                                                     const int32_t *__restrict__ rows,
                                                     const WsHeader *__restrict__ hdr, int bin,
                                                     int32_t *__restrict__ cnt) {
  constexpr int CAP = G * E, R = 256 / G;
  __shared__ SortLds<G, E, float> lds[R];
  if (hdr->status) return;
  const int slot = threadIdx.x / G, l = threadIdx.x % G;
  SortLds<G, E, float> &s = lds[slot];
  // unsigned: a list may hold nearly 2^31 rows
  const uint32_t count = hdr->bin_count[bin];
  const int32_t *list = rows + hdr->bin_start[bin];
  const uint32_t stride = gridDim.x * R;
  const Part &P0 = pr->part[0];
  const SPG_GLOBAL int32_t *bcol0 = gp(P0.bcol);
  const SPG_GLOBAL float *none = nullptr;
  const int K = pr->K;
  uint32_t ri = blockIdx.x * R + slot;
  uint32_t wri = blockIdx.x * R + (int)(threadIdx.x / kWave) * (kWave / G);
  SortNext<G, float> n0, n1, n2;
  n0.row(list, ri, count);
  n0.bounds(P0, nullptr);
  n0.template entry<false>(P0, l);
  int b0 = 0, len = 0;
  if (n0.r >= 0) {
    b0 = gp(P0.brp)[n0.r];
    len = gp(P0.brp)[n0.r + 1] - b0;
  }
  n1.row(list, ri + stride, count);
  n1.bounds(P0, nullptr);
  n2.row(list, ri + 2 * stride, count);
  for (; wri < count; wri += stride, ri += stride) {
    n1.template entry<false>(P0, l);
    uint32_t key[E];
#pragma unroll
    for (int t = 0; t < E; ++t) key[t] = 0xffffffffu;  // past the row: no column
    int P = sort_chunk<G, E, false, false, float>(s, bcol0, none, nullptr, l, b0, len, 1.f, 0, key);
    b0 = len = 0;  // the next row's first entries
    if (n1.r >= 0) {
      b0 = gp(P0.brp)[n1.r];
      len = gp(P0.brp)[n1.r + 1] - b0;
    }
    n2.bounds(P0, nullptr);
    for (int k = 0; k < K; ++k) {  // further entries and parts
      const Part &Pk = pr->part[k];
      uint32_t as = 0, ae = 0;
      if (k == 0) {
        as = (uint32_t)n0.as + G;
        ae = (uint32_t)n0.ae;
      } else if (n0.has) {
        int e0, e1;
        a_row(Pk, n0.i, e0, e1);
        as = (uint32_t)e0;
        ae = (uint32_t)e1;
      }
      while (__any(n0.has && as < ae)) {
        int cb = 0, cl = 0;
        if (n0.has && as + l < ae) {
          const int r = a_entry_row(Pk, n0.i, (int)(as + l));
          cb = gp(Pk.brp)[r];
          cl = gp(Pk.brp)[r + 1] - cb;
        }
        P = min(P, CAP + 1);
        P = sort_chunk<G, E, false, false, float>(s, gp(Pk.bcol), none, nullptr, l, cb, cl, 1.f, P,
                                                  key);
        if (G == kWave || as < ae) as += G;
      }
    }
    group_sort<G, E>(key, l);
    // a lane's first key follows the last one of the lane before it
    const uint32_t prev = (uint32_t)__shfl_up((int)key[E - 1], 1, G);
    int d = key[0] != 0xffffffffu && (l == 0 || key[0] != prev) ? 1 : 0;
#pragma unroll
    for (int t = 1; t < E; ++t) d += key[t] != 0xffffffffu && key[t] != key[t - 1] ? 1 : 0;
    d = group_last<G>(group_incl_scan<G>(d));
    if (n0.has && l == 0) cnt[n0.i] = d;
    n0 = n1;
    n1 = n2;
    n2.row(list, ri + 3 * stride, count);
  }
}

bool sym_sort_ok(int b) { return b >= 1 && b <= 4; }

template <int G, int E>
static void sym_sort(const Problem *dpr, const int32_t *rows, const WsHeader *hdr, int bin,
                     int count, int32_t *cnt, hipStream_t st) {
  constexpr int R = 256 / G;
  int grid = dev_info().cus * 8;
  if (count >= 0) grid = (int)std::min<int64_t>(grid, ((int64_t)count + R - 1) / R);
  hipLaunchKernelGGL((k_sym_sort<G, E>), dim3(std::max(1, grid)), dim3(256), 0, st, dpr, rows, hdr,
                     bin, cnt);
}

void launch_sym_sort(const Problem *dpr, const int32_t *rows, const WsHeader *hdr, int bin,
                     int count, int32_t *cnt, hipStream_t st) {
  switch (bin) {
    case 1: sym_sort<16, 1>(dpr, rows, hdr, bin, count, cnt, st); break;
    case 2: sym_sort<16, 2>(dpr, rows, hdr, bin, count, cnt, st); break;
    case 3: sym_sort<16, 4>(dpr, rows, hdr, bin, count, cnt, st); break;
    default: sym_sort<32, 4>(dpr, rows, hdr, bin, count, cnt, st); break;
  }
}

// Bins served: at most 1024 products a row (beyond, the block bucket kernel
// is faster, see above), and columns that leave the key room for the
// product's number.
bool sort_rows_ok(int b, int64_t n) {
  return b >= 1 && b <= 7 && n <= ((int64_t)1 << (32 - (b + 3)));
}

template <int G, int E, typename VT>
static void num_sort(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int bin, int count,
                     bool pair, const int32_t *crp, int32_t *ccol, VT *cval, int32_t *fb, hipStream_t st) {
  const DevInfo &D = dev_info();
  constexpr int R = 256 / G;
  const int by_waves = sort_waves<G, E>();
  const int by_lds = (int)(D.lds_per_cu / (sizeof(SortLds<G, E, VT>) * R));
  int grid = D.cus * std::max(1, std::min(by_waves, by_lds));
  if (count >= 0) grid = (int)std::min<int64_t>(grid, ((int64_t)count + R - 1) / R);
  if constexpr (sizeof(VT) == 4) {
    if (pair) {
      hipLaunchKernelGGL((k_num_sort<G, E, true, VT>), dim3(std::max(1, grid)), dim3(256), 0, st,
                         dpr, rows, hdr, bin, crp, ccol, cval, fb);
      return;
    }
  }
  hipLaunchKernelGGL((k_num_sort<G, E, false, VT>), dim3(std::max(1, grid)), dim3(256), 0, st, dpr,
                     rows, hdr, bin, crp, ccol, cval, fb);
}

template <typename VT>
static void num_sort_bin(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int bin,
                         int count, bool pair, const int32_t *crp, int32_t *ccol, VT *cval,
                         int32_t *fb, hipStream_t st) {
  switch (bin) {
    case 1: num_sort<16, 1, VT>(dpr, rows, hdr, bin, count, pair, crp, ccol, cval, fb, st); break;
    case 2: num_sort<16, 2, VT>(dpr, rows, hdr, bin, count, pair, crp, ccol, cval, fb, st); break;
    case 3: num_sort<16, 4, VT>(dpr, rows, hdr, bin, count, pair, crp, ccol, cval, fb, st); break;
    case 4: num_sort<32, 4, VT>(dpr, rows, hdr, bin, count, pair, crp, ccol, cval, fb, st); break;
    case 5: num_sort<64, 4, VT>(dpr, rows, hdr, bin, count, pair, crp, ccol, cval, fb, st); break;
    case 6: num_sort<64, 8, VT>(dpr, rows, hdr, bin, count, pair, crp, ccol, cval, fb, st); break;
    default: num_sort<64, 16, VT>(dpr, rows, hdr, bin, count, pair, crp, ccol, cval, fb, st); break;
  }
}

void launch_num_sort(const Problem *dpr, const int32_t *rows, WsHeader *hdr, int bin, int count,
                     bool pair, const int32_t *crp, int32_t *ccol, void *cval, bool f64, int32_t *fb,
                     hipStream_t st) {
  if (f64)
    num_sort_bin<double>(dpr, rows, hdr, bin, count, pair, crp, ccol, static_cast<double *>(cval), fb, st);
  else
    num_sort_bin<float>(dpr, rows, hdr, bin, count, pair, crp, ccol, static_cast<float *>(cval), fb, st);
}

}  // namespace spg
