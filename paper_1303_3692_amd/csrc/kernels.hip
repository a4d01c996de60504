// Device kernels for suffix-array read matching on gfx950 (wave64).
//
// Text layout: 2 bits per base, a=0 c=1 g=2 t=3, base i at bits
// [63-2(i%32)-1, 63-2(i%32)] of word i/32, so comparing two aligned 32-base
// words as unsigned integers compares them lexicographically, and the first
// differing base of two words is clz(x ^ y) / 2.
//
// Search semantics (Section IV, Algorithm 1): with open bounds L = -1 and
// R = n, the LB search moves R to the pivot when the query is not greater
// than the pivot suffix (a prefix match counts as not greater) and ends with
// LB = R; the RB search moves R only when the query is strictly smaller and
// ends with RB = L, i.e. RB + 1 = R.  A suffix that runs out while matching
// is smaller than the query.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "kernels.h"
#include "pivot.h"
#include "radix_sort.h"
#include "split.h"

namespace samatch {
namespace {

constexpr uint32_t kHitExact = 1u;
constexpr uint32_t kHitTooLong = 2u;

// ------------------------------------------------------------------ helpers

__device__ __forceinline__ int min_i(int a, int b) { return a < b ? a : b; }
__device__ __forceinline__ int max_i(int a, int b) { return a > b ? a : b; }

// Probe accounting.  The timed kernels use NoCount (compiles to nothing);
// the instrumented variant counts global probes (one SA entry each), the
// 64-bit text words each probe compares, and probes answered in LDS.
struct NoCount {
    __device__ __forceinline__ void table_probe() {}
    __device__ __forceinline__ void global_probe() {}
    __device__ __forceinline__ void key_probe() {}
    __device__ __forceinline__ void tile_probe() {}
    __device__ __forceinline__ void text_words(uint32_t, uint32_t) {}
    __device__ __forceinline__ void rec_word() {}
    __device__ __forceinline__ void touch(const void *, int) {}
    __device__ __forceinline__ void index_touch(const void *, int) {}
};
// touch(p, bytes): one global access of this lane; the 64-byte segments
// that the wave's active lanes address together are added to `touched`
// (credited to the first active lane), the bytes-touched measure of a
// wave instruction.  index_touch: the same for a load from the index
// (prefix table, row records, suffix array, text), whose addresses are
// scattered; its segments and the load itself are also counted apart
// (`scattered`, `index_loads`), the requests a search makes.
struct Count {
    uint32_t global = 0, words = 0, tile = 0, keys = 0, table = 0, index_loads = 0;
    unsigned long long touched = 0, scattered = 0;
    __device__ __forceinline__ void index_touch(const void *p, int bytes) {
        const unsigned long long before = touched;
        touch(p, bytes);
        scattered += (touched - before) >> 6;
        ++index_loads;
    }
    __device__ __forceinline__ void touch(const void *p, int bytes) {
        const uint64_t a = (uint64_t)(uintptr_t)p;
        const uint64_t s0 = a >> 6;
        const uint64_t active = __ballot(1);
        uint64_t todo = active;
        uint32_t segs = 0;
        while (todo) {
            const int l = __ffsll((unsigned long long)todo) - 1;
            const uint64_t seg = __shfl(s0, l, 64);
            todo &= ~__ballot(s0 == seg);
            ++segs;
        }
        segs += (uint32_t)__popcll(__ballot(((a + (uint64_t)bytes - 1) >> 6) != s0));  // straddling lanes
        if ((threadIdx.x & 63) == __ffsll((unsigned long long)active) - 1) touched += 64ull * segs;
    }
    __device__ __forceinline__ void table_probe() { ++table; }
    __device__ __forceinline__ void global_probe() { ++global; }
    __device__ __forceinline__ void key_probe() { ++global; ++keys; }
    __device__ __forceinline__ void tile_probe() { ++tile; }
    __device__ __forceinline__ void rec_word() { ++keys; }
    // bases [first, end) of the text were compared
    __device__ __forceinline__ void text_words(uint32_t first, uint32_t end) {
        if (end > first) words += ((end - 1) >> 5) - (first >> 5) + 1;
    }
};

// 32 bases of the text starting at base b (bases past the end read as 0; the
// caller never trusts them).  Two neighbouring words joined by a funnel
// shift; the shift by (63 - sh) after a shift by 1 is a shift by 64 - sh
// that also works for sh == 0.
__device__ __forceinline__ uint64_t text_word(const uint64_t *__restrict__ text, uint32_t b) {
    const uint32_t wi = b >> 5;
    const uint32_t sh = (b & 31u) << 1;
    const uint64_t lo = text[wi];
    const uint64_t hi = text[wi + 1];
    return (lo << sh) | ((hi >> 1) >> (63u - sh));
}

template <class Cnt>
__device__ __forceinline__ uint64_t text_word(const uint64_t *__restrict__ text, uint32_t b, Cnt &cnt) {
    cnt.index_touch(text + (b >> 5), 8);
    cnt.index_touch(text + (b >> 5) + 1, 8);
    return text_word(text, b);
}

// Two consecutive 64-bit words with one 16-byte load from an address that
// is only 8-byte aligned (global loads of several dwords need dword
// alignment on this device).
typedef uint64_t u64x2_a8 __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ u64x2_a8 load_u64x2(const uint64_t *p) { return *reinterpret_cast<const u64x2_a8 *>(p); }

// 16 bytes read once: a non-temporal load, so that the caches keep lines
// that are used again (the text, and the row records of repeats) rather than
// prefix-table entries and ASCII reads, which a search touches once (on
// MI355X this took the 250 Mbp / 64M-read batch from 6.47 to 5.93 ms; row
// records loaded like that too: 4.69, through the caches 4.47 ms).
__device__ __forceinline__ uint4 load_stream16(const void *p) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// A 16-byte result, written once and not read again by the kernels.
__device__ __forceinline__ void store_stream16(int4 *p, int4 r) {
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    const i32x4 v = {r.x, r.y, r.z, r.w};
    __builtin_nontemporal_store(v, reinterpret_cast<i32x4 *>(p));
}

// Two consecutive 32-bit words with one 8-byte load, 4-byte aligned.
typedef uint32_t u32x2_a4 __attribute__((ext_vector_type(2), aligned(4)));
__device__ __forceinline__ u32x2_a4 load_u32x2(const uint32_t *p) { return *reinterpret_cast<const u32x2_a4 *>(p); }

// The words of one suffix taken in order: word k (bases p + 32k ..
// p + 32k + 31) joins text words wi + k and wi + k + 1 (wi = p / 32) by a
// funnel shift.  Text words come two per 16-byte load and each is loaded
// once per comparison, so k consecutive suffix words cost 1 + k/2 loads
// (the text carries zero padding words after its end for the loads past it).
struct TextRun {
    const uint64_t *base;  // text + p / 32
    uint32_t sh;           // 2 * (p % 32)
    uint64_t a, b, c;      // text words wi + k, wi + k + 1 and, when `spare`, wi + k + 2
    bool started, spare;

    __device__ __forceinline__ TextRun(const uint64_t *__restrict__ text, uint32_t p)
        : base(text + (p >> 5)), sh((p & 31u) << 1), a(0), b(0), c(0), started(false), spare(false) {}

    // word k of the suffix; successive calls take successive k
    template <class Cnt>
    __device__ __forceinline__ uint64_t word(int k, Cnt &cnt) {
        if (!started) {
            const u64x2_a8 v = load_u64x2(base + k);
            cnt.index_touch(base + k, 16);
            a = v.x;
            b = v.y;
            started = true;
        } else {
            a = b;
            if (spare) {
                b = c;
                spare = false;
            } else {
                const u64x2_a8 v = load_u64x2(base + k + 1);
                cnt.index_touch(base + k + 1, 16);
                b = v.x;
                c = v.y;
                spare = true;
            }
        }
        return (a << sh) | ((b >> 1) >> (63u - sh));
    }
};

// Compare the query P[0..plen) with the suffix at text position p, skipping
// the first 32*k0 bases (known to match).  Returns -1 when P sorts before
// the suffix, 0 when P[0..plen) is a prefix of it, +1 when P sorts after it
// (including when the suffix ends first); lcp gets the exact common-prefix
// length, capped at min(plen, n - p).  The word loop is unrolled over all W
// words and predicated, so the query stays in registers (a run-time index
// into q would move it to scratch memory).
template <int W, class Q, class Cnt>
__device__ __forceinline__ int compare_from(const uint64_t *__restrict__ text, int32_t n,
                                            const Q &q, int plen, int32_t p, int k0,
                                            int &lcp, Cnt &cnt) {
    const int lim = min_i(plen, n - p);
    int res = lim;
    int sign = (lim == plen) ? 0 : 1;
    bool done = false;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        if (!done && k >= k0 && (k << 5) < lim) {
            const uint64_t t = text_word(text, (uint32_t)p + ((uint32_t)k << 5), cnt);
            const uint64_t x = q[k] ^ t;
            if (x) {
                const int mm = (k << 5) + (int)(__clzll((long long)x) >> 1);
                if (mm < lim) {
                    res = mm;
                    sign = q[k] > t ? 1 : -1;
                }
                done = true;
            }
        }
    }
    lcp = res;
    cnt.text_words((uint32_t)p + ((uint32_t)k0 << 5), (uint32_t)p + (uint32_t)min_i(lim, res + 1));
    return sign;
}

// First 16 bytes of a row record: position, length, word 0 (one load).
struct RowHead {
    int32_t pos;
    int32_t len;
    uint64_t key0;
};

__device__ __forceinline__ RowHead row_head(const RowRec *__restrict__ rows, int r) {
    const uint4 v = *reinterpret_cast<const uint4 *>(rows + r);
    RowHead h;
    h.pos = (int32_t)v.x;
    h.len = (int32_t)v.y;
    h.key0 = ((uint64_t)v.w << 32) | v.z;
    return h;
}

// Query words that lie in LDS and are read on demand (the W of the search
// templates otherwise counts words held in registers).
constexpr int kWordsInLds = 0;

// Compares the query P[0..plen) with the suffix at text position p from word k
// on (the words before are known to match); returns and sets what
// compare_from does.  For a query whose words are read as they are needed: a
// loop over two query words at a time, so that it holds few registers and
// stops at the first difference whatever the read's length.  The text words
// of the second of them are loaded together with those of the first (one
// latency for up to 96 bases), and words stay in registers from one turn
// to the next: each text word is loaded once.
template <class Q, class Cnt>
__device__ __forceinline__ int compare_text(const DevIndex &ix, const Q &q, int plen, int32_t p, int k, int &lcp,
                                            Cnt &cnt) {
    const int lim = min_i(plen, ix.n - p);
    const int at_end = (lim == plen) ? 0 : 1;
    lcp = lim;
    if ((k << 5) >= lim) return at_end;
    const uint64_t *tp = ix.text + ((uint32_t)p >> 5) + k;
    const uint32_t sh = ((uint32_t)p & 31u) << 1;
    const uint32_t first = (uint32_t)p + ((uint32_t)k << 5);
    u64x2_a8 a = load_u64x2(tp), b = a;
    cnt.index_touch(tp, 16);
    if ((k << 5) + 32 < lim) {
        b = load_u64x2(tp + 2);
        cnt.index_touch(tp + 2, 16);
    }
    int res = lim, sign = at_end;
    for (;;) {
        uint64_t t = (a.x << sh) | ((a.y >> 1) >> (63u - sh));
        uint64_t w = q[k];
        if (w == t) {
            if ((k << 5) + 32 >= lim) break;
            ++k;
            t = (a.y << sh) | ((b.x >> 1) >> (63u - sh));
            w = q[k];
        }
        if (w != t) {
            const int mm = (k << 5) + (int)(__clzll((long long)(w ^ t)) >> 1);
            if (mm < lim) {
                res = mm;
                sign = w > t ? 1 : -1;
            }
            break;
        }
        if ((k << 5) + 32 >= lim) break;
        ++k;
        tp += 2;
        a = b;
        if ((k << 5) + 32 < lim) {
            b = load_u64x2(tp + 2);
            cnt.index_touch(tp + 2, 16);
        }
    }
    lcp = res;
    cnt.text_words(first, (uint32_t)p + (uint32_t)min_i(lim, res + 1));
    return sign;
}

// compare_row for a query whose words are read from LDS: key0 holds the
// suffix's first key_bases bases (at least 20, at most 32).
template <class Q, class Cnt>
__device__ __forceinline__ int compare_lds(const DevIndex &ix, const Q &q, int plen, int32_t p, uint64_t key0, int h,
                                           int &lcp, Cnt &cnt, int key_bases) {
    const int lim = min_i(plen, ix.n - p);
    const int at_end = (lim == plen) ? 0 : 1;
    lcp = lim;
    int k = h >> 5;
    if (k == 0) {
        const uint64_t q0 = q[0], x = q0 ^ key0;
        const int mm = x ? (int)(__clzll((long long)x) >> 1) : 32;
        if (mm < min_i(key_bases, lim)) {
            lcp = mm;
            return q0 > key0 ? 1 : -1;
        }
        k = key_bases >= 32 ? 1 : 0;
        if (lim <= key_bases) return at_end;
    }
    return compare_text(ix, q, plen, p, k, lcp, cnt);
}

// Probe of one suffix (text position p) whose first key_bases bases (key0,
// the rest of its first word zero) are in hand, with h bases known to
// match: like compare_from, but word 0 comes from key0 and words 1 ..
// kRecWords-1 from the row record (rec; NULL for a node of the LDS tile or
// a prefix-table pivot), loaded only while the words before them tie; later
// words come from the text, and so does word 0 when key0 holds fewer than
// 32 bases, ties on them, and the comparison reaches past them.
template <int W, class Q, class Cnt>
__device__ __forceinline__ int compare_row(const DevIndex &ix, const Q &q, int plen,
                                           const RowRec *__restrict__ rec, int32_t p, uint64_t key0, int h,
                                           int &lcp, Cnt &cnt, int key_bases = 32) {
    if constexpr (W == kWordsInLds) return compare_lds(ix, q, plen, p, key0, h, lcp, cnt, key_bases);
    const int lim = min_i(plen, ix.n - p);
    const int k0 = h >> 5;
    int res = lim;
    int sign = (lim == plen) ? 0 : 1;
    bool done = false;
    uint32_t text_first = 0, text_end = 0;
    TextRun run(ix.text, (uint32_t)p);
#pragma unroll
    for (int k = 0; k < W; ++k) {
        if (!done && k >= k0 && (k << 5) < lim) {
            uint64_t t;
            if (k == 0 && (key_bases >= 32 || lim <= key_bases ||
                           ((q[0] ^ key0) & (~0ull << (64 - 2 * key_bases))) != 0)) {
                t = key0;
            } else if (k > 0 && rec != nullptr && k < kRecWords) {
                t = reinterpret_cast<const uint64_t *>(rec)[1 + k];  // word k of the record
                cnt.rec_word();
                cnt.index_touch(reinterpret_cast<const uint64_t *>(rec) + 1 + k, 8);
            } else {
                t = run.word(k, cnt);
                if (text_end == 0) text_first = (uint32_t)p + ((uint32_t)k << 5);
                text_end = (uint32_t)p + (uint32_t)min_i(lim, (k << 5) + 32);
            }
            const uint64_t x = q[k] ^ t;
            if (x) {
                const int mm = (k << 5) + (int)(__clzll((long long)x) >> 1);
                if (mm < lim) {
                    res = mm;
                    sign = q[k] > t ? 1 : -1;
                }
                done = true;
                if (text_end) text_end = (uint32_t)p + (uint32_t)min_i(lim, mm + 1);
            }
        }
    }
    lcp = res;
    cnt.text_words(text_first, text_end);
    return sign;
}

// Binary search over rows (L, R] with known common-prefix lengths at the
// bounds (lcpL, lcpR, 0 for the open ends).  Every row strictly between
// them shares min(lcpL, lcpR) leading bases with the query, so each probe
// starts comparing at that word.  UPPER = false: first row whose suffix is
// not below P[0..plen) (LB); UPPER = true: first row strictly above every
// extension of P[0..plen) (RB + 1).
template <int W, bool UPPER, class Q, class Cnt>
__device__ __forceinline__ int bounded_search(const DevIndex &ix, const Q &q, int plen, int L, int R,
                              int lcpL, int lcpR, Cnt &cnt) {
    while (R > L + 1) {
        const int piv = midpoint(L, R);
        const RowHead row = row_head(ix.rows, piv);
        cnt.index_touch(ix.rows + piv, 16);
        int lcp;
        cnt.key_probe();
        const int sign = compare_row<W>(ix, q, plen, ix.rows + piv, row.pos, row.key0, min_i(lcpL, lcpR), lcp, cnt);
        const bool go_left = UPPER ? (sign < 0) : (sign <= 0);
        if (go_left) { R = piv; lcpR = lcp; }
        else { L = piv; lcpL = lcp; }
    }
    return R;
}

// State at the end of the LB search: adjacent rows L, R = L + 1 around the
// insertion point of P[0..plen), their common-prefix lengths with P, and for
// each side the last bound before its common-prefix length reached its final
// value (Llt / Rlt) with that bound's length.  Common-prefix lengths only
// grow towards the insertion point, so every row at or beyond Llt (Rlt) on
// that side shares fewer than lcpL (lcpR) bases with P.
struct LbState {
    int L, R, lcpL, lcpR, Llt, lcpLlt, Rlt, lcpRlt;
};

__device__ __forceinline__ void lb_update(LbState &st, int sign, int piv, int lcp) {
    if (sign <= 0) {
        if (lcp > st.lcpR) { st.Rlt = st.R; st.lcpRlt = st.lcpR; }
        st.R = piv; st.lcpR = lcp;
    } else {
        if (lcp > st.lcpL) { st.Llt = st.L; st.lcpLlt = st.lcpL; }
        st.L = piv; st.lcpL = lcp;
    }
}

// LB search of P[0..plen) from the bounds in st to its end, on row records.
template <int W, class Q, class Cnt>
__device__ __forceinline__ void lb_rows(const DevIndex &ix, const Q &q, int plen, LbState &st, Cnt &cnt) {
    while (st.R > st.L + 1) {
        const int piv = midpoint(st.L, st.R);
        const RowHead row = row_head(ix.rows, piv);
        cnt.index_touch(ix.rows + piv, 16);
        int lcp;
        cnt.key_probe();
        const int sign =
            compare_row<W>(ix, q, plen, ix.rows + piv, row.pos, row.key0, min_i(st.lcpL, st.lcpR), lcp, cnt);
        lb_update(st, sign, piv, lcp);
    }
}

// Full LB search of P[0..plen) (lb_tile: its part in the tile, then the rest
// on row records).  The first `levels` probes of every search
// from (-1, n) visit nodes of one fixed implicit binary tree; their pivot
// suffixes (first 32 bases and text position) sit in LDS.  A probe that
// ties on all 32 staged bases continues in global memory at word 1.
template <int W, class Q, class Cnt>
__device__ __forceinline__ void lb_tile(const DevIndex &ix, const uint64_t *s_key, const int32_t *s_sa, int levels,
                          const Q &q, int plen, LbState &st, Cnt &cnt) {
    st.L = -1; st.R = ix.n; st.lcpL = 0; st.lcpR = 0;
    st.Llt = -1; st.lcpLlt = 0; st.Rlt = ix.n; st.lcpRlt = 0;
    int node = 0;
    for (int d = 0; d < levels && st.R > st.L + 1; ++d) {
        const uint64_t key = s_key[node];
        const int32_t p = s_sa[node];
        int lcp;
        cnt.tile_probe();
        const int sign = compare_row<W>(ix, q, plen, nullptr, p, key, min_i(st.lcpL, st.lcpR), lcp, cnt);
        const int piv = midpoint(st.L, st.R);
        lb_update(st, sign, piv, lcp);
        node = 2 * node + (sign <= 0 ? 1 : 2);
    }
}

template <int W, class Q, class Cnt>
__device__ __forceinline__ void lb_search(const DevIndex &ix, const uint64_t *s_key, const int32_t *s_sa, int levels,
                                          const Q &q, int plen, LbState &st, Cnt &cnt) {
    lb_tile<W>(ix, s_key, s_sa, levels, q, plen, st, cnt);
    lb_rows<W>(ix, q, plen, st, cnt);
}

// ---- prefix table
// The table T[v] (v a k-base string) is the first SA row whose suffix is not
// below v.  For a query P with at least k leading ACGT bases and first k
// bases v, every row before T[v] is below P and every row of a suffix that
// does not start with v after them is above it, so the LB search of P runs
// inside the bracket of rows that start with v (see PrefixEntry).

// The entry of the read's first K bases (one 16-byte load).  A table of up
// to kCachedBases bases (1 GiB) is small enough for a batch to come back to its
// lines while caches hold them; a larger one is read past the caches, which
// leaves them to rows and text (MI355X, 4M reads of 100 bases on 1 Mbp, k = 12:
// 191 us cached, 226 not; on 4 Mbp, k = 13: 217 and 232; on 16 Mbp, k = 14: 246
// and 241).
constexpr int kCachedBases = 13;

template <class Cnt>
__device__ __forceinline__ PrefixEntry table_entry(const DevIndex &ix, uint32_t v, Cnt &cnt) {
    const uint4 e = ix.ptab_k <= kCachedBases ? *reinterpret_cast<const uint4 *>(ix.ptab + v)
                                              : load_stream16(ix.ptab + v);
    cnt.index_touch(ix.ptab + v, 16);
    cnt.table_probe();
    return PrefixEntry{e.x, e.y, (int32_t)e.z, e.w};
}

// LB search of P[0..plen) inside the bracket of an entry that has one.
// Rows inside the bracket share k bases with P, so when the search moves a
// bound inside, the other bound's common-prefix length (below k) never
// decides anything and starts as 0.  The first probe takes its pivot
// suffix's position and first k + 16 bases from the entry, with no load of
// its own.
__device__ __forceinline__ void open_bracket(const DevIndex &ix, int row, int size, LbState &st) {
    st.L = row - 1; st.R = row + size; st.lcpL = 0; st.lcpR = 0;
    st.Llt = -1; st.lcpLlt = 0; st.Rlt = ix.n; st.lcpRlt = 0;
}

template <int W, class Q, class Cnt>
__device__ __forceinline__ void lb_search_table(const DevIndex &ix, const PrefixEntry &ent, const Q &q, int plen,
                                                LbState &st, Cnt &cnt) {
    const int K = ix.ptab_k;
    open_bracket(ix, (int)ent.row, (int)ent.size, st);
    const int piv = midpoint(st.L, st.R);
    const uint64_t key = (q[0] & ~(~0ull >> (2 * K))) | ((uint64_t)ent.next << (32 - 2 * K));
    int lcp;
    cnt.global_probe();  // its position and bases came with the entry, not from a record
    const int sign = compare_row<W>(ix, q, plen, nullptr, ent.pos, key, 0, lcp, cnt, K + 16);
    lb_update(st, sign, piv, lcp);
    lb_rows<W>(ix, q, plen, st, cnt);
}

// The read's result from the final state of the LB search of its ACGT
// prefix P[0..mv): exact reads finish with an RB search confined to (LB,
// Rlt]; other reads take the longest matched prefix l = max(lcpL, lcpR) from
// the two rows around the insertion point and find the interval of P[0..l)
// inside the bounds the LB search already bracketed.
template <int W, class Q, class Cnt>
__device__ __forceinline__ int4 finish_read(const DevIndex &ix, const Q &q, int m, int mv, const LbState &st,
                                            Cnt &cnt) {
    if (mv == m && st.lcpR == m) {
        const int hi = bounded_search<W, true>(ix, q, m, st.R, st.Rlt, m, st.lcpRlt, cnt);
        return make_int4(st.R, hi, m, (int)kHitExact);
    }
    // (after a search inside a table bracket l >= k: one of the final
    // bounds is a probed row of the bracket, which shares the k bases)
    const int l = max_i(st.lcpL, st.lcpR);
    if (l == 0) return make_int4(0, ix.n, 0, 0);
    const int lo = (st.lcpL == l) ? bounded_search<W, false>(ix, q, l, st.Llt, st.L, st.lcpLlt, l, cnt) : st.R;
    const int hi = (st.lcpR == l) ? bounded_search<W, true>(ix, q, l, st.R, st.Rlt, l, st.lcpRlt, cnt) : st.R;
    return make_int4(lo, hi, l, 0);
}

// One read: LB search of its ACGT prefix from its table entry or from the
// root, then finish_read.  The empty prefix (an empty read, or one that
// starts with a non-base) matches every suffix.
template <int W, class Q, class Cnt>
__device__ __forceinline__ int4 match_read(const DevIndex &ix, const uint64_t *s_key, const int32_t *s_sa, int levels,
                           bool use_table, const Q &q, int m, int mv, Cnt &cnt) {
    if (mv == 0) return make_int4(0, ix.n, 0, m == 0 ? (int)kHitExact : 0);
    LbState st;
    if (use_table && ix.ptab_k > 0 && mv >= ix.ptab_k) {
        const PrefixEntry ent = table_entry(ix, (uint32_t)(q[0] >> (64 - 2 * ix.ptab_k)), cnt);
        if (ent.size & kPtabAnswer) return make_int4(ent.pos, (int)ent.next, (int)(ent.size & ~kPtabAnswer), 0);
        lb_search_table<W>(ix, ent, q, mv, st, cnt);
    } else {
        lb_search<W>(ix, s_key, s_sa, levels, q, mv, st, cnt);
    }
    return finish_read<W>(ix, q, m, mv, st, cnt);
}

template <int W>
__device__ __forceinline__ void load_query(const uint64_t *__restrict__ src, int nw, uint64_t (&q)[W]) {
#pragma unroll
    for (int k = 0; k < W; ++k) q[k] = k < nw ? src[k] : 0ull;
}

__device__ __forceinline__ uint64_t wave_ballot(bool p) { return __ballot(p); }

// ------------------------------------------------------------------ row keys

// One record per SA row: the suffix's text position and length and its
// first 32 * kRecWords bases (zero past the text end), so that a probe
// fetches position and bases from one line.
__global__ void build_rows_kernel(const uint64_t *__restrict__ text, const int32_t *__restrict__ sa, int32_t n,
                                  RowRec *__restrict__ rows) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const int32_t p = sa[r];
    RowRec rec;
    rec.pos = p;
    rec.len = n - p;
#pragma unroll
    for (int k = 0; k < kRecWords; ++k) rec.key[k] = text_word(text, (uint32_t)p + ((uint32_t)k << 5));
    rows[r] = rec;
}

// ------------------------------------------------------------------ prefix table

// Order key of a row for a k-base table: 2 * (first k bases, zero-padded)
// + 1 for a suffix of at least k bases, without the +1 for a shorter one (it
// sorts before every k-base string it is a proper prefix of).  It does not
// decrease along the suffix array.
__device__ __forceinline__ uint64_t row_order_key(const RowHead &row, int k) {
    return 2 * (row.key0 >> (64 - 2 * k)) + (row.len >= k ? 1u : 0u);
}

// First row whose order key reaches `target`, found by the whole wave, 64 rows
// at a time.
__device__ __forceinline__ uint32_t first_row_from(const DevIndex &ix, int k, uint64_t target, int lane) {
    uint32_t lo = 0, hi = (uint32_t)ix.n;
    while (lo < hi) {
        const uint32_t piv = wave_probe_row(lo, hi, lane);
        const bool reached = piv < hi && row_order_key(row_head(ix.rows, (int)piv), k) >= target;
        const uint64_t r = wave_ballot(reached);
        const int probes = (int)(hi - lo < 64u ? hi - lo : 64u), to = r ? (int)__builtin_ctzll(r) : probes;
        const uint32_t above = __shfl(piv, min_i(to, 63), 64), below = __shfl(piv, max_i(to - 1, 0), 64);
        if (to < probes) hi = above;
        if (to > 0) lo = below + 1;
    }
    return lo;
}

// The prefix table, 4^bases entries (those of one string of k - bases bases)
// per workgroup.  Their rows are neighbours: the workgroup
// finds the first and the last of them, marks in LDS where each string's
// rows start and end (by walking them, or by a search per string where they
// are many), and takes for every string the first row not below it (T) by a
// running minimum from the end.  A string v with rows gets its
// bracket and the suffix at its first pivot.  For one without, the longest
// prefix of v that occurs is the longest that has rows, found by comparing T
// at the ends of ever larger aligned groups of entries, and T there bounds
// its rows.  Two cases search from the root instead: strings of a workgroup
// without any row (all have one answer), and those of a workgroup near
// whose rows a suffix shorter than k sorts (its rows are not aligned to the
// groups; at most k - 1 suffixes are that short).  Bound by the table's
// bytes: 16 Mbp (268 M entries, 4.3 GB) took 16.7 ms as a binary search per
// entry for T and a second pass from the root for the strings without rows,
// 1.3 ms now.
constexpr int kTabThreads = 512;  // at most: a workgroup has no more threads than entries
constexpr int kTabBases = 6;
constexpr int kTabSpan = 1 << (2 * kTabBases);
constexpr int kTabRows = 4;  // entries per thread whose pivots' loads are in flight together
// Rows per string from which a workgroup searches its strings' first rows
// instead of walking all of its rows, which the workgroup with the most of them
// (short strings, a text of one letter) does while the others have finished:
// 16 Mbp, strings of 4 bases (62,500 rows each) 40.6 ms by the walk, 0.02
// searched; 16 M times the same letter, strings of 14 bases 24.6 and 1.5 ms.
// Below it the walk reads fewer lines: it takes each row once, a search
// the logarithm of them.
constexpr uint32_t kTabWalk = 16;

__global__ __launch_bounds__(kTabThreads) void build_prefix_table_kernel(DevIndex ix, int k, int bases,
                                                                         PrefixEntry *__restrict__ tab) {
    __shared__ uint32_t first[kTabSpan + 1];  // a string's first row, then T
    __shared__ uint32_t last[kTabSpan];       // the row after a string's last one, 0 without rows
    __shared__ uint32_t wave_min[kTabThreads / 64];
    __shared__ uint32_t bound[2];
    __shared__ int near_short;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, threads = blockDim.x;
    const int span = 1 << (2 * bases);  // a multiple of the threads, which are full waves
    const uint64_t v0 = (uint64_t)blockIdx.x << (2 * bases);
    if (t == 0) near_short = 0;
    if (wave < 2) {
        const uint32_t r = first_row_from(ix, k, 2 * (v0 + (wave ? (uint64_t)span : 0u)) + 1, lane);
        if (lane == 0) bound[wave] = r;
    }
    __syncthreads();
    const uint32_t r0 = bound[0], r1 = bound[1];  // at most 2^31 - 1; a stride past that needs the last bit
    for (int i = t; i < span; i += threads) {
        first[i] = r1;
        last[i] = 0;
    }
    if (t == 0) first[span] = r1;
    __syncthreads();
    auto order_key = [&](uint32_t r) { return row_order_key(row_head(ix.rows, (int)r), k); };
    if (r1 - r0 <= kTabWalk * (uint32_t)span) {
        for (uint32_t r = r0 + t; r < r1; r += threads) {
            const uint64_t key = order_key(r);
            const int i = (int)((key >> 1) - v0);
            if (key & 1) {
                if (r == r0 || order_key(r - 1) != key) atomicMin(&first[i], r);
                if (r + 1 == r1 || order_key(r + 1) != key) last[i] = r + 1;
            } else {  // below its padded string, above the one before
                atomicMin(&first[i - 1], r);
                near_short = 1;
            }
        }
    } else {
        for (int i0 = t; i0 < span; i0 += kTabRows * threads) {
            uint32_t lo[kTabRows], hi[kTabRows];
#pragma unroll
            for (int u = 0; u < kTabRows; ++u) {
                lo[u] = r0;
                hi[u] = i0 + u * threads < span ? r1 : r0;
            }
            for (uint32_t rows = r1 - r0; rows > 0; rows >>= 1) {
#pragma unroll
                for (int u = 0; u < kTabRows; ++u) {
                    if (lo[u] == hi[u]) continue;
                    const uint32_t mid = lo[u] + (hi[u] - lo[u]) / 2;
                    if (order_key(mid) > 2 * (v0 + (uint64_t)(i0 + u * threads))) hi[u] = mid;
                    else lo[u] = mid + 1;
                }
            }
#pragma unroll
            for (int u = 0; u < kTabRows; ++u)
                if (i0 + u * threads < span) first[i0 + u * threads] = lo[u];
        }
        __syncthreads();
        for (int i = t; i < span; i += threads) {
            uint32_t end = first[i + 1];
            while (end > first[i] && order_key(end - 1) != 2 * (v0 + (uint64_t)i) + 1) {  // below the next padded string
                --end;
                near_short = 1;
            }
            if (end > first[i]) last[i] = end;
        }
    }
    if (t < k && (uint32_t)t < r0 && row_head(ix.rows, (int)r0 - 1 - t).len < k) near_short = 1;
    __syncthreads();
    uint32_t carry = r1;
    for (int base = span - threads; base >= 0; base -= threads) {
        uint32_t x = first[base + t];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_down(x, o, 64);
            if (lane + o < 64) x = x < y ? x : y;
        }
        if (lane == 0) wave_min[wave] = x;
        __syncthreads();
        uint32_t later = carry;  // the least of the waves after this one and of the rounds before
        for (int u = 0; u < threads / 64; ++u) {
            const uint32_t y = wave_min[u];
            if (u > wave) later = later < y ? later : y;
            carry = carry < y ? carry : y;
        }
        first[base + t] = x < later ? x : later;
        __syncthreads();
    }
    const bool none = r0 == r1, search = near_short != 0;
    int4 ans = make_int4(0, 0, 0, 0);
    if (search || none) {
        for (int i = t; i < (search ? span : threads); i += threads) {
            if (last[i]) continue;
            const uint64_t q[1] = {(v0 + (uint64_t)i) << (64 - 2 * k)};
            NoCount cnt;
            ans = match_read<1>(ix, nullptr, nullptr, 0, false, q, k, k, cnt);
            if (search)
                store_stream16(reinterpret_cast<int4 *>(tab + v0) + i,
                               make_int4((int)first[i], (int)(kPtabAnswer | (uint32_t)ans.z), ans.x, ans.y));
        }
    }
    for (int i0 = t; i0 < span; i0 += kTabRows * threads) {
        RowHead h[kTabRows];
#pragma unroll
        for (int u = 0; u < kTabRows; ++u) {
            const int i = i0 + u * threads;
            if (i < span && last[i]) h[u] = row_head(ix.rows, midpoint((int)first[i] - 1, (int)last[i]));
        }
#pragma unroll
        for (int u = 0; u < kTabRows; ++u) {
            const int i = i0 + u * threads;
            if (i >= span) break;
            const uint32_t row = first[i], end = last[i];
            int4 e = make_int4((int)row, (int)(end - row), h[u].pos, (int)(uint32_t)(h[u].key0 >> (32 - 2 * k)));
            if (!end) {
                if (search) continue;  // written above
                if (!none) {
                    int g = 0;
                    uint32_t lo, hi;
                    do {
                        ++g;
                        const int x = i & ~((1 << (2 * g)) - 1);
                        lo = first[x];
                        hi = first[x + (1 << (2 * g))];
                    } while (lo == hi);
                    ans = make_int4((int)lo, (int)hi, k - g, 0);
                }
                e = make_int4((int)row, (int)(kPtabAnswer | (uint32_t)ans.z), ans.x, ans.y);
            }
            store_stream16(reinterpret_cast<int4 *>(tab + v0) + i, e);
        }
    }
    if (blockIdx.x == gridDim.x - 1 && t == 0)  // T[4^k] = n closes the table; it is never looked up
        store_stream16(reinterpret_cast<int4 *>(tab + v0) + span, make_int4(ix.n, 0, 0, 0));
}

// ------------------------------------------------------------------ tile

__global__ void build_tile_kernel(const uint64_t *__restrict__ text, const int32_t *__restrict__ sa,
                                  int32_t n, int levels, uint64_t *key, int32_t *tsa) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int nodes = (1 << levels) - 1;
    if (j >= nodes) return;
    // node j is reached by the bits of j+1 after its leading one: 0 = the
    // query was not above the pivot (R = pivot), 1 = it was (L = pivot)
    const int depth = 31 - __clz(j + 1);
    const int path = (j + 1) - (1 << depth);
    int L = -1, R = n;
    bool live = true;
    for (int i = depth - 1; i >= 0; --i) {
        if (R <= L + 1) { live = false; break; }
        const int piv = midpoint(L, R);
        if ((path >> i) & 1) L = piv; else R = piv;
    }
    if (!live || R <= L + 1) {  // no search reaches this node
        key[j] = 0;
        tsa[j] = 0;
        return;
    }
    const int32_t p = sa[midpoint(L, R)];
    key[j] = text_word(text, (uint32_t)p);
    tsa[j] = p;
}

// ------------------------------------------------------------------ per-read record

// The pack kernel's 8-byte record of a read: its length m (-1: not
// searched), then one word holding the length of its ACGT prefix plus one
// (0: a long read, for the long-read kernel) in the low 16 bits and the
// offset of its packed words in its workgroup's region of qw in the high 16.
struct ReadLen {
    int m, mv, wo;
};

__device__ __forceinline__ int2 encode_len(int m, int mv, int wo) {
    return make_int2(m, (int)(((uint32_t)wo << 16) | (uint32_t)(mv + 1)));
}

__device__ __forceinline__ ReadLen decode_len(int2 v) {
    ReadLen r;
    r.m = v.x;
    r.mv = (int)((uint32_t)v.y & 0xFFFFu) - 1;
    r.wo = (int)((uint32_t)v.y >> 16);
    return r;
}

// ------------------------------------------------------------------ pack

// Per-byte flags (0x80 in each byte) of the four bytes of x that are not
// one of a, c, g, t after forcing lower case: a byte is nonzero after
// xor-ing with a letter unless it is that letter.
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t v) {
    return (((v & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v) & 0x80808080u;
}
__device__ __forceinline__ uint32_t invalid_bytes(uint32_t dw) {
    const uint32_t lc = dw | 0x20202020u;
    return nonzero_bytes(lc ^ 0x61616161u) & nonzero_bytes(lc ^ 0x63636363u) & nonzero_bytes(lc ^ 0x67676767u) &
           nonzero_bytes(lc ^ 0x74747474u);
}

// Four bases (little-endian bytes of dw, the first base in the low byte) to
// 8 bits, first base in the top two bits; `keep` masks the bytes that
// belong to the read.  a->0 c->1 g->2 t->3 for either case, anything else
// becomes 0 and is reported in *bad (0x80 per byte).
__device__ __forceinline__ uint32_t pack4(uint32_t dw, uint32_t keep, uint32_t &bad) {
    bad = invalid_bytes(dw) & keep;
    const uint32_t zero = (bad >> 7) * 0xFFu;  // 0xFF in each flagged byte
    const uint32_t codes = ((dw >> 1) ^ (dw >> 2)) & 0x03030303u & keep & ~zero;
    return ((codes & 3u) << 6) | ((codes >> 4) & 0x30u) | ((codes >> 14) & 0x0Cu) | ((codes >> 24) & 3u);
}

// pack4 with one byte permute instead of four letter tests: the code of a
// byte is ((c >> 1) ^ (c >> 2)) & 3 (a/A -> 0, c/C -> 1, g/G -> 2, t/T ->
// 3), and a byte is a base exactly when, with bit 5 cleared, it equals
// "ACGT"[code] (looked up with v_perm).  Same results as pack4.
__device__ __forceinline__ uint32_t pack4_fast(uint32_t dw, uint32_t keep, uint32_t &bad) {
    uint32_t codes = ((dw >> 1) ^ (dw >> 2)) & 0x03030303u;
    const uint32_t expect = __builtin_amdgcn_perm(0u, 0x54474341u, codes);  // "ACGT"[code] per byte
    bad = nonzero_bytes((dw & 0xDFDFDFDFu) ^ expect) & keep;
    codes &= keep & ~((bad >> 7) * 0xFFu);
    return ((codes & 3u) << 6) | ((codes >> 4) & 0x30u) | ((codes >> 14) & 0x0Cu) | (codes >> 24);
}

// Pack one read from global memory, fetching aligned dwords; an aligned
// dword that holds at least one byte of the read never crosses a page, so
// no fetch can fault.
__device__ __forceinline__ void pack_from_global(const uint8_t *__restrict__ reads, int64_t a, int m,
                                                 uint64_t (&dst)[kWMax + 1], int &mv, uint64_t &w0) {
    mv = m;
    uint64_t word = 0;
    int k = 0;
#pragma unroll
    for (int t = 0; t < kWMax; ++t) dst[t] = 0;
    const uintptr_t start = (uintptr_t)(reads + a);
    const uintptr_t stop = start + (uintptr_t)m;
    for (uintptr_t addr = start & ~(uintptr_t)3; addr < stop; addr += 4) {
        const uint32_t dw = *reinterpret_cast<const uint32_t *>(addr);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uintptr_t at = addr + t;
            if (at < start || at >= stop) continue;
            const int idx = (int)(at - start);
            const uint32_t c = (dw >> (8 * t)) & 0xFFu;
            const uint32_t lc = c | 0x20u;
            const bool ok = lc == 'a' || lc == 'c' || lc == 'g' || lc == 't';
            const uint32_t code = ((c >> 1) ^ (c >> 2)) & 3u;
            if (!ok && idx < mv) mv = idx;
            word |= (uint64_t)(ok ? code : 0u) << (62 - 2 * (idx & 31));
            if ((idx & 31) == 31) {
#pragma unroll
                for (int t = 0; t < kWMax; ++t) dst[t] = (t == k) ? word : dst[t];
                ++k;
                word = 0;
            }
        }
    }
    if ((m & 31) != 0 || m == 0) {
#pragma unroll
        for (int t = 0; t < kWMax; ++t) dst[t] = (t == k) ? word : dst[t];
    }
    w0 = dst[0];
}

// Packing: each workgroup converts the bytes of its 256 consecutive reads
// with coalesced, aligned 16-byte loads into a stream of 2-bit codes in
// LDS (16 bases per word, 12 KB for 48 KB of ASCII) and a flag per byte
// that is not a base; each thread then takes its read's words out of the
// stream with funnel shifts and finds its first non-base from the flags.
// Reads whose bytes are not in the converted span (offsets that are not
// contiguous, or a span larger than 48 KB) take the global path.  The
// packed words go back through LDS so that the workgroup's run of words is
// written with coalesced 16-byte stores.  Read i is reads[offs[i] ..
// offs[i+1]), or reads[offs[i] .. ends[i]) when an end array is given
// (reads scattered over a larger buffer; always the global path).
constexpr int kPackBlock = 256;
constexpr int kPackChunks = 3072;  // 16-byte chunks of ASCII a workgroup converts through LDS (48 KB)
static_assert((kPackChunks + 4) * 6 <= (kPackBlock * kWMax + 8) * 8, "code stream and flags fit the buffer");

// The 0x80 flags of pack4_fast's four bytes as four bits, byte 0 lowest.
__device__ __forceinline__ uint32_t bad_nibble(uint32_t bad) {
    return ((bad >> 7) & 1u) | ((bad >> 14) & 2u) | ((bad >> 21) & 4u) | ((bad >> 28) & 8u);
}

// 16 bytes of ASCII (four little-endian dwords, the first byte lowest) to
// 16 two-bit codes, the first base in the top bits; `bad` becomes nonzero
// when a byte is not a base (its code is then of no meaning).  Bits 1 and 2
// of a base's letter, in either case, count a, c, t, g as 0..3: a dot
// product with the place values of four codes gathers them into a byte, a
// byte permute looks up the letters they stand for to test the bytes, and
// t and g are put in order at the end on all sixteen codes at once.  About
// 30 instructions for 16 bases (shifts, masks and a bit reversal took 60).
__device__ __forceinline__ uint32_t convert16(const uint4 &v, uint32_t &bad) {
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    uint32_t w = 0, diff = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t r = (d[i] >> 1) & 0x03030303u;
        diff |= (d[i] ^ __builtin_amdgcn_perm(0u, 0x47544341u, r)) & 0xDFDFDFDFu;
        w = __builtin_amdgcn_udot4(r, 0x01041040u, w << 8, false);
    }
    bad = diff;
    return w ^ ((w >> 1) & 0x55555555u);
}

// convert16 into codes[c], with a flag bit per byte that is not a base in
// badm[c] (bit i for byte i) and the code of such a byte 0.  Returns
// whether a byte was not a base.
__device__ __forceinline__ bool convert_piece(const uint4 &v, uint32_t *codes, uint16_t *badm, int c) {
    uint32_t any;
    const uint32_t w = convert16(v, any);
    if (any == 0) {
        codes[c] = w;
        badm[c] = 0;
        return false;
    }
    uint32_t bad, code, bits;
    code = pack4_fast(v.x, 0xFFFFFFFFu, bad);
    bits = bad_nibble(bad);
    code = (code << 8) | pack4_fast(v.y, 0xFFFFFFFFu, bad);
    bits |= bad_nibble(bad) << 4;
    code = (code << 8) | pack4_fast(v.z, 0xFFFFFFFFu, bad);
    bits |= bad_nibble(bad) << 8;
    code = (code << 8) | pack4_fast(v.w, 0xFFFFFFFFu, bad);
    bits |= bad_nibble(bad) << 12;
    codes[c] = code;
    badm[c] = (uint16_t)bits;
    return true;
}

// The reference text, packed: one word (32 bases, two 16-byte loads) per
// thread.  Bound by the text's bytes over the bus before it: the host checked
// and packed 16 Mbp in 95 of the 122 ms that the device build took, one byte
// at a time (with this and the steps after it the build takes 4.7).
__global__ __launch_bounds__(256) void pack_text_kernel(const uint8_t *__restrict__ ascii, int64_t n,
                                                        uint64_t *__restrict__ text, int64_t words,
                                                        unsigned long long *__restrict__ first_bad) {
    const int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (w >= words) return;
    uint64_t out = 0;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int64_t p = 32 * w + 16 * half;
        const int64_t left = n - p;
        if (left <= 0) break;
        const uint4 v = load_stream16(ascii + p);
        uint32_t bad;
        uint32_t code = convert16(v, bad);
        if (bad || left < 16) {  // a byte that is not a base, or bytes past the end
            const uint32_t d[4] = {v.x, v.y, v.z, v.w};
            const int take = left < 16 ? (int)left : 16;
            for (int i = take - 1; i >= 0; --i) {
                const uint32_t c = (d[i >> 2] >> (8 * (i & 3))) & 0xDFu;
                if (c != 'A' && c != 'C' && c != 'G' && c != 'T') atomicMin(first_bad, (unsigned long long)(p + i));
            }
            if (take < 16) code &= ~(~0u >> (2 * take));
        }
        out |= (uint64_t)code << (half ? 0 : 32);
    }
    text[w] = out;
}

__global__ __launch_bounds__(kPackBlock) void pack_kernel(const uint8_t *__restrict__ reads,
                                                          const int64_t *__restrict__ offs,
                                                          const int64_t *__restrict__ ends, int64_t nreads,
                                                          BatchBuffers b, BucketTable bt) {
    // the span's bases as a code stream (16 per word, first in the top bits)
    // and a flag per byte that is not a base; later the packed words
    __shared__ uint64_t lds_buf[kPackBlock * kWMax + 8];
    uint32_t *codes = reinterpret_cast<uint32_t *>(lds_buf);
    uint16_t *badm = reinterpret_cast<uint16_t *>(codes + kPackChunks + 4);
    const int64_t r0 = (int64_t)blockIdx.x * kPackBlock;
    const int64_t r1 = r0 + kPackBlock < nreads ? r0 + kPackBlock : nreads;
    const int64_t i = r0 + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x < kStatWords) b.stats[threadIdx.x] = 0ull;
    // with an end array, the workgroup's reads still form one span when each
    // ends where the next starts (the usual case for a request's reads)
    bool contiguous = true;
    if (ends) contiguous = __syncthreads_and(i + 1 >= r1 || ends[i] == offs[i + 1]) != 0;
    const int64_t span0 = offs[r0];
    const int64_t span1 = ends ? (contiguous ? ends[r1 - 1] : span0) : offs[r1];
    const uintptr_t A0 = (uintptr_t)(reads + span0) & ~(uintptr_t)15;
    const uintptr_t A1 = ((uintptr_t)(reads + span1) + 15) & ~(uintptr_t)15;
    const bool staged = contiguous && span1 > span0 && A1 - A0 <= (uintptr_t)kPackChunks * 16u;
    if (staged) {
        // every aligned 16-byte chunk here holds a byte of [span0, span1):
        // coalesced loads, converted on the way into LDS
        const int nvec = (int)((A1 - A0) >> 4);
        const uint4 *src = reinterpret_cast<const uint4 *>(A0);
        for (int c = threadIdx.x; c < nvec; c += kPackBlock) convert_piece(src[c], codes, badm, c);
    }
    __syncthreads();
    uint64_t w[kWMax];
#pragma unroll
    for (int t = 0; t < kWMax; ++t) w[t] = 0;
    int m = -1, mv = 0;
    if (i < nreads) {
        const int64_t a = offs[i], e = ends ? ends[i] : offs[i + 1];
        const int64_t m64 = e - a;
        if (m64 > kShortMax && m64 <= SA_MAX_READ) {
            m = (int)m64;  // long read: packed and searched by the long-read kernel
            mv = -1;
        } else if (m64 >= 0 && m64 <= kShortMax) {
            m = (int)m64;
            mv = m;
            if (staged && a >= span0 && e <= span1) {
                // word k: bases s + 32k .. s + 32k + 31 of the code stream
                const uint32_t st0 = (uint32_t)((uintptr_t)(reads + a) - A0);
#pragma unroll
                for (int k = 0; k < kWMax; ++k) {
                    if (32 * k < m) {
                        const uint32_t bpos = st0 + 32u * (uint32_t)k, q = bpos >> 4, r = bpos & 15u;
                        const uint64_t hi = ((uint64_t)codes[q] << 32) | codes[q + 1];
                        uint64_t x = r ? (hi << (2 * r)) | (codes[q + 2] >> (32 - 2 * r)) : hi;
                        const int rem = m - 32 * k;
                        if (rem < 32) x &= ~0ull << (64 - 2 * rem);
                        w[k] = x;
                    }
                }
                if (m > 0) {  // first byte that is not a base
                    const uint32_t q0 = st0 >> 4, q1 = (st0 + (uint32_t)m - 1) >> 4;
                    for (uint32_t q = q0; q <= q1; ++q) {
                        uint32_t bits = badm[q];
                        if (q == q0) bits &= 0xFFFFu << (st0 & 15u);
                        if (q == q1) bits &= (2u << ((st0 + (uint32_t)m - 1) & 15u)) - 1u;
                        if (bits) {
                            mv = (int)(q * 16u + (uint32_t)__builtin_ctz(bits) - st0);
                            break;
                        }
                    }
                }
            } else {
                uint64_t g[kWMax + 1];
                pack_from_global(reads, a, m, g, mv, g[kWMax]);
#pragma unroll
                for (int t = 0; t < kWMax; ++t) w[t] = (32 * t < m || t == 0) ? g[t] : 0;
            }
        }
    }
    // the words of the workgroup's searched reads, back to back from the
    // start of its region of qw (256 * kWMax words): read i's run starts at
    // word `wo` of the region
    __shared__ uint32_t scan_tmp[kPackBlock / 64];
    const int nw = (i < nreads && m >= 0 && mv >= 0) ? (m > 0 ? (m + 31) >> 5 : 1) : 0;
    uint32_t wo;
    const uint32_t run_words = block_exclusive_scan((uint32_t)nw, wo, scan_tmp);
    __syncthreads();  // the code stream is no longer needed
    uint64_t *slots = lds_buf;
    if (i < nreads) {
#pragma unroll
        for (int t = 0; t < kWMax; ++t)
            if (t < nw) slots[wo + t] = w[t];
        b.qlm[i] = encode_len(m, mv, (int)wo);
        if (bt.keys) {  // sort keys, only when the reads are sorted
            if (m >= 0 && mv < 0) {
                b.key[0][i] = long_read_key(bt.count);
            } else if (m >= 0) {
                int bucket = bt.count - 1;
                for (int j = 0; j < bt.count; ++j)
                    if (m <= bt.edge[j]) { bucket = j; break; }
                b.key[0][i] = ((uint32_t)bucket << 24) | (uint32_t)(w[0] >> 40);
            } else {
                b.key[0][i] = 0;
            }
            b.val[0][i] = (uint32_t)i;
        }
    }
    __syncthreads();
    // 16-byte stores of the used words only (an odd count rounds up within
    // the region, whose size is even)
    uint4 *dst = reinterpret_cast<uint4 *>(b.qw + (size_t)r0 * kWMax);
    const uint4 *srcv = reinterpret_cast<const uint4 *>(slots);
    for (uint32_t c = threadIdx.x; c < (run_words + 1) / 2; c += kPackBlock) dst[c] = srcv[c];
}

// First word of read rid's packed words in qw (its workgroup's region plus
// its offset there, as the pack kernel laid them out).
__device__ __forceinline__ const uint64_t *query_words(const uint64_t *qw, int rid, int wo) {
    return qw + (size_t)(rid & ~(kPackBlock - 1)) * kWMax + wo;
}

// ------------------------------------------------------------------ search

template <int W, class Cnt>
__device__ __forceinline__ void tuned_one(const DevIndex &ix, const uint64_t *s_key, const int32_t *s_sa,
                                          int levels, bool use_table, const BatchBuffers &b, int rid, int m, int mv,
                                          int wo, int4 *out, Cnt &cnt) {
    if (m < 0) {
        out[rid] = make_int4(0, 0, 0, (int)kHitTooLong);
        return;
    }
    uint64_t q[W];
    const uint64_t *src = query_words(b.qw, rid, wo);
    const int nw = m > 0 ? (m + 31) >> 5 : 1;
    load_query<W>(src, nw, q);
#pragma unroll
    for (int k = 0; k < W; ++k)
        if (k < nw) cnt.touch(src + k, 8);
    out[rid] = match_read<W>(ix, s_key, s_sa, levels, use_table, q, m, mv, cnt);
    cnt.touch(out + rid, 16);
}

// LDS written by this wave's lanes is visible to its other lanes.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum a per-lane 64-bit count over the wave and add it to a global counter.
__device__ __forceinline__ void wave_add64(unsigned long long *dst, unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0 && v) atomicAdd(dst, v);
}

// Sum a per-lane count over the wave and add it to a global counter.
__device__ __forceinline__ void wave_add(unsigned long long *dst, uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0 && v) atomicAdd(dst, (unsigned long long)v);
}

// Work split of the persistent kernel, with no global atomics: the reads
// (in input order, or prefix-sorted when the batch is sorted) are cut into
// chunks of 64 (one per lane of a wave) and the chunks into blocks of
// `group` chunks.  Workgroup rank r takes blocks r, r + G, r + 2G, ... (G
// workgroups), so every workgroup sees the same mix of read lengths, and
// all workgroups advance through one window of the order together.  The
// waves of a workgroup share its blocks through a counter in LDS.
// Workgroups are dispatched to the eight XCDs round-robin by id, so ranks
// are assigned XCD by XCD: neighbouring blocks (in a sorted batch, reads
// that visit the same index rows) run in one XCD's L2.
__device__ __forceinline__ int64_t workgroup_rank() {
    const int64_t G = gridDim.x, w = blockIdx.x;
    return (G % 8 == 0) ? (w % 8) * (G / 8) + w / 8 : w;
}

// The workgroup's chunk number c (-1 when its blocks are done; every later one
// lies further on).
__device__ __forceinline__ int64_t nth_chunk(unsigned c, int group, int64_t G, int64_t rank, int64_t nchunks) {
    const int64_t chunk = group == 1 ? (int64_t)c * G + rank
                                     : ((int64_t)(c / (unsigned)group) * G + rank) * group + (c % (unsigned)group);
    return chunk < nchunks ? chunk : -1;
}

// The next chunk of this wave.
__device__ __forceinline__ int64_t take_chunk(unsigned *next, int group, int64_t G, int64_t rank, int lane,
                                              int64_t nchunks) {
    unsigned c = 0;
    if (lane == 0) c = atomicAdd(next, 1u);
    return nth_chunk((unsigned)__builtin_amdgcn_readfirstlane((int)c), group, G, rank, nchunks);
}

// The instrumented kernels' counts, summed over the wave.
__device__ __forceinline__ void add_counts(unsigned long long *stats, const Count &cnt) {
    wave_add(&stats[0], cnt.global);
    wave_add(&stats[1], cnt.words);
    wave_add(&stats[2], cnt.tile);
    wave_add(&stats[5], cnt.keys);
    wave_add(&stats[6], cnt.table);
    wave_add64(&stats[7], cnt.touched);
    wave_add64(&stats[8], cnt.scattered);
    wave_add(&stats[9], cnt.index_loads);
}

// ---- reads packed by the pack kernel

// Persistent kernel: each workgroup stages the top `levels` tree levels in
// LDS once, then its waves take 64-read chunks until the workgroup's blocks
// are done.  Each chunk runs the instantiation for the longest read it
// holds.
template <int BLOCK, bool COUNT>
__global__ __launch_bounds__(BLOCK) void search_packed_kernel(DevIndex ix, int levels, int use_table_i, int group,
                                                              BatchBuffers b, const uint32_t *__restrict__ order,
                                                              int64_t nreads, int4 *__restrict__ out) {
    extern __shared__ uint64_t smem[];
    __shared__ unsigned s_next;
    const int nodes = (1 << levels) - 1;
    uint64_t *s_key = smem;
    int32_t *s_sa = reinterpret_cast<int32_t *>(smem + nodes);
    if (threadIdx.x == 0) s_next = 0u;
    for (int i = threadIdx.x; i < nodes; i += BLOCK) {
        s_key[i] = ix.tile_key[i];
        s_sa[i] = ix.tile_sa[i];
    }
    __syncthreads();
    using Cnt = typename std::conditional<COUNT, Count, NoCount>::type;
    Cnt cnt;
    uint32_t nsearched = 0, nqwords = 0;
    const bool use_table = use_table_i != 0;
    const int lane = threadIdx.x & 63;
    const int64_t nchunks = (nreads + 63) >> 6;
    const int64_t G = gridDim.x, rank = workgroup_rank();
    for (;;) {
        const int64_t chunk = take_chunk(&s_next, group, G, rank, lane, nchunks);
        if (chunk < 0) break;
        const int64_t j = (chunk << 6) + lane;
        const bool active = j < nreads;
        const int rid = active ? (order ? (int)order[j] : (int)j) : 0;
        const ReadLen lm = decode_len(active ? b.qlm[rid] : encode_len(0, 0, 0));
        if (COUNT && active) {
            if (order) cnt.touch(order + j, 4);
            cnt.touch(b.qlm + rid, 8);
        }
        const int m = lm.m;
        const bool short_read = active && !(m >= 0 && lm.mv < 0);  // long reads are the long kernel's
        const int w = max_i(1, (m + 31) >> 5);
        int wc = 1;
#pragma unroll
        for (int t = 2; t <= kWMax; ++t)
            if (wave_ballot(short_read && w >= t)) wc = t;
        if (active && !short_read && m >= 0) b.stats[kLongFlag] = 1ull;  // a long read: the long kernel runs
        if (!short_read) continue;
        if (COUNT && m >= 0) { nsearched++; nqwords += wc; }
        switch (wc) {
            case 1: tuned_one<1>(ix, s_key, s_sa, levels, use_table, b, rid, m, lm.mv, lm.wo, out, cnt); break;
            case 2: tuned_one<2>(ix, s_key, s_sa, levels, use_table, b, rid, m, lm.mv, lm.wo, out, cnt); break;
            case 3: tuned_one<3>(ix, s_key, s_sa, levels, use_table, b, rid, m, lm.mv, lm.wo, out, cnt); break;
            case 4: tuned_one<4>(ix, s_key, s_sa, levels, use_table, b, rid, m, lm.mv, lm.wo, out, cnt); break;
            case 5: tuned_one<5>(ix, s_key, s_sa, levels, use_table, b, rid, m, lm.mv, lm.wo, out, cnt); break;
            case 6: tuned_one<6>(ix, s_key, s_sa, levels, use_table, b, rid, m, lm.mv, lm.wo, out, cnt); break;
            case 7: tuned_one<7>(ix, s_key, s_sa, levels, use_table, b, rid, m, lm.mv, lm.wo, out, cnt); break;
            case 8: tuned_one<8>(ix, s_key, s_sa, levels, use_table, b, rid, m, lm.mv, lm.wo, out, cnt); break;
            case 9: tuned_one<9>(ix, s_key, s_sa, levels, use_table, b, rid, m, lm.mv, lm.wo, out, cnt); break;
            default: tuned_one<10>(ix, s_key, s_sa, levels, use_table, b, rid, m, lm.mv, lm.wo, out, cnt); break;
        }
    }
    if constexpr (COUNT) {
        wave_add(&b.stats[3], nsearched);
        wave_add(&b.stats[4], nqwords);
        add_counts(b.stats, cnt);
    }
}

// ---- reads packed by the search kernel itself

// Rows of a bracket that are looked at together, in one turn, instead of
// queued: as many records as a line holds.  More than half of the brackets of
// several rows have no more (16 Mbp: 4M reads of 100 bases 292 us with none,
// 264 with 2, 261 with 8 or 16; 100,000 of 25 bases 10.0, 9.6, 7.4; 250 Mbp /
// 64M reads 4.79, 4.63, 4.61 ms).
constexpr int kFewRows = 8;

// Words of a queued read's record before its codes: read id, length and
// leading bases, first row and size of its bracket (size 0: search from the
// root).
constexpr int kRecHead = 4;
static_assert(kPoolWords >= kRecHead + SA_MAX_READ / 16, "any read's record fits the pool");

// One wave's LDS area: the code stream (one dummy word, kStagePieces words of
// 16 codes, three words of slack for reads past the last), a bit per piece
// that holds a byte which is not a base, the offsets of the queued reads'
// records, then the records (with two words of slack).
struct WaveArea {
    uint32_t *codes, *bad, *rec_at, *pool;
};

// A query in LDS: word k is 32 codes from code 32k of a stream of 16-code
// words.  c points at the word before the one that holds the first code
// when that one starts it (sh 0), else at the one that holds it: a code
// stream word and the next joined by a right shift of 0..30 bits, so that no
// shift by 32 arises.
struct CodeQuery {
    const uint32_t *c;
    uint32_t sh;
    __device__ __forceinline__ uint32_t half(int j) const { return __builtin_amdgcn_alignbit(c[j], c[j + 1], sh); }
    __device__ __forceinline__ uint64_t operator[](int k) const {
        const uint32_t c0 = c[2 * k], c1 = c[2 * k + 1], c2 = c[2 * k + 2];
        return ((uint64_t)__builtin_amdgcn_alignbit(c0, c1, sh) << 32) | __builtin_amdgcn_alignbit(c1, c2, sh);
    }
};
// The query that starts at code `at` of a stream whose first word (codes
// 0..15) is words[1].
__device__ __forceinline__ CodeQuery code_query(const uint32_t *words, uint32_t at) {
    return CodeQuery{words + ((at + 15u) >> 4), 30u - 2u * ((at + 15u) & 15u)};
}

__device__ __forceinline__ int64_t lane_value(int64_t v, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The largest of the values (below 128) of the lanes in `mask`, the same
// for every lane.
__device__ __forceinline__ int wave_max7(int v, uint64_t mask) {
    int r = 0;
#pragma unroll
    for (int b = 6; b >= 0; --b) {
        const uint64_t t = wave_ballot((v >> b) & 1) & mask;
        if (t) {
            mask = t;
            r |= 1 << b;
        }
    }
    return r;
}

// Start and end of each read of a chunk of `per` reads (none when chunk <
// 0): loads issued here, used later.  Read j ends at offs[j + 1], or at
// ends[j] when an end array is given (reads gathered from anywhere in the
// buffer).
__device__ __forceinline__ void chunk_offsets(const int64_t *__restrict__ offs, const int64_t *__restrict__ ends,
                                              int64_t chunk, int per, int64_t nreads, int lane, int64_t &a,
                                              int64_t &e) {
    const int64_t j = chunk * per + lane;
    const bool act = chunk >= 0 && lane < per && j < nreads;
    a = act ? offs[j] : 0;
    e = act ? (ends ? ends[j] : offs[j + 1]) : 0;
}

// First byte of reads[a .. a + m) that is not a base (m when all are), for a
// read whose bytes lie at code `at` of the staged stream: only the pieces
// flagged in `bad` are looked at again.
__device__ __forceinline__ int first_non_base(const uint8_t *__restrict__ reads, int64_t a, int m, uint32_t at,
                                              const uint32_t *bad) {
    const uint32_t last = (at + (uint32_t)m - 1) >> 4;
    for (uint32_t pc = at >> 4; pc <= last;) {
        const uint32_t w = bad[pc >> 5] >> (pc & 31u);
        if (w == 0) {
            pc = (pc | 31u) + 1u;
            continue;
        }
        pc += (uint32_t)__builtin_ctz(w);
        if (pc > last) break;
        const uint4 v = *reinterpret_cast<const uint4 *>(reads + a + (int64_t)(16u * pc) - (int64_t)at);
        uint32_t b;
        pack4_fast(v.x, 0xFFFFFFFFu, b);
        uint32_t bits = bad_nibble(b);
        pack4_fast(v.y, 0xFFFFFFFFu, b);
        bits |= bad_nibble(b) << 4;
        pack4_fast(v.z, 0xFFFFFFFFu, b);
        bits |= bad_nibble(b) << 8;
        pack4_fast(v.w, 0xFFFFFFFFu, b);
        bits |= bad_nibble(b) << 12;
        if (pc == at >> 4) bits &= 0xFFFFu << (at & 15u);
        if (bits) {
            const int i = (int)(16u * pc + (uint32_t)__builtin_ctz(bits) - at);
            return i < m ? i : m;
        }
        ++pc;
    }
    return m;
}

// Stage `np` 16-byte pieces of ASCII from src as codes (codes[0] is the first
// piece's word) and set the bits of those with a byte that is not a base
// (the first piece is number `first`).  kStageRows loads in flight per lane.
// Returns, the same for every lane, whether there was such a piece.
constexpr int kStageRows = 4;

template <class Cnt>
__device__ __forceinline__ bool stage_pieces(const uint4 *__restrict__ src, int np, uint32_t *codes, uint32_t *bad,
                                             int first, int lane, Cnt &cnt) {
    bool any = false;
#pragma unroll 1
    for (int c0 = 0; c0 < np; c0 += 64 * kStageRows) {
        uint4 r[kStageRows];
#pragma unroll
        for (int u = 0; u < kStageRows; ++u) {
            const int c = c0 + 64 * u + lane;
            if (c < np) {
                r[u] = load_stream16(src + c);
                cnt.touch(src + c, 16);
            }
        }
#pragma unroll
        for (int u = 0; u < kStageRows; ++u) {
            const int c = c0 + 64 * u + lane;
            if (c < np) {
                uint32_t b;
                codes[c] = convert16(r[u], b);
                if (b) {
                    atomicOr(&bad[(first + c) >> 5], 1u << ((first + c) & 31));
                    any = true;
                }
            }
        }
    }
    return __any(any);
}

// The same for reads that lie apart: lane l's first `np` pieces (none: 0) go to
// pieces off, off + 1, ... of the area (off: the sum of np over the lanes
// before), `total` in all.  Each piece's read is found by a binary search over
// the lanes' offsets, so that the loads of all reads are in flight together.
constexpr int kApartRows = 2;  // loads in flight per lane (4 spill registers and gain nothing)

template <class Cnt>
__device__ __forceinline__ bool stage_reads(const uint8_t *__restrict__ reads, int64_t a, int off, int total,
                                            uint32_t *codes, uint32_t *bad, int lane, Cnt &cnt) {
    bool any = false;
#pragma unroll 1
    for (int c0 = 0; c0 < total; c0 += 64 * kApartRows) {
        uint4 r[kApartRows];
#pragma unroll
        for (int u = 0; u < kApartRows; ++u) {
            const int c = c0 + 64 * u + lane;
            int owner = 0;
#pragma unroll
            for (int step = 32; step > 0; step >>= 1)
                if (__shfl(off, owner + step, 64) <= c) owner += step;
            const int k = c - __shfl(off, owner, 64);
            const uint4 *src =
                reinterpret_cast<const uint4 *>((uintptr_t)(reads + __shfl(a, owner, 64)) & ~(uintptr_t)15) + k;
            if (c < total) {
                r[u] = load_stream16(src);
                cnt.touch(src, 16);
            }
        }
#pragma unroll
        for (int u = 0; u < kApartRows; ++u) {
            const int c = c0 + 64 * u + lane;
            if (c < total) {
                uint32_t b;
                codes[c] = convert16(r[u], b);
                if (b) {
                    atomicOr(&bad[c >> 5], 1u << (c & 31));
                    any = true;
                }
            }
        }
    }
    return __any(any);
}

// Searches the wave's queued reads, each by a group of `size` neighbouring
// lanes: as many as the wave has for each read (32 reads: two lanes each;
// one read: all 64), the lanes of a group probing the interval between the
// bounds at as many evenly spaced rows at a time.  A full queue thus takes
// few loads per read, a short one few loads one after the other: with 8
// lanes per read a bracket of 1000 rows takes 4 steps instead of 10, which is
// what bounds small batches (16 Mbp, 20,000 reads of 150 bases: 15.4 us,
// 24.6 with one lane per read; 64 reads of 30-300: 8.0 us, 11.2).  A group
// goes through the searches of finish_read in turn (LB of P[0..v), then LB
// and RB of P[0..l)) without waiting for the other groups.
template <class Cnt>
__device__ __forceinline__ void search_queued(const DevIndex &ix, const uint64_t *t_key, const int32_t *t_sa, int levels,
                                              const WaveArea &w, int queued, int lane, int4 *__restrict__ out, Cnt &cnt) {
    const int bits = 6 - (queued > 1 ? 32 - __builtin_clz((unsigned)queued - 1u) : 0);
    const int size = 1 << bits, sub = lane & (size - 1), first_lane = lane - sub;
    if ((lane >> bits) >= queued) return;
    const uint64_t ones = size == 64 ? ~0ull : (1ull << size) - 1ull;
    const uint32_t share = 0xFFFFFFFFu / (uint32_t)(size + 1) * (uint32_t)(sub + 1);  // of the rows inside, times 2^32
    const uint32_t *r = w.pool + w.rec_at[lane >> bits];
    const CodeQuery q{r + kRecHead - 1, 0};
    // phase 0: LB search of P[0..plen), all of st in use; 1 and 2: LB and RB
    // search of P[0..plen) between st.L and st.R
    int phase = 0, plen = (int)(r[1] >> 16), lo = 0, above = 0, above_lcp = 0;
    LbState st;
    if (r[3]) {
        open_bracket(ix, (int)r[2], (int)r[3], st);
    } else {
        lb_tile<kWordsInLds>(ix, t_key, t_sa, levels, q, plen, st, cnt);
    }
    for (;;) {
        if (st.R == st.L + 1) {
            if (phase == 0) {
                // (the record is read again rather than held in registers through the loop)
                __asm__ volatile("" ::: "memory");
                const bool exact = plen == (int)(r[1] & 0xFFFFu) && st.lcpR == plen;
                const int l = max_i(st.lcpL, st.lcpR);
                if (l == 0) {
                    lo = 0;
                    st.R = ix.n;
                    plen = 0;
                    break;
                }
                plen = l;
                above = st.R;
                above_lcp = st.lcpR;
                lo = st.R;
                phase = 1;
                if (!exact && st.lcpL == l) {  // rows below the insertion point share P[0..l)
                    st.R = st.L;
                    st.lcpR = l;
                    st.L = st.Llt;
                    st.lcpL = st.lcpLlt;
                    continue;
                }
            } else if (phase == 1) {
                lo = st.R;
            }
            if (phase == 2) break;
            if (above_lcp < plen) {  // no row above the insertion point does
                st.R = above;
                break;
            }
            phase = 2;
            st.L = above;
            st.lcpL = above_lcp;
            st.R = st.Rlt;
            st.lcpR = st.lcpRlt;
            continue;
        }
        const int inside = st.R - st.L - 1;
        const bool all = inside <= size;  // every row between the bounds at once
        const int piv = st.L + 1 + (all ? sub : (int)__umulhi((uint32_t)inside, share));
        const bool probe = !all || sub < inside;
        int lcp = 0;
        bool left = false;
        if (probe) {
            const RowHead row = row_head(ix.rows, piv);
            cnt.index_touch(ix.rows + piv, 16);
            cnt.key_probe();
            const int sign = compare_row<kWordsInLds>(ix, q, plen, ix.rows + piv, row.pos, row.key0,
                                                      min_i(st.lcpL, st.lcpR), lcp, cnt);
            left = phase == 2 ? sign < 0 : sign <= 0;
        }
        // the group's first probe that moves R, and the one before it, which moves L
        const int probes = all ? inside : size;
        const uint64_t lefts = (wave_ballot(left) >> first_lane) & ones;
        const int to_r = lefts ? (int)__builtin_ctzll(lefts) : probes;
        const int lane_r = first_lane + min_i(to_r, size - 1), lane_l = first_lane + max_i(to_r - 1, 0);
        const int piv_r = __shfl(piv, lane_r, 64), lcp_r = __shfl(lcp, lane_r, 64);
        const int piv_l = __shfl(piv, lane_l, 64), lcp_l = __shfl(lcp, lane_l, 64);
        if (phase == 0) {
            // the last row on either side that shares fewer bases than the new bound
            const uint64_t fewer_l = (wave_ballot(lcp < lcp_l) >> first_lane) & ones & ((1ull << max_i(to_r - 1, 0)) - 1ull);
            const uint64_t fewer_r =
                to_r < probes ? (wave_ballot(probe && lcp < lcp_r) >> first_lane) & ones & ~((2ull << to_r) - 1ull) : 0ull;
            const int lane_fl = first_lane + (fewer_l ? 63 - (int)__builtin_clzll(fewer_l) : 0);
            const int lane_fr = first_lane + (fewer_r ? (int)__builtin_ctzll(fewer_r) : 0);
            const int piv_fl = __shfl(piv, lane_fl, 64), lcp_fl = __shfl(lcp, lane_fl, 64);
            const int piv_fr = __shfl(piv, lane_fr, 64), lcp_fr = __shfl(lcp, lane_fr, 64);
            if (to_r > 0) {
                if (fewer_l) {
                    st.Llt = piv_fl;
                    st.lcpLlt = lcp_fl;
                } else if (lcp_l > st.lcpL) {
                    st.Llt = st.L;
                    st.lcpLlt = st.lcpL;
                }
            }
            if (to_r < probes) {
                if (fewer_r) {
                    st.Rlt = piv_fr;
                    st.lcpRlt = lcp_fr;
                } else if (lcp_r > st.lcpR) {
                    st.Rlt = st.R;
                    st.lcpRlt = st.lcpR;
                }
            }
        }
        if (to_r > 0) {
            st.L = piv_l;
            st.lcpL = lcp_l;
        }
        if (to_r < probes) {
            st.R = piv_r;
            st.lcpR = lcp_r;
        }
    }
    __asm__ volatile("" ::: "memory");
    if (sub == 0) {
        const int id = (int)r[0], m = (int)(r[1] & 0xFFFFu);
        store_stream16(out + id, make_int4(lo, st.R, plen, plen == m ? (int)kHitExact : 0));
        cnt.touch(out + id, 16);
    }
}

// Pieces of ASCII (aligned 16 bytes) that hold bytes of reads[a .. a + m).
__device__ __forceinline__ int piece_count(const uint8_t *reads, int64_t a, int m) {
    return (int)((((uintptr_t)(reads + a) & 15) + (uint32_t)m + 15) >> 4);
}

// The sum of v over the lanes before this one; total: over all.
__device__ __forceinline__ int wave_excl_sum(int v, int lane, int &total) {
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    total = __builtin_amdgcn_readlane(x, 63);
    return x - v;
}

// A chunk with reads of more than kLongRead bases that does not fit the
// staging area is first staged only kProbePieces pieces a read: most reads are
// settled by their first bases (those that are not from this reference by the
// table's k, those with an error by the first one), and the rest of their
// bytes is never read.  What matches as far as it was staged is staged whole
// in the turns after.  16 Mbp, 400,000 reads of 800 bases 195 us without it,
// 103 with it; 200,000 of 20-1024 87 and 55; 1M of 400 178 and 160; 65,536 of
// 1024 on 10 Mbp 52.6 and 41.6.  From 200 bases on it costs more than it saves
// (4M of 20-300: 393 against 338 us: neighbouring reads share their lines),
// and so it does for chunks that fit half of the area (50,001 of 20-1024:
// 40.3 against 37.2).
constexpr int kLongRead = 320;
constexpr int kProbePieces = 11;
static_assert(64 * kProbePieces <= kStagePieces && 16 * (kProbePieces - 1) >= kMaxPrefixBases,
              "a chunk's first pieces fit, and hold a table's string");

// The search kernel of a batch in input order: it takes the reads as they
// lie in memory (ASCII, with CSR offsets or with an end array) and needs no
// pass before or after it.
//
// Work: chunks of `per` consecutive reads, one read per lane, taken as in
// search_packed_kernel; batches too small to give every wave 64 reads use
// smaller chunks.  For a chunk the wave
//   1. stages the reads' bytes as 2-bit codes in its LDS area: runs of reads
//      that follow each other in memory, as many as fit (reads of up to
//      SA_MAX_READ bases; what does not fit is the next turn's), with
//      coalesced 16-byte loads.  The codes stay in LDS and the comparisons
//      take them from there word by word, so that a query of any length
//      costs no registers;
//   2. looks up each read's prefix-table entry.  An entry that answers the
//      read, or whose bracket is a single row (one comparison then gives the
//      whole result), is finished here;
//   3. queues every other read (brackets of more rows, reads shorter than
//      the table's strings, and all reads when there is no table): its codes
//      and its entry are copied into the wave's record pool.  When the pool
//      is full, or after the last chunk (after each turn with defer == 0), the
//      queued reads are searched together, so that long binary searches run
//      with all lanes busy and hold up nobody (search_queued).
//
// What bounds it: lines. On MI355X a random 16-byte load brings in a 128-byte
// line whatever the cache policy (loads of both halves of a line run at the
// rate of one), at most 52-58 G lines/s.  The 250 Mbp / 64M x 150 batch needs
// about 3.2 per read: 1.3 of ASCII, offsets and results, which alone take 2.0
// ms (5.6 TB/s), the table entry (1.6 ms more), and the text, which hides
// behind them; what is left is the queued searches.  Measured at first (words
// in registers, a second kernel for long reads, set-aside reads read again)
// and now: that batch 5.33 and 4.47 ms; 16 Mbp, 4M x 100 bases 393 and 243
// us, 4M x 20-300 580 and 321 us, 50,001 x 20-1024 264 and 37 us, 65,536 x
// 1024 (on 10 Mbp) 113 and 41 us, 64 x 30-300 30 and 8 us.
template <bool COUNT, bool TILE>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(COUNT ? 1 : kSearchWavesPerSimd))) void search_reads_kernel(
    DevIndex ix, int levels, int use_table_i, int group, int per, int64_t nchunks, int defer, InlineArea area,
    unsigned long long *__restrict__ stats, const uint8_t *__restrict__ reads, const int64_t *__restrict__ offs,
    const int64_t *__restrict__ ends, int64_t nreads, int4 *__restrict__ out) {
    extern __shared__ uint64_t smem[];
    __shared__ unsigned s_next;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // the tree's top levels: in LDS when every search starts there (TILE),
    // else read from memory by the few reads that need them
    const uint64_t *t_key = ix.tile_key;
    const int32_t *t_sa = ix.tile_sa;
    if constexpr (TILE) {
        const int nodes = (1 << levels) - 1;
        uint64_t *s_key = smem;
        int32_t *s_sa = reinterpret_cast<int32_t *>(smem + nodes);
        for (int i = threadIdx.x; i < nodes; i += blockDim.x) {
            s_key[i] = ix.tile_key[i];
            s_sa[i] = ix.tile_sa[i];
        }
        t_key = s_key;
        t_sa = s_sa;
    }
    if (threadIdx.x == 0) s_next = blockDim.x >> 6;
    WaveArea w;
    w.codes = reinterpret_cast<uint32_t *>(smem) + area.first_word + wave * area.wave_words;
    w.bad = w.codes + kStagePieces + 4;
    w.rec_at = w.bad + kStageBadWords;
    w.pool = w.rec_at + kQueueReads;
    using Cnt = typename std::conditional<COUNT, Count, NoCount>::type;
    Cnt cnt;
    uint32_t nsearched = 0, nqwords = 0;
    const bool use_table = use_table_i != 0 && ix.ptab_k > 0;
    const int K = ix.ptab_k;
    const int64_t G = gridDim.x, rank = workgroup_rank();

    // each wave's first chunk goes by its number, so that its loads need not wait for the counter
    int64_t c1 = nth_chunk((unsigned)wave, group, G, rank, nchunks), a1, e1;
    chunk_offsets(offs, ends, c1, per, nreads, lane, a1, e1);
    __syncthreads();  // the counter and the tile are in place
    int64_t a = 0;         // this lane's read of the current chunk: where it starts, its length
    int m = 0, id0 = 0;    // (and lane 0's id)
    uint64_t todo = 0;     // lanes of the current chunk whose reads are not staged yet
    uint64_t pend = 0;     // lanes whose staged reads wait to be queued
    int mv = 0;            // of a staged read: its leading bases, its place in the code stream, its bracket
    uint32_t at = 0, row = 0, size = 0;
    int probes = 0;        // of the current chunk (see kLongRead): 2 before the turn of first pieces, 1 after it
    int queued = 0, used = 0;  // records in the pool, words of it in use (wave-uniform)
    for (;;) {
        if (pend) {
            // as many as fit, each a record of 4 words and its codes
            const CodeQuery q = code_query(w.codes, at);
            const int nd = (mv + 15) >> 4;
            const int ndmax = wave_max7(nd, pend), stride = kRecHead + ndmax;
            const int room = min_i(kQueueReads - queued, (kPoolWords - used) / stride);
            const int my = __popcll(pend & ((1ull << lane) - 1ull));
            const bool mine = (pend >> lane) & 1ull;
            const bool push = mine && my < room;
            const int to = used + my * stride;
            if (push) {
                w.rec_at[queued + my] = (uint32_t)to;
                uint32_t *r = w.pool + to;
                r[0] = (uint32_t)(id0 + lane);
                r[1] = (uint32_t)m | ((uint32_t)mv << 16);
                r[2] = row;
                r[3] = size;
            }
            for (int t = 0; t < ndmax; ++t)
                if (push && t < nd) w.pool[to + kRecHead + t] = q.half(t);
            const uint64_t pushed = wave_ballot(push);
            const int n = __popcll(pushed);
            pend &= ~pushed;
            queued += n;
            used += n * stride;
            wave_lds_sync();
        }
        const bool last = c1 < 0 && todo == 0;
        if (pend || (queued > 0 && (last || defer == 0))) {
            search_queued(ix, t_key, t_sa, levels, w, queued, lane, out, cnt);
            wave_lds_sync();
            queued = 0;
            used = 0;
            continue;
        }
        if (last) break;
        if (todo == 0) {
            // the next chunk; its successor's offsets are loaded meanwhile
            a = a1;
            const int64_t m64 = e1 - a1;
            const int64_t j = c1 * per + lane;
            const bool active = lane < per && j < nreads;
            id0 = (int)(c1 * per);
            c1 = take_chunk(&s_next, group, G, rank, lane, nchunks);
            chunk_offsets(offs, ends, c1, per, nreads, lane, a1, e1);
            const bool valid = active && m64 >= 0 && m64 <= SA_MAX_READ;
            if (COUNT && active) {
                cnt.touch(offs + j, ends ? 8 : 16);
                if (ends) cnt.touch(ends + j, 8);
                if (valid) {
                    nsearched++;
                    nqwords += (uint32_t)max_i(1, (int)((m64 + 31) >> 5));
                }
            }
            if (active && (!valid || m64 == 0))
                store_stream16(out + (id0 + lane), valid ? make_int4(0, ix.n, 0, (int)kHitExact)
                                                : make_int4(0, 0, 0, (int)kHitTooLong));
            m = (int)m64;
            const bool in = valid && m64 > 0;
            todo = wave_ballot(in);
            if (todo == 0) continue;
            probes = 0;
            if (use_table && wave_ballot(in && m > kLongRead)) {
                int total = 0;
                (void)wave_excl_sum(in ? piece_count(reads, a, m) : 0, lane, total);
                probes = total > kStagePieces ? 2 : 0;
            }
        }
        // stage as many of the reads as fit
        if (lane < kStageBadWords) w.bad[lane] = 0;
        wave_lds_sync();
        uint64_t staged = 0;
        bool any_bad = false;
        int have = m;  // bases of this lane's read that get staged
        if (probes) {
            const int limit = probes > 1 ? kProbePieces : kStagePieces;
            int total;
            const bool in = ((todo >> lane) & 1ull) != 0;
            const int np = in ? min_i(piece_count(reads, a, m), limit) : 0;
            const int off = wave_excl_sum(np, lane, total);
            staged = wave_ballot(in && off + np <= kStagePieces);
            total = min_i(total, __builtin_amdgcn_readlane(off + np, 63 - (int)__builtin_clzll(staged)));
            any_bad = stage_reads(reads, a, off, total, w.codes + 1, w.bad, lane, cnt);
            const int skew = (int)((uintptr_t)(reads + a) & 15);
            at = 16u * (uint32_t)off + (uint32_t)skew;
            have = min_i(m, 16 * np - skew);
            todo &= ~staged;
            probes = 1;
        }
        int filled = 0;
        while (!probes && todo) {
            const int f = __ffsll((unsigned long long)todo) - 1;
            const uint8_t *A0 = reinterpret_cast<const uint8_t *>((uintptr_t)(reads + lane_value(a, f)) & ~(uintptr_t)15);
            // the run: lanes f, f + 1, ... while each read starts where the one before ends and still fits
            // (empty ones among them take no room, and are finished already)
            const int64_t e = a + m, before = __shfl_up(e, 1, 64);
            const int64_t stop = (int64_t)((((uintptr_t)(reads + e) + 15) & ~(uintptr_t)15) - (uintptr_t)A0);
            const bool in = ((todo >> lane) & 1ull) != 0;
            const bool ends_run = lane >= f && ((lane > f && a != before) || (!in && e != a) ||
                                                stop > (int64_t)(kStagePieces - filled) * 16);
            const uint64_t cut = wave_ballot(ends_run);
            const int end = cut ? __ffsll((unsigned long long)cut) - 1 : 64;
            if (end == f) break;  // no room for one more
            const int np = (int)(lane_value(stop, end - 1) >> 4);
            if (lane >= f && lane < end) at = 16u * (uint32_t)filled + (uint32_t)((uintptr_t)(reads + a) - (uintptr_t)A0);
            any_bad |= stage_pieces(reinterpret_cast<const uint4 *>(A0), np, w.codes + 1 + filled, w.bad, filled, lane, cnt);
            const uint64_t run = (end == 64 ? ~0ull : (1ull << end) - 1ull) & ~((1ull << f) - 1ull);
            staged |= run & todo;
            todo &= ~run;
            filled += np;
        }
        wave_lds_sync();
        const bool mine = (staged >> lane) & 1ull;
        const CodeQuery q = code_query(w.codes, at);
        mv = have;
        if (any_bad && mine) mv = first_non_base(reads, a, have, at, w.bad);
        size = 0;
        bool queue = mine;
        int4 hit = make_int4(0, ix.n, 0, 0);
        if (mine && mv == 0) {
            queue = false;
        } else if (mine && use_table && mv >= K) {
            const uint64_t q0 = q[0];
            const PrefixEntry ent = table_entry(ix, (uint32_t)(q0 >> (64 - 2 * K)), cnt);
            row = ent.row;
            size = ent.size;
            if (size & kPtabAnswer) {
                hit = make_int4(ent.pos, (int)ent.next, (int)(size & ~kPtabAnswer), 0);
                queue = false;
            } else if (size <= kFewRows) {
                // one row: it is the entry's pivot, whose next 16 bases came along; more: their first 32
                // bases from their records, which lie in a line or two
                int from = 0, lcp = 0;  // the candidate's text is compared from this word on
                int32_t pos = ent.pos;
                int first = (int)row, end = (int)row + 1;
                bool text = true;
                queue = false;
                if (size == 1) {
                    cnt.global_probe();
                    const int lim = min_i(mv, ix.n - pos);
                    const uint32_t x = (uint32_t)((q0 << (2 * K)) >> 32) ^ ent.next;
                    const int same = K + (x ? (int)(__clz((int)x) >> 1) : 16);
                    from = K == 16 ? 1 : 0;
                    lcp = min_i(same, lim);
                    text = same == K + 16 && lim > same;
                } else {
                    first = end = 0;
#pragma unroll 1
                    for (int r = 0; r < (int)size; r += 2) {
                        RowHead h[2];
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            if (r + i < (int)size) {
                                h[i] = row_head(ix.rows, (int)row + r + i);
                                cnt.index_touch(ix.rows + row + r + i, 16);
                                cnt.key_probe();
                            }
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            if (r + i < (int)size) {
                                const uint64_t x = q0 ^ h[i].key0;
                                const int same = min_i(x ? (int)(__clzll((long long)x) >> 1) : 32, min_i(mv, h[i].len));
                                if (same > lcp) {
                                    lcp = same;
                                    first = (int)row + r + i;
                                    pos = h[i].pos;
                                }
                                if (same == lcp) end = (int)row + r + i + 1;
                            }
                    }
                    from = 1;
                    text = lcp == 32 && mv > 32;
                    queue = text && end - first > 1;  // several rows share all 32 bases
                }
                if (text && !queue) compare_text(ix, q, mv, pos, from, lcp, cnt);
                hit = make_int4(first, end, lcp, lcp == m ? (int)kHitExact : 0);
            }
        }
        // a read that matches as far as it was staged, or needs a longer search, is staged whole
        const bool more = mine && have < m && mv == have && (queue || hit.z == mv);
        if (mine && !queue && !more) {
            store_stream16(out + (id0 + lane), hit);
            cnt.touch(out + (id0 + lane), 16);
        }
        pend = wave_ballot(queue && !more);
        todo |= wave_ballot(more);
    }
    if constexpr (COUNT) {
        wave_add(&stats[3], nsearched);
        wave_add(&stats[4], nqwords);
        add_counts(stats, cnt);
    }
}

// Plain kernel, the paper's arrangement (Algorithm 1): one read per
// thread in input order, every search over the whole range (-1, n), every
// probe comparing from the first base, no LDS.  Exact reads take the LB and
// RB searches; other reads add the two neighbour comparisons for l and the
// LB / RB searches of P[0..l).
template <bool UPPER, class Cnt>
__device__ __forceinline__ int plain_search(const DevIndex &ix, const uint64_t (&q)[kWMax], int plen, Cnt &cnt) {
    int L = -1, R = ix.n;
    while (R > L + 1) {
        const int piv = midpoint(L, R);
        int lcp;
        cnt.global_probe();
        cnt.index_touch(ix.sa + piv, 4);
        const int sign = compare_from<kWMax>(ix.text, ix.n, q, plen, ix.sa[piv], 0, lcp, cnt);
        if (UPPER ? (sign < 0) : (sign <= 0)) R = piv; else L = piv;
    }
    return R;
}

template <bool COUNT>
__global__ __launch_bounds__(256) void search_plain_kernel(DevIndex ix, BatchBuffers b, int64_t nreads,
                                                          int4 *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    using Cnt = typename std::conditional<COUNT, Count, NoCount>::type;
    Cnt cnt;
    int4 res = make_int4(0, 0, 0, (int)kHitTooLong);
    const ReadLen lm = decode_len(i < nreads ? b.qlm[i] : encode_len(-1, 0, 0));
    if (COUNT && i < nreads) cnt.touch(b.qlm + i, 8);
    const int m = lm.m;
    const bool long_read = m >= 0 && lm.mv < 0;  // the long kernel's
    if (long_read) b.stats[kLongFlag] = 1ull;
    if (m >= 0 && !long_read) {
        const int mv = lm.mv;
        uint64_t q[kWMax];
        const uint64_t *src = query_words(b.qw, (int)i, lm.wo);
#pragma unroll
        for (int k = 0; k < kWMax; ++k) q[k] = (k << 5) < m ? src[k] : 0ull;
#pragma unroll
        for (int k = 0; k < kWMax; ++k)
            if ((k << 5) < m) cnt.touch(src + k, 8);
        const int lo = plain_search<false>(ix, q, mv, cnt);
        int hi = lo;
        if (mv == m) hi = plain_search<true>(ix, q, m, cnt);
        if (mv == m && lo < hi) {
            res = make_int4(lo, hi, m, (int)kHitExact);
        } else {
            int l = 0, lcp;
            if (lo > 0) {
                cnt.global_probe();
                cnt.index_touch(ix.sa + lo - 1, 4);
                compare_from<kWMax>(ix.text, ix.n, q, mv, ix.sa[lo - 1], 0, lcp, cnt);
                l = max_i(l, lcp);
            }
            if (lo < ix.n) {
                cnt.global_probe();
                cnt.index_touch(ix.sa + lo, 4);
                compare_from<kWMax>(ix.text, ix.n, q, mv, ix.sa[lo], 0, lcp, cnt);
                l = max_i(l, lcp);
            }
            res = make_int4(plain_search<false>(ix, q, l, cnt), plain_search<true>(ix, q, l, cnt), l,
                            l == m ? (int)kHitExact : 0);
        }
    }
    if (i < nreads && !long_read) {
        out[i] = res;
        cnt.touch(out + i, 16);
    }
    if constexpr (COUNT) {
        wave_add(&b.stats[0], cnt.global);
        wave_add(&b.stats[1], cnt.words);
        wave_add(&b.stats[3], m >= 0 && !long_read ? 1u : 0u);
        wave_add(&b.stats[4], m >= 0 && !long_read ? (uint32_t)max_i(1, (m + 31) >> 5) : 0u);
        wave_add64(&b.stats[7], cnt.touched);
        wave_add64(&b.stats[8], cnt.scattered);
        wave_add(&b.stats[9], cnt.index_loads);
    }
}

// Dynamic LDS a search kernel may take (set by prepare_kernels from the
// device's limit per workgroup).
std::atomic<size_t> g_inline_lds{0};

template <class F>
hipError_t allow_lds(F *kernel, size_t bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
}

template <int BLOCK, bool COUNT>
hipError_t launch_packed_block(const DevIndex &ix, int levels, int use_table, int group, int grid,
                               const BatchBuffers &b, const uint32_t *order, int64_t nreads, int4 *out, hipStream_t s) {
    hipLaunchKernelGGL((search_packed_kernel<BLOCK, COUNT>), dim3(grid), dim3(BLOCK), tile_lds_bytes(levels), s, ix,
                       levels, use_table, group, b, order, nreads, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ long reads

// Query words in LDS, read on demand by the comparisons.
struct LdsQuery {
    const uint64_t *p;
    __device__ __forceinline__ uint64_t operator[](int k) const { return p[k]; }
};

// The whole wave packs one read of m <= SA_MAX_READ bases at reads[a..a+m)
// into dst[0 .. 32): lane l converts bases 16l .. 16l+15 from aligned dword
// loads (an aligned dword that holds a byte of the read never crosses a
// page) and writes its half word.  Split in two so that a wave can have the
// loads of several reads in flight before it converts them.
struct PackLoad {
    uint32_t dw[5];
    uint32_t sh;
};

template <class Cnt>
__device__ __forceinline__ PackLoad wave_pack_load(const uint8_t *__restrict__ reads, int64_t a, int m, int lane,
                                                   Cnt &cnt) {
    PackLoad pl;
    const int b0 = 16 * lane;
    const uintptr_t x0 = (uintptr_t)(reads + a + b0);
    const uintptr_t base = x0 & ~(uintptr_t)3;
    const uintptr_t stop = (uintptr_t)(reads + a + m);
    pl.sh = (uint32_t)(x0 & 3u);
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        const bool in = b0 < m && base + 4u * t < stop;
        pl.dw[t] = in ? *reinterpret_cast<const uint32_t *>(base + 4u * t) : 0u;
        if (in) cnt.touch(reinterpret_cast<const void *>(base + 4u * t), 4);
    }
    return pl;
}

// Returns this lane's first non-ACGT base (0x7FFFFFFF if none); the caller
// takes the minimum over the wave.
__device__ __forceinline__ int wave_pack_store(const PackLoad &pl, int m, uint64_t *dst, int lane) {
    const int b0 = 16 * lane;
    uint32_t half = 0;
    int bad_at = 0x7FFFFFFF;
    if (b0 < m) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const int rem = m - b0 - 4 * jj;
            const uint32_t keep = rem >= 4 ? 0xFFFFFFFFu : (rem > 0 ? ((1u << (8 * rem)) - 1u) : 0u);
            uint32_t bad;
            const uint32_t b8 = pack4_fast(__builtin_amdgcn_alignbyte(pl.dw[jj + 1], pl.dw[jj], pl.sh), keep, bad);
            if (bad && bad_at == 0x7FFFFFFF) bad_at = b0 + 4 * jj + (int)(__builtin_ctz(bad) >> 3);
            half = (half << 8) | b8;
        }
    }
    // bases 32k .. 32k+15 (lane 2k) are the high half of word k
    reinterpret_cast<uint32_t *>(dst + (lane >> 1))[(lane & 1) ? 0 : 1] = half;
    return bad_at;
}

// Packs the reads of the lanes in `todo` (a wave-uniform mask; rows `rid`,
// starts `start`, lengths `len` per lane) into their lanes' LDS slots, eight
// reads' loads in flight at a time; *mv of each such lane becomes its
// length up to the first non-ACGT base.
constexpr int kPackInFlight = 8;

template <class Cnt>
__device__ __forceinline__ void wave_pack_reads(const uint8_t *__restrict__ reads, uint64_t todo, int64_t start,
                                                int len, uint64_t (*slot)[kLongWords], int lane, int &mv,
                                                Cnt &cnt) {
    while (todo) {
        int src[kPackInFlight], m[kPackInFlight];
        PackLoad pl[kPackInFlight];
        int nb = 0;
#pragma unroll
        for (int u = 0; u < kPackInFlight; ++u) {
            src[u] = 0;
            m[u] = 0;
            if (todo) {
                src[u] = __ffsll((unsigned long long)todo) - 1;
                todo &= todo - 1;
                m[u] = __shfl(len, src[u], 64);
                pl[u] = wave_pack_load(reads, __shfl(start, src[u], 64), m[u], lane, cnt);
                nb = u + 1;
            }
        }
#pragma unroll
        for (int u = 0; u < kPackInFlight; ++u) {
            if (u < nb) {
                int first_bad = wave_pack_store(pl[u], m[u], slot[src[u]], lane);
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) first_bad = min_i(first_bad, __shfl_xor(first_bad, o, 64));
                if (lane == src[u]) mv = min_i(m[u], first_bad);
            }
        }
    }
}

// One wave per workgroup.  In a sorted batch long reads sort last: each
// workgroup finds where they start, then takes 64-row chunks from there (an
// unsorted batch is scanned from its first read).  For every long read of
// a chunk the whole wave packs it into that lane's LDS slot, 16 bases per
// lane from aligned dword loads (an aligned dword holding a byte of the
// read never crosses a page); then each lane searches its own read with
// the query read from LDS.
template <bool COUNT>
__global__ __launch_bounds__(64) void search_long_kernel(DevIndex ix, const uint8_t *__restrict__ reads,
                                                         const int64_t *__restrict__ offs, BatchBuffers b,
                                                         const uint32_t *__restrict__ order,
                                                         const uint32_t *__restrict__ sorted_key, int key_shift,
                                                         uint32_t key_mask, uint32_t long_field, int use_table_i,
                                                         int64_t nreads, int4 *__restrict__ out) {
    __shared__ uint64_t slot[64][kLongWords];
    __shared__ int64_t s_first;
    const int lane = threadIdx.x;
    // the search kernel before this one flags batches that hold long reads
    if (*reinterpret_cast<volatile const unsigned long long *>(b.stats + kLongFlag) == 0ull) return;
    if (lane == 0) {
        int64_t lo = 0, hi = nreads;  // first sorted row whose key field reaches long_field
        if (sorted_key) {
            while (lo < hi) {
                const int64_t mid = lo + ((hi - lo) >> 1);
                if (((sorted_key[mid] >> key_shift) & key_mask) >= long_field) hi = mid;
                else lo = mid + 1;
            }
        }
        s_first = lo;
    }
    __syncthreads();
    const int64_t first = s_first;
    const int64_t nchunks = (nreads - first + 63) >> 6;
    using Cnt = typename std::conditional<COUNT, Count, NoCount>::type;
    Cnt cnt;
    uint32_t nsearched = 0, nqwords = 0;
    const bool use_table = use_table_i != 0;
    for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const int64_t j = first + (c << 6) + lane;
        const bool act = j < nreads;
        const int rid = act ? (order ? (int)order[j] : (int)j) : 0;
        const ReadLen lm = decode_len(act ? b.qlm[rid] : encode_len(-1, 0, 0));
        if (COUNT && act) {
            if (order) cnt.touch(order + j, 4);
            cnt.touch(b.qlm + rid, 8);
        }
        const bool is_long = act && lm.m >= 0 && lm.mv < 0;
        uint64_t todo = wave_ballot(is_long);
        if (!todo) continue;
        int mv_mine = lm.m;
        wave_pack_reads(reads, todo, is_long ? offs[rid] : 0, lm.m, slot, lane, mv_mine, cnt);
        __syncthreads();  // the slots are written; one wave, so this orders LDS only
        if (is_long) {
            const LdsQuery q{slot[lane]};
            if (COUNT) { nsearched++; nqwords += (uint32_t)((lm.m + 31) >> 5); }
            out[rid] = match_read<kWordsInLds>(ix, nullptr, nullptr, 0, use_table, q, lm.m, mv_mine, cnt);
            cnt.touch(out + rid, 16);
        }
        __syncthreads();  // before the next chunk rewrites the slots
    }
    if constexpr (COUNT) {
        wave_add(&b.stats[3], nsearched);
        wave_add(&b.stats[4], nqwords);
        add_counts(b.stats, cnt);
    }
}

// ------------------------------------------------------------------ suffix tree

// Search of the flattened suffix tree: from the root, take the child that
// continues with the read's next base and compare the read with that
// child's first suffix from the depth already matched; stop where the read
// ends, where no child continues, or where the comparison stops inside the
// edge.  The node or leaf reached holds the rows of the matched prefix: the
// same (lo, hi, l, exact) as the suffix-array searches.
template <class Q>
__device__ __forceinline__ int4 st_match(const uint64_t *__restrict__ text, const int32_t *__restrict__ sa,
                                         int32_t n, const StNode *__restrict__ nodes, int32_t root, const Q &q,
                                         int m, int mv) {
    NoCount cnt;
    int lb = 0, rb = n, d = 0, l = 0;
    int node = root;
    const int plen = mv;
    for (;;) {
        if (d >= plen) {
            l = plen;
            break;
        }
        const int c = (int)((q[d >> 5] >> (62 - 2 * (d & 31))) & 3u);
        const int ch = nodes[node].child[c];
        if (ch == -1) {
            l = d;
            break;
        }
        int clb, crb, cdepth;
        if (ch >= 0) {
            const StNode cn = nodes[ch];
            clb = cn.lb;
            crb = cn.rb;
            cdepth = cn.depth;
        } else {
            clb = -2 - ch;
            crb = clb + 1;
            cdepth = 0;
        }
        const int32_t p = sa[clb];
        if (ch < 0) cdepth = n - p;
        int lcp;
        compare_from<kLongWords>(text, n, q, plen, p, d >> 5, lcp, cnt);
        lb = clb;
        rb = crb;
        if (ch < 0 || lcp < cdepth || plen <= cdepth) {
            l = min_i(lcp, plen);
            break;
        }
        node = ch;
        d = cdepth;
    }
    const int flags = l == m ? (int)kHitExact : 0;
    if (l == 0) return make_int4(0, n, 0, flags);
    return make_int4(lb, rb, l, flags);
}

// One wave per workgroup, 64 reads per chunk in input order: the wave packs
// each read of the chunk into LDS, then every lane walks the tree for its own.
__global__ __launch_bounds__(64) void search_st_kernel(const uint64_t *__restrict__ text,
                                                       const int32_t *__restrict__ sa, int32_t n,
                                                       const StNode *__restrict__ nodes, int32_t root,
                                                       const uint8_t *__restrict__ reads,
                                                       const int64_t *__restrict__ offs, int64_t nreads,
                                                       int4 *__restrict__ out) {
    __shared__ uint64_t slot[64][kLongWords];
    const int lane = threadIdx.x;
    NoCount cnt;
    const int64_t nchunks = (nreads + 63) >> 6;
    for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const int64_t i = (c << 6) + lane;
        const bool act = i < nreads;
        int64_t a = 0;
        int m = -1;
        if (act) {
            a = offs[i];
            const int64_t m64 = offs[i + 1] - a;
            m = (m64 >= 0 && m64 <= SA_MAX_READ) ? (int)m64 : -1;
        }
        const uint64_t todo = wave_ballot(act && m >= 0);
        int mv = m;
        wave_pack_reads(reads, todo, a, m, slot, lane, mv, cnt);
        __syncthreads();  // one wave: orders the LDS slots
        if (act) {
            if (m < 0) {
                out[i] = make_int4(0, 0, 0, (int)kHitTooLong);
            } else {
                const LdsQuery q{slot[lane]};
                out[i] = st_match(text, sa, n, nodes, root, q, m, mv);
            }
        }
        __syncthreads();  // before the next chunk rewrites the slots
    }
}

__global__ void clear_stats_kernel(BatchBuffers b) {
    if (threadIdx.x < kStatWords) b.stats[threadIdx.x] = 0ull;
}

}  // namespace

hipError_t prepare_kernels() {
    hipError_t e;
    int dev = 0, per_block = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess ||
        (e = hipDeviceGetAttribute(&per_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev)) != hipSuccess)
        return e;
    // room for the kernels' static LDS
    const size_t inline_lds = std::min(kLdsBytes, per_block > 256 ? (size_t)per_block - 256 : (size_t)0);
    const size_t tile = tile_lds_bytes(kMaxTileLevels);
    if ((e = allow_lds(search_packed_kernel<256, false>, tile)) != hipSuccess ||
        (e = allow_lds(search_packed_kernel<512, false>, tile)) != hipSuccess ||
        (e = allow_lds(search_packed_kernel<1024, false>, tile)) != hipSuccess ||
        (e = allow_lds(search_packed_kernel<256, true>, tile)) != hipSuccess ||
        (e = allow_lds(search_reads_kernel<false, false>, inline_lds)) != hipSuccess ||
        (e = allow_lds(search_reads_kernel<false, true>, inline_lds)) != hipSuccess ||
        (e = allow_lds(search_reads_kernel<true, false>, inline_lds)) != hipSuccess ||
        (e = allow_lds(search_reads_kernel<true, true>, inline_lds)) != hipSuccess)
        return e;
    g_inline_lds.store(inline_lds);
    return hipSuccess;
}

size_t inline_lds_limit() { return g_inline_lds.load(); }


hipError_t launch_search_st(const uint64_t *text, const int32_t *sa, int32_t n, const StNode *nodes, int32_t root,
                            const uint8_t *reads, const int64_t *offs, int64_t nreads, void *out, int grid,
                            hipStream_t s) {
    hipLaunchKernelGGL(search_st_kernel, dim3((unsigned)(grid > 0 ? grid : 1)), dim3(64), 0, s, text, sa, n, nodes,
                       root, reads, offs, nreads, static_cast<int4 *>(out));
    return hipGetLastError();
}

hipError_t launch_pack_text(const uint8_t *ascii, int64_t n, uint64_t *text, int64_t words,
                            unsigned long long *first_bad, hipStream_t s) {
    hipLaunchKernelGGL(pack_text_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, ascii, n, text, words,
                       first_bad);
    return hipGetLastError();
}

hipError_t launch_build_rows(const uint64_t *text, const int32_t *sa, int32_t n, RowRec *rows, hipStream_t s) {
    const int64_t blocks = ((int64_t)n + 255) / 256;
    hipLaunchKernelGGL(build_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, s, text, sa, n, rows);
    return hipGetLastError();
}

hipError_t launch_build_tile(const uint64_t *text, const int32_t *sa, int32_t n, int levels, uint64_t *key,
                             int32_t *tsa, hipStream_t s) {
    const int nodes = (1 << levels) - 1;
    hipLaunchKernelGGL(build_tile_kernel, dim3((nodes + 255) / 256), dim3(256), 0, s, text, sa, n, levels, key,
                       tsa);
    return hipGetLastError();
}

hipError_t launch_pack(const uint8_t *reads, const int64_t *offs, const int64_t *ends, int64_t nreads,
                       const BatchBuffers &b, const BucketTable &bt, hipStream_t s) {
    const int64_t blocks = (nreads + kPackBlock - 1) / kPackBlock;
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)(blocks > 0 ? blocks : 1)), dim3(kPackBlock), 0, s, reads, offs,
                       ends, nreads, b, bt);
    return hipGetLastError();
}

hipError_t launch_sort(const BatchBuffers &b, int64_t nreads, int lo_bit, int hi_bit, int *which, hipStream_t s) {
    return radix_sort_pairs<uint32_t>(b.key[0], b.val[0], b.key[1], b.val[1], b.hist, b.digit_total, nreads, lo_bit,
                                      hi_bit, which, s);
}

hipError_t launch_search_packed(const DevIndex &ix, int levels, int use_table, int block, int grid, int group,
                                const BatchBuffers &b, const uint32_t *order, int64_t nreads, void *out, bool count,
                                hipStream_t s) {
    int4 *o = static_cast<int4 *>(out);
    if (group < 1) return hipErrorInvalidValue;
    if (count)  // counts do not depend on the workgroup shape or the work split
        return launch_packed_block<256, true>(ix, levels, use_table, group, grid * (block / 256), b, order, nreads, o, s);
    switch (block) {
        case 256: return launch_packed_block<256, false>(ix, levels, use_table, group, grid, b, order, nreads, o, s);
        case 512: return launch_packed_block<512, false>(ix, levels, use_table, group, grid, b, order, nreads, o, s);
        case 1024: return launch_packed_block<1024, false>(ix, levels, use_table, group, grid, b, order, nreads, o, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_search_reads(const DevIndex &ix, int levels, int use_table, int block, int blocks_per_cu, int cus,
                               int group, int defer, unsigned long long *stats, const uint8_t *reads,
                               const int64_t *offs, const int64_t *ends, int64_t nreads, void *out, bool count,
                               hipStream_t s) {
    int4 *o = static_cast<int4 *>(out);
    if (group < 1 || block < 64 || block > 1024) return hipErrorInvalidValue;
    const size_t limit = g_inline_lds.load();
    if (inline_lds_bytes(inline_area(0), block) > limit) return hipErrorInvalidValue;
    // Without a prefix table every search starts at the root: stage the tile,
    // as deep as asked for while it does not cost a workgroup per compute
    // unit its place (MI355X, 4M reads of 100 bases on 16 Mbp in three
    // workgroups of 512 threads: 1.18 ms with 8 levels, 1.39 with 10, which
    // leave room for two).
    const bool tile = !(use_table && ix.ptab_k > 0);
    if (tile) {
        const size_t fit = std::min<size_t>((size_t)blocks_per_cu, limit / inline_lds_bytes(inline_area(0), block));
        while (levels > 1 && inline_lds_bytes(inline_area(levels), block) * fit > limit) --levels;
    }
    const InlineArea area = inline_area(tile ? levels : 0);
    const size_t lds = inline_lds_bytes(area, block);
    if (lds > limit) return hipErrorInvalidValue;
    const SearchSplit sp = search_split(nreads, cus, blocks_per_cu, block / 64, group);
#define SAMATCH_LAUNCH(C, T)                                                                                      \
    hipLaunchKernelGGL((search_reads_kernel<C, T>), dim3(sp.grid), dim3(block), lds, s, ix, levels, use_table, sp.group, \
                       sp.per, sp.chunks, defer, area, stats, reads, offs, ends, nreads, o)
    if (count) {
        if (tile) SAMATCH_LAUNCH(true, true);
        else SAMATCH_LAUNCH(true, false);
    } else {
        if (tile) SAMATCH_LAUNCH(false, true);
        else SAMATCH_LAUNCH(false, false);
    }
#undef SAMATCH_LAUNCH
    return hipGetLastError();
}

hipError_t launch_build_prefix_table(const DevIndex &ix, int k, PrefixEntry *tab, hipStream_t s) {
    // a small table in smaller groups, so that every compute unit has some
    int bases = std::min(k, kTabBases);
    while (bases > 4 && (k - bases) < 5) --bases;
    hipLaunchKernelGGL(build_prefix_table_kernel, dim3(1u << (2 * (k - bases))),
                       dim3(std::min(kTabThreads, 1 << (2 * bases))), 0, s, ix, k, bases, tab);
    return hipGetLastError();
}

hipError_t launch_search_long(const DevIndex &ix, const uint8_t *reads, const int64_t *offs, const BatchBuffers &b,
                              const uint32_t *order, const uint32_t *sorted_key, int key_shift, uint32_t key_mask,
                              uint32_t long_field, int use_table, int grid, int64_t nreads, void *out, bool count,
                              hipStream_t s) {
    int4 *o = static_cast<int4 *>(out);
    const dim3 g((unsigned)(grid > 0 ? grid : 1));
    if (count)
        hipLaunchKernelGGL(search_long_kernel<true>, g, dim3(64), 0, s, ix, reads, offs, b, order, sorted_key,
                           key_shift, key_mask, long_field, use_table, nreads, o);
    else
        hipLaunchKernelGGL(search_long_kernel<false>, g, dim3(64), 0, s, ix, reads, offs, b, order, sorted_key,
                           key_shift, key_mask, long_field, use_table, nreads, o);
    return hipGetLastError();
}

hipError_t launch_clear_stats(const BatchBuffers &b, hipStream_t s) {
    hipLaunchKernelGGL(clear_stats_kernel, dim3(1), dim3(64), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_search_plain(const DevIndex &ix, const BatchBuffers &b, int64_t nreads, void *out, bool count,
                               hipStream_t s) {
    const int64_t blocks = (nreads + 255) / 256;
    const dim3 grid((unsigned)(blocks > 0 ? blocks : 1));
    if (count)
        hipLaunchKernelGGL(search_plain_kernel<true>, grid, dim3(256), 0, s, ix, b, nreads, static_cast<int4 *>(out));
    else
        hipLaunchKernelGGL(search_plain_kernel<false>, grid, dim3(256), 0, s, ix, b, nreads, static_cast<int4 *>(out));
    return hipGetLastError();
}

}  // namespace samatch
