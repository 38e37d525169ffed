// HIP kernels of libtam for gfx950 (CDNA4, wave64).
//
// Mask compile (Section 4.1, valid[n] for every trie node n):
//   k_zero   -- zero fill of the dense table (pure streaming stores).
//   k_probe  -- one lane per non-root node m: the token strings that are suffixes
//               of prefix(m) are found from the longest one (a binary search over
//               its length in the vocabulary's suffix table); a token t of length
//               d = |t| among them is valid at the ancestor d levels up, because
//               t's walk from there ends at m.  This is the paper's crediting of a
//               match to the node |t| bytes back (Section 4.2), done for all nodes
//               at once instead of along a DFS.  It keeps which they are per
//               node, ORs them into the zeroed table with 64-bit atomics (nodes
//               with a dense row) and, for lists, counts per node (without a table
//               under tail compression, it also records each hit listed on a
//               branching node with its rank).
//   k_suf_*  -- the suffix table, once per vocabulary.
//   k_scan_* -- exclusive prefix sum of the counts into row offsets.
//   k_fill   -- writes the hits' token ids into the per-node lists;
//               k_fill_records places the recorded hits instead.
//   k_rows   -- one wave per row builds rows in registers from the lists
//               (canonical rows of handles without a dense table).
// Serving (Section 2, Eq. 1 and the extended transition function):
//   k_apply  -- write-mostly masking of [B, V] logits (lists and tail rows);
//               k_apply_dense for dense-table rows; rows of any alignment.
//   k_advance-- B byte walks along the strings of the blob and over the
//               children that leave them, one wave per row.
//   k_export_dense, k_export_tail -- canonical rows out of the dense table and
//               (tail compression) the suffixes of the nodes below.
// Rows built on demand (lazy computation with a bounded cache, Appendix):
//   k_lazy_assign -- cache lookup and CLOCK replacement for a group of rows;
//               each miss takes a zero spare row, its victim becomes a spare.
//   k_lazy_probe -- the missing rows, from the suffix probes of the node's
//               subtree only, while the victims' rows are cleared; k_apply
//               then reads the cache.
// Trie tables on the device (from the blob and one record per string):
//   k_lay_init, k_lay (positions, tail tables), k_kid_alloc, k_kid_fill (the
//   children that leave a string's own path).
// Fixed-format values (character-position masks):
//   k_format -- every word of the rows of positions 0..L+1, by wave ballots.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstring>
#include <mutex>

#include "tam_internal.hpp"
#include "trie_layout.hpp"

namespace tam {
namespace {

constexpr int kBlock = 256;
constexpr int kWave = 64;
// Apply: two chunks per thread for dense rows, three for tail rows (see k_apply_dense
// and k_apply), while that leaves this many blocks (4 per CU); with fewer, one per
// thread spreads a small batch further.  us per call, one against two or three, new
// rows in every call and, in brackets, after 1 GiB of other traffic.  Tail rows, bf16
// over V = 262,144: 8 rows (344 blocks) 3.00 and 3.30 (5.2 and 5.4), 16 rows (688) 3.79
// and 3.61 (5.7 and 6.3), 32 rows (1,376) 5.45 and 5.07 (8.6 and 7.2), 64 rows 10.4 and
// 9.3 (14.8 and 11.7); V = 32,000, 128 rows (768) 4.37 and 4.20 (5.5 and 6.2), 256 rows
// (1,536) 6.55 and 5.67 (9.6 and 7.8).  Dense rows, V = 262,144: 8 rows (512) 2.54 and
// 2.51 (5.1 and 5.0), 32 rows (2,048) 5.00 and 4.70 (7.3 and 6.0), 64 rows 8.5 and 7.7
// (12.0 and 9.4); V = 32,000, 128 rows (1,024) 3.63 and 3.43 (both 5.1).
constexpr int kDenseChunks = 2, kTailChunks = 3;
constexpr int64_t kApplyWide = 1024;
// k_apply row sources: the valid lists, or with tail compression per row the
// tail's tokens (the suffixes of the nodes below it) or the branching node's dense
// row or list
constexpr int kApplyLists = 1, kApplyTail = 2;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct DevProps {
    int cus = 0;
};

DevProps props_for_current_device() {
    static DevProps cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return DevProps{256};
    if (cache[dev].cus == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            cus <= 0)
            cus = 256;
        cache[dev].cus = cus;
    }
    return cache[dev];
}

// p[i] = value, i < n: 16-byte stores where p is 16-byte aligned.
__global__ void __launch_bounds__(kBlock) k_fill_i32(int32_t *p, int64_t n, int32_t value) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    const int64_t i0 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    int64_t done = 0;
    if ((reinterpret_cast<uintptr_t>(p) & 15) == 0) {
        const uint32_t u = (uint32_t)value;
        const u32x4 v4{u, u, u, u};
        done = n / 4;
        for (int64_t i = i0; i < done; i += stride) reinterpret_cast<u32x4 *>(p)[i] = v4;
        done *= 4;
    }
    for (int64_t i = done + i0; i < n; i += stride) p[i] = value;
}

// ---------------------------------------------------------------- probes ---

// Reversed 16-byte path window ending at blob[pos]: byte k of (lo, hi) is
// blob[pos - k].  Five aligned dword loads; the blob carries 16 zero bytes on
// both sides, so they stay inside it.
__device__ __forceinline__ void load_window(const uint8_t *blob, int64_t pos, uint64_t &lo, uint64_t &hi) {
    const int64_t ws = pos - (kWin - 1);
    const int64_t a = ws & ~int64_t(3);
    const uint32_t *w = reinterpret_cast<const uint32_t *>(blob + a);
    const uint32_t w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3], w4 = w[4];
    const uint32_t sh = (uint32_t)(ws - a) * 8u;
    const uint32_t x0 = (uint32_t)((((uint64_t)w1 << 32) | w0) >> sh);
    const uint32_t x1 = (uint32_t)((((uint64_t)w2 << 32) | w1) >> sh);
    const uint32_t x2 = (uint32_t)((((uint64_t)w3 << 32) | w2) >> sh);
    const uint32_t x3 = (uint32_t)((((uint64_t)w4 << 32) | w3) >> sh);
    lo = __builtin_bswap64(((uint64_t)x3 << 32) | x2);
    hi = __builtin_bswap64(((uint64_t)x1 << 32) | x0);
}

__device__ __forceinline__ uint32_t window_byte(uint64_t lo, uint64_t hi, int k) {
    return (uint32_t)((k < 8 ? lo >> (8 * k) : hi >> (8 * (k - 8))) & 0xffu);
}

__device__ __forceinline__ bool has_len(const DevTables &t, int d) {
    return d < 64 ? ((t.len_mask >> d) & 1ull) != 0 : t.len_present[d] != 0;
}

// The first min(d, 8) reversed bytes of a suffix of d bytes (lo) equal the slot's.
__device__ __forceinline__ bool lo_ok(uint64_t lo, const SlotPay &r, int d) {
    return (d >= 8 ? lo : (lo & (~0ull >> (64 - 8 * d)))) == r.lo;
}

// Reversed bytes 8 .. min(d, 16) - 1 of the suffix (hi) equal the slot's (d > 8).
__device__ __forceinline__ bool hi_ok(uint64_t hi, uint64_t rhi, int d) {
    return (d >= 16 ? hi : (hi & (~0ull >> (64 - 8 * (d - 8))))) == rhi;
}

__device__ __forceinline__ uint64_t home_bucket(const DevTables &t, uint64_t key) {
    return (key & t.slot_mask) / kBucket;
}

// A bucket: its kBucket fingerprints and its base, in one 16-byte load.
struct Bucket {
    u32x4 q[kBucket / 8];
};

__device__ __forceinline__ Bucket load_bucket(const DevTables &t, uint64_t b) {
    const u32x4 *p = reinterpret_cast<const u32x4 *>(t.fps + b * kBucket);
    Bucket k;
#pragma unroll
    for (int i = 0; i < kBucket / 8; ++i) k.q[i] = p[i];
    return k;
}

// The number of the bucket's first string (byte i in bits 24..31 of word i).
__device__ __forceinline__ uint32_t bucket_base(const Bucket &bk) {
    return (bk.q[0].x >> 24) | ((bk.q[0].y >> 24) << 8) | ((bk.q[0].z >> 24) << 16) | (bk.q[0].w & 0xff000000u);
}

// Bit i of *match: slot i holds fingerprint fp; bit i of *empty: slot i is empty.
__device__ __forceinline__ void bucket_masks(const Bucket &bk, uint32_t fp, uint32_t *match, uint32_t *empty) {
    uint32_t mm = 0, ee = 0;
    const uint32_t w[4] = {bk.q[0].x, bk.q[0].y, bk.q[0].z, bk.q[0].w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t a = w[i] & 0xfffu, b = (w[i] >> 12) & 0xfffu;
        mm |= ((a == fp ? 1u : 0u) | (b == fp ? 2u : 0u)) << (2 * i);
        ee |= ((a == 0u ? 1u : 0u) | (b == 0u ? 2u : 0u)) << (2 * i);
    }
    *match = mm;
    *empty = ee;
}

// The suffix of d bytes ending at blob[pos] (window (lo, hi)) equals slot s,
// whose payload m and (d > 8) pay_hi word mhi have just been read: its first 8
// reversed bytes, bytes 8..15, then (d > 16) the bytes beyond the window.
__device__ __forceinline__ bool slot_equals(const DevTables &t, const SlotPay &m, uint64_t mhi, int d, uint64_t lo,
                                            uint64_t hi, int64_t pos) {
    if ((int)m.len != d || !lo_ok(lo, m, d)) return false;
    if (d > 8 && !hi_ok(hi, mhi, d)) return false;
    if (d > kWin) {
        const uint8_t *tb = t.tok_blob + t.tok_off[m.first];
        const uint8_t *pb = t.blob + (pos - d + 1);
        for (int k = 0; k < d - kWin; ++k)
            if (tb[k] != pb[k]) return false;
    }
    return true;
}

// The hit of a suffix of d <= kShortLen bytes (last byte b0, the one before it b1).
__device__ __forceinline__ int32_t short_hit(const DevTables &t, int d, uint32_t b0, uint32_t b1) {
    return t.short_hits[short_index(d, b0, b1)];
}

// Slot (0..kBucket-1) of the first fingerprint fp in bucket bk, or -1.  The
// eight 12-bit fingerprints are compared two per word: a field of
// x = (w ^ fp:fp) & 0xffffff is zero exactly where the fingerprint matches, and
// (x - 0x001001) & ~x sets bit 11 of a zero field; a borrow out of a zero low
// field can flag the high field too, but the lowest flagged field is always a
// true match.  *open: the bucket's last slot is empty, so the bucket was never
// full and a key whose home it is lies in it (slots fill in order and are
// never cleared).
__device__ __forceinline__ int first_match(const Bucket &bk, uint32_t fp, bool *open) {
    const uint32_t fp2 = fp | (fp << 12);
    const uint32_t w[4] = {bk.q[0].x, bk.q[0].y, bk.q[0].z, bk.q[0].w};
    int s = -1;
#pragma unroll
    for (int i = 3; i >= 0; --i) {
        const uint32_t x = (w[i] ^ fp2) & 0xffffffu;
        const uint32_t z = (x - 0x001001u) & ~x & 0x800800u;
        if (z) s = 2 * i + ((z & 0x800u) ? 0 : 1);
    }
    *open = ((w[3] >> 12) & 0xfffu) == 0u;
    return s;
}

// The number of the string of d bytes that ends at blob[pos] (reversed
// window (lo, hi)), with home bucket b and fingerprint fp, or -1; its payload
// goes to *pay.  Buckets are scanned from b until one with an empty slot (load
// <= 1/4 guarantees one exists): a key sits in a later bucket only if every
// bucket before it was full when it was inserted.
__device__ __forceinline__ int32_t probe_from(const DevTables &t, uint64_t b, uint32_t fp, int d, uint64_t lo,
                                              uint64_t hi, int64_t pos, SlotPay *pay) {
    const uint64_t bmask = t.slot_mask / kBucket;
    for (;;) {
        uint32_t match, empty;
        const Bucket bk = load_bucket(t, b);
        bucket_masks(bk, fp, &match, &empty);
        const uint32_t base = bucket_base(bk);
        while (match) {
            const int i = __builtin_ctz(match);
            match &= match - 1;
            const int32_t sl = (int32_t)(base + (uint32_t)i);
            const SlotPay m = t.pay[sl];
            const uint64_t mhi = d > 8 ? t.pay_hi[sl] : 0ull;
            if (slot_equals(t, m, mhi, d, lo, hi, pos)) {
                *pay = m;
                return sl;
            }
        }
        if (empty) return -1;
        b = (b + 1) & bmask;
    }
}

// The same from the string's key (its hash).
__device__ __forceinline__ int32_t probe(const DevTables &t, uint64_t key, int d, uint64_t lo, uint64_t hi,
                                         int64_t pos, SlotPay *pay) {
    return probe_from(t, home_bucket(t, key), fingerprint(key), d, lo, hi, pos, pay);
}

// The hashed lengths are probed in two halves of kLaneLens.
constexpr int kLaneLens = (kWin - kShortLen) / 2;
static_assert(kLaneLens * 2 == kWin - kShortLen, "lengths split evenly");

// The hits (hit_of_slot, or -1) of the suffixes of length d = kD0 + 1 ..
// kD0 + kLaneLens (and, with the lower half, 1 .. kShortLen) of a window (lo,
// hi); only d <= Lw <= kWin are probed.  hit[i] is the hit of length kD0 + 1 + i
// (lower half: hit[kLaneLens + d - 1] for the short d).
// The hash state advances one byte per length, and the lengths are unrolled,
// so every byte extract and mask is a constant.  The home buckets of the
// lane's lengths are loaded together, then the payload (and for lengths beyond
// 8 bytes the pay_hi word) of each first fingerprint match, so the lane waits
// for two memory round trips.  Bit i of the returned mask marks a length its
// home bucket does not settle (a full bucket, or a failed first match): the
// caller probes it with the general probe.
template <int kD0>
__device__ __forceinline__ uint32_t probe_lengths(const DevTables &t, int Lw, uint64_t lo, uint64_t hi,
                                                  int32_t (&hit)[kLaneLens + kShortLen]) {
    if (kD0 == kShortLen) {
        hit[kLaneLens] = short_hit(t, 1, window_byte(lo, hi, 0), 0u);
        hit[kLaneLens + 1] = Lw >= 2 ? short_hit(t, 2, window_byte(lo, hi, 0), window_byte(lo, hi, 1)) : -1;
    } else {
        hit[kLaneLens] = hit[kLaneLens + 1] = -1;
    }
    uint32_t bidx[kLaneLens], fp[kLaneLens];
    bool act[kLaneLens];
    uint32_t h = kHashSeed;
#pragma unroll
    for (int k = 0; k < kD0 + kLaneLens; ++k) {
        h = hash_step(h, window_byte(lo, hi, k));
        if (k >= kD0) {
            const int j = k - kD0, d = k + 1;
            const uint64_t key = hash_final(h);
            bidx[j] = (uint32_t)home_bucket(t, key);
            fp[j] = fingerprint(key);
            act[j] = d <= Lw && has_len(t, d);
        }
    }
    Bucket bk[kLaneLens];
#pragma unroll
    for (int j = 0; j < kLaneLens; ++j)
        if (act[j]) bk[j] = load_bucket(t, bidx[j]);
    int32_t slot[kLaneLens];
    uint32_t pending = 0;
#pragma unroll
    for (int j = 0; j < kLaneLens; ++j) {
        slot[j] = -1;
        if (act[j]) {
            bool open;
            const int sl = first_match(bk[j], fp[j], &open);
            if (sl >= 0) slot[j] = (int32_t)(bucket_base(bk[j]) + (uint32_t)sl);
            if (sl >= 0 || !open) pending |= 1u << j;  // cleared below when the match holds
        }
    }
    SlotPay p[kLaneLens];
    uint64_t phi[kLaneLens];
#pragma unroll
    for (int j = 0; j < kLaneLens; ++j) {
        phi[j] = 0;
        if (slot[j] >= 0) {
            p[j] = t.pay[slot[j]];
            if (kD0 + j + 1 > 8) phi[j] = t.pay_hi[slot[j]];
        }
    }
#pragma unroll
    for (int j = 0; j < kLaneLens; ++j) {
        const int d = kD0 + j + 1;
        hit[j] = -1;
        if (slot[j] >= 0 && (int)p[j].len == d && lo_ok(lo, p[j], d) && (d <= 8 || hi_ok(hi, phi[j], d))) {
            hit[j] = hit_of_slot(slot[j], p[j].first, p[j].count);
            pending &= ~(1u << j);
        }
    }
    return pending;
}

// Writes the token ids of hit x (see hit_of_slot) into the list of node n.
__device__ __forceinline__ void emit(const DevTables &t, int32_t x, int32_t n) {
    if (x >= 0) {
        t.entries[t.row_ptr[n] + atomicAdd(&t.cursor[n], 1)] = x;
        return;
    }
    const SlotPay m = t.pay[-2 - x];
    const int32_t at = t.row_ptr[n] + atomicAdd(&t.cursor[n], (int32_t)m.count);
    int32_t v = m.first;
    for (int k = 0; k < (int)m.count; ++k) {
        t.entries[at + k] = v;
        v = t.dup_next[v];
    }
}

// Number of token ids of hit x.
__device__ __forceinline__ int32_t hit_count(const DevTables &t, int32_t x) {
    return x >= 0 ? 1 : (x == -1 ? 0 : (int32_t)t.pay[-2 - x].count);
}

// Calls f(hit, d) for every token string ending at node m longer than the
// window (d > 16), probing those lengths again (vocabularies rarely have them).
template <typename F>
__device__ __forceinline__ void long_hits(const DevTables &t, int64_t pos, int L, F &&f) {
    uint64_t lo, hi;
    load_window(t.blob, pos, lo, hi);
    uint32_t h = kHashSeed;
    for (int d = 1; d <= kWin; ++d) h = hash_step(h, window_byte(lo, hi, d - 1));
    for (int d = kWin + 1; d <= L; ++d) {
        h = hash_step(h, t.blob[pos - d + 1]);
        if (!has_len(t, d)) continue;
        SlotPay mt;
        const int32_t s = probe(t, hash_final(h), d, lo, hi, pos, &mt);
        if (s >= 0) f(hit_of_slot(s, mt.first, mt.count), d);
    }
}

// The group of probe block b in the groups' grid (0 without groups), and an
// entry of a group array: block-uniform selects, so that the kernel argument is
// never indexed dynamically (which would copy it to scratch memory).
__device__ __forceinline__ int group_of(const RecGroups &rg, int64_t b) {
    return (rg.n > 1 && b >= rg.blk0[1]) + (rg.n > 2 && b >= rg.blk0[2]) + (rg.n > 3 && b >= rg.blk0[3]);
}
template <typename T>
__device__ __forceinline__ T pick(const T (&a)[kMaxRecGroups], int k) {
    return k == 0 ? a[0] : k == 1 ? a[1] : k == 2 ? a[2] : a[3];
}
template <typename T>
__device__ __forceinline__ T pick(const T (&a)[kMaxRecGroups + 1], int k) {
    return k == 0 ? a[0] : k == 1 ? a[1] : k == 2 ? a[2] : a[3];
}

// Hits at distance d <= list_span(m) above node m belong to the valid lists:
// all of them with lists only, the tail ancestors of m with tail compression
// (where the lists hold only tokens longer than the window).
__device__ __forceinline__ int list_span(const DevTables &t, int64_t m) {
    if (t.tail_span) return t.tail_span[m];
    return t.table ? 0 : INT_MAX;
}

// The bits of the lengths 1 .. d (of at most kWin).
__device__ __forceinline__ uint32_t lengths_to(int d) {
    return d >= kWin ? (1u << kWin) - 1u : d <= 0 ? 0u : (1u << d) - 1u;
}

// The hit of length k + 1 in the list of a mask with bit k set.
__device__ __forceinline__ int32_t suf_hit(const DevTables &t, uint32_t off, uint32_t mask, int k) {
    return t.suf_ids[off + __popc(mask & ((1u << k) - 1u))];
}

__device__ __forceinline__ u32x4 suf_bucket(const DevTables &t, uint32_t b) {
    return reinterpret_cast<const u32x4 *>(t.suf_fps)[b];
}

// The first min(len, 16) reversed bytes of a window equal an entry's of length d.
__device__ __forceinline__ bool suf_equal(const SufPay &p, int d, uint64_t lo, uint64_t hi) {
    const uint64_t ml = d >= 8 ? ~0ull : ~0ull >> (64 - 8 * d);
    const uint64_t mh = d >= 16 ? ~0ull : d <= 8 ? 0ull : ~0ull >> (64 - 8 * (d - 8));
    return (int)p.len == d && (lo & ml) == p.lo && (hi & mh) == p.hi;
}

// Bits of the slots whose fingerprint is fp: slot s at bit (s & 3) + 16 * (s >> 2).
__device__ __forceinline__ uint32_t suf_match(u32x4 q, uint32_t fp) {
    const uint32_t fp2 = fp | (fp << 16);
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t x = (q[k] ^ fp2) & 0x7fff7fffu;
        m |= (~(x + 0x7fff7fffu) & 0x80008000u) >> (15 - k);  // a half of x is 0
    }
    return m;
}

__device__ __forceinline__ int32_t suf_entry(uint32_t bucket, int bit) {
    return (int32_t)(bucket * kSufSlots + (uint32_t)((bit & 3) | ((bit >> 4) << 2)));
}

// The number of the entry that equals the window's last d bytes, whose hash
// state is h, or -1: every fingerprint match compared, on to the next bucket
// while keys were moved there.
__device__ __forceinline__ int32_t suf_find(const DevTables &t, uint32_t h, int d, uint64_t lo, uint64_t hi) {
    const uint64_t key = hash_final(h);
    const uint32_t fp = suf_fingerprint(key);
    for (uint32_t b = suf_home(key, t.suf_buckets);; b = b + 1 == t.suf_buckets ? 0 : b + 1) {
        const u32x4 q = suf_bucket(t, b);
        for (uint32_t m = suf_match(q, fp); m; m &= m - 1) {
            const int32_t n = suf_entry(b, __builtin_ctz(m));
            if (suf_equal(t.suf_pay[n], d, lo, hi)) return n;
        }
        if (!(q.w & kSufOver)) return -1;
    }
}

// The search with every step compared (suf_search's rare way out).
__device__ __forceinline__ int32_t suf_search_exact(const DevTables &t, int Lw, uint64_t lo, uint64_t hi) {
    int a = kShortLen, b = kWin + 1;
    int32_t best = -1;
    while (b - a > 1) {
        const int mid = (a + b) / 2;
        int32_t n = -1;
        if (mid <= Lw) {
            uint32_t h = kHashSeed;
            for (int k = 0; k < mid; ++k) h = hash_step(h, window_byte(lo, hi, k));
            n = suf_find(t, h, mid, lo, hi);
        }
        if (n >= 0) {
            best = n;
            a = mid;
        } else {
            b = mid;
        }
    }
    return best;
}

// The token strings that are suffixes of the window's last Lw bytes (1 <= Lw <=
// kWin).  Four dependent probes of one 16-byte load each, taken on the
// fingerprint alone; only the last one that matched is compared: if it holds,
// every shorter one on the way does (they are its token's markers), and a miss
// needs no comparison.  A false match repeats the search with comparisons (1 node
// in 5,000).
__device__ __forceinline__ SufRef suf_search(const DevTables &t, int Lw, uint64_t lo, uint64_t hi) {
    uint32_t hs[kWin + 1];
    uint32_t h = kHashSeed;
#pragma unroll
    for (int k = 1; k <= kWin; ++k) {
        h = hash_step(h, window_byte(lo, hi, k - 1));
        hs[k] = h;
    }
    int32_t best = -1;
    int best_d = 0;
    auto look = [&](int d, uint32_t state) {
        if (d > Lw) return false;
        const uint64_t key = hash_final(state);
        const uint32_t fp = suf_fingerprint(key);
        uint32_t b = suf_home(key, t.suf_buckets);
        u32x4 q = suf_bucket(t, b);
        uint32_t m = suf_match(q, fp);
        while (m == 0 && (q.w & kSufOver)) {  // keys moved on from here (1 bucket in 200)
            b = b + 1 == t.suf_buckets ? 0 : b + 1;
            q = suf_bucket(t, b);
            m = suf_match(q, fp);
        }
        if (m == 0) return false;
        best = suf_entry(b, __builtin_ctz(m));
        best_d = d;
        return true;
    };
    const bool p1 = look(9, hs[9]);
    const bool p2 = look(p1 ? 13 : 5, p1 ? hs[13] : hs[5]);
    const int d3 = p1 ? (p2 ? 15 : 11) : (p2 ? 7 : 3);
    const bool p3 = look(d3, p1 ? (p2 ? hs[15] : hs[11]) : (p2 ? hs[7] : hs[3]));
    const int d4 = p3 ? d3 + 1 : d3 - 1;
    if (d4 > kShortLen) {
        const uint32_t up = p1 ? (p2 ? hs[16] : hs[12]) : (p2 ? hs[8] : hs[4]);
        const uint32_t dn = p1 ? (p2 ? hs[14] : hs[10]) : hs[6];
        look(d4, p3 ? up : dn);
    }
    SufPay pay{};
    if (best >= 0) {
        pay = t.suf_pay[best];
        if (!suf_equal(pay, best_d, lo, hi)) {
            best = suf_search_exact(t, Lw, lo, hi);
            if (best >= 0) pay = t.suf_pay[best];
        }
    }
    if (best >= 0) return SufRef{pay.off, pay.mask, pay.total, 0};
    return t.suf_short[Lw >= 2 ? short_index(2, window_byte(lo, hi, 0), window_byte(lo, hi, 1))
                               : short_index(1, window_byte(lo, hi, 0), 0u)];
}

// Groups a wave's lanes of `in` by the value x: a lane's group's first lane,
// the group's lanes before it, and its size.
__device__ __forceinline__ void wave_groups(int32_t x, uint64_t in, int lane, int *lead, int32_t *before,
                                            int32_t *size) {
    *lead = lane;
    *before = 0;
    *size = 0;
    while (in) {
        const int f = __builtin_ctzll(in);
        const uint64_t same = __ballot(x == __builtin_amdgcn_readlane(x, f)) & in;
        in &= ~same;
        if ((same >> lane) & 1u) {
            *lead = f;
            *before = __popcll(same & ((1ull << lane) - 1));
            *size = __popcll(same);
        }
    }
}

// Probe pass: one lane per node m.  A token t of length d that is a suffix of
// prefix(m) is valid at the ancestor d levels up, node_at[pos - d].  All those of
// up to kWin bytes come from one search for the longest (suf_search) and are kept
// as that entry's list and mask (node_suf), 8 bytes per node; the tails of tail
// compression read their tokens back from there.  Longer tokens are probed where
// needed (long_hits).
// Bound by the search's chain of five dependent loads (the waves wait for 0.77 of
// their time) and its VALU work (816 instructions per wave with records, 689 with
// marks); L2 hit rate 0.87.  Probing every length on its own took 14 bucket loads,
// 4.5 payloads and 64 bytes of hits per node, and every listed hit an atomic of its
// own on the few ancestors that neighbouring nodes share: over a forest of 5.5 M
// nodes 653 us and 1,482 MB read, now 207 us and 547 MB, 37 M L2 requests (370 us
// with the searches alone).
//   do_mark (a table): every hit whose ancestor has a dense row (row_at of its
//     blob position; not a tail) is OR-ed into the zeroed table with a 64-bit
//     atomic, and each block writes the number of valid (node, token) pairs its
//     hits make, tails included, into pairs[blockIdx.x].
//   kCount (lists): the listed hits are counted per node: every hit (lists
//     only); with tail compression and a table, the tails' hits of tokens
//     longer than the window; with tail compression and no table (tail_lists),
//     also every hit on a branching node, and each block then writes its
//     number of valid pairs as do_mark does.
// The grid covers the nodes [m0, m1): every node of the handle, or (lists of a
// forest) one group of whole sets, whose nodes' ancestors are in the group too.
// With tail compression and no table the groups' grid (rg) decides instead:
// this launch runs its probe blocks blk + blockIdx.x.
// kRecords (tail lists) shares the hits out over the block; the others take them
// length by length, unrolled.
template <bool kCount, bool kRecords>
__global__ void __launch_bounds__(kBlock, 8) k_probe(DevTables t, int64_t m0, int64_t m1, int do_mark,
                                                     int32_t *__restrict__ pairs, RecGroups rg, int64_t blk) {
    const int64_t gb = blk + blockIdx.x;  // the block in the grid of pairs (and rec_cnt)
    const int gk = kRecords ? group_of(rg, gb) : 0;
    if (kRecords) {
        m0 = pick(rg.n_lo, gk) + (gb - pick(rg.blk0, gk)) * kBlock;
        m1 = pick(rg.n_hi, gk);
    } else {
        m0 += (int64_t)blockIdx.x * kBlock;
    }
    const int64_t m = m0 + threadIdx.x;
    const int lane = threadIdx.x & (kWave - 1);
    // records: the listed hits of the block, (thread, length - 1) each, and what
    // their threads found
    __shared__ uint16_t s_item[kRecords ? kBlock * kWin : 1];
    __shared__ uint32_t s_off[kRecords ? kBlock : 1], s_mask[kRecords ? kBlock : 1];
    __shared__ int32_t s_pos[kRecords ? kBlock : 1];
    __shared__ int32_t s_n;  // hits, then records left
    if (kRecords) {
        if (threadIdx.x == 0) s_n = 0;
        __syncthreads();
    }
    int32_t found = 0;
    int L = 0, lspan = 0, mspan = INT_MAX;
    // what streams through is loaded and stored past the L2's tables
    const int64_t pos = m < m1 ? __builtin_nontemporal_load(t.node_pos + m) : -1;  // a root ends no token
    unsigned long long *suf_out = reinterpret_cast<unsigned long long *>(t.node_suf + m);
    if (m < m1 && pos < 0) __builtin_nontemporal_store(0ull, suf_out);
    unsigned long long *table = reinterpret_cast<unsigned long long *>(t.table);
    auto mark = [&](int32_t hx, int32_t row) {
        if (row < 0) return;
        if (hx >= 0) {
            atomicOr(table + (int64_t)row * t.Wp + (hx >> 6), 1ull << (hx & 63));
            return;
        }
        const SlotPay mt = t.pay[-2 - hx];  // a string with several token ids (rare)
        int32_t v = mt.first;
        for (int k = 0; k < (int)mt.count; ++k) {
            atomicOr(table + (int64_t)row * t.Wp + (v >> 6), 1ull << (v & 63));
            v = t.dup_next[v];
        }
    };
    if (pos >= 0) {
        L = min(__builtin_nontemporal_load(t.depth + m), t.max_len);
        const int Lw = min(L, kWin);
        lspan = kCount ? list_span(t, m) : 0;  // listed up to here
        if (do_mark) mspan = t.tail_span ? t.tail_span[m] : 0;  // marked beyond
        SufRef r{0, 0, 0, 0};
        if (Lw > 0) {
            uint64_t lo, hi;
            load_window(t.blob, pos, lo, hi);
            r = suf_search(t, Lw, lo, hi);
        }
        __builtin_nontemporal_store((unsigned long long)r.off | ((unsigned long long)r.mask << 32), suf_out);
        found = r.total;
        if (kRecords) {  // on the branching ancestors, beyond the tails
            uint32_t todo = r.mask & ~lengths_to(lspan);
            if (todo) {
                s_off[threadIdx.x] = r.off;
                s_mask[threadIdx.x] = r.mask;
                s_pos[threadIdx.x] = (int32_t)pos;
                int32_t at = atomicAdd(&s_n, __popc(todo));
                for (; todo; todo &= todo - 1) s_item[at++] = (uint16_t)(threadIdx.x << 4 | __builtin_ctz(todo));
            }
        } else {
            // One length after another and unrolled, so that the loads of all come
            // before the first atomic, and the lanes of an atomic have different
            // ancestors (those of consecutive nodes are consecutive).
            const uint32_t todo = do_mark ? r.mask & ~lengths_to(mspan)
                                          : kCount && !t.row_of ? r.mask & lengths_to(lspan) : 0u;
            const int32_t *owner = do_mark ? t.row_at : t.node_at;
            const bool one_each = r.total == __popc(r.mask);  // no string with several ids
            constexpr int H = kWin / 2;
#pragma unroll
            for (int h = 0; h < kWin; h += H) {
                if (!__any((todo >> h) & ((1u << H) - 1u))) continue;
                int32_t hx[H], to[H];
#pragma unroll
                for (int j = 0; j < H; ++j) {
                    const bool on = (todo >> (h + j)) & 1u;
                    hx[j] = on && (do_mark || !one_each) ? suf_hit(t, r.off, r.mask, h + j) : 0;
                    to[j] = on ? owner[pos - h - j - 1] : -1;
                }
#pragma unroll
                for (int j = 0; j < H; ++j) {
                    if (!((todo >> (h + j)) & 1u)) continue;
                    if (!kCount || do_mark)
                        mark(hx[j], to[j]);
                    else
                        atomicAdd(&t.count[to[j]], hit_count(t, hx[j]));
                }
            }
        }
    }
    int32_t *rec = nullptr;
    int32_t reg0 = 0, reg1 = 0;
    // record i of the block: a hit listed at node ln with its rank in the list
    auto put = [&](int32_t hx, int32_t ln, int32_t rank, int32_t i) {
        const int64_t at = (int64_t)reg0 + i;
        if (at >= reg1) {  // more records than the host's bound
            atomicAdd(t.err, 1);
            return;
        }
        rec[3 * at] = ln;
        rec[3 * at + 1] = rank;
        rec[3 * at + 2] = hx;
    };
    if (kRecords) {
        // Only nodes near a branch have listed hits, a few lanes of a wave, and
        // neighbouring nodes' hits land on the same few ancestors.  So the block's
        // threads share the hits out, and a wave counts those of one list node with
        // one atomic (atomics on one address follow one another): over a forest of
        // 5.4 M nodes 222 us for the pass, 370 with an atomic each, 382 with a
        // loop over each lane's own hits; over 1,000 word strings 49.6 against 59.1 us
        // per step with an atomic each.
        __syncthreads();
        const int32_t items = s_n;
        const int64_t o = pick(rg.off0, gk) + (gb - pick(rg.blk0, gk));
        rec = pick(rg.rec, gk);
        reg0 = t.rec_off[o];
        reg1 = t.rec_off[o + 1];
        for (int32_t i0 = 0; i0 < items; i0 += kBlock) {  // uniform over the block
            const int32_t i = i0 + threadIdx.x;
            const bool in = i < items;
            int32_t hx = -1, ln = -1, c = 0;
            if (in) {
                const int l = s_item[i] >> 4, k = s_item[i] & 15;
                hx = suf_hit(t, s_off[l], s_mask[l], k);
                ln = t.node_at[s_pos[l] - k - 1];
                c = hit_count(t, hx);
            }
            int32_t rank = 0;
            if (__any(c > 1)) {  // a string with several ids among them (rare)
                if (in) rank = atomicAdd(&t.count[ln], c);
            } else {
                int lead;
                int32_t before, sum;
                wave_groups(ln, __ballot(in), lane, &lead, &before, &sum);
                if (in && lead == lane) rank = atomicAdd(&t.count[ln], sum);
                rank = __shfl(rank, lead, kWave) + before;
            }
            if (in) put(hx, ln, rank, i);
        }
    }
    // tokens longer than the window (rare), after the shared hits' records
    if (t.max_len > kWin) {  // uniform over the grid
        if (kRecords) __syncthreads();
        if (L > kWin && (do_mark || lspan > kWin || kRecords))
            long_hits(t, pos, L, [&](int32_t hx, int d) {
                const int32_t c = hit_count(t, hx);
                found += c;
                if (d > mspan) mark(hx, t.row_at[pos - d]);
                if (kRecords) {
                    const int32_t ln = t.node_at[pos - d], rank = atomicAdd(&t.count[ln], c);
                    put(hx, ln, rank, atomicAdd(&s_n, 1));
                } else if (d <= lspan) {
                    atomicAdd(&t.count[t.node_at[pos - d]], c);
                }
            });
    }
    if (!do_mark && !kRecords) return;
    // block sum of the pairs
    __shared__ int32_t wsum[kBlock / kWave];
    for (int o = kWave / 2; o > 0; o >>= 1) found += __shfl_xor(found, o, kWave);
    if (lane == 0) wsum[threadIdx.x / kWave] = found;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t total = 0;
        for (int w = 0; w < kBlock / kWave; ++w) total += wsum[w];
        pairs[gb] = total;
        if (kRecords) t.rec_cnt[gb] = s_n;
    }
}

// Threads per probe block's records: one record per thread in a few rounds also
// where most hits are listed (a forest of small word sets, about 1,000 per block: with
// one wave 6 us more per rebuild).
constexpr int kFillThreads = 256;

// The records of probe block blockIdx.x of the groups' grid (tail compression
// without a table): each listed hit's ids go to its node's list at
// row_ptr[node] + rank.
__global__ void __launch_bounds__(kFillThreads) k_fill_records(DevTables t, RecGroups rg) {
    const int64_t b = blockIdx.x;
    const int gk = group_of(rg, b);
    const int64_t o = pick(rg.off0, gk) + (b - pick(rg.blk0, gk));
    const int64_t r0 = t.rec_off[o];
    const int32_t n = min(t.rec_cnt[b], t.rec_off[o + 1] - t.rec_off[o]);
    const int32_t *rec = pick(rg.rec, gk);
    for (int32_t i = threadIdx.x; i < n; i += kFillThreads) {
        const int32_t *r = rec + 3 * (r0 + i);
        const int32_t ln = r[0], rank = r[1], hx = r[2];
        const int64_t at = (int64_t)t.row_ptr[ln] + rank;
        if (hx >= 0) {
            t.entries[at] = hx;
            continue;
        }
        const SlotPay pm = t.pay[-2 - hx];  // a string with several token ids
        int32_t v = pm.first;
        for (int k = 0; k < (int)pm.count; ++k) {
            t.entries[at + k] = v;
            v = t.dup_next[v];
        }
    }
}

// Fill pass (lists): the hits' token ids written into the per-node lists (with
// tail compression those of tokens longer than the window, and without a
// table also those on branching nodes).
__global__ void __launch_bounds__(kBlock) k_fill(DevTables t) {
    const int64_t m = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (m >= t.N) return;
    const int64_t pos = t.node_pos[m];
    if (pos < 0) return;
    const int L = min(t.depth[m], t.max_len);
    const int Lw = min(L, kWin);
    const int span = list_span(t, m);
    const int Ls = t.row_of ? 0 : min(Lw, span);  // tail compression lists long hits only
    const int bspan = t.tail_lists ? t.tail_span[m] : INT_MAX;  // no table: branching nodes' hits too
    const NodeSuf r = t.node_suf[m];
    const uint32_t todo = r.mask & (lengths_to(Ls) | ~lengths_to(bspan));
    int32_t s[kWin], to[kWin];
#pragma unroll
    for (int k = 0; k < kWin; ++k) {
        const bool on = (todo >> k) & 1u;
        s[k] = on ? suf_hit(t, r.off, r.mask, k) : -1;
        to[k] = on ? t.node_at[pos - k - 1] : -1;
    }
    // the places of all (one returning atomic each) before the first store
    int32_t at[kWin];
#pragma unroll
    for (int k = 0; k < kWin; ++k)
        if (s[k] >= 0) at[k] = t.row_ptr[to[k]] + atomicAdd(&t.cursor[to[k]], 1);
#pragma unroll
    for (int k = 0; k < kWin; ++k)
        if (s[k] >= 0) t.entries[at[k]] = s[k];
    if (t.suf_dups)  // strings with several ids
        for (uint32_t left = todo; left; left &= left - 1) {
            const int k = __builtin_ctz(left);
            const int32_t x = suf_hit(t, r.off, r.mask, k);
            if (x < -1) emit(t, x, t.node_at[pos - k - 1]);
        }
    if (L > kWin && (span > kWin || t.tail_lists))
        long_hits(t, pos, L, [&](int32_t hx, int d) {
            if (d <= span || t.tail_lists) emit(t, hx, t.node_at[pos - d]);
        });
}

// Zero fill of n16 16-byte chunks: one chunk per thread, 256 threads (4 KiB)
// per block, plain stores and no grid-stride loop.  Measured on MI355X this
// shape sustains ~6.8 TB/s; more chunks per thread, non-temporal stores or a
// persistent grid-stride grid all write slower, because the blocks in flight
// then no longer sweep one compact window of memory.
__global__ void __launch_bounds__(kBlock) k_zero(u32x4 *__restrict__ p, int64_t n16) {
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c < n16) p[c] = u32x4{0u, 0u, 0u, 0u};
}

// ------------------------------------------------------------------ scan ---

constexpr int kScanItems = 16;
constexpr int kScanTile = kBlock * kScanItems;  // elements per block

// Exclusive scan of one value per thread over the 256-thread block.
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t x, int32_t *total) {
    __shared__ int32_t wave_sums[kBlock / kWave];
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    int32_t inc = x;
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t y = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += y;
    }
    if (lane == kWave - 1) wave_sums[wid] = inc;
    __syncthreads();
    int32_t before = 0, all = 0;
    for (int w = 0; w < kBlock / kWave; ++w) {
        if (w < wid) before += wave_sums[w];
        all += wave_sums[w];
    }
    __syncthreads();
    *total = all;
    return before + inc - x;
}

// A thread's kScanItems consecutive values from base (0 past n): four 16-byte
// loads where the whole run is in range and aligned.
__device__ __forceinline__ void scan_load(const int32_t *in, int64_t base, int64_t n, int32_t (&v)[kScanItems]) {
    if (base + kScanItems <= n && (reinterpret_cast<uintptr_t>(in + base) & 15) == 0) {
#pragma unroll
        for (int q = 0; q < kScanItems / 4; ++q) {
            const u32x4 x = reinterpret_cast<const u32x4 *>(in + base)[q];
            v[4 * q] = (int32_t)x.x;
            v[4 * q + 1] = (int32_t)x.y;
            v[4 * q + 2] = (int32_t)x.z;
            v[4 * q + 3] = (int32_t)x.w;
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) v[k] = base + k < n ? in[base + k] : 0;
}

__global__ void __launch_bounds__(kBlock) k_scan_blocks(const int32_t *in, int64_t n, int32_t *sums) {
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int32_t v[kScanItems];
    scan_load(in, base, n, v);
    int32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) s += v[k];
    int32_t total;
    block_exclusive_scan(s, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// One block: exclusive scan of the nb block sums in place; grand total -> *total_out.
// (Used when the block sums are more than one block of the apply pass adds up.)
__global__ void __launch_bounds__(kBlock) k_scan_top(int32_t *sums, int64_t nb, int32_t *total_out) {
    int32_t carry = 0;
    for (int64_t base = 0; base < nb; base += kScanTile) {
        const int64_t b0 = base + (int64_t)threadIdx.x * kScanItems;
        int32_t v[kScanItems];
        int32_t s = 0;
        for (int k = 0; k < kScanItems; ++k) {
            v[k] = b0 + k < nb ? sums[b0 + k] : 0;
            s += v[k];
        }
        int32_t total;
        int32_t run = carry + block_exclusive_scan(s, &total);
        for (int k = 0; k < kScanItems; ++k) {
            if (b0 + k < nb) sums[b0 + k] = run;
            run += v[k];
        }
        carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total_out = carry;
}

// The scan's second pass, by how a block learns the sum before its own:
// kScanSelf (few blocks: the only pass) reads the counts themselves; kScanOwn (nb
// <= kScanTile) adds up the block sums before its own (at most kScanTile of them,
// from L2); kScanTop takes it from k_scan_top's prefixes.  Without k_scan_top the
// last block writes the grand total.  zero (or null): n values set to 0.
constexpr int kScanTop = 0, kScanOwn = 1, kScanSelf = 2;
// Counting again costs a block 16 KB of reads per block before it, a launch about
// 3 us: up to eight blocks (32,768 nodes) the first pass is left out (rebuild, apply
// and advance over 1,300 nodes with lists, with the cursors cleared here too: 47.7
// -> 44.4 us).
constexpr int64_t kScanSelfBlocks = 8;
__global__ void __launch_bounds__(kBlock) k_scan_apply(const int32_t *in, int64_t n, const int32_t *sums,
                                                       int how, int32_t *out, int32_t *total_out, int32_t *zero) {
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int32_t v[kScanItems];
    scan_load(in, base, n, v);
    int32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) s += v[k];
    int32_t prefix, total;
    if (how == kScanTop) {
        prefix = sums[blockIdx.x];
    } else {
        int32_t p = 0;
        if (how == kScanSelf) {
            for (int64_t b = 0; b < (int64_t)blockIdx.x; ++b) {
                int32_t w[kScanItems];
                scan_load(in, b * kScanTile + (int64_t)threadIdx.x * kScanItems, n, w);
#pragma unroll
                for (int k = 0; k < kScanItems; ++k) p += w[k];
            }
        } else {
            for (int64_t j = threadIdx.x; j < (int64_t)blockIdx.x; j += kBlock) p += sums[j];
        }
        block_exclusive_scan(p, &prefix);
    }
    if (zero)
        for (int64_t i = (int64_t)blockIdx.x * kScanTile + threadIdx.x;
             i < min(n, ((int64_t)blockIdx.x + 1) * kScanTile); i += kBlock)
            zero[i] = 0;
    int32_t run = prefix + block_exclusive_scan(s, &total);
    if (how != kScanTop && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total_out = prefix + total;
    int32_t o[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        o[k] = run;
        run += v[k];
    }
    if (base + kScanItems <= n && (reinterpret_cast<uintptr_t>(out + base) & 15) == 0) {
#pragma unroll
        for (int q = 0; q < kScanItems / 4; ++q)
            reinterpret_cast<u32x4 *>(out + base)[q] =
                u32x4{(uint32_t)o[4 * q], (uint32_t)o[4 * q + 1], (uint32_t)o[4 * q + 2], (uint32_t)o[4 * q + 3]};
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k)
            if (base + k < n) out[base + k] = o[k];
    }
}

// --------------------------------------------------------- suffix table ---

// Built once per vocabulary, after its hash is on the device (see SufPay).

// The scratch set and counts, zero.
__global__ void __launch_bounds__(kBlock) k_suf_init(SufBuild b) {
    const int64_t stride = (int64_t)gridDim.x * kBlock, i0 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    for (int64_t i = i0; i < b.set_slots; i += stride) b.set[i] = 0;
    for (int64_t i = i0; i < b.buckets; i += stride) {
        b.cnt[i] = 0;
        reinterpret_cast<u32x4 *>(b.fps)[i] = u32x4{0u, 0u, 0u, 0u};
    }
    if (i0 == 0) *b.counter = 0;
}

// Every token string's token suffixes of at most kWin bytes (itself included):
// their lengths, their hits in ascending length, and the ids those stand for.  The
// strings of one and two bytes also write their places in the short table.
__global__ void __launch_bounds__(kBlock) k_suf_lists(DevTables t, SufBuild b) {
    const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    SlotPay p{0, -1, 0, 0};
    if (q < b.strings) p = t.pay[q];
    const bool in = p.first >= 0 && (int)p.len <= kWin;
    const uint64_t lo = p.lo, hi = in ? t.pay_hi[q] : 0ull;
    int32_t hit[kWin];  // by length - 1
#pragma unroll
    for (int k = 0; k < kWin; ++k) hit[k] = -1;
    uint32_t mask = 0;
    if (in) {
        const int L = p.len;
        int32_t h0[kLaneLens + kShortLen], h1[kLaneLens + kShortLen];
        const uint32_t p0 = probe_lengths<kShortLen>(t, L, lo, hi, h0);
        const uint32_t p1 = probe_lengths<kShortLen + kLaneLens>(t, L, lo, hi, h1);
#pragma unroll
        for (int k = 0; k < kShortLen; ++k) hit[k] = h0[kLaneLens + k];
#pragma unroll
        for (int k = 0; k < kLaneLens; ++k) {
            hit[kShortLen + k] = h0[k];
            hit[kShortLen + kLaneLens + k] = h1[k];
        }
#pragma unroll
        for (int k = 0; k < kWin; ++k) {
            const int j = k - kShortLen;
            const bool open = j >= 0 && (((j < kLaneLens ? p0 >> j : p1 >> (j - kLaneLens)) & 1u) != 0);
            if (open) {  // the home bucket did not settle it (rare)
                uint32_t hh = kHashSeed;
                for (int i = 0; i <= k; ++i) hh = hash_step(hh, window_byte(lo, hi, i));
                SlotPay mt;
                const int32_t sl = probe(t, hash_final(hh), k + 1, lo, hi, 0, &mt);
                hit[k] = sl >= 0 ? hit_of_slot(sl, mt.first, mt.count) : -1;
            }
            if (hit[k] != -1) mask |= 1u << k;
        }
    }
    int32_t total;
    const int32_t at = block_exclusive_scan(__popc(mask), &total);
    __shared__ int32_t base;
    if (threadIdx.x == 0) base = total ? atomicAdd(b.counter, total) : 0;
    __syncthreads();
    if (q >= b.strings) return;
    const uint32_t off = (uint32_t)(base + at);
    int32_t ids = 0, n = 0;
#pragma unroll
    for (int k = 0; k < kWin; ++k)
        if (hit[k] != -1) {
            b.id_list[off + n++] = hit[k];
            ids += hit_count(t, hit[k]);
        }
    b.str_off[q] = off;
    b.str_mask[q] = mask;
    b.str_total[q] = ids;
    if (in && (int)p.len <= kShortLen && p.len > 0)
        b.shrt[short_index(p.len, window_byte(lo, hi, 0), window_byte(lo, hi, 1))] = SufRef{off, mask, ids, 0};
}

// The rest of the short table: two bytes that are no token have the last byte's
// suffixes; a byte that is no token has none.
__global__ void __launch_bounds__(kBlock) k_suf_short(DevTables t, SufBuild b) {
    const int i = (int)(blockIdx.x * kBlock + threadIdx.x);
    if (i >= kShortEntries || t.short_hits[i] != -1) return;
    const int last = i < 256 ? i : (i - 256) & 0xff;
    b.shrt[i] = i >= 256 && t.short_hits[last] != -1 ? b.shrt[last] : SufRef{0, 0, 0, 0};
}

// A slot of the scratch set: bits 0..3 the entry's length - 1, bits 4..35 one more
// than the string it is a suffix of (0: empty slot), then, once it has its place
// in the table, bits 36..38 its slot and 39..63 how many buckets past its home.
constexpr int kSetSlotBit = 36, kSetMoveBit = 39;

// The entries: every token string of more than kShortLen bytes and its markers,
// each distinct one once (the set compares bytes), one thread per string and
// step of its path.  Bound by its atomics on random lines (83 us for the 1.6 M of
// 262,144 tokens).  The thread that enters it takes its slot in the table: from its home bucket on, the first bucket that
// has not been asked for kSufSlots slots before.
__global__ void __launch_bounds__(kBlock) k_suf_insert(DevTables t, SufBuild b) {
    const int64_t id = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t q = id >> 2;
    if (q >= b.strings) return;
    const SlotPay p = t.pay[q];
    if (p.first < 0 || (int)p.len <= kShortLen || (int)p.len > kWin) return;
    int at[4];
    const int steps = suf_path(p.len, at), j = (int)(id & 3);
    if (j >= steps) return;
    const int d = j == 0 ? at[0] : j == 1 ? at[1] : j == 2 ? at[2] : at[3];
    const uint64_t ml = d >= 8 ? ~0ull : ~0ull >> (64 - 8 * d);
    const uint64_t mh = d >= 16 ? ~0ull : d <= 8 ? 0ull : ~0ull >> (64 - 8 * (d - 8));
    const uint64_t lo = p.lo & ml, hi = t.pay_hi[q] & mh;
    uint32_t h = kHashSeed;
    for (int k = 0; k < d; ++k) h = hash_step(h, window_byte(lo, hi, k));
    const uint64_t key = hash_final(h);
    const unsigned long long code = ((unsigned long long)(q + 1) << 4) | (unsigned)(d - 1);
    const uint64_t smask = (uint64_t)b.set_slots - 1;
    // the set is at most half full, so the walk over it ends
    for (uint64_t i = (key * 0x9e3779b97f4a7c15ull >> 20) & smask;; i = (i + 1) & smask) {
        unsigned long long *slot = reinterpret_cast<unsigned long long *>(b.set + i);
        const unsigned long long old = atomicCAS(slot, 0ull, code);
        if (old == 0) {
            uint32_t bk = suf_home(key, (uint32_t)b.buckets), moved = 0;
            int32_t n;
            // the table has more slots than entries, so a bucket is found
            while ((n = atomicAdd(&b.cnt[bk], 1)) >= kSufSlots) {
                bk = bk + 1 == (uint32_t)b.buckets ? 0 : bk + 1;
                ++moved;
            }
            atomicOr(slot, ((unsigned long long)n << kSetSlotBit) | ((unsigned long long)moved << kSetMoveBit));
            return;
        }
        if ((int)(old & 15) == d - 1) {
            const int64_t o = (int64_t)((old >> 4) & 0xffffffffull) - 1;
            if (((t.pay[o].lo ^ lo) & ml) == 0 && ((t.pay_hi[o] ^ hi) & mh) == 0) return;
        }
    }
}

// The entries' fingerprints and payloads.
__global__ void __launch_bounds__(kBlock) k_suf_fill(DevTables t, SufBuild b) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const uint64_t x = i < b.set_slots ? b.set[i] : 0;
    if (x == 0) return;
    const int d = (int)(x & 15) + 1;
    const int64_t q = (int64_t)((x >> 4) & 0xffffffffull) - 1;
    const uint32_t n = (uint32_t)(x >> kSetSlotBit) & 7u;
    const uint64_t moved = x >> kSetMoveBit;
    const uint64_t ml = d >= 8 ? ~0ull : ~0ull >> (64 - 8 * d);
    const uint64_t mh = d >= 16 ? ~0ull : d <= 8 ? 0ull : ~0ull >> (64 - 8 * (d - 8));
    SufPay e{};
    e.lo = t.pay[q].lo & ml;
    e.hi = t.pay_hi[q] & mh;
    uint32_t h = kHashSeed;
    for (int k = 0; k < d; ++k) h = hash_step(h, window_byte(e.lo, e.hi, k));
    const uint64_t key = hash_final(h);
    const int64_t bk = (int64_t)((suf_home(key, (uint32_t)b.buckets) + moved) % (uint64_t)b.buckets);
    const uint32_t all = b.str_mask[q];
    e.off = b.str_off[q];
    e.mask = (uint16_t)(all & lengths_to(d));
    e.len = (uint16_t)d;
    e.total = __popc((uint32_t)e.mask);
    if (b.str_total[q] != __popc(all)) {  // strings with several ids among them
        e.total = 0;
        for (int k = 0; k < __popc((uint32_t)e.mask); ++k) e.total += hit_count(t, b.id_list[e.off + k]);
    }
    b.pay[bk * kSufSlots + n] = e;
    // slot 7 is taken wherever a key moved on, so its owner says so
    const uint32_t over = n == kSufSlots - 1 && b.cnt[bk] > kSufSlots ? kSufOver >> 16 : 0u;
    reinterpret_cast<uint16_t *>(b.fps)[8 * bk + 2 * (n & 3) + (n >> 2)] = (uint16_t)(suf_fingerprint(key) | over);
}

// ------------------------------------------------------------ row images ---

constexpr int kRowSlots = 8;       // chunks per lane per pass
constexpr int kRowRegBatches = 4;  // 64-entry batches of a row's list held in VGPRs

// One wave per row (grid-stride over rows): the row's list (up to 256 ids) is
// loaded into VGPRs once; each pass then builds 8 chunks per lane in registers
// from it and streams them with non-temporal stores, 64 chunks (1 KiB for
// 16-byte chunks) per store instruction.  No LDS, no barriers: every wave keeps
// a whole row of stores in flight.  Row r is node nodes[r] (r if nodes is
// null), written at out + r*out_stride; a dead or out-of-range node gives a
// zero row.  CW = 64-bit words per chunk (2: 16-byte stores, 1: 8-byte).
template <int CW>
__global__ void __launch_bounds__(kBlock) k_rows(const int32_t *__restrict__ row_ptr,
                                                 const int32_t *__restrict__ entries,
                                                 const int32_t *__restrict__ nodes, int64_t nrows, int64_t N,
                                                 uint64_t *__restrict__ out, int64_t out_stride,
                                                 int64_t out_words) {
    typedef uint32_t chunk_t __attribute__((ext_vector_type(2 * CW)));
    constexpr int kBits = 64 * CW;             // tokens per chunk
    constexpr int kPass = kWave * kRowSlots;   // chunks per pass
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t nwaves = (int64_t)gridDim.x * (kBlock / kWave);
    const int64_t nchunks = out_words / CW;
    for (int64_t r = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave; r < nrows; r += nwaves) {
        const int64_t n = nodes ? (int64_t)nodes[r] : r;
        int32_t b = 0, e = 0;
        if (n >= 0 && n < N) {
            b = row_ptr[n];
            e = row_ptr[n + 1];
        }
        int32_t ent[kRowRegBatches];
#pragma unroll
        for (int i = 0; i < kRowRegBatches; ++i) {
            const int32_t k = b + i * kWave + lane;
            ent[i] = k < e ? entries[k] : 0;
        }
        const int32_t E = e - b;
        chunk_t *dst = reinterpret_cast<chunk_t *>(out + r * out_stride);
        for (int64_t c0 = 0; c0 < nchunks; c0 += kPass) {
            chunk_t val[kRowSlots];
#pragma unroll
            for (int k = 0; k < kRowSlots; ++k) val[k] = chunk_t(0u);
            for (int32_t j = 0; j < E; ++j) {
                int32_t v;
                if (j < kRowRegBatches * kWave) {
                    const int bi = j / kWave;
                    const int32_t src = bi == 0 ? ent[0] : bi == 1 ? ent[1] : bi == 2 ? ent[2] : ent[3];
                    v = __builtin_amdgcn_readlane(src, j % kWave);
                } else {
                    v = entries[b + j];
                }
                const int64_t rel = (int64_t)(v / kBits) - c0;
                if (rel < 0 || rel >= kPass) continue;
                const int k = (int)(rel / kWave), l = (int)(rel % kWave);
                const int dw = (v / 32) % (2 * CW);
                const uint32_t bit = lane == l ? 1u << (v % 32) : 0u;
#pragma unroll
                for (int kk = 0; kk < kRowSlots; ++kk) {
                    if (kk == k) {
#pragma unroll
                        for (int q = 0; q < 2 * CW; ++q)
                            if (q == dw) val[kk][q] |= bit;
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < kRowSlots; ++k) {
                const int64_t c = c0 + k * kWave + lane;
                if (c < nchunks) __builtin_nontemporal_store(val[k], dst + c);
            }
        }
    }
}

// ----------------------------------------------------------------- apply ---

template <typename T>
struct NegInf;
template <>
struct NegInf<uint16_t> {
    static constexpr uint16_t bits = 0xFF80u;
};
template <>
struct NegInf<uint32_t> {
    static constexpr uint32_t bits = 0xFF800000u;
};

// The E mask bits of chunk c of a row shifted by a elements (see row_shift),
// from dense table row trow: the bits of the tokens c E - a .. c E - a + E - 1,
// 0 for tokens below 0 (bits of tokens >= V are 0 in the table, and bytes past
// the row are not read).
template <int E>
__device__ __forceinline__ uint32_t table_bits(const DevTables &t, int64_t trow, int64_t c, int a) {
    const uint8_t *mrow = reinterpret_cast<const uint8_t *>(t.table + trow * t.Wp);
    constexpr uint32_t FULL = (1u << E) - 1u;
    const int64_t i0 = c * E - a;
    if (a == 0) return E == 8 ? (uint32_t)mrow[c] : ((uint32_t)mrow[c >> 1] >> ((c & 1) * 4)) & FULL;
    const int64_t k0 = i0 >> 3, k1 = (i0 + E - 1) >> 3;  // one byte or two neighbours
    const uint32_t x0 = k0 >= 0 ? mrow[k0] : 0u;
    const uint32_t x1 = k1 != k0 && k1 < t.Wp * 8 ? mrow[k1] : 0u;
    return ((x0 | (x1 << 8)) >> (i0 & 7)) & FULL;
}

// One token id per lane (rel = id minus the first element of the block's span;
// >= kSpan: none or outside): each thread sets the bits of its own chunks.  The
// ids inside the span are few, so a ballot keeps only those.
template <int E, int U>
__device__ __forceinline__ void take_ids(uint32_t rel, uint32_t (&bits)[U]) {
    constexpr int kSpan = kBlock * U * E;
    uint64_t in_span = __ballot(rel < (uint32_t)kSpan);
    while (in_span) {
        const int j = __builtin_ctzll(in_span);
        in_span &= in_span - 1;
        const uint32_t r = (uint32_t)__builtin_amdgcn_readlane((int)rel, j);
        const uint32_t lc = r / E;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (lc == (uint32_t)(u * kBlock + threadIdx.x)) bits[u] |= 1u << (r % E);
    }
}

// The same for one id held by the whole wave.
template <int E, int U>
__device__ __forceinline__ void set_id(uint32_t rel, uint32_t (&bits)[U]) {
    constexpr int kSpan = kBlock * U * E;
    if (rel >= (uint32_t)kSpan) return;
    const uint32_t lc = rel / E;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (lc == (uint32_t)(u * kBlock + threadIdx.x)) bits[u] |= 1u << (rel % E);
}

// A chunk is 16 bytes of logits memory (E = 8 bf16 or 4 fp32 elements).  A row
// whose base is `a` elements past a 16-byte boundary (a = 0 when the logits and
// their row stride are 16-byte aligned; an odd vocabulary with contiguous rows
// gives every a) has its chunks shifted by a: chunk c holds the elements c E - a
// .. c E - a + E - 1, and only the row's first and last chunk may be partial.
// So every row, aligned or not, is written in whole 16-byte stores; going
// element by element instead, a decode step (apply + advance) of 64 unaligned
// fp32 rows over V = 128,255 took 23.7 us against 12.9 us this way.
template <typename T>
__device__ __forceinline__ int row_shift(const T *row) {
    return (int)((reinterpret_cast<uintptr_t>(row) & 15) / sizeof(T));
}

// -inf into the elements of a partial chunk [e0, e0 + E) inside [0, V) whose
// bit in bu is 0.  kAligned: e0 >= 0, only the row's end can cut a chunk.
template <typename T, bool kAligned>
__device__ __forceinline__ void mask_partial(T *row, int64_t e0, int64_t V, uint32_t bu) {
    constexpr int E = 16 / (int)sizeof(T);
    const int lim = (int)min<int64_t>(E, V - e0);
    for (int i = kAligned || e0 >= 0 ? 0 : (int)-e0; i < lim; ++i)
        if (!((bu >> i) & 1u)) row[e0 + i] = NegInf<T>::bits;
}

template <typename T>
__device__ __forceinline__ uint32_t neg_word() {
    return sizeof(T) == 2 ? 0xFF80FF80u : 0xFF800000u;
}

// A chunk with -inf in place of the elements whose bit in bu is 0.
template <typename T>
__device__ __forceinline__ u32x4 merge_chunk(u32x4 x, uint32_t bu) {
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (sizeof(T) == 2) {
            const uint32_t two = bu >> (2 * i);
            const uint32_t keep = ((two & 1u) ? 0x0000ffffu : 0u) | ((two & 2u) ? 0xffff0000u : 0u);
            o[i] = (x[i] & keep) | (0xFF80FF80u & ~keep);
        } else {
            o[i] = (bu >> i) & 1u ? x[i] : 0xFF800000u;
        }
    }
    return o;
}

// Chunk [e0, e0 + E) lies inside the row.
template <bool kAligned, int E>
__device__ __forceinline__ bool whole_chunk(int64_t e0, int64_t V) {
    return (kAligned || e0 >= 0) && e0 + E <= V;
}

// List and tail rows.  Grid: x = groups of kBlock*U chunks of one row, y = batch
// row.  Thread i of a block owns chunks c0 + u*kBlock + i, so every store
// instruction covers 4 KiB per block contiguously.  A block's life is the
// dependent loads in front of its stores (node id; row_of with the suffixes of
// the nodes below; their ids; for lists the bounds, then the ids), so a thread
// needs several 16-byte stores for the chip's waves to reach the memory's rate.
// Tail rows, 256 logits rows over V = 262,144, with 1 / 2 / 3 / 4 / 6 chunks per thread,
// us per call.  After 1 GiB of other traffic, as a first pass or a decode behind a
// model's forward meets them (every row's tables come from HBM, and each further
// round of blocks waits for them again): anywhere in a code list 50.0 / 38.6 / 34.8 /
// 31.8 / 28.8, over a forest's decode 51.9 / 40.6 / 36.2 / 34.3 / 31.2, fp32 93 / 68 / 61 / 56 /
// 51.  One call after another on rows that the caches still hold, with two to six:
// 24.6 / 24.9 / 27.6 / 26.4, 26.5 / 26.2 / 29.1 / 27.6, fp32 46.5 / 48.7 / 49.1 / 50.7.  New rows with
// nothing in between: 32.5 / 24.3 / 24.3 / 28.3.  Three is near the best in the caches and 10%
// better than two out of them.
// Plain lists are at the memory's rate with one (25.5 against 26.6 us per step with
// two).
// Write-mostly: a chunk without a valid token is written and not read; a fully
// valid chunk is skipped; a mixed chunk of a tail or branching row is read and
// merged, and stored by the same instruction as the empty ones, so that a 128-byte line holding both is written
// whole (-inf stores into its invalid elements only, without the read, wrote such
// lines in parts: 10,000 word strings from the root 32.0 -> 30.5 us per step, a
// forest 26.9 -> 26.6).  The bits of the block's span come from the
// node's valid list (a ballot over a short list, an LDS bitmap for a long one),
// from the suffixes of the nodes below a tail, or (kApplyTail) from the dense row of a branching node.
// kAligned: every row's base is 16-byte aligned (no shift; computing it all the
// same costs 1-2% of a forest's or a code list's decode step, as does unrolling
// mask_partial).
template <typename T, int kMode, int U, bool kAligned>
__global__ void __launch_bounds__(kBlock) k_apply(DevTables t, const int32_t *__restrict__ node_ids,
                                                  T *__restrict__ logits, int64_t stride) {
    constexpr int E = 16 / (int)sizeof(T);
    constexpr uint32_t FULL = (1u << E) - 1u;
    constexpr int kSpan = kBlock * U * E;  // elements per block
    __shared__ uint32_t bm[kSpan / 32];

    const int64_t V = t.V;
    const int64_t b = blockIdx.y;
    const int32_t n = node_ids[b];
    const bool live = n >= 0 && (int64_t)n < t.N;
    const int64_t c0 = (int64_t)blockIdx.x * kBlock * U;
    T *row = logits + b * stride;
    const int a = kAligned ? 0 : row_shift(row);
    const int64_t nchunks = (V + a + E - 1) / E;
    // the row's source (uniform over the block): its dense table row, its list,
    // or (a tail with tail compression) the suffixes of the nodes on its path
    const int lane = threadIdx.x & (kWave - 1);
    // With tail compression most rows are tails: the suffixes of the nodes on the
    // path below n are loaded together with row_of[n] (lane d-1: those of node
    // n+d, one line for all), and kept only if n turns out to be a tail.
    NodeSuf below{0, 0};
    if (kMode == kApplyTail && live && lane < kWin && lane < t.max_len && (int64_t)n + lane + 1 < t.N)
        below = t.node_suf[n + lane + 1];
    int64_t trow = live ? n : -1;
    if (kMode == kApplyTail && live) trow = t.row_of[n];
    const bool tail_row = kMode == kApplyTail && live && trow < 0;
    // lists: every row; tail compression without a table: the branching rows
    const bool use_list = kMode == kApplyLists || (kMode == kApplyTail && !tail_row && t.table == nullptr);

    uint32_t bits[U];
#pragma unroll
    for (int u = 0; u < U; ++u) bits[u] = 0;
    const uint32_t lo = (uint32_t)(c0 * E - a);  // first element of the span (wraps below 0 in the first one)
    if (tail_row) {
        // lane d-1 takes the token of length d that ends at node n+d, if there is
        // one (the path below a tail has consecutive ids)
        const int Lt = min(min(-1 - (int)trow, kWin), (int)t.max_len);
        const int32_t x = lane < Lt && ((below.mask >> lane) & 1u) ? suf_hit(t, below.off, below.mask, lane) : -1;
        take_ids<E, U>(x >= 0 ? (uint32_t)x - lo : 0xffffffffu, bits);
        // strings with several token ids (rare): walk their id chains
        uint64_t multi = __ballot(x <= -2);
        while (multi) {
            const int j = __builtin_ctzll(multi);
            multi &= multi - 1;
            const SlotPay pm = t.pay[-2 - __builtin_amdgcn_readlane(x, j)];
            int32_t v = pm.first;
            for (int k = 0; k < (int)pm.count; ++k) {
                set_id<E, U>((uint32_t)v - lo, bits);
                v = t.dup_next[v];
            }
        }
        // tokens longer than the window: the tail's list (without such tokens always
        // empty; reading its bounds all the same is one more dependent load in front
        // of the stores: anywhere in a forest 27.9 -> 26.7 us per step)
        if ((t.tail_long || t.tail_lists) && t.max_len > kWin) {
            const int32_t e0 = t.row_ptr[n], e1 = t.row_ptr[n + 1];
            const int32_t *ids = t.entries + e0;  // positions as below
            const uint32_t cnt = (uint32_t)(e1 - e0);
            for (uint32_t k0 = 0; k0 < cnt; k0 += kWave) {
                const uint32_t rel = k0 + lane < cnt ? (uint32_t)ids[k0 + lane] - lo : 0xffffffffu;
                take_ids<E, U>(rel, bits);
            }
        }
    } else if (use_list) {
        const int32_t e0 = live ? t.row_ptr[n] : 0, e1 = live ? t.row_ptr[n + 1] : 0;
        if (e1 - e0 <= kWave) {
            // short list (block-uniform branch): every wave reads the ids into its
            // lanes, keeps those inside the block's span (a ballot), and each thread
            // picks the bits of its own chunks from the few that remain
            take_ids<E, U>(lane < e1 - e0 ? (uint32_t)t.entries[e0 + lane] - lo : 0xffffffffu, bits);
        } else {
            // long list: scatter through an LDS bitmap of the block's span
            constexpr int kIds = 4;
            for (int i = threadIdx.x; i < kSpan / 32; i += kBlock) bm[i] = 0;
            __syncthreads();
            // (four ids per thread loaded together: the roots of a forest 26.1 -> 25.4
            // us per call with two chunks per thread, of 10,000 word strings 31.1 -> 30.0)
            // Positions are counted from the list's start and unsigned: e0 + 1,023 more
            // than a position may exceed 2^31 - 1 at the end of the largest lists.
            const int32_t *ids = t.entries + e0;
            const uint32_t cnt = (uint32_t)(e1 - e0);
            for (uint32_t k0 = threadIdx.x; k0 < cnt; k0 += kIds * kBlock) {
                uint32_t v[kIds];
#pragma unroll
                for (int i = 0; i < kIds; ++i)
                    v[i] = k0 + i * kBlock < cnt ? (uint32_t)ids[k0 + i * kBlock] - lo : 0xffffffffu;
#pragma unroll
                for (int i = 0; i < kIds; ++i)
                    if (v[i] < (uint32_t)kSpan) atomicOr(&bm[v[i] >> 5], 1u << (v[i] & 31));
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t bit = (uint32_t)((u * kBlock + threadIdx.x) * E);
                bits[u] = (bm[bit >> 5] >> (bit & 31)) & FULL;
            }
        }
    } else if (trow >= 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t c = c0 + u * kBlock + threadIdx.x;
            if (c < nchunks) bits[u] = table_bits<E>(t, trow, c, a);
        }
    }

#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t c = c0 + u * kBlock + threadIdx.x;
        if (c >= nchunks) break;
        const uint32_t bu = bits[u];
        if (bu == FULL) continue;
        const int64_t e0 = c * E - a;
        if (whole_chunk<kAligned, E>(e0, V)) {
            u32x4 *p = reinterpret_cast<u32x4 *>(row + e0);
            const uint32_t w = neg_word<T>();
            if (kMode == kApplyLists && bu != 0) {
                // a plain list's row: -inf into the invalid elements only, no read
                // (its chain of loads is the longest already: 23.0 against 27.2 us
                // per call over a forest)
                uint32_t *q = reinterpret_cast<uint32_t *>(p);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (sizeof(T) == 2) {
                        const uint32_t two = (bu >> (2 * i)) & 3u;
                        if (two == 0)
                            q[i] = w;
                        else if (two != 3u)
                            row[e0 + 2 * i + (two == 1u ? 1 : 0)] = NegInf<T>::bits;
                    } else if (!((bu >> i) & 1u)) {
                        q[i] = w;
                    }
                }
                continue;
            }
            u32x4 o{w, w, w, w};
            if (bu != 0) o = merge_chunk<T>(*p, bu);
            __builtin_nontemporal_store(o, p);
        } else {
            mask_partial<T, kAligned>(row, e0, V, bu);
        }
    }
}

// Dense-table rows: block (x, y) takes chunks x * kBlock * U .. of row y, U per
// thread.  The mask bytes are loaded first, then the logits of the mixed chunks,
// then everything is stored, the merged chunks and the empty ones in one
// instruction: a 128-byte line of both is then written whole, where two stores
// in the two arms of a branch wrote it in two parts (256 bf16 rows decoding over
// V = 151,936: 28.0 -> 27.6 us per step; anywhere in a table of V = 262,144 rows:
// 28.2 -> 27.5 us).
// A block's life is the dependent loads in front of its stores (node id, mask
// byte, logits), so it is worth two chunks per thread once the batch fills the
// chip (kApplyWide): the former three rows of one chunk each kept as many
// loads in flight but swept three windows of the logits at once (28.4 us per
// step, 3.1 against 2.9 TB/s over a decode from the root); three chunks take 30.0,
// four 31.5 us per step.
// kAligned: every row's base is 16-byte aligned (no shift).
template <typename T, int U, bool kAligned>
__global__ void __launch_bounds__(kBlock) k_apply_dense(DevTables t, const int32_t *__restrict__ node_ids,
                                                        T *__restrict__ logits, int64_t stride) {
    constexpr int E = 16 / (int)sizeof(T);
    constexpr uint32_t FULL = (1u << E) - 1u;
    const int64_t V = t.V;
    const int64_t b = blockIdx.y;
    const int64_t c0 = (int64_t)blockIdx.x * kBlock * U + threadIdx.x;
    T *row = logits + b * stride;
    const int a = kAligned ? 0 : row_shift(row);
    const int64_t nchunks = (V + a + E - 1) / E;
    const int32_t n = node_ids[b];
    const bool live = n >= 0 && (int64_t)n < t.N;
    uint32_t bits[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t c = c0 + u * kBlock;
        bits[u] = 0;  // a dead row: every token invalid
        if (live && c < nchunks) bits[u] = table_bits<E>(t, n, c, a);
    }
    u32x4 xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t c = c0 + u * kBlock, e0 = c * E - a;
        if (c < nchunks && whole_chunk<kAligned, E>(e0, V) && bits[u] != 0 && bits[u] != FULL)
            xv[u] = *reinterpret_cast<const u32x4 *>(row + e0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t c = c0 + u * kBlock, e0 = c * E - a;
        const uint32_t bu = bits[u];
        if (c >= nchunks || bu == FULL) continue;
        if (whole_chunk<kAligned, E>(e0, V)) {
            const uint32_t w = neg_word<T>();
            u32x4 o{w, w, w, w};
            if (bu != 0) o = merge_chunk<T>(xv[u], bu);
            __builtin_nontemporal_store(o, reinterpret_cast<u32x4 *>(row + e0));
        } else {
            mask_partial<T, kAligned>(row, e0, V, bu);
        }
    }
}

// ------------------------------------------------ node positions, children ---

// The trie's position tables and children, built on the device from the uploaded
// blob and one record per string (lay_string).  The nodes a string creates have
// consecutive ids along consecutive positions, and each string but its set's
// first adds exactly one child that leaves an earlier string's path, so the
// children kept are one entry per string instead of one per node.

__global__ void __launch_bounds__(kBlock) k_lay_init(int32_t *node_at, int64_t blob_bytes, int32_t *kid_cnt,
                                                     int32_t *count, int64_t N, int32_t *err, int32_t *kid_total) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < N) kid_cnt[i] = 0;
    if (i < N && count) count[i] = 0;
    if (i < kBlobPad) node_at[i] = node_at[blob_bytes - kBlobPad + i] = 0;
    if (i == 0) *err = *kid_total = 0;
}

// One wave per string record of [u0, s1) of the group that begins at s0; a record
// that does not fit the tables is counted in *err.  One thread per string wrote
// each table with 64 separate lines per store and walked its characters one after
// another, and the tables took six kernels (positions and tail tables, first
// positions by an atomicMin): 37 us for 500 strings of 60 bytes against 5.8 us, 61
// us for 32,000 strings of a forest against 31 us.
// A launch has fewer than 2^32 threads, so 2^26 waves, and a set may have more
// strings: a launch takes kLayStrings of them.  (Waves striding over the strings
// instead: 25 us more for 500 strings.)
constexpr int64_t kLayStrings = 1 << 18;
static_assert(kLayStrings * kWave < (int64_t(1) << 32), "threads of a launch");
__global__ void __launch_bounds__(kBlock) k_lay(const StrRec *__restrict__ strs, const TailRec *__restrict__ trec,
                                                int64_t s0, int64_t u0, int64_t s1, int64_t blob_bytes, int64_t N,
                                                LayTables o, int32_t *kid_cnt, int32_t *__restrict__ kid_parent,
                                                int32_t *__restrict__ kid_rank, int32_t *err) {
    const int64_t u = u0 + ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (u >= s1) return;  // uniform over the wave
    int32_t par;
    const int32_t bad = lay_string(strs, trec, s0, u, blob_bytes, N, o, lane, kWave, &par);
    if (lane != 0) return;
    if (bad) atomicAdd(err, bad);
    kid_parent[u] = par;  // a node of [0, N), or -1
    if (par >= 0) kid_rank[u] = atomicAdd(&kid_cnt[par], 1);
}

// The ranges of the entries: the first string counted at a parent takes them, one
// atomic per block.
__global__ void __launch_bounds__(kBlock) k_kid_alloc(int64_t K, Walk *walk, const int32_t *__restrict__ kid_cnt,
                                                      const int32_t *__restrict__ kid_parent,
                                                      const int32_t *__restrict__ kid_rank, int32_t *kid_total) {
    const int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int32_t par = u < K ? kid_parent[u] : -1;
    const bool lead = par >= 0 && kid_rank[u] == 0;
    const int32_t n = lead ? kid_cnt[par] : 0;
    const uint32_t byte = lead ? walk[par].nb : 0u;
    int32_t total;
    const int32_t at = block_exclusive_scan(n, &total);
    __shared__ int32_t base;
    if (threadIdx.x == 0) base = total ? atomicAdd(kid_total, total) : 0;
    __syncthreads();
    if (lead) walk[par] = Walk{base + at, byte | ((uint32_t)n << 8)};
}

// Every string's child into its parent's range; the order inside a range is
// free: a lookup matches the child byte.
__global__ void __launch_bounds__(kBlock) k_kid_fill(const StrRec *__restrict__ strs, int64_t K,
                                                     const Walk *__restrict__ walk, Kid *__restrict__ kid,
                                                     const int32_t *__restrict__ kid_parent,
                                                     const int32_t *__restrict__ kid_rank, int32_t *err) {
    const int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int32_t par = u < K ? kid_parent[u] : -1;
    if (par < 0) return;
    const int32_t c = strs[u].first;
    const int64_t at = (int64_t)walk[par].off + kid_rank[u];
    if (at < 0 || at >= K) {
        atomicAdd(err, 1);
        return;
    }
    const Walk w = walk[c];
    kid[at] = Kid{c, w.off, w.nb, 0};
}

__global__ void __launch_bounds__(kBlock) k_tok_heads(const uint32_t *__restrict__ tok_off,
                                                      const uint8_t *__restrict__ tok_blob, int64_t V,
                                                      TokHead *__restrict__ head) {
    const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (v >= V) return;
    const uint32_t o = tok_off[v], len = tok_off[v + 1] - o;
    TokHead h;
#pragma unroll
    for (int k = 0; k < kHeadLen; ++k) h.b[k] = k < (int)len ? tok_blob[o + k] : 0;
    h.b[15] = len <= (uint32_t)kHeadLen ? (uint8_t)len : 255;
    head[v] = h;
}

// ------------------------------------------------- fixed-format strings ---

// Token bytes tb[0..len) at position p of a fixed format: non-empty, within
// the L + 1 characters (the last being the terminator), every byte in its
// position's class.
__device__ __forceinline__ bool format_fits(const DevTables &t, int p, const uint8_t *tb, int len) {
    const int L = t.fmt_L;
    if (len <= 0 || p < 0 || p + len > L + 1) return false;
    for (int i = 0; i < len; ++i) {
        const int q = p + i;
        const uint32_t c = tb[i];
        const bool in = q == L ? c == (uint32_t)t.terminator
                               : ((t.classes[(int64_t)q * 32 + (c >> 3)] >> (c & 7)) & 1u) != 0;
        if (!in) return false;
    }
    return true;
}

// The positions q = 64 k .. 64 k + 63 whose class admits byte c (position L: the
// terminator alone; past it none), bit q - 64 k each.
__device__ __forceinline__ uint64_t class_word(const DevTables &t, int64_t k, uint32_t c) {
    uint64_t x = 0;
    const int64_t q0 = 64 * k;
    const int n = (int)min<int64_t>(64, (int64_t)t.fmt_L - q0);
#pragma unroll 4
    for (int j = 0; j < n; ++j)
        x |= (uint64_t)((t.classes[(q0 + j) * 32 + (c >> 3)] >> (c & 7)) & 1u) << j;
    const int64_t e = (int64_t)t.fmt_L - q0;  // the terminator's position
    if (e >= 0 && e < 64 && c == (uint32_t)t.terminator) x |= 1ull << e;
    return x;
}

// Character-position masks (Appendix, Constraint-Aware Dispatch Beyond Finite
// Sets), written whole: one wave per 64-token word w of every row, 64 positions
// at a time.  LDS holds for every byte the set of positions whose class admits
// it, so lane i finds all positions of a window where token 64 w + i fits with one
// AND per token byte (that set shifted down by the byte's index); the wave's
// ballot over bit j is word w of the window's row j, kept by lane j and stored at
// out[row * stride + w], so no zero fill is needed, and words past V come out
// zero.  Testing every position byte by byte instead was bound by those serial
// checks: a 36-character format over V = 262,144 took 41.5 us, this way 8.7 us.
// The valid (position, token) pairs are counted: per block into
// pairs[blockIdx.x], and/or added to *total.
__global__ void __launch_bounds__(kBlock) k_format(DevTables t, uint64_t *__restrict__ out, int64_t stride,
                                                   int64_t nwords, int32_t *__restrict__ pairs,
                                                   unsigned long long *total) {
    __shared__ uint64_t cls[2][256];  // the window's class words, and the next window's
    static_assert(kBlock == 256, "one thread per byte value");
    const int64_t w = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t v = w * kWave + lane;
    int32_t found = 0;
    int len = 0;
    uint32_t o = 0;
    if (w < nwords && v < t.V) {
        o = t.tok_off[v];
        len = (int)(t.tok_off[v + 1] - o);
    }
    // the token's bytes from i on, eight at a time (three aligned dwords; the
    // token blob is padded)
    auto bytes8 = [&](int i) {
        const uint32_t at = o + (uint32_t)i;
        const uint32_t *q = reinterpret_cast<const uint32_t *>(t.tok_blob + (at & ~3u));
        const uint32_t sh = (at & 3u) * 8u;
        const uint32_t q0 = q[0], q1 = q[1], q2 = q[2];
        return (uint64_t)(uint32_t)((((uint64_t)q1 << 32) | q0) >> sh) |
               ((uint64_t)(uint32_t)((((uint64_t)q2 << 32) | q1) >> sh) << 32);
    };
    const uint64_t head = len > 0 ? bytes8(0) : 0;
    const int64_t rows = (int64_t)t.fmt_L + 2, nwin = (rows + 63) / 64;
    cls[1][threadIdx.x] = class_word(t, 0, threadIdx.x);
    for (int64_t k = 0; k < nwin; ++k) {
        const uint64_t here = cls[1][threadIdx.x];
        const uint64_t next = k + 1 < nwin ? class_word(t, k + 1, threadIdx.x) : 0;
        __syncthreads();  // the last window's reads are done
        cls[0][threadIdx.x] = here;
        cls[1][threadIdx.x] = next;
        __syncthreads();
        if (w >= nwords) continue;  // uniform over the wave
        uint64_t m = len > 0 ? ~0ull : 0;  // bit j: the token fits at position 64 k + j so far
        if (len <= 64) {
            uint64_t x = head;
            for (int i = 0; __any(i < len && m != 0); ++i) {
                if (i >= len || m == 0) continue;
                if (i > 0 && (i & 7) == 0) x = bytes8(i);
                const uint32_t c = (uint32_t)(x >> (8 * (i & 7))) & 0xffu;
                m &= (cls[0][c] >> i) | (i ? cls[1][c] << (64 - i) : 0);
            }
        } else {  // a token longer than a window (rare): position by position
            m = 0;
            for (int j = 0; j < 64; ++j)
                if (64 * k + j < rows && format_fits(t, (int)(64 * k + j), t.tok_blob + o, len)) m |= 1ull << j;
        }
        found += __popcll(m);
        const int n = (int)min<int64_t>(64, rows - 64 * k);
        uint64_t mine = 0;
        if (__any(m != 0)) {
            for (int j = 0; j < n; ++j) {
                const uint64_t word = __ballot((m >> j) & 1u);
                if (lane == j) mine = word;
            }
        }
        if (lane < n) out[(64 * k + lane) * stride + w] = mine;
    }
    __shared__ int32_t wsum[kBlock / kWave];
    for (int o2 = kWave / 2; o2 > 0; o2 >>= 1) found += __shfl_xor(found, o2, kWave);
    if (lane == 0) wsum[threadIdx.x / kWave] = found;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t sum = 0;
        for (int k = 0; k < kBlock / kWave; ++k) sum += wsum[k];
        if (pairs) pairs[blockIdx.x] = sum;
        if (total && sum) atomicAdd(total, (unsigned long long)sum);
    }
}

// --------------------------------------------------------------- advance ---

// The extended transition function, one wave per batch row.  The walk follows
// the string that created the current node n, whose nodes have consecutive ids:
// lane j >= 1 compares the edge byte of node n + j with the token's next j-th
// byte, and has that node's other children beside it (Walk).  So a token along one
// string ends after its first window, its node known without a further load, and
// where the token leaves the string the children there are known: one round trip
// for their entries (a ballot picks the byte), one for the next window, which
// also loads the entries of the child's own children, so that a token that
// leaves again at once (near the root of a large set) takes one trip per branch.
// The run may include the string's terminator but never goes past it (the node
// after T has no children).
// Bound by these dependent trips (cold lines after a large apply): the ids; the
// token's head with the first window; then the branches.  With every child
// listed, and the child ranges by position, node ids, child bytes and token bytes
// behind offsets in tables of their own, a token took five trips and three per
// branch.  256 rows decoding from the root of 10,000 word strings: 10.1 -> 7.0 us
// per call; over a forest 5.6 -> 4.6 us, anywhere in a code list 4.7 -> 4.3 us.
__global__ void __launch_bounds__(kBlock) k_advance(DevTables t, const int32_t *nodes, const int32_t *toks,
                                                    int64_t B, int32_t *out) {
    const int64_t b = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (b >= B) return;  // uniform over the wave
    const int32_t n0 = nodes[b];
    const int32_t v = toks[b];
    int32_t n = TAM_DEAD;
    const bool ok = n0 >= 0 && (int64_t)n0 < t.N && v >= 0 && (int64_t)v < t.V;
    if (t.fmt_L >= 0) {  // character positions: p + |t| when the token fits the classes
        if (ok && lane == 0) {
            const uint32_t o = t.tok_off[v];
            const int len = (int)(t.tok_off[v + 1] - o);
            if (format_fits(t, n0, t.tok_blob + o, len)) n = n0 + len;
        }
        if (lane == 0) out[b] = n;
        return;
    }
    if (ok) {
        // lane j: byte j of the token's head, and node n0 + j for the longest token
        // a head holds
        const uint32_t hb = t.tok_head[v].b[lane & 15];
        Walk w{0, 0x200u};
        if (lane <= kHeadLen && (int64_t)n0 + lane < t.N) w = t.walk[n0 + lane];
        const uint32_t T = (uint32_t)t.terminator;
        int len = (int)__shfl(hb, 15, kWave);
        int64_t a = 0;
        const bool shrt = len <= kHeadLen;
        if (!shrt) {
            a = t.tok_off[v];
            len = (int)(t.tok_off[v + 1] - (uint32_t)a);
        }
        // lanes past kHeadLen of the first window of a longer token count as a
        // mismatch there: the walk then loads the next window instead of branching
        int width = kHeadLen + 1;  // lanes the window covers
        int i = 0;                 // token bytes walked
        Kid e{TAM_DEAD, 0, 0x100u, 0};  // lane j: entry j of n's other children, when held
        bool held = false;
        n = len > 0 ? n0 : TAM_DEAD;
        while (n >= 0 && i < len) {
            // lane 0: the node's own byte; lane j: token byte i + j - 1
            const int j = i + lane - 1;
            uint32_t tb = __shfl(hb, j & 15, kWave);
            if (!shrt) tb = lane > 0 && j < len ? (uint32_t)t.tok_blob[a + j] : 0x100u;
            const bool in = lane < width && lane <= len - i;
            const uint32_t sb = in ? w.nb & 0xffu : 0x200u;
            const uint64_t term = __ballot(sb == T);
            const uint64_t diff = __ballot(lane > 0 && (!in || sb != tb));
            const int f = term ? (int)__builtin_ctzll(term) : kWave;  // the first T
            const int run = diff ? (int)__builtin_ctzll(diff) - 1 : kWave - 1;
            const int k = min(run, f);
            if (f == 0) {  // a final node has no children
                n = TAM_DEAD;
                break;
            }
            n += k;
            i += k;
            if (i >= len) break;  // the token ends inside the string
            if (k == f) {         // it runs past T
                n = TAM_DEAD;
                break;
            }
            if (k < width - 1) {
                // the token leaves the string: the child of n along its next byte
                const int32_t k0 = __shfl(w.off, k, kWave), kn = (int32_t)(__shfl(w.nb, k, kWave) >> 8);
                const uint32_t c = __shfl(tb, k + 1, kWave);
                n = TAM_DEAD;
                int32_t c0 = 0, cn = 0;
                for (int32_t j0 = 0; j0 < kn; j0 += kWave) {
                    if (!(held && k == 0 && j0 == 0)) {
                        e = Kid{TAM_DEAD, 0, 0x100u, 0};
                        if (j0 + lane < kn) e = t.kid[(int64_t)k0 + j0 + lane];
                    }
                    const uint64_t m = __ballot(j0 + lane < kn && (e.nb & 0xffu) == c);
                    if (m) {
                        const int l = (int)__builtin_ctzll(m);
                        n = __shfl(e.node, l, kWave);
                        c0 = __shfl(e.off, l, kWave);
                        cn = (int32_t)(__shfl(e.nb, l, kWave) >> 8);
                        break;
                    }
                }
                ++i;
                if (i < len && c == T) n = TAM_DEAD;  // past T
                if (n < 0 || i >= len) break;
                held = true;
                if (lane < cn) e = t.kid[(int64_t)c0 + lane];
            } else {
                held = false;
            }
            width = kWave;
            w = Walk{0, 0x200u};
            if (lane <= len - i && (int64_t)n + lane < t.N) w = t.walk[n + lane];
        }
    }
    if (lane == 0) out[b] = n;
}

// ---------------------------------------------------------------- export ---

// Lane d - 1: the hit of length d <= Lt starting below tail n (as in k_apply).
__device__ __forceinline__ int32_t tail_hit(const DevTables &t, int32_t n, int lane, int Lt) {
    if (lane >= Lt) return -1;
    const NodeSuf r = t.node_suf[n + lane + 1];
    return (r.mask >> lane) & 1u ? suf_hit(t, r.off, r.mask, lane) : -1;
}

// Rows of the nodes with a dense row; all zero for a dead node and (with tail
// compression) for a tail, whose bits k_export_tail then sets.
__global__ void __launch_bounds__(kBlock) k_export_dense(DevTables t, const int32_t *nodes, uint64_t *out) {
    const int64_t r = blockIdx.y;
    const int64_t w = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (w >= t.W) return;
    const int32_t n = nodes[r];
    const bool live = n >= 0 && (int64_t)n < t.N;
    const int64_t trow = live ? (t.row_of ? (int64_t)t.row_of[n] : (int64_t)n) : -1;
    out[r * t.W + w] = trow >= 0 ? t.table[trow * t.Wp + w] : 0ull;
}

// Tail rows (tail compression), one wave per requested row: the ids of the
// tail's tokens (as in k_apply) OR-ed into the zeroed output row.
__global__ void __launch_bounds__(kBlock) k_export_tail(DevTables t, const int32_t *nodes, int64_t nrows,
                                                        uint64_t *out) {
    const int64_t r = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (r >= nrows) return;
    const int32_t n = nodes[r];
    if (n < 0 || (int64_t)n >= t.N) return;
    const int32_t trow = t.row_of[n];
    if (trow >= 0) return;
    unsigned long long *row = reinterpret_cast<unsigned long long *>(out + r * t.W);
    auto set = [&](int32_t v) { atomicOr(row + (v >> 6), 1ull << (v & 63)); };
    const int Lt = min(min(-1 - trow, kWin), (int)t.max_len);
    const int32_t x = tail_hit(t, n, lane, Lt);
    if (x >= 0) {
        set(x);
    } else if (x <= -2) {
        const SlotPay pm = t.pay[-2 - x];
        int32_t v = pm.first;
        for (int k = 0; k < (int)pm.count; ++k) {
            set(v);
            v = t.dup_next[v];
        }
    }
    if (t.tail_long)
        for (int32_t k = t.row_ptr[n] + lane; k < t.row_ptr[n + 1]; k += kWave) set(t.entries[k]);
}

// |valid[n]| of the requested nodes, one wave per node: the popcount of its
// dense row, the length of its list, or (a tail) its tokens along the path plus
// its long tokens' list; 0 for a dead node.  The same sources as k_apply.
__global__ void __launch_bounds__(kBlock) k_row_counts(DevTables t, const int32_t *nodes, int64_t nrows,
                                                       int32_t *out) {
    const int64_t r = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (r >= nrows) return;  // uniform over the wave
    const int32_t n = nodes[r];
    int32_t c = 0;
    if (n >= 0 && (int64_t)n < t.N) {
        const int64_t trow = t.row_of ? (int64_t)t.row_of[n] : (int64_t)n;
        const bool tail = t.row_of && trow < 0;
        if (t.table && !tail) {
            const uint64_t *row = t.table + trow * t.Wp;
            for (int64_t w = lane; w < t.W; w += kWave) c += __popcll(row[w]);
        } else {
            if (tail) {  // a tail: the token of length d starting below it is the hit of node n + d
                const int Lt = min(min(-1 - (int)trow, kWin), (int)t.max_len);
                const int32_t x = tail_hit(t, n, lane, Lt);
                c = x >= 0 ? 1 : (x <= -2 ? (int32_t)t.pay[-2 - x].count : 0);
            }
            if ((!t.table || t.tail_long) && lane == 0) c += t.row_ptr[n + 1] - t.row_ptr[n];
        }
    }
    for (int o = kWave / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
    if (lane == 0) out[r] = c;
}

// -------------------------------------------------------- rows on demand ---

constexpr int kLazyProbeBlocks = 2048;  // grid of k_lazy_probe (grid-stride; blocks past the work exit)
constexpr int kLazyBatch = 4;           // candidates per thread and round in k_lazy_probe

// Exclusive prefix sum of one value per thread over a block of kLazyGroup
// threads; *total receives the sum.  sh holds kLazyGroup / kWave + 1 values.
// Waves scan their lanes with shuffles; wave 0 then scans the wave totals.
__device__ __forceinline__ int64_t group_scan(int64_t x, int64_t *total, int64_t *sh) {
    constexpr int kWaves = kLazyGroup / kWave;
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    int64_t inc = x;
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t y = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += y;
    }
    if (lane == kWave - 1) sh[wid] = inc;
    __syncthreads();
    if (wid == 0) {
        const int64_t v = lane < kWaves ? sh[lane] : 0;
        int64_t vi = v;
        for (int o = 1; o < kWaves; o <<= 1) {
            const int64_t y = __shfl_up(vi, o, kWave);
            if (lane >= o) vi += y;
        }
        if (lane < kWaves) sh[lane] = vi - v;
        if (lane == kWaves - 1) sh[kWaves] = vi;
    }
    __syncthreads();
    const int64_t before = sh[wid];
    *total = sh[kWaves];
    __syncthreads();
    return before + inc - x;
}

// Cache words that other waves of the same block read back after a barrier:
// work-group scope (the block's waves share one CU and its L1), ordered by the
// work-group fences of __syncthreads.  Nothing outside the block reads them
// before the kernel ends.
__device__ __forceinline__ uint32_t load_wg(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void store_wg(uint32_t *p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Which rows a group of nb batch rows needs built, one block of kLazyGroup
// threads, one thread per batch row.
// kCache (tam_apply_mask):
//   1. Each live row claims its node with a compare-and-swap on slot_of: a
//      slot (>= 0) is a hit; -1 makes the row the builder of the node's row (a
//      miss); -2 - b names builder b to the other rows of that node.  A group
//      without a miss ends here, its rows' slots written.
//   2. Hits stamp their slot with the group's number, so it is not evicted.
//   3. The misses take victims by CLOCK: sweeps from the hand over windows of up
//      to kLazyGroup slots take those not used by the group and without a
//      reference bit, in order, and clear the reference bit of the others they
//      pass; the hand stops after the last slot taken.  With nb <= C at least
//      as many slots are free as there are misses, so two turns of the hand
//      suffice.
//   4. A taken slot drops its old node; each builder records its node, slot,
//      depth and candidate offset for the zero and probe passes, and every
//      batch row its slot (rows_src).
// !kCache (tam_export_rows): every live row is built, into output row b.
template <bool kCache>
__global__ void __launch_bounds__(kLazyGroup) k_lazy_assign(const int32_t *__restrict__ sub_end,
                                                            const int32_t *__restrict__ depth, int64_t N,
                                                            LazyDev z, const int32_t *__restrict__ ids,
                                                            int32_t nb) {
    __shared__ int32_t s_slot[kLazyGroup];
    __shared__ int32_t s_victim[kLazyGroup];
    __shared__ int32_t s_vold[kLazyGroup];
    __shared__ int64_t s_scan[kLazyGroup / kWave + 1];
    __shared__ uint32_t s_u[4];  // group number, -, cut, counter wrapped
    const int tid = threadIdx.x;
    const int32_t n = tid < nb ? ids[tid] : -1;
    const bool live = n >= 0 && (int64_t)n < N;
    const int64_t below = live ? (int64_t)sub_end[n] - n - 1 : 0;
    const int32_t ndep = live ? depth[n] : 0;
    int32_t slot = -1, lead = -1, freed = -1;
    bool miss = live;
    uint32_t group = 0;
    const int64_t C = z.C + z.P;  // the CLOCK sweeps every cache row and passes over the spares
    const int win = (int)min<int64_t>(C, kLazyGroup);
    int64_t hand = 0;
    if (kCache) {
        if (tid == 0) {
            uint32_t g = z.state[0] + 1u;
            s_u[3] = g == 0u ? 1u : 0u;
            if (g == 0u) g = 1u;  // 0 marks a slot never used
            z.state[0] = g;
            s_u[0] = g;
            s_u[1] = z.state[2];  // the spare ring's head
        }
        if (live) {
            const int32_t v = atomicCAS(&z.slot_of[n], -1, -2 - tid);
            miss = v == -1;
            if (v >= 0)
                slot = v;
            else if (v != -1)
                lead = -2 - v;
        }
        __syncthreads();
        group = s_u[0];
        if (s_u[3]) {  // the group counter wrapped: forget every stamp
            for (int64_t c = tid; c < C; c += kLazyGroup) store_wg(&z.stamp[c], 0u);
            __syncthreads();
        }
        if (slot >= 0) {
            store_wg(&z.stamp[slot], group);
            store_wg(&z.ref[slot], 1u);
        }
    }
    s_slot[tid] = slot;
    // no miss in the group (every live row's node is cached): only the rows'
    // slots are written
    if (kCache && !__syncthreads_or(miss ? 1 : 0)) {
        if (tid < nb) z.rows_src[tid] = slot;
        if (tid == 0) {
            z.miss_off[0] = 0;
            *z.miss_count = 0;
        }
        return;
    }
    int64_t nmiss, total;
    const int32_t rank = (int32_t)group_scan(miss ? 1 : 0, &nmiss, s_scan);
    const int64_t off = group_scan(miss ? below : 0, &total, s_scan);
    const int32_t M = (int32_t)nmiss;
    if (kCache) {
        // the hits' stamps are stored (the barrier of the scans above); each
        // window of the sweep loads its slots' stamps, reference bits and
        // nodes in one round trip
        hand = z.state[1];
        int32_t taken = 0;
        const int64_t max_sweeps = 2 * ((C + win - 1) / win) + 2;
        for (int64_t it = 0; it < max_sweeps && taken < M; ++it) {
            const bool in = tid < win;
            int64_t c = hand + tid;
            if (c >= C) c -= C;
            const uint32_t st = in ? load_wg(&z.stamp[c]) : group;
            const uint32_t rf = in ? load_wg(&z.ref[c]) : 1u;
            const int32_t old = in ? z.node_of[c] : -1;
            const bool free_slot = in && st != group && old != -2;  // spares are not victims
            const bool take = free_slot && rf == 0u;
            int64_t avail64;
            const int32_t er = (int32_t)group_scan(take ? 1 : 0, &avail64, s_scan);
            const int32_t need = M - taken, avail = (int32_t)avail64;
            if (take && er == need - 1) s_u[2] = (uint32_t)tid;
            __syncthreads();
            const int cut = avail >= need ? (int)s_u[2] : win - 1;  // last slot the hand passes
            if (tid <= cut) {
                if (take && er < need) {
                    s_victim[taken + er] = (int32_t)c;
                    s_vold[taken + er] = old;
                    store_wg(&z.stamp[c], group);
                } else if (free_slot && rf != 0u) {
                    store_wg(&z.ref[c], 0u);  // second chance
                }
            }
            taken += min(avail, need);
            hand += cut + 1;
            if (hand >= C) hand -= C;
            __syncthreads();
        }
        if (tid == 0) {
            z.state[1] = (uint32_t)hand;
            z.state[2] = (uint32_t)(((int64_t)s_u[1] + taken) % z.P);
        }
        if (miss) {
            const int32_t c = rank < taken ? s_victim[rank] : -1;
            if (c >= 0) {
                // the miss's row is the next spare (zero); its victim c becomes a
                // spare in that place, cleared by this group's build pass
                const int64_t at = ((int64_t)s_u[1] + rank) % z.P;
                const int32_t r = z.spare[at];
                z.spare[at] = c;
                freed = c;
                const int32_t old = s_vold[rank];
                if (old >= 0) z.slot_of[old] = -1;
                z.node_of[c] = -2;
                z.node_of[r] = n;
                z.slot_of[n] = r;
                store_wg(&z.stamp[r], group);
                store_wg(&z.ref[r], 1u);
                s_slot[tid] = r;
            } else {
                // not reached while nb <= C (two turns of the hand find the
                // slots); counted as an error, the rows stay fully masked
                z.slot_of[n] = -1;
                atomicAdd(z.err, 1);
                s_slot[tid] = -1;
            }
        }
        __syncthreads();
        if (tid < nb) z.rows_src[tid] = lead >= 0 ? s_slot[lead] : s_slot[tid];
    }
    if (miss) {
        z.miss_node[rank] = n;
        z.miss_row[rank] = kCache ? s_slot[tid] : tid;
        z.miss_free[rank] = freed;
        z.miss_off[rank] = off;
        z.miss_dep[rank] = ndep;
    }
    if (tid == 0) {
        z.miss_off[M] = total;
        *z.miss_count = M;
    }
}

// The hits of K independent suffixes (the one of d[k] bytes ending at blob
// position pos[k], window (lo[k], hi[k]); act[k] false: none) with their
// memory round trips issued together: short suffixes read short_hits, the
// others their home bucket, then the payload (and pay_hi) of the first
// fingerprint match; a length the home bucket does not settle falls back to
// the general probe.
template <int K>
__device__ __forceinline__ void probe_batch(const DevTables &t, const int64_t (&pos)[K], const int (&d)[K],
                                            const bool (&act)[K], const uint64_t (&lo)[K], const uint64_t (&hi)[K],
                                            int32_t (&hit)[K]) {
    uint64_t key[K];
    bool hashed[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        hit[k] = -1;
        hashed[k] = act[k] && d[k] > kShortLen;
        key[k] = 0;
        if (act[k] && d[k] <= kShortLen) hit[k] = short_hit(t, d[k], window_byte(lo[k], hi[k], 0), window_byte(lo[k], hi[k], 1));
        if (hashed[k]) {
            uint32_t h = kHashSeed;
            for (int j = 0; j < d[k]; ++j)
                h = hash_step(h, j < kWin ? window_byte(lo[k], hi[k], j) : (uint32_t)t.blob[pos[k] - j]);
            key[k] = hash_final(h);
        }
    }
    Bucket bk[K];
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (hashed[k]) bk[k] = load_bucket(t, home_bucket(t, key[k]));
    uint32_t match[K], empty[K];
    int32_t slot[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        match[k] = empty[k] = 0;
        slot[k] = -1;
        if (hashed[k]) {
            bucket_masks(bk[k], fingerprint(key[k]), &match[k], &empty[k]);
            if (match[k]) slot[k] = (int32_t)(bucket_base(bk[k]) + (uint32_t)__builtin_ctz(match[k]));
        }
    }
    SlotPay p[K];
    uint64_t phi[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        phi[k] = 0;
        if (slot[k] >= 0) {
            p[k] = t.pay[slot[k]];
            if (d[k] > 8) phi[k] = t.pay_hi[slot[k]];
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (!hashed[k]) continue;
        if (slot[k] >= 0 && slot_equals(t, p[k], phi[k], d[k], lo[k], hi[k], pos[k])) {
            hit[k] = hit_of_slot(slot[k], p[k].first, p[k].count);
        } else if (!(empty[k] != 0 && (match[k] & (match[k] - 1)) == 0)) {
            SlotPay mt;  // the home bucket does not settle it
            const int32_t sl = probe(t, key[k], d[k], lo[k], hi[k], pos[k], &mt);
            if (sl >= 0) hit[k] = hit_of_slot(sl, mt.first, mt.count);
        }
    }
}

// The candidates of misses: candidate i of miss u is node m = n + 1 + (i -
// miss_off[u]) for the misses the pass covers, a descendant d = depth(m) -
// depth(n) bytes below n (preorder: the subtree is [n, sub_end[n])).  When
// d <= max_len and the last d bytes of prefix(m), the path from n to m, are a
// token string, its ids are valid at n; every token valid at n ends its walk
// at exactly one such m.  set(row, id) records a valid id.
template <typename F>
__device__ __forceinline__ void lazy_candidates(const DevTables &t, const int64_t (&m)[kLazyBatch],
                                                const int (&dep)[kLazyBatch], bool (&act)[kLazyBatch],
                                                const int32_t (&row)[kLazyBatch], F &&set) {
    constexpr int K = kLazyBatch;
    int dm[K], d[K];
    int64_t pos[K];
#pragma unroll
    for (int k = 0; k < K; ++k) dm[k] = act[k] ? t.depth[m[k]] : 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        d[k] = dm[k] - dep[k];
        act[k] = act[k] && row[k] >= 0 && d[k] <= t.max_len && has_len(t, d[k]);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) pos[k] = act[k] ? t.node_pos[m[k]] : 0;
    uint64_t wlo[K], whi[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        wlo[k] = whi[k] = 0;
        if (act[k]) load_window(t.blob, pos[k], wlo[k], whi[k]);
    }
    int32_t hx[K];
    probe_batch<K>(t, pos, d, act, wlo, whi, hx);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (hx[k] == -1) continue;
        if (hx[k] >= 0) {  // one token id (the common case)
            set(row[k], hx[k]);
            continue;
        }
        const SlotPay pm = t.pay[-2 - hx[k]];  // a string with several ids
        int32_t v = pm.first;
        for (int j = 0; j < (int)pm.count; ++j) {
            set(row[k], v);
            v = t.dup_next[v];
        }
    }
}

// The grid-stride pass over the candidates of the misses miss_off covers,
// with 64-bit atomics into the zeroed rows dest + row * stride; block bx of nbx,
// kLazyBatch candidates per thread and round with their loads issued together.
// LDS of the pass: the misses' candidate offsets, nodes, rows and depths.
struct LazyMisses {
    int64_t off[kLazyGroup + 1];
    int32_t node[kLazyGroup], row[kLazyGroup], dep[kLazyGroup];
};

__device__ __forceinline__ void lazy_probe_pass(const DevTables &t, const LazyDev &z, uint64_t *dest, int64_t stride,
                                                int64_t bx, int64_t nbx, LazyMisses &sm) {
    constexpr int K = kLazyBatch;
    int64_t *s_off = sm.off;
    int32_t *s_node = sm.node, *s_row = sm.row, *s_dep = sm.dep;
    const int32_t M = *z.miss_count;
    if (M <= 0) return;
    const int64_t total = z.miss_off[M];
    const int64_t first = bx * kBlock;
    if (first >= total) return;
    for (int i = threadIdx.x; i <= M; i += kBlock) s_off[i] = z.miss_off[i];
    for (int i = threadIdx.x; i < M; i += kBlock) {
        s_node[i] = z.miss_node[i];
        s_row[i] = z.miss_row[i];
        s_dep[i] = z.miss_dep[i];
    }
    __syncthreads();
    unsigned long long *out = reinterpret_cast<unsigned long long *>(dest);
    const int64_t threads = nbx * kBlock;
    for (int64_t base = first + threadIdx.x; base < total; base += K * threads) {
        int64_t m[K];
        int32_t row[K];
        int dep[K];
        bool act[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t i = base + k * threads;
            act[k] = i < total;
            row[k] = -1;
            m[k] = 0;
            dep[k] = 0;
            if (!act[k]) continue;
            int lo = 0, hi = M - 1;  // the last miss whose candidates start at or before i
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_off[mid] <= i)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            row[k] = s_row[lo];
            m[k] = (int64_t)s_node[lo] + 1 + (i - s_off[lo]);
            dep[k] = s_dep[lo];
        }
        lazy_candidates(t, m, dep, act, row, [&](int32_t r, int32_t v) {
            atomicOr(out + (int64_t)r * stride + (v >> 6), 1ull << (v & 63));
        });
    }
}

// The rows of the group's misses, in their cache rows (spares, zero) for
// tam_apply_mask, or straight into the zeroed output rows for tam_export_rows.
// clear (tam_apply_mask): the cache rows the misses freed are zeroed first, so
// that they are zero when a later group takes them as spares.
__global__ void __launch_bounds__(kBlock) k_lazy_probe(DevTables t, LazyDev z, uint64_t *dest, int64_t stride,
                                                       int clear) {
    __shared__ LazyMisses sm;
    if (clear) {
        const int32_t M = *z.miss_count;
        const int32_t per = (int32_t)(t.Wp / 2);  // 16-byte chunks per row
        const int64_t chunks = (int64_t)M * per;
        for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < chunks; i += (int64_t)gridDim.x * kBlock) {
            const int32_t u = (int32_t)(i / per);
            const int32_t r = z.miss_free[u];
            if (r >= 0 && (int64_t)r < z.C + z.P)
                reinterpret_cast<u32x4 *>(z.cache + (int64_t)r * t.Wp)[i - (int64_t)u * per] = u32x4{0u, 0u, 0u, 0u};
        }
    }
    lazy_probe_pass(t, z, dest, stride, blockIdx.x, gridDim.x, sm);
}

// p[i] = first + i, i < n.
__global__ void __launch_bounds__(kBlock) k_iota_i32(int32_t *p, int64_t n, int32_t first) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = first + (int32_t)i;
}

__global__ void __launch_bounds__(kBlock) k_fill_u64(uint64_t *p, int64_t n, uint64_t value) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
        p[i] = value;
}

inline unsigned grid_for(int64_t n, int per_block) {
    return (unsigned)((n + per_block - 1) / per_block);
}

}  // namespace

int64_t scan_tmp_elems(int64_t N) { return (N + kScanTile - 1) / kScanTile + 1; }

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t value, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const unsigned g = (unsigned)std::min<int64_t>(grid_for(n, kBlock), 4096);
    hipLaunchKernelGGL(k_fill_i32, dim3(g), dim3(kBlock), 0, s, p, n, value);
    return hipGetLastError();
}

hipError_t launch_probe(const DevTables &t, bool count, bool mark, int32_t *pairs, hipStream_t s) {
    if (t.N <= 0) return hipSuccess;
    const int do_mark = mark && t.table ? 1 : 0;
    const dim3 grid((unsigned)mark_blocks(t.N));
    if (t.tail_lists) return hipErrorInvalidValue;  // the groups' grid (launch_probe_groups)
    const RecGroups none{};
    if (count)
        hipLaunchKernelGGL((k_probe<true, false>), grid, dim3(kBlock), 0, s, t, (int64_t)0, t.N, do_mark, pairs, none,
                           (int64_t)0);
    else
        hipLaunchKernelGGL((k_probe<false, false>), grid, dim3(kBlock), 0, s, t, (int64_t)0, t.N, do_mark, pairs, none,
                           (int64_t)0);
    return hipGetLastError();
}

// The host checks the groups' grid: consecutive node ranges within [0, N),
// each with as many blocks as its nodes need, blocks and offsets increasing.
static bool groups_ok(const DevTables &t, const RecGroups &rg) {
    if (rg.n < 1 || rg.n > kMaxRecGroups || rg.blk0[0] != 0) return false;
    for (int k = 0; k < rg.n; ++k) {
        const int64_t nodes = rg.n_hi[k] - rg.n_lo[k];
        if (rg.n_lo[k] < 0 || nodes <= 0 || rg.n_hi[k] > t.N || !rg.rec[k]) return false;
        if (rg.blk0[k + 1] - rg.blk0[k] != mark_blocks(nodes)) return false;
        if (k > 0 && (rg.n_lo[k] != rg.n_hi[k - 1] || rg.off0[k] < rg.off0[k - 1] + (rg.blk0[k] - rg.blk0[k - 1]) + 1))
            return false;
    }
    return true;
}

hipError_t launch_probe_groups(const DevTables &t, const RecGroups &rg, int64_t k0, int64_t k1, int32_t *pairs,
                               hipStream_t s) {
    if (!t.tail_lists || t.table || !pairs || !groups_ok(t, rg) || k0 < 0 || k1 > rg.n || k0 >= k1)
        return hipErrorInvalidValue;
    const int64_t b0 = rg.blk0[k0], b1 = rg.blk0[k1];
    hipLaunchKernelGGL((k_probe<true, true>), dim3((unsigned)(b1 - b0)), dim3(kBlock), 0, s, t, (int64_t)0, t.N, 0, pairs,
                       rg, b0);
    return hipGetLastError();
}

hipError_t launch_count_range(const DevTables &t, int64_t m0, int64_t m1, hipStream_t s) {
    if (m1 <= m0) return hipSuccess;
    if (m0 < 0 || m1 > t.N || t.table || t.tail_lists) return hipErrorInvalidValue;
    const RecGroups none{};
    hipLaunchKernelGGL((k_probe<true, false>), dim3((unsigned)mark_blocks(m1 - m0)), dim3(kBlock), 0, s, t, m0, m1, 0,
                       (int32_t *)nullptr, none, (int64_t)0);
    return hipGetLastError();
}

hipError_t launch_lay_init(int32_t *node_at, int64_t blob_bytes, int32_t *kid_cnt, int32_t *count, int64_t N,
                           int32_t *err, int32_t *kid_total, hipStream_t s) {
    if (blob_bytes < 2 * kBlobPad) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_lay_init, dim3(grid_for(std::max<int64_t>(N, kBlobPad), kBlock)), dim3(kBlock), 0, s, node_at,
                       blob_bytes, kid_cnt, count, N, err, kid_total);
    return hipGetLastError();
}

hipError_t launch_lay(const StrRec *strs, const TailRec *trec, int64_t s0, int64_t s1, int64_t blob_bytes, int64_t N,
                      const LayTables &o, int32_t *kid_cnt, int32_t *kid_parent, int32_t *kid_rank, int32_t *err,
                      hipStream_t s) {
    if (s1 <= s0) return hipSuccess;
    if ((trec != nullptr) != (o.row_of != nullptr)) return hipErrorInvalidValue;
    for (int64_t u0 = s0; u0 < s1; u0 += kLayStrings) {
        const int64_t u1 = std::min(u0 + kLayStrings, s1);
        hipLaunchKernelGGL(k_lay, dim3(grid_for(u1 - u0, kBlock / kWave)), dim3(kBlock), 0, s, strs, trec, s0, u0, u1,
                           blob_bytes, N, o, kid_cnt, kid_parent, kid_rank, err);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_kids(const StrRec *strs, int64_t K, int64_t N, Walk *walk, Kid *kid, const int32_t *kid_cnt,
                       const int32_t *kid_parent, const int32_t *kid_rank, int32_t *kid_total, int32_t *err,
                       hipStream_t s) {
    if (K <= 0 || N <= 0) return hipSuccess;
    const dim3 grid(grid_for(K, kBlock));
    hipLaunchKernelGGL(k_kid_alloc, grid, dim3(kBlock), 0, s, K, walk, kid_cnt, kid_parent, kid_rank, kid_total);
    hipLaunchKernelGGL(k_kid_fill, grid, dim3(kBlock), 0, s, strs, K, walk, kid, kid_parent, kid_rank, err);
    return hipGetLastError();
}

hipError_t launch_tok_heads(const uint32_t *tok_off, const uint8_t *tok_blob, int64_t V, TokHead *head, hipStream_t s) {
    if (V <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tok_heads, dim3(grid_for(V, kBlock)), dim3(kBlock), 0, s, tok_off, tok_blob, V, head);
    return hipGetLastError();
}

void suf_sizes(SufBuild &b) {
    // at most 3.2 entries per bucket of eight on average (fewer: equal markers are
    // one entry), so that one bucket in 200 overflows; the scratch set at most
    // half full
    b.buckets = std::min<int64_t>(b.entries * 5 / 16 + 64, INT32_MAX / kSufSlots);  // entry numbers are 31 bits
    b.set_slots = 64;
    while (b.set_slots < 2 * b.entries) b.set_slots <<= 1;
}

hipError_t launch_suffix_table(const DevTables &t, const SufBuild &b, hipStream_t s) {
    if (b.strings < 1 || b.buckets < 1 || b.buckets > INT32_MAX / kSufSlots) return hipErrorInvalidValue;
    const dim3 strings(grid_for(b.strings, kBlock));
    hipLaunchKernelGGL(k_suf_init, dim3((unsigned)std::min<int64_t>(grid_for(b.set_slots, kBlock), 8192)), dim3(kBlock),
                       0, s, b);
    hipLaunchKernelGGL(k_suf_lists, strings, dim3(kBlock), 0, s, t, b);
    hipLaunchKernelGGL(k_suf_short, dim3(grid_for(kShortEntries, kBlock)), dim3(kBlock), 0, s, t, b);
    hipLaunchKernelGGL(k_suf_insert, dim3(grid_for(4 * b.strings, kBlock)), dim3(kBlock), 0, s, t, b);
    hipLaunchKernelGGL(k_suf_fill, dim3(grid_for(b.set_slots, kBlock)), dim3(kBlock), 0, s, t, b);
    return hipGetLastError();
}

int64_t probe_nodes_per_block() { return kBlock; }

hipError_t launch_fill_records(const DevTables &t, const RecGroups &rg, hipStream_t s) {
    if (!groups_ok(t, rg)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_fill_records, dim3((unsigned)rg.blk0[rg.n]), dim3(kFillThreads), 0, s, t, rg);
    return hipGetLastError();
}

hipError_t launch_fill_lists(const DevTables &t, hipStream_t s) {
    if (t.N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3(grid_for(t.N, kBlock)), dim3(kBlock), 0, s, t);
    return hipGetLastError();
}

hipError_t launch_zero(uint64_t *p, int64_t words, hipStream_t s) {
    const int64_t n16 = words / 2;
    if (n16 <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero, dim3(grid_for(n16, kBlock)), dim3(kBlock), 0, s,
                       reinterpret_cast<u32x4 *>(p), n16);
    return hipGetLastError();
}

int64_t mark_blocks(int64_t N) { return (N + kBlock - 1) / kBlock; }

int64_t format_blocks(int64_t Wp) { return (Wp * kWave + kBlock - 1) / kBlock; }

hipError_t launch_format(const DevTables &t, int32_t *pairs, hipStream_t s) {
    hipLaunchKernelGGL(k_format, dim3((unsigned)format_blocks(t.Wp)), dim3(kBlock), 0, s, t, t.table, t.Wp, t.Wp,
                       pairs, (unsigned long long *)nullptr);
    return hipGetLastError();
}

hipError_t launch_scan(const DevTables &t, int32_t *zero, hipStream_t s) {
    const int64_t nb = grid_for(t.N, kScanTile);
    const int how = nb <= kScanSelfBlocks ? kScanSelf : nb <= kScanTile ? kScanOwn : kScanTop;
    if (how != kScanSelf)
        hipLaunchKernelGGL(k_scan_blocks, dim3((unsigned)nb), dim3(kBlock), 0, s, t.count, t.N, t.scan_tmp);
    if (how == kScanTop)
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kBlock), 0, s, t.scan_tmp, nb, t.row_ptr + t.N);
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(kBlock), 0, s, t.count, t.N, t.scan_tmp, how,
                       t.row_ptr, t.row_ptr + t.N, zero);
    return hipGetLastError();
}

hipError_t launch_rows(const DevTables &t, const int32_t *nodes, int64_t nrows, uint64_t *out,
                       int64_t out_stride_words, int64_t out_words, hipStream_t s) {
    if (nrows <= 0 || out_words <= 0) return hipSuccess;
    const bool vec = (out_stride_words & 1) == 0 && (out_words & 1) == 0 &&
                     (reinterpret_cast<uintptr_t>(out) & 15) == 0;
    int per_cu = 0;
    hipError_t e = vec ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_rows<2>, kBlock, 0)
                       : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_rows<1>, kBlock, 0);
    if (e != hipSuccess || per_cu <= 0) per_cu = 4;
    const int64_t waves_needed = nrows;
    const int64_t cap = (int64_t)props_for_current_device().cus * per_cu;
    const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(cap, grid_for(waves_needed, kBlock / kWave)));
    if (vec)
        hipLaunchKernelGGL(k_rows<2>, dim3(g), dim3(kBlock), 0, s, t.row_ptr, t.entries, nodes, nrows, t.N, out,
                           out_stride_words, out_words);
    else
        hipLaunchKernelGGL(k_rows<1>, dim3(g), dim3(kBlock), 0, s, t.row_ptr, t.entries, nodes, nrows, t.N, out,
                           out_stride_words, out_words);
    return hipGetLastError();
}

// Blocks per row of a dense or tail launch.  Consecutive blocks go to the eight XCDs
// in turn, so with a multiple of eight blocks per row each part of every row falls to
// the same XCD; with new rows in every call that was the slower order (not with rows
// that the caches hold, nor behind 1 GiB of other traffic).  One block more, which
// finds no chunk, turns the order by one XCD from row to row.  us per call of 256 rows, new ones in every
// call, with 8 k and 8 k + 1 blocks of two chunks: tail rows, bf16 over V = 262,144 29.8
// and 24.3, fp32 45.2 and 41.8, bf16 over V = 128,255 18.7 and 15.7, fp32 over V = 32,000
// 10.3 and 9.5; dense rows 30.4 and 30.1, 64.4 and 64.5, 18.3 and 17.5, 8.8 and 8.4.  Below two rounds
// of the 2,048 blocks that run at once the block more costs what it gives or more (tail
// rows over V = 128,255, 64 rows 6.30 and 6.45; V = 32,000, 256 rows of 8 and 9 blocks 5.65
// and 6.43).
static unsigned row_blocks(int64_t nchunks, int per, int64_t rows) {
    const unsigned gx = grid_for(nchunks, per);
    return (gx & 7u) == 0 && gx >= 16 && (int64_t)gx * rows >= 4096 ? gx + 1 : gx;
}

// Two chunks per thread for dense rows and three for tail rows while that leaves
// kApplyWide blocks, else one; plain lists always one.  grid.y is limited to 65535
// rows per launch.
template <typename T, bool kAligned>
static hipError_t launch_apply_rows(const DevTables &t, const int32_t *node_ids, int64_t B, T *logits,
                                    int64_t row_stride, int64_t nchunks, hipStream_t s) {
    const int per = kBlock * (t.row_of ? kTailChunks : kDenseChunks);
    const bool wide = (t.row_of || t.table) && (int64_t)grid_for(nchunks, per) * B >= kApplyWide;
    for (int64_t r0 = 0; r0 < B; r0 += 65535) {
        const int64_t rows = std::min<int64_t>(B - r0, 65535);
        const dim3 grid(row_blocks(nchunks, wide ? per : kBlock, rows), (unsigned)rows);
        const dim3 list_grid(grid_for(nchunks, kBlock), (unsigned)rows);
        const int32_t *ids = node_ids + r0;
        T *p = logits + r0 * row_stride;
        if (t.row_of && wide)
            hipLaunchKernelGGL((k_apply<T, kApplyTail, kTailChunks, kAligned>), grid, dim3(kBlock), 0, s, t, ids, p,
                               row_stride);
        else if (t.row_of)
            hipLaunchKernelGGL((k_apply<T, kApplyTail, 1, kAligned>), grid, dim3(kBlock), 0, s, t, ids, p, row_stride);
        else if (wide)
            hipLaunchKernelGGL((k_apply_dense<T, kDenseChunks, kAligned>), grid, dim3(kBlock), 0, s, t, ids, p,
                               row_stride);
        else if (t.table)
            hipLaunchKernelGGL((k_apply_dense<T, 1, kAligned>), grid, dim3(kBlock), 0, s, t, ids, p, row_stride);
        else
            hipLaunchKernelGGL((k_apply<T, kApplyLists, 1, kAligned>), list_grid, dim3(kBlock), 0, s, t, ids, p,
                               row_stride);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T>
static hipError_t launch_apply_typed(const DevTables &t, const int32_t *node_ids, int64_t B, T *logits,
                                     int64_t row_stride, hipStream_t s) {
    constexpr int E = 16 / (int)sizeof(T);
    const bool aligned =
        (reinterpret_cast<uintptr_t>(logits) & 15) == 0 && ((row_stride * (int64_t)sizeof(T)) & 15) == 0;
    const int64_t nchunks = (t.V + (aligned ? 0 : E - 1) + E - 1) / E;  // a shifted row may touch one more
    return aligned ? launch_apply_rows<T, true>(t, node_ids, B, logits, row_stride, nchunks, s)
                   : launch_apply_rows<T, false>(t, node_ids, B, logits, row_stride, nchunks, s);
}

hipError_t launch_apply(const DevTables &t, const int32_t *node_ids, int64_t B, void *logits, int dtype,
                        int64_t row_stride, hipStream_t s) {
    if (dtype == TAM_DTYPE_BF16)
        return launch_apply_typed(t, node_ids, B, static_cast<uint16_t *>(logits), row_stride, s);
    return launch_apply_typed(t, node_ids, B, static_cast<uint32_t *>(logits), row_stride, s);
}

hipError_t launch_advance(const DevTables &t, const int32_t *node_ids, const int32_t *token_ids, int64_t B,
                          int32_t *out, hipStream_t s) {
    if (B <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_advance, dim3(grid_for(B, kBlock / kWave)), dim3(kBlock), 0, s, t, node_ids, token_ids, B,
                       out);
    return hipGetLastError();
}

hipError_t launch_lazy_apply(const DevTables &t, const LazyDev &z, const int32_t *node_ids, int64_t nb,
                             void *logits, int dtype, int64_t row_stride, hipStream_t s) {
    if (nb <= 0) return hipSuccess;
    if (nb > kLazyGroup || nb > z.C || !t.sub_end) return hipErrorInvalidValue;
    if (nb > z.P) return hipErrorInvalidValue;  // a group's misses take at most P spares
    hipLaunchKernelGGL(k_lazy_assign<true>, dim3(1), dim3(kLazyGroup), 0, s, t.sub_end, t.depth, t.N, z, node_ids,
                       (int32_t)nb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lazy_probe, dim3(kLazyProbeBlocks), dim3(kBlock), 0, s, t, z, z.cache, t.Wp, 1);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    // the masking reads the cache as a dense table indexed by cache row
    DevTables tc = t;
    tc.table = z.cache;
    tc.row_of = nullptr;
    tc.N = z.C + z.P;
    tc.R = z.C + z.P;
    return launch_apply(tc, z.rows_src, nb, logits, dtype, row_stride, s);
}

hipError_t launch_lazy_export(const DevTables &t, const LazyDev &z, const int32_t *node_ids, int64_t nb,
                              uint64_t *out, hipStream_t s) {
    if (nb <= 0) return hipSuccess;
    if (nb > kLazyGroup || !t.sub_end) return hipErrorInvalidValue;
    const int64_t words = nb * t.W;
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)std::min<int64_t>(grid_for(words, kBlock), 4096)), dim3(kBlock),
                       0, s, out, words, 0ull);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lazy_assign<false>, dim3(1), dim3(kLazyGroup), 0, s, t.sub_end, t.depth, t.N, z, node_ids,
                       (int32_t)nb);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lazy_probe, dim3(kLazyProbeBlocks), dim3(kBlock), 0, s, t, z, out, t.W, 0);
    return hipGetLastError();
}

hipError_t launch_lazy_reset(const DevTables &t, const LazyDev &z, hipStream_t s) {
    // rows 0 .. C-1 empty, C .. C+P-1 the spares (zeroed), in ring order
    hipError_t e = launch_fill_i32(z.slot_of, t.N, -1, s);
    if (e == hipSuccess) e = launch_fill_i32(z.node_of, z.C, -1, s);
    if (e == hipSuccess) e = launch_fill_i32(z.node_of + z.C, z.P, -2, s);
    if (e == hipSuccess) e = launch_fill_i32(reinterpret_cast<int32_t *>(z.stamp), z.C + z.P, 0, s);
    if (e == hipSuccess) e = launch_fill_i32(reinterpret_cast<int32_t *>(z.ref), z.C + z.P, 0, s);
    if (e == hipSuccess) e = launch_fill_i32(reinterpret_cast<int32_t *>(z.state), 3, 0, s);
    if (e != hipSuccess || z.P <= 0) return e;
    hipLaunchKernelGGL(k_iota_i32, dim3(grid_for(z.P, kBlock)), dim3(kBlock), 0, s, z.spare, z.P, (int32_t)z.C);
    e = hipGetLastError();
    if (e == hipSuccess) e = launch_zero(z.cache + z.C * t.Wp, z.P * t.Wp, s);
    return e;
}

hipError_t launch_row_counts(const DevTables &t, const int32_t *node_ids, int64_t n, int32_t *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_row_counts, dim3(grid_for(n, kBlock / kWave)), dim3(kBlock), 0, s, t, node_ids, n, out);
    return hipGetLastError();
}

hipError_t launch_export_tail(const DevTables &t, const int32_t *node_ids, int64_t n, uint64_t *out, hipStream_t s) {
    if (n <= 0 || !t.row_of) return hipSuccess;
    hipLaunchKernelGGL(k_export_tail, dim3(grid_for(n, kBlock / kWave)), dim3(kBlock), 0, s, t, node_ids, n, out);
    return hipGetLastError();
}

hipError_t launch_export_dense(const DevTables &t, const int32_t *node_ids, int64_t n, uint64_t *out,
                               hipStream_t s) {
    for (int64_t r0 = 0; r0 < n; r0 += 65535) {
        const unsigned rows = (unsigned)std::min<int64_t>(n - r0, 65535);
        hipLaunchKernelGGL(k_export_dense, dim3(grid_for(t.W, kBlock), rows), dim3(kBlock), 0, s, t,
                           node_ids + r0, out + r0 * t.W);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (!t.row_of) return hipSuccess;
    hipLaunchKernelGGL(k_export_tail, dim3(grid_for(n, kBlock / kWave)), dim3(kBlock), 0, s, t, node_ids, n, out);
    return hipGetLastError();
}

// ------------------------------------------- format rows, no allocation ---

// The scratch of tam_format_rows_noalloc: a counter of the valid pairs, then
// the class bits of up to TAM_NOALLOC_MAX_POSITIONS positions, staged from the
// host through kernel arguments.  One copy per GPU, held until the process
// ends; every call on a GPU shares it (overlapping calls race).  Host code
// never names the array itself: it takes the device address that
// hipGetSymbolAddress returns (noalloc_scratch) and passes that to kernels.
constexpr size_t kScratchHeader = 256;
constexpr size_t kScratchBytes = kScratchHeader + 32 * (size_t)TAM_NOALLOC_MAX_POSITIONS;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

namespace {

constexpr int kStagePositions = 64;  // positions per staging launch (2 KiB of kernel arguments)

struct ClassChunk {
    int32_t first, count;                  // positions [first, first + count)
    uint32_t words[kStagePositions * 8];   // their class bits, 32 bytes per position
};

// Copies one chunk of class bits into the scratch (the first chunk also
// clears the pair counter).
__global__ void __launch_bounds__(kBlock) k_stage_classes(ClassChunk c, uint32_t *__restrict__ cls,
                                                          unsigned long long *counter) {
    for (int i = threadIdx.x; i < c.count * 8; i += kBlock) cls[(int64_t)c.first * 8 + i] = c.words[i];
    if (c.first == 0 && threadIdx.x == 0) *counter = 0ull;
}

__global__ void k_store_total(const unsigned long long *counter, int64_t *out) {
    if (threadIdx.x == 0) *out = (int64_t)*counter;
}

std::mutex g_scratch_mutex;
void *g_scratch_ptr[64] = {};

}  // namespace

// The device address of this GPU's scratch, looked up once per device with
// that device current.
hipError_t noalloc_scratch(uint8_t **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> g(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = static_cast<uint8_t *>(g_scratch_ptr[dev]);
    return hipSuccess;
}

hipError_t launch_format_noalloc(const DevTables &t, const uint8_t *classes_host, uint64_t *out, int64_t stride,
                                 int64_t *pairs_out, hipStream_t s) {
    const int64_t L = t.fmt_L;
    if (L < 1 || L > TAM_NOALLOC_MAX_POSITIONS || stride < t.W) return hipErrorInvalidValue;
    uint8_t *base = nullptr;
    hipError_t e = noalloc_scratch(&base);
    if (e != hipSuccess) return e;
    unsigned long long *counter = reinterpret_cast<unsigned long long *>(base);
    uint32_t *cls = reinterpret_cast<uint32_t *>(base + kScratchHeader);
    for (int64_t p0 = 0; p0 < L; p0 += kStagePositions) {
        ClassChunk c;
        c.first = (int32_t)p0;
        c.count = (int32_t)std::min<int64_t>(kStagePositions, L - p0);
        std::memset(c.words, 0, sizeof(c.words));
        std::memcpy(c.words, classes_host + 32 * p0, (size_t)c.count * 32);
        hipLaunchKernelGGL(k_stage_classes, dim3(1), dim3(kBlock), 0, s, c, cls, counter);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    DevTables tf = t;
    tf.classes = reinterpret_cast<const uint8_t *>(cls);
    hipLaunchKernelGGL(k_format, dim3((unsigned)format_blocks(t.W)), dim3(kBlock), 0, s, tf, out, stride, t.W,
                       (int32_t *)nullptr, counter);
    e = hipGetLastError();
    if (e != hipSuccess || !pairs_out) return e;
    hipLaunchKernelGGL(k_store_total, dim3(1), dim3(kWave), 0, s, counter, pairs_out);
    return hipGetLastError();
}

}  // namespace tam
