// Prefix walk over the per-depth arrays, shared by the kernels of libppv_hip.so.
#pragma once
#include "ppv_device.h"
#include "ppv_internal.h"

namespace {

// ------------------------------------------------------------------------------------------
// Prefix walk, one wavefront per prefix (Section 3.2 "Parallel Verification": the search that
// locates a prefix in sorted S; here it descends the per-depth arrays, one 64-way search among
// the children of the current prefix per token, instead of log2|S| probes of whole rows).
// All 64 lanes call it with the same arguments; every result is wave-uniform.
struct Walk {
    uint32_t node;    // the prefix's entry (meaningful when found)
    uint32_t cb, ce;  // its children (when found)
    uint32_t tok;     // its entry's token word with flags (when found and t > 0)
    uint32_t only;    // PPV_NO_SLOT; or the prefix is one of a single member, and this is its one child's token word (token |
                      // PPV_NODE_TERMINAL): cb, ce say 0, 1 then and node is not known (see walk_prefix)
    uint32_t slot;    // the node's slot among the heavy ones, PPV_NO_SLOT if it is not heavy or not known
    uint32_t lo, hi;  // rank range in sorted S; lo == hi == insertion rank when not found
    bool found;       // the prefix is a prefix of at least one member
    bool member;      // the prefix itself is in S
};

__device__ inline uint32_t heavy_slot_of(const IndexView &ix, uint32_t node) {
    return node < ix.heavy_limit ? ix.heavy_slot[node] : PPV_NO_SLOT;
}

// Search `key` among the entries [begin, end) (strictly increasing tokens).  `at` is the first
// position whose token is >= key; on a match tok and child are that entry's and next_child is the child
// offset of the entry after it (the end of the match's own children), else tok = PPV_NO_SLOT.
struct Found {
    uint32_t at, tok, child, next_child;
};
__device__ __forceinline__ Found wave_search(const NodeEnt *__restrict__ ent, uint32_t begin, uint32_t end, uint32_t key,
                                             int lane) {
    uint32_t lo = begin, hi = end;
    while (hi - lo > (uint32_t)(WAVE - 1)) {
        uint32_t n = hi - lo;
        uint32_t step = (n + WAVE - 1) / WAVE;
        uint32_t p = (uint32_t)(lane + 1) * step;
        if (p > n) p = n;
        uint32_t v = ent[lo + p - 1].tok & PPV_NODE_TOKEN;  // 64 pivots, the last one is the last entry
        int c = __popcll(__ballot(v < key));                // pivots below the key
        if (c == WAVE) { lo = hi; break; }                  // everything is below the key
        uint32_t nlo = lo + (uint32_t)c * step;
        uint32_t nhi = lo + (uint32_t)(c + 1) * step;
        if (nhi > hi) nhi = hi;
        lo = nlo;
        hi = nhi;
    }
    // at most 63 candidates: lane l takes entry lo+l, one lane more takes the entry after them
    // (always there: the array ends with a sentinel), which closes the last candidate's children
    const uint32_t n = hi - lo;
    NodeEnt e;
    e.tok = PPV_NO_SLOT;
    e.child = 0;
    if ((uint32_t)lane <= n) e = ent[lo + lane];
    const bool in = (uint32_t)lane < n;
    const uint32_t v = e.tok & PPV_NODE_TOKEN;
    const int c = __popcll(__ballot(in && v < key));
    const uint64_t eq = __ballot(in && v == key);
    const int l = eq ? __ffsll((long long)eq) - 1 : 0;
    return {lo + (uint32_t)c, eq ? lane_value(e.tok, l) : PPV_NO_SLOT, lane_value(e.child, l), lane_value(e.child, l + 1)};
}

// The descent from a known node: token i of the prefix is searched among the children of the node reached
// by tokens 0..i-1, for i = start .. t-1.  `mine` is lane l's token l of the prefix (the first 64 tokens
// in one coalesced load; token i is broadcast from lane i).
template <bool SLOT>
__device__ __forceinline__ Walk walk_from(const IndexView &ix, const int32_t *__restrict__ prefix, int t, int lane,
                                          int32_t mine, int start, uint32_t node, uint32_t tokw, uint32_t cb, uint32_t ce) {
    Walk w;
    w.node = node;
    w.cb = cb;
    w.ce = ce;
    w.tok = tokw;
    w.only = PPV_NO_SLOT;
    w.found = true;
    w.member = false;
    for (int i = start; i < t; i++) {
        const uint32_t key = (uint32_t)((i < WAVE) ? lane_value(mine, i) : prefix[i]);
        const Found hit = wave_search(ix.ent, w.cb, w.ce, key, lane);
        const uint32_t j = hit.at;
        if (hit.tok == PPV_NO_SLOT || key > PPV_NODE_TOKEN) {
            // every member below child j sorts before the prefix; with no such child the prefix
            // sorts after the whole range of the current node
            const uint32_t rank = (j < w.ce) ? ix.node_lo[j] : ix.node_hi[w.node];
            w.lo = rank;
            w.hi = rank;
            w.slot = PPV_NO_SLOT;
            w.found = false;
            w.member = false;
            return w;
        }
        w.node = j;
        w.tok = hit.tok;
        w.cb = hit.child;
        w.ce = hit.next_child;
    }
    w.slot = SLOT ? heavy_slot_of(ix, w.node) : PPV_NO_SLOT;   // (with the ranks: where a caller asked for it after the walk it was a trip to memory more)
    w.lo = ix.node_lo[w.node];
    w.hi = ix.node_hi[w.node];
    w.member = (w.tok & PPV_NODE_TERMINAL) != 0u;
    return w;
}

// Hash of a token string: two sums over the tokens, H_d = sum_{i<=d} (tok_i + 1) * K^i mod 2^32 with two multipliers
// K, mixed into 64 bits at the end.  Sums, because a query needs the hashes of ALL its prefixes at once, lane d that of
// tokens 0..d: one multiplication per lane (by a power that is ready before the tokens have arrived) and one prefix
// sum over the wavefront give them.
constexpr uint32_t PREFIX_HASH_K1 = 0x9E3779B1u, PREFIX_HASH_K2 = 0x85EBCA77u;   // odd
struct PrefixHash {
    uint32_t h1, h2, p1, p2;   // the two sums and the two powers the next token is multiplied by
};
__device__ inline PrefixHash prefix_hash_empty() { return {0u, 0u, 1u, 1u}; }
__device__ inline void prefix_hash_add(PrefixHash &x, uint32_t tok) {
    x.h1 += (tok + 1u) * x.p1;
    x.h2 += (tok + 1u) * x.p2;
    x.p1 *= PREFIX_HASH_K1;
    x.p2 *= PREFIX_HASH_K2;
}
template <uint32_t K> __device__ __forceinline__ uint32_t power_of(int n) {   // K^n, 0 <= n < 64
    uint32_t p = 1u, k = K;
#pragma unroll
    for (int bit = 1; bit < WAVE; bit <<= 1) {
        p *= (n & bit) ? k : 1u;
        k *= k;
    }
    return p;
}
__device__ inline void prefix_hash_finish(uint32_t h1, uint32_t h2, uint32_t size, uint32_t fp_mask, uint32_t *slot,
                                          uint32_t *fp) {
    uint64_t h = ((uint64_t)h1 << 32) | h2;
    h ^= h >> 32;
    h *= 0xD6E8FEB86659FD93ull;
    h ^= h >> 29;
    *slot = __umulhi((uint32_t)(h >> 32), size);
    *fp = ((uint32_t)h & fp_mask) | 1u;
}
// Locates the prefix.  With a look-up table every length of the prefix is probed at once (lane d hashes
// tokens 0..d; a bucket of four entries per trip, one trip nearly always); the deepest hit is checked exactly -- its node
// must have that depth and the first member under it must begin with these tokens -- and the descent then starts
// there: nothing is left to descend when the whole prefix is in the index, one failing step (which yields the rank)
// when it is not.  A hit that fails the check (a fingerprint collision) only costs the shortcut: the descent starts at
// the root.
// A prefix of one member only (nearly all of a set of long sequences) is found by the shortest such prefix of that member,
// whose entry names the member's rank: comparing the member's tokens, in the same trip that checks the hit, gives all
// there is to know -- rank range, membership, the next token -- without looking at a node.  NODE: the node itself is
// wanted (a cursor); it costs two more trips.
// What bounds it is the chain of loads that wait for each other: prefix, bucket, member's tokens (and the root's children
// where nothing was found).  Open addressing at half load, a node by node_at and its entry took 14.5 us for the masks of
// 1,024 prefixes (V = 256k) and 5.6 us for those of 128; 9.4 and 4.1 us this way.
// SLOT: the slot is wanted in the same trip as the ranks, by kernels that hand it over; kernels of a wavefront to a row ask for it where they
// need it, which is no more than the noise of these calls (us, with the slots of all / so, 4,096 rows: mask + sample over codes 9.7 / 9.5, V = 2,000
// bf16 13.4 / 13.1; ppv_sample_next 6.9 / 7.05, 10.3 / 10.2).
// `mine` = first_tokens(prefix, stride, lane), requested by the caller before the prefix's length is known.
__device__ inline int32_t first_tokens(const int32_t *__restrict__ prefix, int stride, int lane) {
    return (lane < stride) ? prefix[lane] : 0;
}
template <bool NODE = false, bool SLOT = true>
__device__ __forceinline__ Walk walk_prefix(const IndexView &ix, const int32_t *__restrict__ prefix, int32_t mine, int t,
                                            int lane) {
    uint32_t node = 0u, tok = 0u, cb = ix.ent[0].child, ce = ix.ent[1].child;   // where the descent starts: the root, or
    int depth = 0;                                                               // the deepest hit
    const uint32_t p1 = power_of<PREFIX_HASH_K1>(lane), p2 = power_of<PREFIX_HASH_K2>(lane);
    int tl = t < WAVE ? t : WAVE;
    tl = tl < ix.l_max ? tl : ix.l_max;   // nothing longer than the longest member is in the index
    if (ix.lookup_buckets != 0u && tl > 0) {
        uint32_t bucket, fp;
        prefix_hash_finish(wave_incl_scan(((uint32_t)mine + 1u) * p1), wave_incl_scan(((uint32_t)mine + 1u) * p2),
                           ix.lookup_buckets, ix.lookup_fp_mask, &bucket, &fp);
        uint32_t hit_x = 0u, hit_y = 0u, hit_z = 0u, hit_w = 0u;   // node or rank, fingerprint (0: none), at, extent
        if (lane < tl) {
            for (uint32_t n = 0; n < ix.lookup_buckets; n++) {   // ends at the first bucket with an empty entry
                typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                const u32x4 *at = (const u32x4 *)(ix.lookup + (size_t)bucket * LOOKUP_BUCKET);
                const u32x4 e0 = at[0], e1 = at[1], e2 = at[2], e3 = at[3];   // filled from the front; fingerprints are not 0
                const uint32_t is0 = e0.y == fp ? ~0u : 0u, is1 = e1.y == fp ? ~is0 : 0u, not01 = ~(is0 | is1);
                const uint32_t is2 = e2.y == fp ? not01 : 0u, is3 = e3.y == fp ? not01 & ~is2 : 0u;   // the first that agrees
                hit_x = (e0.x & is0) | (e1.x & is1) | (e2.x & is2) | (e3.x & is3);
                hit_z = (e0.z & is0) | (e1.z & is1) | (e2.z & is2) | (e3.z & is3);
                hit_w = (e0.w & is0) | (e1.w & is1) | (e2.w & is2) | (e3.w & is3);
                hit_y = is0 | is1 | is2 | is3;
                if (hit_y != 0u || e3.y == 0u) break;
                bucket = bucket + 1u == ix.lookup_buckets ? 0u : bucket + 1u;
            }
        }
        const uint64_t hits = __ballot(hit_y != 0u);
        if (hits) {
            const int D = 63 - __clzll((long long)hits);   // deepest level with a hit: prefix length D + 1
            const uint32_t g = lane_value(hit_x, D), a = lane_value(hit_z, D), ext = lane_value(hit_w, D);
            if ((ext & 0xFFu) == (uint32_t)D + 1u) {   // a node of depth D+1: its first member has D+1 tokens or more
                const int len = (int)(ext >> 8);        // the member's length, if it is the only one (at most a wavefront's)
                if (len == 0) {
                    const bool same = lane > D || ix.x_tok[(size_t)a + lane] == mine;
                    const NodeEnt e0 = ix.ent[g], e1 = ix.ent[g + 1];
                    const uint32_t g_lo = ix.node_lo[g], g_hi = ix.node_hi[g], g_slot = SLOT ? heavy_slot_of(ix, g) : PPV_NO_SLOT;
                    if (__ballot(!same) == 0ull) {
                        if (D + 1 == t) {   // the whole prefix: nothing left to descend
                            Walk w;
                            w.node = g;
                            w.cb = e0.child;
                            w.ce = e1.child;
                            w.tok = e0.tok;
                            w.only = PPV_NO_SLOT;
                            w.slot = g_slot;
                            w.lo = g_lo;
                            w.hi = g_hi;
                            w.found = true;
                            w.member = (e0.tok & PPV_NODE_TERMINAL) != 0u;
                            return w;
                        }
                        node = g;
                        tok = e0.tok;
                        cb = e0.child;
                        ce = e1.child;
                        depth = D + 1;
                    }
                } else {
                    const int32_t x = lane < len ? ix.x_tok[(size_t)a + lane] : 0;
                    const uint64_t differ = __ballot(!(lane < len && lane < tl && x == mine));
                    const int m = differ ? __ffsll((long long)differ) - 1 : WAVE;   // tokens that agree
                    if (m > D) {
                        // (what a member or a prefix of a wavefront's length or more does beyond that is left to the descent)
                        if (!NODE && m < WAVE && (m < len || len < WAVE)) {
                            Walk w;
                            w.node = 0u;
                            w.cb = 0u;
                            w.slot = PPV_NO_SLOT;
                            w.found = m == t;
                            if (w.found) {
                                w.ce = m < len ? 1u : 0u;
                                w.only = m < len ? (uint32_t)lane_value((int)x, m) : PPV_NO_SLOT;
                                if (m + 1 == len && len < WAVE) w.only |= PPV_NODE_TERMINAL;
                                w.tok = m == len ? PPV_NODE_TERMINAL : 0u;
                                w.member = m == len;
                                w.lo = g;
                                w.hi = g + 1u;
                                if (m + 1 < WAVE || len < WAVE) return w;   // (else: whether the child ends the member is not known)
                            } else {   // the prefix leaves the member before it ends, or goes on behind its end
                                w.ce = 0u;
                                w.only = PPV_NO_SLOT;
                                w.tok = 0u;
                                w.member = false;
                                const bool before = m < len && (uint32_t)lane_value(mine, m) < (uint32_t)lane_value((int)x, m);
                                w.lo = w.hi = before ? g : g + 1u;
                                return w;
                            }
                        }
                        node = ix.node_at[(size_t)a + m - 1];
                        tok = ix.ent[node].tok;
                        cb = ix.ent[node].child;
                        ce = ix.ent[node + 1].child;
                        depth = m;
                    }
                }
            }
        }
    }
    return walk_from<SLOT>(ix, prefix, t, lane, mine, depth, node, tok, cb, ce);
}

}  // namespace
