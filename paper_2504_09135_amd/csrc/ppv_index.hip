// Index construction on the device (Algorithm 2, "Prepare"; Section 3.2 "Array Preparation"),
// plus sizes, export, files and release.
//
// The host hands over S as CSR (packed and checked on the way to the device, ppv_pool.hip); the rest runs in kernels:
//   1. sort the rows lexicographically -- token order = integer order, left to right, a sequence that ends sorts
//      before its extensions.  A row's first tokens, as many as fit, make a 64-bit key (token + 1, or 0 past the
//      row's end, most significant first); the keys are radix-sorted.  Rows with equal keys are neighbours then: groups
//      of up to about a thousand of them are ordered by counting, for each row, the rows of its group whose next key is
//      smaller, and the few that agree in that one too token by token; more than a few are counted again by the key after
//      it, and groups beyond a thousand take a radix sort by their rows' next tokens together with the group's number;
//   2. longest common prefix of neighbouring sorted rows; duplicates dropped (S is a set);
//   3. number the prefixes breadth-first.  Row r opens a new prefix of length d+1 iff it is longer than d and shares
//      at most d tokens with the row before it.  One wavefront takes 64 rows, a lane each: a ballot per depth counts
//      what the rows open there, one exclusive scan over (depth, 64 rows) gives every count's first number, and the
//      ballots again give each row its place;
//   4. the same wavefronts write the prefixes' entries, children, rank ranges and look-up entries;
//   5. images and per-word child counts of the heavy prefixes.
//
// What bounds it: for 1M sequences of 18M tokens the arrays are 0.5 GB (0.1 ms at 5 TB/s).  The radix sort over all
// columns that stood here before made 64 passes of five launches over the rows (3.8 ms) and one look-up entry per
// prefix, 17M atomics on a 270 MB table (1.5 ms); see step 4 for which prefixes need an entry.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <new>

#include <cstdlib>

#include "ppv_device.h"
#include "ppv_internal.h"
#include "ppv_walk.h"

extern "C" const char *ppv_status_string(ppv_status s) {
    switch (s) {
        case PPV_OK: return "PPV_OK";
        case PPV_EINVAL: return "PPV_EINVAL: invalid argument";
        case PPV_ENOMEM: return "PPV_ENOMEM: out of memory";
        case PPV_EDEVICE: return "PPV_EDEVICE: HIP call failed";
        case PPV_ERANGE: return "PPV_ERANGE: size beyond what the library supports";
        case PPV_EIO: return "PPV_EIO: file could not be opened, read or written";
    }
    return "unknown ppv_status";
}

namespace {

constexpr int BT = 256;            // threads per workgroup of the build kernels
constexpr int BW = BT / WAVE;      // wavefronts
constexpr int SCAN_ITEMS = 8;      // consecutive items per thread in the scans
constexpr int SCAN_CHUNK = BT * SCAN_ITEMS;
constexpr int SORT_ITEMS = 8;      // keys per thread in a radix pass
constexpr int SORT_CHUNK = BT * SORT_ITEMS;
constexpr int RADIX = 256;
static_assert(RADIX == BT, "one thread per digit in the radix kernels");

#define TRY(x)                          \
    do {                                \
        ppv_status s_ = (x);            \
        if (s_ != PPV_OK) return s_;    \
    } while (0)

inline unsigned blocks_for(uint64_t n) { return (unsigned)((n + BT - 1) / BT); }

// ------------------------------------------------------------------------------------------
// Exclusive scan of f(0..n-1) (sums that the callers keep inside V).
// Three launches: per-chunk sums, scan of the chunk sums by one workgroup, per-chunk scan + base.
template <typename V> __device__ inline V block_exclusive_scan(V x, V *wave_tot, V *block_total) {
    // exclusive prefix of x over the workgroup's BT threads in thread order
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    const V incl = wave_incl_scan(x);
    if (lane == WAVE - 1) wave_tot[wave] = incl;
    __syncthreads();
    V before = 0, total = 0;
    for (int w = 0; w < BW; w++) {
        const V t = wave_tot[w];
        if (w < wave) before += t;
        total += t;
    }
    __syncthreads();
    *block_total = total;
    return before + incl - x;
}

template <typename V, typename F> __global__ __launch_bounds__(BT) void scan_chunk_sums(uint64_t n, F f, V *__restrict__ sums) {
    __shared__ V wave_tot[BW];
    const uint64_t base = (uint64_t)blockIdx.x * SCAN_CHUNK + (uint64_t)threadIdx.x * SCAN_ITEMS;
    V s = 0;
    for (int k = 0; k < SCAN_ITEMS; k++)
        if (base + k < n) s += f(base + k);
    s = wave_sum(s);
    if ((threadIdx.x & (WAVE - 1)) == 0) wave_tot[threadIdx.x / WAVE] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        V t = 0;
        for (int w = 0; w < BW; w++) t += wave_tot[w];
        sums[blockIdx.x] = t;
    }
}

// in place exclusive scan of m values by ONE workgroup; the grand total goes to *total
template <typename V> __global__ __launch_bounds__(BT) void scan_of_sums(V *__restrict__ sums, uint64_t m, V *__restrict__ total) {
    __shared__ V wave_tot[BW];
    V carry = 0;
    for (uint64_t b0 = 0; b0 < m; b0 += SCAN_CHUNK) {
        const uint64_t base = b0 + (uint64_t)threadIdx.x * SCAN_ITEMS;
        V v[SCAN_ITEMS], s = 0;
        for (int k = 0; k < SCAN_ITEMS; k++) {
            v[k] = (base + k < m) ? sums[base + k] : (V)0;
            s += v[k];
        }
        V tot;
        V ex = carry + block_exclusive_scan(s, wave_tot, &tot);
        for (int k = 0; k < SCAN_ITEMS; k++) {
            if (base + k < m) sums[base + k] = ex;
            ex += v[k];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) *total = carry;
}

template <typename V, typename F>
__global__ __launch_bounds__(BT) void scan_apply(uint64_t n, F f, const V *__restrict__ sums, V *out) {
    __shared__ V wave_tot[BW];
    const uint64_t base = (uint64_t)blockIdx.x * SCAN_CHUNK + (uint64_t)threadIdx.x * SCAN_ITEMS;
    V v[SCAN_ITEMS], s = 0;
    for (int k = 0; k < SCAN_ITEMS; k++) {
        v[k] = (base + k < n) ? f(base + k) : (V)0;
        s += v[k];
    }
    V tot;
    V ex = sums[blockIdx.x] + block_exclusive_scan(s, wave_tot, &tot);
    for (int k = 0; k < SCAN_ITEMS; k++) {
        if (base + k < n) out[base + k] = ex;
        ex += v[k];
    }
}

// out[i] = sum of f(0..i-1) for i in [0, n); *d_total = sum of all.  sums: scratch of scan_words(n) values.
// f may read `out` only at the index it is asked for (a scan in place).
inline size_t scan_words(uint64_t n) { return (size_t)((n + SCAN_CHUNK - 1) / SCAN_CHUNK + 1); }
template <typename V, typename F>
ppv_status exclusive_scan(uint64_t n, F f, V *out, V *sums, V *d_total, hipStream_t st) {
    const uint64_t nb = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    if (nb > 0) hipLaunchKernelGGL((scan_chunk_sums<V, F>), dim3((unsigned)nb), dim3(BT), 0, st, n, f, sums);
    hipLaunchKernelGGL(scan_of_sums<V>, dim3(1), dim3(BT), 0, st, sums, nb, d_total);
    if (nb > 0) hipLaunchKernelGGL((scan_apply<V, F>), dim3((unsigned)nb), dim3(BT), 0, st, n, f, (const V *)sums, out);
    PPV_HIP_TRY(hipGetLastError());
    return PPV_OK;
}
template <typename V> struct ValueAt {
    const V *p;
    __device__ V operator()(uint64_t i) const { return p[i]; }
};

// ------------------------------------------------------------------------------------------
// S as it is on the device during a build: tokens in packed form, and rows by offset.
struct PackedTokens {
    const uint16_t *lo;
    const uint8_t *hi;   // nullptr: every token fits 16 bits
    __device__ uint32_t operator[](size_t i) const { return hi ? ((uint32_t)hi[i] << 16) | lo[i] : (uint32_t)lo[i]; }
};
struct FlatTokens {      // a loaded file's
    const int32_t *t;
    __device__ uint32_t operator[](size_t i) const { return (uint32_t)t[i]; }
};
struct KeyShape {
    int bits;    // per token: keys run over 0 .. vocab
    int slots;   // tokens per key
};
__device__ inline uint64_t row_key(const PackedTokens &tok, uint32_t a, uint32_t len, uint32_t from, KeyShape ks) {
    uint64_t k = 0;
    for (int s = 0; s < ks.slots; s++) {
        const uint32_t d = from + (uint32_t)s;
        k = (k << ks.bits) | (d < len ? tok[a + d] + 1u : 0u);   // 0: the row has ended; sorts first
    }
    return k;
}

// ------------------------------------------------------------------------------------------
// 1. sort
__global__ __launch_bounds__(BT) void first_keys(PackedTokens tok, const uint32_t *__restrict__ off, uint32_t n, KeyShape ks,
                                                 uint64_t *__restrict__ key, uint32_t *__restrict__ row) {
    const uint32_t i = blockIdx.x * BT + threadIdx.x;
    if (i >= n) return;
    const uint32_t a = off[i];
    key[i] = row_key(tok, a, off[i + 1] - a, 0u, ks);
    row[i] = i;
}

// One pass of a stable radix sort of (key, row) pairs by eight bits of the key: how often every workgroup's chunk
// holds each digit (digit-major) ...
__global__ __launch_bounds__(BT) void radix_count(const uint64_t *__restrict__ key, uint32_t n, int shift,
                                                  uint32_t *__restrict__ hist, uint32_t n_chunks) {
    __shared__ uint32_t h[RADIX];
    h[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t start = blockIdx.x * SORT_CHUNK;
    uint32_t d[SORT_ITEMS];
#pragma unroll
    for (int j = 0; j < SORT_ITEMS; j++) {
        const uint32_t i = start + j * BT + threadIdx.x;
        d[j] = i < n ? (uint32_t)(key[i] >> shift) & (RADIX - 1) : RADIX;
    }
#pragma unroll
    for (int j = 0; j < SORT_ITEMS; j++)
        if (d[j] < RADIX) atomicAdd(&h[d[j]], 1u);
    __syncthreads();
    hist[(size_t)threadIdx.x * n_chunks + blockIdx.x] = h[threadIdx.x];
}
// ... for each digit (a workgroup each) what the chunks before hold of it, in place, and its total ...
__global__ __launch_bounds__(BT) void radix_before(uint32_t *__restrict__ hist, uint32_t n_chunks, uint32_t *__restrict__ total) {
    __shared__ uint32_t wave_tot[BW];
    uint32_t *h = hist + (size_t)blockIdx.x * n_chunks;
    uint32_t carry = 0;
    for (uint32_t c0 = 0; c0 < n_chunks; c0 += BT) {
        const uint32_t c = c0 + threadIdx.x;
        const uint32_t v = c < n_chunks ? h[c] : 0u;
        uint32_t tot;
        const uint32_t ex = carry + block_exclusive_scan(v, wave_tot, &tot);
        if (c < n_chunks) h[c] = ex;
        carry += tot;
    }
    if (threadIdx.x == 0) total[blockIdx.x] = carry;
}
// ... and every pair to its place.  A wavefront ranks its 512 consecutive keys among themselves, 64 at a time: the
// lanes with the same digit by ballots, after those of the 64s before (a counter per wavefront and digit in LDS).
__global__ __launch_bounds__(BT) void radix_move(const uint64_t *__restrict__ key, const uint32_t *__restrict__ row, uint32_t n,
                                                 int shift, const uint32_t *__restrict__ hist,
                                                 const uint32_t *__restrict__ total, uint32_t n_chunks,
                                                 uint64_t *__restrict__ key_out, uint32_t *__restrict__ row_out) {
    __shared__ uint32_t cnt[BW][RADIX];
    __shared__ uint32_t wave_tot[BW];
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    for (int w = 0; w < BW; w++) cnt[w][threadIdx.x] = 0;
    __syncthreads();
    const uint32_t start = blockIdx.x * SORT_CHUNK + wave * (SORT_ITEMS * WAVE) + lane;
    uint64_t k[SORT_ITEMS];
    uint32_t r[SORT_ITEMS], rank[SORT_ITEMS];
#pragma unroll
    for (int j = 0; j < SORT_ITEMS; j++) {
        const uint32_t i = start + j * WAVE;
        k[j] = i < n ? key[i] : 0ull;
        r[j] = i < n ? row[i] : 0u;
    }
#pragma unroll
    for (int j = 0; j < SORT_ITEMS; j++) {
        const bool valid = start + j * WAVE < n;
        const uint32_t d = (uint32_t)(k[j] >> shift) & (RADIX - 1);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; b++) {
            const uint64_t bal = __ballot((d >> b) & 1u);
            peers &= ((d >> b) & 1u) ? bal : ~bal;
        }
        const int leader = peers ? __ffsll((long long)peers) - 1 : 0;
        uint32_t before = 0;
        if (valid && lane == leader) before = atomicAdd(&cnt[wave][d], (uint32_t)__popcll(peers));
        before = (uint32_t)__shfl((int)before, leader, WAVE);
        rank[j] = before + (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
    }
    __syncthreads();
    {   // counts -> first places, per wavefront and digit (thread = digit)
        uint32_t tot;
        uint32_t at = block_exclusive_scan(total[threadIdx.x], wave_tot, &tot) + hist[(size_t)threadIdx.x * n_chunks + blockIdx.x];
        for (int w = 0; w < BW; w++) {
            const uint32_t c = cnt[w][threadIdx.x];
            cnt[w][threadIdx.x] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < SORT_ITEMS; j++)
        if (start + j * WAVE < n) {
            const uint32_t at = cnt[wave][(uint32_t)(k[j] >> shift) & (RADIX - 1)] + rank[j];
            key_out[at] = k[j];
            row_out[at] = r[j];
        }
}

// sorts (key, row)[n] by the lowest `bits` bits of the keys; the pairs of buffers take turns, the result ends in the first
ppv_status radix_sort(uint64_t *&key, uint64_t *&key2, uint32_t *&row, uint32_t *&row2, uint32_t n, int bits,
                      uint32_t *hist, uint32_t *total, hipStream_t st) {
    const uint32_t nb = (n + SORT_CHUNK - 1) / SORT_CHUNK;
    for (int shift = 0; shift < bits; shift += 8) {
        hipLaunchKernelGGL(radix_count, dim3(nb), dim3(BT), 0, st, (const uint64_t *)key, n, shift, hist, nb);
        hipLaunchKernelGGL(radix_before, dim3(RADIX), dim3(BT), 0, st, hist, nb, total);
        hipLaunchKernelGGL(radix_move, dim3(nb), dim3(BT), 0, st, (const uint64_t *)key, (const uint32_t *)row, n, shift,
                           (const uint32_t *)hist, (const uint32_t *)total, nb, key2, row2);
        std::swap(key, key2);
        std::swap(row, row2);
    }
    PPV_HIP_TRY(hipGetLastError());
    return PPV_OK;
}

// Groups of rows whose tokens compared so far are equal: a byte per sorted position, and heads behind the last.
constexpr int GROUP_PAD = 16;
constexpr uint8_t GROUP_HEAD = 1;   // the first of its group
constexpr uint8_t GROUP_DONE = 2;   // nothing left to order in this group (the rows have ended: they are duplicates)
// Rows of a group are ordered by counting up to this size: size^2 comparisons of two 64-bit words that lie together.
// (The largest group after four tokens of the 1M-sequence Zipf sets: about 500 rows.)
constexpr uint32_t GROUP_COUNT = 1024;
// Rows that agree in the next key too are compared token by token as long as there are no more than this many of them; more
// stay a group for a further round.  A round (a trip to the host and two launches) costs about as much as a row comparing
// three tokens with twenty others, one after the other.  Comparing whole groups that way took 52 to 78 ms instead of 8 for
// 500k rows that share long stems, or are copies of a thousand rows.
constexpr uint32_t GROUP_TOKENS = 16;

__global__ __launch_bounds__(BT) void mark_groups(const uint64_t *__restrict__ key, uint32_t n, uint64_t last_slot,
                                                  uint8_t *__restrict__ group, uint8_t *__restrict__ group2) {
    const uint32_t i = blockIdx.x * BT + threadIdx.x;
    if (i < GROUP_PAD) group[n + i] = group2[n + i] = GROUP_HEAD;
    if (i >= n) return;
    const uint64_t k = key[i];
    group[i] = (uint8_t)(((i == 0u || key[i - 1] != k) ? GROUP_HEAD : 0) | ((k & last_slot) == 0ull ? GROUP_DONE : 0));
}
__device__ inline bool unsettled(const uint8_t *__restrict__ group, uint32_t i, uint32_t n) {
    const uint8_t g = group[i];
    if (g & GROUP_DONE) return false;
    return !(g & GROUP_HEAD) || (i + 1 < n && !(group[i + 1] & GROUP_HEAD));
}
// the next key of the rows that are still to be ordered
__global__ __launch_bounds__(BT) void next_keys(PackedTokens tok, const uint32_t *__restrict__ off,
                                                const uint32_t *__restrict__ row, const uint8_t *__restrict__ group, uint32_t n,
                                                uint32_t depth, KeyShape ks, uint64_t *__restrict__ key) {
    const uint32_t i = blockIdx.x * BT + threadIdx.x;
    if (i >= n || !unsettled(group, i, n)) return;
    const uint32_t r = row[i], a = off[r];
    key[i] = row_key(tok, a, off[r + 1] - a, depth, ks);
}
// Orders the rows of every group of at most GROUP_COUNT, up to groups of more than GROUP_TOKENS that agree in this key too;
// left[0], left[1]: rows in larger groups, and rows in such groups.  depth: tokens that `group` and `key` together have
// covered; complete: no row is longer.
__global__ __launch_bounds__(BT) void order_groups(PackedTokens tok, const uint32_t *__restrict__ off,
                                                   const uint32_t *__restrict__ row, const uint8_t *__restrict__ group,
                                                   const uint64_t *__restrict__ key, uint32_t n, uint32_t depth,
                                                   uint64_t last_slot, int complete, uint32_t *__restrict__ row_out,
                                                   uint8_t *__restrict__ group_out, uint32_t *__restrict__ left) {
    constexpr uint32_t most = GROUP_COUNT;
    const uint32_t i = blockIdx.x * BT + threadIdx.x;
    bool large = false, split = false;
    if (i < n) {
        const uint32_t r = row[i];
        uint8_t g = group[i];
        uint32_t to = i;
        if (unsettled(group, i, n)) {
            // the group's bounds, eight positions at a time
            uint32_t a = i, b = i + 1;
            const uint64_t heads = 0x0101010101010101ull * GROUP_HEAD;
            if (!(g & GROUP_HEAD)) {
                uint32_t w = i >> 3;   // (the bytes at and above i are not looked at)
                uint64_t f = *(const uint64_t *)(group + 8ull * w) & heads & ((1ull << (8 * (i & 7u))) - 1ull);
                while (f == 0ull && i - 8u * w <= most) f = *(const uint64_t *)(group + 8ull * --w) & heads;   // position 0 is a head
                a = f ? 8u * w + (uint32_t)(63 - __clzll((long long)f)) / 8u : 0u;
                large = f == 0ull;
            }
            while (b < n && (b & 7u) && !(group[b] & GROUP_HEAD)) b++;
            if (b < n && !(b & 7u)) {
                uint64_t f = *(const uint64_t *)(group + b) & heads;   // (bytes behind the last position: heads)
                while (f == 0ull && b - i <= most) f = *(const uint64_t *)(group + (b += 8u)) & heads;
                if (f) b += (uint32_t)(__ffsll((long long)f) - 1) / 8u;
                if (b > n) b = n;
            }
            if (!large && b - a <= most) {
                const uint64_t k = key[i];
                uint32_t before = 0, equal = 0;
#pragma unroll 8
                for (uint32_t j = a; j < b; j++) {
                    const uint64_t kj = key[j];
                    before += kj < k ? 1u : 0u;
                    equal += kj == k ? 1u : 0u;
                }
                g = GROUP_HEAD | GROUP_DONE;
                if (equal > GROUP_TOKENS && !complete && (k & last_slot) != 0ull) {   // a group of their own, in the order they are in
                    uint32_t ahead = 0;
                    for (uint32_t j = a; j < i; j++) ahead += key[j] == k ? 1u : 0u;
                    before += ahead;
                    split = true;
                    g = ahead == 0u ? GROUP_HEAD : (uint8_t)0;
                } else if (equal > 1u) {   // rows that agree in this key too: token by token
                    const uint32_t ra = off[r], rl = off[r + 1] - ra;
                    for (uint32_t j = a; j < b; j++) {
                        if (j == i || key[j] != k) continue;
                        int order = 0;   // of row j against row i; -1: before
                        if ((k & last_slot) != 0ull) {
                            const uint32_t q = row[j], qa = off[q], ql = off[q + 1] - qa;
                            const uint32_t m = rl < ql ? rl : ql;
                            uint32_t d = depth;
                            while (d < m && tok[ra + d] == tok[qa + d]) d++;
                            if (d < m) order = tok[qa + d] < tok[ra + d] ? -1 : 1;
                            else order = ql < rl ? -1 : (ql > rl ? 1 : 0);
                        }
                        before += (order < 0 || (order == 0 && j < i)) ? 1u : 0u;
                    }
                }
                to = a + before;
            } else {
                large = true;
            }
        }
        row_out[to] = r;
        group_out[to] = g;
    }
    const uint64_t is_large = __ballot(large), is_split = __ballot(split);
    if ((threadIdx.x & (WAVE - 1)) == 0) {
        if (is_large) atomicAdd(&left[0], (uint32_t)__popcll(is_large));
        if (is_split) atomicAdd(&left[1], (uint32_t)__popcll(is_split));
    }
}
// what is left after order_groups: rows of it before each position | groups of it up to there
struct LargeRows {
    const uint8_t *group;
    uint32_t n;
    __device__ uint64_t operator()(uint64_t i) const {
        if (!unsettled(group, (uint32_t)i, n)) return 0ull;
        return (1ull << 32) | ((group[i] & GROUP_HEAD) ? 1ull : 0ull);
    }
};
// their rows with the next key under the group's number
__global__ __launch_bounds__(BT) void large_keys(PackedTokens tok, const uint32_t *__restrict__ off,
                                                 const uint32_t *__restrict__ row, const uint8_t *__restrict__ group,
                                                 const uint64_t *__restrict__ before, uint32_t n, uint32_t depth, KeyShape ks,
                                                 uint64_t *__restrict__ key, uint32_t *__restrict__ at_row,
                                                 uint32_t *__restrict__ place) {
    const uint32_t i = blockIdx.x * BT + threadIdx.x;
    if (i >= n || !unsettled(group, i, n)) return;
    const uint32_t j = (uint32_t)(before[i] >> 32);
    const uint64_t num = (before[i] & 0xFFFFFFFFull) - ((group[i] & GROUP_HEAD) ? 0ull : 1ull);
    const uint32_t r = row[i], a = off[r];
    key[j] = (num << (ks.bits * ks.slots)) | row_key(tok, a, off[r + 1] - a, depth, ks);
    at_row[j] = r;
    place[j] = i;
}
__global__ __launch_bounds__(BT) void large_back(const uint64_t *__restrict__ key, const uint32_t *__restrict__ at_row,
                                                 const uint32_t *__restrict__ place, uint32_t m, uint64_t last_slot,
                                                 int complete, uint32_t *__restrict__ row, uint8_t *__restrict__ group) {
    const uint32_t j = blockIdx.x * BT + threadIdx.x;
    if (j >= m) return;
    const uint64_t k = key[j];
    row[place[j]] = at_row[j];
    group[place[j]] = (uint8_t)(((j == 0u || key[j - 1] != k) ? GROUP_HEAD : 0) |
                                ((complete || (k & last_slot) == 0ull) ? GROUP_DONE : 0));
}

// ------------------------------------------------------------------------------------------
// 2. common prefix with the previous sorted row; duplicates.  info: common prefix, 0xFFFFFFFF for a duplicate.
constexpr uint32_t DUPLICATE = 0xFFFFFFFFu;
__global__ __launch_bounds__(BT) void neighbour_lcp(PackedTokens tok, const uint32_t *__restrict__ off,
                                                    const uint32_t *__restrict__ row, uint32_t n, uint32_t *__restrict__ info,
                                                    uint64_t *__restrict__ kept) {
    const uint32_t i = blockIdx.x * BT + threadIdx.x;
    if (i >= n) return;
    const uint32_t r = row[i], a = off[r], la = off[r + 1] - a;
    uint32_t c = 0, lb = 0;
    if (i > 0) {
        const uint32_t q = row[i - 1], b = off[q];
        lb = off[q + 1] - b;
        const uint32_t m = la < lb ? la : lb;
        while (c < m && tok[a + c] == tok[b + c]) c++;
    }
    const bool dup = i > 0 && c == la && c == lb;
    info[i] = dup ? DUPLICATE : c;
    kept[i] = dup ? 0ull : (1ull << 32) | la;   // rows | tokens: scanned together
}
// what the later steps know of a row of the index
struct RowMeta {
    uint32_t at;    // where its tokens start in the sorted S
    uint32_t src;   // ... and in the tokens it was given in
    uint32_t lcp;   // tokens shared with the row before
    uint32_t len;
};
__global__ __launch_bounds__(BT) void compact_rows(const uint32_t *__restrict__ off, const uint32_t *__restrict__ row, uint32_t n,
                                                   const uint32_t *__restrict__ info, const uint64_t *__restrict__ place,
                                                   RowMeta *__restrict__ rows) {
    const uint32_t i = blockIdx.x * BT + threadIdx.x;
    if (i >= n || info[i] == DUPLICATE) return;
    const uint32_t r = row[i];
    RowMeta m;
    m.at = (uint32_t)place[i];
    m.src = off[r];
    m.lcp = info[i];
    m.len = off[r + 1] - m.src;
    rows[place[i] >> 32] = m;
}

// ------------------------------------------------------------------------------------------
// 3. how many prefixes each 64 rows open at each depth (depth-major), how many of them get a look-up entry (behind
// the last depth), and the smallest common prefix of the 64.
//
// Look-up entries.  A prefix of one member only -- "alone": nearly all prefixes of long members -- needs no entry of its
// own: the first alone prefix of a row (its "head") has one, and from there the row's tokens are compared and its
// prefixes' numbers read off (node_at).  So a row gets entries for the prefixes it opens up to its head.  Prefixes
// longer than a wavefront are never looked up.
__device__ inline uint32_t shared_len(uint32_t lcp, uint32_t next_lcp) { return lcp > next_lcp ? lcp : next_lcp; }
__device__ inline uint32_t last_entry(uint32_t shared, uint32_t len) {   // longest prefix of the row with an entry
    uint32_t e = shared + 1u;
    e = e < (uint32_t)WAVE ? e : (uint32_t)WAVE;
    return e < len ? e : len;
}
__global__ __launch_bounds__(BT) void count_prefixes(const RowMeta *__restrict__ rows, const uint64_t *__restrict__ totals,
                                                     uint32_t n_groups, int32_t l_max, uint32_t *__restrict__ counts,
                                                     uint32_t *__restrict__ group_lcp) {
    const uint32_t n_rows = (uint32_t)(totals[0] >> 32);
    const int lane = threadIdx.x & (WAVE - 1);
    const uint32_t c = blockIdx.x * BW + threadIdx.x / WAVE;
    if (c >= n_groups) return;   // uniform per wavefront
    const uint32_t r = c * WAVE + lane;
    uint32_t lcp = 0xFFFFFFFFu, len = 0u, next = 0u;
    if (r < n_rows) {
        lcp = rows[r].lcp;
        len = rows[r].len;
        if (r + 1 < n_rows) next = rows[r + 1].lcp;
    }
    const uint32_t entries = r < n_rows && last_entry(shared_len(lcp, next), len) > lcp ? last_entry(shared_len(lcp, next), len) - lcp : 0u;
    const uint32_t n_entries = wave_sum(entries);
    const uint32_t lowest = ~wave_max(~lcp);
    if (lane == 0) {
        counts[(size_t)l_max * n_groups + c] = n_entries;
        group_lcp[c] = lowest;
    }
    const uint32_t longest = wave_max(len), depths = (uint32_t)l_max;
    for (uint32_t d0 = 0; d0 < depths; d0 += WAVE) {   // (unsigned: the step past the longest row there can be is no overflow)
        uint32_t mine = 0u;
        const uint32_t d1 = d0 + WAVE < longest ? d0 + WAVE : longest;
        for (uint32_t d = d0; d < d1; d++) {
            const uint32_t opened = (uint32_t)__popcll(__ballot(lcp <= d && d < len));
            if ((uint32_t)lane == d - d0) mine = opened;
        }
        if (d0 + lane < depths) counts[(size_t)(d0 + lane) * n_groups + c] = mine;
    }
}

// 4. entries, children, rank ranges, look-up entries
struct TrieOut {
    NodeEnt *ent;
    uint32_t *node_lo, *node_hi;
    int32_t *x_tok;
    int64_t *x_off;
    uint32_t *node_at;        // (with a look-up table) number of the alone prefix that ends at this token of the sorted S
    LookupEntry *table;       // nullptr: none
    uint32_t buckets, fp_mask;
};
__device__ inline void insert_entry(const TrieOut &o, const PrefixHash &h, uint32_t node, uint32_t at, uint32_t extent) {
    uint32_t bucket, fp;
    prefix_hash_finish(h.h1, h.h2, o.buckets, o.fp_mask, &bucket, &fp);
    const unsigned long long key = ((unsigned long long)fp << 32) | node;
    for (uint32_t n = 0; n < o.buckets; n++) {   // the table has four times as many places as entries
        LookupEntry *e = o.table + (size_t)bucket * LOOKUP_BUCKET;
        for (uint32_t k = 0; k < LOOKUP_BUCKET; k++)
            if (atomicCAS((unsigned long long *)&e[k].key, 0ull, key) == 0ull) {
                e[k].at = at;
                e[k].extent = extent;
                return;
            }
        bucket = bucket + 1u == o.buckets ? 0u : bucket + 1u;
    }
}
// The tokens of 64 rows are one stretch of the sorted S.  They are gathered into LDS, 16 lanes to a row, and written from
// there; the loop over the depths finds them there and leaves the alone prefixes' numbers in their places, which go
// out as one stretch again.  (Token by token from and to memory, with a lane per row, the kernel took 513 us for 1M
// sequences instead of 218, and gathering the tokens 55 us more.)  `room`: words of LDS per wavefront; rows that need
// more are read from and written to memory as they come.
template <typename TOK>
__global__ __launch_bounds__(BT) void fill_prefixes(TOK tok, const RowMeta *__restrict__ rows, uint32_t n_rows,
                                                    const uint32_t *__restrict__ base, uint32_t n_groups,
                                                    const uint32_t *__restrict__ group_lcp, int32_t l_max, uint32_t n_nodes,
                                                    uint32_t room, TrieOut o) {
    extern __shared__ uint32_t stage_lds[];
    const int lane = threadIdx.x & (WAVE - 1);
    const uint32_t c = blockIdx.x * BW + threadIdx.x / WAVE;
    const uint32_t r = c * WAVE + lane;
    if (c * WAVE >= n_rows) return;   // uniform per wavefront
    uint32_t *st = stage_lds + (threadIdx.x / WAVE) * room;
    if (c == 0 && lane == 0) {        // the empty prefix and the closing sentinel
        o.ent[0].tok = 0u;
        o.ent[0].child = 1u;
        o.node_lo[0] = 0u;
        o.node_hi[0] = n_rows;
        o.ent[n_nodes].tok = PPV_NODE_TOKEN;
        o.ent[n_nodes].child = n_nodes;
    }
    RowMeta m = {0u, 0u, 0xFFFFFFFFu, 0u};
    uint32_t next_lcp = 0u;   // of the row after this one
    if (r < n_rows) {
        m = rows[r];
        if (r + 1 < n_rows) next_lcp = rows[r + 1].lcp;
        o.x_off[r] = m.at;
        if (r + 1 == n_rows) o.x_off[n_rows] = (int64_t)m.at + m.len;
    }
    // numbers of the first prefixes these rows open at depths 0 .. 63 (lane = depth), and so on for the next 64
    const uint32_t depths = (uint32_t)l_max;
    auto firsts = [&](uint32_t d0) {
        const uint32_t d = d0 + (uint32_t)lane;
        return d <= depths ? base[(size_t)d * n_groups + (d < depths ? c : 0u)] : 0u;   // behind the last depth: all prefixes
    };
    uint32_t first_at = firsts(0u);
    const uint32_t at0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)m.at);
    const uint32_t span = wave_max(r < n_rows ? m.at + m.len - at0 : 0u);
    const bool staged = span <= room;
    if (staged) {
        constexpr int L = 16, ROWS = WAVE / L, BATCH = 4;   // lanes to a row, rows at a time, times whose loads go out together
        const uint32_t k0 = lane % L;
        for (int j0 = 0; j0 < WAVE; j0 += ROWS * BATCH) {
            uint32_t src[BATCH], at[BATCH], len[BATCH], v[BATCH][2];
#pragma unroll
            for (int q = 0; q < BATCH; q++) {
                const int from = j0 + q * ROWS + lane / L;
                src[q] = (uint32_t)__shfl((int)m.src, from, WAVE);
                at[q] = (uint32_t)__shfl((int)m.at, from, WAVE) - at0;
                len[q] = (uint32_t)__shfl((int)m.len, from, WAVE);
            }
#pragma unroll
            for (int q = 0; q < BATCH; q++)
#pragma unroll
                for (uint32_t h = 0; h < 2; h++) v[q][h] = k0 + h * L < len[q] ? tok[src[q] + k0 + h * L] : 0u;
#pragma unroll
            for (int q = 0; q < BATCH; q++) {
#pragma unroll
                for (uint32_t h = 0; h < 2; h++)
                    if (k0 + h * L < len[q]) st[at[q] + k0 + h * L] = v[q][h];
                for (uint32_t k = k0 + 2 * L; k < len[q]; k += L) st[at[q] + k] = tok[src[q] + k];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // other lanes' words from here on
        for (uint32_t i = lane; i < span; i += WAVE) o.x_tok[at0 + i] = (int32_t)st[i];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    const uint32_t shared = r < n_rows ? shared_len(m.lcp, next_lcp) : 0u;
    const uint32_t entries_to = o.table && r < n_rows ? last_entry(shared, m.len) : 0u;
    const uint32_t after = (uint32_t)__builtin_amdgcn_readlane((int)next_lcp, WAVE - 1);   // (of the row after these 64)
    const bool last_group = (c + 1) * WAVE >= n_rows;
    const uint64_t below = (1ull << lane) - 1ull;
    const uint32_t longest = wave_max(m.len);
    PrefixHash h = prefix_hash_empty();
    uint64_t opened = __ballot(m.lcp == 0u && m.len > 0u);
    uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first_at);
    for (uint32_t d = 0; d < longest; d++) {
        // what is opened one level down: the children of this level's prefixes
        const uint64_t opened_next = __ballot(m.lcp <= d + 1u && d + 1u < m.len);
        if (((d + 1u) & (WAVE - 1)) == 0u) first_at = firsts(d + 1u);
        const uint32_t first_next = lane_value(first_at, (int)((d + 1u) & (WAVE - 1)));
        const bool opens = m.lcp <= d && d < m.len;
        const bool hashes = d < entries_to && m.lcp < entries_to;
        uint32_t t = 0u;
        if (staged) {
            if (opens || hashes) t = st[m.at - at0 + d];
        } else if (d < m.len) {
            t = tok[m.src + d];
            o.x_tok[m.at + d] = (int32_t)t;
        }
        if (hashes) prefix_hash_add(h, t);
        // where the prefix's range ends: the next row that shares at most d tokens with the row before it
        const uint64_t breaks = __ballot(m.lcp <= d) & ~below & ~(1ull << lane);
        uint32_t hi = breaks ? c * WAVE + (uint32_t)__ffsll((long long)breaks) - 1u : n_rows;
        const bool open_end = opens && !breaks && !last_group;
        if (__ballot(open_end)) {   // (at most one lane) the range goes on behind these 64 rows
            uint32_t end = n_rows;
            if (after <= d) {
                end = (c + 1) * WAVE;
            } else {
                for (uint32_t q = c + 1; q < n_groups; q += WAVE) {
                    const bool found = q + lane < n_groups && group_lcp[q + lane] <= d;
                    const uint64_t bal = __ballot(found);
                    if (bal) {
                        const uint32_t g0 = (q + (uint32_t)__ffsll((long long)bal) - 1u) * WAVE;
                        const bool here = g0 + lane < n_rows && rows[g0 + lane].lcp <= d;
                        const uint64_t bal2 = __ballot(here);
                        if (bal2) end = g0 + (uint32_t)__ffsll((long long)bal2) - 1u;
                        break;
                    }
                }
            }
            if (open_end) hi = end;
        }
        if (opens) {
            const uint32_t g = 1u + first + (uint32_t)__popcll(opened & below);
            const bool ends = m.len == d + 1u;   // the opening row is the prefix itself
            // first child: the first prefix one token longer at or after this row (this row's if it goes on, else the
            // next row's); numbers run on from 64 rows to the next and from a depth to the next
            const uint64_t upto = ends ? below | (1ull << lane) : below;
            NodeEnt e;
            e.tok = ends ? t | PPV_NODE_TERMINAL : t;
            e.child = 1u + first_next + (uint32_t)__popcll(opened_next & upto);
            o.ent[g] = e;
            o.node_lo[g] = r;
            o.node_hi[g] = hi;
            if (o.table && d < (uint32_t)WAVE) {
                const bool alone = d >= shared;
                if (alone) {
                    if (staged) st[m.at - at0 + d] = g;
                    else o.node_at[m.at + d] = g;
                }
                if (d < entries_to)
                    insert_entry(o, h, alone ? r : g, m.at, (d + 1u) | (alone ? (m.len < (uint32_t)WAVE ? m.len : (uint32_t)WAVE) << 8 : 0u));
            }
        }
        opened = opened_next;
        first = first_next;
    }
    if (staged && o.table) {   // (places of prefixes that are not alone hold their tokens: they are not read)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (uint32_t i = lane; i < span; i += WAVE) o.node_at[at0 + i] = st[i];
    }
}

// 5. heavy prefixes
// how many each SCAN_CHUNK entries hold
__global__ __launch_bounds__(BT) void count_heavy(const NodeEnt *__restrict__ ent, uint32_t n_nodes, uint32_t heavy_min,
                                                  uint32_t *__restrict__ sums) {
    __shared__ uint32_t total;
    if (threadIdx.x == 0) total = 0u;
    __syncthreads();
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) {
        const uint64_t g = (uint64_t)blockIdx.x * SCAN_CHUNK + k * BT + threadIdx.x;
        if (g < n_nodes && ent[g + 1].child - ent[g].child > heavy_min) s++;
    }
    s = wave_sum(s);
    if ((threadIdx.x & (WAVE - 1)) == 0 && s) atomicAdd(&total, s);
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}
// second pass over the chunks that hold any: their numbers in increasing order, and their flags
__global__ __launch_bounds__(BT) void list_heavy(NodeEnt *__restrict__ ent, uint32_t n_nodes, uint32_t heavy_min,
                                                 const uint32_t *__restrict__ sums, const uint32_t *__restrict__ n_heavy,
                                                 uint32_t *__restrict__ heavy_node, uint32_t *__restrict__ heavy_limit) {
    __shared__ uint32_t wave_tot[BW];
    const uint32_t before = sums[blockIdx.x];
    if ((blockIdx.x + 1 < gridDim.x ? sums[blockIdx.x + 1] : *n_heavy) == before) return;   // uniform: none here
    const uint32_t base = blockIdx.x * SCAN_CHUNK + threadIdx.x * SCAN_ITEMS;
    uint32_t is = 0, count = 0;
    for (int k = 0; k < SCAN_ITEMS; k++)
        if (base + k < n_nodes && ent[base + k + 1].child - ent[base + k].child > heavy_min) {
            is |= 1u << k;
            count++;
        }
    uint32_t tot;
    uint32_t at = before + block_exclusive_scan(count, wave_tot, &tot);
    for (int k = 0; k < SCAN_ITEMS; k++)
        if ((is >> k) & 1u) {
            heavy_node[at++] = base + k;
            ent[base + k].tok |= PPV_NODE_HEAVY;
            atomicMax(heavy_limit, base + k + 1);
        }
}
// one workgroup per heavy prefix: its children into the image, the children before each word, its slot
constexpr int HT = 1024;
__global__ __launch_bounds__(HT) void fill_heavy(const NodeEnt *__restrict__ ent, const uint32_t *__restrict__ heavy_node,
                                                 const uint32_t *__restrict__ n_heavy, int n_words,
                                                 uint32_t *__restrict__ bits, uint32_t *__restrict__ rank,
                                                 uint32_t *__restrict__ heavy_slot, uint32_t reach) {
    extern __shared__ uint32_t img[];   // [n_words]
    __shared__ uint32_t wave_tot[HT / WAVE];
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    if (blockIdx.x >= *n_heavy) return;
    const uint32_t g = heavy_node[blockIdx.x];
    if (threadIdx.x == 0 && g < reach) heavy_slot[g] = blockIdx.x;
    for (int w = threadIdx.x; w < n_words; w += HT) img[w] = 0u;
    __syncthreads();
    for (uint32_t c = ent[g].child + threadIdx.x; c < ent[g + 1].child; c += HT) {
        const uint32_t v = ent[c].tok & PPV_NODE_TOKEN;
        atomicOr(&img[v >> 5], 1u << (v & 31u));
    }
    __syncthreads();
    uint32_t *b = bits + (size_t)blockIdx.x * (size_t)n_words;
    uint32_t *rk = rank + (size_t)blockIdx.x * (size_t)n_words;
    uint32_t carry = 0;
    for (int w0 = 0; w0 < n_words; w0 += HT) {
        const int w = w0 + threadIdx.x;
        const uint32_t word = w < n_words ? img[w] : 0u;
        const uint32_t c = (uint32_t)__popc(word), incl = wave_incl_scan(c);
        if (lane == WAVE - 1) wave_tot[wave] = incl;
        __syncthreads();
        uint32_t before = 0, total = 0;
        for (int k = 0; k < HT / WAVE; k++) {
            const uint32_t t = wave_tot[k];
            before += k < wave ? t : 0u;
            total += t;
        }
        __syncthreads();
        if (w < n_words) {
            b[w] = word;
            rk[w] = carry + before + incl - c;
        }
        carry += total;
    }
}

// ------------------------------------------------------------------------------------------
// A block of device memory from the pool, cut into arrays: sizes first (add), then the block (take), then addresses.
struct Arena {
    static constexpr int MOST = 32;
    void **slot[MOST];
    size_t at[MOST];
    int n = 0;
    size_t bytes = 0;
    void *block = nullptr;
    template <typename T> void add(T **p, uint64_t count) {
        slot[n] = (void **)p;
        at[n++] = bytes;
        bytes += ((size_t)(count ? count : 1) * sizeof(T) + 255) / 256 * 256;
    }
    ppv_status take() {   // (`bytes` is the block's size from here on)
        TRY(ppv_pool_take(&block, bytes, &bytes));
        for (int i = 0; i < n; i++) *slot[i] = (char *)block + at[i];
        return PPV_OK;
    }
    void *keep() {   // the block belongs to the caller from here on
        void *b = block;
        block = nullptr;
        return b;
    }
};
struct TempArena : Arena {   // given back at the end of the build, when everything that used it has finished
    ~TempArena() {
        if (!block) return;
        ppv_pool_give(block, hipStreamSynchronize(nullptr) == hipSuccess);
    }
};

// What the host has to know of a build under way, written by a kernel into pinned memory.
struct BuildWords {
    uint64_t rows_tokens;                 // rows << 32 | tokens, without duplicates
    uint32_t prefixes, all_counts;        // prefixes; prefixes and look-up entries
    uint32_t large, split;                // rows in groups too large to be ordered by counting; in groups that are to be counted again
    uint32_t heavy, heavy_limit;          // heavy prefixes, one past the last of them
};
static_assert(sizeof(BuildWords) <= PPV_HOST_WORDS_BYTES, "one slot of pinned words");
__global__ void publish(BuildWords *__restrict__ out, const uint64_t *__restrict__ rows_tokens, const uint32_t *__restrict__ prefixes,
                        const uint32_t *__restrict__ all_counts, const uint32_t *__restrict__ left) {
    out->rows_tokens = *rows_tokens;
    out->prefixes = *prefixes;
    out->all_counts = *all_counts;
    out->large = left[0];
    out->split = left[1];
}
__global__ void publish_heavy(BuildWords *__restrict__ out, const uint32_t *__restrict__ heavy) {
    out->heavy = heavy[0];
    out->heavy_limit = heavy[1];
}
struct HostWords {
    volatile BuildWords *w = (volatile BuildWords *)ppv_host_words_take();
    ~HostWords() { ppv_host_words_give((void *)w); }
    BuildWords *dev() const { return (BuildWords *)w; }   // (mapped at the same address)
};

// device words read back by the host; a synchronisation
template <typename T> ppv_status read_back(T *host, const void *dev, size_t count, hipStream_t st) {
    PPV_HIP_TRY(hipMemcpyAsync(host, dev, count * sizeof(T), hipMemcpyDeviceToHost, st));
    PPV_HIP_TRY(hipStreamSynchronize(st));
    return PPV_OK;
}

// 5. Images and per-word child counts of the heavy prefixes, from the finished entries (G of them plus the sentinel).
// Sets the heavy part of the index and of its view.  The index's block has room for HEAVY_GUESS of them (or for as many as
// there can be: with 60 sequences at V = 256,000 for one, 64 KB, where room for all would be 16 MB) among the first
// HEAVY_REACH prefixes, which are filled before the host knows how many there are; more than that (small
// vocabularies, where every second prefix is heavy) get a block of their own.  Ends with a synchronisation.
constexpr uint32_t HEAVY_GUESS = 256, HEAVY_REACH = 1u << 20;
inline uint32_t heavy_min_of(int32_t vocab) { return (uint32_t)std::min<int64_t>(vocab / 32, PPV_LIST_MAX); }
inline uint32_t heavy_at_most(uint32_t G, int32_t vocab) {   // of G prefixes: their children are disjoint
    return (uint32_t)std::max<uint64_t>((G - 1) / (heavy_min_of(vocab) + 1ull), 1);
}
ppv_status finish_heavy(ppv_index *ix, uint32_t G, int32_t vocab, const HostWords &words, hipStream_t st) {
    const int n_words = (vocab + 31) / 32;
    const uint32_t heavy_min = heavy_min_of(vocab), bound = heavy_at_most(G, vocab);
    const uint64_t chunks = ((uint64_t)G + SCAN_CHUNK - 1) / SCAN_CHUNK;
    TempArena tmp;
    uint32_t *sums, *d_heavy, *heavy_node;               // d_heavy: heavy prefixes, one past the last of them
    tmp.add(&sums, chunks + 1);
    tmp.add(&d_heavy, 2);
    tmp.add(&heavy_node, bound);
    TRY(tmp.take());
    PPV_HIP_TRY(hipMemsetAsync(d_heavy, 0, 2 * sizeof(uint32_t), st));
    hipLaunchKernelGGL(count_heavy, dim3((unsigned)chunks), dim3(BT), 0, st, (const NodeEnt *)ix->d_ent, G, heavy_min, sums);
    hipLaunchKernelGGL(scan_of_sums<uint32_t>, dim3(1), dim3(BT), 0, st, sums, chunks, d_heavy);
    hipLaunchKernelGGL(list_heavy, dim3((unsigned)chunks), dim3(BT), 0, st, ix->d_ent, G, heavy_min, (const uint32_t *)sums,
                       (const uint32_t *)d_heavy, heavy_node, d_heavy + 1);
    hipLaunchKernelGGL(publish_heavy, dim3(1), dim3(1), 0, st, words.dev(), (const uint32_t *)d_heavy);
    auto fill = [&](uint32_t most, uint32_t reach) {
        PPV_HIP_TRY(hipMemsetAsync(ix->d_heavy_slot, 0xFF, (size_t)reach * sizeof(uint32_t), st));   // PPV_NO_SLOT
        hipLaunchKernelGGL(fill_heavy, dim3(most), dim3(HT), (size_t)n_words * sizeof(uint32_t), st,
                           (const NodeEnt *)ix->d_ent, (const uint32_t *)heavy_node, (const uint32_t *)d_heavy, n_words,
                           ix->d_heavy_bits, ix->d_heavy_rank, ix->d_heavy_slot, reach);
        PPV_HIP_TRY(hipGetLastError());
        PPV_HIP_TRY(hipStreamSynchronize(st));
        return PPV_OK;
    };
    TRY(fill(std::min(HEAVY_GUESS, bound), std::min(G, HEAVY_REACH)));
    const uint32_t n_heavy = words.w->heavy, limit = words.w->heavy_limit;
    if (n_heavy > HEAVY_GUESS || limit > HEAVY_REACH) {
        Arena keep;
        keep.add(&ix->d_heavy_slot, limit);
        keep.add(&ix->d_heavy_bits, (uint64_t)n_heavy * n_words);
        keep.add(&ix->d_heavy_rank, (uint64_t)n_heavy * n_words);
        TRY(keep.take());
        ix->heavy_block = keep.keep();
        ix->device_bytes += (int64_t)keep.bytes;
        TRY(fill(n_heavy, limit));
    }
    ix->n_heavy = n_heavy;
    ix->view.heavy_slot = ix->d_heavy_slot;
    ix->view.heavy_bits = ix->d_heavy_bits;
    ix->view.heavy_rank = ix->d_heavy_rank;
    ix->view.heavy_limit = limit;
    ix->view.n_heavy = n_heavy;
    ix->view.heavy_min = heavy_min;
    ix->view.n_words = n_words;
    return PPV_OK;
}

// 3. and 4. for rows whose RowMeta is on the device.  counts: (l_max + 1) * n_groups words, already scanned, n_groups
// for as many rows as `rows` has room for; n_prefixes, n_entries: what the scan found.
template <typename TOK>
ppv_status number_prefixes(ppv_index *ix, TOK tok, const RowMeta *rows, uint32_t n_rows, uint32_t n_tok, int32_t l_max,
                           const uint32_t *counts, uint32_t n_groups, const uint32_t *group_lcp, uint32_t n_prefixes,
                           uint32_t n_entries, int32_t vocab, const HostWords &words, hipStream_t st) {
    if (n_prefixes > 0xFFFFFFF0u - 2) return PPV_ERANGE;
    const uint32_t G = n_prefixes + 1;   // with the empty prefix
    // PPV_TUNE_LOOKUP = 0: no table (every prefix is located by the descent).  PPV_TUNE_LOOKUP_WEAK = 1 (tests): one
    // fingerprint for all, so that every probe is a false hit and the exact check has to turn it away.
    const bool lookup = ppv_tuning(PPV_TUNE_LOOKUP) != 0;
    // A bucket per entry: one in fifty is full, so that a query of ten lengths is rarely kept by one of them.
    const uint32_t buckets = lookup ? std::min(n_entries, 0xFFFFFFF0u / LOOKUP_BUCKET) : 0u;
    const uint64_t size = (uint64_t)buckets * LOOKUP_BUCKET;
    Arena keep;
    keep.add(&ix->d_ent, (uint64_t)G + 1);
    keep.add(&ix->d_node_lo, G);
    keep.add(&ix->d_node_hi, G);
    keep.add(&ix->d_x_tok, n_tok);
    keep.add(&ix->d_x_off, (uint64_t)n_rows + 1);
    keep.add(&ix->d_node_at, lookup ? n_tok : 0);
    keep.add(&ix->d_lookup, size);
    const uint64_t n_words = ((uint64_t)vocab + 31) / 32, n_images = std::min(HEAVY_GUESS, heavy_at_most(G, vocab));
    keep.add(&ix->d_heavy_slot, std::min(G, HEAVY_REACH));
    keep.add(&ix->d_heavy_bits, n_images * n_words);
    keep.add(&ix->d_heavy_rank, n_images * n_words);
    TRY(keep.take());
    ix->block = keep.keep();
    ix->device_bytes = (int64_t)keep.bytes;
    if (lookup) PPV_HIP_TRY(hipMemsetAsync(ix->d_lookup, 0, (size_t)size * sizeof(LookupEntry), st));
    TrieOut o;
    o.ent = ix->d_ent;
    o.node_lo = ix->d_node_lo;
    o.node_hi = ix->d_node_hi;
    o.x_tok = ix->d_x_tok;
    o.x_off = ix->d_x_off;
    o.node_at = ix->d_node_at;
    o.table = lookup ? ix->d_lookup : nullptr;
    o.buckets = buckets;
    o.fp_mask = ppv_tuning(PPV_TUNE_LOOKUP_WEAK) == 1 ? 0u : 0xFFFFFFFFu;
    // LDS for what 64 rows hold on average and a quarter more, or for 64 of the longest
    const uint64_t mean = ((uint64_t)n_tok * WAVE + n_rows - 1) / n_rows;
    const uint32_t room = (uint32_t)std::min<uint64_t>(std::min<uint64_t>(mean + mean / 4 + WAVE, (uint64_t)l_max * WAVE), 4096);
    hipLaunchKernelGGL(fill_prefixes<TOK>, dim3(blocks_for(n_rows)), dim3(BT), BW * room * sizeof(uint32_t), st, tok, rows,
                       n_rows, counts, n_groups, group_lcp, l_max, G, room, o);
    PPV_HIP_TRY(hipGetLastError());
    TRY(finish_heavy(ix, G, vocab, words, st));
    ix->n_tokens = n_tok;
    ix->view.ent = ix->d_ent;
    ix->view.node_lo = ix->d_node_lo;
    ix->view.node_hi = ix->d_node_hi;
    ix->view.n_nodes = G;
    ix->view.n_rows = n_rows;
    ix->view.vocab = vocab;
    ix->view.l_max = l_max;
    ix->view.x_tok = ix->d_x_tok;
    ix->view.node_at = ix->d_node_at;
    ix->view.lookup = o.table;
    ix->view.lookup_buckets = buckets;
    ix->view.lookup_fp_mask = o.fp_mask;
    return PPV_OK;
}

ppv_status build_on_device(const int32_t *tokens, const int64_t *offsets, int64_t n_seq, int32_t vocab, ppv_index *ix) {
    if (offsets[0] != 0) return PPV_EINVAL;
    const int64_t total = offsets[n_seq];
    if (total < n_seq) return PPV_EINVAL;                          // some sequence is empty (or offsets decrease)
    if (n_seq > 0xFFFFFFF0ll || total > 0xFFFFFFF0ll) return PPV_ERANGE;
    const uint32_t n = (uint32_t)n_seq;
    hipStream_t st = nullptr;

    // ---- inputs to the device
    uint16_t *d_lo;
    uint8_t *d_hi;
    uint32_t *d_off;
    const bool wide = vocab > 65536;
    TempArena in;
    in.add(&d_lo, (uint64_t)total);
    in.add(&d_hi, wide ? (uint64_t)total : 0);
    in.add(&d_off, (uint64_t)n + 1);
    // ... and what sorting them needs
    uint64_t *key, *key2, *place, *sums64, *d_tot64;
    uint32_t *row, *row2, *hist, *digit_total, *info, *d_word;
    uint8_t *group, *group2;
    RowMeta *rows;
    const uint32_t sort_chunks = (n + SORT_CHUNK - 1) / SORT_CHUNK;
    in.add(&key, n);
    in.add(&key2, n);
    in.add(&row, n);
    in.add(&row2, n);
    in.add(&group, (uint64_t)n + GROUP_PAD);
    in.add(&group2, (uint64_t)n + GROUP_PAD);
    in.add(&hist, (uint64_t)RADIX * sort_chunks);
    in.add(&digit_total, RADIX);
    in.add(&info, n);
    in.add(&place, n);
    in.add(&sums64, scan_words(n));
    in.add(&d_tot64, 1);
    in.add(&d_word, 3);
    in.add(&rows, n);
    TRY(in.take());
    if (!wide) d_hi = nullptr;
    int32_t l_max = 0;
    TRY(ppv_upload_set(tokens, offsets, n_seq, vocab, d_lo, d_hi, d_off, st, &l_max));   // EINVAL: empty sequence, token outside [0, vocab)
    const PackedTokens tok = {d_lo, d_hi};

    // ---- 1. sort
    KeyShape ks;
    ks.bits = 1;
    while ((1ll << ks.bits) <= (int64_t)vocab) ks.bits++;           // keys run over 0 .. vocab
    ks.slots = std::min(64 / ks.bits, l_max);
    const uint64_t last_slot = (1ull << ks.bits) - 1ull;
    const unsigned nb = blocks_for(n);
    hipLaunchKernelGGL(first_keys, dim3(nb), dim3(BT), 0, st, tok, (const uint32_t *)d_off, n, ks, key, row);
    TRY(radix_sort(key, key2, row, row2, n, ks.bits * ks.slots, hist, digit_total, st));
    int64_t depth = ks.slots;                                       // tokens ordered so far
    uint32_t n_groups = 0, *counts, *group_lcp, *sums;
    uint64_t n_counts = 0;
    TempArena cnt;
    auto room_for = [&](uint32_t rows_at_most) {   // the counts of step 3
        n_groups = (rows_at_most + WAVE - 1) / WAVE;
        n_counts = ((uint64_t)l_max + 1) * n_groups;
        if (n_counts > 0xFFFFFFF0ull) return PPV_ERANGE;
        cnt.add(&counts, n_counts);
        cnt.add(&group_lcp, n_groups);
        cnt.add(&sums, scan_words(n_counts));
        return cnt.take();
    };
    // The counts are laid out for the rows that were given, duplicates and all, so that nothing waits for the host to know
    // how many are left; unless that is much (256 MB), for one long row among many short ones.
    const bool by_rows_left = ((uint64_t)l_max + 1) * ((n + WAVE - 1) / WAVE) > (1ull << 26);
    if (!by_rows_left) TRY(room_for(n));
    const HostWords words;
    if (!words.w) return PPV_ENOMEM;

    PPV_HIP_TRY(hipMemsetAsync(d_word, 0, 3 * sizeof(uint32_t), st));   // what order_groups leaves (two words); all counts
    auto order = [&] {   // groups of rows equal so far: what can be ordered by counting
        hipLaunchKernelGGL(next_keys, dim3(nb), dim3(BT), 0, st, tok, (const uint32_t *)d_off, (const uint32_t *)row,
                           (const uint8_t *)group, n, (uint32_t)depth, ks, key);
        hipLaunchKernelGGL(order_groups, dim3(nb), dim3(BT), 0, st, tok, (const uint32_t *)d_off, (const uint32_t *)row,
                           (const uint8_t *)group, (const uint64_t *)key, n, (uint32_t)(depth + ks.slots), last_slot,
                           depth + ks.slots >= l_max ? 1 : 0, row2, group2, d_word);
        std::swap(row, row2);
        std::swap(group, group2);
    };
    // Step 2, and step 3 up to the sizes of the arrays, and the host's look at them.  They are run before it is known
    // whether groups are left (a trip to the host), and again if there were any.
    auto distinct = [&] {
        hipLaunchKernelGGL(neighbour_lcp, dim3(nb), dim3(BT), 0, st, tok, (const uint32_t *)d_off, (const uint32_t *)row, n,
                           info, place);
        TRY(exclusive_scan<uint64_t>(n, ValueAt<uint64_t>{place}, place, sums64, d_tot64, st));
        hipLaunchKernelGGL(compact_rows, dim3(nb), dim3(BT), 0, st, (const uint32_t *)d_off, (const uint32_t *)row, n,
                           (const uint32_t *)info, (const uint64_t *)place, rows);
        return PPV_OK;
    };
    auto count = [&] {
        hipLaunchKernelGGL(count_prefixes, dim3((n_groups + BW - 1) / BW), dim3(BT), 0, st, (const RowMeta *)rows,
                           (const uint64_t *)d_tot64, n_groups, l_max, counts, group_lcp);
        TRY(exclusive_scan<uint32_t>(n_counts, ValueAt<uint32_t>{counts}, counts, sums, d_word + 2, st));
        hipLaunchKernelGGL(publish, dim3(1), dim3(1), 0, st, words.dev(), (const uint64_t *)d_tot64,
                           (const uint32_t *)(counts + (uint64_t)l_max * n_groups), (const uint32_t *)(d_word + 2),
                           (const uint32_t *)d_word);
        PPV_HIP_TRY(hipGetLastError());
        PPV_HIP_TRY(hipStreamSynchronize(st));
        return PPV_OK;
    };
    if (depth < l_max) {
        hipLaunchKernelGGL(mark_groups, dim3(nb), dim3(BT), 0, st, (const uint64_t *)key, n, last_slot, group, group2);
        order();
    }
    uint32_t left[2];
    if (by_rows_left) {
        TRY(read_back(left, d_word, 2, st));
    } else {
        TRY(distinct());
        TRY(count());
        left[0] = words.w->large;
        left[1] = words.w->split;
    }
    const bool again = by_rows_left || left[0] + left[1] > 0;
    while (left[0] + left[1] > 0) {
        if (left[0] > 0) {
            // rows in groups too large to count (and the others that are left): sorted by their next tokens under the group's
            // number
            const uint32_t m = left[0] + left[1];
            TRY(exclusive_scan<uint64_t>(n, LargeRows{group, n}, place, sums64, d_tot64, st));
            uint64_t tot;
            TRY(read_back(&tot, d_tot64, 1, st));
            int group_bits = 1;
            while ((1ull << group_bits) < (tot & 0xFFFFFFFFull)) group_bits++;
            KeyShape ls = ks;
            ls.slots = (int)std::min<int64_t>((64 - group_bits) / ks.bits, l_max - depth);
            uint32_t *lrow = row2, *lrow2 = info, *lplace = (uint32_t *)rows;   // (written by step 2, which comes later)
            uint64_t *lkey = key, *lkey2 = key2;
            hipLaunchKernelGGL(large_keys, dim3(nb), dim3(BT), 0, st, tok, (const uint32_t *)d_off, (const uint32_t *)row,
                               (const uint8_t *)group, (const uint64_t *)place, n, (uint32_t)depth, ls, lkey, lrow, lplace);
            TRY(radix_sort(lkey, lkey2, lrow, lrow2, m, ls.bits * ls.slots + group_bits, hist, digit_total, st));
            depth += ls.slots;
            hipLaunchKernelGGL(large_back, dim3(blocks_for(m)), dim3(BT), 0, st, (const uint64_t *)lkey, (const uint32_t *)lrow,
                               (const uint32_t *)lplace, m, last_slot, depth >= l_max ? 1 : 0, row, group);
        } else {
            depth += ks.slots;   // every group that is left agrees in the tokens of the round before
        }
        if (depth >= l_max) break;
        PPV_HIP_TRY(hipMemsetAsync(d_word, 0, 2 * sizeof(uint32_t), st));
        order();
        TRY(read_back(left, d_word, 2, st));
    }
    if (again) TRY(distinct());
    auto too_many = [&](uint64_t rows_left) { return (uint64_t)l_max * rows_left + 1 > 0xFFFFFFF0ull; };   // (depth, row) pairs are limited to 32 bits
    if (by_rows_left) {
        uint64_t tot;
        TRY(read_back(&tot, d_tot64, 1, st));
        if (too_many(tot >> 32)) return PPV_ERANGE;
        TRY(room_for((uint32_t)(tot >> 32)));
    }
    if (again) TRY(count());
    const uint32_t n_rows = (uint32_t)(words.w->rows_tokens >> 32), n_tok = (uint32_t)words.w->rows_tokens;
    if (too_many(n_rows)) return PPV_ERANGE;
    return number_prefixes(ix, tok, rows, n_rows, n_tok, l_max, counts, n_groups, group_lcp, words.w->prefixes,
                           words.w->all_counts - words.w->prefixes, vocab, words, st);
}

void release(ppv_index *ix) {
    if (!ix) return;
    if (ix->block || ix->heavy_block) {
        // the blocks go to the next index, so every kernel that may still read them has to be over (as hipFree would
        // wait for it); the wait is no part of a capture that another stream may be in
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        int dev = -1;
        (void)hipGetDevice(&dev);
        if (ix->device >= 0 && ix->device != dev) (void)hipSetDevice(ix->device);
        const bool over = hipDeviceSynchronize() == hipSuccess;
        if (ix->device >= 0 && ix->device != dev && dev >= 0) (void)hipSetDevice(dev);
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        (void)hipGetLastError();
        ppv_pool_give(ix->block, over);
        ppv_pool_give(ix->heavy_block, over);
    }
    delete ix;
}

// ------------------------------------------------------------------------------------------
// Persistence.  The file holds what cannot be recomputed cheaply -- the entries (heavy flag cleared), the rank
// ranges and the flat sorted S -- behind a fixed header; the heavy prefixes' images are rebuilt at load.
// Little-endian, as the machine is.
struct FileHeader {
    char magic[8];
    uint32_t version, header_bytes;
    int32_t vocab, l_max;
    uint64_t n_rows, n_nodes, n_tokens;
    uint64_t checksum;      // over the sections, in file order
    uint64_t reserved[9];
};
static_assert(sizeof(FileHeader) == 128, "file header layout");
const char FILE_MAGIC[8] = {'P', 'P', 'V', 'I', 'D', 'X', 0, 1};
constexpr size_t IO_CHUNK = 32u << 20;   // bytes staged per copy

// 64-bit multiply-xor checksum over 8-byte words (the tail is zero-padded); `h` carries across calls whose
// lengths are multiples of 8 except the last of a section
inline uint64_t checksum_words(uint64_t h, const unsigned char *p, size_t n) {
    size_t i = 0;
    for (; i + 8 <= n; i += 8) {
        uint64_t w;
        memcpy(&w, p + i, 8);
        h = (h ^ w) * 0x100000001B3ull;
        h ^= h >> 29;
    }
    if (i < n) {
        uint64_t w = 0;
        memcpy(&w, p + i, n - i);
        h = (h ^ w) * 0x100000001B3ull;
        h ^= h >> 29;
    }
    return h;
}

struct Section {
    void *dev;
    size_t bytes;
    bool entries;   // NodeEnt array: the heavy flag is not stored
};

// A loaded file is only believed as far as it can be checked: the rows have to be rows, in order, and everything else
// in it has to be what numbering those rows' prefixes gives.
__global__ __launch_bounds__(BT) void compare_loaded(const NodeEnt *__restrict__ ent, const uint32_t *__restrict__ node_lo,
                                                     const uint32_t *__restrict__ node_hi, const NodeEnt *__restrict__ f_ent,
                                                     const uint32_t *__restrict__ f_lo, const uint32_t *__restrict__ f_hi,
                                                     uint32_t n_nodes, int32_t *__restrict__ err) {
    const uint32_t g = blockIdx.x * BT + threadIdx.x;
    if (g > n_nodes) return;
    bool bad = (ent[g].tok & ~PPV_NODE_HEAVY) != f_ent[g].tok || ent[g].child != f_ent[g].child;
    if (g < n_nodes) bad = bad || node_lo[g] != f_lo[g] || node_hi[g] != f_hi[g];
    if (bad) atomicOr(err, 1);
}
// the rows of a checked file as the numbering wants them; they have to be in strictly increasing order
__global__ __launch_bounds__(BT) void meta_of_rows(const int32_t *__restrict__ x_tok, const int64_t *__restrict__ x_off,
                                                   uint32_t n_rows, RowMeta *__restrict__ rows, int32_t *__restrict__ err) {
    const uint32_t i = blockIdx.x * BT + threadIdx.x;
    if (i >= n_rows) return;
    const uint32_t a = (uint32_t)x_off[i], la = (uint32_t)(x_off[i + 1] - x_off[i]);
    uint32_t c = 0;
    if (i > 0) {
        const uint32_t b = (uint32_t)x_off[i - 1], lb = a - b;
        const uint32_t m = la < lb ? la : lb;
        while (c < m && x_tok[a + c] == x_tok[b + c]) c++;
        if (c < m ? x_tok[a + c] < x_tok[b + c] : la <= lb) atomicOr(err, 4);
    }
    RowMeta r;
    r.at = a;
    r.src = a;
    r.lcp = c;
    r.len = la;
    rows[i] = r;
}
__global__ __launch_bounds__(BT) void check_loaded_rows(const int32_t *__restrict__ x_tok, const int64_t *__restrict__ x_off,
                                                        uint64_t n_rows, uint64_t n_tokens, int32_t vocab, int32_t l_max,
                                                        int32_t *__restrict__ err, int32_t *__restrict__ reached) {
    const uint64_t i = (uint64_t)blockIdx.x * BT + threadIdx.x;
    bool bad = false;
    if (i < n_rows) {
        const int64_t a = x_off[i], b = x_off[i + 1];
        bad = a < 0 || b <= a || b - a > l_max || (uint64_t)b > n_tokens || (i == 0 && a != 0) ||
              (i == n_rows - 1 && (uint64_t)b != n_tokens);
        if (b - a == l_max) *reached = 1;   // (some row is as long as the file says; all that find one write the same)
    }
    if (i < n_tokens) bad = bad || x_tok[i] < 0 || x_tok[i] >= vocab;
    if (bad) atomicOr(err, 2);
}

ppv_status save_to_file(const ppv_index *ix, const char *path) {
    PPV_HIP_TRY(hipSetDevice(ix->device));
    FILE *f = fopen(path, "wb");
    if (!f) return PPV_EIO;
    unsigned char *stage = new (std::nothrow) unsigned char[IO_CHUNK];
    if (!stage) {
        fclose(f);
        return PPV_ENOMEM;
    }
    FileHeader h;
    memset(&h, 0, sizeof(h));
    memcpy(h.magic, FILE_MAGIC, 8);
    h.version = 1;
    h.header_bytes = sizeof(FileHeader);
    h.vocab = ix->view.vocab;
    h.l_max = ix->view.l_max;
    h.n_rows = ix->view.n_rows;
    h.n_nodes = ix->view.n_nodes;
    h.n_tokens = (uint64_t)ix->n_tokens;
    const Section sec[5] = {{ix->d_ent, ((size_t)h.n_nodes + 1) * sizeof(NodeEnt), true},
                            {ix->d_node_lo, (size_t)h.n_nodes * sizeof(uint32_t), false},
                            {ix->d_node_hi, (size_t)h.n_nodes * sizeof(uint32_t), false},
                            {ix->d_x_off, ((size_t)h.n_rows + 1) * sizeof(int64_t), false},
                            {ix->d_x_tok, (size_t)h.n_tokens * sizeof(int32_t), false}};
    ppv_status st = PPV_OK;
    if (fwrite(&h, sizeof(h), 1, f) != 1) st = PPV_EIO;
    uint64_t sum = 0xCBF29CE484222325ull;
    for (int k = 0; k < 5 && st == PPV_OK; k++)
        for (size_t at = 0; at < sec[k].bytes && st == PPV_OK; at += IO_CHUNK) {
            const size_t n = std::min(IO_CHUNK, sec[k].bytes - at);
            if (hipMemcpy(stage, (const unsigned char *)sec[k].dev + at, n, hipMemcpyDeviceToHost) != hipSuccess) {
                (void)hipGetLastError();
                st = PPV_EDEVICE;
                break;
            }
            if (sec[k].entries)
                for (size_t e = 0; e < n / sizeof(NodeEnt); e++) {
                    NodeEnt ne;
                    memcpy(&ne, stage + e * sizeof(NodeEnt), sizeof(NodeEnt));
                    ne.tok &= ~PPV_NODE_HEAVY;
                    memcpy(stage + e * sizeof(NodeEnt), &ne, sizeof(NodeEnt));
                }
            sum = checksum_words(sum, stage, n);
            if (fwrite(stage, 1, n, f) != n) st = PPV_EIO;
        }
    delete[] stage;
    if (st == PPV_OK) {
        h.checksum = sum;
        if (fseek(f, 0, SEEK_SET) != 0 || fwrite(&h, sizeof(h), 1, f) != 1) st = PPV_EIO;
    }
    if (fclose(f) != 0 && st == PPV_OK) st = PPV_EIO;
    return st;
}

ppv_status load_from_file(FILE *f, ppv_index *ix) {
    FileHeader h;
    if (fread(&h, sizeof(h), 1, f) != 1) return PPV_EINVAL;   // shorter than a header: not an index file
    if (memcmp(h.magic, FILE_MAGIC, 8) != 0 || h.version != 1 || h.header_bytes != sizeof(FileHeader)) return PPV_EINVAL;
    if (h.vocab <= 0 || h.l_max <= 0 || h.n_rows == 0 || h.n_nodes < 2 || h.n_tokens < h.n_rows) return PPV_EINVAL;
    // No row is longer than what the others leave of the tokens, and the file's length vouches for n_tokens: a longest row
    // beyond that would ask for arrays, and for loops over the depths, of any size up to 2^31.
    if ((uint64_t)h.l_max > h.n_tokens - h.n_rows + 1) return PPV_EINVAL;
    if (h.vocab > PPV_MAX_VOCAB || h.n_rows > 0xFFFFFFF0ull || h.n_nodes > 0xFFFFFFF0ull || h.n_tokens > 0xFFFFFFF0ull)
        return PPV_ERANGE;
    const size_t bytes[5] = {((size_t)h.n_nodes + 1) * sizeof(NodeEnt), (size_t)h.n_nodes * sizeof(uint32_t),
                             (size_t)h.n_nodes * sizeof(uint32_t), ((size_t)h.n_rows + 1) * sizeof(int64_t),
                             (size_t)h.n_tokens * sizeof(int32_t)};
    if (fseek(f, 0, SEEK_END) != 0) return PPV_EIO;
    const long end = ftell(f);
    if (end < 0 || (uint64_t)end != sizeof(h) + bytes[0] + bytes[1] + bytes[2] + bytes[3] + bytes[4]) return PPV_EINVAL;
    if (fseek(f, (long)sizeof(h), SEEK_SET) != 0) return PPV_EIO;

    if (hipGetDevice(&ix->device) != hipSuccess) {
        (void)hipGetLastError();
        return PPV_EDEVICE;
    }
    const uint32_t n_rows = (uint32_t)h.n_rows, n_groups = (n_rows + WAVE - 1) / WAVE;
    const uint64_t n_counts = ((uint64_t)h.l_max + 1) * n_groups;
    if (n_counts > 0xFFFFFFF0ull) return PPV_ERANGE;
    NodeEnt *f_ent;
    uint32_t *f_lo, *f_hi, *counts, *group_lcp, *sums, *d_word;
    int64_t *f_off;
    int32_t *f_tok, *d_err;
    uint64_t *d_tot64;
    RowMeta *rows;
    TempArena tmp;
    tmp.add(&f_ent, h.n_nodes + 1);
    tmp.add(&f_lo, h.n_nodes);
    tmp.add(&f_hi, h.n_nodes);
    tmp.add(&f_off, h.n_rows + 1);
    tmp.add(&f_tok, h.n_tokens);
    tmp.add(&rows, n_rows);
    tmp.add(&counts, n_counts);
    tmp.add(&group_lcp, n_groups);
    tmp.add(&sums, scan_words(n_counts));
    tmp.add(&d_tot64, 1);
    tmp.add(&d_word, 1);
    tmp.add(&d_err, 2);
    TRY(tmp.take());
    void *dev[5] = {f_ent, f_lo, f_hi, f_off, f_tok};
    unsigned char *stage = new (std::nothrow) unsigned char[IO_CHUNK];
    if (!stage) return PPV_ENOMEM;
    ppv_status st = PPV_OK;
    uint64_t sum = 0xCBF29CE484222325ull;
    for (int k = 0; k < 5 && st == PPV_OK; k++)
        for (size_t at = 0; at < bytes[k] && st == PPV_OK; at += IO_CHUNK) {
            const size_t n = std::min(IO_CHUNK, bytes[k] - at);
            if (fread(stage, 1, n, f) != n) {
                st = PPV_EIO;
                break;
            }
            sum = checksum_words(sum, stage, n);
            if (hipMemcpy((unsigned char *)dev[k] + at, stage, n, hipMemcpyHostToDevice) != hipSuccess) {
                (void)hipGetLastError();
                st = PPV_EDEVICE;
            }
        }
    delete[] stage;
    if (st != PPV_OK) return st;
    if (sum != h.checksum) return PPV_EINVAL;

    const HostWords words;
    if (!words.w) return PPV_ENOMEM;
    // the checksum guards against damage; these checks guard the kernels against a file that was wrong when written
    hipStream_t s0 = nullptr;
    PPV_HIP_TRY(hipMemsetAsync(d_err, 0, 2 * sizeof(int32_t), s0));   // what is wrong; whether a row of l_max tokens is there
    hipLaunchKernelGGL(check_loaded_rows, dim3(blocks_for(std::max(h.n_rows, h.n_tokens))), dim3(BT), 0, s0,
                       (const int32_t *)f_tok, (const int64_t *)f_off, h.n_rows, h.n_tokens, h.vocab, h.l_max, d_err, d_err + 1);
    PPV_HIP_TRY(hipGetLastError());
    int32_t found[2] = {0, 0}, err = 0;
    TRY(read_back(found, d_err, 2, s0));
    if (found[0] != 0 || found[1] != 1) return PPV_EINVAL;
    hipLaunchKernelGGL(meta_of_rows, dim3(blocks_for(n_rows)), dim3(BT), 0, s0, (const int32_t *)f_tok, (const int64_t *)f_off,
                       n_rows, rows, d_err);
    const uint64_t tot64 = h.n_rows << 32;
    PPV_HIP_TRY(hipMemcpyAsync(d_tot64, &tot64, sizeof(tot64), hipMemcpyHostToDevice, s0));
    hipLaunchKernelGGL(count_prefixes, dim3((n_groups + BW - 1) / BW), dim3(BT), 0, s0, (const RowMeta *)rows,
                       (const uint64_t *)d_tot64, n_groups, h.l_max, counts, group_lcp);
    TRY(exclusive_scan<uint32_t>(n_counts, ValueAt<uint32_t>{counts}, counts, sums, d_word, s0));
    uint32_t n_all, n_pref;
    PPV_HIP_TRY(hipMemcpyAsync(&err, d_err, sizeof(err), hipMemcpyDeviceToHost, s0));
    PPV_HIP_TRY(hipMemcpyAsync(&n_all, d_word, sizeof(n_all), hipMemcpyDeviceToHost, s0));
    TRY(read_back(&n_pref, counts + (uint64_t)h.l_max * n_groups, 1, s0));
    if (err != 0 || (uint64_t)n_pref + 1 != h.n_nodes) return PPV_EINVAL;
    TRY(number_prefixes(ix, FlatTokens{f_tok}, (const RowMeta *)rows, n_rows, (uint32_t)h.n_tokens, h.l_max, counts, n_groups,
                        group_lcp, n_pref, n_all - n_pref, h.vocab, words, s0));
    hipLaunchKernelGGL(compare_loaded, dim3(blocks_for(h.n_nodes + 1)), dim3(BT), 0, s0, (const NodeEnt *)ix->d_ent,
                       (const uint32_t *)ix->d_node_lo, (const uint32_t *)ix->d_node_hi, (const NodeEnt *)f_ent,
                       (const uint32_t *)f_lo, (const uint32_t *)f_hi, (uint32_t)h.n_nodes, d_err);
    PPV_HIP_TRY(hipGetLastError());
    TRY(read_back(&err, d_err, 1, s0));
    return err == 0 ? PPV_OK : PPV_EINVAL;
}

}  // namespace

extern "C" ppv_status ppv_build_index(const int32_t *tokens, const int64_t *offsets, int64_t n_seq, int32_t vocab,
                                      ppv_index_t **out) {
    if (!out) return PPV_EINVAL;
    *out = nullptr;
    if (!tokens || !offsets || n_seq <= 0 || vocab <= 0) return PPV_EINVAL;
    if (vocab > PPV_MAX_VOCAB) return PPV_ERANGE;
    ppv_index *ix = new (std::nothrow) ppv_index();
    if (!ix) return PPV_ENOMEM;
    if (hipGetDevice(&ix->device) != hipSuccess) {
        (void)hipGetLastError();
        delete ix;
        return PPV_EDEVICE;
    }
    ppv_status st = build_on_device(tokens, offsets, n_seq, vocab, ix);
    if (st != PPV_OK) {
        (void)hipDeviceSynchronize();
        (void)hipGetLastError();
        release(ix);
        return st;
    }
    *out = ix;
    return PPV_OK;
}

extern "C" ppv_status ppv_index_info(const ppv_index_t *ix, int64_t *n_distinct, int32_t *l_max, int32_t *vocab,
                                     int64_t *n_prefixes, int64_t *device_bytes) {
    if (!ix) return PPV_EINVAL;
    if (n_distinct) *n_distinct = ix->view.n_rows;
    if (l_max) *l_max = ix->view.l_max;
    if (vocab) *vocab = ix->view.vocab;
    if (n_prefixes) *n_prefixes = (int64_t)ix->view.n_nodes - 1;
    if (device_bytes) *device_bytes = ix->device_bytes;
    return PPV_OK;
}

extern "C" ppv_status ppv_index_export(const ppv_index_t *ix, int32_t *tokens_out, int64_t *offsets_out,
                                       int64_t *n_tokens) {
    if (!ix) return PPV_EINVAL;
    if (n_tokens) *n_tokens = ix->n_tokens;
    if (tokens_out && ix->n_tokens)
        PPV_HIP_TRY(hipMemcpy(tokens_out, ix->d_x_tok, (size_t)ix->n_tokens * sizeof(int32_t), hipMemcpyDeviceToHost));
    if (offsets_out)
        PPV_HIP_TRY(hipMemcpy(offsets_out, ix->d_x_off, ((size_t)ix->view.n_rows + 1) * sizeof(int64_t),
                              hipMemcpyDeviceToHost));
    return PPV_OK;
}

extern "C" void ppv_free_index(ppv_index_t *ix) { release(ix); }

extern "C" ppv_status ppv_index_save(const ppv_index_t *ix, const char *path) {
    if (!ix || !path || !path[0]) return PPV_EINVAL;
    return save_to_file(ix, path);
}

extern "C" ppv_status ppv_index_load(const char *path, ppv_index_t **out) {
    if (!out) return PPV_EINVAL;
    *out = nullptr;
    if (!path || !path[0]) return PPV_EINVAL;
    FILE *f = fopen(path, "rb");
    if (!f) return PPV_EIO;
    ppv_index *ix = new (std::nothrow) ppv_index();
    if (!ix) {
        fclose(f);
        return PPV_ENOMEM;
    }
    ix->device = -1;
    const ppv_status st = load_from_file(f, ix);
    fclose(f);
    if (st != PPV_OK) {
        if (ix->device >= 0) {   // the device was touched: let its work drain before the buffers go
            (void)hipDeviceSynchronize();
            (void)hipGetLastError();
            release(ix);
        } else {
            delete ix;
        }
        return st;
    }
    *out = ix;
    return PPV_OK;
}
