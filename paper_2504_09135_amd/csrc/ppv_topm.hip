// Algorithm 2 with M candidates (the variant the paper ran with M = 50): per row, the M tokens of
// largest probability, one verification per candidate row a + [t_i], and the extended mask.
//
// One workgroup per row.
//   select   P = softmax(logits) is increasing in the logit, so the top M are found on the logits'
//            bit patterns, through an order-preserving 32-bit key per token.  M is small against
//            |V|, so almost every token can be turned away with one comparison:
//              A. the maxima of groups of tokens (half or a quarter of what a lane holds, or for large M every 16 bytes) are histogrammed by
//                 their 11 leading key bits; the bin that holds the M-th largest maximum gives a bound that at
//                 least M tokens reach.  A wavefront holds eight or sixteen chunks of the row (a chunk: 16 bytes a lane) in
//                 registers; when its share of the row is longer, A looks only at those --
//                 the M-th largest of a part of the row is still a lower bound of the row's --
//                 provided the list has room for what the looser bound lets through (else from as
//                 many more of its chunks as it takes).  When A has looked at one set of chunks, the
//                 maxima inside the bound's bin are counted once more by their next five key bits
//                 and the bound moves up inside the bin.  A is over when the prefix has been located, or soon after;
//              B. the tokens that are not below the bound are listed in LDS in token order, each with its
//                 key: usually 1.1 to 1.5 M of them, from registers when A saw the whole row,
//                 else about as many times more as the share is longer than what is held, from the
//                 one pass over the row (the next chunks are asked for before these are
//                 looked at).  Of a chunk the maxima of its 16-byte groups are compared, two chunks at a time on 16-bit keys; the
//                 groups that have a token for the list are queued, one a lane, and listed together;
//              C. a radix select over that short list (the keys' upper halves, counted from the bound, in one
//                 histogram of 256 bins; two more digits of 8 bits for fp32) finds the key T of the
//                 M-th largest token; of the list, the
//                 tokens above T and the first few equal to T, in increasing token id, are chosen, so the set
//                 is unique.
//            What a call of few rows waits for is a chain of steps of the whole workgroup.  128 rows at V = 128,256 bf16, M = 50, us from
//            a wavefront's start, before / now: prefix located 3.1 / 4.1 and A done 5.3 / 6.2 (the row, 256 KB for one compute
//            unit, arrives over the first 4 us: A waited for the prefix, and asked for half of the row later), bound 6.7 / 7.2, list 13.1 / 9.7
//            (2 to 5 us a wavefront for a handful of tokens, each chunk with one listed by itself, and the row's other half on its
//            way), chosen 16.5 / 11.3, written 17.2 / 11.7.  Per call, us before / now: this shape 18.4 / 13.6, V = 32k, 256 rows 11.8 / 9.8,
//            V = 32k, 4,096 rows 73.7 / 56.0, V = 256k, 1,024 rows 115.6 / 98.4, V = 50k fp32, 384 rows 26.5 / 21.2, V = 8,192, 512 rows, M = 1,000
//            20.9 / 16.5.
//            If the list does not fit (a flat row with thousands of equal logits at the cut, M near the number of the row's 16-byte groups, or a
//            workgroup too small to hold it) the same radix select runs over the whole row instead,
//            one histogram pass per digit and two more passes to gather in token order.
//   verify   the M candidate rows share their first |a| tokens, so the prefix is located once
//            (the same walk the full-vocabulary mask uses) and each candidate then needs one
//            binary search for its last token among the prefix's children (their tokens are
//            copied to LDS while the row is on its way) -- or one bit test in the ready-made
//            image of a heavy prefix.  One thread per candidate.
//   extend   the mask row is assembled in LDS and written with whole words.
//   count    a caller that wants only the mask (no candidate list, no verdicts) does not need the top M at all
//            when the prefix has few continuations: token t is among the M most probable iff fewer than M
//            tokens come before it in the order (logit descending, token id ascending).  Those are counted
//            for each child in one pass over the row, two instructions per token and child, with no
//            histogram, no list and no second pass.
// Nothing here is a dense contraction; the row is read from HBM once (64 KB at V = 32k, bf16).
#include <cstdlib>
#include <type_traits>

#include "ppv_device.h"
#include "ppv_internal.h"
#include "ppv_walk.h"

namespace {

constexpr int TOPM_BITS = 11;             // leading key bits of the first digit
constexpr int TOPM_BINS = 1 << TOPM_BITS;   // the histogram shares its LDS with the mask row
constexpr int TOPM_SHIFT = 32 - TOPM_BITS;
constexpr int TOPM_CBINS = 256;   // bins of the histogram over the listed tokens' keys, counted from the bound (the last one: all above)
constexpr int TOPM_WAVES = 16;
constexpr int TOPM_LIST_BIG = 4096, TOPM_LIST_SMALL = 1024;   // capacity of the candidate list (tokens not below the bound),
                                                              // split evenly over the wavefronts; the small one serves M <= 128 at V <= 65,536
constexpr int TOPM_SLOTS = 16;    // list entries per thread at most: the list path needs at least LIST / 16 threads
constexpr int TOPM_HELD = 8;      // chunks of the row a wavefront holds in registers at a time (128 bytes per lane) ...
constexpr int TOPM_HELD_LONG = 16;   // ... where that is the whole share of sixteen wavefronts (see topm_held)

// Bit pattern -> key with the same order as the float value (-0 and +0 share a key).
__device__ inline uint32_t order_key(uint32_t bits) {
    if (bits == 0x80000000u) bits = 0u;
    return bits ^ ((uint32_t)((int32_t)bits >> 31) | 0x80000000u);
}

template <typename T> struct KeyChunk;   // what one 16-byte load per lane covers
template <> struct KeyChunk<float> {
    static constexpr int EPL = 4;
    __device__ static inline void keys(const uint4 &r, uint32_t k[4]) {
        k[0] = order_key(r.x); k[1] = order_key(r.y); k[2] = order_key(r.z); k[3] = order_key(r.w);
    }
    __device__ static inline uint32_t bits_of(const float *row, int v) { return ((const uint32_t *)row)[v]; }
};
template <> struct KeyChunk<uint16_t> {
    static constexpr int EPL = 8;
    __device__ static inline void keys(const uint4 &r, uint32_t k[8]) {
        k[0] = order_key(r.x << 16); k[1] = order_key(r.x & 0xFFFF0000u);
        k[2] = order_key(r.y << 16); k[3] = order_key(r.y & 0xFFFF0000u);
        k[4] = order_key(r.z << 16); k[5] = order_key(r.z & 0xFFFF0000u);
        k[6] = order_key(r.w << 16); k[7] = order_key(r.w & 0xFFFF0000u);
    }
    __device__ static inline uint32_t bits_of(const uint16_t *row, int v) { return (uint32_t)row[v] << 16; }
};

// Keys of this lane's EPL consecutive tokens of chunk c (tokens c*64*EPL + lane*EPL + k).  Returns how
// many of them lie inside the row (the first n of k[]); memory at or beyond token V is never touched.
template <typename T>
__device__ inline int load_keys(const T *__restrict__ row, int V, int c, int lane, uint32_t k[KeyChunk<T>::EPL]) {
    constexpr int EPL = KeyChunk<T>::EPL;
    const int g = (c * WAVE + lane) * EPL;
    if (g + EPL <= V) {
        KeyChunk<T>::keys(*(const uint4 *)(row + g), k);
        return EPL;
    }
    int n = 0;
    for (int j = 0; j < EPL; j++) {
        k[j] = 0u;
        if (g + j < V) {
            k[j] = order_key(KeyChunk<T>::bits_of(row, g + j));
            n = j + 1;
        }
    }
    return n;
}

// This lane's 16 bytes of chunk c (c from `end` on: nothing is read and 0 arrives, as behind the row's end; the caller discards
// that, and the tokens of the row's last group that lie beyond its end).  No condition stands between the caller and
// the load, so loads for the next batch can be in flight while this batch is worked on.  STREAM: the bytes are
// not read again (they need not stay in cache).
template <bool STREAM = true> __device__ inline uint4 load_chunk(const Row &row, int c, int end, int lane) {
    const uint32_t at = (uint32_t)(c < end ? c : 1 << 20) * (WAVE * 16u) + (uint32_t)lane * 16u;
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(row.buf, at, 0, STREAM ? 2 /* non-temporal */ : 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}
// four chunks at once (c .. c+3): four loads in flight per lane
template <bool STREAM>
__device__ inline void load_chunks(const Row &row, int c, int end, int lane, uint4 *r) {
#pragma unroll
    for (int u = 0; u < 4; u++) r[u] = load_chunk<STREAM>(row, c + u, end, lane);
}
// how many of this lane's tokens of chunk c lie inside the row
template <typename T> __device__ inline int n_inside(int V, int c, int lane) {
    constexpr int EPL = KeyChunk<T>::EPL;
    const int r = V - (c * WAVE + lane) * EPL;
    return r < 0 ? 0 : (r > EPL ? EPL : r);
}
template <typename T> __device__ inline void unpack_vals(const uint4 &r, float x[KeyChunk<T>::EPL]) {
    if (sizeof(T) == 4) {
        x[0] = __uint_as_float(r.x); x[1] = __uint_as_float(r.y);
        x[2 % KeyChunk<T>::EPL] = __uint_as_float(r.z); x[3 % KeyChunk<T>::EPL] = __uint_as_float(r.w);
    } else {
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int j = 0; j < 4; j++) {
            x[(2 * j) % KeyChunk<T>::EPL] = __uint_as_float(w[j] << 16);
            x[(2 * j + 1) % KeyChunk<T>::EPL] = __uint_as_float(w[j] & 0xFFFF0000u);
        }
    }
}

// The histogram hist[0..bins) is filled (bins <= 4096).  Finds the digit d with #(digit > d) < need <= #(digit >= d)
// and leaves it in bc[4], with need - #(digit > d) in bc[5].  If fewer than `need` entries were counted,
// bc[4] = 0 and bc[5] = need.  Every thread calls; ends with a barrier.
// The work is wavefront 0's alone, in two levels without a barrier between them: lane l sums a run of consecutive
// bins (runs ordered from the top bin down), a scan over the lanes finds the run in which the count reaches
// `need`, and that run's bins, one per lane, are scanned the same way.  (A scan over all the workgroup's threads
// costs three barriers and was 1.5 to 2.2 us of a 16 us call.)
__device__ inline void pick_digit(const uint32_t *hist, int bins, uint32_t need, uint32_t *bc) {
    if (threadIdx.x < WAVE) {
        const int lane = threadIdx.x;
        const int per = (bins + WAVE - 1) / WAVE;        // bins per lane, at most 64
        const int top_bin = bins - 1 - lane * per;       // lane l: bins top_bin - per + 1 .. top_bin
        const int low_bin = top_bin - per + 1;
        uint32_t s = 0;
        if (low_bin >= 0 && (per & 3) == 0 && (bins & 3) == 0) {   // whole run present and 16-byte aligned
            for (int j = 0; j < per; j += 4) {
                const uint4 h = *(const uint4 *)(hist + low_bin + j);
                s += h.x + h.y + h.z + h.w;
            }
        } else {
            for (int j = 0; j < per; j++)
                if (top_bin - j >= 0) s += hist[top_bin - j];
        }
        const uint32_t incl = wave_incl_scan(s);
        const uint64_t reach = __ballot(incl >= need);
        uint32_t digit = 0u, rest = need;
        if (reach) {   // wave-uniform
            const int l = __ffsll((long long)reach) - 1;                 // the run in which the count reaches need
            const uint32_t above = lane_value(incl - s, l);              // entries in the runs above it
            const int run_top = bins - 1 - l * per;
            const int bin = run_top - lane;                               // level 2: lane j takes bin run_top - j
            const uint32_t h = (lane < per && bin >= 0) ? hist[bin] : 0u;
            const uint32_t incl2 = above + wave_incl_scan(h);
            const uint64_t reach2 = __ballot(lane < per && bin >= 0 && incl2 >= need);
            if (reach2) {   // always: the run's total reaches need
                const int j = __ffsll((long long)reach2) - 1;
                digit = (uint32_t)(run_top - j);
                rest = need - lane_value(incl2 - h, j);
            }
        }
        if (lane == 0) {
            bc[4] = digit;
            bc[5] = rest;
        }
    }
    __syncthreads();
}

// digit p of the radix select: key bits [shift, previous shift)
template <typename T> __device__ inline int digit_shift(int pass) {
    return pass == 0 ? TOPM_SHIFT : (sizeof(T) == 4 ? (pass == 1 ? TOPM_SHIFT - TOPM_BITS : 0) : 16);
}
// bf16: the low 16 bits of a key follow from its sign, so the upper half settles the whole key
template <typename T> __device__ inline uint32_t full_key(uint32_t hi_part) {
    return sizeof(T) == 4 ? hi_part : ((hi_part << 16) | ((hi_part >> 15) & 1u ? 0u : 0xFFFFu));
}

// A barrier for what the workgroup has in LDS: loads from memory stay in flight over it.
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A word that is the same in all lanes, which the compiler does not see of one from LDS.  (Branches on words of LDS were joined again by masks:
// what one side holds was kept, and spilled, on the other.)
__device__ inline uint32_t uniform_word(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

struct TopmLds {
    uint32_t *hist;       // [TOPM_BINS]
    uint32_t *hist3;      // [32] the group maxima inside the bound's bin, by their next five key bits
    uint32_t *hist2;      // [TOPM_CBINS] the listed tokens' keys, counted from the bound (filled while they are listed)
    uint32_t *list_tok;   // [LIST]
    uint32_t *list_key;   // [LIST] the listed tokens' logits (bit patterns, bf16 in the upper half)
    uint32_t *sel;        // [PPV_TOPM_MAX]
    uint32_t *seg_a, *seg_b, *wave_tot;   // [TOPM_WAVES] each
    uint32_t *bc;         // [8]
    uint4 *queue;         // [64] a wavefront: 16 bytes of the row with a token for the list
    uint32_t *queue_tok;  // [64] a wavefront
};

// Radix select over the whole row (any workgroup size, any row): fills sel[0..m) in increasing token id.
template <typename T>
__device__ inline void select_streaming(const T *__restrict__ row, int V, int c0, int c1, int m, const TopmLds &s,
                                        int lane, int wave, int nthreads) {
    constexpr int EPL = KeyChunk<T>::EPL;
    const int tid = threadIdx.x, nw = nthreads / WAVE;
    const int n_pass = sizeof(T) == 4 ? 3 : 2;
    uint32_t hi_part = 0;          // digits settled so far, as the key's leading bits
    uint32_t need = (uint32_t)m;   // how many tokens are still to be taken among those that match hi_part
    int prev_shift = 32;
    for (int pass = 0; pass < n_pass; pass++) {
        const int shift = digit_shift<T>(pass);
        const int bins = 1 << (prev_shift - shift);
        for (int i = tid; i < bins; i += nthreads) s.hist[i] = 0u;
        __syncthreads();
        for (int c = c0; c < c1; c++) {
            uint32_t k[EPL];
            const int n = load_keys<T>(row, V, c, lane, k);
#pragma unroll
            for (int j = 0; j < EPL; j++) {
                const bool match = pass == 0 || (k[j] >> prev_shift) == hi_part;
                if (j < n && match) atomicAdd(&s.hist[(k[j] >> shift) & (uint32_t)(bins - 1)], 1u);
            }
        }
        __syncthreads();
        pick_digit(s.hist, bins, need, s.bc);
        hi_part = (hi_part << (prev_shift - shift)) | s.bc[4];
        need = s.bc[5];
        prev_shift = shift;
        __syncthreads();
    }
    const uint32_t T_key = full_key<T>(hi_part);
    const uint32_t take_eq = need;   // of the tokens whose key equals T_key, the first take_eq in token order

    // gather in token order: counts per wavefront share, then positions from prefix counts
    uint32_t n_gt = 0, n_eq = 0;
    for (int c = c0; c < c1; c++) {
        uint32_t k[EPL];
        const int n = load_keys<T>(row, V, c, lane, k);
#pragma unroll
        for (int j = 0; j < EPL; j++) {
            n_gt += (j < n && k[j] > T_key) ? 1u : 0u;
            n_eq += (j < n && k[j] == T_key) ? 1u : 0u;
        }
    }
    n_gt = wave_sum(n_gt);
    n_eq = wave_sum(n_eq);
    if (lane == 0) {
        s.seg_a[wave] = n_gt;
        s.seg_b[wave] = n_eq;
    }
    __syncthreads();
    uint32_t gt_base = 0, eq_base = 0;   // tokens of either kind in the wavefronts before this one
    for (int w = 0; w < nw; w++)
        if (w < wave) {
            gt_base += s.seg_a[w];
            eq_base += s.seg_b[w];
        }
    for (int c = c0; c < c1; c++) {
        uint32_t k[EPL];
        const int n = load_keys<T>(row, V, c, lane, k);
        uint32_t g = 0, e = 0;
#pragma unroll
        for (int j = 0; j < EPL; j++) {
            g += (j < n && k[j] > T_key) ? 1u : 0u;
            e += (j < n && k[j] == T_key) ? 1u : 0u;
        }
        const uint32_t gi = wave_incl_scan(g), ei = wave_incl_scan(e);
        uint32_t gt_before = gt_base + gi - g, eq_before = eq_base + ei - e;
        const uint32_t first_tok = (uint32_t)((c * WAVE + lane) * EPL);
#pragma unroll
        for (int j = 0; j < EPL; j++) {
            if (j >= n) continue;
            if (k[j] > T_key) {
                const uint32_t pos = gt_before + (eq_before < take_eq ? eq_before : take_eq);
                if (pos < (uint32_t)m) s.sel[pos] = first_tok + j;
                gt_before++;
            } else if (k[j] == T_key) {
                if (eq_before < take_eq) {
                    const uint32_t pos = gt_before + eq_before;
                    if (pos < (uint32_t)m) s.sel[pos] = first_tok + j;
                }
                eq_before++;
            }
        }
        gt_base += last_lane(gi);
        eq_base += last_lane(ei);
    }
    __syncthreads();
}

// Two bf16 values in one word -> their two 16-bit keys, ordered as the values are (-0 just below +0: the
// thresholds below allow for it).
typedef short topm_s2 __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pk_keys(uint32_t w) {
    const topm_s2 sign = __builtin_bit_cast(topm_s2, w) >> 15;   // 0xFFFF under a negative value
    return w ^ (__builtin_bit_cast(uint32_t, sign) | 0x80008000u);
}
// per half: 1 if the key is above the threshold, else 0.  Two packed 16-bit instructions (saturating subtraction,
// minimum with 1), written out because the compiler turns the same expression back into a comparison and a
// select per half.
__device__ inline uint32_t pk_above(uint32_t keys, uint32_t thresholds) {
    uint32_t d, r;
    const uint32_t ones = 0x00010001u;
    asm("v_pk_sub_u16 %0, %1, %2 clamp" : "=v"(d) : "v"(keys), "v"(thresholds));
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(d), "v"(ones));
    return r;
}
__device__ inline uint32_t pk_max(uint32_t a, uint32_t b) {
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(us2, a), __builtin_bit_cast(us2, b)));
}
// How a row is taken by select_listed: a wavefront's share is the chunks c0 .. c1 - 1 of nc.
struct TopmShare {
    int nc, cpw;      // chunks of the row, and of a wavefront (the last ones may have fewer)
    int c0, c1;
    int a_batches;    // batches of `held` chunks of each share that A looks at
    int by_lane;      // 2, 4: A's groups are what a lane has of a batch in every second, every fourth chunk; 0: 16 bytes
};
// With the bound from the whole row the list holds 1.1 to 1.5 m tokens when the bound is taken to the key's
// upper 16 bits (possible when A looks at one batch) and about 4 m of a row of noise when it stays at
// the histogram's bin, a quarter of an octave; from a_batches batches of the share, cpw / (held a_batches)
// times more.  One batch if the list then has room for twice 1.3 m times that, else as few as leave room for
// 4 m times that.  (A list that overflows all the same sends the row to the whole-row select.)
// by_lane: groups of what a lane holds, two or four of them, where A's histogram takes eight or sixteen additions a lane otherwise, nearly all to
// the same few bins.  Tokens thrown into n groups are the largest of n (1 - exp(-tokens / n)) of them: with four groups to a candidate
// the bound lets 1.15 m tokens through.  A vocabulary may be in an order, though, that has all that are likely next to one another, in one
// wavefront's share: its 128 groups then let 125 through for m = 80, its 256 groups 194 for m = 136, which a part of 256 holds, and soon too many
// beyond that.  (In a part of 128 logits that fall as 1.5 log of the id, V = 32k, 256 rows, M = 50, did not fit: 36 us with the whole-row select, 13 with
// groups of 16 bytes.  M = 100, V = 128k bf16, 128 rows, groups of 16 bytes / four a lane: 14.8 / 14.0, logits that fall as above with noise 22.5 / 18.5.
// Of a longer share A sees too little for four: V = 32k, 4,096 rows, M = 100 98 / 69.)
template <typename T, bool KEPT>
__device__ inline TopmShare share_of_row(int V, int m, int list, int held, int wave, int nthreads) {
    constexpr int EPL = KeyChunk<T>::EPL;
    const int nw = nthreads / WAVE;
    TopmShare h;
    h.nc = (V + WAVE * EPL - 1) / (WAVE * EPL);
    h.cpw = (h.nc + nw - 1) / nw;
    h.c0 = wave * h.cpw;
    h.c1 = (h.c0 + h.cpw < h.nc) ? h.c0 + h.cpw : h.nc;
    const int all = (h.cpw + held - 1) / held;
    const long long want = 2ll * m * h.cpw <= (long long)held * list ? 1 : ((long long)m * h.cpw * 4 + (long long)held * list - 1) / ((long long)held * list);
    h.a_batches = KEPT ? 1 : want > all ? all : (int)want;
    h.by_lane = nthreads < 2 * m || list / nw < 256 ? 0 : m <= 80 ? 2 : KEPT && m <= 136 ? 4 : 0;
    return h;
}

// The upper halves of the largest keys of this lane's 16 bytes of two chunks, c and c + 1, side by side (the first in the lower
// half); 0, a key that only NaNs have, where there is no token (`end`: the first chunk that is not to be looked at).  A token may have that
// key too; a group of nothing else then does not count, which makes the bound lower if anything.  -0 is just below +0 here.
template <typename T> __device__ inline uint32_t pair_key(const uint4 &a, const uint4 &b, int V, int c, int end, int lane) {
    uint32_t half[2];   // bf16: the largest of the even and of the odd tokens; fp32: the largest, in the upper half
    const uint4 *w[2] = {&a, &b};
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const bool ragged = (c + i + 1) * WAVE * KeyChunk<T>::EPL > V;   // (wave-uniform) the row ends inside this chunk
        const int n = ragged ? n_inside<T>(V, c + i, lane) : 0;
        const uint32_t v[4] = {w[i]->x, w[i]->y, w[i]->z, w[i]->w};
        uint32_t k[4];
        if (sizeof(T) == 2) {
#pragma unroll
            for (int j = 0; j < 4; j++) k[j] = pk_keys(v[j]);
            if (ragged) {
#pragma unroll
                for (int j = 0; j < 4; j++) k[j] &= (2 * j < n ? 0x0000FFFFu : 0u) | (2 * j + 1 < n ? 0xFFFF0000u : 0u);
            }
            half[i] = pk_max(pk_max(k[0], k[1]), pk_max(k[2], k[3]));
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++) k[j] = v[j] ^ ((uint32_t)((int32_t)v[j] >> 31) | 0x80000000u);
            if (ragged) {
#pragma unroll
                for (int j = 0; j < 4; j++) k[j] = j < n ? k[j] : 0u;
            }
            half[i] = max(max(k[0], k[1]), max(k[2], k[3]));
        }
        if (c + i >= end) half[i] = 0u;   // (wave-uniform)
    }
    const uint32_t upper = __builtin_amdgcn_perm(half[1], half[0], 0x07060302u);
    return sizeof(T) == 4 ? upper : pk_max(upper, __builtin_amdgcn_perm(half[1], half[0], 0x05040100u));
}
// do_group(key): the upper half of the largest key of each of this lane's groups
template <int PAIRS, typename DO> __device__ inline void each_group(const TopmShare &h, const uint32_t (&pairs)[PAIRS], DO do_group) {
    if (h.by_lane) {   // (uniform)
        uint32_t a = pairs[0], b = pairs[1];
#pragma unroll
        for (int p = 2; p < PAIRS; p += 2) {
            a = pk_max(a, pairs[p]);
            b = pk_max(b, pairs[p + 1]);
        }
        if (h.by_lane == 2) a = pk_max(a, b);   // (uniform)
        do_group(a & 0xFFFFu);
        do_group(a >> 16);
        if (h.by_lane == 4) {
            do_group(b & 0xFFFFu);
            do_group(b >> 16);
        }
    } else {
#pragma unroll
        for (int p = 0; p < PAIRS; p++) {
            do_group(pairs[p] & 0xFFFFu);
            do_group(pairs[p] >> 16);
        }
    }
}
// A: the maxima of groups of the row's tokens, and the histogram of their leading key bits (cleared before the workgroup's last
// barrier).  r arrives holding the wavefront's first HELD chunks; pairs: the maxima of the batch that A looks at last, by 16 bytes.
template <typename T, int HELD, bool KEPT>
__device__ inline void group_maxima(const Row &buf, int V, const TopmShare &h, uint32_t *hist, int lane, uint4 (&r)[HELD],
                                    uint32_t (&pairs)[HELD / 2]) {
    const int a_end = h.c0 + h.a_batches * HELD < h.c1 ? h.c0 + h.a_batches * HELD : h.c1;
#pragma unroll
    for (int p = 0; p < HELD / 2; p++) pairs[p] = 0u;   // (a wavefront may have no share)
    for (int c = h.c0; c < a_end; c += HELD) {
        if (!KEPT && c != h.c0) {   // (chunks that A reads from memory are read again in B: from cache)
#pragma unroll
            for (int u = 0; u < HELD; u += 4) load_chunks<false>(buf, c + u, h.c1, lane, r + u);
        }
#pragma unroll
        for (int p = 0; p < HELD / 2; p++) {
            pairs[p] = 0u;
            if (c + 2 * p < h.c1) pairs[p] = pair_key<T>(r[2 * p], r[2 * p + 1], V, c + 2 * p, h.c1, lane);   // (wave-uniform)
        }
        // A lane with many groups adds those in its first one's bin at once: rows whose maxima fall into one or two bins wait for their additions, one
        // lane after the other, and where the row is counted in the end for nothing.  (us, V = 32k bf16, 256 rows, M = 50, mask alone, one by one / so:
        // logits around 12, prefixes of all kinds 10.7 / 10.1, of one continuation 8.1 / 7.5, falling as 1.5 log of the id 8.8 / 7.8; around 0
        // 9.8 / 9.9, 7.1 / 7.2.  With few groups a lane 1 to 3 % slower.)
        if (!h.by_lane && h.cpw > 4) {   // (uniform)
            const uint32_t first = (pairs[0] & 0xFFFFu) >> (16 - TOPM_BITS);
            uint32_t same = 0u;
            each_group(h, pairs, [&](uint32_t key16) {
                const uint32_t bin = key16 >> (16 - TOPM_BITS);
                same += bin == first ? 1u : 0u;
                if (bin != first && key16 != 0u) atomicAdd(&hist[bin], 1u);
            });
            if (first != 0u && same != 0u) atomicAdd(&hist[first], same);   // (bin 0 need not be counted: see select_listed's edge)
        } else {
            each_group(h, pairs, [&](uint32_t key16) {
                if (key16 != 0u) atomicAdd(&hist[key16 >> (16 - TOPM_BITS)], 1u);
            });
        }
    }
}

// From A's maxima to the cut list: bound, short list, radix select over the list.  Needs nthreads >= LIST / TOPM_SLOTS and
// nthreads <= LIST.  Returns false (for every thread alike) when the list did not fit; nothing is chosen then.  Otherwise
// chosen(position, token) is called for each of the m tokens, whose positions are in increasing token id, after the words
// img[0..n_words), which may be the histogram's, have been cleared.  r, pairs: as group_maxima left them, with a barrier since;
// hist2, hist3 and bc[6] were cleared before it.
// The row is read from memory once: a share longer than r gives the bound from its first chunks only (at least m
// of THEIR groups reach it, so at least m tokens of the row do) -- as many batches of HELD chunks as it takes
// for the list to have room for what the looser bound lets through; B reads the batches after the first again, from
// cache, and the rest of the share for the first time.
template <typename T, int LIST, int HELD, bool KEPT, typename CHOSEN>
__device__ inline bool select_listed(const Row &buf, int V, const TopmShare &h, int m, const TopmLds &s, int lane,
                                     int wave, int nthreads, uint4 (&r)[HELD], uint32_t (&pairs)[HELD / 2], uint32_t *img,
                                     int n_words, CHOSEN chosen) {
    constexpr int EPL = KeyChunk<T>::EPL;
    const int tid = threadIdx.x, nw = nthreads / WAVE;
    const int c0 = h.c0, c1 = h.c1;
    const uint32_t R = (uint32_t)(LIST / nw);
    const uint32_t base = (uint32_t)wave * R;
    // At least m groups have their maximum in the bin that is picked or above, so at least m tokens are not below the bin's
    // lower edge.  Where nearly all of the row's groups are asked for, that is below nearly all tokens, and fewer groups than m
    // give no bound at all: the list is not begun.  (us, list / whole-row select, bf16, 64 and 1,024 rows: M = 0.98 of the groups, V = 8,192, 17.5
    // 43.9 / 12.2 36.0; 0.8 of them, V = 10,000 13.0 35.0 / 14.9 45.1, V = 6,000 11.2 25.3 / 12.7 30.3.)
    if (m > (V + EPL - 1) / EPL / 8 * 7) return false;   // (uniform)
    pick_digit(s.hist, TOPM_BINS, (uint32_t)m, s.bc);
    uint32_t edge_key16 = uniform_word(s.bc[4]) << (16 - TOPM_BITS);
    if (edge_key16 == 0u) return false;   // (uniform)
    if (KEPT || h.a_batches == 1) {   // (uniform)
        // A bin is a quarter of an octave wide and holds several times m tokens of a row of noise.  The maxima that
        // A has just seen are still in registers: those inside the bin are counted by their next five key bits, and
        // the bound moves up to the thirty-second of the bin in which the count from the top reaches m.
        const uint32_t bin = s.bc[4], rest = s.bc[5];
        each_group(h, pairs, [&](uint32_t key16) {
            if (key16 >> (16 - TOPM_BITS) == bin) atomicAdd(&s.hist3[key16 & 31u], 1u);   // (bin is not 0: no empty group)
        });
        __syncthreads();
        pick_digit(s.hist3, 32, rest, s.bc);
        edge_key16 |= uniform_word(s.bc[4]);
    }
    // ---- B. the tokens whose keys are not below the edge's, in token order, each wavefront into its own part of the list.
    // Only the keys' upper halves are compared.  (-0 has the key just under +0's in `pairs` and +0's here; an edge at +0 is lowered by one
    // there, so that -0 stays listed: the list may hold more than it need, never less.  C goes by the exact keys.)
    // The groups of 16 bytes that have a token for the list are put into a queue of one per lane, from registers, and then each lane
    // lists what its group holds: one pass of the code that lists, usually, where a wavefront with a token in each of five chunks
    // took five (16 chunks a wavefront, M = 50: 2.2 to 4.5 us).
    uint32_t cnt = 0;   // wave-uniform
    const uint32_t th16 = edge_key16 == 0x8000u ? 0x7FFEu : edge_key16 - 1u;   // listed: key above th16
    const uint32_t th_pk = th16 | (th16 << 16);   // bf16 tokens are compared two at a time
    uint4 *queue = s.queue + wave * WAVE;
    uint32_t *queue_tok = s.queue_tok + wave * WAVE;   // the group's first token
    auto list_group = [&](const uint4 &g, uint32_t first_tok, bool have) __attribute__((always_inline)) {
        const uint32_t w[4] = {g.x, g.y, g.z, g.w};
        uint32_t pm = 0u;   // bit j: token j of this lane's group is listed
        if (sizeof(T) == 2) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint32_t a = pk_above(pk_keys(w[i]), th_pk);
                pm |= ((a | (a >> 15)) & 3u) << (2 * i);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; i++) pm |= order_key(w[i]) >> 16 >= edge_key16 ? 1u << i : 0u;
        }
        const int n = V - (int)first_tok;
        if (n < EPL) pm &= n > 0 ? (1u << n) - 1u : 0u;   // nothing behind the row's end
        if (!have) pm = 0u;
        const uint32_t pc = (uint32_t)__popc(pm);
        const uint32_t incl = wave_incl_scan(pc);
        uint32_t at = cnt + incl - pc;
        while (pm) {
            const uint32_t j = (uint32_t)__ffs((int)pm) - 1u;
            // the token's logit out of the group, by masks (no branch, no indexed register)
            uint32_t bits;
            if (sizeof(T) == 2) {
                const uint32_t m4 = 0u - ((j >> 2) & 1u), m2 = 0u - ((j >> 1) & 1u);
                const uint32_t lo = (w[2] & m4) | (w[0] & ~m4), hi = (w[3] & m4) | (w[1] & ~m4);
                const uint32_t ww = (hi & m2) | (lo & ~m2);
                bits = (ww << ((~j & 1u) << 4)) & 0xFFFF0000u;
            } else {
                const uint32_t m2 = 0u - ((j >> 1) & 1u), m1 = 0u - (j & 1u);
                const uint32_t lo = (w[1] & m1) | (w[0] & ~m1), hi = (w[3] & m1) | (w[2] & ~m1);
                bits = (hi & m2) | (lo & ~m2);
            }
            const uint32_t key = order_key(bits);
            if (at < R) {
                s.list_tok[base + at] = first_tok + j;
                s.list_key[base + at] = key;
            }
            // C's histogram, while the key is at hand: the upper key half, counted from the bound
            const uint32_t rel = (key >> 16) - edge_key16;
            atomicAdd(&s.hist2[rel < (uint32_t)(TOPM_CBINS - 1) ? rel : (uint32_t)(TOPM_CBINS - 1)], 1u);
            at++;
            pm &= pm - 1u;
        }
        cnt += last_lane(incl);
    };
    // N chunks from c + FIRST on, in r[FIRST ..] with their maxima in pairs; what does not fill the queue waits for more (not `last`)
    uint32_t waiting = 0u;   // wave-uniform: groups in the queue
    auto list_some = [&](auto first, auto count, int c, bool last) __attribute__((always_inline)) {
        constexpr int FIRST = decltype(first)::value, N = decltype(count)::value;
        for (uint32_t round = 0;; round += WAVE) {
            uint32_t groups = waiting;
#pragma unroll
            for (int u = FIRST; u < FIRST + N; u++) {
                const uint32_t key16 = (u & 1) ? pairs[u / 2] >> 16 : pairs[u / 2] & 0xFFFFu;
                const bool mine = key16 > th16;
                const uint64_t hit = __ballot(mine);
                if (hit) {   // (uniform) most chunks of a long row have nothing
                    const uint32_t pos = groups + __builtin_amdgcn_mbcnt_hi((uint32_t)(hit >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hit, 0u)) - round;
                    if (mine && pos < (uint32_t)WAVE) {
                        queue[pos] = r[u];
                        queue_tok[pos] = (uint32_t)(((c + u) * WAVE + lane) * EPL);
                    }
                    groups += (uint32_t)__popcll(hit);
                }
            }
            const uint32_t left = groups - round;
            if (left < (uint32_t)WAVE && !(last && left != 0u)) {
                waiting = left;
                break;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (the queue is this wavefront's own)
            const bool have = (uint32_t)lane < left;
            const int at = have ? lane : 0;
            list_group(queue[at], queue_tok[at], have);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (left <= (uint32_t)WAVE || cnt > R) {   // (a list that does not fit is not gone on with)
                waiting = 0u;
                break;
            }
        }
    };
    constexpr int HALF = HELD / 2;
    if (KEPT) {
        list_some(std::integral_constant<int, 0>(), std::integral_constant<int, HELD>(), c0, true);
    } else {
        if (h.a_batches > 1) {   // A has left its last chunks in r
#pragma unroll
            for (int u = 0; u < HELD; u += 4) load_chunks<true>(buf, c0 + u, c1, lane, r + u);
        }
        // the two halves of r take turns: half of the chunks are asked for again as soon as they have been looked at,
        // while the others are looked at
        auto maxima = [&](int p0, int c) __attribute__((always_inline)) {
#pragma unroll
            for (int p = p0; p < p0 + HALF / 2; p++) pairs[p] = pair_key<T>(r[2 * p], r[2 * p + 1], V, c + 2 * p, c1, lane);
        };
        for (int c = c0; c < c1 && cnt <= R; c += HELD) {
            maxima(0, c);
            list_some(std::integral_constant<int, 0>(), std::integral_constant<int, HALF>(), c, false);
#pragma unroll
            for (int u = 0; u < HALF; u++) r[u] = load_chunk(buf, c + HELD + u, c1, lane);
            maxima(HALF / 2, c);
            list_some(std::integral_constant<int, HALF>(), std::integral_constant<int, HALF>(), c, c + HELD >= c1);
#pragma unroll
            for (int u = HALF; u < HELD; u++) r[u] = load_chunk(buf, c + HELD + u, c1, lane);
        }
    }
    if (lane == 0 && cnt > R) atomicOr(&s.bc[6], 1u);
    __syncthreads();
    if (uniform_word(s.bc[6]) != 0u) return false;
    for (int i = tid; i < n_words; i += nthreads) img[i] = 0u;   // (where the queues were)

    // ---- C. the key T of the m-th largest token, from the list: lane l answers for the entries l, l + 64, ... of its
    // wavefront's part.
    const uint32_t *lk = s.list_key + base, *lt = s.list_tok + base;
    // Every listed token's key is at or above the edge key, so the upper 16 key bits, counted from the edge, are small numbers: the one
    // histogram over them that B has filled settles the upper half of T.  A row whose m-th largest token lies
    // further above the bound than the histogram is long (TOPM_CBINS - 1 values of the upper half) goes to the
    // whole-row select.
    pick_digit(s.hist2, TOPM_CBINS, (uint32_t)m, s.bc);
    if (uniform_word(s.bc[4]) == (uint32_t)(TOPM_CBINS - 1)) return false;   // T lies in the overflow bin
    uint32_t hi_part = edge_key16 + s.bc[4], need = s.bc[5];
    if (sizeof(T) == 4) {   // fp32: the lower half of T, eight bits at a time
        for (int shift = 8; shift >= 0; shift -= 8) {
            __syncthreads();
            for (int i = tid; i < 256; i += nthreads) s.hist[i] = 0u;
            __syncthreads();
            for (uint32_t i = (uint32_t)lane; i < cnt; i += WAVE) {
                const uint32_t k = lk[i];
                if ((k >> (shift + 8)) == hi_part) atomicAdd(&s.hist[(k >> shift) & 255u], 1u);
            }
            __syncthreads();
            pick_digit(s.hist, 256, need, s.bc);
            hi_part = (hi_part << 8) | s.bc[4];
            need = s.bc[5];
        }
        for (int i = tid; i < 256; i += nthreads) s.hist[i] = 0u;   // (where img may lie)
    }
    const uint32_t T_key = sizeof(T) == 4 ? hi_part : full_key<T>(hi_part);
    const uint32_t take_eq = need;
    // positions: list order is token order
    uint32_t n_gt = 0, n_eq = 0;   // wave-uniform
    for (uint32_t q = 0; q < cnt; q += WAVE) {
        const uint32_t i = q + (uint32_t)lane;
        const uint32_t k = i < cnt ? lk[i] : 0u;
        n_gt += (uint32_t)__popcll(__ballot(i < cnt && k > T_key));
        n_eq += (uint32_t)__popcll(__ballot(i < cnt && k == T_key));
    }
    if (lane == 0) s.wave_tot[wave] = n_gt | (n_eq << 16);   // both stay below 2^16 (the list has at most 4096 entries)
    __syncthreads();
    const uint32_t before = wave_sum(lane < wave ? s.wave_tot[lane] : 0u);   // entries of either kind in the wavefronts before this one
    uint32_t gt_before = before & 0xFFFFu, eq_before = before >> 16;
    for (uint32_t q = 0; q < cnt; q += WAVE) {
        const uint32_t i = q + (uint32_t)lane;
        const uint32_t k = i < cnt ? lk[i] : 0u;
        const bool is_gt = i < cnt && k > T_key, is_eq = i < cnt && k == T_key;
        const uint64_t gt = __ballot(is_gt), eq = __ballot(is_eq);
        const uint32_t g = gt_before + __builtin_amdgcn_mbcnt_hi((uint32_t)(gt >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)gt, 0u));
        const uint32_t e = eq_before + __builtin_amdgcn_mbcnt_hi((uint32_t)(eq >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eq, 0u));
        const uint32_t pos = g + (e < take_eq ? e : take_eq);
        if ((is_gt || (is_eq && e < take_eq)) && pos < (uint32_t)m) chosen((int)pos, lt[i]);
        gt_before += (uint32_t)__popcll(gt);
        eq_before += (uint32_t)__popcll(eq);
    }
    return true;
}


// ---- mask-only calls, prefixes with at most TOPM_COUNT_MAX children ----
constexpr int TOPM_COUNT_MAX = 8;

// The two thresholds of a child whose logit has the bits `b` (bf16 in the upper half), each in both halves of a
// word: a token at a smaller id comes before the child if its key is above ge, one at a larger id if above gt.
__device__ inline void pk_thresholds(uint32_t b, uint32_t &ge, uint32_t &gt) {
    const uint32_t h = b >> 16;
    const uint32_t key = h ^ ((h & 0x8000u) ? 0xFFFFu : 0x8000u);
    const bool zero = (h & 0x7FFFu) == 0u;
    const uint32_t k_ge = zero ? 0x7FFFu : key, k_gt = zero ? 0x8000u : key;   // -0 and +0 are equal
    const uint32_t t_ge = k_ge ? k_ge - 1u : 0u;
    ge = t_ge | (t_ge << 16);
    gt = k_gt | (k_gt << 16);
}

// Counts, for each of the n children (token tokc[j], logit thr[j], both wave-uniform), the tokens of chunk c that
// come before it in the order of the top-M selection: a larger logit, or an equal one at a smaller token id.
// cnt[j] is this lane's count; for bf16 rows two 16-bit counts side by side (a lane sees at most 4,096 tokens of
// a row), because whole chunks are then counted two tokens at a time on 16-bit keys: three instructions per word
// and child, none of them through a condition register.
template <typename T>
__device__ inline void count_chunk(const uint4 &raw, int V, int c, int lane, int n, const int (&tokc)[TOPM_COUNT_MAX],
                                   const float (&thr)[TOPM_COUNT_MAX], uint32_t (&cnt)[TOPM_COUNT_MAX]) {
    constexpr int EPL = KeyChunk<T>::EPL;
    constexpr bool PACKED = sizeof(T) == 2;
    const int first = c * WAVE * EPL;            // the chunk holds tokens first .. first + 64 * EPL - 1
    const int g = first + lane * EPL;
    const bool ragged = first + WAVE * EPL > V;  // (wave-uniform) the row ends inside this chunk
    float x[EPL];
    uint32_t keys[4] = {0u, 0u, 0u, 0u};
    if (PACKED) {
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int i = 0; i < 4; i++) keys[i] = pk_keys(w[i]);
        if (ragged) {                            // tokens behind the row's end get the lowest key: above no threshold
#pragma unroll
            for (int i = 0; i < 4; i++)
                keys[i] &= (g + 2 * i < V ? 0x0000FFFFu : 0u) | (g + 2 * i + 1 < V ? 0xFFFF0000u : 0u);
        }
    } else {
        unpack_vals<T>(raw, x);
        if (ragged) {
#pragma unroll
            for (int e = 0; e < EPL; e++)
                if (g + e >= V) x[e] = -INFINITY;    // never before a child: compared with ">" (they follow every token)
        }
    }
#pragma unroll
    for (int j = 0; j < TOPM_COUNT_MAX; j++) {
        if (j >= n) break;                       // (wave-uniform)
        const float t = thr[j];
        const bool before = first + WAVE * EPL <= tokc[j];   // every token of the chunk has a smaller id: ties count
        const bool after = first > tokc[j];                   // every token has a larger id: ties do not count
        uint32_t k = 0;
        if (__builtin_expect(before || after, 1)) {   // (all chunks of a row but one per child: the rest is kept out of the loop's way)
            if (PACKED) {
                uint32_t ge, gt;
                pk_thresholds(__float_as_uint(t), ge, gt);
                const uint32_t th = before ? ge : gt;
#pragma unroll
                for (int i = 0; i < 4; i++) k += pk_above(keys[i], th);
            } else if (before) {
#pragma unroll
                for (int e = 0; e < EPL; e++) k += x[e] >= t ? 1u : 0u;
            } else {
#pragma unroll
                for (int e = 0; e < EPL; e++) k += x[e] > t ? 1u : 0u;
            }
        } else if (PACKED) {                     // the child's own chunk (one per child and row): the threshold
                                                 // of each half follows from which side of the child its token lies on
            uint32_t ge, gt;
            pk_thresholds(__float_as_uint(t), ge, gt);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint32_t lo = g + 2 * i < tokc[j] ? ge : gt, hi = g + 2 * i + 1 < tokc[j] ? ge : gt;
                k += pk_above(keys[i], (lo & 0x0000FFFFu) | (hi & 0xFFFF0000u));
            }
        } else {
#pragma unroll
            for (int e = 0; e < EPL; e++) k += (x[e] > t || (x[e] == t && g + e < tokc[j])) ? 1u : 0u;
        }
        cnt[j] += k;
    }
}

// The mask row of a prefix with n <= TOPM_COUNT_MAX children (entries cb .. cb + n - 1, or the one child `only`),
// restricted to the m most probable tokens.  Every thread of the workgroup calls; r holds the wavefront's first HELD chunks; tot[] was
// cleared before the last barrier.
template <typename T, int HELD, bool KEPT>
__device__ inline void count_children(const IndexView &ix, const T *__restrict__ row, const Row &buf, int V, const TopmShare &share,
                                      int m, uint32_t cb, uint32_t only, int n, uint4 (&r)[HELD], uint32_t *tot,
                                      uint32_t *__restrict__ out, int n_words, int lane, int nthreads) {
    // child j in lane j: its token and that token's logit
    uint32_t ctok = 0u;
    float cthr = 0.f;
    if (lane < n) {
        ctok = (only != PPV_NO_SLOT ? only : ix.ent[cb + (uint32_t)lane].tok) & PPV_NODE_TOKEN;
        ctok = ctok < (uint32_t)V ? ctok : 0u;   // (always inside for an index that was built or loaded)
        cthr = __uint_as_float(KeyChunk<T>::bits_of(row, (int)ctok));
    }
    int tokc[TOPM_COUNT_MAX];
    float thr[TOPM_COUNT_MAX];
    uint32_t cnt[TOPM_COUNT_MAX];
#pragma unroll
    for (int j = 0; j < TOPM_COUNT_MAX; j++) {
        tokc[j] = (int)lane_value(ctok, j);
        thr[j] = __uint_as_float(lane_value(__float_as_uint(cthr), j));
        cnt[j] = 0u;
    }
    // the pairs of r take turns: a pair of chunks is asked for again as soon as it has been counted, while the
    // other three pairs are counted or on their way
    for (int c = share.c0; c < share.c1; c += HELD) {
#pragma unroll
        for (int h = 0; h < HELD; h += 2) {
#pragma unroll
            for (int u = h; u < h + 2; u++)
                if (c + u < share.c1) count_chunk<T>(r[u], V, c + u, lane, n, tokc, thr, cnt);
#pragma unroll
            for (int u = h; u < h + 2; u++)
                if (!KEPT) r[u] = load_chunk(buf, c + HELD + u, share.c1, lane);
        }
        if (KEPT) break;
    }
#pragma unroll
    for (int j = 0; j < TOPM_COUNT_MAX; j++) {
        if (j >= n) break;
        const uint32_t w = wave_sum(sizeof(T) == 2 ? (cnt[j] & 0xFFFFu) + (cnt[j] >> 16) : cnt[j]);
        if (lane == 0) atomicAdd(&tot[j], w);
    }
    __syncthreads();
    bool in[TOPM_COUNT_MAX];
#pragma unroll
    for (int j = 0; j < TOPM_COUNT_MAX; j++) in[j] = j < n && tot[j] < (uint32_t)m;
    auto word = [&](int i) {
        uint32_t w = 0u;
#pragma unroll
        for (int j = 0; j < TOPM_COUNT_MAX; j++)
            if (in[j] && (tokc[j] >> 5) == i) w |= 1u << (tokc[j] & 31);
        return w;
    };
    if ((n_words & 3) == 0 && (((uintptr_t)out) & 15u) == 0) {
        for (int i = (int)threadIdx.x; i < (n_words >> 2); i += nthreads)
            ((uint4 *)out)[i] = make_uint4(word(4 * i), word(4 * i + 1), word(4 * i + 2), word(4 * i + 3));
    } else {
        for (int i = (int)threadIdx.x; i < n_words; i += nthreads) out[i] = word(i);
    }
}

// Words of LDS that are the histogram first, then the wavefronts' queues, then the mask row; the children's tokens follow
__host__ __device__ inline int topm_words(int n_words, int nthreads) {
    const int queues = nthreads * 5;
    return max(max(TOPM_BINS, n_words), queues);
}

// KEPT: a wavefront's whole share of the row is in its registers.  (In kernels of their own: held rows need none of the registers of the loop over
// longer shares, 70 for 96 and six spilled, and neither form spills.  us, 1,024 and 4,096 rows at V = 32k bf16, M = 50: 18.6 60.8 / 16.6 55.5.)
template <typename T, int LIST, int HELD, bool KEPT>
__global__ __launch_bounds__(TOPM_WAVES *WAVE, HELD == TOPM_HELD && LIST == TOPM_LIST_SMALL ? 5 : 4) void topm_kernel(const int32_t *__restrict__ prefixes,
                                                                const int32_t *__restrict__ lens,
                                                                const T *__restrict__ logits, int64_t row_stride,
                                                                int32_t stride, int M, int force_streaming,
                                                                int32_t *__restrict__ top_ids,
                                                                uint8_t *__restrict__ mask_V,
                                                                uint32_t *__restrict__ mask, IndexView ix) {
    constexpr bool WHOLE = HELD == TOPM_HELD_LONG;    // a row is no longer than what its wavefronts hold, and is not counted
    extern __shared__ __align__(16) uint32_t smem[];  // topm_lds() bytes, the histogram first
    __shared__ uint32_t list_tok[LIST], list_key[LIST];
    __shared__ uint32_t hist2[TOPM_CBINS], hist3[32];
    __shared__ uint32_t sel[PPV_TOPM_MAX];
    __shared__ uint32_t seg_a[TOPM_WAVES], seg_b[TOPM_WAVES], wave_tot[TOPM_WAVES];
    __shared__ uint32_t bc[8];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int nthreads = blockDim.x, nw = nthreads / WAVE;
    const int V = ix.vocab, n_words = ix.n_words;
    uint32_t *img = smem;                             // [n_words] the row of the mask, in the end
    uint4 *queue = (uint4 *)smem;                     // [nthreads] once the histogram is done with
    uint32_t *queue_tok = smem + 4 * nthreads;        // [nthreads]
    const int m = M < V ? M : V;                      // candidates of this row
    // the tokens of the prefix's children, when they are listed (not a heavy prefix: at most heavy_min of them)
    uint32_t *kids = smem + topm_words(n_words, nthreads);
    const TopmLds lds = {smem, hist3, hist2, list_tok, list_key, sel, seg_a, seg_b, wave_tot, bc, queue, queue_tok};
    const T *row = logits + (size_t)b * (size_t)row_stride;

    const Row buf = row_of(row, V);
    const TopmShare h = share_of_row<T, KEPT>(V, m, LIST, HELD, wave, nthreads);

    const bool listed = force_streaming != 1 && nthreads * TOPM_SLOTS >= LIST && nthreads <= LIST;
    // a caller that asks for the mask alone: prefixes with few children are settled by counting (see count_children)
    const bool counting = force_streaming == 0 && !top_ids && !mask_V;
    int32_t mine = 0;
    int t = 0;
    if (wave == 0) {   // (before the row: memory answers in the order of its requests)
        mine = first_tokens(prefixes + (size_t)b * (size_t)stride, stride, lane);
        t = lens[b];
    }
    if (counting && tid < TOPM_COUNT_MAX) seg_a[tid] = 0u;
    if (listed) {   // what the list select starts from
        for (int i = tid; i < TOPM_BINS; i += nthreads) smem[i] = 0u;
        for (int i = tid; i < TOPM_CBINS; i += nthreads) hist2[i] = 0u;
        if (tid < 32) hist3[tid] = 0u;
        if (tid == 0) bc[6] = 0u;
        lds_barrier();   // (ahead of the row: a wavefront whose requests wait for their turn goes on to nothing else)
    }
    uint4 r[HELD];
    if (listed || counting) {   // in flight while the prefix is located
#pragma unroll
        for (int u = 0; u < HELD; u += 4)
            if (u == 0 || h.cpw > u) load_chunks<true>(buf, h.c0 + u, h.c1, lane, r + u);   // (uniform; a short row has no second half)
    }
    // Counting pays where the selection would read part of the row twice, and of rows that are held.  Of these, where M is large or the launch is,
    // it saves work, and the maxima wait for the walk's verdict; else it saves time on the way, and only wavefront 0's wait, which
    // knows: the others have nothing to do meanwhile, and a row that is not counted is not kept.  (us, mask alone, V = 32k bf16, M = 50, with counting /
    // without, 64, 256 and 512 rows: prefixes with one continuation each 6.8 7.2 9.9 / 8.9 9.3 12.0, prefixes of all kinds 9.6 10.0 12.4 / 9.6 9.8 12.4.  Many continuations are much work where compute
    // units have more than one row: there two are counted at most; with up to eight, prefixes of all kinds took 13.9 us at 512 rows.)
    const bool count_few = counting && !WHOLE && (!listed || h.a_batches > 1 || KEPT);
    const bool count_first = count_few && (!KEPT || nw < 8 || m > 256);
    const uint32_t most = !count_first && gridDim.x > 256u ? 2u : (uint32_t)(sizeof(T) == 2 ? TOPM_COUNT_MAX : TOPM_COUNT_MAX / 2);
    auto is_counted = [&](uint32_t only, uint32_t few) {
        return count_few && few <= most && (only != PPV_NO_SLOT || few <= ix.heavy_min);
    };
    bool maxima = listed;
    if (wave == 0) {   // the part every candidate row shares: locate the prefix once
        t = t < 0 ? 0 : (t > stride ? stride : t);
        const Walk w = walk_prefix(ix, prefixes + (size_t)b * (size_t)stride, mine, t, lane);
        if (lane == 0) {
            bc[0] = w.slot;
            bc[1] = w.found ? 1u : 0u;
            bc[2] = w.found ? w.cb : 0u;
            bc[3] = w.found ? w.ce : 0u;
            bc[7] = w.only;
        }
        if (uniform_word(w.found ? 1u : 0u) == 0u || is_counted(uniform_word(w.only), uniform_word(w.ce - w.cb))) maxima = maxima && !count_few;
    }
    auto verdict = [&](int i) { return uniform_word(bc[i]); };
    if (count_first) {
        __syncthreads();
        maxima = maxima && !is_counted(verdict(7), verdict(3) - verdict(2));
    }
    // The maxima are taken while wavefront 0 is on its way through the index, unless the row may do without them.
    uint32_t pairs[HELD / 2];
    if (maxima) group_maxima<T, HELD, KEPT>(buf, V, h, smem, lane, r, pairs);
    __syncthreads();   // the walk's verdict, and the maxima's histogram
    const bool found = verdict(1) != 0u;
    const uint32_t cb = verdict(2), ce = verdict(3), only = verdict(7);
    const int n = (int)(ce - cb);
    if (counting) {
        uint32_t *out = mask + (size_t)b * (size_t)n_words;
        if (!found || n == 0) {   // no continuation at all: the row of the mask is empty, the logits do not matter
            if ((n_words & 3) == 0 && (((uintptr_t)mask) & 15u) == 0) {
                for (int i = tid; i < (n_words >> 2); i += nthreads) ((uint4 *)out)[i] = make_uint4(0u, 0u, 0u, 0u);
            } else {
                for (int i = tid; i < n_words; i += nthreads) out[i] = 0u;
            }
            return;
        }
        if (!WHOLE && is_counted(only, ce - cb)) {   // (r holds the share's first chunks)
            count_children<T, HELD, KEPT>(ix, row, buf, V, h, m, cb, only, n, r, seg_a, out, n_words, lane, nthreads);
            return;
        }
    }
    // the children's tokens go to LDS while the row is on its way: the candidates are then looked up there
    const bool kids_listed = found && (only != PPV_NO_SLOT || (uint32_t)n <= ix.heavy_min);
    if (only != PPV_NO_SLOT) {
        if (tid == 0) kids[0] = only & PPV_NODE_TOKEN;
    } else if (kids_listed) {
        for (int i = tid; i < n; i += nthreads) kids[i] = ix.ent[cb + (uint32_t)i].tok & PPV_NODE_TOKEN;
    }
    const uint32_t slot = (found && !kids_listed) ? bc[0] : PPV_NO_SLOT;
    // ---- select, and verify what is selected: candidate i is token t
    const uint32_t *image = ix.heavy_bits + (size_t)(slot != PPV_NO_SLOT ? slot : 0u) * (size_t)n_words;
    auto verify = [&](int i, uint32_t t) {
        uint32_t ok = 0;
        if (t < (uint32_t)V) {
            if (slot != PPV_NO_SLOT) {
                ok = (image[t >> 5] >> (t & 31u)) & 1u;
            } else if (kids_listed) {   // first child whose token is not below t
                int lo = 0, hi = n;
                while (lo < hi) {
                    const int mid = lo + (hi - lo) / 2;
                    if (kids[mid] < t) lo = mid + 1;
                    else hi = mid;
                }
                ok = (lo < n && kids[lo] == t) ? 1u : 0u;
            }
            if (ok) atomicOr(&img[t >> 5], 1u << (t & 31u));
        }
        if (top_ids) top_ids[(size_t)b * (size_t)M + i] = t < (uint32_t)V ? (int32_t)t : -1;
        if (mask_V) mask_V[(size_t)b * (size_t)M + i] = (uint8_t)ok;
    };
    // (a wavefront whose part of the list is long has a few of the chosen in each of many rounds: these are verified with all lanes
    // busy, behind one more barrier)
    const bool gather = 2 * m >= nthreads;
    bool done = false;
    if (listed) {
        done = select_listed<T, LIST, HELD, KEPT>(buf, V, h, m, lds, lane, wave, nthreads, r, pairs, img, n_words, [&](int i, uint32_t t) {
            if (gather) sel[i] = t;   // (uniform)
            else verify(i, t);
        });
    }
    if (!done) {
        select_streaming<T>(row, V, h.c0, h.c1, m, lds, lane, wave, nthreads);
        for (int i = tid; i < n_words; i += nthreads) img[i] = 0u;   // the histogram's LDS becomes the mask row
    }
    if (!done || gather) {   // (uniform)
        __syncthreads();
        for (int i = tid; i < m; i += nthreads) verify(i, sel[i]);
    }
    for (int i = m + tid; i < M; i += nthreads) verify(i, PPV_NO_SLOT);   // (fewer tokens than candidates)
    __syncthreads();

    // ---- extend
    uint32_t *out = mask + (size_t)b * (size_t)n_words;
    if ((n_words & 3) == 0 && (((uintptr_t)mask) & 15u) == 0) {
        for (int i = tid; i < (n_words >> 2); i += nthreads) ((uint4 *)out)[i] = ((const uint4 *)img)[i];
    } else {
        for (int i = tid; i < n_words; i += nthreads) out[i] = img[i];
    }
}

// wavefronts per row: a power of two, at most one per chunk; many for a small batch (latency), few for a large one
int topm_waves(int V, ppv_dtype dt, int B) {
    const int per = (dt == PPV_F32 ? 4 : 8) * WAVE;
    const int nc = (V + per - 1) / per;
    int cap = B <= 512 ? 8 : 4;   // measured at V = 32k, M = 50: B = 256: 11.1 / 11.9 us with 8 / 16; B = 4,096: 63 / 90 / 169 us with 4 / 8 / 16
    // long rows (bf16, us per call with 4 / 8 / 16 wavefronts, M = 50 and 1,000): V = 128k: B = 128: 36 / 23 / 19 and 48 / 32 / 23,
    // B = 1,024: 75 / 66 / 83 and 120 / 99 / 102; V = 256k: B = 128: 60 / 37 / 27 and 78 / 49 / 42, B = 1,024: 118 / 117 / 143 (M = 50)
    if (nc <= 4 && B > 512) cap = 2;   // 4 KB rows (V = 1,024 fp32), B = 4,096, M = 50 / 1,000: 39 / 85 us with 1, 32 / 57 with 2, 36 / 64 with 4
    if (nc >= 128 && B <= 256) cap = 16;
    if (nc >= 128 && B <= 2048 && cap < 8) cap = 8;
    if (const int v = ppv_tuning(PPV_TUNE_TOPM_WAVES)) cap = v < TOPM_WAVES ? v : TOPM_WAVES;   // tuning aid (0: the table above)
    int nw = 1;
    while (nw * 2 <= cap && nw * 2 <= nc) nw <<= 1;
    return nw;
}

int chunks_per_wave(int V, ppv_dtype dt, int nw) {
    const int per = (dt == PPV_F32 ? 4 : 8) * WAVE;
    return ((V + per - 1) / per + nw - 1) / nw;
}

// Chunks that a wavefront holds.  The wavefronts of rows with sixteen are alone on their compute unit and may hold sixteen each, which
// is a row of up to 131,072 bf16 or 65,536 fp32 tokens: all of it is asked for at once and looked at in registers.
int topm_held(int V, ppv_dtype dt, int nw) {
    const int cpw = chunks_per_wave(V, dt, nw);
    return nw == TOPM_WAVES && cpw > TOPM_HELD && cpw <= TOPM_HELD_LONG ? TOPM_HELD_LONG : TOPM_HELD;
}

// LDS besides what the kernel declares
size_t topm_lds(const IndexView &ix, int threads) {
    return (size_t)(topm_words(ix.n_words, threads) + (int)(ix.heavy_min ? ix.heavy_min : 1u)) * sizeof(uint32_t);
}

}  // namespace

extern "C" ppv_status ppv_topm_mask(const ppv_index_t *ix, const int32_t *prefixes, int32_t prefix_stride,
                                    const int32_t *lens, const void *logits, ppv_dtype dt, int64_t row_stride,
                                    int32_t M, int32_t B, int32_t *top_ids, uint8_t *mask_V, uint32_t *mask,
                                    void *stream) {
    if (!ix || B < 0 || prefix_stride < 0 || M < 1) return PPV_EINVAL;
    if (M > PPV_TOPM_MAX) return PPV_ERANGE;
    if (B == 0) return PPV_OK;
    if (!prefixes || !lens || !mask || !logits) return PPV_EINVAL;
    if (dt != PPV_F32 && dt != PPV_BF16) return PPV_EINVAL;
    const int V = ix->view.vocab;
    const int64_t per16 = (dt == PPV_F32) ? 4 : 8;
    if (row_stride < V || row_stride % per16 != 0 || ((uintptr_t)logits & 15u) != 0) return PPV_EINVAL;
    const int threads = topm_waves(V, dt, B) * WAVE;
    // testing aid: PPV_TUNE_TOPM_STREAMING = 1 sends every row through the whole-row radix select; 2 keeps the usual
    // select but takes the top M also where counting would do (mask-only calls)
    const int force_streaming = ppv_tuning(PPV_TUNE_TOPM_STREAMING);
    const size_t lds = topm_lds(ix->view, threads);
    const dim3 grid((unsigned)B), block(threads);
    hipStream_t hs = (hipStream_t)stream;
#define PPV_LAUNCH_TOPM(T, LIST, HELD, KEPT)                                                                          \
    hipLaunchKernelGGL((topm_kernel<T, LIST, HELD, KEPT>), grid, block, lds, hs, prefixes, lens, (const T *)logits,    \
                       row_stride, prefix_stride, M, force_streaming, top_ids, mask_V, mask, ix->view)
    // a few hundred tokens reach the bound when M is small and the row not too long (the bound's bin holds a share
    // of the row): then a quarter of the LDS does, and more rows fit a compute unit
    const bool small_list = M <= 128 && V <= 65536;
    const bool long_share = topm_held(V, dt, threads / WAVE) == TOPM_HELD_LONG, kept = chunks_per_wave(V, dt, threads / WAVE) <= TOPM_HELD;
#define PPV_LAUNCH_TOPM_OF(T)                                                         \
    if (long_share) PPV_LAUNCH_TOPM(T, TOPM_LIST_BIG, TOPM_HELD_LONG, true);          \
    else if (small_list && kept) PPV_LAUNCH_TOPM(T, TOPM_LIST_SMALL, TOPM_HELD, true); \
    else if (small_list) PPV_LAUNCH_TOPM(T, TOPM_LIST_SMALL, TOPM_HELD, false);       \
    else if (kept) PPV_LAUNCH_TOPM(T, TOPM_LIST_BIG, TOPM_HELD, true);                \
    else PPV_LAUNCH_TOPM(T, TOPM_LIST_BIG, TOPM_HELD, false)
    if (dt == PPV_F32) {
        PPV_LAUNCH_TOPM_OF(float);
    } else {
        PPV_LAUNCH_TOPM_OF(uint16_t);
    }
#undef PPV_LAUNCH_TOPM_OF
#undef PPV_LAUNCH_TOPM
    PPV_HIP_TRY(hipGetLastError());
    return PPV_OK;
}
