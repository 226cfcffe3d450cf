// Per-step kernels for gfx950 (wave64): next-token scatter (packed mask) with the prefix's rank range,
// fused masked log-softmax + inverse-CDF sample, and the fused decode step (the prefix is located by
// walk_prefix, shared with the top-M kernel).
//
// The logits row is the only large operand.  It is streamed exactly once, in tiles of 4 KB per
// wavefront (four 16-byte loads per lane, issued before any index work so that they are in
// flight while the prefix is located).  Each tile yields (reference, sum of exp relative to it), the
// reference being a value near the tile's maximum; tiles are combined afterwards, so every tile is
// independent and a row can be spread over any number of wavefronts.  The valid set enters in one of two ways:
//   list   at most PPV_LIST_MAX valid tokens: their logits are gathered (they were just streamed,
//          so they come from cache), summed relative to their own maximum, and the sample is
//          located by a scan over the list -- no per-element mask work in the stream;
//   image  more valid tokens: a V-bit image is applied inside the stream (three more ALU
//          operations per element) and the sample is located by re-reading one tile.
// Nothing here is a dense contraction, so no MFMA; the bound is HBM bandwidth, with the exp
// (quarter-rate v_exp_f32) as the main ALU cost.
#include <atomic>
#include <cmath>
#include <cstddef>
#include <mutex>
#include <type_traits>

#include "ppv_device.h"
#include "ppv_internal.h"
#include "ppv_walk.h"

namespace {

constexpr int MASK_THREADS = 256;
constexpr int MAX_WAVES = 16;                 // wavefronts per row (workgroup of up to 1024 threads)
constexpr int LOOP_WAVES = 8;                 // the decode-loop kernel with the list in LDS
constexpr int MAX_TILES = PPV_MAX_TILES;
constexpr float LN2F = 0.693147180559945309417f;
static_assert(PPV_MAX_VOCAB <= MAX_TILES * 1024, "tile bookkeeping too small");

__device__ __forceinline__ float fast_exp2(float y) { return __builtin_amdgcn_exp2f(y); }  // v_exp_f32, 1 ulp
__device__ __forceinline__ float fast_log2(float y) { return __builtin_amdgcn_logf(y); }   // v_log_f32, 1 ulp (normal inputs)
// exp(d) for d <= 0 with the rounding of d*log2(e) compensated (used once per tile, not per token)
// Temperature (Algorithm 1's input T): P = softmax(logits / T).  The division is folded into the constant of the
// exponentials, c = log2(e) / T, so that it costs nothing per token; differences of logits that enter a result
// as they are (a reference minus another) are multiplied by inv = 1 / T.  T = 1 gives c = log2(e), inv = 1.
struct Temper {
    float c;
    float inv;
    float guard;   // how far above an image tile's reference a logit may lie (REF_GUARD * T, see image_stats)
};

__device__ __forceinline__ float exp_scale(float d, float c) {
    float hi = d * c;
    float lo = fmaf(d, c, -hi);
    return fast_exp2(hi) * fmaf(lo, LN2F, 1.0f);
}

// Arguments.  Every kernel takes first what its first loads need (pointers and sizes, 14 words at most) and the structs
// last: the leading scalars are in the wavefronts' registers when these start (-amdgpu-kernarg-preload-count; a struct stays
// in memory), so that a row's words are asked for at once and not after a trip for their addresses.  us per pass before and
// after, the structs first: mask + sample of 4,096 rows at V = 1,024 fp32 11.71 / 11.03 (of 128 at V = 50,265 fp32: no more than
// two runs differ); decoding step by step 2,048 rows at V = 32k 566.5 / 559.1 and 1,024 at V = 50k 269.5 / 265.8.

// ------------------------------------------------------------------------------------------
// ppv_next_token_mask: one workgroup per prefix.
__global__ __launch_bounds__(MASK_THREADS) void mask_kernel(const int32_t *__restrict__ prefixes,
                                                            const int32_t *__restrict__ lens, int32_t stride,
                                                            uint32_t *__restrict__ mask,
                                                            uint32_t *__restrict__ range_lo,
                                                            uint32_t *__restrict__ range_hi,
                                                            uint8_t *__restrict__ member, IndexView ix) {
    extern __shared__ __align__(16) uint32_t smem[];
    const int n_words = ix.n_words;
    uint32_t *img = smem;            // [n_words]
    uint32_t *bc = smem + n_words;   // [5]: slot, found, cb, ce, only
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    if (wave == 0) {
        const int32_t mine = first_tokens(prefixes + (size_t)b * (size_t)stride, stride, lane);
        int t = lens[b];
        t = t < 0 ? 0 : (t > stride ? stride : t);
        Walk w = walk_prefix(ix, prefixes + (size_t)b * (size_t)stride, mine, t, lane);
        if (lane == 0) {
            bc[0] = w.slot;
            bc[1] = w.found ? 1u : 0u;
            bc[2] = w.found ? w.cb : 0u;
            bc[3] = w.found ? w.ce : 0u;
            bc[4] = w.only;
            if (range_lo) range_lo[b] = w.lo;
            if (range_hi) range_hi[b] = w.hi;
            if (member) member[b] = w.member ? 1 : 0;
        }
    }
    __syncthreads();
    const uint32_t slot = bc[0];
    const bool found = bc[1] != 0u;
    const uint32_t cb = bc[2], ce = bc[3];
    uint32_t *out = mask + (size_t)b * (size_t)n_words;
    // rows are written 16 bytes per lane when every row starts on a 16-byte boundary
    const bool wide = (n_words & 3) == 0 && (((uintptr_t)mask) & 15u) == 0;
    const int n_quads = n_words >> 2;
    const uint32_t only = bc[4];
    if (only != PPV_NO_SLOT) {   // one bit
        const int at = (int)((only & PPV_NODE_TOKEN) >> 5);
        const uint32_t bit = 1u << (only & 31u);
        auto word = [&](int i) { return i == at ? bit : 0u; };
        if (wide) {
            for (int i = tid; i < n_quads; i += MASK_THREADS)
                ((uint4 *)out)[i] = make_uint4(word(4 * i), word(4 * i + 1), word(4 * i + 2), word(4 * i + 3));
        } else {
            for (int i = tid; i < n_words; i += MASK_THREADS) out[i] = word(i);
        }
        return;
    }
    if (found && ce - cb > ix.heavy_min) {  // ready-made image: plain copy
        const uint32_t *src = ix.heavy_bits + (size_t)slot * (size_t)n_words;
        if (wide && (((uintptr_t)ix.heavy_bits) & 15u) == 0) {
            for (int i = tid; i < n_quads; i += MASK_THREADS) ((uint4 *)out)[i] = ((const uint4 *)src)[i];
        } else {
            for (int i = tid; i < n_words; i += MASK_THREADS) out[i] = src[i];
        }
        return;
    }
    if (cb == ce) {  // not in S, or a member without extensions
        if (wide) {
            for (int i = tid; i < n_quads; i += MASK_THREADS) ((uint4 *)out)[i] = make_uint4(0u, 0u, 0u, 0u);
        } else {
            for (int i = tid; i < n_words; i += MASK_THREADS) out[i] = 0u;
        }
        return;
    }
    for (int i = tid; i < n_words; i += MASK_THREADS) img[i] = 0u;
    __syncthreads();
    for (uint32_t i = cb + (uint32_t)tid; i < ce; i += MASK_THREADS) {
        uint32_t v = ix.ent[i].tok & PPV_NODE_TOKEN;
        atomicOr(&img[v >> 5], 1u << (v & 31u));
    }
    __syncthreads();
    if (wide) {
        for (int i = tid; i < n_quads; i += MASK_THREADS) ((uint4 *)out)[i] = ((const uint4 *)img)[i];
    } else {
        for (int i = tid; i < n_words; i += MASK_THREADS) out[i] = img[i];
    }
}

// The same for vocabularies of at most 2,048 tokens (a mask row is at most 64 words: one word per lane): one
// wavefront per prefix, four prefixes per workgroup, no LDS and no barrier.  A listed node has at most V / 32 <= 64
// children here, one per lane; each child's bit is set by the lane that holds its word.
constexpr int MASK_SMALL_WORDS = WAVE;
__global__ __launch_bounds__(MASK_THREADS) void mask_rows_kernel(const int32_t *__restrict__ prefixes,
                                                                 const int32_t *__restrict__ lens, int32_t stride, int B,
                                                                 uint32_t *__restrict__ mask,
                                                                 uint32_t *__restrict__ range_lo,
                                                                 uint32_t *__restrict__ range_hi,
                                                                 uint8_t *__restrict__ member, IndexView ix) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int b = blockIdx.x * (MASK_THREADS / WAVE) + threadIdx.x / WAVE;
    if (b >= B) return;  // uniform per wavefront
    const int n_words = ix.n_words;
    const int32_t mine = first_tokens(prefixes + (size_t)b * (size_t)stride, stride, lane);
    int t = lens[b];
    t = t < 0 ? 0 : (t > stride ? stride : t);
    const Walk w = walk_prefix<false, false>(ix, prefixes + (size_t)b * (size_t)stride, mine, t, lane);
    if (lane == 0) {
        if (range_lo) range_lo[b] = w.lo;
        if (range_hi) range_hi[b] = w.hi;
        if (member) member[b] = w.member ? 1 : 0;
    }
    uint32_t word = 0u;
    const uint32_t nchild = w.found ? w.ce - w.cb : 0u;
    if (w.only != PPV_NO_SLOT) {
        if ((uint32_t)lane == (w.only & PPV_NODE_TOKEN) >> 5) word = 1u << (w.only & 31u);
    } else if (nchild > ix.heavy_min) {   // ready-made image
        if (lane < n_words) word = ix.heavy_bits[(size_t)heavy_slot_of(ix, w.node) * (size_t)n_words + lane];
    } else if (nchild > 0u) {      // nchild <= heavy_min <= 64
        const uint32_t tok = (uint32_t)lane < nchild ? (ix.ent[w.cb + (uint32_t)lane].tok & PPV_NODE_TOKEN) : 0u;
        for (uint32_t i = 0; i < nchild; i++) {   // uniform trip count
            const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)tok, (int)i);
            if ((uint32_t)lane == (v >> 5)) word |= 1u << (v & 31u);
        }
    }
    if (lane < n_words) mask[(size_t)b * (size_t)n_words + lane] = word;
}

// ------------------------------------------------------------------------------------------
// Tiles.  A tile is what one wavefront loads with four 16-byte loads per lane: 2048 bf16 or 1024
// fp32 tokens.  Load j of lane l holds the EPL consecutive tokens starting at
// tile*TILE + j*64*EPL + l*EPL, so token order inside a tile is (j, lane, k).
template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr int EPL = 4;  // tokens per 16-byte load
    __device__ static __forceinline__ void unpack(const u32x4 &r, float x[4]) {
        x[0] = __uint_as_float(r.x); x[1] = __uint_as_float(r.y);
        x[2] = __uint_as_float(r.z); x[3] = __uint_as_float(r.w);
    }
};
template <> struct Elem<uint16_t> {  // bf16: widening to fp32 is exact
    static constexpr int EPL = 8;
    __device__ static __forceinline__ void unpack(const u32x4 &r, float x[8]) {
        x[0] = __uint_as_float(r.x << 16); x[1] = __uint_as_float(r.x & 0xFFFF0000u);
        x[2] = __uint_as_float(r.y << 16); x[3] = __uint_as_float(r.y & 0xFFFF0000u);
        x[4] = __uint_as_float(r.z << 16); x[5] = __uint_as_float(r.z & 0xFFFF0000u);
        x[6] = __uint_as_float(r.w << 16); x[7] = __uint_as_float(r.w & 0xFFFF0000u);
    }
};
// The same as unpack, with values that the compiler takes for new ones each time: what is unpacked is used at once and
// not kept in registers for another use of the tile (there is one in a rare case, and tiles are held packed).
template <typename T> __device__ __forceinline__ void unpack_fresh(const u32x4 &r, float x[Elem<T>::EPL]) {
    if (sizeof(T) == 4) {
#pragma unroll
        for (int i = 0; i < 4; i++) x[i] = __uint_as_float(r[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            asm volatile("v_lshlrev_b32 %0, 16, %1" : "=v"(x[(2 * i) % Elem<T>::EPL]) : "v"(r[i]));
            asm volatile("v_and_b32 %0, %2, %1" : "=v"(x[(2 * i + 1) % Elem<T>::EPL]) : "v"(r[i]), "s"(0xFFFF0000u));
        }
    }
}
template <typename T> struct TileGeom {
    static constexpr int EPL = Elem<T>::EPL;
    static constexpr int PER_LOAD = WAVE * EPL;   // tokens covered by one load of the wave
    static constexpr int TILE = 4 * PER_LOAD;     // tokens per tile
    static constexpr int WORDS = TILE / 32;       // mask words per tile
    static constexpr int LANES_PER_WORD = 32 / EPL;
};

struct RawTile {
    u32x4 r[4];
    uint32_t word;   // image path: this lane's word of the tile's mask (requested together with the tile)
};

// A tile is requested with four unconditional 16-byte loads wherever it lies, also at the row's end and behind it; group_of puts
// -inf behind the end when the tile is used.  Nothing is conditional between request and use, so the compiler can
// count the loads in flight and wait for exactly the ones a use needs, and the ragged last tile is one like the others.
// One addition makes the four addresses (clamped into the row by comparisons, as here before, they took twelve).
template <typename T>
__device__ __forceinline__ void load_tile(const Row &row, int tile, int lane, RawTile &rt) {
    const uint32_t at = (uint32_t)tile * (4 * WAVE * 16u) + (uint32_t)lane * 16u;
#pragma unroll
    for (int j = 0; j < 4; j++) rt.r[j] = __builtin_amdgcn_raw_buffer_load_b128(row.buf, at + j * (WAVE * 16u), 0, 2 /* non-temporal */);
}
constexpr int NO_TILE = 1 << 18;   // behind every row: a request that reads nothing
// The tile's tokens that lie inside the row, counted from this lane's first one (PAD: what is behind the row's end counts
// as -inf; only the row's last tile has any of that).
template <typename T> __device__ __forceinline__ int tokens_left(int V, int tile, int lane) {
    return V - tile * TileGeom<T>::TILE - lane * TileGeom<T>::EPL;
}
// group j of a tile, unpacked
template <typename T, bool PAD> __device__ __forceinline__ void group_of(const RawTile &rt, int j, int left, float x[TileGeom<T>::EPL]) {
    unpack_fresh<T>(rt.r[j], x);
    if (PAD) {
        int in = left - j * TileGeom<T>::PER_LOAD;
        asm("" : "+v"(in));   // (or the compiler compares `left` with a constant for each token, each in a register of its own)
#pragma unroll
        for (int k = 0; k < TileGeom<T>::EPL; k++) x[k] = k < in ? x[k] : -INFINITY;
    }
}

// word wi of a V-bit image, with bits at positions >= V cleared (0 beyond the image), in two parts: the load, unconditional
// (clamped index: a conditional load would make later waits conservative), and what is done to the word once it is
// used (at the load it would wait for it, and for every tile asked for before).
__device__ __forceinline__ uint32_t image_word_raw(const uint32_t *__restrict__ image, int wi, int V) {
    const int last = (V + 31) / 32 - 1;
    return image[wi < last ? wi : last];
}
__device__ __forceinline__ uint32_t image_word_fix(uint32_t w, int wi, int V) {
    const int last = (V + 31) / 32 - 1;
    if (wi == last && (V & 31)) w &= (1u << (V & 31)) - 1u;
    return wi <= last ? w : 0u;
}
__device__ __forceinline__ uint32_t image_word(const uint32_t *__restrict__ image, int wi, int V) {
    return image_word_fix(image_word_raw(image, wi, V), wi, V);
}
// the tile's mask word for this lane (lane l < WORDS holds word l of the tile), in the same two parts
template <typename T> __device__ __forceinline__ uint32_t tile_word_raw(const uint32_t *__restrict__ image, int tile, int lane, int V) {
    using G = TileGeom<T>;
    return image_word_raw(image, tile * G::WORDS + (lane < G::WORDS ? lane : 0), V);
}
template <typename T> __device__ __forceinline__ uint32_t tile_word_fix(uint32_t w, int tile, int lane, int V) {
    using G = TileGeom<T>;
    return lane < G::WORDS ? image_word_fix(w, tile * G::WORDS + lane, V) : 0u;
}
template <typename T>
__device__ __forceinline__ uint32_t tile_mask_word(const uint32_t *__restrict__ image, int tile, int lane, int V) {
    return tile_word_fix<T>(tile_word_raw<T>(image, tile, lane, V), tile, lane, V);
}

// mask bits of this lane's EPL tokens of load j, from the tile's mask words (lane l < WORDS holds word l)
template <typename T> __device__ __forceinline__ uint32_t lane_bits(uint32_t tile_word, int j, int lane) {
    using G = TileGeom<T>;
    uint32_t w = (uint32_t)__shfl((int)tile_word, j * (G::WORDS / 4) + lane / G::LANES_PER_WORD, WAVE);
    return (w >> ((lane % G::LANES_PER_WORD) * G::EPL)) & ((1u << G::EPL) - 1u);
}

// References far from 0.  With |m*c| of 2^31 and more the rounding of m*c is beyond the range of exp2, and a product with a
// stand-in for -inf (the type's lowest number, -1e30) is outside fp32.  An exact maximum is therefore taken no lower than
// m*c = -FAR (far tokens weigh nothing against that).  Where a whole row, or its largest token, lies beyond that on either side, the
// differences are taken first: x - m is exact for an x of m's sign, up to twice and down to half its size, and the others weigh nothing.
// (Checked per row and per exact maximum, not per token: 0 to 1 % of a call.  The difference first for every token of these
// tiles took filtered rows of V = 32k, 2,048 of them, from 22.8 us to 25.0, and one argument more for the bound took a decoding
// step of 256 rows from 6.13 to 6.27: a register that the loads ahead of the first tile then waited for.)
constexpr float FAR = 134217728.f;   // 2^27: below it the rounding of m*c is at most four units of the exponent
__device__ __forceinline__ bool far_off(float m, float c) { return fabsf(m * c) >= FAR; }
__device__ __forceinline__ float not_below(float ref, float c) {   // (ref: uniform; -inf, an empty tile, stays that)
    if (__builtin_expect(ref * c <= -FAR, 0) && ref != -INFINITY) {
        asm volatile("" : "+s"(c));   // (computed here: as an argument of the kernel, or ahead of a loop, it costs the usual row a register)
        ref = -FAR * __builtin_amdgcn_rcpf(c);
    }
    return ref;
}
// what to take from the tokens, and what to weigh them against then
struct Shifted {
    float sub, m;
};
__device__ __forceinline__ Shifted shifted(float m, float c) {
    const bool far = far_off(m, c);
    return {far ? m : 0.f, far ? 0.f : m};
}

// Statistics of one tile: a reference m, sum_all = sum exp(x - m), and (image) sum_val over valid tokens.
// Any reference gives the same sums up to rounding as long as they stay inside fp32's range, so neither the maximum nor
// the reduction over the wavefront it would need are computed.
//   without an image   (list_stats) only the sum over all tokens is wanted, and it only ever enters a logarithm: m is the
//          largest of the first 16 bytes of lanes 0 to 3 (two steps within a quad).  Where that is -inf, or so low (REF_LOW)
//          that it is a caller's stand-in for -inf, the row has been filtered; where a token lies more than about REF_GUARD * T
//          above m, the sum is not inside SUM_MOST: then the tile, still in its registers, is summed again with its
//          exact maximum.  (The farther a token lies above m, the larger the arguments
//          of exp and log and the more their rounding weighs: with sums allowed up to 1e30 and m from lane 0 alone, the
//          largest error of logZ_valid went from 2e-6 to 1.1e-5 in rows with a token 55 T above the rest.)
//   image  (image_stats) the sums over valid tokens set the sampling threshold, and with tens of thousands of valid tokens
//          another rounding of them moves a draw now and then: m is the largest of lane 0's own tokens, as long as no token of
//          the tile lies more than REF_GUARD * T above it and it is no stand-in either, else the exact maximum.
// Either way m depends on the row's values alone, not on how the row is split over wavefronts.  m = -inf: an empty tile.
//
// exp(x - m) = 2^(x*c - m*c).  m*c is rounded once (mc); its residual is a factor of the tile's sums (rounding_of).  Without
// an image that factor is left to combine_tiles, which has a tile per lane there.
//
// What a tile costs is the instructions a SIMD issues for it: a quarter of a wavefront's lanes a cycle, an exponential a
// sixteenth.  1,024 fp32 tokens are 16 exponentials, multiply-adds and additions: 384 cycles; 2,048 of bf16, with the
// unpacking, 896.  What surrounds them (addresses, reference, reduction, checks, keeping the result) took about 50 instructions
// and an exponential a tile and takes about 20: one addition for the addresses, reductions of one instruction a step, the
// first group unpacked once, checks by scalar compares, results in a register's lanes until the wavefront's last tile.
// The second copy of the sums for tiles that are summed again stands out of the way of the first.  Tiles that were set aside
// and loaded once more behind the others took filtered rows up to twice as long (constrained_sample, 50 tokens left of
// V = 32k, 2,048 rows: 47.5 us against 25.3; V = 50k fp32, 384 rows: 29.8 against 16.4).
constexpr float REF_GUARD = 40.f;   // exp(40) * 2048 tokens is far inside fp32
constexpr float SUM_MOST = 2.353852668e17f;   // exp(REF_GUARD)
constexpr float REF_LOW = -5e3f;
// (as unsigned numbers, negative floats grow with their size, and infinities and NaNs are above the other positive ones)
__device__ __forceinline__ bool too_low(float ref) { return __float_as_uint(ref) >= __float_as_uint(REF_LOW); }
__device__ __forceinline__ bool settled(float zall) { return __float_as_uint(zall) <= __float_as_uint(SUM_MOST); }
__device__ __forceinline__ float rounding_of(float ref, float c) { return fast_exp2(-fmaf(ref, c, -(ref * c))); }
__device__ __forceinline__ float uniform(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }
template <int EPL> __device__ __forceinline__ float group_sum(const float x[EPL], float c, float mc, float zall) {
#pragma unroll
    for (int k = 0; k < EPL; k++) zall += fast_exp2(fmaf(x[k], c, -mc));
    return zall;
}
template <typename T, bool PAD> __device__ __forceinline__ void list_stats(const RawTile &rt, int left, const Temper &tp, float &m_out, float &zall_out) {
    using G = TileGeom<T>;
    float x[G::EPL];
    group_of<T, PAD>(rt, 0, left, x);
    float mx = x[0];
#pragma unroll
    for (int k = 1; k < G::EPL; k++) mx = fmaxf(mx, x[k]);
    const float ref = uniform(quad_max(mx)), mc = ref * tp.c;
    m_out = ref;
    zall_out = INFINITY;   // (not settled)
    // (before the sums: rows filtered to 50 tokens, the rest -1e4, 2,048 at V = 32k, take 22.9 us like this and 29.3 where every tile is
    // summed first)
    if (__builtin_expect(too_low(ref), 0)) return;   // (uniform)
    float zall = group_sum<G::EPL>(x, tp.c, mc, 0.f);
#pragma unroll
    for (int j = 1; j < 4; j++) {
        __builtin_amdgcn_sched_barrier(0);   // one group's tokens in registers at a time
        group_of<T, PAD>(rt, j, left, x);
        zall = group_sum<G::EPL>(x, tp.c, mc, zall);
    }
    zall_out = wave_sum(zall);
}
template <typename T, bool PAD> __device__ __forceinline__ float lane_max(const RawTile &rt, int left) {
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        float x[TileGeom<T>::EPL];
        group_of<T, PAD>(rt, j, left, x);
#pragma unroll
        for (int k = 0; k < TileGeom<T>::EPL; k++) mx = fmaxf(mx, x[k]);
        __builtin_amdgcn_sched_barrier(0);
    }
    return mx;
}
// the same relative to the exact maximum, for tiles that are not settled by list_stats
template <typename T, bool PAD> __device__ __forceinline__ void exact_stats(const RawTile &rt, int left, const Temper &tp, float &m_out, float &zall_out) {
    using G = TileGeom<T>;
    const float ref = not_below(wave_max(lane_max<T, PAD>(rt, left)), tp.c), mc = ref * tp.c;
    float zall = 0.f;
    if (ref != -INFINITY) {   // (uniform)
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float x[G::EPL];
            group_of<T, PAD>(rt, j, left, x);
            zall = group_sum<G::EPL>(x, tp.c, mc, zall);
            __builtin_amdgcn_sched_barrier(0);
        }
        zall = wave_sum(zall);
    }
    m_out = ref;
    zall_out = zall;
}
template <typename T, bool PAD>
__device__ __forceinline__ void image_stats(const RawTile &rt, uint32_t tile_word, int lane, int left, const Temper &tp,
                                            float &m_out, float &zall_out, float &zval_out) {
    using G = TileGeom<T>;
    const float mx = lane_max<T, PAD>(rt, left);
    float ref = uniform(mx);
    if (too_low(ref) || __ballot(mx > ref + tp.guard) != 0ull) ref = not_below(wave_max(mx), tp.c);   // (uniform)
    float zall = 0.f, zval = 0.f;
    if (ref != -INFINITY) {   // (uniform)
        const float mc = ref * tp.c;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float x[G::EPL];
            group_of<T, PAD>(rt, j, left, x);
            const uint32_t bits = lane_bits<T>(tile_word, j, lane);
#pragma unroll
            for (int k = 0; k < G::EPL; k++) {
                const float e = fast_exp2(fmaf(x[k], tp.c, -mc));
                zall += e;
                const uint32_t keep = (uint32_t)(-(int32_t)((bits >> k) & 1u));
                zval += __uint_as_float(__float_as_uint(e) & keep);
            }
            __builtin_amdgcn_sched_barrier(0);   // one group's tokens in registers at a time
        }
        const float fix = rounding_of(ref, tp.c);
        zall = wave_sum(zall) * fix;
        zval = wave_sum(zval) * fix;
    }
    m_out = ref;
    zall_out = zall;
    zval_out = zval;
}

// A row too far from 0 for its tiles' sums shows in their total, which is then 0, infinite or NaN: a scalar compare.
__device__ __forceinline__ bool no_sum(float za) { return __float_as_uint(za) - 1u >= __float_as_uint(INFINITY) - 1u; }
// ... as does one of nothing but -inf, or with a NaN or +inf, which is left as it is.  (At temperatures below 1e-4 a reference just
// above REF_LOW may be far off, whatever the row's largest token is.)
__device__ __forceinline__ bool is_far(float M, float c) { return fabsf(M) < INFINITY && (far_off(M, c) || REF_LOW * c <= -FAR); }
// A far row's largest token, and the sum over all tokens relative to it: by one wavefront, from memory, in as little code as it takes.
template <typename T> __device__ __forceinline__ void far_row(const T *row, int V, int lane, const Temper &tp, float &M, float &za) {
    constexpr int EPL = Elem<T>::EPL;
    const Row all = row_of(row, V);
    float top = -INFINITY, z = 0.f;
#pragma unroll 1
    for (int pass = 0; pass < 2; pass++) {
#pragma unroll 1
        for (int at = lane * EPL; at < V; at += WAVE * EPL) {
            float x[EPL];
            Elem<T>::unpack(__builtin_amdgcn_raw_buffer_load_b128(all.buf, (uint32_t)at * (uint32_t)sizeof(T), 0, 0), x);
            float m = -INFINITY, e = 0.f;
#pragma unroll
            for (int k = 0; k < EPL; k++) {
                const float v = at + k < V ? x[k] : -INFINITY;
                m = fmaxf(m, v);
                e += fast_exp2((v - top) * tp.c);
            }
            if (pass == 0) top = fmaxf(top, m);
            else z += e;
        }
        if (pass == 0) top = wave_max(top);
    }
    M = top;
    za = wave_sum(z);
}

// Rare path of the image mode (the valid tokens lie far below the row maximum, so sums relative
// to the tile maxima would lose them): maximum over the valid tokens of a tile ...
template <typename T>
__device__ __forceinline__ float tile_valid_max(const RawTile &rt, uint32_t tile_word, int lane) {
    using G = TileGeom<T>;
    float mv = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        float x[G::EPL];
        unpack_fresh<T>(rt.r[j], x);
        const uint32_t bits = lane_bits<T>(tile_word, j, lane);
#pragma unroll
        for (int k = 0; k < G::EPL; k++)
            if ((bits >> k) & 1u) mv = fmaxf(mv, x[k]);
    }
    return wave_max(mv);
}
// ... and the valid sum of a tile relative to a given reference (finite)
template <typename T>
__device__ __forceinline__ float tile_valid_sum(const RawTile &rt, uint32_t tile_word, int lane, const Shifted &ref, float c) {
    using G = TileGeom<T>;
    const float mc = ref.m * c;
    const float fix = fast_exp2(-fmaf(ref.m, c, -mc));
    float z = 0.f;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        float x[G::EPL];
        unpack_fresh<T>(rt.r[j], x);
        const uint32_t bits = lane_bits<T>(tile_word, j, lane);
#pragma unroll
        for (int k = 0; k < G::EPL; k++)
            if ((bits >> k) & 1u) z += fast_exp2(fmaf(x[k] - ref.sub, c, -mc));
    }
    return wave_sum(z) * fix;
}

// Locate the sample inside one tile (IMAGE path).  target is the cumulative valid weight to exceed,
// in units of exp(x - m_tile).  Returns the token id (wave-uniform), or -1 if the tile has no valid
// token with positive weight.  When rounding lets no token exceed the target, the last valid token
// with positive weight is returned.
template <typename T>
__device__ __forceinline__ int locate_in_tile(const RawTile &rt, uint32_t tile_word, int tile, int lane, const Shifted &ref,
                                     double target, float tc) {
    using G = TileGeom<T>;
    const float mc = ref.m * tc;
    const float fix = fast_exp2(-fmaf(ref.m, tc, -mc));
    double before = 0.0;  // valid weight of the loads already passed
    int last_valid = -1;
    for (int j = 0; j < 4; j++) {
        __builtin_amdgcn_sched_barrier(0);   // (one group at a time, as in image_stats)
        float x[G::EPL], e[G::EPL];
        unpack_fresh<T>(rt.r[j], x);
        const uint32_t bits = lane_bits<T>(tile_word, j, lane);
        float grp = 0.f;
        int my_last = -1;
#pragma unroll
        for (int k = 0; k < G::EPL; k++) {
            e[k] = ((bits >> k) & 1u) ? fast_exp2(fmaf(x[k] - ref.sub, tc, -mc)) * fix : 0.f;
            grp += e[k];
            if (e[k] > 0.f) my_last = k;
        }
        const double incl = before + wave_incl_scan((double)grp);
        const uint64_t cross = __ballot(incl > target);
        const int first_tok = tile * G::TILE + j * G::PER_LOAD;
        if (cross) {
            const int l = __ffsll((long long)cross) - 1;
            int id = -1;
            if (lane == l) {
                double c = incl - (double)grp;
                for (int k = 0; k < G::EPL; k++) {
                    c += (double)e[k];
                    if (e[k] > 0.f && c > target) { id = k; break; }
                }
                if (id < 0) id = my_last;  // rounding inside the group
                if (id >= 0) id += first_tok + lane * G::EPL;   // (-1: a target below zero met a lane without a valid token)
            }
            return lane_value(id, l);
        }
        const uint64_t have = __ballot(my_last >= 0);
        if (have) {
            const int l = 63 - __clzll((long long)have);
            last_valid = lane_value(first_tok + lane * G::EPL + my_last, l);
        }
        before = last_lane(incl);
    }
    return last_valid;
}

// ------------------------------------------------------------------------------------------
// One row by one workgroup of `nw` wavefronts.
template <int TILES, int LIST> struct RowSharedT {
    float tile_m[TILES];
    float tile_zall[TILES];
    float tile_zval[TILES];
    float tile_ref[TILES];             // what tile_zval is relative to (the tile maximum, or the valid maximum)
    uint32_t list_tok[LIST + 1];       // valid tokens in increasing order (list path), flags in the top bits
    uint32_t list_child[LIST + 1];     // decode step: child offsets of the listed entries
    float list_e[LIST];                // exp(l - slice max) per listed token
    float slice_m[LIST / WAVE];
    float slice_z[LIST / WAVE];
    int tile_cnt[TILES];               // valid tokens per tile (mask -> list conversion)
    int bc_i[8];
    float bc_f[4];
};
using RowShared = RowSharedT<MAX_TILES, PPV_LIST_MAX>;
// Rows of at most SMALL_TILES tiles whose lists hold at most SMALL_LIST tokens (V <= 2048: the list limit is
// V / 32): 1 KB of LDS per row instead of 18 KB, so that the compute unit is filled by registers, not by LDS.
constexpr int SMALL_TILES = 4, SMALL_LIST = 64;
using RowSharedSmall = RowSharedT<SMALL_TILES, SMALL_LIST>;

struct RowOut {
    int32_t id;        // sampled token or -1
    int32_t pos;       // list path: position of the sampled token in the list, else -1
    float logZ_valid;
    float logZ_all;
    bool mine;         // this thread holds the row's result (wavefront 0 of the workgroup that finishes the row;
                       // every thread of it with ALL)
};

// Words that the workgroups of a split row hand to one another (see SplitRow) are written and read with device-scope
// accesses (each goes to the level of the memory system that all compute units share), so that no fence over the whole
// cache is needed: a device-wide fence per wavefront cost 30 us per launch.
template <typename W> __device__ __forceinline__ void shared_put(W *p, W v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename W> __device__ __forceinline__ W shared_get(const W *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A row shared by `parts` workgroups (see SplitRow); parts == 1: one workgroup has the row to itself and
// nothing else here is looked at.
struct Split {
    int parts;
    int part;             // this workgroup's number, 0 .. parts-1
    SplitRow *row;        // the row's scratch
    uint32_t *arrivals;   // the row's arrival counter
    uint32_t mark;        // of the call
};
template <bool SPLIT> __device__ __forceinline__ Split split_of(int shift) {
    if (!SPLIT) return {1, 0, nullptr, nullptr, 0u};
    return {1 << shift, (int)(blockIdx.x & ((1u << shift) - 1u)), nullptr, nullptr, 0u};
}
// (Where it is needed, not when the kernel starts: on the way through the index there is no room for it in the scalar registers.)
template <bool SPLIT> __device__ __forceinline__ void find_area(Split &sp, SplitScratch *scratch, int b, uint32_t mark) {
    if (!SPLIT) return;
    sp.row = &scratch->row[b];
    sp.arrivals = &scratch->arrivals[b];
    sp.mark = mark;
}
__device__ __forceinline__ void send(Marked *p, float v, uint32_t mark) { shared_put(p, (uint64_t)mark << 32 | __float_as_uint(v)); }
__device__ __forceinline__ void send(MarkedPair *p, float a, float b, uint32_t mark) {
    send(&p->first, a, mark);
    send(&p->second, b, mark);
}
__device__ __forceinline__ void clear(MarkedPair *p) {
    shared_put(&p->first, (Marked)0);
    shared_put(&p->second, (Marked)0);
}
__device__ __forceinline__ MarkedPair look(const MarkedPair *p) { return {shared_get(&p->first), shared_get(&p->second)}; }
__device__ __forceinline__ bool has(Marked w, uint32_t mark) { return (uint32_t)(w >> 32) == mark; }
__device__ __forceinline__ bool has(const MarkedPair &w, uint32_t mark) { return has(w.first, mark) && has(w.second, mark); }
__device__ __forceinline__ float value(Marked w) { return __uint_as_float((uint32_t)w); }
// Waits for words that have been sent, by a whole wavefront: look_again() at all of them as long as one lane's there() is false.  False if they
// do not come: two launches use one area at a time, which no caller may do.  (The row then has no result, and says so: id -1, masses NaN.)
constexpr uint32_t MOST_LOOKS = 1u << 16;      // a word that has been sent comes within microseconds
constexpr uint32_t LOOK_ONCE = 1u << 29;       // of a mark (tests): no further look
template <typename THERE, typename LOOK> __device__ __forceinline__ bool wait_for(const Split &sp, THERE there, LOOK look_again) {
    uint32_t n = 0;
    while (__ballot(!there()) != 0ull) {   // (uniform: what is live here is in scalar registers, of which there are too few)
        if (n++ >= MOST_LOOKS || (sp.mark & LOOK_ONCE)) return false;
        look_again();
    }
    return true;
}
// Counts this workgroup: true for the one that arrives last.  (The count goes from parts - 1 to 0, and from anything that is more: what launches
// that may not have met here leave in it makes some workgroup of a later one the last, which waits for the words of the others.)
__device__ __forceinline__ bool arrive(const Split &sp) { return atomicInc(sp.arrivals, (uint32_t)sp.parts - 1u) >= (uint32_t)sp.parts - 1u; }

// Where the workgroups of a row meet: by wavefront 0 of each, after a barrier behind the last word the workgroup has sent.  True for the
// one that arrives last, which then has every tile's statistics in its LDS; nobody waits for a workgroup that has not arrived.
// A word says by itself whether it is there, so nothing is waited for between the words and the counter, and the words are looked at
// before the counter has answered: one trip to memory that all compute units share, where there were three (the words acknowledged,
// the counter, the words).
// `listed`: of the row's listed tokens, at most 64 (0: there are none, or they need no sums).
template <typename SH> __device__ __forceinline__ bool meet(const Split &sp, SH &sh, int nt, int listed, int lane, bool &lost) {
    constexpr int PER = MAX_TILES / WAVE;
    MarkedPair w[PER], slice = {0u, 0u};
    Marked e = 0u;
    auto look_at_all = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < PER; j++)
            if (j * WAVE < nt) w[j] = look(&sp.row->tile[min(lane + j * WAVE, nt - 1)]);   // (no lane without a word: conditions are registers)
        if (listed) {
            slice = look(&sp.row->slice[0]);
            e = shared_get(&sp.row->list_e[min(lane, listed - 1)]);
        }
    };
    look_at_all();
    int last = 0;   // (its answer is waited for at once)
    if (lane == 0) last = arrive(sp) ? 1 : 0;
    if (!__builtin_amdgcn_readfirstlane(last)) return false;
    const uint32_t mark = sp.mark;
    auto there = [&]() __attribute__((always_inline)) {
        bool all = !listed || (has(slice, mark) && has(e, mark));
#pragma unroll
        for (int j = 0; j < PER; j++)
            if (j * WAVE < nt) all = all && has(w[j], mark);
        return all;
    };
    lost = !wait_for(sp, there, look_at_all);
#pragma unroll
    for (int j = 0; j < PER; j++) {
        const int k = min(lane + j * WAVE, nt - 1);
        if (j * WAVE < nt) {
            sh.tile_m[k] = value(w[j].first);
            sh.tile_zall[k] = value(w[j].second);
        }
    }
    if (listed) {
        if (lane == 0) {
            sh.slice_m[0] = value(slice.first);
            sh.slice_z[0] = value(slice.second);
        }
        if (lane < listed) sh.list_e[lane] = value(e);
    }
    // (zeros, for a graph, all of whose replays have one mark; after the last look, which waits for what was stored before it)
    for (int k = lane; k < nt; k += WAVE) clear(&sp.row->tile[k]);
    if (lane < listed) shared_put(&sp.row->list_e[lane], (Marked)0);
    if (listed && lane == 0) clear(&sp.row->slice[0]);
    return true;
}

enum ValidMode { VALID_NONE = 0, VALID_LIST = 1, VALID_IMAGE = 2 };

// A wavefront's share of a row: of `nw` wavefronts number `wave` has the tiles wave, wave + nw, ...  It takes them from a place
// on that the workgroup's number sets, and the last one, which may be ragged, last.  (Rows that are started together are
// otherwise read in step, and what is asked for at one time lies at the same place of a thousand rows: us per call, in
// step and like this, ppv_sample_next, 1,024 rows, V = 256k bf16 96.2 / 88.4, V = 128k 48.8 / 47.1; the decoding loop, 2,048
// rows at V = 32k, 547.7 / 541.2.  The sixteen places in the order of their bits reversed: neighbours start far apart.)
struct Share {
    int wave, nw, n, turn;   // n: tiles
    __device__ __forceinline__ int first() const { return wave + turn * nw; }
    __device__ __forceinline__ int at(int i) const {   // the i-th tile it takes
        int q = i + turn;
        q = q >= n - 1 ? q - (n - 1) : q;
        return wave + (i < n - 1 ? q : i) * nw;
    }
};
// `wave_v`: the wavefront's number among all that share the row, over all its workgroups
__device__ __forceinline__ Share share_of(int nt, int wave_v, int nw) {
    const int wave = __builtin_amdgcn_readfirstlane(wave_v);   // scalar: loop control stays uniform
    Share s = {wave, nw, 0, 0};
    const int up = nt - wave + nw - 1;
    if ((nw & (nw - 1)) == 0) s.n = up >> __builtin_ctz((unsigned)nw);   // (a division is a hundred cycles before the first load)
    else for (int x = up; x >= nw; x -= nw) s.n++;
    // (where a row has sixteen wavefronts it is nearly alone on its compute unit, and the numbers would only be waited for:
    // constrained_sample, 128 rows at V = 50,265 fp32, 11.0 us without, 11.8 with a turn)
    if ((nw <= 8 || (nw & (nw - 1)) != 0) && s.n > 2) s.turn = (int)((__brev(blockIdx.x) >> 28) * (uint32_t)(s.n - 1) >> 4);
    return s;
}
// Streams a row's tiles through one wavefront's share of the work.  Per tile the statistics go to LDS: under an image at once;
// else, two numbers, they are kept in the lanes of two registers (the wavefront's first tile in lane 0, ...) and written together.
//
// Two register tiles take turns: while one is reduced, the other is on its way.  No load is conditional (see load_tile:
// a tile that is not there costs nothing), so every wait is for loads issued a known number of loads ago.
// `mid` is work of the caller's that needs no tile (the sums over the listed tokens): it is run once, where this
// wavefront has just asked for a tile and would only wait for it.
// X: the share's first tile; `pub`: of a split row, the statistics are left for the workgroup that finishes it.
// IMAGE: the row may have an image (nullptr: it has none; one loop for both, so that the tiles stay in their registers).
template <typename T, bool IMAGE, typename SH, typename MID>
__device__ __forceinline__ void stream_tiles(const Row &row, int V, RawTile &X,
                                    const uint32_t *__restrict__ image, SH &sh, int lane, const Share &share,
                                    const Temper &tp, MID &mid, bool pub, const Split sp) {
    using G = TileGeom<T>;
    if (share.n == 0) {
        mid();
        return;
    }
    float kept_m = 0.f, kept_z = 0.f;   // lane i: the i-th tile since they were written last
    auto write_kept = [&](int n, int i_first) __attribute__((always_inline)) {
        if (lane < n) {
            const int k = share.at(i_first + lane);
            sh.tile_m[k] = kept_m;
            sh.tile_zall[k] = kept_z;
            if (pub) send(&sp.row->tile[k], kept_m, kept_z, sp.mark);
        }
    };
    auto reduce_tile = [&](const RawTile &t, int k, int i, auto pad) __attribute__((always_inline)) {
        constexpr bool PAD = decltype(pad)::value;
        const int left = PAD ? tokens_left<T>(V, k, lane) : 0;
        float m, zall, zval;
        if (IMAGE && image) {
            image_stats<T, PAD>(t, tile_word_fix<T>(t.word, k, lane, V), lane, left, tp, m, zall, zval);
            if (lane == 0) {
                sh.tile_m[k] = m;
                sh.tile_zall[k] = zall;
                sh.tile_zval[k] = zval;
                sh.tile_ref[k] = m;
                if (pub) {
                    send(&sp.row->tile[k], m, zall, sp.mark);
                    send(&sp.row->valid[k], zval, sp.mark);
                }
            }
        } else {
            list_stats<T, PAD>(t, left, tp, m, zall);
            if (__builtin_expect(!settled(zall), 0)) exact_stats<T, PAD>(t, left, tp, m, zall);
            kept_m = lane == (i & (WAVE - 1)) ? m : kept_m;
            kept_z = lane == (i & (WAVE - 1)) ? zall : kept_z;
        }
    };
    auto reduce_last = [&](const RawTile &t, int k, int i) __attribute__((always_inline)) {   // the row's last tile is the last one of its wavefront
        if ((k + 1) * G::TILE > V) reduce_tile(t, k, i, std::true_type());
        else reduce_tile(t, k, i, std::false_type());
    };
    // a tile and its mask word (without an image: of a row of no length, so that the number of loads is the same)
    const Row words = row_of<uint32_t, 3u>(image, IMAGE && image ? (V + 31) / 32 : 0);
    auto fetch_word = [&](RawTile &t, int k) __attribute__((always_inline)) {
        if (IMAGE) t.word = __builtin_amdgcn_raw_buffer_load_b32(words.buf, (uint32_t)(k * G::WORDS + lane) * 4u, 0, 0);
    };
    auto fetch = [&](RawTile &t, int k) __attribute__((always_inline)) {
        load_tile<T>(row, k, lane, t);
        fetch_word(t, k);
    };
    const int n = share.n;
    fetch_word(X, share.first());
    RawTile Y;
    fetch(Y, n > 1 ? share.at(1) : NO_TILE);
    mid();
    int i = 0, written = 0;
    for (; i + 2 < n; i += 2) {
        reduce_tile(X, share.at(i), i, std::false_type());
        fetch(X, share.at(i + 2));
        reduce_tile(Y, share.at(i + 1), i + 1, std::false_type());
        fetch(Y, i + 3 < n ? share.at(i + 3) : NO_TILE);
        if (i + 2 - written == WAVE) {   // (a wavefront with more tiles than lanes: large batches of the loop kernel, two wavefronts to a row)
            if (!(IMAGE && image)) write_kept(WAVE, written);
            written += WAVE;
        }
    }
    if (i + 1 < n) {
        reduce_tile(X, share.at(i), i, std::false_type());
        reduce_last(Y, share.at(i + 1), i + 1);
    } else {
        reduce_last(X, share.at(i), i);
    }
    if (!(IMAGE && image)) write_kept(n - written, written);
}

// Row totals from the per-tile statistics in LDS (without an image: not yet rid of the rounding of their references, see
// list_stats): the largest tile reference M, the sum over all tokens relative
// to it and (image rows) the sum over valid tokens.  Called by a whole wavefront; results are uniform.  The sum over
// all tokens only ever enters a logarithm, so it is added up in fp32 (a tree over at most 256 positive terms: a few
// 1e-7 relative); the valid sum sets the sampling threshold and is added up in fp64.  A far row (see far_off) is summed again
// from memory, and its valid sum left at 0: the caller then sums the valid tokens again, relative to their own maximum.
template <typename SH>
__device__ __forceinline__ void add_tiles(const SH &sh, int nt, int lane, const Temper &tp, bool image, float &M, float &za,
                                     double &zv) {
    if (nt <= WAVE) {   // (uniform) one tile per lane at most: both words in one round of LDS reads, no loops; the
                        // same operations in the same order as below, so the same bits
        const bool have = lane < nt;
        const float m = have ? sh.tile_m[have ? lane : 0] : -INFINITY;
        const float z = have ? sh.tile_zall[have ? lane : 0] : 0.f;
        const float zval = (image && have) ? sh.tile_zval[have ? lane : 0] : 0.f;
        M = wave_max(m);
        float a = 0.f;
        double v = 0.0;
        if (m != -INFINITY) {
            const float sc = exp_scale(m - M, tp.c);
            a = (image ? z : z * rounding_of(m, tp.c)) * sc;
            if (image) v = (double)zval * (double)sc;
        }
        za = wave_sum(a);
        zv = image ? wave_sum(v) : 0.0;
        return;
    }
    M = -INFINITY;
    for (int k = lane; k < nt; k += WAVE) M = fmaxf(M, sh.tile_m[k]);
    M = wave_max(M);
    za = 0.f;
    zv = 0.0;
    for (int k = lane; k < nt; k += WAVE) {
        const float m = sh.tile_m[k];
        if (m != -INFINITY) {
            const float sc = exp_scale(m - M, tp.c);
            const float z = sh.tile_zall[k];
            za += (image ? z : z * rounding_of(m, tp.c)) * sc;
            if (image) zv += (double)sh.tile_zval[k] * (double)sc;   // (the other modes have no per-tile valid sums)
        }
    }
    za = wave_sum(za);
    if (image) zv = wave_sum(zv);
}
template <typename T, typename SH>
__device__ __forceinline__ void combine_tiles(const SH &sh, const T *row, int V, int nt, int lane, const Temper &tp, bool image, float &M,
                                     float &za, double &zv) {
    add_tiles(sh, nt, lane, tp, image, M, za, zv);
    if (__builtin_expect(no_sum(za), 0)) {   // (uniform)
        if (!is_far(M, tp.c)) return;
        far_row<T>(row, V, lane, tp, M, za);
        zv = 0.0;
    }
}

// A list of at most 63 valid tokens that one wavefront holds in registers, entry i in lane i (the per-step decode
// kernel): the sums over the list and the sample, with the arithmetic of the list path of row_sample for a list of
// one slice, so that both give the same bits.  gx: lane i < n_list holds the listed token's logit, the others -inf.
struct RegList {
    bool on;         // (uniform) the row's valid set is held this way
    bool have_gx;    // (uniform) the listed logits have been requested already and are in gx
    uint32_t tokw;   // lane i < n_list: the entry's token word (token | flags)
    float gx;
};
struct ListPick {
    int id, pos;     // sampled token and its position in the list; -1: nothing can be sampled
    float Mv;        // largest listed logit (-inf: no listed token has positive weight)
    double zvl;      // sum of the listed tokens' weights relative to Mv
};
__device__ __forceinline__ ListPick reg_list_pick(float gx, uint32_t tokw, int n_list, float u, int lane, const Temper &tp) {
    ListPick pk;
    pk.id = -1;
    pk.pos = -1;
    pk.zvl = 0.0;
    if (n_list == 1) {
        // One listed token: what the general case below computes, without its reductions and scans over the lanes
        // (every other lane contributes an exact zero): the weight exp(x - x), through the same rounded steps, is
        // the sum; the token is drawn whatever u is, unless its weight is 0.
        const float g = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(gx)));
        const float m = g == g ? g : -INFINITY;   // (a NaN is passed over, as the maximum over the lanes does)
        pk.Mv = m;
        if (m == -INFINITY) return pk;
        const float mc = m * tp.c;
        const float product = fast_exp2(fmaf(m, tp.c, -mc)) * fast_exp2(-fmaf(m, tp.c, -mc));
        const float e = far_off(m, tp.c) ? fast_exp2(m - m) : product;
        pk.zvl = (double)e;
        if (e > 0.f) {
            pk.pos = 0;
            pk.id = (int)((uint32_t)__builtin_amdgcn_readfirstlane((int)tokw) & PPV_NODE_TOKEN);
        }
        return pk;
    }
    const float m = wave_max(gx);
    pk.Mv = m;
    if (m == -INFINITY) return pk;
    float near = m;
    if (__builtin_expect(far_off(m, tp.c), 0)) {   // (uniform)
        gx -= m;
        near = 0.f;
    }
    const float mc = near * tp.c;
    const float fix = fast_exp2(-fmaf(near, tp.c, -mc));
    float e = fast_exp2(fmaf(gx, tp.c, -mc)) * fix;   // gx = -inf gives 0
    const double zvl = (double)wave_sum(e);
    pk.zvl = zvl;
    const double tau = (double)u * zvl;
    double target;
    int s;
    if (zvl > tau) {
        s = 0;
        target = tau;
    } else {
        s = zvl > 0.0 ? 0 : -1;
        target = INFINITY;
    }
    if (!(s >= 0 && lane < n_list)) e = 0.f;
    const double ic = wave_incl_scan((double)e);
    const uint64_t c2 = __ballot(e > 0.f && ic > target);
    const uint64_t h2 = __ballot(e > 0.f);
    if (c2 | h2) {
        const int l = c2 ? __ffsll((long long)c2) - 1 : 63 - __clzll((long long)h2);
        pk.pos = l;
        pk.id = (int)(lane_value(tokw, l) & PPV_NODE_TOKEN);
    }
    return pk;
}

// Streams the row and samples.  Called by every thread of the workgroup with uniform arguments.
//   first        this wave's first tile, already loaded (share_of(...).first())
//   next_row     optional: another row whose first tile (per wave) is to be requested into *next_first
//   mode         VALID_LIST: sh.list_tok[0..n_list) holds the valid tokens (in LDS, barrier done)
//                VALID_IMAGE: image (global memory, V bits) is the valid set
//                VALID_NONE: the valid set is empty
//   ALL          every thread gets the result (one more barrier); otherwise only wavefront 0 does
//   sp           the row's split over workgroups: the wavefronts are then numbered over all its workgroups, and only the
//                workgroup that arrives last goes on to sample (the others return with mine == false)
//   SPLIT        compiled in only for kernels that may share a row between workgroups (the others pay nothing for it)
template <typename T, typename SH, bool ALL, bool SPLIT>
__device__ __forceinline__ RowOut row_sample(const T *__restrict__ row, int V, RawTile &first, int mode, int n_list,
                                    const uint32_t *__restrict__ image, float u, SH &sh, int tid, int nw,
                                    const Temper &tp, const Split &sp, const T *__restrict__ next_row = nullptr,
                                    RawTile *next_first = nullptr) {
    using G = TileGeom<T>;
    const int lane = tid & (WAVE - 1), wave = tid / WAVE;
    const int nt = (V + G::TILE - 1) / G::TILE;
    // the wavefront's number and count over all workgroups of the row: tiles and list slices are dealt out by these
    const int parts = SPLIT ? sp.parts : 1;
    const int vwave = SPLIT ? sp.part * nw + wave : wave, vnw = parts * nw;
    const bool pub = SPLIT && parts > 1;
    const Share share = share_of(nt, vwave, vnw);

    // ---- list path, part 1: ask for the listed tokens' logits now (they are being streamed
    // anyway, so these are cache hits) so that they arrive while the tiles are reduced
    const int ns = (n_list + WAVE - 1) / WAVE;
    float gx = -INFINITY;   // this lane's listed logit of the wave's first slice
    if (mode == VALID_LIST && vwave < ns) {
        const int i = vwave * WAVE + lane;
        if (i < n_list) {
            const uint32_t v = sh.list_tok[i] & PPV_NODE_TOKEN;
            if (sizeof(T) == 4) gx = __uint_as_float(((const uint32_t *)row)[v]);
            else gx = __uint_as_float(((uint32_t)((const uint16_t *)row)[v]) << 16);
        }
    }

    // ---- list path, part 2: sums per slice of 64 listed tokens, relative to the slice maximum.  Run from inside
    // the stream, while the wavefront waits for a tile it has just asked for; after it when there is no such wait.
    auto list_sums = [&]() {
        if (mode != VALID_LIST) return;
        for (int s = vwave; s < ns; s += vnw) {
            const int i = s * WAVE + lane;
            float x = gx;
            if (s != vwave) {
                x = -INFINITY;
                if (i < n_list) {
                    const uint32_t v = sh.list_tok[i] & PPV_NODE_TOKEN;
                    if (sizeof(T) == 4) x = __uint_as_float(((const uint32_t *)row)[v]);
                    else x = __uint_as_float(((uint32_t)((const uint16_t *)row)[v]) << 16);
                }
            }
            const float m = wave_max(x);
            float e = 0.f;
            if (m != -INFINITY) {
                const Shifted ref = shifted(m, tp.c);
                const float mc = ref.m * tp.c;
                const float fix = fast_exp2(-fmaf(ref.m, tp.c, -mc));
                e = fast_exp2(fmaf(x - ref.sub, tp.c, -mc)) * fix;   // x = -inf gives 0
            }
            if (i < n_list) {
                sh.list_e[i] = e;
                if (pub) send(&sp.row->list_e[i], e, sp.mark);
            }
            const float z = wave_sum(e);
            if (lane == 0) {
                sh.slice_m[s] = m;
                sh.slice_z[s] = z;
                if (pub) send(&sp.row->slice[s], m, z, sp.mark);
            }
        }
    };
    // ---- stream: every tile once
    stream_tiles<T, true, SH>(row_of(row, V), V, first, mode == VALID_IMAGE ? image : nullptr, sh, lane, share, tp, list_sums, pub, sp);
    // (decode loop) the row of the next step is known already: ask for this wave's first tile of it
    // now, so that it travels while this row is combined and sampled
    if (next_row && share.n > 0) load_tile<T>(row_of(next_row, V), share.first(), lane, *next_first);
    RowOut none;
    none.id = -1;
    none.pos = -1;
    none.logZ_valid = -INFINITY;
    none.logZ_all = 0.f;
    none.mine = false;
    if (SPLIT && parts > 1) {
        __syncthreads();   // all words of this workgroup have been sent
        const int listed = mode == VALID_LIST ? n_list : 0;
        if (mode != VALID_IMAGE && listed <= WAVE) {
            if (wave != 0) return none;
            bool lost = false;
            if (!meet(sp, sh, nt, listed, lane, lost)) return none;
            if (lane == 0) sh.bc_i[0] = lost ? 2 : 1;
        } else {
            // (many words: by every wavefront, which the rare second pass over an image row needs too; no thread without a word)
            const int nthreads = nw * WAVE;
            const SplitRow *words = sp.row;
            const bool image_row = mode == VALID_IMAGE;
            const uint32_t mark = sp.mark;
            int k = min(tid, nt - 1), i = min(tid, listed - 1);
            const int q = min(tid, ns - 1);   // (at most sixteen slices)
            MarkedPair tile, slice = {0u, 0u};
            Marked valid = 0u, e = 0u;
            auto look_at_tile = [&]() __attribute__((always_inline)) {
                tile = look(&words->tile[k]);
                if (image_row) valid = shared_get(&words->valid[k]);
            };
            auto look_at_list = [&]() __attribute__((always_inline)) {
                if (!image_row) {
                    slice = look(&words->slice[q]);
                    e = shared_get(&words->list_e[i]);
                }
            };
            auto there = [&]() __attribute__((always_inline)) {
                return has(tile, mark) && (image_row ? has(valid, mark) : has(slice, mark) && has(e, mark));
            };
            look_at_tile();
            look_at_list();
            if (tid == 0) sh.bc_i[0] = arrive(sp) ? 1 : 0;
            __syncthreads();
            if (!sh.bc_i[0]) return none;      // uniform for the workgroup
            bool came = true;
            // the first tiles and listed tokens of all threads together, then the second ones, ...
            for (int done = 0; done < nt || done < listed; done += nthreads) {
                k = min(tid + done, nt - 1);
                i = min(tid + done, listed - 1);
                if (done) {
                    look_at_tile();
                    look_at_list();
                }
                came = wait_for(sp, there, [&]() __attribute__((always_inline)) {
                    look_at_tile();
                    look_at_list();
                }) && came;
                sh.tile_m[k] = sh.tile_ref[k] = value(tile.first);
                sh.tile_zall[k] = value(tile.second);
                if (image_row) {
                    sh.tile_zval[k] = value(valid);
                } else {
                    sh.slice_m[q] = value(slice.first);
                    sh.slice_z[q] = value(slice.second);
                    sh.list_e[i] = value(e);
                }
            }
            if (!came) sh.bc_i[0] = 2;
            __syncthreads();
            // (the zeros by the wavefronts that have little left to do)
            const int z0 = nw > 1 ? WAVE : 0;
            if (tid >= z0) {
                for (int k = tid - z0; k < nt; k += nthreads - z0) {
                    clear(&sp.row->tile[k]);
                    if (image_row) shared_put(&sp.row->valid[k], (Marked)0);
                }
                for (int i = tid - z0; i < listed; i += nthreads - z0) {
                    shared_put(&sp.row->list_e[i], (Marked)0);
                    if (i < ns) clear(&sp.row->slice[i]);
                }
            }
        }
    } else {
        __syncthreads();
    }

    // Nobody but wavefront 0 has anything left to do when the result goes to it alone and the set is not an
    // image (whose rare second pass needs every wavefront): the others leave its SIMD to it.
    if (!ALL && mode != VALID_IMAGE && wave != 0) return none;
    // ---- combine (every wave computes the same row totals from LDS; cheap, and saves a broadcast)
    float M, za;
    double zv;
    combine_tiles<T>(sh, row, V, nt, lane, tp, mode == VALID_IMAGE, M, za, zv);
    float R = M;  // reference of the valid sums of the image path

    // ---- image path, rare case: the valid mass is below 2^-18 of the row's largest term, so sums
    // relative to the tile maxima are inaccurate or have underflowed.  Redo the valid sums relative
    // to the maximum over valid tokens (the row is re-read; it is still in cache).
    if (mode == VALID_IMAGE && zv < 3.814697265625e-06) {
        __syncthreads();  // everyone has read tile_zval
        RawTile rt;
        for (int k = wave; k < nt; k += nw) {
            load_tile<T>(row_of(row, V), k, lane, rt);   // (what lies behind the row's end has no mask bit)
            const uint32_t word = tile_mask_word<T>(image, k, lane, V);
            const float mv = tile_valid_max<T>(rt, word, lane);
            if (lane == 0) sh.tile_ref[k] = mv;
        }
        __syncthreads();
        float Mv = -INFINITY;
        for (int k = lane; k < nt; k += WAVE) Mv = fmaxf(Mv, sh.tile_ref[k]);
        Mv = wave_max(Mv);
        __syncthreads();  // everyone has read the per-tile valid maxima
        if (Mv != -INFINITY) {
            for (int k = wave; k < nt; k += nw) {
                load_tile<T>(row_of(row, V), k, lane, rt);
                const uint32_t word = tile_mask_word<T>(image, k, lane, V);
                const float z = tile_valid_sum<T>(rt, word, lane, shifted(Mv, tp.c), tp.c);
                if (lane == 0) {
                    sh.tile_zval[k] = z;
                    sh.tile_ref[k] = Mv;
                }
            }
        } else {
            for (int k = tid; k < nt; k += nw * WAVE) sh.tile_zval[k] = 0.f;
        }
        __syncthreads();
        R = Mv;
        zv = 0.0;
        for (int k = lane; k < nt; k += WAVE) zv += (double)sh.tile_zval[k];
        zv = wave_sum(zv);
    }

    // ---- locate: wave 0
    RowOut out = none;
    out.mine = ALL || wave == 0;
    if (wave == 0) {
        const float l2za = fast_log2(za);
        int id = -1, pos = -1;
        float lzv = -INFINITY;
        if (mode == VALID_IMAGE) {
            if (zv > 0.0) {
                lzv = fmaf(R - M, tp.inv, LN2F * (fast_log2((float)zv) - l2za));
                const double tau = (double)u * zv;
                // first tile whose cumulative valid weight exceeds tau
                double carry = 0.0, before = 0.0;
                int kstar = -1, klast = -1;
                for (int k0 = 0; k0 < nt && kstar < 0; k0 += WAVE) {
                    const int k = k0 + lane;
                    double w = 0.0;
                    if (k < nt && sh.tile_zval[k] > 0.f)
                        w = (double)sh.tile_zval[k] * (double)exp_scale(sh.tile_ref[k] - R, tp.c);
                    const double incl = carry + wave_incl_scan(w);
                    const uint64_t cross = __ballot(incl > tau);
                    const uint64_t have = __ballot(w > 0.0);
                    if (cross) {
                        const int l = __ffsll((long long)cross) - 1;
                        kstar = k0 + l;
                        before = lane_value(incl - w, l);
                    } else if (have) {
                        klast = k0 + 63 - __clzll((long long)have);
                    }
                    carry = last_lane(incl);
                }
                double target;
                int kt;
                if (kstar >= 0) {
                    kt = kstar;
                    target = (tau - before) / (double)exp_scale(sh.tile_ref[kt] - R, tp.c);
                } else {  // rounding: the total never exceeded tau; take the last valid token
                    kt = klast;
                    target = INFINITY;
                }
                if (kt >= 0) {   // (no tile qualifies only when NaNs have poisoned the sums: then nothing is sampled)
                    RawTile lt;
                    load_tile<T>(row_of(row, V), kt, lane, lt);
                    const uint32_t word = tile_mask_word<T>(image, kt, lane, V);
                    id = locate_in_tile<T>(lt, word, kt, lane, shifted(sh.tile_ref[kt], tp.c), target, tp.c);
                }
            }
        } else if (mode == VALID_LIST) {
            float Mv = -INFINITY;
            if (ns == 1) {   // one slice (at most 64 listed tokens, the usual case): nothing to scan over
                Mv = sh.slice_m[0];
            } else {
                if (lane < ns) Mv = sh.slice_m[lane];
                Mv = wave_max(Mv);
            }
            if (Mv != -INFINITY) {
                int s;
                double target, zvl;
                if (ns == 1) {   // the general case below, written out for one slice: same values bit for bit
                    zvl = (double)sh.slice_z[0];
                    const double tau = (double)u * zvl;
                    if (zvl > tau) {
                        s = 0;
                        target = tau;
                    } else {
                        s = zvl > 0.0 ? 0 : -1;
                        target = INFINITY;
                    }
                } else {
                    double w = 0.0, sc = 0.0;
                    if (lane < ns && sh.slice_m[lane] != -INFINITY) {
                        const float d = sh.slice_m[lane] - Mv;
                        sc = d * tp.c < -1000.f ? 0.0 : (double)exp_scale(d, tp.c);   // (a far difference has no product)
                        w = (double)sh.slice_z[lane] * sc;
                    }
                    const double incl = wave_incl_scan(w);
                    zvl = last_lane(incl);
                    const double tau = (double)u * zvl;
                    const uint64_t cross = __ballot(incl > tau);
                    const uint64_t have = __ballot(w > 0.0);
                    if (cross) {
                        s = __ffsll((long long)cross) - 1;
                        target = (tau - lane_value(incl - w, s)) / lane_value(sc, s);
                    } else {
                        s = have ? 63 - __clzll((long long)have) : -1;
                        target = INFINITY;
                    }
                }
                lzv = fmaf(Mv - M, tp.inv, LN2F * (fast_log2((float)zvl) - l2za));
                // (no slice or no token qualifies only when NaNs have poisoned the sums: then nothing is sampled,
                // and above all no position outside the list is ever formed)
                const int i = s * WAVE + lane;
                const float e = (s >= 0 && i < n_list) ? sh.list_e[i] : 0.f;
                const double ic = wave_incl_scan((double)e);
                const uint64_t c2 = __ballot(e > 0.f && ic > target);
                const uint64_t h2 = __ballot(e > 0.f);
                if (c2 | h2) {
                    const int l = c2 ? __ffsll((long long)c2) - 1 : 63 - __clzll((long long)h2);
                    pos = s * WAVE + l;
                    id = (int)(sh.list_tok[pos] & PPV_NODE_TOKEN);
                }
            }
        }
        out.id = id;   // all four are wave-uniform
        out.pos = pos;
        out.logZ_valid = lzv;
        out.logZ_all = fmaf(M, tp.inv, LN2F * l2za);
        if (SPLIT && __builtin_expect(sh.bc_i[0] == 2, 0)) {
            out.id = out.pos = -1;
            out.logZ_valid = out.logZ_all = NAN;
        }
        if (ALL && lane == 0) {
            sh.bc_i[0] = out.id;
            sh.bc_i[1] = out.pos;
            sh.bc_f[0] = out.logZ_valid;
            sh.bc_f[1] = out.logZ_all;
        }
    }
    if (ALL) {
        __syncthreads();
        out.id = sh.bc_i[0];
        out.pos = sh.bc_i[1];
        out.logZ_valid = sh.bc_f[0];
        out.logZ_all = sh.bc_f[1];
    }
    return out;
}

// ------------------------------------------------------------------------------------------
// constrained_sample: the valid set arrives as a packed mask.  Count its bits; a small set is
// unpacked into the token list, a large one is used as an image.
template <typename T, bool SMALL, bool SPLIT>
__global__ __launch_bounds__(SMALL ? SMALL_TILES * WAVE : MAX_WAVES * WAVE) void sample_kernel(const T *__restrict__ logits, int64_t row_stride,
                                                                  const uint32_t *__restrict__ mask, int V,
                                                                  int n_words, int list_max, int shape, SplitScratch *scratch,
                                                                  const float *__restrict__ uniforms,
                                                                  int32_t *__restrict__ ids,
                                                                  float *__restrict__ logZ_valid,
                                                                  float *__restrict__ logZ_all, Temper tp, uint32_t mark) {
    using SH = typename std::conditional<SMALL, RowSharedSmall, RowShared>::type;
    __shared__ SH sh;
    // shape: wavefronts per workgroup << 8 (an argument: blockDim would be waited for), and for SPLIT, where a row is shared by
    // a power of two of consecutive workgroups, that power; mark: the call's
    const int split_shift = shape & 255;
    const int b = SPLIT ? (int)(blockIdx.x >> split_shift) : (int)blockIdx.x;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const int nw = shape >> 8;
    Split sp = split_of<SPLIT>(split_shift);
    const int vwave = sp.part * nw + wave;
    const T *row = logits + (size_t)b * (size_t)row_stride;
    const uint32_t *mrow = mask + (size_t)b * (size_t)n_words;
    // The mask row is read as quads of four words per lane: one wavefront load covers 256 words (8,192 tokens), so a
    // wavefront has few loads to wait for, and those it has are requested two at a time and before the logits tile
    // (memory answers a wavefront in the order of its requests: the few bytes the next steps wait for must not queue
    // behind the 4 KB tile; one word per lane and tile at a time cost a memory round trip per tile, which at 63
    // tiles on 4 wavefronts was most of the kernel).  Words past the row read as 0.
    const int n_groups = ((n_words + 3) / 4 + WAVE - 1) / WAVE;   // <= 32 (PPV_MAX_VOCAB / 8192)
    struct Quad {
        uint32_t w[4];
    };
    auto load_quad = [&](int g) {
        Quad q;
        const int wi = (g * WAVE + lane) * 4;
        if (wi + 4 < n_words) {   // inside the row and not its last word: four loads off one address
            const uint32_t *p = mrow + wi;
#pragma unroll
            for (int j = 0; j < 4; j++) q.w[j] = p[j];
        } else {                  // the row's end: clamped loads, bits past V cleared, 0 beyond
#pragma unroll
            for (int j = 0; j < 4; j++) q.w[j] = image_word(mrow, wi + j, V);
        }
        return q;
    };
    auto bits_of = [](const Quad &q) { return (int)(__popc(q.w[0]) + __popc(q.w[1]) + __popc(q.w[2]) + __popc(q.w[3])); };
    const Quad q0 = load_quad(wave), q1 = load_quad(wave + nw);   // (a group past the row: all zero)
    RawTile first;
    const Share share = share_of((V + TileGeom<T>::TILE - 1) / TileGeom<T>::TILE, vwave, sp.parts * nw);
    load_tile<T>(row_of(row, V), share.first(), lane, first);   // in flight during the mask work

    // valid tokens per group of 64 quads (kept in the tile_cnt array: there are fewer groups than tiles)
    const int incl0 = wave_incl_scan(bits_of(q0));
    {
        const int incl1 = wave_incl_scan(bits_of(q1));
        if (lane == WAVE - 1) {
            if (wave < n_groups) sh.tile_cnt[wave] = incl0;
            if (wave + nw < n_groups) sh.tile_cnt[wave + nw] = incl1;
        }
    }
    for (int g = wave + 2 * nw; g < n_groups; g += nw) {   // long rows on few wavefronts
        const int c = wave_sum(bits_of(load_quad(g)));
        if (lane == 0) sh.tile_cnt[g] = c;
    }
    __syncthreads();
    const int total = wave_sum(lane < n_groups ? sh.tile_cnt[lane] : 0);
    const int mode = total == 0 ? VALID_NONE : (total <= list_max ? VALID_LIST : VALID_IMAGE);
    if (mode == VALID_LIST) {
        // a group's valid tokens go to their places in the list: after those of the groups before it, in lane order
        auto unpack_group = [&](int g, const Quad &q, int incl) {
            const int before = wave_sum(lane < g ? sh.tile_cnt[lane] : 0);
            int at = before + incl - bits_of(q);
            const int wi = (g * WAVE + lane) * 4;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                uint32_t w = q.w[j];
                while (w) {
                    const int bit = __ffs((int)w) - 1;
                    sh.list_tok[at++] = (uint32_t)((wi + j) * 32 + bit);
                    w &= w - 1u;
                }
            }
        };
        if (wave < n_groups && sh.tile_cnt[wave] != 0) unpack_group(wave, q0, incl0);
        for (int g = wave + nw; g < n_groups; g += nw) {
            if (sh.tile_cnt[g] == 0) continue;   // (uniform) most groups of a short list hold nothing
            const Quad q = g == wave + nw ? q1 : load_quad(g);
            unpack_group(g, q, wave_incl_scan(bits_of(q)));
        }
        __syncthreads();
    }
    find_area<SPLIT>(sp, scratch, b, mark);
    RowOut r = row_sample<T, SH, false, SPLIT>(row, V, first, mode, mode == VALID_LIST ? total : 0, mrow, uniforms[b], sh, tid, nw, tp, sp);
    if (r.mine && tid == 0) {
        ids[b] = r.id;
        logZ_valid[b] = r.logZ_valid;
        if (logZ_all) logZ_all[b] = r.logZ_all;
    }
}

// Rows of a single tile (V <= 1,024 fp32 / 2,048 bf16 tokens): one wavefront per row, four rows per workgroup,
// everything in registers -- no LDS, no barrier.  The valid set is applied as bits in the tile (as on the image
// path of the general kernel, with the same rescue when the valid tokens lie far below the row maximum).
//
// What bounds it is the instructions: 4,096 rows are four wavefronts to a SIMD, and each issues some hundreds for its tile.  The valid
// tokens' weights that the sums are made of stay in registers and the token is found from them, where they were computed a second time
// (with the mask's bits brought to their lanes again, and the last token of each lane that has a weight); a row with one valid token needs no
// search.  The lanes' mask bits come from memory, a byte each, not over four exchanges between lanes.  us per call before / after:
// 4,096 rows of constrained_sample at V = 1,024 fp32 5.7 / 4.5, V = 2,048 bf16 8.1 / 5.9; 16,384 rows 14.4 / 11.1, 22.3 / 16.6;
// ppv_sample_next, 4,096 rows 7.1 / 6.3, 9.4 / 7.8.
constexpr int ONE_TILE_ROWS = 4;
struct TileDraw {
    int id;                  // sampled token or -1
    float logZ_valid;
    float m, l2za;           // reference of the row's sum, and log2 of it
};
// bits: this lane's mask bits, group j's in the byte j.  The statistics are image_stats', and the token is locate_in_tile's, with the same
// operations in the same order: a decode step on a row under an image gives the same bits.  (Without the rounding of the reference in the
// weights and in the threshold, sixteen or 32 multiplications and 1 to 3 % of a call fewer, a uniform at the edge between two tokens went to the other one now and then.)
template <typename T, bool PAD>
__device__ __forceinline__ TileDraw draw_in_tile(const T *row, const RawTile &rt, uint32_t bits, float u, int V, int lane, const Temper &tp) {
    using G = TileGeom<T>;
    const int left = tokens_left<T>(V, 0, lane);
    const float mx = lane_max<T, PAD>(rt, left);
    float m = uniform(mx);
    if (too_low(m) || __ballot(mx > m + tp.guard) != 0ull) m = not_below(wave_max(mx), tp.c);   // (uniform)
    float zall = 0.f, zval = 0.f, fix = 0.f;
    float w[4][G::EPL];      // weights of this lane's valid tokens
    if (m != -INFINITY) {    // (uniform)
        const float mc = m * tp.c;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float x[G::EPL];
            group_of<T, PAD>(rt, j, left, x);
#pragma unroll
            for (int k = 0; k < G::EPL; k++) {
                const float e = fast_exp2(fmaf(x[k], tp.c, -mc));
                zall += e;
                w[j][k] = __uint_as_float(__float_as_uint(e) & (uint32_t)(-(int32_t)((bits >> (8 * j + k)) & 1u)));
                zval += w[j][k];
            }
            __builtin_amdgcn_sched_barrier(0);   // one group's tokens in registers at a time
        }
        fix = rounding_of(m, tp.c);
        zall = wave_sum(zall) * fix;
        zval = wave_sum(zval) * fix;
    }
    if (__builtin_expect(no_sum(uniform(zall)), 0) && is_far(m, tp.c)) {   // (uniform)
        far_row<T>(row, V, lane, tp, m, zall);
        zval = 0.f;
    }
    TileDraw d = {-1, -INFINITY, m, fast_log2(zall)};
    const uint64_t some = __ballot(bits != 0u);
    if (!some) return d;
    const bool low = zval < 3.814697265625e-06f;   // below 2^-18 of the largest term: sum again, relative to the valid maximum
    if (__builtin_expect(low || far_off(m, tp.c), 0)) {   // (uniform)
        // (the mask's words from the lanes' bits: word i of the tile in lane i)
        uint32_t word = 0u;
        for (int j = 0; j < 4; j++) {
            for (int p = 0; p < G::LANES_PER_WORD; p++) {
                const int from = (lane % (G::WORDS / 4)) * G::LANES_PER_WORD + p;
                const uint32_t b = ((uint32_t)__shfl((int)bits, from, WAVE) >> (8 * j)) & ((1u << G::EPL) - 1u);
                if (lane / (G::WORDS / 4) == j) word |= b << (p * G::EPL);
            }
        }
        float ref = m;
        if (low) {
            ref = tile_valid_max<T>(rt, word, lane);
            zval = ref != -INFINITY ? tile_valid_sum<T>(rt, word, lane, shifted(ref, tp.c), tp.c) : 0.f;
        }
        if (zval > 0.f) {
            d.logZ_valid = fmaf(ref - m, tp.inv, LN2F * (fast_log2(zval) - d.l2za));
            d.id = locate_in_tile<T>(rt, word, 0, lane, shifted(ref, tp.c), (double)u * (double)zval, tp.c);
        }
        return d;
    }
    if (!(zval > 0.f)) return d;   // (NaNs: nothing is sampled)
    d.logZ_valid = LN2F * (fast_log2(zval) - d.l2za);
    if ((some & (some - 1ull)) == 0ull) {   // (uniform) the valid tokens are one lane's
        const int l = __ffsll((long long)some) - 1;
        const uint32_t only = lane_value(bits, l);
        if ((only & (only - 1u)) == 0u) {   // one valid token
            const int at = __ffs((int)only) - 1;
            d.id = (at >> 3) * G::PER_LOAD + l * G::EPL + (at & 7);
            return d;
        }
    }
    const double target = (double)u * (double)zval;
    double before = 0.0;   // valid weight of the groups already passed
#pragma unroll
    for (int j = 0; j < 4; j++) {
        float grp = 0.f;
#pragma unroll
        for (int k = 0; k < G::EPL; k++) {
            w[j][k] *= fix;
            grp += w[j][k];
        }
        const double incl = before + wave_incl_scan((double)grp);
        const uint64_t cross = __ballot(incl > target);
        if (cross) {   // (uniform)
            const int l = __ffsll((long long)cross) - 1;
            double c = incl - (double)grp;
            int k_at = -1, k_last = -1;
#pragma unroll
            for (int k = 0; k < G::EPL; k++) {
                c += (double)w[j][k];
                if (w[j][k] > 0.f) k_last = k;
                if (k_at < 0 && w[j][k] > 0.f && c > target) k_at = k;
            }
            if (k_at < 0) k_at = k_last;   // rounding inside the group
            if (k_at >= 0) k_at += j * G::PER_LOAD + lane * G::EPL;   // (-1: a target below zero met a lane without a valid token)
            d.id = lane_value(k_at, l);
            return d;
        }
        before = last_lane(incl);
    }
    // rounding: the total never exceeded the target; the last valid token with a weight
#pragma unroll
    for (int j = 0; j < 4; j++) {
        int k_last = -1;
#pragma unroll
        for (int k = 0; k < G::EPL; k++)
            if (w[j][k] > 0.f) k_last = k;
        const uint64_t have = __ballot(k_last >= 0);
        if (have) {
            const int l = 63 - __clzll((long long)have);
            d.id = lane_value(j * G::PER_LOAD + lane * G::EPL + k_last, l);
        }
    }
    return d;
}
template <typename T>
__global__ __launch_bounds__(ONE_TILE_ROWS *WAVE) void sample_one_tile_kernel(const T *__restrict__ logits, int64_t row_stride,
                                                                              const uint32_t *__restrict__ mask,
                                                                              const float *__restrict__ uniforms, int B,
                                                                              int V, int n_words, int32_t *__restrict__ ids,
                                                                              float *__restrict__ logZ_valid,
                                                                              float *__restrict__ logZ_all, Temper tp) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int b = blockIdx.x * ONE_TILE_ROWS + __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    if (b >= B) return;   // uniform per wavefront
    const T *row = logits + (size_t)b * (size_t)row_stride;
    using G = TileGeom<T>;
    // (a row of the mask as a buffer: what is behind its last word is 0)
    const Row words = row_of<uint32_t, 3u>(mask + (size_t)b * (size_t)n_words, n_words);
    uint32_t part[4];
#pragma unroll
    for (int j = 0; j < 4; j++)
        part[j] = __builtin_amdgcn_raw_buffer_load_b8(words.buf, (uint32_t)(j * G::PER_LOAD / 8) + (uint32_t)(lane * G::EPL / 8), 0, 0);
    const float u = uniforms[b];
    RawTile rt;
    load_tile<T>(row_of(row, V), 0, lane, rt);
    uint32_t bits = part[0] | part[1] << 8 | part[2] << 16 | part[3] << 24;
    if (sizeof(T) == 4) bits = (bits >> ((lane & 1) * 4)) & 0x0F0F0F0Fu;   // a byte is two lanes'
    TileDraw d;
    if (V == G::TILE) {
        d = draw_in_tile<T, false>(row, rt, bits, u, V, lane, tp);
    } else {
        const int left = tokens_left<T>(V, 0, lane);
#pragma unroll
        for (int j = 0; j < 4; j++) {   // bits at positions >= V do not count
            const int in = left - j * G::PER_LOAD;
            if (in < G::EPL) bits &= ~(0xFFu << (8 * j)) | (in > 0 ? ((1u << in) - 1u) << (8 * j) : 0u);
        }
        d = draw_in_tile<T, true>(row, rt, bits, u, V, lane, tp);
    }
    if (lane == 0) {
        ids[b] = d.id;
        logZ_valid[b] = d.logZ_valid;
        if (logZ_all) logZ_all[b] = fmaf(d.m, tp.inv, LN2F * d.l2za);
    }
}

// ppv_sample_next for rows of a single tile: the prefix walk of mask_rows_kernel and the arithmetic of
// sample_one_tile_kernel in one wavefront per row; the valid set never exists outside this wavefront's registers
// (lane l holds word l of it, which is also word l of the tile's mask).
template <typename T>
__global__ __launch_bounds__(ONE_TILE_ROWS *WAVE) void sample_next_one_tile_kernel(
    const int32_t *__restrict__ prefixes, const int32_t *__restrict__ lens, const float *__restrict__ uniforms,
    const T *__restrict__ logits, int64_t row_stride, int32_t stride, int B, int32_t *__restrict__ ids,
    float *__restrict__ logZ_valid, uint8_t *__restrict__ member, Temper tp, IndexView ix) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int b = blockIdx.x * ONE_TILE_ROWS + __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    if (b >= B) return;   // uniform per wavefront
    const int V = ix.vocab, n_words = ix.n_words;
    const int32_t mine = first_tokens(prefixes + (size_t)b * (size_t)stride, stride, lane);   // before the tile: answers come in order
    int t = lens[b];
    const float u = uniforms[b];
    RawTile rt;
    const T *row = logits + (size_t)b * (size_t)row_stride;
    load_tile<T>(row_of(row, V), 0, lane, rt);   // in flight during the walk
    t = t < 0 ? 0 : (t > stride ? stride : t);
    const Walk w = walk_prefix<false, false>(ix, prefixes + (size_t)b * (size_t)stride, mine, t, lane);
    uint32_t word = 0u;
    const uint32_t nchild = w.found ? w.ce - w.cb : 0u;
    if (w.only != PPV_NO_SLOT) {
        if ((uint32_t)lane == (w.only & PPV_NODE_TOKEN) >> 5) word = 1u << (w.only & 31u);
    } else if (nchild > ix.heavy_min) {   // ready-made image
        if (lane < n_words) word = ix.heavy_bits[(size_t)heavy_slot_of(ix, w.node) * (size_t)n_words + lane];
    } else if (nchild > 0u) {      // nchild <= heavy_min <= 64: one child per lane
        const uint32_t tok = (uint32_t)lane < nchild ? (ix.ent[w.cb + (uint32_t)lane].tok & PPV_NODE_TOKEN) : 0u;
        for (uint32_t i = 0; i < nchild; i++) {   // uniform trip count
            const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)tok, (int)i);
            if ((uint32_t)lane == (v >> 5)) word |= 1u << (v & 31u);
        }
    }
    uint32_t bits = 0u;
#pragma unroll
    for (int j = 0; j < 4; j++) bits |= lane_bits<T>(word, j, lane) << (8 * j);
    const TileDraw d = V == TileGeom<T>::TILE ? draw_in_tile<T, false>(row, rt, bits, u, V, lane, tp) : draw_in_tile<T, true>(row, rt, bits, u, V, lane, tp);
    if (lane == 0) {
        ids[b] = d.id;
        if (logZ_valid) logZ_valid[b] = d.logZ_valid;
        if (member) member[b] = w.member ? 1 : 0;
    }
}

// ------------------------------------------------------------------------------------------
// ppv_decode_begin: one wavefront per row walks the row's current prefix and leaves the cursor.
__global__ __launch_bounds__(MASK_THREADS) void decode_begin_kernel(const int32_t *__restrict__ prefixes,
                                                                    const int32_t *__restrict__ lens, int32_t stride,
                                                                    int B, RowState *__restrict__ state,
                                                                    uint8_t *__restrict__ active,
                                                                    float *__restrict__ logx, IndexView ix) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int b = blockIdx.x * (MASK_THREADS / WAVE) + threadIdx.x / WAVE;
    if (b >= B) return;  // uniform per wave
    const int32_t mine = first_tokens(prefixes + (size_t)b * (size_t)stride, stride, lane);
    int t = lens[b];
    t = t < 0 ? 0 : (t > stride ? stride : t);
    const Walk w = walk_prefix<true>(ix, prefixes + (size_t)b * (size_t)stride, mine, t, lane);
    if (lane == 0) {
        RowState st;
        st.node = w.found ? w.node : PPV_NO_SLOT;
        st.cb = w.found ? w.cb : 0u;
        st.ce = w.found ? w.ce : 0u;
        st.slot = (w.found && w.ce - w.cb > ix.heavy_min) ? w.slot : PPV_NO_SLOT;
        st.tok0 = st.child0 = st.child1 = st.flags = 0u;   // nothing looked ahead
        state[b] = st;
        active[b] = (w.found && !w.member) ? 1 : 0;
        if (logx) logx[b] = 0.f;
    }
}

// ppv_decode_begin_empty: every row starts from the empty candidate.  The cursor is the root's, the same for all
// rows: no prefix to read, no walk; the lengths are written too, so that a decode loop needs no separate fill.
__global__ __launch_bounds__(MASK_THREADS) void decode_begin_empty_kernel(int B, int32_t *__restrict__ lens,
                                                                          RowState *__restrict__ state,
                                                                          uint8_t *__restrict__ active,
                                                                          float *__restrict__ logx, IndexView ix) {
    const int b = blockIdx.x * MASK_THREADS + threadIdx.x;
    if (b >= B) return;
    RowState st;
    st.node = 0u;
    st.cb = ix.ent[0].child;
    st.ce = ix.ent[1].child;
    st.slot = st.ce - st.cb > ix.heavy_min ? heavy_slot_of(ix, 0u) : PPV_NO_SLOT;
    st.tok0 = st.child0 = st.child1 = st.flags = 0u;   // nothing looked ahead
    lens[b] = 0;
    state[b] = st;
    active[b] = 1;   // the empty sequence is a prefix of every member and is no member itself (members are not empty)
    if (logx) logx[b] = 0.f;
}

// ppv_decode_step / ppv_decode_loop: take the children of the row's prefix as the valid set (list, or
// the ready-made image of a heavy node), stream + sample, append, and report whether the extended
// row is in S.  LOOP: the same for n_steps steps in one launch, one workgroup staying with its row;
// the cursor lives in registers.  Where the row is certain to go on (no child of the current prefix is a member),
// the next step's first tiles are requested early: in chains of single children while this step's last ones are reduced
// (LOOP with REG), and with the list in LDS before the step is sampled.  The other steps of LOOP with REG start with nothing
// requested.
template <typename T, bool LOOP, bool SPLIT, bool REG>
__global__ __launch_bounds__((LOOP && !REG ? LOOP_WAVES : MAX_WAVES) * WAVE, LOOP ? 4 : 1) void decode_kernel(
    uint8_t *__restrict__ active, int32_t *__restrict__ lens, RowState *__restrict__ state, const float *__restrict__ uniforms,
    float *__restrict__ logx, const T *__restrict__ logits, int flags, int shape, int32_t *__restrict__ prefixes,
    int32_t stride, int n_steps, int B, int64_t row_stride, int64_t step_stride, int32_t *__restrict__ ids,
    float *__restrict__ logZ_valid, SplitScratch *scratch, Temper tp, IndexView ix) {
    // flags: from bit 2 on the call's mark (see SplitRow); bit 1 (ppv_decode_first_step): every row starts from the empty candidate here and now -- no flags, length
    // or cursor are read, the root's cursor is taken instead, and all of them are written at the end.
    const int advance = flags & 1;
    const bool fresh = (flags & 2) != 0;
    // advance == 0 (ppv_sample_next): every row takes part, a token is drawn, and nothing of the caller's rows is
    // changed (no append, no cursor, no flags)
    using G = TileGeom<T>;
    constexpr bool STEP_REG = REG && !LOOP, LOOP_REG = REG && LOOP;
    // (the loop kernel's fast steps alternate between two sets of tile statistics, see below)
    __shared__ RowShared shs[LOOP_REG ? 2 : 1];
    RowShared &sh = shs[0];
    // shape: as for sample_kernel (the loop kernel never splits rows)
    const int split_shift = shape & 255;
    static_assert(!(LOOP && SPLIT), "the loop kernel keeps a row in one workgroup");
    const int b = SPLIT ? (int)(blockIdx.x >> split_shift) : (int)blockIdx.x;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const int nw = LOOP ? blockDim.x / WAVE : shape >> 8;   // (the loop kernel's registers come out better with blockDim: 384 rows at V = 50k fp32 142 us against 149)
    Split sp = split_of<SPLIT>(split_shift);
    const int vwave = sp.part * nw + wave;
    // REG: there is a cursor, and a list of at most 63 children is kept in wavefront 0's registers, with a look one level
    // ahead for the next cursor (see RowState); large batches of the loop kernel and calls without a cursor
    // use the list in LDS.  (C3, B = 2,048, the loop step by step: 594 us with the list in LDS, 559 like this.)
    // the independent per-row loads go out together
    uint8_t on = active ? active[b] : (uint8_t)1;
    int t = lens[b];
    RowState st;
    if (REG || state) st = state[b];
    else st.flags = 0u;
    float u = uniforms[b];
    // the running score is read now, not when it is updated at the very end (a load there would stand between the
    // sample and the kernel's last store); unconditional, from an address that always exists
    float logx_in = (logx ? logx : uniforms)[b];
    if (fresh) {   // (uniform) what was loaded is set aside -- the loads themselves stay unconditional, so that the
                   // waits after them stay exact -- for the root's cursor, as ppv_decode_begin_empty writes it
        on = 1;
        t = 0;
        logx_in = 0.f;
        st.node = 0u;
        st.cb = ix.ent[0].child;
        st.ce = ix.ent[1].child;
        st.slot = st.ce - st.cb > ix.heavy_min ? heavy_slot_of(ix, 0u) : PPV_NO_SLOT;
        st.tok0 = st.child0 = st.child1 = st.flags = 0u;
    }
    if (!on) return;  // uniform for the workgroup
    const int V = ix.vocab;
    const T *row = logits + (size_t)b * (size_t)row_stride;
    const int nt = (V + G::TILE - 1) / G::TILE;
    // The cursor comes from memory that the caller owns.  One that cannot be a cursor of this index (a state
    // that never went through ppv_decode_begin, or of another index) must not send a load out of bounds:
    // such a row is treated as having no valid token and retires; a look-ahead that cannot be one is ignored.
    auto check_cursor = [&]() {
        const uint32_t nc = st.ce - st.cb;
        const bool sane = st.node < ix.n_nodes && st.cb <= st.ce && st.ce <= ix.n_nodes &&
                          (st.slot == PPV_NO_SLOT ? nc <= ix.heavy_min : st.slot < ix.n_heavy);
        if (!sane) {
            st.cb = st.ce = 0u;
            st.slot = PPV_NO_SLOT;
        }
        if (st.flags != 1u || (st.tok0 & PPV_NODE_TOKEN) >= (uint32_t)V || st.child0 > st.child1 || st.child1 > ix.n_nodes)
            st.flags = 0u;
    };
    // Register list (wavefront 0): entry i of the node's children in lane i, one entry more than there are children
    // (it closes the last child's own range), and under each child the look-ahead for the next cursor.
    RegList rl;
    rl.on = false;
    rl.have_gx = false;
    rl.tokw = 0u;
    rl.gx = -INFINITY;
    uint32_t rl_child = 0u;                              // lane i <= n: child offset of entry i
    uint32_t ahead_tok = 0u, ahead_child = 0u, ahead_next = 0u;   // lane i < n: ent[child_i].tok / .child, ent[child_i + 1].child
    auto look_ahead = [&](int n) {   // (wavefront 0) every address is clamped into the entry array
        if (lane < n) {
            const uint32_t a0 = rl_child < ix.n_nodes ? rl_child : ix.n_nodes;
            const uint32_t a1 = a0 < ix.n_nodes ? a0 + 1u : ix.n_nodes;
            const NodeEnt e0 = ix.ent[a0];
            ahead_tok = e0.tok;
            ahead_child = e0.child;
            ahead_next = ix.ent[a1].child;
        }
    };
    if (STEP_REG) {
        // with a cursor the small loads go out before the 4 KB tile: memory answers a wavefront in request order
        check_cursor();
        const uint32_t nc = st.ce - st.cb;
        rl.on = nc >= 1u && nc < (uint32_t)WAVE && st.slot == PPV_NO_SLOT;   // (uniform)
        if (rl.on && wave == 0) {
            if (nc == 1u && st.flags == 1u) {   // the cursor knows its only child: its logit can be asked for at once
                rl.tokw = lane == 0 ? st.tok0 : 0u;
                rl_child = lane == 0 ? st.child0 : st.child1;
                rl.have_gx = true;
                if (lane == 0) {
                    const uint32_t v = st.tok0 & PPV_NODE_TOKEN;
                    if (sizeof(T) == 4) rl.gx = __uint_as_float(((const uint32_t *)row)[v]);
                    else rl.gx = __uint_as_float(((uint32_t)((const uint16_t *)row)[v]) << 16);
                }
                look_ahead(1);
            } else if ((uint32_t)lane <= nc) {
                const NodeEnt e = ix.ent[st.cb + (uint32_t)lane];
                rl.tokw = e.tok;
                rl_child = e.child;
            }
        }
        rl.have_gx = __builtin_amdgcn_readfirstlane(rl.have_gx ? 1 : 0) != 0 && wave == 0;
    }
    // without a cursor wavefront 0 locates the prefix from the root: its tokens are asked for before the 4 KB tile as well
    const bool locate = !REG && !state;
    int32_t mine = 0;
    if (locate && wave == 0) mine = first_tokens(prefixes + (size_t)b * (size_t)stride, stride, lane);
    RawTile first;
    const Share share = share_of(nt, vwave, sp.parts * nw);
    load_tile<T>(row_of(row, V), share.first(), lane, first);   // in flight during the index work
    t = t < 0 ? 0 : (t > stride ? stride : t);
    uint32_t only = PPV_NO_SLOT;   // without a cursor, the one child of a prefix of a single member: no node is looked at then
    if (locate) {  // (then it shares what it has found; a single child goes straight into the list)
        if (wave == 0) {
            const Walk w = walk_prefix<LOOP>(ix, prefixes + (size_t)b * (size_t)stride, mine, t, lane);
            if (lane == 0) {
                sh.bc_i[3] = (int)w.slot;
                sh.bc_i[4] = (int)(w.found ? w.node : PPV_NO_SLOT);
                sh.bc_i[5] = (int)(w.found ? w.cb : 0u);
                sh.bc_i[6] = (int)(w.found ? w.ce : 0u);
                sh.bc_i[7] = (int)w.only;
                if (!LOOP && w.only != PPV_NO_SLOT) {
                    sh.list_tok[0] = w.only;
                    sh.list_child[0] = sh.list_child[1] = 0u;
                }
            }
        }
        __syncthreads();
        st.node = (uint32_t)sh.bc_i[4];
        st.cb = (uint32_t)sh.bc_i[5];
        st.ce = (uint32_t)sh.bc_i[6];
        only = (uint32_t)sh.bc_i[7];
        st.slot = (st.node != PPV_NO_SLOT && only == PPV_NO_SLOT && st.ce - st.cb > ix.heavy_min) ? (uint32_t)sh.bc_i[3]
                                                                                                : PPV_NO_SLOT;
        if (LOOP) __syncthreads();
    }
    if (!STEP_REG && (LOOP || only == PPV_NO_SLOT)) check_cursor();
    find_area<SPLIT>(sp, scratch, b, (uint32_t)flags >> 2);
    if (STEP_REG && rl.on) {
        // ---- a short list in wavefront 0's registers.  The sample depends on the listed logits alone, not on the
        // row's totals: wavefront 0 draws the token and works out the next cursor while its tile is still on its
        // way; after the barrier only the stores, the totals and the two masses are left.  (Nothing is stored before
        // the barrier: the other wavefronts read the row's flags and cursor when they start, and one that starts
        // late must not find them changed.)
        const int n = (int)(st.ce - st.cb);
        ListPick pk;
        pk.id = -1;
        pk.pos = -1;
        pk.Mv = -INFINITY;
        pk.zvl = 0.0;
        bool drew = false;
        RowState nx = st;
        uint32_t tokw = 0u;
        if (wave == 0) {
            if (!rl.have_gx) {   // (waits for the entries)
                if (lane < n) {
                    const uint32_t v = rl.tokw & PPV_NODE_TOKEN;
                    if (sizeof(T) == 4) rl.gx = __uint_as_float(((const uint32_t *)row)[v]);
                    else rl.gx = __uint_as_float(((uint32_t)((const uint16_t *)row)[v]) << 16);
                }
                look_ahead(n);
            }
            pk = reg_list_pick(rl.gx, rl.tokw, n, u, lane, tp);
            const bool room = t < stride || !advance;
            drew = pk.id >= 0 && room;
            if (drew) {   // (uniform) the sampled child's entry, the one after it and its look-ahead, out of the lanes
                nx.node = st.cb + (uint32_t)pk.pos;
                tokw = lane_value(rl.tokw, pk.pos);
                nx.cb = lane_value(rl_child, pk.pos);
                nx.ce = lane_value(rl_child, pk.pos + 1);
                nx.tok0 = lane_value(ahead_tok, pk.pos);
                nx.child0 = lane_value(ahead_child, pk.pos);
                nx.child1 = lane_value(ahead_next, pk.pos);
                nx.flags = 1u;
                nx.slot = (tokw & PPV_NODE_HEAVY) ? heavy_slot_of(ix, nx.node) : PPV_NO_SLOT;
            }
        }
        struct {
            __device__ void operator()() const {}
        } nothing;
        stream_tiles<T, false, RowShared>(row_of(row, V), V, first, nullptr, sh, lane, share, tp, nothing,
                                          SPLIT && sp.parts > 1, sp);
        __syncthreads();
        if (wave != 0) return;
        // (of a split row every workgroup has drawn the token, and the one that finishes the row stores it)
        bool lost = false;
        if (SPLIT && sp.parts > 1) {
            if (!meet(sp, sh, nt, 0, lane, lost)) return;
            drew = drew && !lost;
        }
        if (lane == 0) {
            if (ids) ids[b] = drew ? pk.id : -1;
            if (drew) {
                if (advance) {
                    prefixes[(size_t)b * (size_t)stride + t] = pk.id;
                    lens[b] = t + 1;
                    state[b] = nx;
                    if (tokw & PPV_NODE_TERMINAL) active[b] = 0;   // the extended row is itself a member
                    else if (fresh) active[b] = 1;
                }
            } else if (advance) {   // the row stops outside S: no valid token of positive weight, or no room
                if (logx) logx[b] = -INFINITY;
                active[b] = 0;
                if (fresh) {
                    lens[b] = 0;
                    state[b] = st;
                }
            }
        }
        if (pk.Mv == -INFINITY) {   // (uniform) no listed token has positive weight
            if (lane == 0 && logZ_valid) logZ_valid[b] = -INFINITY;
            return;
        }
        float M, za;
        double zv;
        combine_tiles<T>(sh, logits + (size_t)b * (size_t)row_stride, V, nt, lane, tp, false, M, za, zv);
        float lzv = fmaf(pk.Mv - M, tp.inv, LN2F * (fast_log2((float)pk.zvl) - fast_log2(za)));
        if (SPLIT && __builtin_expect(lost, 0)) lzv = NAN;
        if (lane == 0) {
            if (logZ_valid) logZ_valid[b] = lzv;
            if (advance && logx && drew) logx[b] = logx_in + lzv;
        }
        return;
    }
    // running log importance score (tid 0); started from the stored value so that the additions happen in
    // the same order as with one launch per step
    float lx = (LOOP && logx) ? logx_in : 0.f;
    bool done = false;
    // LOOP_REG: hand-over from wavefront 0 to the workgroup, written before a fast step's barrier and read after it
    __shared__ struct {
        int done, drew;
        RowState nx;
    } hand[2];
    for (int s = 0; s < n_steps; s++) {
        const uint32_t cb = st.cb, ce = st.ce, slot = st.slot;
        const int nchild = (int)(ce - cb);
        const int mode = nchild == 0 ? VALID_NONE : (slot != PPV_NO_SLOT ? VALID_IMAGE : VALID_LIST);
        if (LOOP_REG && mode == VALID_LIST && nchild == 1 && st.flags == 1u && (nw >= 8 || nt <= 2 * (nw - 1))) {
            // ---- A chain of prefixes with one child each, the cursor knowing the child (nearly all of a long
            // sequence below its first levels).  Wavefront 0 only draws tokens: each step it takes the listed
            // logit that it asked for a step earlier, advances the cursor, asks for the next step's logit and
            // look-ahead, and after the step's barrier adds up the row's totals.  The other wavefronts only stream, over
            // the steps' ends: the next row's first tiles are requested while this row's last ones are reduced, without a
            // copy of, a condition on or a wait for a tile that is still on its way.  One barrier per step; statistics and
            // hand-over alternate between two buffers as in the fast step below.  The chain ends with the row, or at a
            // prefix that is not of this kind, which the code below takes from there.  (With fewer than eight wavefronts
            // one that only draws is missed by the others: those rows take the fast step.)
            const int ntw = nw - 1;
            const int wave_s = __builtin_amdgcn_readfirstlane(wave);
            auto next_in_chain = [&](const RowState &c) {
                return c.ce - c.cb == 1u && c.flags == 1u && c.slot == PPV_NO_SLOT;
            };
            // whether the row has a step after this one (known from the cursor before the token is drawn)
            auto row_goes_on = [&]() { return !(st.tok0 & PPV_NODE_TERMINAL) && s + 1 < n_steps && t + 1 < stride; };
            bool finished = false;   // the row is done, or out of steps
            if (wave_s == 0) {
                float gx = -INFINITY;
                uint32_t a_tok = 0u, a_child = 0u, a_next = 0u;
                auto ask = [&](const T *r, const RowState &c, float &g, uint32_t &x0, uint32_t &x1, uint32_t &x2) {
                    if (lane == 0) {
                        const uint32_t v = c.tok0 & PPV_NODE_TOKEN;
                        if (sizeof(T) == 4) g = __uint_as_float(((const uint32_t *)r)[v]);
                        else g = __uint_as_float(((uint32_t)((const uint16_t *)r)[v]) << 16);
                        const uint32_t a0 = c.child0 < ix.n_nodes ? c.child0 : ix.n_nodes;
                        const uint32_t a1 = a0 < ix.n_nodes ? a0 + 1u : ix.n_nodes;
                        const NodeEnt g0 = ix.ent[a0];
                        x0 = g0.tok;
                        x1 = g0.child;
                        x2 = ix.ent[a1].child;
                    }
                };
                ask(row, st, gx, a_tok, a_child, a_next);
                for (;;) {
                    const bool more = row_goes_on();
                    const ListPick pk = reg_list_pick(gx, lane == 0 ? st.tok0 : 0u, 1, u, lane, tp);
                    const bool drew = pk.id >= 0 && t < stride;
                    RowState nx = st;
                    nx.flags = 0u;
                    if (drew) {
                        nx.node = st.cb;
                        nx.cb = st.child0;
                        nx.ce = st.child1;
                        nx.tok0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)a_tok);
                        nx.child0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)a_child);
                        nx.child1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)a_next);
                        nx.flags = 1u;
                        nx.slot = (st.tok0 & PPV_NODE_HEAVY) ? heavy_slot_of(ix, nx.node) : PPV_NO_SLOT;
                    }
                    const bool chain_on = drew && more && next_in_chain(nx);
                    // (the answers go straight into the registers the next step reads, whose old contents are used up:
                    // a copy of a value that is still on its way would have to wait for it)
                    const float mv = pk.Mv;
                    const double zvl = pk.zvl;
                    const int drawn = pk.id;
                    if (chain_on) ask(row + step_stride, nx, gx, a_tok, a_child, a_next);
                    if (drew && s + 1 < n_steps) u = uniforms[(size_t)(s + 1) * (size_t)B + b];
                    const bool ends = !drew || (st.tok0 & PPV_NODE_TERMINAL) != 0u;
                    if (lane == 0) {
                        hand[s & 1].done = ends ? 1 : 0;
                        hand[s & 1].drew = drew ? 1 : 0;
                        hand[s & 1].nx = nx;
                        if (drew) prefixes[(size_t)b * (size_t)stride + t] = drawn;
                        if (ids) ids[(size_t)s * (size_t)B + b] = drew ? drawn : -1;
                        if (!drew) lx = -INFINITY;   // the row stops outside S
                        if (logZ_valid && mv == -INFINITY) logZ_valid[(size_t)s * (size_t)B + b] = -INFINITY;
                    }
                    __syncthreads();
                    if (mv != -INFINITY) {
                        float M, za;
                        double zv;
                        combine_tiles<T>(shs[s & 1], row, V, nt, lane, tp, false, M, za, zv);
                        const float lzv = fmaf(mv - M, tp.inv, LN2F * (fast_log2((float)zvl) - fast_log2(za)));
                        if (lane == 0) {
                            if (logZ_valid) logZ_valid[(size_t)s * (size_t)B + b] = lzv;
                            if (drew) lx += lzv;
                        }
                    }
                    done = ends;
                    if (drew) {
                        t += 1;
                        st = nx;
                    }
                    if (ends || s + 1 == n_steps) {
                        finished = true;
                        break;
                    }
                    s += 1;
                    row += step_stride;
                    if (!chain_on) break;
                }
            } else {
                // after the step's barrier; true while the chain goes on
                auto step_over = [&](bool more) __attribute__((always_inline)) {
                    __syncthreads();
                    const bool ends = hand[s & 1].done != 0;
                    const bool drew = hand[s & 1].drew != 0;
                    done = ends;
                    if (drew) {
                        t += 1;
                        st = hand[s & 1].nx;
                    }
                    if (ends || s + 1 == n_steps) {
                        finished = true;
                        return false;
                    }
                    s += 1;
                    row += step_stride;
                    return drew && more && next_in_chain(st);
                };
                auto reduce = [&](const RawTile &tile, int k, RowShared &cur) __attribute__((always_inline)) {
                    if (k >= nt) return;   // (uniform)
                    const int left = tokens_left<T>(V, k, lane);
                    float m, zall;
                    // (one copy of the exact sums for both: 24 steps of 256 rows at V = 32k took 78.4 us with the checks inside and
                    // a copy for each, 75.8 like this)
                    if ((k + 1) * G::TILE > V) list_stats<T, true>(tile, left, tp, m, zall);
                    else list_stats<T, false>(tile, left, tp, m, zall);
                    if (!settled(zall)) exact_stats<T, true>(tile, left, tp, m, zall);
                    if (lane == 0) {
                        cur.tile_m[k] = m;
                        cur.tile_zall[k] = zall;
                    }
                };
                // Two tiles take turns as in stream_tiles, over the steps' ends: behind a row's last two tiles come the next row's
                // first two, asked for while these are reduced.  (No next row: the same loads of no tile.)
                const Share share = share_of(nt, wave_s - 1, ntw);
                const int n = share.n;
                auto tile = [&](int i) { return i < n ? share.at(i) : NO_TILE; };
                RawTile X, Y;
                load_tile<T>(row_of(row, V), tile(0), lane, X);
                load_tile<T>(row_of(row, V), tile(1), lane, Y);
                bool more;
                do {
                    more = row_goes_on();
                    const Row cur = row_of(row, V), next = row_of(more ? row + step_stride : row, more ? V : 0);
                    int i = 0;
                    for (; i + 2 < n; i += 2) {
                        reduce(X, tile(i), shs[s & 1]);
                        load_tile<T>(cur, tile(i + 2), lane, X);
                        reduce(Y, tile(i + 1), shs[s & 1]);
                        load_tile<T>(cur, tile(i + 3), lane, Y);
                    }
                    reduce(X, tile(i), shs[s & 1]);
                    load_tile<T>(next, tile(0), lane, X);
                    reduce(Y, tile(i + 1), shs[s & 1]);
                    load_tile<T>(next, tile(1), lane, Y);
                } while (step_over(more));
            }
            if (finished) break;
            // a prefix of another kind: its step starts below from the row's first tile as the other steps know it
            if (wave < nt) load_tile<T>(row_of(row, V), share.first(), lane, first);
            if (wave_s != 0) u = uniforms[(size_t)s * (size_t)B + b];
            s -= 1;
            continue;
        }
        if (LOOP_REG && mode == VALID_LIST && nchild < WAVE) {
            // ---- A fast step: the children are a short list in wavefront 0's registers.  Wavefront 0 draws the
            // token and works out the next cursor (with its look-ahead) while the tiles are on their way, and hands
            // both to the workgroup through LDS; the step's one barrier says that the tiles' statistics and the
            // hand-over are there.  After it the other wavefronts go straight on to the next step while wavefront 0
            // adds up the row's totals: statistics and hand-over alternate between two buffers, and a buffer is not
            // written again before everybody has passed the barrier after the one it was read behind.
            RowShared &cur = shs[s & 1];
            const bool known = nchild == 1 && st.flags == 1u;   // the cursor knows its only child
            uint32_t e_tok = 0u, e_child = 0u, a_tok = 0u, a_child = 0u, a_next = 0u;
            float gx = -INFINITY;
            if (wave == 0) {
                if (known) {
                    e_tok = lane == 0 ? st.tok0 : 0u;
                    e_child = lane == 0 ? st.child0 : st.child1;
                } else if (lane <= nchild) {
                    const NodeEnt e = ix.ent[cb + (uint32_t)lane];
                    e_tok = e.tok;
                    e_child = e.child;
                }
                if (lane < nchild) {
                    const uint32_t v = e_tok & PPV_NODE_TOKEN;
                    if (sizeof(T) == 4) gx = __uint_as_float(((const uint32_t *)row)[v]);
                    else gx = __uint_as_float(((uint32_t)((const uint16_t *)row)[v]) << 16);
                    const uint32_t a0 = e_child < ix.n_nodes ? e_child : ix.n_nodes;
                    const uint32_t a1 = a0 < ix.n_nodes ? a0 + 1u : ix.n_nodes;
                    const NodeEnt g0 = ix.ent[a0];
                    a_tok = g0.tok;
                    a_child = g0.child;
                    a_next = ix.ent[a1].child;
                }
            }
            ListPick pk;
            pk.id = -1;
            pk.pos = -1;
            pk.Mv = -INFINITY;
            pk.zvl = 0.0;
            if (wave == 0) {
                pk = reg_list_pick(gx, e_tok, nchild, u, lane, tp);
                const bool drew = pk.id >= 0 && t < stride;
                RowState nx = st;
                nx.flags = 0u;
                uint32_t tokw = 0u;
                if (drew) {
                    nx.node = cb + (uint32_t)pk.pos;
                    tokw = lane_value(e_tok, pk.pos);
                    nx.cb = lane_value(e_child, pk.pos);
                    nx.ce = lane_value(e_child, pk.pos + 1);
                    nx.tok0 = lane_value(a_tok, pk.pos);
                    nx.child0 = lane_value(a_child, pk.pos);
                    nx.child1 = lane_value(a_next, pk.pos);
                    nx.flags = 1u;
                    nx.slot = (tokw & PPV_NODE_HEAVY) ? heavy_slot_of(ix, nx.node) : PPV_NO_SLOT;
                }
                if (lane == 0) {
                    hand[s & 1].done = (!drew || (tokw & PPV_NODE_TERMINAL)) ? 1 : 0;
                    hand[s & 1].drew = drew ? 1 : 0;
                    hand[s & 1].nx = nx;
                    if (drew) prefixes[(size_t)b * (size_t)stride + t] = pk.id;
                    if (ids) ids[(size_t)s * (size_t)B + b] = drew ? pk.id : -1;
                    if (!drew) lx = -INFINITY;   // the row stops outside S
                    if (logZ_valid && pk.Mv == -INFINITY) logZ_valid[(size_t)s * (size_t)B + b] = -INFINITY;
                }
            }
            struct {
                __device__ void operator()() const {}
            } nothing;
            stream_tiles<T, false, RowShared>(row_of(row, V), V, first, nullptr, cur, lane, share, tp, nothing, false, sp);
            __syncthreads();
            done = hand[s & 1].done != 0;
            const bool drew = hand[s & 1].drew != 0;
            if (drew) {
                t += 1;
                st = hand[s & 1].nx;
            }
            if (wave == 0 && pk.Mv != -INFINITY) {
                float M, za;
                double zv;
                combine_tiles<T>(cur, row, V, nt, lane, tp, false, M, za, zv);
                const float lzv = fmaf(pk.Mv - M, tp.inv, LN2F * (fast_log2((float)pk.zvl) - fast_log2(za)));
                if (lane == 0) {
                    if (logZ_valid) logZ_valid[(size_t)s * (size_t)B + b] = lzv;
                    if (drew) lx += lzv;
                }
            }
            if (done || s + 1 == n_steps) break;
            row += step_stride;
            if (wave < nt) load_tile<T>(row_of(row, V), share.first(), lane, first);
            u = uniforms[(size_t)(s + 1) * (size_t)B + b];
            continue;
        }
        if (LOOP_REG) __syncthreads();   // (wavefront 0 may still be reading the statistics of a fast step before this one)
        const uint32_t *image = ix.heavy_bits + (size_t)(slot != PPV_NO_SLOT ? slot : 0) * (size_t)ix.n_words;
        int member_child = 0;
        if (mode == VALID_LIST) {
            // children are sorted by token: the list is ready as it is.  One entry more than the
            // children is taken along: it closes the last child's own children range.
            if (LOOP || only == PPV_NO_SLOT) {
                for (int i = tid; i <= nchild; i += nw * WAVE) {
                    const NodeEnt e = ix.ent[cb + i];
                    sh.list_tok[i] = e.tok;
                    sh.list_child[i] = e.child;
                    if (LOOP && !REG && i < nchild && (e.tok & PPV_NODE_TERMINAL)) member_child = 1;
                }
            }
            if (LOOP && !REG) member_child = __syncthreads_or(member_child);
            else if (LOOP || only == PPV_NO_SLOT) __syncthreads();
        }
        // (REG: a third tile in registers here costs more than it saves, in chains, which are spilled for it, and where every step
        // is of this kind too.  us with / without: 800 rows at V = 130k bf16 432 / 398; sets of 2 to 6 tokens, 1,000 rows at V = 32k
        // 66.6 / 60.4, 600 at V = 128k 152 / 142; codes, 256 rows at V = 8,192 bf16 22.0 / 20.0, 512 fp32 26.1 / 25.6)
        const bool more = LOOP && !REG && s + 1 < n_steps && t + 1 < stride && mode != VALID_NONE && !member_child;
        RawTile next_first;
        const T *next_row = more ? row + step_stride : nullptr;
        float next_u = 0.f;
        if (more) next_u = uniforms[(size_t)(s + 1) * (size_t)B + b];
        RowOut r = row_sample<T, RowShared, LOOP, SPLIT>(row, V, first, mode, mode == VALID_LIST ? nchild : 0, image, u, sh,
                                                  tid, nw, tp, sp, next_row, &next_first);
        if (r.mine && tid == 0) {
            const bool room = t < stride || !advance;
            int32_t id = -1;
            done = true;  // no valid token or no room: the row cannot continue
            RowState nx = st;
            nx.flags = 0u;   // (the look-ahead belongs to the node it was made for)
            if (r.id >= 0 && room) {
                id = r.id;
                uint32_t tokw;
                if (mode == VALID_LIST) {
                    nx.node = cb + (uint32_t)r.pos;
                    tokw = sh.list_tok[r.pos];
                    nx.cb = sh.list_child[r.pos];
                    nx.ce = sh.list_child[r.pos + 1];
                } else {  // child index = children before the token's word + set bits below it in the word
                    const uint32_t wv = image[id >> 5];
                    nx.node = cb + ix.heavy_rank[(size_t)slot * (size_t)ix.n_words + (id >> 5)] +
                              (uint32_t)__popc(wv & ((1u << (id & 31)) - 1u));
                    if (nx.node >= ix.n_nodes) nx.node = ix.n_nodes - 1u;   // (only a cursor that paired a slot with another node's children)
                    const NodeEnt e0 = ix.ent[nx.node], e1 = ix.ent[nx.node + 1];
                    tokw = e0.tok;
                    nx.cb = e0.child;
                    nx.ce = e1.child;
                }
                nx.slot = (tokw & PPV_NODE_HEAVY) ? heavy_slot_of(ix, nx.node) : PPV_NO_SLOT;
                done = (tokw & PPV_NODE_TERMINAL) != 0u;   // the extended row is itself a member
                if (advance) prefixes[(size_t)b * (size_t)stride + t] = id;
                lx += r.logZ_valid;
            } else {
                lx = -INFINITY;   // the row stops outside S: its importance score is multiplied by a valid mass of 0
            }
            if (ids) ids[(size_t)s * (size_t)B + b] = id;
            if (logZ_valid) logZ_valid[(size_t)s * (size_t)B + b] = r.logZ_valid;
            if (LOOP) {
                sh.bc_i[2] = done ? 1 : 0;
                sh.bc_i[3] = id >= 0 ? 1 : 0;
                sh.bc_i[4] = (int)nx.node;
                sh.bc_i[5] = (int)nx.cb;
                sh.bc_i[6] = (int)nx.ce;
                sh.bc_i[7] = (int)nx.slot;
            } else if (advance) {
                if (id >= 0) {
                    lens[b] = t + 1;
                    if (state) state[b] = nx;
                } else if (fresh) {
                    lens[b] = 0;
                    if (state) state[b] = st;
                }
                if (logx) logx[b] = logx_in + lx;   // (-inf for a row that drew nothing)
                if (done) active[b] = 0;
                else if (fresh) active[b] = 1;
            }
        }
        if (!LOOP) return;
        __syncthreads();
        done = sh.bc_i[2] != 0;
        if (sh.bc_i[3]) {
            t += 1;
            st.node = (uint32_t)sh.bc_i[4];
            st.cb = (uint32_t)sh.bc_i[5];
            st.ce = (uint32_t)sh.bc_i[6];
            st.slot = (uint32_t)sh.bc_i[7];
            st.flags = 0u;   // the loop kernel does not look ahead
        }
        __syncthreads();   // everyone has the new cursor before LDS is reused
        if (done || s + 1 == n_steps) break;
        row += step_stride;
        if (more) {
            first = next_first;
            u = next_u;
        } else {
            if (wave < nt) load_tile<T>(row_of(row, V), share.first(), lane, first);
            u = uniforms[(size_t)(s + 1) * (size_t)B + b];
        }
    }
    if (LOOP && tid == 0) {
        lens[b] = t;
        if (state) state[b] = st;
        if (logx) logx[b] = lx;
        if (done) active[b] = 0;
    }
}

// T > 0 and finite, or the call is refused; the constants the kernels take (see Temper)
bool temper_for(float temperature, Temper *tp) {
    if (!(temperature > 0.f) || !std::isfinite(temperature)) return false;
    tp->c = (float)(1.44269504088896340736 / (double)temperature);   // log2(e) / T
    tp->inv = (float)(1.0 / (double)temperature);
    tp->guard = REF_GUARD * temperature;
    return std::isfinite(tp->c) && tp->c > 0.f;
}

ppv_status check_logits_args(const void *logits, ppv_dtype dt, int64_t row_stride, int32_t V) {
    if (!logits || V <= 0 || row_stride < V) return PPV_EINVAL;
    if (dt != PPV_F32 && dt != PPV_BF16) return PPV_EINVAL;
    const int64_t per16 = (dt == PPV_F32) ? 4 : 8;
    if (row_stride % per16 != 0 || ((uintptr_t)logits & 15u) != 0) return PPV_EINVAL;
    if (V > PPV_MAX_VOCAB) return PPV_ERANGE;
    return PPV_OK;
}

// Wavefronts per row: a power of two, at most one per tile and at most MAX_WAVES.  A small batch is
// bound by latency and wants every row spread over many wavefronts so that the whole row is in
// flight at once; a large batch is bound by throughput and wants several rows per compute unit, so
// that one row's reduction and sampling phase overlaps another row's loads.  The steps below are
// measured, on the N=1M, V=32k decode loop (TB/s of logits over the whole loop): B=256: 1.05 with
// 16 wavefronts per row, 1.08 with 8, 0.93 with 4; B=512: 1.31 / 1.64 / 1.57; B=1024: 2.28 with 8,
// 2.50 with 4, 2.37 with 2; B=4096: 2.1 with 16, 3.4 with 8, 4.3 with 4, 4.1 with 2; and at
// V=256k: B=256: 3.8 with 16, 1.3 with 2; B=1024: 5.05 with 4, 5.09 with 8, 4.4 with 16.
// `parts`: workgroups per row (see parts_for); the figures then hold for one workgroup's share of the row and for
// the number of workgroups in the launch.
// `cursor_step`: the per-step decode kernel with a cursor, which no longer waits for index entries behind the tiles
// it has asked for: one tile per wavefront, the whole row in flight at once, also at 256 rows (C3, us per launch
// with 8 / 16 wavefronts: 7.9 / 7.6 before the list moved into registers; tiles reduced 3.4 / 2.8 us after the
// cursor is in).
int waves_for(int V, ppv_dtype dt, int B, int parts = 1, bool cursor_step = false) {
    const int tile = (dt == PPV_F32) ? TileGeom<float>::TILE : TileGeom<uint16_t>::TILE;
    const int nt = ((V + tile - 1) / tile + parts - 1) / parts;
    B *= parts;
    int cap = B <= 128 ? 16 : (B <= 512 ? 8 : 4);
    if (cursor_step && B <= 256) cap = 16;
    // long rows in a small batch: one row per compute unit, all of it in flight (constrained_sample, B = 256, us per
    // call with 8 / 16 wavefronts: 32 tiles: 13.2 / 12.0 (fp32 V = 32k), 15.2 / 14.2 (bf16 V = 64k); 63 tiles: 23.6 / 20.6)
    if (nt >= 32 && B <= 256) cap = 16;
    // long rows in a large batch: the loads in flight are the same with fewer rows at a time, and each of these is over
    // sooner.  us with 4 / 8 / 16 wavefronts, decoding loops: V = 200k bf16, B = 1,000: 326 / 289 / 319; V = 128k bf16,
    // B = 1,024: 298 / 287 / 321, B = 1,800: 358 / 341 / 378; V = 50k fp32, B = 1,024: 363 / 352 / 371; V = 32k bf16 (16
    // tiles), B = 1,024: 211 / 219 / 279.  Mask + sample, B = 1,024: V = 200k 92.3 / 89.1 / 88.9, V = 50k fp32
    // 40.7 / 39.5 / 41.7; ppv_sample_next: V = 128k 49.1 / 48.8 / 56.6, V = 50k fp32 36.7 / 37.0 / 40.6.  Below that four are
    // better or as good (constrained_sample / ppv_sample_next, B = 1,024, 4 against 8, 24, 32, 40 and 48 tiles of bf16: 19.2
    // 24.8 29.3 34.6 against 21.4 25.7 30.1 35.0 / 18.1 23.4 27.7 33.0 against 19.4 23.8 28.5 33.0; fp32, 32 and 40 tiles: 22.0
    // 26.5 against 24.8 28.8 / 22.3 26.8 against 23.0 27.3).
    if (nt >= 48 && B > 512) cap = 8;
    // (a part of a row: us per call with 4 / 8 / 16 wavefronts, constrained_sample, list rows, 32 in 4 parts, V = 50k fp32 7.6 / 6.7 /
    // 7.6, V = 128k bf16 9.7 / 7.7 / 8.2, V = 64k 6.7 / 6.5 / 6.4; long parts, 128 rows in 2, V = 256k bf16, 8 / 16: 17.6 / 16.8, 16 rows
    // in 4 11.1 / 9.8, but a step with a cursor 15.4 / 15.8 and 8.8 / 8.9)
    if (parts > 1) cap = nt >= 32 && !cursor_step ? 16 : 8;
    if (const int v = ppv_tuning(PPV_TUNE_WAVES_PER_ROW)) cap = v;   // tuning aid (0: the table above)
    int nw = 1;
    while (nw < nt && nw * 2 <= cap) nw <<= 1;
    return nw;
}

// Workgroups per row.  A batch of fewer rows than the chip has compute units leaves most of it idle with one
// workgroup per row, and a long row alone on a compute unit is bound by that unit's arithmetic.  Such a row is spread over
// 2 .. 16 workgroups: a power of two, six tiles or more each, at most one workgroup per compute unit -- where that takes
// enough of the row off each to pay for the hand-over (see meet): bytes of the row x (1 - 1 / parts), and more of fp32, which
// is half the arithmetic.  us per call unsplit / in 2, 4, 8 parts, list rows of constrained_sample: 32 rows, V = 24k
// fp32 6.4 / 7.0 6.3 6.6, V = 36k fp32 7.0 / 7.1 6.4 6.8, V = 48k bf16 7.1 / 7.0 6.5 7.0, V = 64k bf16 7.9 / 7.0 6.5 7.0, V = 50k
// fp32 8.5 / 7.6 6.7 7.1, V = 128k bf16 10.3 / 9.0 7.7 8.0; 128 rows in 2 parts, V = 48k bf16 7.4 / 7.5, V = 64k 8.2 / 7.7, V = 128k 11.0 /
// 10.7, V = 36k fp32 7.4 / 8.2, V = 50k 9.2 / 9.0.  Rows under an image gain up to twice as much (V = 128k: 32 rows 15.8 / 10.4 in
// 4, 128 rows 16.6 / 14.6 in 2).  A decode step with a cursor has more to lose, unsplit it draws the token while its tiles travel, and
// one without a cursor locates the prefix in each part: 32 rows, V = 64k bf16 7.0 / 6.9 in 4, V = 96k 8.4 / 7.3 in 8, V = 36k fp32
// 6.6 / 7.1 in 4, V = 50k 7.9 / 7.4 in 4; 96 rows in 2, V = 96k bf16 8.8 / 8.9, V = 128k 10.4 / 9.4;
// 128 rows in 2, every compute unit busy, V = 128k 10.5 / 10.4 (ppv_sample_next 11.8 / 12.2), V = 100k fp32 12.6 / 13.1 (14.0 / 14.8),
// V = 256k bf16 16.8 / 15.9; as rows retire a loop's later steps gain (27 steps of 111 rows at V = 98k fp32 335 / 325).
// The first step of a loop, every row under the root's image: 32 rows, V = 48k bf16 10.0 / 9.5 in 4, 128 rows in 2, V = 64k 12.3 / 11.8,
// V = 50k fp32 12.0 / 12.1.  (With three trips to shared memory in the hand-over the line was 160 KB, 180 with a cursor.)
// Above 96 rows a split leaves no compute unit idle, and pays for very long rows alone: constrained_sample behind ppv_next_token_mask, 128
// rows at V = 96k bf16 18.3 / 18.9 in 2, V = 128k 20.6 / 21.0 (behind ppv_topm_mask 30.6 / 31.5), V = 100k fp32 21.2 / 23.2, V = 256k bf16, list
// rows, 17.3 / 16.7.  (Two workgroups that part again where they find the row to be no image row were slower still: 34.0 for 30.6.)
// PPV_TUNE_ROW_SPLIT forces a number of parts.
// The scratch area the parts meet in comes with the stream or the capture; without one (see ppv_split_scratch) rows are not split.
enum RowCall { SAMPLE, LOCATE, STEP, FIRST_STEP };   // LOCATE: without a cursor
int parts_wanted(int V, ppv_dtype dt, int B, RowCall call) {
    const int tile = (dt == PPV_F32) ? TileGeom<float>::TILE : TileGeom<uint16_t>::TILE;
    const int nt = (V + tile - 1) / tile;
    if (B > PPV_SPLIT_MAX_ROWS) return 1;
    int parts = ppv_tuning(PPV_TUNE_ROW_SPLIT);
    if (parts == 0) {
        parts = 1;
        while (B * parts * 2 <= 256 && parts * 2 <= PPV_SPLIT_MAX_PARTS && nt / (parts * 2) >= 6) parts *= 2;
        const double row_kb = (double)V * (dt == PPV_F32 ? 4.0 : 2.0) / 1024.0;
        double least_kb = call == SAMPLE ? (dt == PPV_F32 ? 104.0 : 60.0) : (dt == PPV_F32 ? 140.0 : (call == FIRST_STEP ? 60.0 : 110.0));
        if (B > 96 && call != FIRST_STEP) least_kb = call != STEP ? 200.0 : (dt == PPV_F32 ? 180.0 : 110.0);
        if (row_kb * (1.0 - 1.0 / parts) < least_kb) parts = 1;
    }
    while (parts > 1 && ((parts & (parts - 1)) != 0 || parts * 2 > nt)) parts--;   // a power of two, two tiles each
    return parts;
}
int parts_for(int V, ppv_dtype dt, int B, hipStream_t hs, SplitScratch **scratch, RowCall call) {
    *scratch = nullptr;
    int parts = parts_wanted(V, dt, B, call);
    if (parts > 1) {
        *scratch = ppv_split_scratch(hs, B);
        if (!*scratch) parts = 1;
    }
    return parts;
}
int shift_of(int parts) {
    int sh = 0;
    while ((1 << sh) < parts) sh++;
    return sh;
}

// A mark for a call that splits rows (see SplitRow); 0 for the others.
std::atomic<uint32_t> g_mark_flags{0};
uint32_t mark_for(int split_shift) {
    static std::atomic<uint32_t> last{0};
    uint32_t mark = 0;
    while (split_shift && !mark) mark = ++last & (LOOK_ONCE - 1u);
    return mark | g_mark_flags.load(std::memory_order_relaxed);
}

template <typename T>
void launch_sample(bool small, dim3 grid, dim3 block, hipStream_t hs, const T *lg, int64_t row_stride,
                   const uint32_t *mask, const float *uniforms, int V, int n_words, int list_max, int32_t *ids,
                   float *logZ_valid, float *logZ_all, Temper tp, int split_shift, SplitScratch *scratch) {
#define PPV_LAUNCH_SAMPLE(SMALL, SPLIT)                                                                                  \
    hipLaunchKernelGGL((sample_kernel<T, SMALL, SPLIT>), grid, block, 0, hs, lg, row_stride, mask, V, n_words, \
                       list_max, split_shift | (int)(block.x / WAVE) << 8, scratch, uniforms, ids, logZ_valid, logZ_all, tp, mark_for(split_shift))
    if (split_shift) PPV_LAUNCH_SAMPLE(false, true);
    else if (small) PPV_LAUNCH_SAMPLE(true, false);
    else PPV_LAUNCH_SAMPLE(false, false);
#undef PPV_LAUNCH_SAMPLE
}

constexpr int REG_MAX_ROWS = 1024;   // batches up to here run the loop kernel with the list in registers (two sets of statistics in LDS: fewer rows per compute unit)
template <typename T>
void launch_decode_kernel(bool loop, dim3 grid, dim3 block, hipStream_t hs, const IndexView &view,
                          int32_t *prefixes, int32_t stride, int32_t *lens, uint8_t *active, RowState *rs, const T *lg,
                          int64_t row_stride, int64_t step_stride, const float *uniforms, int n_steps, int B, int32_t *ids,
                          float *logZ_valid, float *logx, Temper tp, int split_shift, SplitScratch *scratch, int flags) {
    const bool reg = rs && (!loop || B <= REG_MAX_ROWS);
#define PPV_LAUNCH_DECODE(LOOP, SPLIT, REG)                                                                               \
    hipLaunchKernelGGL((decode_kernel<T, LOOP, SPLIT, REG>), grid, block, 0, hs, active, lens, rs, uniforms, logx, lg, flags | (int)(mark_for(split_shift) << 2), \
                       split_shift | (int)(block.x / WAVE) << 8, prefixes, stride, n_steps, B, row_stride, step_stride, ids,  \
                       logZ_valid, scratch, tp, view)
    if (split_shift && !loop && reg) PPV_LAUNCH_DECODE(false, true, true);
    else if (split_shift && !loop) PPV_LAUNCH_DECODE(false, true, false);
    else if (loop && reg) PPV_LAUNCH_DECODE(true, false, true);
    else if (loop) PPV_LAUNCH_DECODE(true, false, false);
    else if (reg) PPV_LAUNCH_DECODE(false, false, true);
    else PPV_LAUNCH_DECODE(false, false, false);
#undef PPV_LAUNCH_DECODE
}

}  // namespace

extern "C" ppv_status ppv_next_token_mask(const ppv_index_t *ix, const int32_t *prefixes, int32_t prefix_stride,
                                          const int32_t *lens, int32_t B, uint32_t *mask, uint32_t *range_lo,
                                          uint32_t *range_hi, uint8_t *member, void *stream) {
    if (!ix || B < 0 || prefix_stride < 0) return PPV_EINVAL;
    if (B == 0) return PPV_OK;  // nothing to do; the (possibly null) buffers are not looked at
    if (!prefixes || !lens || !mask) return PPV_EINVAL;
    if (ix->view.n_words <= MASK_SMALL_WORDS) {
        const int rows_per_wg = MASK_THREADS / WAVE;
        hipLaunchKernelGGL(mask_rows_kernel, dim3((unsigned)((B + rows_per_wg - 1) / rows_per_wg)), dim3(MASK_THREADS), 0,
                           (hipStream_t)stream, prefixes, lens, prefix_stride, B, mask, range_lo, range_hi, member, ix->view);
    } else {
        const size_t lds = ((size_t)ix->view.n_words + 5) * sizeof(uint32_t);
        hipLaunchKernelGGL(mask_kernel, dim3((unsigned)B), dim3(MASK_THREADS), lds, (hipStream_t)stream, prefixes,
                           lens, prefix_stride, mask, range_lo, range_hi, member, ix->view);
    }
    PPV_HIP_TRY(hipGetLastError());
    return PPV_OK;
}

// The scratch area of constrained_sample_noalloc: the same SplitScratch that other calls allocate per stream, here
// a fixed array in device memory (every GPU the library runs on holds its own copy until the process ends).  Host
// code never uses the array's name as an address: its address on the current device is looked up once per device.
static __device__ __align__(256) unsigned char scratch[sizeof(SplitScratch)];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_fixed_mu;
SplitScratch *g_fixed_scratch[MAX_DEVICES];   // per device: the address of `scratch` there

ppv_status fixed_scratch(SplitScratch **out) {
    int dev = -1;
    PPV_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return PPV_ERANGE;
    std::lock_guard<std::mutex> lock(g_fixed_mu);
    if (!g_fixed_scratch[dev]) {
        void *ptr = nullptr;
        PPV_HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return PPV_EDEVICE;
        g_fixed_scratch[dev] = (SplitScratch *)ptr;
    }
    *out = g_fixed_scratch[dev];
    return PPV_OK;
}

ppv_status sample_call(const void *logits, ppv_dtype dt, int64_t row_stride, const uint32_t *mask, const float *uniforms,
                       int32_t B, int32_t V, int32_t *ids, float *logZ_valid, float *logZ_all, float temperature,
                       void *stream, bool no_alloc) {
    Temper tp;
    if (B < 0 || !temper_for(temperature, &tp)) return PPV_EINVAL;
    if (B == 0) return PPV_OK;
    if (!mask || !uniforms || !ids || !logZ_valid) return PPV_EINVAL;
    ppv_status st = check_logits_args(logits, dt, row_stride, V);
    if (st != PPV_OK) return st;
    const int n_words = (V + 31) / 32;
    const int list_max = V / 32 < PPV_LIST_MAX ? V / 32 : PPV_LIST_MAX;
    const int tile = (dt == PPV_F32) ? TileGeom<float>::TILE : TileGeom<uint16_t>::TILE;
    const bool small = (V + tile - 1) / tile <= SMALL_TILES && list_max <= SMALL_LIST;   // then threads <= SMALL_TILES * WAVE
    hipStream_t hs = (hipStream_t)stream;
    SplitScratch *scratch = nullptr;
    int parts = 1;
    if (no_alloc) {   // the fixed array: no allocation, a stated largest batch
        if (B > PPV_NOALLOC_MAX_ROWS) return PPV_ERANGE;
        st = fixed_scratch(&scratch);
        if (st != PPV_OK) return st;
        if (!small && V > tile) parts = parts_wanted(V, dt, B, SAMPLE);
    } else if (!small && V > tile) {
        parts = parts_for(V, dt, B, hs, &scratch, SAMPLE);
    }
    const int threads = waves_for(V, dt, B, parts) * WAVE;
    const dim3 grid((unsigned)B * (unsigned)parts), block(threads);
    if (V <= tile) {   // the whole row is one tile
        const dim3 g1((unsigned)((B + ONE_TILE_ROWS - 1) / ONE_TILE_ROWS)), b1(ONE_TILE_ROWS * WAVE);
        if (dt == PPV_F32)
            hipLaunchKernelGGL(sample_one_tile_kernel<float>, g1, b1, 0, hs, (const float *)logits, row_stride, mask, uniforms,
                               B, V, n_words, ids, logZ_valid, logZ_all, tp);
        else
            hipLaunchKernelGGL(sample_one_tile_kernel<uint16_t>, g1, b1, 0, hs, (const uint16_t *)logits, row_stride, mask,
                               uniforms, B, V, n_words, ids, logZ_valid, logZ_all, tp);
        PPV_HIP_TRY(hipGetLastError());
        return PPV_OK;
    }
    if (dt == PPV_F32)
        launch_sample<float>(small, grid, block, hs, (const float *)logits, row_stride, mask, uniforms, V, n_words,
                             list_max, ids, logZ_valid, logZ_all, tp, shift_of(parts), scratch);
    else
        launch_sample<uint16_t>(small, grid, block, hs, (const uint16_t *)logits, row_stride, mask, uniforms, V,
                                n_words, list_max, ids, logZ_valid, logZ_all, tp, shift_of(parts), scratch);
    PPV_HIP_TRY(hipGetLastError());
    return PPV_OK;
}
}  // namespace

ppv_status ppv_split_area_for_tests(void *stream, int32_t fixed, int32_t look_again, void **area, int64_t *bytes, int64_t *words_at) {
    SplitScratch *p = fixed ? nullptr : ppv_split_scratch((hipStream_t)stream, PPV_SPLIT_MAX_ROWS);
    if (fixed) {
        const ppv_status st = fixed_scratch(&p);
        if (st != PPV_OK) return st;
    }
    if (!p) return PPV_ENOMEM;
    g_mark_flags = look_again ? 0u : LOOK_ONCE;
    *area = p;
    *bytes = (int64_t)sizeof(SplitScratch);
    *words_at = (int64_t)offsetof(SplitScratch, row);
    return PPV_OK;
}

extern "C" ppv_status constrained_sample(const void *logits, ppv_dtype dt, int64_t row_stride, const uint32_t *mask,
                                         const float *uniforms, int32_t B, int32_t V, int32_t *ids,
                                         float *logZ_valid, float *logZ_all, float temperature, void *stream) {
    return sample_call(logits, dt, row_stride, mask, uniforms, B, V, ids, logZ_valid, logZ_all, temperature, stream, false);
}

extern "C" ppv_status constrained_sample_noalloc(const void *logits, ppv_dtype dt, int64_t row_stride,
                                                 const uint32_t *mask, const float *uniforms, int32_t B, int32_t V,
                                                 int32_t *ids, float *logZ_valid, float *logZ_all, float temperature,
                                                 void *stream) {
    return sample_call(logits, dt, row_stride, mask, uniforms, B, V, ids, logZ_valid, logZ_all, temperature, stream, true);
}

extern "C" ppv_status ppv_decode_begin(const ppv_index_t *ix, const int32_t *prefixes, int32_t prefix_stride,
                                       const int32_t *lens, int32_t B, uint32_t *state, uint8_t *active, float *logx,
                                       void *stream) {
    if (!ix || B < 0 || prefix_stride < 0) return PPV_EINVAL;
    if (B == 0) return PPV_OK;
    if (!prefixes || !lens || !state || !active) return PPV_EINVAL;
    const int rows_per_wg = MASK_THREADS / WAVE;
    hipLaunchKernelGGL(decode_begin_kernel, dim3((unsigned)((B + rows_per_wg - 1) / rows_per_wg)), dim3(MASK_THREADS), 0,
                       (hipStream_t)stream, prefixes, lens, prefix_stride, B, (RowState *)state, active, logx,
                       ix->view);
    PPV_HIP_TRY(hipGetLastError());
    return PPV_OK;
}

extern "C" ppv_status ppv_decode_begin_empty(const ppv_index_t *ix, int32_t B, int32_t *lens, uint32_t *state,
                                             uint8_t *active, float *logx, void *stream) {
    if (!ix || B < 0) return PPV_EINVAL;
    if (B == 0) return PPV_OK;
    if (!lens || !state || !active) return PPV_EINVAL;
    hipLaunchKernelGGL(decode_begin_empty_kernel, dim3((unsigned)((B + MASK_THREADS - 1) / MASK_THREADS)), dim3(MASK_THREADS),
                       0, (hipStream_t)stream, B, lens, (RowState *)state, active, logx, ix->view);
    PPV_HIP_TRY(hipGetLastError());
    return PPV_OK;
}

namespace {
ppv_status launch_decode(const ppv_index_t *ix, int32_t *prefixes, int32_t prefix_stride, int32_t *lens, uint8_t *active,
                         uint32_t *state, const void *logits, ppv_dtype dt, int64_t row_stride, int64_t step_stride,
                         const float *uniforms, int32_t n_steps, int32_t B, int32_t *ids, float *logZ_valid, float *logx,
                         float temperature, void *stream, bool loop, bool advance = true, bool fresh = false) {
    Temper tp;
    if (!ix || B < 0 || prefix_stride < 0 || n_steps < 0 || !temper_for(temperature, &tp)) return PPV_EINVAL;
    if (B == 0 || n_steps == 0) return PPV_OK;
    if (!prefixes || !lens || (advance && !active) || !uniforms) return PPV_EINVAL;
    ppv_status st = check_logits_args(logits, dt, row_stride, ix->view.vocab);
    if (st != PPV_OK) return st;
    if (loop && n_steps > 1) {
        const int64_t per16 = (dt == PPV_F32) ? 4 : 8;
        if (step_stride % per16 != 0 || step_stride < 0) return PPV_EINVAL;
    }
    hipStream_t hs = (hipStream_t)stream;
    SplitScratch *scratch = nullptr;
    const int parts = loop ? 1 : parts_for(ix->view.vocab, dt, B, hs, &scratch, !state ? LOCATE : (fresh ? FIRST_STEP : STEP));
    int nw = waves_for(ix->view.vocab, dt, B, parts, !loop && state != nullptr);
    const int tile = (dt == PPV_F32) ? TileGeom<float>::TILE : TileGeom<uint16_t>::TILE;
    const int nt = (ix->view.vocab + tile - 1) / tile;
    if (loop) {
        const bool reg = state && B <= REG_MAX_ROWS;
        const int most = reg ? MAX_WAVES : LOOP_WAVES;
        if (nw > most) nw = most;
        // A workgroup of the loop kernel stays with its row for every step, and a row that has no place on the chip waits for
        // another to end.  128 registers are sixteen wavefronts to a compute unit: a row's own up to 256 rows (long rows: up to 320
        // or always, see below), half of them to 512 and for rows of 48 tiles or more, a quarter to 1,024.  us per loop with 16 / 8 / 4: 200 rows, V = 50k fp32
        // 90 / 89 / 131, V = 40k bf16 54 / 59 / 80; 512 rows, V = 16k fp32 80 / 66 / 69, V = 50k bf16 128 / 119 / 132; 1,000 rows,
        // V = 50k fp32 354 / 345 / 375.  (With 168 registers and up to ten wavefronts, one row to a compute unit: 384 rows,
        // V = 50k fp32 142, now 123; 512 rows, V = 32k bf16 98 and 77; 1,000 rows 176 and 134.)  In larger batches two
        // wavefronts, and the list in LDS: what hides a row's dependent phases is other rows on the same compute unit (C3
        // replicas, M prefix-steps/s with 1 / 2 / 4 / 8 wavefronts per row:
        // 4,096 rows: 72 / 81 / 66 / 39; 16,384 rows: 95 / 98 / 77 / 42 -- 6.3 TB/s; the per-step kernel is best with four).
        if (ppv_tuning(PPV_TUNE_WAVES_PER_ROW) == 0) {
            if (reg) {
                // (a few rows above 256, or very long ones: a place to itself is worth more than a place at once.  us per loop with
                // 16 / 8: V = 240k bf16, 264 rows 266 / 308, 512 rows 355 / 370, 600 rows 412 / 425; V = 130k bf16, 264 rows 127 / 158; V = 76k
                // fp32, 320 rows 149 / 168, 384 rows 180 / 174; V = 50k fp32, 264 rows 86 / 102, 512 rows 149 / 141)
                const bool alone = B <= 256 || (B <= 320 && nt >= 48) || nt >= 96;
                nw = alone ? 16 : (B <= 512 || nt >= 48 ? 8 : 4);
                if (nw > nt + 1) nw = nt + 1;   // one draws (see decode_kernel)
                // (16 to 18 tiles on fifteen wavefronts: a few have two tiles and the rest wait for them.  200 rows, V = 16k fp32
                // 42.7 us, and 38.5 with nine wavefronts; with 20 tiles eleven are slower than sixteen, 54.3 against 51.8)
                if (B <= 256 && nt > 15 && nt <= 18) nw = (nt + 1) / 2 + 1;
            } else if (B > REG_MAX_ROWS && nw > 2) {
                nw = 2;
            } else if (B > 512 && nw > 4) {
                nw = 4;
            }
        }
    }
    const dim3 grid((unsigned)B * (unsigned)parts), block(nw * WAVE);
    RowState *rs = (RowState *)state;
    if (!loop) n_steps = 1;
    if (dt == PPV_F32)
        launch_decode_kernel<float>(loop, grid, block, hs, ix->view, prefixes, prefix_stride, lens, active, rs,
                                    (const float *)logits, row_stride, step_stride, uniforms, n_steps, B, ids, logZ_valid,
                                    logx, tp, shift_of(parts), scratch, (advance ? 1 : 0) | (fresh ? 2 : 0));
    else
        launch_decode_kernel<uint16_t>(loop, grid, block, hs, ix->view, prefixes, prefix_stride, lens, active, rs,
                                       (const uint16_t *)logits, row_stride, step_stride, uniforms, n_steps, B, ids,
                                       logZ_valid, logx, tp, shift_of(parts), scratch, (advance ? 1 : 0) | (fresh ? 2 : 0));
    PPV_HIP_TRY(hipGetLastError());
    return PPV_OK;
}
}  // namespace

extern "C" ppv_status ppv_decode_step(const ppv_index_t *ix, int32_t *prefixes, int32_t prefix_stride, int32_t *lens,
                                      uint8_t *active, uint32_t *state, const void *logits, ppv_dtype dt,
                                      int64_t row_stride, const float *uniforms, int32_t B, int32_t *ids,
                                      float *logZ_valid, float *logx, float temperature, void *stream) {
    return launch_decode(ix, prefixes, prefix_stride, lens, active, state, logits, dt, row_stride, 0, uniforms, 1, B, ids,
                         logZ_valid, logx, temperature, stream, false);
}

extern "C" ppv_status ppv_decode_first_step(const ppv_index_t *ix, int32_t *prefixes, int32_t prefix_stride, int32_t *lens,
                                            uint8_t *active, uint32_t *state, const void *logits, ppv_dtype dt,
                                            int64_t row_stride, const float *uniforms, int32_t B, int32_t *ids,
                                            float *logZ_valid, float *logx, float temperature, void *stream) {
    if (!state) return PPV_EINVAL;
    return launch_decode(ix, prefixes, prefix_stride, lens, active, state, logits, dt, row_stride, 0, uniforms, 1, B, ids,
                         logZ_valid, logx, temperature, stream, false, true, true);
}

extern "C" ppv_status ppv_decode_loop(const ppv_index_t *ix, int32_t *prefixes, int32_t prefix_stride, int32_t *lens,
                                      uint8_t *active, uint32_t *state, const void *logits, ppv_dtype dt,
                                      int64_t row_stride, int64_t step_stride, const float *uniforms, int32_t n_steps,
                                      int32_t B, int32_t *ids, float *logZ_valid, float *logx, float temperature,
                                      void *stream) {
    return launch_decode(ix, prefixes, prefix_stride, lens, active, state, logits, dt, row_stride, step_stride, uniforms,
                         n_steps, B, ids, logZ_valid, logx, temperature, stream, true);
}

extern "C" ppv_status ppv_sample_next(const ppv_index_t *ix, const int32_t *prefixes, int32_t prefix_stride,
                                      const int32_t *lens, int32_t B, const void *logits, ppv_dtype dt,
                                      int64_t row_stride, const float *uniforms, int32_t *ids, float *logZ_valid,
                                      float temperature, void *stream) {
    Temper tp;
    if (!ix || B < 0 || prefix_stride < 0 || !temper_for(temperature, &tp)) return PPV_EINVAL;
    if (B == 0) return PPV_OK;
    if (!prefixes || !lens || !uniforms || !ids) return PPV_EINVAL;
    const int V = ix->view.vocab;
    const ppv_status st = check_logits_args(logits, dt, row_stride, V);
    if (st != PPV_OK) return st;
    const int tile = (dt == PPV_F32) ? TileGeom<float>::TILE : TileGeom<uint16_t>::TILE;
    if (V <= tile && ix->view.n_words <= MASK_SMALL_WORDS) {   // the whole row is one tile: one wavefront per row
        const dim3 g1((unsigned)((B + ONE_TILE_ROWS - 1) / ONE_TILE_ROWS)), b1(ONE_TILE_ROWS * WAVE);
        if (dt == PPV_F32)
            hipLaunchKernelGGL(sample_next_one_tile_kernel<float>, g1, b1, 0, (hipStream_t)stream, prefixes, lens,
                               uniforms, (const float *)logits, row_stride, prefix_stride, B, ids, logZ_valid,
                               (uint8_t *)nullptr, tp, ix->view);
        else
            hipLaunchKernelGGL(sample_next_one_tile_kernel<uint16_t>, g1, b1, 0, (hipStream_t)stream, prefixes, lens,
                               uniforms, (const uint16_t *)logits, row_stride, prefix_stride, B, ids, logZ_valid,
                               (uint8_t *)nullptr, tp, ix->view);
        PPV_HIP_TRY(hipGetLastError());
        return PPV_OK;
    }
    // longer rows: the fused decode step without a cursor, told to change nothing of the caller's rows
    return launch_decode(ix, const_cast<int32_t *>(prefixes), prefix_stride, const_cast<int32_t *>(lens), nullptr, nullptr,
                         logits, dt, row_stride, 0, uniforms, 1, B, ids, logZ_valid, nullptr, temperature, stream, false,
                         false);
}
