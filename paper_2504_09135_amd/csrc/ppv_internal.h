// Internal definitions shared by the sources of libppv_hip.so (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ppv.h"

// Device view of the index.  The distinct non-empty prefixes of members ("nodes") are stored in
// breadth-first order: all prefixes of length 1 in sorted order, then all of length 2, ...
// Node 0 is the empty prefix.  Because each depth is sorted, the children of consecutive nodes
// are consecutive, so one offsets array describes all of them: the children of node g are the
// nodes ent[g].child .. ent[g+1].child, in increasing token order.  Token and child offset sit
// side by side, so the one load that searches (or lists) a node's children also brings each
// child's own children range.
//
// Nodes with more than `heavy_min` children ("heavy": the root and a few shallow prefixes) also
// carry their valid set as a ready-made V-bit image plus, per 32-bit word of it, the number of
// children before that word, so that a copy replaces the scatter and the child carrying a given
// token is found with two loads.
constexpr uint32_t PPV_NODE_TERMINAL = 0x80000000u;  // flag in NodeEnt::tok: the prefix itself is in S
constexpr uint32_t PPV_NODE_HEAVY = 0x40000000u;     // flag in NodeEnt::tok: the node has an image
constexpr uint32_t PPV_NODE_TOKEN = 0x3FFFFFFFu;
constexpr uint32_t PPV_NO_SLOT = 0xFFFFFFFFu;
constexpr int PPV_LIST_MAX = 1024;  // a valid set of at most this many tokens is handled as a list

struct NodeEnt {
    uint32_t tok;    // last token of the prefix | flags
    uint32_t child;  // first child; the children end where the next entry's children begin
};

struct alignas(16) LookupEntry {
    uint64_t key;      // fingerprint << 32 | node (or the member's rank, if there is only one under the node); 0: empty
    uint32_t at;       // where the first member under the node starts in x_tok
    uint32_t extent;   // the prefix's length; << 8: that member's length (at most a wavefront's), if it is the only one
};
constexpr uint32_t LOOKUP_BUCKET = 4;   // entries that are looked at together: 64 bytes

struct IndexView {
    const NodeEnt *ent;          // [n_nodes+1] (the last entry is a sentinel that closes the offsets)
    const uint32_t *node_lo;     // [n_nodes]   rank of the first member the prefix is a prefix of
    const uint32_t *node_hi;     // [n_nodes]   one past the rank of the last such member
    const uint32_t *heavy_slot;  // [heavy_limit] slot of a heavy node, PPV_NO_SLOT otherwise
    const uint32_t *heavy_bits;  // [n_heavy, n_words] valid-set images
    const uint32_t *heavy_rank;  // [n_heavy, n_words] children before each word
    // Hashed look-up of prefixes (all lengths of a query are probed at once instead of one level after the other): buckets
    // filled from the front, a full one overflows into the next; lookup_buckets == 0: no table.  A hit is only a hint: it
    // is checked against the tokens of the first member under the prefix it names.  Prefixes of one member only are
    // entered up to the shortest of them (LookupEntry::extent); the longer ones are found by comparing that member's
    // tokens, and their nodes, where they are wanted, by node_at.
    const LookupEntry *lookup;   // [lookup_buckets * LOOKUP_BUCKET]
    const uint32_t *node_at;     // [tokens of S] (with a table) by position in x_tok: the node that ends there, for prefixes of one member
    const int32_t *x_tok;        // sorted S, flat
    uint32_t lookup_buckets;
    uint32_t lookup_fp_mask;     // fingerprint bits in use (all of them; 0 in a test mode that makes every probe a false hit)
    uint32_t heavy_limit;        // nodes >= heavy_limit are not heavy
    uint32_t heavy_min;          // a node is heavy iff it has more than heavy_min children
    uint32_t n_heavy;            // heavy nodes, i.e. rows of heavy_bits / heavy_rank
    uint32_t n_nodes;            // including node 0
    uint32_t n_rows;             // |S| after de-duplication
    int32_t vocab;
    int32_t n_words;             // ceil(vocab / 32)
    int32_t l_max;
};

// A row spread over several workgroups (small batches: fewer rows than compute units).  Every workgroup reduces
// its share of the row's tiles and of the listed tokens and leaves the per-tile / per-slice statistics here; the
// workgroup that arrives last (one device-scope counter per row) takes them all and finishes the row exactly
// as a single workgroup would: the statistics do not depend on who computed them, so results are bit for bit
// those of an unsplit row.  Every word carries the mark of the call that wrote it, so it says by itself whether it has arrived,
// and what another call has left is never taken for it.  (The workgroup that finishes the row puts zeros in their place, for a graph,
// whose replays have one mark.)
constexpr int PPV_MAX_TILES = 256;          // PPV_MAX_VOCAB / 1024 (fp32 tiles are 1024 tokens)
constexpr int PPV_SPLIT_MAX_ROWS = PPV_NOALLOC_MAX_ROWS;   // larger batches fill the chip with one workgroup per row
constexpr int PPV_SPLIT_MAX_PARTS = 16;
typedef uint64_t Marked;                    // a float, and above it the call's mark: never 0, another for every one of 2^29 calls, and
                                            // one for all replays of a captured call
struct MarkedPair {
    Marked first, second;
};
struct SplitRow {
    MarkedPair tile[PPV_MAX_TILES];         // reference, sum over all tokens
    Marked valid[PPV_MAX_TILES];            // sum over valid tokens: rows under an image
    MarkedPair slice[PPV_LIST_MAX / 64];    // largest of 64 listed logits, the sum relative to it
    Marked list_e[PPV_LIST_MAX];
};
struct SplitScratch {
    uint32_t arrivals[PPV_SPLIT_MAX_ROWS];
    SplitRow row[PPV_SPLIT_MAX_ROWS];
};
// The scratch area for `rows` rows (PPV_SPLIT_MAX_ROWS at most) of a call on this stream of the current device, or of the capture
// that the stream is in; nullptr when there is none to be had: the rows are then not split.
SplitScratch *ppv_split_scratch(hipStream_t stream, int rows);
// The area of eager calls on a stream, or constrained_sample_noalloc's array: its address, its size and where the rows' words begin,
// for the tests that look at one or disturb it; look_again 0: calls from now on look once at a word.  (Exported, and not declared in
// ppv.h.)
extern "C" ppv_status ppv_split_area_for_tests(void *stream, int32_t fixed, int32_t look_again, void **area, int64_t *bytes, int64_t *words_at);

// Per-row decoding cursor kept between decode steps (PPV_STATE_WORDS x uint32).  The second half looks one level
// ahead: the entry of the node's first child and the child offset of the entry after it.  For a node with exactly
// one child -- nearly every node below the first few levels of a set of long sequences -- that is the whole valid
// set and the child's own children range, so a decode step on such a node needs no load from the index before it
// can ask for the listed token's logit.  `flags` says whether that half is filled in; it is a cache, never required.
struct RowState {
    uint32_t node;   // entry of the row's current prefix; PPV_NO_SLOT: not a prefix of any member
    uint32_t cb, ce; // its children
    uint32_t slot;   // heavy slot or PPV_NO_SLOT
    uint32_t tok0;   // ent[cb].tok   (token | flags of the first child)      -- when flags == 1
    uint32_t child0; // ent[cb].child (where the first child's children begin)
    uint32_t child1; // ent[cb + 1].child (where they end, if the node has one child)
    uint32_t flags;  // 1: tok0 / child0 / child1 are filled in; anything else: they are not
};
static_assert(sizeof(RowState) == PPV_STATE_WORDS * sizeof(uint32_t), "state layout");

struct ppv_index {
    IndexView view;
    NodeEnt *d_ent;
    uint32_t *d_node_lo, *d_node_hi;
    uint32_t *d_heavy_slot, *d_heavy_bits, *d_heavy_rank;
    LookupEntry *d_lookup;
    uint32_t *d_node_at;
    int32_t *d_x_tok;    // sorted S, flat, no padding: row r is d_x_tok[d_x_off[r] .. d_x_off[r+1])
    int64_t *d_x_off;    // [n_rows + 1]
    int64_t n_tokens;
    int64_t n_heavy;
    int64_t device_bytes;
    void *block, *heavy_block;   // the pool's blocks that the arrays above lie in
    int device;
};

// Device memory kept from one index to the next, and the upload of a set (ppv_pool.hip).  ppv_pool_give:
// `over` says that the device has finished with the block; where the caller's wait failed, the block is not kept.
// `got`: the block's size, which may be more than was asked for.  ppv_pool_empty: everything that is kept goes back to the system.
ppv_status ppv_pool_take(void **out, size_t bytes, size_t *got = nullptr);
void ppv_pool_give(void *block, bool over);
void ppv_pool_empty();
// A little pinned memory that kernels can write (nullptr: none to be had).
constexpr int PPV_HOST_WORDS_BYTES = 64;
void *ppv_host_words_take();
void ppv_host_words_give(void *words);
// Checks S (host CSR) and enqueues its copy to the device in packed form: the tokens' lower 16 bits, the bits above
// them (d_hi, nullptr where the vocabulary has none), the offsets.  Returns when the host arrays have been read.
ppv_status ppv_upload_set(const int32_t *tokens, const int64_t *offsets, int64_t n_seq, int32_t vocab, uint16_t *d_lo,
                          uint8_t *d_hi, uint32_t *d_off, hipStream_t st, int32_t *l_max);

// Current value of a tuning / test switch (PPV_TUNE_* of ppv.h): read from the environment once at load,
// changed by ppv_tuning_set.
int ppv_tuning(int knob);

#define PPV_HIP_TRY(expr)                          \
    do {                                           \
        hipError_t e_ = (expr);                    \
        if (e_ != hipSuccess) {                    \
            (void)hipGetLastError();               \
            return (e_ == hipErrorOutOfMemory) ? PPV_ENOMEM : PPV_EDEVICE; \
        }                                          \
    } while (0)
