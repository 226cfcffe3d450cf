// Wave-level device helpers shared by the kernels of libppv_hip.so (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

constexpr int WAVE = 64;

// wave-level helpers on DPP (data-parallel primitives: a lane reads a neighbour's register inside
// the VALU instruction, no LDS round trip).  Reductions return a wave-uniform value.
constexpr int DPP_QUAD_XOR1 = 0xB1;     // quad_perm [1,0,3,2]
constexpr int DPP_QUAD_XOR2 = 0x4E;     // quad_perm [2,3,0,1]
constexpr int DPP_ROW_SHR1 = 0x111, DPP_ROW_SHR2 = 0x112, DPP_ROW_SHR3 = 0x113, DPP_ROW_SHR4 = 0x114,
              DPP_ROW_SHR8 = 0x118;
constexpr int DPP_ROW_MIRROR = 0x140, DPP_ROW_HALF_MIRROR = 0x141, DPP_ROW_BCAST15 = 0x142, DPP_ROW_BCAST31 = 0x143;

// source lane's value, or 0 where the lane has no source or is masked off
template <int CTRL, int ROW_MASK = 0xF, int BANK_MASK = 0xF> __device__ inline int dpp0(int x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, ROW_MASK, BANK_MASK, true);
}
template <int CTRL, int ROW_MASK = 0xF, int BANK_MASK = 0xF> __device__ inline uint32_t dpp0(uint32_t x) {
    return (uint32_t)dpp0<CTRL, ROW_MASK, BANK_MASK>((int)x);
}
template <int CTRL, int ROW_MASK = 0xF, int BANK_MASK = 0xF> __device__ inline float dpp0(float x) {
    return __int_as_float(dpp0<CTRL, ROW_MASK, BANK_MASK>(__float_as_int(x)));
}
template <int CTRL, int ROW_MASK = 0xF, int BANK_MASK = 0xF> __device__ inline uint64_t dpp0(uint64_t x) {
    return ((uint64_t)dpp0<CTRL, ROW_MASK, BANK_MASK>((uint32_t)(x >> 32)) << 32) | dpp0<CTRL, ROW_MASK, BANK_MASK>((uint32_t)x);
}
template <int CTRL, int ROW_MASK = 0xF, int BANK_MASK = 0xF> __device__ inline double dpp0(double x) {
    return __hiloint2double(dpp0<CTRL, ROW_MASK, BANK_MASK>(__double2hiint(x)),
                            dpp0<CTRL, ROW_MASK, BANK_MASK>(__double2loint(x)));
}
__device__ inline float last_lane(float x) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63)); }
__device__ inline int last_lane(int x) { return __builtin_amdgcn_readlane(x, 63); }
__device__ inline uint32_t last_lane(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }
__device__ inline uint64_t last_lane(uint64_t x) {
    return ((uint64_t)last_lane((uint32_t)(x >> 32)) << 32) | last_lane((uint32_t)x);
}
__device__ inline double last_lane(double x) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 63),
                            __builtin_amdgcn_readlane(__double2loint(x), 63));
}

// value held by lane l (l must be wave-uniform)
__device__ inline int lane_value(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
__device__ inline uint32_t lane_value(uint32_t x, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)x, l); }
__device__ inline double lane_value(double x, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                            __builtin_amdgcn_readlane(__double2loint(x), l));
}

// The reductions of floats are written out: from the builtins the compiler makes three or four instructions of a step
// (a copy, a move across lanes, a NaN made quiet, the operation), and a tile of logits has eight such steps.  A step reads
// other lanes' results of the step before, which takes two idle cycles.
#define PPV_DPP_STEP(OP, CTRL) OP " %0, %0, %0 " CTRL "\n\ts_nop 1\n\t"
#define PPV_DPP_QUAD(OP)                                                      \
    PPV_DPP_STEP(OP, "quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf")        \
    PPV_DPP_STEP(OP, "quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf")
#define PPV_DPP_WAVE(OP)                                                                                        \
    "s_nop 1\n\t" PPV_DPP_QUAD(OP)                                                                              \
    PPV_DPP_STEP(OP, "row_half_mirror row_mask:0xf bank_mask:0xf")                                              \
    PPV_DPP_STEP(OP, "row_mirror row_mask:0xf bank_mask:0xf")       /* every lane: result over its row of 16 */ \
    PPV_DPP_STEP(OP, "row_bcast:15 row_mask:0xa bank_mask:0xf")     /* rows 1, 3 take in rows 0, 2 */           \
    OP " %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf"        /* rows 2, 3 take in lane 31 */
__device__ inline float quad_max(float x) {   // over each four lanes; NaNs are passed over
    asm("s_nop 1\n\t" PPV_DPP_QUAD("v_max_f32_dpp") : "+v"(x));
    return x;
}
__device__ inline float wave_max(float x) {
    asm(PPV_DPP_WAVE("v_max_f32_dpp") : "+v"(x));
    return last_lane(x);
}
// source lane's value, or the lane's own value where it has no source or is masked off
template <int CTRL, int ROW_MASK = 0xF, int BANK_MASK = 0xF> __device__ inline uint32_t dpp_self(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, ROW_MASK, BANK_MASK, false);
}
__device__ inline uint32_t wave_max(uint32_t x) {
    x = max(x, dpp_self<DPP_QUAD_XOR1>(x));
    x = max(x, dpp_self<DPP_QUAD_XOR2>(x));
    x = max(x, dpp_self<DPP_ROW_HALF_MIRROR>(x));
    x = max(x, dpp_self<DPP_ROW_MIRROR>(x));
    x = max(x, dpp_self<DPP_ROW_BCAST15, 0xA>(x));
    x = max(x, dpp_self<DPP_ROW_BCAST31, 0xC>(x));
    return last_lane(x);
}
template <typename V> __device__ inline V wave_sum(V x) {
    x += dpp0<DPP_QUAD_XOR1>(x);
    x += dpp0<DPP_QUAD_XOR2>(x);
    x += dpp0<DPP_ROW_HALF_MIRROR>(x);
    x += dpp0<DPP_ROW_MIRROR>(x);
    x += dpp0<DPP_ROW_BCAST15, 0xA>(x);
    x += dpp0<DPP_ROW_BCAST31, 0xC>(x);
    return last_lane(x);
}
__device__ inline float wave_sum(float x) {   // (the same sums in the same order as above)
    asm(PPV_DPP_WAVE("v_add_f32_dpp") : "+v"(x));
    return last_lane(x);
}
// inclusive prefix sum over the 64 lanes (lane order)
template <typename V> __device__ inline V wave_incl_scan(V x) {
    V t = x;
    t += dpp0<DPP_ROW_SHR1>(x);
    t += dpp0<DPP_ROW_SHR2>(x);
    t += dpp0<DPP_ROW_SHR3>(x);                          // up to 4 consecutive lanes of the row
    t += dpp0<DPP_ROW_SHR4, 0xF, 0xE>(t);
    t += dpp0<DPP_ROW_SHR8, 0xF, 0xC>(t);                // prefix inside each row of 16
    t += dpp0<DPP_ROW_BCAST15, 0xA>(t);
    t += dpp0<DPP_ROW_BCAST31, 0xC>(t);
    return t;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// A row as the memory unit's buffer: its address and its length in bytes, up to the 16 that hold its last token (rows start on
// 16-byte boundaries).  What is asked for behind the length is not read and arrives as 0.
struct Row {
    __amdgpu_buffer_rsrc_t buf;
};
template <typename T, uint32_t PAD = 15u> __device__ __forceinline__ Row row_of(const T *row, int V) {
    // (uniform, which the compiler does not see where the row came with a loop)
    const uint64_t at = (uint64_t)row;
    const uint64_t base = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(at >> 32)) << 32) |
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at);
    const uint32_t bytes = (uint32_t)__builtin_amdgcn_readfirstlane(V) * (uint32_t)sizeof(T);
    return {__builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (bytes + PAD) & ~PAD, 0x00027000)};
}
