// Device-side helpers shared by the kernel files (internal): storage dtype conversion, wavefront reductions, the
// bf16 hi/lo split of fp32 operands, the KV cache's value layout.
#pragma once
#include "common.h"

namespace bs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---- storage dtype helpers ----------------------------------------------------------------------
__device__ __forceinline__ float to_f(float v) { return v; }
__device__ __forceinline__ float to_f(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
template <typename T> __device__ __forceinline__ T from_f(float f);
template <> __device__ __forceinline__ float from_f<float>(float f) { return f; }
// float -> bf16, round to nearest even: gfx950 has the conversion in hardware (v_cvt_pk_bf16_f32, two values per
// instruction), which the compiler emits for a cast to __bf16; four integer instructions per value otherwise
typedef __bf16 bf16x2_hw __attribute__((ext_vector_type(2)));
template <> __device__ __forceinline__ uint16_t from_f<uint16_t>(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

__device__ __forceinline__ float wsum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wmax(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// ---- KV cache layout --------------------------------------------------------------------------------
// Per (sequence, kv head): K is [cache_len][hd] (a key's row is contiguous: MFMA A operand of K.Q^T).
// V of a bf16 cache is stored transposed in blocks of 32 keys, [cache_len/32][hd][32], and inside a block
// the key k = 16t + 4q + e sits at slot 8q + 4t + e: lane (d, q) of the MFMA A operand of V^T.P^T then
// finds its 8 keys in one 16-byte load, in exactly the key order in which the score accumulators of
// K.Q^T hold the probabilities.  cache_len is a multiple of 32.  fp32 caches keep V as [cache_len][hd].
template <typename T> __device__ __forceinline__ size_t v_index(int key, int d, int hd);
template <> __device__ __forceinline__ size_t v_index<float>(int key, int d, int hd) { return (size_t)key * hd + d; }
template <> __device__ __forceinline__ size_t v_index<uint16_t>(int key, int d, int hd) {
    const int k = key & 31;
    const int slot = ((k & 15) >> 2) * 8 + (k >> 4) * 4 + (k & 3);
    return ((size_t)(key >> 5) * hd + d) * 32 + slot;
}

__device__ __forceinline__ uint4 ldg16(const uint16_t* p) { return *reinterpret_cast<const uint4*>(p); }
// NT: the line is asked for as one that nobody reads again (see streams_past_cache)
typedef unsigned int ldg_vec __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ __forceinline__ uint4 ldg16_stream(const uint16_t* p) {
    return NT ? __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const ldg_vec*>(p))) : ldg16(p);
}

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    const bf16x2_hw v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ void split8(const float v[8], uint4& hi, uint4& lo) {
    float r[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = v[e] - to_f(from_f<uint16_t>(v[e]));
    hi = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
    lo = make_uint4(pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3]), pack_bf16(r[4], r[5]), pack_bf16(r[6], r[7]));
}

// four consecutive activations (index a multiple of 4) as two 8-byte stores, one per plane
__device__ __forceinline__ void store_planes4(uint16_t* base, size_t plane, size_t idx, float v0, float v1, float v2, float v3) {
    const uint16_t h0 = from_f<uint16_t>(v0), h1 = from_f<uint16_t>(v1), h2 = from_f<uint16_t>(v2), h3 = from_f<uint16_t>(v3);
    const uint16_t l0 = from_f<uint16_t>(v0 - to_f(h0)), l1 = from_f<uint16_t>(v1 - to_f(h1));
    const uint16_t l2 = from_f<uint16_t>(v2 - to_f(h2)), l3 = from_f<uint16_t>(v3 - to_f(h3));
    *reinterpret_cast<uint2*>(base + idx) = make_uint2((uint32_t)h0 | ((uint32_t)h1 << 16), (uint32_t)h2 | ((uint32_t)h3 << 16));
    *reinterpret_cast<uint2*>(base + plane + idx) = make_uint2((uint32_t)l0 | ((uint32_t)l1 << 16), (uint32_t)l2 | ((uint32_t)l3 << 16));
}

// Tiled activation planes: [K/32][R rows][32 columns].  For the whole-K projections of up to 32 rows (gemm_rows_kernel) R = 16
// or 32 (rows_tiled), so that the B operand of one k step (16 rows x 64 bytes) is one contiguous kilobyte like a weight tile,
// instead of 16 pieces of 16 different cache lines.  A plane is R*K elements whatever the row count; rows >= M are neither
// written nor read.  For the many-row projections (gemm_big.hip) R is the row count rounded up to 16: the 16 rows of a stage that a
// wavefront's transfer moves into LDS are then eight whole cache lines, not halves of sixteen whose other halves are the next stage's.
// R = 32: inside a k step [row / 4][chunk of 8 columns][row % 4][8].  The address unit takes four consecutive lanes at a time, and in
// a B operand these hold one chunk of four rows: here they meet in one 64-byte run instead of four.  With two row tiles the activations are
// most of what O and down request (7B layer, 20 rows: O 14.0 -> 13.2, down 33.5 -> 31.8 us; a pass 4646 -> 4553).  With one tile
// the planes stay row by row: 9 rows touch 5 lines of a k step that way and 6 this way (O and down together 31.5 -> 32.3 us).
__device__ __forceinline__ size_t xt_index(int m, int k, int R) {
    const int in = R == 32 ? (m >> 2) * 128 + ((k >> 3) & 3) * 32 + (m & 3) * 8 + (k & 7) : m * 32 + (k & 31);
    return (size_t)(k >> 5) * (R * 32) + in;
}

// r = rsqrt(mean square + eps) of row m from its per-chunk sums of squares (null: no scaling)
__device__ __forceinline__ float row_rscale(const float* __restrict__ ssq, int nchunks, int m, float inv_d, float eps) {
    if (!ssq) return 1.f;
    float tot = 0.f;
    if (nchunks <= 8) {
        for (int c = 0; c < nchunks; ++c) tot += ssq[(size_t)m * nchunks + c];
    } else {
        for (int c0 = 0; c0 < nchunks; c0 += 8) {    // eight loads in flight: O and down projections leave a sum per tile of columns
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = ssq[(size_t)m * nchunks + min(c0 + i, nchunks - 1)];
#pragma unroll
            for (int i = 0; i < 8; ++i) tot += c0 + i < nchunks ? v[i] : 0.f;
        }
    }
    return 1.0f / sqrtf(tot * inv_d + eps);
}

// ---- weight layouts -------------------------------------------------------------------------------------
// Weight layouts.  Row-major [N][K], or TILED: the matrix is cut into 64-row x 32-column blocks stored
// [N/64][K/32][4][64][8]: inside a block the four 16-row MFMA A tiles follow each other, and inside a tile the
// eight values of lane (row r, k-slot q) sit at lane index r + 16q.  One k step of a wavefront is then one
// contiguous kilobyte and the four wavefronts of a workgroup read 4 KiB runs, which is what HBM serves fastest
// (measured 3.6 -> 4.6 TB/s over the 7B layer shapes against 64-byte pieces 8 KiB apart).
// wlane_ptr: where lane (row local%16, k-slot lq) finds its chunk of k step 0; WSTEP: elements between k steps.
template <bool TILED> struct WSTEP { static constexpr int v = TILED ? 2048 : 32; };
template <bool TILED>
__device__ __forceinline__ const uint16_t* wlane_ptr(const uint16_t* w, int local, int K, int lq) {
    if (TILED) return w + (size_t)(local >> 6) * 64 * K + ((local >> 4) & 3) * 512 + ((local & 15) + 16 * lq) * 8;
    return w + (size_t)local * K + lq * 8;
}

// ---- transfers from memory into LDS -----------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef __attribute__((address_space(1))) const void* global_void_ptr;

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}
// s_waitcnt immediate for "at most n vector-memory operations outstanding" (the other counters unconstrained)
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

// ---- exchange cells {float value, uint32 flag}: device-scope accesses ------------------------------------------------
// Data handed from one workgroup to another INSIDE a kernel travels in 8-byte cells that carry their own flag: one
// store, one load, no fence, and a cell is valid when its flag is the one the reader expects.  The accesses bypass the
// per-die caches (sc1), an 8-byte cell becomes visible as a whole.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
struct DevBuf { __amdgpu_buffer_rsrc_t r; };
__device__ __forceinline__ DevBuf dev_buf(const void* base) {
    DevBuf b;
    b.r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7FFFFFFF, 0x00020000);
    return b;
}
constexpr int AUX_SC1 = 16;
// two cells at cell index c (even): one 16-byte store; each 8-byte cell becomes visible as a whole
__device__ __forceinline__ void st_cells2(DevBuf b, int c, float v0, float v1, unsigned flag) {
    const u32x4 u = {__float_as_uint(v0), flag, __float_as_uint(v1), flag};
    __builtin_amdgcn_raw_buffer_store_b128(u, b.r, c * 8, 0, AUX_SC1);
}
__device__ __forceinline__ void st_cells4(DevBuf b, int c, float v0, float v1, float v2, float v3, unsigned flag) {
    st_cells2(b, c, v0, v1, flag);
    st_cells2(b, c + 2, v2, v3, flag);
}
__device__ __forceinline__ u32x4 ld_cells2(DevBuf b, int c) { return __builtin_amdgcn_raw_buffer_load_b128(b.r, c * 8, 0, AUX_SC1); }
__device__ __forceinline__ u32x2 ld_cell1(DevBuf b, int c) { return __builtin_amdgcn_raw_buffer_load_b64(b.r, c * 8, 0, AUX_SC1); }

}  // namespace bs
