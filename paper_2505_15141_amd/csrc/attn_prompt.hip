// Attention of a prompt chunk: many query rows per head group against the cache, one workgroup per 64 or 128 rows.
#include <math.h>
#include "common.h"
#include "kernels.h"
#include "devutil.h"

namespace bs {

// The decode kernel (attn_mfma_kernel) gives its four wavefronts different keys of the same 32 rows, which is what a pass
// over a long cache with few rows wants; for a prompt chunk it read every K and V block once per 32 rows and wavefront from
// the L2 and ran at 170-250 TFLOP/s.  Here the wavefronts of a workgroup own different rows (16 NT each) and walk the keys
// together: a block of 32 keys (K and V, 16 KB at head_dim 128) goes memory -> LDS once for all of them, two blocks ahead in a
// ring of three, and what bounds the kernel is the matrix cores and the exponentials (two wavefronts per SIMD).
// Rows are ordered by position, then query head (row = position * G + head of the group), so the rows of a workgroup have
// nearly the same causal horizon.  Masks are worked out only in blocks some row of the wavefront does not see whole, the
// outputs are rescaled only when some row's maximum has grown (otherwise the factor is one).  Workgroups start with the
// longest horizons; those of one kv head sit on one die (workgroups go round the 8 dies) and share its keys in the L2.
// S^T = K . Q^T and O^T += V^T . P^T as in the decode kernel, Q and P as hi/lo pairs.
// Measured against it, per layer: 1023 tokens of one prompt (7B shape) 103 -> 37 us; 8 prompts in chunks of 512 tokens (8B
// shape), 512 cached tokens in front on average 354 -> 95 us, 1024 in front 496 -> 175 us (690 TFLOP/s of issued MFMAs).

// Where the 16-byte chunks of a block sit in LDS: chunk c of K row r at slot c ^ r (modulo the chunks of a row), chunk c of V
// row d at slot (c + d / 2) & 3: eight consecutive rows' chunks are eight different bank groups.
template <int HD> struct KvBlock { uint16_t k[32 * HD], v[32 * HD]; };

// four (or eight) 16-byte LDS reads and the wait for them in one block: nothing in flight is left to the compiler
__device__ __forceinline__ void lds_read_k8(u32x4 (&r)[8], const uint32_t (&a)[4]) {        // rows 16 further: 4096 bytes
    asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
                 "ds_read_b128 %4, %8 offset:4096\n\tds_read_b128 %5, %9 offset:4096\n\tds_read_b128 %6, %10 offset:4096\n\tds_read_b128 %7, %11 offset:4096\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
                 : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]) : "memory");
}
__device__ __forceinline__ void lds_read_k8(u32x4 (&r)[4], const uint32_t (&a)[2]) {        // head_dim 64: rows 16 further, 2048 bytes
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %4 offset:2048\n\tds_read_b128 %3, %5 offset:2048\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]) : "v"(a[0]), "v"(a[1]) : "memory");
}
__device__ __forceinline__ void lds_read_v(u32x4 (&r)[8], uint32_t a) {
    asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:1024\n\tds_read_b128 %2, %8 offset:2048\n\tds_read_b128 %3, %8 offset:3072\n\t"
                 "ds_read_b128 %4, %8 offset:4096\n\tds_read_b128 %5, %8 offset:5120\n\tds_read_b128 %6, %8 offset:6144\n\tds_read_b128 %7, %8 offset:7168\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7]) : "v"(a) : "memory");
}
__device__ __forceinline__ void lds_read_v(u32x4 (&r)[4], uint32_t a) {
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:1024\n\tds_read_b128 %2, %4 offset:2048\n\tds_read_b128 %3, %4 offset:3072\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]) : "v"(a) : "memory");
}

template <int HD, int NT>
__global__ __launch_bounds__(256, 2) void attn_prompt_kernel(const float* __restrict__ q, const uint16_t* __restrict__ k_cache,
                                                             const uint16_t* __restrict__ v_cache, const int32_t* __restrict__ pos,
                                                             int B, int q_len, int H, int KVH, int cache_len, float scale,
                                                             int n_rt, uint16_t* __restrict__ out, size_t plane, int tiled) {
    constexpr int DS = HD / 32, DT = HD / 16, ROWS = 64 * NT, FK = HD / 64;      // FK: kilobytes of K (and of V) a wavefront fetches
    __shared__ __attribute__((aligned(16))) KvBlock<HD> kvs[3];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lq = lane >> 4;
    const int n_bk = B * KVH, bk = blockIdx.x % n_bk, rt = n_rt - 1 - blockIdx.x / n_bk;
    const int b = bk / KVH, kvh = bk - b * KVH;
    const int G = H / KVH, R = G * q_len, m_first = b * q_len, r0 = rt * ROWS;
    const int pos0 = pos[m_first];
    if (pos0 < 0) {                                                // sequence left out: zeros
        const int nr = min(ROWS, R - r0);
        for (int idx = threadIdx.x; idx < nr * (HD / 4); idx += 256) {
            const int r = r0 + idx / (HD / 4), c = idx % (HD / 4) * 4;
            const int m = m_first + r / G, col = (kvh * G + r % G) * HD + c;
            store_planes4(out, plane, tiled ? xt_index(m, col, tiled) : (size_t)m * H * HD + col, 0.f, 0.f, 0.f, 0.f);
        }
        return;
    }
    const int n_keys = pos0 + q_len;
    const int nblk = (pos0 + (min(r0 + ROWS, R) - 1) / G + 32) / 32;               // blocks the workgroup's last row sees
    const int w0 = r0 + wave * 16 * NT, wl = min(w0 + 16 * NT, R) - 1;
    const int wblk = w0 < R ? (pos0 + wl / G + 32) / 32 : 0;                       // blocks this wavefront's last row sees
    const int whole_end = w0 < R ? pos0 + w0 / G : 0;                              // keys up to here are seen by all its rows
    const uint16_t* kb = k_cache + ((size_t)b * KVH + kvh) * (size_t)cache_len * HD;
    const uint16_t* vb = v_cache + ((size_t)b * KVH + kvh) * (size_t)cache_len * HD;

    // this lane's sources within a block: piece p = wave + 4 f is the p-th kilobyte of the block's K, and of its V
    uint32_t ksrc[FK], vsrc[FK];
#pragma unroll
    for (int f = 0; f < FK; ++f) {
        const int p = wave + 4 * f;
        const int kr = (p * 512 + lane * 8) / HD, ks = lane & (HD / 8 - 1);
        ksrc[f] = kr * HD + (ks ^ (kr & (HD / 8 - 1))) * 8;
        const int vr = p * 16 + (lane >> 2);
        vsrc[f] = vr * 32 + (((lane & 3) - (vr >> 1)) & 3) * 8;
    }
    auto fill = [&](int blk, int buf) {
        const size_t base = (size_t)min(blk, nblk - 1) * 32 * HD;  // past the end: the last block again, into a buffer nobody reads
#pragma unroll
        for (int f = 0; f < FK; ++f) {
            __builtin_amdgcn_global_load_lds((global_void_ptr)(kb + base + ksrc[f]), (lds_void_ptr)&kvs[buf].k[(wave + 4 * f) * 512], 16, 0, 0);
            __builtin_amdgcn_global_load_lds((global_void_ptr)(vb + base + vsrc[f]), (lds_void_ptr)&kvs[buf].v[(wave + 4 * f) * 512], 16, 0, 0);
        }
    };
    bf16x8 qh[NT][DS], ql[NT][DS];
    int row_pos[NT];
    float m_run[NT], l_run[NT];
    f32x4 o[NT][DT];
#pragma unroll
    for (int x = 0; x < NT; ++x) {
        const int row = w0 + 16 * x + li, rc = min(row, R - 1), qi = rc / G, g = rc - qi * G;
        row_pos[x] = pos0 + qi;
        const float* qrow = q + ((size_t)(m_first + qi) * H + kvh * G + g) * HD;
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
            const float4 a = *reinterpret_cast<const float4*>(qrow + ds * 32 + lq * 8);
            const float4 c = *reinterpret_cast<const float4*>(qrow + ds * 32 + lq * 8 + 4);
            const float v[8] = {a.x * scale, a.y * scale, a.z * scale, a.w * scale, c.x * scale, c.y * scale, c.z * scale, c.w * scale};
            uint4 hi, lo;
            split8(v, hi, lo);
            qh[x][ds] = __builtin_bit_cast(bf16x8, hi); ql[x][ds] = __builtin_bit_cast(bf16x8, lo);
        }
        m_run[x] = -INFINITY; l_run[x] = 0.f;
#pragma unroll
        for (int t = 0; t < DT; ++t) o[x][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    uint32_t ka[DS];                                               // this lane's K chunks of row li of block buffer 0
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) ka[ds] = lds_addr(&kvs[0].k[0]) + li * HD * 2 + (((ds * 4 + lq) ^ (li & (HD / 8 - 1))) * 16);
    const uint32_t va = lds_addr(&kvs[0].v[0]) + li * 64 + ((lq + (li >> 1)) & 3) * 16;

    fill(0, 0);
    fill(1, 1);
    int buf = 0;
    for (int blk = 0; blk < nblk; ++blk) {
        // this wavefront's pieces of the block have landed; behind the barrier everybody's have, and everybody is done with
        // the block before, whose buffer takes the next request (__syncthreads would wait for the requests in flight too)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * FK));
        __builtin_amdgcn_s_barrier();
        fill(blk + 2, buf == 0 ? 2 : buf - 1);
        if (blk < wblk) {
            const uint32_t boff = buf * (uint32_t)sizeof(KvBlock<HD>);
            const int key0 = blk * 32;
            u32x4 kf[2 * DS];
            uint32_t kab[DS];
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) kab[ds] = ka[ds] + boff;
            lds_read_k8(kf, kab);
            f32x4 sc[NT][2];
#pragma unroll
            for (int x = 0; x < NT; ++x) { sc[x][0] = f32x4{0.f, 0.f, 0.f, 0.f}; sc[x][1] = sc[x][0]; }
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int x = 0; x < NT; ++x)
                        sc[x][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[t * DS + ds]), qh[x][ds], sc[x][t], 0, 0, 0);
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int x = 0; x < NT; ++x)
                        sc[x][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[t * DS + ds]), ql[x][ds], sc[x][t], 0, 0, 0);
            }
            // lane holds S^T[key0 + 16t + 4lq + e][row li], in base-2 exponents
            bf16x8 ph[NT], pl[NT];
#pragma unroll
            for (int x = 0; x < NT; ++x) {
                float sv[8], bm = -INFINITY;
                if (key0 + 31 > whole_end) {                       // some row does not see the whole block
#pragma unroll
                    for (int e = 0; e < 8; ++e) sv[e] = key0 + (e >> 2) * 16 + 4 * lq + (e & 3) <= row_pos[x] ? sc[x][e >> 2][e & 3] : -INFINITY;
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) sv[e] = sc[x][e >> 2][e & 3];
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) bm = fmaxf(bm, sv[e]);
                bm = fmaxf(bm, __shfl_xor(bm, 16, 64));
                bm = fmaxf(bm, __shfl_xor(bm, 32, 64));
                // every row sees key 0, so its maximum is finite from the first block on
                if (__any(bm > m_run[x])) {
                    const float m_new = fmaxf(m_run[x], bm), alpha = __builtin_amdgcn_exp2f(m_run[x] - m_new);
                    m_run[x] = m_new;
                    l_run[x] *= alpha;
#pragma unroll
                    for (int t = 0; t < DT; ++t) { o[x][t][0] *= alpha; o[x][t][1] *= alpha; o[x][t][2] *= alpha; o[x][t][3] *= alpha; }
                }
                float pv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) { pv[e] = __builtin_amdgcn_exp2f(sv[e] - m_run[x]); l_run[x] += pv[e]; }
                uint4 hi, lo;
                split8(pv, hi, lo);
                ph[x] = __builtin_bit_cast(bf16x8, hi); pl[x] = __builtin_bit_cast(bf16x8, lo);
            }
            u32x4 vf[DT];
            lds_read_v(vf, va + boff);
            if (key0 + 32 > n_keys) {                              // values of keys past the end may hold anything, NaN patterns too
#pragma unroll
                for (int t = 0; t < DT; ++t)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (key0 + (e >> 2) * 16 + 4 * lq + (e & 3) >= n_keys) vf[t][e >> 1] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
            }
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int x = 0; x < NT; ++x)
                    o[x][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf[t]), ph[x], o[x][t], 0, 0, 0);
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int x = 0; x < NT; ++x)
                    o[x][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf[t]), pl[x], o[x][t], 0, 0, 0);
        }
        buf = buf == 2 ? 0 : buf + 1;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                      // no transfer into LDS is left in flight
#pragma unroll
    for (int x = 0; x < NT; ++x) {
        const int row = w0 + 16 * x + li;
        float l = l_run[x];
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        if (row >= R) continue;
        const int qi = row / G, g = row - qi * G;
        const float inv = l > 0.f ? 1.0f / l : 0.f;
        const int m = m_first + qi, col = (kvh * G + g) * HD + 4 * lq;
#pragma unroll
        for (int t = 0; t < DT; ++t) store_planes4(out, plane, tiled ? xt_index(m, col + 16 * t, tiled) : (size_t)m * H * HD + col + 16 * t, o[x][t][0] * inv, o[x][t][1] * inv, o[x][t][2] * inv, o[x][t][3] * inv);
    }
}

// 128 rows and more per head group, and as many workgroups of 64 rows as compute units: with fewer the decode kernel's key
// splits fill the chip better.
bool attn_prompt_applies(int B, int q_len, int H, int KVH, int hd) {
    const long long R = (long long)(H / KVH) * q_len;
    return (hd == 64 || hd == 128) && R >= 128 && (long long)B * KVH * ((R + 63) / 64) >= 256;
}

int launch_attn_prompt(const float* q, const uint16_t* k_cache, const uint16_t* v_cache, const int32_t* pos, int B, int q_len, int H, int KVH,
                       int hd, int cache_len, uint16_t* out, size_t plane, int tiled, hipStream_t s) {
    BS_REQUIRE(attn_prompt_applies(B, q_len, H, KVH, hd) && cache_len % 32 == 0, BS_ESHAPE, "attn_prompt: B=%d q_len=%d head_dim=%d", B, q_len, hd);
    const int R = H / KVH * q_len;
    const float scale = 1.44269504088896341f / sqrtf((float)hd);   // scores as base-2 exponents
    // two row tiles per wavefront halve the LDS reads per MFMA; with fewer than two such workgroups per compute unit the
    // shorter ones even out the causal horizons better
    const bool wide = (long long)B * KVH * ((R + 127) / 128) >= 512;
    const int n_rt = wide ? (R + 127) / 128 : (R + 63) / 64;
    const dim3 grid(B * KVH * n_rt), block(256);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    const int rc = prof_events(s, &e0, &e1);
    if (rc != BS_OK) return rc;
#define BS_PROMPT(HD, NT) BS_LAUNCH_TIMED((attn_prompt_kernel<HD, NT>), grid, block, 0, s, e0, e1, q, k_cache, v_cache, pos, B, q_len, H, KVH, cache_len, scale, n_rt, out, plane, tiled)
    if (hd == 128) { if (wide) BS_PROMPT(128, 2); else BS_PROMPT(128, 1); }
    else { if (wide) BS_PROMPT(64, 2); else BS_PROMPT(64, 1); }
#undef BS_PROMPT
    BS_LAUNCH_CHECK();
    prof_record(e0, e1, 0.0, 100);
    return BS_OK;
}

}  // namespace bs
