// Device kernels of the transformer forward used by the verification pass (App. A: the target model
// scores all gamma+1 positions in one pass) and by the draft model's steps.
//
//   prep        positions, clamped tokens, RoPE cos/sin table, overflow status
//   embed       token embedding -> fp32 residual stream
//   rmsnorm     completes the fp32 residual from pending split-K partials, normalises it
//   gemm        y = x W^T: bf16 weights streamed once from HBM through MFMA 16x16x32 tiles (the
//               contraction is skinny: M = B*(gamma+1) rows, so it is bound by weight bandwidth),
//               split-K partials out; a many-row variant for prompt chunks and batches (activation
//               stages memory -> LDS directly, 512 x 128 tiles); fp32 variant for the fp32 plumbing
//               configuration
//   resid_sum   bf16 models: completes the residual, writes the planes of gain .* x and partial sums
//               of squares (the RMS scale is applied behind the projection)
//   gemm_dec    the same contraction for one or two rows (draft steps) with the layer's small kernels
//               folded into its epilogues (residual, RoPE + cache write, SwiGLU; RMSNorm by linearity)
//   swiglu      sums gate/up partials, applies silu(g)*u
//   rope_kv     sums q/k/v partials, rotates q and k, writes k/v into the cache
//   attention   q_len causal query rows per head against the contiguous KV cache, split along the
//               keys with online softmax; merge kernel combines the splits
#include <math.h>
#include <initializer_list>
#include <mutex>
#include <vector>
#include <hip/hip_ext.h>
#include "common.h"
#include "kernels.h"
#include "devutil.h"

namespace bs {

// ---- prep ---------------------------------------------------------------------------------------
// One workgroup per sequence and 32 of its rows (a double-precision power, sine and cosine per rotation pair: one workgroup
// for a prompt of 1023 rows took 140 us).  pos[m] = kv_len[b] + kv_base + j, or -1 for a sequence that would run
// past max_len (then nothing of it is written anywhere).  tok[m] = token clamped into [0, V).
constexpr int PREP_ROWS = 32;

// The attention's work items where long sequences are cut into more parts (attn_plan): how many parts sequence b has, and its items.  Long
// sequences come first, so that their parts fall on different compute units.  8 layers of the 7B shape, 8 sequences of 9 rows, one of
// 8000 keys and seven of 500: 2388 us with one part for all, 2014 with the long one's other parts behind the first part of every
// sequence, where two of them came to share a compute unit, 1865 like this; all of 8000 keys 2680 either way.  12 layers of 12 heads of 64, 32
// sequences of one row, one of 8000 keys and the others of 300: 1103 -> 986, all of 8000 2269 -> 2268, all of 4096 1381 -> 1392.  One
// wavefront per sequence, each with its own look at all lengths.
__device__ __forceinline__ void attn_deal(const AttnParts& ap, const int32_t* __restrict__ kv_len, int kv_base, int q_len, int max_len, int B, int b, int pos0) {
    const int lane = threadIdx.x;
    auto keys = [&](int i) -> int {                                // all of them together fit a cache in memory: 31 bits
        const int k = i < B ? (kv_len ? kv_len[i] : 0) + kv_base : -1;
        return k >= 0 && k + q_len <= max_len ? k + q_len : 0;
    };
    auto total = [](int v) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        return v;
    };
    const int k0 = keys(lane);                                     // the first 64 sequences are asked for once
    int sum = k0;
    for (int i = lane + 64; i < B; i += 64) sum += keys(i);
    sum = total(sum);
    auto cut = [&](int own) -> int {                               // a long sequence: as many parts as compute units it would keep busy at an equal share
        if (4ll * own * B <= 5ll * sum) return ap.few;
        const int share = (int)((long long)own * ap.cus / ((long long)sum * ap.kv_heads));
        return share > ap.few ? min(share, ap.most) : ap.few;
    };
    int extra = 0, n_long = 0, extra_before = 0, long_before = 0;
    for (int i0 = 0; i0 < B; i0 += 64) {
        const int n = cut(i0 == 0 ? k0 : keys(i0 + lane)) - ap.few;
        const unsigned long long is_long = __ballot(n > 0), before = b >= i0 + 64 ? ~0ull : b > i0 ? (1ull << (b - i0)) - 1 : 0ull;
        if (!is_long) continue;
        const int both = total(n | ((before >> lane) & 1 ? n << 16 : 0));       // n and those in front of b: at most as many as compute units
        extra += both & 0xFFFF; extra_before += both >> 16;
        n_long += __popcll(is_long); long_before += __popcll(is_long & before);
    }
    const int own = pos0 >= 0 ? cut(pos0 + q_len) : ap.few;
    const int first = own > ap.few ? long_before * ap.few + extra_before : extra + (n_long + b - long_before) * ap.few;
    if (lane < own) ap.items[first + lane] = (long long)(b | lane << 16 | own << 24) << 32 | (unsigned)pos0;
    if (lane == 0) ap.parts[b] = own;
    if (b == 0)
        for (int i = extra + B * ap.few + lane; i < ap.n_items; i += 64) ap.items[i] = -1;
}

__global__ void prep_kernel(const int32_t* __restrict__ q_tokens, int q_stride, const int32_t* __restrict__ kv_len,
                            int kv_base, int q_len, int max_len, int V, int half_hd, float rope_base,
                            int32_t* __restrict__ pos, int32_t* __restrict__ tok, float2* __restrict__ rope,
                            int32_t* __restrict__ status, int B, uint4* __restrict__ clear, size_t clear16, AttnParts ap) {
    const int jblocks = (q_len + PREP_ROWS - 1) / PREP_ROWS;
    if ((int)blockIdx.x >= B * jblocks) {             // the blocks behind the sequences zero the exchange cells
        const size_t nb = gridDim.x - B * jblocks;
        for (size_t i = (size_t)(blockIdx.x - B * jblocks) * blockDim.x + threadIdx.x; i < clear16; i += nb * blockDim.x)
            clear[i] = make_uint4(0u, 0u, 0u, 0u);
        return;
    }
    const int b = blockIdx.x / jblocks, j0 = (blockIdx.x - b * jblocks) * PREP_ROWS, j1 = min(q_len, j0 + PREP_ROWS);
    const int kvl = (kv_len ? kv_len[b] : 0) + kv_base;
    const bool ok = kvl >= 0 && kvl + q_len <= max_len;
    if (!ok && threadIdx.x == 0 && j0 == 0) atomicOr(status, 1);
    if (ap.parts && j0 == 0 && threadIdx.x < 64) attn_deal(ap, kv_len, kv_base, q_len, max_len, B, b, ok ? kvl : -1);
    for (int j = j0 + threadIdx.x; j < j1; j += blockDim.x) {
        const int m = b * q_len + j;
        int t = q_tokens[(size_t)b * q_stride + j];
        if (t < 0 || t >= V) { t = 0; atomicOr(status, 2); }
        tok[m] = t;
        pos[m] = ok ? kvl + j : -1;
    }
    for (int idx = j0 * half_hd + threadIdx.x; idx < j1 * half_hd; idx += blockDim.x) {
        const int j = idx / half_hd, i = idx % half_hd;
        const double inv_freq = pow((double)rope_base, -(double)i / (double)half_hd);   // base^(-2i/hd)
        const double ang = (double)(ok ? kvl + j : 0) * inv_freq;
        double s, c;
        sincos(ang, &s, &c);
        rope[(size_t)(b * q_len + j) * half_hd + i] = make_float2((float)c, (float)s);
    }
}

// ---- embedding ----------------------------------------------------------------------------------
template <typename T>
__global__ void embed_kernel(const int32_t* __restrict__ tok, const T* __restrict__ embed, int d, float* __restrict__ x) {
    const int m = blockIdx.x;
    const T* row = embed + (size_t)tok[m] * d;
    for (int i = threadIdx.x; i < d; i += blockDim.x) x[(size_t)m * d + i] = to_f(row[i]);
}

// ---- activation format ---------------------------------------------------------------------------
// fp32 models keep activations as float [M, K].  bf16 models keep them as TWO bf16 planes hi, lo with
// hi = bf16(v), lo = bf16(v - hi): the MFMA GEMM multiplies the weight tile with both planes, so the
// activations enter the contraction with ~16 significant bits while the weights stream as bf16.  The
// matrix cores have a 20x surplus over the weight bandwidth at these row counts, so the second plane is free.
template <typename T> struct Act;
template <> struct Act<float> {
    static __device__ __forceinline__ void store(void* base, size_t plane, size_t idx, float v) {
        reinterpret_cast<float*>(base)[idx] = v;
    }
};
template <> struct Act<uint16_t> {
    static __device__ __forceinline__ void store(void* base, size_t plane, size_t idx, float v) {
        const uint16_t hi = from_f<uint16_t>(v);
        const uint16_t lo = from_f<uint16_t>(v - to_f(hi));
        reinterpret_cast<uint16_t*>(base)[idx] = hi;
        reinterpret_cast<uint16_t*>(base)[plane + idx] = lo;
    }
};

// Embedding for the fused small-batch schedule: x (fp32), the planes of gain .* x (the next projection's
// input; its epilogue applies the row's RMS scale, the projection being linear) and the row's sum of squares.
__global__ __launch_bounds__(256) void embed_dec_kernel(const int32_t* __restrict__ tok, const uint16_t* __restrict__ embed,
                                                        const float* __restrict__ gain, int d, float* __restrict__ x,
                                                        uint16_t* __restrict__ planes, size_t plane, float* __restrict__ ssq) {
    __shared__ float red[4];
    const int m = blockIdx.x;
    const uint16_t* row = embed + (size_t)tok[m] * d;
    float ss = 0.f;
    for (int i = threadIdx.x; i < d; i += 256) {
        const float v = to_f(row[i]);
        x[(size_t)m * d + i] = v;
        Act<uint16_t>::store(planes, plane, (size_t)m * d + i, v * gain[i]);
        ss += v * v;
    }
    ss = wsum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) ssq[m] = red[0] + red[1] + red[2] + red[3];
}

// ---- RMSNorm (+ pending split-K partials of the previous projection) -----------------------------
// out row r takes input row src = (r / rows_out) * rows_in + (rows_in - rows_out) + r % rows_out
// (rows_out = rows_in: identity; rows_out < rows_in: the trailing rows of every sequence).
// If pend != null the residual row is first completed: x[src] += sum_s pend[s][src][:], and written back.
template <typename T>
__global__ __launch_bounds__(1024) void rmsnorm_kernel(float* __restrict__ x, const float* __restrict__ pend, int pend_ks,
                                                       size_t pend_stride, const float* __restrict__ gain, int d,
                                                       float eps, int rows_in, int rows_out, size_t plane,
                                                       void* __restrict__ out, int tiled) {
    __shared__ float red[16];
    const int r = blockIdx.x;
    const int src = (r / rows_out) * rows_in + (rows_in - rows_out) + r % rows_out;
    float* row = x + (size_t)src * d;
    const float* prow = pend ? pend + (size_t)src * d : nullptr;
    float ss = 0.f;
    // d % 8 == 0 (host check): float4 granules; the split-K partials are independent loads
    for (int i = threadIdx.x * 4; i < d; i += 4096) {
        float4 v = *reinterpret_cast<const float4*>(row + i);
        if (prow) {
            for (int s0 = 0; s0 < pend_ks; s0 += 4) {
                float4 p[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    p[u] = (s0 + u < pend_ks) ? *reinterpret_cast<const float4*>(prow + (size_t)(s0 + u) * pend_stride + i)
                                              : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int u = 0; u < 4; ++u) { v.x += p[u].x; v.y += p[u].y; v.z += p[u].z; v.w += p[u].w; }
            }
            *reinterpret_cast<float4*>(row + i) = v;
        }
        ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
    ss = wsum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) tot += red[w];
    const float scale = 1.0f / sqrtf(tot / (float)d + eps);
    for (int i = threadIdx.x * 4; i < d; i += 4096) {
        const float4 v = *reinterpret_cast<const float4*>(row + i);        // own earlier write, or the input
        const float4 g = *reinterpret_cast<const float4*>(gain + i);
        const size_t idx = tiled ? xt_index(r, i, tiled) : (size_t)r * d + i;        // four columns side by side in either layout
        Act<T>::store(out, plane, idx, v.x * scale * g.x);
        Act<T>::store(out, plane, idx + 1, v.y * scale * g.y);
        Act<T>::store(out, plane, idx + 2, v.z * scale * g.z);
        Act<T>::store(out, plane, idx + 3, v.w * scale * g.w);
    }
}

// ---- residual completion for bf16 models (the 16-row and many-row schedules) ---------------------------
// RMSNorm commutes with the projection that follows it (norm(x) W^T = r * ((gain .* x) W^T), r per row), so the
// row-wide reduction does not have to finish before the projection starts: this kernel only completes the residual
// (x += sum of the pending split-K partials), writes the planes of gain .* x and ONE partial sum of squares per
// 1024-column chunk; the projection's consumer (rope_kv, swiglu) multiplies by r.  grid (rows, ceil(d/1024)):
// every row is spread over several compute units instead of one.
// AHEAD: splits in flight at a time.  They were written by other dies a moment ago, so every turn of the loop is a trip to memory.
template <int AHEAD>
__global__ __launch_bounds__(256) void resid_sum_kernel(float* __restrict__ x, const float* __restrict__ pend, int pend_ks,
                                                        size_t pend_stride, const float* __restrict__ gain, int d, size_t plane,
                                                        uint16_t* __restrict__ out, float* __restrict__ ssq, int tiled) {
    __shared__ float red[4];
    const int r = blockIdx.x, chunk = blockIdx.y, nchunks = gridDim.y;
    const int i = chunk * 1024 + threadIdx.x * 4;                 // d % 8 == 0 (host check): whole float4 granules
    float ss = 0.f;
    if (i < d) {
        float* row = x + (size_t)r * d + i;
        float4 v = *reinterpret_cast<const float4*>(row);
        const float4 g = *reinterpret_cast<const float4*>(gain + i);
        if (pend) {
            const float* prow = pend + (size_t)r * d + i;
            for (int s0 = 0; s0 < pend_ks; s0 += AHEAD) {
                float4 p[AHEAD];
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    p[u] = *reinterpret_cast<const float4*>(prow + (size_t)min(s0 + u, pend_ks - 1) * pend_stride);
                    if (s0 + u >= pend_ks) p[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) { v.x += p[u].x; v.y += p[u].y; v.z += p[u].z; v.w += p[u].w; }
            }
            *reinterpret_cast<float4*>(row) = v;
        }
        ss = v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        store_planes4(out, plane, tiled ? xt_index(r, i, tiled) : (size_t)r * d + i, v.x * g.x, v.y * g.y, v.z * g.z, v.w * g.w);
    }
    ss = wsum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) ssq[(size_t)r * nchunks + chunk] = red[0] + red[1] + red[2] + red[3];
}

// ---- SwiGLU over split-K partials: act = silu(sum_s g) * sum_s u, columns [0,ff) gate, [ff,2ff) up ------
template <typename T>
__global__ void swiglu_kernel(const float* __restrict__ part, int ks, size_t ks_stride, int M, int ff, size_t plane,
                              void* __restrict__ out, int tiled, const float* __restrict__ ssq, int nchunks, float inv_d, float eps) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)M * ff) return;
    const size_t m = idx / ff, j = idx % ff;
    float g = 0.f, u = 0.f;
    for (int s = 0; s < ks; ++s) {
        g += part[(size_t)s * ks_stride + m * 2 * ff + j];
        u += part[(size_t)s * ks_stride + m * 2 * ff + ff + j];
    }
    const float rs = row_rscale(ssq, nchunks, (int)m, inv_d, eps);     // the input rows' RMS scale, if it was deferred
    g *= rs; u *= rs;
    Act<T>::store(out, plane, tiled ? xt_index((int)m, (int)j, tiled) : idx, g / (1.0f + __expf(-g)) * u);
}

// ---- GEMM, bf16 weights streamed through MFMA -------------------------------------------------------
// part[ks][m][n] = sum over the K range of split ks of x[m][k] * W[n][k].
// grid (ceil(N/64), KS), 4 wavefronts; wavefront w owns weight rows n0+16w .. n0+16w+15 (MFMA A operand:
// lane = (row l%16, k-slot l/16), one 16-byte load per 32-wide k slice, straight from HBM into registers,
// a whole stage of KC columns in flight per wavefront plus the next stage prefetched).  The activation
// slice [M, KC] of both planes is staged once per workgroup in LDS (rows padded by 16 bytes so that the
// 16 rows read by one ds_read_b128 phase fall into distinct banks) and shared by the four wavefronts.
// Each wavefront owns its output rows, so no cross-wavefront reduction is needed; split-K partials are
// summed by the consumer kernel.  Three kernels by row count: gemm_bf16_m16_kernel (up to 16 rows: pure weight
// streaming; the layers of a wide model take gemm_rows_kernel instead), this one with two row tiles (17..32 rows, and the
// fallback when K is not a multiple of 32), gemm_bf16_big_kernel from 33 rows on (measured faster from there).

// Column offset of a k slice that starts at k, clamped into the row for the lane whose pointer already sits at k-slot lq
// (tiled: K % 32 == 0, whole slices; row-major: K % 8 == 0, the lane's 8-column chunk must end inside the row).
template <bool TILED>
__device__ __forceinline__ int wclamp(int k, int K, int lq) {
    if (TILED) return min(k, K - 32);
    return max(min(k, K - 8 - lq * 8), -lq * 8);
}

// dst (tiled, rows padded to a multiple of 64 with zeros) <- src (row-major [N][K]); one 16-byte chunk per lane.
__global__ void pack_weights_kernel(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, int N, int K) {
    const size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t per_block = (size_t)(K / 32) * 256;                  // chunks per 64-row block
    const size_t nblocks = (size_t)((N + 63) / 64);
    if (c >= nblocks * per_block) return;
    const int nb = (int)(c / per_block);
    const size_t rem = c % per_block;
    const int step = (int)(rem / 256), in = (int)(rem % 256);
    const int t = in >> 6, lane = in & 63;
    const int n = nb * 64 + t * 16 + (lane & 15), k = step * 32 + (lane >> 4) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (n < N) v = ldg16(src + (size_t)n * K + k);
    *reinterpret_cast<uint4*>(dst + c * 8) = v;
}

template <int MT, int NT, int KC, bool TILED>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmArgs a) {
    constexpr int ROW = KC + 8;                       // padded LDS row (bf16 elements)
    constexpr int NSL = KC / 32;                      // k slices per stage
    __shared__ __attribute__((aligned(16))) uint16_t xs[2][MT * 16][ROW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lq = lane >> 4;
    const int n0 = blockIdx.x * (64 * NT) + wave * (16 * NT);    // this wavefront: NT tiles of 16 weight rows
    const uint16_t* wrow[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        int n = n0 + u * 16 + li;
        if (n >= a.N) n = a.N - 1;
        int seg = 0, local = n;
        if (local >= a.seg_rows[0]) { local -= a.seg_rows[0]; seg = 1; if (local >= a.seg_rows[1]) { local -= a.seg_rows[1]; seg = 2; } }
        wrow[u] = wlane_ptr<TILED>(reinterpret_cast<const uint16_t*>(a.w[seg]), local, a.K, lq);
    }
    const uint16_t* xh = reinterpret_cast<const uint16_t*>(a.x);
    const uint16_t* xl = xh + a.x_plane;
    // stages of this split
    const int nstages = (a.K + KC - 1) / KC;
    const int ks = blockIdx.y, KS = gridDim.y;
    const int st_begin = (int)((long long)nstages * ks / KS), st_end = (int)((long long)nstages * (ks + 1) / KS);

    f32x4 acc[NT][MT];
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[u][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    uint4 wcur[NT][NSL], wnext[NT][NSL];
    auto load_stage = [&](int st, uint4 (&dst)[NT][NSL]) {
        const int kb = st * KC;                       // wrow already points at this lane's k-slot
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int j = 0; j < NSL; ++j) {
                // unconditional and clamped (a select on the loaded value would make the wavefront wait for it right here):
                // columns past K re-read the row's last chunk and meet zero activations, stages past the end are never used
                const int k = wclamp<TILED>(kb + j * 32, a.K, lq);
                dst[u][j] = ldg16(wrow[u] + (size_t)k * (WSTEP<TILED>::v / 32));
            }
    };
    // Activation slice of a stage: 16-byte chunks, rows >= M and columns >= K are zero.  It is requested into registers
    // one stage ahead (behind the weight prefetch) and written to LDS after the MFMAs of the current stage, so the trip
    // to memory hides behind them.
    constexpr int CHUNKS = 2 * MT * 16 * (KC / 8);
    constexpr int XPT = (CHUNKS + 255) / 256;         // chunks per lane
    uint4 xr[XPT];
    auto load_x = [&](int st) {
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int c = threadIdx.x + i * 256;
            const int plane = c / (MT * 16 * (KC / 8));
            const int rem = c % (MT * 16 * (KC / 8));
            const int m = rem / (KC / 8), kc = (rem % (KC / 8)) * 8;
            const int k = st * KC + kc;
            const bool ok = c < CHUNKS && st < st_end && m < a.M && k < a.K;
            const uint4 v = ldg16((plane ? xl : xh) + (ok ? (size_t)m * a.K + k : 0));       // always a valid address
            xr[i] = ok ? v : make_uint4(0, 0, 0, 0);
        }
    };
    auto store_x = [&]() {
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int c = threadIdx.x + i * 256;
            if (c < CHUNKS) {
                const int plane = c / (MT * 16 * (KC / 8));
                const int rem = c % (MT * 16 * (KC / 8));
                *reinterpret_cast<uint4*>(&xs[plane][rem / (KC / 8)][(rem % (KC / 8)) * 8]) = xr[i];
            }
        }
    };
    load_stage(st_begin, wcur);
    load_x(st_begin);
    store_x();
    __syncthreads();
    for (int st = st_begin; st < st_end; ++st) {
        load_stage(st + 1, wnext);                    // prefetch (all zero past the end)
        load_x(st + 1);
#pragma unroll
        for (int j = 0; j < NSL; ++j) {
#pragma unroll
            for (int t = 0; t < MT; ++t) {            // one pair of activation operands serves the NT weight tiles
                const bf16x8 bh = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&xs[0][t * 16 + li][j * 32 + lq * 8]));
                const bf16x8 bl = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&xs[1][t * 16 + li][j * 32 + lq * 8]));
#pragma unroll
                for (int u = 0; u < NT; ++u) {
                    const bf16x8 A = __builtin_bit_cast(bf16x8, wcur[u][j]);
                    acc[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, bh, acc[u][t], 0, 0, 0);
                    acc[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, bl, acc[u][t], 0, 0, 0);
                }
            }
        }
        __syncthreads();                              // every wavefront is done reading this stage's slice
        store_x();
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int j = 0; j < NSL; ++j) wcur[u][j] = wnext[u][j];
    }
    // D[n = n0 + 16u + 4*lq + e][m = 16t + li]: four consecutive n per lane -> one 16-byte store
    float* out = reinterpret_cast<float*>(a.out) + (size_t)ks * a.ks_stride;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        const int nb = n0 + u * 16 + 4 * lq;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const int m = t * 16 + li;
            if (m >= a.M) continue;
            float* o = out + (size_t)m * a.ldo + nb;
            if (nb + 3 < a.N && (reinterpret_cast<uintptr_t>(o) & 15) == 0) {
                *reinterpret_cast<float4*>(o) = make_float4(acc[u][t][0], acc[u][t][1], acc[u][t][2], acc[u][t][3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (nb + e < a.N) o[e] = acc[u][t][e];
            }
        }
    }
}

// ---- GEMM for at most 16 activation rows (LM heads; the layers of models too narrow for gemm_rows_kernel) ----
// Same operand mapping as above, but the whole K range of the workgroup (at most M16_KMAX columns) is
// staged in LDS once, behind the first weight loads, and the loop over 32-wide k slices then runs without
// barriers: each wavefront keeps a ring of M16_DEPTH weight loads (16 rows x 64 bytes each) in flight and
// retires them in order against the in-order memory counter.
constexpr int M16_KMAX = 512;
constexpr int M16_DEPTH = 8;

template <int NT, bool TILED>
__global__ __launch_bounds__(256) void gemm_bf16_m16_kernel(GemmArgs a, int kper) {
    constexpr int ROW = M16_KMAX + 8;
    __shared__ __attribute__((aligned(16))) uint16_t xs[2][16][ROW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lq = lane >> 4;
    const int n0 = blockIdx.x * (64 * NT) + wave * (16 * NT);      // this wavefront: NT tiles of 16 weight rows
    const int ks = blockIdx.y;
    const int k_lo = ks * kper, k_hi = min(a.K, k_lo + kper);       // this workgroup's columns
    const uint16_t* wrow[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        int n = n0 + t * 16 + li;
        if (n >= a.N) n = a.N - 1;
        int seg = 0, local = n;
        if (local >= a.seg_rows[0]) { local -= a.seg_rows[0]; seg = 1; if (local >= a.seg_rows[1]) { local -= a.seg_rows[1]; seg = 2; } }
        wrow[t] = wlane_ptr<TILED>(reinterpret_cast<const uint16_t*>(a.w[seg]), local, a.K, lq);
    }
    const uint16_t* xh = reinterpret_cast<const uint16_t*>(a.x);
    const uint16_t* xl = xh + a.x_plane;
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // phases of at most M16_KMAX columns (one phase unless the caller asked for few splits)
    for (int k_begin = k_lo; k_begin < k_hi; k_begin += M16_KMAX) {
        const int k_end = min(k_hi, k_begin + M16_KMAX);
        const int nsl = (k_end - k_begin + 31) / 32;
        // Unconditional loads (a branch around a load would force the compiler to wait for every outstanding
        // load instead of counting them): slices past the end re-read the last valid 16-byte chunk of the row,
        // which meets zero activations in LDS.
        const int k_last = k_end - 8 - lq * 8;             // last valid chunk start for this lane's k-slot
        auto wload = [&](int t, int j) {
            if (TILED) return ldg16(wrow[t] + (size_t)min(k_begin + j * 32, k_end - 32) * 64);   // K % 32 == 0
            const int k = max(min(k_begin + j * 32, k_last), -lq * 8);   // wrow already points at column lq*8
            return ldg16(wrow[t] + k);
        };
        // Activation slice [16][k_begin..k_end) of both planes: requested first (L2 hits), the weight ring
        // right behind it, so that the LDS fill waits for the slice only (the memory counter retires in order).
        // 2 planes x 16 rows x 64 chunks of 16 bytes = 8 chunks per lane; rows >= M and the tail are zero.
        constexpr int XCH = 2 * 16 * (M16_KMAX / 8) / 256;      // fixed geometry: chunk c -> (plane, row, column) by shifts
        static_assert(M16_KMAX == 512, "chunk decoding below assumes 64 chunks per row");
        uint4 xv[XCH];
#pragma unroll
        for (int u = 0; u < XCH; ++u) {
            const int c = threadIdx.x + u * 256;
            const int plane = c >> 10, m = (c >> 6) & 15, kc = (c & 63) * 8;
            const bool ok = m < a.M && k_begin + kc < k_end;
            const uint16_t* src = (plane ? xl : xh) + (ok ? (size_t)m * a.K + k_begin + kc : 0);   // always a valid address
            xv[u] = ldg16(src);
            const uint32_t keep = ok ? 0xFFFFFFFFu : 0u;
            xv[u].x &= keep; xv[u].y &= keep; xv[u].z &= keep; xv[u].w &= keep;
        }
        uint4 w[NT][M16_DEPTH];
#pragma unroll
        for (int u = 0; u < M16_DEPTH; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t) w[t][u] = wload(t, u);
        if (k_begin != k_lo) __syncthreads();              // the previous phase's LDS reads are done
#pragma unroll
        for (int u = 0; u < XCH; ++u) {
            const int c = threadIdx.x + u * 256;
            *reinterpret_cast<uint4*>(&xs[c >> 10][(c >> 6) & 15][(c & 63) * 8]) = xv[u];
        }
        __syncthreads();
        // M16_DEPTH slices; `more` further ones are behind them: their weights are asked for as these are used up, and the last group
        // asks for nothing (slices of 256 columns, as the layers of a narrow model have, asked for every weight twice)
        auto group = [&](int j0, bool more) {
#pragma unroll
            for (int u = 0; u < M16_DEPTH; ++u) {
                bf16x8 A[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    A[t] = __builtin_bit_cast(bf16x8, w[t][u]);
                    if (more) w[t][u] = wload(t, j0 + M16_DEPTH + u);
                }
                const int j = j0 + u;
                if (more || j < nsl) {
                    const bf16x8 bh = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&xs[0][li][j * 32 + lq * 8]));
                    const bf16x8 bl = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&xs[1][li][j * 32 + lq * 8]));
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[t], bh, acc[t], 0, 0, 0);
                        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[t], bl, acc[t], 0, 0, 0);
                    }
                }
            }
        };
        int j0 = 0;
        for (; j0 + M16_DEPTH < nsl; j0 += M16_DEPTH) group(j0, true);
        group(j0, false);
    }
    float* out = a.out + (size_t)ks * a.ks_stride;
    if (li < a.M) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int nb = n0 + t * 16 + 4 * lq;
            float* o = out + (size_t)li * a.ldo + nb;
            if (nb + 3 < a.N && (reinterpret_cast<uintptr_t>(o) & 15) == 0) {
                *reinterpret_cast<float4*>(o) = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (nb + e < a.N) o[e] = acc[t][e];
            }
        }
    }
}

// ---- fused projections for very few rows (draft steps) ----------------------------------------------
// With one or two activation rows every kernel of a layer is a few microseconds of latency, so the layer
// time is the number of kernels.  Here a workgroup owns 16 output columns over the WHOLE K range: its
// wavefronts split K, add their accumulators through LDS, and wavefront 0 finishes the columns in place:
//   EPI_RESID   x += y; planes of gain_next .* x and the 16-column sums of squares for the next RMSNorm
//   EPI_QKV     RMS scale of the input rows, RoPE on q and k, q out (fp32), k and v into the cache
//   EPI_SWIGLU  gate and up tiles of the same columns side by side: silu(r g) * (r u) as planes
// so a layer is 4 projections + attention + merge instead of 10 kernels.  RMSNorm commutes with the
// projection: norm(x) W^T = r * ((gain .* x) W^T), r = rsqrt(mean(x^2) + eps) per row, so the producer of x
// writes gain .* x and partial sums of squares, and the consumer of the projection multiplies by r.
// The activations come straight from L2 (MFMA B operand: lane = (row l%16, k-slot l/16)); that costs twice
// the weight bytes in L1 traffic at 16 rows, which is why this path is for a handful of rows only.
// Weights are in the tiled layout.

template <int EPI, int DEPTH, bool MERGE>
__global__ __launch_bounds__(512) void gemm_dec_kernel(DecArgs a) {
    __shared__ __attribute__((aligned(16))) float red[8][256];
    extern __shared__ __attribute__((aligned(16))) uint16_t xs[];     // [2 planes][M][K + 8]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, W = blockDim.x >> 6;
    const int li = lane & 15, lq = lane >> 4;
    const int WS = EPI == EPI_SWIGLU ? W / 2 : W;                 // K splits per 16-column tile
    const int grp = wave / WS, split = wave - grp * WS;
    const int n0 = blockIdx.x * 16;
    const int c = n0 + 4 * lq;                                    // lane's four output columns (epilogue)
    const bool row_ok = li < a.M;
    const uint16_t* wmat;
    int local = n0 + li;
    if (EPI == EPI_SWIGLU) wmat = reinterpret_cast<const uint16_t*>(a.w[grp]);
    else {
        int seg = 0;
        if (a.w[1] && local >= a.seg_rows[0]) { local -= a.seg_rows[0]; seg = 1; if (a.w[2] && local >= a.seg_rows[1]) { local -= a.seg_rows[1]; seg = 2; } }
        wmat = reinterpret_cast<const uint16_t*>(a.w[seg]);
    }
    // Everything the epilogue needs from memory is requested now, ahead of the operand streams, so that it has
    // arrived long before wavefront 0 gets there: the rows' sums of squares, the residual and gain (RESID),
    // position and rotation (QKV).
    float ssr[DEC_MAX_ROWS];                                      // this lane's share of each row's sum of squares
#pragma unroll
    for (int m = 0; m < DEC_MAX_ROWS; ++m) ssr[m] = 0.f;
    float4 x_old = make_float4(0.f, 0.f, 0.f, 0.f), g_next = make_float4(0.f, 0.f, 0.f, 0.f);
    float2 rc0 = make_float2(1.f, 0.f), rc1 = make_float2(1.f, 0.f);
    int p_row = -1;
    const int hd_mask = a.hd - 1;                                 // head_dim is 64 or 128
    if (wave == 0) {
        const int m = min(li, a.M - 1);
        if (EPI != EPI_RESID) {
#pragma unroll
            for (int mm = 0; mm < DEC_MAX_ROWS; ++mm) {
                if (mm >= a.M) break;
                for (int t = lane; t < a.ssq_tiles; t += 256) {       // independent loads, four per lane in flight
                    float v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int tt = t + 64 * u;
                        v[u] = a.ssq_in[(size_t)mm * a.ssq_tiles + min(tt, a.ssq_tiles - 1)];
                        if (tt >= a.ssq_tiles) v[u] = 0.f;
                    }
                    ssr[mm] += (v[0] + v[1]) + (v[2] + v[3]);
                }
            }
        }
        if (EPI == EPI_RESID) {
            x_old = *reinterpret_cast<const float4*>(a.x + (size_t)m * a.N + c);
            if (a.gain_next) g_next = *reinterpret_cast<const float4*>(a.gain_next + c);
        }
        if (EPI == EPI_QKV) {
            p_row = a.pos[m];
            const int hc = c & hd_mask;
            rc0 = a.rope[(size_t)m * (a.hd / 2) + hc / 2];
            rc1 = a.rope[(size_t)m * (a.hd / 2) + hc / 2 + 1];
        }
    }
    // ---- activations: both planes of all M rows, whole K, into LDS (a few KB at these row counts) ----
    // First round of 16-byte chunks is requested BEFORE the weight prologue and stored after it, so that the
    // wait for it (the memory counter retires in order) leaves the weight loads in flight.
    const int row_e = a.K + 8;                                    // padded row, elements
    const int kc8 = a.K / 8;                                      // 16-byte chunks per row
    const int kc0 = threadIdx.x < (unsigned)kc8 ? (int)threadIdx.x : 0;       // lanes past the row re-read chunk 0 (not stored)
    uint4 xv0[2 * DEC_MAX_ROWS];
    if (!MERGE) {
#pragma unroll
        for (int pr = 0; pr < 2 * DEC_MAX_ROWS; ++pr) {           // pr = plane * M + row, clamped to the last valid pair
            const int q = min(pr, 2 * a.M - 1);
            const int plane = q >= a.M ? 1 : 0, m = q - plane * a.M;
            xv0[pr] = ldg16(a.xh + (size_t)plane * a.x_plane + (size_t)m * a.K + kc0 * 8);
        }
    }
    const int steps = a.K / 32;
    const int ws_shift = __ffs(WS) - 1;                           // WS is 4 or 8
    const int s_begin = (split * steps) >> ws_shift, s_end = ((split + 1) * steps) >> ws_shift;
    const int n = s_end - s_begin;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const char* wb = reinterpret_cast<const char*>(wmat);
    // byte offsets (every matrix is below 4 GiB: host check); a k step is 4096 bytes of the tiled weights
    uint32_t woff = (uint32_t)(((size_t)(local >> 6) * 64 * a.K + ((local >> 4) & 3) * 512 + ((local & 15) + 16 * lq) * 8 +
                                (size_t)s_begin * 2048) * 2);
    uint4 rw[DEPTH];
    {
        const int nn = max(n, 1) - 1;                             // n == 0: the wavefront re-reads step 0 of its tile and ignores it
        const uint32_t w0 = n > 0 ? woff : (uint32_t)(((size_t)(local >> 6) * 64 * a.K + ((local >> 4) & 3) * 512 + ((local & 15) + 16 * lq) * 8) * 2);
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) rw[u] = ldg16((const uint16_t*)(wb + w0 + min(u, nn) * 4096));   // clamped to the last step
    }
    if (!MERGE) {
#pragma unroll
        for (int pr = 0; pr < 2 * DEC_MAX_ROWS; ++pr)
            if (pr < 2 * a.M && threadIdx.x < (unsigned)kc8) *reinterpret_cast<uint4*>(&xs[pr * row_e + threadIdx.x * 8]) = xv0[pr];
        for (int pr = 0; pr < 2 * a.M; ++pr) {                    // rows longer than the workgroup (8 columns per lane): the rest
            const int plane = pr >= a.M ? 1 : 0, m = pr - plane * a.M;
            for (int kc = threadIdx.x + blockDim.x; kc < kc8; kc += blockDim.x)
                *reinterpret_cast<uint4*>(&xs[pr * row_e + kc * 8]) = ldg16(a.xh + (size_t)plane * a.x_plane + (size_t)m * a.K + kc * 8);
        }
    } else {
        // The activations are the attention output, still as per-split partials (o[hd], max, sum): each lane combines
        // the splits of eight head-dim elements (online over groups of 8 splits, all loads of a group in flight) and
        // writes both planes.  Every workgroup redoes this for the whole row: a few KB from L2, one kernel fewer.
        const size_t pstride = (size_t)a.hd + 4;
        const int hd_shift = __ffs(a.hd) - 1;
        for (int m = 0; m < a.M; ++m)
            for (int kc = threadIdx.x; kc < kc8; kc += blockDim.x) {
                const int col = kc * 8, h = col >> hd_shift, d0 = col & (a.hd - 1);
                const float* base = a.att_part + ((size_t)m * a.H + h) * a.att_splits * pstride;
                float mm = -INFINITY, lsum = 0.f, o[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = 0.f;
                for (int s0 = 0; s0 < a.att_splits; s0 += 8) {
                    float4 oa[8], ob[8];
                    float2 ml[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const float* ps = base + (size_t)min(s0 + u, a.att_splits - 1) * pstride;
                        oa[u] = *reinterpret_cast<const float4*>(ps + d0);
                        ob[u] = *reinterpret_cast<const float4*>(ps + d0 + 4);
                        ml[u] = *reinterpret_cast<const float2*>(ps + a.hd);
                        if (s0 + u >= a.att_splits) ml[u] = make_float2(-INFINITY, 0.f);
                    }
                    float gm = mm;
#pragma unroll
                    for (int u = 0; u < 8; ++u) gm = fmaxf(gm, ml[u].x);
                    if (gm == -INFINITY) continue;
                    const float keep = __expf(mm - gm);                  // 0 when nothing was accumulated yet
                    lsum *= keep;
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] *= keep;
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const float f = (ml[u].x == -INFINITY) ? 0.f : __expf(ml[u].x - gm);
                        if (f == 0.f) continue;                          // an empty split's o[] was never written
                        lsum += ml[u].y * f;
                        o[0] += oa[u].x * f; o[1] += oa[u].y * f; o[2] += oa[u].z * f; o[3] += oa[u].w * f;
                        o[4] += ob[u].x * f; o[5] += ob[u].y * f; o[6] += ob[u].z * f; o[7] += ob[u].w * f;
                    }
                    mm = gm;
                }
                const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
                uint32_t hw[4], lw[4];
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const float v0 = o[e] * inv, v1 = o[e + 1] * inv;
                    const uint16_t h0 = from_f<uint16_t>(v0), h1 = from_f<uint16_t>(v1);
                    hw[e / 2] = (uint32_t)h0 | ((uint32_t)h1 << 16);
                    lw[e / 2] = (uint32_t)from_f<uint16_t>(v0 - to_f(h0)) | ((uint32_t)from_f<uint16_t>(v1 - to_f(h1)) << 16);
                }
                *reinterpret_cast<uint4*>(&xs[(size_t)m * row_e + col]) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
                *reinterpret_cast<uint4*>(&xs[(size_t)(a.M + m) * row_e + col]) = make_uint4(lw[0], lw[1], lw[2], lw[3]);
            }
    }
    __syncthreads();                                              // activations are in LDS
    if (n > 0) {
        // MFMA B operand: lane (row l%16, k-slot l/16); rows >= M feed unused columns of D and read row M-1
        const uint16_t* bh = xs + (size_t)min(li, a.M - 1) * row_e + lq * 8 + s_begin * 32;
        const uint16_t* bl = bh + (size_t)a.M * row_e;
        int j = 0;
        // whole groups whose prefetches (steps j + DEPTH + u) are all inside the range: no clamps, no selects
        for (; j + 2 * DEPTH <= n; j += DEPTH) {
            woff += DEPTH * 4096;
            uint4 Bh[DEPTH], Bl[DEPTH];                           // the group's B operands, all LDS reads in flight together
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                Bh[u] = *reinterpret_cast<const uint4*>(bh + (j + u) * 32);
                Bl[u] = *reinterpret_cast<const uint4*>(bl + (j + u) * 32);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                const bf16x8 A = __builtin_bit_cast(bf16x8, rw[u]);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, Bh[u]), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, Bl[u]), acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);                // keep the refill behind its MFMAs: same registers, no copies
                rw[u] = ldg16((const uint16_t*)(wb + woff + u * 4096));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // last groups: prefetches clamped to the last step, steps past the end meet zero weights
        for (; j < n; j += DEPTH) {
            woff += DEPTH * 4096;
            uint4 Bh[DEPTH], Bl[DEPTH];
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                const int sj = min(j + u, n - 1);
                Bh[u] = *reinterpret_cast<const uint4*>(bh + sj * 32);
                Bl[u] = *reinterpret_cast<const uint4*>(bl + sj * 32);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                uint4 wv = rw[u];
                if (j + u >= n) wv = make_uint4(0u, 0u, 0u, 0u);
                const bf16x8 A = __builtin_bit_cast(bf16x8, wv);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, Bh[u]), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, Bl[u]), acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                const int st = u - max(j + DEPTH + u - (n - 1), 0);      // relative to woff; negative = back inside the range
                rw[u] = ldg16((const uint16_t*)(wb + woff + st * 4096));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    *reinterpret_cast<f32x4*>(&red[wave][lane * 4]) = acc;
    __syncthreads();
    if (wave != 0) return;
    // lane holds D[column n0 + 4*lq + e][row li]
    f32x4 t = {0.f, 0.f, 0.f, 0.f}, t2 = {0.f, 0.f, 0.f, 0.f};
    for (int v = 0; v < WS; ++v) {
        const f32x4 p = *reinterpret_cast<const f32x4*>(&red[v][lane * 4]);
        t[0] += p[0]; t[1] += p[1]; t[2] += p[2]; t[3] += p[3];
    }
    if (EPI == EPI_SWIGLU)
        for (int v = WS; v < 2 * WS; ++v) {
            const f32x4 p = *reinterpret_cast<const f32x4*>(&red[v][lane * 4]);
            t2[0] += p[0]; t2[1] += p[1]; t2[2] += p[2]; t2[3] += p[3];
        }
    float rscale = 1.f;
    if (EPI != EPI_RESID) {      // r = rsqrt(mean square + eps) of the lane's input row
        float mine = 0.f;
#pragma unroll
        for (int mm = 0; mm < DEC_MAX_ROWS; ++mm) {
            const float tot = wsum(ssr[mm]);
            if (li == mm) mine = tot;
        }
        rscale = 1.0f / sqrtf(mine / (float)a.K + a.eps);
    }
    if (EPI == EPI_RESID) {
        float ss = 0.f;
        if (row_ok) {
            float* xp = a.x + (size_t)li * a.N + c;
            float4 xv = x_old;
            xv.x += t[0]; xv.y += t[1]; xv.z += t[2]; xv.w += t[3];
            *reinterpret_cast<float4*>(xp) = xv;
            ss = xv.x * xv.x + xv.y * xv.y + xv.z * xv.z + xv.w * xv.w;
            if (a.gain_next) {
                const float4 g = g_next;
                store_planes4(a.out_planes, a.out_plane, (size_t)li * a.N + c, xv.x * g.x, xv.y * g.y, xv.z * g.z, xv.w * g.w);
            }
        }
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (row_ok && lq == 0 && a.ssq_out) a.ssq_out[(size_t)li * (a.N / 16) + blockIdx.x] = ss;
    } else if (EPI == EPI_SWIGLU) {
        if (row_ok) {
            float h[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float g = t[e] * rscale, u = t2[e] * rscale;
                h[e] = g / (1.0f + __expf(-g)) * u;
            }
            store_planes4(a.out_planes, a.out_plane, (size_t)li * a.N + c, h[0], h[1], h[2], h[3]);
        }
    } else {
        if (row_ok) {
            const int nq = a.H * a.hd, nkv = a.KVH * a.hd;
            const int p = p_row, b = li / a.q_len;
            float v[4] = {t[0] * rscale, t[1] * rscale, t[2] * rscale, t[3] * rscale};
            if (c < nq + nkv) {
                const int hc = c & hd_mask;
                const float2 c0 = rc0, c1 = rc1;
                const float r0 = v[0] * c0.x - v[1] * c0.y, r1 = v[0] * c0.y + v[1] * c0.x;
                const float r2 = v[2] * c1.x - v[3] * c1.y, r3 = v[2] * c1.y + v[3] * c1.x;
                if (c < nq) {
                    *reinterpret_cast<float4*>(a.q_out + (size_t)li * nq + c) = make_float4(r0, r1, r2, r3);
                } else if (p >= 0) {
                    const int kh = (c - nq) >> (__ffs(a.hd) - 1);
                    uint16_t* dst = a.k_cache + (((size_t)b * a.KVH + kh) * a.cache_len + p) * a.hd + hc;
                    *reinterpret_cast<uint2*>(dst) = make_uint2((uint32_t)from_f<uint16_t>(r0) | ((uint32_t)from_f<uint16_t>(r1) << 16),
                                                                (uint32_t)from_f<uint16_t>(r2) | ((uint32_t)from_f<uint16_t>(r3) << 16));
                }
            } else if (p >= 0) {
                const int cv = c - nq - nkv;
                const int vh = cv >> (__ffs(a.hd) - 1), hc = cv & hd_mask;
                uint16_t* base = a.v_cache + ((size_t)b * a.KVH + vh) * (size_t)a.cache_len * a.hd;
#pragma unroll
                for (int e = 0; e < 4; ++e) base[v_index<uint16_t>(p, hc + e, a.hd)] = from_f<uint16_t>(v[e]);
            }
        }
    }
}

// ---- fused projections for a few more rows of a wide model (verification of one to a few sequences) -----------------
// Between 3 and 32 rows the activations are too many to stage whole in every 16-column workgroup, and the 16-row
// kernel above needs a consumer kernel per projection for its split-K partial sums.  On a wide model (about as many
// 16-column units per projection as compute units, or more) there is a third way: one workgroup per compute unit
// owns up to ROWS_UMAX consecutive units over the WHOLE K range, its 8 wavefronts split K, every wavefront streams
// its k steps of all the units and loads the matching activations straight into the MFMA B operand (rows < M only;
// each k slice is read by one wavefront, so LDS would buy nothing, and the B registers are shared by the units),
// the accumulators meet in LDS and wavefront v finishes unit v with the consumer's work: RMS scale + RoPE + q out +
// K/V cache write (EPI_QKV), silu(r g) * (r u) as planes (EPI_SWIGLU, a unit being the gate and the up tile of the
// same 16 columns), residual add + planes of gain_next .* x + the unit's sums of squares (EPI_RESID).  No partial
// sums, no consumer kernel.  The activation planes are tiled (xt_index): with the rows of a k step in 16 different
// cache lines a projection with ONE unit per workgroup (O, down), whose activations are as many bytes as its
// weights, ran a third slower (down projection, 9 rows: 27 against 21 us).
// MT = 2 row tiles serve 17..32 rows: every weight tile meets two B operands, twice the activation loads.
// STREAM: weights as non-temporal loads (7B layer, 9 rows: QKV 22.6 -> 21.7, gate/up 35.0 -> 33.9 us; 20 rows: 26.6 -> 24.6,
// 37.8 -> 36.1).  The LM head's 16-row kernel gained nothing from them.
constexpr int ROWS_UMAX = 4;
constexpr int rows_depth(int nt) { return nt <= 4 ? 4 : 2; }   // k steps in flight per wavefront (3 measured a third slower than 2 or 4)

template <int EPI, int NU, int MT, bool STREAM>
__device__ __forceinline__ void rows_body(const DecArgs& a, const int u0, float* __restrict__ red) {
    constexpr int PER = EPI == EPI_SWIGLU ? 2 : 1, NT = NU * PER, DEPTH = rows_depth(NT);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lq = lane >> 4;
    constexpr int R = 16 * MT;                                     // rows of the tiled planes
    static_assert(NU * MT <= 8, "one wavefront per unit and row tile finishes them");
    // wavefront v finishes unit v % NU of row tile v / NU: row m, if it exists
    const bool fin = wave < NU * MT;
    const int unit = fin ? wave % NU : 0, mrow = 16 * (fin ? wave / NU : 0) + li;
    const bool row_ok = mrow < a.M;
    const int m = min(mrow, a.M - 1);
    bool load_ok[MT];                                              // this lane's rows of the B operands
    int lm[MT];
#pragma unroll
    for (int x = 0; x < MT; ++x) { load_ok[x] = 16 * x + li < a.M; lm[x] = min(16 * x + li, a.M - 1); }
    // what the epilogue needs from memory is requested ahead of the operand streams
    const int c = (u0 + unit) * 16 + 4 * lq;                       // the lane's four output columns there
    const int hd_mask = a.hd - 1;
    float2 rc0 = make_float2(1.f, 0.f), rc1 = make_float2(1.f, 0.f);
    float4 x_old = make_float4(0.f, 0.f, 0.f, 0.f), g_next = make_float4(0.f, 0.f, 0.f, 0.f);
    int p_row = -1;
    if (fin) {
        if (EPI == EPI_QKV) {
            p_row = a.pos[m];
            const int hc = c & hd_mask;
            rc0 = a.rope[(size_t)m * (a.hd / 2) + hc / 2];
            rc1 = a.rope[(size_t)m * (a.hd / 2) + hc / 2 + 1];
        }
        if (EPI == EPI_RESID) {
            x_old = *reinterpret_cast<const float4*>(a.x + (size_t)m * a.N + c);
            if (a.gain_next) g_next = *reinterpret_cast<const float4*>(a.gain_next + c);
        }
    }
    // The input rows' sums of squares come in ssq_tiles pieces per row (4 from the residual kernel, K/16 from an
    // EPI_RESID projection): the lanes (row li, lq) of all wavefronts share the pieces, 8 independent loads each
    // (256 pieces), added up behind the operand streams and combined through LDS with the accumulators.
    float sv[MT][8];
    if (EPI != EPI_RESID) {
#pragma unroll
        for (int x = 0; x < MT; ++x)
#pragma unroll
            for (int i = 0; i < 8; ++i) sv[x][i] = a.ssq_in[(size_t)lm[x] * a.ssq_tiles + min(wave * 4 + lq + 32 * i, a.ssq_tiles - 1)];
    }
    const int steps = a.K / 32;
    const int s_begin = (wave * steps) >> 3, s_end = ((wave + 1) * steps) >> 3;
    const int n = s_end - s_begin, nn = max(n, 1) - 1;
    const int sb = n > 0 ? s_begin : 0;                            // a wavefront without k steps re-reads step 0 and ignores it
    const char* wp[NT];                                            // the wavefront's first k step of every tile (uniform)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        int local = (u0 + t / PER) * 16;
        const void* mat;
        if (EPI == EPI_SWIGLU) mat = a.w[t % PER];
        else {
            int seg = 0;
            if (a.w[1] && local >= a.seg_rows[0]) { local -= a.seg_rows[0]; seg = 1; if (a.w[2] && local >= a.seg_rows[1]) { local -= a.seg_rows[1]; seg = 2; } }
            mat = a.w[seg];
        }
        wp[t] = reinterpret_cast<const char*>(mat) + ((size_t)(local >> 6) * 64 * a.K + ((local >> 4) & 3) * 512 + (size_t)sb * 2048) * 2;
    }
    const uint32_t loff = lane * 16;                               // a k step of a tile is one contiguous kilobyte, 16 bytes per lane
    const uint16_t* bh = a.xh + (size_t)sb * (R * 32) + (MT == 2 ? (li >> 2) * 128 + lq * 32 + (li & 3) * 8 : li * 32 + lq * 8);   // tiled planes (xt_index): a k step is 32 R elements
    const uint16_t* bl = bh + a.x_plane;
    f32x4 acc[NT][MT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int x = 0; x < MT; ++x) acc[t][x] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint4 rw[DEPTH][NT], Bh[DEPTH][MT], Bl[DEPTH][MT];
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
        const int sj = min(u, nn);
#pragma unroll
        for (int x = 0; x < MT; ++x) {
            Bh[u][x] = make_uint4(0u, 0u, 0u, 0u); Bl[u][x] = make_uint4(0u, 0u, 0u, 0u);
            if (load_ok[x]) { Bh[u][x] = ldg16(bh + sj * (R * 32) + x * 512); Bl[u][x] = ldg16(bl + sj * (R * 32) + x * 512); }    // rows >= M stay zero
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) rw[u][t] = ldg16_stream<STREAM>(reinterpret_cast<const uint16_t*>(wp[t] + loff + sj * 4096));
    }
    // DEPTH steps; `more` further ones are behind them: their operands are asked for as these are used up.  The last group asks for
    // nothing: clamped requests there were a quarter of the O projection's loads, and a kernel's end waits for them (7B layer, 9
    // rows: QKV 20.7 -> 19.3, O 9.4 -> 8.9, gate/up 32.9 -> 31.3, down 20.9 -> 20.0 us; a pass 3339 -> 3193, of 20 rows 4553 -> 4272).
    auto group = [&](int j, bool more) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            const bool live = more || j + u < n;                   // steps past the end meet zero weights
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                uint4 wv = rw[u][t];
                if (!live) wv = make_uint4(0u, 0u, 0u, 0u);
                const bf16x8 A = __builtin_bit_cast(bf16x8, wv);
#pragma unroll
                for (int x = 0; x < MT; ++x) {
                    acc[t][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, Bh[u][x]), acc[t][x], 0, 0, 0);
                    acc[t][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, Bl[u][x]), acc[t][x], 0, 0, 0);
                }
            }
            if (!more) continue;
            __builtin_amdgcn_sched_barrier(0);                     // keep the refill behind its MFMAs: same registers, no copies
            const int sj = min(j + DEPTH + u, nn);                 // prefetches clamped to the last step
#pragma unroll
            for (int x = 0; x < MT; ++x)
                if (load_ok[x]) { Bh[u][x] = ldg16(bh + sj * (R * 32) + x * 512); Bl[u][x] = ldg16(bl + sj * (R * 32) + x * 512); }
#pragma unroll
            for (int t = 0; t < NT; ++t) rw[u][t] = ldg16_stream<STREAM>(reinterpret_cast<const uint16_t*>(wp[t] + loff + sj * 4096));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int j = 0;
    for (; j + DEPTH < n; j += DEPTH) group(j, true);
    group(j, false);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int x = 0; x < MT; ++x) *reinterpret_cast<f32x4*>(&red[((wave * NT + t) * MT + x) * 256 + lane * 4]) = acc[t][x];
    float* ssred = red + 8 * NT * MT * 256;                        // [8 wavefronts][R rows]
    if (EPI != EPI_RESID) {
#pragma unroll
        for (int x = 0; x < MT; ++x) {
            float part = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) part += wave * 4 + lq + 32 * i < a.ssq_tiles ? sv[x][i] : 0.f;
            for (int t = wave * 4 + lq + 256; t < a.ssq_tiles; t += 32) part += a.ssq_in[(size_t)lm[x] * a.ssq_tiles + t];
            part += __shfl_xor(part, 16, 64);
            part += __shfl_xor(part, 32, 64);
            if (lq == 0) ssred[wave * R + 16 * x + li] = part;
        }
    }
    __syncthreads();
    if (!fin) return;
    // lane holds D[column c + e][row m] of its unit
    const int xt = wave / NU;
    f32x4 t1 = {0.f, 0.f, 0.f, 0.f}, t2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        const f32x4 p = *reinterpret_cast<const f32x4*>(&red[((v * NT + unit * PER) * MT + xt) * 256 + lane * 4]);
        t1[0] += p[0]; t1[1] += p[1]; t1[2] += p[2]; t1[3] += p[3];
        if (EPI == EPI_SWIGLU) {
            const f32x4 q = *reinterpret_cast<const f32x4*>(&red[((v * NT + unit * PER + 1) * MT + xt) * 256 + lane * 4]);
            t2[0] += q[0]; t2[1] += q[1]; t2[2] += q[2]; t2[3] += q[3];
        }
    }
    if (EPI == EPI_RESID) {
        float ss = 0.f;
        if (row_ok) {
            float4 xv = x_old;
            xv.x += t1[0]; xv.y += t1[1]; xv.z += t1[2]; xv.w += t1[3];
            *reinterpret_cast<float4*>(a.x + (size_t)m * a.N + c) = xv;
            ss = xv.x * xv.x + xv.y * xv.y + xv.z * xv.z + xv.w * xv.w;
            if (a.gain_next)
                store_planes4(a.out_planes, a.out_plane, a.out_tiled ? xt_index(m, c, R) : (size_t)m * a.N + c,
                              xv.x * g_next.x, xv.y * g_next.y, xv.z * g_next.z, xv.w * g_next.w);
        }
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (row_ok && lq == 0 && a.ssq_out) a.ssq_out[(size_t)m * (a.N / 16) + (c >> 4)] = ss;
        return;
    }
    if (!row_ok) return;
    float ssq = 0.f;
#pragma unroll
    for (int v = 0; v < 8; ++v) ssq += ssred[v * R + mrow];
    const float rscale = 1.0f / sqrtf(ssq / (float)a.K + a.eps);  // r = rsqrt(mean square + eps) of the lane's input row
    if (EPI == EPI_SWIGLU) {
        float h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float g = t1[e] * rscale, u = t2[e] * rscale;
            h[e] = g / (1.0f + __expf(-g)) * u;
        }
        store_planes4(a.out_planes, a.out_plane, a.out_tiled ? xt_index(m, c, R) : (size_t)m * a.N + c, h[0], h[1], h[2], h[3]);
    } else {
        const int nq = a.H * a.hd, nkv = a.KVH * a.hd;
        const int p = p_row, b = m / a.q_len;
        const float v[4] = {t1[0] * rscale, t1[1] * rscale, t1[2] * rscale, t1[3] * rscale};
        if (c < nq + nkv) {
            const int hc = c & hd_mask;
            const float r0 = v[0] * rc0.x - v[1] * rc0.y, r1 = v[0] * rc0.y + v[1] * rc0.x;
            const float r2 = v[2] * rc1.x - v[3] * rc1.y, r3 = v[2] * rc1.y + v[3] * rc1.x;
            if (c < nq) {
                *reinterpret_cast<float4*>(a.q_out + (size_t)m * nq + c) = make_float4(r0, r1, r2, r3);
            } else if (p >= 0) {
                const int kh = (c - nq) >> (__ffs(a.hd) - 1);
                uint16_t* dst = a.k_cache + (((size_t)b * a.KVH + kh) * a.cache_len + p) * a.hd + hc;
                *reinterpret_cast<uint2*>(dst) = make_uint2((uint32_t)from_f<uint16_t>(r0) | ((uint32_t)from_f<uint16_t>(r1) << 16),
                                                            (uint32_t)from_f<uint16_t>(r2) | ((uint32_t)from_f<uint16_t>(r3) << 16));
            }
        } else if (p >= 0) {
            const int cv = c - nq - nkv;
            const int vh = cv >> (__ffs(a.hd) - 1), hc = cv & hd_mask;
            uint16_t* base = a.v_cache + ((size_t)b * a.KVH + vh) * (size_t)a.cache_len * a.hd;
#pragma unroll
            for (int e = 0; e < 4; ++e) base[v_index<uint16_t>(p, hc + e, a.hd)] = from_f<uint16_t>(v[e]);
        }
    }
}

// `units` units are dealt to the workgroups in consecutive runs of TU or TU - 1 (host: ceil(units / grid) == TU, grid <= units)
template <int EPI, int TU, int MT, bool STREAM>
__global__ __launch_bounds__(512) void gemm_rows_kernel(DecArgs a, int units) {
    // [8 wavefronts][tiles][row tiles][256] accumulators, then the rows' sums of squares
    __shared__ __attribute__((aligned(16))) float red[8 * TU * (EPI == EPI_SWIGLU ? 2 : 1) * MT * 256 + 8 * 16 * MT];
    const int G = gridDim.x, b = blockIdx.x;
    const int base = units / G, rem = units - base * G;
    const int nu = base + (b < rem ? 1 : 0), u0 = b * base + min(b, rem);
    if (nu == TU) rows_body<EPI, TU, MT, STREAM>(a, u0, red);
    else if (TU > 1 && nu == TU - 1) rows_body<EPI, (TU > 1 ? TU - 1 : 1), MT, STREAM>(a, u0, red);
}

// Split-K factor of the 16-row kernel: the smallest power of two that gives about 450 workgroups (two per
// compute unit keep enough loads in flight; measured on the 7B shapes, more splits only add partial sums
// for the consumer kernels to read), with at least 256 columns per split.
static int m16_splits(int N, int K) {
    const int tiles = (N + 63) / 64;
    int ks = 1;
    while (ks * tiles < 448) ks *= 2;
    const int cap = K / 256 > 1 ? K / 256 : 1;
    if (ks > cap) ks = cap;
    const int kper = ((K + ks - 1) / ks + 31) / 32 * 32;
    return (K + kper - 1) / kper;
}

// ---- GEMM, fp32 (plumbing configuration): one wavefront per output column and four or eight rows, lanes stride K four at a time ----
// Tiny matrices, so a launch is its trips to memory and its shuffles: the chunks of the weight row and of the rows of x are
// asked for together, unconditionally (rows past M repeat the last one), and the rows are spread over workgroups -- eight rows
// one after the other for a batch being verified, one column per lane, took 11.6 us for 20 rows of a 128-wide projection, 24
// rows side by side in a wavefront 8.7 (144 shuffles), now 3.4.
// WIDE, for matrices of 16 MB and more under 48 rows and more: there a launch is the weights coming out of the caches once per
// group of rows.  Eight rows a group, and the groups of a column next to each other in the launch: one layer of 4096 columns
// at 48 / 144 / 1024 rows 2225 -> 1551, 6514 -> 4176, 45371 -> 27824 us, two of 2048 columns at 48 rows 906 -> 870.  With
// fewer rows the padding to eights costs what that gains (two layers of 2048 columns, 20 rows 459 -> 490), with smaller
// matrices the longer chain of a wavefront does (eight layers of 128 columns, 144 rows 358 -> 368).  A sum's order is the same.
template <bool VEC, bool WIDE>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs a) {
    constexpr int F32_RB = WIDE ? 8 : 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = (WIDE ? blockIdx.y : blockIdx.x) * 4 + wave;
    const int group = WIDE ? blockIdx.x : blockIdx.y, groups = WIDE ? gridDim.x : gridDim.y;
    if (n >= a.N) return;
    int seg = 0, local = n;
    if (local >= a.seg_rows[0]) { local -= a.seg_rows[0]; seg = 1; if (local >= a.seg_rows[1]) { local -= a.seg_rows[1]; seg = 2; } }
    const float* w0 = reinterpret_cast<const float*>(a.w[seg]) + (size_t)local * a.K;
    const float* x = reinterpret_cast<const float*>(a.x);
    for (int m0 = group * F32_RB; m0 < a.M; m0 += groups * F32_RB) {       // one turn unless the rows exceed the grid's limit
        float acc[F32_RB];
#pragma unroll
        for (int r = 0; r < F32_RB; ++r) acc[r] = 0.f;
        for (int k = lane * 4; k < a.K; k += 256) {                   // K % 8 == 0 (host check)
            const float4 wv = VEC ? *reinterpret_cast<const float4*>(w0 + k) : make_float4(w0[k], w0[k + 1], w0[k + 2], w0[k + 3]);
            float4 xv[F32_RB];
#pragma unroll
            for (int r = 0; r < F32_RB; ++r) xv[r] = *reinterpret_cast<const float4*>(x + (size_t)min(m0 + r, a.M - 1) * a.K + k);
#pragma unroll
            for (int r = 0; r < F32_RB; ++r) acc[r] = fmaf(xv[r].w, wv.w, fmaf(xv[r].z, wv.z, fmaf(xv[r].y, wv.y, fmaf(xv[r].x, wv.x, acc[r]))));
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int r = 0; r < F32_RB; ++r) acc[r] += __shfl_xor(acc[r], o, 64);
        float mine = 0.f;                                              // lane r stores row r
#pragma unroll
        for (int r = 0; r < F32_RB; ++r) mine = lane == r ? acc[r] : mine;
        if (lane < F32_RB && m0 + lane < a.M) reinterpret_cast<float*>(a.out)[(size_t)(m0 + lane) * a.ldo + n] = mine;
    }
}

int gemm_splits(int dtype, int N, int K, int M) {
    if (dtype != BS_BF16) return 1;
    if (M <= 16) return m16_splits(N, K);
    const int stages = (K + 255) / 256;
    if (M > 32 && K % 32 == 0) return big_splits(N, K, M);
    const int tiles = (N + 63) / 64;
    int ks = (768 + tiles - 1) / tiles;
    if (ks > stages / 2) ks = stages / 2;
    if (ks > 16) ks = 16;
    if (ks < 1) ks = 1;
    return ks;
}

// ---- optional per-launch timing of the weight-streaming GEMM (measurement hook) ----------------------
struct GemmProfile {
    bool on = false;
    std::vector<hipEvent_t> ev;       // pairs (start, stop)
    std::vector<double> bytes;        // algorithmic bytes of each timed launch: the weight tile once
    std::vector<int> mt;
};
static GemmProfile g_prof;
static std::mutex g_prof_mutex;      // launches may come from several host threads

// Switching on starts an empty record; switching off drops the record and its events (collect first).
int profile_enable(int on) {
    std::lock_guard<std::mutex> lock(g_prof_mutex);
    g_prof.on = on != 0;
    for (hipEvent_t e : g_prof.ev) (void)hipEventDestroy(e);
    g_prof.ev.clear(); g_prof.bytes.clear(); g_prof.mt.clear();
    return BS_OK;
}

// Events for one timed launch, or none when the record is off.  Events cannot be recorded into a stream capture: a
// launch that is being captured while the record is on is refused.
int prof_events(hipStream_t s, hipEvent_t* e0, hipEvent_t* e1) {
    *e0 = nullptr; *e1 = nullptr;
    std::lock_guard<std::mutex> lock(g_prof_mutex);
    if (!g_prof.on) return BS_OK;
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    BS_HIP(hipStreamIsCapturing(s, &st));
    BS_REQUIRE(st == hipStreamCaptureStatusNone, BS_ESTATE, "per-launch timing is switched on while the stream is being captured: "
               "switch it off (bs_profile_enable(0)) before capturing");
    BS_HIP(hipEventCreate(e0));
    if (hipEventCreate(e1) != hipSuccess) { (void)hipEventDestroy(*e0); *e0 = nullptr; BS_FAIL(BS_EHIP, "hipEventCreate failed"); }
    return BS_OK;
}
void prof_record(hipEvent_t e0, hipEvent_t e1, double bytes, int cls) {
    if (!e0) return;
    std::lock_guard<std::mutex> lock(g_prof_mutex);
    if (!g_prof.on) { (void)hipEventDestroy(e0); (void)hipEventDestroy(e1); return; }   // switched off in between
    g_prof.ev.push_back(e0); g_prof.ev.push_back(e1);
    g_prof.bytes.push_back(bytes);
    g_prof.mt.push_back(cls);
}

int profile_collect(int mt_filter, double* total_ms, double* total_bytes, long long* launches) {
    std::lock_guard<std::mutex> lock(g_prof_mutex);
    double ms = 0.0, by = 0.0;
    long long n = 0;
    for (size_t i = 0; i < g_prof.bytes.size(); ++i) {
        if (mt_filter > 0 && g_prof.mt[i] != mt_filter) continue;
        BS_HIP(hipEventSynchronize(g_prof.ev[2 * i + 1]));
        float t = 0.f;
        BS_HIP(hipEventElapsedTime(&t, g_prof.ev[2 * i], g_prof.ev[2 * i + 1]));
        ms += t; by += g_prof.bytes[i]; ++n;
    }
    if (total_ms) *total_ms = ms;
    if (total_bytes) *total_bytes = by;
    if (launches) *launches = n;
    return BS_OK;
}

size_t packed_elems(int N, int K) { return (size_t)((N + 63) / 64) * 64 * (size_t)K; }

int launch_pack_weights(const void* src, void* dst, int N, int K, hipStream_t s) {
    BS_REQUIRE(K % 32 == 0 && N >= 1, BS_ESHAPE, "pack_weights: K=%d must be a multiple of 32", K);
    const size_t chunks = packed_elems(N, K) / 8;
    hipLaunchKernelGGL(pack_weights_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, s,
                       (const uint16_t*)src, (uint16_t*)dst, N, K);
    BS_LAUNCH_CHECK();
    return BS_OK;
}

int launch_gemm(int dtype, GemmArgs a, hipStream_t s) {
    if (a.M <= 0 || a.N <= 0) return BS_OK;
    BS_REQUIRE(!a.tiled || (dtype == BS_BF16 && a.K % 32 == 0 && (!a.w[1] || a.seg_rows[0] % 16 == 0) && (!a.w[2] || a.seg_rows[1] % 16 == 0)),
               BS_ESHAPE, "gemm: tiled weights need bf16, K %% 32 == 0 and stacked matrices whose row counts are multiples of 16");
    if (dtype == BS_F32) {
        const int cols = (a.N + 3) / 4;
        const bool wide = a.M >= 48 && (size_t)a.N * a.K >= (size_t)1 << 22 && cols <= 65535;
        const int groups = wide ? (a.M + 7) / 8 : (a.M + 3) / 4;
        const dim3 grid = wide ? dim3(groups, cols) : dim3(cols, groups < 65535 ? groups : 65535), block(256);
        // a caller's LM head need not be 16-byte aligned (the layers' matrices and the activations are)
        const bool vec = ((reinterpret_cast<uintptr_t>(a.w[0]) | reinterpret_cast<uintptr_t>(a.w[1]) | reinterpret_cast<uintptr_t>(a.w[2])) & 15) == 0;
        if (vec && wide) hipLaunchKernelGGL((gemm_f32_kernel<true, true>), grid, block, 0, s, a);
        else if (vec) hipLaunchKernelGGL((gemm_f32_kernel<true, false>), grid, block, 0, s, a);
        else if (wide) hipLaunchKernelGGL((gemm_f32_kernel<false, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((gemm_f32_kernel<false, false>), grid, block, 0, s, a);
        BS_LAUNCH_CHECK();
        return BS_OK;
    }
    const bool big_ok = a.K % 32 == 0;                              // the many-row kernel works in whole 32-column stages
    hipEvent_t e0 = nullptr, e1 = nullptr;
    auto prof_begin = [&]() -> int { return prof_events(s, &e0, &e1); };
    auto prof_end = [&](int mt) -> int {                            // classes by 16-row tiles: 1, 2, 4, 6, 8, 16
        prof_record(e0, e1, (double)a.N * (double)a.K * 2.0, mt <= 1 ? 1 : mt <= 2 ? 2 : mt <= 4 ? 4 : mt <= 6 ? 6 : mt <= 8 ? 8 : 16);
        return BS_OK;
    };
    int rc;
    if (big_ok && a.M > 32) {
        return launch_gemm_big(a, s);
    }
    // up to 32 rows (or K not a multiple of 32: 32 rows at a time)
    const int max_rows = a.M <= 16 ? 16 : 32;
    for (int m0 = 0; m0 < a.M; m0 += max_rows) {
        GemmArgs c = a;
        c.M = (a.M - m0 < max_rows) ? a.M - m0 : max_rows;
        c.x = reinterpret_cast<const uint16_t*>(a.x) + (size_t)m0 * a.K;
        c.out = reinterpret_cast<float*>(a.out) + (size_t)m0 * a.ldo;
        const dim3 grid((a.N + 63) / 64, a.KS), block(256);
        const int kper = ((a.K + a.KS - 1) / a.KS + 31) / 32 * 32;      // columns per split, whole k slices
        if ((rc = prof_begin()) != BS_OK) return rc;
        // one 16-row weight tile per wavefront measured faster than two (3.7 vs 3.2 TB/s over the 7B layer shapes)
        if (a.M <= 16) {
            if (a.tiled) BS_LAUNCH_TIMED((gemm_bf16_m16_kernel<1, true>), grid, block, 0, s, e0, e1, c, kper);
            else BS_LAUNCH_TIMED((gemm_bf16_m16_kernel<1, false>), grid, block, 0, s, e0, e1, c, kper);
        } else {
            if (a.tiled) BS_LAUNCH_TIMED((gemm_bf16_kernel<2, 1, 256, true>), grid, block, 0, s, e0, e1, c);
            else BS_LAUNCH_TIMED((gemm_bf16_kernel<2, 1, 256, false>), grid, block, 0, s, e0, e1, c);
        }
        BS_LAUNCH_CHECK();
        if ((rc = prof_end((c.M + 15) / 16)) != BS_OK) return rc;
    }
    return BS_OK;
}

// ---- RoPE + KV append -----------------------------------------------------------------------------
// grid (M, H + 2*KVH); thread = one rotation pair.  Row layout of the projection: [q heads | k heads | v heads],
// given as split-K partials that are summed here.  q stays fp32; k and v are rounded to the cache dtype.
template <typename T>
__global__ void rope_kv_kernel(const float* __restrict__ part, int ks, size_t ks_stride, const int32_t* __restrict__ pos,
                               const float2* __restrict__ rope, int q_len, int H, int KVH, int hd, int max_len,
                               float* __restrict__ q_out, T* __restrict__ k_cache, T* __restrict__ v_cache,
                               const float* __restrict__ ssq, int nchunks, float inv_d, float eps) {
    const int m = blockIdx.x, head = blockIdx.y, i = threadIdx.x;       // i < hd/2
    const int p = pos[m];
    const int b = m / q_len;
    const int ld = (H + 2 * KVH) * hd;
    const float* src = part + (size_t)m * ld + (size_t)head * hd;
    float x0 = 0.f, x1 = 0.f;
    for (int s = 0; s < ks; ++s) {
        const float2 v = *reinterpret_cast<const float2*>(src + (size_t)s * ks_stride + 2 * i);
        x0 += v.x; x1 += v.y;
    }
    {
        const float rs = row_rscale(ssq, nchunks, m, inv_d, eps);      // the input rows' RMS scale, if it was deferred
        x0 *= rs; x1 *= rs;
    }
    if (head < H + KVH) {
        const float2 cs = rope[(size_t)m * (hd / 2) + i];
        const float r0 = x0 * cs.x - x1 * cs.y, r1 = x0 * cs.y + x1 * cs.x;
        if (head < H) {
            float* dst = q_out + (size_t)m * H * hd + (size_t)head * hd;
            dst[2 * i] = r0; dst[2 * i + 1] = r1;
        } else if (p >= 0) {
            T* dst = k_cache + (((size_t)b * KVH + (head - H)) * max_len + p) * hd;
            dst[2 * i] = from_f<T>(r0); dst[2 * i + 1] = from_f<T>(r1);
        }
    } else if (p >= 0) {
        T* base = v_cache + ((size_t)b * KVH + (head - H - KVH)) * (size_t)max_len * hd;
        base[v_index<T>(p, 2 * i, hd)] = from_f<T>(x0);
        base[v_index<T>(p, 2 * i + 1, hd)] = from_f<T>(x1);
    }
}

// ---- fp32 projections with the work around them -----------------------------------------------------------
// A pass of a small fp32 model is launches: of a layer's nine, four moved a few KB (norm, RoPE + cache write, norm, SwiGLU) and took 2 to 3 us
// each.  Here a wavefront has two columns (a rotation pair; gate and up of a column) under four rows, sums the rows' squares beside the
// products (RMSNorm is linear: r (g .* x) W^T, r per row) and finishes them: RMS scale + RoPE + q + cache write (QKV), silu(r g) r u
// (SWIGLU), x += y (RESID), the logits (HEAD: N rows of the LM head, RMS scale).  The first layer reads the embedding's rows itself, and the first
// RESID leaves x.  A layer is five launches instead of nine, a pass two more instead of four: a round of four steps of a draft of 64 columns and one layer and
// a target of 128 and two, batch 4, 321 -> 246 us (23 of them by attn_kernel).
// The twelve sums of a wavefront (two products and the squares of four rows) are halved in number at each of the first four steps of their
// reduction: 17 exchanges instead of 72.  Sum i ends in lanes 4 i .. 4 i + 3.
template <int N>
__device__ __forceinline__ void halve_sums(float (&v)[16], int lane) {
    const bool up = lane & (4 * N);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float keep = up ? v[i + N] : v[i], give = up ? v[i] : v[i + N];
        v[i] = keep + __shfl_xor(give, 4 * N, 64);
    }
}
__device__ __forceinline__ float reduce16(float (&v)[16]) {
    const int lane = threadIdx.x & 63;
    halve_sums<8>(v, lane); halve_sums<4>(v, lane); halve_sums<2>(v, lane); halve_sums<1>(v, lane);
    float t = v[0];
    t += __shfl_xor(t, 2, 64);
    return t + __shfl_xor(t, 1, 64);
}
template <int EPI, bool VEC>
__global__ __launch_bounds__(256) void f32_fused_kernel(F32Args a) {
    const int lane = threadIdx.x & 63, p = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int c = EPI == F32_SWIGLU ? p : 2 * p;                   // this wavefront's output column, or the first of two
    if (c >= a.N) return;
    const float *w0, *w1;
    if (EPI == F32_SWIGLU) {
        w0 = a.w[0] + (size_t)c * a.K; w1 = a.w[1] + (size_t)c * a.K;
    } else {
        int seg = 0, local = c;                                    // segments are of even length
        if (EPI == F32_QKV && local >= a.nq) { local -= a.nq; seg = 1; if (local >= a.nkv) { local -= a.nkv; seg = 2; } }
        w0 = a.w[seg] + (size_t)local * a.K; w1 = c + 1 < a.N ? w0 + a.K : w0;
    }
    for (int m0 = blockIdx.y * 4; m0 < a.M; m0 += gridDim.y * 4) { // one turn unless the rows exceed the grid's limit
        const float* xr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = min(m0 + r, a.M - 1);
            const int src = EPI == F32_HEAD ? (m / a.rows_out) * a.rows_in + (a.rows_in - a.rows_out) + m % a.rows_out : m;
            xr[r] = a.x + (size_t)(EPI != F32_RESID && a.tok ? a.tok[src] : src) * a.K;
        }
        // what the epilogue needs: lane 4 r finishes row r
        const int m = min(m0 + ((lane >> 2) & 3), a.M - 1);
        int pos = -1;
        float2 cs = make_float2(1.f, 0.f), old = make_float2(0.f, 0.f);
        if (EPI == F32_QKV) {
            pos = a.pos[m];
            if (c < a.nq + a.nkv) cs = a.rope[(size_t)m * (a.hd / 2) + c % a.hd / 2];
        }
        if (EPI == F32_RESID) old = *reinterpret_cast<const float2*>(a.tok ? a.x_old + (size_t)a.tok[m] * a.N + c : a.out + (size_t)m * a.N + c);     // N is even
        float v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = 0.f;
        for (int k = lane * 4; k < a.K; k += 256) {                // K % 8 == 0 (host check)
            float4 u0 = VEC ? *reinterpret_cast<const float4*>(w0 + k) : make_float4(w0[k], w0[k + 1], w0[k + 2], w0[k + 3]);
            float4 u1 = VEC ? *reinterpret_cast<const float4*>(w1 + k) : make_float4(w1[k], w1[k + 1], w1[k + 2], w1[k + 3]);
            float4 xv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) xv[r] = *reinterpret_cast<const float4*>(xr[r] + k);
            if (EPI != F32_RESID) {
                const float4 g = VEC ? *reinterpret_cast<const float4*>(a.gain + k) : make_float4(a.gain[k], a.gain[k + 1], a.gain[k + 2], a.gain[k + 3]);
                u0 = make_float4(u0.x * g.x, u0.y * g.y, u0.z * g.z, u0.w * g.w);
                u1 = make_float4(u1.x * g.x, u1.y * g.y, u1.z * g.z, u1.w * g.w);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] = fmaf(xv[r].w, u0.w, fmaf(xv[r].z, u0.z, fmaf(xv[r].y, u0.y, fmaf(xv[r].x, u0.x, v[r]))));
                v[4 + r] = fmaf(xv[r].w, u1.w, fmaf(xv[r].z, u1.z, fmaf(xv[r].y, u1.y, fmaf(xv[r].x, u1.x, v[4 + r]))));
                if (EPI != F32_RESID) v[8 + r] = fmaf(xv[r].w, xv[r].w, fmaf(xv[r].z, xv[r].z, fmaf(xv[r].y, xv[r].y, fmaf(xv[r].x, xv[r].x, v[8 + r]))));
            }
        }
        const float t = reduce16(v);
        float y0 = t, y1 = __shfl(t, (lane & 15) + 16, 64);
        if (EPI != F32_RESID) {
            const float rs = 1.0f / sqrtf(__shfl(t, (lane & 15) + 32, 64) / (float)a.K + a.eps);
            y0 *= rs; y1 *= rs;
        }
        if (lane >= 16 || (lane & 3) || m0 + (lane >> 2) >= a.M) continue;
        if (EPI == F32_SWIGLU) a.out[(size_t)m * a.N + c] = y0 / (1.0f + __expf(-y0)) * y1;
        if (EPI == F32_RESID) *reinterpret_cast<float2*>(a.out + (size_t)m * a.N + c) = make_float2(old.x + y0, old.y + y1);
        if (EPI == F32_HEAD) {
            float* o = a.out + (size_t)m * a.ldo + c;
            o[0] = y0;
            if (c + 1 < a.N) o[1] = y1;
        }
        if (EPI == F32_QKV) {
            const float2 rot = make_float2(y0 * cs.x - y1 * cs.y, y0 * cs.y + y1 * cs.x);
            const int b = m / a.q_len, d = c % a.hd;
            if (c < a.nq) *reinterpret_cast<float2*>(a.out + (size_t)m * a.nq + c) = rot;
            else if (pos >= 0) {
                const bool key = c < a.nq + a.nkv;
                const int head = (c - a.nq - (key ? 0 : a.nkv)) / a.hd;
                float* dst = (key ? a.k_cache : a.v_cache) + (((size_t)b * (a.nkv / a.hd) + head) * a.cache_len + pos) * a.hd + d;
                *reinterpret_cast<float2*>(dst) = key ? rot : make_float2(y0, y1);
            }
        }
    }
}

// ---- attention -------------------------------------------------------------------------------------
// grid (n_splits x row groups, H, B), 256 lanes.  The keys 0..n_keys-1 (n_keys = pos of the last query row + 1) are cut
// into n_splits chunks of whole 64-key tiles; the 4 wavefronts of a workgroup take 16, 32 or 64 keys of their
// chunk in turn.  Score phase: lane = key.  Value phase: lane = head-dim element (d and d+64).
// A workgroup takes ATT_RB query rows (the shuffles of nine rows at a time were most of what a launch over a short cache does,
// and a prompt chunk's rows ran one group after the other in one workgroup); the keys and values of a turn are in flight before the queries
// are there.  Writes un-normalised partials (m, l, o[hd]) per split, or the output itself where there is one split.  One
// row / 5 rows against 50 keys: 8.9 / 9.1 us each with a wavefront's 64 keys at a time and loads where they are used, 5.0 / 5.5 like this.
constexpr int ATT_RB = 2;
constexpr int ATT_VF = 16;

template <typename T>
__device__ __forceinline__ void load8(const T* p, float out[8]);
template <>
__device__ __forceinline__ void load8<float>(const float* p, float out[8]) {
    const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w; out[4] = b.x; out[5] = b.y; out[6] = b.z; out[7] = b.w;
}
template <>
__device__ __forceinline__ void load8<uint16_t>(const uint16_t* p, float out[8]) {
    const uint4 a = *reinterpret_cast<const uint4*>(p);
    out[0] = __uint_as_float(a.x << 16); out[1] = __uint_as_float(a.x & 0xFFFF0000u);
    out[2] = __uint_as_float(a.y << 16); out[3] = __uint_as_float(a.y & 0xFFFF0000u);
    out[4] = __uint_as_float(a.z << 16); out[5] = __uint_as_float(a.z & 0xFFFF0000u);
    out[6] = __uint_as_float(a.w << 16); out[7] = __uint_as_float(a.w & 0xFFFF0000u);
}

// SHORT, for launches of at most one workgroup per compute unit over caches of up to 512 keys: its loads ahead take 258 registers, one workgroup a compute
// unit instead of four.  Passes of two layers of 512 columns, 8 heads, without -> with: 1 x 1 row at 48 / 120 / 400 keys 59.0 / 60.0 / 71.5 -> 54.6 / 58.5 /
// 71.9 us, 32 x 1 (256 workgroups) 80.7 / 80.8 / 93.2 -> 76.0 / 79.6 / 94.0; with more workgroups what counts is how many fit: 64 x 1 112 / 114 / 140 -> 116 / 123 /
// 155, 16 x 5 at 48 keys 127.8 -> 129.8, prompts of 100 / 300 / 500 tokens 132 / 315 / 494 -> 140 / 370 / 592, 8 of 500 3.60 -> 4.50 ms; 20 rows of 8 heads of 32
// at 5000 keys 121 -> 163.
template <typename T, bool SHORT>
__global__ __launch_bounds__(256) void attn_kernel(const float* __restrict__ q, const T* __restrict__ k_cache,
                                                   const T* __restrict__ v_cache, const int32_t* __restrict__ pos,
                                                   int q_len, int H, int KVH, int hd, int max_len, float scale, int n_splits,
                                                   float* __restrict__ part, float* __restrict__ direct_out) {
    __shared__ float qs[ATT_RB][128];            // scaled query rows
    __shared__ float ps[4][ATT_RB][64];          // per-wavefront probabilities of the current tile
    __shared__ float wm[4][ATT_RB], wl[4][ATT_RB];
    __shared__ float wo[4][ATT_RB][128];
    const int rg = blockIdx.x / n_splits, split = blockIdx.x - rg * n_splits, h = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kvh = h / (H / KVH);
    const int m_first = b * q_len;
    const int pos0 = pos[m_first];
    const size_t pstride = (size_t)hd + 4;       // o[hd], max, sum, 2 pad: rows stay 16-byte aligned
    if (pos0 < 0) {                                // sequence skipped: empty partials, or a zero output
        if (direct_out)
            for (int idx = rg * ATT_RB * hd + threadIdx.x; idx < min(rg * ATT_RB + ATT_RB, q_len) * hd; idx += 256) direct_out[((size_t)(m_first + idx / hd) * H + h) * hd + idx % hd] = 0.f;
        else for (int idx = rg * ATT_RB + threadIdx.x; idx < min(rg * ATT_RB + ATT_RB, q_len); idx += 256) {
            float* dst = part + ((((size_t)(m_first + idx)) * H + h) * n_splits + split) * pstride;
            dst[hd] = -INFINITY; dst[hd + 1] = 0.f;
        }
        return;
    }
    const int n_keys = pos0 + q_len;
    const int tiles = (n_keys + 63) / 64;
    const int tiles_per_split = (tiles + n_splits - 1) / n_splits;
    const int t_begin = split * tiles_per_split;
    const int t_end = min(tiles, t_begin + tiles_per_split);
    const T* kb = k_cache + ((size_t)b * KVH + kvh) * (size_t)max_len * hd;
    const T* vb = v_cache + ((size_t)b * KVH + kvh) * (size_t)max_len * hd;
    const int d0 = lane, d1 = lane + 64;
    // up to 64 keys are dealt to the four wavefronts 16 at a time, up to 128 in turns of 32
    const int k_end = min(t_end * 64, n_keys), len = k_end - t_begin * 64, turn = SHORT && len <= 64 ? 16 : SHORT && len <= 128 ? 32 : 64;
    // 32 dimensions of a turn's keys and, of up to 32 keys, the values of the first ATT_VF are asked for ahead of it
    float kf[4][8], vf0[ATT_VF], vf1[ATT_VF];
    auto ask = [&](int key0) {
        const T* krow = kb + (size_t)min(key0 + lane, n_keys - 1) * hd;
#pragma unroll
        for (int j = 0; j < 4; ++j) load8<T>(krow + min(8 * j, hd - 8), kf[j]);
        if (turn == 64) return;                      // two trips of 32 values a turn
#pragma unroll
        for (int u = 0; u < ATT_VF; ++u) {
            const int vk = min(key0 + u, n_keys - 1);
            vf0[u] = to_f(vb[v_index<T>(vk, min(d0, hd - 1), hd)]);
            vf1[u] = hd > 64 ? to_f(vb[v_index<T>(vk, min(d1, hd - 1), hd)]) : 0.f;
        }
    };
    int key0 = t_begin * 64 + wave * turn;
    if (SHORT) ask(key0);

    {
        const int r0 = rg * ATT_RB, nr = min(ATT_RB, q_len - r0);
        for (int idx = threadIdx.x; idx < ATT_RB * hd; idx += 256) {
            const int r = idx / hd, d = idx % hd;
            qs[r][d] = (r < nr) ? q[((size_t)(m_first + r0 + r) * H + h) * hd + d] * scale : 0.f;
        }
        __syncthreads();
        float mrow[ATT_RB], lrow[ATT_RB], o0[ATT_RB], o1[ATT_RB];
#pragma unroll
        for (int r = 0; r < ATT_RB; ++r) { mrow[r] = -INFINITY; lrow[r] = 0.f; o0[r] = 0.f; o1[r] = 0.f; }

        for (; key0 < k_end; key0 += 4 * turn) {
            const int key = key0 + lane;
            const bool kvalid = lane < turn && key < k_end;
            // ---- scores: lane = key ----
            float s[ATT_RB];
#pragma unroll
            for (int r = 0; r < ATT_RB; ++r) s[r] = 0.f;
            if (kvalid) {
                const T* krow = kb + (size_t)key * hd;
                for (int dd = 0; dd < hd; dd += 32) {                           // 32 dimensions asked for together
                    float kv[4][8];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (!SHORT || dd > 0) load8<T>(krow + min(dd + 8 * j, hd - 8), kv[j]);
                        else
#pragma unroll
                            for (int e = 0; e < 8; ++e) kv[j][e] = kf[j][e];
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int d = dd + 8 * j;
                        if (d >= hd) break;
#pragma unroll
                        for (int r = 0; r < ATT_RB; ++r) {
                            const float4 qa = *reinterpret_cast<const float4*>(&qs[r][d]);
                            const float4 qb = *reinterpret_cast<const float4*>(&qs[r][d + 4]);
                            s[r] += qa.x * kv[j][0] + qa.y * kv[j][1] + qa.z * kv[j][2] + qa.w * kv[j][3] +
                                    qb.x * kv[j][4] + qb.y * kv[j][5] + qb.z * kv[j][6] + qb.w * kv[j][7];
                        }
                    }
                }
            }
            float alpha[ATT_RB];
#pragma unroll
            for (int r = 0; r < ATT_RB; ++r) {
                const bool vis = kvalid && r < nr && key <= pos0 + r0 + r;      // causal
                const float sv = vis ? s[r] : -INFINITY;
                const float mn = fmaxf(mrow[r], wmax(sv));
                const float pr = (mn == -INFINITY) ? 0.f : __expf(sv - mn);
                alpha[r] = (mn == -INFINITY) ? 1.f : __expf(mrow[r] - mn);
                lrow[r] = lrow[r] * alpha[r] + pr;                              // per-lane partial sum
                mrow[r] = mn;
                ps[wave][r][lane] = pr;
            }
            // ---- values: lane = head-dim element ----
#pragma unroll
            for (int r = 0; r < ATT_RB; ++r) { o0[r] *= alpha[r]; o1[r] *= alpha[r]; }
            const int kmax = min(turn, k_end - key0);
            auto add = [&](int k0, float (&v0)[ATT_VF], float (&v1)[ATT_VF]) {
#pragma unroll
                for (int u = 0; u < ATT_VF; u += 4) {
#pragma unroll
                    for (int e = u; e < u + 4; ++e)
                        if (k0 + e >= kmax) { v0[e] = 0.f; v1[e] = 0.f; }       // keys past the end: their probability is zero too
#pragma unroll
                    for (int r = 0; r < ATT_RB; ++r) {
                        const float4 pp = *reinterpret_cast<const float4*>(&ps[wave][r][k0 + u]);
                        o0[r] += pp.x * v0[u] + pp.y * v0[u + 1] + pp.z * v0[u + 2] + pp.w * v0[u + 3];
                        o1[r] += pp.x * v1[u] + pp.y * v1[u + 1] + pp.z * v1[u + 2] + pp.w * v1[u + 3];
                    }
                }
            };
            if (SHORT && turn < 64) add(0, vf0, vf1);
            for (int k0 = SHORT && turn < 64 ? ATT_VF : 0; k0 < kmax; k0 += 2 * ATT_VF) {    // the others 2 ATT_VF at a time
                float v0[2][ATT_VF], v1[2][ATT_VF];
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int u = 0; u < ATT_VF; ++u) {
                        const int vk = key0 + min(k0 + x * ATT_VF + u, kmax - 1);
                        v0[x][u] = to_f(vb[v_index<T>(vk, min(d0, hd - 1), hd)]);
                        v1[x][u] = hd > 64 ? to_f(vb[v_index<T>(vk, min(d1, hd - 1), hd)]) : 0.f;
                    }
                add(k0, v0[0], v1[0]);
                if (k0 + ATT_VF < 64) add(k0 + ATT_VF, v0[1], v1[1]);
            }
            if (SHORT && key0 + 4 * turn < k_end) ask(key0 + 4 * turn);
        }
        // ---- combine the 4 wavefronts ----
#pragma unroll
        for (int r = 0; r < ATT_RB; ++r) {
            const float l = wsum(lrow[r]);
            if (lane == 0) { wm[wave][r] = mrow[r]; wl[wave][r] = l; }
            wo[wave][r][d0] = o0[r];
            wo[wave][r][d1] = o1[r];
        }
        __syncthreads();
        for (int idx = threadIdx.x; idx < nr * hd; idx += 256) {
            const int r = idx / hd, d = idx % hd;
            const float mm = fmaxf(fmaxf(wm[0][r], wm[1][r]), fmaxf(wm[2][r], wm[3][r]));
            float o = 0.f, l = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float f = (wm[w][r] == -INFINITY) ? 0.f : __expf(wm[w][r] - mm);
                o += wo[w][r][d] * f;
                l += wl[w][r] * f;
            }
            if (direct_out) {                          // a single split of the keys: this is the attention output
                direct_out[((size_t)(m_first + r0 + r) * H + h) * hd + d] = l > 0.f ? o / l : 0.f;
                continue;
            }
            float* dst = part + ((((size_t)(m_first + r0 + r)) * H + h) * n_splits + split) * pstride;
            dst[d] = o;
            if (d == 0) { dst[hd] = mm; dst[hd + 1] = l; }
        }
    }
}

// ---- attention, bf16 cache, MFMA ---------------------------------------------------------------------
// grid (n_splits, KVH, B), 4 wavefronts.  Rows of the score matrix = the q_len query positions of the
// H/KVH query heads that share this kv head (16 rows per MFMA tile).  The wavefronts take the 32-key
// blocks of their split in turn:
//   S^T = K . Q^T      A = K rows straight from the cache, B = Q (fp32 queries as a bf16 hi/lo pair)
//   online softmax     a row lives in one lane column (l % 16); its 32 scores sit in 4 lanes -> 2 shuffles
//   O^T += V^T . P^T   A = transposed V block (one 16-byte load per lane), B = P^T taken from the score
//                      accumulators as they are (hi/lo pair), no LDS, no transposes
// Bytes: every K and V element is read once per 16 rows (per 32 with two tiles per wavefront, below).  Un-normalised
// partials (m, l, o[hd]) per split.
// NT = 16-row tiles a wavefront holds at the same time: every K and V block it loads is multiplied with all of them.
// With grouped queries a verification pass has G * (gamma + 1) rows per kv head, more than one tile from 17 rows on, and a
// second workgroup for the second tile walks the whole cache a second time (batch 32, 8192 cached keys, 24 rows: 3.7
// TB/s of distinct K/V bytes against 5.3 with one tile).  Two tiles take about 320 registers, one wavefront per SIMD;
// its next block is therefore requested before the current one is multiplied (two register sets, loop unrolled by two;
// two blocks ahead measured the same).
// Combining the key splits inside this kernel (mg.cells != null; one row tile, all workgroups resident together: host
// check): a workgroup hands its partial over in exchange cells instead of `part`, then the workgroup of split s combines,
// for the rows r = S-1-s, 2S-1-s, ... of its head group (S splits; the last splits hold the fewest keys, often none), the
// partials of all splits as they arrive (bounded polls) and writes the attention output planes -- the hand-over costs
// about 2 us, 1.6 more for every 256 / HD rows beyond the first, where a merge kernel costs five.
// The cells are all zero when the pass starts (prep kernel) and every layer hands over under its own flag.
struct AttnMerge {
    void* cells;                 // [M][H][n_splits][HD + 4] cells: o[HD], max, sum, 2 pad
    uint16_t* out; size_t plane; // attention output planes; tiled: in the layout of the whole-K projections (xt_index)
    int tiled;                   // rows of the tiled planes, 0: row-major (also of the planes of a single split)
    unsigned flag, spin_limit;
    int32_t* status;             // bit 16: a poll ran out of patience
    unsigned* tickets;           // [B][KVH], with `parts`: the workgroups of a sequence cut into several parts that have handed over, of all layers
};

// AHEAD (one row tile): the next block is requested into the registers of the block at hand as they become free.  For launches whose
// wavefronts walk many blocks (launch_attention); a few blocks are not worth the larger kernel (batch 1, 1682 keys in 4 splits: 17.0 us
// without, 17.7 with).
// PARTS (one row tile): every sequence has its own number of splits of the n_splits that `part` and the cells have room for;
// grid (KVH, items) with the sequence, its split and its first position from the items (attn_deal).  Where direct_out is given, a sequence of
// one part writes the output itself, and of one of several the last workgroup to hand over combines the rows; nobody waits for a
// workgroup that has not started.  A variant of its own: in the other kernels the larger code cost 0.8 us a launch (batch 16, head_dim 64).
template <int HD, int NT, bool STREAM, bool AHEAD, bool PARTS>
__global__ __launch_bounds__(256, NT == 2 ? 1 : HD == 64 ? 4 : 2) void attn_mfma_kernel(const float* __restrict__ q, const uint16_t* __restrict__ k_cache,
                                                        const uint16_t* __restrict__ v_cache,
                                                        const int32_t* __restrict__ pos, int q_len, int H, int KVH,
                                                        int cache_len, float scale, float* __restrict__ part, int n_splits,
                                                        uint16_t* __restrict__ direct_out, size_t plane, AttnMerge mg,
                                                        const long long* __restrict__ items) {
    constexpr int DS = HD / 32, DT = HD / 16;
    constexpr int PC = HD + 4;                   // cells of one partial
    __shared__ float wm[4][16], wl[4][16];
    __shared__ __attribute__((aligned(16))) float wo[4][16][HD + 4];
    // blockIdx.x = (group of NT row tiles, split of the keys): with many query rows (a prompt chunk) the groups are
    // spread over workgroups and the keys over few splits; with one group all of gridDim.x are key splits
    int split, rt, n_rt, kvh, b, used, pos0;
    if constexpr (PARTS) {
        const long long item = items[blockIdx.y];    // one load for all of it; behind the last item b and pos0 are negative
        const int deal = (int)(item >> 32);
        kvh = blockIdx.x; b = deal < 0 ? -1 : deal & 0xFFFF; split = (deal >> 16) & 0xFF; used = deal >> 24; rt = 0; n_rt = 1;
        pos0 = (int)item;
        if (used > 1) direct_out = nullptr;
    } else {
        split = blockIdx.x % n_splits; rt = blockIdx.x / n_splits; n_rt = gridDim.x / n_splits; kvh = blockIdx.y; b = blockIdx.z; used = n_splits;
        pos0 = pos[b * q_len];
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lq = lane >> 4;
    const int G = H / KVH, R = G * q_len;
    const int m_first = b * q_len;
    const size_t pstride = (size_t)HD + 4;       // o[HD], max, sum, 2 pad: rows stay 16-byte aligned
    const bool in_cells = PARTS ? mg.cells && !direct_out : mg.cells != nullptr;
    if (pos0 < 0) {                                  // sequence skipped: empty partials (zeros when writing the output itself)
        if (PARTS && b < 0) return;
        if (direct_out) {
            for (int idx = threadIdx.x + rt * 256; idx < R * HD; idx += 256 * n_rt) {
                const int r = idx / HD, d = idx % HD;
                const int m = m_first + r % q_len, head = kvh * G + r / q_len;
                Act<uint16_t>::store(direct_out, plane, mg.tiled ? xt_index(m, head * HD + d, mg.tiled) : ((size_t)m * H + head) * HD + d, 0.f);
            }
            return;
        }
        if (NT == 1 && in_cells) {                   // no workgroup of this sequence polls: the rows' owners write zeros
            for (int rr = n_splits - 1 - split; rr < R; rr += n_splits) {
                const int m = m_first + rr % q_len, head = kvh * G + rr / q_len;
                for (int d = threadIdx.x; d < HD; d += 256)
                    Act<uint16_t>::store(mg.out, mg.plane, mg.tiled ? xt_index(m, head * HD + d, mg.tiled) : ((size_t)m * H + head) * HD + d, 0.f);
            }
            return;
        }
        for (int r = threadIdx.x; r < R; r += 256) {
            const int g = r / q_len, qi = r % q_len;
            float* dst = part + ((((size_t)(m_first + qi)) * H + kvh * G + g) * n_splits + split) * pstride;
            dst[HD] = -INFINITY; dst[HD + 1] = 0.f;
        }
        return;
    }
    const int n_keys = pos0 + q_len;
    const uint16_t* kb = k_cache + ((size_t)b * KVH + kvh) * (size_t)cache_len * HD;
    const uint16_t* vb = v_cache + ((size_t)b * KVH + kvh) * (size_t)cache_len * HD;

    for (int r0 = rt * 16 * NT; r0 < R; r0 += 16 * NT * n_rt) {
        // keys any row of this group may see (causal): up to the group's latest query position
        const int r_last = min(r0 + 16 * NT - 1, R - 1);
        const int qi_max = (r0 / q_len == r_last / q_len) ? r_last % q_len : q_len - 1;
        const int nblk = (pos0 + qi_max + 1 + 31) / 32;
        const int per = (nblk + used - 1) / used;
        const int b_begin = split * per, b_end = min(nblk, b_begin + per);
        // STREAM: K rows of 256 bytes and V are asked for as data nobody reads again (batch 16, 4096 keys, head_dim 128: 212
        // -> 179 us; V alone 192); rows of 128 bytes stay cached, both halves of a line are then served by one request
        // (head_dim 64: a step of the batch 919 -> 890 us)
        auto fetch_k = [&](int blk, uint4 (&kf)[2][DS]) {
            const int key0 = blk * 32;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int krow = min(key0 + t * 16 + li, n_keys - 1);
#pragma unroll
                for (int ds = 0; ds < DS; ++ds) kf[t][ds] = ldg16_stream<STREAM && HD == 128>(kb + (size_t)krow * HD + ds * 32 + lq * 8);
            }
        };
        auto fetch_v = [&](int blk, uint4 (&vf)[DT]) {
#pragma unroll
            for (int t = 0; t < DT; ++t) vf[t] = ldg16_stream<STREAM>(vb + ((size_t)blk * HD + t * 16 + li) * 32 + lq * 8);
        };
        auto fetch = [&](int blk, uint4 (&kf)[2][DS], uint4 (&vf)[DT]) { fetch_k(blk, kf); fetch_v(blk, vf); };
        bool rvalid[NT];
        int row_pos[NT];
        float4 qa[NT][DS][2];
#pragma unroll
        for (int x = 0; x < NT; ++x) {
            const int row = r0 + 16 * x + li;
            rvalid[x] = row < R;
            const int g = rvalid[x] ? row / q_len : 0, qi = rvalid[x] ? row % q_len : 0;
            row_pos[x] = pos0 + qi;
            const float* qrow = q + ((size_t)(m_first + qi) * H + kvh * G + g) * HD;
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) {
                qa[x][ds][0] = *reinterpret_cast<const float4*>(qrow + ds * 32 + lq * 8);
                qa[x][ds][1] = *reinterpret_cast<const float4*>(qrow + ds * 32 + lq * 8 + 4);
            }
        }
        // The wavefront's first block is asked for together with the queries (without a block: the last one, not used).  That, two
        // register sets, four elements a lane where the wavefronts' sums meet and rows combined side by side, us a launch, 7B shape: 1 x 9 rows,
        // 1682 keys in 4 splits 16.9 -> 14.9; 1 x 5 at 705 in 2 15.1 -> 12.6; 1 x 9 at 7909 in 8 28.4 -> 26.7; 2 x 5 at 1805 in 3 19.0 -> 17.1; 8B
        // shape, 2 x 4 at 2504 in 6 18.5 -> 14.9; 32 x 6 at 8198, two row tiles, 168 -> 160.
        uint4 kf0[2][DS], vf0[DT];
        __builtin_amdgcn_sched_barrier(0);
        fetch(min(b_begin + wave, nblk - 1), kf0, vf0);
        __builtin_amdgcn_sched_barrier(0);
        uint4 qh[NT][DS], ql[NT][DS];
        float m_run[NT], l_run[NT];
        f32x4 o[NT][DT];
#pragma unroll
        for (int x = 0; x < NT; ++x) {
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) {
                const float4 a = qa[x][ds][0], c = qa[x][ds][1];
                float v[8] = {a.x, a.y, a.z, a.w, c.x, c.y, c.z, c.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = rvalid[x] ? v[e] * scale : 0.f;
                split8(v, qh[x][ds], ql[x][ds]);
            }
            m_run[x] = -INFINITY; l_run[x] = 0.f;
#pragma unroll
            for (int t = 0; t < DT; ++t) o[x][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        // more (one tile): the next block's keys and values are asked for as soon as their registers are free, under this block's
        // softmax and products.  Four blocks before the end every key is visible to all of the at most 16 query positions (rows
        // that do not exist have zero queries, and nobody reads their sums).  No branch around those loads: the compiler would have to wait for all of them at the next use.
        auto block = [&](int blk, uint4 (&kf)[2][DS], uint4 (&vf)[DT], bool more) {
            const int key0 = blk * 32;
            // ---- values: keys past n_keys may hold anything, even NaN patterns: zero them ----
            if (!more && key0 + 32 > n_keys) {
#pragma unroll
                for (int t = 0; t < DT; ++t) {
                    uint32_t w[4] = {vf[t].x, vf[t].y, vf[t].z, vf[t].w};
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int key = key0 + (e >> 2) * 16 + 4 * lq + (e & 3);
                        if (key >= n_keys) w[e >> 1] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
                    }
                    vf[t] = make_uint4(w[0], w[1], w[2], w[3]);
                }
            }
#pragma unroll
            for (int x = 0; x < NT; ++x) {
                // ---- scores of 32 keys x 16 rows ----
                f32x4 sc[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    sc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ds = 0; ds < DS; ++ds) {
                        const bf16x8 A = __builtin_bit_cast(bf16x8, kf[t][ds]);
                        sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, qh[x][ds]), sc[t], 0, 0, 0);
                        sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, ql[x][ds]), sc[t], 0, 0, 0);
                    }
                }
                if (more) {
                    __builtin_amdgcn_sched_barrier(0);
                    fetch_k(blk + 4, kf);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // lane holds S^T[key0 + 16t + 4lq + e][row li]
                float sv[8];
                float bm = -INFINITY;
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int key = key0 + t * 16 + 4 * lq + e;
                        const bool vis = more || (rvalid[x] && key < n_keys && key <= row_pos[x]);       // causal
                        sv[t * 4 + e] = vis ? sc[t][e] : -INFINITY;
                        bm = fmaxf(bm, sv[t * 4 + e]);
                    }
                bm = fmaxf(bm, __shfl_xor(bm, 16, 64));
                bm = fmaxf(bm, __shfl_xor(bm, 32, 64));
                const float m_new = fmaxf(m_run[x], bm);
                float pv[8];
                float alpha = 1.f, psum = 0.f;
                if (m_new == -INFINITY) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) pv[e] = 0.f;
                } else {
                    alpha = __expf(m_run[x] - m_new);
#pragma unroll
                    for (int e = 0; e < 8; ++e) { pv[e] = __expf(sv[e] - m_new); psum += pv[e]; }
                }
                l_run[x] = l_run[x] * alpha + psum;
                m_run[x] = m_new;
                uint4 ph, pl;
                split8(pv, ph, pl);
#pragma unroll
                for (int t = 0; t < DT; ++t) {
                    o[x][t][0] *= alpha; o[x][t][1] *= alpha; o[x][t][2] *= alpha; o[x][t][3] *= alpha;
                    const bf16x8 A = __builtin_bit_cast(bf16x8, vf[t]);
                    o[x][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, ph), o[x][t], 0, 0, 0);
                    o[x][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, pl), o[x][t], 0, 0, 0);
                }
            }
            if (more) {
                __builtin_amdgcn_sched_barrier(0);
                fetch_v(blk + 4, vf);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if constexpr (NT == 1 && !AHEAD && HD == 64) {
            for (int blk = b_begin + wave; blk < b_end; blk += 4) {
                if (blk != b_begin + wave) fetch(blk, kf0, vf0);
                block(blk, kf0, vf0, false);
            }
        } else if constexpr (NT == 1 && !AHEAD) {
            // two register sets (head_dim 64, which keeps four workgroups on a compute unit, has none to spare): the next block is
            // requested before the one at hand is multiplied
            uint4 kf1[2][DS], vf1[DT];
            int blk = b_begin + wave;
            for (; blk + 4 < b_end; blk += 8) {
                fetch(blk + 4, kf1, vf1);
                block(blk, kf0, vf0, false);
                fetch(min(blk + 8, b_end - 1), kf0, vf0);
                block(blk + 4, kf1, vf1, false);
            }
            if (blk < b_end) block(blk, kf0, vf0, false);
        } else if constexpr (NT == 1) {
            int blk = b_begin + wave;
            if (blk < b_end) {
                for (; blk + 4 < b_end; blk += 4) block(blk, kf0, vf0, true);
                block(blk, kf0, vf0, false);
            }
        } else if (b_begin + wave < b_end) {
            // a request past the wavefront's last block repeats that block: in bounds, never used
            const int blk_last = b_begin + wave + ((b_end - 1 - b_begin - wave) >> 2) * 4;
            uint4 kf1[2][DS], vf1[DT];
            for (int blk = b_begin + wave; blk < b_end; blk += 8) {
                fetch(min(blk + 4, blk_last), kf1, vf1);
                block(blk, kf0, vf0, false);
                if (blk + 4 >= b_end) break;
                fetch(min(blk + 8, blk_last), kf0, vf0);
                block(blk + 4, kf1, vf1, false);
            }
        }
        // ---- combine the 4 wavefronts, one tile at a time: lane holds O^T[d = 16t + 4lq + e][row li] ----
#pragma unroll
        for (int x = 0; x < NT; ++x) {
            const int rbase = r0 + 16 * x;
            if (rbase >= R) break;
            float lr = l_run[x];
            lr += __shfl_xor(lr, 16, 64);
            lr += __shfl_xor(lr, 32, 64);
            __syncthreads();
            if (lq == 0) { wm[wave][li] = m_run[x]; wl[wave][li] = lr; }
#pragma unroll
            for (int t = 0; t < DT; ++t) *reinterpret_cast<f32x4*>(&wo[wave][li][t * 16 + 4 * lq]) = o[x][t];
            __syncthreads();
            // four elements a lane: 9 rows of 128 are two turns instead of eight 
            for (int idx = threadIdx.x; idx < min(16, R - rbase) * (HD / 4); idx += 256) {
                const int r = idx / (HD / 4), d = idx % (HD / 4) * 4;
                const float mm = fmaxf(fmaxf(wm[0][r], wm[1][r]), fmaxf(wm[2][r], wm[3][r]));
                f32x4 ov = {0.f, 0.f, 0.f, 0.f};
                float lv = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float f = (wm[w][r] == -INFINITY) ? 0.f : __expf(wm[w][r] - mm);
                    const f32x4 wv = *reinterpret_cast<const f32x4*>(&wo[w][r][d]);
                    ov[0] += wv[0] * f; ov[1] += wv[1] * f; ov[2] += wv[2] * f; ov[3] += wv[3] * f;
                    lv += wl[w][r] * f;
                }
                const int gg = (rbase + r) / q_len, qq = (rbase + r) % q_len;
                if (direct_out) {                    // a single split of the keys: this is the attention output
                    const int m = m_first + qq, head = kvh * G + gg;
                    const bool some = lv > 0.f;
                    store_planes4(direct_out, plane, mg.tiled ? xt_index(m, head * HD + d, mg.tiled) : ((size_t)m * H + head) * HD + d,
                                  some ? ov[0] / lv : 0.f, some ? ov[1] / lv : 0.f, some ? ov[2] / lv : 0.f, some ? ov[3] / lv : 0.f);
                    continue;
                }
                if (NT == 1 && in_cells) {           // hand the partial over in cells
                    const DevBuf bc = dev_buf(mg.cells);
                    const int c0 = (((m_first + qq) * H + kvh * G + gg) * n_splits + split) * PC;
                    st_cells4(bc, c0 + d, ov[0], ov[1], ov[2], ov[3], mg.flag);
                    if (d == 0) st_cells2(bc, c0 + HD, mm, lv, mg.flag);
                    continue;
                }
                float* dst = part + ((((size_t)(m_first + qq)) * H + kvh * G + gg) * n_splits + split) * pstride;
                *reinterpret_cast<f32x4*>(dst + d) = ov;
                if (d == 0) { dst[HD] = mm; dst[HD + 1] = lv; }
            }
        }
    }
    if constexpr (NT == 1) {
        if (!in_cells) return;
        if constexpr (PARTS) {                       // the sequence's last workgroup combines all rows
            __shared__ int last;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // this wavefront's cells are stored
            __syncthreads();
            if (threadIdx.x == 0) last = atomicAdd(mg.tickets + b * KVH + kvh, 1u) + 1u == mg.flag * used;
            __syncthreads();
            if (!last) return;
            // four (row, head-dim element) pairs of four parts each in flight a lane: 9 rows in 4 parts are two trips to memory
            // (two of two at head_dim 64, which has no registers for more)
            constexpr int IT = HD == 128 ? 4 : 2, PU = IT;
            const DevBuf bc = dev_buf(mg.cells);
            for (int i0 = threadIdx.x; i0 < R * HD; i0 += 256 * IT) {
                float mm[IT], o[IT], l[IT];
                int cell[IT];
                size_t dst[IT];
#pragma unroll
                for (int it = 0; it < IT; ++it) {
                    const int idx = min(i0 + 256 * it, R * HD - 1), r = idx / HD, d = idx % HD, m = m_first + r % q_len, head = kvh * G + r / q_len;
                    mm[it] = -INFINITY; o[it] = 0.f; l[it] = 0.f;
                    cell[it] = (m * H + head) * n_splits * PC;
                    dst[it] = mg.tiled ? xt_index(m, head * HD + d, mg.tiled) : ((size_t)m * H + head) * HD + d;
                }
                for (int s0 = 0; s0 < used; s0 += PU) {
                    u32x2 co[IT][PU];
                    u32x4 cml[IT][PU];
                    unsigned spins = 0;
                    while (true) {                          // handed over before the ticket, so there at once whatever the limit of the waits is
                        asm volatile("" ::: "memory");
                        bool ok = true;
#pragma unroll
                        for (int it = 0; it < IT; ++it)
#pragma unroll
                            for (int u = 0; u < PU; ++u) {
                                const int c0 = cell[it] + min(s0 + u, used - 1) * PC;
                                co[it][u] = ld_cell1(bc, c0 + (i0 + 256 * it) % HD);
                                cml[it][u] = ld_cells2(bc, c0 + HD);
                            }
#pragma unroll
                        for (int it = 0; it < IT; ++it)
#pragma unroll
                            for (int u = 0; u < PU; ++u) ok = ok && co[it][u].y == mg.flag && cml[it][u].y == mg.flag && cml[it][u].w == mg.flag;
                        if (ok) break;
                        if (++spins > (1u << 18)) { atomicOr(mg.status, 16); break; }
                    }
#pragma unroll
                    for (int it = 0; it < IT; ++it) {
                        float gm = mm[it];
#pragma unroll
                        for (int u = 0; u < PU; ++u) gm = fmaxf(gm, __uint_as_float(cml[it][u].x));       // past the end: the last part again
                        if (gm == -INFINITY) continue;
                        const float keep = __expf(mm[it] - gm);       // 0 when nothing was accumulated yet
                        o[it] *= keep; l[it] *= keep;
#pragma unroll
                        for (int u = 0; u < PU; ++u) {
                            const float mv = __uint_as_float(cml[it][u].x);
                            if (s0 + u >= used || mv == -INFINITY) continue;
                            const float f = __expf(mv - gm);
                            l[it] += __uint_as_float(cml[it][u].z) * f;
                            o[it] += __uint_as_float(co[it][u].x) * f;
                        }
                        mm[it] = gm;
                    }
                }
#pragma unroll
                for (int it = 0; it < IT; ++it)
                    if (i0 + 256 * it < R * HD) Act<uint16_t>::store(mg.out, mg.plane, dst[it], l[it] > 0.f ? o[it] / l[it] : 0.f);
            }
            return;
        }
        // ---- combine the splits of this workgroup's rows, 256 / HD of them at a time: lane = (head-dim element d, row, share of the
        // splits).  With fewer rows than that the spare lanes take shares; row and share are uniform in a wavefront. ----
        constexpr int SUBS = 256 / HD;
        constexpr int MU = 8;                        // splits a lane polls in one round (all loads in flight together)
        const DevBuf bc = dev_buf(mg.cells);
        const int d = threadIdx.x % HD, sub = threadIdx.x / HD;
        const int first = n_splits - 1 - split;
        if (first >= R) return;
        const int sh = SUBS == 4 && first + 2 * n_splits < R ? 2 : first + n_splits < R ? 1 : 0;         // 2^sh rows at a time
        const int P = SUBS >> sh, rl = sub & ((1 << sh) - 1), sp0 = sub >> sh;
        for (int rr0 = first; rr0 < R; rr0 += n_splits << sh) {
            const bool live = rr0 + rl * n_splits < R;
            const int rr = live ? rr0 + rl * n_splits : rr0;
            const int m = m_first + rr % q_len, head = kvh * G + rr / q_len;
            const int base = ((m * H + head) * n_splits) * PC;
            float mm = -INFINITY, o = 0.f, l = 0.f;
            for (int s0 = live ? sp0 : n_splits; s0 < n_splits; s0 += MU * P) {
                u32x2 co[MU];
                u32x4 cml[MU];
                unsigned spins = 0;
                while (true) {
                    asm volatile("" ::: "memory");      // the cells change under our feet: every round reads memory again
                    bool ok = true;
#pragma unroll
                    for (int u = 0; u < MU; ++u) {
                        const int sp = min(s0 + u * P, n_splits - 1);       // past the end: the last split again, ignored below
                        co[u] = ld_cell1(bc, base + sp * PC + d);
                        cml[u] = ld_cells2(bc, base + sp * PC + HD);
                    }
#pragma unroll
                    for (int u = 0; u < MU; ++u) ok = ok && co[u].y == mg.flag && cml[u].y == mg.flag && cml[u].w == mg.flag;
                    if (ok) break;
                    if (++spins > mg.spin_limit) { atomicOr(mg.status, 16); break; }
                }
                float gm = mm;
#pragma unroll
                for (int u = 0; u < MU; ++u)
                    if (s0 + u * P < n_splits) gm = fmaxf(gm, __uint_as_float(cml[u].x));
                if (gm == -INFINITY) continue;
                const float keep = __expf(mm - gm);     // 0 when nothing was accumulated yet
                o *= keep; l *= keep;
#pragma unroll
                for (int u = 0; u < MU; ++u) {
                    const float mv = __uint_as_float(cml[u].x);
                    if (s0 + u * P >= n_splits || mv == -INFINITY) continue;
                    const float f = __expf(mv - gm);
                    l += __uint_as_float(cml[u].z) * f;
                    o += __uint_as_float(co[u].x) * f;
                }
                mm = gm;
            }
            if (P > 1) {                             // the shares of a row meet in LDS
                __syncthreads();                     // wo / wm / wl are free again
                wo[sub][0][d] = o;
                if (d == 0) { wm[sub][0] = mm; wl[sub][0] = l; }
                __syncthreads();
                float gm = wm[rl][0];
                for (int p = 1; p < P; ++p) gm = fmaxf(gm, wm[rl + (p << sh)][0]);
                o = l = 0.f;
                for (int p = 0; p < P; ++p) {        // what share 0 stores
                    const float mv = wm[rl + (p << sh)][0], f = (mv == -INFINITY) ? 0.f : __expf(mv - gm);
                    o += wo[rl + (p << sh)][0][d] * f;
                    l += wl[rl + (p << sh)][0] * f;
                }
            }
            if (live && sp0 == 0)
                Act<uint16_t>::store(mg.out, mg.plane, mg.tiled ? xt_index(m, head * HD + d, mg.tiled) : ((size_t)m * H + head) * HD + d,
                                     l > 0.f ? o / l : 0.f);
        }
    }
}

// grid (M*H), threads hd: combine the splits, normalise, store in the storage dtype.  One pass: the (max, sum, o) of
// 16 splits are requested together and folded into a running (max, sum, o) -- the partials were written by other dies
// a moment ago, so every dependent round of loads is a trip to memory.
// PARTS: parts[b] of a sequence's n_splits partials are there, the others hold anything (seq_rows of the grid are one sequence); where
// there is only one the output is there, too.
template <typename T, bool PARTS>
__global__ void attn_merge_kernel(const float* __restrict__ part, int n_splits, int hd, size_t plane, void* __restrict__ out, int tiled_H, int tiled_R,
                                  const int32_t* __restrict__ parts, int seq_rows) {
    const size_t mh = blockIdx.x;
    const int d = threadIdx.x;
    const size_t pstride = (size_t)hd + 4;       // o[hd], max, sum, 2 pad: rows stay 16-byte aligned
    const float* base = part + mh * n_splits * pstride;
    const int used = PARTS ? parts[blockIdx.x / seq_rows] : n_splits;      // asked for together with the first partials
    float mm = -INFINITY, o = 0.f, l = 0.f;
    for (int s0 = 0; s0 < n_splits; s0 += 16) {
        float mv[16], lv[16], ov[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const float* ps = base + (size_t)min(s0 + u, n_splits - 1) * pstride;
            mv[u] = ps[hd]; lv[u] = ps[hd + 1]; ov[u] = ps[d];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (s0 + u >= used) mv[u] = -INFINITY;
        float gm = mm;
#pragma unroll
        for (int u = 0; u < 16; ++u) gm = fmaxf(gm, mv[u]);
        if (gm == -INFINITY) continue;
        const float keep = __expf(mm - gm);       // 0 when nothing was accumulated yet
        o *= keep; l *= keep;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const float f = (mv[u] == -INFINITY) ? 0.f : __expf(mv[u] - gm);
            if (f == 0.f) continue;               // an empty split's o[] was never written
            l += lv[u] * f;
            o += ov[u] * f;
        }
        mm = gm;
    }
    if (PARTS && used == 1) return;
    // tiled_H > 0: planes of tiled_R rows in the layout of the whole-K projections (xt_index), row = mh / H, column = (mh % H) * hd + d
    const size_t idx = tiled_H > 0 ? xt_index((int)(mh / tiled_H), (int)(mh % tiled_H) * hd + d, tiled_R) : mh * hd + d;
    Act<T>::store(out, plane, idx, l > 0.f ? o / l : 0.f);
}

// ---- launchers -----------------------------------------------------------------------------------
int launch_prep(const int32_t* q_tokens, int q_stride, const int32_t* kv_len, int kv_base, int B, int q_len,
                int max_len, int V, int hd, float rope_base, int32_t* pos, int32_t* tok, float2* rope,
                int32_t* status, void* clear, size_t clear_bytes, const AttnParts& ap, hipStream_t s) {
    const int threads = q_len > 16 ? 1024 : 128;
    const size_t clear16 = clear_bytes / 16;
    // one clearing block per 32 KiB, at most 512 (a few MB of attention cells: two or three sweeps per lane)
    int extra = (int)((clear_bytes + 32767) / 32768);
    if (extra > 512) extra = 512;
    hipLaunchKernelGGL(prep_kernel, dim3(B * ((q_len + PREP_ROWS - 1) / PREP_ROWS) + extra), dim3(threads), 0, s, q_tokens, q_stride, kv_len, kv_base, q_len, max_len, V,
                       hd / 2, rope_base, pos, tok, rope, status, B, reinterpret_cast<uint4*>(clear), clear16, ap);
    BS_LAUNCH_CHECK();
    return BS_OK;
}

int launch_embed_dec(const int32_t* tok, const void* embed, const float* gain, int M, int d, float* x, void* planes,
                     size_t plane, float* ssq, hipStream_t s) {
    hipLaunchKernelGGL(embed_dec_kernel, dim3(M), dim3(256), 0, s, tok, (const uint16_t*)embed, gain, d, x, (uint16_t*)planes, plane, ssq);
    BS_LAUNCH_CHECK();
    return BS_OK;
}

// LDS the fused few-row projection needs for its activations; it fits next to the 8 KiB reduction buffer
// inside the 64 KiB a workgroup may use.
static size_t dec_lds_bytes(int M, int K) { return (size_t)2 * M * (K + 8) * 2; }
bool gemm_dec_fits(int M, int K) { return M >= 1 && M <= DEC_MAX_ROWS && K % 32 == 0 && dec_lds_bytes(M, K) <= 56 * 1024; }

int launch_gemm_dec(int epi, const DecArgs& a, hipStream_t s) {
    BS_REQUIRE(gemm_dec_fits(a.M, a.K), BS_ESHAPE, "gemm_dec: %d rows x %d columns of activations do not fit LDS", a.M, a.K);
    BS_REQUIRE(a.M >= 1 && a.M <= 16 && a.K % 32 == 0 && a.N % 16 == 0 && a.K >= 32, BS_ESHAPE, "gemm_dec: M=%d N=%d K=%d", a.M, a.N, a.K);
    BS_REQUIRE((double)a.N * a.K * 2.0 < 4294967296.0 && (double)a.M * a.K * 2.0 < 4294967296.0, BS_ESHAPE,
               "gemm_dec: a matrix of %d x %d exceeds the 32-bit byte offsets of this kernel", a.N, a.K);
    BS_REQUIRE(!a.att_part || (epi == EPI_RESID && a.att_splits >= 1 && (a.hd == 64 || a.hd == 128) && a.K == a.H * a.hd), BS_ESHAPE,
               "gemm_dec: attention partials as input need the O projection's shape (K = %d, H = %d, hd = %d)", a.K, a.H, a.hd);
    BS_REQUIRE(epi != EPI_QKV || (a.hd % 16 == 0 && a.seg_rows[0] % 16 == 0 && a.seg_rows[1] % 16 == 0), BS_ESHAPE, "gemm_dec: head_dim %d", a.hd);
    const int steps = a.K / 32;
    // wavefronts per 16-column tile: about six k steps each, 4 or 8 of them; the gate/up pair takes 4 + 4
    int W = (epi == EPI_SWIGLU) ? 8 : (steps >= 48 ? 8 : 4);
    const bool deep = steps / (epi == EPI_SWIGLU ? 4 : W) > 4;      // ring of 8 unless a wavefront has at most 4 steps
    const dim3 grid(a.N / 16), block(64 * W);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    { const int prc = prof_events(s, &e0, &e1); if (prc != BS_OK) return prc; }
    const size_t lds = dec_lds_bytes(a.M, a.K);
#define BS_DEC(E, MG) do { if (deep) BS_LAUNCH_TIMED((gemm_dec_kernel<E, 8, MG>), grid, block, lds, s, e0, e1, a); \
                           else BS_LAUNCH_TIMED((gemm_dec_kernel<E, 4, MG>), grid, block, lds, s, e0, e1, a); } while (0)
    if (epi == EPI_RESID && a.att_part) BS_DEC(EPI_RESID, true);
    else if (epi == EPI_RESID) BS_DEC(EPI_RESID, false);
    else if (epi == EPI_QKV) BS_DEC(EPI_QKV, false);
    else BS_DEC(EPI_SWIGLU, false);
#undef BS_DEC
    BS_LAUNCH_CHECK();
    prof_record(e0, e1, (double)a.N * (double)a.K * 2.0 * (epi == EPI_SWIGLU ? 2.0 : 1.0), 50);   // class 50: fused few-row projections
    return BS_OK;
}

// The fused projections for up to 32 rows: how many units (16-column tiles of the stacked QKV matrices; gate/up pairs)
// a workgroup gets at most, 0 when the kernel does not apply.  *grid: workgroups (one per compute unit at most).
int gemm_rows_units(int epi, int M, int N, int K, int* grid) {
    if (epi != EPI_QKV && epi != EPI_SWIGLU && epi != EPI_RESID) return 0;
    if (M < 1 || M > ROWS_MAX || K < 32 || K % 32 != 0 || N < 16 || N % 16 != 0) return 0;
    if ((double)N * K * 2.0 >= 4294967296.0 || (double)M * K * 2.0 >= 4294967296.0) return 0;
    const int cus = step_grid();
    if (cus < 8) return 0;
    const int units = N / 16, G = units < cus ? units : cus;
    const int tu = (units + G - 1) / G;
    if (tu > (epi == EPI_SWIGLU ? ROWS_UMAX - 1 : ROWS_UMAX)) return 0;       // at most six weight tiles in flight per wavefront
    if (grid) *grid = G;
    return tu;
}

int launch_gemm_rows(int epi, const DecArgs& a, bool stream, hipStream_t s) {
    int G = 0;
    const int tu = gemm_rows_units(epi, a.M, a.N, a.K, &G);
    BS_REQUIRE(tu >= 1, BS_ESHAPE, "gemm_rows: M=%d N=%d K=%d", a.M, a.N, a.K);
    BS_REQUIRE(epi != EPI_QKV || ((a.hd == 64 || a.hd == 128) && a.seg_rows[0] % 16 == 0 && a.seg_rows[1] % 16 == 0 && a.q_len >= 1), BS_ESHAPE,
               "gemm_rows: head_dim %d", a.hd);
    BS_REQUIRE(epi == EPI_RESID || (a.ssq_in && a.ssq_tiles >= 1), BS_EINVAL, "gemm_rows: the input rows' sums of squares are missing");
    BS_REQUIRE(epi != EPI_RESID || (a.x && (!a.gain_next || a.out_planes)), BS_EINVAL, "gemm_rows: residual or output planes missing");
    BS_REQUIRE(epi != EPI_SWIGLU || (a.out_planes && a.w[0] && a.w[1]), BS_EINVAL, "gemm_rows: gate/up matrices or output planes missing");
    BS_REQUIRE(epi != EPI_QKV || (a.q_out && a.k_cache && a.v_cache && a.pos && a.rope), BS_EINVAL, "gemm_rows: QKV outputs or positions missing");
    BS_REQUIRE(a.xh && a.w[0], BS_EINVAL, "gemm_rows: input planes or weights missing");
    const int units = a.N / 16;
    const dim3 grid(G), block(512);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    { const int prc = prof_events(s, &e0, &e1); if (prc != BS_OK) return prc; }
#define BS_ROWS_MT(E, MT, ST) do { switch (tu) { \
        case 1: BS_LAUNCH_TIMED((gemm_rows_kernel<E, 1, MT, ST>), grid, block, 0, s, e0, e1, a, units); break; \
        case 2: BS_LAUNCH_TIMED((gemm_rows_kernel<E, 2, MT, ST>), grid, block, 0, s, e0, e1, a, units); break; \
        case 3: BS_LAUNCH_TIMED((gemm_rows_kernel<E, 3, MT, ST>), grid, block, 0, s, e0, e1, a, units); break; \
        default: BS_LAUNCH_TIMED((gemm_rows_kernel<E, E == EPI_SWIGLU ? 3 : 4, MT, ST>), grid, block, 0, s, e0, e1, a, units); break; } } while (0)
#define BS_ROWS(E) do { if (a.M <= 16) { if (stream) BS_ROWS_MT(E, 1, true); else BS_ROWS_MT(E, 1, false); } \
                        else { if (stream) BS_ROWS_MT(E, 2, true); else BS_ROWS_MT(E, 2, false); } } while (0)
    if (epi == EPI_QKV) BS_ROWS(EPI_QKV); else if (epi == EPI_SWIGLU) BS_ROWS(EPI_SWIGLU); else BS_ROWS(EPI_RESID);
#undef BS_ROWS_MT
#undef BS_ROWS
    BS_LAUNCH_CHECK();
    prof_record(e0, e1, (double)a.N * (double)a.K * 2.0 * (epi == EPI_SWIGLU ? 2.0 : 1.0), 60);   // class 60: fused projections, up to 32 rows
    return BS_OK;
}

int norm_chunks(int d) { return (d + 1023) / 1024; }

int launch_embed(int dtype, const int32_t* tok, const void* embed, int M, int d, float* x, hipStream_t s) {
    if (dtype == BS_BF16)
        hipLaunchKernelGGL((embed_kernel<uint16_t>), dim3(M), dim3(256), 0, s, tok, (const uint16_t*)embed, d, x);
    else
        hipLaunchKernelGGL((embed_kernel<float>), dim3(M), dim3(256), 0, s, tok, (const float*)embed, d, x);
    BS_LAUNCH_CHECK();
    return BS_OK;
}

int launch_rmsnorm(int dtype, float* x, const float* pend, int pend_ks, size_t pend_stride, const float* gain, int d,
                   float eps, int n_seq, int rows_in, int rows_out, size_t plane, void* out, int tiled, hipStream_t s) {
    const int rows = n_seq * rows_out;
    if (rows <= 0) return BS_OK;
    if (dtype == BS_BF16)
        hipLaunchKernelGGL((rmsnorm_kernel<uint16_t>), dim3(rows), dim3(1024), 0, s, x, pend, pend_ks, pend_stride, gain, d, eps, rows_in, rows_out, plane, out, tiled);
    else
        hipLaunchKernelGGL((rmsnorm_kernel<float>), dim3(rows), dim3(1024), 0, s, x, pend, pend_ks, pend_stride, gain, d, eps, rows_in, rows_out, plane, out, tiled);
    BS_LAUNCH_CHECK();
    return BS_OK;
}

int launch_resid_sum(float* x, const float* pend, int pend_ks, size_t pend_stride, const float* gain, int d, int rows,
                     size_t plane, void* out, float* ssq, int tiled, hipStream_t s) {
    if (rows <= 0) return BS_OK;
    BS_REQUIRE(!tiled || (rows <= tiled && d % 32 == 0), BS_ESHAPE, "resid_sum: tiled planes hold at most %d rows (%d) of a multiple of 32 columns (%d)", tiled, rows, d);
    // up to 8 splits in flight
#define BS_RESID(AHEAD) hipLaunchKernelGGL(resid_sum_kernel<AHEAD>, dim3(rows, norm_chunks(d)), dim3(256), 0, s, x, pend, pend_ks, pend_stride, gain, d, plane, \
                                           (uint16_t*)out, ssq, tiled)
    if (!pend || pend_ks <= 4) BS_RESID(4);
    else BS_RESID(8);
#undef BS_RESID
    BS_LAUNCH_CHECK();
    return BS_OK;
}

int launch_swiglu(int dtype, const float* part, int ks, size_t ks_stride, int M, int ff, size_t plane, void* out, int tiled,
                  const float* ssq, int ssq_n, int d, float eps, hipStream_t s) {
    const size_t n = (size_t)M * ff;
    const dim3 grid((unsigned)((n + 255) / 256)), block(256);
    const float inv_d = 1.0f / (float)d;
    if (dtype == BS_BF16) hipLaunchKernelGGL((swiglu_kernel<uint16_t>), grid, block, 0, s, part, ks, ks_stride, M, ff, plane, out, tiled, ssq, ssq_n, inv_d, eps);
    else hipLaunchKernelGGL((swiglu_kernel<float>), grid, block, 0, s, part, ks, ks_stride, M, ff, plane, out, tiled, ssq, ssq_n, inv_d, eps);
    BS_LAUNCH_CHECK();
    return BS_OK;
}

int launch_rope_kv(int dtype, const float* part, int ks, size_t ks_stride, const int32_t* pos, const float2* rope, int M,
                   int q_len, int H, int KVH, int hd, int max_len, float* q_out, void* k_cache, void* v_cache,
                   const float* ssq, int ssq_n, int d, float eps, hipStream_t s) {
    const dim3 grid(M, H + 2 * KVH), block(hd / 2);
    const float inv_d = 1.0f / (float)d;
    if (dtype == BS_BF16)
        hipLaunchKernelGGL((rope_kv_kernel<uint16_t>), grid, block, 0, s, part, ks, ks_stride, pos, rope, q_len, H, KVH, hd,
                           max_len, q_out, (uint16_t*)k_cache, (uint16_t*)v_cache, ssq, ssq_n, inv_d, eps);
    else
        hipLaunchKernelGGL((rope_kv_kernel<float>), grid, block, 0, s, part, ks, ks_stride, pos, rope, q_len, H, KVH, hd,
                           max_len, q_out, (float*)k_cache, (float*)v_cache, ssq, ssq_n, inv_d, eps);
    BS_LAUNCH_CHECK();
    return BS_OK;
}

// The fused fp32 projections read a matrix once per four rows, from the second time on out of the memory-side cache if it fits there (256 MB).  Against a
// kernel per step: 128 to 1536 columns, 1 to 1024 rows a pass 1.1 to 1.5 times as fast, 2048 columns 1.2 (4 rows) to 1.04 (1024 rows), 4096 columns
// 1.27 up to 40 rows; from 48 rows on gemm_f32_kernel's groups of eight beat them there (48 rows 1551 us against 1752, 1024 rows 28.5 against
// 36.2 ms), whose gate and up matrices are 360 MB.  By a matrix alone, passes of one layer and the LM head of 64 to 131 million elements, kernel per
// step -> fused: 131 million, 32 rows 1091 -> 985 us, 48 rows 1115 -> 1465, 512 rows 9.4 -> 15.4 ms; 66 million, 64 rows 644 -> 628 us, 192 rows 1881 -> 1870, 256 rows
// 2390 -> 2497, 512 rows 4790 -> 5076; 33 million, 192 rows 1008 -> 1001, 256 rows 1287 -> 1322; 16 million, 512 rows 1256 -> 1249.  QKV, which saves
// the launches around it as well, 50 million in two layers: 64 rows 1560 -> 1369, 256 rows 5330 -> 5166, 512 rows 10212 -> 10300.
static bool f32_fits(int M, size_t elems, int rows) { return M < 48 || elems <= 24000000 || (elems <= (size_t)64 << 20 && M < rows); }
bool f32_fused_applies(int M, int d, int ff, int nqkv, int nq) {
    return M < 48 || ((size_t)d * ff <= 12000000 && f32_fits(M, (size_t)nqkv * d, 512) && f32_fits(M, (size_t)nq * d, 512));
}
bool f32_head_applies(int M, int vocab, int d) { return f32_fits(M, (size_t)vocab * d, 256); }

int launch_f32_fused(int epi, const F32Args& a, hipStream_t s) {
    if (a.M <= 0 || a.N <= 0) return BS_OK;
    BS_REQUIRE(a.x && a.w[0] && a.out && a.K % 8 == 0 && (epi == F32_HEAD || a.N % 2 == 0) && (epi == F32_RESID || a.gain), BS_EINVAL, "f32_fused: M=%d N=%d K=%d", a.M, a.N, a.K);
    BS_REQUIRE(epi != F32_QKV || (a.w[1] && a.w[2] && a.pos && a.rope && a.k_cache && a.v_cache && a.nq + 2 * a.nkv == a.N && a.hd >= 2 && a.q_len >= 1), BS_EINVAL, "f32_fused: QKV arguments");
    BS_REQUIRE(epi != F32_SWIGLU || a.w[1], BS_EINVAL, "f32_fused: up matrix missing");
    BS_REQUIRE(epi != F32_RESID || !a.tok || a.x_old, BS_EINVAL, "f32_fused: residual rows missing");
    const int pairs = epi == F32_SWIGLU ? a.N : (a.N + 1) / 2, groups = (a.M + 3) / 4;
    const dim3 grid((pairs + 3) / 4, groups < 65535 ? groups : 65535), block(256);
    // a caller's LM head and final norm need not be 16-byte aligned (the layers' weights and the activations are)
    const bool vec = ((reinterpret_cast<uintptr_t>(a.w[0]) | reinterpret_cast<uintptr_t>(a.gain)) & 15) == 0;
    if (epi == F32_QKV) hipLaunchKernelGGL((f32_fused_kernel<F32_QKV, true>), grid, block, 0, s, a);
    else if (epi == F32_SWIGLU) hipLaunchKernelGGL((f32_fused_kernel<F32_SWIGLU, true>), grid, block, 0, s, a);
    else if (epi == F32_RESID) hipLaunchKernelGGL((f32_fused_kernel<F32_RESID, true>), grid, block, 0, s, a);
    else if (vec) hipLaunchKernelGGL((f32_fused_kernel<F32_HEAD, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((f32_fused_kernel<F32_HEAD, false>), grid, block, 0, s, a);
    BS_LAUNCH_CHECK();
    return BS_OK;
}

// bytes of the exchange cells through which the key splits of `rows` query rows are combined inside the attention kernel
size_t attn_cells_bytes(int rows, int H, int hd, int n_splits) {
    const double b = (double)rows * H * n_splits * (hd + 4) * 8.0;
    return b < 2147483648.0 ? (size_t)b : 0;           // 32-bit cell offsets
}

// workgroups of the one-tile attention kernel that the device holds at the same time, whichever of its variants runs (launch_attention: by the
// length of a split and by what the pass reads): of the variant with the fewest.  Never more than the 2 and 4 a compute unit of its launch bounds, which are
// also the answer without a device (sizes asked for ahead).
static size_t attn_resident_workgroups(int hd) {
    auto ask = [](int bound, std::initializer_list<const void*> variants) -> size_t {
        const int cus = step_grid();
        if (cus <= 0) return (size_t)device_cus() * bound;
        int least = bound;
        for (const void* kernel : variants) {
            int per_cu = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, 0) != hipSuccess || per_cu < 1) return 1;   // 1: never enough, the merge kernel runs
            if (per_cu < least) least = per_cu;
        }
        return (size_t)least * cus;
    };
#define BS_ONE_TILE(HD) {(const void*)&attn_mfma_kernel<HD, 1, true, true, false>, (const void*)&attn_mfma_kernel<HD, 1, false, true, false>, \
                         (const void*)&attn_mfma_kernel<HD, 1, true, false, false>, (const void*)&attn_mfma_kernel<HD, 1, false, false, false>}
    static const size_t c128 = ask(2, BS_ONE_TILE(128)), c64 = ask(4, BS_ONE_TILE(64));      // asked once (initialisation of a local static is thread-safe)
#undef BS_ONE_TILE
    return hd == 128 ? c128 : c64;
}

// How a pass whose attention leaves the output itself (not the few-row schedule) cuts the keys when it may use up to n_splits parts.
AttnPlan attn_plan(int dtype, int B, int q_len, int H, int KVH, int hd, int cache_len, int n_splits) {
    AttnPlan p = {n_splits, n_splits, 0, false};
    if (dtype != BS_BF16 || n_splits <= 1) return p;
    if (attn_prompt_applies(B, q_len, H, KVH, hd)) { p.splits = p.most = 1; return p; }
    const int n_tiles = (H / KVH * q_len + 15) / 16, n_rt = n_tiles >= 2 ? (n_tiles + 1) / 2 : 1, cus = device_cus();
    if (n_tiles >= 2) {
        // Two row tiles a wavefront: one workgroup per group of two and only as many key splits as it takes to reach about a
        // thousand workgroups; a single group keeps all the splits.
        const int want = (int)((4 * cus + (long long)B * KVH * n_rt - 1) / ((long long)B * KVH * n_rt));
        if (n_rt > 1 && want < n_splits) p.splits = p.most = want;
        return p;
    }
    // One row tile: fewer splits than asked for where that is no slower.
    const long long units = (long long)B * KVH;
    const int rows = B * q_len;
    // Combined in the kernel: 3 to 16 rows whose workgroups all fit on the device, counted with the splits asked for, so that a pass of
    // a batch, which may share the device with another stream's, does not come to wait for its own workgroups by being cut less.
    p.in_kernel = rows > DEC_MAX_ROWS && rows <= ATTN_CELL_ROWS && units * n_splits <= (long long)attn_resident_workgroups(hd) &&
                  attn_cells_bytes(rows, H, hd, n_splits) > 0;
    const double unit_mb = 4e-6 * hd * cache_len, merge_us = 4.6 + 8e-4 * rows * H;
    if (hd != 128) {
        // head_dim 64, 4 workgroups per compute unit resident: the fewest splits with the least rounds of 1024 workgroups per split (16
        // sequences of 4097 keys, 12 heads: 6 splits, 1152 workgroups, 36.5 us; 5 splits 35.2; two or fewer workgroups per compute
        // unit have too little in flight: 9 sequences of 8000 keys, 2 splits, a whole pass 8 % longer than with 9).
        const int round = 4 * cus;
        for (int s = n_splits - 1; s >= 1; --s)
            if ((units * s + round - 1) / round * p.splits <= (units * p.splits + round - 1) / round * s) p.splits = s;
    } else {
        // head_dim 128: the least estimated time.  A compute unit streams about 30 KB/us whether it holds one workgroup or two, so what counts
        // is how evenly the workgroups fall on the compute units; all of them together get 6.4 TB/s, and the two bounds add like
        // fourth powers.  Partials and a merge kernel cost 5 us at 20 rows of 32 heads, 8 at 144, and 2 more where workgroups share compute
        // units; combined in the kernel, 0.5 us and 1.55 for each row of a workgroup's share (fitted when it took them one after
        // the other; two at a time cost less, which moves no count of a pass by more than its noise).  16 sequences of 4105 keys, 32 heads: 2 splits 178.6 + 8.5 us, 1 split
        // 168.0.  Whole passes of the 7B shape: 6 sequences of 3007 keys, 1 / 2 / 3 / 4 / 5 splits 6240 / 6505 / 6627 / 6408 / 6596 us;
        // 10 of 6004 keys, 1 / 2 / 3 / 4 splits 11281 / 10266 / 9831 / 9760; 4 of 2053 keys 4378 / 4128 / 4267 / 4158.  Eight layers of it, one
        // sequence, splits combined in the kernel, cache of 900: 3 rows, 1 / 2 splits 781 / 761 us, 5 rows 788 / 782, 9 rows 821 / 836; of 1280:
        // 9 rows, 1 / 2 / 3 splits 858 / 850 / 813, 16 rows 931 / 962 / 911; of 8192: 9 rows, 4 / 6 / 8 / 16 splits 995 / 928 / 894 / 924; 3 sequences
        // of 5 rows, cache of 1280: 927 / 894 / 921.  With a merge kernel: 2 sequences of 9 rows, cache of 600, 1 / 2 splits 926 / 932, of 900 955 / 943;
        // 3 of 6 rows, of 2304, 2 / 5 splits 1024 / 1011; 6 of 5 rows, of 2304, 1 / 4 splits 1227 / 1240.  More splits than that only for a tenth of the estimate.
        const double f = units * unit_mb / 6.4;
        const int group_rows = H / KVH * q_len;
        double best_us = 1e30;
        for (int s = 1; s <= n_splits; ++s) {
            const double c = (double)((units * s + cus - 1) / cus) / s * unit_mb / 0.030;
            const double combine_us = s == 1 ? 0.0 : p.in_kernel ? 0.5 + 1.55 * ((group_rows + s - 1) / s) : merge_us + (units * s > cus ? 2.0 : 0.0);
            const double us = sqrt(sqrt(c * c * c * c + f * f * f * f)) + combine_us;
            if (us < (p.in_kernel ? 0.9 : 0.999) * best_us) { p.splits = s; best_us = us; }
        }
    }
    p.in_kernel = p.in_kernel && p.splits > 1;
    // That is for sequences of about one length.  One that is much longer than the others would end alone, so it is cut into more
    // parts, up to what was asked for (prep_kernel, by the lengths on the device), where that saves it 6 us or, if the others are not cut
    // and its last workgroup has to combine them, twice what that costs.  (The way over the items costs batches of one length up to
    // 1 us a launch: four layers of the 8B's draft, 12 x 2 rows at 3000 keys, 5 splits or up to 7: 304 -> 308 us a pass.)
    const double saved_us = unit_mb / 0.030 * (1.0 / p.splits - 1.0 / n_splits);
    const bool worth = p.splits > 1 ? saved_us > 6.0 : saved_us > 2.0 * (0.5 + 1.55 * (H / KVH) * q_len) && attn_cells_bytes(rows, H, hd, n_splits) > 0;
    p.most = rows > DEC_MAX_ROWS && B < 65536 && !p.in_kernel && worth ? n_splits : p.splits;
    const long long spare = units * (p.most - p.splits), room = cus;           // a long sequence's parts are at most its share of the compute units
    p.n_items = B * p.splits + (int)((spare < room ? spare : room) / KVH);
    return p;
}

int launch_attention(int dtype, const float* q, const void* k_cache, const void* v_cache, const int32_t* pos, int B,
                     int q_len, int H, int KVH, int hd, int max_len, int n_splits, float* part, size_t plane, void* out,
                     int out_tiled, const AttnCells* cells, const AttnParts* ap, bool stream, hipStream_t s) {
    BS_REQUIRE(!out_tiled || (dtype == BS_BF16 && out && B * q_len <= out_tiled), BS_ESHAPE, "attention: tiled output planes hold at most %d rows", out_tiled);
    const float scale = 1.0f / sqrtf((float)hd);
    const dim3 block(256);
    if (dtype == BS_BF16 && out && (!out_tiled || out_tiled > ROWS_MAX) && attn_prompt_applies(B, q_len, H, KVH, hd))
        return launch_attn_prompt(q, reinterpret_cast<const uint16_t*>(k_cache), reinterpret_cast<const uint16_t*>(v_cache), pos, B, q_len, H, KVH, hd,
                                  max_len, reinterpret_cast<uint16_t*>(out), plane, out_tiled, s);
    if (dtype == BS_BF16) {
        const int n_tiles = (H / KVH * q_len + 15) / 16;
        // two tiles per wavefront as soon as there are two: a K or V block then serves 32 rows (verification with grouped
        // queries: 287 -> 225 us per layer at batch 32 / 8192 keys; prompt chunks of a batch: 7-10 % off the prompt pass)
        const int nt = (n_tiles >= 2) ? 2 : 1;
        const int n_rt = (n_tiles + nt - 1) / nt;
        const AttnPlan plan = attn_plan(dtype, B, q_len, H, KVH, hd, max_len, n_splits);
        const int few = out ? plan.splits : n_splits;              // of a sequence about as long as the others
        if (out) n_splits = plan.most;
        if (few == n_splits) ap = nullptr;
        BS_REQUIRE(few == n_splits || (ap && ap->parts && ap->items && (hd == 64 || hd == 128) && nt == 1 && ap->few == few && ap->most == n_splits), BS_EINVAL, "attention: the work items are missing");
        const dim3 mgrid = ap ? dim3(KVH, ap->n_items) : dim3(n_splits * (out ? n_rt : 1), KVH, B);
        uint16_t* direct = (out && few == 1) ? reinterpret_cast<uint16_t*>(out) : nullptr;          // of one part: the output itself
        // the splits combined inside the kernel: one row tile, exchange cells at hand, every workgroup resident at once
        AttnMerge mg = {};
        mg.tiled = out_tiled;
        if (cells && cells->buf && out && (plan.in_kernel || (ap && few == 1))) {
            const size_t need = attn_cells_bytes(B * q_len, H, hd, n_splits);
            BS_REQUIRE(need + (ap ? (size_t)B * KVH * 4 : 0) <= cells->bytes, BS_EWORKSPACE, "attention: %zu bytes of exchange cells", cells->bytes);
            if (ap) mg.tickets = reinterpret_cast<unsigned*>(reinterpret_cast<char*>(cells->buf) + need);
            mg.cells = cells->buf; mg.out = reinterpret_cast<uint16_t*>(out); mg.plane = plane;
            mg.flag = cells->flag; mg.spin_limit = cells->spin_limit; mg.status = cells->status;
        }
        hipEvent_t e0 = nullptr, e1 = nullptr;
        { const int prc = prof_events(s, &e0, &e1); if (prc != BS_OK) return prc; }
        // with several groups of row tiles every group reads the keys again: those loads stay cached
        stream = stream && n_rt == 1;
#define BS_ATTN_ST(HD, NT, ST, AH, PT) BS_LAUNCH_TIMED((attn_mfma_kernel<HD, NT, ST, AH, PT>), mgrid, block, 0, s, e0, e1, q, (const uint16_t*)k_cache, \
                                        (const uint16_t*)v_cache, pos, q_len, H, KVH, max_len, scale, part, n_splits, direct, plane, mg, ap ? ap->items : nullptr)
#define BS_ATTN(HD, NT, AH, PT) do { if (stream) BS_ATTN_ST(HD, NT, true, AH, PT); else BS_ATTN_ST(HD, NT, false, AH, PT); } while (0)
#define BS_ATTN_1(HD, PT) do { if (ahead) BS_ATTN(HD, 1, true, PT); else BS_ATTN(HD, 1, false, PT); } while (0)
        const bool ahead = max_len / few >= 768;              // six blocks and more per wavefront of a full cache
        if (ap) { if (hd == 128) BS_ATTN_1(128, true); else BS_ATTN_1(64, true); }
        else if (hd == 128) { if (nt == 2) BS_ATTN(128, 2, false, false); else BS_ATTN_1(128, false); }
        else if (hd == 64) { if (nt == 2) BS_ATTN(64, 2, false, false); else BS_ATTN_1(64, false); }
        else
            BS_FAIL(BS_ESHAPE, "attention: bf16 caches need head_dim 64 or 128, got %d", hd);
#undef BS_ATTN_1
#undef BS_ATTN_ST
#undef BS_ATTN
        BS_LAUNCH_CHECK();
        prof_record(e0, e1, 0.0, 100);                     // class 100: the split attention kernel (bytes known to the caller)
        if (out && n_splits > 1 && !mg.cells) {
            if (ap)
                hipLaunchKernelGGL((attn_merge_kernel<uint16_t, true>), dim3(B * q_len * H), dim3(hd), 0, s, part, n_splits, hd, plane, out, out_tiled ? H : 0, out_tiled, ap->parts, q_len * H);
            else
                hipLaunchKernelGGL((attn_merge_kernel<uint16_t, false>), dim3(B * q_len * H), dim3(hd), 0, s, part, n_splits, hd, plane, out, out_tiled ? H : 0, out_tiled, (const int32_t*)nullptr, 1);
        }
    } else {
        float* direct = n_splits == 1 ? reinterpret_cast<float*>(out) : nullptr;
        const dim3 grid(n_splits * ((q_len + ATT_RB - 1) / ATT_RB), H, B);
        const bool few = max_len <= 512 && (long long)grid.x * H * B <= device_cus();       // SHORT, see there
        if (few) hipLaunchKernelGGL((attn_kernel<float, true>), grid, block, 0, s, q, (const float*)k_cache, (const float*)v_cache, pos, q_len, H, KVH, hd, max_len, scale, n_splits, part, direct);
        else hipLaunchKernelGGL((attn_kernel<float, false>), grid, block, 0, s, q, (const float*)k_cache, (const float*)v_cache, pos, q_len, H, KVH, hd, max_len, scale, n_splits, part, direct);
        BS_LAUNCH_CHECK();
        if (n_splits > 1) hipLaunchKernelGGL((attn_merge_kernel<float, false>), dim3(B * q_len * H), dim3(hd), 0, s, part, n_splits, hd, plane, out, out_tiled ? H : 0, out_tiled, (const int32_t*)nullptr, 1);
    }
    BS_LAUNCH_CHECK();
    return BS_OK;
}

}  // namespace bs
