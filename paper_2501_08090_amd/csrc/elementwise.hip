// Bandwidth-bound kernels of the decode step: what begins it (embedding gather, rotary table, attention work list), RMSNorm, rotary embedding,
// KV append / gather (the slot contract), and small utilities.  gfx950, wave64.
#include <climits>

#include "attn_plan.h"
#include "kv_layout.h"

namespace chiron {

// ---- RMSNorm: one workgroup per row, row held in registers, wavefront + LDS reduction -------------------
// Also the place where a K-sliced projection into the residual stream is summed: h += sum_s part[s].  The
// slice loads of a thread are independent, so they are issued four at a time.
template <int THREADS, int VPT>  // float4 vectors per thread; covers n <= THREADS*4*VPT
__global__ __launch_bounds__(THREADS) void rmsnorm_kernel(float* __restrict__ h, const float* __restrict__ part, int ks,
                                                          size_t part_stride, const uint16_t* __restrict__ gain, int n,
                                                          float eps, float* __restrict__ out) {
    __shared__ float red[THREADS / 64];
    float* row = h + (size_t)blockIdx.x * n;
    const float* prow = part + (size_t)blockIdx.x * n;
    float* orow = out + (size_t)blockIdx.x * n;
    float4 v[VPT];
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        int j = (i * THREADS + threadIdx.x) * 4;
        if (j < n) {
            v[i] = *reinterpret_cast<const float4*>(row + j);
            if (ks > 0) {
                int s = 0;
                for (; s + 4 <= ks; s += 4) {
                    float4 t[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) t[u] = *reinterpret_cast<const float4*>(prow + (size_t)(s + u) * part_stride + j);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        v[i].x += t[u].x; v[i].y += t[u].y; v[i].z += t[u].z; v[i].w += t[u].w;
                    }
                }
                for (; s < ks; ++s) {
                    float4 t = *reinterpret_cast<const float4*>(prow + (size_t)s * part_stride + j);
                    v[i].x += t.x; v[i].y += t.y; v[i].z += t.z; v[i].w += t.w;
                }
                *reinterpret_cast<float4*>(row + j) = v[i];
            }
            ss += v[i].x * v[i].x + v[i].y * v[i].y + v[i].z * v[i].z + v[i].w * v[i].w;
        }
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int k = 0; k < THREADS / 64; ++k) tot += red[k];
    float inv = 1.0f / sqrtf(tot / (float)n + eps);
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        int j = (i * THREADS + threadIdx.x) * 4;
        if (j < n) {
            uint2 g = *reinterpret_cast<const uint2*>(gain + j);
            float4 o;
            o.x = v[i].x * inv * bf16_lo(g.x);
            o.y = v[i].y * inv * bf16_hi(g.x);
            o.z = v[i].z * inv * bf16_lo(g.y);
            o.w = v[i].w * inv * bf16_hi(g.y);
            *reinterpret_cast<float4*>(orow + j) = o;
        }
    }
}

int32_t launch_rmsnorm(float* h, const float* part, int ks, const uint16_t* gain, int rows, int n, float eps, float* out,
                       hipStream_t st) {
    if (rows == 0) return CHIRON_OK;
    if (n % 4 != 0 || n > 16384) return fail(CHIRON_ERR_SHAPE, "rmsnorm: n=%d must be a multiple of 4, <= 16384", n);
    size_t ps = (size_t)rows * n;
    if (n <= 1024) launch(rmsnorm_kernel<256, 1>, dim3(rows), dim3(256), st, h, part, ks, ps, gain, n, eps, out);
    else if (n <= 4096) launch(rmsnorm_kernel<1024, 1>, dim3(rows), dim3(1024), st, h, part, ks, ps, gain, n, eps, out);
    else if (n <= 8192) launch(rmsnorm_kernel<1024, 2>, dim3(rows), dim3(1024), st, h, part, ks, ps, gain, n, eps, out);
    else launch(rmsnorm_kernel<1024, 4>, dim3(rows), dim3(1024), st, h, part, ks, ps, gain, n, eps, out);
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

// ---- rotary table: fp64 angle and trigonometry, once per step -------------------------------------------
__device__ __forceinline__ void rope_table_entry(int position, int j, int d, float base, float* __restrict__ c, float* __restrict__ s) {
    const double inv_freq = pow((double)base, -2.0 * (double)j / (double)d);
    double sn, cs;
    sincos((double)position * inv_freq, &sn, &cs);
    *c = (float)cs;
    *s = (float)sn;
}

__global__ void rope_table_kernel(const int32_t* __restrict__ pos, int rows, int d, float base, float* __restrict__ cos_t,
                                  float* __restrict__ sin_t) {
    int half = d / 2;
    int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= rows * half) return;
    rope_table_entry(pos[idx / half], idx % half, d, base, cos_t + idx, sin_t + idx);
}

int32_t launch_rope_table(const int32_t* pos, int rows, int d, float base, float* cos_t, float* sin_t, hipStream_t st) {
    if (rows == 0) return CHIRON_OK;
    int n = rows * (d / 2);
    launch(rope_table_kernel, dim3((n + 255) / 256), dim3(256), st, pos, rows, d, base, cos_t, sin_t);
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

// ---- what begins a decode step, in one launch: the attention work list (workgroup 0), the embedding gather
// h[i] = E[tokens[i]] widened to fp32, and the rotary table of every row's position.  All three are bounded by latency (a
// few microseconds each, of which a launch of its own is most); together they take as long as the longest of them.
// Measured against three launches and a work list built request by request: four layers at the 8B widths and 64 requests
// 874 -> 862 us, the two-layer toy decoder 81 -> 73 us; the attention entry point, which launches the work list alone,
// 664 -> 646 us at 32 requests of 28k tokens.
__global__ __launch_bounds__(kPlanThreads) void step_begin_kernel(PlanArgs pa, const uint16_t* __restrict__ table,
                                                                  const int32_t* __restrict__ tokens, int rows, int H, int q_len,
                                                                  int embed_blocks, float* __restrict__ h, int d, float base,
                                                                  float* __restrict__ cos_t, float* __restrict__ sin_t) {
    if (blockIdx.x == 0) {
        attn_plan_block(pa);
    } else if (blockIdx.x <= embed_blocks) {
        const int vecs = H / 8;
        const int64_t t = (int64_t)(blockIdx.x - 1) * kPlanThreads + threadIdx.x;
        if (t >= (int64_t)rows * vecs) return;
        const int i = (int)(t / vecs), j = (int)(t - (int64_t)i * vecs) * 8;
        const uint4 v = *reinterpret_cast<const uint4*>(table + (size_t)tokens[i] * H + j);
        float* out = h + (size_t)i * H + j;
        *reinterpret_cast<float4*>(out) = make_float4(bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y));
        *reinterpret_cast<float4*>(out + 4) = make_float4(bf16_lo(v.z), bf16_hi(v.z), bf16_lo(v.w), bf16_hi(v.w));
    } else {
        const int half = d / 2;
        const int64_t t = (int64_t)(blockIdx.x - 1 - embed_blocks) * kPlanThreads + threadIdx.x;
        if (t >= (int64_t)rows * half) return;
        const int r = (int)(t / half);  // token r % q_len of request r / q_len
        rope_table_entry(pa.seq_lens[r / q_len] + r % q_len, (int)(t - (int64_t)r * half), d, base, cos_t + t, sin_t + t);
    }
}

int32_t launch_step_begin(const AttnWorkspace& ws, const int32_t* seq_lens, const int32_t* bt, int max_blocks, const AttnShape& sh,
                          int n_req, int n_kv, const uint16_t* table, const int32_t* tokens, int H, float* h, int d, float base,
                          float* cos_t, float* sin_t, hipStream_t st) {
    PlanArgs pa;
    int32_t rc = attn_plan_args(ws, seq_lens, bt, max_blocks, sh, n_req, n_kv, &pa);
    if (rc) return rc;
    const int rows = n_req * sh.q_len;
    auto blocks = [](int64_t n) { return (int)((n + kPlanThreads - 1) / kPlanThreads); };
    const int eb = blocks((int64_t)rows * (H / 8)), rb = blocks((int64_t)rows * (d / 2));
    launch(step_begin_kernel, dim3(1 + eb + rb), dim3(kPlanThreads), st, pa, table, tokens, rows, H, sh.q_len, eb, h, d, base, cos_t, sin_t);
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

__global__ __launch_bounds__(256) void rope_kernel(float* __restrict__ x, int ldx, int n_heads, int d,
                                                   const float* __restrict__ cos_t, const float* __restrict__ sin_t) {
    int r = blockIdx.x, half = d / 2;
    float* row = x + (size_t)r * ldx;
    for (int e = threadIdx.x; e < n_heads * half; e += 256) {
        int hd = e / half, j = e % half;
        float c = cos_t[r * half + j], s = sin_t[r * half + j];
        float a = row[hd * d + j], b = row[hd * d + j + half];
        row[hd * d + j] = a * c - b * s;
        row[hd * d + j + half] = b * c + a * s;
    }
}

int32_t launch_rope(float* x, int ldx, int n_heads, int d, const float* cos_t, const float* sin_t, int rows,
                    hipStream_t st) {
    if (rows == 0) return CHIRON_OK;
    launch(rope_kernel, dim3(rows), dim3(256), st, x, ldx, n_heads, d, cos_t, sin_t);
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

// ---- KV append and gather (element order: kv_layout.h) -------------------------------------------------------
// Both directions move 16 bytes per lane.  In a K tile 8 dims of a token are one piece.  In a V tile a piece is 4 tokens
// (positions 4q .. 4q+3) of the dims e and e+16, so a lane takes 8 dims and their partners of four tokens, 8 pieces, and
// transposes them in registers.  Copies, bounded by memory: on 8133 tokens of 8 x 128 (33 MB) the append takes
// 21.5 us (3.1 TB/s read and written; 32 us element by element, where the 2-byte accesses were the bound), the gather of a
// third of them 7.8 us (12.7), the append with three gathers 84 -> 46 us.
// A wave of these kernels does the work of eight and more of the element kernels, one dependent load after the other: few
// tokens take longer (8 x 128: append of 71 tokens 8.4 against 3.6 us, of 517, 2.1 MB of K and V, 6.2 against 5.1; gather of 517
// tokens 4.5 against 3.8).  From about 3 MB on they win (2711 tokens of 8 x 64, 5.6 MB: append 7.0 against 8.0, gather 4.8 against 6.0).
constexpr int64_t kVecAppendBytes = 4 << 20, kVecGatherBytes = 3 << 20;  // K and V
static bool by_pieces(const PoolDesc& p, const void* k, const void* v, int64_t n, int64_t from_bytes) {
    return (((uintptr_t)k | (uintptr_t)v) & 15) == 0 && n * p.n_kv * p.d * 4 >= from_bytes;
}
struct VPieces {
    uint4 u[8];  // piece of dim e0 + i: {e0+i: tokens 0,1 | 2,3; e0+16+i: tokens 0,1 | 2,3}
};
// row of token t: 8 dims (half 0: e0 .., half 1: e0+16 ..) as 16 bytes
__device__ __forceinline__ uint4 v_row_of(const VPieces& p, int t, int half) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint4 &a = p.u[2 * i], &b = p.u[2 * i + 1];
        const uint32_t x = half ? (t < 2 ? a.z : a.w) : (t < 2 ? a.x : a.y), y = half ? (t < 2 ? b.z : b.w) : (t < 2 ? b.x : b.y);
        w[i] = (t & 1) ? (x >> 16) | (y & 0xffff0000u) : (x & 0xffffu) | (y << 16);
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}
__device__ __forceinline__ uint32_t half_of(const uint4& r, int i) {  // value i of a row's 8
    const uint32_t w = i < 2 ? r.x : i < 4 ? r.y : i < 6 ? r.z : r.w;
    return (i & 1) ? w >> 16 : w & 0xffffu;
}
__device__ __forceinline__ VPieces v_pieces_of(const uint4 (&lo)[4], const uint4 (&hi)[4]) {  // [token]: dims e0 .. and e0+16 ..
    VPieces p;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        p.u[i] = make_uint4(half_of(lo[0], i) | half_of(lo[1], i) << 16, half_of(lo[2], i) | half_of(lo[3], i) << 16,
                            half_of(hi[0], i) | half_of(hi[1], i) << 16, half_of(hi[2], i) | half_of(hi[3], i) << 16);
    return p;
}

// One wave per 4 consecutive input tokens, for K (blockIdx.y = 0) or V.  V: four tokens that follow each other in the input and fill positions
// 4q .. 4q+3 of one request are written together by the wave that has the first of them, wherever in its four it is;
// a token that belongs to no such run is written element by element.
__global__ __launch_bounds__(256) void append_kv_vec_kernel(PoolDesc p, int layer, const uint16_t* __restrict__ k,
                                                            const uint16_t* __restrict__ v, const int32_t* __restrict__ bt,
                                                            int max_blocks, const int32_t* __restrict__ seq_idx,
                                                            const int32_t* __restrict__ pos, int64_t n) {
    const int lane = threadIdx.x & 63, row = p.n_kv * p.d, d8 = p.d / 8;
    const int64_t groups = (n + 3) / 4;
    for (int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); g < groups; g += (int64_t)gridDim.x * 4) {
        const int64_t j0 = g * 4;
        const int nt = (int)min((int64_t)4, n - j0);
        // lane l < 10 holds request and position of input token j0 - 3 + l, which is all that decides the four tokens' runs
        const int64_t jl = j0 - 3 + min(lane, 9);
        const bool there = jl >= 0 && jl < n;
        const int my_pos = there ? pos[jl] : -8, my_seq = there ? seq_idx[jl] : -1;
        const int my_block = lane >= 3 && lane < 3 + nt ? bt[(size_t)my_seq * max_blocks + my_pos / kBlockSize] : 0;
        // K: lane = (8-dim piece, token), token fastest: 64 contiguous bytes per piece; all loads before the stores
        if (blockIdx.y == 0) {
            const int t = min(lane & 3, nt - 1);  // (past the end: the last token once more)
            const int slot = __shfl(my_pos, 3 + t) % kBlockSize, block = __shfl(my_block, 3 + t);
            const uint16_t* src = k + (j0 + t) * row;
            const int pieces = p.n_kv * d8;
            for (int c0 = lane >> 2; c0 < pieces; c0 += 128) {
                uint4 x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = *reinterpret_cast<const uint4*>(src + min(c0 + 16 * i, pieces - 1) * 8);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int c = c0 + 16 * i, kvh = c / d8;
                    if (c < pieces) *reinterpret_cast<uint4*>(p.base + tile_base(p, layer, block, kvh) + k_off(slot, (c - kvh * d8) * 8)) = x[i];
                }
            }
            continue;
        }
        // whether a full run of four starts at input token j0 - 3 + l (uniform; l = 0 .. 6)
        auto run_at = [&](int l) {
            const int ps = __shfl(my_pos, l), sq = __shfl(my_seq, l);
            bool ok = ps >= 0 && ps % 4 == 0;
#pragma unroll
            for (int u = 1; u < 4; ++u) ok = ok && __shfl(my_pos, l + u) == ps + u && __shfl(my_seq, l + u) == sq;
            return __builtin_amdgcn_readfirstlane((int)ok) != 0;
        };
        for (int t = 0; t < nt; ++t) {
            const int64_t j = j0 + t;
            const int ps = __builtin_amdgcn_readfirstlane(__shfl(my_pos, 3 + t));
            const int block = __builtin_amdgcn_readfirstlane(__shfl(my_block, 3 + t));
            if (run_at(3 + t)) {
                const int q = ps % kBlockSize / 4;
                for (int c = lane; c < p.n_kv * p.d / 16; c += 64) {  // 8 dims and their partners 16 further
                    const int kvh = c / (p.d / 16), r = c - kvh * (p.d / 16), e0 = r / 2 * 32 + (r & 1) * 8;
                    uint4 lo[4], hi[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint16_t* src = v + (j + u) * row + kvh * p.d + e0;
                        lo[u] = *reinterpret_cast<const uint4*>(src);
                        hi[u] = *reinterpret_cast<const uint4*>(src + 16);
                    }
                    const VPieces vp = v_pieces_of(lo, hi);
                    uint4* dst = reinterpret_cast<uint4*>(p.base + tile_base(p, layer, block, kvh) + 16 * p.d + v_off(4 * q, e0));
#pragma unroll
                    for (int i = 0; i < 8; ++i) dst[i] = vp.u[i];
                }
            } else if (!run_at(3 + t - ps % 4)) {
                for (int e = lane; e < row; e += 64) {
                    const int kvh = e / p.d, dd = e % p.d;
                    p.base[tile_base(p, layer, block, kvh) + 16 * p.d + v_off(ps % kBlockSize, dd)] = v[j * row + e];
                }
            }
        }
    }
}

// few tokens, and input rows that are not 16-byte aligned
__global__ __launch_bounds__(256) void append_kv_kernel(PoolDesc p, int layer, const uint16_t* __restrict__ k,
                                                        const uint16_t* __restrict__ v, const int32_t* __restrict__ bt,
                                                        int max_blocks, const int32_t* __restrict__ seq_idx,
                                                        const int32_t* __restrict__ pos, int64_t n) {
    int row = p.n_kv * p.d;
    for (int64_t j = blockIdx.x; j < n; j += gridDim.x) {
        int ps = pos[j];
        int block = bt[(size_t)seq_idx[j] * max_blocks + ps / kBlockSize];
        int t = ps % kBlockSize;
        for (int e = threadIdx.x; e < row; e += 256) {
            int kvh = e / p.d, dd = e % p.d;
            size_t tb = tile_base(p, layer, block, kvh);
            p.base[tb + k_off(t, dd)] = k[j * row + e];
            p.base[tb + 16 * p.d + v_off(t, dd)] = v[j * row + e];
        }
    }
}

int32_t launch_append_kv(const PoolDesc& p, int layer, const uint16_t* k, const uint16_t* v, const int32_t* bt,
                         int max_blocks, const int32_t* seq_idx, const int32_t* pos, int64_t n, hipStream_t st) {
    if (n == 0) return CHIRON_OK;
    if (by_pieces(p, k, v, n, kVecAppendBytes)) {
        const int64_t wgs = (n + 15) / 16;
        launch(append_kv_vec_kernel, dim3((int)(wgs < 65536 ? wgs : 65536), 2), dim3(256), st, p, layer, k, v, bt, max_blocks, seq_idx, pos, n);
        CHIRON_HIP(hipGetLastError());
        return CHIRON_OK;
    }
    int blocks = (int)(n < 65536 ? n : 65536);
    launch(append_kv_kernel, dim3(blocks), dim3(256), st, p, layer, k, v, bt, max_blocks, seq_idx, pos, n);
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

// One wave per 4 positions 4q .. 4q+3 (of one page), for K (blockIdx.y = 0) or V.
__global__ __launch_bounds__(256) void gather_kv_vec_kernel(PoolDesc p, int layer, const int32_t* __restrict__ bt_row, int len,
                                                            uint16_t* __restrict__ k_out, uint16_t* __restrict__ v_out) {
    const int lane = threadIdx.x & 63, row = p.n_kv * p.d, d8 = p.d / 8;
    for (int q4 = blockIdx.x * 4 + (threadIdx.x >> 6); q4 * 4 < len; q4 += gridDim.x * 4) {
        const int tk0 = q4 * 4, nt = min(4, len - tk0);
        const int block = bt_row[tk0 / kBlockSize], slot0 = tk0 % kBlockSize;
        const int t = min(lane & 3, nt - 1), pieces = p.n_kv * d8;
        for (int c0 = blockIdx.y == 0 ? lane >> 2 : INT_MAX; c0 < pieces; c0 += 128) {  // all loads before the stores
            uint4 x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = min(c0 + 16 * i, pieces - 1), kvh = c / d8;
                x[i] = *reinterpret_cast<const uint4*>(p.base + tile_base(p, layer, block, kvh) + k_off(slot0 + t, (c - kvh * d8) * 8));
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (c0 + 16 * i < pieces) *reinterpret_cast<uint4*>(k_out + (size_t)(tk0 + t) * row + (c0 + 16 * i) * 8) = x[i];
        }
        for (int c = blockIdx.y == 1 ? lane : INT_MAX; c < p.n_kv * p.d / 16; c += 64) {
            const int kvh = c / (p.d / 16), r = c - kvh * (p.d / 16), e0 = r / 2 * 32 + (r & 1) * 8;
            const uint4* src = reinterpret_cast<const uint4*>(p.base + tile_base(p, layer, block, kvh) + 16 * p.d + v_off(slot0, e0));
            VPieces vp;
#pragma unroll
            for (int i = 0; i < 8; ++i) vp.u[i] = src[i];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u < nt) {
                    uint16_t* dst = v_out + (size_t)(tk0 + u) * row + kvh * p.d + e0;
                    *reinterpret_cast<uint4*>(dst) = v_row_of(vp, u, 0);
                    *reinterpret_cast<uint4*>(dst + 16) = v_row_of(vp, u, 1);
                }
        }
    }
}

// few tokens, and outputs that are not 16-byte aligned
__global__ __launch_bounds__(256) void gather_kv_kernel(PoolDesc p, int layer, const int32_t* __restrict__ bt_row,
                                                        int len, uint16_t* __restrict__ k_out,
                                                        uint16_t* __restrict__ v_out) {
    int row = p.n_kv * p.d;
    for (int tk = blockIdx.x; tk < len; tk += gridDim.x) {
        int block = bt_row[tk / kBlockSize];
        int t = tk % kBlockSize;
        for (int e = threadIdx.x; e < row; e += 256) {
            int kvh = e / p.d, dd = e % p.d;
            size_t tb = tile_base(p, layer, block, kvh);
            k_out[(size_t)tk * row + e] = p.base[tb + k_off(t, dd)];
            v_out[(size_t)tk * row + e] = p.base[tb + 16 * p.d + v_off(t, dd)];
        }
    }
}

int32_t launch_gather_kv(const PoolDesc& p, int layer, const int32_t* bt_row, int len, uint16_t* k_out, uint16_t* v_out,
                         hipStream_t st) {
    if (len == 0) return CHIRON_OK;
    if (by_pieces(p, k_out, v_out, len, kVecGatherBytes)) {
        const int wgs = (len + 15) / 16;
        launch(gather_kv_vec_kernel, dim3(wgs < 65536 ? wgs : 65536, 2), dim3(256), st, p, layer, bt_row, len, k_out, v_out);
        CHIRON_HIP(hipGetLastError());
        return CHIRON_OK;
    }
    launch(gather_kv_kernel, dim3(len < 65536 ? len : 65536), dim3(256), st, p, layer, bt_row, len, k_out, v_out);
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

// ---- page migration (eviction to host memory and back): one workgroup per (page, layer), 16-byte copies ------
__global__ __launch_bounds__(256) void swap_kernel(PoolDesc p, const int32_t* __restrict__ bt_row, uint16_t* image,
                                                   int to_image) {
    const int j = blockIdx.x, layer = blockIdx.y;
    const size_t page_elems = (size_t)p.n_kv * 2 * 16 * p.d;
    uint4* pool = reinterpret_cast<uint4*>(p.base + (size_t)layer * (size_t)p.layer_stride + (size_t)bt_row[j] * page_elems);
    uint4* img = reinterpret_cast<uint4*>(image + ((size_t)j * p.n_layers + layer) * page_elems);
    const int n16 = (int)(page_elems / 8);
    for (int e = threadIdx.x; e < n16; e += 256) {
        if (to_image) img[e] = pool[e];
        else pool[e] = img[e];
    }
}

int32_t launch_swap(const PoolDesc& p, const int32_t* bt_row, int n_pages, uint16_t* image, int to_image, hipStream_t st) {
    if (n_pages == 0) return CHIRON_OK;
    launch(swap_kernel, dim3(dim3(n_pages, p.n_layers)), dim3(256), st, p, bt_row, image, to_image);
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

// ---- decode step: sum the K-slices of the QKV projection (whose columns are in packed order), rotate q and k, round k and v to bf16, write them
// at their slots.  One wave per (request, head): lane j owns dims j, j+64, ... of the head. ------------
__global__ __launch_bounds__(64) void rope_append_kernel(PoolDesc p, int layer, const float* __restrict__ qkv, int ks,
                                                         size_t slice_stride, int n_q,
                                                         const float* __restrict__ cos_t,
                                                         const float* __restrict__ sin_t,
                                                         const int32_t* __restrict__ bt, int max_blocks,
                                                         const int32_t* __restrict__ seq_lens, int q_len,
                                                         float* __restrict__ q_out) {
    const int i = blockIdx.x, hd = blockIdx.y, d = p.d, half = d / 2;
    const int ld = (n_q + 2 * p.n_kv) * d;
    const float* row = qkv + (size_t)i * ld + (size_t)hd * d;
    // sum over the K-slices, four independent loads in flight at a time, slices added in ascending order
    auto val = [&](int e) {
        const float* q = row + qkv_packed_dim(e, d);
        float v = 0.f;
        int s = 0;
        for (; s + 4 <= ks; s += 4) {
            float t0 = q[(size_t)s * slice_stride], t1 = q[(size_t)(s + 1) * slice_stride];
            float t2 = q[(size_t)(s + 2) * slice_stride], t3 = q[(size_t)(s + 3) * slice_stride];
            v += t0; v += t1; v += t2; v += t3;
        }
        for (; s < ks; ++s) v += q[(size_t)s * slice_stride];
        return v;
    };
    const int req = i / q_len;  // row i: token i % q_len of request req
    const int ps = seq_lens[req] + i % q_len;
    const int block = bt[(size_t)req * max_blocks + ps / kBlockSize];
    const int t = ps % kBlockSize;
    if (hd < n_q + p.n_kv) {
        for (int j = threadIdx.x; j < half; j += 64) {
            float c = cos_t[(size_t)i * half + j], s = sin_t[(size_t)i * half + j];
            float a = val(j), b = val(j + half);
            float ra = a * c - b * s, rb = b * c + a * s;
            if (hd < n_q) {
                float* qrow = q_out + (size_t)i * n_q * d + (size_t)hd * d;
                qrow[j] = ra;
                qrow[j + half] = rb;
            } else {
                size_t tb = tile_base(p, layer, block, hd - n_q);
                p.base[tb + k_off(t, j)] = f32_to_bf16_rne(ra);
                p.base[tb + k_off(t, j + half)] = f32_to_bf16_rne(rb);
            }
        }
    } else {
        size_t tb = tile_base(p, layer, block, hd - n_q - p.n_kv);
        for (int e = threadIdx.x; e < d; e += 64) p.base[tb + 16 * d + v_off(t, e)] = f32_to_bf16_rne(val(e));
    }
}

int32_t launch_rope_append(const PoolDesc& p, int layer, const float* qkv, int ks, int n_q, const float* cos_t,
                           const float* sin_t, const int32_t* bt, int max_blocks, const int32_t* seq_lens, int q_len,
                           int rows, float* q_out, hipStream_t st) {
    if (rows == 0) return CHIRON_OK;
    size_t stride = (size_t)rows * (n_q + 2 * p.n_kv) * p.d;
    dim3 grid(rows, n_q + 2 * p.n_kv);
    launch(rope_append_kernel, dim3(grid), dim3(64), st, p, layer, qkv, ks, stride, n_q, cos_t, sin_t, bt, max_blocks, seq_lens, q_len, q_out);
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

}  // namespace chiron
