// ee_kernels_f32.hip -- the decode step for EE_F32 models: fp32 kernels for any
// (small) shape.  Nothing is rounded on this path.  At these sizes the step is a
// chain of launches that each wait for memory once or twice, so the kernels are
// built for few launches and few dependent loads: products on the fp32 MFMAs with
// K split over the waves of a workgroup, norms inside the products.  The bandwidth-
// and MFMA-bound work of the large bf16 models lives in ee_kernels_bf16.hip.
#include "ee_device.h"

#include <float.h>

// ------------------------------------------------------------------ GEMM
// out[i][j] = sum_k x[i][k] W[j][k] for list entries i < n, 16 x 16 results per workgroup.
// What bounds it is latency: at K = 256 .. 688 the 16-wide LDS tiles used before took 43 steps of load, barrier,
// multiply, barrier (32 us for K = 688, 10 us for K = 256).  Here 8 waves split K; a wave asks for 16 columns of
// its 16 rows of x and W at a time, straight into the operand registers of v_mfma_f32_16x16x4_f32 (lane l holds
// row l % 16, columns 4 (l / 16) .. +3; the four MFMAs of a chunk take one of them each, which permutes K alike
// on both sides), so all loads of a wave are in flight together; the waves' partial sums are added in wave order
// through LDS.  4 to 5 us at both sizes.
// NORM: x = RMSNorm(h[idx[i]]; gain): the waves also sum the squares of what they load, and the sum over k of
// h[k] gain[k] W[j][k] is multiplied by the row's 1 / sqrt(mean + eps) at the end, so no launch normalises.
// VEC: 16-byte loads (K a multiple of 4, all operands aligned); otherwise element by element.
enum { F32_EPI_STORE = 0, F32_EPI_RESID = 1, F32_EPI_SCALE = 2, F32_EPI_SWIGLU = 3 };
#define F32_WAVES 8

struct F32Gemm {
    const float* X; int ldx;             // NORM: the residual stream, indexed by row id
    const float* W; int N, K;            // SWIGLU: N = F, up row j follows gate row j by F rows
    const int32_t* n_ptr; int B;
    float* out; int ldo;
    const int32_t* idx;
    const float* row_scale;              // SCALE: per row id
    const float* gain; float eps;        // NORM
};

template <bool VEC>
__device__ __forceinline__ float4 f32_load4(const float* p, int k, int K) {
    if constexpr (VEC) return k < K ? *reinterpret_cast<const float4*>(p + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    else return make_float4(k < K ? p[k] : 0.f, k + 1 < K ? p[k + 1] : 0.f, k + 2 < K ? p[k + 2] : 0.f, k + 3 < K ? p[k + 3] : 0.f);
}

template <int EPI, bool NORM, bool VEC>
__global__ void __launch_bounds__(64 * F32_WAVES)
k_f32_gemm(F32Gemm g) {
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    constexpr int NW = EPI == F32_EPI_SWIGLU ? 2 : 1;      // weight rows per result
    __shared__ float red[NW][F32_WAVES][64][4];
    __shared__ float ssq[F32_WAVES][16];
    const int n = min(*g.n_ptr, g.B);
    const int row0 = blockIdx.y * 16;
    if (row0 >= n) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m = lane & 15, kq = lane >> 4;
    const int col0 = blockIdx.x * 16;
    const int xrow = min(row0 + m, n - 1), wrow = min(col0 + m, g.N - 1);   // rows past the end: computed, not written
    const float* x = g.X + (int64_t)(NORM ? g.idx[xrow] : xrow) * g.ldx;
    const float* wp = g.W + (int64_t)wrow * g.K;
    const float* wu = wp + (int64_t)g.N * g.K;             // SWIGLU only
    floatx4 acc[NW] = {};
    float ss = 0.f;
    const int chunks = (g.K + 15) >> 4;
    constexpr int U = 4;                                   // chunks in flight per wave
    for (int c0 = w; c0 < chunks; c0 += F32_WAVES * U) {
        float4 xv[U], wv[U], uv[U], gv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (c0 + u * F32_WAVES) * 16 + 4 * kq;
            xv[u] = f32_load4<VEC>(x, k, g.K);
            wv[u] = f32_load4<VEC>(wp, k, g.K);
            if constexpr (NW == 2) uv[u] = f32_load4<VEC>(wu, k, g.K);
            if constexpr (NORM) gv[u] = f32_load4<VEC>(g.gain, k, g.K);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float xe[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
            const float we[4] = {wv[u].x, wv[u].y, wv[u].z, wv[u].w};
            if constexpr (NORM) {
                const float ge[4] = {gv[u].x, gv[u].y, gv[u].z, gv[u].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) { ss += xe[e] * xe[e]; xe[e] *= ge[e]; }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(xe[e], we[e], acc[0], 0, 0, 0);
            if constexpr (NW == 2) {
                const float ue[4] = {uv[u].x, uv[u].y, uv[u].z, uv[u].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(xe[e], ue[e], acc[1], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < NW; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[q][w][lane][r] = acc[q][r];
    if constexpr (NORM) {
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (kq == 0) ssq[w][m] = ss;
    }
    __syncthreads();
    if (threadIdx.x >= 256) return;
    // thread = 4 * lane + r of the result registers: row 4 (lane / 16) + r, column lane % 16
    const int l = threadIdx.x >> 2, r = threadIdx.x & 3;
    const int rl = 4 * (l >> 4) + r, row = row0 + rl, col = col0 + (l & 15);
    if (row >= n || col >= g.N) return;
    float v[NW];
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        v[q] = 0.f;
#pragma unroll
        for (int k = 0; k < F32_WAVES; ++k) v[q] += red[q][k][l][r];
    }
    if constexpr (NORM) {
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < F32_WAVES; ++k) t += ssq[k][rl];
        const float inv = 1.0f / sqrtf(t / (float)g.K + g.eps);
#pragma unroll
        for (int q = 0; q < NW; ++q) v[q] *= inv;
    }
    if constexpr (EPI == F32_EPI_STORE) g.out[(int64_t)row * g.ldo + col] = v[0];
    else if constexpr (EPI == F32_EPI_RESID) g.out[(int64_t)g.idx[row] * g.ldo + col] += v[0];
    else if constexpr (EPI == F32_EPI_SCALE) g.out[(int64_t)row * g.ldo + col] = v[0] * g.row_scale[g.idx[row]];
    else g.out[(int64_t)row * g.ldo + col] = (v[0] / (1.0f + expf(-v[0]))) * v[NW - 1];
}

// ------------------------------------------------------------------ RoPE + cache append
// buf[i] holds [q (n_q*hd, may be empty) | k (Hkv*hd) | v (Hkv*hd)] of list entry i.
// Rotates q in place and k on its way into the cache, at the row's position.
__global__ void __launch_bounds__(256)
k_f32_rope_append(float* __restrict__ buf, int ld, int n_q, const int32_t* __restrict__ idx,
                  const int32_t* __restrict__ n_ptr, int B, const int32_t* __restrict__ pos,
                  const float* __restrict__ rope, int max_pos, KvView kv, int32_t* __restrict__ status) {
    int i = blockIdx.x;
    int n = min(*n_ptr, B);
    if (i >= n) return;
    int b = idx[i];
    int p = pos[b];
    int hd = kv.head_dim, half = hd >> 1, Hkv = kv.n_kv_heads;
    const int sq = kv_row(kv, b);
    int cap = kv.cap[sq];
    bool ok = p >= 0 && p < cap && p < max_pos;
    if (!ok) {
        if (threadIdx.x == 0) atomicOr(status, 1);
        return;
    }
    float* r = buf + (int64_t)i * ld;
    const float* cs = rope + (int64_t)p * half * 2;
    for (int t = threadIdx.x; t < n_q * half; t += 256) {
        int hh = t / half, j = t % half;
        float c = cs[2 * j], s = cs[2 * j + 1];
        float a = r[hh * hd + j], bb = r[hh * hd + j + half];
        r[hh * hd + j] = a * c - bb * s;
        r[hh * hd + j + half] = bb * c + a * s;
    }
    float* kin = r + n_q * hd;
    float* vin = kin + Hkv * hd;
    for (int t = threadIdx.x; t < Hkv * half; t += 256) {
        int g = t / half, j = t % half;
        float c = cs[2 * j], s = cs[2 * j + 1];
        float a = kin[g * hd + j], bb = kin[g * hd + j + half];
        float* base = reinterpret_cast<float*>(kv.pool) + kv_block(kv, sq, g, cap);
        base[(int64_t)p * hd + j] = a * c - bb * s;
        base[(int64_t)p * hd + j + half] = bb * c + a * s;
    }
    for (int t = threadIdx.x; t < Hkv * hd; t += 256) {
        int g = t / hd, j = t % hd;
        float* base = reinterpret_cast<float*>(kv.pool) + kv_block(kv, sq, g, cap);
        base[(int64_t)cap * hd + (int64_t)p * hd + j] = vin[g * hd + j];
    }
}

// ------------------------------------------------------------------ attention
// One block per (query head, list entry): softmax(q.K^T / sqrt(hd)) V over positions 0..pos.
// VEC (hd a multiple of 4): L lanes (the power of two from hd / 4 up) share a position and take 16 bytes of its
// key or value each, the 256 / L groups take positions in turn, so a wave reads whole cache rows and as many
// positions are in flight as there are groups.  Before, a thread walked one key on its own and hd threads walked
// all values: 9.9 -> 8.4 us at 65 positions of 64 values, and far more beyond (64 rows of up to 1500
// positions: the whole layer 268 -> 88 us).  Other hd: one position per thread, one value per thread.
template <bool VEC>
__global__ void __launch_bounds__(256)
k_f32_attn(const float* __restrict__ qkv, int ld, int Hq, const int32_t* __restrict__ idx,
           const int32_t* __restrict__ n_ptr, int B, const int32_t* __restrict__ pos, KvView kv,
           float* __restrict__ out /* [i][Hq*hd] */, int L) {
    extern __shared__ float sm[];   // VEC: partial outputs [256 / L][hd] (at most 4 * 256) | scores; else q[hd] | scores
    __shared__ float red[4];
    int hq = blockIdx.x, i = blockIdx.y;
    int n = min(*n_ptr, B);
    if (i >= n) return;
    int b = idx[i];
    int hd = kv.head_dim;
    const int sq = kv_row(kv, b);
    int cap = kv.cap[sq];
    int n_pos = min(pos[b] + 1, cap);
    int g = hq / (Hq / kv.n_kv_heads);
    const float* Kb = reinterpret_cast<const float*>(kv.pool) + kv_block(kv, sq, g, cap);
    const float* Vb = Kb + (int64_t)cap * hd;
    const float* qrow = qkv + (int64_t)i * ld + hq * hd;
    float* sc = sm + (VEC ? 1024 : hd);
    const float inv_sqrt = 1.0f / sqrtf((float)hd);
    const int c = 4 * (threadIdx.x & (L - 1)), grp = threadIdx.x / L, groups = 256 / L;     // VEC
    const bool has = c < hd;
    float mx = -FLT_MAX;
    if constexpr (VEC) {
        const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
        const float4 q = has ? *reinterpret_cast<const float4*>(qrow + c) : zero;
        for (int t0 = grp; t0 < n_pos; t0 += 4 * groups) {
            float4 k[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u * groups;
                k[u] = has && t < n_pos ? *reinterpret_cast<const float4*>(Kb + (int64_t)t * hd + c) : zero;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float a = (q.x * k[u].x + q.y * k[u].y) + (q.z * k[u].z + q.w * k[u].w);
                for (int o = L >> 1; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
                const int t = t0 + u * groups;
                if (t >= n_pos) continue;
                a *= inv_sqrt;
                if (c == 0) sc[t] = a;
                mx = fmaxf(mx, a);
            }
        }
    } else {
        float* q = sm;
        for (int t = threadIdx.x; t < hd; t += 256) q[t] = qrow[t];
        __syncthreads();
        for (int t = threadIdx.x; t < n_pos; t += 256) {
            float a = 0.f;
            for (int j = 0; j < hd; ++j) a += q[j] * Kb[(int64_t)t * hd + j];
            a *= inv_sqrt;
            sc[t] = a;
            mx = fmaxf(mx, a);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    float sum = 0.f;
    for (int t = threadIdx.x; t < n_pos; t += 256) {
        float p = expf(sc[t] - mx);
        sc[t] = p;
        sum += p;
    }
    sum = block_sum<256>(sum, red);   // also makes sc[] visible to all threads
    float* orow = out + (int64_t)i * (Hq * hd) + hq * hd;
    if constexpr (VEC) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (has) {
#pragma unroll 4
            for (int t = grp; t < n_pos; t += groups) {
                const float p = sc[t];
                const float4 v = *reinterpret_cast<const float4*>(Vb + (int64_t)t * hd + c);
                acc.x += p * v.x; acc.y += p * v.y; acc.z += p * v.z; acc.w += p * v.w;
            }
            *reinterpret_cast<float4*>(sm + grp * hd + c) = acc;
        }
        __syncthreads();
        for (int j = threadIdx.x; j < hd; j += 256) {
            float a = 0.f;
            for (int k = 0; k < groups; ++k) a += sm[k * hd + j];
            orow[j] = a / sum;
        }
    } else {
        for (int j = threadIdx.x; j < hd; j += 256) {
            float acc = 0.f;
            for (int t = 0; t < n_pos; ++t) acc += sc[t] * Vb[(int64_t)t * hd + j];
            orow[j] = acc / sum;
        }
    }
}

// ------------------------------------------------------------------ logits -> decision
// One block per list entry: largest logit and its lowest column, then the sum of exp(z - max), the confidence
// 1 / sum, and the exit decision of k_exit_decide (ee_kernels_common.hip) in the same launch.
__global__ void __launch_bounds__(256)
k_f32_exit_decide(const float* __restrict__ logits, int V, const int32_t* __restrict__ n_ptr, int B, float threshold,
                  int force_exit, float* __restrict__ head_conf, int32_t* __restrict__ head_tok,
                  uint8_t* __restrict__ head_exit, uint8_t* __restrict__ head_breach) {
    __shared__ float s_m[4];
    __shared__ int s_a[4];
    __shared__ float red[4];
    int i = blockIdx.x;
    int n = min(*n_ptr, B);
    if (i >= n) return;
    const float* z = logits + (int64_t)i * V;
    // Maximum and column as stat_merge takes them: a logit that is NaN is never the maximum, and the row's token is
    // the largest of the others (none: the lowest column); the sum below is NaN then, and the row meets no threshold.
    float m = -FLT_MAX;
    int a = threadIdx.x < V ? threadIdx.x : 0x7fffffff;
    auto take = [&](float m2, int a2) {
        a = m > m2 ? a : (m2 > m ? a2 : min(a, a2));
        m = fmaxf(m, m2);
    };
#pragma unroll 4
    for (int j = threadIdx.x; j < V; j += 256) {
        const float v = z[j];
        if (v > m) { m = v; a = j; }                          // rising j: > keeps the lowest column
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float m2 = __shfl_xor(m, o, 64);
        const int a2 = __shfl_xor(a, o, 64);
        take(m2, a2);
    }
    if ((threadIdx.x & 63) == 0) { s_m[threadIdx.x >> 6] = m; s_a[threadIdx.x >> 6] = a; }
    __syncthreads();
    m = s_m[0]; a = s_a[0];
    for (int w = 1; w < 4; ++w) take(s_m[w], s_a[w]);
    float sum = 0.f;
#pragma unroll 4
    for (int j = threadIdx.x; j < V; j += 256) sum += expf(z[j] - m);
    sum = block_sum<256>(sum, red);
    if (threadIdx.x == 0) {
        const float conf = 1.0f / sum;
        const bool met = conf >= threshold;
        head_conf[i] = conf;
        head_tok[i] = a;
        head_exit[i] = (met || force_exit) ? 1 : 0;
        head_breach[i] = (force_exit && !met) ? 1 : 0;
    }
}

// ------------------------------------------------------------------ host side
static KvView make_view(const ee_model* m, const ee_kv* kv, int layer, const ee_batch* b) {
    return KvView{kv->pool, kv->d_cap, kv->d_off, kv->T, m->cfg.n_kv_heads, m->cfg.head_dim, layer - 1, b->kv_seq};
}

template <int EPI, bool NORM>
static void gemm(const F32Gemm& g, hipStream_t s) {
    const dim3 grid((g.N + 15) / 16, (g.B + 15) / 16), block(64 * F32_WAVES);
    const uintptr_t a = (uintptr_t)g.X | (uintptr_t)g.W | (NORM ? (uintptr_t)g.gain : 0);
    if (g.K % 4 == 0 && g.ldx % 4 == 0 && a % 16 == 0) hipLaunchKernelGGL((k_f32_gemm<EPI, NORM, true>), grid, block, 0, s, g);
    else hipLaunchKernelGGL((k_f32_gemm<EPI, NORM, false>), grid, block, 0, s, g);
}

int f32_layer_forward(const ee_model* m, int layer, ee_kv* kv, ee_batch* b, hipStream_t s) {
    const ee_model_config& c = m->cfg;
    const ee_layer_weights& w = m->layers[layer - 1];
    const ee_batch_layout& L = b->L;
    int B = b->B, d = c.d_model, hd = c.head_dim, qd = c.n_q_heads * hd, F = c.d_ffn;
    int qkv_n = (c.n_q_heads + 2 * c.n_kv_heads) * hd;
    const int32_t* idx = b->st<int32_t>(L.active_idx);
    const int32_t* n_ptr = b->st<int32_t>(L.n_active);
    float* h = b->st<float>(L.h);
    float* qkv = b->wsp<float>(b->W.qkv);
    float* ao = b->wsp<float>(b->W.ao);
    float* act = b->wsp<float>(b->W.act);
    KvView view = make_view(m, kv, layer, b);

    gemm<F32_EPI_STORE, true>(F32Gemm{h, d, (const float*)w.w_qkv, qkv_n, d, n_ptr, B, qkv, qkv_n, idx, nullptr, w.g_attn, c.rms_eps}, s);
    hipLaunchKernelGGL(k_f32_rope_append, dim3(B), dim3(256), 0, s, qkv, qkv_n, c.n_q_heads, idx, n_ptr, B,
                       b->st<int32_t>(L.pos), m->d_rope, c.max_pos, view, b->st<int32_t>(L.status));
    int lanes = 1;                            // lanes that share a position: a power of two that holds hd / 4
    while (4 * lanes < hd) lanes *= 2;
    if (hd % 4 == 0)
        hipLaunchKernelGGL(k_f32_attn<true>, dim3(c.n_q_heads, B), dim3(256), (size_t)(1024 + c.max_pos) * sizeof(float), s, qkv,
                           qkv_n, c.n_q_heads, idx, n_ptr, B, b->st<int32_t>(L.pos), view, ao, lanes);
    else
        hipLaunchKernelGGL(k_f32_attn<false>, dim3(c.n_q_heads, B), dim3(256), (size_t)(hd + c.max_pos) * sizeof(float), s, qkv,
                           qkv_n, c.n_q_heads, idx, n_ptr, B, b->st<int32_t>(L.pos), view, ao, 1);
    gemm<F32_EPI_RESID, false>(F32Gemm{ao, qd, (const float*)w.w_o, d, qd, n_ptr, B, h, d, idx, nullptr, nullptr, 0.f}, s);
    gemm<F32_EPI_SWIGLU, true>(F32Gemm{h, d, (const float*)w.w_gate_up, F, d, n_ptr, B, act, F, idx, nullptr, w.g_ffn, c.rms_eps}, s);
    gemm<F32_EPI_RESID, false>(F32Gemm{act, F, (const float*)w.w_down, d, F, n_ptr, B, h, d, idx, nullptr, nullptr, 0.f}, s);
    EE_LAUNCH_CHECK();
    return EE_OK;
}

int f32_exit_head(const ee_model* m, int e, float th, int force, ee_batch* b, float* dbg, hipStream_t s) {
    const ee_model_config& c = m->cfg;
    const ee_batch_layout& L = b->L;
    int B = b->B, d = c.d_model, V = c.vocab;
    const int32_t* idx = b->st<int32_t>(L.active_idx);
    const int32_t* n_ptr = b->st<int32_t>(L.n_active);
    float* logits = dbg ? dbg : b->wsp<float>(b->W.logits);
    gemm<F32_EPI_SCALE, true>(F32Gemm{b->st<float>(L.h), d, (const float*)m->exits[e].w, V, d, n_ptr, B, logits, V, idx,
                                      b->st<float>(L.row_scale), m->exits[e].gain, c.rms_eps}, s);
    TimedScope t(EE_K_EXIT_DECIDE, s);
    hipLaunchKernelGGL(k_f32_exit_decide, dim3(B), dim3(256), 0, s, logits, V, n_ptr, B, th, force, b->st<float>(L.head_conf),
                       b->st<int32_t>(L.head_tok), b->st<uint8_t>(L.head_exit), b->st<uint8_t>(L.head_breach));
    EE_LAUNCH_CHECK();
    return EE_OK;
}

int f32_fill_kv(const ee_model* m, int from_excl, int to_incl, ee_kv* kv, ee_batch* b, hipStream_t s) {
    const ee_model_config& c = m->cfg;
    const ee_batch_layout& L = b->L;
    int B = b->B, d = c.d_model, hd = c.head_dim;
    int kv_n = 2 * c.n_kv_heads * hd;
    const int32_t* idx = b->st<int32_t>(L.exited_idx);
    const int32_t* n_ptr = b->st<int32_t>(L.n_exited);
    float* kvb = b->wsp<float>(b->W.fill_kv);
    for (int l = from_excl + 1; l <= to_incl; ++l) {
        const ee_layer_weights& w = m->layers[l - 1];
        const float* Wkv = (const float*)w.w_qkv + (int64_t)c.n_q_heads * hd * d;
        gemm<F32_EPI_STORE, true>(F32Gemm{b->st<float>(L.h), d, Wkv, kv_n, d, n_ptr, B, kvb, kv_n, idx, nullptr, w.g_attn, c.rms_eps}, s);
        hipLaunchKernelGGL(k_f32_rope_append, dim3(B), dim3(256), 0, s, kvb, kv_n, 0, idx, n_ptr, B,
                           b->st<int32_t>(L.pos), m->d_rope, c.max_pos, make_view(m, kv, l, b),
                           b->st<int32_t>(L.status));
    }
    EE_LAUNCH_CHECK();
    return EE_OK;
}
