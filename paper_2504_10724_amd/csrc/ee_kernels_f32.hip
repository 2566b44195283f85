// ee_kernels_f32.hip -- the decode step for EE_F32 models: fp32 kernels for any
// (small) shape.  Nothing is rounded on this path.  At these sizes the step is a
// chain of launches that each wait for memory once or twice, so the kernels are
// built for few launches and few dependent loads: products on the fp32 MFMAs with
// K split over the waves of a workgroup, norms inside the products.  The bandwidth-
// and MFMA-bound work of the large bf16 models lives in ee_kernels_bf16.hip.
#include "ee_device.h"

#include <float.h>
#include <algorithm>

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
// ROPE: the q|k|v product, rotation and cache append in one launch.  A workgroup has 16 rotation pairs of one head: columns
// j and j + hd / 2, as SWIGLU has gate and up.  Rotated queries go to out, rotated keys and the values to the
// cache at the row's position.  As a launch of its own rotation and append took 2.6 of the 147 us of the fp32 workload's
// step six times; the K/V of the skipped layers are one launch for 32 layers (blockIdx.z).
// What a launch waits for is a chain of trips to memory, so everything that does not depend on the number of live
// rows is asked for beside it: the row ids, and of the epilogue's operands row id, old value, scale or position.
enum { F32_EPI_RESID = 0, F32_EPI_SCALE = 1, F32_EPI_SWIGLU = 2, F32_EPI_ROPE = 3 };
#define F32_WAVES 8

struct F32Gemm {
    const float* X; int ldx;             // NORM: the residual stream, indexed by row id
    const float* W; int N, K;            // SWIGLU: N = F, up row j follows gate row j by F rows; ROPE: N = all columns of W
    const int32_t* n_ptr; int B;
    float* out; int ldo;
    const int32_t* idx;
    const float* row_scale;              // SCALE: per row id
    const float* gain; float eps;        // NORM
};
#define F32_ROPE_LAYERS 32
struct F32Rope {                         // ROPE
    int n_q, head0;                      // query heads of W, first head of the launch
    const int32_t* pos; const float* rope; int max_pos;
    KvView kv;
    int32_t* status;
    // W and gain of each layer (blockIdx.z).  By value: what the layers were when the call was made, as for every other product
    const float* w[F32_ROPE_LAYERS]; const float* gain[F32_ROPE_LAYERS];
};
struct F32None {};

template <bool VEC>
__device__ __forceinline__ float4 f32_load4(const float* p, int k, int K) {
    if constexpr (VEC) return k < K ? *reinterpret_cast<const float4*>(p + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    else return make_float4(k < K ? p[k] : 0.f, k + 1 < K ? p[k + 1] : 0.f, k + 2 < K ? p[k + 2] : 0.f, k + 3 < K ? p[k + 3] : 0.f);
}

template <int EPI, bool NORM, bool VEC, class P>      // P: F32Rope for ROPE, else F32None
__global__ void __launch_bounds__(64 * F32_WAVES)
k_f32_gemm(F32Gemm g, P p) {
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    constexpr bool ROPE = EPI == F32_EPI_ROPE;
    constexpr int NW = EPI == F32_EPI_SWIGLU || ROPE ? 2 : 1;      // weight rows per result
    constexpr bool BY_ID = NORM || EPI == F32_EPI_RESID || EPI == F32_EPI_SCALE || ROPE;
    __shared__ float4 red[NW][F32_WAVES][64];
    __shared__ float ssq[F32_WAVES][16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m = lane & 15, kq = lane >> 4;
    const int row0 = blockIdx.y * 16;
    // thread = 4 * lane + r of the result registers: row 4 (lane / 16) + r, column lane % 16
    const int el = (threadIdx.x & 255) >> 2, er = threadIdx.x & 3, erl = 4 * (el >> 4) + er, erow = row0 + erl;
    // in a large batch most row groups but the first may be empty: those look at the number of rows before anything else
    if (row0 > 0 && row0 >= min(*g.n_ptr, g.B)) return;
    int id = 0, eid = 0;                                   // row ids: of the row this lane loads, and of the one it writes
    if constexpr (BY_ID) {
        id = g.idx[min(row0 + m, g.B - 1)];
        eid = g.idx[min(erow, g.B - 1)];
        asm volatile("" : "+v"(id), "+v"(eid));            // under way together with the number of rows, not after it
    }
    const int n = min(*g.n_ptr, g.B);
    if (row0 >= n) return;
    // rows past the end are computed, not written: they load the first row
    const int first_id = __builtin_amdgcn_readfirstlane(id);
    const bool in_rows = row0 + m < n, out_row = erow < n;
    if (!in_rows) id = first_id;
    if (!out_row) eid = first_id;
    int col, wrow;                                         // column of the result this thread writes, row of W this lane loads
    int half = 0, head = 0;
    if constexpr (ROPE) {
        half = p.kv.head_dim >> 1;
        const int per_head = (half + 15) >> 4;
        head = p.head0 + blockIdx.x / per_head;
        const int j0 = blockIdx.x % per_head * 16;
        col = j0 + (el & 15);
        wrow = head * 2 * half + min(j0 + m, half - 1);
        g.W = p.w[blockIdx.z];
        g.gain = p.gain[blockIdx.z];
    } else {
        col = blockIdx.x * 16 + (el & 15);
        wrow = min((int)blockIdx.x * 16 + m, g.N - 1);
    }
    const float* x = g.X + (int64_t)(NORM ? id : (in_rows ? row0 + m : row0)) * g.ldx;
    const float* wp = g.W + (int64_t)wrow * g.K;
    const float* wu = wp + (int64_t)(ROPE ? half : g.N) * g.K;      // second weight row
    // what the epilogue needs
    float old = 0.f;
    int at = 0, sq = 0, cap = 0;
    int64_t off = 0;
    float2 cs = make_float2(1.f, 0.f);
    const bool col_ok = col < (ROPE ? half : g.N);
    if constexpr (EPI == F32_EPI_RESID) { if (col_ok) old = g.out[(int64_t)eid * g.ldo + col]; }
    if constexpr (EPI == F32_EPI_SCALE) old = g.row_scale[eid];
    if constexpr (ROPE) {
        at = p.pos[eid];
        sq = kv_row(p.kv, eid);
        cap = p.kv.cap[sq];
        off = p.kv.off[sq];
    }
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
    bool pos_ok = true;
    if constexpr (ROPE) {
        pos_ok = at >= 0 && at < cap && at < p.max_pos;
        if (pos_ok && col_ok) cs = *reinterpret_cast<const float2*>(p.rope + ((int64_t)at * half + col) * 2);
    }
#pragma unroll
    for (int q = 0; q < NW; ++q) red[q][w][lane] = make_float4(acc[q][0], acc[q][1], acc[q][2], acc[q][3]);
    if constexpr (NORM) {
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (kq == 0) ssq[w][m] = ss;
    }
    __syncthreads();
    if (threadIdx.x >= 256 || !out_row || !col_ok) return;
    float v[NW];
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        v[q] = 0.f;
#pragma unroll
        for (int k = 0; k < F32_WAVES; ++k) v[q] += reinterpret_cast<const float*>(&red[q][k][el])[er];
    }
    if constexpr (NORM) {
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < F32_WAVES; ++k) t += ssq[k][erl];
        const float inv = 1.0f / sqrtf(t / (float)g.K + g.eps);
#pragma unroll
        for (int q = 0; q < NW; ++q) v[q] *= inv;
    }
    if constexpr (EPI == F32_EPI_RESID) g.out[(int64_t)eid * g.ldo + col] = old + v[0];
    else if constexpr (EPI == F32_EPI_SCALE) g.out[(int64_t)erow * g.ldo + col] = v[0] * old;
    else if constexpr (EPI == F32_EPI_SWIGLU) g.out[(int64_t)erow * g.ldo + col] = (v[0] / (1.0f + expf(-v[0]))) * v[NW - 1];
    else if constexpr (ROPE) {
        const int hd = 2 * half;
        const bool is_q = head < p.n_q, is_v = head >= p.n_q + p.kv.n_kv_heads;
        const float a = v[0], b = v[NW - 1];
        if (!pos_ok) {                                     // refused: nothing is appended, the queries stay as they are
            if (blockIdx.x == 0 && col == 0) atomicOr(p.status, 1);
            cs = make_float2(1.f, 0.f);
            if (!is_q) return;
        }
        const float x0 = is_v ? a : a * cs.x - b * cs.y, x1 = is_v ? b : b * cs.x + a * cs.y;
        float* dst;
        if (is_q) {
            dst = g.out + (int64_t)erow * g.ldo + head * hd;
        } else {
            const int kvh = head - p.n_q - (is_v ? p.kv.n_kv_heads : 0);
            dst = reinterpret_cast<float*>(p.kv.pool) + ((int64_t)(p.kv.layer0 + blockIdx.z) * p.kv.T + off) * (2LL * p.kv.n_kv_heads * hd) +
                  (int64_t)kvh * 2LL * cap * hd + (is_v ? (int64_t)cap * hd : 0) + (int64_t)at * hd;
        }
        dst[col] = x0;
        dst[col + half] = x1;
    }
}

// ------------------------------------------------------------------ attention
// softmax(q.K^T / sqrt(hd)) V over positions 0..pos, one workgroup per (query head, list entry), hd a multiple of 4.  L
// lanes (the power of two from hd / 4 up) share a position and take 16 bytes of its key and of its value each, asked for
// together, four positions per group of lanes at a time; each group keeps a running maximum, sum and output, which are
// merged over the groups of a wave and over the waves through LDS.  What bounds it is memory latency.  Layer, all scores to
// LDS, then maximum, exponentials and sum over the workgroup, then the values / so: 20 rows of 4 heads of 64, 62 positions 27.0 /
// 25.4 us, 300 33.5 / 27.5, 1500 71.4 / 37.4; one row of 1500 59.8 / 34.7.  (A long row's positions shared out over workgroups
// and merged by another launch: 30 us there, but the host does not know how long rows are, and by the cache's capacity a row
// of 20 positions in room for 2000 paid for it too, 28.4 us instead of 22.1.)
template <int THREADS>
__global__ void __launch_bounds__(THREADS)
k_f32_attn(const float* __restrict__ qkv, int ld, int Hq, const int32_t* __restrict__ idx,
           const int32_t* __restrict__ n_ptr, int B, const int32_t* __restrict__ pos, KvView kv,
           float* __restrict__ out /* [i][Hq*hd] */, int L) {
    constexpr int W = THREADS / 64;
    __shared__ float4 s_o[W][64];
    __shared__ float s_m[W], s_l[W];
    const int hq = blockIdx.x, i = blockIdx.y;
    int b = idx[i];                                         // i < B; beside the number of rows, not after it
    asm volatile("" : "+v"(b));
    const int n = min(*n_ptr, B);
    if (i >= n) return;
    b = __builtin_amdgcn_readfirstlane(b);
    const int hd = kv.head_dim;
    const int sq = kv_row(kv, b);
    const int cap = kv.cap[sq];
    const int n_pos = min(pos[b] + 1, cap);
    const int g = hq / (Hq / kv.n_kv_heads);
    const float* Kb = reinterpret_cast<const float*>(kv.pool) + kv_block(kv, sq, g, cap);
    const float* Vb = Kb + (int64_t)cap * hd;
    const float inv_sqrt = 1.0f / sqrtf((float)hd);
    const int c = 4 * (threadIdx.x & (L - 1)), grp = threadIdx.x / L, groups = THREADS / L;
    const bool has = c < hd;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 q = has ? *reinterpret_cast<const float4*>(qkv + (int64_t)i * ld + hq * hd + c) : zero;
    float m = -FLT_MAX, l = 0.f;
    float4 acc = zero;
    for (int t0 = grp; t0 < n_pos; t0 += 4 * groups) {
        float4 k[4], v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = t0 + u * groups;
            const bool ok = has && t < n_pos;
            k[u] = ok ? *reinterpret_cast<const float4*>(Kb + (int64_t)t * hd + c) : zero;
            v[u] = ok ? *reinterpret_cast<const float4*>(Vb + (int64_t)t * hd + c) : zero;
        }
        float a[4], m_new = m;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[u] = (q.x * k[u].x + q.y * k[u].y) + (q.z * k[u].z + q.w * k[u].w);
            for (int o = L >> 1; o > 0; o >>= 1) a[u] += __shfl_xor(a[u], o, 64);
            a[u] *= inv_sqrt;
            if (t0 + u * groups < n_pos) m_new = fmaxf(m_new, a[u]);
        }
        const float keep = expf(m - m_new);
        l *= keep;
        acc.x *= keep; acc.y *= keep; acc.z *= keep; acc.w *= keep;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float e = t0 + u * groups < n_pos ? expf(a[u] - m_new) : 0.f;
            l += e;
            acc.x += e * v[u].x; acc.y += e * v[u].y; acc.z += e * v[u].z; acc.w += e * v[u].w;
        }
        m = m_new;
    }
    for (int o = L; o < 64; o <<= 1) {                      // the wave's groups
        const float m2 = __shfl_xor(m, o, 64), l2 = __shfl_xor(l, o, 64);
        const float4 a2 = make_float4(__shfl_xor(acc.x, o, 64), __shfl_xor(acc.y, o, 64), __shfl_xor(acc.z, o, 64), __shfl_xor(acc.w, o, 64));
        const float mm = fmaxf(m, m2), w1 = expf(m - mm), w2 = expf(m2 - mm);
        l = l * w1 + l2 * w2;
        acc.x = acc.x * w1 + a2.x * w2; acc.y = acc.y * w1 + a2.y * w2;
        acc.z = acc.z * w1 + a2.z * w2; acc.w = acc.w * w1 + a2.w * w2;
        m = mm;
    }
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane < L) s_o[w][lane] = acc;
    if (lane == 0) { s_m[w] = m; s_l[w] = l; }
    __syncthreads();
    if ((int)threadIdx.x >= L || !has) return;              // the lanes of group 0: four features each
    float mm = s_m[0];
#pragma unroll
    for (int k = 1; k < W; ++k) mm = fmaxf(mm, s_m[k]);
    float sum = 0.f;
    acc = zero;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        const float wk = expf(s_m[k] - mm);
        const float4 o = s_o[k][lane];
        sum += s_l[k] * wk;
        acc.x += o.x * wk; acc.y += o.y * wk; acc.z += o.z * wk; acc.w += o.w * wk;
    }
    *reinterpret_cast<float4*>(out + (int64_t)i * (Hq * hd) + hq * hd + c) = make_float4(acc.x / sum, acc.y / sum, acc.z / sum, acc.w / sum);
}

// The same through the scores of all positions in LDS: maximum, exponentials and sum over the workgroup, then the values.  One
// exponential per position, where the kernel above has one per lane: for many pairs on long rows (two_passes below), and, one
// position and then one value per thread, for other hd.
template <bool VEC>
__global__ void __launch_bounds__(256)
k_f32_attn_scores(const float* __restrict__ qkv, int ld, int Hq, const int32_t* __restrict__ idx,
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

template <int EPI, bool NORM, class P = F32None>
static void gemm(const F32Gemm& g, hipStream_t s, const P& p = P{}, int cols = 0, int nz = 1, bool w_aligned = true) {
    const dim3 grid(cols ? cols : (g.N + 15) / 16, (g.B + 15) / 16, nz), block(64 * F32_WAVES);
    const uintptr_t a = (uintptr_t)g.X | (uintptr_t)g.W | (NORM ? (uintptr_t)g.gain : 0);
    if (g.K % 4 == 0 && g.ldx % 4 == 0 && a % 16 == 0 && w_aligned) hipLaunchKernelGGL((k_f32_gemm<EPI, NORM, true, P>), grid, block, 0, s, g, p);
    else hipLaunchKernelGGL((k_f32_gemm<EPI, NORM, false, P>), grid, block, 0, s, g, p);
}

// queries, keys and values of the rows of a list: heads head0 .. of layers first .. first + nl - 1, one launch per F32_ROPE_LAYERS layers
static void rope_gemm(const ee_model* m, const ee_kv* kv, ee_batch* b, int first, int nl, int head0, const int32_t* idx,
                      const int32_t* n_ptr, hipStream_t s) {
    const ee_model_config& c = m->cfg;
    const int heads = c.n_q_heads + 2 * c.n_kv_heads, per_head = (c.head_dim / 2 + 15) / 16;
    for (const int end = first + nl; first < end; first += F32_ROPE_LAYERS) {
        F32Gemm g{b->st<float>(b->L.h), c.d_model, nullptr, heads * c.head_dim, c.d_model, n_ptr, b->B, b->wsp<float>(b->W.qkv),
                  heads * c.head_dim, idx, nullptr, nullptr, c.rms_eps};
        F32Rope p{c.n_q_heads, head0, b->st<int32_t>(b->L.pos), m->d_rope, c.max_pos, make_view(m, kv, first, b), b->st<int32_t>(b->L.status), {}, {}};
        const int n = std::min(end - first, F32_ROPE_LAYERS);
        bool aligned = true;
        for (int z = 0; z < n; ++z) {
            const ee_layer_weights& w = m->layers[first - 1 + z];
            p.w[z] = (const float*)w.w_qkv; p.gain[z] = w.g_attn;
            aligned = aligned && (((uintptr_t)w.w_qkv | (uintptr_t)w.g_attn) & 15) == 0;
        }
        gemm<F32_EPI_ROPE, true>(g, s, p, (heads - head0) * per_head, n, aligned);
    }
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

    rope_gemm(m, kv, b, layer, 1, 0, idx, n_ptr, s);
    int lanes = 1;                            // lanes that share a position: a power of two that holds hd / 4
    while (4 * lanes < hd) lanes *= 2;
    const int pairs = (b->n_entries > 0 ? b->n_entries : B) * c.n_q_heads, cap = kv->max_cap;
    // Many pairs and room for long rows.  Layer, one pass / two: context passes, 4 heads, 100 entries from 1500 on 55 / 70 us, 200
    // 88 / 84, 300 from 100 on 55 / 58, 600 from 0 on 88 / 85, from 1500 on 210 / 172; 16 heads of 32, 300 entries from 500 on 103 /
    // 93, from 1500 on 178 / 138.  Decode steps, whose rows come from memory: 100 rows of 8 heads of 128, 1500 positions 338 / 322,
    // 150 455 / 450, 250 433 / 456 (700 positions).
    const bool two_passes = cap > 512 && pairs > 768 && (b->kv_seq != nullptr || pairs <= 1100);
    if (hd % 4 == 0 && !two_passes) {
        // Waves of a workgroup, by what the host knows, the (row, head) pairs and the longest row that the cache has room for; rows
        // may be much shorter, so that no choice may cost them what it gives long ones.  Layer, 4 / 8 / 16 waves: 32 pairs, 62
        // positions 22.6 / 23.1 / 24.3 us, 700 39.5 / 32.4 / 28.9; 400 pairs 26.3 / 27.4 / 30.8 and 47.4 / 48.0 / 46.9; 528
        // pairs, 1500 positions 230 / 253 / 255; 800 pairs 352 / 338 / 342, 40 positions 98.6 / 98.4 / 104; 4000 pairs, 40
        // positions 47 / 56 / 73.
        int waves;
        if (cap <= 64) waves = 4;
        else if (pairs <= 256) waves = cap <= 256 ? 8 : 16;
        else if (pairs <= 512) waves = 8;
        else waves = cap > 256 && pairs > 768 && pairs <= 2048 ? 8 : 4;
        auto kern = waves == 4 ? k_f32_attn<256> : waves == 8 ? k_f32_attn<512> : k_f32_attn<1024>;
        hipLaunchKernelGGL(kern, dim3(c.n_q_heads, B), dim3(64 * waves), 0, s, qkv, qkv_n, c.n_q_heads, idx, n_ptr, B,
                           b->st<int32_t>(L.pos), view, ao, lanes);
    } else if (hd % 4 == 0) {
        hipLaunchKernelGGL(k_f32_attn_scores<true>, dim3(c.n_q_heads, B), dim3(256), (size_t)(1024 + c.max_pos) * sizeof(float), s, qkv,
                           qkv_n, c.n_q_heads, idx, n_ptr, B, b->st<int32_t>(L.pos), view, ao, lanes);
    } else {
        hipLaunchKernelGGL(k_f32_attn_scores<false>, dim3(c.n_q_heads, B), dim3(256), (size_t)(hd + c.max_pos) * sizeof(float), s, qkv,
                           qkv_n, c.n_q_heads, idx, n_ptr, B, b->st<int32_t>(L.pos), view, ao, 1);
    }
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
    // key and value heads follow the query heads
    rope_gemm(m, kv, b, from_excl + 1, to_incl - from_excl, m->cfg.n_q_heads, b->st<int32_t>(b->L.exited_idx), b->st<int32_t>(b->L.n_exited), s);
    EE_LAUNCH_CHECK();
    return EE_OK;
}
