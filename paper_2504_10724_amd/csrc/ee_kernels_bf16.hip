// ee_kernels_bf16.hip -- the decode step for EE_BF16 models on gfx950.
//
// Data layout
//   * Weight matrices are streamed from HBM exactly once per call, in the tile
//     order ee_pack_weight produces: a 32(out) x 16(in) tile is 1 KiB and is the
//     B operand of one v_mfma_f32_32x32x16_bf16 as it sits in memory (lane l
//     holds output row l%32, inputs 8*(l/32)..+7), so a wave loads it with one
//     fully coalesced 16-byte-per-lane read and no LDS transpose.  Tiles are
//     ordered K-slice-major (tile (r, c) at slot c * R + r): the workgroups of a
//     launch walk K more or less together, so what they fetch at any moment is
//     one contiguous window of the matrix, spread evenly over the HBM channels,
//     instead of addresses a power of two apart.
//   * Activations that feed a matrix product (normalised rows, attention
//     output, SwiGLU product) are written by their producers in the same tile
//     order (32 rows x 16 columns per tile), i.e. as ready-made A operands.
//   * Everything indexed by "i" is in compacted order (i-th active row);
//     the residual stream, the cache, positions and outputs are indexed by row id.
#include "ee_device.h"

#include <float.h>
#include <algorithm>
#include <type_traits>

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Several layers in one launch (blockIdx.z = layer - first layer): used to produce the keys and
// values of all skipped layers at once.  Null tables / zero strides mean a single-layer launch.
struct ZBatch {
    const void* const*  w_tab;     // per layer: packed W_qkv           (device table, index layer - 1)
    const float* const* g_tab;     // per layer: attention-norm gain
    int     z0;                    // table index of blockIdx.z == 0
    int64_t x_stride;              // uint4 units between the layers' activation matrices
    int64_t out_stride;            // floats between the layers' output matrices
};

// two values rounded to nearest even, a in the low half: one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{a, b}), b2));
}

// silu(g) u: expf and an IEEE division, which stay within 1e-7 of the value before it is rounded to bf16.  On the
// hardware's exponential and reciprocal a round of 256 workgroups takes 3 to 5 us less (gate/up of 256 rows at the
// 70B shape 193 against 198 us, of 1024 entries at the 7B shape 175 against 183), but there the exponential's argument
// is rounded as a product with log2 e, an error that grows with |g|: 2.5e-6 of the value at -80.
__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.0f + expf(-g)) * u; }

// ------------------------------------------------------------------ what the decode attention works on
// What a workgroup of the decode attention has to know before its first load from the cache.  The kernel that normalises a
// row for the q|k|v product, or the append kernel where there is one, leaves one per list entry, in launch order, so that
// the attention kernel starts with a single load instead of the chain order -> row -> position -> cache row -> capacity,
// offset (each a trip to memory).
struct AttnJob {
    int32_t entry;      // list entry
    int32_t n_pos;      // positions read
    int32_t cap;        // capacity of the cache row
    int32_t shares;     // workgroups that share its positions, per kv head
    int64_t off;        // positions of the rows before it
    int32_t pos;        // the row's position
    int32_t pad;
};

// Workgroups that share the positions of one list entry and kv head: as many as keep the live (entry, kv head) pairs
// within the 512 that run at a time (two per CU), but two up to 384 pairs, and no more than leave each of the four
// waves two groups of 32 positions.  `most`: what the host launched, from the capacity.  Taken on the device, because
// only there it is known how many rows are left and how long they are: by the capacities alone, 4 of 16 rows of the
// 70B shape took 24 us with their merge (19 now; 19 with twice the shares whatever is live), one row of 2000
// positions 19 (16).  All rows live, attention and merge: 16 rows of the 70B shape 34 us at 1024 workgroups, 31
// here; 37 rows of 2 kv heads, up to 900 positions, 27 and 17; 12 entries of four contexts at the 7B shape (384
// pairs) 64 unshared, 55 in two; 60 entries (480 pairs) of the 70B shape 46 in two, 41 unshared.
__device__ __forceinline__ int attn_shares(int pairs, int n_pos, int most) {
    return max(1, min(min(most, n_pos >> 8), max(512 / pairs, pairs <= 384 ? 2 : 1)));
}

struct JobArgs {        // jobs == nullptr: none are left
    const int32_t* pos; const int32_t* cap; const int64_t* off;
    AttnJob* jobs;
    int n_kv_heads, most;
};

// Called by every thread of a block of norm_threads that works on list entry i of n: its last wave leaves the entry's job
// at the entry's rank by falling position (ties by entry), so that the longest rows start first and the last round of
// workgroups is short.  Batch row b is cache row b.
#define NORM_THREADS 1024
template <class Row>
__device__ __forceinline__ void leave_job(const JobArgs& a, int i, int n, Row row_of) {
    const int wave0 = blockDim.x - 64;
    if (a.jobs == nullptr || (int)threadIdx.x < wave0) return;
    const int row = row_of(i), mine = a.pos[row];
    int before = 0;
    for (int j = threadIdx.x - wave0; j < n; j += 64) {
        const int kj = a.pos[row_of(j)];
        before += (kj > mine || (kj == mine && j < i)) ? 1 : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
    if ((int)threadIdx.x == wave0) {
        const int cap = a.cap[row], n_pos = max(1, min(mine + 1, cap));
        a.jobs[before] = AttnJob{i, n_pos, cap, attn_shares(n * a.n_kv_heads, n_pos, a.most), a.off[row], mine, 0};
    }
}

// ------------------------------------------------------------------ RMSNorm -> A tiles
// The threads of a block normalise one row (hr: d floats) and write it as list entry
// i of the [Mpad][d] activation matrix in tile order.  Every thread reads only the 8-float chunks
// c = threadIdx.x + blockDim.x j, so a caller may have written those same chunks just before.
// One chunk per thread up to d = 8192, and no wave without one but the one that leaves the attention's job (norm_threads): a row's sum
// of squares adds up the waves' in their order, so that waves without a chunk would add nothing, and the smaller blocks of narrower rows fit on a CU side by side
// (1024 rows of 4096 values, 1024 threads / 512: begin and norm 14.2 / 12.7 us, norm 9.5 / 8.8, finish of two K slices 17.3 / 16.7).
// Sum of the squares of a chunk, its fused multiply-adds written out: every kernel that normalises a row (here, the
// finish of a sliced product, the step begin) has to give the same bits, and left to the compiler which of the
// products of a sum are fused differs from kernel to kernel.
__device__ __forceinline__ float sum_sq8(const float4& a, const float4& b) {
    float s = a.x * a.x;
    s = fmaf(a.y, a.y, s); s = fmaf(a.z, a.z, s); s = fmaf(a.w, a.w, s);
    s = fmaf(b.x, b.x, s); s = fmaf(b.y, b.y, s); s = fmaf(b.z, b.z, s); s = fmaf(b.w, b.w, s);
    return s;
}
// block_sum over the waves that the block has (up to NORM_THREADS / 64)
__device__ __forceinline__ float waves_sum(float v, float* smem) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) smem[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = 0.f;
    for (int i = 0; i < (int)blockDim.x >> 6; ++i) t += smem[i];
    return t;
}
// the row as one 8-float chunk (a, b) per thread (d <= 8 NORM_THREADS; zeros in threads past the row)
__device__ __forceinline__ void rmsnorm_chunk(const float4& a, const float4& b, const float* gain, float eps, int d, uint4* out, int i,
                                              float* red) {
    const int c = threadIdx.x;
    const bool has = c < (d >> 3);
    float4 ga = make_float4(0.f, 0.f, 0.f, 0.f), gb = ga;
    if (has) { ga = reinterpret_cast<const float4*>(gain)[2 * c]; gb = reinterpret_cast<const float4*>(gain)[2 * c + 1]; }
    float ss = 0.f;
    if (has) ss += sum_sq8(a, b);
    ss = waves_sum(ss, red);
    const float inv = 1.0f / sqrtf(ss / (float)d + eps);
    if (!has) return;
    uint4 o;
    o.x = pack2((a.x * inv) * ga.x, (a.y * inv) * ga.y);
    o.y = pack2((a.z * inv) * ga.z, (a.w * inv) * ga.w);
    o.z = pack2((b.x * inv) * gb.x, (b.y * inv) * gb.y);
    o.w = pack2((b.z * inv) * gb.z, (b.w * inv) * gb.w);
    out[afrag_chunk(i, c * 8, d >> 4)] = o;
}

__device__ __forceinline__ void rmsnorm_row(const float* hr_, const float* gain, float eps, int d, uint4* out, int i,
                                            float* red /* NORM_THREADS / 64 floats */) {
    const float4* hr = reinterpret_cast<const float4*>(hr_);
    const float4* g4 = reinterpret_cast<const float4*>(gain);
    int n8 = d >> 3;
    int KB = d >> 4;
    if (n8 <= NORM_THREADS) {
        // one chunk per thread (d <= 8192): it stays in registers; same arithmetic, same bits as below
        const int c = threadIdx.x;
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
        if (c < n8) { a = hr[2 * c]; b = hr[2 * c + 1]; }
        rmsnorm_chunk(a, b, gain, eps, d, out, i, red);
        return;
    }
    float ss = 0.f;
    for (int c = threadIdx.x; c < n8; c += blockDim.x) {
        float4 a = hr[2 * c], b = hr[2 * c + 1];
        ss += sum_sq8(a, b);
    }
    ss = waves_sum(ss, red);
    float inv = 1.0f / sqrtf(ss / (float)d + eps);
    for (int c = threadIdx.x; c < n8; c += blockDim.x) {
        float4 a = hr[2 * c], b = hr[2 * c + 1];
        float4 ga = g4[2 * c], gb = g4[2 * c + 1];
        uint4 o;
        o.x = pack2((a.x * inv) * ga.x, (a.y * inv) * ga.y);
        o.y = pack2((a.z * inv) * ga.z, (a.w * inv) * ga.w);
        o.z = pack2((b.x * inv) * gb.x, (b.y * inv) * gb.y);
        o.w = pack2((b.z * inv) * gb.z, (b.w * inv) * gb.w);
        out[afrag_chunk(i, c * 8, KB)] = o;
    }
}

// one block per list entry i; out is the [Mpad][d] activation matrix in tile order
__global__ void __launch_bounds__(NORM_THREADS)
k_bf16_rmsnorm(const float* __restrict__ h, const int32_t* __restrict__ idx, const int32_t* __restrict__ n_ptr,
               int B, int near, const float* __restrict__ gain, float eps, int d, uint4* __restrict__ out, ZBatch zb, JobArgs ja) {
    __shared__ float red[NORM_THREADS / 64];
    int i = entry_of_block(blockIdx.x, near);
    int n = min(*n_ptr, B);
    if (i >= n) return;
    leave_job(ja, i, n, [&](int j) { return idx[j]; });
    if (zb.g_tab) gain = zb.g_tab[zb.z0 + blockIdx.z];
    out += (int64_t)blockIdx.z * zb.x_stride;
    rmsnorm_row(h + (int64_t)idx[i] * d, gain, eps, d, out, i, red);
}

// ------------------------------------------------------------------ step begin and first norm in one launch
// What k_begin_step (CTX = false) and k_prefill_begin (CTX = true) do for row or entry i, and the operand row of the
// first layer's q|k|v product, RMSNorm of the embedding that was just read: one launch and one pass over h less
// (1999 entries of 8192 values: 22 + 25 us as two launches).  d <= 8 NORM_THREADS.
struct BeginArgs {
    const int32_t* tok; const int32_t* pos; const int32_t* seq;      // pos, seq: context pass
    int n, n_seq, V;
    const uint4* emb;
    float* h;
    int32_t *s_tok, *s_pos, *kv_seq, *active_idx, *n_active, *n_exited, *out_layer, *status;
};

template <bool CTX>
__global__ void __launch_bounds__(NORM_THREADS)
k_bf16_begin_norm(BeginArgs g, int near, const float* __restrict__ gain, float eps, int d, uint4* __restrict__ xout, JobArgs ja) {
    __shared__ float red[NORM_THREADS / 64];
    const int i = entry_of_block(blockIdx.x, near);
    if (i >= g.n) return;
    if constexpr (!CTX) leave_job(ja, i, g.n, [](int j) { return j; });
    int t = g.tok[i];
    const bool bad = t < 0 || t >= g.V;
    if (threadIdx.x == 0) {
        if (bad) atomicOr(g.status, 2);
        if constexpr (CTX) {
            int p = g.pos[i], sq = g.seq[i];
            if (sq < 0 || sq >= g.n_seq) {
                atomicOr(g.status, 1);
                sq = 0;
                p = -1;
            }
            g.s_tok[i] = bad ? 0 : t;
            g.s_pos[i] = p;
            g.kv_seq[i] = sq;
        } else {
            g.out_layer[i] = 0;
        }
        g.active_idx[i] = i;
        if (i == 0) { *g.n_active = g.n; *g.n_exited = 0; }
    }
    if (bad) t = 0;
    const int c = threadIdx.x;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (c < (d >> 3)) {
        const uint4 v = g.emb[(int64_t)t * (d >> 3) + c];
        a = make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
        b = make_float4(__uint_as_float(v.z << 16), __uint_as_float(v.z & 0xffff0000u), __uint_as_float(v.w << 16), __uint_as_float(v.w & 0xffff0000u));
        float4* hp = reinterpret_cast<float4*>(g.h + (int64_t)i * d + c * 8);
        hp[0] = a;
        hp[1] = b;
    }
    rmsnorm_chunk(a, b, gain, eps, d, xout, i, red);
}

// ------------------------------------------------------------------ weight-streaming MFMA GEMM
// out[i][j] = sum_k X[i][k] W[j][k] for the first n rows of X (n read on the device), at most 64.
// A workgroup has WK waves and owns NS consecutive 32-column tile-rows of W and all MS 32-row tiles
// of X; wave wk takes the wk-th slice of the K range, and the WK partial sums of a tile are added in
// a fixed order through LDS.
// 16 bytes that this launch reads once (weights, cached keys and values): a non-temporal load.
// Measured: streams of such loads run 10-13 % faster than ordinary ones, which hold a line of
// the vector cache while they are in flight.
__device__ __forceinline__ uint4 load_nt(const uint4* p) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    u32x4 r = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(r.x, r.y, r.z, r.w);
}

enum { EPI_STORE = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_EXIT = 3 };

struct EpiArgs {
    float*         out;       // STORE: [i][ldo]; RESID: residual stream [row id][ldo]
    int            ldo;
    const int32_t* idx;       // row id of list entry i
    const float*   row_scale; // EXIT: per row id
    float*         part_max;  // EXIT: [i][n_part]
    float*         part_sum;
    int32_t*       part_arg;
    int            n_part;
    float*         dbg_logits;// EXIT, nullable: [i][ldo]
    bf16_t*        act;       // SWIGLU: [Mpad][F] in tile order
    int            KB_act;    // F / 16
};

template <int MS, int NS, int WK, int EPI>
__global__ void __launch_bounds__(64 * WK)
k_bf16_gemm(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp, int KB, int NB_total, int NBs, int nb_off,
            const int32_t* __restrict__ n_ptr, int B, EpiArgs ep, ZBatch zb) {
    constexpr int IPW = 16 / WK;   // accumulator registers each wave finishes after the reduction
    constexpr int GD = 4;          // K tiles per load group
    __shared__ float red[WK * NS * 16 * 64];
    const int n = min(*n_ptr, B);
    if (n <= 0) return;
    if (zb.w_tab) Wp = reinterpret_cast<const uint4*>(zb.w_tab[zb.z0 + blockIdx.z]);
    Xp += (int64_t)blockIdx.z * zb.x_stride;
    ep.out += (int64_t)blockIdx.z * zb.out_stride;
    const int mbs = min(MS, (n + 31) >> 5);
    const int lane = threadIdx.x & 63, wk = threadIdx.x >> 6;
    const int nb0 = blockIdx.x * NS;
    const int kb_lo = (int)(((int64_t)KB * wk) / WK), kb_hi = (int)(((int64_t)KB * (wk + 1)) / WK);
    const uint4* xw = Xp + lane;
    const uint4* ww = Wp + (int64_t)(nb_off + nb0) * 64 + lane;   // tile (r, c) sits at slot c * NBs + r
    const bool has_cols = nb0 + NS <= NB_total;   // uniform over the workgroup

    floatx16 acc[MS][NS];
#pragma unroll
    for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int ns = 0; ns < NS; ++ns)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ms][ns][r] = 0.f;

    if (has_cols) {
        // groups of GD K tiles, the next group's W and X tiles in flight while the current one is
        // multiplied (dead row tiles re-read a live one, so the loads need no branch); groups twice
        // as deep change nothing: with one row tile per wave half of what a CU requests is X
        struct Group { uint4 w[GD][NS]; uint4 x[GD][MS]; };
        auto load_group = [&](int kb) -> Group {
            Group g;
#pragma unroll
            for (int u = 0; u < GD; ++u) {
#pragma unroll
                for (int ns = 0; ns < NS; ++ns) g.w[u][ns] = load_nt(ww + ((int64_t)(kb + u) * NBs + ns) * 64);
#pragma unroll
                for (int ms = 0; ms < MS; ++ms) g.x[u][ms] = xw[((int64_t)min(ms, mbs - 1) * KB + kb + u) * 64];
            }
            return g;
        };
        auto mul_group = [&](const Group& g) {
#pragma unroll
            for (int u = 0; u < GD; ++u)
#pragma unroll
                for (int ms = 0; ms < MS; ++ms) {
                    if (ms < mbs) {
#pragma unroll
                        for (int ns = 0; ns < NS; ++ns)
                            acc[ms][ns] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(g.x[u][ms]), as_bf16x8(g.w[u][ns]),
                                                                                   acc[ms][ns], 0, 0, 0);
                    }
                }
        };
        int kb = kb_lo;
        const int n_groups = (kb_hi - kb_lo) / GD;
        if (n_groups > 0) {
            Group cur = load_group(kb);
            for (int gi = 1; gi < n_groups; ++gi) {
                Group nxt = load_group(kb + GD);
                mul_group(cur);
                cur = nxt;
                kb += GD;
            }
            mul_group(cur);
            kb += GD;
        }
        for (; kb < kb_hi; ++kb) {
#pragma unroll
            for (int ms = 0; ms < MS; ++ms) {
                if (ms < mbs) {
                    uint4 a = xw[((int64_t)ms * KB + kb) * 64];
#pragma unroll
                    for (int ns = 0; ns < NS; ++ns) {
                        uint4 bwv = ww[((int64_t)kb * NBs + ns) * 64];
                        acc[ms][ns] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), as_bf16x8(bwv),
                                                                               acc[ms][ns], 0, 0, 0);
                    }
                }
            }
        }
    }

    // ---- reduction over the K slices and epilogue, one 32-row tile at a time
#pragma unroll
    for (int ms = 0; ms < MS; ++ms) {
        if (ms >= mbs) break;              // uniform over the workgroup
        float v[NS][IPW];
#pragma unroll
        for (int ns = 0; ns < NS; ++ns)
#pragma unroll
            for (int r = 0; r < 16; ++r) red[((wk * NS + ns) * 16 + r) * 64 + lane] = acc[ms][ns][r];
        __syncthreads();
#pragma unroll
        for (int ns = 0; ns < NS; ++ns)
#pragma unroll
            for (int ii = 0; ii < IPW; ++ii) {
                float s = 0.f;
#pragma unroll
                for (int k2 = 0; k2 < WK; ++k2) s += red[((k2 * NS + ns) * 16 + (wk * IPW + ii)) * 64 + lane];
                v[ns][ii] = s;
            }
        __syncthreads();
        if (!has_cols) continue;
#pragma unroll
        for (int ii = 0; ii < IPW; ++ii) {
            const int r = wk * IPW + ii;   // accumulator register index 0..15
            const int row = 32 * ms + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            const bool live = row < n;
            const int cl = lane & 31;
            if (EPI == EPI_STORE) {
                if (live) {
#pragma unroll
                    for (int ns = 0; ns < NS; ++ns)
                        ep.out[(int64_t)row * ep.ldo + 32 * (nb0 + ns) + cl] = v[ns][ii];
                }
            } else if (EPI == EPI_RESID) {
                if (live) {
                    float* hr = ep.out + (int64_t)ep.idx[row] * ep.ldo;
#pragma unroll
                    for (int ns = 0; ns < NS; ++ns) hr[32 * (nb0 + ns) + cl] += v[ns][ii];
                }
            } else if (EPI == EPI_SWIGLU) {
                // rows 2j / 2j+1 of the gate/up matrix are gate / up of output j: neighbouring lanes
                // (same batch row) hold them, the even lane writes the product
#pragma unroll
                for (int ns = 0; ns < NS; ++ns) {
                    const float mine = v[ns][ii], other = __shfl_xor(mine, 1, 64);
                    const float gt = (cl & 1) ? other : mine, up = (cl & 1) ? mine : other;
                    const float a = silu_mul(gt, up);
                    const int col = 16 * (nb0 + ns) + (cl >> 1);
                    if (live && !(cl & 1)) ep.act[afrag_chunk(row, col & ~7, ep.KB_act) * 8 + (col & 7)] = f32_to_bf16(a);
                }
            } else {   // EPI_EXIT
                int col = 32 * nb0 + cl;
                float z = live ? v[0][ii] * ep.row_scale[ep.idx[row]] : 0.f;
                if (live && ep.dbg_logits) ep.dbg_logits[(int64_t)row * ep.ldo + col] = z;
                float mx = z;
                int arg = col;
#pragma unroll
                for (int o = 16; o > 0; o >>= 1) {
                    float m2 = __shfl_xor(mx, o, 64);
                    int a2 = __shfl_xor(arg, o, 64);
                    if (m2 > mx || (m2 == mx && a2 < arg)) { mx = m2; arg = a2; }
                }
                float se = expf(z - mx);
#pragma unroll
                for (int o = 16; o > 0; o >>= 1) se += __shfl_xor(se, o, 64);
                if (live && cl == 0) {
                    int64_t at = (int64_t)row * ep.n_part + nb0;
                    ep.part_max[at] = mx; ep.part_sum[at] = se; ep.part_arg[at] = arg;
                }
            }
        }
    }
}

// ------------------------------------------------------------------ large-batch MFMA GEMM
// 256-row tiles (up to 256 rows per row group), 128 or 256 columns wide, one K slice per
// workgroup, operands fed by LDS-DMA loads (k_bf16_gemm_dma8, k_bf16_gemm_dma2 below).  When K
// is sliced, every slice writes an fp32 partial tile into its own plane and a later kernel adds
// the planes in slice order, so the result does not depend on timing and needs no atomics.
#define BIG_THREADS 256
struct Half { uint4 v[4]; };   // A operands of one K half: 4 row tiles

// One 32x32x16 step of a result tile.  A and B operands have the same register layout, so handing
// them over in the other order gives the transposed tile at no cost: a lane then holds 16 columns of
// ONE batch row (of the tile-row's 32 columns, those at 8 q + 4 (lane / 32) + s, q, s = 0..3, in
// register 4 q + s; lane ^ 32 holds the others).  The exit head wants that: the row statistics
// (maximum, its column, sum of exponentials) need one exchange between the two half-waves instead of
// a 32-lane butterfly per accumulator register (measured: 83 of 230 us of the exit-head product).
// So does the SwiGLU epilogue: gate row j and up row j of the gate/up matrix are neighbouring
// columns, i.e. two registers of one lane.
template <int EPI>
__device__ __forceinline__ floatx16 tile_mfma(const uint4& x, const uint4& w, const floatx16& acc) {
    if constexpr (EPI == EPI_EXIT || EPI == EPI_SWIGLU)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(w), as_bf16x8(x), acc, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(x), as_bf16x8(w), acc, 0, 0, 0);
}

// exp(d), d <= 0 (or NaN) a logit's distance to the tile's maximum: the hardware's base-2 exponential of t = d log2 e, rounded,
// times 1 + r with r = d - t ln 2 what the rounding left; within 1.4e-7 of the value.  (The base-2 exponential alone is off by the
// rounding of t, up to 6e-8 d, and equal distances make the same error, so that it does not average out of a sum.)
// d = -infinity: t is too, r is clipped, the result is 0.  expf, which reduces its argument and tests its range, takes two to
// three times the instructions for each of a lane's up to 128 logits: head of 192 rows at the 70B shape 134.4 us with it, 132.0 so,
// of 200 rows at the 7B shape 86.2 and 84.1.
__device__ __forceinline__ float exp_below(float d) {
    const float t = d * 1.44269504088896340736f;
    const float r = fmaf(-t, -1.90465429995776e-9f, fmaf(-t, 0.693147182464599609f, d));
    const float e = __builtin_amdgcn_exp2f(t);
    return fmaf(e, fminf(r, 1.0f), e);
}

// EXIT: the logit scale of list entry `row` of n, asked for at the start of a kernel, beside its first operands.  In the epilogue
// each was two trips to memory, and a wait for all stores before it: loads and stores return in order.  Head and compaction of 192
// rows at the 70B shape 130.3 -> 129.0 us.
template <int EPI>
__device__ __forceinline__ float exit_scale(const EpiArgs& ep, int row, int n) {
    if constexpr (EPI == EPI_EXIT) return ep.row_scale[ep.idx[min(row, n - 1)]];
    else return 0.f;
}

// v: the 32x32 result of tile-row nb (columns 32 nb ..) for rows row0 .. row0+31; every lane of the wave calls it.  sc (EXIT):
// exit_scale of row row0 + lane % 32
template <int EPI>
__device__ __forceinline__ void epilogue_one(const EpiArgs& ep, const floatx16& v, int row0, int n, int nb, int lane, float sc = 0.f) {
    const int cl = lane & 31;
    if constexpr (EPI == EPI_EXIT) {
        // transposed tile: this lane holds batch row row0 + cl
        const int row = row0 + cl;
        const bool live = row < n;
        const int col0 = 32 * nb + 4 * (lane >> 5);
        float z[16];
        float mx = -FLT_MAX;
        int arg = col0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int col = col0 + 8 * (r >> 2) + (r & 3);        // rising with r: > keeps the lowest column
            z[r] = v[r] * sc;
            if (z[r] > mx) { mx = z[r]; arg = col; }
        }
        if (ep.dbg_logits && live) {
            // registers 4 q .. 4 q + 3 are neighbouring columns of this lane's row: 16 bytes per store (V is a
            // multiple of 32; single values where the caller's array is not aligned for that)
            float* zp = ep.dbg_logits + (int64_t)row * ep.ldo + col0;
            if (((uintptr_t)ep.dbg_logits & 15) == 0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) *reinterpret_cast<float4*>(zp + 8 * q) = make_float4(z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]);
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) zp[8 * (r >> 2) + (r & 3)] = z[r];
            }
        }
        const float m2 = __shfl_xor(mx, 32, 64);
        const int a2 = __shfl_xor(arg, 32, 64);
        if (m2 > mx || (m2 == mx && a2 < arg)) { mx = m2; arg = a2; }
        float ex[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) ex[r] = exp_below(z[r] - mx);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1)                       // in pairs: four roundings on a term's way; one by one fifteen
#pragma unroll
            for (int r = 0; r < o; ++r) ex[r] += ex[r + o];
        float se = ex[0];
        se += __shfl_xor(se, 32, 64);
        if (live && lane < 32) {
            const int64_t at = (int64_t)row * ep.n_part + nb;
            ep.part_max[at] = mx; ep.part_sum[at] = se; ep.part_arg[at] = arg;
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
        // transposed tile of the gate/up matrix (row 2j gate, row 2j+1 up of output j): registers
        // 4q, 4q+1 are gate and up of output 4q + 2h (h = lane / 32) of the tile-row's 16 outputs,
        // registers 4q+2, 4q+3 those of output 4q + 2h + 1.  The half-waves swap two packed pairs so
        // that lane < 32 writes outputs 0..7 and lane >= 32 outputs 8..15 of its batch row as one
        // 16-byte chunk of the next product's operand tiles.
        const int row = row0 + cl, h = lane >> 5;
        uint32_t d[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float g0 = v[4 * q], u0 = v[4 * q + 1], g1 = v[4 * q + 2], u1 = v[4 * q + 3];
            d[q] = pack2(silu_mul(g0, u0), silu_mul(g1, u1));
        }
        const uint32_t r0 = __shfl_xor(h ? d[0] : d[2], 32, 64), r1 = __shfl_xor(h ? d[1] : d[3], 32, 64);
        const uint4 o = h ? make_uint4(r0, d[2], r1, d[3]) : make_uint4(d[0], r0, d[1], r1);
        if (row < n) reinterpret_cast<uint4*>(ep.act)[afrag_chunk(row, 16 * nb + 8 * h, ep.KB_act)] = o;
    } else if constexpr (EPI == EPI_RESID) {
        // h[row id] += v.  All row ids, then all old values, then the stores: taken one result at a time (the stores
        // may alias the loads, so the compiler cannot) the 128 results of a lane were 128 trips to memory, 90 of
        // the 306 us of the O projection of 1999 entries at the 70B shape.
        float* at[16];
        float old[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = row0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            at[r] = ep.out + (int64_t)ep.idx[min(row, n - 1)] * ep.ldo + 32 * nb + cl;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) old[r] = *at[r];
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (row0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3) < n) *at[r] = old[r] + v[r];
    } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = row0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (row < n) ep.out[(int64_t)row * ep.ldo + 32 * nb + cl] = v[r];      // EPI_STORE
        }
    }
}

template <int EPI>
__device__ __forceinline__ void epilogue_tile(const EpiArgs& ep, const floatx16& v0, const floatx16& v1, int row0,
                                              int n, int nb, int lane, float sc) {
    epilogue_one<EPI>(ep, v0, row0, n, nb, lane, sc);
    epilogue_one<EPI>(ep, v1, row0, n, nb + 1, lane, sc);
}

// ------------------------------------------------------------------ results of 16x16x32 MFMAs
// A 32 x 32 block of results as 2 x 2 transposed 16x16 tiles (W is the first operand): v[i][u], lane l: batch row 16 i + l % 16,
// columns 16 u + 4 (l / 16) + s of the block in register s.  What epilogue_one does with a 32x32 tile, to the same bits:
// a 16x16x32 MFMA adds up its 32 products as two 32x32x16 do.
__device__ __forceinline__ floatx4 mfma16(const uint4& x, const uint4& w, const floatx4& acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w), as_bf16x8(x), acc, 0, 0, 0);
}
// lanes below 32: a of both halves of the wave in (x, y), lanes from 32 on: b
__device__ __forceinline__ void halves(float a, float b, float& x, float& y) {
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    x = __uint_as_float(t[0]); y = __uint_as_float(t[1]);
}
// the value of lane ^ 16
__device__ __forceinline__ uint32_t other_row(uint32_t v) {
    const auto t = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (threadIdx.x & 16) ? t[0] : t[1];
}

// v: NB blocks of rows row0 .. row0 + 31, columns 32 nb .. ; every lane of the wave calls it
// sc (EXIT): exit_scale of rows row0 + 16 i + lane % 16
template <int EPI, int NB>
__device__ __forceinline__ void epilogue_blocks(const EpiArgs& ep, const floatx4 (&v)[2][2 * NB], int row0, int n, int nb0, int nb_live,
                                                int lane, const float* sc) {
    const int r16 = lane & 15, g = lane >> 4;
    if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b >= nb_live) break;
            // a lane has outputs 2 g, 2 g + 1 of the 8 of a tile, for four tiles k = 2 i + u; the lanes of a row swap so that
            // group k has all of tile k: one 16-byte chunk of the next product's operand tiles
            uint32_t d[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const floatx4& t = v[k >> 1][2 * b + (k & 1)];
                d[k] = pack2(silu_mul(t[0], t[1]), silu_mul(t[2], t[3]));
            }
            const auto a = __builtin_amdgcn_permlane32_swap(d[0], d[2], false, false), c = __builtin_amdgcn_permlane32_swap(d[1], d[3], false, false);
            const auto lo = __builtin_amdgcn_permlane16_swap(a[0], c[0], false, false), hi = __builtin_amdgcn_permlane16_swap(a[1], c[1], false, false);
            const int row = row0 + 16 * (g >> 1) + r16;
            if (row < n)
                reinterpret_cast<uint4*>(ep.act)[afrag_chunk(row, 16 * (nb0 + b) + 8 * (g & 1), ep.KB_act)] = make_uint4(lo[0], lo[1], hi[0], hi[1]);
        }
    } else if constexpr (EPI == EPI_EXIT) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b >= nb_live) break;
            const int col0 = 32 * (nb0 + b) + 4 * g;
            float z[2][8], mx[2];
            int arg[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                mx[i] = -FLT_MAX;
                arg[i] = col0;
#pragma unroll
                for (int k = 0; k < 8; ++k) {                 // column 16 (k / 4) + k % 4 from col0: rising, > keeps the lowest
                    z[i][k] = v[i][2 * b + (k >> 2)][k & 3] * sc[i];
                    if (z[i][k] > mx[i]) { mx[i] = z[i][k]; arg[i] = col0 + 16 * (k >> 2) + (k & 3); }
                }
                if (ep.dbg_logits && row0 + 16 * i + r16 < n) {
                    // 16 bytes per store (V is a multiple of 32; single values where the caller's array is not aligned for that)
                    float* zp = ep.dbg_logits + (int64_t)(row0 + 16 * i + r16) * ep.ldo + col0;
                    if (((uintptr_t)ep.dbg_logits & 15) == 0) {
#pragma unroll
                        for (int u = 0; u < 2; ++u) *reinterpret_cast<float4*>(zp + 16 * u) = make_float4(z[i][4 * u], z[i][4 * u + 1], z[i][4 * u + 2], z[i][4 * u + 3]);
                    } else {
#pragma unroll
                        for (int k = 0; k < 8; ++k) zp[16 * (k >> 2) + (k & 3)] = z[i][k];
                    }
                }
            }
            // lanes below 32 go on with the rows of i = 0, the others with those of i = 1
            float ma, mb, m;
            halves(mx[0], mx[1], ma, mb);
            const auto ai = __builtin_amdgcn_permlane32_swap((uint32_t)arg[0], (uint32_t)arg[1], false, false);
            int at = (int)ai[0];
            m = ma;
            if (mb > m || (mb == m && (int)ai[1] < at)) { m = mb; at = (int)ai[1]; }
            const float mo = __uint_as_float(other_row(__float_as_uint(m)));
            const int ao = (int)other_row((uint32_t)at);
            if (mo > m || (mo == m && ao < at)) { m = mo; at = ao; }
            float mr[2];
            halves(m, m, mr[0], mr[1]);                       // the maximum of each lane's two rows
            float e[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {                     // in pairs, in epilogue_one's order
                float x, y;
                halves(exp_below(z[0][s] - mr[0]) + exp_below(z[0][4 + s] - mr[0]), exp_below(z[1][s] - mr[1]) + exp_below(z[1][4 + s] - mr[1]), x, y);
                e[s] = x + y;
            }
            float se = (e[0] + e[2]) + (e[1] + e[3]);
            se += __uint_as_float(other_row(__float_as_uint(se)));
            const int row = row0 + 16 * (lane >> 5) + r16;
            if (row < n && !(lane & 16)) {
                const int64_t o = (int64_t)row * ep.n_part + nb0 + b;
                ep.part_max[o] = m; ep.part_sum[o] = se; ep.part_arg[o] = at;
            }
        }
    } else if constexpr (EPI == EPI_RESID) {
        // h[row id] += v: all old values, then the stores (see epilogue_one)
        float* at[2];
        float4 old[2][2 * NB];
#pragma unroll
        for (int i = 0; i < 2; ++i) at[i] = ep.out + (int64_t)ep.idx[min(row0 + 16 * i + r16, n - 1)] * ep.ldo + 32 * nb0 + 4 * g;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int u = 0; u < 2 * NB; ++u)
                if ((u >> 1) < nb_live) old[i][u] = *reinterpret_cast<const float4*>(at[i] + 16 * u);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (row0 + 16 * i + r16 < n) {
#pragma unroll
                for (int u = 0; u < 2 * NB; ++u)
                    if ((u >> 1) < nb_live)
                        *reinterpret_cast<float4*>(at[i] + 16 * u) = make_float4(old[i][u].x + v[i][u][0], old[i][u].y + v[i][u][1],
                                                                                 old[i][u].z + v[i][u][2], old[i][u].w + v[i][u][3]);
            }
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = row0 + 16 * i + r16;
            if (row >= n) continue;
            float* o = ep.out + (int64_t)row * ep.ldo + 32 * nb0 + 4 * g;
#pragma unroll
            for (int u = 0; u < 2 * NB; ++u)
                if ((u >> 1) < nb_live) *reinterpret_cast<float4*>(o + 16 * u) = make_float4(v[i][u][0], v[i][u][1], v[i][u][2], v[i][u][3]);
        }
    }
}

// ------------------------------------------------------------------ tile GEMMs fed by LDS-DMA loads
// No operand passes through registers on its way in: the waves of a workgroup send the X and W
// tiles of a 32-wide K stage straight from global memory into LDS (global_load_lds_dwordx4: 64
// lanes x 16 B per instruction, lane l lands at byte 16 l of the slot), and all MFMA operands are
// read from LDS.  A load that returns into registers holds up the matrix pipe of its SIMD while
// it writes back (measured: streaming time and MFMA time add up, even across waves); a load
// into LDS does not, so here the weight stream runs under the MFMAs.  The loads of a stage are
// issued one behind each MFMA group (a burst would queue up in the vector-memory path and hold the
// wave).  The compiler does not see these loads, so it adds no wait of its own; the waits are
// written out.  Loads past the end of the K slice re-read its last stage.
// Which (row group, column tile x K slice) a workgroup takes.  One row group: blockIdx.x is the
// unit.  Several row groups (context pass; the grid is then one-dimensional with gridDim.x =
// 8 ceil(units / 8) x row groups): workgroups are handed to the 8 XCDs round-robin, each XCD has
// its own L2, and the row groups of a unit read the same weight tiles, so they get block numbers
// 8 apart: same XCD, started one after the other, and the tiles come from HBM once, not once
// per row group.  unit = -1: a block past the last unit.
__device__ __forceinline__ void tile_of_block(int units, int& rg, int& unit) {
    if (gridDim.y == 1 && (int)gridDim.x > units) {
        const int u8 = (units + 7) / 8 * 8, R = gridDim.x / u8;
        const int x = blockIdx.x & 7, q = blockIdx.x >> 3;
        rg = q % R;
        unit = (q / R) * 8 + x;
        if (unit >= units) unit = -1;
    } else {
        rg = blockIdx.y;
        unit = blockIdx.x;
    }
}

// tile and lds_byte are the same in all lanes; going through readfirstlane makes that explicit, so
// that both end up in scalar registers whatever the optimiser did to the address arithmetic
// NT: the tile is read once per launch (weights): a non-temporal load, which does not hold a line of
// the vector cache while it is in flight; activations, which every workgroup re-reads, stay cacheable
template <bool NT = false>
__device__ __forceinline__ void dma_tile(const uint4* tile, unsigned lane_bytes, unsigned lds_byte) {
    const uint64_t a = reinterpret_cast<uint64_t>(tile);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    const uint64_t base = ((uint64_t)hi << 32) | lo;
    const uint32_t slot = __builtin_amdgcn_readfirstlane(lds_byte);
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(slot), "v"(lane_bytes), "s"(base)
                     : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(slot), "v"(lane_bytes), "s"(base)
                     : "memory");
}

// ------------------------------------------------------------------ 128-column tile fed by LDS-DMA loads
// 256 rows x 128 columns per workgroup, waves 2 x 2: wave (wm, wn) owns rows 128 wm .. +127
// and columns 64 wn .. +63 (4 x 2 MFMA tiles, 128 accumulator registers).  LDS: 6 stage buffers x 24 slots: X tile (row tile m, K half kk)
// at 2 m + kk, W tile (column tile nb of the 4, K half kk) at 16 + 2 nb + kk.  A wave sends up to 4 X
// tiles (those of its live row tiles: against re-reading a live tile in place of a dead one, the
// exit head takes 7-10 % less up to 64 rows and QKV 3-5 %) and 2 W tiles per stage and reads the 8 + 4 it needs.  For products with few columns
// (QKV, O projection, exit head) it gives twice as many workgroups per K slice as the 256-column tile.
// Its stages are short (16 MFMAs per wave), so a stage is requested five stages ahead, not three:
// measured against three it takes 5 % off the QKV product at 256 rows and 14 % at 64.
struct BHalf { uint4 v[2]; };

template <int EPI>
__global__ void __launch_bounds__(BIG_THREADS, 1)
k_bf16_gemm_dma2(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp, int KB, int NBs, int nb_off,
                 int n_tiles, int splits, const int32_t* __restrict__ n_ptr, int B, float* __restrict__ partial,
                 int64_t part_plane, int part_ld, EpiArgs ep, ZBatch zb) {
    __shared__ uint4 lds[6][24][64];          // six stage buffers: a stage is requested five stages ahead
    const int n = min(*n_ptr, B);
    int rg, unit;
    tile_of_block(n_tiles * splits, rg, unit);
    if (unit < 0) return;
    const int row_base = rg * 256;
    if (row_base >= n) return;
    if (zb.w_tab) Wp = reinterpret_cast<const uint4*>(zb.w_tab[zb.z0 + blockIdx.z]);
    Xp += (int64_t)blockIdx.z * zb.x_stride;
    ep.out += (int64_t)blockIdx.z * zb.out_stride;
    const int mbs = min(8, (n - row_base + 31) >> 5);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int cnt = max(0, min(4, mbs - 4 * wm));            // live 32-row tiles of this wave
    const int tile = unit / splits, sp = unit % splits;
    const int nbw = (tile * 2 + wn) * 2;                     // first of this wave's two tile-rows of W
    const int KS4 = KB >> 3;
    const int ks_lo = 4 * (int)(((int64_t)KS4 * sp) / splits), ks_hi = 4 * (int)(((int64_t)KS4 * (sp + 1)) / splits);
    const int T = ks_hi - ks_lo;                             // stages of this slice: a positive multiple of 4
    const uint4* xg = Xp + ((int64_t)rg * 8 * KB) * 64;
    const uint4* wg = Wp + (int64_t)(nb_off + tile * 4) * 64;   // the tile's four tile-rows of W
    const unsigned lane_bytes = (unsigned)lane * 16u;
    const unsigned lds0 = (unsigned)(size_t)&lds[0][0][0];

    float sc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) sc[i] = exit_scale<EPI>(ep, row_base + 32 * (4 * wm + i) + (lane & 31), n);

    floatx16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // j-th load of a stage: j = 0..3 X tiles (row tile 2 wave + j/2, K half j%2; sent only if that
    // row tile is live); j = 4, 5 the W slots 2 wave + (j - 4) of the stage's eight (column tile
    // q/2, K half q%2).  A tile's address is the stage's base pointer (scalar, computed once per
    // stage) plus a lane offset that is the same in every stage, so a load costs few instructions.
    unsigned voff[6];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int m = min(2 * wave + (j >> 1), mbs - 1);
        voff[j] = lane_bytes + ((unsigned)(m * KB + (j & 1)) << 10);
    }
#pragma unroll
    for (int j = 4; j < 6; ++j) {
        const int q = 2 * wave + (j - 4), nb = q >> 1, kk = q & 1;
        voff[j] = lane_bytes + ((unsigned)(kk * NBs + nb) << 10);
    }
    auto x_base = [&](int t) { return xg + (int64_t)(2 * (ks_lo + min(t, T - 1))) * 64; };
    auto w_base = [&](int t) { return wg + (int64_t)(2 * (ks_lo + min(t, T - 1))) * NBs * 64; };
    auto issue = [&](const uint4* xs, const uint4* ws, int buf, int j) {
        if (j < 4) dma_tile(xs, voff[j], lds0 + (unsigned)((buf * 24 + (2 * wave + (j >> 1)) * 2 + (j & 1)) << 10));
        else dma_tile<true>(ws, voff[j], lds0 + (unsigned)((buf * 24 + 16 + 2 * wave + (j - 4)) << 10));
    };
    Half a0, a1;
    BHalf b0, b1;
    auto rd_a = [&](Half& o, int buf, int kk, int i) { o.v[i] = (&lds[0][0][lane] + buf * (24 * 64))[((4 * wm + i) * 2 + kk) * 64]; };
    auto rd_b = [&](BHalf& o, int buf, int kk) {
        const uint4* p = &lds[0][0][lane] + buf * (24 * 64);
        o.v[0] = p[(16 + (2 * wn) * 2 + kk) * 64];
        o.v[1] = p[(16 + (2 * wn + 1) * 2 + kk) * 64];
    };
    auto mf_all = [&](const Half& a, const BHalf& bw, int i) {
        acc[i][0] = tile_mfma<EPI>(a.v[i], bw.v[0], acc[i][0]);
        acc[i][1] = tile_mfma<EPI>(a.v[i], bw.v[1], acc[i][1]);
    };
    auto mf_some = [&](const Half& a, const BHalf& bw, int i) {
        if (i < cnt) mf_all(a, bw, i);
    };
#define SB __builtin_amdgcn_sched_barrier(0);
// three stages of this wave's loads (VM of them) may stay in flight: everything up to stage t+2 has landed
#define STAGE_END(VM) asm volatile("s_waitcnt vmcnt(" #VM ") lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // bc / bn / bi: buffers of the current stage, the next one and the one being requested (stage + 5);
    // six buffers and an unroll of four do not divide, so the indices are counted at run time.
    // XL: how many of this wave's two row tiles are live and fetched
#define DMA2_STAGE(MF, XL, VM, U)                                                             \
    { const uint4* xs_ = x_base(t0 + (U) + 5); const uint4* ws_ = w_base(t0 + (U) + 5);       \
    MF(a0, b0, 0); SB if (XL >= 1) issue(xs_, ws_, bi, 0); rd_a(a1, bc, 1, 0); rd_a(a1, bc, 1, 1); rd_b(b1, bc, 1); SB \
    MF(a0, b0, 1); SB if (XL >= 1) issue(xs_, ws_, bi, 1); rd_a(a1, bc, 1, 2); rd_a(a1, bc, 1, 3); SB \
    MF(a0, b0, 2); SB if (XL >= 2) issue(xs_, ws_, bi, 2); SB                                 \
    MF(a0, b0, 3); SB if (XL >= 2) issue(xs_, ws_, bi, 3); SB                                 \
    MF(a1, b1, 0); SB issue(xs_, ws_, bi, 4); rd_a(a0, bn, 0, 0); rd_a(a0, bn, 0, 1); rd_b(b0, bn, 0); SB \
    MF(a1, b1, 1); SB issue(xs_, ws_, bi, 5); rd_a(a0, bn, 0, 2); rd_a(a0, bn, 0, 3); SB      \
    MF(a1, b1, 2); SB                                                                         \
    MF(a1, b1, 3); SB                                                                         \
    STAGE_END(VM) }                                                                           \
    bc = bn; bn = bn == 5 ? 0 : bn + 1; bi = bi == 5 ? 0 : bi + 1;
#define DMA2_LOOP(MF, XL, VM) \
    for (int t0 = 0; t0 < T; t0 += 4) { DMA2_STAGE(MF, XL, VM, 0) DMA2_STAGE(MF, XL, VM, 1) DMA2_STAGE(MF, XL, VM, 2) DMA2_STAGE(MF, XL, VM, 3) }

    // only live row tiles are fetched; the count of loads a wave may leave in flight is per wave
    // and follows from how many X tiles it sends
    const int xl = max(0, min(2, mbs - 2 * wave));
#pragma unroll
    for (int st = 0; st < 5; ++st)
#pragma unroll
        for (int j = 0; j < 6; ++j)
            if (j >= 4 || (j >> 1) < xl) issue(x_base(st), w_base(st), st, j);
    int bc = 0, bn = 1, bi = 5;
    if (xl == 2) { STAGE_END(18) } else if (xl == 1) { STAGE_END(12) } else { STAGE_END(6) }   // stages 0 and 1 have landed
    a1 = Half{};
    b1 = BHalf{};
    rd_a(a0, 0, 0, 0); rd_a(a0, 0, 0, 1); rd_a(a0, 0, 0, 2); rd_a(a0, 0, 0, 3);
    rd_b(b0, 0, 0);
    // a wave that does not send both of its X tiles has fewer than 4 live row tiles
    if (xl == 0) { DMA2_LOOP(mf_some, 0, 6) }
    else if (xl == 1) { DMA2_LOOP(mf_some, 1, 12) }
    else if (cnt == 4) { DMA2_LOOP(mf_all, 2, 18) }
    else { DMA2_LOOP(mf_some, 2, 18) }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#undef DMA2_LOOP
#undef DMA2_STAGE
#undef STAGE_END
#undef SB
#define EPI_ROW(E, ARGS, I) \
    if (4 * wm + (I) < mbs) epilogue_tile<E>(ARGS, acc[I][0], acc[I][1], row_base + 32 * (4 * wm + (I)), n, nbw, lane, sc[I]);
    if (splits > 1) {
        EpiArgs pe = ep;
        pe.out = partial + (int64_t)sp * part_plane;
        pe.ldo = part_ld;
        EPI_ROW(EPI_STORE, pe, 0) EPI_ROW(EPI_STORE, pe, 1) EPI_ROW(EPI_STORE, pe, 2) EPI_ROW(EPI_STORE, pe, 3)
        return;
    }
    EPI_ROW(EPI, ep, 0) EPI_ROW(EPI, ep, 1) EPI_ROW(EPI, ep, 2) EPI_ROW(EPI, ep, 3)
#undef EPI_ROW
}

// ------------------------------------------------------------------ full tiles of 256 and 192 columns: two waves per SIMD in turns
// 256 rows x 32 NT columns per workgroup, eight waves with NA x NB tiles of 16x16 each: as 2 x 4 with 8 x 4 (NT = 8), as 4 x 2
// with 4 x 6 (NT = 6); a wave's 32-row tiles are r0, r0 + STEP, .. so that both waves of a SIMD, w and w + 4, have live rows.
// LDS slots and loads as in the loops of k_bf16_gemm_dma8 and k_bf16_gemm_cols below, which take over where few row tiles are live.
//
// While waves 0 .. 3 multiply, waves 4 .. 7 read their operands of a stage from LDS and send their tiles of the stage four ahead;
// then they change places, at a barrier.  What limits full products is power, of which 16x16x32 MFMAs take less than 32x32x16
// (alone, on random data, 2.08 PFLOP/s against 1.79 to 1.85).  2048 rows of the 70B shape, one machine, loops below / here: gate/up 1454 us,
// matrix pipes busy 77 % of the time at 1.64 GHz / 1338, 76 % at 1.81; down with its K-slice finish 704 / 658; q|k|v, 192 columns, whose
// operands take LDS longer than the MFMAs last, 305 / 311.  Exit head of 1024 entries at the 7B shape 211 / 201, with logits 300..323 /
// 258..267 (the epilogue's 16-byte stores too).
#define SB __builtin_amdgcn_sched_barrier(0)
template <int NT>
struct TurnShape;
template <>
struct TurnShape<8> { static constexpr int NA = 8, NB = 4, STEP = 2; };
template <>
struct TurnShape<6> { static constexpr int NA = 4, NB = 6, STEP = 4; };

// Whether the workgroups of a row group take turns (below: the loops that follow / here).
// One group: with seven live row tiles or more (layer of the 70B shape 200 rows, gate/up 197 / 191 us, down 119 / 112; of the 34B
// shape, 192 columns, 200 rows 160 / 157).  With fewer, memory sets the pace and a wave's turn holds up its requests (gate/up of
// the 70B shape 128 rows 157 / 164..171, 160 174 / 195, of the 34B shape 128 127 / 143, 180 166 / 172).
// Several groups: the last one from five tiles on, as the groups of a column tile read the same weights and keep step only on one loop (layer
// of 400 rows, 144 of them in the second group, that group below / here: 7B shape 354 / 330 us, 34B 718 / 658, 70B 840 / 764; 1700
// rows 1074 / 1064, 2130 / 2076, 2622 / 2564).
// Slices of K: a turn more at the start and at the end of each, and where the groups do not keep step short ones lose more than that.
// All groups in turns, stages of a slice: down of the 2048-wide model 11 (512 rows) 35.5 / 37.7 us, 22 (1024) 49.3 / 50.0, of the 7B shape
// 21 (256 rows) 54.5 / 56.7, 43 (512) 66.0 / 64.5, of the 70B shape 112 (512) 211 / 202.  Planes for the append kernel, whose launches
// leave CUs idle, need longer ones if the last group has the seven tiles that the old loops are good at: q|k|v of the 7B shape 64 (512
// rows) 58.2 / 59.8, (480) 57.0 / 58.4, but (440: six tiles) 59.3 / 57.1, of the 70B shape 85 (512) 85.3 / 83.2.  A last group of fewer tiles: 7B shape
// 300 rows, q|k|v 64 54.5 / 57.5, down 43 59.5 / 61.8, 600 rows, down 68 79.0 / 80.3, on another machine 92 / 85, 34B 300 rows, q|k|v 84
// 80 / 82 and 90 / 86, 7B 1100 rows, down 114 115 / 111.
template <int EPI>
__device__ __forceinline__ bool takes_turns(int n, int row_base, int splits, int stages) {
    const int groups = (n + 255) >> 8, from = groups > 1 ? 5 : 7;
    const int live = (n - row_base + 31) >> 5, last = (n - 256 * (groups - 1) + 31) >> 5;      // row tiles from this group on, of the last one
    const bool longer = last < from || (EPI == EPI_STORE && last >= 7);
    return live >= from && (splits == 1 || stages >= (longer ? 65 : 40));
}

struct TurnCtx {
    uint4*       lds;        // [5][32][64]
    const uint4* xg;         // row tile 0, K tile 0 of the row group
    const uint4* wg;         // column tile 0 of the workgroup, K tile 0
    int KB, NBs, ks_lo, T;   // stages ks_lo .. ks_lo + T - 1
    int row_base, n, nb0, nt_live;
};

template <int EPI, int NT>
__device__ __forceinline__ void tile_in_turns(const TurnCtx& c, const EpiArgs& ep) {
    using S = TurnShape<NT>;
    constexpr int NA = S::NA, NB = S::NB;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int later = wave >> 2;
    const int r0 = NT == 8 ? later : 2 * ((wave >> 1) & 1) + later, c0 = NB / 2 * (NT == 8 ? wave & 3 : wave & 1);
    const int rows = c.n - c.row_base, mbs = min(8, (rows + 31) >> 5);
    int cnt = 0;                                             // live 16-row tiles among the wave's
#pragma unroll
    for (int i = 0; i < NA / 2; ++i) cnt += max(0, min(2, (rows - 32 * (r0 + S::STEP * i) + 15) >> 4));
    const unsigned lane_bytes = (unsigned)lane * 16u;
    const unsigned lds0 = (unsigned)(size_t)c.lds;
    const bool sends_x = wave < mbs, sends_w = wave < NT;
    float sc[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) sc[i] = exit_scale<EPI>(ep, c.row_base + 32 * (r0 + S::STEP * (i >> 1)) + 16 * (i & 1) + (lane & 15), c.n);

    floatx4 acc[NA][NB];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    // j-th load of a stage: j = 0, 1 the X tile of row tile `wave`, K half j; j = 2, 3 the W tile of
    // column tile `wave`, K half j - 2.  Address = the stage's base pointer (scalar, once per stage)
    // plus a lane offset that is the same in every stage.
    unsigned voff[4];
#pragma unroll
    for (int j = 0; j < 2; ++j) voff[j] = lane_bytes + ((unsigned)(min(wave, mbs - 1) * c.KB + j) << 10);
#pragma unroll
    for (int j = 2; j < 4; ++j) voff[j] = lane_bytes + ((unsigned)((j - 2) * c.NBs + min(wave, c.nt_live - 1)) << 10);
    auto x_base = [&](int t) { return c.xg + (int64_t)(2 * (c.ks_lo + min(t, c.T - 1))) * 64; };
    auto w_base = [&](int t) { return c.wg + (int64_t)(2 * (c.ks_lo + min(t, c.T - 1))) * c.NBs * 64; };
    // Operand of a 16x16x32 MFMA from the two tiles (K halves, 1 KiB each) of 32 rows: lane l has row l % 16 and K octet l / 16,
    // the tiles' lanes are 32 rows x 2 octets; rows 16 to 31 are 256 bytes further
    const char* lane_at = reinterpret_cast<const char*>(c.lds) + (lane >> 5) * 1024 + ((lane >> 4) & 1) * 512 + (lane & 15) * 16;
    auto next = [](int buf) { return buf == 4 ? 0 : buf + 1; };

    // what a wave sends is fixed, and with it the count of loads it may leave in flight: each combination runs its own copy
    auto loop = [&](auto xl_, auto wl_, auto all_) {
        constexpr bool XL = decltype(xl_)::value, WL = decltype(wl_)::value, ALL = decltype(all_)::value;
        constexpr int L = 2 * (XL ? 1 : 0) + 2 * (WL ? 1 : 0);
        auto issue = [&](int t, int buf) {
            const uint4 *xs = x_base(t), *ws = w_base(t);
            const unsigned at = lds0 + (unsigned)((buf * 32 + wave * 2) << 10);
            if constexpr (XL) { dma_tile(xs, voff[0], at); dma_tile(xs, voff[1], at + 1024); }
            if constexpr (WL) { dma_tile<true>(ws, voff[2], at + 16384); dma_tile<true>(ws, voff[3], at + 17408); }
        };
#pragma unroll
        for (int st = 0; st < 4; ++st) issue(st, st);
        uint4 a[NA], b[NB];
#pragma unroll
        for (int i = 0; i < NA; ++i) a[i] = make_uint4(0, 0, 0, 0);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(3 * L) : "memory");         // stage 0 has landed
        if (later) asm volatile("s_barrier" ::: "memory");
        int bc = 0, bi = 4;                                  // buffers of the current stage and of the one being requested
        for (int t = 0; t < c.T; ++t) {
            SB;
            const char* at = lane_at + bc * 32768;
#pragma unroll
            for (int j = 0; j < NB; ++j) b[j] = *reinterpret_cast<const uint4*>(at + 16384 + (c0 + (j >> 1)) * 2048 + (j & 1) * 256);
#pragma unroll
            for (int i = 0; i < NA; ++i)
                if (ALL || i < cnt) a[i] = *reinterpret_cast<const uint4*>(at + (r0 + S::STEP * (i >> 1)) * 2048 + (i & 1) * 256);
            issue(t + 4, bi);
            // The operands have been read (their buffer is filled again from the phase after the next on).  Between the two phases
            // of a stage every wave waits for its loads of the next stage, which is first read after this barrier or the one after.
            if (later) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(3 * L) : "memory");
            else asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            SB;
#pragma unroll
            for (int i = 0; i < NA; ++i)
                if (ALL || i < cnt) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) acc[i][j] = mfma16(a[i], b[j], acc[i][j]);
                }
            SB;
            if (later) asm volatile("s_barrier" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(3 * L) : "memory");
            bc = next(bc); bi = next(bi);
        }
        if (!later) asm volatile("s_barrier" ::: "memory");  // as many barriers as the others
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    using Yes = std::true_type;
    using No = std::false_type;
    const bool all = cnt == NA;                              // only waves that send X have all their rows live
    if (NT == 8 || sends_w) { if (!sends_x) loop(No{}, Yes{}, No{}); else if (all) loop(Yes{}, Yes{}, Yes{}); else loop(Yes{}, Yes{}, No{}); }
    else { if (!sends_x) loop(No{}, No{}, No{}); else if (all) loop(Yes{}, No{}, Yes{}); else loop(Yes{}, No{}, No{}); }

#pragma unroll
    for (int i = 0; i < NA / 2; ++i) {
        if (2 * i >= cnt) break;
        floatx4 v[2][NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) { v[0][j] = acc[2 * i][j]; v[1][j] = acc[2 * i + 1][j]; }
        epilogue_blocks<EPI, NB / 2>(ep, v, c.row_base + 32 * (r0 + S::STEP * i), c.n, c.nb0 + c0, c.nt_live - c0, lane, sc + 2 * i);
    }
}

#undef SB

// ------------------------------------------------------------------ 256-column tile, two waves per SIMD
// 256 rows x 256 columns per workgroup, eight waves (2 x 4): wave (wm, wn) owns rows
// 128 wm .. +127 and columns 64 wn .. +63 (4 x 2 MFMA tiles, 128 accumulator registers), so two waves
// share a SIMD and one computes while the other waits at a barrier or for LDS (an MFMA-only
// kernel issues 10 % more per SIMD with two waves than with one).  Used for the
// products with many columns (gate/up with the SwiGLU epilogue, down, the K/V of skipped layers).  LDS: 5 stage buffers x 32 slots
// (X tile (row tile m, K half kk) at 2 m + kk, W tile (column tile nb of 8, K half kk) at
// 16 + 2 nb + kk) = all 160 KiB.  A wave sends 2 X and 2 W tiles per stage, four stages ahead, and
// may leave two stages in flight at the barrier: a load has two to three stages to land.
template <int EPI>
__global__ void __launch_bounds__(512, 2)
k_bf16_gemm_dma8(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp, int KB, int NBs, int nb_off,
                 int n_tiles, int splits, const int32_t* __restrict__ n_ptr, int B, float* __restrict__ partial,
                 int64_t part_plane, int part_ld, EpiArgs ep, ZBatch zb) {
    __shared__ uint4 lds[5][32][64];
    const int n = min(*n_ptr, B);
    int rg, unit;
    tile_of_block(n_tiles * splits, rg, unit);
    if (unit < 0) return;
    const int row_base = rg * 256;
    if (row_base >= n) return;
    if (zb.w_tab) Wp = reinterpret_cast<const uint4*>(zb.w_tab[zb.z0 + blockIdx.z]);
    Xp += (int64_t)blockIdx.z * zb.x_stride;
    ep.out += (int64_t)blockIdx.z * zb.out_stride;
    const int mbs = min(8, (n - row_base + 31) >> 5);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int cnt = max(0, min(4, mbs - 4 * wm));            // live 32-row tiles of this wave
    const int tile = unit / splits, sp = unit % splits;
    const int nbw = (tile * 4 + wn) * 2;                     // first of this wave's two tile-rows of W
    const int KS4 = KB >> 3;
    const int ks_lo = 4 * (int)(((int64_t)KS4 * sp) / splits), ks_hi = 4 * (int)(((int64_t)KS4 * (sp + 1)) / splits);
    const int T = ks_hi - ks_lo;                             // stages of this slice: a positive multiple of 4
    const uint4* xg = Xp + ((int64_t)rg * 8 * KB) * 64;
    const uint4* wg = Wp + (int64_t)(nb_off + tile * 8) * 64;   // the tile's eight tile-rows of W
    if (splits > 1) {
        ep.out = partial + (int64_t)sp * part_plane;
        ep.ldo = part_ld;
    }
    if (takes_turns<EPI>(n, row_base, splits, T)) {
        const TurnCtx c{&lds[0][0][0], xg, wg, KB, NBs, ks_lo, T, row_base, n, tile * 8, 8};
        if (splits > 1) tile_in_turns<EPI == EPI_RESID ? EPI_STORE : EPI, 8>(c, ep);     // others than these two are never sliced
        else tile_in_turns<EPI, 8>(c, ep);
        return;
    }
    const unsigned lane_bytes = (unsigned)lane * 16u;
    const unsigned lds0 = (unsigned)(size_t)&lds[0][0][0];

    float sc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) sc[i] = exit_scale<EPI>(ep, row_base + 32 * (4 * wm + i) + (lane & 31), n);

    floatx16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // j-th load of a stage: j = 0, 1 the X tile of row tile `wave`, K half j (sent only if that row
    // tile is live); j = 2, 3 the W tile of column tile `wave`, K half j - 2.  Address = the stage's base pointer (scalar, once per stage) plus a lane
    // offset that is the same in every stage.
    unsigned voff[4];
#pragma unroll
    for (int j = 0; j < 2; ++j) voff[j] = lane_bytes + ((unsigned)(min(wave, mbs - 1) * KB + j) << 10);
#pragma unroll
    for (int j = 2; j < 4; ++j) voff[j] = lane_bytes + ((unsigned)((j - 2) * NBs + wave) << 10);
    auto x_base = [&](int t) { return xg + (int64_t)(2 * (ks_lo + min(t, T - 1))) * 64; };
    auto w_base = [&](int t) { return wg + (int64_t)(2 * (ks_lo + min(t, T - 1))) * NBs * 64; };
    auto issue = [&](const uint4* xs, const uint4* ws, int buf, int j) {
        if (j < 2) dma_tile(xs, voff[j], lds0 + (unsigned)((buf * 32 + wave * 2 + j) << 10));
        else dma_tile<true>(ws, voff[j], lds0 + (unsigned)((buf * 32 + 16 + wave * 2 + (j - 2)) << 10));
    };
    Half a0, a1;
    BHalf b0, b1;
    auto rd_a = [&](Half& o, int buf, int kk, int i) { o.v[i] = (&lds[0][0][lane] + buf * (32 * 64))[((4 * wm + i) * 2 + kk) * 64]; };
    auto rd_b = [&](BHalf& o, int buf, int kk) {
        const uint4* p = &lds[0][0][lane] + buf * (32 * 64);
        o.v[0] = p[(16 + (2 * wn) * 2 + kk) * 64];
        o.v[1] = p[(16 + (2 * wn + 1) * 2 + kk) * 64];
    };
    auto mf_all = [&](const Half& a, const BHalf& bw, int i) {
        acc[i][0] = tile_mfma<EPI>(a.v[i], bw.v[0], acc[i][0]);
        acc[i][1] = tile_mfma<EPI>(a.v[i], bw.v[1], acc[i][1]);
    };
    auto mf_some = [&](const Half& a, const BHalf& bw, int i) {
        if (i < cnt) mf_all(a, bw, i);
    };
#define SB __builtin_amdgcn_sched_barrier(0);
// two stages of this wave's loads (VM of them) may stay in flight: everything up to stage t+2 has landed
#define STAGE_END(VM) asm volatile("s_waitcnt vmcnt(" #VM ") lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // bc / bn / bi: buffers of the current stage, the next one and the one being requested (stage + 4)
#define DMA8_STAGE(MF, XL, VM, U)                                                             \
    { const uint4* xs_ = x_base(t0 + (U) + 4); const uint4* ws_ = w_base(t0 + (U) + 4);       \
    MF(a0, b0, 0); SB if (XL) issue(xs_, ws_, bi, 0); rd_a(a1, bc, 1, 0); rd_a(a1, bc, 1, 1); rd_b(b1, bc, 1); SB \
    MF(a0, b0, 1); SB if (XL) issue(xs_, ws_, bi, 1); rd_a(a1, bc, 1, 2); rd_a(a1, bc, 1, 3); SB \
    MF(a0, b0, 2); SB                                                                         \
    MF(a0, b0, 3); SB                                                                         \
    MF(a1, b1, 0); SB issue(xs_, ws_, bi, 2); rd_a(a0, bn, 0, 0); rd_a(a0, bn, 0, 1); rd_b(b0, bn, 0); SB \
    MF(a1, b1, 1); SB issue(xs_, ws_, bi, 3); rd_a(a0, bn, 0, 2); rd_a(a0, bn, 0, 3); SB      \
    MF(a1, b1, 2); SB                                                                         \
    MF(a1, b1, 3); SB                                                                         \
    STAGE_END(VM) }                                                                           \
    bc = bn; bn = bn == 4 ? 0 : bn + 1; bi = bi == 4 ? 0 : bi + 1;
#define DMA8_LOOP(MF, XL, VM) \
    for (int t0 = 0; t0 < T; t0 += 4) { DMA8_STAGE(MF, XL, VM, 0) DMA8_STAGE(MF, XL, VM, 1) DMA8_STAGE(MF, XL, VM, 2) DMA8_STAGE(MF, XL, VM, 3) }

    // only live row tiles are fetched: wave w sends the X tiles of row tile w if there is one, and
    // the count of loads it may leave in flight follows (the counter is per wave)
    const bool sends_x = wave < mbs;
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j >= 2 || sends_x) issue(x_base(st), w_base(st), st, j);
    int bc = 0, bn = 1, bi = 4;
    if (sends_x) { STAGE_END(8) } else { STAGE_END(4) }   // stages 0 and 1 have landed
    a1 = Half{};
    b1 = BHalf{};
    rd_a(a0, 0, 0, 0); rd_a(a0, 0, 0, 1); rd_a(a0, 0, 0, 2); rd_a(a0, 0, 0, 3);
    rd_b(b0, 0, 0);
    if (!sends_x) { DMA8_LOOP(mf_some, false, 4) }         // such a wave has fewer than 4 live tiles
    else if (cnt == 4) { DMA8_LOOP(mf_all, true, 8) }
    else { DMA8_LOOP(mf_some, true, 8) }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#undef DMA8_LOOP
#undef DMA8_STAGE
#undef STAGE_END
#undef SB
#define EPI_ROW(E, ARGS, I) \
    if (4 * wm + (I) < mbs) epilogue_tile<E>(ARGS, acc[I][0], acc[I][1], row_base + 32 * (4 * wm + (I)), n, nbw, lane, sc[I]);
    if (splits > 1) {
        EPI_ROW(EPI_STORE, ep, 0) EPI_ROW(EPI_STORE, ep, 1) EPI_ROW(EPI_STORE, ep, 2) EPI_ROW(EPI_STORE, ep, 3)
        return;
    }
    EPI_ROW(EPI, ep, 0) EPI_ROW(EPI, ep, 1) EPI_ROW(EPI, ep, 2) EPI_ROW(EPI, ep, 3)
#undef EPI_ROW
}

// ------------------------------------------------------------------ tile of 192 columns
// 256 rows x 192 columns per workgroup, for products whose column tiles fill the 256 CUs badly at 128 or 256 columns
// (gate/up of the 34B shape has 1376 tile-rows: 344 workgroups of 4 take two rounds, 172 of 8 leave a third of the
// CUs idle, 230 of 6 run in one round; with several row groups gate/up of 1024 entries at the 7B shape is 344
// workgroups of 8, two rounds of 90 us, and 460 of 6, two rounds of 76).  Same operand path, staging and waits as
// k_bf16_gemm_dma8; eight waves as 4 x 2, wave (wm, wn) owns row tiles 2 wm, 2 wm + 1 and column tiles 3 wn .. 3 wn + 2: six
// MFMA tiles each, two waves per SIMD.  (Before, the six column tiles were dealt out 2, 2, 1, 1 over the SIMDs, which at full rows
// ran at the pace of the fuller ones: 256 rows 175 -> 169 us, and no faster than 256 columns with several row groups.)
// LDS: 5 stage buffers of 32 slots, X tile (row tile m, K half kk) at 2 m + kk, W tile (column tile nb, K half
// kk) at 16 + 2 nb + kk; wave w sends the X tiles of row tile w (if live) and the W tiles of column
// tile w (if w < 6), four stages ahead.  The last workgroup of a product whose tile-rows are no
// multiple of 6 re-reads its last tile-row in place of the missing ones and drops their results.
#define COLS_NT 6       /* column tiles of a workgroup */
#define COLS_NR 2       /* row tiles of a wave */
#define COLS_NC 3       /* column tiles of a wave */
struct ColsCtx {
    uint4*       lds;        // [5][32][64]
    const uint4* xg;
    const uint4* wg;
    int KB, NBs, ks_lo, T, mbs, nt_live, wave, lane, row_base, n, nb0;
};

template <int EPI>
__device__ __forceinline__ void cols_wave(const ColsCtx& c, const int r0, const int c0, const EpiArgs& ep) {
    const int wave = c.wave, lane = c.lane;
    const int cnt = max(0, min(COLS_NR, c.mbs - r0));              // live row tiles among the wave's
    const unsigned lane_bytes = (unsigned)lane * 16u;
    const unsigned lds0 = (unsigned)(size_t)c.lds;
    const bool sends_x = wave < c.mbs, sends_w = wave < COLS_NT;
    float sc[COLS_NR];
#pragma unroll
    for (int i = 0; i < COLS_NR; ++i) sc[i] = exit_scale<EPI>(ep, c.row_base + 32 * (r0 + i) + (lane & 31), c.n);

    floatx16 acc[COLS_NR][COLS_NC];
#pragma unroll
    for (int i = 0; i < COLS_NR; ++i)
#pragma unroll
        for (int j = 0; j < COLS_NC; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // j-th load of a stage: j = 0, 1 the X tile of row tile `wave`, K half j; j = 2, 3 the W tile of
    // column tile `wave`, K half j - 2.  Address = the stage's base pointer (scalar, once per stage)
    // plus a lane offset that is the same in every stage.
    unsigned voff[4];
#pragma unroll
    for (int j = 0; j < 2; ++j) voff[j] = lane_bytes + ((unsigned)(min(wave, c.mbs - 1) * c.KB + j) << 10);
#pragma unroll
    for (int j = 2; j < 4; ++j) voff[j] = lane_bytes + ((unsigned)((j - 2) * c.NBs + min(wave, c.nt_live - 1)) << 10);
    auto x_base = [&](int t) { return c.xg + (int64_t)(2 * (c.ks_lo + min(t, c.T - 1))) * 64; };
    auto w_base = [&](int t) { return c.wg + (int64_t)(2 * (c.ks_lo + min(t, c.T - 1))) * c.NBs * 64; };
    auto issue = [&](const uint4* xs, const uint4* ws, int buf, int j) {
        if (j < 2) dma_tile(xs, voff[j], lds0 + (unsigned)((buf * 32 + wave * 2 + j) << 10));
        else dma_tile<true>(ws, voff[j], lds0 + (unsigned)((buf * 32 + 16 + wave * 2 + (j - 2)) << 10));
    };
    uint4 a[2][COLS_NR], b[2][COLS_NC];                                 // [K half][row tile], [K half][column tile]
    auto slot = [&](int buf, int s_) { return (c.lds + lane + buf * (32 * 64))[s_ * 64]; };
    auto rd_a = [&](int buf, int kk, int i) { a[kk][i] = slot(buf, (r0 + i) * 2 + kk); };
    auto rd_b = [&](int buf, int kk, int j) { b[kk][j] = slot(buf, 16 + (c0 + j) * 2 + kk); };

    int bc = 0, bn = 1, bi = 4;   // buffers of the current stage, the next one and the one being requested (stage + 4)
    // One stage: the MFMAs of K half 0 while K half 1 is read from LDS and the X tiles of stage + 4 are
    // requested, then those of K half 1 while K half 0 of the next stage is read and the W tiles are
    // requested; the loads are issued one behind an MFMA group each.  Two stages of this wave's loads
    // may stay in flight at the barrier: everything up to stage + 2 has landed.
    auto stage = [&](auto xl_, auto wl_, auto all_, int t_req) {
        constexpr bool XL = decltype(xl_)::value, WL = decltype(wl_)::value, ALL = decltype(all_)::value;
        const uint4* xs = x_base(t_req);
        const uint4* ws = w_base(t_req);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int rb = kk == 0 ? bc : bn;                 // buffer the other K half is read from
            const int ok = 1 - kk;
#pragma unroll
            for (int g = 0; g < COLS_NR; ++g) {
                if (ALL || g < cnt) {
#pragma unroll
                    for (int j = 0; j < COLS_NC; ++j) acc[g][j] = tile_mfma<EPI>(a[kk][g], b[kk][j], acc[g][j]);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (g == 0) {
                    if (kk == 0 ? XL : WL) issue(xs, ws, bi, 2 * kk);
                    rd_a(rb, ok, 0); rd_b(rb, ok, 0); rd_b(rb, ok, 1);
                } else {
                    if (kk == 0 ? XL : WL) issue(xs, ws, bi, 2 * kk + 1);
                    rd_a(rb, ok, 1); rd_b(rb, ok, 2);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * (2 * (XL ? 1 : 0) + 2 * (WL ? 1 : 0))) : "memory");
        bc = bn; bn = bn == 4 ? 0 : bn + 1; bi = bi == 4 ? 0 : bi + 1;
    };
    auto slice = [&](auto xl_, auto wl_, auto all_) {
        constexpr bool XL = decltype(xl_)::value, WL = decltype(wl_)::value;
#pragma unroll
        for (int st = 0; st < 4; ++st)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j < 2 ? XL : WL) issue(x_base(st), w_base(st), st, j);
        // stages 0 and 1 have landed
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * (2 * (XL ? 1 : 0) + 2 * (WL ? 1 : 0))) : "memory");
#pragma unroll
        for (int i = 0; i < COLS_NR; ++i) { rd_a(0, 0, i); a[1][i] = a[0][i]; }
#pragma unroll
        for (int j = 0; j < COLS_NC; ++j) { rd_b(0, 0, j); b[1][j] = b[0][j]; }
        for (int t0 = 0; t0 < c.T; t0 += 4) {
            stage(xl_, wl_, all_, t0 + 4); stage(xl_, wl_, all_, t0 + 5); stage(xl_, wl_, all_, t0 + 6); stage(xl_, wl_, all_, t0 + 7);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    using Yes = std::true_type;
    using No = std::false_type;
    // the count of loads a wave may leave in flight is per wave and follows from what it sends, so each
    // combination runs its own copy of the loop; a wave whose two row tiles are live (the common case)
    // runs a copy without the live-tile test
    // (at most six row tiles are live here, so that a wave that sends X sends W too)
    const bool all = cnt == COLS_NR;
    if (sends_x)      { if (all) slice(Yes{}, Yes{}, Yes{}); else slice(Yes{}, Yes{}, No{}); }
    else if (sends_w) { slice(No{}, Yes{}, No{}); }
    else              { slice(No{}, No{}, No{}); }

#pragma unroll
    for (int i = 0; i < COLS_NR; ++i) {
        if (i >= cnt) continue;
#pragma unroll
        for (int j = 0; j < COLS_NC; ++j)
            if (c0 + j < c.nt_live)
                epilogue_one<EPI>(ep, acc[i][j], c.row_base + 32 * (r0 + i), c.n, c.nb0 + c0 + j, lane, sc[i]);
    }
}

template <int EPI>
__global__ void __launch_bounds__(512, 2)
k_bf16_gemm_cols(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp, int KB, int NBs, int nb_off, int NB_total,
                 int n_tiles, const int32_t* __restrict__ n_ptr, int B, EpiArgs ep, ZBatch zb) {
    __shared__ uint4 lds[5][32][64];
    const int n = min(*n_ptr, B);
    int rg, tile;
    tile_of_block(n_tiles, rg, tile);
    if (tile < 0) return;
    const int row_base = rg * 256;
    if (row_base >= n) return;
    if (zb.w_tab) Wp = reinterpret_cast<const uint4*>(zb.w_tab[zb.z0 + blockIdx.z]);
    Xp += (int64_t)blockIdx.z * zb.x_stride;
    ep.out += (int64_t)blockIdx.z * zb.out_stride;
    if (takes_turns<EPI>(n, row_base, 1, KB >> 1)) {
        const TurnCtx t{&lds[0][0][0], Xp + ((int64_t)rg * 8 * KB) * 64, Wp + (int64_t)(nb_off + tile * COLS_NT) * 64, KB, NBs, 0, KB >> 1,
                        row_base, n, tile * COLS_NT, min(COLS_NT, NB_total - tile * COLS_NT)};
        tile_in_turns<EPI, COLS_NT>(t, ep);
        return;
    }
    ColsCtx c;
    c.lds = &lds[0][0][0];
    c.KB = KB; c.NBs = NBs;
    c.ks_lo = 0;
    c.T = KB >> 1;                                            // stages: a positive multiple of 4 (K is a multiple of 128)
    c.mbs = (n - row_base + 31) >> 5;                        // at most six (takes_turns)
    c.nt_live = min(COLS_NT, NB_total - tile * COLS_NT);
    c.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    c.lane = threadIdx.x & 63;
    c.row_base = row_base; c.n = n; c.nb0 = tile * COLS_NT;
    c.xg = Xp + ((int64_t)rg * 8 * KB) * 64;
    c.wg = Wp + (int64_t)(nb_off + tile * COLS_NT) * 64;            // the tile's COLS_NT tile-rows of W
    cols_wave<EPI>(c, COLS_NR * (c.wave >> 1), COLS_NC * (c.wave & 1), ep);
}

// ------------------------------------------------------------------ few rows: each wave streams on its own
// Products of at most 128 rows are a stream of weights, and what the tile kernels above lose there is depth: their
// stages are shared by the waves of a workgroup, so each ends in a barrier, and with room for 256 rows in a stage
// three of them (30 KiB at 32 rows) are on their way at a time, while a CU can keep more.  Here nothing is shared:
// wave w of a workgroup takes the K tiles 4 i + w of the workgroup's K slice (so that all waves of a launch walk K
// together), with the NS tile-rows of W and the MS row tiles of X of each in a ring of its own, filled by LDS-DMA
// loads up to D tiles ahead and waited for by the wave's own load counter; the four partial sums are added in wave
// order through LDS at the end.  Up to 64 rows two workgroups fit on a CU.  Of an X tile only the 8-row pieces (whole
// lines) that hold live rows are fetched; the rest of its slot keeps what was there, and reaches only results that
// are not written.  K is a multiple of 64, the last workgroup of a slice re-reads its last tile-row in place of
// missing ones.  More rows than 32 MS are taken in row groups (tile_of_block).
constexpr int few_depth(int MS, int NS) { return (MS > 2 ? 40 : 20) / (MS + NS); }     // KiB of a wave's ring

template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// the wait before a wave's last tiles: `left` more of L loads each may be under way (left < D)
template <int L, int D>
__device__ __forceinline__ void wait_tail(int left) {
    if constexpr (D > 1) {
        if (left >= D - 1) { wait_loads<(D - 1) * L>(); return; }
        wait_tail<L, D - 1>(left);
    } else {
        wait_loads<0>();
    }
}

template <int MS, int NS, int EPI>
__global__ void __launch_bounds__(256, MS > 2 ? 1 : 2)
k_bf16_gemm_few(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp, int KB, int NBs, int nb_off, int NB_total, int splits,
                const int32_t* __restrict__ n_ptr, int B, float* __restrict__ partial, int64_t part_plane, int part_ld, EpiArgs ep,
                ZBatch zb) {
    constexpr int T = NS + MS, D = few_depth(MS, NS);
    __shared__ uint4 lds[4 * D * T * 64];
    static_assert(4 * D * T >= 16 * NS, "the partial sums of a row tile share the rings");
    int rg, unit;
    tile_of_block((NB_total + NS - 1) / NS * splits, rg, unit);
    const int row_base = rg * (32 * MS), n = min(*n_ptr, B) - row_base;      // rows of this row group and after it
    if (unit < 0 || n <= 0) return;
    if (zb.w_tab) Wp = reinterpret_cast<const uint4*>(zb.w_tab[zb.z0 + blockIdx.z]);
    Xp += (int64_t)blockIdx.z * zb.x_stride + (int64_t)rg * MS * KB * 64;
    ep.out += (int64_t)blockIdx.z * zb.out_stride;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = unit / splits, sp = unit % splits;
    const int nb0 = tile * NS, nt_live = min(NS, NB_total - nb0);
    const int quads = KB >> 2;                               // a step of the workgroup: one K tile per wave
    const int q_lo = (int)((int64_t)quads * sp / splits), S = (int)((int64_t)quads * (sp + 1) / splits) - q_lo;
    const unsigned lane_bytes = (unsigned)lane * 16u, ring = (unsigned)(size_t)&lds[wave * D * T * 64];
    float sc[MS];
#pragma unroll
    for (int m = 0; m < MS; ++m) sc[m] = exit_scale<EPI>(ep, row_base + 32 * m + (lane & 31), row_base + n);
    const uint4* wp = Wp + ((int64_t)(4 * q_lo + wave) * NBs + nb_off + nb0) * 64;   // tile (r, c) of W sits at slot c * NBs + r
    const uint4* xp = Xp + (int64_t)(4 * q_lo + wave) * 64;
    unsigned wv[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) wv[j] = lane_bytes + ((unsigned)min(j, nt_live - 1) << 10);

    floatx16 acc[MS][NS];
#pragma unroll
    for (int m = 0; m < MS; ++m)
#pragma unroll
        for (int j = 0; j < NS; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][j][r] = 0.f;

    auto stream = [&](auto live_) {                          // live_: row tiles that hold rows
        constexpr int ML = decltype(live_)::value, L = NS + ML;
        auto issue = [&](int slot) {
            const unsigned at = ring + (unsigned)(slot * T << 10);
#pragma unroll
            for (int j = 0; j < NS; ++j) dma_tile<true>(wp, wv[j], at + (unsigned)(j << 10));
#pragma unroll
            for (int m = 0; m < ML; ++m)
                if ((lane & 31) < ((n - 32 * m + 7) & ~7))   // lanes of the first eight rows always: the load is counted
                    dma_tile(xp, lane_bytes + ((unsigned)(m * KB) << 10), at + (unsigned)((NS + m) << 10));
            wp += (int64_t)4 * NBs * 64;
            xp += 4 * 64;
        };
        for (int i = 0; i < min(D, S); ++i) issue(i);
        int slot = 0;
        for (int s = 0; s < S; ++s) {
            if (s + D <= S) wait_loads<(D - 1) * L>();
            else wait_tail<L, D>(S - 1 - s);
            const uint4* t = &lds[(wave * D + slot) * T * 64 + lane];
            uint4 w[NS], x[ML];
#pragma unroll
            for (int j = 0; j < NS; ++j) w[j] = t[j * 64];
#pragma unroll
            for (int m = 0; m < ML; ++m) x[m] = t[(NS + m) * 64];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before the slot is filled again
            if (s + D < S) issue(slot);
#pragma unroll
            for (int m = 0; m < ML; ++m)
#pragma unroll
                for (int j = 0; j < NS; ++j) acc[m][j] = tile_mfma<EPI>(x[m], w[j], acc[m][j]);
            slot = slot + 1 == D ? 0 : slot + 1;
        }
    };
    if (MS == 1 || n > 32 * (MS - 1)) stream(std::integral_constant<int, MS>{});
    else if (MS > 2 && n > 32 * (MS - 2)) stream(std::integral_constant<int, (MS > 2 ? MS - 1 : 1)>{});
    else if (MS > 3 && n > 32) stream(std::integral_constant<int, (MS > 3 ? 2 : 1)>{});
    else stream(std::integral_constant<int, 1>{});
    float4* red = reinterpret_cast<float4*>(lds);            // [wave][tile-row][4 registers][lane]
#pragma unroll
    for (int m = 0; m < MS; ++m) {
        if (32 * m >= n) break;
        __syncthreads();                                     // the rings, or the row tile before, have been read
#pragma unroll
        for (int j = 0; j < NS; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                red[((wave * NS + j) * 4 + q) * 64 + lane] = make_float4(acc[m][j][4 * q], acc[m][j][4 * q + 1], acc[m][j][4 * q + 2], acc[m][j][4 * q + 3]);
        __syncthreads();
        if (wave < nt_live) {                                // tile-row `wave`
            floatx16 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float4 t = red[(wave * 4 + q) * 64 + lane];
#pragma unroll
                for (int k = 1; k < 4; ++k) {
                    const float4 u = red[((k * NS + wave) * 4 + q) * 64 + lane];
                    t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
                }
                v[4 * q] = t.x; v[4 * q + 1] = t.y; v[4 * q + 2] = t.z; v[4 * q + 3] = t.w;
            }
            if (splits > 1) {
                EpiArgs pe = ep;
                pe.out = partial + (int64_t)sp * part_plane;
                pe.ldo = part_ld;
                epilogue_one<EPI_STORE>(pe, v, row_base + 32 * m, row_base + n, nb0 + wave, lane);
            } else {
                epilogue_one<EPI>(ep, v, row_base + 32 * m, row_base + n, nb0 + wave, lane, sc[m]);
            }
        }
    }
}

// ------------------------------------------------------------------ RoPE + cache append
// buf[i] = [q (n_q heads, may be 0) | k (Hkv heads) | v (Hkv heads)], fp32, hd = 128.
// Queries are rotated and written as a bf16 pair (hi, lo) with hi + lo = q to 16
// mantissa bits, so that the attention kernel can feed them to the bf16 matrix
// cores without giving up fp32-grade scores.  Keys are rotated, rounded and
// appended; values are rounded and appended in the grouped layout.
// alone: no other entry's position shares a line of the cache with this one's (rows of a decode step).  An append then touches 32
// lines of a row and kv head for 16 bytes of a key's and 2 of a value's each, half a million lines for 512 rows of the 7B shape.
// As ordinary stores they stay in L2 until the attention's stream drives them out, one by one between its reads; non-temporal
// ones leave at once.  512 rows of the 7B shape, append 32 -> 36 us, attention 807 -> 765..790, machine to machine (its loads alone
// 776 before; without any append 703), 64 rows 117 -> 112..115, 256 rows of the 70B shape 233 -> 230.  In a context pass neighbours complete each other's lines in L2:
// append of 1024 entries 25 us, 55 non-temporal.
__device__ __forceinline__ void append8(bf16_t* at, uint2 v, bool alone) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    if (alone) __builtin_nontemporal_store((u32x2{v.x, v.y}), reinterpret_cast<u32x2*>(at));
    else *reinterpret_cast<uint2*>(at) = v;
}
__device__ __forceinline__ void append2(bf16_t* at, bf16_t v, bool alone) {
    if (alone) __builtin_nontemporal_store(v, at);
    else *at = v;
}

__global__ void __launch_bounds__(256)
k_bf16_rope_append(const float* __restrict__ buf, int ld, int n_q, const int32_t* __restrict__ idx,
                   const int32_t* __restrict__ n_ptr, int B, int near, const int32_t* __restrict__ pos,
                   const float* __restrict__ rope, int max_pos, KvView kv, bf16_t* __restrict__ q_hi,
                   bf16_t* __restrict__ q_lo, int32_t* __restrict__ status, int64_t z_stride,
                   int32_t* __restrict__ order, AttnJob* __restrict__ jobs, int most_shares, int tile_entries, bool alone, int splits, int64_t plane,
                   const float* __restrict__ planes, int ld_planes, int from) {
    int i = entry_of_block(blockIdx.x, near);
    int n = min(*n_ptr, B);
    if (i >= n) return;
    buf += (int64_t)blockIdx.z * z_stride;     // several layers in one launch: blockIdx.z = layer offset
    kv.layer0 += blockIdx.z;
    int b = idx[i];
    int p = pos[b];
    const int sq = kv_row(kv, b);
    const int cap = kv.cap[sq];
    if ((order != nullptr || jobs != nullptr) && blockIdx.y == 0 && threadIdx.x < 64 && i % tile_entries == 0) {
        // launch order of the attention workgroups: tiles of tile_entries list entries (one in a decode
        // step) by falling context length (that of a tile's last entry, as a context comes in rising
        // order; ties by tile), so that the longest start first and the last round of workgroups is short.
        // Rank of this tile = how many tiles come before it; the ranks form a permutation.
        auto key = [&](int tile) { return pos[idx[min(n, (tile + 1) * tile_entries) - 1]]; };
        const int tile = i / tile_entries, tiles = (n + tile_entries - 1) / tile_entries;
        const int mine = key(tile);
        int before = 0;
        for (int j = threadIdx.x; j < tiles; j += 64) {
            const int kj = key(j);
            before += (kj > mine || (kj == mine && j < tile)) ? 1 : 0;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
        if (threadIdx.x == 0) {
            if (jobs != nullptr) {
                const int n_pos = max(1, min(p + 1, cap));
                jobs[before] = AttnJob{tile, n_pos, cap, attn_shares(n * kv.n_kv_heads, n_pos, most_shares), kv.off[sq], p, 0};
            } else {
                order[before] = tile;
            }
        }
    }
    const int hd = 128, half = 64;
    int Hkv = kv.n_kv_heads;
    if (p < 0 || p >= cap || p >= max_pos) {
        if (threadIdx.x == 0) atomicOr(status, 1);
        return;
    }
    // columns before `from` are finished in buf; those from there on are `splits` K-slice planes of the product
    // (plane floats apart, ld_planes wide): their sum in slice order is the value
    const float* r0 = buf + (int64_t)i * ld;
    const float* rp = planes + (int64_t)i * ld_planes - from;
    // four consecutive values at once (x is a multiple of 4, from of 128: 16-byte loads from every plane)
    auto rd4 = [&](int x) -> float4 {
        if (x < from) return *reinterpret_cast<const float4*>(r0 + x);
        float4 v = *reinterpret_cast<const float4*>(rp + x);
        for (int q = 1; q < splits; ++q) {
            const float4 u = *reinterpret_cast<const float4*>(rp + x + (int64_t)q * plane);
            v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
        }
        return v;
    };
    auto pack4 = [](float a, float b, float c, float d) -> uint2 { return make_uint2(pack2(a, b), pack2(c, d)); };
    const float* cs = rope + (int64_t)p * half * 2;
    // The work of a row, in items of four rotation pairs (q, k) or four values (v), is dealt out over
    // the threads of the gridDim.y blocks that share the row: items [0, nq4) rotate queries, the next
    // nk4 rotate and append keys, the last nv4 append values.
    // A thread of the value items takes the values f, f + 64, f + 128, f + 192 of a block of 256, so that a wave's
    // 2-byte stores (16 bytes apart in the cache) touch 8 lines per store instead of 32.
    const int nq4 = n_q * (half / 4), nk4 = Hkv * (half / 4), nv4 = (Hkv * hd + 255) / 256 * 64;
    const int kin = n_q * hd;
    const int vin = kin + Hkv * hd;
    for (int t = blockIdx.y * 256 + threadIdx.x; t < nq4 + nk4 + nv4; t += 256 * gridDim.y) {
        if (t < nq4 + nk4) {
            const bool is_q = t < nq4;
            const int u = is_q ? t : t - nq4;
            const int hh = u >> 4, j0 = (u & 15) * 4;                 // head, first of the four pairs
            const int x = (is_q ? 0 : kin) + hh * hd + j0;
            const float4 a = rd4(x), bb = rd4(x + half);
            const float4 cs0 = *reinterpret_cast<const float4*>(cs + 2 * j0);       // c0 s0 c1 s1
            const float4 cs1 = *reinterpret_cast<const float4*>(cs + 2 * j0 + 4);   // c2 s2 c3 s3
            const float x0[4] = {a.x * cs0.x - bb.x * cs0.y, a.y * cs0.z - bb.y * cs0.w,
                                 a.z * cs1.x - bb.z * cs1.y, a.w * cs1.z - bb.w * cs1.w};
            const float x1[4] = {bb.x * cs0.x + a.x * cs0.y, bb.y * cs0.z + a.y * cs0.w,
                                 bb.z * cs1.x + a.z * cs1.y, bb.w * cs1.z + a.w * cs1.w};
            if (is_q) {
                const int64_t o = ((int64_t)i * n_q + hh) * hd + j0;
                const uint2 h0 = pack4(x0[0], x0[1], x0[2], x0[3]), h1 = pack4(x1[0], x1[1], x1[2], x1[3]);
                *reinterpret_cast<uint2*>(q_hi + o) = h0;
                *reinterpret_cast<uint2*>(q_hi + o + half) = h1;
                float l0[4], l1[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    l0[k] = x0[k] - bf16_to_f32(f32_to_bf16(x0[k]));
                    l1[k] = x1[k] - bf16_to_f32(f32_to_bf16(x1[k]));
                }
                *reinterpret_cast<uint2*>(q_lo + o) = pack4(l0[0], l0[1], l0[2], l0[3]);
                *reinterpret_cast<uint2*>(q_lo + o + half) = pack4(l1[0], l1[1], l1[2], l1[3]);
            } else {
                // four consecutive features of a key sit side by side in the cache (same octet)
                bf16_t* base = reinterpret_cast<bf16_t*>(kv.pool) + kv_block(kv, sq, hh, cap);
                append8(base + k_bf16_offset(p, j0, hd), pack4(x0[0], x0[1], x0[2], x0[3]), alone);
                append8(base + k_bf16_offset(p, j0 + half, hd), pack4(x1[0], x1[1], x1[2], x1[3]), alone);
            }
        } else {
            const int u = t - nq4 - nk4;
            const int f0 = (u >> 6) * 256 + (u & 63);
            // the four values of a plane are asked for together (value by value, each through its planes, 20 rows of
            // 4 kv heads in four slices took 9.7 us between events instead of 7.8); past the last value the last one is read again
            float v[4];
            int x[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                x[k] = vin + min(f0 + 64 * k, Hkv * hd - 1);
                v[k] = x[k] < from ? r0[x[k]] : rp[x[k]];
            }
            for (int q = 1; q < splits; ++q) {
                float u[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) u[k] = x[k] < from ? 0.f : rp[x[k] + (int64_t)q * plane];
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = x[k] < from ? v[k] : v[k] + u[k];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int f = f0 + 64 * k;
                if (f >= Hkv * hd) break;
                bf16_t* base = reinterpret_cast<bf16_t*>(kv.pool) + kv_block(kv, sq, f >> 7, cap);
                append2(base + v_bf16_offset(p, f & 127, hd), f32_to_bf16(v[k]), alone);
            }
        }
    }
}

// ------------------------------------------------------------------ decode attention
// One workgroup per (kv head g, list entry i); its waves (four, or one for short rows) take the 32-position
// groups of the row's cache round-robin and are merged at the end.  Per group:
//   S^T[pos][head] = K[pos][:] . q[head][:]   two 16x16x32 MFMAs per 32 features
//   online softmax over positions (fp32, per head)
//   O^T[feat][head] += V^T[feat][pos] P^T[pos][head]
// The G = H_q/H_kv query heads that share the kv head are the N dimension of
// the MFMAs, so each cached element is read from HBM once and used G times.
// The result registers of the score MFMAs are, lane for lane, the P operand
// of the value MFMAs (the grouped V layout is chosen to make that so).
// q and P enter as bf16 (hi, lo) pairs: two MFMAs each, fp32-grade products.
// The work of one workgroup: list entries first .. first + cnt - 1 of kv head g, share `share` of n_splits of
// the position groups.  AHEAD: a wave asks for its next group before it works on the current one.
#define ATTN_SHARE 132      /* floats of one head's share of a row: a multiple of four, so that they move 16 bytes at a time */
template <int WAVES>
struct AttnShared {
    float m[WAVES][16];
    float l[WAVES][16];
    float o[WAVES][16][132];    // 128 features; rows of 132 floats put a 16-byte access of the 16 columns into different banks
};

// Rotation and append in the attention of a decode step (FUSED): the q|k|v product's result is taken as it is (from buf, or
// as `splits` K-slice planes, as in k_bf16_rope_append; some columns so and others so is for context passes).  Wave 0 and 1 rotate the queries of
// the workgroup's heads (features 32 c + .. and 32 c + 64 + .. are pairs, c = 0 and 1) and leave them as (hi, lo) pairs in
// LDS, wave 3 rotates and appends the key and appends the value, all while the other waves' first cached keys and values are
// on their way.  The group that holds the new position is read after the barrier, from L2.  As a launch of its own this took 3.5 to 4 us on a few
// rows; which calls come here: append_in_attn.
struct QkvIn {
    const float* buf; int ld;                               // of the planes too
    const float* planes; int splits; int64_t plane;
    const float* rope; int max_pos;
    int32_t* status;
    // N times 4 columns of entry i (x[k] a multiple of 4): the loads of two planes under way together
    template <int N>
    __device__ __forceinline__ void rd4(int i, const int (&x)[N], float4 (&v)[N]) const {
        const bool done = splits == 1;
        const float* p = (done ? buf : planes) + (int64_t)i * ld;
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = *reinterpret_cast<const float4*>(p + x[k]);
        if (done) return;
        for (int q = 1; q < splits; q += 2) {
            float4 u[2][N];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int k = 0; k < N; ++k) u[h][k] = *reinterpret_cast<const float4*>(p + x[k] + min(q + h, splits - 1) * plane);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (q + h >= splits) break;
#pragma unroll
                for (int k = 0; k < N; ++k) { v[k].x += u[h][k].x; v[k].y += u[h][k].y; v[k].z += u[h][k].z; v[k].w += u[h][k].w; }
            }
        }
    }
};

// four rotation pairs: columns j .. j + 3 (a) with j + 64 .. (b), cs = cos, sin of the first
__device__ __forceinline__ void rotate4(const float4& a, const float4& b, const float* cs, float (&x0)[4], float (&x1)[4]) {
    const float4 c0 = *reinterpret_cast<const float4*>(cs), c1 = *reinterpret_cast<const float4*>(cs + 4);
    x0[0] = a.x * c0.x - b.x * c0.y; x0[1] = a.y * c0.z - b.y * c0.w; x0[2] = a.z * c1.x - b.z * c1.y; x0[3] = a.w * c1.z - b.w * c1.w;
    x1[0] = b.x * c0.x + a.x * c0.y; x1[1] = b.y * c0.z + a.y * c0.w; x1[2] = b.z * c1.x + a.z * c1.y; x1[3] = b.w * c1.z + a.w * c1.w;
}

// what wave w of the workgroup (kv head g, job) does of it; qs: [c][hi, lo][lane]
__device__ __forceinline__ void rotate_append(uint4 (&qs)[4][2][64], const QkvIn& in, const KvView& kv, const AttnJob& job, int Hq, int g,
                                              bool appends) {
    const int G = Hq / kv.n_kv_heads, i = job.entry, p = job.pos;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, n16 = lane & 15, gq = lane >> 4;
    const bool ok = p >= 0 && p < job.cap && p < in.max_pos;
    const float* cs = in.rope + (int64_t)(ok ? p : 0) * 128;
    if (w < 2) {
        const int x = (g * G + (n16 < G ? n16 : 0)) * 128 + 32 * w + 8 * gq;      // columns without a head read head 0
        float lo[8], hi[8];
        const int xs[4] = {x, x + 4, x + 64, x + 68};
        float4 v[4];
        in.rd4(i, xs, v);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float x0[4], x1[4];
            rotate4(v[h], v[2 + h], cs + 2 * (32 * w + 8 * gq + 4 * h), x0, x1);
#pragma unroll
            for (int k = 0; k < 4; ++k) { lo[4 * h + k] = x0[k]; hi[4 * h + k] = x1[k]; }
        }
        auto put = [&](int c, const float (&v)[8]) {
            uint32_t a[4], b[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                a[k] = pack2(v[2 * k], v[2 * k + 1]);
                b[k] = pack2(v[2 * k] - __uint_as_float(a[k] << 16), v[2 * k + 1] - __uint_as_float(a[k] & 0xffff0000u));
            }
            qs[c][0][lane] = make_uint4(a[0], a[1], a[2], a[3]);
            qs[c][1][lane] = make_uint4(b[0], b[1], b[2], b[3]);
        };
        put(w, lo);
        put(w + 2, hi);
        return;
    }
    if (!appends || w != 3) return;
    if (!ok) {
        if (lane == 0 && g == 0) atomicOr(in.status, 1);
        return;
    }
    bf16_t* base = reinterpret_cast<bf16_t*>(kv.pool) + ((int64_t)kv.layer0 * kv.T + job.off) * (2LL * kv.n_kv_heads * 128) +
                   (int64_t)g * 2LL * job.cap * 128;
    // lanes 0 .. 15 four pairs of the key each, lanes 32 .. 63 four values each
    if (lane < 16) {
        const int j0 = 4 * lane, x = (Hq + g) * 128 + j0;
        const int xs[2] = {x, x + 64};
        float4 v[2];
        in.rd4(i, xs, v);
        float x0[4], x1[4];
        rotate4(v[0], v[1], cs + 2 * j0, x0, x1);
        *reinterpret_cast<uint2*>(base + k_bf16_offset(p, j0, 128)) = make_uint2(pack2(x0[0], x0[1]), pack2(x0[2], x0[3]));
        *reinterpret_cast<uint2*>(base + k_bf16_offset(p, j0 + 64, 128)) = make_uint2(pack2(x1[0], x1[1]), pack2(x1[2], x1[3]));
    } else if (lane >= 32) {
        const int f = 4 * (lane - 32);
        const int xs[1] = {(Hq + kv.n_kv_heads + g) * 128 + f};
        float4 v[1];
        in.rd4(i, xs, v);
        bf16_t* at = base + v_bf16_offset(p, f, 128);         // neighbouring features are 8 positions apart
        at[0] = f32_to_bf16(v[0].x); at[8] = f32_to_bf16(v[0].y); at[16] = f32_to_bf16(v[0].z); at[24] = f32_to_bf16(v[0].w);
    }
}

template <bool PAIR, bool AHEAD, bool FUSED, int WAVES>
__device__ __forceinline__ void attn_streams(AttnShared<WAVES>& sm, const bf16_t* __restrict__ q_hi, const bf16_t* __restrict__ q_lo,
                                             int Hq, const int32_t* __restrict__ idx, const int32_t* __restrict__ pos,
                                             const KvView& kv, uint4* __restrict__ ao, int KB_ao, int n_splits, int share,
                                             float* __restrict__ part, int most, int g, int first, int cnt,
                                             const AttnJob& job = AttnJob{}, const QkvIn& in = QkvIn{}, uint4 (*qs)[2][64] = nullptr) {
    const int G = Hq / kv.n_kv_heads;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int n16 = lane & 15, gq = lane >> 4;
    for (int r0 = 0; r0 < cnt;) {
    int r1 = r0 + 1, cap, n_pos;                            // n_pos: positions read, the longest of the run
    const bf16_t* Kb;
    int my_ent = 0, my_np, n_col = G;
    if constexpr (PAIR) {
        const int sq = kv_row(kv, idx[first + r0]);
        while (r1 < cnt && kv_row(kv, idx[first + r1]) == sq) ++r1;
        n_col = (r1 - r0) * G;                               // live MFMA columns
        cap = kv.cap[sq];
        n_pos = 1;
        for (int j = r0; j < r1; ++j) n_pos = max(n_pos, min(pos[idx[first + j]] + 1, cap));
        my_ent = n16 < n_col ? n16 / G : 0;                  // this lane's column: entry, head, positions
        my_np = n16 < n_col ? max(1, min(pos[idx[first + r0 + my_ent]] + 1, cap)) : 0;
        Kb = reinterpret_cast<const bf16_t*>(kv.pool) + kv_block(kv, sq, g, cap);
    } else {
        cap = job.cap;
        n_pos = job.n_pos;
        my_np = n16 < n_col ? n_pos : 0;
        Kb = reinterpret_cast<const bf16_t*>(kv.pool) +
             ((int64_t)kv.layer0 * kv.T + job.off) * (2LL * kv.n_kv_heads * 128) + (int64_t)g * 2LL * cap * 128;
    }
    const int my_e = first + r0 + my_ent;
    const int my_head = n16 - my_ent * G;

    bf16x8 qh[4], ql[4];
    if constexpr (!FUSED) {
        // Columns without a head read head 0 (their results are not written): eight 16-byte loads.  With a condition
        // on them they became 32 loads of 4 bytes, each with a branch of its own, at the start of every run of
        // entries: 1024 rows of 30 to 100 positions at the 7B shape 438 us, 362 now; 16 rows of the 70B shape in
        // eight shares with their merge 36.4, 33.9; long contexts within 1 %.
        const int64_t qo = ((int64_t)my_e * Hq + (int64_t)g * G + (n16 < n_col ? my_head : 0)) * 128 + 8 * gq;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            qh[c] = as_bf16x8(*reinterpret_cast<const uint4*>(q_hi + qo + 32 * c));
            ql[c] = as_bf16x8(*reinterpret_cast<const uint4*>(q_lo + qo + 32 * c));
        }
    }
    const int n_groups = (n_pos + 31) >> 5;
    // with n_splits > 1 this workgroup covers the share-th share of the position groups (at most 2^26 of them, 16 shares)
    const int g_lo = (int)((unsigned)(n_groups * share) / (unsigned)n_splits);
    const int g_hi = (int)((unsigned)(n_groups * (share + 1)) / (unsigned)n_splits);
    // K and V tiles of one 32-position group as this lane holds them for the MFMAs
    struct KVTiles { uint4 k[2][4]; uint4 v[8]; };
    auto load_kv = [&](int t) -> KVTiles {
        KVTiles x;
        // K: two blocks of 16 positions; slice c of a block is 1 KiB, lane l takes bytes 16 l ..
        const bf16_t* k0 = Kb + (int64_t)t * 8192 + lane * 8;      // the group's 16 KiB: K blocks, then V
        const bf16_t* k1 = k0 + 2048;
        const bf16_t* vg = k0 + 4096;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            x.k[0][c] = load_nt(reinterpret_cast<const uint4*>(k0 + 512 * c));
            x.k[1][c] = load_nt(reinterpret_cast<const uint4*>(k1 + 512 * c));
        }
#pragma unroll
        for (int hb = 0; hb < 8; ++hb) x.v[hb] = load_nt(reinterpret_cast<const uint4*>(vg + hb * 512));
        return x;
    };
    // Decode: a wave asks for its next group before it works on the current one (two workgroups per
    // CU then; against three workgroups that load and compute in turn: -2..4 % from 64 to 192 rows,
    // equal at 256).  Context pass with two entries per workgroup: three workgroups, no prefetch
    // (0.8 % faster there).
    KVTiles nxt;
    if constexpr (AHEAD) {
        const int t0 = min(g_lo + w, max(g_hi - 1, 0));                     // a group this workgroup's row has
        // it holds the position that is appended below, or belongs to the wave that appends and waits for its stores
        const bool late = FUSED && (t0 == n_groups - 1 || w == 3);
        if (!late) nxt = load_kv(t0);
        if constexpr (FUSED) {
            rotate_append(*reinterpret_cast<uint4 (*)[4][2][64]>(qs), in, kv, job, Hq, g, share == n_splits - 1);
            // the appending wave: key and value have arrived in L2
            if (w == 3) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (late) nxt = load_kv(t0);
#pragma unroll
            for (int c = 0; c < 4; ++c) { qh[c] = as_bf16x8(qs[c][0][lane]); ql[c] = as_bf16x8(qs[c][1][lane]); }
        }
    }

    const float inv_sqrt = 1.0f / sqrtf(128.0f);
    const float NEG = -1.0e30f;
    float m_run = NEG, l_run = 0.f;
    floatx4 O[8];
#pragma unroll
    for (int hb = 0; hb < 8; ++hb) O[hb] = floatx4{0.f, 0.f, 0.f, 0.f};

    for (int t = g_lo + w; t < g_hi; t += WAVES) {
        const int p0 = t << 5;
        KVTiles cur;
        if constexpr (AHEAD) {
            cur = nxt;
            if (t + WAVES < g_hi) nxt = load_kv(t + WAVES);
        } else {
            cur = load_kv(t);
        }
        floatx4 S0 = {0.f, 0.f, 0.f, 0.f}, S1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            bf16x8 a0 = as_bf16x8(cur.k[0][c]);
            bf16x8 a1 = as_bf16x8(cur.k[1][c]);
            S0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, qh[c], S0, 0, 0, 0);
            S0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, ql[c], S0, 0, 0, 0);
            S1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, qh[c], S1, 0, 0, 0);
            S1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, ql[c], S1, 0, 0, 0);
        }
        // S0[r]: position p0 + 4 gq + r ; S1[r]: position p0 + 16 + 4 gq + r ; head n16
        float s[8];
        float mx = NEG;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r]     = (p0 + 4 * gq + r < my_np) ? S0[r] * inv_sqrt : NEG;
            s[4 + r] = (p0 + 16 + 4 * gq + r < my_np) ? S1[r] * inv_sqrt : NEG;
            mx = fmaxf(mx, fmaxf(s[r], s[4 + r]));
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx);
        const float alpha = __expf(m_run - m_new);
        float pv[8], lsum = 0.f;
#pragma unroll
        for (int r = 0; r < 8; ++r) { pv[r] = __expf(s[r] - m_new); lsum += pv[r]; }
        l_run = l_run * alpha + lsum;
        m_run = m_new;
        uint4 ph, pl;
        {
            bf16_t hi[8], lo[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                hi[r] = f32_to_bf16(pv[r]);
                lo[r] = f32_to_bf16(pv[r] - bf16_to_f32(hi[r]));
            }
            ph = make_uint4(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16),
                            hi[4] | ((uint32_t)hi[5] << 16), hi[6] | ((uint32_t)hi[7] << 16));
            pl = make_uint4(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16),
                            lo[4] | ((uint32_t)lo[5] << 16), lo[6] | ((uint32_t)lo[7] << 16));
        }
        const bool partial = p0 + 32 > n_pos;
#pragma unroll
        for (int hb = 0; hb < 8; ++hb) {
            uint4 vv = cur.v[hb];
            if (partial) {
                // element j of the chunk is position p0 + 4 gq + j (j < 4) or p0 + 16 + 4 gq + j - 4
                uint32_t* vw = reinterpret_cast<uint32_t*>(&vv);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    int pj = p0 + ((j < 4) ? (4 * gq + j) : (16 + 4 * gq + j - 4));
                    if (pj >= n_pos) vw[j >> 1] &= (j & 1) ? 0x0000ffffu : 0xffff0000u;
                }
            }
            O[hb] = O[hb] * alpha;
            O[hb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vv), as_bf16x8(ph), O[hb], 0, 0, 0);
            O[hb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vv), as_bf16x8(pl), O[hb], 0, 0, 0);
        }
    }
    // O[hb][r]: feature 16 hb + 4 gq + r of head n16 (unnormalised), this wave's positions
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    if (gq == 0) { sm.m[w][n16] = m_run; sm.l[w][n16] = l_run; }
    if (n16 < n_col) {
#pragma unroll
        for (int hb = 0; hb < 8; ++hb)
            *reinterpret_cast<float4*>(&sm.o[w][n16][16 * hb + 4 * gq]) = make_float4(O[hb][0], O[hb][1], O[hb][2], O[hb][3]);
    }
    __syncthreads();
    for (int tt = threadIdx.x; tt < n_col * 16; tt += 64 * WAVES) {
        const int head = tt >> 4, c0 = (tt & 15) * 8;      // head = MFMA column
        const int i = first + r0 + head / G;
        const int hq = head % G;
        float M = sm.m[0][head];
#pragma unroll
        for (int k = 1; k < WAVES; ++k) M = fmaxf(M, sm.m[k][head]);
        float Lsum = 0.f, o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < WAVES; ++k) {
            const float wgt = __expf(sm.m[k][head] - M);
            Lsum += sm.l[k][head] * wgt;
            const float4 u = *reinterpret_cast<const float4*>(&sm.o[k][head][c0]), v = *reinterpret_cast<const float4*>(&sm.o[k][head][c0 + 4]);
            o[0] += u.x * wgt; o[1] += u.y * wgt; o[2] += u.z * wgt; o[3] += u.w * wgt;
            o[4] += v.x * wgt; o[5] += v.y * wgt; o[6] += v.z * wgt; o[7] += v.w * wgt;
        }
        if (n_splits == 1) {
            uint4 pk = make_uint4(pack2(o[0] / Lsum, o[1] / Lsum), pack2(o[2] / Lsum, o[3] / Lsum),
                                  pack2(o[4] / Lsum, o[5] / Lsum), pack2(o[6] / Lsum, o[7] / Lsum));
            int col = (g * G + hq) * 128 + c0;
            ao[afrag_chunk(i, col, KB_ao)] = pk;
        } else {
            // unnormalised share: [i][kv head][share, `most` of them][head][132] = 128 features, max, sum, two unused
            float* p = part + ((((int64_t)i * kv.n_kv_heads + g) * most + share) * 16 + hq) * ATTN_SHARE;
            *reinterpret_cast<float4*>(p + c0) = make_float4(o[0], o[1], o[2], o[3]);
            *reinterpret_cast<float4*>(p + c0 + 4) = make_float4(o[4], o[5], o[6], o[7]);
            if (c0 == 0) { p[128] = M; p[129] = Lsum; }
        }
    }
    r0 = r1;
    if (r0 < cnt) __syncthreads();         // the merge has read the shared arrays before the next run writes them
    }
}

template <bool PAIR, int WAVES>
__global__ void __launch_bounds__(64 * WAVES, PAIR ? 3 : 2)
k_bf16_attn(const bf16_t* __restrict__ q_hi, const bf16_t* __restrict__ q_lo, int Hq,
            const int32_t* __restrict__ idx, const int32_t* __restrict__ n_ptr, int B,
            const int32_t* __restrict__ pos, KvView kv, uint4* __restrict__ ao, int KB_ao, int most,
            float* __restrict__ part, const AttnJob* __restrict__ jobs) {
    __shared__ AttnShared<WAVES> sm;
    const int n = min(*n_ptr, B);
    // PAIR (context pass and other passes over list entries, 2 G <= 16): the workgroup serves the E = 16 / G
    // list entries E y .. E y + E - 1.  Consecutive entries that read the same cache row (a context passed
    // in rising position order) share its K/V stream: entry j of such a run has its G heads in the MFMA
    // columns G j .. G j + G - 1, each column masked at its own entry's position.  With one query head per
    // kv head 16 entries share a stream, with eight heads two.  A change of cache row inside the E entries
    // starts another run, served after the first.
    if constexpr (PAIR) {
        const int E = 16 / (Hq / kv.n_kv_heads), first = E * (int)blockIdx.y;
        if (first >= n) return;
        attn_streams<true, false, false, WAVES>(sm, q_hi, q_lo, Hq, idx, pos, kv, ao, KB_ao, 1, 0, nullptr, 1, blockIdx.x, first, min(E, n - first));
    } else {
        const AttnJob job = jobs[blockIdx.y];  // longest contexts first; slots from n on are not read further
        if ((int)blockIdx.y >= n || (int)blockIdx.z >= job.shares) return;
        attn_streams<false, true, false, WAVES>(sm, q_hi, q_lo, Hq, idx, pos, kv, ao, KB_ao, job.shares, blockIdx.z, part, most, blockIdx.x,
                                  job.entry, 1, job);
    }
}

// The attention of a decode step with rotation and append: batch row b owns cache row b, and no workgroup reads what another
// one appends.
__global__ void __launch_bounds__(256, 2)
k_bf16_attn_decode(QkvIn in, int Hq, const int32_t* __restrict__ n_ptr, int B, KvView kv, uint4* __restrict__ ao, int KB_ao, int most,
                   float* __restrict__ part, const AttnJob* __restrict__ jobs) {
    __shared__ AttnShared<4> sm;
    __shared__ uint4 qs[4][2][64];
    const int n = min(*n_ptr, B);
    const AttnJob job = jobs[blockIdx.y];      // longest contexts first; slots from n on are not read further
    if ((int)blockIdx.y >= n || (int)blockIdx.z >= job.shares) return;
    attn_streams<false, true, true, 4>(sm, nullptr, nullptr, Hq, nullptr, nullptr, kv, ao, KB_ao, job.shares, blockIdx.z, part, most,
                                    blockIdx.x, job.entry, 1, job, in, qs);
}

// ------------------------------------------------------------------ context-pass attention
// What bounds the kernel above in a context pass: 16 MFMA columns per workgroup, so with eight query heads
// per kv head two entries share a pass over the keys and values and a 2000-entry call streams them 1000
// times.  Here a workgroup serves a tile of 4 C 16-column blocks (C per wave; 4 C E entries with E = 16 / G):
// the keys and values of its cache row go through LDS in stages of 64 positions, two stage buffers filled by
// LDS-DMA loads, and every wave works through all of them for its own columns, so no merge follows.  Scores
// and P V take the same operands as above (queries and probabilities as bf16 pairs hi + lo).  Exponentials
// are base 2 with the scale folded in, and a column's running maximum is only raised (and its sums rescaled)
// when it grows by more than 2^8, which leaves the sums in fp32 range and the result unchanged.
// Measured (70B shape, 1999 entries of three contexts of 1400 to 2200 positions): 585 -> 275 to 355 us, machine to
// machine, at 2 us of MFMAs in 4.3 us per stage and pair of waves; what is left is the softmax arithmetic, which the other wave
// of the SIMD covers in part, at the 1.65 GHz the power limit leaves beside the products of the layer.  7B
// shape, 1024 entries of four prompts (C = 1): 73 -> 35 us.  All eight K reads of a group are asked for
// before its first MFMA and the V reads before the softmax; with a read in front of each product C = 2 took
// 315 us, and with one register too many (a spill's reload waits for the stage just requested) up to 760.
// Entries of a tile that name more than two cache rows are served by attn_streams instead, one workgroup per
// E entries as above: the workgroups y = sub * tiles + t, sub = 0 .. 4 C - 1, exist for that; on a tile of
// one or two rows only sub = 0 works.
// A column's probability is 0 at the positions it is masked at, but 0 times a value that is infinite or NaN is NaN,
// and the entries of a tile read each other's positions: a tile with such a result is served again entry group
// by entry group, so that a token with a NaN, or an entry refused for its position, reaches no further among
// the entries of its call than it did when all calls went that way.
#define CTX_STAGE 2048                        /* uint4 of a stage: two groups of 32 positions, 16 KiB each */

// maximum over the four lanes that hold a column (lane, lane ^ 16, lane ^ 32, lane ^ 48)
__device__ __forceinline__ float column_max(float v) {
    auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Returns, alike in all waves, whether a result came out infinite or NaN.
template <int C>
__device__ __forceinline__ bool attn_tile(uint4* lds, const bf16_t* __restrict__ q_hi, const bf16_t* __restrict__ q_lo, int Hq,
                                          const int32_t* __restrict__ idx, const int32_t* __restrict__ pos, const KvView& kv,
                                          uint4* __restrict__ ao, int KB_ao, int g, int first, int cnt) {
    const int G = Hq / kv.n_kv_heads, E = 16 / G;
    const int lane = threadIdx.x & 63, n16 = lane & 15, gq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned lane_bytes = (unsigned)lane * 16u, lds0 = (unsigned)(size_t)lds;
    const float scale2 = (1.0f / sqrtf(128.0f)) * 1.44269504088896340736f;    // exp(x) = 2^(x log2 e)
    const float NEG = -1.0e30f;
    float odd = 0.f;                                         // NaN once a result is infinite or NaN
    for (int r0 = 0; r0 < cnt;) {
        const int sq = __builtin_amdgcn_readfirstlane(kv_row(kv, idx[first + r0]));
        int r1 = r0 + 1;
        while (r1 < cnt && __builtin_amdgcn_readfirstlane(kv_row(kv, idx[first + r1])) == sq) ++r1;
        const int cap = kv.cap[sq];
        int n_pos = 1;                                       // positions read: the longest of the run
        for (int j = r0 + lane; j < r1; j += 64) n_pos = max(n_pos, min(pos[idx[first + j]] + 1, cap));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) n_pos = max(n_pos, __shfl_xor(n_pos, o, 64));
        n_pos = __builtin_amdgcn_readfirstlane(n_pos);
        const uint4* Kb = reinterpret_cast<const uint4*>(reinterpret_cast<const bf16_t*>(kv.pool) + kv_block(kv, sq, g, cap));
        const uint64_t kv_base = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)Kb >> 32)) << 32) |
                                 (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)Kb);
        const int n_groups = (n_pos + 31) >> 5, n_st = (n_groups + 1) >> 1;

        // this lane's column of each block: entry, head, positions (0: a column without an entry of the run)
        int ent[C], np[C];
        bf16x8 qh[C][4], ql[C][4];
        int lo_np = 0x7fffffff, hi_np = 0;                   // over the wave's live columns
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const int e = (w * C + j) * E + n16 / G;
            const bool live = n16 < E * G && e >= r0 && e < r1;
            ent[j] = live ? first + e : -1;
            np[j] = live ? max(1, min(pos[idx[first + e]] + 1, cap)) : 0;
            const uint4 z = make_uint4(0, 0, 0, 0);
            const int64_t qo = ((int64_t)(first + (live ? e : r0)) * Hq + (int64_t)g * G + n16 % G) * 128 + 8 * gq;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                qh[j][c] = as_bf16x8(live ? *reinterpret_cast<const uint4*>(q_hi + qo + 32 * c) : z);
                ql[j][c] = as_bf16x8(live ? *reinterpret_cast<const uint4*>(q_lo + qo + 32 * c) : z);
            }
            int l = live ? np[j] : 0x7fffffff, h = np[j];
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) { l = min(l, __shfl_xor(l, o, 64)); h = max(h, __shfl_xor(h, o, 64)); }
            lo_np = min(lo_np, l);
            hi_np = max(hi_np, h);
        }
        lo_np = __builtin_amdgcn_readfirstlane(lo_np);
        hi_np = __builtin_amdgcn_readfirstlane(hi_np);
        float m_run[C], l_run[C];
        floatx4 O[C][8];
#pragma unroll
        for (int j = 0; j < C; ++j) {
            m_run[j] = NEG; l_run[j] = 0.f;
#pragma unroll
            for (int hb = 0; hb < 8; ++hb) O[j][hb] = floatx4{0.f, 0.f, 0.f, 0.f};
        }

        // wave w sends pieces 8 w .. 8 w + 7 (1 KiB each) of a stage; a group past the last one of the row is
        // replaced by the last one (its positions are masked)
        auto issue = [&](int t) {
            const int grp = min(2 * t + (w >> 1), n_groups - 1);
            const uint4* src = reinterpret_cast<const uint4*>(kv_base + ((uint64_t)grp << 14) + ((w & 1) << 13));
            const unsigned dst = lds0 + (unsigned)((t & 1) * CTX_STAGE + w * 512) * 16u;
#pragma unroll
            for (int p = 0; p < 8; ++p) dma_tile(src + p * 64, lane_bytes, dst + (unsigned)p * 1024u);
        };
        // the queries are in registers before the first LDS-DMA load: a wait for them inside the loop would wait
        // for the stage that has just been asked for
#pragma unroll
        for (int j = 0; j < C; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) asm volatile("" : "+v"(qh[j][c]), "+v"(ql[j][c]));
        __syncthreads();                                     // an earlier run's last stage has been read
        issue(0);
        for (int t = 0; t < n_st; ++t) {
            // this wave's pieces of stage t have landed; after the barrier everybody's have, and the other
            // buffer (stage t - 1) has been read by all waves
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (t + 1 < n_st) issue(t + 1);
            const int p0 = t << 6;
            if (p0 >= hi_np) continue;                       // no column of this wave reaches this stage
            const uint4* st = lds + (t & 1) * CTX_STAGE + lane;
            const bool edge = p0 + 64 > lo_np;               // a column of the wave ends inside this stage
#pragma unroll 1
            for (int q = 0; q < 2; ++q) {                    // 32 positions from pg on, their K and V at kvg
                const uint4* kvg = st + q * 1024;
                const int pg = p0 + 32 * q;
                if (pg >= hi_np) break;
                bf16x8 kf[8];
#pragma unroll
                for (int c = 0; c < 4; ++c) { kf[c] = as_bf16x8(kvg[c * 64]); kf[4 + c] = as_bf16x8(kvg[256 + c * 64]); }
                floatx4 S[C][2];                             // [pb][r]: position pg + 16 pb + 4 gq + r of column n16
#pragma unroll
                for (int j = 0; j < C; ++j) S[j][0] = S[j][1] = floatx4{0.f, 0.f, 0.f, 0.f};
                __builtin_amdgcn_sched_barrier(0);           // all eight K reads are under way before the first MFMA
#pragma unroll
                for (int c = 0; c < 4; ++c) {
#pragma unroll
                    for (int j = 0; j < C; ++j) {
                        S[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[c], qh[j][c], S[j][0], 0, 0, 0);
                        S[j][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[4 + c], qh[j][c], S[j][1], 0, 0, 0);
                    }
#pragma unroll
                    for (int j = 0; j < C; ++j) {
                        S[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[c], ql[j][c], S[j][0], 0, 0, 0);
                        S[j][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[4 + c], ql[j][c], S[j][1], 0, 0, 0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                uint4 vf[8];                                 // under way during the softmax
#pragma unroll
                for (int hb = 0; hb < 8; ++hb) vf[hb] = kvg[512 + hb * 64];
                __builtin_amdgcn_sched_barrier(0);
                if (edge) {
                    asm volatile("");                        // a branch, not 8 C selects in every group
#pragma unroll
                    for (int j = 0; j < C; ++j) {
                        const int end = np[j] - pg - 4 * gq; // the lane's positions 16 pb + r from here on are masked
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (16 * (i >> 2) + (i & 3) >= end) S[j][i >> 2][i & 3] = NEG;
                    }
                }
                float mx[C];
                bool raise = false;
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    mx[j] = NEG;
#pragma unroll
                    for (int i = 0; i < 8; ++i) mx[j] = fmaxf(mx[j], S[j][i >> 2][i & 3]);
                    mx[j] = column_max(mx[j]) * scale2;
                    raise = raise || mx[j] > m_run[j] + 8.0f;
                }
                if (__any(raise)) {
#pragma unroll
                    for (int j = 0; j < C; ++j) {
                        const float m_new = mx[j] > m_run[j] + 8.0f ? mx[j] : m_run[j];
                        const float alpha = __builtin_amdgcn_exp2f(m_run[j] - m_new);
                        m_run[j] = m_new;
                        l_run[j] *= alpha;
#pragma unroll
                        for (int hb = 0; hb < 8; ++hb) O[j][hb] = O[j][hb] * alpha;
                    }
                }
                uint4 ph[C], pl[C];
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    float pv[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) pv[i] = __builtin_amdgcn_exp2f(fmaf(S[j][i >> 2][i & 3], scale2, -m_run[j]));
                    l_run[j] += ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
                    uint32_t hw[4], lw[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        hw[i] = pack2(pv[2 * i], pv[2 * i + 1]);
                        lw[i] = pack2(pv[2 * i] - __uint_as_float(hw[i] << 16), pv[2 * i + 1] - __uint_as_float(hw[i] & 0xffff0000u));
                    }
                    ph[j] = make_uint4(hw[0], hw[1], hw[2], hw[3]);
                    pl[j] = make_uint4(lw[0], lw[1], lw[2], lw[3]);
                }
                if (pg + 32 > n_pos) {                       // what lies beyond the row's positions was never written
                    const int end = n_pos - pg - 4 * gq;     // element e of a lane's chunk is position e (e < 4) or 12 + e
#pragma unroll
                    for (int hb = 0; hb < 8; ++hb) {
                        uint32_t* vw = reinterpret_cast<uint32_t*>(&vf[hb]);
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if ((e < 4 ? e : 12 + e) >= end) vw[e >> 1] &= (e & 1) ? 0x0000ffffu : 0xffff0000u;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int half = 0; half < 2; ++half) {
#pragma unroll
                    for (int j = 0; j < C; ++j)
#pragma unroll
                        for (int u = 4 * half; u < 4 * half + 4; ++u)
                            O[j][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vf[u]), as_bf16x8(ph[j]), O[j][u], 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < C; ++j)
#pragma unroll
                        for (int u = 4 * half; u < 4 * half + 4; ++u)
                            O[j][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vf[u]), as_bf16x8(pl[j]), O[j][u], 0, 0, 0);
                }
            }
        }
        // O[j][hb][r]: feature 16 hb + 4 gq + r of column n16 of block j
        int chunk0 = (g * G + n16 % G) * 128;
        asm volatile("" : "+v"(chunk0));                     // the addresses below are not worth registers in the loop
#pragma unroll
        for (int j = 0; j < C; ++j) {
            float l = l_run[j];
            l += __shfl_xor(l, 16, 64);
            l += __shfl_xor(l, 32, 64);
            if (ent[j] < 0) continue;
#pragma unroll
            for (int hb = 0; hb < 8; ++hb) {
                const int col = chunk0 + 16 * hb + 4 * gq;
                O[j][hb] = O[j][hb] / l;
#pragma unroll
                for (int r = 0; r < 4; ++r) odd = fmaf(O[j][hb][r], 0.f, odd);
                uint2* dst = reinterpret_cast<uint2*>(ao + afrag_chunk(ent[j], col & ~7, KB_ao)) + ((col >> 2) & 1);
                *dst = make_uint2(pack2(O[j][hb][0], O[j][hb][1]), pack2(O[j][hb][2], O[j][hb][3]));
            }
        }
        r0 = r1;
    }
    return __syncthreads_or(odd != 0.f);
}

template <int C>
__global__ void __launch_bounds__(256, 2)
k_bf16_attn_ctx(const bf16_t* __restrict__ q_hi, const bf16_t* __restrict__ q_lo, int Hq, const int32_t* __restrict__ idx,
                const int32_t* __restrict__ n_ptr, int B, const int32_t* __restrict__ pos, KvView kv, uint4* __restrict__ ao,
                int KB_ao, const int32_t* __restrict__ order) {
    __shared__ uint4 lds[2 * CTX_STAGE];
    static_assert(sizeof(AttnShared<4>) <= sizeof(lds), "the merge arrays share the stage buffers");
    const int n = min(*n_ptr, B);
    const int E = 16 / (Hq / kv.n_kv_heads), TE = 4 * C * E;
    const int tiles = gridDim.y / (4 * C);                   // of the batch's capacity; n entries fill the first ones
    const int sub = blockIdx.y / tiles, t = blockIdx.y % tiles;
    if (t * TE >= n) return;
    const int first = order[t] * TE, cnt = min(TE, n - first);
    const int lane = threadIdx.x & 63;
    int changes = 0;                                         // cache-row changes inside the tile
    for (int j = lane; j + 1 < cnt; j += 64) changes += kv_row(kv, idx[first + j]) != kv_row(kv, idx[first + j + 1]) ? 1 : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) changes += __shfl_xor(changes, o, 64);
    int k = sub, k_end = sub + 1;                            // entry groups this workgroup serves one by one
    if (__builtin_amdgcn_readfirstlane(changes) <= 1) {
        if (sub != 0 || !attn_tile<C>(lds, q_hi, q_lo, Hq, idx, pos, kv, ao, KB_ao, blockIdx.x, first, cnt)) return;
        k_end = 4 * C;
        __syncthreads();                                     // what the tile wrote comes before what follows
    }
    for (; k < k_end && k * E < cnt; ++k) {
        attn_streams<true, true, false, 4>(*reinterpret_cast<AttnShared<4>*>(lds), q_hi, q_lo, Hq, idx, pos, kv, ao, KB_ao, 1, 0, nullptr,
                                 1, blockIdx.x, first + k * E, min(E, cnt - k * E));
        __syncthreads();                                     // the merge has read the shared arrays
    }
}

// merges the position shares of k_bf16_attn in share order: one workgroup per (kv head, list entry)
__global__ void __launch_bounds__(256)
k_bf16_attn_merge(const float* __restrict__ part, int Hq, int Hkv, int most, const AttnJob* __restrict__ jobs,
                  const int32_t* __restrict__ n_ptr, int B, uint4* __restrict__ ao, int KB_ao) {
    const int g = blockIdx.x;
    const int n = min(*n_ptr, B);
    const int i = jobs[blockIdx.y].entry, shares = jobs[blockIdx.y].shares;
    if ((int)blockIdx.y >= n || shares == 1) return;         // a single share wrote the result itself
    const int G = Hq / Hkv;
    const int head = threadIdx.x >> 4, c0 = (threadIdx.x & 15) * 8;
    if (head >= G) return;
    const float* base = part + (((int64_t)i * Hkv + g) * most * 16 + head) * ATTN_SHARE;
    float M = -1.0e30f;
    for (int q = 0; q < shares; ++q) M = fmaxf(M, base[(int64_t)q * 16 * ATTN_SHARE + 128]);
    float L = 0.f, o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int q = 0; q < shares; ++q) {
        const float* p = base + (int64_t)q * 16 * ATTN_SHARE;
        const float4 u = *reinterpret_cast<const float4*>(p + c0), v = *reinterpret_cast<const float4*>(p + c0 + 4);
        const float wq = __expf(p[128] - M);
        L += p[129] * wq;
        o[0] += u.x * wq; o[1] += u.y * wq; o[2] += u.z * wq; o[3] += u.w * wq;
        o[4] += v.x * wq; o[5] += v.y * wq; o[6] += v.z * wq; o[7] += v.w * wq;
    }
    uint4 pk = make_uint4(pack2(o[0] / L, o[1] / L), pack2(o[2] / L, o[3] / L), pack2(o[4] / L, o[5] / L),
                          pack2(o[6] / L, o[7] / L));
    ao[afrag_chunk(i, (g * G + head) * 128 + c0, KB_ao)] = pk;
}

// ------------------------------------------------------------------ host side
static KvView make_view(const ee_model* m, const ee_kv* kv, int layer, const ee_batch* b) {
    return KvView{kv->pool, kv->d_cap, kv->d_off, kv->T, m->cfg.n_kv_heads, m->cfg.head_dim, layer - 1, b->kv_seq};
}

// Blocks that share a row in k_bf16_rope_append: one item per thread, up to eight blocks, as long as the launch stays
// within 8192 blocks (four rounds on the chip: each block first waits for its entry's row, position and cache row),
// but four.  7B shape: 64 rows 8.5 us with four blocks, 8.1 with eight, 1024 context entries 32 and 22; seven
// skipped layers of 32 rows 12.2 with one block, 9.0 with six.  70B shape: 256 rows 14.6 with four, 13.7 with six,
// 1999 context entries 40 and 48.
static int rope_blocks(int n_q, int n_kv, int rows) {
    const int items = n_q * 16 + n_kv * 16 + (n_kv * 128 + 255) / 256 * 64;
    return std::min({8, (items + 255) / 256, std::max(4, 8192 / rows)});
}

// picks the tile configuration from the row capacity of the batch: at most 64 rows come here (gemm_tiled)
template <int NS, int EPI>
static void gemm(const void* X, const void* W, int N, int K, int NBs, int nb_off, const int32_t* n_ptr, int B,
                 const EpiArgs& ep, hipStream_t s, const ZBatch& zb = ZBatch{}, int nz = 1) {
    auto kern = B <= 32 ? k_bf16_gemm<1, NS, 8, EPI> : k_bf16_gemm<2, NS, 8, EPI>;
    hipLaunchKernelGGL(kern, dim3((N / 32 + NS - 1) / NS, 1, nz), dim3(64 * 8), 0, s, (const uint4*)X, (const uint4*)W, K / 16, N / 32, NBs, nb_off,
                       n_ptr, B, ep, zb);
}

// Adds the K-slice planes in slice order into out.  One thread per 4 consecutive columns.
__global__ void __launch_bounds__(256)
k_splitk_finish(const float* __restrict__ partial, int64_t plane, int ld, int splits, int N,
                const int32_t* __restrict__ n_ptr, int B, float* __restrict__ out, int ldo) {
    const int n = min(*n_ptr, B);
    const int row = blockIdx.y;
    if (row >= n) return;
    const int col = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (col >= N) return;
    const float* p = partial + (int64_t)row * ld + col;
    float4 sum = *reinterpret_cast<const float4*>(p);
    for (int q = 1; q < splits; ++q) {
        float4 v = *reinterpret_cast<const float4*>(p + (int64_t)q * plane);
        sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
    }
    *reinterpret_cast<float4*>(out + (int64_t)row * ldo + col) = sum;
}

// Residual finish of a K-sliced product, one block per list entry: h[row id] += sum of the
// slice planes (in slice order, as k_splitk_finish does), and, if a gain is given, the RMSNorm
// of the updated row straight into the operand matrix of the next product.
__global__ void __launch_bounds__(NORM_THREADS)
k_splitk_resid_norm(const float* __restrict__ partial, int64_t plane, int ld, int splits, int N,
                    const int32_t* __restrict__ n_ptr, int B, int near, float* h, int ldh, const int32_t* __restrict__ idx,
                    const float* gain, float eps, uint4* xout, JobArgs ja) {
    __shared__ float red[NORM_THREADS / 64];
    const int n = min(*n_ptr, B);
    const int i = entry_of_block(blockIdx.x, near);
    if (i >= n) return;
    leave_job(ja, i, n, [&](int j) { return idx[j]; });
    float* hrow = h + (int64_t)idx[i] * ldh;
    const float* prow = partial + (int64_t)i * ld;
    if ((N >> 3) <= NORM_THREADS) {
        // at most one 8-float chunk per thread (d <= 8192): the updated chunk stays in registers for
        // the norm instead of being read back twice; same arithmetic, same bits as the general path
        const int c = threadIdx.x;
        const bool has = c < (N >> 3);
        float4 o0 = make_float4(0.f, 0.f, 0.f, 0.f), o1 = o0;
        if (has) {
            const float* p = prow + c * 8;
            float4 s0 = *reinterpret_cast<const float4*>(p), s1 = *reinterpret_cast<const float4*>(p + 4);
#pragma unroll 4
            for (int q = 1; q < splits; ++q) {
                const float4 v0 = *reinterpret_cast<const float4*>(p + (int64_t)q * plane);
                const float4 v1 = *reinterpret_cast<const float4*>(p + (int64_t)q * plane + 4);
                s0.x += v0.x; s0.y += v0.y; s0.z += v0.z; s0.w += v0.w;
                s1.x += v1.x; s1.y += v1.y; s1.z += v1.z; s1.w += v1.w;
            }
            float4* hp = reinterpret_cast<float4*>(hrow + c * 8);
            o0 = hp[0]; o1 = hp[1];
            o0.x += s0.x; o0.y += s0.y; o0.z += s0.z; o0.w += s0.w;
            o1.x += s1.x; o1.y += s1.y; o1.z += s1.z; o1.w += s1.w;
            hp[0] = o0; hp[1] = o1;
        }
        if (gain == nullptr) return;
        float ss = 0.f;
        if (has) ss += sum_sq8(o0, o1);
        ss = waves_sum(ss, red);
        const float inv = 1.0f / sqrtf(ss / (float)N + eps);
        if (has) {
            const float4* g4 = reinterpret_cast<const float4*>(gain);
            const float4 ga = g4[2 * c], gb = g4[2 * c + 1];
            uint4 o;
            o.x = pack2((o0.x * inv) * ga.x, (o0.y * inv) * ga.y);
            o.y = pack2((o0.z * inv) * ga.z, (o0.w * inv) * ga.w);
            o.z = pack2((o1.x * inv) * gb.x, (o1.y * inv) * gb.y);
            o.w = pack2((o1.z * inv) * gb.z, (o1.w * inv) * gb.w);
            xout[afrag_chunk(i, c * 8, N >> 4)] = o;
        }
        return;
    }
    for (int c = threadIdx.x; c < (N >> 3); c += blockDim.x) {
        const float* p = prow + c * 8;
        float4 s0 = *reinterpret_cast<const float4*>(p), s1 = *reinterpret_cast<const float4*>(p + 4);
#pragma unroll 4
        for (int q = 1; q < splits; ++q) {
            const float4 v0 = *reinterpret_cast<const float4*>(p + (int64_t)q * plane);
            const float4 v1 = *reinterpret_cast<const float4*>(p + (int64_t)q * plane + 4);
            s0.x += v0.x; s0.y += v0.y; s0.z += v0.z; s0.w += v0.w;
            s1.x += v1.x; s1.y += v1.y; s1.z += v1.z; s1.w += v1.w;
        }
        float4* hp = reinterpret_cast<float4*>(hrow + c * 8);
        float4 o0 = hp[0], o1 = hp[1];
        o0.x += s0.x; o0.y += s0.y; o0.z += s0.z; o0.w += s0.w;
        o1.x += s1.x; o1.y += s1.y; o1.z += s1.z; o1.w += s1.w;
        hp[0] = o0; hp[1] = o1;
    }
    if (gain != nullptr) rmsnorm_row(hrow, gain, eps, N, xout, i, red);   // reads back this thread's own chunks
}

// Tile-rows per workgroup (NS) and K slices of k_bf16_gemm_few: the pair with the shortest estimate.  Workgroups are
// taken in rounds of one per CU; a round lasts as long as its slowest bound, softened (4-norm), of what a CU gets at most
// (50 GB/s, weights and live lines of X), memory (6.3 TB/s of weights) and both kinds over all CUs (15 TB/s).  The constants
// are fitted to products of four shapes at 1, 16 and 48 rows, each with NS 1 .. 4 and 1 .. 16 slices: of the 48, the pair
// chosen is on average 0.7 % and at most 4 % above the best one (q|k|v of the 70B shape, 1 row: 30.9 us with 3 and two
// slices; 40.3 with 1 and one, 47.6 with 4 and one).  A slice keeps 32 K tiles, eight per wave.
struct FewShape { int NS = 4, splits = 1; };
static FewShape few_shape(int tile_rows, int KB, int rows, int nz, int max_splits) {
    const int quads = KB / 4, groups = (rows + 127) / 128;
    const float x_kib = (std::min(rows, 128) + 7) / 8 * 0.25f;      // KiB of X per K tile
    FewShape best;
    float best_t = 1e30f;
    for (int NS = 1; NS <= 4; ++NS)
        for (int sp = 1; sp <= max_splits && (sp == 1 || quads / sp >= 8); ++sp) {
            const int wgs = (tile_rows + NS - 1) / NS * sp * nz * groups, full = wgs / 256, last = wgs % 256;
            const float steps = 4.0f * ((quads + sp - 1) / sp), w = steps * NS, wx = w + steps * x_kib;    // KiB of a workgroup
            auto round = [&](int c) {
                const float a = wx / 50.f, m = c * w / 6300.f, x = c * wx / 15000.f;
                return std::sqrt(std::sqrt(a * a * a * a + m * m * m * m + x * x * x * x));
            };
            float t = (rows > 64 ? 0.7f : 0.3f) * sp + (sp > 1 ? (float)sp * rows * tile_rows * (32 * 8) / 4.0e6f : 0.f);       // us
            t += std::max(0, full + (last > 0) - 2);
            if (full > 0) t += full * round(256);
            if (last > 0) t += round(last);
            if (t < best_t) { best_t = t; best = FewShape{NS, sp}; }
        }
    return best;
}

// threads of a block that normalises a row of d values: one per chunk of 8 up to NORM_THREADS, and a wave for the attention's job where there is room
static int norm_threads(int d, const JobArgs& jobs) {
    const int chunks = (d / 8 + 63) / 64 * 64;
    return std::min(NORM_THREADS, chunks + (jobs.jobs != nullptr ? 64 : 0));
}

// what the caller wants done with the K-slice planes of a product
struct SliceTail {
    const float* norm_gain = nullptr;   // RESID: also normalise the updated rows with this gain ...
    float        eps = 0.f;
    uint4*       norm_out = nullptr;    // ... into this operand matrix
    bool*        norm_done = nullptr;   // set when that happened
    int          defer_most = 0;        // STORE: leave up to so many planes to the caller ...
    int*         splits_out = nullptr;  // ... who gets their number (1 = the result is in out already)
    int*         from_out = nullptr;    // ... and, from a caller that can take a part of the columns so, the first one in planes
    JobArgs      jobs = {};             // RESID: the attention jobs to leave beside the norm
};

// the launch that adds the K-slice planes of a product, where there are any and the caller does not do it itself
template <int EPI>
static void finish_slices(const ee_batch* b, int N, int splits, const int32_t* n_ptr, int B, const EpiArgs& ep, hipStream_t s,
                          const SliceTail& tail) {
    if (tail.splits_out) *tail.splits_out = splits;
    if (splits == 1) return;
    const int64_t plane = (int64_t)((B + 31) / 32 * 32) * N;
    if (EPI == EPI_RESID) {
        hipLaunchKernelGGL(k_splitk_resid_norm, dim3(entry_grid(B)), dim3(norm_threads(N, tail.jobs)), 0, s, b->wsp<float>(b->W.gemm_part),
                           plane, N, splits, N, n_ptr, B, entry_near(B), ep.out, ep.ldo, ep.idx, tail.norm_gain, tail.eps, tail.norm_out, tail.jobs);
        if (tail.norm_gain && tail.norm_done) *tail.norm_done = true;
    } else if (splits > tail.defer_most) {
        if (tail.splits_out) *tail.splits_out = 1;
        hipLaunchKernelGGL(k_splitk_finish, dim3((N / 4 + 255) / 256, B), dim3(256), 0, s, b->wsp<float>(b->W.gemm_part), plane, N, splits, N,
                           n_ptr, B, ep.out, ep.ldo);
    }
}

// Whether the products of one launch take the 256-column tile: it loads each activation tile once per 256 columns instead
// of once per 128, which is worth it when it still gives every CU a workgroup
static bool wide_tiles(int N, int row_groups, int nz) { return N % 256 == 0 && N / 256 * row_groups * nz >= 200; }

// how full the rounds of one workgroup per CU are
static float rounds_filled(int wgs) { return wgs == 0 ? 0.f : (float)wgs / (float)((wgs + 255) / 256 * 256); }

// Whether a product takes k_bf16_gemm_few: up to 128 rows, from 4 MiB of weights on (below, launches wait for memory
// once or twice whatever the kernel: O of a 576-wide model 6.7 us on the weight-streaming kernel and its norm 3.3, 9.5
// here).  Where a tile width fills its rounds to 80 % gate/up stays with the tile kernels: they read X once per 192 or 256
// columns (gate/up of the 70B shape, 224 workgroups, 16 rows 141 and 142 us, 48 rows 143 and 149, 128 rows 157 and 189).
// Elsewhere, tile kernels with the streaming kernel / this one, whole
// launches with the finish: 7B shape 16 rows q|k|v 25.1 / 21.6 us, O 17.4 / 15.3, gate/up 39.8 / 31.2 (172 workgroups / 230),
// down 25.1 / 22.7, 72 rows 31.3 / 27.1, 22.4 / 21.3, 48.4 / 38.7, 30.4 / 29.3; 2048-wide model gate/up 16 rows 22.6 / 13.5, 72
// rows 28.5 / 21.0; 70B shape 16 rows q|k|v 33.8 / 30.9, O 34.1 / 30.4, down 82.3 / 76.9, 128 rows 46.3 / 44.4, 47.4 / 45.3,
// 101 / 94; exit head of the 70B shape 64 rows 89 / 86, 72 rows 106 / 93.
// A head whose 256-column tiles fill their rounds to 77 % stays with them too: 4096 wide, tiles / here, 64 rows of 51200 logits
// (200 tiles) 83.6 and 89.1 us, of 65536 (256) 99.7 and 103.3, of 102400 (400) 160 and 178, of 131072 (512) 206 and 220, 128 rows
// 213 and 267, one row 202 and 235; of 98304 (384, 75 %) 160 / 147, of 76800 (300) 150 / 132, of 40960 (tiles of 128) 96.4 / 76.7.
// Above 128 rows an X tile per 128 columns is too much (head of the 7B shape 144 rows 65 / 115) where the tile kernels can
// run (N and K multiples of 128); for other shapes the whole range is here: layer of 576 / 2880 values and 72 rows 79 / 56
// and 211 / 100 us on the streaming kernel / here, 400 rows 293 / 76 and 977 / 227, context pass of 2048 entries 392 / 143
// and 1518 / 696.
template <int EPI>
static bool few_rows(int N, int K, int rows, int B) {
    const bool on_grid = N % 128 == 0 && K % 128 == 0;
    if (!on_grid && B > 64) return true;
    if (rows > 128 || (int64_t)N * K < ((int64_t)2 << 20)) return false;
    if (!on_grid) return true;
    if (EPI == EPI_EXIT) return !(wide_tiles(N, 1, 1) && rounds_filled(N / 256) >= 0.77f);
    if (EPI != EPI_SWIGLU) return true;
    float fill = 0.f;                                        // widths: as gate/up takes them below
    for (int t = 8; t >= 4; t -= 2) {
        const int wgs = (N / 32 + t - 1) / t;
        if (t < 8 || N % 256 == 0) fill = std::max(fill, (float)(N / 32) / (float)((wgs + 255) / 256 * 256 * t));
    }
    return fill < 0.8f;
}

template <int EPI>
static void launch_few(const ee_batch* b, const void* X, const void* W, int N, int K, int NBs, int nb_off, const int32_t* n_ptr, int B,
                       int rows, const EpiArgs& ep, hipStream_t s, const ZBatch& zb, int nz, const SliceTail& tail) {
    const int Mpad = (B + 31) / 32 * 32, groups = (rows + 127) / 128;
    float* part = b->wsp<float>(b->W.gemm_part);
    int most = 1;                                            // slices: only where somebody adds the planes
    if (nz == 1 && (EPI == EPI_RESID || (EPI == EPI_STORE && tail.defer_most > 0)))
        most = (int)std::min<size_t>(16, b->W.gemm_part_bytes / ((size_t)Mpad * N * sizeof(float)));
    const FewShape f = few_shape(N / 32, K / 16, rows, nz, most);
    const int units = (N / 32 + f.NS - 1) / f.NS * f.splits;
    const dim3 grid(groups > 1 ? (units + 7) / 8 * 8 * groups : units, 1, nz);      // see tile_of_block
    auto go = [&](auto ms_, auto ns_) {
        hipLaunchKernelGGL((k_bf16_gemm_few<decltype(ms_)::value, decltype(ns_)::value, EPI>), grid, dim3(256), 0, s, (const uint4*)X,
                           (const uint4*)W, K / 16, NBs, nb_off, N / 32, f.splits, n_ptr, B, part, (int64_t)Mpad * N, N, ep, zb);
    };
    auto go_ns = [&](auto ms_) {
        if (f.NS == 4) go(ms_, std::integral_constant<int, 4>{});
        else if (f.NS == 3) go(ms_, std::integral_constant<int, 3>{});
        else if (f.NS == 2) go(ms_, std::integral_constant<int, 2>{});
        else go(ms_, std::integral_constant<int, 1>{});
    };
    if (rows <= 32) go_ns(std::integral_constant<int, 1>{});
    else if (rows <= 64) go_ns(std::integral_constant<int, 2>{});
    else if (rows <= 96) go_ns(std::integral_constant<int, 3>{});
    else go_ns(std::integral_constant<int, 4>{});
    finish_slices<EPI>(b, N, f.splits, n_ptr, B, ep, s, tail);
    if (tail.from_out) *tail.from_out = 0;
}

// Several layers in one launch (K/V of skipped layers): the kernel whose waves stream alone, the tile kernels, or the
// weight-streaming one.  They add K up in different orders, so that this choice decides the bits; which tile does not,
// and such a launch is never sliced.
enum class Fill { stream, few, tiles };
static Fill fill_kernel(int N, int K, int rows, int nz) {
    const int64_t weights = (int64_t)N * K * nz;
    const bool large = weights >= ((int64_t)16 << 20);       // 32 MiB; two layers of 4 MiB 17.1 us on the streaming kernel, 17.6 on few
    if (N % 128 != 0 || K % 128 != 0) return rows > 64 || large ? Fill::few : Fill::stream;
    const int wide = N % 256 == 0 ? N / 256 * nz : 0, narrow = N / 128 * nz;       // column tiles
    if (rows <= 128) {
        // Tiles of 256 columns read X once per 256 columns, if they fill their rounds (seven layers of the 7B shape, 64 rows
        // 95 us and 99 on few), and with more than 96 rows so do tiles of 128 (three layers of the 7B shape, 128 rows 68.9 / 72.7,
        // sixteen of 1 MiB 41.1 / 43.0); elsewhere few (five layers of the 7B shape, 62 %, 64 rows 93 / 76, 128 rows 117.8 / 113.7, 60
        // of 128 leaving 97.8 / 86.0; ten of the 70B shape, 62 %, 113.0 / 117.2 with all 128 rows leaving, 94.2 / 91.5 with 60)
        const bool filled = rounds_filled(wide) >= 0.8f || (rows > 96 && wide < 200 && rounds_filled(narrow) >= 0.75f);
        // Few workgroups and few rows: one per tile-row on the streaming kernel, one round of them, is the shorter start up to 96 MiB
        // of weights, 64 up to 16 rows where they are more than 128.  Streaming / few: eight layers of 4 MiB (256 tile-rows) 1 row 14.2 /
        // 15.9 us, 32 rows 17.0 / 18.9; two of 16 MiB (128) 16.9 / 19.1 and 18.8 / 20.9, four (256) 20.9 / 20.2 and 24.1 / 25.0; two of
        // the 70B shape (128) 27.1 / 28.3 and 30.8 / 32.2, three 32.0 / 29.9 and 36.4 / 37.0; ten of 4 MiB 18.7 / 17.5 and 22.6 / 21.9
        const int tile_rows = N / 32 * nz;
        const bool short_start = rows <= 32 && tile_rows <= 256 && weights < ((int64_t)(rows <= 16 && tile_rows > 128 ? 32 : 48) << 20);
        if ((rows > 64 || large) && !filled && !short_start) return Fill::few;
        // The whole fill, streaming / tile kernel: up to 64 rows the tile kernel needs the 256-column tiles of all layers to fill
        // the chip, up to 32 also well filled rounds of workgroups: seven layers of the 7B shape (224 tiles) 1 row 90 / 79
        // us, 40 rows 144 / 94; 40 layers of the 70B shape (320) 1 row 240 / 274
        if (rows <= 64 && (wide < 200 || (rows <= 32 && rounds_filled(wide) < 0.75f))) return Fill::stream;
    }
    // more than 128 rows: always the tiles, so that a range gives the same bits in one launch or several.  (Two row groups of 128 on
    // few: 256 rows, two layers of the 70B shape 109 / 59 us, but eight, at 129 rows, 106 / 132.)
    return Fill::tiles;
}

// A product on the kernel whose waves stream alone (few_rows) or on the 256-row tile kernels, 128, 192 or 256 columns
// wide, K sliced so that about one workgroup per CU runs; returns false where the weight-streaming kernel is the better
// choice (at most 64 rows).  nz > 1 layers in one launch: the kernel that a launch of nz_as of them would take.
template <int EPI>
static bool gemm_tiled(const ee_batch* b, const void* X, const void* W, int N, int K, int NBs, int nb_off,
                     const int32_t* n_ptr, int B, const EpiArgs& ep, hipStream_t s, const ZBatch& zb = ZBatch{},
                     int nz = 1, const SliceTail& tail = SliceTail{}, int nz_as = 1) {
    const int rows = b->n_entries > 0 ? b->n_entries : B;    // in a context pass what the call has, not what the batch could hold
    const Fill fill_as = nz > 1 ? fill_kernel(N, K, rows, nz_as) : Fill::tiles;
    if (nz > 1 ? fill_as == Fill::few : few_rows<EPI>(N, K, rows, B)) {
        launch_few<EPI>(b, X, W, N, K, NBs, nb_off, n_ptr, B, rows, ep, s, zb, nz, tail);
        return true;
    }
    if (N % 128 != 0 || K % 128 != 0 || fill_as == Fill::stream) return false;
    int row_groups = (rows + 255) / 256;
    int Mpad = (B + 31) / 32 * 32;
    int KS = K / 32;
    auto launch_cols = [&]() {
        const int n_tiles = (N / 32 + 5) / 6;
        const dim3 grid(row_groups > 1 ? (n_tiles + 7) / 8 * 8 * row_groups : n_tiles, 1, 1);      // see tile_of_block
        hipLaunchKernelGGL((k_bf16_gemm_cols<EPI>), grid, dim3(512), 0, s, (const uint4*)X, (const uint4*)W, K / 16, NBs, nb_off,
                           N / 32, n_tiles, n_ptr, B, ep, zb);
        if (tail.splits_out) *tail.splits_out = 1;
        if (tail.from_out) *tail.from_out = 0;
        return true;
    };
    // or when K is long enough that a deeper K slicing costs little
    // (long K: with more than 128 rows the 256-column tile's halved activation traffic outweighs its
    // doubled K-slice planes; up to 128 rows the 128-column tile is 2-8 % faster on the down projection)
    bool wide = wide_tiles(N, row_groups, nz) || (N % 256 == 0 && EPI == EPI_RESID && K >= 2 * N && rows > 128);
    // K slices of a narrow product when the launch is left to itself: about one workgroup per CU
    auto slices_for = [&](int tiles) {
        int sp = (256 + tiles / 2) / tiles;
        // rounding up may push the launch past one round of 256 workgroups (96 column tiles x 3 slices):
        // one slice fewer then runs in a single round with longer slices and one plane less
        while (sp > 1 && tiles * sp > 256 && tiles * (sp - 1) >= 176) --sp;
        return sp;
    };
    auto fit_slices = [&](int sp) {
        while (sp > 1 && KS / sp < 16) --sp;               // every slice keeps at least 16 K steps (> 4)
        while (sp > 1 && (size_t)sp * Mpad * N * sizeof(float) > b->W.gemm_part_bytes) --sp;
        return sp;
    };
    const bool sliceable = (EPI == EPI_STORE || EPI == EPI_RESID) && nz == 1;
    int splits = 0;                                        // 0: not decided yet
    if (!wide && N % 256 == 0 && row_groups >= 2 && nz == 1) {
        // several row groups (context pass, batches above 256): the products are bound by the MFMAs and by
        // what a CU can pull from L2, and the 256-column tile moves a quarter less per MFMA issued
        const int ww = (N / 256) * row_groups, wn = (N / 128) * row_groups;
        if (sliceable && ww <= 256) {
            // a product that may be K-sliced: the 256-column tile with as many slices (at most 4) as keep
            // it inside one round of workgroups, against the 128-column tile with the slices it would get
            // below; ties go to the 256-column tile unless it needs 4 planes for it.  (70B shape, context
            // pass, per launch with the kernel that adds the planes: QKV at 512 entries 134 -> 104 us, at
            // 1024 entries 219 -> 198 us; O projection at 768 entries 158 -> 124 us, at 1024 168 -> 148 us.)
            const int s_w = fit_slices(std::min(4, 256 / ww));
            const int s_n = fit_slices(wn < 200 ? slices_for(wn) : 1);
            const float f_w = rounds_filled(ww * s_w), f_n = rounds_filled(wn * s_n);
            wide = f_w > f_n || (f_w == f_n && s_w < 4);
            splits = wide ? s_w : s_n;
        } else {
            wide = rounds_filled(ww) >= rounds_filled(wn);
        }
    }
    if constexpr (EPI == EPI_SWIGLU) if (row_groups == 1 && nz == 1) {
        // one row group (decode; with several the product is MFMA bound and the rule above stands).
        // Tile width for the widest product: 256, 192 or 128 columns, whichever makes the column tiles cost
        // the fewest rounds of 256 workgroups times the tile's width (what a round costs a CU in operand
        // traffic); ties go to the wider tile, which re-reads the activations less often.  (224 columns
        // were measured too, for the 70B shape's 1792 tile-rows = 256 x 7: within 2 % of 256 columns.)
        const int NB = N / 32;
        int nt = 4, best = 1 << 30;
        for (int t = 8; t >= 4; t -= 2) {
            if (t == 8 && N % 256 != 0) continue;
            const int wgs = (NB + t - 1) / t * row_groups * nz, cost = (wgs + 255) / 256 * t;
            if (cost < best) { best = cost; nt = t; }
        }
        if (nt == 6) return launch_cols();
        wide = nt == 8;
    }
    int n_tiles = wide ? N / 256 : N / 128;
    if (splits == 0) splits = sliceable && n_tiles * row_groups < 200 ? fit_slices(slices_for(n_tiles * row_groups)) : 1;
    if (nz == 1 && rows <= 256 && n_tiles * splits <= (rows > 160 ? 128 : 112) && (int64_t)N * K >= ((int64_t)2 << 20)) {
        // half of the CUs would idle: two row groups of 128 (2048-wide model, 192 rows: q|k|v 20.2 us in 96 workgroups, 18.0
        // here, O 22.7 / 19.8, gate/up 30.3 / 27.2; with 172 workgroups the tiles stay: gate/up of the 7B shape 54.8 / 85).
        // Little more than one group's rows: head of 16000 logits, 8192 wide (125 workgroups), 129 rows 107 / 113, 160 108 / 112, 180
        // 113.0 / 112.3, 256 128 / 105; of 14080 (110) 129 rows 107.0 / 106.8.
        launch_few<EPI>(b, X, W, N, K, NBs, nb_off, n_ptr, B, rows, ep, s, zb, nz, tail);
        return true;
    }
    if (tail.from_out) *tail.from_out = 0;
    // row groups that have rows: known in a context pass; in a decode step the rows that have left may leave one
    const int live_groups = (b->n_entries + 255) / 256;
    if (EPI == EPI_STORE && tail.defer_most > 0 && tail.from_out && wide && splits == 1 && nz == 1 && live_groups > 1 &&
        32 % live_groups == 0) {
        // More tiles than fit whole rounds of 256 workgroups: the column tiles that do run unsliced, the rest in
        // a second launch, K-sliced so that it fills one short round (QKV of 1999 entries at the 70B shape: 320
        // tiles, two rounds 360 us; 256 tiles 215 us and 64 in four slices 62, with 14 more where they are added).
        // Only where the row groups of whole column tiles fill an XCD's 32 CUs (32 % live_groups): tile_of_block
        // keeps a column tile on one XCD, so with seven groups 36 column tiles are 35 workgroups on some XCDs and
        // 28 on others, two rounds again (1600 entries: 345 + 39 us against 298 + 31 unsplit; 7B shape, 1600
        // entries 220 against 183, 3072 364 against 296).
        // By the batch's capacity instead of the call's entries, 64 entries in a batch of 2048 (7B shape) took two
        // launches for 48 tiles: 79 us instead of 52.
        const int full = n_tiles * live_groups / 256 * 256 / live_groups, rest = n_tiles - full;
        const int N2 = rest * 256;
        int sp = full > 0 && rest > 0 ? std::min({4, 256 / (rest * live_groups), KS / 16}) : 1;
        while (sp > 1 && (size_t)sp * Mpad * N2 * sizeof(float) > b->W.gemm_part_bytes) --sp;
        if (sp > 1) {
            hipLaunchKernelGGL((k_bf16_gemm_dma8<EPI>), dim3((full + 7) / 8 * 8 * row_groups), dim3(512), 0, s, (const uint4*)X,
                               (const uint4*)W, K / 16, NBs, nb_off, full, 1, n_ptr, B, (float*)nullptr, (int64_t)0, 0, ep, zb);
            hipLaunchKernelGGL((k_bf16_gemm_dma8<EPI>), dim3((rest * sp + 7) / 8 * 8 * row_groups), dim3(512), 0, s, (const uint4*)X,
                               (const uint4*)W, K / 16, NBs, nb_off + full * 8, rest, sp, n_ptr, B, b->wsp<float>(b->W.gemm_part),
                               (int64_t)Mpad * N2, N2, ep, zb);
            *tail.splits_out = sp;
            *tail.from_out = full * 256;
            return true;
        }
    }
    if (EPI != EPI_RESID && splits == 1 && nz == 1 && row_groups > 1) {
        // Several row groups: 192 columns where they cost fewer rounds of workgroups times a round's length.  A round of
        // 256 / 192 / 128 columns takes 1 / 0.82 / 0.73, the last one down to 0.85 of that when it is nearly empty.  (192: gate/up of 400
        // to 2048 rows 0.79 to 0.83, q|k|v of the 70B shape 0.88.  128: 0.59 to 0.63 against full groups of 256 columns, which a choice
        // between 192 and 128 has not hung on.)  Gate/up 256 / 192 columns: 7B shape 400 rows 89 / 76 us (172 / 230
        // workgroups), 768 entries 176 / 146, 1024 182 / 157, 1536 271 / 228, 2048 282 / 300 (688 / 920, not taken); 34B 512 entries 345 / 303, 1024
        // 543 / 588 (not taken); 70B 512 377 / 427 (not taken).  q|k|v: 7B shape 1536 entries 182 / 158, 2048 186 / 179, 70B 1024 174 / 156,
        // 2048 355 / 318.
        auto cost = [](int wgs, float round) {
            const int full = (wgs - 1) / 256;
            return round * ((float)full + 0.85f + 0.15f * (float)(wgs - 256 * full) / 256.f);
        };
        if (cost((N / 32 + 5) / 6 * row_groups, 0.82f) < cost(n_tiles * row_groups, wide ? 1.0f : 0.73f)) return launch_cols();
    }
    dim3 grid(n_tiles * splits, row_groups, nz);
    if (row_groups > 1) grid = dim3((n_tiles * splits + 7) / 8 * 8 * row_groups, 1, nz);   // see tile_of_block
    if (wide)
        hipLaunchKernelGGL((k_bf16_gemm_dma8<EPI>), grid, dim3(512), 0, s, (const uint4*)X, (const uint4*)W,
                           K / 16, NBs, nb_off, n_tiles, splits, n_ptr, B, b->wsp<float>(b->W.gemm_part),
                           (int64_t)Mpad * N, N, ep, zb);
    else
        hipLaunchKernelGGL((k_bf16_gemm_dma2<EPI>), grid, dim3(BIG_THREADS), 0, s, (const uint4*)X, (const uint4*)W,
                           K / 16, NBs, nb_off, n_tiles, splits, n_ptr, B, b->wsp<float>(b->W.gemm_part),
                           (int64_t)Mpad * N, N, ep, zb);
    finish_slices<EPI>(b, N, splits, n_ptr, B, ep, s, tail);
    return true;
}

// How the attention of a context pass is tiled: C 16-column blocks per wave (0: not tiled), entries per tile.
// Two blocks per wave read each K and V operand from LDS half as often, one block gives twice the
// workgroups: two where that still leaves two workgroups per CU (70B shape, 1999 entries, one machine: 275 us against
// 310 with one), one from one workgroup per CU on (256 entries, 1500 cached: layer 558 -> 539 us; 600 entries of
// four contexts: 1284 -> 1239 us).  Below that the kernel that splits a row's positions over its waves stays.
// What counts is the entries of the call, not the batch's capacity: 64 entries at positions from 1936 on take 41 us
// in a batch of 2048 (79 as four tiles of 16, 32 workgroups), 100 of two contexts of 3000 in a batch of 1024 61 (197).
// Speculative rounds keep it too: their runs are a few drafts long.
struct CtxTiles { int C = 0, tile_entries = 1, tiles = 0; };
static CtxTiles ctx_tiles(const ee_model_config& c, const ee_batch* b) {
    CtxTiles r;
    const int G = c.n_q_heads / c.n_kv_heads, E = 16 / G;
    if (b->n_entries == 0) return r;
    for (int C = 2; C >= 1; --C) {
        const int te = 4 * C * E, tiles = (b->n_entries + te - 1) / te;
        if (tiles * c.n_kv_heads < 256 * C || tiles * 4 * C > 65535) continue;
        r.C = C; r.tile_entries = te; r.tiles = tiles;
        break;
    }
    return r;
}

// Most workgroups per (row, kv head) of the decode attention (attn_shares).  Positions are shared only where a row may be worth
// the launch that merges them: room for 672 positions (attention and merge of 8 kv heads, 1 row of 500: layer 1 us
// longer shared, of 950: 3 us shorter), with 192 pairs 1024 (60 rows of 4 kv heads, 650: 78.5 us shared, 75.3 whole,
// 950: 84.1 and 81.1; 12 rows of 32, 650: 120.5 and 117.6).  The host knows the room, not the rows: short ones in a large cache
// pay for the merge launch too (4 rows of 40 to 200 positions of the 70B shape, attention 11.2 us, 12.7 with room for 3000 more).
static int attn_most(const ee_model_config& c, const ee_kv* kv, const ee_batch* b) {
    const int pairs = c.n_kv_heads * b->B;
    int most = pairs >= 512 || kv->max_cap < (pairs >= 192 ? 1024 : 672) ? 1 : std::min({16, (1024 + pairs - 1) / pairs, kv->max_cap / 256});
    while (most > 1 && (size_t)b->Mpad * c.n_kv_heads * most * 16 * ATTN_SHARE * 4 > b->W.attn_part_bytes) --most;
    return most;
}

// Whether rotation and append are part of the attention (k_bf16_attn_decode): in a decode step (with entries that name their
// cache row one may read what another appends), up to 768 (row, kv head) pairs.  Beyond, the workgroups' start is no longer hidden
// and costs more than the launch.  Layer, separate / together: 7B shape 8 rows (256 pairs) 103.7 / 101.0 us, 20 rows (640)
// 121.6 / 119.5, 40 (1280) 118.7 / 122.5, 512 1106 / 1141; 34B 128 rows (1024) 419 / 422; 2048-wide model 100 rows (400) 98.1 /
// 93.4; 576-wide model 20 rows (40) 43.1 / 41.0.
static bool append_in_attn(const ee_model_config& c, const ee_batch* b) { return b->kv_seq == nullptr && c.n_kv_heads * b->B <= 768; }

// the jobs that the kernel which normalises for a layer's q|k|v product leaves; elsewhere the append kernel does
static JobArgs attn_jobs(const ee_model_config& c, const ee_kv* kv, const ee_batch* b) {
    if (!append_in_attn(c, b)) return JobArgs{};
    return JobArgs{b->st<int32_t>(b->L.pos), kv->d_cap, kv->d_off, b->wsp<AttnJob>(b->W.attn_order), c.n_kv_heads, attn_most(c, kv, b)};
}

static bool begin_norm_fits(const ee_model* m) {
    return m->cfg.d_model <= 8 * NORM_THREADS && (uintptr_t)m->emb % 16 == 0;
}

int bf16_begin_step(const ee_model* m, const ee_kv* kv, ee_batch* b, hipStream_t s, bool* x_ready) {
    *x_ready = begin_norm_fits(m);
    if (!*x_ready) return launch_begin_step(m, b, s);
    const ee_batch_layout& L = b->L;
    TimedScope t(EE_K_EMBED, s);
    BeginArgs g{};
    g.tok = b->st<int32_t>(L.tok_in); g.n = b->B; g.V = m->cfg.vocab; g.emb = (const uint4*)m->emb; g.h = b->st<float>(L.h);
    g.active_idx = b->st<int32_t>(L.active_idx); g.n_active = b->st<int32_t>(L.n_active);
    g.n_exited = b->st<int32_t>(L.n_exited); g.out_layer = b->st<int32_t>(L.out_layer); g.status = b->st<int32_t>(L.status);
    hipLaunchKernelGGL(k_bf16_begin_norm<false>, dim3(entry_grid(b->B)), dim3(norm_threads(m->cfg.d_model, attn_jobs(m->cfg, kv, b))), 0, s, g, entry_near(b->B),
                       (const float*)m->layers[0].g_attn, m->cfg.rms_eps, m->cfg.d_model, b->wsp<uint4>(b->W.x), attn_jobs(m->cfg, kv, b));
    EE_LAUNCH_CHECK();
    return EE_OK;
}

int bf16_prefill_begin(const ee_model* m, const ee_kv* kv, ee_batch* b, const int32_t* tok, const int32_t* pos,
                       const int32_t* seq, int n, hipStream_t s, bool* x_ready) {
    *x_ready = begin_norm_fits(m);
    if (!*x_ready) return launch_prefill_begin(m, kv, b, tok, pos, seq, n, s);
    const ee_batch_layout& L = b->L;
    TimedScope t(EE_K_EMBED, s);
    BeginArgs g{};
    g.tok = tok; g.pos = pos; g.seq = seq; g.n = n; g.n_seq = kv->B; g.V = m->cfg.vocab; g.emb = (const uint4*)m->emb;
    g.h = b->st<float>(L.h); g.s_tok = b->st<int32_t>(L.tok_in); g.s_pos = b->st<int32_t>(L.pos);
    g.kv_seq = b->wsp<int32_t>(b->W.kv_seq); g.active_idx = b->st<int32_t>(L.active_idx);
    g.n_active = b->st<int32_t>(L.n_active); g.n_exited = b->st<int32_t>(L.n_exited); g.status = b->st<int32_t>(L.status);
    hipLaunchKernelGGL(k_bf16_begin_norm<true>, dim3(entry_grid(n)), dim3(norm_threads(m->cfg.d_model, JobArgs{})), 0, s, g, entry_near(n),
                       (const float*)m->layers[0].g_attn, m->cfg.rms_eps, m->cfg.d_model, b->wsp<uint4>(b->W.x), JobArgs{});
    EE_LAUNCH_CHECK();
    return EE_OK;
}

// x_ready: the operand matrix already holds RMSNorm(h; attention gain of this layer).
// tail_gain (with x_done): if the last product of the layer is finished from K-slice planes, that
// kernel also leaves RMSNorm(h; tail_gain) in the operand matrix and sets *x_done.
int bf16_layer_forward(const ee_model* m, int layer, ee_kv* kv, ee_batch* b, hipStream_t s, bool x_ready,
                       const float* tail_gain, bool* x_done) {
    const ee_model_config& c = m->cfg;
    const ee_layer_weights& w = m->layers[layer - 1];
    const ee_batch_layout& L = b->L;
    int B = b->B, d = c.d_model, hd = c.head_dim, qd = c.n_q_heads * hd, F = c.d_ffn;
    int qkv_n = (c.n_q_heads + 2 * c.n_kv_heads) * hd;
    const int32_t* idx = b->st<int32_t>(L.active_idx);
    const int32_t* n_ptr = b->st<int32_t>(L.n_active);
    float* h = b->st<float>(L.h);
    uint4* x = b->wsp<uint4>(b->W.x);
    float* qkv = b->wsp<float>(b->W.qkv);
    uint4* ao = b->wsp<uint4>(b->W.ao);
    bf16_t* act = b->wsp<bf16_t>(b->W.act);
    KvView view = make_view(m, kv, layer, b);
    const CtxTiles ctx = ctx_tiles(c, b);
    const int pairs = c.n_kv_heads * B, most = attn_most(c, kv, b);
    const JobArgs jobs = attn_jobs(c, kv, b);

    if (!x_ready) {
        TimedScope t(EE_K_NORM, s);
        hipLaunchKernelGGL(k_bf16_rmsnorm, dim3(entry_grid(B)), dim3(norm_threads(d, jobs)), 0, s, h, idx, n_ptr, B, entry_near(B), w.g_attn, c.rms_eps, d, x, ZBatch{}, jobs);
    }
    EpiArgs e1{};
    e1.out = qkv; e1.ldo = qkv_n; e1.idx = idx;
    int qkv_splits = 1, qkv_from = 0;
    const bool together = append_in_attn(c, b);
    {
        TimedScope t(EE_K_GEMM_QKV, s);
        SliceTail st;                  // K-slice planes of q|k|v are added up by the append kernel, or the attention, which takes all columns so
        st.defer_most = 1 << 30; st.splits_out = &qkv_splits; st.from_out = together ? nullptr : &qkv_from;
        if (!gemm_tiled<EPI_STORE>(b, x, w.w_qkv, qkv_n, d, qkv_n / 32, 0, n_ptr, B, e1, s, ZBatch{}, 1, st))
            gemm<1, EPI_STORE>(x, w.w_qkv, qkv_n, d, qkv_n / 32, 0, n_ptr, B, e1, s);
    }
    if (qkv_splits == 1) qkv_from = qkv_n;             // nothing is in planes
    if (!together) {
        TimedScope t(EE_K_ROPE_APPEND, s);
        // neighbouring entries share lines of the cache only where they are positions of one row (context pass)
        const int near = b->kv_seq != nullptr ? entry_near(B) : 1;
        hipLaunchKernelGGL(k_bf16_rope_append, dim3(near > 1 ? entry_grid(B) : B, rope_blocks(c.n_q_heads, c.n_kv_heads, B)), dim3(256), 0, s, qkv, qkv_n, c.n_q_heads, idx, n_ptr, B, near,
                           b->st<int32_t>(L.pos), m->d_rope, c.max_pos, view, b->wsp<bf16_t>(b->W.q_hi),
                           b->wsp<bf16_t>(b->W.q_lo), b->st<int32_t>(L.status), (int64_t)0,
                           ctx.C ? b->wsp<int32_t>(b->W.attn_order) : nullptr, ctx.C ? nullptr : b->wsp<AttnJob>(b->W.attn_order),
                           most, ctx.tile_entries, b->kv_seq == nullptr, qkv_splits, (int64_t)b->Mpad * (qkv_n - qkv_from), b->wsp<float>(b->W.gemm_part),
                           qkv_n - qkv_from, qkv_from);
    }
    {
        TimedScope t(EE_K_ATTENTION, s);
        // context pass: 16 / G entries per workgroup, which share the K/V stream where they sit in the same cache row
        const int G = c.n_q_heads / c.n_kv_heads;
        const bool pair = b->kv_seq != nullptr && pairs >= 512 && 2 * G <= 16;
        if (together) {
            const QkvIn in{qkv, qkv_n, b->wsp<float>(b->W.gemm_part), qkv_splits, (int64_t)b->Mpad * qkv_n, m->d_rope, c.max_pos,
                           b->st<int32_t>(L.status)};
            hipLaunchKernelGGL(k_bf16_attn_decode, dim3(c.n_kv_heads, B, most), dim3(256), 0, s, in, c.n_q_heads, n_ptr, B, view, ao, qd / 16,
                               most, b->wsp<float>(b->W.attn_part), b->wsp<AttnJob>(b->W.attn_order));
        } else if (ctx.C) {
            auto kern = ctx.C == 2 ? k_bf16_attn_ctx<2> : k_bf16_attn_ctx<1>;
            hipLaunchKernelGGL(kern, dim3(c.n_kv_heads, ctx.tiles * 4 * ctx.C), dim3(256), 0, s, b->wsp<bf16_t>(b->W.q_hi),
                               b->wsp<bf16_t>(b->W.q_lo), c.n_q_heads, idx, n_ptr, B, b->st<int32_t>(L.pos), view, ao,
                               qd / 16, b->wsp<int32_t>(b->W.attn_order));
        } else if (pair)
            hipLaunchKernelGGL((k_bf16_attn<true, 4>), dim3(c.n_kv_heads, (B + 16 / G - 1) / (16 / G), 1), dim3(256), 0, s, b->wsp<bf16_t>(b->W.q_hi),
                               b->wsp<bf16_t>(b->W.q_lo), c.n_q_heads, idx, n_ptr, B, b->st<int32_t>(L.pos), view, ao,
                               qd / 16, 1, b->wsp<float>(b->W.attn_part), b->wsp<AttnJob>(b->W.attn_order));
        else
        {
            // Room for at most 8 groups of 32 positions per row and many rows: a wave takes a whole row, so that nothing is merged and eight
            // rows start on a CU at a time.  Layer, four waves / one: 7B shape 300 rows of 20 to 30 positions 330 / 287 us, of 125
            // to 250 439 / 436, 40 rows of 60 117.5 / 113.5; 34B 400 rows of 60 746 / 729; longer rows 0.5 to 2 % the other way (two
            // waves lie between).
            const bool one = pairs > 768 && kv->max_cap <= 256;
            auto kern = one ? k_bf16_attn<false, 1> : k_bf16_attn<false, 4>;
            hipLaunchKernelGGL(kern, dim3(c.n_kv_heads, B, most), dim3(one ? 64 : 256), 0, s, b->wsp<bf16_t>(b->W.q_hi),
                               b->wsp<bf16_t>(b->W.q_lo), c.n_q_heads, idx, n_ptr, B, b->st<int32_t>(L.pos), view, ao,
                               qd / 16, most, b->wsp<float>(b->W.attn_part), b->wsp<AttnJob>(b->W.attn_order));
        }
        if (most > 1 && ctx.C == 0)
            hipLaunchKernelGGL(k_bf16_attn_merge, dim3(c.n_kv_heads, B), dim3(256), 0, s, b->wsp<float>(b->W.attn_part),
                               c.n_q_heads, c.n_kv_heads, most, b->wsp<AttnJob>(b->W.attn_order), n_ptr, B, ao, qd / 16);
    }
    EpiArgs e2{};
    e2.out = h; e2.ldo = d; e2.idx = idx;
    bool ffn_x_done = false;
    {
        TimedScope t(EE_K_GEMM_O, s);
        SliceTail st;                  // the finish of a sliced product also normalises for the FFN
        st.norm_gain = w.g_ffn; st.eps = c.rms_eps; st.norm_out = x; st.norm_done = &ffn_x_done;
        if (!gemm_tiled<EPI_RESID>(b, ao, w.w_o, d, qd, d / 32, 0, n_ptr, B, e2, s, ZBatch{}, 1, st))
            gemm<1, EPI_RESID>(ao, w.w_o, d, qd, d / 32, 0, n_ptr, B, e2, s);
    }
    if (!ffn_x_done) {
        TimedScope t(EE_K_NORM, s);
        hipLaunchKernelGGL(k_bf16_rmsnorm, dim3(entry_grid(B)), dim3(norm_threads(d, JobArgs{})), 0, s, h, idx, n_ptr, B, entry_near(B), w.g_ffn, c.rms_eps, d, x, ZBatch{}, JobArgs{});
    }
    EpiArgs e3{};
    e3.act = act; e3.KB_act = F / 16; e3.idx = idx;
    {
        TimedScope t(EE_K_GEMM_GATE_UP, s);
        if (!gemm_tiled<EPI_SWIGLU>(b, x, w.w_gate_up, 2 * F, d, 2 * F / 32, 0, n_ptr, B, e3, s))
            gemm<2, EPI_SWIGLU>(x, w.w_gate_up, 2 * F, d, 2 * F / 32, 0, n_ptr, B, e3, s);
    }
    {
        TimedScope t(EE_K_GEMM_DOWN, s);
        SliceTail st;
        st.norm_gain = tail_gain; st.eps = c.rms_eps; st.norm_out = x; st.norm_done = x_done;
        if (tail_gain) st.jobs = jobs;
        if (!gemm_tiled<EPI_RESID>(b, act, w.w_down, d, F, d / 32, 0, n_ptr, B, e2, s, ZBatch{}, 1, st))
            gemm<1, EPI_RESID>(act, w.w_down, d, F, d / 32, 0, n_ptr, B, e2, s);
    }
    EE_LAUNCH_CHECK();
    return EE_OK;
}

int bf16_exit_head(const ee_model* m, int e, float th, int force, ee_batch* b, float* dbg, hipStream_t s,
                   bool x_ready) {
    const ee_model_config& c = m->cfg;
    const ee_batch_layout& L = b->L;
    int B = b->B, d = c.d_model, V = c.vocab;
    const int32_t* idx = b->st<int32_t>(L.active_idx);
    const int32_t* n_ptr = b->st<int32_t>(L.n_active);
    uint4* x = b->wsp<uint4>(b->W.x);
    if (!x_ready) {
        TimedScope t(EE_K_NORM, s);
        hipLaunchKernelGGL(k_bf16_rmsnorm, dim3(entry_grid(B)), dim3(norm_threads(d, JobArgs{})), 0, s, b->st<float>(L.h), idx, n_ptr, B, entry_near(B),
                           m->exits[e].gain, c.rms_eps, d, x, ZBatch{}, JobArgs{});
    }
    EpiArgs ep{};
    ep.idx = idx; ep.row_scale = b->st<float>(L.row_scale);
    ep.part_max = b->wsp<float>(b->W.part_max); ep.part_sum = b->wsp<float>(b->W.part_sum);
    ep.part_arg = b->wsp<int32_t>(b->W.part_arg); ep.n_part = V / 32;
    ep.dbg_logits = dbg; ep.ldo = V;
    {
        TimedScope t(EE_K_EXIT_GEMM, s);
        if (!gemm_tiled<EPI_EXIT>(b, x, m->exits[e].w, V, d, V / 32, 0, n_ptr, B, ep, s))
            gemm<1, EPI_EXIT>(x, m->exits[e].w, V, d, V / 32, 0, n_ptr, B, ep, s);
    }
    EE_LAUNCH_CHECK();
    return launch_exit_decide(b, V / 32, th, force, s);
}

// layers_as: the keys and values are those of fills of so many layers, bit for bit
static int fill_kv(const ee_model* m, int from_excl, int to_incl, ee_kv* kv, ee_batch* b, hipStream_t s, const int32_t* idx,
                   const int32_t* n_ptr, int layers_as) {
    const ee_model_config& c = m->cfg;
    const ee_batch_layout& L = b->L;
    int B = b->B, d = c.d_model, hd = c.head_dim;
    int kv_n = 2 * c.n_kv_heads * hd;
    int nl = to_incl - from_excl;                       // layers to fill: from_excl + 1 .. to_incl
    if (idx == nullptr) { idx = b->st<int32_t>(L.exited_idx); n_ptr = b->st<int32_t>(L.n_exited); }
    uint4* x = b->wsp<uint4>(b->W.fill_x);              // [layer][Mpad][d] normalised exit rows, tile order
    float* kvb = b->wsp<float>(b->W.fill_kv);           // [layer][Mpad][2 H_kv hd]
    TimedScope t(EE_K_FILL_KV, s);
    // all layers of the range in three launches (blockIdx.z = layer): the layers differ only in
    // their norm gain and their W_k / W_v
    ZBatch zb{};
    zb.w_tab = m->d_wqkv_tab; zb.g_tab = m->d_gattn_tab; zb.z0 = from_excl;
    zb.x_stride = (int64_t)b->Mpad * d / 8; zb.out_stride = (int64_t)b->Mpad * kv_n;
    hipLaunchKernelGGL(k_bf16_rmsnorm, dim3(entry_grid(B), 1, nl), dim3(norm_threads(d, JobArgs{})), 0, s, b->st<float>(L.h), idx, n_ptr, B, entry_near(B),
                       (const float*)nullptr, c.rms_eps, d, x, zb, JobArgs{});
    // key and value rows are the last 2*H_kv*hd rows of W_qkv: tile-rows H_q*hd/32 onwards
    EpiArgs ep{};
    ep.out = kvb; ep.ldo = kv_n; ep.idx = idx;
    int NBs = (c.n_q_heads + 2 * c.n_kv_heads) * hd / 32, nb_off = c.n_q_heads * hd / 32;
    int splits = 1;
    // one layer's K-slice planes, of all columns, are added up by the append kernel, up to eight of them (70B shape, added there / in a
    // launch before it: 129 rows, sixteen planes, 35.7 / 34.3 us; 300 rows, eight, 38.7 / 40.0)
    SliceTail st;
    st.defer_most = nl == 1 ? 8 : 0; st.splits_out = &splits;
    if (!gemm_tiled<EPI_STORE>(b, x, nullptr, kv_n, d, NBs, nb_off, n_ptr, B, ep, s, zb, nl, st, layers_as))
        gemm<1, EPI_STORE>(x, nullptr, kv_n, d, NBs, nb_off, n_ptr, B, ep, s, zb, nl);
    const int near = b->kv_seq != nullptr ? entry_near(B) : 1;
    hipLaunchKernelGGL(k_bf16_rope_append, dim3(near > 1 ? entry_grid(B) : B, rope_blocks(0, c.n_kv_heads, B * nl), nl), dim3(256), 0, s, kvb, kv_n, 0, idx, n_ptr, B, near,
                       b->st<int32_t>(L.pos), m->d_rope, c.max_pos, make_view(m, kv, from_excl + 1, b),
                       (bf16_t*)nullptr, (bf16_t*)nullptr, b->st<int32_t>(L.status), zb.out_stride,
                       (int32_t*)nullptr, (AttnJob*)nullptr, 1, 1, false, splits, (int64_t)b->Mpad * kv_n, b->wsp<float>(b->W.gemm_part), kv_n,
                       splits == 1 ? kv_n : 0);
    EE_LAUNCH_CHECK();
    return EE_OK;
}

int bf16_fill_kv(const ee_model* m, int from_excl, int to_incl, ee_kv* kv, ee_batch* b, hipStream_t s, const int32_t* idx,
                 const int32_t* n_ptr) {
    return fill_kv(m, from_excl, to_incl, kv, b, s, idx, n_ptr, to_incl - from_excl);
}

int bf16_fill_ranges(const ee_model* m, const int32_t* bounds, int n, bool singles_apart, ee_kv* kv, ee_batch* b, hipStream_t s,
                     const int32_t* idx, const int32_t* n_ptr) {
    const ee_model_config& c = m->cfg;
    auto kernel = [&](int layers) { return fill_kernel(2 * c.n_kv_heads * c.head_dim, c.d_model, b->B, layers); };
    int rc = EE_OK;
    for (int i = 0, j; i < n && rc == EE_OK; i = j) {
        int layers = bounds[i + 1] - bounds[i];              // of a range of several whose kernel the launch takes
        for (j = i + 1; j < n && !(layers == 1 && singles_apart); ++j) {
            const int next = bounds[j + 1] - bounds[j];
            if (next == 1 ? singles_apart : layers > 1 && kernel(next) != kernel(layers)) break;
            if (layers == 1) layers = next;
        }
        rc = fill_kv(m, bounds[i], bounds[j], kv, b, s, idx, n_ptr, layers > 1 ? layers : bounds[j] - bounds[i]);
    }
    return rc;
}
