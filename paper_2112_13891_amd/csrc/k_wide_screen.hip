// k_wide_screen.hip -- the FP32 step for wide rows (padded D = 64, 128, 256) by
// a screen of the pairs on the matrix cores (gfx950).
//
// The update needs 3 D FP32 operations a pair, and in wide rows nearly all of
// them go to pairs whose weight is exactly zero: distances grow with D, and a
// Gaussian weight is +0 in FP32 from q = |x - s|^2 = 150 packed units on (the
// flat window ends at h^2).  So an iteration is two kernels:
//   1. wide_mask_kernel: a bit per seed and point, set unless a lower bound of
//      q rules the pair out.  The bound comes from one bf16 product per pair on
//      the matrix cores, 2 s.x with s and x relative to the first row:
//          q >= (1 - 2^-7 - 2^-10) (|s|^2 + |x|^2) - (2 s.x)_bf16 .
//      A bf16 factor is within 2^-8 of its value (8 significant bits), so 2 s.x
//      is off by at most (2^-7 + 2^-16) 2 |s||x| <= (2^-7 + 2^-16) (|s|^2 + |x|^2):
//      coordinates at 1 + 2^-8, which round down to 1, take nearly all of it.
//      The FP32 sums (256 products, each norm's chain of 128) are off by less
//      than 2^-14 of |s|^2 + |x|^2; the further 2^-10 covers them 16 times.
//   2. wide_eval_kernel: a workgroup per seed lists its set bits in LDS and
//      evaluates those pairs as the all-pairs form does, in FP32 differences;
//      then the update, the shift and the convergence test, and the seed's
//      operand for the next iteration.
// A pair left out has weight exactly +0 (or lies outside the flat window), or,
// from the second update on, a weight below 2^-33 / n of the seed's last W (a
// mean-shift step never lowers the density), in all below 2^-33 of it where an
// FP32 sum rounds at 2^-25.  Rows that are not finite are never left out.
//
// The screen's products are cheap (50,001 x 500 x 128: 6.4 GFLOP); what bounds
// the form is the rows that the seeds read again, D * 4 bytes a kept pair from
// L2: 625,000 kept pairs of 512 bytes an update there, 10.7 TB/s.
// 50,001 points, 500 seeds, 40 clusters, D = 128: an update 830 us over all
// pairs (k_step_wide.hip), 17.5 + 30 us here; two updates with their set-up 1,720
// -> 133 us.  With every pair within reach three updates cost 2.4 -> 1.5 ms there
// and 9.0 -> 3.2 ms at D = 256; at D = 64 0.69 -> 0.83 ms, since every seed reads
// all rows (6.4 GB an update, 24 TB/s) where the all-pairs form reads a row once
// for 64 seeds.

#include "step_common.h"

namespace fms {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr float kNormShare = 1.0f - 1.0f / 128.0f - 1.0f / 1024.0f;
constexpr float kNever = 3e38f;          // no finite product reaches it
constexpr float kZeroQ = 160.0f;         // exp2(-q) == +0 for q >= 150
constexpr float kDropped = 34.0f;        // log2 of W over all that is left out, and 1 of margin
constexpr float kFlatMargin = 1.001f;
constexpr int kEvalWaves = 8;
constexpr int kEvalPoints = 64 * kEvalWaves * 32;   // points listed at once: 32 bits a thread
// A lane adds this many pairs in a row before its sums are added up across
// lanes.  Where points repeat, additions of equal terms all round the same way:
// one update of seeds that see 120,001 points of seven values (D = 128) was off
// by 1.3e-5 h, and is by 1.1e-7 h now (50,001 x 500 pairs, all near, three
// updates: D = 128 1,374 -> 1,403 us, D = 64 and 256 within 1 %).
constexpr int kEvalRun = 32;

// Points as operands: per 32 points and block of 16 coordinates, lane l holds
// point l % 32, coordinates 8 (l / 32) ... + 7.  One wave per 32 points.  With
// Xp, the rows (of d coordinates) are packed on the way.
template <int D>
__global__ __launch_bounds__(kThreads) void wide_points_kernel(const float* __restrict__ X, int n, int d, float scale,
                                                               int tiles, float* __restrict__ Xp,
                                                               bf16x8* __restrict__ pf, float* __restrict__ nx) {
    // differences of packed coordinates, rounded as the exact distances have
    // them: fused with the scaling, a column of equal large values (1.6e9, h = 1)
    // put points and seeds 2 ulp apart in the screen alone
#pragma clang fp contract(off)
    constexpr int KB = D / 16;
    const int t = blockIdx.x * kWaves + (threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5;
    if (t >= tiles) return;
    const int p = t * 32 + (lane & 31);
    const float* row = X + (long long)(p < n ? p : 0) * d;
    float nn = 0.0f;
#pragma unroll 4
    for (int kb = 0; kb < KB; ++kb) {
        const int k0 = kb * 16 + half * 8;
        float x[8], r[8];
#pragma unroll
        for (int q = 0; q < 8; q += 4) {
            if (k0 + q + 4 <= d) {   // wide loads
#pragma unroll
                for (int e = q; e < q + 4; ++e) {
                    x[e] = row[k0 + e] * scale;
                    r[e] = X[k0 + e] * scale;
                }
            } else {
#pragma unroll
                for (int e = q; e < q + 4; ++e) {
                    x[e] = k0 + e < d ? row[k0 + e] * scale : 0.0f;
                    r[e] = k0 + e < d ? X[k0 + e] * scale : 0.0f;
                }
            }
        }
        if (Xp && p < n) {
            float4* out = reinterpret_cast<float4*>(Xp + (long long)p * D + k0);
            out[0] = make_float4(x[0], x[1], x[2], x[3]);
            out[1] = make_float4(x[4], x[5], x[6], x[7]);
        }
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float u = x[e] - r[e];
            nn = fmaf(u, u, nn);
            v[e] = (__bf16)u;
        }
        pf[((long long)t * KB + kb) * 64 + lane] = p < n ? v : bf16x8{};
    }
    nn += __shfl_xor(nn, 32);
    // a row that is not finite stays in every seed's list; rows past the last in none
    if (half == 0) nx[p] = p < n ? (nn < 1e37f ? kNormShare * nn : __builtin_nanf("")) : kNever;
}

// The reach of a seed in q.
__device__ __forceinline__ float seed_reach(int kern, float h2, float W, int n) {
    if (kern != MS_KERNEL_GAUSSIAN) return h2 * kFlatMargin;
    if (!(W > 0.0f)) return kZeroQ;   // first update
    return fminf(kZeroQ, fmaxf(kDropped + __builtin_amdgcn_logf((float)n) - __builtin_amdgcn_logf(W), 1.0f));
}

// One seed's operand and share of the test, by one wave: lane l holds
// coordinates l, l + 64, ... in u (original units).
template <int D>
__device__ __forceinline__ void store_seed(int j, const float (&u)[D / 64], bool active, float reach, float scale,
                                           const float* __restrict__ Xp, __bf16* sf, float* crow) {
#pragma clang fp contract(off)   // as in wide_points_kernel
    constexpr int KB = D / 16;
    const int lane = threadIdx.x & 63;
    float nn = 0.0f;
#pragma unroll
    for (int i = 0; i < D / 64; ++i) {
        const int k = lane + 64 * i;
        const float v = u[i] * scale - Xp[k];
        nn = fmaf(v, v, nn);
        sf[((((long long)(j >> 5) * KB + (k >> 4)) * 64) + (j & 31) + 32 * ((k >> 3) & 1)) * 8 + (k & 7)] =
            (__bf16)(2.0f * v);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) nn += __shfl_xor(nn, off);
    if (lane == 0) crow[j] = active ? (nn < 1e37f ? kNormShare * nn - reach : __builtin_nanf("")) : kNever;
}

// Seeds of a step call in, a wave each: as launch_seed_init_from_array, and
// their operands (slots past the last one never match).
template <int D>
__global__ __launch_bounds__(kThreads) void wide_load_kernel(const float* __restrict__ seeds,
                                                             const uint8_t* __restrict__ conv_in, int d, int m,
                                                             int slots, int kern, float h2, float scale, int n,
                                                             const float* __restrict__ Xp, float* S, int32_t* act0,
                                                             uint8_t* status, int32_t* iters, float* shift2, Ctl* ctl,
                                                             __bf16* sf, float* crow) {
    const int j = blockIdx.x * kWaves + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (j >= slots) return;
    float u[D / 64];
#pragma unroll
    for (int i = 0; i < D / 64; ++i) {
        const int k = lane + 64 * i;
        u[i] = j < m && k < d ? seeds[(long long)j * d + k] : 0.0f;
        if (j < m) S[(long long)j * D + k] = u[i];
    }
    const uint8_t st = j < m ? conv_in[j] : (uint8_t)ST_CONVERGED;
    store_seed<D>(j, u, st == ST_ACTIVE, seed_reach(kern, h2, 0.0f, n), scale, Xp, sf, crow);
    if (lane == 0 && j < m) {
        status[j] = st;
        iters[j] = 0;
        shift2[j] = __builtin_nanf("");
        if (st == ST_ACTIVE) act0[atomicAdd(&ctl->count[0], 1)] = j;
    }
}

// The seeds of a batch before its first update, a wave each; slots past the
// last one never match.
template <int D>
__global__ __launch_bounds__(kThreads) void wide_seeds_kernel(const float* __restrict__ S,
                                                              const uint8_t* __restrict__ status, int m, int slots,
                                                              int kern, float h2, float scale, int n,
                                                              const float* __restrict__ Xp, __bf16* sf, float* crow) {
    const int j = blockIdx.x * kWaves + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (j >= slots) return;
    float u[D / 64];
#pragma unroll
    for (int i = 0; i < D / 64; ++i) u[i] = j < m ? S[(long long)j * D + lane + 64 * i] : 0.0f;
    store_seed<D>(j, u, j < m && status[j] == ST_ACTIVE, seed_reach(kern, h2, 0.0f, n), scale, Xp, sf, crow);
}

// The point of a bit: bits 16 h + r are register r of half h of the product.
__device__ __forceinline__ int bit_point(int b) { return (b & 3) | ((b & 12) << 1) | ((b >> 2) & 4); }

// A wave takes 64 points (a word of every seed's bits) past the seed tiles of
// its share: rows of the product are points, columns seeds, so that a lane
// gathers 32 bits of one seed.
template <int D>
__global__ __launch_bounds__(kThreads) void wide_mask_kernel(StepArgs a, int t, WideScreen w, int stiles) {
    constexpr int KB = D / 16;
    const int m = active_count(a.ctl, t);
    if (blockIdx.y == 0) step_prologue(a, t, m);   // one workgroup of the whole grid
    if (m == 0) return;
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int word = blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (word >= w.words) return;
    const bf16x8* pf = reinterpret_cast<const bf16x8*>(w.pf) + (long long)word * 2 * KB * 64 + lane;
    bf16x8 p0[KB], p1[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        p0[kb] = pf[kb * 64];
        p1[kb] = pf[(KB + kb) * 64];
    }
    f32x16 i0, i1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 u = reinterpret_cast<const float4*>(w.nx)[word * 16 + 2 * q + half];
        const float4 v = reinterpret_cast<const float4*>(w.nx)[word * 16 + 8 + 2 * q + half];
        i0[4 * q] = -u.x;
        i0[4 * q + 1] = -u.y;
        i0[4 * q + 2] = -u.z;
        i0[4 * q + 3] = -u.w;
        i1[4 * q] = -v.x;
        i1[4 * q + 1] = -v.y;
        i1[4 * q + 2] = -v.z;
        i1[4 * q + 3] = -v.w;
    }
    // no bit past the last point, whatever the seed
    const int left = a.n - word * 64;
    unsigned vlo = ~0u, vhi = ~0u;
    if (left < 64) {
        vlo = vhi = 0;
        for (int b = 0; b < 32; ++b) {
            vlo |= bit_point(b) < left ? 1u << b : 0u;
            vhi |= 32 + bit_point(b) < left ? 1u << b : 0u;
        }
    }
    const int s0 = (int)((long long)stiles * blockIdx.y / gridDim.y);
    const int s1 = (int)((long long)stiles * (blockIdx.y + 1) / gridDim.y);
    for (int st = s0; st < s1; ++st) {
        const float c = w.crow[st * 32 + (lane & 31)];
        const bf16x8* sf = reinterpret_cast<const bf16x8*>(w.sf) + (long long)st * KB * 64 + lane;
        f32x16 E0 = i0, E1 = i1;   // 2 s.x less the points' share
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const bf16x8 sv = sf[kb * 64];
            E0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p0[kb], sv, E0, 0, 0, 0);
            E1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p1[kb], sv, E1, 0, 0, 0);
        }
        unsigned b0 = 0, b1 = 0;
#pragma unroll
        for (int r = 15; r >= 0; --r) {   // kept unless ruled out: a NaN is kept
            b0 = 2 * b0 + (E0[r] < c ? 0u : 1u);
            b1 = 2 * b1 + (E1[r] < c ? 0u : 1u);
        }
        const unsigned own = b0 | (b1 << 16), other = __shfl_xor(own, 32);
        const unsigned lo = ((own & 0xffffu) | (other << 16)) & vlo;
        const unsigned hi = ((own >> 16) | (other & 0xffff0000u)) & vhi;
        if (half == 0) w.mask[(long long)(st * 32 + lane) * w.words + word] = lo | ((unsigned long long)hi << 32);
    }
}

// Sum over L neighbouring lanes, the same in each: every step adds two values
// that commute.
template <int CTRL>
__device__ __forceinline__ float row_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int L>
__device__ __forceinline__ float lanes_sum(float v) {
    if constexpr (L == 16) {
        v = row_add<0x128>(v);   // row_ror:8
        v = row_add<0x124>(v);
        v = row_add<0x122>(v);
        return row_add<0x121>(v);
    } else {
        static_assert(L == 8);
        v = row_add<0xb1>(v);    // quad_perm:[1,0,3,2]
        v = row_add<0x4e>(v);    // quad_perm:[2,3,0,1]
        return row_add<0x141>(v);   // row_half_mirror: the other quad of 8
    }
}

// A workgroup per active seed.  LP lanes hold a pair, D / LP coordinates each;
// 64 / LP pairs to a wave, U rows in flight per lane.  At least 8 coordinates a
// lane: with 4 (D = 64 by 16 lanes) the lanes' sum and the exponential are a
// third of the work (50,001 x 500 pairs, all near, three updates: 1,010 us, 834
// with 8 lanes).
template <int D, int KERN>
__global__ __launch_bounds__(64 * kEvalWaves) void wide_eval_kernel(StepArgs a, int t, WideScreen w) {
    constexpr int LP = D == 64 ? 8 : 16;     // lanes per pair
    constexpr int G = 64 / LP;               // pairs of a wave
    constexpr int C4 = D / (4 * LP);         // float4 groups per lane
    constexpr int U = D == 256 ? 2 : 4;
    constexpr int V = 4 * C4 + 1;            // a lane's sums: coordinates, weight
    constexpr int Q = (V + 3) / 4;
    const int m = active_count(a.ctl, t);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = lane % LP, grp = lane / LP;
    __shared__ unsigned short list[kEvalPoints];
    __shared__ int wcnt[kEvalWaves];
    __shared__ float red[kEvalWaves][D + 1];
    const unsigned* mask32 = reinterpret_cast<const unsigned*>(w.mask);
    const float4* X4 = reinterpret_cast<const float4*>(a.Xp);
    for (int slot = blockIdx.x; slot < m; slot += gridDim.x) {
        const int j = a.act_in[slot];
        float* sj = a.S + (long long)j * D;
        float s[4 * C4], acc[V], sum[Q];
#pragma unroll
        for (int q = 0; q < C4; ++q) {
            const float4 v = reinterpret_cast<const float4*>(sj)[q * LP + sub];
            s[4 * q] = v.x * a.scale;
            s[4 * q + 1] = v.y * a.scale;
            s[4 * q + 2] = v.z * a.scale;
            s[4 * q + 3] = v.w * a.scale;
        }
#pragma unroll
        for (int k = 0; k < V; ++k) acc[k] = 0.0f;
#pragma unroll
        for (int q = 0; q < Q; ++q) sum[q] = 0.0f;
        auto fold = [&] {
            auto take = [&](int k) {
                if (k >= V) return 0.0f;
                const float v = acc[k];
                acc[k] = 0.0f;
                return v;
            };
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const float a4 = take(4 * q), b4 = take(4 * q + 1), c4 = take(4 * q + 2), d4 = take(4 * q + 3);
                sum[q] += rows4(a4, b4, c4, d4);
            }
        };
        const int words32 = 2 * w.words;
        for (int w0 = 0; w0 < words32; w0 += 64 * kEvalWaves) {
            // the points of the set bits, in order
            const int wi = w0 + (int)threadIdx.x;
            unsigned bits = wi < words32 ? mask32[(long long)j * words32 + wi] : 0u;
            const int cnt = __popc(bits);
            int x = cnt;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(x, off);
                if (lane >= off) x += y;
            }
            __syncthreads();   // the last list and counts are no longer read
            if (lane == 63) wcnt[wave] = x;
            __syncthreads();
            int at = x - cnt, len = 0;
#pragma unroll
            for (int v = 0; v < kEvalWaves; ++v) {
                if (v < wave) at += wcnt[v];
                len += wcnt[v];
            }
            while (bits) {
                const int b = __builtin_ctz(bits);
                bits &= bits - 1;
                list[at++] = (unsigned short)(threadIdx.x * 32 + bit_point(b));
            }
            __syncthreads();
            len = __builtin_amdgcn_readfirstlane(len);
            // kEvalRun pairs a lane, then the fold (its test within one loop: 5 %)
            for (int c0 = wave * G * U; c0 < len; c0 += kEvalWaves * G * kEvalRun) {
                const int c1 = min(len, c0 + kEvalWaves * G * kEvalRun);
                for (int i0 = c0; i0 < c1; i0 += kEvalWaves * G * U) {
                    float4 x4[U][C4];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i = i0 + u * G + grp;
                        const long long p = (long long)w0 * 32 + list[i < len ? i : i0];
#pragma unroll
                        for (int q = 0; q < C4; ++q) x4[u][q] = X4[p * (D / 4) + q * LP + sub];
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        float dx[4 * C4], q2 = 0.0f;
#pragma unroll
                        for (int q = 0; q < C4; ++q) {
                            dx[4 * q] = x4[u][q].x - s[4 * q];
                            dx[4 * q + 1] = x4[u][q].y - s[4 * q + 1];
                            dx[4 * q + 2] = x4[u][q].z - s[4 * q + 2];
                            dx[4 * q + 3] = x4[u][q].w - s[4 * q + 3];
                        }
#pragma unroll
                        for (int k = 0; k < 4 * C4; ++k) q2 = fmaf(dx[k], dx[k], q2);
                        q2 = lanes_sum<LP>(q2);
                        float wt;
                        if (KERN == MS_KERNEL_GAUSSIAN) wt = __builtin_amdgcn_exp2f(-q2);
                        else wt = q2 <= a.h2 ? 1.0f : 0.0f;
                        if (i0 + u * G + grp < len) {
                            acc[4 * C4] += wt;
#pragma unroll
                            for (int k = 0; k < 4 * C4; ++k) acc[k] = fmaf(wt, dx[k], acc[k]);
                        }
                    }
                }
                fold();
            }
        }
        // the pairs of a wave, then the waves in order
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const float v = LP == 8 ? row_add<0x128>(sum[q]) : sum[q];   // row_ror:8
            const int k = 4 * q + rows4_value(lane);
            if ((lane & 15) < LP) {
                if (k < 4 * C4) red[wave][(k >> 2) * 4 * LP + sub * 4 + (k & 3)] = v;
                else if (k == 4 * C4 && sub == 0) red[wave][D] = v;
            }
        }
        __syncthreads();
        if (wave == 0) {
            constexpr int C = D / 64;
            float v[C], u[C], W = 0.0f, part2 = 0.0f;
#pragma unroll
            for (int i = 0; i < C; ++i) v[i] = 0.0f;
#pragma unroll
            for (int g = 0; g < kEvalWaves; ++g) {
                W += red[g][D];
#pragma unroll
                for (int i = 0; i < C; ++i) v[i] += red[g][lane + 64 * i];
            }
            int res = 0;
#pragma unroll
            for (int i = 0; i < C; ++i) u[i] = sj[lane + 64 * i];
            if (!(W > 0.0f) || !isfinite(W)) {
                if (lane == 0) a.status[j] = ST_FAILED;
            } else {
                const float inv = a.inv_scale / W;
                bool finite = true;
                float rn = 1.0f;
                if (a.metric == MS_METRIC_COSINE) {
                    float nn = 0.0f;
#pragma unroll
                    for (int i = 0; i < C; ++i) {
                        const float y = u[i] + v[i] * inv;
                        nn = fmaf(y, y, nn);
                    }
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) nn += __shfl_xor(nn, off);
                    rn = 1.0f / sqrtf(nn);
                    finite = nn > 0.0f && isfinite(rn);
                }
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    float dk;
                    if (a.metric == MS_METRIC_COSINE) {
                        const float y = (u[i] + v[i] * inv) * rn;
                        dk = y - u[i];
                        finite = finite && isfinite(y);
                        u[i] = y;
                    } else {
                        dk = v[i] * inv;
                        finite = finite && isfinite(dk);
                        u[i] += dk;
                    }
                    part2 = fmaf(dk, dk, part2);
                }
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) part2 += __shfl_xor(part2, off);
                finite = __ballot(!finite) == 0;
#pragma unroll
                for (int i = 0; i < C; ++i) sj[lane + 64 * i] = u[i];
                res = !finite ? 0 : (part2 < a.thr2 ? 2 : 1);
                if (lane == 0) {
                    a.iters[j] += 1;
                    a.shift2[j] = part2;
                    if (!finite) a.status[j] = ST_FAILED;
                    else if (res == 2) a.status[j] = ST_CONVERGED;
                }
            }
            // (the cosine step raises the density too, the kernel being convex in
            // s.x on unit vectors; its next pass keeps the bound of the first one)
            const float Wk = a.metric == MS_METRIC_COSINE ? 0.0f : W;
            store_seed<D>(j, u, res == 1, seed_reach(KERN, a.h2, Wk, a.n), a.scale, a.Xp,
                          reinterpret_cast<__bf16*>(w.sf), w.crow);
            if (lane == 0) {
                if (res == 1) a.act_out[atomicAdd(&a.ctl->count[(t + 1) % 3], 1)] = j;
                else if (res == 2) add_converged(a.ctl, t, 1);
            }
        }
        __syncthreads();   // red is written again
    }
}

template <int D>
hipError_t launch_screen_t(Batch& b, int t, hipStream_t s) {
    StepArgs a;
    a.Xp = b.Xp;
    a.n = b.n;
    a.d = b.d;
    a.min_chunk = b.sh.MC;
    a.S = b.S;
    a.act_in = b.act[t & 1];
    a.act_out = b.act[(t + 1) & 1];
    a.status = b.status;
    a.iters = b.iters;
    a.shift2 = b.shift2;
    a.part = b.part;
    a.red = nullptr;
    a.prog = b.prog;
    a.ctl = b.ctl;
    a.h2 = b.h * b.h;
    a.scale = b.scale;
    a.inv_scale = b.inv_scale;
    a.thr2 = b.thr2;
    a.metric = b.metric;
    const int stiles = (b.n_seeds + 31) / 32;
    if (t == 0 && !b.screen.loaded)
        hipLaunchKernelGGL((wide_seeds_kernel<D>), dim3((stiles * 32 + kWaves - 1) / kWaves), dim3(kThreads), 0, s,
                           b.S, b.status, b.n_seeds, stiles * 32, b.kernel, a.h2, b.scale, b.n, b.Xp,
                           (__bf16*)b.screen.sf, b.screen.crow);
    // as many waves as their registers allow at once, the seed tiles split where
    // the points alone are too few (D = 128: 17.6 us at 768 workgroups, 20 at 512,
    // 1,024 and 2,048; D = 256: 18 at 512, 21 at 768)
    const int pb = (b.screen.words + kWaves - 1) / kWaves;
    const int want = D == 256 ? 512 : 768;
    const int split_most = pb < want ? want / pb : 1;
    const int split = split_most < stiles ? split_most : stiles;
    hipLaunchKernelGGL((wide_mask_kernel<D>), dim3(pb, split), dim3(kThreads), 0, s, a, t, b.screen, stiles);
    const int blocks = b.n_seeds < 65536 ? b.n_seeds : 65536;
    if (b.kernel == MS_KERNEL_GAUSSIAN)
        hipLaunchKernelGGL((wide_eval_kernel<D, MS_KERNEL_GAUSSIAN>), dim3(blocks), dim3(64 * kEvalWaves), 0, s, a, t,
                           b.screen);
    else
        hipLaunchKernelGGL((wide_eval_kernel<D, MS_KERNEL_FLAT>), dim3(blocks), dim3(64 * kEvalWaves), 0, s, a, t,
                           b.screen);
    return hipGetLastError();
}

}  // namespace

// The bits take n / 8 bytes a seed: up to 256 MB.
bool wide_screen_ok(int D, long long n, long long m) {
    return D >= 64 && ((m + 31) / 32 * 32) * ((n + 63) / 64) <= (1LL << 25);
}

size_t wide_screen_carve(WideScreen& w, char* base, int D, int n, int m) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* p = base ? base + off : nullptr;
        off += (bytes + 255) / 256 * 256;
        return p;
    };
    const size_t slots = (size_t)(m + 31) / 32 * 32;
    w.words = (n + 63) / 64;
    w.pf = take((size_t)w.words * 64 * D * 2);
    w.nx = (float*)take((size_t)w.words * 64 * 4);
    w.sf = take(slots * D * 2);
    w.crow = (float*)take(slots * 4);
    w.mask = (unsigned long long*)take(slots * w.words * 8);
    return off;
}

hipError_t launch_wide_screen_points(const WideScreen& w, const float* X, int n, int d, float scale, float* Xp, int D,
                                     hipStream_t s) {
    const int tiles = 2 * w.words;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((tiles + kWaves - 1) / kWaves), dim3(kThreads), 0, s, X, n, d, scale, tiles,
                           Xp, reinterpret_cast<bf16x8*>(w.pf), w.nx);
        return hipGetLastError();
    };
    if (D == 64) return go(wide_points_kernel<64>);
    if (D == 128) return go(wide_points_kernel<128>);
    if (D == 256) return go(wide_points_kernel<256>);
    return hipErrorInvalidValue;
}

hipError_t launch_wide_screen_load(const float* seeds, const uint8_t* conv_in, Batch& b, hipStream_t s) {
    if (b.metric == MS_METRIC_COSINE) return hipErrorInvalidValue;   // unit seeds: launch_seed_init_from_array
    const int slots = (b.n_seeds + 31) / 32 * 32;
    const dim3 g((slots + kWaves - 1) / kWaves);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, g, dim3(kThreads), 0, s, seeds, conv_in, b.d, b.n_seeds, slots, b.kernel, b.h * b.h,
                           b.scale, b.n, b.Xp, b.S, b.act[0], b.status, b.iters, b.shift2, b.ctl,
                           (__bf16*)b.screen.sf, b.screen.crow);
        return hipGetLastError();
    };
    b.screen.loaded = true;
    if (b.sh.D == 64) return go(wide_load_kernel<64>);
    if (b.sh.D == 128) return go(wide_load_kernel<128>);
    if (b.sh.D == 256) return go(wide_load_kernel<256>);
    return hipErrorInvalidValue;
}

hipError_t launch_iteration_screen(Batch& b, int t, hipStream_t s) {
    if (b.sh.R != 1 || b.sh.DP != b.sh.D) return hipErrorInvalidValue;
    if (b.sh.D == 64) return launch_screen_t<64>(b, t, s);
    if (b.sh.D == 128) return launch_screen_t<128>(b, t, s);
    if (b.sh.D == 256) return launch_screen_t<256>(b, t, s);
    return hipErrorInvalidValue;
}

}  // namespace fms
