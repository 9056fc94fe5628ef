// k_runs.hip -- points grouped into 64-point tiles around sampled pivots, for
// the seed form (k_seed.hip: one cloud at D >= 8, many at any D up to 32) and the
// differentiable form (k_adjoint_runs.hip: any D up to 32) (gfx950).
//
// Each cloud samples one pivot per 128 points (at fixed strides, at most
// 1,024).  A point belongs to the run of its nearest pivot, or, farther than
// `far` from every pivot, to one of kFarRuns runs by that distance.  Runs are
// padded to whole tiles, so that no tile spans two runs: the order of the runs
// does not matter (the block forms of k_sort.hip need neighbouring pivots in
// neighbouring blocks and walk a chain over all pivots for it, 440 us of one
// workgroup at 1,024 pivots).  Two radix passes over the run number put the
// points in order.
//
// The nearest pivot is searched on the matrix cores: E = 2 x.p - |p|^2 - |x|^2
// = -|x - p|^2 with x and p relative to the cloud's first row and split into two
// bf16 parts each (hi.hi + hi.lo + lo.hi, and one product for the norms split
// in three); the largest of 32 x 32 E values of a tile is found with the row
// number in the lowest mantissa bits.  262,144 x 32 against 1,024 pivots took
// 413 us with FP32 differences on the vector units.  The choice is only a
// grouping and need not be exact; what must hold are the distance bounds kept
// with it, which carry the error bound of E: the largest distance of a near
// run's points from their pivot, and for a far run the least distance of its
// points from any pivot.

#include <algorithm>

#include "step_common.h"

namespace fms {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ int pivots_of(long long nc) {
    if (nc <= 0) return 0;
    const long long P = nc / kRunPoints;
    return (int)(P < 1 ? 1 : (P > kRunPivotMax ? kRunPivotMax : P));
}

// Offsets of every cloud: rows, pivots, 32-pivot tiles, 256-row tiles.  One
// workgroup; each thread takes a stretch of clouds.
__global__ __launch_bounds__(1024) void run_plan_kernel(const long long* __restrict__ src, int n_each, int ncl,
                                                        long long* xo, int32_t* poff, int32_t* ptoff,
                                                        int32_t* rtoff, unsigned long long* dense) {
    if (dense && threadIdx.x < 2) dense[threadIdx.x] = 0;
    __shared__ int s[3][1024];
    const int per = (ncl + 1023) / 1024;
    const int c0 = min(ncl, (int)threadIdx.x * per), c1 = min(ncl, c0 + per);
    auto rows = [&](int c) { return src ? src[c + 1] - src[c] : (long long)n_each; };
    int a[3] = {0, 0, 0};
    for (int c = c0; c < c1; ++c) {
        const long long nc = rows(c);
        const int P = pivots_of(nc);
        a[0] += P;
        a[1] += (P + 31) / 32;
        a[2] += (int)((nc + 255) / 256);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) s[q][threadIdx.x] = a[q];
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        int v[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] = (int)threadIdx.x >= off ? s[q][threadIdx.x - off] : 0;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 3; ++q) s[q][threadIdx.x] += v[q];
        __syncthreads();
    }
    int b[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) b[q] = s[q][threadIdx.x] - a[q];
    for (int c = c0; c < c1; ++c) {
        const long long nc = rows(c);
        const int P = pivots_of(nc);
        xo[c] = src ? src[c] : (long long)c * n_each;
        poff[c] = b[0];
        ptoff[c] = b[1];
        rtoff[c] = b[2];
        b[0] += P;
        b[1] += (P + 31) / 32;
        b[2] += (int)((nc + 255) / 256);
    }
    if (threadIdx.x == 1023) {
        xo[ncl] = src ? src[ncl] : (long long)ncl * n_each;
        poff[ncl] = s[0][1023];
        ptoff[ncl] = s[1][1023];
        rtoff[ncl] = s[2][1023];
    }
}

// v in three bf16 parts
__device__ __forceinline__ void split3(float v, __bf16& h, __bf16& m, __bf16& l) {
    h = (__bf16)v;
    const float r = v - (float)h;
    m = (__bf16)r;
    l = (__bf16)(r - (float)m);
}

// Operands of 32 pivots (rows of the product), one wave per tile of pivots:
// per block of 16 coordinates the hi and the lo part, then the norms
// (-|p|^2 in three parts, and ones for the points' norms).  Lane l: row l % 32,
// entries 8 (l / 32) ... + 7 of the block.  Rows past the last pivot get a
// norm that never wins.
template <int KB>
__global__ __launch_bounds__(64) void run_pivots_kernel(const float* __restrict__ X, int d, float scale,
                                                        const long long* __restrict__ xo,
                                                        const int32_t* __restrict__ poff,
                                                        const int32_t* __restrict__ ptoff, int ncl, int D, int DP, int ptot,
                                                        float* pivots, float* pivot_rows, char* frag) {
    const int c = upper_cloud(ptoff, ncl, blockIdx.x);
    const int lane = threadIdx.x, half = lane >> 5;
    const int P = poff[c + 1] - poff[c];
    const long long x0 = xo[c], nc = xo[c + 1] - x0;
    const int j = ((int)blockIdx.x - ptoff[c]) * 32 + (lane & 31);
    const bool live = j < P;
    const float* row = X + (x0 + (live ? (long long)j * nc / P : 0)) * d;
    const float* ref = X + x0 * d;
    bf16x8* out = reinterpret_cast<bf16x8*>(frag + (long long)blockIdx.x * (2 * KB + 1) * 1024);
    float nn = 0.0f;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        bf16x8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = kb * 16 + half * 8 + e;
            const float v = (live && k < d) ? (row[k] - ref[k]) * scale : 0.0f;
            if (pivots && live && k < D) pivots[(long long)k * ptot + poff[c] + j] = k < d ? row[k] * scale : 0.0f;
            if (pivot_rows && live && k < DP) pivot_rows[(long long)(poff[c] + j) * DP + k] = k < d ? row[k] : 0.0f;
            nn = fmaf(v, v, nn);
            // a reference that overflows in packed units makes every distance
            // from it NaN: all points of the cloud go to its last far run
            if (live && k < d) nn = fmaf(0.0f, ref[k] * scale, nn);
            hi[e] = (__bf16)v;
            lo[e] = (__bf16)(v - (float)hi[e]);
        }
        out[(2 * kb) * 64 + lane] = hi;
        out[(2 * kb + 1) * 64 + lane] = lo;
    }
    nn += __shfl_xor(nn, 32);
    bf16x8 nv = {};
    if (half == 0) {
        __bf16 h, m, l;
        split3(live ? -nn : -1e30f, h, m, l);
        nv[0] = h;
        nv[1] = m;
        nv[2] = l;
        nv[3] = nv[4] = nv[5] = (__bf16)1.0f;
    }
    out[2 * KB * 64 + lane] = nv;
}

// Nearest pivot of 256 rows of one cloud, 64 per wave (two column tiles of 32),
// against all pivots of the cloud, whose operands pass through LDS four tiles
// at a time.  keys = run number, vals = row; dpiv = the distance bound of the
// file comment (lower bound for a far row, upper bound for a near one).
template <int KB, bool VEC>
__global__ __launch_bounds__(256) void run_near_kernel(const float* __restrict__ rows, int ld, int d, float scale,
                                                       const long long* __restrict__ roff,
                                                       const int32_t* __restrict__ rtoff, int ncl, int single_m,
                                                       const float* __restrict__ X, int xld,
                                                       const long long* __restrict__ xo,
                                                       const int32_t* __restrict__ poff,
                                                       const int32_t* __restrict__ ptoff,
                                                       const char* __restrict__ frag, float far, unsigned* keys,
                                                       int* vals, float* dpiv, int32_t* near_pivot) {
    constexpr int F = 2 * KB + 1;
    constexpr int CH = 4;
    __shared__ bf16x8 sf[CH * F * 64];
    const int c = single_m >= 0 ? 0 : upper_cloud(rtoff, ncl, blockIdx.x);
    const long long r0 = single_m >= 0 ? 0 : roff[c];
    const long long r1 = single_m >= 0 ? (long long)single_m : roff[c + 1];
    const long long base = r0 + (long long)(single_m >= 0 ? blockIdx.x : blockIdx.x - rtoff[c]) * 256;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
    const float* ref = X + xo[c] * xld;
    const int P = poff[c + 1] - poff[c];
    const int pt0 = ptoff[c], npt = ptoff[c + 1] - pt0;

    bf16x8 bh[2][KB], bl[2][KB], bn[2];
    float xx[2];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        const long long p = base + wave * 64 + ct * 32 + (lane & 31);
        const float* row = rows + (p < r1 ? p : r1 - 1) * ld;
        float nn = 0.0f;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const int k0 = kb * 16 + half * 8;
            float xr[8];
            if constexpr (VEC) {   // d = 16 KB, rows aligned
                const float4 u0 = *reinterpret_cast<const float4*>(row + k0);
                const float4 u1 = *reinterpret_cast<const float4*>(row + k0 + 4);
                const float t[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) xr[e] = t[e] - ref[k0 + e];
            } else {
#pragma unroll
                for (int q = 0; q < 8; q += 4) {
                    if (k0 + q + 4 <= d) {   // wide loads
#pragma unroll
                        for (int e = q; e < q + 4; ++e) xr[e] = row[k0 + e] - ref[k0 + e];
                    } else {
#pragma unroll
                        for (int e = q; e < q + 4; ++e) xr[e] = k0 + e < d ? row[k0 + e] - ref[k0 + e] : 0.0f;
                    }
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float v = xr[e] * scale;
                nn = fmaf(v, v, nn);
                const float v2 = 2.0f * v;
                bh[ct][kb][e] = (__bf16)v2;
                bl[ct][kb][e] = (__bf16)(v2 - (float)bh[ct][kb][e]);
            }
        }
        nn += __shfl_xor(nn, 32);
        xx[ct] = nn;
        bn[ct] = bf16x8{};
        if (half == 0) {
            __bf16 h, m, l;
            split3(-nn, h, m, l);
            bn[ct][0] = bn[ct][1] = bn[ct][2] = (__bf16)1.0f;
            bn[ct][3] = h;
            bn[ct][4] = m;
            bn[ct][5] = l;
        }
    }
    float best[2] = {-__builtin_inff(), -__builtin_inff()};
    int bt[2] = {0, 0};
    const bf16x8* gf = reinterpret_cast<const bf16x8*>(frag) + (long long)pt0 * F * 64;
    for (int t0 = 0; t0 < npt; t0 += CH) {
        const int cnt = min(CH, npt - t0);
        __syncthreads();
        for (int e = threadIdx.x; e < cnt * F * 64; e += 256) sf[e] = gf[(long long)t0 * F * 64 + e];
        __syncthreads();
        for (int t = 0; t < cnt; ++t) {
            const bf16x8* af = sf + t * F * 64 + lane;
            bf16x8 ah[KB], al[KB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                ah[kb] = af[(2 * kb) * 64];
                al[kb] = af[(2 * kb + 1) * 64];
            }
            const bf16x8 an = af[2 * KB * 64];
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) {
                f32x16 E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(an, bn[ct], f32x16{}, 0, 0, 0);
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) {
                    E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[kb], bl[ct][kb], E, 0, 0, 0);
                    E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[kb], bh[ct][kb], E, 0, 0, 0);
                    E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[kb], bh[ct][kb], E, 0, 0, 0);
                }
                // register r holds row (r % 4) + 8 (r / 4) + 4 half
                float m = -__builtin_inff();
#pragma unroll
                for (int r = 0; r < 16; ++r) m = fmaxf(m, __int_as_float((__float_as_int(E[r]) & ~15) | r));
                if (m > best[ct]) {
                    best[ct] = m;
                    bt[ct] = t0 + t;
                }
            }
        }
    }
    // the two halves of a column, then lane l takes column tile l / 32
    float qe = 0.0f, x2 = 0.0f;
    int pv = 0;
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        const int r = __float_as_int(best[ct]) & 15;
        int pj = bt[ct] * 32 + (r & 3) + 8 * (r >> 2) + 4 * half;
        const float ob = __shfl_xor(best[ct], 32);
        const int op = __shfl_xor(pj, 32);
        float b = best[ct];
        if (ob > b || (ob == b && op < pj)) {
            b = ob;
            pj = op;
        }
        if (ct == half) {
            qe = -b;
            pv = pj;
            x2 = xx[ct];
        }
    }
    const long long p = base + wave * 64 + half * 32 + (lane & 31);
    if (p >= r1) return;
    qe = fmaxf(qe, 0.0f);
    if (pv >= P) pv = P - 1;   // only when no E was a number
    // |p|^2 <= 2 |x|^2 + 2 q for the nearest pivot: the bound of E's error
    const float eps = (3.0f * x2 + 2.0f * qe) * (1.0f / 8192.0f);
    const bool fine = qe + eps < 3e38f;
    const float dist = fine ? __builtin_amdgcn_sqrtf(qe) : 0.0f;
    const bool is_far = !fine || dist > far;
    unsigned run = (unsigned)(poff[c] + kFarRuns * c);
    if (is_far)
        run += (unsigned)P + (fine ? (unsigned)fminf((dist - far) * (4.0f / far), (float)(kFarRuns - 1)) : kFarRuns - 1u);
    else
        run += (unsigned)pv;
    keys[p] = run;
    vals[p] = (int)p;
    if (near_pivot) {   // seeds: the pivot itself, and an upper bound
        near_pivot[p] = pv;
        dpiv[p] = fine ? __builtin_amdgcn_sqrtf(qe + eps) * 1.0001f : __builtin_inff();
    } else {
        float b = 0.0f;
        if (fine) b = is_far ? __builtin_amdgcn_sqrtf(fmaxf(qe - eps, 0.0f)) * 0.9999f
                             : __builtin_amdgcn_sqrtf(qe + eps) * 1.0001f;
        dpiv[p] = b;
    }
}

// First sorted position of every run, and the empty bounds: position i opens the runs between the
// key before it and its own.
__global__ void run_starts_kernel(const unsigned* __restrict__ keys, int n, int runs,
                                  const int32_t* __restrict__ poff, int ncl, int32_t* start, float* bound) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < runs) {   // of a run without points; the fill takes its points' in
        const int c = upper_cloud_runs(poff, ncl, i);
        bound[i] = i >= poff[c + 1] + kFarRuns * c ? __builtin_inff() : 0.0f;
    }
    if (i > n) return;
    const int from = i == 0 ? 0 : (int)keys[i - 1] + 1;
    const int to = i == n ? runs : (int)keys[i];
    for (int r = from; r <= to; ++r) start[r] = i;
}

// First tile of every run, in run order.  One workgroup; each thread takes a stretch of runs.
__global__ __launch_bounds__(1024) void run_tiles_kernel(const int32_t* __restrict__ start, int runs,
                                                         int32_t* tile_start) {
    __shared__ int s[1024];
    const int per = (runs + 1023) / 1024;
    const int r0 = min(runs, (int)threadIdx.x * per), r1 = min(runs, r0 + per);
    int a = 0;
#pragma unroll 8
    for (int r = r0; r < r1; ++r) a += (start[r + 1] - start[r] + 63) / 64;
    s[threadIdx.x] = a;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int v = (int)threadIdx.x >= off ? s[threadIdx.x - off] : 0;
        __syncthreads();
        s[threadIdx.x] += v;
        __syncthreads();
    }
    int b = s[threadIdx.x] - a;
#pragma unroll 8
    for (int r = r0; r < r1; ++r) {
        tile_start[r] = b;
        b += (start[r + 1] - start[r] + 63) / 64;
    }
    if (threadIdx.x == 1023) tile_start[runs] = s[1023];
}

// The run of every tile (by the workgroup above: 35 of its 45 us at 19,000 runs).
__global__ void run_of_tile_kernel(const int32_t* __restrict__ tile_start, int runs, int32_t* tile_run) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= runs) return;
    for (int t = tile_start[r]; t < tile_start[r + 1]; ++t) tile_run[t] = r;
}

// One wave per tile: gathers the run's rows, in packed units, and folds its
// points' bounds into the run's (integer atomics on the float's pattern, which
// is monotone from 0 up: the same result in any order).
template <int D>
__global__ __launch_bounds__(256) void run_fill_kernel(const float* __restrict__ X, int d, float scale, int vec4,
                                                       const int* __restrict__ vals,
                                                       const float* __restrict__ dpiv,
                                                       const int32_t* __restrict__ start,
                                                       const int32_t* __restrict__ tile_start,
                                                       const int32_t* __restrict__ tile_run, int runs,
                                                       const int32_t* __restrict__ poff, int ncl, int row_major,
                                                       float* tiles, float* bound, int32_t* rows) {
    constexpr int DP = D <= 4 ? 4 : D;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= tile_start[runs]) return;
    const int r = tile_run[t];
    const int pos = start[r] + (t - tile_start[r]) * 64 + lane;
    const int end = start[r + 1];
    const bool live = pos < end;
    const int row = live ? vals[pos] : -1;
    const float dp = live ? dpiv[row] : 0.0f;
    float x[DP];
#pragma unroll
    for (int k = 0; k < DP; ++k) x[k] = 0.0f;
    if (live) {
        if (vec4) {
            const float4* src = reinterpret_cast<const float4*>(X + (long long)row * d);
#pragma unroll
            for (int q = 0; q < DP / 4; ++q) {
                if (4 * q < d) {
                    const float4 v = src[q];
                    x[4 * q] = v.x * scale;
                    x[4 * q + 1] = v.y * scale;
                    x[4 * q + 2] = v.z * scale;
                    x[4 * q + 3] = v.w * scale;
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < D; ++k)
                if (k < d) x[k] = X[(long long)row * d + k] * scale;
        }
    }
    // runs of a cloud: its pivots', then the far ones
    const int c = upper_cloud_runs(poff, ncl, r);
    const bool far = r >= poff[c + 1] + kFarRuns * c;
    float v = live ? (far ? -dp : dp) : -__builtin_inff();   // far runs: the smallest
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    if (lane == 0) {
        if (far) atomicMin(reinterpret_cast<int*>(bound) + r, __float_as_int(fmaxf(-v, 0.0f)));
        else atomicMax(reinterpret_cast<int*>(bound) + r, __float_as_int(fmaxf(v, 0.0f)));
    }
    if (!live) x[0] = kPadCoord;
    const int ostep = row_major ? 1 : 64;
    float4* out = reinterpret_cast<float4*>(tiles) + (long long)t * (DP / 4) * 64 + lane * (row_major ? DP / 4 : 1);
#pragma unroll
    for (int q = 0; q < DP / 4; ++q) out[q * ostep] = make_float4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
    if (rows) rows[t * 64 + lane] = row;
}

// Ball of each run of row-major tiles, one wave per run: the mean of its rows
// and the largest distance from it (packed units, rounded up).  In 16-D a ball
// around the mean of a run has 0.7 of the radius around one of its points.  A
// run too long for one wave (far points of a cloud without clusters) gets an
// infinite radius, and so does one with a point whose distance from the mean is
// not finite: no distance from such a ball rules its points out.
constexpr int kBallRows = 8192;
template <int D>
__global__ __launch_bounds__(256) void run_ball_kernel(const float* __restrict__ tiles,
                                                       const int32_t* __restrict__ start,
                                                       const int32_t* __restrict__ tile_start, int runs, float scale,
                                                       float* balls) {
    constexpr int DP = D <= 4 ? 4 : D;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= runs) return;
    const int cnt = start[r + 1] - start[r];
    if (cnt > kBallRows) {
        if (lane < DP) balls[(long long)r * (DP + 4) + lane] = 0.0f;
        if (lane == 0) balls[(long long)r * (DP + 4) + DP] = __builtin_inff();
        return;
    }
    const float4* src = reinterpret_cast<const float4*>(tiles) + (long long)tile_start[r] * 64 * (DP / 4);
    auto row = [&](int i, float (&x)[DP]) {
#pragma unroll
        for (int q = 0; q < DP / 4; ++q) {
            const float4 v = src[(long long)i * (DP / 4) + q];
            x[4 * q] = v.x;
            x[4 * q + 1] = v.y;
            x[4 * q + 2] = v.z;
            x[4 * q + 3] = v.w;
        }
    };
    float c[DP];
#pragma unroll
    for (int k = 0; k < DP; ++k) c[k] = 0.0f;
    for (int i = lane; i < cnt; i += 64) {
        float x[DP];
        row(i, x);
#pragma unroll
        for (int k = 0; k < DP; ++k) c[k] += x[k];
    }
    const float inv = 1.0f / (float)(cnt > 0 ? cnt : 1);
#pragma unroll
    for (int k = 0; k < DP; ++k) c[k] = k < D ? lane_value(wave_add63(c[k]), 63) * inv : 0.0f;
    float r2 = 0.0f;
    bool fin = true;
    for (int i = lane; i < cnt; i += 64) {
        float x[DP], q = 0.0f;
        row(i, x);
#pragma unroll
        for (int k = 0; k < D; ++k) q = fmaf(x[k] - c[k], x[k] - c[k], q);
        r2 = fmaxf(r2, q);   // passes a NaN over
        fin = fin && isfinite(q);
    }
    const bool allfin = __ballot(!fin) == 0;
    r2 = -lane_value(wave_min63(-r2), 63);
    if (lane == 0) {
        float* o = balls + (long long)r * (DP + 4);
#pragma unroll
        for (int k = 0; k < DP; ++k) o[k] = c[k];
        o[DP] = allfin ? sqrtf(r2) * scale * 1.0001f + 1e-30f : __builtin_inff();
    }
}

// Row-major tiles of other rows in an index's order (a row per slot).
template <int D>
__global__ __launch_bounds__(256) void run_regroup_kernel(const float* __restrict__ S, int d,
                                                          const int32_t* __restrict__ rows,
                                                          const int32_t* __restrict__ tile_start, int runs,
                                                          float* tiles) {
    constexpr int DP = D <= 4 ? 4 : D;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= tile_start[runs] * 64) return;
    const int row = rows[e];
    float4* out = reinterpret_cast<float4*>(tiles) + (long long)e * (DP / 4);
#pragma unroll
    for (int q = 0; q < DP / 4; ++q) {
        float x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = (row >= 0 && 4 * q + k < d) ? S[(long long)row * d + 4 * q + k] : 0.0f;
        out[q] = make_float4(x[0], x[1], x[2], x[3]);
    }
}

hipError_t launch_balls(const RunIndex& r, const float* tiles, float* balls, hipStream_t s) {
    const dim3 bg((r.sz.runs + 3) / 4);
#define FMS_CASE(DD)                                                                                            \
    case DD:                                                                                                    \
        hipLaunchKernelGGL((run_ball_kernel<DD>), bg, dim3(256), 0, s, tiles, r.run_start, r.tile_start,         \
                           r.sz.runs, r.scale, balls);                                                          \
        break;
    switch (r.D) {
        FMS_CASE(1) FMS_CASE(2) FMS_CASE(3) FMS_CASE(4) FMS_CASE(8) FMS_CASE(16) FMS_CASE(32)
        default: return hipErrorInvalidValue;
    }
#undef FMS_CASE
    return hipGetLastError();
}

// Distances between the pivots, rounded down (1e-4 relative).
__global__ __launch_bounds__(256) void pivot_pairs_kernel(const float* __restrict__ pv, int P, int D, float* out) {
    const int j = blockIdx.x * 256 + threadIdx.x, i = blockIdx.y;
    if (j >= P) return;
    float q = 0.0f;
    for (int k = 0; k < D; ++k) {
        const float u = pv[(long long)k * P + j] - pv[(long long)k * P + i];
        q = fmaf(u, u, q);
    }
    out[(long long)i * P + j] = sqrtf(q) * 0.9999f;
}

// RunIndex::dense from every kDenseRow-th pivot, 256 runs to a workgroup.  kDenseReach
// is the reach of a seed amid 2^12 to 2^18 points (k_seed.hip).  Sums of whole
// numbers: any order.
constexpr int kDenseRow = 16;
constexpr float kDenseReach = 7.0f;
__global__ __launch_bounds__(256) void run_dense_kernel(const float* __restrict__ pv, int P, int D,
                                                        const float* __restrict__ bound,
                                                        const int32_t* __restrict__ tile_start, float reach,
                                                        unsigned long long* dense) {
    __shared__ int s[2][4];
    const int i = blockIdx.x * kDenseRow;
    int near = 0, all = 0;
    const int j = blockIdx.y * 256 + threadIdx.x;
    if (j < P) {
        float q = 0.0f;
#pragma unroll 16
        for (int k = 0; k < D; ++k) {
            const float u = pv[(long long)k * P + j] - pv[(long long)k * P + i];
            q = fmaf(u, u, q);
        }
        const int tiles = tile_start[j + 1] - tile_start[j];
        all += tiles;
        if (sqrtf(q) - bound[j] <= reach) near += tiles;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        near += __shfl_xor(near, off);
        all += __shfl_xor(all, off);
    }
    if ((threadIdx.x & 63) == 0) {
        s[0][threadIdx.x >> 6] = near;
        s[1][threadIdx.x >> 6] = all;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const unsigned long long w = (unsigned long long)(tile_start[i + 1] - tile_start[i]);
        const int* v = s[threadIdx.x];
        atomicAdd(&dense[threadIdx.x], w * (unsigned long long)(v[0] + v[1] + v[2] + v[3]));
    }
}

void add_cloud(RunSizes& z, long long nc) {
    const int P = run_pivots(nc);
    z.ptot += P;
    z.pmax = std::max(z.pmax, P);
    z.ptiles += (P + 31) / 32;
    z.rtiles += (int)((nc + 255) / 256);
}

void finish_sizes(RunSizes& z) {
    z.runs = z.ptot + kFarRuns * z.ncl;
    // every run but the empty ones may leave one tile partly filled
    z.max_tiles = std::max(1, std::min(z.n, z.n / 64 + z.runs));
}

int radix_passes(int runs) {
    int bits = 1;
    while (bits < 31 && (1 << bits) < runs) ++bits;
    return (bits + 7) / 8;
}

#define FMS_KB(D_, ...)                                              \
    do {                                                             \
        if ((D_) <= 16) { constexpr int KB = 1; __VA_ARGS__; }       \
        else if ((D_) == 32) { constexpr int KB = 2; __VA_ARGS__; }  \
        else return hipErrorInvalidValue;                            \
    } while (0)

}  // namespace

int run_pivots(long long nc) {
    if (nc <= 0) return 0;
    return (int)std::max(1LL, std::min((long long)kRunPivotMax, nc / kRunPoints));
}

RunSizes run_sizes(const long long* x_off, int ncl) {
    RunSizes z;
    z.ncl = ncl;
    z.n = (int)x_off[ncl];
    for (int c = 0; c < ncl; ++c) add_cloud(z, x_off[c + 1] - x_off[c]);
    finish_sizes(z);
    return z;
}

RunSizes run_sizes_equal(int ncl, int n_each) {
    RunSizes z;
    z.ncl = ncl;
    z.n = ncl * n_each;
    for (int c = 0; c < ncl; ++c) add_cloud(z, n_each);
    finish_sizes(z);
    return z;
}

hipError_t launch_run_index(RunIndex& r, const float* X, const long long* xo_src, int n_each, float scale,
                            float far, hipStream_t s) {
    const RunSizes& z = r.sz;
    r.scale = scale;
    r.far = far;
    r.X = X;
    if (z.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(run_plan_kernel, dim3(1), dim3(1024), 0, s, xo_src, n_each, z.ncl, r.xo, r.poff, r.ptoff,
                       r.rtoff, r.dense);
    FMS_KB(r.D, hipLaunchKernelGGL((run_pivots_kernel<KB>), dim3(z.ptiles), dim3(64), 0, s, X, r.d, scale, r.xo,
                                   r.poff, r.ptoff, z.ncl, r.D, r.DP, z.ptot, r.pivots, r.pivot_rows, r.frag));
    const int vec4 = r.d % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0;
    auto near = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(z.rtiles), dim3(256), 0, s, X, r.d, r.d, scale, r.xo, r.rtoff, z.ncl, -1, X,
                           r.d, r.xo, r.poff, r.ptoff, r.frag, far, r.k0, r.v0, r.dpiv, (int32_t*)nullptr);
    };
    FMS_KB(r.D, if (vec4 && r.d == 16 * KB) near(run_near_kernel<KB, true>); else near(run_near_kernel<KB, false>));
    unsigned* keys;
    int* vals;
    hipError_t e = launch_radix_pairs(r.k0, r.k1, r.v0, r.v1, r.radix, z.n, radix_passes(z.runs), &keys, &vals, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(run_starts_kernel, dim3((std::max(z.n, z.runs) + 256) / 256), dim3(256), 0, s, keys, z.n, z.runs,
                       r.poff, z.ncl, r.run_start, r.run_bound);
    hipLaunchKernelGGL(run_tiles_kernel, dim3(1), dim3(1024), 0, s, r.run_start, z.runs, r.tile_start);
    hipLaunchKernelGGL(run_of_tile_kernel, dim3((z.runs + 255) / 256), dim3(256), 0, s, r.tile_start, z.runs,
                       r.tile_run);
    const dim3 fg((z.max_tiles + 3) / 4);
#define FMS_CASE(DD)                                                                                          \
    case DD:                                                                                                  \
        hipLaunchKernelGGL((run_fill_kernel<DD>), fg, dim3(256), 0, s, X, r.d, r.row_major ? 1.0f : scale,    \
                           vec4, vals, r.dpiv, r.run_start, r.tile_start, r.tile_run, z.runs, r.poff, z.ncl,  \
                           r.row_major ? 1 : 0, r.tiles, r.run_bound, r.rows);                                                              \
        break;
    switch (r.D) {
        FMS_CASE(1) FMS_CASE(2) FMS_CASE(3) FMS_CASE(4) FMS_CASE(8) FMS_CASE(16) FMS_CASE(32)
        default: return hipErrorInvalidValue;
    }
#undef FMS_CASE
    if (r.row_major) return launch_balls(r, r.tiles, r.ball_rows, s);
    if (r.dense)   // far: 8 packed units, whatever the kernel's units are
        hipLaunchKernelGGL(run_dense_kernel, dim3((z.ptot + kDenseRow - 1) / kDenseRow, (z.ptot + 255) / 256), dim3(256), 0, s, r.pivots,
                           z.ptot, r.D, r.run_bound, r.tile_start, kDenseReach / 8.0f * far, r.dense);
    return hipGetLastError();
}

hipError_t launch_run_regroup(const RunIndex& r, const float* S, float* tiles, float* balls, hipStream_t s) {
    const dim3 g((unsigned)(((long long)r.sz.max_tiles * 64 + 255) / 256));
#define FMS_CASE(DD)                                                                                           \
    case DD:                                                                                                   \
        hipLaunchKernelGGL((run_regroup_kernel<DD>), g, dim3(256), 0, s, S, r.d, r.rows, r.tile_start,          \
                           r.sz.runs, tiles);                                                                  \
        break;
    switch (r.D) {
        FMS_CASE(1) FMS_CASE(2) FMS_CASE(3) FMS_CASE(4) FMS_CASE(8) FMS_CASE(16) FMS_CASE(32)
        default: return hipErrorInvalidValue;
    }
#undef FMS_CASE
    return launch_balls(r, tiles, balls, s);
}

hipError_t launch_run_seeds(const RunIndex& r, const float* S, int m, RunSeeds& q, hipStream_t s) {
    if (r.sz.ncl != 1) return hipErrorInvalidValue;
    const int P = r.sz.ptot;
    FMS_KB(r.D, hipLaunchKernelGGL((run_near_kernel<KB, false>), dim3((m + 255) / 256), dim3(256), 0, s, S, r.DP,
                                   r.d, r.scale, nullptr, nullptr, 1, m, r.X, r.d, r.xo, r.poff, r.ptoff, r.frag,
                                   r.far, q.k0, q.v0, q.dist, q.near));
    hipLaunchKernelGGL(pivot_pairs_kernel, dim3((P + 255) / 256, P), dim3(256), 0, s, r.pivots, P, r.D, q.ppair);
    unsigned* keys;
    const hipError_t e =
        launch_radix_pairs(q.k0, q.k1, q.v0, q.v1, q.tmp, m, radix_passes(r.sz.runs), &keys, &q.order, s);
    return e;
}

}  // namespace fms
