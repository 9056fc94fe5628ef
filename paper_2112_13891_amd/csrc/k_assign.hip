// k_assign.hip -- nearest-mode labelling ("cluster x by the distance to
// modes", Algorithm 2, final loop) and the input finiteness scan, for gfx950.
//
// One lane per point: the point row stays in registers, the modes stream
// through LDS tiles shared by the workgroup, and the lane keeps the two
// smallest squared distances.  Distances are FP32 direct differences (the
// expanded |x|^2 + |m|^2 - 2 x.m form cancels badly at large coordinates).
// Modes are scanned in increasing index with a strict '<', so ties go to
// the lowest index, as the oracle's argmin does.
//
// Wide rows and many modes (assign_mfma_kernel): the expanded form on the matrix
// cores only tells which modes can be the nearest; their distances are then
// computed as above, so labels and margins are bit for bit those of the scan.

#include "fms_internal.h"

namespace fms {

namespace {

constexpr int kT = 256;

template <int D>
__global__ __launch_bounds__(kT) void assign_kernel(const float* __restrict__ X, int n, int d,
                                                    const float* __restrict__ modes, int k,
                                                    int32_t* __restrict__ labels,
                                                    float* __restrict__ margin) {
    constexpr int TM = (D <= 4) ? 1024 : (4096 / D);   // modes per LDS tile (16 KB)
    __shared__ float tile[TM * D];
    const int i = blockIdx.x * kT + threadIdx.x;
    float x[D];
    const bool live = i < n;
#pragma unroll
    for (int q = 0; q < D; ++q) x[q] = (live && q < d) ? X[(long long)i * d + q] : 0.0f;
    float best = __builtin_inff(), second = __builtin_inff();
    int arg = 0;
    for (int base = 0; base < k; base += TM) {
        const int cnt = min(TM, k - base);
        __syncthreads();
        for (int e = threadIdx.x; e < cnt * D; e += kT) {
            const int j = e / D, q = e % D;
            tile[e] = (q < d) ? modes[(long long)(base + j) * d + q] : 0.0f;
        }
        __syncthreads();
        for (int j = 0; j < cnt; ++j) {
            float dd = 0.0f;
#pragma unroll
            for (int q = 0; q < D; ++q) {
                const float t = x[q] - tile[j * D + q];
                dd = fmaf(t, t, dd);
            }
            if (dd < best) {
                second = best;
                best = dd;
                arg = base + j;
            } else if (dd < second) {
                second = dd;
            }
        }
    }
    if (live) {
        labels[i] = arg;
        if (margin) margin[i] = (k > 1) ? sqrtf(second) - sqrtf(best) : __builtin_inff();
    }
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// Candidates by matrix products.  With x and m relative to the first mode and
// split into two bf16 parts each,
//     E = 2 x.m - |m|^2 - |x|^2 = -|x - m|^2
// is a sum of hi.hi + hi.lo + lo.hi and of the norms split in three, off by less
// than eps = 2^-13 (3 |x|^2 + 2 q) for a mode at squared distance q (a bf16 part
// is within 2^-8 of its value: lo.lo and what the lo parts leave out are below
// 3 2^-16 of 2 |x||m|, the matrix unit's sums off by less than 2^-17 of their
// largest term, and |x|^2 + |m|^2 <= 3 |x|^2 + 2 q).  A first pass over the
// modes finds the largest E of every point (with MARGIN: the second largest);
// a mode whose E lies more than 2 eps below it cannot be the nearest (second
// nearest) in FP32 either.  The second pass lists the modes within that band,
// and their distances are computed by direct differences in the order of
// assign_kernel.  A point whose list overflows, or whose bound is not finite,
// scans all modes.
//
// A workgroup of four waves takes 256 points, a wave two column tiles of 32;
// the modes pass in tiles of 32, split to bf16 in LDS by the workgroup (the
// next tile's rows loaded ahead).  The matrix unit (7 products of 32 x 32 x 16
// a tile and pass at D = 32), the rest of the two passes on the VALU and the
// barriers take a similar time each.  Rows of exactly D coordinates are read
// in wide loads: by single coordinates, the points' and the candidates' rows
// alone cost 50 us of the first form's 194 us.
constexpr int kAsgCand = 10;

template <int D, bool MARGIN>
__global__ __launch_bounds__(kT) void assign_mfma_kernel(const float* __restrict__ X, int n, int d,
                                                         const float* __restrict__ modes, int k,
                                                         int32_t* __restrict__ labels, float* __restrict__ margin) {
    constexpr int KB = D <= 16 ? 1 : D / 16;
    constexpr int F = 2 * KB + 1;
    constexpr int EPT = D / 8;   // coordinates of a mode tile per thread
    __shared__ __attribute__((aligned(16))) __bf16 sf[2][F * 64 * 8];
    __shared__ int cand[kT / 64][2][kAsgCand][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
    const int base = blockIdx.x * kT + wave * 64;

    // this wave's points as the right operand
    bf16x8 bh[2][KB], bl[2][KB], bn[2];
    float x2[2];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        const int p = base + ct * 32 + (lane & 31);
        const float* row = X + (long long)(p < n ? p : n - 1) * d;
        float nn = 0.0f;
        float xv[KB][8];
        if (D >= 16 && d == D) {   // whole rows, in wide loads
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int e = 0; e < 8; ++e) xv[kb][e] = row[kb * 16 + half * 8 + e] - modes[kb * 16 + half * 8 + e];
        } else {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int c = kb * 16 + half * 8 + e;
                    xv[kb][e] = c < d ? row[c] - modes[c] : 0.0f;
                }
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float v = xv[kb][e];
                nn = fmaf(v, v, nn);
                bh[ct][kb][e] = (__bf16)(2.0f * v);
                bl[ct][kb][e] = (__bf16)(2.0f * v - (float)bh[ct][kb][e]);
            }
        nn += __shfl_xor(nn, 32);
        x2[ct] = nn;
        bn[ct] = bf16x8{};
        if (half == 0) {
            const __bf16 h = (__bf16)(-nn);
            const float r = -nn - (float)h;
            const __bf16 m = (__bf16)r;
            bn[ct][0] = bn[ct][1] = bn[ct][2] = (__bf16)1.0f;
            bn[ct][3] = h;
            bn[ct][4] = m;
            bn[ct][5] = (__bf16)(r - (float)m);
        }
    }

    // mode tiles: row threadIdx / 8 of the tile, coordinates EPT (threadIdx % 8) ..
    const int mrow = threadIdx.x >> 3, mseg = threadIdx.x & 7;
    float mv[EPT], ref[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) ref[e] = mseg * EPT + e < d ? modes[mseg * EPT + e] : 0.0f;
    auto load = [&](int t) {
        const int j = t * 32 + mrow;
        const float* src = modes + (long long)(j < k ? j : 0) * d;
        if (d == D) {
#pragma unroll
            for (int e = 0; e < EPT; ++e) mv[e] = src[mseg * EPT + e] - ref[e];
        } else {
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                const int c = mseg * EPT + e;
                mv[e] = c < d ? src[c] - ref[e] : 0.0f;
            }
        }
    };
    auto store = [&](int t) {
        __bf16* f = sf[t & 1];
        float nn = 0.0f;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int c = mseg * EPT + e;
            const __bf16 h = (__bf16)mv[e];
            nn = fmaf(mv[e], mv[e], nn);
            const int at = (mrow + 32 * ((c & 15) >> 3)) * 8 + (c & 7);
            f[(2 * (c >> 4)) * 512 + at] = h;
            f[(2 * (c >> 4) + 1) * 512 + at] = (__bf16)(mv[e] - (float)h);
        }
        // the row's norm over its eight threads
        nn += __shfl_xor(nn, 1);
        nn += __shfl_xor(nn, 2);
        nn += __shfl_xor(nn, 4);
        if (mseg == 0) {
            const float v = t * 32 + mrow < k ? -nn : -1e30f;   // rows past the last mode never win
            const __bf16 h = (__bf16)v;
            const float r = v - (float)h;
            const __bf16 m = (__bf16)r;
            bf16x8 nv = {};
            nv[0] = h;
            nv[1] = m;
            nv[2] = (__bf16)(r - (float)m);
            nv[3] = nv[4] = nv[5] = (__bf16)1.0f;
            *reinterpret_cast<bf16x8*>(f + 2 * KB * 512 + mrow * 8) = nv;
        }
    };
    // what the stores leave alone stays zero: the norms' upper half, and the
    // padding coordinates of a single block
    for (int e = threadIdx.x; e < 2 * F * 512 / 8; e += kT) reinterpret_cast<bf16x8*>(sf)[e] = bf16x8{};
    __syncthreads();

    const int tiles = (k + 31) / 32;
    // f(tile, E of the first column tile, E of the second) for every tile of modes
    auto pass = [&](auto&& f) {
        load(0);
        store(0);
        if (tiles > 1) load(1);
        __syncthreads();
        for (int t = 0; t < tiles; ++t) {
            if (t + 1 < tiles) store(t + 1);
            if (t + 2 < tiles) load(t + 2);
            const bf16x8* af = reinterpret_cast<const bf16x8*>(sf[t & 1]) + lane;
            const bf16x8 an = af[2 * KB * 64];
            f32x16 E0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(an, bn[0], f32x16{}, 0, 0, 0);
            f32x16 E1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(an, bn[1], f32x16{}, 0, 0, 0);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const bf16x8 ah = af[(2 * kb) * 64], al = af[(2 * kb + 1) * 64];
                E0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl[0][kb], E0, 0, 0, 0);
                E1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl[1][kb], E1, 0, 0, 0);
                E0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh[0][kb], E0, 0, 0, 0);
                E1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh[1][kb], E1, 0, 0, 0);
                E0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh[0][kb], E0, 0, 0, 0);
                E1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh[1][kb], E1, 0, 0, 0);
            }
            f(t, 0, E0);
            f(t, 1, E1);
            __syncthreads();
        }
    };

    // the largest (two) E of every point
    float e1[2], e2[2];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) e1[ct] = e2[ct] = -__builtin_inff();
    pass([&](int, int ct, const f32x16& E) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (MARGIN) e2[ct] = fmaxf(e2[ct], fminf(e1[ct], E[r]));
            e1[ct] = fmaxf(e1[ct], E[r]);
        }
    });
    float thr[2];
    bool scan[2];   // this point scans all modes
    int cnt[2];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        const float o1 = __shfl_xor(e1[ct], 32);
        float top = fmaxf(e1[ct], o1);
        if (MARGIN) top = fmaxf(fmaxf(e2[ct], __shfl_xor(e2[ct], 32)), fminf(e1[ct], o1));
        const float q = fmaxf(-top, 0.0f);
        thr[ct] = top - (3.0f * x2[ct] + 2.0f * q) * (1.0f / 4096.0f) - 1e-30f;
        scan[ct] = !(thr[ct] > -1e29f);
        cnt[ct] = 0;
    }
    // the modes within the band
    pass([&](int t, int ct, const f32x16& E) {
        float m = E[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) m = fmaxf(m, E[r]);
        if (__ballot(m >= thr[ct])) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (E[r] >= thr[ct]) {
                    if (cnt[ct] < kAsgCand) cand[wave][ct][cnt[ct]][lane] = t * 32 + (r & 3) + 8 * (r >> 2) + 4 * half;
                    ++cnt[ct];
                }
            }
        }
    });

    // a row by its lane, zeros past d; a full row in wide loads
    auto load_padded = [&](const float* row, float* v) {
        if (d == D) {
#pragma unroll
            for (int q = 0; q < D; ++q) v[q] = row[q];
        } else {
#pragma unroll
            for (int q = 0; q < D; ++q) v[q] = q < d ? row[q] : 0.0f;
        }
    };
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        const int p = base + ct * 32 + (lane & 31);
        const int over = (scan[ct] || cnt[ct] > kAsgCand) ? 1 : 0;
        const bool all = (over | __shfl_xor(over, 32)) != 0;   // either half's list; every lane shuffles
        float x[D];
        const float* row = X + (long long)(p < n ? p : n - 1) * d;
        load_padded(row, x);
        float best = __builtin_inff(), second = __builtin_inff();
        int arg = 0x7fffffff;
        // the scan's halves: even and odd modes
        const int count = all ? (k - half + 1) / 2 : cnt[ct];
        for (int i = 0; __ballot(i < count); ++i) {
            if (i < count) {
                const int j = all ? 2 * i + half : cand[wave][ct][i < kAsgCand ? i : 0][lane];
                float dd = 0.0f, y[D];
                load_padded(modes + (long long)j * d, y);
#pragma unroll
                for (int q = 0; q < D; ++q) {
                    const float t = x[q] - y[q];
                    dd = fmaf(t, t, dd);
                }
                // the lowest index among equals, in whatever order they come
                if (dd < best || (dd == best && j < arg && dd < __builtin_inff())) {
                    second = best;
                    best = dd;
                    arg = j;
                } else if (dd < second) {
                    second = dd;
                }
            }
        }
        const float ob = __shfl_xor(best, 32), os = __shfl_xor(second, 32);
        const int oa = __shfl_xor(arg, 32);
        const float lose = fmaxf(best, ob);
        second = fminf(fminf(second, os), lose);
        if (ob < best || (ob == best && oa < arg)) {
            best = ob;
            arg = oa;
        }
        if (half == 0 && p < n) {
            labels[p] = arg == 0x7fffffff ? 0 : arg;   // no distance is a number: the scan's start
            if (MARGIN) margin[p] = (k > 1) ? sqrtf(second) - sqrtf(best) : __builtin_inff();
        }
    }
}

__global__ void check_finite_kernel(const float* __restrict__ X, long long count,
                                    int32_t* flag) {
    long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    bool bad = false;
    for (; e < count; e += stride) bad = bad || !isfinite(X[e]);
    if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

}  // namespace

// Modes from which the candidates come from the matrix cores: under them the
// points' setup and the exact distances cost more than the passes save.
// Measured against the direct form (assign_kernel), us:
//   D = 32, 262,144 points: k = 64 44 -> 27, 500 210 -> 76
//   D = 64,  50,000 points: k = 64 44 -> 22, 500 276 -> 73
//   D = 16,  30,000 points: k = 64 13.5 -> 11.4, 500 78 -> 43
//   D = 8,  100,000 points: k = 64 10.5 -> 11.1, 128 18 -> 15, 500 63 -> 37
//   d = 9,  200,000 points (rows short of D): k = 64 16 -> 20, 500 101 -> 55
bool assign_by_matrix(int D, int d, int k) {
    return D >= 8 && D <= 64 && k >= (D >= 16 && d == D ? 64 : 128);
}

hipError_t launch_assign(const float* X, int n, int d, const float* modes, int k,
                         int32_t* labels, float* margin, hipStream_t s) {
    const int blocks = (n + kT - 1) / kT;
    const int Dw = step_shape(d).D;
    if (assign_by_matrix(Dw, d, k)) {
#define FMS_CASE(DD)                                                                                             \
    if (Dw == DD) {                                                                                              \
        if (margin)                                                                                              \
            hipLaunchKernelGGL((assign_mfma_kernel<DD, true>), dim3(blocks), dim3(kT), 0, s, X, n, d, modes, k,  \
                               labels, margin);                                                                  \
        else                                                                                                     \
            hipLaunchKernelGGL((assign_mfma_kernel<DD, false>), dim3(blocks), dim3(kT), 0, s, X, n, d, modes, k, \
                               labels, margin);                                                                  \
        return hipGetLastError();                                                                                \
    }
        FMS_CASE(8) FMS_CASE(16) FMS_CASE(32) FMS_CASE(64)
#undef FMS_CASE
    }
    switch (Dw) {
#define FMS_CASE(DD)                                                                       \
    case DD:                                                                               \
        hipLaunchKernelGGL(assign_kernel<DD>, dim3(blocks), dim3(kT), 0, s, X, n, d, modes, \
                           k, labels, margin);                                             \
        break;
        FMS_CASE(1)
        FMS_CASE(2)
        FMS_CASE(3)
        FMS_CASE(4)
        FMS_CASE(8)
        FMS_CASE(16)
        FMS_CASE(32)
        FMS_CASE(64)
        FMS_CASE(128)
        FMS_CASE(256)
#undef FMS_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_check_finite(const float* X, long long count, int32_t* flag, hipStream_t s) {
    long long blocks = (count + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(check_finite_kernel, dim3((unsigned)blocks), dim3(256), 0, s, X, count,
                       flag);
    return hipGetLastError();
}

}  // namespace fms
