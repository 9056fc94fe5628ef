// k_adjoint_runs.hip -- the differentiable Gaussian update and its adjoint in
// FP32 over pivot runs (gfx950): the arithmetic of k_adjoint.hip on the pairs
// that can matter.
//
// The points and the seeds are grouped into runs around sampled pivots
// (k_runs.hip), 64 rows to a tile.  A workgroup holds one tile, a row per
// lane, and its eight waves stream the other side's tiles through wave-uniform
// (scalar) loads, tile by tile in turn; the wave sums are added in wave order.
// Every lane knows its distance from a run's centre and the run's radius, so a
// run is passed over when it is out of every lane's reach, and a row when half
// of its coordinates already put it there.  On the clouds of the batched
// recipe (D = 16, 2..40 clusters, h = 1) a tenth of the pairs remains; on data
// without clusters every pair does, at the price of the grouping.
//
// What is out of reach: weights that are exactly zero in FP32 (q >= 150, with
// q = |x - s|^2 in units of 2 h^2 / log2 e; the test uses 160), and weights
// below 2^-33 / n of the seed's sum W (n points).  The latter add up to at most
// 2^-33 W, where an FP32 sum rounds at 2^-25 W; in dL/dX they are terms below
// 2^-33 / n of the upstream gradient.  In the seed passes W is bounded from
// below by the nearest pivot, which is a point; the point pass has W itself.
//
// One pass over the pairs gives the update and dL/ds together: with
// dx = x - s and delta = sum w dx / W,
//     dL/ds = (sum w (g.dx) dx / W - (g.delta) delta) / h^2,
// the same sums as beta_ij = w_ij g.(x_i - s'_j) / (h^2 W_j) gives (see
// k_adjoint.hip), with s'_j left outside them.
//
// Bound by the vector units (D = 16: 54, 87 and 89 lane-ops a pair for the
// update, the seed pass and the point pass; all pairs of overlapping clusters at
// D = 3 run at 80 % of their rate).  8 clouds of 16,384 x 16, one call: update
// 2,050 -> 490 us, adjoint 8,600 -> 1,500 us, of which the index 75 us.

#include <algorithm>
#include <cmath>

#include "step_common.h"

namespace fms {

namespace {

constexpr int kT = 512;           // eight waves share a tile: short workgroups balance uneven runs
constexpr int kWv = kT / 64;
constexpr float kZeroQ = 160.0f;
constexpr float kDropped = 33.0f;
constexpr int kFoldTiles = 4;

// One side of the pairs: runs in cloud order (k_runs.hip).
struct Side {
    const float* rows;          // 64 rows of `ld` floats per tile
    int ld;
    const float* pivot_rows;    // stride DP
    const float* ball_rows;     // centre of each run (stride DP + 4), its radius at DP
    const float* run_bound;     // the far runs' bounds are used where this is not NULL
    const int32_t* tile_start;
    const int32_t* run_start;
    const int32_t* poff;
    const float* runq;          // per run: the largest q that counts (point pass), or NULL
};

struct AdjArgs {
    Side own, other;
    const int32_t* own_tile_run;
    const int32_t* own_rows;    // original row of each slot, -1: padding
    int own_runs, ncl, d;
    float c, scale, ih2;        // exp2(c |dx|^2); packed units per input unit; 1 / h^2
    float neg;                  // 33 + log2 n
    const float* G;
    float* out;                 // S_out; or dS / dX, added into
    float* sg;                  // seed pass: rows for the point pass (s, g, 1/W, -g.delta)
    float* runq;                // seed pass: the seed runs' largest q, as the float's bits
};

enum { FWD = 0, DS = 1, DX = 2 };

template <int D, int MODE>
__global__ __launch_bounds__(kT) void adj_runs_kernel(AdjArgs a) {
    constexpr int DP = D <= 4 ? 4 : D;
    constexpr int V = MODE == FWD ? D + 1 : (MODE == DS ? 2 * D + 1 : 2 * D);
    constexpr int VR = MODE == DX ? D : V;   // sums a wave passes on
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = blockIdx.x;
    if (tile >= a.own.tile_start[a.own_runs]) return;
    const int orun = a.own_tile_run[tile];
    const int c = upper_cloud_runs(a.own.poff, a.ncl, orun);
    const int p0 = __builtin_amdgcn_readfirstlane(a.other.poff[c]);
    const int P = __builtin_amdgcn_readfirstlane(a.other.poff[c + 1]) - p0;
    const int run0 = p0 + kFarRuns * __builtin_amdgcn_readfirstlane(c);

    const int row = a.own_rows[tile * 64 + lane];
    const bool live = row >= 0;
    float s[D], g[MODE == DS ? D : 1];
    const float* own = a.own.rows + (long long)(tile * 64 + lane) * a.own.ld;
#pragma unroll
    for (int k = 0; k < D; ++k) s[k] = live ? own[k] : 0.0f;
    if constexpr (MODE == DS) {
#pragma unroll
        for (int k = 0; k < D; ++k) g[k] = (live && k < a.d) ? a.G[(long long)row * a.d + k] : 0.0f;
    }

    constexpr int kGroups = (kRunPivotMax + kFarRuns + 63) / 64;
    constexpr bool kTileSums = D <= 8;
    __shared__ float red[(kTileSums ? kWv - 1 : kWv) * VR * 64];
    __shared__ float umin[kWv][64];
    __shared__ float wfirst_d[kWv];
    __shared__ int wfirst[kWv];
    __shared__ unsigned long long near_mask[kGroups];

    // distances (packed units) from rows of the other side, by lane
    auto dist_to = [&](const_f32_ptr p) {
        float q = 0.0f;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const float u = s[k] - p[k];
            q = fmaf(u, u, q);
        }
        return __builtin_amdgcn_sqrtf(q) * a.scale;
    };
    const const_f32_ptr pv = wave_uniform_const(a.other.pivot_rows);
    const const_f32_ptr bv = wave_uniform_const(a.other.ball_rows);
    const bool bounds = MODE != DX || a.other.run_bound != nullptr;
    // the nearest pivot (a point) of each lane, and the pivot nearest to any
    float ub = __builtin_inff(), first_d = 1e18f;
    int first = 0;
    for (int e = wave; bounds && e < P; e += kWv) {
        const float dist = dist_to(pv + (long long)(p0 + e) * DP);
        ub = fminf(ub, dist);
        if (MODE != DX) {
            const float m = lane_value(wave_min63(live ? dist : 1e18f), 63);
            if (m < first_d) {
                first_d = m;
                first = e;
            }
        }
    }
    umin[wave][lane] = ub;
    if (lane == 0) {
        wfirst[wave] = first;
        wfirst_d[wave] = first_d;
    }
    if (threadIdx.x < kGroups) near_mask[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWv; ++w) ub = fminf(ub, umin[w][lane]);
    first = 0;
    first_d = 1e18f;
    for (int w = 0; w < kWv; ++w)
        if (wfirst_d[w] < first_d) {
            first_d = wfirst_d[w];
            first = wfirst[w];
        }
    first = __builtin_amdgcn_readfirstlane(first);
    ub *= 1.001f;
    // seed passes: the largest q that counts for the lane's seed
    const float toraw = 1.0f / (a.scale * a.scale);
    float rq = fminf(kZeroQ, a.neg + ub * ub), reach = sqrtf(rq);
    // a cloud with a point that is not finite (in its last far run, whose bound
    // is then 0): none of its pairs is left out by half a distance
    const float least_q =
        MODE != DX && D >= 16 && a.other.run_bound[run0 + P + kFarRuns - 1] == 0.0f ? __builtin_inff() : 0.0f;
    float far_q = live ? fmaxf(rq * toraw, least_q) : -1.0f;

    // near: run e of this cloud is within some lane's reach
    auto is_near = [&](int e, float lim) {
        const const_f32_ptr p = bv + (long long)(run0 + e) * (DP + 4);
        bool near = !(dist_to(p) - p[DP] > lim);   // a NaN is near
        if (bounds && e >= P) near = near && !(a.other.run_bound[run0 + e] - ub > lim);
        return __ballot(near && live) != 0;
    };
    for (int e = wave; e < P + kFarRuns; e += kWv) {
        if (a.other.tile_start[run0 + e] == a.other.tile_start[run0 + e + 1]) continue;
        const float lim = MODE == DX ? sqrtf(a.other.runq[run0 + e]) : reach;
        if (is_near(e, lim) && lane == 0) atomicOr(&near_mask[e >> 6], 1ull << (e & 63));
    }
    __syncthreads();

    // narrow rows: each tile's 64 terms are summed apart and then added, which
    // keeps the chains short (at D = 3 a wave adds thousands of terms; dL/dX of
    // overlapping clusters was off by 1.1e-6 without and the all-pairs form by
    // 7.9e-7).  Wide rows: every kFoldTiles tiles the sums are added into the
    // wave's place in LDS (where points repeat, additions of equal terms all
    // round the same way: 16,384 x 8,192 pairs of seven points, D = 32, dL/dS
    // was off by 7.1e-6 and the all-pairs form by 2.5e-6)
    float acc[V], sum[kTileSums ? V : 1];
#pragma unroll
    for (int k = 0; k < V; ++k) acc[k] = 0.0f;
    if constexpr (kTileSums) {
#pragma unroll
        for (int k = 0; k < V; ++k) sum[k] = 0.0f;
    }
    float* const place = red + wave * VR * 64 + lane;   // wide rows
    float folded_W = 0.0f;
    int unfolded = 0;
    if constexpr (!kTileSums) {
#pragma unroll
        for (int k = 0; k < VR; ++k) place[k * 64] = 0.0f;
    }
    auto to_place = [&]() {
        if (MODE != DX) folded_W += acc[MODE != DX ? D : 0];
#pragma unroll
        for (int k = 0; k < VR; ++k) {
            place[k * 64] += MODE == DX ? fmaf(-a.ih2, acc[MODE == DX ? D + k : k], acc[k]) : acc[k];
            acc[k] = 0.0f;
            if (MODE == DX) acc[MODE == DX ? D + k : k] = 0.0f;
        }
        unfolded = 0;
    };
    auto fold = [&]() {
        if constexpr (kTileSums) {
#pragma unroll
            for (int k = 0; k < V; ++k) {
                sum[k] += acc[k];
                acc[k] = 0.0f;
            }
        } else if (++unfolded == kFoldTiles) {
            to_place();
        }
    };
    auto wave_W = [&]() {
        if constexpr (kTileSums && MODE != DX) return sum[D];
        else return folded_W + acc[MODE != DX ? D : 0];
    };
    int turn = 0;
    const const_f32_ptr rows = wave_uniform_const(a.other.rows);
    // one run: its tiles dealt to the waves in turn
    auto do_run = [&](int e) {
            const int t0 = __builtin_amdgcn_readfirstlane(a.other.tile_start[run0 + e]);
            const int t1 = __builtin_amdgcn_readfirstlane(a.other.tile_start[run0 + e + 1]);
            const int cnt = __builtin_amdgcn_readfirstlane(a.other.run_start[run0 + e + 1] - a.other.run_start[run0 + e]);
            const int w0 = t0 + ((wave - turn) & (kWv - 1));
            turn = (turn + t1 - t0) & (kWv - 1);
            if (w0 >= t1) return;
            if (MODE == DX) {
                far_q = live ? a.other.runq[run0 + e] * toraw : -1.0f;
            } else {
                // the wave's sum so far is a better bound of W than the nearest
                // pivot: fewer rows count, and perhaps none of this run
                const float better = a.neg + 0.01f - __builtin_amdgcn_logf(wave_W());
                if (__ballot(live && better < rq)) {
                    rq = fminf(rq, fmaxf(better, 1.0f));
                    reach = sqrtf(rq);
                    far_q = live ? fmaxf(rq * toraw, least_q) : -1.0f;
                    if (!is_near(e, reach)) return;
                }
            }
            for (int t = w0; t < t1; t += kWv) {
                const int n = min(64, cnt - (t - t0) * 64);
                const const_f32_ptr base = rows + (long long)t * 64 * a.other.ld;
                if constexpr (MODE != DX) {
                    stream_rows<D, DP>(base, n, [&](const float (&x)[D]) {
                        float dx[D], q = 0.0f;
                        constexpr int H = D >= 16 ? D / 2 : D;
#pragma unroll
                        for (int k = 0; k < H; ++k) {
                            dx[k] = x[k] - s[k];
                            q = fmaf(dx[k], dx[k], q);
                        }
                        if constexpr (H < D) {
                            if (!__ballot(!(q > far_q && q < 3e38f))) return;
#pragma unroll
                            for (int k = H; k < D; ++k) {
                                dx[k] = x[k] - s[k];
                                q = fmaf(dx[k], dx[k], q);
                            }
                        }
                        const float w = __builtin_amdgcn_exp2f(q * a.c);
                        acc[D] += w;
#pragma unroll
                        for (int k = 0; k < D; ++k) acc[k] = fmaf(w, dx[k], acc[k]);
                        if constexpr (MODE == DS) {
                            float gdx = 0.0f;
#pragma unroll
                            for (int k = 0; k < D; ++k) gdx = fmaf(g[k], dx[k], gdx);
                            const float wg = w * gdx;
#pragma unroll
                            for (int k = 0; k < D; ++k) acc[D + 1 + k] = fmaf(wg, dx[k], acc[D + 1 + k]);
                        }
                    });
                } else {
                    // a seed's row: s, g, 1 / W, -g.delta (wide rows: the next row's
                    // loads put ahead gained nothing, the vector units are busy)
                    constexpr int LD = 2 * DP + 4;
                    auto pair = [&](const float (&r)[LD]) {
                        float dx[D], q = 0.0f;
                        constexpr int H = D >= 16 ? D / 2 : D;
#pragma unroll
                        for (int k = 0; k < H; ++k) {
                            dx[k] = s[k] - r[k];
                            q = fmaf(dx[k], dx[k], q);
                        }
                        if constexpr (H < D) {
                            if (!__ballot(!(q > far_q && q < 3e38f))) return;
#pragma unroll
                            for (int k = H; k < D; ++k) {
                                dx[k] = s[k] - r[k];
                                q = fmaf(dx[k], dx[k], q);
                            }
                        }
                        float gdx = r[2 * DP + 1];   // -g.delta
#pragma unroll
                        for (int k = 0; k < D; ++k) gdx = fmaf(r[DP + k], dx[k], gdx);
                        const float w = __builtin_amdgcn_exp2f(q * a.c);
                        const float aa = w * r[2 * DP];   // w_ij / W_j
                        const float bb = aa * gdx;        // h^2 beta_ij
#pragma unroll
                        for (int k = 0; k < D; ++k) {
                            acc[k] = fmaf(aa, r[DP + k], acc[k]);
                            acc[D + k] = fmaf(bb, dx[k], acc[D + k]);
                        }
                    };
                    if constexpr (D <= 8) {
                        stream_rows<LD, LD>(base, n, pair);
                    } else {
                        for (int p = 0; p < n; ++p) {
                            float r[LD];
#pragma unroll
                            for (int k = 0; k < LD; ++k) r[k] = base[p * LD + k];
                            pair(r);
                        }
                    }
                }
                fold();
            }
    };
    // the listed runs, the one nearest to the tile first: W is soon known well
    const int groups = (P + kFarRuns + 63) / 64;
    int gi = -1;
    unsigned long long mk = 0;
    auto next = [&]() {
        for (;;) {
            while (!mk) {
                if (++gi >= groups) return -1;
                mk = (unsigned long long)wave_uniform((long long)near_mask[gi]);
            }
            const int e = gi * 64 + __builtin_ctzll(mk);
            mk &= mk - 1;
            if (e != first) return e;
        }
    };
    int e = -1;
    if (MODE != DX && ((near_mask[first >> 6] >> (first & 63)) & 1ull)) {
        e = first;
    } else {
        first = -1;
        e = next();
    }
    while (e >= 0) {
        do_run(e);
        e = next();
    }

    if constexpr (kTileSums) {
#pragma unroll
        for (int k = 0; k < V; ++k) acc[k] = sum[k];
        if constexpr (MODE == DX) {
#pragma unroll
            for (int k = 0; k < D; ++k) acc[k] = fmaf(-a.ih2, acc[D + k], acc[k]);
        }
        // the wave sums in wave order
        if (wave > 0) {
#pragma unroll
            for (int k = 0; k < VR; ++k) red[((wave - 1) * VR + k) * 64 + lane] = acc[k];
        }
    } else {
        to_place();
    }
    __syncthreads();
    if (wave > 0) return;
    // the last additions and the products of sums in FP64: they are few, and
    // sum w (g.dx) dx and (g.delta) delta cancel where delta is large
    auto tot = [&](int k) {
        double v = kTileSums ? acc[k] : 0.0f;
#pragma unroll
        for (int w = 0; w < (kTileSums ? kWv - 1 : kWv); ++w) v += red[(w * VR + k) * 64 + lane];
        return v;
    };
    if constexpr (MODE == DX) {
        if (!live) return;
#pragma unroll
        for (int k = 0; k < D; ++k)
            if (k < a.d) a.out[(long long)row * a.d + k] += (float)tot(k);
    } else {
        const double Wd = tot(D), iw = 1.0 / Wd;
        const float W = (float)Wd;
        if constexpr (MODE == FWD) {
            if (!live) return;
#pragma unroll
            for (int k = 0; k < D; ++k)
                if (k < a.d) a.out[(long long)row * a.d + k] = s[k] + (float)(tot(k) * iw);
        } else {
            double gdel = 0.0;
#pragma unroll
            for (int k = 0; k < D; ++k) gdel += g[k] * (tot(k) * iw);
            if (live) {
#pragma unroll
                for (int k = 0; k < D; ++k)
                    if (k < a.d)
                        a.out[(long long)row * a.d + k] +=
                            (float)(a.ih2 * ((tot(D + 1 + k) - gdel * tot(k)) * iw));
            }
            // the point pass reads the seeds' rows in this order; a padding row
            // weighs nothing
            float* o = a.sg + (long long)(tile * 64 + lane) * (2 * DP + 4);
#pragma unroll
            for (int k = 0; k < D; ++k) {
                o[k] = s[k];
                o[DP + k] = g[k];
            }
            o[2 * DP] = live ? (float)iw : 0.0f;
            o[2 * DP + 1] = live ? -(float)gdel : 0.0f;
            // a seed without weight (1/W not finite), or whose g.delta is not
            // finite, is seen by every point
            float q = 0.0f;
            if (live)
                q = (W > 0.0f && isfinite((float)iw) && isfinite((float)gdel))
                        ? fminf(kZeroQ, fmaxf(a.neg + 1.0f - __builtin_amdgcn_logf(W), 1.0f))
                        : __builtin_inff();
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) q = fmaxf(q, __shfl_xor(q, off));
            if (lane == 0) atomicMax(reinterpret_cast<int*>(a.runq) + orun, __float_as_int(q));
        }
    }
}

__global__ void zero_floats_kernel(float* a, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = 0.0f;
}

// Buffers of one call out of one block of memory (NULL: sizes only).
struct Bump {
    char* base;
    size_t off = 0;
    template <typename T>
    int alloc(T** out, size_t count) {
        *out = base ? reinterpret_cast<T*>(base + off) : nullptr;
        off += (std::max<size_t>(count * sizeof(T), 256) + 255) / 256 * 256;
        return 0;
    }
};

struct AdjBuffers {
    RunIndex x, s;   // s: the seeds' own index, the points' (same rows), or the points' order over the seeds' rows
    float *sg = nullptr, *runq = nullptr;
};

size_t carve_points(RunIndex& x, char* base, int nb, int n, int d) {
    Bump w{base};
    x.row_major = true;
    (void)run_index_alloc(x, run_sizes_equal(nb, n), d, true, [&](auto** p, size_t c) { return w.alloc(p, c); });
    return w.off;
}

// The points' index lies in `plan` or, if that is NULL, before the rest.
size_t carve_runs(AdjBuffers& b, char* base, char* plan, bool planned, int nb, int n, int m, int d, bool same,
                  bool adjoint) {
    const size_t own = carve_points(b.x, planned ? plan : base, nb, n, d);
    Bump w{base, planned ? 0 : own};
    auto alloc = [&](auto** p, size_t c) { return w.alloc(p, c); };
    b.s.row_major = true;
    if (m == n) {
        b.s = b.x;   // (its scale is set with b.x's)
        if (!same) {   // seeds that started from the points keep the points' order
            (void)w.alloc(&b.s.tiles, (size_t)b.x.sz.max_tiles * 64 * b.x.DP);
            (void)w.alloc(&b.s.ball_rows, (size_t)b.x.sz.runs * (b.x.DP + 4));
        }
    } else {
        (void)run_index_alloc(b.s, run_sizes_equal(nb, m), d, true, alloc);
    }
    if (adjoint) {
        (void)w.alloc(&b.sg, (size_t)b.s.sz.max_tiles * 64 * (2 * b.s.DP + 4));
        (void)w.alloc(&b.runq, (size_t)b.s.sz.runs);
    }
    return w.off;
}

Side side_of(const RunIndex& r) {
    return Side{r.tiles, r.DP, r.pivot_rows, r.ball_rows, r.run_bound, r.tile_start, r.run_start, r.poff, nullptr};
}

template <int D>
void launch_modes(const AdjArgs& seeds, const AdjArgs& points, bool adjoint, int stiles, int xtiles, hipStream_t s) {
    if (!adjoint) {
        hipLaunchKernelGGL((adj_runs_kernel<D, FWD>), dim3(stiles), dim3(kT), 0, s, seeds);
        return;
    }
    hipLaunchKernelGGL((adj_runs_kernel<D, DS>), dim3(stiles), dim3(kT), 0, s, seeds);
    hipLaunchKernelGGL((adj_runs_kernel<D, DX>), dim3(xtiles), dim3(kT), 0, s, points);
}

}  // namespace

// Where the runs are the better form.  A workgroup takes one tile of 64 rows and
// walks all of its near tiles, so they want many tiles on either side (few
// seeds: 60,000 x 2,500, D = 16, update and adjoint 2,490 us against 968 over
// all pairs), clouds that several runs divide (1,000 points: 1,135 and 903; 256
// points, 1,030 clouds: 26 ms and 1.0), and pairs enough to pay for the index.
// Update and adjoint over runs and over all pairs (k_adjoint.hip), us, clusters
// that mostly overlap at D <= 8:
//   D = 16: 8,192^2 562 / 383, 4 x 4,096^2 537 / 426, 8 x 4,096^2 687 / 746,
//           11,600^2 487 / 796, 64 x 2,100^2 1,286 / 1,398, 65,536 x 16,384 1,458 / 6,055
//   D = 32: 8,192^2 662 / 703, 4 x 4,096^2 647 / 711, 64 x 2,100^2 2,689 / 2,783
//   D = 8:  8 x 4,096^2 590 / 420, 16,384^2 1,353 / 842, 16 x 10,000 x 4,096 1,613 / 1,678
//   D = 3:  8 x 4,096^2 454 / 249, 16,384^2 998 / 514
// At D <= 8 reach is wide against such clouds and nothing is left out; the runs
// are kept for the larger clouds, where their sums by tiles are ten times closer
// (8 x 16,384^2, D = 3: 1.2e-7 and 1.2e-6 off) and where clouds that are wide
// against h gain (8 x 8,200^2, D = 3, centres 30 h apart: 570 and 1,708, two updates).
bool adjoint_runs_ok(int nb, int n, int m, int d, bool adjoint, bool planned) {
    if (d > 32) return false;
    if ((long long)nb * std::max(n, m) > (1LL << 28)) return false;   // tile slots stay in 32 bits
    const int D = step_shape(d).D, least = std::min(n, m);
    const long long pairs = (long long)nb * n * m;
    if (D <= 8) {
        // more seeds than points: few tiles of points with long lists (8,192 x
        // 20,000, D = 3: 829 over runs, 323 over all pairs)
        if (least < 8192 || m > n) return false;
    } else {
        if (least < 2048 || (long long)nb * least < 8192) return false;
    }
    // the update alone, without a plan: the index takes 60 to 100 us of it
    return pairs >= (D == 16 || !(adjoint || planned) ? 1LL << 27 : 1LL << 26);
}

size_t adjoint_runs_bytes(int nb, int n, int m, int d, bool same, bool adjoint, bool planned) {
    AdjBuffers b;
    return carve_runs(b, nullptr, nullptr, planned, nb, n, m, d, same, adjoint);
}

size_t points_plan_bytes(int nb, int n, int d) {
    RunIndex x;
    return carve_points(x, nullptr, nb, n, d);
}

static float packed(double h) { return (float)std::sqrt(1.4426950408889634 / (2.0 * h * h)); }

hipError_t launch_points_plan(const float* X, int nb, int n, int d, double h, void* plan, hipStream_t s) {
    RunIndex x;
    carve_points(x, (char*)plan, nb, n, d);
    return launch_run_index(x, X, nullptr, n, packed(h), 8.0f, s);
}

hipError_t launch_adjoint_runs(const float* X, int nb, int n, const float* S, int m, int d, double h, float* S_out,
                               const float* G, float* dS, float* dX, void* ws, const void* plan, hipStream_t s) {
    const bool same = S == X && m == n, adjoint = G != nullptr;
    AdjBuffers b;
    carve_runs(b, (char*)ws, (char*)const_cast<void*>(plan), plan != nullptr, nb, n, m, d, same, adjoint);
    const float scale = packed(h);
    hipError_t e = hipSuccess;
    b.x.scale = scale;
    if (!plan) e = launch_run_index(b.x, X, nullptr, n, scale, 8.0f, s);
    if (e != hipSuccess) return e;
    if (m == n && !same) {
        e = launch_run_regroup(b.x, S, b.s.tiles, b.s.ball_rows, s);
        b.s.run_bound = nullptr;
    } else if (m != n) {
        e = launch_run_index(b.s, S, nullptr, m, scale, 8.0f, s);
    }
    if (e != hipSuccess) return e;
    AdjArgs a{};
    a.own = side_of(b.s);
    a.other = side_of(b.x);
    a.own_tile_run = b.s.tile_run;
    a.own_rows = b.s.rows;
    a.own_runs = b.s.sz.runs;
    a.ncl = nb;
    a.d = d;
    a.c = (float)(-1.4426950408889634 / (2.0 * h * h));
    a.scale = scale;
    a.ih2 = (float)(1.0 / (h * h));
    a.neg = kDropped + (float)std::log2((double)n) + 0.01f;
    a.G = G;
    a.out = adjoint ? dS : S_out;
    a.sg = b.sg;
    a.runq = b.runq;
    AdjArgs p = a;
    if (adjoint) {
        hipLaunchKernelGGL(zero_floats_kernel, dim3((b.s.sz.runs + 255) / 256), dim3(256), 0, s, b.runq, b.s.sz.runs);
        p.own = side_of(b.x);
        p.other = side_of(b.s);
        p.other.rows = b.sg;
        p.other.ld = 2 * b.s.DP + 4;
        p.other.runq = b.runq;
        p.own_tile_run = b.x.tile_run;
        p.own_rows = b.x.rows;
        p.own_runs = b.x.sz.runs;
        p.out = dX;
    }
    const int st = b.s.sz.max_tiles, xt = b.x.sz.max_tiles;
    switch (b.x.D) {
        case 1: launch_modes<1>(a, p, adjoint, st, xt, s); break;
        case 2: launch_modes<2>(a, p, adjoint, st, xt, s); break;
        case 3: launch_modes<3>(a, p, adjoint, st, xt, s); break;
        case 4: launch_modes<4>(a, p, adjoint, st, xt, s); break;
        case 8: launch_modes<8>(a, p, adjoint, st, xt, s); break;
        case 16: launch_modes<16>(a, p, adjoint, st, xt, s); break;
        case 32: launch_modes<32>(a, p, adjoint, st, xt, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace fms
