// k_seed.hip -- the FP32 update with a workgroup per seed (or per few seeds)
// that runs all of the seeds' iterations in one launch (gfx950).
//
// The update of Section II-B has no exchange between seeds: a seed's next
// position needs the points and its own position only.  So a workgroup owns R
// seeds, keeps them in registers, and iterates until they converge (Algorithms
// 1-2, "while not converge") or max_iter updates are done.  Nothing leaves the
// workgroup between two updates: no partial sums in memory, no reduction or
// compaction launch, no host poll.  Only a batch that stops early on its
// converged count (Section II-C with gamma < 1) needs all seeds in step; it
// takes the forms that launch per iteration.
//
// Lanes hold POINTS and the seed is wave-uniform (scalar registers), the
// reverse of the seed-tile forms.  Points come as tiles of 64 (one per lane),
// coordinates in float4 groups: tile t, group g, lane l at
// ((t * D/4 + g) * 64 + l) * 4, so that every load is 1 KB contiguous.  With a
// ball (centre, radius) per tile, each wave tests 64 tiles at once (lane =
// tile) and walks the set bits of the ballot: a seed evaluates only the tiles
// within its own reach, where a 64-seed tile evaluates the union of 64
// seeds' tiles.  In the fit of 200,000 x 3-D points that is 3.3 % of the pairs
// instead of 35 %.  The near tiles are neighbours in the spatial order, so the
// workgroup lists them in LDS first and its waves take the entries in turn.
//
// The tiles come in one of two orders.
//   Rows (d <= 4): the packed rows as they are (few points: every tile is
//     evaluated), or in Morton order with a ball per tile.
//   Runs (k_runs.hip; every d up to 32, one cloud or many): runs of tiles
//     around sampled pivots.  The ball of a run is its pivot and its farthest
//     point; a run of points far from every pivot has a lower bound of that
//     distance, and a seed within u of some pivot sees none of its points
//     closer than the bound minus u.
//
// What a tile may be left out for (the Gaussian): every pair of it is beyond
// the distance where the FP32 weight is exactly zero (q >= 150; the test uses
// 160), or has a weight below 2^-33 / n of the seed's weight sum W.  At most n
// such terms are dropped, in total below 2^-33 W, where an FP32 sum rounds at
// 2^-25 W.  W is bounded from below without any sum: a ball of
// radius r at distance c holds a point within c + r (a pivot is a point
// itself), so W >= 2^-(c + r)^2 for the nearest one; after the first update
// the W of the previous one serves (a mean-shift step never lowers the
// density).  The flat window leaves out the tiles wholly outside it.
//
// With the list made beforehand the tiles' loads run ahead of the arithmetic
// with no test between them.  The waves test consecutive groups of 64 balls
// (contiguous loads; with the tiles dealt to the waves one by one a pass over
// 3,125 balls took 7 us instead of 2).  The list is kept while the seeds stay
// within a slack of where it was made, the reach being that much longer; late
// iterations move far less and skip the geometry.
//
// The lane sums are added by fixed DPP steps, the waves' sums in wave order:
// no floating-point atomics, the same result on every run.

#include <algorithm>

#include "step_common.h"

namespace fms {

namespace {

constexpr float kSeedZero = 160.0f;      // exp2(-q) == +0 in FP32 for q >= 150
constexpr float kSeedDropped = 33.0f;    // the terms left out are below 2^-33 of the sum in all
constexpr float kSeedFlatMargin = 1.001f;
constexpr float kSlack = 0.25f;          // packed units
constexpr int kSegGroups = 96;           // groups of 64 tiles listed at once (24 KB: six workgroups a CU)
constexpr int kSeedMaxWaves = 16;
// waves per SIMD the register count must allow
constexpr int seed_min_waves(int D) { return D >= 16 ? 3 : 4; }
constexpr int kXcdRun = 64;
// Workgroups of one launch: fewer than 2^32 threads, with at most 16 waves each.
constexpr int kSeedLaunch = 1 << 21;
// wide rows need the registers that 16 waves in one workgroup would not have
constexpr int seed_max_waves(int D, int R) { return D <= 4 && R == 1 ? kSeedMaxWaves : 8; }

// LDS of a seed's list over runs: masks, entries, counts, pivot distances.
__host__ __device__ constexpr size_t run_lds(int cap) { return ((size_t)cap / 64 * 8 + (size_t)cap * 12 + 16 + 15) / 16 * 16; }

// PW: every wave of a workgroup has a seed of its own (and a list), instead of
// a share of one seed's tiles.  Where seeds reach an eighth of the tiles and
// more, all these reads through L2 bound the update; waves that walk nearly the
// same list at nearly the same time find them in L1.  262,144 x 32-D points,
// seeds sharing and own, us: 2 clusters, 8,192 seeds, three updates 45,000 and
// 14,900; 7 clusters, 4,000 seeds, two 3,300 and 2,000; 80 clusters, 8,192
// seeds, three 1,100 and 1,900.  Registers for two waves a SIMD: with three,
// 250 bytes of scratch a lane and 15,500.
constexpr int kOwnWaves = 4;

// A lane adds at most this many tiles in a row; then its sums go to a second
// set.  Where points repeat (quantised data), additions of equal terms all
// round the same way, and the error grows with their number: one update of
// seeds that see 1,108 tiles of seven different points was off by 8e-6 h, and
// is by 2e-7 h now.  The second set is V registers a lane.  At D = 32 three
// waves a SIMD leave none: there it is sums over rows of 16 lanes (`rows4`) in
// LDS, 2.3 KB a wave (262,144 points, 2 clusters, 700 seeds, three updates:
// 3,400 us without it, 3,700 in registers that spill, 3,260 so).  At D = 8 the
// rows cost 9 % (8,192 seeds of 4,000 near points each), the registers 1 %.
constexpr int kFoldTiles = 32;
__host__ __device__ constexpr bool fold_rows(int D, bool PW) { return D == 32 && !PW; }
__host__ __device__ constexpr int fold_quads(int D) { return (D + 4) / 4; }

template <int D, int R, int KERN, bool RUNS, bool PW>
__global__ __launch_bounds__(64 * seed_max_waves(D, R), PW ? 2 : seed_min_waves(D)) void seed_iterate_kernel(SeedArgs a) {
    constexpr int DP = D <= 4 ? 4 : D;
    constexpr int G4 = DP / 4;
    constexpr int V = D + 1;
    constexpr bool kFoldRows = fold_rows(D, PW);
    constexpr int kFoldQuads = fold_quads(D);
    static_assert(!kFoldRows || R == 1);
    constexpr int NWMAX = seed_max_waves(D, R);
    static_assert(R * DP <= 64, "one wave holds the coordinates of the seeds");
    const int lane = threadIdx.x & 63;
    const int hwave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = PW ? 0 : hwave;
    const int NW = PW ? 1 : blockDim.x >> 6;
    static_assert(!PW || RUNS, "a seed per wave: runs only");
    // the waves that share a seed wait for each other
    auto sync = [&] {
        if constexpr (PW) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    };

    if (RUNS && a.dense && (kDensePart * a.dense[0] > a.dense[1]) != PW) return;

    // this workgroup's seeds and its cloud's tiles.  Workgroups are dealt to
    // the eight XCDs in turn; an XCD takes kXcdRun seed groups in a row, so
    // that seeds that are close (or in one cloud) read their tiles through one
    // L2, from the end of the order: the seeds far from every pivot come last
    // in it and see every far tile, so they start first and on all XCDs.
    const int xi = (int)blockIdx.x >> 3;
    const int wg = a.wgs - 1 - (((xi / kXcdRun) * 8 + ((int)blockIdx.x & 7)) * kXcdRun + xi % kXcdRun);
    if (wg < 0) return;
    const int j0 = PW ? (a.wg0 + wg) * (int)(blockDim.x >> 6) + hwave : (a.wg0 + wg) * R;
    if (PW && j0 >= a.m) return;
    // rows: tiles [0, nball), a ball each; runs: the cloud's pivots
    // [ball0, ball0 + nball), whose runs start at run0
    int ball0 = 0, nball = a.tiles, run0 = 0;
    if constexpr (RUNS) {
        const int c = a.seg ? upper_cloud(a.seg, a.ncl, j0) : 0;
        ball0 = __builtin_amdgcn_readfirstlane(a.poff[c]);
        nball = __builtin_amdgcn_readfirstlane(a.poff[c + 1]) - ball0;
        run0 = ball0 + kFarRuns * __builtin_amdgcn_readfirstlane(c);
    }
    const bool culled = RUNS || a.geom != nullptr;

    __shared__ float red[2][NWMAX][R * V];
    __shared__ float wub[R][NWMAX];
    __shared__ unsigned wcnt[NWMAX];
    // rows: `list` holds tiles.  Runs: `list` holds the first tile of each
    // listed run and `list_pre` the tiles listed before it; a lower bound of a
    // seed's distance from every pivot stays in `dist_s`.  The top bits of an entry say which of
    // the R seeds reach it.
    // (Runs: sized by the largest cloud, so that many small clouds' workgroups
    // fit a CU.)
    __shared__ unsigned rows_list[RUNS ? 1 : kSegGroups * 64];
    __shared__ unsigned long long rows_mask[RUNS ? 1 : kSegGroups];
    __shared__ unsigned char near_who[RUNS || R == 1 ? 1 : kSegGroups * 64];
    extern __shared__ __attribute__((aligned(16))) unsigned long long dyn[];
    static_assert(!RUNS || R == 1, "runs: one seed per workgroup");
    const int cap = a.run_cap;   // whole groups
    unsigned long long* const dyn_s = dyn + (PW ? hwave * (int)(run_lds(cap) / 8) : 0);
    unsigned long long* const near_mask = RUNS ? dyn_s : rows_mask;
    unsigned* const list = RUNS ? reinterpret_cast<unsigned*>(dyn_s + cap / 64) : rows_list;
    int* const list_pre = reinterpret_cast<int*>(list + cap);   // cap + 1
    float* const dist_s = reinterpret_cast<float*>(list_pre + cap + 1);
    float* const folded_s = reinterpret_cast<float*>(dyn) + (RUNS ? run_lds(cap) / 4 : 0) + hwave * kFoldQuads * 64 + lane;

    // lane (r, k) holds coordinate k of seed r, in every wave
    const int r_of = lane / DP, k_of = lane % DP;
    int id[R];
    unsigned act = 0;   // bit r: seed r still iterates
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int slot = j0 + r;
        id[r] = -1;
        if (slot < a.m) {
            id[r] = __builtin_amdgcn_readfirstlane(a.order ? a.order[slot] : slot);
            if (a.status[id[r]] == ST_ACTIVE) act |= 1u << r;
        }
    }
    act = __builtin_amdgcn_readfirstlane(act);
    if (!act) return;
    float sv = 0.0f;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r_of == r && id[r] >= 0) sv = a.S[(long long)id[r] * DP + k_of];

    // Ball g * 64 + l is lane l of group g.  A segment is as many groups as fit
    // the list; with one segment (always, for runs) the list may be kept from
    // one update to the next.
    const int groups = (nball + 63) / 64;
    const bool keep = RUNS || groups <= kSegGroups;
    int points = nball * 64;
    if constexpr (RUNS) points = (a.tile_start[run0 + nball + kFarRuns] - a.tile_start[run0]) * 64;
    // A cloud with a point that is not finite (or overflows) has it in its last
    // far run, whose bound is then 0: every seed of the cloud fails by it, also
    // by a coordinate that the first half of a distance does not hold
    bool whole = false;
    if constexpr (RUNS && D >= 16) whole = a.run_bound[run0 + nball + kFarRuns - 1] == 0.0f;
    const float negligible = kSeedDropped + __builtin_amdgcn_logf((float)points) + 0.01f;
    const float4* __restrict__ T4 = reinterpret_cast<const float4*>(a.T);

    float reach[R], rq[R], wprev[R], last_sh2[R];   // reach and its square
    float ub[R];             // some point (runs: some pivot) lies within ub
    int nit[R];
    int result[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        reach[r] = 0.0f;
        rq[r] = __builtin_inff();   // nothing is left out without geometry
        ub[r] = __builtin_inff();
        wprev[r] = -1.0f;
        last_sh2[r] = __builtin_nanf("");
        nit[r] = 0;
        result[r] = ST_ACTIVE;
    }
    float sref = 0.0f;       // where the masks were made
    bool have_list = false;
    int len = 0;             // listed tiles
    int nlisted = 0;         // listed runs
    unsigned evaluated = 0;  // tiles this wave evaluated, over seeds and iterations
    int executed = 0;        // updates run, over the seeds

    int it = 0;
    for (; it < a.max_iter && act; ++it) {
        const float svs = sv * a.scale;
        float s[R][D];   // wave-uniform: scalar registers
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int k = 0; k < D; ++k) s[r][k] = lane_value(svs, r * DP + k);

        // f(g, r, inside, distance of seed r from the ball's centre, radius)
        // for the lane's ball of this wave's groups g0 + wave, + NW, ... < g1,
        // several groups' loads at once
        auto balls = [&](int g0, int g1, auto&& f) {
            constexpr int B = D <= 4 ? 4 : (D <= 16 ? 2 : 1);
#pragma unroll 1
            for (int g = g0 + wave; g < g1; g += B * NW) {
                float c[B][D], rad[B];
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    const int e = (g + i * NW) * 64 + lane;
                    const int t = ball0 + (e < nball ? e : 0);
#pragma unroll
                    for (int k = 0; k < D; ++k) c[i][k] = a.geom[(long long)k * a.geom_ld + t];
                    rad[i] = RUNS ? 0.0f : a.geom[(long long)D * a.geom_ld + t];
                }
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    if (g + i * NW < g1) {
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            float d2 = 0.0f;
#pragma unroll
                            for (int k = 0; k < D; ++k) {
                                const float u = s[r][k] - c[i][k];
                                d2 = fmaf(u, u, d2);
                            }
                            f(g + i * NW, r, (g + i * NW) * 64 + lane < nball, __builtin_amdgcn_sqrtf(d2), rad[i]);
                        }
                    }
                }
            }
        };

        bool remake = culled;
        if (remake && have_list) {
            float d2 = sv - sref;
            d2 = d2 * d2;
#pragma unroll
            for (int off = DP / 2; off >= 1; off >>= 1) d2 += __shfl_xor(d2, off);
            const float moved = sqrtf(d2) * a.scale;
            const bool far = !(moved <= a.slack) && ((act >> r_of) & 1u);
            remake = __ballot(far) != 0;
        }
        if (remake) {
            float moved[R];   // since the last list
            if (RUNS && it > 0) {
                float d2 = (sv - sref) * a.scale;
                d2 = d2 * d2;
#pragma unroll
                for (int off = DP / 2; off >= 1; off >>= 1) d2 += __shfl_xor(d2, off);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    moved[r] = 1.001f * sqrtf(lane_value(d2, r * DP));
                    ub[r] += moved[r];
                }
            }
            sref = sv;
            const bool by_row = RUNS && it == 0 && a.pnear != nullptr;
            if (by_row) {
#pragma unroll
                for (int r = 0; r < R; ++r) ub[r] = id[r] >= 0 ? a.pdist[id[r]] : 0.0f;
            }
            if (RUNS) sync();   // the last list is no longer read
            if (it == 0 && !by_row && (RUNS || KERN == MS_KERNEL_GAUSSIAN)) {
                balls(0, groups, [&](int g, int r, bool in, float dist, float rad) {
                    if (in) {
                        ub[r] = fminf(ub[r], dist + rad);   // a NaN never lowers it
                        if (RUNS) dist_s[g * 64 + lane] = dist;
                    }
                });
#pragma unroll
                for (int r = 0; r < R; ++r) {
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) ub[r] = fminf(ub[r], __shfl_xor(ub[r], off));
                    if (lane == 0) wub[r][hwave] = ub[r];
                }
                sync();
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    float u = wub[r][PW ? hwave : 0];
                    for (int w = 1; w < NW; ++w) u = fminf(u, wub[r][w]);
                    ub[r] = 1.001f * u;
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (KERN == MS_KERNEL_GAUSSIAN) {
                    // -log2 W, at most (1 of margin on the previous update's)
                    const float q = it == 0 ? ub[r] * ub[r] : 1.0f - __builtin_amdgcn_logf(wprev[r]);
                    rq[r] = fminf(kSeedZero, fmaxf(negligible + q, 1.0f));
                    reach[r] = sqrtf(rq[r]);
                } else {
                    reach[r] = a.flat_reach;
                    rq[r] = reach[r] * reach[r];
                }
                if (whole) rq[r] = __builtin_inff();
            }
            if constexpr (RUNS) {
                // near runs by their balls, far runs by their bounds.  A
                // pivot's distance is computed again only where the bound from
                // the last list, or from the seed's nearest pivot
                // (|s - p| >= |p' - p| - |s - p'|), does not rule it out: all
                // 1,024 distances of 8,192 seeds at D = 32 read 1 GB and took
                // 107 us a pass
                auto test = [&](int e, float bound) {
                    unsigned who = 0;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float lim = reach[r] + a.slack;
                        bool out;
                        if (e < nball) {
                            float l;
                            float& kept = dist_s[e];
                            if (by_row) l = id[r] >= 0 ? a.ppair[(long long)a.pnear[id[r]] * nball + e] - ub[r] : 0.0f;
                            else l = kept - (it > 0 ? moved[r] : 0.0f);
                            if ((by_row || it > 0) && !(l - bound > lim)) {
                                float d2 = 0.0f;
#pragma unroll
                                for (int k = 0; k < D; ++k) {
                                    const float u = s[r][k] - a.geom[(long long)k * a.geom_ld + ball0 + e];
                                    d2 = fmaf(u, u, d2);
                                }
                                l = __builtin_amdgcn_sqrtf(d2);
                            }
                            kept = l;
                            out = l - bound > lim;   // a NaN is near
                        } else {
                            out = bound - ub[r] > lim;
                        }
                        who |= (!out && ((act >> r) & 1u)) ? 1u << r : 0u;
                    }
                    return who;
                };
                const int nrun = nball + kFarRuns;
                const int rgroups = (nrun + 63) / 64;
#pragma unroll 1
                for (int g = wave; g < rgroups; g += NW) {
                    const int e = g * 64 + lane;
                    unsigned who = 0;
                    if (e < nrun) who = test(e, a.run_bound[run0 + e]);
                    if (e < nrun && a.tile_start[run0 + e] == a.tile_start[run0 + e + 1]) who = 0;
                    const unsigned long long mk = __ballot(who != 0);
                    if (lane == 0) near_mask[g] = mk;
                }
                sync();
                // entries before each group, then the entries with their tiles
                // counted in run order
                int before = 0;
                const int gc = lane < rgroups ? __popcll(near_mask[lane]) : 0;
                int x = gc;
#pragma unroll
                for (int off = 1; off < 32; off <<= 1) {
                    const int y = __shfl_up(x, off);
                    if (lane >= off) x += y;
                }
                before = x - gc;
                const int nlist = __builtin_amdgcn_readlane(x, 31);
#pragma unroll 1
                for (int g = wave; g < rgroups; g += NW) {
                    const unsigned long long mk = (unsigned long long)wave_uniform((long long)near_mask[g]);
                    const int at = __builtin_amdgcn_readlane(before, g);
                    if ((mk >> lane) & 1ull) {
                        const int e = g * 64 + lane, q = at + __popcll(mk & ((1ull << lane) - 1ull));
                        const int t = a.tile_start[run0 + e];
                        list[q] = (unsigned)t;
                        list_pre[q] = a.tile_start[run0 + e + 1] - t;
                    }
                }
                sync();
                // prefix of the listed runs' tiles, by wave 0
                if (wave == 0) {
                    int total = 0;
                    for (int q0 = 0; q0 < nlist; q0 += 64) {
                        const int c = q0 + lane < nlist ? list_pre[q0 + lane] : 0;
                        int v = c;
#pragma unroll
                        for (int off = 1; off < 64; off <<= 1) {
                            const int y = __shfl_up(v, off);
                            if (lane >= off) v += y;
                        }
                        if (q0 + lane < nlist) list_pre[q0 + lane] = total + v - c;
                        total += __builtin_amdgcn_readlane(v, 63);
                    }
                    if (lane == 0) list_pre[nlist] = total;
                }
                sync();
                nlisted = nlist;
                len = __builtin_amdgcn_readfirstlane(list_pre[nlist]);
            }
            have_list = keep;
        }

        float acc[R][V];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int k = 0; k < V; ++k) acc[r][k] = 0.0f;
        float sum[kFoldRows ? 1 : R][kFoldRows ? 1 : V];
        if constexpr (kFoldRows) {
#pragma unroll
            for (int q = 0; q < kFoldQuads; ++q) folded_s[q * 64] = 0.0f;
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int k = 0; k < V; ++k) sum[r][k] = 0.0f;
        }
        int run = 0;   // tiles since the last fold, at most
        auto fold = [&] {
            if constexpr (kFoldRows) {
                auto take = [&](int k) {
                    if (k >= V) return 0.0f;
                    const float v = acc[0][k];
                    acc[0][k] = 0.0f;
                    return v;
                };
#pragma unroll
                for (int q = 0; q < kFoldQuads; ++q) {
                    const float v0 = take(4 * q), v1 = take(4 * q + 1), v2 = take(4 * q + 2), v3 = take(4 * q + 3);
                    folded_s[q * 64] += rows4(v0, v1, v2, v3);
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int k = 0; k < V; ++k) {
                        sum[r][k] += acc[r][k];
                        acc[r][k] = 0.0f;
                    }
            }
            run = 0;
        };

        for (int g0 = 0; g0 < (RUNS ? 1 : groups); g0 += kSegGroups) {
            if constexpr (!RUNS) {
                const int g1 = min(groups, g0 + kSegGroups);
                if (remake) {
                    unsigned who = 0;   // seeds that reach the lane's tile
                    sync();   // the last list and its masks are no longer read
                    balls(g0, g1, [&](int g, int r, bool in, float dist, float rad) {
                        // a NaN (a ball without a finite centre) stays near
                        const bool near = in && !(dist - rad > reach[r] + (keep ? a.slack : 0.0f));
                        who = (r == 0 ? 0u : who) | ((near && ((act >> r) & 1u)) ? 1u << r : 0u);
                        if (r == R - 1) {
                            const unsigned long long mk = __ballot(who != 0);
                            if (lane == 0) near_mask[g - g0] = mk;
                            if (R > 1) near_who[(g - g0) * 64 + lane] = (unsigned char)who;
                        }
                    });
                    sync();
                    // entries before each group: a scan of the groups' counts
                    int before[(kSegGroups + 63) / 64];
                    len = 0;
#pragma unroll
                    for (int q = 0; q < (kSegGroups + 63) / 64; ++q) {
                        const int gi = q * 64 + lane;
                        const int cnt = gi < g1 - g0 ? __popcll(near_mask[gi]) : 0;
                        int x = cnt;
#pragma unroll
                        for (int off = 1; off < 64; off <<= 1) {
                            const int y = __shfl_up(x, off);
                            if (lane >= off) x += y;
                        }
                        before[q] = len + x - cnt;
                        len += __builtin_amdgcn_readlane(x, 63);
                    }
                    for (int gi = wave; gi < g1 - g0; gi += NW) {
                        const unsigned long long mk = (unsigned long long)wave_uniform((long long)near_mask[gi]);
                        if (!mk) continue;
                        const int at = __builtin_amdgcn_readlane(gi < 64 ? before[0] : before[1], gi & 63);
                        if ((mk >> lane) & 1ull)
                            list[at + __popcll(mk & ((1ull << lane) - 1ull))] =
                                (unsigned)((g0 + gi) * 64 + lane) |
                                (R > 1 ? (unsigned)near_who[gi * 64 + lane] << 28 : 0u);
                    }
                    sync();
                } else if (!culled) {
                    len = min((g1 - g0) * 64, nball - g0 * 64);
                }
            }
            // this wave's entries: wave, wave + NW, ...
            const int mine_n = len > wave ? (len - wave + NW - 1) / NW : 0;
            if (mine_n == 0) continue;
            evaluated += mine_n;
            // walk the tiles in batches of U, the next batch's loads in flight
            // while one computes; lane i of `ids` holds entry i of the current 64
            constexpr int U = D <= 8 ? 4 : (D <= 16 ? 2 : 1);
            float4 xa[U][G4], xb[U][G4];
            unsigned wa[U], wb[U];
            unsigned ids = 0;
            int next = 0;
            auto fetch = [&](float4 (&x)[U][G4], unsigned (&who)[U]) {
                const int cnt = min(U, mine_n - next);
                if ((next & 63) == 0) {
                    const int e = (next + lane < mine_n ? next + lane : 0) * NW + wave;
                    if constexpr (RUNS) {
                        // the listed run that holds tile e
                        int lo = 0, hi = nlisted;
                        while (hi - lo > 1) {
                            const int mid = (lo + hi) >> 1;
                            if (list_pre[mid] <= e) lo = mid;
                            else hi = mid;
                        }
                        ids = list[lo] + (unsigned)(e - list_pre[lo]);
                    } else {
                        ids = culled ? list[e] : (unsigned)(g0 * 64 + e);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    // past the end: the last entry again, not used
                    const int e = (next + u < mine_n ? next + u : mine_n - 1) & 63;
                    const unsigned v = (unsigned)__builtin_amdgcn_readlane((int)ids, e);
                    who[u] = (R > 1 && culled) ? v >> 28 : (1u << R) - 1u;
                    const long long t = (R > 1 && culled) ? (v & 0x0fffffffu) : v;
#pragma unroll
                    for (int q = 0; q < G4; ++q) x[u][q] = T4[(t * G4 + q) * 64 + lane];
                }
                next += U;
                return cnt;
            };
            auto compute = [&](const float4 (&xv)[U][G4], const unsigned (&who)[U], int cnt) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (u >= cnt) break;
                    float x[DP];
#pragma unroll
                    for (int q = 0; q < G4; ++q) {
                        x[4 * q] = xv[u][q].x;
                        x[4 * q + 1] = xv[u][q].y;
                        x[4 * q + 2] = xv[u][q].z;
                        x[4 * q + 3] = xv[u][q].w;
                    }
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        if (R > 1 && !((who[u] & act) >> r & 1u)) continue;
                        float dx[D];
                        float q = 0.0f;
                        constexpr int H = D >= 16 ? D / 2 : D;
#pragma unroll
                        for (int k = 0; k < H; ++k) {
                            dx[k] = x[k] - s[r][k];
                            q = fmaf(dx[k], dx[k], q);
                        }
                        if constexpr (H < D) {
                            // half the coordinates put every point of most far
                            // tiles beyond the reach (a coordinate that is not
                            // finite does not: it fails the seed)
                            if (!__ballot(!(q > rq[r] && q < 3e38f))) continue;
#pragma unroll
                            for (int k = H; k < D; ++k) {
                                dx[k] = x[k] - s[r][k];
                                q = fmaf(dx[k], dx[k], q);
                            }
                        }
                        if constexpr (D >= 8) {
                            if (!__ballot(!(q > rq[r] && q < 3e38f))) continue;
                        }
                        float w;
                        if (KERN == MS_KERNEL_GAUSSIAN)
                            w = __builtin_amdgcn_exp2f(-q);
                        else
                            w = (q <= a.h2) ? 1.0f : 0.0f;
                        acc[r][D] += w;
#pragma unroll
                        for (int k = 0; k < D; ++k) acc[r][k] = fmaf(w, dx[k], acc[r][k]);
                    }
                }
            };
            int na = fetch(xa, wa);
            for (;;) {
                int nb = 0;
                if (next < mine_n) nb = fetch(xb, wb);
                compute(xa, wa, na);
                if (!nb) break;
                na = 0;
                if (next < mine_n) na = fetch(xa, wa);
                compute(xb, wb, nb);
                if (!na) break;
                if ((run += 2 * U) >= kFoldTiles) fold();
            }
            run += 2 * U;
        }

        // lanes, then waves in order; every wave makes the same update
        const int par = it & 1;
        if constexpr (kFoldRows) {
            fold();
#pragma unroll
            for (int q = 0; q < kFoldQuads; ++q) {
                float t = folded_s[q * 64];
                t = dpp_add<0x128, 0xf>(t);   // row_ror:8
                t = dpp_add<0x124, 0xf>(t);
                t = dpp_add<0x122, 0xf>(t);
                t = dpp_add<0x121, 0xf>(t);
                const int k = 4 * q + rows4_value(lane);
                if ((lane & 15) == 0 && k < V) red[par][hwave][k] = t;
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    const float v = wave_add63(sum[r][k] + acc[r][k]);
                    if (lane == 63) red[par][hwave][r * V + k] = v;
                }
        }
        sync();
        float v = 0.0f, W = 0.0f;
        if (r_of < R) {
            for (int w = 0; w < NW; ++w) {
                if (k_of < D) v += red[par][PW ? hwave : w][r_of * V + k_of];
                W += red[par][PW ? hwave : w][r_of * V + D];
            }
        }
        const bool okW = W > 0.0f && isfinite(W);
        const float inv = a.inv_scale / W;
        float ns, dk;
        if (a.metric == MS_METRIC_COSINE) {
            const float u = sv + v * inv;
            float nn = u * u;
#pragma unroll
            for (int off = DP / 2; off >= 1; off >>= 1) nn += __shfl_xor(nn, off);
            const float rn = 1.0f / sqrtf(nn);
            ns = u * rn;
            dk = ns - sv;
            if (!(nn > 0.0f) || !isfinite(rn)) dk = __builtin_nanf("");
        } else {
            dk = v * inv;
            ns = sv + dk;
        }
        float sh2 = dk * dk;
#pragma unroll
        for (int off = DP / 2; off >= 1; off >>= 1) sh2 += __shfl_xor(sh2, off);
        // a non-finite coordinate makes the sum of squares non-finite; a sum
        // that only overflows is told apart by the coordinates themselves
        const unsigned long long bad = __ballot(r_of < R && k_of < D && !(isfinite(dk) && isfinite(ns)));
        bool mine = false;   // this lane's seed takes its new position
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (!((act >> r) & 1u)) continue;
            const float Wr = lane_value(W, r * DP);
            const float shr = lane_value(sh2, r * DP);
            ++executed;
            if (!(Wr > 0.0f) || !isfinite(Wr)) {
                result[r] = ST_FAILED;
                act &= ~(1u << r);
                continue;
            }
            mine = mine || r_of == r;
            ++nit[r];
            last_sh2[r] = shr;
            wprev[r] = Wr;
            const unsigned long long lanes = ((DP == 64 ? 0ull : (1ull << DP)) - 1ull) << (r * DP);
            if (bad & lanes) {
                result[r] = ST_FAILED;
                act &= ~(1u << r);
            } else if (shr < a.thr2) {
                result[r] = ST_CONVERGED;
                act &= ~(1u << r);
                if (a.ctl && wave == 0 && lane == 0) atomicAdd(&a.ctl->conv_it[it], 1);
            }
        }
        if (mine && okW) sv = ns;
    }

    // the output pointers are read from the argument block here, so that they
    // hold no scalar registers during the iterations
    auto* ka = (const __attribute__((address_space(4))) SeedArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ka));
    if (wave == 0) {
        float* S = ka->S;
        int32_t* iters = ka->iters;
        float* shift2 = ka->shift2;
        uint8_t* status = ka->status;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (id[r] < 0) continue;
            if (r_of == r && nit[r] > 0) S[(long long)id[r] * DP + k_of] = sv;
            if (lane == 0) {
                if (nit[r] > 0) {
                    iters[id[r]] += nit[r];
                    shift2[id[r]] = last_sh2[r];
                }
                if (result[r] != ST_ACTIVE) status[id[r]] = (uint8_t)result[r];
            }
        }
    }
    Ctl* ctl = ka->ctl;
    if (ctl) {
        if (lane == 0) wcnt[hwave] = evaluated;
        sync();
        if (wave == 0 && lane == 0) {
            unsigned long long e = 0;
            for (int w = 0; w < NW; ++w) e += wcnt[PW ? hwave : w];
            atomicMax(&ctl->iters_run, it);
            atomicAdd((unsigned long long*)&ctl->pairs, (unsigned long long)executed * (unsigned long long)ka->n);
            if (ka->count_exact)
                atomicAdd((unsigned long long*)&ctl->refined[(blockIdx.x % kRefinedSlots) * kRefinedStride],
                          e * 64ull);
        }
    }
}

// Points of 64-point tiles, D <= 4: ball of each tile (midpoint of the bounding
// box, largest distance from it, rounded up) in structure-of-arrays form, and
// the rows past the last point filled so that they weigh nothing.  One wave
// per tile.  A tile with a coordinate that is not finite gets a NaN centre:
// it is never left out.
template <int D>
__global__ __launch_bounds__(256) void tile_ball_kernel(float* T, int n, int tiles, float* geom, int ld) {
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (t >= tiles) return;
    const int i = t * 64 + lane;
    float4* row = reinterpret_cast<float4*>(T) + i;
    const bool live = i < n;
    if (!live) *row = make_float4(kPadCoord, kPadCoord, kPadCoord, kPadCoord);
    if (!geom) return;
    const float4 p = *row;
    const float x[4] = {p.x, p.y, p.z, p.w};
    float c[D], r2 = 0.0f;
    bool fin = true;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        float lo = live ? x[k] : __builtin_inff(), hi = live ? x[k] : -__builtin_inff();
        fin = fin && (!live || isfinite(x[k]));
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            lo = fminf(lo, __shfl_xor(lo, off));
            hi = fmaxf(hi, __shfl_xor(hi, off));
        }
        c[k] = 0.5f * (lo + hi);
        const float u = live ? x[k] - c[k] : 0.0f;
        r2 = fmaf(u, u, r2);
    }
    const bool allfin = __ballot(!fin) == 0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) r2 = fmaxf(r2, __shfl_xor(r2, off));
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < D; ++k) geom[(long long)k * ld + t] = allfin ? c[k] : __builtin_nanf("");
        geom[(long long)D * ld + t] = sqrtf(r2) * 1.0001f + 1e-30f;
    }
}

// Seeds of a step call in (m x d, stride d) and out, one coordinate per thread.
__global__ void seed_load_kernel(const float* __restrict__ seeds, const uint8_t* __restrict__ conv_in, int d, int DP,
                                 int m, float* S, uint8_t* status, int32_t* iters, float* shift2) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < (long long)m * DP; e += stride) {
        const int j = (int)(e / DP), k = (int)(e % DP);
        S[e] = k < d ? seeds[(long long)j * d + k] : 0.0f;
        if (k == 0) {
            status[j] = conv_in[j];
            iters[j] = 0;
            shift2[j] = __builtin_nanf("");
        }
    }
}

__global__ void seed_store_kernel(const float* __restrict__ S, int DP, int d, int m,
                                  const uint8_t* __restrict__ status, const int32_t* __restrict__ it,
                                  const float* __restrict__ sh, float* seeds, uint8_t* conv, int32_t* iters,
                                  float* shift2) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < (long long)m * d; e += stride) {
        const int j = (int)(e / d), k = (int)(e % d);
        seeds[e] = S[(long long)j * DP + k];
        if (k == 0) {
            conv[j] = status[j];
            iters[j] = it[j];
            if (it[j] > 0) shift2[j] = sh[j];
        }
    }
}

// Blocks of 256 for that many elements, a stride more than once where a launch
// of all of them would have 2^32 threads.
dim3 element_grid(long long total) { return dim3((unsigned)std::min<long long>((total + 255) / 256, 1 << 22)); }

// D >= 8: rows to tiles as they are, with the tail filled up (no balls).
__global__ void pack_tiles_kernel(const float* __restrict__ X, int n, int d, int D, float scale, float* T) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int G4 = D / 4, tiles = (n + 63) / 64;
    if (e >= (long long)tiles * G4 * 64) return;
    const int lane = (int)(e & 63), q = (int)((e >> 6) % G4);
    const long long i = (e >> 6) / G4 * 64 + lane;
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (i < n && 4 * q + k < d) ? X[i * d + 4 * q + k] * scale : 0.0f;
    if (i >= n && q == 0) v[0] = kPadCoord;
    reinterpret_cast<float4*>(T)[e] = make_float4(v[0], v[1], v[2], v[3]);
}

template <int D, int R, bool RUNS, bool PW = false>
hipError_t launch_seed_t(SeedArgs a, int kernel, int wgs, int nw, hipStream_t s) {
    const size_t lds = (RUNS ? run_lds(a.run_cap) * (PW ? nw : 1) : 0) +
                       (fold_rows(D, PW) ? (size_t)nw * fold_quads(D) * 256 : 0);
    // from the last seeds down, as within a launch: the far ones start first
    for (int w1 = wgs; w1 > 0; w1 = a.wg0) {
        a.wgs = std::min(w1, kSeedLaunch);
        a.wg0 = w1 - a.wgs;
        const dim3 g((a.wgs + 8 * kXcdRun - 1) / (8 * kXcdRun) * (8 * kXcdRun));
        if (kernel == MS_KERNEL_GAUSSIAN)
            hipLaunchKernelGGL((seed_iterate_kernel<D, R, MS_KERNEL_GAUSSIAN, RUNS, PW>), g, dim3(64 * nw), lds, s, a);
        else
            hipLaunchKernelGGL((seed_iterate_kernel<D, R, MS_KERNEL_FLAT, RUNS, PW>), g, dim3(64 * nw), lds, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_seed_load(const float* seeds, const uint8_t* conv_in, int d, int m, Batch& b, hipStream_t s) {
    if (b.metric == MS_METRIC_COSINE) return hipErrorInvalidValue;   // unit seeds: launch_seed_init_from_array
    const long long total = (long long)m * b.sh.DP;
    hipLaunchKernelGGL(seed_load_kernel, element_grid(total), dim3(256), 0, s, seeds, conv_in, d,
                       b.sh.DP, m, b.S, b.status, b.iters, b.shift2);
    return hipGetLastError();
}

hipError_t launch_seed_store(const Batch& b, int m, float* seeds, uint8_t* conv, int32_t* iters, float* shift2,
                             hipStream_t s) {
    const long long total = (long long)m * b.d;
    hipLaunchKernelGGL(seed_store_kernel, element_grid(total), dim3(256), 0, s, b.S, b.sh.DP, b.d,
                       m, b.status, b.iters, b.shift2, seeds, conv, iters, shift2);
    return hipGetLastError();
}

hipError_t launch_pack_tiles(const float* X, int n, int d, int D, float scale, float* T, hipStream_t s) {
    const long long total = (long long)((n + 63) / 64) * (D / 4) * 64;
    hipLaunchKernelGGL(pack_tiles_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, X, n, d, D, scale, T);
    return hipGetLastError();
}

hipError_t launch_tile_ball(float* T, int n, int D, float* geom, int ld, hipStream_t s) {
    const int tiles = (n + 63) / 64;
    const dim3 g((tiles + 3) / 4);
    switch (D) {
        case 1: hipLaunchKernelGGL((tile_ball_kernel<1>), g, dim3(256), 0, s, T, n, tiles, geom, ld); break;
        case 2: hipLaunchKernelGGL((tile_ball_kernel<2>), g, dim3(256), 0, s, T, n, tiles, geom, ld); break;
        case 3: hipLaunchKernelGGL((tile_ball_kernel<3>), g, dim3(256), 0, s, T, n, tiles, geom, ld); break;
        case 4: hipLaunchKernelGGL((tile_ball_kernel<4>), g, dim3(256), 0, s, T, n, tiles, geom, ld); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Seeds per workgroup and waves per workgroup for m seeds.  Few seeds: one per
// workgroup, split over as many waves as fill the 1,024 SIMDs about four deep.
// Many: four neighbours per workgroup share the loaded tiles.  Measured, 200,000
// x 3-D points, all updates of a batch (7 or so) in one launch, us:
//   m       1 seed: 4 / 8 / 16 waves     4 seeds: 1 / 2 / 4 waves
//   128       46 / 33 / 33
//   512       47 / 40 / 61
//   1,024     58 / 69 / 109
//   2,048     96 / 124 / 206
//   8,192    315 / 424 / 752              555 / 316 / 209
//   32,768                               1449 / 898 / 643
// (one update launched as a step over 64-seed tiles and a finalize: 31 us at
// 512 seeds, 220 us for a batch; 1.54 ms at 200,000 seeds against 1.28 here).
// Wide rows, 262,144 x 32-D points in runs, 3 updates, us:
//   m       1 seed: 1 / 2 / 4 / 8 waves   2 seeds: 1 / 2 / 4 waves
//   128      159 / 90 / 56 / 43
//   1,024    229 / 159 / 151 / 175          325 / 182 / 125
//   8,192    557 / 469 / 510 / 869          620 / 511 / 546
// (64-seed tiles: 2,530 us an update at 8,192 seeds).  Two seeds share the
// loads but leave two waves a SIMD: one seed per workgroup.
// At D <= 4 the number of points matters too: a seed alone reads all the points
// within its reach, which grow with n, and from some n on that, not the walk
// over the lists, is the time.  Then two or four neighbours share them.  Five
// updates of clustered (50 blobs, 3-D), evenly spread (2-D) and entirely reached
// points (one blob), us, seeds a workgroup and waves:
//   n, m                  1, 4 or 8           2, 8            4, 8
//   200,000   1,000     152   240   703   168  236  559
//   400,000   2,000     306   722  2567                    276   467  1512
//   1,000,000 1,000     459  1340  3151   379  787 2431
//   1,000,000 2,000     662  2635  7601                    484   960  3587
//   4,000,000 2,000    3147 13403 61153                   1610  4113 13926
//                        4, 4                               4, 8
//   400,000   4,000     385   772  2967                    420   739  2825
//   1,000,000 4,000     748  1765  7301                    741  1625  6748
//   4,000,000 8,192    3918 13339 52859                   3821 11764 50614
// (the order of the seeds is 10 us: at 400,000 points two updates of 600 to
// 1,500 clustered seeds were 7 to 11 % slower with it).
SeedShape seed_shape(int D, long long m, long long n) {
    SeedShape sh;
    if (D <= 4) {
        const bool many = n > (1 << 19);
        sh.R = m > 2048 ? 4 : (many && m > 512 ? (m > 1024 ? 4 : 2) : 1);
        sh.nw = m <= 512 || (many && sh.R > 1) ? 8 : 4;
    } else {
        sh.R = 1;
        sh.nw = m <= 512 ? 8 : (m <= 2048 ? 4 : 2);
    }
    return sh;
}

// The seeds of many clouds: one per workgroup.
SeedShape seed_shape_batched(long long m) {
    SeedShape sh;
    sh.R = 1;
    sh.nw = m <= 512 ? 8 : (m <= 2048 ? 4 : (m <= 8192 ? 2 : 1));
    return sh;
}

hipError_t launch_seed_iterate(SeedArgs a, int D, int kernel, const SeedShape& sh, int wgs, hipStream_t s) {
    if (sh.nw < 1 || sh.nw > seed_max_waves(D, sh.R)) return hipErrorInvalidValue;
    a.slack = kernel == MS_KERNEL_GAUSSIAN ? kSlack : 0.25f * sqrtf(a.h2) * a.scale;
    a.flat_reach = sqrtf(a.h2 * kSeedFlatMargin);
    if (wgs < 1) return hipSuccess;
    // one of two launches runs, by the index's estimate (RunIndex::dense)
    if (a.dense) {
        const int g = (wgs + kOwnWaves - 1) / kOwnWaves;
        hipError_t e = hipErrorInvalidValue;
        if (D == 16) e = launch_seed_t<16, 1, true, true>(a, kernel, g, kOwnWaves, s);
        if (D == 32) e = launch_seed_t<32, 1, true, true>(a, kernel, g, kOwnWaves, s);
        if (e != hipSuccess) return e;
    }
#define FMS_CASE(DD, RR, RUNS) \
    if (D == DD && sh.R == RR && (a.poff != nullptr) == RUNS) return launch_seed_t<DD, RR, RUNS>(a, kernel, wgs, sh.nw, s);
    FMS_CASE(1, 1, false) FMS_CASE(2, 1, false) FMS_CASE(3, 1, false) FMS_CASE(4, 1, false)
    FMS_CASE(1, 2, false) FMS_CASE(2, 2, false) FMS_CASE(3, 2, false) FMS_CASE(4, 2, false)
    FMS_CASE(1, 4, false) FMS_CASE(2, 4, false) FMS_CASE(3, 4, false) FMS_CASE(4, 4, false)
    FMS_CASE(1, 1, true) FMS_CASE(2, 1, true) FMS_CASE(3, 1, true) FMS_CASE(4, 1, true)
    FMS_CASE(8, 1, true) FMS_CASE(16, 1, true) FMS_CASE(32, 1, true)
    FMS_CASE(8, 1, false) FMS_CASE(16, 1, false) FMS_CASE(32, 1, false)
#undef FMS_CASE
    return hipErrorInvalidValue;
}

}  // namespace fms
