// k_adjoint.hip -- the differentiable Gaussian update and its hand-written
// adjoint, for gfx950, in FP32 or FP64.
//
// Forward (the batched update of Section II-B for every seed, no stopping):
//     w_ij = exp(-|s_j - x_i|^2 / (2 h^2)),  W_j = sum_i w_ij,
//     s'_j = s_j + delta_j,  delta_j = sum_i w_ij (x_i - s_j) / W_j .
// Reverse, for an upstream gradient g_j = dL/ds'_j (derived from the
// forward: ds'_j/dw_ij = (x_i - s'_j)/W_j, dw_ij/ds_j = w_ij (x_i - s_j)/h^2,
// and the direct path ds'_j/dx_i = (w_ij/W_j) I):
//     beta_ij = w_ij * g_j.(x_i - s'_j) / (h^2 W_j)
//     dL/ds_j += sum_i beta_ij (x_i - s_j)
//     dL/dx_i += sum_j (w_ij / W_j) g_j + beta_ij (s_j - x_i)
// Two passes over the pairs (three for wide rows: one_pass()) recompute the
// weights each time; no m x n weight matrix is ever stored.  Lanes are rows of one set (64 to a wave);
// the other set's rows stream past in wave-uniform (scalar) loads, split over
// the four waves of a workgroup, whose sums join in LDS in wave order, and over
// chunk_count() workgroups, whose partials a reduction kernel adds in chunk
// order: results are bitwise reproducible.
//
// These sizes (FP64, and FP32 under the run form's line) leave the chip idle
// before they fill it, so the split follows the sizes.  2 clouds of 1,501
// points, d = 8, FP64, two updates and their adjoints, with 8 fixed chunks of
// 256-row blocks (96 workgroups a pass) and now: update 42 -> 15 us, update and
// dS 90 -> 18, dX 102 -> 21, reductions 6 -> 4 each; what is left is the FP64
// VALU (an exponential and 3 to 6 operations a coordinate) and the latency of
// the reductions.

#include "fms_internal.h"

namespace fms {

namespace {

constexpr int kT = 256;
constexpr int kRows = 64;        // rows of a workgroup: its lanes
constexpr int kW = kT / kRows;   // waves, each with its share of the inner rows

// Inner-sum chunks of a pass over `rows` x `inner` pairs of nb clouds: enough
// workgroups for three waves a SIMD while a wave keeps 16 inner rows, and never
// under two, so that no partial sum is longer than an eighth of the whole.
int chunk_count(int nb, long long rows, long long inner) {
    const long long blocks = nb * ((rows + kRows - 1) / kRows);
    long long c = (768 + blocks - 1) / blocks;
    const long long most = inner / (16 * kW);
    if (c > most) c = most;
    if (c > 64) c = 64;
    return c < 2 ? 2 : (int)c;
}

// Sums acc over the workgroup's waves in wave order; the last wave ends with the total.
template <typename T, int N>
__device__ __forceinline__ void join_waves(T* acc) {
    __shared__ T red[N][kRows];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int w = 0; w < kW; ++w) {
        if (wave == w) {
            if (w > 0) {
#pragma unroll
                for (int k = 0; k < N; ++k) acc[k] += red[k][lane];
            }
            if (w < kW - 1) {
#pragma unroll
                for (int k = 0; k < N; ++k) red[k][lane] = acc[k];
            }
        }
        __syncthreads();
    }
}

// The inner rows [first, last) of this wave.
__device__ __forceinline__ void inner_range(int inner, int& first, int& last) {
    const long long part = (long long)blockIdx.y * kW + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long parts = (long long)gridDim.y * kW;
    first = (int)(inner * part / parts);
    last = (int)(inner * (part + 1) / parts);
}

template <typename T>
__device__ __forceinline__ T expw(T q, T c);   // exp(c q), c = -1/(2h^2)
template <>
__device__ __forceinline__ float expw<float>(float q, float c) {
    return __builtin_amdgcn_exp2f(q * c);       // c pre-multiplied by log2(e)
}
template <>
__device__ __forceinline__ double expw<double>(double q, double c) {
    return exp(q * c);
}

// Per-pass per-row state loaded once per lane.
template <typename T, int D>
struct Row {
    T v[D];
};

// Row `row` of a d-column array, zero-padded to D.  EXACT (d == D) loads
// with compile-time offsets, which lets wave-uniform rows become wide scalar
// loads; otherwise each column is guarded.
template <typename T, int D, bool EXACT>
__device__ __forceinline__ void load_row(const T* __restrict__ A, long long row, int d, T* out) {
    if constexpr (EXACT) {
#pragma unroll
        for (int k = 0; k < D; ++k) out[k] = A[row * D + k];
    } else {
#pragma unroll
        for (int k = 0; k < D; ++k) out[k] = (k < d) ? A[row * d + k] : T(0);
    }
}

// Forward partials: lane = seed j, chunk of points.  part[(b*chunks + c)*(D+1) + k][m]
template <typename T, int D, bool EXACT>
__global__ __launch_bounds__(kT) void fwd_partial_kernel(const T* __restrict__ X, int n,
                                                         const T* __restrict__ S, int m, int d,
                                                         T c, T* __restrict__ part) {
    const int b = blockIdx.z, chunk = blockIdx.y, lane = threadIdx.x & 63;
    const int j = blockIdx.x * kRows + lane;
    const T* Xb = X + (long long)b * n * d;
    T s[D], acc[D + 1];
    load_row<T, D, EXACT>(S + (long long)b * m * d, j < m ? j : 0, d, s);
#pragma unroll
    for (int k = 0; k <= D; ++k) acc[k] = T(0);
    int p0, p1;
    inner_range(n, p0, p1);
    for (int i = p0; i < p1; ++i) {
        T x[D];
        load_row<T, D, EXACT>(Xb, i, d, x);
        T dx[D], q = T(0);
#pragma unroll
        for (int k = 0; k < D; ++k) {
            dx[k] = x[k] - s[k];
            q = fma(dx[k], dx[k], q);
        }
        const T w = expw<T>(q, c);
        acc[D] += w;
#pragma unroll
        for (int k = 0; k < D; ++k) acc[k] = fma(w, dx[k], acc[k]);
    }
    join_waves<T, D + 1>(acc);
    if (threadIdx.x >= kT - kRows && j < m) {
        T* out = part + ((long long)b * gridDim.y + chunk) * (D + 1) * m + j;
#pragma unroll
        for (int k = 0; k <= D; ++k) out[(long long)k * m] = acc[k];
    }
}

// Reduce forward partials: S_out = s + delta; keeps delta and 1/W per seed.
// A thread per coordinate and seed; W is summed by each.
template <typename T, int D>
__global__ void fwd_reduce_kernel(const T* __restrict__ part, const T* __restrict__ S, int m,
                                  int d, int chunks, T* S_out, T* delta, T* invW) {
    const int b = blockIdx.z, k = blockIdx.y;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= m) return;
    T a = T(0), w = T(0);
    const T* p = part + (long long)b * chunks * (D + 1) * m + j;
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) {
        a += p[((long long)c * (D + 1) + k) * m];
        w += p[((long long)c * (D + 1) + D) * m];
    }
    const T iw = T(1) / w;
    const long long row = (long long)b * m + j;
    if (invW && k == 0) invW[row] = iw;
    const T dk = a * iw;
    if (delta) delta[row * d + k] = dk;
    if (S_out) S_out[row * d + k] = S[row * d + k] + dk;
}

// The update and dS in one pass over the pairs: with W and delta not known
// before its end, dS is taken from
//     sum_i beta_ij (x_i - s_j) = (B_j - (g_j.delta_j) A_j) / (h^2 W_j),
//     A_j = sum_i w_ij (x_i - s_j),  B_j = sum_i w_ij g_j.(x_i - s_j) (x_i - s_j) .
// part[(b*chunks + c)*(2D+1) + k][m]: A, W, B.
template <typename T, int D, bool EXACT>
__global__ __launch_bounds__(kT) void fwd_ds_partial_kernel(const T* __restrict__ X, int n,
                                                            const T* __restrict__ S, int m, int d,
                                                            T c, const T* __restrict__ G,
                                                            T* __restrict__ part) {
    const int b = blockIdx.z, chunk = blockIdx.y, lane = threadIdx.x & 63;
    const int j = blockIdx.x * kRows + lane;
    const T* Xb = X + (long long)b * n * d;
    T s[D], g[D], acc[2 * D + 1];
    load_row<T, D, EXACT>(S + (long long)b * m * d, j < m ? j : 0, d, s);
    load_row<T, D, EXACT>(G + (long long)b * m * d, j < m ? j : 0, d, g);
#pragma unroll
    for (int k = 0; k <= 2 * D; ++k) acc[k] = T(0);
    int p0, p1;
    inner_range(n, p0, p1);
    for (int i = p0; i < p1; ++i) {
        T x[D];
        load_row<T, D, EXACT>(Xb, i, d, x);
        T dx[D], q = T(0), gdx = T(0);
#pragma unroll
        for (int k = 0; k < D; ++k) {
            dx[k] = x[k] - s[k];
            q = fma(dx[k], dx[k], q);
            gdx = fma(g[k], dx[k], gdx);
        }
        const T w = expw<T>(q, c);
        const T wg = w * gdx;
        acc[D] += w;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            acc[k] = fma(w, dx[k], acc[k]);
            acc[D + 1 + k] = fma(wg, dx[k], acc[D + 1 + k]);
        }
    }
    join_waves<T, 2 * D + 1>(acc);
    if (threadIdx.x >= kT - kRows && j < m) {
        T* out = part + ((long long)b * gridDim.y + chunk) * (2 * D + 1) * m + j;
#pragma unroll
        for (int k = 0; k <= 2 * D; ++k) out[(long long)k * m] = acc[k];
    }
}

// dS += from the partials above, and 1/W and g.delta for the dX pass.  Lanes
// are seeds, the waves share the sums; these are in FP64, so that the
// difference loses nothing.
template <typename T, int D>
__global__ __launch_bounds__(kT) void fwd_ds_reduce_kernel(const T* __restrict__ part, int m, int d, int chunks,
                                                           double inv_h2, const T* __restrict__ G, T* dS,
                                                           T* __restrict__ invW, T* __restrict__ gdel_out) {
    __shared__ double sum[2 * D + 1][kRows];
    const int b = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = blockIdx.x * kRows + lane;
    const T* p = part + (long long)b * chunks * (2 * D + 1) * m + (j < m ? j : 0);
    for (int k = wave; k <= 2 * D; k += kW) {
        double a = 0.0;
#pragma unroll 8
        for (int c = 0; c < chunks; ++c) a += (double)p[((long long)c * (2 * D + 1) + k) * m];
        sum[k][lane] = a;
    }
    __syncthreads();
    if (j >= m) return;
    const long long row = (long long)b * m + j;
    const double iw = 1.0 / sum[D][lane];
    double gd = 0.0;
#pragma unroll
    for (int k = 0; k < D; ++k)
        if (k < d) gd = fma((double)G[row * d + k], sum[k][lane] * iw, gd);
    if (wave == 0) {
        invW[row] = (T)iw;
        gdel_out[row] = (T)gd;
    }
    for (int k = wave; k < d; k += kW)
        dS[row * d + k] += (T)((sum[D + 1 + k][lane] - gd * sum[k][lane]) * (inv_h2 * iw));
}

// Rows up to which the one pass keeps its sums in registers: past it (FP32
// D = 64, FP64 D >= 32) the update and dS are passes of their own.
template <typename T, int D>
constexpr bool one_pass() {
    return D * sizeof(T) <= 128;
}

// dS partials: lane = seed j, chunk of points.
template <typename T, int D, bool EXACT>
__global__ __launch_bounds__(kT) void ds_partial_kernel(const T* __restrict__ X, int n,
                                                        const T* __restrict__ S, int m, int d,
                                                        T c, T inv_h2, const T* __restrict__ G,
                                                        const T* __restrict__ delta,
                                                        const T* __restrict__ invW,
                                                        T* __restrict__ gdel_out,
                                                        T* __restrict__ part) {
    const int b = blockIdx.z, chunk = blockIdx.y, lane = threadIdx.x & 63;
    const int j = blockIdx.x * kRows + lane;
    const int jj = j < m ? j : 0;
    const long long row = (long long)b * m + jj;
    const T* Xb = X + (long long)b * n * d;
    T s[D], g[D], acc[D];
    load_row<T, D, EXACT>(S + (long long)b * m * d, jj, d, s);
    load_row<T, D, EXACT>(G + (long long)b * m * d, jj, d, g);
    T gdel = T(0);
#pragma unroll
    for (int k = 0; k < D; ++k)
        if (k < d) gdel = fma(g[k], delta[row * d + k], gdel);
    if (chunk == 0 && threadIdx.x < kRows && j < m) gdel_out[row] = gdel;   // g_j . delta_j, read by the dX pass
    const T coef = inv_h2 * invW[row];
#pragma unroll
    for (int k = 0; k < D; ++k) acc[k] = T(0);
    int p0, p1;
    inner_range(n, p0, p1);
    for (int i = p0; i < p1; ++i) {
        T x[D];
        load_row<T, D, EXACT>(Xb, i, d, x);
        T dx[D], q = T(0), gdx = T(0);
#pragma unroll
        for (int k = 0; k < D; ++k) {
            dx[k] = x[k] - s[k];
            q = fma(dx[k], dx[k], q);
            gdx = fma(g[k], dx[k], gdx);
        }
        // g.(x - s') = g.(x - s) - g.delta
        const T beta = expw<T>(q, c) * (gdx - gdel) * coef;
#pragma unroll
        for (int k = 0; k < D; ++k) acc[k] = fma(beta, dx[k], acc[k]);
    }
    join_waves<T, D>(acc);
    if (threadIdx.x >= kT - kRows && j < m) {
        T* out = part + ((long long)b * gridDim.y + chunk) * D * m + j;
#pragma unroll
        for (int k = 0; k < D; ++k) out[(long long)k * m] = acc[k];
    }
}

// dX partials: lane = point i, chunk of seeds.
template <typename T, int D, bool EXACT>
__global__ __launch_bounds__(kT) void dx_partial_kernel(const T* __restrict__ X, int n,
                                                        const T* __restrict__ S, int m, int d,
                                                        T c, T inv_h2, const T* __restrict__ G,
                                                        const T* __restrict__ gdel,
                                                        const T* __restrict__ invW,
                                                        T* __restrict__ part) {
    const int b = blockIdx.z, chunk = blockIdx.y, lane = threadIdx.x & 63;
    const int i = blockIdx.x * kRows + lane;
    const T* Sb = S + (long long)b * m * d;
    const T* Gb = G + (long long)b * m * d;
    const T* Eb = gdel + (long long)b * m;
    const T* Wb = invW + (long long)b * m;
    T x[D], acc[D];
    load_row<T, D, EXACT>(X + (long long)b * n * d, i < n ? i : 0, d, x);
#pragma unroll
    for (int k = 0; k < D; ++k) acc[k] = T(0);
    int j0, j1;
    inner_range(m, j0, j1);
    for (int j = j0; j < j1; ++j) {
        T s[D], g[D];
        load_row<T, D, EXACT>(Sb, j, d, s);
        load_row<T, D, EXACT>(Gb, j, d, g);
        const T iw = Wb[j];
        const T gd = Eb[j];
        T dx[D], q = T(0), gdx = T(0);
#pragma unroll
        for (int k = 0; k < D; ++k) {
            dx[k] = x[k] - s[k];
            q = fma(dx[k], dx[k], q);
            gdx = fma(g[k], dx[k], gdx);
        }
        const T w = expw<T>(q, c);
        const T a = w * iw;                              // w_ij / W_j
        const T beta = a * (gdx - gd) * inv_h2;          // beta_ij
#pragma unroll
        for (int k = 0; k < D; ++k) acc[k] = fma(a, g[k], fma(-beta, dx[k], acc[k]));
    }
    join_waves<T, D>(acc);
    if (threadIdx.x >= kT - kRows && i < n) {
        T* out = part + ((long long)b * gridDim.y + chunk) * D * n + i;
#pragma unroll
        for (int k = 0; k < D; ++k) out[(long long)k * n] = acc[k];
    }
}

// out[row, k] += sum over chunks of part (chunk order).  A thread per element.
template <typename T, int D>
__global__ void add_reduce_kernel(const T* __restrict__ part, int rows, int d, int chunks, T* out) {
    const int b = blockIdx.z, k = blockIdx.y;
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= rows) return;
    T a = T(0);
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) a += part[(((long long)b * chunks + c) * D + k) * rows + r];
    out[((long long)b * rows + r) * d + k] += a;
}

template <typename T>
T weight_coef(double h) {
    return sizeof(T) == 4 ? T(-1.4426950408889634 / (2.0 * h * h)) : T(-1.0 / (2.0 * h * h));
}

template <typename T, int D>
hipError_t fwd_t(const T* X, int nb, int n, const T* S, int m, int d, double h, T* S_out,
                 T* delta, T* invW, T* part, hipStream_t s) {
    const int chunks = chunk_count(nb, m, n);
    dim3 g1((m + kRows - 1) / kRows, chunks, nb);
    if (d == D)
        hipLaunchKernelGGL((fwd_partial_kernel<T, D, true>), g1, dim3(kT), 0, s, X, n, S, m, d,
                           weight_coef<T>(h), part);
    else
        hipLaunchKernelGGL((fwd_partial_kernel<T, D, false>), g1, dim3(kT), 0, s, X, n, S, m, d,
                           weight_coef<T>(h), part);
    dim3 g2((m + 255) / 256, d, nb);
    hipLaunchKernelGGL((fwd_reduce_kernel<T, D>), g2, dim3(256), 0, s, part, S, m, d, chunks, S_out,
                       delta, invW);
    return hipGetLastError();
}

template <typename T, int D, bool EXACT>
hipError_t adj_passes(const T* X, int nb, int n, const T* S, int m, int d, double h, const T* G,
                      T* delta, T* invW, T* gdel, T* part, T* dS, T* dX, hipStream_t s) {
    const T c = weight_coef<T>(h);
    const T ih2 = T(1.0 / (h * h));
    const int cs = chunk_count(nb, m, n), cx = chunk_count(nb, n, m);
    const dim3 gs((m + kRows - 1) / kRows, cs, nb);
    if constexpr (one_pass<T, D>()) {
        hipLaunchKernelGGL((fwd_ds_partial_kernel<T, D, EXACT>), gs, dim3(kT), 0, s, X, n, S, m, d, c, G, part);
        hipLaunchKernelGGL((fwd_ds_reduce_kernel<T, D>), dim3(gs.x, nb), dim3(kT), 0, s, part, m, d, cs,
                           1.0 / (h * h), G, dS, invW, gdel);
    } else {
        const hipError_t e = fwd_t<T, D>(X, nb, n, S, m, d, h, nullptr, delta, invW, part, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((ds_partial_kernel<T, D, EXACT>), gs, dim3(kT), 0, s, X, n, S, m, d, c, ih2, G, delta,
                           invW, gdel, part);
        hipLaunchKernelGGL((add_reduce_kernel<T, D>), dim3((m + 255) / 256, d, nb), dim3(256), 0, s,
                           part, m, d, cs, dS);
    }
    hipLaunchKernelGGL((dx_partial_kernel<T, D, EXACT>), dim3((n + kRows - 1) / kRows, cx, nb), dim3(kT), 0,
                       s, X, n, S, m, d, c, ih2, G, gdel, invW, part);
    hipLaunchKernelGGL((add_reduce_kernel<T, D>), dim3((n + 255) / 256, d, nb), dim3(256), 0, s,
                       part, n, d, cx, dX);
    return hipGetLastError();
}

template <typename T, int D>
hipError_t adj_t(const T* X, int nb, int n, const T* S, int m, int d, double h, const T* G,
                 T* dS, T* dX, T* delta, T* invW, T* gdel, T* part, hipStream_t s) {
    if (d == D) return adj_passes<T, D, true>(X, nb, n, S, m, d, h, G, delta, invW, gdel, part, dS, dX, s);
    return adj_passes<T, D, false>(X, nb, n, S, m, d, h, G, delta, invW, gdel, part, dS, dX, s);
}

struct Ws {
    char* base;
    size_t part, delta, invw, gdel;
};

Ws carve(void* ws, int nb, int n, int m, int d, int bytes) {
    const int D = step_shape(d).D;
    const long long rs = (long long)chunk_count(nb, m, n) * m, rx = (long long)chunk_count(nb, n, m) * n;
    Ws w;
    w.base = (char*)ws;
    w.part = 0;
    size_t off = (size_t)nb * (2 * D + 1) * (size_t)(rs > rx ? rs : rx) * bytes;
    off = (off + 255) & ~(size_t)255;
    w.delta = off;
    off += (size_t)nb * m * d * bytes;
    off = (off + 255) & ~(size_t)255;
    w.invw = off;
    off += (size_t)nb * m * bytes;
    off = (off + 255) & ~(size_t)255;
    w.gdel = off;
    return w;
}

#define FMS_ADJ_DSWITCH(D_, CALL)                           \
    switch (D_) {                                           \
        case 1: { constexpr int DD = 1; return CALL; }      \
        case 2: { constexpr int DD = 2; return CALL; }      \
        case 3: { constexpr int DD = 3; return CALL; }      \
        case 4: { constexpr int DD = 4; return CALL; }      \
        case 8: { constexpr int DD = 8; return CALL; }      \
        case 16: { constexpr int DD = 16; return CALL; }    \
        case 32: { constexpr int DD = 32; return CALL; }    \
        case 64: { constexpr int DD = 64; return CALL; }    \
        default: return hipErrorInvalidValue;               \
    }

}  // namespace

size_t adjoint_workspace_bytes(int nb, int n, int m, int d, int bytes) {
    Ws w = carve(nullptr, nb, n, m, d, bytes);
    return w.gdel + (size_t)nb * m * bytes + 256;
}

hipError_t launch_forward_update(const void* X, int nb, int n, const void* S, int m, int d,
                                 double h, void* S_out, int bytes, void* ws, hipStream_t s) {
    Ws w = carve(ws, nb, n, m, d, bytes);
    const int D = step_shape(d).D;
    if (bytes == 4) {
        FMS_ADJ_DSWITCH(D, (fwd_t<float, DD>((const float*)X, nb, n, (const float*)S, m, d, h,
                                             (float*)S_out, nullptr, nullptr,
                                             (float*)(w.base + w.part), s)));
    }
    FMS_ADJ_DSWITCH(D, (fwd_t<double, DD>((const double*)X, nb, n, (const double*)S, m, d, h,
                                          (double*)S_out, nullptr, nullptr,
                                          (double*)(w.base + w.part), s)));
}

hipError_t launch_step_adjoint(const void* X, int nb, int n, const void* S, int m, int d,
                               double h, const void* G, void* dS, void* dX, int bytes, void* ws,
                               hipStream_t s) {
    Ws w = carve(ws, nb, n, m, d, bytes);
    const int D = step_shape(d).D;
    if (bytes == 4) {
        FMS_ADJ_DSWITCH(D, (adj_t<float, DD>((const float*)X, nb, n, (const float*)S, m, d, h,
                                             (const float*)G, (float*)dS, (float*)dX,
                                             (float*)(w.base + w.delta),
                                             (float*)(w.base + w.invw),
                                             (float*)(w.base + w.gdel),
                                             (float*)(w.base + w.part), s)));
    }
    FMS_ADJ_DSWITCH(D, (adj_t<double, DD>((const double*)X, nb, n, (const double*)S, m, d, h,
                                          (const double*)G, (double*)dS, (double*)dX,
                                          (double*)(w.base + w.delta),
                                          (double*)(w.base + w.invw),
                                          (double*)(w.base + w.gdel),
                                          (double*)(w.base + w.part), s)));
}

}  // namespace fms
