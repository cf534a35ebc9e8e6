// Compensation factors from the quantization error, on the GPU, in fp64.
//
// The paper takes the compensation factors from the singular value
// decomposition of the residual E = W - W_hat (Section 4.1) and relies on the
// truncated SVD being the best rank-r approximation, its squared Frobenius
// error being the sum of the squared tail singular values (Appendix B.2,
// Eckart-Young-Mirsky).  With E = U diag(sigma) V^T, sigma descending:
//
//     A = diag(sqrt(sigma[:r_max])) V^T[:r_max]        (r_max x d_in)
//     B = U[:, :r_max] diag(sqrt(sigma[:r_max]))       (d_out x r_max)
//
// so B[:, :r] A[:r] is the rank-r truncation for every r <= r_max; the sign of
// each singular pair makes the largest-magnitude entry of the U column
// positive (first index on ties).
//
// Steps (all fp64, one stream, the host waits once):
//  1. E = W - s (q - z) elementwise.
//  2. The Gram matrix over the smaller side, C = E^T E (d_in <= d_out) or
//     C = E E^T, with a tiled fp64 MFMA GEMM (64 x 64 tiles through LDS).
//  3. Eigen-decomposition C = X diag(lambda) X^T, X for the leading r_max only:
//     Householder reduction to tridiagonal T = Q^T C Q, one launch per
//     reflector; T split into blocks where a coupling is within the
//     reduction's rounding; every eigenvalue of each block by bisection on
//     Sturm counts, 64 points of an interval per wave and round; eigenvectors
//     of the blocks by inverse iteration, one lane per vector, with the
//     vectors of a block's close eigenvalues orthogonalised among each other
//     and all of them then made orthonormal to rounding; X = Q Z.
//  4. sigma = sqrt(lambda), descending.  If X holds right vectors V:
//     A = sqrt(sigma) V^T and
//     B = E V / sqrt(sigma) (= U sqrt(sigma)); if it holds left vectors U:
//     B = U sqrt(sigma) and A = U^T E / sqrt(sigma).
//  5. Sign fix on the U column, rounding to fp16 (one rounding from fp64).
//
// The Gram route squares the condition number: singular values far below
// sqrt(eps) * sigma_max carry absolute, not relative, accuracy.  The factors
// only use the leading ones.

#include <type_traits>

#include "cl_device.h"
#include "cl_internal.h"

namespace cl {

namespace {

// Sweep 1 leaves |T| eps / gap of the neighbours in a vector, sweep 2 its square
// (an unlucky start vector included).
constexpr int kInverseSweeps = 2, kMaxSweeps = 8;
// What the vectors are checked for after a sweep: |T z - lambda z| relative to
// |T|, and the inner products of different ones.  Ordinary residuals reach 1e-15
// and eps / gap; 175,000 near-degenerate ones on the CPU 2e-12 and 6e-10.
constexpr double kResidualTol = 1e-10, kOrthogonalTol = 1e-8;
// Bisection rounds: 65-section of an interval of width 2 |T| down to 2^-53 |T|.
constexpr int kSections = 9;
// Eigenvalues of a block closer than this (relative to |T|) have their vectors
// orthogonalised; beyond it inverse iteration alone leaves them orthogonal to
// better than 1e-9, which the last step (check_kernel) squares.
constexpr double kCluster = 1e-6;
// A coupling e_i is dropped, and T falls into two blocks there, where it is
// within kDrop sqrt(n) (|d_i| + |d_i+1|): the rounding of the n reflectors
// before it.  Left in, it does not separate the two sides and inverse iteration
// divides by it.
constexpr double kDrop = 4.5e-16;
// Shifts of one block's eigenvalues are kept this far apart (relative to |T|),
// about two roundings of an eigenvalue: with equal shifts every vector of a
// cluster turns into the one nearest the shift (the same is done in Jessup and
// Ipsen's analysis of inverse iteration and in LAPACK's xSTEIN).
constexpr double kShift = 4e-16;

size_t up256(size_t n) { return (n + 255) / 256 * 256; }

struct CompLayout {
    size_t E, C, V, tau, lam, row_lam, d, e, de, p, blk, order, rank_of, bounds, scale, sign, Xr, P, total;
};

CompLayout comp_layout(int d_out, int d_in, int r_max) {
    const size_t n = static_cast<size_t>(d_in <= d_out ? d_in : d_out);
    const size_t big = static_cast<size_t>(d_in > d_out ? d_in : d_out);
    CompLayout l;
    l.E = 0;
    l.C = l.E + up256(static_cast<size_t>(d_out) * d_in * 8);
    l.V = l.C + up256(n * n * 8);
    l.tau = l.V + up256(n * n * 8);
    l.lam = l.tau + up256(n * 8);
    l.row_lam = l.lam + up256(n * 8);
    l.d = l.row_lam + up256(n * 8);
    l.e = l.d + up256(n * 8);
    l.de = l.e + up256(n * 8);
    l.p = l.de + up256(n * 16);
    l.blk = l.p + up256(n * 16);
    l.order = l.blk + up256(n * 8);
    l.rank_of = l.order + up256(n * 4);
    l.bounds = l.rank_of + up256(n * 4);
    l.scale = l.bounds + 256;
    l.sign = l.scale + up256(static_cast<size_t>(r_max) * 8 + 8);
    l.Xr = l.sign + up256(static_cast<size_t>(r_max) * 8 + 8);
    l.P = l.Xr + up256(static_cast<size_t>(r_max) * n * 8 + 8);
    l.total = l.P + up256(static_cast<size_t>(r_max) * big * 8 + 8);
    return l;
}

__device__ __forceinline__ double h2d(uint16_t h) {
    return static_cast<double>(f16_bits_to_f32(h));
}

// E[o][c] = W[o][c] - s (q - z), one thread per element
__global__ __launch_bounds__(256) void residual_kernel(const float* __restrict__ W, QW w, double* __restrict__ E) {
    const size_t idx = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    const size_t total = static_cast<size_t>(w.d_out) * w.d_in;
    if (idx >= total) return;
    const int o = static_cast<int>(idx / w.d_in);
    const int c = static_cast<int>(idx - static_cast<size_t>(o) * w.d_in);
    // code c: bits bits * c .. of the row's bit string (3-bit codes can
    // straddle two words)
    const uint32_t* row = w.q + static_cast<size_t>(o) * (static_cast<size_t>(w.d_in) * w.bits / 32);
    const int bp = w.bits * c;
    uint64_t two = row[bp >> 5];
    if ((bp & 31) + w.bits > 32) two |= static_cast<uint64_t>(row[(bp >> 5) + 1]) << 32;
    const uint32_t code = static_cast<uint32_t>(two >> (bp & 31)) & ((1u << w.bits) - 1u);
    const size_t gi = static_cast<size_t>(o) * (w.d_in / w.G) + c / w.G;
    const double what = h2d(w.s[gi]) * (static_cast<double>(code) - h2d(w.z[gi]));
    E[idx] = static_cast<double>(W[idx]) - what;
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

// out[i * ldo + j] = sum_k X[i * xi + k * xk] * Y[j * yj + k * yk]  (fp64)
// 64 x 64 output tile per 256-thread workgroup, each wave a 32 x 32 quadrant
// of it on v_mfma_f64_16x16x4_f64; k in steps of 16 through two LDS buffers,
// the next step's loads in flight during this one's products (a lone
// workgroup per CU has nothing else to hide them).  XK1 / YK1: the operand is
// contiguous along k (else along i / j), which decides the load order so that
// loads coalesce.  Bound by the matrix cores' fp64 rate and, at 16 x 16 tiles,
// by one workgroup's chain of k steps: 1024 x 1024 x 4096 245 us (fp64 FMAs on the
// VALU, 4 x 4 outputs a thread: 748).
template <bool XK1, bool YK1>
__global__ __launch_bounds__(256) void gemm_nt_f64(const double* __restrict__ X, size_t xi, size_t xk,
                                                   const double* __restrict__ Y, size_t yj, size_t yk, int I, int J,
                                                   int K, double* __restrict__ out, size_t ldo) {
    constexpr int BT = 64, BK = 16;
    __shared__ double xs[2][BK][BT + 1];
    __shared__ double ys[2][BK][BT + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, r = lane & 15;
    const int i0 = blockIdx.y * BT, j0 = blockIdx.x * BT;
    const int wi = 32 * (wave >> 1), wj = 32 * (wave & 1);
    // element l of this thread: row (of the tile) and k of the step
    auto row_of = [&](bool k1, int l) { const int e = tid + 256 * l; return k1 ? e / BK : e & (BT - 1); };
    auto k_of = [&](bool k1, int l) { const int e = tid + 256 * l; return k1 ? e & (BK - 1) : e / BT; };
    double xr[4], yr[4];
    auto load = [&](int k0) {
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            const int gi = i0 + row_of(XK1, l), gk = k0 + k_of(XK1, l);
            xr[l] = (gi < I && gk < K) ? X[gi * xi + gk * xk] : 0.0;
            const int gj = j0 + row_of(YK1, l), gkj = k0 + k_of(YK1, l);
            yr[l] = (gj < J && gkj < K) ? Y[gj * yj + gkj * yk] : 0.0;
        }
    };
    auto store = [&](int st) {
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            xs[st][k_of(XK1, l)][row_of(XK1, l)] = xr[l];
            ys[st][k_of(YK1, l)][row_of(YK1, l)] = yr[l];
        }
    };
    f64x4 acc[2][2] = {};
    load(0);
    store(0);
    __syncthreads();
    for (int k0 = 0, st = 0; k0 < K; k0 += BK, st ^= 1) {
        if (k0 + BK < K) load(k0 + BK);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 4) {
            double a[2], b[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                a[u] = xs[st][kk + g][wi + 16 * u + r];
                b[u] = ys[st][kk + g][wj + 16 * u + r];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 2; ++v)
                    acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[v], acc[u][v], 0, 0, 0);
        }
        if (k0 + BK < K) store(st ^ 1);
        __syncthreads();
    }
    // lane (g, r) holds rows 4 e + g of column r of a 16 x 16 tile
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int gi = i0 + wi + 16 * u + 4 * e + g, gj = j0 + wj + 16 * v + r;
                if (gi < I && gj < J) out[gi * ldo + gj] = acc[u][v][e];
            }
}

// Sum over the 256 threads of a workgroup, in a fixed order; red: 4 doubles
// that the previous use has been read out of.
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__device__ __forceinline__ double block_sum_f64(double v, double* red) {
    v = wave_sum_f64(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// 1 / q to about an ulp: the hardware estimate and two Newton steps.
__device__ __forceinline__ double recip_f64(double q) {
    double r = __builtin_amdgcn_rcp(q);
    r = fma(r, fma(-q, r, 1.0), r);
    return fma(r, fma(-q, r, 1.0), r);
}

// Step k of the Householder reduction, one launch per step.  On entry the
// rows and columns >= k of C still miss step k - 1's update
// C -= v w^T + w v^T, w = tau p - (tau^2 / 2)(p . v) v, where p = C v came out
// of the launch before.  Every workgroup forms w, the updated row k and from
// it the next reflector (v_k+1 = 1, tail scaled) for itself; then it updates
// its rows and multiplies each by the new v on the way, so C is read and
// written once per step.  A thread owns the same CPT columns throughout (v, w
// and the new v stay in its registers) and R rows at a time; the first R
// rows' loads are issued before the reductions.  Row i always belongs to
// workgroup i mod grid.  Bound by the chain of one launch (two reductions; 4.0
// us a step at <= 256 columns, 6.5 at 1024) up to n ~ 2000, beyond by the 16
// n^2 bytes.  The whole call at 1024 x 4096, r_max 128: 134 -> 7.5 ms, 4096 x
// 4096: 4.9 -> 0.11 s, against cyclic Jacobi (10 to 18 sweeps of n - 1 rounds
// of two launches over C and X).
template <int CPT, int R>
__global__ __launch_bounds__(256) void householder_step_kernel(double* __restrict__ C, int n, int k,
                                                               double* __restrict__ V,
                                                               const double* __restrict__ p_in,
                                                               double* __restrict__ p_out, double* __restrict__ tau,
                                                               double* __restrict__ d, double* __restrict__ e) {
    __shared__ double red[2][4];
    __shared__ double rows[2][R][4];
    __shared__ double next;
    const int tid = threadIdx.x, b = blockIdx.x, G = gridDim.x;
    const int col0 = (k & ~63) + tid;
    const double* vp = V + static_cast<size_t>(k > 0 ? k - 1 : 0) * n;
    const bool upd = k > 0;
    int i = b;
    if (i < k + 1) i += (k + 1 - i + G - 1) / G * G;

    double a[R][CPT];
    auto load_rows = [&](int i0) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int iu = i0 + u * G;
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const int j = col0 + 256 * c;
                a[u][c] = (iu < n && j > k && j < n) ? C[static_cast<size_t>(iu) * n + j] : 0.0;
            }
        }
    };

    double v[CPT], w[CPT], x[CPT];
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int j = col0 + 256 * c;
        const bool in = j >= k && j < n;
        v[c] = in && upd ? vp[j] : 0.0;
        w[c] = in && upd ? p_in[j] : 0.0;
        x[c] = in ? C[static_cast<size_t>(k) * n + j] : 0.0;
    }
    const double tp = upd ? tau[k - 1] : 0.0;
    const double pk = upd ? p_in[k] : 0.0;
    load_rows(i);
#pragma unroll
    for (int c = 0; c < CPT; ++c) s = fma(v[c], w[c], s);
    s = block_sum_f64(s, red[0]);
    const double h = 0.5 * tp * tp * s;
    const double wk = fma(tp, pk, -h);           // v_k = 1
    double q = 0.0;
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int j = col0 + 256 * c;
        w[c] = fma(tp, w[c], -h * v[c]);
        x[c] = fma(-wk, v[c], x[c] - w[c]);
        if (j == k && b == 0) d[k] = x[c];
        if (j == k + 1) next = x[c];
        if (j > k + 1) q = fma(x[c], x[c], q);   // zero past n
    }
    if (k + 1 >= n) return;                      // the last diagonal entry
    q = block_sum_f64(q, red[1]);
    const double x0 = next;
    double t = 0.0, beta = x0, inv = 0.0;
    // a tail whose squares fall out of the normal range (E is fp32, so it is
    // below 1e-55 of |T|) is left, for t would not fit v any more
    if (q > 1e-290) {
        const double norm = sqrt(fma(x0, x0, q));
        beta = x0 >= 0.0 ? -norm : norm;
        t = (beta - x0) / beta;
        inv = 1.0 / (x0 - beta);
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int j = col0 + 256 * c;
        x[c] = j == k + 1 ? 1.0 : (j > k + 1 ? x[c] * inv : 0.0);
        if (b == 0 && j > k && j < n) V[static_cast<size_t>(k) * n + j] = x[c];
    }
    if (b == 0 && tid == 0) { tau[k] = t; e[k] = beta; }

    for (int par = 0; i < n; i += R * G, par ^= 1) {
        double acc[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int iu = i + u * G < n ? i + u * G : n - 1;
            const double vi = upd ? vp[iu] : 0.0;
            const double wi = upd ? fma(tp, p_in[iu], -h * vi) : 0.0;
            acc[u] = 0.0;
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const int j = col0 + 256 * c;
                const double val = fma(-vi, w[c], fma(-wi, v[c], a[u][c]));
                if (i + u * G < n && j > k && j < n) {
                    if (tp != 0.0) C[static_cast<size_t>(iu) * n + j] = val;
                    acc[u] = fma(val, x[c], acc[u]);
                }
            }
        }
        if (i + R * G < n) load_rows(i + R * G);
#pragma unroll
        for (int u = 0; u < R; ++u) acc[u] = wave_sum_f64(acc[u]);
        if ((tid & 63) == 0) {
#pragma unroll
            for (int u = 0; u < R; ++u) rows[par][u][tid >> 6] = acc[u];
        }
        __syncthreads();
        if (tid < R && i + tid * G < n) {
            const double* r = rows[par][tid];
            p_out[i + tid * G] = (r[0] + r[1]) + (r[2] + r[3]);
        }
    }
}

// The couplings within the rounding dropped (e set to zero); blk[i] = the rows
// of i's block; (d_i, e_i-1^2) pairs for the Sturm counts; bounds = {lower and
// upper end of the Gershgorin discs, |T|, smallest pivot, 1 if T is not
// finite, (check_kernel's) worst check over its tolerance}.  One workgroup, a run of rows per thread.
__global__ __launch_bounds__(256) void tridiagonal_prep_kernel(const double* __restrict__ d, double* __restrict__ e,
                                                               int n, double2* __restrict__ de,
                                                               int2* __restrict__ blk, double* __restrict__ bounds) {
    __shared__ double red[3][4];
    __shared__ int edge[3][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, per = (n + 255) / 256;
    const int i0 = min(tid * per, n), i1 = min(i0 + per, n);
    const double tol = kDrop * sqrt(static_cast<double>(n));
    for (int i = i0; i < i1; ++i)
        if (i + 1 < n && fabs(e[i]) <= tol * (fabs(d[i]) + fabs(d[i + 1]))) e[i] = 0.0;
    __syncthreads();
    auto starts = [&](int i) { return i == 0 || e[i - 1] == 0.0; };
    double l = 1e308, h = -1e308, m = 0.0;
    int f = n, t = -1, bad = 0;
    for (int i = i0; i < i1; ++i) {
        const double el = i > 0 ? e[i - 1] : 0.0, er = i + 1 < n ? e[i] : 0.0;
        const double di = d[i], rad = fabs(el) + fabs(er);
        bad |= !(fabs(di) + rad < 1e300);
        de[i] = make_double2(di, el * el);
        l = fmin(l, di - rad);
        h = fmax(h, di + rad);
        m = fmax(m, el * el);
        if (starts(i)) {
            f = min(f, i);
            t = i;
        }
    }
    // the last start at or before this thread's rows, the first one after them
    int beg = t, end = f;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int p = __shfl_up(beg, off, 64), q = __shfl_down(end, off, 64);
        if (lane >= off) beg = max(beg, p);
        if (lane + off < 64) end = min(end, q);
        l = fmin(l, __shfl_xor(l, off, 64));
        h = fmax(h, __shfl_xor(h, off, 64));
        m = fmax(m, __shfl_xor(m, off, 64));
        bad |= __shfl_xor(bad, off, 64);
    }
    if (lane == 63) edge[0][wave] = beg;
    if (lane == 0) {
        edge[1][wave] = end;
        edge[2][wave] = bad;
        red[0][wave] = l; red[1][wave] = h; red[2][wave] = m;
    }
    __syncthreads();
    beg = __shfl_up(beg, 1, 64);
    end = __shfl_down(end, 1, 64);
    if (lane == 0) beg = 0;
    if (lane == 63) end = n;
    for (int w = 0; w < 4; ++w) {
        if (w < wave) beg = max(beg, edge[0][w]);
        if (w > wave) end = min(end, edge[1][w]);
    }
    for (int i = i0; i < i1; ++i) {
        if (starts(i)) beg = i;
        blk[i].x = beg;
    }
    for (int i = i1 - 1; i >= i0; --i) {
        blk[i].y = end;
        if (starts(i)) end = i;
    }
    if (tid == 0) {
        for (int w = 1; w < 4; ++w) {
            l = fmin(l, red[0][w]);
            h = fmax(h, red[1][w]);
            m = fmax(m, red[2][w]);
            bad |= edge[2][w];
        }
        const double norm = fmax(fabs(l), fabs(h));
        const double pad = 4e-16 * norm * sqrt(static_cast<double>(n));
        bounds[0] = l - pad;
        bounds[1] = h + pad;
        bounds[2] = norm;
        bounds[3] = 2.3e-308 * fmax(1.0, m);
        bounds[4] = bad;
        bounds[5] = 0.0;
    }
}

// row_lam[j] for row j of a block: the block's (j - first row)-th largest
// eigenvalue, one wave each: the number of eigenvalues below x is the number
// of negative pivots of T - x; each round every lane counts at one of 64
// points of the interval.
__global__ __launch_bounds__(256) void bisect_kernel(const double2* __restrict__ de, const int2* __restrict__ blk,
                                                     int n, const double* __restrict__ bounds,
                                                     double* __restrict__ row_lam) {
    const int j = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (j >= n) return;
    const int beg = blk[j].x, end = blk[j].y;
    const int lane = threadIdx.x & 63, below = end - 1 - j;
    double lo = bounds[0], hi = bounds[1];
    const double pivmin = bounds[3];
    for (int round = 0; round < kSections; ++round) {
        const double width = (hi - lo) * (1.0 / 65.0);
        const double x = fma(width, lane + 1.0, lo);
        int count = 0;
        double q = 1.0;
#pragma unroll 8
        for (int i = beg; i < end; ++i) {
            const double2 t = de[i];
            q = fma(-t.y, recip_f64(q), t.x - x);
            if (fabs(q) < pivmin) q = -pivmin;
            count += q < 0.0;
        }
        const unsigned long long above = __ballot(count > below);
        const int first = above ? __builtin_ctzll(above) : 64;
        const double base = lo;
        if (first < 64) hi = fma(width, first + 1.0, base);
        if (first > 0) lo = fma(width, static_cast<double>(first), base);
    }
    if (lane == 0) row_lam[j] = bounds[2] == 0.0 ? 0.0 : 0.5 * (lo + hi);
}

// The blocks' eigenvalues in one descending order (ties by row): lam, sigma;
// order[rank] = row, rank_of[row] = rank.  A single block is in order already,
// and stays in it where T is not finite (the order of NaNs is no permutation).
__global__ __launch_bounds__(256) void order_kernel(const double* __restrict__ row_lam, const int2* __restrict__ blk,
                                                    int n, const double* __restrict__ bounds,
                                                    double* __restrict__ lam, int* __restrict__ order,
                                                    int* __restrict__ rank_of, float* __restrict__ sigma) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const double l = row_lam[j];
    int rank = j;
    if (blk[0].y < n && bounds[4] == 0.0) {
        rank = 0;
        for (int q = 0; q < n; ++q) {
            const double v = row_lam[q];
            rank += v > l || (v == l && q < j);
        }
    }
    lam[rank] = l;
    order[rank] = j;
    rank_of[j] = rank;
    if (sigma) sigma[rank] = static_cast<float>(sqrt(l > 0.0 ? l : 0.0));
}

// Entry i of start vector j, in [-1, 1): the high half of a Weyl sequence (its
// steps 2^64 over the golden ratio and over the square root of two) squared
// twice.
__device__ __forceinline__ double start_entry(int i, int j) {
    uint64_t x = (i + 1) * 0x9E3779B97F4A7C15ull + (j + 1) * 0xB504F333F9DE6484ull;
    x = x * x + x;
    x = (x >> 32) | (x << 32);
    x = x * x + x;
    return static_cast<double>(static_cast<uint32_t>(x >> 32)) * 0x1p-31 - 1.0;
}

// One inverse iteration of vectors j0 .. j0 + nb - 1, a lane each, on the rows
// of the vector's block (zero elsewhere): Gaussian elimination of T - shift
// with partial pivoting, the right-hand side (the last iterate, |T| scaled; a
// fixed pseudo-random vector at first) carried along, then back substitution.
// Pivots below the rounding of |T| count as that: the vectors of a cluster
// would otherwise differ in scale by their ratio and agree in every digit.  S:
// the rows of the upper factor (reciprocal pivot, two off-diagonals) and the
// reduced right-hand side, nb of each per row; Z[i][j] the iterates, scale[j]
// their reciprocal norms.
__global__ __launch_bounds__(64) void inverse_iteration_kernel(const double* __restrict__ d,
                                                               const double* __restrict__ e, int n,
                                                               double* __restrict__ bounds,
                                                               const double* __restrict__ row_lam,
                                                               const int2* __restrict__ blk,
                                                               const int* __restrict__ order, int j0, int nb,
                                                               int r_max, bool first, double* __restrict__ S,
                                                               double* __restrict__ Z, double* __restrict__ scale) {
    const int t = blockIdx.x * 64 + threadIdx.x;
    if (t == 0) bounds[5] = 0.0;                  // the check that follows the sweep
    if (t >= nb) return;
    const int j = j0 + t, row = order[j], beg = blk[row].x, end = blk[row].y;
    const size_t plane = static_cast<size_t>(n) * nb;
    double *U0 = S + t, *U1 = U0 + plane, *U2 = U1 + plane, *Y = U2 + plane;
    const double norm = bounds[2] > 0.0 ? bounds[2] : 1.0, tiny = 1.1e-16 * norm, apart = kShift * norm;
    double l = row_lam[row];
    for (int q = row; q > beg && row_lam[q - 1] - row_lam[q] <= apart; --q) l -= apart;
    const double sc = first ? norm : norm * scale[j];
    auto rhs = [&](int i) -> double {
        return sc * (first ? start_entry(i, j) : Z[static_cast<size_t>(i) * r_max + j]);
    };
    double a = d[beg] - l, b = beg + 1 < end ? e[beg] : 0.0, y = rhs(beg);
#pragma unroll 4
    for (int i = beg; i + 1 < end; ++i) {
        const double ei = e[i], dn = d[i + 1] - l, en = i + 2 < end ? e[i + 1] : 0.0, yn = rhs(i + 1);
        const size_t at = static_cast<size_t>(i) * nb;
        const bool keep = fabs(a) >= fabs(ei);
        double pivot = keep ? a : ei;
        if (fabs(pivot) < tiny) pivot = copysign(tiny, pivot);
        const double ui = recip_f64(pivot), m = (keep ? ei : a) * ui;
        U0[at] = ui;
        U1[at] = keep ? b : dn;
        U2[at] = keep ? 0.0 : en;
        Y[at] = keep ? y : yn;
        const double a2 = keep ? fma(-m, b, dn) : fma(-m, dn, b);
        b = keep ? en : -m * en;
        y = keep ? fma(-m, y, yn) : fma(-m, yn, y);
        a = a2;
    }
    if (fabs(a) < tiny) a = copysign(tiny, a);
    double x1 = y * recip_f64(a), x2 = 0.0, ss = x1 * x1;
    Z[static_cast<size_t>(end - 1) * r_max + j] = x1;
#pragma unroll 4
    for (int i = end - 2; i >= beg; --i) {
        const size_t at = static_cast<size_t>(i) * nb;
        const double x = fma(-U2[at], x2, fma(-U1[at], x1, Y[at])) * U0[at];
        Z[static_cast<size_t>(i) * r_max + j] = x;
        ss = fma(x, x, ss);
        x2 = x1;
        x1 = x;
    }
    for (int i = 0; i < beg; ++i) Z[static_cast<size_t>(i) * r_max + j] = 0.0;
    for (int i = end; i < n; ++i) Z[static_cast<size_t>(i) * r_max + j] = 0.0;
    scale[j] = ss > 0.0 ? 1.0 / sqrt(ss) : 0.0;
}

// Sums over the wave of 8 values per lane: lane l is left with the sum of value
// l >> 3 (bits 5, 4, 3 of l choose the halves that it keeps).
__device__ __forceinline__ double wave_sum8_f64(double (&v)[8]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int h = 4, off = 32; h > 0; h >>= 1, off >>= 1) {
        const bool upper = lane & off;
#pragma unroll
        for (int u = 0; u < h; ++u) {
            const double keep = upper ? v[u + h] : v[u], give = upper ? v[u] : v[u + h];
            v[u] = keep + __shfl_xor(give, off, 64);
        }
    }
    double s = v[0];
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    return s;
}

// The iterates to unit length (scale 1), and those of a block's runs of
// eigenvalues closer than kCluster |T| orthogonal: classical Gram-Schmidt
// against 8 vectors at a time, twice (once leaves the rounding that the first
// pass's cancellation magnified).  One workgroup per run; the vectors of its
// other ranks leave at once.  Vectors of eigenvalue zero are multiplied by
// sigma = 0 afterwards and stay as they are.  A thread keeps its CPT entries
// of the vector in registers and reads the finished ones from rows W[rank][i]
// of a copy.  Bound by the chain of a run, 2.4 us for each 8 vectors and pass:
// 1024 x 1024 of rank 4, 252 eigenvalues of rounding size in one run, 46 ms the
// call (one vector at a time, modified Gram-Schmidt on the columns of Z: 221).
template <int CPT>
__global__ __launch_bounds__(256) void orthogonalise_kernel(const double* __restrict__ row_lam,
                                                            const int2* __restrict__ blk,
                                                            const int* __restrict__ order,
                                                            const int* __restrict__ rank_of,
                                                            const double* __restrict__ bounds, int n, int r_max,
                                                            double* __restrict__ Z, double* __restrict__ scale,
                                                            double* W) {
    constexpr int QB = 8, KEEP = CPT <= 4 ? CPT : 1;   // entries kept between the two uses of a vector
    __shared__ double red[2][QB][4];
    const int tid = threadIdx.x, lane = tid & 63;
    const double tol = kCluster * bounds[2];
    int s = order[blockIdx.x];
    const int beg = blk[s].x, end = blk[s].y;
    auto close = [&](int i) { return i > beg && row_lam[i] > 0.0 && row_lam[i - 1] - row_lam[i] <= tol; };
    if (close(s)) return;
    const int head = s;
    int par = 0;
    double z[CPT];
    do {
        const int m = rank_of[s];
        const double sm = scale[m];
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int i = tid + 256 * c;
            z[c] = i < n ? sm * Z[static_cast<size_t>(i) * r_max + m] : 0.0;
        }
        for (int pass = 0; pass < 2 && s > head; ++pass) {
            for (int q0 = head; q0 < s; q0 += QB) {
                const double* row[QB];
                double w[QB][KEEP], dot[QB];
#pragma unroll
                for (int u = 0; u < QB; ++u) {
                    row[u] = W + static_cast<size_t>(rank_of[min(q0 + u, s - 1)]) * n;
                    dot[u] = 0.0;
                }
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    const int i = min(tid + 256 * c, n - 1);     // z[c] is 0 past n
#pragma unroll
                    for (int u = 0; u < QB; ++u) {
                        const double v = row[u][i];
                        dot[u] = fma(z[c], v, dot[u]);
                        if (KEEP == CPT) w[u][c < KEEP ? c : 0] = v;
                    }
                }
                const double d = wave_sum8_f64(dot);
                if ((lane & 7) == 0) red[par][lane >> 3][tid >> 6] = d;
                __syncthreads();
#pragma unroll
                for (int u = 0; u < QB; ++u) {
                    const double* r = red[par][u];
                    dot[u] = q0 + u < s ? (r[0] + r[1]) + (r[2] + r[3]) : 0.0;
                }
                par ^= 1;
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    const int i = min(tid + 256 * c, n - 1);
                    double v = z[c];
#pragma unroll
                    for (int u = 0; u < QB; ++u)
                        v = fma(-dot[u], KEEP == CPT ? w[u][c < KEEP ? c : 0] : row[u][i], v);
                    z[c] = tid + 256 * c < n ? v : 0.0;
                }
            }
            double ss = 0.0;
#pragma unroll
            for (int c = 0; c < CPT; ++c) ss = fma(z[c], z[c], ss);
            ss = block_sum_f64(ss, red[par][0]);
            par ^= 1;
            const double inv = ss > 0.0 ? 1.0 / sqrt(ss) : 0.0;
#pragma unroll
            for (int c = 0; c < CPT; ++c) z[c] *= inv;
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int i = tid + 256 * c;
            if (i < n) {
                Z[static_cast<size_t>(i) * r_max + m] = z[c];
                W[static_cast<size_t>(m) * n + i] = z[c];
            }
        }
        __syncthreads();                         // the row of W is there, and scale[m] was read
        if (tid == 0) scale[m] = 1.0;
        ++s;
    } while (s < end && close(s) && rank_of[s] < r_max);
}

// bounds[5] = the worst of vector j's |T z - lambda z| / |T| and of its inner
// products with the others, each over its tolerance (products with vectors of
// eigenvalue zero apart); 1e300 where one is not a number.  Row j of M = (3 I -
// Z^T Z) / 2: Z M is orthonormal to the square of Z's own error, 1e-9 to 1e-18
// (one step of Newton's iteration for the polar factor).  One workgroup per
// vector; a thread sums every parts-th row of one other's product, a wave's
// threads along a row of Z.  The bits of a positive double are in its order.
// Bound by the chain of its loads, 16 at a time: 128 vectors of 1024, 44 us (the
// products on the matrix cores, four workgroups for want of tiles, and the check
// in a launch of its own 62 + 13 us).
__global__ __launch_bounds__(256) void check_kernel(const double* __restrict__ d, const double* __restrict__ e, int n,
                                                    const double* __restrict__ lam, int r_max,
                                                    const double* __restrict__ Z, double* __restrict__ M,
                                                    double* __restrict__ bounds) {
    __shared__ double red[4], part[256];
    const int j = blockIdx.x, tid = threadIdx.x;
    const double norm = bounds[2] > 0.0 ? bounds[2] : 1.0, l = lam[j];
    auto z = [&](int i) { return Z[static_cast<size_t>(i) * r_max + j]; };
    double ss = 0.0;
    for (int i = tid; i < n; i += 256) {
        double v = (d[i] - l) * z(i);
        if (i > 0) v = fma(e[i - 1], z(i - 1), v);
        if (i + 1 < n) v = fma(e[i], z(i + 1), v);
        ss = fma(v, v, ss);
    }
    ss = block_sum_f64(ss, red);
    double worst = sqrt(ss) / (norm * kResidualTol);
    const int parts = 256 / r_max, k = tid % r_max, p = tid / r_max;
    double g = 0.0;
    if (p < parts) {
#pragma unroll 16
        for (int i = p; i < n; i += parts) g = fma(z(i), Z[static_cast<size_t>(i) * r_max + k], g);
    }
    part[tid] = g;
    __syncthreads();
    if (tid < r_max) {
        for (int u = 1; u < parts; ++u) g += part[u * r_max + tid];
        const double one = tid == j ? 1.0 : 0.0;
        const double off = tid == j || (l > 0.0 && lam[tid] > 0.0) ? g - one : 0.0;
        M[static_cast<size_t>(j) * r_max + tid] = fma(-0.5, off, one);
        const double o = fabs(off) / kOrthogonalTol;
        worst = o <= worst ? worst : o;
    }
    if (!(worst < 1e300)) worst = 1e300;
    atomicMax(reinterpret_cast<unsigned long long*>(bounds + 5), __builtin_bit_cast(unsigned long long, worst));
}

// X = Q Z: the reflectors applied in reverse to vector j, one workgroup each,
// CPT entries per thread in registers; the next reflector is loaded while
// this one's dot product is summed.  Xr[j][i] = X[i][j].
template <int CPT>
__global__ __launch_bounds__(256) void back_transform_kernel(const double* __restrict__ V,
                                                             const double* __restrict__ tau, int n, int r_max,
                                                             const double* __restrict__ Z,
                                                             double* __restrict__ Xr) {
    __shared__ double red[2][4];
    const int j = blockIdx.x, tid = threadIdx.x;
    double z[CPT], v[CPT];
    auto load = [&](int k) {
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int i = tid + 256 * c;
            v[c] = i > k && i < n ? V[static_cast<size_t>(k) * n + i] : 0.0;
        }
    };
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int i = tid + 256 * c;
        z[c] = i < n ? Z[static_cast<size_t>(i) * r_max + j] : 0.0;
    }
    if (n > 2) load(n - 3);
    for (int k = n - 3; k >= 0; --k) {
        double dot = 0.0, u[CPT];
        const double t = tau[k];
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            u[c] = v[c];
            dot = fma(v[c], z[c], dot);
        }
        if (k > 0) load(k - 1);
        dot = -t * block_sum_f64(dot, red[k & 1]);
#pragma unroll
        for (int c = 0; c < CPT; ++c) z[c] = fma(dot, u[c], z[c]);
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int i = tid + 256 * c;
        if (i < n) Xr[static_cast<size_t>(j) * n + i] = z[c];
    }
}

// sign[j] = +-1 so that the largest-magnitude entry (first index on ties) of
// U column j, u[i * stride + j * jstride] for i < len, becomes positive.
__global__ __launch_bounds__(256) void sign_kernel(const double* __restrict__ u, size_t stride, size_t jstride, int len,
                                                   double* __restrict__ sign) {
    __shared__ double bv[256];
    __shared__ int bi[256];
    const int j = blockIdx.x;
    double best = -1.0, val = 0.0;
    int bidx = 0x7fffffff;
    for (int i = threadIdx.x; i < len; i += 256) {
        const double x = u[i * stride + j * jstride];
        if (fabs(x) > best) { best = fabs(x); bidx = i; val = x; }
    }
    bv[threadIdx.x] = best;
    bi[threadIdx.x] = bidx;
    __shared__ double vv[256];
    vv[threadIdx.x] = val;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            const double o = bv[threadIdx.x + s];
            const int oi = bi[threadIdx.x + s];
            if (o > bv[threadIdx.x] || (o == bv[threadIdx.x] && oi < bi[threadIdx.x])) {
                bv[threadIdx.x] = o;
                bi[threadIdx.x] = oi;
                vv[threadIdx.x] = vv[threadIdx.x + s];
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) sign[j] = vv[0] < 0.0 ? -1.0 : 1.0;
}

// fp16 factors.  right: X held right vectors (Xr = V^T rows, P = E V);
// otherwise left vectors (Xr = U^T rows, P = U^T E).
__global__ __launch_bounds__(256) void factor_a_kernel(const double* __restrict__ Xr, const double* __restrict__ P,
                                                       const double* __restrict__ lam, const double* __restrict__ sign,
                                                       int r_max, int d_in, bool right, uint16_t* __restrict__ A) {
    const size_t idx = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    if (idx >= static_cast<size_t>(r_max) * d_in) return;
    const int j = static_cast<int>(idx / d_in);
    const double sg = sqrt(lam[j] > 0.0 ? lam[j] : 0.0);
    const double root = sqrt(sg);
    double v;
    if (right) v = root * Xr[idx];
    else v = sg > 0.0 ? P[idx] / root : 0.0;
    A[idx] = f64_to_f16_rne(sign[j] * v);
}

__global__ __launch_bounds__(256) void factor_b_kernel(const double* __restrict__ Xr, const double* __restrict__ P,
                                                       const double* __restrict__ lam, const double* __restrict__ sign,
                                                       int r_max, int d_out, bool right, uint16_t* __restrict__ B) {
    const size_t idx = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    if (idx >= static_cast<size_t>(d_out) * r_max) return;
    const int o = static_cast<int>(idx / r_max), j = static_cast<int>(idx % r_max);
    const double sg = sqrt(lam[j] > 0.0 ? lam[j] : 0.0);
    const double root = sqrt(sg);
    double v;
    if (right) v = sg > 0.0 ? P[idx] / root : 0.0;                 // P is [d_out][r_max]
    else v = root * Xr[static_cast<size_t>(j) * d_out + o];
    B[idx] = f64_to_f16_rne(sign[j] * v);
}

unsigned grid1(size_t n) { return static_cast<unsigned>((n + 255) / 256); }

template <bool XK1, bool YK1>
void gemm(const double* X, size_t xi, size_t xk, const double* Y, size_t yj, size_t yk, int I, int J, int K,
          double* out, size_t ldo, hipStream_t st) {
    dim3 grid((J + 63) / 64, (I + 63) / 64);
    hipLaunchKernelGGL((gemm_nt_f64<XK1, YK1>), grid, dim3(256), 0, st, X, xi, xk, Y, yj, yk, I, J, K, out, ldo);
}

}  // namespace

bool comp_fits(int d_out, int d_in) {
    const int n = d_in <= d_out ? d_in : d_out;
    return n <= 8192 && static_cast<long long>(d_out) * d_in <= (1ll << 31);
}

size_t comp_workspace_bytes(int d_out, int d_in, int r_max) {
    return comp_layout(d_out, d_in, r_max).total;
}

namespace {

// Columns per thread for `cols` columns over 256 threads.
template <typename F>
void by_columns(int cols, F f) {
    if (cols <= 256) f(std::integral_constant<int, 1>());
    else if (cols <= 512) f(std::integral_constant<int, 2>());
    else if (cols <= 1024) f(std::integral_constant<int, 4>());
    else if (cols <= 2048) f(std::integral_constant<int, 8>());
    else if (cols <= 4096) f(std::integral_constant<int, 16>());
    else f(std::integral_constant<int, 32>());
}

}  // namespace

hipError_t launch_build_compensation(const float* W, const QW& w, int r_max, uint16_t* A, uint16_t* B, float* sigma,
                                     void* ws, hipStream_t st, int* sweeps_out) {
    const int d_out = w.d_out, d_in = w.d_in;
    const bool right = d_in <= d_out;              // Gram over d_in: eigenvectors are V
    const int n = right ? d_in : d_out;
    const CompLayout l = comp_layout(d_out, d_in, r_max);
    char* base = static_cast<char*>(ws);
    auto at = [&](size_t off) { return reinterpret_cast<double*>(base + off); };
    double *E = at(l.E), *C = at(l.C), *V = at(l.V), *tau = at(l.tau), *lam = at(l.lam), *d = at(l.d), *e = at(l.e);
    double *p[2] = {at(l.p), at(l.p) + n}, *bounds = at(l.bounds), *scale = at(l.scale), *sign = at(l.sign);
    double *Xr = at(l.Xr), *P = at(l.P);
    double* row_lam = at(l.row_lam);
    double2* de = reinterpret_cast<double2*>(base + l.de);
    int2* blk = reinterpret_cast<int2*>(base + l.blk);
    int *order = reinterpret_cast<int*>(base + l.order), *rank_of = reinterpret_cast<int*>(base + l.rank_of);
    hipError_t err;

    const size_t total = static_cast<size_t>(d_out) * d_in;
    hipLaunchKernelGGL(residual_kernel, dim3(grid1(total)), dim3(256), 0, st, W, w, E);
    // Gram: C[i][j] = sum_k E_k,i E_k,j over the larger side
    if (right) gemm<false, false>(E, 1, d_in, E, 1, d_in, n, n, d_out, C, n, st);
    else gemm<true, true>(E, d_in, 1, E, d_in, 1, n, n, d_in, C, n, st);

    for (int k = 0; k < n; ++k) {
        by_columns(n - (k & ~63), [&](auto cpt) {
            // rows in hand per workgroup, and workgroups: two per CU where the
            // trailing matrix has the rows (1024 x 4096 7.97 -> 7.37 ms, 4096 x
            // 4096 128 -> 105 ms against 256 workgroups of 4 rows in hand)
            constexpr int CPT = decltype(cpt)::value, R = CPT <= 2 ? 1 : 2, G = CPT == 1 ? 256 : 512;
            hipLaunchKernelGGL((householder_step_kernel<CPT, R>), dim3(n < G ? n : G), dim3(256), 0, st, C, n, k, V,
                               p[k & 1], p[(k & 1) ^ 1], tau, d, e);
        });
    }
    hipLaunchKernelGGL(tridiagonal_prep_kernel, dim3(1), dim3(256), 0, st, d, e, n, de, blk, bounds);
    hipLaunchKernelGGL(bisect_kernel, dim3((n + 3) / 4), dim3(256), 0, st, de, blk, n, bounds, row_lam);
    hipLaunchKernelGGL(order_kernel, dim3(grid1(n)), dim3(256), 0, st, row_lam, blk, n, bounds, lam, order, rank_of,
                       sigma);
    // sweeps of inverse iteration, two at first and then one at a time, until
    // the vectors pass the check; each time the host waits for its outcome (W
    // has been read then, and a fault of the work so far is reported by this call)
    int sweeps = 0;
    do {
        // C is free now: the eliminations of n / 4 vectors at a time (4 planes
        // of n each); the iterates in P until the product with E needs it, the
        // finished ones row by row, then the check's M, in Xr; the
        // orthonormal ones in C
        const int batch = n < 4 ? 1 : n / 4, until = sweeps == 0 ? kInverseSweeps : sweeps + 1;
        for (; r_max > 0 && sweeps < until; ++sweeps) {
            for (int j0 = 0; j0 < r_max; j0 += batch) {
                const int nb = r_max - j0 < batch ? r_max - j0 : batch;
                hipLaunchKernelGGL(inverse_iteration_kernel, dim3((nb + 63) / 64), dim3(64), 0, st, d, e, n, bounds,
                                   row_lam, blk, order, j0, nb, r_max, sweeps == 0, C, P, scale);
            }
            by_columns(n, [&](auto cpt) {
                hipLaunchKernelGGL((orthogonalise_kernel<decltype(cpt)::value>), dim3(r_max), dim3(256), 0, st, row_lam,
                                   blk, order, rank_of, bounds, n, r_max, P, scale, Xr);
            });
        }
        if (r_max > 0) {
            hipLaunchKernelGGL(check_kernel, dim3(r_max), dim3(256), 0, st, d, e, n, lam, r_max, P, Xr, bounds);
            gemm<true, false>(P, r_max, 1, Xr, 1, r_max, n, r_max, r_max, C, r_max, st);
            by_columns(n, [&](auto cpt) {
                hipLaunchKernelGGL((back_transform_kernel<decltype(cpt)::value>), dim3(r_max), dim3(256), 0, st, V, tau,
                                   n, r_max, C, Xr);
            });
        }
        if ((err = hipGetLastError()) != hipSuccess) return err;
        double state[2];                          // T not finite; the worst check
        if ((err = hipMemcpyAsync(state, bounds + 4, sizeof(state), hipMemcpyDeviceToHost, st)) != hipSuccess)
            return err;
        if ((err = hipStreamSynchronize(st)) != hipSuccess) return err;
        *sweeps_out = r_max > 0 ? sweeps : 1;
        if (state[0] != 0.0) {
            *sweeps_out = 0;
            return hipErrorNotReady;
        }
        if (r_max == 0 || state[1] <= 1.0) break;
        if (sweeps == kMaxSweeps) return hipErrorNotReady;
    } while (true);

    if (r_max > 0) {
        if (right) {
            // P[o][j] = sum_c E[o][c] V[c][j]
            gemm<true, true>(E, d_in, 1, Xr, d_in, 1, d_out, r_max, d_in, P, r_max, st);
            hipLaunchKernelGGL(sign_kernel, dim3(r_max), dim3(256), 0, st, P, static_cast<size_t>(r_max),
                               static_cast<size_t>(1), d_out, sign);
        } else {
            // P[j][c] = sum_o U[o][j] E[o][c]
            gemm<true, false>(Xr, d_out, 1, E, 1, d_in, r_max, d_in, d_out, P, d_in, st);
            hipLaunchKernelGGL(sign_kernel, dim3(r_max), dim3(256), 0, st, Xr, static_cast<size_t>(1),
                               static_cast<size_t>(d_out), d_out, sign);
        }
        hipLaunchKernelGGL(factor_a_kernel, dim3(grid1(static_cast<size_t>(r_max) * d_in)), dim3(256), 0, st, Xr, P,
                           lam, sign, r_max, d_in, right, A);
        hipLaunchKernelGGL(factor_b_kernel, dim3(grid1(static_cast<size_t>(d_out) * r_max)), dim3(256), 0, st, Xr, P,
                           lam, sign, r_max, d_out, right, B);
    }
    return hipGetLastError();
}

}  // namespace cl
