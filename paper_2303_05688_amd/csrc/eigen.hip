// The variational step of the ASCI loop on one GPU (Sec. II.C): the
// Hamiltonian over a determinant set by the double loop over determinant
// pairs, stored as CSR, its product with a vector, and the Davidson method
// (Alg. 5) with the shifted-Jacobi (diagonal) preconditioner.
//
// H: rows in the order of the determinant set, columns ascending, both
// triangles and the diagonal stored.  Matrix elements use the same
// Slater-Condon routines (and the same operation order) as the search.
#include "pairs.h"

#include <cmath>
#include <cstring>

namespace asci {

namespace {

constexpr int kChunk = 4096;      // counts per chunk of the row-pointer scan

// 64-bit exclusive scan of the counts by row and share, chunk by chunk; a
// row starts with its first share
__global__ __launch_bounds__(256) void k_chunk_sums(const uint32_t *__restrict__ cnt, size_t n,
                                                    unsigned long long *__restrict__ sums)
{
    __shared__ unsigned long long s[256];
    const size_t base = (size_t)blockIdx.x * kChunk;
    unsigned long long acc = 0;
    for (uint32_t i = threadIdx.x; i < kChunk && base + i < n; i += 256) acc += cnt[base + i];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = s[0];
}

__global__ __launch_bounds__(256) void k_chunk_scan(const uint32_t *__restrict__ cnt, size_t n, uint32_t shares,
                                                    const unsigned long long *__restrict__ base,
                                                    int64_t *__restrict__ start, int64_t *__restrict__ rowptr)
{
    constexpr int per = kChunk / 256;
    __shared__ unsigned long long s[256];
    const size_t c0 = (size_t)blockIdx.x * kChunk + threadIdx.x * per;
    uint32_t v[per];
    unsigned long long tot = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        v[k] = (c0 + k < n) ? cnt[c0 + k] : 0u;
        tot += v[k];
    }
    s[threadIdx.x] = tot;
    __syncthreads();
    // Hillis-Steele inclusive scan of the thread totals
    for (int d = 1; d < 256; d <<= 1) {
        const unsigned long long add = (int)threadIdx.x >= d ? s[threadIdx.x - d] : 0ull;
        __syncthreads();
        s[threadIdx.x] += add;
        __syncthreads();
    }
    unsigned long long run = base[blockIdx.x] + s[threadIdx.x] - tot;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        if (c0 + k < n) {
            start[c0 + k] = (int64_t)run;
            if ((c0 + k) % shares == 0) rowptr[(c0 + k) / shares] = (int64_t)run;
        }
        run += v[k];
    }
}

// ---------------------------------------------------------------- vectors
// y = H x, one wavefront per row (lane-strided, then a fixed shuffle tree)
__global__ __launch_bounds__(256) void k_spmv(const int64_t *__restrict__ rowptr, const int32_t *__restrict__ cols,
                                              const double *__restrict__ vals, const double *__restrict__ x,
                                              double *__restrict__ y, uint32_t nrows)
{
    const uint32_t row = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= nrows) return;
    double acc = 0.0;
    for (int64_t k = rowptr[row] + lane; k < rowptr[row + 1]; k += 64) acc = acc + vals[k] * x[cols[k]];
    for (int d = 32; d >= 1; d >>= 1) acc = acc + __shfl_xor(acc, d, 64);
    if (lane == 0) y[row] = acc;
}

constexpr int kDotBlocks = 512;
constexpr int kMaxSub = 48;           // largest Davidson subspace
constexpr int kPartLd = kMaxSub + 4;  // partial sums: a row per block; behind the columns' the three norms
enum { kNormR = kMaxSub, kNormT = kMaxSub + 1, kNormV = kMaxSub + 2 };
constexpr int kDotCols = 4;           // columns a workgroup of k_multidot takes: one read of x for four

struct SubCoef {
    double c[kMaxSub];
};

// the block's sum of acc in thread 0, in one order whatever the kernel (a tree
// over the threads, halves first)
__device__ __forceinline__ double block_tree(double acc, double *s_red)
{
    const int tid = threadIdx.x;
    __syncthreads();
    s_red[tid] = acc;
    __syncthreads();
    if (tid < 64) {
        acc = (s_red[tid] + s_red[tid + 128]) + (s_red[tid + 64] + s_red[tid + 192]);
        for (int w = 32; w >= 1; w >>= 1) acc = acc + __shfl_down(acc, w, 64);
    }
    return acc;
}

// sum over the nb blocks' partials of column j, ascending; 32 loads in flight
__device__ __forceinline__ double sum_partials(const double *__restrict__ partial, int j, int nb)
{
    double acc = 0.0;
    for (int b0 = 0; b0 < nb; b0 += 32) {
        double v[32];
#pragma unroll
        for (int k = 0; k < 32; ++k) v[k] = b0 + k < nb ? partial[(size_t)(b0 + k) * kPartLd + j] : 0.0;
#pragma unroll
        for (int k = 0; k < 32; ++k) acc = acc + v[k];
    }
    return acc;
}

// partial[b][j] = sum over block b's share of i of V[j][i] * x[i], for the
// kDotCols columns of blockIdx.y.  At 5000 rows one workgroup for all of 12
// columns took 7.1 us, most of it in the barriers of one column after another.
__global__ __launch_bounds__(256) void k_multidot(const double *__restrict__ V, size_t ld, int m,
                                                  const double *__restrict__ x, size_t n,
                                                  double *__restrict__ partial)
{
    __shared__ double s_red[256];
    const int j0 = blockIdx.y * kDotCols;
    double acc[kDotCols] = {};
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const double xi = x[i];
#pragma unroll
        for (int j = 0; j < kDotCols; ++j)
            if (j0 + j < m) acc[j] = acc[j] + V[(size_t)(j0 + j) * ld + i] * xi;
    }
#pragma unroll
    for (int j = 0; j < kDotCols; ++j) {
        if (j0 + j >= m) break;
        const double t = block_tree(acc[j], s_red);
        if (threadIdx.x == 0) partial[(size_t)blockIdx.x * kPartLd + j0 + j] = t;
    }
}

// out[0, m) and the three norms behind them
__global__ __launch_bounds__(64) void k_rowsum(const double *__restrict__ partial, int m, int nb,
                                               double *__restrict__ out)
{
    const int j = threadIdx.x;
    if (j < m || (j >= kMaxSub && j < kPartLd - 1)) out[j] = sum_partials(partial, j, nb);
}

// The Ritz vector u = V c, wc = W c, the residual wc - theta u and from it
// t = residual / (D - theta), the denominator kept away from zero; the partial
// sums of their squares.  restart: u and wc become the first columns.
__global__ __launch_bounds__(256) void k_ritz(double *__restrict__ V, double *__restrict__ W, size_t ld, int m,
                                              SubCoef c, double theta, const double *__restrict__ diag, size_t n,
                                              double *__restrict__ u, double *__restrict__ t, int restart,
                                              double *__restrict__ partial)
{
    __shared__ double s_red[256];
    double rr = 0.0, tt = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        double a = 0.0, b = 0.0;
#pragma unroll 4
        for (int j = 0; j < m; ++j) {
            a = a + c.c[j] * V[(size_t)j * ld + i];
            b = b + c.c[j] * W[(size_t)j * ld + i];
        }
        u[i] = a;
        if (restart) {
            V[i] = a;
            W[i] = b;
        }
        const double r = b - theta * a;
        double d = diag[i] - theta;
        if (fabs(d) < 1e-8) d = d < 0.0 ? -1e-8 : 1e-8;
        const double x = r / d;
        t[i] = x;
        rr = rr + r * r;
        tt = tt + x * x;
    }
    rr = block_tree(rr, s_red);
    tt = block_tree(tt, s_red);
    if (threadIdx.x == 0) {
        partial[(size_t)blockIdx.x * kPartLd + kNormR] = rr;
        partial[(size_t)blockIdx.x * kPartLd + kNormT] = tt;
    }
}

// t = t - sum_j h[j] V[j], h the sums of the dots' partials; norm: the partial
// sums of t's squares too
__global__ __launch_bounds__(256) void k_orth(const double *__restrict__ V, size_t ld, int m, size_t n,
                                              double *__restrict__ t, const double *__restrict__ dots,
                                              double *__restrict__ norm)
{
    __shared__ double s_h[kMaxSub], s_red[256];
    if ((int)threadIdx.x < m) s_h[threadIdx.x] = sum_partials(dots, (int)threadIdx.x, (int)gridDim.x);
    __syncthreads();
    double tt = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        double acc = t[i];
#pragma unroll 4
        for (int j = 0; j < m; ++j) acc = acc - s_h[j] * V[(size_t)j * ld + i];
        t[i] = acc;
        tt = tt + acc * acc;
    }
    if (!norm) return;
    tt = block_tree(tt, s_red);
    if (threadIdx.x == 0) norm[(size_t)blockIdx.x * kPartLd + kNormV] = tt;
}

// y = x / |x|, the square of |x| in the partial sums of column kNormV
__global__ __launch_bounds__(256) void k_normalise(const double *__restrict__ x, size_t n,
                                                   const double *__restrict__ partial, double *__restrict__ y)
{
    __shared__ double s_a;
    if (threadIdx.x == 0) s_a = 1.0 / sqrt(sum_partials(partial, kNormV, (int)gridDim.x));
    __syncthreads();
    const double a = s_a;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) y[i] = a * x[i];
}

// the partial sums of x's squares, column kNormV
__global__ __launch_bounds__(256) void k_norm(const double *__restrict__ x, size_t n, double *__restrict__ partial)
{
    __shared__ double s_red[256];
    double tt = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) tt = tt + x[i] * x[i];
    tt = block_tree(tt, s_red);
    if (threadIdx.x == 0) partial[(size_t)blockIdx.x * kPartLd + kNormV] = tt;
}

// The sign that cyclic Jacobi rotations (Golub and Van Loan, Sec. 8.5) give the
// eigenvector vec of A: one sweep after the other until a column of their
// product is within 0.99 of it (mostly one or two; none once the first vector
// of the subspace is).  Every rotation is by at most 45 degrees, so the column
// keeps its side from there on.
double jacobi_sign(const std::vector<double> &A_in, int ld, int m, const double *vec)
{
    double A[kMaxSub][kMaxSub], Q[kMaxSub][kMaxSub];  // Q: a column of the product per row
    for (int i = 0; i < m; ++i)
        for (int j = 0; j < m; ++j) {
            A[i][j] = A_in[(size_t)i * ld + j];
            Q[i][j] = i == j ? 1.0 : 0.0;
        }
    double best = 0.0;
    for (int sweep = 0;; ++sweep) {
        best = 0.0;
        for (int k = 0; k < m; ++k) {
            double x = 0.0;
            for (int j = 0; j < m; ++j) x += Q[k][j] * vec[j];
            if (std::fabs(x) > std::fabs(best)) best = x;
        }
        if (!(std::fabs(best) < 0.99) || sweep == 30) break;
        for (int p = 0; p < m - 1; ++p)
            for (int q = p + 1; q < m; ++q) {
                const double apq = A[p][q];
                if (apq == 0.0) continue;
                const double app = A[p][p], aqq = A[q][q];
                const double tau = (aqq - app) / (2.0 * apq);
                const double t = (tau >= 0.0 ? 1.0 : -1.0) / (std::fabs(tau) + std::sqrt(1.0 + tau * tau));
                const double c = 1.0 / std::sqrt(1.0 + t * t), s = t * c;
                for (int k = 0; k < m; ++k) {
                    const double x = A[p][k], y = A[q][k];
                    A[p][k] = c * x - s * y;
                    A[q][k] = s * x + c * y;
                    const double u = Q[p][k], v = Q[q][k];
                    Q[p][k] = c * u - s * v;
                    Q[q][k] = s * u + c * v;
                }
                A[p][p] = app - t * apq;
                A[q][q] = aqq + t * apq;
                A[p][q] = A[q][p] = 0.0;
                for (int k = 0; k < m; ++k) {
                    A[k][p] = A[p][k];
                    A[k][q] = A[q][k];
                }
            }
    }
    return best < 0.0 ? -1.0 : 1.0;
}

// Lowest eigenpair of a small symmetric matrix (the first m rows and columns of
// A, leading dimension ld): Householder reduction to tridiagonal form (Golub
// and Van Loan, Alg. 8.3.1), the lowest eigenvalue by bisection on Sturm counts
// (Sec. 8.4.1), its vector by inverse iteration.  m = 20 takes 50 us with the
// sign; Jacobi rotations to the end, which this took the place of, took 123 and
// left larger residuals.
void small_lowest(const std::vector<double> &A_in, int ld, int m, double &theta, double *vec)
{
    double A[kMaxSub][kMaxSub], d[kMaxSub], e[kMaxSub], x[kMaxSub], p[kMaxSub];
    for (int i = 0; i < m; ++i)
        for (int j = 0; j < m; ++j) A[i][j] = A_in[(size_t)i * ld + j];
    double beta[kMaxSub];  // reflector k: rows k+1.. of column k hold its vector
    for (int k = 0; k + 2 < m; ++k) {
        double sigma = 0.0;
        for (int i = k + 2; i < m; ++i) sigma += A[i][k] * A[i][k];
        const double x0 = A[k + 1][k];
        beta[k] = 0.0;
        e[k] = x0;
        if (sigma == 0.0) continue;
        const double mu = std::sqrt(x0 * x0 + sigma);
        const double v0 = x0 <= 0.0 ? x0 - mu : -sigma / (x0 + mu);
        e[k] = mu;
        beta[k] = 2.0 * v0 * v0 / (sigma + v0 * v0);
        A[k + 1][k] = 1.0;
        for (int i = k + 2; i < m; ++i) A[i][k] /= v0;
        double pv = 0.0;
        for (int i = k + 1; i < m; ++i) {
            double acc = 0.0;
            for (int j = k + 1; j < m; ++j) acc += A[i][j] * A[j][k];
            p[i] = beta[k] * acc;
            pv += p[i] * A[i][k];
        }
        for (int i = k + 1; i < m; ++i) p[i] -= 0.5 * beta[k] * pv * A[i][k];
        for (int i = k + 1; i < m; ++i)
            for (int j = k + 1; j < m; ++j) A[i][j] -= A[i][k] * p[j] + p[i] * A[j][k];
    }
    double lo = 0.0, hi = 0.0, norm = 0.0;
    if (m >= 2) e[m - 2] = A[m - 1][m - 2];
    for (int i = 0; i < m; ++i) {
        d[i] = A[i][i];
        const double r = (i > 0 ? std::fabs(e[i - 1]) : 0.0) + (i + 1 < m ? std::fabs(e[i]) : 0.0);
        lo = i == 0 ? d[i] - r : std::min(lo, d[i] - r);
        hi = i == 0 ? d[i] : std::min(hi, d[i]);  // no eigenvalue bound is larger than a diagonal element
        norm = std::max(norm, std::fabs(d[i]) + r);
    }
    const double tiny = std::max(norm, 1e-250) * 0x1p-52;
    // lo has no eigenvalue below it, hi (a little above the smallest diagonal element) at least one
    hi += tiny;
    lo -= tiny;
    for (int it = 0; it < 200; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (!(mid > lo && mid < hi)) break;
        bool below = false;
        double q = d[0] - mid;
        for (int i = 0; !(below = q < 0.0) && i + 1 < m; ++i) {
            if (q == 0.0) q = tiny;
            q = d[i + 1] - mid - e[i] * e[i] / q;
        }
        if (below) hi = mid;
        else lo = mid;
    }
    theta = 0.5 * (lo + hi);
    // (T - theta) = P L U by rows, pivoting between neighbours
    double u0[kMaxSub], u1[kMaxSub], u2[kMaxSub], l[kMaxSub];
    bool sw[kMaxSub];
    {
        double a = d[0] - theta, b = m > 1 ? e[0] : 0.0;
        for (int i = 0; i + 1 < m; ++i) {
            const double s0 = e[i], s1 = d[i + 1] - theta, s2 = i + 2 < m ? e[i + 1] : 0.0;
            sw[i] = std::fabs(s0) > std::fabs(a);
            if (sw[i]) {
                l[i] = a / s0;
                u0[i] = s0;
                u1[i] = s1;
                u2[i] = s2;
                a = b - l[i] * s1;
                b = -l[i] * s2;
            } else {
                if (std::fabs(a) < tiny) a = tiny;
                l[i] = s0 / a;
                u0[i] = a;
                u1[i] = b;
                u2[i] = 0.0;
                a = s1 - l[i] * b;
                b = s2;
            }
        }
        u0[m - 1] = std::fabs(a) < tiny ? tiny : a;
        u1[m - 1] = u2[m - 1] = 0.0;
    }
    for (int i = 0; i < m; ++i) x[i] = 1.0;
    for (int it = 0; it < 4; ++it) {
        if (it > 0)
            for (int i = 0; i + 1 < m; ++i) {
                if (sw[i]) std::swap(x[i], x[i + 1]);
                x[i + 1] -= l[i] * x[i];
            }
        double big = 0.0;
        for (int i = m - 1; i >= 0; --i) {
            double r = x[i];
            if (i + 1 < m) r -= u1[i] * x[i + 1];
            if (i + 2 < m) r -= u2[i] * x[i + 2];
            x[i] = r / u0[i];
            big = std::max(big, std::fabs(x[i]));
        }
        for (int i = 0; i < m; ++i) x[i] /= big;
    }
    for (int k = m - 3; k >= 0; --k) {
        if (beta[k] == 0.0) continue;
        double acc = 0.0;
        for (int i = k + 1; i < m; ++i) acc += A[i][k] * x[i];
        acc *= beta[k];
        for (int i = k + 1; i < m; ++i) x[i] -= acc * A[i][k];
    }
    double nrm = 0.0;
    for (int i = 0; i < m; ++i) nrm += x[i] * x[i];
    nrm = std::sqrt(nrm);
    for (int i = 0; i < m; ++i) vec[i] = x[i] / nrm;
    if (jacobi_sign(A_in, ld, m, vec) < 0.0)
        for (int i = 0; i < m; ++i) vec[i] = -vec[i];
}

}  // namespace

// ---------------------------------------------------------------- HMat
HMat::~HMat() { release(); }

void HMat::release()
{
    if (rowptr || cols || vals || diag) {
        (void)hipSetDevice(device);
        (void)hipFree(rowptr);
        (void)hipFree(cols);
        (void)hipFree(vals);
        (void)hipFree(diag);
    }
    rowptr = nullptr;
    cols = nullptr;
    vals = nullptr;
    diag = nullptr;
    nrows = nnz = 0;
}

void hmat_build(asci_ctx *ctx, const double *h, const double *eri, int n, int na, int nb, const uint64_t *dets,
                int64_t ndets, double ecore, HMat &H, hipStream_t s)
{
    require(ndets >= 1 && ndets < ((int64_t)1 << 31), ASCI_EINVAL, "ndets must be in [1, 2^31)");
    validate_dets(ctx, dets, ndets, n, na, nb, s);
    H.release();
    H.device = ctx->device;
    const uint32_t nd = (uint32_t)ndets;
    // couplings are counted and placed by row and column share
    const uint32_t shares = pair_shares(nd);
    const size_t ncnt = (size_t)nd * shares;
    const uint32_t nchunks = (uint32_t)((ncnt + kChunk - 1) / kChunk);
    Arena &ar = ctx->main;
    ar.reset();
    ar.reserve((size_t)(2 * n * n + n) * 8 + ncnt * 12 + (size_t)nchunks * 8 + 4096);
    ar.reset();
    double *jk = ar.take<double>((size_t)2 * n * n + n);
    uint32_t *cnt = ar.take<uint32_t>(ncnt);
    int64_t *start = ar.take<int64_t>(ncnt);
    unsigned long long *csum = ar.take<unsigned long long>(nchunks);
    ASCI_HIP(hipMalloc((void **)&H.rowptr, ((size_t)nd + 1) * sizeof(int64_t)));
    ASCI_HIP(hipMalloc((void **)&H.diag, (size_t)nd * sizeof(double)));
    fault_clear(s);
    pair_prepare(h, eri, n, dets, nd, ecore, jk, H.diag, s);

    PairArgs g{};
    g.dets = dets;
    g.nd = nd;
    g.n = n;
    g.h = h;
    g.eri = eri;
    g.hdiag = H.diag;
    g.cnt = cnt;
    g.start = start;
    Profiler *prof = &ctx->prof;
    {
        ProfScope ps(prof, "hbuild_count", 0.0, s);
        launch_pairs<kPairCount>(g, s);
    }
    k_chunk_sums<<<nchunks, 256, 0, s>>>(cnt, ncnt, csum);
    ASCI_LAUNCH_CHECK();
    // chunk bases on the host (one value per 4096 counts)
    std::vector<unsigned long long> hb(nchunks);
    ASCI_HIP(hipMemcpyAsync(hb.data(), csum, nchunks * sizeof(unsigned long long), hipMemcpyDeviceToHost, s));
    ASCI_HIP(hipStreamSynchronize(s));
    unsigned long long tot = 0;
    for (uint32_t c = 0; c < nchunks; ++c) {
        const unsigned long long v = hb[c];
        hb[c] = tot;
        tot += v;
    }
    ASCI_HIP(hipMemcpyAsync(csum, hb.data(), nchunks * sizeof(unsigned long long), hipMemcpyHostToDevice, s));
    k_chunk_scan<<<nchunks, 256, 0, s>>>(cnt, ncnt, shares, csum, start, H.rowptr);
    ASCI_LAUNCH_CHECK();
    const int64_t nnz = (int64_t)tot;
    ASCI_HIP(hipMemcpyAsync(H.rowptr + nd, &nnz, sizeof(int64_t), hipMemcpyHostToDevice, s));
    ASCI_HIP(hipMalloc((void **)&H.cols, (size_t)std::max<int64_t>(nnz, 1) * sizeof(int32_t)));
    ASCI_HIP(hipMalloc((void **)&H.vals, (size_t)std::max<int64_t>(nnz, 1) * sizeof(double)));
    g.cols = H.cols;
    g.vals = H.vals;
    {
        ProfScope ps(prof, "hbuild_fill", 12.0 * (double)nnz, s);
        launch_pairs<kPairFill>(g, s);
    }
    HostStage &hst = ctx->stage;
    hst.reserve(256);
    fault_fetch((unsigned int *)((char *)hst.ptr + 64), s);
    ASCI_HIP(hipStreamSynchronize(s));
    fault_check(*(unsigned int *)((char *)hst.ptr + 64), "the Hamiltonian build");
    H.nrows = ndets;
    H.nnz = nnz;
}

void hmat_matvec(const HMat &H, const double *x, double *y, hipStream_t s, Profiler *prof)
{
    ProfScope ps(prof, "spmv", 12.0 * (double)H.nnz + 16.0 * (double)H.nrows, s);
    k_spmv<<<(unsigned)((H.nrows + 3) / 4), 256, 0, s>>>(H.rowptr, H.cols, H.vals, x, y, (uint32_t)H.nrows);
    ASCI_LAUNCH_CHECK();
}

// ---------------------------------------------------------------- Davidson (Alg. 5)
// The subspace V (orthonormal columns) and W = H V grow one vector per
// iteration; the projected matrix V^T W is solved on the host; the residual
// of the lowest Ritz pair is preconditioned by (D - theta)^-1, orthogonalised
// twice against V and appended.  A full subspace restarts from the Ritz vector.
//
// An iteration is queued as a whole and read back once: the sums that steer the
// vectors (overlaps, norms) are taken from their partials by the kernels that
// need them, and what decides on the host (the residual, independence, the new
// column of the projected matrix) comes back together.  At 5000 rows an
// iteration of about 30 launches and six read-backs took 154 us, now 55; at
// 120,000 rows 821 and 422.
//
// A converged iteration would append one vector in vain, so where convergence
// is near the residual is read back ahead of that: in the first iteration (the
// guess may be an eigenvector) and once the last residual was within kNear of
// the tolerance.  From a converged guess, without and with it, 5000 rows take
// 0.122 and 0.076 ms, 60,000 rows 0.405 and 0.222.  A read-back costs about 12
// us: too much for every iteration of a few thousand rows.
constexpr double kNear = 4.0;
DavidsonOut davidson(asci_ctx *ctx, const HMat &H, const double *guess, const DavidsonOpts &o, double *vec,
                     hipStream_t s)
{
    const size_t N = (size_t)H.nrows;
    const int mmax = std::max(2, std::min(o.max_subspace, kMaxSub));
    Arena &ar = ctx->main;
    ar.reset();
    ar.reserve((size_t)2 * mmax * N * 8 + 2 * N * 8 + (size_t)kDotBlocks * kPartLd * 2 * 8 + kPartLd * 8 + 64 * 256);
    ar.reset();
    double *V = ar.take<double>((size_t)mmax * N);
    double *W = ar.take<double>((size_t)mmax * N);
    double *u = ar.take<double>(N), *t = ar.take<double>(N);
    // partial sums: what is read back, and the two passes of the orthogonalisation
    double *part = ar.take<double>((size_t)kDotBlocks * kPartLd);
    double *hpart = ar.take<double>((size_t)kDotBlocks * kPartLd);
    double *dsmall = ar.take<double>(kPartLd);
    Profiler *prof = &ctx->prof;
    const unsigned nb = (unsigned)std::min<size_t>(kDotBlocks, std::max<size_t>(1, (N + 255) / 256));
    HostStage &hst = ctx->stage;
    hst.reserve(kPartLd * sizeof(double));
    double *h_down = (double *)hst.ptr;

    auto dots = [&](const double *M, int m, const double *x, double *out) {
        k_multidot<<<dim3(nb, (unsigned)((m + kDotCols - 1) / kDotCols)), 256, 0, s>>>(M, N, m, x, N, out);
        ASCI_LAUNCH_CHECK();
    };
    // sums of the first m columns of part, and the norms, in h_down
    auto read_sums = [&](int m) {
        k_rowsum<<<1, 64, 0, s>>>(part, m, (int)nb, dsmall);
        ASCI_LAUNCH_CHECK();
        ASCI_HIP(hipMemcpyAsync(h_down, dsmall, kPartLd * sizeof(double), hipMemcpyDeviceToHost, s));
        ASCI_HIP(hipStreamSynchronize(s));
    };
    // V[m] = t / |t| (|t|^2 in part), W[m] = H V[m], their overlaps with V[0..m] in part
    auto append = [&](int m) {
        k_normalise<<<nb, 256, 0, s>>>(t, N, part, V + (size_t)m * N);
        ASCI_LAUNCH_CHECK();
        hmat_matvec(H, V + (size_t)m * N, W + (size_t)m * N, s, prof);
        dots(V, m + 1, W + (size_t)m * N, part);
        read_sums(m + 1);
    };

    // start vector: the guess, else the unit vector of the lowest diagonal element
    if (guess) {
        ASCI_HIP(hipMemcpyAsync(t, guess, N * sizeof(double), hipMemcpyDeviceToDevice, s));
    } else {
        std::vector<double> d(N);
        ASCI_HIP(hipMemcpyAsync(d.data(), H.diag, N * sizeof(double), hipMemcpyDeviceToHost, s));
        ASCI_HIP(hipStreamSynchronize(s));
        size_t best = 0;
        for (size_t i = 1; i < N; ++i)
            if (d[i] < d[best]) best = i;
        std::vector<double> e(N, 0.0);
        e[best] = 1.0;
        ASCI_HIP(hipMemcpyAsync(t, e.data(), N * sizeof(double), hipMemcpyHostToDevice, s));
        ASCI_HIP(hipStreamSynchronize(s));
    }
    k_norm<<<nb, 256, 0, s>>>(t, N, part);
    ASCI_LAUNCH_CHECK();
    append(0);
    require(std::sqrt(h_down[kNormV]) > 0.0, ASCI_EINVAL, "Davidson guess vector is zero");
    int m = 1;
    std::vector<double> A((size_t)mmax * mmax, 0.0);
    A[0] = h_down[0];

    DavidsonOut out{0.0, 0.0, 0, false};
    SubCoef c;
    for (int it = 1; it <= o.max_iter; ++it) {
        double theta;
        small_lowest(A, mmax, m, theta, c.c);
        // a full subspace restarts from the Ritz vector (u, W u) alone
        const bool restart = m == mmax;
        k_ritz<<<nb, 256, 0, s>>>(V, W, N, m, c, theta, H.diag, N, u, t, restart ? 1 : 0, part);
        ASCI_LAUNCH_CHECK();
        out.energy = theta;
        out.iters = it;
        if (it == 1 || out.resid <= kNear * o.tol) {
            read_sums(0);
            out.resid = std::sqrt(h_down[kNormR]);
            if (out.resid <= o.tol) {
                out.converged = true;
                break;
            }
        }
        if (restart) {
            std::fill(A.begin(), A.end(), 0.0);
            A[0] = theta;
            m = 1;
        }
        // t orthogonalised against V[0..m) twice, normalised into V[m]
        for (int pass = 0; pass < 2; ++pass) {
            dots(V, m, t, hpart);
            k_orth<<<nb, 256, 0, s>>>(V, N, m, N, t, hpart, pass == 1 ? part : nullptr);
            ASCI_LAUNCH_CHECK();
        }
        append(m);
        out.resid = std::sqrt(h_down[kNormR]);
        if (out.resid <= o.tol) {
            out.converged = true;
            break;
        }
        // nothing independent is left
        if (!(std::sqrt(h_down[kNormV]) > 1e-12 * std::max(std::sqrt(h_down[kNormT]), 1e-300))) break;
        // new row and column of the projected matrix: V^T (H v_m)
        for (int i = 0; i <= m; ++i) {
            A[(size_t)i * mmax + m] = h_down[i];
            A[(size_t)m * mmax + i] = h_down[i];
        }
        ++m;
    }
    // the Ritz vector of the last projected solve
    ASCI_HIP(hipMemcpyAsync(vec, u, N * sizeof(double), hipMemcpyDeviceToDevice, s));
    ASCI_HIP(hipStreamSynchronize(s));
    return out;
}

}  // namespace asci
