// The double loop over the determinant pairs of a set (Sec. II.C): couplings
// counted, written as CSR rows, or summed into the energy.  A wavefront holds
// a few rows and tests 64 column determinants of a tile in LDS at a time
// (exclusive or and popcount); the pairs that pass, a few in a thousand, go to
// a queue of the wavefront and are evaluated 64 at a time, so that every lane
// has an element to form.  Evaluated where they were found, a test's few hits
// left most lanes idle for the length of an element.  20,000 determinants of
// (16e,20o) took 0.26 ms to test (count) and 2.86 ms to fill, now 0.12 and 0.33
// ms; the energy of 10,000 took 21.3 ms on 40 workgroups of one row a thread,
// now 0.077 ms.  Bound by the latency of the elements' scattered reads.
// Singles, whose elements are sums over the occupied orbitals, have a queue of
// their own.
#pragma once

#include "hamiltonian.h"

#include <algorithm>

namespace asci {

namespace {

constexpr int kPairBlock = 256;    // 4 wavefronts
constexpr int kPairTile = 1024;    // column determinants staged in LDS per tile
constexpr int kPairQueue = 128;    // entries of one queue: fewer than 64 left over, and one test's 64
enum PairMode { kPairCount, kPairFill, kPairEnergy };

struct PairArgs {
    const uint64_t *dets;
    uint32_t nd;
    int n;
    const double *h, *eri;
    const double *hdiag;     // H_ii (k_pair_diag)
    uint32_t tiles, shares;  // column tiles of one share; shares (blockIdx.y)
    uint32_t *cnt;           // count: couplings per row and share
    const int64_t *start;    // fill: their first place
    int32_t *cols;
    double *vals;
    const double *c;         // energy: coefficients
    double *partial;         // energy: one sum per wavefront
};

// <a|H|i> for two different determinants a = (aa, ab) and i = (ia, ib), a single
// or a double apart: the excitation is read from i to a
__device__ __forceinline__ double pair_element(const PairArgs &g, uint64_t aa, uint64_t ab, uint64_t ia, uint64_t ib)
{
    const int n = g.n;
    const int ea = popc64(aa ^ ia) >> 1, eb = popc64(ab ^ ib) >> 1;
    if (ea == 1 && eb == 0) return single_value(g.h, g.eri, n, ia, ib, lowbit(ia & ~aa), lowbit(aa & ~ia));
    if (ea == 0 && eb == 1) return single_value(g.h, g.eri, n, ib, ia, lowbit(ib & ~ab), lowbit(ab & ~ib));
    if (ea == 1 && eb == 1)
        return double_opp_value(g.eri, n, ia, ib, lowbit(ia & ~aa), lowbit(aa & ~ia), lowbit(ib & ~ab),
                                lowbit(ab & ~ib));
    if (ea == 2) return double_same_value(g.eri, n, ia, ia & ~aa, aa & ~ia);
    return double_same_value(g.eri, n, ib, ib & ~ab, ab & ~ib);
}

// a wavefront's queued pairs
struct PairQueue {
    uint32_t col[kPairQueue];
    uint32_t pos[kPairQueue];  // fill: place in its row and share
    uint8_t row[kPairQueue];
};

// M: the word a spin string is tested in (32 bits where every orbital fits);
// kPairRows: rows per wavefront
template <int MODE, typename M, int kPairRows>
__global__ __launch_bounds__(kPairBlock) void k_pairs(PairArgs g)
{
    __shared__ M ta[kPairTile], tb[kPairTile];
    __shared__ PairQueue queues[MODE == kPairCount ? 1 : 2 * (kPairBlock / 64)];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint64_t lt = (1ull << lane) - 1ull;
    const uint32_t row0 = (blockIdx.x * (kPairBlock / 64) + (uint32_t)wv) * kPairRows;
    PairQueue *q0 = &queues[MODE == kPairCount ? 0 : 2 * wv], *q1 = &queues[MODE == kPairCount ? 0 : 2 * wv + 1];
    uint32_t n0 = 0, n1 = 0;  // entries: doubles and equal determinants, singles
    M ra[kPairRows], rb[kPairRows];
    uint32_t run[kPairRows];
#pragma unroll
    for (int t = 0; t < kPairRows; ++t) {
        const bool ok = row0 + t < g.nd;
        ra[t] = ok ? (M)g.dets[2 * (size_t)(row0 + t)] : (M)0;
        rb[t] = ok ? (M)g.dets[2 * (size_t)(row0 + t) + 1] : (M)0;
        run[t] = 0u;
    }
    double acc = 0.0;
    // evaluates the first m entries of a queue and moves the rest to its front
    auto flush = [&](PairQueue *q, uint32_t &count, uint32_t m) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if ((uint32_t)lane < m) {
            const uint32_t j = q->col[lane], i = row0 + q->row[lane];
            const uint64_t ia = g.dets[2 * (size_t)i], ib = g.dets[2 * (size_t)i + 1];
            const uint64_t ja = g.dets[2 * (size_t)j], jb = g.dets[2 * (size_t)j + 1];
            // a determinant that the set holds twice couples to its copy by H_ii
            const double v = ia == ja && ib == jb ? g.hdiag[i] : pair_element(g, ia, ib, ja, jb);
            if (MODE == kPairFill) {
                const int64_t at = g.start[(size_t)i * g.shares + blockIdx.y] + (int64_t)q->pos[lane];
                g.cols[at] = (int32_t)j;
                g.vals[at] = v;
            } else {
                // both triangles; a row with itself once
                acc = acc + (i == j ? 1.0 : 2.0) * (g.c[i] * v * g.c[j]);
            }
        }
        const uint32_t left = count - m;  // below 64
        const uint32_t c = q->col[m + min((uint32_t)lane, 63u)], p = MODE == kPairFill ? q->pos[m + (uint32_t)lane] : 0u;
        const uint8_t r = q->row[m + (uint32_t)lane];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if ((uint32_t)lane < left) {
            q->col[lane] = c;
            if (MODE == kPairFill) q->pos[lane] = p;
            q->row[lane] = r;
        }
        count = left;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    const uint32_t all = (g.nd + kPairTile - 1) / kPairTile;
    const uint32_t t0 = blockIdx.y * g.tiles, t1 = min(all, t0 + g.tiles);
    for (uint32_t tile = t0; tile < t1; ++tile) {
        const uint32_t j0 = tile * kPairTile, tn = min((uint32_t)kPairTile, g.nd - j0);
        // the energy takes each pair once: tiles left of every row of the workgroup are done
        if (MODE == kPairEnergy && j0 + tn <= blockIdx.x * (kPairBlock / 64) * kPairRows) continue;
        __syncthreads();
        for (uint32_t k = threadIdx.x; k < tn; k += kPairBlock) {
            ta[k] = (M)g.dets[2 * (size_t)(j0 + k)];
            tb[k] = (M)g.dets[2 * (size_t)(j0 + k) + 1];
        }
        __syncthreads();
        for (uint32_t c = 0; c < tn; c += 64) {
            const uint32_t jl = c + (uint32_t)lane, j = j0 + jl;
            const bool in = jl < tn;
            const M ca = in ? ta[jl] : (M)0, cb = in ? tb[jl] : (M)0;
#pragma unroll
            for (int t = 0; t < kPairRows; ++t) {
                if (row0 + t >= g.nd) break;  // the same for the whole wavefront
                const int d = __popcll((uint64_t)(M)(ra[t] ^ ca)) + __popcll((uint64_t)(M)(rb[t] ^ cb));
                bool hit = in && d <= 4;
                if (MODE == kPairEnergy) hit = hit && j >= row0 + t;
                const uint64_t m = __ballot(hit);
                if (MODE == kPairCount) {
                    run[t] += (uint32_t)__popcll(m);
                    continue;
                }
                if (m == 0ull) continue;
                const uint64_t single = __ballot(hit && d == 2), other = m & ~single;
                if (hit) {
                    const bool s = (single >> lane) & 1ull;
                    PairQueue *q = s ? q1 : q0;
                    const uint32_t at = s ? n1 + (uint32_t)__popcll(single & lt) : n0 + (uint32_t)__popcll(other & lt);
                    q->col[at] = j;
                    q->row[at] = (uint8_t)t;
                    if (MODE == kPairFill) q->pos[at] = run[t] + (uint32_t)__popcll(m & lt);
                }
                run[t] += (uint32_t)__popcll(m);
                n0 += (uint32_t)__popcll(other);
                n1 += (uint32_t)__popcll(single);
                if (n0 >= 64u) flush(q0, n0, 64u);
                if (n1 >= 64u) flush(q1, n1, 64u);
            }
        }
    }
    if (MODE == kPairCount) {
        if (lane == 0) {
#pragma unroll
            for (int t = 0; t < kPairRows; ++t)
                if (row0 + t < g.nd) g.cnt[(size_t)(row0 + t) * g.shares + blockIdx.y] = run[t];
        }
        return;
    }
    if (n0) flush(q0, n0, n0);
    if (n1) flush(q1, n1, n1);
    if (MODE == kPairEnergy) {
        for (int d = 32; d >= 1; d >>= 1) acc = acc + __shfl_xor(acc, d, 64);
        if (lane == 0) g.partial[((size_t)blockIdx.y * gridDim.x + blockIdx.x) * (kPairBlock / 64) + wv] = acc;
    }
}

// Rows per wavefront: eight share each column read, but a set of less than
// 131,072 determinants then has fewer than 16 wavefronts a CU to hide the
// elements' reads behind (H of 20,000 filled in 1.35 ms with eight rows, 0.51
// ms with two).
inline int pair_rows(uint32_t nd) { return nd >= 131072u ? 8 : (nd >= 65536u ? 4 : 2); }
inline unsigned pair_blocks(uint32_t nd)
{
    const uint32_t rows = (uint32_t)(kPairBlock / 64 * pair_rows(nd));
    return (nd + rows - 1) / rows;
}

// Column shares of a row: the reference and the singles couple to most of a set,
// so that the wavefront with their rows would run long after the others
// (energy of 10,000 determinants 0.28 ms in one share, 0.077 ms in ten).
inline uint32_t pair_shares(uint32_t nd)
{
    return std::max(1u, std::min((nd + kPairTile - 1) / kPairTile, 16384u / pair_blocks(nd)));
}

template <int MODE, typename M>
inline void launch_pairs_m(PairArgs g, hipStream_t s)
{
    g.shares = pair_shares(g.nd);
    g.tiles = ((g.nd + kPairTile - 1) / kPairTile + g.shares - 1) / g.shares;
    const dim3 grid(pair_blocks(g.nd), g.shares);
    switch (pair_rows(g.nd)) {
    case 8: k_pairs<MODE, M, 8><<<grid, kPairBlock, 0, s>>>(g); break;
    case 4: k_pairs<MODE, M, 4><<<grid, kPairBlock, 0, s>>>(g); break;
    default: k_pairs<MODE, M, 2><<<grid, kPairBlock, 0, s>>>(g); break;
    }
    ASCI_LAUNCH_CHECK();
}
template <int MODE>
inline void launch_pairs(const PairArgs &g, hipStream_t s)
{
    if (g.n <= 32) launch_pairs_m<MODE, uint32_t>(g, s);
    else launch_pairs_m<MODE, uint64_t>(g, s);
}

// J_pq = (pp|qq), X_pq = (pp|qq) - (pq|qp), h_pp: the tables of H_aa
__global__ __launch_bounds__(kPairBlock) void k_pair_table(const double *__restrict__ eri, const double *__restrict__ h,
                                                           int n, double *__restrict__ jk)
{
    const int t = blockIdx.x * kPairBlock + threadIdx.x;
    if (t >= n * n) return;
    const int p = t / n, q = t % n;
    jk[t] = eri4(eri, n, p, p, q, q);
    jk[n * n + t] = eri4(eri, n, p, p, q, q) - eri4(eri, n, p, q, q, p);
    if (q == 0) jk[2 * n * n + p] = h[(size_t)p * n + p];
}

// H_ii of every determinant, the tables in LDS.  A diagonal element is a sum
// over all its orbital pairs, read one after the other: in the pair sweep it
// would hold the 63 other lanes of its queue's turn for that long.
__global__ __launch_bounds__(64) void k_pair_diag(const uint64_t *__restrict__ dets, uint32_t nd,
                                                  const double *__restrict__ jk, int n, double ecore,
                                                  double *__restrict__ out)
{
    extern __shared__ __align__(16) unsigned char pair_smem[];
    double *tab = reinterpret_cast<double *>(pair_smem);
    for (int t = threadIdx.x; t < 2 * n * n + n; t += 64) tab[t] = jk[t];
    __syncthreads();
    const uint32_t i = blockIdx.x * 64 + threadIdx.x;
    if (i < nd)
        out[i] = diag_value(tab, tab + n * n, tab + 2 * n * n, n, ecore, dets[2 * (size_t)i], dets[2 * (size_t)i + 1]);
}

// the tables (2 n^2 + n doubles at jk) and H_ii
inline void pair_prepare(const double *h, const double *eri, int n, const uint64_t *dets, uint32_t nd, double ecore,
                         double *jk, double *hdiag, hipStream_t s)
{
    k_pair_table<<<(unsigned)((n * n + kPairBlock - 1) / kPairBlock), kPairBlock, 0, s>>>(eri, h, n, jk);
    ASCI_LAUNCH_CHECK();
    const size_t lds = (size_t)(2 * n * n + n) * 8;
    ASCI_HIP(hipFuncSetAttribute((const void *)k_pair_diag, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    k_pair_diag<<<(nd + 63) / 64, 64, lds, s>>>(dets, nd, jk, n, ecore, hdiag);
    ASCI_LAUNCH_CHECK();
}

}  // namespace

}  // namespace asci
