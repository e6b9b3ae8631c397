// Variational energy E = sum_ij C_i H_ij C_j over a determinant set: the E_k
// of Eq. (1), by the double loop over determinant pairs that the paper uses to
// build H (Sec. II.C).  Each pair is formed once (H is symmetric) and counted
// twice; the wavefronts' sums are added in a fixed order.
#include "pairs.h"

namespace asci {

namespace {

// deterministic sum of the partial sums: one block, fixed order
__global__ __launch_bounds__(1024) void k_sum(const double *__restrict__ x, uint32_t n, double *__restrict__ out)
{
    __shared__ double s[1024];
    double acc = 0.0;
    for (uint32_t i = threadIdx.x; i < n; i += 1024) acc = acc + x[i];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 512; w >= 1; w >>= 1) {
        if (threadIdx.x < (unsigned)w) s[threadIdx.x] = s[threadIdx.x] + s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s[0];
}

}  // namespace

double energy_device(asci_ctx *ctx, const double *h, const double *eri, int n, const uint64_t *dets,
                     const double *coeffs, int64_t ndets, double ecore, hipStream_t s)
{
    require(ndets >= 1 && ndets < (1ll << 31), ASCI_EINVAL, "ndets out of range");
    const uint32_t nd = (uint32_t)ndets;
    Arena &ar = ctx->main;
    const size_t parts = (size_t)pair_blocks(nd) * pair_shares(nd) * (kPairBlock / 64);
    ar.reset();
    ar.reserve(parts * 8 + (size_t)nd * 8 + ((size_t)2 * n * n + n) * 8 + 4096);
    ar.reset();
    double *partial = ar.take<double>(parts);
    double *jk = ar.take<double>((size_t)2 * n * n + n);
    double *hdiag = ar.take<double>(nd);
    double *out = ar.take<double>(1);
    fault_clear(s);
    pair_prepare(h, eri, n, dets, nd, ecore, jk, hdiag, s);
    PairArgs g{};
    g.dets = dets;
    g.nd = nd;
    g.n = n;
    g.h = h;
    g.eri = eri;
    g.hdiag = hdiag;
    g.c = coeffs;
    g.partial = partial;
    launch_pairs<kPairEnergy>(g, s);
    k_sum<<<1, 1024, 0, s>>>(partial, (uint32_t)parts, out);
    ASCI_LAUNCH_CHECK();
    HostStage &hs = ctx->stage;
    hs.reserve(256);
    ASCI_HIP(hipMemcpyAsync(hs.ptr, out, sizeof(double), hipMemcpyDeviceToHost, s));
    fault_fetch((unsigned int *)((char *)hs.ptr + 64), s);
    ASCI_HIP(hipStreamSynchronize(s));
    fault_check(*(unsigned int *)((char *)hs.ptr + 64), "the energy double loop");
    return *(double *)hs.ptr;
}

}  // namespace asci
