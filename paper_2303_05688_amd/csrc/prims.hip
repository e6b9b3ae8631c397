// Device primitives for the search: exclusive scan, stable merge and radix
// sorts, and radix selection.  Written for 64-wide wavefronts (gfx950): ranking inside a
// wave uses ballots, blocks are 256 threads (4 waves).
#include <algorithm>
#include "asci_internal.h"

namespace asci {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kItems = 16;
constexpr int kTile = kThreads * kItems;  // 4096
static_assert(kTile == kScanTile, "scan tile");

// a host bound on a count, tightened by the count on the device when given
__device__ __forceinline__ size_t dev_n(size_t n, const uint32_t *dn) { return dn ? min(n, (size_t)*dn) : n; }

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// exclusive scan across a block of NW waves; every thread must call it
template <int NW>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *s_tmp, uint32_t &total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = wave_incl_scan(v);
    if (lane == 63) s_tmp[w] = x;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        uint32_t t = s_tmp[i];
        base += (i < w) ? t : 0u;
        tot += t;
    }
    total = tot;
    __syncthreads();
    return base + x - v;
}

// ---------------------------------------------------------------- scan
__global__ __launch_bounds__(kThreads) void k_scan_reduce(const uint32_t *__restrict__ in, size_t n,
                                                          uint32_t *__restrict__ partial, const uint32_t *dn)
{
    __shared__ uint32_t s_tmp[kWaves];
    n = dev_n(n, dn);
    const size_t base = (size_t)blockIdx.x * kTile;
    uint32_t s = 0;
    if (base + kTile <= n && (reinterpret_cast<uintptr_t>(in) & 15u) == 0) {
        // a whole tile: 16-byte loads, coalesced across the block
        const uint4 *p = reinterpret_cast<const uint4 *>(in + base);
#pragma unroll
        for (int i = 0; i < kTile / 4 / kThreads; ++i) {
            const uint4 q = p[i * kThreads + threadIdx.x];
            s += (q.x + q.y) + (q.z + q.w);
        }
    } else {
        for (int i = threadIdx.x; i < kTile; i += kThreads) {
            size_t j = base + i;
            if (j < n) s += in[j];
        }
    }
    uint32_t tot;
    block_excl_scan<kWaves>(s, s_tmp, tot);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void k_scan_partials(uint32_t *__restrict__ partial, uint32_t np,
                                                        uint32_t *__restrict__ d_total)
{
    __shared__ uint32_t s_tmp[16];
    uint32_t carry = 0;
    for (uint32_t c0 = 0; c0 < np; c0 += 1024) {
        uint32_t j = c0 + threadIdx.x;
        uint32_t v = j < np ? partial[j] : 0u;
        uint32_t tot;
        uint32_t e = block_excl_scan<16>(v, s_tmp, tot);
        if (j < np) partial[j] = carry + e;
        carry += tot;
    }
    if (threadIdx.x == 0 && d_total) *d_total = carry;
}

// short inputs (at most kScanSmall elements): one workgroup, one launch,
// chunks of 16384 scanned in turn with a running carry, 16-byte loads (33,000
// elements took 20 us in chunks of 4096 of single words: each chunk waits for
// its loads)
constexpr size_t kScanSmall = 65536;
__global__ __launch_bounds__(1024) void k_scan_small(const uint32_t *in, uint32_t *out, uint32_t n,
                                                     uint32_t *__restrict__ d_total, const uint32_t *dn)
{
    __shared__ uint32_t s_tmp[16];
    n = (uint32_t)dev_n(n, dn);
    const bool aligned = ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15u) == 0;
    uint32_t carry = 0;
    for (uint32_t c0 = 0; c0 < n; c0 += 1024u * kItems) {
        const uint32_t j0 = c0 + threadIdx.x * (uint32_t)kItems;
        const bool full = aligned && j0 + kItems <= n;
        uint32_t v[kItems], sum = 0;
        if (full) {
#pragma unroll
            for (int i = 0; i < kItems / 4; ++i) {
                const uint4 q = reinterpret_cast<const uint4 *>(in + j0)[i];
                v[4 * i] = q.x;
                v[4 * i + 1] = q.y;
                v[4 * i + 2] = q.z;
                v[4 * i + 3] = q.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < kItems; ++i) v[i] = j0 + i < n ? in[j0 + i] : 0u;
        }
#pragma unroll
        for (int i = 0; i < kItems; ++i) sum += v[i];
        uint32_t tot;
        uint32_t e = carry + block_excl_scan<16>(sum, s_tmp, tot);
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            const uint32_t x = v[i];
            v[i] = e;
            e += x;
        }
        if (full) {
#pragma unroll
            for (int i = 0; i < kItems / 4; ++i)
                reinterpret_cast<uint4 *>(out + j0)[i] = make_uint4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
        } else {
#pragma unroll
            for (int i = 0; i < kItems; ++i)
                if (j0 + i < n) out[j0 + i] = v[i];
        }
        carry += tot;
    }
    if (threadIdx.x == 0 && d_total) *d_total = carry;
}

__global__ __launch_bounds__(kThreads) void k_scan_down(const uint32_t *in, uint32_t *out, size_t n,
                                                        const uint32_t *__restrict__ partial, const uint32_t *dn)
{
    __shared__ uint32_t s_tmp[kWaves];
    n = dev_n(n, dn);
    const size_t base = (size_t)blockIdx.x * kTile + (size_t)threadIdx.x * kItems;
    // a whole tile with aligned ends moves each thread's 16 items as four
    // 16-byte words (the scan may run in place: every word is read before the
    // block's barrier and written after it)
    const bool full = (size_t)blockIdx.x * kTile + kTile <= n &&
                      ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15u) == 0;
    uint32_t v[kItems];
    uint32_t s = 0;
    if (full) {
        const uint4 *p = reinterpret_cast<const uint4 *>(in + base);
#pragma unroll
        for (int i = 0; i < kItems / 4; ++i) {
            const uint4 q = p[i];
            v[4 * i] = q.x;
            v[4 * i + 1] = q.y;
            v[4 * i + 2] = q.z;
            v[4 * i + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            size_t j = base + i;
            v[i] = j < n ? in[j] : 0u;
        }
    }
#pragma unroll
    for (int i = 0; i < kItems; ++i) s += v[i];
    uint32_t tot;
    uint32_t e = block_excl_scan<kWaves>(s, s_tmp, tot) + partial[blockIdx.x];
    if (full) {
        uint4 *p = reinterpret_cast<uint4 *>(out + base);
#pragma unroll
        for (int i = 0; i < kItems / 4; ++i) {
            uint4 q;
            q.x = e;
            e += v[4 * i];
            q.y = e;
            e += v[4 * i + 1];
            q.z = e;
            e += v[4 * i + 2];
            q.w = e;
            e += v[4 * i + 3];
            p[i] = q;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            size_t j = base + i;
            if (j < n) out[j] = e;
            e += v[i];
        }
    }
}

// ---------------------------------------------------------------- merge sort
// Keys of KW words, the first the most significant, ties by position (a stable
// sort), a 32-bit payload: chunks sorted in LDS by a bitonic network, then eight
// runs at a time merged, every element finding its place by a binary search in
// the seven other runs.  One launch for the chunks, one more for each factor of
// eight, where a radix sort of 8-bit digits takes three launches a digit (the
// 2000 scores of a small search took 24 launches, about 110 us).  73,000 scores
// of a bound of 3e5 (8e12o): three merges of 11.7 us, four at a time five of 9.0;
// with the reads of each search behind its own branch 16 at a time took 22.
constexpr int kSortT = 512;
constexpr uint32_t kSortWays = 8;
constexpr int kSortChunk = 1024;  // one pair a thread and stage: 17 us (a chunk of 4096 took 47)

template <int KW>
struct SortKeys {
    uint64_t *w[KW];
};

template <int KW>
__device__ __forceinline__ bool words_less(const uint64_t (&a)[KW], const uint64_t (&b)[KW])
{
#pragma unroll
    for (int k = 0; k + 1 < KW; ++k)
        if (a[k] != b[k]) return a[k] < b[k];
    return a[KW - 1] < b[KW - 1];
}

// orders a wavefront's LDS accesses (see the stages that need no barrier)
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The payload is the position.  score: the key (of one word) is
// ~|score|, so that ascending keys are descending |score|
template <int KW>
__global__ __launch_bounds__(kSortT) void k_sort_chunks(SortKeys<KW> in, const double *__restrict__ score,
                                                        SortKeys<KW> out, uint32_t *__restrict__ oval, size_t n,
                                                        const uint32_t *dn)
{
    constexpr int CH = kSortChunk;
    __shared__ uint64_t x[KW][CH];
    __shared__ uint16_t ix[CH];
    n = dev_n(n, dn);
    const size_t base = (size_t)blockIdx.x * CH;
    if (base >= n) return;  // uniform
    const uint32_t m = (uint32_t)min(n - base, (size_t)CH);
    uint32_t p = 2;
    while (p < m) p <<= 1;
    for (uint32_t i = threadIdx.x; i < p; i += kSortT) {
#pragma unroll
        for (int k = 0; k < KW; ++k)
            x[k][i] = i < m ? (score ? ~abs_order(score[base + i]) : in.w[k][base + i]) : ~0ull;
        ix[i] = (uint16_t)i;  // a pad's position is above every record's
    }
    __syncthreads();
    // pair t of a stage is (i, i + jj); up to jj = 64 a wavefront's pairs lie in
    // its own 128 elements, so those stages need no barrier between them
    for (uint32_t k2 = 2; k2 <= p; k2 <<= 1) {
        for (uint32_t jj = k2 >> 1; jj > 0; jj >>= 1) {
            for (uint32_t t = threadIdx.x; t < p / 2; t += kSortT) {
                const uint32_t i = 2u * (t & ~(jj - 1u)) + (t & (jj - 1u)), o = i + jj;
                uint64_t a[KW], b[KW];
#pragma unroll
                for (int k = 0; k < KW; ++k) {
                    a[k] = x[k][i];
                    b[k] = x[k][o];
                }
                const uint16_t ia = ix[i], ib = ix[o];
                const bool gt = words_less<KW>(b, a) || (!words_less<KW>(a, b) && ib < ia);
                if (gt == ((i & k2) == 0u)) {
#pragma unroll
                    for (int k = 0; k < KW; ++k) {
                        x[k][i] = b[k];
                        x[k][o] = a[k];
                    }
                    ix[i] = ib;
                    ix[o] = ia;
                }
            }
            if (jj > 64u || (jj == 1u && k2 >= 128u)) __syncthreads();
            else wave_order();
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < m; i += kSortT) {
#pragma unroll
        for (int k = 0; k < KW; ++k) out.w[k][base + i] = x[k][i];
        oval[base + i] = (uint32_t)(base + ix[i]);
    }
}

// merges the runs of `width` elements kSortWays at a time
template <int KW>
__global__ __launch_bounds__(kThreads) void k_sort_merge(SortKeys<KW> in, const uint32_t *__restrict__ ival,
                                                         SortKeys<KW> out, uint32_t *__restrict__ oval, size_t n,
                                                         size_t width, const uint32_t *dn)
{
    n = dev_n(n, dn);
    const size_t g = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (g >= n) return;
    const size_t base = g / (kSortWays * width) * (kSortWays * width), off = g - base;
    const uint32_t run = (uint32_t)(off / width);
    uint64_t key[KW];
#pragma unroll
    for (int k = 0; k < KW; ++k) key[k] = in.w[k][g];
    // elements of the other runs that come first: smaller ones, and in the runs
    // before this element's equal ones too; all searches take a step together,
    // their reads ahead of the first comparison, so that a step waits once
    uint32_t l[kSortWays], r[kSortWays];
    const uint32_t n32 = (uint32_t)n, b32 = (uint32_t)base, w32 = (uint32_t)width;
    uint32_t d = b32 + ((uint32_t)off - run * w32);
#pragma unroll
    for (uint32_t o = 0; o < kSortWays; ++o) {
        l[o] = (uint32_t)min(base + o * width, n);
        r[o] = o == run ? l[o] : (uint32_t)min(base + (o + 1) * width, n);
        d -= l[o];
    }
    for (size_t w = width; w; w >>= 1) {  // uniform: a run of w elements takes bits(w) steps
        uint64_t y[kSortWays][KW];
#pragma unroll
        for (uint32_t o = 0; o < kSortWays; ++o) {
            const uint32_t m = min(l[o] + (r[o] - l[o]) / 2u, n32 - 1u);
#pragma unroll
            for (int k = 0; k < KW; ++k) y[o][k] = in.w[k][m];
        }
#pragma unroll
        for (uint32_t o = 0; o < kSortWays; ++o) {
            const uint32_t m = l[o] + (r[o] - l[o]) / 2u;
            const bool open = l[o] < r[o];
            const bool before = o < run ? !words_less<KW>(key, y[o]) : words_less<KW>(y[o], key);
            l[o] = open && before ? m + 1u : l[o];
            r[o] = open && !before ? m : r[o];
        }
    }
#pragma unroll
    for (uint32_t o = 0; o < kSortWays; ++o) d += l[o];
#pragma unroll
    for (int k = 0; k < KW; ++k) out.w[k][d] = key[k];
    oval[d] = ival[g];
}

// ---------------------------------------------------------------- radix sort
// Long inputs: stable LSD passes of 8 bits, tiles of kTile records.  A merge of
// eight runs reads each of them at log2(width) scattered places for every
// element, and its runs outgrow the cache; a digit pass streams.  The sort of
// the k best of 1.3e8 pairs (16e20o), ms, merged and by digits: k = 3e5 0.09 and
// 0.25, 1e6 0.30 and 0.35, 3e6 0.80 and 0.47, 2e7 7.3 and 2.4.
constexpr size_t kRadixFrom = (size_t)3 << 19;

__global__ __launch_bounds__(kThreads) void k_rs_keys(const double *__restrict__ score, uint64_t *__restrict__ key,
                                                      uint32_t *__restrict__ val, size_t n, const uint32_t *dn)
{
    n = dev_n(n, dn);
    const size_t j = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (j >= n) return;
    if (score) key[j] = ~abs_order(score[j]);
    val[j] = (uint32_t)j;
}

// counts of every digit per tile; a tile past a count on the device writes zeros
__global__ __launch_bounds__(kThreads) void k_rs_hist(const uint64_t *__restrict__ key, size_t n, int shift,
                                                      uint32_t *__restrict__ hist, uint32_t nblocks, const uint32_t *dn)
{
    __shared__ uint32_t h[kWaves][256];
    n = dev_n(n, dn);
    const int tid = threadIdx.x, w = tid >> 6;
    for (int i = tid; i < kWaves * 256; i += kThreads) (&h[0][0])[i] = 0u;
    __syncthreads();
    const size_t base = (size_t)blockIdx.x * kTile;
    for (int i = tid; i < kTile; i += kThreads)
        if (base + i < n) atomicAdd(&h[w][(uint32_t)(key[base + i] >> shift) & 0xFFu], 1u);
    __syncthreads();
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) c += h[i][tid];
    hist[(size_t)tid * nblocks + blockIdx.x] = c;
}

// Stable scatter of one tile.  Tile order is (wave, row, lane), which is the
// input order, so equal digits keep their input order.
__global__ __launch_bounds__(kThreads) void k_rs_scatter(const uint64_t *__restrict__ ikey,
                                                         const uint32_t *__restrict__ ival, uint64_t *__restrict__ okey,
                                                         uint32_t *__restrict__ oval, size_t n, int shift,
                                                         const uint32_t *__restrict__ hist, uint32_t nblocks,
                                                         const uint32_t *dn)
{
    __shared__ uint64_t s_key[kTile];
    __shared__ uint32_t s_val[kTile];
    __shared__ uint32_t s_wcnt[kWaves][256];
    __shared__ uint32_t s_dbase[256], s_gbase[256], s_tmp[kWaves];
    n = dev_n(n, dn);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const size_t tile0 = (size_t)blockIdx.x * kTile;
    if (tile0 >= n) return;  // uniform
    for (int i = tid; i < kWaves * 256; i += kThreads) (&s_wcnt[0][0])[i] = 0u;
    __syncthreads();
    uint64_t rk[kItems];
    uint32_t rv[kItems], rrank[kItems];
    const uint64_t lt = (1ull << lane) - 1ull;
    const size_t wbase = tile0 + (size_t)w * 64 * kItems;
#pragma unroll
    for (int s = 0; s < kItems; ++s) {
        const size_t j = wbase + (size_t)s * 64 + lane;
        const bool valid = j < n;
        rk[s] = valid ? ikey[j] : 0ull;
        rv[s] = valid ? ival[j] : 0u;
        const uint32_t d = (uint32_t)(rk[s] >> shift) & 0xFFu;
        const uint64_t peers = wave_match(d, valid, 8);
        const uint32_t before = s_wcnt[w][d];
        rrank[s] = before + (uint32_t)__popcll(peers & lt);
        wave_order();
        if (valid && (peers & lt) == 0ull) s_wcnt[w][d] = before + (uint32_t)__popcll(peers);
        wave_order();
    }
    __syncthreads();
    {
        uint32_t run = 0;
#pragma unroll
        for (int i = 0; i < kWaves; ++i) {
            const uint32_t c = s_wcnt[i][tid];
            s_wcnt[i][tid] = run;
            run += c;
        }
        uint32_t tot;
        s_dbase[tid] = block_excl_scan<kWaves>(run, s_tmp, tot);
        s_gbase[tid] = hist[(size_t)tid * nblocks + blockIdx.x];
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kItems; ++s) {
        if (wbase + (size_t)s * 64 + lane < n) {
            const uint32_t d = (uint32_t)(rk[s] >> shift) & 0xFFu;
            const uint32_t at = min(s_dbase[d] + s_wcnt[w][d] + rrank[s], (uint32_t)kTile - 1u);
            s_key[at] = rk[s];
            s_val[at] = rv[s];
        }
    }
    __syncthreads();
    const uint32_t tn = (uint32_t)min(n - tile0, (size_t)kTile);
    for (uint32_t i = tid; i < tn; i += kThreads) {
        const uint64_t k = s_key[i];
        const uint32_t d = (uint32_t)(k >> shift) & 0xFFu;
        const size_t g = (size_t)s_gbase[d] + (i - s_dbase[d]);
        if (g < n) {
            okey[g] = k;
            oval[g] = s_val[i];
        }
    }
}

// ---------------------------------------------------------------- radix select
constexpr int kSelBins = 2048;
static_assert(sizeof(SelectState::hist) == kSelBins * sizeof(uint32_t), "one counter a bin");

__global__ __launch_bounds__(1024) void k_sel_init(SelectState *st, uint64_t k, const uint32_t *dk,
                                                   unsigned int *count)
{
    if (threadIdx.x == 0) {
        st->prefix = 0ull;
        st->mask = 0ull;
        st->krem = dk ? min(k, (uint64_t)*dk) : k;
        st->done = 0u;
        if (count) *count = 0u;
    }
    for (int i = threadIdx.x; i < kSelBins; i += 1024) st->hist[i] = 0u;
}

// takes a digit from the counters of a pass (the largest whose entries, with
// those above it, reach krem) and clears them for the next one
__device__ __forceinline__ void sel_pick(SelectState *st, int shift, int bits, uint64_t prefix, uint64_t mask,
                                         uint32_t *s_tmp)
{
    // thread t holds bins kSelBins - 1 - 8t downwards: a scan over the threads
    // counts the entries above every bin
    constexpr int PER = kSelBins / kThreads;
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        c[k] = __hip_atomic_load(&st->hist[kSelBins - 1 - PER * (int)threadIdx.x - k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sum += c[k];
    }
    uint32_t tot;
    uint64_t above = block_excl_scan<kWaves>(sum, s_tmp, tot);
    const uint64_t need = st->krem;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int d = kSelBins - 1 - PER * (int)threadIdx.x - k;
        // one thread holds the digit: above < need <= above + its count (need
        // is at most the number of entries)
        if (above < need && above + c[k] >= need) {
            st->krem = need - above;
            st->prefix = prefix | ((uint64_t)d << shift);
            st->mask = mask | (((1ull << bits) - 1ull) << shift);
        }
        above += c[k];
        st->hist[d] = 0u;
    }
    if (threadIdx.x == 0) st->done = 0u;
}

__global__ __launch_bounds__(kThreads) void k_sel_pick(SelectState *st, int shift, int bits)
{
    __shared__ uint32_t s_tmp[kWaves];
    sel_pick(st, shift, bits, st->prefix, st->mask, s_tmp);
}

// One digit: every workgroup counts its entries of the selected prefix.  PICK:
// the last one to finish takes the digit, which saves a launch but has every
// workgroup report to one counter in turn (about 50 ns each): only for the few
// workgroups of a short input.
template <bool PICK>
__global__ __launch_bounds__(kThreads) void k_sel_hist(const double *__restrict__ score, size_t n, int shift, int bits,
                                                       SelectState *st, const uint32_t *dn)
{
    __shared__ uint32_t h[kSelBins];
    __shared__ uint32_t s_tmp[kWaves];
    __shared__ bool last;
    n = dev_n(n, dn);
    for (int i = threadIdx.x; i < kSelBins; i += kThreads) h[i] = 0u;
    __syncthreads();
    const uint64_t prefix = st->prefix, mask = st->mask;
    const uint32_t dmask = (1u << bits) - 1u;
    // the workgroups stride over the tiles, so that few of them add their
    // counts to the global bins (the leading digits of |A| fall into very few
    // bins, and atomics on one address serialise)
    for (size_t base = (size_t)blockIdx.x * kTile; base < n; base += (size_t)gridDim.x * kTile) {
        for (int i = threadIdx.x; i < kTile; i += kThreads) {
            const size_t j = base + i;
            if (j < n) {
                const uint64_t o = abs_order(score[j]);
                if ((o & mask) == prefix) atomicAdd(&h[(uint32_t)(o >> shift) & dmask], 1u);
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kSelBins; i += kThreads)
        if (h[i]) atomicAdd(&st->hist[i], h[i]);
    if (!PICK) return;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(&st->done, 1u) + 1u == gridDim.x;
    __syncthreads();
    if (!last) return;
    __threadfence();
    sel_pick(st, shift, bits, prefix, mask, s_tmp);
}

// the entries that still match the selected prefix, copied (in any order:
// only their count per digit matters) to a smaller array
__global__ __launch_bounds__(kThreads) void k_sel_compact(const double *__restrict__ score, size_t n,
                                                          const SelectState *__restrict__ st, double *__restrict__ out,
                                                          unsigned int *__restrict__ count, const uint32_t *dn)
{
    n = dev_n(n, dn);
    const uint64_t prefix = st->prefix, mask = st->mask;
    const size_t base = (size_t)blockIdx.x * kTile;
    const int lane = threadIdx.x & 63;
    const uint64_t lt = (1ull << lane) - 1ull;
    if (base >= n) return;  // uniform
    for (int i = threadIdx.x; i < kTile; i += kThreads) {
        const size_t j = base + i;
        const double v = j < n ? score[j] : 0.0;
        const bool keep = j < n && (abs_order(v) & mask) == prefix;
        const uint64_t b = __ballot(keep);
        unsigned int at = 0;
        if (lane == 0 && b) at = atomicAdd(count, (unsigned int)__popcll(b));
        at = __shfl(at, 0, 64);
        if (keep) out[at + __popcll(b & lt)] = v;
    }
}

}  // namespace

__global__ __launch_bounds__(64) void k_fill_u32(uint32_t *p, uint32_t n, uint32_t v)
{
    for (uint32_t i = blockIdx.x * 64 + threadIdx.x; i < n; i += gridDim.x * 64) p[i] = v;
}

void fill_u32(uint32_t *p, size_t n, uint32_t v, hipStream_t s)
{
    if (n == 0) return;
    k_fill_u32<<<(unsigned)std::min<size_t>((n + 63) / 64, 4096), 64, 0, s>>>(p, (uint32_t)n, v);
    ASCI_LAUNCH_CHECK();
}

void scan_u32(const uint32_t *in, uint32_t *out, size_t n, uint32_t *d_total, Arena &ar, hipStream_t s,
              Profiler *prof, const uint32_t *dn)
{
    if (n == 0) {
        if (d_total) {
            k_fill_u32<<<1, 64, 0, s>>>(d_total, 1, 0u);
            ASCI_LAUNCH_CHECK();
        }
        return;
    }
    ProfScope ps(prof, "scan", 8.0 * n, s);
    if (n <= kScanSmall) {
        k_scan_small<<<1, 1024, 0, s>>>(in, out, (uint32_t)n, d_total, dn);
        ASCI_LAUNCH_CHECK();
        return;
    }
    size_t nb = (n + kTile - 1) / kTile;
    require(nb <= (1u << 26), ASCI_EINVAL, "scan too long");
    uint32_t *partial = ar.take<uint32_t>(nb);
    k_scan_reduce<<<(unsigned)nb, kThreads, 0, s>>>(in, n, partial, dn);
    ASCI_LAUNCH_CHECK();
    k_scan_partials<<<1, 1024, 0, s>>>(partial, (uint32_t)nb, d_total);
    ASCI_LAUNCH_CHECK();
    k_scan_down<<<(unsigned)nb, kThreads, 0, s>>>(in, out, n, partial, dn);
    ASCI_LAUNCH_CHECK();
}

template <int KW>
int merge_sort(uint64_t *(*keys)[2], uint32_t *vals[2], const double *score, size_t n, hipStream_t s, Profiler *prof,
               const uint32_t *dn)
{
    require(n < (1ull << 32), ASCI_EINVAL, "sort: too many records");
    if (n == 0) return 0;
    constexpr size_t CH = kSortChunk;
    ProfScope ps(prof, "sort", (8.0 * KW + 4.0) * 2.0 * n, s);
    SortKeys<KW> k[2];
    for (int i = 0; i < KW; ++i)
        for (int b = 0; b < 2; ++b) k[b].w[i] = keys[i][b];
    k_sort_chunks<KW><<<(unsigned)((n + CH - 1) / CH), kSortT, 0, s>>>(k[0], score, k[1], vals[1], n, dn);
    ASCI_LAUNCH_CHECK();
    int cur = 1;
    for (size_t width = CH; width < n; width *= kSortWays) {
        k_sort_merge<KW><<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(k[cur], vals[cur], k[cur ^ 1],
                                                                                      vals[cur ^ 1], n, width, dn);
        ASCI_LAUNCH_CHECK();
        cur ^= 1;
    }
    return cur;
}

size_t sort_bytes(size_t n)
{
    const size_t nb = (n + kTile - 1) / kTile;
    return n > kRadixFrom ? nb * 256 * 4 + (nb * 256 / kTile + 1) * 4 + 512 : 0;
}

int sort_keys(uint64_t *keys[2], uint32_t *vals[2], const double *score, size_t n, int bits, Arena &ar, hipStream_t s,
              Profiler *prof, const uint32_t *dn)
{
    if (n <= kRadixFrom || ar.capacity() - ar.used() < sort_bytes(n)) {
        uint64_t *k[1][2] = {{keys[0], keys[1]}};
        return merge_sort<1>(k, vals, score, n, s, prof, dn);
    }
    require(n < (1ull << 32), ASCI_EINVAL, "sort: too many records");
    ProfScope ps(prof, "sort", (8.0 + 4.0) * 2.0 * n, s);
    const size_t nb = (n + kTile - 1) / kTile;
    uint32_t *hist = ar.take<uint32_t>(nb * 256);
    const size_t mark = ar.used();
    k_rs_keys<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(score, keys[0], vals[0], n, dn);
    ASCI_LAUNCH_CHECK();
    int cur = 0;
    for (int shift = 0; shift < bits; shift += 8, cur ^= 1) {
        k_rs_hist<<<(unsigned)nb, kThreads, 0, s>>>(keys[cur], n, shift, hist, (uint32_t)nb, dn);
        ASCI_LAUNCH_CHECK();
        scan_u32(hist, hist, nb * 256, nullptr, ar, s);
        ar.reset();
        (void)ar.take<char>(mark);
        k_rs_scatter<<<(unsigned)nb, kThreads, 0, s>>>(keys[cur], vals[cur], keys[cur ^ 1], vals[cur ^ 1], n, shift, hist,
                                                       (uint32_t)nb, dn);
        ASCI_LAUNCH_CHECK();
    }
    return cur;
}

template int merge_sort<2>(uint64_t *(*)[2], uint32_t *[2], const double *, size_t, hipStream_t, Profiler *, const uint32_t *);
template int merge_sort<3>(uint64_t *(*)[2], uint32_t *[2], const double *, size_t, hipStream_t, Profiler *, const uint32_t *);

Profiler::~Profiler()
{
    for (auto &p : pending_) {
        (void)hipEventDestroy(p.a);
        (void)hipEventDestroy(p.b);
    }
    for (auto e : pool_) (void)hipEventDestroy(e);
}

hipEvent_t Profiler::get_event()
{
    if (!pool_.empty()) {
        hipEvent_t e = pool_.back();
        pool_.pop_back();
        return e;
    }
    hipEvent_t e;
    ASCI_HIP(hipEventCreate(&e));
    return e;
}

int Profiler::begin(const char *name, double bytes, hipStream_t s)
{
    int idx = -1;
    for (size_t i = 0; i < entries.size(); ++i)
        if (entries[i].name == name) idx = (int)i;
    if (idx < 0) {
        entries.push_back(ProfEntry{name});
        idx = (int)entries.size() - 1;
    }
    Pending p{idx, get_event(), get_event(), bytes};
    ASCI_HIP(hipEventRecord(p.a, s));
    pending_.push_back(p);
    return (int)pending_.size() - 1;
}

void Profiler::end(int token, hipStream_t s) { ASCI_HIP(hipEventRecord(pending_[token].b, s)); }

void Profiler::set_bytes(int token, double bytes)
{
    if (token >= 0 && (size_t)token < pending_.size()) pending_[(size_t)token].bytes = bytes;
}

void Profiler::collect()
{
    for (auto &p : pending_) {
        float ms = 0.f;
        ASCI_HIP(hipEventSynchronize(p.b));
        ASCI_HIP(hipEventElapsedTime(&ms, p.a, p.b));
        ProfEntry &e = entries[p.entry];
        e.ms += ms;
        e.launches += 1;
        e.bytes += p.bytes;
        pool_.push_back(p.a);
        pool_.push_back(p.b);
    }
    pending_.clear();
}

void Profiler::reset()
{
    collect();
    entries.clear();
}

void radix_select_abs(const double *score, size_t n, uint64_t k, SelectState *d_state, hipStream_t s,
                      Profiler *prof, const SelectWork *work, const uint32_t *dn, const uint32_t *dk)
{
    require(k >= 1 && k <= n, ASCI_EINVAL, "radix select: k out of range");
    // Few scores: 32 workgroups a pass, the last of which picks the digit.  More:
    // a launch of its own picks it, and the entries that match two digits are
    // copied out.  At 9e5 scores the first took 178 us, the second 90; at 2e5 54 and 75.
    bool few = n <= ((size_t)1 << 18);
    if (few) work = nullptr;
    const unsigned nb = (unsigned)((n + kTile - 1) / kTile);
    k_sel_init<<<1, 1024, 0, s>>>(d_state, k, dk, work ? work->d_count : nullptr);
    ASCI_LAUNCH_CHECK();
    const double *x = score;
    // the 63 bits of |A|, most significant first
    for (int pass = 0, shift = 63; pass < 6; ++pass) {
        const int bits = pass < 3 ? 11 : 10;
        shift -= bits;
        if (pass == 2 && work) {
            ProfScope ps(prof, "select_compact", 8.0 * n, s);
            k_sel_compact<<<nb, kThreads, 0, s>>>(x, n, d_state, work->tmp, work->d_count, dn);
            ASCI_LAUNCH_CHECK();
            x = work->tmp;
            dn = work->d_count;
            few = true;
        }
        ProfScope ps(prof, "select_hist", 8.0 * n, s);
        if (few) {
            k_sel_hist<true><<<std::min(nb, 32u), kThreads, 0, s>>>(x, n, shift, bits, d_state, dn);
            ASCI_LAUNCH_CHECK();
        } else {
            k_sel_hist<false><<<std::min(nb, 2048u), kThreads, 0, s>>>(x, n, shift, bits, d_state, dn);
            ASCI_LAUNCH_CHECK();
            k_sel_pick<<<1, kThreads, 0, s>>>(d_state, shift, bits);
            ASCI_LAUNCH_CHECK();
        }
    }
}

}  // namespace asci
