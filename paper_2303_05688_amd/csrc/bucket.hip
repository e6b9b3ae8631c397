// Sort-and-accumulate of one class batch by buckets (Alg. 2, the sort on
// the target bitstring and the sum per unique target), built for LDS:
//
//   segments: contiguous record ranges in key order; the classes of the batch
//             are the first segments (the generator lays records out class by
//             class).
//   split   : a segment larger than the capacity of one wavefront's LDS share
//             is split, stably, into up to 256 key ranges bounded by splitters
//             sampled from it (sample sort: the ranges are balanced however
//             skewed the keys are, and they keep key order), with per-tile
//             histograms laid out segment by segment, one global exclusive
//             scan and a ranked scatter into the other buffer.  Repeat level
//             by level.  A sampled key that fills several quantiles gets a
//             range of its own, so a range that stays too large either divides
//             at the next level or holds a single key.  Ranges of at most one
//             tile that a wavefront cannot hold yet are split last, each by one
//             workgroup in one read and one write of its records.
//   finish  : one wavefront per final segment, with no barrier: it sorts the
//             segment's record indices in its LDS share (stable LSD on a 32-bit
//             window of each key that holds the bits varying inside the
//             segment), puts the values in sorted order, sums every run of
//             equal keys in record order (record order is ascending core
//             index), drops input determinants (and, after an earlier class
//             batch, candidates below the pool's k-th |A|), forms H_aa and
//             A_a, and writes the surviving candidates, compacted, at the
//             segment's start in slot arrays; a bit per slot marks them.
//   collect : the marked slots, in slot (= key) order, are copied to the pool.
//
// Keys are handled as the 2n-bit value (alpha << n) | beta: one word for
// n <= 32, two words (hi = alpha, lo = beta) above.
#include "hamiltonian.h"

#include <algorithm>
#include <type_traits>
#include <vector>

namespace asci {

namespace {

constexpr int kTileT = 1024;          // threads of the scatter: two workgroups of 16 waves per CU
constexpr int kTileItems = 4;
constexpr int kHistT = 256;           // threads of the histogram pass
constexpr int kTileN = kTileT * kTileItems;  // 4096 records per tile

// Records one wavefront finishes: an eighth of the workgroup capacity that
// finish_cap names (eight wavefronts share a workgroup and its tables), and 256
// at least.  Shares of 128, for a finish_cap of 1024, were slower than 256 at
// every size: ms, 128 and 256, 8e12o 0.30 and 0.27, 16e20o of 1.3e8 pairs 9.4 and
// 7.3, 24e30o of 2.7e8 30.6 and 24.1, 20e36o of 9.7e7 15.2 and 12.7.
constexpr int kFinishWaves = 8;
inline int wave_cap(int finish_cap) { return (finish_cap >= 4096 ? 4096 : 2048) / kFinishWaves; }

struct Seg {
    uint32_t start, size, meta;  // meta: buf (bit 0) | single key (bit 1)
};

__host__ __device__ __forceinline__ uint32_t seg_buf(const Seg &s) { return s.meta & 1u; }
__host__ __device__ __forceinline__ bool seg_single(const Seg &s) { return (s.meta >> 1) & 1u; }
__host__ __device__ __forceinline__ uint32_t make_meta(uint32_t buf, bool single) { return buf | (single ? 2u : 0u); }

constexpr int kMaxSplit = 256;       // ranges per split
constexpr int kSplitSample = 8;      // samples per range

template <int W>
__device__ __forceinline__ bool key_less(uint64_t alo, uint64_t ahi, uint64_t blo, uint64_t bhi)
{
    return W == 1 ? alo < blo : (ahi < bhi || (ahi == bhi && alo < blo));
}

// a value every lane of the wavefront holds, moved to a scalar register
__device__ __forceinline__ uint32_t uniform32(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ uint64_t uniform64(uint64_t x)
{
    return (uint64_t)uniform32((uint32_t)x) | ((uint64_t)uniform32((uint32_t)(x >> 32)) << 32);
}

// One data-parallel-primitive step: x of another lane (row_shr:n within a row
// of 16 lanes, row_bcast:15 / row_bcast:31 across rows), 0 where there is none.
// Every lane of the wavefront must be active.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_from(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}

// x of the lane before, `first` in lane 0
__device__ __forceinline__ uint32_t lane_before(uint32_t x, uint32_t first)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)x, 0x138, 0xF, 0xF, false);
}

// inclusive sum over the lanes: six register moves, where a shuffle would make
// six round trips through the LDS unit
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x)
{
    x += dpp_from<0x111, 0xF>(x);
    x += dpp_from<0x112, 0xF>(x);
    x += dpp_from<0x114, 0xF>(x);
    x += dpp_from<0x118, 0xF>(x);
    x += dpp_from<0x142, 0xA>(x);
    x += dpp_from<0x143, 0xC>(x);
    return x;
}

// OR over the lanes, in a scalar register
__device__ __forceinline__ uint32_t wave_or(uint32_t x)
{
    x |= dpp_from<0x111, 0xF>(x);
    x |= dpp_from<0x112, 0xF>(x);
    x |= dpp_from<0x114, 0xF>(x);
    x |= dpp_from<0x118, 0xF>(x);
    x |= dpp_from<0x142, 0xA>(x);
    x |= dpp_from<0x143, 0xC>(x);
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ uint64_t wave_or64(uint64_t x)
{
    return (uint64_t)wave_or((uint32_t)x) | ((uint64_t)wave_or((uint32_t)(x >> 32)) << 32);
}

// Orders the LDS accesses of one wavefront around it (its lanes run in
// lockstep and the LDS unit takes a wavefront's accesses in order, so only the
// compiler has to be held back).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// exclusive scan over the block (NW waves); every thread must call it
template <int NW>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *s_tmp, uint32_t &total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t x = wave_incl_scan(v);
    if (lane == 63) s_tmp[w] = x;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const uint32_t t = s_tmp[i];
        base += (i < w) ? t : 0u;
        tot += t;
    }
    total = tot;
    __syncthreads();
    return base + x - v;
}

__device__ __forceinline__ uint32_t dev_count(uint32_t n, const uint32_t *dn) { return dn ? min(n, *dn) : n; }

// ---------------------------------------------------------------- split level
// ranges of a split: about half the capacity each, 3 to 256 (three ranges have
// the two splitters that can isolate one key)
__host__ __device__ __forceinline__ uint32_t split_ranges(uint32_t size, uint32_t cap)
{
    const uint64_t want = ((uint64_t)size * 2 + cap - 1) / cap;
    return (uint32_t)(want < 3 ? 3 : (want > (uint64_t)kMaxSplit ? (uint64_t)kMaxSplit : want));
}
__host__ __device__ __forceinline__ uint32_t seg_tiles(uint32_t size) { return (size + kTileN - 1) / kTileN; }
// where a segment's splitters start: a segment larger than cap has at most
// 2 size / cap of them, so the disjoint segments' ranges do not overlap
__host__ __device__ __forceinline__ size_t split_at(uint32_t start, uint32_t cap)
{
    return (size_t)((uint64_t)start * 2 / cap);
}
// bounds of one level's tiles and histogram entries, for nseg segments of more
// than cap records out of P
inline size_t level_tiles(size_t P, size_t nseg) { return P / kTileN + nseg; }
inline size_t level_hist(size_t P, size_t nseg, size_t cap)
{
    return P / (kTileN / kMaxSplit) + std::min<size_t>((size_t)kMaxSplit * nseg, 2 * P / cap + 3 * nseg);
}

struct SplitArgs {
    const Seg *segs;            // large segments of this level
    const uint32_t *tile_base;  // per segment: first tile
    const uint32_t *hist_base;  // per segment: first histogram entry
    const uint32_t *tile_seg;   // per tile: its segment
    uint32_t ntiles;            // bound; the count is lev[0]
    const uint32_t *lev;        // tiles, histogram entries of the level
    uint32_t *hist;             // segment-major, range-major inside a segment, then tile
    uint64_t *klo[2], *khi[2];
    double *val[2];
    uint32_t cap;
    const uint64_t *spl_lo, *spl_hi;  // splitters, at split_at of each segment
    uint8_t *dig;                     // per record: its range, from the histogram pass
};

struct KeyBufs {
    const uint64_t *lo[2], *hi[2];
};

// Splitters of every large segment: kSplitSample records per range, taken at
// even strides (the records are in generation order, not key order, so a
// strided pick is a fair sample), sorted in LDS by a bitonic network; the
// splitters are the sample's quantiles.  A quantile equal to the one before it
// becomes the next larger key, so that a key which fills more than one quantile
// has a range of its own.
template <int W, int T>
__global__ __launch_bounds__(T) void k_seg_splitters(const Seg *__restrict__ segs, uint32_t cap, KeyBufs kb,
                                                       uint64_t *__restrict__ g_lo, uint64_t *__restrict__ g_hi,
                                                       uint32_t nseg, const uint32_t *dn_seg)
{
    constexpr int kMaxSample = kMaxSplit * kSplitSample;
    __shared__ uint64_t x_lo[kMaxSample];
    __shared__ uint64_t x_hi[W == 2 ? kMaxSample : 1];
    const uint32_t ns = dev_count(nseg, dn_seg);
    for (uint32_t s = blockIdx.x; s < ns; s += gridDim.x) {
        const Seg sg = segs[s];
        const uint32_t nb = split_ranges(sg.size, cap);
        const uint32_t m = min(sg.size, nb * (uint32_t)kSplitSample);
        uint32_t p = 1;
        while (p < m) p <<= 1;
        const uint64_t *klo = kb.lo[seg_buf(sg)], *khi = kb.hi[seg_buf(sg)];
        __syncthreads();  // the previous segment's samples are read
        for (uint32_t i = threadIdx.x; i < p; i += T) {
            if (i < m) {
                const size_t j = (size_t)sg.start + (size_t)(((uint64_t)2 * i + 1) * sg.size / (2 * (uint64_t)m));
                x_lo[i] = klo[j];
                if (W == 2) x_hi[i] = khi[j];
            } else {
                x_lo[i] = ~0ull;
                if (W == 2) x_hi[i] = ~0ull;
            }
        }
        __syncthreads();
        // pair t of a stage is (i, i + jj) with i = t with a zero bit inserted at
        // jj: every lane works, and up to jj = 64 a wavefront's 64 pairs lie in
        // its own 128 elements, so those stages need no barrier between them
        for (uint32_t k = 2; k <= p; k <<= 1) {
            for (uint32_t jj = k >> 1; jj > 0; jj >>= 1) {
                for (uint32_t t = threadIdx.x; t < p / 2; t += T) {
                    const uint32_t i = 2u * (t & ~(jj - 1u)) + (t & (jj - 1u)), o = i + jj;
                    const bool up = (i & k) == 0;
                    const uint64_t al = x_lo[i], bl = x_lo[o];
                    const uint64_t ah = W == 2 ? x_hi[i] : 0ull, bh = W == 2 ? x_hi[o] : 0ull;
                    if (key_less<W>(bl, bh, al, ah) == up) {
                        x_lo[i] = bl;
                        x_lo[o] = al;
                        if (W == 2) {
                            x_hi[i] = bh;
                            x_hi[o] = ah;
                        }
                    }
                }
                if (jj > 64u || (jj == 1u && k >= 128u)) __syncthreads();
                else wave_sync();
            }
        }
        __syncthreads();
        const size_t at = split_at(sg.start, cap);
        for (uint32_t j = threadIdx.x; j + 1u < nb; j += T) {
            const uint32_t q = (uint32_t)(((uint64_t)(j + 1) * m) / nb);
            const uint32_t q0 = (uint32_t)(((uint64_t)j * m) / nb);
            uint64_t lo = x_lo[q], hi = W == 2 ? x_hi[q] : 0ull;
            if (j > 0 && lo == x_lo[q0] && (W == 1 || hi == x_hi[q0])) {
                ++lo;  // the next larger key (no stored key is all ones)
                if (W == 2 && lo == 0ull) ++hi;
            }
            g_lo[at + j] = lo;
            if (W == 2) g_hi[at + j] = hi;
        }
    }
}

// the segment of a tile: the last one that starts at or before it
__device__ __forceinline__ uint32_t seg_of_tile(const uint32_t *tile_base, uint32_t ns, uint32_t t)
{
    uint32_t l = 0, r = ns;  // tile_base[l] <= t
    while (r - l > 1u) {
        const uint32_t m = (l + r) >> 1;
        if (tile_base[m] <= t) l = m;
        else r = m;
    }
    return l;
}

// One workgroup lays a level out: first tile and first histogram entry of
// every large segment, the totals, cleared skip flags and next-level count, and
// (tile_seg given: few tiles) the segment of every tile.
__global__ __launch_bounds__(1024) void k_level_plan(const Seg *__restrict__ segs, uint32_t nseg, uint32_t cap,
                                                     uint32_t *__restrict__ tile_base,
                                                     uint32_t *__restrict__ hist_base, uint32_t *__restrict__ skip,
                                                     uint32_t *__restrict__ lev, uint32_t *__restrict__ nnext,
                                                     uint32_t *__restrict__ tile_seg, const uint32_t *dn_seg,
                                                     uint32_t *__restrict__ nlevels, uint32_t *__restrict__ nrec)
{
    __shared__ uint32_t s_tmp[16], s_rec;
    const uint32_t ns = dev_count(nseg, dn_seg);
    uint32_t tiles = 0, entries = 0, rec = 0;
    if (threadIdx.x == 0) s_rec = 0u;
    for (uint32_t b = 0; b < ns; b += 4096) {
        const uint32_t s0 = b + threadIdx.x * 4u;
        uint32_t t[4], e[4], st = 0, se = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            t[k] = e[k] = 0u;
            if (s0 + k < ns) {
                const uint32_t size = segs[s0 + k].size;
                t[k] = seg_tiles(size);
                e[k] = t[k] * split_ranges(size, cap);
                rec += size;
            }
            st += t[k];
            se += e[k];
        }
        uint32_t tt, et;
        uint32_t at = tiles + block_scan<16>(st, s_tmp, tt), ae = entries + block_scan<16>(se, s_tmp, et);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (s0 + k < ns) {
                tile_base[s0 + k] = at;
                hist_base[s0 + k] = ae;
                skip[s0 + k] = 0u;
            }
            at += t[k];
            ae += e[k];
        }
        tiles += tt;
        entries += et;
    }
    if (threadIdx.x == 0) {
        lev[0] = tiles;
        lev[1] = entries;
        *nnext = 0u;
        if (ns > 0u) ++*nlevels;
    }
    if (nrec) {  // timing only: the records of the level
        __syncthreads();
        atomicAdd(&s_rec, rec);
        __syncthreads();
        if (threadIdx.x == 0) *nrec = s_rec;
    }
    if (!tile_seg) return;
    __syncthreads();  // the block's own writes of tile_base
    for (uint32_t t = threadIdx.x; t < tiles; t += 1024) tile_seg[t] = seg_of_tile(tile_base, ns, t);
}

__global__ __launch_bounds__(256) void k_tile_seg(const uint32_t *__restrict__ tile_base, uint32_t nseg,
                                                  const uint32_t *__restrict__ lev, uint32_t *__restrict__ tile_seg,
                                                  const uint32_t *dn_seg)
{
    const uint32_t ns = dev_count(nseg, dn_seg), nt = lev[0];
    for (uint32_t t = blockIdx.x * 256 + threadIdx.x; t < nt; t += gridDim.x * 256)
        tile_seg[t] = seg_of_tile(tile_base, ns, t);
}

// Tiles of a level, XCD-contiguous: the tiles [x * per, (x + 1) * per) go to
// XCD x (workgroups are handed to the 8 XCDs in turn), taken by that XCD's
// workgroups in turn.  With a grid of 8 * per workgroups each takes one tile.
#define FOR_LEVEL_TILES(a, t)                                                          \
    const uint32_t nt_all_ = min((a).ntiles, (a).lev[0]);                             \
    const uint32_t per_ = (nt_all_ + 7u) / 8u, slots_ = max(gridDim.x >> 3, 1u);      \
    for (uint32_t i_ = blockIdx.x >> 3, t = (blockIdx.x & 7u) * per_ + i_;            \
         i_ < per_ && t < nt_all_; i_ += slots_, t = (blockIdx.x & 7u) * per_ + i_)

template <int W>
__global__ __launch_bounds__(kHistT) void k_split_hist(SplitArgs a)
{
    __shared__ uint32_t h[kHistT / 64][256];
    __shared__ uint64_t spl_lo[kMaxSplit - 1];
    __shared__ uint64_t spl_hi[W == 2 ? kMaxSplit - 1 : 1];
    FOR_LEVEL_TILES(a, t) {
        const uint32_t s = a.tile_seg[t];
        const Seg sg = a.segs[s];
        const uint32_t nt = seg_tiles(sg.size), tl = t - a.tile_base[s];
        const uint32_t nb = split_ranges(sg.size, a.cap);
        const uint32_t buf = seg_buf(sg);
        const size_t at = split_at(sg.start, a.cap);
        __syncthreads();  // the previous tile's counts are written out
        for (int i = threadIdx.x; i < (kHistT / 64) * 256; i += kHistT) (&h[0][0])[i] = 0u;
        // unused splitters hold the largest key
        for (uint32_t j = threadIdx.x; j < kMaxSplit - 1; j += kHistT) {
            const bool used = j + 1u < nb;
            spl_lo[j] = used ? a.spl_lo[at + j] : ~0ull;
            if (W == 2) spl_hi[j] = used ? a.spl_hi[at + j] : ~0ull;
        }
        __syncthreads();
        const uint32_t r0 = tl * kTileN, r1 = min(sg.size, r0 + kTileN);
        const int wv = threadIdx.x >> 6;
        // four records per step, their searches interleaved
        for (uint32_t rb = r0 + threadIdx.x; rb < r1; rb += 4 * kHistT) {
            uint64_t lo[4], hi[4];
            uint32_t dg[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t r = rb + (uint32_t)k * kHistT;
                const size_t j = (size_t)sg.start + (r < r1 ? r : r0);
                lo[k] = a.klo[buf][j];
                hi[k] = W == 2 ? a.khi[buf][j] : 0ull;
                dg[k] = 0u;
            }
            // the range of a key is the number of splitters <= it, by binary
            // lifting over the 255 entries: no branches
#pragma unroll
            for (uint32_t step = 128; step >= 1; step >>= 1) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t m = dg[k] + step - 1u;
                    const bool le = W == 1 ? spl_lo[m] <= lo[k]
                                           : (spl_hi[m] < hi[k] || (spl_hi[m] == hi[k] && spl_lo[m] <= lo[k]));
                    dg[k] += le ? step : 0u;
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t r = rb + (uint32_t)k * kHistT;
                if (r < r1) {
                    const uint32_t d = min(dg[k], nb - 1u);
                    a.dig[(size_t)sg.start + r] = (uint8_t)d;
                    atomicAdd(&h[wv][d], 1u);
                }
            }
        }
        __syncthreads();
        const uint32_t d = threadIdx.x;
        if (d < nb) {
            uint32_t c = 0;
#pragma unroll
            for (int i = 0; i < kHistT / 64; ++i) c += h[i][d];
            a.hist[(size_t)a.hist_base[s] + (size_t)d * nt + tl] = c;
        }
    }
}

// Greedy grouping of consecutive parts of sizes pre[i + 1] - pre[i], i < m,
// into groups of at most cap records (a larger part is a group of its own):
// next[i] is the end of the group that would start at part i, mark[i] tells
// whether one does.  Pointer doubling: after round r every start within 2^r
// groups of the first is marked.  pre, next, jump (m + 1 entries each) and mark
// lie in LDS; the T threads tid of a block (or of a wavefront, with sync to
// match) share the work, at most P parts each.
template <int P, typename Sync>
__device__ __forceinline__ void greedy_groups(const uint32_t *pre, uint32_t m, uint32_t cap, uint16_t *next,
                                              uint16_t *jump, uint8_t *mark, uint32_t tid, uint32_t T, Sync sync)
{
    uint32_t bits = 1;
    while ((1u << bits) <= m) ++bits;
#pragma unroll
    for (int c = 0; c < P; ++c) {
        const uint32_t i = tid + (uint32_t)c * T;
        if (i > m) continue;
        uint32_t l = i;  // largest l <= m with pre[l] - pre[i] <= cap
        for (uint32_t step = 1u << (bits - 1u); step; step >>= 1)
            if (l + step <= m && pre[l + step] - pre[i] <= cap) l += step;
        const uint32_t nx = i >= m ? m : max(l, i + 1u);
        next[i] = (uint16_t)nx;
        jump[i] = (uint16_t)nx;
        mark[i] = i == 0u ? 1 : 0;
    }
    sync();
    for (uint32_t r = 0; r < bits; ++r) {
        uint32_t j2[P];
#pragma unroll
        for (int c = 0; c < P; ++c) {
            const uint32_t i = tid + (uint32_t)c * T;
            const uint32_t j = i <= m ? jump[i] : m;
            if (i <= m && mark[i]) mark[j] = 1;
            j2[c] = jump[j];
        }
        sync();
#pragma unroll
        for (int c = 0; c < P; ++c) {
            const uint32_t i = tid + (uint32_t)c * T;
            if (i <= m) jump[i] = (uint16_t)j2[c];
        }
        sync();
    }
}

// where new segments go: finals, segments of one tile at most, larger ones
struct SegLists {
    Seg *finals, *small, *next;
    uint32_t *nfinal, *nsmall, *nnext, *overflow;
    uint32_t finals_cap, small_cap, next_cap;
};
__device__ __forceinline__ void put_seg(Seg *list, uint32_t cap, uint32_t i, const Seg &c, uint32_t *overflow)
{
    if (i < cap) list[i] = c;
    else atomicOr(overflow, 1u);
}
// appends the wavefront's segments (kind 0 none, 1 final, 2 small, 3 next): one
// atomic per list
__device__ __forceinline__ void append_segs(const SegLists &l, uint32_t kind, const Seg &c)
{
    const int lane = threadIdx.x & 63;
    const uint64_t lt = (1ull << lane) - 1ull;
    const uint64_t f = __ballot(kind == 1u), m = __ballot(kind == 2u), x = __ballot(kind == 3u);
    uint32_t at = 0;
    if (lane == 0 && f) at = atomicAdd(l.nfinal, (uint32_t)__popcll(f));
    if (lane == 1 && m) at = atomicAdd(l.nsmall, (uint32_t)__popcll(m));
    if (lane == 2 && x) at = atomicAdd(l.nnext, (uint32_t)__popcll(x));
    const uint32_t bf = (uint32_t)__builtin_amdgcn_readlane((int)at, 0);
    const uint32_t bm = (uint32_t)__builtin_amdgcn_readlane((int)at, 1);
    const uint32_t bx = (uint32_t)__builtin_amdgcn_readlane((int)at, 2);
    if (kind == 1u) put_seg(l.finals, l.finals_cap, bf + (uint32_t)__popcll(f & lt), c, l.overflow);
    if (kind == 2u) put_seg(l.small, l.small_cap, bm + (uint32_t)__popcll(m & lt), c, l.overflow);
    if (kind == 3u) put_seg(l.next, l.next_cap, bx + (uint32_t)__popcll(x & lt), c, l.overflow);
}

// Children of every large segment, one wavefront per segment (no barrier).
// Ranges larger than the capacity become small or large segments, or
// single-key finals; runs of consecutive smaller ranges are coalesced into
// final segments of at most `cap` records.  A segment whose records all fall in
// one range has one key (its splitters would otherwise divide it): it is not
// moved (skip[s] = 1) and becomes a single-key final in its buffer.
constexpr int kChildWaves = 4;
template <int W>
__global__ __launch_bounds__(64 * kChildWaves) void k_split_children(const Seg *__restrict__ segs, uint32_t nseg,
                                                        const uint32_t *__restrict__ hist_base,
                                                        const uint32_t *__restrict__ scan, uint32_t cap,
                                                        const uint64_t *__restrict__ spl_lo,
                                                        const uint64_t *__restrict__ spl_hi,
                                                        uint32_t *__restrict__ skip, SegLists lists,
                                                        const uint32_t *dn_seg)
{
    __shared__ uint32_t s_pre[kChildWaves][kMaxSplit + 1];
    __shared__ uint16_t s_next[kChildWaves][kMaxSplit + 2], s_jump[kChildWaves][kMaxSplit + 2];
    __shared__ uint8_t s_mark[kChildWaves][kMaxSplit + 2];
    const uint32_t ns = dev_count(nseg, dn_seg);
    const uint32_t wv = uniform32(threadIdx.x >> 6), lane = threadIdx.x & 63;
    uint32_t *pre = s_pre[wv];
    for (uint32_t s = blockIdx.x * kChildWaves + wv; s < ns; s += gridDim.x * kChildWaves) {
        const Seg sg = segs[s];
        const uint32_t nt = seg_tiles(sg.size), nb = split_ranges(sg.size, cap);
        const size_t b0 = (size_t)hist_base[s], sp = split_at(sg.start, cap);
        const uint32_t base = scan[b0];
        wave_sync();
        bool one_key[kMaxSplit / 64];
#pragma unroll
        for (int c = 0; c < kMaxSplit / 64; ++c) {
            const uint32_t d = (uint32_t)c * 64 + lane;
            one_key[c] = false;
            if (d < nb) pre[d] = scan[b0 + (size_t)d * nt] - base;
            // range d holds one key when its bounds are consecutive keys
            if (d > 0 && d + 1u < nb) {
                const size_t at = sp + d;
                const uint64_t lo = spl_lo[at - 1] + 1ull;
                one_key[c] = W == 1 ? spl_lo[at] == lo
                                    : (spl_lo[at] == lo && spl_hi[at] == spl_hi[at - 1] + (lo == 0ull ? 1ull : 0ull));
            }
        }
        if (lane == 0) pre[nb] = sg.size;
        wave_sync();
        greedy_groups<kMaxSplit / 64 + 1>(pre, nb, cap, s_next[wv], s_jump[wv], s_mark[wv], lane, 64u, [] { wave_sync(); });
#pragma unroll
        for (int c = 0; c < kMaxSplit / 64; ++c) {
            const uint32_t d = (uint32_t)c * 64 + lane;
            if ((uint32_t)c * 64 >= nb) break;  // uniform
            uint32_t kind = 0;
            Seg ch{0u, 0u, 0u};
            if (d < nb && s_mark[wv][d]) {
                const uint32_t size = pre[s_next[wv][d]] - pre[d];
                const bool whole = size == sg.size;  // more than cap records: a single range
                if (size > 0u) kind = size <= cap || one_key[c] ? 1u : (size <= kTileN ? 2u : 3u);
                if (whole) {
                    skip[s] = 1u;
                    if (!one_key[c]) raise_fault(kFaultSlot);
                    kind = 1u;
                }
                ch = Seg{sg.start + pre[d], size, make_meta(seg_buf(sg) ^ (whole ? 0u : 1u), size > cap)};
            }
            append_segs(lists, kind, ch);
        }
    }
}

template <int W>
// eight waves per SIMD (64 VGPRs): the load, rank and write phases of four
// workgroups' worth of waves overlap on each CU
__global__ __launch_bounds__(kTileT) __attribute__((amdgpu_waves_per_eu(8))) void k_split_scatter(SplitArgs a,
                                                          const uint32_t *__restrict__ skip)
{
    constexpr int NW = kTileT / 64;
    __shared__ uint64_t s_lo[kTileN];
    __shared__ uint64_t s_hi[W == 2 ? kTileN : 1];
    __shared__ double s_val[kTileN];
    __shared__ uint16_t s_wcnt[NW][256];  // counts and prefixes below kTileN
    __shared__ uint32_t s_dbase[256];
    __shared__ uint32_t s_gbase[256];
    __shared__ uint32_t s_tmp[NW];
    __shared__ uint8_t s_dg[kTileN];

    FOR_LEVEL_TILES(a, t) {
    const uint32_t s = a.tile_seg[t];
    if (skip[s]) continue;  // uniform per block
    const Seg sg = a.segs[s];
    const uint32_t nt = seg_tiles(sg.size), tl = t - a.tile_base[s], nb = split_ranges(sg.size, a.cap);
    const uint32_t ib = seg_buf(sg), ob = ib ^ 1u;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    __syncthreads();  // the previous tile's records are written out
    for (int i = tid; i < NW * 256; i += kTileT) (&s_wcnt[0][0])[i] = 0u;
    __syncthreads();
    const uint32_t r0 = tl * kTileN, rn = min(sg.size - r0, (uint32_t)kTileN);
    uint64_t rlo[kTileItems], rhi[kTileItems];
    double rv[kTileItems];
    uint32_t rrank[kTileItems], rd[kTileItems];
    const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int q = 0; q < kTileItems; ++q) {
        const uint32_t li = (uint32_t)wv * 64 * kTileItems + (uint32_t)q * 64 + lane;
        const bool valid = li < rn;
        const size_t j = (size_t)sg.start + r0 + li;
        rlo[q] = valid ? a.klo[ib][j] : 0ull;
        rhi[q] = (W == 2 && valid) ? a.khi[ib][j] : 0ull;
        rv[q] = valid ? a.val[ib][j] : 0.0;
        const uint32_t d = valid ? (uint32_t)a.dig[j] : 0u;
        rd[q] = d;
        const uint64_t peers = wave_match(d, valid, 8);
        const uint32_t before = s_wcnt[wv][d];
        rrank[q] = before + (uint32_t)__popcll(peers & lt);
        if (valid && (peers & lt) == 0ull) s_wcnt[wv][d] = before + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    {
        const int d = tid;
        uint32_t run = 0;
        if (d < 256) {
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const uint32_t c = s_wcnt[i][d];
                s_wcnt[i][d] = run;
                run += c;
            }
        }
        uint32_t tot;
        const uint32_t e = block_scan<NW>(d < 256 ? run : 0u, s_tmp, tot);
        if ((uint32_t)d < nb) {
            s_dbase[d] = e;
            const size_t b0 = (size_t)a.hist_base[s];
            s_gbase[d] = sg.start + (a.hist[b0 + (size_t)d * nt + tl] - a.hist[b0]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kTileItems; ++q) {
        const uint32_t li = (uint32_t)wv * 64 * kTileItems + (uint32_t)q * 64 + lane;
        if (li < rn) {
            const uint32_t d = rd[q];
            const uint32_t p = min(s_dbase[d] + s_wcnt[wv][d] + rrank[q], (uint32_t)kTileN - 1u);
            s_lo[p] = rlo[q];
            if (W == 2) s_hi[p] = rhi[q];
            s_val[p] = rv[q];
            s_dg[p] = (uint8_t)d;
        }
    }
    __syncthreads();
    const uint32_t seg_end = sg.start + sg.size;
    for (uint32_t i = tid; i < rn; i += kTileT) {
        const uint64_t lo = s_lo[i];
        const uint64_t hi = W == 2 ? s_hi[i] : 0ull;
        const uint32_t d = s_dg[i];
        const uint32_t g = s_gbase[d] + (i - s_dbase[d]);
        if (g >= sg.start && g < seg_end) {
            a.klo[ob][g] = lo;
            if (W == 2) a.khi[ob][g] = hi;
            a.val[ob][g] = s_val[i];
        }
    }
    }
}

// Splits a segment of at most one tile (and more than cap records) into finals,
// in place, one workgroup per segment: the records are read once into
// registers, 16 samples a range are ranked against each other in LDS, and the
// records are written back range by range, each range in record order.  The
// separate splitter, histogram, scan and scatter launches of a level would read
// the records twice more and leave most of every tile empty.  A range of a
// single key that exceeds cap is a single-key final; one of several keys (the
// sample misled, as happens where targets have hundreds of contributions each)
// is split again by the same workgroup, on samples of its own: every split
// divides a range of several keys, so this ends.  Left to a later launch, such
// ranges sent small searches of dense spaces back to the step-by-step path (3.9
// million pairs of 13 + 6 electrons in 14 orbitals 1.16 ms, now 0.52).  Of
// 17,500 cycles a segment of 1000 records, 4900 went into ranking the samples
// (one thread counted all others for each) and 3500 into grouping the ranges by
// pointer doubling: 1.3e8 records of 16e20o took 1.29 ms, now 1.10 (3.8 TB/s).
constexpr int kSmallT = 512;
constexpr int kSmallItems = kTileN / kSmallT;
constexpr int kSmallMax = 64;      // ranges: half of cap each
constexpr int kSmallSample = 512;  // samples at most
constexpr int kMinCap = 2048 / kFinishWaves;  // the smallest wave_cap
template <int W>
__global__ __launch_bounds__(kSmallT) __attribute__((amdgpu_waves_per_eu(4))) void k_small_split(
    const Seg *__restrict__ segs, uint32_t nseg, const uint32_t *dn_seg, uint32_t cap, uint64_t *__restrict__ klo0,
    uint64_t *__restrict__ klo1, uint64_t *__restrict__ khi0, uint64_t *__restrict__ khi1, double *__restrict__ val0,
    double *__restrict__ val1, SegLists lists)
{
    constexpr int NW = kSmallT / 64;
    __shared__ uint64_t s_lo[kTileN];
    __shared__ uint64_t s_hi[W == 2 ? kTileN : 1];
    // the values of two-word keys take the array of the low words after these are written
    __shared__ double s_val[W == 1 ? kTileN : 1];
    __shared__ uint64_t q_lo[kSmallMax], q_hi[W == 2 ? kSmallMax : 1];
    __shared__ uint16_t s_wcnt[NW][kSmallMax];
    __shared__ uint32_t s_rank[kSmallSample];
    // ranges to be split again: disjoint, of more than cap of the segment's records
    __shared__ Seg s_left[kTileN / kMinCap];
    __shared__ uint32_t s_nleft;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint64_t lt = (1ull << lane) - 1ull;
    const uint32_t ns = dev_count(nseg, dn_seg);
    uint32_t left = 0;  // entries of s_left
    for (uint32_t s = blockIdx.x; left > 0u || s < ns;) {  // uniform
        Seg sg;
        if (left > 0u) {
            sg = s_left[--left];
        } else {
            sg = segs[s];
            s += gridDim.x;
        }
        const uint32_t size = sg.size, buf = seg_buf(sg);
        uint64_t *klo = (buf ? klo1 : klo0) + sg.start, *khi = W == 2 ? (buf ? khi1 : khi0) + sg.start : nullptr;
        double *val = (buf ? val1 : val0) + sg.start;
        // every wavefront takes the same whole number of rows of 64 records
        const uint32_t rows = (size + 64u * NW - 1u) / (64u * NW), r0 = (uint32_t)wv * rows * 64u + (uint32_t)lane;
        uint64_t lo[kSmallItems], hi[W == 2 ? kSmallItems : 1];
        double v[kSmallItems];
#pragma unroll
        for (int q = 0; q < kSmallItems; ++q) {
            const uint32_t r = r0 + (uint32_t)q * 64;
            const bool in = (uint32_t)q < rows && r < size;
            lo[q] = in ? klo[r] : 0ull;
            if (W == 2) hi[q] = in ? khi[r] : 0ull;
            v[q] = in ? val[r] : 0.0;
        }
        const uint32_t nb = min(max((2u * size + cap - 1u) / cap, 3u), (uint32_t)kSmallMax);
        const uint32_t m = min(min(size, 16u * nb), (uint32_t)kSmallSample);
        __syncthreads();  // the previous segment's LDS is read
        for (uint32_t i = tid; i < m; i += kSmallT) {
            const uint32_t j = (uint32_t)(((uint64_t)(2u * i + 1u) * size) / (2u * m));
            s_lo[i] = klo[j];
            if (W == 2) s_hi[i] = khi[j];
        }
        for (int i = tid; i < NW * kSmallMax; i += kSmallT) (&s_wcnt[0][0])[i] = 0u;
        if (tid < kSmallSample) s_rank[tid] = 0u;
        __syncthreads();
        // splitter j is the sample of rank q_j = j m / nb (ties by index): every
        // sample counts the ones below it and takes the splitters of its rank;
        // one equal to the splitter before it becomes the next larger key below
        // (the samples that one counts are shared out among the threads of the block)
        {
            uint32_t lg = 6;
            while ((1u << lg) < m) ++lg;
            const uint32_t i = (uint32_t)tid & ((1u << lg) - 1u), part = (uint32_t)tid >> lg;
            const uint32_t share = (m + ((uint32_t)kSmallT >> lg) - 1u) / ((uint32_t)kSmallT >> lg);
            if (i < m) {
                const uint64_t xl = s_lo[i], xh = W == 2 ? s_hi[i] : 0ull;
                const uint32_t j1 = min((part + 1u) * share, m);
                uint32_t rank = 0;
#pragma unroll 4
                for (uint32_t j = part * share; j < j1; ++j) {
                    const uint64_t yl = s_lo[j], yh = W == 2 ? s_hi[j] : 0ull;
                    const bool eq = yl == xl && (W == 1 || yh == xh);
                    rank += (key_less<W>(yl, yh, xl, xh) || (eq && j < i)) ? 1u : 0u;
                }
                atomicAdd(&s_rank[i], rank);
            }
        }
        __syncthreads();
        if ((uint32_t)tid < m) {
            const uint32_t rank = s_rank[tid];
            const uint32_t j = (rank * nb + m - 1u) / m;  // smallest j with j m / nb >= rank
            if (j > 0u && j < nb && (j * m) / nb == rank) {
                q_lo[j] = s_lo[tid];
                if (W == 2) q_hi[j] = s_hi[tid];
            }
        }
        __syncthreads();
        uint64_t ql = 0ull, qh = 0ull;
        bool one_key = false;
        if (tid > 0 && (uint32_t)tid < nb) {
            ql = q_lo[tid];
            qh = W == 2 ? q_hi[tid] : 0ull;
            if (tid > 1 && ql == q_lo[tid - 1] && (W == 1 || qh == q_hi[tid - 1])) {
                ++ql;
                if (W == 2 && ql == 0ull) ++qh;
            }
        }
        __syncthreads();
        if (tid < kSmallMax) {
            const bool used = tid > 0 && (uint32_t)tid < nb;
            q_lo[tid] = used ? ql : ~0ull;
            if (W == 2) q_hi[tid] = used ? qh : ~0ull;
        }
        __syncthreads();
        if (tid > 0 && (uint32_t)tid + 1u < nb) {
            const uint64_t nl = q_lo[tid] + 1ull;
            one_key = W == 1 ? q_lo[tid + 1] == nl
                             : (q_lo[tid + 1] == nl && q_hi[tid + 1] == q_hi[tid] + (nl == 0ull ? 1ull : 0ull));
        }
        // the range of a key is the number of splitters <= it; stable ranks by
        // wavefront, row and lane
        uint32_t dr[kSmallItems];  // range | rank << 8
        uint32_t nbits = 1;
        while ((1u << nbits) < nb) ++nbits;
#pragma unroll
        for (int q = 0; q < kSmallItems; ++q) {
            dr[q] = 0;
            if ((uint32_t)q >= rows) continue;  // uniform
            uint32_t d = 0;
            for (uint32_t step = 1u << (nbits - 1u); step; step >>= 1) {
                const uint32_t k = min(d + step, (uint32_t)kSmallMax - 1u);
                const bool le = W == 1 ? q_lo[k] <= lo[q] : (q_hi[k] < hi[q] || (q_hi[k] == hi[q] && q_lo[k] <= lo[q]));
                d += le ? step : 0u;
            }
            d = min(d, nb - 1u);
            const bool valid = r0 + (uint32_t)q * 64 < size;
            const uint64_t peers = wave_match(d, valid, (int)nbits);
            const uint32_t before = s_wcnt[wv][d];
            wave_sync();
            dr[q] = d | ((before + (uint32_t)__popcll(peers & lt)) << 8);
            if (valid && (peers & lt) == 0ull) s_wcnt[wv][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
            wave_sync();
        }
        __syncthreads();
        uint32_t kind = 0;  // wavefront 0, lane d: a final that starts at range d
        Seg c{0u, 0u, 0u};
        if (wv == 0) {
            // lane d: the bases of range d
            uint32_t run = 0;
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const uint32_t x = s_wcnt[i][lane];
                s_wcnt[i][lane] = (uint16_t)run;
                run += x;
            }
            const uint32_t e = wave_incl_scan(run) - run;
#pragma unroll
            for (int i = 0; i < NW; ++i) s_wcnt[i][lane] = (uint16_t)(s_wcnt[i][lane] + e);
            // Greedy groups of consecutive ranges, of at most cap records (a larger
            // range is a group of its own), one after the other: two to four for
            // most segments.
            const uint32_t end = e + run;
            for (uint32_t a = 0; a < nb;) {  // uniform
                const uint32_t start = (uint32_t)__builtin_amdgcn_readlane((int)e, (int)a);
                const uint64_t in = __ballot((uint32_t)lane >= a && (uint32_t)lane < nb && end - start <= cap);
                const uint32_t last = in ? 63u - (uint32_t)__clzll((long long)in) : a;
                if ((uint32_t)lane == a) {
                    const uint32_t gs = (uint32_t)__builtin_amdgcn_readlane((int)end, (int)last) - start;
                    if (gs > 0u) kind = gs <= cap || one_key ? 1u : 3u;
                    c = Seg{sg.start + start, gs, make_meta(buf, gs > cap && one_key)};
                }
                a = last + 1u;
            }
        }
        __syncthreads();
        // records to LDS in range order
#pragma unroll
        for (int q = 0; q < kSmallItems; ++q) {
            const uint32_t r = r0 + (uint32_t)q * 64;
            if ((uint32_t)q < rows && r < size) {
                const uint32_t p = min((uint32_t)s_wcnt[wv][dr[q] & 0xFFu] + (dr[q] >> 8), (uint32_t)kTileN - 1u);
                dr[q] = p;
                s_lo[p] = lo[q];
                if (W == 2) s_hi[p] = hi[q];
                else s_val[p] = v[q];
            }
        }
        __syncthreads();
        for (uint32_t i = tid; i < size; i += kSmallT) {
            klo[i] = s_lo[i];
            if (W == 2) khi[i] = s_hi[i];
            else val[i] = s_val[i];
        }
        if (W == 2) {
            __syncthreads();
            double *sv = reinterpret_cast<double *>(s_lo);
#pragma unroll
            for (int q = 0; q < kSmallItems; ++q)
                if ((uint32_t)q < rows && r0 + (uint32_t)q * 64 < size) sv[dr[q]] = v[q];
            __syncthreads();
            for (uint32_t i = tid; i < size; i += kSmallT) val[i] = sv[i];
        }
        if (wv == 0) {
            const uint64_t again = __ballot(kind == 3u);
            if (kind == 3u) s_left[left + (uint32_t)__popcll(again & lt)] = c;
            if (lane == 0) s_nleft = left + (uint32_t)__popcll(again);
            append_segs(lists, kind == 3u ? 0u : kind, c);
        }
        __syncthreads();  // the records, and what is left, are written
        left = s_nleft;
    }
}

// ---------------------------------------------------------------- finish
struct FinishArgs {
    const Seg *finals;
    const uint64_t *klo[2], *khi[2];
    const double *val[2];
    int n;
    const double *jk;           // J, J-K (n^2 each), h_pp (n)
    SpinTables st;              // E(alpha), E(beta) by string rank (optional)
    const uint64_t *thr;        // candidates with abs_order(A) below *thr cannot enter the top k (optional)
    double ecore, E0, eps;      // eps > 0: keep a pair only if |H_ai C_i / (E0 - H_aa)| > eps
    uint64_t *clo, *chi;        // slot arrays (batch positions)
    double *cnum, *cscore;
    unsigned long long *mask;   // a bit per slot: holds a candidate (cleared by the caller)
    uint32_t *tcnt;             // candidates per tile of kSlotTile slots (cleared by the caller)
    uint32_t nfinal;
    const uint32_t *dn_final;   // device: final segments (nfinal is then a bound; optional)
    int part;                   // kAll, or the final segments of a pilot, or all but those
    uint32_t *runs;             // distinct targets are added to it (optional)
    PsiSet psi;                 // input determinants (exclusion)
    int na, nb;
    int stage_x;                // some strings have no table: J-K (triangle) and h_pp are staged in LDS
    uint32_t tab_bytes;         // LDS of the staged tables
    uint32_t wave_bytes;        // LDS of one wavefront
    uint32_t amax;              // alpha strings one wavefront caches (a power of two)
    const double *bounds;       // k_diag_bounds: with a threshold, targets are rejected by a bound (optional)
    uint32_t qcap;              // targets that a wavefront queues
};
constexpr uint32_t kMinRanks = 256;

constexpr uint32_t kSlotTile = 4096;  // slots per collect tile
enum { kAll = 0, kPilotPart = 1, kRestPart = 2 };
// A pilot takes every 16th final segment: of more, fewer are left to gain from;
// fewer bound the k-th |A| less tightly (every 8th, 16th and 32nd, ms: 16e20o of
// 2^27 pairs, k = P / 256 6.64, 6.76, 6.93, k = P / 8192 6.17, 6.08, 6.08; 24e30o
// of 2^28 pairs, k = P / 1024 20.3, 20.1, 20.2).
constexpr uint32_t kPilot = 16;

// final segments of a part, and the i-th of them
__host__ __device__ __forceinline__ uint32_t part_count(uint32_t nf, int part)
{
    const uint32_t np = (nf + kPilot - 1u) / kPilot;
    return part == kAll ? nf : (part == kPilotPart ? np : nf - np);
}
__device__ __forceinline__ uint32_t part_index(uint32_t i, int part)
{
    return part == kAll ? i : (part == kPilotPart ? i * kPilot : i + i / (kPilot - 1u) + 1u);
}

// The tables a finish reads and the electron counts.  The counts are the same
// for every string of a search, so that the walks over a string's set bits
// below run a uniform number of steps.  Each table lies in one known memory (a
// pointer that may be either makes every access a flat one): X, h_pp and the
// binomials in LDS, J there too when JL.
template <bool JL>
struct Diag {
    // J (JL: its lower triangle row by row, else n^2), X = J - K (its strict
    // upper triangle row by row), h_pp
    const double *J, *X, *hd;
    const double *e[2];        // E(alpha), E(beta) by string rank, or null
    uint32_t last[2];          // the largest rank
    const uint32_t *binom;
    int n, ne[2];
};

// index of the lowest set bit; n - 1 for an empty word (a string with fewer
// electrons than it should have, from inputs that fail validation, must not
// send an access out of its table)
template <typename M>
__device__ __forceinline__ uint32_t low_orb(M m, int n)
{
    return min((uint32_t)__builtin_ctzg(m, (int)(8 * sizeof(M))), (uint32_t)n - 1u);
}

// load(i, orbital) for the ne lowest set bits of m, ascending, then add of what
// it returned, in the same order; the loads of four are in flight at a time
template <typename M, typename L, typename A>
__device__ __forceinline__ void for_bits(M m, int n, int ne, L load, A add)
{
    int i = 0;
    for (; i + 4 <= ne; i += 4) {
        decltype(load(0, 0u)) x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[k] = load(i + k, low_orb(m, n));
            m &= m - 1;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) add(x[k]);
    }
    if (i < ne) {  // one to three more
        decltype(load(0, 0u)) x[3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k == 0 || i + k < ne) {
                x[k] = load(i + k, low_orb(m, n));
                m &= m - 1;
            }
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k == 0 || i + k < ne) add(x[k]);
    }
}

// c_q(alpha) = sum over p in alpha of J_pq, p ascending; alpha is uniform
template <bool JL, typename M>
__device__ __forceinline__ double column_sum(const Diag<JL> &D, M alpha, uint32_t q)
{
    const uint32_t n = (uint32_t)D.n, qb = q * (q + 1u) / 2u;
    double c = 0.0;
    for_bits(alpha, D.n, D.ne[0],
             [&](int, uint32_t p) { return D.J[JL ? (q >= p ? qb + p : p * (p + 1u) / 2u + q) : p * n + q]; },
             [&](double x) { c = c + x; });
    return c;
}

// E(s) in the order of spin_energy: h_pp ascending, then the pairs p < q row by row
template <bool JL, typename M>
__device__ __forceinline__ double spin_energy_u(const Diag<JL> &D, int ne, M s)
{
    double e = 0.0;
    for_bits(s, D.n, ne, [&](int, uint32_t q) { return D.hd[q]; }, [&](double x) { e = e + x; });
    for (int i = 0; i + 1 < ne; ++i) {
        const uint32_t p = low_orb(s, D.n);
        s &= s - 1;
        // the strict upper triangle's row p starts at p n - p (p + 3) / 2 - 1 for column 0
        const int row = (int)(p * (uint32_t)D.n) - (int)(p * (p + 3u) / 2u + 1u);
        for_bits(s, D.n, ne - 1 - i, [&](int, uint32_t q) { return D.X[max(row + (int)q, 0)]; }, [&](double x) { e = e + x; });
    }
    return e;
}

// rank of the string in the combinatorial number system
template <bool JL, typename M>
__device__ __forceinline__ uint32_t spin_rank_u(const Diag<JL> &D, int ne, M s)
{
    uint32_t r = 0;
    for_bits(s, D.n, ne, [&](int i, uint32_t q) { return D.binom[(i + 1) * (D.n + 1) + (int)q]; }, [&](uint32_t x) { r += x; });
    return r;
}

// E of one spin string (0 = alpha, 1 = beta): looked up when tabulated
template <bool JL, typename M>
__device__ __forceinline__ double spin_e(const Diag<JL> &D, int spin, M s)
{
    return D.e[spin] ? D.e[spin][min(spin_rank_u(D, D.ne[spin], s), D.last[spin])] : spin_energy_u(D, D.ne[spin], s);
}

// H_aa = ((ecore + E(alpha)) + E(beta)) + E(alpha, beta)
template <bool JL, typename M>
__device__ __forceinline__ double diag_tab(const Diag<JL> &D, double ecore, M a, M b)
{
    double cross = 0.0;
    for (M m = b; m; m &= m - 1) cross = cross + column_sum(D, a, low_orb(m, D.n));
    return ((ecore + spin_e(D, 0, a)) + spin_e(D, 1, b)) + cross;
}

// The key as one 2n-bit value (alpha << n) | beta.  Bits [o, o + 32) of it:
template <int W>
__device__ __forceinline__ uint32_t key_window(uint64_t lo, uint64_t hi, int n, int o)
{
    if (W == 1) return o < 64 ? (uint32_t)(lo >> o) : 0u;
    if (o >= n) return (uint32_t)(hi >> (o - n));
    uint64_t x = lo >> o;
    if (n - o < 32) x |= hi << (n - o);
    return (uint32_t)x;
}

// OR a 32-bit window c into bits [o, o + 32) of the key (bits past 2n are 0 in c)
template <int W>
__device__ __forceinline__ void key_put(uint32_t c, int o, int n, uint64_t &lo, uint64_t &hi)
{
    if (W == 1) {
        lo |= (uint64_t)c << o;
        return;
    }
    if (o >= n) {
        hi |= (uint64_t)c << (o - n);
        return;
    }
    const uint64_t nmask = (n == 64) ? ~0ull : ((1ull << n) - 1ull);
    lo |= ((uint64_t)c << o) & nmask;
    if (n - o < 32) hi |= (uint64_t)c >> (n - o);
}

// f(source shift, width mask, destination shift) for every run of set bits of
// m, lowest first; returns the number of set bits.  m is uniform, so the walk
// is scalar work.
template <typename F>
__device__ __forceinline__ int for_bit_runs(uint64_t m, int at, F f)
{
    while (m) {
        const int s = __builtin_ctzll(m);
        const uint64_t t = ~(m >> s);
        const int len = t ? __builtin_ctzll(t) : 64 - s;
        const uint64_t wm = len >= 64 ? ~0ull : (1ull << len) - 1ull;
        f(s, wm, at);
        at += len;
        m &= ~(wm << s);
    }
    return at;
}

// lowest varying key bit (-1: none) and one past the highest
template <int W>
__device__ __forceinline__ int key_low(uint64_t vlo, uint64_t vhi, int n)
{
    if (vlo) return __builtin_ctzll(vlo);
    if (W == 2 && vhi) return n + __builtin_ctzll(vhi);
    return -1;
}
template <int W>
__device__ __forceinline__ int key_top(uint64_t vlo, uint64_t vhi, int n)
{
    if (W == 2 && vhi) return n + 64 - __builtin_clzll(vhi);
    if (vlo) return 64 - __builtin_clzll(vlo);
    return 0;
}

// LDS share of one wavefront: 64 * IT records.  The sort permutes 16-bit
// record indices (ix), ranking them by a 32-bit window of each key that holds
// its varying bits (ck); the values stay in registers meanwhile, so that their
// array holds the digit counters (two 16-bit counters a word).  After the sort
// ix holds the run heads (position, and bit 15 where the alpha string
// changes) and ck each run's window, or its record where the keys have to be
// read back.  Behind it lies the alpha cache: c_q(alpha) of amax strings.
template <int IT>
struct WaveLds {
    static constexpr int CAP = 64 * IT;
    static constexpr int DIGITS = 256 * IT;  // counters that fit over the values
    uint32_t ck[CAP];
    uint16_t ix[CAP + 8];
    union {
        double val[CAP + 2];  // val[CAP] stays 0: what a lane past the end of its run adds
        uint32_t cnt[DIGITS / 2];
    };
    static_assert(sizeof(cnt) <= sizeof(double) * CAP && sizeof(val) > sizeof(double) * CAP,
                  "the counters lie below the zero, and the zero inside the values");
};
template <int IT>
constexpr int digit_bits()
{
    return IT == 8 ? 11 : 10;
}

// exclusive scan of N counter words per lane, in place: a word's two 16-bit
// counters become the bases of their digits
template <int N>
__device__ __forceinline__ void scan_counters(uint32_t *cnt)
{
    uint32_t *c = cnt + (threadIdx.x & 63) * N;
    uint32_t x[N], mine = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = c[i];
#pragma unroll
    for (int i = 0; i < N; ++i) mine += (x[i] & 0xFFFFu) + (x[i] >> 16);
    uint32_t base = wave_incl_scan(mine) - mine;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint32_t lo = base + (x[i] & 0xFFFFu);
        c[i] = base | (lo << 16);
        base = lo + (x[i] >> 16);
    }
}

// The values [p0, p1) added in order: eight or four whole ones at a time, then
// the last three at most (past the end +0.0, which leaves the sum's bits alone:
// it starts at +0.0 and so never is -0.0).  Eight at a time with a bound check
// on each took three times the instructions.
template <int IT>
__device__ __forceinline__ double run_sum(const WaveLds<IT> &S, uint32_t p0, uint32_t p1)
{
    double sum = 0.0;
    uint32_t j = p0;
    for (; j + 8 <= p1; j += 8) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = S.val[j + (uint32_t)k];
#pragma unroll
        for (int k = 0; k < 8; ++k) sum = sum + v[k];
    }
    if (j + 4 <= p1) {
        double v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = S.val[j + (uint32_t)k];
#pragma unroll
        for (int k = 0; k < 4; ++k) sum = sum + v[k];
        j += 4;
    }
    double v[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] = S.val[j + (uint32_t)k < p1 ? j + (uint32_t)k : (uint32_t)WaveLds<IT>::CAP];
#pragma unroll
    for (int k = 0; k < 3; ++k) sum = sum + v[k];
    return sum;
}

// marks the slots [start, start + written) and counts them in their tiles
__device__ __forceinline__ void mark_slots(const FinishArgs &f, uint32_t start, uint32_t written)
{
    if (written == 0) return;
    const int lane = threadIdx.x & 63;
    const uint32_t end = start + written, w0 = start >> 6, w1 = (end - 1u) >> 6;
    for (uint32_t w = w0 + (uint32_t)lane; w <= w1; w += 64) {
        unsigned long long m = ~0ull;
        if (w == w0) m &= ~0ull << (start & 63u);
        if (w == w1) m &= ~0ull >> (63u - ((end - 1u) & 63u));
        atomicOr(&f.mask[w], m);
    }
    const uint32_t t0 = start / kSlotTile, t1 = (end - 1u) / kSlotTile;
    if (lane == 0) {
        const uint32_t first = min(end, (t0 + 1u) * kSlotTile) - start;
        atomicAdd(&f.tcnt[t0], first);
        if (t1 != t0) atomicAdd(&f.tcnt[t1], written - first);  // a segment holds at most 512 candidates
    }
}

// a segment of one key with more records than a wavefront's share: summed in
// record order, 64 * IT values at a time staged in LDS
template <int W, int IT, bool JL>
__device__ __forceinline__ void finish_single(const FinishArgs &f, const Diag<JL> &D, WaveLds<IT> &S, const Seg &sg)
{
    constexpr int CAP = WaveLds<IT>::CAP;
    const int n = f.n, lane = threadIdx.x & 63;
    const uint64_t nmask = (n == 64) ? ~0ull : ((1ull << n) - 1ull);
    const uint64_t lo = f.klo[seg_buf(sg)][sg.start], hi = W == 2 ? f.khi[seg_buf(sg)][sg.start] : 0ull;
    if (psi_contains(f.psi, lo, hi)) return;
    const double *gv = f.val[seg_buf(sg)] + sg.start;
    const uint64_t a = W == 1 ? (lo >> n) : hi, b = W == 1 ? (lo & nmask) : lo;
    const double den = f.E0 - (n <= 32 ? diag_tab<JL, uint32_t>(D, f.ecore, (uint32_t)a, (uint32_t)b)
                                       : diag_tab<JL, uint64_t>(D, f.ecore, a, b));
    double sum = 0.0;
    bool kept = false;
    for (uint32_t r0 = 0; r0 < sg.size; r0 += CAP) {
        wave_sync();
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            const uint32_t r = r0 + (uint32_t)(k * 64 + lane);
            double v = r < sg.size ? gv[r] : 0.0;
            bool in = r < sg.size;
            if (f.eps > 0.0) in = in && fabs(v / den) > f.eps;
            // a dropped value adds +0.0, which leaves the sum's bits alone (it
            // starts at +0.0 and so never is -0.0)
            S.val[k * 64 + lane] = in ? v : 0.0;
            kept |= __ballot(in) != 0ull;
        }
        wave_sync();
        const uint32_t m = min(sg.size - r0, (uint32_t)CAP);
        for (uint32_t j = 0; j < m; j += 16) {
            double v[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) v[k] = S.val[j + k];  // past the end: zeros
#pragma unroll
            for (int k = 0; k < 16; ++k) sum = sum + v[k];
        }
    }
    const double score = sum / den;
    if (!kept || (f.thr && abs_order(score) < *f.thr)) return;
    if (lane == 0) {
        f.clo[sg.start] = lo;
        if (W == 2) f.chi[sg.start] = hi;
        if (f.cnum) f.cnum[sg.start] = sum;
        f.cscore[sg.start] = score;
    }
    mark_slots(f, sg.start, 1u);
}

// Targets whose sum a bound on the diagonal element did not reject: a
// wavefront's own queue in LDS, evaluated 64 at a time.
template <int W>
struct Queue {
    uint64_t *lo, *hi;
    double *sum;
    uint32_t *slot;
    uint32_t n;
};
template <int W>
constexpr size_t queue_entry()
{
    return 8 * W + 12;
}

// the last (at most 64) targets of the queue: diagonal, score, exclusion, slot
template <int W, bool JL>
__device__ __forceinline__ void finish_queued(const FinishArgs &f, const Diag<JL> &D, Queue<W> &Q, uint64_t thr)
{
    const uint32_t lane = threadIdx.x & 63, cnt = min(Q.n, 64u);
    wave_sync();
    Q.n -= cnt;
    if (lane < cnt) {
        const uint32_t i = Q.n + lane;
        const uint64_t lo = Q.lo[i], hi = W == 2 ? Q.hi[i] : 0ull;
        const double sum = Q.sum[i];
        const uint32_t at = Q.slot[i];
        const int n = f.n;
        const uint64_t nmask = (n == 64) ? ~0ull : ((1ull << n) - 1ull);
        const uint64_t a = W == 1 ? (lo >> n) : hi, b = W == 1 ? (lo & nmask) : lo;
        const double den = f.E0 - (n <= 32 ? diag_tab<JL, uint32_t>(D, f.ecore, (uint32_t)a, (uint32_t)b)
                                           : diag_tab<JL, uint64_t>(D, f.ecore, a, b));
        const double score = sum / den;
        if (abs_order(score) >= thr && !psi_contains(f.psi, lo, hi)) {
            f.clo[at] = lo;
            if (W == 2) f.chi[at] = hi;
            if (f.cnum) f.cnum[at] = sum;
            f.cscore[at] = score;
            atomicOr(&f.mask[at >> 6], 1ull << (at & 63u));
            atomicAdd(&f.tcnt[at / kSlotTile], 1u);
        }
    }
    wave_sync();
}

__device__ __forceinline__ double readlane_f64(double x, int l)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    return __longlong_as_double((long long)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l) |
                                            ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l) << 32)));
}

// sum over the lanes, by register moves
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_from_f64(double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    return __longlong_as_double((long long)((uint64_t)dpp_from<CTRL, ROWS>((uint32_t)u) |
                                            ((uint64_t)dpp_from<CTRL, ROWS>((uint32_t)(u >> 32)) << 32)));
}
__device__ __forceinline__ double wave_sum(double x)
{
    x = x + dpp_from_f64<0x111, 0xF>(x);
    x = x + dpp_from_f64<0x112, 0xF>(x);
    x = x + dpp_from_f64<0x114, 0xF>(x);
    x = x + dpp_from_f64<0x118, 0xF>(x);
    x = x + dpp_from_f64<0x142, 0xA>(x);
    x = x + dpp_from_f64<0x143, 0xC>(x);
    return readlane_f64(x, 63);
}

// the smaller one; NaN if either is
__device__ __forceinline__ double min_nan(double x, double m)
{
    return m != m || m <= x ? m : x;
}

// A lower bound of the sum of nb of the lanes' v, all of the lanes in `fixed`
// among them and the others from `free`: for every level l, the sum of the
// nfree smallest v is at least nfree l + sum over free of min(v - l, 0), and
// equal to it where l is the nfree-th smallest.  l follows the strings that
// come by; it only decides how tight the bound is.
__device__ __forceinline__ double least_columns(double v, uint64_t fixed, uint64_t free, int nb, double step, double &level)
{
    const int lane = threadIdx.x & 63;
    const int nfree = nb - (int)__popcll(fixed);
    const bool below = !(v >= level) && ((free >> lane) & 1ull);
    const double sum = wave_sum(((fixed >> lane) & 1ull) ? v : (below ? v - level : 0.0)) + (double)nfree * level;
    level = level + (double)(nfree - (int)__popcll(__ballot(below))) * step;
    return sum;
}

// E(s) of one uniform string from its table, lane q the orbital q
template <bool JL, typename M>
__device__ __forceinline__ double spin_e_lanes(const Diag<JL> &D, int spin, M s)
{
    const uint32_t lane = threadIdx.x & 63, n = (uint32_t)D.n;
    const uint64_t below = (uint64_t)s & ((1ull << lane) - 1ull);
    uint32_t r = 0;
    if (lane < n && (((uint64_t)s >> lane) & 1ull))
        r = D.binom[min((uint32_t)__popcll(below) + 1u, (uint32_t)D.ne[spin]) * (n + 1u) + lane];
    r = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(r), 63);
    return D.e[spin][min(r, D.last[spin])];
}

// one final segment of at most 64 * IT records, by one wavefront; its distinct keys
template <int W, int IT, bool JL>
__device__ __forceinline__ uint32_t finish_segment(const FinishArgs &f, const Diag<JL> &D, WaveLds<IT> &S, double *acache,
                                               const Seg &sg, uint64_t thr, bool prune, double &level, uint32_t &queued,
                                               Queue<W> &Q)
{
    using M = std::conditional_t<W == 1, uint32_t, uint64_t>;  // a spin string
    constexpr int CAP = WaveLds<IT>::CAP;
    constexpr int DB = digit_bits<IT>();
    static_assert(1 << DB == WaveLds<IT>::DIGITS, "the digit counters lie over the values");
    const int n = f.n;
    const int lane = threadIdx.x & 63;
    const uint64_t lt = (1ull << lane) - 1ull;
    const uint32_t size = sg.size;
    const uint64_t nmask = (n == 64) ? ~0ull : ((1ull << n) - 1ull);
    const uint64_t *gk = f.klo[seg_buf(sg)] + sg.start;
    const uint64_t *gh = f.khi[seg_buf(sg)] + sg.start;
    const double *gv = f.val[seg_buf(sg)] + sg.start;

    // record r = k * 64 + lane in registers; the bits that vary inside the
    // segment are those in which some key differs from the first
    uint64_t rk[IT], rh[W == 2 ? IT : 1];
    double rv[IT];
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const uint32_t r = (uint32_t)(k * 64 + lane);
        rk[k] = r < size ? gk[r] : 0ull;
        if (W == 2) rh[k] = r < size ? gh[r] : 0ull;
        rv[k] = r < size ? gv[r] : 0.0;
    }
    const uint64_t k0lo = uniform64(rk[0]), k0hi = W == 2 ? uniform64(rh[0]) : 0ull;
    uint64_t var_lo = 0ull, var_hi = 0ull;
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const uint32_t r = (uint32_t)(k * 64 + lane);
        var_lo |= r < size ? rk[k] ^ k0lo : 0ull;
        if (W == 2) var_hi |= r < size ? rh[k] ^ k0hi : 0ull;
    }
    var_lo = wave_or64(var_lo);
    if (W == 2) var_hi = wave_or64(var_hi);
    const uint64_t and_lo = k0lo & ~var_lo, and_hi = k0hi & ~var_hi;
    const int low = key_low<W>(var_lo, var_hi, n);
    const int span = low < 0 ? 0 : key_top<W>(var_lo, var_hi, n) - low;
    const int nvar = __popcll(var_lo) + (W == 2 ? __popcll(var_hi) : 0);
    // The window: the key's bits [low, low + 32) where the span fits, else its
    // varying bits packed together; more than 32 varying bits take several
    // windows of the span, and the keys are read back from memory (cache).
    const bool packed = span > 32 && nvar <= 32;
    const bool multi = nvar > 32;
    const int bits = packed ? nvar : span;
    // digits of equal width, at most DB bits: as few passes as that allows
    const int npass = (bits + DB - 1) / DB;
    const int dw = npass ? (bits + npass - 1) / npass : 1;
    const int per_win = multi ? 32 / dw : max(npass, 1);
    // window bits at or above this one belong to the alpha string
    const int aw = packed ? __popcll(W == 1 ? (var_lo & nmask) : var_lo) : n - low;

    if (packed) {
        uint32_t w[IT];
#pragma unroll
        for (int k = 0; k < IT; ++k) w[k] = 0u;
        const int d = for_bit_runs(var_lo, 0, [&](int s, uint64_t m, int to) {
#pragma unroll
            for (int k = 0; k < IT; ++k) w[k] |= (uint32_t)((rk[k] >> s) & m) << to;
        });
        if (W == 2)
            (void)for_bit_runs(var_hi, d, [&](int s, uint64_t m, int to) {
#pragma unroll
                for (int k = 0; k < IT; ++k) w[k] |= (uint32_t)((rh[k] >> s) & m) << to;
            });
#pragma unroll
        for (int k = 0; k < IT; ++k) S.ck[k * 64 + lane] = w[k];
    } else if (!multi && npass) {
#pragma unroll
        for (int k = 0; k < IT; ++k) S.ck[k * 64 + lane] = key_window<W>(rk[k], W == 2 ? rh[k] : 0ull, n, low);
    }
    uint32_t c[IT], rec[IT];  // after the sort: window and record at position q * 64 + lane
    uint32_t hd = 0;          // bit q: run head there, bit 16 + q: alpha head
    // Stable LSD radix sort of the record indices.  A record's rank among equal
    // digits is the counter value that its LDS atomic returns: one instruction
    // a row of 64 records, where a ballot match takes four a digit bit (which
    // made 8-bit digits the widest that paid).  The order in which one
    // instruction's lanes reach a counter is not specified, so nothing is taken
    // on trust: the run-head pass compares every neighbouring pair, and a
    // segment found out of (key, record) order is sorted again from the start
    // with ballot ranks, whose order is defined.
    for (int attempt = 0;; ++attempt) {
        const bool ballots = attempt > 0;  // uniform
        bool first = true;
        wave_sync();
        if (npass == 0) {
            // one key: no pass runs, the order is the identity
#pragma unroll
            for (int k = 0; k < IT; ++k) S.ix[k * 64 + lane] = (uint16_t)(k * 64 + lane);
        }
        for (int p0 = 0; p0 < npass; p0 += per_win) {
            if (multi) {
                wave_sync();
#pragma unroll
                for (int k = 0; k < IT; ++k) {
                    const uint32_t r = (uint32_t)(k * 64 + lane);
                    if (r < size) S.ck[r] = key_window<W>(gk[r], W == 2 ? gh[r] : 0ull, n, low + p0 * dw);
                }
                wave_sync();
            }
            for (int p = p0; p < min(p0 + per_win, npass); ++p) {
                const int sh = (p - p0) * dw;
                const uint32_t dmask = (1u << dw) - 1u;
                const uint32_t words = max(1u << (dw - 1), 64u);
                for (uint32_t i = (uint32_t)lane; i < words; i += 64) S.cnt[i] = 0u;
                uint32_t item[IT], dg[IT];  // record | rank << 16, digit
#pragma unroll
                for (int q = 0; q < IT; ++q)
                    item[q] = first ? (uint32_t)(q * 64 + lane) : (uint32_t)S.ix[q * 64 + lane] & (uint32_t)(CAP - 1);
#pragma unroll
                for (int q = 0; q < IT; ++q) dg[q] = (S.ck[item[q]] >> sh) & dmask;
                first = false;
                wave_sync();
                if (!ballots) {
#pragma unroll
                    for (int q = 0; q < IT; ++q) {
                        const uint32_t hs = (dg[q] & 1u) * 16u;
                        if ((uint32_t)(q * 64 + lane) < size)
                            item[q] |= ((atomicAdd(&S.cnt[dg[q] >> 1], 1u << hs) >> hs) & 0xFFFFu) << 16;
                        wave_sync();
                    }
                } else {
                    uint16_t *c16 = reinterpret_cast<uint16_t *>(&S.cnt[0]);
#pragma unroll
                    for (int q = 0; q < IT; ++q) {
                        const bool valid = (uint32_t)(q * 64 + lane) < size;
                        const uint64_t peers = wave_match(dg[q], valid, dw);
                        const uint32_t before = c16[dg[q]];
                        wave_sync();
                        if (valid) {
                            item[q] |= (before + (uint32_t)__popcll(peers & lt)) << 16;
                            if ((peers & lt) == 0ull) c16[dg[q]] = (uint16_t)(before + (uint32_t)__popcll(peers));
                        }
                        wave_sync();
                    }
                }
                wave_sync();
                switch (words) {  // uniform
                case 64: scan_counters<1>(S.cnt); break;
                case 128: scan_counters<2>(S.cnt); break;
                case 256: scan_counters<4>(S.cnt); break;
                case 512: scan_counters<8>(S.cnt); break;
                default: if (IT >= 8) scan_counters<IT >= 8 ? 16 : 1>(S.cnt); break;
                }
                wave_sync();
                {
                    const uint16_t *c16 = reinterpret_cast<const uint16_t *>(&S.cnt[0]);
#pragma unroll
                    for (int q = 0; q < IT; ++q)
                        if ((uint32_t)(q * 64 + lane) < size) {
                            const uint32_t d = min((uint32_t)c16[dg[q]] + (item[q] >> 16), (uint32_t)CAP - 1u);
                            S.ix[d] = (uint16_t)(item[q] & 0xFFFFu);
                        }
                }
                wave_sync();
            }
        }
        // values to LDS in record order; then runs of equal keys and the alpha
        // strings among them, row by row of the sorted positions: the position
        // before a lane's is the lane before's, or the last of the row before
#pragma unroll
        for (int k = 0; k < IT; ++k) S.val[k * 64 + lane] = rv[k];
        wave_sync();
#pragma unroll
        for (int q = 0; q < IT; ++q) rec[q] = (uint32_t)S.ix[q * 64 + lane] & (uint32_t)(CAP - 1);
        if (!multi) {
#pragma unroll
            for (int q = 0; q < IT; ++q) c[q] = npass ? S.ck[rec[q]] : 0u;
        } else {
#pragma unroll
            for (int q = 0; q < IT; ++q) c[q] = rec[q];  // a run's key is read back through its record
        }
        hd = 0;
        bool bad = false;
        uint32_t pc = 0, pr = 0;  // last lane of the row before
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            if ((uint32_t)q * 64 >= size) break;  // uniform
            const uint32_t j = (uint32_t)(q * 64 + lane);
            const uint32_t bc = lane_before(c[q], pc), br = lane_before(rec[q], pr);
            pc = (uint32_t)__builtin_amdgcn_readlane((int)c[q], 63);
            pr = (uint32_t)__builtin_amdgcn_readlane((int)rec[q], 63);
            bool head, ahead, order;  // order: out of (key, record) order
            if (!multi) {
                const uint32_t x = c[q] ^ bc;
                head = x != 0u;
                ahead = aw < 32 && (x >> max(aw, 0)) != 0u;
                order = head ? c[q] < bc : rec[q] <= br;
            } else {
                const bool in = j > 0u && j < size;
                const uint64_t klo = in ? gk[rec[q]] : 0ull, khi = W == 2 && in ? gh[rec[q]] : 0ull;
                const uint64_t plo = in ? gk[br] : 0ull, phi = W == 2 && in ? gh[br] : 0ull;
                head = klo != plo || khi != phi;
                ahead = W == 1 ? (klo >> n) != (plo >> n) : khi != phi;
                order = head ? key_less<W>(klo, khi, plo, phi) : rec[q] <= br;
            }
            if (j < size) {
                bad |= j != 0u && order;
                hd |= (j == 0u || head ? 1u : 0u) << q;
                hd |= (j == 0u || ahead ? 1u : 0u) << (16 + q);
            }
        }
        if (ballots || __ballot(bad) == 0ull) break;
    }
    uint32_t nruns = 0;
    {
        double gval[IT];
#pragma unroll
        for (int q = 0; q < IT; ++q) gval[q] = S.val[rec[q]];
        wave_sync();  // every lane holds its values, windows and records
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            if ((uint32_t)q * 64 >= size) break;  // uniform
            S.val[q * 64 + lane] = gval[q];
            const bool head = (hd >> q) & 1u;
            const uint64_t m = __ballot(head);
            if (head) {
                const uint32_t at = nruns + (uint32_t)__popcll(m & lt);
                S.ix[at] = (uint16_t)((uint32_t)(q * 64 + lane) | (((hd >> (16 + q)) & 1u) << 15));
                S.ck[at] = c[q];
            }
            nruns += (uint32_t)__popcll(m);
        }
        if (lane == 0) S.ix[nruns] = (uint16_t)size;
        wave_sync();
    }
    const auto run_key = [&](uint32_t w, uint64_t &lo, uint64_t &hi) {
        if (multi) {
            lo = gk[w];
            hi = W == 2 ? gh[w] : 0ull;
        } else if (packed) {
            const int d = for_bit_runs(var_lo, 0, [&](int s, uint64_t m, int to) { lo |= ((uint64_t)(w >> to) & m) << s; });
            if (W == 2)
                (void)for_bit_runs(var_hi, d, [&](int s, uint64_t m, int to) { hi |= ((uint64_t)(w >> to) & m) << s; });
        } else if (npass) {
            key_put<W>(w, low, n, lo, hi);
        }
    };
    // a score is below thr for certain where |N| < tlow |E0 - H_aa| (the margin
    // covers the roundings of both sides; no test for a bound that is not finite)
    const double tlow = thr < 0x7FE0000000000000ull ? __longlong_as_double((long long)thr) * (1.0 - 0x1p-40) : 0.0;
    const uint32_t amask = f.amax - 1u;
    if (prune) {
        // Sums first; a run goes to the queue unless |N| < tlow times a bound of
        // its denominator: E(alpha), a least E(beta) and the least sum of columns
        // that the segment's beta strings can have, less a margin far above what
        // the roundings of either side can amount to.
        const uint64_t bfix = W == 1 ? (and_lo & nmask) : and_lo, bfree = W == 1 ? (var_lo & nmask) : var_lo;
        const double margin = f.bounds[0], emin = f.bounds[1], step = f.bounds[3];
        uint32_t nq = 0;
        double lb_last = 0.0, lb_carry = 0.0;  // of the last alpha string so far, and at the batch's start
        for (uint32_t base = 0; base < nruns; base += 64) {
            const uint32_t u = base + (uint32_t)lane;
            const bool act = u < nruns;
            double sum = 0.0, lb = 0.0;
            uint32_t w = 0;
            uint64_t lo = and_lo, hi = and_hi;
            bool ahead = false;
            if (act) {
                const uint32_t h0 = S.ix[u], p0 = h0 & 0x7FFFu, p1 = (uint32_t)S.ix[u + 1] & 0x7FFFu;
                ahead = (h0 >> 15) != 0u;
                w = S.ck[u];
                sum = run_sum(S, p0, p1);
                if (ahead) run_key(w, lo, hi);
            }
            const M a = (M)(W == 1 ? (lo >> n) : hi);
            const uint64_t heads = __ballot(ahead);
            for (uint64_t fresh = heads; fresh; fresh &= fresh - 1ull) {
                const int hl = __ffsll((long long)fresh) - 1;
                M as = (M)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)a, hl);
                if (W == 2) as |= (M)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)a >> 32), hl) << 32);
                const double e = spin_e_lanes(D, 0, as);
                const double cq = lane < n ? column_sum(D, as, (uint32_t)lane) : 0.0;
                const double x = least_columns(cq, bfix, bfree, D.ne[1], step, level);
                const double b = (((f.ecore + e) + emin) + x - f.E0) - margin;
                if (lane >= hl) lb = b;
                lb_last = b;
            }
            if (heads == 0ull || lane < __ffsll((long long)heads) - 1) lb = lb_carry;
            lb_carry = lb_last;
            const double least = tlow * lb;
            const bool keep = act && !(lb > 0.0 && least > 1e-280 && fabs(sum) < least);
            const uint64_t kb = __ballot(keep);
            const uint32_t cnt = (uint32_t)__popcll(kb);
            while (Q.n + cnt > f.qcap) finish_queued<W, JL>(f, D, Q, thr);
            if (keep) {
                const uint32_t at = (uint32_t)__popcll(kb & lt), i = Q.n + at;
                if (!ahead) run_key(w, lo, hi);
                Q.lo[i] = lo;
                if (W == 2) Q.hi[i] = hi;
                Q.sum[i] = sum;
                Q.slot[i] = sg.start + nq + at;
            }
            Q.n += cnt;
            nq += cnt;
        }
        queued += nq;
        wave_sync();
        return nruns;
    }
    // Runs, 64 at a time: key, diagonal, sum in record order, score, exclusion;
    // a ballot places the surviving candidates, compacted, in run order.
    uint32_t written = 0, nalpha = 0;
    double ea_last = 0.0;  // E(alpha) of the last string so far
    for (uint32_t base = 0; base < nruns; base += 64) {
        const uint32_t u = base + (uint32_t)lane;
        const bool act = u < nruns;
        bool keep = false;
        uint64_t lo = and_lo, hi = and_hi;
        double sum = 0.0, score = 0.0, eb = 0.0, cross = 0.0, ea = 0.0;
        uint32_t p0 = 0, p1 = 0;
        bool ahead = false;
        if (act) {
            const uint32_t h0 = S.ix[u];
            p0 = h0 & 0x7FFFu;
            p1 = (uint32_t)S.ix[u + 1] & 0x7FFFu;
            ahead = (h0 >> 15) != 0u;
            run_key(S.ck[u], lo, hi);
        }
        const M a = (M)(W == 1 ? (lo >> n) : hi), b = (M)(W == 1 ? (lo & nmask) : lo);
        // without a threshold every candidate asks the exclusion filter: its
        // word is read first, so that the latency overlaps the work below
        const uint64_t fh = psi_filter_hash(lo, hi), fb = psi_filter_bits(fh);
        uint64_t fw = 0ull;
        if (act && !thr) fw = f.psi.filter[psi_filter_word(fh, f.psi.fmask)];
        // Alpha strings: the n-th string of the segment takes slot n mod amax
        // of the cache.  The lanes are taken in turns of at most amax strings;
        // a turn's new strings are the alpha heads among its lanes.
        const uint64_t heads = __ballot(ahead);
        const uint32_t ai = nalpha + (uint32_t)__popcll(heads & (lt | (1ull << lane))) - 1u;
        nalpha += (uint32_t)__popcll(heads);
        // E(alpha) by the lane of its head; its table entry, like E(beta)'s
        // below, is a read at random from memory that is waited for at the end
        double ea_head = 0.0;
        if (ahead) ea_head = spin_e(D, 0, a);
        for (uint64_t pend = __ballot(act); pend;) {
            const int l0 = __ffsll((long long)pend) - 1;
            const uint32_t a0 = (uint32_t)__builtin_amdgcn_readlane((int)ai, l0);
            const bool turn = ((pend >> lane) & 1ull) && ai - a0 < f.amax;
            const uint64_t tm = __ballot(turn);
            for (uint64_t fresh = tm & heads; fresh; fresh &= fresh - 1ull) {
                // c_q(alpha) of the head's string, q by lane
                const int hl = __ffsll((long long)fresh) - 1;
                const uint32_t sl = (uint32_t)__builtin_amdgcn_readlane((int)ai, hl) & amask;
                M as = (M)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)a, hl);
                if (W == 2) as |= (M)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)a >> 32), hl) << 32);
                if (lane < n) acache[sl * (uint32_t)n + (uint32_t)lane] = column_sum(D, as, (uint32_t)lane);
            }
            wave_sync();
            if (turn) {
                // E(alpha, beta), and the rank of beta in the same walk over its orbitals
                const double *cs = acache + (ai & amask) * (uint32_t)n;
                if (D.e[1]) {
                    struct Two {
                        double x;
                        uint32_t r;
                    };
                    uint32_t r = 0;
                    for_bits(b, n, D.ne[1], [&](int i, uint32_t q) { return Two{cs[q], D.binom[(i + 1) * (n + 1) + (int)q]}; },
                             [&](const Two &t) {
                                 cross = cross + t.x;
                                 r += t.r;
                             });
                    eb = D.e[1][min(r, D.last[1])];
                } else {
                    for_bits(b, n, D.ne[1], [&](int, uint32_t q) { return cs[q]; }, [&](double x) { cross = cross + x; });
                }
            }
            pend &= ~tm;
            if (pend) wave_sync();  // the next turn reuses slots this one reads
        }
        if (!D.e[1] && act) eb = spin_energy_u(D, D.ne[1], b);
        if (act) {
            if (f.eps <= 0.0) {
                // the run's values, in sorted (= record, ascending core) order
                sum = run_sum(S, p0, p1);
                keep = true;
            }
            {
                // of the alpha head at or before this lane, or of the last batch
                const uint64_t hm = heads & (lt | (1ull << lane));
                const double x = __shfl(ea_head, hm ? 63 - __clzll((long long)hm) : 0, 64);
                ea = hm ? x : ea_last;
            }
            const double den = f.E0 - (((f.ecore + ea) + eb) + cross);
            if (f.eps > 0.0) {
                // Alg. 2's threshold, per pair
                for (uint32_t j = p0; j < p1; ++j) {
                    const double v = S.val[j];
                    if (fabs(v / den) > f.eps) {
                        sum = sum + v;
                        keep = true;
                    }
                }
            }
            const double least = tlow * fabs(den);
            keep = keep && !(least > 1e-280 && fabs(sum) < least);
            if (keep) {
                score = sum / den;
                keep = abs_order(score) >= thr;
            }
            // an input determinant is not a candidate: the table is probed only
            // when the filter bits are set
            if (thr && keep) fw = f.psi.filter[psi_filter_word(fh, f.psi.fmask)];
            if (keep && (fw & fb) == fb) {
                uint32_t sl = psi_hash(lo, hi, f.psi.mask);
                bool found = false;
                for (uint32_t t = f.psi.state[sl]; t != 0u; t = f.psi.state[sl]) {
                    if (f.psi.lo[sl] == lo && f.psi.hi[sl] == hi) {
                        found = true;
                        break;
                    }
                    sl = (sl + 1u) & f.psi.mask;
                }
                keep = !found;
            }
        }
        if (heads) {
            const int hl = 63 - __clzll((long long)heads);
            const uint64_t x = (uint64_t)__double_as_longlong(ea_head);
            ea_last = __longlong_as_double((long long)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, hl) |
                                                       ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), hl) << 32)));
        }
        const uint64_t kb = __ballot(keep);
        if (keep) {
            const size_t d = (size_t)sg.start + written + (uint32_t)__popcll(kb & lt);
            f.clo[d] = lo;
            if (W == 2) f.chi[d] = hi;
            if (f.cnum) f.cnum[d] = sum;
            f.cscore[d] = score;
        }
        written += (uint32_t)__popcll(kb);
    }
    mark_slots(f, sg.start, written);
    return nruns;
}

// A resident grid: every wavefront strides over the final segments on its own
// (no barrier after the tables are staged), so that the load, sort and run
// phases of the sixteen wavefronts of a CU overlap.  Bound by VALU issue (about
// 60 % of the SIMD cycles) and, behind it, LDS.  One workgroup per segment of
// 4096 records, with a barrier between phases, issued VALU work 35 % of the time
// and waited 72 %; per launch, then and now: 9.6e8 records of 24e30o 24.3 and
// 14.4 ms, 1.3e8 of 16e20o 2.98 and 1.68 ms, 9.7e7 two-word ones of 20e36o 7.5
// and 5.45 ms.  Under a threshold the bounds leave 2 of 134 targets a segment
// of 24e30o to evaluate (8 of 103 of 16e20o): 10.1 ms per launch.
template <int W, int IT, bool JL>
__global__ __launch_bounds__(64 * kFinishWaves) __attribute__((amdgpu_waves_per_eu(4))) void k_finish(FinishArgs f)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int NT = 64 * kFinishWaves;
    const int n = f.n;
    const int tid = threadIdx.x;
    double *lx = reinterpret_cast<double *>(smem_raw);        // X, h_pp: where a string has no table
    double *lj = lx + (f.stage_x ? n * (n - 1) / 2 + n : 0);  // J
    uint32_t *lb = reinterpret_cast<uint32_t *>(lj + (JL ? n * (n + 1) / 2 : 0));  // binomials
    if (f.stage_x) {
        for (int t = tid; t < n * n; t += NT) {
            const int p = t / n, q = t % n;
            if (q > p) lx[p * n - (p * (p + 3) / 2 + 1) + q] = f.jk[n * n + t];
        }
        for (int t = tid; t < n; t += NT) lx[n * (n - 1) / 2 + t] = f.jk[2 * n * n + t];
    }
    if (JL)  // J_pq = J_qp bit for bit (the integrals are checked symmetric)
        for (int t = tid; t < n * n; t += NT) {
            const int p = t / n, q = t % n;
            if (q <= p) lj[p * (p + 1) / 2 + q] = f.jk[t];
        }
    if (f.st.binom)
        for (int t = tid; t < (f.st.kmax + 1) * (n + 1); t += NT) lb[t] = f.st.binom[t];
    const Diag<JL> D{JL ? lj : f.jk,  lx, lx + n * (n - 1) / 2, {f.st.e[0], f.st.e[1]}, {f.st.last[0], f.st.last[1]},
                     lb, n, {f.na, f.nb}};
    const uint32_t wv = uniform32((uint32_t)tid >> 6);
    unsigned char *mine = smem_raw + f.tab_bytes + wv * f.wave_bytes;
    WaveLds<IT> &S = *reinterpret_cast<WaveLds<IT> *>(mine);
    double *acache = reinterpret_cast<double *>(mine + ((sizeof(WaveLds<IT>) + 15) & ~size_t(15)));
    if ((tid & 63) < 2) S.val[WaveLds<IT>::CAP + (tid & 63)] = 0.0;
    __syncthreads();
    const uint32_t nf = part_count(dev_count(f.nfinal, f.dn_final), f.part);
    // thr: a lower bound of the final k-th |A|, from a pilot or earlier class batches, if any
    const uint64_t thr = f.thr ? *f.thr : 0ull;
    // the queue takes the place of the alpha cache, which the pruned path has no use for
    bool prune = thr != 0ull && !(f.eps > 0.0) && f.bounds;
    double level = prune ? f.bounds[2] : 0.0;
    Queue<W> Q;
    Q.lo = reinterpret_cast<uint64_t *>(acache);
    Q.hi = W == 2 ? Q.lo + f.qcap : nullptr;
    Q.sum = reinterpret_cast<double *>(Q.lo + W * f.qcap);
    Q.slot = reinterpret_cast<uint32_t *>(Q.sum + f.qcap);
    Q.n = 0;
    uint32_t runs = 0, tried = 0, queued = 0;
    const uint32_t step = gridDim.x * kFinishWaves;
    uint32_t i = blockIdx.x + gridDim.x * wv;
    Seg next = i < nf ? f.finals[part_index(i, f.part)] : Seg{0u, 0u, 0u};
    for (; i < nf; i += step) {
        const Seg sg = next;
        if (nf - i > step) next = f.finals[part_index(i + step, f.part)];
        if (seg_single(sg)) {
            finish_single<W, IT, JL>(f, D, S, sg);
            ++runs;
        } else {
            const uint32_t r = finish_segment<W, IT, JL>(f, D, S, acache, sg, thr, prune, level, queued, Q);
            runs += r;
            // An E0 among the diagonal elements leaves no bound.  Where more than a
            // quarter of the targets are queued, a wavefront goes on without: with
            // all of them queued a launch of 24e30o takes 28 ms, without bounds
            // 14.4, and with 2 % of them 10.
            tried += prune ? r : 0u;
            if (prune && tried >= 256u && queued > tried / 4u) {
                while (Q.n) finish_queued<W, JL>(f, D, Q, thr);
                prune = false;
            }
        }
    }
    while (Q.n) finish_queued<W, JL>(f, D, Q, thr);
    if (f.runs && (tid & 63) == 0 && runs) atomicAdd(f.runs, runs);
}

// ---------------------------------------------------------------- bounds
// out[i] = least of x[256 i, 256 i + 256)
__global__ __launch_bounds__(256) void k_block_min(const double *__restrict__ x, uint32_t n, double *__restrict__ out)
{
    __shared__ double s_m[4];
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    double m = i < n ? x[i] : __longlong_as_double(0x7FF0000000000000ll);
    for (int d = 32; d >= 1; d >>= 1) m = min_nan(__shfl_xor(m, d, 64), m);
    if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = min_nan(min_nan(s_m[0], s_m[1]), min_nan(s_m[2], s_m[3]));
}

// What bounds a diagonal element from below.
//   out[0]  the margin that covers the roundings of a bound and of a diagonal
//           element: each adds at most n^2 + n table entries, so it is off by
//           less than 2^-40 of the sum of all their magnitudes (n <= 64)
//   out[1]  the least E(beta)
//   out[2]  a first level for least_columns, out[3] the step of its search: from
//           the columns of na average orbitals
__global__ __launch_bounds__(1024) void k_diag_bounds(const double *__restrict__ jk, int n, int na, int nb, double E0,
                                                      double ecore, const double *__restrict__ emin, uint32_t nmin,
                                                      double *__restrict__ out)
{
    __shared__ double s_t[16], s_m[16], s_c[64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int q = wv; q < n; q += 16) {
        const double c = wave_sum(lane < n ? jk[q * n + lane] : 0.0);
        if (lane == 0) s_c[q] = c * ((double)na / n);
    }
    double t = 0.0, m = __longlong_as_double(0x7FF0000000000000ll);
    for (int i = threadIdx.x; i < 2 * n * n + n; i += 1024) t = t + fabs(jk[i]);
    for (uint32_t i = threadIdx.x; i < nmin; i += 1024) m = min_nan(emin[i], m);
    t = wave_sum(t);
    for (int d = 32; d >= 1; d >>= 1) m = min_nan(__shfl_xor(m, d, 64), m);
    if (lane == 0) {
        s_t[wv] = t;
        s_m[wv] = m;
    }
    __syncthreads();
    if (wv == 0) {
        const double c = lane < n ? s_c[lane] : 0.0;
        int rank = 0;
        for (int r = 0; r < n; ++r) rank += s_c[r] < c || (s_c[r] == c && r < lane) ? 1 : 0;
        const double lo = readlane_f64(c, max(__ffsll((long long)__ballot(lane < n && rank == 0)) - 1, 0));
        const double hi = readlane_f64(c, max(__ffsll((long long)__ballot(lane < n && rank == n - 1)) - 1, 0));
        const double lev = readlane_f64(c, max(__ffsll((long long)__ballot(lane < n && rank == max(nb - 1, 0))) - 1, 0));
        if (lane == 0) {
            for (int i = 1; i < 16; ++i) {
                t = t + s_t[i];
                m = min_nan(s_m[i], m);
            }
            out[0] = 0x1p-36 * ((t + fabs(E0)) + fabs(ecore));
            out[1] = m;
            out[2] = lev;
            out[3] = (hi - lo) / (2.0 * n);
        }
    }
}

// ---------------------------------------------------------------- pilot
// |A| in bins of the exponent and five mantissa bits, 2^-56 to 2^8 (what lies
// outside goes to the first or last)
constexpr uint32_t kPilotBins = 2048, kPilotBase = (1023u - 56u) << 5;
__device__ __forceinline__ uint32_t pilot_bin(double score)
{
    const uint32_t x = (uint32_t)(abs_order(score) >> 47);
    return x <= kPilotBase ? 0u : min(x - kPilotBase, kPilotBins - 1u);
}

// the candidates of the pilot's segments by bin of |A|, one wavefront a segment
__global__ __launch_bounds__(1024) void k_pilot_hist(const Seg *__restrict__ finals, uint32_t nf,
                                                     const unsigned long long *__restrict__ mask,
                                                     const double *__restrict__ score, uint32_t *__restrict__ hist)
{
    __shared__ uint32_t s_h[kPilotBins];
    for (uint32_t t = threadIdx.x; t < kPilotBins; t += 1024) s_h[t] = 0u;
    __syncthreads();
    const uint32_t np = part_count(nf, kPilotPart), lane = threadIdx.x & 63;
    for (uint32_t i = blockIdx.x * 16 + (threadIdx.x >> 6); i < np; i += gridDim.x * 16) {
        const Seg sg = finals[part_index(i, kPilotPart)];
        const uint32_t m = seg_single(sg) ? 1u : sg.size;
        for (uint32_t r = lane; r < m; r += 64) {
            const uint32_t at = sg.start + r;
            if ((mask[at >> 6] >> (at & 63u)) & 1ull) atomicAdd(&s_h[pilot_bin(score[at])], 1u);
        }
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < kPilotBins; t += 1024)
        if (s_h[t]) atomicAdd(&hist[t], s_h[t]);
}

// the lower edge of the bin that holds the k-th largest |A|; 0 with fewer
__global__ __launch_bounds__(1024) void k_pilot_pick(const uint32_t *__restrict__ hist, uint64_t k,
                                                     uint64_t *__restrict__ thr)
{
    __shared__ uint32_t s_tmp[16];
    // bins in descending order, two a thread
    const uint32_t b = kPilotBins - 1u - 2u * threadIdx.x;
    const uint32_t x = hist[b], y = hist[b - 1u];
    uint32_t tot;
    const uint64_t before = block_scan<16>(x + y, s_tmp, tot);
    if (threadIdx.x == 0 && tot < k) *thr = 0ull;
    if (before < k && k <= before + x) *thr = b ? (uint64_t)(b + kPilotBase) << 47 : 0ull;
    else if (before + x < k && k <= before + x + y) *thr = b > 1u ? (uint64_t)(b - 1u + kPilotBase) << 47 : 0ull;
}

// ---------------------------------------------------------------- collect
// one block per tile of slots: copies the marked ones, in order, to the pool
template <int W>
__global__ __launch_bounds__(256) void k_collect(const unsigned long long *__restrict__ mask, size_t P,
                                                 uint32_t ntile, const uint32_t *__restrict__ tcnt,
                                                 const uint32_t *__restrict__ off, const uint64_t *__restrict__ clo,
                                                 const uint64_t *__restrict__ chi, const double *__restrict__ cnum,
                                                 const double *__restrict__ cscore, uint64_t *__restrict__ plo,
                                                 uint64_t *__restrict__ phi, double *__restrict__ pnum,
                                                 double *__restrict__ pscore, size_t base, size_t cap)
{
    static_assert(kSlotTile == 64 * 64, "one mask word a lane");
    __shared__ unsigned long long s_m[64];
    __shared__ uint32_t s_at[64];
    const int lane = threadIdx.x & 63;
    for (uint32_t t = blockIdx.x; t < ntile; t += gridDim.x) {
        if (tcnt[t] == 0u) continue;  // uniform per block
        const size_t s0 = (size_t)t * kSlotTile;
        __syncthreads();  // the previous tile's words are read
        if (threadIdx.x < 64) {
            const unsigned long long m = s0 + (size_t)lane * 64 < P ? mask[s0 / 64 + lane] : 0ull;
            const uint32_t c = (uint32_t)__popcll(m);
            s_m[lane] = m;
            s_at[lane] = off[t] + wave_incl_scan(c) - c;
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x >> 6; i < 64; i += 4) {
            const unsigned long long m = s_m[i];
            if (!((m >> lane) & 1ull)) continue;
            const size_t s = s0 + i * 64 + (uint32_t)lane;
            const size_t d = base + s_at[i] + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
            if (d >= cap) {
                raise_fault(kFaultSlot);
                continue;
            }
            plo[d] = clo[s];
            if (W == 2) phi[d] = chi[s];
            if (pnum) pnum[d] = cnum[s];
            pscore[d] = cscore[s];
        }
    }
}

constexpr uint32_t kMaxClassSegs = 2048;  // classes of one batch

// the first segments: classes larger than the capacity, and runs of
// consecutive smaller ones coalesced into finals of at most `cap` records
__global__ __launch_bounds__(1024) void k_class_segs(uint32_t nc, uint32_t nq, const uint32_t *__restrict__ offsets,
                                                     const uint32_t *__restrict__ total, uint32_t cap, SegLists lists,
                                                     uint32_t *__restrict__ ctr, uint32_t nrec)
{
    // Bounds are clamped to the record buffer (nrec records): counts that
    // overrun it (inputs that fail validation) cannot send a segment past it.
    __shared__ uint32_t s_start[kMaxClassSegs + 1];
    __shared__ uint16_t s_next[kMaxClassSegs + 2], s_jump[kMaxClassSegs + 2];
    __shared__ uint8_t s_mark[kMaxClassSegs + 2];
    if (threadIdx.x < 8) ctr[threadIdx.x] = 0u;
    for (uint32_t c = threadIdx.x; c < nc; c += 1024) s_start[c] = min(offsets[(size_t)c * nq], nrec);
    if (threadIdx.x == 0) s_start[nc] = min(*total, nrec);
    __threadfence();  // the counters are zero before any wavefront adds to them
    __syncthreads();
    greedy_groups<3>(s_start, nc, cap, s_next, s_jump, s_mark, threadIdx.x, 1024u, [] { __syncthreads(); });
    for (uint32_t b = 0; b < nc; b += 1024) {
        const uint32_t c = b + threadIdx.x;
        uint32_t size = 0;
        if (c < nc && s_mark[c]) size = s_start[s_next[c]] - s_start[c];
        // offsets that wrapped round (inputs that fail validation) give no segment
        if (size > nrec || (size && (uint64_t)s_start[c] + size > nrec)) size = 0;
        const uint32_t kind = size == 0u ? 0u : (size <= cap ? 1u : (size <= (uint32_t)kTileN ? 2u : 3u));
        append_segs(lists, kind, size ? Seg{s_start[c], size, make_meta(0u, false)} : Seg{0u, 0u, 0u});
    }
}

}  // namespace

// ---------------------------------------------------------------- host side
// A bound: the split, finish and collect of P records in nc classes take less
// (see level_tiles, level_hist) for every finish capacity.
size_t bucket_workspace_bytes(size_t P, size_t nc, int W, int finish_cap)
{
    const size_t cap = finish_cap >= 4096 ? 4096 : (finish_cap >= 2048 ? 2048 : 1024);
    const size_t finals = nc + P / 8 + 65536, level = P / cap + nc + 16;
    const size_t tiles = (P + kTileN - 1) / kTileN + level;
    return finals * sizeof(Seg) + 2 * level * sizeof(Seg) + level * 16 + tiles * (256 * 8 + 8) +
           level * ((kMaxSplit - 1) * 8 * W + 32) + P + 256 + finals * (8 * 2 + 4 * 4 + 8) + (finals + tiles * 256) / 1024 +
           (4 << 20);
}

// LDS per workgroup: two workgroups share a CU
constexpr size_t kFinishLdsBudget = 80 * 1024;

template <int W, int IT>
static int launch_finish(FinishArgs &fa, const BucketArgs &b, uint32_t nf, int part, hipStream_t s, Profiler *prof)
{
    fa.part = part;
    nf = part_count(nf, part);
    const size_t base = (sizeof(WaveLds<IT>) + 15) & ~size_t(15);
    const size_t n = (size_t)b.n, entry = n * 8;  // of the alpha cache
    // strings without a table are evaluated from X and h_pp, those with one are
    // ranked; J is staged where every wavefront keeps room for two alpha strings
    fa.stage_x = !b.st.e[0] || !b.st.e[1] ? 1 : 0;
    size_t tab = (fa.stage_x ? (n * (n - 1) / 2 + n) * 8 : 0) + (b.st.binom ? (size_t)(b.st.kmax + 1) * (n + 1) * 4 : 0);
    // a wavefront's alpha strings and its queue share one region
    auto region = [&](size_t strings) { return std::max(strings * entry, fa.bounds ? 64 * queue_entry<W>() : 0); };
    auto total = [&](size_t tables, size_t strings) {
        return ((tables + 15) & ~size_t(15)) + kFinishWaves * ((base + region(strings) + 15) & ~size_t(15));
    };
    const bool jl = total(tab + n * (n + 1) / 2 * 8, 2) <= kFinishLdsBudget;
    if (jl) tab += n * (n + 1) / 2 * 8;
    tab = (tab + 15) & ~size_t(15);
    fa.amax = 1;
    while (fa.amax < 32 && total(tab, 2 * fa.amax) <= kFinishLdsBudget) fa.amax *= 2;
    fa.tab_bytes = (uint32_t)tab;
    fa.wave_bytes = (uint32_t)((base + region(fa.amax) + 15) & ~size_t(15));
    fa.qcap = (uint32_t)std::min<size_t>(region(fa.amax) / queue_entry<W>(), 128);
    const size_t lds = tab + (size_t)kFinishWaves * fa.wave_bytes;
    void (*kernel)(FinishArgs) = jl ? k_finish<W, IT, true> : k_finish<W, IT, false>;
    const void *fn = (const void *)kernel;
    constexpr int NT = 64 * kFinishWaves;
    ASCI_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    int dev = 0, ncu = 0, per_cu = 0;
    ASCI_HIP(hipGetDevice(&dev));
    ASCI_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    ASCI_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, NT, lds));
    // one resident grid; few segments are spread one wavefront to a workgroup
    const uint32_t grid = std::min<uint32_t>(nf, (uint32_t)std::max(1, ncu * std::max(per_cu, 1)));
    // bytes: every record read once; the candidates it writes are added once
    // their number is known (finish_bytes)
    ProfScope ps(prof, part == kPilotPart ? "finish_pilot" : "finish",
                 (8.0 * W + 8.0) * (double)b.P / (part == kPilotPart ? kPilot : 1), s);
    kernel<<<grid, NT, lds, s>>>(fa);
    ASCI_LAUNCH_CHECK();
    return ps.tok;
}

// algorithmic bytes of a finish launch: records read, candidates written
// (key and score, plus N_a when every candidate is kept)
static void finish_bytes(const BucketArgs &b, int W)
{
    if (b.prof && b.finish_tok >= 0)
        b.prof->set_bytes(b.finish_tok, (8.0 * W + 8.0) * (double)b.P +
                                            (8.0 * W + 8.0 + (b.cnum ? 8.0 : 0.0)) * (double)b.V);
}

constexpr size_t kQueuedRecords = (size_t)1 << 28;

// device counters of one batch
enum { kCtrFinal = 0, kCtrLarge = 1 /* and 2: per level parity */, kCtrOverflow = 3, kCtrSmall = 4, kCtrLevels = 6 };

// Split levels, finish, and the scan that places the candidates.  With dev
// nothing is read back: b.dev_levels levels and the small split run on launch
// shapes sized for bounds (the caller checks b.dn_nlarge and b.dn_overflow);
// else the host reads the number of large segments once per level and stops
// when none is left.
template <int W>
static void accumulate(BucketArgs &b, Arena &ar, hipStream_t s, Profiler *prof, HostStage *hs, bool dev)
{
    const uint32_t cap = (uint32_t)wave_cap(b.finish_cap);
    const size_t P = b.P;
    const uint32_t finals_cap = (uint32_t)std::min<size_t>(b.nc + P / 8 + 65536, 0xFFFFFFF0u);
    const uint32_t level_cap = (uint32_t)(P / cap + 16);  // disjoint segments of more than cap records
    Seg *finals = ar.take<Seg>(finals_cap);
    Seg *lv[2] = {ar.take<Seg>(level_cap), ar.take<Seg>(level_cap)};
    Seg *small = ar.take<Seg>(level_cap);
    uint32_t *ctr = ar.take<uint32_t>(8);
    uint32_t *hcnt = hs ? (uint32_t *)hs->ptr : nullptr;
    SegLists lists{finals, small, lv[0], ctr + kCtrFinal, ctr + kCtrSmall, ctr + kCtrLarge, ctr + kCtrOverflow,
                   finals_cap, level_cap, level_cap};
    require(b.nc <= kMaxClassSegs, ASCI_EINVAL, "too many classes in one batch");
    k_class_segs<<<1, 1024, 0, s>>>(b.nc, b.nq, b.offsets, b.total, cap, lists, ctr,
                                    (uint32_t)std::min<size_t>(P, 0xFFFFFFFFu));
    ASCI_LAUNCH_CHECK();
    auto read_counts = [&]() {
        ASCI_HIP(hipMemcpyAsync(hcnt, ctr, 8 * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
        ASCI_HIP(hipStreamSynchronize(s));
        require(hcnt[kCtrOverflow] == 0, ASCI_EDEVICE, "bucket segment list overflow");
    };
    uint8_t *dig = ar.take<uint8_t>(P + 1);
    uint64_t *spl_lo = ar.take<uint64_t>(2 * P / cap + 1);
    uint64_t *spl_hi = W == 2 ? ar.take<uint64_t>(2 * P / cap + 1) : nullptr;
    uint32_t *lev_tot = ar.take<uint32_t>(4);
    // per-kernel timing: the records of each level, for the bytes its passes move
    const bool timed = prof && prof->on;
    uint32_t *level_rec = ar.take<uint32_t>(64);
    std::vector<int> tok_hist, tok_scatter;
    const size_t mark = ar.used();
    const KeyBufs kb{{b.klo[0], b.klo[1]}, {b.khi[0], b.khi[1]}};
    int lev = 0;
    // One split level of the large segments of list lev & 1: nlarge of them, or
    // (queued) at most nlarge, their number on the device, on grids of at most
    // gmax workgroups.
    auto split_level = [&](uint32_t nlarge, bool queued, uint32_t gmax) {
        ar.reset();
        (void)ar.take<char>(mark);
        require(lev < 64, ASCI_EDEVICE, "bucket split did not converge");
        Seg *segs = lv[lev & 1];
        const uint32_t *dn_seg = queued ? ctr + kCtrLarge + (lev & 1) : nullptr;
        lists.next = lv[(lev & 1) ^ 1];
        lists.nnext = ctr + kCtrLarge + ((lev & 1) ^ 1);
        const uint32_t ntiles = (uint32_t)level_tiles(P, nlarge);
        const size_t nhist = level_hist(P, nlarge, cap);
        uint32_t *tbase = ar.take<uint32_t>((size_t)nlarge + 1);
        uint32_t *hbase = ar.take<uint32_t>((size_t)nlarge + 1);
        uint32_t *skip = ar.take<uint32_t>((size_t)nlarge + 1);
        uint32_t *tseg = ar.take<uint32_t>((size_t)ntiles + 1);
        uint32_t *hist = ar.take<uint32_t>(nhist + 1);
        // launch shapes: per-segment kernels stride over the level's segments,
        // tile kernels over its tiles (eight XCD groups of workgroups)
        const unsigned g_seg = std::min(nlarge, gmax);
        const unsigned g_tiles = 8u * std::min((ntiles + 7) / 8, gmax / 8);
        const bool few = ntiles <= 8192;
        k_level_plan<<<1, 1024, 0, s>>>(segs, nlarge, cap, tbase, hbase, skip, lev_tot, lists.nnext, few ? tseg : nullptr,
                                        dn_seg, ctr + kCtrLevels, timed ? level_rec + lev : nullptr);
        ASCI_LAUNCH_CHECK();
        if (!few) {
            k_tile_seg<<<std::min((ntiles + 255) / 256, 1024u), 256, 0, s>>>(tbase, nlarge, lev_tot, tseg, dn_seg);
            ASCI_LAUNCH_CHECK();
        }
        {
            ProfScope ps(prof, "split_sample", 0.0, s);
            // class-sized segments of the first level sort up to 2048 samples:
            // more threads per sort; later levels sort a few hundred
            if (lev == 0) k_seg_splitters<W, 1024><<<g_seg, 1024, 0, s>>>(segs, cap, kb, spl_lo, spl_hi, nlarge, dn_seg);
            else k_seg_splitters<W, 256><<<g_seg, 256, 0, s>>>(segs, cap, kb, spl_lo, spl_hi, nlarge, dn_seg);
            ASCI_LAUNCH_CHECK();
        }
        SplitArgs sa;
        sa.segs = segs;
        sa.tile_base = tbase;
        sa.hist_base = hbase;
        sa.tile_seg = tseg;
        sa.ntiles = ntiles;
        sa.lev = lev_tot;
        sa.hist = hist;
        sa.klo[0] = b.klo[0];
        sa.klo[1] = b.klo[1];
        sa.khi[0] = b.khi[0];
        sa.khi[1] = b.khi[1];
        sa.val[0] = b.val[0];
        sa.val[1] = b.val[1];
        sa.cap = cap;
        sa.spl_lo = spl_lo;
        sa.spl_hi = spl_hi;
        sa.dig = dig;
        {
            ProfScope ps(prof, "split_hist", 0.0, s);
            tok_hist.push_back(ps.tok);
            k_split_hist<W><<<g_tiles, kHistT, 0, s>>>(sa);
            ASCI_LAUNCH_CHECK();
        }
        scan_u32(hist, hist, nhist, nullptr, ar, s, prof, lev_tot + 1);
        k_split_children<W><<<(g_seg + kChildWaves - 1) / kChildWaves, 64 * kChildWaves, 0, s>>>(
            segs, nlarge, hbase, hist, cap, spl_lo, spl_hi, skip, lists, dn_seg);
        ASCI_LAUNCH_CHECK();
        {
            ProfScope ps(prof, "split_scatter", 0.0, s);
            tok_scatter.push_back(ps.tok);
            k_split_scatter<W><<<g_tiles, kTileT, 0, s>>>(sa, skip);
            ASCI_LAUNCH_CHECK();
        }
        ++lev;
    };
    // The segments of one tile at most, each by one workgroup; nsm: their number
    // on the device (nsmall is then a bound).
    auto small_split = [&](uint32_t nsmall, uint32_t *nsm, uint32_t gmax) {
        if (nsmall == 0) return;
        ProfScope ps(prof, "small_split", 0.0, s);
        k_small_split<W><<<std::min(nsmall, gmax), kSmallT, 0, s>>>(
            small, nsmall, nsm, cap, b.klo[0], b.klo[1], b.khi[0], b.khi[1], b.val[0], b.val[1], lists);
        ASCI_LAUNCH_CHECK();
    };
    constexpr uint32_t kAnyGrid = 1u << 30;
    if (dev) {
        for (int l = 0; l < b.dev_levels; ++l) split_level(level_cap, true, 2048u);
        small_split(level_cap, ctr + kCtrSmall, 4096u);
        // what is left in list lev & 1 fails the call
        b.dn_nlarge = ctr + kCtrLarge + (lev & 1);
        b.dn_overflow = ctr + kCtrOverflow;
        b.dn_levels = ctr + kCtrLevels;
    } else {
        // What most batches need is queued at once: a read-back between two
        // levels leaves the chip idle for about 35 us (8a5b23o, 4.6e7 records: five
        // read-backs, now one).  A large segment has more records than a tile.
        // Above 2^28 records a level takes long enough, and its grid is better
        // sized by its count.
        bool small_done = P <= kQueuedRecords;
        if (small_done) {
            for (int l = 0; l < (P <= ((size_t)1 << 19) ? 1 : 2); ++l) split_level((uint32_t)(P / kTileN + 1), true, kAnyGrid);
            small_split(level_cap, ctr + kCtrSmall, 16384u);
        }
        read_counts();
        if (small_done && hcnt[kCtrLarge + (lev & 1)] > 0) {
            fill_u32(ctr + kCtrSmall, 1, 0u, s);  // the ones so far are split
            small_done = false;
        }
        while (hcnt[kCtrLarge + (lev & 1)] > 0) {
            split_level(hcnt[kCtrLarge + (lev & 1)], false, kAnyGrid);
            read_counts();
        }
        if (!small_done && hcnt[kCtrSmall] > 0) {
            small_split(hcnt[kCtrSmall], nullptr, kAnyGrid);
            read_counts();
        }
        b.levels = hcnt[kCtrLevels];
        if (timed && lev > 0) {
            std::vector<uint32_t> rec((size_t)lev);
            ASCI_HIP(hipMemcpyAsync(rec.data(), level_rec, rec.size() * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
            ASCI_HIP(hipStreamSynchronize(s));
            for (size_t l = 0; l < rec.size(); ++l) {
                if (tok_hist[l] >= 0) prof->set_bytes(tok_hist[l], 8.0 * W * rec[l]);
                if (tok_scatter[l] >= 0) prof->set_bytes(tok_scatter[l], 2.0 * (8.0 * W + 8.0) * rec[l]);
            }
        }
    }
    ar.reset();
    (void)ar.take<char>(mark);
    const uint32_t nf = dev ? finals_cap : hcnt[kCtrFinal];
    b.nfinal = nf;
    // candidate marks: a bit per slot, a count per tile of slots, cleared together
    const uint32_t ntile = (uint32_t)((P + kSlotTile - 1) / kSlotTile);
    const size_t mwords = 2 * (size_t)ntile * (kSlotTile / 64);
    uint32_t *marks = ar.take<uint32_t>(mwords + ntile + 1);
    fill_u32(marks, mwords + ntile, 0u, s);
    b.mask = reinterpret_cast<unsigned long long *>(marks);
    b.tcnt = marks + mwords;
    b.ntile = ntile;
    if (nf) {
        FinishArgs fa;
        fa.finals = finals;
        for (int i = 0; i < 2; ++i) {
            fa.klo[i] = b.klo[i];
            fa.khi[i] = b.khi[i];
            fa.val[i] = b.val[i];
        }
        fa.n = b.n;
        fa.na = b.na;
        fa.nb = b.nb;
        fa.jk = b.jk;
        fa.st = b.st;
        fa.thr = b.thr;
        fa.ecore = b.ecore;
        fa.E0 = b.E0;
        fa.eps = b.eps;
        fa.clo = b.clo;
        fa.chi = b.chi;
        fa.cnum = b.cnum;
        fa.cscore = b.cscore;
        fa.mask = b.mask;
        fa.tcnt = b.tcnt;
        fa.nfinal = nf;
        fa.dn_final = dev ? ctr + kCtrFinal : nullptr;
        fa.psi = b.psi;
        fa.bounds = b.bounds;
        b.prof = prof;
        auto finish = [&](int part) {
            if (cap == 512) b.finish_tok = launch_finish<W, 8>(fa, b, nf, part, s, prof);
            else b.finish_tok = launch_finish<W, 4>(fa, b, nf, part, s, prof);
        };
        fa.runs = b.pilot_k > 0 ? b.runs : nullptr;
        if (b.pilot_k > 0) {
            uint64_t *thr = ar.take<uint64_t>(1);
            uint32_t *hist = ar.take<uint32_t>(kPilotBins);
            fill_u32(hist, kPilotBins, 0u, s);
            finish(kPilotPart);
            k_pilot_hist<<<std::min(part_count(nf, kPilotPart) / 16 + 1, 256u), 1024, 0, s>>>(finals, nf, b.mask, b.cscore,
                                                                                            hist);
            ASCI_LAUNCH_CHECK();
            k_pilot_pick<<<1, 1024, 0, s>>>(hist, b.pilot_k, thr);
            ASCI_LAUNCH_CHECK();
            fa.thr = thr;
            finish(kRestPart);
        } else {
            finish(kAll);
        }
    }
    uint32_t *off = ar.take<uint32_t>((size_t)ntile + 1);
    uint32_t *d_v = ar.take<uint32_t>(4);
    scan_u32(b.tcnt, off, ntile, d_v, ar, s, nullptr);
    b.off = off;
    b.dn_V = d_v;
    b.dn_nfinal = ctr + kCtrFinal;
}

template <int W>
void bucket_accumulate(BucketArgs &b, Arena &ar, hipStream_t s, Profiler *prof, HostStage &hs)
{
    accumulate<W>(b, ar, s, prof, &hs, false);
    uint32_t *hcnt = (uint32_t *)hs.ptr;
    ASCI_HIP(hipMemcpyAsync(hcnt + 6, b.dn_V, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    if (b.pilot_k > 0) ASCI_HIP(hipMemcpyAsync(hcnt + 7, b.runs, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    b.h_v = hcnt + 6;
    if (b.defer_v) {
        b.V = ~0u;  // unknown until bucket_read_v
    } else {
        ASCI_HIP(hipStreamSynchronize(s));
        b.V = hcnt[6];
        b.h_runs = hcnt[7];
        finish_bytes(b, W);
    }
}

template <int W>
void bucket_accumulate_dev(BucketArgs &b, Arena &ar, hipStream_t s)
{
    accumulate<W>(b, ar, s, nullptr, nullptr, true);
    b.V = (uint32_t)std::min<size_t>(b.P, 0xFFFFFFFFu);  // a bound: the count is *dn_V
}

template <int W>
int bucket_collect(BucketArgs &b, hipStream_t s, Profiler *prof)
{
    if (b.nfinal == 0 || b.V == 0) return -1;
    // with the count still in flight the bytes are set once it is known
    ProfScope ps(prof, "collect", b.defer_v ? 0.0 : (8.0 * W + 8.0) * 2.0 * b.V, s);
    k_collect<W><<<std::min<uint32_t>(b.ntile, 65536u), 256, 0, s>>>(b.mask, b.P, b.ntile, b.tcnt, b.off, b.clo, b.chi,
                                                                     b.cnum, b.cscore, b.pool_lo, b.pool_hi,
                                                                     b.pool_num, b.pool_score, b.pool_base, b.pool_cap);
    ASCI_LAUNCH_CHECK();
    return ps.tok;
}

void bucket_diag_bounds(const double *jk, int n, int na, int nb, double E0, double ecore, const double *etab, uint32_t ntab,
                        double *tmp, double *out, hipStream_t s)
{
    const uint32_t nmin = (ntab + kMinRanks - 1) / kMinRanks;
    k_block_min<<<nmin, kMinRanks, 0, s>>>(etab, ntab, tmp);
    ASCI_LAUNCH_CHECK();
    k_diag_bounds<<<1, 1024, 0, s>>>(jk, n, na, nb, E0, ecore, tmp, nmin, out);
    ASCI_LAUNCH_CHECK();
}

void bucket_read_v(BucketArgs &b, hipStream_t s)
{
    if (!b.defer_v) return;
    ASCI_HIP(hipStreamSynchronize(s));
    b.V = *b.h_v;
    b.h_runs = b.h_v[1];
    b.defer_v = false;
    finish_bytes(b, b.n <= 32 ? 1 : 2);
}

// sum of N_a * A_a over the batch's candidates: per tile of slots (each lane
// its marked slots in order, then a fixed tree), then a fixed-order tree over
// the tiles
__global__ __launch_bounds__(256) void k_pt2_tiles(const unsigned long long *__restrict__ mask, size_t P,
                                                   uint32_t ntile, const uint32_t *__restrict__ tcnt,
                                                   const double *__restrict__ cnum,
                                                   const double *__restrict__ cscore, double *__restrict__ part)
{
    __shared__ double sh[256];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (uint32_t t = blockIdx.x; t < ntile; t += gridDim.x) {
        double e = 0.0;
        if (tcnt[t]) {
            const size_t s0 = (size_t)t * kSlotTile;
            for (uint32_t i = (uint32_t)wv; i < kSlotTile / 64; i += 4) {
                if (s0 + (size_t)i * 64 >= P) break;
                const unsigned long long m = mask[s0 / 64 + i];
                const size_t s = s0 + (size_t)i * 64 + (uint32_t)lane;
                if ((m >> lane) & 1ull) e = e + cnum[s] * cscore[s];
            }
        }
        __syncthreads();
        sh[threadIdx.x] = e;
        __syncthreads();
        for (int w = 128; w >= 1; w >>= 1) {
            if ((int)threadIdx.x < w) sh[threadIdx.x] = sh[threadIdx.x] + sh[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) part[t] = sh[0];
    }
}

__global__ __launch_bounds__(1024) void k_sum_fixed(const double *__restrict__ x, uint32_t n, double *__restrict__ out)
{
    __shared__ double sh[1024];
    double acc = 0.0;
    for (uint32_t i = threadIdx.x; i < n; i += 1024) acc = acc + x[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 512; w >= 1; w >>= 1) {
        if (threadIdx.x < (unsigned)w) sh[threadIdx.x] = sh[threadIdx.x] + sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0];
}

double bucket_pt2(BucketArgs &b, Arena &ar, hipStream_t s, HostStage &hs)
{
    if (b.nfinal == 0) return 0.0;
    double *part = ar.take<double>(b.ntile);
    double *tot = ar.take<double>(1);
    k_pt2_tiles<<<std::min<uint32_t>(b.ntile, 65536u), 256, 0, s>>>(b.mask, b.P, b.ntile, b.tcnt, b.cnum, b.cscore, part);
    ASCI_LAUNCH_CHECK();
    k_sum_fixed<<<1, 1024, 0, s>>>(part, b.ntile, tot);
    ASCI_LAUNCH_CHECK();
    double *h = (double *)((char *)hs.ptr + 128);
    ASCI_HIP(hipMemcpyAsync(h, tot, sizeof(double), hipMemcpyDeviceToHost, s));
    ASCI_HIP(hipStreamSynchronize(s));
    return *h;
}

// the collect of the device-driven variant: counts read on the device
template <int W>
void bucket_collect_dev(BucketArgs &b, hipStream_t s)
{
    k_collect<W><<<std::min<uint32_t>(b.ntile, 65536u), 256, 0, s>>>(b.mask, b.P, b.ntile, b.tcnt, b.off, b.clo, b.chi,
                                                                     b.cnum, b.cscore, b.pool_lo, b.pool_hi,
                                                                     b.pool_num, b.pool_score, b.pool_base, b.pool_cap);
    ASCI_LAUNCH_CHECK();
}

template void bucket_accumulate_dev<1>(BucketArgs &, Arena &, hipStream_t);
template void bucket_accumulate_dev<2>(BucketArgs &, Arena &, hipStream_t);
template void bucket_collect_dev<1>(BucketArgs &, hipStream_t);
template void bucket_collect_dev<2>(BucketArgs &, hipStream_t);

uint32_t *bucket_fault_word() { return fault_word(); }
void bucket_fault_fetch(unsigned int *dst, hipStream_t s) { fault_fetch(dst, s); }

template void bucket_accumulate<1>(BucketArgs &, Arena &, hipStream_t, Profiler *, HostStage &);
template void bucket_accumulate<2>(BucketArgs &, Arena &, hipStream_t, Profiler *, HostStage &);
template int bucket_collect<1>(BucketArgs &, hipStream_t, Profiler *);
template int bucket_collect<2>(BucketArgs &, hipStream_t, Profiler *);

}  // namespace asci
