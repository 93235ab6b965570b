// Binning of (Gaussian, tile) pairs and the device radix sort that builds
// the depth-indexed per-tile Gaussian lists (paper Sec. II-A: the scattering
// intensity is computed along depth-indexed Gaussian lists; the third radar
// coordinate serves as the sorting depth).
//
//   1. records are sorted by (fl32 depth, index) with a stable LSD radix
//      sort of 32-bit keys (index order is the initial order, the first
//      pass generates the indices); with up to SEG_MAX views each view's
//      records are sorted among themselves (a segmented sort), so the order
//      is view-major and the reads by record index that follow stay inside
//      one view at a time; with more views they are sorted together;
//   2. their computation-plane pair counts are scanned in that order and
//      every record emits (tile bucket, record) pairs in depth order;
//   3. a stable LSD radix sort of the pairs on the bucket id yields, per
//      tile, the Gaussians in depth order (segmented by view when the
//      records were: only the tile bits within a view are sorted);
//   4. tile ranges [start, end) are read off the sorted bucket ids;
//   5. after pass A, records with a nonzero intensity emit their
//      imaging-plane pairs in index order (after the computation-plane
//      ones) and the same sort groups them by tile, the order only fixing
//      the FP32 summation order of pass B.
//
// Small views get their lists without the sorts (k_view_rank, k_view_counts,
// k_tile_lists), and small calls no imaging-plane lists at all.
//
// Sort blocks work on runs of tiles of 4096 items (256 threads x 16), or of
// 2048 or 1024 where there are few.
#include "common.hpp"

#include <algorithm>
#include <cstring>

namespace sdgr {
namespace {

constexpr int SB = 256;          // threads per sort/scan block
constexpr int SI_LARGE = 16;     // items per thread and tile
constexpr int SI_MIDDLE = 8;
constexpr int SI_SMALL = 4;
constexpr int MAX_RADIX = 1 << 10;

inline unsigned nblocks(int64_t n, int sn) { return (unsigned)((n + sn - 1) / sn); }

__global__ void __launch_bounds__(256) k_fill(uint32_t* p, uint32_t v, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}


__global__ void __launch_bounds__(256) k_iota(uint32_t* p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = (uint32_t)i;
}

// Digit width of a sort: the fewest passes of at most 10 bits, then the
// narrowest digit (8 to 10 bits) that covers the key in that many passes. A
// key of no bits (one bucket) has a width too: the segment table of a sort is
// set up by it whether or not the sort makes a pass.
inline int digit_bits(int bits)
{
    const int passes = std::max(1, (bits + 9) / 10);
    const int d = (bits + passes - 1) / passes;
    return d < 8 ? 8 : d;
}

// Sort grids have at most max_blocks blocks; each takes a contiguous
// run of tiles of the actual item count, so the per-block digit
// counts (digit-major, R x nb words) and their scan stay small however long
// the array is.
inline unsigned sort_grid(int64_t cap, unsigned max_blocks, int sn)
{
    return std::min(nblocks(cap, sn), max_blocks);
}

// Items of a sort tile: small tiles where the large ones would be too few
// blocks; only with 8-bit digits, whose counts fit the same space for four
// times the blocks. The depth sort of 160k records takes 57 us with tiles of
// 1024 items, 62 of 2048, 76 of 4096; of 500k 70, 67 and 79; of 640k 96, 83
// and 87; of 1.6M 135, 110 and 104; the sort of 2.8M pairs with their
// positions 43, 40 and 46.
constexpr int64_t SORT_SMALL = int64_t(1) << 18, SORT_MIDDLE = int64_t(1) << 20,
                  SORT_MIDDLE_PAIRS = int64_t(1) << 22;

int sort_tile_items(int64_t cap, int bits, bool positions)
{
    if (digit_bits(bits) != 8) return SB * SI_LARGE;
    if (cap <= SORT_SMALL) return SB * SI_SMALL;
    return SB * (cap <= (positions ? SORT_MIDDLE_PAIRS : SORT_MIDDLE) ? SI_MIDDLE : SI_LARGE);
}

struct SortSpan {
    int64_t n;      // items
    uint32_t nb;    // blocks with items
    uint32_t tpb;   // tiles per block
};

__device__ __forceinline__ SortSpan sort_span(const uint32_t* n_dev, uint32_t grid, int sn)
{
    SortSpan sp;
    sp.n = *n_dev;
    const uint32_t tiles = (uint32_t)((sp.n + sn - 1) / sn);
    sp.tpb = max(1u, (tiles + grid - 1) / grid);
    sp.nb = (tiles + sp.tpb - 1) / sp.tpb;
    return sp;
}

// Items of one sort block: a run of tiles of the whole array, or (segmented
// sorts) a run of tiles of one segment. Digits are taken from key - kb; slot is
// the block's column in the digit-major count matrix of stride columns.
struct BlockItems {
    int64_t first, end;
    uint32_t tiles, stride, kb;
    int s;
};

template <int SN>
__device__ __forceinline__ bool span_items(const uint32_t* n_dev, BlockItems& bi)
{
    const SortSpan sp = sort_span(n_dev, gridDim.x, SN);
    if (blockIdx.x >= sp.nb) return false;
    bi.first = (int64_t)blockIdx.x * sp.tpb * SN;
    bi.end = sp.n;
    bi.tiles = sp.tpb;
    bi.stride = sp.nb;
    bi.kb = 0u;
    bi.s = 0;
    return true;
}

// Segment of block b: the last s with tp[s] <= b (empty segments own no
// block, so the block lands in the non-empty one that follows them).
template <int SN>
__device__ __forceinline__ bool seg_items(const SegTable* t, int S, uint32_t* s_tp, BlockItems& bi)
{
    for (int k = threadIdx.x; k <= S; k += blockDim.x) s_tp[k] = t->tp[k];
    __syncthreads();
    const uint32_t T = s_tp[S], b = blockIdx.x;
    if (b >= T) return false;
    int lo = 0, hi = S - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_tp[mid] <= b) lo = mid; else hi = mid - 1;
    }
    const uint32_t tpb = t->tpb;
    bi.s = lo;
    bi.first = (int64_t)t->seg[lo] + (int64_t)(b - s_tp[lo]) * tpb * SN;
    bi.end = min(bi.first + (int64_t)tpb * SN, (int64_t)t->seg[lo + 1]);
    bi.tiles = tpb;
    bi.stride = T;
    bi.kb = t->kb[lo];
    return true;
}

// Segment table of a segmented sort: item offsets (views' records, or the
// computation-plane pair offsets the emission wrote for the first record of
// each view), key bases, and the block offsets of every segment, with as
// many tiles per block as keep the blocks near MAX_SORT_BLOCKS.
__global__ void __launch_bounds__(SEG_MAX)
k_seg_setup(const DevView* __restrict__ views, int nv, int64_t records,
            const uint32_t* __restrict__ n_dev, int pairs, uint32_t max_blocks, uint32_t sn,
            SegTable* __restrict__ t)
{
    __shared__ uint32_t s_seg[SEG_MAX + 1];
    __shared__ uint8_t s_empty[SEG_MAX];
    __shared__ uint32_t s_w[SEG_MAX / WAVE];
    const int tid = threadIdx.x;
    const uint32_t n = *n_dev;
    if (tid < nv) {
        const int64_t r0 = views[tid].rec_off;
        const int64_t r1 = tid + 1 < nv ? views[tid + 1].rec_off : records;
        s_empty[tid] = r1 <= r0;
        s_seg[tid] = pairs ? t->seg[tid] : (uint32_t)r0;
    }
    __syncthreads();
    if (tid == 0) {
        // empty segments start where the next one does; all clamped to n
        // (0 after a pair overflow)
        uint32_t next = n;
        for (int v = nv - 1; v >= 0; --v) {
            const uint32_t o = s_empty[v] ? next : min(s_seg[v], next);
            s_seg[v] = o;
            next = o;
        }
        s_seg[nv] = n;
    }
    __syncthreads();
    const uint32_t len = tid < nv ? s_seg[tid + 1] - s_seg[tid] : 0u;
    const uint32_t tiles = (len + sn - 1) / sn;
    uint32_t all_tiles, total;
    (void)block_excl_scan_256(tiles, s_w, all_tiles);
    const uint32_t tpb = max(1u, (all_tiles + max_blocks - 1) / max_blocks);
    __syncthreads();   // s_w is reused by the second scan
    const uint32_t tp = block_excl_scan_256((tiles + tpb - 1) / tpb, s_w, total);
    if (tid < nv) {
        t->seg[tid] = s_seg[tid];
        t->tp[tid] = tp;
        t->kb[tid] = pairs ? (uint32_t)views[tid].tile_c : 0u;
    }
    if (tid == 0) {
        t->seg[nv] = n;
        t->tp[nv] = total;
        t->tpb = tpb;
    }
}

// Block digit histogram over the block's tiles, one LDS atomic per item, in
// HIST_COPIES counters per digit picked by lane (the high digits of a depth
// are few). Keys come four at a time. (Grouping a wave's lanes by digit first,
// with a ballot match over the digit bits, was slower for every key set here,
// the pair keys of a few busy tiles included.)
constexpr int HIST_COPIES = 4;
struct __attribute__((packed, aligned(4))) Key4 { uint32_t v[4]; };

template <int BITS, bool SEG, int SI>
__global__ void __launch_bounds__(SB)
k_radix_hist(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ n_dev, int shift,
             uint32_t* __restrict__ hist, const SegTable* __restrict__ segt, int S)
{
    constexpr int R = 1 << BITS, SN = SB * SI;
    static_assert(SI % 4 == 0, "keys are loaded four at a time");
    __shared__ uint32_t h[R * HIST_COPIES];
    __shared__ uint32_t s_tp[SEG ? SEG_MAX + 1 : 1];
    BlockItems bi;
    if constexpr (SEG) {
        if (!seg_items<SN>(segt, S, s_tp, bi)) return;
    } else {
        if (!span_items<SN>(n_dev, bi)) return;
    }
    const int tid = threadIdx.x;
    for (int d = tid; d < R * HIST_COPIES; d += SB) h[d] = 0;
    __syncthreads();
    const uint32_t copy = (uint32_t)tid & (HIST_COPIES - 1);
    auto count = [&](uint32_t key) {
        atomicAdd(&h[(((key - bi.kb) >> shift) & (R - 1)) * HIST_COPIES + copy], 1u);
    };
    const int64_t n = bi.end;
    for (uint32_t t = 0; t < bi.tiles; ++t) {
        const int64_t base = bi.first + (int64_t)t * SN;
        if (base >= n) break;
        if (base + SN <= n) {
            Key4 key[SI / 4];
#pragma unroll
            for (int k = 0; k < SI / 4; ++k)
                key[k] = *reinterpret_cast<const Key4*>(keys + base + (k * SB + tid) * 4);
#pragma unroll
            for (int k = 0; k < SI / 4; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) count(key[k].v[j]);
        } else {
            for (int64_t idx = base + tid; idx < n; idx += SB) count(keys[idx]);
        }
    }
    __syncthreads();
    for (int d = tid; d < R; d += SB) {
        uint32_t sum = 0u;
#pragma unroll
        for (int c = 0; c < HIST_COPIES; ++c) sum += h[d * HIST_COPIES + c];
        hist[(int64_t)d * bi.stride + blockIdx.x] = sum;
    }
}

// Spine of one pass: block d turns row d of the digit-major block counts
// into its exclusive prefix over blocks, in place, and writes the digit's
// total to tot[d] (the scatter adds the prefix over digits).
__global__ void __launch_bounds__(SB)
k_radix_spine(uint32_t* __restrict__ hist, uint32_t* __restrict__ tot,
              const uint32_t* __restrict__ n_dev, unsigned grid, int sn,
              const SegTable* __restrict__ segt, int S)
{
    constexpr int PER = MAX_SORT_BLOCKS / SB;
    __shared__ uint32_t wtot[SB / WAVE];
    // a segmented sort's blocks (one tile each) may exceed MAX_SORT_BLOCKS:
    // the row is taken MAX_SORT_BLOCKS at a time with a running carry
    const uint32_t nb = segt ? segt->tp[S] : sort_span(n_dev, grid, sn).nb;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
    uint32_t* row = hist + (int64_t)blockIdx.x * nb;
    uint32_t carry = 0u;
    for (uint32_t base = 0; base < nb; base += MAX_SORT_BLOCKS) {
        uint32_t v[PER], sum = 0u;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t b = base + (uint32_t)(tid * PER + k);
            v[k] = b < nb ? row[b] : 0u;
            sum += v[k];
        }
        uint32_t inc = sum;
#pragma unroll
        for (int dd = 1; dd < WAVE; dd <<= 1) {
            const uint32_t c = __shfl_up(inc, dd, WAVE);
            if (lane >= dd) inc += c;
        }
        if (lane == WAVE - 1) wtot[w] = inc;
        __syncthreads();
        uint32_t run = carry + inc - sum, all = 0u;
#pragma unroll
        for (int ww = 0; ww < SB / WAVE; ++ww) {
            if (ww < w) run += wtot[ww];
            all += wtot[ww];
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t b = base + (uint32_t)(tid * PER + k);
            if (b < nb) row[b] = run;
            run += v[k];
        }
        carry += all;
        __syncthreads();   // wtot is rewritten by the next chunk
    }
    if (tid == 0) tot[blockIdx.x] = carry;
}

// Stable scatter, one tile at a time over the block's tiles. Each wave ranks
// its own quarter of consecutive items in SI rounds of 64 (ballot
// match over the digit bits, per-wave digit counters in LDS, no block
// barrier); the block then turns the per-wave counts into digit-major local
// offsets, places the items in LDS in digit order and writes them out so
// that the items of one digit leave as a contiguous run. The block's next
// position per digit carries over from tile to tile. With vin null the
// values are the items' input positions. V2 moves a second value array
// along (vin2 null: the input positions).
template <int BITS, bool SEG, bool V2, int SI>
__global__ void __launch_bounds__(SB)
k_radix_scatter(const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                const uint32_t* __restrict__ n_dev, int shift,
                const uint32_t* __restrict__ offs, const uint32_t* __restrict__ tot,
                const SegTable* __restrict__ segt, int S,
                const uint32_t* __restrict__ vin2, uint32_t* __restrict__ vout2)
{
    constexpr int R = 1 << BITS, SN = SB * SI;
    constexpr int NW = SB / WAVE;
    constexpr int DPT = R / SB;                  // digits per thread
    __shared__ uint32_t wc[NW][R];              // per-wave digit counters, then offsets
    __shared__ uint32_t gbase[R];               // global position minus local offset
    __shared__ uint32_t wsum[NW];
    __shared__ uint32_t s_key[SN];
    __shared__ uint32_t s_val[SN];
    __shared__ uint32_t s_val2[V2 ? SN : 1];
    __shared__ uint32_t s_tp[SEG ? SEG_MAX + 1 : 1];
    BlockItems bi;
    if constexpr (SEG) {
        if (!seg_items<SN>(segt, S, s_tp, bi)) return;
    } else {
        if (!span_items<SN>(n_dev, bi)) return;
    }
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
    const int64_t n = bi.end;
    uint32_t run[DPT];   // next output position of my digits
    {
        // items of all smaller digits (exclusive scan of the digit totals;
        // segmented: of the segment's digit totals, from the segment start)
        uint32_t t[DPT], pb[DPT], sum = 0u, seg0 = 0u;
        const int64_t col = blockIdx.x;
#pragma unroll
        for (int k = 0; k < DPT; ++k) {
            const int64_t row = (int64_t)(tid * DPT + k) * bi.stride;
            if constexpr (SEG) {
                const uint32_t b0 = s_tp[bi.s], b1 = s_tp[bi.s + 1];
                const uint32_t p0 = offs[row + b0];
                const uint32_t p1 = b1 < bi.stride ? offs[row + b1] : tot[tid * DPT + k];
                t[k] = p1 - p0;
                pb[k] = offs[row + col] - p0;
            } else {
                t[k] = tot[tid * DPT + k];
                pb[k] = offs[row + col];
            }
            sum += t[k];
        }
        if constexpr (SEG) seg0 = segt->seg[bi.s];
        uint32_t inc = sum;
#pragma unroll
        for (int dd = 1; dd < WAVE; dd <<= 1) {
            const uint32_t c = __shfl_up(inc, dd, WAVE);
            if (lane >= dd) inc += c;
        }
        if (lane == WAVE - 1) wsum[w] = inc;
        __syncthreads();
        uint32_t base = inc - sum;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww)
            if (ww < w) base += wsum[ww];
#pragma unroll
        for (int k = 0; k < DPT; ++k) {
            run[k] = seg0 + base + pb[k];
            base += t[k];
        }
        __syncthreads();   // wsum is reused per tile
    }
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (WAVE - lane));
    uint32_t key[SI], val[SI], rank[SI], val2[V2 ? SI : 1];
    auto load_tile = [&](int64_t blk) {
#pragma unroll
        for (int k = 0; k < SI; ++k) {
            const int64_t idx = blk + (int64_t)w * (SI * WAVE) + k * WAVE + lane;
            const bool valid = idx < n;
            key[k] = valid ? kin[idx] : 0u;
            val[k] = valid ? (vin ? vin[idx] : (uint32_t)idx) : 0u;
            if constexpr (V2) val2[k] = valid ? (vin2 ? vin2[idx] : (uint32_t)idx) : 0u;
        }
    };
    const int64_t first = bi.first;
    load_tile(first);
    for (uint32_t t = 0; t < bi.tiles; ++t) {
        const int64_t blk = first + (int64_t)t * SN;
        if (blk >= n) break;
        const uint32_t cnt_blk = (uint32_t)min((int64_t)SN, n - blk);
#pragma unroll
        for (int k = 0; k < DPT; ++k)
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) wc[ww][tid * DPT + k] = 0u;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < SI; ++k) {
            const int64_t idx = blk + (int64_t)w * (SI * WAVE) + k * WAVE + lane;
            const bool valid = idx < n;
            const uint32_t d = ((key[k] - bi.kb) >> shift) & (R - 1);
            uint64_t m = __ballot(valid);
#pragma unroll
            for (int b = 0; b < BITS; ++b) {
                const uint64_t bb = __ballot((d >> b) & 1u);
                m &= ((d >> b) & 1u) ? bb : ~bb;
            }
            const uint32_t before = valid ? wc[w][d] : 0u;
            rank[k] = before + (uint32_t)__popcll(m & below);
            __builtin_amdgcn_wave_barrier();
            if (valid && (m & below) == 0ull) wc[w][d] = before + (uint32_t)__popcll(m);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        __syncthreads();
        // digit totals of the tile, exclusive scan over digits (digit-major)
        uint32_t tot[DPT], sum = 0u;
#pragma unroll
        for (int k = 0; k < DPT; ++k) {
            uint32_t c = 0u;
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) c += wc[ww][tid * DPT + k];
            tot[k] = c;
            sum += c;
        }
        uint32_t inc = sum;
#pragma unroll
        for (int dd = 1; dd < WAVE; dd <<= 1) {
            const uint32_t c = __shfl_up(inc, dd, WAVE);
            if (lane >= dd) inc += c;
        }
        if (lane == WAVE - 1) wsum[w] = inc;
        __syncthreads();
        uint32_t lofs = inc - sum;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww)
            if (ww < w) lofs += wsum[ww];
#pragma unroll
        for (int k = 0; k < DPT; ++k) {
            const int d = tid * DPT + k;
            gbase[d] = run[k] - lofs;
            run[k] += tot[k];
            uint32_t o = lofs;
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) {
                const uint32_t c = wc[ww][d];
                wc[ww][d] = o;
                o += c;
            }
            lofs += tot[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < SI; ++k) {
            const int64_t idx = blk + (int64_t)w * (SI * WAVE) + k * WAVE + lane;
            if (idx < n) {
                const uint32_t d = ((key[k] - bi.kb) >> shift) & (R - 1);
                const uint32_t pos = wc[w][d] + rank[k];
                s_key[pos] = key[k];
                s_val[pos] = val[k];
                if constexpr (V2) s_val2[pos] = val2[k];
            }
        }
        // the next tile's items load while this one is written out
        if (t + 1 < bi.tiles && blk + SN < n) load_tile(blk + SN);
        __syncthreads();
#pragma unroll 4
        for (uint32_t i = tid; i < cnt_blk; i += SB) {
            const uint32_t k = s_key[i];
            const uint32_t g = gbase[((k - bi.kb) >> shift) & (R - 1)] + i;
            if (kout) kout[g] = k;
            vout[g] = s_val[i];
            if constexpr (V2) vout2[g] = s_val2[i];
        }
    }
}

// Grid of a sort pass: a segmented sort's blocks take a run of tiles of
// their segment, and every segment may end in a shorter block.
inline unsigned pass_grid(int64_t cap, int S, bool seg, unsigned max_blocks, int sn)
{
    return sort_grid(cap, max_blocks, sn) + (seg ? (unsigned)S : 0u);
}

template <int BITS, bool SEG, int SI>
hipError_t radix_passes(uint32_t* keys[2], uint32_t* vals[2], int64_t cap, const uint32_t* n_dev,
                        int bits, bool iota_vals, uint32_t* hist, int* cur, hipStream_t s,
                        int shift0, const SegTable* segt, int S, bool keys_out,
                        uint32_t* const* vals2, unsigned max_blocks)
{
    constexpr int R = 1 << BITS;
    const unsigned grid = pass_grid(cap, S, SEG, max_blocks, SB * SI);
    uint32_t* tot = hist + (int64_t)R * grid;   // digit totals after the counts
    for (int shift = shift0; shift < shift0 + bits; shift += BITS) {
        hipLaunchKernelGGL((k_radix_hist<BITS, SEG, SI>), dim3(grid), dim3(SB), 0, s, keys[*cur],
                           n_dev, shift, hist, segt, S);
        hipLaunchKernelGGL(k_radix_spine, dim3(R), dim3(SB), 0, s, hist, tot, n_dev, grid,
                           SB * SI, SEG ? segt : nullptr, S);
        const uint32_t* vin = (iota_vals && shift == shift0) ? nullptr : vals[*cur];
        // the last pass writes no keys when the caller needs only the values
        uint32_t* kout = (keys_out || shift + BITS < shift0 + bits) ? keys[*cur ^ 1] : nullptr;
        if (vals2) {
            const uint32_t* vin2 = shift == shift0 ? nullptr : vals2[*cur];
            hipLaunchKernelGGL((k_radix_scatter<BITS, SEG, true, SI>), dim3(grid), dim3(SB), 0, s,
                               keys[*cur], vin, kout, vals[*cur ^ 1], n_dev, shift, hist, tot,
                               segt, S, vin2, vals2[*cur ^ 1]);
        } else {
            hipLaunchKernelGGL((k_radix_scatter<BITS, SEG, false, SI>), dim3(grid), dim3(SB), 0, s,
                               keys[*cur], vin, kout, vals[*cur ^ 1], n_dev, shift, hist, tot,
                               segt, S, nullptr, nullptr);
        }
        *cur ^= 1;
    }
    return hipGetLastError();
}

template <bool SEG>
hipError_t radix_sort_t(uint32_t* keys[2], uint32_t* vals[2], int64_t cap, const uint32_t* n_dev,
                        int bits, bool iota_vals, uint32_t* hist, int* cur, hipStream_t s,
                        int shift0, const SegTable* segt, int S, bool keys_out,
                        uint32_t* const* vals2, unsigned max_blocks)
{
    switch (digit_bits(bits)) {
    case 8:
        switch (sort_tile_items(cap, bits, vals2 != nullptr)) {
        case SB * SI_SMALL:
            return radix_passes<8, SEG, SI_SMALL>(keys, vals, cap, n_dev, bits, iota_vals, hist,
                                                  cur, s, shift0, segt, S, keys_out, vals2,
                                                  max_blocks);
        case SB * SI_MIDDLE:
            return radix_passes<8, SEG, SI_MIDDLE>(keys, vals, cap, n_dev, bits, iota_vals, hist,
                                                   cur, s, shift0, segt, S, keys_out, vals2,
                                                   max_blocks);
        default:
            break;
        }
        return radix_passes<8, SEG, SI_LARGE>(keys, vals, cap, n_dev, bits, iota_vals, hist, cur,
                                              s, shift0, segt, S, keys_out, vals2, max_blocks);
    case 9:
        return radix_passes<9, SEG, SI_LARGE>(keys, vals, cap, n_dev, bits, iota_vals, hist, cur,
                                              s, shift0, segt, S, keys_out, vals2, max_blocks);
    default:
        return radix_passes<10, SEG, SI_LARGE>(keys, vals, cap, n_dev, bits, iota_vals, hist, cur,
                                               s, shift0, segt, S, keys_out, vals2, max_blocks);
    }
}

hipError_t radix_sort(uint32_t* keys[2], uint32_t* vals[2], int64_t cap, const uint32_t* n_dev,
                      int bits, bool iota_vals, uint32_t* hist, int* which, hipStream_t s,
                      int shift0, const SegTable* segt, int S, bool keys_out,
                      uint32_t* const* vals2, unsigned max_blocks)
{
    int cur = 0;
    *which = 0;
    if (cap <= 0) return hipSuccess;
    if (bits <= 0) {
        // one bucket: the input is the result, and every item's position its own
        if (vals2)
            hipLaunchKernelGGL(k_iota, dim3((unsigned)((cap + 255) / 256)), dim3(256), 0, s,
                               vals2[0], cap);
        return hipGetLastError();
    }
    if (segt && (S < 1 || S > SEG_MAX)) return hipErrorInvalidValue;
    const hipError_t e =
        segt ? radix_sort_t<true>(keys, vals, cap, n_dev, bits, iota_vals, hist, &cur, s, shift0,
                                  segt, S, keys_out, vals2, max_blocks)
             : radix_sort_t<false>(keys, vals, cap, n_dev, bits, iota_vals, hist, &cur, s, shift0,
                                   nullptr, 0, keys_out, vals2, max_blocks);
    *which = cur;
    return e;
}

// Tile rectangles of the records in depth order, and the computation-plane
// pair count of each block of 256 (the emission scans within the block). A
// workgroup takes four blocks of 256, so each lane has four gathers in
// flight.
constexpr int GATHER_BLOCKS = 4;

__global__ void __launch_bounds__(256)
k_gather_rects(const uint32_t* __restrict__ order, const uint2* __restrict__ rect, int64_t n,
               uint2* __restrict__ rect_sorted, uint32_t* __restrict__ bsum)
{
    __shared__ uint32_t s_w[GATHER_BLOCKS][4];
    // each XCD walks a contiguous part of the order: in view-major order its
    // reads stay inside a view or two, which its L2 holds
    const uint32_t blk = xcd_block(blockIdx.x, gridDim.x);
    uint32_t o[GATHER_BLOCKS];
#pragma unroll
    for (int k = 0; k < GATHER_BLOCKS; ++k) {
        const int64_t i = ((int64_t)blk * GATHER_BLOCKS + k) * 256 + threadIdx.x;
        o[k] = i < n ? order[i] : 0u;
    }
    uint2 rc[GATHER_BLOCKS];
#pragma unroll
    for (int k = 0; k < GATHER_BLOCKS; ++k) {
        const int64_t i = ((int64_t)blk * GATHER_BLOCKS + k) * 256 + threadIdx.x;
        rc[k] = i < n ? rect[o[k]] : make_uint2(0u, 0u);
    }
#pragma unroll
    for (int k = 0; k < GATHER_BLOCKS; ++k) {
        const int64_t i = ((int64_t)blk * GATHER_BLOCKS + k) * 256 + threadIdx.x;
        if (i < n) rect_sorted[i] = rc[k];
        const uint32_t c = ((rc[k].x >> 16) - (rc[k].x & 0xFFFF)) *
                           ((rc[k].y >> 16) - (rc[k].y & 0xFFFF));
        uint32_t sum = c;
#pragma unroll
        for (int d = 1; d < WAVE; d <<= 1) sum += (uint32_t)__shfl_xor((int)sum, d, WAVE);
        // 64 counts of under 2^24 cannot wrap; larger ones saturate (a sum
        // above every capacity)
        if (__ballot(c >> 24) != 0ull) {
            unsigned long long all = c;
#pragma unroll
            for (int d = 1; d < WAVE; d <<= 1)
                all += (unsigned long long)__shfl_xor((long long)all, d, WAVE);
            sum = (uint32_t)min(all, 0xFFFFFFFFull);
        }
        if (lane_id() == 0) s_w[k][threadIdx.x / WAVE] = sum;
    }
    __syncthreads();
    if (threadIdx.x < GATHER_BLOCKS) {
        const int64_t b = (int64_t)blk * GATHER_BLOCKS + threadIdx.x;
        unsigned long long sum = 0ull;
        for (int w = 0; w < 4; ++w) sum += s_w[threadIdx.x][w];
        if (b * 256 < n) bsum[b] = (uint32_t)min(sum, 0xFFFFFFFFull);
    }
}

// Exclusive scan in place of the per-block counts, one workgroup walking
// them 8192 at a time with a running carry (coalesced loads and stores
// through LDS, each thread scanning 8 consecutive counts, the next 8192
// loading meanwhile); the total
// optionally becomes a pair count in status (0 and the overflow flag when
// above the capacity). The total has 64 bits: 8192 counts of 256 records each
// pass 2^32 where 262144 Gaussians have grown over 16384 tiles. The offsets
// have 32, unused after an overflow; the threads keep the total beside them
// (scanned in 64 bits too, the two scans of 72 views of 200k took 6 us more).
__global__ void __launch_bounds__(1024)
k_scan_blocks(uint32_t* __restrict__ a, int64_t n, int64_t cap, uint32_t* __restrict__ status,
              int slot)
{
    constexpr int ITEMS = 8, NT = 1024, NWV = NT / WAVE, CH = NT * ITEMS;
    __shared__ uint32_t s_v[CH + CH / 32];   // padded: index k -> k + k / 32
    __shared__ uint32_t s_w[NWV];
    __shared__ uint32_t s_carry;
    __shared__ unsigned long long s_all[NWV];
    auto pad = [](int k) { return k + (k >> 5); };
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
    if (tid == 0) s_carry = 0u;
    unsigned long long all = 0ull;   // the thread's counts
    // the next chunk's counts load while this one is scanned and written
    uint32_t nx[ITEMS];
    auto load = [&](int64_t base) {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int64_t idx = base + k * NT + tid;
            nx[k] = idx < n ? a[idx] : 0u;
        }
    };
    load(0);
    for (int64_t base = 0; base < n; base += CH) {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            s_v[pad(k * NT + tid)] = nx[k];
            all += nx[k];
        }
        __syncthreads();
        if (base + CH < n) load(base + CH);
        uint32_t v[ITEMS], sum = 0u;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            v[k] = s_v[pad(tid * ITEMS + k)];
            sum += v[k];
        }
        uint32_t inc = sum;
#pragma unroll
        for (int d = 1; d < WAVE; d <<= 1) {
            const uint32_t t = __shfl_up(inc, d, WAVE);
            if (lane >= d) inc += t;
        }
        if (lane == WAVE - 1) s_w[w] = inc;
        __syncthreads();
        uint32_t off = 0u, total = 0u;
#pragma unroll
        for (int k = 0; k < NWV; ++k) {
            if (k < w) off += s_w[k];
            total += s_w[k];
        }
        uint32_t run = s_carry + off + inc - sum;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            s_v[pad(tid * ITEMS + k)] = run;
            run += v[k];
        }
        __syncthreads();   // everyone has read s_carry and s_w; s_v holds the prefixes
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int64_t idx = base + k * NT + tid;
            if (idx < n) a[idx] = s_v[pad(k * NT + tid)];
        }
        if (tid == 0) s_carry += total;
        __syncthreads();
    }
    if (slot < 0) return;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1)
        all += (unsigned long long)__shfl_xor((long long)all, d, WAVE);
    if (lane == 0) s_all[w] = all;
    __syncthreads();
    if (tid == 0) {
        unsigned long long tot = 0ull;
        for (int k = 0; k < NWV; ++k) tot += s_all[k];
        const bool over = tot > (unsigned long long)cap;
        status[ST_OVERFLOW] |= over ? 1u : 0u;
        status[slot] = over ? 0u : (uint32_t)tot;
    }
}

// View of a record through a copy of the view offsets in LDS (records in
// depth order come from all views at random unless the depth sort was
// segmented by view).
constexpr int LDS_VIEWS = 512;

// Pair writes of one wave's records (a loop per record would leave most lanes
// idle and store single words: the computation plane's pairs of 16 views of
// 2M Gaussians took 831 us instead of 374). Record (lane) l
// owns the wave's pairs [ex[l], ex[l] + cnt_l) in row-major order over its
// tile rectangle (width w, first tile local0, tile row stride txn); the key
// is kadd + local, or (local << 8) | kadd for view-major imaging keys. The
// lanes take the wave's pairs 64 at a time, each finding its pair's record
// by binary search over the offsets (the largest l with ex[l] <= j owns j:
// records without pairs share their offset with the next record), so each
// store writes 64 consecutive entries whatever the spread of the counts.
struct EmitWaves {
    uint32_t ex[4][WAVE];
    uint32_t local0[4][WAVE];
    uint32_t w[4][WAVE];
    uint32_t txn[4][WAVE];
    uint32_t kadd[4][WAVE];
    uint32_t val[4][WAVE];
};

__device__ __forceinline__ void emit_wave_pairs(const EmitWaves& L, int w, uint32_t lane,
                                                uint64_t o0, uint32_t total, uint64_t lim,
                                                bool vm, uint32_t* __restrict__ pkey,
                                                uint32_t* __restrict__ pval)
{
    for (uint32_t j = lane; j < total; j += WAVE) {
        uint32_t l = 0;
#pragma unroll
        for (uint32_t step = WAVE / 2; step > 0; step >>= 1)
            if (L.ex[w][l + step] <= j) l += step;
        const uint32_t t = j - L.ex[w][l], rw = L.w[w][l];
        const uint32_t row = t / rw, col = t - row * rw;
        const uint32_t local = L.local0[w][l] + row * L.txn[w][l] + col;
        const uint64_t o = o0 + j;
        if (o < lim) {
            pkey[o] = ikey_encode(vm, (int)L.kadd[w][l], L.kadd[w][l], local);
            pval[o] = L.val[w][l];
        }
    }
}

// Offsets of a wave's records relative to the wave (ex: block-relative
// exclusive offsets), stored with the records' emission data; returns the
// wave's pair count and its first offset in *ex0.
__device__ __forceinline__ uint32_t stage_wave_records(EmitWaves& L, int w, uint32_t lane,
                                                       uint32_t ex, uint32_t cnt, uint2 rc,
                                                       uint32_t txn, uint32_t kadd, uint32_t val,
                                                       uint32_t* ex0)
{
    const uint32_t first = __shfl(ex, 0, WAVE);
    const uint32_t total = __shfl(ex + cnt, WAVE - 1, WAVE) - first;
    const uint32_t tx0 = rc.x & 0xFFFF, tx1 = rc.x >> 16, ty0 = rc.y & 0xFFFF;
    L.ex[w][lane] = ex - first;
    L.local0[w][lane] = ty0 * txn + tx0;
    L.w[w][lane] = tx1 - tx0;
    L.txn[w][lane] = txn;
    L.kadd[w][lane] = kadd;
    L.val[w][lane] = val;
    *ex0 = first;
    return total;
}

// Computation-plane pairs of the records in depth order: each record's
// (tile bucket, record) for every tile of its rectangle at its scanned
// offset, so each tile's pairs leave in depth order. A wave writes its
// records' pairs 64 at a time (see EmitWaves).
// A workgroup takes EMIT_BLOCKS blocks of 256 records, their loads in flight
// together: 4 from EMIT_LARGE records on (72 views of 200k Gaussians 107 us
// instead of 132 with one, 16 views of 2M 374 instead of 480), one below (one
// view of 500k 12 us, with 4 it is 18).
constexpr int64_t EMIT_LARGE = 2000000;

template <int EMIT_BLOCKS>
__global__ void __launch_bounds__(256)
k_emit_c(const DevView* __restrict__ views, int nv, int64_t records,
         const uint32_t* __restrict__ dval, const uint2* __restrict__ rect_sorted,
         const uint32_t* __restrict__ bscan, int64_t cap_c, const uint32_t* __restrict__ status,
         uint32_t* __restrict__ pkey, uint32_t* __restrict__ pval, uint32_t* __restrict__ seg,
         uint32_t* __restrict__ dord, uint32_t* __restrict__ poff)
{
    __shared__ uint32_t s_w[EMIT_BLOCKS][4];
    __shared__ EmitWaves L;
    __shared__ int64_t s_off[LDS_VIEWS];
    __shared__ int32_t s_tile[LDS_VIEWS], s_tx[LDS_VIEWS];
    const bool cached = nv <= LDS_VIEWS;
    const uint32_t lane = lane_id();
    const int w = threadIdx.x / WAVE;
    const int64_t b0 = (int64_t)blockIdx.x * EMIT_BLOCKS;
    uint2 rc[EMIT_BLOCKS];
    uint32_t rec[EMIT_BLOCKS], first[EMIT_BLOCKS];
#pragma unroll
    for (int k = 0; k < EMIT_BLOCKS; ++k) {
        const int64_t p = (b0 + k) * 256 + threadIdx.x;
        rc[k] = p < records ? rect_sorted[p] : make_uint2(0u, 0u);
        rec[k] = p < records ? dval[p] : 0u;
        first[k] = (b0 + k) * 256 < records ? bscan[b0 + k] : 0u;
    }
    if (cached)
        for (int k = threadIdx.x; k < nv; k += blockDim.x) {
            s_off[k] = views[k].rec_off;
            s_tile[k] = views[k].tile_c;
            s_tx[k] = views[k].txc;
        }
    const uint64_t lim = min((uint64_t)status[ST_PAIRS_C], (uint64_t)cap_c);
    const bool over = status[ST_OVERFLOW] != 0u;
    __syncthreads();
    auto view_of = [&](int64_t x) {
        int lo = 0, hi = nv - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_off[mid] <= x) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
#pragma unroll
    for (int k = 0; k < EMIT_BLOCKS; ++k) {
        const int64_t p = (b0 + k) * 256 + threadIdx.x;
        const bool in = p < records;
        const uint32_t cnt = ((rc[k].x >> 16) - (rc[k].x & 0xFFFFu)) *
                             ((rc[k].y >> 16) - (rc[k].y & 0xFFFFu));
        // offset: the block's prefix plus the counts of its records before
        uint32_t tot;
        const uint32_t ex = block_excl_scan_256(cnt, s_w[k], tot);
        // the first pair of this depth rank's record and the record
        // (deterministic mode)
        if (in && poff) poff[p] = first[k] + ex;
        if (in && dord) dord[p] = rec[k];
        uint32_t tile0 = 0u, txc = 0u;
        if (cached) {
            // view-major order (segmented depth sort): the first record of
            // each view marks where the view's pairs start
            const int v = in ? view_of(seg ? p : (int64_t)rec[k]) : 0;
            if (in && seg && s_off[v] == p) seg[v] = first[k] + ex;
            tile0 = (uint32_t)s_tile[v];
            txc = (uint32_t)s_tx[v];
        } else if (in && cnt) {
            const int v = find_view(nv, (int64_t)rec[k], [&](int j) { return views[j].rec_off; });
            tile0 = (uint32_t)views[v].tile_c;
            txc = (uint32_t)views[v].txc;
        }
        if (over) continue;
        uint32_t ex0;
        const uint32_t total =
            stage_wave_records(L, w, lane, ex, cnt, rc[k], txc, tile0, rec[k], &ex0);
        wave_lds_sync();
        emit_wave_pairs(L, w, lane, (uint64_t)first[k] + ex0, total, lim, false, pkey, pval);
        wave_lds_sync();
    }
}

// Deterministic sums over the computation-plane pairs: thread = depth rank
// p, its record's pairs are [poff[p], next) before the pair sort (one
// record's tiles, row by row); their rows of NC partials are added in that
// order. Bound by the rows' bytes. (One array per component, read one after
// the other: 132 us for both sums of 24 views of 60k Gaussians.) After a
// pair overflow the lists are empty and no partial was written: nothing is
// summed (the call's results are void anyway).
template <int NC>
__global__ void __launch_bounds__(256)
k_reduce_pairs(const uint32_t* __restrict__ dord, const uint32_t* __restrict__ poff,
               int64_t records, const uint32_t* __restrict__ status,
               const float* __restrict__ part, float* __restrict__ out, int64_t out_rec)
{
    static_assert(NC == 1 || NC % 2 == 0, "rows are read two floats at a time");
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= records || status[ST_OVERFLOW]) return;
    const uint32_t kc = status[ST_PAIRS_C];
    const uint32_t lo = min(poff[p], kc);
    const uint32_t hi = p + 1 < records ? min(poff[p + 1], kc) : kc;
    const uint32_t r = dord[p];
    float acc[NC] = {};
    for (uint32_t i = lo; i < hi; ++i) {
        const float* row = part + (uint64_t)i * NC;
        if constexpr (NC == 1) {
            acc[0] += row[0];
        } else {
#pragma unroll
            for (int k = 0; k < NC; k += 2) {
                const float2 v = *reinterpret_cast<const float2*>(row + k);
                acc[k] += v.x;
                acc[k + 1] += v.y;
            }
        }
    }
    float* o = out + (int64_t)r * out_rec;
#pragma unroll
    for (int k = 0; k < NC; ++k) o[k] = acc[k];
}

// The stored-hit pass A backward's per-pair partials, summed per record.
// A wave takes RT_ROUNDS x 256 consecutive pair positions (pre-sort order,
// where each record's pairs are contiguous); per round each lane reads the
// touched marks and rows of four consecutive positions, coalesced. The
// rows name their record, and runs of equal record over the touched rows
// are summed: in the lane first, where a run with a run of another record
// on both sides is complete and stored at once; then across the lanes, by
// a segmented scan of each lane's last run (a lane's first run closes with
// the sum carried from the lanes below), the run still open after the last
// lane carrying into the next round. A run with a run of another record
// before and after it inside the wave has every pair in the wave, and its
// sums are stored (this runs before the tiles whose hits are re-derived add
// theirs with atomics). The wave's first and last runs may go on in the
// neighbouring waves and are added with atomics, which is why the rows of
// the records pass A visits start at zero (the image backward clears them).
// Skipped after a pair overflow.
constexpr int RT_ROUNDS = 4;
constexpr int RT_LANE = 4;   // consecutive positions per lane and round
constexpr int RT_WAVE = RT_ROUNDS * WAVE * RT_LANE;

// Six segmented inclusive lane sums that share their segment flags (the
// DPP steps of seg_incl_scan).
template <int CTRL, int ROWS>
__device__ __forceinline__ void seg_sum6_step(float (&x)[6], int& f)
{
    const int fl = dpp_from<CTRL, ROWS>(f);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const float xl = __int_as_float(dpp_from<CTRL, ROWS>(__float_as_int(x[k])));
        x[k] = f ? x[k] : xl + x[k];
    }
    f |= fl;
}

__device__ __forceinline__ void seg_incl_scan6(float (&x)[6], bool head)
{
    int f = head ? 1 : 0;
    seg_sum6_step<0x111, 0xF>(x, f);
    seg_sum6_step<0x112, 0xF>(x, f);
    seg_sum6_step<0x114, 0xF>(x, f);
    seg_sum6_step<0x118, 0xF>(x, f);
    seg_sum6_step<0x142, 0xA>(x, f);
    seg_sum6_step<0x143, 0xC>(x, f);
}

__global__ void __launch_bounds__(256)
k_reduce_touched(int64_t cap, int64_t records, const uint32_t* __restrict__ status,
                 const unsigned char* __restrict__ touched, const float* __restrict__ part,
                 float* __restrict__ grad_c)
{
    constexpr uint32_t NONE = 0xFFFFFFFFu;
    const int lane = lane_id();
    const int64_t base = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE) * RT_WAVE;
    if (status[ST_OVERFLOW]) return;
    const int64_t kc = min((int64_t)status[ST_PAIRS_C], cap);
    if (base >= kc) return;   // wave-uniform
    // touched marks of the lane's four positions per round, one word each
    // (the marks array has four bytes of slack past the capacity)
    uint32_t tw[RT_ROUNDS];
#pragma unroll
    for (int r = 0; r < RT_ROUNDS; ++r) {
        const int64_t i = base + (int64_t)(r * WAVE + lane) * RT_LANE;
        uint32_t w = 0u;
        if (i < kc) {
            w = *reinterpret_cast<const uint32_t*>(touched + i);
            const int64_t left = kc - i;   // marks past the pair count are not read
            if (left < RT_LANE) w &= (1u << (8 * left)) - 1u;
        }
        tw[r] = w;
    }
    auto put = [&](uint32_t rec, const float (&v)[6], bool add) {
        if ((int64_t)rec >= records) return;
        float* g = grad_c + (int64_t)rec * GC_STRIDE;
        if (add) {
#pragma unroll
            for (int k = 0; k < 6; ++k) unsafeAtomicAdd(&g[k], v[k]);
        } else {
            reinterpret_cast<float4*>(g)[0] = make_float4(v[0], v[1], v[2], v[3]);
            reinterpret_cast<float2*>(g)[2] = make_float2(v[4], v[5]);
        }
    };
    uint32_t ckey = NONE;      // record of the run open after the last lane (wave-uniform)
    float cs[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};   // its sums so far
    bool first = true;         // no run of the wave has closed yet
#pragma unroll
    for (int r = 0; r < RT_ROUNDS; ++r) {
        const int64_t i0 = base + (int64_t)(r * WAVE + lane) * RT_LANE;
        float4 ra[RT_LANE], rb[RT_LANE];
#pragma unroll
        for (int j = 0; j < RT_LANE; ++j) {
            ra[j] = rb[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if ((tw[r] >> (8 * j)) & 0xFFu) {
                const float4* src = reinterpret_cast<const float4*>(
                    part + (uint64_t)(i0 + j) * HIT_PART_STRIDE);
                ra[j] = src[0];
                rb[j] = src[1];
            }
        }
        // the lane's runs: the first one's sums, the last (open) one's sums
        int nr = 0;
        uint32_t fkey = NONE, lkey = NONE;
        float fs[6], ls[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) fs[k] = ls[k] = 0.0f;
#pragma unroll
        for (int j = 0; j < RT_LANE; ++j) {
            if (!((tw[r] >> (8 * j)) & 0xFFu)) continue;
            const uint32_t key = __float_as_uint(rb[j].z);
            const float v[6] = {ra[j].x, ra[j].y, ra[j].z, ra[j].w, rb[j].x, rb[j].y};
            if (nr > 0 && key == lkey) {
#pragma unroll
                for (int k = 0; k < 6; ++k) ls[k] += v[k];
                continue;
            }
            if (nr == 1) {
#pragma unroll
                for (int k = 0; k < 6; ++k) fs[k] = ls[k];   // the first run ends
            } else if (nr > 1) {
                put(lkey, ls, false);   // a run between two others in the lane
            }
            if (nr == 0) fkey = key;
            ++nr;
            lkey = key;
#pragma unroll
            for (int k = 0; k < 6; ++k) ls[k] = v[k];
        }
        const uint64_t m = __ballot(nr > 0);
        if (m) {
            // the open run ends where this round's first touched row names
            // another record
            const uint32_t fk = (uint32_t)__builtin_amdgcn_readlane((int)fkey,
                                                                    __ffsll((long long)m) - 1);
            if (ckey != NONE && fk != ckey) {
                if (lane == 0) put(ckey, cs, first);
                first = false;
                ckey = NONE;
#pragma unroll
                for (int k = 0; k < 6; ++k) cs[k] = 0.0f;
            }
        }
        const uint64_t below = m & ((1ull << lane) - 1ull);
        const uint64_t above = lane == WAVE - 1 ? 0ull : m & ~((2ull << lane) - 1ull);
        // the open record at the nearest lane with rows below, and the first
        // record of the nearest one above (every lane takes part)
        const int lb = below ? 63 - __clzll((long long)below) : lane;
        const int la = above ? __ffsll((long long)above) - 1 : lane;
        const uint32_t pk_ = (uint32_t)__shfl((int)lkey, lb, WAVE);
        const uint32_t nk = (uint32_t)__shfl((int)fkey, la, WAVE);
        const uint32_t prev = below ? pk_ : ckey;
        const bool head = nr > 1 || (nr == 1 && fkey != prev);
        float x[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) x[k] = ls[k] + (lane == 0 && !head ? cs[k] : 0.0f);
        seg_incl_scan6(x, head || lane == 0);
        // the sums carried into the lane: the open run after the lane below
        float cin[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const float xb = __int_as_float(from_lane_below(__float_as_int(x[k])));
            cin[k] = lane == 0 ? cs[k] : xb;
        }
        // closings: a lane's first run when a second one starts in it, and
        // its last run when the next lane with rows starts another record
        const bool close_first = nr > 1;
        const bool close_last = nr > 0 && above && nk != lkey;
        const uint64_t cm = __ballot(close_first || close_last);
        const bool lead = first && cm && lane == __ffsll((long long)cm) - 1;
        if (close_first) {
            float t[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) t[k] = fs[k] + (prev == fkey ? cin[k] : 0.0f);
            put(fkey, t, lead);
        }
        if (close_last) put(lkey, x, lead && !close_first);
        if (cm) first = false;
        if (m) ckey = (uint32_t)__builtin_amdgcn_readlane((int)lkey, 63 - __clzll((long long)m));
#pragma unroll
        for (int k = 0; k < 6; ++k)
            cs[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[k]), WAVE - 1));
    }
    if (ckey != NONE && lane == 0) put(ckey, cs, true);
}

// Imaging-plane tile ranges (deterministic pass B): runs of equal keys in
// the sorted imaging-plane keys, indexed by the tile's imaging bucket minus
// tiles_c (keys (tile within the view << 8) | view when vm).
__global__ void __launch_bounds__(256)
k_ranges_i(const DevView* __restrict__ views, const uint32_t* __restrict__ keys,
           const uint32_t* __restrict__ status, int64_t cap_i, int64_t tiles_c, int64_t tiles_i,
           int vm, uint2* __restrict__ ranges)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = min((int64_t)status[ST_PAIRS_I], cap_i);
    if (p >= n) return;
    const uint32_t k = keys[p];
    const int64_t t = vm ? (int64_t)views[k & 0xFFu].tile_i - tiles_c + (k >> 8)
                         : (int64_t)k - tiles_c;
    if (t < 0 || t >= tiles_i) return;
    if (p == 0 || keys[p - 1] != k) ranges[t].x = (uint32_t)p;
    if (p == n - 1 || keys[p + 1] != k) ranges[t].y = (uint32_t)(p + 1);
}

// Imaging-plane pairs of the records in index order, only for the records
// whose intensity is nonzero (cnt_i = 0 otherwise); written after the
// first cap_c entries of the pair arrays.
__global__ void __launch_bounds__(256)
k_emit_i(const DevView* __restrict__ views, int nv, int64_t records,
         const uint2* __restrict__ rect_i, const uint32_t* __restrict__ cnt_i,
         const uint32_t* __restrict__ bscan, int64_t cap_c, int64_t cap_i, int vm,
         const uint32_t* __restrict__ status, uint32_t* __restrict__ pkey,
         uint32_t* __restrict__ pval)
{
    __shared__ uint32_t s_w[4];
    __shared__ EmitWaves L;
    const uint32_t lane = lane_id();
    const int w = threadIdx.x / WAVE;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t cnt = p < records ? cnt_i[p] : 0u;
    // offset: the block's prefix plus the counts of the block's records before
    uint32_t tot;
    const uint32_t ex = block_excl_scan_256(cnt, s_w, tot);
    if (status[ST_OVERFLOW]) return;
    const uint64_t lim = min((uint64_t)status[ST_PAIRS_I], (uint64_t)cap_i);
    uint2 ri = make_uint2(0u, 0u);
    uint32_t kadd = 0u, txi = 1u;
    if (cnt) {
        const int v = find_view(nv, p, [&](int k) { return views[k].rec_off; });
        const DevView& V = views[v];
        ri = rect_i[p];
        txi = (uint32_t)V.txi;
        kadd = vm ? (uint32_t)v : (uint32_t)V.tile_i;
    }
    uint32_t ex0;
    const uint32_t total =
        stage_wave_records(L, w, lane, ex, cnt, ri, txi, kadd, (uint32_t)p, &ex0);
    __syncthreads();
    emit_wave_pairs(L, w, lane, (uint64_t)bscan[blockIdx.x] + ex0, total, lim, vm != 0,
                    pkey + cap_c, pval + cap_c);
}

// The same where there are many records: a wave takes a block of 256, four to
// a lane, and compacts the few with pairs (a fifth of the vehicle's) into one
// table, from which it writes 64 pairs at a time. Per 64 records there were
// two dozen pairs to write, so most of the time went into what is done once
// per wave. A wave's pairs are a chain, though, so with many pairs a record it
// takes more records until there are enough waves: the number grows as the
// square of the pairs. Scan and emission, a wave per 64 records and per 256:
// 200k vehicle (2.0 pairs a record in the plan) 8 views 19.5 and 20.1 us, 13
// views 27.7 and 26.3, 26 views 44 and 36, 72 views 114 and 82; 200k building
// (1.6) 36 views of 50k 26 and 28, 30 views 56 and 51; 2M block (6.1) 5 views
// 113 and 118, 8 views 181 and 182, 16 views 355 and 341; 1M block in 14 views
// (2.8) 136 and 122; 100k cube (17) 20 views 32 and 37.
constexpr int64_t EMIT_I_MANY = 2000000;
constexpr double EMIT_I_WIDE = 700000.0;   // records, times the square of the pairs a record

struct EmitTable {
    uint32_t ex[4][256];       // first pair, relative to the wave's
    uint32_t local0[4][256];   // first tile
    uint32_t wr[4][256];       // rectangle width, record within the block << 16
    uint32_t txn[4][256];      // the view's tile row stride
    uint32_t kadd[4][256];     // the view's part of the key
};

__global__ void __launch_bounds__(256)
k_emit_i_many(const DevView* __restrict__ views, int nv, int64_t records,
              const uint2* __restrict__ rect_i, const uint32_t* __restrict__ cnt_i,
              const uint32_t* __restrict__ bscan, int64_t cap_c, int64_t cap_i, int vm,
              const uint32_t* __restrict__ status, uint32_t* __restrict__ pkey,
              uint32_t* __restrict__ pval)
{
    __shared__ EmitTable L;
    const uint32_t lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
    const int64_t block = (int64_t)blockIdx.x * 4 + w, p0 = block * 256, p = p0 + 4 * lane;
    if (p0 >= records || status[ST_OVERFLOW]) return;
    const uint64_t lim = min((uint64_t)status[ST_PAIRS_I], (uint64_t)cap_i);
    uint32_t cnt[4] = {0u, 0u, 0u, 0u};
    if (p + 4 <= records) {
        const uint4 c = *reinterpret_cast<const uint4*>(cnt_i + p);
        cnt[0] = c.x;
        cnt[1] = c.y;
        cnt[2] = c.z;
        cnt[3] = c.w;
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (p + k < records) cnt[k] = cnt_i[p + k];
    }
    uint2 ri[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) ri[k] = cnt[k] ? rect_i[p + k] : make_uint2(0u, 0u);
    // pairs and records with pairs of the lanes below
    const uint32_t mine = cnt[0] + cnt[1] + cnt[2] + cnt[3];
    const uint32_t some = (cnt[0] ? 1u : 0u) + (cnt[1] ? 1u : 0u) + (cnt[2] ? 1u : 0u) +
                          (cnt[3] ? 1u : 0u);
    uint32_t ex = mine, slot = some;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        const uint32_t a = __shfl_up(ex, d, WAVE), b = __shfl_up(slot, d, WAVE);
        if ((int)lane >= d) {
            ex += a;
            slot += b;
        }
    }
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)ex, WAVE - 1);
    const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)slot, WAVE - 1);
    if (total == 0u) return;
    ex -= mine;
    slot -= some;
    // the wave's records mostly lie in one view: one look-up for all
    const int v0 = find_view(nv, p0, [&](int q) { return views[q].rec_off; });
    const int64_t v0_end = v0 + 1 < nv ? views[v0 + 1].rec_off : records;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (!cnt[k]) continue;
        const int v = p + k < v0_end
                          ? v0 : find_view(nv, p + k, [&](int q) { return views[q].rec_off; });
        const uint32_t txn = (uint32_t)views[v].txi;
        L.ex[w][slot] = ex;
        L.local0[w][slot] = (ri[k].y & 0xFFFFu) * txn + (ri[k].x & 0xFFFFu);
        L.wr[w][slot] = ((ri[k].x >> 16) - (ri[k].x & 0xFFFFu)) | (4u * lane + k) << 16;
        L.txn[w][slot] = txn;
        L.kadd[w][slot] = vm ? (uint32_t)v : (uint32_t)views[v].tile_i;
        ex += cnt[k];
        ++slot;
    }
    wave_lds_sync();
    const uint64_t o0 = bscan[block];
    const uint32_t top = n > 1u ? 0x80000000u >> __clz((int)(n - 1u)) : 0u;
    for (uint32_t j = lane; j < total; j += WAVE) {
        uint32_t l = 0u;
        for (uint32_t step = top; step > 0u; step >>= 1)
            if (l + step < n && L.ex[w][l + step] <= j) l += step;
        const uint32_t t = j - L.ex[w][l], wr = L.wr[w][l], rw = wr & 0xFFFFu;
        const uint32_t row = t / rw, col = t - row * rw;
        const uint32_t local = L.local0[w][l] + row * L.txn[w][l] + col;
        const uint64_t o = o0 + j;
        if (o < lim) {
            pkey[cap_c + o] = ikey_encode(vm != 0, (int)L.kadd[w][l], L.kadd[w][l], local);
            pval[cap_c + o] = (uint32_t)p0 + (wr >> 16);
        }
    }
}

// ---- computation-plane lists of small views
// Where every view has at most VL_MAX records, three kernels take the place
// of the depth sort, the binning, the pair sort and the tile ranges: every
// record counts the records before it in its view, a workgroup per view
// counts the pairs of its tiles, and a workgroup per tile walks the view's
// records in depth order and writes its own list. The lists, their places
// and the pairs' positions in record order are those of the sorts, which are
// 23 to 29 launches of about 4 us moving a few hundred KB.
constexpr int VL_THREADS = 1024;
constexpr int VL_WAVES = VL_THREADS / WAVE;

// Depth rank of each record in its view: a workgroup takes 64 records (lane
// = record), its waves share out the keys they are compared with, which are
// scalar loads. Two VALU operations a pair, a fifth of their rate where there
// are this few waves: 7300 records in each of three views take 22 us, 1000 in one view 8, where the radix sort's
// 12 launches took 66 and 48 (and a radix sort in one workgroup's LDS 35 and
// 10).
__global__ void __launch_bounds__(VL_THREADS)
k_view_rank(const DevView* __restrict__ views, const uint32_t* __restrict__ dkey,
            const uint2* __restrict__ rect, uint32_t* __restrict__ order,
            uint2* __restrict__ rect_sorted)
{
    __shared__ uint32_t s_n[VL_WAVES][WAVE];
    const DevView& V = views[blockIdx.y];
    const int n = V.n, i0 = (int)blockIdx.x * WAVE;
    if (i0 >= n) return;
    const int64_t rec0 = V.rec_off;
    const uint32_t* keys = dkey + rec0;
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
    const int i = i0 + lane;
    const uint32_t mine = keys[min(i, n - 1)];
    const int per = (n + VL_WAVES - 1) / VL_WAVES;
    const int j0 = min(n, w * per), j1 = min(n, j0 + per);
    const int a1 = max(j0, min(j1, i0)), b1 = max(a1, min(j1, i0 + WAVE));
    uint32_t cnt = 0u;
    // equal keys keep their order: those of earlier records count as smaller
#pragma unroll 16
    for (int j = j0; j < a1; ++j) cnt += keys[j] <= mine ? 1u : 0u;
    for (int j = a1; j < b1; ++j) {
        const uint32_t k = keys[j];
        cnt += k < mine || (k == mine && j < i) ? 1u : 0u;
    }
#pragma unroll 16
    for (int j = b1; j < j1; ++j) cnt += keys[j] < mine ? 1u : 0u;
    s_n[w][lane] = cnt;
    __syncthreads();
    if (w != 0 || i >= n) return;
    const uint2 rc = rect[rec0 + i];
    uint32_t rank = 0u;
#pragma unroll
    for (int k = 0; k < VL_WAVES; ++k) rank += s_n[k][lane];
    order[rec0 + rank] = (uint32_t)(rec0 + i);
    rect_sorted[rec0 + rank] = rc;
}

// Block-wide exclusive prefix of v over VL_THREADS threads.
__device__ __forceinline__ uint32_t view_scan(uint32_t v, uint32_t* s_w, uint32_t& total)
{
    const int lane = lane_id(), w = (int)threadIdx.x / WAVE;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        const uint32_t t = __shfl_up(inc, d, WAVE);
        if (lane >= d) inc += t;
    }
    __syncthreads();   // s_w may still be read from the scan before
    if (lane == WAVE - 1) s_w[w] = inc;
    __syncthreads();
    uint32_t off = 0u;
    total = 0u;
#pragma unroll
    for (int k = 0; k < VL_WAVES; ++k) {
        if (k < w) off += s_w[k];
        total += s_w[k];
    }
    return off + inc - v;
}

// A view's pair offsets per depth rank, its tiles' ranges relative to its
// first pair, and its pair count. A tile's count is the number of rectangles
// that cover it: four marks per record in a difference array over the tiles
// (with a border), then prefix sums along the rows and the columns.
__global__ void __launch_bounds__(VL_THREADS)
k_view_counts(const DevView* __restrict__ views, const uint2* __restrict__ rect_sorted,
              uint32_t* __restrict__ rank_off, uint2* __restrict__ ranges,
              unsigned long long* __restrict__ vtot)
{
    __shared__ uint32_t s_t[VL_TILES];
    __shared__ uint32_t s_w[VL_WAVES];
    const DevView& V = views[blockIdx.x];
    const int64_t rec0 = V.rec_off;
    const int n = V.n, txc = V.txc, tyc = V.tyc;
    const int tid = threadIdx.x;
    const int gw = txc + 1, cells = gw * (tyc + 1);
    for (int k = tid; k < cells; k += VL_THREADS) s_t[k] = 0u;
    __syncthreads();
    constexpr int GRP = 8;   // records of a thread in flight, consecutive ranks
    uint32_t carry = 0u, total;
    for (int p0 = 0; p0 < n; p0 += VL_THREADS * GRP) {
        uint2 rc[GRP];
        uint32_t cnt[GRP], sum = 0u;
#pragma unroll
        for (int k = 0; k < GRP; ++k) {
            const int p = p0 + tid * GRP + k;
            rc[k] = p < n ? rect_sorted[rec0 + p] : make_uint2(0u, 0u);
        }
#pragma unroll
        for (int k = 0; k < GRP; ++k) {
            const uint32_t tx0 = rc[k].x & 0xFFFFu, tx1 = rc[k].x >> 16;
            const uint32_t y0 = rc[k].y & 0xFFFFu, y1 = rc[k].y >> 16;
            cnt[k] = (tx1 - tx0) * (y1 - y0);
            if (cnt[k]) {
                atomicAdd(&s_t[y0 * gw + tx0], 1u);
                atomicAdd(&s_t[y0 * gw + tx1], 0xFFFFFFFFu);
                atomicAdd(&s_t[y1 * gw + tx0], 0xFFFFFFFFu);
                atomicAdd(&s_t[y1 * gw + tx1], 1u);
            }
            sum += cnt[k];
        }
        uint32_t off = carry + view_scan(sum, s_w, total);
        carry += total;
#pragma unroll
        for (int k = 0; k < GRP; ++k) {
            const int p = p0 + tid * GRP + k;
            if (p < n) rank_off[rec0 + p] = off;
            off += cnt[k];
        }
    }
    if (tid == 0) vtot[blockIdx.x] = carry;
    __syncthreads();
    constexpr int STEP = 8;
    auto prefix = [&](int at, int count, int stride) {
        uint32_t acc = 0u;
        for (int i = 0; i < count; i += STEP) {
            uint32_t v[STEP];
#pragma unroll
            for (int j = 0; j < STEP; ++j) v[j] = i + j < count ? s_t[at + (i + j) * stride] : 0u;
#pragma unroll
            for (int j = 0; j < STEP; ++j) {
                acc += v[j];
                if (i + j < count) s_t[at + (i + j) * stride] = acc;
            }
        }
    };
    for (int y = tid; y < tyc; y += VL_THREADS) prefix(y * gw, txc, 1);
    __syncthreads();
    for (int x = tid; x < txc; x += VL_THREADS) prefix(x, tyc, gw);
    __syncthreads();
    // tiles in row-major order, VL_TILES / VL_THREADS to a thread
    constexpr int PER = VL_TILES / VL_THREADS;
    uint32_t c[PER];
    uint32_t sum = 0u;
    const int t0 = tid * PER, tiles = txc * tyc;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int t = t0 + k, y = t / txc;
        c[k] = t < tiles ? s_t[y * gw + t - y * txc] : 0u;
        sum += c[k];
    }
    uint32_t off = view_scan(sum, s_w, total);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (t0 + k < tiles) ranges[V.tile_c + t0 + k] = make_uint2(off, off + c[k]);
        off += c[k];
    }
}

// The list of one tile (a workgroup): which of the view's records, in depth
// order, cover it (a wave takes a quarter of them, 64 at a time), then the
// list's entries at the places k_view_counts found. Sets the pair count (0
// and the overflow flag above the capacity, with empty ranges).
constexpr int TL_WAVES = 4;
constexpr int TL_CHUNKS = VL_MAX / WAVE / TL_WAVES;   // of 64 records, per wave

__global__ void __launch_bounds__(TL_WAVES * WAVE)
k_tile_lists(const DevView* __restrict__ views, int nv, int64_t cap_c,
             const uint32_t* __restrict__ order, const uint2* __restrict__ rect_sorted,
             const uint32_t* __restrict__ rank_off, const unsigned long long* __restrict__ vtot,
             uint32_t* __restrict__ status, uint2* __restrict__ ranges,
             uint32_t* __restrict__ pkey, uint32_t* __restrict__ pval,
             uint32_t* __restrict__ ppos, uint32_t* __restrict__ dord,
             uint32_t* __restrict__ poff)
{
    __shared__ uint64_t s_m[TL_WAVES][TL_CHUNKS];
    __shared__ unsigned long long s_before[TL_WAVES], s_all[TL_WAVES];
    __shared__ uint32_t s_n[TL_WAVES];
    const int tid = threadIdx.x, lane = lane_id(), w = tid / WAVE;
    const uint32_t tile = blockIdx.x;
    const int vi = find_view(nv, (int64_t)tile, [&](int k) { return (int64_t)views[k].tile_c; });
    const DevView& V = views[vi];
    const int64_t rec0 = V.rec_off;
    const int n = V.n, chunks = (n + WAVE - 1) / WAVE, per = (chunks + TL_WAVES - 1) / TL_WAVES;
    const uint32_t local = tile - (uint32_t)V.tile_c;
    const uint32_t ty = local / (uint32_t)V.txc, tx = local - ty * (uint32_t)V.txc;
    // pairs of the views before, and of all
    unsigned long long before = 0ull, all = 0ull;
    for (int k = tid; k < nv; k += TL_WAVES * WAVE) {
        const unsigned long long c = vtot[k];
        all += c;
        if (k < vi) before += c;
    }
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        before += (unsigned long long)__shfl_xor((long long)before, d, WAVE);
        all += (unsigned long long)__shfl_xor((long long)all, d, WAVE);
    }
    auto covers = [&](uint2 rc) {
        return tx >= (rc.x & 0xFFFFu) && tx < rc.x >> 16 && ty >= (rc.y & 0xFFFFu) &&
               ty < rc.y >> 16;
    };
    const int c0 = w * per, c1 = min(chunks, c0 + per);
    uint32_t count = 0u;
    constexpr int AHEAD = 8;   // loads in flight
    for (int cb = c0; cb < c1; cb += AHEAD) {
        uint2 rc[AHEAD];
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            const int p = (cb + k) * WAVE + lane;
            rc[k] = cb + k < c1 && p < n ? rect_sorted[rec0 + p] : make_uint2(0u, 0u);
        }
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            const uint64_t m = __ballot(covers(rc[k]));
            if (lane == 0 && cb + k < c1) s_m[w][cb + k - c0] = m;
            count += (uint32_t)__popcll(m);
        }
    }
    if (lane == 0) {
        s_before[w] = before;
        s_all[w] = all;
        s_n[w] = count;
    }
    const uint2 rg = ranges[tile];
    __syncthreads();
    before = all = 0ull;
#pragma unroll
    for (int k = 0; k < TL_WAVES; ++k) {
        before += s_before[k];
        all += s_all[k];
    }
    const bool over = all > (unsigned long long)cap_c;
    if (tile == 0 && tid == 0) {
        status[ST_OVERFLOW] |= over ? 1u : 0u;
        status[ST_PAIRS_C] = over ? 0u : (uint32_t)all;
    }
    if (tid == 0)
        ranges[tile] = over || rg.y <= rg.x ? make_uint2(0u, 0u)
                                            : make_uint2((uint32_t)before + rg.x,
                                                         (uint32_t)before + rg.y);
    // (deterministic mode) the first pair and the record of every depth rank:
    // the view's tiles take equal parts
    if (poff) {
        const int64_t tiles = (int64_t)V.txc * V.tyc;
        const int p1 = (int)((int64_t)n * (local + 1) / tiles);
        for (int p = (int)((int64_t)n * local / tiles) + tid; p < p1; p += TL_WAVES * WAVE) {
            poff[rec0 + p] = (uint32_t)before + rank_off[rec0 + p];
            dord[rec0 + p] = order[rec0 + p];
        }
    }
    if (over) return;
    uint32_t o = (uint32_t)before + rg.x;
    for (int k = 0; k < w; ++k) o += s_n[k];
    const uint64_t lower = (1ull << lane) - 1ull;
    for (int cb = c0; cb < c1; cb += AHEAD) {
        uint64_t m[AHEAD];
        uint32_t rec[AHEAD], off[AHEAD];
        uint2 rc[AHEAD];
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            m[k] = cb + k < c1 ? s_m[w][cb + k - c0] : 0ull;
            const int64_t p = rec0 + (cb + k) * WAVE + lane;
            rec[k] = off[k] = 0u;
            rc[k] = make_uint2(0u, 0u);
            if (m[k] >> lane & 1ull) {
                rec[k] = order[p];
                if (ppos) {
                    rc[k] = rect_sorted[p];
                    off[k] = rank_off[p];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            if (m[k] >> lane & 1ull) {
                const uint32_t at = o + (uint32_t)__popcll(m[k] & lower);
                pkey[at] = tile;
                pval[at] = rec[k];
                if (ppos) {
                    const uint32_t rx = rc[k].x & 0xFFFFu, rw = (rc[k].x >> 16) - rx;
                    ppos[at] = (uint32_t)before + off[k] + (ty - (rc[k].y & 0xFFFFu)) * rw + tx - rx;
                }
            }
            o += (uint32_t)__popcll(m[k]);
        }
    }
}

// Tile ranges from the sorted bucket ids, four keys per thread (one 16-byte
// load when the four are in range) and the neighbours of the first and last.
__global__ void __launch_bounds__(256)
k_ranges(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ n_dev, int64_t buckets,
         uint2* __restrict__ ranges)
{
    const int64_t p0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    const int64_t n = *n_dev;
    if (p0 >= n) return;
    uint32_t k[4];
    if (p0 + 4 <= n) {
        const uint4 q = *reinterpret_cast<const uint4*>(keys + p0);
        k[0] = q.x; k[1] = q.y; k[2] = q.z; k[3] = q.w;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) k[i] = p0 + i < n ? keys[p0 + i] : 0xFFFFFFFFu;
    }
    const uint32_t before = p0 > 0 ? keys[p0 - 1] : 0xFFFFFFFFu;
    const uint32_t after = p0 + 4 < n ? keys[p0 + 4] : 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t p = p0 + i;
        if (p >= n || k[i] >= buckets) continue;
        const uint32_t prev = i == 0 ? before : k[i - 1];
        const uint32_t next = i == 3 ? after : k[i + 1];
        if (p == 0 || prev != k[i]) ranges[k[i]].x = (uint32_t)p;
        if (p == n - 1 || next != k[i]) ranges[k[i]].y = (uint32_t)(p + 1);
    }
}

inline unsigned grid256(int64_t n) { return (unsigned)((n + 255) / 256); }

// Fills and small host tables of a call in one launch. The tables come
// through the kernel arguments: the runtime copies the argument block at
// launch, so the host buffer may be released as soon as the launch returns
// and the copy stays stream-ordered. A block per SETUP_WORDS words filled
// (16-byte stores where aligned), the first one also stores the tables. Each
// fill and table alone was a launch of 2 to 5 us (a forward of 1000 Gaussians
// with 11 launches fewer: 86 -> 63 us).
constexpr int SETUP_DATA = 3072;
constexpr int SETUP_WORDS = 4096;
constexpr int SETUP_PIECES = 2;
struct SetupArgs {
    SetupFill fill[Setup::FILLS];
    uint32_t first[Setup::FILLS + 1];   // first block of each fill, then their count
    int32_t nfill;
    int32_t words[SETUP_PIECES];
    uint32_t* dst[SETUP_PIECES];
    uint32_t data[SETUP_DATA / 4];
};

__global__ void __launch_bounds__(256) k_setup(SetupArgs a)
{
    const int tid = threadIdx.x;
    if (blockIdx.x == 0) {
        for (int i = tid; i < a.words[0]; i += 256) a.dst[0][i] = a.data[i];
        for (int i = tid; i < a.words[1]; i += 256) a.dst[1][i] = a.data[a.words[0] + i];
    }
    const uint32_t b = blockIdx.x;
    if (b >= a.first[a.nfill]) return;
    int k = 0;
    while (b >= a.first[k + 1]) ++k;
    const uint32_t v = a.fill[k].v;
    const int64_t at = (int64_t)(b - a.first[k]) * SETUP_WORDS;
    uint32_t* p = a.fill[k].p + at;
    const int n = (int)min(a.fill[k].n - at, (int64_t)SETUP_WORDS);
    int done = 0;
    if ((reinterpret_cast<uintptr_t>(p) & 15) == 0) {
        for (int i = tid; i < n / 4; i += 256) reinterpret_cast<uint4*>(p)[i] = make_uint4(v, v, v, v);
        done = n & ~3;
    }
    for (int i = done + tid; i < n; i += 256) p[i] = v;
}

}  // namespace

void Setup::fill(uint32_t* p, uint32_t v, int64_t n)
{
    if (n > 0 && nfill < FILLS) fills[nfill] = SetupFill{p, n, v};
    if (n > 0) ++nfill;
}

void Setup::table(void* dst, const void* src, size_t bytes)
{
    if (ntable < TABLES) tables[ntable] = Table{dst, src, bytes};
    ++ntable;
}

hipError_t Setup::launch(hipStream_t s) const
{
    if (nfill > FILLS || ntable > TABLES) return hipErrorInvalidValue;
    SetupArgs a;
    a.nfill = nfill;
    a.first[0] = 0;
    for (int k = 0; k < nfill; ++k) {
        const int64_t blocks = (fills[k].n + SETUP_WORDS - 1) / SETUP_WORDS;
        if (a.first[k] + blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
        a.fill[k] = fills[k];
        a.first[k + 1] = a.first[k] + (uint32_t)blocks;
    }
    int t = 0;
    size_t off = 0;
    bool any = nfill > 0;
    // the fills go with the first of as many launches as the tables need
    do {
        size_t used = 0;
        int pieces = 0;
        for (int k = 0; k < SETUP_PIECES; ++k) {
            a.words[k] = 0;
            a.dst[k] = nullptr;
        }
        while (t < ntable && pieces < SETUP_PIECES && used < SETUP_DATA) {
            const size_t n = std::min(tables[t].bytes - off, (size_t)SETUP_DATA - used);
            if (n & 3) return hipErrorInvalidValue;
            memcpy(reinterpret_cast<char*>(a.data) + used,
                   static_cast<const char*>(tables[t].src) + off, n);
            a.dst[pieces] = reinterpret_cast<uint32_t*>(static_cast<char*>(tables[t].dst) + off);
            a.words[pieces++] = (int32_t)(n / 4);
            used += n;
            off += n;
            if (off == tables[t].bytes) {
                ++t;
                off = 0;
            }
            any = true;
        }
        if (any)
            hipLaunchKernelGGL(k_setup, dim3(std::max(a.first[a.nfill], 1u)), dim3(256), 0, s, a);
        a.nfill = 0;
    } while (t < ntable);
    return hipGetLastError();
}

size_t radix_hist_words(int64_t cap)
{
    // counts (up to one block per tile and a partial tile per segment),
    // digit totals
    return (size_t)MAX_RADIX * (pass_grid(cap > 0 ? cap : 1, SEG_MAX, true, MAX_SORT_BLOCKS, SB * SI_LARGE) + 1);
}

int radix_passes_for(int bits)
{
    if (bits <= 0) return 0;
    const int d = digit_bits(bits);
    return (bits + d - 1) / d;
}

hipError_t launch_radix_sort_u32(uint32_t* keys[2], uint32_t* vals[2], int64_t cap,
                                 const uint32_t* n_dev, int bits, bool iota_vals, uint32_t* hist,
                                 int* which, hipStream_t s, int shift0, const SegTable* segt,
                                 int S, bool keys_out, uint32_t* const* vals2,
                                 unsigned max_blocks)
{
    if (max_blocks < SB || max_blocks > MAX_SORT_BLOCKS) return hipErrorInvalidValue;
    return radix_sort(keys, vals, cap, n_dev, bits, iota_vals, hist, which, s, shift0, segt, S,
                      keys_out, vals2, max_blocks);
}

hipError_t launch_seg_setup(const DevView* views, int nv, int64_t records, const uint32_t* n_dev,
                            int64_t cap, int bits, bool pairs, bool positions, SegTable* segt,
                            hipStream_t s, unsigned max_blocks)
{
    if (nv < 1 || nv > SEG_MAX) return hipErrorInvalidValue;
    if (max_blocks < SB || max_blocks > MAX_SORT_BLOCKS) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_seg_setup, dim3(1), dim3(SEG_MAX), 0, s, views, nv, records, n_dev,
                       pairs ? 1 : 0, (uint32_t)max_blocks,
                       (uint32_t)sort_tile_items(cap, bits, positions), segt);
    return hipGetLastError();
}

namespace {
// dst |= src[0] (one word; for accumulating a status flag on the device)
__global__ void k_or_word(const uint32_t* __restrict__ src, uint32_t* __restrict__ dst)
{
    if (threadIdx.x == 0) {
        const uint32_t v = src[0];
        if (v) dst[0] |= v;
    }
}
}  // namespace

hipError_t launch_or_word(const uint32_t* src, uint32_t* dst, hipStream_t s)
{
    hipLaunchKernelGGL(k_or_word, dim3(1), dim3(64), 0, s, src, dst);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3(grid256(n)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_gather_rects(const uint32_t* order, const uint2* rect, int64_t n,
                               uint2* rect_sorted, uint32_t* bsum, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const unsigned grid = (unsigned)((n + 256 * GATHER_BLOCKS - 1) / (256 * GATHER_BLOCKS));
    hipLaunchKernelGGL(k_gather_rects, dim3(grid), dim3(256), 0, s, order, rect, n, rect_sorted,
                       bsum);
    return hipGetLastError();
}

hipError_t launch_scan_blocks(uint32_t* bsum, int64_t n, int64_t cap, uint32_t* status,
                              int status_slot, hipStream_t s)
{
    hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(1024), 0, s, bsum, n, cap, status,
                       status_slot);
    return hipGetLastError();
}

hipError_t launch_emit_pairs_c(const DevView* views, int nv, int64_t records,
                               const uint32_t* dval_sorted, const uint2* rect_sorted,
                               const uint32_t* bscan_c, int64_t cap_c, const uint32_t* status,
                               uint32_t* pkey, uint32_t* pval, uint32_t* seg, uint32_t* dord,
                               uint32_t* poff, hipStream_t s)
{
    if (records <= 0) return hipSuccess;
    if (seg && nv > LDS_VIEWS) return hipErrorInvalidValue;
    const bool large = records >= EMIT_LARGE;
    const int64_t per = large ? 4 : 1;
    hipLaunchKernelGGL(large ? k_emit_c<4> : k_emit_c<1>, dim3(grid256((records + per - 1) / per)),
                       dim3(256), 0, s, views, nv, records, dval_sorted, rect_sorted, bscan_c,
                       cap_c, status, pkey, pval, seg, dord, poff);
    return hipGetLastError();
}

hipError_t launch_reduce_pairs(const uint32_t* dord, const uint32_t* poff, int64_t records,
                               const uint32_t* status, const float* part, int ncomp, float* out,
                               int64_t out_rec, hipStream_t s)
{
    if (records <= 0) return hipSuccess;
    if (ncomp == 1)
        hipLaunchKernelGGL(k_reduce_pairs<1>, dim3(grid256(records)), dim3(256), 0, s, dord, poff,
                           records, status, part, out, out_rec);
    else if (ncomp == PART_G)
        hipLaunchKernelGGL(k_reduce_pairs<PART_G>, dim3(grid256(records)), dim3(256), 0, s, dord,
                           poff, records, status, part, out, out_rec);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_reduce_touched(int64_t cap, int64_t records, const uint32_t* status,
                                 const unsigned char* touched, const float* part, float* grad_c,
                                 hipStream_t s)
{
    if (records <= 0 || cap <= 0) return hipSuccess;
    constexpr int64_t per_block = 4 * (int64_t)RT_WAVE;   // four waves of 256 threads
    const int64_t grid = (cap + per_block - 1) / per_block;
    if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_reduce_touched, dim3((unsigned)grid), dim3(256), 0, s, cap, records,
                       status, touched, part, grad_c);
    return hipGetLastError();
}

hipError_t launch_ranges_i(const DevView* views, const uint32_t* keys, const uint32_t* status,
                           int64_t cap_i, int64_t tiles_c, int64_t tiles_i, bool vm,
                           uint2* ranges, hipStream_t s)
{
    hipError_t e = launch_fill_u32((uint32_t*)ranges, 0u, 2 * tiles_i, s);
    if (e != hipSuccess || cap_i <= 0) return e;
    hipLaunchKernelGGL(k_ranges_i, dim3(grid256(cap_i)), dim3(256), 0, s, views, keys, status,
                       cap_i, tiles_c, tiles_i, vm ? 1 : 0, ranges);
    return hipGetLastError();
}

hipError_t launch_emit_pairs_i(const DevView* views, int nv, int64_t records,
                               const uint2* rect_i, const uint32_t* cnt_i,
                               const uint32_t* bscan_i, int64_t cap_c, int64_t cap_i, bool vm,
                               const uint32_t* status, uint32_t* pkey, uint32_t* pval,
                               hipStream_t s)
{
    if (records <= 0) return hipSuccess;
    const double pairs = (double)cap_i / (double)records;
    const bool many =
        records >= EMIT_I_MANY && (double)records >= EMIT_I_WIDE * pairs * pairs;
    const int64_t per = many ? 4 : 1;
    hipLaunchKernelGGL(many ? k_emit_i_many : k_emit_i, dim3(grid256((records + per - 1) / per)),
                       dim3(256), 0, s, views, nv, records, rect_i, cnt_i, bscan_i, cap_c, cap_i,
                       vm ? 1 : 0, status, pkey, pval);
    return hipGetLastError();
}

hipError_t launch_tile_ranges(const uint32_t* keys, int64_t cap, const uint32_t* n_dev,
                              int64_t buckets, uint2* ranges, hipStream_t s)
{
    if (cap <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_ranges, dim3(grid256((cap + 3) / 4)), dim3(256), 0, s, keys, n_dev,
                       buckets, ranges);
    return hipGetLastError();
}

hipError_t launch_view_lists(const DevView* views, int nv, int64_t max_records, int64_t tiles_c,
                             int64_t cap_c, const uint32_t* dkey, const uint2* rect,
                             uint32_t* order, uint2* rect_sorted, uint32_t* rank_off,
                             unsigned long long* vtot, uint32_t* status, uint2* ranges,
                             uint32_t* pkey, uint32_t* pval, uint32_t* ppos, uint32_t* dord,
                             uint32_t* poff, hipStream_t s)
{
    if (nv < 1 || max_records > VL_MAX) return hipErrorInvalidValue;
    if (max_records > 0)
        hipLaunchKernelGGL(k_view_rank, dim3((unsigned)((max_records + WAVE - 1) / WAVE),
                                             (unsigned)nv),
                           dim3(VL_THREADS), 0, s, views, dkey, rect, order, rect_sorted);
    hipLaunchKernelGGL(k_view_counts, dim3((unsigned)nv), dim3(VL_THREADS), 0, s, views,
                       rect_sorted, rank_off, ranges, vtot);
    hipLaunchKernelGGL(k_tile_lists, dim3((unsigned)tiles_c), dim3(TL_WAVES * WAVE), 0, s, views,
                       nv, cap_c, order, rect_sorted, rank_off, vtot, status, ranges, pkey, pval,
                       ppos, dord, poff);
    return hipGetLastError();
}

}  // namespace sdgr
