// Rasterizers of the SAR Gaussian splatting renderer (paper Sec. II-A,
// scattering intensity and imaging; Sec. II-B, their gradients).
//
// Computation plane (order matters: front-to-back along each ray)
//   One wave64 owns one 8x8 tile, or a workgroup does where few tiles would
//   leave the device idle: lane l handles ray (l % 8, l / 8); only non-empty
//   tiles run, longest lists first. Every
//   (tile, Gaussian) pair carries a 64-bit mask of the tile cells inside the
//   footprint ellipse, and every 64 consecutive pairs of the sorted array (a
//   chunk) the OR of their masks (k_pair_masks). The tile's depth-sorted list
//   is walked chunk by chunk: chunks whose summary misses every ray still in
//   play are skipped unread, the next chunks' masks are prefetched, and in
//   those that are read the 64 masks are bit-transposed (lane = ray: which
//   entries cover my cell) and the hits compacted, so that lane = hit.
//   pass A forward : alpha = 1 - exp(-kappa f), A_i += alpha T, T *= exp(-kappa f);
//                    per-entry sums in LDS (FP64 atomics: one takes 8 to 27
//                    cycles for a wave, an FP32 one 192), one global atomic
//                    per (tile, Gaussian); a ray leaves after its optical
//                    depth reaches tau_max.
//   pass A backward: back to front from each ray's last contributing entry:
//                    tau -= kappa f, T = exp(-tau), dL/dalpha = T (c - U),
//                    U <- c alpha + (1 - alpha) U (division-free), c = P dL/dI.
// Imaging plane (order-free additive layover)
//   pass B forward : fixed 128-entry segments of the sorted (tile, Gaussian)
//                    pair array, one wave each (balanced however long a
//                    tile's list is); footprint masks computed on the fly
//                    and bit-transposed, so lane = pixel sums only the
//                    entries covering it; partial pixel sums are added to
//                    the image at tile boundaries. Small calls and the
//                    deterministic mode: a workgroup per tile.
//   pass B backward: one thread per record walks its footprint ellipse and
//                    gathers dL/dS (no atomics).
#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "common.hpp"

namespace sdgr {
namespace {

constexpr uint32_t B_SEGMENT = 128;    // pair entries per pass-B forward wave

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) v = max(v, (uint32_t)__shfl_xor((int)v, d, WAVE));
    return v;
}

// Number of set bits of `mask` below this lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// ---- wave64 data movement without the LDS crossbar --------------------
// Lane i reads lane i ^ S: S = 32 and 16 through the gfx950 permlane swaps,
// S = 8 by a DPP row rotation, S = 4 by DPP row shifts, S = 2 and 1 by DPP
// quad permutes.
template <int S>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v)
{
    const int lane = lane_id();
    if constexpr (S == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return lane < 32 ? r[1] : r[0];
    } else if constexpr (S == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (lane & 16) ? r[0] : r[1];
    } else if constexpr (S == 8) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true);
    } else if constexpr (S == 4) {
        const uint32_t from_below = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
        const uint32_t from_above = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x104, 0xF, 0xF, false);
        return (lane & 4) ? from_below : from_above;
    } else if constexpr (S == 2) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);
    } else {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);
    }
}

template <int S>
__device__ __forceinline__ uint64_t xor_lane64(uint64_t v)
{
    return ((uint64_t)xor_lane<S>((uint32_t)(v >> 32)) << 32) | xor_lane<S>((uint32_t)v);
}

// 64x64 bit-matrix transpose across the wave: on return, bit j of lane i is
// bit i of lane j's input. Recursive block swap: at step s, lanes i and i ^ s
// exchange the s-wide bit blocks that sit off the diagonal. It is bound by
// instruction issue (few waves share a SIMD in the rasterizers), so each step
// uses what moves most per instruction: the two 32-bit halves are exchanged
// whole by one permlane32 swap, the 16-bit blocks of both words by byte
// permutes around one permlane16 swap, whose unpacking is the packing of the
// 8-bit step (byte selectors that depend on the lane, one DPP rotation), and
// the blocks within bytes by a DPP move, a rotate and a bit-field insert per
// word: 30 instructions where shifting, masking and selecting both forms of
// every block took about 120. N transposes go step by step together, so that
// no instruction waits on the one before it.
struct TransposeLane {
    uint32_t send8, keep8, lo8, hi8;   // byte selectors of the 8-bit step
    uint32_t rot4, rot2, rot1;         // rotations of the partner's word
    uint32_t m4, m2, m1;               // bits of the own word that stay
};

__device__ __forceinline__ TransposeLane transpose_lane()
{
    const int l = lane_id();
    const bool u8 = (l & 8) != 0, u4 = (l & 4) != 0, u2 = (l & 2) != 0, u1 = (l & 1) != 0;
    TransposeLane t;
    t.send8 = u8 ? 0x06020400u : 0x07030501u;
    t.keep8 = u8 ? 0x07030501u : 0x06020400u;
    t.lo8 = u8 ? 0x01050004u : 0x05010400u;
    t.hi8 = u8 ? 0x03070206u : 0x07030602u;
    t.rot4 = u4 ? 4u : 28u;
    t.rot2 = u2 ? 2u : 30u;
    t.rot1 = u1 ? 1u : 31u;
    t.m4 = u4 ? 0xF0F0F0F0u : 0x0F0F0F0Fu;
    t.m2 = u2 ? 0xCCCCCCCCu : 0x33333333u;
    t.m1 = u1 ? 0xAAAAAAAAu : 0x55555555u;
    return t;
}

// Own blocks of word x where `keep` is set, the partner's (lane ^ S) moved
// next to them elsewhere.
template <int S>
__device__ __forceinline__ uint32_t transpose_bits(uint32_t x, uint32_t keep, uint32_t rot)
{
    uint32_t r;
    if constexpr (S == 4) {
        // lane + 4 in banks 0 and 2 of each row, lane - 4 in banks 1 and 3
        r = (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x104, 0xF, 0x5, false);
        r = (uint32_t)__builtin_amdgcn_update_dpp((int)r, (int)x, 0x114, 0xF, 0xA, false);
    } else {
        r = xor_lane<S>(x);
    }
    r = __builtin_amdgcn_alignbit(r, r, rot);
    return (x & keep) | (r & ~keep);   // one three-operand bit operation
}

template <int N>
__device__ __forceinline__ void transpose64_n(uint64_t (&v)[N], const TransposeLane& t)
{
    uint32_t lo[N], hi[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const auto r = __builtin_amdgcn_permlane32_swap((uint32_t)v[i], (uint32_t)(v[i] >> 32),
                                                        false, false);
        lo[i] = r[0];
        hi[i] = r[1];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        // low halves of both words, high halves of both words
        const uint32_t a = __builtin_amdgcn_perm(hi[i], lo[i], 0x05040100u);
        const uint32_t b = __builtin_amdgcn_perm(hi[i], lo[i], 0x07060302u);
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        lo[i] = r[0];
        hi[i] = r[1];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint32_t s = __builtin_amdgcn_perm(hi[i], lo[i], t.send8);
        const uint32_t k = __builtin_amdgcn_perm(hi[i], lo[i], t.keep8);
        const uint32_t r = xor_lane<8>(s);
        lo[i] = __builtin_amdgcn_perm(r, k, t.lo8);
        hi[i] = __builtin_amdgcn_perm(r, k, t.hi8);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        lo[i] = transpose_bits<4>(lo[i], t.m4, t.rot4);
        hi[i] = transpose_bits<4>(hi[i], t.m4, t.rot4);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        lo[i] = transpose_bits<2>(lo[i], t.m2, t.rot2);
        hi[i] = transpose_bits<2>(hi[i], t.m2, t.rot2);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        lo[i] = transpose_bits<1>(lo[i], t.m1, t.rot1);
        hi[i] = transpose_bits<1>(hi[i], t.m1, t.rot1);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = ((uint64_t)hi[i] << 32) | lo[i];
}

__device__ __forceinline__ uint64_t transpose64(uint64_t v, const TransposeLane& t)
{
    uint64_t one[1] = {v};
    transpose64_n(one, t);
    return one[0];
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
    v += xor_lane64<1>(v);
    v += xor_lane64<2>(v);
    v += xor_lane64<4>(v);
    v += xor_lane64<8>(v);
    v += xor_lane64<16>(v);
    v += xor_lane64<32>(v);
    return v;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ void or_step(uint32_t& x)
{
    x |= (uint32_t)dpp_from<CTRL, ROWS>((int)x);
}

// OR of a word over the lanes up to each one; the last lane holds the wave's.
__device__ __forceinline__ uint32_t or_scan_u32(uint32_t x)
{
    or_step<0x111, 0xF>(x);
    or_step<0x112, 0xF>(x);
    or_step<0x114, 0xF>(x);
    or_step<0x118, 0xF>(x);
    or_step<0x142, 0xA>(x);
    or_step<0x143, 0xC>(x);
    return x;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ void seg_affine_step(float& a, float& b, int& f)
{
    // lanes without a source see the identity map (a = 1, b = 0)
    const float al = __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(1.0f), __float_as_int(a), CTRL, ROWS, 0xF, false));
    const float bl = __int_as_float(dpp_from<CTRL, ROWS>(__float_as_int(b)));
    const int fl = dpp_from<CTRL, ROWS>(f);
    if (!f) {
        b = a * bl + b;
        a = a * al;
    }
    f |= fl;
}

// Segmented inclusive composition of the affine maps U -> a U + b held by
// the lanes, earlier lanes applied first: lane l gets f_l o ... o f_head.
__device__ __forceinline__ void seg_incl_affine(float& a, float& b, bool head)
{
    int f = head ? 1 : 0;
    seg_affine_step<0x111, 0xF>(a, b, f);
    seg_affine_step<0x112, 0xF>(a, b, f);
    seg_affine_step<0x114, 0xF>(a, b, f);
    seg_affine_step<0x118, 0xF>(a, b, f);
    seg_affine_step<0x142, 0xA>(a, b, f);
    seg_affine_step<0x143, 0xC>(a, b, f);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ void sum_step_u32(uint32_t& x)
{
    x += (uint32_t)dpp_from<CTRL, ROWS>((int)x);
}

// Wave totals of N values at once (inclusive scans, step by step over all
// of them, read at the last lane).
template <int N>
__device__ __forceinline__ void wave_total_u32_n(uint32_t (&x)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) sum_step_u32<0x111, 0xF>(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) sum_step_u32<0x112, 0xF>(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) sum_step_u32<0x114, 0xF>(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) sum_step_u32<0x118, 0xF>(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) sum_step_u32<0x142, 0xA>(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) sum_step_u32<0x143, 0xC>(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = (uint32_t)__builtin_amdgcn_readlane((int)x[i], WAVE - 1);
}

// Exclusive prefix sum of small unsigned counts over the 64 lanes.
__device__ __forceinline__ uint32_t wave_excl_scan_u32(uint32_t v)
{
    uint32_t x = v;
    sum_step_u32<0x111, 0xF>(x);
    sum_step_u32<0x112, 0xF>(x);
    sum_step_u32<0x114, 0xF>(x);
    sum_step_u32<0x118, 0xF>(x);
    sum_step_u32<0x142, 0xA>(x);
    sum_step_u32<0x143, 0xC>(x);
    return x - v;
}

// Direct global-to-LDS loads (gfx950): every lane's 16 (or 4) bytes land
// at dst + lane * 16 (or 4) without passing through registers, so a batch's
// gathers all stay in flight until one wait.
__device__ __forceinline__ void load16_to_lds(const void* src, void* dst_wave_base)
{
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)src,
                                     (void __attribute__((address_space(3)))*)dst_wave_base,
                                     16, 0, 0);
}

__device__ __forceinline__ void load4_to_lds(const void* src, void* dst_wave_base)
{
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)src,
                                     (void __attribute__((address_space(3)))*)dst_wave_base,
                                     4, 0, 0);
}

__device__ __forceinline__ void wait_all_memory()
{
    __builtin_amdgcn_s_waitcnt(0);
}

// Gather of one 32-byte record per lane (every lane takes part, each with a
// valid id). A lane's two 16-byte loads would touch one line twice, and the L1
// stalls on a line that is still in flight, so the lanes of a pair load the
// two halves of the even lane's record, then those of the odd lane's: both
// halves of a line in one instruction, and swap what belongs to the other.
__device__ __forceinline__ float4 dpp_pair_swap(float4 v)
{
    return make_float4(__uint_as_float(xor_lane<1>(__float_as_uint(v.x))),
                       __uint_as_float(xor_lane<1>(__float_as_uint(v.y))),
                       __uint_as_float(xor_lane<1>(__float_as_uint(v.z))),
                       __uint_as_float(xor_lane<1>(__float_as_uint(v.w))));
}

struct RecPair { float4 a, b; };   // halves of the even and of the odd lane's record

__device__ __forceinline__ RecPair load_rec_pair(const CRec* __restrict__ crec, uint32_t id)
{
    const uint32_t ie = (uint32_t)__builtin_amdgcn_mov_dpp((int)id, 0xA0, 0xF, 0xF, true);
    const uint32_t io = (uint32_t)__builtin_amdgcn_mov_dpp((int)id, 0xF5, 0xF, 0xF, true);
    const float4* base = reinterpret_cast<const float4*>(crec);
    const uint32_t half = (uint32_t)lane_id() & 1u;
    return RecPair{base[2u * (uint64_t)ie + half], base[2u * (uint64_t)io + half]};
}

// The records of the lanes' ids straight into LDS, both halves of lane i's at
// dst[2 i] and dst[2 i + 1]: a pair of lanes loads the halves of one record,
// so each line is touched by one instruction.
__device__ __forceinline__ void load_recs_to_lds(const CRec* __restrict__ crec, uint32_t id,
                                                 float4* dst)
{
    const int lane = lane_id();
    const float4* base = reinterpret_cast<const float4*>(crec);
    const uint32_t lo = (uint32_t)__shfl((int)id, lane / 2, WAVE);
    const uint32_t hi = (uint32_t)__shfl((int)id, WAVE / 2 + lane / 2, WAVE);
    load16_to_lds(&base[2u * (uint64_t)lo + (lane & 1)], dst);
    load16_to_lds(&base[2u * (uint64_t)hi + (lane & 1)], dst + WAVE);
}

__device__ __forceinline__ CRec own_rec(const RecPair& p)
{
    const bool odd = (lane_id() & 1) != 0;
    auto pick = [&](const float4& x, const float4& y) {
        return make_float4(odd ? x.x : y.x, odd ? x.y : y.y, odd ? x.z : y.z, odd ? x.w : y.w);
    };
    const float4 other = dpp_pair_swap(pick(p.a, p.b));
    return CRec{pick(other, p.a), pick(p.b, other)};
}

struct TileCell {
    int v;
    int tx, ty;
    int col, row;
    bool inside;
};

// Tile coordinates of a bucket id (computation-plane ids first, then
// imaging-plane ids), and this lane's cell.
__device__ __forceinline__ TileCell tile_cell(const DevView* views, int nv, int64_t bucket,
                                              bool comp_plane)
{
    TileCell t;
    if (comp_plane)
        t.v = find_view(nv, bucket, [&](int k) { return (int64_t)views[k].tile_c; });
    else
        t.v = find_view(nv, bucket, [&](int k) { return (int64_t)views[k].tile_i; });
    const DevView& V = views[t.v];
    const int64_t local = bucket - (comp_plane ? V.tile_c : V.tile_i);
    const int tx_n = comp_plane ? V.txc : V.txi;
    t.tx = (int)(local % tx_n);
    t.ty = (int)(local / tx_n);
    const int lane = lane_id();
    t.col = t.tx * TILE + (lane & (TILE - 1));
    t.row = t.ty * TILE + (lane / TILE);
    t.inside = comp_plane ? (t.col < V.Wc && t.row < V.Hc) : (t.col < V.W && t.row < V.H);
    return t;
}

// Tile coordinates and this lane's pixel of an imaging-plane key (view-major
// when vm, else a global bucket id).
__device__ __forceinline__ TileCell tile_cell_i(const DevView* views, int nv, uint32_t key, bool vm)
{
    if (!vm) return tile_cell(views, nv, (int64_t)key, false);
    TileCell t;
    t.v = (int)(key & 0xFFu);
    const DevView& V = views[t.v];
    const uint32_t local = key >> 8;
    t.tx = (int)(local % (uint32_t)V.txi);
    t.ty = (int)(local / (uint32_t)V.txi);
    const int lane = lane_id();
    t.col = t.tx * TILE + (lane & (TILE - 1));
    t.row = t.ty * TILE + (lane / TILE);
    t.inside = t.col < V.W && t.row < V.H;
    return t;
}

// Footprint mask of every computation-plane pair (bit 8 * row + col for
// the tile cells inside the ellipse q < q_max), and per 64-pair chunk of
// the sorted array (aligned to the array, so a chunk may span two tiles)
// the OR of its masks. A block takes PM_ITEMS runs of 256 pairs, each wave
// one chunk of every run, so that each lane has PM_ITEMS independent record
// reads in flight.
constexpr int PM_ITEMS = 4;

template <bool TIGHT>
__global__ void __launch_bounds__(256)
k_pair_masks(const DevView* __restrict__ views, int nv, int64_t cap, RasterParams rp,
             const uint32_t* __restrict__ status, const uint32_t* __restrict__ pkey,
             const uint32_t* __restrict__ pvals, const CRec* __restrict__ crec,
             uint64_t* __restrict__ pmask, uint64_t* __restrict__ psum)
{
    constexpr int BP = 256 * PM_ITEMS;
    const int64_t kc = min(cap, (int64_t)status[ST_PAIRS_C]);
    const uint32_t nblk = (uint32_t)((kc + BP - 1) / BP);
    const int64_t base = (int64_t)xcd_block(blockIdx.x, nblk) * BP + threadIdx.x;
    if (base - lane_id() >= kc) return;   // whole wave past the end
    uint32_t bucket[PM_ITEMS], r[PM_ITEMS];
#pragma unroll
    for (int k = 0; k < PM_ITEMS; ++k) {
        const int64_t p = base + k * 256;
        bucket[k] = p < kc ? pkey[p] : 0u;
        r[k] = p < kc ? pvals[p] : 0u;
    }
    RecPair g[PM_ITEMS];
#pragma unroll
    for (int k = 0; k < PM_ITEMS; ++k) g[k] = load_rec_pair(crec, r[k]);   // (record 0 past the end)
#pragma unroll
    for (int k = 0; k < PM_ITEMS; ++k) {
        const int64_t p = base + k * 256;
        if (p - lane_id() >= kc) break;   // this and later chunks of the wave are past the end
        uint64_t m = 0ull;
        const CRec rec = own_rec(g[k]);
        if (p < kc) {
            const int v = find_view(nv, (int64_t)bucket[k],
                                    [&](int j) { return (int64_t)views[j].tile_c; });
            const DevView& V = views[v];
            const int local = (int)(bucket[k] - (uint32_t)V.tile_c);
            m = footprint_mask<TIGHT>(rec.q.x, rec.q.y, rec.q.z, rec.q.w, rec.w.x, rp.q_max,
                                      local % V.txc, local / V.txc);
            pmask[p] = m;
        }
        const uint32_t olo = or_scan_u32((uint32_t)m), ohi = or_scan_u32((uint32_t)(m >> 32));
        if (lane_id() == WAVE - 1) psum[p / WAVE] = ((uint64_t)ohi << 32) | olo;
    }
}

// A block of `take` units of the hit stream for a tile's records (the whole
// wave calls): from part `sub` if it has room, else from another part whose
// counter shows room, wherever it lies; sub is where the tile goes on. Only a
// tile that finds its part full looks at others, HIT_LOOK - 1 spread over the
// stream. Where these are mostly full too it asks once more and, in vain,
// raises its part's counter past HIT_FULL, so that the tiles after it in that
// part stop at their first request. Pass A of 500k Gaussians in one view, whose
// stream fills everywhere, takes 134 us; with all 64 counters read and as many
// requests as they promise 177, with the mark and three requests 144.
constexpr int HIT_TRIES = 3;
constexpr uint32_t HIT_LOOK = 8, HIT_STEP = 71;   // (a prime past HIT_SUBS: all parts in turn)
constexpr unsigned long long HIT_FULL = 1ull << 40;

__device__ __forceinline__ bool take_hit_block(const RasterParams& rp, uint32_t take,
                                               uint32_t& sub, uint32_t& top)
{
    const uint32_t lane = (uint32_t)lane_id();
    const unsigned long long cap = rp.hit_sub_cap;
    auto ask = [&](uint32_t s) {
        unsigned long long at = 0ull;
        if (lane == 0u)
            at = atomicAdd(&rp.hit_tops[s * HIT_TOP_STRIDE], (unsigned long long)take);
        return ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane(
                    (int)(uint32_t)(at >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at);
    };
    unsigned long long at = ask(sub);
    if (at + take > cap) {
        if (at >= HIT_FULL) return false;
        const uint32_t first = sub, parts = min(rp.hit_subs, HIT_LOOK);
        auto part = [&](uint32_t k) { return (first + HIT_STEP * k) % rp.hit_subs; };
        unsigned long long used = cap;
        if (lane > 0u && lane < parts)
            used = __hip_atomic_load(&rp.hit_tops[part(lane) * HIT_TOP_STRIDE], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
        // parts at least half free: where they are a quarter, the stream fills
        // unevenly; else it fills everywhere
        uint64_t room = __ballot(2u * used <= cap && used + take <= cap);
        const bool ample = 4u * (uint32_t)__popcll(room) >= parts;
        if (!ample) room = __ballot(used + take <= cap);
        for (int k = 0;; ++k, room &= room - 1ull) {
            if (room == 0ull || k == (ample ? HIT_TRIES : 1)) {
                if (lane == 0u && !ample)
                    atomicAdd(&rp.hit_tops[first * HIT_TOP_STRIDE], HIT_FULL);
                return false;
            }
            sub = part((uint32_t)__builtin_ctzll(room));
            at = ask(sub);
            if (at + take <= cap) break;
        }
    }
    top = sub * rp.hit_sub_cap + (uint32_t)at;
    return true;
}

// Pass A forward, one wave per non-empty 8x8 tile; the wave's rays are the
// tile's 64 cells. The list is walked in 64-entry chunks aligned to the
// global pair array; a chunk whose footprint summary misses every ray still
// in play is skipped without reading its entries. Chunks that are read are
// taken in batches (of HB_CHUNKS where the hits are stored, else twice
// A_BATCH): their masks are loaded together, then the records of the entries
// any live ray needs are gathered together, so a batch pays two memory
// latencies. Inside a chunk the 64x64 bit matrix of
// footprint masks is transposed (lane = ray: which entries cover my cell),
// the (ray, entry) hits are compacted ray-major into LDS, and the wave
// takes them 64 at a time, lane = hit: each ray's optical depth in front of
// each of its hits is a segmented prefix sum, so a round costs the same
// however the hits are spread over the rays. Per-entry sums collect in LDS
// and leave with one global atomic per (tile, entry).
constexpr int A_BATCH = 4;
// Hits of a compaction group: all of a batch's when at most half of these
// are left, else each ray's next GROUP_RAY.
constexpr uint32_t GROUP_RAY = 16;
constexpr uint32_t GROUP_HITS = WAVE * GROUP_RAY;
// Chunks of a batch where hits are stored (and entry slots of the backward).
constexpr int HB_CHUNKS = 4;
constexpr int HB_SLOTS = HB_CHUNKS * WAVE;
constexpr int HB_CHUNK_BITS = 2, HB_RAY_SHIFT = 6 + HB_CHUNK_BITS;
static_assert(HB_CHUNKS == 1 << HB_CHUNK_BITS, "chunk index bits of a stored hit");

// Where hits are stored, up to this many tiles go to k_raster_a_fwd_hits, nine
// waves to a tile, which halves the chain of a long list: 8 views of 20k
// Gaussians in 88 tiles 100 -> 63 us, 20 views of 80k in 718 tiles 142 -> 91.
// More tiles fill the device with a wave each: 72 views of 200k in 2601 tiles
// 375 against 453, 36 views of 50k in 6360 shorter ones 145 against 341. Near
// the line, a wave and nine to a tile: a vehicle of 80k in 1193 tiles 153 and
// 136, 1526 161 and 178, 1789 163 and 205; of 200k in 1216 264 and 213, 1558 270
// and 273, 1829 286 and 313; a building of 50k in 1218 83 and 70, 1566 90 and
// 87, 1916 89 and 106; a block of 200k in 1553 74 and 67.
constexpr uint32_t HF_TILES = 1536;

// DET: deterministic mode (per-pair partials at their pre-sort positions).
// HITS: the hits are stored for the backward. Only then is a group cut by ray;
// without stored hits the groups are whole chunks of up to 4096 hits. (The
// backward that re-derives hits takes either: tiles that find the stream full
// come to it from groups cut by ray, within 1e-5 of the stored hits' sums.)
template <bool DET, bool HITS>
__global__ void __launch_bounds__(WAVE) __attribute__((amdgpu_waves_per_eu(1, HITS ? 8 : 2)))
k_raster_a_fwd(const DevView* __restrict__ views, int nv, RasterParams rp,
               const uint32_t* __restrict__ status, const uint32_t* __restrict__ worklist,
               const uint2* __restrict__ ranges, const uint32_t* __restrict__ pvals,
               const uint64_t* __restrict__ pmask, const uint64_t* __restrict__ psum,
               const CRec* __restrict__ crec,
               float* __restrict__ A, float* __restrict__ tau, uint32_t* __restrict__ nlast)
{
    constexpr int NB = HITS ? HB_CHUNKS : 2 * A_BATCH;
    constexpr int HKB = NB == 4 ? 2 : 3;   // bits of a hit's chunk index
    constexpr int HRS = 6 + HKB;           // shift of a hit's ray index
    static_assert(NB == 4 || NB == 8, "chunk index bits");
    static_assert(!HITS || NB <= 4 * ((int)HIT_HEADER_UNITS - 1), "chunk ids of a stored-hit record");
    __shared__ float4 s_q[NB][WAVE];
    __shared__ float s_wc[NB][WAVE], s_wk[NB][WAVE];   // conic c and extinction
    __shared__ double s_A[NB][WAVE + 1];      // per-entry sums
    __shared__ uint32_t s_chk[NB];
    constexpr uint32_t GROUP_MAX = HITS ? GROUP_HITS : WAVE * WAVE;
    __shared__ uint16_t s_hit[GROUP_MAX];     // (ray, chunk, entry) packed, ray-major
    // per ray during a group: first hit in s_hit, optical depth, transmittance,
    // last list position used (one 16-byte read per hit)
    struct alignas(16) RayF { uint32_t o; float t, T; uint32_t last; };
    __shared__ RayF s_ray[WAVE];
    const int lane = threadIdx.x;
    const TransposeLane tl = transpose_lane();
    const uint32_t ntiles = status[ST_WORK_TILES];
    if (blockIdx.x >= ntiles || (HITS && ntiles <= HF_TILES)) return;
    const int64_t bucket = worklist[blockIdx.x];
    const TileCell tc = tile_cell(views, nv, bucket, true);
    const DevView& V = views[tc.v];
    const float x0 = (float)(tc.tx * TILE) + 0.5f, y0 = (float)(tc.ty * TILE) + 0.5f;
    const uint2 rg = ranges[bucket];
#pragma unroll
    for (int k = 0; k < NB; ++k) s_A[k][lane] = 0.0;
    float T = 1.0f, t = 0.0f;
    bool alive = tc.inside;
    uint32_t last = 0;
    uint32_t n_iter = 0, n_hits = 0, n_batch = 0, n_extra = 0;   // work counters
    uint64_t live = __ballot(alive);
    // per-entry sums of the last processed batch leave with one atomic each;
    // they are sent once the next batch's loads have landed, so the wait for
    // those loads never waits for the atomics
    uint32_t r_prev[NB], r_cur[NB];   // record of my entry in each chunk
    uint32_t d_prev[NB], d_cur[NB];   // deterministic mode: its pair's position before the sort
    // stored hits: this tile's chain of batch records (h_on while the stream
    // has room; h_prev becomes HIT_OVERFLOW when it runs out), the block of
    // the stream the tile writes into [h_top, h_end) and the block size it
    // takes next, the current record and its hit count
    bool h_on = HITS;
    uint32_t h_top = 0u, h_end = 0u, h_blk = 128u, h_prev = HIT_NONE, h_rec = 0u, h_kept = 0u;
    uint32_t h_prev2 = HIT_NONE;   // the record before h_prev
    uint32_t h_seq = 0u;           // records stored
    uint32_t h_sub = HITS ? blockIdx.x % rp.hit_subs : 0u;   // part of the stream
    // (a nonzero sum means a live ray hit the entry, so its record was
    // gathered and r_prev holds it: all eight sums are read at once, without
    // a branch per chunk)
    auto flush = [&]() {
        float a[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) a[k] = (float)s_A[k][lane];
#pragma unroll
        for (int k = 0; k < NB; ++k) s_A[k][lane] = 0.0;
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (a[k] != 0.0f) {
                if constexpr (DET) rp.part[d_prev[k]] = a[k];
                else unsafeAtomicAdd(&A[r_prev[k]], a[k]);
            }
        }
    };
    const uint32_t c_first = rg.x / WAVE, c_end = (rg.y + WAVE - 1) / WAVE;
    for (uint32_t g0 = c_first; g0 < c_end && live != 0ull; g0 += WAVE) {
        const uint64_t sm = g0 + lane < c_end ? psum[g0 + lane] : 0ull;
        uint64_t todo = __ballot((sm & live) != 0ull);   // chunks to read, in order
        // up to NB chunks per batch: their masks and values are fetched one
        // batch ahead (in flight while the current batch's hits are
        // processed), then the records the live rays need
        uint32_t chk_n[NB], r_n[NB], d_n[NB];
        uint64_t m_n[NB];
        int nb_n = 0;
        auto fetch = [&]() {
            nb_n = 0;
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                chk_n[k] = 0u;
                if (todo != 0ull) {
                    chk_n[k] = g0 + (uint32_t)__builtin_ctzll(todo);
                    todo &= todo - 1ull;
                    nb_n = k + 1;
                }
            }
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const uint32_t e = chk_n[k] * WAVE + lane;
                const bool in = k < nb_n && e >= rg.x && e < rg.y;
                m_n[k] = in ? pmask[e] : 0ull;
                r_n[k] = in ? pvals[e] : 0u;
                if constexpr (DET) d_n[k] = in ? rp.ppos[e] : 0u;
            }
        };
        fetch();
        while (nb_n > 0 && live != 0ull) {
            ++n_batch;
            const int nb = nb_n;
            // the batch's chunks; col[k] is first lane = entry (the cells it
            // covers), then transposed to lane = ray (the entries covering it)
            uint64_t col[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                col[k] = m_n[k];
                r_cur[k] = r_n[k];
                if constexpr (DET) d_cur[k] = d_n[k];
            }
            // records straight into LDS, all in flight together (entries no
            // live ray needs read record 0, one shared line)
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const bool need = (col[k] & live) != 0ull;
                const uint32_t rk = need ? r_cur[k] : 0u;
                const float* w = reinterpret_cast<const float*>(&crec[rk].w);
                load16_to_lds(&crec[rk].q, &s_q[k][0]);
                load4_to_lds(w, &s_wc[k][0]);
                load4_to_lds(w + 1, &s_wk[k][0]);
                if (lane == k) s_chk[k] = chk_n[k];
            }
            // the transposes run while the records come in; rays already out
            // of play and unused chunk slots keep no hits
            transpose64_n(col, tl);
#pragma unroll
            for (int k = 0; k < NB; ++k) col[k] = (k < nb && alive) ? col[k] : 0ull;
            wait_all_memory();
            wave_lds_sync();
            fetch();   // the next batch's masks and values
            flush();
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                r_prev[k] = r_cur[k];
                if constexpr (DET) d_prev[k] = d_cur[k];
            }
            uint32_t hk[HITS ? 1 : NB];   // hits of each chunk over the wave
            if constexpr (!HITS) {
                // (at most 4096 each: summed two to a word)
                uint32_t tot[NB / 2];
#pragma unroll
                for (int i = 0; i < NB / 2; ++i)
                    tot[i] = (uint32_t)__popcll(col[2 * i]) |
                             ((uint32_t)__popcll(col[2 * i + 1]) << 16);
                wave_total_u32_n(tot);
#pragma unroll
                for (int i = 0; i < NB / 2; ++i) {
                    hk[2 * i] = tot[i] & 0xFFFFu;
                    hk[2 * i + 1] = tot[i] >> 16;
                }
            }
            // The batch's hits in groups, compacted ray-major (front to back
            // along each ray) and taken 64 per round. Stored hits: all that
            // are left when they are few, else each ray's next GROUP_RAY;
            // after each group the rays that reached tau_max drop their
            // remaining hits, so dense lists do not compact and evaluate what
            // lies behind. Otherwise consecutive chunks whose hits fit s_hit.
            bool fresh = true;   // no record of this batch is stored yet
            int g0 = 0, g1 = NB;
            for (uint32_t group = 0;; ++group) {
                uint32_t nr = 0, H, o, o_end;
                if constexpr (HITS) {
#pragma unroll
                    for (int k = 0; k < NB; ++k) nr += (uint32_t)__popcll(col[k]);
                    if (__ballot(nr != 0u) == 0ull) break;
                    // hits left and hits of a limited group, scanned together
                    // (at most 64 x 256 and 64 x GROUP_RAY: two to a word)
                    const uint32_t lim = min(nr, GROUP_RAY);
                    const uint32_t both = nr | (lim << 16);
                    const uint32_t ex = wave_excl_scan_u32(both);
                    const uint32_t tot =
                        (uint32_t)__builtin_amdgcn_readlane((int)(ex + both), WAVE - 1);
                    const bool few = (tot & 0xFFFFu) <= GROUP_HITS / 2;
                    H = few ? (tot & 0xFFFFu) : (tot >> 16);
                    o = few ? (ex & 0xFFFFu) : (ex >> 16);
                    o_end = o + (few ? nr : lim);
                } else {
                    if (g0 >= nb || live == 0ull) break;
                    H = 0u;
                    bool open = true;
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        if (k < g0 || k >= nb || !open) continue;
                        if (H + hk[k] <= GROUP_MAX) {
                            H += hk[k];
                            g1 = k + 1;
                        } else {
                            open = false;
                        }
                    }
#pragma unroll
                    for (int k = 0; k < NB; ++k)
                        if (k >= g0 && k < g1) nr += (uint32_t)__popcll(col[k]);
                    o = wave_excl_scan_u32(nr);
                    o_end = o + nr;
                }
                if (group > 0) ++n_extra;
                if (h_on) {
                    // room for the group's record (header and at most every
                    // hit); a new block when the tile's is short (sizes
                    // doubling up to 16 KB, so short tiles waste little and
                    // long ones seldom ask)
                    const uint32_t units = HIT_HEADER_UNITS + (H + 7u) / 8u;
                    if (h_end - h_top < units) {
                        const uint32_t take = max(units, h_blk);
                        h_blk = min(2u * h_blk, 1024u);
                        h_on = take_hit_block(rp, take, h_sub, h_top);
                        h_end = h_top + take;
                        if (!h_on) h_prev = HIT_OVERFLOW;
                    }
                }
                h_rec = h_top;
                h_kept = 0u;
                uint32_t w = o;
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    if (!HITS && (k < g0 || k >= g1)) continue;
                    uint32_t half[2] = {(uint32_t)col[k], (uint32_t)(col[k] >> 32)};
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const uint32_t tag = (uint32_t)((lane << HRS) | (k << 6) | (q << 5));
                        while (half[q] != 0u && w < o_end) {
                            const uint32_t j = (uint32_t)__builtin_ctz(half[q]);
                            half[q] &= half[q] - 1u;
                            s_hit[w++] = (uint16_t)(tag | j);
                        }
                    }
                    col[k] = ((uint64_t)half[1] << 32) | half[0];
                }
                s_ray[lane] = RayF{o, t, T, last};
                wave_lds_sync();
                for (uint32_t base = 0; base < H; base += WAVE) {
                    ++n_iter;
                    const uint32_t L = base + lane;
                    const bool valid = L < H;
                    const uint32_t hv = valid ? (uint32_t)s_hit[L] : 0u;
                    const int rr = (int)(hv >> HRS), k = (int)((hv >> 6) & ((1u << HKB) - 1u)),
                              j = (int)(hv & 63u);
                    // ray state and entry record, read together (lanes past
                    // the last hit read entry 0 of ray 0 and ignore it)
                    const RayF rs = s_ray[rr];
                    const float4 g = s_q[k][j];
                    const float gc = s_wc[k][j], gk = s_wk[k][j];
                    const uint32_t pos = s_chk[k] * WAVE + (uint32_t)j - rg.x;   // list position
                    const int seg0 = valid ? max((int)rs.o - (int)base, 0) : lane;
                    bool real = false;
                    float x = 0.0f, E = 1.0f;
                    if (valid) {
                        const float dx = x0 + (float)(rr & (TILE - 1)) - g.x;
                        const float dy = y0 + (float)(rr / TILE) - g.y;
                        const float q = quadform(g, gc, dx, dy);
                        if (q < rp.q_max) {
                            real = true;
                            x = gk * ((__expf(-0.5f * q) - rp.eps) * rp.inv1meps);
                            E = __expf(-x);
                        }
                    }
                    const float incl = seg_incl_scan(x, lane == seg0);
                    const float excl = incl - x;
                    const float tr = valid ? rs.t : 0.0f;
                    const float Tr = valid ? rs.T : 1.0f;
                    // a ray's hits are processed up to the first one reached
                    // with an optical depth of tau_max (a prefix of its segment)
                    const uint64_t stop =
                        __ballot(valid && rp.shadowing && !(tr + excl < rp.tau_max));
                    const uint64_t after = stop & (~0ull << seg0);
                    const bool proc = valid && (after == 0ull || lane < __builtin_ctzll(after));
                    if (h_on) {
                        // the processed hits, in processing order
                        const uint64_t kb = __ballot(proc);
                        if (proc)
                            reinterpret_cast<uint16_t*>(
                                rp.hits + h_rec + HIT_HEADER_UNITS)[h_kept + lanes_below(kb)] =
                                (uint16_t)hv;
                        h_kept += (uint32_t)__popcll(kb);
                    }
                    if (proc && real) {
                        // at least FLT_MIN, so that A > 0 marks exactly the
                        // records some ray used (the exact alpha T is > 0
                        // for every footprint hit)
                        const float a = fmaxf(
                            (1.0f - E) * (rp.shadowing ? Tr * __expf(-excl) : 1.0f), FLT_MIN);
                        atomicAdd(&s_A[k][j], (double)a);
                    }
                    n_hits += (uint32_t)__popcll(__ballot(proc && real));
                    // the last processed hit of each ray in this round updates the ray
                    const int nxt = from_lane_above(proc ? (int)hv : -1);
                    const bool endseg = proc && (lane == WAVE - 1 || (nxt >> HRS) != rr);
                    float tn = tr + incl;
                    if constexpr (HITS) {
                        // stopped in front of a further hit of its own: done,
                        // also where this sum rounds to just below tau_max
                        const int fol = from_lane_above(valid ? (int)hv : -1);
                        if (lane < WAVE - 1 && (fol >> HRS) == rr && rp.shadowing)
                            tn = fmaxf(tn, rp.tau_max);
                    }
                    wave_lds_sync();
                    if (endseg)
                        s_ray[rr] = RayF{rs.o, tn, rp.shadowing ? Tr * __expf(-incl) : Tr,
                                         pos + 1u};
                    wave_lds_sync();
                }
                {
                    const RayF rs = s_ray[lane];
                    t = rs.t;
                    T = rs.T;
                    last = rs.last;
                }
                if (rp.shadowing && t >= rp.tau_max) {
                    alive = false;
                    if constexpr (HITS) {
#pragma unroll
                        for (int k = 0; k < NB; ++k) col[k] = 0ull;
                    }
                }
                live = __ballot(alive);
                g0 = g1;
                wave_lds_sync();
                if (h_on && h_kept > 0u) {   // the group's record
                    if (lane == 0)
                        rp.hits[h_rec] =
                            make_uint4(h_prev, h_kept, (h_seq << 1) | (fresh ? 1u : 0u), h_prev2);
                    if (lane == 1)
                        rp.hits[h_rec + 1] = make_uint4(s_chk[0], s_chk[1], s_chk[2], s_chk[3]);
                    ++h_seq;
                    h_prev2 = h_prev;
                    h_prev = h_rec;
                    h_top = h_rec + HIT_HEADER_UNITS + (h_kept + 7u) / 8u;
                    fresh = false;
                }
            }
            wave_lds_sync();
        }
    }
    flush();
    if (HITS && lane == 0) rp.hit_tail[bucket] = h_prev;
    if (rp.work) {
        const uint32_t used = wave_max_u32(last);   // list prefix any ray used
        const uint64_t stopped = __ballot(tc.inside && rp.shadowing && t >= rp.tau_max);
        if (lane == 0) {
            atomicAdd(&rp.work[4], (unsigned long long)n_iter);
            atomicAdd(&rp.work[0], (unsigned long long)n_hits);
            atomicAdd(&rp.work[7], (unsigned long long)used);
            atomicMax(&rp.work[8], (unsigned long long)n_batch);
            atomicAdd(&rp.work[10], (unsigned long long)n_extra);
            atomicAdd(&rp.work[12], (unsigned long long)__popcll(stopped));
            atomicMax(&rp.work[13], (unsigned long long)used);
        }
    }
    if (tc.inside) {
        const int64_t ray = V.ray_off + (int64_t)tc.row * V.Wc + tc.col;
        tau[ray] = t;
        nlast[ray] = last;
    }
}

// Pass A forward with the hits stored for the backward, for few tiles: a
// workgroup of nine waves takes a tile. The list is walked in the same batches
// of four chunks, in three stages a step apart (a step is a group of hits):
//   four waves prepare the next group: load and transpose a chunk each and
//     compact the hits ray-major together. Masks and record ids are loaded two
//     batches ahead, records one batch ahead. Which rays are in play is known
//     up to the group before the current one; hits of rays that stop in that
//     are evaluated in vain;
//   four waves evaluate the current group, 256 hits at a time, 64 to a wave:
//     the segmented prefix sums along the rays run in each wave, and the one
//     ray that crosses from a wave into the next is carried over through LDS;
//   the last wave sends the per-entry sums of the group before and copies its
//     hits to the stream (memory operations complete in order, so a wave that
//     also stored would wait for its atomics whenever it waits for a load).
// Bound by the chain of batches of the longest lists, most of it dependent
// instructions and LDS accesses: a single wave that does all of it takes 4 us
// a batch (k_raster_a_fwd, the better one where tiles fill the device).
constexpr int HF_THREADS = (2 * HB_CHUNKS + 1) * WAVE;

// One group of hits, from the preparing waves.
struct HitGroup {
    uint32_t H, base, off;   // hits; chunk k of the batch is base + byte k of off
    uint32_t flags;          // 1: no group, the list is done, 2: first of its batch
    int par, buf;            // buffers of its batch's records (of two, of three)
};

// What a wave of the evaluation tells the others about its 64 hits.
struct HitFwdInfo {
    uint32_t kept, kept0;   // hits processed, and those of its first lane's ray
    uint32_t bits;          // 1: first lane processed, 2: its last ray stopped, 4: one ray only
};

__global__ void __launch_bounds__(HF_THREADS)
k_raster_a_fwd_hits(const DevView* __restrict__ views, int nv, RasterParams rp,
                    const uint32_t* __restrict__ status, const uint32_t* __restrict__ worklist,
                    const uint2* __restrict__ ranges, const uint32_t* __restrict__ pvals,
                    const uint64_t* __restrict__ pmask, const uint64_t* __restrict__ psum,
                    const CRec* __restrict__ crec, float* __restrict__ A,
                    float* __restrict__ tau, uint32_t* __restrict__ nlast)
{
    constexpr int NB = HB_CHUNKS, HRS = HB_RAY_SHIFT;
    static_assert(NB <= 4 * ((int)HIT_HEADER_UNITS - 1), "chunk ids of a stored-hit record");
    __shared__ float4 s_q[2][NB][WAVE];
    __shared__ float2 s_w[2][NB][WAVE];       // conic c and extinction
    __shared__ uint32_t s_rec[3][NB][WAVE];   // record of each entry
    __shared__ double s_A[NB][WAVE + 1];      // per-entry sums
    __shared__ uint32_t s_cnt[NB][WAVE];      // hits per chunk and ray
    __shared__ uint16_t s_hit[2][GROUP_HITS]; // (ray, chunk, entry) packed, ray-major
    __shared__ uint32_t s_o[2][WAVE];         // per ray: its first hit in s_hit
    __shared__ HitGroup s_group[2];
    // per ray: optical depth, transmittance, last list position used
    struct alignas(16) RayF { float t, T; uint32_t last, pad; };
    __shared__ RayF s_ray[WAVE];
    __shared__ float s_tail[NB];              // sum of the last ray's hits in each wave's round
    __shared__ HitFwdInfo s_info[NB];
    __shared__ uint4 s_out[GROUP_HITS / 8];   // the group's processed hits, in order
    const uint32_t ntiles = status[ST_WORK_TILES];
    if (blockIdx.x >= ntiles || ntiles > HF_TILES) return;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
    const int w = wave & (NB - 1);
    const int64_t bucket = worklist[blockIdx.x];
    const TileCell tc = tile_cell(views, nv, bucket, true);
    const DevView& V = views[tc.v];
    const uint2 rg = ranges[bucket];
    if (wave < NB) s_A[w][lane] = 0.0;
    if (wave == 0) s_ray[lane] = RayF{0.0f, 1.0f, 0u, 0u};
    __syncthreads();
    // Every wave meets the same barriers: three per 256 hits of a group, at
    // least three per group, and three before the first.
    auto rounds = [](uint32_t H) { return max(1u, (H + NB * WAVE - 1) / (NB * WAVE)); };

    if (wave < NB) {   // ---- the next group
        const TransposeLane tl = transpose_lane();
        const uint32_t c_first = rg.x / WAVE, c_end = (rg.y + WAVE - 1) / WAVE;
        bool alive = tc.inside;
        uint64_t live = __ballot(alive);
        // a batch: up to NB chunks whose footprint summary meets a ray in
        // play, from one group of 64 chunks (loads are unconditional, so that
        // waiting for one waits for no other)
        struct Batch {
            uint32_t base, off;
            int nb;
            __device__ uint32_t chunk(int k) const { return base + ((off >> (8 * k)) & 0xFFu); }
        };
        uint32_t g0 = c_first;
        auto summary = [&](uint32_t g) { return psum[min(g + lane, c_end - 1u)]; };
        auto meets = [&](uint64_t sm) {
            return __ballot(g0 + lane < c_end && (sm & live) != 0ull);
        };
        uint64_t ahead = summary(g0);
        uint64_t todo = meets(ahead);
        ahead = summary(g0 + WAVE);
        auto next = [&]() {
            while (todo == 0ull && g0 + WAVE < c_end) {
                g0 += WAVE;
                todo = meets(ahead);
                ahead = summary(g0 + WAVE);
            }
            Batch b{g0, 0u, 0};
#pragma unroll
            for (int k = 0; k < NB; ++k)
                if (todo != 0ull) {
                    b.off |= (uint32_t)__builtin_ctzll(todo) << (8 * k);
                    todo &= todo - 1ull;
                    b.nb = k + 1;
                }
            return b;
        };
        // the wave's chunk of a batch: cells covered and record of the lane's entry
        struct Entry {
            uint64_t m;
            uint32_t rec;
            bool in;
            __device__ uint64_t cells() const { return in ? m : 0ull; }
        };
        auto fetch = [&](const Batch& b) {
            const uint32_t e = b.chunk(w) * WAVE + lane;
            const bool in = w < b.nb && e >= rg.x && e < rg.y;
            const uint32_t at = in ? e : rg.x;
            return Entry{pmask[at], pvals[at], in};
        };
        // (entries no ray in play needs read record 0, one shared line)
        auto gather = [&](const Entry& e) {
            return load_rec_pair(crec, (e.cells() & live) != 0ull ? e.rec : 0u);
        };
        Batch cur = next(), nx = next();
        Entry e_cur = fetch(cur), e_nx = fetch(nx);
        RecPair rec = gather(e_cur);
        uint32_t N = 0u, done = 0u, idx = 0u;   // the ray's hits in the batch, those taken, and
                                                // the index of the wave's next one
        uint32_t half[2] = {0u, 0u};            // the wave's entries left that cover the ray
        int par = 0, buf = 0;
        uint32_t b_base = 0u, b_off = 0u;   // the batch's chunks
        uint32_t n_batch = 0, n_extra = 0;   // work counters
        uint32_t H = 0u;   // of the group being evaluated
        for (int p = 1;; p ^= 1) {
            // rays that reached tau_max drop their remaining hits
            if (rp.shadowing && s_ray[lane].t >= rp.tau_max) {
                alive = false;
                done = N;
                half[0] = half[1] = 0u;
            }
            live = __ballot(alive);
            const bool fresh = __ballot(done != N) == 0ull;
            const bool end = fresh && (cur.nb == 0 || live == 0ull);
            const uint32_t base = cur.base, off = cur.off;
            if (fresh && !end) {
                if (n_batch > 0u) {
                    par ^= 1;
                    buf = buf == 2 ? 0 : buf + 1;
                }
                ++n_batch;
                const Batch nn = next();
                const Entry e_nn = fetch(nn);
                const CRec own = own_rec(rec);
                s_q[par][w][lane] = own.q;
                s_w[par][w][lane] = make_float2(own.w.x, own.w.y);
                s_rec[buf][w][lane] = e_cur.rec;
                rec = gather(e_nx);
                // lane = ray: the entries of the wave's chunk covering it
                uint64_t col = transpose64(e_cur.cells(), tl);
                if (!alive) col = 0ull;
                s_cnt[w][lane] = (uint32_t)__popcll(col);
                half[0] = (uint32_t)col;
                half[1] = (uint32_t)(col >> 32);
                cur = nx;
                nx = nn;
                e_cur = e_nx;
                e_nx = e_nn;
            } else {
                n_extra += end ? 0u : 1u;
            }
            __syncthreads();
            HitGroup g{0u, 0u, 0u, 1u, par, buf};
            if (!end) {
                if (fresh) {
                    N = done = idx = 0u;
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        const uint32_t c = s_cnt[k][lane];
                        if (k < w) idx += c;
                        N += c;
                    }
                    b_base = base;
                    b_off = off;
                }
                // all hits that are left when they are few, else each ray's
                // next GROUP_RAY (both scanned together: at most 64 x 256 and
                // 64 x GROUP_RAY, two to a word)
                const uint32_t left = N - done, lim = min(left, GROUP_RAY);
                const uint32_t both = left | (lim << 16);
                const uint32_t ex = wave_excl_scan_u32(both);
                const uint32_t tot =
                    (uint32_t)__builtin_amdgcn_readlane((int)(ex + both), WAVE - 1);
                const bool few = (tot & 0xFFFFu) <= GROUP_HITS / 2;
                const uint32_t o = few ? (ex & 0xFFFFu) : (ex >> 16);
                const uint32_t to = done + (few ? left : lim);
                g = HitGroup{few ? (tot & 0xFFFFu) : (tot >> 16), b_base, b_off, fresh ? 2u : 0u,
                             par, buf};
                if (w == 0) s_o[p ^ 1][lane] = o;
                uint16_t* out = s_hit[p ^ 1] + o;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const uint32_t tag = (uint32_t)((lane << HRS) | (w << 6) | (q << 5));
                    while (half[q] != 0u && idx < to) {
                        const uint32_t j = (uint32_t)__builtin_ctz(half[q]);
                        half[q] &= half[q] - 1u;
                        out[idx - done] = (uint16_t)(tag | j);
                        ++idx;
                    }
                }
                done = to;
            }
            if (w == 0 && lane == 0) s_group[p ^ 1] = g;
            __syncthreads();
            __syncthreads();
            for (uint32_t k = rounds(H); k > 1u; --k) {
                __syncthreads();
                __syncthreads();
                __syncthreads();
            }
            if (end) break;
            H = g.H;
        }
        if (rp.work && w == 0 && lane == 0) {
            atomicMax(&rp.work[8], (unsigned long long)n_batch);
            atomicAdd(&rp.work[10], (unsigned long long)n_extra);
        }
    } else if (wave < 2 * NB) {   // ---- the current group
        const float x0 = (float)(tc.tx * TILE) + 0.5f, y0 = (float)(tc.ty * TILE) + 0.5f;
        uint32_t n_iter = 0, n_hits = 0;   // work counters
        __syncthreads();
        __syncthreads();
        __syncthreads();
        for (int p = 0;; p ^= 1) {
            const HitGroup G = s_group[p];
            if (G.flags & 1u) break;
            uint32_t kept = 0u;   // hits of the group processed so far
            for (uint32_t base = 0; base == 0u || base < G.H; base += NB * WAVE) {
                const uint32_t b0 = base + (uint32_t)w * WAVE, L = b0 + lane;
                n_iter += b0 < G.H ? 1u : 0u;
                const bool valid = L < G.H;
                const uint32_t hv = valid ? (uint32_t)s_hit[p][L] : 0u;
                const int rr = (int)(hv >> HRS), k = (int)((hv >> 6) & (NB - 1u)),
                          j = (int)(hv & 63u);
                // ray state and entry record, read together (lanes past the
                // last hit read entry 0 of ray 0 and ignore it)
                const RayF rs = s_ray[rr];
                const uint32_t ro = s_o[p][rr];
                const float4 g = s_q[G.par][k][j];
                const float2 g2 = s_w[G.par][k][j];
                // the ray of the next hit, the next wave's first for lane 63
                const int fol = L + 1u < G.H ? (int)((uint32_t)s_hit[p][L + 1u] >> HRS) : -1;
                const int seg0 = valid ? max((int)ro - (int)b0, 0) : lane;
                bool real = false;
                float x = 0.0f, E = 1.0f;
                if (valid) {
                    const float dx = x0 + (float)(rr & (TILE - 1)) - g.x;
                    const float dy = y0 + (float)(rr / TILE) - g.y;
                    const float q = quadform(g, g2.x, dx, dy);
                    if (q < rp.q_max) {
                        real = true;
                        x = g2.y * ((__expf(-0.5f * q) - rp.eps) * rp.inv1meps);
                        E = __expf(-x);
                    }
                }
                float incl = seg_incl_scan(x, lane == seg0);
                if (lane == WAVE - 1) s_tail[w] = incl;
                __syncthreads();
                // the lanes whose ray began in a wave before
                const bool crossed = valid && ro < b0;
                {
                    const uint32_t o0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)ro);
                    float carry = 0.0f;
                    for (int v = w - 1; v >= 0 && o0 < base + (uint32_t)(v + 1) * WAVE; --v)
                        carry += s_tail[v];
                    if (crossed) incl += carry;
                }
                const float excl = incl - x;
                const float tr = valid ? rs.t : 0.0f;
                const float Tr = valid ? rs.T : 1.0f;
                // a ray's hits are processed up to the first one reached with
                // an optical depth of tau_max (a prefix of its segment)
                const uint64_t stop = __ballot(valid && rp.shadowing && !(tr + excl < rp.tau_max));
                const uint64_t after = stop & (~0ull << seg0);
                bool proc = valid && (after == 0ull || lane < __builtin_ctzll(after));
                {
                    const uint64_t kb = __ballot(proc), cr = __ballot(crossed);
                    const int s63 = __builtin_amdgcn_readlane(seg0, WAVE - 1);
                    if (lane == 0)
                        s_info[w] = HitFwdInfo{(uint32_t)__popcll(kb), (uint32_t)__popcll(kb & cr),
                                               (uint32_t)(kb & 1ull) |
                                                   ((stop & (~0ull << s63)) != 0ull ? 2u : 0u) |
                                                   (cr == ~0ull ? 4u : 0u)};
                }
                __syncthreads();
                // hits kept by the waves before, and whether the ray that
                // crosses into this wave, or into the next, was stopped before
                uint32_t at = kept;
                bool dead = false, dead_in = false, next_first = false;
#pragma unroll
                for (int v = 0; v < NB; ++v) {
                    const HitFwdInfo f = s_info[v];
                    if (v == w) dead_in = dead;
                    if (v == w + 1) next_first = !dead && (f.bits & 1u) != 0u;
                    const uint32_t n = f.kept - (dead ? f.kept0 : 0u);
                    if (v < w) at += n;
                    kept += n;
                    dead = (f.bits & 2u) != 0u || (dead && (f.bits & 4u) != 0u);
                }
                if (crossed && dead_in) proc = false;
                {
                    const uint64_t kb = __ballot(proc);
                    if (proc)
                        reinterpret_cast<uint16_t*>(s_out)[at + lanes_below(kb)] = (uint16_t)hv;
                }
                if (proc && real) {
                    // at least FLT_MIN, so that A > 0 marks exactly the
                    // records some ray used (the exact alpha T is > 0 for
                    // every footprint hit)
                    const float a = fmaxf(
                        (1.0f - E) * (rp.shadowing ? Tr * __expf(-excl) : 1.0f), FLT_MIN);
                    atomicAdd(&s_A[k][j], (double)a);
                }
                n_hits += (uint32_t)__popcll(__ballot(proc && real));
                // the last processed hit of each ray updates the ray; a ray
                // stopped in front of a further hit of its own is done, also
                // where its sum rounds to just below tau_max
                const int nxt = from_lane_above(proc ? rr : -1);
                const bool own_next = fol == rr;
                const bool goes_on = lane == WAVE - 1 ? own_next && next_first : nxt == rr;
                if (proc && !goes_on) {
                    float tn = tr + incl;
                    if (own_next && rp.shadowing && (lane < WAVE - 1 || w < NB - 1))
                        tn = fmaxf(tn, rp.tau_max);
                    const uint32_t chunk = G.base + ((G.off >> (8 * k)) & 0xFFu);
                    s_ray[rr] = RayF{tn, rp.shadowing ? Tr * __expf(-incl) : Tr,
                                     chunk * WAVE + (uint32_t)j - rg.x + 1u, 0u};
                }
                __syncthreads();
            }
        }
        if (rp.work && lane == 0) {
            atomicAdd(&rp.work[4], (unsigned long long)n_iter);
            atomicAdd(&rp.work[0], (unsigned long long)n_hits);
        }
    } else {   // ---- what the group before leaves to store
        // this tile's chain of records (h_on while the stream has room; h_prev
        // becomes HIT_OVERFLOW when it runs out), the block of the stream the
        // tile writes into [h_top, h_end) and the block size it takes next
        bool h_on = true;
        uint32_t h_top = 0u, h_end = 0u, h_blk = 128u, h_prev = HIT_NONE, h_prev2 = HIT_NONE;
        uint32_t h_seq = 0u;                         // records stored
        uint32_t h_sub = blockIdx.x % rp.hit_subs;   // part of the stream
        HitGroup G{0u, 0u, 0u, 1u, 0, 0};
        uint32_t kept = 0u;   // hits of it processed
        bool fresh = true;    // no record of its batch is stored yet
        auto store_hits = [&]() {
            if (G.flags & 1u) return;
            if (G.flags & 2u) fresh = true;
            if (h_on && kept > 0u) {
                // room for the group's record; a new block when the tile's is
                // short (sizes doubling up to 16 KB, so short tiles waste
                // little and long ones seldom ask)
                const uint32_t words = (kept + 7u) / 8u, units = HIT_HEADER_UNITS + words;
                if (h_end - h_top < units) {
                    const uint32_t take = max(units, h_blk);
                    h_blk = min(2u * h_blk, 1024u);
                    h_on = take_hit_block(rp, take, h_sub, h_top);
                    h_end = h_top + take;
                    if (!h_on) h_prev = HIT_OVERFLOW;
                }
                if (h_on) {
                    uint4* to = rp.hits + h_top;
                    for (uint32_t i = lane; i < words; i += WAVE) to[HIT_HEADER_UNITS + i] = s_out[i];
                    if (lane == 0)
                        to[0] = make_uint4(h_prev, kept, (h_seq << 1) | (fresh ? 1u : 0u), h_prev2);
                    if (lane == 1)
                        to[1] = make_uint4(G.base + (G.off & 0xFFu), G.base + ((G.off >> 8) & 0xFFu),
                                           G.base + ((G.off >> 16) & 0xFFu), G.base + (G.off >> 24));
                    ++h_seq;
                    h_prev2 = h_prev;
                    h_prev = h_top;
                    h_top += units;
                }
            }
            if (kept > 0u) fresh = false;
        };
        auto store_sums = [&]() {
            if (G.flags & 1u) return;
            // (a nonzero sum means that a ray in play hit the entry)
            double a[NB];
            uint32_t r[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                a[k] = s_A[k][lane];
                r[k] = s_rec[G.buf][k][lane];
            }
#pragma unroll
            for (int k = 0; k < NB; ++k) s_A[k][lane] = 0.0;
#pragma unroll
            for (int k = 0; k < NB; ++k)
                if ((float)a[k] != 0.0f) unsafeAtomicAdd(&A[r[k]], (float)a[k]);
        };
        __syncthreads();
        __syncthreads();
        __syncthreads();
        for (int p = 0;; p ^= 1) {
            const HitGroup next = s_group[p];
            if (next.flags & 1u) break;
            store_hits();
            uint32_t n = 0u;
            for (uint32_t k = rounds(next.H), k0 = k; k > 0u; --k) {
                __syncthreads();
                if (k == k0) store_sums();
                __syncthreads();
                bool dead = false;
#pragma unroll
                for (int v = 0; v < NB; ++v) {
                    const HitFwdInfo f = s_info[v];
                    n += f.kept - (dead ? f.kept0 : 0u);
                    dead = (f.bits & 2u) != 0u || (dead && (f.bits & 4u) != 0u);
                }
                __syncthreads();
            }
            G = next;
            kept = n;
        }
        store_hits();
        store_sums();
        const RayF rs = s_ray[lane];
        if (lane == 0) rp.hit_tail[bucket] = h_prev;
        if (tc.inside) {
            const int64_t ray = V.ray_off + (int64_t)tc.row * V.Wc + tc.col;
            tau[ray] = rs.t;
            nlast[ray] = rs.last;
        }
        if (rp.work) {
            const uint32_t used = wave_max_u32(rs.last);   // list prefix any ray used
            const uint64_t stopped =
                __ballot(tc.inside && rp.shadowing && rs.t >= rp.tau_max);
            if (lane == 0) {
                atomicAdd(&rp.work[7], (unsigned long long)used);
                atomicAdd(&rp.work[12], (unsigned long long)__popcll(stopped));
                atomicMax(&rp.work[13], (unsigned long long)used);
            }
        }
    }
}

// Zero every view's image before the segmented accumulation.
__global__ void __launch_bounds__(256)
k_zero_images(const DevView* __restrict__ views, int nv, int64_t pixels, float* __restrict__ images)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= pixels) return;
    const int v = find_view(nv, p, [&](int k) { return views[k].pix_off; });
    images[views[v].img_off + (p - views[v].pix_off)] = 0.0f;
}

// Pass B forward over fixed B_SEGMENT-entry segments of the sorted imaging-plane
// pair array (one wave each, balanced however long a tile's list is).
// Lane = entry: gather the record, compute its footprint mask on the
// entry's tile; then, per run of entries of one tile, the masks are
// bit-transposed and lane = pixel sums only the entries covering it. The
// partial pixel sums are added to the image when the tile changes.
__global__ void __launch_bounds__(RASTER_THREADS)
k_raster_b_fwd(const DevView* __restrict__ views, int nv, RasterParams rp, int64_t cap_c,
               const uint32_t* __restrict__ status, const uint32_t* __restrict__ pkey,
               const uint32_t* __restrict__ pvals, const float4* __restrict__ iq,
               const float2* __restrict__ iw, float* __restrict__ images, int vm)
{
    __shared__ float4 s_q[RASTER_WAVES][WAVE];
    __shared__ float2 s_w[RASTER_WAVES][WAVE];
    const int w = threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
    const TransposeLane tl = transpose_lane();
    const uint32_t ki = status[ST_PAIRS_I];
    const uint32_t nblk = (uint32_t)(((uint64_t)ki + (uint64_t)B_SEGMENT * RASTER_WAVES - 1) /
                                     ((uint64_t)B_SEGMENT * RASTER_WAVES));
    const uint64_t seg = (uint64_t)xcd_block(blockIdx.x, nblk) * RASTER_WAVES + w;
    const uint64_t p0 = (uint64_t)cap_c + seg * B_SEGMENT;
    const uint64_t pend = (uint64_t)cap_c + ki;
    if (p0 >= pend) return;
    const uint32_t p1 = (uint32_t)min(pend, p0 + B_SEGMENT);
    uint32_t cur = 0xFFFFFFFFu;
    float acc = 0.0f, px = 0.0f, py = 0.0f;
    int64_t pix = -1;
    unsigned long long n_iter = 0, n_hits = 0;   // work counters
    // software pipeline over the 64-entry steps: the records of step s + 1
    // and the keys and record ids of step s + 2 load while step s runs
    const uint32_t e0 = (uint32_t)p0 + lane;
    uint32_t key_n = e0 < p1 ? pkey[e0] : 0xFFFFFFFFu;
    uint32_t r_n = e0 < p1 ? pvals[e0] : 0u;
    float4 g_n = iq[r_n];
    float2 g2_n = iw[r_n];
    uint32_t key_nn = e0 + WAVE < p1 ? pkey[e0 + WAVE] : 0xFFFFFFFFu;
    uint32_t r_nn = e0 + WAVE < p1 ? pvals[e0 + WAVE] : 0u;
    for (uint32_t b0 = (uint32_t)p0; b0 < p1; b0 += WAVE) {
        const uint32_t e = b0 + lane;
        const bool in = e < p1;
        const uint32_t key = key_n;
        const float4 g = g_n;
        const float2 g2 = g2_n;
        key_n = key_nn;
        g_n = iq[r_nn];
        g2_n = iw[r_nn];
        key_nn = e + 2 * WAVE < p1 ? pkey[e + 2 * WAVE] : 0xFFFFFFFFu;
        r_nn = e + 2 * WAVE < p1 ? pvals[e + 2 * WAVE] : 0u;
        uint64_t m = 0ull;
        if (in) {
            s_q[w][lane] = g;
            s_w[w][lane] = g2;
            const TileCell tk = tile_cell_i(views, nv, key, vm != 0);
            if (g2.y != 0.0f)   // zero intensity adds nothing
                m = footprint_mask<false>(g.x, g.y, g.z, g.w, g2.x, rp.q_max, tk.tx, tk.ty);
        }
        wave_lds_sync();
        uint64_t rest = __ballot(in);
        while (rest != 0ull) {
            // the run of entries of the first remaining tile (keys are sorted)
            const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)key,
                                                                  __builtin_ctzll(rest));
            const uint64_t sel = __ballot(in && key == k) & rest;
            rest &= ~sel;
            if (k != cur) {   // tile change: flush the partial sums
                if (pix >= 0 && acc != 0.0f) unsafeAtomicAdd(&images[pix], acc);
                const TileCell tc = tile_cell_i(views, nv, k, vm != 0);
                const DevView& V = views[tc.v];
                px = tc.col + 0.5f;
                py = tc.row + 0.5f;
                pix = tc.inside ? V.img_off + (int64_t)tc.row * V.W + tc.col : -1;
                acc = 0.0f;
                cur = k;
            }
            uint64_t col = transpose64(((sel >> lane) & 1ull) ? m : 0ull, tl);
            if (pix < 0) col = 0ull;
            for (;;) {
                if (__ballot(col != 0ull) == 0ull) break;
                ++n_iter;
                if (col != 0ull) {
                    const int j = __builtin_ctzll(col);
                    col &= col - 1ull;
                    const float4 g = s_q[w][j];
                    const float2 g2 = s_w[w][j];
                    const float dx = px - g.x, dy = py - g.y;
                    const float q = quadform(g, g2.x, dx, dy);
                    if (q < rp.q_max) {
                        ++n_hits;
                        acc += (__expf(-0.5f * q) - rp.eps) * rp.inv1meps * g2.y;
                    }
                }
            }
        }
        wave_lds_sync();
    }
    if (pix >= 0 && acc != 0.0f) unsafeAtomicAdd(&images[pix], acc);
    if (rp.work) {
        n_hits = wave_sum_u64(n_hits);
        if (lane == 0) {
            atomicAdd(&rp.work[6], n_iter);
            atomicAdd(&rp.work[2], n_hits);
        }
    }
}

// Sum of the first cnt (up to 64) of a wave's records on the lane's pixel, for
// the kernels where a workgroup has a tile of the image.
struct TileSum {
    float acc = 0.0f;
    unsigned long long n_iter = 0, n_hits = 0;   // work counters

    __device__ __forceinline__ void add(const float4* q4, const float2* w2, uint32_t cnt,
                                        const TileCell& tc, const RasterParams& rp,
                                        const TransposeLane& tl)
    {
        const int lane = lane_id();
        const float px = tc.col + 0.5f, py = tc.row + 0.5f;
        uint64_t m = 0ull;
        if ((uint32_t)lane < cnt) {
            const float4 g = q4[lane];
            const float2 g2 = w2[lane];
            if (g2.y != 0.0f)   // zero intensity adds nothing
                m = footprint_mask<false>(g.x, g.y, g.z, g.w, g2.x, rp.q_max, tc.tx, tc.ty);
        }
        // the transpose exchanges bits between lanes: every lane takes part,
        // pixels outside the image drop their column afterwards
        uint64_t col = transpose64(m, tl);
        if (!tc.inside) col = 0ull;
        while (__ballot(col != 0ull) != 0ull) {
            ++n_iter;
            if (col != 0ull) {
                const int j = __builtin_ctzll(col);
                col &= col - 1ull;
                const float4 g = q4[j];
                const float2 g2 = w2[j];
                const float q = quadform(g, g2.x, px - g.x, py - g.y);
                if (q < rp.q_max) {
                    ++n_hits;
                    acc += (__expf(-0.5f * q) - rp.eps) * rp.inv1meps * g2.y;
                }
            }
        }
    }

    __device__ __forceinline__ void count(const RasterParams& rp) const
    {
        if (!rp.work) return;
        const unsigned long long hits = wave_sum_u64(n_hits);
        if (lane_id() == 0) {
            atomicAdd(&rp.work[6], n_iter);
            atomicAdd(&rp.work[2], hits);
        }
    }
};

constexpr int BT_WAVES = 8;

// The waves' sums in wave order, stored once per pixel.
__device__ __forceinline__ void store_tile(float (*s_acc)[WAVE], int w, float acc,
                                           const TileCell& tc, const DevView& V,
                                           float* __restrict__ images)
{
    const int lane = lane_id();
    s_acc[w][lane] = acc;
    __syncthreads();
    if (w != 0 || !tc.inside) return;
    float sum = 0.0f;
#pragma unroll
    for (int k = 0; k < BT_WAVES; ++k) sum += s_acc[k][lane];
    images[V.img_off + (int64_t)tc.row * V.W + tc.col] = sum;
}

// Deterministic pass B: a workgroup per imaging tile (bucket tiles_c + t), its
// list in equal runs of whole chunks over the waves, which take 64 entries at
// a time: lane = entry while the records load and the footprint masks form,
// then lane = pixel adding the entries that cover it in list order. Every
// pixel is written once, by a plain store on the zeroed image, from the
// waves' sums in their order, so repeated runs agree bit for bit. Bound by
// the longest list's chain of chunks (a wave per tile took 183 us for 24 views
// of 60k Gaussians).
__global__ void __launch_bounds__(BT_WAVES * WAVE)
k_raster_b_tile(const DevView* __restrict__ views, int nv, RasterParams rp, int64_t cap_c,
                int64_t tiles_c, const uint2* __restrict__ ranges_i,
                const uint32_t* __restrict__ pvals, const float4* __restrict__ iq,
                const float2* __restrict__ iw, float* __restrict__ images)
{
    __shared__ float4 s_q[BT_WAVES][WAVE];
    __shared__ float2 s_w[BT_WAVES][WAVE];
    __shared__ float s_acc[BT_WAVES][WAVE];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE), lane = lane_id();
    const uint2 rg = ranges_i[blockIdx.x];
    if (rg.y <= rg.x) return;
    const TransposeLane tl = transpose_lane();
    const TileCell tc = tile_cell(views, nv, tiles_c + blockIdx.x, false);
    const DevView& V = views[tc.v];
    const uint32_t chunks = (rg.y - rg.x + WAVE - 1) / WAVE;
    const uint32_t per = (chunks + BT_WAVES - 1) / BT_WAVES;
    const uint32_t e0 = min(rg.y, rg.x + (uint32_t)w * per * WAVE);
    const uint32_t e1 = min(rg.y, e0 + per * WAVE);
    TileSum sum;
    // records one chunk ahead, their ids two
    auto id = [&](uint32_t b) { return b + lane < e1 ? pvals[cap_c + b + lane] : 0u; };
    uint32_t r_n = id(e0);
    float4 g_n = iq[r_n];
    float2 g2_n = iw[r_n];
    r_n = id(e0 + WAVE);
    for (uint32_t b = e0; b < e1; b += WAVE) {
        s_q[w][lane] = g_n;
        s_w[w][lane] = g2_n;
        g_n = iq[r_n];
        g2_n = iw[r_n];
        r_n = id(b + 2 * WAVE);
        wave_lds_sync();
        sum.add(s_q[w], s_w[w], min(e1 - b, (uint32_t)WAVE), tc, rp, tl);
        wave_lds_sync();
    }
    store_tile(s_acc, w, sum.acc, tc, V, images);
}

// Pass B without lists, for few records per tile: a workgroup takes a tile
// of the image and goes over the view's records itself. Each wave takes an
// equal run of them, keeps those whose rectangle has the tile and whose
// intensity is not zero, and adds them to its pixels 64 at a time as pass B
// does; the waves' sums meet in LDS and every pixel is stored once. It takes
// the place of the scan, the emission, the sort (3 to 6 launches), the
// zeroing and the tile sums, which were bound by their launches. Also counts
// the pairs the lists would have (for the overflow flag).
__global__ void __launch_bounds__(BT_WAVES * WAVE)
k_raster_b_direct(const DevView* __restrict__ views, int nv, RasterParams rp, int64_t tiles_c,
                  int64_t cap_i, const uint32_t* __restrict__ bsum, int64_t nbsum,
                  uint32_t* __restrict__ status, const uint2* __restrict__ rect,
                  const float4* __restrict__ iq, const float2* __restrict__ iw,
                  float* __restrict__ images)
{
    __shared__ float4 s_q[BT_WAVES][2 * WAVE];
    __shared__ float2 s_w[BT_WAVES][2 * WAVE];
    __shared__ float s_acc[BT_WAVES][WAVE];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE), lane = lane_id();
    const TransposeLane tl = transpose_lane();
    const TileCell tc = tile_cell(views, nv, tiles_c + blockIdx.x, false);
    const DevView& V = views[tc.v];
    const int64_t rec0 = V.rec_off;
    const int n = V.n, chunks = (n + WAVE - 1) / WAVE, per = (chunks + BT_WAVES - 1) / BT_WAVES;
    const int c0 = w * per, c1 = min(chunks, c0 + per);
    const uint32_t tx = (uint32_t)tc.tx, ty = (uint32_t)tc.ty;
    TileSum sum;
    uint32_t kept = 0u;
    auto put = [&](float4 g, float2 g2) {
        const bool hit = g2.y != 0.0f;   // zero intensity adds nothing
        const uint64_t m = __ballot(hit);
        if (m == 0ull) return;
        if (hit) {
            const uint32_t at = kept + lanes_below(m);
            s_q[w][at] = g;
            s_w[w][at] = g2;
        }
        kept += (uint32_t)__popcll(m);
        wave_lds_sync();
        if (kept < WAVE) return;
        sum.add(s_q[w], s_w[w], WAVE, tc, rp, tl);
        kept -= WAVE;
        wave_lds_sync();
        if ((uint32_t)lane < kept) {
            s_q[w][lane] = s_q[w][WAVE + lane];
            s_w[w][lane] = s_w[w][WAVE + lane];
        }
        wave_lds_sync();
    };
    constexpr int AHEAD = 4;   // chunks whose loads are in flight together
    for (int cb = c0; cb < c1; cb += AHEAD) {
        uint2 rc[AHEAD];
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            const int p = (cb + k) * WAVE + lane;
            rc[k] = cb + k < c1 && p < n ? rect[rec0 + p] : make_uint2(0u, 0u);
        }
        float4 g[AHEAD];
        float2 g2[AHEAD];
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            const int64_t r = rec0 + (cb + k) * WAVE + lane;
            g[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            g2[k] = make_float2(0.0f, 0.0f);
            if (tx >= (rc[k].x & 0xFFFFu) && tx < rc[k].x >> 16 && ty >= (rc[k].y & 0xFFFFu) &&
                ty < rc[k].y >> 16) {
                g[k] = iq[r];
                g2[k] = iw[r];
            }
        }
        put(g[0], g2[0]);
        put(g[1], g2[1]);
        put(g[2], g2[2]);
        put(g[3], g2[3]);
    }
    if (kept) sum.add(s_q[w], s_w[w], kept, tc, rp, tl);
    store_tile(s_acc, w, sum.acc, tc, V, images);
    if (blockIdx.x == 0 && w == 1) {
        unsigned long long pairs = 0ull;
        for (int64_t k = lane; k < nbsum; k += WAVE) pairs += bsum[k];
        pairs = wave_sum_u64(pairs);
        if (lane == 0) {
            const bool over = pairs > (unsigned long long)cap_i;
            status[ST_OVERFLOW] |= over ? 1u : 0u;
            status[ST_PAIRS_I] = over ? 0u : (uint32_t)pairs;
        }
    }
    sum.count(rp);
}

struct __attribute__((packed, aligned(4))) Float4Unaligned { float v[4]; };

// Imaging-plane backward, one thread per used record (view, Gaussian): the
// additive image formation has no order, so each thread walks its own
// footprint ellipse q < q_max row by row (exact column span from the conic,
// widened by one pixel), gathers dL/dS there and keeps its moments about the
// centre in registers -- no atomics, no tile list; dL/dI and the centre and
// conic gradients are linear in those. Bound by the address units, a lane's
// pixels lying in lines of their own: 16 views of a 2M-Gaussian block take
// 3.2 ms, with a load per pixel 4.3; then by the records' bytes (72 views of one
// vehicle of 200k 179 -> 168 us; of the one bench.py draws, with more and larger
// footprints, the stage hardly gained: 262 -> 260). It also clears the record's computation-plane gradient
// sums for pass A.
__global__ void __launch_bounds__(256)
k_image_bwd(const DevView* __restrict__ views, const DevScene* __restrict__ scenes, int nv,
            int64_t records, RasterParams rp, const uint32_t* __restrict__ status,
            const uint32_t* __restrict__ active, const float4* __restrict__ iq,
            const float2* __restrict__ iw, const float* __restrict__ prec,
            const float* __restrict__ dimg, float* __restrict__ grad_i,
            CRec* __restrict__ crec, float* __restrict__ grad_c)
{
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if ((int64_t)blockIdx.x * blockDim.x >= (int64_t)status[ST_ACTIVE]) return;
    unsigned long long hits = 0;
    if (t0 < (int64_t)status[ST_ACTIVE]) {
    const int64_t r = active[t0];
    const int v = find_view(nv, r, [&](int k) { return views[k].rec_off; });
    const DevView& V = views[v];
    const float4 g = iq[r];
    const float2 g2 = iw[r];
    const float a = g.z, b = g.w, c = g2.x, I = g2.y;
    const float det = a * c - b * b;
    float dI = 0.f, dcx = 0.f, dcy = 0.f, da = 0.f, db = 0.f, dc = 0.f;
    if (det > 0.0f && a > 0.0f) {
        const float qm = rp.q_max;
        const float ry = sqrtf(qm * a / det);
        const int W = V.W;
        // clamp in float before converting (far-away centres stay in range)
        const int row0 = (int)fmaxf(0.0f, ceilf(g.y - ry - 0.5f) - 1.0f);
        const int row1 = (int)fminf((float)(V.H - 1), floorf(g.y + ry - 0.5f) + 1.0f);
        // the column span only bounds the pixels tested (one pixel of slack
        // each side; q < q_max decides), so 1/a by one reciprocal is enough
        const float inv_a = 1.0f / a;
        const float* G = dimg + V.img_off;
        float sG = 0.f, s0 = 0.f, sx = 0.f, sy = 0.f, sxx = 0.f, sxy = 0.f, syy = 0.f;
        for (int row = row0; row <= row1; ++row) {
            const float dy = row + 0.5f - g.y;
            const float D = a * qm - det * dy * dy;
            if (D < -1e-4f * a * qm) continue;   // rows an FP32 q < q_max can still reach
            const float half = sqrtf(fmaxf(D, 0.0f)) * inv_a;
            const float xc = g.x - b * dy * inv_a;
            const int col0 = (int)fmaxf(0.0f, ceilf(xc - half - 0.5f) - 1.0f);
            const int col1 = (int)fminf((float)(W - 1), floorf(xc + half - 0.5f) + 1.0f);
            const float* Grow = G + (int64_t)row * W;
            // sums over the row of w, w dx and w dx^2, w = G e
            float r0 = 0.f, r1 = 0.f, r2 = 0.f;
            // four columns' cotangents in one load (the columns past the span
            // are not used; past the row's end they are not read)
            for (int c0 = col0; c0 <= col1; c0 += 4) {
                Float4Unaligned Gq;
                if (c0 + 3 < W) {
                    Gq = *reinterpret_cast<const Float4Unaligned*>(Grow + c0);
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) Gq.v[u] = c0 + u < W ? Grow[c0 + u] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int col = c0 + u;
                    const float dx = col + 0.5f - g.x;
                    const float q = quadform(g, c, dx, dy);
                    const bool in = q < qm && col <= col1;
                    if (rp.work) hits += in ? 1ull : 0ull;
                    const float Gp = in ? Gq.v[u] : 0.0f;
                    const float w = in ? Gq.v[u] * __expf(-0.5f * q) : 0.0f;
                    const float wx = w * dx;
                    sG += Gp;
                    r0 += w;
                    r1 += wx;
                    r2 += wx * dx;
                }
            }
            s0 += r0;
            sx += r1;
            sy += dy * r0;
            sxx += r2;
            sxy += dy * r1;
            syy += dy * dy * r0;
        }
        // (an infinite cotangent, of whichever sign, outweighs the rest: the
        // difference would make it NaN)
        dI = (isinf(s0) ? s0 : s0 - rp.eps * sG) * rp.inv1meps;
        const float k = -0.5f * I * rp.inv1meps;   // dL/dq = k w
        dcx = -2.0f * k * (a * sx + b * sy);
        dcy = -2.0f * k * (b * sx + c * sy);
        da = k * sxx;
        db = 2.0f * k * sxy;
        dc = k * syy;
    }
    float4* gi = reinterpret_cast<float4*>(grad_i + r * GC_STRIDE);
    gi[0] = make_float4(dcx, dcy, da, db);
    gi[1] = make_float4(dc, dI, 0.0f, 0.0f);
    // c = P dL/dI for pass A (P the record's phase factor), in the record
    // pass A's backward gathers per hit
    reinterpret_cast<float*>(&crec[r].w)[3] =
        (prec ? prec[r] : scenes[V.scene].amp[r - V.rec_off] * (float)V.pscale) * dI;
    // pass A backward adds into the record's computation-plane sums
    float4* gc = reinterpret_cast<float4*>(grad_c + r * GC_STRIDE);
    gc[0] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    gc[1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    if (rp.work) {   // one atomic per wave
#pragma unroll
        for (int d = 1; d < WAVE; d <<= 1)
            hits += (unsigned long long)__shfl_xor((long long)hits, d, WAVE);
        if (lane_id() == 0 && hits) atomicAdd(&rp.work[3], hits);
    }
}

// Pass A backward, same tiling, chunk batches and hit compaction as the
// forward, but back to front from each ray's last contributing entry:
// tau -= kappa f, dL/dalpha = exp(-tau) (c - U), U <- c alpha + (1 - alpha) U,
// with c = P dL/dI. A ray takes part in a chunk only if it used an entry at
// or past the chunk's start in the forward, so the chunks behind the point
// where most rays saturated are skipped as in the forward. Within a round
// (lane = hit, hits of a ray back to front) the optical depth is a
// segmented prefix sum and U a segmented prefix composition of the affine
// maps U -> (1 - alpha) U + c alpha. The six per-entry gradient sums collect
// in LDS and leave with one global atomic each per (tile, entry).
// Two variants, by list length (the worklist holds the long lists first;
// when long lists are the majority the first variant runs every tile):
//   FLUSHER (lists of at least 2^(LONG_LIST_BITS - 1) entries): a second wave
//     of the workgroup sends each batch's atomics while the first goes on,
//     so a long chain of batches never waits on them; two sum buffers;
//   short lists: one wave sends its own atomics, one buffer: less LDS, so
//     more tiles run per CU.
// The short lists are bound by the float atomics, which every XCD sends on to
// memory: a request per entry and sum was 148M requests and 9.1 ms of the
// 16-view block of 2M Gaussians (10.6 ms both variants); eight entries to an
// instruction, the six sums of one in one request, and batches of 4 chunks
// (24 KB of LDS instead of 48) made both variants 5.0 ms.
constexpr int LONG_LIST_BITS = 12;

// Hits of a compaction group of the backward: all of a batch's when at most
// BG_HITS are left, else each ray's next BG_RAY.
constexpr uint32_t BG_RAY = 32, BG_HITS = WAVE * BG_RAY;

// Tiles a workgroup looks at for one without stored hits (none has them in
// most calls: a workgroup per tile that only finds its own stored took the
// two launches 38 us for the 74k tiles of 72 views).
constexpr int BWD_TILES = 8;

template <bool FLUSHER, bool DET>
__global__ void __launch_bounds__(FLUSHER ? 2 * WAVE : WAVE) __attribute__((amdgpu_waves_per_eu(1, 2)))
k_raster_a_bwd(const DevView* __restrict__ views, int nv,
               RasterParams rp, const uint32_t* __restrict__ status,
               const uint32_t* __restrict__ worklist, const uint2* __restrict__ ranges,
               const uint32_t* __restrict__ pvals, const uint64_t* __restrict__ pmask,
               const uint64_t* __restrict__ psum, const CRec* __restrict__ crec,
               const float* __restrict__ tau, const uint32_t* __restrict__ nlast,
               float* __restrict__ grad_c, int64_t stride)
{
    constexpr int NB = A_BATCH;
    constexpr int HKB = 2;         // bits of a hit's chunk index
    constexpr int HRS = 6 + HKB;   // shift of a hit's ray index
    static_assert(NB == 1 << HKB, "chunk index bits");
    __shared__ float4 s_rec[NB][2 * WAVE];   // both halves of each entry's record
    // per-entry gradient sums (rows padded by one: they differ in bank), in
    // two buffers with the flusher: the second wave of the workgroup sends
    // one batch's sums with atomics while the first accumulates the next
    // batch in the other
    constexpr int GB = FLUSHER ? 2 : 1;
    __shared__ double s_G[GB][NB][6][WAVE + 1];
    __shared__ uint32_t s_rf[GB][FLUSHER ? NB : 1][WAVE];   // records of the handed-off entries
    __shared__ uint2 s_list[WAVE];            // entries being sent: lane, destination
    __shared__ uint32_t s_cmd[GB][WAVE];      // per entry lane: chunks gathered (bits), last flag
    __shared__ uint32_t s_chk[NB];
    __shared__ uint16_t s_hit[BG_HITS];    // (ray, chunk, entry) packed, ray-major, back to front
    // per ray during a chunk: first hit in s_hit, optical depth, U
    struct alignas(16) RayB { uint32_t o; float t, U, pad; };
    __shared__ RayB s_ray[WAVE];
    // worklist entries [0, nlong) hold the long lists; when they are the
    // majority the run is bound by their chains and the flusher variant
    // takes every tile (short ones then fill its gaps)
    const uint32_t ntiles = status[ST_WORK_TILES];
    uint32_t nlong = status[WL_BINS_WORD + 33 + LONG_LIST_BITS];
    if (2u * nlong >= ntiles) nlong = ntiles;
    const uint32_t w0 = FLUSHER ? 0u : nlong, w1 = FLUSHER ? nlong : ntiles;
    // tiles whose hits the forward stored run in k_raster_a_bwd_hits, mostly
    // all of them: a workgroup then looks at BWD_TILES tiles for one without
    uint64_t todo_tiles = w0 + blockIdx.x < w1 ? 1ull : 0ull;
    if (!DET && rp.hits != nullptr) {
        const uint32_t wi = w0 + blockIdx.x + (uint32_t)lane_id() * gridDim.x;
        todo_tiles = __ballot(lane_id() < BWD_TILES && wi < w1 &&
                              rp.hit_tail[worklist[min(wi, w1 - 1u)]] == HIT_OVERFLOW);
    }
    constexpr uint32_t LAST = 1u << 31;
    // The six sums of a batch's touched entries (cmd: their chunks per lane,
    // rec: where each lane's go) leave with one atomic each, eight entries to
    // an instruction: the lanes of one entry add to one 32-byte row, which is
    // one request to memory instead of six. The sums are cleared for reuse.
    auto send = [&](int hb, uint32_t cmd, const uint32_t (&rec)[NB]) {
        const int lane = lane_id();
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const uint64_t m = __ballot((cmd >> k) & 1u);
            if (m == 0ull) continue;
            if ((cmd >> k) & 1u) {
                const uint32_t at = lanes_below(m);
                s_list[at] = make_uint2((uint32_t)lane, rec[k]);
            }
            wave_lds_sync();
            const int n = __popcll(m), c = lane & 7;
            for (int e = lane >> 3; e < n; e += WAVE / 8) {
                if (c >= 6) continue;
                const uint2 el = s_list[e];
                const float v = (float)s_G[hb][k][c][el.x];
                s_G[hb][k][c][el.x] = 0.0;
                if (v == 0.0f) continue;
                if constexpr (DET) rp.part[(int64_t)el.y * PART_G + c] = v;
                else unsafeAtomicAdd(&grad_c[(int64_t)el.y * GC_STRIDE + c], v);
            }
            wave_lds_sync();
        }
    };
    while (todo_tiles != 0ull) {   // the same for both waves
        const uint32_t wi = w0 + blockIdx.x + (uint32_t)__builtin_ctzll(todo_tiles) * gridDim.x;
        todo_tiles &= todo_tiles - 1ull;
        if (FLUSHER && threadIdx.x >= WAVE) {
            // the flusher: per hand-off, the six sums of every handed-off entry
            // leave with one atomic each, and the buffer is cleared for reuse
            const int fl = threadIdx.x - WAVE;
            for (int hb = 0;; hb ^= 1) {
                __syncthreads();
                const uint32_t cmd = s_cmd[hb][fl];
                uint32_t rec[NB];
#pragma unroll
                for (int k = 0; k < NB; ++k) rec[k] = s_rf[hb][k][fl];
                send(hb, cmd, rec);
                if (cmd & LAST) break;
            }
            __syncthreads();
            continue;
        }
        const int lane = threadIdx.x;
        const TransposeLane tl = transpose_lane();
        const int64_t bucket = worklist[wi];
        const TileCell tc = tile_cell(views, nv, bucket, true);
        const DevView& V = views[tc.v];
        const float x0 = (float)(tc.tx * TILE) + 0.5f, y0 = (float)(tc.ty * TILE) + 0.5f;
        const uint2 rg = ranges[bucket];
        const int64_t ray = V.ray_off + (int64_t)tc.row * V.Wc + tc.col;
        const uint32_t n_mine = tc.inside ? nlast[ray] : 0u;   // entries [0, n_mine) were used
        float t = tc.inside ? tau[ray] : 0.0f;
        float U = 0.0f;
#pragma unroll
        for (int b = 0; b < GB; ++b)
#pragma unroll
            for (int k = 0; k < NB; ++k)
#pragma unroll
                for (int c = 0; c < 6; ++c) s_G[b][k][c][lane] = 0.0;
        unsigned long long n_iter = 0, n_hits = 0;   // work counters
        unsigned long long n_batch = 0, n_extra = 0;
        const uint32_t n_max = wave_max_u32(n_mine);
        const uint32_t e_end = rg.x + n_max;           // exclusive end of the used entries
        // the six per-entry sums of the last processed batch leave once the next
        // batch's loads have landed: handed to the flusher wave (the barrier also
        // returns the buffer it emptied last), or sent by this wave before the
        // next batch accumulates into the same buffer
        uint32_t got_prev = 0u;
        // where each entry's sums go: its record, or in deterministic mode its
        // pair's position before the sort
        uint32_t r_prev[NB], r_cur[NB];
        int hb = 0;                        // buffer the current batch accumulates in
        auto flush = [&](bool last) {
            if constexpr (FLUSHER) {
#pragma unroll
                for (int k = 0; k < NB; ++k) s_rf[hb][k][lane] = r_prev[k];
                s_cmd[hb][lane] = got_prev | (last ? LAST : 0u);
                __syncthreads();
                hb ^= 1;
            } else {
                send(0, got_prev, r_prev);
            }
            got_prev = 0u;
        };
        // One round of up to 64 hits, lane = hit (each ray's hits contiguous,
        // back to front; `head` marks a ray's first hit in the round, rs is its
        // state before the round): optical depths and U by segmented scans, the
        // per-entry gradient sums into LDS, each ray's state after its last hit
        // back to s_ray.
        auto hit_round = [&](const uint32_t hv, const bool valid, const bool head, const RayB rs) {
            const int rr = (int)(hv >> HRS), k = (int)((hv >> 6) & ((1u << HKB) - 1u)),
                      j = (int)(hv & 63u);
            const float4 g = s_rec[k][2 * j], g2 = s_rec[k][2 * j + 1];
            const float cj = g2.w;
            bool real = false;
            float x = 0.0f, E = 1.0f, ex = 0.0f, f = 0.0f, dx = 0.0f, dy = 0.0f;
            float c = 0.0f;
            if (valid) {
                dx = x0 + (float)(rr & (TILE - 1)) - g.x;
                dy = y0 + (float)(rr / TILE) - g.y;
                const float q = quadform(g, g2.x, dx, dy);
                if (q < rp.q_max) {
                    real = true;
                    c = cj;
                    ex = __expf(-0.5f * q);
                    f = (ex - rp.eps) * rp.inv1meps;
                    x = g2.y * f;
                    E = __expf(-x);
                }
            }
            const float sx = seg_incl_scan(x, head);   // this and the later hits
            float sa = E, sb = real ? c * (1.0f - E) : 0.0f;
            seg_incl_affine(sa, sb, head);
            float ea = __int_as_float(from_lane_below(__float_as_int(sa)));
            float eb = __int_as_float(from_lane_below(__float_as_int(sb)));
            if (head) {
                ea = 1.0f;
                eb = 0.0f;
            }
            const float tr = valid ? rs.t : 0.0f;
            const float Ur = valid ? rs.U : 0.0f;
            if (real) {
                float dalpha;
                if (rp.shadowing) {
                    const float Tn = __expf(-fmaxf(tr - sx, 0.0f));
                    dalpha = Tn * (c - (ea * Ur + eb));
                } else {
                    dalpha = c;
                }
                const float dxx = dalpha * E;   // d alpha / d x = exp(-x)
                const float dq = dxx * g2.y * (-0.5f * ex * rp.inv1meps);
                atomicAdd(&s_G[hb][k][0][j], (double)(-2.0f * dq * (g.z * dx + g.w * dy)));
                atomicAdd(&s_G[hb][k][1][j], (double)(-2.0f * dq * (g.w * dx + g2.x * dy)));
                atomicAdd(&s_G[hb][k][2][j], (double)(dq * dx * dx));
                atomicAdd(&s_G[hb][k][3][j], (double)(2.0f * dq * dx * dy));
                atomicAdd(&s_G[hb][k][4][j], (double)(dq * dy * dy));
                atomicAdd(&s_G[hb][k][5][j], (double)(dxx * f));
            }
            const uint64_t hbits = __ballot(real);
            if (lane == 0) n_hits += (unsigned long long)__popcll(hbits);
            const int nxt = from_lane_above(valid ? (int)hv : -1);
            const bool endseg = valid && (lane == WAVE - 1 || (nxt >> HRS) != rr);
            wave_lds_sync();
            if (endseg && rp.shadowing) s_ray[rr] = RayB{rs.o, tr - sx, sa * Ur + sb, 0.0f};
            wave_lds_sync();
        };
        const int64_t c_first = rg.x / WAVE, c_end = (int64_t)(e_end + WAVE - 1) / WAVE;
        for (int64_t g1 = c_end; g1 > c_first && n_max > 0u; g1 -= WAVE) {
            const int64_t g0 = max(c_first, g1 - (int64_t)WAVE);
            // lane = chunk g0 + lane: the rays that used an entry at or past its start
            const int64_t cpos = (g0 + lane) * WAVE - (int64_t)rg.x;
            uint64_t live_c = 0ull;
            for (int rr = 0; rr < WAVE; ++rr) {
                const uint32_t nm = (uint32_t)__builtin_amdgcn_readlane((int)n_mine, rr);
                if ((int64_t)nm > cpos) live_c |= 1ull << rr;
            }
            const uint64_t sm = g0 + lane < g1 ? psum[g0 + lane] : 0ull;
            uint64_t todo = __ballot((sm & live_c) != 0ull);   // chunks to read, back to front
            // up to NB chunks per batch: their masks and values are fetched one
            // batch ahead (in flight while the current batch's hits are
            // processed), then the records the rays need
            uint32_t chk_n[NB], rec_n[NB], r_n[NB];
            uint64_t lv_n[NB], m_n[NB];
            int nb_n = 0;
            auto fetch = [&]() {
                nb_n = 0;
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    chk_n[k] = 0u;
                    lv_n[k] = 0ull;
                    if (todo != 0ull) {
                        const int hi = 63 - __builtin_clzll(todo);
                        todo &= ~(1ull << hi);
                        chk_n[k] = (uint32_t)g0 + (uint32_t)hi;
                        const uint32_t l0 =
                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)live_c, hi);
                        const uint32_t l1 =
                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(live_c >> 32), hi);
                        lv_n[k] = ((uint64_t)l1 << 32) | l0;
                        nb_n = k + 1;
                    }
                }
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    const uint32_t e = chk_n[k] * WAVE + lane;
                    const bool in = k < nb_n && e >= rg.x && e < e_end;
                    m_n[k] = in ? pmask[e] : 0ull;
                    rec_n[k] = in ? pvals[e] : 0u;
                    if constexpr (DET) r_n[k] = in ? rp.ppos[e] : 0u;
                    else r_n[k] = rec_n[k];
                }
            };
            fetch();
            while (nb_n > 0) {
                ++n_batch;
                uint32_t got = 0u;
                const int nb = nb_n;
                uint64_t m[NB];   // lane = entry: the cells it covers
                {
                    uint32_t chk[NB];
                    uint64_t lv[NB];
                    uint32_t* r = r_cur;
                    uint32_t rec[NB];
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        chk[k] = chk_n[k];
                        lv[k] = lv_n[k];
                        m[k] = m_n[k];
                        rec[k] = rec_n[k];
                        r[k] = r_n[k];
                    }
                    // records straight into LDS, all in flight together (entries
                    // no ray needs read record 0 of the view, one shared line)
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        const bool need = (m[k] & lv[k]) != 0ull;
                        got |= need ? 1u << k : 0u;
                        load_recs_to_lds(crec, need ? rec[k] : (uint32_t)V.rec_off, &s_rec[k][0]);
                    }
#pragma unroll
                    for (int k = 0; k < NB; ++k)
                        if (lane == k) s_chk[k] = chk[k];
                }
                wait_all_memory();
                wave_lds_sync();
                fetch();   // the next batch's masks and values
                flush(false);
                got_prev = got;
#pragma unroll
                for (int k = 0; k < NB; ++k) r_prev[k] = r_cur[k];
                // the batch's chunks, transposed: bit j of col[k] is entry j of
                // chunk k covering my cell that my ray used in the forward
                // (all transposed together, as in the forward)
                uint64_t col[NB];
#pragma unroll
                for (int k = 0; k < NB; ++k) col[k] = m[k];
                transpose64_n(col, tl);
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    uint64_t used = 0ull;
                    if (k < nb) {
                        const int64_t pos0 = (int64_t)s_chk[k] * WAVE - rg.x;
                        const int64_t nu = (int64_t)n_mine - pos0;   // used: positions < n_mine
                        used = nu >= WAVE ? ~0ull : (nu <= 0 ? 0ull : ((1ull << nu) - 1ull));
                    }
                    col[k] &= used;
                }
                // the batch's hits in groups, compacted ray-major, back to front
                // (the batch's chunks come back to front), and taken 64 per
                // round: all that are left when they are few, else each ray's
                // next BG_RAY
                for (bool more = false;; more = true) {
                    uint32_t nr = 0;
#pragma unroll
                    for (int k = 0; k < NB; ++k) nr += (uint32_t)__popcll(col[k]);
                    if (__ballot(nr != 0u) == 0ull) break;
                    n_extra += more ? 1u : 0u;
                    // hits left and hits of a limited group, scanned together
                    // (at most 64 x 256 and 64 x BG_RAY: two to a word)
                    const uint32_t lim = min(nr, BG_RAY);
                    const uint32_t both = nr | (lim << 16);
                    const uint32_t excl = wave_excl_scan_u32(both);
                    const uint32_t tot =
                        (uint32_t)__builtin_amdgcn_readlane((int)(excl + both), WAVE - 1);
                    const bool few = (tot & 0xFFFFu) <= BG_HITS;
                    const uint32_t H = few ? (tot & 0xFFFFu) : (tot >> 16);
                    const uint32_t o = few ? (excl & 0xFFFFu) : (excl >> 16);
                    const uint32_t o_end = o + (few ? nr : lim);
                    {
                        uint32_t w = o;
#pragma unroll
                        for (int k = 0; k < NB; ++k) {
                            uint32_t half[2] = {(uint32_t)col[k], (uint32_t)(col[k] >> 32)};
#pragma unroll
                            for (int q = 1; q >= 0; --q) {
                                const uint32_t tag =
                                    (uint32_t)((lane << HRS) | (k << 6) | (q << 5));
                                while (half[q] != 0u && w < o_end) {
                                    const uint32_t j = 31u - (uint32_t)__builtin_clz(half[q]);
                                    half[q] &= ~(1u << j);
                                    s_hit[w++] = (uint16_t)(tag | j);
                                }
                            }
                            col[k] = ((uint64_t)half[1] << 32) | half[0];
                        }
                        s_ray[lane] = RayB{o, t, U, 0.0f};
                        wave_lds_sync();
                        for (uint32_t base = 0; base < H; base += WAVE) {
                            ++n_iter;
                            const uint32_t L = base + lane;
                            const bool valid = L < H;
                            const uint32_t hv = valid ? (uint32_t)s_hit[L] : 0u;
                            // ray state (lanes past the last hit read ray 0 and ignore it)
                            const RayB rs = s_ray[hv >> HRS];
                            const int seg0 = valid ? max((int)rs.o - (int)base, 0) : lane;
                            hit_round(hv, valid, lane == seg0, rs);
                        }
                        {
                            const RayB rs = s_ray[lane];
                            t = rs.t;
                            U = rs.U;
                        }
                        wave_lds_sync();
                    }
                }
                wave_lds_sync();
            }
        }
        flush(true);
        if (rp.work) {
            n_hits = wave_sum_u64(n_hits);
            if (lane == 0) {
                atomicAdd(&rp.work[5], n_iter);
                atomicAdd(&rp.work[1], n_hits);
                atomicMax(&rp.work[9], n_batch);
                atomicAdd(&rp.work[11], n_extra);
                atomicAdd(&rp.work[FLUSHER ? 14 : 15], 1ull);
                atomicAdd(&rp.work[17], 1ull);
            }
        }
        if constexpr (FLUSHER) __syncthreads();
        else wave_lds_sync();
    }
}

// Pass A backward over the hits the forward stored (RasterParams::hits).
// A workgroup takes a tile and walks its records back to front. The chain
// along the rays (optical depth and U, carried from hit to hit) is serial,
// everything else is not, so the work is split over its waves, a step being
// up to HB_HELPERS rounds of 64 hits from the back of one record:
//   helper waves, one round of the step each: the chain of loads (hit words
//     of the step three ahead, list entries' record ids, records), then the
//     footprint, x = kappa f and c = P dL/dI of each hit, handed to the main
//     wave one step ahead; one step later the six gradient terms
//     from the main wave's dL/dx, added per entry slot of the batch in LDS;
//   the main wave: the rounds of the step one after the other, lane = hit
//     (each ray's hits contiguous and back to front): optical depths and U by
//     segmented scans, dL/dx per hit, each ray's state after its last hit.
// Once a batch's records are done, one more wave stores each touched entry's
// six sums with plain stores at its pair's position before the pair sort and
// marks it (a buffer per batch, two in turn), and launch_reduce_touched adds
// them per record (float atomics, one per sum, would cost several times the
// whole pass); an entry whose record has no other tile stores its sums as the
// record's directly. One barrier per step. One wave that loaded, evaluated
// and scanned its rounds alone, with a second one storing, took 2.8 us per
// round on the longest tiles (a full memory latency in each, however far
// ahead the loads were issued).
// Records that do not fit the stream, record numbers that do not fall along
// the walk, record ids past the record count and list positions past the pair
// count end the walk or are skipped, so a stream that holds anything else
// cannot send the kernel out of bounds or keep it going.
constexpr int HB_HELPERS = 4;
constexpr int HB_THREADS = (2 + HB_HELPERS) * WAVE;

// A step's rounds: the stream index of the first of its n hit words (n = 0
// once the chain is done; round r's lane i takes word base + n - 1 - 64 r -
// i), whether it ends its batch, the batch's buffer and its chunks' list
// positions / 64 (lane k: chunk k).
struct HitStep {
    uint64_t base;
    uint32_t n, chunks;
    int buf;
    bool last;
};

// What a helper keeps of a hit from its evaluation to its gradient terms.
struct HitTerm {
    float dx, dy, a, b, c, dqx, f;   // offsets, conic, d(q)/d(x) factor, footprint
    uint32_t id, pos;                // record and pair position (HIT_NONE: it has one tile)
    uint32_t slot;                   // entry slot, bit 16: inside the footprint
};

// (80 registers: four workgroups to a CU instead of three, 36 views of 50k
// Gaussians 229 -> 197 us)
__global__ void __launch_bounds__(HB_THREADS) __attribute__((amdgpu_waves_per_eu(6, 6)))
k_raster_a_bwd_hits(const DevView* __restrict__ views, int nv, RasterParams rp,
                    const uint32_t* __restrict__ status, const uint32_t* __restrict__ worklist,
                    const uint32_t* __restrict__ pvals, const CRec* __restrict__ crec,
                    const float* __restrict__ tau, float* __restrict__ grad_c, int64_t stride)
{
    // per batch buffer: the slots' sums, each touched slot's record
    // (HIT_NONE: untouched) and pair position (HIT_NONE: the record has only
    // this tile)
    __shared__ double s_G[2][6][HB_SLOTS];
    __shared__ uint32_t s_rec[2][HB_SLOTS];
    __shared__ uint32_t s_pos[2][HB_SLOTS];
    // per batch, two in turn: record id and pair position of its list entries
    __shared__ uint2 s_ent[2][HB_SLOTS];
    // per step, two in turn: x (then dL/dx), c and the ray (-1: no hit) of
    // each hit, the step's hits, and the batch buffer it completes (2: none)
    __shared__ float2 s_in[2][HB_HELPERS][WAVE];
    __shared__ signed char s_key[2][HB_HELPERS][WAVE];
    __shared__ uint32_t s_n[2], s_done[2];
    __shared__ float2 s_ray[WAVE];   // per ray: optical depth, U
    if (blockIdx.x >= status[ST_WORK_TILES]) return;
    const int64_t bucket = worklist[blockIdx.x];
    const uint32_t tail = rp.hit_tail[bucket];
    if (tail == HIT_OVERFLOW) return;   // k_raster_a_bwd re-derives this tile's hits
    for (int i = threadIdx.x; i < 2 * HB_SLOTS; i += HB_THREADS) {
        (&s_rec[0][0])[i] = HIT_NONE;
#pragma unroll
        for (int c = 0; c < 6; ++c) s_G[i / HB_SLOTS][c][i % HB_SLOTS] = 0.0;
    }
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
    const TileCell tc = tile_cell(views, nv, bucket, true);
    const DevView& V = views[tc.v];

    if (wave == 0) {   // the main wave
        const int64_t ray = V.ray_off + (int64_t)tc.row * V.Wc + tc.col;
        s_ray[lane] = make_float2(tc.inside ? tau[ray] : 0.0f, 0.0f);
        uint32_t n_iter = 0;   // work counter
        __syncthreads();
        for (int t = 0;; ++t) {
            const uint32_t n = s_n[t & 1];
            if (n == 0u) break;
            for (uint32_t r = 0; r * WAVE < n; ++r) {
                ++n_iter;
                float2& hit = s_in[t & 1][r][lane];
                const float2 in = hit;
                const int key = s_key[t & 1][r][lane];
                const float E = __expf(-in.x);
                const bool valid = key >= 0;
                const int rr = valid ? key : 0;
                const float2 rs = s_ray[rr];
                // the neighbours' rays, read by every lane (a cross-lane read
                // inside a condition would see the lanes it skips as zero)
                const int below = from_lane_below(key), above = from_lane_above(key);
                const bool head = !valid || lane == 0 || below != key;
                const float c = in.y;
                const float sx = seg_incl_scan(in.x, head);   // this and the later hits
                float sa = E, sb = c * (1.0f - E);
                seg_incl_affine(sa, sb, head);
                float ea = __int_as_float(from_lane_below(__float_as_int(sa)));
                float eb = __int_as_float(from_lane_below(__float_as_int(sb)));
                if (head) {
                    ea = 1.0f;
                    eb = 0.0f;
                }
                const float tr = valid ? rs.x : 0.0f;
                const float Ur = valid ? rs.y : 0.0f;
                float dalpha = c;
                if (rp.shadowing) {
                    const float Tn = __expf(-fmaxf(tr - sx, 0.0f));
                    dalpha = Tn * (c - (ea * Ur + eb));
                }
                hit.x = dalpha * E;   // d alpha / d x = exp(-x)
                const bool endseg = valid && (lane == WAVE - 1 || above != key);
                wave_lds_sync();
                if (endseg && rp.shadowing) s_ray[rr] = make_float2(tr - sx, sa * Ur + sb);
                wave_lds_sync();
            }
            __syncthreads();
        }
        // the helpers' last terms, then their last sums
        if (n_iter != 0u) __syncthreads();
        if (rp.work && lane == 0) {
            atomicAdd(&rp.work[5], (unsigned long long)n_iter);
            atomicAdd(&rp.work[16], 1ull);
        }
        return;
    }

    if (wave == 1 + HB_HELPERS) {
        // the storing wave, which loads nothing: a wait for a load would wait
        // for every store before it
        const uint32_t kc = status[ST_PAIRS_C];
        __syncthreads();
        // step t: the batch whose last terms were added in the step before
        bool drained = false;   // step t - 1 was the first empty one
        for (int t = 0;; ++t) {
            const uint32_t n = drained ? 0u : s_n[t & 1];
            const uint32_t fb = t > 0 ? s_done[(t - 1) & 1] : 2u;
            if (fb < 2u) {
#pragma unroll
                for (int i = 0; i < HB_CHUNKS; ++i) {
                    const int sl = i * WAVE + lane;
                    const uint32_t rk = s_rec[fb][sl];
                    if (rk == HIT_NONE) continue;
                    // one store path: a record with no other tile takes its
                    // sums directly (its eight floats: six sums and two
                    // spare), any other entry its pair's partial row (six
                    // sums, the record, a spare); the mark of a direct store
                    // lands in the spare byte at the pair count, which the
                    // reduction never reads
                    const uint32_t pos = s_pos[fb][sl];
                    const bool one = pos == HIT_NONE;
                    float v[6];
#pragma unroll
                    for (int c = 0; c < 6; ++c) {
                        v[c] = (float)s_G[fb][c][sl];
                        s_G[fb][c][sl] = 0.0;
                    }
                    s_rec[fb][sl] = HIT_NONE;
                    if (!one && pos >= kc) continue;
                    float4* dst = reinterpret_cast<float4*>(
                        one ? grad_c + (int64_t)rk * GC_STRIDE
                            : rp.hit_part + (uint64_t)pos * HIT_PART_STRIDE);
                    dst[0] = make_float4(v[0], v[1], v[2], v[3]);
                    dst[1] = make_float4(v[4], v[5], __uint_as_float(rk), 0.0f);
                    rp.hit_touched[one ? kc : pos] = 1;
                }
            }
            if (drained || (t == 0 && n == 0u)) return;
            __syncthreads();
            drained = n == 0u;
        }
    }

    // a helper wave
    const int hw = wave - 1;
    const uint32_t kc = status[ST_PAIRS_C];
    const uint32_t rec0 = (uint32_t)V.rec_off;   // read by lanes without a hit
    const float x0 = (float)(tc.tx * TILE) + 0.5f, y0 = (float)(tc.ty * TILE) + 0.5f;
    const uint32_t* hw32 = reinterpret_cast<const uint32_t*>(rp.hits);
    const uint16_t* hit16 = reinterpret_cast<const uint16_t*>(rp.hits);
    const uint64_t cap = rp.hit_cap;
    uint32_t n_hits = 0, n_batch = 0;   // work counters

    // the cursor: the record steps are taken from, its number in the tile, its
    // hits not yet taken, whether it is the first of its batch, its header (lanes 0..7; chunk k's
    // list position in lane 4 + k), the record before it and the headers of
    // the two before it (a header names both, so two loads are in flight and
    // a step does not wait for one)
    uint32_t cur = HIT_NONE, left = 0u, prev = HIT_NONE, first = 0u, chunks = 0u;
    uint32_t pend = 0u, pend2 = 0u, seq = 1u << 31;   // (past every record's number)
    int buf = 0;
    auto load_header = [&](uint32_t r) {
        return lane < 4 * (int)HIT_HEADER_UNITS && (uint64_t)r + HIT_HEADER_UNITS <= cap
                   ? hw32[(uint64_t)r * 4 + lane] : 0u;
    };
    auto enter = [&](uint32_t r, uint32_t header) {
        const uint32_t pv = (uint32_t)__builtin_amdgcn_readlane((int)header, 0);
        const uint32_t kept = (uint32_t)__builtin_amdgcn_readlane((int)header, 1);
        const uint32_t mark = (uint32_t)__builtin_amdgcn_readlane((int)header, 2);
        const uint32_t pv2 = (uint32_t)__builtin_amdgcn_readlane((int)header, 3);
        if (kept == 0u || (uint64_t)r + HIT_HEADER_UNITS + (kept + 7u) / 8u > cap ||
            mark >> 1 >= seq) {
            cur = HIT_NONE;
            return;
        }
        first = mark & 1u;
        seq = mark >> 1;
        chunks = header;
        cur = r;
        left = kept;
        prev = seq > 0u ? pv : HIT_NONE;
        pend = pend2;
        pend2 = load_header(pv2);   // (zeros for none: no hits, the walk ends)
    };
    auto next = [&]() {
        HitStep q{0, 0u, 0u, buf, false};
        if (cur != HIT_NONE && left == 0u) {
            if (prev == HIT_NONE) cur = HIT_NONE;
            else enter(prev, pend);
        }
        if (cur == HIT_NONE) return q;
        q.n = min(left, (uint32_t)(HB_HELPERS * WAVE));
        left -= q.n;
        q.base = ((uint64_t)cur + HIT_HEADER_UNITS) * 8 + left;
        // a batch's records share their chunks, so its sums stay in one
        // buffer until the first of them is done
        q.last = left == 0u && (first != 0u || prev == HIT_NONE);
        q.chunks = chunks;
        if (q.last) buf ^= 1;
        return q;
    };
    const uint32_t my = (uint32_t)(hw * WAVE + lane);   // my hit of a step, from its end
    auto load_hit = [&](const HitStep& q) {
        return my < q.n ? (uint32_t)hit16[q.base + q.n - 1u - my] : 0u;
    };
    // record id (HIT_NONE: no hit) and pair position of the hit's list entry
    struct Entry { uint32_t id, pos; };
    auto load_entry = [&](uint32_t hv, const HitStep& q) {
        const uint32_t chunk =
            (uint32_t)__shfl((int)q.chunks, 4 + (int)((hv >> 6) & (HB_CHUNKS - 1)), WAVE);   // all lanes take part
        const uint32_t pos = chunk * WAVE + (hv & 63u);
        Entry e{HIT_NONE, 0u};
        if (my < q.n && pos < kc) e = Entry{pvals[pos], rp.hit_ppos[pos]};
        return e;
    };
    auto gather = [&](uint32_t id) {
        return load_rec_pair(crec, (int64_t)id < stride ? id : rec0);
    };
    // the same for my chunk of a batch's list entries (lane = entry)
    auto load_chunk = [&](const HitStep& q) {
        const uint32_t chunk = (uint32_t)__builtin_amdgcn_readlane((int)q.chunks, 4 + hw);
        const uint32_t pos = chunk * WAVE + (uint32_t)lane;
        Entry e{HIT_NONE, 0u};
        if (q.n != 0u && pos < kc) e = Entry{pvals[pos], rp.hit_ppos[pos]};
        return e;
    };
    // footprint and attenuation of the hit; its part of the main wave's input
    auto evaluate = [&](uint32_t hv, const Entry& e, const CRec& R, const HitStep& q, int t) {
        HitTerm o;
        const bool valid = my < q.n;
        const int rr = (int)((hv >> HB_RAY_SHIFT) & (uint32_t)(WAVE - 1));
        float2 in = make_float2(0.0f, 0.0f);
        o.dx = x0 + (float)(rr & (TILE - 1)) - R.q.x;
        o.dy = y0 + (float)(rr / TILE) - R.q.y;
        o.a = R.q.z;
        o.b = R.q.w;
        o.c = R.w.x;
        o.id = e.id;
        o.pos = __float_as_uint(R.w.z) == 1u ? HIT_NONE : e.pos;
        o.slot = hv & (uint32_t)(HB_SLOTS - 1);
        o.dqx = o.f = 0.0f;
        if (valid && (int64_t)e.id < stride) {
            const float qf = quadform(R.q, R.w.x, o.dx, o.dy);
            if (qf < rp.q_max) {
                const float ex = __expf(-0.5f * qf);
                o.f = (ex - rp.eps) * rp.inv1meps;
                o.dqx = R.w.y * (-0.5f * ex * rp.inv1meps);
                o.slot |= 1u << 16;
                in.x = R.w.y * o.f;
                in.y = R.w.w;
            }
        }
        s_in[t & 1][hw][lane] = in;
        s_key[t & 1][hw][lane] = (signed char)(valid ? rr : -1);
        if (hw == 0 && lane == 0) s_n[t & 1] = q.n;
        n_hits += (uint32_t)__popcll(__ballot((o.slot >> 16) & 1u));
        return o;
    };
    // steps t - 1 .. t + 3 and what is loaded for them, relative to step t
    HitStep st[5];   // [0]: t - 1
    HitTerm term[3];
    uint32_t h[5];
    Entry en[4], chunk4;
    RecPair rec;
    st[0] = HitStep{0, 0u, 0u, 0, false};
    if ((uint64_t)tail + HIT_HEADER_UNITS <= cap) {
        const uint32_t header = load_header(tail);
        pend2 = load_header((uint32_t)__builtin_amdgcn_readlane((int)header, 0));
        enter(tail, header);
    }
#pragma unroll
    for (int i = 1; i < 5; ++i) {
        st[i] = next();
        h[i] = load_hit(st[i]);
    }
#pragma unroll
    for (int i = 1; i < 4; ++i) en[i] = load_entry(h[i], st[i]);
    {
        const RecPair r1 = gather(en[1].id);
        rec = gather(en[2].id);
        chunk4 = load_chunk(st[4]);
        term[1] = evaluate(h[1], en[1], own_rec(r1), st[1], 0);
    }
    bool fresh4 = true;   // step t + 3's entries are not in s_ent yet
    __syncthreads();
    for (int t = 0;; ++t) {
        // loads of later steps, waited for at the start of the next step
        const bool fresh_far = st[4].last;
        const HitStep far = next();
        const uint32_t h_far = load_hit(far);
        Entry chunk_far{HIT_NONE, 0u};
        if (fresh_far) chunk_far = load_chunk(far);
        const RecPair rec_far = gather(en[3].id);
        // the entries of step t + 3's batch, for the hits of its steps
        if (fresh4) s_ent[st[4].buf][hw * WAVE + lane] = make_uint2(chunk4.id, chunk4.pos);
        // the gradient terms of step t - 1
        if (t > 0 && ((term[0].slot >> 16) & 1u)) {
            const HitTerm& m = term[0];
            const int gb = st[0].buf, sl = (int)(m.slot & (uint32_t)(HB_SLOTS - 1));
            const float dxx = s_in[(t - 1) & 1][hw][lane].x;
            const float dq = dxx * m.dqx;
            s_rec[gb][sl] = m.id;
            s_pos[gb][sl] = m.pos;
            atomicAdd(&s_G[gb][0][sl], (double)(-2.0f * dq * (m.a * m.dx + m.b * m.dy)));
            atomicAdd(&s_G[gb][1][sl], (double)(-2.0f * dq * (m.b * m.dx + m.c * m.dy)));
            atomicAdd(&s_G[gb][2][sl], (double)(dq * m.dx * m.dx));
            atomicAdd(&s_G[gb][3][sl], (double)(2.0f * dq * m.dx * m.dy));
            atomicAdd(&s_G[gb][4][sl], (double)(dq * m.dy * m.dy));
            atomicAdd(&s_G[gb][5][sl], (double)(dxx * m.f));
        }
        if (hw == 0) {
            n_batch += st[0].last ? 1u : 0u;
            if (lane == 0) s_done[t & 1] = st[0].last ? (uint32_t)st[0].buf : 2u;
        }
        // step t + 1 for the main wave
        const bool more = st[1].n != 0u;
        if (more) term[2] = evaluate(h[2], en[2], own_rec(rec), st[2], t + 1);
        else if (t == 0) break;   // nothing at all
        __syncthreads();          // one per step, and one for the first empty step
        if (!more) break;
        __builtin_amdgcn_sched_barrier(0);   // the loads are waited for after the barrier
#pragma unroll
        for (int i = 0; i < 4; ++i) st[i] = st[i + 1];
        st[4] = far;
        term[0] = term[1];
        term[1] = term[2];
        h[2] = h[3];
        h[3] = h[4];
        h[4] = h_far;
        en[2] = en[3];
        {
            const uint2 e = s_ent[st[3].buf][h[3] & (uint32_t)(HB_SLOTS - 1)];
            en[3] = my < st[3].n ? Entry{e.x, e.y} : Entry{HIT_NONE, 0u};
        }
        chunk4 = chunk_far;
        fresh4 = fresh_far;
        rec = rec_far;
    }
    if (rp.work && lane == 0) {
        atomicAdd(&rp.work[1], (unsigned long long)n_hits);
        if (hw == 0) atomicMax(&rp.work[9], (unsigned long long)n_batch);
    }
}

// Non-empty computation-plane tiles, longest lists first (binned by the
// bit length of the list size), so the heaviest tiles start earliest. Three
// steps over global bins (bins[0..32] counts, bins[33..65] cursors): count
// per bin, turn the counts into starts (one workgroup; the tile count goes
// to status[ST_WORK_TILES]), place each tile at its bin's cursor. What
// bounds them is atomics on the few busy bins: one global atomic per tile
// had each step take 4.3 ns a tile (2.26 ms for the two on 262k tiles, 49 us
// each on 9k). A block takes WL_TILES tiles, counts them in LDS, with one LDS
// atomic per bin a wave's tiles fall in, and sends one atomic per bin.
constexpr int WL_PER = 4;
constexpr int WL_TILES = 256 * WL_PER;
constexpr int WL_BINS_N = 33;

__device__ __forceinline__ int list_bin(const uint2* __restrict__ ranges, int64_t t,
                                        int64_t tiles_c)
{
    if (t >= tiles_c) return 0;
    const uint2 rg = ranges[t];
    return rg.y > rg.x ? 32 - __clz(rg.y - rg.x) : 0;   // 0: nothing to do
}

// Adds the wave's tiles to the block's counts, one LDS atomic for the lanes
// of each bin (a loop over the bins among them waits for one atomic after
// the other: 21 us for 9216 tiles in one workgroup); returns the tile's place
// among the block's tiles of its bin.
__device__ __forceinline__ uint32_t bin_rank(uint32_t* s_cnt, int bin)
{
    uint64_t same = __ballot(bin != 0);
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        const uint64_t bit = __ballot((bin >> b) & 1);
        same &= ((bin >> b) & 1) ? bit : ~bit;
    }
    uint32_t first = 0u;
    if (bin != 0 && lanes_below(same) == 0u)
        first = atomicAdd(&s_cnt[bin], (uint32_t)__popcll(same));
    const int lead = same ? __builtin_ctzll(same) : 0;   // (no bin: any lane)
    return (uint32_t)__shfl((int)first, lead, WAVE) + lanes_below(same);
}

__global__ void __launch_bounds__(256)
k_worklist_count(const uint2* __restrict__ ranges, int64_t tiles_c, uint32_t* __restrict__ bins)
{
    __shared__ uint32_t s_cnt[WL_BINS_N];
    if (threadIdx.x < WL_BINS_N) s_cnt[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * WL_TILES + threadIdx.x;
    int bin[WL_PER];
#pragma unroll
    for (int k = 0; k < WL_PER; ++k) bin[k] = list_bin(ranges, t0 + k * 256, tiles_c);
#pragma unroll
    for (int k = 0; k < WL_PER; ++k) (void)bin_rank(s_cnt, bin[k]);
    __syncthreads();
    if (threadIdx.x < WL_BINS_N && s_cnt[threadIdx.x])
        atomicAdd(&bins[threadIdx.x], s_cnt[threadIdx.x]);
}

__global__ void k_worklist_starts(uint32_t* __restrict__ bins, uint32_t* __restrict__ status)
{
    if (threadIdx.x != 0) return;
    uint32_t acc = 0;
    for (int lvl = 32; lvl >= 1; --lvl) {
        bins[33 + lvl] = acc;
        acc += bins[lvl];
    }
    status[ST_WORK_TILES] = acc;
}

__global__ void __launch_bounds__(256)
k_worklist_place(const uint2* __restrict__ ranges, int64_t tiles_c, uint32_t* __restrict__ bins,
                 uint32_t* __restrict__ worklist)
{
    __shared__ uint32_t s_cnt[WL_BINS_N], s_base[WL_BINS_N];
    if (threadIdx.x < WL_BINS_N) s_cnt[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * WL_TILES + threadIdx.x;
    int bin[WL_PER];
    uint32_t rank[WL_PER];
#pragma unroll
    for (int k = 0; k < WL_PER; ++k) bin[k] = list_bin(ranges, t0 + k * 256, tiles_c);
#pragma unroll
    for (int k = 0; k < WL_PER; ++k) rank[k] = bin_rank(s_cnt, bin[k]);
    __syncthreads();
    if (threadIdx.x < WL_BINS_N)
        s_base[threadIdx.x] =
            s_cnt[threadIdx.x] ? atomicAdd(&bins[33 + threadIdx.x], s_cnt[threadIdx.x]) : 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < WL_PER; ++k)
        if (bin[k]) worklist[s_base[bin[k]] + rank[k]] = (uint32_t)(t0 + k * 256);
}

// The three steps in one workgroup, for at most WL_SMALL tiles (64 tiles in 3
// us, 9216 in 13, 16384 in 16; the three launches take 12, 18 and 18).
constexpr int WL_SMALL_THREADS = 1024;
constexpr int WL_SMALL_PER = 16;
constexpr int64_t WL_SMALL = WL_SMALL_THREADS * WL_SMALL_PER;

__global__ void __launch_bounds__(WL_SMALL_THREADS)
k_worklist_small(const uint2* __restrict__ ranges, int64_t tiles_c, uint32_t* __restrict__ bins,
                 uint32_t* __restrict__ status, uint32_t* __restrict__ worklist)
{
    __shared__ uint32_t s_cnt[WL_BINS_N], s_base[WL_BINS_N];
    if (threadIdx.x < WL_BINS_N) s_cnt[threadIdx.x] = 0u;
    __syncthreads();
    int bin[WL_SMALL_PER];
    uint32_t rank[WL_SMALL_PER];
#pragma unroll
    for (int k = 0; k < WL_SMALL_PER; ++k)
        bin[k] = list_bin(ranges, (int64_t)(k * WL_SMALL_THREADS) + threadIdx.x, tiles_c);
#pragma unroll
    for (int k = 0; k < WL_SMALL_PER; ++k)
        rank[k] = k * WL_SMALL_THREADS < tiles_c ? bin_rank(s_cnt, bin[k]) : 0u;
    __syncthreads();
    if (threadIdx.x < WAVE) {
        // bins in descending order of length: lane l holds bin 32 - l
        const int lane = threadIdx.x, b = 32 - lane;
        const uint32_t c = lane < 32 ? s_cnt[b] : 0u;
        uint32_t inc = c;
#pragma unroll
        for (int d = 1; d < 32; d <<= 1) {
            const uint32_t t = __shfl_up(inc, d, WAVE);
            if (lane >= d) inc += t;
        }
        if (lane < 32) {
            s_base[b] = inc - c;
            bins[b] = c;
            bins[33 + b] = inc;
        }
        if (lane == 31) status[ST_WORK_TILES] = inc;
        if (lane == 32) bins[0] = bins[33] = 0u;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < WL_SMALL_PER; ++k)
        if (bin[k])
            worklist[s_base[bin[k]] + rank[k]] = (uint32_t)(k * WL_SMALL_THREADS + threadIdx.x);
}

inline unsigned raster_grid(int64_t waves)
{
    return (unsigned)((waves + RASTER_WAVES - 1) / RASTER_WAVES);
}

inline unsigned grid256(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t launch_pair_masks(const DevView* views, int nv, int64_t cap_c, const RasterParams& rp,
                             bool tight,
                             const uint32_t* status, const uint32_t* pkey,
                             const uint32_t* pvals, const CRec* crec,
                             uint64_t* pmask, uint64_t* psum, hipStream_t s)
{
    if (cap_c <= 0) return hipSuccess;
    const unsigned grid = (unsigned)((cap_c + 256 * PM_ITEMS - 1) / (256 * PM_ITEMS));
    if (tight)
        hipLaunchKernelGGL(k_pair_masks<true>, dim3(grid), dim3(256), 0, s, views, nv, cap_c, rp,
                           status, pkey, pvals, crec, pmask, psum);
    else
        hipLaunchKernelGGL(k_pair_masks<false>, dim3(grid), dim3(256), 0, s, views, nv, cap_c, rp,
                           status, pkey, pvals, crec, pmask, psum);
    return hipGetLastError();
}

hipError_t launch_tile_worklist(const uint2* ranges, int64_t tiles_c, uint32_t* worklist,
                                uint32_t* bins, uint32_t* status, hipStream_t s)
{
    if (tiles_c <= WL_SMALL) {
        hipLaunchKernelGGL(k_worklist_small, dim3(1), dim3(WL_SMALL_THREADS), 0, s, ranges,
                           tiles_c, bins, status, worklist);
        return hipGetLastError();
    }
    const unsigned wl_grid = (unsigned)((tiles_c + WL_TILES - 1) / WL_TILES);
    if (tiles_c > 0)
        hipLaunchKernelGGL(k_worklist_count, dim3(wl_grid), dim3(256), 0, s, ranges, tiles_c,
                           bins);
    hipLaunchKernelGGL(k_worklist_starts, dim3(1), dim3(64), 0, s, bins, status);
    if (tiles_c > 0)
        hipLaunchKernelGGL(k_worklist_place, dim3(wl_grid), dim3(256), 0, s, ranges, tiles_c,
                           bins, worklist);
    return hipGetLastError();
}

hipError_t launch_raster_a_fwd(const DevView* views, int nv, int64_t tiles_c,
                               const RasterParams& rp, const uint32_t* status,
                               const uint32_t* worklist, const uint2* ranges,
                               const uint32_t* pvals, const uint64_t* pmask,
                               const uint64_t* psum, const CRec* crec,
                               float* A, float* tau, uint32_t* nlast, hipStream_t s)
{
    if (tiles_c <= 0) return hipSuccess;
    auto run = [&](auto det, auto hits) {
        hipLaunchKernelGGL((k_raster_a_fwd<decltype(det)::value, decltype(hits)::value>),
                           dim3((unsigned)tiles_c), dim3(WAVE), 0, s, views, nv, rp, status,
                           worklist, ranges, pvals, pmask, psum, crec, A, tau, nlast);
    };
    if (rp.ppos) {
        run(std::true_type{}, std::false_type{});
    } else if (rp.hits) {
        // (the number of tiles with lists is known on the device only)
        hipLaunchKernelGGL(k_raster_a_fwd_hits,
                           dim3((unsigned)std::min<int64_t>(tiles_c, HF_TILES)),
                           dim3(HF_THREADS), 0, s, views, nv, rp, status, worklist, ranges, pvals,
                           pmask, psum, crec, A, tau, nlast);
        if (tiles_c > (int64_t)HF_TILES) run(std::false_type{}, std::true_type{});
    } else {
        run(std::false_type{}, std::false_type{});
    }
    return hipGetLastError();
}

hipError_t launch_raster_b_fwd(const DevView* views, int nv, int64_t pixels, int64_t cap_c,
                               int64_t cap_i, const RasterParams& rp, const uint32_t* status,
                               const uint32_t* pkey, const uint32_t* pvals, const float4* iq,
                               const float2* iw, float* images, bool zeroed, bool vm,
                               hipStream_t s)
{
    if (pixels <= 0) return hipSuccess;
    if (!zeroed)
        hipLaunchKernelGGL(k_zero_images, dim3(grid256(pixels)), dim3(256), 0, s, views, nv,
                           pixels, images);
    if (cap_i <= 0) return hipGetLastError();
    const int64_t segs = (cap_i + B_SEGMENT - 1) / B_SEGMENT;
    hipLaunchKernelGGL(k_raster_b_fwd, dim3(raster_grid(segs)), dim3(RASTER_THREADS), 0, s, views,
                       nv, rp, cap_c, status, pkey, pvals, iq, iw, images, vm ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_raster_b_direct(const DevView* views, int nv, int64_t tiles_c, int64_t tiles_i,
                                  int64_t records, int64_t cap_i, const RasterParams& rp,
                                  const uint32_t* bsum, uint32_t* status, const uint2* rect,
                                  const float4* iq, const float2* iw, float* images,
                                  hipStream_t s)
{
    if (tiles_i <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_raster_b_direct, dim3((unsigned)tiles_i), dim3(BT_WAVES * WAVE), 0, s,
                       views, nv, rp, tiles_c, cap_i, bsum, (records + 255) / 256, status, rect,
                       iq, iw, images);
    return hipGetLastError();
}

hipError_t launch_raster_b_tiles(const DevView* views, int nv, int64_t pixels, int64_t cap_c,
                                 int64_t cap_i, int64_t tiles_c, int64_t tiles_i,
                                 const RasterParams& rp, const uint32_t* status,
                                 const uint32_t* pkey, const uint32_t* pvals, const float4* iq,
                                 const float2* iw, uint2* ranges_i, float* images, bool zeroed,
                                 bool vm, hipStream_t s)
{
    if (pixels <= 0) return hipSuccess;
    if (!zeroed)
        hipLaunchKernelGGL(k_zero_images, dim3(grid256(pixels)), dim3(256), 0, s, views, nv,
                           pixels, images);
    if (cap_i <= 0 || tiles_i <= 0) return hipGetLastError();
    hipError_t e = launch_ranges_i(views, pkey + cap_c, status, cap_i, tiles_c, tiles_i, vm,
                                   ranges_i, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_raster_b_tile, dim3((unsigned)tiles_i), dim3(BT_WAVES * WAVE), 0, s,
                       views, nv, rp, cap_c, tiles_c, ranges_i, pvals, iq, iw, images);
    return hipGetLastError();
}

hipError_t launch_image_bwd(const DevView* views, const DevScene* scenes, int nv,
                            int64_t records, const RasterParams& rp, const uint32_t* status,
                            const uint32_t* active, const float4* iq, const float2* iw,
                            const float* prec, const float* dimg, float* grad_i, CRec* crec,
                            float* grad_c, hipStream_t s)
{
    if (records <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_image_bwd, dim3(grid256(records)), dim3(256), 0, s, views, scenes, nv,
                       records, rp, status, active, iq, iw, prec, dimg, grad_i, crec, grad_c);
    return hipGetLastError();
}

hipError_t launch_raster_a_bwd_hits(const DevView* views, int nv, int64_t tiles_c,
                                    const RasterParams& rp, const uint32_t* status,
                                    const uint32_t* worklist, const uint32_t* pvals,
                                    const CRec* crec, const float* tau, float* grad_c,
                                    int64_t stride, hipStream_t s)
{
    if (tiles_c <= 0 || !rp.hits || rp.ppos) return hipSuccess;
    hipLaunchKernelGGL(k_raster_a_bwd_hits, dim3((unsigned)tiles_c), dim3(HB_THREADS), 0, s, views,
                       nv, rp, status, worklist, pvals, crec, tau, grad_c, stride);
    return hipGetLastError();
}

hipError_t launch_raster_a_bwd(const DevView* views, int nv, int64_t tiles_c,
                               const RasterParams& rp, const uint32_t* status,
                               const uint32_t* worklist, const uint2* ranges,
                               const uint32_t* pvals, const uint64_t* pmask,
                               const uint64_t* psum, const CRec* crec,
                               const float* tau, const uint32_t* nlast, float* grad_c,
                               int64_t stride, hipStream_t s)
{
    if (tiles_c <= 0) return hipSuccess;
    // long lists (the front of the worklist), then the short ones
    auto two = [&](auto det) {
        constexpr bool D = decltype(det)::value;
        const int64_t per = !D && rp.hits ? BWD_TILES : 1;
        const unsigned grid = (unsigned)((tiles_c + per - 1) / per);
        hipLaunchKernelGGL((k_raster_a_bwd<true, D>), dim3(grid), dim3(2 * WAVE), 0, s, views, nv,
                           rp, status, worklist, ranges, pvals, pmask, psum, crec, tau, nlast,
                           grad_c, stride);
        hipLaunchKernelGGL((k_raster_a_bwd<false, D>), dim3(grid), dim3(WAVE), 0, s, views, nv,
                           rp, status, worklist, ranges, pvals, pmask, psum, crec, tau, nlast,
                           grad_c, stride);
    };
    if (rp.ppos)
        two(std::true_type{});
    else
        two(std::false_type{});
    return hipGetLastError();
}

}  // namespace sdgr
