// Device code shared by the kernels that select the outlier channels for themselves: every
// workgroup folds the column maxima, selects (Sec. III-C) and derives the scale (Eq. 1 on Body), a
// thread per chunk of 8 channels, instead of reading the results of a selection kernel.
#pragma once
#include "muxq_kernels.h"

namespace muxq {
namespace {

// The largest magnitude among the channels of `raw` (8 fp16) that `listed` does not name, in the
// low half, and among those it names, in the high half (fp16 magnitudes order like integers).
__device__ __forceinline__ uint32_t chunk_maxima(uint4 raw, uint32_t listed)
{
    uint32_t d[4] = {raw.x & 0x7fff7fffu, raw.y & 0x7fff7fffu, raw.z & 0x7fff7fffu, raw.w & 0x7fff7fffu};
    uint32_t l = 0;
    if (__ballot(listed != 0) != 0) {                    // (most waves have no listed channel)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t two = listed >> (2 * i);
            const uint32_t out = (two & 1u) * 0xffffu | (two >> 1 & 1u) * 0xffff0000u;
            l = pk_max_u16(l, d[i] & out);
            d[i] &= ~out;
        }
        l = max(l & 0xffffu, l >> 16);
    }
    const uint32_t m = pk_max_u16(pk_max_u16(d[0], d[1]), pk_max_u16(d[2], d[3]));
    return max(m & 0xffffu, m >> 16) | (l << 16);
}

__device__ __forceinline__ float f32_of_half_bits(uint32_t h)
{
    return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
}

// Scale, multiplier and zero point (Eq. 1; the zero point of the unlisted channels' codes is even,
// see the selection kernel) from the two maxima of chunk_maxima over a row, or over the call.
__device__ __forceinline__ void call_scale(uint32_t maxima, float shrink, float qmax, float &sx, float &inv, int &z)
{
    const float nm = fmaxf(0.f, f32_of_half_bits(maxima & 0xffffu)), lm = fmaxf(0.f, f32_of_half_bits(maxima >> 16));
    const float am = fmaxf(nm, lm * shrink);             // exact: max |Body| (Eq. 4)
    sx = am > 0.f ? am / qmax : 0.f;                     // correctly rounded binary32 divisions
    inv = am > 0.f ? qmax / am : 0.f;
    const int c = (int)fminf(__builtin_rintf(nm * inv), qmax);
    z = min(c + (c & 1), (127 - c) & ~1);
}

// Maximum (two packed uint16) over the wave, in lane 63; sum of the lanes up to and including this
// one.  (Cross-lane moves of the vector ALU: a permute through LDS is ten times their latency.)
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t dpp_zero(uint32_t v)     // lanes without a source get 0
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_max_u16x2_to_lane63(uint32_t v)
{
    v = pk_max_u16(v, dpp_zero<0x111>(v));                   // row_shr 1, 2, 4, 8: lane 15 of a row of 16
    v = pk_max_u16(v, dpp_zero<0x112>(v));
    v = pk_max_u16(v, dpp_zero<0x114>(v));
    v = pk_max_u16(v, dpp_zero<0x118>(v));
    v = pk_max_u16(v, dpp_zero<0x142, 0xa>(v));              // lane 15 of a row to the next one
    return pk_max_u16(v, dpp_zero<0x143, 0xc>(v));           // lane 31 to the upper half
}
// ... over each LANES (16 or 64) neighbouring lanes, in all of them.
template <int LANES>
__device__ __forceinline__ uint32_t lanes_max_u16x2(uint32_t v)
{
    if (LANES == 64) return (uint32_t)__builtin_amdgcn_readlane((int)wave_max_u16x2_to_lane63(v), 63);
    v = pk_max_u16(v, dpp_zero<0x121>(v));                   // rotations of a row of 16 by 1, 2, 4, 8
    v = pk_max_u16(v, dpp_zero<0x122>(v));
    v = pk_max_u16(v, dpp_zero<0x124>(v));
    return pk_max_u16(v, dpp_zero<0x128>(v));
}
__device__ __forceinline__ int wave_inclusive_sum(int x)
{
    uint32_t v = (uint32_t)x;
    v += dpp_zero<0x111>(v);
    v += dpp_zero<0x112>(v);
    v += dpp_zero<0x114>(v);
    v += dpp_zero<0x118>(v);
    v += dpp_zero<0x142, 0xa>(v);
    return (int)(v + dpp_zero<0x143, 0xc>(v));
}

// Eight fp16 values, or their magnitudes, with those that are NaN (magnitudes above infinity's) zeroed: a
// NaN in X must not hide the other channels from the scale of the call, or of its row.
__device__ __forceinline__ uint4 drop_nan(uint4 mx)
{
    uint32_t d[4] = {mx.x, mx.y, mx.z, mx.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if ((d[i] & 0x7fffu) > 0x7c00u) d[i] &= 0xffff0000u;
        if ((d[i] >> 16 & 0x7fffu) > 0x7c00u) d[i] &= 0xffffu;
    }
    return make_uint4(d[0], d[1], d[2], d[3]);
}

// chunk_maxima over the chunks that the lanes of a wave hold of a row, in lane 63, without NaNs.  (Every lane of the wave
// calls.)  A NaN wins the integer comparison, so it shows in the result, and only then the maxima are taken again without it.
__device__ __forceinline__ uint32_t wave_row_maxima(uint4 raw, uint32_t listed)
{
    const uint32_t m = wave_max_u16x2_to_lane63(chunk_maxima(raw, listed));
    const uint32_t top = (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
    if ((top & 0xffffu) <= 0x7c00u && (top >> 16) <= 0x7c00u) return m;
    return wave_max_u16x2_to_lane63(chunk_maxima(drop_nan(raw), listed));
}

// Whether a lane of the wave has a NaN among its magnitudes.
__device__ __forceinline__ bool wave_has_nan(uint4 mx)
{
    const muxq_u16x2 inf = {0x7c00, 0x7c00};
    const uint32_t d[4] = {mx.x, mx.y, mx.z, mx.w};
    uint32_t over = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        over |= __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(muxq_u16x2, d[i]), inf));
    return __ballot(over != 0) != 0;
}

// What select_channels returns: for this thread's chunk (in the waves that hold chunks), and for the call.
struct Selected {
    uint32_t listed;     // bit i: channel i of the chunk is listed
    int first;           // rank of the chunk's first candidate
    int used, found;     // listed channels, candidates
    uint32_t maxima;     // chunk_maxima over all channels (want_max)
};

// The channels of a chunk whose column maxima are over the threshold, one bit each.  `cut` is the
// threshold as the bits of the largest fp16 magnitude that is not over it (magnitude_cut), so that
// two channels are compared in one instruction; a NaN is never over it.  (All lanes of a wave call.)
__device__ __forceinline__ uint32_t chunk_candidates(uint4 mx, float threshold, int cut)
{
    if (cut < 0 || wave_has_nan(mx)) {                   // (a negative threshold: every number is over it)
        float v[8];
        widen8(mx, v);
        uint32_t cand = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) cand |= (v[i] > threshold ? 1u : 0u) << i;
        return cand;
    }
    const muxq_u16x2 cut2 = {(unsigned short)cut, (unsigned short)cut}, one = {1, 1};
    const uint32_t d[4] = {mx.x, mx.y, mx.z, mx.w};
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const muxq_u16x2 over = __builtin_elementwise_sub_sat(__builtin_bit_cast(muxq_u16x2, d[i]), cut2);
        m |= __builtin_bit_cast(uint32_t, __builtin_elementwise_min(over, one)) << (2 * i);
    }
    return (m | m >> 15) & 0xffu;
}
// (On the host, in every call with a threshold: the conversion to fp16, rounded towards zero.  A search over the values took 0.11 us.)
inline int magnitude_cut(float threshold)
{
    if (!(threshold >= 0.f)) return -1;
    if (threshold > 65504.f) return threshold == __builtin_inff() ? 0x7c00 : 0x7bff;
    if (threshold < 0x1p-14f) return (int)(threshold * 0x1p24f);         // subnormal: in units of 2^-24 (and -0)
    return (int)(__builtin_bit_cast(uint32_t, threshold) >> 13) - ((127 - 15) << 10);
}

// Sec. III-C with the capacity rule: the r_cap lowest candidates are listed.  The first `n_seg` pieces
// of 64 chunks are in one wave each; a thread of those (`holds`, the same in a wave) brings the column maxima `mx`
// (magnitudes) of chunk 64 seg + lane and its candidates.  All waves of the workgroup call, 16 at most; one
// barrier, two more where the list overflows: the caller's LDS writes before are visible after, what it read before may be overwritten
// after, and s_tot and s_max (16 entries each) not before another barrier.
// A chain of latencies that every workgroup walks: 16 waves that all work out everything are bound by
// their instructions (four waves on a SIMD), so only the waves that hold chunks do, and what all need of the waves' results
// is read by 16 lanes side by side (8192 x 1024, from the column maxima to the list 1.5 -> 0.9 us).
__device__ __forceinline__ Selected select_channels(uint4 mx, uint32_t cand, bool holds, int seg, int n_seg, int r_cap,
                                                    bool want_max, int *s_tot, uint32_t *s_max)
{
    const int lane = threadIdx.x & 63;
    Selected r;
    r.listed = cand;
    int incl = 0;
    if (holds) {
        incl = wave_inclusive_sum(__builtin_popcount(cand));
        uint32_t top = 0;
        if (want_max) {
            if (wave_has_nan(mx)) mx = drop_nan(mx);
            top = wave_max_u16x2_to_lane63(chunk_maxima(mx, cand));
        }
        if (lane == 63) {
            s_tot[seg] = incl;
            s_max[seg] = top;
        }
    }
    lds_barrier();
    const bool in = (lane & 15) < n_seg;
    uint32_t tot = in ? (uint32_t)s_tot[lane & 15] : 0u, m = in ? s_max[lane & 15] : 0u;
    tot += dpp_zero<0x111>(tot);                         // row_shr 1, 2, 4, 8: sums over a row of 16 lanes
    tot += dpp_zero<0x112>(tot);
    tot += dpp_zero<0x114>(tot);
    tot += dpp_zero<0x118>(tot);
    if (want_max) {
        m = pk_max_u16(m, dpp_zero<0x111>(m));
        m = pk_max_u16(m, dpp_zero<0x112>(m));
        m = pk_max_u16(m, dpp_zero<0x114>(m));
        m = pk_max_u16(m, dpp_zero<0x118>(m));
    }
    r.found = __builtin_amdgcn_readlane((int)tot, 15);
    r.maxima = (uint32_t)__builtin_amdgcn_readlane((int)m, 15);
    r.first = incl - __builtin_popcount(cand) + (seg > 0 ? __builtin_amdgcn_readlane((int)tot, max(seg, 1) - 1) : 0);
    r.used = min(r.found, r_cap);
    if (r.found > r_cap) {
        if (holds) {
            uint32_t kept = 0;
            int rank = r.first;
            for (uint32_t mm = cand; mm != 0; mm &= mm - 1, ++rank)
                if (rank < r_cap) kept |= mm & (0u - mm);
            r.listed = kept;
        }
        if (want_max) {
            const uint32_t top = holds ? wave_max_u16x2_to_lane63(chunk_maxima(mx, r.listed)) : 0u;
            lds_barrier();                               // s_max is consumed
            if (holds && lane == 63) s_max[seg] = top;
            lds_barrier();
            r.maxima = 0;
            for (int i = 0; i < n_seg; ++i) r.maxima = pk_max_u16(r.maxima, s_max[i]);
        }
    }
    return r;
}

// The selection results of the call as the workspace keeps them: col_absmax, col_slot, col_mask and, with one scale per
// call, col_scale; the list, its padding and counts.  Every workgroup has them, and each stores the chunks of few
// waves (store_share): all by one workgroup, that one ended 0.5 to 1.5 us after the others.  Called by the waves that hold
// chunks, `c` being the thread's; the padding and counts go out from the first workgroup.
__device__ __forceinline__ bool store_share(int seg) { return seg % (int)gridDim.x == (int)blockIdx.x; }
__device__ __forceinline__ void store_selection(const Selected &r, uint4 mx, int c, int C, int CA, int r_cap,
                                                bool with_scale, float inv, float shrink, float *col_absmax,
                                                float *col_scale, int32_t *col_slot, uint8_t *col_mask, int32_t *idx)
{
    if (c < CA) {
        int slots[8];
        int rank = r.first;
        float v[8];
        widen8(mx, v);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const bool l = ((r.listed >> i) & 1u) != 0;
            slots[i] = l ? rank : -1;
            if (l) idx[rank] = c * 8 + i;
            rank += l ? 1 : 0;
        }
        int4 *cs = (int4 *)(col_slot + c * 8);
        cs[0] = make_int4(slots[0], slots[1], slots[2], slots[3]);
        cs[1] = make_int4(slots[4], slots[5], slots[6], slots[7]);
        col_mask[c] = (uint8_t)r.listed;
        if (c < C) {
            float4 *cm = (float4 *)(col_absmax + c * 8);
            cm[0] = make_float4(v[0], v[1], v[2], v[3]);
            cm[1] = make_float4(v[4], v[5], v[6], v[7]);
        }
        if (with_scale) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = c < C ? inv * (slots[i] >= 0 ? shrink : 1.0f) : 0.f;
            float4 *sc = (float4 *)(col_scale + c * 8);
            sc[0] = make_float4(v[0], v[1], v[2], v[3]);
            sc[1] = make_float4(v[4], v[5], v[6], v[7]);
        }
    }
}
__device__ __forceinline__ void store_list_rest(const Selected &r, int r_cap, int32_t *idx, int32_t *n_outliers)
{
    for (int j = r.used + (int)threadIdx.x; j < max(r_cap, 1); j += (int)blockDim.x) idx[j] = -1;
    if (threadIdx.x == 0) {
        n_outliers[0] = r.used;
        n_outliers[1] = r.found;
    }
}

}  // namespace
}  // namespace muxq
