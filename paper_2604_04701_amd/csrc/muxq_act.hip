// The activation side with the selection inside the quantisers.
//
// The selection (Sec. III-C: which channels are outlier channels; Eq. 1: the scale taken on Body)
// needs the column maxima of all of X and very little work, and as a kernel of its own it cost 6-8 us
// between two streaming kernels: one workgroup reading up to 320 KB of slab maxima at what one CU
// can fetch (~100 GB/s), and the launch.  Here the abs-max pass leaves few slabs (narrow blocks of
// columns, 64 KB in all), and every workgroup of the quantiser folds them and selects for itself,
// while its first rows of X are on their way.  With few tokens the abs-max pass goes as well: the
// workgroups fold X itself (`slabs` are its rows).  The results go into the workspace in shares of the workgroups.
//
// Bound by memory: X twice (the second time mostly out of the memory-side cache), the codes once.
#include "muxq_select.h"

namespace muxq {
namespace {

constexpr int kActThreads = 1024, kActWaves = kActThreads / 64;
constexpr int kActMaxK = 8 * kActThreads;              // one chunk of 8 channels per thread in the selection
constexpr int kActMaxCap = 1024;

// Column maxima of |X| per row slab, like k_col_absmax_partial, but a workgroup covers only 128
// columns and many rows: the same number of workgroups leaves a quarter of the slabs.  (64 columns leave
// an eighth, but 16384 x 5120 from HBM then takes 5 us more; 256 columns, 64-128 KB to fold, cost the
// quantisers 1-2 us.)
constexpr int kNarrowLanes = 16;
__global__ __launch_bounds__(512) void k_col_absmax_narrow(const uint16_t *__restrict__ x, int rows, int cols, int ld,
                                                           int k_pad, int rows_per_block,
                                                           uint16_t *__restrict__ partial)
{
    constexpr int LANES = kNarrowLanes, RW = 64 / LANES, RB = 8 * RW;    // rows of a wave's load, of a workgroup's
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col0 = blockIdx.x * LANES * 8 + (lane % LANES) * 8;
    const int r0 = blockIdx.y * rows_per_block, r1 = min(rows, r0 + rows_per_block);
    uint4 mx = make_uint4(0, 0, 0, 0);
    if (col0 < cols) {
        const uint16_t *p = x + col0;
        int row = r0 + wave * RW + lane / LANES;
        for (; row + 3 * RB < r1; row += 4 * RB) {
            const uint4 v0 = *(const uint4 *)(p + (size_t)row * ld);
            const uint4 v1 = *(const uint4 *)(p + (size_t)(row + RB) * ld);
            const uint4 v2 = *(const uint4 *)(p + (size_t)(row + 2 * RB) * ld);
            const uint4 v3 = *(const uint4 *)(p + (size_t)(row + 3 * RB) * ld);
            mx = absmax_step(absmax_step(absmax_step(absmax_step(mx, v0), v1), v2), v3);
        }
        for (; row < r1; row += RB) mx = absmax_step(mx, *(const uint4 *)(p + (size_t)row * ld));
    }
    __shared__ uint4 red[512];
    red[threadIdx.x] = mx;
    lds_barrier();
    if (wave != 0) return;
    for (int w = 1; w < 8; ++w) mx = absmax_step(mx, red[w * 64 + lane]);
#pragma unroll
    for (int off = LANES; off < 64; off <<= 1)
        mx = absmax_step(mx, make_uint4(__shfl_xor((int)mx.x, off), __shfl_xor((int)mx.y, off),
                                        __shfl_xor((int)mx.z, off), __shfl_xor((int)mx.w, off)));
    if (lane < LANES && col0 < k_pad) *(uint4 *)(partial + (size_t)blockIdx.y * k_pad + col0) = mx;  // zeros in the K padding
}

// Many slabs (a producer's) -> one, in slab 0: 64 chunks per workgroup, four threads to a chunk, which
// reads and writes nothing but its own columns.
__global__ __launch_bounds__(256) void k_fold_slabs(uint16_t *partial, int n_slabs, int k_pad)
{
    __shared__ uint4 part[256];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63), g = threadIdx.x >> 6;
    uint4 mx = make_uint4(0, 0, 0, 0);
    if (c < k_pad / 8)
        for (int s0 = g; s0 < n_slabs; s0 += 32) {
            uint4 q[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)              // (past the end the last slab again)
                q[j] = *(const uint4 *)(partial + (size_t)min(s0 + 4 * j, n_slabs - 1) * k_pad + c * 8);
#pragma unroll
            for (int j = 0; j < 8; ++j) mx = absmax_step(mx, q[j]);
        }
    part[threadIdx.x] = mx;
    lds_barrier();                                   // (every read of the slabs is back: its value is in LDS)
    if (g != 0 || c >= k_pad / 8) return;
    for (int j = 1; j < 4; ++j) mx = absmax_step(mx, part[j * 64 + threadIdx.x]);
    *(uint4 *)(partial + c * 8) = mx;
}

struct ActShared {
    uint4 part[kActThreads];
    uint16_t slot[kActMaxK];             // list position of each listed channel
    int idx[kActMaxCap];                 // the list
    uint8_t mask[kActThreads];           // per chunk of 8 channels: which are listed
    int tot[kActWaves];
    uint32_t max[kActWaves];
    float amax;                          // given list only
    float sx, inv;                       // one scale per call
    int z;
};

// This thread's part of the fold, of N slabs p, p + P, ... at most.  The loads of N slabs are all
// requested at once, and the workgroup's first rows of X behind them (load_x): loads come back in the order they
// were issued, and the fold would wait for X as well.  (Past the end the last slab again: a branch per load would
// serialise the loads.  N fits the slabs there are, because what 16 waves read twice counts: always eight of them, 0.2-0.4 us; a form for five as
// well, 0.0 us.)
template <int N, typename LoadX>
__device__ __forceinline__ uint4 fold_slabs(const ActArgs &a, int c, int p, int P, bool on, LoadX &&load_x)
{
    const uint16_t *const src = a.slabs + (size_t)c * 8;
    uint4 q[N], mx = make_uint4(0, 0, 0, 0);
    if (on)
#pragma unroll
        for (int j = 0; j < N; ++j) q[j] = *(const uint4 *)(src + (size_t)min(p + j * P, a.n_slabs - 1) * a.slab_ld);
    __builtin_amdgcn_sched_barrier(0);
    load_x();
    __builtin_amdgcn_sched_barrier(0);
    if (on)
#pragma unroll
        for (int j = 0; j < N; ++j) mx = absmax_step(mx, q[j]);
    return mx;
}

// Fold, selection and list for the whole workgroup.  WANT_MAX: false where neither the candidates (a
// list fixed offline) nor the scale (one per token) need the column maxima.
// load_x (WANT_MAX): requests the workgroup's first rows of X.
// WANT_SCALE: the scale of the call is left in `sh`.
template <bool WANT_MAX, bool WANT_SCALE, typename LoadX>
__device__ __forceinline__ Selected act_select(const ActArgs &a, ActShared &sh, float shrink, uint4 &mx, LoadX &&load_x)
{
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), C = a.K / 8, CA = a.k_pad / 8;
    const int n_seg = (CA + 63) / 64;                    // waves that hold chunks in the selection
    const bool holds = wave < n_seg;
    mx = make_uint4(0, 0, 0, 0);
    if (WANT_MAX) {
        const int P = quotient(a.wg_waves * 64, a.by_chunks), p = quotient(tid, a.by_chunks), c = tid - p * CA;
        const bool on = p < P && c < C && p < a.n_slabs;
        if (a.n_slabs <= P) {
            mx = fold_slabs<1>(a, c, p, P, on, load_x);
        } else if (a.n_slabs <= 2 * P) {
            mx = fold_slabs<2>(a, c, p, P, on, load_x);
        } else if (a.n_slabs <= 4 * P) {
            mx = fold_slabs<4>(a, c, p, P, on, load_x);
        } else {
            mx = fold_slabs<8>(a, c, p, P, on, load_x);
            for (int sl = p + 8 * P; on && sl < a.n_slabs; sl += 8 * P) {
                uint4 q[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    q[j] = *(const uint4 *)(a.slabs + (size_t)c * 8 + (size_t)min(sl + j * P, a.n_slabs - 1) * a.slab_ld);
#pragma unroll
                for (int j = 0; j < 8; ++j) mx = absmax_step(mx, q[j]);
            }
        }
        if (P > 1) {
            sh.part[tid] = mx;
            lds_barrier();
            if (holds) {
                const int G = min(P, a.n_slabs), at = min(tid, CA - 1);
                mx = make_uint4(0, 0, 0, 0);
                for (int g = 0; g < G; g += 4) {         // (past the end the last part again)
                    uint4 q[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) q[j] = sh.part[min(g + j, G - 1) * CA + at];
#pragma unroll
                    for (int j = 0; j < 4; ++j) mx = absmax_step(mx, q[j]);
                }
                if (tid >= CA) mx = make_uint4(0, 0, 0, 0);
            }
        }
    }
    uint32_t cand = 0;
    if (holds) {
        if (a.static_mask != nullptr)
            cand = tid < C ? a.static_mask[tid] : 0u;
        else if (WANT_MAX) {
            cand = chunk_candidates(mx, a.threshold, a.cut);
            if (tid >= C) cand = 0;
        }
    }
    const Selected r = select_channels(mx, cand, holds, wave, n_seg, a.r_cap, WANT_SCALE, sh.tot, sh.max);
    if (holds) {
        if (tid < CA) sh.mask[tid] = (uint8_t)r.listed;
        int rank = r.first;
        for (uint32_t mm = r.listed; mm != 0; mm &= mm - 1, ++rank) {
            const int k = tid * 8 + __builtin_ctz(mm);
            sh.slot[k] = (uint16_t)rank;
            sh.idx[rank] = k;
        }
    }
    if (WANT_SCALE && wave == a.wg_waves - 1) {           // (as a rule a wave without chunks)
        float sx, inv;
        int z;
        call_scale(r.maxima, shrink, a.qmax, sx, inv, z);
        if ((tid & 63) == 0) {
            sh.sx = sx;
            sh.inv = inv;
            sh.z = z;
        }
    }
    lds_barrier();
    return r;
}

// Eq. 7: the weight rows that meet Aux, w_aux[n][j] = w_q[n][idx[j]], and cn[n], the sum of channel n's
// other weight codes (+ cn_bias): 16 lanes per output channel, 64 channels per step of a workgroup of 16 waves.  The
// bytes of the first step are requested before the rows of X are worked on and written after it.
struct ActGather {
    int v[4], row_sum;
};
__device__ __forceinline__ ActGather gather_request(const ActArgs &a, const ActShared &sh, int n, int used)
{
    ActGather g;
    g.row_sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) g.v[i] = 0;
    if (a.cn == nullptr || n >= a.N) return g;
    g.row_sum = a.w_row_sum[n];
    const int sub = threadIdx.x & 15;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (sub + 16 * i < used) g.v[i] = a.w_q[packed_index(n, sh.idx[sub + 16 * i], a.k_pad)];
    return g;
}
__device__ __forceinline__ void gather_finish(const ActArgs &a, const ActShared &sh, int n, int used, const ActGather &g)
{
    if (a.cn == nullptr) return;
    const int sub = threadIdx.x & 15;
    int sum = 0;
    if (n < a.N) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = sub + 16 * i;
            if (a.w_aux != nullptr && j < a.r_cap) a.w_aux[packed_index(n, j, a.r_cap)] = (int8_t)g.v[i];
            sum += g.v[i];
        }
        for (int j = sub + 64; j < a.r_cap; j += 16) {           // lists beyond 64 entries
            const int v = j < used ? a.w_q[packed_index(n, sh.idx[j], a.k_pad)] : 0;
            if (a.w_aux != nullptr) a.w_aux[packed_index(n, j, a.r_cap)] = (int8_t)v;
            sum += v;
        }
    }
    for (int off = 8; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if (sub == 0 && n < a.N) a.cn[n] = g.row_sum - sum + a.cn_bias;
}
__device__ __forceinline__ void gather_rest(const ActArgs &a, const ActShared &sh, int used, const ActGather &first)
{
    const int per = a.wg_waves * 4, n0 = (int)blockIdx.x * per + ((int)threadIdx.x >> 4);       // channels per workgroup and step
    gather_finish(a, sh, n0, used, first);
    if (a.cn == nullptr) return;
    for (int nb = ((int)blockIdx.x + (int)gridDim.x) * per; nb < a.N; nb += (int)gridDim.x * per) {    // (N in the ten thousands)
        const int n = nb + ((int)threadIdx.x >> 4);
        gather_finish(a, sh, n, used, gather_request(a, sh, n, used));
    }
}

// 8 codes, stored at agent scope: written through, where a usual store leaves them dirty in L2 until the kernel ends.
__device__ __forceinline__ void store_through(int8_t *dst, uint2 codes)
{
    __hip_atomic_store((unsigned long long *)dst, __builtin_bit_cast(unsigned long long, codes), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Aux columns past the list, zeroed for an equal share of the rows: four codes to a store.
__device__ __forceinline__ void zero_aux_rest(const ActArgs &a, int used)
{
    const int per = (a.M + (int)gridDim.x - 1) / (int)gridDim.x, r1 = min(a.M, ((int)blockIdx.x + 1) * per);
    for (int r = (int)blockIdx.x * per + ((int)threadIdx.x >> 4); r < r1; r += a.wg_waves * 4)
        for (int j = ((int)threadIdx.x & 15) * 4; j < a.r_cap; j += 64) {
            int8_t *const dst = a.aux_q + packed_index(r, j, a.r_cap);
            if (j >= used)
                *(uint32_t *)dst = 0u;
            else
                for (int i = max(used - j, 0); i < 4; ++i) dst[i] = 0;
        }
}

// One activation scale for the call.  The unit of work is 8 rows x 64 channels: 16 bytes of X a lane, and half a block of
// the packed codes, 512 contiguous bytes, which go out as whole lines.  A wave keeps to one column of blocks, so its
// lanes' channels, masks and all of an address but one scalar are fixed, and the work per code is the
// quantisation itself, 3 vector instructions and a share of the packing; it takes every `groups`-th block of 8 rows, up to U
// of them in flight, a request behind each one that is worked on.  All workgroups walk X together: what is in flight at one
// time is one contiguous piece of memory.  (A range of rows for each workgroup puts all of them on the same few memory
// channels where a range is a multiple of a large power of two: 16384 x 5120 from HBM 65 us instead of 45 us.)
// Few codes (up to 10 MB) are written through: stored as usual they all are dirty in the L2s when the kernel ends, and
// wait to be written back then (us a call, through / as usual: 4096 x 512 -> 256 17.1 / 17.3, 16384 x 512 (8 MB) -> 256 21.5 / 22.0, 16384 x 512 -> 1024
// 28.7 / 29.1, 8192 x 1024 (8 MB) -> 256 22.4 / 22.6, 2048 x 4096 -> 256 21.8 / 22.0).  With more of them the L2s write while the kernel runs anyway, and do it
// better by themselves: from 10 to 20 MB no difference (24576 x 512 25.5 / 25.6, 12288 x 1024 25.5 / 25.5), then up to 2 % (8192 x 4096 61.3 / 60.0, 40000 x 1024
// 59.4 / 58.5), once none (16384 x 5120 112.3 / 112.6).
// Against rows of 64 chunks to a wave, four rows requested at a time (64-byte pieces of the codes): 8192 x 1024 11.8 -> 9.4 us, 8192
// x 4096 30.2 -> 25.3 us (100 MB, 4.0 TB/s with the selection in it), a call of 9000 x 520 -> 1000 38.4 -> 28.8 us.  U = 2; 3, 4, 6
// and 8 are up to 2 % slower.
// GIVEN: the list and the column maxima are the caller's (muxq_build_aux): any list of channels, each
// named once, and any binary32 maxima.
template <bool GIVEN>
__global__ __launch_bounds__(kActThreads) void k_quantize_select(const ActArgs a)
{
    __shared__ ActShared sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int C = a.K / 8, CA = a.k_pad / 8, CB = a.k_pad / 64;
    constexpr int U = 2;
    const int G = a.groups, g = (int)blockIdx.x * a.waves + wave, rg = quotient(g, a.by_pieces), cb = g - rg * CB;
    const int nb = (a.M + 7) >> 3;
    int rb = wave < a.waves && rg < G ? rg : nb;         // block of 8 rows (waves without one: past the end)
    const int c = cb * 8 + (lane & 7), lr = lane >> 3;
    const bool in_c = c < C;
    const uint16_t *const xc = a.x + min(c, C - 1) * 8;  // (lanes of the K padding read the last channels)
    uint4 raw[U];
    auto load = [&](int b) { return *(const uint4 *)(xc + (size_t)min(b * 8 + lr, a.M - 1) * a.ldx); };
    auto load_first = [&] {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (rb + u * G < nb) raw[u] = load(rb + u * G);
    };
    if (GIVEN) load_first();

    const float shrink = __uint_as_float((uint32_t)(127 - a.exp) << 23);  // 2^-exp
    float sx, inv;
    int z = 0, used;
    if (GIVEN) {
        used = max(0, min(a.n_outliers[0], a.r_cap));
        if (tid < CA) sh.mask[tid] = 0;
        if (tid == 0) sh.amax = 0.f;
        lds_barrier();
        for (int j = tid; j < used; j += a.wg_waves * 64) {
            const int k = a.idx[j];
            if (k >= 0 && k < a.K) {
                sh.slot[k] = (uint16_t)j;
                atomicOr((uint32_t *)(sh.mask + ((k >> 3) & ~3)), 1u << ((k & 7) + 8 * ((k >> 3) & 3)));
            }
        }
        lds_barrier();
        float amax = 0.f;
        if (tid < C) {
            const uint32_t m = sh.mask[tid];
#pragma unroll
            for (int i = 0; i < 8; ++i) amax = fmaxf(amax, a.col_absmax[tid * 8 + i] * ((m >> i) & 1u ? shrink : 1.0f));
        }
        for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
        if ((tid & 63) == 0) atomicMax((uint32_t *)&sh.amax, __float_as_uint(amax));
        lds_barrier();
        amax = sh.amax;
        sx = amax > 0.f ? amax / a.qmax : 0.f;       // correctly rounded binary32 divisions (Eq. 1)
        inv = amax > 0.f ? a.qmax / amax : 0.f;
        if (blockIdx.x == 0 && tid == 0) {
            a.x_scale[0] = sx;
            a.x_scale[1] = inv;
        }
    } else {
        uint4 mx;
        const Selected sel = act_select<true, true>(a, sh, shrink, mx, load_first);
        used = sel.used;
        sx = sh.sx;
        inv = sh.inv;
        z = sh.z;
        if (tid < CA && store_share(wave))
            store_selection(sel, mx, tid, C, CA, a.r_cap, true, inv, shrink, a.col_absmax, a.col_scale, a.col_slot, a.col_mask, a.idx);
        if (blockIdx.x == 0) {
            store_list_rest(sel, a.r_cap, a.idx, a.n_outliers);
            if (tid == 0) {
                a.x_scale[0] = sx;
                a.x_scale[1] = inv;
                a.zero_point[0] = z;
            }
        }
    }
    const ActGather g_aux = gather_request(a, sh, (int)blockIdx.x * a.wg_waves * 4 + (tid >> 4), used);

    const float inv_listed = inv * shrink, magic = 12582912.0f + (float)z;
    const uint32_t mask = rb < nb && in_c ? sh.mask[c] : 0u;
    const bool wave_listed = __ballot(mask != 0) != 0;
    const uint32_t keep = in_c ? ~0u : 0u;               // K padding of Body: zeros
    const bool through = (size_t)a.M * a.k_pad <= (size_t)10 << 20;
    // the multiplier and the rounding constant of each of the thread's channels, once: where the list is
    // full its entries are the lowest channels (the capacity rule), all in the first columns, and codes put
    // right one by one made those waves the last (64 of 4096 channels: 34 us against 27 us)
    float mul[8], mag[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const bool l = ((mask >> i) & 1u) != 0;
        mul[i] = l ? inv_listed : inv;
        mag[i] = l ? 12582912.0f : magic;
    }
    while (rb < nb) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (rb >= nb) break;
            const f16x8 h = __builtin_bit_cast(f16x8, raw[u]);
            if (rb + U * G < nb) raw[u] = load(rb + U * G);
            uint32_t q[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) q[i] = quant_word((float)h[i], mul[i], a.qmax, mag[i]);
            const uint2 packed = make_uint2(pack_low_bytes(q[0], q[1], q[2], q[3]) & keep, pack_low_bytes(q[4], q[5], q[6], q[7]) & keep);
            const int r = rb * 8 + lr;
            if (r < a.M) {
                int8_t *const dst = a.body_q + ((size_t)(rb >> 1) * CB + cb) * 1024 + (rb & 1) * 512;      // = packed_index(8 rb, 64 cb)
                if (through)
                    store_through(dst + lane * 8, packed);
                else
                    *(uint2 *)(dst + lane * 8) = packed;
                if (wave_listed)
                    for (uint32_t mm = mask; mm != 0; mm &= mm - 1) {          // Aux (Eq. 5)
                        const int i = __builtin_ctz(mm);
                        a.aux_q[packed_index(r, sh.slot[c * 8 + i], a.r_cap)] =
                            (int8_t)((i < 4 ? packed.x : packed.y) >> ((i & 3) * 8));
                    }
            }
            rb += G;
        }
    }
    zero_aux_rest(a, used);
    gather_rest(a, sh, used, g_aux);
}

// One activation scale per row.  A wave takes 64 / LANES rows x NB pieces of LANES chunks, 16 bytes of each piece a lane, in
// registers from the rows' maxima to the codes: with 16 lanes to a row, what is worked out for a row (its maximum over the lanes, the
// scale, two divisions) is worked out for 4 rows at once, and the codes go out as 256 contiguous bytes.  The next rows are
// requested piece by piece as these are worked on.  (All at once before the maxima, whether there are any or not: calls with several steps of
// rows up to 4 KB 1-2 % faster, with one step 0.5 us slower; and as a kernel of its own for several steps an MLP, whose two layers then run
// different ones, 2-3 us slower: 8192 x 440 -> 1760 -> 440 66.0 / 68.6, 9000 x 264 58.2 / 60.2.)  Rows longer than that are in `pieces` waves, whose maxima meet in LDS (one
// barrier per step; the two halves of `s_piece` take turns).  Against single rows of up to 4 x 64 chunks a wave: 16384 x 1280
// 24.8 -> 21.8 us (63 MB, with the selection in it), a call of 60000 x 1280 -> 512 138 -> 122 us.  The codes are written through, however many:
// as usual / through, calls with N = 256, 4096 x 512 18.4 / 18.3, 16384 x 512 (8 MB) 25.2 / 24.3, 16384 x 1280 (21 MB) 39.0 / 38.4, 8192 x 4096 (33 MB)
// 65.6 / 64.3, 16384 x 5120 (84 MB) 116.7 / 115.9, 30000 x 4096 (123 MB) 158.9 / 158.2; only with N = 1024 and from 100 MB on as usual is ahead by 0.5 %.
// A kernel starts with a cold instruction cache, and what is unrolled NB times is kept short (1 KB of code takes about 0.12 us
// to fetch: 10 pieces with everything unrolled was 2 us slower than 4 on 1024 x 768): the column masks of the maxima come from LDS, and pieces
// with a listed channel or K padding are put aside, in LDS, for a rolled loop.
// STATIC: the list was fixed offline (a kernel of its own: nothing waits for slabs, and the rows are requested first).
template <int NB, int LANES, bool STATIC>
__global__ __launch_bounds__(kActThreads) void k_rows_select(const ActArgs a)
{
    constexpr int R = 64 / LANES;
    static_assert(NB * LANES <= 128, "what is put aside fits LDS");
    __shared__ ActShared sh;
    __shared__ __attribute__((aligned(16))) uint32_t s_piece[2][kActWaves * 4 * R];
    __shared__ uint4 s_aside[kActWaves][NB][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int C = a.K / 8, CA = a.k_pad / 8;
    const int S = a.pieces, S4 = (S + 3) & ~3, P = a.groups, p = quotient(wave, a.by_pieces), seg = wave - p * S;
    const int c0 = seg * NB * LANES + lane % LANES, lr = lane / LANES, n_rb = (a.M + R - 1) / R;
    uint4 raw[NB];
    auto chunk = [&](int j) { return min(c0 + j * LANES, C - 1); };          // (past the end the last chunk again)
    auto row_of = [&](int rb) { return a.x + (size_t)min(min(rb, n_rb - 1) * R + lr, a.M - 1) * a.ldx; };
    auto load = [&](const uint16_t *row, int j) { return *(const uint4 *)(row + chunk(j) * 8); };
    const int stride = (int)gridDim.x * P;
    int rb = (int)blockIdx.x * P + p;
    auto load_first = [&] {
        if (p < P && rb < n_rb) {
            const uint16_t *const row = row_of(rb);
#pragma unroll
            for (int j = 0; j < NB; ++j) raw[j] = load(row, j);
        }
    };
    if (STATIC) load_first();
    if (tid < 2 * kActWaves * 4 * R) (&s_piece[0][0])[tid] = 0;

    const float shrink = __uint_as_float((uint32_t)(127 - a.exp) << 23);  // 2^-exp
    uint4 mx;
    const Selected sel = act_select<!STATIC, false>(a, sh, shrink, mx, load_first);
    if (!STATIC) {
        if (tid < CA && store_share(wave))
            store_selection(sel, mx, tid, C, CA, a.r_cap, false, 0.f, shrink, a.col_absmax, a.col_scale, a.col_slot, a.col_mask, a.idx);
        if (blockIdx.x == 0) store_list_rest(sel, a.r_cap, a.idx, a.n_outliers);
    }
    const int used = __builtin_amdgcn_readfirstlane(sel.used);       // (the same in every lane)
    const ActGather g = gather_request(a, sh, (int)blockIdx.x * a.wg_waves * 4 + (tid >> 4), used);
    // magnitudes of the unlisted channels of each chunk (the parts of the fold have been read)
    uint4 *const s_unlisted = sh.part;
    if (tid < C) {
        const uint32_t m = sh.mask[tid];
        uint32_t d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i] = (m >> (2 * i) & 1u ? 0u : 0x7fffu) | (m >> (2 * i + 1) & 1u ? 0u : 0x7fff0000u);
        s_unlisted[tid] = make_uint4(d[0], d[1], d[2], d[3]);
    }
    uint32_t aside = 0;                                  // which pieces are not all unlisted channels
#pragma unroll 1
    for (int j = 0; j < NB; ++j) {
        const int c = c0 + j * LANES;
        if (__ballot(c >= C || sh.mask[min(c, C - 1)] != 0) != 0) aside |= 1u << j;
    }
    aside = __builtin_amdgcn_readfirstlane(aside);
    lds_barrier();

    // (the same number of steps for all waves: they meet at the barrier)
    for (int step = 0, r0 = (int)blockIdx.x * P; r0 < n_rb; ++step, r0 += stride, rb += stride) {
        const bool on = p < P && rb < n_rb;
        uint32_t m = 0;
        if (on) {
            // listed and unlisted apart, two halves to a word
            uint32_t nm = 0, lm = 0;
            auto take = [&](const uint4 &v, const uint4 &k) {
                nm = pk_max_u16(pk_max_u16(pk_max_u16(nm, v.x & k.x), pk_max_u16(v.y & k.y, v.z & k.z)), v.w & k.w);
                lm = pk_max_u16(pk_max_u16(pk_max_u16(lm, v.x & ~k.x & 0x7fff7fffu), pk_max_u16(v.y & ~k.y & 0x7fff7fffu, v.z & ~k.z & 0x7fff7fffu)),
                                v.w & ~k.w & 0x7fff7fffu);
            };
            auto both = [&] { return max(nm & 0xffffu, nm >> 16) | max(lm & 0xffffu, lm >> 16) << 16; };
#pragma unroll
            for (int j = 0; j < NB; ++j) take(raw[j], s_unlisted[chunk(j)]);
            m = lanes_max_u16x2<LANES>(both());
            // (a NaN wins the integer comparison, so it shows; the maxima are taken again without it)
            if (__ballot((m & 0xffffu) > 0x7c00u || (m >> 16) > 0x7c00u) != 0) {
                const uint16_t *const row = row_of(rb);
                nm = lm = 0;
#pragma unroll 1
                for (int j = 0; j < NB; ++j) take(drop_nan(load(row, j)), s_unlisted[chunk(j)]);
                m = lanes_max_u16x2<LANES>(both());
            }
        }
        if (S > 1) {
            if (on && lane % LANES == 0) s_piece[step & 1][(p * R + lr) * S4 + seg] = m;
            lds_barrier();
            if (on)
                for (int i = 0; i < S; i += 4) {
                    const uint4 o = *(const uint4 *)&s_piece[step & 1][(p * R + lr) * S4 + i];
                    m = pk_max_u16(m, pk_max_u16(pk_max_u16(o.x, o.y), pk_max_u16(o.z, o.w)));
                }
        }
        if (!on) continue;
        const int row = rb * R + lr;
        float sx, inv;
        int z;
        call_scale(m, shrink, a.qmax, sx, inv, z);
        if (seg == 0 && lane % LANES == 0 && row < a.M) {
            a.x_scale[row] = sx;
            a.x_scale[a.M + row] = inv;
            ((int32_t *)a.x_scale)[2 * (size_t)a.M + row] = z;
        }
        const float inv_listed = inv * shrink, magic = 12582912.0f + (float)z;
        const bool more = rb + stride < n_rb;
        const uint16_t *const next = row_of(rb + stride);
        int8_t *const dst = a.body_q + packed_index(row, c0 * 8, a.k_pad);
        constexpr int PIECE = LANES / 8 * 1024;          // bytes of packed codes from piece to piece
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const uint4 v = raw[j];
            if (more) raw[j] = load(next, j);
            if ((aside >> j & 1u) != 0) {
                s_aside[wave][j][lane] = v;
            } else {
                const f16x8 h = __builtin_bit_cast(f16x8, v);
                uint32_t q[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) q[i] = quant_word((float)h[i], inv, a.qmax, magic);
                const uint2 packed = make_uint2(pack_low_bytes(q[0], q[1], q[2], q[3]), pack_low_bytes(q[4], q[5], q[6], q[7]));
                if (row < a.M) store_through(dst + j * PIECE, packed);
            }
        }
#pragma unroll 1
        for (uint32_t rest = aside; rest != 0; rest &= rest - 1) {
            const int j = __builtin_ctz(rest), c = c0 + j * LANES;
            const f16x8 h = __builtin_bit_cast(f16x8, s_aside[wave][j][lane]);
            const uint32_t mask = c < C ? (uint32_t)sh.mask[c] : 0u;
            uint32_t q[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {                // listed channels: shrunk, no z
                const bool l = ((mask >> i) & 1u) != 0;
                q[i] = quant_word((float)h[i], l ? inv_listed : inv, a.qmax, l ? 12582912.0f : magic);
            }
            uint2 packed = make_uint2(pack_low_bytes(q[0], q[1], q[2], q[3]), pack_low_bytes(q[4], q[5], q[6], q[7]));
            if (c >= C) packed = make_uint2(0, 0);       // K padding of Body
            if (row < a.M && c < CA) {
                store_through(dst + j * PIECE, packed);
                for (uint32_t mm = mask; mm != 0; mm &= mm - 1) {      // Aux (Eq. 5)
                    const int i = __builtin_ctz(mm);
                    a.aux_q[packed_index(row, sh.slot[c * 8 + i], a.r_cap)] = (int8_t)((i < 4 ? packed.x : packed.y) >> ((i & 3) * 8));
                }
            }
        }
    }
    zero_aux_rest(a, used);
    gather_rest(a, sh, used, g);
}

// muxq_detect_outliers: the fold and the list by themselves, one workgroup.  Bound by latency (5120 channels 5.5 -> 4.7 us against
// the kernel that also leaves what the separate quantisers read).  8 waves instead of 16 would do up to 4096 channels and are neither better nor
// worse: both kernels of a call replayed 20 times, 1 x 256 5.0 / 5.0 us, 64 x 2048 5.1 / 5.1, 1 x 4096 5.3 / 5.2, 1024 x 1024 5.5 / 5.8, 300 x 3072 5.6 / 5.4.
__global__ __launch_bounds__(kActThreads) void k_detect_select(const ActArgs a)
{
    __shared__ ActShared sh;
    const int tid = threadIdx.x;
    uint4 mx;
    const Selected sel = act_select<true, false>(a, sh, 1.f, mx, [] {});
    if (tid < a.K / 8) {
        float v[8];
        widen8(mx, v);
        if (((uintptr_t)a.col_absmax & 15) == 0) {
            ((float4 *)(a.col_absmax + tid * 8))[0] = make_float4(v[0], v[1], v[2], v[3]);
            ((float4 *)(a.col_absmax + tid * 8))[1] = make_float4(v[4], v[5], v[6], v[7]);
        } else {
            for (int i = 0; i < 8; ++i) a.col_absmax[tid * 8 + i] = v[i];
        }
    }
    for (int j = tid; j < sel.used; j += kActThreads) a.idx[j] = sh.idx[j];
    store_list_rest(sel, a.r_cap, a.idx, a.n_outliers);
}

}  // namespace

bool act_select_fits(int k_pad, int r_cap) { return k_pad <= kActMaxK && r_cap <= kActMaxCap; }

// With one scale per call and X beyond what the 256 MB memory-side cache keeps, both passes stream from HBM, and the
// 2048 small workgroups of the separate kernels do that better than 256 large ones; the selection kernel between
// them no longer weighs.  us a layer, separate kernels / these, 64 output channels: 20505 x 4096 (168 MB) 97 / 98, 24409 x
// 4096 (200 MB) 138 / 140, 146481 x 4096 (1.2 GB) 707 / 777, 78121 x 1280 (200 MB) 133 / 145; up to 1024 channels these
// win at any size: 97657 x 1024 (200 MB) 133 / 131; so do they with very long rows (73241 x 8192 765 / 734).  (With one scale per row the separate kernel is always the slower one.)
bool act_select_pays(int M, int K) { return K <= 1024 || K > 6144 || (size_t)M * K * 2 < ((size_t)176 << 20); }

// The same for muxq_build_aux, whose list and maxima come from outside: 40000 x 4096 (328 MB) 100 / 116 us, 50000 x 5120
// (512 MB) 175 / 152, 97657 x 1024 (200 MB) 66 / 58; short rows 250001 x 256 (128 MB) 54 / 68, 500001 x 256 (256 MB)
// 135 / 120, 312497 x 512 (320 MB) 113 / 120.
bool act_given_pays(int M, int K)
{
    const size_t mib = ((size_t)M * K * 2) >> 20;
    return !(mib >= 288 && K >= 1024 && K < 5120) && !(mib >= 60 && (K <= 256 ? mib < 200 : K <= 512));
}

// And for the abs-max pass by itself, blocks of 512 columns / narrow ones: 262144 x 4096 (2 GB) 332 / 353 us, 256 MB of 4096
// channels narrow 4 % faster, 400000 x 256 84 / 34.
bool absmax_narrow_pays(int M, int K) { return K < 2048 || (size_t)M * K * 2 < ((size_t)480 << 20); }

hipError_t launch_col_absmax_narrow(const void *x_fp16, int rows, int cols, int ld, int k_pad, uint16_t *partial,
                                    int *n_slabs, hipStream_t s)
{
    // about one workgroup per CU, at least 64 rows each
    const int gx = (k_pad / 8 + kNarrowLanes - 1) / kNarrowLanes;
    int gy = max(1, min(kMaxSlabs, 256 / gx));
    gy = max(1, min(gy, (rows + 63) / 64));
    const int rpb = ((rows + gy - 1) / gy + 63) & ~63;
    gy = (rows + rpb - 1) / rpb;
    *n_slabs = gy;
    return launch_kernel(k_col_absmax_narrow, dim3(gx, gy), dim3(512), 0, s,
                         (const uint16_t *)x_fp16, rows, cols, ld, k_pad, rpb, partial);
}

hipError_t launch_fold_slabs(uint16_t *partial, int n_slabs, int k_pad, hipStream_t s)
{
    return launch_kernel(k_fold_slabs, dim3((k_pad / 8 + 63) / 64), dim3(256), 0, s, partial, n_slabs, k_pad);
}

// The form of k_rows_select: single rows in pieces of 2 x 64 chunks, or 4 rows in pieces of 4 or 5 x 16, by the least of three estimates.
// One step, or rows beyond 4 KB: bound by the vector instructions, about 60 for a piece of 64 lanes x 16 bytes and 200 for what is worked
// out once per row, times the waves on a SIMD and the steps (19 shapes, 24 x 5120 to 60000 x 1280: the fastest or within 1 %; us a call, single
// rows / 4 rows x 4 / 4 rows x 5: 512 x 4096 -> 1024 21.8 / 22.4 / 22.7, 2000 x 1280 -> 1280 23.6 / 22.8 / 23.0, 8192 x 4096 -> 1024 81.1 / 73.7 / 74.6).
// Several steps of shorter rows: the latency of a step counts as well (the 8 in the estimate), and the barrier of rows in several waves, most of
// all from step to step; fitted to 232 calls in each form.  There the groups are also spread evenly over the steps, unless the last one is
// nearly empty.  us a call, single rows of up to 4 x 64 chunks as before the three forms / the first estimate for all / now: 10240 x 1024 -> 256
// 29.1 / 30.4 / 28.2, 20000 x 1024 38.3 / 40.7 / 38.4, 9004 x 896 static 21.7 / 23.5 / 20.3, 16384 x 1424 44.4 / 46.6 / 43.5, 16384 x 1592 47.5 / 50.2 / 48.6; 16386 x 576,
// whose second step is one group, evenly 30.1, otherwise 28.3.  With one step the second estimate takes single rows up to 4096 x 1000, no
// faster by themselves, and an MLP of them is slower: 4096 x 768 -> 3072 -> 768 per token 69.0 / 71.2.
// Returns the groups of rows; pieces: waves to a group, at_once: groups of a workgroup at a time.
int row_form(int M, int k_pad, int &form, int &pieces, int &at_once)
{
    static const struct { int pieces, lanes; } kForms[3] = {{2, 64}, {4, 16}, {5, 16}};
    // (more than one step: of 4 rows to a wave in pieces of 4 x 16 chunks)
    const bool short_rows = k_pad <= 2048 && M > 4 * 256 * (kActWaves / ((k_pad / 8 + 63) / 64));
    int groups = 0;
    long long best = -1;
    for (int f = 0; f < 3; ++f) {
        const int NB = kForms[f].pieces, rows = 64 / kForms[f].lanes, n = (M + rows - 1) / rows;
        const int S = (k_pad / 8 + NB * kForms[f].lanes - 1) / (NB * kForms[f].lanes);
        const int most = 256 * (kActWaves / S), steps = (n + most - 1) / most;
        int P = min(kActWaves / S, (n + 255) / 256);
        if (short_rows && steps > 1 && (n - 1) % most >= most / 8) P = (n + 256 * steps - 1) / (256 * steps);
        const int waves = (P * S + 3) / 4;
        const long long cost = !short_rows ? (long long)steps * waves * (60 * NB + 200)
                               : (long long)steps * (waves + 8) * (60 * NB + (rows == 1 ? 140 : 70)) + (S == 1 ? 0 : steps == 1 ? 1000 : 4680);
        if (best >= 0 && cost >= best) continue;
        best = cost;
        form = f;
        groups = n;
        pieces = S;
        at_once = P;
    }
    return groups;
}

hipError_t launch_detect_select(const ActArgs &args, hipStream_t s)
{
    ActArgs a = args;
    a.by_chunks = divisor(a.k_pad / 8);
    a.cut = magnitude_cut(a.threshold);
    a.wg_waves = kActWaves;
    return launch_kernel(k_detect_select, dim3(1), dim3(kActThreads), 0, s, a);
}

hipError_t launch_quantize_select(const ActArgs &args, bool per_token, bool given, hipStream_t s)
{
    ActArgs a = args;
    a.by_chunks = divisor(a.k_pad / 8);
    const bool is_static = a.static_mask != nullptr;
    if (!given && !is_static) a.cut = magnitude_cut(a.threshold);
    // every workgroup selects for itself, so no more of them than are resident at once, but enough for
    // a share of the weight side each (4 output channels a wave)
    const int most = 256;
    int units, form = 0;                                 // units: what a wave takes at a time
    if (!per_token) {
        // columns of 64 channels, and as many waves as there are blocks of 8 rows in them
        const int columns = a.k_pad / 64, blocks = (a.M + 7) / 8;
        a.by_pieces = divisor(columns);
        a.waves = (int)min((long long)kActWaves, ((long long)columns * blocks + most - 1) / most);
        units = (int)min((long long)most * a.waves, (long long)columns * blocks);
    } else {
        units = row_form(a.M, a.k_pad, form, a.pieces, a.groups);
        a.by_pieces = divisor(a.pieces);
        a.waves = a.groups * a.pieces;
    }
    // A workgroup of 8 waves where they are enough, for the rows, the chunks and a step of the weight side: what all waves do, the
    // selection above all, is bound by the issue of its instructions.  us a call with 16 / 8: 100 x 2000 -> 640 13.3 / 12.3, 1024 x 768
    // -> 3072 17.9 / 17.7, 40 x 3000 -> 3000 14.4 / 14.1; 50 x 1000 -> 16384 (two steps of the weight side) 14.9 / 16.1.
    a.wg_waves = max(a.waves, (a.k_pad + 511) / 512) <= 8 && (a.cn == nullptr || a.N <= most * 32) ? 8 : kActWaves;
    const int weight_side = a.cn != nullptr ? (a.N + 4 * a.wg_waves - 1) / (4 * a.wg_waves) : 1;
    const int grid = min(max((units + (per_token ? a.groups : a.waves) - 1) / (per_token ? a.groups : a.waves), weight_side), most);
    if (!per_token) a.groups = min(grid * a.waves / (a.k_pad / 64), (a.M + 7) / 8);
    void (*kern)(const ActArgs);
    if (!per_token)
        kern = given ? k_quantize_select<true> : k_quantize_select<false>;
    else if (form == 0)
        kern = is_static ? k_rows_select<2, 64, true> : k_rows_select<2, 64, false>;
    else if (form == 1)
        kern = is_static ? k_rows_select<4, 16, true> : k_rows_select<4, 16, false>;
    else
        kern = is_static ? k_rows_select<5, 16, true> : k_rows_select<5, 16, false>;
    return launch_kernel(kern, dim3(grid), dim3(a.wg_waves * 64), 0, s, a);
}

}  // namespace muxq
