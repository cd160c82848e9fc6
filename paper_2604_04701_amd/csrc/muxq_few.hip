// The whole MUXQ linear layer for few tokens (a decode step) as ONE launch.
//
// With few rows of X every stage of the layer is short, and what a call costs is the launches
// and the memory round trips between them: a dependent launch takes 4-5 us on this chip however
// little it does, and a GEMM kernel made of 64 x 64 or 128 x 128 output tiles leaves most CUs
// without a tile.  So here every workgroup does the activation side of ALL rows for itself --
// column maxima, outlier selection, codes, kept in LDS -- and then the product for 16 output
// channels at a time.  What bounds it now: the instructions that every wave repeats and the latencies between them, up to
// about 8 K elements of X (1 x 768 -> 2304: 4.5 us inside the kernel), the vector ALU work of the codes, repeated on
// every CU, beyond (8 x 5120: 3 of 9.5 us).
// Measured, us per call, four launches with a selection kernel against this kernel with 16 waves (see few_waves): 1 x 768 -> 2304 18.8 / 8.4,
// 1 x 8192 -> 1024 49.1 / 10.1, 8 x 1280 -> 5120 -> 1280 (an MLP with both layers in this kernel, two launches instead of eight)
// 61.5 / 24.7, 16 x 2560 -> 2560 28.8 / 11.2, 2 x 4096 -> 16384 36.8 / 20.5; against the launches that
// would run here without it, see few_tokens_fit.
//
// Product.  A block of the packed weight layout is 16 output channels x 64 input channels, 1 KiB
// contiguous, which is exactly the first operand of one v_mfma_i32_16x16x64_i8: lane l takes the
// 16 bytes of channel l % 16 at input channels 16 (l / 16).  Weights therefore go from memory
// straight to registers, each byte once per call, in loads of whole KiB; the waves of the
// workgroup split K, and their INT32 partial sums meet in LDS (integer adds: any order gives the
// same sum).  The loads of the first 16 channels are issued before anything else, so that the
// activation side runs in the shadow of their latency.
//
// Everything a caller may read from the workspace afterwards (the muxq_workspace_layout regions)
// is written as by the separate launches: the selection results and the codes in shares by
// the workgroups, w_aux and cn by the workgroup that owns the channels.
#include "muxq_select.h"

namespace muxq {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

constexpr int kFewMaxWaves = 16;                             // of a workgroup, see few_waves
constexpr int kFewMaxK = 8 * 64 * kFewMaxWaves;              // one 8-channel chunk per thread in the selection
constexpr int kFewMaxM = 64;
constexpr int kFewGrid = 256;                               // workgroups, one to a CU (see few_two_on_a_cu)
constexpr int kFewTwoM = 4;                                  // most rows with which two share a CU
// Weight blocks of a wave, all in registers, by 16-row blocks of tokens: enough for the K that
// few_tokens_fit lets through.  (Eight for all of them made the forms above 16 tokens spill to scratch.)
constexpr int few_loads(int row_blocks) { return row_blocks == 1 ? kFewMaxK / 64 / kFewMaxWaves : row_blocks == 2 ? 3 : 1; }

// What the kernel needs besides FewArgs, worked out on the host: the division of its waves and LDS.
struct FewPlan {
    int waves;               // of a workgroup
    int pieces, groups;      // a row of X is `pieces` pieces of 64 chunks (8 channels each); rows in flight at once
    int div;                 // wave / pieces == wave * div >> 16
    int share_parts, share_len;          // codes for the caller: a row in so many parts of so many 16-byte units
    int codes, aux, waux, red, idx, part, total;     // LDS offsets (X itself at 0)
    int cut;                 // the threshold, see chunk_candidates
};

FewPlan few_plan(int M, int K, int k_pad, int r_cap, int grid, int waves)
{
    FewPlan P;
    P.waves = waves;
    P.pieces = (k_pad / 8 + 63) / 64;
    P.groups = waves / P.pieces;
    P.div = 65536 / P.pieces + 1;
    P.share_parts = grid / M > 1 ? grid / M : 1;
    const int units = k_pad / 16;
    P.share_len = (units + P.share_parts - 1) / P.share_parts;
    int off = M * K * 2;                                     // X, row after row
    P.codes = off; off += M * k_pad;                         // codes of Body, tight rows
    P.aux = off;   off += M * r_cap;                         // codes of Aux
    P.waux = off;  off += 16 * r_cap;                        // Aux weight rows of the current 16 channels
    P.red = off;   off += (M + 15) / 16 * 1024;              // partial sums
    P.idx = off;   off += r_cap * 4;                         // the list
    // partial column maxima, before there are codes or sums
    P.part = P.codes;
    if (P.part + waves * 1024 > off) off = P.part + waves * 1024;
    P.total = off;
    return P;
}

// Byte of (row, column) in an LDS code matrix of M rows and `cols` columns: blocks of 16 rows x 64
// columns like the packed layout, the last one with as many rows as there are; the four 16-byte
// chunks of a row are XOR-swizzled with row bits, so that the 16 rows a fragment read touches at
// one chunk fall into different banks.
__device__ __forceinline__ int few_code_pos(int row, int col, int M, int cols)
{
    const int mb = row >> 4, r = row & 15, rows = min(16, M - (mb << 4));
    return (mb << 4) * cols + (col >> 6) * (rows << 6) + (r << 6) + ((((col >> 4) & 3) ^ (r >> 2)) << 4) + (col & 15);
}

// MB: 16-row blocks of tokens (1, 2 or 4).  TOKEN: one activation scale per row.
// (Loops over rows are kept rolled: a kernel starts with a cold instruction cache, and straight-line
// code for eight rows takes longer to fetch than to run.)
template <int MB, bool TOKEN>
__global__ __launch_bounds__(kFewMaxWaves * 64) void k_linear_few(const FewArgs a, const FewPlan L)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    typedef __attribute__((address_space(3))) void *lptr_t;
    constexpr int LOADS = few_loads(MB);
    __shared__ __attribute__((aligned(16))) int s_tot[kFewMaxWaves];
    __shared__ __attribute__((aligned(16))) uint32_t s_max[kFewMaxWaves];
    __shared__ uint32_t s_row[kFewMaxM * kFewMaxWaves];     // per token: the maxima of a row's pieces
    __shared__ float s_sx[kFewMaxM], s_inv[kFewMaxM];
    __shared__ int s_z[kFewMaxM];
    __shared__ uint32_t s_pick[kFewMaxK / 8];            // per chunk: which channels are listed, rank of the first << 8

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, K = a.K, k_pad = a.k_pad, N = a.N, r_cap = a.r_cap;
    const int W = L.waves, threads = W * 64;
    unsigned char *const codes = lds + L.codes;
    unsigned char *const aux = lds + L.aux;
    unsigned char *const waux = lds + L.waux;
    int *const red = (int *)(lds + L.red);
    int *const idx_lds = (int *)(lds + L.idx);
    const int C = K / 8, CA = k_pad / 8;                 // 8-channel chunks: real, with the padding
    const int KB = k_pad / 64, nblk = (N + 15) >> 4, n_mb = (M + 15) >> 4;
    const int ln = lane & 15, lq = lane >> 4;            // MFMA lane: row of the block, 16-byte chunk

    // Activation side: a wave owns piece `seg` of the rows p, p + P, ...; a thread its chunk c there.
    const int S = L.pieces, P = L.groups;
    const int p = wave * L.div >> 16, seg = wave - p * S, c = seg * 64 + lane;
    const bool in_c = c < C && p < P;
    const int row0 = p < P ? p : M;                      // (waves without a row: none)
    const unsigned char *const xc = lds + c * 16;        // this thread's chunk, + row * 2 K

    // X goes straight to LDS, all of it in flight at once (the wave's 64 x 16 bytes are contiguous)
    {
        const __amdgpu_buffer_rsrc_t r_x = __builtin_amdgcn_make_buffer_rsrc(
            (void *)a.x, 0, (int)(((unsigned)(M - 1) * (unsigned)a.ldx + (unsigned)K) * 2u), 0x00020000);
        if (in_c)
            for (int row = row0; row < M; row += P)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(r_x, (lptr_t)(lds + row * K * 2 + seg * 1024), 16,
                                                         (unsigned)c * 16u, (unsigned)row * (unsigned)a.ldx * 2u, 0, 0);
    }
    const bool is_static = a.static_mask != nullptr;
    const bool want_max = !(TOKEN && is_static);
    uint32_t listed = 0;                                 // bit i: channel 8 c + i is listed
    uint4 mx = make_uint4(0, 0, 0, 0);                   // column maxima
    if (in_c && is_static) listed = a.static_mask[c];
    if (in_c && a.slabs != nullptr && want_max)          // left by the producer of X; one or two
        for (int sl = 0; sl < a.n_slabs; ++sl)
            mx = absmax_step(mx, *(const uint4 *)(a.slabs + (size_t)sl * k_pad + c * 8));

    // the weight blocks of the first 16 channels, on their way during all that follows
    int nb = blockIdx.x;
    v4i w[LOADS];
    auto load_weights = [&](int nblock) {
        const int8_t *src = a.w_q + (size_t)nblock * k_pad * 16 + ln * 64 + lq * 16;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int kb = wave + i * W;
            if (kb < KB) w[i] = *(const v4i *)(src + (size_t)kb * 1024);
        }
    };
    load_weights(nb);
    // constants of the epilogue (waves 0 .. n_mb - 1: lane = token ln, channels n .. n + 3)
    v4i rs = {0, 0, 0, 0};
    float4 sw = make_float4(0.f, 0.f, 0.f, 0.f);
    f16x4 bias = {0, 0, 0, 0};
    auto load_consts = [&](int nblock) {
        const int n = nblock * 16 + lq * 4;
        if (wave < n_mb && n < N) {                      // N % 8 == 0: a run of 4 is in or out as a whole
            rs = *(const v4i *)(a.w_row_sum + n);
            const int st = a.w_per_channel ? 1 : 0, n0 = a.w_per_channel ? n : 0;
            sw = make_float4(a.w_scale[n0], a.w_scale[n0 + st], a.w_scale[n0 + 2 * st], a.w_scale[n0 + 3 * st]);
            if (a.bias != nullptr) {
#pragma unroll
                for (int i = 0; i < 4; ++i) bias[i] = a.bias[n + i];
            }
        }
    };
    load_consts(nb);

    // X has landed (and with it the weights: both come from memory at the same time); a wave reads
    // back only what it loaded itself
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0)
    asm volatile("" ::: "memory");

    // ---- column maxima of |X| (Sec. III-C) ----
    if (want_max && a.slabs == nullptr) {
        if (in_c)
            for (int row = row0; row < M; row += P) mx = absmax_step(mx, *(const uint4 *)(xc + row * K * 2));
        if (min(P, M) > 1) {                             // the row groups' parts meet
            uint4 *const part = (uint4 *)(lds + L.part);
            part[tid] = mx;
            lds_barrier();
            if (p == 0)
                for (int g = 1; g < min(P, M); ++g) mx = absmax_step(mx, part[(g * S + seg) * 64 + lane]);
        }
    }

    // ---- selection (Sec. III-C) with the capacity rule ----
    const float shrink = __uint_as_float((uint32_t)(127 - a.exp) << 23);  // 2^-exp
    // (in the waves of the first row group; the others take the lists over)
    const bool holds = p == 0;
    if (holds && !is_static) {
        listed = chunk_candidates(mx, a.threshold, L.cut);
        if (!in_c) listed = 0;
    }
    const Selected sel = select_channels(mx, listed, holds, seg, S, r_cap, !TOKEN, s_tot, s_max);
    const int used = sel.used;
    const uint32_t call_max = sel.maxima;
    // (the parts of the maxima, which may lie here, were read before the barrier of the selection)
    for (int i = tid * 4; i < M * r_cap; i += threads * 4) *(uint32_t *)(aux + i) = 0u;
    for (int i = tid * 4; i < 16 * r_cap; i += threads * 4) *(uint32_t *)(waux + i) = 0u;
    for (int i = tid; i < n_mb * 256; i += threads) red[i] = 0;
    if (holds) {
        int rank = sel.first;
        for (uint32_t mm = sel.listed; mm != 0; mm &= mm - 1, ++rank) idx_lds[rank] = c * 8 + __builtin_ctz(mm);
        s_pick[c] = sel.listed | (uint32_t)sel.first << 8;
    }
    lds_barrier();
    const uint32_t pick = p < P ? s_pick[c] : 0u;
    listed = pick & 0xffu;
    const int first = (int)(pick >> 8);

    float inv = 0.f, sx_call = 0.f;
    int z = 0;
    if (TOKEN) {
        // ---- max|Body| of every row: a wave's piece first ----
        for (int row = row0; row < M; row += P) {
            uint4 raw = make_uint4(0, 0, 0, 0);
            if (in_c) raw = *(const uint4 *)(xc + row * K * 2);
            const uint32_t m = wave_row_maxima(raw, listed);
            if (lane == 63) s_row[row * kFewMaxWaves + seg] = m;
        }
        lds_barrier();
        if (tid < M) {
            uint32_t m = 0;
            for (int s = 0; s < S; ++s) m = pk_max_u16(m, s_row[tid * kFewMaxWaves + s]);
            float sx, iv;
            int zz;
            call_scale(m, shrink, a.qmax, sx, iv, zz);
            s_sx[tid] = sx;
            s_inv[tid] = iv;
            s_z[tid] = zz;
            if (blockIdx.x == 0) {
                a.x_scale[tid] = sx;
                a.x_scale[M + tid] = iv;
                a.zero_point[tid] = zz;
            }
        }
        lds_barrier();
    } else {
        call_scale(call_max, shrink, a.qmax, sx_call, inv, z);
    }

    // Eq. 7: the weights of the listed channels, 16 per output channel and step; on their way while
    // the codes are formed (the lines have just been read, as part of the weight blocks)
    const int g_row = tid & 15, g_slot = tid >> 4;       // `slots` at a time
    const int slots = threads >> 4;
    int g_w = 0;
    auto gather_weights = [&](int nblock, int j) -> int {
        return a.w_q[(size_t)nblock * k_pad * 16 + (size_t)(idx_lds[j] >> 6) * 1024 + g_row * 64 + (idx_lds[j] & 63)];
    };
    if (g_slot < used) g_w = gather_weights(nb, g_slot);

    // ---- codes of Body and Aux (Eq. 1, 4, 5) into LDS ----
    const bool wave_listed = __ballot(listed != 0) != 0;
    if (p < P && c < CA) {
        for (int row = row0; row < M; row += P) {
            if (TOKEN) {
                inv = s_inv[row];
                z = s_z[row];
            }
            uint4 raw = make_uint4(0, 0, 0, 0);
            if (c < C) raw = *(const uint4 *)(xc + row * K * 2);
            const float magic = 12582912.0f + (float)z;
            const f16x8 h = __builtin_bit_cast(f16x8, raw);
            uint32_t q[8];
            if (wave_listed) {
                // listed channels: Body = x 2^-exp and one rounded product (the factor is a power of
                // two: its place does not matter), no zero point
                const float inv_l = inv * shrink;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool l = ((listed >> j) & 1u) != 0;
                    q[j] = quant_word((float)h[j], l ? inv_l : inv, a.qmax, l ? 12582912.0f : magic);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) q[j] = quant_word((float)h[j], inv, a.qmax, magic);
            }
            uint2 packed = make_uint2(pack_low_bytes(q[0], q[1], q[2], q[3]), pack_low_bytes(q[4], q[5], q[6], q[7]));
            if (c >= C) packed = make_uint2(0, 0);       // K padding of Body
            int slot = first;
            for (uint32_t mm = listed; mm != 0; mm &= mm - 1, ++slot) {          // Aux (Eq. 5)
                const int j = __builtin_ctz(mm);
                aux[few_code_pos(row, slot, M, r_cap)] = (uint8_t)((j < 4 ? packed.x : packed.y) >> ((j & 3) * 8));
            }
            *(uint2 *)(codes + few_code_pos(row, c * 8, M, k_pad)) = packed;
        }
    }
    auto keep_weights = [&](int nblock) {                // -> LDS; longer lists: the rest directly
        if (g_slot < used) waux[few_code_pos(g_row, g_slot, 16, r_cap)] = (uint8_t)g_w;
        for (int j = g_slot + slots; j < used; j += slots)
            waux[few_code_pos(g_row, j, 16, r_cap)] = (uint8_t)gather_weights(nblock, j);
    };
    keep_weights(nb);
    // ---- the selection results, for the caller ----
    if (want_max) {
        if (holds && (MB == 1 ? blockIdx.x == 0 : store_share(seg)))         // (with few rows the first has the time)
            store_selection(sel, mx, c, C, CA, r_cap, !TOKEN, inv, shrink, a.col_absmax, a.col_scale, a.col_slot, a.col_mask, a.idx);
        if (blockIdx.x == 0) {
            store_list_rest(sel, r_cap, a.idx, a.n_outliers);
            if (tid == 0 && !TOKEN) {
                a.x_scale[0] = sx_call;
                a.x_scale[1] = inv;
                a.zero_point[0] = z;
            }
        }
    }
    lds_barrier();
    // ---- this workgroup's share of the codes, for the caller: part of a row, or whole rows ----
    if ((int)blockIdx.x < M * L.share_parts)
        for (int row = (int)blockIdx.x % M; row < M; row += gridDim.x) {
            const int u0 = ((int)blockIdx.x / M) * L.share_len, u1 = min(k_pad / 16, u0 + L.share_len);
            for (int u = u0 + tid; u < u1; u += threads)
                *(uint4 *)(a.body_q + packed_index(row, u * 16, k_pad)) = *(const uint4 *)(codes + few_code_pos(row, u * 16, M, k_pad));
            if ((int)blockIdx.x < M && tid < r_cap / 16)
                *(uint4 *)(a.aux_q + packed_index(row, tid * 16, r_cap)) = *(const uint4 *)(aux + few_code_pos(row, tid * 16, M, r_cap));
        }

    // ---- products, 16 output channels at a time ----
    const int t_aux = (used + 63) >> 6;
    auto frag = [&](const unsigned char *m, int cols, int mb, int kb) -> v4i {
        const int rows = min(16, M - mb * 16), r = min(ln, rows - 1);     // rows past M feed outputs that are not stored
        return *(const v4i *)(m + mb * 16 * cols + kb * (rows << 6) + (r << 6) + ((lq ^ (r >> 2)) << 4));
    };
    for (; nb < nblk; nb += gridDim.x) {
        const int n = nb * 16 + lq * 4;
        const bool epi = wave < n_mb && n < N;
        v4i acc[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int kb = wave + i * W;
            if (kb >= KB) break;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                if (mb < n_mb)
                    acc[mb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[i], frag(codes, k_pad, mb, kb), acc[mb], 0, 0, 0);
        }
        if (nb + (int)gridDim.x < nblk) {
            load_weights(nb + gridDim.x);
            if (g_slot < used) g_w = gather_weights(nb + gridDim.x, g_slot);
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            if (mb < n_mb) {
#pragma unroll
                for (int v = 0; v < 4; ++v) atomicAdd(&red[(mb * 4 + v) * 64 + lane], acc[mb][v]);
            }
        lds_barrier();

        // the Aux weight rows, for the caller (a static block has them already)
        if (a.w_aux != nullptr)
            for (int u = tid; u < r_cap; u += threads) {       // 16 rows x r_cap / 16 pieces
                const int row = u & 15, col = u & ~15;
                if (nb * 16 + row < N)
                    *(uint4 *)(a.w_aux + packed_index(nb * 16 + row, col, r_cap)) =
                        *(const uint4 *)(waux + few_code_pos(row, col, 16, r_cap));
            }
        if (wave < n_mb) {
            const int mb = wave;
            // Aux product, and (second operand all ones) each channel's sum over the listed weights
            v4i ax = {0, 0, 0, 0}, sum = {0, 0, 0, 0};
            const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
            for (int t = 0; t < t_aux; ++t) {
                const v4i wa = *(const v4i *)(waux + (t << 10) + (ln << 6) + ((lq ^ (ln >> 2)) << 4));
                ax = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa, frag(aux, r_cap, mb, t), ax, 0, 0, 0);
                sum = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa, ones, sum, 0, 0, 0);
            }
            const int m = mb * 16 + ln;
            const float sx = TOKEN ? s_sx[min(m, M - 1)] : sx_call;
            if (TOKEN) z = s_z[min(m, M - 1)];
            const v4i cn = rs - sum;
            const float swv[4] = {sw.x, sw.y, sw.z, sw.w};
            f16x4 out;
            v4i total;
            uint32_t hmax[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                // Eq. 7 on INT32 accumulators, modulo 2^32 like every form of the GEMM
                total[i] = (int)((uint32_t)red[(mb * 4 + i) * 64 + lane] + ((uint32_t)ax[i] << a.exp) - (uint32_t)ax[i] -
                                 (uint32_t)z * (uint32_t)cn[i]);
                const float sc = sx * swv[i];
                float y = sc * (float)total[i];          // Eq. 3
                if (a.bias != nullptr) y = y + (float)bias[i];
                out[i] = (_Float16)y;
                // fused activation: on the fp16 value the layer would have stored
                if (a.gelu) out[i] = (_Float16)gelu_tanh_f32((float)out[i]);
                hmax[i] = m < M ? (uint32_t)__builtin_bit_cast(unsigned short, (_Float16)out[i]) & 0x7fffu : 0u;
            }
            if (epi && m < M) {
                *(f16x4 *)(a.y + (size_t)m * a.ldy + n) = out;
                if (a.dbg_acc != nullptr) *(v4i *)(a.dbg_acc + (size_t)m * N + n) = total;
            }
            if (a.cn != nullptr && epi && mb == 0 && ln == 0) *(v4i *)(a.cn + n) = cn + a.cn_bias;
            if (a.next_slabs != nullptr) {               // column maxima over the tokens, for the next layer
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    hmax[i] = max(hmax[i], dpp_zero<0x111>(hmax[i]));
                    hmax[i] = max(hmax[i], dpp_zero<0x112>(hmax[i]));
                    hmax[i] = max(hmax[i], dpp_zero<0x114>(hmax[i]));
                    hmax[i] = max(hmax[i], dpp_zero<0x118>(hmax[i]));
                }
                if (ln == 15) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) red[(mb * 4 + i) * 64 + lane] = (int)hmax[i];
                }
            }
        }
        lds_barrier();
        if (a.next_slabs != nullptr && tid < 16) {
            uint32_t m = 0;
            for (int mb = 0; mb < n_mb; ++mb) m = max(m, (uint32_t)red[(mb * 4 + (tid & 3)) * 64 + (tid >> 2) * 16 + 15]);
            if (nb * 16 + tid >= N) m = 0;
            for (int sl = 0; sl < a.next_count; ++sl)              // the whole maximum sits in slab 0
                a.next_slabs[(size_t)sl * a.next_ld + nb * 16 + tid] = sl == 0 ? (uint16_t)m : (uint16_t)0;
        }
        if (nb + (int)gridDim.x < nblk) {
            load_consts(nb + gridDim.x);
            keep_weights(nb + gridDim.x);                // (waux is consumed: the barrier above)
            if (a.next_slabs != nullptr) lds_barrier();
            for (int i = tid; i < n_mb * 256; i += threads) red[i] = 0;
            lds_barrier();
        }
    }
    // the K padding of the next layer's slabs past the last 16 channels of this one
    if (a.next_slabs != nullptr && blockIdx.x == 0)
        for (int i = nblk * 16 + tid; i < a.next_ld; i += threads)
            for (int sl = 0; sl < a.next_count; ++sl) a.next_slabs[(size_t)sl * a.next_ld + i] = 0;
}

}  // namespace

// Waves of a workgroup.  Every wave walks through the whole kernel, much of which is not divided among them (about 800
// instructions, 4 cycles each), so with four waves on a SIMD small calls are bound by their issue.  A long K, whose weights
// want many loads in flight, takes 16 all the same, else many rows 12 and few rows 8; whole row groups of waves, since a thread has one
// chunk of the rows, and no more weight blocks to a wave than it has registers for.  us a call with 8 / 12 / 16: 1 x 768 -> 2304 6.8 /
// 7.1 / 7.4, 4 x 1024 -> 1024 7.2 / 7.6 / 8.0, 8 x 1280 -> 5120 10.9 / 10.0 / 10.4, 16 x 1280 -> 3840 14.5 / 11.4 / 12.0, 3 x 3000 -> 8000
// 13.7 / 12.4 / 12.4, 8 x 4096 -> 4096 13.6 / 13.6 / 12.4.
// Whole row groups are 9 to 15 waves with a K beyond 4096.  Where the workgroups walk over N, the weights decide, and 16 it is, the rest of
// them for the weights alone: whole groups / 16, 1 x 4368 -> 6424 13.2 / 12.3, 1 x 4608 -> 14336 22.0 / 20.2, 4 x 3072 -> 10240 15.0 / 14.5; with
// one block of 16 channels to a workgroup 8 x 4608 -> 1280 11.0 / 11.2, 4 x 6144 -> 1280 9.5 / 9.5.  Where 8 would be 6, as three pieces make
// them, 12 walk over N faster unless two workgroups share the CU (6 / 12 waves): 5 x 1280 -> 12288 12.7 / 11.8, per token 13.4 / 12.3, 6 x
// 1536 -> 8192 10.2 / 9.8; one block of channels 6 x 1536 -> 4096 7.2 / 7.5.  Rows of four pieces take 16 from the fifth block of channels on (12
// / 16): 5 x 2048 -> 24576 21.1 / 19.6, per token 22.1 / 20.4, 6 x 1600 -> 24576 19.8 / 18.9; 8 x 2048 -> 12288 13.2 / 13.4.
int few_waves(int M, int N, int k_pad)
{
    const int pieces = (k_pad / 8 + 63) / 64, loads = few_loads((M + 15) / 16);
    if (pieces > 4 ? N > 16 * kFewGrid : pieces == 4 && M > kFewTwoM && N > 4 * 16 * kFewGrid) return kFewMaxWaves;
    const bool few = M * pieces <= 20 && !(pieces == 3 && M > kFewTwoM && N > 16 * kFewGrid);
    const int want = pieces > 4 ? 16 : few ? 8 : 12;
    int waves = max(want / pieces, 1) * pieces;
    while (waves * loads * 64 < k_pad) waves += pieces;
    return min(waves, kFewMaxWaves);
}

// Whether two workgroups share a CU where there are more blocks of 16 output channels than CUs (two of at most 8 waves do not hinder each
// other much while few rows' codes are to be formed): us a call, walking over N / so: 1 x 1600 -> 6400 9.1 / 8.0, 1 x 2048 -> 16384 15.6 / 12.1,
// 4 x 1024 -> 12288 11.4 / 9.8, 4 x 512 -> 8192 8.6 / 8.0; with 6 waves 1 x 1280 -> 5120 8.2 / 7.4, 4 x 1536 -> 12288 12.8 / 10.6; 8 x 512 -> 8192
// 8.5 / 8.8, 16 x 512 -> 8192 9.4 / 10.2.
bool few_two_on_a_cu(int M, int waves) { return M <= kFewTwoM && waves <= 8; }

// Most rows in turn (see few_tokens_fit) with the maxima given by the layer before.  The separate launches then are one less, and what
// they cost the host is hidden by that layer, so the line lies at fewer turns than without.  us of both layers of an MLP (the first one a
// quarter of the second's K wide), the second in separate launches / in this kernel (turns):
//   N <= 4096  32 x 512 -> 128 18.8 / 17.9 (3), 48 x 512 20.1 / 21.1 (4), 16 x 1024 -> 256 17.7 / 17.1 (3), 20 x 1024 18.3 / 18.4 (4), 16 x 1536 -> 384
//          17.8 / 17.3 (4), 20 x 1536 18.2 / 18.4 (5), 12 x 2048 -> 512 18.6 / 18.3 (4), 14 x 2048 18.7 / 18.8 (5); a longer K 10 x 3072 -> 768 18.7 / 18.3 (5),
//          12 x 3072 19.3 / 19.7 (6), 5 x 5120 -> 1280 21.7 / 20.9, 8 x 5120 21.9 / 22.7, 5 x 4608 -> 1152 21.4 / 21.1, 8 x 4608 22.0 / 23.0, 5 x 4608 -> 4096
//          22.1 / 22.5, 4 x 5120 -> 4096 21.3 / 21.2
//   per token  24 x 512 -> 128 19.5 / 19.0 (2), 12 x 1024 -> 256 18.5 / 18.2 (2), 16 x 1024 19.1 / 19.2 (3), 9 x 2048 -> 512 19.6 / 19.3 (3), 10 x 2048 19.9 /
//          19.9 (4), 8 x 3072 -> 768 20.0 / 19.8 (4), 9 x 3072 20.4 / 20.5 (5), 6 x 4096 -> 1024 20.0 / 19.7, -> 4096 20.6 / 21.1, 3 x 4608 -> 2560 21.5 /
//          21.0, 4 x 4608 22.2 / 22.4
//   beyond 24 x 512 -> 8192 18.9 / 18.8 (2), 32 x 512 19.2 / 19.3 (3), 12 x 1024 18.3 / 18.1 (2), 16 x 1024 18.5 / 18.7 (3), -> 5120 19.1 / 18.5, 6 x 1024 ->
//          12288 20.0 / 19.8 (1), 10 x 1024 20.7 / 20.9 (2), 5 x 2048 -> 8192 18.6 / 19.2 (2), two workgroups on a CU 4 x 2048 18.6 / 18.3; 4 x 3072 -> 8192
//          19.7 / 19.4 (2), 4 x 3072 -> 5120 19.1 / 19.3, 2 x 6400 -> 5120 24.5 / 25.2 (2), per token 3 x 4096 -> 8192 22.0 / 21.7, 4 x 4096 21.9 / 22.5 (2)
int given_turns(int M, int K, int N, int k_pad, int pieces, bool per_token)
{
    if (N > 4096) {
        if (few_two_on_a_cu(M, few_waves(M, N, k_pad))) return M;
        if (pieces <= 3) return pieces > 1 && N > 8192 ? 1 : per_token || N > 6400 ? 2 : 3;
        return pieces > 4 && N > 6400 && K <= 6144 && !(per_token && M * K > 12 * 1024) ? 2 : 1;
    }
    if (!per_token) return pieces <= 2 ? 3 : pieces > 4 && N <= 2560 ? 5 : 4;
    if (M * K > (N > 2560 ? 20 : 24) * 1024) return 0;
    return pieces <= 2 ? 2 : pieces > 4 && pieces <= 8 ? 4 : 3;
}

// Most rows in turn where a layer follows that takes the column maxima from this one, with more than one block of 16 output channels to a
// workgroup.  What the separate launches cost the host is hidden by that layer, which leaves the time of the kernels.  us of an MLP of widths K,
// 4 K, K, its second layer in separate launches, the first one in separate launches / in this kernel (turns):
//   N <= 5120  16 x 1040 23.0 / 22.2 (4), 13 x 1280 23.1 / 22.7 (4), 16 x 1280 23.4 / 23.0 (4)
//   beyond 13 x 1440 23.2 / 23.5 (4), 16 x 1520 23.5 / 24.1 (4), 10 x 1600 23.7 / 24.2 (4)
//   per token  9 x 1120 23.9 / 23.2 (3), 12 x 1120 24.0 / 23.9 (3), 9 x 1280 23.9 / 23.7 (3), 12 x 1280 24.0 / 24.2 (3), 16 x 1120 24.3 / 24.7 (4); beyond 6
//          x 1520 23.7 / 23.8 (2), 9 x 1440 24.0 / 24.3 (3), 16 x 1520 24.4 / 26.0 (4), four pieces 5 x 1600 24.2 / 24.6 (2), 9 x 1600 24.5 / 25.3 (3)
// (two rows in turn beyond N = 8192, and one with more than four pieces, are what ran before the line of calls by themselves went further.)
int handing_turns(int M, int K, int N, int k_pad, int pieces, bool per_token)
{
    if (pieces <= 2) return M;
    if (pieces > 4) return 1;
    if (!per_token) return N <= 5120 ? 4 : N <= 8192 ? 3 : 2;
    if (N <= 5120) return M * K <= 14 * 1024 ? 3 : 2;
    return pieces == 3 ? 2 : few_two_on_a_cu(M, few_waves(M, N, k_pad)) ? 2 : 1;
}

// X and its codes have to fit LDS together (about 42 K elements); below that the line against the separate
// launches (selecting quantiser and GEMM, two or three of them, which cost the host alone 9.8 us) lies where what grows here
// outweighs the launches saved: the rows that a wave works on one after the other (`turns`, counted for 12 waves and 16 whatever few_waves
// gives, so that a row more never brings a call back) and the elements in them, which every workgroup repeats, and the walk over N, 16
// channels per workgroup at a time with barriers between, from N = 4096 on.  us per call, the separate launches / this kernel (turns), with
// the maxima not given:
//   N <= 4096  18 x 2048 10.9 / 9.7, 30 x 1024 9.9 / 8.8, 60 x 512 9.9 / 9.2; from the ninth piece on the elements decide 8 x 4608 -> 2560 11.6 / 11.3,
//          7 x 4608 -> 4096 12.0 / 12.1, 8 x 4608 12.0 / 12.4, 8 x 5120 -> 4096 12.2 / 12.7, 4 x 8192 13.7 / 13.4
//   per token, whose maxima are one more walk over the rows  48 x 512 11.0 / 10.3 (4), 60 x 512 10.9 / 11.3 (5), 24 x 768 10.6 / 10.1 (4), 30 x 768 10.7 /
//          10.9 (5), 16 x 1536 10.7 / 10.4 (4), 15 x 2048 11.8 / 11.3 (5), 18 x 2048 11.6 / 12.4 (6), 12 x 2560 12.2 / 12.0 (4, 30 K elements), 15 x 2560
//          12.2 / 13.2, 10 x 3072 -> 2560 12.3 / 11.6 (5), 6 x 4096 -> 2560 11.7 / 11.3 (3), -> 4096 12.0 / 12.1, 8 x 4096 11.8 / 12.2; from the ninth piece on
//          5 x 4608 -> 2560 12.2 / 11.8, 6 x 4608 12.3 / 12.6, 3 x 4608 -> 4096 12.3 / 11.6, 4 x 4608 12.4 / 12.4, 4 x 8192 -> 768 13.6 / 12.6
//   to 12288, up to four pieces  36 x 768 -> 8192 12.4 / 11.0 (6), -> 12288 13.1 / 13.1, 12 x 1536 -> 12288 12.8 / 12.7 (3), 16 x 1536 12.9 / 13.1, 12 x 1600 ->
//          8192 11.2 / 10.8 (4), 15 x 1600 11.1 / 11.2, 9 x 1600 -> 12288 13.0 / 13.0 (3), 12 x 1600 13.2 / 13.4; per token 48 x 512 -> 8192 12.7 / 11.7
//          (4), 24 x 768 11.4 / 11.5 (4), 18 x 768 -> 12288 13.0 / 12.4 (3), 12 x 1536 -> 8192 11.9 / 11.8 (3), 16 x 1536 12.0 / 12.7, -> 5120 12.0 / 12.1, 8
//          x 1536 -> 12288 13.5 / 13.3 (2), 12 x 1536 13.7 / 14.2, 9 x 1600 -> 5120 11.5 / 11.2 (3), 12 x 1600 11.6 / 12.1, 6 x 2048 -> 8192 11.7 / 11.7 (2)
//   to 12288, more pieces  2 x 3072 -> 5120 11.0 / 11.2 (1), 4 x 3072 11.2 / 11.5, 4 x 4096 12.3 / 12.8: up to N = 6400 the GEMM does not fill the CUs and
//          this kernel walks two steps all the same; 9 x 2560 -> 8192 12.4 / 12.1 (3), 12 x 2560 12.4 / 12.6, 3 x 4608 13.7 / 13.7 (3), 4 x 4608 13.9 / 14.1,
//          3 x 5120 -> 12288 18.6 / 18.2 (3), 2 x 8192 -> 8192 17.7 / 17.6 (2); per token 2 x 3072 12.7 / 12.1 (1), 4 x 3072 12.7 / 12.8, 2 x 5120 15.1 /
//          14.7 (2), 3 x 5120 15.1 / 15.4, 1 x 6400 16.5 / 15.8, 2 x 6400 16.4 / 16.7
//   to 16384, where the GEMM still has direct tiles and this kernel takes a step more  3 x 2560 15.4 / 16.7, 5 x 1024 12.6 / 13.1, 5 x 2048 14.2 /
//          15.8, but 8 x 512 12.1 / 10.8; two workgroups on a CU 4 x 2048 14.1 / 12.7
//   beyond, where it has not  8 x 4096 -> 24576 38.1 / 32.9, 10 x 4096 38.3 / 33.4, 12 x 3072 26.9 / 25.1, 12 x 2560 -> 20480 23.7 / 20.9, per token 9 x 2560
//          -> 24576 24.8 / 24.2, 12 x 2560 24.9 / 25.3 (4); four pieces 9 x 2048 -> 24576 21.5 / 20.3 (3), per token 22.6 / 21.4, 9 x 1600 19.3 / 19.4
// Long lists move it the other way (8 x 1280 -> 4096, 160 channels of at most 1024 listed, 19.6 / 11.0 with the separate launches of
// before): capacities above 64 keep wider lines.
bool few_tokens_fit(int M, int K, int N, int k_pad, int r_cap, bool per_token, bool maxima_given, bool hands_maxima)
{
    if (M > kFewMaxM || k_pad > 64 * kFewMaxWaves * few_loads((M + 15) / 16) || few_plan(M, K, k_pad, r_cap, 1, kFewMaxWaves).total > kFewLdsBytes)
        return false;
    const bool fewest = M <= 8, long_lists = r_cap > 64;
    if (N > (M > 32 ? 8192 : K > 1536 ? (fewest && K > 3072 ? 32768 : 24576) : fewest ? 16384 : 12288)) return false;
    if (!long_lists) {
        const int pieces = (k_pad / 8 + 63) / 64, at_once = max((pieces > 4 ? 16 : 12) / pieces, 1), turns = (M + at_once - 1) / at_once;
        if (N > 12288) {
            if (pieces > 4) return N > 16384 && !(per_token && pieces == 5 && turns > 3);
            return pieces == 1 || few_two_on_a_cu(M, few_waves(M, N, k_pad)) || (pieces == 4 && N > 16384 && turns <= 3);
        }
        if (maxima_given) {
            if (turns > given_turns(M, K, N, k_pad, pieces, per_token)) return false;
            if (N > 4096) return true;
        } else if (N > 4096) {
            if (hands_maxima && turns > handing_turns(M, K, N, k_pad, pieces, per_token)) return false;
            if (pieces > 4) return turns <= (N <= 6400 ? 1 : per_token ? 1 + (pieces > 8 && K <= 6144) : 3 - (K > 6144));
            const int most = !per_token ? (pieces <= 2 ? 6 : N <= 8192 || pieces == 3 ? 4 : 3)
                           : pieces <= 2 ? 4 - (N > 8192) : pieces == 3 ? 4 - (N > 6400) - (N > 8192) : 3 - (N > 6400);
            return turns <= most && M * K <= 24 * 1024;
        } else if (!per_token) {
            if (pieces > 8 && M * K > 34 * 1024 && N > 2560) return false;
        } else if (pieces > 8) {
            if (N > 2560 ? turns > 3 : M * K > 26 * 1024 && (N > 1536 || turns > 4)) return false;
        } else if (turns > (pieces <= 3 ? 4 : pieces <= 6 ? 5 : 3) || M * K > 31 * 1024) {
            if (pieces <= 3 || M * K > 26 * 1024 || (pieces > 6 && N > 2560)) return false;
        }
    }
    if (M <= 20) return true;
    if (M <= 32) return M * K <= (M <= 24 ? 36 : 32) * 1024;
    return K <= 512 ? M <= (per_token ? 48 : 64) : M <= 40 && M * K <= 32 * 1024 && !per_token;
}

typedef void (*few_kernel_t)(const FewArgs, const FewPlan);
static few_kernel_t few_kernel(int row_blocks, bool token)
{
    switch (row_blocks) {
    case 1: return token ? k_linear_few<1, true> : k_linear_few<1, false>;
    case 2: return token ? k_linear_few<2, true> : k_linear_few<2, false>;
    default: return token ? k_linear_few<4, true> : k_linear_few<4, false>;
    }
}

hipError_t few_prepare_device()
{
    for (int i = 0; i < 6; ++i) {
        const hipError_t e = hipFuncSetAttribute((const void *)few_kernel(1 + i / 2, i % 2 != 0),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kFewLdsBytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_linear_few(const FewArgs &a, hipStream_t s)
{
    const hipError_t e = gemm_prepare_device();
    if (e != hipSuccess) return e;
    // every workgroup repeats the activation side: no more of them than are resident at once
    const int nblk = (a.N + 15) / 16, waves = few_waves(a.M, a.N, a.k_pad), grid = min(nblk, few_two_on_a_cu(a.M, waves) ? 2 * kFewGrid : kFewGrid);
    FewPlan plan = few_plan(a.M, a.K, a.k_pad, a.r_cap, grid, waves);
    plan.cut = a.static_mask != nullptr ? 0 : magnitude_cut(a.threshold);
    return launch_kernel(few_kernel((a.M + 15) / 16, a.x_per_token != 0), dim3(grid), dim3(plan.waves * 64), plan.total, s,
                         a, plan);
}

}  // namespace muxq
