// INT8 x INT8 -> INT32 MFMA GEMM of the MUXQ linear layer for gfx950, with the
// Aux product, the (2^exp - 1) recombination (Eq. 7) and the dequantising
// epilogue (Eq. 3) fused in.
//
// Orientation.  Both operands are stored K-contiguous: activations a_q[m][k]
// and the packed weight w_q[n][k].  The MFMA computes D = A.B with A = a
// 32(n) x 32(k) block of the weight and B = a 32(k) x 32(m) block of the
// activations, i.e. the tile of Y transposed.  In the 32x32 accumulator layout
// each lane then owns ONE token m and runs of 4 consecutive output channels
// n, which are contiguous in row-major Y: the epilogue stores 8-byte fp16x4
// packets without any shuffle.
//
// K loop.  The Aux product is simply a few extra K tiles placed FIRST: the
// accumulators after the Aux tiles hold acc_aux; they are multiplied once by
// c = 2^exp - 1 and the Body tiles are then accumulated on top, which gives
// acc_body + c * acc_aux in exact integer arithmetic with one set of
// accumulators.  The number of Aux tiles is read from device memory
// (n_outliers[0]) so no host synchronisation is needed.
//
// Power.  Under INT8 MFMA load the chip is power-limited, and what the matrix pipes
// draw depends on how much their operands toggle.  Two things keep that down without
// changing any result: the activation codes of the unlisted channels come with a
// zero point (non-negative; the epilogue takes z * cn[n] off the accumulators), and
// the accumulators start at a positive offset instead of 0, so that they do not keep
// changing sign (see kCnBias / kAccBias; the Aux weighting lets the offset pass
// through, the epilogue removes it).  The weights are the first MFMA operand and the
// narrow activation codes the second: the other way round draws more.
//
// Four kernels share that scheme:
//   k_gemm_i8_persist8  256 x 256 tile, 8 waves (2 per SIMD), K step 64, one
//                   persistent workgroup per CU.  Operand tiles go global -> LDS
//                   directly (buffer_load_dwordx4 ... lds, no staging registers)
//                   into a ring of LDS stages, two K steps ahead; fragments are
//                   double-buffered in registers so ds_read_b128 of the next K
//                   sub-step overlaps the MFMAs of the current one; one
//                   workgroup barrier per K step, placed between the two
//                   sub-steps so that it never waits on data.
//   k_gemm_i8_persist4  the same kernel body with a 128 x 128 tile and 4 waves,
//                   two workgroups per CU, where its rounds of tiles are fewer
//                   than three times those of the 256 x 256 form (gemm_form).
//   k_gemm_i8_persist_half  the same with a 128 (n) x 256 (m) tile and 4 waves, two workgroups per
//                   CU, each with its own barriers: one computes under the other's epilogue.
//   k_gemm_i8_direct  small tiles (16 x 16 to 64 x 64), operands from memory straight to
//                   registers, the waves of a workgroup split K: for problems
//                   with too few larger tiles to fill the chip.
//
// LDS rows are 64 bytes (one K step); the four 16-byte chunks of a row are
// XOR-swizzled with row bits so that a ds_read_b128 of 32 rows x one chunk is
// spread over all banks without padding (a direct-to-LDS load needs the LDS
// image of a wave to be contiguous, so padding is not an option; the swizzle
// is applied on the global-address side instead).
//
// Workgroup -> tile map.  Workgroups are dealt round-robin to the 8 XCDs, each
// with its own L2; workgroup i belongs to XCD i % 8.  Tiles are grouped in blocks
// of sup_m x sup_n, as many as an XCD works on at one time, so that its L2 holds
// sup_m + sup_n operand panels for sup_m * sup_n tiles.  Blocks are dealt to the
// XCDs in turn, one to each where there are no more tiles than CUs; where ragged
// blocks would make that take more rounds than the number of tiles needs, the
// tiles are instead put in one order, block after block, and split evenly.
#include "muxq_kernels.h"

#include <atomic>
#include <mutex>

// Compiled four times, as device binaries that are loaded when the first of their kernels is used: this file with the usual
// kernels, and muxq_gemm_own.hip, _gelu.hip and _codes.hip, which include it, with those of part_of.  (All in one binary
// loading the library took 2.9 ms and a program's first call 10 ms, with 200 kernels; so 1.1 and 3.7 ms, with 210.)
#ifndef MUXQ_GEMM_PART
#define MUXQ_GEMM_PART 0
#endif

namespace muxq {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 64;   // K step (bytes of one LDS row)

struct TileMap {
    int tiles_m, tiles_n, sup_m, sup_n;
    int at_once;          // even split: tiles an XCD works on at a time; 0: blocks dealt in turn
    int n_super, super_n; // blocks, and blocks per row of blocks
    int full, rest;       // even split: full rounds, tiles of the last one
    Divisor by_block, by_sup_n, by_super_n, by_at_once, by_band, by_band_block, by_last_band_block, by_last_cols;
    // by_block: sup_m sup_n; by_band: sup_m tiles_n; by_band_block: rows of a band x sup_n; `last`: the
    // last, ragged band of rows or block of columns
};

// 16-byte chunk position of logical chunk `chunk` in LDS row `row`.
template <int SWZ>
__device__ __forceinline__ int swizzle(int row, int chunk)
{
    if constexpr (SWZ == 0)
        return chunk ^ ((row >> 1) & 3);
    else if constexpr (SWZ == 1)
        return chunk ^ ((row >> 2) & 3);
    else if constexpr (SWZ == 2)
        return chunk ^ (row & 3);
    else
        return chunk;
}

// Brings all cache lines of the kernel's arguments in at once.  The tile map reads its fields behind
// branches, and each first touch of a 64-byte line of arguments is a round trip to memory
// (24 x 5120 -> 1280 4.84 -> 4.65 us, 512 x 1024 -> 1024 5.60 -> 5.39 us; the persistent forms have no use for it).
__device__ __forceinline__ void fetch_arguments()
{
    constexpr int LINES = (sizeof(GemmArgs) + sizeof(TileMap) + 63) / 64;
    static_assert(LINES == 5, "one operand below for each line");
    const __attribute__((address_space(4))) int *const p =
        (const __attribute__((address_space(4))) int *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" ::"s"(p[0]), "s"(p[16]), "s"(p[32]), "s"(p[48]), "s"(p[64]));
}

// Tile j of the share of XCD `xcd`: 1, or 0 past the end of the share, or -1 where a ragged block has
// no tile (j + 1 may have one).
// (12288 x 1280 -> 1280 is 240 tiles for 256 CUs; dealt as blocks of 4 x 5 tiles, half of the XCDs had
// two rounds, 39 us, split evenly one, 23 us.  Where both take the same number of rounds whole blocks
// are better: 16384 x 1280 -> 3840 84 us, split evenly 87-90 us.)
__device__ __forceinline__ int tile_of_share(const TileMap &tm, int xcd, int j, int &tile_m, int &tile_n)
{
    if (tm.at_once == 0) {
        const int r = quotient(j, tm.by_block), in_block = j - r * tm.sup_m * tm.sup_n, st = r * 8 + xcd;
        if (st >= tm.n_super) return 0;
        const int row = quotient(in_block, tm.by_sup_n), bm = quotient(st, tm.by_super_n);
        tile_m = bm * tm.sup_m + row;
        tile_n = (st - bm * tm.super_n) * tm.sup_n + in_block - row * tm.sup_n;
        return tile_m < tm.tiles_m && tile_n < tm.tiles_n ? 1 : -1;
    }
    const int r = quotient(j, tm.by_at_once);
    int idx;
    if (r < tm.full) {
        idx = (r * 8 + xcd) * tm.at_once + (j - r * tm.at_once);
    } else {
        const int jr = j - tm.full * tm.at_once;
        if (jr >= tm.rest / 8 + (xcd < tm.rest % 8 ? 1 : 0)) return 0;
        idx = tm.full * 8 * tm.at_once + tm.rest / 8 * xcd + min(tm.rest % 8, xcd) + jr;
    }
    const int band = quotient(idx, tm.by_band), in_band = idx - band * tm.sup_m * tm.tiles_n;
    const bool last = (band + 1) * tm.sup_m > tm.tiles_m;
    const int rows = last ? tm.tiles_m - band * tm.sup_m : tm.sup_m;
    const int block = last ? quotient(in_band, tm.by_last_band_block) : quotient(in_band, tm.by_band_block);
    const int in_block = in_band - block * rows * tm.sup_n;
    const bool last_cols = (block + 1) * tm.sup_n > tm.tiles_n;
    const int cols = last_cols ? tm.tiles_n - block * tm.sup_n : tm.sup_n;
    const int row = last_cols ? quotient(in_block, tm.by_last_cols) : quotient(in_block, tm.by_sup_n);
    tile_m = band * tm.sup_m + row;
    tile_n = block * tm.sup_n + in_block - row * cols;
    return 1;
}

__device__ __forceinline__ bool tile_of_workgroup(const TileMap &tm, int &tile_m, int &tile_n)
{
    return tile_of_share(tm, (int)blockIdx.x & 7, (int)blockIdx.x >> 3, tile_m, tile_n) > 0;
}

// acc <- c * acc with c = 2^e - 1, as (acc << e) - acc (two full-rate VALU ops).  The
// accumulators start at an offset B (see kCnBias) that is to come through unscaled:
// c * (acc - B) + B = c * acc - fix with fix = (c - 1) * B.
template <int FN, int FM>
__device__ __forceinline__ void scale_acc(v16i (&acc)[FN][FM], int e, int fix)
{
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
        {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[fn][fm][v] = (int)(((unsigned)acc[fn][fm][v] << e) + (0u - (unsigned)fix - (unsigned)acc[fn][fm][v]));
            // one fragment at a time: keeps the number of temporaries small when the
            // accumulators live in the accumulation registers
            __builtin_amdgcn_sched_barrier(0);
        }
}

// The same step when Aux was quantised on a scale of its own (s_aux, the other reading of
// Eq. 5): the Aux accumulators are brought onto Body's scale, acc <- rne(rho * acc) with
// rho = (2^e - 1) s_aux / s_x <= 2^e - 1, and the Body steps then accumulate on top as before.
// Against the sum of Eq. 7 taken after dequantisation this rounds the Aux term to a whole
// unit of s_x s_w[n]: at most half such a unit of error per output.
template <int FN, int FM>
__device__ __forceinline__ void scale_acc_rho(v16i (&acc)[FN][FM], float rho, int bias)
{
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
        {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[fn][fm][v] = (int)__builtin_rintf(rho * (float)(acc[fn][fm][v] - bias)) + bias;
            __builtin_amdgcn_sched_barrier(0);
        }
}

// The same with one activation scale per token: a lane's accumulators of fragment column fm
// belong to one token, whose factor rho[fm] the row quantiser left behind the token scales.
template <int FN, int FM>
__device__ __forceinline__ void scale_acc_rho_tok(v16i (&acc)[FN][FM], const float (&rho)[FM], int bias)
{
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
        {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[fn][fm][v] = (int)__builtin_rintf(rho[fm] * (float)(acc[fn][fm][v] - bias)) + bias;
            __builtin_amdgcn_sched_barrier(0);
        }
}

// Where the per-token factors rho[m] = (2^e - 1) s_aux[m] / s_x[m] of such a launch are:
// the fifth array of x_scale (after s_x[M], qmax / max|Body[m]|, z[m], s_aux[M]).
__device__ __forceinline__ const float *aux_rho_tok(const GemmArgs &a) { return a.x_scale + 4 * (size_t)a.M; }

// (2^e - 1) s_aux / s_x of a launch whose Aux codes have their own scale, else 0.
__device__ __forceinline__ float aux_rho(const GemmArgs &a)
{
    if (!a.aux_own_scale || a.x_per_token) return 0.f;
    const float sx = a.x_scale[0], sa = a.x_scale[2];
    return sx > 0.f ? ((float)((1 << a.exp_shift) - 1) * sa) / sx : 0.f;
}

// Whether Y goes out as a stream.  Rows on 128-byte lines: a store instruction writes whole lines, and Y, which
// is not read here again, stays out of the operands' way in L2 (16384 x 1280 -> 3840 90 us through L2, 87 us as a
// stream).  Rows on 64-byte boundaries: whole transfers still, but half lines, which L2 would join.  That is worth
// more while the memory-side cache takes Y in, and less once it does not, or while the L2s themselves hold it (768
// input channels, us through L2 / as a stream: 1000 -> 20000 24.5 / 22.5, 2000 -> 20000 43 / 47, 12000 -> 20000
// 250 / 202).  Other rows: the transfers at the ends of a piece are completed by the neighbouring piece, which only
// happens in L2 (3001 -> 4808 19 / 27, 12000 -> 10000 111 / 145).
__host__ __device__ __forceinline__ bool stream_rows(const GemmArgs &a)
{
    const uintptr_t start = (uintptr_t)a.y | (uintptr_t)a.ldy * 2;
    const size_t mib = ((size_t)a.M * a.N * 2) >> 20;
    return start % 128 == 0 || (start % 64 == 0 && (mib < 48 || mib >= 256));
}

// How a persistent kernel stores Y: through L2 or as a stream half of a wave's channels at a time, or through L2 with
// all pieces of a row one after the other, so that L2 still has a line that two of them share when the second comes.  The last
// pays where Y is more than the L2s hold, 32 MiB (us a call, by halves / together: 11330 x 448 -> 14296 186 / 148, 13653 x 520 ->
// 10608 174 / 148, 4837 x 1600 -> 10168 113 / 104, 8811 x 776 -> 5264 72.5 / 71.0); below, the first stores come too late
// (11873 x 312 -> 680 30.3 / 31.3, 14185 x 120 -> 520 23.7 / 24.1, but 3001 x 1592 -> 4808 43.0 / 42.1).  Not in the 128 x 128
// tiles, whose waves have one piece of a row, nor with the GELU, whose work per output is twice as much (11608 x 760 -> 5368 105.0 /
// 108.9, 5239 x 1728 -> 7224 100.3 / 98.4).
enum Store { kStoreL2, kStoreStream, kStoreTogether, kStores };

// 16 bytes of Y.  STREAM: non-temporal (chosen by stream_rows).  Compile time: a branch at each store costs
// 1 us per tile.
template <bool STREAM>
__device__ __forceinline__ void store_y(const GemmArgs &a, int m, int n, v4i v)
{
    v4i *const dst = (v4i *)(a.y + (size_t)m * a.ldy + n);
    if (STREAM)
        __builtin_nontemporal_store(v, dst);
    else
        *dst = v;
}

// Eq. 3: Y = fp16((s_x * s_w[n]) * float(acc) + bias[n]).  Lane layout of the
// 32x32 accumulator: token m = lane % 32, output channels
// n = 8 * (v / 4) + 4 * (lane / 32) + v % 4 for register v of 16, so a lane holds
// runs of 4 channels of ONE token: stored directly, a wave instruction would
// touch 32 rows of Y with 16 bytes each.  Instead each wave transposes its
// fp16 results through a private LDS patch, 32 tokens at a time, whose row padding
// of 16 B spreads the 8-byte writes of the 32 tokens over the banks.
//
// Epilogue of the persistent kernels: the wave's LDS patch
// holds 32 tokens x 64 channels (two fragments), so a tile's epilogue runs
// FM x FN/2 rounds of { 8 ds_write_b64, 4 ds_read_b128, 4 stores of 8 rows x 128 B }.
// Exactly FM * (FN / 2) * 4 store instructions are issued for a tile, partial or not.
// Bound by its vector ALU work and by the latency of reading the constants: a group of 4 channels is read once
// for the FM tokens of a lane, one group ahead, and the later token's results stay in the registers of the
// accumulators they replace until the patch is free.
// The vector-memory counter completes in issue order, so a vector load issued
// here would have to wait for every operand load still in flight.  So the wave's constants come straight into
// `chan` (LDS) by direct-to-LDS loads issued with the tile's first K step (raw values: FN * 32 weight scales, then
// FN * 32 fp16 bias values, then FM * 32 token scales, the channels' cn, the tokens' z and rho), and what a launch
// has of them is known at compile time (Epi): a run-time flag costs a select or an add of zero per output, and this
// epilogue is bound by its vector ALU work (seven operations per output in the per-vector setting).  One kernel for
// each, chosen on the host: with eleven epilogues behind one K loop the compiler left no vector registers for reading the
// constants ahead.  (It still spills 30 to 190 scalar registers, 190 to 260 then; with the tile map read anew for each tile it is 30
// to 70, and 13 shapes stay within 0.7 %, so those cost nothing that can be measured.)
// (one kernel each and the reads ahead, us a call: 1024 x 768 -> 3072 19.9 -> 18.1, 8192 x 1024 -> 1024 30.5 -> 28.0, 3001 x
// 1592 -> 4808 per vector 43.3 -> 41.6, 16384 x 1280 -> 3840 per vector 113.3 -> 108.4, 8192 x 4096 -> 16384 428 -> 422)
enum Epi {
    kEpiAny,          // flags at run time; exports the raw accumulators when asked (debugging; drains the memory queue
                      // once per tile) and takes any row stride of Y
    kEpiGeneral,      // flags at run time
    kEpiPlain, kEpiBias, kEpiChan, kEpiChanBias,          // one activation scale, no zero point (muxq_gemm_i8)
    kEpiPlainZ, kEpiBiasZ, kEpiChanZ, kEpiChanBiasZ,      // one activation scale, zero point
    kEpiToken, kEpiTokenBias,                             // scales per token, zero points per token
    kEpiVector, kEpiVectorBias,                           // the same with a scale per channel as well
    kEpis
};
constexpr int kChanFloats = 128 + 64 + 64 + 128 + 64 + 64;   // per-wave LDS for the tile's constants

// kEpiAny: the rows m + p * 8 + lane / 8 of Y from channel n on.  A buffer for the 8 rows of each store, whose offsets reach
// rows 2^28 elements apart; by address beyond.  (512 x 2048 -> 16384 with rows 2^25 elements apart: by address 36.2 us, so
// 32.0.)
constexpr int kBufferLdy = (1 << 28) - 64;
__device__ __forceinline__ void put_any(const GemmArgs &a, const v4i (&v)[4], int m, int n, int lane)
{
    constexpr unsigned PAST = 0xfffffc00u;
    static_assert((unsigned)kBufferLdy * 16u <= PAST, "the range check drops what is past the buffer");
    const bool stream = stream_rows(a);
    if (a.ldy <= kBufferLdy) {
        const unsigned off = n < a.N ? (unsigned)(lane >> 3) * (unsigned)a.ldy * 2u + (unsigned)n * 2u : PAST;
        const auto buffer = [&](int p) {
            return __builtin_amdgcn_make_buffer_rsrc((void *)(a.y + (size_t)(m + p * 8) * a.ldy), 0,
                                                     (int)((unsigned)min(max(a.M - m - p * 8, 0), 8) * (unsigned)a.ldy * 2u), 0x00020000);
        };
        if (stream) {
#pragma unroll
            for (int p = 0; p < 4; ++p) __builtin_amdgcn_raw_buffer_store_b128(v[p], buffer(p), off, 0, 2);
        } else {
#pragma unroll
            for (int p = 0; p < 4; ++p) __builtin_amdgcn_raw_buffer_store_b128(v[p], buffer(p), off, 0, 0);
        }
    } else {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int row = m + p * 8 + (lane >> 3);
            if (n < a.N && row < a.M) {
                if (stream) store_y<true>(a, row, n, v[p]);
                else store_y<false>(a, row, n, v[p]);
            }
        }
    }
}

// -1: decided at run time from the arguments
constexpr bool epi_flags(int e) { return e <= kEpiGeneral; }
constexpr int epi_chan(int e)
{
    return epi_flags(e) ? -1 : e == kEpiChan || e == kEpiChanBias || e == kEpiChanZ || e == kEpiChanBiasZ || e >= kEpiVector;
}
constexpr int epi_bias(int e)
{
    return epi_flags(e) ? -1 : e == kEpiBias || e == kEpiChanBias || e == kEpiBiasZ || e == kEpiChanBiasZ || e == kEpiTokenBias ||
                                   e == kEpiVectorBias;
}
constexpr int epi_token(int e) { return epi_flags(e) ? -1 : e >= kEpiToken; }
constexpr int epi_zero(int e) { return epi_flags(e) ? -1 : e >= kEpiPlainZ; }
// Whether the accumulators of a launch with the zero point 0 start at kAccBias all the same.  Not in the 128 x 128 tiles: there
// it gains 1 % without outliers (8192 x 1024 -> 1024 27.8 / 27.6 us), and the branch costs the other calls 1 to 2.5 %
// (with outliers, a scale per channel: 1024 x 768 -> 3072 19.0 / 19.5, 8192 x 1024 -> 1024 30.1 / 30.4).
constexpr bool z_offset(int fn) { return fn == 4; }

// The accumulators carry a zero-point term z * cn[n] (cn per channel, int32; z per launch or per token), which is
// taken off in integers (one 24-bit multiply-add), so the result is the accumulator of Eq. 7 exactly; `sub_bias`
// (see kAccBias) comes off as well, and is known to be zero with one zero point per launch (0 among them: z_none).
// GELU (compile time): the result goes through the tanh GELU, applied to the fp16 value the
// layer would have stored, and `mx` (FN / 2 entries) collects, per lane, the running maxima of
// the |fp16| values the lane stores (its 8 channels of each half, over its rows).
template <int FN, int FM, int ROW_BYTES, int EPI, int STORE, bool GELU>
__device__ __forceinline__ void epilogue_patch(const GemmArgs &a, const v16i (&acc)[FN][FM],
                                               int m_base, int n_base, int lane,
                                               unsigned char *patch, float *chan, float sx,
                                               float sw0, int z_launch, int sub_bias, uint4 *mx)
{
    constexpr int WCH = epi_chan(EPI), TOK = epi_token(EPI), BIAS = epi_bias(EPI), ZC = epi_zero(EPI);
    const bool w_chan = WCH < 0 ? a.w_per_channel != 0 : WCH != 0;
    const bool x_tok = TOK < 0 ? a.x_per_token != 0 : TOK != 0;
    const bool has_zc = ZC < 0 ? a.cn != nullptr : ZC != 0;
    if (ZC == 1 && TOK == 0) sub_bias = 0;
    const float s_tensor = sx * sw0;
    static_assert((FN == 4 || FN == 2) && FM == 2, "the constants' layout holds up to 128 channels and 64 tokens per wave");
    // (what follows from the lane number is worked out anew for each tile: kept through the K loop it would spill)
    asm volatile("" : "+v"(lane));
    const int fr = lane & 31, fh = lane >> 5;
    _Float16 *const chan_bias = (_Float16 *)(chan + 128);
    float *const chan_tok = chan + 128 + 64;
    int *const chan_zc = (int *)(chan + 256);      // cn of the wave's 128 channels
    int *const chan_ztok = (int *)(chan + 384);    // z of the wave's 64 tokens (per-token setting)
    // One zero point for the launch and that is 0: the accumulators started at kAccBias, which comes off in the place of
    // z * cn[n], as 1 * kAccBias.
    const bool z_none = z_offset(FN) && has_zc && !x_tok && z_launch == 0;
    if (z_none) chan_zc[lane] = chan_zc[64 + lane] = kAccBias;
    int negz[FM];                                  // this lane's tokens
    float sxt[FM];
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) {
        negz[fm] = !has_zc ? 0 : x_tok ? -chan_ztok[fm * 32 + fr] : z_none ? -1 : -z_launch;
        sxt[fm] = x_tok ? chan_tok[fm * 32 + fr] : sx;
    }
    // Y of the wave's rows of one fragment, as a buffer that ends with row M - 1: a store needs one 32-bit add, and
    // rows past M are dropped by the range check.
    const int piece = lane & 7;
    unsigned y_off[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) y_off[p] = (unsigned)(p * 8 + (lane >> 3)) * (unsigned)a.ldy * 2u + (unsigned)(n_base + piece * 8) * 2u;
    // constants of the 4 channels of group e (fragment e / 4, run e % 4), read one group ahead of their use
    struct Group { float4 w; f16x4 b; v4i z; };
    const auto group = [&](int e) {
        const int at = e * 8 + 4 * fh;
        Group c;
        c.w = make_float4(sw0, sw0, sw0, sw0);
        c.b = f16x4{0, 0, 0, 0};
        c.z = v4i{0, 0, 0, 0};
        // (with flags: what the launch has not was loaded as zeros)
        if (WCH < 0) {
            const float4 w = *(const float4 *)(chan + at);
            if (w_chan) c.w = w;
        } else if (WCH != 0) c.w = *(const float4 *)(chan + at);
        if (BIAS != 0) c.b = *(const f16x4 *)(chan_bias + at);
        if (ZC != 0) c.z = *(const v4i *)(chan_zc + at);
        return c;
    };
    // Raw accumulators, debugging aid: plain per-lane stores.  Before the results, which go into the accumulators' registers
    // (behind them both were held, 38 to 102 registers spilled: 8192 x 2048 -> 8192 311 us, so 206).
    if (EPI == kEpiAny && !GELU && a.dbg_acc != nullptr) {
#pragma unroll
        for (int e = 0; e < FN * 4; ++e) {
            const int n = n_base + e * 8 + 4 * fh;
            const v4i z = group(e).z;
#pragma unroll
            for (int fm = 0; fm < FM; ++fm) {
                const int m = m_base + fm * 32 + fr;
                v4i raw;
#pragma unroll
                for (int i = 0; i < 4; ++i) raw[i] = __mul24(z[i], negz[fm]) + acc[e / 4][fm][4 * (e % 4) + i] - sub_bias;
                if (n < a.N && m < a.M) *(v4i *)(a.dbg_acc + (size_t)m * a.N + n) = raw;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    Group cst = group(0);
    // patch -> Y: 8 lanes cover the 128 bytes of one token, 8 tokens per instruction
    const auto put = [&](int h, int fm) {
        // (no branch at a store: lanes past N get an offset past the end)
        const bool n_in = n_base + h * 64 + piece * 8 < a.N;
        unsigned off[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) off[p] = n_in ? y_off[p] + h * 128 : 1u << 31;
        const int rows = __builtin_amdgcn_readfirstlane(min(max(a.M - m_base - fm * 32, 0), 32));
        const __amdgpu_buffer_rsrc_t r_y = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(a.y + (size_t)(m_base + fm * 32) * a.ldy), 0, (int)((unsigned)rows * (unsigned)a.ldy * 2u), 0x00020000);
        v4i v[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int row = p * 8 + (lane >> 3);
            v[p] = *(const v4i *)(patch + row * ROW_BYTES + piece * 16);
            if (EPI != kEpiAny) __builtin_amdgcn_raw_buffer_store_b128(v[p], r_y, off[p], 0, STORE == kStoreStream ? 2 : 0);
            if (GELU) {
                const unsigned keep = n_in && row < rows ? ~0u : 0u;
                const uint4 u = __builtin_bit_cast(uint4, v[p]);
                mx[h] = absmax_step(mx[h], make_uint4(u.x & keep, u.y & keep, u.z & keep, u.w & keep));
            }
        }
        if (EPI == kEpiAny) put_any(a, v, m_base + fm * 32, n_base + h * 64 + piece * 8, lane);
    };
    // Results that wait for the patch, in the registers of accumulators that are done with: kStoreTogether those of all
    // pieces, which then go out one after the other, else those of half of the channels.
    constexpr bool TOGETHER = STORE == kStoreTogether;
    f16x4 held[FN / 2][FM][8];
#pragma unroll
    for (int h = 0; h < FN / 2; ++h) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const Group nxt = h * 8 + e + 1 < FN * 4 ? group(h * 8 + e + 1) : cst;
            const int fn = 2 * h + e / 4, g = e % 4;
            const float wv[4] = {cst.w.x, cst.w.y, cst.w.z, cst.w.w};
#pragma unroll
            for (int fm = 0; fm < FM; ++fm) {
                f16x4 out;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // Eq. 3: one binary32 product of the two scales, whichever granularity
                    const float sc = WCH == 0 && TOK == 0 ? s_tensor : sxt[fm] * wv[i];
                    int t = acc[fn][fm][4 * g + i];
                    if (ZC != 0) t = __mul24(cst.z[i], negz[fm]) + t;
                    float y = sc * (float)(t - sub_bias);
                    if (BIAS != 0) y = y + (float)cst.b[i];   // + 0 without a bias: changes no finite value
                    // The product is a binary32 value: without a bias and before the GELU the compiler folded it and the
                    // conversion into one mixed-precision instruction with a single rounding.  (With flags it took the
                    // conversions out of their groups and spilled 20 to 47 registers.)
                    if (epi_flags(EPI) || (GELU && BIAS == 0)) asm volatile("" : "+v"(y));
                    out[i] = (_Float16)y;
                    if (GELU) out[i] = (_Float16)gelu_tanh_f32((float)out[i]);
                }
                if (fm == 0 && (!TOGETHER || h == 0)) *(f16x4 *)(patch + fr * ROW_BYTES + (e * 8 + 4 * fh) * 2) = out;
                else held[h][fm][e] = out;
            }
            cst = nxt;
            __builtin_amdgcn_sched_barrier(0);     // bounds the live temporaries (see scale_acc)
        }
        if (!TOGETHER) {
#pragma unroll
            for (int fm = 0; fm < FM; ++fm) {
                if (fm > 0) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) *(f16x4 *)(patch + fr * ROW_BYTES + (e * 8 + 4 * fh) * 2) = held[h][fm][e];
                }
                put(h, fm);
            }
        }
    }
    if (TOGETHER) {
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int h = 0; h < FN / 2; ++h) {
                if (fm + h > 0) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) *(f16x4 *)(patch + fr * ROW_BYTES + (e * 8 + 4 * fh) * 2) = held[h][fm][e];
                }
                put(h, fm);
            }
    }
}

__device__ __forceinline__ int aux_tiles(const GemmArgs &a)
{
    int used = 0;
    if (a.n_outliers != nullptr && a.r_cap > 0) used = max(0, min(a.n_outliers[0], a.r_cap));
    used = __builtin_amdgcn_readfirstlane(used);
    return (used + BK - 1) / BK;
}

// s_waitcnt that only constrains vmcnt (gfx9 encoding: vmcnt[3:0] | expcnt[6:4]
// | lgkmcnt[11:8] | vmcnt[5:4] << 14).
constexpr int waitcnt_vm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }
// ... and additionally waits for every LDS access of this wave (lgkmcnt = 0).
constexpr int waitcnt_vm_lds(int n) { return (n & 15) | (7 << 4) | (0 << 8) | ((n >> 4) << 14); }
constexpr int waitcnt_lds_only() { return waitcnt_vm_lds(63); }

// --------------------------------------------------------------------------
// Persistent form of the 256 x 256 kernel: one workgroup per CU walks a list of
// tiles, and the K steps of all its tiles form ONE continuous stream through
// the LDS ring.  The operand loads of the next tile's first K steps are issued
// during the last K steps of the current tile, so there is no load latency at
// tile boundaries, and the stores of a tile's epilogue drain while the next
// tile is already being computed.  The epilogue's LDS patches lie behind the
// ring, so the ring keeps filling during an epilogue (or, OVERLAY, in the one stage
// that nothing is loaded into meanwhile).
//
// The DMA instructions of a K step (four, in the 256 x 256 form) are spread over the first eight MFMAs
// (one per two MFMAs) instead of being issued back to back: a burst of 32 DMA
// instructions per CU backs up the texture-address unit, and a wave blocked on
// issuing a load cannot issue its MFMAs either.
//
// Ragged edges clamp the 16-row BLOCK index of an operand load (never the row),
// so every lane offset is a launch constant: rows of the last block beyond M or
// N are read from the padded packed buffer and only feed outputs that are never
// stored.
// --------------------------------------------------------------------------
struct PersistTile {
    int j;            // index in the XCD's share, see tile_of_share; -1 when exhausted
    int tile_m, tile_n;
};

// The tile map of a persistent kernel, read from its arguments anew: its 26 fields kept in scalar registers all
// through the K loop make the forms with Aux on its own scale spill 110 more of them (8192 x 1280 -> 3840 69.0 us,
// read anew once per tile 67.1 us).  The other forms have the room, and the reads cost them 0.4 us a tile
// (16384 x 1280 -> 3840 per token).  The kernels' parameters are (GemmArgs, TileMap).
__device__ __forceinline__ TileMap tile_map_argument()
{
    static_assert(sizeof(GemmArgs) % alignof(TileMap) == 0, "the second parameter follows the first");
    typedef const __attribute__((address_space(4))) char *arg_ptr_t;
    arg_ptr_t p = (arg_ptr_t)__builtin_amdgcn_kernarg_segment_ptr() + sizeof(GemmArgs);
    asm volatile("" : "+s"(p));              // (the compiler no longer knows that it has read these before)
    return *(const TileMap *)p;
}

// The first tile of this XCD's share at or after j, in steps of `stride` workgroups of the XCD.
template <bool ANEW>
__device__ __forceinline__ PersistTile tile_at(const TileMap &map, int j, int stride)
{
    const TileMap tm = ANEW ? tile_map_argument() : map;
    PersistTile p;
    p.tile_m = p.tile_n = 0;
    int st;
    while ((st = tile_of_share(tm, (int)blockIdx.x & 7, j, p.tile_m, p.tile_n)) < 0) j += stride;
    p.j = st > 0 ? j : -1;
    return p;
}

// The tile is WN x WM waves of FN x FM fragments of 32 x 32.  Built as 2 x 4 waves of
// 4 x 2 (256 x 256, two waves per SIMD, each 128 (n) x 64 (m)), 1 x 4 of 4 x 2 (128 x 256)
// and 2 x 2 of 2 x 2 (128 x 128, for problems with few tiles).
// OWN (compile time): the launch's Aux codes have a scale of their own (GemmArgs::aux_own_scale),
// 1 with one activation scale per launch, 2 with one per token; forms of their own so that the
// usual kernel's register allocation does not carry the floating-point rescale of the
// accumulators (nor the per-launch form the per-token factors: 109 spilled registers in one kernel).
// GELU (compile time): the fused-activation form (GemmArgs::gelu): every epilogue applies the
// GELU and, with slab_out, the workgroup leaves the column maxima of its tile of Y.
template <int STAGES, int WN, int WM, int FN, int FM, int EPI, int OWN, bool GELU, int STORE>
__device__ __forceinline__ void gemm_persist_body(const GemmArgs &a, const TileMap &tm)
{
    constexpr int NWAVES = WN * WM, TN = WN * FN * 32, TM = WM * FM * 32, SWZ = 1;
    constexpr int NMFMA = FN * FM;           // MFMAs per wave per K sub-step
    constexpr int NFRAG = FN + FM;           // fragment reads per wave per K sub-step
    constexpr int STAGE_BYTES = (TN + TM) * BK;
    constexpr int RING_BYTES = STAGES * STAGE_BYTES;
    constexpr int DEPTH = STAGES - 1;        // K steps in flight ahead of the one being computed
    constexpr int LHN = TN / 16 / NWAVES, LHM = TM / 16 / NWAVES;   // DMA instructions per wave, K step and operand
    static_assert(TN % (32 * NWAVES) == 0 && TM % (32 * NWAVES) == 0 && FN * 2 % LHN == 0 && FM * 2 % LHM == 0,
                  "the waves share the blocks of both operands evenly, a fragment's two blocks with one wave");
    constexpr int LOADS = LHN + LHM;
    constexpr int DMA_EVERY = NMFMA / LOADS; // one DMA instruction per this many MFMAs
    constexpr int REGION = LOADS * 1024;     // a wave's part of a stage: what it loads itself
    constexpr int PATCH_ROW = 2 * 64 + 16;   // epilogue patch: 32 tokens x 64 channels fp16 (+ pad)
    constexpr int PATCH_BYTES = 32 * PATCH_ROW;
    // global stores per wave per full tile (with the fused GELU one more: the column maxima)
    constexpr int STORES = FM * (FN / 2) * 4 + (GELU ? 1 : 0);
    static_assert(LOADS <= NMFMA && NFRAG <= NMFMA, "schedule does not fit");
    constexpr bool OVERLAY = REGION >= PATCH_BYTES;
    static_assert((DEPTH - 1) * LOADS + STORES + 8 < 64, "vmcnt has 6 bits");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    typedef __attribute__((address_space(3))) void *lptr_t;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_n = (wave % WN) * (FN * 32), wave_m = (wave / WN) * (FM * 32);
    constexpr int CONST_AT = RING_BYTES + (OVERLAY ? 0 : NWAVES * PATCH_BYTES);
    float *const chan = (float *)(lds + CONST_AT) + wave * kChanFloats;

    const int t_aux = aux_tiles(a);
    const int k_tiles = a.k_pad / BK;
    const int stride = (int)gridDim.x >> 3;  // the grid is a multiple of the 8 XCDs

    PersistTile cur_tile = tile_at<OWN != 0>(tm, (int)blockIdx.x >> 3, stride);
    if (cur_tile.j < 0) return;
    if (a.wg_ticks != nullptr) {             // measurement aid: when this workgroup started
        if (tid == 0) a.wg_ticks[2 * blockIdx.x] = wall_clock64();
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // keeps the store out of the loop's load accounting
    }
    // launch constants of the epilogue, fetched before any operand load is in flight
    const float sx = a.x_scale[0];
    const float sw0 = a.w_scale[0];
    const bool has_zc = epi_zero(EPI) < 0 ? a.cn != nullptr : epi_zero(EPI) != 0;
    const bool x_tok = epi_token(EPI) < 0 ? a.x_per_token != 0 : epi_token(EPI) != 0;
    const int z_launch = has_zc && !x_tok ? a.zero_point[0] : 0;
    // where the accumulators start (see kCnBias): what comes off with z * cn[n], or by itself (see kAccBias), and
    // what the Aux weighting has to take off
    const int sub_bias = has_zc && !x_tok ? 0 : kAccBias;
    // (A zero point of 0, where the unlisted channels use the whole range, as without outliers: kAccBias all the same, which
    // the epilogue takes off in the place of z * cn.  Started at 0 / so, us: 8192 x 4096 -> 16384 474 / 458, 16384 x 1280 ->
    // 3840 112 / 109, naive 4096 x 4096 -> 4096 71.7 / 69.8.)
    const int acc_bias = has_zc && !x_tok && (z_launch != 0 || !z_offset(FN)) ? z_launch * a.cn_bias : kAccBias, acc_fix = ((1 << a.exp_shift) - 2) * acc_bias;
    const float rho = OWN == 1 ? aux_rho(a) : 0.f;
    // the tile's constants that come by DMA: weight scales (2 loads), bias, token scales, cn (2), z and rho per token
    constexpr bool L_W = epi_chan(EPI) != 0, L_B = epi_bias(EPI) != 0, L_T = epi_token(EPI) != 0, L_Z = epi_zero(EPI) != 0,
                   L_ZT = L_T && L_Z, L_RHO = OWN == 2;
    constexpr int CONST_LOADS = 2 * L_W + L_B + L_T + 2 * L_Z + L_ZT + L_RHO;

    // ---- DMA side -------------------------------------------------------------
    // One buffer_load ... lds instruction moves one 1 KiB block of the packed layout
    // (16 rows x 64 B) into 1 KiB of contiguous LDS: lane l lands at byte 16 l, i.e.
    // row l / 4, physical chunk l % 4, and fetches the logical chunk the swizzle maps
    // there.  The address is resource base + per-lane offset (a launch constant) +
    // a scalar offset (row block and K step), so a load costs one scalar add.
    // The stream of K steps runs DEPTH steps ahead of the compute loop, through the
    // phases { Aux steps, Body steps } of one tile after the other.
    const unsigned lane_off = (unsigned)((lane >> 2) * 64 + swizzle<SWZ>(lane >> 2, lane & 3) * 16);
    const unsigned body_rowblock = (unsigned)k_tiles * 1024u;          // bytes per 16 packed rows
    const unsigned aux_rowblock = (unsigned)(a.r_cap / BK) * 1024u;
    const int nblk_n = (a.N + 15) >> 4, nblk_m = (a.M + 15) >> 4;
    constexpr int RSRC_FLAGS = 0x00020000;   // raw buffer of dwords, offset checked against the size
    // resources of the phase the stream is in (rebuilt at each phase change, which is rare)
    __amdgpu_buffer_rsrc_t r_w, r_x;

    PersistTile dma_tile = cur_tile;
    // The tile after the current one, worked out at the end of each epilogue, where the scalar unit has
    // time: at the phase change all waves would wait for it.  With fewer K steps per tile than the
    // stream runs ahead, the stream may need the tile after that one and works it out itself.
    const bool known_next = t_aux + k_tiles > DEPTH;
    PersistTile nx_tile = tile_at<OWN != 0>(tm, cur_tile.j + stride, stride);
    bool d_aux;                 // phase of the stream
    int d_left;                 // K steps left in the phase
    unsigned d_w[LHN], d_x[LHM];  // scalar byte offsets of the next step's blocks
#define MUXQ_DMA_PHASE(aux_)                                                                    \
    do {                                                                                        \
        const bool ax_ = (aux_);                                                                \
        const unsigned rb_ = ax_ ? aux_rowblock : body_rowblock;                                \
        _Pragma("unroll") for (int i_ = 0; i_ < LHN; ++i_)                                      \
            d_w[i_] = rb_ * (unsigned)min(dma_tile.tile_n * (TN / 16) + wave * LHN + i_, nblk_n - 1); \
        _Pragma("unroll") for (int i_ = 0; i_ < LHM; ++i_)                                      \
            d_x[i_] = rb_ * (unsigned)min(dma_tile.tile_m * (TM / 16) + wave * LHM + i_, nblk_m - 1); \
        r_w = __builtin_amdgcn_make_buffer_rsrc((void *)(ax_ ? a.w_aux : a.w_q), 0,             \
                                                (int)((unsigned)nblk_n * rb_), RSRC_FLAGS);     \
        r_x = __builtin_amdgcn_make_buffer_rsrc((void *)(ax_ ? a.aux_q : a.a_q), 0,             \
                                                (int)((unsigned)nblk_m * rb_), RSRC_FLAGS);     \
        d_aux = ax_;                                                                            \
        d_left = ax_ ? t_aux : k_tiles;                                                         \
    } while (0)
    // Rare path, once per phase: Aux -> Body of the same tile, Body -> next tile.
    // After the last step of the last tile the stream keeps re-reading that step
    // into stages nobody reads, so the number of loads in flight stays uniform.
#define MUXQ_DMA_NEXT_PHASE                                                                     \
    do {                                                                                        \
        if (d_aux) {                                                                            \
            MUXQ_DMA_PHASE(false);                                                              \
        } else {                                                                                \
            const PersistTile nx_ = known_next ? nx_tile : tile_at<OWN != 0>(tm, dma_tile.j + stride, stride); \
            if (nx_.j >= 0) {                                                                   \
                dma_tile = nx_;                                                                 \
                MUXQ_DMA_PHASE(t_aux > 0);                                                      \
            } else {                                                                            \
                _Pragma("unroll") for (int i_ = 0; i_ < LHN; ++i_) d_w[i_] -= 1024u;            \
                _Pragma("unroll") for (int i_ = 0; i_ < LHM; ++i_) d_x[i_] -= 1024u;            \
                d_left = 1;                                                                     \
            }                                                                                   \
        }                                                                                       \
    } while (0)
    MUXQ_DMA_PHASE(t_aux > 0);
    int st_dma = 0;                            // byte offset of the stage the next DMA fills
    // DMA instruction j of a step: the wave's weight blocks, then its activation blocks
#define MUXQ_DMA(j_)                                                                            \
    do {                                                                                        \
        if ((j_) < LHN)                                                                         \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r_w,                                       \
                (lptr_t)(lds + st_dma + wave * REGION + (j_) * 1024), 16, lane_off, d_w[(j_) < LHN ? (j_) : 0], 0, 0); \
        else                                                                                    \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r_x,                                       \
                (lptr_t)(lds + st_dma + wave * REGION + (j_) * 1024), 16, lane_off, d_x[(j_) < LHN ? 0 : (j_) - LHN], 0, 0); \
    } while (0)
#define MUXQ_DMA_STEP_DONE                                                                      \
    do {                                                                                        \
        _Pragma("unroll") for (int i_ = 0; i_ < LHN; ++i_) d_w[i_] += 1024u;                    \
        _Pragma("unroll") for (int i_ = 0; i_ < LHM; ++i_) d_x[i_] += 1024u;                    \
        --d_left;                                                                               \
        st_dma = st_dma + STAGE_BYTES == RING_BYTES ? 0 : st_dma + STAGE_BYTES;                 \
    } while (0)

    // ---- fragment read addresses (byte offsets inside a stage) --------------------
    const int fr = lane & 31, fh = lane >> 5;
    int w_rd[2], x_rd[2];                      // [kk]
    {
        // (whole blocks of 16 rows behind row fr keep the swizzle bits)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int in_frag = fr * BK + swizzle<SWZ>(fr, kk * 2 + fh) * 16;
            w_rd[kk] = wave_n / (16 * LHN) * REGION + in_frag;
            x_rd[kk] = wave_m / (16 * LHM) * REGION + LHN * 1024 + in_frag;
        }
    }
    // fragment read q of a K sub-step: q < FN -> weight fragment q, else activation fragment q - FN
#define MUXQ_RD(wf_, xf_, stage_base_, kk_, q_)                                                 \
    do {                                                                                        \
        if ((q_) < FN) wf_[(q_)] = *(const v4i *)((stage_base_) + w_rd[kk_] + ((q_) * 2 / LHN) * REGION + ((q_) * 2 % LHN) * 1024); \
        else xf_[(q_) - FN] = *(const v4i *)((stage_base_) + x_rd[kk_] + (((q_) - FN) * 2 / LHM) * REGION + (((q_) - FN) * 2 % LHM) * 1024); \
    } while (0)
#define MUXQ_MFMA(q_, wf_, xf_)                                                                 \
    acc[(q_) / FM][(q_) % FM] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf_[(q_) / FM], xf_[(q_) % FM], acc[(q_) / FM][(q_) % FM], 0, 0, 0)
#define MUXQ_PIN __builtin_amdgcn_sched_barrier(0)

    // ---- prologue: DEPTH K steps in flight, step 0 landed, its first fragments read ----
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
#pragma unroll
        for (int j = 0; j < LOADS; ++j) MUXQ_DMA(j);
        MUXQ_DMA_STEP_DONE;
        if (d_left == 0) MUXQ_DMA_NEXT_PHASE;
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm((DEPTH - 1) * LOADS));
    __builtin_amdgcn_s_barrier();
    v4i wfA[FN], xfA[FM], wfB[FN], xfB[FM];
#pragma unroll
    for (int q = 0; q < NFRAG; ++q) MUXQ_RD(wfA, xfA, lds, 0, q);
    __builtin_amdgcn_s_waitcnt(waitcnt_lds_only());

    int st_cur = 0;                // byte offset of the stage being computed
    bool stores_pending = false;   // the previous tile's stores may still be in the vmcnt queue

    // One K step.  First half: MFMAs on the fragments of K sub-step 0; in their shadow
    // the fragment reads of sub-step 1 and this step's DMA instructions, spread evenly
    // (a burst of loads backs up the address unit, and a wave blocked on issuing a load
    // cannot issue its MFMAs either).  The stage the DMA refills was last read in the
    // first half of the previous step, i.e. before the barrier every wave has passed
    // since.  Then the next K step must have landed (this wave's part: everything but
    // the newest DEPTH - 1 steps of DMA, which complete in issue order; everybody's
    // part: the barrier), and the fragment reads of this stage must be complete before
    // another wave may refill it after the barrier.  Second half: sub-step 1, and the
    // first fragments of the next step.
    // Wave priority: the second half of a step runs at a higher priority than the first
    // (which carries the DMA instructions).  Of the two waves of a SIMD the one further
    // along then wins the issue arbitration: 6 % fewer cycles per tile, 2 % less time
    // (the chip is power-limited: most of a cycle gain comes back as a lower clock).
    // Only in the 8-wave form: with two 4-wave workgroups per CU it costs 3-4 %.
    // The first step of a tile (FIRST_ = 1) is written out on its own: only there can
    // the previous tile's stores still sit in the queue, and only there are the tile's
    // epilogue constants fetched (straight into the wave's `chan`: they queue behind the
    // step's operand loads and land K steps before use), so the steady-state step keeps
    // a single wait and no branches.
#define MUXQ_KSTEP(FIRST_)                                                                      \
    do {                                                                                        \
        const unsigned char *const cur_ = lds + st_cur;                                         \
        if (NWAVES == 8) __builtin_amdgcn_s_setprio(0);                                         \
        MUXQ_PIN;                                                                               \
        _Pragma("unroll") for (int q = 0; q < NMFMA; ++q) {                                     \
            MUXQ_MFMA(q, wfA, xfA);                                                             \
            if (q < NFRAG) MUXQ_RD(wfB, xfB, cur_, 1, q);                                       \
            if (q % DMA_EVERY == 0 && q / DMA_EVERY < LOADS) MUXQ_DMA(q / DMA_EVERY);           \
            if (q == NMFMA - 1) MUXQ_DMA_STEP_DONE;                                             \
            MUXQ_PIN;                                                                           \
        }                                                                                       \
        if (FIRST_) {                                                                           \
            MUXQ_CONST_LOADS;                                                                   \
            if (stores_pending)                                                                 \
                __builtin_amdgcn_s_waitcnt(waitcnt_vm_lds((DEPTH - 1) * LOADS + STORES + CONST_LOADS)); \
            else                                                                                \
                __builtin_amdgcn_s_waitcnt(waitcnt_vm_lds((DEPTH - 1) * LOADS + CONST_LOADS));  \
            stores_pending = false;                                                             \
        } else {                                                                                \
            __builtin_amdgcn_s_waitcnt(waitcnt_vm_lds((DEPTH - 1) * LOADS));                    \
        }                                                                                       \
        __builtin_amdgcn_s_barrier();                                                           \
        if (NWAVES == 8) __builtin_amdgcn_s_setprio(1);                                         \
        MUXQ_PIN;                                                                               \
        const int st_next_ = st_cur + STAGE_BYTES == RING_BYTES ? 0 : st_cur + STAGE_BYTES;     \
        const unsigned char *const nxt_ = lds + st_next_;                                       \
        _Pragma("unroll") for (int q = 0; q < NMFMA; ++q) {                                     \
            MUXQ_MFMA(q, wfB, xfB);                                                             \
            if (q < NFRAG) MUXQ_RD(wfA, xfA, nxt_, 0, q);                                       \
            if (q == NMFMA - 2 && d_left == 0) MUXQ_DMA_NEXT_PHASE;                             \
            if (q == NMFMA - 1) st_cur = st_next_;                                              \
            MUXQ_PIN;                                                                           \
        }                                                                                       \
        __builtin_amdgcn_s_waitcnt(waitcnt_lds_only());                                         \
    } while (0)
    // The constants' resources are built on the spot (a feature that is off gets a
    // zero-sized resource, whose loads return zeros without touching memory).  Whole
    // offsets go into the per-lane operand: that is the part the buffer range check
    // covers, so channels past N and tokens past M read zeros.
#define MUXQ_CONST_LOAD(base_, on_, size_, chan_, at_)                                          \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(                                                   \
        __builtin_amdgcn_make_buffer_rsrc((on_) ? (void *)(base_) : (void *)a.w_scale, 0, (on_) ? (size_) : 0, RSRC_FLAGS), \
        (lptr_t)(chan + (chan_)), 4, (at_), 0, 0, 0)
#define MUXQ_CONST_LOADS                                                                        \
    do {                                                                                        \
        const int n_w_ = cur_tile.tile_n * TN + wave_n, m_w_ = cur_tile.tile_m * TM + wave_m;   \
        if constexpr (L_W) {                                                                    \
            MUXQ_CONST_LOAD(a.w_scale, a.w_per_channel, a.N * 4, 0, (n_w_ + lane) * 4);         \
            MUXQ_CONST_LOAD(a.w_scale, a.w_per_channel, a.N * 4, 64, (n_w_ + 64 + lane) * 4);   \
        }                                                                                       \
        if constexpr (L_B) MUXQ_CONST_LOAD(a.bias, a.bias != nullptr, a.N * 2, 128, (n_w_ + 2 * lane) * 2); \
        if constexpr (L_T) MUXQ_CONST_LOAD(a.x_scale, a.x_per_token, a.M * 4, 192, (m_w_ + lane) * 4); \
        if constexpr (L_Z) {                                                                    \
            MUXQ_CONST_LOAD(a.cn, a.cn != nullptr, a.N * 4, 256, (n_w_ + lane) * 4);            \
            MUXQ_CONST_LOAD(a.cn, a.cn != nullptr, a.N * 4, 320, (n_w_ + 64 + lane) * 4);       \
        }                                                                                       \
        if constexpr (L_ZT)                                                                     \
            MUXQ_CONST_LOAD(a.zero_point, a.cn != nullptr && a.x_per_token, a.M * 4, 384, (m_w_ + lane) * 4); \
        if constexpr (L_RHO) MUXQ_CONST_LOAD(aux_rho_tok(a), true, a.M * 4, 448, (m_w_ + lane) * 4); \
    } while (0)

    // fused-GELU form: per-wave column maxima of the tile (fp16 magnitudes of the wave's FN * 32 channels), in
    // the place that only the forms with a factor per token use among the wave's constants
    static_assert(FN * 32 * 2 <= 64 * 4, "column maxima do not fit");
    const auto wave_colmax = [&](int wm, int wn) {
        return (unsigned short *)((float *)(lds + CONST_AT) + (wm * WN + wn) * kChanFloats + 448);
    };

    const int t_all = t_aux + k_tiles;
    while (cur_tile.j >= 0) {
        v16i acc[FN][FM];
#pragma unroll
        for (int fn = 0; fn < FN; ++fn)
#pragma unroll
            for (int fm = 0; fm < FM; ++fm)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[fn][fm][v] = acc_bias;

        // The Aux steps, then (after weighting the Aux accumulators by c = 2^exp - 1)
        // the Body steps.
        MUXQ_KSTEP(1);
#pragma unroll 1
        for (int t = 1; t < t_all; ++t) {
            if (t == t_aux) {                                    // acc_aux -> c * acc_aux
                if constexpr (OWN == 2) {
                    // one factor per token: staged with the tile's constants (issued with the
                    // first K step, so everything older has to land first)
                    float rho_t[FM];
                    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lds(0));
                    asm volatile("" ::: "memory");       // the reads below stay behind the wait
#pragma unroll
                    for (int fm = 0; fm < FM; ++fm) rho_t[fm] = chan[448 + fm * 32 + (lane & 31)];
                    scale_acc_rho_tok<FN, FM>(acc, rho_t, acc_bias);
                } else if constexpr (OWN == 1) scale_acc_rho<FN, FM>(acc, rho, acc_bias);
                else scale_acc<FN, FM>(acc, a.exp_shift, acc_fix);
            }
            MUXQ_KSTEP(0);
        }

        // ---- epilogue of this tile; the ring keeps its loads in flight meanwhile ----
        unsigned char *const patch = OVERLAY ? lds + (st_cur == 0 ? RING_BYTES - STAGE_BYTES : st_cur - STAGE_BYTES) + wave * REGION
                                             : lds + RING_BYTES + wave * PATCH_BYTES;
        const int m_base = cur_tile.tile_m * TM + wave_m, n_base = cur_tile.tile_n * TN + wave_n;
        [[maybe_unused]] const bool full = cur_tile.tile_m * TM + TM <= a.M && cur_tile.tile_n * TN + TN <= a.N;
        // a one-step tile has not yet waited past its constants' loads
        if (CONST_LOADS > 0 && t_all == 1) __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        if constexpr (GELU) {
            uint4 mxh[FN / 2];
#pragma unroll
            for (int h = 0; h < FN / 2; ++h) mxh[h] = make_uint4(0, 0, 0, 0);
            epilogue_patch<FN, FM, PATCH_ROW, EPI, STORE, true>(a, acc, m_base, n_base, lane, patch, chan, sx, sw0, z_launch, sub_bias, mxh);
            if (a.slab_out != nullptr) {
                // A lane holds the maxima of its 8 channels of each half over the rows it stored;
                // the 8 lane groups of a wave hold different rows: fold them through the wave's
                // patch (a wave's LDS operations execute in order), then the WM waves that share
                // the channels through wg_colmax, and every wave stores TN / NWAVES channels.
#pragma unroll
                for (int h = 0; h < FN / 2; ++h) {
                    // (lanes exchange data through LDS here: the fences keep the compiler from
                    // moving one lane's accesses across the other lanes' -- to a single lane
                    // the addresses it reads and the one it writes look unrelated)
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    *(uint4 *)(patch + lane * 16) = mxh[h];
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    if (lane < 8) {
                        uint4 m = make_uint4(0, 0, 0, 0);
#pragma unroll
                        for (int g = 0; g < 8; ++g) m = absmax_step(m, *(const uint4 *)(patch + (g * 8 + lane) * 16));
                        *(uint4 *)(wave_colmax(wave / WN, wave % WN) + h * 64 + lane * 8) = m;
                    }
                }
                __builtin_amdgcn_s_waitcnt(waitcnt_lds_only());
                __builtin_amdgcn_s_barrier();
                constexpr int CH_PER_WAVE = TN / NWAVES;          // 32 channels, lanes 0..3
                const int c0 = wave * CH_PER_WAVE + lane * 8;
                const int n = cur_tile.tile_n * TN + c0;
                // (in a full tile every wave issues this store: the wait counts rely on it)
                if (lane < CH_PER_WAVE / 8 && n < a.slab_ld) {
                    uint4 m = make_uint4(0, 0, 0, 0);
#pragma unroll
                    for (int wm = 0; wm < WM; ++wm) m = absmax_step(m, *(const uint4 *)(wave_colmax(wm, c0 / (FN * 32)) + c0 % (FN * 32)));
                    *(uint4 *)(a.slab_out + (size_t)cur_tile.tile_m * a.slab_ld + n) = m;
                }
            }
        } else {
            epilogue_patch<FN, FM, PATCH_ROW, EPI, STORE, false>(a, acc, m_base, n_base, lane, patch, chan, sx, sw0, z_launch, sub_bias, nullptr);
        }
        // (a buffer store is issued for a partial tile as well; a store by address or of the column maxima is not)
        if ((EPI != kEpiAny || (full && a.dbg_acc == nullptr)) && (!GELU || (full && a.slab_out != nullptr))) {
            stores_pending = true;           // exactly STORES stores and no loads were issued
        } else {
            __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // unknown number of vector-memory operations: drain
        }
        cur_tile = nx_tile;
        if (cur_tile.j >= 0) nx_tile = tile_at<OWN != 0>(tm, cur_tile.j + stride, stride);
    }
    // Drain the unused tail loads before the workgroup's LDS is released.
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lds(0));
    if (a.wg_ticks != nullptr && tid == 0) a.wg_ticks[2 * blockIdx.x + 1] = wall_clock64();
#undef MUXQ_KSTEP
#undef MUXQ_CONST_LOADS
#undef MUXQ_DMA_PHASE
#undef MUXQ_DMA_NEXT_PHASE
#undef MUXQ_DMA
#undef MUXQ_DMA_STEP_DONE
#undef MUXQ_RD
#undef MUXQ_MFMA
#undef MUXQ_PIN
#undef MUXQ_CONST_LOAD
}

template <int STAGES, int EPI, int OWN, bool GELU, int STORE>
__global__ __launch_bounds__(512) void k_gemm_i8_persist8(const GemmArgs a, const TileMap tm)
{
    gemm_persist_body<STAGES, 2, 4, 4, 2, EPI, OWN, GELU, STORE>(a, tm);
}

// 128 (n) x 256 (m) tiles, 4 waves of 128 x 64, two workgroups per CU.  The epilogue's patches lie in the ring, in the
// stage that was computed last: every wave's in the part that it will load itself, so that its own loads follow its own
// stores to Y, and no wave still reads operands there (the barrier of the tile's last step came after the last read).
template <int STAGES, int EPI, int OWN, bool GELU, int STORE>
__global__ __launch_bounds__(256, 2) void k_gemm_i8_persist_half(const GemmArgs a, const TileMap tm)
{
    gemm_persist_body<STAGES, 1, 4, 4, 2, EPI, OWN, GELU, STORE>(a, tm);
}

// 128 x 128 tiles, 4 waves of 64 x 64: for problems whose 256 x 256 tiles would leave the last, or the
// only, round on the chip half empty.
template <int STAGES, int EPI, int OWN, bool GELU, int STORE>
__global__ __launch_bounds__(256, EPI == kEpiAny ? 2 : 1) void k_gemm_i8_persist4(const GemmArgs a, const TileMap tm)
{
    gemm_persist_body<STAGES, 2, 2, 2, 2, EPI, OWN, GELU, STORE>(a, tm);
}

#if MUXQ_GEMM_PART == 0

// --------------------------------------------------------------------------
// Problems with too few tiles for the forms above: 16 TNB x 16 TMB tiles, and the waves of a
// workgroup split K.  A block of the packed layout (16 rows x 64 codes, 1 KiB) is one operand of
// v_mfma_i32_16x16x64_i8 as it lies there -- lane l takes the 16 bytes of row l % 16 at 16 (l / 16)
// -- so fragments go from memory straight to registers: no LDS image, no barrier in the K loop,
// and every byte a workgroup reads is read by one wave once.  A wave keeps the loads of DEPTH K
// steps in flight.  The waves' INT32 partial sums meet in LDS (integer adds: any order gives the
// same sum).  Bound by what a CU fetches (operands come from L2 at 80-100 GB/s per CU) and by the
// latencies at its start and end; the matrix pipes, which run this MFMA shape at 60 % of the
// 32x32x32 rate, do not matter.
// The Aux K steps all belong to the last wave (which has the fewest Body steps), come first there
// and are weighted before its Body steps, as in the other forms.
// What counts beside the bytes is that no request waits for anything and nothing waits for a request it does not use: the first
// Aux step and the epilogue's constants, token scales and zero points are requested with the first Body steps, without
// branches.  (Before, a wave waited for all its first loads for the sake of a constant, the last wave was 2.6 us behind the others
// with Aux, every DEPTH steps all loads were waited for, and the end began with two loads: 512 x 4096 -> 1024 11.6 -> 10.1 us,
// 24 x 5120 -> 1280 6.9 -> 6.0.)
// --------------------------------------------------------------------------
template <int TNB, int TMB, int DEPTH, int W>
__global__ __launch_bounds__(W * 64) void k_gemm_i8_direct(const GemmArgs a, const TileMap tm)
{
    fetch_arguments();
    constexpr int FRAGS = TNB * TMB, NQ = TNB * 4;       // n quads per tile row
    __shared__ __attribute__((aligned(16))) v4i part[W * FRAGS * 64];
    __shared__ uint32_t s_colmax[TNB * 16];

    int tile_m, tile_n;
    if (!tile_of_workgroup(tm, tile_m, tile_n)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk_n = (a.N + 15) >> 4, nblk_m = (a.M + 15) >> 4;
    const int k_tiles = a.k_pad / BK;
    const int lane_off = (lane & 15) * 64 + (lane >> 4) * 16;
    // ragged edges: the last block again (it only feeds outputs that are not stored)
    int bn[TNB], bm[TMB];
#pragma unroll
    for (int i = 0; i < TNB; ++i) bn[i] = min(tile_n * TNB + i, nblk_n - 1);
#pragma unroll
    for (int i = 0; i < TMB; ++i) bm[i] = min(tile_m * TMB + i, nblk_m - 1);

    v4i acc[TNB][TMB];
#pragma unroll
    for (int i = 0; i < TNB; ++i)
#pragma unroll
        for (int j = 0; j < TMB; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    // The last wave's first Aux step, requested before anything else: its Body steps wait for it.  (Read whether or not there
    // are listed channels; the count comes at the same time.)
    const int aux_row_bytes = a.r_cap / BK * 1024;             // bytes of 16 packed Aux rows
    const bool aux_wave = wave == W - 1 && a.n_outliers != nullptr && a.r_cap > 0;
    typedef const __attribute__((address_space(4))) int32_t *scalar_ptr_t;       // (a scalar load: nothing queues behind it)
    const int32_t n_listed = *(scalar_ptr_t)(uintptr_t)(aux_wave ? (const void *)a.n_outliers : (const void *)a.x_scale);
    // (The other waves read 16 bytes of the weights: behind a branch the values were copied, and the copy waited for.)
    v4i wa[TNB], xa[TMB];
    const int8_t *const wa_src = aux_wave ? a.w_aux : a.w_q, *const xa_src = aux_wave ? a.aux_q : a.w_q;
    const int aux_off = aux_wave ? lane_off : 0, aux_rows = aux_wave ? aux_row_bytes : 0;
#pragma unroll
    for (int i = 0; i < TNB; ++i) wa[i] = *(const v4i *)(wa_src + (size_t)bn[i] * aux_rows + aux_off);
#pragma unroll
    for (int i = 0; i < TMB; ++i) xa[i] = *(const v4i *)(xa_src + (size_t)bm[i] * aux_rows + aux_off);

    v4i wf[DEPTH][TNB], xf[DEPTH][TMB];
    const int8_t *wp[TNB], *xp[TMB];
#pragma unroll
    for (int i = 0; i < TNB; ++i) wp[i] = a.w_q + (size_t)bn[i] * k_tiles * 1024 + lane_off;
#pragma unroll
    for (int i = 0; i < TMB; ++i) xp[i] = a.a_q + (size_t)bm[i] * k_tiles * 1024 + lane_off;
    const int nk = (k_tiles - wave + W - 1) / W;          // Body steps of this wave: wave, wave + W, ...
    auto load = [&](int d, int step) {
        const int off = (wave + min(step, nk - 1) * W) * 1024;     // past the end: the last step again, unused
#pragma unroll
        for (int i = 0; i < TNB; ++i) wf[d][i] = *(const v4i *)(wp[i] + off);
#pragma unroll
        for (int i = 0; i < TMB; ++i) xf[d][i] = *(const v4i *)(xp[i] + off);
    };
    if (nk > 0) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) load(d, d);
    }

    // Epilogue constants: a thread finishes 4 channels (n quad nq) of the tokens m0, m0 + MSTEP, ...  Requested behind the
    // first K steps and not touched before the end: no branches, what there is not is read from another place.
    constexpr int MSTEP = W * 64 / NQ, MT = (TMB * 16 + MSTEP - 1) / MSTEP;
    const int nq = tid % NQ, m0 = tid / NQ;
    const int n = tile_n * TNB * 16 + nq * 4;
    const bool n_in = n < a.N;                            // N % 8 == 0: a run of 4 is in or out as a whole
    const int nc = min(n, a.N - 4), w_at = a.w_per_channel ? nc : 0, w_step = a.w_per_channel ? 1 : 0;
    const unsigned short *const bias_src = a.bias != nullptr ? (const unsigned short *)a.bias : (const unsigned short *)a.w_scale;
    const int b_at = a.bias != nullptr ? nc : 0, b_step = a.bias != nullptr ? 1 : 0;
    float swv[4];
    unsigned short bias[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        swv[i] = a.w_scale[w_at + i * w_step];
        bias[i] = bias_src[b_at + i * b_step];
    }
    const v4i cn_raw = *(const v4i *)(a.cn != nullptr ? (const void *)(a.cn + nc) : (const void *)a.w_q);
    const int32_t *const z_src = a.cn != nullptr ? a.zero_point : (const int32_t *)a.x_scale;
    float sxv[MT];
    int zv[MT];
#pragma unroll
    for (int k = 0; k < MT; ++k) {
        const int tok = a.x_per_token ? min(tile_m * TMB * 16 + m0 + k * MSTEP, a.M - 1) : 0;
        sxv[k] = a.x_scale[tok];
        zv[k] = z_src[tok];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (tid < TNB * 16) s_colmax[tid] = 0;

    if (aux_wave) {
        const int t_aux = (max(0, min(n_listed, a.r_cap)) + BK - 1) / BK;
        // (the first step by itself: in one loop with the others it would wait for the Body loads too)
        if (t_aux > 0) {
#pragma unroll
            for (int i = 0; i < TNB; ++i)
#pragma unroll
                for (int j = 0; j < TMB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa[i], xa[j], acc[i][j], 0, 0, 0);
        }
        for (int t = 1; t < t_aux; ++t) {
            v4i wn[TNB], xn[TMB];
#pragma unroll
            for (int i = 0; i < TNB; ++i) wn[i] = *(const v4i *)(a.w_aux + (size_t)bn[i] * aux_row_bytes + t * 1024 + lane_off);
#pragma unroll
            for (int i = 0; i < TMB; ++i) xn[i] = *(const v4i *)(a.aux_q + (size_t)bm[i] * aux_row_bytes + t * 1024 + lane_off);
#pragma unroll
            for (int i = 0; i < TNB; ++i)
#pragma unroll
                for (int j = 0; j < TMB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wn[i], xn[j], acc[i][j], 0, 0, 0);
        }
        if (t_aux > 0 && !a.aux_own_scale) {              // acc_aux -> (2^e - 1) acc_aux
#pragma unroll
            for (int i = 0; i < TNB; ++i)
#pragma unroll
                for (int j = 0; j < TMB; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        acc[i][j][v] = (int)(((unsigned)acc[i][j][v] << a.exp_shift) - (unsigned)acc[i][j][v]);
        } else if (t_aux > 0) {                           // ... or onto Body's scale
            const float rho = aux_rho(a);
#pragma unroll
            for (int j = 0; j < TMB; ++j) {
                float r = rho;
                if (a.x_per_token) r = aux_rho_tok(a)[min((tile_m * TMB + j) * 16 + (lane & 15), a.M - 1)];
#pragma unroll
                for (int i = 0; i < TNB; ++i)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[i][j][v] = (int)__builtin_rintf(r * (float)acc[i][j][v]);
            }
        }
    }
    auto multiply = [&](int d) {
#pragma unroll
        for (int i = 0; i < TNB; ++i)
#pragma unroll
            for (int j = 0; j < TMB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf[d][i], xf[d][j], acc[i][j], 0, 0, 0);
    };
    // (no condition on a request in the loop: where one may have been left out, the compiler waits for all of them)
    int t = 0;
    for (; t + 2 * DEPTH <= nk; t += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            multiply(d);
            load(d, t + d + DEPTH);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
        if (t + d < nk) multiply(d);
        if (t + d + DEPTH < nk) load(d, t + d + DEPTH);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (t + d + DEPTH < nk) multiply(d);

    // Partial sums to LDS.  A 16 x 16 fragment has its lane (token l % 16, n quad q = l / 16) in slot
    // 16 q + (token + 4 nb + q) % 16: free of bank conflicts for this store and for the reads below.
    {
        const int m = lane & 15, q = lane >> 4;
#pragma unroll
        for (int i = 0; i < TNB; ++i)
#pragma unroll
            for (int j = 0; j < TMB; ++j)
                part[(wave * FRAGS + i * TMB + j) * 64 + q * 16 + ((m + 4 * i + q) & 15)] = acc[i][j];
    }
    lds_barrier();
    uint32_t mx[4] = {0, 0, 0, 0};
    const v4i cn = cn_raw - a.cn_bias;
#pragma unroll
    for (int k = 0; k < MT; ++k) {
        const int mt = m0 + k * MSTEP;
        if (mt >= TMB * 16) break;
        const int nb = nq >> 2, q = nq & 3, j = mt >> 4, m = tile_m * TMB * 16 + mt;
        const v4i *src = part + (nb * TMB + j) * 64 + q * 16 + (((mt & 15) + 4 * nb + q) & 15);
        v4i sum = src[0];
#pragma unroll
        for (int w = 1; w < W; ++w) sum += src[w * FRAGS * 64];
        if (!n_in || m >= a.M) continue;
        if (a.cn != nullptr) sum -= cn * zv[k];
        f16x4 out;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float y = (sxv[k] * swv[i]) * (float)sum[i];  // Eq. 3
            if (a.bias != nullptr) y = y + (float)__builtin_bit_cast(_Float16, bias[i]);
            out[i] = (_Float16)y;
            if (a.gelu) {
                out[i] = (_Float16)gelu_tanh_f32((float)out[i]);
                mx[i] = max(mx[i], (uint32_t)__builtin_bit_cast(unsigned short, (_Float16)out[i]) & 0x7fffu);
            }
        }
        *(f16x4 *)(a.y + (size_t)m * a.ldy + n) = out;
        if (a.dbg_acc != nullptr) *(v4i *)(a.dbg_acc + (size_t)m * a.N + n) = sum;
    }
    if (a.slab_out != nullptr) {                          // the tile's column maxima, for the next layer
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (mx[i] != 0) atomicMax(&s_colmax[nq * 4 + i], mx[i]);
        lds_barrier();
        const int ch = tile_n * TNB * 16 + tid;
        if (tid < TNB * 16 && ch < a.slab_ld) a.slab_out[(size_t)tile_m * a.slab_ld + ch] = (uint16_t)s_colmax[tid];
        // zeros in the K padding past the last tile
        if (tile_n == tm.tiles_n - 1)
            for (int i = tm.tiles_n * TNB * 16 + tid; i < a.slab_ld; i += W * 64) a.slab_out[(size_t)tile_m * a.slab_ld + i] = 0;
    }
}

// at_once: tiles an XCD works on at a time.  grid: workgroups for one tile each, a multiple of 8.
TileMap make_tile_map(const GemmArgs &a, int TN, int TM, int &grid, bool persistent = false, int at_once = 32)
{
    TileMap tm;
    tm.tiles_m = (a.M + TM - 1) / TM;
    tm.tiles_n = (a.N + TN - 1) / TN;
    const int total = tm.tiles_m * tm.tiles_n, even = (total + 7) / 8;
    // No more tiles than the chip works on at one time: eight blocks, one for each XCD, as square as there are,
    // if no XCD's CUs (32) get a tile more by them than by an even split, whose shares straddle blocks
    // (300 x 2560 -> 7680, 3 x 60 tiles: 16.2 us split evenly, 13.5 us in blocks of 3 x 8; 256 x 2048 -> 16384 15.7, 14.3 us).
    int square = 0;
    if (persistent && total <= at_once * 8)
        for (int bands = 1; bands <= 8; ++bands) {
            const int strips = 8 / bands, m = (tm.tiles_m + bands - 1) / bands, n = (tm.tiles_n + strips - 1) / strips;
            if ((m * n + 31) / 32 <= (even + 31) / 32 && (square == 0 || m + n < square)) {
                square = m + n;
                tm.sup_m = m;
                tm.sup_n = n;
            }
        }
    if (square == 0) {
        tm.sup_m = min(at_once > 32 ? 8 : 4, tm.tiles_m);
        tm.sup_n = min(at_once / tm.sup_m, tm.tiles_n);
    }
    const int super_m = (tm.tiles_m + tm.sup_m - 1) / tm.sup_m;
    tm.super_n = (tm.tiles_n + tm.sup_n - 1) / tm.sup_n;
    tm.n_super = super_m * tm.super_n;
    // otherwise whole blocks if they fill at least one round and no XCD's CUs get a tile more
    const int block_rounds = (tm.n_super + 7) / 8, most = block_rounds * tm.sup_m * tm.sup_n;
    const bool blocks = square != 0 || (total >= at_once * 8 && (most + 31) / 32 <= (even + 31) / 32);
    tm.at_once = blocks ? 0 : at_once;
    tm.full = total / (at_once * 8);
    tm.rest = total - tm.full * at_once * 8;
    const int last_rows = tm.tiles_m - (super_m - 1) * tm.sup_m, last_cols = tm.tiles_n - (tm.super_n - 1) * tm.sup_n;
    tm.by_block = divisor(tm.sup_m * tm.sup_n);
    tm.by_sup_n = divisor(tm.sup_n);
    tm.by_super_n = divisor(tm.super_n);
    tm.by_at_once = divisor(at_once);
    tm.by_band = divisor(tm.sup_m * tm.tiles_n);
    tm.by_band_block = divisor(tm.sup_m * tm.sup_n);
    tm.by_last_band_block = divisor(last_rows * tm.sup_n);
    tm.by_last_cols = divisor(last_cols);
    grid = tm.at_once ? (total + 7) / 8 * 8 : block_rounds * 8 * tm.sup_m * tm.sup_n;
    return tm;
}

#endif  // MUXQ_GEMM_PART == 0

// LDS bytes of a persistent kernel: the operand ring, the waves' epilogue patches and constants.
enum PersistTileForm { kTile256, kTile128, kTileHalf };
constexpr int tile_n_of(int t) { return t == kTile256 ? 256 : 128; }
constexpr int tile_m_of(int t) { return t == kTile128 ? 128 : 256; }
constexpr int waves_of(int t) { return t == kTile256 ? 8 : 4; }
template <int STAGES, int TILE>
constexpr int persist_lds_bytes()
{
    return STAGES * (tile_n_of(TILE) + tile_m_of(TILE)) * BK +
           waves_of(TILE) * ((TILE == kTileHalf ? 0 : 32 * (2 * 64 + 16)) + kChanFloats * 4);
}

typedef void (*persist_kernel_t)(const GemmArgs, const TileMap);

// The persistent kernels of one tile: what is fused or rescaled x what the epilogue applies x how Y is stored (kEpiAny
// decides that itself).  nullptr: not built.
enum PersistKind { kKindUsual, kKindOwn, kKindOwnToken, kKindGelu, kKinds };
template <int TILE, int EPI, int OWN, bool GELU>
persist_kernel_t persist_kernel_of(int store)
{
    constexpr int STAGES = 3;
    // (a form that is not built stands for the plain one)
    constexpr int AS_STREAM = EPI == kEpiAny ? kStoreL2 : kStoreStream;
    constexpr int AS_TOGETHER = epi_flags(EPI) || GELU || TILE == kTile128 ? kStoreL2 : kStoreTogether;
#define MUXQ_FORM(STORE_)                                                         \
    (TILE == kTile256   ? k_gemm_i8_persist8<STAGES, EPI, OWN, GELU, STORE_>      \
     : TILE == kTile128 ? k_gemm_i8_persist4<STAGES, EPI, OWN, GELU, STORE_>      \
                        : k_gemm_i8_persist_half<STAGES, EPI, OWN, GELU, STORE_>)
    return store == kStoreStream ? MUXQ_FORM(AS_STREAM) : store == kStoreTogether ? MUXQ_FORM(AS_TOGETHER) : MUXQ_FORM(kStoreL2);
#undef MUXQ_FORM
}
// Which binary a kernel is in: 1 own scales of Aux, 2 the fused GELU, 3 what a layer has no use for in its calls (the
// accumulator export, far rows, muxq_gemm_i8 on its own).
constexpr int part_of(int kind, int epi)
{
    return kind == kKindOwn || kind == kKindOwnToken ? 1 : kind == kKindGelu ? 2 : epi == kEpiAny || (epi >= kEpiPlain && epi <= kEpiChanBias) ? 3 : 0;
}

// The kernels of this binary.
template <int TILE>
persist_kernel_t persist_kernel_here(int kind, int epi, int store)
{
#define MUXQ_CASE(KIND_, EPI_, OWN_, GELU_)                                                        \
    static_assert(part_of(KIND_, EPI_) == MUXQ_GEMM_PART, "in another binary");                    \
    case KIND_ * kEpis + EPI_: return persist_kernel_of<TILE, EPI_, OWN_, GELU_>(store)
    switch (kind * kEpis + epi) {
#if MUXQ_GEMM_PART == 0
        MUXQ_CASE(kKindUsual, kEpiPlainZ, 0, false);
        MUXQ_CASE(kKindUsual, kEpiBiasZ, 0, false);
        MUXQ_CASE(kKindUsual, kEpiChanZ, 0, false);
        MUXQ_CASE(kKindUsual, kEpiChanBiasZ, 0, false);
        MUXQ_CASE(kKindUsual, kEpiToken, 0, false);
        MUXQ_CASE(kKindUsual, kEpiTokenBias, 0, false);
        MUXQ_CASE(kKindUsual, kEpiVector, 0, false);
        MUXQ_CASE(kKindUsual, kEpiVectorBias, 0, false);
#elif MUXQ_GEMM_PART == 1
        MUXQ_CASE(kKindOwn, kEpiAny, 1, false);
        MUXQ_CASE(kKindOwn, kEpiPlainZ, 1, false);
        MUXQ_CASE(kKindOwn, kEpiBiasZ, 1, false);
        MUXQ_CASE(kKindOwn, kEpiChanZ, 1, false);
        MUXQ_CASE(kKindOwn, kEpiChanBiasZ, 1, false);
        MUXQ_CASE(kKindOwnToken, kEpiAny, 2, false);
        MUXQ_CASE(kKindOwnToken, kEpiToken, 2, false);
        MUXQ_CASE(kKindOwnToken, kEpiTokenBias, 2, false);
        MUXQ_CASE(kKindOwnToken, kEpiVector, 2, false);
        MUXQ_CASE(kKindOwnToken, kEpiVectorBias, 2, false);
#elif MUXQ_GEMM_PART == 2
        MUXQ_CASE(kKindGelu, kEpiAny, 0, true);
        MUXQ_CASE(kKindGelu, kEpiGeneral, 0, true);
        MUXQ_CASE(kKindGelu, kEpiPlainZ, 0, true);
        MUXQ_CASE(kKindGelu, kEpiBiasZ, 0, true);
        MUXQ_CASE(kKindGelu, kEpiChanBiasZ, 0, true);
        MUXQ_CASE(kKindGelu, kEpiTokenBias, 0, true);
        MUXQ_CASE(kKindGelu, kEpiVectorBias, 0, true);
#else
        MUXQ_CASE(kKindUsual, kEpiAny, 0, false);
        MUXQ_CASE(kKindUsual, kEpiPlain, 0, false);
        MUXQ_CASE(kKindUsual, kEpiBias, 0, false);
        MUXQ_CASE(kKindUsual, kEpiChan, 0, false);
        MUXQ_CASE(kKindUsual, kEpiChanBias, 0, false);
#endif
    default: return nullptr;
    }
#undef MUXQ_CASE
}

}  // namespace

template <int PART> const void *persist_kernel_of_part(int tile, int kind, int epi, int store);
template <> const void *persist_kernel_of_part<MUXQ_GEMM_PART>(int tile, int kind, int epi, int store)
{
    return (const void *)(tile == kTile256   ? persist_kernel_here<kTile256>(kind, epi, store)
                          : tile == kTile128 ? persist_kernel_here<kTile128>(kind, epi, store)
                                             : persist_kernel_here<kTileHalf>(kind, epi, store));
}

#if MUXQ_GEMM_PART == 0

template <> const void *persist_kernel_of_part<1>(int tile, int kind, int epi, int store);
template <> const void *persist_kernel_of_part<2>(int tile, int kind, int epi, int store);
template <> const void *persist_kernel_of_part<3>(int tile, int kind, int epi, int store);

namespace {

persist_kernel_t persist_kernel(int tile, int kind, int epi, int store)
{
    const int part = part_of(kind, epi);
    return (persist_kernel_t)(part == 1   ? persist_kernel_of_part<1>(tile, kind, epi, store)
                              : part == 2 ? persist_kernel_of_part<2>(tile, kind, epi, store)
                              : part == 3 ? persist_kernel_of_part<3>(tile, kind, epi, store)
                                          : persist_kernel_of_part<0>(tile, kind, epi, store));
}


// What the launcher needs to know about a device, found once per device (gemm_prepare_device).
constexpr int kMaxDevices = 64;
std::atomic<int> g_device_cus[kMaxDevices];      // 0 = not prepared yet
std::mutex g_prepare_mutex;

// The persistent kernels take more LDS than a kernel may without asking, so each needs an attribute set on each device, which
// loads its binary: for a kernel's first launch, and in muxq_init for all (first launches under capture).
std::atomic<unsigned char> g_lds_set[kMaxDevices][3][kKinds * kEpis * kStores];

template <int STAGES, int TILE>
hipError_t set_persist_lds(int dev, int kind, int epi, int store, persist_kernel_t k)
{
    std::atomic<unsigned char> &set = g_lds_set[dev][TILE][(kind * kEpis + epi) * kStores + store];
    if (set.load(std::memory_order_acquire) != 0) return hipSuccess;
    std::lock_guard<std::mutex> lock(g_prepare_mutex);
    const hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             persist_lds_bytes<STAGES, TILE>());
    if (e == hipSuccess) set.store(1, std::memory_order_release);
    return e;
}

template <int STAGES, int TILE>
hipError_t set_all_persist_lds(int dev)
{
    for (int i = 0; i < kKinds * kEpis * kStores; ++i) {
        const int kind = i / kStores / kEpis, epi = i / kStores % kEpis, store = i % kStores;
        const persist_kernel_t k = persist_kernel(TILE, kind, epi, store);
        const hipError_t e = k == nullptr ? hipSuccess : set_persist_lds<STAGES, TILE>(dev, kind, epi, store, k);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t prepare_current_device(int dev)
{
    std::lock_guard<std::mutex> lock(g_prepare_mutex);
    if (g_device_cus[dev].load(std::memory_order_acquire) != 0) return hipSuccess;
    hipError_t e;
    if ((e = few_prepare_device()) != hipSuccess) return e;
    int cus = 0;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    int n_cu = cus > 0 ? cus / 8 * 8 : 8;   // a multiple of the 8 XCDs keeps workgroup i on XCD i % 8
    if (n_cu < 8) n_cu = 8;
    g_device_cus[dev].store(n_cu, std::memory_order_release);
    return hipSuccess;
}

// CU count (rounded down to a multiple of 8) of the current device, preparing it on first use.
hipError_t current_device_cus(int &n_cu, int &dev)
{
    dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    n_cu = g_device_cus[dev].load(std::memory_order_acquire);
    if (n_cu != 0) return hipSuccess;
    if ((e = prepare_current_device(dev)) != hipSuccess) return e;
    n_cu = g_device_cus[dev].load(std::memory_order_acquire);
    return hipSuccess;
}

template <int STAGES, int TILE>
hipError_t launch_persist(const GemmArgs &a, hipStream_t s)
{
    int total;
    const TileMap tm = make_tile_map(a, tile_n_of(TILE), tile_m_of(TILE), total, true, TILE == kTile256 ? 32 : 64);
    constexpr int lds_bytes = persist_lds_bytes<STAGES, TILE>();
    constexpr int wgs_per_cu = 160 * 1024 / lds_bytes;     // by LDS; registers allow at least as many
    static_assert(wgs_per_cu >= 1, "ring too deep");
    const int kind = a.gelu ? kKindGelu : !a.aux_own_scale ? kKindUsual : a.x_per_token ? kKindOwnToken : kKindOwn;
    const int store = stream_rows(a) ? kStoreStream : (size_t)a.M * a.N * 2 > (size_t)32 << 20 ? kStoreTogether : kStoreL2;
    int epi = (a.x_per_token ? a.w_per_channel ? kEpiVector : kEpiToken
                             : (a.cn != nullptr ? kEpiPlainZ : kEpiPlain) + (a.w_per_channel ? 2 : 0)) + (a.bias != nullptr ? 1 : 0);
    // (32 rows of Y 2^25 elements apart are beyond the 32-bit offsets of the usual kernels' buffer.  Buffers of 8 rows in
    // all kernels: 16384 x 1280 -> 3840 per vector 112.3 -> 113.5 us.)
    if (a.dbg_acc != nullptr || a.ldy >= 1 << 25) epi = kEpiAny;
    persist_kernel_t kern = persist_kernel(TILE, kind, epi, store);
    // (the GELU without a bias: c_fc has one, so those are one kernel)
    if (kern == nullptr && kind == kKindGelu) kern = persist_kernel(TILE, kind, epi = kEpiGeneral, store);
    if (kern == nullptr) return hipErrorInvalidDeviceFunction;
    int n_cu = 0, dev = 0;
    hipError_t e = current_device_cus(n_cu, dev);
    if (e != hipSuccess || (e = set_persist_lds<STAGES, TILE>(dev, kind, epi, store, kern)) != hipSuccess) return e;
    const int grid = total < n_cu * wgs_per_cu ? total : n_cu * wgs_per_cu;
    return launch_kernel(kern, dim3(grid), dim3(waves_of(TILE) * 64), lds_bytes, s, a, tm);
}

template <int TNB, int TMB, int DEPTH, int W>
hipError_t launch_direct(const GemmArgs &a, hipStream_t s)
{
    int grid;
    const TileMap tm = make_tile_map(a, TNB * 16, TMB * 16, grid);
    return launch_kernel(k_gemm_i8_direct<TNB, TMB, DEPTH, W>, dim3(grid), dim3(W * 64), 0, s, a, tm);
}

}  // namespace

hipError_t gemm_prepare_device()
{
    int n_cu = 0, dev = 0;
    return current_device_cus(n_cu, dev);
}

hipError_t gemm_prepare_all()
{
    int n_cu = 0, dev = 0;
    hipError_t e = current_device_cus(n_cu, dev);
    if (e == hipSuccess) e = set_all_persist_lds<3, kTile256>(dev);
    if (e == hipSuccess) e = set_all_persist_lds<3, kTile128>(dev);
    if (e == hipSuccess) e = set_all_persist_lds<3, kTileHalf>(dev);
    return e;
}

enum GemmForm {
    kPersist128, kPersist256, kPersistHalf,
    kDirect16x16, kDirect16x32, kDirect32x32, kDirect32x64, kDirect64x64       // channels x tokens
};

// Which form runs a shape fastest was measured over 289 shapes (M up to 16384, K 256..5120, N 256..16384,
// each form forced in turn).  us per call, by form:
//   24 x 5120 -> 1280    16x16 5.3,  16x32 6.0,  32x32 8.2,  persistent 128 27.6
//   32 x 768 -> 2304     16x32 4.1,  32x32 4.7,  persistent 128 9.3
// and since the direct forms' requests no longer wait, as whole calls:
//   128 x 1024 -> 4096   32x32 14.6,  32x64 14.3,  64x64 15.7,  16x32 16.2,  persistent 128 17.5
//   512 x 1024 -> 1024   32x32 14.8,  32x64 14.7,  64x64 15.7,  persistent 128 17.8
//   768 x 768 -> 768     64x64 16.1,  32x32 17.3,  persistent 128 17.5
//   512 x 4096 -> 1024   32x64 18.7,  32x32 20.1,  64x64 21.1,  persistent 128 31.1
//   512 x 1024 -> 2048   64x64 15.9,  persistent 128 18.2,  32x32 19.0
//   1024 x 512 -> 1024   64x64 15.6,  persistent 128 16.4,  32x32 18.8
//   400 x 256 -> 2560    persistent 128 14.8,  64x64 20.1,  32x32 20.3
//   512 x 1024 -> 3072   persistent 128 18.4,  64x64 21.9,  32x32 23.0
// (a form with 64 x 64 tiles staged through registers, which was the choice up to K = 512, is 3 to 14 % slower than the
// better of these on all of 31 shapes with K from 8 to 512, and gone)
//
// off_lines: rows of Y off 64-byte boundaries, no GELU (it matters for the tiles of 256 tokens alone, whose slabs are the same)
static GemmForm gemm_form(int M, int N, int k_pad, bool off_lines = false)
{
    const auto tiles = [&](int tn, int tm) { return (long)((N + tn - 1) / tn) * ((M + tm - 1) / tm); };
    const long t64 = tiles(64, 64), t128 = tiles(128, 128), t256 = tiles(256, 256);
    // Too few tiles for the others: the smallest tile that gives no more workgroups than CUs, or, while
    // K is short, than are resident at once (a long K is bound by what the CUs fetch, and two small
    // tiles on a CU fetch more than one large one).
    const bool short_k = k_pad <= 1536;
    if (!short_k && tiles(16, 16) <= 256) return kDirect16x16;
    if (tiles(16, 32) <= (short_k ? 320 : 256)) return kDirect16x32;
    if (tiles(32, 32) <= (short_k ? 512 : 256)) return kDirect32x32;
    if (!short_k && tiles(32, 64) <= 256) return kDirect32x64;
    if (t64 <= 256) return kDirect64x64;
    // One row of tiles: half of a 64 x 64 tile and three quarters of a persistent one would be empty.  To three workgroups of 32 x 32 on a
    // CU, with one K step or from 12 on (us a call, 32 x 32 / persistent 128): 16 x 64 -> 20000 12.9 / 13.9, 32 x 768 -> 16392 15.1 / 16.1, 16 x 1536
    // -> 24576 17.7 / 20.8; 32 x 256 -> 20000 15.9 / 14.3, 32 x 512 -> 20000 15.9 / 15.0, with 800 tiles 32 x 768 -> 25600 17.9 / 16.3.
    if (tiles(32, 32) <= 768 && short_k && (k_pad <= 64 || k_pad >= 768)) return kDirect32x32;
    // A round of 256 tiles of 256 x 256 takes as long as three of 256 tiles of 128 x 128 (1024 channels:
    // 20-23 us and 5.3 us + 5.3 us each; the ratio holds from K = 768 to 5120), so the larger tile
    // wins where its last round is full enough: 8192 x 1024 -> 1024 14 us against 19 us,
    // 16384 x 1024 -> 1024 24 us against 21 us.
    const long rounds128 = (t128 + 255) / 256, rounds256 = (t256 + 255) / 256;
    const bool square128 = rounds128 < 3 * rounds256 || (rounds256 >= 3 && rounds128 == 3 * rounds256);
    // 128 x 256, two workgroups per CU.  A round of 512 tiles does the work of one of 256 tiles of 256 x 256 and
    // computes one tile under the other's epilogue, but fetches half as much again per K step: by the sweep (in K steps) 1.15
    // steps + 4 against steps + 7, and a last round of at most 256 tiles, one to a CU, is 0.62 of a full one.  us, 256 x 256 /
    // 128 x 256: 8192 x 1024 -> 4096 55.3 / 53.5, 5239 x 1728 -> 7224 122 / 108, 10796 x 1480 -> 3664 with GELU 123 / 110,
    // 16384 x 1280 -> 3840 111 / 117, 8192 x 4096 -> 16384 434 / 480 (K below 512 was not in the sweep).  Where
    // the rows of Y are off 64-byte boundaries the narrower tile shares more lines with other workgroups, and with 100 MiB of
    // Y or more that is counted as 1.1 (14061 x 752 -> 12600 207 / 228, 6569 x 912 -> 14704 121 / 133, 13653 x 520 -> 10608 142 /
    // 155; the line is not sharp: 15259 x 1856 -> 4464 169 / 164, 11828 x 584 -> 8744 131 / 130; with the GELU, or on 64 bytes, 6589 x
    // 568 -> 14432, 128 x 256 is 4 to 9 % the faster).  Of 80 more shapes the rule is then within 2.5 % of the best
    // form for all but one round half full (749 x 952 -> 11104 25.0 / 25.9) and 3399 x 536 -> 12024 (128 x 128 49.4 / 53.2).
    // Against 128 x 128 it reads a quarter less through LDS, which pays with a long K: a round 0.415 steps - 0.3 (16384 x 5120
    // -> 1280 203 / 191, 4352 x 5120 -> 4680 142 / 132, 16059 x 1432 -> 2152 107 / 102), and in two nearly full rounds
    // from K = 2048 on (8192 x 4096 -> 1024 80.3 / 76.5; 8192 x 1024 -> 1024 31.2 / 31.9; with 384 tiles even, with 270 7 %
    // slower), if that is one tile for each CU: where M leaves half a row of tiles empty it can be more, and then one CU works
    // on two (1040 x 2072 -> 6968, 275 tiles, 32.3 / 39.2; 1642 x 5024 -> 4744, 266, 59.4 / 73.7).  By 27 shapes with K from
    // 2048 to 5120: to 256 tiles 0.99 to 1.05 times as fast, from 258 to 275 tiles 0.78 to 0.85.
    const long t_half = tiles(128, 256), last = t_half % 512, steps = k_pad / 64 + 1;
    const long half = (100 * (t_half / 512) + (last == 0 ? 0 : last <= 256 ? 62 : 100)) * (115 * steps + 400) / 100;
    if (square128) {
        if (rounds128 == 2 ? k_pad >= 2048 && t128 > 448 && t_half <= 256
                           : rounds128 >= 5 && k_pad >= 1024 && 10 * half < rounds128 * (415 * steps - 300)) return kPersistHalf;
        return kPersist128;
    }
    const bool wide = off_lines && (size_t)M * N * 2 >= (size_t)100 << 20;
    return k_pad >= 512 && (wide ? half * 11 / 10 : half) < rounds256 * 100 * (steps + 7) ? kPersistHalf : kPersist256;
}

// (The callers divide by it: a form without a case here does not compile.)
#pragma clang diagnostic push
#pragma clang diagnostic error "-Wswitch"
int gemm_tile_rows(int M, int N, int k_pad)
{
    switch (gemm_form(M, N, k_pad)) {
    case kPersist256: case kPersistHalf: return 256;
    case kPersist128: return 128;
    case kDirect64x64: case kDirect32x64: return 64;
    case kDirect32x32: case kDirect16x32: return 32;
    case kDirect16x16: return 16;
    }
    __builtin_unreachable();
}
#pragma clang diagnostic pop

const char *gemm_kernel_name(int M, int N, int k_pad)
{
    switch (gemm_form(M, N, k_pad)) {
    case kPersist256: return "k_gemm_i8_persist8";
    case kPersist128: return "k_gemm_i8_persist4";
    case kPersistHalf: return "k_gemm_i8_persist_half";
    default: return "k_gemm_i8_direct";
    }
}

hipError_t launch_gemm(const GemmArgs &a, hipStream_t s)
{
    const bool off_lines = !a.gelu && (((uintptr_t)a.y | (uintptr_t)a.ldy * 2) % 64) != 0;
    switch (gemm_form(a.M, a.N, a.k_pad, off_lines)) {
    case kPersist256: return launch_persist<3, kTile256>(a, s);
    case kPersist128: return launch_persist<3, kTile128>(a, s);
    case kPersistHalf: return launch_persist<3, kTileHalf>(a, s);
    case kDirect16x16: return launch_direct<1, 1, 8, 8>(a, s);
    case kDirect16x32: return launch_direct<1, 2, 6, 4>(a, s);
    case kDirect32x32: return launch_direct<2, 2, 6, 4>(a, s);
    case kDirect32x64: return launch_direct<2, 4, 6, 4>(a, s);
    case kDirect64x64: return launch_direct<4, 4, 4, 4>(a, s);
    }
    return hipErrorInvalidValue;
}

#endif  // MUXQ_GEMM_PART == 0

}  // namespace muxq
