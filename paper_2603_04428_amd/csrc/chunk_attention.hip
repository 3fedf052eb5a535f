// Chunked-append causal attention over paged Q4 KV caches (Sec. 3.4 chunked prefill, Sec. 3.5 cross-phase
// append, Sec. 3.6 causal and sliding-window masks): every agent brings q_len new query tokens whose K/V have
// already been quantize-appended, and query token c of agent a attends to the first
// seq_len[a] - (q_len-1-c) tokens of that agent's cache -- the chunk's own keys in their Q4 form included.
//
// Unlike decode this is a dense contraction: the q_len * n_rep query rows that share one KV head form the
// M side of two GEMMs per KV tile (S = Q K^T, O += P V), so it runs on the matrix cores.  What bounds it is each wave's
// own chain (operand reads, dependent products, scales, maximum, exponentials, products) and the barrier behind it, with two
// waves per SIMD to fill the gaps: matrix pipe and LDS are each busy 46 % of the time.  A vector instruction takes
// 4.5 clocks of the issue port, a 32x32x16 matrix instruction about 5 (and 32 of the pipe), a 16x16x32 one 8.6 (and
// 17): the products are cut so that what a wave prepares itself (scales, weights) serves 32 query rows, and what can be prepared once
// (unpacked keys, values) all rows of the workgroup.
//
//  * A workgroup of eight waves owns 256 query rows of one (layer, agent, KV head) -- 256/n_rep consecutive chunk
//    positions times the n_rep query heads of the group -- 32 rows per wave; or 128 rows, when its waves 0..3 take the
//    first and waves 4..7 the second half of every tile's tokens (KSPLIT = 2: short chunks).
//  * A wave multiplies 64 tokens at a time as two interleaved pieces of 32 (the second chain of matrix instructions runs
//    while the first one's results are on their way), 256-wide heads one piece: a KV tile is 32 to 128 tokens.  Measured,
//    one piece / two: 70 tokens of four agents, 128-wide 60.6 / 50.5 us, 512 tokens of ten agents, six layers 2,878 /
//    2,738 us; 24 tokens of five agents, 192 + 128-wide 170 / 154 us.
//  * KV tiles are fetched as Q4 (codes + scale/bias, prefetched one tile ahead into registers) and staged
//    ONCE per workgroup in LDS: V_hat dequantized to binary16, row-major, K as matrix operands (a lane's A operand is exactly
//    one code word, masked in place into eight binary16 subnormals: c 2^-24 and, for odd nibbles, 16 c 2^-24 against q/16), [word][token].  The dims inside
//    a word appear in the order the nibble masks deliver them (0,4,1,5,2,6,3,7): the query operand uses the same order
//    for K, the output store undoes it for V_hat.
//  * Unpacking while staging instead of in every one of the eight waves takes 96 of 305 vector instructions out of a wave's
//    32 tokens (256-wide).  Measured, one call, packed / unpacked: 256-wide 512 tokens of ten agents of 4K-32K 2,440 / 2,356
//    us, of one behind 8,000 123.7 / 121.8; 128-wide, four agents, two layers 424 / 414; 192 + 128 265 / 257; 64-wide 107 /
//    100.  It is 8.6 % fewer clocks on the long call, of which the power limit gives a third back: 1.87 -> 1.81 GHz.  Where
//    the unpacked tile does not fit into LDS (chunk_unpacks_keys) the code words are staged as they are and masked by each
//    wave.  Whole numbers in place of the subnormals, in the one form and not in the other, gave the two forms different bits:
//    the matrix core's sums are 2e-8 off with them and 8e-7 with subnormals.  Outputs do not show that (errors against 64 bits
//    3.275e-4 and 3.277e-4).  They cost 4 instructions a word more and save the bias term's change of unit, 16 a piece: whole numbers /
//    subnormals 64-wide, ten agents, six layers 597 / 613 us, 128-wide, ten agents, three layers 2,043 / 2,072, 192 + 128 1,257 / 1,243, 256 1,944 / 1,937.
//  * K stays factored, S^T = sum_g s[t,g] (C_g Q_g^T) + b Qsum^T: the matrix core multiplies the codes exactly, and the
//    per-(token, group) scale meets the binary32 result of each group; the bias term is one more matrix
//    instruction per 32 tokens whose contraction runs over the groups (group sums of q split into a binary16 high
//    and low part).  A K row dequantized to binary16 would carry an absolute rounding error of 2^-11 |K_hat|,
//    which the large channels of real key caches turn into score errors of several 1e-3.  V_hat is dequantized
//    to binary16 (its rounding error is relative to the values that are averaged).
//  * The wave computes S^T (tokens are the M rows), so that the probabilities come out of the matrix core already in
//    the register layout the second GEMM wants for its B operand (P^T); no shuffle or LDS round trip between the
//    GEMMs.  O^T = V_hat^T P^T accumulates in binary32; its A operand wants 8 tokens of one dim per lane, which two
//    transposing LDS reads (ds_read_b64_tr_b16) deliver straight from the row-major tile: in a group of 16 lanes, lane
//    4e + c points at 4 consecutive dims (chunk c) of token e, and element e of what lane j receives is half j % 4 of
//    the chunk that lane 4e + j / 4 addressed, i.e. dim j of token e.
//  * M row m of a 32-token product stands for token perm(m) = 16 (m/16) + 8 ((m/4)%2) + 2 (m%4) + (m/8)%2: the rows one
//    transposing read touches are then two tokens apart, and with a pitch of 8 banks (mod 64) the four tokens x 64
//    bytes of half a wave fall into all 64 banks.
//  * At 256-wide heads the accumulators of 32 rows (128 registers) leave no room for the whole query operand (64) if
//    two waves are to share a SIMD: what does not fit (QREG) lies in LDS, in operand order; some of it at 128 and 192 too.
//    With KSPLIT = 2 the two waves of a row group read one copy, which the first one writes before the barrier in front of
//    the tile loop.
//  * Softmax is online, per query row (= per lane column): scores in binary32, log2 domain.  The reference of a row moves when
//    the row exceeds it by more than kSlack, which rescales the accumulators.  (Moving all rows of a wave together rescales less
//    often, 0.5 % over 25 calls, and makes a row's rounding depend on the rows beside it.)
//    The denominator sums the weights in binary32, as they are before they are rounded for the product.  (A sum of the
//    rounded ones is 8 instructions fewer per 32 tokens and up to 7 % closer where few tokens dominate, but a token in front
//    of 131,071 of weight 2^-25.2 then comes out 1.9e-3 off.)
//  * A wave works a step ahead of itself: step i takes the scores of tile i and then, between the matrix instructions of the
//    product of tile i - 1, the softmax of tile i.  The tiles are staged beside the scores, V one step behind K.  Measured
//    against scores, softmax and product one after the other, one call: 256-wide 512 tokens of ten agents of 6,000, three layers 1,844 /
//    1,821 us (4.05e6 / 3.80e6 clocks; the power limit lowers the clock by the half of that), a window of 1,024 330 / 311;
//    128-wide two layers of four agents 406 / 396, 192 + 128 253 / 248, 64-wide 599 / 584 (with the references of a wave moved together
//    and a denominator of rounded weights, 0.9 % of it).  The first step is a copy of its own
//    without a product, which a unit of few tiles would feel: with a product of zeros / without, 94 tokens of two agents behind
//    900, 128-wide, six layers 201 / 191 us (append included), 70 tokens of four agents 57.7 / 56.0, 256-wide 71.0 / 68.5, 700 tokens behind 300
//    49.3 / 47.0.  (A branch round the product inside the loop made the compiler copy or spill the accumulators.)
//  * Every variant runs without scratch memory or spills, and build.py refuses one that does not: in a build that spilled, the compiler
//    put a spill behind a loop over part of the threads but before all were switched on again.  What the tile loop does not
//    need is therefore worked out again behind it from opaque copies (lane_again, fresh).  What still diverges: the prefix sums
//    over the agents (ChunkStream::fill) and the staging of threads without a share (k_on, v_on, k_params_writer).
//  * Two forms of launch: one workgroup per unit (layer, agent, KV head, row tile); or, given a workspace, where the units are
//    fewer than two per compute unit and it gains something (chunk_rules.h), one workgroup per compute unit, each with an
//    equal contiguous range of all units' tiles.  A unit cut by a range's end leaves un-normalised sums, maxima and
//    denominators of every part in the workspace, and a second small kernel merges them in order.
//
// Measured, 256-wide heads, a 512-token chunk, one layer: ten agents of 4K-32K tokens (20,700 in the mean) 2.09 ms = 823 TFLOP/s
// with shares, 2.45 without; one agent behind 8,000 0.120 ms with, 0.315 without; 48 layers of ten agents, one unit per
// workgroup, 88.1 to 89.9 ms = 921 to 903 TFLOP/s (boxes differ).  There a wave issues 271 vector and 33 matrix instructions per 32 tokens (305 and 33 while every
// wave unpacked the keys) and waits to issue 22 % of the time; the clock falls as the pipe fills (on one box 1.99 GHz at 42 %, 1.92 at 45 %; others
// run at 1.95 to 1.99 at 46 %), so a clock saved is worth about half.  64 rows per wave at one wave per SIMD (half the LDS reads per row, the accumulators
// in the accumulator file): 3.64e6 clocks against 3.21e6, because one wave issues one instruction of any kind in five clocks.
// Holding the second wave of a SIMD half a step behind by two barriers per step cost 15 %.  Wave priorities by phase,
// deeper operand reads: no change.
#include <utility>

#include "chunk_rules.h"
#include "q4_device.h"
#include "q4kv_internal.h"

namespace q4kv {
namespace {

constexpr int kChunkWaves = 8;
constexpr int kChunkThreads = kChunkWaves * kWave;
constexpr int kRowsWave = 32; // query rows per wave
constexpr int kSub = 32;      // tokens per matrix tile of scores
constexpr float kNegBig = -1.0e30f;
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kMaxChunkWindowLayers = 128; // layers per call when every layer brings its own window

typedef float float16_t __attribute__((ext_vector_type(16)));

// A unit that several workgroups share: the record of the workgroup it begins in, how many records it has (0: none; the
// others are the first ones of the workgroups that follow), its place in the output.
struct ChunkShared {
    int slots, first_record, qt, kvh;
    int64_t token_row; // (layer in call * agents + agent) * q_len
};

struct ChunkParams {
    const uint32_t *k_codes, *v_codes;
    const uint16_t *k_scale, *k_bias, *v_scale, *v_bias;
    const uint16_t *q;
    uint16_t *out;
    const int32_t *block_table, *seq_len;
    float *part_acc;                // records of units that several workgroups share: [2 grid][wave][DV / 8][lane][4]
    float *part_ml;                 // [2 grid][wave][32 rows][2]: running maximum (log2 units), denominator
    ChunkShared *shared;            // [grid]: the unit that begins in a workgroup's range and goes on past it
    int num_blocks, kv_heads, q_heads, num_agents, max_blocks, max_seq_len, window, q_len;
    int layer_begin, layers_in_call, q_tiles;
    float score_scale;
    int per_layer_windows;          // 1: layer_window[] holds the window of every layer of the call
    int layer_window[kMaxChunkWindowLayers];
};

// ---------------------------------------------------------------------------------------------- units and ranges

struct ChunkUnit {
    int li, agent, kvh, qt; // layer in call, agent, KV head, row tile
};

// The tokens the rows of one row tile see: chunk position c sees [first(c), vis(c)), vis(c) = n - (q_len - 1 - c).
template <int QPOS, int TILE>
__device__ __forceinline__ void visible_range(const ChunkParams &p, int n, int window, int qt, int &t_begin, int &t_end)
{
    const int pos0 = qt * QPOS;                                             // first chunk position of the row tile
    t_end = n - (p.q_len - 1 - min(p.q_len - 1, pos0 + QPOS - 1));          // exclusive; may be <= 0
    const int vis_first = n - (p.q_len - 1 - pos0);
    t_begin = window > 0 && vis_first > window ? (vis_first - window) & ~(TILE - 1) : 0;
}

// tiles a unit counts for when all are dealt out (a unit that sees nothing still has rows of zeros to write)
template <int QPOS, int TILE>
__device__ __forceinline__ int unit_tiles(const ChunkParams &p, int n, int window, int qt)
{
    int t_begin, t_end;
    visible_range<QPOS, TILE>(p, n, window, qt, t_begin, t_end);
    return t_end > t_begin ? (t_end - t_begin + TILE - 1) / TILE : 1;
}

__device__ __forceinline__ int clamped_length(const ChunkParams &p, int agent)
{
    const int n = p.seq_len[agent];
    return n < 0 ? 0 : (n > p.max_seq_len ? p.max_seq_len : n);
}

__device__ __forceinline__ int scalar(int v) { return __builtin_amdgcn_readfirstlane(v); }

// All tiles of a call in the order (layer, agent, KV head, row tile, tile), one window for all layers.  pre[a] = tiles of
// the agents before a in one layer, pre[num_agents] = tiles of a layer, len[a] the agent's length; in LDS, filled by the
// first wave.
template <int QPOS, int TILE>
struct ChunkStream {
    const int *pre, *len;

    __device__ __forceinline__ static void fill(const ChunkParams &p, int *pre, int *len, int lane)
    {
        int total = 0;
        for (int a0 = 0; a0 < p.num_agents; a0 += kWave) {
            const int a = a0 + lane;
            int mine = 0, n = 0;
            if (a < p.num_agents) {
                n = clamped_length(p, a);
                for (int qt = 0; qt < p.q_tiles; ++qt) mine += unit_tiles<QPOS, TILE>(p, n, p.window, qt);
                mine *= p.kv_heads;
            }
            int incl = mine;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const int up = __shfl_up(incl, off, kWave);
                if (lane >= off) incl += up;
            }
            if (a < p.num_agents) {
                pre[a] = total + incl - mine;
                len[a] = n;
            }
            total += __shfl(incl, kWave - 1, kWave);
        }
        if (lane == 0) pre[p.num_agents] = total;
    }
    // the unit that tile x belongs to, the tile's number inside it, the unit's tiles, the agent's length
    __device__ __forceinline__ ChunkUnit locate(const ChunkParams &p, int x, int &at, int &tiles, int &n) const
    {
        ChunkUnit u;
        int agents = p.num_agents;
        asm volatile("" : "+s"(agents)); // else the address below is kept in a vector register from one part to the next
        const int layer_tiles = scalar(pre[agents]);
        u.li = x / layer_tiles;
        int r = x - u.li * layer_tiles;
        int lo = 0, hi = p.num_agents - 1; // largest a with pre[a] <= r (every agent has tiles)
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (scalar(pre[mid]) <= r) lo = mid; else hi = mid - 1;
        }
        u.agent = lo;
        r -= scalar(pre[lo]);
        const int per_head = (scalar(pre[lo + 1]) - scalar(pre[lo])) / p.kv_heads;
        u.kvh = r / per_head;
        r -= u.kvh * per_head;
        n = scalar(len[lo]);
        u.qt = 0;
        while (r >= (tiles = unit_tiles<QPOS, TILE>(p, n, p.window, u.qt))) {
            r -= tiles;
            ++u.qt;
        }
        at = r;
        return u;
    }
};

// ---------------------------------------------------------------------------------------------- small helpers

__device__ __forceinline__ half2_t pk_fma(half2_t a, half2_t b, half2_t c) { return a * b + c; }

// two nibble positions of a word pair as exact small integers in binary16:
// ((w & mask) | 0x6400.6400) is 1024 + c (or 1024 + 16c for the upper nibble of a byte); subtracting 1024 is exact
__device__ __forceinline__ half2_t nibbles_lo(uint32_t w)
{
    return bits_to_half2((w & 0x000F000Fu) | 0x64006400u) - half2_t{(half_t)1024.0f, (half_t)1024.0f};
}
__device__ __forceinline__ half2_t nibbles_hi16(uint32_t w) // 16 * code
{
    return bits_to_half2((w & 0x00F000F0u) | 0x64006400u) - half2_t{(half_t)1024.0f, (half_t)1024.0f};
}

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4_t *lds_short4_ptr;

// x[i] (op) x[i ^ 32] without touching LDS
__device__ __forceinline__ float xor32_max(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}
__device__ __forceinline__ float xor32_sum(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}

// Four normalised values of one query row at positions 8 j + 4 h .. + 3 of an 8-dim word of V_hat (h = lane / 32):
// dims (0,4,1,5) in the lower half of the wave, (2,6,3,7) in the upper.  The halves trade pairs, after which each
// lane holds four consecutive dims: 0..3 below, 4..7 above.
__device__ __forceinline__ void store_row_quad(uint16_t *word, int h, float a, float b, float c, float d)
{
    const uint32_t first = half2_to_bits(half2_t{(half_t)a, (half_t)c}), second = half2_to_bits(half2_t{(half_t)b, (half_t)d});
    const auto r = __builtin_amdgcn_permlane32_swap(first, second, false, false);
    *reinterpret_cast<uint2 *>(word + 4 * h) = make_uint2((uint32_t)r[0], (uint32_t)r[1]);
}

// How the threads of a workgroup share the staging of one tile of DIM-wide code rows: as many threads per row
// as fit, each with 2, 4 or 8 consecutive words (never across a quantization group).
template <int DIM, int THREADS, int TILE>
struct Stage {
    static constexpr int WORDS = DIM / 8; // code words per row
    static constexpr int WPT = TILE * (WORDS / 2) <= THREADS ? 2 : (TILE * (WORDS / 4) <= THREADS ? 4 : 8);
    static constexpr int TPR = WORDS / WPT; // threads per row
    static constexpr int ACTIVE = TILE * TPR;
    static_assert(WORDS % WPT == 0 && ACTIVE <= THREADS, "tile split");
};

template <bool B> struct Flag { static constexpr bool value = B; };
template <int I> struct Index { static constexpr int value = I; };
template <class F, int... I>
__device__ __forceinline__ void for_each_index(F &&f, std::integer_sequence<int, I...>) { (f(Index<I>()), ...); }
// f(Index<0>()) ... f(Index<N - 1>()): a loop that is unrolled whatever its size, with indexes that `if constexpr` can see
template <int N, class F>
__device__ __forceinline__ void unrolled(F &&f) { for_each_index(f, std::make_integer_sequence<int, N>()); }

// ---------------------------------------------------------------------------------------------- attention

// 32-token pieces of a tile that a wave multiplies at once.  Two give it two independent chains of matrix instructions
// and half the barriers; at 256-wide heads there are no registers for the second one's scores and products.
constexpr int chunk_pieces(int dk) { return dk == 256 ? 1 : 2; }
// KV tokens per tile
constexpr int chunk_tile(int dk, int ksplit) { return kSub * chunk_pieces(dk) * ksplit; }
// Whether the K tile is unpacked when it is staged: two tiles of K and V_hat and the query operand have 160 KB.  128 rows of
// 256-wide heads (64-token tiles) would need 182, of 192 + 128-wide ones (128 tokens) 193.
constexpr bool chunk_unpacks_keys(int dk, int ksplit) { return dk <= 128 || ksplit == 1; }

// KSPLIT 1: 256 rows per workgroup; 2: 128 rows, the two halves of the waves share the tokens of a tile.
// SHARES: the workgroup takes an equal share of all tiles; else one unit.
// BF: scale and bias are stored as bfloat16 (converted to binary16 when a row is staged).
template <int DK, int DV, int NREP, int KSPLIT, bool SHARES, bool BF>
__global__ __launch_bounds__(kChunkThreads, 2) void chunk_attention_kernel(ChunkParams p)
{
    constexpr int GK = DK / kGroup, GV = DV / kGroup;
    constexpr int ROWGROUPS = kChunkWaves / KSPLIT;       // waves that own rows of their own
    constexpr int QPOS = ROWGROUPS * kRowsWave / NREP;    // chunk positions per workgroup
    constexpr int KPITCH = DK / 8 + 4; // words; an odd multiple of 4: 16 rows x 16 bytes fall into all 64 banks
    constexpr int VPITCH = DV + 16;    // halves; 8 banks mod 64 (40 at 64-wide rows), see above
    constexpr int DTILES = DV / 32;    // 32-dim tiles of O^T
    constexpr int NP = chunk_pieces(DK), TILE = chunk_tile(DK, KSPLIT);
    constexpr bool KFULL = chunk_unpacks_keys(DK, KSPLIT);
    // matrix instructions (4 per group) whose query operand stays in registers; the rest lie in LDS
    // (as many as leave every variant without scratch memory)
    constexpr int QREG = DK == 256 ? (KFULL ? 5 : 4) : (DK == 192 ? 7 : (DK == 128 && KSPLIT == 1 && !SHARES ? 5 : 4));
    constexpr int QLDS = 4 * GK - QREG;
    constexpr int QROWS = ROWGROUPS * kWave; // lanes that hold query operands of their own
    typedef Stage<DK, kChunkThreads, TILE> SK; // staging of the K rows of a tile ...
    typedef Stage<DV, kChunkThreads, TILE> SV; // ... and of its V rows

    // two tiles each: while the waves multiply against one, they unpack the next into the other
    // K, unpacked: the 8 codes of a word as a matrix operand, [word][token]; else the code words as they are in the pool
    __shared__ __attribute__((aligned(16))) uint32_t k_lds[2][KFULL ? TILE * DK / 2 : TILE * KPITCH];
    __shared__ __attribute__((aligned(16))) half_t v_lds[2][TILE * VPITCH];   // V_hat
    // K scale [group][token]: a lane's first 8 scores take tokens 8 (lane / 32) .. + 7 of its 32, the last 8 those 16 further on
    __shared__ __attribute__((aligned(16))) half_t ks_lds[2][GK * TILE];
    // K bias [token][8]: groups 0..3 (zero padded) twice, against the high and the low parts of the group sums of q
    __shared__ __attribute__((aligned(16))) half_t kb_lds[2][TILE * 8];
    __shared__ __attribute__((aligned(16))) half8_t q_lds[QLDS > 0 ? QLDS * QROWS : 1];
    __shared__ int s_pre[kMaxStreamAgents + 1], s_len[kMaxStreamAgents];

    const int wave = scalar(threadIdx.x / kWave);

    // ---- the range of tiles this workgroup takes: whole unit blockIdx (consecutive workgroups of one XCD share a KV
    // head), or an equal share of all tiles (consecutive shares on one XCD)
    const ChunkStream<QPOS, TILE> stream{s_pre, s_len};
    int x = 0, x1 = 1, per = 1, worker = 0;
    if constexpr (SHARES) {
        if (wave == 0) ChunkStream<QPOS, TILE>::fill(p, s_pre, s_len, threadIdx.x);
        __syncthreads();
        const int total = p.layers_in_call * scalar(s_pre[p.num_agents]), grid = gridDim.x;
        per = (total + grid - 1) / grid;
        worker = grid % kXcds == 0 ? (int)(blockIdx.x % kXcds) * (grid / kXcds) + (int)(blockIdx.x / kXcds) : (int)blockIdx.x;
        x = worker * per; // below total + grid: far inside 32 bits
        x1 = min(total, x + per);
        if (threadIdx.x == 0) p.shared[worker].slots = 0; // this thread writes it again when a unit goes on past the range
        if (x >= x1) return;
    }
    if constexpr (GK < 4) { // bias slots of groups the rows do not have: zero once (their q sums are zero too)
        static_assert(TILE * 8 % kChunkThreads == 0, "words of the two tiles' slots: the same number for every thread");
#pragma unroll
        for (int i = 0; i < TILE * 8; i += kChunkThreads) reinterpret_cast<uint32_t *>(&kb_lds[0][0])[i + threadIdx.x] = 0u;
        __syncthreads();
    }

    const int range_begin = x;
    while (x < x1) {
        // Everything derived from the thread's index is worked out anew for every part: kept from one to the next (the
        // compiler would lift it out of this loop) it costs two dozen registers that the tile loop does not have.
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & (kWave - 1), qn = lane % 32, h = lane / 32;
        ChunkUnit u;
        int begin = 0, tiles = 0, part_end, n;
        if constexpr (SHARES) {
            u = stream.locate(p, x, begin, tiles, n);
            part_end = min(tiles, begin + (x1 - x));
        } else {
            const int slot = blockIdx.x / kXcds, xcd = blockIdx.x % kXcds;
            const int unit = slot / p.q_tiles * kXcds + xcd;
            if (unit >= p.layers_in_call * p.num_agents * p.kv_heads) return;
            u.qt = slot % p.q_tiles;
            u.kvh = unit % p.kv_heads;
            u.agent = unit / p.kv_heads % p.num_agents;
            u.li = unit / (p.kv_heads * p.num_agents);
            part_end = 1;
        }
        // Row group; with KSPLIT 2 the half of a tile's tokens.  Waves w and w + 4 share a SIMD.  They are the two halves of one row
        // group where all groups have rows of the chunk, else neighbours are, so that the groups that have some spread over all
        // SIMDs.  Neighbours / halves w and w + 4: 2 tokens of two agents of up to 5,000, 192 + 128-wide, four layers 124 / 141
        // us, 9 of four of 2,600, 256-wide, five layers 199 / 221; 70 of four, 128-wide, all live but in the last tile, four layers 199 / 195.
        const bool all_live = KSPLIT == 1 || u.qt * QPOS + (ROWGROUPS - 1) * kRowsWave / NREP < p.q_len;
        const int rg = all_live ? wave % ROWGROUPS : wave / KSPLIT, my_sub = all_live ? wave / ROWGROUPS : wave % KSPLIT;
        // ---- this lane's query row: column qn of its wave's 32 (both halves of the wave hold the same row).  Asked for before
        // the length and the block table, which are two trips to memory for the first tile (0.3-0.6 us of every call).
        // Rows of q and of the output: a uniform place for the row tile and 32 bits per lane from there.
        const int64_t tile_row = (((int64_t)u.li * p.num_agents + u.agent) * p.q_len + u.qt * QPOS) * p.q_heads + u.kvh * NREP;
        auto row_in_tile = [&](int pos, int r) __attribute__((always_inline)) {
            uint32_t heads = p.q_heads;
            asm volatile("" : "+s"(heads)); // else it is moved to a vector register that is kept for the next part
            return (uint32_t)pos * heads + (uint32_t)(r % NREP);
        };
        const int my_row = rg * kRowsWave + qn;
        uint4 q_raw[GK][4];
        {
            const uint16_t *src = p.q + tile_row * DK + (uint64_t)row_in_tile(min(my_row / NREP, p.q_len - 1 - u.qt * QPOS), my_row) * DK + 32 * h;
#pragma unroll
            for (int g = 0; g < GK; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) q_raw[g][i] = *reinterpret_cast<const uint4 *>(src + kGroup * g + 8 * i);
        }
        if constexpr (!SHARES) n = scalar(clamped_length(p, u.agent));
        const int layer = p.layer_begin + u.li;
        const int window = p.per_layer_windows ? p.layer_window[u.li] : p.window;
        int t_begin, t_end;
        visible_range<QPOS, TILE>(p, n, window, u.qt, t_begin, t_end);
        const int part_t0 = t_begin + begin * TILE;
        const int part_t1 = SHARES ? min(t_end, t_begin + part_end * TILE) : t_end; // exclusive; may be <= part_t0

        // ---- KV tile staging: raw Q4 in registers one tile ahead.  A thread takes WPT consecutive words of one token's
        // K row and (the same ones when the rows are equally wide) of one token's V row; with rows that do not divide
        // evenly the last waves stage nothing
        const int32_t *table = p.block_table + (int64_t)u.agent * p.max_blocks;
        uint32_t kraw[SK::WPT], vraw[SV::WPT];
        uint32_t ksb[2], vsb[2]; // scale / bias bits of the group this thread unpacks
        // 16 consecutive lanes take 16 consecutive tokens (and the same part of the row): their 16-byte LDS stores of K
        // then fall into 16 different bank groups, like the operand reads
        const bool k_on = SK::ACTIVE == kChunkThreads || tid < SK::ACTIVE, v_on = SV::ACTIVE == kChunkThreads || tid < SV::ACTIVE;
        const int k_tok = k_on ? (tid % 16) + 16 * (tid / (16 * SK::TPR)) : 0, k_w0 = k_on ? ((tid / 16) % SK::TPR) * SK::WPT : 0;
        const int v_tok = v_on ? (tid % 16) + 16 * (tid / (16 * SV::TPR)) : 0, v_w0 = v_on ? ((tid / 16) % SV::TPR) * SV::WPT : 0;
        const uint32_t k_off = 4 * (k_tok * SK::WORDS + k_w0), v_off = 4 * (v_tok * SV::WORDS + v_w0);
        // the thread's place, worked out again: kept through the tile loop (or out of this one) it would cost registers
        auto lane_again = []() __attribute__((always_inline)) {
            int t = threadIdx.x;
            asm volatile("" : "+v"(t));
            return t & (kWave - 1);
        };
        // what follows from k_off or v_off is worked out where it is needed: kept, each would take a register through the tile loop
        auto fresh = [](uint32_t v) __attribute__((always_inline)) {
            asm volatile("" : "+v"(v));
            return v;
        };
        auto params_at = [&](uint32_t words_at) __attribute__((always_inline)) { return (fresh(words_at) >> 5) * 2; };
        // A block id outside the pool: the tile's (unconditional) loads go to the agent's own first block instead -- to
        // block 0 only if that id is outside the pool as well -- and everything they bring is discarded.
        const int own0 = scalar(table[0]);
        const int fallback_blk = own0 >= 0 && own0 < p.num_blocks ? own0 : 0;
        // Fetched well before it is needed: a trip to memory in the tile loop otherwise.  No branch (a load that may or may not be
        // in flight makes the compiler wait for all), and entries past the row are told apart where they are used.
        auto block_of = [&](int t0) __attribute__((always_inline)) { return table[min(t0 / kBlockTokens, p.max_blocks - 1)]; };
        auto tile_row0 = [&](int t0, int entry, bool &ok) __attribute__((always_inline)) {
            const int blk = scalar(entry);
            ok = blk >= 0 && blk < p.num_blocks && t0 / kBlockTokens < p.max_blocks;
            return (((int64_t)layer * p.num_blocks + (ok ? blk : fallback_blk)) * p.kv_heads + u.kvh) * kBlockTokens + (t0 % kBlockTokens);
        };
        auto load_words = [&](const uint32_t *src, auto &dst) __attribute__((always_inline)) {
            constexpr int N = sizeof(dst) / sizeof(uint32_t);
            if constexpr (N % 4 == 0) {
#pragma unroll
                for (int i = 0; i < N / 4; ++i) {
                    const uint4 t = *reinterpret_cast<const uint4 *>(src + 4 * i);
                    dst[4 * i] = t.x; dst[4 * i + 1] = t.y; dst[4 * i + 2] = t.z; dst[4 * i + 3] = t.w;
                }
            } else {
                const uint2 t = *reinterpret_cast<const uint2 *>(src);
                dst[0] = t.x; dst[1] = t.y;
            }
        };
        // a uniform base and a 32-bit byte offset per lane
        auto at = [](auto *base, uint32_t byte_off) __attribute__((always_inline)) {
            asm volatile("" : "+v"(byte_off)); // else base + offset is kept as one 64-bit pointer per lane and array
            return reinterpret_cast<decltype(base)>(reinterpret_cast<const char *>(base) + byte_off);
        };
        // threads without a share load row 0 of the tile again (a valid address) and never store
        auto load_k = [&](int64_t row0) __attribute__((always_inline)) {
            load_words(at(p.k_codes + row0 * SK::WORDS, k_off), kraw);
            const uint32_t params = params_at(k_off);
            ksb[0] = *at(p.k_scale + row0 * GK, params);
            ksb[1] = *at(p.k_bias + row0 * GK, params);
        };
        auto load_v = [&](int64_t row0) __attribute__((always_inline)) {
            load_words(at(p.v_codes + row0 * SV::WORDS, v_off), vraw);
            const uint32_t params = params_at(v_off);
            vsb[0] = *at(p.v_scale + row0 * GV, params);
            vsb[1] = *at(p.v_bias + row0 * GV, params);
        };
        // Dequantization of the staged rows happens one code word (8 dims, one 16-byte store) at a time, so that the
        // matrix loops below can take a word between their steps.  Rows of an unreachable block and rows at or past
        // t_end (never visible, possibly never written) become zeros, so that no stale bit pattern can reach an
        // accumulator.
        struct RowDequant {
            half2_t s2, s16, b2;
        };
        auto row_params = [&](const uint32_t (&sb)[2], bool ok) __attribute__((always_inline)) {
            RowDequant r;
            // bfloat16 parameters of binary16-range data convert exactly (8 significant bits into 11) unless they are
            // below 2^-14, where the difference is far below what binary16 operands resolve anyway
            const half_t s_in = BF ? (half_t)bf16_bits_to_float((uint16_t)sb[0]) : __builtin_bit_cast(half_t, (uint16_t)sb[0]);
            const half_t b_in = BF ? (half_t)bf16_bits_to_float((uint16_t)sb[1]) : __builtin_bit_cast(half_t, (uint16_t)sb[1]);
            const half_t s = ok ? s_in : (half_t)0.0f;
            const half_t b = ok ? b_in : (half_t)0.0f;
            r.s2 = half2_t{s, s};
            r.b2 = half2_t{b, b};
            r.s16 = r.s2 * half2_t{(half_t)0.0625f, (half_t)0.0625f};
            return r;
        };
        auto store_word = [&](half_t *dst, uint32_t raw, const RowDequant &r) __attribute__((always_inline)) {
            const uint32_t w8 = raw >> 8;
            const half2_t v0 = pk_fma(nibbles_lo(raw), r.s2, r.b2);     // dims 0, 4
            const half2_t v1 = pk_fma(nibbles_hi16(raw), r.s16, r.b2);  // dims 1, 5
            const half2_t v2 = pk_fma(nibbles_lo(w8), r.s2, r.b2);      // dims 2, 6
            const half2_t v3 = pk_fma(nibbles_hi16(w8), r.s16, r.b2);   // dims 3, 7
            *reinterpret_cast<uint4 *>(dst) = make_uint4(half2_to_bits(v0), half2_to_bits(v1), half2_to_bits(v2), half2_to_bits(v3));
        };
        auto store_codes = [&](uint32_t *dst, const uint32_t (&raw)[SK::WPT]) __attribute__((always_inline)) {
            if constexpr (SK::WPT % 4 == 0) {
#pragma unroll
                for (int w = 0; w < SK::WPT; w += 4)
                    *reinterpret_cast<uint4 *>(dst + w) = make_uint4(raw[w], raw[w + 1], raw[w + 2], raw[w + 3]);
            } else {
                *reinterpret_cast<uint2 *>(dst) = make_uint2(raw[0], raw[1]);
            }
        };
        // a code word as the A operand of a matrix instruction: the nibbles masked in place are binary16 subnormals
        // c 2^-24 (dims 0, 4, 2, 6 of the word) and 16 c 2^-24 (dims 1, 5, 3, 7)
        auto code_operand = [&](uint32_t w) __attribute__((always_inline)) {
            const uint32_t w8 = w >> 8;
            return __builtin_bit_cast(half8_t, make_uint4(w & 0x000F000Fu, w & 0x00F000F0u, w8 & 0x000F000Fu, w8 & 0x00F000F0u));
        };
        auto store_unpacked = [&](uint32_t *dst, uint32_t w) __attribute__((always_inline)) {
            *reinterpret_cast<half8_t *>(dst) = code_operand(w);
        };
        // scale and bias of a K row go to LDS beside the codes, written by the thread that holds the first word of the
        // group.  In token order: in the scores' order every wave worked out the place with 22 instructions a tile instead of 12.
        const bool k_params_writer = k_on && (k_w0 * 8) % kGroup == 0;
        auto store_k_params = [&](int b, const RowDequant &r) __attribute__((always_inline)) {
            const int at = (int)(fresh(k_off) / 4), tok = at / SK::WORDS, grp = at % SK::WORDS / 8;
            ks_lds[b][grp * TILE + tok] = r.s2.x;
            kb_lds[b][tok * 8 + grp] = r.b2.x;
            kb_lds[b][tok * 8 + 4 + grp] = r.b2.x;
        };
        auto row_ok = [&](int t0, int tok, bool ok_tile) __attribute__((always_inline)) { return ok_tile && (t0 + tok < t_end); };
        const int k_dst = KFULL ? (k_w0 * TILE + k_tok) * 4 : k_tok * KPITCH + k_w0, v_dst = v_tok * VPITCH + v_w0 * 8;
        constexpr int kWordStep = TILE * 4; // from one word's operands to the next one's

        // the first tile is on its way while the queries are unpacked
        const int t_last = part_t0 < part_t1 ? part_t0 + (part_t1 - 1 - part_t0) / TILE * TILE : 0; // start of the last tile
        const int second = min(part_t0 + TILE, t_last);
        bool ok_next = false, ok_cur = false;
        int64_t row_next = 0;
        if (part_t0 < part_t1) { // entry 0 of the table is there already
            const int entry0 = part_t0 < kBlockTokens ? own0 : block_of(part_t0), entry1 = second < kBlockTokens ? own0 : block_of(second);
            const int64_t row_a = tile_row0(part_t0, entry0, ok_cur);
            row_next = tile_row0(second, entry1, ok_next);
            load_k(row_a);
            load_v(row_a);
        }

        // ---- what this lane's row sees, and its query operand
        const bool wave_live = u.qt * QPOS + rg * kRowsWave / NREP < p.q_len; // the wave's first row; wave-uniform
        // rows past the chunk repeat its last position (and are not stored)
        auto row_sees = [&](int pos) __attribute__((always_inline)) { return n - (p.q_len - 1 - min(pos, p.q_len - 1)); };
        auto row_hides = [&](int vis) __attribute__((always_inline)) { return window > 0 && vis > window ? vis - window : 0; };
        // tokens inside [all_first, all_vis) are visible to every row of this wave and need no masks
        const int all_vis = row_sees(u.qt * QPOS + rg * kRowsWave / NREP);
        const int all_first = row_hides(row_sees(u.qt * QPOS + (rg * kRowsWave + kRowsWave - 1) / NREP));
        half8_t qop[QREG]; // [matrix instruction 4 g + i]: the 8 dims of word 8 g + 4 h + i
        half8_t qsop;         // lower half of the wave: group sums of q, high parts in slots 0..3, low parts in 4..7; else 0
        {
            float qs[GK];
#pragma unroll
            for (int g = 0; g < GK; ++g) {
                qs[g] = 0.0f;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // 8 dims in the order the nibble masks emit them: 0,4,1,5,2,6,3,7; the odd ones divided by 16
                    // because their codes arrive 16 times larger
                    const uint4 raw = q_raw[g][i];
                    const half2_t e01 = bits_to_half2(raw.x), e23 = bits_to_half2(raw.y);
                    const half2_t e45 = bits_to_half2(raw.z), e67 = bits_to_half2(raw.w);
                    const half_t sixteenth = (half_t)0.0625f;
                    const half8_t v = half8_t{e01.x, e45.x, e01.y * sixteenth, e45.y * sixteenth,
                                              e23.x, e67.x, e23.y * sixteenth, e67.y * sixteenth};
                    qs[g] += ((float)e01.x + (float)e01.y) + ((float)e23.x + (float)e23.y) +
                             ((float)e45.x + (float)e45.y) + ((float)e67.x + (float)e67.y);
                    if (4 * g + i < QREG) qop[4 * g + i < QREG ? 4 * g + i : 0] = v;
                    else if (my_sub == 0) q_lds[(4 * g + i - QREG) * QROWS + rg * kWave + lane] = v;
                }
            }
            half_t part[8];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float v = g < GK ? xor32_sum(qs[g < GK ? g : 0]) : 0.0f;
                const half_t hi = (half_t)v;
                part[g] = h == 0 ? hi : (half_t)0.0f;
                part[4 + g] = h == 0 ? (half_t)(v - (float)hi) : (half_t)0.0f;
            }
            qsop = half8_t{part[0], part[1], part[2], part[3], part[4], part[5], part[6], part[7]};
        }
        float16_t o_acc[DTILES]; // O^T: lane column = query row, register i = row position 8 (i/4) + 4 h + i%4
#pragma unroll
        for (int d = 0; d < DTILES; ++d)
#pragma unroll
            for (int i = 0; i < 16; ++i) o_acc[d][i] = 0.0f;
        // m_run: the reference the exponentials are taken against.  It moves only when a tile's maximum exceeds it by more than
        // kSlack (log2 units), so the accumulators are rescaled a few times per row, not once per tile.
        // (A reference that is the row's maximum gives the largest weight without rounding.  Error against 64 bits, 512 tokens behind
        // 8,000, 256-wide, with a denominator of rounded weights, slack 3 / 4 / 5 / 8: 3.27e-4 / 3.31e-4 / 3.35e-4 / 3.5e-4; 8 would be 2 % faster.)
        constexpr float kSlack = 3.0f;
        float m_run = kNegBig, l_run = 0.0f; // l_run: this lane's tokens only

        // operand reads: K row of M row qn; V_hat by the transposing read (token 8 h + 2 e (+ 1), dims 16 (lane/16 % 2) + 4 c)
        const int m_token = 16 * (qn / 16) + 8 * ((qn / 4) % 2) + 2 * (qn % 4) + (qn / 8) % 2;
        const int k_lane = KFULL ? 4 * h * kWordStep + m_token * 4 : m_token * KPITCH + 4 * h;
        constexpr int kPiece = KFULL ? kSub * 4 : kSub * KPITCH; // from one 32-token piece to the next
        const int v_lane = (8 * h + 2 * ((lane % 16) / 4)) * VPITCH + 16 * ((lane / 16) % 2) + 4 * (lane % 4);

        // One barrier per tile.  Step i takes the scores of tile i and, while its softmax is worked out, the product of tile
        // i - 1; it stages V of tile i and K of tile i + 1 and asks for the tiles behind those.
        int buf = 0, t0 = part_t0, entry_ahead = -1;
        const int sub = my_sub * NP; // this wave's NP pieces of 32 tokens
        float16_t zero;
        half8_t pt[2 * NP]; // P^T of the tile before, [16-token step]
#pragma unroll
        for (int i = 0; i < 16; ++i) zero[i] = 0.0f;

        // ---- S^T = sum_g s_g (C_g Q_g^T) + b Qsum^T in binary32, in units of 2^-24
        constexpr float kUnit = 0x1p-24f;
        auto scores = [&](float16_t (&st)[NP], bool more, int64_t row_ahead) __attribute__((always_inline)) {
            const uint32_t *k_row = k_lds[buf] + sub * kPiece + k_lane;
            const half_t *ks_row = ks_lds[buf] + sub * kSub + 8 * (lane_again() / 32);
            const half_t *kb_row = kb_lds[buf] + (sub * kSub + (KFULL ? (int)(fresh(k_lane) / 4) % kSub : m_token)) * 8;
            auto q_operand = [&](auto index) __attribute__((always_inline)) { // matrix instruction 4 group + i
                constexpr int k = index.value;
                if constexpr (k < QREG) return qop[k];
                else return q_lds[(k - QREG) * QROWS + rg * kWave + lane];
            };
            // this lane's token: the operands of the kKeysAhead matrix instructions to come, or the code words 8 g + 4 h .. + 3
            constexpr int kKeysAhead = 2;
            uint4 words[NP], keys[kKeysAhead][NP];
            auto load_keys = [&](int k, int n) __attribute__((always_inline)) { // matrix instruction k of piece n
                return *reinterpret_cast<const uint4 *>(k_row + n * kPiece + (8 * (k / 4) + k % 4) * kWordStep);
            };
#pragma unroll
            for (int n = 0; n < NP; ++n) {
                const half8_t ba = *reinterpret_cast<const half8_t *>(kb_row + n * kSub * 8);
                st[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ba, qsop, zero, 0, 0, 0);
            }
#pragma unroll
            for (int n = 0; n < NP; ++n) {
                if constexpr (KFULL) {
#pragma unroll
                    for (int k = 0; k < kKeysAhead; ++k) keys[k][n] = load_keys(k, n);
                } else {
                    words[n] = *reinterpret_cast<const uint4 *>(k_row + n * kPiece);
                }
            }
            half8_t qk = q_operand(Index<0>());
            const RowDequant kr = row_params(ksb, row_ok(t0 + TILE, (int)(fresh(k_off) / (4 * SK::WORDS)), ok_next && more));
            const RowDequant vr = row_params(vsb, row_ok(t0, (int)(fresh(v_off) / (4 * SV::WORDS)), ok_cur));
            if constexpr (!KFULL) {
                if (k_on) store_codes(k_lds[buf ^ 1] + k_dst, kraw);
            }
            if (k_params_writer) store_k_params(buf ^ 1, kr);
            float16_t d[NP];
            uint4 sc[NP], sc1[NP]; // scales of the lane's first and last 8 scores
            uint32_t w4[NP][4];
            unrolled<4 * GK>([&](auto index) __attribute__((always_inline)) {
                constexpr int k = index.value, g = k / 4, i = k % 4;
                if constexpr (i == 0) {
#pragma unroll
                    for (int n = 0; n < NP; ++n) {
                        if constexpr (!KFULL) {
                            w4[n][0] = words[n].x; w4[n][1] = words[n].y; w4[n][2] = words[n].z; w4[n][3] = words[n].w;
                        }
                        d[n] = zero;
                    }
                }
                const half8_t qi = qk;
                if constexpr (k + 1 < 4 * GK) qk = q_operand(Index<k + 1>());
#pragma unroll
                for (int n = 0; n < NP; ++n) {
                    if constexpr (i == 2) sc[n] = *reinterpret_cast<const uint4 *>(ks_row + g * TILE + n * kSub);
                    if constexpr (i == 3) sc1[n] = *reinterpret_cast<const uint4 *>(ks_row + g * TILE + n * kSub + 16);
                    half8_t a;
                    if constexpr (KFULL) {
                        a = __builtin_bit_cast(half8_t, keys[k % kKeysAhead][n]);
                        if constexpr (k + kKeysAhead < 4 * GK) keys[k % kKeysAhead][n] = load_keys(k + kKeysAhead, n);
                    } else {
                        if constexpr (i == 3 && g + 1 < GK) words[n] = *reinterpret_cast<const uint4 *>(k_row + n * kPiece + 8 * (g + 1));
                        a = code_operand(w4[n][i]);
                    }
                    d[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, qi, d[n], 0, 0, 0);
                }
                // the next tile's K, then this one's V, a word at a time; behind each its registers are free for the tile after that
                constexpr int kWords = (KFULL ? SK::WPT : 0) + SV::WPT, kFirstV = kWords - SV::WPT;
                unrolled<kWords>([&](auto word) __attribute__((always_inline)) {
                    constexpr int w = word.value;
                    if constexpr (w * 4 * GK / kWords == k) {
                        if constexpr (w < kFirstV) {
                            if (k_on) store_unpacked(k_lds[buf ^ 1] + k_dst + w * kWordStep, kraw[w]);
                        } else {
                            if (v_on) store_word(v_lds[buf] + v_dst + 8 * (w - kFirstV), vraw[w - kFirstV], vr);
                        }
                    }
                });
                constexpr int kAfterK = kFirstV > 0 ? (kFirstV - 1) * 4 * GK / kWords : 0;
                if constexpr (k == kAfterK) load_k(row_ahead);
                if constexpr (k == (kWords - 1) * 4 * GK / kWords) {
                    load_v(row_next);
                    entry_ahead = block_of(min(t0 + 3 * TILE, t_last)); // for the next step: a trip to memory in every one otherwise
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (i == 3) {
#pragma unroll
                    for (int n = 0; n < NP; ++n) {
                        const uint32_t s8[8] = {sc[n].x, sc[n].y, sc[n].z, sc[n].w, sc1[n].x, sc1[n].y, sc1[n].z, sc1[n].w};
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const half2_t sh = bits_to_half2(s8[4 * (e / 8) + e % 4]); // tokens 2 (e % 4) and one more of 8
                            const float prev = g == 0 ? st[n][e] * kUnit : st[n][e]; // the bias term enters in the products' unit
                            st[n][e] = fmaf((float)((e & 4) ? sh.y : sh.x), d[n][e], prev);
                        }
                        // pinned: else the multiplies of all groups sink to the scores' first use and every product stays live
#pragma unroll
                        for (int e = 0; e < 16; e += 8)
                            asm volatile("" : "+v"(st[n][e]), "+v"(st[n][e + 1]), "+v"(st[n][e + 2]), "+v"(st[n][e + 3]), "+v"(st[n][e + 4]),
                                         "+v"(st[n][e + 5]), "+v"(st[n][e + 6]), "+v"(st[n][e + 7]));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        };

        auto stage_keys = [&](int b, const RowDequant &kr) __attribute__((always_inline)) {
            if (k_params_writer) store_k_params(b, kr);
            if constexpr (KFULL) {
#pragma unroll
                for (int w = 0; w < SK::WPT; ++w)
                    if (k_on) store_unpacked(k_lds[b] + k_dst + w * kWordStep, kraw[w]);
            } else if (k_on) {
                store_codes(k_lds[b] + k_dst, kraw);
            }
        };
        // what `scores` does beside its matrix instructions: ksb and kraw hold tile t0 + TILE, vsb and vraw tile t0
        auto stage_only = [&](bool more, int64_t row_ahead) __attribute__((always_inline)) {
            const RowDequant kr = row_params(ksb, row_ok(t0 + TILE, (int)(fresh(k_off) / (4 * SK::WORDS)), ok_next && more));
            const RowDequant vr = row_params(vsb, row_ok(t0, (int)(fresh(v_off) / (4 * SV::WORDS)), ok_cur));
            stage_keys(buf ^ 1, kr);
            load_k(row_ahead);
#pragma unroll
            for (int w = 0; w < SV::WPT; ++w)
                if (v_on) store_word(v_lds[buf] + v_dst + 8 * w, vraw[w], vr);
            load_v(row_next);
            entry_ahead = block_of(min(t0 + 3 * TILE, t_last));
        };

        // ---- online softmax of the scores per query row (lane column) and their P^T, in kItems pieces
        struct Softmax {
            float mx = kNegBig, m_new = 0.0f, sum = 0.0f;
            bool moved = false;
            uint32_t next[8 * NP];
        };
        constexpr int kItems = 10 * NP + 1;
        auto softmax_item = [&](auto index, Softmax &x, const float16_t (&st)[NP], float zs) __attribute__((always_inline)) {
            constexpr int j = index.value;
            if constexpr (j < 2 * NP) { // the maximum, before the scale is applied (which is positive)
#pragma unroll
                for (int i = 0; i < 8; ++i) x.mx = fmaxf(x.mx, st[j / 2][8 * (j % 2) + i]);
            } else if constexpr (j == 2 * NP) {
                x.mx = xor32_max(x.mx * zs); // the row's tokens live in two lanes
                const bool mine = x.mx > m_run + kSlack; // of this row alone: its bits do not depend on its neighbours
                x.m_new = mine ? x.mx : m_run;
                x.moved = __builtin_amdgcn_ballot_w64(mine) != 0ull;
            } else {
                constexpr int e = j - 2 * NP - 1;
                const float a = __builtin_amdgcn_exp2f(fmaf(st[e / 8][2 * (e % 8)], zs, -x.m_new));
                const float b = __builtin_amdgcn_exp2f(fmaf(st[e / 8][2 * (e % 8) + 1], zs, -x.m_new));
                const half2_t w = half2_t{(half_t)a, (half_t)b};
                x.sum += a; // the weights themselves: a long tail of weights that round to little or nothing still counts
                x.sum += b;
                x.next[e] = half2_to_bits(w);
                asm volatile("" : "+v"(x.next[e]), "+v"(x.sum)); // else the additions are put off and every weight stays live
            }
        };
        auto softmax_done = [&](const Softmax &x) __attribute__((always_inline)) {
            m_run = x.m_new;
            l_run += x.sum;
#pragma unroll
            for (int s = 0; s < 2 * NP; ++s)
                pt[s] = __builtin_bit_cast(half8_t, make_uint4(x.next[4 * s], x.next[4 * s + 1], x.next[4 * s + 2], x.next[4 * s + 3]));
        };

        // ---- O^T += V_hat^T P^T of the tile before, the operand reads ahead; between the matrix instructions the softmax of the
        // scores (SOFT), whose P^T the next step multiplies
        auto product = [&](auto soft, const float16_t (&st)[NP], float zs) __attribute__((always_inline)) {
            constexpr bool SOFT = soft.value;
            constexpr int kPerTile = 2 * NP, kSteps = kPerTile * DTILES, kAhead = 2;
            const half_t *v_row = v_lds[buf ^ 1] + sub * kSub * VPITCH + fresh(v_lane);
            auto load_va = [&](int step) __attribute__((always_inline)) { // step = 2 NP * dim tile + 16-token step
                const half_t *src = v_row + (step % kPerTile) * 16 * VPITCH + (step / kPerTile) * 32;
                const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)src);
                const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(src + VPITCH));
                return __builtin_bit_cast(half8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            };
            half8_t va[kAhead];
#pragma unroll
            for (int s = 0; s < kAhead; ++s) va[s] = load_va(s);
            Softmax x;
            unrolled<kSteps>([&](auto index) __attribute__((always_inline)) {
                constexpr int s = index.value;
                const half8_t a = va[s % kAhead];
                if constexpr (s + kAhead < kSteps) va[s % kAhead] = load_va(s + kAhead);
                o_acc[s / kPerTile] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, pt[s % kPerTile], o_acc[s / kPerTile], 0, 0, 0);
                if constexpr (SOFT) {
                    constexpr int first = (s * kItems + kSteps - 1) / kSteps, last = ((s + 1) * kItems + kSteps - 1) / kSteps;
                    unrolled<last - first>([&](auto j) __attribute__((always_inline)) { softmax_item(Index<first + j.value>(), x, st, zs); });
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (SOFT) {
                if (__builtin_expect(x.moved, 0)) { // rare after a unit's first tiles
                    const float alpha = __builtin_amdgcn_exp2f(m_run - x.m_new);
                    l_run *= alpha;
#pragma unroll
                    for (int d = 0; d < DTILES; ++d)
#pragma unroll
                        for (int i = 0; i < 16; ++i) o_acc[d][i] *= alpha;
                }
                softmax_done(x);
            }
        };
        if (part_t0 < part_t1) {
            stage_keys(0, row_params(ksb, row_ok(part_t0, k_tok, ok_cur)));
            load_k(row_next);
            entry_ahead = block_of(min(part_t0 + 2 * TILE, t_last));
            __syncthreads();
            auto look_ahead = [&](int64_t &row_ahead, bool &ok_ahead) __attribute__((always_inline)) {
                const int t_ahead = min(t0 + 2 * TILE, t_last); // past the end: the last tile again, never used
                row_ahead = tile_row0(t_ahead, entry_ahead, ok_ahead);
            };
            auto end_step = [&](int64_t row_ahead, bool ok_ahead) __attribute__((always_inline)) {
                ok_cur = ok_next;
                ok_next = ok_ahead;
                row_next = row_ahead;
                t0 += TILE;
                __syncthreads(); // every wave is done with these buffers and has filled its part of the others
                buf ^= 1;
            };
            int64_t row_ahead;
            bool ok_ahead;
            auto step = [&](auto first) __attribute__((always_inline)) {
                const int ts = t0 + kSub * sub;
                look_ahead(row_ahead, ok_ahead);
                float16_t st[NP];
                scores(st, t0 + TILE < part_t1, row_ahead);
                // tokens that every row of the wave sees need no masks; the path with masks assumes nothing of the scale
                float zs = p.score_scale / kUnit;
                if (__builtin_expect(!(ok_cur && ts >= all_first && ts + NP * kSub <= all_vis && p.score_scale > 0.0f), 0)) {
                    const int ln = lane_again();
                    const int row_vis = row_sees(u.qt * QPOS + (rg * kRowsWave + ln % 32) / NREP), row_first = row_hides(row_vis);
#pragma unroll
                    for (int n = 0; n < NP; ++n)
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int t = ts + kSub * n + 16 * (i / 8) + 8 * (ln / 32) + 2 * (i % 4) + ((i / 4) & 1);
                            const float z = st[n][i] * zs;
                            st[n][i] = ok_cur && t < row_vis && t >= row_first ? z : 2.0f * kNegBig; // a weight of 0 against any reference
                        }
                    zs = 1.0f;
                }
                if constexpr (first.value) {
                    Softmax x;
                    unrolled<kItems>([&](auto j) __attribute__((always_inline)) { softmax_item(j, x, st, zs); });
                    softmax_done(x);
                } else {
                    product(Flag<true>(), st, zs);
                }
                end_step(row_ahead, ok_ahead);
            };
            if (wave_live) {
                step(Flag<true>()); // no tile before: no product
                while (t0 < part_t1) step(Flag<false>());
                float16_t none[NP];
                product(Flag<false>(), none, 0.0f);
            } else { // no rows of the chunk: this wave only does its part of the staging, and leaves the rest of its SIMD to the others
                do {
                    look_ahead(row_ahead, ok_ahead);
                    stage_only(t0 + TILE < part_t1, row_ahead);
                    end_step(row_ahead, ok_ahead);
                } while (t0 < part_t1);
            }
        }

        float l_tot = xor32_sum(l_run);
        if constexpr (KSPLIT == 2) if (part_t1 - part_t0 > kSub * NP) { // else the upper half has seen no token
            // The upper half of the waves hands its sums to the lower one through the V buffers, a few dim tiles at a
            // time; the maxima and denominators travel in the K buffers.
            constexpr int MT = (int)(2 * TILE * VPITCH * sizeof(half_t) / (ROWGROUPS * kWave * 16 * sizeof(float))) < DTILES
                                   ? (int)(2 * TILE * VPITCH * sizeof(half_t) / (ROWGROUPS * kWave * 16 * sizeof(float))) : DTILES;
            static_assert(MT >= 1, "room for one dim tile");
            const int ln = lane_again();
            float *ml = reinterpret_cast<float *>(&k_lds[0][0]);
            float *xch = reinterpret_cast<float *>(&v_lds[0][0]);
            if (my_sub == 1 && wave_live) {
                ml[(rg * 2) * kWave + ln] = m_run;
                ml[(rg * 2 + 1) * kWave + ln] = l_tot;
            }
            __syncthreads();
            float w_lo = 1.0f, w_hi = 0.0f;
            if (my_sub == 0 && wave_live) {
                const float m_hi = ml[(rg * 2) * kWave + ln], l_hi = ml[(rg * 2 + 1) * kWave + ln];
                const float m_new = fmaxf(m_run, m_hi);
                w_lo = __builtin_amdgcn_exp2f(m_run - m_new);
                w_hi = __builtin_amdgcn_exp2f(m_hi - m_new);
                l_tot = fmaf(l_hi, w_hi, l_tot * w_lo);
                m_run = m_new;
            }
#pragma unroll
            for (int d0 = 0; d0 < DTILES; d0 += MT) {
                if (my_sub == 1 && wave_live) {
#pragma unroll
                    for (int d = d0; d < d0 + MT && d < DTILES; ++d)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            *reinterpret_cast<float4_t *>(xch + (((rg * MT + d - d0) * 4 + j) * kWave + ln) * 4) =
                                float4_t{o_acc[d][4 * j], o_acc[d][4 * j + 1], o_acc[d][4 * j + 2], o_acc[d][4 * j + 3]};
                }
                __syncthreads();
                if (my_sub == 0 && wave_live) {
#pragma unroll
                    for (int d = d0; d < d0 + MT && d < DTILES; ++d)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float4_t v = *reinterpret_cast<const float4_t *>(xch + (((rg * MT + d - d0) * 4 + j) * kWave + ln) * 4);
#pragma unroll
                            for (int e = 0; e < 4; ++e) o_acc[d][4 * j + e] = fmaf(v[e], w_hi, o_acc[d][4 * j + e] * w_lo);
                        }
                }
                __syncthreads();
            }
        }

        const bool whole = !SHARES || (begin == 0 && part_end == tiles);
        if (wave_live && my_sub == 0) {
            if (whole) { // ---- normalise and store
                const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
                const int ln = lane_again();
                const int r = rg * kRowsWave + ln % 32;
                const bool store = u.qt * QPOS + r / NREP < p.q_len;
                uint16_t *dst = p.out + tile_row * DV + (uint64_t)row_in_tile(r / NREP, r) * DV;
#pragma unroll
                for (int d = 0; d < DTILES; ++d)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float a = o_acc[d][4 * j] * inv, b = o_acc[d][4 * j + 1] * inv;
                        const float e = o_acc[d][4 * j + 2] * inv, f = o_acc[d][4 * j + 3] * inv;
                        if (store) store_row_quad(dst + 32 * d + 8 * j, ln / 32, a, b, e, f);
                    }
            } else { // ---- this workgroup's part of a shared unit, un-normalised
                const int64_t rec = ((int64_t)worker * 2 + (x - begin > range_begin ? 1 : 0)) * ROWGROUPS + rg;
                const int ln = lane_again();
                float *acc = p.part_acc + (rec * (DV / 8) * kWave + ln) * 4;
#pragma unroll
                for (int d = 0; d < DTILES; ++d)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        *reinterpret_cast<float4_t *>(acc + (d * 4 + j) * kWave * 4) =
                            float4_t{o_acc[d][4 * j], o_acc[d][4 * j + 1], o_acc[d][4 * j + 2], o_acc[d][4 * j + 3]};
                if (ln < 32) *reinterpret_cast<float2 *>(p.part_ml + (rec * kRowsWave + ln) * 2) = make_float2(m_run, l_tot);
            }
        }
        if (SHARES && threadIdx.x == 0 && begin == 0 && part_end < tiles) {
            ChunkShared *s = p.shared + worker;
            s->slots = (x + tiles - 1) / per - worker + 1;
            s->first_record = worker * 2 + (x > range_begin ? 1 : 0);
            s->qt = u.qt;
            s->kvh = u.kvh;
            s->token_row = ((int64_t)u.li * p.num_agents + u.agent) * p.q_len;
        }
        x += SHARES ? part_end - begin : 1;
        // A part of no tokens has had no barrier, and the next one may place the row groups differently: a wave that is late would
        // write this part's queries over the next one's.
        if constexpr (SHARES && KSPLIT == 2) if (part_t0 >= part_t1) __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------- merging shared units

constexpr int kMergeThreads = 256;
constexpr int kMergeQuads = 2; // float4 pieces of a lane that a wave merges at a time
constexpr int kMergeBatch = 4; // records whose pieces are asked for together

// pieces a unit's merge is cut into: one wave each
template <int DV, int ROWGROUPS>
constexpr int merge_items() { return ROWGROUPS * (DV / 8 / kMergeQuads); }
template <int DV, int ROWGROUPS>
constexpr int merge_parts() { return merge_items<DV, ROWGROUPS>() / (kMergeThreads / kWave); }

// The unit that begins in worker w's range and goes on past it: workgroups (w, part) merge its records in worker order.
// Reading the records once is all there is to do, so every wave has the loads of four records in flight, and takes two pieces
// of each: of what was tried (records at a time x pieces: 2 x 4, 4 x 4, 8 x 2, 4 x 2) one agent of 8,000 tokens, 256-wide,
// two layers takes 258.2, 261.0, 254.8, 254.4 us, four agents of up to 6,000, 128-wide, four layers 202.5, 203.3, 205.7, 201.1
// (two records at a time behind a first pass over the maxima: 260.3 and 202.9).
template <int DV, int NREP, int ROWGROUPS>
__global__ __launch_bounds__(kMergeThreads) void chunk_merge_kernel(ChunkParams p)
{
    constexpr int QPOS = ROWGROUPS * kRowsWave / NREP, PARTS = merge_parts<DV, ROWGROUPS>();
    constexpr int kQuads = DV / 8; // float4 pieces per lane and record
    static_assert(merge_items<DV, ROWGROUPS>() % (kMergeThreads / kWave) == 0, "whole workgroups");
    const int worker = blockIdx.x / PARTS, part = blockIdx.x % PARTS;
    const ChunkShared u = p.shared[worker];
    if (u.slots == 0) return;
    const int lane = threadIdx.x & (kWave - 1), wave = scalar(threadIdx.x / kWave), qn = lane % 32, h = lane / 32;
    const int item = part * (kMergeThreads / kWave) + wave;
    const int rg = item / (kQuads / kMergeQuads), quad0 = item % (kQuads / kMergeQuads) * kMergeQuads;
    if (u.qt * QPOS + rg * kRowsWave / NREP >= p.q_len) return; // a row group past the chunk left no record
    auto record = [&](int s) { return (int64_t)(s == 0 ? u.first_record : (worker + s) * 2) * ROWGROUPS + rg; };
    auto max_and_sum = [&](int s) { return *reinterpret_cast<const float2 *>(p.part_ml + (record(s) * kRowsWave + qn) * 2); };
    // kBatch records at a time, everything of them asked for together: a unit of that many costs one trip to memory.  The
    // reference moves batch by batch.
    float m_ref = kNegBig, l = 0.0f;
    float4_t o[kMergeQuads];
#pragma unroll
    for (int k = 0; k < kMergeQuads; ++k) o[k] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
    for (int s0 = 0; s0 < u.slots; s0 += kMergeBatch) {
        float2 ml[kMergeBatch];
        float4_t v[kMergeBatch][kMergeQuads];
#pragma unroll
        for (int b = 0; b < kMergeBatch; ++b) {
            const int s = s0 + b < u.slots ? s0 + b : u.slots - 1; // repeats of the last record are not used
            ml[b] = max_and_sum(s);
            const float4_t *src = reinterpret_cast<const float4_t *>(p.part_acc) + (record(s) * kQuads + quad0) * kWave + lane;
#pragma unroll
            for (int k = 0; k < kMergeQuads; ++k) v[b][k] = src[k * kWave];
        }
        if (s0 + kMergeBatch > u.slots) { // the repeats get no weight, and nothing to give it to: zero times an infinite sum is NaN
            asm volatile(""); // a branch: whole batches do not pay for the selects
#pragma unroll
            for (int b = 1; b < kMergeBatch; ++b)
                if (s0 + b >= u.slots) {
                    ml[b].y = 0.0f;
#pragma unroll
                    for (int k = 0; k < kMergeQuads; ++k) v[b][k] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
                }
        }
        float m_new = m_ref;
#pragma unroll
        for (int b = 0; b < kMergeBatch; ++b)
            if (ml[b].y > 0.0f) m_new = fmaxf(m_new, ml[b].x);
        const float keep = __builtin_amdgcn_exp2f(m_ref - m_new); // 1 when the reference stays
        m_ref = m_new;
        l *= keep;
#pragma unroll
        for (int k = 0; k < kMergeQuads; ++k) o[k] *= keep;
#pragma unroll
        for (int b = 0; b < kMergeBatch; ++b) {
            const float wgt = ml[b].y > 0.0f ? __builtin_amdgcn_exp2f(ml[b].x - m_ref) : 0.0f;
            l = fmaf(ml[b].y, wgt, l);
#pragma unroll
            for (int k = 0; k < kMergeQuads; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e) o[k][e] = fmaf(v[b][k][e], wgt, o[k][e]);
        }
    }
    const float inv = l > 0.0f ? 1.0f / l : 0.0f;
    const int r = rg * kRowsWave + qn, c = u.qt * QPOS + r / NREP;
    if (c >= p.q_len) return;
    uint16_t *dst = p.out + ((u.token_row + c) * p.q_heads + u.kvh * NREP + r % NREP) * DV + 8 * quad0;
#pragma unroll
    for (int k = 0; k < kMergeQuads; ++k) store_row_quad(dst + 8 * k, h, o[k][0] * inv, o[k][1] * inv, o[k][2] * inv, o[k][3] * inv);
}

// ---------------------------------------------------------------------------------------------- launch

ChunkSizes chunk_sizes(const q4kv_spec &s, int num_agents, int q_len, int layers, int compute_units)
{
    return ChunkSizes{(int64_t)layers * num_agents * s.num_kv_heads, (int64_t)q_len * (s.num_q_heads / s.num_kv_heads), compute_units};
}

template <int DK, int DV, int NREP, int KSPLIT, bool SHARES>
hipError_t launch_chunk_k(const AttentionArgs &a, hipStream_t stream)
{
    constexpr int ROWGROUPS = kChunkWaves / KSPLIT;
    constexpr int QPOS = ROWGROUPS * kRowsWave / NREP;
    ChunkParams p;
    p.k_codes = a.k.codes; p.k_scale = a.k.scale; p.k_bias = a.k.bias;
    p.v_codes = a.v.codes; p.v_scale = a.v.scale; p.v_bias = a.v.bias;
    p.q = a.q; p.out = a.out; p.block_table = a.block_table; p.seq_len = a.seq_len;
    p.num_blocks = a.k.num_blocks; p.kv_heads = a.spec.num_kv_heads; p.q_heads = a.spec.num_q_heads;
    p.num_agents = a.num_agents; p.max_blocks = a.max_blocks; p.max_seq_len = a.max_seq_len;
    p.window = a.window; p.q_len = a.q_len;
    p.per_layer_windows = a.layer_window != nullptr;
    if (p.per_layer_windows && a.layers_in_call == 1) {
        p.window = a.layer_window[0];
        p.per_layer_windows = 0;
    }
    for (int i = 0; i < kMaxChunkWindowLayers; ++i)
        p.layer_window[i] = (p.per_layer_windows && i < a.layers_in_call) ? a.layer_window[i] : 0;
    p.layer_begin = a.layer_begin; p.layers_in_call = a.layers_in_call;
    p.q_tiles = (a.q_len + QPOS - 1) / QPOS;
    p.score_scale = a.sm_scale * kLog2e;
    p.part_acc = a.part_acc; p.part_ml = a.part_ml;
    p.shared = reinterpret_cast<ChunkShared *>(a.part_ml + 2 * (size_t)a.chunk_workers * ROWGROUPS * kRowsWave * 2);
    const int64_t units = (int64_t)a.layers_in_call * a.num_agents * a.spec.num_kv_heads;
    const int64_t grid = SHARES ? a.chunk_workers : (units + kXcds - 1) / kXcds * kXcds * p.q_tiles;
    if (grid <= 0) return hipSuccess;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    if (a.spec.param_format == Q4KV_PARAMS_BF16)
        hipLaunchKernelGGL((chunk_attention_kernel<DK, DV, NREP, KSPLIT, SHARES, true>), dim3((unsigned)grid), dim3(kChunkThreads), 0, stream, p);
    else
        hipLaunchKernelGGL((chunk_attention_kernel<DK, DV, NREP, KSPLIT, SHARES, false>), dim3((unsigned)grid), dim3(kChunkThreads), 0, stream, p);
    if constexpr (SHARES)
        hipLaunchKernelGGL((chunk_merge_kernel<DV, NREP, ROWGROUPS>), dim3((unsigned)grid * merge_parts<DV, ROWGROUPS>()),
                           dim3(kMergeThreads), 0, stream, p);
    return hipGetLastError();
}

template <int DK, int DV, int NREP>
hipError_t launch_chunk_t(const AttentionArgs &a, hipStream_t stream)
{
    int tokens[kMaxChunkWindowLayers]; // what a workgroup sees; one entry unless the layers have windows of their own
    const int n = a.layer_window ? a.layers_in_call : 1;
    for (int i = 0; i < n; ++i) tokens[i] = visible_tokens(a.max_seq_len, a.layer_window ? a.layer_window[i] : a.window, a.q_len, NREP);
    const ChunkSizes sizes = chunk_sizes(a.spec, a.num_agents, a.q_len, a.layers_in_call, a.compute_units);
    // a.chunk_workers > 0: the workspace holds two records for each of that many workgroups
    const bool shares = a.chunk_workers > 0 && n == 1 && shares_pay(sizes, DK, tokens[0]);
    const int rows = shares ? rows_shared(sizes, tokens[0]) : rows_alone(sizes, tokens, n);
    if (shares) return rows == 256 ? launch_chunk_k<DK, DV, NREP, 1, true>(a, stream) : launch_chunk_k<DK, DV, NREP, 2, true>(a, stream);
    return rows == 256 ? launch_chunk_k<DK, DV, NREP, 1, false>(a, stream) : launch_chunk_k<DK, DV, NREP, 2, false>(a, stream);
}

template <int DK, int DV>
hipError_t launch_chunk_d(const AttentionArgs &a, int n_rep, hipStream_t stream)
{
    switch (n_rep) {
    case 1: return launch_chunk_t<DK, DV, 1>(a, stream);
    case 2: return launch_chunk_t<DK, DV, 2>(a, stream);
    case 4: return launch_chunk_t<DK, DV, 4>(a, stream);
    case 8: return launch_chunk_t<DK, DV, 8>(a, stream);
    default: return hipErrorInvalidValue;
    }
}

} // namespace

// The file is compiled once for each key width (Q4KV_CHUNK_WIDTH): 32 kernels a time, all four at once.
template <int DK>
hipError_t launch_chunk_width(const AttentionArgs &a, int n_rep, hipStream_t stream);
template <>
hipError_t launch_chunk_width<Q4KV_CHUNK_WIDTH>(const AttentionArgs &a, int n_rep, hipStream_t stream)
{
    return launch_chunk_d<Q4KV_CHUNK_WIDTH, Q4KV_CHUNK_WIDTH == 192 ? 128 : Q4KV_CHUNK_WIDTH>(a, n_rep, stream);
}

#if Q4KV_CHUNK_WIDTH == 64
template <> hipError_t launch_chunk_width<128>(const AttentionArgs &a, int n_rep, hipStream_t stream);
template <> hipError_t launch_chunk_width<192>(const AttentionArgs &a, int n_rep, hipStream_t stream);
template <> hipError_t launch_chunk_width<256>(const AttentionArgs &a, int n_rep, hipStream_t stream);

size_t chunk_workspace_bytes(const q4kv_spec &s, int num_agents, int q_len, int max_seq_len, int layers, int compute_units,
                             size_t &acc_bytes)
{
    acc_bytes = 0;
    const ChunkSizes sizes = chunk_sizes(s, num_agents, q_len, layers, compute_units);
    if (!chunk_supported(s) || !shares_fit(sizes, num_agents, max_seq_len)) return 0;
    // a window can only make a call take fewer rows per workgroup than this
    const size_t rows = 2 * (size_t)compute_units * rows_shared(sizes, max_seq_len);
    acc_bytes = rows * s.v_dim * sizeof(float);
    // The size tells a workspace that was made for such a call from any other.  Those of decode calls are multiples of 8
    // (plan and counters in pieces of 256 bytes, records of (v_dim + 2) floats), and so is the static array's, so 4 more bytes
    // make it one of its own.
    return acc_bytes + rows * 2 * sizeof(float) + compute_units * sizeof(ChunkShared) + 4;
}

bool chunk_supported(const q4kv_spec &s)
{
    const int n_rep = s.num_q_heads / s.num_kv_heads;
    const bool rep_ok = n_rep == 1 || n_rep == 2 || n_rep == 4 || n_rep == 8;
    const bool square = (s.k_dim == 64 || s.k_dim == 128 || s.k_dim == 256) && s.v_dim == s.k_dim;
    const bool mla_per_head = s.k_dim == 192 && s.v_dim == 128; // decompressed per-head MLA cache (Sec. 3.6)
    return rep_ok && (square || mla_per_head) && !s.v_aliases_k;
}

hipError_t launch_chunk_attention(const AttentionArgs &a, hipStream_t stream)
{
    const int n_rep = a.spec.num_q_heads / a.spec.num_kv_heads;
    switch (a.spec.k_dim) {
    case 64: return launch_chunk_width<64>(a, n_rep, stream);
    case 128: return launch_chunk_width<128>(a, n_rep, stream);
    case 192: return launch_chunk_width<192>(a, n_rep, stream);
    case 256: return launch_chunk_width<256>(a, n_rep, stream);
    default: return hipErrorInvalidValue;
    }
}
#endif

} // namespace q4kv
