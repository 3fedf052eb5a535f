// Batched decode attention over a shared-latent Q4 cache (Sec. 3.6, the MLA-shaped spec: one latent row per
// token serves as K in full and as V in its first v_dim elements; 16 query heads read it):
//   out[l][a][h] = softmax(sm * q_h C_hat^T) C_hat[:, :v_dim],   C_hat = code*scale + bias   (Sec. 3.2, 3.4)
//
// A cached token costs k_dim/2 + 4*k_dim/64 bytes and 2*16*(k_dim + v_dim) flops, about 100 flop/byte, so the
// pass is still HBM-bound but only if both contractions run on the matrix cores and the vector ALUs do little
// more than unpack nibbles.  Per wave (one per SIMD, 512 registers, no synchronisation between waves):
//
//  * Work decomposition: the stream-K tile stream of stream_k.h, 64-token tiles, one partial (acc, m, l) per
//    (unit, wave) intersection.  The records of a unit (16 heads x 512 values x about 9 waves: 290 KB) are merged by
//    a kernel of their own with one thread per four output values: left to the last wave that leaves the unit, as
//    the GQA decode path does with its far smaller records, the merge took that one wave 50 round trips to memory
//    and the call 0.75 instead of 0.40 ms.
//  * A tile's code rows are contiguous in the pool; they travel HBM -> LDS directly (global_load_lds, 16 bytes
//    per lane) into one of two buffers while the other is being consumed, so no register holds a code word
//    before it is used.  Scale and bias (18 + 18 bytes per token) go through registers and are re-laid in LDS
//    in the two orders the matrix instructions want.
//  * Scores, transposed:  S^T[t][h] = sum_g s[t,g] * (C_g Q_g^T)[t][h] + (b Qsum^T)[t][h].
//    C_g Q_g^T is two v_mfma_f32_16x16x32_f16 per 16 tokens and group: operand A is a code word masked in place
//    (nibbles become binary16 subnormals, see q4_device.h), operand B the query in the matching element order.
//    The bias term is one more instruction per 16 tokens, its contraction index running over the groups with
//    the group sums of q split into binary16 high and low parts.
//  * Row i of set j is the token whose scores lane slot i/4 receives (slot_token below), so the lane that receives S^T
//    for (head, four tokens of a set) is the lane that must supply P^T for the same tokens as operand B of the second
//    contraction: probabilities never leave their registers.
//  * Output, transposed:  O^T[e][h] = sum_t c[t,e] * (p[h,t] s[t,g(e)])  +  sum_t b[t,g(e)] p[h,t].
//    Operand A wants 8 tokens of one element per lane while a word holds 8 elements of one token: the transposing LDS
//    read of 4-bit elements (ds_read_b64_tr_b4) gives a lane 16 tokens of one element, and the four masks that unpack a
//    code word for the scores unpack 8 tokens here.  One read and ten vector instructions feed four matrix instructions.
//    (Eight 4-byte reads, eight masks and sixteen v_perm per four operands before: 77 LDS instructions more per tile.)
//  * Online softmax per tile of 64 tokens, lane-local denominators, accumulators rescaled only when some
//    head's running maximum moved far.
//
// What bounds it is one instruction stream per SIMD (an instruction every five clocks): 1,132 vector, 206 matrix and 123
// LDS instructions per 64-token tile (counted on the device, per tile of a whole call).  27 layers of five agents of 32,768
// tokens: 342-355 us a call, 4.1 TB/s, plan and combine included (405 us with 1,414 vector and 200 LDS instructions: results copied
// out of accumulator registers, per-byte permutes, selects for hidden tokens in every tile).
#include "q4_device.h"
#include "q4kv_internal.h"
#include "stream_k.h"

namespace q4kv {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kHeads = 16;          // query heads per latent head: the M (or N) extent of the matrix tiles
constexpr float kNegBig = -1.0e30f; // "minus infinity" that survives subtraction
constexpr float kLog2e = 1.4426950408889634f;
constexpr uint32_t kLiftScaleBits = 0x5BE0; // binary16 252: 2^8 times that is still below 65504

typedef __attribute__((address_space(3))) void *lds_ptr_t;
typedef const __attribute__((address_space(1))) void *global_ptr_t;

// The records of a call: maxima and denominators, number per unit.  A planned call brings a second pair, for a plan made in a
// workspace with room for more records (slots 0: this one has not); which of them holds stands in the plan's signature.
struct Records {
    float *ml;
    int slots;
};
__device__ __forceinline__ bool fine_plan(const int32_t *plan, int signature, const Records &fine)
{
    return fine.slots > 0 && plan[5] == (signature ^ kFineRecords);
}

struct MlaParams {
    const uint32_t *codes;
    const uint16_t *scale, *bias;
    const uint16_t *q;
    StreamParams stream;
    float *part_acc;
    Records records, fine;
    int q_heads;
    float score_scale; // sm_scale * log2(e): scores are kept in log2 units
};

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// x[i] (op) x[i ^ 16], x[i] (op) x[i ^ 32] without touching LDS
__device__ __forceinline__ float xor16_max(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}
__device__ __forceinline__ float xor32_max(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}
__device__ __forceinline__ float xor16_sum(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ float xor32_sum(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
// the value lane i ^ 16 holds
__device__ __forceinline__ float xor16_other(float x, bool odd_row)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __builtin_bit_cast(float, (uint32_t)(odd_row ? r[0] : r[1]));
}

// The 64 tokens of a tile as 4 slots q (a lane's contraction slot) x 4 sets j of 16 consecutive tokens x 4 rows r.  Odd
// sets turn the slots round by one, so that the 16 rows a transposing read takes for one slot (all j and r) lie two by two
// in 8 bank groups (the row pitch is 8 banks modulo 64) instead of four by four in 4.
__device__ __forceinline__ constexpr int slot_token(int q, int j, int r) { return 16 * j + 4 * ((q + (j & 1)) & 3) + r; }

__device__ __forceinline__ half8_t words_to_half8(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    return __builtin_bit_cast(half8_t, make_uint4(a, b, c, d));
}

__device__ __forceinline__ half8_t code_operand(uint32_t w)
{
    const uint32_t w8 = w >> 8;
    return words_to_half8(w & 0x000F000Fu, w & 0x00F000F0u, w8 & 0x000F000Fu, w8 & 0x00F000F0u);
}

typedef int int2_t __attribute__((ext_vector_type(2)));
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) int2_t *lds_int2_ptr;

__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, a), __builtin_bit_cast(ushort2_t, b)));
}

__device__ __forceinline__ float half_of(uint32_t pair, int hi)
{
    return half_bits_to_float((uint16_t)(hi ? pair >> 16 : pair & 0xffffu));
}

// GK, GV: quantization groups of the latent row and of its value part (k_dim = 64 GK, v_dim = 64 GV <= k_dim).
// BF: scale and bias are stored as bfloat16; they are converted to binary16 (exactly, for parameters of binary16-range
// data above 2^-14) when a tile's parameters are re-laid in LDS, everything after that is the same.
template <int GK, int GV, bool BF>
__global__ __launch_bounds__(kThreads, 1) void mla_decode_kernel(const MlaParams p)
{
    static_assert(GV <= 8 && GV <= GK && GK <= 10, "group counts");
    constexpr int DK = GK * kGroup, DV = GV * kGroup;
    constexpr int W = DK / 8;               // code words per token row
    constexpr int kTileWords = kWave * W;   // one tile of code rows
    constexpr int kLoads = kTileWords / (kWave * 4); // 1 KiB transfers per tile
    constexpr int BTP = GK > 8 ? 12 : 8;    // binary16 slots per token in the token-major bias copy

    __shared__ __attribute__((aligned(16))) uint32_t codes_all[kWaves][2][kTileWords]; // two tile buffers per wave
    // scale and bias of the tile, [tile half][group][slot q][8]: one 16-byte read gives a lane the 8 tokens of its
    // contraction slots, register r the tokens slot_token(q, 2 half, r) and slot_token(q, 2 half + 1, r)
    __shared__ __attribute__((aligned(16))) uint16_t sc_all[kWaves][2][GK][4][8];
    __shared__ __attribute__((aligned(16))) uint16_t bg_all[kWaves][2][GV][4][8];
    // bias again, token-major [64][BTP] (groups 0..7, then groups 8.. and zero padding): operand of the score bias term
    __shared__ __attribute__((aligned(16))) uint16_t bt_all[kWaves][kWave * BTP + 8];

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = uniform(tid / kWave);
    const int gw = blockIdx.x * kWaves + wave; // this wave's index in the launch

    const bool fine = fine_plan(p.stream.plan, p.stream.plan_signature, p.fine);
    StreamParams sp = p.stream;
    if (fine) sp.plan_signature ^= kFineRecords;
    const TileStream ts(sp);
    const int per = ts.per, N = ts.N;
    const long long x_begin = (long long)gw * per;
    if (x_begin >= N) return;
    const int x0 = (int)x_begin;
    const int x1 = (int)min((long long)N, x_begin + per);

    uint32_t *const bufs = &codes_all[wave][0][0];
    uint16_t *const sc = &sc_all[wave][0][0][0][0];
    uint16_t *const bg = &bg_all[wave][0][0][0][0];
    uint16_t *const bt = bt_all[wave];

    // lane roles: col = row of an A operand / column of a B operand or result; qk = the lane's contraction slot
    // (8 of 32 indices) in an operand, the row quad in a result
    const int col = lane % 16, qk = lane / 16;
    const int row_even = col, row_odd = 4 * ((col / 4 + 1) & 3) + col % 4; // token (in its set) behind A row `col`, sets 0, 2 / 1, 3
    const int v_row = slot_token(qk, col / 4, col % 4); // token whose codes this lane points the transposing reads at
    // where token `lane` sits in sc / bg (half index, without the group)
    const int tok_set = lane / 16, tok_q = (((lane % 16) / 4) - (tok_set & 1)) & 3;
    const int tok_at = tok_q * 8 + 2 * (lane % 4) + (tok_set & 1), tok_h2 = tok_set / 2;

    Cursor cur = ts.locate(x0);

    constexpr int PW = GK / 2, PT = GK % 2; // whole words and odd halves of a row of scales (or biases)
    uint32_t sraw[PW + PT], braw[PW + PT];  // scale / bias bits of token `lane` of the tile in flight

    // Start the transfer of a tile: kLoads instructions move 1 KiB each straight from global memory into LDS
    // (lane i's 16 bytes land at M0 + offset + 16 i), then the lane's scale and bias loads.  The transfers are
    // written as asm statements so that the compiler neither tracks them nor makes later LDS reads of the
    // other buffer wait for them; the tile loop waits for them itself (vmcnt) before it touches the buffer.
    auto issue_tile = [&](const Cursor &c, int buf) __attribute__((always_inline)) {
        const uint32_t *src = p.codes + c.row * W; // wave-uniform
        const uint32_t dst = (uint32_t)(uintptr_t)(lds_ptr_t)(bufs + buf * kTileWords);
        const uint32_t lane_off = lane * 16;
#pragma unroll
        for (int i = 0; i < kLoads; i += 4) {
            const uint32_t *s4k = src + i * (kWave * 4);
            const uint32_t d4k = dst + i * 1024;
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(s4k), "s"(d4k) : "memory", "m0");
            if (i + 1 < kLoads)
                asm volatile("global_load_lds_dwordx4 %0, %1 offset:1024" ::"v"(lane_off), "s"(s4k) : "memory");
            if (i + 2 < kLoads)
                asm volatile("global_load_lds_dwordx4 %0, %1 offset:2048" ::"v"(lane_off), "s"(s4k) : "memory");
            if (i + 3 < kLoads)
                asm volatile("global_load_lds_dwordx4 %0, %1 offset:3072" ::"v"(lane_off), "s"(s4k) : "memory");
        }
        const uint16_t *sp = p.scale + (c.row + lane) * GK;
        const uint16_t *bp = p.bias + (c.row + lane) * GK;
        __builtin_memcpy(sraw, sp, 4 * PW); // rows of an odd number of groups are only 2-byte aligned
        __builtin_memcpy(braw, bp, 4 * PW);
        if constexpr (PT) {
            sraw[PW] = sp[GK - 1];
            braw[PW] = bp[GK - 1];
        }
    };

    half8_t qop[GK][2]; // query operand per (group, word pair member): element order of code_operand, odd elements / 16
    half8_t qsop;       // group sums of q: slots of qk 0 = high parts of groups 0..7, qk 1 = low parts, qk 2 / 3 = groups 8..
    int x = x0;
    int buf = 0;        // tile buffer the current tile arrives in

    issue_tile(cur, 0);
    while (x < x1) {
        // ---- a unit (or the part of it inside this wave's range) begins: its 16 query heads as operand B of the
        // score contraction.  Lane (head col, slot qk) holds, for group g and word r, the 8 elements of word
        // 8g + 2qk + r in the order code_operand emits codes (0,4,1,5,2,6,3,7), odd elements divided by 16
        // because their codes arrive 16 times larger.
        const int64_t unit0 =
            ((int64_t)cur.li * p.stream.num_agents + cur.agent) * p.q_heads + (int64_t)cur.kvh * kHeads;
        int slot, slots_unused;
        ts.slot_of(cur, gw, slot, slots_unused);
        {
            const uint16_t *qrow = p.q + (unit0 + col) * DK + 16 * qk;
            float qs[GK];
#pragma unroll
            for (int g = 0; g < GK; ++g) {
                float sum = 0.0f;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const uint4 raw = *reinterpret_cast<const uint4 *>(qrow + g * kGroup + 8 * r);
                    const half2_t e01 = bits_to_half2(raw.x), e23 = bits_to_half2(raw.y);
                    const half2_t e45 = bits_to_half2(raw.z), e67 = bits_to_half2(raw.w);
                    const half_t sixteenth = (half_t)0.0625f;
                    qop[g][r] = half8_t{e01.x, e45.x, e01.y * sixteenth, e45.y * sixteenth,
                                        e23.x, e67.x, e23.y * sixteenth, e67.y * sixteenth};
                    sum += ((float)e01.x + (float)e01.y) + ((float)e23.x + (float)e23.y) +
                           ((float)e45.x + (float)e45.y) + ((float)e67.x + (float)e67.y);
                }
                qs[g] = xor32_sum(xor16_sum(sum)); // all four slots of a head now hold the group's sum
            }
            half_t part[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                // slot qk, element e: qk 0 -> high part of group e, qk 1 -> low part of group e,
                // qk 2 -> high part of group 8 + e, qk 3 -> low part of group 8 + e
                const float lo_grp = e < GK ? qs[e] : 0.0f;
                const float hi_grp = 8 + e < GK ? qs[(8 + e) < GK ? 8 + e : 0] : 0.0f;
                const float v = qk >= 2 ? hi_grp : lo_grp;
                const half_t hi = (half_t)v;
                part[e] = (qk & 1) ? (half_t)(v - (float)hi) : hi;
            }
            qsop = half8_t{part[0], part[1], part[2], part[3], part[4], part[5], part[6], part[7]};
        }
        float4_t acc[4 * GV]; // [16-element column block]: rows = elements, columns = heads
        float4_t pbacc = float4_t{0.0f, 0.0f, 0.0f, 0.0f}; // rows = groups: sum_t b[t,g] p[h,t]
#pragma unroll
        for (int c = 0; c < 4 * GV; ++c) acc[c] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        float m_run = kNegBig, l_run = 0.0f; // of head `col`; l_run covers this lane's tokens only
        bool first_tile = true, unit_ends;
        // The query operand lives in accumulator registers, which matrix instructions read directly; without this the
        // allocator moved it about in every tile (65 instructions; 27 layers of five agents of 32K tokens 359 -> 346 us)
#pragma unroll
        for (int g = 0; g < GK; ++g) asm volatile("" : "+a"(qop[g][0]), "+a"(qop[g][1]));
        asm volatile("" : "+a"(qsop));

        do { // ---- the tiles of the unit
            const uint32_t *cb = bufs + buf * kTileWords;
            const bool last_of_wave = x + 1 >= x1;
            Cursor nxt = cur;
            if (!last_of_wave) ts.step(nxt);
            unit_ends = last_of_wave || nxt.j == 0;

            // everything of this tile has landed: codes in `cb`, scale / bias in registers
            __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt(0)
            const int tok = cur.t0 + lane;
            const bool tok_valid = cur.reachable && tok >= cur.first && tok < cur.n;
            // wave-uniform: some token of the tile lies outside the agent's visible range
            const bool edge = !(cur.reachable && cur.t0 >= cur.first && cur.t0 + kWave <= cur.n);
            uint32_t s_top = 0; // the larger of this token's value scales, two halves apart
            {
                uint32_t s[PW + PT], b[PW + PT];
                if constexpr (BF) {
                    auto both = [](uint32_t w) {
                        return (uint32_t)float_to_half_bits(bf16_bits_to_float((uint16_t)(w & 0xffffu))) |
                               (uint32_t)float_to_half_bits(__builtin_bit_cast(float, w & 0xffff0000u)) << 16;
                    };
#pragma unroll
                    for (int i = 0; i < PW + PT; ++i) {
                        s[i] = both(sraw[i]);
                        b[i] = both(braw[i]);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < PW + PT; ++i) {
                        s[i] = sraw[i];
                        b[i] = braw[i];
                    }
                }
                // rows outside the agent's range may hold anything: their scale and bias become zero so that no NaN
                // or infinity reaches a matrix operand (codes are nibbles and always finite)
                if (__builtin_expect(edge, 0)) {
                    asm volatile(""); // a branch: interior tiles (nearly all) must not pay for the selects
#pragma unroll
                    for (int i = 0; i < PW + PT; ++i) {
                        s[i] = tok_valid ? s[i] : 0u;
                        b[i] = tok_valid ? b[i] : 0u;
                    }
                }
                uint16_t *s_at = sc + tok_h2 * GK * 32 + tok_at, *b_at = bg + tok_h2 * GV * 32 + tok_at;
#pragma unroll
                for (int g = 0; g < GK; ++g) s_at[g * 32] = (uint16_t)(g % 2 ? s[g / 2] >> 16 : s[g / 2]);
#pragma unroll
                for (int g = 0; g < GV; ++g) b_at[g * 32] = (uint16_t)(g % 2 ? b[g / 2] >> 16 : b[g / 2]);
                uint2 *btw = reinterpret_cast<uint2 *>(bt + lane * BTP);
#pragma unroll
                for (int i = 0; i < BTP / 4; ++i)
                    btw[i] = make_uint2(2 * i < PW + PT ? b[2 * i] : 0u, 2 * i + 1 < PW + PT ? b[2 * i + 1] : 0u);
#pragma unroll
                for (int i = 0; i < GV / 2; ++i) s_top = i == 0 ? s[0] : pk_max_u16(s_top, s[i]);
            }
            // wave-uniform: some value scale of the tile is too large for probabilities up to 2^7 (see the softmax)
            const int parts = __builtin_amdgcn_ballot_w64((s_top & 0xffffu) > kLiftScaleBits || (s_top >> 16) > kLiftScaleBits) != 0ull ? 2 : 1;
            // the next tile starts travelling (into the buffer the previous tile was read from)
            // (behind the last tile nothing does: the wave would have to wait for it before it leaves; 3,000 to 9,000
            // tokens of five agents, eight layers, a plan, an append and a call each: 334 -> 321 us)
            if (!last_of_wave) issue_tile(nxt, buf ^ 1);
            __builtin_amdgcn_sched_barrier(0);
            wave_lds_sync();

            // A tile with a large value scale is taken in two parts, first the even rows r of every slot, then the odd ones (see the
            // softmax); everything that the second part reads is still in LDS.
            int part = 0;
            do {
                // ---- scores of the 64 tokens, four 16-token sets: z[j][r] is token slot_token(qk, j, r), head col, in units of
                // 2^-24 / score_scale.  Every operand register is read again from LDS for the next set (the scales: for
                // the next pair of sets) right after its last use: with one wave per SIMD nothing else hides the latency.
                float z[4][4];
                const float4_t zero = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
                const uint32_t *const k_at[2] = {cb + row_even * W + 2 * qk, cb + row_odd * W + 2 * qk};
                const uint16_t *const bt_at[2] = {bt + row_even * BTP + ((GK > 8 && qk >= 2) ? 8 : 0),
                                                  bt + row_odd * BTP + ((GK > 8 && qk >= 2) ? 8 : 0)};
                const uint16_t *const sc_at = sc + qk * 8;
                uint2 kw[GK]; // code words 8g + 2qk, 8g + 2qk + 1 of this lane's row
                uint4 s8[GK]; // scales of the tokens this lane gets results for, two sets
                uint2 b0, b1; // bias row (slots as in qsop)
                b0 = *reinterpret_cast<const uint2 *>(bt_at[0]);
                b1 = *reinterpret_cast<const uint2 *>(bt_at[0] + 4);
#pragma unroll
                for (int g = 0; g < GK; ++g) {
                    kw[g] = *reinterpret_cast<const uint2 *>(k_at[0] + 8 * g);
                    s8[g] = *reinterpret_cast<const uint4 *>(sc_at + g * 32);
                }
                // value side: column block c of the tile's rows, 16 tokens x 16 elements per slot, transposed by the read
                const uint32_t *const v_at = cb + v_row * W;
                auto load_columns = [&](int c) __attribute__((always_inline)) {
                    return __builtin_amdgcn_ds_read_tr4_b64_v2i32((lds_int2_ptr)(v_at + 2 * c));
                };
                constexpr int kAhead = 4;
                int2_t vw[kAhead];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint2 c0 = b0, c1 = b1;
                    if (qk >= 2) {
                        c1 = make_uint2(0u, 0u);
                        if (GK <= 8) c0 = make_uint2(0u, 0u);
                    }
                    // bias term: A = b[t][.], B = group sums of q
                    float4_t sum = __builtin_amdgcn_mfma_f32_16x16x32_f16(words_to_half8(c0.x, c0.y, c1.x, c1.y), qsop, zero, 0, 0, 0);
                    if (j < 3) {
                        b0 = *reinterpret_cast<const uint2 *>(bt_at[(j + 1) & 1] + (j + 1) * 16 * BTP);
                        b1 = *reinterpret_cast<const uint2 *>(bt_at[(j + 1) & 1] + (j + 1) * 16 * BTP + 4);
                    }
                    float4_t d[GK];
#pragma unroll
                    for (int g = 0; g < GK + 1; ++g) {
                        if (g < GK) {
                            d[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(code_operand(kw[g].x), qop[g][0], zero, 0, 0, 0);
                            d[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(code_operand(kw[g].y), qop[g][1], d[g], 0, 0, 0);
                            if (j < 3) kw[g] = *reinterpret_cast<const uint2 *>(k_at[(j + 1) & 1] + (j + 1) * 16 * W + 8 * g);
                        }
                        if (g == 0) {
#pragma unroll
                            for (int r = 0; r < 4; ++r) sum[r] *= 0x1p-24f; // the products' unit
                        } else { // the results of the group before
                            const uint32_t s4[4] = {s8[g - 1].x, s8[g - 1].y, s8[g - 1].z, s8[g - 1].w};
#pragma unroll
                            for (int r = 0; r < 4; ++r) sum[r] = fmaf(half_of(s4[r], j & 1), d[g - 1][r], sum[r]);
                            if (j == 1) s8[g - 1] = *reinterpret_cast<const uint4 *>(sc_at + (GK + g - 1) * 32);
                            if (j == 3 && g <= kAhead) vw[g - 1] = load_columns(g - 1);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) z[j][r] = sum[r];
                }

                // ---- online softmax of head col over the tile.  m_run is the reference the exponentials are taken against,
                // not the exact running maximum: it moves only when a tile's maximum exceeds it by more than 7 (in log2
                // units) and then to 4 below that maximum, so the accumulators are rescaled a handful of times per unit instead of
                // in every other tile.  p <= 2^7 then, and p * s stays inside binary16 for scales up to kLiftScale with one binary
                // place to spare: the maximum is rounded once more than the exponents are, and from 2^18 on that is a few per
                // cent of p (at 2^19, with the line at 504, 130.25 * 504 was infinite).  In a tile with a
                // larger one (values spread over thousands) the even rows keep p <= 2^2.5, against the maximum itself: the widest
                // group that can be stored, +-65504, has the scale 8736 (as bfloat16 8768), and 2^2.5 * 8768 = 49600.  The
                // odd rows, whose p is divided by 16 below, follow with the reference 4 lower: the division costs no bits there either.
                float zs = p.score_scale * kCodeScaleA;
                if (__builtin_expect(!(p.score_scale > 0.0f), 0)) { // the maximum may not be taken before the scale is applied
                    asm volatile("");
#pragma unroll
                    for (int i = 0; i < 16; ++i) z[i / 4][i % 4] *= zs;
                    zs = 1.0f;
                }
                if (__builtin_expect(edge, 0)) {
                    int t0 = cur.t0;
                    asm volatile("" : "+s"(t0)); // else the comparisons move out of the two parts' loop, into every tile
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int t = t0 + slot_token(qk, j, r);
                            if (!(cur.reachable && t >= cur.first && t < cur.n)) z[j][r] = -INFINITY;
                        }
                }
                float slack = 7.0f, below = 4.0f, m_ref = m_run;
                if (__builtin_expect(parts > 1, 0)) {
                    asm volatile("");
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if ((i & 1) != part) z[i / 4][i % 4] = -INFINITY;
                    slack = part == 0 ? 2.5f : 6.5f;
                    below = part == 0 ? 0.0f : 4.0f;
                    m_ref += part == 0 ? 4.0f : -4.0f; // from 4 below the maximum to the maximum, and back
                }
                float mt = -INFINITY;
#pragma unroll
                for (int i = 0; i < 16; ++i) mt = fmaxf(mt, z[i / 4][i % 4]);
                mt = xor32_max(xor16_max(mt)) * zs;
                const bool above = mt > m_ref + slack; // the same in the four lanes of a head
                const float m_new = above ? mt - below : m_ref;
                float psum = 0.0f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float pr = __builtin_amdgcn_exp2f(fmaf(z[i / 4][i % 4], zs, -m_new)); // 0 for a masked token
                    z[i / 4][i % 4] = pr;
                    psum += pr;
                }
                if (!first_tile && __builtin_amdgcn_ballot_w64(m_new != m_run) != 0ull) { // in a unit's first tile all sums are zero
                    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new); // 1 for a head whose reference stays
                    l_run *= alpha;
                    pbacc *= alpha;
#pragma unroll
                    for (int c = 0; c < 4 * GV; ++c) acc[c] *= alpha;
                }
                l_run += psum;
                m_run = m_new;

                // ---- values: per tile half, B = p * s of tokens slot_token(qk, 2 h2 + {0, 1}, r) in register r, in two binary16
                // terms.  The product of two binary16 numbers minus its rounded value is a binary16 number again (barring
                // underflow), so hi + lo carries p s to about 22 bits.  With hi alone an agent of a handful of tokens,
                // where one or two rounding errors of p s make up the whole error of an output, can leave the tolerance
                // when the latent holds channels of several times the usual magnitude.
                // The codes of the odd rows r arrive 16 times larger (code_operand): their p is a sixteenth.  That costs
                // no bits, because the reference lies 4 below the maximum.
                half2_t p16[2][4];
#pragma unroll
                for (int h2 = 0; h2 < 2; ++h2) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) p16[h2][r] = half2_t{(half_t)z[2 * h2][r], (half_t)z[2 * h2 + 1][r]};
                    const half8_t pop = words_to_half8(half2_to_bits(p16[h2][0]), half2_to_bits(p16[h2][1]), half2_to_bits(p16[h2][2]),
                                                       half2_to_bits(p16[h2][3]));
                    // bias sums of this half: rows = groups (rows past GV repeat a valid row, unused)
                    const int g_row = (col % 8) < GV ? (col % 8) : GV - 1;
                    const uint4 b8 = *reinterpret_cast<const uint4 *>(bg + ((h2 * GV + g_row) * 4 + qk) * 8);
                    pbacc = __builtin_amdgcn_mfma_f32_16x16x32_f16(words_to_half8(b8.x, b8.y, b8.z, b8.w), pop, pbacc, 0, 0, 0);
                    const half2_t sixteenth = half2_t{(half_t)0.0625f, (half_t)0.0625f};
                    p16[h2][1] *= sixteenth;
                    p16[h2][3] *= sixteenth;
                }
                half8_t ps_hi[2], ps_lo[2];
                auto scaled = [&](int g) __attribute__((always_inline)) {
#pragma unroll
                    for (int h2 = 0; h2 < 2; ++h2) {
                        const uint4 sv = *reinterpret_cast<const uint4 *>(sc_at + (h2 * GK + g) * 32);
                        const half2_t s2[4] = {bits_to_half2(sv.x), bits_to_half2(sv.y), bits_to_half2(sv.z), bits_to_half2(sv.w)};
                        half2_t hi[4], lo[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            hi[r] = p16[h2][r] * s2[r];
                            lo[r] = __builtin_elementwise_fma(p16[h2][r], s2[r], -hi[r]);
                        }
                        ps_hi[h2] = words_to_half8(half2_to_bits(hi[0]), half2_to_bits(hi[1]), half2_to_bits(hi[2]), half2_to_bits(hi[3]));
                        ps_lo[h2] = words_to_half8(half2_to_bits(lo[0]), half2_to_bits(lo[1]), half2_to_bits(lo[2]), half2_to_bits(lo[3]));
                    }
                };
                half8_t cop[2] = {code_operand((uint32_t)vw[0].x), code_operand((uint32_t)vw[0].y)};
#pragma unroll
                for (int c = 0; c < 4 * GV; ++c) {
                    if (c % 4 == 0) scaled(c / 4);
                    if (c + kAhead < 4 * GV) vw[c % kAhead] = load_columns(c + kAhead);
                    const half8_t a0 = cop[0], a1 = cop[1];
                    acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, ps_hi[0], acc[c], 0, 0, 0);
                    acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, ps_lo[0], acc[c], 0, 0, 0);
                    acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, ps_hi[1], acc[c], 0, 0, 0);
                    acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, ps_lo[1], acc[c], 0, 0, 0);
                    if (c + 1 < 4 * GV) { // the next block's operands, while this one is multiplied
                        cop[0] = code_operand((uint32_t)vw[(c + 1) % kAhead].x);
                        cop[1] = code_operand((uint32_t)vw[(c + 1) % kAhead].y);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                wave_lds_sync(); // the next tile rewrites sc / bg / bt
                first_tile = false;
            } while (__builtin_expect(++part < parts, 0));
            cur = nxt;
            buf ^= 1;
            ++x;
        } while (!unit_ends);

        // ---- this wave's share of the unit is complete: one partial per query head, written straight from the
        // accumulators.  Lane (head col, quad qk) holds elements 4 qk .. 4 qk + 3 of every column block; of the bias sums
        // it holds groups 4 (qk % 2) + r.
        const float l_tot = xor32_sum(xor16_sum(l_run));
        const bool odd = (qk & 1) != 0;
        float pb[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float other = xor16_other(pbacc[r], odd);
            pb[r] = odd ? other : pbacc[r];
            pb[4 + r] = odd ? pbacc[r] : other;
        }
        const int64_t rec = (unit0 + col) * (fine ? p.fine.slots : p.records.slots) + slot;
        float *dst = p.part_acc + rec * DV + 4 * qk;
#pragma unroll
        for (int c = 0; c < 4 * GV; ++c) {
            float4_t o;
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] = fmaf(acc[c][r], kCodeScaleA, pb[c / 4]);
            *reinterpret_cast<float4_t *>(dst + 16 * c) = o;
        }
        if (qk == 0) {
            float *ml = (fine ? p.fine.ml : p.records.ml) + rec * 2;
            ml[0] = m_run;
            ml[1] = l_tot;
        }
    }
}

// Merge the partials of every (layer, agent, query head) in slot order: binary32, output binary16.  A thread owns
// four consecutive output elements of one head (16-byte loads); v_dim / 4 threads share a head.
// B: records whose loads are issued together.
template <int B>
__global__ __launch_bounds__(kThreads) void combine_kernel(const float *__restrict__ part_acc,
                                                           const Records records, const Records fine,
                                                           const int32_t *__restrict__ plan, uint16_t *__restrict__ out,
                                                           int q_heads, int kv_heads, int num_agents, int v_dim,
                                                           int layers, long long units, int signature)
{
    const bool is_fine = fine_plan(plan, signature, fine);
    if (!is_fine && plan[5] != signature) return; // a plan made for other arguments: the attention launch did nothing either
    const int max_slots = is_fine ? fine.slots : records.slots;
    const int threads_per_unit = v_dim / 4;
    const long long unit = (long long)blockIdx.x * (kThreads / threads_per_unit) + threadIdx.x / threads_per_unit;
    if (unit >= units) return; // (layer in call, agent, query head)
    const int e = (threadIdx.x % threads_per_unit) * 4;
    const int qh = (int)(unit % q_heads);
    const int agent = (int)((unit / q_heads) % num_agents);
    const int li = (int)(unit / ((long long)q_heads * num_agents));
    const int kvh = qh / (q_heads / kv_heads);
    PlanView pv;
    pv.plan = plan;
    pv.A = num_agents;
    pv.L = layers;
    const int per = plan[1];
    const int cb = pv.layer_class_off(li);
    const int32_t *tpre = pv.tpre(cb);
    const int tiles = tpre[agent + 1] - tpre[agent];
    int slots = 0;
    if (tiles > 0) {
        const long long u0 = (long long)plan[pv.lt_off() + li] + (long long)kvh * pv.tiles_per_head(cb) + tpre[agent];
        slots = (int)((u0 + tiles - 1) / per - u0 / per) + 1;
    }
    const float *ml = (is_fine ? fine.ml : records.ml) + unit * max_slots * 2;
    const float *acc = part_acc + unit * max_slots * v_dim + e;
    // B slots at a time: every load of a group is issued before anything is computed, so a unit costs one memory round trip per
    // group.  Past the last slot a group reads that slot again and gives it no weight.  The running reference moves group by
    // group (with one group: exactly the maximum over all slots, then one weighted sum in slot order).
    float m = kNegBig, denom = 0.0f;
    float4 o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int s0 = 0; s0 < slots; s0 += B) {
        float mm[B], ll[B];
        float4 a[B];
#pragma unroll
        for (int k = 0; k < B; ++k) {
            const int at = min(s0 + k, slots - 1);
            const float2 t = *reinterpret_cast<const float2 *>(ml + 2 * at);
            mm[k] = t.x;
            ll[k] = s0 + k < slots ? t.y : 0.0f;
            a[k] = *reinterpret_cast<const float4 *>(acc + (long long)at * v_dim);
        }
        float m_new = m;
#pragma unroll
        for (int k = 0; k < B; ++k)
            if (ll[k] > 0.0f) m_new = fmaxf(m_new, mm[k]);
        const float keep = __builtin_amdgcn_exp2f(m - m_new); // 1 when the reference stays, 0 while nothing was added yet
        denom *= keep;
        o.x *= keep; o.y *= keep; o.z *= keep; o.w *= keep;
#pragma unroll
        for (int k = 0; k < B; ++k) {
            if (!(ll[k] > 0.0f)) continue;
            const float wgt = __builtin_amdgcn_exp2f(mm[k] - m_new);
            denom = fmaf(wgt, ll[k], denom);
            o.x = fmaf(wgt, a[k].x, o.x);
            o.y = fmaf(wgt, a[k].y, o.y);
            o.z = fmaf(wgt, a[k].z, o.z);
            o.w = fmaf(wgt, a[k].w, o.w);
        }
        m = m_new;
    }
    const float inv = denom > 0.0f ? 1.0f / denom : 0.0f;
    const uint32_t lo = (uint32_t)float_to_half_bits(o.x * inv) | ((uint32_t)float_to_half_bits(o.y * inv) << 16);
    const uint32_t hi = (uint32_t)float_to_half_bits(o.z * inv) | ((uint32_t)float_to_half_bits(o.w * inv) << 16);
    *reinterpret_cast<uint2 *>(out + unit * v_dim + e) = make_uint2(lo, hi);
}

hipError_t launch_combine(const AttentionArgs &a, hipStream_t stream)
{
    const int64_t units = (int64_t)a.layers_in_call * a.num_agents * a.q_len * a.spec.num_q_heads;
    if (units == 0) return hipSuccess;
    const int units_per_block = kThreads / (a.spec.v_dim / 4); // v_dim is a multiple of 64 and at most 1,024 here
    const int64_t blocks = (units + units_per_block - 1) / units_per_block;
    // Up to two workgroups per compute unit the kernel is a chain of trips to memory, and a long agent of a short call has up to
    // a hundred records: sixteen of them a trip (one layer, five agents of 32K tokens, a call 55.2 -> 48.1 us).  With more, the
    // memory is busy and a unit has about nine records: four.
    const auto kernel = blocks <= 2 * a.compute_units ? combine_kernel<16> : combine_kernel<4>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kThreads), 0, stream, a.part_acc, Records{a.part_ml, a.max_slots},
                       Records{a.fine_ml, a.fine_slots}, a.plan, a.out, a.spec.num_q_heads, a.spec.num_kv_heads, a.num_agents,
                       a.spec.v_dim, a.layers_in_call, (long long)units, a.plan_signature);
    return hipGetLastError();
}

template <int GK, int GV, bool BF>
hipError_t launch_mla_t(const AttentionArgs &a, hipStream_t stream)
{
    MlaParams p;
    p.codes = a.k.codes; p.scale = a.k.scale; p.bias = a.k.bias;
    p.q = a.q;
    p.stream = stream_params(a);
    p.part_acc = a.part_acc;
    p.records = Records{a.part_ml, a.max_slots};
    p.fine = Records{a.fine_ml, a.fine_slots};
    p.q_heads = a.spec.num_q_heads;
    p.score_scale = a.sm_scale * kLog2e;
    hipLaunchKernelGGL((mla_decode_kernel<GK, GV, BF>), dim3(a.grid_workgroups), dim3(kThreads), 0, stream, p);
    return hipGetLastError();
}

} // namespace

bool mla_decode_supported(const q4kv_spec &s)
{
    return s.v_aliases_k && s.num_q_heads == kHeads * s.num_kv_heads && s.k_dim == 576 && s.v_dim == 512;
}

// every wave walks a tile range of its own
hipError_t launch_mla_decode_plan(const AttentionArgs &a, hipStream_t stream)
{
    return launch_plan(a, a.grid_workgroups * kWaves, 1, stream);
}

hipError_t launch_mla_decode_attention(const AttentionArgs &a, hipStream_t stream)
{
    hipError_t e = a.spec.param_format == Q4KV_PARAMS_BF16 ? launch_mla_t<9, 8, true>(a, stream) : launch_mla_t<9, 8, false>(a, stream);
    return e == hipSuccess ? launch_combine(a, stream) : e;
}

} // namespace q4kv
