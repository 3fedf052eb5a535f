// How a chunk call is cut into workgroups: host arithmetic on sizes alone (the lengths are on the device), in a header of
// its own so that it can be checked without a GPU.  Every figure beside a rule is the time of one attention call in us,
// 256 compute units, binary16 parameters, both sides measured in turn.
#pragma once
#include <cstdint>

namespace q4kv {

constexpr int kXcds = 8;              // compute dies; consecutive workgroups go to consecutive dies
constexpr int kMaxStreamAgents = 256; // agents of a call whose tiles are dealt out evenly

struct ChunkSizes {
    int64_t units; // (layer, agent, KV head) triples of the call
    int64_t rows;  // query rows of a unit: q_len * query heads per KV head
    int compute_units;
};

inline int64_t row_tiles(const ChunkSizes &s, int rows_per_workgroup) { return (s.rows + rows_per_workgroup - 1) / rows_per_workgroup; }

// Time of a 128-row workgroup in that of a 256-row one over the same tokens: its staging does not shrink, its start and
// end do not either.  Measured on full rounds of one layer, 256-, 128- and 192 + 128-wide heads: 0.58, 0.60, 0.58 at 1,712
// tokens, 0.50, 0.55, 0.60 at 6,512; on a chip with few workgroups 0.66 (812), 0.57 (2,512), 0.54-0.57 (8,512).
inline double half_rows_time(double tokens)
{
    const double t = 0.56 + 80.0 / tokens;
    return t < 0.85 ? t : 0.85;
}

// Time of a call with one unit per workgroup, in tokens of a 256-row workgroup, when every unit sees `tokens`.  A unit's row
// tiles all lie on one die (they share its keys), a compute unit holds one workgroup at a time, so a die takes
// rounds of compute_units / 8.
inline double time_alone(const ChunkSizes &s, int rows, double tokens)
{
    const int64_t per_die = (s.units + kXcds - 1) / kXcds * row_tiles(s, rows), places = s.compute_units / kXcds > 0 ? s.compute_units / kXcds : 1;
    return (double)((per_die + places - 1) / places) * tokens * (rows == 128 ? half_rows_time(tokens) : 1.0);
}

// The same when the layers differ in what they see (tokens[0 .. layers), a window each): the workgroups that follow fill
// in behind shorter ones, so it is the average load and, at worst, the longest unit behind it.
inline double time_alone(const ChunkSizes &s, int rows, const int *tokens, int layers)
{
    double sum = 0.0, longest = 0.0;
    for (int i = 0; i < layers; ++i) {
        const double t = tokens[i] * (rows == 128 ? half_rows_time(tokens[i]) : 1.0);
        sum += t;
        longest = t > longest ? t : longest;
    }
    const double per_die = (double)((s.units + kXcds - 1) / kXcds) * (double)row_tiles(s, rows);
    return sum / layers * per_die * kXcds / s.compute_units + longest;
}

// Rows per workgroup when every unit has a workgroup of its own: whichever is done first.  256 rows cost less per row, 128
// are twice the workgroups.  Measured, 128 / 256 rows: 512 tokens behind 8,000, 256-wide, one agent (32 workgroups of
// 256) 316 / 584, four agents, two rounds of 128 against one of 256, 563 / 545 (6,000 tokens, two layers); three
// rounds against two 825 / 941, five against three 1,357 / 1,447, six against three 1,627 / 1,524.  128-wide, one
// agent 183 / 320, two rounds against one 392 / 375.  192 + 128: 210 / 372.  64-wide: 134 / 239.  Twelve layers, five of six
// with a window of 1,024, 256-wide, 512 tokens behind 6,000: one agent 426 / 559, four 1,152 / 1,214, ten 2,931 / 2,886;
// 128-wide: one agent 398 / 436, four 1,344 / 1,122.
inline int rows_alone(const ChunkSizes &s, const int *tokens, int layers)
{
    bool same = true;
    for (int i = 1; i < layers; ++i) same = same && tokens[i] == tokens[0];
    const double narrow = same ? time_alone(s, 128, tokens[0]) : time_alone(s, 128, tokens, layers);
    const double wide = same ? time_alone(s, 256, tokens[0]) : time_alone(s, 256, tokens, layers);
    return narrow < wide ? 128 : 256;
}

// The tokens that a workgroup of 256 rows sees at most (never 0): the bound of the lengths, or its window and its own positions.
inline int visible_tokens(int max_seq_len, int window, int q_len, int n_rep)
{
    const int positions = q_len < 256 / n_rep ? q_len : 256 / n_rep;
    const int64_t seen = window > 0 ? (int64_t)window + positions : max_seq_len;
    const int64_t tokens = seen < max_seq_len ? seen : max_seq_len;
    return tokens > 0 ? (int)tokens : 1;
}

// Rows per workgroup of a call with equal shares.  128 where 256 would be padding: 128 query rows of 256-wide heads, ten
// agents of 4K-32K tokens 295 / 473 (128 / 256 rows), 280 rows of 128-wide heads, four agents of up to 6K 53 / 61, 300 rows of
// 192 + 128-wide ones behind 2,000 41.0 / 42.8, behind 8,000 66 / 74.  And where a compute unit's share is short: every
// workgroup of a shared unit leaves a record of its rows, and half the rows are half the record.  The line is at 448 tokens
// per compute unit; between 250 and 1,000 the sides differ by 6 %, either way, but for one point (512 new tokens, one agent, tokens per compute unit: 256-wide 250 65.6 / 68.3, 400 73.7 / 77.7, 560 87.4 / 90.7, 1,000 120 / 122,
// 2,200 221 / 214; 128-wide 250 51.0 / 50.8, 400 56.5 / 55.6, 560 65.8 / 62.4; 192 + 128 100 37.1 / 40.7, 400 54.0 / 63.6, 750
// 72.8 / 71.2; 64-wide 76 24.6 / 34.5, 282 38.5 / 40.5), so one line does for all widths: over 460 calls a line for each width
// gave nothing.
inline int rows_shared(const ChunkSizes &s, int tokens)
{
    const int64_t wide = row_tiles(s, 256), narrow = row_tiles(s, 128);
    if (0.6 * narrow < wide) return 128;
    return (double)s.units * wide * tokens < 448.0 * s.compute_units ? 128 : 256;
}

// Whether a call may share its tiles out at all, whatever its lengths and window turn out to be: what a workspace is sized
// for.  The line is at two units per compute unit: a workgroup that takes an equal share holds its compute unit
// until the call ends, and a decode step on another stream, which gets in whenever a workgroup ends, waits for that
// long.  48 layers of 512 tokens behind 16,384 (1,536 units) take 7.63 ms with one unit per workgroup, 8.04 with equal
// shares; decode steps of 0.76 ms beside them then take 2.1 and 4.9 ms.  Below the line: layer by layer, 0.84 ms steps beside
// 512 tokens of ten agents of 4K-32K take 1.7 ms without shares and 2.65 with, beside one agent's (0.13 ms a call) 0.92.  Alone
// equal shares would go on to win for a while: 256-wide, four agents of 2K-6K, units per compute unit 1.5 632 / 608 (alone /
// shares), 2 844 / 804, 3 1,225 / 1,151, 4 1,585 / 1,515, 6 2,269 / 2,319; 128-wide 2 456 / 441, 4 838 / 802, 6 1,185 / 1,168.
inline bool shares_fit(const ChunkSizes &s, int num_agents, int max_seq_len)
{
    const int64_t units = s.units * row_tiles(s, rows_shared(s, max_seq_len));
    return num_agents <= kMaxStreamAgents && max_seq_len > 256 && units < 2 * (int64_t)s.compute_units &&
           units * (max_seq_len / 32 + 2) < 0x3fffffff; // tiles (of 32 tokens and more) are numbered with 32-bit integers
}

// Whether equal shares are done before one unit per workgroup.  They even the load out, but every workgroup begins and ends up
// to two units more, leaves their records and a second kernel merges them: about 100 (256-wide) or 300 tokens of a 256-row
// workgroup, and up to 550 (250 at 192 + 128, 500 below) more as the units become as many as the compute
// units.  One unit per workgroup / equal shares, 256-wide: 512 tokens behind 2,000 112 / 71, behind 8,000 316 / 138, ten agents of 4K-32K 2,000 / 1,840; 2 tokens
// of ten agents behind 280 25.1 / 37.0, 512 of three behind 280 50.7 / 66.1, behind 700 67.4 / 80.5, behind 1,500 101 / 103.
// 128-wide: 512 behind 280 30.9 / 41.8, behind 700 39.7 / 48.6, behind 2,000 66.6 / 61.9, behind 8,000 183 / 124; 16 of
// ten agents behind 280 19.7 / 23.4, behind 1,500 43.7 / 32.7; a window of 1,024 on 512 behind 16,000 36 / 46.  192 + 128: 70
// of ten agents behind 280 22.1 / 37.9, 2 of three behind 700 27.9 / 23.2, 512 of one behind 1,500 62 / 50.  Over 486 calls with
// lengths from 280 to 32K, always sharing below two units per compute unit took 5 % longer in the mean and up to 1.7 times
// as long; where this takes the slower form the other is 3 to 12 % faster.
inline bool shares_pay(const ChunkSizes &s, int k_dim, int tokens)
{
    const int rows = rows_shared(s, tokens);
    const double units = (double)(s.units * row_tiles(s, rows)) / s.compute_units;
    const double shared = units * tokens * (rows == 128 ? half_rows_time(tokens) : 1.0);
    const double alone = time_alone(s, rows_alone(s, &tokens, 1), tokens);
    const double start = k_dim == 256 ? 100.0 : 300.0, more = k_dim == 256 ? 550.0 : (k_dim == 192 ? 250.0 : 500.0);
    return alone - shared > start + more * (units < 1.0 ? units : 1.0);
}

} // namespace q4kv
