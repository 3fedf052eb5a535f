// How a chunk call is cut into workgroups: host arithmetic on sizes alone (the lengths are on the device), in a header of
// its own so that it can be checked without a GPU.  Every figure beside a rule is the time of one attention call in us,
// 256 compute units, binary16 parameters, both sides measured in turn, on the kernel as it is unless it says otherwise.  (The lines
// were drawn on a kernel without softmax beside the product, whose waves without rows cost as much as others; they still hold.)
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
// end do not either.  Measured on full rounds of one layer, 256-, 128- and 192 + 128-wide heads: 0.57, 0.59, 0.58 at 1,712
// tokens, 0.56, 0.55, 0.55 at 6,512; on a chip with few workgroups 0.63-0.68 (812), 0.61 (2,512), 0.58-0.61 (8,512).
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
// 256) 315 / 517, four agents, two rounds of 128 against one of 256, 526 / 470 (6,000 tokens, two layers); three
// rounds against two 799 / 874, six against three 1,602 / 1,428.  128-wide, one agent 167 / 291, two rounds against one
// 359 / 327.  192 + 128: 197 / 333.  64-wide: 129 / 220.  Twelve layers, five of six with a window of 1,024, 256-wide, 512 tokens
// behind 6,000: four agents 1,136 / 1,135, ten 2,919 / 2,703; 128-wide: four 1,236 / 1,063.  Over 2,500 calls (2 to 700 tokens of
// 1 to 12 agents behind 100 to 24,000) the better side is 0.1 % faster in the mean.
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
// agents of 4K-32K tokens 315 / 394 (128 / 256 rows), 280 rows of 128-wide heads, four agents of up to 6K 43.3 / 44.3, 300 rows of
// 192 + 128-wide ones behind 2,000 38.8 / 39.7, behind 8,000 65 / 68.  And where a compute unit's share is short: every
// workgroup of a shared unit leaves a record of its rows, and half the rows are half the record.  The line is at 448 tokens
// per compute unit; between 250 and 1,000 the sides differ by 6 %, either way, but for one point (512 new tokens, one agent, tokens per compute unit: 256-wide 250 55.9 / 58.4, 400 65.7 / 68.1, 560 78.5 / 81.6, 1,000 115 / 115,
// 2,200 209 / 202; 128-wide 250 40.3 / 38.5, 400 45.5 / 43.7, 560 51.7 / 49.2; 192 + 128 100 32.7 / 35.5, 400 47.3 / 52.6, 750
// 64.2 / 64.8; 64-wide 76 23.2 / 26.9, 282 32.7 / 31.6): over 2,500 calls no line between 250 and 1,000 is 0.02 % better.
inline int rows_shared(const ChunkSizes &s, int tokens)
{
    const int64_t wide = row_tiles(s, 256), narrow = row_tiles(s, 128);
    if (0.6 * narrow < wide) return 128;
    return (double)s.units * wide * tokens < 448.0 * s.compute_units ? 128 : 256;
}

// Whether a call may share its tiles out at all, whatever its lengths and window turn out to be: what a workspace is sized
// for.  The line is at two units per compute unit: a workgroup that takes an equal share holds its compute unit
// until the call ends, and a decode step on another stream, which gets in whenever a workgroup ends, waits for that
// long.  48 layers of 512 tokens behind 16,384 (1,536 units) take 7.15 ms with one unit per workgroup, 7.47 with equal
// shares; decode steps of 0.76 ms beside them took 2.1 and 4.9 ms when the line was drawn (7.63 and 8.04 ms of chunk).  Below the line,
// of that time too: layer by layer, 0.84 ms steps beside 512 tokens of ten agents of 4K-32K take 1.7 ms without shares and 2.65 with, beside
// one agent's (0.13 ms a call) 0.92.  Alone equal shares go on to win at 128-wide heads: four agents of 6,000, units per compute unit 2 510 / 509 (alone /
// shares), 4 1,013 / 994, 6 1,515 / 1,486; 256-wide 1.5 792 / 745, 2 941 / 955, 3 1,405 / 1,452, 6 2,800 / 2,881.
inline bool shares_fit(const ChunkSizes &s, int num_agents, int max_seq_len)
{
    const int64_t units = s.units * row_tiles(s, rows_shared(s, max_seq_len));
    return num_agents <= kMaxStreamAgents && max_seq_len > 256 && units < 2 * (int64_t)s.compute_units &&
           units * (max_seq_len / 32 + 2) < 0x3fffffff; // tiles (of 32 tokens and more) are numbered with 32-bit integers
}

// Whether equal shares are done before one unit per workgroup.  They even the load out, but every workgroup begins and ends up
// to two units more, leaves their records and a second kernel merges them: about 100 (256-wide) or 300 tokens of a 256-row
// workgroup, and up to 550 (250 at 192 + 128, 500 below) more as the units become as many as the compute
// units.  One unit per workgroup / equal shares, 256-wide: 512 tokens behind 2,000 107 / 61, behind 8,000 315 / 120, ten agents of 4K-32K 2,455 / 2,088; 2 tokens
// of ten agents behind 280 16.8 / 29.7, 512 of three behind 280 47.1 / 59.5, behind 700 62.0 / 69.2, behind 1,500 93.5 / 92.0.
// 128-wide: 512 behind 280 26.8 / 37.1, behind 700 34.1 / 42.6, behind 2,000 58.0 / 53.1, behind 8,000 167 / 109; 16 of
// ten agents behind 280 13.1 / 21.7, behind 1,500 29.9 / 26.9; a window of 1,024 on 512 behind 16,000 32.3 / 43.7.  192 + 128: 70
// of ten agents behind 280 17.9 / 34.4, 2 of three behind 700 17.8 / 17.3, 512 of one behind 1,500 57 / 42.  Over 2,500 calls the best
// form is 0.9 % faster in the mean than the one this takes (always sharing below two units per compute unit: 9.1 %, and up to twice the time).
// 87 of them are more than 10 % slower than the best, most of them a few tokens behind 300 to 1,100 that share and need not (2 to 140 tokens,
// 256-wide: up to 1.4 times): starts of 200 (256-wide) and 360 tokens would leave 49 and 0.7 %.
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
