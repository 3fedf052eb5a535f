// How a chunk call is cut into workgroups: host arithmetic on sizes alone (the lengths are on the device), in a header of
// its own so that it can be checked without a GPU.  Every figure beside a rule is the time of one attention call in us,
// 256 compute units, binary16 parameters, both sides measured in turn.
#pragma once
#include <cstdint>

namespace q4kv {

constexpr int kXcds = 8; // compute dies; consecutive workgroups go to consecutive dies

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

} // namespace q4kv
