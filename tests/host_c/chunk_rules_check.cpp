// Prints what the launch rules of the chunk kernel say for the calls given on the command line -- rows per workgroup without shares;
// with them; 1 if shares pay; 1 if a workspace is sized for them -- six numbers and a list each: key width, agents, units,
// rows of a unit, query heads per KV head, max_seq_len, then q_len and the windows ("512:0" or "512:1024,0").
#include <cstdio>
#include <cstdlib>

#include "../../paper_2603_04428_amd/csrc/chunk_rules.h"

int main(int argc, char **argv)
{
    for (int i = 1; i + 6 < argc; i += 7) {
        const int k_dim = atoi(argv[i]), agents = atoi(argv[i + 1]), n_rep = atoi(argv[i + 4]), max_seq_len = atoi(argv[i + 5]);
        const q4kv::ChunkSizes s{atoll(argv[i + 2]), atoll(argv[i + 3]), 256};
        char *at = argv[i + 6];
        const int q_len = (int)strtol(at, &at, 10);
        int tokens[128], n = 0;
        while (*at) tokens[n++] = q4kv::visible_tokens(max_seq_len, (int)strtol(at + 1, &at, 10), q_len, n_rep);
        printf("%d %d %d %d\n", q4kv::rows_alone(s, tokens, n), q4kv::rows_shared(s, tokens[0]),
               n == 1 && q4kv::shares_pay(s, k_dim, tokens[0]), q4kv::shares_fit(s, agents, max_seq_len));
    }
    return 0;
}
