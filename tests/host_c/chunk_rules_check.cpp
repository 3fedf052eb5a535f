// Prints what the launch rules of the chunk kernel say for the calls given on the command line, four numbers and a list each:
// units, rows of a unit, query heads per KV head, max_seq_len, then q_len and the windows ("512:0" or "512:1024,0").
#include <cstdio>
#include <cstdlib>

#include "../../paper_2603_04428_amd/csrc/chunk_rules.h"

int main(int argc, char **argv)
{
    for (int i = 1; i + 4 < argc; i += 5) {
        const int n_rep = atoi(argv[i + 2]), max_seq_len = atoi(argv[i + 3]);
        const q4kv::ChunkSizes s{atoll(argv[i]), atoll(argv[i + 1]), 256};
        char *at = argv[i + 4];
        const int q_len = (int)strtol(at, &at, 10);
        int tokens[128], n = 0;
        while (*at) tokens[n++] = q4kv::visible_tokens(max_seq_len, (int)strtol(at + 1, &at, 10), q_len, n_rep);
        printf("%d\n", q4kv::rows_alone(s, tokens, n));
    }
    return 0;
}
