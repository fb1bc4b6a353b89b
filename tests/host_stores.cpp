// CPU-only check of the rule that leaves a call's stores to the L2 (kv_engine.hpp): for each
// line "vec piece layer_first block_bytes run n_out n_in" on stdin, 1 or 0 on stdout.  The out
// slots are runs of `run` consecutive ones with gaps between them.
#include <cstdio>
#include <vector>

#include "../paper_2601_20309_amd/csrc/kv_engine.hpp"

int main()
{
    long long piece, block, n_out, n_in;
    int vec, layer_first, run;
    while (std::scanf("%d %lld %d %lld %d %lld %lld", &vec, &piece, &layer_first, &block, &run, &n_out, &n_in) == 7) {
        std::vector<int32_t> slots;
        for (long long i = 0; i < n_out; i++) slots.push_back((int32_t)(i + i / run));
        std::printf("%d\n", dkv::leaves_to_l2(vec, (uint64_t)piece, layer_first != 0, (uint64_t)block, slots.data(), n_out, n_in) ? 1 : 0);
    }
    return 0;
}
