// Prints the attention plan of every line of "batch max_pages_per_req n_q_heads n_kv_heads head_dim max_spec_len dtype"
// read from standard input: split and direct flag of a chain call, of a tree call, tokens per block, bytes of
// both and of the query, wavefronts per row of the chain's combine kernel.  With an argument: possible splits per request of
// the chain call, whether the main kernel merges them, whether the chain's, and the tree's, wavefronts split a unit's rows.
#include <cstdio>

#include "../../paper_2503_05096_amd/csrc/adaspec_internal.h"

int main(int argc, char **)
{
    adaspec_attn_dims d = {};
    d.page_size = 16;
    d.num_pages = 1;
    while (scanf("%d %d %d %d %d %d %d", &d.batch, &d.max_pages_per_req, &d.n_q_heads, &d.n_kv_heads, &d.head_dim, &d.max_spec_len,
                 &d.dtype) == 7) {
        d.out_dtype = d.dtype;
        d.total_q = d.batch * (d.max_spec_len + 1);
        const adaspec::AttnKind kind = adaspec::attn_kind(d);
        const adaspec::AttnPlan chain = adaspec::make_attn_plan(d, kind, false), tree = adaspec::make_attn_plan(d, kind, true);
        if (argc > 1) {
            printf("%d %d %d %d\n", chain.per_req, (int)chain.merged, (int)chain.row_split, (int)tree.row_split);
            continue;
        }
        printf("%d %d %d %d %d %zu %zu %zu %d\n", chain.split_tokens, (int)chain.direct, tree.split_tokens, (int)tree.direct,
               chain.block_tokens, chain.total_bytes, tree.total_bytes, adaspec_verify_attn_workspace_bytes(&d), adaspec::attn_combine_waves(chain, d));
    }
    return 0;
}
