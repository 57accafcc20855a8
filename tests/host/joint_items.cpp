// Reads mixed batches "n_q n_kv d page | prefix rows | query tokens and own keys of every row" (all rows carry the prefix) and prints how
// many row-tiled items their attention has and how many of them are joint (expand_batch; host arithmetic alone).  Ends with a
// message if some query token does not see the template once and its own keys once, up to itself, through its request's block table.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "relserve_internal.h"

using namespace relserve;

#define EXPECT(cond) do { if (!(cond)) { std::printf("FAILED line %d: %s\n", __LINE__, #cond); return 1; } } while (0)

int main() {
    int n_q, n_kv, d, page, prefix, rows;
    while (std::scanf("%d %d %d %d %d %d", &n_q, &n_kv, &d, &page, &prefix, &rows) == 6) {
        std::vector<int32_t> q(rows), own(rows), q_start(1, 0), ctx, pid(rows, 0);
        int max_blocks = 0;
        for (int r = 0; r < rows; ++r) {
            if (std::scanf("%d %d", &q[r], &own[r]) != 2) return 1;
            q_start.push_back(q_start.back() + q[r]);
            ctx.push_back(prefix + own[r]);
            max_blocks = std::max(max_blocks, (ctx[r] + page - 1) / page);
        }
        std::vector<int32_t> table((size_t)rows * max_blocks, 0);
        int next = prefix / page;
        for (int r = 0; r < rows; ++r)
            for (int i = 0; i < (ctx[r] + page - 1) / page; ++i) table[(size_t)r * max_blocks + i] = i < prefix / page ? i : next++;
        relserve_layer_config cfg{};
        cfg.hidden = n_q * d; cfg.n_q_heads = n_q; cfg.n_kv_heads = n_kv; cfg.head_dim = d; cfg.mlp_dim = 8; cfg.page_size = page;
        relserve_batch_desc desc{};
        desc.num_reqs = rows; desc.q_start = q_start.data(); desc.ctx_len = ctx.data(); desc.block_table = table.data();
        desc.max_blocks = max_blocks; desc.num_pages = next; desc.prefix_id = pid.data(); desc.num_prefixes = 1; desc.prefix_len = &prefix;
        HostBatch hb;
        if (const int32_t st = expand_batch(cfg, desc, true, &hb)) { std::printf("status %d\n", st); return 1; }
        const ItemLists& il = hb.items;
        const int T = hb.T, tile_tok = ATTN_BLOCK_M / (n_q / n_kv);
        std::vector<int> shared(T, 0), self(T, 0);
        int n_joint = 0, longest = 1 << 30;
        for (const AttnItem& it : il.items_prefix) {
            EXPECT(it.n_tok >= 1 && it.n_tok <= tile_tok && it.key_begin == 0 && it.key_end == prefix && (it.flags & ITEM_WRITE_PARTIAL));
            for (int i = 0; i < it.n_tok; ++i) ++shared[il.attn_tok[it.tok_off + i]];
        }
        for (const AttnItem& it : il.items_tile) {
            EXPECT(it.n_tok >= 1 && it.n_tok <= tile_tok);
            const int32_t* tok = il.attn_tok.data() + it.tok_off;
            if (!(it.flags & ITEM_JOINT)) {
                EXPECT(it.key_begin == prefix && (it.flags & ITEM_INIT_PARTIAL));
                for (int i = 0; i < it.n_tok; ++i) {
                    EXPECT(hb.tok_req[tok[i]] == it.bt_req && hb.tok_pos[tok[i]] < it.key_end);
                    ++self[tok[i]];
                }
                continue;
            }
            ++n_joint;
            EXPECT(it.flags == ITEM_JOINT && it.key_begin == 0 && it.key_end == prefix);
            const int32_t* seg = il.attn_tok.data() + it.pad0;
            int blocks = (prefix + 63) / 64, covered = 0;
            for (int i = 0; i < it.n_tok; ++i) ++shared[tok[i]];
            for (const int32_t* s = seg + 1; covered < it.n_tok; s += 4) {
                EXPECT(s + 4 <= il.attn_tok.data() + il.attn_tok.size());
                EXPECT(s[2] == covered && s[3] >= 1 && s[1] > prefix && s[1] <= ctx[s[0]]);
                for (int i = s[2]; i < s[2] + s[3]; ++i) {
                    EXPECT(hb.tok_req[tok[i]] == s[0] && hb.tok_pos[tok[i]] < s[1]);
                    ++self[tok[i]];
                }
                covered += s[3];
                blocks += (s[1] - prefix + 63) / 64;
            }
            EXPECT(covered == it.n_tok && seg[0] == blocks && blocks <= longest);   // longest first
            longest = blocks;
        }
        for (const AttnItem& it : il.items_split) ++self[it.pad0];
        for (int t = 0; t < T; ++t) EXPECT(shared[t] == 1 && self[t] >= 1);
        std::printf("%d %d\n", (int)il.items_tile.size(), n_joint);
    }
    return 0;
}
