// Reads batches of decode rows "n_q n_kv d page | rows prefix members | own keys of every row" and prints how their attention is
// cut (expand_batch; host arithmetic alone): scratch slots, longest wave item, longest prefix item in keys, the same two of the
// list without slots.  Ends with a message if the items of a list do not cover every row's keys exactly once, if a slot
// is written twice, read without being written or out of range, or if a row that has parts is not merged.
#include <algorithm>
#include <cstdio>
#include <map>
#include <utility>
#include <vector>

#include "relserve_internal.h"

using namespace relserve;

#define EXPECT(cond) do { if (!(cond)) { std::printf("FAILED line %d: %s\n", __LINE__, #cond); return false; } } while (0)

static bool check(const ItemLists& il, const relserve_layer_config& cfg, const std::vector<int32_t>& ctx, int& longest_own, int& longest_prefix) {
    const int B = (int)ctx.size(), tile_tok = ATTN_BLOCK_M / (cfg.n_q_heads / cfg.n_kv_heads);
    std::vector<std::vector<std::pair<int, int>>> keys(B);   // per row: key ranges of its items
    std::map<int, int> slot_row;                             // slot -> row that wrote it (plan with slots, or chunks of rows)
    std::vector<int> from_prefix(B, 0), finished(B, 0);
    longest_own = longest_prefix = 0;
    for (const AttnItem& it : il.items_prefix) {
        EXPECT(it.n_tok >= 1 && it.n_tok <= tile_tok && it.key_begin < it.key_end && it.key_begin % 64 == 0);
        EXPECT(it.flags & ITEM_WRITE_PARTIAL);
        EXPECT(((it.flags & ITEM_SLOTS) != 0) == (il.n_scratch_slots > 0));
        longest_prefix = std::max(longest_prefix, it.key_end - it.key_begin);
        for (int i = 0; i < it.n_tok; ++i) {
            const int t = il.attn_tok[it.tok_off + i];
            keys[t].push_back({it.key_begin, it.key_end});
            ++from_prefix[t];
            if (it.flags & ITEM_SLOTS) EXPECT(slot_row.emplace(il.attn_tok[it.pad0 + i] + it.pad1, t).second);
        }
    }
    EXPECT(il.items_tile.empty());
    for (const AttnItem& it : il.items_split) {
        EXPECT(it.n_tok == 1 && it.key_begin < it.key_end);
        longest_own = std::max(longest_own, it.key_end - it.key_begin);
        keys[it.pad0].push_back({it.key_begin, it.key_end});
        if (it.flags & ITEM_WRITE_PARTIAL) EXPECT(slot_row.emplace(it.pad1, it.pad0).second);
        else ++finished[it.pad0];
    }
    const int cap = il.n_scratch_slots > 0 ? il.n_scratch_slots : (int)split_slot_cap(B);
    EXPECT(il.n_scratch_slots <= scratch_slot_cap(cfg.n_q_heads, cfg.head_dim));
    size_t merged = 0;
    for (const MergeItem& m : il.merge_items) {
        ++finished[m.tok];
        for (int c = 0; c < m.n_chunks; ++c, ++merged) {
            const auto s = slot_row.find(m.first_slot + c);
            EXPECT(m.first_slot + c < cap && s != slot_row.end() && s->second == m.tok);
        }
    }
    EXPECT(merged == slot_row.size());
    for (int t = 0; t < B; ++t) {
        EXPECT(finished[t] == 1);
        std::sort(keys[t].begin(), keys[t].end());
        int at = 0;
        for (auto [b, e] : keys[t]) {
            EXPECT(b == at);
            at = e;
        }
        EXPECT(at == ctx[t]);
    }
    return true;
}

int main() {
    relserve_layer_config cfg{};
    int rows, prefix, members;
    while (std::scanf("%d %d %d %d %d %d %d", &cfg.n_q_heads, &cfg.n_kv_heads, &cfg.head_dim, &cfg.page_size, &rows, &prefix, &members) == 7) {
        cfg.hidden = cfg.n_q_heads * cfg.head_dim, cfg.mlp_dim = 512, cfg.rms_eps = 1e-5f, cfg.rope_base = 10000.0f;
        const int P = cfg.page_size;
        std::vector<int32_t> ctx(rows), q_start(rows + 1), pid(rows), bt, plen;
        int max_blocks = 1, next = prefix / P;
        for (int r = 0; r < rows; ++r) {
            if (std::scanf("%d", &ctx[r]) != 1) return 2;
            pid[r] = prefix > 0 && r < members ? 0 : -1;
            ctx[r] += pid[r] == 0 ? prefix : 0;
            q_start[r + 1] = r + 1;
            max_blocks = std::max(max_blocks, (ctx[r] + P - 1) / P);
        }
        bt.assign((size_t)rows * max_blocks, 0);
        for (int r = 0; r < rows; ++r)
            for (int i = 0; i < (ctx[r] + P - 1) / P; ++i) bt[(size_t)r * max_blocks + i] = pid[r] == 0 && i < prefix / P ? i : next++;
        if (prefix > 0) plen.push_back(prefix);
        relserve_batch_desc d{};
        d.num_reqs = rows, d.max_blocks = max_blocks, d.q_start = q_start.data(), d.ctx_len = ctx.data(), d.block_table = bt.data();
        d.prefix_id = pid.data(), d.num_prefixes = (int32_t)plen.size(), d.prefix_len = plen.data(), d.num_pages = next;
        HostBatch hb;
        if (int rc = expand_batch(cfg, d, true, &hb)) {
            std::printf("FAILED: status %d\n", rc);
            return 1;
        }
        int own, pre, own2 = 0, pre2 = 0;
        if (!check(hb.items, cfg, ctx, own, pre)) return 1;
        if (hb.items.n_scratch_slots > 0 && !check(hb.no_slots, cfg, ctx, own2, pre2)) return 1;
        std::printf("%d %d %d %d %d\n", hb.items.n_scratch_slots, own, pre, own2, pre2);
    }
    return 0;
}
