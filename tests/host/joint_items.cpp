// Reads mixed batches "n_q n_kv d page | prefix groups rows | query tokens and own keys of every row" (every row carries the prefix of its
// group, the groups one behind the other) and prints how
// many row-tiled items their attention has, how many of them are joint, whether the template's state of decode rows is kept in
// slots, and how many items are joint without slots (expand_batch; host arithmetic alone).  Ends with a message if some query token does not see the template once and its own
// keys once, up to itself, through its request's block table, or if a slot is out of range, written twice or not merged.
#include <algorithm>
#include <cstdio>
#include <set>
#include <vector>

#include "relserve_internal.h"

using namespace relserve;

#define EXPECT(cond) do { if (!(cond)) { std::printf("FAILED line %d: %s\n", __LINE__, #cond); return 1; } } while (0)

static int check(const HostBatch& hb, const ItemLists& il, const std::vector<int32_t>& q, const std::vector<int32_t>& own,
                 const std::vector<int32_t>& ctx, int prefix, int tile_tok, int& n_joint) {
    const int T = hb.T;
    std::vector<int> shared(T, 0), self(T, 0);
    std::set<int> written;
    int longest = 1 << 30;
    auto prefix_item = [&](const AttnItem& it) {
        EXPECT(it.n_tok >= 1 && it.n_tok <= tile_tok && it.key_begin % 64 == 0 && it.key_end <= prefix && (it.flags & ITEM_WRITE_PARTIAL));
        EXPECT(((it.flags & ITEM_SLOTS) != 0) == il.in_slots);
        for (int i = 0; i < it.n_tok; ++i) {
            shared[il.attn_tok[it.tok_off + i]] += it.key_end - it.key_begin;
            if (it.flags & ITEM_SLOTS) EXPECT(written.insert(il.attn_tok[it.pad0 + i] + it.pad1).second);
        }
        return 0;
    };
    for (const AttnItem& it : il.items_prefix)
        if (prefix_item(it)) return 1;
    for (const AttnItem& it : il.items_tile) {
        EXPECT(it.n_tok >= 1 && it.n_tok <= tile_tok);
        const int32_t* tok = il.attn_tok.data() + it.tok_off;
        const int blocks = it.flags & ITEM_JOINT ? il.attn_tok[it.pad0] : (it.key_end - it.key_begin + 63) / 64;
        EXPECT(blocks <= longest);   // longest first
        longest = blocks;
        if (it.flags & ITEM_WRITE_PARTIAL) {
            if (prefix_item(it)) return 1;
        } else if (!(it.flags & ITEM_JOINT)) {
            EXPECT(it.key_begin == prefix && (it.flags & ITEM_INIT_PARTIAL));
            for (int i = 0; i < it.n_tok; ++i) {
                EXPECT(hb.tok_req[tok[i]] == it.bt_req && hb.tok_pos[tok[i]] < it.key_end);
                self[tok[i]] += own[it.bt_req];
            }
        } else {
            ++n_joint;
            EXPECT(it.flags == ITEM_JOINT && it.key_begin == 0 && it.key_end == prefix);
            const int32_t* seg = il.attn_tok.data() + it.pad0;
            int all = (prefix + 63) / 64, covered = 0;
            for (int i = 0; i < it.n_tok; ++i) shared[tok[i]] += prefix;
            for (const int32_t* s = seg + 1; covered < it.n_tok; s += 4) {
                EXPECT(s + 4 <= il.attn_tok.data() + il.attn_tok.size());
                EXPECT(s[2] == covered && s[3] >= 1 && s[1] > prefix && s[1] <= ctx[s[0]]);
                for (int i = s[2]; i < s[2] + s[3]; ++i) {
                    EXPECT(hb.tok_req[tok[i]] == s[0] && hb.tok_pos[tok[i]] < s[1]);
                    self[tok[i]] += own[s[0]];
                }
                covered += s[3];
                all += (s[1] - prefix + 63) / 64;
            }
            EXPECT(covered == it.n_tok && seg[0] == all);
        }
    }
    for (const AttnItem& it : il.items_split) {
        EXPECT(it.key_begin >= prefix && it.key_begin < it.key_end);
        self[it.pad0] += it.key_end - it.key_begin;
        if (it.flags & ITEM_WRITE_PARTIAL) EXPECT(written.insert(it.pad1).second);
    }
    for (int t = 0; t < T; ++t) EXPECT(shared[t] == prefix && self[t] == own[hb.tok_req[t]]);
    size_t merged = 0;
    for (const MergeItem& m : il.merge_items) {
        EXPECT(q[hb.tok_req[m.tok]] == 1 && m.n_chunks > 1);
        for (int c = 0; c < m.n_chunks; ++c) EXPECT(written.count(m.first_slot + c));
        merged += m.n_chunks;
    }
    EXPECT(merged == written.size());
    const int64_t cap = il.n_scratch_slots > 0 ? il.n_scratch_slots : split_slot_cap(T);
    EXPECT(written.empty() || (*written.begin() >= 0 && *written.rbegin() < cap));
    return 0;
}

int main() {
    int n_q, n_kv, d, page, prefix, groups, rows;
    while (std::scanf("%d %d %d %d %d %d %d", &n_q, &n_kv, &d, &page, &prefix, &groups, &rows) == 7) {
        std::vector<int32_t> q(rows), own(rows), q_start(1, 0), ctx, pid(rows, 0);
        int max_blocks = 0;
        for (int r = 0; r < rows; ++r) {
            if (std::scanf("%d %d", &q[r], &own[r]) != 2) return 1;
            q_start.push_back(q_start.back() + q[r]);
            ctx.push_back(prefix + own[r]);
            pid[r] = r * groups / rows;
            max_blocks = std::max(max_blocks, (ctx[r] + page - 1) / page);
        }
        std::vector<int32_t> table((size_t)rows * max_blocks, 0);
        const std::vector<int32_t> prefix_len(groups, prefix);
        const int shared = prefix / page;
        int next = groups * shared;
        for (int r = 0; r < rows; ++r)
            for (int i = 0; i < (ctx[r] + page - 1) / page; ++i) table[(size_t)r * max_blocks + i] = i < shared ? pid[r] * shared + i : next++;
        relserve_layer_config cfg{};
        cfg.hidden = n_q * d; cfg.n_q_heads = n_q; cfg.n_kv_heads = n_kv; cfg.head_dim = d; cfg.mlp_dim = 8; cfg.page_size = page;
        relserve_batch_desc desc{};
        desc.num_reqs = rows; desc.q_start = q_start.data(); desc.ctx_len = ctx.data(); desc.block_table = table.data();
        desc.max_blocks = max_blocks; desc.num_pages = next; desc.prefix_id = pid.data(); desc.num_prefixes = groups; desc.prefix_len = prefix_len.data();
        HostBatch hb;
        if (const int32_t st = expand_batch(cfg, desc, true, &hb)) { std::printf("status %d\n", st); return 1; }
        int n_joint = 0, other = 0;
        if (check(hb, hb.items, q, own, ctx, prefix, ATTN_BLOCK_M / (n_q / n_kv), n_joint)) return 1;
        if (hb.items.in_slots && check(hb, hb.no_slots, q, own, ctx, prefix, ATTN_BLOCK_M / (n_q / n_kv), other)) return 1;
        std::printf("%d %d %d %d\n", (int)hb.items.items_tile.size(), n_joint, (int)hb.items.in_slots, hb.items.in_slots ? other : n_joint);
    }
    return 0;
}
