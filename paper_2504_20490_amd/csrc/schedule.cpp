// Cost-sorted, XCD-aware work lists for packed variable-length causal attention.
//
// The paper balances mixed-length sequences across pipelines with a cost model
// evaluated on the CPU while the GPU is busy (Appendix "Scenario-specific
// Planning", mixed-length case).  Inside one GPU the same long tail appears
// again: under the causal mask q tile t of a sequence visits t+1 key tiles, so
// one 16K sequence holds most of a pack's work.  The list built here is the
// on-device analogue: every (sequence, tile, head) is an item with a known cost,
// and the order in which workgroups pick items up is planned on the host, once
// per pack, and reused by every layer and both passes.
//
// Placement follows the chip: workgroups are handed to the 8 XCDs round-robin by
// workgroup index and every XCD has its own L2.  Items that stream the same K/V
// (all q tiles and all query heads of one (sequence, kv head)) are therefore kept
// in the same queue (= the same XCD) and adjacent in it, so that one tile's K/V
// fetch is an L2 hit for its neighbours.  Chains heavier than a fraction of the
// total are cut into segments so that queues can be balanced; segments go to the
// least-loaded queue, heaviest first (longest-processing-time rule), and a queue
// runs its segments in order of their most expensive item.
#include "schedule.hpp"

#include <algorithm>
#include <numeric>

namespace hspmd {

std::string check_pack(const int32_t* cu, int32_t num_seqs, int32_t hq, int32_t hkv) {
    if (!cu) return "cu_seqlens is NULL";
    if (num_seqs < 0) return "num_seqs is negative";
    if (hq <= 0 || hkv <= 0) return "head counts must be positive";
    if (hq % hkv != 0) return "local_q_heads must be a multiple of local_kv_heads (cut an uneven share on KV-group boundaries)";
    if (cu[0] != 0) return "cu_seqlens[0] must be 0";
    for (int32_t i = 0; i < num_seqs; ++i)
        if (cu[i + 1] < cu[i]) return "cu_seqlens must be non-decreasing";
    return std::string();
}

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

int64_t item_cost(hspmd_list_kind kind, int32_t seq_len, int32_t tile, int32_t group) {
    if (kind == HSPMD_LIST_DKV) {
        const int64_t first_row = (int64_t)tile * kDkvKTile;          // rows r >= first key of the tile
        if (first_row >= seq_len) return 0;
        return ceil_div(seq_len - first_row, kDkvQTile) * group;
    }
    const int64_t last_key = std::min<int64_t>(seq_len, (int64_t)(tile + 1) * kFwdQTile);
    if ((int64_t)tile * kFwdQTile >= seq_len) return 0;
    return ceil_div(last_key, kFwdKTile);
}

// The placement, shared by the packed and the block lists: chains are cut into segments, segments are assigned to queues
// by the longest-processing-time rule, each queue is ordered, the queues are interleaved.
//
// The list is rebuilt for every pack, on the host, ahead of that pack's first kernel, so its cost counts.  Two facts keep
// it at a few nanoseconds per item: the kv heads of a sequence have equal chains, so costs and cuts are computed once per
// sequence and not per head; and nothing but segment descriptors is sorted, items are generated once, straight into their
// slots.  A whole refill (two lists and their upload), against chains held as vectors of items: 57 sequences of 32 .. 506
// tokens, 16 heads (2 x 2496 items) 231 -> 38 us; 14 sequences, 32 heads on 8 (16576 + 4144 items) 167 -> 67 us.
namespace {

// A run of items of one sequence's chain; the chains of all `copies` kv heads of the sequence hold it.
struct SegmentClass {
    int64_t cost, first_cost;   // of the whole run; of its first (most expensive) item
    int64_t order0, stride;     // creation index of kv head g's copy: order0 + g * stride
    int32_t seq, first, count;
};

// Walks the segments of all kv heads in the order (key descending, creation index ascending): `visit(class, kv head)`.
// Copies of one class carry consecutive heads and classes of one sequence alternate head by head, so only the classes are
// sorted and runs of equal keys within a sequence are walked head-first.
template <typename Key, typename Visit>
void walk_segments(const std::vector<SegmentClass>& classes, int32_t copies, Key key, Visit visit) {
    std::vector<int32_t> by_key(classes.size());
    std::iota(by_key.begin(), by_key.end(), 0);
    std::stable_sort(by_key.begin(), by_key.end(), [&](int32_t a, int32_t b) { return key(classes[a]) > key(classes[b]); });
    for (size_t i = 0; i < by_key.size();) {
        size_t end = i + 1;
        while (end < by_key.size() && key(classes[by_key[end]]) == key(classes[by_key[i]]) &&
               classes[by_key[end]].seq == classes[by_key[i]].seq)
            ++end;
        for (int32_t g = 0; g < copies; ++g)
            for (size_t j = i; j < end; ++j) visit(classes[by_key[j]], g);
        i = end;
    }
}

// chain_len(s): items of one kv head's chain of sequence s, most expensive first; cost_of(s, i): of its i-th item;
// make(s, g, i): that item for kv head g.  one_head: a chain holds one item per tile, not one per query head of a group.
template <typename Item, typename ChainLen, typename Cost, typename Make>
std::vector<Item> place_chains(int32_t num_seqs, int32_t kv_heads, int32_t num_queues, bool one_head, ChainLen chain_len,
                               Cost cost_of, Make make, Item pad) {
    int64_t total_cost = 0;
    for (int32_t s = 0; s < num_seqs; ++s) {
        const int32_t n = chain_len(s);
        for (int32_t i = 0; i < n; ++i) total_cost += cost_of(s, i);
    }
    total_cost *= kv_heads;

    // cut chains into segments no heavier than 1/(4 * queues) of the total; fewer than two chains per queue are cut finer:
    // their few segments left the heaviest queue a tenth above the mean (5 heads: one document of 16001 tokens, forward 355 ->
    // 345, dK/dV 612 -> 586 us; one of 24976 tokens 445 -> 416, dQ 592 -> 550, dK/dV 802 -> 749 us).  With more chains the
    // coarse cut balances as well and keeps more of a chain's K and V in one L2.  (Chains with several query heads keep the coarse
    // cut, so that a group's heads of one tile stay together.)
    int64_t chains = 0;
    for (int32_t s = 0; s < num_seqs; ++s) chains += chain_len(s) > 0 ? kv_heads : 0;
    const int64_t parts = one_head && chains < 2 * (int64_t)num_queues ? 16 : 4;
    const int64_t cap = std::max<int64_t>(1, total_cost / (num_queues * parts));
    std::vector<SegmentClass> classes;
    int64_t segments = 0;
    for (int32_t s = 0; s < num_seqs; ++s) {
        const int32_t n = chain_len(s);
        if (n <= 0) continue;
        const size_t first_class = classes.size();
        SegmentClass seg{0, 0, 0, 0, s, 0, 0};
        for (int32_t i = 0; i < n; ++i) {
            // an item that only writes zeros (block variant) still occupies a workgroup slot: weight 1, so that
            // such items spread over the queues instead of piling up in one
            const int64_t c = std::max<int64_t>(1, cost_of(s, i));
            if (seg.count > 0 && seg.cost + c > cap) {
                classes.push_back(seg);
                seg = SegmentClass{0, 0, 0, 0, s, i, 0};
            }
            if (seg.count == 0) seg.first_cost = c;
            ++seg.count;
            seg.cost += c;
        }
        classes.push_back(seg);
        const int64_t per_head = (int64_t)(classes.size() - first_class);
        for (int64_t k = 0; k < per_head; ++k) {
            classes[first_class + k].order0 = segments + k;
            classes[first_class + k].stride = per_head;
        }
        segments += per_head * kv_heads;
    }
    if (classes.empty()) return {};

    // longest-processing-time assignment: each segment, heaviest first, goes to the least loaded queue (the lowest index
    // among equals).  The loads are a binary heap whose root is replaced, never popped and pushed.
    struct Load {
        int64_t load;
        int32_t queue;
        bool before(const Load& o) const { return load != o.load ? load < o.load : queue < o.queue; }
    };
    std::vector<Load> heap((size_t)num_queues);
    for (int32_t x = 0; x < num_queues; ++x) heap[x] = Load{0, x};   // sorted, hence a heap
    std::vector<int32_t> queue_of((size_t)segments);
    std::vector<int64_t> length((size_t)num_queues, 0);
    walk_segments(classes, kv_heads, [](const SegmentClass& c) { return c.cost; }, [&](const SegmentClass& c, int32_t g) {
        Load root = heap[0];
        queue_of[(size_t)(c.order0 + g * c.stride)] = root.queue;
        length[(size_t)root.queue] += c.count;
        root.load += c.cost;
        size_t at = 0;
        for (size_t child = 1; child < heap.size(); child = 2 * at + 1) {
            if (child + 1 < heap.size() && heap[child + 1].before(heap[child])) ++child;
            if (!heap[child].before(root)) break;
            heap[at] = heap[child];
            at = child;
        }
        heap[at] = root;
    });

    // inside a queue: segments by their most expensive item, then creation order; slot p belongs to queue
    // p % num_queues, short queues are padded at their end
    const int64_t longest = *std::max_element(length.begin(), length.end());
    std::vector<Item> out((size_t)(longest * num_queues), pad);
    std::vector<int64_t> cursor((size_t)num_queues);
    std::iota(cursor.begin(), cursor.end(), (int64_t)0);
    walk_segments(classes, kv_heads, [](const SegmentClass& c) { return c.first_cost; }, [&](const SegmentClass& c, int32_t g) {
        int64_t& slot = cursor[(size_t)queue_of[(size_t)(c.order0 + g * c.stride)]];
        for (int32_t i = c.first; i < c.first + c.count; ++i, slot += num_queues) out[(size_t)slot] = make(c.seq, g, i);
    });
    return out;
}

}  // namespace

// The two orders without placement: used only to measure what the default order buys.
static std::vector<hspmd_work_item> build_plain_list(hspmd_list_kind kind, const int32_t* cu, int32_t num_seqs,
                                                     int32_t hq, int32_t hkv, hspmd_order order) {
    const int32_t group = hq / hkv;
    const int tile_rows = (kind == HSPMD_LIST_DKV) ? kDkvKTile : kFwdQTile;
    const int32_t heads = (kind == HSPMD_LIST_DKV) ? hkv : hq;
    std::vector<hspmd_work_item> out;
    for (int32_t s = 0; s < num_seqs; ++s) {
        const int32_t len = cu[s + 1] - cu[s];
        if (len <= 0) continue;
        const int32_t n_tiles = (int32_t)ceil_div(len, tile_rows);
        for (int32_t t = 0; t < n_tiles; ++t)
            for (int32_t h = 0; h < heads; ++h) out.push_back({cu[s], len, t, h});
    }
    if (order == HSPMD_ORDER_COST)
        std::stable_sort(out.begin(), out.end(), [&](const hspmd_work_item& a, const hspmd_work_item& b) {
            return item_cost(kind, a.seq_len, a.tile, group) > item_cost(kind, b.seq_len, b.tile, group);
        });
    return out;
}

std::vector<hspmd_work_item> build_work_list(hspmd_list_kind kind, const int32_t* cu, int32_t num_seqs,
                                             int32_t hq, int32_t hkv, int32_t num_queues, hspmd_order order) {
    if (order != HSPMD_ORDER_XCD_COST) return build_plain_list(kind, cu, num_seqs, hq, hkv, order);
    const int32_t group = hq / hkv;
    const int tile_rows = (kind == HSPMD_LIST_DKV) ? kDkvKTile : kFwdQTile;

    // a chain: all items that share one (sequence, kv head), most expensive first
    auto tile_of = [=](int32_t len, int32_t i) {
        return kind == HSPMD_LIST_DKV ? i : (int32_t)ceil_div(len, tile_rows) - 1 - i / group;
    };
    return place_chains<hspmd_work_item>(
        num_seqs, hkv, num_queues, kind == HSPMD_LIST_DKV || group == 1,
        [&](int32_t s) {
            const int32_t n_tiles = (int32_t)ceil_div(cu[s + 1] - cu[s], tile_rows);
            return kind == HSPMD_LIST_DKV ? n_tiles : n_tiles * group;
        },
        [&](int32_t s, int32_t i) {
            const int32_t len = cu[s + 1] - cu[s];
            return item_cost(kind, len, tile_of(len, i), group);
        },
        [&](int32_t s, int32_t g, int32_t i) {
            const int32_t len = cu[s + 1] - cu[s];
            return hspmd_work_item{cu[s], len, tile_of(len, i), kind == HSPMD_LIST_DKV ? g : g * group + i % group};
        },
        hspmd_work_item{0, 0, -1, 0});
}

PassLoad pass_load(hspmd_list_kind kind, const int32_t* cu, int32_t num_seqs, int32_t hq, int32_t hkv) {
    const int tile_rows = (kind == HSPMD_LIST_DKV) ? kDkvKTile : kFwdQTile;
    PassLoad load;
    for (int32_t s = 0; s < num_seqs; ++s) {
        const int32_t len = cu[s + 1] - cu[s], n_tiles = (int32_t)ceil_div(len, tile_rows);
        for (int32_t t = 0; t < n_tiles; ++t) {
            const int64_t c = item_cost(kind, len, t, hq / hkv);
            load.total += c;
            load.heaviest = std::max(load.heaviest, c);
        }
    }
    load.total *= (kind == HSPMD_LIST_DKV) ? hkv : hq;
    return load;
}

// ------------------------------------------------------------------------------ cost model
// The paper's planner dispatches mixed-length sequences with a cost model evaluated on the CPU (Appendix
// "Scenario-specific Planning", mixed-length case); this is the per-operator predictor for the attention
// kernels of this library.  Fitted by relative least squares to 40 packs per head_dim: mean absolute error
// 6-8 %, at most 15-32 % (on packs that take about a hundred microseconds).
PassCost pass_cost_coefficients(hspmd_list_kind kind, int32_t head_dim) {
    static const PassCost k128[3] = {{13.1, 1.655, 10.37}, {7.6, 2.168, 18.64}, {24.8, 1.620, 11.66}};
    static const PassCost k64[3] = {{13.1, 1.045, 6.22}, {7.6, 1.239, 9.02}, {18.5, 1.062, 6.41}};
    return (head_dim == 64 ? k64 : k128)[(int)kind];
}

double estimate_pass_us(hspmd_list_kind kind, const int32_t* cu, int32_t num_seqs, int32_t hq, int32_t hkv, int32_t head_dim) {
    const std::vector<hspmd_work_item> list = build_work_list(kind, cu, num_seqs, hq, hkv, kNumXcd);
    if (list.empty()) return 0.0;
    const PassCost c = pass_cost_coefficients(kind, head_dim);
    const int32_t group = hq / hkv;
    // workgroups resident per XCD: 32 compute units, two workgroups each in the forward and dQ passes, one in dK/dV
    const double slots = kind == HSPMD_LIST_DKV ? 32.0 : 64.0;
    double queue_weight[kNumXcd] = {0};
    double heaviest = 0.0;
    for (size_t p = 0; p < list.size(); ++p) {
        if (list[p].tile < 0) continue;
        const double w = (double)item_cost(kind, list[p].seq_len, list[p].tile, group) * c.step_us + c.item_us;
        queue_weight[p % kNumXcd] += w;
        heaviest = std::max(heaviest, w);
    }
    double worst = 0.0;
    for (double w : queue_weight) worst = std::max(worst, w);
    return c.launch_us + std::max(worst / slots, heaviest);
}

// ------------------------------------------------------------------------------ block variant
std::string check_block_pack(const int32_t* cu_q, const int32_t* cu_k, const int32_t* q_pos, const int32_t* k_pos,
                             int32_t num_seqs, int32_t hq, int32_t hkv) {
    if (!cu_q || !cu_k) return "cu_seqlens is NULL";
    if (num_seqs < 0) return "num_seqs is negative";
    if (num_seqs > 0 && (!q_pos || !k_pos)) return "chunk positions are NULL";
    if (hq <= 0 || hkv <= 0) return "head counts must be positive";
    if (hq % hkv != 0) return "local_q_heads must be a multiple of local_kv_heads (cut an uneven share on KV-group boundaries)";
    if (cu_q[0] != 0 || cu_k[0] != 0) return "cu_seqlens[0] must be 0";
    for (int32_t i = 0; i < num_seqs; ++i) {
        if (cu_q[i + 1] < cu_q[i] || cu_k[i + 1] < cu_k[i]) return "cu_seqlens must be non-decreasing";
        if (q_pos[i] < 0 || k_pos[i] < 0) return "chunk positions must be non-negative";
        // positions of the last row / key must stay in int32 together with the tile arithmetic
        if ((int64_t)q_pos[i] + (cu_q[i + 1] - cu_q[i]) > (int64_t)1 << 30 ||
            (int64_t)k_pos[i] + (cu_k[i + 1] - cu_k[i]) > (int64_t)1 << 30)
            return "chunk position + length above 2^30";
    }
    return std::string();
}

int64_t block_item_cost(hspmd_list_kind kind, const hspmd_block_item& it, int32_t group) {
    if (kind == HSPMD_LIST_DKV) {
        // rows r >= key0 - offset see the tile's first key
        if ((int64_t)it.tile * kDkvKTile >= it.k_len) return 0;
        const int64_t first_row = std::max<int64_t>(0, (int64_t)it.tile * kDkvKTile - it.offset);
        const int64_t first_qt = first_row / kDkvQTile;
        const int64_t n_qt = ceil_div(it.q_len, kDkvQTile);
        return std::max<int64_t>(0, n_qt - first_qt) * group;
    }
    if ((int64_t)it.tile * kFwdQTile >= it.q_len) return 0;
    const int64_t last_row = std::min<int64_t>(it.q_len, (int64_t)(it.tile + 1) * kFwdQTile);   // exclusive
    const int64_t kv_end = std::max<int64_t>(0, std::min<int64_t>(it.k_len, last_row + it.offset));
    return ceil_div(kv_end, kFwdKTile);
}

std::vector<hspmd_block_item> build_block_list(hspmd_list_kind kind, const int32_t* cu_q, const int32_t* cu_k,
                                               const int32_t* q_pos, const int32_t* k_pos, int32_t num_seqs,
                                               int32_t hq, int32_t hkv, int32_t num_queues) {
    const int32_t group = hq / hkv;
    const int tile_rows = (kind == HSPMD_LIST_DKV) ? kDkvKTile : kFwdQTile;
    auto rows_of = [&](int32_t s) { return (kind == HSPMD_LIST_DKV) ? cu_k[s + 1] - cu_k[s] : cu_q[s + 1] - cu_q[s]; };
    auto make = [&](int32_t s, int32_t g, int32_t i) {
        hspmd_block_item it{cu_q[s], cu_q[s + 1] - cu_q[s], cu_k[s], cu_k[s + 1] - cu_k[s], q_pos[s] - k_pos[s], 0, 0, q_pos[s]};
        it.tile = kind == HSPMD_LIST_DKV ? i : (int32_t)ceil_div(rows_of(s), tile_rows) - 1 - i / group;
        it.head = kind == HSPMD_LIST_DKV ? g : g * group + i % group;
        return it;
    };
    // most expensive first inside a chain (with a shift the cost is still monotone in the tile index)
    return place_chains<hspmd_block_item>(
        num_seqs, hkv, num_queues, kind == HSPMD_LIST_DKV || group == 1,
        [&](int32_t s) {
            const int32_t n_tiles = (int32_t)ceil_div(rows_of(s), tile_rows);   // rows of the outputs the list owns
            return kind == HSPMD_LIST_DKV ? n_tiles : n_tiles * group;
        },
        [&](int32_t s, int32_t i) { return block_item_cost(kind, make(s, 0, i), group); }, make,
        hspmd_block_item{0, 0, 0, 0, 0, -1, 0, 0});
}

PassLoad block_pass_load(hspmd_list_kind kind, const int32_t* cu_q, const int32_t* cu_k, const int32_t* q_pos,
                         const int32_t* k_pos, int32_t num_seqs, int32_t hq, int32_t hkv) {
    const int tile_rows = (kind == HSPMD_LIST_DKV) ? kDkvKTile : kFwdQTile;
    PassLoad load;
    for (int32_t s = 0; s < num_seqs; ++s) {
        hspmd_block_item it{cu_q[s], cu_q[s + 1] - cu_q[s], cu_k[s], cu_k[s + 1] - cu_k[s], q_pos[s] - k_pos[s], 0, 0, q_pos[s]};
        const int32_t n_tiles = (int32_t)ceil_div(kind == HSPMD_LIST_DKV ? it.k_len : it.q_len, tile_rows);
        for (it.tile = 0; it.tile < n_tiles; ++it.tile) {
            const int64_t c = block_item_cost(kind, it, hq / hkv);
            load.total += c;
            load.heaviest = std::max(load.heaviest, c);
        }
    }
    load.total *= (kind == HSPMD_LIST_DKV) ? hkv : hq;
    return load;
}

}  // namespace hspmd
