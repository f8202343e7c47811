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
#include <cmath>
#include <limits>
#include <new>
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

// (inlined by force where a list's costs are summed, twice per item)
static inline __attribute__((always_inline)) int64_t item_steps(hspmd_list_kind kind, int32_t seq_len, int32_t tile, int32_t group) {
    if (kind == HSPMD_LIST_DKV) {
        const int64_t first_row = (int64_t)tile * kDkvKTile;          // rows r >= first key of the tile
        if (first_row >= seq_len) return 0;
        return ceil_div(seq_len - first_row, kDkvQTile) * group;
    }
    const int64_t last_key = std::min<int64_t>(seq_len, (int64_t)(tile + 1) * kFwdQTile);
    if ((int64_t)tile * kFwdQTile >= seq_len) return 0;
    return ceil_div(last_key, kFwdKTile);
}

int64_t item_cost(hspmd_list_kind kind, int32_t seq_len, int32_t tile, int32_t group) {
    return item_steps(kind, seq_len, tile, group);
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

// Workgroups that an XCD holds at once: two per compute unit in the forward and dQ passes, one in the dK/dV pass.  At tile width 64 a
// unit holds three of the dQ and two of the dK/dV pass; a list does not know its width, and the lines drawn with these numbers hold
// there too (order_last_items on ten packs of width 64: forward 0.85 to 1.01 of the time, dQ 0.87 to 1.00, dK/dV 0.82 to 1.01).
constexpr int32_t kResidentRows = 64, kResidentKeys = 32;

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

// Cuts the chains into segments no heavier than `cap`.  chain_len, cost_of: see place_chains.  (Inlined by force: called from two
// places it is not, and neither are then the costs and items of the list: a refill's lists take up to twice as long.)
template <typename ChainLen, typename Cost>
__attribute__((always_inline)) inline std::vector<SegmentClass> cut_chains(int32_t num_seqs, int32_t kv_heads, int64_t cap, ChainLen chain_len, Cost cost_of) {
    std::vector<SegmentClass> classes;
    int64_t segments = 0;
    for (int32_t s = 0; s < num_seqs; ++s) {
        const int32_t n = (int32_t)chain_len(s);
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
    return classes;
}

struct Assignment {
    std::vector<int32_t> queue_of;   // per segment, by creation index
    std::vector<int64_t> length;     // items per queue
    int64_t heaviest = 0;            // cost of the heaviest queue
};

// Longest-processing-time assignment: each segment, heaviest first, goes to the least loaded queue (the lowest index among
// equals).  The loads are a binary heap whose root is replaced, never popped and pushed.
Assignment assign_segments(const std::vector<SegmentClass>& classes, int32_t kv_heads, int32_t num_queues) {
    struct Load {
        int64_t load;
        int32_t queue;
        bool before(const Load& o) const { return load != o.load ? load < o.load : queue < o.queue; }
    };
    std::vector<Load> heap((size_t)num_queues);
    for (int32_t x = 0; x < num_queues; ++x) heap[x] = Load{0, x};   // sorted, hence a heap
    std::vector<int32_t> queue_of((size_t)classes.size() * (size_t)kv_heads);
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
    int64_t heaviest = 0;
    for (const Load& l : heap) heaviest = std::max(heaviest, l.load);
    return Assignment{std::move(queue_of), std::move(length), heaviest};
}

// The last items of a queue, once and a half as many as it has workgroups at once, go by cost and not chain by chain where the
// chains are alike (the last starts with an item at least half as heavy as the first's): a chain's heavy items would start when
// the queue runs dry.  Measured, chain by chain and by cost (us, sustained; forward, dQ, dK/dV): 5 x 2697, 8 heads, head_dim 80 77.4
// / 69.5, 100.4 / 88.0, 138.2 / 124.2; 4 x 4096, 12 heads 222 / 200, 289 / 273; 3 x 1500, 32 heads 77.6 / 68.8, 106.8 / 94.9, 142.3 /
// 139.2; 16 x 800, 8 heads 40.9 / 39.1, 58.7 / 53.2, 74.9 / 68.7; one of 5067, 24 heads, width 64 107 / 100, 126 / 118, 165 / 155.
// Not where the last chains are cheap anyway (41 log-normal sequences, 16 heads 49.5 / 52.0); nor where items are short, in the
// rows lists below 13 steps (12 x 700, 16 heads 42.4 / 45.0), in the dK/dV list below 10; nor where more than five rounds make the
// end a small part, against which K and V (Q and dO) are fetched again: dK/dV of 6 x 2048, 16 heads, six rounds 228 / 233.
template <typename Item, typename Cost>
__attribute__((noinline)) void order_last_items(const std::vector<SegmentClass>& classes, int32_t kv_heads, const Assignment& placed,
                                                int64_t resident, int64_t least_cost, Cost cost_of_item, std::vector<Item>& out) {
    const size_t queues = placed.length.size();
    std::vector<int64_t> heaviest(queues, 0), lightest(queues, std::numeric_limits<int64_t>::max());
    for (const SegmentClass& c : classes)
        for (int32_t g = 0; g < kv_heads; ++g) {
            const size_t x = (size_t)placed.queue_of[(size_t)(c.order0 + g * c.stride)];
            heaviest[x] = std::max(heaviest[x], c.first_cost);
            lightest[x] = std::min(lightest[x], c.first_cost);
        }
    std::vector<std::pair<int64_t, Item>> last;
    for (size_t x = 0; x < queues; ++x) {
        const int64_t length = placed.length[x];
        if (length <= resident || length > 5 * resident || heaviest[x] < least_cost || 2 * lightest[x] < heaviest[x]) continue;
        const int64_t window = std::min(length, resident * 3 / 2);
        Item* const first = out.data() + (size_t)(length - window) * queues + x;
        last.clear();
        for (int64_t i = 0; i < window; ++i) last.emplace_back(cost_of_item(first[(size_t)i * queues]), first[(size_t)i * queues]);
        std::stable_sort(last.begin(), last.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
        for (int64_t i = 0; i < window; ++i) first[(size_t)i * queues] = last[(size_t)i].second;
    }
}

// chain_len(s): items of one kv head's chain of sequence s, most expensive first; cost_of(s, i): of its i-th item;
// make(s, g, i): that item for kv head g; cost_of_item(item): its cost.  finer_slots: workgroups that a queue holds at once, for
// lists whose chains may be cut finer and whose end may go by cost, else 0 (rows lists of grouped heads: a finer cut would part the
// heads of one tile, and an end by cost has not been measured there).
template <typename Item, typename ChainLen, typename Cost, typename Make, typename ItemCost>
std::vector<Item> place_chains(int32_t num_seqs, int32_t kv_heads, int32_t num_queues, int32_t finer_slots, ChainLen chain_len,
                               Cost cost_of, Make make, ItemCost cost_of_item, Item pad) {
    int64_t total_cost = 0, chains = 0;
    for (int32_t s = 0; s < num_seqs; ++s) {
        const int64_t n = chain_len(s);
        if (n > std::numeric_limits<int32_t>::max()) throw std::bad_alloc();   // no list of that size can be held
        for (int32_t i = 0; i < n; ++i) total_cost += cost_of(s, i);
        if (n > 0) chains += kv_heads;
    }
    total_cost *= kv_heads;

    // segments no heavier than 1/(4 * queues) of the total
    const int64_t cap = std::max<int64_t>(1, total_cost / ((int64_t)num_queues * 4));
    std::vector<SegmentClass> classes = cut_chains(num_seqs, kv_heads, cap, chain_len, cost_of);
    if (classes.empty()) return {};
    Assignment placed = assign_segments(classes, kv_heads, num_queues);
    // Fewer than two chains per queue leave few segments, and the heaviest queue up to a tenth above the mean.  They are cut four
    // times finer where that is what the pass waits for: not when the queues are balanced (a chain's K and V then stay in one
    // L2), when the heaviest item outlasts the work per slot, or when items cost alike and come in rounds anyway.  Measured, coarse
    // and fine (us; forward, dQ, dK/dV): one document of 16001 tokens, 5 heads 339 / 326, 454 / 442, 590 / 555; 12 heads 716 /
    // 682, 987 / 926, 1349 / 1287; dK/dV of 20000 tokens, 2 KV heads of 4, width 64 1169 / 1064.  Coarse by these rules: 8 heads,
    // balanced, 476 / 483; a block of 8192 rows and keys, 8 KV heads of 4, balanced, dK/dV 900 / 944; 12 heads of 2000 tokens,
    // forward, heaviest item five times the work per slot, 30 / 33.  (That last rule costs where only dQ gains: one head
    // of 24151 tokens, forward 254 / 256, dQ 259 / 250.)
    if (finer_slots > 0 && chains < 2 * (int64_t)num_queues) {
        int64_t heaviest_item = 0, total = 0, items = 0;
        for (const SegmentClass& c : classes) {
            heaviest_item = std::max(heaviest_item, c.first_cost);
            total += c.cost * kv_heads;
            items += (int64_t)c.count * kv_heads;
        }
        const double queue = (double)total / num_queues;
        if ((double)placed.heaviest > 1.03 * queue && (double)heaviest_item < 3.0 * queue / finer_slots &&
            (double)heaviest_item > 1.1 * (double)total / (double)items) {
            const int64_t fine = std::max<int64_t>(1, total_cost / ((int64_t)num_queues * 16));
            classes = cut_chains(num_seqs, kv_heads, fine, chain_len, cost_of);
            placed = assign_segments(classes, kv_heads, num_queues);
        }
    }

    // inside a queue: segments by their most expensive item, then creation order; slot p belongs to queue
    // p % num_queues, short queues are padded at their end
    const std::vector<int32_t>& queue_of = placed.queue_of;
    const int64_t longest = *std::max_element(placed.length.begin(), placed.length.end());
    std::vector<Item> out((size_t)(longest * num_queues), pad);
    std::vector<int64_t> cursor((size_t)num_queues);
    std::iota(cursor.begin(), cursor.end(), (int64_t)0);
    walk_segments(classes, kv_heads, [](const SegmentClass& c) { return c.first_cost; }, [&](const SegmentClass& c, int32_t g) {
        int64_t& slot = cursor[(size_t)queue_of[(size_t)(c.order0 + g * c.stride)]];
        for (int32_t i = c.first; i < c.first + c.count; ++i, slot += num_queues) out[(size_t)slot] = make(c.seq, g, i);
    });
    if (finer_slots > 0 && longest > finer_slots)
        order_last_items(classes, kv_heads, placed, finer_slots, finer_slots == kResidentRows ? 13 : 10, cost_of_item, out);
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
    auto tile_of = [=](int32_t len, int32_t i) __attribute__((always_inline)) {
        return kind == HSPMD_LIST_DKV ? i : (int32_t)ceil_div(len, tile_rows) - 1 - i / group;
    };
    return place_chains<hspmd_work_item>(
        num_seqs, hkv, num_queues, kind == HSPMD_LIST_DKV ? kResidentKeys : group == 1 ? kResidentRows : 0,
        [&](int32_t s) {
            const int64_t n_tiles = ceil_div(cu[s + 1] - cu[s], tile_rows);
            return kind == HSPMD_LIST_DKV ? n_tiles : n_tiles * group;
        },
        [&](int32_t s, int32_t i) __attribute__((always_inline)) {
            const int32_t len = cu[s + 1] - cu[s];
            return item_steps(kind, len, tile_of(len, i), group);
        },
        [&](int32_t s, int32_t g, int32_t i) __attribute__((always_inline)) {
            const int32_t len = cu[s + 1] - cu[s];
            return hspmd_work_item{cu[s], len, tile_of(len, i), kind == HSPMD_LIST_DKV ? g : g * group + i % group};
        },
        [&](const hspmd_work_item& it) { return item_cost(kind, it.seq_len, it.tile, group); }, hspmd_work_item{0, 0, -1, 0});
}

PassLoad pass_load(hspmd_list_kind kind, const int32_t* cu, int32_t num_seqs, int32_t hq, int32_t hkv) {
    const int tile_rows = (kind == HSPMD_LIST_DKV) ? kDkvKTile : kFwdQTile;
    PassLoad load;
    for (int32_t s = 0; s < num_seqs; ++s) {
        const int32_t len = cu[s + 1] - cu[s], n_tiles = (int32_t)ceil_div(len, tile_rows);
        load.items += n_tiles;
        for (int32_t t = 0; t < n_tiles; ++t) {
            const int64_t c = item_cost(kind, len, t, hq / hkv);
            load.total += c;
            load.heaviest = std::max(load.heaviest, c);
        }
    }
    load.total *= (kind == HSPMD_LIST_DKV) ? hkv : hq;
    load.items *= (kind == HSPMD_LIST_DKV) ? hkv : hq;
    return load;
}

// ------------------------------------------------------------------------------ dispatch of a pass
// The rules below take every slot of the list for an item.  Padding slots (at most a queue's last few, more only on packs of few
// chains) thus count as work, which leaves packs at the edge of a rule with whole items.
namespace {

// Whether the forward and the dQ pass work on half items (64 rows, two waves of a workgroup sharing each 32-row block).  A
// step of a half item takes 0.6 to 0.85 of a whole item's (each tile is copied for half the rows), so halves pay when the
// heaviest item is what the pass waits for: when it is at least twice as long as the work per slot (two workgroups per compute
// unit), six steps of prologue and stores per half item included; and when it is long enough for what the halves cost, which
// grows with their number (above 128 items there are more of them than compute units).  Measured, forward and dQ pass, whole
// -> halves (us): heaviest item 32 steps, 4 per slot (136 items) 36.7 -> 27.8, 43.5 -> 29.3; 220 steps, 26 per slot 187 ->
// 145, 213 -> 131; 93 steps, 30 per slot 94 -> 83, 121 -> 104; but 42 steps, 28 per slot 75 -> 83, 98 -> 105; 251 steps, 156
// per slot 336 -> 376, 450 -> 445; 8 x 2048, 32 heads 304 -> 425, 450 -> 534; and 2 steps, 128 items 11.6 -> 13.2, 8 steps,
// 192 items 17.2 -> 19.7, 20.2 -> 21.3; at tile width 64 the latter 9.9 -> 12.2 and 13.4 -> 17.0.  Of 201 packs at three
// widths, measured in either form, none that this rule halves takes more than 1.02 of its time whole; the halved forwards take
// 0.89 on average, the dQ passes 0.81.
bool split_rows(hspmd_list_kind kind, const PassLoad& load, int64_t slots, int32_t head_dim) {
    const double workgroups = 512.0, heaviest = (double)load.heaviest, items = (double)slots;
    const double least = kind == HSPMD_LIST_FWD ? std::max(5.0, (head_dim <= 64 ? 6 : 5) + 0.08 * (items - 96))
                                                : items > 128 ? 8 + 0.05 * (items - 128) : 2;
    const double per_slot = ((double)load.total + 6.0 * 2.0 * (double)slots) / workgroups;
    return heaviest + 6.0 >= 2.0 * per_slot && heaviest >= least;
}

// Where an item of the forward or the dQ pass goes to two teams of four waves, one workgroup of eight per compute unit: half as many
// iterations per item, at the price of what the teams' sums cost at the end of an item and of the second workgroup that would have
// covered its loads and stores.  Half items: where each has a unit to itself, more or less, and is long (at most 240 slots: lists in the
// arguments, the only ones that these kernels take).  Whole items: where the
// heaviest is longer than the work per slot, and not so much that halves are better.  Measured, without and with (us; F forward,
// Q dQ pass; steps of the heaviest item, slots of the list with its padding; ratio = (heaviest + 6) / work per slot as in split_rows):
//   half items, one team / two: one head of 8192 tokens (128, 144) F 88.9 / 68.9, Q 82 / 73; 4 heads of 4096 (64, 168) F 52 / 44;
//   width 64, 8 heads of 2048 (32, 128) F 21.4 / 18.4, Q 18.7 / 18.4; lost where shorter or more (2 x 1024, 8 heads F 18.3 / 19.7, Q 20.4 / 22.6; 184 slots,
//   40 steps F 35.7 / 40.6; 200 slots, 100 steps Q 67.7 / 72).
//   whole items, one team / two: 5 heads of 16001 (251, 816, ratio 1.47) F 321 / 310, Q 438 / 414; width 64, 8 heads of 8192 (128, 512, 1.74)
//   F 99 / 86, Q 116 / 99, 2 of 16384 (256, 336, 3.62) F 155 / 130; against halves width 80, 318 items of 477 slots, 1.98 F 296 / 256, Q 338 /
//   307; lost at lower ratios (12 heads of 8192, 1.1 F 199 / 208, Q 267 / 280), for dQ at higher ones, where halves win (134 steps, 270
//   slots, 3.9 Q 114 / 136), and with heads in groups, which already share tiles in the L1 (24 on 6, 74 steps, 1.7 F 99 / 110).
//   Lists without padding (one sequence on 8 heads, say) end together by themselves, with halves and with whole items: there the dQ pass asks
//   for a little more (ratio 1.52 at 109 steps Q 169 / 181, 124 steps 190 / 199), and so does the forward at width 64 against halves below 80
//   steps (45 steps F 27.4 / 30.1, 56 33.8 / 36.6, 76 45.2 / 46.9; with padding 45 steps 35.6 / 31.7).  At head_dim above 112 whole items
//   against halves gain nothing below 80 steps (64 steps F 53.9 / 56.6, 77 69.1 / 71.0; 107 119 / 103).
// Over 677 packs of five widths, one to 40 heads, the passes that this takes run in 0.86 (F, width 64), 0.89 (F) and 0.93 (Q) of the time on
// average; 18 of 831 lose more than 1 %, the worst F 1.08 (24.4 / 26.4) and Q 1.02.
int teams_of_rows(hspmd_list_kind kind, bool halves, const PassLoad& load, int64_t slots, int32_t group, int32_t head_dim, bool in_arguments,
                  bool* whole) {
    const double heaviest = (double)load.heaviest, items = (double)slots;
    const double ratio = (heaviest + 6.0) / (((double)load.total + 6.0 * 2.0 * items) / 512.0);
    const bool fwd = kind == HSPMD_LIST_FWD, narrow = head_dim <= 64;
    const bool even = load.items == slots;   // no queue is shorter than the others
    *whole = !halves;
    const double least = (fwd ? narrow ? 17 : 30 : narrow ? 32 : 48) + (fwd ? 0.25 : 1.2) * std::max(0.0, items - 128);
    if (halves && in_arguments && ratio >= 4.2 && heaviest >= least) return 2;
    const double from = fwd ? (narrow ? 1.35 + 0.3 * 64 / heaviest : 1.3 + 0.5 * 64 / heaviest) + (group == 1 ? 0.0 : narrow ? 0.1 : 0.35)
                            : (narrow ? 1.35 : even ? 1.45 : 1.4) + 0.2 * 64 / heaviest;
    const double to = fwd ? narrow ? halves && even && heaviest < 80 ? 2.5 : 9.0 : 3.4 : narrow ? 2.3 : 2.0;
    const double longer = fwd ? narrow ? 44 : halves && head_dim > 112 ? 80 : 64 : 100;
    if ((fwd || group == 1) && items >= (fwd && narrow ? 150 : 250) && heaviest >= longer && ratio >= from && ratio <= to) {
        *whole = true;
        return 2;
    }
    return 1;
}

// Whether the dK/dV pass gives every item to two workgroups (each with half of its keys and half of its time).  The pass takes
// as long as its heaviest item or as the work that one workgroup slot gets, whichever is longer; a half item costs 0.68 of the
// whole one alone on its compute unit and 0.65 (2 x 0.65 = 1.3 in all) on a full chip, because both halves copy every Q / dO
// tile, and an item costs about eight steps beside its tiles.  At tile width 64, where two whole items share a unit but halves
// do not, a full chip takes 1.6 for the halves; and with more halves than units a quarter of a half item is lost at the end.
// Measured, whole and split (us): heaviest item 32 steps, 8.5 per slot (2 sequences, 8 heads) 50 and 41; 60 steps, 16 per slot
// (8 KV heads of 4) 85 and 61; 238 steps, 118 per slot (one head, width 128) 306 and 259; but 196 steps, 136 per slot 290 and
// 321; 3 steps, 168 items 17 and 23; 8 x 2048, 32 heads 652 and 826; 10 x 512, 4 heads (160 items) 22.9 and 30.1; width 64,
// one document of 16384 tokens, 2 heads 216 and 229.  Of the same packs none that this rule halves takes more than 1.01 of its
// time whole, 0.85 on average.  (Since then the halves' tile loop has become 8 % faster, 36.9 -> 33.8 us on 2 sequences, 8 heads, and the
// whole items' by 0 to 5 %; the line is the one drawn before that and errs towards whole items.)
bool split_dkv(const PassLoad& load, int64_t slots, int32_t head_dim) {
    const double heaviest = (double)load.heaviest, total = (double)load.total, items = (double)slots;
    const double units = 256.0;   // compute units; whole items of tile width 64 fit a unit twice
    const double workgroups = head_dim <= 64 ? 2 * units : units, full = head_dim <= 64 ? 1.6 : 1.3;
    const double whole = std::max(heaviest + 8, (total + 8 * items) / workgroups);
    const double tail = 2 * items > units ? 0.25 * (0.5 * full * total / items + 8) : 0.0;
    const double split = std::max(0.68 * heaviest + 8, (full * total + 8 * 2 * items) / units + tail);
    return split < 0.9 * whole;
}

// Whether the dK/dV pass draws its items in persistent workgroups (tile width 128, whole items, packed plans): at least 1024
// slots, between 3.2 and 6 steps per slot on average, 9 at head_dim up to 112, and no item that alone takes most of the pass.
// One workgroup fits a compute unit there, so the time between two of them is exposed, most of all, by the measurements, where
// chains of two, four or eight items bring heavy and light items up in step with the order in which an XCD hands its
// workgroups out.  Against that, the next item's loads wait for the last one's stores inside a workgroup, which short items
// feel.  Measured, one workgroup per item and persistent (us, head_dim 128, the same tile loop in both): 33 x 400 tokens, 16 heads
// (4 steps) 179 and 140; 78 x 512, 16 heads (5) 434 and 362; 67 x 300, 8 heads (3) 99 and 100; 43 x 64, 24 heads (1) 47 and 47; 438
// sequences, one of 3026, one head (5, the longest 48) 70.5 and 69.8; head_dim 104, 7 x 1024, 40 heads (9) 238 and 221, head_dim 96, 40 x
// 512, 16 heads 200 and 177; items of two heads: 66 x 400, 16 heads on 8 255 and 190; head_dim 104, 39 x 512, 32 on 16 327 and 274.
// The upper bounds were drawn with a tile loop that lost 2-4 % inside an item loop.  Items of one head go on to persistent_dkv; for
// items of several heads they are on the safe side (head_dim 104, 16 x 1000, 32 heads on 16, 17 steps, 356 and 333, is not taken).
bool short_items(const PassLoad& load, int64_t slots, int32_t head_dim) {
    const double per_unit = (double)(load.total + 8 * slots) / 256.0;
    return slots >= 4 * 256 && 5 * load.total > 16 * slots && load.total <= (head_dim > 112 ? 6 : 9) * slots &&
           (double)load.heaviest + 8 <= 0.8 * per_unit;
}

}  // namespace

Dispatch pass_dispatch(hspmd_list_kind kind, const PassLoad& load, int64_t slots, int32_t head_dim, bool block) {
    if (kind != HSPMD_LIST_DKV) return split_rows(kind, load, slots, head_dim) ? Dispatch::kHalves : Dispatch::kWhole;
    if (split_dkv(load, slots, head_dim)) return Dispatch::kHalves;
    return !block && head_dim > 64 && short_items(load, slots, head_dim) ? Dispatch::kPersistent : Dispatch::kWhole;
}

RowsForm rows_form(hspmd_list_kind kind, const PassLoad& load, int64_t slots, int32_t group, int32_t head_dim, bool in_arguments) {
    const bool halves = split_rows(kind, load, slots, head_dim);
    bool whole = !halves;
    const int teams = teams_of_rows(kind, halves, load, slots, group, head_dim, in_arguments, &whole);
    return RowsForm{!whole, teams};
}

// Items of one query head are drawn by persistent workgroups up to 48 steps (64 at head_dim up to 112), now that the instructions of
// the tile loop do not depend on the loop around it: at least 1536 slots (six per compute unit), more than 3.2 steps per slot, no
// item that alone takes most of the pass.  Measured, one workgroup per item and persistent (us, the same tile loop in both): 8 x 2048,
// 32 heads (17 steps) 671 and 641; 7 x 1024, 40 heads (9) 252 and 236; 10 x 1448, 16 heads (12) 250 and 237; 24 of 900 and 1025, 12 heads
// (8) 247 and 239; 8 x 4096, 16 heads, head_dim 104 (33) 1071 and 1053.  Longer items gain nothing (32768 tokens, 24 heads, 58 steps,
// 2619 and 2620), items of several heads lose (65536 tokens, 32 heads on 8, a whole step 34263 and 34880), and so do short ones (2160
// of 3 steps 142 and 144, 3136 of one tile 95 and 108).  Of 42 packs of 1120 to 2500 items of one head, five to fifty steps, three
// widths: above 1536 items 0.95 to 1.02 of the time, 0.99 on average; below, where there are five rounds of items and fewer, 0.99 to 1.02,
// 1.006 on average (5 x 1300, 24 heads 146 and 148; 8 x 1300, 16 heads, head_dim 104 151 and 156; 7 x 2440, 8 heads 185 and 189).
bool persistent_dkv(Dispatch form, const PassLoad& load, int64_t slots, int32_t group, int32_t head_dim) {
    if (form != Dispatch::kWhole || head_dim <= 64) return form == Dispatch::kPersistent;
    const double per_unit = (double)(load.total + 8 * slots) / 256.0;
    return group == 1 && slots >= 6 * 256 && 5 * load.total > 16 * slots && load.total <= (head_dim > 112 ? 48 : 64) * slots &&
           (double)load.heaviest + 8 <= 0.8 * per_unit;
}

// ------------------------------------------------------------------------------ pieces of dK/dV items
// An item walks the query tiles of every head of its group, so on packs of few KV heads the first key tiles of a long sequence
// outlast everything else.  Items above a limit are dealt out by query heads (the walk's outer loop) or, where heads are not
// grouped, by query tiles: every share leaves its sums of dK and dV as fp32 in memory, and a kernel behind the pass adds them up in the order of
// heads and tiles.  That costs a launch and
// the way of the sums through memory, about seven steps and 0.025 per share, and the shares' own prologues and stores.
// Measured, the dK/dV pass without and with, sums included (us): 8 query heads on 2 KV heads, 3000 and 500 tokens 146 / 70, 2048 tokens 100 /
// 42, 512 tokens 36 / 21, 16384 tokens 1171 / 996; 8 on 1, 4096 tokens 354 / 102; 16 on 4, 8192 tokens 599 / 513; 28 on 7, 1947 tokens 104 / 95; width
// 64, 8 on 2, 8192 tokens 273 / 159; by tiles: one head of 8192 tokens 100 / 56, width 64, 2 heads of 16384 208 / 157.  Of 62 packs of 256 to 32000
// tokens, 1 to 8 KV heads and groups of 2 to 8, the 38 that this takes run in 0.74 of the time on average, 0.99 at worst; of 61 packs of 1000 to
// 50000 tokens and 1 to 8 heads, most of one query head each, 18 in 0.75, 0.96 at worst.  The line is at 0.9 of the steps because idle time comes
// back as clock: at 0.95 it also takes 32 heads on 8, 9 sequences of 103 .. 3079 321 / 322, and 10 on 5, head_dim 104, 8 of up to 12995 877 / 893.
// Closer still, at 0.77, where the shares are whole items in one to two rounds and the items were halves: the estimate takes two workgroups
// that follow each other on a unit for the sum of their steps, and without its halves a long share starts last.  One sequence of 3596 tokens,
// 16 heads on 8 111 / 124; 5438 tokens, 10 on 5, head_dim 80 82 / 89; 2332, 27 on 9 99 / 108; 3000, 16 on 8 87 / 90.  At 0.72 for groups of more than
// five heads, whose shares of two heads and more come out uneven (8622 to 9779 tokens among 17 sequences, 21 on 3, 1.02 to 1.09 of the time
// on whole items).  Where the items were whole too, in more than three and a half rounds, at 0.87 (24268 tokens, 24 on 3, head_dim 104 1597 /
// 1821; 36016, 20 on 4, 80 424 / 442), and for those groups at head_dim above 112, in more than three, at 0.8 (13584 tokens, 40 on 5 1324 /
// 1433; 25631, 21 on 3 2307 / 2405; but 23554, 9 on 3 549 / 475).  Of 900 packs of 256 to
// 40000 tokens, 1 to 16 KV heads and groups of 1 to 8 that the line at 0.9 takes 35 lost more than 1 %, with these 3 (35.1 / 36.4 the worst); the 107 that
// they leave with their items would have taken 0.97 of the time on average.  Of 2568 that these lines take 10 lose more than 1 %; 0.68 on average.
// Not against half items of single heads that are more than the units hold at once (5000, 3000 and 300 tokens, 3 heads 72 / 80; 16001 tokens, 2
// heads 274 / 282).  Limits finer than a quarter of the mean only add sums; a limit of the mean leaves queues of 41 heavy shares on 32 units (8192
// tokens, 16 on 4 617).
namespace {

// What the dK/dV pass takes, in steps, and whether on half items (split_dkv): its longest item, or its work and what the last items
// leave idle at the end.
double dkv_steps(double heaviest, double total, double items, int32_t head_dim, bool* halves) {
    const PassLoad load{(int64_t)total, (int64_t)heaviest, (int64_t)items};
    *halves = split_dkv(load, (int64_t)items, head_dim);
    const double units = 256.0;
    if (*halves) {
        const double full = head_dim <= 64 ? 1.6 : 1.3;
        return std::max(0.68 * heaviest + 8, (full * total + 16 * items) / units + 0.25 * heaviest);
    }
    return std::max(heaviest + 8, (total + 8 * items) / (head_dim <= 64 ? 2 * units : units) + 0.35 * heaviest);
}

constexpr int64_t kLeastDealt = 9;   // steps: shorter items are not worth what the sums cost

// How an item of `per_head` steps a head is dealt out where a share may hold `limit` steps.
struct Deal {
    int32_t heads, parts;   // heads of a share; shares of a head's tiles
    Deal(int64_t per_head, int64_t limit, int32_t group)
        : heads((int32_t)std::min<int64_t>(group, std::max<int64_t>(1, limit / std::max<int64_t>(1, per_head)))),
          parts(group == 1 && per_head > limit ? (int32_t)ceil_div(per_head, limit) : 1) {}
    int64_t shares(int32_t group) const { return ceil_div(group, heads) * parts; }
    int64_t heaviest(int64_t per_head) const { return heads * ceil_div(per_head, parts); }
};

}  // namespace

// One sequence of n query tiles with a query head per KV head, in shares of six steps, has n (n + 12) / 24 of them a head, one with groups at
// most n / 2 a query head; of 377 packs of 192 to 65536 tokens that are dealt out without this bound, none has more.  Single heads: of
// 7500 packs on 16 to 40 of them none would be dealt out (their items come in too many rounds), so those plans keep no room.
int64_t most_areas(int64_t tokens, int32_t hq, int32_t hkv, int32_t head_dim) {
    const int64_t n = ceil_div(tokens, kDkvQTile), group = hq / hkv, most = kMostSumsBytes / sums_area_bytes(head_dim);
    if (n * group < kLeastDealt || (group == 1 && hkv > 15) || hkv > HeadPiece::kMostKvHeads || group > HeadPiece::kMostGroup) return 0;
    return n > 24 * most ? most : std::min(most, ceil_div(hq * n * (n + 12), 24));
}

bool build_piece_list(const int32_t* cu, int32_t num_seqs, int32_t hq, int32_t hkv, int32_t num_queues, const PassLoad& load,
                      int64_t slots, int32_t head_dim, int64_t most_items, PieceList& out) {
    const int32_t group = hq / hkv;
    const int64_t room = most_areas(cu[num_seqs], hq, hkv, head_dim);
    if (load.heaviest < kLeastDealt || room == 0) return false;
    const double units = head_dim <= 64 ? 512.0 : 256.0, items = (double)slots;
    bool halves = false;
    const double now = dkv_steps((double)load.heaviest, (double)load.total, items, head_dim, &halves);
    const double mean = ((double)load.total + 8 * items) / units;
    const bool whole_now = !halves;
    double rounds = 0.0;   // of the shares, on the chip's workgroups
    int64_t best = 0;
    if (group == 1 && halves && slots > 240) return false;
    double least = 0.9 * now;
    if (std::max(mean, 8.0) + 7 >= least) return false;   // what is left with every share as short as can be
    const bool short_list = most_items < slots + HeadPiece::kMostAreas;   // (coarser limits, so that some list fits)
    for (const double share : {2.0, 1.4, 1.0, 0.7, 0.5, 0.25}) {
        if (share > 1.0 && !short_list) continue;
        const int64_t limit = std::max<int64_t>(6, (int64_t)(share * mean));   // (a share of a head's tiles then has three and more)
        if (load.heaviest <= limit) continue;
        int64_t heaviest = 0, more = 0, areas = 0, parts = 1;
        for (int32_t s = 0; s < num_seqs; ++s) {
            const int32_t len = cu[s + 1] - cu[s], n_tiles = (int32_t)ceil_div(len, kDkvKTile);
            if (n_tiles > HeadPiece::kMostTiles) return false;
            for (int32_t t = 0; t < n_tiles; ++t) {
                const int64_t per_head = item_steps(HSPMD_LIST_DKV, len, t, 1);
                if (per_head * group <= limit) {   // neither this nor any later item is dealt out
                    heaviest = std::max(heaviest, per_head * group);
                    break;
                }
                const Deal deal(per_head, limit, group);
                const int64_t pieces = deal.shares(group);
                heaviest = std::max(heaviest, deal.heaviest(per_head));
                parts = std::max<int64_t>(parts, deal.parts);
                more += (pieces - 1) * hkv;
                if (pieces > 1) areas += pieces * hkv;
            }
        }
        if (areas > room || parts > HeadPiece::kMostParts || slots + more + (short_list ? 16 : 0) > most_items) continue;   // (16: padding of short queues)
        bool h = false;
        const double then = dkv_steps((double)heaviest, (double)load.total, items + (double)more, head_dim, &h) + 7 + 0.025 * (double)areas;
        if (then < least) {
            least = then;
            best = limit;
            halves = h;
            rounds = (items + (double)more) / units;
        }
    }
    if (best == 0) return false;
    if (!halves) {   // (see above)
        const double closer = group > 5 ? 0.72 : 0.77;
        const double line = !whole_now ? (rounds > 1.15 && rounds < 2.3 ? closer : 0.9)
                                       : group > 5 && head_dim > 112 && rounds > 3.0 ? 0.8 : rounds > 3.5 ? 0.87 : 0.9;
        if (least >= line * now) return false;
    }

    struct Share {
        int64_t cost;
        int32_t tile, area0, pieces;   // area0: kv head 0's first area
        uint32_t deal;                 // as HeadPiece's
    };
    std::vector<std::vector<Share>> shares((size_t)num_seqs);
    out = PieceList();
    for (int32_t s = 0; s < num_seqs; ++s) {
        const int32_t len = cu[s + 1] - cu[s], n_tiles = (int32_t)ceil_div(len, kDkvKTile);
        for (int32_t t = 0; t < n_tiles; ++t) {
            const Deal deal(item_steps(HSPMD_LIST_DKV, len, t, 1), best, group);
            const int32_t pieces = (int32_t)deal.shares(group);
            for (int32_t index = 0; index < pieces; ++index) {
                const HeadPiece x{0, len, (uint32_t)t, (uint32_t)deal.heads | (uint32_t)deal.parts << 8 | (uint32_t)index << 15};
                shares[s].push_back(Share{(int64_t)x.n_heads(group) * (x.end_tile() - x.first_tile()), t, (int32_t)out.areas, pieces, x.deal});
            }
            if (pieces > 1) out.areas += (int64_t)pieces * hkv;
        }
        std::stable_sort(shares[s].begin(), shares[s].end(), [](const Share& a, const Share& b) { return a.cost > b.cost; });
    }
    out.halves = halves;
    out.items = place_chains<HeadPiece>(
        num_seqs, hkv, num_queues, kResidentKeys, [&](int32_t s) { return (int64_t)shares[s].size(); },
        [&](int32_t s, int32_t i) { return shares[s][i].cost; },
        [&](int32_t s, int32_t g, int32_t i) {
            const Share& x = shares[s][i];
            const int32_t area = x.pieces > 1 ? x.area0 + g * x.pieces + (int32_t)(x.deal >> 15) : 0;
            return HeadPiece{cu[s], cu[s + 1] - cu[s], (uint32_t)x.tile | (uint32_t)g << 14 | (uint32_t)area << 21, x.deal};
        },
        [&](const HeadPiece& it) { return (int64_t)it.n_heads(group) * (it.end_tile() - it.first_tile()); }, HeadPiece{0, 0, 0, 0});
    if ((int64_t)out.items.size() > most_items) return false;   // (short queues are padded)
    for (const HeadPiece& it : out.items)
        if (!it.padding() && it.index() == 0 && it.shares(group) > 1) out.dealt.push_back(it);
    return true;
}

// ------------------------------------------------------------------------------ cost model
// The paper's planner dispatches mixed-length sequences with a cost model evaluated on the CPU (Appendix
// "Scenario-specific Planning", mixed-length case); this is the per-operator predictor for the attention kernels of this library.
// A pass takes a launch time and, of two times, a little more than the longer (the fourth root of the sum of their fourth
// powers: where they are close, part of the chip idles at the end): the weight of the heaviest XCD queue -- steps x step time
// + a fixed time per item -- shared by the workgroups that an XCD holds, and the heaviest item on a chip that is otherwise
// idle.  Half items take the stated shares of a whole one's times.  Fitted by relative least squares to 124 packs at each of
// five widths, before the dK/dV loop was written step by step and short lists went into the arguments; with these kernels the mean
// |error| on such packs is 6-8 % per pass, 95 % of them are within 20 %, the others (passes of a few steps per item or with a single
// item per workgroup) within 43 %; 7 % of the forward and 5 % of the backward together with the present forms.  A new fit would take off up to
// a percent of the mean.
namespace {

struct PassCost { double step_us, item_us, alone_us; };               // alone_us: a step with one workgroup per unit or fewer
struct PassFixed { double launch_us, half_step, half_alone, half_item; };   // half_*: shares of a whole item's times
struct Shares { double step, alone, item; };
// the same shares where two teams of waves take an item: whole items, half items (fitted to 205 and 143 forwards, 48 and 71 dQ passes;
// mean |error| 3 to 5 %)
constexpr Shares kTeamShares[2][2] = {{{1.19, 0.65, 1.30}, {0.80, 0.51, 0.98}}, {{1.18, 0.69, 1.01}, {0.68, 0.49, 0.85}}};
constexpr PassFixed kPassFixed[3] = {{1.6, 0.64, 0.75, 0.83}, {0.0, 0.62, 0.61, 0.67}, {0.0, 0.52, 0.70, 0.84}};
// head_dim up to 64, 80, 96, 112, 128: each has kernels of its own
constexpr PassCost kPassCost[3][5] = {
    {{1.092, 6.86, 0.692}, {1.359, 7.88, 0.845}, {1.447, 8.07, 0.835}, {1.686, 9.25, 0.849}, {1.712, 9.12, 0.858}},
    {{1.919, 11.16, 0.593}, {1.701, 12.25, 0.786}, {1.859, 12.98, 0.827}, {2.206, 13.94, 0.876}, {2.331, 14.86, 0.896}},
    {{1.724, 10.78, 0.835}, {1.357, 11.48, 0.938}, {1.405, 11.83, 1.075}, {1.659, 13.52, 1.059}, {1.666, 13.82, 1.163}}
};

}  // namespace

void pack_features(const int32_t* cu, int32_t num_seqs, int32_t hq, int32_t hkv, int32_t head_dim, PassFeatures (&out)[3]) {
    const int32_t group = hq / hkv;
    // one list serves the forward and the dQ pass, as in a plan
    const std::vector<hspmd_work_item> rows = build_work_list(HSPMD_LIST_FWD, cu, num_seqs, hq, hkv, kNumXcd);
    const std::vector<hspmd_work_item> keys = build_work_list(HSPMD_LIST_DKV, cu, num_seqs, hq, hkv, kNumXcd);
    const bool in_arguments = std::max(rows.size(), keys.size()) <= 240;
    auto walk = [](const auto& list, auto real, auto cost_of, PassFeatures& f) {
        f.heaviest = 0.0;
        for (size_t p = 0; p < list.size(); ++p) {
            if (!real(list[p])) continue;
            const double cost = (double)cost_of(list[p]);
            f.heaviest = std::max(f.heaviest, cost);
            f.queue_steps[p % kNumXcd] += cost;
            f.queue_items[p % kNumXcd] += 1.0;
        }
    };
    auto real = [](const hspmd_work_item& it) { return it.tile >= 0; };
    PassFeatures& fwd = out[HSPMD_LIST_FWD] = PassFeatures();
    PassFeatures& dkv = out[HSPMD_LIST_DKV] = PassFeatures();
    walk(rows, real, [&](const hspmd_work_item& it) { return item_cost(HSPMD_LIST_FWD, it.seq_len, it.tile, group); }, fwd);
    out[HSPMD_LIST_DQ] = fwd;
    const PassLoad row_load = pass_load(HSPMD_LIST_FWD, cu, num_seqs, hq, hkv), key_load = pass_load(HSPMD_LIST_DKV, cu, num_seqs, hq, hkv);
    for (const hspmd_list_kind kind : {HSPMD_LIST_FWD, HSPMD_LIST_DQ}) {
        const RowsForm form = rows_form(kind, row_load, (int64_t)rows.size(), group, head_dim, in_arguments);
        out[kind].halves = form.halves;
        out[kind].teams = form.teams;
    }
    PieceList pieces;
    if (!keys.empty() && build_piece_list(cu, num_seqs, hq, hkv, kNumXcd, key_load, (int64_t)keys.size(), head_dim,
                                          in_arguments ? 240 : std::numeric_limits<int32_t>::max(), pieces)) {
        dkv.halves = pieces.halves;
        dkv.areas = pieces.areas;
        walk(pieces.items, [](const HeadPiece& it) { return !it.padding(); },
             [&](const HeadPiece& it) { return (int64_t)it.n_heads(group) * (it.end_tile() - it.first_tile()); }, dkv);
    } else {
        dkv.halves = pass_dispatch(HSPMD_LIST_DKV, key_load, (int64_t)keys.size(), head_dim, false) == Dispatch::kHalves;
        walk(keys, real, [&](const hspmd_work_item& it) { return item_cost(HSPMD_LIST_DKV, it.seq_len, it.tile, group); }, dkv);
    }
}

double estimate_pass_us(hspmd_list_kind kind, const PassFeatures& f, int32_t head_dim) {
    if (f.heaviest == 0.0) return 0.0;   // an empty pack
    const bool narrow = head_dim <= 64;
    const PassCost c = kPassCost[(int)kind][narrow ? 0 : std::max(1, (head_dim + 15) / 16 - 4)];
    const PassFixed fixed = kPassFixed[(int)kind];
    const Shares share = f.teams == 2 ? kTeamShares[(int)kind][f.halves] : f.halves ? Shares{fixed.half_step, fixed.half_alone, fixed.half_item}
                                                                                   : Shares{1.0, 1.0, 1.0};
    const double step = c.step_us * share.step * (f.halves ? 2 : 1), item = c.item_us * share.item * (f.halves ? 2 : 1);
    // workgroups resident per XCD: 32 compute units, two workgroups each in the forward and dQ passes, one in dK/dV; at tile
    // width 64 three in the dQ pass and two in dK/dV with whole items
    const double per_unit = kind == HSPMD_LIST_DKV ? (narrow && !f.halves ? 2 : 1) : (narrow && kind == HSPMD_LIST_DQ ? 3 : 2);
    double shared = 0.0;
    for (int x = 0; x < kNumXcd; ++x) shared = std::max(shared, f.queue_steps[x] * step + f.queue_items[x] * item);
    shared /= 32.0 * per_unit;
    const double alone = f.heaviest * c.alone_us * share.alone + c.item_us * share.item;
    // (items that are dealt out: what adding up their sums takes)
    return fixed.launch_us + (f.areas > 0 ? 5.0 + 0.03 * (double)f.areas : 0.0) +
           std::sqrt(std::sqrt(shared * shared * shared * shared + alone * alone * alone * alone));
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
        num_seqs, hkv, num_queues, kind == HSPMD_LIST_DKV ? kResidentKeys : group == 1 ? kResidentRows : 0,
        [&](int32_t s) {
            const int64_t n_tiles = ceil_div(rows_of(s), tile_rows);   // rows of the outputs the list owns
            return kind == HSPMD_LIST_DKV ? n_tiles : n_tiles * group;
        },
        [&](int32_t s, int32_t i) __attribute__((always_inline)) { return block_item_cost(kind, make(s, 0, i), group); }, make,
        [&](const hspmd_block_item& it) { return block_item_cost(kind, it, group); },
        hspmd_block_item{0, 0, 0, 0, 0, -1, 0, 0});
}

PassLoad block_pass_load(hspmd_list_kind kind, const int32_t* cu_q, const int32_t* cu_k, const int32_t* q_pos,
                         const int32_t* k_pos, int32_t num_seqs, int32_t hq, int32_t hkv) {
    const int tile_rows = (kind == HSPMD_LIST_DKV) ? kDkvKTile : kFwdQTile;
    PassLoad load;
    for (int32_t s = 0; s < num_seqs; ++s) {
        hspmd_block_item it{cu_q[s], cu_q[s + 1] - cu_q[s], cu_k[s], cu_k[s + 1] - cu_k[s], q_pos[s] - k_pos[s], 0, 0, q_pos[s]};
        const int32_t n_tiles = (int32_t)ceil_div(kind == HSPMD_LIST_DKV ? it.k_len : it.q_len, tile_rows);
        load.items += n_tiles;
        for (it.tile = 0; it.tile < n_tiles; ++it.tile) {
            const int64_t c = block_item_cost(kind, it, hq / hkv);
            load.total += c;
            load.heaviest = std::max(load.heaviest, c);
        }
    }
    load.total *= (kind == HSPMD_LIST_DKV) ? hkv : hq;
    load.items *= (kind == HSPMD_LIST_DKV) ? hkv : hq;
    return load;
}

}  // namespace hspmd
