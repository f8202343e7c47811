// Host-side construction of the cost-sorted work lists (no GPU code in here).
#pragma once
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/hspmd_attn.h"

namespace hspmd {

// Tile geometry shared by the scheduler and the kernels.
constexpr int kFwdQTile = 128;   // q rows per forward / dQ work item (4 waves x 32 rows)
constexpr int kFwdKTile = 64;    // keys per inner step of the forward / dQ kernels
constexpr int kDkvKTile = 128;   // keys per dK/dV work item (4 waves x 32 keys)
constexpr int kDkvQTile = 64;    // q rows per inner step of the dK/dV kernel
constexpr int kNumXcd = 8;       // XCDs of an MI355X: workgroup p lands on XCD p % 8

// Validates cu_seqlens / head counts; returns an empty string when fine.
std::string check_pack(const int32_t* cu, int32_t num_seqs, int32_t hq, int32_t hkv);

// Cost (number of inner steps) of one item.
int64_t item_cost(hspmd_list_kind kind, int32_t seq_len, int32_t tile, int32_t group);

// What a pass has to do, in inner steps: all items together, and the heaviest one (the pass takes at least that long); and the number
// of items, which the list's length exceeds by its padding.
struct PassLoad {
    int64_t total = 0, heaviest = 0, items = 0;
};
PassLoad pass_load(hspmd_list_kind kind, const int32_t* cu, int32_t num_seqs, int32_t hq, int32_t hkv);
PassLoad block_pass_load(hspmd_list_kind kind, const int32_t* cu_q, const int32_t* cu_k, const int32_t* q_pos,
                         const int32_t* k_pos, int32_t num_seqs, int32_t hq, int32_t hkv);

// Builds the launch-ordered list (see hspmd_attn_schedule in the public header).
std::vector<hspmd_work_item> build_work_list(hspmd_list_kind kind, const int32_t* cu, int32_t num_seqs,
                                             int32_t hq, int32_t hkv, int32_t num_queues,
                                             hspmd_order order = HSPMD_ORDER_XCD_COST);

// How a pass deals out the items of its list: a workgroup per item, half items, or persistent workgroups (dK/dV of packed
// plans; the forward is always persistent).  `slots`: length of the list, padding included.
enum class Dispatch { kWhole, kHalves, kPersistent };
Dispatch pass_dispatch(hspmd_list_kind kind, const PassLoad& load, int64_t slots, int32_t head_dim, bool block);
// How the forward or the dQ pass of a packed plan deals out its items: `halves` as pass_dispatch says, except where `teams` is 2 (two
// teams of four waves share an item's key tiles), which may also take whole items where pass_dispatch says halves.
struct RowsForm {
    bool halves;
    int teams;
};
// in_arguments: the list travels in the launch's arguments.
RowsForm rows_form(hspmd_list_kind kind, const PassLoad& load, int64_t slots, int32_t group, int32_t head_dim, bool in_arguments);
// Whether the dK/dV pass of a packed plan draws its items in persistent workgroups: also where pass_dispatch says whole items.
bool persistent_dkv(Dispatch form, const PassLoad& load, int64_t slots, int32_t group, int32_t head_dim);

// ---- dK/dV items, dealt out by query heads, or, where heads are not grouped, by query tiles
// A share of an item, as long as an ordinary item.  Its dK and dV go to area `area()` as fp32 sums that one more kernel adds up, or,
// where it is the only share, to their own place.
struct HeadPiece {
    int32_t token_start, seq_len;   // as hspmd_work_item
    uint32_t where, deal;           // tile 14 bits, kv head 7, area 11; heads of a share 8, shares of a head's tiles 7, number of the share 10
    static constexpr int64_t kMostTiles = 1 << 14, kMostKvHeads = 1 << 7, kMostAreas = 1 << 10, kMostGroup = 255, kMostParts = 127;
    constexpr bool padding() const { return deal == 0; }
    constexpr int tile() const { return (int)(where & 0x3fff); }
    constexpr int head() const { return (int)(where >> 14 & 0x7f); }
    constexpr int area() const { return (int)(where >> 21); }
    constexpr int heads() const { return (int)(deal & 0xff); }
    constexpr int parts() const { return (int)(deal >> 8 & 0x7f); }
    constexpr int index() const { return (int)(deal >> 15); }
    constexpr int shares(int group) const { return (group + heads() - 1) / heads() * parts(); }
    // the share's query heads of the group, and the query tiles that it walks of each
    constexpr int first_head() const { return index() / parts() * heads(); }
    constexpr int n_heads(int group) const { return group - first_head() < heads() ? group - first_head() : heads(); }
    constexpr int diagonal() const { return tile() * (kDkvKTile / kDkvQTile); }
    constexpr int end() const { return (seq_len + kDkvQTile - 1) / kDkvQTile; }
    constexpr int first_tile() const { return diagonal() + (end() - diagonal()) * (index() % parts()) / parts(); }
    constexpr int end_tile() const { return diagonal() + (end() - diagonal()) * (index() % parts() + 1) / parts(); }
};
static_assert(sizeof(HeadPiece) == sizeof(hspmd_work_item), "lists of either travel alike");
// The sums of a share: dK and dV of an item's keys, fp32, at the tile width that head_dim runs at; and the most that a pass may keep.
constexpr int64_t sums_area_bytes(int32_t head_dim) { return 2 * kDkvKTile * (head_dim <= 64 ? 64 : 128) * 4; }
constexpr int64_t kMostSumsBytes = 64 << 20;
static_assert(kMostSumsBytes / sums_area_bytes(64) <= HeadPiece::kMostAreas, "an area's number fits its field");
// The most areas that a pack of `tokens` tokens may ask for: by the token count alone and never less for more tokens, so that a
// workspace made for the largest pack serves every smaller one.  0: none can be dealt out.
int64_t most_areas(int64_t tokens, int32_t hq, int32_t hkv, int32_t head_dim);
struct PieceList {
    std::vector<HeadPiece> items;    // launch order, as build_work_list's
    std::vector<HeadPiece> dealt;    // the first share of every item that has several
    int64_t areas = 0;
    bool halves = false;             // the unit of work is half a piece
};
// The dK/dV list of a pack by pieces, where that pays (`load`, `slots`: of the ordinary list), with at most `most_items`
// of them; else false.
bool build_piece_list(const int32_t* cu, int32_t num_seqs, int32_t hq, int32_t hkv, int32_t num_queues, const PassLoad& load,
                      int64_t slots, int32_t head_dim, int64_t most_items, PieceList& out);

// ---- cost model: predicted kernel times (microseconds) of the three passes for a pack
// What the model knows of a pass: the form that it takes, and the inner steps and items (or shares of items) of each queue.
struct PassFeatures {
    bool halves = false;
    int teams = 1;
    int64_t areas = 0;   // of a dK/dV pass whose items are dealt out
    double heaviest = 0.0, queue_steps[kNumXcd] = {0.0}, queue_items[kNumXcd] = {0.0};
};
void pack_features(const int32_t* cu, int32_t num_seqs, int32_t hq, int32_t hkv, int32_t head_dim, PassFeatures (&out)[3]);
double estimate_pass_us(hspmd_list_kind kind, const PassFeatures& f, int32_t head_dim);

// ---- block variant (one step of context-parallel attention): per sequence a query chunk and a key chunk
// with positions inside the sequence; key j is visible to row r iff j <= r + (q_pos - k_pos).
std::string check_block_pack(const int32_t* cu_q, const int32_t* cu_k, const int32_t* q_pos, const int32_t* k_pos,
                             int32_t num_seqs, int32_t hq, int32_t hkv);

// Cost (number of inner steps) of one block item; 0 when the item only writes zeros.
int64_t block_item_cost(hspmd_list_kind kind, const hspmd_block_item& item, int32_t group);

// Launch-ordered list of the block variant: same placement rules as build_work_list.  Every tile that owns
// output rows gets an item, also when nothing is visible to it (it then writes zeros).
std::vector<hspmd_block_item> build_block_list(hspmd_list_kind kind, const int32_t* cu_q, const int32_t* cu_k,
                                               const int32_t* q_pos, const int32_t* k_pos, int32_t num_seqs,
                                               int32_t hq, int32_t hkv, int32_t num_queues);

}  // namespace hspmd
