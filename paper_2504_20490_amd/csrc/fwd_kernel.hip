// Forward kernel: one workgroup per (sequence, 128-row q tile, q head) work item.
//
// Each of the 4 waves owns 32 query rows.  For every 64-key tile of the causal prefix the
// workgroup stages K and V in LDS (coalesced 16-byte global->LDS copies, double buffered, one
// barrier per tile); each wave computes S^T = K Q^T on MFMA (keys along rows, its queries along
// columns), runs the online-softmax recurrence with one lane per query, and feeds the bf16
// P^T fragments straight back into MFMA as the B operand of O^T += V^T P^T, V^T being read
// from the row-major V tile with the LDS transpose read.
//
// The loop is software-pipelined by one tile: the MFMAs of S^T(kt+1) run under the exp work of tile kt's
// first key block, the first MFMAs of tile kt's P V under that of its second key block.  K therefore
// runs one tile ahead of V in LDS.  Both phases are written MFMA step by MFMA step (operand reads a few
// steps ahead, a scheduling barrier after each step).  Tiles that lie wholly below the diagonal take
// code without any mask; only the tiles on the diagonal compare key and row indices.  With BLOCK the
// query rows and the keys are separate chunks and the diagonal is shifted (one step of context-parallel
// attention): partial O in fp32, LSE = -inf for rows that see no key.
#include "attn_device.hpp"
#include "fwd_tiles.hpp"
#include "kernels.hpp"
#include "schedule.hpp"

namespace hspmd {

namespace {

// KD: 16-column steps of head_dim that hold data (D / 16, or fewer when head_dim ends before the tile width: the steps
// beyond it would multiply the zero padding of the query fragments); the product whose output is head_dim wide takes
// (KD + 1) / 2 blocks of 32 columns.  8 x 2048, 32 heads, head_dim 96: 6 steps and 3 blocks instead of 7 and 4, 282 -> 256 us.
template <int D, int KD>
struct FwdGeom {
    static_assert(KD >= 1 && KD <= D / 16, "k-steps inside the tile width");
    static constexpr int KK = KD;       // k-steps of S^T = K Q^T
    static constexpr int DB = (KD + 1) / 2;   // 32-row blocks of O^T that hold data
    static constexpr int kTileBytes = kFwdKTile * D * 2;
};

// NB: 32-key blocks of every tile that the wave takes: both, or one when two waves share the tile (SPLIT)
template <int D, int KD, int NB>
struct FwdState {
    using G = FwdGeom<D, KD>;
    bf16x8 qf[G::KK];      // this lane's query row (B operand of S^T = K Q^T)
    f32x16 acc[G::DB];     // O^T accumulator
    f32x16 s[NB];          // S^T of the current tile, one fragment per 32-key block
    float m, l;            // running row max of the raw scores; this lane's share of the running row sum
    float tnext;           // this lane's maximum over s[] as it stands (all keys taken as visible)
    int rm[G::KK];         // per-lane LDS offsets of the K fragments (row-major read), block 0 of a tile
    int tr[G::DB][2];      // per-lane LDS offsets of the V^T fragments (transpose read), k-step 0 of a tile
};

// this wave's single copy instructions of one whole K tile and one whole V tile
template <int D>
struct FwdTileLoad {
    using Copy = TileCopy<D, kFwdKTile>;
    const Copy* copy;
    const uint16_t* k_row;   // first row of the K tile, this kv head, column 0
    const uint16_t* v_row;
    uint32_t k_dst;          // LDS byte addresses
    uint32_t v_dst;
    int wave;
    __device__ __forceinline__ void k_piece(int i) const {
#pragma unroll
        for (int n = 0; n < Copy::kPerWave; ++n)
            if (n == i) copy->issue_full_one_at(n, k_dst, k_row, wave);
    }
    __device__ __forceinline__ void v_piece(int i) const {
#pragma unroll
        for (int n = 0; n < Copy::kPerWave; ++n)
            if (n == i) copy->issue_full_one_at(n, v_dst, v_row, wave);
    }
};

// this lane's maximum over its 16 NB scores of a tile (v_max3: two scores per instruction)
template <int NB>
__device__ __forceinline__ float lane_max(const f32x16 (&s)[NB]) {
    float t = fmaxf(s[0][0], s[0][1]);
#pragma unroll
    for (int e = 2; e < 16 * NB; ++e) t = fmaxf(t, s[e >> 4][e & 15]);   // a chain: pairs of steps become one v_max3
    return t;
}

__device__ __forceinline__ float pair_max(float x) {
    // v_permlane32_swap: first result = the value held by lane l % 32, second = the value of lane l % 32 + 32
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// One iteration on key tile kt, whose scores are already in st.s:
//   first  : VALU only: running max of tile kt; accumulator rescale if some lane's max moved
//   phase A: MFMA S^T(kt+1) = K(kt+1) Q^T   |  VALU: exp2, row sum, bf16 pack of tile kt's first key block
//   phase B: MFMA O^T += V(kt)^T P^T(kt)     |  VALU: the same for its second key block, under the first MFMAs
// kbuf: K tile kt+1; vbuf: V tile kt.  MASK: tile kt touches the diagonal (keys beyond a lane's own row get
// weight 0); LAST: there is no tile kt+1.
// SPREAD: the iteration also issues this wave's share of the copies of K(kt+2) and V(kt+1), both whole
// tiles, one instruction per MFMA step of phase A.  Issued back to back after the barrier, the copies of
// all waves queue up in front of the CU's one address unit.
// SOME (block variant, half items, teams): a lane's row may have no visible key so far, or, with a share of the keys, none with a finite score (its
// running max is still -inf): the maximum that the exponentials are taken against is then replaced by 0, which keeps every
// weight and the rescale factor at 0.
// NB = 1: the wave's only 32-key block of the tile is part of the addresses; its eight score pairs all go under the
// MFMAs of phase A, the copies too (two per step where the phase has fewer steps than copies).
template <int D, int KD, int NB, bool MASK, bool LAST, bool SPREAD, bool SOME>
__device__ __forceinline__ void fwd_iteration(FwdState<D, KD, NB>& st, const char* kbuf, const char* vbuf, float c,
                                              int dkey /* my_row - key0 - 4 * (lane / 32) */,
                                              const FwdTileLoad<D>& load) {
    using G = FwdGeom<D, KD>;
    constexpr int KK = G::KK, DB = G::DB;
    constexpr int NP = FwdTileLoad<D>::Copy::kPerWave;   // copy instructions per wave and tile

    // ---------------- running max of tile kt and the (rare) accumulator rescale: a short VALU-only stretch
    if constexpr (MASK) {
        // element i of block jb is key 32 jb + 8 (i / 4) + i % 4 (+ 4 (lane / 32), folded into dkey)
#pragma unroll
        for (int jb = 0; jb < NB; ++jb)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (32 * jb + 8 * (i >> 2) + (i & 3) > dkey) st.s[jb][i] = -INFINITY;
    }
    // An unmasked tile's maximum was taken while the scores were still warm: under the last MFMAs of the iteration
    // that produced them, which have no other VALU work to run beside them (st.tnext).
    float tmax = st.tnext;
    if constexpr (MASK) tmax = lane_max(st.s);
    tmax = pair_max(tmax);
    // st.m is the reference that the exponentials are taken against, not the exact running maximum: it moves only
    // when the maximum has risen by more than kMaxSlack in the exponent (base-2) domain.  Weights then lie in
    // (0, 2^kMaxSlack] instead of (0, 1] -- the same relative precision in bf16 and fp32, and O and LSE do not depend on
    // the reference -- while the accumulator rescale, which a moving maximum of ANY of the wave's 32 rows triggers,
    // becomes rare after the first tiles.  (-inf - -inf = NaN compares false: a row without a visible key keeps -inf.)
    constexpr float kMaxSlack = 8.f;
    const float m_new = (tmax - st.m) * c > kMaxSlack ? tmax : st.m;
    const float m_ref = (SOME && m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = fast_exp2((st.m - m_ref) * c);
    const float mc = m_ref * c;
    if (__any(m_new > st.m)) {      // wave-uniform: skip the accumulator rescale when no lane's max moved
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) st.acc[db][i] *= alpha;
    }
    st.m = m_new;
    __builtin_amdgcn_sched_barrier(0);

    // The two waves of a SIMD (one of each resident workgroup) compete for its issue slots: the one that is in its
    // MFMA phases goes first, so that the matrix pipe does not wait behind the other's VALU-only stretch.
    __builtin_amdgcn_s_setprio(1);
    // ---------------- phase A: S^T(kt+1) on the MFMA, exp2 / row sum / bf16 pack of tile kt on the VALU.
    // Written out step by step with a scheduling barrier after each: step n issues the K fragment read of
    // MFMA n + kAheadK, MFMA n, and the softmax work on two scores.
    f32x16 sn[NB];
    float psum = 0.f;
    union { u32x4 u; bf16x8 v; } pw[2 * NB];
    auto softmax_pair = [&](int n) {   // scores 2n, 2n+1 of the tile's 32 per lane -> one packed bf16 pair
        const int jb = n >> 3, i = (n & 7) * 2;
        const float e0 = fast_exp2(fmaf(st.s[jb][i], c, -mc));
        const float e1 = fast_exp2(fmaf(st.s[jb][i + 1], c, -mc));
        psum += e0 + e1;
        // the sum is needed only at the end of the iteration, and left alone the compiler keeps all 32 weights in
        // registers and adds them up there, in one stretch of 32 VALU instructions with no MFMA to run under;
        // an (empty) statement that reads and writes the sum keeps each pair's two additions in this step
        asm volatile("" : "+v"(psum));
        pw[jb * 2 + (i >> 3)].u[(i >> 1) & 3] = pack_bf16(e0, e1);
    };
    if constexpr (!LAST) {
        constexpr int kAheadK = 4;
        constexpr int NM = NB * KK;              // MFMAs of the phase
        static_assert(NB == 1 || 2 * NP <= NM, "one copy instruction per MFMA step");
        // the tile's key blocks in turn: consecutive MFMAs take the same query fragment, and none continues its predecessor's chain
        // (one block after the other / in turn, interleaved: 8 x 2048, 32 heads, width 64 200.2 / 198.2 us; 6001 tokens, 32 heads on 8 96.5 /
        // 96.0; 8 x 2048, 32 heads 303.6 / 302.9; 8 x 4096, head_dim 104 522 / 521; short sequences of width 64 46.9 / 47.1)
        auto k_frag = [&](int n) {
            return *reinterpret_cast<const bf16x8*>(kbuf + st.rm[n / NB] + (n % NB) * 32 * D * 2);
        };
        bf16x8 kq[kAheadK + 1];
#pragma unroll
        for (int n = 0; n < kAheadK; ++n) kq[n] = k_frag(n);
#pragma unroll
        for (int jb = 0; jb < NB; ++jb)
#pragma unroll
            for (int i = 0; i < 16; ++i) sn[jb][i] = 0.f;
#pragma unroll
        for (int n = 0; n < NM; ++n) {
            if (n + kAheadK < NM) kq[(n + kAheadK) % (kAheadK + 1)] = k_frag(n + kAheadK);
            sn[n % NB] = mfma(kq[n % (kAheadK + 1)], st.qf[n / NB], sn[n % NB]);
            // the first 8 of the 16 score pairs (key block 0, P fragments 0 and 1) spread over the NM MFMAs; the
            // other 8 go under the first P V MFMAs of phase B, which only need fragments 0 and 1
            if constexpr (NB == 1) {
#pragma unroll
                for (int x = n * 8 / NM; x < (n + 1) * 8 / NM; ++x) softmax_pair(x);
            } else if constexpr (NM > 8) {
                // pairs 0 .. NM/2 - 1 at the even steps; with fewer than 16 steps the remaining ones at the last odd steps
                if (n % 2 == 0) softmax_pair(n / 2);
                else if (7 - (NM - 1 - n) / 2 >= NM / 2) softmax_pair(7 - (NM - 1 - n) / 2);
            } else {
                static_assert(NM == 8, "eight score pairs over the steps of the phase");
                softmax_pair(n);
            }
            if constexpr (SPREAD && NB == 1) {
#pragma unroll
                for (int x = n * 2 * NP / NM; x < (n + 1) * 2 * NP / NM; ++x) {
                    if (x < NP) load.k_piece(x);
                    else load.v_piece(x - NP);
                }
            } else if constexpr (SPREAD) {
                // all copies early in the iteration: both tiles are needed right after the next barrier
                if (n < NP) load.k_piece(n);
                else if (n < 2 * NP) load.v_piece(n - NP);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int n = 0; n < 8; ++n) softmax_pair(n);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---------------- phase B: O^T += V(kt)^T P^T(kt), transpose reads kAheadV MFMAs ahead
    {
        constexpr int kAheadV = 3;
        constexpr int NM = 2 * NB * DB;
        auto v_frag = [&](int n) {
            const int t = n / DB, db = n % DB;
            const int off = t * 16 * D * 2;
            union { struct { s16x4 a, b; } s; bf16x8 v; } u;
            u.s.a = lds_transpose_read(vbuf + st.tr[db][0] + off);
            u.s.b = lds_transpose_read(vbuf + st.tr[db][1] + off);
            return u.v;
        };
        bf16x8 vq[kAheadV + 1];
#pragma unroll
        for (int n = 0; n < kAheadV; ++n) vq[n] = v_frag(n);
        // the next tile's maximum, a share of its 32 scores per step (the scores are complete since phase A)
        float tnext = -INFINITY;
        auto max_share = [&](int e0, int count) {
#pragma unroll
            for (int e = e0; e < e0 + count; ++e) tnext = fmaxf(tnext, sn[e >> 4][e & 15]);   // a chain: v_max3 per pair
            // (an empty statement on the running value keeps the share in its step: nothing else needs the value
            // before the end of the iteration, and the compiler would collect all 32 there)
            asm volatile("" : "+v"(tnext));
        };
#pragma unroll
        for (int n = 0; n < NM; ++n) {
            if (n + kAheadV < NM) vq[(n + kAheadV) % (kAheadV + 1)] = v_frag(n + kAheadV);
            st.acc[n % DB] = mfma(vq[n % (kAheadV + 1)], pw[n / DB].v, st.acc[n % DB]);
            // score pairs 8 .. 15 (key block 1, P fragments 2 and 3) under the MFMAs of fragments 0 and 1
            if constexpr (NB == 1) {
                if (!LAST) max_share(n * 16 / NM, (n + 1) * 16 / NM - n * 16 / NM);
            } else if (n < NM / 2) {
#pragma unroll
                for (int x = n * 16 / NM; x < (n + 1) * 16 / NM; ++x) softmax_pair(8 + x);
            } else if (!LAST) {
                const int h = n - NM / 2;
                max_share(h * 64 / NM, (h + 1) * 64 / NM - h * 64 / NM);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!LAST) st.tnext = tnext;
    }
    __builtin_amdgcn_s_setprio(0);
    st.l = st.l * alpha + psum;
    if constexpr (!LAST) {
#pragma unroll
        for (int jb = 0; jb < NB; ++jb) st.s[jb] = sn[jb];
    }
}

}  // namespace

// SPLIT: the unit of work is half an item, 64 rows; two waves share each 32-row block, one takes the first 32-key block of
// every tile, the other the second, each with a running maximum and sum of its own, and their results meet in LDS at the
// end.  Same copies and LDS per tile, half the products: for packs whose longest item outlasts the rest of the pass.
// More: InlineList when the work list is the second argument; TwoTeams when two teams of four waves take an item's key tiles in
// turn (the workgroup then has eight waves).
// Two teams: what bounds a pass whose longest item outlasts the rest is the number of iterations of that item, each of which takes a
// step's latency (barrier, first operand reads, softmax chain) whatever else is idle.  With the tiles dealt out in turn there are
// half as many; a SIMD then holds a wave of either team, as it does with two workgroups per unit.  The teams hold a maximum and a sum of
// their own and meet in LDS, as the halves of a tile do.  One head of 8192 tokens 88.9 -> 68.9 us (half items), 5 heads of 16001 321 ->
// 310 (whole), width 64, 8 heads of 8192 99 -> 86.  The choice is in teams_of_rows.
template <int D, bool BLOCK, int KD, bool SPLIT, typename... More>
__global__ __launch_bounds__(kThreads * teams_of<More...>, 2) void fwd_kernel(FwdParams p, More...) {
    constexpr int TEAMS = teams_of<More...>;
    using G = FwdGeom<D, KD>;
    constexpr int BQ = SPLIT ? kFwdQTile / 2 : kFwdQTile, BK = kFwdKTile;
    constexpr int NB = SPLIT ? 1 : 2;
    constexpr int KK = G::KK, DB = G::DB;
    constexpr int kTileBytes = G::kTileBytes;
    constexpr int kTeamBytes = 4 * kTileBytes;   // K tiles kt+1 / kt+2 and V tiles kt / kt+1: two buffers each
    constexpr int kRowBlocks = BQ / 32, kShares = TEAMS * (SPLIT ? 2 : 1);   // waves that share a row block
    __shared__ __attribute__((aligned(1024))) char lds[TEAMS * kTeamBytes];
    // the slot handed round after an item, double-buffered: between two hand-overs there is one barrier, and with a single
    // word the leader could overwrite it before a late wave has read it (items that only write zeros pass no other barrier)
    __shared__ int next_slot[2];
    __shared__ float2 row_stats[kShares > 1 ? (kShares - 1) * kRowBlocks * 64 : 1];   // (maximum, sum) that the other waves of a row block hand to the first
    char* const kbuf0 = lds;
    char* const vbuf0 = lds + 2 * kTileBytes;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = TEAMS > 1 ? wave_id & 3 : wave_id, team = TEAMS > 1 ? wave_id >> 2 : 0;
    const uint32_t kdst0 = lds_address(lds) + team * kTeamBytes, vdst0 = kdst0 + 2 * kTileBytes;   // the team's buffers as copy destinations
    const int row_block = SPLIT ? wave & 1 : wave, key_block = SPLIT ? wave >> 1 : 0;   // this wave's 32 rows; its keys of a tile
    const int share = team * (SPLIT ? 2 : 1) + key_block;
    const int hh = lane >> 5;
    const int hd = p.head_dim;   // elements per head in memory, <= D (columns hd .. D-1 exist only in LDS and registers)
    const float c = p.scale_log2;

    // what does not depend on the item: copy geometry and per-lane LDS offsets of the operand fragments
    TileCopy<D, BK> kvcopy;   // K and V share stride and geometry
    kvcopy.init(p.kv_stride, wave, lane, hd);
    int rm[KK], tr[DB][2];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) rm[kk] = tile_offset<D>(lane & 31, kk * 16 + hh * 8);
    {
        const int c16 = lane & 15;
        const int row = (hh << 2) + (c16 >> 2);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int col = db * 32 + (((lane >> 4) & 1) << 4) + ((c16 & 3) << 2);
            tr[db][0] = tile_offset<D>(row, col);
            tr[db][1] = tile_offset<D>(row + 8, col);
        }
    }
    if constexpr (kShares > 1) {
        const int skip = team * kTeamBytes + key_block * 32 * D * 2;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) rm[kk] += skip;
#pragma unroll
        for (int db = 0; db < DB; ++db) { tr[db][0] += skip; tr[db][1] += skip; }
    }

    // ---- one work item: a 128-row q tile of one (sequence, q head)
    ItemQueue queue;
    queue.init(p.queue);
    int drawn = 0;
    auto run_item = [&](const ItemGeom& item, int half) {
        // The lane index as the item's own code sees it: an empty statement makes it a new value per item, so that what
        // the prologue and the epilogue derive from it (row numbers, addresses of the staged stores) is computed per
        // item.  Derived from the kernel-wide lane index, those values would be loop-invariant, would be moved out of
        // the item loop and would then occupy registers all through the tile loop, which has none to spare.
        int lane = tid & 63;
        asm volatile("" : "+v"(lane));
        const int hh = lane >> 5;
        // the item's state is a new object: nothing of the previous item stays alive (a state kept across items would
        // hold the previous scores in registers through the prologue, wherever a wave might have no tile of its own)
        FwdState<D, KD, NB> st;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) st.rm[kk] = rm[kk];
#pragma unroll
        for (int db = 0; db < DB; ++db) { st.tr[db][0] = tr[db][0]; st.tr[db][1] = tr[db][1]; }
        const int Lq = item.q_len, L = item.k_len, off = item.offset;   // L: keys of the chunk (= rows when !BLOCK)
        const int h = item.head, hk = h / p.group;
        const int q_row0 = item.tile * kFwdQTile + (SPLIT ? half * BQ : 0);
        if (SPLIT && q_row0 >= Lq) {   // the last item of a sequence may have no second half
            if (tid == 0) drawn = queue.draw();
            return;
        }
        const int wave_row0 = q_row0 + row_block * 32;
        const int my_row = wave_row0 + (lane & 31);

        const uint16_t* qbase = p.q + (int64_t)item.q_start * p.q_stride + (int64_t)h * hd;
        const uint16_t* kbase = p.k + (int64_t)item.k_start * p.kv_stride + (int64_t)hk * hd;
        const uint16_t* vbase = p.v + (int64_t)item.k_start * p.kv_stride + (int64_t)hk * hd;

        // last key this lane's row may see (key j is visible to row r iff j <= r + off), as an index into the chunk
        const int my_limit = BLOCK ? min(my_row + off, L - 1) : my_row;
        const FwdTiles tiles = fwd_tiles(SPLIT, Lq, L, off, q_row0, row_block, key_block, TEAMS, team);
        const int n_tiles = tiles.n_tiles, n_tiles_w = tiles.n_tiles_w;
        if (BLOCK && tiles.n_passes == 0) {
            // no key of the chunk is visible to any row of the tile: O = 0, LSE = -inf
            if (my_row < Lq && share == 0) {
                float* orow = p.o_f32 + ((int64_t)(item.q_start + my_row) * p.q_heads + h) * hd;
    #pragma unroll
                for (int c4 = 0; c4 < D / 8; ++c4)
                    if (hh * (D / 2) + c4 * 4 < hd)
                        *reinterpret_cast<f32x4*>(orow + hh * (D / 2) + c4 * 4) = f32x4{0.f, 0.f, 0.f, 0.f};
                if (hh == 0) p.lse[(int64_t)h * p.total_tokens + item.q_start + my_row] = -INFINITY;
            }
            if (tid == 0) drawn = queue.draw();
            return;
        }

        auto tile_of = [=](int kt) { return TEAMS > 1 ? kt * TEAMS + team : kt; };   // the item's number of the team's tile kt
        auto first_key = [=](int kt) { return tile_of(kt) * BK; };
        // K(0), V(0), K(1)
        if (TEAMS == 1 || n_tiles > 0) {
            kvcopy.issue(kdst0, kbase, p.kv_stride, first_key(0), L, wave, lane);
            kvcopy.issue(vdst0, vbase, p.kv_stride, first_key(0), L, wave, lane);
        }
        if (n_tiles > 1) kvcopy.issue(kdst0 + kTileBytes, kbase, p.kv_stride, first_key(1), L, wave, lane);

    #pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            union { u32x4 u; bf16x8 v; } t;
            t.u = u32x4{0u, 0u, 0u, 0u};
            if (my_row < Lq && kk * 16 + hh * 8 < hd)
                t.u = *reinterpret_cast<const u32x4*>(qbase + (int64_t)my_row * p.q_stride + kk * 16 + hh * 8);
            st.qf[kk] = t.v;
        }
    #pragma unroll
        for (int db = 0; db < DB; ++db)
    #pragma unroll
            for (int i = 0; i < 16; ++i) st.acc[db][i] = 0.f;
        st.m = -INFINITY;
        st.l = 0.f;

        wait_tile_loads();
        __syncthreads();
        // S^T(0), not pipelined
        if (n_tiles_w > 0)
    #pragma unroll
        for (int jb = 0; jb < NB; ++jb) {
    #pragma unroll
            for (int i = 0; i < 16; ++i) st.s[jb][i] = 0.f;
    #pragma unroll
            for (int kk = 0; kk < KK; ++kk)
                st.s[jb] = mfma(*reinterpret_cast<const bf16x8*>(kbuf0 + st.rm[kk] + jb * 32 * D * 2), st.qf[kk], st.s[jb]);
        }
        st.tnext = n_tiles_w > 0 ? lane_max(st.s) : -INFINITY;
        // iteration 0 issues K(2) into the buffer that S^T(0) has just been read from: every wave must be done with it (a
        // wave may run ahead of another: one whose rows lie past the end of the chunk reads nothing here, and the waves of the
        // other resident workgroup hold some back)
        if (tiles.reuses_first_k()) __syncthreads();

        // iteration kt: K(kt+1) in kbuf[(kt+1) & 1], V(kt) in vbuf[kt & 1]; issues K(kt+2) -> kbuf[kt & 1] and
        // V(kt+1) -> vbuf[(kt+1) & 1], both free since the barrier at the top
        FwdTileLoad<D> no_load{};
        auto step = [&](int kt, auto masked, auto last) {
            if (kt > 0) {
                wait_tile_loads();
                __syncthreads();   // K(kt+1) and V(kt) have landed; every wave is done with iteration kt-1
            }
            if (kt + 2 < n_tiles) kvcopy.issue(kdst0 + (kt & 1) * kTileBytes, kbase, p.kv_stride, first_key(kt + 2), L, wave, lane);
            if (kt + 1 < n_tiles) kvcopy.issue(vdst0 + ((kt + 1) & 1) * kTileBytes, vbase, p.kv_stride, first_key(kt + 1), L, wave, lane);
            fwd_iteration<D, KD, NB, decltype(masked)::value, decltype(last)::value, false, BLOCK || (kShares > 1)>(
                st, kbuf0 + ((kt + 1) & 1) * kTileBytes, vbuf0 + (kt & 1) * kTileBytes, c,
                my_limit - first_key(kt) - key_block * 32 - 4 * hh, no_load);
        };
        // the same for an unmasked tile whose successors kt+1 and kt+2 are whole tiles: their copies need no case
        // distinction and are issued from inside the iteration
        // `parity` = kt & 1, as a run-time value or as a std::integral_constant: with a constant the LDS buffers of the
        // iteration are compile-time offsets and the operand reads need no address arithmetic
        auto step_spread = [&](int kt, auto parity) {
            const int par = parity;
            if (kt > 0) {
                wait_tile_loads();
                __syncthreads();
            }
            FwdTileLoad<D> load;
            load.copy = &kvcopy;
            load.k_row = kbase + (int64_t)tile_of(kt + 2) * BK * p.kv_stride;
            load.v_row = vbase + (int64_t)tile_of(kt + 1) * BK * p.kv_stride;
            load.k_dst = kdst0 + par * kTileBytes;
            load.v_dst = vdst0 + (1 - par) * kTileBytes;
            load.wave = wave;
            fwd_iteration<D, KD, NB, false, false, true, BLOCK || (kShares > 1)>(st, kbuf0 + (1 - par) * kTileBytes, vbuf0 + par * kTileBytes, c,
                                                        my_limit - first_key(kt) - 4 * hh, load);
        };
        // a tile past this wave's own diagonal: the barrier and the wave's share of the copies, nothing else
        auto idle = [&](int kt) {
            if (kt > 0) {
                wait_tile_loads();
                __syncthreads();
            }
            if (kt + 2 < n_tiles) kvcopy.issue(kdst0 + (kt & 1) * kTileBytes, kbase, p.kv_stride, first_key(kt + 2), L, wave, lane);
            if (kt + 1 < n_tiles) kvcopy.issue(vdst0 + ((kt + 1) & 1) * kTileBytes, vbase, p.kv_stride, first_key(kt + 1), L, wave, lane);
        };
        // separate loops instead of branches inside one: unmasked tiles (with and without whole successors), masked
        // tiles, and the wave's final tile (which has no successor to compute scores for); the large register state
        // then meets at a join once per loop, not per tile.  Every wave passes the barrier of every tile of the
        // workgroup, in whichever loop it happens to be.
        const int n_plain = tiles.n_plain, n_spread = tiles.n_spread;
        int kt = 0;
        // the long loop of a long sequence runs in pairs (even tile, odd tile) with constant buffer offsets
        for (; kt + 1 < n_spread; kt += 2) {
            step_spread(kt, std::integral_constant<int, 0>{});
            step_spread(kt + 1, std::integral_constant<int, 1>{});
        }
        for (; kt < n_spread; ++kt) step_spread(kt, kt & 1);
        for (; kt < n_plain; ++kt) step(kt, std::false_type{}, std::false_type{});
        for (; kt < n_tiles_w - 1; ++kt) step(kt, std::true_type{}, std::false_type{});
        if (n_tiles_w > 0) {
            step(kt, std::true_type{}, std::true_type{});   // the wave's final tile touches its diagonal (always, when !BLOCK)
            ++kt;
        }
        for (; kt < tiles.n_passes; ++kt) idle(kt);

        // the next slot is requested when the tiles are done (not earlier: a slot reserved at the start of a long item
        // would wait for that item while other workgroups run out of work) and looked at after the stores
        if (tid == 0) drawn = queue.draw();
        float l_row = st.l + partner32(st.l);
        // O leaves through LDS (free once every wave has left the tile loop) so that every store instruction writes
        // whole rows; a row that saw no key (BLOCK only) has l = 0 and m = -inf: O = 0, LSE = -inf
        __syncthreads();
        if constexpr (kShares > 1) {
            constexpr int kArea = 32 * D * 4;
            auto area = [&](int x) { return lds + (x * kRowBlocks + row_block) * kArea; };   // of share x; share 0's is where O is staged
            auto stats = [&](int x) -> float2& { return row_stats[((x - 1) * kRowBlocks + row_block) * 64 + lane]; };
            if (share > 0) {
    #pragma unroll
                for (int db = 0; db < DB; ++db)
    #pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4)
                        *reinterpret_cast<f32x4*>(area(share) + ((db * 4 + i4) * 64 + lane) * 16) =
                            f32x4{st.acc[db][4 * i4], st.acc[db][4 * i4 + 1], st.acc[db][4 * i4 + 2], st.acc[db][4 * i4 + 3]};
                stats(share) = make_float2(st.m, l_row);
            }
            __syncthreads();
            if (share > 0) return;
            // (a wave that met no key has m = -inf, l = 0, O = 0: its factor is exp2(-inf) = 0)
            float m = st.m;
    #pragma unroll
            for (int x = 1; x < kShares; ++x) m = fmaxf(m, stats(x).x);
            const float m_ref = m == -INFINITY ? 0.f : m;
            float fa = fast_exp2((st.m - m_ref) * c);
    #pragma unroll
            for (int x = 1; x < kShares; ++x) {
                const float2 other = stats(x);
                const float fb = fast_exp2((other.x - m_ref) * c);
    #pragma unroll
                for (int db = 0; db < DB; ++db)
    #pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        const f32x4 y = *reinterpret_cast<const f32x4*>(area(x) + ((db * 4 + i4) * 64 + lane) * 16);
    #pragma unroll
                        for (int j = 0; j < 4; ++j) st.acc[db][4 * i4 + j] = st.acc[db][4 * i4 + j] * fa + y[j] * fb;
                    }
                l_row = l_row * fa + other.y * fb;
                fa = 1.f;
            }
            st.m = m;
        }
        const float inv = (!BLOCK || l_row > 0.f) ? 1.f / l_row : 0.f;
        const int rows = min(32, Lq - wave_row0);
        const int64_t row0_elem = ((int64_t)(item.q_start + wave_row0) * p.q_heads + h) * hd;
        // the normaliser differs per row (= per lane): scale the fragments in place, then store with factor 1
    #pragma unroll
        for (int db = 0; db < DB; ++db)
    #pragma unroll
            for (int i = 0; i < 16; ++i) st.acc[db][i] *= inv;
        if constexpr (BLOCK) {
            store_tile_f32<D, false>(lds + row_block * (32 * D * 4), st.acc, 1.f, p.o_f32 + row0_elem, (int64_t)p.q_heads * hd, rows,
                                     hd, lane);
        } else {
            store_tile_bf16<D>(lds + row_block * (32 * D * 2), st.acc, 1.f, p.o + row0_elem, (int64_t)p.q_heads * hd, rows, hd, lane);
        }
        if (my_row < Lq && hh == 0)
            p.lse[(int64_t)h * p.total_tokens + item.q_start + my_row] =
                (!BLOCK || l_row > 0.f) ? (st.m * c + __log2f(l_row)) * kLn2 : -INFINITY;

    };

    // ---- the persistent loop: the first item is the workgroup's own slot, the others are drawn from its queue
    // (SPLIT: the entries of a queue are half items, an item's second half, which sees more keys, before its first)
    int slot = blockIdx.x;
    for (int turn = 0;; turn ^= 1) {
        const int list_slot = SPLIT ? slot / (2 * kQueues) * kQueues + slot % kQueues : slot;
        if (SPLIT && list_slot >= p.num_items) break;
        const ItemGeom item = load_item<BLOCK, has_inline_list<More...>>(p, list_slot);
        if (item.tile < 0) break;          // padding at the end of the queue: nothing left
        run_item(item, 1 - slot / kQueues % 2);
        if (tid == 0) next_slot[turn] = drawn;
        __syncthreads();                   // publishes the slot; every wave has left the item's LDS areas
        slot = __builtin_amdgcn_readfirstlane(next_slot[turn]);
        if (!SPLIT && slot >= p.num_items) break;
    }
    if (tid == 0) queue.leave();
}

namespace {

template <int D, int KD, typename... List>
void launch(const FwdParams& p, unsigned workgroups, bool block, bool split, hipStream_t stream, const List&... list) {
    const dim3 grid(workgroups), threads(kThreads), both_teams(2 * kThreads);
    const TwoTeams two{};
    if constexpr (D == 64 || sizeof...(List) == 0) {   // (whole items at tile width 128: only lists too long for the arguments)
        if (p.teams == 2 && !split) {
            hipLaunchKernelGGL((fwd_kernel<D, false, KD, false, List..., TwoTeams>), grid, both_teams, 0, stream, p, list..., two);
            return;
        }
    }
    if constexpr (sizeof...(List) != 0) {               // (half items: only lists in the arguments)
        if (p.teams == 2 && split) {
            hipLaunchKernelGGL((fwd_kernel<D, false, KD, true, List..., TwoTeams>), grid, both_teams, 0, stream, p, list..., two);
            return;
        }
    }
    if (block && split) hipLaunchKernelGGL((fwd_kernel<D, true, KD, true, List...>), grid, threads, 0, stream, p, list...);
    else if (block) hipLaunchKernelGGL((fwd_kernel<D, true, KD, false, List...>), grid, threads, 0, stream, p, list...);
    else if (split) hipLaunchKernelGGL((fwd_kernel<D, false, KD, true, List...>), grid, threads, 0, stream, p, list...);
    else hipLaunchKernelGGL((fwd_kernel<D, false, KD, false, List...>), grid, threads, 0, stream, p, list...);
}

// the kernel whose contraction over head_dim has as many 16-column steps as hold data, and whose products of output
// width head_dim have as many 32-column blocks (three up to 96)
template <typename... List>
void launch_width(const FwdParams& p, int head_dim, unsigned workgroups, bool block, bool split, hipStream_t stream, const List&... list) {
    if (tile_width(head_dim) == 64) launch<64, 4>(p, workgroups, block, split, stream, list...);
    else if (contraction_steps(head_dim) <= 5) launch<128, 5>(p, workgroups, block, split, stream, list...);
    else if (contraction_steps(head_dim) == 6) launch<128, 6>(p, workgroups, block, split, stream, list...);
    else if (contraction_steps(head_dim) == 7) launch<128, 7>(p, workgroups, block, split, stream, list...);
    else launch<128, 8>(p, workgroups, block, split, stream, list...);
}

}  // namespace

hipError_t launch_fwd(const FwdParams& params, const InlineList* list, int head_dim, int64_t num_items, bool block, hipStream_t stream) {
    if (num_items == 0) return hipSuccess;
    const bool split = params.split != 0;
    const int64_t slots = split ? 2 * ((num_items + kQueues - 1) / kQueues * kQueues) : num_items;
    // a short list has a workgroup for every slot: nothing to draw, and no round trip to the counters at the end of the item
    FwdParams p = params;
    const int64_t workgroups = list != nullptr ? slots : persistent_grid(slots, p.teams == 2 ? 1 : 2);
    if (workgroups <= 0) return hipErrorInvalidDevice;
    if (workgroups == slots) p.queue = nullptr;
    if (list) launch_width(p, head_dim, (unsigned)workgroups, block, split, stream, *list);
    else launch_width(p, head_dim, (unsigned)workgroups, block, split, stream);
    return hipGetLastError();
}

}  // namespace hspmd
