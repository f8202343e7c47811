// Backward dK/dV pass: one workgroup per (sequence, 128-key tile, kv head).
//
// Each of the 4 waves owns 32 keys (K and V rows stay in registers as MFMA B operands) and walks
// over the query heads of the KV group and, per head, over the 32-row query blocks at or below the
// diagonal.  Per block b:
//     G1(b): S' = Q_b K^T - LSE/scale, dP' = dO_b V^T - D    (16 MFMA, operands read along tile rows; the
//            statistics are the initial accumulator values)
//     V(b) : P = exp2(S' c), dS = P dP'                       (VALU, one lane per key)
//     G2(b): dV^T += dO_b^T P, dK^T += Q_b^T dS               (16 MFMA, operands by LDS transpose read)
// The group loop runs inside the workgroup, so dK/dV need no atomics.
//
// The kernel holds two fp32 accumulators of 32 x D per wave, which leaves room for only one wave
// per SIMD; one wave is one in-order instruction stream, so the loop is software-pipelined inside the
// wave and the instruction count per MFMA is kept low.  Iteration i is one basic block in two phases:
//     phase A: MFMA G2(i-1)  |  first half of V(i)   |  LDS reads: Q/dO rows and statistics of block i+1
//     phase B: MFMA G1(i+1)  |  second half of V(i)  |  LDS reads: Q^T/dO^T of block i (for G2(i) next time)
// so every MFMA operand is requested half an iteration (16 MFMAs) before its use and the exp/multiply work
// of one block is spread under the MFMAs of its neighbours.  S'/dP' are double buffered (block i is still
// being consumed while G1(i+1) accumulates).  The order is written out step by step, see dkv_iteration.
//
// LDS: four stages of {Q tile, dO tile (64 rows each), -LSE/scale [64], -D [64]}.  While iterations
// 2t and 2t+1 work on tile t and read ahead into tile t+1, tiles t+2 and t+3 are in flight
// (global -> LDS copies; t+3 goes into the stage that tile t-1 occupied).  One barrier per tile.
#include <type_traits>

#include "attn_device.hpp"
#include "kernels.hpp"
#include "schedule.hpp"

namespace hspmd {

namespace {

// KD: 16-column steps of the contractions over head_dim (G1) that hold data: D / 16, or fewer when head_dim ends
// before the tile width (the steps beyond it would multiply the zero padding of the K / V fragments); the products whose
// output is head_dim wide (G2) take (KD + 1) / 2 blocks of 32 columns.  8 x 2048, 32 heads, head_dim 96: 6 steps and 3 blocks
// instead of 7 and 4, 618 -> 527 us.
template <int D, int KD = D / 16>
struct DkvGeom {
    static_assert(KD >= 1 && KD <= D / 16, "k-steps inside the tile width");
    static constexpr int DB = (KD + 1) / 2;                // 32-row blocks of dK^T / dV^T that hold data
    static constexpr int KK = 2 * DB;                      // fragments per G2 operand (2 k-steps x DB row blocks)
    static constexpr int K1 = KD;                          // k-steps over head_dim of G1
    static constexpr int kTileBytes = kDkvQTile * D * 2;   // one 64-row tile
    static constexpr int kBlockBytes = 32 * D * 2;         // one 32-row block of it
    static constexpr int kStatBytes = 1024;                // -LSE/scale [64] at +0, -D [64] at +256
    static constexpr int kStageBytes = 2 * kTileBytes + kStatBytes;
    static constexpr int kStages = 4;
};

template <int D, int KD>
struct DkvState {
    using G = DkvGeom<D, KD>;
    bf16x8 kf[G::K1], vf[G::K1];           // this wave's 32 keys: K rows, V rows (B operands)
    f32x16 dk[G::DB], dv[G::DB];           // dK^T, dV^T accumulators
    f32x16 s[2], dp[2];                    // S - LSE/scale and dP - D: [i & 1] of block i, [~i & 1] of block i+1
    bf16x8 qf[G::K1], dof[G::K1];          // Q, dO rows of block i+1 (A operands of G1), live inside an iteration
    bf16x8 qtf[G::KK], dotf[G::KK];        // Q^T, dO^T of block i-1 (A operands of G2), index tt*DB + db
    bf16x8 pprev[2], dsprev[2];            // P, dS of block i-1 as bf16 B operands
};

// per-lane LDS byte addresses (stage base included) of the operand fragments
template <int D, int KD>
struct DkvAddr {
    using G = DkvGeom<D, KD>;
    int rm[G::KK];         // row-major fragment kk of a 32-row block (Q tile; dO tile is + kTileBytes)
    int tr[G::DB][2];      // transposed fragment: column block db, 8-row part
    int st;                // statistics
};

// The global -> LDS copies of one whole 64-row tile (Q chunks, dO chunks, one statistics row), cut into
// this wave's single instructions so that an iteration can issue them one at a time between its MFMAs:
// issued back to back after the barrier, the copies of all four waves queue up in front of the CU's one
// address unit and every wave sits in its issue slot for hundreds of cycles with nothing else to run.
template <int D>
struct DkvTileLoad {
    using Copy = TileCopy<D, kDkvQTile>;
    static constexpr int kPieces = 2 * Copy::kPerWave + 1;
    const Copy* qcopy;
    const Copy* docopy;
    const uint16_t* q_row;      // first row of the tile, this head, column 0
    const uint16_t* do_row;
    const float* stat;          // -LSE/scale (even waves) or -D (odd waves) of the tile's first row
    uint32_t stage;             // LDS byte addresses
    uint32_t stat_dst;
    int wave, lane;
    template <int N>
    __device__ __forceinline__ void piece() const {
        if constexpr (N < Copy::kPerWave) {
            qcopy->template issue_full_one<N>(stage, q_row, wave);
        } else if constexpr (N < 2 * Copy::kPerWave) {
            docopy->template issue_full_one<N - Copy::kPerWave>(stage + DkvGeom<D>::kTileBytes, do_row, wave);
        } else if constexpr (N == 2 * Copy::kPerWave) {
            global_to_lds<4>(stat, (uint32_t)lane * 4u, stat_dst);
        }
    }
    // the same with the index as an argument that is constant after unrolling
    __device__ __forceinline__ void piece_at(int n) const {
        if (n < Copy::kPerWave) qcopy->issue_full_one_at(n, stage, q_row, wave);
        else if (n < 2 * Copy::kPerWave)
            docopy->issue_full_one_at(n - Copy::kPerWave, stage + DkvGeom<D>::kTileBytes, do_row, wave);
        else if (n == 2 * Copy::kPerWave) global_to_lds<4>(stat, (uint32_t)lane * 4u, stat_dst);
    }
};

__device__ __forceinline__ bf16x8 lds_read128(const char* lds, int addr) {
    return *reinterpret_cast<const bf16x8*>(lds + addr);
}

template <int D>
__device__ __forceinline__ bf16x8 lds_read_tr(const char* lds, int a0, int a1) {
    const s16x4 lo = lds_transpose_read(lds + a0);
    const s16x4 hi = lds_transpose_read(lds + a1);
    union { struct { s16x4 a, b; } s; bf16x8 v; } u;
    u.s.a = lo;
    u.s.b = hi;
    return u.v;
}

// One pipelined iteration on block i (RB = i & 1 selects the accumulator pair that holds its S' / dP').
//   `cur`: addresses in the stage of block i's tile; `ahead`: addresses in the stage of block i+1's tile.
//   WHOLE: the wave takes both 32-row blocks of every tile in turn, so RB is also block i's position inside its tile and
//   block i+1 sits at the other one (of the next tile when RB == 1).  Otherwise the wave takes the same block of every
//   tile and the position is part of the addresses.
// dkey = my_key - (first row of block i) - 4 * (lane / 32): element e of an accumulator fragment is a
// masked (row < key) pair iff 8 * (e / 4) + e % 4 < dkey.
// SPREAD: the iteration also issues its share of the copies of a later tile (`load`), one instruction at a time.
//
// Both phases are written MFMA step by MFMA step: a step issues its MFMA, two or three LDS reads, a share of the exp / multiply
// work and at most one copy, and ends in a scheduling barrier.  With one wave per SIMD the order of the instruction stream is
// what overlaps, and left to scheduling hints it depended on what surrounded the loop: inside a loop over items one phase's 16
// LDS reads ended up behind its MFMAs.  Against the hints (us, sustained): half items of 2 sequences, 8 heads 36.9 -> 33.8; blocks
// of a ring of four over 32768 tokens, 24 heads 350 -> 338 each; 8 x 4096, 16 heads, head_dim 104 1000 -> 974; long packs, which
// the power limit decides, unchanged.  The exp work is spread evenly: in the first 12 of 16 steps it takes 5 % longer.  Whole items of
// tile width 64 have two waves per SIMD, which cover each other, and less MFMA work per score: there the compiler orders each phase by
// a hint (short sequences 68.8 us against 70.2 step by step), and so it does for some items of several query heads, see
// dkv_iteration_hinted.
template <int D, int KD, int RB, bool MASK, bool SPREAD, bool WHOLE>
__device__ __forceinline__ void dkv_iteration(DkvState<D, KD>& st, const char* lds, const DkvAddr<D, KD>& ahead,
                                              const DkvAddr<D, KD>& cur, int dkey, float c, const DkvTileLoad<D>& load) {
    using G = DkvGeom<D, KD>;
    constexpr int KK = G::KK, DB = G::DB, K1 = G::K1;
    constexpr int NRB = RB ^ 1;
    constexpr int CUR = WHOLE ? RB : 0, AHEAD = WHOLE ? NRB : 0;   // positions of blocks i and i+1 beyond the addresses
    constexpr int NA = 2 * KK, NB = 2 * K1;                        // MFMA steps of the two phases
    constexpr bool kSteps = D == 128 || !WHOLE;
    // this iteration's share of the copies, spread evenly over its steps
    constexpr int kAll = DkvTileLoad<D>::kPieces;
    constexpr int kFirstPiece = WHOLE && RB == 1 ? kAll / 2 : 0;
    constexpr int kPieces = !SPREAD ? 0 : !WHOLE ? kAll : RB == 0 ? kAll / 2 : kAll - kAll / 2;
    auto copies = [&](int step) {
        if constexpr (kPieces > 0) {
#pragma unroll
            for (int x = 0; x < kPieces; ++x)
                if ((2 * x + 1) * (NA + NB) / (2 * kPieces) == step) load.piece_at(kFirstPiece + x);
        }
    };

    // The exp / multiply work of half a block (8 elements, one B operand of P and one of dS): four pairs, four shares each.  An
    // empty statement on a share's results keeps it in its step: nothing else needs them before the end of the phase.
    u32x4 pw, dw;
    float p0 = 0.f, p1 = 0.f, d0 = 0.f;
    auto share = [&](int half, int x) {
        const int e = 8 * half + x / 4 * 2, w = x / 4;
        if (x % 4 == 0) {
            p0 = st.s[RB][e] * c;
            p1 = st.s[RB][e + 1] * c;
            if constexpr (kSteps) asm volatile("" : "+v"(p0), "+v"(p1));
        } else if (x % 4 == 1) {
            p0 = fast_exp2(p0);
            p1 = fast_exp2(p1);
            if constexpr (kSteps) asm volatile("" : "+v"(p0), "+v"(p1));
        } else if (x % 4 == 2) {
            if (MASK && (8 * (e >> 2) + (e & 3) < dkey)) p0 = 0.f;
            if (MASK && (8 * ((e + 1) >> 2) + ((e + 1) & 3) < dkey)) p1 = 0.f;
            uint32_t pair = pack_bf16(p0, p1);
            d0 = p0 * st.dp[RB][e];
            if constexpr (kSteps) asm volatile("" : "+v"(pair), "+v"(d0));
            pw[w] = pair;
        } else {
            uint32_t pair = pack_bf16(d0, p1 * st.dp[RB][e + 1]);
            if constexpr (kSteps) asm volatile("" : "+v"(pair));
            dw[w] = pair;
        }
    };
    auto end_step = [] {
        if constexpr (kSteps) __builtin_amdgcn_sched_barrier(0);
    };

    // ================= phase A: G2(i-1); reads of block i+1 =================
    // the statistics go straight into the accumulators: rows 8 j + 4 (lane / 32) .. + 3 in registers 4 j .. 4 j + 3
    auto read_ahead = [&](int r) {
        if (r < 8) {
            const int i4 = r / 2;
            const f32x4 a = *reinterpret_cast<const f32x4*>(lds + ahead.st + AHEAD * 128 + i4 * 32 + (r & 1) * 256);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (r & 1) st.dp[NRB][4 * i4 + j] = a[j];
                else st.s[NRB][4 * i4 + j] = a[j];
            }
        } else {
            const int kk = (r - 8) / 2;
            if (r & 1) st.dof[kk] = lds_read128(lds, ahead.rm[kk] + AHEAD * G::kBlockBytes + G::kTileBytes);
            else st.qf[kk] = lds_read128(lds, ahead.rm[kk] + AHEAD * G::kBlockBytes);
        }
    };
    constexpr int kReadsA = 8 + 2 * K1;
    static_assert(kReadsA <= 2 * NA, "two reads a step");
#pragma unroll
    for (int n = 0; n < NA; ++n) {
        const int kk = n / 2, tt = kk / DB, db = kk % DB;
        if (n % 2 == 0) st.dv[db] = mfma(st.dotf[kk], st.pprev[tt], st.dv[db]);
        else st.dk[db] = mfma(st.qtf[kk], st.dsprev[tt], st.dk[db]);
#pragma unroll
        for (int r = 2 * n; r < 2 * n + 2; ++r)
            if (r < kReadsA) read_ahead(r);
#pragma unroll
        for (int x = n * 16 / NA; x < (n + 1) * 16 / NA; ++x) share(0, x);
        copies(n);
        end_step();
    }
    if constexpr (!kSteps) {
        // per MFMA: LDS reads and a share of the VALU work
        InterleaveHint<NA, 2, (MASK ? 4 : 3), 0, 0x402>::apply();
        __builtin_amdgcn_sched_barrier(0);
    }

    // ================= phase B: G1(i+1) on top of the statistics; transpose reads of block i =================
    union { u32x4 u; bf16x8 v; } cv;
    cv.u = pw; st.pprev[0] = cv.v;
    cv.u = dw; st.dsprev[0] = cv.v;
    auto read_back = [&](int r) {
        const int kk = r / 2, tt = kk / DB, db = kk % DB;
        const int off = (CUR * 2 + tt) * 16 * D * 2;   // 16 tile rows per k-step
        if (r % 2 == 0) st.dotf[kk] = lds_read_tr<D>(lds, cur.tr[db][0] + off + G::kTileBytes, cur.tr[db][1] + off + G::kTileBytes);
        else st.qtf[kk] = lds_read_tr<D>(lds, cur.tr[db][0] + off, cur.tr[db][1] + off);
    };
    // the two accumulation chains in turn: an MFMA that continues a chain does not follow its predecessor directly
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        if (n % 2 == 0) st.s[NRB] = mfma(st.qf[n / 2], st.kf[n / 2], st.s[NRB]);
        else st.dp[NRB] = mfma(st.dof[n / 2], st.vf[n / 2], st.dp[NRB]);
#pragma unroll
        for (int r = n * 2 * KK / NB; r < (n + 1) * 2 * KK / NB; ++r) read_back(r);
#pragma unroll
        for (int x = n * 16 / NB; x < (n + 1) * 16 / NB; ++x) share(1, x);
        copies(NA + n);
        end_step();
    }
    if constexpr (!kSteps) {
        InterleaveHint<NB, 2, (MASK ? 4 : 3), 1, 0x402>::apply();
        __builtin_amdgcn_sched_barrier(0);
    }
    cv.u = pw; st.pprev[1] = cv.v;
    cv.u = dw; st.dsprev[1] = cv.v;
}

// The same iteration of a whole item, its order left to the compiler by hints: per MFMA two LDS reads and a share of the other work,
// copies at fixed places among the LDS reads (the copies are ordered against LDS accesses, the reads are tied to the MFMAs by the
// hints): pieces 0-3 in the first iteration of a tile, 4-8 in the second.
//
// For packed items of several query heads with all eight contraction steps, one tile per trip (see GROUPS below).  They gain nothing
// from the order above and lose a little.  Interleaved in one process (us, hints / steps in trips of two): 65536 tokens, 32 heads on 8
// 16188 / 16306, on other boxes 15948 / 16033, 16057 / 16156 and 17455 / 17813; 5 sequences of 700 .. 2500, 32 on 8 237.0 / 238.5;
// 64 x 512, 32 on 16 520.4 / 521.7; 4 x 4096, 32 on 16 1003 / 1005; 2 x 8192 and 16384 tokens, 32 on 8 equal.  On the box of 17455,
// steps with one tile a trip take 18070, trips of hints inside the function above 17862.  The others keep the steps: narrower heads
// (2 x 8192, 32 on 8, head_dim 104 1775 / 1747, 96 1534 / 1517, 80 1479 / 1459; 64 x 512, 32 on 16, 104 535 / 527), blocks (6 x 2178,
// 24 on 8 370 / 354; 2 x 8192, 32 on 8 1938 / 1819), persistent workgroups (head_dim 104 288 / 282).
template <int D, int KD, int RB, bool MASK, bool SPREAD>
__device__ __forceinline__ void dkv_iteration_hinted(DkvState<D, KD>& st, const char* lds, const DkvAddr<D, KD>& ahead,
                                                     const DkvAddr<D, KD>& cur, int dkey, float c, const DkvTileLoad<D>& load) {
    using G = DkvGeom<D, KD>;
    constexpr int KK = G::KK, DB = G::DB, K1 = G::K1;
    constexpr int NRB = RB ^ 1;
    constexpr int P0 = RB == 0 ? 0 : 4;   // first piece of this iteration

    // element e of an accumulator fragment -> packed bf16 pair index; one half = 8 elements = one B operand
    auto softmax_half = [&](int half, u32x4& pw, u32x4& dw) {
#pragma unroll
        for (int e = 8 * half; e < 8 * half + 8; e += 2) {
            float p0 = fast_exp2(st.s[RB][e] * c);
            float p1 = fast_exp2(st.s[RB][e + 1] * c);
            if (MASK && (8 * (e >> 2) + (e & 3) < dkey)) p0 = 0.f;
            if (MASK && (8 * ((e + 1) >> 2) + ((e + 1) & 3) < dkey)) p1 = 0.f;
            pw[(e >> 1) & 3] = pack_bf16(p0, p1);
            dw[(e >> 1) & 3] = pack_bf16(p0 * st.dp[RB][e], p1 * st.dp[RB][e + 1]);
        }
    };

    // ================= phase A =================
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(lds + ahead.st + NRB * 128 + i4 * 32);
        const f32x4 b = *reinterpret_cast<const f32x4*>(lds + ahead.st + NRB * 128 + i4 * 32 + 256);
#pragma unroll
        for (int j = 0; j < 4; ++j) { st.s[NRB][4 * i4 + j] = a[j]; st.dp[NRB][4 * i4 + j] = b[j]; }
    }
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) {
        st.qf[kk] = lds_read128(lds, ahead.rm[kk] + NRB * G::kBlockBytes);
        st.dof[kk] = lds_read128(lds, ahead.rm[kk] + NRB * G::kBlockBytes + G::kTileBytes);
        if constexpr (SPREAD) {
            if (kk == KK / 4 - 1) load.template piece<P0>();
            if (kk == 3 * KK / 4 - 1) load.template piece<P0 + 1>();
        }
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        const int tt = kk / DB, db = kk % DB;
        st.dv[db] = mfma(st.dotf[kk], st.pprev[tt], st.dv[db]);
        st.dk[db] = mfma(st.qtf[kk], st.dsprev[tt], st.dk[db]);
    }
    u32x4 pw0, dw0;
    softmax_half(0, pw0, dw0);
    InterleaveHint<2 * KK, 2, (MASK ? 4 : 3), 0, 0x402>::apply();
    __builtin_amdgcn_sched_barrier(0);

    // ================= phase B =================
    union { u32x4 u; bf16x8 v; } cv;
    cv.u = pw0; st.pprev[0] = cv.v;
    cv.u = dw0; st.dsprev[0] = cv.v;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int off = (RB * 2 + tt) * 16 * D * 2;   // 16 tile rows per k-step
            st.qtf[tt * DB + db] = lds_read_tr<D>(lds, cur.tr[db][0] + off, cur.tr[db][1] + off);
            st.dotf[tt * DB + db] = lds_read_tr<D>(lds, cur.tr[db][0] + off + G::kTileBytes, cur.tr[db][1] + off + G::kTileBytes);
            if constexpr (SPREAD) {
                if (tt == 0 && db == DB - 1) load.template piece<P0 + 2>();
                if (tt == 1 && db == DB / 2 - 1) load.template piece<P0 + 3>();
                if (RB == 1 && tt == 1 && db == DB - 1) load.template piece<P0 + 4>();
            }
        }
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) {
        st.s[NRB] = mfma(st.qf[kk], st.kf[kk], st.s[NRB]);
        st.dp[NRB] = mfma(st.dof[kk], st.vf[kk], st.dp[NRB]);
    }
    u32x4 pw1, dw1;
    softmax_half(1, pw1, dw1);
    cv.u = pw1; st.pprev[1] = cv.v;
    cv.u = dw1; st.dsprev[1] = cv.v;
    InterleaveHint<2 * K1, (K1 == KK ? 2 : 3), (MASK ? 4 : 3), 1, 0x402>::apply();
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace

// Tile width 64: the accumulators are half as large, so two workgroups fit a compute unit (248 registers per wave, 2 x 68 KB
// of LDS) and one hides the other's prologue, stores and waits.  Against one workgroup with 280 registers: 16384 tokens in
// sequences of 32 .. 512, 16 heads: 98 -> 62 us; 8 x 2048, 32 heads: 396 -> 298 us; 2 x 8192, 8 heads on 2: 444 -> 413 us.
//
// SPLIT: a workgroup takes half an item, 64 keys; the waves are two pairs over the keys, and one pair takes the first
// 32-row block of every tile, the other the second.  Same copies and LDS per tile, half the products, so a half item takes
// 0.68 of the time: for packs whose longest item outlasts the rest of the pass.  The two
// accumulator pairs of a key meet in LDS at the end, in one fixed order.
//
// PERSIST: the workgroup draws items from its queue until none is left (as the forward does), for packs of many items (short_items and
// persistent_dkv in schedule.cpp).
//
// GROUPS: whole packed items of several query heads at head_dim above 112, one workgroup each; every head is walked one tile at a time,
// in the compiler's order (dkv_iteration_hinted).
//
// List: nothing, InlineList when the work list is the second argument, or HeadPieces where items are dealt out by query heads and tiles: a share
// leaves fp32 sums in its area (build_piece_list in schedule.cpp).
template <int D, bool BLOCK, int KD, bool SPLIT, bool PERSIST, bool GROUPS, typename... List>
__global__ __launch_bounds__(kThreads, (D == 64 && !SPLIT ? 2 : 1)) void bwd_dkv_kernel(BwdParams p, List...) {
    static_assert(!PERSIST || (!BLOCK && !SPLIT), "whole items of packed plans only");
    static_assert(!GROUPS || (KD == 8 && !BLOCK && !SPLIT && !PERSIST), "whole items of packed plans, head_dim above 112");
    constexpr bool kPieces = has_pieces<List...>;
    static_assert(!kPieces || (!BLOCK && !PERSIST && !GROUPS), "packed plans, a workgroup per share");
    constexpr bool kTrips = !SPLIT && !GROUPS && D == 128;   // whole items, two tiles a trip
    using G = DkvGeom<D, KD>;
    constexpr int BKV = SPLIT ? kDkvKTile / 2 : kDkvKTile, BQ = kDkvQTile;
    constexpr int KK = G::KK, DB = G::DB, K1 = G::K1;
    __shared__ __attribute__((aligned(1024))) char lds[G::kStages * G::kStageBytes];

    // workgroups p and p + 8 of 16 take the halves of an item: like the item itself they belong to XCD p % 8
    int slot = SPLIT ? (int)(blockIdx.x / (2 * kQueues)) * kQueues + (int)(blockIdx.x % kQueues) : (int)blockIdx.x;
    if (SPLIT && slot >= p.num_items) return;
    PersistentLoop<PERSIST> loop;
    loop.init(p.queue);
    do {
    ItemGeom item;
    int first_head = 0, n_heads = p.group;   // query heads of the group that this workgroup walks
    int share_first = 0, share_end = 0;      // kPieces: the query tiles
    if constexpr (kPieces) {
        const HeadPiece it = load_piece<has_inline_list<List...>>(p, slot);
        if (it.padding()) break;
        item = ItemGeom{it.token_start, it.seq_len, it.token_start, it.seq_len, 0, it.tile(), it.head(), 0};
        first_head = it.first_head();
        n_heads = it.n_heads(p.group);
        share_first = it.first_tile();
        share_end = it.end_tile();
    } else {
        item = load_item<BLOCK, has_inline_list<List...>>(p, slot);
    }
    if (item.tile < 0) break;
    const int tid = threadIdx.x, lane = loop.item_lane();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = item.q_len, Lk = item.k_len, shift = item.offset, g = item.head;   // L: rows of the chunk
    const int first_q_head = g * p.group + first_head;
    const int key0 = item.tile * kDkvKTile + (SPLIT ? (int)(blockIdx.x / kQueues % 2) * BKV : 0);
    if (SPLIT && key0 >= Lk) return;             // the last item of a sequence may have no second half
    const int row_block = SPLIT ? wave >> 1 : 0;   // the 32-row block of every tile that is this wave's
    const int wave_key0 = key0 + (SPLIT ? wave & 1 : wave) * 32;
    const int my_key = wave_key0 + (lane & 31);
    const int hh = lane >> 5;
    const bool valid = my_key < Lk;

    int hd = p.head_dim;   // elements per head in memory, <= D (columns hd .. D-1 exist only in LDS and registers)
    // (a value of its own: spilled as one group with its neighbours among the parameters, it leaves a stack object behind)
    if constexpr (kPieces) asm volatile("" : "+s"(hd));
    const uint16_t* kbase = p.k + (int64_t)item.k_start * p.kv_stride + (int64_t)g * hd;
    const uint16_t* vbase = p.v + (int64_t)item.k_start * p.kv_stride + (int64_t)g * hd;

    constexpr int kLoadsPerTile = 2 * (BQ * D * 2 / 1024) / 4 + 1;   // per wave: Q and dO chunks + one statistics copy
    // tiles: for each head of the group, q tiles first_qt .. n_qt-1 (rows at or below the diagonal: row r sees
    // key j iff j <= r + shift, so the tile's first key is seen by the rows from key0 - shift on)
    const int diagonal_qt = max(0, key0 - shift) / BQ;
    // (the second half of an item starts a tile further down.  A share of one head's tiles has three and more, so the half finds some in its
    // first share too; other shares hold the whole range, and where that is one tile the item has no second half)
    const int first_qt = kPieces ? max(diagonal_qt, share_first) : diagonal_qt;
    const int n_qt = kPieces ? share_end : (L + BQ - 1) / BQ;
    const int per_head = max(0, n_qt - first_qt);
    const int n_tiles = per_head * n_heads;
    if (BLOCK && per_head == 0) {
        // no row of the chunk sees these keys
        if (valid && row_block == 0) {
            const int64_t row_elem = ((int64_t)(item.k_start + my_key) * p.kv_heads + g) * hd;
#pragma unroll
            for (int c4 = 0; c4 < D / 8; ++c4) {
                if (hh * (D / 2) + c4 * 4 >= hd) continue;
                store_grad4(p.dk, row_elem + hh * (D / 2) + c4 * 4, p.grad_f32 != 0, 0.f, 0.f, 0.f, 0.f);
                store_grad4(p.dv, row_elem + hh * (D / 2) + c4 * 4, p.grad_f32 != 0, 0.f, 0.f, 0.f, 0.f);
            }
        }
        return;
    }

    // global -> LDS copy of tile u (flattened over heads) into a stage, statistics included
    const uint32_t lds0 = lds_address(lds);   // copy destinations are LDS byte addresses
    TileCopy<D, BQ> qcopy, docopy;
    qcopy.init(p.q_stride, wave, lane, hd);
    docopy.init((int64_t)p.q_heads * hd, wave, lane, hd);
    auto load_tile = [&](int u, int stage_index) {
        const uint32_t stage = lds0 + stage_index * G::kStageBytes;
        const int hq = first_q_head + u / per_head;
        const int row0 = (n_qt - 1 - u % per_head) * BQ;   // q tiles are walked from the end of the sequence down
        const uint16_t* qb = p.q + (int64_t)item.q_start * p.q_stride + (int64_t)hq * hd;
        const uint16_t* dob = p.d_o + ((int64_t)item.q_start * p.q_heads + hq) * hd;
        // even waves: -LSE/scale of the 64 rows; odd waves: -D (waves 2, 3 repeat the copies of waves 0, 1 so that
        // every wave has the same number of loads in flight)
        const int which = wave & 1;
        const uint32_t stat_dst = stage + 2 * G::kTileBytes + which * 256;
        const int64_t stat0 = (int64_t)hq * p.total_tokens + item.q_start + row0;
        if (row0 + BQ <= L) {
            qcopy.issue_full(stage, qb, p.q_stride, row0, wave);
            docopy.issue_full(stage + G::kTileBytes, dob, (int64_t)p.q_heads * hd, row0, wave);
            global_to_lds<4>((which == 0 ? p.nlse : p.negd) + stat0, (uint32_t)lane * 4u, stat_dst);
        } else {
            // last tile of a head: rows past the end read a finite duplicate; their -LSE/scale reads -inf, so P = 0
            qcopy.issue_clamped(stage, qb, p.q_stride, row0, L, wave, lane);
            docopy.issue_clamped(stage + G::kTileBytes, dob, (int64_t)p.q_heads * hd, row0, L, wave, lane);
            const int r = row0 + lane;
            const int64_t stat = stat0 + min(lane, L - 1 - row0);
            const float* src = (which == 0) ? ((r < L) ? p.nlse + stat : p.ninf_pad) : p.negd + stat;
            global_to_lds<4>(src, stat_dst);
        }
    };

    load_tile(0, 0);
    if (n_tiles > 1) load_tile(1, 1);
    if (n_tiles > 2) load_tile(2, 2);

    DkvState<D, KD> st;
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) {
        union { u32x4 u; bf16x8 v; } a, b;
        a.u = u32x4{0u, 0u, 0u, 0u};
        b.u = u32x4{0u, 0u, 0u, 0u};
        if (valid && kk * 16 + hh * 8 < hd) {
            a.u = *reinterpret_cast<const u32x4*>(kbase + (int64_t)my_key * p.kv_stride + kk * 16 + hh * 8);
            b.u = *reinterpret_cast<const u32x4*>(vbase + (int64_t)my_key * p.kv_stride + kk * 16 + hh * 8);
        }
        st.kf[kk] = a.v;
        st.vf[kk] = b.v;
    }
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) { st.dk[db][i] = 0.f; st.dv[db][i] = 0.f; }
    const float c = p.scale_log2;

    // per-lane fragment offsets inside a stage
    DkvAddr<D, KD> off;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) off.rm[kk] = tile_offset<D>(lane & 31, kk * 16 + hh * 8);
    {
        const int c16 = lane & 15;
        const int row = (hh << 2) + (c16 >> 2);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int col = db * 32 + (((lane >> 4) & 1) << 4) + ((c16 & 3) << 2);
            off.tr[db][0] = tile_offset<D>(row, col);
            off.tr[db][1] = tile_offset<D>(row + 8, col);
        }
    }
    off.st = 2 * G::kTileBytes + hh * 16;
    if constexpr (SPLIT) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) off.rm[kk] += row_block * G::kBlockBytes;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            off.tr[db][0] += row_block * G::kBlockBytes;
            off.tr[db][1] += row_block * G::kBlockBytes;
        }
        off.st += row_block * 128;
    }
    // `off` holds the addresses of the current tile's stage and is moved from stage to stage by adding the
    // distance (one set of address registers instead of one per stage in use)
    auto shifted = [&](const DkvAddr<D, KD>& a0, int bytes) {
        DkvAddr<D, KD> a;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) a.rm[kk] = a0.rm[kk] + bytes;
#pragma unroll
        for (int db = 0; db < DB; ++db) { a.tr[db][0] = a0.tr[db][0] + bytes; a.tr[db][1] = a0.tr[db][1] + bytes; }
        a.st = a0.st + bytes;
        return a;
    };

    wait_tile_loads();
    __syncthreads();   // tiles 0, 1 and 2 are in LDS

    // prologue: G1(0) computed directly on top of block 0's statistics; P = dS = 0 for the non-existent block -1
    {
        const DkvAddr<D, KD>& a0 = off;   // stage 0
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            const f32x4 a = *reinterpret_cast<const f32x4*>(lds + a0.st + i4 * 32);
            const f32x4 b = *reinterpret_cast<const f32x4*>(lds + a0.st + i4 * 32 + 256);
#pragma unroll
            for (int j = 0; j < 4; ++j) { st.s[0][4 * i4 + j] = a[j]; st.dp[0][4 * i4 + j] = b[j]; }
        }
#pragma unroll
        for (int kk = 0; kk < K1; ++kk) {
            st.s[0] = mfma(lds_read128(lds, a0.rm[kk]), st.kf[kk], st.s[0]);
            st.dp[0] = mfma(lds_read128(lds, a0.rm[kk] + G::kTileBytes), st.vf[kk], st.dp[0]);
        }
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            st.qtf[kk] = lds_read128(lds, a0.rm[kk]);      // any finite operand: it meets P = dS = 0
            st.dotf[kk] = st.qtf[kk];
        }
        union { u32x4 u; bf16x8 v; } z;
        z.u = u32x4{0u, 0u, 0u, 0u};
        st.pprev[0] = st.pprev[1] = st.dsprev[0] = st.dsprev[1] = z.v;
    }

    // One tile = two iterations.  The two q tiles next to the diagonal hold the (row < key) pairs of some wave
    // and take the masked code; all other tiles take the unmasked code.  Two loops instead of a branch inside
    // one: the ~400 live registers then meet at a join once per head, not once per iteration.
    int stage = 0;   // stage of tile u
    DkvTileLoad<D> no_load{};
    // S' and dP' of a tile's first block come out of the matrix core in the tile before.  Told nothing, the compiler copies all 32 of
    // them to vector registers where a loop or a branch begins; held in accumulation registers up to here (an empty statement),
    // they are copied one by one under the MFMAs of the steps that use them.
    auto hold_in_acc = [&] {
        if constexpr (kTrips) asm volatile("" : "+a"(st.s[0]), "+a"(st.dp[0]));
    };
    // `par`: SPLIT, where a tile is one iteration: the accumulator pair that holds the tile's S' / dP'.  Otherwise, 0 for the item's
    // first tile, 1 for the first and 2 for the second tile of a trip
    auto tile_step = [&](int u, int qt, auto masked, auto par) {
        constexpr bool kMask = decltype(masked)::value;
        constexpr int kPar = decltype(par)::value;
        if (u > 0) {
            // tile u+1 must have landed; the copies of tile u+2 (the newest kLoadsPerTile of this wave) may still fly
            if (u + 2 < n_tiles) wait_tile_loads_except<kLoadsPerTile>(); else wait_tile_loads();
            __syncthreads();   // ... for every wave; and every wave is done with tile u-1
        }
        const int stage1 = stage + 1 == G::kStages ? 0 : stage + 1;
        const int stage3 = (stage + 3) % G::kStages;
        if (u + 3 < n_tiles) load_tile(u + 3, stage3);
        // block 2u+2 lives in the next tile; the last tile has none: it re-reads itself (result unused)
        const int to_next = (stage1 - stage) * G::kStageBytes;
        const DkvAddr<D, KD> next = shifted(off, u + 1 < n_tiles ? to_next : 0);
        const int dkey0 = my_key - shift - qt * BQ - row_block * 32 - 4 * hh;
        hold_in_acc();
        if constexpr (SPLIT) {
            dkv_iteration<D, KD, kPar, kMask, false, false>(st, lds, next, off, dkey0, c, no_load);
        } else if constexpr (GROUPS) {
            dkv_iteration_hinted<D, KD, 0, kMask, false>(st, lds, off, off, dkey0, c, no_load);
            dkv_iteration_hinted<D, KD, 1, kMask, false>(st, lds, next, off, dkey0 - 32, c, no_load);
        } else {
            dkv_iteration<D, KD, 0, kMask, false, true>(st, lds, off, off, dkey0, c, no_load);
            dkv_iteration<D, KD, 1, kMask, false, true>(st, lds, next, off, dkey0 - 32, c, no_load);
        }
        off = shifted(off, to_next);
        stage = stage1;
    };
    // The same for an unmasked tile that is at least three tiles above the head's last one: the tile loaded
    // meanwhile (u + 3) belongs to the same head and is a whole tile, so its copies need no case distinction
    // and are issued from inside the two iterations.
    // `load` arrives pointing at the first rows of tile qt - 3 of the head and leaves pointing one tile lower.
    auto tile_step_spread = [&](int u, int qt, DkvTileLoad<D>& load, auto par) {
        constexpr int kPar = decltype(par)::value;
        if constexpr (kPar < 2) hold_in_acc();
        if (kPar >= 1 || u > 0) {
            wait_tile_loads_except<kLoadsPerTile>();   // u + 2 < n_tiles here
            __syncthreads();
        }
        const int stage1 = stage + 1 == G::kStages ? 0 : stage + 1;
        const int stage3 = stage == 0 ? G::kStages - 1 : stage - 1;   // (stage + 3) % kStages
        load.stage = lds0 + stage3 * G::kStageBytes;
        load.stat_dst = load.stage + 2 * G::kTileBytes + (wave & 1) * 256;
        const int to_next = (stage1 - stage) * G::kStageBytes;
        const DkvAddr<D, KD> next = shifted(off, to_next);
        const int dkey0 = my_key - shift - qt * BQ - row_block * 32 - 4 * hh;
        if constexpr (SPLIT) {
            dkv_iteration<D, KD, kPar, false, true, false>(st, lds, next, off, dkey0, c, load);
        } else if constexpr (GROUPS) {
            dkv_iteration_hinted<D, KD, 0, false, true>(st, lds, off, off, dkey0, c, load);
            dkv_iteration_hinted<D, KD, 1, false, true>(st, lds, next, off, dkey0 - 32, c, load);
        } else {
            dkv_iteration<D, KD, 0, false, true, true>(st, lds, off, off, dkey0, c, load);
            dkv_iteration<D, KD, 1, false, true, true>(st, lds, next, off, dkey0 - 32, c, load);
        }
        off = shifted(off, to_next);
        load.q_row -= (int64_t)BQ * p.q_stride;
        load.do_row -= (int64_t)BQ * p.q_heads * hd;
        load.stat -= BQ;
        stage = stage1;
    };
    // Every head is walked from its LAST q tile down to the diagonal.  All key tiles of one (sequence, kv head)
    // run on one XCD at about the same time; walking down from the common end keeps them on the same Q / dO
    // tiles at the same time (one L2 fill serves them all), whereas walking up from each item's own diagonal
    // would spread them over the whole sequence.
    // q tiles that hold some (row, key) pair above the shifted diagonal for the keys of this workgroup:
    // qt BQ + shift < key0 + BKV - 1; the two nearest the diagonal when there is no shift
    const int n_masked = BLOCK ? (key0 + BKV - 2 - shift < 0 ? 0 : max(0, min(per_head, (key0 + BKV - 2 - shift) / BQ - first_qt + 1)))
                               : kPieces ? max(0, min(BKV / BQ - (first_qt - diagonal_qt), per_head)) : min(BKV / BQ, per_head);
    const int n_general = max(3, n_masked);   // tiles below this index (from the diagonal) take the general path
    // SPLIT: tiles are walked in pairs, one per accumulator pair; after a single tile the pairs change places
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    using Second = std::integral_constant<int, 2>;
    auto swap_pairs = [&] { st.s[0] = st.s[1]; st.dp[0] = st.dp[1]; };
    for (int h = 0, u = 0; h < n_heads; ++h) {
        int j = per_head - 1;
        if (j >= n_general) {
            const int hq = first_q_head + h;
            const int64_t row = item.q_start + (int64_t)(first_qt + j - 3) * BQ;   // first row of the tile loaded first
            DkvTileLoad<D> load;
            load.qcopy = &qcopy;
            load.docopy = &docopy;
            load.q_row = p.q + row * p.q_stride + (int64_t)hq * hd;
            load.do_row = p.d_o + (row * p.q_heads + hq) * hd;
            load.stat = ((wave & 1) == 0 ? p.nlse : p.negd) + (int64_t)hq * p.total_tokens + row;
            load.wave = wave;
            load.lane = lane;
            if constexpr (kTrips) {
                // Two tiles a trip, in one basic block: a conditional barrier in it, or one tile a trip, gathers the copies of S' and
                // dP' (see hold_in_acc) where the block begins, with no MFMA beside them.  8 x 2048, 32 heads 639 -> 610 us against
                // 623, the pack of 32768 tokens 2563 -> 2564 against 2604; four tiles a trip 623 and 2595 (7 KB of code more to fetch).
                if (u == 0) {
                    tile_step_spread(u, first_qt + j, load, Even{});
                    --j, ++u;
                }
                for (; j > n_general; j -= 2, u += 2) {
                    tile_step_spread(u, first_qt + j, load, Odd{});
                    tile_step_spread(u + 1, first_qt + j - 1, load, Second{});
                }
                if (j >= n_general) {
                    tile_step_spread(u, first_qt + j, load, Odd{});
                    --j, ++u;
                }
            } else if constexpr (SPLIT) {
                for (; j > n_general; j -= 2, u += 2) {
                    tile_step_spread(u, first_qt + j, load, Even{});
                    tile_step_spread(u + 1, first_qt + j - 1, load, Odd{});
                }
            }
            if constexpr (!kTrips)
            for (; j >= n_general; --j, ++u) {
                tile_step_spread(u, first_qt + j, load, Even{});
                if constexpr (SPLIT) swap_pairs();
            }
        }
        for (; j >= n_masked; --j, ++u) {
            tile_step(u, first_qt + j, std::false_type{}, Even{});
            if constexpr (SPLIT) swap_pairs();
        }
        for (; j >= 0; --j, ++u) {
            tile_step(u, first_qt + j, std::true_type{}, Even{});
            if constexpr (SPLIT) swap_pairs();
        }
    }

    loop.draw();
    // epilogue: G2 of the last block
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        const int tt = kk / DB, db = kk % DB;
        st.dv[db] = mfma(st.dotf[kk], st.pprev[tt], st.dv[db]);
        st.dk[db] = mfma(st.qtf[kk], st.dsprev[tt], st.dk[db]);
    }

    // whole rows per store instruction, staged through LDS (free once every wave has left the tile loop)
    int area = -1;   // where the sums of a share go
    if constexpr (kPieces) {
        int again = slot;   // (read here and not kept through the tile loop)
        asm volatile("" : "+s"(again));
        const HeadPiece it = load_piece<has_inline_list<List...>>(p, again);
        if (it.shares(p.group) > 1) area = it.area();
    }
    const bool sums = kPieces && area >= 0;
    const bool rope = !sums && p.rope_table != nullptr;
    __syncthreads();
    constexpr int kWaveArea = 32 * D * 4;
    static_assert(!SPLIT || 8 * kWaveArea <= G::kStages * G::kStageBytes, "exchange and staging areas");
    char* wave_lds = lds + wave * kWaveArea;
    if constexpr (SPLIT) {
        // the waves of a key pair hold the two row blocks' shares: the first hands its dV over and stores dK, the second
        // hands its dK over and stores dV
        auto slot16 = [&](int w, int db, int i4) {
            return reinterpret_cast<f32x4*>(lds + w * kWaveArea + ((db * 4 + i4) * 64 + lane) * 16);
        };
        auto hand_over = [&](const f32x16 (&x)[DB]) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4)
                    *slot16(wave, db, i4) = f32x4{x[db][4 * i4], x[db][4 * i4 + 1], x[db][4 * i4 + 2], x[db][4 * i4 + 3]};
        };
        auto take_over = [&](f32x16 (&x)[DB]) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const f32x4 y = *slot16(wave ^ 2, db, i4);
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[db][4 * i4 + j] += y[j];
                }
        };
        if (row_block == 0) hand_over(st.dv);
        else hand_over(st.dk);
        __syncthreads();
        if (row_block == 0) take_over(st.dk);
        else take_over(st.dv);
        wave_lds += 4 * kWaveArea;   // the partner may still read this wave's exchange area
    }
    const bool stores_dk = !SPLIT || row_block == 0, stores_dv = !SPLIT || row_block == 1;
    const int64_t row0_elem = sums ? (int64_t)(wave_key0 - item.tile * kDkvKTile) * D : ((int64_t)(item.k_start + wave_key0) * p.kv_heads + g) * hd;
    const int64_t row_stride = sums ? D : (int64_t)p.kv_heads * hd;
    float* const dk_f32 = sums ? p.piece_sums + (int64_t)area * (2 * kDkvKTile * D) : static_cast<float*>(p.dk);
    float* const dv_f32 = sums ? p.piece_sums + (int64_t)area * (2 * kDkvKTile * D) + kDkvKTile * D : static_cast<float*>(p.dv);
    const int rows = min(32, Lk - wave_key0);
    if (!stores_dk) {
    } else if (rope) {
        // dK with respect to the keys before their rotary embedding; key positions inside the sequence
        store_tile_rope_transposed<D>(wave_lds, st.dk, p.scale, p.dk, row0_elem, p.grad_f32 != 0, row_stride, rows, hd,
                                      p.rope_table + (int64_t)(item.q_pos - item.offset + wave_key0) * hd, lane);
    } else if (sums || p.grad_f32 != 0) {
        store_tile_f32<D, false>(wave_lds, st.dk, sums ? 1.f : p.scale, dk_f32 + row0_elem, row_stride, rows, hd, lane);
    } else {
        store_tile_bf16<D>(wave_lds, st.dk, p.scale, static_cast<uint16_t*>(p.dk) + row0_elem, row_stride, rows, hd, lane);
    }
    if (!stores_dv) {
    } else if (sums || p.grad_f32 != 0) {
        store_tile_f32<D, false>(wave_lds, st.dv, 1.f, dv_f32 + row0_elem, row_stride, rows, hd, lane);
    } else {
        store_tile_bf16<D>(wave_lds, st.dv, 1.f, static_cast<uint16_t*>(p.dv) + row0_elem, row_stride, rows, hd, lane);
    }
    } while (loop.next(slot, p.num_items));
    loop.leave();
}

// Sum of an item's areas, in the order of the heads and tiles.  A workgroup takes 16 keys of the item whose first share its entry of the list
// is; a thread four columns of the lower half of a row and the four that the rotary embedding pairs them with, of dK and dV.  Bound by
// the areas' way out of L2 and memory.
template <typename... List>
__global__ __launch_bounds__(kThreads) void bwd_piece_sums_kernel(BwdParams p, List...) {
    const HeadPiece it = load_piece<has_inline_list<List...>>(p, blockIdx.x / (kDkvKTile / 16));
    if (it.padding() || it.index() != 0) return;
    const int areas = it.shares(p.group);
    if (areas == 1) return;
    const int hd = p.head_dim, half = hd / 2, pairs = hd / 8, width = hd <= 64 ? 64 : 128;
    const int row = (int)(blockIdx.x % (kDkvKTile / 16)) * 16 + (int)threadIdx.x / 16, c = (int)threadIdx.x % 16;
    const int position = it.tile() * kDkvKTile + row;
    if (position >= it.seq_len || c >= pairs) return;
    const int64_t area = 2 * kDkvKTile * (int64_t)width;
    const float* at = p.piece_sums + it.area() * area + (int64_t)row * width + c * 4;
    f32x4 k_lo{0.f, 0.f, 0.f, 0.f}, k_hi = k_lo, v_lo = k_lo, v_hi = k_lo;
    for (int i = 0; i < areas; ++i, at += area) {
        k_lo += *reinterpret_cast<const f32x4*>(at);
        k_hi += *reinterpret_cast<const f32x4*>(at + half);
        v_lo += *reinterpret_cast<const f32x4*>(at + kDkvKTile * width);
        v_hi += *reinterpret_cast<const f32x4*>(at + kDkvKTile * width + half);
    }
    k_lo *= p.scale;
    k_hi *= p.scale;
    if (p.rope_table != nullptr) {
        const float* t = p.rope_table + ((int64_t)position * half + c * 4) * 2;
        const f32x4 t01 = *reinterpret_cast<const f32x4*>(t), t23 = *reinterpret_cast<const f32x4*>(t + 4);
        const f32x4 cs{t01[0], t01[2], t23[0], t23[2]}, sn{t01[1], t01[3], t23[1], t23[3]};
        const f32x4 lo = k_lo, hi = k_hi;
        k_lo = lo * cs + hi * sn;
        k_hi = hi * cs - lo * sn;
    }
    const int64_t elem = ((int64_t)(it.token_start + position) * p.kv_heads + it.head()) * hd + c * 4;
    const bool f32 = p.grad_f32 != 0;
    store_grad4(p.dk, elem, f32, k_lo[0], k_lo[1], k_lo[2], k_lo[3]);
    store_grad4(p.dk, elem + half, f32, k_hi[0], k_hi[1], k_hi[2], k_hi[3]);
    store_grad4(p.dv, elem, f32, v_lo[0], v_lo[1], v_lo[2], v_lo[3]);
    store_grad4(p.dv, elem + half, f32, v_hi[0], v_hi[1], v_hi[2], v_hi[3]);
}

namespace {

template <int D, int KD, typename... List>
hipError_t launch_dkv(const BwdParams& p, int64_t num_items, bool block, hipStream_t stream, const List&... list) {
    const dim3 threads(kThreads);
    if (p.piece_sums != nullptr) {
        const HeadPieces shares{};
        if (p.split != 0) hipLaunchKernelGGL((bwd_dkv_kernel<D, false, KD, true, false, false, List..., HeadPieces>), dim3((unsigned)((num_items + kQueues - 1) / kQueues * kQueues * 2)), threads, 0, stream, p, list..., shares);
        else hipLaunchKernelGGL((bwd_dkv_kernel<D, false, KD, false, false, false, List..., HeadPieces>), dim3((unsigned)num_items), threads, 0, stream, p, list..., shares);
        return hipGetLastError();
    }
    if (p.split != 0) {
        const dim3 grid((unsigned)((num_items + kQueues - 1) / kQueues * kQueues * 2));
        if (block) hipLaunchKernelGGL((bwd_dkv_kernel<D, true, KD, true, false, false, List...>), grid, threads, 0, stream, p, list...);
        else hipLaunchKernelGGL((bwd_dkv_kernel<D, false, KD, true, false, false, List...>), grid, threads, 0, stream, p, list...);
    } else {
        const dim3 grid((unsigned)num_items);
        if constexpr (D == 128 && sizeof...(List) == 0) {   // (an inline list is too short for persistent workgroups)
            if (!block && p.persist) {
                const int workgroups = persistent_grid(num_items, 1);
                if (workgroups > 0) {
                    hipLaunchKernelGGL((bwd_dkv_kernel<D, false, KD, false, true, false>), dim3((unsigned)workgroups), threads, 0, stream, p);
                    return hipGetLastError();
                }
                if (p.persist == 1) return hipErrorInvalidDevice;
            }
        }
        if constexpr (KD == 8 && sizeof...(List) == 0) {   // (with the list in the arguments the two walks take the same time)
            if (!block && p.group > 1) {
                hipLaunchKernelGGL((bwd_dkv_kernel<D, false, KD, false, false, true>), grid, threads, 0, stream, p);
                return hipGetLastError();
            }
        }
        if (block) hipLaunchKernelGGL((bwd_dkv_kernel<D, true, KD, false, false, false, List...>), grid, threads, 0, stream, p, list...);
        else hipLaunchKernelGGL((bwd_dkv_kernel<D, false, KD, false, false, false, List...>), grid, threads, 0, stream, p, list...);
    }
    return hipGetLastError();
}

template <typename... List>
hipError_t launch_dkv_width(const BwdParams& p, int head_dim, int64_t num_items, bool block, hipStream_t stream, const List&... list) {
    if (tile_width(head_dim) == 64) return launch_dkv<64, 4>(p, num_items, block, stream, list...);
    if (contraction_steps(head_dim) <= 5) return launch_dkv<128, 5>(p, num_items, block, stream, list...);
    if (contraction_steps(head_dim) == 6) return launch_dkv<128, 6>(p, num_items, block, stream, list...);
    if (contraction_steps(head_dim) == 7) return launch_dkv<128, 7>(p, num_items, block, stream, list...);
    return launch_dkv<128, 8>(p, num_items, block, stream, list...);
}

}  // namespace

hipError_t launch_bwd_dkv(const BwdParams& p, const InlineList* list, int head_dim, int64_t num_items, bool block, hipStream_t stream) {
    if (num_items == 0) return hipSuccess;
    return list ? launch_dkv_width(p, head_dim, num_items, block, stream, *list)
                : launch_dkv_width(p, head_dim, num_items, block, stream);
}

hipError_t launch_piece_sums(const BwdParams& p, const InlineList* list, int64_t count, hipStream_t stream) {
    if (count == 0) return hipSuccess;
    const dim3 grid((unsigned)(count * (kDkvKTile / 16))), threads(kThreads);
    if (list) hipLaunchKernelGGL((bwd_piece_sums_kernel<InlineList>), grid, threads, 0, stream, p, *list);
    else hipLaunchKernelGGL((bwd_piece_sums_kernel<>), grid, threads, 0, stream, p);
    return hipGetLastError();
}

}  // namespace hspmd
