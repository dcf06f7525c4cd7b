// wavefront_impl.h -- the strip sweep shared by the pair sweep (wavefront.hip)
// and the tile sweep (tile.hip).  See wavefront.hip for the design.
#pragma once

#include "twed_dispatch.h"

namespace twed {

// Polls of a predecessor's progress word before a wave gives up (tens of
// seconds either way: an LDS poll takes about 0.1 us with its sleep, a
// global one a few us).
constexpr uint32_t kMaxPollsLds = 1u << 28;
constexpr uint32_t kMaxPollsGlobal = 1u << 24;
// The error word (a global load, a few us) is read once every kErrEvery
// polls, so a waiting wave notices its predecessor's progress within one
// poll.
constexpr uint32_t kErrEvery = 64;

template <typename AT>
struct alignas(2 * sizeof(AT)) Pair2 {
    AT dp;
    AT x;
};

// Rows per global handoff (one window of the 64-lane boundary register).
// Inside a workgroup the handoff comes every 1 << sub_shift steps (8, 16 or
// 32; a kernel argument).
constexpr int kWindow = 64;
// Rows of one in-group boundary kept in LDS (power of two), plus one slot
// that absorbs the writes of lanes without a row.  Row r sits at slot
// (r - 1) mod 128: the rows a sub-chunk of steps reads or writes then fill
// consecutive slots without a wrap (sub-chunks start at multiples of their
// length, and rows t + 1 come in and rows t - 63 go out at step t), so a step
// reaches them at a constant offset from an address kept in a register.
constexpr int kRing = 128;
__host__ __device__ constexpr int ring_slot(int r) { return (r - 1) & (kRing - 1); }
// Most steps between two updates of the boundary addresses.
constexpr int kMaxUnroll = 4;
// No row of any lane (rows run from -63).
constexpr int kNoRow = -0x40000000;

// Rows of A reach the lanes through LDS: every 64 steps lane l of a wave loads
// row t + l and writes it to the wave's ring, and at step t lane l reads row
// t - l.  The ring holds 64-row chunks c - 1 and c, always contiguous (chunk c
// even at rows 64 .. 127, odd at rows 128 .. 191 and again at 0 .. 63), so a
// step needs no address wrap.  Read from global memory by every lane at every
// step, a row came 64 times through the L1 (2 KB per wave and step for 32-byte
// rows, at 64 B per cycle) and its latency, three steps of a narrow strip, was
// often not hidden: 3-D FP32 strips took 150 ns per step whatever their width.
// Samples whose rings do not fit the LDS beside the rest keep the global reads.
template <typename CT, int DIMT, int G>
constexpr bool kRowRing = kRingRows * Row<CT, DIMT>::kStride * (int)sizeof(CT) * G <= kRingBytes;
static_assert(kRingRows == 3 * kWave + 2, "two chunks, one of them twice, and two rows read ahead");
// resident_group of a kernel.
template <typename CT, int DIMT, int PM>
constexpr int kResidentGroup = kRowRing<CT, DIMT, 4> || PM == kLp ? 4 : 1;

template <typename CT, typename AT, int DIMT, int G>
struct GroupShared {
    alignas(16) CT rows[G][kRowRing<CT, DIMT, G> ? kRingRows * Row<CT, DIMT>::kStride : 1];
    Pair2<AT> ring[G > 1 ? G - 1 : 1][kRing + 1];  // boundary of wave w, read by wave w+1
    Pair2<AT> in_stage[kWindow + 1];               // wave 0's left boundary, one global window
    Pair2<AT> in_next[kWindow];                    // the next window, when it is there early
    Pair2<AT> out_stage[kRing + 1];                // wave G-1's right boundary before it goes out
    Pair2<AT> dummy[kWave + kMaxUnroll];           // takes the boundary writes of lanes 0 .. 62
    int prod[G + 2];                               // rows of that boundary written; a sink; "all" (no wave to wait for)
    int cons[G];                                   // rows of wave w's left boundary consumed
    uint32_t ticket[G];                            // ticket value seen by each wave (wave 0's is the claim)
};

// Bounded wait until *p >= need (uniform across the wave).  A wave that gives
// up marks the error word (the result strip then reports NaN) and carries
// on, and once the word is set no wave waits any more (it is read every
// kErrEvery polls), so every wave still reaches the end of the grid after at
// most one time-out.
__device__ __forceinline__ void wait_progress(const uint32_t *p, uint32_t need, uint32_t *err)
{
    uint32_t polls = 0;
    while (load_progress(p) < need) {
        if (polls % kErrEvery == kErrEvery - 1 && load_progress(err) != 0u) break;
        __builtin_amdgcn_s_sleep(1);
        if (++polls > kMaxPollsGlobal) {
            __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
    }
}

// The same for a count in LDS: of the boundary rows that wave w - 1 of the group
// has written or wave w has read.  Returns the count seen last.
// All LDS operations of a compute unit are performed one after another, those of
// a wave in its order, so rows written before a count are there for whoever has
// read the count, and neither side waits for what else it has in flight (with
// workgroup fences, which wait for every load and store: the 8-D pair of 10^6
// samples 866 ms, now 855; 30,000 x 30,000 1-D in FP64 4.69 ms, now 4.63).
__device__ __forceinline__ int wait_rows(const int *prod, int need, uint32_t *err)
{
    uint32_t polls = 0;
    int seen;
    while ((seen = __builtin_amdgcn_readfirstlane(
                __hip_atomic_load(prod, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))) < need) {
        if (polls % kErrEvery == kErrEvery - 1 && load_progress(err) != 0u) break;
        if (polls >= 4) __builtin_amdgcn_s_sleep(1);  // not yet under way: leave the SIMD to others
        if (++polls > kMaxPollsLds) {
            __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
    }
    return seen;
}

// Block boundaries and extra outputs of the tile sweep (TILE kernels only;
// pair sweeps pass an empty set).  Cells are (DP, X = DP + e) pairs.
//   top     row 0 of the block, columns 0..nB (null: the pad row of a pair)
//   left    column 0 of the block, rows 0..nA (null: the pad column)
//   bottom  receives row nA, columns 1..nB
//   right   receives column nB, rows 1..nA
//   ckrow   receives rows ck_rows, 2*ck_rows, ... below nA (nB + 1 cells
//           each; column 0 is left to the host)
//   ckcol   receives columns ck_cols, 2*ck_cols, ... left of nB (nA + 1
//           cells each; row 0 is left to the host); ck_cols is a multiple
//           of the strip width
//   dirs    (DIRS kernels, K = 1) the move into every cell, in sweep order:
//           strip s, 32 steps, lane, 64 bits of two per step (1 the match, 2 the
//           deletion in B from the cell on the left, 0 the deletion in A from
//           the cell above); ceil((nA + 64) / 32) * 64 words per strip
//   dummy   64*K cells that lanes without a cell to store write instead
template <typename AT>
struct TileIO {
    const Pair2<AT> *top;
    const Pair2<AT> *left;
    Pair2<AT> *bottom;
    Pair2<AT> *right;
    Pair2<AT> *ckrow;
    Pair2<AT> *ckcol;
    Pair2<AT> *dummy;
    uint64_t *dirs;
    int ck_rows;
    int ck_cols;
};

// Strip widths compiled for a sample dimension: beyond 16 components a lane
// holds at most two columns (wider strips would not fit the register file).
template <int DIMT, int K>
constexpr bool kStripCompiled = DIMT <= 16 || K <= 2;

// One strip of 64*K columns swept by one wave.  Its left boundary (DP and X =
// DP + e of column c0-1, per row) comes from the previous strip: through LDS
// when that strip belongs to the same workgroup (counted every kSub = 1 <<
// sub_shift rows), through a global slot and flag otherwise (every kWindow
// rows, agent-scope release/acquire).  Its right boundary goes the
// same two ways to the next strip.
//
// rowsA points at row 0 of A, with kRowPad rows before it and kRowPadTail after
// row nA.  Lanes that have not started yet, or have finished, sweep rows
// outside 1..nA (with the ring, rows of zeros before row 0) and compute values
// nobody uses, so the row address needs no clamp.
//
// What bounds a step: with one wave on a SIMD, everything the step issues, so
// the loop holds no branch, no address arithmetic beyond one update every four
// steps and no scalar test; the cells themselves are the floor.  Before this
// form a step of one FP64 1-D column took 178 ns, now 100; with the width rule
// 30,000 x 30,000 samples went from 10.5 to 4.9 ms, 1,000 x 1,000 from 355 to
// 181 us, 100,000 x 100,000 3-D in FP32 from 29.6 to 22.2 ms.
//
// A tile sweep (TILE) starts from a given top row and left column instead of
// the pad row and column.  A lane processes rows 0 and below before its
// first real row; in a pair sweep those rows keep the +inf state of the pad
// row, and in a tile the lane loads its top-row cells at the step where it
// sits on row 0, so that row 1 starts from them.
template <typename CT, typename AT, int DIMT, int PM, int K, int G, bool DUMP, bool TILE, int REC, bool DIRS>
__device__ __forceinline__ void sweep_strip(GroupShared<CT, AT, DIMT, G> &sh, int w, int g, int s, int cbase,
                                            const CT *__restrict__ rowsA,
                                            const CT *__restrict__ rowsB, int nA, int nB, const CostArgs<CT> &ca,
                                            Pair2<AT> *bnd, uint32_t *flags, uint32_t *err, int nStrips, CT beta,
                                            AT *out, AT *dump, int sub_shift, const TileIO<AT> &io)
{
    static_assert(REC == kRecTwed || TILE, "sibling recurrences run as tiles");
    static_assert(!DIRS || TILE, "moves are recorded by tile sweeps");
    static_assert(!DIRS || K == 1, "moves are packed by lane");
    const int kSub = DIRS ? 32 : 1 << sub_shift;
    constexpr int S = Row<CT, DIMT>::kStride;
    constexpr int W = kWave * K;
    const int lane = threadIdx.x & (kWave - 1);
    const AT INF = pinf<AT>();
    // ---- columns of this lane (the strip's first column is 1 + cbase)
    const int c0 = 1 + cbase + lane * K;
    Lane<CT, AT, DIMT, K> L;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        Row<CT, DIMT> b;
        const int c = c0 + j <= nB ? c0 + j : nB;
        load_row<CT, DIMT>(rowsB, c, b);
#pragma unroll
        for (int k = 0; k < DIMT; ++k) L.bx[j][k] = b.x[k];
        L.bt[j] = b.t;
        L.bdel[j] = kShifted<AT> ? (AT)(b.del - beta) : (AT)b.del;
        L.up[j] = INF;   // DP(0, c)
        L.xp[j] = INF;   // DP(0, c) + e(0, c)
    }

    const bool in_global = w == 0 && (s > 0 || (TILE && io.left != nullptr));
    const bool in_lds = w > 0;
    const bool has_out = s + 1 < nStrips;
    const bool out_lds = has_out && w < G - 1;
    const bool out_global = has_out && w == G - 1;
    // global slots alternate between consecutive groups (see the header comment)
    const Pair2<AT> *in_slot = (TILE && s == 0) ? io.left : bnd + (size_t)((g + 1) & 1) * (size_t)(nA + 1);
    Pair2<AT> *out_slot = bnd + (size_t)(g & 1) * (size_t)(nA + 1);
    const uint32_t *in_flag = flags + (g > 0 ? g - 1 : 0);
    uint32_t *out_flag = flags + g;

    // column nB sits in the last strip, at lane lstar, column jstar
    const bool result_strip = s == nStrips - 1;
    const int qs = (nB - 1) - cbase;
    const int lstar = qs / K, jstar = qs - (qs / K) * K;

    // Operands shifted in from lane l-1 after each step: sh_l is the left
    // operand DP(r, c0-1) of the next step, sh_xo its up-left operand
    // X(r-1, c0-1) = DP + e, and sh_x the X value that becomes sh_xo one
    // step later.  Lane 0 takes them from the strip's left boundary
    // instead: +inf on the pad row and column, except X(0, 0) = 0 (minus
    // the offset) for the first strip.
    AT sh_l = INF;
    AT sh_x = (lane == 0 && s == 0) ? -(AT)beta : INF;
    AT sh_xo = INF;
    Pair2<AT> *ck_col = nullptr;
    if constexpr (TILE) {
        // X(0, c0 - 1) of this strip: from the top row, else the corner
        AT x0 = INF;
        if (io.top != nullptr) x0 = io.top[cbase].x;
        else if (s == 0) x0 = io.left != nullptr ? io.left[0].x : AT(0);
        sh_x = lane == 0 ? x0 : INF;
        if (io.ckcol != nullptr && has_out && (cbase + W) % io.ck_cols == 0)
            ck_col = io.ckcol + (size_t)((cbase + W) / io.ck_cols - 1) * (size_t)(nA + 1);
    }

    // A tile's top-row cells wait in registers for the step at which the lane
    // sits on row 0, and the cells of a row that is stored (the last, or a
    // checkpoint) until every lane has swept it.  A strip follows the one before
    // it by some 110 steps, so what the 64 steps around such a row cost more than
    // others is paid again in every strip along the front: dummy stores by the
    // other lanes, a branch, a load or the wait for stores at the next hand-over.
    // (Forward sweep of a path of 100,000 8-D samples: 53.4 ms with dummy stores,
    // 38.8 with branches, now 36.)  Wide strips have no registers to spare.
    constexpr bool kCellsKept = TILE && K <= 2;
    Pair2<AT> tops[kCellsKept ? K : 1], kept[kCellsKept ? K : 1];
    if constexpr (kCellsKept) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            tops[j] = io.top != nullptr ? io.top[c0 + j <= nB ? c0 + j : nB] : Pair2<AT>{INF, INF};
            kept[j] = Pair2<AT>{INF, INF};
        }
    }
    // the first checkpoint row not yet passed by every lane, and where it goes
    // (rows at least 128 apart, so that one is kept at a time)
    int ck_next = io.ck_rows;
    Pair2<AT> *ck_row = io.ckrow;
    const bool rows_kept =
        kCellsKept && !DIRS && (io.ckrow == nullptr || (io.bottom == nullptr && io.ck_rows >= 2 * kWave));

    const int T = nA + kWave;  // lane 63 reaches row nA at step nA + 63
    // The last strip stops once lane lstar has swept row nA (its lanes past
    // lstar hold columns beyond nB): the result is then in that lane's
    // registers, and the step loop carries no test for it.
    const int T_run = result_strip ? nA + lstar + 1 : T;
    // Rows are read kAhead steps ahead of their use: from the wave's ring in
    // LDS, or from global memory (large samples).
    // (Wide strips of large samples, whose columns fill the registers, have none
    // left for the ring's loads.)
    constexpr int kRowWords = S * (int)sizeof(CT) / 4;
    constexpr bool RR = kRowRing<CT, DIMT, G> && kRowWords * K <= 96;
    // One row read ahead, not two, and steps kept apart, two to a turn: for rows of
    // 17 .. 32 FP64 components, or the rows in flight alone fill the registers
    // (32-D, 3,000 x 300 samples: 1.23 ms with two ahead and four to a turn, now
    // 1.00; pairs in strips of two columns, which read no ring, keep four), and for
    // more than eight components in general Lp, whose powers, inlined for every
    // component of four steps, overrun the instruction cache (FP64 12-D, 10,000 x
    // 800 samples: 68.7 ms, now 62.9).
    constexpr bool kTwoSteps = (kRowWords > 64 && (RR || TILE)) || (PM == kLp && DIMT > 8);
    // How many steps ahead of its use a row and a boundary cell are read: an LDS
    // read takes about as long as a narrow strip's step (1-D FP64: 1,000 x 1,000
    // samples 181 -> 174 us, 30,000 x 30,000 4.88 -> 4.69 ms from one to two).
    constexpr int kAhead = RR && !kTwoSteps ? 2 : 1;
    constexpr int V = 16 / (int)sizeof(CT);
    typedef CT vec __attribute__((ext_vector_type(V)));
    CT *const rows_lds = &sh.rows[w][0];
    vec fetched[S / V];
    auto fetch = [&](int t) {  // rows t .. t + 63, a row per lane (those past nA + 64 repeat a padding row)
        const int r = t + lane < nA + kRowPad ? t + lane : nA + kRowPad;
        const vec *p = reinterpret_cast<const vec *>(rowsA + (ptrdiff_t)r * S);
#pragma unroll
        for (int v = 0; v < S / V; ++v) fetched[v] = p[v];
    };
    auto put = [&](int slot) {
        vec *p = reinterpret_cast<vec *>(rows_lds + (slot + lane) * S);
#pragma unroll
        for (int v = 0; v < S / V; ++v) p[v] = fetched[v];
    };
    static_assert(kRowPad <= kRowPadTail && kWave <= kRowPadTail, "rows up to nA + 64 are read");
    Row<CT, DIMT> row[4];
    Pair2<AT> nbs[2];
    const CT *row_at;  // row t - lane, the row lane `lane` works on at step t
    if constexpr (RR) {
        // lanes that have not reached row 0 sweep rows of zeros
#pragma unroll
        for (int v = 0; v < S / V; ++v) fetched[v] = vec{};
        put(0);
        fetch(0);
        row_at = rows_lds;
    } else {
        row_at = rowsA - (ptrdiff_t)lane * S;
        load_row<CT, DIMT>(row_at, 0, row[0]);
    }
    // Lane 0's left operands of the next step come from one LDS read at a
    // wave-uniform address (a broadcast: no cross-lane moves, no lane
    // selection): from the ring of the previous wave of the group, or from
    // in_stage, which holds one window of the global slot (or +inf: the pad
    // column of the first strip).  Lane 63's output of every step -- the
    // strip's right boundary -- goes to the ring of the next wave, or to
    // out_stage when it leaves the group through global memory, from where
    // whole windows are copied out.  Every lane executes that store, the others
    // into cells nobody reads: masking them off took five scalar instructions
    // and a branch per step, which a strip alone on its SIMD pays for in full.
    // In-group hand-over: this wave's count goes to prod_out, the count of the
    // wave before comes from prod_in.
    const int *const prod_in = in_lds ? &sh.prod[w - 1] : &sh.prod[G + 1];
    int *const prod_out = out_lds ? &sh.prod[w] : &sh.prod[G];
    int counted = 0, consumed = 0;  // the last counts seen: of the wave before, and by the wave behind
    const bool has_in = in_global || in_lds;
    if (!has_in) sh.in_stage[lane] = Pair2<AT>{INF, INF};
    // boundary row t + 1 sits at in_src[t & in_mask]: ring slot t mod 128, or
    // in_stage slot t mod 64
    const int in_mask = in_lds ? kRing - 1 : kWindow - 1;
    const Pair2<AT> *const in_src = in_lds ? &sh.ring[w > 0 ? w - 1 : 0][0] : &sh.in_stage[0];
    Pair2<AT> *const out_ring = out_lds ? &sh.ring[w < G - 1 ? w : 0][0] : &sh.out_stage[0];

    // The next global window is fetched ahead when it is already published:
    // its flag is read at the start of the window's second-to-last sub-chunk
    // (the load completes behind that sub-chunk's steps), checked at the last
    // one, and the window's rows go to in_next there.  Otherwise the window
    // start waits for the flag.  (Rows held in registers until the window
    // starts lengthened the step loop: the 8-D pair of 10^6 samples ran in 896
    // ms instead of 884.)
    const int q_last = (kWindow >> sub_shift) - 1;
    uint32_t ahead_flag = 0;
    bool ahead = false;
    for (int t0 = 0; t0 < T_run; t0 += kSub) {
        const int q = (t0 >> sub_shift) & ((kWindow >> sub_shift) - 1);  // sub-chunk within the window
        const int wb = t0 - q * kSub;                          // window start
        const int steps = T_run - t0 < kSub ? T_run - t0 : kSub;
        const bool flagged = !TILE || s > 0;  // a tile's left column is there from the start
        if (RR && q == 0) {
            // (LDS accesses of one wave complete in order; the fences keep the
            // compiler from moving a row read across these writes)
            const int odd = (t0 / kWave) & 1;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            put(odd ? 2 * kWave : kWave);
            if (odd) put(0);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (t0 + kWave < T_run) fetch(t0 + kWave);
            row_at = rows_lds + ((odd ? 2 * kWave : kWave) - lane) * S;
            load_row<CT, DIMT>(row_at, 0, row[0]);
            if constexpr (kAhead == 2) load_row<CT, DIMT>(row_at, 1, row[1]);
        }
        if (in_global && q == 0) {
            if (ahead) {
                sh.in_stage[lane] = sh.in_next[lane];
            } else {
                if (flagged) {
                    const uint32_t need = (uint32_t)(t0 + kWindow < nA ? t0 + kWindow : nA);
                    wait_progress(in_flag, need, err);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                }
                // rows t0 + 1 .. t0 + 64 of the boundary
                const int rr = t0 + 1 + lane < nA ? t0 + 1 + lane : nA;
                sh.in_stage[lane] = in_slot[rr];
            }
            ahead = false;
        }
        // (the flag's value is taken wave-uniform only where it is used, so
        // the wave does not wait for the load where it is issued)
        if (in_global && flagged && q_last > 0 && q == q_last - 1)
            ahead_flag = __hip_atomic_load(in_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (in_global && q == q_last && wb + kWindow < T_run) {
            const int nb0 = wb + kWindow;  // the next window's start
            const uint32_t need = (uint32_t)(nb0 + kWindow < nA ? nb0 + kWindow : nA);
            if (!flagged || (q_last > 0 && wave_uniform(ahead_flag) >= need)) {
                if (flagged) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                const int rr = nb0 + 1 + lane < nA ? nb0 + 1 + lane : nA;
                sh.in_next[lane] = in_slot[rr];
                ahead = true;
            }
        }
        {
            // the rows this sub-chunk reads, t0 + 1 .. t0 + steps, are in the ring
            const int need = t0 + steps < nA ? t0 + steps : nA;
            if (counted < need) counted = wait_rows(prod_in, need, err);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        if (out_lds) {
            // this sub-chunk writes rows up to t0 + steps - 64 into the ring,
            // over the slots of rows up to 128 earlier: the next wave must
            // have read those
            const int last_w = t0 + steps - kWave;
            if (consumed < last_w - kRing) consumed = wait_rows(&sh.cons[w + 1], last_w - kRing, err);
        }

        // This sub-chunk's first boundary cells: row t0 + 1 in, row t0 - 63 out
        // (rows -63 .. 0 of the first 64 steps land in the slots of rows 65 ..
        // 128, which are written again with those rows, at steps 128 .. 191,
        // before anyone may read them).
        const Pair2<AT> *in_at = in_src + (t0 & in_mask);
        Pair2<AT> *out_at = has_out && lane == kWave - 1 ? out_ring + ring_slot(t0 - (kWave - 1)) : &sh.dummy[lane];
        const int out_step = has_out && lane == kWave - 1 ? 1 : 0;
        // Tiles: which rows of interest do lanes reach in this sub-chunk: row 0
        // (top row), nA (bottom row), a checkpoint row?  Or is this the strip
        // that hands out column nB at every step?
        bool sp_top = false, sp_rows = false, sp_right = false;
        int ck_lo = kNoRow, ck_hi = kNoRow;  // checkpoint rows
        int keep = kNoRow;                   // the row whose cells are kept
        int top_step = kNoRow;               // the step at which this lane is on row 0
        if constexpr (TILE) {
            const int r_lo = t0 - (kWave - 1), r_hi = t0 + steps - 1;  // rows the lanes touch
            sp_top = io.top != nullptr && t0 < kWave;
            if (sp_top) top_step = lane;
            if constexpr (!DIRS) {
                sp_right = io.right != nullptr && result_strip;
                if (io.ckrow != nullptr) {
                    // at most two checkpoint rows (ck_rows >= 64) are among the
                    // at most 95 rows of the range
                    if (ck_next < r_lo) {
                        ck_next += io.ck_rows;
                        ck_row += nB + 1;
                    }
                    if (ck_next <= r_hi && ck_next < nA) ck_lo = ck_next;
                    if (ck_next + io.ck_rows <= r_hi && ck_next + io.ck_rows < nA) ck_hi = ck_next + io.ck_rows;
                }
                const bool last_row = io.bottom != nullptr && nA <= r_hi;
                if (rows_kept) keep = last_row ? nA : ck_lo;
                sp_rows = last_row || ck_lo != kNoRow;
            }
        }
        uint32_t d_lo = 0, d_hi = 0;  // this sub-chunk's moves, the last step in the highest bits
        // One step: sweep row t - lane with `use`, read row t + kAhead - lane into
        // `fill`; OFF is the step's place in its unrolled run.  Steps take turns
        // with the row buffers, so a row read ahead never has to be copied.  SP
        // (tile sweeps): lanes meet a row of interest in this sub-chunk; the
        // other sub-chunks run without testing for them at every step.  Where
        // cells are kept, the step only selects by lane.
        auto step = [&]<bool SP, int OFF>(int i, Row<CT, DIMT> &use, Row<CT, DIMT> &fill, Pair2<AT> &nb,
                                         Pair2<AT> &nb_next) {
            static_assert(OFF < kMaxUnroll, "sh.dummy has room for this many");
            const int t = t0 + i;
            load_row<CT, DIMT>(row_at, OFF + kAhead, fill);
            // boundary row t + kAhead, which lane 0 meets kAhead steps on (nb is
            // row t + 1)
            nb_next = in_at[OFF + kAhead - 1];

            AT left = sh_l, xl;
            if constexpr (TILE) {
                if constexpr (DIRS) {
                    uint32_t code;
                    if constexpr (REC == kRecTwed)
                        code = lane_row_dirs<CT, AT, DIMT, PM>(L, use, left, sh_xo, xl, ca.nu, ca.p, ca.invp);
                    else
                        code = lane_row_sibling<CT, AT, DIMT, PM, K, REC, true>(L, use, left, sh_xo, xl, ca.p, ca.invp);
                    d_lo = __builtin_amdgcn_alignbit(d_hi, d_lo, 2);
                    d_hi = __builtin_amdgcn_alignbit(code == 0 ? 1u : code & 2u, d_hi, 2);
                } else {
                    if constexpr (REC == kRecTwed)
                        lane_row<CT, AT, DIMT, PM, K>(L, use, left, sh_xo, xl, ca.nu, ca.p, ca.invp, beta);
                    else
                        (void)lane_row_sibling<CT, AT, DIMT, PM, K, REC, false>(L, use, left, sh_xo, xl, ca.p,
                                                                                ca.invp);
                }
              if constexpr (SP) {
                // the lane sits on row 0: its top-row cells replace the pad state
                if (kCellsKept || sp_top) {
                    const bool own = t == top_step;
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        Pair2<AT> v;
                        if constexpr (kCellsKept) v = tops[j];
                        else v = io.top[c0 + j <= nB ? c0 + j : nB];
                        L.up[j] = own ? v.dp : L.up[j];
                        L.xp[j] = own ? v.x : L.xp[j];
                    }
                    left = own ? L.up[K - 1] : left;
                    xl = own ? L.xp[K - 1] : xl;
                }
                if constexpr (kCellsKept && !DIRS) {
                    const bool own = t - lane == keep;
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        kept[j].dp = own ? L.up[j] : kept[j].dp;
                        kept[j].x = own ? L.xp[j] : kept[j].x;
                    }
                }
                // (every lane stores; lanes without a cell of the row write the
                // dummy cells)
                auto store_row = [&](int r, Pair2<AT> *row) {
                    if (r <= t && r >= t - (kWave - 1)) {
#pragma unroll
                        for (int j = 0; j < K; ++j) {
                            Pair2<AT> *dst = t - lane == r && c0 + j <= nB ? row + (c0 + j) : io.dummy + lane * K + j;
                            *dst = Pair2<AT>{L.up[j], L.xp[j]};
                        }
                    }
                };
                if (!DIRS && !rows_kept) {
                    if (io.bottom != nullptr) store_row(nA, io.bottom);
                    if (ck_lo != kNoRow) store_row(ck_lo, ck_row);
                    if (ck_hi != kNoRow) store_row(ck_hi, ck_row + (nB + 1));
                }
                // column nB (lane lstar, column jstar of the last strip)
                if (!DIRS && sp_right && t - lstar >= 1 && t - lstar <= nA) {
                    AT dp = L.up[0], x = L.xp[0];
#pragma unroll
                    for (int j = 1; j < K; ++j) {
                        if (j == jstar) {
                            dp = L.up[j];
                            x = L.xp[j];
                        }
                    }
                    io.right[t - lstar] = Pair2<AT>{lane_value(dp, lstar), lane_value(x, lstar)};
                }
              }
            } else {
                lane_row<CT, AT, DIMT, PM, K>(L, use, left, sh_xo, xl, ca.nu, ca.p, ca.invp, beta);
            }

            if constexpr (DUMP) {
                const int r = t - lane;
                if (r >= 1 && r <= nA) {
#pragma unroll
                    for (int j = 0; j < K; ++j)
                        if (c0 + j <= nB)
                            dump[(size_t)r * (size_t)(nB + 1) + (size_t)(c0 + j)] =
                                kShifted<AT> ? (AT)((double)L.up[j] + (double)beta * (double)(r + c0 + j))
                                             : L.up[j];
                }
            }
            sh_xo = sh_x;
            sh_l = shift_in(left, nb.dp);
            sh_x = shift_in(xl, nb.x);
            out_at[OFF] = Pair2<AT>{left, xl};  // (lane 63: row t - 63 of the strip's right boundary)
            // Wide strips fill the SIMD by themselves; steps mixed with their
            // neighbours would only cost registers.
            if constexpr (kRowWords * K > 96 || kTwoSteps) __builtin_amdgcn_sched_barrier(0);
        };
        auto advance = [&](int n) {
            row_at += n * S;
            in_at += n;
            out_at += n * out_step;
        };
        auto run = [&]<bool SP>() {
            int i = 0;
            if constexpr (kAhead == 2) {
                nbs[0] = in_at[0];
                for (; i + kMaxUnroll <= steps; i += kMaxUnroll) {
                    step.template operator()<SP, 0>(i, row[0], row[2], nbs[0], nbs[1]);
                    step.template operator()<SP, 1>(i + 1, row[1], row[3], nbs[1], nbs[0]);
                    step.template operator()<SP, 2>(i + 2, row[2], row[0], nbs[0], nbs[1]);
                    step.template operator()<SP, 3>(i + 3, row[3], row[1], nbs[1], nbs[0]);
                    advance(kMaxUnroll);
                }
                for (; i < steps; ++i) {  // the end of the sweep
                    step.template operator()<SP, 0>(i, row[0], row[2], nbs[0], nbs[1]);
                    row[0] = row[1];
                    row[1] = row[2];
                    nbs[0] = nbs[1];
                    advance(1);
                }
            } else if constexpr (kTwoSteps) {
#pragma unroll 1
                for (; i + 2 <= steps; i += 2) {
                    step.template operator()<SP, 0>(i, row[0], row[1], nbs[0], nbs[0]);
                    step.template operator()<SP, 1>(i + 1, row[1], row[0], nbs[0], nbs[0]);
                    advance(2);
                }
                if (i < steps) {  // the end of the sweep
                    step.template operator()<SP, 0>(i, row[0], row[1], nbs[0], nbs[0]);
                    row[0] = row[1];
                    advance(1);
                }
            } else {
                for (; i + kMaxUnroll <= steps; i += kMaxUnroll) {
                    step.template operator()<SP, 0>(i, row[0], row[1], nbs[0], nbs[0]);
                    step.template operator()<SP, 1>(i + 1, row[1], row[0], nbs[0], nbs[0]);
                    step.template operator()<SP, 2>(i + 2, row[0], row[1], nbs[0], nbs[0]);
                    step.template operator()<SP, 3>(i + 3, row[1], row[0], nbs[0], nbs[0]);
                    advance(kMaxUnroll);
                }
                for (; i < steps; ++i) {  // the end of the sweep
                    step.template operator()<SP, 0>(i, row[0], row[1], nbs[0], nbs[0]);
                    row[0] = row[1];
                    advance(1);
                }
            }
        };
        if constexpr (TILE) {
            if (sp_top || sp_rows || sp_right) run.template operator()<true>();
            else run.template operator()<false>();
        } else {
            run.template operator()<false>();
        }

        const int tend = t0 + steps;        // steps done so far
        const int last = tend - kWave;      // last boundary row complete
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (in_lds) {
            // rows up to tend have been read
            __hip_atomic_store(&sh.cons[w], tend, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __hip_atomic_store(prod_out, tend - kWave, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (out_global && (q == (kWindow >> sub_shift) - 1 || tend >= T)) {
            // the window's rows, tend - 127 + lane for lanes kWave - (tend -
            // wb) .. 63, from out_stage to the slot (lanes without a row of
            // this window write slot row 0, which no consumer reads: no
            // lane-conditional branch)
            const int ws = tend - wb;
            int r = tend - 2 * kWave + 1 + lane;
            r = (lane >= kWave - ws && r >= 1 && r <= nA) ? r : 0;
            out_slot[r] = sh.out_stage[r > 0 ? ring_slot(r) : kRing];
            if (last >= 1) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                __hip_atomic_store(out_flag, (uint32_t)(last < nA ? last : nA), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if constexpr (DIRS)  // (behind the hand-over, which waits for outstanding stores)
            io.dirs[((size_t)s * (size_t)((T + 31) / 32) + (size_t)(t0 / 32)) * kWave + lane] =
                ((uint64_t)d_hi << 32 | d_lo) >> (2 * (32 - steps));
        if constexpr (TILE) {
            if (keep != kNoRow && (tend - 1 >= keep + kWave - 1 || tend >= T_run)) {
                // every lane (with a column of the block) has swept the row
                Pair2<AT> *to = keep == nA ? io.bottom : ck_row;
#pragma unroll
                for (int j = 0; j < (kCellsKept ? K : 0); ++j)
                    *(c0 + j <= nB ? to + (c0 + j) : io.dummy + lane * K + j) = kept[j];
            }
            // a checkpoint column at this strip's right edge, window by window
            if (ck_col != nullptr && (q == (kWindow >> sub_shift) - 1 || tend >= T)) {
                const int ws = tend - wb;
                const int r = tend - 2 * kWave + 1 + lane;
                const bool ok = lane >= kWave - ws && r >= 1 && r <= nA;
                *(ok ? ck_col + r : io.dummy + lane) = out_ring[ok ? ring_slot(r) : kRing];
            }
        }
    }
    if (result_strip) {
        // DP(nA, nB): column jstar of lane lstar after its sweep of row nA
        // (wave-uniform; every lane stores the same value)
        AT res = L.up[0];
#pragma unroll
        for (int j = 1; j < K; ++j)
            if (j == jstar) res = L.up[j];
        res = lane_value(res, lstar);
        if (kShifted<AT>) res = (AT)((double)res + (double)beta * (double)(nA + nB));
        if (load_progress(err) != 0u) res = __builtin_nan("");
        out[0] = res;
    }
}

// Persistent workgroups of G waves.  A workgroup claims a group g of G
// consecutive strips from an atomic ticket (wave 0 claims, LDS broadcasts),
// so the group it waits for has always been claimed by a running workgroup:
// no co-residency assumption, no deadlock.  Inside the group, wave w sweeps
// strip g*G + w: body(w, g, s).
//
// Two global slots suffice: group g+2 writes row r of its boundary only
// after group g+1 has read row r from the slot both use (it reads a row
// before its own last wave can produce that row).
template <int G, typename Shared, typename Body>
__device__ __forceinline__ void claim_groups(Shared &sh, uint32_t *ticket, int nStrips, Body &&body)
{
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int nGroups = (nStrips + G - 1) / G;
    for (;;) {
        __syncthreads();  // the previous group is done with the LDS
        // Every thread takes part in the claim and only thread 0 counts, so
        // there is no branch around the atomic; wave 0's lane-0 value is the
        // group, published through LDS.
        const uint32_t mine = atomicAdd(ticket, threadIdx.x == 0 ? 1u : 0u);
        __hip_atomic_store(&sh.ticket[w], (uint32_t)__builtin_amdgcn_readlane((int)mine, 0), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(&sh.prod[w], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(&sh.prod[G + 1], 0x7fffffff, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(&sh.cons[w], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        const int g = (int)__hip_atomic_load(&sh.ticket[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (g >= nGroups) break;
        const int s = g * G + w;
        if (s < nStrips) body(w, g, s);
    }
}

// Strips of one width: strip s starts at column 1 + s*64*K.
template <typename CT, typename AT, int DIMT, int PM, int K, int G, bool DUMP, bool TILE, int REC = kRecTwed,
          bool DIRS = false>
__global__ __launch_bounds__(kWave * G) void wavefront_kernel(const CT *__restrict__ rowsA,
                                                             const CT *__restrict__ rowsB, int nA, int nB,
                                                             CostArgs<CT> ca, Pair2<AT> *bnd, uint32_t *flags,
                                                             uint32_t *ticket, uint32_t *err, int nStrips,
                                                             const CT *beta_ptr, AT *out, AT *dump, int sub_shift,
                                                             TileIO<AT> io)
{
    __shared__ GroupShared<CT, AT, DIMT, G> sh;
    const CT beta = kShifted<AT> ? beta_ptr[0] : CT(0);
    claim_groups<G>(sh, ticket, nStrips, [&](int w, int g, int s) {
        sweep_strip<CT, AT, DIMT, PM, K, G, DUMP, TILE, REC, DIRS>(sh, w, g, s, s * kWave * K, rowsA, rowsB, nA, nB,
                                                                   ca, bnd, flags, err, nStrips, beta, out, dump,
                                                                   sub_shift, io);
    });
}

// Strips of two widths: strips 0 .. s1-1 hold K columns per lane, the rest
// K2 < K.  A strip starts one pipeline lag (in its own steps) after the one
// before it and runs nA + 63 steps, so with every strip resident the sweep
// ends when the last strip does: narrower strips at the end of the row
// finish sooner, and the spare workgroup slots that uniform strips would
// leave idle take the extra strips.  Cells and their arithmetic do not
// depend on the strip widths.
template <typename CT, typename AT, int DIMT, int PM, int K, int K2, int G>
__global__ __launch_bounds__(kWave * G) void wavefront_mixed_kernel(const CT *__restrict__ rowsA,
                                                                   const CT *__restrict__ rowsB, int nA, int nB,
                                                                   CostArgs<CT> ca, Pair2<AT> *bnd, uint32_t *flags,
                                                                   uint32_t *ticket, uint32_t *err, int nStrips,
                                                                   int s1, const CT *beta_ptr, AT *out,
                                                                   int sub_shift)
{
    static_assert(K2 < K, "the second width is the narrower one");
    __shared__ GroupShared<CT, AT, DIMT, G> sh;
    const CT beta = kShifted<AT> ? beta_ptr[0] : CT(0);
    claim_groups<G>(sh, ticket, nStrips, [&](int w, int g, int s) {
        if (s < s1)
            sweep_strip<CT, AT, DIMT, PM, K, G, false, false, kRecTwed, false>(
                sh, w, g, s, s * kWave * K, rowsA, rowsB, nA, nB, ca, bnd, flags, err, nStrips, beta, out,
                nullptr, sub_shift, TileIO<AT>{});
        else
            sweep_strip<CT, AT, DIMT, PM, K2, G, false, false, kRecTwed, false>(
                sh, w, g, s, s1 * kWave * K + (s - s1) * kWave * K2, rowsA, rowsB, nA, nB, ca, bnd, flags, err,
                nStrips, beta, out, nullptr, sub_shift, TileIO<AT>{});
    });
}

template <typename CT, typename AT, int DIMT, int PM, int K, int G, bool TILE, int REC = kRecTwed,
          bool DIRS = false>
int occupancy_kg()
{
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, wavefront_kernel<CT, AT, DIMT, PM, K, G, false, TILE, REC, DIRS>,
                                                     kWave * G, 0) != hipSuccess)
        return 0;
    return blocks;
}

template <typename CT, typename AT, int DIMT, int PM, int K, int G, bool TILE, int REC = kRecTwed,
          bool DIRS = false>
size_t scratch_kg()
{
    hipFuncAttributes attr{};
    if (hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(wavefront_kernel<CT, AT, DIMT, PM, K, G, false, TILE, REC, DIRS>)) !=
        hipSuccess)
        return (size_t)-1;
    return attr.localSizeBytes;
}

template <typename CT, typename AT, int DIMT, int PM, int K, bool TILE>
int occupancy_k(int G)
{
    switch (G) {
    case 1: return occupancy_kg<CT, AT, DIMT, PM, K, 1, TILE>();
    case 4: return occupancy_kg<CT, AT, DIMT, PM, K, 4, TILE>();
    case 8: return occupancy_kg<CT, AT, DIMT, PM, K, 8, TILE>();
    default: return 0;
    }
}

}  // namespace twed
