// batch.hip -- many TWED pairs in one persistent launch.
//
// The paper's batch mode (section "cuTWED Implementation Remarks") maps
// (series pair, diagonal entry) onto a 2-D grid and fills the whole distance
// matrix; its section "Validation using Real Datasets" notes that the
// symmetric case needs only the upper triangle.  Here each pair is swept by
// one wave with the whole band in registers: one series is spread over the 64
// lanes (K = ceil(n/64) columns per lane, K <= KMAX), the other streams through
// them, and the three live diagonals never leave the register file.  A pair
// alone spreads its shorter series; pairs in a chain the one they share,
// whichever is shorter.  Waves pull pairs from an atomic ticket; in the symmetric
// mode the series are visited longest-first so the expensive pairs start
// first and the cheap ones fill the tail.  Results are bitwise equal to the
// single-pair sweep: both evaluate every cell with the same lane code, and
// the cell arithmetic is symmetric under transposition.
#include "twed_dispatch.h"

#include <math.h>
#include <algorithm>

namespace twed {

int batch_kmax(int dimt)
{
    if (dimt <= 1) return 16;
    if (dimt <= 4) return 8;
    if (dimt <= 8) return 4;
    if (dimt <= 16) return 2;
    return 1;
}

template <int DIMT>
__host__ __device__ constexpr int kmax_of()
{
    return DIMT <= 1 ? 16 : (DIMT <= 4 ? 8 : (DIMT <= 8 ? 4 : (DIMT <= 16 ? 2 : 1)));
}

// Sweeps one pair with one wave; returns DP(nA, nB) in every lane (samples
// too wide for the chained sweep below).  Pairs
// here are short enough that the FP32 offset is zero (the single-pair sweep
// applies one only beyond kOffsetMinLength samples), so the two paths stay
// bitwise equal.
template <typename CT, typename AT, int DIMT, int PM, int K>
__device__ __forceinline__ AT sweep_pair(const CT *__restrict__ rowsA, int nA, const CT *__restrict__ rowsB,
                                         int nB, const CostArgs<CT> &ca)
{
    const int lane = threadIdx.x & (kWave - 1);
    const AT INF = pinf<AT>();
    const int c0 = 1 + lane * K;
    Lane<CT, AT, DIMT, K> L;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        Row<CT, DIMT> b;
        load_row<CT, DIMT>(rowsB, c0 + j <= nB ? c0 + j : nB, b);
#pragma unroll
        for (int k = 0; k < DIMT; ++k) L.bx[j][k] = b.x[k];
        L.bt[j] = b.t;
        L.bdel[j] = (AT)b.del;
        L.up[j] = INF;
        L.xp[j] = INF;
    }
    const int q = nB - 1;
    const int lstar = q / K, jstar = q - (q / K) * K;

    AT sh_l = INF;
    AT sh_x = lane == 0 ? -AT(0) : INF;  // X(0,0) = -beta with beta = 0
    AT sh_xo = INF;
    // Lane l reads row t - l at step t with no clamping: before row 0 and
    // past row nA it reads a neighbouring series or the 64 zero rows that pad
    // every packed buffer (rows -63 .. nA + 64 are touched).  Those rows only
    // meet +inf operands (before row 0) or feed no result (past row nA).
    // For wide samples, lanes whose columns all lie past nB (they feed no
    // result: values only flow to higher lanes) read lane 0's row, which the
    // wave's load then serves once instead of fetching rows nobody needs.
    const int row_lane = (DIMT < 8 || c0 <= nB) ? lane : 0;
    const CT *pa = rowsA - (ptrdiff_t)row_lane * Row<CT, DIMT>::kStride;
    Row<CT, DIMT> ra, rb;
    load_row<CT, DIMT>(pa, 0, ra);
    auto step = [&](const Row<CT, DIMT> &row) {
        AT left = sh_l, xl;
        lane_row<CT, AT, DIMT, PM, K>(L, row, left, sh_xo, xl, ca.nu, ca.p, ca.invp, CT(0));
        sh_xo = sh_x;
        sh_l = shift_in(left, INF);
        sh_x = shift_in(xl, INF);
    };
    const int T = nA + lstar + 1;  // last step: lane lstar finishes row nA
    int t = 0;
    // two steps per iteration: the band registers alternate without copies
    for (; t + 2 <= T; t += 2) {
        load_row<CT, DIMT>(pa, t + 1, rb);
        step(ra);
        load_row<CT, DIMT>(pa, t + 2, ra);
        step(rb);
    }
    if (t < T) step(ra);
    AT res = L.up[0];
#pragma unroll
    for (int j = 1; j < K; ++j)
        if (j == jstar) res = L.up[j];
    return lane_value(res, lstar);
}

template <typename CT, typename AT, int DIMT, int PM, int K, int KHI>
__device__ __forceinline__ AT sweep_dispatch(int k, const CT *rowsA, int nA, const CT *rowsB, int nB,
                                             const CostArgs<CT> &ca)
{
    if constexpr (K > kmax_of<DIMT>() || K > KHI) {
        return AT(0);
    } else {
        if (k == K) return sweep_pair<CT, AT, DIMT, PM, K>(rowsA, nA, rowsB, nB, ca);
        return sweep_dispatch<CT, AT, DIMT, PM, K + 1, KHI>(k, rowsA, nA, rowsB, nB, ca);
    }
}

// Items item0 .. nItems-1; pairs of KLO..KHI columns per lane (clipped to
// what the sample width allows) are swept, the others left to other launches.
template <typename CT, typename AT, int DIMT, int PM, int KLO, int KHI>
__global__ __launch_bounds__(64) void batch_kernel(const CT *__restrict__ rowsX, const CT *__restrict__ rowsY,
                                                   const int64_t *__restrict__ offX,
                                                   const int64_t *__restrict__ offY,
                                                   const int32_t *__restrict__ order,
                                                   const int64_t *__restrict__ pairs, int64_t nX, int64_t nY,
                                                   int64_t item0, int64_t nItems, int mode, CostArgs<CT> ca, AT *D,
                                                   uint32_t *ticket, int chunk)
{
    constexpr int S = Row<CT, DIMT>::kStride;
    constexpr int KMAX = kmax_of<DIMT>() < KHI ? kmax_of<DIMT>() : KHI;
    // A ticket is `chunk` consecutive items: for short pairs one atomic per
    // pair on a single counter would cost more than the pair itself.
    for (;;) {
        const int64_t first = item0 + (int64_t)next_ticket(ticket) * chunk;
        if (first >= nItems) break;
        const int64_t last = first + chunk < nItems ? first + chunk : nItems;
        for (int64_t item = first; item < last; ++item) {
            int64_t a, b;
            if (mode == kSymmetric) {
                // item -> (i < j) over the length-sorted order: j-th group holds
                // the pairs (0..j-1, j).
                int64_t j = (int64_t)((1.0 + sqrt(1.0 + 8.0 * (double)item)) * 0.5);
                while (j * (j - 1) / 2 > item) --j;
                while ((j + 1) * j / 2 <= item) ++j;
                const int64_t i = item - j * (j - 1) / 2;
                a = order[i];
                b = order[j];
            } else if (mode == kRect) {
                a = item / nY;
                b = item - a * nY;
            } else {
                a = pairs[2 * item];
                b = pairs[2 * item + 1];
            }
            // a pair-list entry outside the collections yields NaN
            const bool ok = a >= 0 && a < nX && b >= 0 && b < nY;
            if (!ok) {  // uniform: one item per wave
                D[item] = (AT)__builtin_nan("");
                continue;
            }
            const int64_t xa = offX[a], la = offX[a + 1] - xa;
            const int64_t yb = offY[b], lb = offY[b + 1] - yb;
            const CT *ra = rowsX + (xa + a) * S;
            const CT *rb = rowsY + (yb + b) * S;
            // shorter operand across the lanes
            const bool swap = lb > la;
            const CT *rowsA = swap ? rb : ra;
            const CT *rowsB = swap ? ra : rb;
            const int nA = (int)(swap ? lb : la);
            const int nB = (int)(swap ? la : lb);
            const int k = (nB + kWave - 1) / kWave;
            // Pairs wider than one wave are swept by the single-pair path instead.
            if (k >= KLO && k <= KMAX) {
                // d is the same in every lane; every lane stores it (one
                // transaction), so the loop body holds no lane-conditional branch.
                const AT d = sweep_dispatch<CT, AT, DIMT, PM, KLO, KMAX>(k, rowsA, nA, rowsB, nB, ca);
                if (mode == kSymmetric) {
                    D[a * nX + b] = d;
                    D[b * nX + a] = d;
                } else {
                    D[item] = d;
                }
            }
        }
    }
}

// ---- chained sweep ---------------------------------------------------------------
//
// A wave sweeps a chain of pairs that share one series: the shared series'
// columns stay in the lanes' registers and the rows of the other series run
// through them back to back, each preceded by its pad row.  Swept one pair at
// a time, every pair fills and drains a 64-lane pipeline (64 steps beside the
// 60 .. 700 of its rows) and reloads the columns; in a chain only the first
// pair fills it and only the last drains it.
//
// The pad row of a streamed series carries x[0] = del = +inf: a lane that
// sweeps it leaves +inf (or NaN, which a minimum ignores just the same) in
// every cell of its columns, i.e. the pad row of the next pair, whatever the
// previous pair left there.  Only lane 0 needs more: X(0, 0) = 0 enters its
// up-left operand one step before it meets row 1.
//
// Rows come from a ring in LDS: every 64 steps each lane loads one row of the
// stream (the series of a chain may lie anywhere) and writes it to the ring,
// and at step t lane l reads row t - l.  The ring holds 64-row chunks c - 1
// and c, always contiguous: chunk c even at rows 64 .. 127, odd at rows
// 128 .. 191 and again at 0 .. 63, so a step needs no address wrap.  A row
// read is one LDS access per 16 bytes instead of a global one (1-D FP64: 32
// bytes by 64 lanes, 32 cycles of the L1 per step).
//
// Every cell is evaluated with the arithmetic of the single-pair sweep, in
// which the two series have symmetric roles, so the results are bitwise equal
// to it whichever series is shared.
//
// Rows of up to 48 bytes (the ring then fits 16 waves per compute unit) are
// chained; wider samples, whose cells cost enough to hide a pair's fill, are
// swept one pair at a time (batch_kernel).
constexpr int kChainRowBytes = 48;
template <typename CT, int DIMT>
constexpr bool kChained = Row<CT, DIMT>::kStride * (int)sizeof(CT) <= kChainRowBytes;

constexpr int kChainMax = kWave;  // pairs per chain: a lane describes each

template <typename CT, int DIMT>
struct ChainShared {
    alignas(16) CT ring[(3 * kWave + 1) * Row<CT, DIMT>::kStride];
    int64_t base[kChainMax];     // row index of each series' row 0
    int start[kChainMax + 1];    // its place in the stream; the stream's length
};

__device__ __forceinline__ int64_t lane_value64(int64_t v, int lane)
{
    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane) << 32) |
                     (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, lane));
}

// Whether the chain's steps are held apart so that each row read stays a whole
// step ahead of its use.  1-D samples: left to itself the compiler reads the rows
// of two steps at the end of the first, and the wave waits out the LDS latency
// once in two steps (all pairs of 400 series: FP64 of 57 samples 320 us, now 260;
// FP32 of 569 4.57 ms, now 4.03, of 1,017 12.2, now 11.4).  Not in FP64 above six
// columns, where kStepsAligned does it for less, nor at 10 and 11 FP32 columns,
// which lose 2 .. 6% (of 633 4.73 ms without, 5.00 with) though their loops are
// the others' instructions in the others' order.  Wider samples lose (20,000 pairs
// of 310 4-D FP32 samples 955 us without, 1,049 with).
template <typename CT, typename AT, int DIMT, int K>
constexpr bool kReadsPinned = DIMT == 1 && (sizeof(CT) == 8   ? K <= 6
                                            : sizeof(AT) == 4 ? K != 10 && K != 11
                                                              : true);

// Whether a step begins at an even word of the code.  FP64 steps are runs of
// 8-byte instructions, and one that begins at an odd word takes 15 .. 19% longer:
// where a loop falls is the accident of the code before it (all pairs of 400 1-D
// series, ms, odd and even: of 761 samples 16.3 and 13.6, of 1,017 28.0 and 22.8;
// of 633 11.9 and 9.7).  The operands put the directive before the step's first
// instruction and the next row's read behind it, a step ahead.
template <typename CT, int DIMT, int K>
constexpr bool kStepsAligned = DIMT == 1 && sizeof(CT) == 8 && K > 6;

// Sweeps the chain described by sh.start and sh.base (E series of `rows`)
// against the nB columns of rowsB.  Lane e gets DP(nA_e, nB) of series e.
template <typename CT, typename AT, int DIMT, int PM, int K>
__device__ __forceinline__ AT sweep_chain(ChainShared<CT, DIMT> &sh, const CT *__restrict__ rows, int E,
                                          const CT *__restrict__ rowsB, int nB, const CostArgs<CT> &ca)
{
    constexpr int S = Row<CT, DIMT>::kStride;
    constexpr int V = 16 / (int)sizeof(CT);
    constexpr int kNever = 0x7fffffff;
    const int lane = threadIdx.x & (kWave - 1);
    const AT INF = pinf<AT>();
    const int c0 = 1 + lane * K;
    Lane<CT, AT, DIMT, K> L;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        Row<CT, DIMT> b;
        load_row<CT, DIMT>(rowsB, c0 + j <= nB ? c0 + j : nB, b);
#pragma unroll
        for (int k = 0; k < DIMT; ++k) L.bx[j][k] = b.x[k];
        L.bt[j] = b.t;
        L.bdel[j] = (AT)b.del;
        L.up[j] = INF;
        L.xp[j] = INF;
    }
    const int q = nB - 1;
    const int lstar = q / K, jstar = q - (q / K) * K;
    const int total = __builtin_amdgcn_readfirstlane(sh.start[E]);
    const int T = total + lstar;  // the last series' row nA leaves lane lstar at step T - 1

    // this lane's row of the next chunk: stream row g = 64 c + lane
    typedef CT vec __attribute__((ext_vector_type(V)));
    vec fetched[S / V];
    int fe = 0;  // the series that holds stream row g
    uint32_t g = lane;
    const int64_t base0 = lane_value64(sh.base[0], 0);
    auto fetch = [&]() {
        const int gg = g < (uint32_t)total ? (int)g : total - 1;
        int r = gg;
        int64_t base = base0;
        // (a pair alone needs no search; its table reads would be waited for every 64
        // steps, which a cell of more components hides)
        if (DIMT > 1 || E > 1) {
            for (;;) {
                const bool past = gg >= sh.start[fe + 1];
                fe += past ? 1 : 0;
                if (__ballot(past) == 0) break;
            }
            r = gg - sh.start[fe];
            base = sh.base[fe];
        }
        const vec *p = reinterpret_cast<const vec *>(rows + (base + r) * S);
#pragma unroll
        for (int v = 0; v < S / V; ++v) fetched[v] = p[v];
        if (r == 0) {  // the pad row
            fetched[0][0] = pinf<CT>();
            fetched[(DIMT + 1) / V][(DIMT + 1) % V] = pinf<CT>();
        }
        g += kWave;
    };
    auto put = [&](int slot) {
        vec *p = reinterpret_cast<vec *>(sh.ring + (slot + lane) * S);
#pragma unroll
        for (int v = 0; v < S / V; ++v) p[v] = fetched[v];
    };

    // Lane 0 receives no lane's value: its shifted-in operands are +inf (the
    // pad column) and stay so, because each shift writes over an operand that
    // is already used up and whose lane 0 it leaves alone (no register is set
    // to +inf per step: 4 of 16 overhead instructions of a step pair).
    AT sh_l = INF, sh_x = INF, sh_xo = INF;
    auto step = [&](const Row<CT, DIMT> &row) {
        AT left = sh_l, xl;
        lane_row<CT, AT, DIMT, PM, K>(L, row, left, sh_xo, xl, ca.nu, ca.p, ca.invp, CT(0));
        const AT x = shift_in(xl, sh_xo);
        sh_xo = sh_x;
        sh_x = x;
        sh_l = shift_in(left, sh_l);
    };

    AT res = INF;
    int e_in = 0, e_out = 0;
    auto start_of = [&](int e) { return __builtin_amdgcn_readfirstlane(sh.start[e]); };
    // Steps after which lane 0's up-left operand becomes X(0, 0) = 0 (it has
    // swept the pad row of pair e_in and meets row 1 next) or, one step later,
    // its stale copy +inf again; and the step after which lane lstar holds the
    // result of pair e_out.
    int t_in = 0, t_out = start_of(1) - 1 + lstar;
    bool stale = false;
    fetch();
    int t = 0;
    Row<CT, DIMT> ra, rb;
    for (int c = 0;; ++c) {
        const int odd = c & 1;
        // (LDS accesses of one wave complete in order; the fences keep the
        // compiler from moving a row read across these writes)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        put(odd ? 2 * kWave : kWave);
        if (odd) put(0);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if ((c + 1) * kWave < T) fetch();
        const CT *pr = sh.ring + ((odd ? 2 * kWave : kWave) - lane) * S;  // row 64 c - lane
        load_row<CT, DIMT>(pr, 0, ra);
        const int stop = T < (c + 1) * kWave ? T : (c + 1) * kWave;
        while (t < stop) {
            const int ev = t_in < t_out ? t_in : t_out;
            const int lim = ev < stop ? ev + 1 : stop;
            // two steps per iteration: the band registers alternate without copies
            auto ahead = [] {
                if constexpr (kReadsPinned<CT, AT, DIMT, K>) __builtin_amdgcn_sched_barrier(0);
            };
            for (; t + 2 <= lim; t += 2) {
                if constexpr (kStepsAligned<CT, DIMT, K>)
                    asm volatile(".p2align 3" : "+v"(ra.x[0]), "+v"(ra.t), "+v"(ra.del));
                load_row<CT, DIMT>(pr, 1, rb);
                ahead();
                step(ra);
                load_row<CT, DIMT>(pr, 2, ra);
                ahead();
                step(rb);
                pr += 2 * S;
            }
            if (t < lim) {
                load_row<CT, DIMT>(pr, 1, rb);
                step(ra);
                ra = rb;
                pr += S;
                ++t;
            }
            if (t - 1 == t_in) {
                if (!stale) {
                    sh_xo = lane == 0 ? AT(0) : sh_xo;
                    ++t_in;
                } else {
                    sh_x = lane == 0 ? INF : sh_x;
                    ++e_in;
                    t_in = e_in < E ? start_of(e_in) : kNever;
                }
                stale = !stale;
            }
            if (t - 1 == t_out) {
                AT r = L.up[0];
#pragma unroll
                for (int j = 1; j < K; ++j)
                    if (j == jstar) r = L.up[j];
                r = lane_value(r, lstar);
                res = lane == e_out ? r : res;
                ++e_out;
                t_out = e_out < E ? start_of(e_out + 1) - 1 + lstar : kNever;
            }
        }
        if (t >= T) break;
    }
    return res;
}

template <typename CT, typename AT, int DIMT, int PM, int K, int KHI>
__device__ __forceinline__ AT chain_dispatch(int k, ChainShared<CT, DIMT> &sh, const CT *rows, int E,
                                             const CT *rowsB, int nB, const CostArgs<CT> &ca)
{
    if constexpr (K > kmax_of<DIMT>() || K > KHI) {
        return AT(0);
    } else {
        if (k == K) return sweep_chain<CT, AT, DIMT, PM, K>(sh, rows, E, rowsB, nB, ca);
        return chain_dispatch<CT, AT, DIMT, PM, K + 1, KHI>(k, sh, rows, E, rowsB, nB, ca);
    }
}

// Waves per SIMD a chain kernel is held to (the registers the compiler may use).
template <typename CT, typename AT, int DIMT, int KHI>
constexpr int chain_waves()
{
    if (KHI > kBatchNarrowMax) return sizeof(AT) == 4 ? 2 : 1;
    if (KHI > kBatchSlimMax) return sizeof(AT) == 4 ? (DIMT == 1 ? 4 : 3) : (DIMT == 1 ? 3 : 2);
    return sizeof(AT) == 4 ? (DIMT == 1 ? 7 : 5) : (DIMT == 1 ? 4 : 3);
}

// Items item0 .. nItems-1 as batch_kernel takes them, in chains: a ticket of
// `chunk` consecutive items is cut into runs that share a series (symmetric:
// the shorter one, order[j]; rectangular: X_a, or Y_b when y_fixed, whose
// items then run b-major; pair list: whichever of the first item's two series
// the longer run of equal indices has).  A pair alone, or one whose shared
// series is too long for the lanes, takes its shorter series as columns.
template <typename CT, typename AT, int DIMT, int PM, int KLO, int KHI>
__global__ __launch_bounds__(64, (chain_waves<CT, AT, DIMT, KHI>())) void batch_chain_kernel(const CT *__restrict__ rowsX, const CT *__restrict__ rowsY,
                                                         const int64_t *__restrict__ offX,
                                                         const int64_t *__restrict__ offY,
                                                         const int32_t *__restrict__ order,
                                                         const int64_t *__restrict__ pairs, int64_t nX, int64_t nY,
                                                         int64_t item0, int64_t nItems, int mode, CostArgs<CT> ca,
                                                         AT *D, uint32_t *ticket, int chunk, int y_fixed)
{
    constexpr int S = Row<CT, DIMT>::kStride;
    constexpr int KMAX = kmax_of<DIMT>() < KHI ? kmax_of<DIMT>() : KHI;
    __shared__ ChainShared<CT, DIMT> sh;
    const int lane = threadIdx.x;
    // lanes that have not reached row 0 yet sweep these rows (values unused)
    for (int k = lane; k < 2 * kWave * S; k += kWave) sh.ring[k] = CT(0);
    for (;;) {
        const int64_t first = item0 + (int64_t)next_ticket(ticket) * chunk;
        if (first >= nItems) break;
        const int64_t last = first + chunk < nItems ? first + chunk : nItems;
        for (int64_t item = first; item < last;) {
            // lane e's pair (lanes past the run repeat item's and are dropped)
            int run = last - item < kChainMax ? (int)(last - item) : kChainMax;
            int64_t a, b;
            int64_t f = 0, s0 = 0;  // shared and first streamed index (symmetric, rectangular)
            bool fix_x;             // the shared series is X_a
            if (mode == kSymmetric) {
                int64_t j = (int64_t)((1.0 + sqrt(1.0 + 8.0 * (double)item)) * 0.5);
                while (j * (j - 1) / 2 > item) --j;
                while ((j + 1) * j / 2 <= item) ++j;
                s0 = item - j * (j - 1) / 2;
                run = j - s0 < run ? (int)(j - s0) : run;
                a = order[s0 + (lane < run ? lane : 0)];
                b = f = order[j];
                fix_x = false;
            } else if (mode == kRect) {
                const int64_t nF = y_fixed ? nX : nY;  // streamed series
                f = item / nF;
                s0 = item - f * nF;
                run = nF - s0 < run ? (int)(nF - s0) : run;
                const int64_t s = s0 + (lane < run ? lane : 0);
                a = y_fixed ? s : f;
                b = y_fixed ? f : s;
                fix_x = !y_fixed;
            } else {
                const int64_t at = item + (lane < run ? lane : 0);
                a = pairs[2 * at];
                b = pairs[2 * at + 1];
                const bool ok = a >= 0 && a < nX && b >= 0 && b < nY;
                const uint64_t in = run < kChainMax ? (1ull << run) - 1 : ~0ull;
                const uint64_t good = __ballot(ok) & in;
                if (!(good & 1)) {  // an entry outside the collections yields NaN
                    D[item] = (AT)__builtin_nan("");
                    ++item;
                    continue;
                }
                const uint64_t same_a = __ballot(a == lane_value64(a, 0)) & good;
                const uint64_t same_b = __ballot(b == lane_value64(b, 0)) & good;
                const int run_a = same_a == ~0ull ? kChainMax : __builtin_ctzll(~same_a);
                const int run_b = same_b == ~0ull ? kChainMax : __builtin_ctzll(~same_b);
                fix_x = run_a >= run_b;
                run = fix_x ? run_a : run_b;
                if (lane >= run) {  // (their own entries may lie outside the collections)
                    a = 0;
                    b = 0;
                }
            }
            const int64_t xa = offX[a], la = offX[a + 1] - xa;
            const int64_t yb = offY[b], lb = offY[b + 1] - yb;
            const int64_t la0 = lane_value64(la, 0), lb0 = lane_value64(lb, 0);
            int64_t nF = fix_x ? la0 : lb0;
            if (run == 1 || nF > (int64_t)KMAX * kWave) {
                run = 1;
                fix_x = lb0 > la0;
                nF = fix_x ? la0 : lb0;
            }
            const int64_t k64 = (nF + kWave - 1) / kWave;
            if (k64 < KLO || k64 > KMAX) {  // left to another launch
                ++item;
                continue;
            }
            // The stream: each series behind its pad row.  A pair alone needs no sum
            // over the lanes.  Pair lists whose neighbours share nothing, 1-D FP32 in
            // 128 .. 512 samples: 2,048 pairs 135 us with the sum and the table reads,
            // now 127 (swept from global rows without a ring 131; 50,000 FP64 pairs in
            // 20 .. 100 samples 341, 268 and 410 us).
            const int64_t nS = fix_x ? lb : la;
            int64_t end = lane < run ? nS + 1 : 0;
            if (run > 1) {
#pragma unroll
                for (int d = 1; d < kWave; d <<= 1) {
                    const int64_t o = __shfl_up((long long)end, d, kWave);
                    end += lane >= d ? o : 0;
                }
                // (at most 2^30 rows in a chain of several)
                const uint64_t fits = __ballot(end <= (int64_t(1) << 30));
                const int most = fits == ~0ull ? kChainMax : __builtin_ctzll(~fits);
                run = most < run ? (most > 1 ? most : 1) : run;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            sh.start[0] = 0;
            sh.start[lane + 1] = (int)end;  // (entries past the run are not read)
            sh.base[lane] = fix_x ? yb + b : xa + a;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const int64_t fr = fix_x ? lane_value64(xa + a, 0) : lane_value64(yb + b, 0);
            const AT d = chain_dispatch<CT, AT, DIMT, PM, KLO, KMAX>((int)k64, sh, fix_x ? rowsY : rowsX, run,
                                                                    (fix_x ? rowsX : rowsY) + fr * S, (int)nF, ca);
            // Lanes past the run store lane 0's result again (no lane-conditional
            // branch at the loop's end).  Where each result goes is worked out
            // again here: holding it through the sweep costs registers.
            const int e = lane < run ? lane : 0;
            const AT v = lane < run ? d : lane_value(d, 0);
            if (mode == kSymmetric) {
                const int64_t s = order[s0 + e];
                D[s * nX + f] = v;
                D[f * nX + s] = v;
            } else if (mode == kRect) {
                D[y_fixed ? (s0 + e) * nY + f : f * nY + s0 + e] = v;
            } else {
                D[item + e] = v;
            }
            item += run;
        }
    }
}

// Calls f<KLO, KHI>() with the widths of a class, as far as the sample width
// allows them (a class that reaches beyond KMAX stops there).
template <typename CT, typename AT, int DIMT, int PM, typename F>
static auto by_class(int cls, F &&f)
{
    constexpr int KM = kmax_of<DIMT>();
    if constexpr (KM > kBatchSlimMax) {
        if (cls == kBatchSlim) return f.template operator()<1, kBatchSlimMax>();
        if (cls == kBatchMid) return f.template operator()<kBatchSlimMax + 1, kBatchNarrowMax>();
    }
    if constexpr (KM > kBatchNarrowMax) {
        if (cls == kBatchNarrow) return f.template operator()<1, kBatchNarrowMax>();
        if (cls == kBatchWide) return f.template operator()<kBatchNarrowMax + 1, KM>();
    }
    return f.template operator()<1, KM>();
}

template <typename CT, typename AT, int DIMT, int PM>
static int batch_occupancy(int cls)
{
    return by_class<CT, AT, DIMT, PM>(cls, [&]<int KLO, int KHI>() -> int {
        int blocks = 0;
        hipError_t e;
        if constexpr (kChained<CT, DIMT>)
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, batch_chain_kernel<CT, AT, DIMT, PM, KLO, KHI>,
                                                             kWave, 0);
        else
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, batch_kernel<CT, AT, DIMT, PM, KLO, KHI>, kWave,
                                                             0);
        return e == hipSuccess ? blocks : 0;
    });
}

int batch_default_chunk(Prec prec, int dimt, double mean_x, double mean_y, bool y_fixed, int64_t items, int workers)
{
    int64_t chunk;
    if (row_stride(prec, dimt) * (int)cost_size(prec) <= kChainRowBytes) {
        // A chain of E series of r rows costs about 64 steps beside its E r
        // (its fill), and at the end of the launch the waves wait for the last
        // tickets, a share of about 2 E w / (3 items): the sum is least near
        // E = sqrt(100 items / (r w)).  Measured: 1-D FP32, 2,048 series of
        // 64 .. 1,024, 107 ms at E = 1, 101 at 4 .. 6, 110 at 32; 1-D FP64,
        // 500 series of 100 .. 500, 4.02 ms at 1, 3.71 at 4, 5.19 at 32.
        const double rows = (y_fixed ? mean_x : mean_y) + 1.0;
        const double best = sqrt(100.0 * (double)items / (rows * (double)workers));
        chunk = std::max<int64_t>(1, std::min<int64_t>(kChainMax, (int64_t)(best + 0.5)));
    } else {
        // about 64k cells of work per ticket for short pairs, while leaving
        // at least four tickets per wave
        const double cells = mean_x * mean_y;
        chunk = std::max<int64_t>(1, std::min<int64_t>(32, (int64_t)(65536.0 / std::max(cells, 1.0))));
        chunk = std::min<int64_t>(chunk, std::max<int64_t>(1, items / (4 * (int64_t)workers)));
    }
    return (int)chunk;
}

hipError_t launch_batch(Prec prec, const CostParams &cp, const BatchArgs &a, hipStream_t st)
{
    return by_prec(prec, cp.dimt, cp.pm, [&]<typename CT, typename AT, int DIMT, int PM>() -> hipError_t {
        return by_class<CT, AT, DIMT, PM>(a.kclass, [&]<int KLO, int KHI>() -> hipError_t {
            if constexpr (kChained<CT, DIMT>)
                hipLaunchKernelGGL((batch_chain_kernel<CT, AT, DIMT, PM, KLO, KHI>), dim3(a.grid), dim3(kWave), 0, st,
                                   (const CT *)a.rowsX, (const CT *)a.rowsY, a.offX, a.offY, a.order, a.pairs, a.nX,
                                   a.nY, a.item0, a.nItems, a.mode, CostArgs<CT>::make(cp), (AT *)a.D, a.ticket,
                                   a.chunk > 1 ? a.chunk : 1, a.y_fixed);
            else
                hipLaunchKernelGGL((batch_kernel<CT, AT, DIMT, PM, KLO, KHI>), dim3(a.grid), dim3(kWave), 0, st,
                                   (const CT *)a.rowsX, (const CT *)a.rowsY, a.offX, a.offY, a.order, a.pairs, a.nX,
                                   a.nY, a.item0, a.nItems, a.mode, CostArgs<CT>::make(cp), (AT *)a.D, a.ticket,
                                   a.chunk > 1 ? a.chunk : 1);
            return hipGetLastError();
        });
    });
}

int batch_max_workers(Prec prec, const CostParams &cp, int kclass)
{
    int per_cu = 0;
    hipError_t e = by_prec(prec, cp.dimt, cp.pm, [&]<typename CT, typename AT, int DIMT, int PM>() -> hipError_t {
        per_cu = batch_occupancy<CT, AT, DIMT, PM>(kclass);
        return hipSuccess;
    });
    if (e != hipSuccess || per_cu <= 0) return 0;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return per_cu * cus;
}

template <typename AT>
__global__ void diag_zero_kernel(AT *D, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        D[i * n + i] = AT(0);
}

template <typename AT>
__global__ void copy_one_kernel(const AT *src, AT *dst)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) dst[0] = src[0];
}

hipError_t launch_batch_diag_zero(Prec prec, void *D, int64_t n, hipStream_t st)
{
    const int grid = (int)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
    if (prec == kF32)
        hipLaunchKernelGGL(diag_zero_kernel<float>, dim3(grid), dim3(256), 0, st, (float *)D, n);
    else
        hipLaunchKernelGGL(diag_zero_kernel<double>, dim3(grid), dim3(256), 0, st, (double *)D, n);
    return hipGetLastError();
}

hipError_t launch_copy_one(Prec prec, const void *src, void *dst, hipStream_t st)
{
    if (prec == kF32)
        hipLaunchKernelGGL(copy_one_kernel<float>, dim3(1), dim3(64), 0, st, (const float *)src, (float *)dst);
    else
        hipLaunchKernelGGL(copy_one_kernel<double>, dim3(1), dim3(64), 0, st, (const double *)src, (double *)dst);
    return hipGetLastError();
}

}  // namespace twed
