// query.hip -- one short query against many series.
//
// A workgroup of four waves sweeps 64 pairs, one per lane, column by column (a
// sample of every lane's series at a time). Wave w owns the query's rows w R +
// 1 .. (w + 1) R: their DP column is in its registers, and it computes the
// point costs of all its rows for a column before the row above them is due.
// The recurrence itself needs the previous wave's last row of the same column,
// so wave w runs it w columns later, on point costs kept in registers, and
// hands (DP, X) of its last row on through LDS, two barriers per column.
//
// Every cell is evaluated with the arithmetic of lane_row (transposed, which
// changes nothing: the point and time terms are symmetric and the minimum is
// exact), so results are bitwise those of the wave-per-pair sweep and of
// twed_pair. That sweep spends most of its lanes and steps filling and draining
// a 64-lane pipeline for a few hundred cells.
//
// Bound: FP64 issue (28-D L2: 77 instructions per cell). One wave per 64 pairs,
// as before, left SIMDs idle (938 waves for 60,000 series) and read the query's
// row from LDS for every cell: 15 16-byte reads of 64 lanes, twice the LDS time
// the cell's arithmetic takes. Here the query's components are scalar operands,
// the same for every lane, loaded four rows ahead, and the lanes' samples are
// read from LDS once for all rows of the wave. The samples are staged by the
// whole workgroup, consecutive threads reading consecutive bytes, one column
// ahead of their use. 28 samples in R^28 against 60,000 series of 28, FP64: 377
// -> 231 us a call; of 20 .. 36 samples, FP64 441 -> 285, FP32 343 -> 151; against
// 2,000 series of 28 FP32 249 -> 83. Held to 128 registers (seven rows a wave),
// four workgroups, four waves per SIMD, share a compute unit and all 938 run at
// once: a tenth faster than at 132 registers; eight rows do not fit and run three
// to a unit. Ten rows a wave in three waves (fewer scalar loads) took a tenth
// longer.
//
// RAW: the series are read as the caller holds them (Y: dim components per
// sample, TY: timestamps) instead of as staged rows, and each sample's deletion
// cost is computed (by wave 0, which passes it on) from the sample before it
// with the staging kernel's arithmetic, so a collection queried once needs no
// staging pass.
#include "twed_dispatch.h"

namespace twed {

constexpr int kQueryWaves = 4;

template <typename AT>
struct QueryHandOff {
    AT dp[kWave], x[kWave];
};

// Elements between the staged samples of two lanes: the components, the
// timestamp and (staged rows) the deletion cost, padded to an odd number of
// 16-byte units, so that eight lanes' reads of one unit cover all LDS banks.
inline int query_pitch(int dim, int dimt, int elem, bool raw)
{
    const int v = 16 / elem;
    const int units = raw ? (dim + 1 + v - 1) / v : (dimt + 2 + v - 1) / v;
    return (units | 1) * v;
}

// RM: rows a wave owns (the last wave that has rows maybe fewer).
template <typename CT, typename AT, int DIMT, int PM, bool RAW, int RM>
__global__ __launch_bounds__(kWave *kQueryWaves, RM <= 7 ? 4 : 3) void batch_query_kernel(
    const CT *__restrict__ rowsQ, int nQ, const CT *__restrict__ rowsY, const CT *__restrict__ Yraw,
    const CT *__restrict__ TYraw, int dim, int pitch, int wide, const int64_t *__restrict__ offY, int64_t nY, CostArgs<CT> ca,
    AT *D)
{
    constexpr int W = kQueryWaves;
    constexpr int S = Row<CT, DIMT>::kStride;
    constexpr int V = 16 / (int)sizeof(CT);               // elements per 16-byte unit
    constexpr int NB = (DIMT + V - 1) / V;                // units that hold components
    constexpr int NU = RAW ? NB : S / V;                  // units staged per sample
    constexpr int kLoads = (NU + W - 1) / W;              // units a thread stages per column
    static_assert(RM <= kRowPad, "rows before the query's first are read (and not used)");
    typedef CT vec __attribute__((ext_vector_type(V)));
    typedef const CT __attribute__((address_space(4))) *Scalars;
    extern __shared__ __align__(16) char query_lds[];
    CT *const stage = reinterpret_cast<CT *>(query_lds);  // two columns of 64 samples
    // The hand-over has two buffers in turn, or one, read behind the step's second
    // barrier, for FP64 samples of more than 16 components: four workgroups then
    // fit the LDS of a compute unit at every dimension (40,960 bytes each at 32).
    // With two buffers three did, from 30 components on (staged rows: from 17 on),
    // and 938 workgroups ran as 768 and 170.
    constexpr int kHands = sizeof(CT) == 8 && DIMT > 16 ? 1 : 2;
    __shared__ QueryHandOff<AT> hand[W - 1][kHands];
    __shared__ CT dels[4][kWave];  // deletion costs of the last four columns
    __shared__ int64_t place[2][kWave];  // element of every lane's sample in Y (or rowsY)
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const Scalars q = (Scalars)(uintptr_t)rowsQ;
    const AT INF = pinf<AT>();

    const int64_t item = (int64_t)blockIdx.x * kWave + lane;
    const bool ok = item < nY;
    const int64_t b = ok ? item : (int64_t)blockIdx.x * kWave;  // idle lanes repeat a pair and store nothing
    const int64_t yb = offY[b];
    const int lb = (int)(offY[b + 1] - yb);
    int maxL = lb;
#pragma unroll
    for (int m = kWave / 2; m >= 1; m >>= 1) {
        const int o = __shfl_xor(maxL, m, kWave);
        maxL = o > maxL ? o : maxL;
    }
    maxL = __builtin_amdgcn_readfirstlane(maxL);
    // rows of this wave: row r of [RM - nr, RM) is query row row0 + r
    const int nr = nQ - w * RM < RM ? nQ - w * RM : RM;  // may be <= 0 (this wave only stages samples)
    const int row0 = w * RM + 1 - (RM - nr);
    const int last_wave = (nQ - 1) / RM;

    // columns past a series' end repeat its last sample (nothing reads them)
    auto sample = [&](int j) { return yb + (j <= lb ? j : lb) - 1; };
    auto place_of = [&](int j) { return RAW ? sample(j) * dim : (sample(j) + 1 + b) * S; };
    vec fetched[kLoads];
    CT fetched_t = CT(0);
    auto staged = [&](int j, int p) { return stage + (((j & 1) << 6) + p) * pitch; };
    const int t_at = RAW ? dim : DIMT;  // where a staged sample's timestamp sits
    auto fetch = [&](int j) {
#pragma unroll
        for (int n = 0; n < kLoads; ++n) {
            const int u = tid + n * kWave * W;
            const int p = u / NU, k = (u - p * NU) * V;
            vec v = {};
            if (p < kWave) {
                if constexpr (!RAW) {
                    v = *reinterpret_cast<const vec *>(rowsY + place[j & 1][p] + k);
                } else if (k < dim) {
                    const CT *src = Yraw + place[j & 1][p] + k;
                    if (wide) {
                        v = *reinterpret_cast<const vec *>(src);
                    } else {
#pragma unroll
                        for (int e = 0; e < V; ++e) v[e] = k + e < dim ? src[e] : CT(0);
                    }
                }
            }
            fetched[n] = v;
        }
        if constexpr (RAW)
            if (w == 0) fetched_t = TYraw[sample(j)];
    };
    auto put = [&](int j) {
#pragma unroll
        for (int n = 0; n < kLoads; ++n) {
            const int u = tid + n * kWave * W;
            const int p = u / NU, k = (u - p * NU) * V;
            if (p >= kWave || (RAW && k >= dim)) continue;
            CT *dst = staged(j, p) + k;
            if (RAW && k + V > dim) {  // the timestamp follows the last component
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (k + e < dim) dst[e] = fetched[n][e];
            } else {
                *reinterpret_cast<vec *>(dst) = fetched[n];
            }
        }
        if constexpr (RAW)
            if (w == 0) staged(j, lane)[t_at] = fetched_t;
    };

    // One unit of the sum over components of row r's point distance.
    auto add = [&](CT sum, CT a, CT x) -> CT {
        const CT d = a - x;
        if constexpr (DIMT == 1 || PM == kL1) return sum + fabs_(d);
        else if constexpr (PM == kL2) return fma_(d, d, sum);
        else return sum + (fabs_(d) > CT(0) ? pow_(fabs_(d), ca.p) : CT(0));
    };
    auto root = [&](CT sum) -> CT {
        if constexpr (DIMT == 1 || PM == kL1) return sum;
        else if constexpr (PM == kL2) return sqrt_(sum);
        else return sum > CT(0) ? pow_(sum, ca.invp) : CT(0);
    };
    place[1][lane] = place_of(1);  // (every wave writes the same values)
    place[0][lane] = place_of(2);
    __syncthreads();
    fetch(1);
    put(1);

    AT up[RM], xq[RM];  // DP(i, j - 1) and X(i, j - 1) of the wave's rows
#pragma unroll
    for (int r = 0; r < RM; ++r) up[r] = xq[r] = INF;
    AT res = INF;

    // The sweep of a wave that runs the recurrence DELAY columns after the
    // point costs (DELAY = w).
    auto sweep = [&]<int DELAY>() {
        CT e[DELAY + 1][RM];
        AT x_above = DELAY == 0 ? AT(0) : INF;  // X of the row above, one column back; X(0, 0) = 0
        // column j of the wave's rows, from point costs ec, DP of the row
        // above and the column's deletion cost
        auto column = [&](int j, int s, const CT (&ec)[RM], AT above, CT del) {
            AT diag = x_above;
#pragma unroll
            for (int r = 0; r < RM; ++r) {
                if (r >= RM - nr) {
                    const AT ee = (AT)ec[r];
                    const AT dela = (AT)q[(int64_t)(row0 + r) * S + DIMT + 1];
                    const AT v = dmin(dmin(diag + ee, above + dela), up[r] + (AT)del);
                    diag = xq[r];
                    xq[r] = v + ee;
                    up[r] = v;
                    above = v;
                }
            }
            if constexpr (DELAY < W - 1) {
                QueryHandOff<AT> &h = hand[DELAY][s % kHands];
                h.dp[lane] = up[RM - 1];
                h.x[lane] = xq[RM - 1];
            }
            if constexpr (DELAY == 0) dels[j & 3][lane] = del;
            if (DELAY == last_wave) res = j == lb ? up[RM - 1] : res;
        };
        AT above_next = INF, x_next = INF;  // one buffer: DP and X of the row above, handed over at the step before
        const int steps = maxL + last_wave;
        for (int s = 1; s <= steps; ++s) {
            __syncthreads();
            if (s < maxL) fetch(s + 1);
            if (w == 0 && s + 2 <= maxL) place[s & 1][lane] = place_of(s + 2);
            if constexpr (DELAY > 0) {
                const int j = s - DELAY;
                if (j >= 1 && j <= maxL && nr > 0) {
                    const QueryHandOff<AT> &h = hand[DELAY - 1][(s - 1) % kHands];
                    const AT above = kHands == 1 ? above_next : h.dp[lane], xn = kHands == 1 ? x_next : h.x[lane];
                    column(j, s, e[DELAY - 1], above, dels[j & 3][lane]);
                    x_above = xn;
                }
#pragma unroll
                for (int n = DELAY; n > 0; --n)
#pragma unroll
                    for (int r = 0; r < RM; ++r) e[n][r] = e[n - 1][r];
            }
            if (s <= maxL && nr > 0) {
                const CT *smp = (const CT *)__builtin_assume_aligned(staged(s, lane), 16);
                CT sum[RM];
#pragma unroll
                for (int r = 0; r < RM; ++r) sum[r] = CT(0);
                // C components at k0 of every row: the samples' once, the
                // query's four rows at a time, the next four loaded (after
                // these have come: scalar loads return out of order, so a wait
                // is for all of them) before these rows' arithmetic
                auto block = [&]<int C>(int k0) {
                    constexpr int H = 4;
                    CT x[C], a[2][H][C];
#pragma unroll
                    for (int c = 0; c < C; ++c) x[c] = smp[k0 + c];
                    auto load = [&](int r, CT (&d)[H][C]) {
#pragma unroll
                        for (int h = 0; h < H; ++h)
#pragma unroll
                            for (int c = 0; c < C; ++c)
                                if (r + h < RM) d[h][c] = q[(int64_t)(row0 + r + h) * S + k0 + c];
                    };
                    load(0, a[0]);
#pragma unroll
                    for (int r = 0; r < RM; r += H) {
                        CT (&cur)[H][C] = a[(r / H) & 1];
                        asm volatile("" ::"s"(cur[0][0]));
                        if (r + H < RM) load(r + H, a[(r / H + 1) & 1]);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int c = 0; c < C; ++c)
#pragma unroll
                            for (int h = 0; h < H; ++h)
                                if (r + h < RM) sum[r + h] = add(sum[r + h], cur[h][c], x[c]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                if constexpr (DIMT <= 4) {
                    block.template operator()<DIMT>(0);
                } else {
                    int k0 = 0;
                    for (; k0 + 4 <= dim; k0 += 4) block.template operator()<4>(k0);
                    for (; k0 < dim; ++k0) block.template operator()<1>(k0);
                }
                const CT t = smp[t_at];
#pragma unroll
                for (int r = 0; r < RM; ++r)
                    e[0][r] = fma_(ca.nu, fabs_(q[(int64_t)(row0 + r) * S + DIMT] - t), root(sum[r]));
                if constexpr (DELAY == 0) {
                    CT del;
                    if constexpr (RAW) {
                        const CT *before = staged(s - 1, lane);
                        CT d = CT(0), tp = CT(0);
                        if (s > 1) {
                            for (int k = 0; k < dim; ++k) d = add(d, smp[k], before[k]);
                            tp = before[t_at];
                        } else {
                            for (int k = 0; k < dim; ++k) d = add(d, smp[k], CT(0));
                        }
                        del = fma_(ca.nu, fabs_(t - tp), root(d)) + ca.lambda;
                    } else {
                        del = smp[DIMT + 1];
                    }
                    column(s, s, e[0], INF, del);  // the pad row above is +inf
                    x_above = INF;
                }
            }
            __syncthreads();  // (the sample before this column's is read above)
            if constexpr (DELAY > 0 && kHands == 1) {
                above_next = hand[DELAY - 1][0].dp[lane];
                x_next = hand[DELAY - 1][0].x[lane];
            }
            if (s < maxL) put(s + 1);
        }
    };
    if (w == 0) sweep.template operator()<0>();
    if (w == 1) sweep.template operator()<1>();
    if (w == 2) sweep.template operator()<2>();
    if (w == 3) sweep.template operator()<3>();
    if (ok && w == last_wave) D[item] = res;
}

hipError_t launch_batch_lane(Prec prec, const CostParams &cp, const void *rowsQ, int nQ, const void *rowsY,
                            const void *Yraw, const void *TYraw, const int64_t *offY, int64_t nY, void *D, hipStream_t st)
{
    if (nQ < 1 || nQ > kLaneMaxQuery) return hipErrorInvalidValue;
    const int grid = (int)((nY + kWave - 1) / kWave);
    return by_prec(prec, cp.dimt, cp.pm, [&]<typename CT, typename AT, int DIMT, int PM>() -> hipError_t {
        // 16-byte loads of the caller's samples where their alignment allows them
        const int wide = ((uintptr_t)Yraw % 16 == 0 && (size_t)cp.dim * sizeof(CT) % 16 == 0) ? 1 : 0;
        auto launch = [&]<bool RAW, int RM>() {
            const int pitch = query_pitch(cp.dim, DIMT, (int)sizeof(CT), RAW);
            hipLaunchKernelGGL((batch_query_kernel<CT, AT, DIMT, PM, RAW, RM>), dim3(grid), dim3(kWave * kQueryWaves),
                               (size_t)2 * kWave * pitch * sizeof(CT), st, (const CT *)rowsQ, nQ, (const CT *)rowsY,
                               (const CT *)Yraw, (const CT *)TYraw, cp.dim, pitch, wide, offY, nY,
                               CostArgs<CT>::make(cp), (AT *)D);
            return hipGetLastError();
        };
        // The rows a wave owns: the fewest compiled that hold the query in four
        // waves.  A wave computes the point costs of all RM rows, so the query's rows
        // fill the first waves instead of being spread over the four (FP64, 60,000
        // series of 20 .. 36 samples in R^32: 4 rows 247 us spread, now 138; 24 staged
        // rows 328, now 289).  Two rows only for small samples: of more components the
        // collection's samples bound a short query, and four rows in one wave leave
        // the others to stage them (one row, 200,000 series in R^28 FP32: 262 us at
        // two rows a wave, 220 at four).
        auto by_rows = [&]<bool RAW>() {
            if constexpr (DIMT <= 4)
                if (nQ <= 2 * kQueryWaves) return launch.template operator()<RAW, 2>();
            if (nQ <= 4 * kQueryWaves) return launch.template operator()<RAW, 4>();
            if (nQ <= 7 * kQueryWaves) return launch.template operator()<RAW, 7>();
            return launch.template operator()<RAW, kLaneMaxQuery / kQueryWaves>();
        };
        return Yraw ? by_rows.template operator()<true>() : by_rows.template operator()<false>();
    });
}

}  // namespace twed
