// tile_capi.hip -- extern "C" entry points of the tile sweep and of the
// alignment path (host code: argument checks, workspace layout, dispatch).
//
// A block of the DP matrix is swept from its top row and left column of
// (DP, X = DP + e) cells (section "Improved Time Warp Edit Distance": the
// band is the whole state), which gives resumable sweeps of long pairs and
// the column shards a multi-GPU sweep would hand from GPU to GPU.  The path
// is read back block by block from moves recorded during a second sweep of
// each block the path crosses (section "Time Warp Edit Distance" names
// backtracking over the forward problem's choices).
#include "../../include/twed.h"
#include "capi_util.h"
#include "twed_kernels.h"

#include <algorithm>
#include <cstdint>
#include <cstdlib>

using namespace twed;
using namespace twed::capi;

namespace {

constexpr int64_t kTailWords = 4;      // work ticket, wait error word, two spare words
constexpr size_t kDummyCells = 512;    // 64 lanes x up to 8 columns
constexpr int64_t kDefaultBlock = 4096;
constexpr size_t kCell = 16;           // one (DP, X) pair of FP64

int simds()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 1024;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 1024;
    return cus * 4;
}

bool tile_prec(const twed_params *prm, Prec *out)
{
    if (prm->precision == TWED_F64) *out = kF64;
    else if (prm->precision == TWED_F32_ACC64) *out = kF32Acc64;
    else return false;
    return true;
}

struct Sweep {
    int K, G;
};

// The recurrence a sweep runs: kRecTwed, or a sibling (kRecDtw, kRecEdit,
// kRecIndel; see twed_device.h).
size_t sweep_scratch(int rec, Prec prec, const CostParams &cp, int K, int G)
{
    return rec == kRecTwed ? tile_scratch_bytes(prec, cp, K, G) : dp_scratch_bytes(rec, prec, cp, K, G);
}

int sweep_workers(int rec, Prec prec, const CostParams &cp, int K, int G)
{
    return rec == kRecTwed ? tile_max_workers(prec, cp, K, G) : dp_max_workers(rec, prec, cp, K, G);
}

// Strip width and group of a sweep of nA x nB cells: the pair sweep's rule
// (resident_strip_width, groups of resident_group, while the strips fit one wave
// per SIMD; beyond that the widest strip that leaves three strips for every four
// SIMDs, in groups of eight where four fit at all), with kernels that have no
// scratch at all.
Sweep tile_sweep(int rec, int strip_k, int64_t nA, int64_t nB, Prec prec, const CostParams &cp)
{
    const int64_t n_simds = simds();
    const int G4 = resident_group(prec, cp.dimt, cp.pm);
    auto fits = [&](int K, int G) { return sweep_scratch(rec, prec, cp, K, G) == 0; };
    const int any[] = {1, G4 == 4 ? 2 : 0, 4, 8, 0};  // (the pair sweep's reason for one column)
    const int one[] = {strip_k, 0};
    int G = G4;
    int K = resident_strip_width(one[0] > 0 ? one : any, nA, nB, prec, cp, resident_slots(n_simds, G4),
                                 [&](int k) { return fits(k, G4); });
    if (K == 0) {
        K = one[0] > 0 ? one[0] : 1;
        if (one[0] <= 0 && G4 == 4) {
            for (int k : {8, 4, 2}) {
                if ((nB + 64 * k - 1) / (64 * k) * 4 >= n_simds * 3 && (fits(k, 8) || fits(k, G4))) {
                    K = k;
                    break;
                }
            }
        }
        if (G4 == 4 && fits(K, 8)) G = 8;
    }
    // TWED_WAVEFRONT_GROUP (4 or 8) overrides the group of plain TWED tile
    // sweeps for tuning runs
    if (const char *env = std::getenv("TWED_WAVEFRONT_GROUP")) {
        const int g = std::atoi(env);
        if (rec == kRecTwed && (g == 4 || g == 8) && fits(K, g)) G = g;
    }
    return Sweep{K, G};
}

// Staged rows, handoff slots, flags and scratch of one sweep of nA x nB.
struct SweepBuffers {
    void *rowsA, *rowsB, *bnd, *dummy, *tmp;
    uint32_t *flags;
    int64_t zero_words;
};

void take_sweep(Carver &c, SweepBuffers &b, Prec prec, int dimt, int64_t nA, int64_t nB)
{
    b.rowsA = take_rows(c, prec, dimt, nA + 1);
    b.rowsB = take_rows(c, prec, dimt, nB + 1);
    b.bnd = c.take((size_t)2 * (size_t)(nA + 1) * kCell);
    b.zero_words = (nB + 63) / 64 + kTailWords;
    b.flags = (uint32_t *)c.take((size_t)b.zero_words * 4);
    b.dummy = c.take(kDummyCells * kCell);
    b.tmp = c.take(8);
}

twed_status run_tile(int rec, Prec prec, const CostParams &cp, Sweep sw, const void *rowsA, const void *rowsB,
                     int64_t nA, int64_t nB, const SweepBuffers &b, const TileArgs &t, void *out, hipStream_t st)
{
    WavefrontArgs w{};
    w.rowsA = rowsA;
    w.rowsB = rowsB;
    w.nA = nA;
    w.nB = nB;
    w.bnd = b.bnd;
    w.flags = b.flags;
    w.ticket = b.flags + (b.zero_words - kTailWords);
    w.beta = w.ticket + 2;
    w.nStrips = (nB + 64 * sw.K - 1) / (64 * sw.K);
    w.out = out;
    w.dump = nullptr;
    w.group = sw.G;
    w.sub_shift = kSubShift;
    const int workers = sweep_workers(rec, prec, cp, sw.K, sw.G);
    if (workers <= 0) return fail(TWED_ERR_DEVICE, "occupancy query failed");
    w.grid = (int)std::min<int64_t>((w.nStrips + sw.G - 1) / sw.G, workers);
    const hipError_t e = rec == kRecTwed ? launch_tile(prec, cp, sw.K, w, t, st)
                                         : launch_dp(rec, prec, cp, sw.K, w, t, st);
    if (e != hipSuccess) return fail_hip(e, "tile sweep launch");
    return TWED_OK;
}

twed_status check_series(const void *A, const void *TA, int64_t nA, const void *B, const void *TB, int64_t nB)
{
    if (!A || !TA || !B || !TB) return fail(TWED_ERR_INVALID, "NULL array argument");
    if (nA < 1 || nB < 1) return fail(TWED_ERR_INVALID, "series lengths must be >= 1");
    if (nA > kMaxLen || nB > kMaxLen) return fail(TWED_ERR_UNSUPPORTED, "series longer than 2^31 - 130");
    return TWED_OK;
}

size_t row_bytes(Prec prec, int dimt) { return (size_t)row_stride(prec, dimt) * cost_size(prec); }

// ---- path layout ---------------------------------------------------------------

struct PathGeometry {
    Sweep fwd;
    int64_t H, Wc, nr, nc;
};

PathGeometry path_geometry(int rec, const twed_params *prm, int64_t nA, int64_t nB, int64_t block, Prec prec,
                           const CostParams &cp)
{
    PathGeometry g{};
    const int64_t want = block > 0 ? block : kDefaultBlock;
    g.fwd = tile_sweep(rec, prm->strip_k, nA, nB, prec, cp);
    const int64_t W = 64 * (int64_t)g.fwd.K;
    g.H = std::max<int64_t>(64, want);
    g.Wc = (std::max(want, W) + W - 1) / W * W;
    g.nr = (nA - 1) / g.H;
    g.nc = (nB - 1) / g.Wc;
    return g;
}

// Edit and indel distances start from finite row 0 / column 0 (i, i).
bool finite_edges(int rec) { return rec == kRecEdit || rec == kRecIndel; }

// Blocks swept again with moves while the walk is in one of them: that block,
// its neighbours up and to the left, and the blocks that the direction of the
// last few walks leads to.  A block's sweep takes several times as long as its
// walk (1.5 ms against 0.2 for 4,096 x 4,096 8-D cells), so it has to start
// several walks ahead.  Each block has a slot; there are more slots than blocks
// wanted, so that a new block need not wait for the sweep of one that is no
// longer wanted.  (With the neighbours only, in four slots, every block was waited
// for; with squares of blocks the launches held each other up.)
constexpr int kPathAhead = 8;  // walks
constexpr int kPathSlots = 24, kPathSlotsMin = 4;

int path_slots(int64_t nr, int64_t nc)
{
    return (int)std::clamp<int64_t>((nr + 1) * (nc + 1), kPathSlotsMin, kPathSlots);
}

struct WantedBlocks {
    int64_t r[kMaxDirsBlocks], c[kMaxDirsBlocks];
    int n = 0, near = 0;  // blocks 0 .. near - 1 are the walk's and those it may enter next
    int limit;
    bool add(int64_t br, int64_t bc)
    {
        if (br < 0 || bc < 0 || n >= limit) return false;
        for (int i = 0; i < n; ++i)
            if (r[i] == br && c[i] == bc) return false;
        r[n] = br;
        c[n++] = bc;
        return true;
    }
};

// The walk is in block (br, bc), having come `up` blocks up and `left` blocks to
// the left in its last few walks.
WantedBlocks wanted_blocks(int64_t br, int64_t bc, int64_t up, int64_t left, int limit)
{
    WantedBlocks w;
    w.limit = limit;
    w.add(br, bc);
    w.add(br - 1, bc);
    w.add(br, bc - 1);
    w.near = w.n;
    w.add(br - 1, bc - 1);
    if (up + left == 0) up = br, left = bc;  // no walk yet: towards (0, 0)
    if (br == 0) up = 0, left = 1;
    if (bc == 0) up = 1, left = 0;
    for (int64_t j = 2; j <= kPathAhead && up + left > 0; ++j) {
        const int64_t lo = j * up / (up + left), hi = (j * up + up + left - 1) / (up + left);
        w.add(br - lo, bc - (j - lo));
        w.add(br - hi, bc - (j - hi));
        if (j == 2) {
            w.add(br - 2, bc - 1);
            w.add(br - 1, bc - 2);
        }
    }
    return w;
}

// What one block sweep writes: boundary, flags, dummy cells, result and moves.
struct BlockBuffers {
    void *bnd, *dummy, *tmp;
    uint32_t *flags;
    void *dirs;
};

struct PathLayout {
    SweepBuffers b;
    BlockBuffers slot[kPathSlots];
    int64_t zero_words;  // of a slot's flags
    void *ckrow, *ckcol, *row0, *col0;
    int64_t *st;
    size_t total;
};

PathLayout path_layout(char *base, int rec, const twed_params *prm, int64_t nA, int64_t nB, const PathGeometry &g,
                       Prec prec, int slots)
{
    Carver c{base};
    PathLayout L{};
    take_sweep(c, L.b, prec, dimt_for(prm->dim), nA, nB);
    L.st = (int64_t *)c.take(4 * sizeof(int64_t));
    if (finite_edges(rec)) {
        L.row0 = c.take((size_t)(nB + 1) * kCell);
        L.col0 = c.take((size_t)(nA + 1) * kCell);
    }
    L.ckrow = c.take((size_t)g.nr * (size_t)(nB + 1) * kCell);
    L.ckcol = c.take((size_t)g.nc * (size_t)(nA + 1) * kCell);
    const int64_t bh = std::min(g.H, nA), bw = std::min(g.Wc, nB);
    L.zero_words = (bw + 63) / 64 + kTailWords;
    for (int k = 0; k < slots; ++k) {
        BlockBuffers &u = L.slot[k];
        u.bnd = c.take((size_t)2 * (size_t)(bh + 1) * kCell);
        u.flags = (uint32_t *)c.take((size_t)L.zero_words * 4);
        u.dummy = c.take(kDummyCells * kCell);
        u.tmp = c.take(8);
        u.dirs = c.take(dirs_bytes(bh, bw));
    }
    L.total = c.used;
    return L;
}

// Side streams and events of the backward pass; the destructor waits for
// their work (speculative block sweeps may still run) before releasing them.
// Three streams, taken in turn: with the caller's they fit four hardware queues,
// and the sweeps started for the walk three blocks earlier have ended.
constexpr int kPathStreams = 3;
struct PathStreams {
    hipStream_t s[kPathStreams] = {};
    hipEvent_t done[kPathSlots] = {};
    hipEvent_t fwd = nullptr;
    hipError_t create(int slots)
    {
        hipError_t e = hipEventCreateWithFlags(&fwd, hipEventDisableTiming);
        for (int k = 0; k < kPathStreams && e == hipSuccess; ++k)
            e = hipStreamCreateWithFlags(&s[k], hipStreamNonBlocking);
        for (int k = 0; k < slots && e == hipSuccess; ++k)
            e = hipEventCreateWithFlags(&done[k], hipEventDisableTiming);
        return e;
    }
    ~PathStreams()
    {
        for (int k = 0; k < kPathStreams; ++k) {
            if (s[k]) {
                (void)hipStreamSynchronize(s[k]);
                (void)hipStreamDestroy(s[k]);
            }
        }
        for (hipEvent_t ev : done)
            if (ev) (void)hipEventDestroy(ev);
        if (fwd) (void)hipEventDestroy(fwd);
    }
};

// The path of one pair under recurrence `rec` (A/TA/B/TB as staged by
// twed_pair; TA, TB null for the siblings).  Runs after argument checks.
twed_status path_impl(int rec, const void *A, const void *TA, int64_t nA, const void *B, const void *TB, int64_t nB,
                      const twed_params *prm, int64_t block, double *out, int64_t *path, int64_t *path_len,
                      void *workspace, size_t ws_bytes, Prec prec, hipStream_t st)
{
    twed_status s;
    const CostParams cp = cost_params(prm);
    const PathGeometry g = path_geometry(rec, prm, nA, nB, block, prec, cp);
    if (g.H > 0x40000000LL || g.Wc > 0x40000000LL) return fail(TWED_ERR_UNSUPPORTED, "block too large");
    // (a workspace too small for all slots gets the four it takes at least)
    int slots = path_slots(g.nr, g.nc);
    if (path_layout(nullptr, rec, prm, nA, nB, g, prec, slots).total > ws_bytes) slots = kPathSlotsMin;
    if ((s = check_workspace(workspace, ws_bytes, path_layout(nullptr, rec, prm, nA, nB, g, prec, slots).total)) !=
        TWED_OK)
        return s;
    const PathLayout L = path_layout((char *)workspace, rec, prm, nA, nB, g, prec, slots);
    const SweepBuffers &b = L.b;
    hipError_t e;
#define TRY(call, what)                                \
    do {                                               \
        e = (call);                                    \
        if (e != hipSuccess) return fail_hip(e, what); \
    } while (0)
    // forward sweep of the whole pair, keeping checkpoint rows and columns
    TRY(launch_stage(prec, cp, A, TA, nullptr, 1, nA, nA, nA + 1, b.rowsA, b.flags, b.zero_words, st), "staging");
    TRY(launch_stage(prec, cp, B, TB, nullptr, 1, nB, nB, nB + 1, b.rowsB, nullptr, 0, st), "staging");
    if (finite_edges(rec)) {
        TRY(launch_index_cells(L.row0, nB, st), "boundary");
        TRY(launch_index_cells(L.col0, nA, st), "boundary");
    }
    TileArgs t{};
    t.top = L.row0;
    t.left = L.col0;
    t.dummy = b.dummy;
    t.ckrow = g.nr > 0 ? L.ckrow : nullptr;
    t.ckcol = g.nc > 0 ? L.ckcol : nullptr;
    t.ck_rows = (int)g.H;
    t.ck_cols = (int)g.Wc;
    s = run_tile(rec, prec, cp, g.fwd, b.rowsA, b.rowsB, nA, nB, b, t, out, st);
    if (s != TWED_OK) return s;
    // Backwards, block by block: sweep the block again recording moves, walk
    // it.  While the walk runs on the caller's stream, the blocks it and the
    // next walk can leave into are swept on a side stream, all in one launch,
    // so that their moves are ready or nearly so when a walk gets there.
    const int64_t cap = nA + nB + 1;
    TRY(launch_walk_init(L.st, nA, nB, st), "walk set-up");
    const size_t rb = row_bytes(prec, dimt_for(prm->dim));
    PathStreams ps;
    TRY(ps.create(slots), "stream set-up");
    TRY(hipEventRecord(ps.fwd, st), "event record");
    for (int k = 0; k < kPathStreams; ++k) TRY(hipStreamWaitEvent(ps.s[k], ps.fwd, 0), "stream wait");
    int64_t held[kPathSlots][3];  // block row and column, and the launch that sweeps it
    for (int k = 0; k < slots; ++k) held[k][0] = held[k][1] = held[k][2] = -1;
    auto slot_of = [&](int64_t qr, int64_t qc) {
        for (int k = 0; k < slots; ++k)
            if (held[k][0] == qr && held[k][1] == qc) return k;
        return -1;
    };
    // block (br, bc) to be swept into slot k
    auto block_args = [&](int k, int64_t br, int64_t bc) {
        const int64_t r0 = br * g.H, r1 = std::min(r0 + g.H, nA);
        const int64_t c0 = bc * g.Wc, c1 = std::min(c0 + g.Wc, nB);
        const BlockBuffers &sb = L.slot[k];
        DirsArgs u{};
        u.rowsA = (const char *)b.rowsA + r0 * rb;
        u.rowsB = (const char *)b.rowsB + c0 * rb;
        u.nA = r1 - r0;
        u.nB = c1 - c0;
        u.bnd = sb.bnd;
        u.flags = sb.flags;
        u.ticket = sb.flags + (L.zero_words - kTailWords);
        u.dummy = sb.dummy;
        u.out = sb.tmp;
        u.dirs = sb.dirs;
        if (br > 0)
            u.top = (const char *)L.ckrow + ((size_t)(br - 1) * (size_t)(nB + 1) + (size_t)c0) * kCell;
        else if (L.row0)
            u.top = (const char *)L.row0 + (size_t)c0 * kCell;
        if (bc > 0)
            u.left = (const char *)L.ckcol + ((size_t)(bc - 1) * (size_t)(nA + 1) + (size_t)r0) * kCell;
        else if (L.col0)
            u.left = (const char *)L.col0 + (size_t)r0 * kCell;
        return u;
    };
    int64_t hst[4] = {0, 0, 0, 0};
    int64_t launches = 0;
    constexpr int kTrail = 4;  // walks whose blocks tell the direction
    int64_t trail[kTrail][2] = {};
    const int64_t max_blocks = g.nr + g.nc + 3;
    for (int64_t it = 0;; ++it) {
        TRY(hipMemcpyAsync(hst, L.st, sizeof(hst), hipMemcpyDeviceToHost, st), "walk state read");
        TRY(hipStreamSynchronize(st), "walk state read");
        if (hst[3] == 1) break;
        if (hst[3] != 0 || it > max_blocks || hst[0] < 1 || hst[1] < 1)
            return fail(TWED_ERR_DEVICE, "the path could not be followed (non-finite distance or a timed-out sweep)");
        const int64_t br = (hst[0] - 1) / g.H, bc = (hst[1] - 1) / g.Wc;
        auto walk = [&](int kc) -> hipError_t {
            hipError_t e2 = hipStreamWaitEvent(st, ps.done[kc], 0);
            if (e2 != hipSuccess) return e2;
            return launch_walk(L.slot[kc].dirs, br * g.H, bc * g.Wc, std::min(g.H, nA - br * g.H), L.st, path, cap,
                               finite_edges(rec), st);
        };
        const bool swept = slot_of(br, bc) >= 0;
        if (swept) TRY(walk(slot_of(br, bc)), "walk");
        // A slot whose block is not among those wanted now may be overwritten:
        // every walk that read it has finished (the caller's stream was
        // synchronised), and its own sweep is waited for.
        const int64_t *from = trail[it >= kTrail ? it % kTrail : 0];
        const int64_t up = it > 0 ? from[0] - br : 0, left = it > 0 ? from[1] - bc : 0;
        const WantedBlocks want = wanted_blocks(br, bc, up, left, std::min(slots, kMaxDirsBlocks));
        trail[it % kTrail][0] = br;
        trail[it % kTrail][1] = bc;
        bool keep[kPathSlots] = {};
        int missing = 0;
        bool near = false;
        for (int i = 0; i < want.n; ++i) {
            const int k = slot_of(want.r[i], want.c[i]);
            if (k >= 0) keep[k] = true;
            else ++missing, near = near || i < want.near;
        }
        // A walk leaves a few blocks missing; they wait for the next one's, so
        // that a launch brings more blocks: only as many launches run at a time as
        // there are side streams.
        if (near || missing > kPathSlotsMin) {
            ++launches;
            hipStream_t side = ps.s[launches % kPathStreams];
            DirsArgs todo[kMaxDirsBlocks];
            int at[kMaxDirsBlocks], nt = 0;
            for (int i = 0; i < want.n; ++i) {
                if (slot_of(want.r[i], want.c[i]) >= 0) continue;
                // of the slots that hold no wanted block (there is one: no more
                // blocks are wanted than there are slots) the one swept longest ago
                int k = -1;
                for (int f = 0; f < slots; ++f)
                    if (!keep[f] && (k < 0 || held[f][2] < held[k][2])) k = f;
                keep[k] = true;
                if (held[k][0] >= 0) TRY(hipStreamWaitEvent(side, ps.done[k], 0), "stream wait");
                held[k][0] = want.r[i];
                held[k][1] = want.c[i];
                held[k][2] = launches;
                todo[nt] = block_args(k, want.r[i], want.c[i]);
                at[nt++] = k;
            }
            TRY(launch_zero_flags(todo, nt, L.zero_words, side), "flag reset");
            TRY(launch_dirs(rec, prec, cp, todo, nt, side), "block sweep");
            for (int i = 0; i < nt; ++i) TRY(hipEventRecord(ps.done[at[i]], side), "event record");
        }
        if (!swept) TRY(walk(slot_of(br, bc)), "walk");
    }
    // later work on the caller's stream (and its reuse of the workspace)
    // stays behind speculative sweeps still running
    for (int k = 0; k < slots; ++k)
        if (held[k][0] >= 0) TRY(hipStreamWaitEvent(st, ps.done[k], 0), "stream wait");
    TRY(launch_order(L.st, path, path_len, cap, st), "path order");
    // the path and its length are complete when the call returns
    TRY(hipStreamSynchronize(st), "path order");
#undef TRY
    return TWED_OK;
}

// The recurrence of a twed_dp kind, or -1.
int rec_of(int32_t kind)
{
    switch (kind) {
    case TWED_DP_DTW: return kRecDtw;
    case TWED_DP_EDIT: return kRecEdit;
    case TWED_DP_LCS: return kRecIndel;
    default: return -1;
    }
}

twed_status check_dp(int32_t kind, const twed_params *prm, Prec *prec)
{
    twed_status s = check_params(prm);
    if (s != TWED_OK) return s;
    if (rec_of(kind) < 0) return fail(TWED_ERR_INVALID, "unknown twed_dp_kind");
    if (kind != TWED_DP_DTW && prm->dim != 1)
        return fail(TWED_ERR_UNSUPPORTED, "edit distance and LCS compare 1-D samples (dim = 1)");
    if (!(prm->strip_k == 0 || prm->strip_k == 1 || prm->strip_k == 2 || prm->strip_k == 8))
        return fail(TWED_ERR_UNSUPPORTED, "twed_dp takes strip_k 0, 1, 2 or 8");
    if (!tile_prec(prm, prec)) return fail(TWED_ERR_UNSUPPORTED, "twed_dp takes TWED_F64 or TWED_F32_ACC64");
    return TWED_OK;
}

}  // namespace

extern "C" {

size_t twed_pair_tile_workspace_size(int64_t rows, int64_t cols, const twed_params *prm)
{
    Prec prec;
    if (rows < 1 || cols < 1 || rows > kMaxLen || cols > kMaxLen) return 0;
    if (check_params(prm) != TWED_OK || !tile_prec(prm, &prec)) return 0;
    Carver c{nullptr};
    SweepBuffers b{};
    take_sweep(c, b, prec, dimt_for(prm->dim), rows, cols);
    return c.used;
}

twed_status twed_pair_tile(const void *A, const void *TA, int64_t nA, const void *B, const void *TB, int64_t nB,
                           const twed_params *prm, int64_t r0, int64_t r1, int64_t c0, int64_t c1,
                           const twed_cell *top, const twed_cell *left, twed_cell *bottom, twed_cell *right,
                           double *corner, void *workspace, size_t ws_bytes, hipStream_t st)
{
    last_error().clear();
    twed_status s = check_params(prm);
    if (s != TWED_OK) return s;
    if ((s = check_series(A, TA, nA, B, TB, nB)) != TWED_OK) return s;
    if (!(0 <= r0 && r0 < r1 && r1 <= nA && 0 <= c0 && c0 < c1 && c1 <= nB))
        return fail(TWED_ERR_INVALID, "the block must satisfy 0 <= r0 < r1 <= nA and 0 <= c0 < c1 <= nB");
    if (r0 > 0 && !top) return fail(TWED_ERR_INVALID, "a block below row 0 needs its top row");
    if (c0 > 0 && !left) return fail(TWED_ERR_INVALID, "a block right of column 0 needs its left column");
    Prec prec;
    if (!tile_prec(prm, &prec)) return fail(TWED_ERR_UNSUPPORTED, "tiles take TWED_F64 or TWED_F32_ACC64");
    const int64_t nAt = r1 - r0, nBt = c1 - c0;
    const size_t need = twed_pair_tile_workspace_size(nAt, nBt, prm);
    if ((s = check_workspace(workspace, ws_bytes, need)) != TWED_OK) return s;
    Carver c{(char *)workspace};
    SweepBuffers b{};
    const int dimt = dimt_for(prm->dim);
    take_sweep(c, b, prec, dimt, nAt, nBt);
    const CostParams cp = cost_params(prm);
    const size_t es = cost_size(prec) * (size_t)prm->dim, ts = cost_size(prec);
    hipError_t e = launch_stage(prec, cp, (const char *)A + r0 * es, (const char *)TA + r0 * ts, nullptr, 1, nAt,
                                nAt, nAt + 1, b.rowsA, b.flags, b.zero_words, st, r0 > 0);
    if (e != hipSuccess) return fail_hip(e, "staging launch");
    e = launch_stage(prec, cp, (const char *)B + c0 * es, (const char *)TB + c0 * ts, nullptr, 1, nBt, nBt, nBt + 1,
                     b.rowsB, nullptr, 0, st, c0 > 0);
    if (e != hipSuccess) return fail_hip(e, "staging launch");
    TileArgs t{};
    t.top = top;
    t.left = left;
    t.bottom = bottom;
    t.right = right;
    t.dummy = b.dummy;
    return run_tile(kRecTwed, prec, cp, tile_sweep(kRecTwed, prm->strip_k, nAt, nBt, prec, cp), b.rowsA, b.rowsB, nAt,
                    nBt, b, t, corner ? (void *)corner : b.tmp, st);
}

size_t twed_pair_path_workspace_size(int64_t nA, int64_t nB, const twed_params *prm, int64_t block)
{
    Prec prec;
    if (nA < 1 || nB < 1 || nA > kMaxLen || nB > kMaxLen || block < 0) return 0;
    if (check_params(prm) != TWED_OK || !tile_prec(prm, &prec)) return 0;
    const CostParams cp = cost_params(prm);
    const PathGeometry g = path_geometry(kRecTwed, prm, nA, nB, block, prec, cp);
    return path_layout(nullptr, kRecTwed, prm, nA, nB, g, prec, path_slots(g.nr, g.nc)).total;
}

twed_status twed_pair_path(const void *A, const void *TA, int64_t nA, const void *B, const void *TB, int64_t nB,
                           const twed_params *prm, int64_t block, double *out, int64_t *path, int64_t *path_len,
                           void *workspace, size_t ws_bytes, hipStream_t st)
{
    last_error().clear();
    twed_status s = check_params(prm);
    if (s != TWED_OK) return s;
    if ((s = check_series(A, TA, nA, B, TB, nB)) != TWED_OK) return s;
    if (!out || !path || !path_len) return fail(TWED_ERR_INVALID, "NULL output argument");
    if (block < 0) return fail(TWED_ERR_INVALID, "block must be >= 0");
    Prec prec;
    if (!tile_prec(prm, &prec)) return fail(TWED_ERR_UNSUPPORTED, "the path takes TWED_F64 or TWED_F32_ACC64");
    return path_impl(kRecTwed, A, TA, nA, B, TB, nB, prm, block, out, path, path_len, workspace, ws_bytes, prec, st);
}

size_t twed_dp_workspace_size(int32_t kind, int64_t nA, int64_t nB, const twed_params *prm)
{
    Prec prec;
    if (nA < 1 || nB < 1 || nA > kMaxLen || nB > kMaxLen) return 0;
    if (check_dp(kind, prm, &prec) != TWED_OK) return 0;
    Carver c{nullptr};
    SweepBuffers b{};
    take_sweep(c, b, prec, dimt_for(prm->dim), nA, nB);
    c.take((size_t)(nA + nB + 2) * kCell);
    return c.used;
}

twed_status twed_dp(int32_t kind, const void *A, int64_t nA, const void *B, int64_t nB, const twed_params *prm,
                    double *out, void *workspace, size_t ws_bytes, hipStream_t st)
{
    last_error().clear();
    Prec prec;
    twed_status s = check_dp(kind, prm, &prec);
    if (s != TWED_OK) return s;
    if (!A || !B || !out) return fail(TWED_ERR_INVALID, "NULL array argument");
    if (nA < 1 || nB < 1) return fail(TWED_ERR_INVALID, "series lengths must be >= 1");
    if (nA > kMaxLen || nB > kMaxLen) return fail(TWED_ERR_UNSUPPORTED, "series longer than 2^31 - 130");
    if ((s = check_workspace(workspace, ws_bytes, twed_dp_workspace_size(kind, nA, nB, prm))) != TWED_OK) return s;
    const int rec = rec_of(kind);
    Carver c{(char *)workspace};
    SweepBuffers b{};
    take_sweep(c, b, prec, dimt_for(prm->dim), nA, nB);
    void *row0 = c.take((size_t)(nB + 1) * kCell);
    void *col0 = c.take((size_t)(nA + 1) * kCell);
    const CostParams cp = cost_params(prm);
    hipError_t e = launch_stage(prec, cp, A, nullptr, nullptr, 1, nA, nA, nA + 1, b.rowsA, b.flags, b.zero_words, st);
    if (e != hipSuccess) return fail_hip(e, "staging launch");
    e = launch_stage(prec, cp, B, nullptr, nullptr, 1, nB, nB, nB + 1, b.rowsB, nullptr, 0, st);
    if (e != hipSuccess) return fail_hip(e, "staging launch");
    TileArgs t{};
    t.dummy = b.dummy;
    if (finite_edges(rec)) {
        if ((e = launch_index_cells(row0, nB, st)) != hipSuccess) return fail_hip(e, "boundary");
        if ((e = launch_index_cells(col0, nA, st)) != hipSuccess) return fail_hip(e, "boundary");
        t.top = row0;
        t.left = col0;
    }
    s = run_tile(rec, prec, cp, tile_sweep(rec, prm->strip_k, nA, nB, prec, cp), b.rowsA, b.rowsB, nA, nB, b, t, out, st);
    if (s != TWED_OK) return s;
    if (kind == TWED_DP_LCS && (e = launch_lcs_finish(out, nA, nB, st)) != hipSuccess) return fail_hip(e, "LCS");
    return TWED_OK;
}

size_t twed_dp_path_workspace_size(int32_t kind, int64_t nA, int64_t nB, const twed_params *prm, int64_t block)
{
    Prec prec;
    if (nA < 1 || nB < 1 || nA > kMaxLen || nB > kMaxLen || block < 0) return 0;
    if (check_dp(kind, prm, &prec) != TWED_OK) return 0;
    const int rec = rec_of(kind);
    const CostParams cp = cost_params(prm);
    const PathGeometry g = path_geometry(rec, prm, nA, nB, block, prec, cp);
    return path_layout(nullptr, rec, prm, nA, nB, g, prec, path_slots(g.nr, g.nc)).total;
}

twed_status twed_dp_path(int32_t kind, const void *A, int64_t nA, const void *B, int64_t nB, const twed_params *prm,
                         int64_t block, double *out, int64_t *path, int64_t *path_len, void *workspace,
                         size_t ws_bytes, hipStream_t st)
{
    last_error().clear();
    Prec prec;
    twed_status s = check_dp(kind, prm, &prec);
    if (s != TWED_OK) return s;
    if (!A || !B) return fail(TWED_ERR_INVALID, "NULL array argument");
    if (nA < 1 || nB < 1) return fail(TWED_ERR_INVALID, "series lengths must be >= 1");
    if (nA > kMaxLen || nB > kMaxLen) return fail(TWED_ERR_UNSUPPORTED, "series longer than 2^31 - 130");
    if (!out || !path || !path_len) return fail(TWED_ERR_INVALID, "NULL output argument");
    if (block < 0) return fail(TWED_ERR_INVALID, "block must be >= 0");
    s = path_impl(rec_of(kind), A, nullptr, nA, B, nullptr, nB, prm, block, out, path, path_len, workspace, ws_bytes,
                  prec, st);
    if (s != TWED_OK) return s;
    if (kind == TWED_DP_LCS) {
        const hipError_t e = launch_lcs_finish(out, nA, nB, st);
        if (e != hipSuccess) return fail_hip(e, "LCS");
    }
    return TWED_OK;
}

}  // extern "C"
