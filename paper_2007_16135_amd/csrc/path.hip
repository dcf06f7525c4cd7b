// path.hip -- reading an optimal alignment path back from recorded moves.
//
// The paper's section "Time Warp Edit Distance" notes that the alignment
// path follows by backtracking over the choices of the forward problem.  The
// block sweep records the move into every cell of a block (two bits, in sweep
// order) and the walk below follows them from a cell of the block back to the
// block's top row or left column.  The path is written from its end, (nA, nB), so
// the cells come out in reverse; a last pass puts them in order.
#include "twed_device.h"
#include "twed_kernels.h"

namespace twed {

namespace {

// One wave.  The walk is a chain of dependent steps, so what it costs is the
// latency of one link.  320 steps of the strip it is in (the rows it can meet in
// that strip's 64 columns) go to LDS, and those of the strip to the left are
// requested while it walks.  Lane l then shifts the moves of 32 rows of column l
// into 64 bits: bit 2k says that row k is left by a match, bit 2k + 1 by a
// deletion in B.  The chain runs on scalar registers and links columns, not
// cells: entered at row k, a column is left at its highest bit p at or below 2k +
// 1, and the next one is entered at row (p - 1) / 2, rounded up.  All that is
// noted is the entry row, in the column's lane; the lanes then store the cells
// of their columns side by side.  (Moves as bytes, followed one by one in LDS
// with 64 scattered loads per 64 x 64 window: 1,230 us for the part of a path in
// a block of 4,096 x 4,096.)
// st = {r, c, n, status} in global coordinates; status 0 running, 1 reached
// (0, 0), -1 failed.
//
// With free_edges (edit and indel distances, whose row 0 and column 0 are
// finite) a walk that reaches row 0 or column 0 follows it to (0, 0); for
// TWED and DTW those cells are +inf and reaching one is an error.
constexpr int kWalkPieces = 10;  // of 32 steps
constexpr int kWalkSteps = 32 * kWalkPieces;
constexpr int kWalkVecs = kWalkPieces * 512 / 1024;  // 16-byte loads per lane
typedef uint32_t WalkVec __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)(uint64_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)((uint64_t)hi << 32 | lo);
}

__device__ __forceinline__ uint64_t lane_mask64(uint64_t v, int l)
{
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return (uint64_t)hi << 32 | lo;
}

// Sum of v over lanes 0 .. lane.
__device__ __forceinline__ int wave_prefix_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

__global__ __launch_bounds__(kWave) void walk_kernel(const char *__restrict__ dirs, int64_t r0, int64_t c0,
                                                     int nAt, int64_t *st, int64_t *rev, int64_t cap, int free_edges)
{
    __shared__ alignas(16) uint64_t win[2][kWalkPieces * kWave];
    const int lane = threadIdx.x;
    if (st[3] != 0) return;
    int64_t n = uniform64(st[2]);
    // the current cell, local to the block
    int rr = (int)(uniform64(st[0]) - r0), cc = (int)(uniform64(st[1]) - c0);
    int status = 0;
    const int64_t strip_bytes = ((int64_t)nAt + kWave + 31) / 32 * 512;
    // steps base .. base + 319 of strip s (base a multiple of 32), 16 bytes per
    // lane and load (those behind the strip's last step repeat its last 16)
    WalkVec ahead[kWalkVecs];
    auto request = [&](int s, int base) {
        const char *p = dirs + (int64_t)s * strip_bytes;
#pragma unroll
        for (int v = 0; v < kWalkVecs; ++v) {
            const int64_t at = (int64_t)(base / 32) * 512 + v * 1024 + lane * 16;
            ahead[v] = *reinterpret_cast<const WalkVec *>(p + (at < strip_bytes - 16 ? at : strip_bytes - 16));
        }
    };
    // the rows q - 31 .. q of all columns sit at steps q - 31 .. q + 63: with 224
    // steps before the entry row, 193 rows further up are still covered
    auto base_for = [](int q) { return q > 224 ? (q - 224) / 32 * 32 : 0; };
    auto covers = [](int base, int q) {
        return (q > 31 ? q - 31 : 0) >= base && q + kWave - 1 < base + kWalkSteps;
    };
    // Two windows in LDS: the one walked on, and the next, which `ahead` goes to
    // when the strip ends, before its last cells are stored, so that no load is
    // waited for behind a store just made.  (One wave: its LDS accesses complete in order, and the fences keep
    // the compiler to that order.)
    int at = 0, cur_s = -1, cur_base = 0, next_s = -1, next_base = 0;
    bool pending = false;
    auto settle = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int v = 0; v < kWalkVecs; ++v) reinterpret_cast<WalkVec *>(win[at ^ 1])[v * kWave + lane] = ahead[v];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        pending = false;
    };
    auto start = [&](int s, int base) {
        next_s = s;
        next_base = base;
        request(s, base);
        pending = true;
    };
    while (rr > 0 && cc > 0) {
        const int s = (cc - 1) / kWave;
        int l = (cc - 1) - s * kWave;
        if (cur_s != s || !covers(cur_base, rr)) {
            if (next_s != s || !covers(next_base, rr)) start(s, base_for(rr));
            if (pending) settle();
            at ^= 1;
            cur_s = next_s;
            cur_base = next_base;
            next_s = -1;
            if (s > 0) start(s - 1, base_for(rr));
        }
        // moves of rows wr .. rr = wr + 31 of column `lane` (words outside the
        // window hold rows above the block only)
        const int wr = rr - 31;
        const int f = wr + lane - cur_base, sh = 2 * (f & 31), piece = f >> 5;
        auto word = [&](int i) {
            return win[at][(i < 0 ? 0 : (i < kWalkPieces ? i : kWalkPieces - 1)) * kWave + lane];
        };
        const uint64_t moves = word(piece) >> sh | (word(piece + 1) << 1) << (63 - sh);
        // Bits up to `stop` end the walk: the window's first row, met again in
        // the next window, or rows above the block.
        const int stop = wr < 0 ? 1 - 2 * wr : 1;
        const uint64_t ends = moves | ~0ull >> (63 - stop);
        int p = 63, p2, entered = -1;
        do {
            entered = lane == l ? p : entered;
            p2 = p - __builtin_clzll(lane_mask64(ends, l) << (63 - p));
            p = (p2 - 1) | 1;
            --l;
        } while (min(l, p - stop - 1) >= 0);
        if (p2 <= stop) ++l;  // upwards to the window's end, the column goes on
        // each crossed column's cells: rows k_in .. k_out
        const int k_in = entered >> 1, e_in = entered < 0 ? 0 : entered;
        const int end = e_in - __builtin_clzll(ends << (63 - e_in));
        const int k_out = (end > stop ? end : stop + 2) >> 1;
        const int count = entered < 0 ? 0 : k_in - k_out + 1;
        const int upto = wave_prefix_sum(count), dn = __builtin_amdgcn_readlane(upto, kWave - 1);
        if (n + dn > cap) {
            status = -1;
            break;
        }
        if (pending && l < 0) settle();
        if (count > 0) {
            int64_t *to = rev + 2 * (n + dn - upto);  // columns to the right come first
            const int64_t col = c0 + (int64_t)s * kWave + lane + 1;
            for (int q = k_in; q >= k_out; --q, to += 2) {
                to[0] = r0 + wr + q;
                to[1] = col;
            }
        }
        n += dn;
        rr = wr + (p >> 1);
        cc = s * kWave + l + 1;
    }
    int64_t r = r0 + rr, c = c0 + cc;
    if (status == 0 && (r == 0 || c == 0)) {
        status = -1;
        if ((r == 0 && c == 0) || free_edges) {
            while (n < cap) {
                if (lane == 0) {
                    rev[2 * n] = r;
                    rev[2 * n + 1] = c;
                }
                ++n;
                if (r == 0 && c == 0) break;
                if (r > 0) --r;
                else --c;
            }
            status = (r == 0 && c == 0) ? 1 : -1;
        }
    }
    st[0] = r;  // every lane stores the same values
    st[1] = c;
    st[2] = n;
    st[3] = status;
}

// path[k] = rev[n - 1 - k] for the n cells, and *len = n (0 on failure).
__global__ void order_kernel(const int64_t *st, int64_t *path, int64_t *len)
{
    const int64_t n = st[3] == 1 ? st[2] : 0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n / 2; k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t a = k, b = n - 1 - k;
        const int64_t ai = path[2 * a], aj = path[2 * a + 1];
        path[2 * a] = path[2 * b];
        path[2 * a + 1] = path[2 * b + 1];
        path[2 * b] = ai;
        path[2 * b + 1] = aj;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *len = n;
}

__global__ void walk_init_kernel(int64_t *st, int64_t nA, int64_t nB)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st[0] = nA;
        st[1] = nB;
        st[2] = 0;
        st[3] = 0;
    }
}

}  // namespace

hipError_t launch_walk_init(int64_t *st, int64_t nA, int64_t nB, hipStream_t s)
{
    hipLaunchKernelGGL(walk_init_kernel, dim3(1), dim3(1), 0, s, st, nA, nB);
    return hipGetLastError();
}

hipError_t launch_walk(const void *dirs, int64_t r0, int64_t c0, int64_t nAt, int64_t *st, int64_t *rev, int64_t cap,
                       bool free_edges, hipStream_t s)
{
    hipLaunchKernelGGL(walk_kernel, dim3(1), dim3(kWave), 0, s, (const char *)dirs, r0, c0, (int)nAt, st, rev, cap,
                       free_edges ? 1 : 0);
    return hipGetLastError();
}

namespace {
// cells[i] = (i, i): row 0 or column 0 of the edit and indel distances.
__global__ void index_cells_kernel(double *cells, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += (int64_t)gridDim.x * blockDim.x) {
        cells[2 * i] = (double)i;
        cells[2 * i + 1] = (double)i;
    }
}

// LCS length from the indel distance: (nA + nB - I) / 2.
__global__ void lcs_finish_kernel(double *out, int64_t nA, int64_t nB)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) out[0] = ((double)(nA + nB) - out[0]) * 0.5;
}
}  // namespace

hipError_t launch_index_cells(void *cells, int64_t n, hipStream_t s)
{
    int64_t g = (n + 256) / 256;
    if (g > 1024) g = 1024;
    hipLaunchKernelGGL(index_cells_kernel, dim3((int)g), dim3(256), 0, s, (double *)cells, n);
    return hipGetLastError();
}

hipError_t launch_lcs_finish(double *out, int64_t nA, int64_t nB, hipStream_t s)
{
    hipLaunchKernelGGL(lcs_finish_kernel, dim3(1), dim3(1), 0, s, out, nA, nB);
    return hipGetLastError();
}

hipError_t launch_order(const int64_t *st, int64_t *path, int64_t *len, int64_t cap, hipStream_t s)
{
    int64_t g = (cap / 2 + 255) / 256;
    if (g < 1) g = 1;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(order_kernel, dim3((int)g), dim3(256), 0, s, st, path, len);
    return hipGetLastError();
}

}  // namespace twed

namespace twed {

namespace {
__global__ void zero32_kernel(uint32_t *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}
}  // namespace

hipError_t launch_zero32(uint32_t *p, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t g = (n + 255) / 256;
    if (g > 1024) g = 1024;
    hipLaunchKernelGGL(zero32_kernel, dim3((int)g), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

namespace {
struct FlagList {
    uint32_t *p[kMaxDirsBlocks];
};

__global__ void zero_flags_kernel(FlagList f, int64_t words)
{
    for (int64_t i = threadIdx.x; i < words; i += blockDim.x) f.p[blockIdx.x][i] = 0u;
}
}  // namespace

hipError_t launch_zero_flags(const DirsArgs *blocks, int n, int64_t words, hipStream_t s)
{
    if (n <= 0 || words <= 0) return hipSuccess;
    if (n > kMaxDirsBlocks) return hipErrorInvalidValue;
    FlagList f{};
    for (int i = 0; i < n; ++i) f.p[i] = blocks[i].flags;
    hipLaunchKernelGGL(zero_flags_kernel, dim3(n), dim3(256), 0, s, f, words);
    return hipGetLastError();
}

}  // namespace twed
