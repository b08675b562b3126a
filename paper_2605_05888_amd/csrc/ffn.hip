// Expert computation (Section II-A, step 3): grouped SwiGLU FFN over ragged,
// expert-contiguous row segments whose offsets live on the device.
//
//   GEMM1  a[m, f] = silu(xp[m,:] . W_gate[e,f,:]) * (xp[m,:] . W_up[e,f,:])
//   GEMM2  y[m, c] = a[m,:] . W_down[e,c,:]
//
// Both operands of both GEMMs have the reduction index contiguous, so every lane
// fetches its matrix-core operand (8 consecutive bf16 of one row) with a single
// 16-byte LDS read.  bf16 path: v_mfma_f32_32x32x16_bf16, fp32 accumulators,
// operand tiles brought global -> LDS without staging registers into a ring of
// XOR-swizzled units (grouped_gemm.h), one barrier per K tile.  GEMM1 keeps gate and up columns of the same f in one wavefront, so
// the activation is applied to the accumulators and `g`, `u` never reach memory.
//
// Launches with few rows and few tiles go to ffn_thin.hip (use_thin below), fp32 to ffn_f32.hip.
//
// Scheduling is device side: a small kernel turns seg_offsets into a tile table
// (expert, first row, end row, column tile), ordered so that tiles that run
// together share weight tiles; workgroup ids are spread so that each XCD's L2
// sees a compact patch of that order.  Nothing about the routing result is read
// on the host.
#include <atomic>

#include "common.h"
#include "ffn_gemm.h"
#include "ffn_thin.h"

namespace moe {

// ------------------------------------------------------------------------
// tile table
// ------------------------------------------------------------------------
constexpr int kSchedThreads = 256;
// relative cost of a light, a middle and a full tile, for sharing out the workgroup slots (middle: by its time; 246 random launches
// with all three take 0.995, 0.998, 1, 1.003 of the time with 4, 5, 6, 7)
constexpr int kLightCost = 3, kMidCost = 5, kHeavyCost = 7;
#ifndef MOE_ORDER_LONG_FIRST
#define MOE_ORDER_LONG_FIRST 1
#endif
// experts with at most this many rows go through the shallow tile geometry
constexpr int kLightRows = 64;

// Experts come in three classes by their rows (geometries in ffn_gemm.h): full tiles, middle, light; the table holds them in this
// order, and inside a class by expert, column tile, row tile.  The GEMM's persistent workgroups draw from two streams: full tiles,
// and light ones.  Middle tiles wait for memory as light ones do, and without full tiles they go with them (0.85 of the time with
// 256-row tiles in their place, 36 random launches).  Next to full tiles they do so where at least a sixth of all tiles are light:
// then a good part of the workgroups streams from the start (41 experts, 13 / 14 / 14 of the classes, K 3840, N 1216: 317 -> 244
// us).  With fewer light tiles they end the full tiles' stream, as the shorter ones (44 experts, 7 middle, 37 full, K 2688, N 1280:
// 249 -> 203).  211 random launches with middle and full tiles, time over that without middle tiles: always with the light ones
// 0.934, up to 1.24; always behind the full ones 0.915, up to 1.14; this 0.918, up to 1.08.
constexpr int kMidWithLight = 6;
// Row tiles of an expert with `rows` rows: a remainder of at most `extra` rows rides with the last
// full tile instead of forming a tile of its own.
__device__ __forceinline__ int row_tiles(int32_t rows, int BM, int extra)
{
    const int full = rows / BM, rest = rows - full * BM;
    return full > 0 && rest <= extra ? full : full + (rest > 0 ? 1 : 0);
}

__device__ __forceinline__ int32_t clamped_rows(const int32_t *seg_offsets, int e, int64_t M, int64_t &lo)
{
    int64_t hi = seg_offsets[e + 1];
    lo = seg_offsets[e];
    lo = lo < 0 ? 0 : (lo > M ? M : lo);
    hi = hi < lo ? lo : (hi > M ? M : hi);
    return (int32_t)(hi - lo);
}

// One launch builds the tables of both GEMMs: blockIdx.y picks the set of arguments.
struct TableArgs {
    int BM, extra; // rows of a tile; rows beyond them that the last full one may take
    int mid_rows;  // experts with more than light_rows and up to so many rows are one tile of the middle geometry
    int n_tiles, max_tiles, out_cols;
    TileTableHeader *hdr;
    TileEntry *table;
};

__global__ __launch_bounds__(kSchedThreads) void build_tile_table(
    const int32_t *__restrict__ seg_offsets, int E_local, int64_t M, int light_rows,
    TableArgs gemm1, TableArgs gemm2, int32_t *__restrict__ ready)
{
    const TableArgs &args = blockIdx.y == 0 ? gemm1 : gemm2;
    if (blockIdx.y == 0) // arrival counters of the row tiles start at zero with every schedule
        for (int64_t i = (int64_t)blockIdx.x * kSchedThreads + threadIdx.x; i < M; i += (int64_t)gridDim.x * kSchedThreads)
            ready[i] = 0;
    const int n_tiles = args.n_tiles, max_tiles = args.max_tiles, BM = args.BM, extra = args.extra;
    TileTableHeader *__restrict__ hdr = args.hdr;
    TileEntry *__restrict__ table = args.table;
    // first tile of each expert among those of its class: full [0], middle [1], light [2]
    constexpr int kClasses = 3;
    __shared__ int32_t start[kClasses][MOE_MAX_EXPERTS + 1];
    __shared__ int32_t wave_tot[kClasses][kSchedThreads / kWave];
    const int mid_rows = args.mid_rows;
    auto class_of = [&](int32_t rows) { return rows <= light_rows ? 2 : rows <= mid_rows ? 1 : 0; };
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    // exclusive scans of tiles per expert; a thread owns a contiguous run of experts
    const int per = (E_local + kSchedThreads - 1) / kSchedThreads;
    const int e_lo = tid * per;
    int32_t mine[kClasses] = {0, 0, 0};
    for (int j = 0; j < per; ++j) {
        const int e = e_lo + j;
        if (e < E_local) {
            int64_t lo;
            const int32_t rows = clamped_rows(seg_offsets, e, M, lo);
            mine[class_of(rows)] += row_tiles(rows, BM, extra) * n_tiles;
        }
    }
    int32_t inc[kClasses] = {mine[0], mine[1], mine[2]};
    for (int d = 1; d < kWave; d <<= 1) {
#pragma unroll
        for (int c = 0; c < kClasses; ++c) {
            const int32_t t = __shfl_up(inc[c], d);
            if (lane >= d)
                inc[c] += t;
        }
    }
    if (lane == kWave - 1) {
        for (int c = 0; c < kClasses; ++c)
            wave_tot[c][wave] = inc[c];
    }
    __syncthreads();
    int32_t run[kClasses] = {inc[0] - mine[0], inc[1] - mine[1], inc[2] - mine[2]};
    for (int w = 0; w < wave; ++w) {
        for (int c = 0; c < kClasses; ++c)
            run[c] += wave_tot[c][w];
    }
    for (int j = 0; j < per; ++j) {
        const int e = e_lo + j;
        if (e < E_local) {
            int64_t lo;
            const int32_t rows = clamped_rows(seg_offsets, e, M, lo);
            for (int c = 0; c < kClasses; ++c)
                start[c][e] = run[c];
            run[class_of(rows)] += row_tiles(rows, BM, extra) * n_tiles;
        }
    }
    if (tid == kSchedThreads - 1) { // the last thread's running sums are the totals
        for (int c = 0; c < kClasses; ++c)
            start[c][E_local] = run[c];
    }
    __syncthreads();
    // ends of the classes in the table (the bound cannot be reached by monotone offsets within [0, M])
    auto end_of = [&](int32_t tiles) { return tiles < max_tiles ? tiles : max_tiles; };
    const int32_t end_full = end_of(start[0][E_local]), end_mid = end_of(end_full + start[1][E_local]);
    const int32_t total = end_of(end_mid + start[2][E_local]);
    if (blockIdx.x == 0 && tid == 0) {
        const int32_t len0 = end_full > 0 && (int64_t)(total - end_mid) * kMidWithLight < total ? end_mid : end_full;
        hdr->len[0] = len0;
        hdr->len[1] = total - len0;
        hdr->end_full = end_full;
        hdr->end_mid = end_mid;
        // share of the workgroup slots that take stream 1 first: its tiles' share of the work
        const int64_t w_mid = (int64_t)(end_mid - end_full) * kMidCost;
        const int64_t wl = (int64_t)(total - end_mid) * kLightCost + (len0 == end_full ? w_mid : 0);
        const int64_t wh = (int64_t)end_full * kHeavyCost + (len0 == end_full ? 0 : w_mid);
        hdr->light_slots = len0 > 0 ? (int32_t)((32 * wl + (wl + wh) / 2) / (wl + wh)) : 32;
        hdr->done = 0;
        hdr->error = 0;
        hdr->epoch = 0;
        hdr->all_done = 0;
        hdr->magic = kTableMagic;
        hdr->rows = (int32_t)M;
        hdr->out_cols = args.out_cols;
        for (int s = 0; s < 2; ++s)
            for (int x = 0; x < kXcds; ++x)
                hdr->next[s][x] = 0;
    }
    for (int L = blockIdx.x * kSchedThreads + tid; L < total; L += gridDim.x * kSchedThreads) {
        const int c = L < end_full ? 0 : L < end_mid ? 1 : 2;
        const int32_t pos = L - (c == 0 ? 0 : c == 1 ? end_full : end_mid); // place among the tiles of its class
        int lo_e = 0, hi_e = E_local;             // last e with start[c][e] <= pos: the expert that owns it
        while (hi_e - lo_e > 1) {
            const int mid = (lo_e + hi_e) >> 1;
            if (start[c][mid] <= pos)
                lo_e = mid;
            else
                hi_e = mid;
        }
        const int e = lo_e;
        int64_t lo;
        const int32_t n_rows_e = clamped_rows(seg_offsets, e, M, lo);
        const int m_tiles = row_tiles(n_rows_e, BM, extra);
        // Inside an expert the tiles go in blocks of kOrderRows x kOrderCols (row tiles x column
        // tiles): the 32 tiles an XCD takes together (one per compute unit) then share 8 weight tiles
        // and 4 activation tiles in its L2, instead of 32 and one.
        const int local = pos - start[c][e];
        const int band_tiles = kOrderRows * n_tiles; // tiles of a full band of kOrderRows row tiles
        int rb = local / band_tiles;
        const int last_band = (m_tiles - 1) / kOrderRows;
        rb = rb > last_band ? last_band : rb;
        const int h = m_tiles - rb * kOrderRows < kOrderRows ? m_tiles - rb * kOrderRows : kOrderRows;
        const int in_band = local - rb * band_tiles;
        const int cb = in_band / (kOrderCols * h);
        const int in_block = in_band - cb * kOrderCols * h;
        TileEntry t;
        t.expert = e;
        int row_in_band = in_block % h, col_in_block = in_block / h;
#if MOE_ORDER_LONG_FIRST
        // The expert's last row tile takes another time than the full ones: longer when a remainder rides
        // with it, shorter when it is ragged.  Inside a block the long tiles are handed out first and the
        // short ones last, so that the workgroups that finish their previous tile early take the long ones
        // (it is the same set of tiles per block either way).
        if (rb == last_band && h > 1 && n_rows_e != m_tiles * BM) {
            const int wb = n_tiles - cb * kOrderCols < kOrderCols ? n_tiles - cb * kOrderCols : kOrderCols;
            const bool tall = n_rows_e > m_tiles * BM;
            const int first = tall ? wb : 0;                  // tiles of the odd row handed out before the others
            if (tall && in_block < wb) {
                row_in_band = h - 1, col_in_block = in_block;
            } else if (!tall && in_block >= wb * (h - 1)) {
                row_in_band = h - 1, col_in_block = in_block - wb * (h - 1);
            } else {
                row_in_band = (in_block - first) % (h - 1), col_in_block = (in_block - first) / (h - 1);
            }
        }
#endif
        const int row_tile = rb * kOrderRows + row_in_band;
        // rows that the expert's last tile computes beyond its BM
        const int ext = row_tile == m_tiles - 1 && n_rows_e > m_tiles * BM ? n_rows_e - m_tiles * BM : 0;
        t.n_tile = (cb * kOrderCols + col_in_block) | (ext << kTileColBits);
        t.m0 = (int32_t)lo + row_tile * BM;
        t.m_end = (int32_t)lo + n_rows_e;
        table[L] = t;
    }
}

// ------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------
// upper bound of the down projection's 256-column tiles up to which the narrow form is used
#ifndef MOE_NARROW_TILE_BOUND
#define MOE_NARROW_TILE_BOUND 256
#endif
constexpr int kNarrowTileBound = MOE_NARROW_TILE_BOUND;

struct FfnPlan {
    bool thin1, thin2; // GEMM1 / GEMM2 by ffn_thin.hip: that table holds row tiles only
    bool narrow2; // the down projection runs with NarrowSet
    int BM, out_cols1, out_cols2;
    int n_tiles1, n_tiles2, max_m_tiles1, max_m_tiles2;
    size_t off_a, off_hdr1, off_tab1, off_hdr2, off_tab2, off_ready, total;
};

// Few rows per expert, and so few of the tiled kernel's tiles that compute units stay idle: ffn_thin.hip.  GEMM1 / GEMM2,
// every expert with the rows given, tiled -> thin, us:
//   4 experts, H 2048, F 1408 (44 / 64 tiles):   1: 40 / 23 -> 16 / 12    16: 42 / 25 -> 17 / 12    32: 46 / 28 -> 20 / 12
//   8 experts, H 7168, F 2048 (128 / 448 tiles): 1: 136 / 63 -> 91 / 49   16: 135 / 63 -> 102 / 56  32: 140 / 64 -> 114 / 64
//   2 experts, H 4096, F 14336 (224 / 64 tiles): 1: 91 / 104 -> 85 / 49   16: 96 / 110 -> 101 / 59  32: 98 / 112 -> 116 / 67
//   8 experts, H 4096, F 14336 (896 / 256 tiles): 1: 352 / 159 -> 323 / 176                         32: 372 / 167 -> 415 / 220
// A tile of a short reduction is mostly start and end, hence the higher limit there.  With many experts (128 of H = F =
// 2880: 642 / 334 -> 830 / 405) thin workgroups are too short-lived themselves.  The bound on M keeps the worst case, all
// rows with one expert, at a few passes over its weights, all but the first from the caches.
// Where the lines lie: both forms on 4000 random launches that the lines take, 1 - 128 experts, K 512 - 16384, rows spread
// evenly, by Zipf's law or all with one expert: twice as fast in the median, 0.2 % of them more than 1 % slower.  Up to
// 64 tiles thin never lost.  Beyond that every block of columns reads the rows of A again, which counts with rows * K: 4
// experts, K 7168, N 4096, 31 rows each 82 -> 96, 16 experts, K 15488, N 896, 16 rows 120 -> 125, but 16 rows of K 6464 62
// -> 53.  Above 176 tiles long reductions lose, spread rows at least: 8 experts, K 5120, N 3264, 2 rows 62 -> 72, K 6976, N
// 8640, 1 row 137 -> 151, but 12 experts, K 3584, N 1728, 2 rows 76 -> 70.  Above 384 tiles of 256 weight rows the thin
// form's last round decides: 8 experts, N 6400, K 1280, 13 rows 64 -> 77, K 1984, 8 rows 86 -> 95, but 16 experts, N 3136, K
// 1024, 16 rows 36 -> 23.
constexpr int kThinMaxRows = 256;
// tiles: of the tiled form, tile_rows weight rows each
static bool use_thin(int64_t M, int64_t experts, int64_t tiles, int tile_rows, int64_t Kdim)
{
    if (M > kThinMaxRows || M > 32 * experts)
        return false;
    const int64_t reread = M * Kdim / (8192 * experts); // columns of A per expert, in units of 8192
    if (tiles <= 128)
        return tiles <= 64 || reread < 24;
    if (tiles <= 224 && M <= 4 * experts && (Kdim <= 4096 || (tiles <= 176 && reread < 3)))
        return true;
    if (M > 16 * experts || Kdim > 2048)
        return false;
    return tiles <= 384 || (tiles <= 448 && (tile_rows == 128 || Kdim <= 1024 || M <= 2 * experts));
}
// Workgroups of four blocks of weight rows instead of two read the rows of A half as often: better once there are some
// rows and enough workgroups (8 experts, H 7168, F 2048, 16 rows each, 512 of them: 114 -> 102 us; one row: 91 -> 91; 2
// experts, F 14336, 1 row: 85 -> 92; 128 of them, K 14336: 49 -> 81).
static bool wide_thin(int64_t M, int64_t experts, int64_t workgroups) { return M > 4 * experts && workgroups >= 384; }

// From so many columns on 32 rows, whose bytes bound the tiled form's stores, take 4 GiB, more than a byte count holds.  The thin
// form stores to 64-bit addresses and takes any number of rows (a pass over the weights for 64 of them).
constexpr int64_t kThinCols = (int64_t)1 << 26;

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

static FfnPlan make_plan(int64_t M, int64_t H, int64_t F, int E_local)
{
    FfnPlan p;
    p.BM = BigTile<true>::BM;
    p.out_cols1 = BigTile<true>::kOutCols; // GEMM1 writes BN/2 columns of `a` per tile
    p.narrow2 = (M / BigTile<false>::BM + E_local) * ceil_div(H, BigTile<false>::kOutCols) <= kNarrowTileBound;
    p.out_cols2 = p.narrow2 ? NarrowBig<false>::kOutCols : BigTile<false>::kOutCols;
    p.n_tiles1 = (int)ceil_div(F, p.out_cols1);
    p.n_tiles2 = (int)ceil_div(H, p.out_cols2);
    p.max_m_tiles1 = p.max_m_tiles2 = (int)(M / p.BM) + E_local;
    size_t o = 0;
    p.off_a = o;
    o = align_up(o + (size_t)M * F * 2, 256);
    p.off_hdr1 = o;
    o += kTileTableHeaderBytes;
    p.off_tab1 = o;
    o = align_up(o + (size_t)p.max_m_tiles1 * p.n_tiles1 * sizeof(TileEntry), 256);
    p.off_hdr2 = o;
    o += kTileTableHeaderBytes;
    p.off_tab2 = o;
    o = align_up(o + (size_t)p.max_m_tiles2 * p.n_tiles2 * sizeof(TileEntry), 256);
    p.off_ready = o; // per row: arrival counter of the row tile that starts there (dependency-driven launches)
    o = align_up(o + (size_t)M * sizeof(int32_t), 256);
    p.total = o;
    // (the workspace's layout is the tiled form's, so that its size keeps growing with M)
    const int thin_tiles = (int)(M / kThinRows + E_local < M ? M / kThinRows + E_local : M);
    const int64_t experts = E_local < M ? E_local : M;
    p.thin1 = (F >= kThinCols || use_thin(M, experts, experts * p.n_tiles1, 256, H)) && thin_tiles <= p.max_m_tiles1 * p.n_tiles1;
    p.thin2 = (H >= kThinCols || use_thin(M, experts, experts * p.n_tiles2, p.out_cols2, F)) && thin_tiles <= p.max_m_tiles2 * p.n_tiles2;
    if (p.thin1) {
        p.max_m_tiles1 = thin_tiles, p.n_tiles1 = 1;
        p.out_cols1 = wide_thin(M, experts, experts * ceil_div(F, 32)) ? 32 : 16;
    }
    if (p.thin2) {
        p.max_m_tiles2 = thin_tiles, p.n_tiles2 = 1;
        p.out_cols2 = wide_thin(M, experts, experts * ceil_div(H, 64)) ? 64 : 32;
    }
    return p;
}

size_t ffn_workspace_bytes(int64_t M, int64_t H, int64_t F, int E_local, int dtype)
{
    if (dtype == MOE_F32)
        return align_up((size_t)M * F * 4, 256);
    return make_plan(M, H, F, E_local).total;
}

// Per-device facts, cached on first use.  Entries are written with relaxed atomics and every writer
// stores the same value, so threads that race on the first call of a device do no harm.
constexpr int kMaxDevices = 64;
static int current_device()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
        return -1;
    return dev;
}

static int compute_units()
{
    static std::atomic<int> cus[kMaxDevices];
    const int dev = current_device();
    int n = dev >= 0 ? cus[dev].load(std::memory_order_relaxed) : 0;
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev < 0 ? 0 : dev) != hipSuccess || n <= 0)
            return kXcds * 32;
        if (dev >= 0)
            cus[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

int workgroup_slots()
{
    int g = compute_units() / kXcds * kXcds; // (LDS: one workgroup per compute unit)
    if (g > kMaxGemmWorkgroups)
        g = kMaxGemmWorkgroups / kXcds * kXcds;
    return g < kXcds ? kXcds : g;
}

void allow_lds(const void *kern, size_t lds_bytes, std::atomic<uint64_t> &raised)
{
    const int dev = current_device();
    if (dev < 0 || !(raised.load(std::memory_order_relaxed) >> dev & 1)) {
        (void)hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (dev >= 0)
            raised.fetch_or(uint64_t(1) << dev, std::memory_order_relaxed);
    }
}

// Weight rows a multiple of 4 KiB apart: workgroups that all start at column 0 ask the same few memory channels, and
// being equally fast they go on doing so.  Such a launch starts every column tile (experts with one shallow row tile) or
// block of eight (so that tiles that share operands in an XCD's L2 stay together) 2 KiB further on.  GEMM1 of 64 experts,
// F 2560, 16 / 144 rows each, us: K 2048 276 / 349 -> 230 / 312, K 4096 481 / 645 -> 430 / 566, K 6144 716 / 949 -> 640 /
// 831, K 8192 904 / 1192 -> 843 / 1088.  Other strides spread by themselves and lose up to 4 % (K 2560, 3072, 3584).  Above
// 8192 the rows of A that the turned tiles share no longer fit the L2 (K 14336, 256 rows: 268 -> 281).  From 256 rows per
// expert on the matrix cores bound the launch, and it takes channels that streaming would not fill where there are fewer
// tiles than compute units, or one or two starting points only: of 900 random launches (K 2048 - 8192, unturned -> turned)
// those within all the lines take 0.95 of the time in the median, below 64 rows 0.93; with 256 to 600 rows it is 1.00, with
// fewer than 192 tiles 1.01 (64 experts, K 4096, N 256, 40 rows 53 -> 65), with two column tiles 1.01 (256 experts, K 2048,
// N 256, 12 rows 98 -> 104).
constexpr int kChannelStride = 4096, kTurnTiles = 16, kMaxTurnedK = 8192, kMinTurnedTiles = 192;
constexpr int64_t kMaxTurnedRows = 256;

// tiles: column tiles of the launch's tile width
static int turn_of(int64_t M, int E_local, int Kdim, int64_t tiles)
{
    const int64_t experts = E_local < M ? E_local : M; // at most so many have rows
    const bool turned = (int64_t)Kdim * 2 % kChannelStride == 0 && Kdim <= kMaxTurnedK && M < kMaxTurnedRows * E_local &&
                        tiles > 2 && tiles * experts >= kMinTurnedTiles;
    return turned ? kTurnTiles : 0;
}

static GemmArgs gemm_args(const uint16_t *A, int64_t M, int E_local, int Kdim, int Ndim, const uint16_t *B0, const uint16_t *B1,
                          uint16_t *C, TileTableHeader *hdr, const TileEntry *table, int out_cols)
{
    GemmArgs g = {};
    g.A = A, g.M = M, g.Kdim = Kdim, g.Ndim = Ndim, g.B0 = B0, g.B1 = B1, g.C = C, g.hdr = hdr, g.table = table;
    g.gather_div = 1;
    g.k_turn = turn_of(M, E_local, Kdim, ceil_div(Ndim, out_cols));
    return g;
}

int check_ffn_shape(int dtype, int64_t H, int64_t F)
{
    if (dtype == MOE_BF16 && (H % 64 != 0 || F % 64 != 0))
        return fail(MOE_ERR_UNSUPPORTED,
                    "bf16 moe_grouped_ffn needs H and F to be multiples of 64 (got H=%lld, F=%lld)",
                    (long long)H, (long long)F);
    return MOE_OK;
}

// polls (about a microsecond each) a dependent tile spends on its rows before it gives up: seconds
constexpr int64_t kDefaultWaitLimit = (int64_t)1 << 22;

struct FfnWorkspace {
    uint16_t *a;
    TileTableHeader *hdr1, *hdr2;
    TileEntry *tab1, *tab2;
    int max1, max2;
    int32_t *ready;
};

static FfnWorkspace carve(const FfnPlan &p, void *ws)
{
    unsigned char *w = static_cast<unsigned char *>(ws);
    FfnWorkspace k;
    k.a = reinterpret_cast<uint16_t *>(w + p.off_a);
    k.hdr1 = reinterpret_cast<TileTableHeader *>(w + p.off_hdr1);
    k.tab1 = reinterpret_cast<TileEntry *>(w + p.off_tab1);
    k.hdr2 = reinterpret_cast<TileTableHeader *>(w + p.off_hdr2);
    k.tab2 = reinterpret_cast<TileEntry *>(w + p.off_tab2);
    k.max1 = p.max_m_tiles1 * p.n_tiles1;
    k.max2 = p.max_m_tiles2 * p.n_tiles2;
    k.ready = reinterpret_cast<int32_t *>(w + p.off_ready);
    return k;
}


int launch_ffn_schedule(int dtype, int64_t M, int64_t H, int64_t F, int E_local,
                        const int32_t *seg_offsets, void *ws, hipStream_t st)
{
    if (dtype == MOE_F32)
        return MOE_OK; // the fp32 kernels look their expert up per row
    const FfnPlan p = make_plan(M, H, F, E_local);
    const FfnWorkspace k = carve(p, ws);
    const int max_both = k.max1 > k.max2 ? k.max1 : k.max2;
    hipLaunchKernelGGL(build_tile_table, dim3((unsigned)ceil_div(max_both, kSchedThreads), 2),
                       dim3(kSchedThreads), 0, st, seg_offsets, E_local, M, kLightRows,
                       TableArgs{p.thin1 ? kThinRows : p.BM, p.thin1 ? 0 : BigTile<true>::kExtra, p.thin1 ? 0 : kMidRows, p.n_tiles1, k.max1, p.out_cols1, k.hdr1, k.tab1},
                       TableArgs{p.thin2 ? kThinRows : p.BM, p.thin2 ? 0 : BigTile<false>::kExtra, p.thin2 ? 0 : kMidRows, p.n_tiles2, k.max2, p.out_cols2, k.hdr2, k.tab2},
                       k.ready);
    return check_launch("moe_ffn_schedule");
}

// gather_rows == nullptr: xp holds the M rows.  Otherwise xp is x[N, H] and row m is x[gather_rows[m] / K].
int launch_ffn_gate_up(const void *xp, int dtype, int64_t M, int64_t H, int64_t F, int E_local,
                       const int32_t *seg_offsets, const void *W_gate, const void *W_up, void *ws,
                       hipStream_t st, const int32_t *gather_rows, int K, int64_t N)
{
    if (dtype == MOE_F32) {
        return launch_ffn_f32_gate_up(static_cast<const float *>(xp), M, H, F, E_local, seg_offsets,
                                      static_cast<const float *>(W_gate), static_cast<const float *>(W_up),
                                      static_cast<float *>(ws), gather_rows, K, st);
    }
    const FfnPlan p = make_plan(M, H, F, E_local);
    const FfnWorkspace k = carve(p, ws);
    const uint16_t *xpb = static_cast<const uint16_t *>(xp);
    const uint16_t *wg = static_cast<const uint16_t *>(W_gate), *wu = static_cast<const uint16_t *>(W_up);
    if (p.thin1) {
        launch_thin_gate_up(xpb, M, H, F, wg, wu, k.a, k.hdr1, k.tab1, p.max_m_tiles1, p.out_cols1, gather_rows, K, (uint32_t)(N * H * 2), st);
        return check_launch("moe_ffn_gate_up");
    }
    GemmArgs g = gemm_args(xpb, M, E_local, (int)H, (int)F, wg, wu, k.a, k.hdr1, k.tab1, p.out_cols1);
    if (gather_rows) {
        g.gather_rows = gather_rows, g.gather_div = K, g.gather_bytes = (uint32_t)(N * H * 2);
        launch_gate_up_gather(g, st);
    } else {
        launch_gate_up(g, st);
    }
    return check_launch("moe_ffn_gate_up");
}

int launch_ffn_down(int dtype, int64_t M, int64_t H, int64_t F, int E_local,
                    const int32_t *seg_offsets, const void *W_down, void *y, void *ws, hipStream_t st)
{
    if (dtype == MOE_F32) {
        return launch_ffn_f32_down(static_cast<const float *>(ws), M, H, F, E_local, seg_offsets,
                                   static_cast<const float *>(W_down), static_cast<float *>(y), st);
    }
    const FfnPlan p = make_plan(M, H, F, E_local);
    const FfnWorkspace k = carve(p, ws);
    const uint16_t *wd = static_cast<const uint16_t *>(W_down);
    uint16_t *yb = static_cast<uint16_t *>(y);
    if (p.thin2) {
        launch_thin_down(k.a, M, H, F, wd, yb, k.hdr2, k.tab2, p.max_m_tiles2, p.out_cols2, nullptr, 1, nullptr, st);
        return check_launch("moe_ffn_down");
    }
    const GemmArgs g = gemm_args(k.a, M, E_local, (int)F, (int)H, wd, nullptr, yb, k.hdr2, k.tab2, p.out_cols2);
    if (p.narrow2)
        launch_down_narrow(g, st);
    else
        launch_down(g, st);
    return check_launch("moe_ffn_down");
}

// Both GEMMs in one launch, the second consuming the first's rows tile by tile (after launch_ffn_schedule).
int launch_ffn_gate_up_down(const void *xp, int64_t M, int64_t H, int64_t F, int E_local, const void *W_gate,
                            const void *W_up, const void *W_down, void *y, void *ws, int64_t wait_limit,
                            hipStream_t st)
{
    const FfnPlan p = make_plan(M, H, F, E_local);
    const FfnWorkspace k = carve(p, ws);
    if (p.thin1 || p.thin2) { // a table of another form: two launches
        const int rc = launch_ffn_gate_up(xp, MOE_BF16, M, H, F, E_local, nullptr, W_gate, W_up, ws, st, nullptr, 1, 0);
        return rc != MOE_OK ? rc : launch_ffn_down(MOE_BF16, M, H, F, E_local, nullptr, W_down, y, ws, st);
    }
    GemmArgs g1 = gemm_args(static_cast<const uint16_t *>(xp), M, E_local, (int)H, (int)F, static_cast<const uint16_t *>(W_gate),
                            static_cast<const uint16_t *>(W_up), k.a, k.hdr1, k.tab1, p.out_cols1);
    GemmArgs g2 = gemm_args(k.a, M, E_local, (int)F, (int)H, static_cast<const uint16_t *>(W_down), nullptr,
                            static_cast<uint16_t *>(y), k.hdr2, k.tab2, p.out_cols2);
    g1.ready = g2.ready = k.ready;
    g1.hdr_dep = g2.hdr_dep = k.hdr1;
    g1.ready_per_launch = g2.ready_per_launch = BigTile<true>::kWaves * p.n_tiles1;
    g1.wait_limit = g2.wait_limit = wait_limit > 0 ? wait_limit : kDefaultWaitLimit;
    if (p.narrow2)
        launch_gate_up_and_down_narrow(g1, g2, st);
    else
        launch_gate_up_and_down(g1, g2, st);
    return check_launch("moe_ffn_gate_up_down");
}

// Waits for `st`, then reads the two tables' error words.
int ffn_status(int64_t M, int64_t H, int64_t F, int E_local, const void *ws, hipStream_t st)
{
    const FfnPlan p = make_plan(M, H, F, E_local);
    const FfnWorkspace k = carve(p, const_cast<void *>(ws));
    int32_t err[2] = {0, 0};
    if (hipMemcpyAsync(&err[0], &k.hdr1->error, sizeof(int32_t), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipMemcpyAsync(&err[1], &k.hdr2->error, sizeof(int32_t), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return check_launch("moe_ffn_status") != MOE_OK ? MOE_ERR_LAUNCH
                                                        : fail(MOE_ERR_LAUNCH, "moe_ffn_status: copy failed");
    for (int g = 0; g < 2; ++g) {
        if (err[g] == kNoScheduleError)
            return fail(MOE_ERR_STATE, "GEMM%d ran over a workspace that moe_ffn_schedule had not filled for M=%lld "
                                       "(and this H, F, E_local)", g + 1, (long long)M);
        if (err[g] == kDependencyTimeout)
            return fail(MOE_ERR_STATE, "GEMM%d gave up waiting for rows of the first GEMM (poll limit reached); "
                                       "its output is incomplete", g + 1);
    }
    return MOE_OK;
}

// ------------------------------------------------------------------------
// down projection with the combine in its epilogue
// ------------------------------------------------------------------------
__global__ void fill_zero_16B(u32x4 *__restrict__ p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        p[i] = u32x4{0u, 0u, 0u, 0u};
}

// sums[N*H] fp32 -> out[N*H] bf16, eight elements per thread
__global__ void round_sums_bf16(const f32x4 *__restrict__ sums, u32x4 *__restrict__ out, int64_t n8)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n8)
        return;
    const f32x4 a = __builtin_nontemporal_load(&sums[2 * i]), b = __builtin_nontemporal_load(&sums[2 * i + 1]);
    u32x4 o;
    o[0] = pack_bf16x2(a[0], a[1]);
    o[1] = pack_bf16x2(a[2], a[3]);
    o[2] = pack_bf16x2(b[0], b[1]);
    o[3] = pack_bf16x2(b[2], b[3]);
    out[i] = o;
}

int launch_ffn_down_combine(int64_t N, int K, int64_t H, int64_t F, int E_local, const void *W_down,
                            const int32_t *row_of_slot, const float *topk_w, float *sums, void *out,
                            void *ws, hipStream_t st)
{
    const int64_t M = N * K;
    const FfnPlan p = make_plan(M, H, F, E_local);
    const FfnWorkspace k = carve(p, ws);
    const int64_t n16 = N * H / 4, n8 = N * H / 8;
    hipLaunchKernelGGL(fill_zero_16B, dim3((unsigned)ceil_div(n16, 256)), dim3(256), 0, st,
                       reinterpret_cast<u32x4 *>(sums), n16);
    const uint16_t *wd = static_cast<const uint16_t *>(W_down);
    if (p.thin2) {
        launch_thin_down(k.a, M, H, F, wd, sums, k.hdr2, k.tab2, p.max_m_tiles2, p.out_cols2, row_of_slot, K, topk_w, st);
    } else {
        GemmArgs g = gemm_args(k.a, M, E_local, (int)F, (int)H, wd, nullptr, reinterpret_cast<uint16_t *>(sums), k.hdr2, k.tab2,
                               p.out_cols2);
        g.gather_rows = row_of_slot, g.gather_div = K, g.scatter_w = topk_w;
        if (p.narrow2)
            launch_down_scatter_narrow(g, st);
        else
            launch_down_scatter(g, st);
    }
    hipLaunchKernelGGL(round_sums_bf16, dim3((unsigned)ceil_div(n8, 256)), dim3(256), 0, st,
                       reinterpret_cast<const f32x4 *>(sums), static_cast<u32x4 *>(out), n8);
    return check_launch("moe_ffn_down_combine");
}

}  // namespace moe
