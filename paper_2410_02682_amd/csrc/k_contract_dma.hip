// Block contraction with direct global->LDS staging: which shapes take it, with which tiles (the kernel is in k_contract_dma.h),
// and the aggregation of the tile-ordered partial slabs it writes.
#include <algorithm>

#include "k_contract_dma.h"

namespace eg {

bool contract_dma_eligible(const ContractParams &p)
{
    if (p.ragged || (p.in_dtype != EG_BF16 && p.in_dtype != EG_F32)) return false;
    const bool f32 = p.in_dtype == EG_F32;
    const int64_t es = f32 ? 4 : 2, epc = 16 / es, bk = 128 / es;
    if (p.m.n < 1 || p.n.n < 1 || p.k.n < 1) return false;
    // every run of the innermost K label starts a stage; along a K-contiguous operand 16-byte chunks must be whole and
    // aligned, so runs are whole chunks and start on chunk boundaries
    const int64_t run = p.k.n == 1 ? p.K : p.k.ext[p.k.n - 1];
    (void)bk;
    if (p.a_kcontig || p.b_kcontig) {
        if (run % epc) return false;
        for (int i = 0; i + 1 < p.k.n; i++)
            if ((p.a_kcontig && p.k.s0[i] % epc) || (p.b_kcontig && p.k.s1[i] % epc)) return false;
    }
    // Lane offsets count from the tile's first row and must stay below 2^31 bytes: rows of a tile must not lie before
    // its first row (strides nested, outermost first), and 256 rows plus the k-rows of a stage must span less.
    auto tile_span = [](const DimList &g) -> int64_t {            // largest offset of a row within 255 rows of another
        int64_t inner = 1, span = 0;
        for (int i = g.n - 1; i >= 0; i--) {
            if (g.s0[i] < 0) return -1;
            if (i + 1 < g.n && g.s0[i] < g.s0[i + 1] * g.ext[i + 1]) return -1;
            const int64_t steps = std::min<int64_t>(g.ext[i] - 1, 255 / inner + 1);
            span += steps * g.s0[i];
            inner *= g.ext[i];
        }
        return span;
    };
    const int kin = p.k.n - 1;
    const int64_t sx = tile_span(p.m), sy = tile_span(p.n);
    if (sx < 0 || sy < 0) return false;
    const int64_t lim = ((1ll << 31) - 256) / es;                           // elements
    if (sx + (p.a_kcontig ? 64 : 64 * std::max<int64_t>(p.k.s0[kin], 1)) >= lim) return false;
    if (sy + (p.b_kcontig ? 64 : 64 * std::max<int64_t>(p.k.s1[kin], 1)) >= lim) return false;
    if (p.a_kcontig ? p.k.s0[p.k.n - 1] != 1 : (p.m.s0[p.m.n - 1] != 1 || p.m.ext[p.m.n - 1] % epc)) return false;
    if (p.b_kcontig ? p.k.s1[p.k.n - 1] != 1 : (p.n.s0[p.n.n - 1] != 1 || p.n.ext[p.n.n - 1] % epc)) return false;
    if (!p.a_kcontig && p.M < epc) return false;
    if (!p.b_kcontig && p.N < epc) return false;
    if (((uintptr_t)p.x & 15) || ((uintptr_t)p.y & 15)) return false;
    return true;
}

// compute units of the current device, rounded down to whole XCD rounds (0: the device cannot be queried)
static int dma_cu_count()
{
    static int n_cu = 0;
    if (!n_cu) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
        n_cu = prop.multiProcessorCount > 8 ? prop.multiProcessorCount / 8 * 8 : 8;
    }
    return n_cu;
}

void contract_dma_variant(const ContractParams &p, int &tm, int &tn, int &nw, int &ns)
{
    const int n_cu = dma_cu_count();
    // Tile shape.  256 x 256, one workgroup per compute unit, is the fastest per flop on long reductions (fewest bytes into LDS per
    // flop, full 128-byte lines from operands contiguous along K).  256 x 128 with half-depth stages runs two workgroups per unit,
    // one's per-tile phases under the other's MFMAs; its main loop is a fifth slower (64-byte requests for operands contiguous
    // along K, a barrier every 16 MFMAs), so it is taken only where tiles are mostly per-tile work or where the wider tile would be
    // padding: reductions of up to 128 elements (config 4's scores: 0.42 -> 0.38 ms) and blocks whose last 256 columns are at most
    // half filled (config 4's P x V with 128 columns: 0.31 -> 0.30 ms).  128 x 128 tiles, two workgroups per unit, are taken
    // when they are all resident at once, i.e. when larger tiles would leave at least half of the compute units without work
    // (measured: 64 tiles of 256 x 256 ran 1.5-1.8x faster as 256 small ones; 160 of them 1.4x slower as 640 small ones, which
    // need a second round).
    const bool f32 = p.in_dtype == EG_F32;
    const int64_t tuples = p.n_tuples * p.n_batch;
    auto count = [&](int tm, int tn) { return tuples * ((p.M + tm - 1) / tm) * ((p.N + tn - 1) / tn); };
    const int64_t small = count(128, 128);
    const int64_t ntail = p.N % 256;
    if (p.carry) tm = tn = 256;
    else if (small <= 2 * n_cu || p.n_totals > 1) tm = tn = 128;
    else if (!f32 && (p.K <= 128 || (ntail > 0 && ntail <= 128 && p.N < 1024))) { tm = 256; tn = 128; }
    else if (4 * count(256, 256) * 10 > small * 14) tm = tn = 128;
    else tm = tn = 256;
    if (p.force_tile_m && p.force_tile_n) { tm = p.force_tile_m; tn = p.force_tile_n; }   // tr_set_contract_variant: comparisons and tests
    if (f32 && tm != tn) tn = tm;
    nw = (tm == 256 && tn == 256 && (f32 || p.force_waves != 4)) ? 8 : 4;
    ns = tm == 256 && tn == 128 ? 3 : 2;
    // 128 x 128 tiles of which each compute unit has one at most: eight waves in two groups and four stages instead of four waves and
    // two (781 cycles per stage instead of 1457, but 1 us more before and after: 2048 x 2048 x 2048 33.6 -> 27.3 us, 2048 x 256 x
    // 2048 12.0 -> 12.9).  Not with partial slabs, whose tile order is that of four waves, nor for fp32, whose MFMAs take the
    // time of a stage four times over.
    if (tm == 128 && tn == 128 && !f32 && !p.out.slab_elems && small <= n_cu && p.force_waves != 4 && p.K * std::max(p.n_totals, 1) >= 512) { nw = 8; ns = 4; }
}

// Does a contraction with n_agg blocks along its aggregated labels run faster when one workgroup walks over a tile's blocks and keeps
// the totals of their sums (128 x 128 tiles: totals and sums together take the registers that 256 x 256 tiles need for the sums
// alone), than as partial slabs and an aggregation?  p: the parameters of the latter.  The sums are the same in the same order (with
// four stages the two groups' halves are added last).  Estimated from these rates, in us: a stage of a 128 x 128 tile 0.45 with four
// stages in LDS, 0.65 with two, 1.0 for two tiles at once, of a 256 x 256 tile 1.5, 2.5 for a tile's slab, and the slabs' way through memory at 5.3 TB/s.
//                                                            slabs        totals
//   8192 x (8 x 512) x 4096 to fp32                         342 + 216       302
//   4096 x (8 x 512) x 1024 to fp32                          58 + 28         45
//   65536 x (16 x 1024) x 4096 to fp32                     9000 + 3240     9600
//   8192 x (8 x 1376) x 4096 to fp32                        705 + 212       790
//   2048 x (2 x 1024) x 2048 to bf16                         28 + 12         27
//   8192 x (2 x 4096) x 8192 to bf16                        860 + 115      1150
//   512 x (2 x 1840) x 1536 to bf16                              34.4        38.3
//   1024 x (8 x 12800) x 10240 to bf16                     1860 + 56          -      (160 large tiles: the pieces fill the chip)
// Under 32 tiles the blocks' own workgroups are worth more than the launch that is saved (unless the reduction is a few stages long).
// While the totals' tiles fit the compute units once, both ways are estimated to a few percent instead, with what a block costs that is
// walked over (its offsets, the folding of its sums) and what an aggregation does for small slabs: 420 shapes of 16 to 1536
// elements a block and 140 of 1024 to 8192, each on both ways; the way taken is 0.2 % slower than the better one on average and nowhere more
// than 4 % slower than slabs, apart from two shapes (11 and 6 %).  (2632 x (16 x 128) x 144 to fp32: slabs 22.8 us, totals 32.0; 4608 x
// (3 x 1536) x 952 29.9 and 39.5; 696 x (4 x 320) x 648 13.8 and 17.7; 1072 x (16 x 128) x 2968 85 and 37.)
bool contract_totals_pay(const ContractParams &p, int64_t n_agg, int out_bytes)
{
    const int n_cu = dma_cu_count();
    if (!n_cu || n_agg < 2 || n_agg > INT32_MAX || p.n_tuples % n_agg) return false;
    if (p.force_tile_m || p.force_tile_n) return false;                   // comparisons of tile shapes are about the two-stage path
    const bool f32 = p.in_dtype == EG_F32;
    const int64_t outs = p.n_tuples / n_agg * p.n_batch;
    auto count = [&](int t) { return outs * ((p.M + t - 1) / t) * ((p.N + t - 1) / t); };
    auto rounds = [](int64_t tiles, int64_t wgs) { return (double)((tiles + wgs - 1) / wgs); };
    const int64_t small = count(128), large = count(256);
    if (small < 32 || small * n_agg >= (1ll << 31)) return false;
    if (p.force_kernel == 2) return true;                                  // asked for by name: this form of the kernel at any such size
    const double n = (double)n_agg, stages = (double)((p.K * (f32 ? 4 : 2) + 127) / 128);
    if (small <= n_cu) {
        const double mb = (double)outs * p.M * p.N * (4 * n + out_bytes) * 1e-6;
        const double totals = f32 ? 8 + n * (2.1 * stages + 0.6) : p.K * n_agg >= 512 ? 7.2 + n * (0.42 * stages + 0.8) : 6 + n * (0.52 * stages + 0.65);
        int tm, tn, nw, ns;
        contract_dma_variant(p, tm, tn, nw, ns);                          // the blocks' own tiles
        const int64_t tiles = outs * n_agg * ((p.M + tm - 1) / tm) * ((p.N + tn - 1) / tn);
        double slabs;
        if (tm == 256 && tn == 256) slabs = f32 ? 13.4 + rounds(tiles, n_cu) * (2.7 + 6.5 * stages) + 0.23 * mb + 0.15 * n : 9.1 + rounds(tiles, n_cu) * (2.85 + 1.06 * stages) + 0.28 * mb;
        else if (tm == 256) slabs = 12.9 + rounds(tiles, 2 * n_cu) * (0.23 + 1.07 * stages) + 0.234 * mb + 0.17 * n;
        else if (tiles <= n_cu) slabs = (f32 ? 8 + 2.1 * stages : 6.6 + 0.525 * stages) + 0.44 * mb + 0.3 * n;
        else if (tiles <= 2 * n_cu) slabs = f32 ? 7.9 + 3.4 * stages + 0.37 * mb + 0.6 * n : 9.9 + 0.57 * stages + 0.32 * mb + 0.23 * n;
        else slabs = 9.9 + rounds(tiles, 2 * n_cu) * (1.5 + (f32 ? 4.1 : 1.0) * stages) + 0.28 * mb;
        return totals < slabs;
    }
    const double two = f32 ? 4.1 : 1.0, big = f32 ? 8.0 : 1.5;                              // us per stage: two 128 x 128 tiles, a 256 x 256 tile
    const double totals = rounds(small, 2 * n_cu) * (two * stages * n + 2.5);
    const double join = small * n_agg <= 2 * n_cu ? two * stages : rounds(large * n_agg, n_cu) * (big * stages + 2.5);
    const double bytes = (double)outs * p.M * p.N * (4 * n + out_bytes);
    return totals < join + 5 + bytes / 5.3e6;
}

// Two blocks of long reductions on whole 256 x 256 tiles: a workgroup multiplies a tile's blocks one after the other and the first
// one's sums wait for the second's in the first slab.  Saves the other slab's way through memory and the aggregation, for a read
// (some 12 us per tile) that nothing covers.  us, two blocks of K (slabs and aggregation / totals in registers / this):
//   4096 x 4096    K = 1024 109 / 75 / 86      2048 155 / 134 / 132    4096 248 / 254 / 226
//   8192 x 4096    K = 1024 197 / 141 / 155    2048 291 / 264 / 246    4096 481 / 495 / 439
//   16384 x 4096   K = 1024 372 / 280 / 283    2048 569 / 522 / 486    4096 973 / 1026 / 937
//   5120 x 4096    K = 4096 333 / 310 / 373    (a second round of 64 tiles, twice as long: whole rounds only)
// Four blocks, whose totals are read and written in between: 491 / 527 / 478 at 4096 x 4096 of K = 4096, 1122 / 1046 / 1132 at 16384 x
// 4096 of 2048; left to the others.
bool contract_carry_pays(const ContractParams &p, int64_t n_agg)
{
    const int n_cu = dma_cu_count();
    if (!n_cu || n_agg != 2 || p.n_tuples % 2 || p.in_dtype == EG_F32 || p.M % 256 || p.N % 256 || p.K < 2048) return false;
    if (p.force_tile_m || p.force_tile_n || p.force_waves == 4) return false;
    int tm, tn, nw, ns;
    contract_dma_variant(p, tm, tn, nw, ns);
    if (tm != 256 || tn != 256) return false;
    const int64_t tiles = p.n_tuples / 2 * p.n_batch * (p.M / 256) * (p.N / 256);
    return 2 * tiles < (1ll << 31) && 2 * ((tiles + n_cu - 1) / n_cu) <= (2 * tiles + n_cu - 1) / n_cu;
}

int launch_contract_dma(ContractParams &p, void *stream)
{
    if (!p.x || !p.y || !p.out.ptr) return fail(EG_ERR_NULL, "contraction: NULL operand");
    if (!contract_dma_eligible(p)) return fail(EG_ERR_LIMIT, "contraction: shape not eligible for the direct-to-LDS kernel");
    const int n_cu = dma_cu_count();
    if (!n_cu) return fail(EG_ERR_HIP, "cannot query the device");
    const bool f32 = p.in_dtype == EG_F32;
    const int64_t tuples = p.n_tuples * p.n_batch;
    int tm, tn, nw, ns;
    contract_dma_variant(p, tm, tn, nw, ns);
    if (p.tile_order && ns == 4) return fail(EG_ERR_LIMIT, "contraction: the four-stage kernel has no tile order");
    if (p.carry && (tm != 256 || tn != 256 || nw != 8 || f32 || p.n_totals != 2 || p.out.slab_elems || p.tile_order || p.M % 256 || p.N % 256)) return fail(EG_ERR_LIMIT, "contraction: sums wait in memory for those of a second block, whole 256 x 256 tiles of bf16 operands");
    if (!p.carry && p.n_totals > 1 && (tm != 128 || tn != 128 || p.out.slab_elems)) return fail(EG_ERR_LIMIT, "contraction: totals are kept by 128 x 128 tiles, in place of partial slabs");
    if (p.tile_order && (p.M % tm || p.N % tn || !p.out.slab_elems)) return fail(EG_ERR_LIMIT, "contraction: tile-ordered partial slabs need whole tiles");
    // the variant: stage depth and waves follow from the tile shape
    const int kb = (tm == 256 && tn == 128) ? 64 : 128;
    p.tiles_m = (int32_t)((p.M + tm - 1) / tm);
    p.tiles_n = (int32_t)((p.N + tn - 1) / tn);
    const int64_t wgs = tuples * p.tiles_m * p.tiles_n;
    if (wgs < 1 || wgs >= (1ll << 31)) return fail(EG_ERR_LIMIT, "contraction has %lld output tiles", (long long)wgs);
    // persistent workgroups: as many as fit the chip at once, a multiple of 8 so that every XCD gets the same number
    const int64_t resident = (2 * dma::lds_bytes(tm, tn, kb, 2, nw, ns) <= 160 * 1024 ? 2 : 1) * (int64_t)n_cu;
    p.total_tiles = (int32_t)wgs;
    p.grid = (int32_t)(wgs < resident ? wgs : resident);
    // wide epilogue stores need Z contiguous along the innermost N label and every other Z offset a multiple of 8 elements
    bool vec = p.n.s1[p.n.n - 1] == 1 && p.n.ext[p.n.n - 1] % 8 == 0 && ((uintptr_t)p.out.ptr & 15) == 0 && p.out.slab_elems % 8 == 0;
    for (int i = 0; i < p.m.n; i++) vec = vec && p.m.s1[i] % 8 == 0;
    for (int i = 0; i + 1 < p.n.n; i++) vec = vec && p.n.s1[i] % 8 == 0;
    for (int i = 0; i < p.batch.n; i++) vec = vec && p.batch.s2[i] % 8 == 0;
    for (int l = 0; l < p.ts.n; l++) vec = vec && p.ts.step_z[l] % 8 == 0;
    p.out_vec = vec ? 1 : 0;
    // Stages per tile.  Where an operand is contiguous along the one K label and its blocks start inside a 128-byte line
    // (a slice of 1376 bf16: every other block starts 64 bytes into a line), stages that start at the block's first k fetch
    // two half lines per row and stage (config 4's down projection: 830 against 1030-1090 TFLOP/s with aligned slices).
    // k_align lays the stages on that operand's lines instead; the set of offsets the tuples' blocks can have decides how
    // many stages that takes, and a tile whose own offset needs one fewer runs an empty last stage.
    const int64_t es = f32 ? 4 : 2, bk = kb / es, run = p.k.n == 1 ? p.K : p.k.ext[p.k.n - 1];
    const int64_t stages0 = (p.K / run) * ((run + bk - 1) / bk);
    p.k_align = 0;
    p.k_stages = (int32_t)stages0;
    if (kb == 128 && p.k.n == 1 && stages0 >= 8) {
        // largest offset (in 16-byte chunks, 0..7) of a block's first row inside its line; -1: rows differ among themselves
        auto worst = [&](const void *base, int which) -> int {
            auto bytes = [&](int64_t elems) { return (uint64_t)(elems * es); };
            const DimList &rows = which == 0 ? p.m : p.n;
            for (int i = 0; i < rows.n; i++)
                if (rows.ext[i] > 1 && bytes(rows.s0[i]) % 128) return -1;
            for (int i = 0; i < p.batch.n; i++)
                if (p.batch.ext[i] > 1 && bytes(which == 0 ? p.batch.s0[i] : p.batch.s1[i]) % 128) return -1;
            unsigned set = 1u << (((uintptr_t)base % 128) / 16);
            for (int l = 0; l < p.ts.n; l++) {
                const uint64_t st = bytes(which == 0 ? p.ts.step_x[l] : p.ts.step_y[l]);
                if (st % 16) return -1;
                unsigned next = 0;
                for (int i = 0; i < p.ts.d[l] && i < 8; i++)
                    for (int r = 0; r < 8; r++)
                        if (set >> r & 1) next |= 1u << ((r + i * (st / 16)) % 8);
                set = next;
            }
            int w = 0;
            for (int r = 0; r < 8; r++)
                if (set >> r & 1) w = r;
            return w;
        };
        const int wx = p.a_kcontig ? worst(p.x, 0) : 0, wy = p.b_kcontig ? worst(p.y, 1) : 0;
        const int which = wx > 0 ? 1 : (wy > 0 ? 2 : 0);
        if (which) {
            const int64_t skip = (which == 1 ? wx : wy) * (16 / es);
            const int64_t stages = (p.K + skip + bk - 1) / bk;
            if (stages == stages0 || (stages == stages0 + 1 && stages0 >= 32)) {     // (an extra stage in 22 costs what whole lines gain)
                p.k_align = which;
                p.k_stages = (int32_t)stages;
            }
        }
    }
    if (p.carry) return wgs * p.n_totals < (1ll << 31) ? dma::launch_carry(p, stream) : fail(EG_ERR_LIMIT, "contraction has too many tiles");
    if (p.n_totals > 1) return dma::launch_totals(p, ns, stream);
    if (tm == 128) return dma::launch_128(p, ns, stream);
    if (tn == 128) return dma::launch_256x128(p, stream);
    return dma::launch_256(p, nw, stream);
}

// ------------------------------------------------------------------------------------------------
// Aggregation of tile-ordered partial slabs (AggTilesParams).
// The sums run over the slabs in ascending order in fp32 with one final cast, as in the dense-layout kernels
// (Section 4.2: the aggregation operator over the tuples that share an output block).
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ int64_t agg_tiles_offset(const DimList &g, int64_t idx, bool batch)
{
    int64_t o = 0;
    uint32_t rem = (uint32_t)idx;
    for (int i = g.n - 1; i >= 0; i--) {
        const uint32_t e = (uint32_t)g.ext[i], q = rem / e, k = rem - q * e;
        rem = q;
        o += (int64_t)k * (batch ? g.s2[i] : g.s1[i]);
    }
    return o;
}

// One workgroup per wave patch of an output tile, 32 rows at a time; the next 32 rows' slabs are fetched meanwhile.  (A workgroup
// per band of 32 rows across the whole tile, all loads issued at once, was 1.5 % faster on 16 slabs and 5-15 % slower on 2-8.)
template <int N>
__global__ __launch_bounds__(256) void k_aggregate_patches(const AggTilesParams p)
{
    fetch_params<sizeof(AggTilesParams)>();
    __shared__ int64_t zr[128], zc[128];               // Z offsets of the patch's rows and columns
    __shared__ __attribute__((aligned(16))) float rows[32 * (128 + 4)];    // 32 rows of the patch on their way from register order to row order
    const int tid = threadIdx.x;
    const int WN = p.nw / 2, RT = p.tm / 64, NT = p.tn / WN / 32;
    const int PR = 32 * RT, PC = 32 * NT, pitch = PC + 4;
    // workgroup -> (output block, batch entry, tile row, tile column, wave of the join kernel)
    const uint32_t wave = blockIdx.x % (uint32_t)p.nw;
    int64_t T = blockIdx.x / (uint32_t)p.nw;
    const int64_t tile = T;
    const int64_t tile_n = T % p.tiles_n; T /= p.tiles_n;
    const int64_t tile_m = T % p.tiles_m; T /= p.tiles_m;
    const int64_t bidx = T % p.n_batch, grp = T / p.n_batch;
    const int64_t bz = group_offset_z(p.ts, grp) + agg_tiles_offset(p.batch, bidx, true);
    const int64_t row0 = tile_m * p.tm + (wave / WN) * PR, col0 = tile_n * p.tn + (wave % WN) * PC;
    if (tid < PR) zr[tid] = agg_tiles_offset(p.m, row0 + tid, false);
    else if (tid - PR < PC) zc[tid - PR] = agg_tiles_offset(p.n, col0 + (tid - PR), false);
    const float *src = p.partials + tile * ((int64_t)p.tm * p.tn) + (int64_t)wave * (RT * NT * 1024);
    const int lane = tid & 63, g4 = tid >> 6;          // chunk (k * 4 + g4) * 64 + lane of the patch, k = i * NT + j
    const int64_t slab4 = p.slab_stride / 4;
    const int orow = tid >> 3, oc0 = (tid & 7) * (PC / 8);    // on the way out: 8 threads per row, PC / 8 consecutive columns each
    // the sums of row tile i (NT chunks per thread); the loads of tile i + 1 are issued before tile i's rows are written out
    auto sums = [&](int i, f32x4 (&acc)[4]) {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if (j >= NT) break;
            const f32x4 *s4 = (const f32x4 *)src + ((i * NT + j) * 4 + g4) * 64 + lane;
            if (N > 0) {
                f32x4 v[N > 0 ? N : 1];
#pragma unroll
                for (int a = 0; a < N; a++) v[a] = __builtin_nontemporal_load(s4 + a * slab4);
                acc[j] = v[0];
#pragma unroll
                for (int a = 1; a < N; a++) acc[j] += v[a];
            } else {
                acc[j] = __builtin_nontemporal_load(s4);
                for (int64_t a = 1; a < p.n_agg; a++) acc[j] += __builtin_nontemporal_load(s4 + a * slab4);
            }
        }
    };
    f32x4 cur[4], nxt[4];
    sums(0, cur);
    for (int i = 0; i < RT; i++) {
        __syncthreads();                               // the tables are there; the previous rows have been read
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if (j >= NT) break;
            float *d = rows + (8 * g4 + 4 * (lane >> 5)) * pitch + j * 32 + (lane & 31);
            d[0] = cur[j].x; d[pitch] = cur[j].y; d[2 * pitch] = cur[j].z; d[3 * pitch] = cur[j].w;
        }
        if (i + 1 < RT) sums(i + 1, nxt);
        __syncthreads();
        const float *r = rows + orow * pitch + oc0;
        const int64_t zb = bz + zr[i * 32 + orow];
        if (p.vec) {                                    // Z runs along the columns: whole 16-byte pieces
            if (p.out_dtype == EG_BF16) {
                for (int c = 0; c < PC / 8; c += 8) {
                    const f32x4 a = *(const f32x4 *)(r + c), b = *(const f32x4 *)(r + c + 4);
                    uint4 o;
                    o.x = pack_bf16x2(a.x, a.y); o.y = pack_bf16x2(a.z, a.w); o.z = pack_bf16x2(b.x, b.y); o.w = pack_bf16x2(b.z, b.w);
                    *(uint4 *)((uint16_t *)p.out + zb + zc[oc0 + c]) = o;
                }
            } else {
                for (int c = 0; c < PC / 8; c += 4) *(f32x4 *)((float *)p.out + zb + zc[oc0 + c]) = *(const f32x4 *)(r + c);
            }
        } else {
            for (int c = 0; c < PC / 8; c++) store_elem(p.out, p.out_dtype, zb + zc[oc0 + c], r[c]);
        }
#pragma unroll
        for (int j = 0; j < 4; j++) cur[j] = nxt[j];
    }
}

int launch_aggregate_tiles(AggTilesParams &p, void *stream)
{
    if (!p.partials || !p.out) return fail(EG_ERR_NULL, "aggregation of tiles: NULL operand");
    const bool shape = (p.tm == 256 && p.tn == 256 && (p.nw == 8 || p.nw == 4)) || (p.tm == 256 && p.tn == 128 && p.nw == 4) || (p.tm == 128 && p.tn == 128 && p.nw == 4);
    if (!shape) return fail(EG_ERR_LIMIT, "aggregation of tiles: no join kernel writes %d x %d tiles with %d waves", p.tm, p.tn, p.nw);
    if (p.n_agg < 1 || p.tiles < 1 || p.tiles_m < 1 || p.tiles_n < 1 || p.n_batch < 1) return fail(EG_ERR_LIMIT, "aggregation of tiles: empty input");
    if (p.tiles % ((int64_t)p.tiles_m * p.tiles_n * p.n_batch)) return fail(EG_ERR_LIMIT, "aggregation of tiles: the tile count is no whole number of output blocks");
    if (p.slab_stride < p.tiles * p.tm * p.tn || p.slab_stride % 4 || ((uintptr_t)p.partials & 15)) return fail(EG_ERR_LIMIT, "aggregation of tiles: slabs overlap or are not 16-byte aligned");
    if (p.out_dtype != EG_F32 && p.out_dtype != EG_BF16) return fail(EG_ERR_DTYPE, "aggregation of tiles: result dtype");
    const int64_t wgs = p.tiles * p.nw;
    if (wgs >= (1ll << 31)) return fail(EG_ERR_LIMIT, "aggregation of tiles: %lld workgroups", (long long)wgs);
    // 16-byte stores along the rows: Z contiguous along the innermost column label in runs of whole pieces, everything else 8-aligned
    bool vec = p.n.s1[p.n.n - 1] == 1 && p.n.ext[p.n.n - 1] % 8 == 0 && ((uintptr_t)p.out & 15) == 0;
    for (int i = 0; i < p.m.n; i++) vec = vec && p.m.s1[i] % 8 == 0;
    for (int i = 0; i + 1 < p.n.n; i++) vec = vec && p.n.s1[i] % 8 == 0;
    for (int i = 0; i < p.batch.n; i++) vec = vec && p.batch.s2[i] % 8 == 0;
    for (int l = 0; l < p.ts.n; l++) vec = vec && p.ts.step_z[l] % 8 == 0;
    p.vec = vec ? 1 : 0;
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid((unsigned)wgs), block(256);
    switch (p.n_agg) {
    case 2: EG_LAUNCH(k_aggregate_patches<2>, grid, block, 0, st, p); break;
    case 4: EG_LAUNCH(k_aggregate_patches<4>, grid, block, 0, st, p); break;
    case 8: EG_LAUNCH(k_aggregate_patches<8>, grid, block, 0, st, p); break;
    case 16: EG_LAUNCH(k_aggregate_patches<16>, grid, block, 0, st, p); break;
    default: EG_LAUNCH(k_aggregate_patches<0>, grid, block, 0, st, p); break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(EG_ERR_HIP, "k_aggregate_tiles launch failed: %s", hipGetErrorString(e));
    return EG_OK;
}

}  // namespace eg
