// Block contraction (bf16 or fp32 operands, fp32 accumulation) with direct global->LDS staging, no register round trip.
//
// Same operation as k_contract.hip (the per-block kernel K of Section 4.3 of the paper for (x) = multiply,
// (+) = sum, all tuples of the join in one launch), specialised for blocks of at least 128 x 128:
//   * 256 x 256 output tiles, 8 waves per workgroup (two per SIMD), each owning a 128x64 patch = 4x2 MFMA 32x32 tiles;
//     or 256 x 128 tiles with 4 waves of the same 128x64 patch, stages half as deep and two workgroups per compute unit,
//     so that one workgroup's epilogue, addressing and first loads run under the other's MFMAs;
//     or 128 x 128 tiles with 4 waves and two workgroups per compute unit when large tiles would leave the chip idle;
//     or, where a compute unit has one such tile at most, 128 x 128 with 8 waves in two groups of four and one workgroup per unit;
//   * persistent workgroups, each walking over its share of the output tiles;
//   * every 16-byte chunk of both operand tiles travels global memory -> LDS directly; the chunk a lane
//     fetches is chosen so that the contiguous 1 KiB an instruction deposits is already the swizzled layout;
//   * a stage is 128 (or 64) bytes of k per tile row (64 or 32 k of bf16, 32 k of fp32) and four (two) k-steps: one
//     32x32x16 bf16 MFMA per 32x32 tile and step, or four 32x32x2 fp32 MFMAs on the four k a 16-byte chunk brings;
//   * an operand contiguous along K sits in LDS as [row][128 bytes of k] and is read with 16-byte reads; an operand
//     contiguous along M or N sits as [k][TS mn] and is read with the 16-bit transposing LDS read (bf16), which
//     hands every lane four consecutive k for its own column, or with four 4-byte reads (fp32);
//   * two LDS stages: the loads of stage t+1 are in flight while the MFMAs of stage t run (256 x 128 tiles three, the eight-wave
//     128 x 128 tile four: two and three stages in flight);
//   * what becomes of the blocks along aggregated labels is a template parameter: partial slabs, totals in registers (128 x 128), or
//     a first block's sums that wait in memory for the second's (256 x 256);
//   * the loads are buffer loads with a 2 GiB descriptor: a lane whose chunk lies beyond K in the last,
//     partial stage is given an offset outside the descriptor, fetches nothing and deposits zeros.
// Several K labels: every run of the innermost one starts a stage of its own (a run of 96 k is a full stage and
// a half-filled one), so a stage never straddles two runs.
// Requirements (checked on the host): along a K-contiguous operand runs are whole 16-byte chunks on chunk boundaries;
// byte offsets within a tile (256 rows, 64 k-rows) fit 31 bits and rows do not lie before their tile's first row.
// Anything else goes to the register-staged kernel.
#pragma once

#include <hip/hip_runtime.h>

#include "eg_device.h"

namespace eg {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

namespace dma {

// Element type: bf16 (F32 = false) or fp32.  A stage holds 128 bytes of k per row: 64 k of bf16, 32 k of fp32, and is
// four k-steps either way (one 32x32x16 bf16 MFMA, or four 32x32x2 fp32 MFMAs on the four k a 16-byte chunk brings).
template <bool F32> struct Elem {
    static constexpr int ES = F32 ? 4 : 2;         // bytes per element
    static constexpr int EPC = 16 / ES;            // elements per 16-byte chunk
};

#define EG_LDS(p) ((__attribute__((address_space(3))) void *)(p))
#define EG_GLB(p) ((const __attribute__((address_space(1))) void *)(p))

__device__ __forceinline__ void decode_group2(const DimList &g, int64_t idx, int64_t &o0, int64_t &o1)
{
    o0 = o1 = 0;
    if (g.n == 1) { o0 = idx * g.s0[0]; o1 = idx * g.s1[0]; return; }
    uint32_t rem = (uint32_t)idx;
    for (int i = g.n - 1; i >= 0; i--) {
        uint32_t e = (uint32_t)g.ext[i], q = rem / e, k = rem - q * e;
        rem = q;
        o0 += (int64_t)k * g.s0[i];
        o1 += (int64_t)k * g.s1[i];
    }
}

// Per-lane source offsets (bytes, relative to the first row of the operand's tile: `origin` is that row's
// element offset in the block) of the chunks this lane fetches per stage (NW waves per workgroup, T rows or columns
// of this operand per tile, KB bytes of k per row and stage), without the k advance.
//   KC: a row holds CR = KB/16 chunks, so one 1 KiB instruction deposits RPI = 64/CR rows (8 for KB = 128, 16 for 64):
//       instruction i of wave w deposits rows (NW i+w)*RPI .. +RPI-1, lane -> row +lane/CR, physical chunk lane%CR,
//       logical chunk (lane%CR) ^ key(row), key = (row>>1)&7 for 128-byte rows, (row>>2)&3 for 64-byte rows: the 16 rows a
//       16-byte LDS read instruction touches in one pass then fall into 16 different 16-byte bank groups.
//   MC: a k-row holds CPR = T/8 chunks, so one instruction deposits KR = 64/CPR k-rows (2 for T = 256, 4 for
//       T = 128): instruction i of wave w deposits k-rows KR (NW i+w) .. +KR-1, lane -> k-row +lane/CPR,
//       physical chunk lane%CPR, logical chunk (lane%CPR) ^ 4*(krow%4), krow%4 = (KR w + lane/CPR)%4.
template <bool KC, int NW, int T, int KB, bool F32>
struct Src {
    static constexpr int ES = Elem<F32>::ES, EPC = Elem<F32>::EPC;
    static constexpr int LD = T * KB / 1024 / NW;         // direct loads of this operand per wave and stage
    static constexpr int CR = KB / 16, RPI = 64 / CR;     // chunks per row of a KC tile, rows per 1 KiB instruction
    static constexpr int CPR = T / EPC, KR = 64 / CPR;    // chunks per k-row of an MC tile, k-rows per 1 KiB instruction
    static_assert(LD >= 1 && LD * NW * 1024 == T * KB, "a stage of this operand is a whole number of 1 KiB instructions per wave");
    static_assert(KB == 128 || KB == 64, "rows of 128 or 64 bytes of k");
    static_assert((NW * KR) % 4 == 0, "the swizzle key of an MC chunk must not depend on the instruction index");
    uint32_t boff[LD];        // byte offset of the chunk instruction i fetches, relative to the stage's first k
    int kl;                   // k (within the stage) of chunk 0 of this lane; chunk i sits at kl (KC) or kl + KR NW i (MC)

    __device__ __forceinline__ void init(const DimList &grp, int64_t first, int64_t extent, int64_t origin, int64_t k_inner_stride, int wave, int lane)
    {
        if (KC) {
            // LDS row of this lane's chunk is (NW i+wave)*RPI + lane/CR; its swizzle key does not depend on i
            const int key = KB == 128 ? ((wave * 4 + (lane >> 4)) & 7) : ((lane >> 4) & 3);
            const int lc = (lane % CR) ^ key;
            kl = lc * EPC;
#pragma unroll
            for (int i = 0; i < LD; i++) {
                int64_t r = first + (NW * i + wave) * RPI + lane / CR;
                r = r < extent ? r : extent - 1;
                int64_t o0, o1;
                decode_group2(grp, r, o0, o1);
                boff[i] = (uint32_t)((o0 - origin + lc * EPC) * ES);
            }
        } else {
            // bf16: chunks of four consecutive k-rows are XOR-ed apart for the transposing reads; fp32 fragments are read
            // with 4-byte reads of 32 consecutive columns, which need no swizzle
            const int kr4 = (KR * wave + lane / CPR) & 3;
            const int lc = F32 ? lane % CPR : (lane % CPR) ^ (4 * kr4);
            int64_t m = first + lc * EPC;
            m = m + EPC <= extent ? m : extent - EPC;
            int64_t o0, o1;
            decode_group2(grp, m, o0, o1);
            kl = KR * wave + lane / CPR;
#pragma unroll
            for (int i = 0; i < LD; i++)
                boff[i] = (uint32_t)((o0 - origin + (KR * NW * i + kl) * k_inner_stride) * ES);
        }
    }
    // offset handed to load i of a stage whose valid k are kmin .. krem-1: beyond the descriptor when the chunk's k is outside
    // (past the end of the reduction, or, in a tile's first stage, before its start)
    __device__ __forceinline__ uint32_t voff(int i, int krem, int kmin) const
    {
        const int k = KC ? kl : kl + KR * NW * i;
        return (uint32_t)(k - kmin) < (uint32_t)(krem - kmin) ? boff[i] : 0x80000000u;
    }
};

// LDS byte address of the fragment chunk lane `lane` feeds to the MFMA for 32-row tile `t32` (rows t32*32..+31
// of the wave's 128) at k-step ks (16 k per step).  KC layout: one 16-byte read.
template <int KB>
__device__ __forceinline__ int kc_frag_off(int row, int ks, int lane)
{
    const int lc = 2 * ks + (lane >> 5);
    const int key = KB == 128 ? (row >> 1) & 7 : (row >> 2) & 3;
    return row * KB + ((lc ^ key) << 4);                    // 16 consecutive rows hit 16 distinct 16-byte bank groups
}

// MC layout: two transposing 8-byte reads (k = 8*(lane/32) + 0..3 and +4..7 of the k-step); TS: columns of the operand's tile.
template <int TS>
__device__ __forceinline__ int mc_frag_off(int col0, int ks, int lane, int second)
{
    const int s = lane & 15;
    const int kr = 16 * ks + 8 * (lane >> 5) + (s >> 2) + 4 * second;
    const int n = col0 + 16 * ((lane >> 4) & 1) + 4 * (s & 3);
    const int pc = (n >> 3) ^ (4 * (s >> 2));
    return kr * (TS * 2) + (pc << 4) + ((n & 7) << 1);
}

// Fragments of one k-step (16 k of bf16, 8 k of fp32): RT 32-row A fragments and NT 32-column B fragments of this wave
// (row0, col0: first row / column of the wave's patch inside the tile).  A fragment is 16 bytes per lane: eight bf16
// (k = 8 * (lane / 32) + 0..7 of the step) or four fp32 (k = 4 * (lane / 32) + 0..3).
template <bool KC, int TS, int KB, bool F32>
__device__ __forceinline__ u32x4 load_frag(const char *l, int first, int ks, int lane)
{
    if (KC) return *(const u32x4 *)(l + kc_frag_off<KB>(first + (lane & 31), ks, lane));
    if (F32) {
        const char *q = l + (8 * ks + 4 * (lane >> 5)) * (TS * 4) + (first + (lane & 31)) * 4;
        u32x4 v;
        v.x = *(const uint32_t *)q; v.y = *(const uint32_t *)(q + TS * 4); v.z = *(const uint32_t *)(q + 2 * TS * 4); v.w = *(const uint32_t *)(q + 3 * TS * 4);
        return v;
    }
    short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v *)EG_LDS(l + mc_frag_off<TS>(first, ks, lane, 0)));
    short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v *)EG_LDS(l + mc_frag_off<TS>(first, ks, lane, 1)));
    u32x4 v;
    short4v *dst = (short4v *)&v;
    dst[0] = lo; dst[1] = hi;
    return v;
}

template <bool A_KC, bool B_KC, int RT, int NT, int TM, int TN, int KB, bool F32>
__device__ __forceinline__ void load_frags(const char *la, const char *lb, int ks, u32x4 (&a)[RT], u32x4 (&b)[NT], int row0, int col0, int lane)
{
#pragma unroll
    for (int i = 0; i < RT; i++) a[i] = load_frag<A_KC, TM, KB, F32>(la, row0 + i * 32, ks, lane);
#pragma unroll
    for (int j = 0; j < NT; j++) b[j] = load_frag<B_KC, TN, KB, F32>(lb, col0 + j * 32, ks, lane);
}

// One 32x32 tile's share of a k-step.
template <bool F32>
__device__ __forceinline__ void mma(const u32x4 &a, const u32x4 &b, f32x16 &acc)
{
    if (F32) {
        // the elements are copied out first: a bit cast applied directly to an element of a vector reference read element 0 every time
        const uint32_t a0 = a.x, a1 = a.y, a2 = a.z, a3 = a.w, b0 = b.x, b1 = b.y, b2 = b.z, b3 = b.w;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a0), __uint_as_float(b0), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a1), __uint_as_float(b1), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a2), __uint_as_float(b2), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a3), __uint_as_float(b3), acc, 0, 0, 0);
    } else {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
    }
}

// MFMAs of one k-step for rows [I0, I1) of this wave's RT x NT grid of 32x32 tiles.
template <int I0, int I1, int RT, int NT, bool F32>
__device__ __forceinline__ void mfma_rows(const u32x4 (&a)[RT], const u32x4 (&b)[NT], f32x16 (&acc)[RT][NT])
{
#pragma unroll
    for (int i = I0; i < I1; i++)
#pragma unroll
        for (int j = 0; j < NT; j++) mma<F32>(a[i], b[j], acc[i][j]);
}

// What is uniform over a workgroup about one output tile.
struct TileInfo {
    int64_t m0, n0;          // first row / column of the tile inside the block
    const char *xb, *yb;     // X and Y at the tuple's blocks, the batch entry and the tile's first row / column
    int64_t ox0, oy0;        // element offsets of that first row / column inside the block (what lane offsets are relative to)
    int64_t bz, agg;         // Z element offset of the tuple's block and batch entry; aggIdx of the tuple
    int64_t slab_tile;       // with tile-ordered partial slabs: the tile's place in its slab
};

// Output tiles are TM x TN; the NW waves of a workgroup form a 2 x NW/2 grid of patches; a stage holds KB bytes of k per row.
//   256 x 256, KB = 128, NW = 8: two waves per SIMD, each owning 128 x 64; one wave's MFMAs cover the other's LDS reads
//       and barrier waits.  One workgroup per compute unit (154 KiB of LDS): every tile's addressing, first loads and
//       epilogue run with the matrix pipes idle, which is what short reductions consist of.
//   256 x 128, KB = 64, NW = 4: the same 128 x 64 patch per wave (the same LDS reads per MFMA), stages half as deep, 64 KiB
//       of LDS: two workgroups per compute unit, not in step with each other, so one's per-tile phases and barrier waits
//       run under the other's MFMAs.
//   256 x 256, KB = 128, NW = 4: one wave per SIMD, each owning 128 x 128 (two thirds of the LDS read traffic, nothing to
//       cover a wave's own waits); kept for comparison.
//   128 x 128, KB = 128, NW = 4: patches of 64 x 64, 78 KiB of LDS, two workgroups per compute unit.  For launches with too
//       few larger tiles to fill the chip, and for totals in registers.
//   128 x 128, KB = 128, NW = 8, four stages: two groups of four waves, each with patches of 64 x 64 over the whole tile and half
//       of a stage's k-steps, 132 KiB of LDS, one workgroup per compute unit.  For launches of one tile per compute unit.
//
// The kernel is persistent: the workgroups of a compute unit walk over their share of the tiles.  While a tile's
// epilogue runs, the first two stages of the workgroup's next tile are already on their way into LDS, and the
// next tile's addressing was worked out while the current tile waited for its own first stage.
// LDS of one workgroup: the stages, two sets of Z offset tables, the waves' epilogue staging rows
// (with three or four stages the staging rows lie in the last stage's buffer, which is free while an epilogue runs)
constexpr int lds_bytes(int TM, int TN, int KB, int WM, int NW, int NS)
{
    return NS * (TM + TN) * KB + 2 * (TM + TN) * 8 + (NS == 2 ? NW * 8 * (32 * (TN / (NW / WM) / 32) * 4 + 32) : 0);          // (NS = 4: staging in a stage's buffer)
}

// NS: LDS stages (2, 3 or 4); REM: the stage count modulo NS (NS = 4: not used, 0).
// MODE 1: one tile over n_totals blocks, whose totals stay in registers; 2: as 0, but a tile's two
// blocks follow one another and the first one's sums wait in memory (p.carry) for the second.
// Four stages (KG = 2): two groups of waves share the tile, each takes half of a stage's k-steps.
template <int TM, int TN, int KB, int NS, int WM, int NW, bool A_KC, bool B_KC, int REM, bool F32, int MODE>
__global__ __launch_bounds__(NW * 64, 2 * lds_bytes(TM, TN, KB, WM, NW, NS) <= 160 * 1024 ? 2 : 1) void k_contract_dma(const ContractParams p)
{
    constexpr bool TOT = MODE == 1, CARRY = MODE == 2;
    constexpr int ES = Elem<F32>::ES, EPC = Elem<F32>::EPC, BK = KB / ES;
    constexpr int KS = KB / 32;                       // k-steps per stage (32 bytes of k each)
    constexpr int KG = NS == 4 ? 2 : 1;               // groups of waves, each with the whole tile and its own k-steps of a stage
    constexpr int WN = NW / KG / WM;                  // waves side by side
    constexpr int RT = TM / WM / 32, NT = TN / WN / 32;    // 32x32 MFMA tiles per wave: RT down, NT across
    constexpr int LDA = TM * KB / 1024 / NW, LDB = TN * KB / 1024 / NW, NLD = LDA + LDB;   // direct loads per wave and stage
    constexpr int TILE_BYTES = TM * KB;               // X's tile of one stage: KB bytes of k per row; Y's follows it
    constexpr int STAGE_BYTES = (TM + TN) * KB;
    constexpr int TBL = (TM + TN) * 8;                // one set of Z offset tables (TM rows, TN columns)
    static_assert(KS == 4 || KS == 2, "a stage is four or two k-steps");
    constexpr int CW = 32 * NT, PITCH = CW * 4 + 32, WBUF = 8 * PITCH;   // epilogue staging: 8 rows of a wave's patch
    // Separate LDS objects for the stages and for the epilogue: the compiler can then tell that the fragment
    // reads of one stage, or the epilogue's staging, never alias the direct loads in flight into another object,
    // and does not wait for them.
    __shared__ __attribute__((aligned(1024))) char lds0[STAGE_BYTES];
    __shared__ __attribute__((aligned(1024))) char lds1[STAGE_BYTES];
    __shared__ __attribute__((aligned(1024))) char lds2[NS >= 3 ? STAGE_BYTES : 16];
    __shared__ __attribute__((aligned(1024))) char lds3[NS >= 4 ? STAGE_BYTES : 16];
    char *const ldsl = NS == 4 ? lds3 : lds2;         // three or four stages: the last one's buffer holds the staging rows during an epilogue
    __shared__ __attribute__((aligned(16))) char ldsx[2 * TBL + (NS == 2 ? NW * WBUF : 0)];    // two sets of Z offset tables (+ staging)
    static_assert(NS == 2 || ((NS == 3 || NS == 4) && NW * WBUF <= STAGE_BYTES), "three or four stages: the staging rows fit one of them");
    static_assert(REM >= 0 && REM < NS, "REM is the stage count modulo NS");
    static_assert(NS * STAGE_BYTES + 2 * TBL + (NS == 2 ? NW * WBUF : 0) == lds_bytes(TM, TN, KB, WM, NW, NS), "lds_bytes() is what decides the workgroups per compute unit");
    fetch_params<sizeof(ContractParams)>();
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % (NW / KG) / WN, wn = wave % WN;
    const int kg = KG == 2 ? __builtin_amdgcn_readfirstlane(wave / (NW / KG)) : 0;
    const int row0 = wm * (32 * RT), col0 = wn * (32 * NT);

    // ---- this workgroup's tiles: logical ids first, first + stride, ...; concurrent ids share an XCD ----
    const uint32_t total = (uint32_t)p.total_tiles, G = gridDim.x;
    uint32_t first, stride, count;
    if ((G & 7) == 0) {
        const uint32_t per = total / 8, rem = total % 8, x = blockIdx.x % 8, j = blockIdx.x / 8;
        const uint32_t nx = per + (x < rem ? 1 : 0);
        stride = G / 8;
        first = x * per + (x < rem ? x : rem) + j;
        count = j < nx ? (nx - j + stride - 1) / stride : 0;
    } else {
        stride = G;
        first = blockIdx.x;
        count = first < total ? (total - first + G - 1) / G : 0;
    }
    if (count == 0) return;
    if (CARRY) count *= 2;                            // (a tile's two blocks one after the other)

    auto uniform_ptr = [](const char *q) {            // the buffer descriptors must live in scalar registers
        const uint64_t v = (uint64_t)q;
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
        return (const char *)(((uint64_t)hi << 32) | lo);
    };
    // logical id -> (tuple, batch entry, tile); tiles are walked in groups of 8 tile rows
    auto tile_info = [&](uint32_t it, TileInfo &t) {
        const uint32_t walk = CARRY ? it / 2 : it, block = CARRY ? it % 2 : 0;
        const uint32_t logical = first + walk * stride;
        const uint32_t tiles = (uint32_t)p.tiles_m * (uint32_t)p.tiles_n;
        const uint32_t tb = logical / tiles, tl = logical - tb * tiles;
        constexpr uint32_t GM = 8;
        const uint32_t span = GM * (uint32_t)p.tiles_n;
        const uint32_t grp = tl / span, first_m = grp * GM;
        const uint32_t gsz = ((uint32_t)p.tiles_m - first_m) < GM ? ((uint32_t)p.tiles_m - first_m) : GM;
        const uint32_t tile_m = first_m + (tl - grp * span) % gsz;
        const uint32_t tile_n = (tl - grp * span) / gsz;
        const uint32_t nb = (uint32_t)p.n_batch, tuple = tb / nb, bidx = tb - tuple * nb;
        int64_t bx, by, bz, agg = 0;
        if (MODE) group_offsets(p.ts, tuple, bx, by, bz);
        else decode_tuple(p.ts, tuple, bx, by, bz, agg);
        if constexpr (CARRY) {
            int64_t ox, oy;
            agg_offsets(p.ts, block, ox, oy);
            bx += ox;
            by += oy;
            agg = block;
        }
        uint32_t rem = bidx;
        for (int i = p.batch.n - 1; i >= 0; i--) {
            uint32_t e = (uint32_t)p.batch.ext[i], q = rem / e, k = rem - q * e;
            rem = q;
            bx += (int64_t)k * p.batch.s0[i];
            by += (int64_t)k * p.batch.s1[i];
            bz += (int64_t)k * p.batch.s2[i];
        }
        t.m0 = (int64_t)tile_m * TM;
        t.n0 = (int64_t)tile_n * TN;
        // lane offsets are 32 bits and count from the tile's first row (an operand contiguous along M or N reads whole
        // 8-element chunks, so near the block's edge its first chunk may start up to 7 elements before the tile)
        int64_t unused;
        const int64_t fm = A_KC || t.m0 + EPC <= p.M ? t.m0 : p.M - EPC, fn = B_KC || t.n0 + EPC <= p.N ? t.n0 : p.N - EPC;
        decode_group2(p.m, fm, t.ox0, unused);
        decode_group2(p.n, fn, t.oy0, unused);
        t.xb = uniform_ptr((const char *)p.x + (bx + t.ox0) * ES);
        t.yb = uniform_ptr((const char *)p.y + (by + t.oy0) * ES);
        t.bz = bz;
        t.agg = agg;
        if (CARRY) t.slab_tile = (int64_t)tb * tiles + tile_m * (uint32_t)p.tiles_n + tile_n;
        else t.slab_tile = p.tile_order ? ((tuple_group(p.ts, tuple) * nb + bidx) * (int64_t)p.tiles_m + tile_m) * (int64_t)p.tiles_n + tile_n : 0;
    };
    const int kin = p.k.n - 1;                        // innermost K label: every stage lies inside one run of it
    const int32_t run = p.k.n == 1 ? (int32_t)p.K : p.k.ext[kin];   // k of one run of the innermost K label
    const int64_t nkb = p.k_stages, nk = TOT ? nkb * p.n_totals : nkb;     // stages per block and per tile: every run starts a stage of its own

    TileInfo cur, nxt;
    Src<A_KC, NW, TM, KB, F32> sa;
    Src<B_KC, NW, TN, KB, F32> sb;
    const char *xb, *yb;                              // bases the direct loads currently work from
    const char *xt, *yt;                              // TOT: the tile's bases; the blocks along the aggregated labels start at offsets from these
    uint32_t blk = 0;                                 // TOT: block the next stage belongs to, and how many of its stages are left
    int32_t blk_left = 0;

    // Uniform source pointers of consecutive stages, and how many k each has (a full stage, less at the end of a run of
    // the innermost K label, 0 past the end: every lane of its direct loads then deposits zeros without fetching).
    // Inside a run a stage lies one fixed step after the one before; where a run ends (several fused K labels) the
    // next stage starts the next run and its offsets are decoded afresh, so a stage never straddles two runs and the
    // main loop's scalar work per stage is two additions almost always.
    const int64_t dka = (int64_t)BK * p.k.s0[kin] * ES, dkb = (int64_t)BK * p.k.s1[kin] * ES;
    // With p.k_align (one K label, an operand contiguous along it whose rows all start at the same offset inside a 128-byte
    // line) a tile's stages are laid on that operand's lines: the first one starts `kskip` elements before the block's
    // first k, those elements are not fetched (zeros), and every later stage fetches whole lines instead of the halves of two.
    const char *ga_n, *gb_n;
    int32_t k_n, run_left;                            // first k of the current run; what is left of it (and of the skipped elements), 0 past the end
    int kskip = 0, kmin_n = 0;
    auto first_stage = [&]() {
        k_n = 0;
        ga_n = xb - (int64_t)kskip * p.k.s0[kin] * ES;
        gb_n = yb - (int64_t)kskip * p.k.s1[kin] * ES;
        run_left = run + kskip;
        kmin_n = kskip;
    };
    auto enter_block = [&]() {
        if constexpr (TOT) {
            int64_t ox, oy;
            agg_offsets(p.ts, blk, ox, oy);
            xb = uniform_ptr(xt + ox * ES);
            yb = uniform_ptr(yt + oy * ES);
            blk_left = (int32_t)nkb;
        }
        kskip = p.k_align ? (int)(((uint32_t)(uintptr_t)(p.k_align == 1 ? xb : yb) & 127u) / ES) : 0;
        first_stage();
    };
    auto next_stage = [&](const char *&ga, const char *&gb, int &krem, int &kmin) {
        ga = ga_n;
        gb = gb_n;
        krem = run_left < BK ? run_left : BK;
        kmin = kmin_n;
        kmin_n = 0;
        run_left -= BK;
        ga_n += dka;
        gb_n += dkb;
        if constexpr (TOT) blk_left--;
        if (run_left <= 0) {
            run_left = 0;
            k_n = k_n < (int32_t)p.K ? k_n + run : k_n;
            if (k_n < (int32_t)p.K) {
                int64_t ka, kb;
                decode_group2(p.k, k_n, ka, kb);       // offset of the next run's first k in X and in Y
                ga_n = xb + ka * ES;
                gb_n = yb + kb * ES;
                run_left = run;
            } else if constexpr (TOT) {
                if (blk_left == 0 && blk + 1 < (uint32_t)p.n_totals) {
                    blk++;
                    enter_block();
                }
            }
        }
    };
    // direct load i (0..LDA-1: X tile, LDA..NLD-1: Y tile) of a stage into the LDS stage at `dst`: a 2 GiB buffer descriptor
    // on the uniform stage base + a 32-bit lane offset (in-block offsets are below 2^31; 2^31 itself means "no fetch, zeros")
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    auto dma = [&](int i, const char *ga, const char *gb, int krem, int kmin, char *dst) {
        if (i < LDA) {
            __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)ga, 0, (int)0x80000000u, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, EG_LDS(dst + (NW * i + wave_u) * 1024), 16, (int)sa.voff(i, krem, kmin), 0, 0, 0);
        } else {
            __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)gb, 0, (int)0x80000000u, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, EG_LDS(dst + TILE_BYTES + (NW * (i - LDA) + wave_u) * 1024), 16, (int)sb.voff(i - LDA, krem, kmin), 0, 0, 0);
        }
    };
    // The same load written out by hand, for the loads that travel during an epilogue: the compiler keeps track of
    // direct loads it issued itself and would hold the epilogue's first LDS access until they have landed.  These
    // are waited for by the explicit vmcnt(0) and barrier at the head of the tile loop.  M0 (the LDS base of a
    // direct load) is put back, so the compiler's own picture of it stays right.
    auto dma_untracked = [&](int i, const char *ga, const char *gb, int krem, int kmin, char *dst) {
        const bool isa = i < LDA;
        const uint64_t base = (uint64_t)(isa ? ga : gb);
        u32x4 rs;
        rs.x = (uint32_t)base;
        rs.y = (uint32_t)(base >> 32) & 0xffffu;       // stride 0
        rs.z = 0x80000000u;
        rs.w = 0x00020000u;
        const uint32_t l = (uint32_t)(uintptr_t)EG_LDS(dst + (isa ? 0 : TILE_BYTES) + (NW * (isa ? i : i - LDA) + wave_u) * 1024);
        const uint32_t off = isa ? sa.voff(i, krem, kmin) : sb.voff(i - LDA, krem, kmin);
        uint32_t keep;
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
                     : "=&s"(keep) : "s"(l), "v"(off), "s"(rs) : "memory");
    };
    auto issue = [&](const char *ga, const char *gb, int krem, int kmin, char *dst) {
#pragma unroll
        for (int i = 0; i < NLD; i++) dma_untracked(i, ga, gb, krem, kmin, dst);
    };
    const char *ga2, *gb2;
    int kr2, km2;
    // per-lane addressing of tile t, then its first two stages on their way, of four stages three (their LDS buffers must be free)
    auto start_tile = [&](const TileInfo &t) {
        sa.init(p.m, t.m0, p.M, t.ox0, p.k.s0[kin], wave, lane);
        sb.init(p.n, t.n0, p.N, t.oy0, p.k.s1[kin], wave, lane);
        xb = xt = uniform_ptr(t.xb);
        yb = yt = uniform_ptr(t.yb);
        blk = 0;
        enter_block();
        next_stage(ga2, gb2, kr2, km2);
        issue(ga2, gb2, kr2, km2, lds0);
        next_stage(ga2, gb2, kr2, km2);
        if (NS == 4 || nk > 1) issue(ga2, gb2, kr2, km2, lds1);
        if constexpr (NS == 4) {
            next_stage(ga2, gb2, kr2, km2);
            issue(ga2, gb2, kr2, km2, lds2);
        }
    };

    // Software pipeline.  Fragment registers alternate between two sets (f0 = a0/b0, f1 = a1/b1).  Each k-step
    // issues its first NT MFMAs, then the LDS reads of the next k-step, then its other 3 NT MFMAs, so the reads
    // return while the matrix pipe is busy.  The last k-step of a stage runs after the barrier, together with
    // the direct loads of the stage after next and the first fragment reads of the next stage.
    // sched_barrier pins this order against the compiler's own scheduling.
    f32x16 acc[RT][NT];
    u32x4 a0[RT], b0[NT], a1[RT], b1[NT];
#define EG_PIN() __builtin_amdgcn_sched_barrier(0)
#define EG_FRAGS(BUF, KSTEP, NA, NB) load_frags<A_KC, B_KC, RT, NT, TM, TN, KB, F32>(BUF, BUF + TILE_BYTES, KSTEP, NA, NB, row0, col0, lane)
#define EG_KSTEP(FA, FB, NA, NB, BUF, KS_NEXT)                                                    \
    mfma_rows<0, 1, RT, NT, F32>(FA, FB, acc); EG_PIN();                                                   \
    EG_FRAGS(BUF, KS_NEXT, NA, NB); EG_PIN();                                                      \
    mfma_rows<1, RT, RT, NT, F32>(FA, FB, acc); EG_PIN();
    // the direct loads of a stage are spread over the RT * NT MFMAs of a k-step: those that follow MFMA q
#define EG_DMA_AFTER(Q, C)                                                                        \
    if (has2) { _Pragma("unroll") for (int d = (Q) * NLD / (RT * NT); d < ((Q) + 1) * NLD / (RT * NT); d++) dma(d, ga2, gb2, kr2, km2, C); }
#define EG_STAGE_NEXT(C, O, HAS_NEXT2) /* one stage; its successor is already in flight into O */     \
    do {                                                                                          \
        mfma_rows<0, 1, RT, NT, F32>(a0, b0, acc); EG_PIN();                                               \
        const bool has2 = (HAS_NEXT2);                                                            \
        next_stage(ga2, gb2, kr2, km2);          /* scalar work rides under the MFMAs */               \
        EG_FRAGS(C, 1, a1, b1); EG_PIN();                                                         \
        mfma_rows<1, RT, RT, NT, F32>(a0, b0, acc); EG_PIN();                                               \
        if constexpr (KS == 4) {                                                                  \
            EG_KSTEP(a1, b1, a0, b0, C, 2)                                                        \
            EG_KSTEP(a0, b0, a1, b1, C, 3)                                                        \
        }                                                                                         \
        __builtin_amdgcn_s_waitcnt(0x0F70); /* vmcnt(0): this wave's deposits for O landed */     \
        __syncthreads();                    /* everybody's landed; everybody has left C */        \
        EG_PIN();                                                                                 \
        /* last k-step: the MFMAs carry the direct loads of the stage after next into C */        \
        _Pragma("unroll") for (int j = 0; j < NT; j++) {                                          \
            mma<F32>(a1[0], b1[j], acc[0][j]); EG_PIN();                                          \
            EG_DMA_AFTER(j, C)                                                                    \
            EG_PIN();                                                                             \
        }                                                                                         \
        EG_FRAGS(O, 0, a0, b0); EG_PIN();                                                         \
        _Pragma("unroll") for (int q = 0; q < (RT - 1) * NT; q++) {                               \
            mma<F32>(a1[1 + q / NT], b1[q % NT], acc[1 + q / NT][q % NT]); EG_PIN();              \
            EG_DMA_AFTER(NT + q, C)                                                               \
            EG_PIN();                                                                             \
        }                                                                                         \
    } while (0)

    // Three or four stages: while stage s is computed, stage s+1 has landed or is landing and the later ones are in
    // flight; the loads of stage s+NS go into s's buffer once every wave has its last fragments of s in registers.  A load
    // has two or three full stages to arrive.  The wait before the barrier leaves the younger stages' loads outstanding.
#define EG_STAGEN(C, O, S)                                                                        \
    do {                                                                                          \
        mfma_rows<0, 1, RT, NT, F32>(a0, b0, acc); EG_PIN();                                               \
        const bool has2 = (S) + NS < nk;    /* what EG_DMA_AFTER issues: stage s+NS into C */     \
        next_stage(ga2, gb2, kr2, km2);                                                                \
        EG_FRAGS(C, 1, a1, b1); EG_PIN();                                                         \
        mfma_rows<1, RT, RT, NT, F32>(a0, b0, acc); EG_PIN();                                               \
        if constexpr (KS == 4) {                                                                  \
            EG_KSTEP(a1, b1, a0, b0, C, 2)                                                        \
            EG_KSTEP(a0, b0, a1, b1, C, 3)                                                        \
        }                                                                                         \
        /* vmcnt(NLD per later stage): stage s+1 has landed, the later ones may still travel; lgkmcnt(0): this wave's reads of C */ \
        /* have returned.  A bare barrier: __syncthreads() would add a fence that waits for every outstanding load. */ \
        if ((S) + 2 < nk) __builtin_amdgcn_s_waitcnt(0x0070 | (NLD & 15) | ((NLD >> 4) << 14)); \
        else __builtin_amdgcn_s_waitcnt(0x0070);                                                  \
        __builtin_amdgcn_s_barrier();                                                             \
        EG_PIN();                                                                                 \
        _Pragma("unroll") for (int j = 0; j < NT; j++) {                                          \
            mma<F32>(a1[0], b1[j], acc[0][j]); EG_PIN();                                          \
            EG_DMA_AFTER(j, C)                                                                    \
            EG_PIN();                                                                             \
        }                                                                                         \
        EG_FRAGS(O, 0, a0, b0); EG_PIN();                                                         \
        _Pragma("unroll") for (int q = 0; q < (RT - 1) * NT; q++) {                               \
            mma<F32>(a1[1 + q / NT], b1[q % NT], acc[1 + q / NT][q % NT]); EG_PIN();              \
            EG_DMA_AFTER(NT + q, C)                                                               \
            EG_PIN();                                                                             \
        }                                                                                         \
    } while (0)

    // Four stages, two groups of four waves, one of each group on every SIMD: a wave of 64 x 64 issues some 180 instructions for
    // the 16 MFMAs of a whole stage, more than their 512 cycles hold, so each group takes two of its four k-steps and the groups'
    // sums are added at the end (and each fragment is still read once per 64 x 64).  A stage's fragments are read into a second set
    // of registers under the MFMAs of the stage before; its buffer is free from the first MFMA of the stage on.  Loads past the
    // last stage fetch nothing and deposit zeros: no branches, and the same number in flight at every wait.
#define EG_STAGE4(B, C, O)                                                                        \
    do {                                                                                          \
        EG_FRAGS(C, kg * 2 + 1, a1, b1); EG_PIN();                                                \
        mfma_rows<0, RT, RT, NT, F32>(a0, b0, acc); EG_PIN();                                     \
        next_stage(ga2, gb2, kr2, km2); EG_PIN();            /* scalar work rides under the MFMAs */ \
        EG_FRAGS(O, kg * 2, a0, b0); EG_PIN();                                                    \
        _Pragma("unroll") for (int q = 0; q < RT * NT; q++) {                                     \
            mma<F32>(a1[q / NT], b1[q % NT], acc[q / NT][q % NT]); EG_PIN();                      \
            _Pragma("unroll") for (int d = q * NLD / (RT * NT); d < (q + 1) * NLD / (RT * NT); d++) dma(d, ga2, gb2, kr2, km2, B); \
            EG_PIN();                                                                             \
        }                                                                                         \
        __builtin_amdgcn_s_waitcnt(0x0F70 | (NLD & 15) | ((NLD >> 4) << 14));                     \
        __builtin_amdgcn_s_barrier();                                                             \
        EG_PIN();                                                                                 \
    } while (0)

    // TOT: a block's sums, scaled and rounded as its partial slab would have held them, are added to the totals in ascending order
    f32x16 tot[TOT ? RT : 1][TOT ? NT : 1];
    int64_t behind = 0;                               // stages of the current block that have been multiplied
    auto fold = [&]() {
        if constexpr (TOT) {
#pragma clang fp contract(off)
            if (++behind == nkb) {
                behind = 0;
                u32x4 z = {0, 0, 0, 0};
                asm volatile("" : "+v"(z));
#pragma unroll
                for (int i = 0; i < RT; i++)
#pragma unroll
                    for (int j = 0; j < NT; j++) {
#pragma unroll
                        for (int r = 0; r < 16; r++) {
                            const float s = p.alpha * acc[i][j][r];
                            tot[i][j][r] = tot[i][j][r] + s;
                        }
                        // Cleared by a matrix instruction, which writes the registers in place: zeros assigned here made the compiler
                        // move all accumulators once per stage.
                        f32x16 zero;
#pragma unroll
                        for (int r = 0; r < 16; r++) zero[r] = 0.f;
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, z), __builtin_bit_cast(bf16x8, z), zero, 0, 0, 0);
                    }
            }
        }
    };
    const bool out_bf16 = p.out.dtype == EG_BF16;
    const float alpha = MODE ? 1.f : p.alpha;         // (totals are scaled already)

    tile_info(0, cur);
    start_tile(cur);
    for (uint32_t it = 0;; it++) {
        const bool more = it + 1 < count;
        // while the first stages travel: the next tile's uniform addressing and this tile's Z offset tables
        // (256 rows, 256 columns; two sets in turn, so a wave already in the next tile cannot disturb a slower one)
        if (more) tile_info(it + 1, nxt);
        int64_t *zrow = (int64_t *)(ldsx + (it & 1) * TBL), *zcol = zrow + TM;
        if (!p.tile_order)                            // (tile-ordered partial slabs need no Z offsets)
        for (int e = tid; e < TM + TN; e += NW * 64) {
            int64_t unused, z;
            if (e < TM) {
                const int64_t m = cur.m0 + e;
                decode_group2(p.m, m < p.M ? m : 0, unused, z);
            } else {
                const int64_t n = cur.n0 + (e - TM);
                decode_group2(p.n, n < p.N ? n : 0, unused, z);
            }
            zrow[e] = z;
        }
#pragma unroll
        for (int i = 0; i < RT; i++)
#pragma unroll
            for (int j = 0; j < NT; j++)
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    acc[i][j][r] = 0.f;
                    if constexpr (TOT) tot[i][j][r] = -0.f;     // the one value that leaves any first sum as it is
                }
        __builtin_amdgcn_s_waitcnt(0x0F70);           // the stages that start_tile issued (and the previous tile's stores) are done
        __syncthreads();
        if constexpr (NS == 3) {
            // the last buffer held the previous tile's staging rows until this barrier: its stage goes out now
            next_stage(ga2, gb2, kr2, km2);
            if (nk > NS - 1) {
#pragma unroll
                for (int i = 0; i < NLD; i++) dma(i, ga2, gb2, kr2, km2, ldsl);
            }
        }
        if constexpr (NS < 4) EG_FRAGS(lds0, 0, a0, b0);
        // Every stage, the last one included, runs the same straight-line code (the last one pays for one idle
        // barrier and a set of unused fragment reads): an MFMA under a branch inside the loop would make the
        // compiler shuffle the accumulator registers.  The stage count modulo the number of buffers is a template parameter.
        if constexpr (NS == 2) {
            if (REM) {
                EG_STAGE_NEXT(lds0, lds1, 2 < nk); fold();
                for (int64_t st = 1; st < nk; st += 2) {
                    EG_STAGE_NEXT(lds1, lds0, st + 2 < nk); fold();
                    EG_STAGE_NEXT(lds0, lds1, st + 3 < nk); fold();
                }
            } else {
                for (int64_t st = 0; st < nk; st += 2) {
                    EG_STAGE_NEXT(lds0, lds1, st + 2 < nk); fold();
                    EG_STAGE_NEXT(lds1, lds0, st + 3 < nk); fold();
                }
            }
        } else if constexpr (NS == 3) {
            int64_t st = 0;
            for (; st + 3 <= nk; st += 3) {
                EG_STAGEN(lds0, lds1, st); fold();
                EG_STAGEN(lds1, lds2, st + 1); fold();
                EG_STAGEN(lds2, lds0, st + 2); fold();
            }
            if constexpr (REM >= 1) { EG_STAGEN(lds0, lds1, st); fold(); }
            if constexpr (REM == 2) { EG_STAGEN(lds1, lds2, st + 1); fold(); }
        } else {
            EG_FRAGS(lds0, kg * 2, a0, b0);
            int64_t st = 0;
            for (; st + 4 <= nk; st += 4) {
                EG_STAGE4(lds3, lds0, lds1); fold();
                EG_STAGE4(lds0, lds1, lds2); fold();
                EG_STAGE4(lds1, lds2, lds3); fold();
                EG_STAGE4(lds2, lds3, lds0); fold();
            }
            if (st < nk) { EG_STAGE4(lds3, lds0, lds1); fold(); }
            if (st + 1 < nk) { EG_STAGE4(lds0, lds1, lds2); fold(); }
            if (st + 2 < nk) { EG_STAGE4(lds1, lds2, lds3); fold(); }
        }
        if constexpr (TOT) {
#pragma unroll
            for (int i = 0; i < RT; i++)
#pragma unroll
                for (int j = 0; j < NT; j++) acc[i][j] = tot[i][j];
        }
        if constexpr (NS == 4) __builtin_amdgcn_s_waitcnt(0x0F70);      // the zeros deposited past the last stage have landed
        __syncthreads();                              // every wave has left the stages
        // the two groups exchange halves of their sums: group g goes on with row tile g of the patch
        constexpr int RTE = RT / KG;                  // row tiles of a wave in the epilogue
        const int erow0 = row0 + kg * RTE * 32;
        f32x16 own[RTE][NT];
        if constexpr (KG == 2) {
            static_assert(RT == 2 && TM * TN * 4 == 2 * STAGE_BYTES, "a row tile each; two stage buffers hold half of the groups' sums");
            f32x4 *mail = (f32x4 *)(kg ? lds2 : lds3) + wave % (NW / KG) * (NT * 256) + lane;
            const f32x4 *got = (const f32x4 *)(kg ? lds3 : lds2) + wave % (NW / KG) * (NT * 256) + lane;
#pragma unroll
            for (int j = 0; j < NT; j++)
#pragma unroll
                for (int r = 0; r < 16; r++) own[0][j][r] = kg ? acc[1][j][r] : acc[0][j][r];
#pragma unroll
            for (int j = 0; j < NT; j++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    f32x4 v;
#pragma unroll
                    for (int r = 0; r < 4; r++) v[r] = kg ? acc[0][j][4 * g + r] : acc[1][j][4 * g + r];
                    mail[(j * 4 + g) * 64] = v;
                }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < NT; j++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    const f32x4 v = got[(j * 4 + g) * 64];
#pragma unroll
                    for (int r = 0; r < 4; r++) own[0][j][4 * g + r] += v[r];
                }
            __syncthreads();                          // the buffers are free for the next tile's stages
        } else {
#pragma unroll
            for (int i = 0; i < RT; i++)
#pragma unroll
                for (int j = 0; j < NT; j++) own[i][j] = acc[i][j];
        }
        // (three stages: the staging rows lie in a stage buffer the compiler has seen direct loads go into; all of those have
        // landed, and saying so here keeps it from waiting again, for the next tile's loads too, in front of the staging)
        if constexpr (NS >= 3) __builtin_amdgcn_s_waitcnt(0x0F70);
        if (more) start_tile(nxt);                    // travels during the epilogue

        // ---- epilogue of the current tile -----------------------------------------------------------
        // lane holds column (lane % 32) and rows 8*(r/4) + 4*(lane/32) + r%4 of each 32x32 tile
        char *zb = (char *)p.out.ptr + (p.out.slab_elems ? cur.agg * p.out.slab_elems * 4 : 0);
        // Everything per-lane below is derived from a lane id the compiler cannot see through, or it would work
        // out the addressing of all the unrolled stores once, before the tile loop, and keep it in scratch memory.
        int elane = lane;
        asm volatile("" : "+v"(elane));
        const int lrow = elane & 31, lhalf = elane >> 5;
        char *wbuf = (NS >= 3 ? ldsl : ldsx + 2 * TBL) + wave_u * WBUF;   // this wave's staging rows
        const bool slab = p.out.slab_elems != 0;
        const int mrem = (int)(p.M - cur.m0 < TM ? p.M - cur.m0 : TM);     // rows / columns of the tile inside the block
        const int nrem = (int)(p.N - cur.n0 < TN ? p.N - cur.n0 : TN);
        bool carried = false;
        if constexpr (CARRY) {
            // The first block's sums, scaled and rounded as its partial slab would have held them, wait in memory in register order
            // while the second block is multiplied; every lane reads back what it wrote itself (8192 x (2 x 4096) x 8192: 998 -> 921 us).
#pragma clang fp contract(off)
            char *tb = (char *)uniform_ptr((const char *)(p.carry + cur.slab_tile * (TM * TN) + wave_u * (RT * NT * 1024)));
            const uint32_t lo = (uint32_t)elane * 16;
            // (one sequence for both blocks: under a branch each, 380 registers went through scratch memory)
            carried = cur.agg == 0;
            f32x4 had[2][4];
            auto fetch = [&](int q, f32x4 (&v)[4]) {
#pragma unroll
                for (int g = 0; g < 4; g++) v[g] = carried ? f32x4{-0.f, -0.f, -0.f, -0.f} : __builtin_nontemporal_load((const f32x4 *)(tb + (q * 4 + g) * 1024 + lo));
            };
            fetch(0, had[0]);
#pragma unroll
            for (int q = 0; q < RT * NT; q++) {
                if (q + 1 < RT * NT) fetch(q + 1, had[(q + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const float s = p.alpha * own[q / NT][q % NT][r];
                    own[q / NT][q % NT][r] = had[q & 1][r >> 2][r & 3] + s;
                }
                if (carried) {
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        const f32x16 &o = own[q / NT][q % NT];
                        const f32x4 val = {o[4 * g], o[4 * g + 1], o[4 * g + 2], o[4 * g + 3]};
                        __builtin_nontemporal_store(val, (f32x4 *)(tb + (q * 4 + g) * 1024 + lo));
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (carried) {
        } else if (KG == 1 && !CARRY && p.tile_order) {
            // Partial slabs in tile order (the launcher set this only for whole tiles): every accumulator register group goes out
            // as it is, 16 bytes per lane and 1 KiB per instruction, no staging; the aggregation kernel undoes the layout.
            float *tb = (float *)zb + cur.slab_tile * (TM * TN) + (int64_t)wave_u * (RT * NT * 4 * 64 * 4);
#pragma unroll
            for (int i = 0; i < RTE; i++)
#pragma unroll
                for (int j = 0; j < NT; j++)
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        const f32x4 val = {alpha * own[i][j][4 * g], alpha * own[i][j][4 * g + 1], alpha * own[i][j][4 * g + 2], alpha * own[i][j][4 * g + 3]};
                        __builtin_nontemporal_store(val, (f32x4 *)(tb + (((i * NT + j) * 4 + g) * 64 + elane) * 4));
                    }
        } else if (p.out_vec) {
            // Z is contiguous along the tile's columns: each wave stages 8 rows x CW columns of its patch at a time
            // in LDS (the row pitch leaves 32 bytes of padding, which keeps the two half-waves on different banks)
            // and writes them out as whole row segments, 16 bytes per lane.  LDS operations of one wave execute
            // in order, so no barrier is needed.
            // The 16 passes are software-pipelined: the stores of a pass are issued after the LDS writes and reads of
            // the next one, so a pass's LDS round trip is hidden behind the next pass's LDS traffic (the wave's LDS
            // operations stay in order, so the single staging buffer is enough).
            constexpr int LPR_F = CW / 4, RPI_F = 64 / LPR_F;     // fp32 out: lanes per row, rows per store instruction
            constexpr int LPR_B = CW / 8, RPI_B = 64 / LPR_B;     // bf16 out
            static_assert(RPI_F <= 8 && RPI_B <= 8, "a store instruction covers at most the 8 staged rows");
            constexpr int NV4 = CW / 32;                          // 16-byte LDS reads per lane and pass
            const int lc = out_bf16 ? elane % LPR_B : elane % LPR_F, lr = out_bf16 ? elane / LPR_B : elane / LPR_F;
            const int c = col0 + lc * (out_bf16 ? 8 : 4);         // first of this lane's 8 or 4 consecutive columns
            const int64_t zc = cur.bz + zcol[c];
            const bool cok = c < nrem;
            f32x4 rd[2][NV4];
            int64_t zr[2][NV4];
            auto write_pass = [&](int i, int q) {
#pragma unroll
                for (int j = 0; j < NT; j++)
#pragma unroll
                    for (int rr = 0; rr < 4; rr++)
                        *(float *)(wbuf + (4 * lhalf + rr) * PITCH + (j * 32 + lrow) * 4) = alpha * own[i][j][4 * q + rr];
            };
            auto read_pass = [&](int i, int q, f32x4 (&v)[NV4], int64_t (&z)[NV4]) {
                if (!out_bf16) {
#pragma unroll
                    for (int h = 0; h < 8 / RPI_F; h++) {
                        const int row = RPI_F * h + lr;
                        v[h] = *(const f32x4 *)(wbuf + row * PITCH + lc * 16);
                        z[h] = zrow[erow0 + i * 32 + 8 * q + row];
                    }
                } else {
#pragma unroll
                    for (int h = 0; h < 8 / RPI_B; h++) {
                        const int row = RPI_B * h + lr;
                        v[2 * h] = *(const f32x4 *)(wbuf + row * PITCH + lc * 32);
                        v[2 * h + 1] = *(const f32x4 *)(wbuf + row * PITCH + lc * 32 + 16);
                        z[2 * h] = zrow[erow0 + i * 32 + 8 * q + row];
                    }
                }
            };
            auto store_pass = [&](int i, int q, const f32x4 (&v)[NV4], const int64_t (&z)[NV4]) {
                if (!out_bf16) {
#pragma unroll
                    for (int h = 0; h < 8 / RPI_F; h++) {
                        const int rr = erow0 + i * 32 + 8 * q + RPI_F * h + lr;
                        if (cok && rr < mrem) {
                            f32x4 *dst = (f32x4 *)((float *)zb + z[h] + zc);
                            const f32x4 val = v[h];
                            if (slab) __builtin_nontemporal_store(val, dst);   // partial slabs are read much later, by another kernel
                            else *dst = val;
                        }
                    }
                } else {
#pragma unroll
                    for (int h = 0; h < 8 / RPI_B; h++) {
                        const int rr = erow0 + i * 32 + 8 * q + RPI_B * h + lr;
                        uint4 o;
                        o.x = pack_bf16x2(v[2 * h].x, v[2 * h].y); o.y = pack_bf16x2(v[2 * h].z, v[2 * h].w);
                        o.z = pack_bf16x2(v[2 * h + 1].x, v[2 * h + 1].y); o.w = pack_bf16x2(v[2 * h + 1].z, v[2 * h + 1].w);
                        if (cok && rr < mrem) *(uint4 *)((uint16_t *)zb + z[2 * h] + zc) = o;
                    }
                }
            };
#pragma unroll
            for (int ps = 0; ps < 4 * RTE; ps++) {
                write_pass(ps >> 2, ps & 3);
                read_pass(ps >> 2, ps & 3, rd[ps & 1], zr[ps & 1]);
                __builtin_amdgcn_sched_barrier(0);
                if (ps > 0) store_pass((ps - 1) >> 2, (ps - 1) & 3, rd[(ps - 1) & 1], zr[(ps - 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
            store_pass(RTE - 1, 3, rd[1], zr[1]);
        } else {
            int64_t zn[NT];
            bool nok[NT];
#pragma unroll
            for (int j = 0; j < NT; j++) {
                const int c = col0 + j * 32 + lrow;
                zn[j] = cur.bz + zcol[c];
                nok[j] = c < nrem;
            }
#pragma unroll
            for (int i = 0; i < RTE; i++) {
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const int rr = erow0 + i * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3);
                    if (rr < mrem) {
                        const int64_t zm = zrow[rr];
#pragma unroll
                        for (int j = 0; j < NT; j++) {
                            if (!nok[j]) continue;
                            const float val = alpha * own[i][j][r];
                            const int64_t off = zm + zn[j];
                            if (out_bf16) ((uint16_t *)zb)[off] = f32_to_bf16(val);
                            else ((float *)zb)[off] = val;
                        }
                    }
                    asm volatile("" ::: "memory");     // keep the scheduler from hoisting all 64 row lookups at once
                }
            }
        }
        if (!more) break;
        cur = nxt;
    }
#undef EG_STAGEN
#undef EG_STAGE_NEXT
#undef EG_DMA_AFTER
#undef EG_KSTEP
#undef EG_FRAGS
#undef EG_PIN
}

template <int TM, int TN, int KB, int NS, int WM, int NW, bool A_KC, bool B_KC, int REM, bool F32, int MODE>
static int launch_one(ContractParams &p, void *stream)
{
    EG_LAUNCH((k_contract_dma<TM, TN, KB, NS, WM, NW, A_KC, B_KC, REM, F32, MODE>), dim3((unsigned)p.grid), dim3(NW * 64), 0, (hipStream_t)stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(EG_ERR_HIP, "k_contract_dma launch failed: %s", hipGetErrorString(e));
    return EG_OK;
}

template <int TM, int TN, int KB, int NS, int WM, int NW, bool A_KC, bool B_KC, bool F32, int MODE>
static int launch_rem(ContractParams &p, void *stream)
{
    const int rem = (int)((MODE == 1 ? (int64_t)p.k_stages * p.n_totals : p.k_stages) % NS);
    if (NS == 4 || rem == 0) return launch_one<TM, TN, KB, NS, WM, NW, A_KC, B_KC, 0, F32, MODE>(p, stream);
    if constexpr (NS < 4) if (rem == 1) return launch_one<TM, TN, KB, NS, WM, NW, A_KC, B_KC, 1, F32, MODE>(p, stream);
    if constexpr (NS == 3) if (rem == 2) return launch_one<TM, TN, KB, NS, WM, NW, A_KC, B_KC, 2, F32, MODE>(p, stream);
    return fail(EG_ERR_LIMIT, "k_contract_dma: stage count");
}

template <int TM, int TN, int KB, int NS, int WM, int NW, bool F32, int MODE = 0>
static int launch_layout(ContractParams &p, void *stream)
{
    if (p.a_kcontig) return p.b_kcontig ? launch_rem<TM, TN, KB, NS, WM, NW, true, true, F32, MODE>(p, stream) : launch_rem<TM, TN, KB, NS, WM, NW, true, false, F32, MODE>(p, stream);
    return p.b_kcontig ? launch_rem<TM, TN, KB, NS, WM, NW, false, true, F32, MODE>(p, stream) : launch_rem<TM, TN, KB, NS, WM, NW, false, false, F32, MODE>(p, stream);
}

// one per unit of instantiations; each returns eg_status
int launch_256(ContractParams &p, int nw, void *stream);              // 256 x 256
int launch_256x128(ContractParams &p, void *stream);
int launch_128(ContractParams &p, int ns, void *stream);              // 128 x 128, two or four stages
int launch_totals(ContractParams &p, int ns, void *stream);           // ... which keeps the totals of n_totals blocks
int launch_carry(ContractParams &p, void *stream);                     // 256 x 256, two blocks, the first one's sums wait in memory

}  // namespace dma

}  // namespace eg
