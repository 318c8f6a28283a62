// Block contraction on MFMA: the per-block kernel K of Section 4.3 of the paper for (x) = multiply,
// (+) = sum, i.e. Z'[l_Z] = sum over l_agg of X^{kX}[l_X] * Y^{kY}[l_Y] on one joined pair of blocks.
//
// Every tuple of the join is viewed as a strided batched matrix product: labels in X, Y and Z are batch
// labels, labels in X and Z form M, labels in Y and Z form N, labels in X and Y only form K.  One launch
// covers all tuples: workgroup -> (tuple, batch index, M tile, N tile).  Tiles are staged through LDS in
// 16-byte chunks with an XOR swizzle; an operand that is contiguous along M or N instead of K is
// transposed in registers on its way into LDS, so the MFMA feed is identical for every layout.
// fp32 accumulation for whole vectors, 64-bit totals for ragged products and a compensation term for other ragged sums;
// the epilogue either writes fp32 partial blocks (slab aggIdx) or casts once to the vertex dtype.
//
// Ragged operands (extents, strides or addresses that are no whole 16-byte vectors) run through the same tiles: a
// vector that lies inside one run of the contiguous label is one load of element alignment, the last one of the last run
// is read so many elements earlier and shifted, and one that crosses into the next run is put together element by element.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "eg_device.h"

namespace eg {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// RAG: operands of any alignment.  WIDE: products and sums in 64 bits (v_mfma_f64_16x16x4), see launch_ragged.
template <int BM_, int BN_, int WM_, int WN_, bool BF16_, bool RAG_ = false, bool WIDE_ = false>
struct Cfg {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
    static constexpr bool BF16 = BF16_, RAG = RAG_, WIDE = WIDE_;
    static constexpr bool TOTALS = RAG_ && BF16_ && !WIDE_;   // a stage's sums in 32 bits, their totals in 64
    static constexpr int ESZ = BF16_ ? 2 : 4;             // element bytes
    static constexpr int EPC = 16 / ESZ;                  // elements per 16-byte chunk
    static constexpr int BK = 8 * EPC;                    // 8 chunks = 128 bytes per tile row
    static constexpr int WAVES_M = BM / WM, WAVES_N = BN / WN;
    static constexpr int THREADS = WAVES_M * WAVES_N * 64;
    static constexpr int MF = WIDE_ ? 16 : 32;            // rows and columns of one MFMA
    static constexpr int MT = WM / MF, NT = WN / MF;      // MFMA tiles per wave
    static constexpr int NVA = BM * 8 / THREADS;          // 16-byte vectors per thread per stage
    static constexpr int NVB = BN * 8 / THREADS;
    static constexpr int LDS_A = BM * 128, LDS_B = BN * 128;
    static constexpr int LDS_BYTES = 2 * (LDS_A + LDS_B);
    static_assert(BM % WM == 0 && BN % WN == 0 && WM % 32 == 0 && WN % 32 == 0, "tile shape");
    static_assert((BM * 8) % THREADS == 0 && (BN * 8) % THREADS == 0, "tile / thread split");
    static_assert(THREADS % 8 == 0 && THREADS % (BM / EPC) == 0 && THREADS % (BN / EPC) == 0, "loader split");
};

// Swizzled byte offset of 16-byte chunk `chunk` (0..7) in tile row `row`.
__device__ __forceinline__ int lds_off(int row, int chunk) { return row * 128 + ((chunk ^ ((row ^ (row >> 3)) & 7)) << 4); }

// index within a role group -> element offsets in the two tensors that carry the group
__device__ __forceinline__ void decode_group(const DimList &g, int64_t idx, int64_t &o0, int64_t &o1)
{
    o0 = o1 = 0;
    if (g.n == 1) {
        o0 = idx * g.s0[0];
        o1 = idx * g.s1[0];
        return;
    }
    uint32_t rem = (uint32_t)idx;
    for (int i = g.n - 1; i >= 0; i--) {
        uint32_t e = (uint32_t)g.ext[i], q = rem / e, k = rem - q * e;
        rem = q;
        o0 += (int64_t)k * g.s0[i];
        o1 += (int64_t)k * g.s1[i];
    }
}

// Gathers element j of each of the NV register vectors (one k-row each) into consecutive k order.
template <int NV, bool BF16>
__device__ __forceinline__ void transpose_store(const uint4 (&v)[NV], char *lds_tile, int row0, int kfirst)
{
    constexpr int EPC = BF16 ? 8 : 4;
    constexpr int G = NV < EPC ? NV : EPC;          // k-values per LDS write (stay inside one 16-byte chunk)
#pragma unroll
    for (int j = 0; j < EPC; j++) {
        const int row = row0 + j;
#pragma unroll
        for (int g0 = 0; g0 < NV; g0 += G) {
            const int k = kfirst + g0;              // first k of this group within the stage
            char *dst = lds_tile + lds_off(row, k / EPC) + (k % EPC) * (BF16 ? 2 : 4);
            if (BF16) {
                uint32_t w[G / 2];
#pragma unroll
                for (int q = 0; q < G / 2; q++) {
                    const uint32_t *a = (const uint32_t *)&v[g0 + 2 * q];
                    const uint32_t *b = (const uint32_t *)&v[g0 + 2 * q + 1];
                    uint32_t lo = (j & 1) ? (a[j >> 1] >> 16) : (a[j >> 1] & 0xffffu);
                    uint32_t hi = (j & 1) ? (b[j >> 1] & 0xffff0000u) : (b[j >> 1] << 16);
                    w[q] = lo | hi;
                }
                if (G == 8) *(uint4 *)dst = make_uint4(w[0], w[1], w[2], w[3]);
                else if (G == 4) *(uint2 *)dst = make_uint2(w[0], w[1]);
                else *(uint32_t *)dst = w[0];
            } else {
                uint32_t w[G];
#pragma unroll
                for (int q = 0; q < G; q++) w[q] = ((const uint32_t *)&v[g0 + q])[j];
                if (G == 4) *(uint4 *)dst = make_uint4(w[0], w[1], w[2], w[3]);
                else if (G == 2) *(uint2 *)dst = make_uint2(w[0], w[1]);
                else *(uint32_t *)dst = w[0];
            }
        }
    }
}

// 16 bytes of EPC elements from an address that is a multiple of the element size only
template <bool BF16>
__device__ __forceinline__ uint4 load_elem_aligned(const char *p)
{
    uint4 v;
    __builtin_memcpy(&v, __builtin_assume_aligned(p, BF16 ? 2 : 4), 16);
    return v;
}

// the same number of elements, each from its own offset: at(j) is element j's offset, or -1 for a zero
template <bool BF16, typename F>
__device__ __forceinline__ uint4 gather_elems(const char *base, F at)
{
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll 1
    for (int j = 0; j < (BF16 ? 8 : 4); j++) {          // rare: code size and registers count more than its speed
        const int64_t o = at(j);
        uint32_t e = 0;
        if (o >= 0) e = BF16 ? (uint32_t)((const uint16_t *)base)[o] << (16 * (j & 1)) : ((const uint32_t *)base)[o];
#pragma unroll
        for (int q = 0; q < 4; q++) w[q] |= q == (BF16 ? j >> 1 : j) ? e : 0u;
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// elements s .. EPC-1 of a vector, moved to the front; zeros behind them
template <bool BF16>
__device__ __forceinline__ uint4 drop_elems(uint4 v, int s)
{
    const int b = s * (BF16 ? 16 : 32);
    if (b == 0) return v;
    uint64_t lo = (uint64_t)v.y << 32 | v.x, hi = (uint64_t)v.w << 32 | v.z;
    if (b >= 64) {
        lo = hi >> (b - 64);
        hi = 0;
    } else {
        lo = lo >> b | hi << (64 - b);
        hi >>= b;
    }
    return make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
}

// position of idx inside the innermost run of a group
__device__ __forceinline__ int32_t run_pos(const DimList &g, int64_t idx)
{
    return g.n == 1 ? (int32_t)idx : (int32_t)((uint32_t)idx % (uint32_t)g.ext[g.n - 1]);
}

// One operand's loader state: which rows / k-rows this thread fetches and where they land in LDS.
template <int ROWS, int NV, int THREADS, bool BF16, bool RAG>
struct Loader {
    static constexpr int EPC = BF16 ? 8 : 4;
    static constexpr int CM = ROWS / EPC;            // mn-chunks per k-row (mn-contiguous mode)
    const char *base;                                // operand base for this (tuple, batch, tile)
    int64_t row_off[NV];                             // k-contiguous mode: element offset of each fetched row
    int64_t mn_off;                                  // mn-contiguous mode: element offset of the chunk start
    bool kcontig;
    bool cross;                                      // ragged, mn-contiguous mode: the chunk crosses into another run
    int back;                                        // ragged, mn-contiguous mode: elements by which the chunk at the edge is read earlier
    int32_t m_first;                                 // its first index in the group
    uint4 reg[NV];

    // gsel: 0 -> K strides of X (s0), 1 -> K strides of Y (s1)
    __device__ __forceinline__ void init(const void *ptr, int64_t base_off, const DimList &grp, int64_t first, int64_t extent,
                                         bool kc, int tid)
    {
        kcontig = kc;
        cross = false;
        back = 0;
        m_first = 0;
        base = (const char *)ptr + base_off * (BF16 ? 2 : 4);
        if (kc) {
#pragma unroll
            for (int i = 0; i < NV; i++) {
                int64_t r = first + (tid >> 3) + i * (THREADS / 8);
                r = r < extent ? r : extent - 1;                 // clamp: rows past the edge are never stored
                int64_t o0, o1;
                decode_group(grp, r, o0, o1);
                row_off[i] = o0;
            }
            mn_off = 0;
        } else {
            int64_t m = first + (int64_t)(tid % CM) * EPC;
            if (RAG) {
                m_first = (int32_t)(m < extent ? m : extent - 1);
                const int32_t run = grp.ext[grp.n - 1], over = run_pos(grp, m_first) + EPC - run;
                // The last chunk of the edge reads the EPC elements that end there and drops what lies in front of its own:
                // element by element it took 6 us a stage where the others take 2 (1000 x 3001 x 1530: 290 us, 98 now)
                if (over > 0 && m_first + EPC > extent && run >= EPC) back = over;
                else cross = over > 0;
                m = m_first - back;
            } else m = m + EPC <= extent ? m : extent - EPC;            // extent is a multiple of EPC (checked on the host)
            int64_t o0, o1;
            decode_group(grp, m, o0, o1);
            mn_off = o0;
#pragma unroll
            for (int i = 0; i < NV; i++) row_off[i] = 0;
        }
    }

    // Issues the global loads of the stage starting at k0.  which: 0 = X strides of K, 1 = Y strides.
    // (grp and extent: the row group, read only for chunks that cross the end of a run)
    __device__ __forceinline__ void fetch(const DimList &kgrp, int which, int64_t k0, int64_t K, int tid, const DimList &grp, int64_t extent)
    {
        if (kcontig) {
            const int64_t k = k0 + (tid & 7) * EPC;
            int64_t o0, o1;
            decode_group(kgrp, k < K ? k : 0, o0, o1);
            const int64_t ko = which ? o1 : o0;
            if (RAG) {
                const int32_t run = kgrp.ext[kgrp.n - 1], over = run_pos(kgrp, k < K ? k : 0) + EPC - run;
                const int early = over > 0 ? over : 0;               // as at the edge of the rows: read early, drop what is in front
                if (k < K && (early == 0 || (k + EPC > K && run >= EPC))) {
#pragma unroll
                    for (int i = 0; i < NV; i++) reg[i] = load_elem_aligned<BF16>(base + (row_off[i] + ko - early) * (BF16 ? 2 : 4));
                    if (early) {
#pragma unroll
                        for (int i = 0; i < NV; i++) reg[i] = drop_elems<BF16>(reg[i], early);
                    }
                } else if (k >= K) {
#pragma unroll
                    for (int i = 0; i < NV; i++) reg[i] = make_uint4(0, 0, 0, 0);
                } else {
#pragma unroll 1
                    for (int i = 0; i < NV; i++) {
                        int64_t ro = row_off[0];                     // row_off[i] without a register array indexed at run time
#pragma unroll
                        for (int q = 1; q < NV; q++) ro = q == i ? row_off[q] : ro;
                        const uint4 v = gather_elems<BF16>(base, [&](int j) -> int64_t {
                            if (k + j >= K) return -1;
                            int64_t a0, a1;
                            decode_group(kgrp, k + j, a0, a1);
                            return ro + (which ? a1 : a0);
                        });
#pragma unroll
                        for (int q = 0; q < NV; q++)
                            if (q == i) reg[q] = v;
                    }
                }
                return;
            }
#pragma unroll
            for (int i = 0; i < NV; i++) {
                if (k < K) reg[i] = *(const uint4 *)(base + (row_off[i] + ko) * (BF16 ? 2 : 4));
                else reg[i] = make_uint4(0, 0, 0, 0);
            }
        } else {
            const int64_t kfirst = k0 + (int64_t)(tid / CM) * NV;
            if (RAG && cross) {
#pragma unroll 1
                for (int i = 0; i < NV; i++) {
                    const int64_t k = kfirst + i;
                    int64_t o0, o1;
                    decode_group(kgrp, k < K ? k : 0, o0, o1);
                    const int64_t ko = which ? o1 : o0;
                    const uint4 v = gather_elems<BF16>(base, [&](int j) -> int64_t {       // rows past the edge repeat the last one
                        if (k >= K) return -1;
                        const int64_t m = m_first + j < extent ? m_first + j : extent - 1;
                        int64_t a0, a1;
                        decode_group(grp, m, a0, a1);
                        return a0 + ko;
                    });
#pragma unroll
                    for (int q = 0; q < NV; q++)
                        if (q == i) reg[q] = v;
                }
                return;
            }
#pragma unroll
            for (int i = 0; i < NV; i++) {
                const int64_t k = kfirst + i;
                int64_t o0, o1;
                decode_group(kgrp, k < K ? k : 0, o0, o1);
                const int64_t ko = which ? o1 : o0;
                if (RAG) {
                    if (k < K) reg[i] = load_elem_aligned<BF16>(base + (mn_off + ko) * (BF16 ? 2 : 4));
                    else reg[i] = make_uint4(0, 0, 0, 0);
                } else if (k < K) reg[i] = *(const uint4 *)(base + (mn_off + ko) * (BF16 ? 2 : 4));
                else reg[i] = make_uint4(0, 0, 0, 0);
            }
            if (RAG && back) {
#pragma unroll
                for (int i = 0; i < NV; i++) reg[i] = drop_elems<BF16>(reg[i], back);
            }
        }
    }

    __device__ __forceinline__ void commit(char *lds_tile, int tid) const
    {
        if (kcontig) {
#pragma unroll
            for (int i = 0; i < NV; i++) {
                const int row = (tid >> 3) + i * (THREADS / 8);
                *(uint4 *)(lds_tile + lds_off(row, tid & 7)) = reg[i];
            }
        } else {
            transpose_store<NV, BF16>(reg, lds_tile, (tid % CM) * EPC, (tid / CM) * NV);
        }
    }
};

// TOTALS: four waves per SIMD (128 registers, nothing spilled) hide the stages' loads better than the compiler's three:
// 4001 x 3001 x 4099 578 -> 447 us.
template <typename C>
__global__ __launch_bounds__(C::THREADS, C::TOTALS ? 4 : 1) void k_contract(const ContractParams p)
{
    fetch_params<sizeof(ContractParams)>();
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;

    // ---- workgroup -> (tuple, batch, tile); consecutive logical ids stay on one XCD -----------------
    const int64_t total = (int64_t)gridDim.x;
    int64_t logical;
    {
        const int64_t per = total / 8, rem = total % 8;
        const int64_t x = blockIdx.x % 8, j = blockIdx.x / 8;
        logical = x * per + (x < rem ? x : rem) + j;
    }
    const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n;
    const int64_t tb = logical / tiles;
    const int tl = (int)(logical - tb * tiles);
    constexpr int GM = 8;                                    // tile rows walked together for L2 reuse
    const int span = GM * p.tiles_n;
    const int grp = tl / span, first_m = grp * GM;
    const int gsz = (p.tiles_m - first_m) < GM ? (p.tiles_m - first_m) : GM;
    const int tile_m = first_m + (tl - grp * span) % gsz;
    const int tile_n = (tl - grp * span) / gsz;
    const int64_t tuple = tb / p.n_batch, bidx = tb - tuple * p.n_batch;

    int64_t bx, by, bz, agg;
    decode_tuple(p.ts, tuple, bx, by, bz, agg);
    {
        uint32_t rem = (uint32_t)bidx;
        for (int i = p.batch.n - 1; i >= 0; i--) {
            uint32_t e = (uint32_t)p.batch.ext[i], q = rem / e, k = rem - q * e;
            rem = q;
            bx += (int64_t)k * p.batch.s0[i];
            by += (int64_t)k * p.batch.s1[i];
            bz += (int64_t)k * p.batch.s2[i];
        }
    }
    const int64_t m0 = (int64_t)tile_m * C::BM, n0 = (int64_t)tile_n * C::BN;

    Loader<C::BM, C::NVA, C::THREADS, C::BF16, C::RAG> la;
    Loader<C::BN, C::NVB, C::THREADS, C::BF16, C::RAG> lb;
    la.init(p.x, bx, p.m, m0, p.M, p.a_kcontig != 0, tid);
    lb.init(p.y, by, p.n, n0, p.N, p.b_kcontig != 0, tid);

    constexpr int AR = C::WIDE ? 4 : 16;                     // accumulators per lane of one MFMA
    typedef typename std::conditional<C::TOTALS, double, float>::type total_t;
    typedef total_t totals __attribute__((ext_vector_type(16)));
    typename std::conditional<C::WIDE, f64x4, totals>::type acc[C::MT][C::NT];
#pragma unroll
    for (int i = 0; i < C::MT; i++)
#pragma unroll
        for (int j = 0; j < C::NT; j++)
#pragma unroll
            for (int r = 0; r < AR; r++) acc[i][j][r] = 0;

    const int64_t nk = (p.K + C::BK - 1) / C::BK;
    la.fetch(p.k, 0, 0, p.K, tid, p.m, p.M);
    lb.fetch(p.k, 1, 0, p.K, tid, p.n, p.N);
    la.commit(smem, tid);
    lb.commit(smem + C::LDS_A, tid);
    __syncthreads();

    const int lrow = lane & 31, lhalf = lane >> 5;
    for (int64_t kt = 0; kt < nk; kt++) {
        const int cur = (int)(kt & 1);
        const char *sa = smem + cur * (C::LDS_A + C::LDS_B);
        const char *sb = sa + C::LDS_A;
        if (kt + 1 < nk) {
            la.fetch(p.k, 0, (kt + 1) * C::BK, p.K, tid, p.m, p.M);
            lb.fetch(p.k, 1, (kt + 1) * C::BK, p.K, tid, p.n, p.N);
        }
        if constexpr (C::WIDE) {
            // lane: row or column lane % 16, k = lane / 16 of four.  An MFMA takes 64 cycles, so element reads keep up
            auto elem = [&](const char *tile, int row, int k) -> double {
                const char *q = tile + lds_off(row, k / C::EPC) + (k % C::EPC) * C::ESZ;
                return C::BF16 ? (double)bf16_to_f32(*(const uint16_t *)q) : (double)*(const float *)q;
            };
            const int64_t left = p.K - kt * C::BK;           // slots behind the last k hold zeros: whole groups of them are left out
            const int groups = left >= C::BK ? C::BK / 4 : (int)((left + 3) / 4);
            for (int ks = 0; ks < groups; ks++) {
                const int k = 4 * ks + (lane >> 4);
                double a[C::MT], b[C::NT];
#pragma unroll
                for (int i = 0; i < C::MT; i++) a[i] = elem(sa, wm * C::WM + i * 16 + (lane & 15), k);
#pragma unroll
                for (int j = 0; j < C::NT; j++) b[j] = elem(sb, wn * C::WN + j * 16 + (lane & 15), k);
#pragma unroll
                for (int i = 0; i < C::MT; i++)
#pragma unroll
                    for (int j = 0; j < C::NT; j++) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
            }
        } else if constexpr (C::TOTALS) {
            // The products of a stage (64 at most) are added from zero on the matrix instruction and their sum goes to a 64-bit
            // total: 16 conversions and additions per 32 x 32 of a stage, hidden behind its loads (figures at launch_ragged)
            uint4 b[C::NT][4];
#pragma unroll
            for (int j = 0; j < C::NT; j++)
#pragma unroll
                for (int ks = 0; ks < 4; ks++) b[j][ks] = *(const uint4 *)(sb + lds_off(wn * C::WN + j * 32 + lrow, 2 * ks + lhalf));
#pragma unroll
            for (int i = 0; i < C::MT; i++) {
                uint4 a[4];
#pragma unroll
                for (int ks = 0; ks < 4; ks++) a[ks] = *(const uint4 *)(sa + lds_off(wm * C::WM + i * 32 + lrow, 2 * ks + lhalf));
#pragma unroll
                for (int j = 0; j < C::NT; j++) {
                    f32x16 part;
#pragma unroll
                    for (int r = 0; r < 16; r++) part[r] = 0.f;
#pragma unroll
                    for (int ks = 0; ks < 4; ks++)
                        part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8 *)&a[ks], *(const bf16x8 *)&b[j][ks], part, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 16; r++) acc[i][j][r] += (double)part[r];
                }
            }
        } else
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
            uint4 a[C::MT], b[C::NT];
#pragma unroll
            for (int i = 0; i < C::MT; i++) a[i] = *(const uint4 *)(sa + lds_off(wm * C::WM + i * 32 + lrow, 2 * ks + lhalf));
#pragma unroll
            for (int j = 0; j < C::NT; j++) b[j] = *(const uint4 *)(sb + lds_off(wn * C::WN + j * 32 + lrow, 2 * ks + lhalf));
#pragma unroll
            for (int i = 0; i < C::MT; i++)
#pragma unroll
                for (int j = 0; j < C::NT; j++) {
                    if (C::BF16) {
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8 *)&a[i], *(const bf16x8 *)&b[j], acc[i][j], 0, 0, 0);
                    } else {
                        const float *fa = (const float *)&a[i];
                        const float *fb = (const float *)&b[j];
#pragma unroll
                        for (int q = 0; q < 4; q++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[q], fb[q], acc[i][j], 0, 0, 0);
                    }
                }
        }
        if (kt + 1 < nk) {
            char *na = smem + (cur ^ 1) * (C::LDS_A + C::LDS_B);
            la.commit(na, tid);
            lb.commit(na + C::LDS_A, tid);
        }
        __syncthreads();
    }

    // ---- epilogue: lane holds column (lane % 32) and rows 8*(r/4) + 4*(lane/32) + r%4 of each 32x32 tile; in 64 bits
    // column (lane % 16) and rows 4*r + lane/16 of each 16x16 tile ----
    char *zb = (char *)p.out.ptr + (p.out.slab_elems ? agg * p.out.slab_elems * 4 : 0);
    const bool out_bf16 = p.out.dtype == EG_BF16;
#pragma unroll
    for (int j = 0; j < C::NT; j++) {
        const int64_t n = n0 + wn * C::WN + j * C::MF + (lane & (C::MF - 1));
        if (n >= p.N) continue;
        int64_t oy_unused, zn;
        decode_group(p.n, n, oy_unused, zn);
#pragma unroll
        for (int i = 0; i < C::MT; i++) {
#pragma unroll
            for (int r = 0; r < AR; r++) {
                const int64_t m = m0 + wm * C::WM + i * C::MF + (C::WIDE ? 4 * r + (lane >> 4) : 8 * (r >> 2) + 4 * lhalf + (r & 3));
                if (m >= p.M) continue;
                int64_t ox_unused, zm;
                decode_group(p.m, m, ox_unused, zm);
                const float val = C::WIDE || C::TOTALS ? (float)((double)p.alpha * acc[i][j][r]) : p.alpha * (float)acc[i][j][r];
                const int64_t off = bz + zm + zn;
                if (out_bf16) ((uint16_t *)zb)[off] = f32_to_bf16(val);
                else ((float *)zb)[off] = val;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Ragged products whose contracted label is one run and whose operands' contiguous labels are one run each: 64 x 64 tiles
// of four waves as above, with loads that need no branches, so that several stages of them can be in flight.  A vector that
// would cross the end of its run is read so many elements earlier, and moved into place (zeros behind it) on its way into
// LDS; k-rows past the end are read from the last one and replaced by zeros there.  A workgroup walks over the blocks
// along the aggregated labels (n_totals) as one sequence of stages, its 64-bit totals go on over all of them.
//   WIDE (results of 32 bits, fp32 operands): v_mfma_f64_16x16x4, bound by its 64 cycles.  Which k a slot of the instruction
//       stands for is free, so a lane takes its 16-byte chunks g and g + 4 of a stage's eight whole: 8 LDS reads a stage
//       instead of 64 of single elements, each followed by the instruction that waits for it.
//   otherwise (bf16 to bf16): a stage's sums on the bf16 instruction from zero, added to 64-bit totals; bound by the latency of the
//       loads, of which two stages are in flight (with four, 195 registers and a workgroup fewer on the compute unit: the same).
// us before (the tiles above: one stage of loads in flight, branches around them) and now: 1000 x 3001 x 1530 to bf16 98 and 52, 1000 x
// 1530 x 1003 to fp32 123 and 72, 3001 x 1000 x 1530 to fp32 in eight blocks 287 and 215, 1121 x 319 x 647 fp32 33 and 20, 707 x 22867 x
// 767 in eight 688 and 260.  264 shapes of 300 to 5100 rows and columns and 17 to 300 contracted elements, the rule for short ones
// (contract_ragged_short) applied, 0.94 to 1.55 times as fast.
// ------------------------------------------------------------------------------------------------
template <bool BF16, bool WIDE>
__global__ __launch_bounds__(256, WIDE ? 2 : 3) void k_contract_ragged(const ContractParams p)
{
    fetch_params<sizeof(ContractParams)>();
    constexpr int ES = BF16 ? 2 : 4, EPC = 16 / ES, BK = 128 / ES, NV = 2, CM = 64 / EPC;    // elements per chunk, k of a stage, vectors per thread and operand
    constexpr int D = 2;                                     // stages in flight
    constexpr int TILE = 64 * 128;                           // bytes of one operand's stage
    __shared__ __attribute__((aligned(16))) char lds[2][2 * TILE];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;

    // ---- workgroup -> (output block, batch entry, tile); consecutive logical ids stay on one XCD ----
    const uint32_t total = gridDim.x, per = total / 8, rem8 = total % 8, xcd = blockIdx.x % 8;
    const uint32_t logical = xcd * per + (xcd < rem8 ? xcd : rem8) + blockIdx.x / 8;
    const uint32_t tiles = (uint32_t)p.tiles_m * (uint32_t)p.tiles_n, tb = logical / tiles, tl = logical - tb * tiles;
    constexpr uint32_t GM = 8;                               // tile rows walked together for L2 reuse
    const uint32_t span = GM * (uint32_t)p.tiles_n, grp = tl / span, first_m = grp * GM;
    const uint32_t gsz = (uint32_t)p.tiles_m - first_m < GM ? (uint32_t)p.tiles_m - first_m : GM;
    const int64_t m0 = (int64_t)(first_m + (tl - grp * span) % gsz) * 64, n0 = (int64_t)((tl - grp * span) / gsz) * 64;
    const uint32_t tuple = tb / (uint32_t)p.n_batch, bidx = tb - tuple * (uint32_t)p.n_batch;
    const uint32_t blocks = p.n_totals > 1 ? (uint32_t)p.n_totals : 1u;
    int64_t bx, by, bz, agg = 0;
    if (blocks > 1) group_offsets(p.ts, tuple, bx, by, bz);
    else decode_tuple(p.ts, tuple, bx, by, bz, agg);
    {
        uint32_t rem = bidx;
        for (int i = p.batch.n - 1; i >= 0; i--) {
            const uint32_t e = (uint32_t)p.batch.ext[i], q = rem / e, k = rem - q * e;
            rem = q;
            bx += (int64_t)k * p.batch.s0[i];
            by += (int64_t)k * p.batch.s1[i];
            bz += (int64_t)k * p.batch.s2[i];
        }
    }

    // ---- one operand's side of the loads ----
    const int32_t K = (int32_t)p.K;
    struct Side {
        int64_t off[NV];                                     // element offset of the row (along k) or of the chunk (otherwise, off[0])
        int64_t ks;                                          // element stride of k
        int32_t k;                                           // first k of this thread's vectors inside a stage
        int32_t back;                                        // chunk at the edge, read so many elements earlier
        bool kc;
    };
    auto side = [&](const DimList &g, int64_t first, int64_t extent, bool kc, int64_t ks) {
        Side d;
        d.kc = kc;
        d.ks = ks;
        d.back = 0;
        int64_t unused;
        if (kc) {
            d.k = (tid & 7) * EPC;
#pragma unroll
            for (int i = 0; i < NV; i++) {
                const int64_t r = first + (tid >> 3) + i * 32;
                decode_group(g, r < extent ? r : extent - 1, d.off[i], unused);      // rows past the edge are never stored
            }
        } else {
            d.k = tid / CM * NV;
            int64_t m = first + (int64_t)(tid % CM) * EPC;
            m = m < extent ? m : extent - 1;
            if (m + EPC > extent) { d.back = (int32_t)(m + EPC - extent); m = extent - EPC; }
            decode_group(g, m, d.off[0], unused);
            d.off[1] = 0;
        }
        return d;
    };
    const Side A = side(p.m, m0, p.M, p.a_kcontig != 0, p.k.s0[0]), B = side(p.n, n0, p.N, p.b_kcontig != 0, p.k.s1[0]);
    const char *xt = (const char *)p.x + bx * ES, *yt = (const char *)p.y + by * ES;
    auto load_side = [&](const Side &d, const char *base, int32_t k0, uint4 (&v)[NV]) {
        if (d.kc) {
            int32_t k = k0 + d.k;
            k = k + EPC <= K ? k : K - EPC;
#pragma unroll
            for (int i = 0; i < NV; i++) v[i] = load_elem_aligned<BF16>(base + (d.off[i] + k) * ES);
        } else {
#pragma unroll
            for (int i = 0; i < NV; i++) {
                int32_t k = k0 + d.k + i;
                k = k < K ? k : K - 1;
                v[i] = load_elem_aligned<BF16>(base + (d.off[0] + (int64_t)k * d.ks) * ES);
            }
        }
    };
    // a stage's vectors into LDS; whole: all of its k exist
    auto store_side = [&](const Side &d, int32_t k0, bool whole, bool edge, uint4 (&v)[NV], char *tile) {
        if (d.kc) {
            if (!whole) {
                const int32_t over = k0 + d.k + EPC - K;     // elements behind the last k
#pragma unroll
                for (int i = 0; i < NV; i++)
                    if (over > 0) v[i] = over < EPC ? drop_elems<BF16>(v[i], over) : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < NV; i++) *(uint4 *)(tile + lds_off((tid >> 3) + i * 32, tid & 7)) = v[i];
        } else {
            if (edge) {
#pragma unroll
                for (int i = 0; i < NV; i++) v[i] = drop_elems<BF16>(v[i], d.back);
            }
            if (!whole) {
#pragma unroll
                for (int i = 0; i < NV; i++)
                    if (k0 + d.k + i >= K) v[i] = make_uint4(0, 0, 0, 0);
            }
            transpose_store<NV, BF16>(v, tile, (tid % CM) * EPC, d.k);
        }
    };
    const bool edge_a = !A.kc && m0 + 64 > p.M, edge_b = !B.kc && n0 + 64 > p.N;

    // ---- stages: the loads run D stages ahead of the arithmetic, over the ends of blocks; past the last stage they repeat it ----
    const int32_t per_block = (K + BK - 1) / BK;
    const int64_t nst = (int64_t)per_block * blocks;
    uint32_t lblk = 0;
    int32_t lk = 0, sk = 0;                                  // next stage to load (block, first k); next one to store
    const char *xl = xt, *yl = yt;
    int64_t loaded = 0;
    if (blocks > 1) {
        int64_t ox, oy;
        agg_offsets(p.ts, 0, ox, oy);
        xl = xt + ox * ES;
        yl = yt + oy * ES;
    }
    auto load = [&](uint4 (&a)[NV], uint4 (&b)[NV]) {
        load_side(A, xl, lk, a);
        load_side(B, yl, lk, b);
        if (++loaded < nst) {
            lk += BK;
            if (lk >= K) {
                lk = 0;
                lblk++;
                int64_t ox, oy;
                agg_offsets(p.ts, lblk, ox, oy);
                xl = xt + ox * ES;
                yl = yt + oy * ES;
            }
        }
    };
    auto store = [&](uint4 (&a)[NV], uint4 (&b)[NV], char *dst) {
        const bool whole = sk + BK <= K;
        store_side(A, sk, whole, edge_a, a, dst);
        store_side(B, sk, whole, edge_b, b, dst + TILE);
        sk = sk + BK < K ? sk + BK : 0;
    };

    uint4 ra[D][NV], rb[D][NV];
#pragma unroll
    for (int d = 0; d < D; d++) load(ra[d], rb[d]);
    store(ra[0], rb[0], lds[0]);
    load(ra[0], rb[0]);
    __syncthreads();

    constexpr int AR = WIDE ? 4 : 16;
    typedef double totals __attribute__((ext_vector_type(AR)));
    constexpr int MT = WIDE ? 2 : 1;
    totals acc[MT][MT];
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
        for (int j = 0; j < MT; j++)
#pragma unroll
            for (int r = 0; r < AR; r++) acc[i][j][r] = 0;
    const int c16 = lane & 15, g = lane >> 4, lrow = lane & 31, lhalf = lane >> 5;
    int32_t ck = 0;                                          // first k of the stage that is multiplied
    [[maybe_unused]] uint4 wa[2][2], wb[2][2];               // WIDE: row or column tile, chunk g or g + 4
    [[maybe_unused]] auto fragments = [&](const char *buf, int h) {
#pragma unroll
        for (int i = 0; i < 2; i++) {
            wa[i][h] = *(const uint4 *)(buf + lds_off(wm * 32 + i * 16 + c16, g + 4 * h));
            wb[i][h] = *(const uint4 *)(buf + TILE + lds_off(wn * 32 + i * 16 + c16, g + 4 * h));
        }
    };
    [[maybe_unused]] auto half = [&](int h) {
        if constexpr (WIDE) {
            auto elem = [](const uint4 &v, int e) -> double {
                const uint32_t w = ((const uint32_t *)&v)[BF16 ? e >> 1 : e];
                return BF16 ? (double)__uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16)) : (double)__uint_as_float(w);
            };
#pragma unroll
            for (int e = 0; e < EPC; e++) {
                double x[2], y[2];
#pragma unroll
                for (int i = 0; i < 2; i++) { x[i] = elem(wa[i][h], e); y[i] = elem(wb[i][h], e); }
#pragma unroll
                for (int i = 0; i < 2; i++)
#pragma unroll
                    for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i], y[j], acc[i][j], 0, 0, 0);
            }
        }
    };
    if constexpr (WIDE) {
        fragments(lds[0], 0);
        fragments(lds[0], 1);
    }
    auto stage = [&](const char *cur, char *nxt, uint4 (&a)[NV], uint4 (&b)[NV]) {
        const char *sa = cur, *sb = cur + TILE;
        if constexpr (WIDE) {
            // the fragments were read under the MFMAs of the stage before, half of them (chunks g, chunks g + 4) at a time, so that
            // a wave alone on its SIMD does not wait for them
            store(a, b, nxt);
            load(a, b);
            half(0);
            const bool second = ck + BK / 2 < K;             // (chunks 4 to 7 of a last stage may hold zeros only)
            __syncthreads();
            fragments(nxt, 0);
            if (second) half(1);
            fragments(nxt, 1);
            ck = ck + BK < K ? ck + BK : 0;
            return;
        } else {
            uint4 fa[4], fb[4];
#pragma unroll
            for (int ks = 0; ks < 4; ks++) {
                fa[ks] = *(const uint4 *)(sa + lds_off(wm * 32 + lrow, 2 * ks + lhalf));
                fb[ks] = *(const uint4 *)(sb + lds_off(wn * 32 + lrow, 2 * ks + lhalf));
            }
            f32x16 part;
#pragma unroll
            for (int r = 0; r < 16; r++) part[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 4; ks++)
                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8 *)&fa[ks], *(const bf16x8 *)&fb[ks], part, 0, 0, 0);
            store(a, b, nxt);
            load(a, b);
#pragma unroll
            for (int r = 0; r < 16; r++) acc[0][0][r] += (double)part[r];
        }
        ck = ck + BK < K ? ck + BK : 0;
        __syncthreads();
    };
    for (int64_t st = 0; st < nst; st += D) {
#pragma unroll
        for (int d = 0; d < D; d++) {
            if (st + d >= nst) break;
            stage(lds[d & 1], lds[(d + 1) & 1], ra[(d + 1) % D], rb[(d + 1) % D]);
        }
    }

    // ---- epilogue: lane holds column (lane % 32) and rows 8*(r/4) + 4*(lane/32) + r%4 of its 32x32 tile; WIDE: column lane % 16
    // and rows 4*r + lane/16 of each 16x16 tile ----
    char *zb = (char *)p.out.ptr + (p.out.slab_elems ? agg * p.out.slab_elems * 4 : 0);
#pragma unroll
    for (int j = 0; j < MT; j++) {
        const int64_t n = n0 + wn * 32 + (WIDE ? j * 16 + c16 : lrow);
        if (n >= p.N) continue;
        int64_t unused, zn;
        decode_group(p.n, n, unused, zn);
#pragma unroll
        for (int i = 0; i < MT; i++)
#pragma unroll
            for (int r = 0; r < AR; r++) {
                const int64_t m = m0 + wm * 32 + (WIDE ? i * 16 + 4 * r + g : 8 * (r >> 2) + 4 * lhalf + (r & 3));
                if (m >= p.M) continue;
                int64_t zm;
                decode_group(p.m, m, unused, zm);
                const float val = (float)((double)p.alpha * acc[i][j][r]);
                const int64_t off = bz + zm + zn;
                if (p.out.dtype == EG_BF16) ((uint16_t *)zb)[off] = f32_to_bf16(val);
                else ((float *)zb)[off] = val;
            }
    }
}

// operands the kernel above takes: one run each along the contracted label and along what they are contiguous in, a chunk at least
bool contract_ragged_streams(const ContractParams &p)
{
    if (!p.ragged || p.otimes != EG_MUL || p.oplus != EG_AGG_SUM || p.k.n != 1) return false;
    const int epc = p.in_dtype == EG_BF16 ? 8 : 4;
    if (p.K < epc || p.K >= (1ll << 30)) return false;
    return (p.a_kcontig || (p.m.n == 1 && p.M >= epc)) && (p.b_kcontig || (p.n.n == 1 && p.N >= epc));
}

// A reduction of a stage or two under more tiles than run at once: the loads that the kernel above keeps in flight have nothing to run
// ahead of, and the tiles with run-by-run loads, of which more fit a compute unit, are faster (us there and here: 5101 x 31 x 3801 to
// bf16 36 and 43, x 97 48 and 47; bf16 to fp32 x 33 64 and 90, x 97 118 and 134, x 127 136 and 134, 2001 x 33 x 1403 14.4 and 17.7; fp32 x 33
// 72 and 79, x 63 90 and 88).
bool contract_ragged_short(const ContractParams &p, double tiles)
{
    if (p.n_totals > 1) return false;
    if (!p.wide) return p.K <= 64 && tiles > 1024;
    return p.K <= (p.in_dtype == EG_BF16 ? 112 : 72) && tiles > 512;
}

// Do they run faster with a tile's blocks one after another in one workgroup than each with its own, slabs and an aggregation?  Both
// ways in us, by rounds of 256 tiles (of two and three workgroups on a compute unit a round costs 0.8 to 0.9) and stages, with what a
// block costs that is walked over, and the slabs' way through memory at some 1.6 TB/s (they are small); two launches take 10 us at the
// least.  A stage of bf16 operands on the fp64 instruction may be cut short by half.  From 420 shapes of 17 to 2500 rows and columns
// and blocks of 9 to 1500 elements, each on both ways: the way taken is 0.5 to 1.5 % slower than the better one on average and
// at most 8 % slower than slabs.  (315 x (16 x 324) x 200 to bf16: slabs 16.9 us, totals 88.9; 1871 x (3 x 1335) x 706 bf16 to fp32
// 259 and 300; 3001 x (8 x 125) x 1530 fp32 287 and 215; 2477 x (8 x 81) x 1273 to bf16 85 and 41.)
bool contract_ragged_totals_pay(const ContractParams &p, int64_t n_agg, int out_bytes)
{
    if (n_agg < 2 || n_agg > INT32_MAX || p.n_tuples % n_agg || !contract_ragged_streams(p)) return false;
    const bool bf = p.in_dtype == EG_BF16;
    const double outs = (double)(p.n_tuples / n_agg * p.n_batch), tiles = outs * ((p.M + 63) / 64) * ((p.N + 63) / 64), n = (double)n_agg;
    const double mb = outs * p.M * p.N * (4 * n + out_bytes) * 1e-6, c = std::ceil(tiles / 256), w = std::ceil(tiles * n / 256);
    const double stages = bf && p.wide ? (double)((p.K + 31) / 32) / 2 : (double)((p.K + (bf ? 63 : 31)) / (bf ? 64 : 32));
    double totals, slabs;
    if (!p.wide) {
        totals = 6.1 + n * (0.62 * stages + 0.35) * std::max(1.0, 0.8 * c);
        slabs = 8.0 + std::max(1.0, 0.8 * w) * (0.632 * stages - 0.469) + 0.611 * mb;
    } else if (bf) {
        totals = 6.0 + n * (2.4 * stages + 0.6) * c;
        slabs = 6.9 + w * (2.58 * stages + 0.78) + 0.563 * mb;
    } else {
        totals = 7.2 + n * (1.35 * stages + 0.35) * std::max(1.0, 0.9 * c);
        slabs = 7.5 + std::max(1.0, 0.8 * w) * (1.454 * stages - 0.387) + 0.73 * mb;
    }
    return totals < std::max(slabs, 10.0);
}

static int launch_ragged_streams(ContractParams &p, void *stream)
{
    p.tiles_m = (int32_t)((p.M + 63) / 64);
    p.tiles_n = (int32_t)((p.N + 63) / 64);
    const int64_t wgs = p.n_tuples * p.n_batch * p.tiles_m * p.tiles_n;
    if (wgs < 1 || wgs >= (1ll << 31)) return fail(EG_ERR_LIMIT, "contraction needs %lld workgroups", (long long)wgs);
    const dim3 grid((unsigned)wgs), block(256);
    if (!p.wide) EG_LAUNCH((k_contract_ragged<true, false>), grid, block, 0, (hipStream_t)stream, p);
    else if (p.in_dtype == EG_BF16) EG_LAUNCH((k_contract_ragged<true, true>), grid, block, 0, (hipStream_t)stream, p);
    else EG_LAUNCH((k_contract_ragged<false, true>), grid, block, 0, (hipStream_t)stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(EG_ERR_HIP, "k_contract_ragged launch failed: %s", hipGetErrorString(e));
    return EG_OK;
}

// ------------------------------------------------------------------------------------------------
// The same tiling for any other scalar function (x) and reduction (+) of Section 3 of the paper (squared
// difference with sum, absolute difference with max, ...): no matrix instruction fits, so the tile is worked
// on the vector ALU.  256 threads as a 16 x 16 grid, each thread an 8 x 8 block of the 128 x 128 tile (4 x 4 of
// 64 x 64) with rows ty + 16 i and columns tx + 16 j (the 16 lanes that differ in tx read 16 consecutive LDS rows, which the
// swizzle spreads over all banks, and write consecutive columns).  Operands pass through the same loaders and
// the same LDS layout as above.  The reduction runs over exactly K values: zero-filled tail slots are skipped,
// since (x)(0, 0) need not be the identity of (+).
// ------------------------------------------------------------------------------------------------
// Bound by the issue of vector instructions: two of different waves go out together, so a SIMD whose second wave waits runs at half
// its rate.  Hence three workgroups per compute unit (168 registers a lane), no instruction right behind the one it waits for, and
// maxima of two k in one.  8192 x 1024 x 8192 cut 2 x 2 x 2, ms: squared differences 3.55 -> 2.61 (fp32), 3.14 -> 2.54 (bf16),
// largest absolute difference 2.94 -> 2.16, 2.68 -> 2.19; that is 26 to 32e12 label combinations a second, of 36e12 that a
// subtract and a multiply-add in registers reach.  Sums of blocks kept in the result instead of slabs (no aggregation, 0.13 ms
// each) cost the accumulators' registers: 2.89 ms.
template <typename C, int OT> constexpr int alu_waves() { return C::RAG || OT < 0 ? 2 : 3; }

template <typename C, int OT, int OP>
__global__ __launch_bounds__(C::THREADS, (alu_waves<C, OT>())) void k_contract_alu(const ContractParams p)
{
    fetch_params<sizeof(ContractParams)>();
    static_assert(C::BM == C::BN && (C::BM == 128 || C::BM == 64) && C::THREADS == 256, "16 x 16 threads of 8 x 8 or 4 x 4 outputs");
    constexpr int R = C::BM / 16;                            // rows and columns of a thread
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;

    const int64_t total = (int64_t)gridDim.x;
    int64_t logical;
    {
        const int64_t per = total / 8, rem = total % 8;
        const int64_t x = blockIdx.x % 8, j = blockIdx.x / 8;
        logical = x * per + (x < rem ? x : rem) + j;
    }
    const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n;
    const int64_t tb = logical / tiles;
    const int tl = (int)(logical - tb * tiles);
    const int tile_m = tl % p.tiles_m, tile_n = tl / p.tiles_m;
    const int64_t tuple = tb / p.n_batch, bidx = tb - tuple * p.n_batch;

    int64_t bx, by, bz, agg;
    decode_tuple(p.ts, tuple, bx, by, bz, agg);
    {
        uint32_t rem = (uint32_t)bidx;
        for (int i = p.batch.n - 1; i >= 0; i--) {
            uint32_t e = (uint32_t)p.batch.ext[i], q = rem / e, k = rem - q * e;
            rem = q;
            bx += (int64_t)k * p.batch.s0[i];
            by += (int64_t)k * p.batch.s1[i];
            bz += (int64_t)k * p.batch.s2[i];
        }
    }
    const int64_t m0 = (int64_t)tile_m * C::BM, n0 = (int64_t)tile_n * C::BN;

    Loader<C::BM, C::NVA, C::THREADS, C::BF16, C::RAG> la;
    Loader<C::BN, C::NVB, C::THREADS, C::BF16, C::RAG> lb;
    la.init(p.x, bx, p.m, m0, p.M, p.a_kcontig != 0, tid);
    lb.init(p.y, by, p.n, n0, p.N, p.b_kcontig != 0, tid);

    float acc[R][R];
    const float ident = oplus_identity(OP >= 0 ? OP : p.oplus);
#pragma unroll
    for (int i = 0; i < R; i++)
#pragma unroll
        for (int j = 0; j < R; j++) acc[i][j] = ident;
    // Ragged sums carry a compensation term (Kahan), as the one-output-per-lane kernel that took such shapes before did:
    // the same terms in the same order, four more instructions per term.  Only the ragged form has it at all: left unused in
    // the others it stayed in scratch memory where the operators are read at run time (1744 bytes a lane, 1472 without it).
    constexpr int CN = C::RAG ? R : 1;
    [[maybe_unused]] float comp[CN][CN];
    if constexpr (C::RAG) {
#pragma unroll
        for (int i = 0; i < R; i++)
#pragma unroll
            for (int j = 0; j < R; j++) comp[i][j] = 0.f;
    }

    const int64_t nk = (p.K + C::BK - 1) / C::BK;

    // element e of a 16-byte chunk
    auto elem_of = [](const uint4 &v, int e) -> float {
        const uint32_t w = ((const uint32_t *)&v)[C::BF16 ? e >> 1 : e];
        return C::BF16 ? __uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16)) : __uint_as_float(w);
    };
    // one 16-byte chunk (EPC consecutive k) of the thread's 8 rows and 8 columns; `valid` k of it count
    [[maybe_unused]] auto chunk = [&](const char *sa, const char *sb, int c, int valid) {
        uint4 a[R], b[R];
#pragma unroll
        for (int i = 0; i < R; i++) a[i] = *(const uint4 *)(sa + lds_off(ty + 16 * i, c));
#pragma unroll
        for (int j = 0; j < R; j++) b[j] = *(const uint4 *)(sb + lds_off(tx + 16 * j, c));
#pragma unroll
        for (int e = 0; e < C::EPC; e++) {
            if (e >= valid) break;
            float xs[R], ys[R];
#pragma unroll
            for (int i = 0; i < R; i++) {
                const uint32_t wa = ((const uint32_t *)&a[i])[C::BF16 ? e >> 1 : e], wb = ((const uint32_t *)&b[i])[C::BF16 ? e >> 1 : e];
                xs[i] = C::BF16 ? __uint_as_float((e & 1) ? (wa & 0xffff0000u) : (wa << 16)) : __uint_as_float(wa);
                ys[i] = C::BF16 ? __uint_as_float((e & 1) ? (wb & 0xffff0000u) : (wb << 16)) : __uint_as_float(wb);
            }
#pragma unroll
            for (int i = 0; i < R; i++)
#pragma unroll
                for (int j = 0; j < R; j++) acc[i][j] = oplus_t<OP>(p.oplus, acc[i][j], otimes_t<OT, false>(p.otimes, xs[i], ys[j], p.alpha));
            __builtin_amdgcn_sched_barrier(0);       // one k at a time: unpacking all of a chunk ahead of its use costs registers
        }
    };

    // The same for the two compiled pairs, a whole chunk.  Four columns at a time: 48 registers of operands instead of 64 let a third
    // workgroup onto the compute unit.  A row's four differences are taken before the previous row's are used (pinned: as the
    // compiler orders them, every difference is followed by the instruction that waits for it).
    // (Row + 64 has the swizzle key of row, so four offsets serve eight rows.)
    [[maybe_unused]] int pa[4], pb[4];
#pragma unroll
    for (int i = 0; i < 4; i++) { pa[i] = lds_off(ty + 16 * i, 0); pb[i] = C::LDS_A + lds_off(tx + 16 * i, 0); }
    [[maybe_unused]] auto whole_chunk = [&](int c) {
        constexpr bool PAIR = OT == EG_ABSDIFF && OP == EG_AGG_MAX;          // a maximum takes two k in one instruction
        constexpr int STEP = PAIR ? 2 : 1;
        uint4 a[R];
#pragma unroll
        for (int i = 0; i < R; i++) a[i] = *(const uint4 *)(smem + (pa[i & 3] ^ (c << 4)) + (i >> 2) * 8192);
#pragma unroll
        for (int h = 0; h < R / 4; h++) {
            uint4 b[4];
#pragma unroll
            for (int j = 0; j < 4; j++) b[j] = *(const uint4 *)(smem + (pb[j] ^ (c << 4)) + h * 8192);
#pragma unroll
            for (int e = 0; e < C::EPC; e += STEP) {
                float d[2][STEP][4];
                auto differences = [&](int i) {
#pragma unroll
                    for (int q = 0; q < STEP; q++) {
                        const float x = elem_of(a[i], e + q);
#pragma unroll
                        for (int j = 0; j < 4; j++) d[i & 1][q][j] = x - elem_of(b[j], e + q);
                        asm volatile("" : "+v"(d[i & 1][q][0]), "+v"(d[i & 1][q][1]), "+v"(d[i & 1][q][2]), "+v"(d[i & 1][q][3]));
                    }
                };
                differences(0);
#pragma unroll
                for (int i = 0; i < R; i++) {
                    if (i + 1 < R) differences(i + 1);
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        // (written out: fmaxf makes the compiler quieten the running maximum first, which is never a signalling NaN here)
                        if constexpr (PAIR) asm volatile("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(acc[i][4 * h + j]) : "v"(d[i & 1][0][j]), "v"(d[i & 1][STEP - 1][j]));
                        else asm volatile("v_fmac_f32 %0, %1, %1" : "+v"(acc[i][4 * h + j]) : "v"(d[i & 1][0][j]));
                    }
                }
            }
        }
    };

    // One LDS stage, no register prefetch: a stage is some ten microseconds of arithmetic per wave, the other
    // workgroups on the compute unit cover the loads, and the registers are needed for the 8 x 8 block.
    const char *sa = smem, *sb = smem + C::LDS_A;
    // (the compiled pairs take whole stages here and the rest behind the loop: with both in it, all accumulators were moved once per chunk)
    const int64_t nloop = !C::RAG && OT >= 0 ? p.K / C::BK : nk;
    for (int64_t kt = 0; kt < nloop; kt++) {
        la.fetch(p.k, 0, kt * C::BK, p.K, tid, p.m, p.M);
        lb.fetch(p.k, 1, kt * C::BK, p.K, tid, p.n, p.N);
        la.commit(smem, tid);
        lb.commit(smem + C::LDS_A, tid);
        __syncthreads();
        const int64_t left = p.K - kt * C::BK;
        if constexpr (C::RAG) {
            // one k at a time, read as elements (the compensation terms take the registers of whole chunks)
            const int n = left < C::BK ? (int)left : C::BK;
#pragma unroll 1
            for (int k = 0; k < n; k++) {
                auto elem = [&](const char *tile, int row) -> float {
                    const char *q = tile + lds_off(row, k / C::EPC) + (k % C::EPC) * C::ESZ;
                    return C::BF16 ? bf16_to_f32(*(const uint16_t *)q) : *(const float *)q;
                };
                float xs[R], ys[R];
#pragma unroll
                for (int i = 0; i < R; i++) { xs[i] = elem(sa, ty + 16 * i); ys[i] = elem(sb, tx + 16 * i); }
#pragma unroll
                for (int i = 0; i < R; i++)
#pragma unroll
                    for (int j = 0; j < R; j++) {
                        const float v = otimes_t<OT, false>(p.otimes, xs[i], ys[j], p.alpha);
                        if ((OP >= 0 ? OP : p.oplus) == EG_AGG_SUM) {
                            const float u = v - comp[i][j], s = acc[i][j] + u;
                            comp[i][j] = (s - acc[i][j]) - u;
                            acc[i][j] = s;
                        } else {
                            acc[i][j] = oplus_t<OP>(p.oplus, acc[i][j], v);
                        }
                    }
            }
        } else if constexpr (OT >= 0) {
#pragma unroll 1
            for (int c = 0; c < 8; c++) whole_chunk(c);
        } else if (left >= C::BK) {
#pragma unroll 1
            for (int c = 0; c < 8; c++) chunk(sa, sb, c, C::EPC);
        } else {
            for (int c = 0; c * C::EPC < left; c++) chunk(sa, sb, c, (int)(left - c * C::EPC < C::EPC ? left - c * C::EPC : C::EPC));
        }
        __syncthreads();
    }
    if constexpr (!C::RAG && OT >= 0) {
        if (nloop < nk) {
            la.fetch(p.k, 0, nloop * C::BK, p.K, tid, p.m, p.M);
            lb.fetch(p.k, 1, nloop * C::BK, p.K, tid, p.n, p.N);
            la.commit(smem, tid);
            lb.commit(smem + C::LDS_A, tid);
            __syncthreads();
            const int left = (int)(p.K - nloop * C::BK);
#pragma unroll 1
            for (int c = 0; c < left / C::EPC; c++) whole_chunk(c);
#pragma unroll 1
            for (int k = left / C::EPC * C::EPC; k < left; k++) {
                auto elem = [&](const char *tile, int row) -> float {
                    const char *q = tile + lds_off(row, k / C::EPC) + (k % C::EPC) * C::ESZ;
                    return C::BF16 ? bf16_to_f32(*(const uint16_t *)q) : *(const float *)q;
                };
                float xs[R], ys[R];
#pragma unroll
                for (int i = 0; i < R; i++) { xs[i] = elem(sa, ty + 16 * i); ys[i] = elem(sb, tx + 16 * i); }
#pragma unroll
                for (int i = 0; i < R; i++)
#pragma unroll
                    for (int j = 0; j < R; j++) acc[i][j] = oplus_t<OP>(p.oplus, acc[i][j], otimes_t<OT, false>(p.otimes, xs[i], ys[j], p.alpha));
            }
        }
    }

    char *zb = (char *)p.out.ptr + (p.out.slab_elems ? agg * p.out.slab_elems * 4 : 0);
    const bool out_bf16 = p.out.dtype == EG_BF16;
    int64_t zn[R];
#pragma unroll
    for (int j = 0; j < R; j++) {
        const int64_t n = n0 + tx + 16 * j;
        int64_t unused;
        decode_group(p.n, n < p.N ? n : 0, unused, zn[j]);
    }
#pragma unroll
    for (int i = 0; i < R; i++) {
        const int64_t m = m0 + ty + 16 * i;
        if (m >= p.M) continue;
        int64_t unused, zm;
        decode_group(p.m, m, unused, zm);
#pragma unroll
        for (int j = 0; j < R; j++) {
            if (n0 + tx + 16 * j >= p.N) continue;
            const int64_t off = bz + zm + zn[j];
            if (out_bf16) ((uint16_t *)zb)[off] = f32_to_bf16(acc[i][j]);
            else ((float *)zb)[off] = acc[i][j];
        }
    }
}

template <typename C, int OT, int OP>
static int launch_alu(ContractParams &p, void *stream)
{
    p.tiles_m = (int32_t)((p.M + C::BM - 1) / C::BM);
    p.tiles_n = (int32_t)((p.N + C::BN - 1) / C::BN);
    const int64_t wgs = p.n_tuples * p.n_batch * p.tiles_m * p.tiles_n;
    if (wgs < 1 || wgs >= (1ll << 31)) return fail(EG_ERR_LIMIT, "contraction needs %lld workgroups", (long long)wgs);
    static bool attr_set = false;
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)k_contract_alu<C, OT, OP>, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_A + C::LDS_B) != hipSuccess)
            return fail(EG_ERR_HIP, "cannot reserve %d bytes of LDS", C::LDS_A + C::LDS_B);
        attr_set = true;
    }
    EG_LAUNCH((k_contract_alu<C, OT, OP>), dim3((unsigned)wgs), dim3(C::THREADS), C::LDS_A + C::LDS_B, (hipStream_t)stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(EG_ERR_HIP, "k_contract_alu launch failed: %s", hipGetErrorString(e));
    return EG_OK;
}

template <typename C>
static int launch_alu_ops(ContractParams &p, void *stream)
{
    // The compiled pairs: 64 x 64 tiles while there are fewer than two 128 x 128 ones for a compute unit.  A wave alone on its SIMD issues
    // one instruction in the time of two, and a small launch is as long as a tile (192 x (2 x 192) x 1984 to fp32
    // 68.3 us with 128 x 128, 30.5 with 64 x 64; 256 x (2 x 512) x 512 158 and 62; 1280 x (2 x 52) x 2304, 360 tiles, 40.4 and 35.1; from 512
    // on the large ones: 2048 x (2 x 256) x 3072, 768 tiles, 157 and 176).
    if constexpr (!C::RAG && C::BM == 128) {
        const int64_t tiles = p.n_tuples * p.n_batch * ((p.M + 127) / 128) * ((p.N + 127) / 128);
        if (tiles < 512 && ((p.otimes == EG_SQDIFF && p.oplus == EG_AGG_SUM) || (p.otimes == EG_ABSDIFF && p.oplus == EG_AGG_MAX)))
            return launch_alu_ops<Cfg<64, 64, 32, 32, C::BF16>>(p, stream);
    }
    // the paper's two examples are compiled in; any other pair reads its operators at run time, which the ragged form does not
    // (9.6 us per contracted element of a tile against 1.0): of others it has the sum of absolute differences only
    if (p.otimes == EG_SQDIFF && p.oplus == EG_AGG_SUM) return launch_alu<C, EG_SQDIFF, EG_AGG_SUM>(p, stream);
    if (p.otimes == EG_ABSDIFF && p.oplus == EG_AGG_MAX) return launch_alu<C, EG_ABSDIFF, EG_AGG_MAX>(p, stream);
    if constexpr (C::BM == 64) {
        return fail(EG_ERR_BAD_OP, "contraction: no 64 x 64 tiles for scalar function %d", p.otimes);
    } else if constexpr (C::RAG) {
        if (p.otimes == EG_ABSDIFF && p.oplus == EG_AGG_SUM) return launch_alu<C, EG_ABSDIFF, EG_AGG_SUM>(p, stream);
        return fail(EG_ERR_BAD_OP, "contraction: no tiles for scalar function %d of ragged operands", p.otimes);
    } else {
        return launch_alu<C, -1, -1>(p, stream);
    }
}

template <typename C>
static int launch_cfg(ContractParams &p, void *stream)
{
    p.tiles_m = (int32_t)((p.M + C::BM - 1) / C::BM);
    p.tiles_n = (int32_t)((p.N + C::BN - 1) / C::BN);
    const int64_t wgs = p.n_tuples * p.n_batch * p.tiles_m * p.tiles_n;
    if (wgs < 1 || wgs >= (1ll << 31)) return fail(EG_ERR_LIMIT, "contraction needs %lld workgroups", (long long)wgs);
    static bool attr_set = false;
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)k_contract<C>, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES) != hipSuccess)
            return fail(EG_ERR_HIP, "cannot reserve %d bytes of LDS", C::LDS_BYTES);
        attr_set = true;
    }
    EG_LAUNCH(k_contract<C>, dim3((unsigned)wgs), dim3(C::THREADS), C::LDS_BYTES, (hipStream_t)stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(EG_ERR_HIP, "k_contract launch failed: %s", hipGetErrorString(e));
    return EG_OK;
}

// Blocks with at least 128 rows or columns take the direct-to-LDS kernel when their layout allows; force_kernel
// (tr_set_contract_variant) forces one of the two.  A handful of small fp32 blocks (configuration 1: eight blocks of
// 128^3) is a latency chain of slow MFMAs on as many compute units, which 64 x 64 tiles of the register-staged kernel
// spread over four times as many.  (Skinny products included: with 8192 x 4096 x 32..96 the half-empty tiles of that
// kernel still finish in 0.045 ms against 0.105-0.124 ms here.)
bool contract_takes_dma(const ContractParams &p)
{
    if (p.otimes != EG_MUL || p.oplus != EG_AGG_SUM) return false;
    const int64_t tiles128 = p.n_tuples * p.n_batch * ((p.M + 127) / 128) * ((p.N + 127) / 128);
    const bool tiny_f32 = p.in_dtype == EG_F32 && tiles128 <= 64;
    const bool want_dma = p.force_kernel ? p.force_kernel == 2 : ((p.M >= 128 || p.N >= 128) && !tiny_f32);
    return want_dma && contract_dma_eligible(p);
}

// Ragged operands.  Such shapes were summed with a compensation term before, to a unit in the last place of a 32-bit sum,
// which an fp32 accumulator does not reach, so no sum is left to one.  Results of bf16 from bf16 operands run on the bf16 matrix
// instruction one stage of 64 at a time, the stages' sums are added in 64 bits.  Results of 32 bits, and of fp32 operands, run
// on the fp64 matrix instruction, exact products and 64-bit sums.  64 x 64 tiles throughout: the 64-bit totals take 128
// registers of a 128 x 128 tile's lanes, and with one wave per SIMD left, or two of half the tile, nothing hides the loads
// (4001 x 3001 x 4099: 447 us with 64 x 64, 557 with 128 x 64, 592 with 128 x 128; 439 with 128 x 128 and plain fp32 sums).
// Operands of one run each take k_contract_ragged; the forms with run-by-run loads are left for the others (two contracted labels that
// do not join, runs of a few elements) and for short reductions under many tiles.  Against one output per lane, which ran such shapes before there were tiles: fp32
// 1121 x 319 x 646 371 us, 20 now; a classifier's step of 1000 x 3001 x 1530 x 1003 23.5 ms, 0.50 now.
static int launch_ragged(ContractParams &p, void *stream)
{
    if (p.otimes != EG_MUL || p.oplus != EG_AGG_SUM) {
        if (p.n_totals > 1) return fail(EG_ERR_LIMIT, "contraction: no totals of blocks on this form");
        if (p.otimes < EG_MUL || p.otimes > EG_SILU_MUL) return fail(EG_ERR_BAD_OP, "contraction: scalar function %d is not binary", p.otimes);
        if (p.in_dtype == EG_BF16) return launch_alu_ops<Cfg<128, 128, 64, 64, true, true>>(p, stream);
        return launch_alu_ops<Cfg<128, 128, 64, 64, false, true>>(p, stream);
    }
    if (contract_ragged_streams(p) && !contract_ragged_short(p, (double)(p.n_tuples * p.n_batch * ((p.M + 63) / 64) * ((p.N + 63) / 64)))) {
        if (!p.wide && p.in_dtype != EG_BF16) return fail(EG_ERR_LIMIT, "contraction: ragged fp32 operands are summed in 64 bits");
        return launch_ragged_streams(p, stream);
    }
    if (p.n_totals > 1) return fail(EG_ERR_LIMIT, "contraction: no totals of blocks on this form");
    if (p.wide) {
        if (p.in_dtype == EG_BF16) return launch_cfg<Cfg<64, 64, 32, 32, true, true, true>>(p, stream);
        return launch_cfg<Cfg<64, 64, 32, 32, false, true, true>>(p, stream);
    }
    if (p.in_dtype != EG_BF16) return fail(EG_ERR_LIMIT, "contraction: ragged fp32 operands are summed in 64 bits");
    return launch_cfg<Cfg<64, 64, 32, 32, true, true>>(p, stream);
}

int launch_contract(ContractParams &p, void *stream)
{
    // what the kernel assumes, re-checked here so that a wrong table can never reach the device
    if (!p.x || !p.y || !p.out.ptr) return fail(EG_ERR_NULL, "contraction: NULL operand");
    if (p.m.n < 1 || p.n.n < 1 || p.k.n < 1 || p.M < 1 || p.N < 1 || p.K < 1 || p.n_batch < 1 || p.n_tuples < 1)
        return fail(EG_ERR_LIMIT, "contraction: empty role group");
    if (p.ragged) {
        const bool one_a = p.a_kcontig ? p.k.s0[p.k.n - 1] == 1 : p.m.s0[p.m.n - 1] == 1;
        const bool one_b = p.b_kcontig ? p.k.s1[p.k.n - 1] == 1 : p.n.s0[p.n.n - 1] == 1;
        if (!one_a || !one_b) return fail(EG_ERR_LIMIT, "contraction: operand is not contiguous along its innermost label");
        return launch_ragged(p, stream);
    }
    const int epc = p.in_dtype == EG_BF16 ? 8 : 4;
    const bool ok_a = p.a_kcontig ? (p.k.s0[p.k.n - 1] == 1 && p.k.ext[p.k.n - 1] % epc == 0)
                                  : (p.m.s0[p.m.n - 1] == 1 && p.m.ext[p.m.n - 1] % epc == 0);
    const bool ok_b = p.b_kcontig ? (p.k.s1[p.k.n - 1] == 1 && p.k.ext[p.k.n - 1] % epc == 0)
                                  : (p.n.s0[p.n.n - 1] == 1 && p.n.ext[p.n.n - 1] % epc == 0);
    if (!ok_a || !ok_b) return fail(EG_ERR_LIMIT, "contraction: operand is not vectorisable along its contiguous label");
    if (((uintptr_t)p.x & 15) || ((uintptr_t)p.y & 15)) return fail(EG_ERR_LIMIT, "contraction: operands must be 16-byte aligned");
    if (p.otimes != EG_MUL || p.oplus != EG_AGG_SUM) {
        if (p.otimes < EG_MUL || p.otimes > EG_SILU_MUL) return fail(EG_ERR_BAD_OP, "contraction: scalar function %d is not binary", p.otimes);
        if (p.in_dtype == EG_BF16) return launch_alu_ops<Cfg<128, 128, 64, 64, true>>(p, stream);
        return launch_alu_ops<Cfg<128, 128, 64, 64, false>>(p, stream);
    }
    const int64_t tiles128 = p.n_tuples * p.n_batch * ((p.M + 127) / 128) * ((p.N + 127) / 128);
    if (contract_takes_dma(p)) return launch_contract_dma(p, stream);
    if (p.n_totals > 1) return fail(EG_ERR_LIMIT, "contraction: totals of blocks are kept by the direct-to-LDS kernel only");
    if (tiles128 <= 64) {
        if (p.in_dtype == EG_BF16) return launch_cfg<Cfg<64, 64, 32, 32, true>>(p, stream);
        return launch_cfg<Cfg<64, 64, 32, 32, false>>(p, stream);
    }
    if (p.in_dtype == EG_BF16) return launch_cfg<Cfg<128, 128, 64, 64, true>>(p, stream);
    // fp32 shapes the direct-to-LDS kernel cannot take: 256 x 256 tiles (eight waves of 128 x 64) once there are enough
    // of them to occupy half the chip (measured 98-113 TFLOP/s on 4096^3 and 8192^3 against 81-101 with 128 x 128 tiles)
    const int64_t tiles256 = p.n_tuples * p.n_batch * ((p.M + 255) / 256) * ((p.N + 255) / 256);
    if (tiles256 >= 128) return launch_cfg<Cfg<256, 256, 128, 64, false>>(p, stream);
    return launch_cfg<Cfg<128, 128, 64, 64, false>>(p, stream);
}

}  // namespace eg
