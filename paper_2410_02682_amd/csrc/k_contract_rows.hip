// Block contraction of a few rows with a large matrix (a token's activations times a weight matrix): X has at most 16 rows, each
// contiguous along the one contracted label; Y is whole 16-byte vectors along its columns or along the contracted label.
//
// Bound by the way of Y from memory.  The 128 x 128 tiles spend their LDS, barriers and stages on rows that are not there; here
// every wave streams its own part of Y into registers, two iterations of 4 or 8 KiB in flight (four were slower: waves have four
// to sixteen iterations, and branches around the loads make the compiler wait for all of them), and feeds it to 16x16x32 MFMAs
// whose other operand is X, padded to 16 rows by loads outside its descriptor.  No LDS before the end, where the eight waves of a
// workgroup, which split its part of the contracted label, add their sums in ascending order.  us with Y from memory, aggregation
// of the pieces included, tiles and now: 8 x 4096 x 4096 24.0 and 11.6 (33.5 MB), 8 x 4096 x 11008 30.1 and 22.4 (4.0 TB/s),
// 8 x (8 x 1376) x 4096 30.8 and 22.7, 8 x 4096 x 4096 with Y along k 23.6 and 10.6.
//   Y contiguous along its columns: a lane takes VC neighbouring columns of eight consecutive k and turns them around in
//       registers (v_perm), which gives VC fragments; fragment f of lane c stands for column VC * c + f of the wave's 16 * VC.
//   Y contiguous along k: a lane's 16 bytes are a fragment already; a wave takes 16 columns and 128 k per iteration (256 took 155
//       registers, one workgroup to a compute unit, and launches of a few more than 256 a second round: 8 x 768 x 12160 16.6 -> 12.7).
// A launch is cut along the contracted label into at most as many pieces as the vertex has partial slabs: so many that the busiest
// compute unit has the least to fetch (rows_us).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "eg_device.h"

namespace eg {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

namespace rows {

constexpr int kWaves = 8;

__device__ __forceinline__ void decode(const DimList &g, int64_t idx, int64_t &o0, int64_t &o1)
{
    o0 = o1 = 0;
    uint32_t rem = (uint32_t)idx;
    for (int i = g.n - 1; i >= 0; i--) {
        const uint32_t e = (uint32_t)g.ext[i], q = rem / e, k = rem - q * e;
        rem = q;
        o0 += (int64_t)k * g.s0[i];
        o1 += (int64_t)k * g.s1[i];
    }
}

// YK: Y is contiguous along k.  VC: columns of a lane (8 or 4) when it is not.
template <bool YK, int VC>
__global__ __launch_bounds__(kWaves * 64, 2) void k_contract_rows(const ContractParams p)
{
    fetch_params<sizeof(ContractParams)>();
    constexpr int COLS = YK ? 16 : 16 * VC, KI = YK ? 128 : 32, NL = YK ? 4 : 8;      // columns of a workgroup, k of an iteration, loads of Y per iteration
    constexpr int NX = KI / 32;                                              // fragments of X per iteration
    constexpr int PITCH = COLS + 4;
    __shared__ __attribute__((aligned(16))) float sums[kWaves][16 * PITCH];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15, g = lane >> 4;
    // Where rows of Y are no whole 128-byte lines, neighbouring strips share lines: they run on one XCD then and find them in its L2
    // (16 x (4 x 2768) x 8624 82 -> 71 us; with whole lines 34.6 -> 36.0 on 15 x 5544 x 11264, so not there).
    uint32_t strip = blockIdx.x, part = blockIdx.y;
    if (p.k_align) {
        const uint32_t id = blockIdx.y * gridDim.x + blockIdx.x, total = gridDim.x * gridDim.y, per = total / 8, rem8 = total % 8, xcd = id % 8;
        const uint32_t logical = xcd * per + (xcd < rem8 ? xcd : rem8) + id / 8;
        part = logical / gridDim.x;
        strip = logical - part * gridDim.x;
    }
    const int64_t n0 = (int64_t)strip * COLS;
    const int32_t piece = (int32_t)part, M = (int32_t)p.M;

    // this wave's k: a part of the piece, whole iterations of 32 (p.k_stages: k per piece)
    const int32_t K = (int32_t)p.K, first = piece * p.k_stages, last = first + p.k_stages < K ? first + p.k_stages : K;
    const int32_t share = ((p.k_stages + kWaves - 1) / kWaves + 31) / 32 * 32;
    const int32_t kb = first + wave * share, ke = kb + share < last ? kb + share : last;

    // lane offsets in bytes from the wave's first k; a chunk outside is given an offset outside the descriptor and arrives as zeros
    const int64_t sx = p.k.s0[0], sy = p.k.s1[0];                            // element strides of k
    int64_t xo, yo, unused;
    decode(p.m, c16 < M ? c16 : 0, xo, unused);
    const int64_t col = n0 + (YK ? c16 : VC * c16);
    const bool inside = col < p.N;                                           // (N is a multiple of VC)
    decode(p.n, inside ? col : 0, yo, unused);
    auto uniform = [](const char *q) {
        const uint64_t v = (uint64_t)q;
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));   // (they return int)
        return (const char *)(((uint64_t)hi << 32) | lo);
    };
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)uniform((const char *)p.x + (int64_t)kb * sx * 2), 0, (int)0x80000000u, 0x00020000);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void *)uniform((const char *)p.y + (int64_t)kb * sy * 2), 0, (int)0x80000000u, 0x00020000);
    const uint32_t x0 = (uint32_t)(xo + 8 * g) * 2, y0 = (uint32_t)(yo + 8 * g * sy) * 2, ystep = (uint32_t)sy * 2;
    const int32_t kn = ke - kb;                                              // may be negative: nothing to do

    u32x4 xf[2][NX], yf[2][NL];
    auto load = [&](int32_t k, u32x4 (&x)[NX], u32x4 (&y)[NL]) {             // k from the wave's first one
#pragma unroll
        for (int j = 0; j < NL; j++) {
            const int32_t kk = k + 8 * g + (YK ? 32 * j : j);
            const uint32_t o = inside && kk < kn ? y0 + (uint32_t)(k + (YK ? 32 * j : j)) * ystep : 0x80000000u;
            if (YK || VC == 8) y[j] = __builtin_amdgcn_raw_buffer_load_b128(ry, (int)o, 0, 2);
            else {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(ry, (int)o, 0, 2);
                y[j].x = v.x; y[j].y = v.y;
            }
        }
#pragma unroll
        for (int j = 0; j < NX; j++) {
            const int32_t kk = k + 32 * j;
            x[j] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(c16 < M && kk + 8 * g < kn ? x0 + (uint32_t)kk * 2 : 0x80000000u), 0, 0);
        }
    };
    constexpr int NF = YK ? 1 : VC;                                          // fragments of 16 columns
    f32x4 acc[NF];
#pragma unroll
    for (int f = 0; f < NF; f++) acc[f] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const u32x4 (&x)[NX], const u32x4 (&y)[NL]) {
        if constexpr (YK) {
#pragma unroll
            for (int j = 0; j < NL; j++)
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[j]), __builtin_bit_cast(bf16x8, y[j]), acc[0], 0, 0, 0);
        } else {
#pragma unroll
            for (int d = 0; d < VC / 2; d++) {                               // columns 2 d and 2 d + 1: eight k each, from eight rows
                u32x4 lo, hi;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    lo[j] = __builtin_amdgcn_perm(y[2 * j + 1][d], y[2 * j][d], 0x05040100u);
                    hi[j] = __builtin_amdgcn_perm(y[2 * j + 1][d], y[2 * j][d], 0x07060302u);
                }
                acc[2 * d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[0]), __builtin_bit_cast(bf16x8, lo), acc[2 * d], 0, 0, 0);
                acc[2 * d + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[0]), __builtin_bit_cast(bf16x8, hi), acc[2 * d + 1], 0, 0, 0);
            }
        }
    };
    // two iterations in flight; loads behind the last k fetch nothing
    load(0, xf[0], yf[0]);
    for (int32_t k = 0; k < kn; k += 2 * KI) {
        load(k + KI, xf[1], yf[1]);
        multiply(xf[0], yf[0]);
        load(k + 2 * KI, xf[0], yf[0]);
        multiply(xf[1], yf[1]);
    }

    // lane: column c16 of a fragment, rows 4 g .. 4 g + 3
#pragma unroll
    for (int r = 0; r < 4; r++) {
        float *s = sums[wave] + (4 * g + r) * PITCH + NF * c16;
        if constexpr (NF == 1) s[0] = acc[0][r];
        else {
#pragma unroll
            for (int f = 0; f < NF; f += 4) *(f32x4 *)(s + f) = (f32x4){acc[f][r], acc[f + 1][r], acc[f + 2][r], acc[f + 3][r]};
        }
    }
    __syncthreads();
    char *zb = (char *)p.out.ptr + (p.out.slab_elems ? piece * p.out.slab_elems * 4 : 0);
    for (int e = tid; e < M * COLS; e += kWaves * 64) {
        const int m = e / COLS, c = e % COLS;
        if (n0 + c >= p.N) continue;
        float s = sums[0][m * PITCH + c];
#pragma unroll
        for (int w = 1; w < kWaves; w++) s += sums[w][m * PITCH + c];
        int64_t zm, zn;
        decode(p.m, m, unused, zm);
        decode(p.n, n0 + c, unused, zn);
        s *= p.alpha;
        if (p.out.dtype == EG_BF16) ((uint16_t *)zb)[zm + zn] = f32_to_bf16(s);
        else ((float *)zb)[zm + zn] = s;
    }
}

}  // namespace rows

// p: a contraction in one piece (no blocks, no batch label).  The MFMA rows beyond M are idle, and a wave's part of Y has to
// be long enough to be a stream.
bool contract_rows_suits(const ContractParams &p)
{
    if (p.ragged || p.in_dtype != EG_BF16 || p.otimes != EG_MUL || p.oplus != EG_AGG_SUM) return false;
    if (p.force_kernel || p.force_tile_m || p.force_waves) return false;
    if (p.n_tuples != 1 || p.n_batch != 1 || p.k.n != 1 || !p.a_kcontig || p.k.s0[0] != 1) return false;
    if (p.M > 16 || p.N < 64 || p.K < 256 || p.K >= (1 << 30)) return false;
    auto span = [](const DimList &g, const int64_t *s) { int64_t t = 0; for (int i = 0; i < g.n; i++) { if (s[i] < 0) return (int64_t)1 << 40; t += (g.ext[i] - 1) * s[i]; } return t; };
    if (p.k.s1[0] < 1) return false;
    // 32-bit byte offsets from a wave's first k, iterations past the last one included
    const int64_t over = p.K + 2048;
    if (over + span(p.m, p.m.s0) >= (1ll << 30) || over * p.k.s1[0] + span(p.n, p.n.s0) >= (1ll << 30)) return false;
    if (((uintptr_t)p.x & 15) || ((uintptr_t)p.y & 15)) return false;
    // Y along k: a strip of 16 columns fetches X whole, which is as much again at 16 rows; the tiles stream large matrices of whole
    // 128-byte lines faster then (16 x 4096 x 14336 34.2 us on the tiles, 39.7 here; 16 x 2560 x 12288 1.14 times faster here, 12 x 4096 x
    // 8128 1.07, and 16 x 9168 x 12288, whose rows are no whole lines, 1.23; 8 x 8192 x 14336 63.0 and 62.2 from memory, but 42 and 62
    // where the matrix stays in the last-level cache from call to call)
    if (p.b_kcontig && p.M > 4 && p.K * p.N > (p.M > 8 ? 40000000 : 80000000) && p.n.s0[p.n.n - 1] % 64 == 0) return false;
    return true;
}

// us of a launch in so many pieces, beyond what all of them have: the busiest compute unit's share of Y at the rate a unit fetches it
// (strips of 128 columns keep more in flight than those of 64), or all of it at the memory's; and an aggregation's.  Over 90 shapes of
// either layout, Y from memory, each in 1 to 8 pieces and with either strip, its choice is 0.3 (0.6) % slower than the best on average
// and 6 % at most; of up to 64 pieces (65536 and 100352 by 64 to 320) the aggregation takes little more than of eight.  (One piece from 160 strips on, 256 workgroups and more below, took 29.7 us for 15 x (4 x 768) x 9240, now 18.8; 31.7 for
// 8 x 7936 x 6400, now 22.6: workgroups beyond 256 made a second round.)
static double rows_us(const ContractParams &p, bool wide, int64_t pieces)
{
    const int64_t cols = p.b_kcontig ? 16 : wide ? 128 : 64, on_unit = ((p.N + cols - 1) / cols * pieces + 255) / 256;
    const double unit = p.b_kcontig ? 18e3 : wide ? 28e3 : 20e3, memory = p.b_kcontig ? 4e6 : 6e6;          // bytes per us
    const double us = std::max((double)p.K * p.N * 2 / memory, (double)(on_unit * cols * 2 * ((p.K + pieces - 1) / pieces)) / unit);
    return us + (pieces > 1 ? 1.5 + 0.2 * std::min<int64_t>(pieces, 8) + 0.02 * pieces + (double)(p.M * p.N * 4 * pieces) / 2e6 : 0);
}

static bool rows_wide(const ContractParams &p, int64_t pieces) { return !p.b_kcontig && rows_us(p, true, pieces) < rows_us(p, false, pieces); }

// How many pieces the contracted label is cut into, of at most `slabs` and of 256 elements at least; and so many that
// no wave sums up more of it than a slab's block does.  0: more than a grid has room for, not for this kernel
constexpr int64_t kMaxPieces = 65535;
int contract_rows_pieces(const ContractParams &p, int64_t slabs)
{
    const int64_t least = (slabs + rows::kWaves - 1) / rows::kWaves, most = std::max(least, std::min(std::min(slabs, p.K / 256), kMaxPieces));
    int64_t best = least;
    double us = -1;
    for (int w = 0; w < (p.b_kcontig ? 1 : 2); w++) {
        // the fewest, and of all numbers that give the busiest unit the same number of workgroups the largest
        const int64_t cols = p.b_kcontig ? 16 : w ? 128 : 64, strips = (p.N + cols - 1) / cols;
        int64_t s = least;
        for (int64_t u = (strips * least + 255) / 256, tries = 0; tries < 16; u++, tries++) {
            const double t = rows_us(p, w != 0, s);
            if (us < 0 || t < us) { best = s; us = t; }
            if (s == most) break;
            s = std::min(std::max(256 * u / strips, s), most);
        }
    }
    return best <= kMaxPieces ? (int)best : 0;
}

int launch_contract_rows(ContractParams &p, int pieces, void *stream)
{
    if (!p.x || !p.y || !p.out.ptr) return fail(EG_ERR_NULL, "contraction: NULL operand");
    if (!contract_rows_suits(p) || pieces < 1 || pieces > kMaxPieces || (pieces > 1) != (p.out.slab_elems != 0)) return fail(EG_ERR_LIMIT, "contraction: shape not eligible for the few-row kernel");
    p.k_stages = (int32_t)(((p.K + pieces - 1) / pieces + 31) / 32 * 32);
    p.k_align = !p.b_kcontig && p.k.s1[0] * 2 % 128 != 0;
    const bool wide = rows_wide(p, pieces);
    const int cols = p.b_kcontig ? 16 : wide ? 128 : 64;
    const dim3 grid((unsigned)((p.N + cols - 1) / cols), (unsigned)pieces), block(rows::kWaves * 64);
    hipStream_t st = (hipStream_t)stream;
    if (p.b_kcontig) EG_LAUNCH((rows::k_contract_rows<true, 8>), grid, block, 0, st, p);
    else if (wide) EG_LAUNCH((rows::k_contract_rows<false, 8>), grid, block, 0, st, p);
    else EG_LAUNCH((rows::k_contract_rows<false, 4>), grid, block, 0, st, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(EG_ERR_HIP, "k_contract_rows launch failed: %s", hipGetErrorString(e));
    return EG_OK;
}

}  // namespace eg
