// dd_gemm.hip -- bf16 matrix products of the transformer block around the
// attention (the projections and the MLP of one OpenLM block) on gfx950
// matrix cores:  C[M, N] = op(A) op(B),  bf16 inputs, fp32 accumulation.
//
//   op(A) = A, stored [M][K] with row stride lda, or A^T with A stored [K][M]
//   op(B) = B, stored [K][N] with row stride ldb, or B^T with B stored [N][K]
//
// A forward projection y = x W is (A, B) = (x, W); the backward's input
// gradient dx = dy W^T is (dy, W^T) and its weight gradient dW = x^T dy is
// (x^T, dy).
//
// One workgroup (8 waves) computes a 256 x 256 tile of C.  The K axis is
// walked in 64-wide steps; the A and B tiles of a step are two halves of 128
// rows (columns) each, in two LDS stages (128 KiB).  Wave (wm, wn) owns rows
// 64 wm .. +63 of each A half and columns 32 wn .. +31 of each B half: four
// 64 x 32 quadrants, one per pair of halves.  A step is four phases, one
// quadrant's 16 products each:
//
//   phase            1        2        3        4
//   products         A0 B0    A0 B1    A1 B1    A1 B0
//   LDS reads        B0       B1       A1       A0 of the next step
//   loads started    A0       B0       B1       A1, all of step + 2
//
// The loads refill the half that the phase before has read, so each has six
// phases (1.5 steps) to arrive; a phase waits only for the loads that the
// next phase's reads need (vmcnt(12): six halves stay in flight).  Waves 4-7
// run half a phase behind waves 0-3 (one extra barrier before the loop): on
// every SIMD one wave issues its 16 products while the other reads its next
// operands and starts loads.  Loads go directly from global memory to LDS
// and waits are explicit: the compiler would otherwise wait for every load
// before each transposing LDS read.
//
// What bounds it: power.  At 8192^3 the matrix pipes are busy 76-83% of the
// time (50% with one barrier per step and all waves in phase) at a shader
// clock of 1.4-1.7 GHz of 2.4; the 32x32x16 product kept them 89% busy at 1.35
// GHz and was 7% slower, so the 16x16x32 product is used.  At K = 2048 they
// are busy 69-75%: tile starts and ends.  Measured (TFLOP/s, one barrier per
// step -> now): 8192^3 A B^T 1,134 -> 1,480-1,565, A B 1,068 -> 1,373-1,555
// (within 1% of A B^T where both were timed in one process), A^T B 997 ->
// 1,420; 65,536 x 5632 x 2048 A B^T 1,151 -> 1,410; 2048 x 5632 x 65,536 A^T B
// 863 -> 1,173-1,220.
//
// Every 64 x 64 sub-tile sits in LDS as the matrix stores it, 128-byte rows
// of swizzled 16-byte chunks.  An operand stored with its reduction axis
// along the rows (A^T, B) is read with the transposing LDS read; one stored
// with it along the columns is read row-wise.  Both give a lane the 8
// consecutive k of its row or column.
//
// Each product is issued as D = op(B)^T op(A)^T, so a lane's accumulator holds
// 4 consecutive columns of C: the epilogue writes 8 bytes per lane and
// accumulator to an LDS copy of the tile, and the tile then goes to memory
// in full 16-byte rows.  With split-K (weight gradients, whose reduction axis
// is the 65,536 tokens), every split writes an fp32 partial tile to the
// caller's workspace and a second kernel sums them.
#include "dd_device.hpp"
#include "dd_tile.hpp"
#include "dd_internal.h"
#include "dd_launch.hpp"
#include "dd_routes.hpp"
#include "dd_attn.h"

#include <algorithm>

namespace dd {

struct GemmTile {
    static constexpr int BM = 256, BN = 256, BK = 64, NW = 8;
    static constexpr int SUB = 64 * 64;        // elements of one 64 x 64 sub-tile
    static constexpr int HALF = 2 * SUB;       // half of the A (or B) tile of one K step
    static constexpr int SIDE = 4 * HALF;      // A (or B): two halves x two stages
};

// Waits until at most N of this wave's vector-memory operations are in
// flight and all its LDS reads have returned, then joins the workgroup's
// barrier.
template <int N>
__device__ __forceinline__ void wait_and_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void plain_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" : : : "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Chunk swizzle of the sub-tiles that are read along rows: 64 lanes read 16
// consecutive rows at four neighbouring chunks, and the LDS serves them in
// groups of 16 lanes that are not consecutive (lanes 0-3, 12-15, 20-23,
// 24-27 and so on).  With swz<64>, made for 32 rows at two chunks, such a
// read has two-way bank conflicts.
__device__ __forceinline__ int row_swz(int r) { return (r >> 1) & 7; }

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Row strides (elements) from which a load's per-lane byte offset, up to 7
// rows, may not fit 32 bits; the loads then take per-lane 64-bit addresses.
constexpr long long kGemmWideStride = 1LL << 28;

// What becomes of the tile (EPI):
//   kEpiStore      C = op(A) op(B), plus R (bf16, row stride ldc, may be C
//                  itself) added to the rounded product before the final
//                  rounding if given
//   kEpiPart       an fp32 partial tile of split blockIdx.y to P
//                  ([splits][groups][M][N])
//   kEpiSwiglu     half of the tile's columns are A B[0] and half the same
//                  columns of A B[1]: C[0] and C[1] receive them, C[2]
//                  silu(C[0]) * C[1] of the rounded values
//   kEpiSwigluBwd  the rounded tile is the gradient of silu(U) * V: C[0] and
//                  C[1] receive the gradients of U and V (row stride ldc)
enum GemmEpi { kEpiStore, kEpiPart, kEpiSwiglu, kEpiSwigluBwd };

// One launch computes, with the same strides,
//   groups:   C[g] = op(A[0]) op(B[g]), g < groups, or
//   segments: C[0] = sum over s < segs of op(A[s]) op(B[s])
// (one of the two counts is 1).
struct GemmOperands {
    const uint16_t *A[3], *B[3];
    uint16_t *C[3];
    const uint16_t *R, *U, *V;
    float *P;
};

// Sizes: M x N per group, K per segment; k_len of a split (segs * K without
// splits); tiles_n = tile columns of all groups; xm: tile_of.
struct GemmSizes {
    int M, N, K, k_len, tiles_n, xm;
    long long lda, ldb, ldc;
};

// Tile of block `id`.  Workgroups are dispatched round-robin over the 8 XCDs
// (block id % 8), each with its own L2.  XCD x takes every xm-th tile row
// from row x % xm on and one of 8 / xm blocks of columns, in bands of kGR of
// its rows; a band is walked in groups of 32 tiles (one per CU of the XCD),
// each group column by column, so the tiles that run at the same time share
// their A and B panels in one L2.  xm = 0: row by row (tile_rows_step).
constexpr int kGR = 4;

__device__ __forceinline__ void tile_of(int id, int tiles_m, int tiles_n, int xm, int &tm, int &tn)
{
    if (xm == 0) {
        tm = id / tiles_n;
        tn = id - tm * tiles_n;
        return;
    }
    const int x = id % kXcds, k = id / kXcds;
    const int rows_x = tiles_m / xm, cols_x = tiles_n * xm / kXcds;
    const int band = k / (kGR * cols_x), rem = k - band * kGR * cols_x;
    const int gr = min(kGR, rows_x - band * kGR);  // rows of this band
    const int gc = 32 / gr, grp = rem / (gr * gc), w = rem - grp * gr * gc;
    tm = (band * kGR + w % gr) * xm + x % xm;
    tn = x / xm * cols_x + grp * gc + w / gr;
}

// LDS position (elements) of the four columns c .. c + 3 of row r of the
// finished BM x BN bf16 tile.  With kEpiSwiglu the column halves are two
// tiles of their own.  A row's 4-element group x sits at x ^ (2 (r mod 16))
// (mod 8 where a row has 16 groups), which keeps the two groups of a 16-byte piece adjacent and spreads one
// write instruction's 16 rows over the LDS banks.
template <int BM, int BN, int EPI>
__device__ __forceinline__ int epi_off(int r, int c)
{
    constexpr int W = EPI == kEpiSwiglu ? BN / 2 : BN;
    return c / W * (BM * W) + r * W + 4 * (((c % W) >> 2) ^ (2 * (r & (W == 64 ? 7 : 15))));
}

// Writes the finished tile of rows m0 .., columns n0 .. from LDS to memory.
template <int BM, int BN, int EPI>
__device__ __forceinline__ void epi_store(const uint16_t *lds, const GemmOperands &op, int grp,
                                          int m0, int n0, long long ldc, int tid)
{
    constexpr int W = EPI == kEpiSwiglu ? BN / 2 : BN, CPR = W / 8;
    uint16_t *C = op.C[EPI == kEpiStore ? grp : 0];
#pragma unroll 4
    for (int it = 0; it < BM * CPR / 512; ++it) {
        const int idx = it * 512 + tid, r = idx / CPR, c = idx % CPR * 8;
        const u32x4 v = *reinterpret_cast<const u32x4 *>(lds + epi_off<BM, W, kEpiStore>(r, c));
        const long long at = (m0 + r) * ldc + n0 + c;
        if constexpr (EPI == kEpiSwiglu) {
            const u32x4 w =
                *reinterpret_cast<const u32x4 *>(lds + BM * W + epi_off<BM, W, kEpiStore>(r, c));
            float x[8], y[8], z[8];
            unpack8(v, x);
            unpack8(w, y);
#pragma unroll
            for (int t = 0; t < 8; ++t)
                z[t] = swiglu(x[t], y[t]);
            *reinterpret_cast<u32x4 *>(C + at) = v;
            *reinterpret_cast<u32x4 *>(op.C[1] + at) = w;
            *reinterpret_cast<u32x4 *>(op.C[2] + at) = pack8f(z);
        } else if constexpr (EPI == kEpiSwigluBwd) {
            float d[8], x[8], y[8], dx[8], dy[8];
            unpack8(v, d);
            unpack8(*reinterpret_cast<const u32x4 *>(op.U + at), x);
            unpack8(*reinterpret_cast<const u32x4 *>(op.V + at), y);
#pragma unroll
            for (int t = 0; t < 8; ++t)
                swiglu_grad(x[t], y[t], d[t], dx[t], dy[t]);
            *reinterpret_cast<u32x4 *>(C + at) = pack8f(dx);
            *reinterpret_cast<u32x4 *>(op.C[1] + at) = pack8f(dy);
        } else if (op.R != nullptr) {
            float x[8], y[8];
            unpack8(v, x);
            unpack8(*reinterpret_cast<const u32x4 *>(op.R + at), y);
#pragma unroll
            for (int t = 0; t < 8; ++t)
                x[t] += y[t];
            *reinterpret_cast<u32x4 *>(C + at) = pack8f(x);
        } else {
            *reinterpret_cast<u32x4 *>(C + at) = v;
        }
    }
}

// The pointers of the K steps still to load: moves one step on, or to the
// next segment's start (all scalar).
struct GemmWalk {
    const uint16_t *pa, *pb, *a1, *b1, *a2, *b2;
    int left, seg_steps;

    __device__ __forceinline__ void init(const GemmOperands &p, int grp, long long oa,
                                         long long ob, int steps)
    {
        pa = p.A[0] + oa;
        pb = p.B[grp] + ob;
        a1 = p.A[1] + oa;
        b1 = p.B[1] + ob;
        a2 = p.A[2] + oa;
        b2 = p.B[2] + ob;
        left = seg_steps = steps;
    }
    __device__ __forceinline__ void next(long long ka, long long kb)
    {
        const bool sw = --left == 0;
        pa = sw ? a1 : pa + ka;
        pb = sw ? b1 : pb + kb;
        a1 = sw ? a2 : a1;
        b1 = sw ? b2 : b1;
        left = sw ? seg_steps : left;
    }
};

// TA: A is stored [K][M]; TB: B is stored [N][K]; WIDE: a row stride of A
// or B is at least kGemmWideStride.
template <bool TA, bool TB, int EPI, bool WIDE>
__global__ void __launch_bounds__(512, 1)
gemm_kernel(GemmOperands op, GemmSizes sz)
{
    const long long lda = sz.lda, ldb = sz.ldb, ldc = sz.ldc;
    using T = GemmTile;
    __shared__ __attribute__((aligned(1024))) uint16_t lds[2 * T::SIDE];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l16 = lane & 15, g = lane >> 4;
    const int wm = wave >> 2, wn = wave & 3;
    const int tiles_n = sz.tiles_n;
    int tm, tn;
    tile_of(static_cast<int>(blockIdx.x), sz.M / T::BM, tiles_n, sz.xm, tm, tn);
    // Columns of one matrix B[g] (C[g]) in a tile.
    constexpr int NC = EPI == kEpiSwiglu ? T::BN / 2 : T::BN;
    const int m0 = tm * T::BM, tpg = sz.N / NC, grp = tn / tpg, n0 = (tn - grp * tpg) * NC;
    const int kbeg = static_cast<int>(blockIdx.y) * sz.k_len;
    const int nkt = sz.k_len / T::BK;

    // Loads: sub-tile rows of 128 bytes, eight of them per wave instruction
    // (1 KiB); lane i takes row 8 wave + i / 8, stored chunk i % 8.
    const int qr = lane >> 3, qrow = 8 * wave + qr;
    const int xa = ((lane & 7) ^ (TA ? swz<64>(qrow) : row_swz(qrow))) * 8;
    const int xb = ((lane & 7) ^ (TB ? row_swz(qrow) : swz<64>(qrow))) * 8;
    const long long va = (qr * lda + xa) * 2, vb = (qr * ldb + xb) * 2;  // bytes
    GemmWalk at;
    at.init(op, grp,
            8 * wave * lda + (TA ? static_cast<long long>(kbeg) * lda + m0
                                 : static_cast<long long>(m0) * lda + kbeg),
            8 * wave * ldb + (TB ? static_cast<long long>(n0) * ldb + kbeg
                                 : static_cast<long long>(kbeg) * ldb + n0),
            sz.K / T::BK);
    // Sub-tile s starts 64 rows (stored along the tile's rows) or 64 columns
    // further; K step kt moves 64 rows or columns.
    const long long sa = TA ? 64 : 64 * lda, sb = TB ? 64 * ldb : 64;
    const long long ka = TA ? 64 * lda : 64, kb = TB ? 64 : 64 * ldb;
    const uint32_t lds0 = lds_base_sgpr(lds) + 1024u * wave;
    auto load = [&](const uint16_t *p, long long v, uint32_t l) __attribute__((always_inline)) {
        if constexpr (WIDE)
            dma_b128(reinterpret_cast<const char *>(p) + v, l);
        else
            dma_b128_off(p, static_cast<uint32_t>(v), l);
    };
    // From half 0 to half 1 of B: the next 128 columns, or the other matrix.
    const long long hb = EPI == kEpiSwiglu ? op.B[1] - op.B[0] : 2 * sb;
    // Half h of A (B) of the next K step to load, into stage S.
    auto load_a = [&](int h, int S) __attribute__((always_inline)) {
        const uint16_t *p = at.pa;
        const uint32_t l = lds0 + 2u * (2 * h + S) * T::HALF;
        load(p + 2 * h * sa, va, l);
        load(p + 2 * h * sa + sa, va, l + 2u * T::SUB);
    };
    auto load_b = [&](int h, int S) __attribute__((always_inline)) {
        const uint16_t *p = at.pb + h * hb;
        const uint32_t l = lds0 + 2u * (T::SIDE + (2 * h + S) * T::HALF);
        load(p, vb, l);
        load(p + sb, vb, l + 2u * T::SUB);
    };

    // Fragments.  A half h: rows 64 wm + 16 i .. +15 of the half, i.e.
    // sub-tile wm; B half h: columns 32 wn + 16 j .. +15, i.e. sub-tile
    // wn / 2.  A lane holds the eight k = 32 kk + 8 g .. +7 of its row.
    // Row reads take them in one piece; transposed reads in two pieces of
    // four k, whose lane 4 e + c of a 16-lane group addresses row e, columns
    // 4 c .. 4 c + 3.
    const int e4 = l16 >> 2, c4 = l16 & 3;
    const uint16_t *fa[TA ? 8 : 2], *fb[TB ? 2 : 4];
    {
        const uint16_t *as = lds + wm * T::SUB;
        const uint16_t *bs = lds + T::SIDE + (wn >> 1) * T::SUB;
        if constexpr (TA) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                fa[i] = as + tile_off<64>(8 * g + 4 * (i & 1) + e4, 16 * (i >> 1) + 4 * c4);
        } else {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
                fa[kk] = as + 64 * l16 + (((4 * kk + g) ^ row_swz(l16)) << 3);
        }
        if constexpr (TB) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
                fb[kk] = bs + 64 * (32 * (wn & 1) + l16) + (((4 * kk + g) ^ row_swz(l16)) << 3);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                fb[j] = bs + tile_off<64>(8 * g + 4 * (j & 1) + e4,
                                          32 * (wn & 1) + 16 * (j >> 1) + 4 * c4);
        }
    }
    bf16x8 a0[4][2], a1[4][2], b0[2][2], b1[2][2];
    auto read_a = [&](bf16x8 (&f)[4][2], int h, int S) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const int o = (2 * h + S) * T::HALF;
                if constexpr (TA)
                    f[i][kk] = join(lds_tr4(fa[2 * i] + (o + 2048 * kk)),
                                    lds_tr4(fa[2 * i + 1] + (o + 2048 * kk)));
                else
                    f[i][kk] = lds_row8(fa[kk] + (o + 1024 * i));
            }
    };
    auto read_b = [&](bf16x8 (&f)[2][2], int h, int S) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const int o = (2 * h + S) * T::HALF;
                if constexpr (TB)
                    f[j][kk] = lds_row8(fb[kk] + (o + 1024 * j));
                else
                    f[j][kk] = join(lds_tr4(fb[2 * j] + (o + 2048 * kk)),
                                    lds_tr4(fb[2 * j + 1] + (o + 2048 * kk)));
            }
    };

    f32x4 acc[2][2][4][2];  // [A half][B half][i][j]
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[x >> 1][x & 1][i][j] = f32x4{};
    auto multiply = [&](f32x4 (&c)[4][2], const bf16x8 (&a)[4][2],
                        const bf16x8 (&b)[2][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    c[i][j] = mfma16(b[j][kk], a[i][kk], c[i][j]);  // rows n, columns m
    };
    auto products = [&](f32x4 (&c)[4][2], const bf16x8 (&a)[4][2],
                        const bf16x8 (&b)[2][2]) __attribute__((always_inline)) {
        __builtin_amdgcn_s_setprio(1);
        multiply(c, a, b);
        __builtin_amdgcn_s_setprio(0);
        plain_barrier();
    };

    // One K step from stage S.  MODE 0: also starts the loads of the step
    // after the next one; 1, 2: the last step but one, the last step.
    auto step = [&](auto stage, auto mode) __attribute__((always_inline)) {
        constexpr int S = decltype(stage)::value, MODE = decltype(mode)::value;
        read_b(b0, 0, S);
        if constexpr (MODE == 0)
            load_a(0, S);
        wait_and_barrier<MODE == 0 ? 12 : MODE == 1 ? 10 : 2>();
        products(acc[0][0], a0, b0);
        read_b(b1, 1, S);
        if constexpr (MODE == 0)
            load_b(0, S);
        wait_and_barrier<MODE == 0 ? 12 : MODE == 1 ? 8 : 0>();
        products(acc[0][1], a0, b1);
        read_a(a1, 1, S);
        if constexpr (MODE == 0)
            load_b(1, S);
        wait_and_barrier<MODE == 0 ? 12 : MODE == 1 ? 6 : 0>();
        products(acc[1][1], a1, b1);
        if constexpr (MODE != 2)
            read_a(a0, 0, 1 - S);
        if constexpr (MODE == 0) {
            load_a(1, S);
            at.next(ka, kb);
        }
        wait_and_barrier<MODE == 0 ? 12 : MODE == 1 ? 4 : 0>();
        products(acc[1][0], a1, b0);
    };

    // The loop takes K steps in pairs, stage 0 first; an odd count starts with
    // a step of its own in stage 1.
    auto load_step = [&](int S) __attribute__((always_inline)) {
        load_a(0, S);
        load_b(0, S);
        load_b(1, S);
        load_a(1, S);
        at.next(ka, kb);
    };
    if (nkt == 1) {
        // Nothing to overlap: one wait for the step's tiles, no phases.  5632 x
        // 3072, us, with one barrier per step / in four phases / here: 15.4 /
        // 16.6 / 15.1.  (Two steps, 18.7 / 19.1, lose 2-4% for A B^T only and
        // gained nothing without the phases.)
        load_step(0);
        wait_and_barrier<0>();
        read_a(a0, 0, 0);
        read_b(b0, 0, 0);
        multiply(acc[0][0], a0, b0);
        read_b(b1, 1, 0);
        multiply(acc[0][1], a0, b1);
        read_a(a1, 1, 0);
        multiply(acc[1][1], a1, b1);
        multiply(acc[1][0], a1, b0);
    } else {
        const int s0 = nkt & 1;
        load_step(s0);
        load_step(1 - s0);
        wait_and_barrier<8>();
        read_a(a0, 0, s0);
        // Phase 1 refills the half just read: as in the loop, only after a
        // barrier that every wave reaches with its reads returned (a load of
        // one wave writes rows that all the others read).
        wait_and_barrier<8>();
        // The second group of four waves runs half a phase behind the first:
        // on every SIMD one wave issues products while the other reads and
        // loads.
        if (wm == 1)
            plain_barrier();
        for (int kt = 2 - s0; kt < nkt; kt += 2) {
            if (kt > 1)
                step(IC<0>{}, IC<0>{});
            step(IC<1>{}, IC<0>{});
        }
        step(IC<0>{}, IC<1>{});
        step(IC<1>{}, IC<2>{});
        if (wm == 0)
            plain_barrier();
    }

    // Accumulator (ha, hb, i, j), register e: row m = 128 ha + 64 wm + 16 i +
    // l16, column n = 128 hb + 32 wn + 16 j + 4 g + e of the tile.
    if constexpr (EPI == kEpiPart) {
        const int N = sz.N;
        float *dst = op.P + static_cast<long long>(blockIdx.y * (tiles_n / tpg) + grp) * sz.M * N;
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            const int ha = x >> 3, i = (x >> 1) & 3, hb = x & 1;
            const long long m = m0 + 128 * ha + 64 * wm + 16 * i + l16;
#pragma unroll
            for (int j = 0; j < 2; ++j)
                *reinterpret_cast<f32x4 *>(dst + m * N + n0 + 128 * hb + 32 * wn + 16 * j + 4 * g) =
                    acc[ha][hb][i][j];
        }
    } else {
        // The tile in bf16 through LDS, then to memory in 16-byte pieces of
        // rows.
        __syncthreads();
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            const int ha = x >> 3, i = (x >> 1) & 3, hb = x & 1;
            const int r = 128 * ha + 64 * wm + 16 * i + l16;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const f32x4 v = acc[ha][hb][i][j];
                *reinterpret_cast<bf16x4 *>(lds + epi_off<T::BM, T::BN, EPI>(
                                                      r, 128 * hb + 32 * wn + 16 * j + 4 * g)) =
                    pack4(v[0], v[1], v[2], v[3]);
            }
        }
        __syncthreads();
        epi_store<T::BM, T::BN, EPI>(lds, op, grp, m0, n0, ldc, tid);
    }
}

// ---------------------------------------------------------------------------
// Smaller tiles, for products whose 256 x 256 tiles would leave CUs idle:
// 128 x 128 (SmallTile) and 256 x 128 (TallTile).  Eight waves in two groups
// that run half a phase apart, as in the large kernel; a phase is 16 products
// of every wave: one K step of the small tile (a wave owns 64 x 32), half of
// one (32 k) of the tall tile (64 x 64).  With one workgroup per CU nothing
// else hides a load's latency, so further stages beside the one being read
// are in flight: three of four for the small tile (128 KiB; two or four more
// measured the same or slower), two of three for the tall one (144 KiB).
//
// What bounds the loop: no throughput, but the turn of the two groups.  A step
// of the small tile takes 0.41 us (about 900 clocks), of which its products
// fill 512 and its 96 KiB of LDS reads about as many (220-256 bytes per clock
// measured); of the tall one 0.60 us (1024 clocks of products, 128 KiB).
// Waves wait at barriers and for loads 31-43% of their cycles and to issue
// 29-39%, of that on LDS 6-12%.  Letting each group take half of the k for the
// whole small tile reads 64 KiB a step and measured 6% faster at K = 5632, 5%
// slower at K = 1024 (the sums have to be added at the end).
// 2048 x 1024 x 1024: 21.1 us on 32 large tiles, 11.4-12.6 on small ones.
struct SmallTile {
    static constexpr int BM = 128, BN = 128, BK = 64, NST = 4;
    static constexpr int PH = 1;  // phases per K step
};
struct TallTile {
    static constexpr int BM = 256, BN = 128, BK = 64, NST = 3;
    static constexpr int PH = 2;
};

template <typename T, bool TA, bool TB, int EPI, bool WIDE>
__global__ void __launch_bounds__(512, 1)
gemm_mid_kernel(GemmOperands op, GemmSizes sz)
{
    const long long lda = sz.lda, ldb = sz.ldb, ldc = sz.ldc;
    constexpr int SUB = 64 * 64;
    constexpr int NA = T::BM / 64, NB = T::BN / 64;   // sub-tiles of A, of B
    constexpr int STAGE = (NA + NB) * SUB;
    constexpr int LPS = NA + NB;                      // a wave's loads per step
    constexpr int WN = T::BM == 256 ? 2 : 4;          // waves along N
    constexpr int NJ = T::BN / WN / 16;               // 16-column blocks per wave
    __shared__ __attribute__((aligned(1024))) uint16_t lds[T::NST * STAGE];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l16 = lane & 15, g = lane >> 4;
    const int wm = wave / WN, wn = wave % WN, group = wave >> 2;
    const int tiles_n = sz.tiles_n;
    int tm, tn;
    tile_of(static_cast<int>(blockIdx.x), sz.M / T::BM, tiles_n, sz.xm, tm, tn);
    // Columns of one matrix B[g] (C[g]) in a tile.
    constexpr int NC = EPI == kEpiSwiglu ? T::BN / 2 : T::BN;
    const int m0 = tm * T::BM, tpg = sz.N / NC, grp = tn / tpg, n0 = (tn - grp * tpg) * NC;
    const int kbeg = static_cast<int>(blockIdx.y) * sz.k_len;
    const int nkt = sz.k_len / T::BK;

    const int qr = lane >> 3, qrow = 8 * wave + qr;
    const int xa = ((lane & 7) ^ (TA ? swz<64>(qrow) : row_swz(qrow))) * 8;
    const int xb = ((lane & 7) ^ (TB ? row_swz(qrow) : swz<64>(qrow))) * 8;
    const long long va = (qr * lda + xa) * 2, vb = (qr * ldb + xb) * 2;  // bytes
    GemmWalk at;
    at.init(op, grp,
            8 * wave * lda + (TA ? static_cast<long long>(kbeg) * lda + m0
                                 : static_cast<long long>(m0) * lda + kbeg),
            8 * wave * ldb + (TB ? static_cast<long long>(n0) * ldb + kbeg
                                 : static_cast<long long>(kbeg) * ldb + n0),
            sz.K / T::BK);
    const long long sa = TA ? 64 : 64 * lda, sb = TB ? 64 * ldb : 64;
    const long long ka = TA ? 64 * lda : 64, kb = TB ? 64 : 64 * ldb;
    const uint32_t lds0 = lds_base_sgpr(lds) + 1024u * wave;
    // From sub-tile 0 to sub-tile 1 of B: the next 64 columns, or the other matrix.
    const long long hb = EPI == kEpiSwiglu ? op.B[1] - op.B[0] : sb;
    // Load i of the next K step to load, into stage st: the A sub-tiles, then
    // the B sub-tiles.
    auto load = [&](int i, int st) __attribute__((always_inline)) {
        const uint32_t l = lds0 + 2u * (STAGE * st + i * SUB);
        const uint16_t *p = i < NA ? at.pa + i * sa : at.pb + (i - NA) * hb;
        const long long v = i < NA ? va : vb;
        if constexpr (WIDE)
            dma_b128(reinterpret_cast<const char *>(p) + v, l);
        else
            dma_b128_off(p, static_cast<uint32_t>(v), l);
    };

    const int e4 = l16 >> 2, c4 = l16 & 3;
    int fa[TA ? 8 : 2], fb[TB ? 2 : 2 * NJ];  // element offsets in a stage
    {
        // The wave's first column inside its B sub-tile.
        const int as = wm * SUB, bs = (NA + wn * 16 * NJ / 64) * SUB, bc = wn * 16 * NJ % 64;
        if constexpr (TA) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                fa[i] = as + tile_off<64>(8 * g + 4 * (i & 1) + e4, 16 * (i >> 1) + 4 * c4);
        } else {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
                fa[kk] = as + 64 * l16 + (((4 * kk + g) ^ row_swz(l16)) << 3);
        }
        if constexpr (TB) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
                fb[kk] = bs + 64 * (bc + l16) + (((4 * kk + g) ^ row_swz(l16)) << 3);
        } else {
#pragma unroll
            for (int j = 0; j < 2 * NJ; ++j)
                fb[j] = bs + tile_off<64>(8 * g + 4 * (j & 1) + e4, bc + 16 * (j >> 1) + 4 * c4);
        }
    }
    f32x4 acc[4][NJ];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            acc[i][j] = f32x4{};

    const int first = min(nkt, T::NST - 1);
    for (int kt = 0; kt < first; ++kt) {
#pragma unroll
        for (int i = 0; i < LPS; ++i)
            load(i, kt);
        at.next(ka, kb);
    }
    if (nkt > T::NST - 2)
        wait_and_barrier<LPS *(T::NST - 2)>();
    else
        wait_and_barrier<0>();
    if (group == 1)
        plain_barrier();
    int rs = 0, ws = T::NST - 1;  // the stages read and refilled by a step
    for (int kt = 0; kt < nkt; ++kt) {
        const uint16_t *st = lds + rs * STAGE;
        constexpr int KK = 2 / T::PH;  // 32-wide parts of the step in a phase
#pragma unroll
        for (int ph = 0; ph < T::PH; ++ph) {
            bf16x8 a[4][KK], b[NJ][KK];
#pragma unroll
            for (int x = 0; x < KK; ++x) {
                const int kk = ph * KK + x;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    if constexpr (TB)
                        b[j][x] = lds_row8(st + fb[kk] + 1024 * j);
                    else
                        b[j][x] = join(lds_tr4(st + fb[2 * j] + 2048 * kk),
                                       lds_tr4(st + fb[2 * j + 1] + 2048 * kk));
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (TA)
                        a[i][x] = join(lds_tr4(st + fa[2 * i] + 2048 * kk),
                                       lds_tr4(st + fa[2 * i + 1] + 2048 * kk));
                    else
                        a[i][x] = lds_row8(st + fa[kk] + 1024 * i);
                }
            }
            // The stage that the step before has read is refilled; before the
            // next step starts, its own loads have to be there (the steps
            // after it may be in flight).
            const int ahead = nkt - 1 - kt;  // steps after this one
            if (ahead >= T::NST - 1) {
#pragma unroll
                for (int i = ph * LPS / T::PH; i < (ph + 1) * LPS / T::PH; ++i)
                    load(i, ws);
            }
            if (ph + 1 < T::PH) {
                wait_and_barrier<63>();
            } else {
                if (ahead >= T::NST - 1) {
                    at.next(ka, kb);
                    wait_and_barrier<LPS *(T::NST - 2)>();
                } else if (T::NST == 4 && ahead == 2) {
                    wait_and_barrier<LPS>();
                } else {
                    wait_and_barrier<0>();
                }
                ws = rs;
                rs = rs + 1 == T::NST ? 0 : rs + 1;
            }
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int x = 0; x < KK; ++x)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        acc[i][j] = mfma16(b[j][x], a[i][x], acc[i][j]);  // rows n, columns m
            __builtin_amdgcn_s_setprio(0);
            plain_barrier();
        }
    }
    if (group == 0)
        plain_barrier();

    // Accumulator (i, j), register e: row m = 64 wm + 16 i + l16, column
    // n = 16 NJ wn + 16 j + 4 g + e of the tile; stored as in the large kernel.
    if constexpr (EPI == kEpiPart) {
        const int N = sz.N;
        float *dst = op.P + static_cast<long long>(blockIdx.y * (tiles_n / tpg) + grp) * sz.M * N;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                *reinterpret_cast<f32x4 *>(dst + static_cast<long long>(m0 + 64 * wm + 16 * i + l16) * N +
                                           n0 + 16 * NJ * wn + 16 * j + 4 * g) = acc[i][j];
    } else {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 64 * wm + 16 * i + l16;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const f32x4 v = acc[i][j];
                *reinterpret_cast<bf16x4 *>(
                    lds + epi_off<T::BM, T::BN, EPI>(r, 16 * NJ * wn + 16 * j + 4 * g)) =
                    pack4(v[0], v[1], v[2], v[3]);
            }
        }
        __syncthreads();
        epi_store<T::BM, T::BN, EPI>(lds, op, grp, m0, n0, ldc, tid);
    }
}

// C[g] = sum over splits of P (fp32 [splits][groups][M][N]) rounded to bf16;
// 8 elements per thread, grid-stride.
__global__ void __launch_bounds__(256)
gemm_reduce_kernel(GemmOperands op, int groups, long long MN, int splits, long long ldc, int N)
{
    const float *__restrict__ P = op.P;
    const uint16_t *R = op.R;
    const long long all = groups * MN;
    const long long stride = static_cast<long long>(gridDim.x) * 256;
    for (long long v = static_cast<long long>(blockIdx.x) * 256 + threadIdx.x; v < all / 8;
         v += stride) {
        const long long e0 = v * 8;
        f32x4 s0 = *reinterpret_cast<const f32x4 *>(P + e0);
        f32x4 s1 = *reinterpret_cast<const f32x4 *>(P + e0 + 4);
        for (int s = 1; s < splits; ++s) {
            s0 += *reinterpret_cast<const f32x4 *>(P + s * all + e0);
            s1 += *reinterpret_cast<const f32x4 *>(P + s * all + e0 + 4);
        }
        const int grp = static_cast<int>(e0 / MN);
        const long long m = (e0 - grp * MN) / N, n = e0 % N;
        if (R != nullptr) {
            const bf16x8 r = as_bf16x8(*reinterpret_cast<const u32x4 *>(R + m * ldc + n));
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                s0[t] = static_cast<float>(static_cast<__bf16>(s0[t])) + static_cast<float>(r[t]);
                s1[t] = static_cast<float>(static_cast<__bf16>(s1[t])) + static_cast<float>(r[t + 4]);
            }
        }
        *reinterpret_cast<bf16x8 *>(op.C[grp] + m * ldc + n) =
            join(pack4(s0[0], s0[1], s0[2], s0[3]), pack4(s1[0], s1[1], s1[2], s1[3]));
    }
}

#define DD_GEMM_INST(TA, TB, EPI)                                                                \
    template __global__ void gemm_kernel<TA, TB, EPI, false>(GemmOperands, GemmSizes);           \
    template __global__ void gemm_kernel<TA, TB, EPI, true>(GemmOperands, GemmSizes);            \
    template __global__ void gemm_mid_kernel<TallTile, TA, TB, EPI, false>(GemmOperands,         \
                                                                           GemmSizes);           \
    template __global__ void gemm_mid_kernel<TallTile, TA, TB, EPI, true>(GemmOperands,          \
                                                                          GemmSizes);            \
    template __global__ void gemm_mid_kernel<SmallTile, TA, TB, EPI, false>(GemmOperands,        \
                                                                            GemmSizes);          \
    template __global__ void gemm_mid_kernel<SmallTile, TA, TB, EPI, true>(GemmOperands,         \
                                                                           GemmSizes)
DD_GEMM_INST(false, false, kEpiStore);
DD_GEMM_INST(false, false, kEpiPart);
DD_GEMM_INST(false, true, kEpiStore);
DD_GEMM_INST(false, true, kEpiPart);
DD_GEMM_INST(true, false, kEpiStore);
DD_GEMM_INST(true, false, kEpiPart);
DD_GEMM_INST(false, false, kEpiSwiglu);
DD_GEMM_INST(false, true, kEpiSwigluBwd);
#undef DD_GEMM_INST

static GemmPlan plan_on_device(int M, long long N, long long K, bool may_split)
{
    return gemm_plan(M, N, K, may_split, device_cu_count());
}

// xm of tile_of: the one whose groups of 32 tiles read the fewest panels per
// tile, of those that divide the tiles evenly (0: none does).  Eight tile rows
// of a weight gradient, taken a row per XCD, read 24 B panels for 24 tiles
// (2048 x 6144, K = 16,384: 430 us); as 4 x 6 tiles per XCD 400 us.
static int tile_rows_step(int tiles_m, int tiles_n)
{
    int best = 0;
    double least = 0;
    for (int xm = kXcds; xm >= 1; xm /= 2) {
        if (tiles_m % xm || tiles_n * xm % kXcds)
            continue;
        const double gr = std::min(kGR, tiles_m / xm);
        const double gc = std::min(32 / gr, static_cast<double>(tiles_n * xm / kXcds));
        const double panels = (gr + gc) / (gr * gc);
        if (best == 0 || panels < least) {
            best = xm;
            least = panels;
        }
    }
    return best;
}

size_t gemm_workspace_bytes(int M, int N, int K, int groups)
{
    const GemmPlan p = plan_on_device(M, static_cast<long long>(groups) * N, K, true);
    return p.splits > 1 ? static_cast<size_t>(p.splits) * groups * M * N * sizeof(float) : 0;
}

int launch_gemm(const GemmArgs &a)
{
    hipStream_t st = static_cast<hipStream_t>(a.stream);
    // Columns of all groups (of both matrices for kEpiSwiglu).
    const bool swiglu = a.kind == GemmArgs::kSwiglu;
    const long long cols = static_cast<long long>(swiglu ? 2 : a.groups) * a.N;
    const GemmPlan plan =
        plan_on_device(a.M, cols, static_cast<long long>(a.segs) * a.K, a.may_split);
    const int splits = plan.splits;
    const int bm = plan.tile == GemmPlan::kSmall ? SmallTile::BM : GemmTile::BM;
    const int bn = plan.tile == GemmPlan::kLarge ? GemmTile::BN : SmallTile::BN;
    GemmOperands op{};
    for (int i = 0; i < 3; ++i) {
        op.A[i] = static_cast<const uint16_t *>(a.A[i]);
        op.B[i] = static_cast<const uint16_t *>(a.B[i]);
        op.C[i] = static_cast<uint16_t *>(a.C[i]);
    }
    op.R = static_cast<const uint16_t *>(a.R);
    op.U = static_cast<const uint16_t *>(a.U);
    op.V = static_cast<const uint16_t *>(a.V);
    op.P = static_cast<float *>(a.workspace);
    const int tiles_n = static_cast<int>(cols / bn);
    const GemmSizes sz{a.M, a.N, a.K, a.K / splits * a.segs, tiles_n,
                       tile_rows_step(a.M / bm, tiles_n), a.lda, a.ldb, a.ldc};
    const dim3 grid(static_cast<unsigned>(a.M / bm) * tiles_n, static_cast<unsigned>(splits));
    const bool wide = a.lda >= kGemmWideStride || a.ldb >= kGemmWideStride;
    auto pick = [&](auto ta, auto tb, auto epi) {
        constexpr bool TA = decltype(ta)::value, TB = decltype(tb)::value;
        constexpr int E = decltype(epi)::value;
        if (plan.tile == GemmPlan::kSmall)
            return wide ? gemm_mid_kernel<SmallTile, TA, TB, E, true>
                        : gemm_mid_kernel<SmallTile, TA, TB, E, false>;
        if (plan.tile == GemmPlan::kTall)
            return wide ? gemm_mid_kernel<TallTile, TA, TB, E, true>
                        : gemm_mid_kernel<TallTile, TA, TB, E, false>;
        return wide ? gemm_kernel<TA, TB, E, true> : gemm_kernel<TA, TB, E, false>;
    };
    auto form = [&](auto epi) {
        return a.trans_a   ? pick(IC<1>{}, IC<0>{}, epi)
               : a.trans_b ? pick(IC<0>{}, IC<1>{}, epi)
                           : pick(IC<0>{}, IC<0>{}, epi);
    };
    const auto kern = swiglu                                ? pick(IC<0>{}, IC<0>{}, IC<kEpiSwiglu>{})
                      : a.kind == GemmArgs::kSwigluBackward ? pick(IC<0>{}, IC<1>{}, IC<kEpiSwigluBwd>{})
                      : splits > 1                          ? form(IC<kEpiPart>{})
                                                            : form(IC<kEpiStore>{});
    hipError_t e = launch_kernel(kern, grid, dim3(512), st, op, sz);
    if (e != hipSuccess || splits == 1)
        return e == hipSuccess ? DD_OK : DD_ERR_HIP;
    const long long MN = static_cast<long long>(a.M) * a.N;
    const unsigned blocks =
        static_cast<unsigned>(std::min<long long>((a.groups * MN / 8 + 255) / 256, 8192));
    e = launch_kernel(gemm_reduce_kernel, dim3(blocks), dim3(256), st, op, a.groups, MN, splits,
                      a.ldc, a.N);
    return e == hipSuccess ? DD_OK : DD_ERR_HIP;
}

}  // namespace dd
