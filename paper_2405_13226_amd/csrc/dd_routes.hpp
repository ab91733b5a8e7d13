// dd_routes.hpp -- which kernel form a call takes: an attention call by the
// number of its 128-row blocks, the row length L, the mask and the number of
// CUs, a product by its sizes.  Plain C++, so that a host program can ask where
// a shape goes.
//
// Attention: groups of waves share a block's tiles.  The workgroups of a small
// grid are all resident at once, so the heaviest block's chain of tiles is the
// launch's time, and the groups shorten it.  A larger grid is balanced by dispatch (or
// by the persistent forms' walk), and the groups cost it their final sum and
// their share of a CU.  That balance is what the causal mask makes uneven and
// documents more so: without the causal mask every block has the same work, a
// grid that covers the CUs gains nothing, and the groups stop at one block per
// CU or two.
//
// The figures of the attention rules are graph-replayed times with two (or four) groups over
// those with one, per row length and blocks, causal / not causal / causal with
// documents (log-normal lengths, median 600); a rule takes the groups where
// they gain.
#pragma once

#include <algorithm>
#include <cmath>

namespace dd {

// Blocks up to which the groups pay under the causal mask: two per CU, with
// documents two and a half.  D = 128 forward: 512 blocks of 4096 0.78, 640 of
// 4096 1.10, with documents 0.77.
inline bool causal_small_grid(long long blocks, bool docs, long long cus)
{
    return 2 * blocks <= (docs ? 5 : 4) * cus;
}

// Forward: groups over a query block's key tiles.
// D = 64, up to a block per CU: L = 64 (one tile) 1.14 / 1.14 / 1.12, 128 0.97 /
// 1.06 / 0.98, 160 1.02 / 1.03 / 1.02, 256 0.92 / 0.98 / 0.92, 512 0.84 / 0.89 /
// 0.84; four groups from 769 on (L = 2048 0.70 / 0.73 / 0.69).  Up to two: L =
// 256 1.06 / 1.10 / 1.04, 300 1.00 / 1.03 / 1.03, 512 0.96 / 1.03 / 0.97, 700
// 0.87 / 0.93 / 0.86.  Beyond: L = 1536 1.09 / 1.00 / 1.05 (768), 2048 0.84 /
// 0.98 / 0.99 (768) and 1.00 / 1.01 / 1.03 (1280), 4096 0.76 / 0.95 / 0.76 (768)
// and 0.91 / 0.99 / 0.80 (1280), 8192 1.00 / 1.03 / 0.71 (1280).
// D = 128, up to a block per CU: L = 64 1.21 / 1.24 / 1.21, 160 1.07 / 1.12 /
// 1.05, 256 1.00 / 1.07 / 0.96, 300 0.92 / 0.93 / 0.93, 2048 0.82 / 0.84 /
// 0.76.  Beyond: L = 4096 0.79 / 1.14 / 0.70 (320), 0.78 / 1.08 / 0.74 (512);
// L = 2048 1.23 times faster at 320, equal from 480 on: not taken.
inline int fwd_key_groups(int D, long long blocks, int L, bool causal, bool docs, long long cus)
{
    if (D == 64) {
        if (L <= 192)
            return 1;
        if (blocks <= cus)
            return L > 768 ? 4 : 2;
        if (blocks <= 2 * cus)
            return L > (causal ? 384 : 512) ? 2 : 1;
        return L >= 2048 && blocks <= (!causal ? 3 : L > 2048 ? 5 : 4) * cus ? 2 : 1;
    }
    if (blocks <= cus)
        return L > 256 ? 2 : 1;
    return causal && L > 2048 && causal_small_grid(blocks, docs, cus) ? 2 : 1;
}

// dQ: groups over a query block's key tiles, where it runs by itself (the
// ratios are of the whole backward).
// D = 64, up to a block per CU 0.93 / 0.97 / 0.92 (L = 300); with RoPE, which
// has no one-kernel backward, dQ and dK/dV together L = 64 1.20, 128 and 160
// 1.05, 200 0.95.  Up to two: L = 300
// 1.02 / 1.05 / 1.03, 512 1.02 / 1.02 / 1.01, 700 0.94 / 0.98 / 0.96, 1024 0.97 /
// 0.98 / 0.97; four groups over two (512 blocks): L = 8192 0.89 for 0.93 / 0.98
// for 0.95 / 0.83 for 0.85.  Beyond: L = 4096 0.88 / 1.00 / 0.90 (1024), 0.98 /
// 1.01 / 0.90 (1280); L = 3000 1.09 / 1.02 / 1.04 (2040).
// D = 128: L = 4096 0.93 / 1.04 / 0.94 (384), 0.89 / 1.01 / 0.88 (512), 1.01 /
// 0.99 / 0.90 (640), 1.03 / 1.01 / 0.98 (768); L = 1024 0.96 / 1.01 / 0.93 (256).
inline int dq_key_groups(int D, long long blocks, int L, bool causal, bool docs, long long cus)
{
    if (D == 64) {
        if (L <= 512)
            return L > 192 && blocks <= cus ? 2 : 1;
        if (blocks <= 2 * cus)
            return L > 2048 && causal ? 4 : 2;
        return L > 2048 && blocks <= 6 * cus ? 2 : 1;
    }
    return (L > 768 && blocks <= cus) || (L > 2048 && causal && causal_small_grid(blocks, docs, cus))
               ? 2
               : 1;
}

// dK/dV at D = 64: groups over a key block's query tiles.  Up to a block per
// CU 0.92 / 0.94 / 0.86 (L = 2048), not for the shortest rows (see dQ).  L =
// 4096: 0.85 / 1.07 / 0.86 (512), 1.00 / 0.99 / 0.84 (640), 1.04 / 1.00 / 0.93
// (768); L = 3000 1.05 / 0.99 / 0.87 (648).  (At D = 128 the paired waves fill
// a CU's registers with one group.)
inline int dkdv_query_groups(long long blocks, int L, bool causal, bool docs, long long cus)
{
    return (L > 192 && blocks <= cus) ||
                   (L > 2048 && causal && causal_small_grid(blocks, docs, cus))
               ? 2
               : 1;
}

// Whether dK/dV and dQ run as one launch (blocks of each).  Its workgroups
// fill a CU, so it pays while both kernels' blocks fit the chip once; longer
// rows, whose heaviest blocks take longer than the average ones, gain further.
// One launch over the other route.  128 blocks: D = 64 L = 160 0.90 / 0.86 /
// 0.90, 256 0.68 / 0.50 / 0.66; D = 128 L = 64 0.94 / 0.98 / 0.91, 512 0.66 /
// 0.71 / 0.65.  144: D = 64 L = 256 1.08 / 0.80 / 1.07, 300 0.84 / 1.01 / 0.84,
// 512 0.75 / 1.07 / 0.77; D = 128 L = 256 1.12 / 1.16 / 1.07, 300 0.81 / 1.13 /
// 0.82, 512 0.68 / 1.10 / 0.70.  160: D = 64 L = 512 1.05 / 1.05 / 0.90, 600
// 0.65 / 0.77 / 0.81; D = 128 L = 512 1.03 / 1.08 / 0.86, 600 0.74 / 0.89 / 0.91.
// 320, L = 4096: D = 64 0.65 / 0.87 / 0.46, D = 128 0.83 / 0.83 / 0.54; 228, L =
// 1536, D = 128: 0.71 / 1.04 / 0.63.  At D = 64 the one-kernel backward keeps
// rows of at most 128 tokens.
inline bool bwd_together(int D, long long blocks, int L, bool causal, bool rope, long long cus)
{
    if (D == 64 && !rope && L <= 128)
        return false;
    return 2 * blocks <= cus || (causal && L > 256 && 16 * blocks <= 9 * cus) ||
           (L > 512 && 8 * blocks <= 5 * cus) ||
           (L > (causal ? 1024 : 2048) && 4 * blocks <= 5 * cus);
}

// How a product of these sizes runs: on tiles of 256 x 256, 256 x 128 or
// 128 x 128 (the value is log2 of the tiles per 256 x 256), with the K axis in
// `splits` parts (1: none; more need the workspace).
struct GemmPlan {
    enum Tile { kLarge, kTall, kSmall } tile;
    int splits;
};

// Estimated time (us) of `tiles` tiles with `splits` K parts: rounds of
// workgroups over the CUs (one per CU), each a start-up and tail plus its K
// steps, then the partial sums' write and read.  The constants are fits to
// graph-replayed products.  One round of large, tall and small tiles: 2048 x
// 1024 at K = 1024 takes 21 / 15-17 / 12.5-13 us, at K = 5632 88 / 58 / 42-47
// (with two splits 59 / 44 / 40); 2048 x 2816 at K = 1024 (88, 176 and 352
// workgroups) 23 / 17 / 23.  A full chip runs slower, large tiles for their
// power: 8192 x 2048 at K = 2048 (256, 512, 1024 workgroups) 54 / 69 / 86.
inline double gemm_cost(double tiles, double cus, double steps, double splits, double mn,
                        int tile)
{
    const double wgs = tiles * splits, rounds = std::ceil(wgs / cus);
    const double part = std::min(wgs / cus, 1.0);  // CUs in use
    const double step = tile == GemmPlan::kSmall  ? (part < 1 ? 0.42 : 0.55)
                        : tile == GemmPlan::kTall ? (part < 1 ? 0.60 + 0.15 * part : 0.95)
                                                  : (part < 1 ? 1.02 + 0.2 * part : 1.4);
    const double reduce = splits > 1 ? 6.0 + splits * mn * 8.0 / 4.0e6 : 0.0;
    return rounds * (std::ceil(steps / splits) * step + 6.0) + reduce;
}

// The cheapest tile and number of K splits (1, 2, 4, ...) for a product of
// M x N (all groups' columns together) over K.  Splits are multiples of 64
// and at least 1024 long, and more of them than two large tiles per CU are
// never needed.
inline GemmPlan gemm_plan(int M, long long N, long long K, bool may_split, int cus)
{
    cus = std::max(cus, 1);
    const long long tiles = static_cast<long long>(M / 256) * (N / 256);
    GemmPlan best{GemmPlan::kLarge, 1};
    double cost = -1;
    for (int s = 1;; s *= 2) {
        for (const GemmPlan::Tile tile : {GemmPlan::kLarge, GemmPlan::kTall, GemmPlan::kSmall}) {
            const double c = gemm_cost(static_cast<double>(tiles << tile), cus, K / 64.0, s,
                                       static_cast<double>(M) * N, tile);
            if (cost < 0 || c < cost) {
                cost = c;
                best = GemmPlan{tile, s};
            }
        }
        if (!may_split || tiles * s >= 2LL * cus || K / (2 * s) < 1024 ||
            (K / (2 * s)) % 64 != 0)
            return best;
    }
}

}  // namespace dd
