// na_launch.h -- host-side launchers of the HIP kernels (internal to libna.so).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "na_common.h"

namespace na {

// Forward: q, k, v, o in dtype (0 fp32, 1 fp16, 2 bf16); lse fp32.
hipError_t launch_forward(const Geo& g, int rank, int D, int dtype, int qm, const void* q,
                          const void* k, const void* v, void* o, float* lse, float scale,
                          hipStream_t s);

// Backward: one launch of dK/dV-role and dQ-role workgroups (Delta in-kernel).
hipError_t launch_backward(const Geo& g, int rank, int D, int dtype, int m, const void* q,
                           const void* k, const void* v, const void* o, const float* lse,
                           const void* dout, void* dq, void* dk, void* dv, float scale,
                           hipStream_t s);

// Largest number of 16-key blocks in any workgroup's halo (interior tiles).
inline int max_halo_blocks(const Geo& g, int rank) {
    int nb = 1;
    for (int a = 0; a < rank; ++a) {
        const int n0 = group_len(g.L[a], g.d[a], 0);
        int e = std::min(g.T[a], n0) + g.k[a] - 1;
        e = std::min(e, n0);
        nb *= (a == rank - 1) ? (e + 15) / 16 : e;
    }
    return nb;
}

// LDS of the mask tables (MaskRows): one per outer wave position of the workgroup,
// a row of 32 bytes per 16-token block of the box, rounded to whole stages (of at
// most 16 blocks).  Larger tables are not used.
constexpr size_t kMaskTableBytes = 16384;
inline int mask_table_rows(int blocks) { return (blocks + 15) & ~15; }
inline size_t mask_table_bytes(const Geo& g, int rank) {
    int waves = 1;
    for (int a = 0; a < rank - 1; ++a) waves *= g.WGd[a];
    return (size_t)waves * g.tab_rows * 32;
}

// The narrow form of a two-block tiling (32 queries per wave, four waves): the
// same workgroup tile and halo, its halo rows held in one 16-key block each, but
// waves cut along the innermost axis so that a wave needs eight columns of every
// row; a tile is then four rows of eight keys.  Small inner windows leave most of
// a 16-key block unused otherwise: with k = 7 a 2 x 2 x 8 wave tile visits
// 8 x 8 x 16 = 1024 keys per query and a 4 x 4 x 2 one 10 x 10 x 8 = 800.
// Re-cuts g and returns true where that visits at least a tenth fewer tiles.  Forward,
// 8 heads, ordinary / narrow, us (D = 32, 64, 128): 16 x 64 x 64, 7^3 d = 1, 2, 2 fp16
// 141 / 105, 172 / 142, 361 / 282, bf16 143 / 93, 182 / 134, 361 / 275; 16 x 64 x 64,
// 9 x 9 x 5 bf16 205 / 117, 266 / 191, 533 / 368; 4 x 75 x 117, 11 x 5 d = 1, 3 bf16
// 34 / 23, 46 / 37, 94 / 78.
inline bool narrow_form(Geo& g, int rank, int nb_max) {
    const int in = rank - 1;
    if (g.T[in] + g.k[in] - 1 > 16) return false;  // one block per halo row
    auto rows = [&](const int* wt) {
        int r = 1;
        for (int a = 0; a < in; ++a)
            r *= std::min(wt[a] + g.k[a] - 1, group_len(g.L[a], g.d[a], 0));
        return r;
    };
    const int tiles = (rows(g.WT) + 1) / 2;  // pairs of 16-key rows
    int best = 0, bt[kMaxRank] = {1, 1, 1};
    for (int w = 2; w <= 4 && w + g.k[in] - 1 <= 8; w *= 2) {
        const int nin = g.T[in] / w;  // waves along the innermost axis
        if (nin != 2 && nin != 4) continue;
        for (int s = 0; s < in; ++s) {  // the other split, if any, along outer axis s
            int t[kMaxRank] = {g.T[0], g.T[1], g.T[2]};
            t[in] = w;
            t[s] /= 4 / nin;
            int slots = 0;
            for (int a = 0; a < in; ++a) slots += 2 * (t[a] - 1);
            if (t[s] < 1 || slots > 15) continue;
            const int nt = (rows(t) + 3) / 4;
            if (!best || nt < best) {
                best = nt;
                for (int a = 0; a < kMaxRank; ++a) bt[a] = t[a];
            }
        }
    }
    Geo n = g;
    n.tab_rows = mask_table_rows(nb_max);
    for (int a = 0; a < kMaxRank; ++a) n.WGd[a] = g.T[a] / bt[a];
    if (!best || best * 10 > tiles * 9 || mask_table_bytes(n, rank) > kMaskTableBytes) return false;
    g.tab_rows = n.tab_rows;
    auto lg = [](int x) { return 31 - __builtin_clz((unsigned)x); };
    for (int a = 0; a < kMaxRank; ++a) {
        g.WT[a] = bt[a];
        g.WGd[a] = g.T[a] / bt[a];
        g.lgWT[a] = lg(g.WT[a]);
        g.lgWGd[a] = lg(g.WGd[a]);
    }
    return true;
}

// Geometry of the unfused operators (filled on the host).  A rank-r problem
// occupies the last r axes; the leading ones are inert (extent, window and
// dilation 1, token stride 0).
struct UGeo {
    int L[kMaxRank], k[kMaxRank], d[kMaxRank], causal[kMaxRank];
    int ts[kMaxRank];   // token stride of each axis (0 for inert axes)
    int kst[kMaxRank];  // stride of each axis's window offset in a weight row
    int N;              // tokens per (batch, head)
    int ell;            // weights per row: prod k
    int64_t rows;       // batch * heads * N
    FastDiv fd_L[kMaxRank], fd_d[kMaxRank], fd_k[kMaxRank];
};

// The unfused operators (na_unfused.hip): x, y, z are the op's operands.
enum {
    kUnfusedPN = 0,        // z[i, e] = scale * x_i . y_j(i,e)            (weights z)
    kUnfusedSoftmax = 1,   // z = softmax of each row of z in place; lse  (weights z)
    kUnfusedNN = 2,        // z_i = scale * sum_e x[i, e] y_j(i,e)        (weights x)
    kUnfusedIN = 3,        // z_j = scale * sum_i x[i, e(i,j)] y_i         (weights x)
    kUnfusedSoftmaxBwd = 4 // z = x * (z - rowsum(x * z)) in place          (probs x)
};
hipError_t launch_unfused(const UGeo& u, int D, int dtype, int op, const void* x, const void* y,
                          void* z, float* lse, float scale, hipStream_t s);

// Per-axis window starts and inverse ranges (absolute coordinates), int32.
hipError_t launch_debug_windows(int rank, const int* L, const int* k, const int* d, const int* c,
                                int* start, int* inv_lo, int* inv_hi, hipStream_t s);

}  // namespace na
