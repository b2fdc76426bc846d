// na_fwd.hip -- fused neighborhood-attention forward for gfx950.
//
// Fused NA (Sec. 3.3, Fig. "fna-vis"): queries are tiled in their own 1-D /
// 2-D / 3-D layout; the key/value tile is the halo that covers every
// neighbourhood of the query tile; scores go through the NA mask and an online
// softmax (Sec. 2) and straight into the product with V.  Only the output and
// the per-query logsumexp are written.  Dilation is handled as extra
// workgroups over the sub-lattices x = g (mod d) (Sec. 3.4).
//
// MI355X mapping:
//   * workgroup = W waves (4; 8 for large 1-D problems) = one query tile of
//     one (batch, head, dilation group); each wave owns QM x 16 queries of it
//     (a sub-box);
//   * the workgroup's key halo is cut into blocks of 16 keys that run along
//     the innermost axis; stages of SB blocks go straight from HBM to LDS
//     (16-byte direct-to-LDS loads, double buffered when there is more than
//     one stage), K and V both as swizzled unpadded rows; V^T fragments are
//     gathered with the transposed LDS read, so no transposed copy exists;
//   * a wave only runs the matrix cores on blocks that intersect its own
//     sub-box halo, and evaluates the mask only on blocks that are not inside
//     every one of its windows;
//   * S^T = K Q^T (16 keys x 16 queries per MFMA) leaves each query's scores
//     in one lane column; the row maximum needs two lane-swap steps, and P^T
//     feeds O^T = V^T P^T directly as the B operand;
//   * scores are scaled once into base 2 (so the row maximum maps to exactly
//     exp2(0) = 1 and a window of one key returns V bit for bit); the running
//     maximum is only raised (and O rescaled) when a row's maximum grows by
//     more than kLazy, which keeps every P <= 2^kLazy.  Each lane tests its
//     own share of a row against the threshold; the cross-lane row maximum is
//     formed only in the (rare) raising branch;
//   * with one query block per wave, 16-bit types sum each row of the rounded
//     P on the matrix cores: one more MFMA with an all-ones V^T block leaves
//     the full row sum in every lane (with two blocks the extra accumulators
//     would cost a wave of occupancy, so those sum with v_dot2).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "na_launch.h"
#include "na_stage.h"

namespace na {

constexpr float kLazy = 8.f;  // base-2 headroom before the running max is raised

template <int R, int D, typename T, int SB, int W = 4>
struct FwdCfg {
    static constexpr int kWaves = W;
    static constexpr int kThreads = W * kWave;
    static constexpr int kKeys = SB * 16;  // keys per stage
    static constexpr int kTileBytes = kKeys * Rows<T, D>::kRowBytes;
    static constexpr size_t kBufBytes = 2 * kTileBytes;  // K rows, then V rows
    using Ld = DirectRows<T, D, kKeys, W, (R > 1)>;
    static_assert(SB % 2 == 0 && SB <= 32, "stage blocks are tested by one lane each");
};

// Waves per SIMD the register allocation must allow: four for the 16-bit
// kernels that fit 128 VGPRs (every one at D <= 64, and the one-block ones at
// D = 128); the others take what they need.
template <int D, typename T, int QM>
constexpr int fwd_min_waves() {
    return sizeof(T) == 2 && (D <= 64 || QM == 1) ? 4 : 1;
}

// c = scale * log2(e): scores are kept in base 2.  SHORT = 1: every halo row
// holds at most two 16-key blocks (rank >= 2), so the inner-axis mask is a
// per-lane constant; SHORT = 0: general masking with mask-free full blocks.
// QM_ blocks of 16 queries per wave on 16x16x32 steps; SHORT = 2: the narrow form of a
// two-block tiling, one block of 32 queries on 32x32x16 steps (narrow_form).
template <int R, int D, typename T, int QM_, int SB, int SHORT, int W>
__global__ __launch_bounds__(W * kWave, (fwd_min_waves<D, T, QM_>())) void na_fwd_kernel(
    Geo g, const T* __restrict__ qg, const T* __restrict__ kg, const T* __restrict__ vg,
    T* __restrict__ og, float* __restrict__ lseg, float c) {
    using C = FwdCfg<R, D, T, SB, W>;
    constexpr bool kNar = SHORT == 2;
    constexpr int Q = kNar ? 32 : 16, QM = kNar ? 1 : QM_;
    using Ops = TileOps<T, D, Q>;
    using x8 = typename Tr<T>::x8;
    extern __shared__ __align__(16) unsigned char smem_raw[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // (masked: the launch has W waves, which lets the compiler drop the
    // staging loops' bounds tests)
    const int wave = uniform((tid >> 6) & (W - 1));
    const int col = lane & (Q - 1);  // query column of this lane
    const int grp = lane / Q;        // Q-lane group

    // ---- workgroup -> (bh, dilation group, tile) ----
    fetch_geo<R>(g);
    asm volatile("" ::"s"(qg), "s"(kg), "s"(vg), "s"(og), "s"(lseg), "s"(c));
    const int bid = xcd_remap(blockIdx.x, g.nwg);
    int bh, gc[kMaxRank], tc[kMaxRank], n[kMaxRank], to[kMaxRank];
    decode_workgroup<R>(g, bid, bh, gc, tc, n);

    Box<R> halo;
#pragma unroll
    for (int a = 0; a < R; ++a) {
        to[a] = tc[a] * g.T[a];
        if (to[a] >= n[a]) return;  // tile beyond this (shorter) group: uniform exit
        const int last = min(to[a] + g.T[a], n[a]) - 1;
        const bool ca = g.causal[a] != 0;
        halo.lo[a] = win_start(to[a], n[a], g.k[a], ca);
        halo.E[a] = win_last(last, n[a], g.k[a], ca) + 1 - halo.lo[a];
    }
    halo.finish(g, gc);

    const size_t slice = (size_t)bh * g.N * D;
    const T* kb = kg + slice;
    const T* vb = vg + slice;
    const int tstep = g.d[R - 1];  // token step along the innermost axis

    // ---- staging: K and V rows straight to LDS, one address set for both ----
    // The first stage is issued as soon as the halo is known, so that its
    // loads are in flight during the per-wave and per-lane set-up below.
    typename C::Ld ld;
    auto issue_stage = [&](int s, int buf) {
        ld.template compute<kNar>(halo, s * SB, tstep, wave, lane);
        unsigned char* tile = smem_raw + buf * C::kBufBytes;
        ld.issue(kb, tile, wave);
        ld.issue(vb, tile + C::kTileBytes, wave);
    };
    issue_stage(0, 0);

    // ---- this wave's query sub-box: its halo and the keys inside all of its windows ----
    int wc[kMaxRank], wo[kMaxRank];
    unravel_pow2<R>(wave, g.lgWGd, wc);
    bool wave_live = true;
    WaveRange<R> wr;
    MaskRows<R> mrows;  // narrow form
#pragma unroll
    for (int a = 0; a < R; ++a) {
        wo[a] = to[a] + wc[a] * g.WT[a];
        if (wo[a] >= n[a]) wave_live = false;
        const int f = min(wo[a], n[a] - 1);
        const int l = min(wo[a] + g.WT[a], n[a]) - 1;
        const bool ca = g.causal[a] != 0;
        const int sf = win_start(f, n[a], g.k[a], ca), sl = win_start(l, n[a], g.k[a], ca);
        const int ef = win_last(f, n[a], g.k[a], ca), el = win_last(l, n[a], g.k[a], ca);
        wr.set(a, sf - halo.lo[a], el + 1 - halo.lo[a], sl - halo.lo[a], ef + 1 - halo.lo[a]);
        if (kNar && a < R - 1)
            mrows.set(a, sf - halo.lo[a], el + 1 - sf, sl - sf, ef + 1 - sf);
    }
    const int col0 = kNar ? min(wr.lo[R - 1], 8) : 0;  // narrow form: the wave's first column
    if constexpr (kNar) {
        if ((wave & (g.WGd[R - 1] - 1)) == 0 && wave_live)
            mrows.write_table(g, halo, smem_raw + g.tab_off, wave >> g.lgWGd[R - 1], lane);
    }

    // ---- per-lane queries: validity, window starts (relative to the halo), Q ----
    int qs[QM][kMaxRank];
    bool qvalid[QM];
    size_t qoff[QM];
    x8 qf[QM][Ops::kKS];
#pragma unroll
    for (int m = 0; m < QM; ++m) {
        int cc[kMaxRank];
        unravel_pow2<R>(m * Q + col, g.lgWT, cc);
        bool ok = wave_live;
        int tok = 0;
#pragma unroll
        for (int a = 0; a < R; ++a) {
            int p = wo[a] + cc[a];
            if (p >= n[a]) ok = false;
            p = min(p, n[a] - 1);
            qs[m][a] = mask_start(p, n[a], g.k[a], g.causal[a] != 0) - halo.lo[a];
            tok += (gc[a] + g.d[a] * p) * g.ts[a];
        }
        qvalid[m] = ok;
        qoff[m] = slice + (size_t)tok * D;
#pragma unroll
        // unconditional: qoff points at a real (clamped) query even for absent
        // slots, whose results are discarded; no wait before the K/V loads
        for (int s = 0; s < Ops::kKS; ++s)
            qf[m][s] = ld_x8<T>(qg + qoff[m] + s * Ops::kStep + grp * 8);
    }

    Ops ops;
    ops.init(lane, col0);
    i32x4 pen{};  // narrow form: this lane's mask operand
    unsigned tab_lane = 0;
    if constexpr (kNar) {
        unsigned pm = mrows.operand();
#pragma unroll
        for (int a = 0; a < R - 1; ++a)
            pm = mrows.operand(pm, a, qs[0][a], qs[0][a] + g.k[a] - 1);
        pen = mrows.pack_operand(pm, grp);
        tab_lane = g.tab_off + (wave >> g.lgWGd[R - 1]) * g.tab_rows * 32 + (col >> 3) * 32 +
                   grp * 16;
    }

    // ---- online-softmax state (per lane: its query column) ----
    // mref: running reference (base 2, -inf until the row sees a key);
    // negm = -mref (0 while mref = -inf) is the scores' addend and thr the
    // score above which the reference must be raised.
    // Row sums: with kMfmaSum, lsum[m] accumulates the row sums of the rounded
    // P on the matrix cores; otherwise each lane sums its share of P in
    // lrow[m], reduced across the lane groups at the end.
    // Two blocks per wave: the matrix cores at D = 32, and in 1-D at D = 64,
    // where the two extra accumulators leave the occupancy as it is
    // (elsewhere they cost a wave per SIMD).
    constexpr bool kMfmaSum = sizeof(T) == 2 && (QM == 1 || D <= 32 || (R == 1 && D <= 64));
    // Score addends folded into the accumulators.  Not for D = 128 (the
    // addend vectors would cost it occupancy) nor bf16 (rounding c*Q to 8
    // mantissa bits would add an error comparable to that of P itself).
    constexpr bool kFoldAdd = D <= 64 && !std::is_same_v<T, __bf16>;
    x8 ones = Ops::ones_frag(lane);
    // kept in four registers for the whole loop: rebuilt from the constant
    // it would cost three moves per tile
    if constexpr (kMfmaSum) {
        i32x4 u = __builtin_bit_cast(i32x4, ones);
        asm volatile("" : "+v"(u));
        ones = __builtin_bit_cast(x8, u);
    }
    typename Ops::Acc oacc[QM][Ops::kDB];
    f32x4 lsum[QM];
    float mref[QM], negm[QM], thr[QM], lrow[QM];
    // kFoldAdd: negm in all four slots, the accumulator seed of full tiles,
    // kept as a vector so the matrix cores read it in place (no per-tile splat)
    f32x4 negm4[QM];
#pragma unroll
    for (int m = 0; m < QM; ++m) {
        mref[m] = -INFINITY;
        negm[m] = 0.f;
        negm4[m] = f32x4{0.f, 0.f, 0.f, 0.f};
        thr[m] = -INFINITY;
        lsum[m] = f32x4{0.f, 0.f, 0.f, 0.f};
        lrow[m] = 0.f;
#pragma unroll
        for (int db = 0; db < Ops::kDB; ++db) oacc[m][db] = typename Ops::Acc{} * 0.f;
    }
    // Halo rows of at most two 16-key blocks (the usual 2-D / 3-D case): the
    // inner-axis test of this lane's key slots is fixed for the whole
    // kernel, so it is folded into per-slot FMA addends (negm where valid,
    // -inf where not), refreshed only when the reference moves.  Block bi of
    // a tile has inner block index bi when rows hold two blocks, else 0.
    constexpr bool short_rows = SHORT != 0 && R > 1;
    // (the narrow form's tiles hold the wave's eight columns of four rows, so a lane's
    // addends repeat: without kFoldAdd four of them serve the tile, and the mask product
    // seeds the scores.  A second tile for the addends would spill Q at D = 64 and reload
    // it for every tile: 16 x 64 x 64, 7^3 bf16, 8 heads 225 us so, 134 us now; the
    // ordinary form takes 182)
    Tile<Q> ain[QM];
    f32x4 ain4[QM];
    auto refresh_addends = [&](int m) {
        if constexpr (kNar && !kFoldAdd) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool v = (unsigned)(col0 + grp * 4 + r - qs[m][R - 1]) <
                               (unsigned)g.k[R - 1];
                ain4[m][r] = v ? negm[m] : -INFINITY;
            }
        } else {
#pragma unroll
            for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                for (int r = 0; r < Tile<Q>::kN; ++r) {
                    const int ib = halo.nbr == 2 ? bi : 0;
                    const int pos = kNar ? col0 + grp * 4 + (r & 3) : ib * 16 + grp * 4 + r;
                    const bool v = (unsigned)(pos - qs[m][R - 1]) < (unsigned)g.k[R - 1];
                    ain[m].set(bi, r, v ? negm[m] : -INFINITY);
                }
        }
    };
    if (short_rows) {
#pragma unroll
        for (int m = 0; m < QM; ++m) refresh_addends(m);
    }

    const int nst = (halo.nb + SB - 1) / SB;
    wait_vmem();
    __syncthreads();
    // kFoldAdd: Q scaled once by c = scale*log2(e) and rounded to T, so the
    // matrix cores produce base-2 scores (after the wait: the loads above are
    // in flight together)
    if constexpr (kFoldAdd)
#pragma unroll
    for (int m = 0; m < QM; ++m)
#pragma unroll
        for (int st = 0; st < Ops::kKS; ++st)
#pragma unroll
            for (int j = 0; j < 8; ++j) qf[m][st][j] = Tr<T>::cvt((float)qf[m][st][j] * c);
    // (the narrow form without it: masked before the scaling)
    float cs = c;
    if constexpr (kNar && !kFoldAdd) cs = give_sign<T>(qf[0], c);

    ChunkTests<R, SB> ct;  // this wave's block tests, 64 blocks at a time
    for (int s = 0; s < nst; ++s) {
        if (s + 1 < nst) issue_stage(s + 1, (s + 1) & 1);
        const unsigned char* ks = smem_raw + (s & 1) * C::kBufBytes;

        if (wave_live) {
            // the halo's blocks are tested against this wave's queries (one
            // block per lane, 64 at a time); the wave then visits only the
            // tiles (block pairs) with a relevant block, reading their
            // coordinates back from the lanes
            ct.stage(wr, halo, s, lane);
            const uint64_t relm = ct.rel_bits();
            const uint64_t fullm = ct.full_bits();
            const uint64_t ofullm = ct.ofull_bits();
            uint64_t tiles = (relm | (relm >> 1)) & 0x5555555555555555ull;
            if constexpr (kNar) tiles = (tiles | (tiles >> 2)) & 0x1111111111111111ull;
            // The body of one tile (block pair tp), by kind: 0 general; 1 both
            // blocks inside every window of the wave's queries (no mask); 2 short
            // rows, both blocks inside every window along the outer axes (the
            // mask is the per-lane inner-axis addend alone, used in place); 3 / 4
            // short rows, only the first / second block so.
            auto tile = [&](int tp, auto tile_kind) {
                constexpr int kKind = decltype(tile_kind)::value;
                constexpr bool kFull = kKind == 1;
                // block bi inside every window along the outer axes
                constexpr bool kOF[2] = {kKind == 2 || kKind == 3, kKind == 2 || kKind == 4};
                bool rel[2], full[2];
                int boc[2][kMaxRank], bin0[2];
#pragma unroll
                for (int bi = 0; bi < 2; ++bi) {
                    const int j = tp * 2 + bi;
                    rel[bi] = kFull || kOF[bi] || ((relm >> j) & 1);
                    full[bi] = kFull || ((fullm >> j) & 1);
                    bin0[bi] = ct.inner0(j);
#pragma unroll
                    for (int a = 0; a < R - 1; ++a) boc[bi][a] = ct.outer(j, a);
                }

                // ---- S^T = K Q^T for both blocks ----
                // Both blocks are read and multiplied without a branch: a block
                // outside this wave's halo is masked below, and every row of
                // the stage buffer holds finite data (missing keys are
                // stand-in rows).  The V fragments of the tile are read here
                // too (D = 32), so one LDS round trip serves the whole tile.
                constexpr int kRowB = Rows<T, D>::kRowBytes;
                const unsigned char* kt = ks + tp * 32 * kRowB;
                x8 kf[Ops::kF];
                ops.rows(kt, kf);
                constexpr bool kEarlyV = D == 32 && Q == 16;
                constexpr bool kMidV = D <= 64 && Q == 32;
                x8 vf[Ops::kF];
                if (kEarlyV) ops.template cols<C::kTileBytes>(kt, vf);
                if (Q == 32) __builtin_amdgcn_sched_barrier(0);
                // ---- Y^T = c K Q^T + A, A the addend: -m on valid pairs, -inf on masked ----
                // (base 2, relative to the running reference m).  With kFoldAdd the
                // accumulator starts at A and Q is prescaled, so the matrix cores
                // produce Y; otherwise one FMA per score applies c and A.
                auto score_addend = [&](int m, int bi) {
                    f32x4 add;
                    if (!short_rows && full[bi]) {
                        add = f32x4{negm[m], negm[m], negm[m], negm[m]};
                    } else {
                        bool outer_ok = rel[bi];
                        if (!kOF[bi]) {
#pragma unroll
                            for (int a = 0; a < R - 1; ++a)
                                outer_ok = outer_ok &&
                                           (unsigned)(boc[bi][a] - qs[m][a]) < (unsigned)g.k[a];
                        }
                        // generic rows: slot r is valid when base + r lies in [0, lim),
                        // lim folding the outer axes in (0 fails every slot)
                        const int base = bin0[bi] + grp * 4 - qs[m][R - 1];
                        const unsigned lim = outer_ok ? (unsigned)g.k[R - 1] : 0u;
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            add[r] = short_rows ? (outer_ok ? ain[m].at(bi, r) : -INFINITY)
                                     : (unsigned)(base + r) < lim ? negm[m] : -INFINITY;
                    }
                    return add;
                };
                Tile<Q> sacc[QM];
                if constexpr (kNar) {
                    // what the outer axes mask (on top of the inner-axis addends)
                    const i32x4 rows = lds16(smem_raw + tab_lane + (s * SB + tp * 2) * 32);
#pragma unroll
                    for (int m = 0; m < QM; ++m) {
                        sacc[m] = kFoldAdd ? ain[m] : splat_tile<Q>(0.f);
                        sacc[m].v = mma_bf16(rows, pen, sacc[m].v);
#pragma unroll
                        for (int n_ = 0; n_ < Ops::kF; ++n_)
                            Ops::score(sacc[m], kf[n_], n_, qf[m]);
                    }
                } else {
#pragma unroll
                    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                        for (int m = 0; m < QM; ++m) {
                            const int n0 = bi * Ops::kKS;
                            // (the first product of a full tile reads negm4 in place, of an
                            // outer-full tile of short rows the inner addends)
                            if (kFoldAdd && !short_rows && full[bi])
                                sacc[m].b[bi] = Tr<T>::mma(kf[n0], qf[m][0], negm4[m]);
                            else if (kFoldAdd && short_rows && kOF[bi])
                                sacc[m].b[bi] = Tr<T>::mma(kf[n0], qf[m][0], ain[m].b[bi]);
                            else
                                sacc[m].b[bi] = Tr<T>::mma(kf[n0], qf[m][0],
                                                           kFoldAdd ? score_addend(m, bi)
                                                                    : f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                            for (int n_ = n0 + 1; n_ < n0 + Ops::kKS; ++n_)
                                Ops::score(sacc[m], kf[n_], n_, qf[m]);
                        }
                }
                if (kMidV) ops.template cols<C::kTileBytes>(kt, vf);

                // ---- online softmax per query block ----
                x8 pf[QM][Ops::kPF];
#pragma unroll
                for (int m = 0; m < QM; ++m) {
                    constexpr int kN = Tile<Q>::kN;
                    float y[2][kN];
                    if constexpr (kFoldAdd) {
#pragma unroll
                        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                            for (int r = 0; r < kN; ++r) y[bi][r] = sacc[m].at(bi, r);
                    } else {
#pragma unroll
                        for (int bi = 0; bi < 2; ++bi) {
                            f32x4 add;
                            if constexpr (kNar)
                                add = ain4[m];
                            else
                                add = score_addend(m, bi);
#pragma unroll
                            for (int r = 0; r < kN; ++r)
                                y[bi][r] = fmaf(sacc[m].at(bi, r), cs, add[r & 3]);
                        }
                    }
                    // this lane's share of the row; the row maximum exceeds the
                    // threshold exactly when some lane's share does
                    // (a chain, so that it becomes v_max3 instructions)
                    float lmax = y[0][0];
#pragma unroll
                    for (int r = 1; r < 2 * kN; ++r) lmax = fmaxf(lmax, y[r / kN][r % kN]);
                    // raise the reference on the first valid key of a row, or when
                    // the row grows by more than kLazy (rare, wave-uniform branch)
                    if (__builtin_amdgcn_ballot_w64(lmax > thr[m])) {
                        const float ymax = col_max<Q>(lmax);
                        const bool raise = ymax > thr[m];
                        const float dlt = raise ? ymax : 0.f;
                        // a row without a reference has nothing to rescale (and its
                        // first maximum may lie below -128: exp2(-dlt) = inf)
                        const float alpha = thr[m] == -INFINITY ? 0.f : fast_exp2(-dlt);
                        mref[m] = raise ? dlt - negm[m] : mref[m];
                        const bool seen = mref[m] != -INFINITY;
                        negm[m] = seen ? -mref[m] : 0.f;
                        negm4[m] = f32x4{negm[m], negm[m], negm[m], negm[m]};
                        thr[m] = seen ? kLazy : -INFINITY;
                        if (short_rows) refresh_addends(m);
                        if constexpr (kMfmaSum)
                            lsum[m] *= alpha;
                        else
                            lrow[m] *= alpha;
#pragma unroll
                        for (int db = 0; db < Ops::kDB; ++db) oacc[m][db] *= alpha;
#pragma unroll
                        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                            for (int r = 0; r < kN; ++r) y[bi][r] -= dlt;
                    }
                    float p[2][kN];
#pragma unroll
                    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                        for (int r = 0; r < kN; ++r) p[bi][r] = fast_exp2(y[bi][r]);
                    Ops::pack(pf[m], p);
                    if constexpr (!kMfmaSum)
#pragma unroll
                    for (int i = 0; i < Ops::kPF; ++i) lrow[m] = row_sum8<T>(pf[m][i], lrow[m]);
                }

                // ---- O^T += V^T P^T (and the row sums, ones^T P^T) ----
                if (!kEarlyV && !kMidV) ops.template cols<C::kTileBytes>(kt, vf);
#pragma unroll
                for (int n_ = 0; n_ < Ops::kF; ++n_)
#pragma unroll
                    for (int m = 0; m < QM; ++m) Ops::accum(oacc[m], vf[n_], n_, pf[m]);
                if constexpr (kMfmaSum) {
#pragma unroll
                    for (int m = 0; m < QM; ++m) Ops::colsum(lsum[m], ones, pf[m]);
                }
            };
            // Tiles of two full blocks (kind 1, rows of more than two blocks) or
            // of two outer-full blocks (kind 2, short rows) are visited first, by
            // bodies without per-block branches, then (short rows) those with one
            // outer-full block; the order of tiles is free in the online softmax.
            // (narrow form: every tile, of four rows, runs the one body)
            if constexpr (!kNar) run_tile_kinds<short_rows>(tiles, fullm, ofullm, tile);
            while (tiles) {
                const int tp = __builtin_ctzll(tiles) >> 1;
                tiles &= tiles - 1;
                tile(tp, std::integral_constant<int, 0>{});
            }
        }

        // the next stage's rows have landed, and this stage's buffer is free for
        // the loads issued next (no buffer is reused after the last stage)
        if (s + 1 < nst) {
            wait_vmem();
            __syncthreads();
        }
    }

    // ---- epilogue: normalise, store O (rounded once) and the natural-log LSE ----
#pragma unroll
    for (int m = 0; m < QM; ++m) {
        const float l = kMfmaSum ? Ops::colsum_of(lsum[m], lane) : col_sum<Q>(lrow[m]);
        if (!qvalid[m]) continue;
        Ops::store(og + qoff[m], oacc[m], grp, 1.f / l);
        if (grp == 0) lseg[qoff[m] / D] = (mref[m] + __log2f(l)) * kLn2;
    }
}

// ---- host-side launch ----
// Largest number of 16-key blocks in one halo row (interior tiles).
static int max_row_blocks(const Geo& g, int rank) {
    const int a = rank - 1;
    const int n0 = group_len(g.L[a], g.d[a], 0);
    const int e = std::min(std::min(g.T[a], n0) + g.k[a] - 1, n0);
    return (e + 15) / 16;
}

template <int R, int D, typename T, int QM, int SB, int W = 4>
static hipError_t launch_fwd_inst(const Geo& g0, const void* q, const void* k, const void* v,
                                  void* o, float* lse, float scale, hipStream_t stream) {
    using C = FwdCfg<R, D, T, SB, W>;
    // The register bound asks for no more workgroups (of W waves, over the CU's
    // four SIMDs) than its 160 KiB of LDS holds, with double buffers (stages of
    // 16 blocks are used only when the halo fits in one: single) and 8 KiB of mask
    // tables.  (Larger ones leave three workgroups per CU at D = 64, which still is the
    // faster: 9 x 9 x 5 windows, tables of 9 KiB, 250 us in the ordinary form, 191 so.)
    constexpr size_t kTab = R > 1 && sizeof(T) == 2 && QM == 2 ? 8192 : 0;
    static_assert(fwd_min_waves<D, T, QM>() * 4 / W *
                          ((SB >= 16 ? 1 : 2) * C::kBufBytes + kTab) <= 160 * 1024,
                  "register bound beyond the LDS occupancy");
    if (g0.WGd[0] * g0.WGd[1] * g0.WGd[2] != W) return hipErrorInvalidConfiguration;
    const bool short_rows = R > 1 && max_row_blocks(g0, R) <= 2;
    auto kern = na_fwd_kernel<R, D, T, QM, SB, 0, W>;
    if constexpr (R > 1)  // (1-D halos have one row: never short)
        if (short_rows) kern = na_fwd_kernel<R, D, T, QM, SB, 1, W>;
    const int nb_max = max_halo_blocks(g0, R);
    size_t lds = (nb_max > SB ? 2 : 1) * C::kBufBytes;
    Geo g = g0;
    if constexpr (R > 1 && sizeof(T) == 2 && QM == 2) {
        if (narrow_form(g, R, nb_max)) {
            kern = na_fwd_kernel<R, D, T, QM, SB, 2, W>;
            g.tab_off = (int)lds;
            lds += mask_table_bytes(g, R);
        }
    }
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(g.nwg), dim3(C::kThreads), lds, stream, g,
                       static_cast<const T*>(q), static_cast<const T*>(k),
                       static_cast<const T*>(v), static_cast<T*>(o), lse, scale * kLog2e);
    return hipGetLastError();
}

template <int R, int D, typename T>
static hipError_t launch_fwd_qm(const Geo& g, int qm, const void* q, const void* k, const void* v,
                                void* o, float* lse, float scale, hipStream_t stream) {
    if constexpr (sizeof(T) == 4) {
        if (qm == 1) return launch_fwd_inst<R, D, T, 1, 2>(g, q, k, v, o, lse, scale, stream);
        return launch_fwd_inst<R, D, T, 2, 2>(g, q, k, v, o, lse, scale, stream);
    } else {
        // One block per wave at D = 128: stages of half the keys, so that the
        // four waves per SIMD the registers allow also fit in LDS.
        constexpr int kSB1 = D == 128 ? 2 : 4;
        // 1-D: eight waves share each (twice as large) stage
        if constexpr (R == 1) {
            if (g.WGd[0] == 8) {
                if (qm == 1)
                    return launch_fwd_inst<R, D, T, 1, kSB1 * 2, 8>(g, q, k, v, o, lse, scale, stream);
                return launch_fwd_inst<R, D, T, 2, 8, 8>(g, q, k, v, o, lse, scale, stream);
            }
        }
        // one LDS stage covering the whole halo when it is small and D is 32
        if constexpr (D == 32) {
            if (max_halo_blocks(g, R) <= 16) {
                if (qm == 1) return launch_fwd_inst<R, D, T, 1, 16>(g, q, k, v, o, lse, scale, stream);
                return launch_fwd_inst<R, D, T, 2, 16>(g, q, k, v, o, lse, scale, stream);
            }
        }
        if (qm == 1) return launch_fwd_inst<R, D, T, 1, kSB1>(g, q, k, v, o, lse, scale, stream);
        return launch_fwd_inst<R, D, T, 2, 4>(g, q, k, v, o, lse, scale, stream);
    }
}

template <int R, typename T>
static hipError_t launch_fwd_d(const Geo& g, int D, int qm, const void* q, const void* k,
                               const void* v, void* o, float* lse, float scale, hipStream_t s) {
    switch (D) {
        case 32: return launch_fwd_qm<R, 32, T>(g, qm, q, k, v, o, lse, scale, s);
        case 64: return launch_fwd_qm<R, 64, T>(g, qm, q, k, v, o, lse, scale, s);
        case 128: return launch_fwd_qm<R, 128, T>(g, qm, q, k, v, o, lse, scale, s);
    }
    return hipErrorInvalidValue;
}

template <typename T>
static hipError_t launch_fwd_r(const Geo& g, int rank, int D, int qm, const void* q, const void* k,
                               const void* v, void* o, float* lse, float scale, hipStream_t s) {
    switch (rank) {
        case 1: return launch_fwd_d<1, T>(g, D, qm, q, k, v, o, lse, scale, s);
        case 2: return launch_fwd_d<2, T>(g, D, qm, q, k, v, o, lse, scale, s);
        case 3: return launch_fwd_d<3, T>(g, D, qm, q, k, v, o, lse, scale, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_forward(const Geo& g, int rank, int D, int dtype, int qm, const void* q,
                          const void* k, const void* v, void* o, float* lse, float scale,
                          hipStream_t s) {
    switch (dtype) {
        case 0: return launch_fwd_r<float>(g, rank, D, qm, q, k, v, o, lse, scale, s);
        case 1: return launch_fwd_r<_Float16>(g, rank, D, qm, q, k, v, o, lse, scale, s);
        case 2: return launch_fwd_r<__bf16>(g, rank, D, qm, q, k, v, o, lse, scale, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace na
