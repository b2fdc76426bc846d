// na_bwd.hip -- fused neighborhood-attention backward for gfx950.
//
// The backward pass is built from the three operators of Sec. 3.1, each run
// fused so that no attention weight reaches global memory:
//   PN  dP = dO V^T        (PN applied to the output gradient and V)
//   NN  dQ = scale dA K    over each query's neighbourhood
//   IN  dK = scale dA^T Q, dV = P^T dO  over each key's inverse neighbourhood
// with dA = P * (dP - Delta), Delta = rowsum(dO * O), and P recomputed from
// the logsumexp saved by the forward pass.  One launch, two workgroup roles,
// no atomics and no workspace, so the result is deterministic:
//   dK/dV role  one workgroup per key tile; its queries are the union of the
//               tile's inverse neighbourhoods (Sec. 3.1: the relation is not
//               symmetric and a key may be attended by up to k + floor(k/2)
//               queries per axis); Delta of every staged query is formed
//               while staging, from the O and dO rows
//   dQ role     one workgroup per query tile over its key halo, like the
//               forward pass; Delta of its own queries from their fragments
// The roles are independent, so they share the GPU instead of running as
// consecutive launches.
#include <algorithm>
#include <type_traits>

#include "na_launch.h"
#include "na_stage.h"

namespace na {

// Addressing of the stage loads of a kernel with M blocks per wave (see Addr).
template <int R, int D, typename T, int M>
constexpr Addr bwd_addr() {
    if (sizeof(T) != 2 || (R == 3 && D == 128)) return Addr::kByBlock;
    return R == 2 && M == 1 && D <= 64 ? Addr::kUntracked : Addr::kByLane;
}

// ---------------------------------------------------------------------------
// dQ: query-major, over each query tile's key halo.
// ---------------------------------------------------------------------------
template <int R, int D, typename T, int SB>
struct DqCfg {
    static constexpr int kThreads = 4 * kWave;
    static constexpr int kKeys = SB * 16;
    static constexpr int kTileBytes = kKeys * Rows<T, D>::kRowBytes;
    static constexpr size_t kBufBytes = 2 * kTileBytes;  // K rows, then V rows
    template <int M>
    using Ld = DirectRows<T, D, kKeys, 4, (R > 1), bwd_addr<R, D, T, M>()>;
};

// QM blocks of 16 queries per wave on 16x16x32 steps.
// SHORT = 1: every halo row holds at most two 16-key blocks (rank >= 2), so
// the inner-axis mask is a per-lane constant (chosen on the host).
// SHORT = 2: the narrow form of a QM = 2 tiling, one block of 32 queries on 32x32x16
// steps with the outer-axis masks from a MaskRows table.
// braw: the workgroup's index among the dQ-role workgroups.
template <int R, int D, typename T, int QM_, int SB, int SHORT>
__device__ __forceinline__ void dq_role(const Geo& g, int braw, unsigned char* smem_raw,
                                        const T* __restrict__ qg, const T* __restrict__ kg,
                                        const T* __restrict__ vg, const T* __restrict__ og,
                                        const T* __restrict__ dog, const float* __restrict__ lseg,
                                        T* __restrict__ dqg, float scale_log2, float scale) {
    using C = DqCfg<R, D, T, SB>;
    constexpr bool kNar = SHORT == 2;
    constexpr int Q = kNar ? 32 : 16, QM = kNar ? 1 : QM_;
    using Ops = TileOps<T, D, Q>;
    using x8 = typename Tr<T>::x8;
    constexpr int kRowB = Rows<T, D>::kRowBytes;
    constexpr int kN = Tile<Q>::kN;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = uniform((tid >> 6) & (C::kThreads / kWave - 1));  // (bounds the staging loops)
    const int col = lane & (Q - 1);
    const int grp = lane / Q;

    const int bid = xcd_remap(braw, g.nwg);
    int bh, gc[kMaxRank], tc[kMaxRank], n[kMaxRank], to[kMaxRank];
    decode_workgroup<R>(g, bid, bh, gc, tc, n);

    Box<R> halo;
#pragma unroll
    for (int a = 0; a < R; ++a) {
        to[a] = tc[a] * g.T[a];
        if (to[a] >= n[a]) return;
        const int last = min(to[a] + g.T[a], n[a]) - 1;
        const bool ca = g.causal[a] != 0;
        halo.lo[a] = win_start(to[a], n[a], g.k[a], ca);
        halo.E[a] = win_last(last, n[a], g.k[a], ca) + 1 - halo.lo[a];
    }
    halo.finish(g, gc);

    const size_t slice = (size_t)bh * g.N * D;
    const T* kb = kg + slice;
    const T* vb = vg + slice;

    // The first stage is issued as soon as the halo is known, so that its
    // loads are in flight during the per-wave and per-lane set-up below.
    const int tstep = g.d[R - 1];
    typename C::template Ld<QM_> ld;
    auto issue_stage = [&](int s, int buf) {
        ld.template compute<false>(halo, s * SB, tstep, wave, lane);
        unsigned char* tile = smem_raw + buf * C::kBufBytes;
        ld.issue(kb, tile, wave);
        ld.issue(vb, tile + C::kTileBytes, wave);
    };
    issue_stage(0, 0);

    int wc[kMaxRank], wo[kMaxRank];
    unravel_pow2<R>(wave, g.lgWGd, wc);
    bool wave_live = true;
    WaveRange<R> wr;
    MaskRows<R> mrows;  // kNar
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

    int qs[QM][kMaxRank];
    bool qvalid[QM];
    size_t qoff[QM];
    x8 qf[QM][Ops::kKS], gf[QM][Ops::kKS], of[QM][Ops::kKS];
    float lse2[QM], dlt[QM];
#pragma unroll
    for (int m = 0; m < QM; ++m) {
        int c[kMaxRank];
        unravel_pow2<R>(m * Q + col, g.lgWT, c);
        bool ok = wave_live;
        int tok = 0;
#pragma unroll
        for (int a = 0; a < R; ++a) {
            int p = wo[a] + c[a];
            if (p >= n[a]) ok = false;
            p = min(p, n[a] - 1);
            qs[m][a] = mask_start(p, n[a], g.k[a], g.causal[a] != 0) - halo.lo[a];
            tok += (gc[a] + g.d[a] * p) * g.ts[a];
        }
        qvalid[m] = ok;
        qoff[m] = slice + (size_t)tok * D;
#pragma unroll
        // unconditional: qoff points at a real (clamped) query even for absent
        // slots, whose results are discarded
        for (int s = 0; s < Ops::kKS; ++s) {
            const int e = s * Ops::kStep + grp * 8;
            qf[m][s] = ld_x8<T>(qg + qoff[m] + e);
            gf[m][s] = ld_x8<T>(dog + qoff[m] + e);
            of[m][s] = ld_x8<T>(og + qoff[m] + e);
        }
        lse2[m] = lseg[qoff[m] / D] * kLog2e;
    }

    Ops ops;
    ops.init(lane, col0);
    i32x4 pen{};  // kNar: this lane's mask operand, and its part of a tile's rows
    unsigned tab_lane = 0;
    if constexpr (kNar) {
        unsigned pm = mrows.operand();
#pragma unroll
        for (int a = 0; a < R - 1; ++a)
            pm = mrows.operand(pm, a, qs[0][a], qs[0][a] + g.k[a] - 1);
        pen = mrows.pack_operand(pm, grp);
        tab_lane = g.tab_off + (wave >> g.lgWGd[R - 1]) * g.tab_rows * 32 +
                   (col >> 3) * 32 + grp * 16;
    }

    typename Ops::Acc dqacc[QM][Ops::kDB];
#pragma unroll
    for (int m = 0; m < QM; ++m)
#pragma unroll
        for (int db = 0; db < Ops::kDB; ++db) dqacc[m][db] = typename Ops::Acc{};
    // Halo rows of at most two 16-key blocks: the inner-axis test of this
    // lane's 4 key slots is fixed, folded with -lse2 into per-slot addends.
    constexpr bool short_rows = SHORT != 0 && R > 1;
    // Score addends folded into the accumulators (not for D = 128 or bf16,
    // as in the forward)
    constexpr bool kFoldAdd = D <= 64 && !std::is_same_v<T, __bf16>;
    // (narrow form: as in the forward)
    Tile<Q> ain[QM];
    f32x4 ain4{};
    if constexpr (kNar && !kFoldAdd)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            ain4[r] = (unsigned)(col0 + grp * 4 + r - qs[0][R - 1]) < (unsigned)g.k[R - 1]
                          ? -lse2[0]
                          : -INFINITY;
#pragma unroll
    for (int m = 0; m < QM; ++m)
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int r = 0; r < kN; ++r) {
                const int ib = halo.nbr == 2 ? bi : 0;
                const int pos = kNar ? col0 + grp * 4 + (r & 3) : ib * 16 + grp * 4 + r;
                ain[m].set(bi, r, (unsigned)(pos - qs[m][R - 1]) < (unsigned)g.k[R - 1]
                                      ? -lse2[m]
                                      : -INFINITY);
            }

    const int nst = (halo.nb + SB - 1) / SB;
    // Delta = dO . O of this lane's queries: 4 lanes hold a query's D slots
#pragma unroll
    for (int m = 0; m < QM; ++m) {
        float part = 0.f;
#pragma unroll
        for (int s = 0; s < Ops::kKS; ++s) part = dot8<T>(of[m][s], gf[m][s], part);
        dlt[m] = col_sum<Q>(part);
    }
    wait_vmem();
    __syncthreads();
    // -lse2 in all four slots: the accumulator seed of full tiles (kFoldAdd)
    f32x4 nlse4[QM];
#pragma unroll
    for (int m = 0; m < QM; ++m) nlse4[m] = f32x4{-lse2[m], -lse2[m], -lse2[m], -lse2[m]};
    // kFoldAdd: Q scaled once by c = scale*log2(e) and rounded to T
    if constexpr (kFoldAdd)
#pragma unroll
    for (int m = 0; m < QM; ++m)
#pragma unroll
        for (int st = 0; st < Ops::kKS; ++st)
#pragma unroll
            for (int j = 0; j < 8; ++j) qf[m][st][j] = Tr<T>::cvt((float)qf[m][st][j] * scale_log2);
    float cs = scale_log2;
    if constexpr (kNar && !kFoldAdd) cs = give_sign<T>(qf[0], scale_log2);

    ChunkTests<R, SB> ct;  // this wave's block tests, 64 blocks at a time
    for (int s = 0; s < nst; ++s) {
        if (s + 1 < nst) issue_stage(s + 1, (s + 1) & 1);
        const unsigned char* ks = smem_raw + (s & 1) * C::kBufBytes;
        const unsigned char* vs = ks + C::kTileBytes;

        if (wave_live) {
            // blocks are tested one per lane, 64 at a time; only tiles with a
            // relevant block are visited, their coordinates read back from the
            // lanes
            ct.stage(wr, halo, s, lane);
            const uint64_t relm = ct.rel_bits();
            const uint64_t fullm = ct.full_bits();
            const uint64_t ofullm = ct.ofull_bits();
            uint64_t tiles = (relm | (relm >> 1)) & 0x5555555555555555ull;
            if constexpr (kNar) tiles = (tiles | (tiles >> 2)) & 0x1111111111111111ull;
            // The body of one tile (block pair tp), by kind, as in the forward:
            // 0 general; 1 both blocks inside every window of the wave's queries;
            // 2 short rows, both blocks inside every window along the outer axes;
            // 3 / 4 short rows, only the first / second block so.
            auto tile = [&](int tp, auto tile_kind) {
                constexpr int kKind = decltype(tile_kind)::value;
                constexpr bool kFull = kKind == 1;
                // block bi inside every range along the outer axes
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

                // Y^T = c K Q^T + A (A: -lse2 on valid pairs, -inf on masked; with
                // kFoldAdd the accumulator starts at A and Q is prescaled by c) and
                // dP^T - Delta = V dO^T - Delta (the accumulator starts at -Delta)
                auto score_addend = [&](int m, int bi) {
                    f32x4 add;
                    if (!short_rows && full[bi]) {
                        add = f32x4{-lse2[m], -lse2[m], -lse2[m], -lse2[m]};
                    } else {
                        bool outer_ok = rel[bi];
                        if (!kOF[bi]) {
#pragma unroll
                            for (int a = 0; a < R - 1; ++a)
                                outer_ok = outer_ok &&
                                           (unsigned)(boc[bi][a] - qs[m][a]) < (unsigned)g.k[a];
                        }
                        // generic rows: slot r is valid when base + r lies in [0, lim)
                        const int base = bin0[bi] + grp * 4 - qs[m][R - 1];
                        const unsigned lim = outer_ok ? (unsigned)g.k[R - 1] : 0u;
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            add[r] = short_rows ? (outer_ok ? ain[m].at(bi, r) : -INFINITY)
                                     : (unsigned)(base + r) < lim ? -lse2[m] : -INFINITY;
                    }
                    return add;
                };
                const unsigned char* kt = ks + tp * 32 * kRowB;
                if constexpr (kNar) {
                    // Every row of the tile is multiplied (rows that no query of the wave
                    // needs are masked): the inner-axis addends, plus what the outer axes
                    // mask, seed the scores.
                    x8 fr[Ops::kF];
                    ops.rows(kt, fr);
                    const i32x4 rows = lds16(smem_raw + tab_lane + (s * SB + tp * 2) * 32);
                    Tile<Q> sacc, pacc;
                    sacc = kFoldAdd ? ain[0] : splat_tile<Q>(0.f);
                    sacc.v = mma_bf16(rows, pen, sacc.v);
#pragma unroll
                    for (int n_ = 0; n_ < Ops::kF; ++n_) Ops::score(sacc, fr[n_], n_, qf[0]);
                    x8 fv[Ops::kF];
                    ops.rows(kt + C::kTileBytes, fv);
                    pacc = splat_tile<Q>(0.f);
#pragma unroll
                    for (int n_ = 0; n_ < Ops::kF; ++n_) Ops::score(pacc, fv[n_], n_, gf[0]);
                    // K^T for dQ^T += K^T dA^T, read while the products run
                    x8 fc[Ops::kF];
                    ops.template cols<0>(kt, fc);
                    // dA^T = P^T (dP^T - Delta), P = exp2(Y^T)
                    float ds[2][kN];
#pragma unroll
                    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                        for (int r = 0; r < kN; ++r) {
                            float y = sacc.at(bi, r);
                            if constexpr (!kFoldAdd) y = fmaf(y, cs, ain4[r & 3]);
                            ds[bi][r] = fast_exp2(y) * (pacc.at(bi, r) - dlt[0]);
                        }
                    x8 dsf[Ops::kPF];
                    Ops::pack(dsf, ds);
#pragma unroll
                    for (int n_ = 0; n_ < Ops::kF; ++n_) Ops::accum(dqacc[0], fc[n_], n_, dsf);
                    return;
                } else {
                f32x4 sacc[QM][2], pacc[QM][2];
#pragma unroll
                for (int bi = 0; bi < 2; ++bi) {
                    if (rel[bi]) {
                        const int boff = (tp * 2 + bi) * 16 * kRowB;
#pragma unroll
                        for (int st = 0; st < Ops::kKS; ++st) {
                            const x8 kf = ops.rf.read(ks + boff, st);
                            const x8 vf = ops.rf.read(vs + boff, st);
#pragma unroll
                            for (int m = 0; m < QM; ++m) {
                                if (st > 0)
                                    sacc[m][bi] = Tr<T>::mma(kf, qf[m][st], sacc[m][bi]);
                                else if (kFoldAdd && !short_rows && full[bi])
                                    sacc[m][bi] = Tr<T>::mma(kf, qf[m][0], nlse4[m]);  // in place
                                else if (kFoldAdd && short_rows && kOF[bi])
                                    sacc[m][bi] =
                                        Tr<T>::mma(kf, qf[m][0], ain[m].b[bi]);  // in place
                                else
                                    sacc[m][bi] = Tr<T>::mma(kf, qf[m][0],
                                                             kFoldAdd ? score_addend(m, bi)
                                                                      : f32x4{0.f, 0.f, 0.f, 0.f});
                                const f32x4 nd = f32x4{-dlt[m], -dlt[m], -dlt[m], -dlt[m]};
                                pacc[m][bi] = Tr<T>::mma(vf, gf[m][st], st == 0 ? nd : pacc[m][bi]);
                            }
                        }
                    } else {
#pragma unroll
                        for (int m = 0; m < QM; ++m) {
                            const float s0 = kFoldAdd ? -INFINITY : 0.f;
                            sacc[m][bi] = f32x4{s0, s0, s0, s0};
                            pacc[m][bi] = f32x4{0.f, 0.f, 0.f, 0.f};
                        }
                    }
                }

                // dA^T = P^T (dP^T - Delta), P = exp2(Y^T)
                x8 dsf[QM][Ops::kPF];
#pragma unroll
                for (int m = 0; m < QM; ++m) {
                    float ds[2][4];
#pragma unroll
                    for (int bi = 0; bi < 2; ++bi) {
                        f32x4 y = sacc[m][bi];
                        if constexpr (!kFoldAdd) {
                            const f32x4 add = score_addend(m, bi);
#pragma unroll
                            for (int r = 0; r < 4; ++r) y[r] = fmaf(y[r], scale_log2, add[r]);
                        }
#pragma unroll
                        for (int r = 0; r < 4; ++r) ds[bi][r] = fast_exp2(y[r]) * pacc[m][bi][r];
                    }
                    Ops::pack(dsf[m], ds);
                }

                // dQ^T += K^T dA^T (K^T read transposed from the K rows)
#pragma unroll
                for (int db = 0; db < Ops::kDB; ++db) {
                    const x8 kf = ops.cf.read(kt, db, lane);
#pragma unroll
                    for (int m = 0; m < QM; ++m) Ops::accum(dqacc[m], kf, db, dsf[m]);
                }
                }
            };
            // the specialised tiles first (the order of tiles does not matter; the
            // narrow form has one body)
            if constexpr (!kNar) run_tile_kinds<short_rows>(tiles, fullm, ofullm, tile);
            while (tiles) {
                const int tp = __builtin_ctzll(tiles) >> 1;
                tiles &= tiles - 1;
                tile(tp, std::integral_constant<int, 0>{});
            }
        }

        if (s + 1 < nst) {  // (no buffer is reused after the last stage)
            wait_vmem();
            __syncthreads();
        }
    }

#pragma unroll
    for (int m = 0; m < QM; ++m) {
        if (!qvalid[m]) continue;
        Ops::store(dqg + qoff[m], dqacc[m], grp, scale);
    }
}

// ---------------------------------------------------------------------------
// dK, dV: key-major, over the union of the key tile's inverse neighbourhoods.
// ---------------------------------------------------------------------------
// DIN: -Delta of every query comes from memory (written by a pre-pass), so
// neither O rows nor a Delta pass are needed.
template <int R, int D, typename T, int SB, bool DIN = false>
struct DkvCfg {
    static constexpr int kThreads = 4 * kWave;
    static constexpr int kRows = SB * 16;  // queries per stage
    static constexpr int kTileBytes = kRows * Rows<T, D>::kRowBytes;
    // Without DIN, one staged query per thread (the whole box in one stage):
    // each thread forms Delta of its query from its O row in registers, and
    // no O tile is staged.  Otherwise O rows are staged beside Q and dO.
    static constexpr bool kRegDelta = !DIN && kRows == kThreads;
    static constexpr int kTiles = (DIN || kRegDelta) ? 2 : 3;
    // Q rows, dO rows, [O rows,] then fp32 -lse2 and -Delta per query
    static constexpr size_t kFloatOff = (size_t)kTiles * kTileBytes;
    static constexpr size_t kBufBytes = kFloatOff + 2 * kRows * sizeof(float);
    template <int M>
    using Ld = DirectRows<T, D, kRows, 4, (R > 1), bwd_addr<R, D, T, M>()>;
};

// SHORT = 1: every query-box row holds at most two 16-query blocks (rank >= 2).
// braw: the workgroup's index among the nwk dK/dV-role workgroups (nwk is
// g.nwg rounded up to a multiple of the 8 XCDs; the surplus ones exit).
// DIN: ndg holds -Delta of every query ([B * H * N] fp32, from the pre-pass).
template <int R, int D, typename T, int KM, int SB, int SHORT, bool DIN>
__device__ __forceinline__ void dkdv_role(const Geo& g, int braw, int nwk,
                                          unsigned char* smem_raw, const T* __restrict__ qg,
                                          const T* __restrict__ kg, const T* __restrict__ vg,
                                          const T* __restrict__ og, const T* __restrict__ dog,
                                          const float* __restrict__ lseg,
                                          const float* __restrict__ ndg, T* __restrict__ dkg,
                                          T* __restrict__ dvg, float scale_log2, float scale) {
    using C = DkvCfg<R, D, T, SB, DIN>;
    using Ops = TileOps<T, D, 16>;
    using x8 = typename Tr<T>::x8;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = uniform((tid >> 6) & (C::kThreads / kWave - 1));  // (bounds the staging loops)
    const int col = lane & 15;  // key column of this lane
    const int grp = lane >> 4;

    const int bid = xcd_remap(braw, nwk);
    if (bid >= g.nwg) return;
    int bh, gc[kMaxRank], tc[kMaxRank], n[kMaxRank], to[kMaxRank];
    decode_workgroup<R>(g, bid, bh, gc, tc, n);

    // key tile [to, last] and the box of queries attending to it
    Box<R> ibox;
#pragma unroll
    for (int a = 0; a < R; ++a) {
        to[a] = tc[a] * g.T[a];
        if (to[a] >= n[a]) return;
        const int last = min(to[a] + g.T[a], n[a]) - 1;
        const bool ca = g.causal[a] != 0;
        ibox.lo[a] = inv_lo(to[a], n[a], g.k[a], ca);
        ibox.E[a] = inv_hi(last, n[a], g.k[a], ca) + 1 - ibox.lo[a];
    }
    ibox.finish(g, gc);

    const size_t slice = (size_t)bh * g.N * D;
    const T* qb = qg + slice;
    const T* gb = dog + slice;
    const T* ob = og + slice;
    const float* lb = lseg + (size_t)bh * g.N;
    const float* nb_ = DIN ? ndg + (size_t)bh * g.N : nullptr;

    const int tstep = g.d[R - 1];
    typename C::template Ld<KM> ld;
    using L = Rows<T, D>;
    // the stage's per-query values as loaded (row tid of the stage), and
    // whether the row holds a query; combined only where they are stored
    float lse_raw = 0.f, ndl_raw = 0.f;
    bool row_ok = false;
    i32x4 orow[L::kSegs];  // kRegDelta: this thread's O row
    auto issue_stage = [&](int s, int buf) {
        ld.template compute<false>(ibox, s * SB, tstep, wave, lane);
        unsigned char* tile = smem_raw + buf * C::kBufBytes;
        ld.issue(qb, tile, wave);
        ld.issue(gb, tile + C::kTileBytes, wave);
        if constexpr (!DIN && !C::kRegDelta) ld.issue(ob, tile + 2 * C::kTileBytes, wave);
        // Every thread loads (threads past the stage's rows read a real token
        // too, whose values are never stored), with nothing computed from the
        // loaded values here: they are combined only in put_floats, so that
        // no wait for them (nor for the staging loads above) is needed before
        // the stage's tiles run.
        {
            int valid;
            const int tok0 = ibox.block_token(s * SB + (tid >> 4), valid);
            row_ok = (tid & 15) < valid;
            const int tk = row_ok ? tok0 + (tid & 15) * tstep : 0;  // token 0: safe stand-in
            lse_raw = lb[tk];
            if constexpr (DIN) ndl_raw = nb_[tk];  // already -Delta
            if constexpr (C::kRegDelta) {
#pragma unroll
                for (int sg = 0; sg < L::kSegs; ++sg)
                    orow[sg] = ld16<i32x4>(ob + (size_t)tk * D + sg * L::kVec);
            }
        }
    };
    // The first stage is issued as soon as the query box is known, so that
    // its loads are in flight during the per-wave and per-lane set-up below.
    issue_stage(0, 0);

    // this wave's key sub-box: the queries that attend to any / all of its keys
    int wc[kMaxRank], wo[kMaxRank];
    unravel_pow2<R>(wave, g.lgWGd, wc);
    bool wave_live = true;
    WaveRange<R> wr;
#pragma unroll
    for (int a = 0; a < R; ++a) {
        wo[a] = to[a] + wc[a] * g.WT[a];
        if (wo[a] >= n[a]) wave_live = false;
        const int f = min(wo[a], n[a] - 1);
        const int l = min(wo[a] + g.WT[a], n[a]) - 1;
        const bool ca = g.causal[a] != 0;
        wr.set(a, inv_lo(f, n[a], g.k[a], ca) - ibox.lo[a],
               inv_hi(l, n[a], g.k[a], ca) + 1 - ibox.lo[a],
               inv_lo(l, n[a], g.k[a], ca) - ibox.lo[a],
               inv_hi(f, n[a], g.k[a], ca) + 1 - ibox.lo[a]);
    }

    // per-lane keys: group coordinates, K and V fragments
    int kc[KM][kMaxRank];
    bool kvalid[KM];
    size_t koff[KM];
    x8 kf[KM][Ops::kKS], vf[KM][Ops::kKS];
#pragma unroll
    for (int m = 0; m < KM; ++m) {
        int c[kMaxRank];
        unravel_pow2<R>(m * 16 + col, g.lgWT, c);
        bool ok = wave_live;
        int tok = 0;
#pragma unroll
        for (int a = 0; a < R; ++a) {
            int p = wo[a] + c[a];
            if (p >= n[a]) ok = false;
            p = min(p, n[a] - 1);
            kc[m][a] = p;
            tok += (gc[a] + g.d[a] * p) * g.ts[a];
        }
        kvalid[m] = ok;
        koff[m] = slice + (size_t)tok * D;
#pragma unroll
        // unconditional: koff points at a real (clamped) key even for absent
        // slots, whose results are discarded
        for (int s = 0; s < Ops::kKS; ++s) {
            kf[m][s] = ld_x8<T>(kg + koff[m] + s * Ops::kStep + grp * 8);
            vf[m][s] = ld_x8<T>(vg + koff[m] + s * Ops::kStep + grp * 8);
        }
    }

    // A query q attends to this lane's key j exactly when q lies in j's
    // inverse range [inv_lo(j), inv_hi(j)] on every axis (contiguous, since
    // window starts are non-decreasing): per lane, relative to the query box.
    int ilo[KM][kMaxRank], ispan[KM][kMaxRank];
#pragma unroll
    for (int m = 0; m < KM; ++m)
#pragma unroll
        for (int a = 0; a < R; ++a) {
            const bool ca = g.causal[a] != 0;
            const int lo = inv_lo(kc[m][a], n[a], g.k[a], ca);
            ilo[m][a] = lo - ibox.lo[a];
            ispan[m][a] = inv_hi(kc[m][a], n[a], g.k[a], ca) - lo;
        }
    // Query-box rows of at most two 16-query blocks: the inner-axis test of
    // this lane's 4 query slots is fixed, folded into 0 / -inf addends.
    constexpr bool short_rows = SHORT != 0 && R > 1;
    // Score addends folded into the accumulators (not for D = 128 or bf16,
    // as in the forward)
    constexpr bool kFoldAdd = D <= 64 && !std::is_same_v<T, __bf16>;
    float ain[KM][2][4];
#pragma unroll
    for (int m = 0; m < KM; ++m)
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ib = ibox.nbr == 2 ? bi : 0;
                ain[m][bi][r] = (unsigned)(ib * 16 + grp * 4 + r - ilo[m][R - 1]) <=
                                        (unsigned)ispan[m][R - 1]
                                    ? 0.f
                                    : -INFINITY;
            }
    auto floats = [&](int buf) {
        return reinterpret_cast<float*>(smem_raw + buf * C::kBufBytes + C::kFloatOff);
    };
    // 16-byte dot product in fp32
    auto dot16 = [&](i32x4 a, i32x4 b, float acc) {
        if constexpr (sizeof(T) == 2) {
            return dot8<T>(__builtin_bit_cast(x8, a), __builtin_bit_cast(x8, b), acc);
        } else {
            const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
            return fmaf(x[3], y[3], fmaf(x[2], y[2], fmaf(x[1], y[1], fmaf(x[0], y[0], acc))));
        }
    };
    // Delta = dO . O of the stage's staged queries (dO from its LDS rows; O
    // from its LDS rows with kThreads / kRows lanes per query reduced by lane
    // shuffles, or from the thread's registers); the float area holds -lse2
    // and -Delta per staged query
    auto delta_pass = [&](int buf) {
        const unsigned char* gt = smem_raw + buf * C::kBufBytes + C::kTileBytes;
        if constexpr (DIN) {
            (void)gt;
        } else if constexpr (C::kRegDelta) {
            float acc = 0.f;
#pragma unroll
            for (int sg = 0; sg < L::kSegs; ++sg) acc = dot16(lds16(gt + L::off(tid, sg)), orow[sg], acc);
            floats(buf)[C::kRows + tid] = -acc;  // staged negated: -Delta
        } else {
            constexpr int kP = C::kThreads / C::kRows;
            constexpr int kSpt = (L::kSegs + kP - 1) / kP;
            const unsigned char* ot = gt + C::kTileBytes;
            const int row = tid / kP, part = tid % kP;
            float acc = 0.f;
#pragma unroll
            for (int i = 0; i < kSpt; ++i) {
                const int seg = part * kSpt + i;
                if (seg < L::kSegs) {
                    const int o = L::off(row, seg);
                    acc = dot16(lds16(gt + o), lds16(ot + o), acc);
                }
            }
#pragma unroll
            for (int w = 1; w < kP; w <<= 1) acc += __shfl_xor(acc, w, kWave);
            if (part == 0) floats(buf)[C::kRows + row] = -acc;  // staged negated: -Delta
        }
    };
    Ops ops;
    ops.init(lane);
    constexpr int kRowB = Rows<T, D>::kRowBytes;

    typename Ops::Acc dkacc[KM][Ops::kDB], dvacc[KM][Ops::kDB];
#pragma unroll
    for (int m = 0; m < KM; ++m)
#pragma unroll
        for (int d = 0; d < Ops::kDB; ++d) {
            dkacc[m][d] = typename Ops::Acc{};
            dvacc[m][d] = typename Ops::Acc{};
        }

    const int nst = (ibox.nb + SB - 1) / SB;
    // the per-query floats of a stage: -lse2, and -Delta when it comes from memory
    auto put_floats = [&](int buf) {
        if (tid < C::kRows) {
            floats(buf)[tid] = row_ok ? -lse_raw * kLog2e : 0.f;  // staged negated: -lse2
            if constexpr (DIN) floats(buf)[C::kRows + tid] = row_ok ? ndl_raw : 0.f;
        }
    };
    put_floats(0);
    wait_vmem();
    __syncthreads();
    delta_pass(0);
    // kFoldAdd: K scaled once by c = scale*log2(e) and rounded to T
    if constexpr (kFoldAdd)
#pragma unroll
    for (int m = 0; m < KM; ++m)
#pragma unroll
        for (int st = 0; st < Ops::kKS; ++st)
#pragma unroll
            for (int j = 0; j < 8; ++j) kf[m][st][j] = Tr<T>::cvt((float)kf[m][st][j] * scale_log2);
    if constexpr (!DIN) __syncthreads();  // Delta of the first stage written

    ChunkTests<R, SB> ct;  // this wave's block tests, 64 blocks at a time
    for (int s = 0; s < nst; ++s) {
        if (s + 1 < nst) issue_stage(s + 1, (s + 1) & 1);
        const unsigned char* qs = smem_raw + (s & 1) * C::kBufBytes;
        const unsigned char* gs = qs + C::kTileBytes;
        const float* ls = floats(s & 1);
        const float* dls = ls + C::kRows;

        if (wave_live) {
            // blocks are tested one per lane, 64 at a time; only tiles with a
            // relevant block are visited, their coordinates read back from the
            // lanes
            ct.stage(wr, ibox, s, lane);
            const uint64_t relm = ct.rel_bits();
            const uint64_t fullm = ct.full_bits();
            const uint64_t ofullm = ct.ofull_bits();
            uint64_t tiles = (relm | (relm >> 1)) & 0x5555555555555555ull;
            // The body of one tile (block pair tp), by kind: 0 general; 1 both
            // query blocks attend every key of the wave; 2 short rows, both
            // blocks inside the wave's inverse ranges along the outer axes; 3 / 4
            // short rows, only the first / second block so.
            auto tile = [&](int tp, auto tile_kind) {
                constexpr int kKind = decltype(tile_kind)::value;
                constexpr bool kFull = kKind == 1;
                // block bi inside every range along the outer axes
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

                const unsigned char* qt = qs + tp * 32 * kRowB;
                // -lse2 and -Delta of the 2 x 4 queries this lane holds
                f32x4 nlse[2], ndl[2];
#pragma unroll
                for (int bi = 0; bi < 2; ++bi) {
                    const int srow = (tp * 2 + bi) * 16 + grp * 4;
                    nlse[bi] = ld16<f32x4>(ls + srow);
                    ndl[bi] = ld16<f32x4>(dls + srow);
                }

                // Y = c Q K^T + A (A: -lse2 on valid pairs, -inf on masked; with
                // kFoldAdd the accumulator starts at A and K is prescaled by c) and
                // dP - Delta = dO V^T - Delta (rows: queries, columns: this wave's
                // keys; the accumulator starts at -Delta)
                auto score_addend = [&](int m, int bi) {
                    f32x4 add;
                    if (!short_rows && full[bi]) {
                        add = nlse[bi];
                    } else {
                        bool outer_ok = rel[bi];
                        if (!kOF[bi]) {
#pragma unroll
                            for (int a = 0; a < R - 1; ++a)
                                outer_ok = outer_ok && (unsigned)(boc[bi][a] - ilo[m][a]) <=
                                                           (unsigned)ispan[m][a];
                        }
                        // generic rows: slot r is valid when base + r lies in [0, lim)
                        const int base = bin0[bi] + grp * 4 - ilo[m][R - 1];
                        const unsigned lim = outer_ok ? (unsigned)ispan[m][R - 1] + 1u : 0u;
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            add[r] = short_rows ? (outer_ok ? nlse[bi][r] + ain[m][bi][r] : -INFINITY)
                                     : (unsigned)(base + r) < lim ? nlse[bi][r] : -INFINITY;
                    }
                    return add;
                };
                f32x4 sacc[KM][2], pacc[KM][2];
#pragma unroll
                for (int bi = 0; bi < 2; ++bi) {
                    if (rel[bi]) {
                        const int boff = (tp * 2 + bi) * 16 * kRowB;
#pragma unroll
                        for (int st = 0; st < Ops::kKS; ++st) {
                            const x8 qa = ops.rf.read(qs + boff, st);
                            const x8 ga = ops.rf.read(gs + boff, st);
#pragma unroll
                            for (int m = 0; m < KM; ++m) {
                                if (st > 0)
                                    sacc[m][bi] = Tr<T>::mma(qa, kf[m][st], sacc[m][bi]);
                                else if (kFoldAdd && !short_rows && full[bi])
                                    sacc[m][bi] = Tr<T>::mma(qa, kf[m][0], nlse[bi]);  // in place
                                else
                                    sacc[m][bi] = Tr<T>::mma(qa, kf[m][0],
                                                             kFoldAdd ? score_addend(m, bi)
                                                                      : f32x4{0.f, 0.f, 0.f, 0.f});
                                pacc[m][bi] = Tr<T>::mma(ga, vf[m][st], st == 0 ? ndl[bi] : pacc[m][bi]);
                            }
                        }
                    } else {
#pragma unroll
                        for (int m = 0; m < KM; ++m) {
                            const float s0 = kFoldAdd ? -INFINITY : 0.f;
                            sacc[m][bi] = f32x4{s0, s0, s0, s0};
                            pacc[m][bi] = f32x4{0.f, 0.f, 0.f, 0.f};
                        }
                    }
                }

                // P = exp2(Y), dA = P (dP - Delta)
                x8 pf[KM][Ops::kPF], dsf[KM][Ops::kPF];
#pragma unroll
                for (int m = 0; m < KM; ++m) {
                    float p[2][4], ds[2][4];
#pragma unroll
                    for (int bi = 0; bi < 2; ++bi) {
                        f32x4 y = sacc[m][bi];
                        if constexpr (!kFoldAdd) {
                            const f32x4 add = score_addend(m, bi);
#pragma unroll
                            for (int r = 0; r < 4; ++r) y[r] = fmaf(y[r], scale_log2, add[r]);
                        }
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float pv = fast_exp2(y[r]);
                            p[bi][r] = pv;
                            ds[bi][r] = pv * pacc[m][bi][r];
                        }
                    }
                    Ops::pack(pf[m], p);
                    Ops::pack(dsf[m], ds);
                }

                // dV^T += dO^T P and dK^T += Q^T dA (transposed reads of the rows)
#pragma unroll
                for (int d = 0; d < Ops::kDB; ++d) {
                    const x8 ga = ops.cf.read(gs + tp * 32 * kRowB, d, lane);
                    const x8 qa = ops.cf.read(qt, d, lane);
#pragma unroll
                    for (int m = 0; m < KM; ++m) {
                        Ops::accum(dvacc[m], ga, d, pf[m]);
                        Ops::accum(dkacc[m], qa, d, dsf[m]);
                    }
                }
            };
            // the specialised tiles first (the order of tiles does not matter);
            // 16-bit types at D <= 64 only (the compiler fails on the others)
            if constexpr (sizeof(T) == 2 && D <= 64)
                run_tile_kinds<short_rows>(tiles, fullm, ofullm, tile);
            while (tiles) {
                const int tp = __builtin_ctzll(tiles) >> 1;
                tiles &= tiles - 1;
                tile(tp, std::integral_constant<int, 0>{});
            }
        }

        if (s + 1 < nst) {  // (no buffer is reused after the last stage)
            put_floats((s + 1) & 1);
            wait_vmem();
            __syncthreads();
            if (!DIN) {
                delta_pass((s + 1) & 1);
                __syncthreads();
            }
        }
    }

#pragma unroll
    for (int m = 0; m < KM; ++m) {
        if (!kvalid[m]) continue;
        Ops::store(dkg + koff[m], dkacc[m], grp, scale);
        Ops::store(dvg + koff[m], dvacc[m], grp, 1.f);
    }
}

// ---------------------------------------------------------------------------
// the kernel: workgroups [0, nwk) take the dK/dV role, the next g.nwg the dQ
// role (dK/dV first: its workgroups carry more work and start earlier)
// ---------------------------------------------------------------------------
// 16-bit types with D <= 64 are held to 2 waves per SIMD (<= 256 registers),
// and to 3 (<= 168) for rank 1: there the few values that no longer fit are
// spilled outside the tile loop (the dQ role's per-stage state), and the
// third wave hides more of the tile loop's latency (1-D k = 1023 backward:
// -7 %).  Ranks 2 and 3 would spill inside the loop.
// ROLE 0 runs both roles in one grid; ROLE 1 only the dK/dV role (nwk
// workgroups) and ROLE 2 only the dQ role (g.nwg workgroups), each as a
// launch of its own with its own register budget.  ROLE 1 stages 128
// queries per stage at D = 64, double-buffered: about 67 KiB
// of LDS, so two workgroups share a CU, two waves per SIMD whatever the
// registers, and a tighter bound would only spill.  Rank 1 at D = 64 stages
// 64 queries instead (about 34 KiB), which leaves room for the third wave,
// and D = 32 stages 128 (about 34 KiB): four waves at rank 1, three above.
// D = 128 (rank 1, one block per wave) stages 32 queries or keys, so that the
// three waves its registers allow (152-166 VGPRs) fit in LDS.  The single launch
// stages 32 keys in its dQ role too (SBQ in launch_bwd_inst), which takes its LDS
// from 64 to 48 KiB: 1-D 8192 x 16 heads k = 255 fp16 143 -> 128 us, 32768 x 8 k = 127
// 236 -> 212 us.
// Where the split form exists: 16-bit types at D <= 64, and at D = 128 for rank 1 with
// one block per wave.
template <int R, int D, typename T, int M>
constexpr bool has_split() {
    return sizeof(T) == 2 && (D <= 64 || (R == 1 && M == 1));
}

template <int R, int D, typename T, int M, int ROLE>
constexpr int bwd_min_waves() {
    if constexpr (D == 128 && ROLE != 0) return has_split<R, D, T, M>() ? 3 : 1;
    if constexpr (ROLE == 2) return sizeof(T) == 2 && D <= 64 ? (M == 1 ? 5 : 3) : 2;
    if constexpr (ROLE == 1) return R == 1 && D == 64 ? 3 : (D == 32 ? (R == 1 ? 4 : 3) : 2);
    return sizeof(T) == 2 && D <= 64 ? (R == 1 ? 3 : 2) : 1;
}

template <int R, int D, typename T, int M, int SBQ, int SBK, int SHORT, int ROLE>
__global__ __launch_bounds__(256, (bwd_min_waves<R, D, T, M, ROLE>())) void na_bwd_kernel(
    Geo g, int nwk, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
    const T* __restrict__ o, const T* __restrict__ dout, const float* __restrict__ lse,
    const float* __restrict__ ndelta, T* __restrict__ dq, T* __restrict__ dk, T* __restrict__ dv,
    float scale_log2, float scale) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int b = blockIdx.x;
    if constexpr (ROLE == 1) {
        dkdv_role<R, D, T, M, SBK, SHORT, true>(g, b, nwk, smem_raw, q, k, v, o, dout, lse,
                                                   ndelta, dk, dv, scale_log2, scale);
    } else if constexpr (ROLE == 2) {
        dq_role<R, D, T, M, SBQ, SHORT>(g, b, smem_raw, q, k, v, o, dout, lse, dq, scale_log2,
                                           scale);
    } else {
        if (b < nwk)
            dkdv_role<R, D, T, M, SBK, SHORT, false>(g, b, nwk, smem_raw, q, k, v, o, dout,
                                                        lse, nullptr, dk, dv, scale_log2, scale);
        else
            dq_role<R, D, T, M, SBQ, SHORT>(g, b - nwk, smem_raw, q, k, v, o, dout, lse, dq,
                                               scale_log2, scale);
    }
}

// ---------------------------------------------------------------------------
// host-side launch
// ---------------------------------------------------------------------------
// Longest extent along one axis, over every tile and both group lengths of a
// dilated axis, of a workgroup's key halo (inverse = false) or of the box of
// queries attending to its key tile (inverse = true).  Window starts grow by
// at most one per position, so a halo never exceeds min(T, n) + k - 1; an
// inverse box can (every key within k - 1 of the start is attended by query
// 0), so the tiles near a border are evaluated one by one and a single
// interior tile (extent T + k - 1) stands for the rest.  Causal axes have no
// such border growth.
static int max_box_extent(int L, int d, int k, int T, bool causal, bool inverse) {
    int best = 0;
    const int n0 = group_len(L, d, 0);
    for (int n = n0; n >= n0 - 1; --n) {
        if (n < n0 && L % d == 0) break;  // every group has length n0
        // along a causal axis both boxes are [start(first), last] and
        // [first, min(last + k - 1, n - 1)]: never wider than T + k - 1
        if (!inverse || causal) {
            best = std::max(best, std::min(std::min(T, n) + k - 1, n));
            continue;
        }
        const int nt = (n + T - 1) / T;
        const int edge = k / T + 2;  // tiles that can reach within k of a border
        for (int i = 0; i < nt; ++i) {
            if (i > edge && i < nt - edge) continue;
            const int to = i * T, last = std::min(to + T, n) - 1;
            best = std::max(best, inv_hi(last, n, k, false) + 1 - inv_lo(to, n, k, false));
        }
    }
    return best;
}

// 16-token blocks of the largest box with per-axis extents e[]: rows along
// the innermost axis are cut into blocks.
static int box_blocks(const int* e, int rank) {
    int nb = (e[rank - 1] + 15) / 16;
    for (int a = 0; a < rank - 1; ++a) nb *= e[a];
    return nb;
}

// Delta pre-pass of the split backward: nd[row] = -sum_c dO[row, c] O[row, c]
// in fp32, the lanes of a 16-byte segment group sharing a row.
template <typename T, int D>
__global__ __launch_bounds__(256) void na_delta_kernel(const T* __restrict__ o,
                                                       const T* __restrict__ dout,
                                                       float* __restrict__ nd, int64_t rows) {
    using L = Rows<T, D>;
    constexpr int kSegs = L::kSegs;  // lanes per row (a power of two dividing 64)
    const int seg = threadIdx.x % kSegs;
    const int64_t step = (int64_t)gridDim.x * (256 / kSegs);
    for (int64_t row = (int64_t)blockIdx.x * (256 / kSegs) + threadIdx.x / kSegs; row < rows;
         row += step) {
        const i32x4 a = ld16<i32x4>(o + row * D + seg * L::kVec);
        const i32x4 b = ld16<i32x4>(dout + row * D + seg * L::kVec);
        float acc;
        if constexpr (sizeof(T) == 2) {
            using x8 = typename Tr<T>::x8;
            acc = dot8<T>(__builtin_bit_cast(x8, a), __builtin_bit_cast(x8, b), 0.f);
        } else {
            const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
            acc = fmaf(x[3], y[3], fmaf(x[2], y[2], fmaf(x[1], y[1], x[0] * y[0])));
        }
#pragma unroll
        for (int w = 1; w < kSegs; w <<= 1) acc += __shfl_xor(acc, w, kWave);
        if (seg == 0) nd[row] = -acc;
    }
}

// hq / hk: most blocks in any dQ halo / dK-dV query box; a role whose boxes
// all fit in one stage gets a single LDS buffer.
//
// One launch runs both roles (dK/dV workgroups first).  The split form, for
// large 16-bit problems (has_split), runs three launches instead: a Delta
// pre-pass writing -Delta of every query into dq (scratch until the last
// launch overwrites it), the dK/dV role reading it (no O rows, no Delta pass,
// one barrier per stage, stages of SBS blocks), then the dQ role; each role
// runs at the occupancy its own registers and LDS allow.
template <int R, int D, typename T, int M, int SBQ, int SBK>
static hipError_t launch_bwd_sb(const Geo& g0, bool short_rows, bool split, int hq, int hk,
                                const void* q, const void* k, const void* v, const void* o,
                                const float* lse, const void* dout, void* dq, void* dk, void* dv,
                                float scale, hipStream_t stream) {
    using CQ = DqCfg<R, D, T, SBQ>;
    using CK = DkvCfg<R, D, T, SBK>;
    const size_t lds_q = (hq > SBQ ? 2 : 1) * CQ::kBufBytes;
    const size_t lds_k = (hk > SBK ? 2 : 1) * CK::kBufBytes;
    // No register bound asks for more waves per SIMD (workgroups of four
    // waves per CU) than a CU's 160 KiB of LDS holds, with double buffers
    // (stages of 16 blocks are used only when every box fits in one: single).
    constexpr size_t kCuLds = 160 * 1024;
    constexpr size_t kLdsQ = (SBQ >= 16 ? 1 : 2) * CQ::kBufBytes;
    constexpr size_t kLdsK = (SBK >= 16 ? 1 : 2) * CK::kBufBytes;
    static_assert(bwd_min_waves<R, D, T, M, 0>() * (kLdsQ > kLdsK ? kLdsQ : kLdsK) <= kCuLds,
                  "one-launch register bound beyond the LDS occupancy");
    static_assert(bwd_min_waves<R, D, T, M, 2>() * (kLdsQ + (R > 1 && M == 2 ? kMaskTableBytes : 0)) <=
                      kCuLds,
                  "dQ-launch register bound beyond the LDS occupancy");
    const int nwk = (g0.nwg + 7) & ~7;
    auto launch = [&](auto kern, const Geo& g, size_t lds, int grid,
                      const float* nd) -> hipError_t {
        if (lds > 65536) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(4 * kWave), lds, stream, g, nwk,
                           static_cast<const T*>(q), static_cast<const T*>(k),
                           static_cast<const T*>(v), static_cast<const T*>(o),
                           static_cast<const T*>(dout), lse, nd, static_cast<T*>(dq),
                           static_cast<T*>(dk), static_cast<T*>(dv), scale * kLog2e, scale);
        return hipGetLastError();
    };
    if constexpr (has_split<R, D, T, M>()) {
        if (split) {
            // query blocks per stage of the dK/dV launch (see bwd_min_waves)
            constexpr int SBS = D == 32 ? 8 : D == 128 ? 2 : (R == 1 ? 4 : 8);
            const size_t lds_ks = (hk > SBS ? 2 : 1) * DkvCfg<R, D, T, SBS, true>::kBufBytes;
            static_assert(bwd_min_waves<R, D, T, M, 1>() * 2 *
                                  DkvCfg<R, D, T, SBS, true>::kBufBytes <= kCuLds,
                          "dK/dV-launch register bound beyond the LDS occupancy");
            auto kk = na_bwd_kernel<R, D, T, M, SBQ, SBS, 0, 1>;
            auto kq = na_bwd_kernel<R, D, T, M, SBQ, SBK, 0, 2>;
            Geo gq = g0;
            size_t lds_tab = 0;  // the narrow form's tables, behind the stages
            if constexpr (R > 1) {
                if (short_rows) {
                    kk = na_bwd_kernel<R, D, T, M, SBQ, SBS, 1, 1>;
                    kq = na_bwd_kernel<R, D, T, M, SBQ, SBK, 1, 2>;
                }
                if constexpr (M == 2)
                    if (narrow_form(gq, R, hq)) {
                        kq = na_bwd_kernel<R, D, T, M, SBQ, SBK, 2, 2>;
                        gq.tab_off = (int)lds_q;
                        lds_tab = mask_table_bytes(gq, R);
                    }
            }
            float* nd = static_cast<float*>(dq);
            const int64_t rows = (int64_t)g0.BH * g0.N;
            constexpr int kRowsPerBlock = 256 / Rows<T, D>::kSegs;
            const int64_t blocks = std::min<int64_t>((rows + kRowsPerBlock - 1) / kRowsPerBlock,
                                                     int64_t(1) << 18);
            hipLaunchKernelGGL((na_delta_kernel<T, D>), dim3((unsigned)blocks), dim3(256), 0,
                               stream, static_cast<const T*>(o), static_cast<const T*>(dout), nd,
                               rows);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            e = launch(kk, g0, lds_ks, nwk, nd);
            if (e != hipSuccess) return e;
            return launch(kq, gq, lds_q + lds_tab, g0.nwg, nullptr);
        }
    }
    (void)split;
    auto kern = na_bwd_kernel<R, D, T, M, SBQ, SBK, 0, 0>;
    if constexpr (R > 1)  // (1-D boxes have one row: never short)
        if (short_rows) kern = na_bwd_kernel<R, D, T, M, SBQ, SBK, 1, 0>;
    return launch(kern, g0, std::max(lds_q, lds_k), nwk + g0.nwg, nullptr);
}

template <int R, int D, typename T, int M>
static hipError_t launch_bwd_inst(const Geo& g, const void* q, const void* k, const void* v,
                                  const void* o, const float* lse, const void* dout, void* dq,
                                  void* dk, void* dv, float scale, hipStream_t stream) {
    int eq[kMaxRank], ek[kMaxRank];
    for (int a = 0; a < R; ++a) {
        eq[a] = max_box_extent(g.L[a], g.d[a], g.k[a], g.T[a], g.causal[a] != 0, false);
        ek[a] = max_box_extent(g.L[a], g.d[a], g.k[a], g.T[a], g.causal[a] != 0, true);
    }
    const int hq = box_blocks(eq, R), hk = box_blocks(ek, R);
    // rows of every halo (dQ) and query box (dK/dV) hold at most 2 blocks
    const bool short_rows = R > 1 && (eq[R - 1] + 15) / 16 <= 2 && (ek[R - 1] + 15) / 16 <= 2;
    // The split form of 1-D problems needs a large grid: its two more launches and the
    // tail of each cost 10 to 20 us.  One launch / split, us: D = 128 at 1024 workgroups
    // (16384 tokens x 4 heads, k = 600) 116 / 137, at 2048 (8192 x 16, k = 512 causal)
    // 190 / 187, at 4096 (32768 x 8, k = 512) 403 / 384; D = 64 at 256 (2048 x 8, k = 512
    // causal) 17 / 27, at 2048 (32768 x 8, k = 1023) 271 / 277, at 4096 (32768 x 16,
    // k = 1023) 568 / 548; D = 32 at 2048 162 / 169, at 4096 323 / 309.
    constexpr int kSplitGrid = D == 128 ? 2048 : 4096;
    const bool split = g.bwd_split == 2 || (g.bwd_split && (R != 1 || g.nwg >= kSplitGrid));
    // D = 32, 16-bit: boxes of up to 16 blocks are staged whole (one stage)
    if constexpr (sizeof(T) == 2 && D == 32) {
        if (hq <= 16 && hk <= 16)
            return launch_bwd_sb<R, D, T, M, 16, 16>(g, short_rows, split, hq, hk, q, k, v, o, lse,
                                                         dout, dq, dk, dv, scale, stream);
    }
    constexpr int SBQ = sizeof(T) == 4 || (D == 128 && has_split<R, D, T, M>()) ? 2 : 4;
    constexpr int SBK = (sizeof(T) == 4 || D == 128) ? 2 : 4;
    return launch_bwd_sb<R, D, T, M, SBQ, SBK>(g, short_rows, split, hq, hk, q, k, v, o, lse, dout,
                                                   dq, dk, dv, scale, stream);
}

template <int R, int D, typename T>
static hipError_t launch_bwd_m(const Geo& g, int m, const void* q, const void* k, const void* v,
                               const void* o, const float* lse, const void* dout, void* dq,
                               void* dk, void* dv, float scale, hipStream_t s) {
    if (m == 1) return launch_bwd_inst<R, D, T, 1>(g, q, k, v, o, lse, dout, dq, dk, dv, scale, s);
    return launch_bwd_inst<R, D, T, 2>(g, q, k, v, o, lse, dout, dq, dk, dv, scale, s);
}

template <int R, typename T>
static hipError_t launch_bwd_d(const Geo& g, int D, int m, const void* q, const void* k,
                               const void* v, const void* o, const float* lse, const void* dout,
                               void* dq, void* dk, void* dv, float scale, hipStream_t s) {
    switch (D) {
        case 32: return launch_bwd_m<R, 32, T>(g, m, q, k, v, o, lse, dout, dq, dk, dv, scale, s);
        case 64: return launch_bwd_m<R, 64, T>(g, m, q, k, v, o, lse, dout, dq, dk, dv, scale, s);
        case 128: return launch_bwd_m<R, 128, T>(g, m, q, k, v, o, lse, dout, dq, dk, dv, scale, s);
    }
    return hipErrorInvalidValue;
}

template <typename T>
static hipError_t launch_bwd_r(const Geo& g, int rank, int D, int m, const void* q, const void* k,
                               const void* v, const void* o, const float* lse, const void* dout,
                               void* dq, void* dk, void* dv, float scale, hipStream_t s) {
    switch (rank) {
        case 1: return launch_bwd_d<1, T>(g, D, m, q, k, v, o, lse, dout, dq, dk, dv, scale, s);
        case 2: return launch_bwd_d<2, T>(g, D, m, q, k, v, o, lse, dout, dq, dk, dv, scale, s);
        case 3: return launch_bwd_d<3, T>(g, D, m, q, k, v, o, lse, dout, dq, dk, dv, scale, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_backward(const Geo& g, int rank, int D, int dtype, int m, const void* q,
                           const void* k, const void* v, const void* o, const float* lse,
                           const void* dout, void* dq, void* dk, void* dv, float scale,
                           hipStream_t s) {
    switch (dtype) {
        case 0: return launch_bwd_r<float>(g, rank, D, m, q, k, v, o, lse, dout, dq, dk, dv, scale, s);
        case 1: return launch_bwd_r<_Float16>(g, rank, D, m, q, k, v, o, lse, dout, dq, dk, dv, scale, s);
        case 2: return launch_bwd_r<__bf16>(g, rank, D, m, q, k, v, o, lse, dout, dq, dk, dv, scale, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace na
