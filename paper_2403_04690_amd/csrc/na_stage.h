// na_stage.h -- direct global -> LDS staging of token rows, the swizzled LDS
// row layout the matrix-core fragments are read from, and the halo geometry
// those rows come from.
#pragma once

#include <type_traits>

#include "na_common.h"

namespace na {

// A box of tokens in group coordinates, [lo, lo + E) per axis, cut into rows
// along the innermost axis and each row into 16-token blocks (rows are padded
// to a multiple of 16; padding slots hold a stand-in token and are always
// masked).
template <int R>
struct Box {
    int lo[kMaxRank];
    int E[kMaxRank];
    int nbr;  // blocks per row
    int nb;   // total blocks
    FastDiv fd_nbr;
    FastDiv fd_E[kMaxRank];
    // token (within the (batch, head) slice) of the box's first position, and
    // the token distance of one step along each axis in group coordinates
    int tok_lo;
    int tstride[kMaxRank];

    // Block counts and divisors; gc[] is the dilation group of each axis.
    __device__ __forceinline__ void finish(const Geo& g, const int* gc) {
        nbr = (E[R - 1] + 15) >> 4;
        nb = nbr;
#pragma unroll
        for (int a = 0; a < R - 1; ++a) nb *= E[a];
        if constexpr (R > 1) fd_nbr.init(nbr);  // (1-D boxes are one row)
#pragma unroll
        for (int a = 1; a < R - 1; ++a) fd_E[a].init(E[a]);
        tok_lo = 0;
#pragma unroll
        for (int a = 0; a < R; ++a) {
            tstride[a] = g.d[a] * g.ts[a];
            tok_lo += (gc[a] + g.d[a] * lo[a]) * g.ts[a];
        }
    }

    // Outer coordinates (relative to lo) and first inner coordinate of block b
    // (blocks past the box get coordinates past it too).
    __device__ __forceinline__ void block_coords(int b, int* oc, int& inner0) const {
        if constexpr (R == 1) {  // one row: no division
            inner0 = b * 16;
            return;
        }
        int row = fd_nbr.div(b);
        inner0 = (b - row * nbr) * 16;
#pragma unroll
        for (int a = R - 2; a >= 1; --a) {
            const int nx = fd_E[a].div(row);
            oc[a] = row - nx * E[a];
            row = nx;
        }
        if (R >= 2) oc[0] = row;
    }

    // The same for staging, where blocks past the end stand for the last one.
    __device__ __forceinline__ int block_first(int b, int& valid) const {
        return block_token(b < nb ? b : nb - 1, valid);
    }

    // Token (within the (batch, head) slice) of slot 0 of block b, and how many
    // slots of the block hold a token of the box (0 for blocks past the end).
    // Slot j of the block is token + j * g.d[R-1].
    __device__ __forceinline__ int block_token(int b, int& valid) const {
        int oc[kMaxRank];
        int inner0;
        block_coords(b, oc, inner0);
        oc[R - 1] = inner0;
        const int left = E[R - 1] - inner0;
        valid = b < nb ? (left > 16 ? 16 : left) : 0;
        int tok = tok_lo;
#pragma unroll
        for (int a = 0; a < R; ++a) tok += oc[a] * tstride[a];
        return tok;
    }
};

// Per-wave block tests against a box of the other side: a block is relevant
// when it intersects [lo, hi) on every axis, and full when it lies inside
// [flo, fhi) on every axis (all its pairs with the wave's tokens are valid).
// Each range is kept as its start and its length (0 when empty), so that
// every test is one unsigned comparison.
template <int R>
struct WaveRange {
    int lo[kMaxRank], rlen[kMaxRank], flo[kMaxRank], flen[kMaxRank];
    int ilen;  // inner axis: blocks [i0, i0 + 16) meeting [lo, hi) have i0 - lo + 15 < ilen
    int iflen;  // inner axis: blocks inside [flo, fhi) have i0 - flo < iflen

    // Axis a: relevant range [lo_, hi_) (never empty), full range [flo_, fhi_).
    __device__ __forceinline__ void set(int a, int lo_, int hi_, int flo_, int fhi_) {
        lo[a] = lo_;
        rlen[a] = hi_ - lo_;
        flo[a] = flo_;
        flen[a] = fhi_ > flo_ ? fhi_ - flo_ : 0;
        if (a == R - 1) {
            ilen = hi_ - lo_ + 15;
            iflen = fhi_ - flo_ > 15 ? fhi_ - flo_ - 15 : 0;
        }
    }

    // rel: block b meets some window of the wave's queries; full: it lies
    // inside all of them; outer_full: inside all of them along the outer axes
    // (the innermost axis not tested).
    __device__ __forceinline__ void test(const Box<R>& box, int b, int* oc, int& inner0, bool& rel,
                                         bool& full, bool& outer_full) const {
        box.block_coords(b, oc, inner0);
        const bool in_box = b < box.nb;
        bool r_ = in_box, f_ = in_box;
#pragma unroll
        for (int a = 0; a < R - 1; ++a) {
            r_ = r_ & ((unsigned)(oc[a] - lo[a]) < (unsigned)rlen[a]);
            f_ = f_ & ((unsigned)(oc[a] - flo[a]) < (unsigned)flen[a]);
        }
        outer_full = f_;
        rel = r_ & ((unsigned)(inner0 - lo[R - 1] + 15) < (unsigned)ilen);
        full = f_ & ((unsigned)(inner0 - flo[R - 1]) < (unsigned)iflen);
    }
    __device__ __forceinline__ void test(const Box<R>& box, int b, int* oc, int& inner0, bool& rel,
                                         bool& full) const {
        bool outer_full;
        test(box, b, oc, inner0, rel, full, outer_full);
    }
};

// A wave's block tests taken 64 blocks at a time, one block per lane, instead
// of once per stage: a stage of SB blocks (SB divides 64) reads its bits from
// the chunk's masks, and a block's coordinates back from the lane that tested
// it.  Stages of 16 blocks or more (a whole halo, staged once) are tested
// stage by stage, with no chunk bookkeeping.
template <int R, int SB>
struct ChunkTests {
    static_assert(64 % SB == 0, "stages tile the 64-block chunks");
    static constexpr int kChunk = SB >= 16 ? SB : 64;  // blocks tested at a time
    static constexpr uint64_t kSel = SB == 64 ? ~0ull : (1ull << SB) - 1;
    int loc[kMaxRank], lin0;  // this lane's block: outer coordinates, first inner coordinate
    uint64_t rel, full, ofull;  // the chunk's blocks: relevant, full, full along the outer axes
    int j0;  // the stage's first block within the chunk

    // Stage s (stages are visited in order from 0).
    __device__ __forceinline__ void stage(const WaveRange<R>& wr, const Box<R>& box, int s,
                                          int lane) {
        j0 = (s * SB) & (kChunk - 1);
        if (j0 == 0) {
            bool r, f, o;
            wr.test(box, s * SB + lane, loc, lin0, r, f, o);
            rel = __builtin_amdgcn_ballot_w64(r);
            full = __builtin_amdgcn_ballot_w64(f);
            ofull = __builtin_amdgcn_ballot_w64(o);
        }
    }
    // bit j: block s * SB + j of the stage
    __device__ __forceinline__ uint64_t rel_bits() const { return (rel >> j0) & kSel; }
    __device__ __forceinline__ uint64_t full_bits() const { return (full >> j0) & kSel; }
    __device__ __forceinline__ uint64_t ofull_bits() const { return (ofull >> j0) & kSel; }
    // first inner coordinate and outer coordinate a of the stage's block j
    __device__ __forceinline__ int inner0(int j) const {
        return __builtin_amdgcn_readlane(lin0, j0 + j);
    }
    __device__ __forceinline__ int outer(int j, int a) const {
        return __builtin_amdgcn_readlane(loc[a], j0 + j);
    }
};

// Runs the tiles (bit 2 tp of `tiles`: block pair tp) whose kind allows a
// specialised body, removing them from `tiles`, which keeps the general ones
// (kind 0).  Kinds: 1 both blocks full (rows of more than two blocks); for
// short rows, 2 both blocks full along the outer axes, 3 / 4 only the first /
// second.  The order of tiles is free in the online softmax and in the sums.
template <bool SHORT_ROWS, typename F>
__device__ __forceinline__ void run_tile_kinds(uint64_t& tiles, uint64_t full, uint64_t ofull,
                                               F&& tile) {
    auto run = [&](uint64_t set, auto kind) {
        while (set) {
            const int tp = __builtin_ctzll(set) >> 1;
            set &= set - 1;
            tile(tp, kind);
        }
    };
    if constexpr (SHORT_ROWS) {
        const uint64_t of0 = ofull & 0x5555555555555555ull;
        const uint64_t of1 = (ofull >> 1) & 0x5555555555555555ull;
        run(tiles & of0 & of1, std::integral_constant<int, 2>{});
        run(tiles & of0 & ~of1, std::integral_constant<int, 3>{});
        run(tiles & ~of0 & of1, std::integral_constant<int, 4>{});
        tiles &= ~(of0 | of1);
    } else {
        const uint64_t pairs = full & (full >> 1) & 0x5555555555555555ull;
        run(tiles & pairs, std::integral_constant<int, 1>{});
        tiles &= ~pairs;
    }
}

// ---------------------------------------------------------------------------
// Outer-axis masks as a matrix product (32x32x16 kernels, short rows).  Along an axis the
// box positions a wave needs, counted from the first, fall into three runs: the
// first nlow are missing from the windows of the wave's later tokens, those from
// nfirst on (past the first token's window) from the earlier ones', and what lies
// between belongs to all.  With one slot per position of the outer runs (15 at most,
// checked on the host), a box row's operand has kMaskRow in the slots its coordinates
// fall into, a token's operand kMaskTok in the slots it misses, and their product is
// what to add to the pair's score: 0, or -inf, to which the product of the two bf16
// values of largest magnitude overflows (1.1e77).  Slot 15 marks rows that no token of
// the wave needs.  One 32x32x16 bf16 step per tile (32 cycles of the matrix core) takes
// the place of two compares per axis, row and lane and a select per score.
// ---------------------------------------------------------------------------
constexpr unsigned kMaskRow = 0x7f7fu, kMaskTok = 0xff7fu;  // bf16 3.39e38, -3.39e38

template <int R>
struct MaskRows {
    int lo[kMaxRank], len[kMaxRank], nlow[kMaxRank], nfirst[kMaxRank], slot[kMaxRank];

    // Axis a: the wave needs positions [lo, lo + len) of the box; nlow and nfirst as
    // above.
    NA_HD void set(int a, int lo_, int len_, int nlow_, int nfirst_) {
        lo[a] = lo_;
        len[a] = len_;
        nlow[a] = nlow_;
        nfirst[a] = nfirst_;
        slot[a] = a == 0 ? 0 : slot[a - 1] + nlow[a - 1] + len[a - 1] - nfirst[a - 1];
    }

    // Slots of the box row at outer coordinates oc (relative to the box).
    NA_HD unsigned row_slots(const int* oc) const {
        unsigned m = 0;
#pragma unroll
        for (int a = 0; a < R - 1; ++a) {
            const int x = oc[a] - lo[a];
            if ((unsigned)x >= (unsigned)len[a]) {
                m |= 1u << 15;
            } else {
                if (x < nlow[a]) m |= 1u << (slot[a] + x);
                if (x >= nfirst[a]) m |= 1u << (slot[a] + nlow[a] + x - nfirst[a]);
            }
        }
        return m;
    }

    // Table `idx` of the workgroup: 16 bf16 slots per block of the box, as the waves
    // at one outer position need them; blocks past the box are marked.
    __device__ __forceinline__ void write_table(const Geo& g, const Box<R>& box,
                                                unsigned char* tab, int idx, int lane) const {
        tab += idx * g.tab_rows * 32;
        for (int row = lane; row < g.tab_rows; row += kWave) {
            int oc[kMaxRank], inner0;
            box.block_coords(row, oc, inner0);
            const unsigned m = row < box.nb ? row_slots(oc) : 1u << 15;
            st16<i32x4>(tab + row * 32, expand(m, kMaskRow));
            st16<i32x4>(tab + row * 32 + 16, expand(m >> 8, kMaskRow));
        }
    }

    // Mask operand of a token, slots 8 grp .. 8 grp + 7: start with operand(), then
    // axis by axis the token's own range [first, last] of box positions.
    NA_HD static unsigned operand() { return 1u << 15; }
    NA_HD unsigned operand(unsigned m, int a, int first, int last) const {
        const int nh = len[a] - nfirst[a];
        const int miss = min(max(first - lo[a], 0), nlow[a]);           // first positions missed
        const int have = min(max(last + 1 - lo[a] - nfirst[a], 0), nh);  // last ones reached
        m |= ((1u << miss) - 1u) << slot[a];
        m |= (((1u << nh) - 1u) & ~((1u << have) - 1u)) << (slot[a] + nlow[a]);
        return m;
    }
    __device__ __forceinline__ static i32x4 pack_operand(unsigned m, int grp) {
        return expand(m >> (8 * grp), kMaskTok);
    }

  private:
    // bits 0..7 of m as eight 16-bit values: v where set
    __device__ __forceinline__ static i32x4 expand(unsigned m, unsigned v) {
        i32x4 r;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            r[j] = (int)(((m >> (2 * j)) & 1u ? v : 0u) | ((m >> (2 * j + 1)) & 1u ? v << 16 : 0u));
        return r;
    }
};

// ---------------------------------------------------------------------------
// LDS rows: D elements of T per token, row-major and unpadded, cut into
// 16-byte segments; segment s of row r is stored at position s ^ swz(r).
// The swizzle is linear in the low four row bits and was chosen so that both
// reads of 16-row fragments below are free of bank conflicts:
//   * 16-byte reads of one segment down 16 consecutive rows (MFMA operands
//     whose contraction runs along D);
//   * transposed 8-byte reads of 4 consecutive rows x 2 adjacent segments per
//     16 lanes (operands whose contraction runs along the tokens).  The LDS
//     serves 256 bytes a cycle, lane groups 0 and 2, then 1 and 3 (counted:
//     with rows r and r + 8 on the same pair of segments a third of all LDS
//     cycles were conflicts, with those of this swizzle none).  Conflict-free
//     reads took the dK/dV launch of the 1-D k = 1023 backward from 352 to
//     336 us and its dQ launch from 258 to 244 us.
// The narrow form's reads (RowFrag32, ColFrag32) are not: their eight-column rows start
// anywhere in a block, and rows 16 apart share a swizzle (counted on 16 x 64 x 64, 7^3 fp16:
// 31 % of the LDS cycles of the forward and 38 % of dQ's are conflicts).
// ---------------------------------------------------------------------------
template <typename T, int D>
struct Rows {
    static constexpr int kSegs = D * (int)sizeof(T) / 16;  // segments per row
    static constexpr int kRowBytes = D * (int)sizeof(T);
    static constexpr int kVec = 16 / (int)sizeof(T);  // elements per segment
    static_assert(kSegs == 4 || kSegs == 8 || kSegs == 16 || kSegs == 32, "segments per row");

    __device__ __forceinline__ static constexpr int swz(int r) {
        constexpr int c0 = kSegs == 4 ? 0 : kSegs == 32 ? 1 : 2;
        constexpr int c1 = kSegs == 4 ? 2 : kSegs == 32 ? 2 : 4;
        constexpr int c2 = kSegs == 4 ? 3 : kSegs == 8 ? 3 : kSegs == 16 ? 9 : 4;
        constexpr int c3 = kSegs >= 16 ? 8 : 2;
        return (-(r & 1) & c0) ^ (-((r >> 1) & 1) & c1) ^ (-((r >> 2) & 1) & c2) ^
               (-((r >> 3) & 1) & c3);
    }
    // byte offset of logical segment s of row r
    __device__ __forceinline__ static int off(int r, int s) {
        return r * kRowBytes + ((s ^ swz(r)) << 4);
    }
};

// Waits until this wave's outstanding vector memory operations (including
// direct-to-LDS loads) have completed.
__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

typedef __attribute__((address_space(3))) void lds_void;

// x, with its value hidden from the optimiser.
__device__ __forceinline__ int opaque(int x) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(x));
#endif
    return x;
}

// Stages ROWS token rows into an LDS tile with 16-byte direct-to-LDS loads
// (no register round trip): wave instruction t writes the tile's 16-byte
// positions [64 t, 64 t + 64), i.e. 64 / kSegs rows of one 16-row block, and
// lane l loads the segment that the swizzle puts at position 64 t + l.
// Rows past the end of a box row are replaced by the first row of their block,
// blocks past the end of the box by its last one (data of the box that the masks
// exclude).  Several tensors with the same rows share one
// set of per-lane source offsets.  With BLOCKWISE, when a block takes several
// instructions, wave w of the W takes the consecutive ones [w * kPerWave,
// (w + 1) * kPerWave), so that one block decode serves all of a block's
// instructions (2-D / 3-D boxes, whose decode has divisions); otherwise the
// waves take the instructions round-robin (measured faster for 1-D boxes).
// How a load is addressed:
//   kByLane   scalar slice base + 32-bit lane offset (16-bit types, whose slices are
//             below 2^32 bytes): one base register pair for every load;
//   kByBlock  scalar base per block + lane offset: no vector add per load, but a
//             register pair each.  fp32, whose lane offsets may exceed 32 bits, and the
//             3-D backward at D = 128, measured by block / by lane 16 x 64 x 64, 7^3
//             1664 / 1735 us, 8 x 96 x 96, 5 x 7 x 7 1200 / 1295.  Elsewhere by lane is the
//             faster or within 1 %: 1-D k = 255 causal bf16 D = 64 forward 23.7 / 22.8,
//             3-D 9 x 9 x 5 bf16 D = 64 forward 191 / 186, 2-D 128 x 128 k = 13 d = 2 bf16
//             D = 32 backward 103.4 / 97.6;
//   kUntracked  as kByLane, in inline assembly (load_lds below).
enum class Addr { kByLane, kByBlock, kUntracked };

template <typename T, int D, int ROWS, int W = 4, bool BLOCKWISE = false,
          Addr ADDR = (sizeof(T) == 2 ? Addr::kByLane : Addr::kByBlock)>
struct DirectRows {
    using L = Rows<T, D>;
    static constexpr int kRowsPerInstr = 64 / L::kSegs;
    static constexpr int kInstr = ROWS * L::kSegs / 64;  // wave instructions per tensor
    static constexpr int kPerWave = (kInstr + W - 1) / W;
    // wave instruction u of this wave
    __device__ __forceinline__ static int instr(int wave, int u) {
        return BLOCKWISE && kRowsPerInstr < 16 ? wave * kPerWave + u : wave + W * u;
    }
    static_assert(ROWS % 16 == 0 && kInstr >= 1, "whole blocks per stage");
    // A block costs its first token (uniform, on the scalar unit).
    // Offsets count bytes, fp32 ones elements (32 bits hold either).
    static constexpr int kUnit = sizeof(T) == 2 ? 1 : 4;
    static constexpr uint32_t kRowUnits = L::kRowBytes / kUnit;
    static_assert(ADDR == Addr::kByBlock || sizeof(T) == 2, "32-bit byte offsets");
    uint32_t base[kPerWave];  // kByBlock: the stage's blocks' first tokens within the slice
    uint32_t cur[kPerWave];   // this lane's segment, from there; else within the slice

    // Rows of stage-local blocks b0, b0 + 1, ... of the box; tstep is the token
    // distance between consecutive slots of a block.  AFRESH forms the lane's part
    // for each stage again: kernels without registers to spare would spill it in
    // the tile loop.
    template <bool AFRESH, int R>
    __device__ __forceinline__ void compute(const Box<R>& box, int b0, int tstep, int wave,
                                            int lane) {
        if (AFRESH) lane = opaque(lane);
        const uint32_t rstep = (uint32_t)tstep * kRowUnits;
        // (round-robin instructions of a wave cover the same rows of their blocks when
        // W instructions make whole blocks)
        constexpr int kKinds =
            (BLOCKWISE && kRowsPerInstr < 16) || W * kRowsPerInstr % 16 != 0 ? kPerWave : 1;
        int row[kKinds];
        uint32_t seg0[kKinds], seg[kKinds];
#pragma unroll
        for (int u = 0; u < kKinds; ++u) {
            row[u] = ((instr(wave, u) * kRowsPerInstr) & 15) + lane / L::kSegs;
            seg0[u] = (uint32_t)(((lane % L::kSegs) ^ L::swz(row[u])) * (16 / kUnit));
            seg[u] = (uint32_t)row[u] * rstep + seg0[u];
        }
#pragma unroll
        for (int u = 0; u < kPerWave; ++u) {
            const int t = instr(wave, u);
            if (t < kInstr) {
                int valid;
                const int tok0 = box.block_first(b0 + ((t * kRowsPerInstr) >> 4), valid);
                const int k = kKinds == 1 ? 0 : u;
                base[u] = (uint32_t)tok0 * kRowUnits;
                cur[u] = row[k] < valid ? seg[k] : seg0[k];
                if (ADDR != Addr::kByBlock) cur[u] += base[u];
            }
        }
    }

    __device__ __forceinline__ void issue(const T* slice, unsigned char* tile, int wave) const {
#pragma unroll
        for (int u = 0; u < kPerWave; ++u) {
            const int t = instr(wave, u);
            if (t >= kInstr) continue;
            const unsigned char* src = reinterpret_cast<const unsigned char*>(slice);
            if (ADDR == Addr::kByBlock) src += (size_t)base[u] * kUnit;
            if constexpr (ADDR == Addr::kUntracked)
                load_lds(src, cur[u], tile + t * 1024);
            else
                __builtin_amdgcn_global_load_lds(static_cast<const void*>(src + (size_t)cur[u] * kUnit),
                                                 (lds_void*)(tile + t * 1024), 16, 0, 0);
        }
    }

    // 16 bytes per lane from base + off to consecutive LDS positions from dst, in inline
    // assembly: the compiler cannot tell the stage buffers apart and waits,
    // before a transposed LDS read of the current stage, for the next stage's loads too.
    // It has no output registers; every wait for it is wait_vmem().  (m0 is reserved: the
    // compiler sets it right where it needs it, so writing it here disturbs nothing.)
    // A vector memory instruction may read a scalar register five wait states after a
    // vector instruction wrote it (a value read back from a lane: a first lane's, a spilled
    // one), and one that uses m0 one after its write; the compiler keeps neither distance
    // inside assembly, so the block does: the move and four idle states.
    // Used by the 2-D backwards of one block per wave at D <= 64, tracked / untracked, us:
    // 56 x 56 k = 7 D = 32 fp16, 128 slices 61.6 / 59.7, 128 x 128 k = 13 d = 2 D = 64 fp16
    // 159.2 / 156.6, 96 x 96 k = 21 d = 2 D = 64 bf16 104.9 / 102.2 (56 x 56 k = 7 D = 64
    // bf16 loses, 40.9 / 41.6).  Elsewhere it gains nothing or loses: 1-D k = 1023 forward
    // fp16 166 / 166, bf16 166 / 170, 3-D 7^3 backward bf16 565 / 582.
    __device__ __forceinline__ static void load_lds(const unsigned char* base, uint32_t off,
                                                    unsigned char* dst) {
#if defined(__HIP_DEVICE_COMPILE__)
        const unsigned m0 = (unsigned)(size_t)(lds_void*)dst;
        static_assert(kUnit == 1, "16-bit types");
        asm volatile(
            "s_mov_b32 m0, %2\n\t"
            "s_nop 3\n\t"
            "global_load_lds_dwordx4 %0, %1"
            :
            : "v"(off), "s"(base), "s"(m0)
            : "memory");
#endif
    }
};

// 16-byte and 8-byte LDS reads.
__device__ __forceinline__ i32x4 lds16(const unsigned char* p) {
    return *reinterpret_cast<const i32x4*>(p);
}

// Operand fragment of 16 rows x 32 contraction slots whose contraction runs
// along D (MFMA A/B layout: lane l holds row l % 16, slots 8 (l / 16) .. +7
// = elements st * 32 + 8 (l / 16) .. +7 of its row).  rowoff[] is from
// frag_offsets(); tile points at the first of the 16 rows.
template <typename T, int D>
struct RowFrag {
    using L = Rows<T, D>;
    static constexpr int kKS = D / 32;
    static constexpr int kN = sizeof(T) == 2 ? 1 : 2;  // 16-byte reads per fragment
    int off[kKS][kN];
    __device__ __forceinline__ void init(int lane) {
        const int r = lane & 15, g = lane >> 4;
#pragma unroll
        for (int st = 0; st < kKS; ++st)
#pragma unroll
            for (int n = 0; n < kN; ++n) off[st][n] = L::off(r, (st * 32 + g * 8) / L::kVec + n);
    }
    __device__ __forceinline__ typename Tr<T>::x8 read(const unsigned char* tile, int st) const {
        using x8 = typename Tr<T>::x8;
        if constexpr (sizeof(T) == 2) {
            return __builtin_bit_cast(x8, lds16(tile + off[st][0]));
        } else {
            const f32x4 a = __builtin_bit_cast(f32x4, lds16(tile + off[st][0]));
            const f32x4 b = __builtin_bit_cast(f32x4, lds16(tile + off[st][1]));
            return x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        }
    }
};

// Transposed operand fragment: 16 columns d = db*16 + (l % 16) of D against
// 32 token slots, slot j of lane l holding token row
//   4 (l / 16) + j          (j < 4)   and   16 + 4 (l / 16) + j - 4   (j >= 4)
// of a 32-row tile -- the token order of a result tile of two 16-token
// blocks (result lane l holds rows 4 (l / 16) .. +3 of each block), so a
// probability or gradient tile feeds the next product without a shuffle.
// 16-bit types use the gfx950 transposed LDS read (each 16-lane group
// gathers 4 rows x 16 columns); fp32 reads the eight values one by one.
template <typename T, int D>
struct ColFrag {
    using L = Rows<T, D>;
    static constexpr int kDB = D / 16;
    int off[kDB];
    __device__ __forceinline__ void init(int lane) {
        const int g = lane >> 4, i = lane & 15;
        if constexpr (sizeof(T) == 2) {
            // lane 16g + 4s + q supplies row 4g + s, columns db*16 + 4q .. +3
            const int r = 4 * g + (i >> 2), q = i & 3;
#pragma unroll
            for (int db = 0; db < kDB; ++db)
                off[db] = L::off(r, (db * 16 + 4 * q) / L::kVec) + (q & 1) * 8;
        } else {
#pragma unroll
            for (int db = 0; db < kDB; ++db) off[db] = 0;
        }
    }
    __device__ __forceinline__ typename Tr<T>::x8 read(const unsigned char* tile, int db,
                                                       int lane) const {
        using x8 = typename Tr<T>::x8;
        if constexpr (sizeof(T) == 2) {
            typedef short s16x4 __attribute__((ext_vector_type(4)));
            typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
            const i32x2 a = __builtin_bit_cast(
                i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tile + off[db])));
            const i32x2 b = __builtin_bit_cast(
                i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                           (lds_s16x4*)(tile + 16 * L::kRowBytes + off[db])));
            return __builtin_bit_cast(x8, i32x4{a[0], a[1], b[0], b[1]});
        } else {
            const int g = lane >> 4, d = db * 16 + (lane & 15);
            x8 v;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int r = (j < 4 ? 0 : 16) + 4 * g + (j & 3);
                v[j] = *reinterpret_cast<const float*>(tile + L::off(r, d / L::kVec) +
                                                       (d % L::kVec) * 4);
            }
            return v;
        }
    }
};

// The same two reads for the 32x32x16 steps of the narrow form (16-bit types).  The 32
// rows of a tile are eight columns (col0 .. col0 + 7) of four consecutive 16-row blocks:
// row r is staged row 16 (r / 8) + col0 + r % 8.
// Row fragment st: lane l holds row l % 32, elements st * 16 + 8 (l / 32) .. +7.
// One offset per lane: fragment st's segment is that of fragment 0 with bits of
// st flipped in, (2 st + l / 32) ^ swz = 2 st ^ (l / 32 ^ swz), so its offset is
// formed where it is used (kept apart they would cost three more registers).
template <typename T, int D>
struct RowFrag32 {
    static_assert(sizeof(T) == 2, "16-bit types");
    using L = Rows<T, D>;
    static constexpr int kKS = D / 16;
    int off;
    __device__ __forceinline__ void init(int lane, int col0) {
        const int r = lane & 31;
        off = L::off((r >> 3) * 16 + col0 + (r & 7), lane >> 5);
    }
    __device__ __forceinline__ void read(const unsigned char* tile,
                                         typename Tr<T>::x8 (&f)[kKS]) const {
        const int o = opaque(off);  // (not hoisted out of the tile loop)
#pragma unroll
        for (int st = 0; st < kKS; ++st)
            f[st] = __builtin_bit_cast(typename Tr<T>::x8, lds16(tile + (o ^ (st << 5))));
    }
};

// Transposed fragment of columns d = db * 32 + l % 32 against rows 16 bi .. +15 of the
// tile: slot j of lane l is row 4 (l / 32) + j (j < 4) or 8 + 4 (l / 32) + j - 4
// (j >= 4) of them, the rows that lane holds of a 32x32 result tile, so such a tile
// feeds the next product without a shuffle.
// (Again one offset per lane: column block db flips segment bits, and slots 4 .. 7 lie
// in the next 16-row block, with the same swizzle.)
template <typename T, int D>
struct ColFrag32 {
    static_assert(sizeof(T) == 2, "16-bit types");
    using L = Rows<T, D>;
    static constexpr int kDB = D / 32;
    static constexpr int kBlk = 32 * L::kRowBytes;  // from bi = 0 to bi = 1
    static constexpr int kSec = 16 * L::kRowBytes;  // to slots 4 .. 7
    int off;
    __device__ __forceinline__ void init(int lane, int col0) {
        // 16-lane group (2 h + e): rows 4 h + s, columns db * 32 + e * 16 + 4 q .. +3
        const int h = lane >> 5, e = (lane >> 4) & 1, i = lane & 15;
        const int r = col0 + 4 * h + (i >> 2), q = i & 3;
        off = L::off(r, (e * 16 + 4 * q) / 8) + (q & 1) * 8;
    }
    // Every fragment of the tile, (db, bi) at 2 db + bi, and the wait for them, in
    // inline-assembly blocks: the compiler takes the transposed read for an access
    // to any staged row and would wait before it for every direct-to-LDS load in
    // flight, the next stage's included.
    // The rows start EXTRA bytes past `tile`.
    template <int EXTRA>
    __device__ __forceinline__ void read(const unsigned char* tile,
                                         typename Tr<T>::x8 (&f)[2 * kDB]) const {
        static_assert(EXTRA + kBlk + kSec < 65536, "immediate offsets");
#if defined(__HIP_DEVICE_COMPILE__)
        typedef const __attribute__((address_space(3))) unsigned char lds_u8;
        const int o = opaque(off);  // (not hoisted out of the tile loop)
        if constexpr (kDB == 1) {
            i32x2 r[4];
            asm volatile(
                "ds_read_b64_tr_b16 %0, %4 offset:%5\n\t"
                "ds_read_b64_tr_b16 %1, %4 offset:%6\n\t"
                "ds_read_b64_tr_b16 %2, %4 offset:%7\n\t"
                "ds_read_b64_tr_b16 %3, %4 offset:%8\n\t"
                "s_waitcnt lgkmcnt(0)"
                : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
                : "v"((lds_u8*)(tile + o)), "n"(EXTRA), "n"(EXTRA + kSec), "n"(EXTRA + kBlk),
                  "n"(EXTRA + kBlk + kSec)
                : "memory");
#pragma unroll
            for (int i = 0; i < 2; ++i) f[i] = cat(r[2 * i], r[2 * i + 1]);
        } else {
#pragma unroll
            for (int db = 0; db < kDB; db += 2) {
                const int o0 = o ^ (db << 6), o1 = o ^ ((db + 1) << 6);
                i32x2 r[8];
                asm volatile(
                    "ds_read_b64_tr_b16 %0, %8 offset:%10\n\t"
                    "ds_read_b64_tr_b16 %1, %8 offset:%11\n\t"
                    "ds_read_b64_tr_b16 %4, %9 offset:%10\n\t"
                    "ds_read_b64_tr_b16 %5, %9 offset:%11\n\t"
                    "ds_read_b64_tr_b16 %2, %8 offset:%12\n\t"
                    "ds_read_b64_tr_b16 %3, %8 offset:%13\n\t"
                    "ds_read_b64_tr_b16 %6, %9 offset:%12\n\t"
                    "ds_read_b64_tr_b16 %7, %9 offset:%13\n\t"
                    "s_waitcnt lgkmcnt(0)"
                    : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]),
                      "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
                    : "v"((lds_u8*)(tile + o0)), "v"((lds_u8*)(tile + o1)), "n"(EXTRA),
                      "n"(EXTRA + kSec), "n"(EXTRA + kBlk), "n"(EXTRA + kBlk + kSec)
                    : "memory");
#pragma unroll
                for (int i = 0; i < 4; ++i) f[2 * db + i] = cat(r[2 * i], r[2 * i + 1]);
            }
        }
#endif
    }

  private:
    __device__ __forceinline__ static typename Tr<T>::x8 cat(i32x2 a, i32x2 b) {
        return __builtin_bit_cast(typename Tr<T>::x8, i32x4{a[0], a[1], b[0], b[1]});
    }
};

// The fragments and products of one tile, 32 staged rows (two 16-row blocks)
// against a block of Q tokens held in registers, by Q.  kF fragments cover the
// 32 rows in either orientation.
//   rows(): the tile's rows as A operand, contraction along D;
//   cols(): transposed, contraction along the 32 rows;
//   score(): s += a row fragment x the register fragments b[];
//   accum(): acc[] += a transposed fragment x p, p the tile's values rounded to T.
template <typename T, int D, int Q>
struct TileOps;

template <typename T, int D>
struct TileOps<T, D, 16> {
    using x8 = typename Tr<T>::x8;
    using Acc = f32x4;
    static constexpr int kStep = 32, kKS = D / 32, kDB = D / 16, kF = D / 16, kPF = 1;
    RowFrag<T, D> rf;
    ColFrag<T, D> cf;
    int lane;
    __device__ __forceinline__ void init(int lane_, int = 0) {
        lane = lane_;
        rf.init(lane_);
        cf.init(lane_);
    }
    // fragment n = bi * kKS + st
    __device__ __forceinline__ void rows(const unsigned char* tile, x8 (&f)[kF]) const {
#pragma unroll
        for (int n = 0; n < kF; ++n)
            f[n] = rf.read(tile + (n / kKS) * 16 * Rows<T, D>::kRowBytes, n % kKS);
    }
    template <int EXTRA = 0>
    __device__ __forceinline__ void cols(const unsigned char* tile, x8 (&f)[kF]) const {
#pragma unroll
        for (int n = 0; n < kF; ++n) f[n] = cf.read(tile + EXTRA, n, lane);
    }
    // product of row fragment n with the register fragments
    __device__ __forceinline__ static void score(Tile<16>& s, x8 f, int n, const x8 (&b)[kKS]) {
        s.b[n / kKS] = Tr<T>::mma(f, b[n % kKS], s.b[n / kKS]);
    }
    __device__ __forceinline__ static void accum(Acc (&acc)[kDB], x8 f, int n, const x8 (&p)[kPF]) {
        acc[n] = Tr<T>::mma(f, p[0], acc[n]);
    }
    // Column sums of p on the matrix cores: sum += ones^T p, column c's in every
    // entry (ones_frag: all ones).
    __device__ __forceinline__ static x8 ones_frag(int) {
        x8 o;
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = (T)1.0f;
        return o;
    }
    __device__ __forceinline__ static void colsum(f32x4& sum, x8 ones, const x8 (&p)[kPF]) {
        sum = Tr<T>::mma(ones, p[0], sum);
    }
    __device__ __forceinline__ static float colsum_of(f32x4 sum, int) { return sum[0]; }
    __device__ __forceinline__ static void pack(x8 (&pf)[kPF], const float (&p)[2][4]) {
        pf[0] = x8{Tr<T>::cvt(p[0][0]), Tr<T>::cvt(p[0][1]), Tr<T>::cvt(p[0][2]),
                   Tr<T>::cvt(p[0][3]), Tr<T>::cvt(p[1][0]), Tr<T>::cvt(p[1][1]),
                   Tr<T>::cvt(p[1][2]), Tr<T>::cvt(p[1][3])};
    }
    // the token row of D elements at p from the column accumulators, scaled
    __device__ __forceinline__ static void store(T* p, const Acc (&acc)[kDB], int grp, float f) {
#pragma unroll
        for (int db = 0; db < kDB; ++db) st_x4<T>(p + db * 16 + grp * 4, acc[db] * f);
    }
};

template <typename T, int D>
struct TileOps<T, D, 32> {
    using x8 = typename Tr<T>::x8;
    using Acc = f32x16;
    static constexpr int kStep = 16, kKS = D / 16, kDB = D / 32, kF = D / 16, kPF = 2;
    RowFrag32<T, D> rf;
    ColFrag32<T, D> cf;
    __device__ __forceinline__ void init(int lane, int col0) {
        rf.init(lane, col0);
        cf.init(lane, col0);
    }
    __device__ __forceinline__ void rows(const unsigned char* tile, x8 (&f)[kF]) const {
        rf.read(tile, f);
    }
    // fragment n = db * 2 + bi
    template <int EXTRA = 0>
    __device__ __forceinline__ void cols(const unsigned char* tile, x8 (&f)[kF]) const {
        cf.template read<EXTRA>(tile, f);
    }
    __device__ __forceinline__ static void score(Tile<32>& s, x8 f, int n, const x8 (&b)[kKS]) {
        s.v = Tr<T>::mma(f, b[n], s.v);
    }
    __device__ __forceinline__ static void accum(Acc (&acc)[kDB], x8 f, int n, const x8 (&p)[kPF]) {
        acc[n >> 1] = Tr<T>::mma(f, p[n & 1], acc[n >> 1]);
    }
    // Column sums of p with 16x16x32 steps, whose operand B has lane l at column
    // l % 16 and slots 8 (l / 16): the lanes of columns c and c + 16 fall into one
    // column there, so the left operand has ones for the even lane groups in its
    // even rows and for the odd groups in its odd rows, and a lane finds the sum
    // of its own column in the entry of its group's parity (half the matrix time
    // of a 32x32x16 step per fragment, and four registers instead of sixteen).
    __device__ __forceinline__ static x8 ones_frag(int lane) {
        x8 o;
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = (T)(((lane >> 4) & 1) == (lane & 1) ? 1.0f : 0.0f);
        return o;
    }
    __device__ __forceinline__ static void colsum(f32x4& sum, x8 ones, const x8 (&p)[kPF]) {
        sum = Tr<T>::mma(ones, p[0], sum);
        sum = Tr<T>::mma(ones, p[1], sum);
    }
    __device__ __forceinline__ static float colsum_of(f32x4 sum, int lane) {
        return (lane >> 4) & 1 ? sum[1] : sum[0];
    }
    __device__ __forceinline__ static void pack(x8 (&pf)[kPF], const float (&p)[2][8]) {
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
            pf[bi] = x8{Tr<T>::cvt(p[bi][0]), Tr<T>::cvt(p[bi][1]), Tr<T>::cvt(p[bi][2]),
                        Tr<T>::cvt(p[bi][3]), Tr<T>::cvt(p[bi][4]), Tr<T>::cvt(p[bi][5]),
                        Tr<T>::cvt(p[bi][6]), Tr<T>::cvt(p[bi][7])};
    }
    __device__ __forceinline__ static void store(T* p, const Acc (&acc)[kDB], int grp, float f) {
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                st_x4<T>(p + db * 32 + i * 8 + grp * 4,
                         f32x4{acc[db][4 * i], acc[db][4 * i + 1], acc[db][4 * i + 2],
                               acc[db][4 * i + 3]} * f);
    }
};

}  // namespace na
