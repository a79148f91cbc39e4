// Arguments and addressing of the GEMM kernel on smaller tiles (amap_gemm_ring.hip); the address functions are
// compiled for the GPU and for the host, where its replay walks them.
#pragma once

#include "amap_gemm.hpp"

namespace amap_gemm {

// One operand (or one source of a gathered A): element (x, k), x = m or n, lies at base + dx(x) + k part.
struct RingOperand {
    const uint16_t *src;
    uint32_t base;
    uint32_t steps;   // gathered A: k-steps of this source
    int32_t kss;      // X form: source elements between consecutive k inside a k-step (K form: 1)
    Digits dx;
};

// Workgroup -> output tile.  Every XCD (workgroup b runs on XCD b % 8) gets one contiguous eighth of the sequence
// that walks the tiles in bands of `group` rows, down the band first: its share is a compact block of tiles, so the A rows and
// W columns its workgroups have in common are fetched into its L2 once.
struct RingTiles {
    uint32_t tiles_m, tiles_n, group;
    FastDiv f_band, f_group, f_last;   // division by group * tiles_n, by group, by the rows of the last band
};
AMAP_HD void ring_tile(const RingTiles &r, uint32_t b, uint32_t grid, uint32_t &tm, uint32_t &tn) {
    const uint32_t t = xcd_remap(b, grid);
    const uint32_t band = fdiv(t, r.f_band), first = band * r.group, at = t - first * r.tiles_n;
    const bool last = first + r.group > r.tiles_m;
    const uint32_t rows = last ? r.tiles_m - first : r.group;
    tn = fdiv(at, last ? r.f_last : r.f_group);
    tm = first + (at - tn * rows);
}

// Runs of A along k shorter than a k-step, of one length (k has two digits): where a lane's chunk lies follows from where
// it lay a step before.  ext = length of a run, rem = elements of a step past its last whole run, step = bytes a step moves
// the chunk, carry = bytes more where it passes the end of a run.
struct RingRuns {
    uint32_t ext, rem, step, carry;
};
AMAP_HD void ring_runs_next(const RingRuns &r, uint32_t &low, uint32_t &off) {
    low += r.rem;
    const bool over = low >= r.ext;
    low -= over ? r.ext : 0u;
    off += r.step + (over ? r.carry : 0u);
}

struct RingCommon {
    uint16_t *C;
    uint32_t M, N, steps;
    RingTiles map;
    T2Steps a_steps, w_steps;
    Digits a_dk;      // runs of A shorter than a step: k per lane
    RingRuns a_runs;
    RingOperand w;
    uint16_t store_mapped, stream;   // stream: the product goes past the caches (see stores_stream)
    uint32_t obase;
    Digits om, on;
};
template <int NSEG>
struct RingArgs : RingCommon {
    RingOperand a[NSEG];
};

// Index x of a dimension -> its offset.  The digits of a dimension nest (digit j + 1 counts what digit j wraps; the plan
// refuses others), so n digits take n - 1 divisions, and the one digit that most dimensions have none; digits_offset4
// takes eight, with nothing to decide.  The short way is the faster one where a product has few tiles and the decode
// is not hidden behind another tile's work (the tiles smaller than 128 x 128, and those with 8 wavefronts):
// attention output of one sequence, M = 512, K = N = 1024, 6.5 us of kernel time against 7.0, M = 999, K = N = 768
// 6.4 / 6.9.  With several tiles a compute unit its branches cost more than they save: 1x1 conv behind a concat,
// M = 100352, K = 320, N = 256, 27.5 us against 25.7.
template <bool SHORT>
AMAP_HD uint32_t ring_digits(const Digits &d, uint32_t x) {
    if constexpr (!SHORT) return digits_offset4(d, x);
    if (d.n <= 1) return x * (uint32_t)d.ss[0];
    uint32_t off = 0;
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
#endif
    for (uint32_t j = 0; j + 1 < (uint32_t)kMaxDigits; ++j) {
        if (j + 1 >= d.n) break;
        const uint32_t q = fdiv(x, d.fext[j]);
        off += (x - q * d.ext[j]) * (uint32_t)d.ss[j];
        x = q;
    }
    return off + x * (uint32_t)d.ss[d.n - 1];
}

// A load block is the 1 KiB of LDS that one load instruction of a wavefront fills in lane order.
// K form: block b = rows 8 b .. 8 b + 7, 64 k each; lane i brings row 8 b + i / 8, physical chunk i % 8.
AMAP_HD uint32_t ring_k_chunk(uint32_t b, uint32_t lane) { return (lane & 7u) ^ (((b & 1u) << 2) | (lane >> 4)); }
// X form: block b = 512 / BX rows of k, BX elements each; lane i brings one 8-element chunk of one of them.
template <int BX>
AMAP_HD uint32_t ring_x_k(uint32_t b, uint32_t lane) {
    return b * (512u / BX) + lane / (BX / 8);
}
template <int BX>
AMAP_HD uint32_t ring_x_chunk(uint32_t b, uint32_t lane) {
    const uint32_t k = ring_x_k<BX>(b, lane);
    return (lane % (BX / 8)) ^ ((BX >= 128 ? k & 3u : (k >> 1) & 1u) << 2);
}
// byte offset of a lane's 16 bytes of load block b, for the first k-step of the operand; rows (columns) past the last
// one read the last one again, their products are never stored
template <bool X, int BX, bool SHORT>
AMAP_HD uint32_t ring_offset(const Digits &dx, uint32_t base, int32_t kss, uint32_t x0, uint32_t xn, uint32_t b, uint32_t lane) {
    if constexpr (X) {
        uint32_t x = x0 + 8u * ring_x_chunk<BX>(b, lane);
        x = x + 8u <= xn ? x : xn - 8u;
        return 2u * (base + ring_digits<SHORT>(dx, x) + ring_x_k<BX>(b, lane) * (uint32_t)kss);
    } else {
        uint32_t x = x0 + 8u * b + (lane >> 3);
        x = x < xn ? x : xn - 1u;
        return 2u * (base + ring_digits<SHORT>(dx, x) + 8u * ring_k_chunk(b, lane));
    }
}
// The same for block first + j of a wavefront, less the offset that its load instruction adds on both sides, plus
// kRingBias, which the scalar base lacks: what a lane adds is zero-extended and must not be negative.
constexpr uint32_t kRingBias = 3072;
template <bool X, int BX, bool SHORT>
AMAP_HD uint32_t ring_block_offset(const Digits &dx, uint32_t base, int32_t kss, uint32_t x0, uint32_t xn, uint32_t first, uint32_t j, uint32_t lane) {
    return ring_offset<X, BX, SHORT>(dx, base, kss, x0, xn, first + j, lane) + (kRingBias - 1024u * (j % 4u));
}
// The walk over the k-steps (see T2Steps): a plain step is one subtraction and one addition, a carry (rare) looks the
// levels up in the argument block.
struct RingWalk {
    uint32_t left, c1, c2;   // plain steps to the next carry; steps done on the levels above
    int64_t d0;
};
AMAP_HD RingWalk ring_walk_begin(const T2Steps &s) { return RingWalk{s.e[0], 0, 0, s.dl[0]}; }
AMAP_HD int64_t ring_walk_next(RingWalk &w, const T2Steps &s) {
    if (--w.left != 0) return w.d0;
    w.left = s.e[0];
    if (++w.c1 < s.e[1]) return s.dl[1];
    w.c1 = 0;
    if (++w.c2 < s.e[2]) return s.dl[2];
    w.c2 = 0;
    return s.dl[3];
}
// LDS reads of fragment f (32 rows or columns from x_base + 32 f) and sub-step kk (16 k), bytes from the operand's part of
// a stage.  K form: 16 bytes, row lane % 32, k = 16 kk + 8 (lane / 32).  X form (hi = 0, 1): lane = 16 g + s supplies
// the 8 bytes at k = 16 kk + 8 (g / 2) + s / 4 + 4 hi, x = 16 (g % 2) + 4 (s % 4) and receives four consecutive k of one x.
AMAP_HD uint32_t ring_k_frag(uint32_t lane, uint32_t x_base, uint32_t f, uint32_t kk) {
    return x_base * 128u + (((lane & 31u) * 128u + (((lane >> 5) ^ ((lane >> 1) & 7u)) << 4)) ^ (kk << 5)) + f * 4096u;
}
template <int BX>
AMAP_HD uint32_t ring_x_frag(uint32_t lane, uint32_t x_base, uint32_t f, uint32_t kk, uint32_t hi) {
    const uint32_t gq = lane >> 4, sq = lane & 15u;
    const uint32_t block = ((x_base >> 5) + f) ^ (BX >= 128 ? sq >> 2 : sq >> 3);
    return (16u * kk + 8u * (gq >> 1) + (sq >> 2) + 4u * hi) * (2u * BX) + block * 64u + (gq & 1u) * 32u + (sq & 3u) * 8u;
}
// LDS byte address of 16-byte chunk cv of row `row` of the staged output tile
template <int BN>
AMAP_HD uint32_t ring_c_slot(uint32_t row, uint32_t cv) {
    return row * (2u * BN) + ((cv ^ (BN >= 128 ? row & 15u : (row >> 1) & 7u)) << 4);
}

// Stores of a staged output tile by WAVES wavefronts, BN / 8 lanes to a row: wavefront w's lane l stores row row_of_store(p, 64 w + l) at
// pass p.  For a mapped store each lane decodes one row of its wavefront's, row_of_lane, and store p takes the offset from
// lane_of_store(p, l) of the same wavefront.
template <int BM, int BN, int WAVES>
struct RingStore {
    static constexpr uint32_t kCv = BN / 8, kWaveRows = 64 / kCv, kRows = WAVES * kWaveRows, kPasses = BM / kRows;
    static_assert(kPasses * kWaveRows <= 64, "a row per lane");
    static_assert(kPasses >= 1 && BM % kRows == 0, "every row of the tile is stored");
    static AMAP_HD uint32_t row_of_store(uint32_t p, uint32_t tid) { return p * kRows + tid / kCv; }
    static AMAP_HD uint32_t row_of_lane(uint32_t wave, uint32_t lane) { return lane / kWaveRows % kPasses * kRows + wave * kWaveRows + lane % kWaveRows; }
    static AMAP_HD uint32_t lane_of_store(uint32_t p, uint32_t lane) { return p * kWaveRows + lane / kCv; }
};

// The tiles there are (W8: 8 wavefronts; DEEP: 8 wavefronts and four stages, one workgroup to a compute unit; LOAD: four wavefronts
// that compute and four that load).
enum RingShape { RS_32x64 = 0, RS_64x64, RS_64x128, RS_128x128, RS_128x128_W8, RS_128x128_DEEP, RS_64x64_LOAD, RS_192x128 };

// A product as the ring kernel runs it: tile, wavefronts, forms of the operands (X: runs along m / n), arguments.
struct RingPlan {
    RingShape shape;
    int bm, bn, waves;   // wavefronts that compute
    const char *more;    // for a trace: what else the shape has
    bool ax, wx;
    int klane;    // runs of A along k shorter than a k-step: 1 of one length (k has two digits), 2 more digits
    int n_seg;
    RingArgs<kMaxSeg> args;
};

// Plan the product described by g (its maps already decoded into digits, no source of 2^31 - 2048 elements or more); false if
// its form has no ring kernel, or if the 256 x 256-tile kernel takes it as well (tile256) and is the faster one.
bool ring_plan(const GemmArgs &g, int amode, int wmode, bool tile256, uint32_t n_cu, RingPlan &p);
amap_status ring_launch(const RingPlan &p, hipStream_t stream);
// Host replay of a plan: every load against a_bytes[source] / w_bytes, every fragment read against the element the
// operands' maps name, every vector of the output stored once.  Returns the number of errors.
int64_t ring_replay(const RingPlan &p, const GemmArgs &g, const int64_t *a_bytes, int64_t w_bytes);

}  // namespace amap_gemm
