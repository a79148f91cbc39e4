// The product of amap_gemm.hip on smaller output tiles: out[m,n] = bf16( sum_k A[m,k] * W[k,n] ), both operands read
// through composed maps (the consumer loads of the paper's eq. 4), the product stored through one (eq. "store").
//
// One output tile per workgroup of 2 to 8 wavefronts, k in steps of BK through a ring of NST LDS stages.  Both
// operands go from global memory straight into LDS (global_load_lds, 16 bytes per lane): no staging registers, no
// LDS-write instructions, and because every lane brings its own address the map's digits cost nothing in the loop:
// a lane's rows (or its 8 columns) are decoded once per tile, a k-step moves one scalar base.
//   operand with runs along k ("K" form): stage [row][64 k], 128 bytes per row, 16-byte chunks XOR-ed with row / 2, so
//     that the 16 rows an LDS read serves together cover all banks;
//   operand with runs along m or n ("X" form: a channel-major activation, a row-major weight): stage [k][x], read with
//     the transposing LDS read (ds_read_b64_tr_b16), which hands every lane four consecutive k of one x; chunks XOR-ed
//     so that the four k rows of such a read lie in different banks.
// A step waits for its own loads only (vmcnt counts the loads of the NST - 2 later steps that may stay in flight),
// passes one barrier, issues the loads of step s + NST - 1 into the stage that step s - 1 has just left, and computes.
// What bounds a step on small tiles is LDS: the loads' writes (64 bytes a clock and compute unit on their own) and the
// fragment reads share about 113 bytes a clock, 48 KB per step of 64 x 64 x 64 (0.18 us; measured 0.14 .. 0.20), 72 KB of
// 64 x 128 (0.27; 0.23 .. 0.31), 96 KB of 128 x 128 (0.36; 0.40 .. 0.47).  A compute unit with one such tile gets its operands at
// 93 bytes a ns at most, whatever the tile and however many steps are in flight (64 x 64 0.175 us a step, 128 x 128 0.35).  Level or slower: wavefronts that share a tile along k
// and so read less (64 x 128, M = 2400, K = 1280: 11.0 against 9.9 us), two steps per barrier, more stages, reads or loads
// placed elsewhere among the matrix instructions.
#include "amap_gemm_ring.hpp"
#include "amap_launch.hpp"

#include <algorithm>
#include <cstring>
#include <type_traits>
#include <vector>

using namespace amap_dev;
using namespace amap_detail;
using namespace amap_gemm;

namespace {

// the part of the argument block in front of the epilogue's tables and of the second source of a gathered A
constexpr uint32_t kRingArgTouch = sizeof(RingArgs<1>);

// Wavefronts that only load (T::LOAD of them, behind those that compute): the same waits without the wavefront's own LDS reads, which it has none of.
template <int N>
__device__ __forceinline__ void ring_landed() {
    static_assert(N < 64, "vmcnt");
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"(N) : "memory");
}
template <int L, int R>
__device__ __forceinline__ void ring_landed_step(uint32_t later) {
    if constexpr (R == 0) {
        ring_landed<0>();
    } else {
        if (later >= (uint32_t)R)
            ring_landed<R * L>();
        else
            ring_landed_step<L, R - 1>(later);
    }
}

// wait until the loads of all but the `later` newest steps (L loads each per wavefront) have landed, then meet the
// other wavefronts; the compiler does not know of these loads.  (lgkmcnt: this wavefront's reads of the stage that is
// refilled next are done.)
template <int N>
__device__ __forceinline__ void ring_wait() {
    static_assert(N < 64, "vmcnt");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(N) : "memory");
}
template <int L, int R>
__device__ __forceinline__ void ring_wait_step(uint32_t later) {
    if constexpr (R == 0) {
        ring_wait<0>();
    } else {
        if (later >= (uint32_t)R)
            ring_wait<R * L>();
        else
            ring_wait_step<L, R - 1>(later);
    }
}

// Load blocks j = 0 .. N - 1 of a wavefront: lane i's 16 bytes of block j land at lds + 1024 j + 16 i.  The instruction's
// offset counts on both sides, so one write of M0 serves four blocks (ring_block_offset takes it off the address).
template <int N>
__device__ __forceinline__ void ring_load(const char *base, const uint32_t (&off)[N], uint32_t lds) {
#pragma unroll
    for (int j = 0; j < N; j += 4) {
        const uint32_t at = lds + 1024u * j;
        if (j + 4 <= N)
            asm volatile(
                "s_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %4\n\tglobal_load_lds_dwordx4 %1, %4 offset:1024\n\t"
                "global_load_lds_dwordx4 %2, %4 offset:2048\n\tglobal_load_lds_dwordx4 %3, %4 offset:3072" ::"v"(off[j]),
                "v"(off[j + 1 < N ? j + 1 : 0]), "v"(off[j + 2 < N ? j + 2 : 0]), "v"(off[j + 3 < N ? j + 3 : 0]), "s"(base), "s"(at)
                : "memory");
        else if (j + 3 == N)
            asm volatile("s_mov_b32 m0, %4\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %3\n\tglobal_load_lds_dwordx4 %1, %3 offset:1024\n\t"
                         "global_load_lds_dwordx4 %2, %3 offset:2048" ::"v"(off[j]),
                         "v"(off[j + 1 < N ? j + 1 : 0]), "v"(off[j + 2 < N ? j + 2 : 0]), "s"(base), "s"(at)
                         : "memory");
        else if (j + 2 <= N)
            asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024" ::"v"(off[j]),
                         "v"(off[j + 1 < N ? j + 1 : 0]), "s"(base), "s"(at)
                         : "memory");
        else
            load_to_lds16(base, off[j], at);
    }
}

template <class T>
__global__ __launch_bounds__(64 * (T::WVM * T::WVN + T::LOAD), T::OCC) void amap_gemm_ring_kernel(const RingArgs<T::NSEG> g) {
    constexpr int BM = T::BM, BN = T::BN, BK = T::BK, NST = T::NST;
    constexpr int kCompute = T::WVM * T::WVN, kWaves = kCompute + T::LOAD, kLoad = T::LOAD ? T::LOAD : kCompute;   // wavefronts that compute, all, that load
    constexpr int XM = BM / T::WVM, XN = BN / T::WVN;         // a wavefront's part of the tile
    constexpr bool AX = T::AX, WX = T::WX;
    constexpr uint32_t kABytes = BM * BK * 2, kWBytes = BN * BK * 2, kStage = kABytes + kWBytes;
    constexpr int NA = kABytes / (1024 * kLoad), NW = kWBytes / (1024 * kLoad);   // loads per loading wavefront and step
    constexpr int FM = XM / 32, FN = XN / 32;                 // 32 x 32 tiles per wavefront
    {
        // every 64-byte line of the argument block that the prologue reads, fetched side by side: read where they are
        // needed, the digit tables are one scalar-cache miss after the other in front of the first load
        const uint32_t *const arg = reinterpret_cast<const uint32_t *>(&g);
        uint32_t x = 0;
#pragma unroll
        for (uint32_t at = 0; at < kRingArgTouch / 4; at += 16) x |= arg[at];
        asm volatile("" ::"s"(x));
    }
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t wm = wave / T::WVN, wn = wave % T::WVN;   // (used by the wavefronts that compute)
    const uint32_t lwave = T::LOAD == 0 ? wave : wave < kCompute ? 0u : wave - kCompute;   // a loading wavefront's share of the blocks
    uint32_t tm, tn;
    ring_tile(g.map, blockIdx.x, gridDim.x, tm, tn);
    const uint32_t m0 = tm * BM, n0 = tn * BN;

    // ---- per-lane byte offsets of this wavefront's load blocks, and the scalar bases they are added to
    static_assert(NA >= 1 && NW >= 1, "ring_load");
    uint32_t a_off[NA], w_off[NW];
#pragma unroll
    for (int j = 0; j < NA; ++j) a_off[j] = ring_block_offset<AX, BM, T::SHORT>(g.a[0].dx, g.a[0].base, g.a[0].kss, m0, g.M, lwave * NA, j, lane);
#pragma unroll
    for (int j = 0; j < NW; ++j) w_off[j] = ring_block_offset<WX, BN, T::SHORT>(g.w.dx, g.w.base, g.w.kss, n0, g.N, lwave * NW, j, lane);
    const char *ka = reinterpret_cast<const char *>(g.a[0].src) - kRingBias, *kw = reinterpret_cast<const char *>(g.w.src) - kRingBias;
    RingWalk a_walk = ring_walk_begin(g.a_steps), w_walk = ring_walk_begin(g.w_steps);
    uint32_t seg = 0, seg_left = g.a[0].steps;   // NSEG > 1: the source the stream reads, and its k-steps to go
    int64_t seg_step = 2 * (int64_t)g.a[0].kss * BK;
    // KLANE, runs of A shorter than a step: what k adds to a lane's two chunk orders.  Decoded from k each step it costs two
    // chains of divisions and reads of the argument block between a step's barrier and its loads; with runs of one length
    // (KLANE 1, a head's rows) it follows from the step before.  Runs of 80: M = 300, K = 960, N = 1000 8.4 us decoded, 7.3 us
    // carried on; M = 6300, K = 1600, N = 4096 108 and 99.5 us; M = 3600, K = 1280, N = 2048 26.8 and 26.1 us; runs of 32:
    // M = 8000, K = 256, N = 2048 16.9 and 16.3 us.
    uint32_t ld_k = 0, kl[2] = {}, kl_low[2] = {};
    auto chunk_of = [&](uint32_t par) __attribute__((always_inline)) { return 8u * ring_k_chunk(lwave * NA + par, lane); };
    if constexpr (T::KLANE) {
#pragma unroll
        for (uint32_t par = 0; par < 2; ++par) {
            const uint32_t c8 = chunk_of(par);
            kl[par] = 2u * (ring_digits<T::SHORT>(g.a_dk, c8) - c8);
            kl_low[par] = c8 - fdiv(c8, g.a_dk.fext[0]) * g.a_dk.ext[0];
        }
    }
    const uint32_t lds_a = __builtin_amdgcn_readfirstlane(lwave * (NA * 1024u)), lds_w = __builtin_amdgcn_readfirstlane(kABytes + lwave * (NW * 1024u));
    auto issue = [&](uint32_t stage) __attribute__((always_inline)) {
        if constexpr (T::NSEG > 1) {
            if (seg_left == 0) {   // the next source of a gathered A: its own rows, strides and pointer
                ++seg;
                const RingOperand &s = g.a[seg];
                seg_left = s.steps;
                seg_step = 2 * (int64_t)s.kss * BK;
                ka = reinterpret_cast<const char *>(s.src) - kRingBias;
#pragma unroll
                for (int j = 0; j < NA; ++j) a_off[j] = ring_block_offset<AX, BM, T::SHORT>(s.dx, s.base, s.kss, m0, g.M, lwave * NA, j, lane);
            }
        }
        if constexpr (T::KLANE) {
            uint32_t off[NA];
#pragma unroll
            for (int j = 0; j < NA; ++j) off[j] = a_off[j] + kl[j & 1];
            ring_load<NA>(ka, off, lds_a + stage);
        } else {
            ring_load<NA>(ka, a_off, lds_a + stage);
        }
        ring_load<NW>(kw, w_off, lds_w + stage);
        if constexpr (T::NSEG > 1) {
            --seg_left;
            ka += seg_step;
        } else if constexpr (!T::KLANE) {
            ka += ring_walk_next(a_walk, g.a_steps);
        }
        kw += ring_walk_next(w_walk, g.w_steps);
        if constexpr (T::KLANE) {
#pragma unroll
            for (uint32_t par = 0; par < 2; ++par) {
                if constexpr (T::KLANE == 1)
                    ring_runs_next(g.a_runs, kl_low[par], kl[par]);
                else
                    kl[par] = 2u * (ring_digits<T::SHORT>(g.a_dk, ld_k + BK + chunk_of(par)) - chunk_of(par));
            }
            ld_k += BK;
        }
    };

    // ---- fragment addresses.  What does not depend on the stage is kept per lane, the stage and the fragment go into
    // the instruction's offset: K form, one address per sub-step; X form, one per fragment
    constexpr int kSub = BK / 16;
    uint32_t a_frag[AX ? FM : kSub], w_frag[WX ? FN : kSub];
#pragma unroll
    for (int i = 0; i < (AX ? FM : kSub); ++i) a_frag[i] = AX ? ring_x_frag<BM>(lane, wm * XM, i, 0, 0) : ring_k_frag(lane, wm * XM, 0, i);
#pragma unroll
    for (int i = 0; i < (WX ? FN : kSub); ++i) w_frag[i] = kABytes + (WX ? ring_x_frag<BN>(lane, wn * XN, i, 0, 0) : ring_k_frag(lane, wn * XN, 0, i));
    auto read_frag = [&](auto x_form, auto bx, const auto &addr, uint32_t stage, uint32_t f, uint32_t kk) __attribute__((always_inline)) -> bf16x8 {
        if constexpr (!x_form.value) {
            return __builtin_bit_cast(bf16x8, *reinterpret_cast<lds_u32x4 *>(addr[kk] + (stage + f * 4096u)));
        } else {
            typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
            constexpr uint32_t kRow = 2u * bx.value;   // bytes per k
            const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(reinterpret_cast<lds_bf16x4 *>(addr[f] + (stage + kk * 16u * kRow)));
            const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(reinterpret_cast<lds_bf16x4 *>(addr[f] + (stage + (kk * 16u + 4u) * kRow)));
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    };
    using std::integral_constant;
    constexpr integral_constant<bool, AX> ax{};
    constexpr integral_constant<bool, WX> wx{};
    constexpr integral_constant<int, BM> bm{};
    constexpr integral_constant<int, BN> bn{};

    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    const uint32_t steps = g.steps;
    constexpr int L = NA + NW;
    if constexpr (T::LOAD) {
        // Loading is left to wavefronts of their own: a load instruction holds its wavefront until the address unit takes it, and
        // with one small tile on a compute unit nothing else fills that time.  A loading wavefront is one barrier per step:
        // its loads of the next step have landed, the stage of the step before is free, its next loads go there.  The others have the
        // whole step's fragments in registers and read the next step's into each as its last MFMA is issued.
        // 32 x 64 tiles, M = 256 and 512, K = N = 1024: 5.5 -> 4.8 us and 5.7 -> 4.9 us, M = N = 512, K = 2560 9.4 -> 8.7 us.
        // (64 x 64 tiles so 12.0 -> 11.5 us and 6.7 -> 6.4, but 0 .. 8 % slower from two tiles per unit on; 128 x 128 level.)
        static_assert(NST >= 4, "the stage a step leaves is refilled a step later");
        uint32_t left = steps - 1u;
        if (wave >= kCompute) {
#pragma unroll
            for (int s = 0; s < NST - 1; ++s)
                if ((uint32_t)s < steps) issue((uint32_t)s * kStage);
            ring_landed_step<L, NST - 2>(left);
            uint32_t to = (NST - 1) * kStage;
            for (; left >= (uint32_t)NST - 1u; --left) {
                ring_landed<(NST - 3) * L>();
                issue(to);
                to = to == (NST - 1) * kStage ? 0u : to + kStage;
            }
            for (; left; --left) ring_landed_step<L, NST - 3>(left - 1u);
        } else {
            bf16x8 fa[kSub][FM], fw[kSub][FN];
            asm volatile("s_barrier" ::: "memory");   // the first step has landed
#pragma unroll
            for (int kk = 0; kk < kSub; ++kk) {
#pragma unroll
                for (int i = 0; i < FM; ++i) fa[kk][i] = read_frag(ax, bm, a_frag, 0, i, kk);
#pragma unroll
                for (int j = 0; j < FN; ++j) fw[kk][j] = read_frag(wx, bn, w_frag, 0, j, kk);
            }
            uint32_t next = kStage;
            for (;;) {
                if (left) asm volatile("s_barrier" ::: "memory");   // the next step has landed; the last one's fragments have all been used
                __builtin_amdgcn_sched_barrier(0);
                uint32_t a_next[AX ? FM : kSub], w_next[WX ? FN : kSub];
#pragma unroll
                for (int i = 0; i < (AX ? FM : kSub); ++i) a_next[i] = a_frag[i] + next;
#pragma unroll
                for (int i = 0; i < (WX ? FN : kSub); ++i) w_next[i] = w_frag[i] + next;
#pragma unroll
                for (int kk = 0; kk < kSub; ++kk)
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int j = 0; j < FN; ++j) {
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[kk][j], fa[kk][i], acc[i][j], 0, 0, 0);
                            __builtin_amdgcn_sched_barrier(0);
                            // (after the last step: a stale stage, read and unused)
                            if (j == FN - 1) fa[kk][i] = read_frag(ax, bm, a_next, 0, i, kk);
                            if (i == FM - 1) fw[kk][j] = read_frag(wx, bn, w_next, 0, j, kk);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                next = next == (NST - 1) * kStage ? 0u : next + kStage;
                if (left-- == 0) break;
            }
        }
    } else {
        // Two sets of fragments, PK sub-steps of 16 k each: one is read while the other feeds the matrix cores.
        constexpr int PK = T::PK, kPhases = kSub / PK;
        static_assert(kSub % PK == 0 && (kPhases % 2 == 0 || (kPhases == 1 && NST % 2 == 0)), "the fragment sets alternate");
        bf16x8 fa[2][PK][FM], fw[2][PK][FN];
        auto read_one = [&](uint32_t set, uint32_t stage, uint32_t ph, int r) __attribute__((always_inline)) {
            if (r >= PK * (FM + FN)) return;
            const uint32_t kk = (uint32_t)(r / (FM + FN)), f = (uint32_t)(r % (FM + FN));
            if (f < (uint32_t)FM)
                fa[set][kk][f] = read_frag(ax, bm, a_frag, stage, f, ph * PK + kk);
            else
                fw[set][kk][f - FM] = read_frag(wx, bn, w_frag, stage, f - FM, ph * PK + kk);
        };
        // the MFMAs of one phase on fragment set `set`, the reads of the next phase (ph of `stage`) spread under them
        auto phase = [&](uint32_t set, uint32_t stage, uint32_t ph) __attribute__((always_inline)) {
            constexpr int kMf = PK * FM * FN, kRd = PK * (FM + FN), kPer = (kRd + kMf - 1) / kMf;
#pragma unroll
            for (int q = 0; q < kMf; ++q) {
#pragma unroll
                for (int r = 0; r < kPer; ++r) read_one(set ^ 1u, stage, ph, q * kPer + r);
                const int kk = q / (FM * FN), i = q / FN % FM, j = q % FN;
                // W as the row operand: the 32 x 32 result is C^T, a lane holds four consecutive n of one row m
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[set][kk][j], fa[set][kk][i], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        };

#pragma unroll
        for (int s = 0; s < NST; ++s)
            if ((uint32_t)s < steps) issue((uint32_t)s * kStage);
        ring_wait_step<L, NST - 1>(steps - 1u);
#pragma unroll
        for (int r = 0; r < PK * (FM + FN); ++r) read_one(0, 0, 0, r);
        // the ring once around per pass: stages and fragment sets are constants, a read is one instruction
        uint32_t left = steps - 1u;
        for (;;) {
            bool done = false;
#pragma unroll
            for (int st = 0; st < NST; ++st) {
                if (done) break;
                const uint32_t cur = st * kStage, next = (st + 1) % NST * kStage, set0 = kPhases == 1 ? st & 1 : 0;
#pragma unroll
                for (int ph = 0; ph + 1 < kPhases; ++ph) phase(set0 ^ (ph & 1u), cur, ph + 1);
                // the last fragments of this step are read: its stage is free once every wavefront is here, and the next step's
                // loads (all but those of up to NST - 2 later steps) have landed
                if (left) ring_wait_step<L, NST - 2>(left - 1u);
                if (left >= (uint32_t)NST) issue(cur);
                __builtin_amdgcn_sched_barrier(0);
                phase(set0 ^ ((kPhases - 1) & 1u), next, 0);   // (after the last step: a stale stage, read and unused)
                if (left-- == 0) done = true;
            }
            if (done) break;
        }
    }

    // ---- epilogue: the tile rounded to bf16 in LDS (the ring is free once every wavefront has passed), then whole rows
    // of 16-byte stores.  Accumulator v of a 32 x 32 tile in lane l: m = l % 32, n = 8 (v / 4) + 4 (l / 32) + v % 4.
    __syncthreads();
    const uint32_t row_l = lane & 31u, half = lane >> 5;
    if (T::LOAD == 0 || wave < kCompute) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    u32x2 o;
                    o.x = pack_bf16(acc[i][j][4 * q], acc[i][j][4 * q + 1]);
                    o.y = pack_bf16(acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
                    const uint32_t row = wm * XM + 32u * i + row_l, chunk = wn * (XN / 8) + 4u * j + q;
                    *reinterpret_cast<__attribute__((address_space(3))) u32x2 *>(ring_c_slot<BN>(row, chunk) + ((half ^ ((row >> 4) & 1u)) << 3)) = o;
                }
    }
    __syncthreads();
    typedef RingStore<BM, BN, kWaves> Store;
    const uint32_t cv = tid % Store::kCv, n = n0 + cv * 8u;
    const bool n_ok = n < g.N;
    const uint32_t n_off = g.store_mapped ? g.obase + ring_digits<T::SHORT>(g.on, n_ok ? n : 0u) : n;
    // A mapped store: a lane decodes one of its wavefront's rows, and every store asks the lane that has its row (see the
    // epilogue of the 256 x 256 kernel).
    uint32_t row_off = 0;
    if (g.store_mapped) {
        const uint32_t m = m0 + Store::row_of_lane(wave, lane);
        row_off = ring_digits<T::SHORT>(g.om, m < g.M ? m : g.M - 1u);
    }
    const uint32_t M = g.M, N = g.N;
    uint16_t *const C = g.C;
    const bool mapped = g.store_mapped;
    auto store_tile = [&](auto stream) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t p = 0; p < Store::kPasses; ++p) {
            const uint32_t row = Store::row_of_store(p, tid), m = m0 + row;
            u32x4 x = *reinterpret_cast<lds_u32x4 *>(ring_c_slot<BN>(row, cv));
            if ((row >> 4) & 1u) x = u32x4{x.z, x.w, x.x, x.y};
            size_t off = (size_t)m * N + n_off;
            if (mapped) off = n_off + (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * Store::lane_of_store(p, lane)), (int)row_off);
            if (m < M && n_ok) store_c(C + off, x, stream);
        }
    };
    // A along m: past the caches only.  us through the caches by past them, over 190 pointwise convolutions: whole 64-byte pieces 1.00 (outputs
    // of up to 1 MB, 40), 1.01 (4 MB, 9), 1.08 .. 1.10 (32 MB, 18), 1.19 (beyond, 3); rows of no whole pieces 0.94 .. 0.98 in the mean at
    // any size, 0.63 to 1.28 one by one (120; M = 29008, K = 96, N = 1000 25.1 and 15.9 us, M = 65072, K = 512, N = 360 36.6 and 47.0):
    // no line has been drawn for these.
    if constexpr (AX)
        store_tile(std::true_type{});
    else
        stores_by_kind(g.stream, store_tile);
}

template <class T>
amap_status launch(const RingArgs<kMaxSeg> &full, uint32_t grid, hipStream_t stream) {
    constexpr int kRing = T::NST * (T::BM + T::BN) * T::BK * 2, kTile = T::BM * T::BN * 2, lds = kRing > kTile ? kRing : kTile;
    static_assert(lds <= 160 * 1024, "what a compute unit has");
    if constexpr (lds > 65536) {   // what a launch may ask for without it
        static LdsReservation reserved;
        const hipError_t r = reserved.on_current_device({reinterpret_cast<const void *>(amap_gemm_ring_kernel<T>)}, lds);
        if (r != hipSuccess) {
            set_last_error("amap_gemm_ring_kernel: cannot reserve its LDS stages", hipGetErrorString(r));
            return AMAP_E_HIP;
        }
    }
    RingArgs<T::NSEG> g;
    static_cast<RingCommon &>(g) = full;
    for (int i = 0; i < T::NSEG; ++i) g.a[i] = full.a[i];
    const hipError_t e = launch_kernel<amap_gemm_ring_kernel<T>>(dim3(grid), dim3(64 * (T::WVM * T::WVN + T::LOAD)), lds, stream, g);
    if (e != hipSuccess) {
        set_last_error("amap_gemm_ring_kernel", hipGetErrorString(e));
        return AMAP_E_HIP;
    }
    return AMAP_OK;
}

template <int BM_, int BN_, int BK_, int NST_, int PK_, int WVM_, int WVN_, int OCC_, bool AX_, bool WX_, int NSEG_, int KLANE_, int LOAD_ = 0>
struct Shape {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, NST = NST_, PK = PK_, WVM = WVM_, WVN = WVN_, OCC = OCC_, NSEG = NSEG_;
    static constexpr bool AX = AX_, WX = WX_;
    static constexpr bool SHORT = PK_ == 2 || BM_ * BN_ < 128 * 128;   // see ring_digits
    static constexpr int LOAD = LOAD_;     // wavefronts that only load (0: those that compute load as well)
    static constexpr int KLANE = KLANE_;   // 0: whole steps of k in a run of A; 1, 2: shorter runs, of one length / of any digits
};

}  // namespace

namespace amap_gemm {

// k-steps of bk elements over the digits of k; false if a step could straddle two digits
static bool ring_steps(const Digits &d, uint32_t bk, T2Steps &s) {
    if (d.n == 0 || d.mult[0] != 1 || (d.n > 1 && d.ext[0] % bk)) return false;
    const int64_t st[kMaxDigits] = {(int64_t)bk * d.ss[0], d.ss[1], d.ss[2], d.ss[3]};
    const uint32_t e[kMaxDigits] = {(d.ext[0] + bk - 1) / bk, d.ext[1], d.ext[2], d.ext[3]};
    int64_t back = 0;   // from the last step of the levels below to their first one
    int at = 0;         // levels of one step (runs of exactly bk) are left out: the walk carries where it must only
    for (int j = 0; j < kMaxDigits; ++j) {
        if (e[j] == 1u && j + 1 < kMaxDigits) continue;
        s.dl[at] = 2 * (st[j] - back);
        back += (int64_t)(e[j] - 1u) * st[j];
        if (at + 1 < kMaxDigits) s.e[at] = j + 1 < kMaxDigits ? e[j] : 0xFFFFFFFFu;
        ++at;
    }
    for (; at < kMaxDigits; ++at) {
        s.dl[at] = 0;
        if (at + 1 < kMaxDigits) s.e[at] = 0xFFFFFFFFu;
    }
    return true;
}

// digit j + 1 counts what digit j wraps (see ring_digits)
static bool nested(const Digits &d) {
    uint64_t mult = 1;
    for (uint32_t j = 0; j < d.n; ++j) {
        if (d.mult[j] != mult) return false;
        mult *= d.ext[j];
    }
    return true;
}

static Digits one_digit(uint32_t ext, int32_t ss) {
    Digits d;
    std::memset(&d, 0, sizeof(d));
    d.n = 1;
    for (int j = 0; j < kMaxDigits; ++j) {
        d.mult[j] = 1;
        d.ext[j] = j ? 1u : ext;
        d.ss[j] = j ? 0 : ss;
        d.fmult[j] = make_fastdiv(1);
        d.fext[j] = make_fastdiv(d.ext[j]);
    }
    return d;
}

// 64 x 64 or 128 x 128 tiles: time in us, `step` per tile and 64 k plus `tile` per tile of a compute unit's share after 4 us for
// the launch, the first loads and the last stores.  Fitted to measurements with K = 256 .. 2560 and 1 .. 32 tiles per compute
// unit (for instance 128 x 128 tiles, K = 1024: 256 tiles 13.9 us, 512 21.2, 1024 38.5, 2048 71.6; 64 x 64 tiles: 512 9.8, 1024
// 16.9, 2048 27.7).
static double share_of(uint64_t tiles, double k64, uint32_t n_cu, double step, double tile) {
    const double q = (double)tiles / n_cu, up = (double)((tiles + n_cu - 1) / n_cu);
    // up to two tiles share a compute unit, so a few more tiles than units cost less than a second round
    const double rounds = q <= 2.0 ? 0.5 * (std::max(q, 1.0) + up) : up;
    return 4.0 + rounds * (step * k64 + tile);
}

// The shapes against each other, and the 256 x 256 tiles against them: time in us, `launch` for the launch, the first
// loads and the last stores, `tile` per tile of the busiest compute unit, and for every 64 k of its tiles s1 where it has one
// and all units do, s2 for two (they share the unit), `more` for each further one; from s0 to s1 up to one tile per unit (the
// fewer units work, the faster each).  What lies between whole numbers of tiles per unit counts for `up` of the next one.
// Along k: fitted to 1195 products of K = 256 .. 2560 timed on the device, operands in three sets of buffers in turn, each row over the
// tiles per unit at which its shape is considered and most where it is near the best (128 x 128 by 4 wavefronts is counted as by 8).
// Along m and n: fitted to 700 pointwise convolutions, the device's time as well.
// A row with s2 = 0 is of a shape that one tile per unit is all there is to: it has no figures beyond.
struct RingCost {
    float launch, s0, s1, s2, more, tile, up;
};
static double estimate(const RingCost &c, uint64_t tiles, double k64, uint32_t n_cu) {
    const double q = (double)tiles / n_cu, up = (double)((tiles + n_cu - 1) / n_cu), e = q > 1.0 ? q + c.up * (up - q) : 1.0;
    if (q > 1.0 && c.s2 == 0.f) return 1e30;
    const double step = c.s0 + (c.s1 - c.s0) * std::min(q, 1.0) + (c.s2 - c.s1) * (std::min(e, 2.0) - 1.0) + c.more * std::max(e - 2.0, 0.0);
    return c.launch + c.tile * e + step * k64;
}
// by RingShape: whole steps of k in a run of A; shorter runs; both operands along m and n
static const RingCost kCostK[] = {{2.79f, .100f, .146f, .258f, .215f, .34f, .66f}, {2.94f, .176f, .237f, .365f, .213f, .24f, .63f},
                                  {3.71f, .253f, .315f, .635f, .240f, .07f, .60f}, {1.78f, .453f, .661f, .814f, .617f, 1.81f, .60f},
                                  {1.78f, .453f, .661f, .814f, .617f, 1.81f, .60f}, {3.84f, .226f, .521f, 0.f, 0.f, 1.f, 0.f},
                                  {3.60f, .133f, .192f, 0.f, 0.f, .10f, 0.f}, {5.10f, .339f, .604f, 0.f, 0.f, 0.f, 0.f}};
static const RingCost kCostRuns[] = {{3.11f, .110f, .161f, .281f, .282f, .11f, .76f}, {3.04f, .225f, .270f, .446f, .240f, .00f, .62f},
                                     {3.52f, .286f, .361f, .688f, .567f, .00f, .63f}, {1.38f, .457f, .738f, 1.09f, .512f, 1.90f, .31f},
                                     {1.38f, .457f, .738f, 1.09f, .512f, 1.90f, .31f}, {3.22f, .361f, .594f, 0.f, 0.f, 1.f, 0.f},
                                     {3.55f, .165f, .244f, 0.f, 0.f, .00f, 0.f}, {4.30f, .600f, .720f, 0.f, 0.f, 0.f, 0.f}};
static const RingCost kCostX[] = {{}, {2.67f, .439f, .537f, .567f, .238f, .347f, .475f}, {2.63f, .495f, .673f, .714f, .306f, .505f, .623f},
                                  {2.38f, .646f, 1.16f, 1.25f, .389f, 1.23f, .279f}};

// rows, columns, wavefronts that compute, what else there is to say (in a trace)
static const struct { int bm, bn, waves; const char *more; } kRingTile[] = {{32, 64, 2, ", 2 more load"}, {64, 64, 4, ""}, {64, 128, 4, ""}, {128, 128, 4, ""}, {128, 128, 8, ""},
                                                                            {128, 128, 8, ", four stages"}, {64, 64, 4, ", 4 more load"}, {192, 128, 8, ""}};

// The shape of a product's tiles, and its estimate.  Measured on 354 other products along k: 0.8 % off the best shape each has, where
// the shapes and figures before this were 3.2 % off.  Along m 2 % off the best over the 700 that the figures were fitted to; of 140 others
// 0.8 % over 119 (the worst 13 %), and 26 % over the 21 of the fewest tiles, which keep 128 x 128 (see below; none takes more than 5.5 us).
static RingShape ring_shape(const GemmArgs &g, const RingPlan &p, uint32_t n_cu, double &best) {
    RingShape shape = RS_128x128;
    best = 1e30;
    const double k64 = g.K / 64.0;
    auto tiles = [&](int bm, int bn) { return (uint64_t)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn); };
    const double q64x128 = (double)tiles(64, 128) / n_cu;
    auto consider = [&](RingShape s, double times = 1.0) {
        const double t = times * estimate((p.ax ? kCostX : p.klane ? kCostRuns : kCostK)[s], tiles(kRingTile[s].bm, kRingTile[s].bn), k64, n_cu);
        if (t < best) best = t, shape = s;
    };
    if (p.ax || g.n_seg > 1) {
        // a weight along k with A along m, sources gathered along k: 128 x 128 only
        consider(RS_128x128);
        // Smaller tiles where 128 x 128 leave compute units idle, or N or M half of a tile empty: M = 15408, K = 608, N = 128
        // 13.7 -> 8.9 us, M = 8624, K = 256, N = 512 9.3 -> 8.2, M = 50176, K = 288, N = 64 10.1 -> 8.7; M = 100352, K = 320, N = 256
        // stays (25.9 against 29).  Few tiles of a short walk too: M = 832, K = 224, N = 128 6.2 -> 4.5, M = 768, K = 96, N = 128
        // 5.2 -> 4.0; but the fewest of all, where the call takes what issuing it takes (M = 288, K = 256, N = 128 5.3 and 4.2).
        if (p.ax && p.wx && (tiles(128, 128) >= 16 || g.M > 512 || g.K > 256)) {
            // Rows of C of no whole 64-byte pieces that one tile of 128 columns holds: two tiles of 64 share a piece of each of them.  The 58
            // products (N = 72 .. 120) whose shape the factor decides take 0.946 of the time without it, none more; wider rows are shared
            // by any tiles, and 120 products with N = 136 .. 1096 took 1.036 of it (M = 3920, K = 32, N = 200 3.78 against 3.62 us).
            consider(RS_64x64, g.N % 32 && g.N > 64 && g.N < 128 ? 1.06 : 1.0);
            consider(RS_64x128);
        }
        return shape;
    }
    // 128 x 128 tiles come two to a compute unit.  8 wavefronts each where the busiest unit's last pair is whole, 4 where a single tile is
    // left over, which 8 finish no sooner; beyond eight tiles that counts for little.  Time by 8 / by 4 in the mean (products), by
    // the tiles of the busiest unit, K >= 768:
    //   3  1.02 (57)   4  0.97 (34)   5  1.02 (62)   6  0.97 (37)   7  1.01 (20)   8  0.96 (23)   9 .. 12  0.99 (40)   more  0.99 (26)
    // up to 2 (any K) 0.95;  below K = 768  3  1.00   4  0.98   5  1.02   6  1.01   7  0.99   8  0.97.  us by 8 / by 4: 1.97 tiles per unit,
    // K = 1024 19.2 / 20.1   2.88, K = 2048 53.2 / 52.5   3.47, K = 2048 59.0 / 61.6   4.12, K = 1024 44.6 / 43.4   5.21, K = 1024 48.5 / 50.3
    const uint64_t up128 = (tiles(128, 128) + n_cu - 1) / n_cu;
    // (K = 768 and six tiles: 0.95 to 1.02; K = 768 .. 1023 and more than eight: 0.95 to 1.02 as well)
    const bool by8 = up128 <= 2 || (up128 > 8 ? g.K >= 1024 : up128 % 2 == 0 && g.K >= (up128 == 6 ? 960u : 768u));
    const bool small = share_of(tiles(64, 64), k64, n_cu, 0.19, 0.35) < share_of(tiles(128, 128), k64, n_cu, 0.47, 1.4);
    consider(small ? RS_64x64 : up128 <= 2 ? RS_128x128_W8 : RS_128x128);
    const uint64_t t64 = tiles(64, 64), t128 = tiles(128, 128);
    if (p.klane < 2) {
        // three stages of 64 x 128 while two workgroups find room on every compute unit and the walk is long enough to pay for them:
        // M = 2400, K = 1280, N = 768 10.7 -> 9.5 us, M = 1322, K = N = 2048 22.3 -> 20.2, M = 825, K = 768, N = 2304 8.0 -> 7.4,
        // M = 1864, K = 640, N = 1000 8.3 -> 7.7, but M = 396, K = 512, N = 4096 5.4 -> 5.9, M = 1020, N = 1536 6.0 -> 6.2.  Under two
        // thirds of a tile per unit it has to be longer still (64 x 64 tiles are then one to a unit, and few units have two): 41 products
        // of K = 640 .. 959 were 3 % slower as 64 x 128 (M = 345, K = 704, N = 3072 6.2 -> 6.7, 6.6 -> 7.0 with operands out of the L2s),
        // 24 of K = 960 .. 1279 from 6 % faster to 8 % slower, 18 longer ones 4 % faster, runs shorter than a step 3 to 10 %.
        // Above one and a half per unit (64 x 64 tiles come three to a unit and would need a fourth) less will do: M = 1305, K = 512,
        // N = 3072 10.5 -> 9.1, M = 3717, N = 1024 4 % faster.  Beyond two the 128 x 128 tiles, with less LDS traffic, are up to 1.4 times
        // as fast
        const uint32_t least_k = q64x128 > 1.5 ? 384u : p.klane || 3.0 * q64x128 >= 2.0 ? 640u : 1280u;
        if (q64x128 <= 2.0 && g.K >= least_k) consider(RS_64x128);
        // Few tiles: 32 x 64 by two wavefronts that compute and two that load: M = 518, K = 2560, N = 512 12.0 (64 x 64) -> 8.7 us, M = 256,
        // K = N = 1024 5.9 -> 4.7, M = 49, K = 2560, N = 768 10.5 -> 7.2.  Very few tiles only with a long walk, and none of a short one:
        // there both take what issuing the call takes (M = 435, K = 384, N = 768 4.6 and 4.1 us, M = 62, K = 640, N = 768 5.1 and 4.3).
        // Runs of A shorter than a step cost the wavefronts that only load nothing: from K = 256 on (runs of 32, M = 44, K = 384, N = 1024
        // 4.35 -> 4.0).
        if (g.K >= (p.klane ? 256u : 512u) && (t64 >= 16 || (t64 >= 8 && g.K >= 896))) consider(RS_32x64);
        // 64 x 64 with loading wavefronts while no unit has two of them: M = 1000, K = N = 1024 6.7 -> 6.3 us, M = 576, K = 2048, N = 1024
        // 10.2 -> 8.9; beyond that 5 to 18 % slower, the other wavefronts' tiles fill the time already.
        if (t64 >= 16 && t64 <= n_cu) consider(RS_64x64_LOAD);
        // One 128 x 128 tile to a unit: four stages, three steps of operands on their way, instead of two stages for each of two
        // workgroups of which a unit has but one: M = 2618, K = 2560, N = 1000 28 -> 21.5 us, M = 2445, K = 1280, N = 1024 15.3 -> 12.2,
        // M = 1016, K = 1024, N = 3072 12.7 -> 10.9.  Up to half a unit's worth of tiles the smaller ones are ahead; nearly all
        // units busy, a short walk ends sooner on more, smaller workgroups (M = 970, K = 1024, N = 4096 14.8 against 13.4).
        if (2 * t128 > n_cu && t128 <= n_cu && (20 * t128 <= 17 * (uint64_t)n_cu || g.K >= 1280)) consider(RS_128x128_DEEP);
        // A few more 128 x 128 tiles than units put two on some of them while the others wait: 192 x 128 go once around, with half as much again
        // for the matrix cores to each byte that a unit is handed. 512 <= K < 768 4 % faster (26 products), from 768 on 8 % (73):
        // M = 2048, K = 768, N = 2304 12.1 -> 11.1 us, stored by heads 12.5 -> 11.4, M = 9618, K = 1600, N = 512 21.2 -> 18.8, in runs of 80
        // 24.5 -> 21.9 (one card, operands in three sets of buffers; 4 to 5 % on another); K = 384 0 to 3 % slower. (160 x 128, or four stages:
        // 0 to 4 % faster.)
        if (t128 > n_cu && tiles(192, 128) <= n_cu && g.K >= 512) consider(RS_192x128);
    }
    if (shape == RS_128x128 && by8) shape = RS_128x128_W8;
    return shape;
}

bool ring_plan(const GemmArgs &g, int amode, int wmode, bool tile256, uint32_t n_cu, RingPlan &p) {
    if (g.padded || g.n_seg > (uint32_t)kMaxSeg) return false;
    p.ax = amode == A_RUNS_M;
    p.wx = wmode != W_MAPPED_K;
    p.klane = 0;
    p.n_seg = (int)g.n_seg;
    // k in steps of 64 where a run along k is a 128-byte row of the stage; of 32 (more workgroups per compute unit: 39.8
    // against 42.8 us on a pointwise convolution [100352,256] x [256,512], 30.7 against 44.8 us gathered from four
    // sources) where both operands have theirs along m and n
    const uint32_t bk = p.ax && p.wx ? 32 : 64;
    if (g.K % bk) return false;
    std::memset(&p.args, 0, sizeof(p.args));
    RingArgs<kMaxSeg> &r = p.args;
    r.C = g.C;
    r.M = g.M;
    r.N = g.N;
    r.steps = g.K / bk;
    if (g.n_seg > 1) {
        for (uint32_t j = 0; j < g.n_seg; ++j) {
            const uint32_t len = g.seg_kend[j] - (j ? g.seg_kend[j - 1] : 0u);
            if (g.seg_dk[j].n != 1 || len % bk) return false;
            r.a[j] = RingOperand{g.seg_src[j], g.seg_sbase[j], len / bk, g.seg_dk[j].ss[0], g.seg_dm[j]};
        }
    } else {
        r.a[0] = RingOperand{g.A_src, g.sbase, r.steps, g.dk.ss[0], g.dm};
        if (!ring_steps(g.dk, bk, r.a_steps)) {
            if (p.ax) return false;
            p.klane = g.dk.n == 2 ? 1 : 2;
            r.a_dk = g.dk;
            if (p.klane == 1) {
                const uint32_t e = g.dk.ext[0], s0 = (uint32_t)g.dk.ss[0], s1 = (uint32_t)g.dk.ss[1];
                r.a_runs = RingRuns{e, bk % e, 2u * (bk % e * s0 + bk / e * s1), 2u * (s1 - e * s0)};
            }
        }
    }
    if (wmode == W_PLAIN) {
        r.w = RingOperand{g.W, 0, r.steps, (int32_t)g.N, one_digit(g.N, 1)};
        ring_steps(one_digit(g.K, (int32_t)g.N), bk, r.w_steps);
    } else {
        r.w = RingOperand{g.W, g.wbase, r.steps, g.wk.ss[0], g.wn};
        if (!ring_steps(g.wk, bk, r.w_steps)) return false;
    }
    if (!nested(r.a[0].dx) || !nested(r.w.dx) || (p.klane && !nested(r.a_dk)) || (g.store_mapped && (!nested(g.om) || !nested(g.on)))) return false;
    for (uint32_t j = 1; j < g.n_seg; ++j)
        if (!nested(r.a[j].dx)) return false;
    r.store_mapped = (uint16_t)g.store_mapped;
    r.obase = g.obase;
    r.om = g.om;
    r.on = g.on;
    r.stream = p.ax || stores_stream(g.M, g.N, g.store_mapped ? g.on.ext[0] : g.N);   // (A along m: the kernel has the one kind)

    // ---- the tile
    double t;
    p.shape = ring_shape(g, p, n_cu, t);
    if (tile256) {
        // The 256 x 256-tile kernel takes the product as well, and is ahead where its tiles fill the chip a whole number of
        // times (M = 8192, K = 1024, N = 4096 63 against 69 us; M = 4608, N = 2048 25.1 against 27.3) and behind it where they
        // leave units idle (M = 2048, K = 768, N = 2304 20.9 against 12.9 us, M = 512, K = N = 1024 23.7 against 5.8).  Its time,
        // fitted to the same products: the busier the chip the lower its clock; partial tiles add their masks.
        const uint64_t n256 = (uint64_t)((g.M + 255) / 256) * ((g.N + 255) / 256), rounds = (n256 + n_cu - 1) / n_cu, wgs = (n256 + rounds - 1) / rounds;
        const double step256 = 0.96 + 0.53 * (double)wgs / n_cu;
        const double t256 = 4.0 + (g.M % 256 || g.N % 256 ? 1.5 : 0.0) + (double)rounds * (g.K / 64.0) * step256 + 5.5 * (double)(rounds - 1);
        if (t > t256) return false;
    }
    p.bm = kRingTile[p.shape].bm;
    p.bn = kRingTile[p.shape].bn;
    p.waves = kRingTile[p.shape].waves;
    p.more = kRingTile[p.shape].more;
    r.map.tiles_m = (uint32_t)((g.M + p.bm - 1) / p.bm);
    r.map.tiles_n = (uint32_t)((g.N + p.bn - 1) / p.bn);
    if ((uint64_t)r.map.tiles_m * r.map.tiles_n >= (1ull << 31)) return false;
    // bands of 8 tile rows: the 32 or so tiles an XCD works on at a time are then a compact block (4 or 32 rows: 0 .. 4 % slower)
    r.map.group = std::min<uint32_t>(8, r.map.tiles_m);
    if ((uint64_t)r.map.group * r.map.tiles_n >= (1ull << 31)) return false;
    r.map.f_band = make_fastdiv(r.map.group * r.map.tiles_n);
    r.map.f_group = make_fastdiv(r.map.group);
    const uint32_t last = r.map.tiles_m % r.map.group;
    r.map.f_last = make_fastdiv(last ? last : r.map.group);
    return true;
}

namespace {
// the kernel shapes that exist, each handed to f as a type
template <bool AX, bool WX, int NSEG, int KLANE, class F>
void with_tile(const RingPlan &p, F f) {
    switch (p.shape) {
    case RS_32x64:
        if constexpr (!AX && NSEG == 1 && KLANE < 2) f(Shape<32, 64, 64, 5, 2, 1, 2, 2, false, WX, 1, KLANE, 2>());
        break;
    case RS_64x64:
        if constexpr (AX && WX)
            f(Shape<64, 64, 32, 4, 2, 2, 2, 4, true, true, NSEG, 0>());
        else if constexpr (!AX && NSEG == 1)
            f(Shape<64, 64, 64, 3, 2, 2, 2, 3, false, WX, 1, KLANE>());
        break;
    case RS_64x128:
        if constexpr (AX && WX)
            f(Shape<64, 128, 32, 3, 1, 2, 2, 4, true, true, NSEG, 0>());
        else if constexpr (!AX && NSEG == 1 && KLANE < 2)
            f(Shape<64, 128, 64, 3, 2, 2, 2, 2, false, WX, 1, KLANE>());
        break;
    case RS_192x128:
        if constexpr (!AX && NSEG == 1 && KLANE < 2) f(Shape<192, 128, 64, 3, 2, 2, 4, 2, false, WX, 1, KLANE>());
        break;
    case RS_64x64_LOAD:
        if constexpr (!AX && NSEG == 1 && KLANE < 2) f(Shape<64, 64, 64, 5, 2, 2, 2, 2, false, WX, 1, KLANE, 4>());
        break;
    case RS_128x128_DEEP:
        if constexpr (!AX && NSEG == 1 && KLANE < 2) f(Shape<128, 128, 64, 4, 2, 2, 4, 2, false, WX, 1, KLANE>());
        break;
    case RS_128x128_W8:
        if constexpr (!AX && NSEG == 1) f(Shape<128, 128, 64, 2, 2, 2, 4, 4, false, WX, 1, KLANE>());
        break;
    default:
        if constexpr (AX && WX)
            f(Shape<128, 128, 32, 2, 1, 2, 2, 4, true, true, NSEG, 0>());
        else if constexpr (AX || NSEG > 1)
            f(Shape<128, 128, 64, 2, 1, 2, 2, 2, AX, WX, NSEG, 0>());
        else
            f(Shape<128, 128, 64, 2, 1, 2, 2, 2, false, WX, 1, KLANE>());
    }
}
template <bool AX, bool WX, class F>
void with_sources(const RingPlan &p, F f) {
    if (p.n_seg > 1)
        with_tile<AX, WX, kMaxSeg, 0>(p, f);
    else if (p.klane == 1)
        with_tile<AX, WX, 1, !AX ? 1 : 0>(p, f);
    else if (p.klane)
        with_tile<AX, WX, 1, !AX ? 2 : 0>(p, f);
    else
        with_tile<AX, WX, 1, 0>(p, f);
}
template <class F>
void with_shape(const RingPlan &p, F f) {
    if (p.ax && p.wx)
        with_sources<true, true>(p, f);
    else if (p.ax)
        with_sources<true, false>(p, f);
    else if (p.wx)
        with_sources<false, true>(p, f);
    else
        with_sources<false, false>(p, f);
}

// every load, fragment read and store of one kernel shape, with the kernel's own address functions
template <class T>
int64_t replay(const RingArgs<kMaxSeg> &r, const GemmArgs &g, const int64_t *a_bytes, int64_t w_bytes) {
    constexpr int BM = T::BM, BN = T::BN, BK = T::BK, kCompute = T::WVM * T::WVN, kWaves = kCompute + T::LOAD, kLoad = T::LOAD ? T::LOAD : kCompute, XM = BM / T::WVM, XN = BN / T::WVN;
    constexpr uint32_t NA = BM * BK * 2 / (1024 * kLoad), NW = BN * BK * 2 / (1024 * kLoad);
    int64_t errors = 0;
    const uint32_t grid = r.map.tiles_m * r.map.tiles_n;
    std::vector<uint8_t> written((size_t)g.M * g.N / 8, 0), seen(grid, 0);
    std::vector<int64_t> lds_a(BM * BK / 8), lds_w(BN * BK / 8);   // source element of every 16-byte slot of a stage
    for (uint32_t b = 0; b < grid; ++b) {
        uint32_t tm, tn;
        ring_tile(r.map, b, grid, tm, tn);
        if (tm >= r.map.tiles_m || tn >= r.map.tiles_n || seen[tm * r.map.tiles_n + tn]++) {
            ++errors;
            continue;
        }
        const uint32_t m0 = tm * BM, n0 = tn * BN;
        int64_t ka = 0, kw = 0;
        std::vector<uint32_t> kl(kLoad * 64 * 2), low(kl.size());   // as the kernel's kl, kl_low
        for (size_t i = 0; T::KLANE && i < kl.size(); ++i) {
            const uint32_t c8 = 8u * ring_k_chunk((uint32_t)(i / 128) * NA + (i & 1u), (uint32_t)(i / 2 % 64));
            kl[i] = 2u * (ring_digits<T::SHORT>(r.a_dk, c8) - c8);
            low[i] = c8 - fdiv(c8, r.a_dk.fext[0]) * r.a_dk.ext[0];
        }
        RingWalk ao = ring_walk_begin(r.a_steps), wo = ring_walk_begin(r.w_steps);
        uint32_t seg = 0, left = r.a[0].steps, seg_k0 = 0;
        for (uint32_t s = 0; s < r.steps; ++s) {
            if (T::NSEG > 1 && left == 0) {
                seg_k0 += r.a[seg].steps * BK;
                ++seg;
                left = r.a[seg].steps;
                ka = 0;
            }
            const RingOperand &A = r.a[seg];
            for (uint32_t wave = 0; wave < (uint32_t)kLoad; ++wave)
                for (uint32_t lane = 0; lane < 64; ++lane) {
                    const size_t at_kl = (wave * 64 + lane) * 2;
                    for (uint32_t j = 0; j < NA; ++j) {
                        const uint32_t b1 = wave * NA + j;
                        const uint32_t off = ring_block_offset<T::AX, BM, T::SHORT>(A.dx, A.base, A.kss, m0, r.M, wave * NA, j, lane) + (T::KLANE ? kl[at_kl + (j & 1u)] : 0u);
                        const int64_t at = ka - (int64_t)kRingBias + (int64_t)off + 1024 * (int64_t)(j % 4u);   // (the instruction's offset)
                        if (at < 0 || at + 16 > a_bytes[seg] || at % 16) ++errors;
                        lds_a[b1 * 64 + lane] = at / 2;
                    }
                    for (uint32_t j = 0; j < NW; ++j) {
                        const uint32_t b1 = wave * NW + j;
                        const uint32_t off = ring_block_offset<T::WX, BN, T::SHORT>(r.w.dx, r.w.base, r.w.kss, n0, r.N, wave * NW, j, lane);
                        const int64_t at = kw - (int64_t)kRingBias + (int64_t)off + 1024 * (int64_t)(j % 4u);
                        if (at < 0 || at + 16 > w_bytes || at % 16) ++errors;
                        lds_w[b1 * 64 + lane] = at / 2;
                    }
                    for (uint32_t par = 0; T::KLANE && par < 2; ++par) {
                        if (T::KLANE == 1) {
                            ring_runs_next(r.a_runs, low[at_kl + par], kl[at_kl + par]);
                        } else {
                            const uint32_t c8 = 8u * ring_k_chunk(wave * NA + par, lane);
                            kl[at_kl + par] = 2u * (ring_digits<T::SHORT>(r.a_dk, (s + 1) * BK + c8) - c8);
                        }
                    }
                }
            --left;
            if (T::NSEG > 1)
                ka += 2 * (int64_t)A.kss * BK;
            else if (!T::KLANE)
                ka += ring_walk_next(ao, r.a_steps);
            kw += ring_walk_next(wo, r.w_steps);
            // the element the map wants at (m, k) / (k, n)
            auto want_a = [&](uint32_t m, uint32_t k) -> int64_t {
                if (g.n_seg > 1) return (int64_t)(uint32_t)(g.seg_sbase[seg] + digits_offset4(g.seg_dm[seg], m) + digits_offset4(g.seg_dk[seg], k - seg_k0));
                return (int64_t)(uint32_t)(g.sbase + digits_offset4(g.dm, m) + digits_offset4(g.dk, k));
            };
            auto want_w = [&](uint32_t k, uint32_t n) -> int64_t {
                if (g.wn.n == 0) return (int64_t)k * g.N + n;   // plain row-major
                return (int64_t)(uint32_t)(g.wbase + digits_offset4(g.wk, k) + digits_offset4(g.wn, n));
            };
            for (uint32_t w2 = 0; w2 < (uint32_t)std::max(T::WVM, T::WVN); ++w2)
                for (uint32_t kk = 0; kk < BK / 16; ++kk)
                    for (uint32_t lane = 0; lane < 64; ++lane) {
                        const uint32_t gq = lane >> 4, sq = lane & 15u;
                        auto check = [&](bool x_form, uint32_t k_addr, const uint32_t *x_addr, const std::vector<int64_t> &lds, uint32_t x0, uint32_t x_lim, auto want) {
                            if (!x_form) {
                                const uint32_t x = x0 + (lane & 31u);
                                if (x < x_lim && lds[k_addr / 16] != want(x, s * BK + 16 * kk + 8 * (lane >> 5))) ++errors;
                                return;
                            }
                            for (uint32_t hi = 0; hi < 2; ++hi) {
                                const uint32_t x = x0 + 16 * (gq & 1u) + 4 * (sq & 3u), k = s * BK + 16 * kk + 8 * (gq >> 1) + (sq >> 2) + 4 * hi;
                                if (x < x_lim && lds[x_addr[hi] / 16] + (x_addr[hi] % 16) / 2 != want(x, k)) ++errors;
                            }
                        };
                        for (uint32_t f = 0; w2 < (uint32_t)T::WVM && f < XM / 32; ++f) {
                            const uint32_t xb = w2 * XM, xa[2] = {ring_x_frag<BM>(lane, xb, f, kk, 0), ring_x_frag<BM>(lane, xb, f, kk, 1)};
                            check(T::AX, ring_k_frag(lane, xb, f, kk), xa, lds_a, m0 + xb + 32 * f, r.M, want_a);
                        }
                        for (uint32_t f = 0; w2 < (uint32_t)T::WVN && f < XN / 32; ++f) {
                            const uint32_t xb = w2 * XN, xa[2] = {ring_x_frag<BN>(lane, xb, f, kk, 0), ring_x_frag<BN>(lane, xb, f, kk, 1)};
                            check(T::WX, ring_k_frag(lane, xb, f, kk), xa, lds_w, n0 + xb + 32 * f, r.N, [&](uint32_t n, uint32_t k) { return want_w(k, n); });
                        }
                    }
        }
        // the stores: the rows that a wavefront's lanes decode, then every lane of every pass
        typedef RingStore<BM, BN, kWaves> Store;
        for (uint32_t wave = 0; wave < (uint32_t)kWaves; ++wave) {
            uint32_t row_off[64] = {};
            for (uint32_t lane = 0; lane < 64 && r.store_mapped; ++lane) {
                const uint32_t m = m0 + Store::row_of_lane(wave, lane);
                row_off[lane] = ring_digits<T::SHORT>(r.om, m < r.M ? m : r.M - 1u);
            }
            for (uint32_t p = 0; p < Store::kPasses; ++p)
                for (uint32_t lane = 0; lane < 64; ++lane) {
                    const uint32_t tid = wave * 64 + lane, m = m0 + Store::row_of_store(p, tid), n = n0 + 8 * (tid % Store::kCv);
                    if (m >= r.M || n >= r.N) continue;
                    const int64_t off = r.store_mapped ? (int64_t)(uint32_t)(r.obase + ring_digits<T::SHORT>(r.on, n) + row_off[Store::lane_of_store(p, lane)])
                                                       : (int64_t)m * r.N + n;
                    const int64_t want = g.store_mapped ? (int64_t)(uint32_t)(g.obase + digits_offset4(g.om, m) + digits_offset4(g.on, n)) : (int64_t)m * g.N + n;
                    if (off != want || off % 8 || off < 0 || off + 8 > (int64_t)g.M * g.N || written[(size_t)off / 8]++) ++errors;
                }
        }
    }
    for (uint8_t w : written)
        if (w != 1) ++errors;
    return errors;
}
}  // namespace

amap_status ring_launch(const RingPlan &p, hipStream_t stream) {
    const uint32_t grid = p.args.map.tiles_m * p.args.map.tiles_n;
    amap_status st = AMAP_E_HIP;
    with_shape(p, [&](auto shape) { st = launch<decltype(shape)>(p.args, grid, stream); });
    return st;
}

int64_t ring_replay(const RingPlan &p, const GemmArgs &g, const int64_t *a_bytes, int64_t w_bytes) {
    int64_t errors = -1;
    with_shape(p, [&](auto shape) { errors = replay<decltype(shape)>(p.args, g, a_bytes, w_bytes); });
    return errors;
}

}  // namespace amap_gemm
