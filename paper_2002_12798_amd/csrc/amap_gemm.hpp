// What the GEMM kernels share: the argument block, the decoding of the operands' maps into digits, and the
// device helpers every one of them uses.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "amap_index.hpp"
#include "amap_plan.hpp"

namespace amap_gemm {

using namespace amap_dev;
using amap_detail::Piece;

constexpr int kGemmThreads = 256;
constexpr int kMaxDigits = 4;
constexpr int kMaxSeg = 8;  // sources of an A operand gathered along k

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// One dst dimension of the A map written as mixed-radix digits of its index:
// digit j = (x / mult[j]) % ext[j] contributes digit * ss[j] source elements.
struct Digits {
    uint32_t n;
    uint32_t mult[kMaxDigits], ext[kMaxDigits];
    int32_t ss[kMaxDigits];
    FastDiv fmult[kMaxDigits], fext[kMaxDigits];
};

// The k-steps of an operand of the 256 x 256-tile kernel as an odometer over the digits of k, so that the kernel
// moves from one step to the next with a few scalar additions instead of decoding k: level 0 counts the
// 64-element blocks of the contiguous lowest digit, level j >= 1 is digit j.  A step that carries into level j
// (levels below j return to 0, level j goes up by one) moves the operand's address by dl[j] bytes.
struct T2Steps {
    uint32_t e[kMaxDigits - 1];   // extents of levels 0 .. 2 (the top level ends with K)
    int64_t dl[kMaxDigits];
};

// A padded operand (Section 2.1: the load of a pad operator composed into the consumer load): the one
// data piece covers, per dimension, index lo + sum_j i_j * mult[j] with i_j < ext[j]; an index is decoded
// in the radices rad[j] = mult[j + 1] / mult[j] of the PADDED tensor and lies in the piece iff every
// digit stays below the piece's extent.  Everything else reads the pad constant.
struct PadBox {
    uint32_t lo;
    uint32_t rad[kMaxDigits];   // rad of the outermost digit: 0 = unbounded
    FastDiv frad[kMaxDigits];
};

struct GemmArgs {
    const uint16_t *A_src;
    const uint16_t *W;
    uint16_t *C;
    uint32_t M, N, K;
    uint32_t sbase;
    uint32_t tiles_m, tiles_n;
    uint32_t a_row_ss;  // tile256 kernel: source elements between consecutive m inside a 256-row tile
    int64_t a_base;     // tile256 kernel: sbase in 64 bits (its tile and k-step offsets are 64-bit: operands of 2^31 elements and more)
    uint32_t w_row_ss;  // tile256 kernel, W with runs along k (a weight kept as [N,K]): source elements between consecutive n
    T2Steps a_steps, w_steps;   // tile256 kernel: the k-steps of A (and of a W with runs along k) as odometers over the digits of k
    Digits dm, dk;
    // store side (Section 2, eq. "store"): element (m, n) of the product goes to
    // out[obase + om(m) + on(n)]; store_mapped = 0 means the plain row-major C
    uint32_t store_mapped, obase;
    uint32_t stream;    // tile256 kernel: the product goes past the caches (always but for partial tiles whose rows or runs are no whole 64-byte pieces)
    Digits om, on;
    // W read through a map as well: element (k, n) of W is W[wbase + wk(k) + wn(n)]
    uint32_t wbase;
    Digits wk, wn;
    // A gathered from several sources, one per range of k (a concat along the reduction
    // dimension that is never materialised): segment j covers k in [seg_kend[j-1], seg_kend[j])
    // and reads seg_src[j] at seg_sbase[j] + seg_dm[j](m) + seg_dk[j](k - seg_kend[j-1]).
    // n_seg <= 1: the single-source fields above are used instead.
    // A with padding: padded = 1, the data piece's box per dimension, the pad constant (two bf16 per word)
    uint32_t padded, pad_word;
    PadBox pm, pk;
    uint32_t n_seg;
    uint32_t seg_kend[kMaxSeg];
    uint32_t seg_sbase[kMaxSeg];
    const uint16_t *seg_src[kMaxSeg];
    Digits seg_dm[kMaxSeg], seg_dk[kMaxSeg];
};

// Whether the ring kernel, with A along k, stores the product past the caches (non-temporal).  Not where its rows (or a mapped store's
// runs) are no whole 64-byte pieces, which is what memory writes: a piece is then stored by two instructions, and past the caches each of
// them goes to memory by itself.  us past the caches / through them, the ring kernel: M = 126, K = 960, N = 1000 4.7 / 4.3   M = 469, K = 640
// 4.9 / 4.5   M = 16000, K = 512 24.4 / 23.1.  Beyond what the L2s hold (32 MB) lines are written back before they are whole, and past the
// caches is ahead again (M = 32192, K = 512, N = 1000 44.5 / 54.1), as it is with whole pieces at any size (M = 3000, K = 640, N = 1920
// 10.7 / 11.6; products split into heads of 32 8 % faster in the mean).
// The other kernels: the ring kernel with A along m and whole 256 x 256 tiles store past the caches, partial 256 x 256 tiles by their rows or runs
// alone, at any size (N = 1000, M = 32192, K = 512 49.2 / 41.2   M = 16000 26.0 / 22.3   N = 1024, M = 32192 37.8 / 39.1).
inline bool stores_stream(uint64_t M, uint64_t N, uint32_t run) { return run % 32 == 0 || M * N * 2 > (32u << 20); }
// f(true_type) or f(false_type), the stores past the caches or through them.  They differ in one bit of the instruction only, and the
// compiler would merge the ends of the two arms into one kind.
template <class F>
__device__ __forceinline__ void stores_by_kind(bool stream, F f) {
    if (stream) {
        f(std::true_type{});
        asm volatile("; past the caches");
    } else {
        f(std::false_type{});
    }
}
template <class STREAM>
__device__ __forceinline__ void store_c(uint16_t *at, u32x4 x, STREAM) {
    if constexpr (STREAM::value)
        __builtin_nontemporal_store(x, reinterpret_cast<u32x4 *>(at));
    else
        *reinterpret_cast<u32x4 *>(at) = x;
}

// How the W operand is fetched: plain row-major [K,N]; through a map whose
// contiguous runs lie along n (same 4 x 8 blocks, transposed in registers); or
// through a map whose runs lie along k (a transposed weight: vectors go to LDS
// as they are, like the A operand).
enum WMode { W_PLAIN = 0, W_MAPPED_N = 1, W_MAPPED_K = 2 };

// How the A operand is fetched: 16-byte runs of the source along k (vectors go to
// LDS as they are), or along m (an operand kept transposed, or a channel-major
// activation feeding a pointwise convolution: 4 k x 8 m blocks, transposed in
// registers like the W operand whose runs lie along n).
enum AMode { A_RUNS_K = 0, A_RUNS_M = 1 };

__device__ __forceinline__ uint32_t digits_offset(const Digits &d, uint32_t x) {
    uint32_t off = 0;
    for (uint32_t j = 0; j < d.n; ++j) {
        const uint32_t q = fdiv(x, d.fmult[j]);
        const uint32_t dig = q - fdiv(q, d.fext[j]) * d.ext[j];
        off += dig * (uint32_t)d.ss[j];
    }
    return off;
}

// two fp32 -> two bf16 (round to nearest even; the hardware conversion of gfx950)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;

// all digits of one dimension, fixed trip count (unused digits have extent 1 and stride 0)
__host__ __device__ __forceinline__ uint32_t digits_offset4(const Digits &d, uint32_t x) {
    uint32_t off = 0;
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
#endif
    for (uint32_t j = 0; j < (uint32_t)kMaxDigits; ++j) {
        const uint32_t q = fdiv(x, d.fmult[j]);
        const uint32_t dig = q - fdiv(q, d.fext[j]) * d.ext[j];
        off += dig * (uint32_t)d.ss[j];
    }
    return off;
}

// 16 bytes per lane from global memory straight into LDS: lane i lands at lds_base + 16 i
__device__ __forceinline__ void load_to_lds16(const void *base, uint32_t byte_off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_off), "s"(base), "s"(lds_base) : "memory");
}

// counters of levels 0 .. 2 of one operand's odometer; all 0 at the first k-step of a tile
struct T2Odo {
    uint32_t c0, c1, c2;
};
// one k-step on: the byte delta to the next step's base (not called at the last step of a tile)
__host__ __device__ __forceinline__ int64_t t2_odo_advance(T2Odo &o, const T2Steps &s) {
    if (++o.c0 < s.e[0]) return s.dl[0];
    o.c0 = 0;
    if (++o.c1 < s.e[1]) return s.dl[1];
    o.c1 = 0;
    if (++o.c2 < s.e[2]) return s.dl[2];
    o.c2 = 0;
    return s.dl[3];
}
}  // namespace amap_gemm
