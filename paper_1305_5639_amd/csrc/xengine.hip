// X-engine: the correlation of Section 2, Eq. 2, over the triangle of
// non-redundant input pairs (Section 4), as a batched Hermitian rank-A update
// on MFMA:  for each channel k,  C_k += X_k^H X_k,  X_k = [A spectra x N inputs].
//
// Complex arithmetic on real MFMA.  With x = xr + j xi,
//   Re C_ij = sum_a xr_i xr_j + xi_i xi_j
//   Im C_ij = sum_a xr_i xi_j - xi_i xr_j
// so each 32x32 output block takes four real MFMAs per K step:
//   re += Ar*Br, re += Ai*Bi, im += Ar*Bi, im += Ai*(-Br),
// where A holds rows i (the conjugated input) and B columns j.  The negated
// operand is formed in registers (sign flip for float forms, a byte-wise SWAR
// negate for int8, exact because the int8 range is symmetric).
//
// Tiling.  A workgroup owns a TILE x TILE block (rows I, columns J <= I) of
// one channel's triangle, TILE = 64 or 128.  Its waves form a 2 x (TILE / 32)
// grid: each wave owns TILE / 2 rows and one 32-column block, as 32x32 MFMA
// blocks with separate real and imaginary accumulators (TILE = 128: 8 waves of
// 64 x 32, 512 threads, for FP32 4 waves of 64 x 64; TILE = 64: 4 waves of 32 x
// 32).  FP32 is summed as three BF16 parts (below).  On diagonal blocks
// the waves whose columns lie wholly right of their rows idle, and a wave
// whose first 32 rows do skips that row block.  The K loop walks time blocks
// through a two-slot LDS ring filled by direct global-to-LDS copies
// (global_load_lds_dwordx4): each stage holds the TILE unpadded 128-byte rows
// (both planes) of each operand, with each row's 16-byte chunks XOR-swizzled
// so that 16 consecutive rows cover all 64 LDS banks.  Every lane reads 32
// bytes per (row block, plane) per stage, which is one K step for FP8
// (32x32x64), two for int8 (32x32x32) and FP16 (32x32x16), one per pair of parts
// for FP32 (32x32x16).  Because the same K assignment is used for both operands, the
// spectrum-to-slot order inside a stage does not matter.
//
// Workgroups map XCD-major (each XCD takes a contiguous range of
// (channel, block) items) so one channel's blocks share an L2.
// The epilogue scales by s_k^2 (float forms) and adds into the persistent
// lower-triangle accumulators (or writes them on the first call of an
// integration); autos get an exactly zero imaginary part, as Eq. 2 gives.
#include <algorithm>
#include <type_traits>

#include "corr_internal.h"

namespace corr {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Device-memory pointers in the global address space.  Loads and stores
// through them compile to global_* instructions even where the pointer was
// itself read from memory (a descriptor); a generic pointer would give flat_*
// instructions, which also count against the LDS wait counter and so make
// every LDS wait drain the prefetch loads as well.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const uint8_t gu8;
typedef __attribute__((address_space(1))) const u32x4 gu4;
typedef __attribute__((address_space(1))) const float gf32;

// LDS ring.  A stage is one time block of the TILE rows of both operand
// slabs: 128-byte rows (both planes), two slots.  Rows have no padding; the
// 16-byte chunk c of row r sits in slot c ^ swz(r).  A 16-byte-per-lane LDS
// read is served 16 lanes (16 consecutive rows here) per cycle from 64 banks
// of 4 bytes; swz makes those 16 rows cover all 64 banks.  A lane's fragment
// of one (row, plane) and stage is kNT = 2 chunks (32 bytes).
constexpr int kRB = 2 * kRowBytes;                     // LDS row bytes
constexpr int kCPP = kRowBytes / 16;                   // 16-byte chunks per plane
constexpr int kNT = 2;                                 // chunks per lane fragment
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }
// LDS of a block: two ring slots of 2 TILE rows, and for FP32 a word (16 bytes).
constexpr int ring_bytes(int tile) { return 2 * 2 * tile * kRB; }
constexpr int lds_bytes(int prec, int tile) { return ring_bytes(tile) + (prec == P_FP32 ? 16 : 0); }

// Per-precision fragment type and MFMA step for NT chunks per lane.  A
// fragment feeds NSUB MFMAs (sub-step e of the fragment).  The same chunk to
// K-slot assignment is used for both operands, so which spectra share an MFMA
// does not matter.
template <int PREC, int NT> struct XT;

template <int NT> struct XT<P_FP32, NT> {
    using Acc = f32x16;
    typedef float Frag __attribute__((ext_vector_type(4 * NT)));   // 4 NT spectra
    static constexpr int NSUB = 4 * NT;
    static __device__ __forceinline__ Frag load(const uint8_t *p, const int *o) {
        Frag f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const f32x4 v = *reinterpret_cast<const f32x4 *>(p + o[t]);
#pragma unroll
            for (int i = 0; i < 4; ++i) f[4 * t + i] = v[i];
        }
        return f;
    }
    static __device__ __forceinline__ Frag neg(Frag b) { return -b; }
    static __device__ __forceinline__ void mfma(Acc &c, const Frag &a, const Frag &b, int e) {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], c, 0, 0, 0);
    }
};

// FP16 and int8 share the integer fragment: NT x 16 bytes, one MFMA per chunk.
template <int PREC, int NT> struct XTInt {
    typedef int Frag __attribute__((ext_vector_type(4 * NT)));
    static constexpr int NSUB = NT;
    static __device__ __forceinline__ Frag load(const uint8_t *p, const int *o) {
        Frag f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const i32x4 v = *reinterpret_cast<const i32x4 *>(p + o[t]);
#pragma unroll
            for (int i = 0; i < 4; ++i) f[4 * t + i] = v[i];
        }
        return f;
    }
    static __device__ __forceinline__ i32x4 part(const Frag &f, int e) {
        return i32x4{f[4 * e], f[4 * e + 1], f[4 * e + 2], f[4 * e + 3]};
    }
};

template <int NT> struct XT<P_FP16, NT> : XTInt<P_FP16, NT> {
    using Acc = f32x16;
    using Frag = typename XTInt<P_FP16, NT>::Frag;
    static __device__ __forceinline__ Frag neg(Frag b) { return b ^ (int)0x80008000u; }
    static __device__ __forceinline__ void mfma(Acc &c, const Frag &a, const Frag &b, int e) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, XTInt<P_FP16, NT>::part(a, e)),
                                                   __builtin_bit_cast(f16x8, XTInt<P_FP16, NT>::part(b, e)), c, 0,
                                                   0, 0);
    }
};

template <int NT> struct XT<P_INT8, NT> : XTInt<P_INT8, NT> {
    using Acc = i32x16;
    using Frag = typename XTInt<P_INT8, NT>::Frag;
    // Byte-wise 0 - b without borrows between bytes (exact: the range is +-127).
    static __device__ __forceinline__ Frag neg(Frag b) {
        return (Frag)((0x80808080u - ((__typeof__(b))b & 0x7f7f7f7f)) ^ (~b & (int)0x80808080u));
    }
    static __device__ __forceinline__ void mfma(Acc &c, const Frag &a, const Frag &b, int e) {
        c = __builtin_amdgcn_mfma_i32_32x32x32_i8(XTInt<P_INT8, NT>::part(a, e), XTInt<P_INT8, NT>::part(b, e), c,
                                                  0, 0, 0);
    }
};

template <int NT> struct XT<P_FP8, NT> {
    static_assert(NT == 2, "the FP8 MFMA takes 32 bytes per lane");
    using Acc = f32x16;
    using Frag = i32x8;
    static constexpr int NSUB = 1;
    static __device__ __forceinline__ Frag load(const uint8_t *p, const int *o) {
        const i32x4 a = *reinterpret_cast<const i32x4 *>(p + o[0]);
        const i32x4 b = *reinterpret_cast<const i32x4 *>(p + o[1]);
        return Frag{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    }
    static __device__ __forceinline__ Frag neg(Frag b) { return b ^ (int)0x80808080u; }
    // Format code 0 = FP8 E4M3 for both operands; E8M0 scale 127 = 2^0.
    static __device__ __forceinline__ void mfma(Acc &c, const Frag &a, const Frag &b, int) {
        c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
    }
};

// Wave layout of a TILE x TILE block: WR x WC waves, each owning QS rows (FR
// blocks of 32) and QC columns (FC blocks of 32).  The FP16, FP8 and int8
// forms take narrow waves, 64 x 32 (TILE = 128, 8 waves) or 32 x 32 (TILE =
// 64, 4 waves): their complex accumulators fit 64 registers, so four waves
// share each SIMD, and while some wait at a barrier or on LDS the others issue
// MFMAs.  FP32 with TILE = 128 takes 4 waves of 64 x 64, two per SIMD: its
// fragments are split on the vector ALU after the LDS read, and a wave of
// twice the columns splits each row half as often.
template <int PREC, int TILE> struct WaveGrid {
    static constexpr int FR = TILE / 64;               // 32-row blocks per wave
    static constexpr int FC = PREC == P_FP32 ? TILE / 64 : 1;   // 32-column blocks per wave
    static constexpr int QS = 32 * FR;                 // rows per wave
    static constexpr int QC = 32 * FC;                 // columns per wave
    static constexpr int WC = TILE / QC;               // waves across the columns
    static constexpr int NW = TILE / QS * WC;          // waves
    static constexpr int THREADS = 64 * NW;
    static constexpr int EU = FR * FC > 2 ? 2 : 4;     // waves per SIMD
};

// Row blocks a wave one block wide leaves out: SKIP = 1, a diagonal wave's first,
// lying wholly above the diagonal; SKIP = 2, a last one wholly past the inputs.
// (In waves two blocks wide the branch costs more registers than there are.)
template <int FR, int SKIP> constexpr bool skipped(int f) {
    return (SKIP == 1 && f == 0) || (SKIP == 2 && f == FR - 1);
}

// One stage of a wave's FR x FC blocks of 32x32.  pa / pb point at the lane's
// row (row block 0) and column (column block 0) in the stage; off[plane][t]
// are the lane's swizzled chunk offsets in a row.  Four real products per
// block (Re += Ar Br + Ai Bi, Im += Ar Bi + Ai (-Br)).  The column fragments
// are read once, each row block's fragments just before its MFMAs, and
// (except for FP8, whose MFMA takes both chunks) one 16-byte chunk at a time,
// which keeps the live fragment registers few enough for four waves per SIMD.
// TRI: rows and columns are the same, and blocks above the diagonal are left
// out.
template <int PREC, int FR, int FC, int SKIP, bool TRI = false, typename Acc>
__device__ __forceinline__ void wave_stage(Acc (&re)[FR][FC], Acc (&im)[FR][FC], const uint8_t *pa,
                                           const uint8_t *pb, const int (&off)[2][kNT]) {
    constexpr int NC = PREC == P_FP8 ? 1 : kNT;        // chunk groups per stage
    constexpr int NTC = kNT / NC;                      // chunks per fragment
    using X = XT<PREC, NTC>;
    // The compiler's MFMA / LDS-read interleaving strategies, chosen per form
    // by measurement: FP16 at 1024 x 4096 x 1024 17.27 -> 16.54 ms and at 512 x
    // 2048 x 2048 4.24 -> 4.14 ms (strategy 0); int8 at 512 x 2048 x 2048
    // 2.44 -> 2.38 ms (strategy 1).  FP8, whose fragments take both chunks at
    // once, spills under either and keeps none.
    if constexpr (PREC == P_FP16) __builtin_amdgcn_iglp_opt(0);
    else if constexpr (PREC == P_INT8) __builtin_amdgcn_iglp_opt(1);
#pragma unroll
    for (int t = 0; t < NC; ++t) {
        typename X::Frag b0[FC], b1[FC], nb[FC];
#pragma unroll
        for (int c = 0; c < FC; ++c) {
            b0[c] = X::load(pb + c * 32 * kRB, off[0] + t * NTC);
            b1[c] = X::load(pb + c * 32 * kRB, off[1] + t * NTC);
            nb[c] = X::neg(b0[c]);
        }
#pragma unroll
        for (int f = 0; f < FR; ++f) {
            if (skipped<FR, SKIP>(f)) continue;
            const typename X::Frag a0 = TRI ? b0[f] : X::load(pa + f * 32 * kRB, off[0] + t * NTC);
            const typename X::Frag a1 = TRI ? b1[f] : X::load(pa + f * 32 * kRB, off[1] + t * NTC);
#pragma unroll
            for (int c = 0; c < FC; ++c) {
                if (TRI && c > f) continue;
#pragma unroll
                for (int e = 0; e < X::NSUB; ++e) {
                    X::mfma(re[f][c], a0, b0[c], e);   // + xr_i xr_j
                    X::mfma(im[f][c], a0, b1[c], e);   // + xr_i xi_j
                    X::mfma(re[f][c], a1, b1[c], e);   // + xi_i xi_j
                    X::mfma(im[f][c], a1, nb[c], e);   // - xi_i xr_j
                }
            }
        }
    }
}

// ---- FP32 on the BF16 matrix cores ------------------------------------------
// A float32 is the exact sum of three BF16 values (8 significand bits each,
// rounded to nearest, so the parts carry signs and all 24 bits are held).  Of
// the nine products of two such sums the six largest are formed; what is left
// out is at most 2^-24 of the product (2^-24.01 of x * x at x = 1.0038986, above
// 2^-25 for 2% of all significands), and has one sign where the inputs do not
// change.  Six 32x32x16 BF16 MFMAs (8 passes each) stand in for eight 32x32x2 FP32
// ones (16 passes each).
// Bound: the matrix cores' BF16 rate under the power limit (1024 inputs x 512
// channels x 1024 spectra: 16.6 ms = 132 TFLOP/s with FP32 MFMAs, 11.6 ms = 190
// TFLOP/s split, which is 1140 TFLOP/s of BF16 products; the BF16 library
// product reaches 1158 on this card).  Error against 64 bits, relative to the
// triangle's norm, with FP32 MFMAs and split, 130 inputs x 64 channels x
// 1024 spectra (4096; long_tile below): noise 6.2e-7 and 1.6e-7 (1.2e-6 and 1.5e-7),
// a source common to all inputs, in quadrature, 6.0e-7 and 2.9e-7 (1.2e-6 and
// 2.9e-7), a tone without noise 6.3e-7 and 4.4e-7 (1.3e-6 and 7.5e-7), constant inputs
// 1.1e-5 and 2.2e-6 (4.2e-5 and 3.9e-6).  The gain is in the sums; a product alone
// (the other spectra zero) is rounded once by an FP32 MFMA, and up to twice as far off
// here.  A launch that leaves most of the chip idle waits for the splitting in each
// time block: 130 x 130 inputs x 16 channels x 576 spectra 43.6 -> 47.2 us.
//
// The matrix cores take BF16 values and products below the normal range as
// zero, an error of 2^-126 in each of A * 24 products.  That is nothing beside
// sqrt(C_ii C_jj) where both inputs have a value of at least kLeast (2^-40) in the
// integration, or are zero.  Values above kMost have no finite parts.
constexpr float kLeast = 0x1p-40f, kMost = 0x1p127f;
// A block with a value or a sum that the split does not carry is summed again, with
// FP32 MFMAs.  The values are looked at every kLook time blocks, from the first on,
// and the split ends there (512 inputs x 512 channels x 1024 spectra, all values small
// 7.3 -> 4.8 ms, one input small 5.4 -> 3.9, an infinity in the middle 5.4 -> 4.7; usual
// data 3.0 either way, and with FP32 MFMAs in blocks of 64 alone 4.4).
constexpr int kLook = 16;
__device__ __forceinline__ bool unfit(float most) {
    return !(most <= kMost) || (most != 0.0f && most < kLeast);
}
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
struct Split {
    i32x4 p[3];                                        // 8 spectra of each part, largest first
};

typedef float f32x8 __attribute__((ext_vector_type(8)));

// The lane's 8 spectra of one (row, plane) and stage.
__device__ __forceinline__ f32x8 load8(const uint8_t *p, int o) {
    const f32x4 a = *reinterpret_cast<const f32x4 *>(p + o), b = *reinterpret_cast<const f32x4 *>(p + (o ^ 16));
    return f32x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
}

// The same, split; most: their largest magnitude so far, NaN once there is one.
__device__ __forceinline__ Split split8(f32x8 v, float &most) {
    Split s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x = v[2 * i], y = v[2 * i + 1];
        most = __builtin_elementwise_maximum(__builtin_elementwise_maximum(most, __builtin_fabsf(x)),
                                             __builtin_fabsf(y));
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const bf16x2 h{(__bf16)x, (__bf16)y};
            const uint32_t u = __builtin_bit_cast(uint32_t, h);
            s.p[q][i] = (int)u;
            if (q < 2) {
                x -= __builtin_bit_cast(float, u << 16);
                y -= __builtin_bit_cast(float, u & 0xffff0000u);
            }
        }
    }
    return s;
}

__device__ __forceinline__ void mfma_bf16(f32x16 &c, i32x4 a, i32x4 b) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                0, 0);
}

// wave_stage for FP32, split.  a / b: where in LDS the lane's first chunk of the
// real plane of its row (row block 0) and column (column block 0) is; the
// other chunks and the imaginary plane differ from it by one bit each.  The
// real sums take a stage's 16 spectra from zero, smallest products first, and
// are added to the running ones on the vector ALU: with the products going
// straight into the running sums the autos, which only grow, lost accuracy
// (1024 spectra: 1.3e-6 against 6.2e-7 with FP32 MFMAs).  The imaginary sums go
// straight in: inputs in quadrature make them grow like autos, and they then lie
// between (1024 spectra: 2.8e-7 rms, real sums 7.7e-8, FP32 MFMAs 4.3e-7).  a1 is
// negated in place for the products that enter with a minus sign.
template <int FR, int FC, bool TRI = false, typename Acc>
__device__ __forceinline__ void wave_stage_split(Acc (&re)[FR][FC], Acc (&im)[FR][FC], const uint8_t *smem, int a,
                                                 int b, float (&most)[FR + FC]) {
    // (a wave of one block, with registers to spare, reads everything at once)
    f32x8 ra0, ra1;
    if constexpr (FR * FC == 1 && !TRI) {
        ra0 = load8(smem, a);
        ra1 = load8(smem, a ^ kRowBytes);
    }
    Split b0[FC], b1[FC];
#pragma unroll
    for (int c = 0; c < FC; ++c) {
        const f32x8 r0 = load8(smem + c * 32 * kRB, b), r1 = load8(smem + c * 32 * kRB, b ^ kRowBytes);
        b0[c] = split8(r0, most[c]);
        b1[c] = split8(r1, most[c]);
    }
    constexpr int PA[6] = {0, 1, 2, 0, 1, 0}, PB[6] = {2, 1, 0, 1, 0, 0};
#pragma unroll
    for (int f = 0; f < FR; ++f) {
        if constexpr (FR * FC > 1 && !TRI) {
            ra0 = load8(smem + f * 32 * kRB, a);
            ra1 = load8(smem + f * 32 * kRB, a ^ kRowBytes);
        }
        const Split a0 = TRI ? b0[f] : split8(ra0, most[FC + f]);
        Split a1 = TRI ? b1[f] : split8(ra1, most[FC + f]);
#pragma unroll
        for (int c = 0; c < FC; ++c) {
            if (TRI && c > f) continue;
            Acc r = {0};
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                mfma_bf16(r, a1.p[PA[q]], b1[c].p[PB[q]]);             // + xi_i xi_j
                mfma_bf16(im[f][c], a0.p[PA[q]], b1[c].p[PB[q]]);      // + xr_i xi_j
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) a1.p[q] ^= (int)0x80008000u;
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                mfma_bf16(im[f][c], a1.p[PA[q]], b0[c].p[PB[q]]);      // - xi_i xr_j
                mfma_bf16(r, a0.p[PA[q]], b0[c].p[PB[q]]);             // + xr_i xr_j
            }
            if (c + 1 < FC && !(TRI && c == f))
#pragma unroll
                for (int q = 0; q < 3; ++q) a1.p[q] ^= (int)0x80008000u;
            re[f][c] += r;
        }
    }
}

// Asynchronous copy of 16 bytes per lane from global memory, base + off (base
// uniform), into LDS at lds + 16 * lane (the LDS address is taken from M0).  Issued as inline
// assembly so that the compiler, which cannot tell ring slots apart, does not
// wait for every copy in flight before each LDS read; completion is awaited
// explicitly with wait_vm.  The kernels here give the compiler no other use
// of M0.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(gu8 *base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds)
                 : "memory", "m0");
}

#pragma clang diagnostic pop

// Wait until at most n vector-memory operations of this wave are in flight.
template <int n> __device__ __forceinline__ void wait_vm() {
    static_assert(n >= 0 && n < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14));
}

// A value that is the same in every lane, kept in a scalar register (integer
// divisions run on the vector ALU and would leave it in a vector one).
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Where a block's results go.  Triangle (RECT = false): the lower-triangle
// product i(i+1)/2 + j of rows and columns below N with j <= i, B per
// channel.  Rectangle (RECT = true): rows [r0, r_end) x columns [c0, c_end),
// row-major, (i - r0) (c_end - c0) + (j - c0), B per channel; the two ranges
// do not overlap, so no pair is an auto.
struct OutMap {
    int r0, r_end, c0, c_end;
};

// The whole K loop and epilogue of one TILE x TILE block of channel k, rows
// I0.., columns J0.., by the waves of WaveGrid<PREC, TILE>.
// Time blocks stream through a two-slot LDS ring by direct global-to-LDS
// copies: the copy of time block t + 1 is issued when block t starts and
// lands while its MFMAs run.  The copies bypass registers, so the block
// keeps two workgroups per CU.  A diagonal block copies its one slab of rows
// once and reads both operands from it.  Rows past N copy row N - 1;
// they only feed outputs that are not written.  In the last time block,
// spectra past the valid count are zeroed in LDS once it lands.
template <int PREC, int TILE, bool RECT = false>
__device__ __forceinline__ void tile(uint8_t *smem, const uint8_t *__restrict__ base_k, int64_t t_stride, int N,
                                     int n_tb, int tv,
                                     int I0, int J0, int k, const float *__restrict__ scale2,
                                     void *__restrict__ acc_out, const void *acc_in, int64_t B, int first_call,
                                     int tid,
                                     OutMap om = OutMap{}) {
    constexpr int NT = kNT, RB = kRB, CPP = kCPP;
    using Acc = typename XT<PREC, NT>::Acc;
    constexpr int ES = PREC == P_FP32 ? 4 : (PREC == P_FP16 ? 2 : 1);
    constexpr int TB = kRowBytes / ES;
    using G = WaveGrid<PREC, TILE>;
    constexpr int QS = G::QS, QC = G::QC, FR = G::FR, FC = G::FC, WC = G::WC, NW = G::NW, THREADS = G::THREADS;
    constexpr int OPB = TILE * RB;                      // one operand slab of a stage
    constexpr int STG = 2 * OPB;                        // one stage
    constexpr int L = STG / (NW * 1024);                // 1 KB copies per wave per stage
    static_assert(2 * STG == ring_bytes(TILE) && L < 64 && L % 2 == 0, "ring geometry");
    const int wave = tid >> 6, lane = tid & 63;
    const int wi = wave / WC, wj = wave % WC;
    const int m = lane & 31, h = lane >> 5;
    const bool diag = !RECT && I0 == J0;
    // on a diagonal block, a wave whose columns all lie right of its rows
    // idles; one whose first 32 rows do skips that row block.  A wave whose
    // rows or columns all lie past the inputs (past the rectangle) idles; one
    // whose last 32 rows do skips that row block.
    const int rlim = RECT ? om.r_end : N, clim = RECT ? om.c_end : N;
    const bool dwave = FR > 1 && FC == 1 && diag && 32 * wj > wi * QS + 31;
    const bool lwave = FR > 1 && FC == 1 && I0 + wi * QS + (FR - 1) * 32 >= rlim;
    const bool active = !(diag && QC * wj > wi * QS + QS - 1) && I0 + wi * QS < rlim && J0 + wj * QC < clim &&
                        !(dwave && lwave);
    const int S = n_tb;                                 // stages

    // Copy j of this wave covers stage bytes [g KB, (g + 1) KB), g = NW j + wave;
    // lane l writes bytes 16 l of it: slab o, row r, slot sl, which holds
    // chunk c = sl ^ swz(r), i.e. bytes [16 (c % CPP), +16) of plane c / CPP.
    // The swizzled chunk is the same for every j: NW copies advance a multiple
    // of 16 rows.
    static_assert(NW * 1024 / RB % 16 == 0 && OPB % (NW * 1024) == 0, "copies advance whole swizzle periods");
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const uint64_t gaddr = (uint64_t)(uintptr_t)base_k;
    gu8 *const gbase = (gu8 *)(uintptr_t)((uint64_t)(uint32_t)uniform((int)(uint32_t)gaddr) |
                                          (uint64_t)(uint32_t)uniform((int)(gaddr >> 32)) << 32);
    // A diagonal block's two slabs are the same rows: it copies slab 0 only
    // (copies j < L / 2 cover stage bytes [0, OPB)) and reads both operands
    // from it.
    auto issue = [&](int t) {
        gu8 *src = gbase + (int64_t)t * t_stride;
        const uint32_t dst = lds0 + (uint32_t)((t & 1) * STG + wave * 1024);
        int x = tid;
        if constexpr (PREC == P_FP32) asm volatile("" : "+v"(x));   // (rebuild the offsets: its registers are full)
        const int r = x >> 3, c = (x & 7) ^ swz(r);
        const uint32_t col = (uint32_t)((c / CPP) * kRowBytes + (c % CPP) * 16);
#pragma unroll
        for (int j = 0; j < L; ++j) {
            if (diag && j >= L / 2) continue;
            constexpr int STEP = NW * 1024 / RB;       // rows per copy of the workgroup
            const int row = min((j < L / 2 ? I0 + j * STEP : J0 + (j - L / 2) * STEP) + r, N - 1);
            dma16(src, (uint32_t)row * RB + col,
                  __builtin_amdgcn_readfirstlane(dst + (uint32_t)(NW * j * 1024)));
        }
    };
    // Zero spectra >= tv of the landed last time block.
    auto fix_tail = [&](int t) {
        uint8_t *sm = smem + (t & 1) * STG;
        for (int q = tid; q < STG / 16; q += THREADS) {
            const int bo = q * 16, r = (bo % OPB) / RB, c = ((bo % RB) / 16) ^ swz(r);
            const int first = ((c % CPP) * 16) / ES;     // spectrum index of the chunk's first element
            if (first + 16 / ES <= tv) continue;
            uint32_t *wd = reinterpret_cast<uint32_t *>(sm + bo);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t msk = 0;
#pragma unroll
                for (int bb = 0; bb < 4; ++bb)
                    if (first + (4 * d + bb) / ES < tv) msk |= 0xffu << (8 * bb);
                wd[d] &= msk;
            }
        }
    };

    // The lane's fragment chunk offsets within a row (the rows of a fragment
    // read are m modulo 32, and swz depends on r mod 16 only).
    int off[2][NT];
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
        for (int t = 0; t < NT; ++t) off[pl][t] = 16 * ((pl * CPP + h * NT + t) ^ swz(m));

    Acc re[FR][FC], im[FR][FC];
    float most[FR + FC] = {};                          // (FP32) the lane's columns' and rows' largest values

    const uint8_t *pa0 = smem + (wi * QS + m) * RB;
    const uint8_t *pb0 = smem + (diag ? 0 : OPB) + (wj * QC + m) * RB;
    const bool tail = tv < TB;

    // (FP32) set where a wave has met a value that the split does not carry
    int *const stop = reinterpret_cast<int *>(smem + ring_bytes(TILE));
    auto met_unfit = [&] {
        bool b = false;
#pragma unroll
        for (int i = 0; i < FR + FC; ++i) b |= unfit(most[i]);
        return b;
    };

    // The sums over all stages; SPLIT (FP32): on the BF16 matrix cores, up to a value
    // that they do not carry.
    auto sum = [&](auto split) {
        constexpr bool SPLIT = decltype(split)::value;
        if (SPLIT && tid == 0) *stop = 0;              // (written again after the first barrier only)
#pragma unroll
        for (int f = 0; f < FR; ++f)
#pragma unroll
            for (int c = 0; c < FC; ++c)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    re[f][c][r] = 0;
                    im[f][c][r] = 0;
                }
        __builtin_amdgcn_s_setprio(2);                 // (see the copies in the loop)
        issue(0);
        __builtin_amdgcn_s_setprio(0);
        for (int t = 0; t < S; ++t) {
            wait_vm<0>();                               // this wave's copies of block t landed
            __syncthreads();                            // block t landed; the other slot is free
            if (SPLIT && t % kLook == 1 && uniform(*stop)) break;
            // The copies go out at a raised wave priority, ahead of the MFMAs of
            // the other waves on the SIMD (the first block's copies too: a
            // further 0.2-1%; the FP16, FP8 and int8 forms otherwise
            // unchanged within 1%).
            __builtin_amdgcn_s_setprio(2);
            if (t + 1 < S) issue(t + 1);
            __builtin_amdgcn_s_setprio(0);
            if (tail && t == S - 1) {
                fix_tail(t);
                __syncthreads();
            }
            if (!active) continue;
            const int so = (t & 1) * STG;
            // one uniform branch per stage keeps the MFMA stream branch-free
            if constexpr (SPLIT) {
                int x = tid;
                asm volatile("" : "+v"(x));            // (rebuilt, not kept: see issue)
                const int row = x & 31, w = x >> 6, chunk = 16 * ((x >> 5 & 1) * NT ^ swz(row));
                wave_stage_split<FR, FC>(re, im, smem + so, (w / WC * QS + row) * RB + chunk,
                                         (diag ? 0 : OPB) + (w % WC * QC + row) * RB + chunk, most);
                if (t % kLook == 0 && met_unfit()) *stop = 1;
            } else if constexpr (PREC == P_FP32) {
                wave_stage<PREC, FR, FC, 0>(re, im, pa0 + so, pb0 + so, off);
            } else {
                if (dwave) wave_stage<PREC, FR, FC, 1>(re, im, pa0 + so, pb0 + so, off);
                else if (PREC != P_FP8 && lwave)       // (a third FP8 body would spill)
                    wave_stage<PREC, FR, FC, 2>(re, im, pa0 + so, pb0 + so, off);
                else wave_stage<PREC, FR, FC, 0>(re, im, pa0 + so, pb0 + so, off);
            }
        }
    };
    if constexpr (PREC == P_FP32) {
        // Under one whole block of spectra there are too few roundings for the
        // split to gain accuracy (1 to 3 spectra: 5e-8 against 3e-8 to 5e-8
        // relative), and little to do: FP32 MFMAs.  They also sum a block
        // again where the split met a value it cannot carry (see kLeast), or left
        // a sum that is not finite.
        bool plain = S == 1 && tail;
        if (!plain) {
            sum(std::true_type{});
            float bad = met_unfit() ? 1.0f : 0.0f;
            if (active) {
#pragma unroll
                for (int f = 0; f < FR; ++f)
#pragma unroll
                    for (int c = 0; c < FC; ++c)
#pragma unroll
                        for (int r = 0; r < 16; ++r) bad += 0.0f * re[f][c][r] + 0.0f * im[f][c][r];
            }
            plain = __syncthreads_or(bad != 0.0f);
        }
        if (plain) sum(std::false_type{});
    } else {
        sum(std::false_type{});
    }
    // Epilogue.  Element r of a 32x32 block is (row 8(r/4) + 4h + r%4, column m).
    // The writes are streaming (non-temporal) so that they displace fewer of the
    // spectra rows other blocks still read from L2 (FP8, 1024 inputs x 4096
    // channels: 9.45 -> 9.1-9.3 ms).  Pairs outside the triangle (rectangle) or
    // past N read a valid place and are not written.  Offsets within a channel
    // fit 32 bits (N(N+1)/2 and N^2 < 2^31 for N <= 8192).
    using E = typename std::conditional<PREC == P_INT8, int, float>::type;
    typedef E T2 __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(1))) T2 gT2;
    gT2 *out = (gT2 *)acc_out + (int64_t)k * B;
    const gT2 *in = (const gT2 *)acc_in + (int64_t)k * B;   // the sums so far (== out except when dumping)
    const float s2 = (PREC != P_INT8 && scale2) ? ((gf32 *)scale2)[k] : 1.0f;
    if constexpr (TILE == 128) {
        // 128-input blocks: row block f of every wave is laid out in LDS as 64 rows
        // of TILE pairs, and the workgroup writes it from there row by row: a row's
        // places are computed once, and its 1 KB goes out as one run of 16-byte
        // stores.  Straight from the registers, as below, each pair had its place
        // computed and rows went out in runs of 256 bytes: 512 inputs x 2048
        // channels x 128 FP8 spectra 0.76 -> 0.56 ms, 1024 x 1024 x 256 1.35 -> 1.1-1.2,
        // 512 x 2048 x 32 FP32 0.99 -> 0.73; nothing where the sums take long.
        typedef E T4 __attribute__((ext_vector_type(4)));
        typedef T4 T4u __attribute__((aligned(8)));
        typedef __attribute__((address_space(1))) T4u gT4;
        static_assert(64 * TILE * sizeof(T2) <= ring_bytes(TILE) && TILE / QS == 2, "a row block of all waves fits the ring");
        T2 *const rows = reinterpret_cast<T2 *>(smem);
        constexpr int R = 64 / NW;                         // rows per wave
        const int j = J0 + 2 * lane;                       // the lane's two columns are j and j + 1
#pragma unroll
        for (int f = 0; f < FR; ++f) {
            __syncthreads();                               // the ring, or the last row block, has been read
            if (active && !(dwave && skipped<FR, 1>(f)) && !(lwave && skipped<FR, 2>(f))) {
                T2 *w = rows + (wi * 32 + 4 * h) * TILE + wj * QC + m;
#pragma unroll
                for (int c = 0; c < FC; ++c)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        w[(8 * (r >> 2) + (r & 3)) * TILE + 32 * c] = T2{re[f][c][r], im[f][c][r]};
            }
            __syncthreads();
            int o[R];
            bool one[R], two[R];                           // whether the lane's first and second pair are written
            T2 old[R][2];
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int lr = wave * R + q;
                const int i = I0 + (lr >> 5) * QS + f * 32 + (lr & 31);
                if constexpr (RECT) {
                    one[q] = i < om.r_end && j < om.c_end;
                    two[q] = i < om.r_end && j + 1 < om.c_end;
                    o[q] = (i - om.r0) * (om.c_end - om.c0) + (j - om.c0);
                } else {
                    one[q] = i < N && j <= i;
                    two[q] = i < N && j + 1 <= i;
                    o[q] = i * (i + 1) / 2 + j;
                }
            }
            if (!first_call) {
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    old[q][0] = in[one[q] ? o[q] : 0];
                    old[q][1] = in[two[q] ? o[q] + 1 : 0];
                }
            }
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int lr = wave * R + q;
                const int i = I0 + (lr >> 5) * QS + f * 32 + (lr & 31);
                T4 v = *reinterpret_cast<const T4 *>(rows + lr * TILE + 2 * lane);
                if constexpr (PREC != P_INT8) v *= s2;
                if (!RECT && i == j) v[1] = 0;             // autos
                if (!RECT && i == j + 1) v[3] = 0;
                if (!first_call) v += T4{old[q][0].x, old[q][0].y, old[q][1].x, old[q][1].y};
                if (two[q]) __builtin_nontemporal_store(v, (gT4 *)&out[o[q]]);
                else if (one[q]) __builtin_nontemporal_store(T2{v[0], v[1]}, &out[o[q]]);
            }
        }
    } else {
        // 64-input blocks, one 32x32 block a wave: from the registers (rows of
        // 512 bytes through LDS gained nothing: 200 inputs x 8192 channels x 128
        // FP8 spectra 0.43 -> 0.46-0.50 ms, 100 x 2048 x 500 FP16 0.125 -> 0.129).
        // All accumulator reads are issued before any of the writes.
        static_assert(FR * FC == 1, "one block a wave");
        if (!active) return;
        const int j = J0 + wj * QC + m;
        int idx[16];
        uint32_t ok = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = I0 + wi * QS + 8 * (r >> 2) + 4 * h + (r & 3);
            bool inside;
            int o;
            if constexpr (RECT) {
                inside = i < om.r_end && j < om.c_end;
                o = (i - om.r0) * (om.c_end - om.c0) + (j - om.c0);
            } else {
                inside = i < N && j <= i;
                o = i * (i + 1) / 2 + j;
            }
            ok |= (uint32_t)inside << r;
            idx[r] = inside ? o : 0;
        }
        T2 old[16];
        if (!first_call) {
#pragma unroll
            for (int r = 0; r < 16; ++r) old[r] = in[idx[r]];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = I0 + wi * QS + 8 * (r >> 2) + 4 * h + (r & 3);
            T2 v{re[0][0][r], im[0][0][r]};
            if constexpr (PREC != P_INT8) v *= s2;
            if (!RECT && i == j) v.y = 0;              // autos
            if (!first_call) v += old[r];
            if ((ok >> r) & 1u) __builtin_nontemporal_store(v, &out[idx[r]]);
        }
    }
}

// The same in calls longer than kSegment time blocks, FP32: piece by piece, each
// added to the sums in memory.  Running float sums take a rounding error per time
// block, and where the blocks bring nearly the same (a tone without noise) those
// errors have one sign: they grow with the blocks that one running sum takes
// (such tones, 130 inputs, error relative to the triangle's norm with FP32 MFMAs, in
// one piece and in pieces: 8192 spectra 1.8e-6, 2.9e-6, 7e-7; 2048, one piece, 8.8e-7
// and 8.0e-7).  A piece costs one more pass over the block's sums: 512 inputs x 512
// channels x 2048 spectra 6.4 ms, one piece; 256 x 1024 x 4096 7.54 ms either way.
constexpr int kSegment = 128;
template <int PREC, int TILE, bool RECT = false>
__device__ __forceinline__ void long_tile(uint8_t *smem, const uint8_t *__restrict__ base_k, int64_t t_stride, int N,
                                          int n_tb, int tv, int I0, int J0, int k, const float *__restrict__ scale2,
                                          void *__restrict__ acc_out, const void *acc_in, int64_t B, int first_call,
                                          int tid, OutMap om = OutMap{}) {
    if constexpr (PREC != P_FP32) {
        tile<PREC, TILE, RECT>(smem, base_k, t_stride, N, n_tb, tv, I0, J0, k, scale2, acc_out, acc_in, B, first_call,
                               tid, om);
    } else {
        for (int t0 = 0; t0 < n_tb; t0 += kSegment) {
            if (t0) __syncthreads();                   // every wave is done with smem
            int t = tid;
            asm volatile("" : "+v"(t));                // (the block's addresses are not kept across pieces)
            const bool last = n_tb - t0 <= kSegment;
            tile<PREC, TILE, RECT>(smem, base_k + (int64_t)t0 * t_stride, t_stride, N, last ? n_tb - t0 : kSegment,
                                   last ? tv : kRowBytes / 4, I0, J0, k, scale2, acc_out, t0 ? acc_out : acc_in, B,
                                   t0 ? 0 : first_call, t, om);
        }
    }
}

// Lower-triangle block t of a tiling with blocks (bi, bj), bj <= bi, in the
// order (0,0), (1,0), (1,1), (2,0), ...
__device__ __forceinline__ void tri_block(int t, int &bi, int &bj) {
    int b = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while (b * (b + 1) / 2 > t) --b;
    while ((b + 1) * (b + 2) / 2 <= t) ++b;
    bi = b;
    bj = t - b * (b + 1) / 2;
}

// zflag (may be null): a device flag that, when set, makes this the first
// call of an integration whatever first_call says (the accumulators of a
// batch sub-array are then logically zero, whatever they hold).
template <int PREC, int TILE>
__global__ __launch_bounds__((WaveGrid<PREC, TILE>::THREADS)) __attribute__((amdgpu_waves_per_eu((WaveGrid<PREC, TILE>::EU)))) void xengine_kernel(
    const uint8_t *__restrict__ spec, int N, int n_tiles, int n_work, int n_tb, int tv,
    int64_t k_stride, int64_t t_stride, const float *__restrict__ scale2, void *__restrict__ acc_out,
    const void *acc_in, int64_t B, int first_call, const int *__restrict__ zflag) {
    __shared__ __attribute__((aligned(16))) uint8_t smem[lds_bytes(PREC, TILE)];
    const int per = (n_work + 7) / 8;
    const int w = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (w >= n_work) return;
    const int k = uniform(w / n_tiles);
    int bi, bj;
    tri_block(w % n_tiles, bi, bj);
    bi = uniform(bi);
    bj = uniform(bj);
    const int fc = zflag && *zflag ? 1 : first_call;
    long_tile<PREC, TILE>(smem, spec + (int64_t)k * k_stride, t_stride, N, n_tb, tv, bi * TILE, bj * TILE, k, scale2,
                          acc_out, acc_in, B, fc, threadIdx.x);
}

// Small arrays, N <= 32 NB inputs (NB = 1, or 2 for FP32): one workgroup per channel,
// whose waves each take every KS-th time block of the whole triangle into
// accumulators of their own, through a two-slot ring of their own, and add them
// up through LDS at the end.  What bounds such an array is the chain of time
// blocks, each a copy's latency and a few MFMAs long: in a 64-input block one to
// three waves out of four walked all of it behind a barrier per time block.
// Bounds: copy latency (16 inputs x 64 channels x 1024 FP32 spectra: 74 -> 14 us)
// and, with many channels, the matrix cores' idle half and the copies (16 x 8192
// x 1024 int8: 95 -> 62 us, 4.3 TB/s).
template <int NB> struct SmallGrid {
    static constexpr int KS = NB == 1 ? 8 : 4;         // waves
    static constexpr int THREADS = 64 * KS;
    static constexpr int STG = NB * 32 * kRB;          // bytes of a stage
    static constexpr int L = STG / 1024;               // 1 KB copies per stage
    static constexpr int EU = NB == 1 ? 4 : 2;         // waves per SIMD (two workgroups per CU by LDS)
};

template <int PREC, int NB>
__global__ __launch_bounds__((SmallGrid<NB>::THREADS)) __attribute__((amdgpu_waves_per_eu((SmallGrid<NB>::EU)))) void xengine_small_kernel(
    const uint8_t *__restrict__ spec, int N, int C, int n_tb, int tv, int64_t k_stride, int64_t t_stride,
    const float *__restrict__ scale2, void *__restrict__ acc_out, const void *acc_in, int64_t B, int first_call,
    const int *__restrict__ zflag) {
    using G = SmallGrid<NB>;
    using Acc = typename XT<PREC, kNT>::Acc;
    using E = typename std::conditional<PREC == P_INT8, int, float>::type;
    constexpr int KS = G::KS, STG = G::STG, L = G::L;
    constexpr int ES = PREC == P_FP32 ? 4 : (PREC == P_FP16 ? 2 : 1);
    __shared__ __attribute__((aligned(16))) uint8_t smem[KS * 2 * STG];
    const int per = (C + 7) / 8;
    const int k = (blockIdx.x % 8) * per + blockIdx.x / 8;   // XCD-major
    if (k >= C) return;
    const int wave = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int m = lane & 31, h = lane >> 5;
    const int n = n_tb > wave ? (n_tb - wave + KS - 1) / KS : 0;   // this wave's time blocks
    uint8_t *const ring = smem + wave * 2 * STG;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)ring;
    gu8 *const gbase = (gu8 *)spec + (int64_t)k * k_stride;

    auto issue = [&](int i) {
        gu8 *src = gbase + (int64_t)(wave + KS * i) * t_stride;
#pragma unroll
        for (int j = 0; j < L; ++j) {
            const int r = j * 8 + (lane >> 3), c = (lane & 7) ^ swz(r);
            dma16(src, (uint32_t)(min(r, N - 1) * kRB + c * 16), uniform((int)(lds0 + (i & 1) * STG + j * 1024)));
        }
    };
    // Zero spectra >= tv of this wave's landed last time block.
    auto fix_tail = [&](int i) {
        for (int q = lane; q < STG / 16; q += 64) {
            const int r = q / (kRB / 16), c = (q % (kRB / 16)) ^ swz(r);
            const int first = (c % kCPP) * 16 / ES;
            uint32_t *wd = reinterpret_cast<uint32_t *>(ring + (i & 1) * STG + q * 16);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t msk = 0;
#pragma unroll
                for (int bb = 0; bb < 4; ++bb)
                    if (first + (4 * d + bb) / ES < tv) msk |= 0xffu << (8 * bb);
                wd[d] &= msk;
            }
        }
    };
    int off[2][kNT];
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
        for (int t = 0; t < kNT; ++t) off[pl][t] = 16 * ((pl * kCPP + h * kNT + t) ^ swz(m));

    const bool tail = tv < kRowBytes / ES;
    Acc re[NB][NB], im[NB][NB];
    float most[2 * NB] = {};
    auto met_unfit = [&] {
        bool b = false;
#pragma unroll
        for (int i = 0; i < NB; ++i) b |= unfit(most[i]);
        return b;
    };
    auto sum = [&](auto split) {
#pragma unroll
        for (int f = 0; f < NB; ++f)
#pragma unroll
            for (int c = 0; c <= f; ++c)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    re[f][c][r] = 0;
                    im[f][c][r] = 0;
                }
        if (n > 0) issue(0);
        auto block = [&](int i) {
            // the slot's last reads are done; the next block goes out before
            // this one is waited for
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (i + 1 < n) {
                issue(i + 1);
                asm volatile("s_waitcnt vmcnt(%0)" : : "n"(L) : "memory");
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            if (tail && wave + KS * i == n_tb - 1) {
                fix_tail(i);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
            const uint8_t *p = ring + (i & 1) * STG + m * kRB;
            if constexpr (decltype(split)::value)
                wave_stage_split<NB, NB, true>(re, im, p, off[0][0], off[0][0], most);
            else
                wave_stage<PREC, NB, NB, 0, true>(re, im, p, p, off);
        };
        if constexpr (decltype(split)::value) {
            // The values are looked at once, after two blocks, and by each wave for
            // itself: it sees all inputs.  Not where looking shows and there is little to
            // end: 16 inputs x 64 channels x 1024 spectra, 8 blocks a wave, F + X 18.2 ->
            // 18.3 us, and 20 x 4096 x 1024 small values 472 us without, usual data 188;
            // 48 x 4096 x 512, 8 blocks of a larger triangle, 711 without and 522.
            for (int i = 0, end = n > (NB == 1 ? 8 : 4) ? 2 : n;; end = n) {
                for (; i < end; ++i) block(i);
                if (end == n) break;
                if (__any(met_unfit())) {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the block on its way)
                    break;
                }
            }
        } else {
            for (int i = 0; i < n; ++i) block(i);
        }
    };
    if constexpr (PREC == P_FP32) {                    // (the rules of tile())
        bool plain = n_tb == 1 && tail;                // (the last piece of a long call may be that)
        if (!plain) {
            sum(std::true_type{});
            float bad = met_unfit() ? 1.0f : 0.0f;
#pragma unroll
            for (int f = 0; f < NB; ++f)
#pragma unroll
                for (int c = 0; c <= f; ++c)
#pragma unroll
                    for (int r = 0; r < 16; ++r) bad += 0.0f * re[f][c][r] + 0.0f * im[f][c][r];
            plain = __syncthreads_or(bad != 0.0f);
        }
        if (plain) sum(std::false_type{});
    } else {
        sum(std::false_type{});
    }

    // Each block's sums of all waves through LDS; wave w then adds up and
    // writes elements R w .. R w + R - 1 of it (their places as in tile()).
    constexpr int R = 16 / KS;
    static_assert(KS * 32 * 64 * 4 <= KS * 2 * STG, "the sums of a block fit the rings");
    E *const red = reinterpret_cast<E *>(smem);
    typedef E T2 __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(1))) T2 gT2;
    gT2 *out = (gT2 *)acc_out + (int64_t)k * B;
    const gT2 *in = (const gT2 *)acc_in + (int64_t)k * B;
    const float s2 = (PREC != P_INT8 && scale2) ? ((gf32 *)scale2)[k] : 1.0f;
    const bool write = (zflag && *zflag) || first_call;
#pragma unroll
    for (int f = 0; f < NB; ++f)
#pragma unroll
    for (int c = 0; c <= f; ++c) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            red[(wave * 32 + r) * 64 + lane] = re[f][c][r];
            red[(wave * 32 + 16 + r) * 64 + lane] = im[f][c][r];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int r = R * wave + q;
            const int i = 32 * f + 8 * (r >> 2) + 4 * h + (r & 3), j = 32 * c + m;
            E a = red[r * 64 + lane], b = red[(16 + r) * 64 + lane];
#pragma unroll
            for (int w = 1; w < KS; ++w) {
                a += red[(w * 32 + r) * 64 + lane];
                b += red[(w * 32 + 16 + r) * 64 + lane];
            }
            if (i < N && j <= i) {
                const int o = i * (i + 1) / 2 + j;
                T2 v;
                if constexpr (PREC == P_INT8) v = T2{a, i == j ? 0 : b};
                else v = T2{a * s2, i == j ? 0.0f : b * s2};
                if (!write) {
                    const T2 old = in[o];
                    v.x += old.x;
                    v.y += old.y;
                }
                __builtin_nontemporal_store(v, &out[o]);
            }
        }
    }
}

// Rectangle X-engine: rows [r0, r0 + ni) against columns [c0, c0 + nj) in
// TILE x TILE blocks (nbi x nbj per channel), XCD-major like xengine_kernel.
template <int PREC, int TILE>
__global__ __launch_bounds__((WaveGrid<PREC, TILE>::THREADS)) __attribute__((amdgpu_waves_per_eu((WaveGrid<PREC, TILE>::EU)))) void xengine_rect_kernel(
    const uint8_t *__restrict__ spec, int N, int nbi, int nbj, int n_work, int n_tb, int tv, int64_t k_stride,
    int64_t t_stride, const float *__restrict__ scale2, void *__restrict__ out, int64_t B, int first_call, OutMap om) {
    __shared__ __attribute__((aligned(16))) uint8_t smem[lds_bytes(PREC, TILE)];
    const int per = (n_work + 7) / 8;
    const int w = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (w >= n_work) return;
    const int nb = nbi * nbj;
    const int k = uniform(w / nb), bi = uniform((w % nb) / nbj), bj = uniform(w % nbj);
    long_tile<PREC, TILE, true>(smem, spec + (int64_t)k * k_stride, t_stride, N, n_tb, tv, om.r0 + bi * TILE,
                                om.c0 + bj * TILE, k,
                                scale2, out, out, B, first_call, threadIdx.x, om);
}

// Persistent X-engine over many sub-arrays with blocks of TILE inputs, so
// uneven sub-arrays share one launch.  Work items are (sub-array, channel,
// block); XCD x's queue holds channels [x C/8, (x+1) C/8) of every sub-array,
// so the blocks of one channel run on one XCD and share its L2.  A workgroup
// takes items from its own XCD's queue through that queue's atomic counter
// (the ticket for the next item is taken while the current one runs), and
// once it is drained from the other queues in turn; every workgroup ends
// after one failed take on each of the eight queues.  Within a queue the
// descriptors follow their sorted order (largest item first) and a workgroup
// finds its descriptor by binary search over the queue offsets.
template <int PREC, int TILE>
__global__ __launch_bounds__((WaveGrid<PREC, TILE>::THREADS)) __attribute__((amdgpu_waves_per_eu((WaveGrid<PREC, TILE>::EU)))) void xengine_batched_kernel(
    const XQueue *__restrict__ plan, const XDesc *__restrict__ all_desc, unsigned int *__restrict__ counter) {
    __shared__ __attribute__((aligned(16))) uint8_t smem[lds_bytes(PREC, TILE)];
    __shared__ unsigned int s_item;
    const int tid = threadIdx.x;
    const int n_desc = plan->n_desc;
    const XDesc *__restrict__ desc = all_desc + plan->desc_offset;
    const int home = blockIdx.x % kXcds;
    for (int s = 0; s < kXcds; ++s) {
        const int x = (home + s) % kXcds;
        unsigned int *cnt = counter + x * kCounterStride;
        const int64_t qlen = plan->qlen[x];
        if (tid == 0) s_item = atomicAdd(cnt, 1u);
        __syncthreads();
        // uniform across the workgroup: keep it (and the descriptor fields it
        // selects) in scalar registers
        int64_t item = (unsigned int)__builtin_amdgcn_readfirstlane((int)s_item);
        __syncthreads();                                // s_item free for reuse
        // the descriptor of the last item and its item range in this queue:
        // a workgroup's items rise, so most items reuse it without a search
        int cur = 0, cur_fc = 0;
        int64_t c_lo = 1, c_hi = 0;
        while (item < qlen) {
            // take the next ticket now; its latency overlaps this item's loads
            unsigned int next = 0;
            if (tid == 0) next = atomicAdd(cnt, 1u);
            if (item < c_lo || item >= c_hi) {
                int lo = 0, hi = n_desc - 1;            // last descriptor with qbegin[x] <= item
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (desc[mid].qbegin[x] <= item) lo = mid; else hi = mid - 1;
                }
                cur = lo;
                c_lo = desc[lo].qbegin[x];
                c_hi = lo + 1 < n_desc ? desc[lo + 1].qbegin[x] : qlen;
                // the sub-array's flag is cleared only after the launch, so
                // every item of it reads the same value
                const int *zf = desc[lo].zflag;
                cur_fc = zf && *(const __attribute__((address_space(1))) int *)zf ? 1 : desc[lo].first_call;
            }
            const XDesc &d = desc[cur];
            const int64_t local = item - d.qbegin[x];
            const int k = uniform(x * d.C / kXcds + (int)(local / d.n_tiles));
            int bi, bj;
            tri_block((int)(local % d.n_tiles), bi, bj);
            bi = uniform(bi);
            bj = uniform(bj);
            // an opaque copy of the thread index keeps the block body's
            // per-lane address arithmetic inside the loop instead of live
            // across it (which cost registers and occupancy)
            int t = tid;
            asm volatile("" : "+v"(t));
            long_tile<PREC, TILE>(smem, d.spec + (int64_t)k * d.k_stride, d.tb_stride, d.N, d.n_tb, d.tv, bi * TILE,
                                  bj * TILE, k,
                                  d.scale2, d.acc, d.acc, d.B, cur_fc, t);
            if (tid == 0) s_item = next;
            __syncthreads();                            // also: every wave is done with smem
            item = (unsigned int)__builtin_amdgcn_readfirstlane((int)s_item);
            __syncthreads();
        }
    }
}

__global__ void reset_counters_kernel(unsigned int *counter) { counter[threadIdx.x * kCounterStride] = 0u; }

// After a batched launch: clear the zero flag of every sub-array in the plan.
__global__ void clear_flags_kernel(const XQueue *__restrict__ plan, const XDesc *__restrict__ desc) {
    const int n = plan[0].n_desc + plan[1].n_desc;
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        if (desc[i].zflag) *desc[i].zflag = 0;
}

__global__ void set_flag_kernel(int *flag, int v) { *flag = v; }

template <int PREC, int TILE>
hipError_t launch_x(int C, int N, int n_spectra, const void *spec, SpecLayout lay,
                    const float *scale2, void *acc, const void *acc_in, int first_call, const int *zflag,
                    hipStream_t stream) {
    const int TB = time_block(PREC);
    const int n_tb = (n_spectra + TB - 1) / TB;
    const int tv = n_spectra - (n_tb - 1) * TB;
    const int n_blk = (N + TILE - 1) / TILE;
    const int n_tiles = n_blk * (n_blk + 1) / 2;
    const int64_t n_work = (int64_t)C * n_tiles;
    if (n_tb <= 0 || n_work <= 0 || n_work > ((int64_t)1 << 30)) return hipErrorInvalidValue;
    const int grid = (int)((n_work + 7) / 8) * 8;
    const int64_t B = (int64_t)N * (N + 1) / 2;
    hipLaunchKernelGGL((xengine_kernel<PREC, TILE>), dim3(grid), dim3(WaveGrid<PREC, TILE>::THREADS), 0, stream,
                       static_cast<const uint8_t *>(spec), N, n_tiles, (int)n_work, n_tb, tv, lay.ks, lay.ts,
                       scale2, acc, acc_in, B, first_call, zflag);
    return hipGetLastError();
}

template <int PREC, int NB>
hipError_t launch_small(int C, int N, int n_spectra, const void *spec, SpecLayout lay, const float *scale2, void *acc,
                        const void *acc_in, int first_call, const int *zflag, hipStream_t stream) {
    const int TB = time_block(PREC);
    const int n_tb = (n_spectra + TB - 1) / TB;
    const int tv = n_spectra - (n_tb - 1) * TB;
    if (n_tb <= 0 || C <= 0 || N < 1 || N > 32 * NB) return hipErrorInvalidValue;
    // FP32: in pieces like long_tile(), kSegment time blocks to a wave, each a launch
    // (in one launch their loop cost the kernel 4%: 20 inputs x 1024 channels x 4096
    // spectra 0.182 -> 0.189 ms)
    const int piece = PREC == P_FP32 ? kSegment * SmallGrid<NB>::KS : n_tb;
    for (int t0 = 0; t0 < n_tb; t0 += piece) {
        const bool last = n_tb - t0 <= piece;
        hipLaunchKernelGGL((xengine_small_kernel<PREC, NB>), dim3((C + 7) / 8 * 8), dim3(SmallGrid<NB>::THREADS), 0,
                           stream, static_cast<const uint8_t *>(spec) + t0 * lay.ts, N, C, last ? n_tb - t0 : piece,
                           last ? tv : TB, lay.ks, lay.ts, scale2, acc, t0 ? acc : acc_in, (int64_t)N * (N + 1) / 2,
                           t0 ? 0 : first_call, t0 ? nullptr : zflag);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int PREC>
hipError_t launch_xp(int tile, int C, int N, int n_spectra, const void *spec, SpecLayout lay,
                     const float *scale2, void *acc, const void *acc_in, int first_call, const int *zflag,
                     hipStream_t stream) {
    // The small kernel from as many time blocks as its split of them gains from
    // (its reduction costs the same whatever their number): FP32, whose blocks
    // take longest, 32 inputs x 8192 channels: 2 blocks 59 -> 54 us, 4 blocks 92 ->
    // 61, 16 blocks 270 -> 148; FP16 6 blocks 54 -> 47, 8 blocks 73 -> 58, int8 8
    // blocks 76 -> 61, but int8 2 blocks 33 -> 38.  Over 32 inputs FP32 alone: 64 x
    // 4096 channels, 4 blocks 84 -> 64 us, 32 blocks 517 -> 325; FP16 64 x 2048, 32
    // blocks, 104 -> 112.
    const int n_tb = (n_spectra + time_block(PREC) - 1) / time_block(PREC);
    if (tile == 64 && N <= 32 && n_tb >= (PREC == P_FP32 ? 4 : 6))
        return launch_small<PREC, 1>(C, N, n_spectra, spec, lay, scale2, acc, acc_in, first_call, zflag, stream);
    if constexpr (PREC == P_FP32)
        if (tile == 64 && N <= 64 && n_tb >= 4)
            return launch_small<PREC, 2>(C, N, n_spectra, spec, lay, scale2, acc, acc_in, first_call, zflag, stream);
    if (tile == 64)
        return launch_x<PREC, 64>(C, N, n_spectra, spec, lay, scale2, acc, acc_in, first_call, zflag, stream);
    if (tile == 128)
        return launch_x<PREC, 128>(C, N, n_spectra, spec, lay, scale2, acc, acc_in, first_call, zflag, stream);
    return hipErrorInvalidValue;
}

}  // namespace

template <int PREC, int TILE>
hipError_t launch_rect_t(int C, int N, int n_spectra, const void *spec, SpecLayout lay, const float *scale2,
                         void *out, int first_call, int r0, int ni, int c0, int nj,
                         hipStream_t stream) {
    const int TB = time_block(PREC);
    const int n_tb = (n_spectra + TB - 1) / TB;
    const int tv = n_spectra - (n_tb - 1) * TB;
    const int nbi = (ni + TILE - 1) / TILE, nbj = (nj + TILE - 1) / TILE;
    const int64_t n_work = (int64_t)C * nbi * nbj;
    if (n_tb <= 0 || n_work <= 0 || n_work > ((int64_t)1 << 30) || r0 < 0 || c0 < 0 || r0 + ni > N || c0 + nj > N)
        return hipErrorInvalidValue;
    const int grid = (int)((n_work + 7) / 8) * 8;
    hipLaunchKernelGGL((xengine_rect_kernel<PREC, TILE>), dim3(grid), dim3(WaveGrid<PREC, TILE>::THREADS), 0, stream,
                       static_cast<const uint8_t *>(spec), N, nbi, nbj, (int)n_work, n_tb, tv,
                       lay.ks, lay.ts, scale2, out, (int64_t)ni * nj, first_call,
                       OutMap{r0, r0 + ni, c0, c0 + nj});
    return hipGetLastError();
}

template <int PREC>
hipError_t launch_rect_p(int tile, int C, int N, int n_spectra, const void *spec, SpecLayout lay,
                         const float *scale2, void *out, int first_call, int r0, int ni, int c0, int nj,
                         hipStream_t stream) {
    if (tile == 64)
        return launch_rect_t<PREC, 64>(C, N, n_spectra, spec, lay, scale2, out, first_call, r0, ni, c0, nj, stream);
    if (tile == 128)
        return launch_rect_t<PREC, 128>(C, N, n_spectra, spec, lay, scale2, out, first_call, r0, ni, c0, nj, stream);
    return hipErrorInvalidValue;
}

hipError_t launch_xengine_rect(int prec, int tile, int C, int N, int n_spectra, const void *spec, SpecLayout lay,
                               const float *scale2, void *out, int first_call, int r0, int ni, int c0, int nj,
                               hipStream_t stream) {
    switch (prec) {
    case P_FP32: return launch_rect_p<P_FP32>(tile, C, N, n_spectra, spec, lay, scale2, out, first_call, r0, ni, c0, nj, stream);
    case P_FP16: return launch_rect_p<P_FP16>(tile, C, N, n_spectra, spec, lay, scale2, out, first_call, r0, ni, c0, nj, stream);
    case P_FP8: return launch_rect_p<P_FP8>(tile, C, N, n_spectra, spec, lay, scale2, out, first_call, r0, ni, c0, nj, stream);
    case P_INT8: return launch_rect_p<P_INT8>(tile, C, N, n_spectra, spec, lay, scale2, out, first_call, r0, ni, c0, nj, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_xengine(int prec, int tile, int C, int N, int n_spectra, const void *spec, SpecLayout lay,
                          const float *scale2, void *acc, const void *acc_in, int first_call, hipStream_t stream,
                          const int *zflag) {
#define CORR_X_ARGS tile, C, N, n_spectra, spec, lay, scale2, acc, acc_in, first_call, zflag, stream
    switch (prec) {
    case P_FP32: return launch_xp<P_FP32>(CORR_X_ARGS);
    case P_FP16: return launch_xp<P_FP16>(CORR_X_ARGS);
    case P_FP8: return launch_xp<P_FP8>(CORR_X_ARGS);
    case P_INT8: return launch_xp<P_INT8>(CORR_X_ARGS);
#undef CORR_X_ARGS
    default: return hipErrorInvalidValue;
    }
}

template <int PREC, int TILE>
hipError_t launch_batched_t(const XQueue *d_plan, const XDesc *d_desc, unsigned int *counter, int grid,
                            hipStream_t stream) {
    hipLaunchKernelGGL((xengine_batched_kernel<PREC, TILE>), dim3(grid), dim3(WaveGrid<PREC, TILE>::THREADS), 0, stream, d_plan, d_desc,
                       counter);
    return hipGetLastError();
}

template <int TILE>
hipError_t launch_batched_p(int prec, const XQueue *d_plan, const XDesc *d_desc, unsigned int *counter, int grid,
                            hipStream_t stream) {
    switch (prec) {
    case P_FP32: return launch_batched_t<P_FP32, TILE>(d_plan, d_desc, counter, grid, stream);
    case P_FP16: return launch_batched_t<P_FP16, TILE>(d_plan, d_desc, counter, grid, stream);
    case P_FP8: return launch_batched_t<P_FP8, TILE>(d_plan, d_desc, counter, grid, stream);
    case P_INT8: return launch_batched_t<P_INT8, TILE>(d_plan, d_desc, counter, grid, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_xengine_batched(int prec, const XQueue *d_plan, const XDesc *d_desc, int launch_group,
                                  unsigned int *counters, int num_cus, hipStream_t stream) {
    if (num_cus <= 0 || (launch_group & ~3)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(reset_counters_kernel, dim3(1), dim3(2 * kXcds), 0, stream, counters);
    hipError_t e = hipGetLastError();
    // 128-input blocks first (the larger items), two workgroups per CU; then
    // 64-input blocks, four workgroups per CU.
    // (grids rounded to a multiple of the XCD count, as the kernel assumes)
    const int g128 = std::max(kXcds, 2 * num_cus / kXcds * kXcds), g64 = std::max(kXcds, 4 * num_cus / kXcds * kXcds);
    if (e == hipSuccess && (launch_group & 2))
        e = launch_batched_p<128>(prec, d_plan + 1, d_desc, counters + kXcds * kCounterStride, g128, stream);
    if (e == hipSuccess && (launch_group & 1))
        e = launch_batched_p<64>(prec, d_plan, d_desc, counters, g64, stream);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(256), 0, stream, d_plan, d_desc);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_set_flag(int *flag, int v, hipStream_t stream) {
    hipLaunchKernelGGL(set_flag_kernel, dim3(1), dim3(1), 0, stream, flag, v);
    return hipGetLastError();
}

}  // namespace corr
