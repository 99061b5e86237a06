// F-engine: channelising FFT (Section 2, Eq. 1) with a fused requantise
// epilogue that writes the X-engine's time-blocked planar spectra layout.
//
// One workgroup of TH threads (256, or 512 for some sizes)
// transforms T = TH PT / C consecutive spectra of
// one input (64 KB of complex64 voltages, one contiguous coalesced run); every
// thread holds PT = 32 complex values.  The FFT is a Stockham autosort transform
// with radices up to 32 done in registers: one pass for C <= 32, two for
// C <= 1024 (one LDS round trip), three above.  The first pass reads straight
// from global memory; the others read and write LDS rows whose index is padded
// (one slot every 16 or 32, plus a few per row, chosen per C) so that the
// strided Stockham stores and loads are free of bank conflicts.  The last pass
// maps neighbouring lanes to neighbouring spectra of one channel; its values
// are scaled by inv_s[k], rounded to the spectra element type and staged in
// LDS as [channel][spectrum][part], which turns the channel-major FFT output
// into runs of consecutive spectra per channel, parted into the (channel,
// input, plane) rows of the X-engine layout as they are stored.  From kGatherMinC channels on, a workgroup's staged output
// goes instead to a scratch buffer in workgroup order, and fgather_kernel
// assembles the rows from those pieces.
//
// Twiddles between passes are float32 values of exp(-j 2 pi m / C) computed
// in float64 on the host: log2(R) table reads per butterfly, the other powers
// as products (at most log2(R) - 1 deep).  The twiddles inside a radix-R
// butterfly are constants.  Workgroups are numbered XCD-major (each XCD takes
// a contiguous range of work items), so the workgroups that fill the same
// 128-byte spectra rows run on one XCD at about the same time and their
// partial-row stores merge in that XCD's L2.
//
// Real-input form (Section 5: 8-bit real samples, transform length 2C): the
// 2C samples of a block are read as C complex values z[n] = x[2n] + j x[2n+1]
// straight from the int8 stream, transformed by the same C-point FFT, and the
// length-2C spectrum's channels k < C are split out of it after the last
// pass (one more LDS round trip for the partner value Z[C - k]).
#include "corr_internal.h"

#include <algorithm>

namespace corr {
namespace {

constexpr int kMaxC = 8192;                       // channels, at most

// The complex FP32 form at 2048 and 4096 channels stores straight into the
// held rows (in 16-byte pieces of each) instead of through the chunked gather:
// 2048 channels from 256-thread workgroups, two per CU (1024 inputs x 512
// spectra: 5.1 ms; one 512-thread workgroup per CU with 32-byte pieces 6.4; the
// gather 7.1-7.8), 4096 channels from 512-thread ones (512 x 256: 3.8 ms; 256
// threads with 8-byte pieces 5.8; the gather 4.2).  At 8192 channels (1 or 2
// spectra per workgroup) the gather stays faster, and so it does for every
// low-precision form, whose larger workgroups measured 35-75% slower.
template <int C, int PREC, bool REAL>
constexpr bool fp32_direct() {
    return !REAL && PREC == P_FP32 && (C == 2048 || C == 4096);
}

// Threads per workgroup: 256, or 512 for the low-precision complex forms at C =
// 512 and 1024, where twice the spectra per workgroup (so half as many
// partial output rows) measured 3-10% faster on 2^28 samples for int8 and FP8
// and more for FP16 (512 inputs x 512 channels x 512 spectra 0.41 -> 0.33 ms,
// 256 x 1024 x 64 0.062 -> 0.043); at 256 channels
// they gained nothing; and for fp32_direct as said there.  From 2048 channels the
// chunked store and gather leave no partial rows to save.
template <int C, int PREC, bool REAL>
constexpr int threads() {
    if (fp32_direct<C, PREC, REAL>()) return C == 2048 ? 256 : 512;
    return (!REAL && PREC != P_FP32 && (C == 512 || C == 1024)) ? 512 : 256;
}

// Complex values per thread.  64 once paid at C >= 4096, where 32 left a
// workgroup so few spectra that its held-row stores went out in 1- to
// 4-byte pieces; with the chunked store and gather used from 2048 channels
// on, 32 (no spills) is faster at every size (4096 channels x 1024 inputs x
// 1024 FP8: 16.2 -> 14.5 ms; 8192 x 256 x 128 int8: 1.53 -> 1.15 ms).  A
// workgroup of TH threads transforms T = TH kPT / C spectra; the helpers below
// take T and TH.
constexpr int kPT = 32;

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// exp(-j 2 pi k / 32), k = 0..15.
__constant__ const float kW32[16][2] = {
    {1.000000000f, -0.000000000f},  {0.980785280f, -0.195090322f},  {0.923879533f, -0.382683432f},
    {0.831469612f, -0.555570233f},  {0.707106781f, -0.707106781f},  {0.555570233f, -0.831469612f},
    {0.382683432f, -0.923879533f},  {0.195090322f, -0.980785280f},  {0.000000000f, -1.000000000f},
    {-0.195090322f, -0.980785280f}, {-0.382683432f, -0.923879533f}, {-0.555570233f, -0.831469612f},
    {-0.707106781f, -0.707106781f}, {-0.831469612f, -0.555570233f}, {-0.923879533f, -0.382683432f},
    {-0.980785280f, -0.195090322f},
};

// x * exp(-j 2 pi k / R) for a compile-time k / R, with the trivial angles exact.
template <int R, int K>
__device__ __forceinline__ float2 rot(float2 x) {
    constexpr int k32 = K * (32 / R);                  // angle in units of 2 pi / 32, < 16
    if constexpr (k32 == 0) return x;
    else if constexpr (k32 == 8) return make_float2(x.y, -x.x);      // -j
    else return cmul(x, make_float2(kW32[k32][0], kW32[k32][1]));
}

// Forward R-point DFT in registers (R a power of two, <= 32), decimation in
// time: two R/2-point DFTs of the even and odd samples joined by W_R^k.
template <int R> struct Dft {
    template <int K = 0>
    static __device__ __forceinline__ void join(float2 *v, const float2 *e, const float2 *o) {
        if constexpr (K < R / 2) {
            const float2 t = rot<R, K>(o[K]);
            v[K] = cadd(e[K], t);
            v[K + R / 2] = csub(e[K], t);
            join<K + 1>(v, e, o);
        }
    }
    static __device__ __forceinline__ void run(float2 *v) {
        if constexpr (R == 1) {
            return;
        } else if constexpr (R == 2) {
            const float2 a = v[0], b = v[1];
            v[0] = cadd(a, b);
            v[1] = csub(a, b);
        } else {
            float2 e[R / 2], o[R / 2];
#pragma unroll
            for (int i = 0; i < R / 2; ++i) {
                e[i] = v[2 * i];
                o[i] = v[2 * i + 1];
            }
            Dft<R / 2>::run(e);
            Dft<R / 2>::run(o);
            join(v, e, o);
        }
    }
};

// Radices of the passes (product C, each <= 32) and the LDS row padding:
// element i of a row is stored at i + (i >> SH), rows are C + (C >> SH) + EX
// apart.  The paddings come from a bank-mapping simulation of every pass.
template <int C> struct Plan;
template <> struct Plan<16> { static constexpr int NP = 1, R0 = 16, R1 = 1, R2 = 1, SH = 5, EX = 0; };
template <> struct Plan<32> { static constexpr int NP = 1, R0 = 32, R1 = 1, R2 = 1, SH = 5, EX = 0; };
template <> struct Plan<64> { static constexpr int NP = 2, R0 = 8, R1 = 8, R2 = 1, SH = 5, EX = 1; };
template <> struct Plan<128> { static constexpr int NP = 2, R0 = 8, R1 = 16, R2 = 1, SH = 4, EX = 1; };
template <> struct Plan<256> { static constexpr int NP = 2, R0 = 16, R1 = 16, R2 = 1, SH = 4, EX = 1; };
template <> struct Plan<512> { static constexpr int NP = 2, R0 = 16, R1 = 32, R2 = 1, SH = 4, EX = 1; };
template <> struct Plan<1024> { static constexpr int NP = 2, R0 = 32, R1 = 32, R2 = 1, SH = 5, EX = 2; };
template <> struct Plan<2048> { static constexpr int NP = 3, R0 = 8, R1 = 16, R2 = 16, SH = 4, EX = 4; };
template <> struct Plan<4096> { static constexpr int NP = 3, R0 = 16, R1 = 16, R2 = 16, SH = 4, EX = 8; };
template <> struct Plan<8192> { static constexpr int NP = 3, R0 = 8, R1 = 32, R2 = 32, SH = 5, EX = 0; };

constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x / 2); }

// Butterfly q of thread tid in a pass of radix R maps to (spectrum t, index
// j), with b = tid + TH q (TH threads per workgroup):
//   MAP_PLAIN : (b / (C/R), b % (C/R));
//   MAP_REMAP : (b % T, b / T), the last pass, so that neighbouring lanes hold
//               neighbouring spectra of one channel;
//   MAP_PAIRED: the last pass of the real-input form when C/R >= 2 and the Q
//               butterflies of a thread are even in number: t = tid % T, and
//               with g = tid / T, G = TH / T, butterfly q < Q/2 takes
//               j = g + G q while butterfly Q-1-q takes its mirror C/R - j (C/R/2
//               in place of the mirror of j = 0), so a thread holds channel k
//               and channel C - k of the same spectrum together.
enum { MAP_PLAIN = 0, MAP_REMAP = 1, MAP_PAIRED = 2 };

template <int C, int T, int TH, int R, int MAP>
__device__ __forceinline__ void bfly_index(int tid, int q, int &t, int &j) {
    const int b = tid + TH * q;
    if constexpr (MAP == MAP_REMAP) {
        t = b % T;
        j = b / T;
    } else if constexpr (MAP == MAP_PAIRED) {
        constexpr int Q = T * C / TH / R, CR = C / R, G = TH / T;
        static_assert(T <= TH && Q % 2 == 0 && CR == G * Q, "paired mapping needs T | TH and even Q");
        t = tid % T;
        const int g = tid / T;
        if (q < Q / 2) {
            j = g + G * q;
        } else {
            const int j1 = g + G * (Q - 1 - q);
            j = j1 ? CR - j1 : CR / 2;
        }
    } else {
        t = b / (C / R);
        j = b % (C / R);
    }
}

// LDS index of element i of spectrum t (rows padded as Plan<C> says).
template <int C>
__device__ __forceinline__ int lidx(int t, int i) {
    using P = Plan<C>;
    return t * (C + (C >> P::SH) + P::EX) + i + (i >> P::SH);
}

// The same for fields that share no bits: the padding of their sum is the sum
// of their paddings.  Everything a thread reads or writes in LDS then lies at
// one place that its index gives (at) plus compile-time offsets (step), which
// are immediates of the LDS instructions; left to itself the compiler shifts
// and masks anew for each element (250-300 of the 2000 vector instructions of a
// thread at 2048 and 4096 channels).
template <int C> __device__ __forceinline__ constexpr int pad(int x) { return x + (x >> Plan<C>::SH); }
template <int C> constexpr int row_stride() { return pad<C>(C) + Plan<C>::EX; }

// Element j + r C/R of spectrum t, (t, j) = butterfly b = tid + TH q by MAP_PLAIN
// or MAP_REMAP.
template <int C, int T, int TH, int R, int MAP> struct ReadAt {
    static_assert(MAP != MAP_PAIRED, "mirrored indices are not sums");
    static __device__ __forceinline__ constexpr int t_of(int b) { return MAP == MAP_REMAP ? b % T : b / (C / R); }
    static __device__ __forceinline__ constexpr int j_of(int b) { return MAP == MAP_REMAP ? b / T : b % (C / R); }
    static __device__ __forceinline__ constexpr int at(int b) { return t_of(b) * row_stride<C>() + pad<C>(j_of(b)); }
    static __device__ __forceinline__ constexpr int step(int q, int r) { return at(TH * q) + pad<C>(r * (C / R)); }
};

// Element (j/NS) NS R + j mod NS + r NS of spectrum t, (t, j) = butterfly
// tid + TH q by MAP_PLAIN.
template <int C, int T, int TH, int R, int NS> struct WriteAt {
    static __device__ __forceinline__ constexpr int at(int b) {
        const int j = b % (C / R);
        return b / (C / R) * row_stride<C>() + pad<C>(j / NS * NS * R) + pad<C>(j % NS);
    }
    static __device__ __forceinline__ constexpr int step(int q, int r) { return at(TH * q) + pad<C>(r * NS); }
};

// First Stockham pass, radix R: butterfly (t, j) takes x[t][j + r C/R] straight
// from global memory (spectra past n_spectra read as zero) and does an R-point
// DFT; no twiddles precede the first pass.  The loads are unconditional so that
// all of a thread's loads are in flight together: a load under a branch whose
// value is converted inside it would be waited for one by one.  A padding
// spectrum reads a row of zeros with radix 8: one choice of address in place of
// one for each value (128 channels real-input int8 0.235 -> 0.227 ms, 8192 FP32
// 0.98 -> 0.89).  With radices 16 and 32 it reads spectrum 0 (which always
// exists) and zeroes what it read: without the choice between them and the
// first sums (or the conversions in its sight) the compiler joins other
// multiplications and additions there, and the spectra round otherwise.
__device__ float2 zero_row[kMaxC];                // (device globals start as zeros; never written)
template <bool> __device__ __forceinline__ float2 to_f2(float2 x) { return x; }
// Two signed bytes.  SIGNED: by conversions that take a byte with its sign as it
// is (the compiler extends each first).
template <bool SIGNED> __device__ __forceinline__ float2 to_f2(char2 x) {
    if constexpr (!SIGNED) return make_float2((float)x.x, (float)x.y);
    uint16_t u;
    __builtin_memcpy(&u, &x, 2);
    float2 f;
    asm("v_cvt_f32_i32_sdwa %0, sext(%1) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0" : "=v"(f.x) : "v"((uint32_t)u));
    asm("v_cvt_f32_i32_sdwa %0, sext(%1) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1" : "=v"(f.y) : "v"((uint32_t)u));
    return f;
}

// Load of one input element: plain, or as one 64-bit word, plain or non-temporal
// (streaming).  The word forms round alike; the compiler's choice of fused
// multiply-adds after a plain load is another at 16 and 32 channels.
enum Load { LOAD_PLAIN, LOAD_WORD, LOAD_STREAM };
template <int LD>
__device__ __forceinline__ float2 ld_in(const float2 *p) {
    if constexpr (LD != LOAD_PLAIN) {
        const unsigned long long *q = reinterpret_cast<const unsigned long long *>(p);
        const unsigned long long u = LD == LOAD_STREAM ? __builtin_nontemporal_load(q) : *q;
        float2 r;
        __builtin_memcpy(&r, &u, sizeof r);
        return r;
    } else {
        return *p;
    }
}
template <int LD>
__device__ __forceinline__ char2 ld_in(const char2 *p) {
    return *p;
}

template <int C, int T, int TH, int R, int LD, typename Src>
__device__ __forceinline__ void first_pass(float2 *v, const Src *__restrict__ src, int a0, int n_spectra,
                                           int tid) {
    constexpr int Q = T * C / TH / R, CR = C / R;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        int t, j;
        bfly_index<C, T, TH, R, MAP_PLAIN>(tid, q, t, j);
        float2 *x = v + q * R;
        constexpr bool ZEROS = R <= 8;
        const bool ok = a0 + t < n_spectra;
        const Src *row = (ok || !ZEROS ? src + (int64_t)(ok ? a0 + t : 0) * C : reinterpret_cast<const Src *>(zero_row)) + j;
        Src raw[R];
#pragma unroll
        for (int r = 0; r < R; ++r) raw[r] = ld_in<LD>(row + r * CR);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float2 f = to_f2<ZEROS>(raw[r]);
            x[r] = make_float2(ok || ZEROS ? f.x : 0.f, ok || ZEROS ? f.y : 0.f);
        }
        Dft<R>::run(x);
    }
}

// A later pass of radix R after NS points have been combined: butterfly (t, j)
// (already holding x[t][j + r C/R]) multiplies element r by
// W_C^(r (j mod NS) C/(NS R)) and does an R-point DFT.
template <int C, int T, int TH, int R, int NS, int MAP>
__device__ __forceinline__ void later_pass(float2 *v, const float2 *__restrict__ tw, int tid) {
    constexpr int Q = T * C / TH / R;
    constexpr int LR = ilog2(R);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        int t, j;
        bfly_index<C, T, TH, R, MAP>(tid, q, t, j);
        float2 *x = v + q * R;
        const int m = (j % NS) * (C / (NS * R));
        float2 wp[LR];                                 // W^(m 2^i)
#pragma unroll
        for (int i = 0; i < LR; ++i) wp[i] = tw[m << i];
        float2 w[R];
#pragma unroll
        for (int r = 1; r < R; ++r) {
            const int hb = 31 - __builtin_clz(r);
            w[r] = (r == (1 << hb)) ? wp[hb] : cmul(w[r - (1 << hb)], wp[hb]);
            x[r] = cmul(x[r], w[r]);
        }
        Dft<R>::run(x);
    }
}

// Stockham reordering between a pass (radix R1 after NS1 points) and the next
// (radix R2): butterfly (t, j) of the first writes element r to
// x[t][(j/NS1) NS1 R1 + j mod NS1 + r NS1], butterfly (t', j') of the next
// reads x[t'][j' + r C/R2].  SPLIT: the LDS holds one float per element, so
// the real parts go first and the imaginary parts second, each component read
// back taking the registers of one just written (half the LDS, so more
// workgroups per CU); otherwise whole complex values in one round.
// wait_first: the LDS may still be read by an earlier exchange.
template <int C, int T, int TH, int R1, int NS1, int R2, int MAP2, bool SPLIT>
__device__ __forceinline__ void exchange(float2 *v, float *lds, int tid, bool wait_first) {
    constexpr int PT = T * C / TH;
    constexpr int Q1 = PT / R1, Q2 = PT / R2;
    // Sums of a place and an immediate (see pad), except with whole complex
    // values in three passes, where they let the compiler join LDS reads in
    // pairs of 8 bytes, which were slower (FP32 8192 channels 1.02 -> 1.14 ms,
    // 4096 3.86 -> 4.0), and mirrored indices, which are no sums.
    constexpr bool SUMS = SPLIT || Plan<C>::NP < 3;
    using W = WriteAt<C, T, TH, R1, NS1>;
    const int w0 = W::at(tid);
    // where element (q, r) goes
    auto here = [&](int q, int r) {
        if constexpr (!SUMS) {
            int t, j;
            bfly_index<C, T, TH, R1, MAP_PLAIN>(tid, q, t, j);
            return lidx<C>(t, (j / NS1) * NS1 * R1 + (j % NS1) + r * NS1);
        } else {
            return w0 + W::step(q, r);
        }
    };
    // where the next pass's element (q, r) lies
    auto next = [&](int q, int r) {
        if constexpr (!SUMS) {
            int t, j;
            bfly_index<C, T, TH, R2, MAP2>(tid, q, t, j);
            return lidx<C>(t, j + r * (C / R2));
        } else if constexpr (MAP2 == MAP_PAIRED) {
            int t, j;
            bfly_index<C, T, TH, R2, MAP2>(tid, q, t, j);
            return lidx<C>(t, j) + pad<C>(r * (C / R2));
        } else {
            using N = ReadAt<C, T, TH, R2, MAP2>;
            return N::at(tid) + N::step(q, r);
        }
    };
    if constexpr (!SPLIT) {
        float2 *l2 = reinterpret_cast<float2 *>(lds);
        if (wait_first) __syncthreads();
#pragma unroll
        for (int q = 0; q < Q1; ++q)
#pragma unroll
            for (int r = 0; r < R1; ++r) l2[here(q, r)] = v[q * R1 + r];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q2; ++q)
#pragma unroll
            for (int r = 0; r < R2; ++r) v[q * R2 + r] = l2[next(q, r)];
        return;
    }
    float xr[PT];
#pragma unroll
    for (int comp = 0; comp < 2; ++comp) {
        if (comp == 1 || wait_first) __syncthreads();
#pragma unroll
        for (int q = 0; q < Q1; ++q)
#pragma unroll
            for (int r = 0; r < R1; ++r) lds[here(q, r)] = comp ? v[q * R1 + r].y : v[q * R1 + r].x;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q2; ++q)
#pragma unroll
            for (int r = 0; r < R2; ++r) {
                const float e = lds[next(q, r)];
                if (comp == 0) xr[q * R2 + r] = e;
                else v[q * R2 + r] = make_float2(xr[q * R2 + r], e);
            }
    }
}

// Radix, butterflies per thread and index range of the last pass of Plan<C>,
// and how the real-input form finds the partner Z[C - k] of each Z[k]: in the
// same thread (MAP_PAIRED, or C/R = 1 where every butterfly has j = 0), else
// through LDS.
template <int C> struct Last {
    using P = Plan<C>;
    static constexpr int RL = P::NP == 1 ? P::R0 : (P::NP == 2 ? P::R1 : P::R2);
    static constexpr int Q = kPT / RL, CR = C / RL;
    static constexpr bool PAIRED = CR >= 2 && Q % 2 == 0;
    static constexpr bool REAL_VIA_LDS = CR >= 2 && Q % 2 == 1;
};

// The passes of Plan<C>; v ends with the last pass's outputs in registers,
// laid out by mapping LMAP.
template <int C, int T, int TH, bool SPLIT, int LMAP, int LD, typename Src>
__device__ __forceinline__ void fft(float2 *v, float *lds, const Src *__restrict__ src, int a0, int n_spectra,
                                    const float2 *__restrict__ tw, int tid) {
    using P = Plan<C>;
    first_pass<C, T, TH, P::R0, LD>(v, src, a0, n_spectra, tid);
    if constexpr (P::NP == 2) {
        exchange<C, T, TH, P::R0, 1, P::R1, LMAP, SPLIT>(v, lds, tid, false);
        later_pass<C, T, TH, P::R1, P::R0, LMAP>(v, tw, tid);
    } else if constexpr (P::NP == 3) {
        exchange<C, T, TH, P::R0, 1, P::R1, MAP_PLAIN, SPLIT>(v, lds, tid, false);
        later_pass<C, T, TH, P::R1, P::R0, MAP_PLAIN>(v, tw, tid);
        exchange<C, T, TH, P::R1, P::R0, P::R2, LMAP, SPLIT>(v, lds, tid, true);
        later_pass<C, T, TH, P::R2, P::R0 * P::R1, LMAP>(v, tw, tid);
    }
}

// X[k] and X[C - k] of the length-2C real-input spectrum from z = Z[k],
// p = Z[C - k] of the C-point transform of z[n] = x[2n] + j x[2n+1] and
// w = W_2C^k = exp(-j pi k / C):
//   E = (z + conj p) / 2,  O = (z - conj p) / 2j,
//   X[k] = E + w O,  X[C - k] = conj(E - w O)   (W_2C^(C-k) = -conj w).
__device__ __forceinline__ void split_pair(float2 &z, float2 &p, float2 w) {
    const float er = 0.5f * (z.x + p.x), ei = 0.5f * (z.y - p.y);
    const float orr = 0.5f * (z.y + p.y), oi = 0.5f * (p.x - z.x);
    const float wr = w.x * orr - w.y * oi, wi = w.x * oi + w.y * orr;
    z = make_float2(er + wr, ei + wi);
    p = make_float2(er - wr, wi - ei);
}

// One last-pass butterfly with j = 0: u[r] = Z[r C/RL].  X[0] = Re Z[0] +
// Im Z[0] (real); X[C/2] = conj Z[C/2]; the others pair r with RL - r.
template <int C, int RL>
__device__ __forceinline__ void split_j0(float2 *u, const float2 *__restrict__ tw2) {
    constexpr int CR = C / RL;
    u[0] = make_float2(u[0].x + u[0].y, 0.f);
    if constexpr (RL >= 2) {
        u[RL / 2] = make_float2(u[RL / 2].x, -u[RL / 2].y);
#pragma unroll
        for (int r = 1; r < RL / 2; ++r) split_pair(u[r], u[RL - r], tw2[r * CR]);
    }
}

// Real-input split with every partner in the same thread (MAP_PAIRED, or
// C/R = 1).  In MAP_PAIRED butterfly q < Q/2 (index j) pairs element r with
// element RL-1-r of butterfly Q-1-q (index C/R - j); the thread with g = 0
// instead holds j = 0 in butterfly 0 and j = C/R/2 in butterfly Q-1, each
// paired with itself (r with RL - r, and r with RL-1-r).
template <int C, int T, int TH, int RL>
__device__ __forceinline__ void real_split_regs(float2 *v, const float2 *__restrict__ tw2, int tid) {
    constexpr int Q = T * C / TH / RL, CR = C / RL;
    if constexpr (CR == 1) {
#pragma unroll
        for (int q = 0; q < Q; ++q) split_j0<C, RL>(v + q * RL, tw2);
    } else {
        constexpr int G = TH / T;
        const int g = tid / T;
#pragma unroll
        for (int q = 0; q < Q / 2; ++q) {
            float2 *a = v + q * RL, *b = v + (Q - 1 - q) * RL;
            if (q == 0 && g == 0) {
                split_j0<C, RL>(a, tw2);
#pragma unroll
                for (int r = 0; r < RL / 2; ++r) split_pair(b[r], b[RL - 1 - r], tw2[CR / 2 + r * CR]);
            } else {
                const int j = g + G * q;
#pragma unroll
                for (int r = 0; r < RL; ++r) split_pair(a[r], b[RL - 1 - r], tw2[j + r * CR]);
            }
        }
    }
}

// Real-input split through LDS, for last passes whose butterflies per thread
// are odd in number (a single butterfly, so no pairing within the thread):
// with P = Z[(C - k) mod C] of the C-point transform Z of z[n] = x[2n] + j x[2n+1],
//   E = (Z[k] + conj P) / 2,  O = (Z[k] - conj P) / 2j,  X[k] = E + W_2C^k O,
// k < C, W_2C^k = exp(-j pi k / C) = tw2[k].  v holds Z[k] as the last pass
// left it (k = j + r C/RL of spectrum t, butterfly b = tid + TH q, (t, j) =
// (b % T, b / T)) and receives X[k] in the same places.  The partner values
// travel through LDS in natural [t][k] order, one component at a time when
// SPLIT.  The LDS may still be read by the last reordering on entry.
template <int C, int T, int TH, int RL, bool SPLIT>
__device__ __forceinline__ void real_split_lds(float2 *v, float *lds, const float2 *__restrict__ tw2, int tid) {
    constexpr int PT = T * C / TH;
    constexpr int Q = PT / RL, CR = C / RL;
    float pr[PT];                                      // partner real parts (SPLIT)
#pragma unroll
    for (int comp = 0; comp < (SPLIT ? 2 : 1); ++comp) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            int t, j;
            bfly_index<C, T, TH, RL, MAP_REMAP>(tid, q, t, j);
#pragma unroll
            for (int r = 0; r < RL; ++r) {
                const int i = lidx<C>(t, j + r * CR);
                if constexpr (SPLIT) lds[i] = comp ? v[q * RL + r].y : v[q * RL + r].x;
                else reinterpret_cast<float2 *>(lds)[i] = v[q * RL + r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            int t, j;
            bfly_index<C, T, TH, RL, MAP_REMAP>(tid, q, t, j);
#pragma unroll
            for (int r = 0; r < RL; ++r) {
                const int k = j + r * CR;
                const int i = lidx<C>(t, (C - k) & (C - 1));
                if (SPLIT && comp == 0) {
                    pr[q * RL + r] = lds[i];
                    continue;
                }
                float2 P;
                if constexpr (SPLIT) P = make_float2(pr[q * RL + r], lds[i]);
                else P = reinterpret_cast<const float2 *>(lds)[i];
                const float2 Z = v[q * RL + r];
                const float2 w = tw2[k];
                const float er = 0.5f * (Z.x + P.x), ei = 0.5f * (Z.y - P.y);
                const float orr = 0.5f * (Z.y + P.y), oi = 0.5f * (P.x - Z.x);
                v[q * RL + r] = make_float2(er + (w.x * orr - w.y * oi), ei + (w.x * oi + w.y * orr));
            }
        }
    }
}

// ---- requantisation --------------------------------------------------------
// Both parts of a spectrum value, scaled, as the pair of elements (re low) that
// is staged.
template <int PREC> struct Pair;
template <> struct Pair<P_FP32> {
    using T = float2;
    static constexpr int ES = 4;
    static __device__ __forceinline__ T conv(float re, float im) { return make_float2(re, im); }
};
template <> struct Pair<P_FP16> {
    using T = uint32_t;
    static constexpr int ES = 2;
    static __device__ __forceinline__ T conv(float re, float im) {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));   // RNE, saturating
        return __builtin_bit_cast(uint32_t, h2{(_Float16)fminf(fmaxf(re, -65504.0f), 65504.0f),
                                               (_Float16)fminf(fmaxf(im, -65504.0f), 65504.0f)});
    }
};
// OCP E4M3 (gfx950's FP8 format), round half to even, saturating at +-448: the
// values are clamped to the largest finite E4M3 magnitude first, so the
// hardware conversion (round to nearest even) never overflows.
template <> struct Pair<P_FP8> {
    using T = uint16_t;
    static constexpr int ES = 1;
    static __device__ __forceinline__ T conv(float re, float im) {
        re = fminf(fmaxf(re, -448.0f), 448.0f);
        im = fminf(fmaxf(im, -448.0f), 448.0f);
        return (uint16_t)__builtin_amdgcn_cvt_pk_fp8_f32(re, im, 0, false);
    }
};
// Round half to even, symmetric clamp.  Added to 1.5 * 2^23 a clamped value is
// rounded so, and the sum's low byte is the integer.
template <> struct Pair<P_INT8> {
    using T = uint16_t;
    static constexpr int ES = 1;
    static __device__ __forceinline__ uint32_t bits(float y) {
        return __float_as_uint(fminf(fmaxf(y, -127.0f), 127.0f) + 12582912.0f);
    }
    static __device__ __forceinline__ T conv(float re, float im) {
        return (uint16_t)__builtin_amdgcn_perm(bits(im), bits(re), 0x0c0c0400u);
    }
};

template <int NB> struct Bytes;
template <> struct Bytes<1> { using T = uint8_t; };
template <> struct Bytes<2> { using T = uint16_t; };
template <> struct Bytes<4> { using T = uint32_t; };
template <> struct Bytes<8> { using T = uint2; };
template <> struct Bytes<16> { using T = uint4; };

// Word d of plane pl's elements of N pairs of ES bytes each that lie in the
// words w(i): pair e (e < N) in bytes [2 ES pos(e), +2 ES) of them.
template <int ES, typename Words, typename Pos>
__device__ __forceinline__ uint32_t plane_word(const Words &w, const Pos &pos, int pl, int d) {
    if constexpr (ES == 4) {
        return w(2 * pos(d) + pl);
    } else if constexpr (ES == 2) {
        return __builtin_amdgcn_perm(w(pos(2 * d + 1)), w(pos(2 * d)), pl ? 0x07060302u : 0x05040100u);
    } else {
        const int e0 = pos(4 * d), e1 = pos(4 * d + 1), e2 = pos(4 * d + 2), e3 = pos(4 * d + 3);
        if (e0 / 2 == e1 / 2 && e2 / 2 == e3 / 2)      // (a word holds two pairs)
            return __builtin_amdgcn_perm(w(e2 / 2), w(e0 / 2), pl ? 0x07050301u : 0x06040200u);
        const uint32_t b0 = 2 * (e0 & 1) + pl, b1 = 4 + 2 * (e1 & 1) + pl, b2 = 2 * (e2 & 1) + pl,
                       b3 = 4 + 2 * (e3 & 1) + pl;
        const uint32_t lo = __builtin_amdgcn_perm(w(e1 / 2), w(e0 / 2), b0 | b1 << 8 | 0x0c0c0000u);
        const uint32_t hi = __builtin_amdgcn_perm(w(e3 / 2), w(e2 / 2), b2 | b3 << 8 | 0x0c0c0000u);
        return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
    }
}

// REAL: the input is int8 real samples (ld in bytes, block a at byte a*2C of
// its row) and tw2 holds exp(-j pi k / C); otherwise complex64 voltages (ld in
// complex samples, block a at sample a*C) and tw2 is unused.  inv_scale is
// never null (the host passes a table of ones for "no scale").
template <int C, int PREC, bool REAL>
__global__ __launch_bounds__((threads<C, PREC, REAL>())) __attribute__((amdgpu_waves_per_eu(
    PREC == P_FP32 || (REAL && Last<C>::REAL_VIA_LDS) ? 2 : 3))) void fengine_kernel(
    const void *__restrict__ in, int64_t ld, int N, int n_spectra, int n_valid_pad,
    int n_work, const float *__restrict__ inv_scale,
    const float2 *__restrict__ tw, const float2 *__restrict__ tw2, uint8_t *__restrict__ spec, int64_t k_stride,
    int64_t t_stride, int tb0, float *__restrict__ scale2) {
    using PR = Pair<PREC>;
    constexpr int TH = threads<C, PREC, REAL>();      // threads per workgroup
    constexpr int PT = kPT;
    constexpr int T = TH * PT / C;                     // spectra per workgroup
    using P = Plan<C>;
    static_assert(P::R0 * P::R1 * P::R2 == C, "radix plan must multiply to C");
    constexpr int RL = Last<C>::RL;                    // last radix
    constexpr int LMAP = REAL && Last<C>::PAIRED ? MAP_PAIRED : MAP_REMAP;
    constexpr int CP = C + (C >> P::SH) + P::EX;       // LDS row stride (floats)
    constexpr int ES = PR::ES;
    constexpr int TB = kRowBytes / ES;                 // spectra per time block
    constexpr int S = T * ES;                          // bytes of one staged row
    constexpr int CH = S < 16 ? S : 16;                // store chunk
    // The low-precision forms keep one float per element in LDS: the FFT's
    // reorderings move one component at a time, which halves the buffer so
    // three workgroups share a CU.  FP32, whose wider output staging needs the
    // registers that would allow that, keeps whole complex values (two
    // workgroups per CU, one round per reordering), and so does the
    // real-input form where the partners of its split step come through LDS.
    constexpr bool SPLIT = PREC != P_FP32 && !(REAL && Last<C>::REAL_VIA_LDS);
    // LD: int8 and FP8 read the voltages with streaming (non-temporal) loads from
    // 256 channels on (512 inputs x 256 channels x 1024 spectra int8 0.28 ms,
    // without 0.32; 512 x 512 x 512 0.31, 0.34; 512 x 1024 x 512 0.72, 0.77; above that
    // within 2%).  Below, a wave's loads of one spectrum are a few lines or part
    // of one, gone before the next load of the rest (1024 x 32 x 8192 1.14 ms,
    // without 0.54; 1024 x 64 x 4096 0.58, 0.54).  FP32 and FP16 gain nothing or lose.
    constexpr int LD = REAL || PREC == P_FP32 || PREC == P_FP16 ? LOAD_PLAIN : C >= 256 ? LOAD_STREAM : LOAD_WORD;
    // GATHER: stores go to the chunk scratch (passed as spec) in natural
    // order, [workgroup][plane][channel][spectrum], contiguous per workgroup.
    constexpr bool GATHER = C >= kGatherMinC && !fp32_direct<C, PREC, REAL>();
    static_assert(!GATHER || T <= TB, "a gathered workgroup must lie within one time block");
    constexpr int LF = SPLIT ? 1 : 2;                  // floats per LDS element
    static_assert(2 * C * S <= T * CP * 4 * LF, "staging must fit the FFT buffer");

    __shared__ __attribute__((aligned(16))) float lds[T * CP * LF];
    const int tid = threadIdx.x;

    // XCD-major work order: XCD x = blockIdx % 8 takes items [x*per, (x+1)*per).
    // Items run input-fastest within a time block, GPT workgroups per (time
    // block, input): the workgroups running together on an XCD then fill
    // whole 128-byte lines (k, tb, p) of consecutive inputs, which merge in
    // its L2 and leave it as contiguous runs.
    constexpr int GPT = TB > T ? TB / T : 1;
    const int per = (n_work + 7) / 8;
    const int w = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (w >= n_work) return;
    // the X-engine's s_k^2, written here rather than by a launch of its own
    // (2 us of each call: 16-station F + X 21.8 -> 20.3 us)
    if (scale2) for_share(w, n_work, TH, tid, C, [&](int k) { scale2[k] = square_of_scale(inv_scale[k]); });
    const int rest = w / GPT;
    const int p = rest % N;
    const int a0 = ((rest / N) * GPT + w % GPT) * T;

    float2 v[PT];
    if constexpr (REAL) {
        const char2 *src = reinterpret_cast<const char2 *>(static_cast<const int8_t *>(in) + (int64_t)p * ld);
        fft<C, T, TH, SPLIT, LMAP, LOAD_PLAIN>(v, lds, src, a0, n_spectra, tw, tid);
        if constexpr (Last<C>::REAL_VIA_LDS) real_split_lds<C, T, TH, RL, SPLIT>(v, lds, tw2, tid);
        else real_split_regs<C, T, TH, RL>(v, tw2, tid);
    } else {
        fft<C, T, TH, SPLIT, LMAP, LD>(v, lds, static_cast<const float2 *>(in) + (int64_t)p * ld, a0, n_spectra, tw,
                                   tid);
    }

    // v[q RL + r] holds channel k = j + r C/RL of spectrum t for last-pass
    // butterfly q, (t, j) as mapping LMAP gives them.  The values are requantised
    // and staged in LDS as pairs, [channel][spectrum][part]: one conversion and
    // one LDS write for both parts where they had two (2048 channels int8 5.87 ->
    // 5.72 ms with the gather, 64 channels FP32 0.29 -> 0.24, 4096 FP32 3.70 -> 3.42,
    // 8192 FP16 0.37 -> 0.33).  From there they go as runs
    // of consecutive spectra to the rows (k, tb, p, plane) at spec + tb t_stride +
    // k k_stride + p 128 + plane 64, or, for GATHER, as the staged block stands.
    constexpr int CR = C / RL;
    using PT2 = typename PR::T;
    uint8_t *stage = reinterpret_cast<uint8_t *>(lds);
    __syncthreads();                                   // every thread is done reading lds
#pragma unroll
    for (int q = 0; q < PT / RL; ++q) {
        int t, j;
        bfly_index<C, T, TH, RL, LMAP>(tid, q, t, j);
#pragma unroll
        for (int r = 0; r < RL; ++r) {
            const int k = j + r * CR;
            const float sc = inv_scale[k];
            const float2 y = v[q * RL + r];
            *reinterpret_cast<PT2 *>(stage + (k * T + t) * (2 * ES)) = PR::conv(y.x * sc, y.y * sc);
        }
    }
    __syncthreads();
    if constexpr (GATHER) {
        uint4 *dst = reinterpret_cast<uint4 *>(spec + (int64_t)w * (2 * C * S));
        for (int c = tid; c < 2 * C * S / 16; c += TH)
            if (a0 < n_valid_pad) dst[c] = reinterpret_cast<const uint4 *>(stage)[c];
    } else {
        using V = typename Bytes<CH>::T;
        constexpr int CPR = S / CH;                    // chunks per staged row
        for (int c = tid; c < C * CPR; c += TH) {
            const int k = c / CPR, a = a0 + c % CPR * (CH / ES);
            if (a >= n_valid_pad) continue;
            uint32_t u[CH / 2], o[2][CH / 4];          // CH / ES pairs; their planes
            __builtin_memcpy(u, stage + c * 2 * CH, 2 * CH);
#pragma unroll
            for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                for (int d = 0; d < CH / 4; ++d)
                    o[pl][d] = plane_word<ES>([&](int i) { return u[i]; }, [](int e) { return e; }, pl, d);
            uint8_t *dst = spec + (int64_t)(tb0 + a / TB) * t_stride + (int64_t)k * k_stride +
                           (int64_t)p * (2 * kRowBytes) + a % TB * ES;
            V x;
            __builtin_memcpy(&x, o[0], CH);
            *reinterpret_cast<V *>(dst) = x;
            __builtin_memcpy(&x, o[1], CH);
            *reinterpret_cast<V *>(dst + kRowBytes) = x;
        }
    }
}

// Second step of a gathered F-engine chunk: the scratch holds, for chunk time
// block tbl, chunk input i and piece g < GPT = TB / T, workgroup w = (tbl np + i)
// GPT + g's pairs, [channel][spectrum][part] (piece g = spectra g T .. g T + T - 1
// of the block).  A thread takes one 16-byte quarter v of both planes' 64-byte
// rows (k, tb, p) of KG neighbouring channels: 16-byte loads from each of its
// pieces, the pairs parted and put in order in registers, 16-byte stores.  Of a
// wave's lanes those of the four quarters write whole rows, and those of 16
// channel groups read 256 bytes together.  Bound: HBM.  (One channel per thread,
// so up to 16 loads of 1 to 8 bytes for each store: 2048 channels int8, 8.6 GB,
// 1.96 ms, now 1.66 = 5.2 TB/s, the copy rate; 4096 FP8 1.20 -> 0.92; 8192 FP16
// 0.24 -> 0.16.)
template <int ES, int T>
__global__ __launch_bounds__(256) void fgather_kernel(const uint8_t *__restrict__ scr, uint8_t *__restrict__ spec,
                                                      int log2c, int np, int64_t total, int64_t ks, int64_t ts,
                                                      int tb_first, int p0) {
    constexpr int PB = 2 * ES * T;                     // bytes of a piece of one channel
    constexpr int TB = kRowBytes / ES, GPT = TB / T, VE = 16 / ES;   // elements of a row, pieces, of a quarter
    constexpr int NP = VE / T > 0 ? VE / T : 1;        // pieces of a quarter
    constexpr int KG = PB < 16 ? 16 / PB : 1;          // channels
    constexpr int L = PB > 16 ? PB / 16 : 1;           // loads per piece
    static_assert(NP * T == VE, "a quarter is whole pieces");
    const int C = 1 << log2c;
    const int64_t wg_bytes = (int64_t)C * PB;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const int v = (int)(e & 3);
    const int64_t r = e >> 2;
    const int k0 = (int)(r & (C / KG - 1)) * KG;
    const int64_t r2 = r / (C / KG);
    const int i = (int)(r2 % np), tbl = (int)(r2 / np);
    const uint8_t *src = scr + ((int64_t)(tbl * np + i) * GPT + v * NP) * wg_bytes + (int64_t)k0 * PB;
    uint8_t *dst = spec + (int64_t)(tb_first + tbl) * ts + (int64_t)k0 * ks + (int64_t)(p0 + i) * (2 * kRowBytes) +
                   v * 16;
    uint4 in[NP * L];
#pragma unroll
    for (int u = 0; u < NP * L; ++u)
        in[u] = *reinterpret_cast<const uint4 *>(src + u / L * wg_bytes + u % L * 16);
    uint32_t a[NP * L * 4];
    __builtin_memcpy(a, in, sizeof a);
    const auto word = [&](int x) { return a[x]; };
#pragma unroll
    for (int g = 0; g < KG; ++g)
#pragma unroll
        for (int pl = 0; pl < 2; ++pl) {
            // element s of the quarter: pair (g, s mod T) of piece s / T
            const auto pos = [&](int s) { return s / T * (16 * L / (2 * ES)) + g * T + s % T; };
            uint4 out;
            out.x = plane_word<ES>(word, pos, pl, 0);
            out.y = plane_word<ES>(word, pos, pl, 1);
            out.z = plane_word<ES>(word, pos, pl, 2);
            out.w = plane_word<ES>(word, pos, pl, 3);
            *reinterpret_cast<uint4 *>(dst + g * ks + pl * kRowBytes) = out;
        }
}

template <int PREC, int C, bool REAL>
hipError_t launch_c(int N, const void *in, int64_t ld, int n_spectra, const float *inv_scale,
                    const float2 *tw, const float2 *tw2, void *spec, SpecLayout lay, FScratch scr, int tb0,
                    float *scale2, hipStream_t stream) {
    constexpr int TH = threads<C, PREC, REAL>();
    constexpr int T = TH * kPT / C;
    const int TB = time_block(PREC);
    const int n_tb = (n_spectra + TB - 1) / TB;
    auto run = [&](const void *src, int n_in, int ns, uint8_t *dst, int first_tb, float *s2) -> hipError_t {
        const int n_valid_pad = (ns + TB - 1) / TB * TB;
        const int groups = (n_valid_pad + T - 1) / T;
        const int64_t n_work = (int64_t)n_in * groups;
        if (n_work <= 0 || n_work > (int64_t)1 << 30) return hipErrorInvalidValue;
        const int grid = (int)((n_work + 7) / 8) * 8;
        hipLaunchKernelGGL((fengine_kernel<C, PREC, REAL>), dim3(grid), dim3(TH), 0, stream, src, ld, n_in, ns,
                           n_valid_pad, (int)n_work, inv_scale, tw, tw2, dst, lay.ks, lay.ts, first_tb, s2);
        return hipGetLastError();
    };
    if constexpr (C < kGatherMinC || fp32_direct<C, PREC, REAL>()) {
        return run(in, N, n_spectra, static_cast<uint8_t *>(spec), tb0, scale2);
    } else {
        // Chunks of whole time blocks of all inputs, or of one time block of
        // a range of inputs, each filling at most the scratch.
        constexpr int ES = Pair<PREC>::ES, KG = 2 * ES * T < 16 ? 16 / (2 * ES * T) : 1;
        const int64_t unit = (int64_t)C * 2 * kRowBytes;
        if (!scr.buf || scr.bytes < unit) return hipErrorInvalidValue;
        const int np = (int)std::min<int64_t>(N, scr.bytes / unit);
        const int ntb = np == N ? (int)std::min<int64_t>(n_tb, scr.bytes / (unit * N)) : 1;
        int log2c = 0;
        while ((1 << log2c) < C) ++log2c;
        uint8_t *sb = static_cast<uint8_t *>(scr.buf);
        for (int tbc = 0; tbc < n_tb; tbc += ntb) {
            const int s0 = tbc * TB;
            const int ns = std::min(ntb * TB, n_spectra - s0);
            const int ntb_c = (ns + TB - 1) / TB;
            for (int p0 = 0; p0 < N; p0 += np) {
                const int npc = std::min(np, N - p0);
                const void *src = REAL ? static_cast<const void *>(static_cast<const int8_t *>(in) + p0 * ld +
                                                                   (int64_t)s0 * 2 * C)
                                       : static_cast<const void *>(static_cast<const float2 *>(in) + p0 * ld +
                                                                   (int64_t)s0 * C);
                hipError_t e = run(src, npc, ns, sb, 0, tbc == 0 && p0 == 0 ? scale2 : nullptr);
                if (e != hipSuccess) return e;
                const int64_t total = (int64_t)ntb_c * npc * 4 * (C / KG);
                hipLaunchKernelGGL((fgather_kernel<ES, T>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, sb,
                                   static_cast<uint8_t *>(spec), log2c, npc, total, lay.ks, lay.ts, tb0 + tbc, p0);
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
        }
        return hipSuccess;
    }
}

template <int PREC, bool REAL>
hipError_t launch_p(int C, int N, const void *in, int64_t ld, int n_spectra, const float *inv_scale,
                    const float2 *tw, const float2 *tw2, void *spec, SpecLayout lay, FScratch scr, int tb0,
                    float *scale2, hipStream_t stream) {
#define CORR_FENGINE_CASE(c)                                                                            \
    case c: return launch_c<PREC, c, REAL>(N, in, ld, n_spectra, inv_scale, tw, tw2, spec, lay, scr, tb0, scale2, stream);
    switch (C) {
        CORR_FENGINE_CASE(16)
        CORR_FENGINE_CASE(32)
        CORR_FENGINE_CASE(64)
        CORR_FENGINE_CASE(128)
        CORR_FENGINE_CASE(256)
        CORR_FENGINE_CASE(512)
        CORR_FENGINE_CASE(1024)
        CORR_FENGINE_CASE(2048)
        CORR_FENGINE_CASE(4096)
        CORR_FENGINE_CASE(8192)
    default: return hipErrorInvalidValue;
    }
#undef CORR_FENGINE_CASE
}

template <bool REAL>
hipError_t launch_any(int prec, int C, int N, const void *in, int64_t ld, int n_spectra, const float *inv_scale,
                      const float2 *tw, const float2 *tw2, void *spec, SpecLayout lay, FScratch scr, int tb0,
                      float *scale2, hipStream_t stream) {
    switch (prec) {
    case P_FP32: return launch_p<P_FP32, REAL>(C, N, in, ld, n_spectra, inv_scale, tw, tw2, spec, lay, scr, tb0, scale2, stream);
    case P_FP16: return launch_p<P_FP16, REAL>(C, N, in, ld, n_spectra, inv_scale, tw, tw2, spec, lay, scr, tb0, scale2, stream);
    case P_FP8: return launch_p<P_FP8, REAL>(C, N, in, ld, n_spectra, inv_scale, tw, tw2, spec, lay, scr, tb0, scale2, stream);
    case P_INT8: return launch_p<P_INT8, REAL>(C, N, in, ld, n_spectra, inv_scale, tw, tw2, spec, lay, scr, tb0, scale2, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_fengine(int prec, int C, int N, const float2 *volts, int64_t ld, int n_spectra,
                          const float *inv_scale, const float2 *twiddle, void *spec, SpecLayout lay, FScratch scr,
                          int first_tb, float *scale2, hipStream_t stream) {
    return launch_any<false>(prec, C, N, volts, ld, n_spectra, inv_scale, twiddle, nullptr, spec, lay, scr, first_tb,
                             scale2, stream);
}

hipError_t launch_fengine_real8(int prec, int C, int N, const int8_t *samples, int64_t ld, int n_spectra,
                                const float *inv_scale, const float2 *twiddle, const float2 *twiddle2n, void *spec,
                                SpecLayout lay, FScratch scr, int first_tb, float *scale2, hipStream_t stream) {
    return launch_any<true>(prec, C, N, samples, ld, n_spectra, inv_scale, twiddle, twiddle2n, spec, lay, scr,
                            first_tb, scale2, stream);
}

}  // namespace corr
