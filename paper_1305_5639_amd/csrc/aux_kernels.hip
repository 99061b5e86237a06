// Data-movement kernels around the two engines: caller spectra in and out of
// the time-blocked planar layout, dump layout/order conversion and a zero fill.  None of these is on the F -> X hot path; the
// spectra moves are LDS-tiled transposes, the rest coalesced element maps.
#include "corr_internal.h"

namespace corr {
namespace {

constexpr int kThreads = 256;


// Caller spectra <-> held rows.  For channel k and time block tb, the TB
// public rows a = tb*TB + t hold the 2N columns (2p + plane) of that channel
// contiguously; the held layout wants each column's TB values contiguous (one
// 64-byte plane row).  That is a TB x 2N transpose per (k, tb).  One
// workgroup moves a tile of kCols columns: TB public segments of kCols * ES
// bytes <-> kCols held rows of 64 bytes, 16 KB either way, through LDS.  Both
// sides move 16-byte vectors; the LDS row of public row t stores its 16-byte
// chunks XOR-swizzled by the held vector t falls in, so the gathers of one
// wave (16 columns x 4 held vectors) hit distinct banks.
constexpr int kCols = 256;

template <typename T>
__device__ __forceinline__ int lds_elem(int t, int j) {
    constexpr int ES = (int)sizeof(T), VE = 16 / ES, W = kCols * ES;
    const int byte = j * ES, chunk = byte >> 4;
    const int tg = (t / VE) & 3;
    return t * W + ((chunk ^ (tg * ES)) << 4) + (byte & 15);
}

// Byte-wise max(b, -127) of four int8 values: a byte equal to 0x80 (-128)
// becomes 0x81 (-127), every other byte is unchanged.  x marks the -128 bytes
// as zero bytes; the zero-byte test below is exact (no borrow between bytes).
__device__ __forceinline__ uint32_t sat_int8x4(uint32_t v) {
    const uint32_t x = v ^ 0x80808080u;
    const uint32_t nz = ((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x;
    return v | ((~nz & 0x80808080u) >> 7);
}

// INGEST: public src -> held dst (the tail of the last block zero-filled);
// else held src -> public dst.  VEC: public rows 16-byte aligned (2N * ES a
// multiple of 16, base aligned), so public segments move as vectors.  SAT8
// (int8 ingest): -128 is read as -127, the symmetric range the X-engine's
// exact negation and the int32 overflow bound assume.
template <typename T, bool INGEST, bool VEC, bool SAT8 = false>
__global__ __launch_bounds__(kThreads) void relayout_kernel(const uint8_t *__restrict__ src,
                                                             uint8_t *__restrict__ dst, int C, int N,
                                                             int n_spectra, int n_tb, int n_cc, SpecLayout lay,
                                                             UserScale us) {
    constexpr int ES = (int)sizeof(T), TB = kRowBytes / ES, VE = 16 / ES, W = kCols * ES;
    constexpr int PUB_VECS = TB * (W / 16);             // 1024 either side
    __shared__ __align__(16) uint8_t lds[TB * W];
    const int64_t g = blockIdx.x;
    const int cc = (int)(g % n_cc);
    const int tb = (int)((g / n_cc) % n_tb);
    const int k = (int)(g / ((int64_t)n_cc * n_tb));
    const int cols = 2 * N, c_base = cc * kCols;
    const int64_t pub_row = (int64_t)cols * ES;         // bytes per public (a, k) row
    uint8_t *held = (INGEST ? dst : const_cast<uint8_t *>(src)) + (int64_t)tb * lay.ts + (int64_t)k * lay.ks;

    auto pub_addr = [&](int t, int col) -> int64_t {
        return ((int64_t)(tb * TB + t) * C + k) * pub_row + (int64_t)col * ES;
    };
    if (INGEST) {
        if (us.scale2)
            for (int64_t c = g * kThreads + threadIdx.x; c < us.C; c += (int64_t)gridDim.x * kThreads)
                us.scale2[c] = us.inv ? square_of_scale(us.inv[c]) : 1.0f;
        for (int i = threadIdx.x; i < PUB_VECS; i += kThreads) {
            const int t = i / (W / 16), c = i % (W / 16);
            const int a = tb * TB + t, col0 = c_base + c * VE;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (a < n_spectra && col0 < cols) {
                if (VEC && col0 + VE <= cols) {
                    v = *reinterpret_cast<const uint4 *>(src + pub_addr(t, col0));
                } else {
                    T e[VE];
                    for (int u = 0; u < VE; ++u)
                        e[u] = col0 + u < cols ? *reinterpret_cast<const T *>(src + pub_addr(t, col0 + u)) : T(0);
                    __builtin_memcpy(&v, e, 16);
                }
            }
            if constexpr (SAT8) {
                v.x = sat_int8x4(v.x);
                v.y = sat_int8x4(v.y);
                v.z = sat_int8x4(v.z);
                v.w = sat_int8x4(v.w);
            }
            *reinterpret_cast<uint4 *>(lds + lds_elem<T>(t, c * VE)) = v;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < kCols * 4; i += kThreads) {
            const int j = i >> 2, hv = i & 3, col = c_base + j;
            if (col >= cols) continue;
            T e[VE];
            for (int u = 0; u < VE; ++u) e[u] = *reinterpret_cast<const T *>(lds + lds_elem<T>(hv * VE + u, j));
            uint4 v;
            __builtin_memcpy(&v, e, 16);
            *reinterpret_cast<uint4 *>(held + (int64_t)col * kRowBytes + hv * 16) = v;
        }
    } else {
        for (int i = threadIdx.x; i < kCols * 4; i += kThreads) {
            const int j = i >> 2, hv = i & 3, col = c_base + j;
            if (col >= cols) continue;
            const uint4 v = *reinterpret_cast<const uint4 *>(held + (int64_t)col * kRowBytes + hv * 16);
            T e[VE];
            __builtin_memcpy(e, &v, 16);
            for (int u = 0; u < VE; ++u) *reinterpret_cast<T *>(lds + lds_elem<T>(hv * VE + u, j)) = e[u];
        }
        __syncthreads();
        for (int i = threadIdx.x; i < PUB_VECS; i += kThreads) {
            const int t = i / (W / 16), c = i % (W / 16);
            const int a = tb * TB + t, col0 = c_base + c * VE;
            if (a >= n_spectra || col0 >= cols) continue;
            const uint4 v = *reinterpret_cast<const uint4 *>(lds + lds_elem<T>(t, c * VE));
            if (VEC && col0 + VE <= cols) {
                *reinterpret_cast<uint4 *>(dst + pub_addr(t, col0)) = v;
            } else {
                T e[VE];
                __builtin_memcpy(e, &v, 16);
                for (int u = 0; u < VE && col0 + u < cols; ++u)
                    *reinterpret_cast<T *>(dst + pub_addr(t, col0 + u)) = e[u];
            }
        }
    }
}

// Row and column of lower-triangle product b = i(i+1)/2 + j.
__device__ __forceinline__ void pair_of(int64_t b, int &i, int &j) {
    int r = (int)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
    while ((int64_t)r * (r + 1) / 2 > b) --r;
    while ((int64_t)(r + 1) * (r + 2) / 2 <= b) ++r;
    i = r;
    j = (int)(b - (int64_t)r * (r + 1) / 2);
}

// Index of product (i, j), i <= j, in the upper triangle's rows.
__device__ __forceinline__ int64_t upper_index(int N, int i, int j) {
    return (int64_t)i * N - (int64_t)i * (i - 1) / 2 + (j - i);
}

// C_ji from C_ij.
__device__ __forceinline__ int2 conj_of(int2 v, int is_int) {
    return make_int2(v.x, is_int ? -v.y : __float_as_int(-__int_as_float(v.y)));
}

// The dump conversions read the accumulators once, in whole rows, and turn
// them around in LDS, so that the writes are whole rows too.  Bound: HBM.  (One
// thread per output element, dividing its index into a pair and reading the
// accumulator there, against now: 300 inputs x 1024 channels full 0.51 -> 0.28 ms,
// full baseline-major 1.04 -> 0.28; 256 x 1024 lower baseline-major 0.26 -> 0.13,
// upper 0.29 -> 0.16; 1024 x 256 full 1.67 -> 0.59.)

// Channel-major upper triangle or full matrix: a workgroup takes the products
// of 32 rows I and 32 columns J <= I of one channel (gridDim.y: channels), the
// mirrored ones through LDS.
constexpr int kTile = 32;
template <bool FULL>
__global__ __launch_bounds__(kThreads) void dump_mirror_kernel(const int2 *__restrict__ acc, int2 *__restrict__ dst,
                                                                int N, int is_int, const int *__restrict__ zflag) {
    __shared__ int2 t[kTile][kTile + 1];
    const bool zero = zflag && *zflag;
    const int64_t Bl = (int64_t)N * (N + 1) / 2;
    const int k = blockIdx.y;
    int bi, bj;
    pair_of(blockIdx.x, bi, bj);
    const int x = threadIdx.x % kTile, y0 = threadIdx.x / kTile;
    const int2 *src = acc + k * Bl;
    int2 *out = dst + k * (FULL ? (int64_t)N * N : Bl);
    constexpr int R = kTile * kTile / kThreads;        // products per thread
    int2 v[R];                                         // (read together: places outside read product 0)
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = bi * kTile + y0 + q * (kThreads / kTile), j = bj * kTile + x;
        v[q] = src[i < N && j <= i ? (int64_t)i * (i + 1) / 2 + j : 0];
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int y = y0 + q * (kThreads / kTile), i = bi * kTile + y, j = bj * kTile + x;
        if (zero) v[q] = make_int2(0, 0);
        t[y][x] = v[q];
        if (FULL && i < N && j <= i) out[(int64_t)i * N + j] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int y = y0; y < kTile; y += kThreads / kTile) {
        const int i = bi * kTile + x, j = bj * kTile + y;   // product (j, i) of the upper triangle
        if (i >= N || j > i || (FULL && j == i)) continue;
        out[FULL ? (int64_t)j * N + i : upper_index(N, j, i)] = i == j ? t[x][y] : conj_of(t[x][y], is_int);
    }
}

// Baseline-major dumps, in any layout: a workgroup takes 64 products of 32
// channels.
constexpr int kProducts = 64;
__global__ __launch_bounds__(kThreads) void dump_baseline_kernel(const int2 *__restrict__ acc, int2 *__restrict__ dst,
                                                                  int C, int N, int layout, int is_int,
                                                                  const int *__restrict__ zflag) {
    __shared__ int2 t[kTile][kProducts + 1];
    __shared__ int pi[kProducts], pj[kProducts];
    const bool zero = zflag && *zflag;
    const int64_t Bl = (int64_t)N * (N + 1) / 2;
    const int64_t b0 = (int64_t)blockIdx.x * kProducts;
    const int k0 = blockIdx.y * kTile;
    {
        constexpr int R = kTile * kProducts / kThreads;   // products per thread
        const int x = threadIdx.x % kProducts, y0 = threadIdx.x / kProducts;
        int2 v[R];                                     // (read together: places outside read product 0)
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int k = k0 + y0 + q * (kThreads / kProducts);
            v[q] = acc[b0 + x < Bl && k < C ? k * Bl + b0 + x : 0];
        }
        if (layout != 0 && threadIdx.x < kProducts && b0 + threadIdx.x < Bl)
            pair_of(b0 + threadIdx.x, pi[threadIdx.x], pj[threadIdx.x]);
#pragma unroll
        for (int q = 0; q < R; ++q) t[y0 + q * (kThreads / kProducts)][x] = zero ? make_int2(0, 0) : v[q];
    }
    __syncthreads();
    const int x = threadIdx.x % kTile;
    if (k0 + x >= C) return;
#pragma unroll
    for (int y = threadIdx.x / kTile; y < kProducts; y += kThreads / kTile) {
        if (b0 + y >= Bl) break;
        const int2 v = t[x][y];
        if (layout == 0) {
            dst[(b0 + y) * C + k0 + x] = v;
            continue;
        }
        const int i = pi[y], j = pj[y];
        const int2 w = i == j ? v : conj_of(v, is_int);
        if (layout == 1) {
            dst[upper_index(N, j, i) * C + k0 + x] = w;
        } else {
            dst[((int64_t)i * N + j) * C + k0 + x] = v;
            if (i != j) dst[((int64_t)j * N + i) * C + k0 + x] = w;
        }
    }
}

// dst = src, n elements, or zeros where *zflag is set.
template <typename V>
__global__ void dump_copy_kernel(const V *__restrict__ src, V *__restrict__ dst, int64_t n,
                                 const int *__restrict__ zflag) {
    const bool zero = zflag && *zflag;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        dst[e] = zero ? V{} : src[e];
}

__global__ void zero_kernel(uint32_t *__restrict__ p, int64_t n) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        p[e] = 0u;
}

int grid_for(int64_t n) {
    int64_t g = (n + kThreads - 1) / kThreads;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (int)g;
}

// nk: channels moved (the grid); C stays the channel stride of the public
// layout, so a public pointer advanced by k0 channels moves channels
// [k0, k0 + nk) to held channels [0, nk).
template <typename T, bool INGEST, bool SAT8 = false>
hipError_t relayout_t(int C, int N, int n_spectra, SpecLayout lay, const void *src, void *dst, UserScale us,
                      hipStream_t s, int nk = -1) {
    constexpr int TB = kRowBytes / (int)sizeof(T);
    const int n_tb = (n_spectra + TB - 1) / TB;
    const int n_cc = (2 * N + kCols - 1) / kCols;
    const int64_t grid = (int64_t)(nk < 0 ? C : nk) * n_tb * n_cc;
    if (grid < 1) return hipSuccess;
    if (grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const void *pub = INGEST ? src : dst;
    const bool vec = (2 * N * (int)sizeof(T)) % 16 == 0 && reinterpret_cast<uintptr_t>(pub) % 16 == 0;
    const uint8_t *in = static_cast<const uint8_t *>(src);
    uint8_t *out = static_cast<uint8_t *>(dst);
    if (vec)
        hipLaunchKernelGGL((relayout_kernel<T, INGEST, true, SAT8>), dim3((unsigned)grid), dim3(kThreads), 0, s, in,
                           out, C, N, n_spectra, n_tb, n_cc, lay, us);
    else
        hipLaunchKernelGGL((relayout_kernel<T, INGEST, false, SAT8>), dim3((unsigned)grid), dim3(kThreads), 0, s, in,
                           out, C, N, n_spectra, n_tb, n_cc, lay, us);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_ingest(int prec, int C, int N, int n_spectra, SpecLayout lay, const void *src, void *spec,
                         UserScale us, hipStream_t stream) {
    switch (elem_bytes(prec)) {
    case 4: return relayout_t<uint32_t, true>(C, N, n_spectra, lay, src, spec, us, stream);
    case 2: return relayout_t<uint16_t, true>(C, N, n_spectra, lay, src, spec, us, stream);
    default:
        if (prec == P_INT8) return relayout_t<uint8_t, true, true>(C, N, n_spectra, lay, src, spec, us, stream);
        return relayout_t<uint8_t, true>(C, N, n_spectra, lay, src, spec, us, stream);
    }
}

hipError_t launch_ingest_channels(int prec, int C, int k0, int nk, int N, int n_spectra, SpecLayout lay,
                                  const void *src, void *spec, UserScale us, hipStream_t stream) {
    if (k0 < 0 || nk < 1 || k0 + nk > C) return hipErrorInvalidValue;
    const uint8_t *s0 = static_cast<const uint8_t *>(src) + (int64_t)k0 * 2 * N * elem_bytes(prec);
    switch (elem_bytes(prec)) {
    case 4: return relayout_t<uint32_t, true>(C, N, n_spectra, lay, s0, spec, us, stream, nk);
    case 2: return relayout_t<uint16_t, true>(C, N, n_spectra, lay, s0, spec, us, stream, nk);
    default:
        if (prec == P_INT8) return relayout_t<uint8_t, true, true>(C, N, n_spectra, lay, s0, spec, us, stream, nk);
        return relayout_t<uint8_t, true>(C, N, n_spectra, lay, s0, spec, us, stream, nk);
    }
}

hipError_t launch_export(int prec, int C, int N, int n_spectra, SpecLayout lay, const void *spec, void *dst,
                         hipStream_t stream) {
    switch (elem_bytes(prec)) {
    case 4: return relayout_t<uint32_t, false>(C, N, n_spectra, lay, spec, dst, UserScale{}, stream);
    case 2: return relayout_t<uint16_t, false>(C, N, n_spectra, lay, spec, dst, UserScale{}, stream);
    default: return relayout_t<uint8_t, false>(C, N, n_spectra, lay, spec, dst, UserScale{}, stream);
    }
}

hipError_t launch_dump_convert(int C, int N, int layout, int order, int is_int, const void *acc, void *dst,
                               hipStream_t stream, const int *zflag) {
    const int2 *a = static_cast<const int2 *>(acc);
    int2 *d = static_cast<int2 *>(dst);
    const int64_t Bl = (int64_t)N * (N + 1) / 2, n = (N + kTile - 1) / kTile;
    if (order != 0) {
        const dim3 grid((unsigned)((Bl + kProducts - 1) / kProducts), (unsigned)((C + kTile - 1) / kTile));
        hipLaunchKernelGGL(dump_baseline_kernel, grid, dim3(kThreads), 0, stream, a, d, C, N, layout, is_int, zflag);
    } else if (layout == 0) {
        hipLaunchKernelGGL(dump_copy_kernel<int2>, dim3(grid_for(Bl * C)), dim3(kThreads), 0, stream, a, d, Bl * C,
                           zflag);
    } else if (layout == 1) {
        hipLaunchKernelGGL(dump_mirror_kernel<false>, dim3((unsigned)(n * (n + 1) / 2), (unsigned)C), dim3(kThreads), 0,
                           stream, a, d, N, is_int, zflag);
    } else {
        hipLaunchKernelGGL(dump_mirror_kernel<true>, dim3((unsigned)(n * (n + 1) / 2), (unsigned)C), dim3(kThreads), 0,
                           stream, a, d, N, is_int, zflag);
    }
    return hipGetLastError();
}

hipError_t launch_dump_copy(const void *acc, void *dst, int64_t n_words, const int *zflag, hipStream_t stream) {
    // accumulators are 8-byte pairs, C * B of them (C even): 16-byte vectors
    if (n_words % 4) return hipErrorInvalidValue;
    hipLaunchKernelGGL(dump_copy_kernel<int4>, dim3(grid_for(n_words / 4)), dim3(kThreads), 0, stream,
                       static_cast<const int4 *>(acc), static_cast<int4 *>(dst), n_words / 4, zflag);
    return hipGetLastError();
}

hipError_t launch_zero(void *p, int64_t n_words, hipStream_t stream) {
    hipLaunchKernelGGL(zero_kernel, dim3(grid_for(n_words)), dim3(kThreads), 0, stream, static_cast<uint32_t *>(p),
                       n_words);
    return hipGetLastError();
}

}  // namespace corr
