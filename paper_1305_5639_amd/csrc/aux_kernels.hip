// Data-movement kernels around the two engines: caller spectra in and out of
// the time-blocked planar layout, dump layout/order conversion and a zero fill.
// The spectra moves and the dump conversions are tiled transposes through LDS.
#include "corr_internal.h"

namespace corr {
namespace {

constexpr int kThreads = 256;


// Caller spectra <-> held rows.  The public row of a spectrum holds C x 2N
// columns (k, 2p + plane) one after the other; the held layout wants each
// column's TB values of a time block contiguous (one 64-byte plane row).  That is
// a TB x C 2N transpose per time block, in tiles of kCols columns whatever their
// channels (a tile of one channel's columns would be part empty: 48 inputs have
// 96): TB public segments of kCols * ES bytes <-> kCols held rows of 64 bytes.  A
// thread moves 4 16-byte vectors either way, the public ones from 4 / ES
// neighbouring spectra, which it transposes in registers into dwords of 4 / ES
// spectra of one column; LDS holds a tile's dwords as [16 bytes of columns]
// [column][dword] with 4 dwords of padding, so that a wave's 16 vectors x 4 dwords
// hit distinct banks on the public side, and the held side reads whole vectors.
// Bound: HBM, and for small calls the latency of one load and one store.
// (Per-channel tiles with a scalar path where 2N ES is no multiple of 16, loads
// under branches and a byte or half at a time out of LDS, against now, ingest and
// export: 48 inputs x 256 channels x 512 int8 12.2 -> 9.4 us, 7.1 -> 6.7; 300 x 256 x
// 1000 int8 198 -> 49, 251 -> 55; 300 x 1024 x 1000 FP16 465 -> 449, 686 -> 486 = 5.1
// TB/s, the copy rate; 1 input x 1024 x 4096 int8 with its X pass 182 -> 22.)
constexpr int kCols = 256;

// Byte-wise max(b, -127) of four int8 values: a byte equal to 0x80 (-128)
// becomes 0x81 (-127), every other byte is unchanged.  x marks the -128 bytes
// as zero bytes; the zero-byte test below is exact (no borrow between bytes).
__device__ __forceinline__ uint32_t sat_int8x4(uint32_t v) {
    const uint32_t x = v ^ 0x80808080u;
    const uint32_t nz = ((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x;
    return v | ((~nz & 0x80808080u) >> 7);
}

// w[r]: 4 bytes of row r, elements of ES bytes -> w[i]: the 4 / ES rows of element
// i.  Its own inverse.
template <int ES>
__device__ __forceinline__ void transpose(uint32_t *w) {
    if constexpr (ES == 2) {
        const uint32_t a = w[0], b = w[1];
        w[0] = __builtin_amdgcn_perm(b, a, 0x05040100);
        w[1] = __builtin_amdgcn_perm(b, a, 0x07060302);
    } else if constexpr (ES == 1) {
        const uint32_t a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400);
        const uint32_t b = __builtin_amdgcn_perm(w[1], w[0], 0x07030602);
        const uint32_t c = __builtin_amdgcn_perm(w[3], w[2], 0x05010400);
        const uint32_t d = __builtin_amdgcn_perm(w[3], w[2], 0x07030602);
        w[0] = __builtin_amdgcn_perm(c, a, 0x05040100);
        w[1] = __builtin_amdgcn_perm(c, a, 0x07060302);
        w[2] = __builtin_amdgcn_perm(d, b, 0x05040100);
        w[3] = __builtin_amdgcn_perm(d, b, 0x07060302);
    }
}

// INGEST: public src -> held dst (the tail of the last block zero-filled);
// else held src -> public dst.  n_cols = channels moved x 2N; pub_row: bytes
// between spectra of the public side.  Public vectors may lie at any multiple of
// ES (a channel slice begins anywhere); the last one of a row may be part of 16
// bytes.  SAT8 (int8 ingest): -128 is read as -127, the symmetric range the
// X-engine's exact negation and the int32 overflow bound assume.
template <typename T, bool INGEST, bool SAT8 = false>
__global__ __launch_bounds__(kThreads) void relayout_kernel(const uint8_t *__restrict__ src,
                                                             uint8_t *__restrict__ dst, uint32_t n_cols, uint32_t cols,
                                                             int64_t pub_row, int n_spectra, int n_ct, bool blocks_first,
                                                             SpecLayout lay, UserScale us) {
    constexpr int ES = (int)sizeof(T), TB = kRowBytes / ES, VE = 16 / ES;
    constexpr int RI = 4 / ES;                          // spectra of a dword
    constexpr int CS = VE * 16 + 4;                     // LDS dwords of one vector's columns
    __shared__ __align__(16) uint32_t lds[kCols / VE * CS];
    const int n_tb = gridDim.x / n_ct;
    const int tb = blocks_first ? blockIdx.x % n_tb : blockIdx.x / n_ct;
    const uint32_t f0 = (uint32_t)(blocks_first ? blockIdx.x / n_tb : blockIdx.x % n_ct) * kCols;
    const int tid = threadIdx.x, tg = tid / 64 * 4 + tid % 64 / 16;
    const bool whole = f0 + kCols <= n_cols;            // no column past the end

    // thread's public vectors: spectra a0 + r < n_spectra, r < RI; columns
    // f0 + (16 q + tid % 16) VE, q < ES
    const int a0 = tb * TB + tg * RI;
    auto first_col = [&](int q) -> uint32_t { return f0 + (uint32_t)(q * 16 + tid % 16) * VE; };
    auto pub_addr = [&](int r, uint32_t col) -> int64_t { return (int64_t)(a0 + r) * pub_row + (int64_t)col * ES; };
    auto word = [&](int q, int i) -> uint32_t & { return lds[(q * 16 + tid % 16) * CS + i * 16 + tg]; };
    auto held_rows = [&](auto &&move) {
#pragma unroll
        for (int it = 0; it < kCols * 4 / kThreads; ++it) {
            const int j = it * (kThreads / 4) + tid / 4, hv = tid % 4;
            const uint32_t f = f0 + j;
            if (f >= n_cols) continue;
            const uint32_t k = f / cols, col = f - k * cols;
            move(lds + j / VE * CS + j % VE * 16 + hv * 4,
                 (int64_t)tb * lay.ts + (int64_t)k * lay.ks + (int64_t)col * kRowBytes + hv * 16);
        }
    };

    uint32_t w[ES][4][RI];                              // [vector column][dword][spectrum]
    if constexpr (INGEST) {
        if (us.scale2)
            for (int64_t c = (int64_t)blockIdx.x * kThreads + tid; c < us.C; c += (int64_t)gridDim.x * kThreads)
                us.scale2[c] = us.inv ? square_of_scale(us.inv[c]) : 1.0f;
        uint4 v[ES][RI];
        if (whole) {
#pragma unroll
            for (int q = 0; q < ES; ++q)
#pragma unroll
                for (int r = 0; r < RI; ++r) {
                    // past the last spectrum: any row of the block that there is
                    const int64_t o = a0 + r < n_spectra ? pub_addr(r, first_col(q))
                                                         : (int64_t)tb * TB * pub_row + (int64_t)first_col(q) * ES;
                    __builtin_memcpy(&v[q][r], src + o, 16);
                }
        } else {
#pragma unroll
            for (int q = 0; q < ES; ++q)
#pragma unroll
                for (int r = 0; r < RI; ++r) {
                    const uint32_t col = first_col(q);
                    v[q][r] = make_uint4(0, 0, 0, 0);
                    if (a0 + r >= n_spectra) continue;
                    if (col + VE <= n_cols) {
                        __builtin_memcpy(&v[q][r], src + pub_addr(r, col), 16);
                    } else {
                        T e[VE];
                        for (int u = 0; u < VE; ++u)
                            e[u] = col + u < n_cols ? *reinterpret_cast<const T *>(src + pub_addr(r, col + u)) : T(0);
                        __builtin_memcpy(&v[q][r], e, 16);
                    }
                }
        }
#pragma unroll
        for (int q = 0; q < ES; ++q) {
#pragma unroll
            for (int r = 0; r < RI; ++r) {
                uint32_t x[4] = {v[q][r].x, v[q][r].y, v[q][r].z, v[q][r].w};
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    if constexpr (SAT8) x[d] = sat_int8x4(x[d]);
                    w[q][d][r] = a0 + r < n_spectra ? x[d] : 0;
                }
            }
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                transpose<ES>(w[q][d]);
#pragma unroll
                for (int i = 0; i < RI; ++i) word(q, d * RI + i) = w[q][d][i];
            }
        }
        __syncthreads();
        held_rows([&](const uint32_t *l, int64_t o) {
            *reinterpret_cast<uint4 *>(dst + o) = *reinterpret_cast<const uint4 *>(l);
        });
    } else {
        held_rows([&](uint32_t *l, int64_t o) {
            *reinterpret_cast<uint4 *>(l) = *reinterpret_cast<const uint4 *>(src + o);
        });
        __syncthreads();
#pragma unroll
        for (int q = 0; q < ES; ++q) {
            const uint32_t col = first_col(q);
            if (col >= n_cols) continue;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
#pragma unroll
                for (int i = 0; i < RI; ++i) w[q][d][i] = word(q, d * RI + i);
                transpose<ES>(w[q][d]);
            }
#pragma unroll
            for (int r = 0; r < RI; ++r) {
                if (a0 + r >= n_spectra) continue;
                const uint4 v = make_uint4(w[q][0][r], w[q][1][r], w[q][2][r], w[q][3][r]);
                if (whole || col + VE <= n_cols) {
                    __builtin_memcpy(dst + pub_addr(r, col), &v, 16);
                } else {
                    T e[VE];
                    __builtin_memcpy(e, &v, 16);
                    for (int u = 0; u < VE && col + u < n_cols; ++u)
                        *reinterpret_cast<T *>(dst + pub_addr(r, col + u)) = e[u];
                }
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
    const uint32_t cols = 2 * (uint32_t)N;
    const int64_t n_cols = (int64_t)(nk < 0 ? C : nk) * cols, n_ct = (n_cols + kCols - 1) / kCols;
    const int64_t grid = n_ct * n_tb;
    if (grid < 1) return hipSuccess;
    if (grid > 0x7fffffffLL || n_cols > 0xffffffffLL - kCols) return hipErrorInvalidConfiguration;
    // Neighbouring workgroups take neighbouring columns, or, where a spectrum's
    // columns are 1 MB and more, the time blocks of the same columns (ingest and
    // export: 300 inputs x 1024 channels x 1000 FP16, 1.2 MB, 449 and 486 us, by
    // columns 469 and 477; 512 x 1024 x 512 FP8, 1 MB, 200 and 205, 207 and 219;
    // 512 x 2048 x 128 FP16, 4 MB, 210 and 204, 222 and 222; but 48 x 256 x 512 int8,
    // 24 KB, 11.5 and 5.9, 9.4 and 6.7; 256 x 256 x 500 FP32, 512 KB, 84.9 and 104,
    // 83.0 and 102).
    const bool blocks_first = n_cols * (int)sizeof(T) >= 1 << 20;
    hipLaunchKernelGGL((relayout_kernel<T, INGEST, SAT8>), dim3((unsigned)grid), dim3(kThreads), 0, s,
                       static_cast<const uint8_t *>(src), static_cast<uint8_t *>(dst), (uint32_t)n_cols, cols,
                       (int64_t)C * cols * (int)sizeof(T), n_spectra, (int)n_ct, blocks_first,
                       lay, us);
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
