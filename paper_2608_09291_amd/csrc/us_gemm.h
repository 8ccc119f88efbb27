// Dense INT8 GEMM on the int8 matrix cores: the kernel and its
// configurations (us_gemm.hip has the entry point).
//
// Y = W X, W int8 M x K, X int8 N x K (row n = column n of X), Y int32 N x M.
// A wavefront owns R row blocks x C column blocks of 16. WM x WN wavefronts
// of a workgroup share their operands through LDS (one barrier per chunk),
// and WK such groups split K and combine in LDS. A chunk is 128 bytes of k of
// every row and column.
//
// What bounds it is getting operands into a CU: HBM at few columns (W is read
// once), L2 at many (every workgroup reads its rows and columns). So operands
// go straight into LDS in whole 128-byte lines, 8 rows per load (118 B/ns per
// CU from L2 against 38 for the matrix layout's 16 rows x 64 bytes, as
// measured), the tile grows with the problem, and all columns are one launch
// instead of one pass over W per 32 columns.
//
// us per call, the register kernel before it -> this one, weights rotating past
// the 256 MB cache: 4096x11008 N = 8 15.1 -> 10.5, N = 32 24.9 -> 14.8, N = 256
// 195 -> 29; 12288x4096 N = 512 333 -> 45; 8192x8192 N = 1024 900 -> 78. Over
// three copies of the weights, which that cache holds, 4096x11008 takes 9.0 at
// N = 8 and 22.3 at N = 256. Over 60 drawn shapes (M, K 256-16384) the choice
// of gemm_pick takes 0.79 of the time at N = 1-16, 0.61 at 17-32, 0.29 at
// 33-128 and 0.13 above (geometric means; the slowest, a call of 2 us, 0.4 us
// more). Non-temporal weight loads were up to 20 % slower.
#ifndef UNIONSPARSE_US_GEMM_H
#define UNIONSPARSE_US_GEMM_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>
#include <utility>

namespace us_gemm_detail {

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) i32x4 lds_i4;

constexpr int kMaxLds = 160 * 1024;
constexpr int kBufferDword3 = 0x00020000;                 // raw buffer, 32-bit data (gfx9 family)

// R, C, WM, WN, WK as above, NB operand stages, LW wavefronts per SIMD the
// registers are bound for; s, a, b, e: cost in us (gemm_cost).
struct GemmCfg {
    int R, C, WM, WN, WK, NB, LW;
    float s, a, b, e;
};

// The built configurations; costs fitted, one configuration at a time, to the
// sweep above. The list is what a greedy choice from 29 left (mean loss
// against the fastest of them: 2 %).
#define US_GEMM_CFGS(X)                                    \
    X(1, 1, 1, 1, 1, 2, 8, 0.00f, 0.27f, 0.146f, 0.15f)    \
    X(1, 1, 1, 1, 8, 2, 6, 0.07f, 0.00f, 0.179f, 0.12f)    \
    X(1, 1, 1, 1, 4, 2, 8, 0.31f, 0.20f, 0.186f, 0.02f)    \
    X(2, 1, 1, 1, 4, 2, 6, 0.20f, 0.30f, 0.271f, 0.14f)    \
    X(2, 1, 1, 1, 8, 2, 3, 0.19f, 0.51f, 0.199f, 0.21f)    \
    X(2, 2, 1, 1, 4, 1, 4, 0.30f, 0.39f, 0.365f, 0.17f)    \
    X(2, 2, 1, 1, 8, 1, 3, 0.22f, 0.67f, 0.179f, 0.12f)    \
    X(4, 2, 1, 1, 4, 1, 3, 0.50f, 0.58f, 0.533f, 0.40f)    \
    X(4, 2, 1, 1, 8, 1, 2, 0.93f, 1.05f, 0.093f, 0.09f)    \
    X(4, 4, 1, 1, 4, 1, 2, 0.82f, 0.84f, 0.696f, 1.05f)    \
    X(4, 4, 1, 1, 8, 1, 2, 0.78f, 1.45f, 0.273f, 0.56f)    \
    X(2, 4, 2, 2, 1, 2, 3, 0.00f, 0.42f, 0.262f, 1.12f)    \
    X(4, 4, 2, 2, 1, 2, 2, 0.00f, 0.52f, 0.401f, 2.30f)

#define US_GEMM_ROW(...) {__VA_ARGS__},
constexpr GemmCfg kGemmCfgs[] = {US_GEMM_CFGS(US_GEMM_ROW)};
#undef US_GEMM_ROW
constexpr int kNumGemmCfgs = sizeof(kGemmCfgs) / sizeof(kGemmCfgs[0]);

template <int R, int C, int WM, int WN, int WK, int NB>
struct GemmStage {
    static constexpr int kRows = 16 * R * WM, kCols = 16 * C * WN;
    static constexpr int kBuf = 128 * (kRows + kCols);    // one chunk of a K group's operands
    static constexpr int kGroup = NB * kBuf;
    static constexpr int kTotal = WK * kGroup;
    static constexpr int kShare = kTotal / (WM * WN * WK) / 1024;  // combine blocks (1 KB) per wavefront
};

// 16 bytes per lane straight into LDS: lane l writes LDS [lds + 16 l, + 16).
// M0 holds the LDS base and is set here only (the compiler keeps nothing in
// it). The callers order their LDS reads with vmcnt waits and barriers.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void gemm_dma16(u32x4 desc, uint32_t lds, uint32_t voff) {
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :
                     : "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(voff), "s"(desc)
                     : "memory", "m0");
}
#pragma clang diagnostic pop

template <int R, int C, int WM, int WN, int WK, int NB, int LW>
__global__ __launch_bounds__(64 * WM * WN * WK, LW) void us_gemm_i8_kernel(const int8_t *w, const int8_t *x, int m_, int k_,
                                                                          int n_, int n_tiles, int32_t *y) {
    using S = GemmStage<R, C, WM, WN, WK, NB>;
    constexpr int WG = WM * WN;                            // wavefronts of a K group
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    const uint32_t lds0 = (uint32_t)(size_t)(lds_u32 *)lds;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave / WG, wg = wave % WG, wm = wg % WM, wn = wg / WM;
    // Column tiles of one row group take consecutive places on one XCD.
    const uint32_t slot = blockIdx.x >> 3;
    const uint32_t group = (slot / (uint32_t)n_tiles) * 8u + (blockIdx.x & 7u);
    const int n0 = (int)(slot % (uint32_t)n_tiles) * S::kCols;
    const int nrb = m_ / 16;
    if (group * (WM * R) >= (uint32_t)nrb) return;         // whole workgroup
    const int64_t row0 = (int64_t)group * S::kRows;

    const uint32_t unkb = (uint32_t)k_ / 64u;
    const uint32_t kb0 = (uint32_t)wk * (unkb / WK) + min((uint32_t)wk, unkb % WK);
    const uint32_t nk = unkb / WK + ((uint32_t)wk < unkb % WK ? 1u : 0u);      // >= 1
    const uint32_t nchunk = WG > 1 ? ((unkb + WK - 1) / WK + 1) / 2 : (nk + 1) / 2;

    // Operands of this workgroup: rows past M and columns past N lie outside
    // the buffers and read zero.
    const uint32_t K = (uint32_t)k_;
    auto desc_of = [&](const int8_t *p, uint32_t rows) {   // the K slice's first byte of `rows` rows on
        const uint64_t a = (uint64_t)(size_t)(p + 64u * kb0);
        return (u32x4){(uint32_t)a, (uint32_t)(a >> 32) & 0xFFFFu, rows * K - 64u * kb0, (uint32_t)kBufferDword3};
    };
    const u32x4 wd = desc_of(w + row0 * k_, (uint32_t)min((int64_t)S::kRows, (int64_t)m_ - row0));
    const u32x4 xd = desc_of(x + (int64_t)n0 * k_, (uint32_t)min(S::kCols, n_ - n0));
    const uint32_t st = lds0 + (uint32_t)(wk * S::kGroup);

    // Load b of a chunk brings rows 8 b .. 8 b + 7, 128 bytes each: lane
    // 8 c + p the 16-byte piece p ^ c ^ (b mod 2) of row c, so that the reads
    // of 16 rows below fall in different banks. In a chunk whose second half
    // lies past the slice, those weights read zero.
    const uint32_t lc = (uint32_t)lane >> 3, lq = ((uint32_t)lane & 7u) ^ lc;
    auto load = [&](uint32_t c, uint32_t buf) {
        const uint32_t dst = st + buf * S::kBuf;
        const uint32_t v = lc * K + 16u * lq + 128u * c;
        const uint32_t vw = 2u * c + (lq >> 2) < nk ? v : 0x80000000u;
#pragma unroll
        for (int b0 = 0; b0 < S::kRows / 8; b0 += WG) {
            const int b = b0 + wg;
            if (S::kRows / 8 % WG == 0 || b < S::kRows / 8) {
                const uint32_t o = (vw ^ (uint32_t)(16 * (b & 1))) + (uint32_t)(8 * b) * K;
                gemm_dma16(wd, dst + 1024u * b, o);
            }
        }
#pragma unroll
        for (int b0 = 0; b0 < S::kCols / 8; b0 += WG) {
            const int b = b0 + wg;
            if (S::kCols / 8 % WG == 0 || b < S::kCols / 8)
                gemm_dma16(xd, dst + 128u * S::kRows + 1024u * b, (v ^ (uint32_t)(16 * (b & 1))) + (uint32_t)(8 * b) * K);
        }
    };
    const int rr = lane & 15, g = lane >> 4;
    const uint32_t rd0 = 1024u * (uint32_t)(rr >> 3) + 128u * (uint32_t)(rr & 7);
    const uint32_t rs = (uint32_t)((rr & 7) ^ (rr >> 3));
    const uint32_t rd[2] = {rd0 + 16u * ((uint32_t)g ^ rs), rd0 + 16u * ((4u + (uint32_t)g) ^ rs)};
    const uint32_t st_w = st + 2048u * (uint32_t)(R * wm), st_x = st + 128u * S::kRows + 2048u * (uint32_t)(C * wn);

    i32x4 acc[R][C];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int cb = 0; cb < C; ++cb) acc[r][cb] = (i32x4){0, 0, 0, 0};

    load(0, 0);
    auto step = [&](uint32_t c, uint32_t buf, auto more) {
        __builtin_amdgcn_s_waitcnt(0);
        if constexpr (WG > 1) __builtin_amdgcn_s_barrier();
        __asm__ volatile("" ::: "memory");
        if constexpr (NB == 2)
            if constexpr (decltype(more)::value) load(c + 1, buf ^ 1u);
        const uint32_t o = NB == 2 ? buf * S::kBuf : 0u;
        i32x4 a[2][R], b[2][C];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int r = 0; r < R; ++r) a[u][r] = *(const lds_i4 *)(size_t)(st_w + o + rd[u] + 2048u * r);
#pragma unroll
            for (int cb = 0; cb < C; ++cb) b[u][cb] = *(const lds_i4 *)(size_t)(st_x + o + rd[u] + 2048u * cb);
        }
        if constexpr (NB == 1) {
            __asm__ volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): the stage has been read
            __asm__ volatile("" ::: "memory");
            if constexpr (decltype(more)::value) load(c + 1, 0);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int cb = 0; cb < C; ++cb)
#pragma unroll
                for (int r = 0; r < R; ++r) acc[r][cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(b[u][cb], a[u][r], acc[r][cb], 0, 0, 0);
        __asm__ volatile("" ::: "memory");
    };
    static_assert(WG == 1 || NB == 2, "shared stages are double-buffered");
    uint32_t c = 0;
    for (; c + 1 < nchunk; ++c) step(c, c & 1u, std::integral_constant<bool, true>());
    step(c, c & 1u, std::integral_constant<bool, false>());

    // Lane (rr, g), element v of a block: row rr, column 4 g + v.
    constexpr int kBlocks = R * C;
    if constexpr (WK == 1) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t m = row0 + 16 * (R * wm + r) + rr;
            if (m >= m_) break;                            // (whole row blocks)
#pragma unroll
            for (int cb = 0; cb < C; ++cb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int n = n0 + 16 * (C * wn + cb) + 4 * g + v;
                    if (n < n_) y[(int64_t)n * m_ + m] = acc[r][cb][v];
                }
        }
    } else {
        constexpr int kPer = S::kShare < kBlocks ? S::kShare : kBlocks;
        static_assert(kPer >= 1, "a wavefront's share of the LDS holds at least one block");
        const uint32_t mine = lds0 + (uint32_t)((wg * WK + wk) * kPer) * 1024u + 4u * lane;
#pragma unroll
        for (int b0 = 0; b0 < kBlocks; b0 += kPer) {
            __syncthreads();
#pragma unroll
            for (int b = 0; b < kPer; ++b) {
                if (b0 + b < kBlocks) {
                    const i32x4 t = acc[(b0 + b) / C][(b0 + b) % C];
#pragma unroll
                    for (int v = 0; v < 4; ++v) *(lds_u32 *)(size_t)(mine + 1024 * b + 256 * v) = (uint32_t)t[v];
                }
            }
            __syncthreads();
            const int rows_now = 4 * (kBlocks - b0 < kPer ? kBlocks - b0 : kPer);
            for (int q = wave; q < WG * rows_now; q += WG * WK) {              // wave-uniform
                const int s = q / rows_now, bv = q % rows_now, blk = b0 + (bv >> 2), v = bv & 3;
                const int64_t m = row0 + 16 * (R * (s % WM) + blk / C) + rr;
                const int n = n0 + 16 * (C * (s / WM) + blk % C) + 4 * g + v;
                const uint32_t at = lds0 + (uint32_t)(s * WK * kPer) * 1024u + (uint32_t)bv * 256u + 4u * lane;
                int32_t sum = 0;
#pragma unroll
                for (int k = 0; k < WK; ++k) sum += (int32_t) * (const lds_u32 *)(size_t)(at + (uint32_t)(k * kPer * 1024));
                if (m < m_ && n < n_) y[(int64_t)n * m_ + m] = sum;
            }
        }
    }
}

template <int R, int C, int WM, int WN, int WK, int NB, int LW>
hipError_t launch_gemm(const int8_t *w, const int8_t *x, int32_t *y, int M, int K, int N, hipStream_t s) {
    using S = GemmStage<R, C, WM, WN, WK, NB>;
    auto kern = us_gemm_i8_kernel<R, C, WM, WN, WK, NB, LW>;
    // Allow more than 64 KB of dynamic LDS: once per instantiation and device.
    if constexpr (S::kTotal > 65536) {
        static std::atomic<unsigned long long> attr_set{0};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) dev = 0;
        const unsigned long long bit = 1ull << (dev & 63);
        if (!(attr_set.load(std::memory_order_acquire) & bit)) {
            const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
            if (e != hipSuccess) return e;
            attr_set.fetch_or(bit, std::memory_order_release);
        }
    }
    const int tiles = (N + S::kCols - 1) / S::kCols;
    const int64_t groups8 = ((M / 16 + WM * R - 1) / (WM * R) + 7) / 8;
    constexpr int kLds = S::kTotal;
    hipLaunchKernelGGL(kern, dim3((unsigned)(8 * groups8 * tiles)), dim3(64 * WM * WN * WK), kLds, s, w, x, M, K, N, tiles, y);
    return hipGetLastError();
}

constexpr float kNoLaunch = 3e38f;

// Cost of a configuration in us: generations of the workgroups that the CUs
// hold, each a start s, per chunk the larger of one wavefront's latency a and
// the busiest SIMD's share b v (v wavefronts on it), blended a little, and
// e v for the combine and the stores. A grid of 2^32 threads or more cannot be
// launched. (Always inlined: every call has a constant configuration, which
// leaves two of its ten divisions.)
__attribute__((always_inline)) inline float gemm_cost(const GemmCfg &c, int64_t nrb, int nkb, int N, int n_cu) {
    const int w = c.WM * c.WN * c.WK, lds = c.WK * c.NB * 128 * 16 * (c.R * c.WM + c.C * c.WN);
    const int64_t groups = (nrb + c.R * c.WM - 1) / (c.R * c.WM), cols = 16 * c.C * c.WN, tiles = (N + cols - 1) / cols;
    if ((groups + 7) / 8 * tiles >= ((int64_t)1 << 23) / w) return kNoLaunch;
    const int by_lds = kMaxLds / lds, by_regs = 4 * c.LW / w > 0 ? 4 * c.LW / w : 1;
    int per_cu = by_lds < by_regs ? by_lds : by_regs;
    if (per_cu > 16) per_cu = 16;
    const int64_t slots = (int64_t)n_cu * per_cu;
    const float chunks = (float)(((nkb + c.WK - 1) / c.WK + 1) / 2);
    float t = 0.0f;
    for (int64_t left = groups * tiles; left > 0;) {
        // (whole generations at once: they cost the same)
        const int64_t gens = left > slots ? left / slots : 1, g = left < slots ? left : slots;
        const float v = 0.25f * (float)(w * ((g + n_cu - 1) / n_cu)), iss = c.b * v;
        t += (float)gens * (c.s + chunks * (0.9f * (c.a > iss ? c.a : iss) + 0.1f * (c.a + iss)) + c.e * v);
        left -= gens * g;
    }
    return t;
}

// What a large matrix takes at up to 8 columns instead of the configuration of
// lowest cost. The costs were fitted to M <= 16384 and know no HBM limit. With
// rows of 1 KB and more they send larger matrices to config 0 (no K slices),
// which streams W at 4.2-4.8 TB/s where it has fewer than 8 wavefronts per CU
// to request it, or rows a multiple of 4 KB apart, against 5.2-6 with four
// slices; and with rows above 8 KB to four slices, each wavefront's own above
// 2 KB (4.4 TB/s against 5.5 with eight). us per call at N = 1, that choice ->
// this one, against the kernel that this file replaced (16 rows x 64 bytes
// into registers): 28672x1536 10.3 -> 9.2 against 10.1, 31744x2048 12.9 -> 12.4
// against 13.8, 28672x4096 26.3 -> 22.5 against 23.3, 28672x8192 45.4 -> 41.0
// against 49.0, 53248x4096 46.5 -> 40.4 against 45.9, 28672x11008 80.9 -> 59.9
// against 67.1, 16384x16384 62.4 -> 48.6 against 54.5. Config 1 (eight slices)
// holds two workgroups per CU; where that leaves a second, part-filled
// generation, four slices (five per CU) are faster up to 8 KB: 12288x8192
// 20.8 -> 18.0 against 20.2, 8720x8192 17.9 -> 14.0 against 19.1. With more
// wavefronts config 0 stays (49152x2048 17.6 against 18.1), and above 8
// columns, where it already was ahead, the lowest cost (53248x4096 N = 16 43.0
// against 44.4).
inline int gemm_narrow(int best, int64_t nrb, int nkb, int n_cu) {
    if (nkb > 128) return best == 0 || best == 3 ? 4 : best;
    if (best == 1 && nrb > 2 * (int64_t)n_cu) return 2;
    return best == 0 && nkb >= 16 && (nrb < 8 * (int64_t)n_cu || nkb % 64 == 0) ? 2 : best;
}
static_assert(kGemmCfgs[2].R == 1 && kGemmCfgs[2].WK == 4 && kGemmCfgs[3].R == 2 && kGemmCfgs[3].WK == 4 &&
                  kGemmCfgs[4].R == 2 && kGemmCfgs[4].WK == 8,
              "gemm_narrow names configurations by their place in the list");

// The configuration with the lowest cost. Wide tiles are left out where more
// than half of their columns would be empty; the first configuration takes
// every shape, up to the rows of one grid (2^30 / column tiles), and the last
// one, with the fewest workgroups, what then is left.
template <int... I>
inline int gemm_pick(int64_t nrb, int nkb, int N, int n_cu, std::integer_sequence<int, I...>) {
    int best = -1;
    float cost = 0.0f;
    const auto consider = [&](auto k) __attribute__((always_inline)) {
        constexpr GemmCfg c = kGemmCfgs[decltype(k)::value];
        if (k > 0 && c.WK > nkb) return;                   // at least 64 k per slice
        if (k > 0 && c.C * c.WN > 1 && 16 * c.C * c.WN >= 2 * (N + 15)) return;
        const float t = gemm_cost(c, nrb, nkb, N, n_cu);
        if (best < 0 || t < cost) {
            best = k;
            cost = t;
        }
    };
    (consider(std::integral_constant<int, I>()), ...);
    if (cost >= kNoLaunch) return (int)sizeof...(I) - 1;
    return N <= 8 ? gemm_narrow(best, nrb, nkb, n_cu) : best;
}

inline int gemm_pick(int64_t nrb, int nkb, int N, int n_cu) {
    return gemm_pick(nrb, nkb, N, n_cu, std::make_integer_sequence<int, kNumGemmCfgs>());
}

}  // namespace us_gemm_detail

#endif  // UNIONSPARSE_US_GEMM_H
