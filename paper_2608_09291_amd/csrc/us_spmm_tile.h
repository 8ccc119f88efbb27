// IE-BME x INT4 -> INT32 sparse product on gfx950: the tile kernel, which
// automatic calls of every width take, except some of up to 32 columns
// (use_tile, tall), up to 48 columns at K = 64, and matrices of more than 2^22
// rows. Same operation and format as the chunked kernel of us_spmm_kernel.h
// (Section VI: the UnionSparse kernel, its LSPD decode and split-K); what
// differs:
//
//  * Wavefront tile. A wavefront multiplies R row blocks by C column blocks of
//    16, so that an expanded activation operand feeds R matrix instructions
//    and a decoded weight operand C of them. The chunked kernel decodes W and
//    expands X once per 16 x 32 outputs, and reads W again for every 32
//    columns; here all columns are one launch. Both expansions compete with
//    the matrix instructions for issue: a SIMD with four wavefronts was
//    measured to take 7.5 ns per v_mfma_i32_16x16x64_i8 with up to two other
//    vector instructions beside it, 9.3 with three, 12.0 with four, 14.4 with
//    six, 16.4 with eight, and 1 ns for each further one.
//
//  * Lane groups take LTs, not segments. A chunk is four LTs of a row block.
//    Lane (rr, g) owns mask row i = rr / 2, area row rr % 2 of LT g, and
//    matrix instruction j multiplies segment j of LT g in lane group g: a
//    product sums over all 64 k slots, so the four groups may come from four
//    LTs as long as both operands agree. A lane thus keeps one mask row and
//    one slot address for all four segments (no exchange through LDS), and
//    its activations for all four are the 2 x 16 consecutive bytes of LT g,
//    read with two 16-byte LDS reads and no transposition.
//
//  * Activations go straight into LDS, 8 columns x 128 bytes per load, lanes
//    along the row: 16 rows x 64 bytes per load was measured at 38 B/ns per
//    CU from L2, 8 x 128 at 118, contiguous bytes at 133. The 16-byte pieces
//    are placed with an XOR so that the reads of 16 columns fall in different
//    banks. With WM > 1 the WM wavefronts of a K slice stack along M and
//    share two such stages (one barrier per chunk); with WM = 1 every
//    wavefront has its own and takes it into registers before requesting the
//    next chunk's.
//
//  * One chunk ahead. At the top of a chunk the wavefront waits for
//    everything it has requested, and requests the next chunk before (NB = 2
//    payload stages) or after (NB = 1) decoding this one. Payload ranges of
//    64 chunks are worked out at once, one chunk per lane, so that a request
//    is a few scalar instructions.
//
// Measured against the chunked kernel (us per call, launched back to back on
// weights that rotate past the 256 MB cache, 50 % sparse where not said,
// before -> after): 12288x4096 N = 1024 301 -> 59, 4096x11008 N = 256 81 -> 26,
// N = 100 37 -> 16, 28672x8192 70 % sparse N = 32 35 -> 24, 13824x5120 60 %
// N = 16 11.9 -> 9.3, 28672x8192 70 % N = 1 21.2 -> 19.2 and reordered N = 5
// 25.2 -> 20.3, 11008x4096 N = 8 7.0 -> 6.7, 1024x4096 N = 8 4.1 -> 3.6.
// Geometric means over 330 drawn shapes (M 256-28672, K 256-28672, every
// weight form) with the choice of tile_pick: 0.24 of the time at N = 33-1024,
// 0.83 at 17-32, 0.92 at 1-16.
#ifndef UNIONSPARSE_US_SPMM_TILE_H
#define UNIONSPARSE_US_SPMM_TILE_H

#include <utility>

#include "us_spmm_kernel.h"

namespace us_spmm_detail {

// A configuration: R row blocks x C column blocks per wavefront, WM
// wavefronts along M that share activations, WK K slices, NB payload stages,
// LW wavefronts per SIMD the registers are bound for (8 is 7 for reordered
// LTs, whose permutation words do not fit), JS steps a chunk's four
// segments are decoded in (2 halves the decoded operands held at a time).
// s, a, b, e: its cost in us (tile_cost).
struct TileCfg {
    int R, C, WM, WK, NB, LW, JS;
    float s, a, b, e;
};

// The built configurations: what a greedy choice from 43 left. Their cost
// constants were fitted to the sweeps described above, then refined for the
// smallest mean loss against the fastest of all 43 (1 % at N = 1-32, 3 %
// above).
#define US_TILE_CFGS(X)                                            \
    X(1, 1, 1, 2, 2, 8, 1, 0.300f, 0.554f, 0.266f, 0.318f)         \
    X(1, 1, 1, 4, 1, 8, 1, 0.092f, 0.685f, 0.292f, 0.160f)         \
    X(1, 1, 1, 8, 2, 8, 1, 0.380f, 0.560f, 0.266f, 0.070f)         \
    X(1, 1, 1, 16, 2, 8, 1, 0.711f, 0.450f, 0.224f, 0.080f)        \
    X(2, 1, 1, 4, 2, 5, 1, 1.317f, 0.660f, 0.400f, 0.080f)         \
    X(1, 2, 1, 2, 2, 5, 1, 0.477f, 0.630f, 0.347f, 0.281f)         \
    X(1, 2, 1, 4, 1, 5, 1, 0.370f, 0.760f, 0.363f, 0.110f)         \
    X(1, 2, 1, 8, 2, 5, 1, 0.680f, 0.855f, 0.365f, 0.070f)         \
    X(2, 2, 1, 4, 1, 4, 1, 0.700f, 1.030f, 0.585f, 0.220f)         \
    X(2, 3, 1, 2, 2, 3, 1, 1.120f, 0.980f, 0.699f, 0.750f)         \
    X(2, 3, 1, 4, 2, 3, 1, 0.637f, 0.980f, 0.727f, 0.514f)         \
    X(2, 4, 1, 1, 2, 2, 1, 0.939f, 0.976f, 0.774f, 1.730f)         \
    X(2, 4, 1, 4, 2, 2, 1, 0.710f, 1.044f, 0.795f, 0.800f)         \
    X(2, 4, 1, 8, 2, 2, 1, 1.178f, 1.700f, 0.606f, 0.330f)         \
    X(4, 4, 2, 2, 1, 2, 2, 1.898f, 2.060f, 1.426f, 2.400f)         \
    X(2, 8, 4, 1, 1, 3, 1, 0.000f, 1.845f, 0.998f, 2.556f)         \
    X(3, 8, 4, 1, 1, 2, 1, 0.000f, 2.028f, 1.281f, 5.387f)

#define US_TILE_ROW(...) {__VA_ARGS__},
constexpr TileCfg kTileCfgs[] = {US_TILE_CFGS(US_TILE_ROW)};
#undef US_TILE_ROW
constexpr int kNumTileCfgs = sizeof(kTileCfgs) / sizeof(kTileCfgs[0]);
constexpr int kTileMaxM = 1 << 22;   // 128 columns of Y stay within 2^31 bytes

struct TileArgs {
    SpmmArgs a;
    int32_t nrb;         // row blocks of 16
    int32_t n_tiles;     // column tiles of 16 C columns
};

// LDS of a workgroup: every wavefront's NB x R payload stages (a chunk of
// four LTs each; a window may read on into what follows), then every K
// slice's activation stages.
template <int R, int C, int WM, int WK, int NB, int BITS>
struct TileStage {
    static constexpr int KC = 4;                              // LTs of a row block per chunk
    static constexpr int kPieces = 8 * BITS * KC + 2;         // 16-byte payload pieces of one row block's chunk
    static constexpr int kLoads = (kPieces + 63) / 64;
    static constexpr int kPay = 16 * kPieces;
    static constexpr int kWave = NB * R * kPay;               // payload stages of one wavefront
    static constexpr int kXBuf = 2048 * C;                    // 16 C columns x 128 bytes
    static constexpr int kGroup = (WM > 1 ? 2 : 1) * kXBuf;   // activation stages of one K slice
    static constexpr int kTotal = WM * WK * kWave + WK * kGroup;
    static constexpr int kShare = kTotal / (WM * WK) / 1024;  // combine blocks (1 KB) per wavefront
};

// 16 bytes per lane straight into LDS, as dma16, default cache policy (the
// activations are read by every row group). No memory clobber: it only writes
// a stage that nothing reads before the next wait and barrier, and the
// compiler may schedule this chunk's LDS reads around it.
__device__ __forceinline__ void dma16_x(u32x4 desc, uint32_t lds, uint32_t voff) {
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :
                     : "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(voff), "s"(desc)
                     : "m0");
}

// Two dwords shifted left by one nibble in one 64-bit shift, which issues as
// fast as a 32-bit one (4 cycles); the nibble that crosses from the first
// into the second lands in a low nibble, which every user masks off. (Written
// as assembly because the compiler, seeing the masks, splits it again.)
__device__ __forceinline__ uint2 shl4(uint32_t a, uint32_t b) {
    const u32x2 v = (u32x2){a, b};
    u32x2 q;
    __asm__("v_lshlrev_b64 %0, 4, %1" : "=v"(q) : "v"(v));
    return make_uint2(q.x, q.y);
}

// place_slots with the shift of both dwords in one instruction.
template <int BITS>
__device__ __forceinline__ i32x4 place_slots2(uint2 w, uint2 sel) {
    if constexpr (BITS == 4) {
        const uint32_t p0 = __builtin_amdgcn_perm(w.y, w.x, sel.x);
        const uint32_t p1 = __builtin_amdgcn_perm(w.y, w.x, sel.y);
        const uint2 q = shl4(p0, p1);
        return (i32x4){(int32_t)(q.x & kHiNib), (int32_t)(q.y & kHiNib), (int32_t)(p0 & kHiNib), (int32_t)(p1 & kHiNib)};
    } else {
        return place_slots<BITS>(w, sel);
    }
}

template <int R, int C, int WM, int WK, int NB, int LW, int JS, bool PERM, int BITS>
__global__ __launch_bounds__(64 * WM * WK, PERM && LW == 8 ? 7 : LW) void us_spmm_tile_kernel(
    const uint32_t *off, const uint32_t *bm32, const uint8_t *x, int32_t nkb_, int32_t n_, int32_t k_,
    int32_t pay_bytes, const uint8_t *pay, const float *scale, int32_t nrb, int32_t n_tiles, int32_t *y, float *yf,
    const uint32_t *perm32, int32_t m_) {
    using S = TileStage<R, C, WM, WK, NB, BITS>;
    constexpr int KC = S::KC;
    constexpr uint32_t kSlotsPerByte = 4 / BITS;
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ u32x2 lut[256];
    const uint32_t lds0 = (uint32_t)(size_t)(lds_u32 *)lds;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave / WM, wm = wave % WM;
    // Workgroups go to the XCDs in turn: the column tiles of one row group
    // take consecutive places on one XCD, whose L2 then serves their common
    // weights.
    const uint32_t slot = blockIdx.x >> 3;
    const uint32_t group = (slot / (uint32_t)n_tiles) * 8u + (blockIdx.x & 7u);
    const int n0 = (int)(slot % (uint32_t)n_tiles) * (16 * C);
    if (group * (WM * R) >= (uint32_t)nrb) return;            // whole workgroup
    const uint32_t rb0 = (group * WM + wm) * R;
    const int N = n_;

    const uint32_t unkb = (uint32_t)nkb_;
    const uint32_t kb0 = (uint32_t)wk * (unkb / WK) + min((uint32_t)wk, unkb % WK);
    const uint32_t nk = unkb / WK + ((uint32_t)wk < unkb % WK ? 1u : 0u);      // >= 1
    // (with shared activations every slice of the workgroup takes as many
    // chunks as the longest, the last one possibly empty)
    const uint32_t nchunk = WM > 1 ? ((unkb + WK - 1) / WK + KC - 1) / KC : (nk + KC - 1) / KC;

    const int rr = lane & 15;
    const int i = rr >> 1;
    const int g = lane >> 4;
    const uint32_t amask = (rr & 1) ? ~0u : 0u;
    const uint32_t st = lds0 + (uint32_t)(wave * S::kWave);
    const uint32_t st_x = lds0 + (uint32_t)(WM * WK * S::kWave + wk * S::kGroup);

    // The slice's offsets, masks and permutations. Row blocks past the matrix
    // repeat the last one; their sums are dropped.
    __amdgpu_buffer_rsrc_t off_s[R], bm_s[R];
    [[maybe_unused]] __amdgpu_buffer_rsrc_t perm_s[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint64_t t0 = (uint64_t)min(rb0 + r, (uint32_t)nrb - 1u) * unkb + kb0;
        off_s[r] = __builtin_amdgcn_make_buffer_rsrc((void *)(off + t0), (short)0, (int)(4u * (nk + 1u)), kBufferDword3);
        bm_s[r] = __builtin_amdgcn_make_buffer_rsrc((void *)(bm32 + 8 * t0), (short)0, (int)(32u * nk), kBufferDword3);
        if constexpr (PERM)
            perm_s[r] = __builtin_amdgcn_make_buffer_rsrc((void *)(perm32 + 2 * t0), (short)0, (int)(8u * nk), kBufferDword3);
    }

    // Activation staging: load b brings columns 8 b .. 8 b + 7 of the tile,
    // lane 8 c + p the piece p ^ c ^ (b mod 2) (16 bytes: half p mod 2 of LT
    // p / 2) of column c. Columns past N read zero, bytes past a row whatever
    // follows it (their weights are zero).
    const uint32_t xrow = (uint32_t)k_ >> 1;
    const uint64_t xa64 = (uint64_t)(size_t)x;
    const u32x4 xdesc =
        (u32x4){(uint32_t)xa64, (uint32_t)(xa64 >> 32) & 0xFFFFu, (uint32_t)N * xrow, (uint32_t)kBufferDword3};
    const uint32_t xc = (uint32_t)lane >> 3;
    const uint32_t xbase = ((uint32_t)n0 + xc) * xrow + 32u * kb0;
    const uint32_t xq0 = 16u * (((uint32_t)lane & 7u) ^ xc);  // even 8-column blocks; odd ones xor 16
    auto load_x = [&](uint32_t c, uint32_t buf) {
        const uint32_t v = xbase + 128u * c;
#pragma unroll
        for (int b0 = 0; b0 < 2 * C; b0 += WM) {
            const int b = b0 + wm;
            if ((2 * C % WM == 0 || b < 2 * C) && n0 + 8 * b < N)   // (blocks past N feed no output)
                dma16_x(xdesc, st_x + buf * S::kXBuf + 1024u * b, v + (uint32_t)(8 * b) * xrow + (xq0 ^ (uint32_t)(16 * (b & 1))));
        }
    };
    // Piece (kb = g, half h) of column 16 cb + rr.
    const uint32_t xr0 = st_x + 1024u * (uint32_t)(rr >> 3) + 128u * (uint32_t)(rr & 7);
    const uint32_t xs = (uint32_t)((rr & 7) ^ (rr >> 3));
    const uint32_t xr[2] = {xr0 + 16u * ((2u * g) ^ xs), xr0 + 16u * ((2u * g + 1u) ^ xs)};

    constexpr bool kShared = WM > 1;

    i32x4 acc[R][C];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int cb = 0; cb < C; ++cb) acc[r][cb] = (i32x4){0, 0, 0, 0};

    // A chunk's mask rows (zero past the slice) and offsets, first and end of
    // LT g (past the slice those of its last LT).
    u32x2 ov[R];
    uint32_t mv[R];
    [[maybe_unused]] uint32_t pv[R];
    auto load_rows = [&](uint32_t c) {
        const uint32_t j = KC * c + (uint32_t)g, jo = min(j, nk - 1u);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            mv[r] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(bm_s[r], 32 * j + 4 * i, 0, 0);
            ov[r] = (u32x2)__builtin_amdgcn_raw_buffer_load_b64(off_s[r], 4 * jo, 0, 0);
            if constexpr (PERM)
                pv[r] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(perm_s[r], 8 * j + 4 * (rr & 1), 0, 0);
        }
    };
    // Payload ranges of 64 chunks, one per lane: first staged byte and length.
    uint32_t pa0[R], plen[R];
    auto load_ranges = [&](uint32_t c0) {
        uint32_t ob[R], oe[R];
        const uint32_t j0 = min(KC * (c0 + (uint32_t)lane), nk), j1 = min(j0 + KC, nk);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ob[r] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(off_s[r], 4 * j0, 0, 0);
            oe[r] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(off_s[r], 4 * j1, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            pa0[r] = us_range::first_byte<BITS>(ob[r], (uint32_t)pay_bytes);
            plen[r] = us_range::value_bytes<BITS>(oe[r], pa0[r], (uint32_t)pay_bytes, (uint32_t)S::kPieces);
        }
    };
    uint32_t base[R];                                         // first staged byte of the chunk being decoded
    auto load_payload = [&](uint32_t c, uint32_t buf) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t A0 = lane_value(pa0[r], (int)(c & 63u)), len = lane_value(plen[r], (int)(c & 63u));
            const uint32_t area = st + (buf * R + r) * S::kPay;
            const uint64_t pa = (uint64_t)(size_t)pay + A0;
            const u32x4 desc = (u32x4){(uint32_t)pa, (uint32_t)(pa >> 32), len, (uint32_t)kBufferDword3};
            base[r] = A0;
#pragma unroll
            for (int u = 0; u < S::kLoads; ++u) {
                if (u + 1 < S::kLoads || S::kPieces % 64 == 0) {
                    dma16(desc, area + 1024u * u, (uint32_t)(16 * lane + 1024 * u), 0u);
                } else if (len > 1024u * u) {                 // a nearly full chunk: wave-uniform
                    __asm__ volatile("" ::: "memory");        // (keeps this a scalar branch)
                    if (lane < S::kPieces - 64 * u) dma16(desc, area + 1024u * u, (uint32_t)(16 * lane + 1024 * u), 0u);
                }
            }
        }
    };
    // Mask row and slot address of lane (rr, g)'s row in LT g of the chunk.
    uint32_t dm[R], ds[R];
    auto rows = [&](uint32_t buf) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t m = mv[r];
            uint32_t ex = dpp_row<0x112>((uint32_t)__popc(m));
            ex += dpp_row<0x112>(ex);
            ex += dpp_row<0x114>(ex);
            ex += dpp_row<0x118>(ex);
            const uint32_t at = kSlotsPerByte * (st + ((NB == 2 ? buf : 0u) * R + r) * S::kPay - base[r]);
            uint32_t s = at + (ov[r].x >> 1) + (amask & ((ov[r].y - ov[r].x) >> 2)) + ex;
            if constexpr (PERM) {
                const uint32_t row = (pv[r] >> (4 * i)) & 15u;        // original row of reordered row 8 a + i
                const int to = 4 * (int)(16u * g + (((row << 1) & 14u) | (row >> 3)));
                m = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)m);
                s = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)s);
            }
            dm[r] = m;
            ds[r] = s;
        }
    };
    // Segment j of LT g, for every lane group g: one MFMA's weight operand.
    auto decode = [&](int r, int j) {
        const uint32_t m = dm[r];
        const uint32_t s = j == 0 ? ds[r] : ds[r] + (uint32_t)__popc(m & ((1u << (8 * j)) - 1u));
        const u32x2 sv = lut[(m >> (8 * j)) & 0xFFu];
        return place_slots2<BITS>(slot_window<BITS>(s), make_uint2(sv.x, sv.y));
    };
    auto load_b = [&](uint32_t buf, int cb, int h) {
        return *(const lds_u4 *)(size_t)(xr[h] + (kShared ? buf * S::kXBuf : 0u) + 2048u * cb);
    };

    load_ranges(0);
    load_rows(0);
    load_x(0, 0);
    // Dequant scales of this lane's rows (row 8 (rr mod 2) + rr / 2 of every
    // row block), requested now so that the epilogue does not wait for them.
    const uint32_t m_in = 8u * (uint32_t)(rr & 1) + (uint32_t)i;
    float sc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) sc[r] = scale ? scale[min(rb0 + r, (uint32_t)nrb - 1u) * 16u + m_in] : 0.0f;
    for (int e = threadIdx.x; e < 256; e += 64 * WM * WK) lut[e] = perm_selectors<BITS>((uint32_t)e);
    load_payload(0, 0);
    __syncthreads();

    auto step = [&](uint32_t c, uint32_t buf, auto more) {
        __builtin_amdgcn_s_waitcnt(0);
        if constexpr (kShared) __builtin_amdgcn_s_barrier();  // this chunk's activations are in place, the last one's read
        __asm__ volatile("" ::: "memory");
        rows(buf);
        if constexpr (decltype(more)::value && kShared) load_x(c + 1, buf ^ 1u);
        if constexpr (decltype(more)::value) load_rows(c + 1);
        constexpr int KJ = KC / JS;                           // weight operands decoded at a time
        i32x4 w[R][KJ];
        auto decode_all = [&](int j0) {
#pragma unroll
            for (int j = 0; j < KJ; ++j)
#pragma unroll
                for (int r = 0; r < R; ++r) w[r][j] = decode(r, j0 + j);
        };
        [[maybe_unused]] u32x4 xb[kShared ? 1 : C][2];
        if constexpr (!kShared) {
#pragma unroll
            for (int cb = 0; cb < C; ++cb)
#pragma unroll
                for (int h = 0; h < 2; ++h) xb[cb][h] = load_b(0, cb, h);
        }
        auto request = [&]() {
            __asm__ volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xC07F);               // lgkmcnt(0): the stages have been read
            __asm__ volatile("" ::: "memory");
            if constexpr (decltype(more)::value) {
                if constexpr (!kShared) load_x(c + 1, 0u);
                if (((c + 1) & 63u) == 0) load_ranges(c + 1);
                load_payload(c + 1, NB == 2 ? buf ^ 1u : 0u);
            }
            __asm__ volatile("" ::: "memory");
        };
        if constexpr (NB == 2) request();
#pragma unroll
        for (int js = 0; js < JS; ++js) {
            decode_all(KJ * js);
            if constexpr (NB == 1)
                if (js == JS - 1) request();
            // Column blocks in turn; the next block's activations are read
            // while this one's are multiplied.
            typedef uint32_t bvec __attribute__((ext_vector_type(KJ)));
            bvec b0, b1, n0v, n1v;
            auto get = [&](int cb, bvec &v0, bvec &v1) {
                if constexpr (kShared) {
                    v0 = *(const __attribute__((address_space(3))) bvec *)(size_t)(xr[0] + buf * S::kXBuf + 2048u * cb + 4u * KJ * js);
                    v1 = *(const __attribute__((address_space(3))) bvec *)(size_t)(xr[1] + buf * S::kXBuf + 2048u * cb + 4u * KJ * js);
                } else {
                    for (int j = 0; j < KJ; ++j) v0[j] = xb[cb][0][KJ * js + j], v1[j] = xb[cb][1][KJ * js + j];
                }
            };
            get(0, b0, b1);
#pragma unroll
            for (int cb = 0; cb < C; ++cb) {
                if (cb + 1 < C) get(cb + 1, n0v, n1v);
                if constexpr (kShared) __asm__ volatile("" ::: "memory");
#pragma unroll
                for (int j = 0; j < KJ; j += 2) {
                    const int j1 = KJ > 1 ? j + 1 : j;
                    const uint2 s0 = shl4(b0[j], b0[j1]), s1 = shl4(b1[j], b1[j1]);
#pragma unroll
                    for (int t = 0; t < (KJ > 1 ? 2 : 1); ++t) {
                        const i32x4 b = (i32x4){(int32_t)((t ? s0.y : s0.x) & kHiNib), (int32_t)(b0[j + t] & kHiNib),
                                                (int32_t)((t ? s1.y : s1.x) & kHiNib), (int32_t)(b1[j + t] & kHiNib)};
#pragma unroll
                        for (int r = 0; r < R; ++r)
                            acc[r][cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(b, w[r][j + t], acc[r][cb], 0, 0, 0);
                    }
                }
                b0 = n0v;
                b1 = n1v;
            }
        }
        __asm__ volatile("" ::: "memory");
    };
    // Issue priority falls by one step per quarter of the slice: a SIMD's
    // arbiter otherwise favours its oldest wavefronts, which then run at
    // nearly the speed of a lone one while the youngest finish alone.
    const uint32_t p1 = (nchunk + 3) / 4, p2 = (nchunk + 1) / 2, p3 = (3 * nchunk + 3) / 4;
    __builtin_amdgcn_s_setprio(3);
    uint32_t c = 0;
    for (; c + 1 < nchunk; ++c) {
        if (c == p1) __builtin_amdgcn_s_setprio(2);
        if (c == p2) __builtin_amdgcn_s_setprio(1);
        if (c == p3) __builtin_amdgcn_s_setprio(0);
        step(c, c & 1u, std::integral_constant<bool, true>());
    }
    step(c, c & 1u, std::integral_constant<bool, false>());

    // Stores through buffers over this tile's columns of Y and Yf: columns
    // past N lie outside them and are dropped. (At most 128 columns of 4 M
    // bytes, 2^31 in all: the host takes this path for M <= 2^22. Sizes and
    // offsets of buffers are unsigned.)
    constexpr int kShift = BITS == 4 ? 8 : 10;
    constexpr int kBlocks = R * C;
    const uint32_t row4 = 4u * (uint32_t)m_;                  // bytes of one column of Y
    const uint32_t tile_bytes = row4 * (uint32_t)min(16 * C, N - n0);
    const __amdgpu_buffer_rsrc_t ydst =
        __builtin_amdgcn_make_buffer_rsrc((void *)(y + (int64_t)n0 * m_), (short)0, (int)tile_bytes, kBufferDword3);
    const __amdgpu_buffer_rsrc_t fdst = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(yf + (scale ? (int64_t)n0 * m_ : 0)), (short)0, scale ? (int)tile_bytes : 0, kBufferDword3);
    // Lane (rr, g), element v: row 8 (rr & 1) + rr / 2 of its row block, column 4 g + v.
    const uint32_t lane_off = 4u * m_in + (uint32_t)(4 * g) * row4;
    if constexpr (WK == 1) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (rb0 + r >= (uint32_t)nrb) break;
            const uint32_t at = lane_off + 64u * (rb0 + r);
#pragma unroll
            for (int cb = 0; cb < C; ++cb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int32_t yv = acc[r][cb][v] >> kShift;
                    const uint32_t o = at + (uint32_t)(16 * cb + v) * row4;
                    __builtin_amdgcn_raw_buffer_store_b32((uint32_t)yv, ydst, o, 0, 0);
                    if (scale) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)yv * sc[r]), fdst, o, 0, 0);
                }
        }
    } else {
        // Split-K combine, a few 16 x 16 blocks per wavefront and round: the
        // WK partials of a block's element row (64 lanes) are summed by one
        // of the wavefronts that made them.
        constexpr int kPer = S::kShare < kBlocks ? S::kShare : kBlocks;
        static_assert(kPer >= 1, "a wavefront's share of the LDS holds at least one block");
        const uint32_t mine = lds0 + (uint32_t)((wm * WK + wk) * kPer) * 1024u + 4u * lane;
#pragma unroll
        for (int b0 = 0; b0 < kBlocks; b0 += kPer) {
            __syncthreads();
#pragma unroll
            for (int b = 0; b < kPer; ++b) {
                if (b0 + b < kBlocks) {
                    const i32x4 a = acc[(b0 + b) / C][(b0 + b) % C];
#pragma unroll
                    for (int v = 0; v < 4; ++v) lds_store(mine + 1024 * b + 256 * v, (uint32_t)a[v]);
                }
            }
            __syncthreads();
            const int rows_now = 4 * (kBlocks - b0 < kPer ? kBlocks - b0 : kPer);
            for (int q = wk; q < rows_now; q += WK) {                     // wave-uniform
                const int blk = b0 + (q >> 2), v = q & 3;
                const uint32_t rb = rb0 + (uint32_t)(blk / C);
                if (rb >= (uint32_t)nrb) continue;
                const uint32_t at = lds0 + (uint32_t)(wm * WK * kPer) * 1024u + (uint32_t)q * 256u + 4u * lane;
                int32_t s = 0;
#pragma unroll
                for (int k = 0; k < WK; ++k) s += (int32_t)lds_load(at + (uint32_t)(k * kPer * 1024));
                const int32_t yv = s >> kShift;
                const uint32_t o = lane_off + 64u * rb + (uint32_t)(16 * (blk % C) + v) * row4;
                __builtin_amdgcn_raw_buffer_store_b32((uint32_t)yv, ydst, o, 0, 0);
                if (scale) {
                    float f = sc[0];
#pragma unroll
                    for (int r = 1; r < R; ++r) f = blk / C == r ? sc[r] : f;
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)yv * f), fdst, o, 0, 0);
                }
            }
        }
    }
}

template <int R, int C, int WM, int WK, int NB, int LW, int JS, bool PERM, int BITS>
hipError_t launch_tile(const TileArgs &t, hipStream_t s) {
    auto kern = us_spmm_tile_kernel<R, C, WM, WK, NB, LW, JS, PERM, BITS>;
    static std::atomic<unsigned long long> attr_set{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    const unsigned long long bit = 1ull << (dev & 63);
    if (!(attr_set.load(std::memory_order_acquire) & bit)) {
        const hipError_t e =
            hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds - kLutBytes);
        if (e != hipSuccess) return e;
        attr_set.fetch_or(bit, std::memory_order_release);
    }
    const SpmmArgs &a = t.a;
    const int groups8 = ((t.nrb + WM * R - 1) / (WM * R) + 7) / 8;
    constexpr int kLds = TileStage<R, C, WM, WK, NB, BITS>::kTotal;
    hipLaunchKernelGGL(kern, dim3(8 * groups8 * t.n_tiles), dim3(64 * WM * WK), kLds, s, a.off, a.bm32, a.x, a.nkb, a.N,
                       a.K, a.pay_bytes, a.pay, a.scale, t.nrb, t.n_tiles, a.y, a.yf, a.perm32, a.M);
    return hipGetLastError();
}

template <bool PERM, int BITS>
hipError_t launch_tile_cfg(int idx, const TileArgs &t, hipStream_t s) {
    int k = 0;
#define US_TILE_CASE(R, C, WM, WK, NB, LW, JS, ...) \
    if (idx == k++) return launch_tile<R, C, WM, WK, NB, LW, JS, PERM, BITS>(t, s);
    US_TILE_CFGS(US_TILE_CASE)
#undef US_TILE_CASE
    return hipErrorInvalidValue;
}

// The instantiations of each weight form, in translation units of their own:
// 4-bit rows in stored order, row-reordered 4-bit, 2-bit.
hipError_t launch_tile_plain(int idx, const TileArgs &t, hipStream_t s);
hipError_t launch_tile_perm(int idx, const TileArgs &t, hipStream_t s);
hipError_t launch_tile_w2(int idx, const TileArgs &t, hipStream_t s);

// LDS bytes of a workgroup of configuration c, the selector table included.
inline int tile_lds(const TileCfg &c, int bits) {
    return kLutBytes + c.WM * c.WK * c.NB * c.R * 16 * (8 * bits * 4 + 2) + c.WK * (c.WM > 1 ? 2 : 1) * 2048 * c.C;
}

// Cost of a configuration in us. Workgroups run in generations of what the
// CUs hold; a generation costs s, then per chunk the larger of one
// wavefront's latency a and the busiest SIMD's share b v (v wavefronts on
// it), blended a little as neither hides the other entirely, and e v for the
// combine and the stores. (Always inlined: every call has a constant
// configuration, which leaves two of its ten divisions.)
__attribute__((always_inline)) inline float tile_cost(const TileCfg &c, int nrb, int nkb, int N, int bits, int n_cu) {
    const int w = c.WM * c.WK;
    const long tiles = (N + 16 * c.C - 1) / (16 * c.C), groups = (nrb + c.R * c.WM - 1) / (c.R * c.WM);
    const int by_lds = kMaxLds / tile_lds(c, bits), by_regs = 4 * c.LW / w > 0 ? 4 * c.LW / w : 1;
    const int per_cu = by_lds < by_regs ? by_lds : by_regs;
    const long slots = (long)n_cu * per_cu;
    const float chunks = (float)(((nkb + c.WK - 1) / c.WK + 3) / 4);
    float t = 0.0f;
    for (long left = groups * tiles; left > 0;) {
        // (whole generations at once: they cost the same)
        const long gens = left > slots ? left / slots : 1, g = left < slots ? left : slots;
        const float v = 0.25f * (float)(w * ((g + n_cu - 1) / n_cu)), lat = c.a, iss = c.b * v;
        t += (float)gens * (c.s + chunks * (0.9f * (lat > iss ? lat : iss) + 0.1f * (lat + iss)) + c.e * v);
        left -= gens * g;
    }
    return t;
}

// The configuration with the lowest cost (its index), or -1 if K is too short
// for every configuration of that width.
template <int... I>
inline int tile_pick(int nrb, int nkb, int N, int bits, int n_cu, std::integer_sequence<int, I...>) {
    int best = -1;
    float cost = 0.0f;
    const auto consider = [&](auto k) __attribute__((always_inline)) {
        constexpr TileCfg c = kTileCfgs[decltype(k)::value];
        if (c.WK > nkb) return;                                // at least one LT per slice
        if (c.C > 1 && 16 * c.C >= N + 16) return;             // a whole column block would be empty
        const float t = bits == 2 ? tile_cost(c, nrb, nkb, N, 2, n_cu) : tile_cost(c, nrb, nkb, N, 4, n_cu);
        if (best < 0 || t < cost) {
            best = k;
            cost = t;
        }
    };
    (consider(std::integral_constant<int, I>()), ...);
    return best;
}

inline int tile_pick(int nrb, int nkb, int N, int bits, int n_cu) {
    return tile_pick(nrb, nkb, N, bits, n_cu, std::make_integer_sequence<int, kNumTileCfgs>());
}

}  // namespace us_spmm_detail

#endif  // UNIONSPARSE_US_SPMM_TILE_H
