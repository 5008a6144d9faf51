// Device code shared by the GEMM kernels: the operands of a launch, tile positions and the epilogue.
#pragma once
#include <type_traits>

#include "osc_internal.h"
#include "lds_dma.h"

namespace osc {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int GT = 256;  // 4 wavefronts, arranged 2 x 2 over the workgroup tile
enum { MODE_DUAL = 0, MODE_FP8 = 1, MODE_MX8 = 2 };  // MX8: E4M3 codes with E8M0 block scales on both operands

struct KArgs {
    const uint8_t* Xq;
    const uint8_t* Xs;
    const float* xs;
    const uint8_t* B;
    int64_t bpitch;  // bytes per row of B
    const int32_t* row_map;
    const int32_t* off;
    int E;
    const uint8_t* Wpack;
    size_t pack_stride, off_q, off_s, off_l, off_z;
    int64_t wlpitch;  // bytes per row of W_L^T
    int M, N, K, K_o;
    void* Y;
    int y_bf16;
    int64_t ldy;
    int tiles_n;
};



struct TilePos {
    int m0, n0, row_begin, row_end;
    const uint8_t* wp;
    bool valid;
};

// Workgroups are dealt round-robin to the 8 XCDs; renumber so that each XCD owns a contiguous
// run of tiles and its L2 sees neighbouring tiles.  Single problem: tiles walk down bands of 8
// m-tiles.  Grouped: m-tiles are numbered expert by expert (the grid is an upper bound).
template <int BM, int BN>
__device__ __forceinline__ TilePos tile_at(const KArgs& a, int tile);

template <int BM, int BN>
__device__ __forceinline__ TilePos locate_tile(const KArgs& a) {
    int tile = blockIdx.x;
    if (a.off) {
        // grouped: XCD x takes m-tiles x, x+8, ... and walks the n-tiles of each in turn (they share
        // the activation rows).  The surplus m-tiles at the end of the numbering (the grid is an
        // upper bound, a multiple of 8 m-tiles) are then spread over all XCDs.
        const int x = tile & 7, sidx = tile >> 3;
        tile = ((sidx / a.tiles_n) * 8 + x) * a.tiles_n + sidx % a.tiles_n;
    } else {
        const int per = gridDim.x >> 3;
        if (tile < (per << 3)) tile = (tile & 7) * per + (tile >> 3);
    }
    return tile_at<BM, BN>(a, tile);
}

// position of tile number `tile` (numbered so that neighbours share operand panels)
template <int BM, int BN>
__device__ __forceinline__ TilePos tile_at(const KArgs& a, int tile) {
    TilePos p;
    p.row_begin = 0;
    p.row_end = a.M;
    p.wp = a.Wpack;
    p.valid = true;
    int tm_idx, tn_idx;
    if (a.off) {
        // m-tiles are numbered expert by expert.  Every wavefront finds the expert of m-tile j by
        // itself: 64 experts at a time, one per lane, prefix sum of their tile counts, first lane
        // whose running total exceeds j.  (A serial walk over the offsets costs one dependent
        // memory round trip per expert.)
        tn_idx = tile % a.tiles_n;
        const int j = tile / a.tiles_n;
        const int lane = threadIdx.x & 63;
        int before = 0, e_found = -1, j_in = 0;
        for (int e0 = 0; e0 < a.E; e0 += 64) {
            const int e = e0 + lane;
            const int b = e < a.E ? a.off[e] : 0;
            const int n = e < a.E ? a.off[e + 1] - b : 0;
            const int te = (n + BM - 1) / BM;
            int ps = te;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int v = __shfl_up(ps, d);
                if (lane >= d) ps += v;
            }
            const int total = __shfl(ps, 63);
            if (j < before + total) {
                const int l = __ffsll((unsigned long long)__ballot(before + ps > j)) - 1;
                e_found = e0 + l;
                j_in = j - (before + __shfl(ps, l) - __shfl(te, l));
                p.row_begin = __shfl(b, l);
                p.row_end = p.row_begin + __shfl(n, l);
                break;
            }
            before += total;
        }
        e_found = __builtin_amdgcn_readfirstlane(e_found);
        j_in = __builtin_amdgcn_readfirstlane(j_in);
        p.row_begin = __builtin_amdgcn_readfirstlane(p.row_begin);
        p.row_end = __builtin_amdgcn_readfirstlane(p.row_end);
        if (e_found < 0) {  // surplus workgroup (the grid is an upper bound)
            p.valid = false;
            e_found = 0;
        }
        tm_idx = j_in;
        p.wp += (size_t)e_found * a.pack_stride;
    } else {
        const int tiles_m = (a.M + BM - 1) / BM;
        const int band = tile / (8 * a.tiles_n), within = tile - band * 8 * a.tiles_n;
        const int rows = min(8, tiles_m - band * 8);
        tm_idx = band * 8 + within % rows;
        tn_idx = within / rows;
    }
    p.m0 = p.row_begin + tm_idx * BM;
    p.n0 = tn_idx * BN;
    return p;
}

// First column in the tile of block j of wavefront column w (of WN), TN blocks each: pairs of blocks first, then the last blocks of an
// odd TN side by side.  So every pair begins on a 128-byte line of bf16 results and two last blocks share one.  With a wavefront's blocks in a
// row, 128 x 192 tiles had half of their pairs across two lines: 512 x 12288 x 4096 wrote 14.3 MB for 12.0, now 12.3, and 12.0 with the halves of
// a shared line stored plainly, so that they meet in L2; 25.9 -> 25.6 us with the quantiser, 1000 x 6144 x 4096 24.0 -> 23.5.  (64 x 128 tiles, whose
// wavefronts hold a last block each, stream it: 128 x 8192 x 4096 13.5 us, 13.6 with plain stores, 1000 x 2048 x 2048 10.1 and 10.3.)
template <int TN, int WN>
constexpr int block_col(int w, int j) {
    return TN % 2 && j == TN - 1 ? 32 * (WN * (TN - 1) + w) : 32 * (w * (TN & ~1) + j);
}

// Column in the tile that lane r = p % 32 of block p / 32 (of TN * WN) holds with store_pairs below: the kernel places that weight row of the tile on
// LDS row p.  Blocks 2b and 2b + 1 of a wavefront share 64 columns: a lane's two results of one row are neighbours, and lanes r and
// r ^ 16 hold four columns in a row.  In the last block of an odd TN those lanes hold neighbours.
template <int TN, int WN = 1>
constexpr int pair_col(int p) {
    const int w = TN % 2 ? (int)((uint32_t)p / (32 * TN)) : 0, o = TN % 2 ? (int)((uint32_t)p % (32 * TN)) : p & 63;
    const int c = o & 15, h = (o >> 4) & 1, j = o >> 5;
    if (TN % 2 && j == TN - 1) return block_col<TN, WN>(w, j) + 2 * c + h;
    return (TN % 2 ? block_col<TN, WN>(w, j & ~1) : p & ~63) + 4 * c + 2 * h + (j & 1);
}
template <int TN, int WN>
constexpr bool pairs_on_lines() {  // every column of the tile once, pairs of blocks on whole lines of bf16
    uint32_t seen[TN * WN] = {};
    for (int p = 0; p < 32 * TN * WN; ++p) seen[pair_col<TN, WN>(p) / 32] |= 1u << (pair_col<TN, WN>(p) % 32);
    for (int b = 0; b < TN * WN; ++b)
        if (seen[b] != ~0u || (b % TN % 2 == 0 && b % TN + 1 < TN && block_col<TN, WN>(b / TN, b % TN) % 64 != 0)) return false;
    return true;
}
static_assert(pairs_on_lines<1, 4>() && pairs_on_lines<2, 2>() && pairs_on_lines<2, 4>() && pairs_on_lines<3, 2>() && pairs_on_lines<4, 2>(), "tile's columns");

// Where lane r finds its row's scale word of a pair of weight blocks' first block: a block's words lie in the order of the rows, four
// bytes each, `block` bytes from block to block; the second block's is the word behind it.  A read takes every second word of two
// blocks, so with 32 banks lanes r and r ^ 8 meet wherever the blocks' 16-byte pieces lie (exchanging the half stages of every second block
// changed no count): 2.3 cycles a read by the counter.  That is off the critical path: with every conflict gone (words of other rows, so
// wrong results) attention and feed-forward blocks of 8192 tokens and the experts run 0 to 0.4 % faster, one round of 128 x 192 tiles 0.8 %.
// Both words by one 8-byte read, which the lane halves shift: 8192 tokens, attention block 253 -> 259 us, feed-forward 892 -> 900;
// words requested in the order of the lanes (MXFP8, persistent kernel): no conflicts, 8192 x 4096 x 12288 387 -> 391 us.
__device__ __forceinline__ uint32_t pair_scale(int r, uint32_t block) {
    return ((uint32_t)(r >> 3) & 1) * block + (4 * ((uint32_t)r & 7) + 2 * ((uint32_t)r >> 4)) * 4;
}

// Where four bf16 columns of a row leave at once (two in the last block of 64 x 128 tiles), the flowing, DMA, staged and ring kernels stream
// them past the caches; the persistent kernel stores plainly, which its next tiles gain by (8192 x 24576 x 4096 dual path 520 -> 501 us in a
// feed-forward block, the SwiGLU pass behind it 81.7 -> 79.6; 8192 x 1024 x 4096 on the flowing kernel 25.8 -> 27.3).  fp32 results and those
// that leave element by element are plain stores everywhere.
template <bool CACHED, class T>
__device__ __forceinline__ void store_y(T v, uint8_t* p) {
    if constexpr (CACHED) *reinterpret_cast<T*>(p) = v;
    else __builtin_nontemporal_store(v, reinterpret_cast<T*>(p));
}

// Epilogue: WM x WN wavefronts of TM x TN blocks of 32 x 32, columns dealt to the lanes as pair_col() says.  Result register k of
// lane (q, r) is row 8 (k / 4) + 4 q + k % 4 of its block.  Turning "one column, sixteen rows a lane" into rows takes one
// conversion per two results and one exchange of lanes r and r ^ 16 per four (per two in the last block of an odd TN), and 16
// lanes store 128 (64) bytes of a row.  With the columns in order it took three rounds of lane exchanges, seven instructions per
// two results, for 16-byte stores: 8192 x 8192 x 512 dual path 53 us then, 48 now; 300 x 4096 x 2048 8.2 and 7.3;
// 8192 x 24576 x 4096 482 and 456 (with the first products of a tile starting from zero, see the persistent kernel).
// LDS_SCALES (FP8): the tile's BM row scales and BN column scales are read from `tile_scales` in LDS (past the end of Y any
// values), not from memory.  WHOLE: the tile lies inside Y.  ACC_REGS: the accumulators fill the accumulation registers, and
// every result is read from there by itself (left to the compiler, whole blocks are copied and spilled at the head of the
// epilogue: 82 registers in the MXFP8 form of the persistent kernel).
template <int MODE, int TM, int TN, int WN, int WM, bool LDS_SCALES = false, bool WHOLE = false, bool ACC_REGS = false>
__device__ __forceinline__ void store_pairs(const KArgs& a, const TilePos& tp, v16f (&acc)[TM][TN],
                                            const float* tile_scales = nullptr) {
    constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN;
    typedef float v2f4 __attribute__((ext_vector_type(2), aligned(4)));  // (wide stores need 4-byte alignment only)
    typedef unsigned int u32x4_4 __attribute__((ext_vector_type(4), aligned(4)));
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / WN, wn = wave % WN, q = lane >> 5, r = lane & 31;
    int64_t ldy = a.ldy;
    if constexpr (ACC_REGS) {  // the asm reads below are not known to the compiler as reads of a matrix instruction's result
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 15\n\ts_nop 15");
        __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("" : "+s"(ldy));  // the row addresses are worked out here: hoisted out of the tile loop they spill
    // KIND 2: tile inside Y; 1: columns inside, rows tested; 0: everything tested, bf16 element by element
    auto store = [&](auto kind_tag, auto bf16_tag) __attribute__((always_inline)) {
        constexpr int KIND = decltype(kind_tag)::value;
        constexpr bool BF16 = decltype(bf16_tag)::value;
        constexpr int SZ = BF16 ? 2 : 4;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row0 = tp.m0 + wm * (TM * 32) + i * 32, rl = 4 * q;  // uniform, this lane's
            float xr[16];
            if constexpr (MODE == MODE_FP8) {
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const int row = row0 + rl + 8 * (k >> 2) + (k & 3);
                    if constexpr (LDS_SCALES) xr[k] = tile_scales[row - tp.m0];
                    else xr[k] = a.xs[KIND == 2 ? row : min(row, tp.row_end - 1)];
                }
            }
            auto column_scale = [&](int col) __attribute__((always_inline)) -> float {
                if constexpr (MODE != MODE_FP8) return 1.0f;
                else if constexpr (LDS_SCALES) return tile_scales[BM + col - tp.n0];
                else return reinterpret_cast<const float*>(tp.wp + a.off_s)[KIND >= 1 ? col : min(col, a.N - 1)];
            };
            auto result = [&](int j, int k, float scale) __attribute__((always_inline)) -> float {
                float v = acc[i][j][k];
                if constexpr (ACC_REGS) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(acc[i][j][k]));
                if constexpr (MODE == MODE_FP8) return v * (xr[k] * scale);
                else return v;
            };
            // two neighbouring columns of a row, at p
            auto store2 = [&](uint8_t* p, int row, int col, v2f v) __attribute__((always_inline)) {
                if (KIND < 2 && !WHOLE && row >= tp.row_end) return;
                if constexpr (BF16) {
                    const uint32_t word = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, v2bf));
                    if constexpr (KIND >= 1) {
                        store_y<WHOLE || (TN > 1)>(word, p);
                    } else {
                        uint16_t* const dst = reinterpret_cast<uint16_t*>(p);
                        if (WHOLE || col < a.N) dst[0] = (uint16_t)word;
                        if (WHOLE || col + 1 < a.N) dst[1] = (uint16_t)(word >> 16);
                    }
                } else {
                    float* const dst = reinterpret_cast<float*>(p);
                    if (KIND >= 1 || WHOLE || col + 1 < a.N) *reinterpret_cast<v2f4*>(dst) = v;
                    else if (col < a.N) dst[0] = v.x;
                }
            };
#pragma unroll
            for (int j = 0; j < TN; j += 2) {
                const int col0 = tp.n0 + block_col<TN, WN>(wn, j);
                uint8_t* p = reinterpret_cast<uint8_t*>(a.Y) + SZ * ((int64_t)row0 * ldy + col0);
                if constexpr (TN % 2 == 1)
                    if (j + 1 == TN) {
                        const int held = 2 * (r & 15) + (r >> 4);
                        const float cs = column_scale(col0 + held);
                        p += SZ * ((rl + (r >> 4)) * ldy + 2 * (r & 15));
#pragma unroll
                        for (int k = 0; k < 16; k += 2) {
                            const u32x2 o = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, result(j, k, cs)),
                                                                             __builtin_bit_cast(uint32_t, result(j, k + 1, cs)), false, false);
                            const uint32_t o0 = o.x, o1 = o.y;
                            store2(p, row0 + rl + (r >> 4) + 8 * (k >> 2) + (k & 2), col0 + 2 * (r & 15),
                                   (v2f){__builtin_bit_cast(float, o0), __builtin_bit_cast(float, o1)});
                            p += (k & 2 ? 6 : 2) * SZ * ldy;
                        }
                        break;
                    }
                const int jr = j + 1 < TN ? j + 1 : j;
                const int lc = 4 * (r & 15) + 2 * (r >> 4);  // this lane's columns lc, lc + 1 of the pair's 64
                const float c0 = column_scale(col0 + lc), c1 = column_scale(col0 + lc + 1);
                auto both = [&](int k) __attribute__((always_inline)) -> v2f { return (v2f){result(j, k, c0), result(jr, k, c1)}; };
                if constexpr (BF16 && KIND >= 1) {
                    const uint32_t off = 2u * (uint32_t)((rl + (r >> 4)) * (int)ldy + 4 * (r & 15));
#pragma unroll
                    for (int k = 0; k < 16; k += 2) {
                        // lanes 0..15 of a half keep row k of both lanes of an exchange, lanes 16..31 row k + 1
                        const u32x2 out = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, __builtin_convertvector(both(k), v2bf)),
                                                                           __builtin_bit_cast(uint32_t, __builtin_convertvector(both(k + 1), v2bf)),
                                                                           false, false);
                        if (KIND == 2 || row0 + rl + (r >> 4) + 8 * (k >> 2) + (k & 2) < tp.row_end)
                            store_y<WHOLE>(out, p + off);
                        p += (k & 2 ? 6 : 2) * SZ * ldy;
                    }
                } else if constexpr (KIND >= 1) {
                    p += SZ * ((rl + (r >> 4)) * ldy + 4 * (r & 15));
#pragma unroll
                    for (int k = 0; k < 16; k += 2) {
                        const v2f a0 = both(k), a1 = both(k + 1);
                        const float x0 = a0.x, y0 = a0.y, x1 = a1.x, y1 = a1.y;
                        const u32x2 x = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x0), __builtin_bit_cast(uint32_t, x1), false, false);
                        const u32x2 y = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, y0), __builtin_bit_cast(uint32_t, y1), false, false);
                        if (KIND == 2 || row0 + rl + (r >> 4) + 8 * (k >> 2) + (k & 2) < tp.row_end)
                            *reinterpret_cast<u32x4_4*>(p) = (u32x4_4){x.x, y.x, x.y, y.y};
                        p += (k & 2 ? 6 : 2) * SZ * ldy;
                    }
                } else {
                    p += SZ * (rl * ldy + lc);
#pragma unroll
                    for (int k = 0; k < 16; ++k) {
                        store2(p, row0 + rl + 8 * (k >> 2) + (k & 3), col0 + lc, both(k));
                        p += ((k & 3) == 3 ? 5 : 1) * SZ * ldy;
                    }
                }
            }
        }
    };
    const std::integral_constant<int, 0> any{};
    const std::integral_constant<int, 1> rows{};
    const std::integral_constant<int, 2> inside{};
    // bf16: 8-byte stores of four columns
    const bool wide = !a.y_bf16 || ((ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(a.Y) & 7) == 0);
    if (wide && (WHOLE || (tp.n0 + BN <= a.N && tp.m0 + BM <= tp.row_end))) {
        if (a.y_bf16) store(inside, std::true_type{});
        else store(inside, std::false_type{});
    } else if (!WHOLE && wide && tp.n0 + BN <= a.N) {
        if (a.y_bf16) store(rows, std::true_type{});
        else store(rows, std::false_type{});
    } else {
        if (a.y_bf16) store(any, std::true_type{});
        else if (!WHOLE) store(any, std::false_type{});
    }
}

// Flowing kernel (gemm_flow.hip).  flow_choose: the tile that should be fastest for one problem (-1: too few stages for
// any) and what it should cost; flow_fits: whether a tile (0: 128 x 256, 1: 128 x 192, 2: 128 x 128, 3: 64 x 128;
// experts: 0 only) can serve a launch.
bool flow_fits(int mode, int tile, int stages, bool grouped, int E);
int flow_choose(int mode, int64_t M, int64_t N, int stages, int ncu, double* cost);
int launch_flow(const KArgs& a, int mode, int tile, hipStream_t st);

}  // namespace osc
