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

// LDS_SCALES (FP8): the row scales of the tile's BM rows and the column scales of its BN columns are read from
// `tile_scales` in LDS (all BM + BN floats, past the end of Y any values) instead of global memory.
// WM x WN wavefronts of TM x TN blocks of 32 x 32.
template <int MODE, int TM, int TN, int WN = 2, bool LDS_SCALES = false, int WM = 2>
__device__ __forceinline__ void store_result(const KArgs& a, const TilePos& tp, v16f (&acc)[TM][TN],
                                             const float* tile_scales = nullptr) {
    constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave / WN, wn = wave % WN, q = lane >> 5, r = lane & 31;
    const int m0 = tp.m0, n0 = tp.n0, row_end = tp.row_end;
    const uint8_t* wp = tp.wp;
    // ---- epilogue ---------------------------------------------------------------------------
    // Result register k of lane (q, r): row 8*(k/4) + 4*q + k%4, column r of its 32x32 tile.
    // fp32: every register is one 128-byte row segment per half-wave.  bf16: neighbouring lanes
    // swap one register of each pair so that every lane owns two adjacent columns of one row and
    // writes them as one 32-bit word (even lanes row k, odd lanes row k+1).
    const float* wsc = (MODE == MODE_FP8) ? reinterpret_cast<const float*>(wp + a.off_s) : nullptr;
    const int odd = r & 1;
    const int wu_m = __builtin_amdgcn_readfirstlane(wm), wu_n = __builtin_amdgcn_readfirstlane(wn);
    // byte offset of this lane's four columns inside a 32x32 result tile: row 4q + r%4, columns 4(r/4) ..
    const uint32_t yoff8 = 2u * (uint32_t)((4 * q + (r & 3)) * (int)a.ldy + (r & ~3));
    const bool hi2 = (r & 2) != 0;
    // 16-byte stores of eight bf16 columns need rows that keep 16-byte alignment
    const bool wide16 = (a.ldy & 7) == 0 && (reinterpret_cast<uintptr_t>(a.Y) & 15) == 0;
    // byte selector of step 2: even lanes [own.lo, other.lo], odd lanes [other.hi, own.hi]
    const uint32_t sel12 = odd ? 0x03020706u : 0x05040100u;
    auto store_tile = [&](auto kind_tag) __attribute__((always_inline)) {
        // 2: tile entirely inside Y, no bounds tests; 1: all columns inside, rows tested (ragged
        // last tile of a problem or an expert); 0: everything tested, 2-byte stores
        constexpr int KIND = decltype(kind_tag)::value;
        constexpr bool FULL = KIND == 2;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int rbase = m0 + wm * (TM * 32) + i * 32 + 4 * q;
            float xr[16];
            if (MODE == MODE_FP8) {
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const int row = rbase + 8 * (k >> 2) + (k & 3);
                    if constexpr (LDS_SCALES) xr[k] = tile_scales[row - m0];
                    else xr[k] = a.xs[FULL ? row : min(row, row_end - 1)];
                }
            }
            int j0 = 0;
            if constexpr (KIND >= 1 && TN >= 2) {
                if (a.y_bf16 && wide16) {
                    // 16-byte stores: the two exchange rounds described below, on two neighbouring tiles,
                    // then a third between lanes l and l^4: lanes of even column groups complete eight
                    // adjacent columns of the left tile, the others of the right tile, so one store
                    // instruction writes eight rows of 128 contiguous bytes.
                    const bool lo4 = (r & 4) != 0;
                    const uint32_t yoff16 = 2u * (uint32_t)((4 * q + (r & 3)) * (int)a.ldy + (r & ~3) + (lo4 ? 28 : 0));
#pragma unroll
                    for (int jp = 0; jp + 1 < TN; jp += 2) {
                        u32x2 o[2][4];
#pragma unroll
                        for (int s2 = 0; s2 < 2; ++s2) {
                            const int j = jp + s2;
                            float cs = 1.0f;
                            if (MODE == MODE_FP8) cs = LDS_SCALES ? tile_scales[BM + wn * (TN * 32) + j * 32 + r] : wsc[n0 + wn * (TN * 32) + j * 32 + r];
                            uint32_t P[8], W[8];
#pragma unroll
                            for (int k = 0; k < 8; ++k) {
                                const float v0 = (MODE == MODE_FP8) ? acc[i][j][2 * k] * (xr[2 * k] * cs) : acc[i][j][2 * k];
                                const float v1 = (MODE == MODE_FP8) ? acc[i][j][2 * k + 1] * (xr[2 * k + 1] * cs)
                                                                     : acc[i][j][2 * k + 1];
                                const v2f pair = {v0, v1};
                                P[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, v2bf));
                            }
#pragma unroll
                            for (int k = 0; k < 8; ++k) {
                                const uint32_t Q = (uint32_t)__builtin_amdgcn_mov_dpp((int)P[k], 0xB1, 0xF, 0xF, true);
                                W[k] = __builtin_amdgcn_perm(Q, P[k], sel12);
                            }
#pragma unroll
                            for (int h = 0; h < 4; ++h) {
                                const uint32_t ra = (uint32_t)__builtin_amdgcn_mov_dpp((int)W[2 * h], 0x4E, 0xF, 0xF, true);
                                const uint32_t rb = (uint32_t)__builtin_amdgcn_mov_dpp((int)W[2 * h + 1], 0x4E, 0xF, 0xF, true);
                                o[s2][h] = (u32x2){hi2 ? rb : W[2 * h], hi2 ? W[2 * h + 1] : ra};
                            }
                        }
                        uint8_t* const ybase = reinterpret_cast<uint8_t*>(a.Y) +
                            2 * ((int64_t)(m0 + wu_m * (TM * 32) + i * 32) * a.ldy + n0 + wu_n * (TN * 32) + jp * 32);
#pragma unroll
                        for (int h = 0; h < 4; ++h) {
                            // lane + 4 sends its left-tile words down, lane - 4 its right-tile words up
                            const uint32_t dx = (uint32_t)__builtin_amdgcn_mov_dpp((int)o[0][h].x, 0x104, 0xF, 0xF, true);
                            const uint32_t dy = (uint32_t)__builtin_amdgcn_mov_dpp((int)o[0][h].y, 0x104, 0xF, 0xF, true);
                            const uint32_t ux = (uint32_t)__builtin_amdgcn_mov_dpp((int)o[1][h].x, 0x114, 0xF, 0xF, true);
                            const uint32_t uy = (uint32_t)__builtin_amdgcn_mov_dpp((int)o[1][h].y, 0x114, 0xF, 0xF, true);
                            const u32x4 out = {lo4 ? ux : o[0][h].x, lo4 ? uy : o[0][h].y, lo4 ? o[1][h].x : dx,
                                               lo4 ? o[1][h].y : dy};
                            uint8_t* const hbase = ybase + 2 * (int64_t)(8 * h) * a.ldy;
                            if (FULL || rbase + 8 * h + (r & 3) < row_end)
                                __builtin_nontemporal_store(out, reinterpret_cast<u32x4*>(hbase + yoff16));
                        }
                    }
                    j0 = TN & ~1;
                }
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (j < j0) continue;  // stored in pairs above
                const int col = n0 + wn * (TN * 32) + j * 32 + r;
                float cs = 1.0f;
                if (MODE == MODE_FP8) cs = LDS_SCALES ? tile_scales[BM + col - n0] : wsc[FULL ? col : min(col, a.N - 1)];
                float v[16];
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    v[k] = (MODE == MODE_FP8) ? acc[i][j][k] * (xr[k] * cs) : acc[i][j][k];
                if (a.y_bf16 && KIND >= 1) {
                    // 8-byte stores: two rounds of exchanges inside each quad of lanes turn "one column,
                    // sixteen rows per lane" into "four adjacent columns of one row per lane".
                    //  1. pairs of result registers (rows R, R+1 of column c) are rounded to packed bf16;
                    //  2. lanes c, c^1 swap halves: even lanes get row R, odd lanes row R+1, columns c&~1, +1;
                    //  3. lanes l, l^2 swap words of register pairs (k, k+2): lanes 0,1 of a quad complete
                    //     rows R, R+1, lanes 2,3 rows R+2, R+3, columns 4b .. 4b+3.
                    // Each step runs over all registers of the tile before the next one starts, so the
                    // single wavefront of a SIMD always has independent instructions to issue.
                    uint8_t* const ybase = reinterpret_cast<uint8_t*>(a.Y) +
                        2 * ((int64_t)(m0 + wu_m * (TM * 32) + i * 32) * a.ldy + n0 + wu_n * (TN * 32) + j * 32);
                    uint32_t P[8], W[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const v2f pair = {v[2 * k], v[2 * k + 1]};
                        P[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, v2bf));
                    }
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const uint32_t Q = (uint32_t)__builtin_amdgcn_mov_dpp((int)P[k], 0xB1, 0xF, 0xF, true);
                        W[k] = __builtin_amdgcn_perm(Q, P[k], sel12);
                    }
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        // both words cross to lane l^2; each lane keeps one of its own and one of the other's
                        // (every crossing has a single use, so it folds into the select that consumes it)
                        const uint32_t ra = (uint32_t)__builtin_amdgcn_mov_dpp((int)W[2 * h], 0x4E, 0xF, 0xF, true);
                        const uint32_t rb = (uint32_t)__builtin_amdgcn_mov_dpp((int)W[2 * h + 1], 0x4E, 0xF, 0xF, true);
                        const u32x2 out = {hi2 ? rb : W[2 * h], hi2 ? W[2 * h + 1] : ra};
                        uint8_t* const hbase = ybase + 2 * (int64_t)(8 * h) * a.ldy;
                        if (FULL || rbase + 8 * h + (r & 3) < row_end)
                            __builtin_nontemporal_store(out, reinterpret_cast<u32x2*>(hbase + yoff8));
                    }
                } else if (a.y_bf16) {
                    uint16_t* Y = reinterpret_cast<uint16_t*>(a.Y);
#pragma unroll
                    for (int k = 0; k < 16; k += 2) {
                        const float send = odd ? v[k] : v[k + 1];
                        // neighbour lane's value: DPP quad_perm [1,0,3,2]
                        const float recv = __builtin_bit_cast(
                            float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), 0xB1, 0xF, 0xF, false));
                        const float lo = odd ? recv : v[k], hi = odd ? v[k + 1] : recv;
                        const int row = rbase + 8 * (k >> 2) + (k & 3) + odd;
                        const int c0 = col - odd;
                        uint16_t* dst = Y + (int64_t)row * a.ldy + c0;
                        const uint32_t word =
                            (uint32_t)f32_to_bf16_rne(lo) | ((uint32_t)f32_to_bf16_rne(hi) << 16);
                        if (row < row_end) {
                            if (c0 < a.N) dst[0] = (uint16_t)word;
                            if (c0 + 1 < a.N) dst[1] = (uint16_t)(word >> 16);
                        }
                    }
                } else {
                    float* Y = reinterpret_cast<float*>(a.Y);
#pragma unroll
                    for (int k = 0; k < 16; ++k) {
                        const int row = rbase + 8 * (k >> 2) + (k & 3);
                        if (FULL || (row < row_end && (KIND == 1 || col < a.N))) Y[(int64_t)row * a.ldy + col] = v[k];
                    }
                }
            }
        }
    };
    // 32-bit stores of bf16 pairs need an even leading dimension and a 4-byte aligned Y
    const bool cols = (n0 + BN <= a.N) &&
                      (!a.y_bf16 || (((a.ldy & 3) == 0) && ((reinterpret_cast<uintptr_t>(a.Y) & 7) == 0)));
    if (cols && m0 + BM <= row_end)
        store_tile(std::integral_constant<int, 2>{});
    else if (cols)
        store_tile(std::integral_constant<int, 1>{});
    else
        store_tile(std::integral_constant<int, 0>{});
}

// Flowing kernel (gemm_flow.hip).  flow_choose: the tile that should be fastest for one problem (-1: too few stages for
// any) and what it should cost; flow_fits: whether a tile (0: 128 x 256, 1: 128 x 192, 2: 128 x 128, 3: 64 x 128;
// experts: 0 only) can serve a launch.
bool flow_fits(int mode, int tile, int stages, bool grouped, int E);
int flow_choose(int mode, int64_t M, int64_t N, int stages, int ncu, double* cost);
int launch_flow(const KArgs& a, int mode, int tile, hipStream_t st);

}  // namespace osc
