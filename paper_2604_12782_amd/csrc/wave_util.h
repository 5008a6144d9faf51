// 64-lane reductions and the row/segment work split shared by the streaming kernels (device code only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace osc {

// 64-lane reductions on the vector ALU alone (DPP inside each row of 16 lanes, then four lane
// reads).
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v, const int ctrl_sel) {
    const int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
    int l2, h2;
    switch (ctrl_sel) {
        case 0: l2 = __builtin_amdgcn_mov_dpp(lo, 0xB1, 0xF, 0xF, true); h2 = __builtin_amdgcn_mov_dpp(hi, 0xB1, 0xF, 0xF, true); break;    // lane ^ 1
        case 1: l2 = __builtin_amdgcn_mov_dpp(lo, 0x4E, 0xF, 0xF, true); h2 = __builtin_amdgcn_mov_dpp(hi, 0x4E, 0xF, 0xF, true); break;    // lane ^ 2
        case 2: l2 = __builtin_amdgcn_mov_dpp(lo, 0x141, 0xF, 0xF, true); h2 = __builtin_amdgcn_mov_dpp(hi, 0x141, 0xF, 0xF, true); break;  // 7 - lane
        default: l2 = __builtin_amdgcn_mov_dpp(lo, 0x140, 0xF, 0xF, true); h2 = __builtin_amdgcn_mov_dpp(hi, 0x140, 0xF, 0xF, true); break; // 15 - lane
    }
    return (uint64_t)(uint32_t)h2 << 32 | (uint32_t)l2;
}
__device__ __forceinline__ uint64_t lane_u64(uint64_t v, const int l) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l) << 32 |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
}
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const uint64_t u = dpp_u64(v, s);
        v = u > v ? u : v;
    }
    const uint64_t a = lane_u64(v, 0), b = lane_u64(v, 16), c = lane_u64(v, 32), d = lane_u64(v, 48);
    const uint64_t ab = a > b ? a : b, cd = c > d ? c : d;
    return ab > cd ? ab : cd;
}
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
    for (int s = 0; s < 4; ++s) v += dpp_u64(v, s);
    return (lane_u64(v, 0) + lane_u64(v, 16)) + (lane_u64(v, 32) + lane_u64(v, 48));
}


__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true));
    v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true));
    v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true));
    v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true));
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    return max(max(a, b), max(c, d));
}

// ---- packed 16-bit magnitudes and 8-bit codes ------------------------------------------------
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
// element-wise maximum of two pairs of 16-bit magnitudes (one packed instruction)
__device__ __forceinline__ uint32_t max_pair(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
typedef unsigned int codes8 __attribute__((ext_vector_type(2)));  // eight one-byte codes
// E4M3 codes of eight bf16 values times `inv` (one rounded multiplication each), saturating at +-448
__device__ __forceinline__ codes8 fp8_codes(const uint32_t (&w)[4], float inv) {
    float p[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t lo = w[k] << 16, hi = w[k] & 0xffff0000u;
        p[2 * k] = __builtin_amdgcn_fmed3f(__fmul_rn(__builtin_bit_cast(float, lo), inv), -448.0f, 448.0f);
        p[2 * k + 1] = __builtin_amdgcn_fmed3f(__fmul_rn(__builtin_bit_cast(float, hi), inv), -448.0f, 448.0f);
    }
    int r0 = 0, r1 = 0;
    r0 = __builtin_amdgcn_cvt_pk_fp8_f32(p[0], p[1], r0, false);
    r0 = __builtin_amdgcn_cvt_pk_fp8_f32(p[2], p[3], r0, true);
    r1 = __builtin_amdgcn_cvt_pk_fp8_f32(p[4], p[5], r1, false);
    r1 = __builtin_amdgcn_cvt_pk_fp8_f32(p[6], p[7], r1, true);
    return (codes8){(uint32_t)r0, (uint32_t)r1};
}
// E4M3 codes of eight bf16 values (four packed words) with E8M0 scale code `code`, of which no value's
// exponent exceeds code + 8: the scaled conversion rounds x * 2^(127 - code) to nearest even but does not
// saturate, so magnitudes are clamped to 448 * 2^(code - 127) first, as bit patterns, two at a time
// (the codes of multiply, clamp to +-448, convert for every finite value and scale, at half the instructions).
// Products that left the bf16 range come out of exponent 255, where no bf16 pattern is the limit (448 * 2^120):
// such a block takes the multiplication and saturates as everywhere else (infinities to +-448, NaN to -448).
__device__ __forceinline__ codes8 mxfp8_codes(const uint32_t (&w)[4], uint32_t code) {
    typedef __bf16 v2bf_ __attribute__((ext_vector_type(2)));
    typedef short v2s_ __attribute__((ext_vector_type(2)));
    const uint32_t lim = ((code + 8u) << 7 | 0x60u) * 0x00010001u;
    const float scale = __builtin_bit_cast(float, code << 23);
    if (__builtin_expect(code == 247u, 0)) return fp8_codes(w, 0x1p-120f);
    uint32_t c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t mag = w[k] & 0x7fff7fffu;
        c[k] = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, mag), __builtin_bit_cast(u16x2, lim)));
        c[k] |= w[k] & 0x80008000u;
    }
    v2s_ lo = {0, 0}, hi = {0, 0};
    lo = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(lo, __builtin_bit_cast(v2bf_, c[0]), scale, false);
    lo = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(lo, __builtin_bit_cast(v2bf_, c[1]), scale, true);
    hi = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(hi, __builtin_bit_cast(v2bf_, c[2]), scale, false);
    hi = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(hi, __builtin_bit_cast(v2bf_, c[3]), scale, true);
    return (codes8){__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
}

// ---- work split of the row-streaming kernels: (row, 1024-channel segment) items --------------
constexpr int SEG_CHUNKS = 128;             // chunks per segment (two per lane)
constexpr int SEG_CH = SEG_CHUNKS * 8;      // channels per segment


struct QItem {
    int m, seg;
};
// linear work item (four per workgroup trip) -> (row, segment).  A block of 4 * quads rows (row_split) is
// 4*quads*nseg items; XCD x = workgroup % 8 owns blocks x, x+8, ...
__device__ __forceinline__ QItem quant_item(int wg, int wave, int nseg, int quads, int M) {
    const int per_block = quads * nseg;      // workgroups per block
    const int x = wg & 7, s = wg >> 3;
    const int block = x + 8 * (s / per_block);
    const int it = (s % per_block) * 4 + wave;  // item within the block, row-major (row, segment)
    QItem q;
    q.m = block * 4 * quads + it / nseg;
    q.seg = it % nseg;
    if (q.m >= M) q.m = -1;
    return q;
}

// The list of protected channels, expanded once per workgroup of T threads: one bit per channel, the list as 16-bit words, and the
// first entry of every segment (nseg + 1 of them; the list is ascending, so a segment owns a run).
template <int T>
__device__ __forceinline__ void list_expand(const int32_t* __restrict__ oidx, int K_o, int K, int nseg, int t, uint32_t* bits, int* colstart,
                                            uint16_t* och) {
    for (int i = t; i < (K >> 5); i += T) bits[i] = 0;
    __syncthreads();
    for (int o = t; o < K_o; o += T) {
        const int c = oidx[o];
        const int prev = o ? oidx[o - 1] : -1;
        if (c >= 0 && c < K) atomicOr(&bits[c >> 5], 1u << (c & 31));
        och[o] = (uint16_t)c;
        // segments that start between the previous listed channel and this one start here
        for (int s = (prev < 0 ? -1 : prev / SEG_CH) + 1; s <= c / SEG_CH && s <= nseg; ++s) colstart[s] = o;
        if (o == K_o - 1)
            for (int s = c / SEG_CH + 1; s <= nseg; ++s) colstart[s] = K_o;
    }
    __syncthreads();
}

// What a wavefront needs of the list of protected channels for the segment that its rows are in, kept in registers from row to
// row: AND masks of its lanes' two chunks, and where the segment's run of B columns comes from (two entries a lane; a longer
// run goes on in LDS).
struct SegmentList {
    int seg = -1, run0 = 0, run1 = 0;
    uint32_t keep[2][4];
    int from[2];
    __device__ __forceinline__ void take(int s, int lane, int nchunk, const uint32_t* bits, const int* colstart, const uint16_t* och) {
        seg = s;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c = s * SEG_CHUNKS + lane + 64 * i;
            const int b = c < nchunk ? reinterpret_cast<const uint8_t*>(bits)[c] : 0xff;  // one bit per channel; past the end of the row zeros
#pragma unroll
            for (int k = 0; k < 4; ++k) keep[i][k] = ((b >> (2 * k)) & 1 ? 0u : 0xffffu) | ((b >> (2 * k + 1)) & 1 ? 0u : 0xffff0000u);
        }
        run0 = __builtin_amdgcn_readfirstlane(colstart[s]);
        run1 = __builtin_amdgcn_readfirstlane(colstart[s + 1]);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int o = run0 + lane + 64 * i;
            from[i] = o < run1 ? (int)och[o] - s * SEG_CH : -1;
        }
    }
    // raw: the segment as it was
    __device__ __forceinline__ void gather(uint16_t* brow, const uint16_t* raw, int lane, const uint16_t* och) const {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t o = (uint32_t)(run0 + lane + 64 * i);
            if (o < (uint32_t)run1) brow[o] = raw[from[i]];
        }
#pragma unroll 1
        for (int o = run0 + 128 + lane; o < run1; o += 64) brow[o] = raw[(int)och[o] - seg * SEG_CH];
    }
};

}  // namespace osc
