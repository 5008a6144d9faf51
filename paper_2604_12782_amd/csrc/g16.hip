// 4-bit formats whose scale group is 16 channels (Section 3.1: G in {16, 32, 64}; Table 2, row
// G = 16; NVFP4 is named in the abstract and the conclusion): the OSC-enhanced quantiser (Alg. 2)
// and the dual-path layer (Eq. dual-path) for
//   format 0: E2M1 elements, one E8M0 scale per 16 channels (shared exponent floor(log2 amax) - 2);
//   format 1: NVFP4 - E2M1 elements, one E4M3 scale per 16 channels, one single-precision scale per
//             tensor, each step one IEEE single-precision operation (see osc.h).
// The matrix core scales blocks of 32 with powers of two only, so neither format can be multiplied
// as 4-bit operands.  What the formats buy is bytes: in the weight-bound (decode) regime of Table 2
// the layer streams 0.56 bytes per weight instead of 1.  The GEMM here is that regime's kernel: the
// 4-bit codes travel through HBM, L2 and LDS as they are and are expanded to bf16 in registers with
// their scale folded in (E2M1 x E8M0 and E2M1 x E4M3 are exact in bf16), then multiplied on the bf16
// (NVFP4: fp16) matrix core into fp32; the tensor scales are applied once, before the bf16 branch is added.
#include "osc_internal.h"
#include "lds_dma.h"
#include "wave_util.h"

namespace osc {

typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int QT16 = 256;

// ------------------------------------------------------------------------------------------
// Quantiser: the work split, the table expansion and the gather of quant_mxfp4_osc_kernel (one
// wavefront per 1024-channel segment of a row, two 16-byte chunks per lane); a block of 16 channels
// is two neighbouring lanes, its scale byte leaves as one of four in a 32-bit word (plain row-major
// [M, K/16], so K must be a multiple of 64).
// ------------------------------------------------------------------------------------------
template <int FMT>
__global__ void __launch_bounds__(QT16) quant_fp4_g16_kernel(
    const uint16_t* __restrict__ X, int M, int K, int64_t ldx, const int32_t* __restrict__ oidx, int K_o, float ts,
    uint8_t* __restrict__ Xq, uint8_t* __restrict__ Xs, uint16_t* __restrict__ B, int64_t ldb, int nseg, int quads, int total_wg) {
    extern __shared__ uint32_t smem[];
    const int nchunk = K >> 3;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    u32x4* strip = reinterpret_cast<u32x4*>(smem) + wave * SEG_CHUNKS;
    uint32_t* keep = smem + 4 * SEG_CHUNKS * 4;
    int* colstart = reinterpret_cast<int*>(keep + (K >> 1));
    uint16_t* och = reinterpret_cast<uint16_t*>(colstart + nseg + 1);
    if (K_o > 0) {
        for (int i = t; i < (K >> 1); i += QT16) keep[i] = 0xffffffffu;
        for (int i = t; i <= nseg; i += QT16) colstart[i] = K_o;
        __syncthreads();
        for (int o = t; o < K_o; o += QT16) {
            const int c = oidx[o];
            const int prev = o ? oidx[o - 1] : -1;
            if (c >= 0 && c < K) atomicAnd(&keep[c >> 1], (c & 1) ? 0x0000ffffu : 0xffff0000u);
            och[o] = (uint16_t)c;
            for (int sgm = (prev < 0 ? -1 : prev / SEG_CH) + 1; sgm <= c / SEG_CH && sgm <= nseg; ++sgm) colstart[sgm] = o;
        }
        __syncthreads();
    }
    const float d6 = __fmul_rn(6.0f, ts);
    for (int wg = blockIdx.x; wg < total_wg; wg += gridDim.x) {
        const QItem cur = quant_item(wg, wave, nseg, quads, M);
        if (cur.m < 0) continue;
        const int m = cur.m, cbase = cur.seg * SEG_CHUNKS;
        const u32x4* src = reinterpret_cast<const u32x4*>(X + (int64_t)m * ldx);
        uint32_t* dst = reinterpret_cast<uint32_t*>(Xq + (int64_t)m * (K >> 1));
        uint32_t* sdst = reinterpret_cast<uint32_t*>(Xs + (int64_t)m * (K >> 4));
        u32x4 v[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c = cbase + lane + 64 * i;
            v[i] = (u32x4){0u, 0u, 0u, 0u};
            if (c < nchunk) v[i] = __builtin_nontemporal_load(src + c);
        }
        if (K_o > 0) {
            strip[lane] = v[0];
            strip[lane + 64] = v[1];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c = cbase + lane + 64 * i;
            u32x4 w = v[i];
            if (K_o > 0 && c < nchunk) w &= *reinterpret_cast<const u32x4*>(keep + 4 * c);  // steps 2-3 of Section 3.2
            const u32x4 ab = w & 0x7fff7fffu;
            uint32_t a = max(max(ab.x & 0xffffu, ab.x >> 16), max(ab.y & 0xffffu, ab.y >> 16));
            a = max(a, max(max(ab.z & 0xffffu, ab.z >> 16), max(ab.w & 0xffffu, ab.w >> 16)));
            a = max(a, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, 0xB1, 0xF, 0xF, false));  // the block's other lane
            uint32_t code, out = 0;
            const uint32_t w4[4] = {w.x, w.y, w.z, w.w};
            if (FMT == 0) {
                code = (uint32_t)max((int)(a >> 7) - 2, 0);
                const float scale = __builtin_bit_cast(float, code << 23);
                out = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(out, __builtin_bit_cast(v2bf, w4[0]), scale, 0);
                out = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(out, __builtin_bit_cast(v2bf, w4[1]), scale, 1);
                out = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(out, __builtin_bit_cast(v2bf, w4[2]), scale, 2);
                out = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(out, __builtin_bit_cast(v2bf, w4[3]), scale, 3);
            } else {
                const float amax = __builtin_bit_cast(float, a << 16);
                const float q = fminf(__fdiv_rn(amax, d6), 448.0f);
                code = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(q, q, 0, false) & 0xffu;
                const float sval = __builtin_amdgcn_cvt_f32_fp8((int)code, 0);
                const float inv = sval == 0.0f ? 0.0f : __fdiv_rn(1.0f, __fmul_rn(ts, sval));
                float lo[4], hi[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    lo[k] = __fmul_rn(__builtin_bit_cast(float, w4[k] << 16), inv);
                    hi[k] = __fmul_rn(__builtin_bit_cast(float, w4[k] & 0xffff0000u), inv);
                }
                out = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(out, lo[0], hi[0], 1.0f, 0);
                out = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(out, lo[1], hi[1], 1.0f, 1);
                out = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(out, lo[2], hi[2], 1.0f, 2);
                out = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(out, lo[3], hi[3], 1.0f, 3);
            }
            // four blocks (eight lanes) -> one 32-bit word in the first of the eight lanes
            uint32_t word = code;
            word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)code, 0x102, 0xF, 0xF, true) << 8;   // lane + 2
            word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)code, 0x104, 0xF, 0xF, true) << 16;  // lane + 4
            word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)code, 0x106, 0xF, 0xF, true) << 24;  // lane + 6
            if ((lane & 7) == 0 && c < nchunk) sdst[c >> 3] = word;
            if (c < nchunk) __builtin_nontemporal_store(out, dst + c);
        }
        if (B) {
            uint16_t* brow = B + (int64_t)m * ldb;
            if (K_o > 0) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                const uint16_t* raw = reinterpret_cast<const uint16_t*>(strip);
                const int o1 = colstart[cur.seg + 1];
                for (int o = colstart[cur.seg] + lane; o < o1; o += 64) brow[o] = raw[(int)och[o] - cur.seg * SEG_CH];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            if (cur.seg == nseg - 1)
                for (int o = K_o + lane; o < (int)ldb; o += 64) brow[o] = 0;  // padding columns: +0
        }
    }
}

int launch_quant_fp4_g16(const uint16_t* X, int64_t M, int64_t K, int64_t ldx, const int32_t* oidx, int32_t K_o, int fmt,
                         float ts, uint8_t* Xq, uint8_t* Xs, uint16_t* B, int64_t ldb, hipStream_t st) {
    const int64_t nchunk = K / 8;
    const int nseg = (int)((nchunk + SEG_CHUNKS - 1) / SEG_CHUNKS);
    size_t smem = 4 * SEG_CHUNKS * 16;
    if (K_o > 0) smem += (size_t)(K / 2) * 4 + (size_t)(nseg + 1) * 4 + (size_t)K_o * 2;
    if (smem > 160 * 1024)
        return fail(OSC_ERR_UNSUPPORTED, "quantize: K=%lld with K_o=%d needs %zu bytes of LDS", (long long)K, (int)K_o, smem);
    auto kern = fmt == 0 ? quant_fp4_g16_kernel<0> : quant_fp4_g16_kernel<1>;
    if (smem > 48 * 1024) {
        static LdsReserved lds_reserved[2];
        if (int rc = reserve_lds(reinterpret_cast<const void*>(kern), smem, lds_reserved[fmt])) return rc;
    }
    const RowSplit split = row_split(M, nseg);
    const int64_t total_wg = split.wgs;
    if (total_wg > 0x7fffffff) return fail(OSC_ERR_UNSUPPORTED, "quantize: M=%lld too large", (long long)M);
    const int grid = (int)(total_wg < 2048 ? total_wg : 2048);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(QT16), smem, st, X, (int)M, (int)K, ldx, oidx, (int)K_o, ts, Xq, Xs, B, ldb,
                       nseg, split.quads, (int)total_wg);
    return check_launch("quant_fp4_g16_kernel");
}

// A dword of codes (8 channels of one scale block) as a matrix-core operand, the block scale folded in.
//   format 0: the conversion instruction multiplies by a power of two (it takes only the exponent of
//             its scale operand, which is all an E8M0 scale has): E2M1 x 2^e, exact in bf16.
//   format 1: an E4M3 scale has a mantissa, so the codes become fp16 (exact) and are multiplied by the
//             scale as packed fp16: an E2M1 value times an E4M3 value has at most six significant bits
//             and lies in [2^-10, 2688], exact in fp16; the main phase then runs on the fp16 matrix
//             core (the bf16 branch keeps the bf16 one; both accumulate into the same fp32 registers).
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
template <int FMT>
struct Scales16;
template <>
struct Scales16<0> {
    typedef v8bf operand;
    float s[4];
    // the four scale bytes of a lane; a zero byte is 2^-127
    __device__ __forceinline__ explicit Scales16(uint32_t w) {
#pragma unroll
        for (int b = 0; b < 4; ++b) s[b] = __builtin_bit_cast(float, max(((w >> (8 * b)) & 0xffu) << 23, 0x00400000u));
    }
    __device__ __forceinline__ operand expand(uint32_t w, int b) const {
        const v2bf p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, s[b], 0), p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, s[b], 1),
                   p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, s[b], 2), p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, s[b], 3);
        return (v8bf){p0.x, p0.y, p1.x, p1.y, p2.x, p2.y, p3.x, p3.y};
    }
};
template <>
struct Scales16<1> {
    typedef v8h operand;
    v2h s[2];  // exact: every E4M3 value is an fp16 value
    __device__ __forceinline__ explicit Scales16(uint32_t w) {
        s[0] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w, 1.0f, false);
        s[1] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w, 1.0f, true);
    }
    __device__ __forceinline__ operand expand(uint32_t w, int b) const {
        const _Float16 sh = s[b >> 1][b & 1];
        const v2h ss = {sh, sh};
        const v2h p0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 0) * ss, p1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 1) * ss,
                  p2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 2) * ss, p3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 3) * ss;
        return (v8h){p0.x, p0.y, p1.x, p1.y, p2.x, p2.y, p3.x, p3.y};
    }
};

struct G16Args {
    const uint8_t* Xq;
    const uint8_t* Xs;
    const uint8_t* B;
    int64_t bpitch;
    const uint8_t* Wq;
    const uint8_t* Ws;
    const uint8_t* WL;
    int64_t wlpitch;
    int M, N, K, K_o;
    float ts;  // product of the two tensor scales (1 for format 0)
    void* Y;
    int y_bf16;
    int64_t ldy;
};

// ------------------------------------------------------------------------------------------
// Streaming GEMM, up to 16 rows (32 where that leaves CUs idle: rule below).  A workgroup owns 16 rows of X and 16 NT output
// channels; its NW wavefronts take the 128-byte lines of the reduction axis (256 four-bit channels = 16 scale blocks
// per row and line, then the bf16 lines of the branch) in turn and never synchronise until the end.  A wavefront loads
// the next line (eight lanes per row) into one of two register sets while it takes the current one through a strip of
// LDS of its own into matrix-core layout, expands it in registers and multiplies.
// Layout of v_mfma_f32_16x16x32_{f16,bf16} (lane = 16 q + r): row r, eight elements of block q; which elements is free
// as long as both operands agree.  A lane takes pieces 2q and 2q + 1 of its row's line, 64 codes in eight dwords: dword
// m feeds instruction m, and its scale block is 4q + m / 2, byte m / 2 of the word that the lane loads for its row.
// What bounds it: the vector work of the expansion, a conversion per two values and in NVFP4 a product per two as well,
// 32 (64) instructions per 16 rows or channels and line.  32 rows of X per 32 channels, 16 of them copies at up to 16
// tokens, made that twice what it has to be, on 384 workgroups for 256 CUs; 16 rows and 48 channels are half of it and
// one workgroup per CU at N = 12288.  16 tokens, weights from HBM, us, wide kernel below -> this one:
//   12288 x 4096  NVFP4 13.1 -> 8.8, E8M0 11.4 -> 8.5      4096 x 12288  15.2 -> 9.9, 13.9 -> 9.7      4096 x 4096  6.9 -> 4.9, 6.1 -> 4.8
// and 32 tokens: 4096 x 4096  8.5 -> 7.0, 7.9 -> 6.8; but 12288 x 4096 from the last-level cache 11.8 -> 12.5 and 9.9 -> 11.8,
// and 33 to 128 tokens in tiles of 32 or 64 rows 1.0 to 1.3 times slower: these stay on the wide kernel.
// ------------------------------------------------------------------------------------------
template <int FMT, int NT, int NW>
__global__ void __launch_bounds__(64 * NW) gemm_g16_kernel(G16Args a) {
    constexpr int MT = 1;  // 16-row tiles of X
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int q = lane >> 4, r = lane & 15;
    // two blocks of rows: workgroups b and b + 8, which run on the same die, share the weights of a strip
    const bool two = a.M > 16 * MT;
    const int strip_n = two ? (int)(blockIdx.x >> 4) * 8 + (int)(blockIdx.x & 7) : (int)blockIdx.x;
    const int n0 = strip_n * (16 * NT), m0 = two ? (int)(blockIdx.x >> 3 & 1) * (16 * MT) : 0;
    if (n0 >= a.N) return;  // (the grid is whole groups of eight strips)
    const uint32_t rowbytes = (uint32_t)a.K >> 1, srow = (uint32_t)a.K >> 4;
    const int nL = (int)(rowbytes >> 7);
    const int nLT = nL + ((a.K_o * 2 + 127) >> 7);
    // instruction h of a 16-row tile loads rows 8h .. 8h+7, eight lanes per line
    const int lrow = lane >> 3;
    const uint32_t p0 = (uint32_t)(lane & 7) * 16u;
    uint32_t ow[NT][2], owb[NT][2], osw[NT], ox[MT][2], oxb[MT][2], osx[MT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t n = (uint32_t)min(n0 + 16 * j + 8 * h + lrow, a.N - 1);
            ow[j][h] = n * rowbytes + p0;
            owb[j][h] = n * (uint32_t)a.wlpitch + p0;
        }
        osw[j] = (uint32_t)min(n0 + 16 * j + r, a.N - 1) * srow + 4u * q;
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t g = (uint32_t)min(m0 + 16 * i + 8 * h + lrow, a.M - 1);
            ox[i][h] = g * rowbytes + p0;
            oxb[i][h] = g * (uint32_t)a.bpitch + p0;
        }
        osx[i] = (uint32_t)min(m0 + 16 * i + r, a.M - 1) * srow + 4u * q;
    }
    // one line of the workgroup's rows per wavefront (weights, then X); later the partial sums
    constexpr int STRIP = 16 * (NT + MT) * 128;
    __shared__ __attribute__((aligned(16))) uint8_t lds_s[NW * (STRIP > MT * NT * 1024 ? STRIP : MT * NT * 1024)];
    uint8_t* const strip = lds_s + wave * STRIP;
    float* const red = reinterpret_cast<float*>(lds_s);
    uint32_t wpos[2], rpos[2];  // places in a 16-row tile: written (instruction h), read (piece 2q + h)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        wpos[h] = (uint32_t)st128_off(8 * h + lrow, lane & 7);
        rpos[h] = (uint32_t)st128_off(r, 2 * q + h);
    }
    struct Line {
        u32x4 w[NT][2], x[MT][2];
        uint32_t sw[NT], sx[MT];
    };
    v4f acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
    bool scaled = FMT == 0;  // the tensor scales go on once, before the first branch line

    // line L into S (a branch line fetches the last scale words again, unused)
    auto load = [&](int L, Line& S) __attribute__((always_inline)) {
        const bool main = L < nL;
        const uint32_t lo = (uint32_t)(main ? L : L - nL) * 128u, ls = (uint32_t)min(L, nL - 1) * 16u;
        const uint8_t *const wb = (main ? a.Wq : a.WL) + lo, *const xb = (main ? a.Xq : a.B) + lo;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
                S.w[j][h] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wb + (main ? ow[j][h] : owb[j][h])));
            S.sw[j] = *reinterpret_cast<const uint32_t*>(a.Ws + (osw[j] + ls));
        }
#pragma unroll
        for (int i = 0; i < MT; ++i) {
#pragma unroll
            for (int h = 0; h < 2; ++h) S.x[i][h] = *reinterpret_cast<const u32x4*>(xb + (main ? ox[i][h] : oxb[i][h]));
            S.sx[i] = *reinterpret_cast<const uint32_t*>(a.Xs + (osx[i] + ls));
        }
    };
    auto compute = [&](int L, const Line& S) __attribute__((always_inline)) {
        // through the wavefront's strip into matrix-core layout (LDS runs a wavefront's operations in order)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int j = 0; j < NT; ++j) *reinterpret_cast<u32x4*>(strip + j * 2048 + wpos[h]) = S.w[j][h];
#pragma unroll
            for (int i = 0; i < MT; ++i) *reinterpret_cast<u32x4*>(strip + (NT + i) * 2048 + wpos[h]) = S.x[i][h];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (L < nL) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u32x4 cw[NT], cx[MT];
#pragma unroll
                for (int j = 0; j < NT; ++j) cw[j] = *reinterpret_cast<const u32x4*>(strip + j * 2048 + rpos[h]);
#pragma unroll
                for (int i = 0; i < MT; ++i) cx[i] = *reinterpret_cast<const u32x4*>(strip + (NT + i) * 2048 + rpos[h]);
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    typename Scales16<FMT>::operand fx[MT];
#pragma unroll
                    for (int i = 0; i < MT; ++i) fx[i] = Scales16<FMT>(S.sx[i]).expand(cx[i][m], 2 * h + m / 2);
#pragma unroll
                    for (int j = 0; j < NT; ++j) {
                        const typename Scales16<FMT>::operand fw = Scales16<FMT>(S.sw[j]).expand(cw[j][m], 2 * h + m / 2);
#pragma unroll
                        for (int i = 0; i < MT; ++i) {
                            if constexpr (FMT == 0) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx[i], fw, acc[i][j], 0, 0, 0);
                            else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fx[i], fw, acc[i][j], 0, 0, 0);
                        }
                    }
                }
            }
        } else {
            if (!scaled) {
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) acc[i][j] *= a.ts;
                scaled = true;
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const u32x4 fw = *reinterpret_cast<const u32x4*>(strip + j * 2048 + rpos[h]);
#pragma unroll
                    for (int i = 0; i < MT; ++i) {
                        const u32x4 fx = *reinterpret_cast<const u32x4*>(strip + (NT + i) * 2048 + rpos[h]);
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, fx), __builtin_bit_cast(v8bf, fw), acc[i][j], 0, 0, 0);
                    }
                }
        }
    };
    if (wave < nLT) {
        // two sets written out in turn: a copy from one to the other would wait for the loads in flight
        Line sa, sb;
        int L = wave;
        load(L, sa);
#pragma unroll 1
        for (; L + 2 * NW < nLT; L += 2 * NW) {
            load(L + NW, sb);
            compute(L, sa);
            load(L + 2 * NW, sa);
            compute(L + NW, sb);
        }
        if (L + NW < nLT) {
            load(L + NW, sb);
            compute(L, sa);
            compute(L + NW, sb);
        } else {
            compute(L, sa);
        }
    }
    if (!scaled) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] *= a.ts;
    }
    // ---- sum the NW partial results in a fixed order, store ----
    __syncthreads();  // every wavefront is done with its strip
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k) red[((wave * MT * NT + i * NT + j) * 4 + k) * 64 + lane] = acc[i][j][k];
    __syncthreads();
    for (int u = t; u < MT * NT * 256; u += 64 * NW) {
        const int l = u & 63, k = (u >> 6) & 3, ij = u >> 8;
        const int row = m0 + 16 * (ij / NT) + 4 * (l >> 4) + k, col = n0 + 16 * (ij % NT) + (l & 15);
        if (row >= a.M || col >= a.N) continue;
        float v = red[u];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += red[w * MT * NT * 256 + u];
        if (a.y_bf16) reinterpret_cast<uint16_t*>(a.Y)[(int64_t)row * a.ldy + col] = f32_to_bf16_rne(v);
        else reinterpret_cast<float*>(a.Y)[(int64_t)row * a.ldy + col] = v;
    }
}

template <int FMT, int NT, int NW>
static int launch_g16(const G16Args& a, hipStream_t st) {
    const unsigned strips = (unsigned)((a.N + 16 * NT - 1) / (16 * NT)), grid = a.M > 16 ? (strips + 7) / 8 * 16 : strips;  // M <= 32
    hipLaunchKernelGGL((gemm_g16_kernel<FMT, NT, NW>), dim3(grid), dim3(64 * NW), 0, st, a);
    note_gemm(GEMM_G16_ROWS16, NT);
    return check_launch("gemm_g16_kernel");
}

// Channels / 16 of a workgroup: the smallest ceil(workgroups / CUs) x (1 + NT), the smaller one among equals (a launch
// lasts as long as the CU with the most workgroups, a workgroup as long as its expansion takes).  0: the wide kernel, which
// expands as many rows for 32 of X as two row blocks here and the weights once: more than 16 rows, where a CU would get more
// than one workgroup or one of more than 32 channels (32 rows, wide -> here, us, weights cached and from HBM: E8M0 2048 x 4096
// 5.9 -> 4.0 and 6.3 -> 5.0, 4096 x 4096 6.1 -> 5.9 and 7.9 -> 6.8; 6144 x 8192 9.3 and 11.7, 13.4 and 14.1; 8192 x 4096 6.9 and 8.8,
// 8.7 and 10.5; NVFP4 8.1 and 9.5, 9.6 and 11.0; very long rows of E8M0 gain from HBM only: 4096 x 12288 12.0 and 12.5, 17.4 -> 15.1).
static int g16_rows16_tile(int64_t M, int64_t N, int ncu) {
    int best = 1;
    int64_t best_cost = INT64_MAX, best_per = 0;
    for (int nt = 1; nt <= 4; ++nt) {
        const int64_t wgs = (N + 16 * nt - 1) / (16 * nt) * ((M + 15) / 16), per = (wgs + ncu - 1) / ncu, cost = per * (1 + nt);
        if (cost < best_cost) {
            best_cost = cost;
            best_per = per;
            best = nt;
        }
    }
    return M <= 16 || (M <= 32 && best_per == 1 && best <= 2) ? best : 0;
}

template <int FMT>
static int launch_g16_rows16(const G16Args& a, int nt, hipStream_t st) {
    switch (nt) {
        case 1: return launch_g16<FMT, 1, 8>(a, st);
        case 2: return launch_g16<FMT, 2, 8>(a, st);
        case 3: return launch_g16<FMT, 3, 8>(a, st);
        default: return launch_g16<FMT, 4, 8>(a, st);
    }
}

// ------------------------------------------------------------------------------------------
// Wide form, more rows: one workgroup per 32 output channels and 32 rows of X; its wavefronts take the
// 128-byte lines in turn.  A wavefront moves a line global -> LDS by DMA into a strip of its own (codes in whole
// 128-byte lines, the 16 scale bytes of every row beside them), expands it in registers and multiplies.
// K order inside a line: the bf16 matrix core pairs lane half q of one operand with lane half q of
// the other, nothing else, so a lane takes the 16 contiguous bytes [32j + 16q, +16) of its row for
// the four MFMAs 4j .. 4j+3 (dword t feeds MFMA 4j+t); those 32 channels are scale blocks 4j+2q and
// 4j+2q+1, applied during the expansion.
// ------------------------------------------------------------------------------------------
template <int FMT, int NW>
__global__ void __launch_bounds__(64 * NW) gemm_g16_wide_kernel(G16Args a) {
    constexpr int IMG = 64 * 128 + 64 * 16;  // codes of 32 weight rows and 32 X rows, then their scale bytes
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int q = lane >> 5, r = lane & 31;
    const int n0 = blockIdx.x * 32, mb = blockIdx.y * 32;
    const int rowbytes = a.K >> 1, srow = a.K >> 4;
    const int nL = rowbytes >> 7;
    const int nLB = (a.K_o * 2 + 127) >> 7;
    const int nLT = nL + nLB;
    uint8_t* const strip = lds + wave * (2 * IMG);

    // DMA instruction i (0..7) moves rows 8i .. 8i+7 of the image (rows 0-31 weights, 32-63 X): lane ->
    // row 8i + lane/8, piece position lane%8 holding piece (lane%8) ^ swz8(row); instruction 8 moves
    // the 16 scale bytes of row `lane`
    uint32_t o_fp4[8], o_br[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = 8 * i + (lane >> 3);
        const uint32_t piece = (uint32_t)((lane & 7) ^ swz8(row)) * 16u;
        const uint32_t g = row < 32 ? (uint32_t)min(n0 + row, a.N - 1) : (uint32_t)min(mb + row - 32, a.M - 1);
        o_fp4[i] = g * (uint32_t)rowbytes + piece;
        o_br[i] = g * (uint32_t)(row < 32 ? a.wlpitch : a.bpitch) + piece;
    }
    const uint32_t o_sc = (lane < 32 ? (uint32_t)min(n0 + lane, a.N - 1) : (uint32_t)min(mb + lane - 32, a.M - 1)) * (uint32_t)srow;
    const uint8_t* const sc_base = lane < 32 ? a.Ws : a.Xs;

    v16f acc;
#pragma unroll
    for (int k = 0; k < 16; ++k) acc[k] = 0.0f;

#define G16_FETCH(L_, IMG_)                                                                              \
    {                                                                                                    \
        uint8_t* dst__ = strip + (IMG_)*IMG;                                                             \
        if ((L_) < nL) {                                                                                 \
            _Pragma("unroll") for (int i = 0; i < 8; ++i)                                                \
                load_to_lds16((i < 4 ? a.Wq : a.Xq) + ((size_t)(L_)*128 + o_fp4[i]), dst__ + i * 1024);  \
            load_to_lds16(sc_base + ((size_t)(L_)*16 + o_sc), dst__ + 8192);                             \
        } else if ((L_) < nLT) {                                                                         \
            _Pragma("unroll") for (int i = 0; i < 8; ++i)                                                \
                load_to_lds16((i < 4 ? a.WL : a.B) + ((size_t)((L_)-nL) * 128 + o_br[i]), dst__ + i * 1024); \
            load_to_lds16(sc_base + o_sc, dst__ + 8192); /* keeps the count of requests per line fixed */ \
        }                                                                                                \
    }
    bool scaled = FMT == 0;  // the tensor scales go on once, before the first branch line
    int L = wave, img = 0;
    G16_FETCH(L, 0)
#pragma unroll 1
    for (; L < nLT; L += NW) {
        G16_FETCH(L + NW, img ^ 1)
        if (L + NW < nLT) wait_vmcnt<9>(); else wait_vmcnt<0>();
        const uint8_t* src = strip + img * IMG;
        if (L < nL) {
            const u32x4 sw = *reinterpret_cast<const u32x4*>(src + 8192 + r * 16);
            const u32x4 sx = *reinterpret_cast<const u32x4*>(src + 8192 + (32 + r) * 16);
            const uint32_t swv[4] = {sw.x, sw.y, sw.z, sw.w}, sxv[4] = {sx.x, sx.y, sx.z, sx.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const u32x4 cw = *reinterpret_cast<const u32x4*>(src + st128_off(r, 2 * j + q));
                const u32x4 cx = *reinterpret_cast<const u32x4*>(src + st128_off(32 + r, 2 * j + q));
                const Scales16<FMT> bw(swv[j] >> (16 * q)), bx(sxv[j] >> (16 * q));
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const typename Scales16<FMT>::operand fx = bx.expand(cx[k], k >> 1), fw = bw.expand(cw[k], k >> 1);
                    if constexpr (FMT == 0) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx, fw, acc, 0, 0, 0);
                    else acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(fx, fw, acc, 0, 0, 0);
                }
            }
        } else {
            if (!scaled) {
#pragma unroll
                for (int k = 0; k < 16; ++k) acc[k] *= a.ts;
                scaled = true;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const u32x4 fw = *reinterpret_cast<const u32x4*>(src + st128_off(r, 4 * q + i));
                const u32x4 fx = *reinterpret_cast<const u32x4*>(src + st128_off(32 + r, 4 * q + i));
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, fx), __builtin_bit_cast(v8bf, fw), acc, 0, 0, 0);
            }
        }
        img ^= 1;
    }
#undef G16_FETCH
    if (!scaled) {
#pragma unroll
        for (int k = 0; k < 16; ++k) acc[k] *= a.ts;
    }
    // ---- sum the NW partial results in a fixed order, store ----
    __syncthreads();
    float* const red = reinterpret_cast<float*>(lds);  // [NW][16][64]
#pragma unroll
    for (int k = 0; k < 16; ++k) red[(wave * 16 + k) * 64 + lane] = acc[k];
    __syncthreads();
#pragma unroll
    for (int k0 = 0; k0 < 16; k0 += NW) {
        const int k = k0 + wave;
        if (k >= 16) break;
        float v = red[k * 64 + lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += red[(w * 16 + k) * 64 + lane];
        const int row = mb + 8 * (k >> 2) + 4 * q + (k & 3), col = n0 + r;
        if (row < a.M && col < a.N) {
            if (a.y_bf16)
                reinterpret_cast<uint16_t*>(a.Y)[(int64_t)row * a.ldy + col] = f32_to_bf16_rne(v);
            else
                reinterpret_cast<float*>(a.Y)[(int64_t)row * a.ldy + col] = v;
        }
    }
}

int launch_dual_gemm_g16(const uint8_t* Xq, const uint8_t* Xs, float xts, const uint16_t* B, int64_t ldb, const uint8_t* Wq,
                         const uint8_t* Ws, const uint16_t* WLt, int64_t ldwl, float wts, int64_t M, int64_t N, int64_t K,
                         int32_t K_o, int fmt, void* Y, int y_dtype, int64_t ldy, hipStream_t st) {
    G16Args a;
    a.Xq = Xq;
    a.Xs = Xs;
    a.B = reinterpret_cast<const uint8_t*>(B);
    a.bpitch = ldb * 2;
    a.Wq = Wq;
    a.Ws = Ws;
    a.WL = reinterpret_cast<const uint8_t*>(WLt);
    a.wlpitch = ldwl * 2;
    a.M = (int)M;
    a.N = (int)N;
    a.K = (int)K;
    a.K_o = K_o;
    a.ts = fmt == 0 ? 1.0f : xts * wts;
    a.Y = Y;
    a.y_bf16 = y_dtype == OSC_DT_BF16;
    a.ldy = ldy;
    const int64_t lim = (int64_t)1 << 32;
    if (M * (K / 2) >= lim || N * (K / 2) >= lim || M * a.bpitch >= lim || N * a.wlpitch >= lim)
        return fail(OSC_ERR_UNSUPPORTED, "gemm: an operand of 4 GiB or more");
    const int ncu = cu_count();
    if (ncu <= 0) return fail(OSC_ERR_HIP, "gemm: cannot read the number of compute units");
    if (const int nt = g16_rows16_tile(M, N, ncu)) return fmt == 0 ? launch_g16_rows16<0>(a, nt, st) : launch_g16_rows16<1>(a, nt, st);
    const dim3 grid((unsigned)((N + 31) / 32), (unsigned)((M + 31) / 32));
    constexpr int IMG = 64 * 128 + 64 * 16;
    // eight wavefronts when the grid leaves CUs idle, four otherwise (two workgroups per CU)
    const bool wide = (int64_t)grid.x * grid.y <= ncu;
    const size_t smem = (size_t)(wide ? 8 : 4) * 2 * IMG;
#define G16_LAUNCH(F_, NW_)                                                                               \
    {                                                                                                     \
        auto kern = gemm_g16_wide_kernel<F_, NW_>;                                                             \
        static LdsReserved lds_reserved;                                                                  \
        if (int rc = reserve_lds(reinterpret_cast<const void*>(kern), smem, lds_reserved)) return rc; \
        hipLaunchKernelGGL(kern, grid, dim3(64 * NW_), smem, st, a);                                      \
    }
    if (fmt == 0) {
        if (wide) G16_LAUNCH(0, 8) else G16_LAUNCH(0, 4)
    } else {
        if (wide) G16_LAUNCH(1, 8) else G16_LAUNCH(1, 4)
    }
#undef G16_LAUNCH
    note_gemm(GEMM_G16_WIDE, wide ? 8 : 4);
    return check_launch("gemm_g16_wide_kernel");
}

}  // namespace osc
