// Producer fusion: RMSNorm (the operation in front of the attention and FFN projections, positions
// 1 and 3 of Section 2.1) and the OSC-enhanced quantiser (Section 3.2, Alg. 2) in one pass over
// the row, so that the normalised activations never travel through HBM.
#include "osc_internal.h"
#include "wave_util.h"

namespace osc {

typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int FT = 256;  // four wavefronts, one row each at a time
constexpr int64_t MAX_GRID = 1 << 22;  // workgroups of a one-trip launch (the kernels walk on from there)

// bf16(a * r) for the two halves of a packed word, one single-precision multiplication each
__device__ __forceinline__ uint32_t scale_pair(uint32_t w, float r) {
    const uint32_t lo = w << 16, hi = w & 0xffff0000u;
    const v2f p = {__builtin_bit_cast(float, lo) * r, __builtin_bit_cast(float, hi) * r};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(p, v2bf));
}
// bf16(t * g), element by element (the product of two bf16 values is exact in single precision)
__device__ __forceinline__ uint32_t mul_pair(uint32_t t, uint32_t g) {
    const uint32_t tl = t << 16, th = t & 0xffff0000u, gl = g << 16, gh = g & 0xffff0000u;
    const v2f p = {__builtin_bit_cast(float, tl) * __builtin_bit_cast(float, gl),
                   __builtin_bit_cast(float, th) * __builtin_bit_cast(float, gh)};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(p, v2bf));
}
// The fixed-point sum of squares, floor(x^2 / u) summed over the row with u = 2^(2e - 296) (e the row's
// largest biased exponent), comes out of the double-precision FMA itself: the accumulator starts at
// 2^52 * u, so its last place is u for as long as fewer than 2^52 units are added (a lane adds at most
// 192 terms below 2^44 units each); x^2 is exact in double; and with the double-precision rounding
// mode set to "toward zero" the one rounding of fma(x, x, acc) drops exactly the fraction of a unit,
// because acc is a whole number of units.  The mode is a wavefront's own state.  It is switched
// by the two statements below, which take the accumulators as operands so that every operation that
// produces or consumes them stays between the switches, and each FMA is written out so that it cannot
// be merged or moved across them.
constexpr int F64_ROUND_TOWARD_ZERO = 3, F64_ROUND_NEAREST = 0;
template <int ROUND>
__device__ __forceinline__ void f64_round_mode(double& a, double& b) {
    asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), %2\n\ts_nop 1" : "+v"(a), "+v"(b) : "n"(ROUND));
}
__device__ __forceinline__ void sq_add(double& acc, uint32_t fbits) {
    const double x = (double)__builtin_bit_cast(float, fbits);
    asm volatile("v_fma_f64 %0, %1, %1, %0" : "+v"(acc) : "v"(x));
}

// Scale code and E2M1 codes of chunk c (eight normalised channels, y: pairs of bf16) of a row; four neighbouring lanes hold
// a 32-channel group, sixteen the four scale bytes of one word.
__device__ __forceinline__ void quant_chunk(const uint32_t (&y)[4], int lane, int c, bool valid, uint32_t* __restrict__ dst,
                                            uint8_t* __restrict__ sdst) {
    const uint32_t a2 = max_pair(max_pair(y[0] & 0x7fff7fffu, y[1] & 0x7fff7fffu),
                                 max_pair(y[2] & 0x7fff7fffu, y[3] & 0x7fff7fffu));
    uint32_t a = max(a2 & 0xffffu, a2 >> 16);
    a = max(a, (uint32_t)__builtin_amdgcn_mov_dpp((int)a, 0xB1, 0xF, 0xF, true));
    a = max(a, (uint32_t)__builtin_amdgcn_mov_dpp((int)a, 0x4E, 0xF, 0xF, true));
    const uint32_t code = (uint32_t)max((int)(a >> 7) - 2, 0);
    uint32_t word = code;
    word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)code, 0x104, 0xF, 0xF, true) << 8;
    word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)code, 0x108, 0xF, 0xF, true) << 16;
    word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)code, 0x10C, 0xF, 0xF, true) << 24;
    if ((lane & 15) == 0 && valid) *reinterpret_cast<uint32_t*>(sdst + (c >> 4) * 128) = word;
    const float scale = __builtin_bit_cast(float, code << 23);
    uint32_t out = 0;
    out = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(out, __builtin_bit_cast(v2bf, y[0]), scale, 0);
    out = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(out, __builtin_bit_cast(v2bf, y[1]), scale, 1);
    out = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(out, __builtin_bit_cast(v2bf, y[2]), scale, 2);
    out = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(out, __builtin_bit_cast(v2bf, y[3]), scale, 3);
    if (valid) __builtin_nontemporal_store(out, dst + c);
}

// A wavefront owns a whole row: lane l holds the 16-byte chunks l, l + 64, ... (NCI of them), so
// the two row-wide reductions (largest exponent, sum of squares) are register work plus DPP.
// The sum of squares is an integer in fixed point relative to the row's largest exponent: exact
// up to a truncation 2^-42 below the largest term and independent of any order, so the
// normalised row, and every code derived from it, is reproducible bit for bit.
// LDS: per-wave strip of the normalised row (for the gather) | keep masks | gamma | channel list.
template <int NCI, bool FULL>
__global__ void __launch_bounds__(FT) rmsnorm_quant_mxfp4_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ gamma, double eps, int M, int K, int64_t ldx,
    const int32_t* __restrict__ oidx, int K_o, uint8_t* __restrict__ Xq, uint8_t* __restrict__ Xs,
    uint16_t* __restrict__ B, int64_t ldb, uint16_t* __restrict__ Xn) {
    extern __shared__ uint32_t smem[];
    const int Kg = K >> 5, Kg4 = (Kg + 3) >> 2;
    const int nchunk = K >> 3;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);  // uniform: row and segment arithmetic stays on the scalar unit
    u32x4* strip = reinterpret_cast<u32x4*>(smem) + wave * (NCI * 64);
    uint32_t* keep = smem + 4 * NCI * 64 * 4;
    u32x4* gam = reinterpret_cast<u32x4*>(keep + (K >> 1));
    uint16_t* och = reinterpret_cast<uint16_t*>(gam + nchunk);

    for (int i = t; i < (K >> 1); i += FT) keep[i] = 0xffffffffu;
    for (int i = t; i < nchunk; i += FT) gam[i] = reinterpret_cast<const u32x4*>(gamma)[i];
    __syncthreads();
    for (int o = t; o < K_o; o += FT) {
        const int c = oidx[o];
        if (c >= 0 && c < K) atomicAnd(&keep[c >> 1], (c & 1) ? 0x0000ffffu : 0xffff0000u);
        och[o] = (uint16_t)c;
    }
    __syncthreads();

    for (int m = blockIdx.x * 4 + wave; m < M; m += gridDim.x * 4) {
        const u32x4* src = reinterpret_cast<const u32x4*>(X + (int64_t)m * ldx);
        u32x4 v[NCI];
#pragma unroll
        for (int i = 0; i < NCI; ++i) {
            const int c = lane + 64 * i;
            v[i] = (u32x4){0u, 0u, 0u, 0u};
            if ((FULL || c < nchunk)) v[i] = __builtin_nontemporal_load(src + c);
        }
        // largest exponent of the row
        uint32_t am2 = 0;
#pragma unroll
        for (int i = 0; i < NCI; ++i) {
            const u32x4 ab = v[i] & 0x7fff7fffu;
            am2 = max_pair(am2, max_pair(max_pair(ab.x, ab.y), max_pair(ab.z, ab.w)));
        }
        const int e = max(1, (int)(wave_max_u32(max(am2 & 0xffffu, am2 >> 16)) >> 7));
        // sum of squares in units of 2^(2e - 296): exact per lane (see sq_add), the 64 lane sums are
        // added as integers
        const double base = __builtin_bit_cast(double, (uint64_t)(1023 + 52 + 2 * e - 296) << 52);
        double s0 = base, s1 = base;
        f64_round_mode<F64_ROUND_TOWARD_ZERO>(s0, s1);
#pragma unroll
        for (int i = 0; i < NCI; ++i) {
            const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                sq_add(s0, w[k] << 16);
                sq_add(s1, w[k] & 0xffff0000u);
            }
        }
        f64_round_mode<F64_ROUND_NEAREST>(s0, s1);
        const double units = ((s0 - base) + (s1 - base)) * __builtin_bit_cast(double, (uint64_t)(1023 + 296 - 2 * e) << 52);
        const uint64_t S = wave_sum_u64((uint64_t)units);
        const double mean = ldexp((double)S, 2 * e - 296) / (double)K;
        const float r = (float)(1.0 / sqrt(mean + eps));

        uint32_t* dst = reinterpret_cast<uint32_t*>(Xq + (int64_t)m * (K >> 1));
        uint8_t* sdst = Xs + (int64_t)(m >> 5) * Kg4 * 128 + (m & 31) * 4;
#pragma unroll
        for (int i = 0; i < NCI; ++i) {
            const int c = lane + 64 * i;
            const u32x4 g = (FULL || c < nchunk) ? gam[c] : (u32x4){0u, 0u, 0u, 0u};
            uint32_t y[4] = {mul_pair(scale_pair(v[i].x, r), g.x), mul_pair(scale_pair(v[i].y, r), g.y),
                             mul_pair(scale_pair(v[i].z, r), g.z), mul_pair(scale_pair(v[i].w, r), g.w)};
            const u32x4 yv = {y[0], y[1], y[2], y[3]};
            if (Xn && (FULL || c < nchunk)) __builtin_nontemporal_store(yv, reinterpret_cast<u32x4*>(Xn + (int64_t)m * K) + c);
            if (K_o > 0) {
                strip[c] = yv;  // back-up (step 2 of Section 3.2)
                if ((FULL || c < nchunk)) {
                    const u32x4 kp = *reinterpret_cast<const u32x4*>(keep + 4 * c);
                    y[0] &= kp.x, y[1] &= kp.y, y[2] &= kp.z, y[3] &= kp.w;  // zero (step 3)
                }
            }
            quant_chunk(y, lane, c, FULL || c < nchunk, dst, sdst);
        }
        if (B) {
            uint16_t* brow = B + (int64_t)m * ldb;
            if (K_o > 0) {
                // the strip was written by this wavefront; LDS runs a wavefront's operations in order
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                const uint16_t* raw = reinterpret_cast<const uint16_t*>(strip);
                for (int o = lane; o < K_o; o += 64) brow[o] = raw[och[o]];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            for (int o = K_o + lane; o < (int)ldb; o += 64) brow[o] = 0;  // padding columns: +0
        }
    }
}

// The same for few rows: a workgroup of four wavefronts owns a row, thread t the chunks t, t + 256, ... (NCH of them).  One
// wavefront per row leaves most SIMDs empty below a few thousand rows and is then a chain of 1100 vector instructions;
// here it is 300, with three more barriers (largest exponent, sum, the row for the gather).  The sum of squares is an
// integer that does not depend on how it is split, so the results are the same bits.  us, a
// wavefront per row -> a workgroup per row (calls in a row; 4.3 is the host's rate):
//   K = 4096   16 rows 5.7 -> 4.5   100: 6.0 -> 4.4   500: 6.7 -> 5.1   1000: 7.1 -> 6.5   2000: 9.0 -> 9.6   8192: 22 -> 27
//   K = 12288  16 rows 13.3 -> 7.2  100: 14.1 -> 8.5  500: 14.9 -> 10.5 1000: 16.4 -> 19.7
template <int NCH>
__global__ void __launch_bounds__(FT) rmsnorm_quant_mxfp4_row_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ gamma, double eps, int K, int64_t ldx,
    const int32_t* __restrict__ oidx, int K_o, uint8_t* __restrict__ Xq, uint8_t* __restrict__ Xs,
    uint16_t* __restrict__ B, int64_t ldb, uint16_t* __restrict__ Xn) {
    extern __shared__ uint32_t smem[];
    __shared__ uint32_t top[4];
    __shared__ uint64_t sums[4];
    const int Kg4 = ((K >> 5) + 3) >> 2, nchunk = K >> 3, m = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    u32x4* const strip = reinterpret_cast<u32x4*>(smem);  // the normalised row
    uint32_t* const keep = smem + NCH * 256 * 4;
    const u32x4* const src = reinterpret_cast<const u32x4*>(X + (int64_t)m * ldx);
    u32x4 v[NCH], g[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = t + 256 * i;
        v[i] = g[i] = (u32x4){0u, 0u, 0u, 0u};
        if (c < nchunk) {
            v[i] = __builtin_nontemporal_load(src + c);
            g[i] = reinterpret_cast<const u32x4*>(gamma)[c];
        }
    }
    const int och0 = t < K_o ? oidx[t] : -1;
    if (K_o > 0) {
#pragma unroll
        for (int i = 0; i < NCH; ++i) *reinterpret_cast<u32x4*>(keep + 4 * (t + 256 * i)) = (u32x4){~0u, ~0u, ~0u, ~0u};
    }
    uint32_t am2 = 0;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const u32x4 ab = v[i] & 0x7fff7fffu;
        am2 = max_pair(am2, max_pair(max_pair(ab.x, ab.y), max_pair(ab.z, ab.w)));
    }
    const uint32_t wtop = wave_max_u32(max(am2 & 0xffffu, am2 >> 16));
    if (lane == 0) top[wave] = wtop;
    __syncthreads();
    for (int o = t; o < K_o; o += FT) {
        const int och = o == t ? och0 : oidx[o];
        if (och >= 0 && och < K) atomicAnd(&keep[och >> 1], (och & 1) ? 0x0000ffffu : 0xffff0000u);
    }
    const int e = max(1, (int)(max(max(top[0], top[1]), max(top[2], top[3])) >> 7));
    const double base = __builtin_bit_cast(double, (uint64_t)(1023 + 52 + 2 * e - 296) << 52);
    double s0 = base, s1 = base;
    f64_round_mode<F64_ROUND_TOWARD_ZERO>(s0, s1);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            sq_add(s0, w[k] << 16);
            sq_add(s1, w[k] & 0xffff0000u);
        }
    }
    f64_round_mode<F64_ROUND_NEAREST>(s0, s1);
    const double units = ((s0 - base) + (s1 - base)) * __builtin_bit_cast(double, (uint64_t)(1023 + 296 - 2 * e) << 52);
    const uint64_t wsum = wave_sum_u64((uint64_t)units);
    if (lane == 0) sums[wave] = wsum;
    __syncthreads();  // sums and keep masks
    const uint64_t S = (sums[0] + sums[1]) + (sums[2] + sums[3]);
    const double mean = ldexp((double)S, 2 * e - 296) / (double)K;
    const float r = (float)(1.0 / sqrt(mean + eps));

    uint32_t* const dst = reinterpret_cast<uint32_t*>(Xq + (int64_t)m * (K >> 1));
    uint8_t* const sdst = Xs + (int64_t)(m >> 5) * Kg4 * 128 + (m & 31) * 4;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = t + 256 * i;
        uint32_t y[4] = {mul_pair(scale_pair(v[i].x, r), g[i].x), mul_pair(scale_pair(v[i].y, r), g[i].y),
                         mul_pair(scale_pair(v[i].z, r), g[i].z), mul_pair(scale_pair(v[i].w, r), g[i].w)};
        const u32x4 yv = {y[0], y[1], y[2], y[3]};
        if (Xn && c < nchunk) __builtin_nontemporal_store(yv, reinterpret_cast<u32x4*>(Xn + (int64_t)m * K) + c);
        if (K_o > 0) {
            strip[c] = yv;
            const u32x4 kp = *reinterpret_cast<const u32x4*>(keep + 4 * c);
            y[0] &= kp.x, y[1] &= kp.y, y[2] &= kp.z, y[3] &= kp.w;
        }
        quant_chunk(y, lane, c, c < nchunk, dst, sdst);
    }
    if (B) {
        uint16_t* const brow = B + (int64_t)m * ldb;
        if (K_o > 0) {
            __syncthreads();
            const uint16_t* const raw = reinterpret_cast<const uint16_t*>(strip);
            for (int o = t; o < K_o; o += FT) {
                const int c = o == t ? och0 : oidx[o];
                brow[o] = c >= 0 && c < K ? raw[c] : 0;
            }
        }
        for (int o = K_o + t; o < (int)ldb; o += FT) brow[o] = 0;  // padding columns: +0
    }
}

template <int NCH>
static int launch_row(const uint16_t* X, const uint16_t* gamma, double eps, int64_t M, int64_t K, int64_t ldx, const int32_t* oidx,
                      int32_t K_o, uint8_t* Xq, uint8_t* Xs, uint16_t* B, int64_t ldb, uint16_t* Xn, hipStream_t st) {
    const size_t smem = (size_t)NCH * 256 * 32;  // the row and its keep masks, at most 48 KB
    hipLaunchKernelGGL(rmsnorm_quant_mxfp4_row_kernel<NCH>, dim3((unsigned)M), dim3(FT), smem, st, X, gamma, eps, (int)K, ldx, oidx,
                       (int)K_o, Xq, Xs, B, ldb, Xn);
    return check_launch("rmsnorm_quant_mxfp4_row_kernel");
}

// LDS of the kernel with a row per wavefront; its limit on K_o holds for both kernels
static size_t rmsnorm_lds(int64_t nci, int64_t K, int32_t K_o) {
    const int64_t chunks = nci <= 4 ? 4 : nci <= 8 ? 8 : nci <= 16 ? 16 : 24;
    return (size_t)4 * chunks * 64 * 16 + (size_t)(K / 2) * 4 + (size_t)K * 2 + (size_t)K_o * 2 + 16;
}

template <int NCI>
static int launch_fused_nci(const uint16_t* X, const uint16_t* gamma, double eps, int64_t M, int64_t K, int64_t ldx,
                            const int32_t* oidx, int32_t K_o, uint8_t* Xq, uint8_t* Xs, uint16_t* B, int64_t ldb,
                            uint16_t* Xn, hipStream_t st) {
    const size_t smem = rmsnorm_lds(NCI, K, K_o);
    if (smem > 160 * 1024)
        return fail(OSC_ERR_UNSUPPORTED, "rmsnorm+quantize: K=%lld with K_o=%d needs %zu bytes of LDS", (long long)K,
                    (int)K_o, smem);
    // FULL: every lane holds NCI whole chunks, so the per-chunk bounds tests (and the branches they cost) drop out
    auto kern = K == (int64_t)NCI * 512 ? rmsnorm_quant_mxfp4_kernel<NCI, true> : rmsnorm_quant_mxfp4_kernel<NCI, false>;
    if (smem > 48 * 1024) {
        static LdsReserved lds_reserved;
        if (int rc = reserve_lds(reinterpret_cast<const void*>(kern), smem, lds_reserved)) return rc;
    }
    const int64_t want = (M + 3) / 4;
    // as many workgroups as the chip holds at once (LDS decides how many per CU), each wavefront then
    // takes several rows: measured 29 us against 31.6 us with one row per wavefront at 8192 x 4096
    // (requesting a wavefront's next row ahead of time made it slower again: 31.3 us)
    int per_cu = (int)((160 * 1024) / smem);
    per_cu = per_cu < 1 ? 1 : (per_cu > 8 ? 8 : per_cu);
    const int cap = 256 * per_cu;
    const int grid = (int)(want < cap ? want : cap);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(FT), smem, st, X, gamma, eps, (int)M, (int)K, ldx, oidx, (int)K_o, Xq,
                       Xs, B, ldb, Xn);
    return check_launch("rmsnorm_quant_mxfp4_kernel");
}

int launch_rmsnorm_quant_mxfp4(const uint16_t* X, const uint16_t* gamma, float eps, int64_t M, int64_t K, int64_t ldx,
                               const int32_t* oidx, int32_t K_o, uint8_t* Xq, uint8_t* Xs, uint16_t* B, int64_t ldb,
                               uint16_t* Xn, hipStream_t st) {
    const int64_t nci = (K / 8 + 63) / 64;
    const double e = (double)eps;
    // up to four rows per CU (wide rows: two) the workgroup per row is ahead: figures at the kernel
    const int ncu = cu_count();
    if (M >= 1 && M <= (int64_t)(nci > 8 ? 2 : 4) * (ncu > 0 ? ncu : 256) && nci <= 24 && rmsnorm_lds(nci, K, K_o) <= 160 * 1024) {
        if (nci <= 4) return launch_row<1>(X, gamma, e, M, K, ldx, oidx, K_o, Xq, Xs, B, ldb, Xn, st);
        if (nci <= 8) return launch_row<2>(X, gamma, e, M, K, ldx, oidx, K_o, Xq, Xs, B, ldb, Xn, st);
        if (nci <= 16) return launch_row<4>(X, gamma, e, M, K, ldx, oidx, K_o, Xq, Xs, B, ldb, Xn, st);
        return launch_row<6>(X, gamma, e, M, K, ldx, oidx, K_o, Xq, Xs, B, ldb, Xn, st);
    }
    if (nci <= 4) return launch_fused_nci<4>(X, gamma, e, M, K, ldx, oidx, K_o, Xq, Xs, B, ldb, Xn, st);
    if (nci <= 8) return launch_fused_nci<8>(X, gamma, e, M, K, ldx, oidx, K_o, Xq, Xs, B, ldb, Xn, st);
    if (nci <= 16) return launch_fused_nci<16>(X, gamma, e, M, K, ldx, oidx, K_o, Xq, Xs, B, ldb, Xn, st);
    if (nci <= 24) return launch_fused_nci<24>(X, gamma, e, M, K, ldx, oidx, K_o, Xq, Xs, B, ldb, Xn, st);
    return fail(OSC_ERR_UNSUPPORTED, "rmsnorm+quantize: K=%lld exceeds 12288", (long long)K);
}

// ------------------------------------------------------------------------------------------
// SwiGLU fused with the MXFP8 quantiser of the W_2 fallback (position 4 of Section 2.1; Section
// 3.4; Section 4.1: MXFP8 for the W_2 inputs): y = bf16(bf16(silu(g)) * u) goes straight from
// registers into E4M3 codes and E8M0 scales.
//
// silu is defined as a fixed sequence of correctly rounded single-precision operations (osc.h), but only
// its bf16 rounding is ever used and its argument is a bf16 value, so there are 65536 cases.  The
// sequence below (hardware exp2 and reciprocal, one Newton step on the reciprocal) gives the defined
// sequence's bf16 result in every one of them with a finite gate (compared value by value on the
// device; without the Newton step g = 5.9375, whose silu lies on a rounding boundary, comes out one
// step high).  Eight vector instructions, two of them at quarter rate, instead of 28: the kernels
// below are streams bound by HBM again at every size.  They replaced a 128 KB table in LDS
// (one workgroup per CU, and a 4.7 us launch in front of every call to fill it).
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float silu_bf16_exact(float g) {
    const float z = __builtin_amdgcn_fmed3f(g, -86.0f, 86.0f);
    const float d = 1.0f + __builtin_amdgcn_exp2f(z * -0x1.715476p+0f);
    float r = __builtin_amdgcn_rcpf(d);
    r = __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
    return g * r;
}
// bf16(bf16(silu(g)) * u) for the two halves of a packed word
__device__ __forceinline__ uint32_t swiglu_pair(uint32_t g, uint32_t u) {
    const uint32_t gl = g << 16, gh = g & 0xffff0000u;
    const v2f s = {silu_bf16_exact(__builtin_bit_cast(float, gl)), silu_bf16_exact(__builtin_bit_cast(float, gh))};
    const uint32_t t = __builtin_bit_cast(uint32_t, __builtin_convertvector(s, v2bf));
    return mul_pair(t, u);
}
__device__ __forceinline__ uint32_t max_mag4(const uint32_t (&w)[4]) {  // two 16-bit maxima
    return max_pair(max_pair(w[0] & 0x7fff7fffu, w[1] & 0x7fff7fffu), max_pair(w[2] & 0x7fff7fffu, w[3] & 0x7fff7fffu));
}
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Chunk c (eight channels) of a row: activation, scale code and E4M3 codes; four neighbouring lanes hold a 32-channel block,
// sixteen the four scale bytes of one word.
__device__ __forceinline__ void swiglu_mxfp8_chunk(const u32x4 gv, const u32x4 uv, int lane, int c, bool ok, u32x4* yrow, u32x2* dst, uint8_t* sdst) {
    const uint32_t ww[4] = {swiglu_pair(gv.x, uv.x), swiglu_pair(gv.y, uv.y), swiglu_pair(gv.z, uv.z), swiglu_pair(gv.w, uv.w)};
    if (yrow && ok) __builtin_nontemporal_store((u32x4){ww[0], ww[1], ww[2], ww[3]}, yrow + c);
    const uint32_t a2 = max_mag4(ww);
    uint32_t a = max(a2 & 0xffffu, a2 >> 16);
    a = max(a, (uint32_t)__builtin_amdgcn_mov_dpp((int)a, 0xB1, 0xF, 0xF, true));  // lane ^ 1
    a = max(a, (uint32_t)__builtin_amdgcn_mov_dpp((int)a, 0x4E, 0xF, 0xF, true));  // lane ^ 2
    const uint32_t code = (uint32_t)max((int)(a >> 7) - 8, 0);  // E8M0 code = max(E - 8, 0)
    uint32_t word = code;
    word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)code, 0x104, 0xF, 0xF, true) << 8;
    word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)code, 0x108, 0xF, 0xF, true) << 16;
    word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)code, 0x10C, 0xF, 0xF, true) << 24;
    if ((lane & 15) == 0 && ok) *reinterpret_cast<uint32_t*>(sdst + (c >> 4) * 128) = word;
    const u32x2 out = mxfp8_codes(ww, code);
    // Stored plainly, for the GEMM that reads them next.  Pass and GEMM together, us, streamed -> plain: 32768 x 768 -> 2048 columns 88.1 -> 80.1,
    // 262144 x 768 -> 2048 647 -> 609, 6000 x 12288 -> 512 121.5 -> 115.2, 16384 x 12288 -> 4096 847 -> 834; 24576 x 12288 -> 4096 1282 -> 1293,
    // 100000 x 2048 -> 2048 549 -> 557.  No bound on the size: none would part the gains from the losses, which are large only where a
    // GEMM of few columns follows many rows (16384 x 12288 -> 512 258 -> 278).  The pass by itself gets 5 to 10 % slower (8192 x 12288 78.7 -> 86.2).
    if (ok) dst[c] = out;
}

// 4 B read and 1 B written per element.  One (row, 1024-channel segment) per wavefront and trip as in
// the quantisers; a lane's four 16-byte loads per trip on up to eight wavefronts per SIMD keep enough
// bytes in flight.  8192 x 12288: 98.9 -> 79.0 us (6.4 TB/s), 1000 x 12288: 16.9 -> 12.9 us with streaming stores, table launch
// included in the old figures; 86 to 89 and 13.9 with the plain ones that the GEMM behind gains by.
__global__ void __launch_bounds__(FT) swiglu_quant_mxfp8_kernel(const uint16_t* __restrict__ G,
                                                                const uint16_t* __restrict__ U, int M, int K,
                                                                int64_t ldg, int64_t ldu, uint8_t* __restrict__ Xq,
                                                                uint8_t* __restrict__ Xs, uint16_t* __restrict__ Yn,
                                                                int nseg, int quads, int total_wg) {
    const int Kg = K >> 5, Kg4 = (Kg + 3) >> 2;
    const int nchunk = K >> 3;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    for (int wg = blockIdx.x; wg < total_wg; wg += gridDim.x) {
        const QItem it = quant_item(wg, wave, nseg, quads, M);
        if (it.m < 0) continue;  // uniform over the wavefront
        const int m = it.m;
        const u32x4* gsrc = reinterpret_cast<const u32x4*>(G + (int64_t)m * ldg);
        const u32x4* usrc = reinterpret_cast<const u32x4*>(U + (int64_t)m * ldu);
        const int c0 = it.seg * SEG_CHUNKS + lane;
        u32x4 gv[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}}, uv[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (c0 + 64 * i < nchunk) {
                gv[i] = __builtin_nontemporal_load(gsrc + c0 + 64 * i);
                uv[i] = __builtin_nontemporal_load(usrc + c0 + 64 * i);
            }
        u32x2* dst = reinterpret_cast<u32x2*>(Xq + (int64_t)m * K);
        uint8_t* sdst = Xs + (int64_t)(m >> 5) * Kg4 * 128 + (m & 31) * 4;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c = c0 + 64 * i;
            swiglu_mxfp8_chunk(gv[i], uv[i], lane, c, c < nchunk, Yn ? reinterpret_cast<u32x4*>(Yn + (int64_t)m * K) : nullptr, dst, sdst);
        }
    }
}

// Rows of whole 128-channel words but not of whole segments: the chunks of all rows in one line, 128 per wavefront, so that no
// lane is idle (a segment per row leaves a quarter of them idle at 768 channels and half at 512).  Every die takes a run of
// rows of its own: the four-byte scale words of a 32-row block meet in one L2.  A kernel of its own: with rows by lane instead of by
// wavefront whole segments are 3 to 6 % slower.
__global__ void __launch_bounds__(FT) swiglu_quant_mxfp8_flat_kernel(const uint16_t* __restrict__ G, const uint16_t* __restrict__ U, int M, int K,
                                                                     int64_t ldg, int64_t ldu, uint8_t* __restrict__ Xq,
                                                                     uint8_t* __restrict__ Xs, uint16_t* __restrict__ Yn) {
    const int Kg4 = ((K >> 5) + 3) >> 2, nchunk = K >> 3;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int first = (((int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3)) * 4 + wave) * SEG_CHUNKS;  // gridDim.x: a multiple of 8
    const int row = first / nchunk, col = first - row * nchunk;
    if (row >= M) return;  // uniform over the wavefront
    int m[2], c[2];
    u32x4 gv[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}}, uv[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        m[i] = row;
        c[i] = col + lane + 64 * i;
#pragma unroll
        for (int k = 0; k < 2; ++k) {  // nchunk >= 64, c < nchunk + 128
            const bool over = c[i] >= nchunk;
            c[i] -= over ? nchunk : 0;
            m[i] += over ? 1 : 0;
        }
        if (m[i] < M) {
            gv[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(G + (int64_t)m[i] * ldg) + c[i]);
            uv[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(U + (int64_t)m[i] * ldu) + c[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
        swiglu_mxfp8_chunk(gv[i], uv[i], lane, c[i], m[i] < M, Yn ? reinterpret_cast<u32x4*>(Yn + (int64_t)m[i] * K) : nullptr,
                           reinterpret_cast<u32x2*>(Xq + (int64_t)m[i] * K), Xs + (int64_t)(m[i] >> 5) * Kg4 * 128 + (m[i] & 31) * 4);
}

int launch_swiglu_quant_mxfp8(const uint16_t* G, const uint16_t* U, int64_t M, int64_t K, int64_t ldg, int64_t ldu,
                              uint8_t* Xq, uint8_t* Xs, uint16_t* Yn, hipStream_t st) {
    const int64_t nchunk = K / 8;
    const int nseg = (int)((nchunk + SEG_CHUNKS - 1) / SEG_CHUNKS);
    const RowSplit split = row_split(M, nseg);
    const int64_t total_wg = split.wgs;
    if (total_wg > 0x7fffffff) return fail(OSC_ERR_UNSUPPORTED, "swiglu+quantize: M=%lld too large", (long long)M);
    // One trip per workgroup: the hardware hands out new workgroups as old ones drain, which beats walking a
    // fixed grid at every size of whole segments (8192 x 12288: 79 us, a grid of 8192 86 us, of 2048 92 us; with plain stores 89, 89.6
    // and 93, with the GEMM behind it 413, 417 and 417).
    // Rows of less than a segment are the exception.
    const int64_t flat_wg = (M * nchunk + 4 * SEG_CHUNKS - 1) / (4 * SEG_CHUNKS) + 7;
    // All rows' chunks in one line where segments would leave a fifth of the lanes or more idle, and lanes for a thousand segments
    // in all (us: 32768 x 512 22.3 -> 16.9, x 640 23.6 -> 20.8, x 768 25.8 -> 23.7, 8192 x 1152 13.4 -> 11.6, 4096 x 3200
    // 14.8 -> 14.3, 2000 x 512 3.5 -> 3.2; beyond: 2000 x 1920 5.7 -> 6.1, 4096 x 11136 39 -> 44; with fewer rows idle lanes cost
    // nothing and the division per wavefront does: 32 x 512 2.65 -> 2.86, 512 x 768 3.0 -> 3.3, 1000 x 2304 4.4 -> 4.5)
    if (K % 128 == 0 && K >= 512 && 4 * nseg * SEG_CHUNKS >= 5 * nchunk && M * (nseg * SEG_CHUNKS - nchunk) >= 1000 * SEG_CHUNKS && M * nchunk < ((int64_t)1 << 30) && flat_wg <= MAX_GRID) {
        const unsigned wgs = (unsigned)(flat_wg / 8 * 8);
        hipLaunchKernelGGL(swiglu_quant_mxfp8_flat_kernel, dim3(wgs), dim3(FT), 0, st, G, U, (int)M, (int)K, ldg, ldu, Xq, Xs, Yn);
        return check_launch("swiglu_quant_mxfp8_flat_kernel");
    }
    const int64_t cap = K >= SEG_CH ? MAX_GRID : 4096;
    const int grid = (int)(total_wg < cap ? total_wg : cap);
    hipLaunchKernelGGL(swiglu_quant_mxfp8_kernel, dim3(grid), dim3(FT), 0, st, G, U, (int)M, (int)K, ldg, ldu, Xq,
                       Xs, Yn, nseg, split.quads, (int)total_wg);
    return check_launch("swiglu_quant_mxfp8_kernel");
}

// ------------------------------------------------------------------------------------------
// SwiGLU fused with the per-token FP8 quantiser (Section 3.4: the W_2 inputs stay in 8 bits; this
// is the per-token e4m3 form of that fallback): y = bf16(bf16(silu(g)) * u) stays in registers between
// the row's amax reduction and the conversion, so gate and up are read once and y is never written
// unless asked for.  WPR wavefronts share a row (thread t of them holds chunks t, t + 64 WPR, ...): one
// for rows of at most 2048 channels (no barrier), four for longer ones, so that a few hundred rows
// still occupy the chip and the row's values fit few registers (with a wavefront per row and the table
// 1000 x 12288 took 30.9 us, now 13.0; 8192 x 12288 95.5 -> 84.6 us, 32768 x 768 37.3 -> 24.7 us).
//
// CACHED: codes are stored plainly, for the GEMM that reads them next, but for 120 MB or more of them in rows of at most 1024 channels.
// Pass and GEMM together, us, streamed -> plain: 32768 x 768 -> 2048 columns 89.1 -> 81.6, 150000 x 768 -> 2048 (110 MB) 377 -> 353,
// 200000 x 768 -> 2048 (146 MB) 500 -> 513, 262144 x 768 -> 2048 651 -> 687, 262144 x 512 -> 2048 (128 MB) 501 -> 514; longer rows
// 6000 x 12288 -> 512 122.9 -> 103.4, 8192 x 12288 -> 4096 398 -> 387, 16384 x 12288 -> 4096 820 -> 802, 100000 x 2048 -> 2048 556 -> 550.
// The pass by itself gets 2 to 12 % slower (8192 x 12288 85.6 -> 87.6, 1000 x 12288 12.1 -> 13.6).
// ------------------------------------------------------------------------------------------
template <int CPT, int WPR, bool CACHED = true>
__global__ void __launch_bounds__(FT) swiglu_quant_fp8_kernel(const uint16_t* __restrict__ G,
                                                              const uint16_t* __restrict__ U, int M, int K,
                                                              int64_t ldg, int64_t ldu, uint8_t* __restrict__ X8,
                                                              float* __restrict__ xs, uint16_t* __restrict__ Yn) {
    static_assert(WPR == 1 || WPR == 4, "a wavefront or the workgroup per row");
    __shared__ uint32_t red[2][4];  // two copies by parity of the trip: one barrier per row
    const int t = WPR == 1 ? threadIdx.x & 63 : threadIdx.x, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nchunk = K >> 3;
    int par = 0;
    for (int m = WPR == 1 ? blockIdx.x * 4 + wave : blockIdx.x; m < M; m += gridDim.x * (4 / WPR), par ^= 1) {
        const u32x4* gsrc = reinterpret_cast<const u32x4*>(G + (int64_t)m * ldg);
        const u32x4* usrc = reinterpret_cast<const u32x4*>(U + (int64_t)m * ldu);
        u32x4 gv[CPT], uv[CPT];
        uint32_t y[CPT][4];
        uint32_t a2 = 0;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            const int c = t + 64 * WPR * i;
            gv[i] = uv[i] = (u32x4){0u, 0u, 0u, 0u};
            if (c < nchunk) {
                gv[i] = __builtin_nontemporal_load(gsrc + c);
                uv[i] = __builtin_nontemporal_load(usrc + c);
            }
        }
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            const int c = t + 64 * WPR * i;
            y[i][0] = swiglu_pair(gv[i].x, uv[i].x);
            y[i][1] = swiglu_pair(gv[i].y, uv[i].y);
            y[i][2] = swiglu_pair(gv[i].z, uv[i].z);
            y[i][3] = swiglu_pair(gv[i].w, uv[i].w);
            a2 = max_pair(a2, max_mag4(y[i]));
            if (Yn && c < nchunk)
                __builtin_nontemporal_store((u32x4){y[i][0], y[i][1], y[i][2], y[i][3]},
                                            reinterpret_cast<u32x4*>(Yn + (int64_t)m * K) + c);
        }
        uint32_t a = wave_max_u32(max(a2 & 0xffffu, a2 >> 16));
        if constexpr (WPR == 4) {
            if ((t & 63) == 0) red[par][wave] = a;
            __syncthreads();
            a = max(max(red[par][0], red[par][1]), max(red[par][2], red[par][3]));
        }
        const float amax = __builtin_bit_cast(float, a << 16);
        float scale = 1.0f, inv = 1.0f;
        if (amax >= 0x1p-100f) {
            scale = __fdiv_rn(amax, 448.0f);
            inv = __fdiv_rn(448.0f, amax);
        }
        if (t == 0) xs[m] = scale;
        u32x2* dst = reinterpret_cast<u32x2*>(X8 + (int64_t)m * K);
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            const int c = t + 64 * WPR * i;
            if (c < nchunk) {
                if constexpr (CACHED) dst[c] = fp8_codes(y[i], inv);
                else __builtin_nontemporal_store(fp8_codes(y[i], inv), dst + c);
            }
        }
    }
}

int launch_swiglu_quant_fp8(const uint16_t* G, const uint16_t* U, int64_t M, int64_t K, int64_t ldg, int64_t ldu,
                            uint8_t* X8, float* xs, uint16_t* Yn, hipStream_t st) {
    const int64_t nchunk = K / 8;
    if (nchunk > 8 * FT) return fail(OSC_ERR_UNSUPPORTED, "swiglu+fp8 quantize: K=%lld exceeds 16384", (long long)K);
    const bool wave_rows = nchunk <= 4 * 64;
    // one row (four short rows) per workgroup, as above: 8192 x 12288 81 us, 81.5 on a grid of 8192, 87 on one of 2048
    const int64_t want = wave_rows ? (M + 3) / 4 : M;
    const int grid = (int)(want < MAX_GRID ? want : MAX_GRID);
    const int64_t cpt = wave_rows ? (nchunk + 63) / 64 : (nchunk + FT - 1) / FT;
    const bool streamed = K <= 1024 && M * K >= ((int64_t)120 << 20);
#define OSC_SLAUNCH(...)                                                                                             \
    hipLaunchKernelGGL((swiglu_quant_fp8_kernel<__VA_ARGS__>), dim3(grid), dim3(FT), 0, st, G, U, (int)M, (int)K, ldg, ldu, X8, \
                       xs, Yn)
    if (streamed) {
        if (cpt <= 1) OSC_SLAUNCH(1, 1, false);
        else OSC_SLAUNCH(2, 1, false);
    } else if (wave_rows) {
        if (cpt <= 1) OSC_SLAUNCH(1, 1);
        else if (cpt <= 2) OSC_SLAUNCH(2, 1);
        else OSC_SLAUNCH(4, 1);
    } else if (cpt <= 2) OSC_SLAUNCH(2, 4);
    else if (cpt <= 4) OSC_SLAUNCH(4, 4);
    else if (cpt <= 6) OSC_SLAUNCH(6, 4);
    else OSC_SLAUNCH(8, 4);
#undef OSC_SLAUNCH
    return check_launch("swiglu_quant_fp8_kernel");
}

}  // namespace osc
