// Flowing GEMM kernel: dual path, per-token FP8 and MXFP8 on operand rows that are whole 128-byte lines; tiles of
// medium size for one problem, 128 x 256 for experts.
#include "gemm_tile.h"

namespace osc {

// ------------------------------------------------------------------------------------------
// One persistent workgroup of eight wavefronts (two per SIMD) per CU walks a list of tiles.  A stage is 128 bytes of
// every operand row, as in the DMA kernel; a ring of NSTG stages in LDS is filled by global->LDS DMA three or four
// stages ahead of the products, across tile borders, and a stage costs one barrier:
//
//   first half:   products on X (first half of stage T, registers)   | fragments of the second half -> Yf;
//                                                                      SPLIT: rest of the requests for stage T + LEAD - 1
//   barrier:      this wavefront's requests for stage T + 1 have landed; all have read stage T
//   second half:  products on Yf                                     | (first) requests for stage T + LEAD into the slot of T;
//                                                                      first half of stage T + 1 -> X
//
// so fragments are read half a stage before the products that need them, and no wait in the loop is for a request
// younger than stage T + 1 (requests are counted: the scale words and tile scales that only some wavefronts fetch are
// left out of the count, which makes those wait for a little more than they must).  With LAG the barrier does not wait
// for the reads of stage T: the requests go to the slot of stage T - 1 instead, whose reads the products of T have
// waited for.  That is for the smallest tile, whose few products cover no LDS latency.
//
// Experts: the running tile counts and first rows go into LDS once; a tile's expert is found by one parallel comparison.
// The entries of a row map travel a tile ahead (every wavefront fetches those that its own requests need), the scale
// words of rows that do not start at a 32-row block are gathered word by word.  128 experts of 1536 x 2048 with about 256
// rows each: 103 us against 117 for 256-row tiles and a second launch; without the result stores 90, without the
// requests 76 (HBM: 364 MB, 70 us at the rate of a copy); skipping the empty half of an expert's last tile is 3 to 4 % of it.
//
// What bounds it.  128 x 256 tiles, K = 4096 (FP8): the matrix cores are busy 75 % of the kernel's cycles, but the clock is
// 1.7 GHz (2.35 without fragment reads and requests, 1.8 without requests): power.  Reading the fragments of 64 x 64
// outputs per wavefront costs twice the LDS traffic of the persistent kernel's 128 x 128, which is why whole rounds of
// 256 x 256 tiles stay there (8192 x 24576 x 4096: 470 to 495 us there, 545 to 575 here).  64 x 128 tiles: 24 KB of
// requests per stage and CU, 17 to 21 TB/s.  Tried: four wavefronts of twice the size (35 us against 25 on
// 8192 x 1024 x 4096: nothing covers a wavefront that waits for its request to be taken); results kept as bf16 and stored
// during the next tile's stages (no change, though without any stores the kernel is 10 to 20 % faster); raised wave
// priority around the products (4 to 7 % slower); fragments read in the first one or two slots (no change).
// Figures against the kernels that had these calls stand beside the launcher's rule.  With LEAD stages a tile or fewer the load
// cursor crosses several tiles: the FP8 tile scales then have more copies, and with one stage the row map is waited for.
// ------------------------------------------------------------------------------------------

// FP8: copies of the tile scales.  The load cursor fetches those of the tile that its next stage belongs to, LEAD + 1 stages
// ahead of the products: the next tile, or with no more than LEAD stages a tile (FEW) up to the fourth from here.
constexpr int tile_scale_copies(bool few) { return few ? 5 : 2; }

// LDS of one ring slot: the operand rows of a stage, 128 bytes each, then its scale words in whole 1 KB requests
template <int MODE, int BM, int BN>
struct FlowSlot {
    static constexpr int BLK = (BM + BN) / 32;
    static constexpr int SBB = MODE == MODE_DUAL ? 256 : 128;  // scale bytes per 32 rows and stage
    static constexpr int ROWS = (BM + BN) * 128;
    static constexpr int SCL = MODE == MODE_FP8 ? 0 : (BM / 32) * SBB + ((BN / 32) * SBB + 1023) / 1024 * 1024;
    static constexpr int SCL1 = MODE == MODE_FP8 ? 0 : (BLK * SBB + 1023) / 1024 * 1024;
    static constexpr int BYTES = ROWS + (SCL > SCL1 ? SCL : SCL1);
};

// FEW: LEAD stages a tile or fewer.  A form of its own because the others run up to half a percent slower with its bookkeeping.
template <int MODE, int WM, int WN, int TM, int TN, int NSTG, bool LAG, bool GROUPED, bool FEW>
__global__ void __launch_bounds__(64 * WM * WN) gemm_flow_kernel(KArgs a, int ntiles) {
    constexpr bool DUAL = MODE == MODE_DUAL, FP8 = MODE == MODE_FP8, MX = MODE == MODE_MX8;
    constexpr int NW = WM * WN, RPP = 8 * NW, BM = 32 * TM * WM, BN = 32 * TN * WN;
    constexpr int LA = BM / RPP, LB = BN / RPP, NLD = LA + LB;
    constexpr int NBA = BM / 32, NBB = BN / 32, NBLK = NBA + NBB;
    using Slot = FlowSlot<MODE, BM, BN>;
    constexpr int SBB = Slot::SBB, BPR = 1024 / SBB, PPB = SBB / 16;  // 32-row blocks per 16-byte request, pieces per block
    constexpr int HR = TM + TN;
    constexpr int LEAD = LAG ? NSTG - 1 : NSTG;  // stages between the compute cursor and the load cursor
    static_assert(BM % RPP == 0 && BN % RPP == 0, "tile does not split over the wavefronts");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / WN, wn = wave % WN, q = lane >> 5, r = lane & 31;
    const int Kg4 = ((a.K >> 5) + 3) >> 2;
    const uint32_t rowbytes = DUAL ? (uint32_t)a.K >> 1 : (uint32_t)a.K;
    const int nTA = (int)(rowbytes >> 7);
    const int nTB = DUAL ? (a.K_o * 2 + 127) >> 7 : 0;
    const int nT = nTA + nTB;  // without FEW more than LEAD (the host sees to it)
    // behind the ring: FP8, the row and column scales of NTSC tiles in turn; grouped, the experts' running tile
    // counts and first rows; mapped rows, 64 entries per wavefront
    constexpr int NTSC = tile_scale_copies(FEW);
    float* const tsc = reinterpret_cast<float*>(lds + NSTG * Slot::BYTES);
    int* const cum_l = reinterpret_cast<int*>(lds + NSTG * Slot::BYTES + (FP8 ? NTSC * (BM + BN) * 4 : 0));  // [E + 1]
    int* const off_l = cum_l + a.E + 1;                                                                   // [E + 1]
    int* const map_l = off_l + a.E + 1;                                                                   // [NW][64]
    const bool mapped = GROUPED && DUAL && a.row_map != nullptr;
    const int tiles_m = (a.M + BM - 1) / BM;

    if constexpr (GROUPED) {
        if (wave == 0) {
            int before = 0;
            for (int e0 = 0; e0 < a.E; e0 += 64) {
                const int e = e0 + lane;
                const int b = e < a.E ? a.off[e] : 0, n = e < a.E ? a.off[e + 1] - b : 0;
                const int te = n > 0 ? (n + BM - 1) / BM * a.tiles_n : 0;
                int ps = te;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const int u = __shfl_up(ps, d);
                    if (lane >= d) ps += u;
                }
                if (e < a.E) {
                    cum_l[e] = before + ps - te;
                    off_l[e] = b;
                }
                before += __shfl(ps, 63);
            }
            if (lane == 0) {
                cum_l[a.E] = before;
                off_l[a.E] = a.off[a.E];
            }
        }
        __syncthreads();
        ntiles = __builtin_amdgcn_readfirstlane(cum_l[a.E]);
    }
    // this workgroup's tiles: ltile, ltile + step, ... below last.  Every XCD owns a contiguous run of tiles, as many
    // (to within one) as the others, and no more than its workgroups where there is a workgroup per tile
    const int xcd = blockIdx.x & 7, step = (gridDim.x + 7 - xcd) >> 3;
    const int per = ntiles >> 3, extra = ntiles & 7;
    int ltile = xcd * per + min(xcd, extra);
    const int last = ltile + per + (xcd < extra ? 1 : 0);
    ltile += blockIdx.x >> 3;
    if (ltile >= last) return;
    int left = FEW ? (last - ltile + step - 1) / step * nT : 0;  // stages from the compute cursor on

    auto find_tile = [&](int v) __attribute__((always_inline)) -> TilePos {
        TilePos p;
        p.valid = true;
        if constexpr (GROUPED) {
            // the last expert whose first tile number is <= v: experts without tiles share that number with
            // their successor
            int cnt = 0;
            for (int e0 = 0; e0 < a.E; e0 += 64) {
                const int e = e0 + lane;
                cnt += __popcll(__ballot(e < a.E && cum_l[e < a.E ? e : 0] <= v));
            }
            const int e = __builtin_amdgcn_readfirstlane(cnt - 1);
            const int first = __builtin_amdgcn_readfirstlane(cum_l[e]), all = __builtin_amdgcn_readfirstlane(cum_l[e + 1]) - first;
            p.row_begin = __builtin_amdgcn_readfirstlane(off_l[e]);
            p.row_end = __builtin_amdgcn_readfirstlane(off_l[e + 1]);
            const int mt = all / a.tiles_n, in = v - first;
            const int tn = in / mt;  // an expert's row tiles of one column strip are neighbours: they share its weights
            p.m0 = p.row_begin + (in - tn * mt) * BM;
            p.n0 = tn * BN;
            p.wp = a.Wpack + (size_t)e * a.pack_stride;
        } else {
            const int band = v / (8 * a.tiles_n), within = v - band * 8 * a.tiles_n;
            const int rows = min(8, tiles_m - band * 8);
            p.row_begin = 0;
            p.row_end = a.M;
            p.m0 = (band * 8 + within % rows) * BM;
            p.n0 = (within / rows) * BN;
            p.wp = a.Wpack;
        }
        return p;
    };

    // ---- load cursor ---------------------------------------------------------------------------------
    const uint32_t c8 = (uint32_t)((t & 7) ^ swz8(t >> 3)) * 16u;
    TilePos ld = find_tile(ltile), cur = ld;
    int lT = 0, lslot = 0, lpar = 0;
    uint32_t ga[LA], gb[LB], voa[LA], vob[LB];
    const uint8_t *pa, *pb;
    const uint8_t* psc = nullptr;  // this lane's scale source
    uint32_t so = 0;
    // scale requests of a stage: which wavefronts issue one, and of which width
    const bool gather_s = GROUPED;  // rows that do not start at a 32-row block: A's scale words lane by lane
    const int nreq4 = FP8 ? 0 : gather_s ? (DUAL ? NBA : (NBA + 1) / 2) : 0;
    const int nreq16 = FP8 ? 0 : gather_s ? (NBB + BPR - 1) / BPR : (NBLK + BPR - 1) / BPR;
    static_assert(FP8 || (GROUPED ? (DUAL ? NBA : (NBA + 1) / 2) + (NBB + BPR - 1) / BPR : (NBLK + BPR - 1) / BPR) <= NW, "scale requests");

    auto request_map = [&](const TilePos& p) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the entries that these replace have been read
        const int idx = lane < 32 ? wave * 8 + (lane & 7) + RPP * min(lane >> 3, LA - 1) : min(wave, NBA - 1) * 32 + r;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(a.row_map + min(p.m0 + idx, p.row_end - 1)),
                                         (__attribute__((address_space(3))) void*)(map_l + wave * 64), 4, 0, 0);
    };
    auto enter_tile = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < LA; ++i) ga[i] = (uint32_t)min(ld.m0 + (t >> 3) + RPP * i, ld.row_end - 1);
#pragma unroll
        for (int i = 0; i < LB; ++i) gb[i] = (uint32_t)min(ld.n0 + pair_col<TN, WN>((t >> 3) + RPP * i), a.N - 1);
        int gs = min(ld.m0 + wave * 32 + r, ld.row_end - 1);
        if (mapped) {
#pragma unroll
            for (int i = 0; i < LA; ++i) ga[i] = (uint32_t)map_l[wave * 64 + i * 8 + (lane >> 3)];
            gs = map_l[wave * 64 + 32 + r];
        }
#pragma unroll
        for (int i = 0; i < LA; ++i) voa[i] = ga[i] * rowbytes + c8;
#pragma unroll
        for (int i = 0; i < LB; ++i) vob[i] = gb[i] * rowbytes + c8;
        pa = a.Xq;
        pb = ld.wp + a.off_q;
        lT = 0;
        so = 0;
        const uint8_t* const wsb = ld.wp + a.off_s;
        if constexpr (DUAL || MX) {
            const uint32_t pitch = (uint32_t)Kg4 * 128u;
            if constexpr (GROUPED) {
                if (wave < nreq4) {
                    if (MX) gs = min(ld.m0 + wave * 64 + lane, ld.row_end - 1);
                    psc = a.Xs + ((size_t)((uint32_t)gs >> 5) * pitch + ((uint32_t)gs & 31) * 4u + (DUAL ? q * 128u : 0u));
                } else {
                    const int b = min((wave - nreq4) * BPR + lane / PPB, NBB - 1);
                    psc = wsb + ((size_t)min((ld.n0 >> 5) + b, (a.N - 1) >> 5) * pitch + (uint32_t)(lane % PPB) * 16u);
                }
            } else {
                const int b = min(wave * BPR + lane / PPB, NBLK - 1);
                psc = (b < NBA ? a.Xs + (size_t)min((ld.m0 >> 5) + b, (ld.row_end - 1) >> 5) * pitch
                               : wsb + (size_t)min((ld.n0 >> 5) + b - NBA, (a.N - 1) >> 5) * pitch) + (lane % PPB) * 16u;
            }
        }
        if constexpr (FP8) {
            const float* const wcs = reinterpret_cast<const float*>(wsb);
#pragma unroll
            for (int k = 0; k < (BM + BN) / 64; k += NW)
                if (k + wave < (BM + BN) / 64) {
                    const int idx = (k + wave) * 64 + lane;
                    const float* src = idx < BM ? a.xs + min(ld.m0 + idx, ld.row_end - 1) : wcs + min(ld.n0 + idx - BM, a.N - 1);
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                                     (__attribute__((address_space(3))) void*)(tsc + lpar * (BM + BN) + (k + wave) * 64), 4, 0, 0);
                }
        }
    };
    // data request number l of the stage under the load cursor
    auto load_one = [&](int l) __attribute__((always_inline)) {
        uint8_t* const dst = lds + lslot * Slot::BYTES + wave * 1024;
        if (l < LA) load_to_lds16(pa + voa[l < LA ? l : 0], dst + l * (RPP * 128));
        else load_to_lds16(pb + vob[l >= LA ? l - LA : 0], dst + BM * 128 + (l - LA) * (RPP * 128));
    };
    // the stage's scale words, then one stage further; past the last tile's last stage the cursor stands still
    auto finish_stage = [&]() __attribute__((always_inline)) {
        if constexpr (DUAL || MX) {
            uint8_t* const scl = lds + lslot * Slot::BYTES + Slot::ROWS;
            if (wave < nreq4)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(psc + so),
                                                 (__attribute__((address_space(3))) void*)(scl + wave * 256), 4, 0, 0);
            else if (wave < nreq4 + nreq16)
                load_to_lds16(psc + so, scl + (GROUPED ? NBA * SBB + (wave - nreq4) * 1024 : wave * 1024));
        }
        lslot = lslot + 1 == NSTG ? 0 : lslot + 1;
        ++lT;
        pa += 128;
        pb += 128;
        if (lT < nTA) so += SBB;
        if (DUAL && lT == nTA && lT < nT) {
            pa = a.B;
            pb = ld.wp + a.off_l;
#pragma unroll
            for (int i = 0; i < LA; ++i) voa[i] = ga[i] * (uint32_t)a.bpitch + c8;
#pragma unroll
            for (int i = 0; i < LB; ++i) vob[i] = gb[i] * (uint32_t)a.wlpitch + c8;
        }
        if (lT == nT && ltile + step < last) {
            if (FEW && mapped && nT == 1) wait_vmcnt<0>();  // the map entries have been asked for since the last barrier
            ltile += step;
            ld = find_tile(ltile);
            lpar = lpar + 1 == NTSC ? 0 : lpar + 1;
            enter_tile();
            if (mapped && ltile + step < last) request_map(find_tile(ltile + step));
        }
    };

    // ---- compute side ----------------------------------------------------------------------------------
    u32x4 X[HR][2], Yf[HR][2];  // fragments of the first and second half of a stage
    int sX[HR], sY[HR];
    v16f acc[TM][TN];
    const int ra0 = wm * (TM * 32) + r, rb0 = BM + wn * (TN * 32) + r;
    int cslot = 0;
    // fragment read u (0 .. 2 HR - 1) of half H of the stage in slot s; 8 bits need both pieces of a block for one MFMA
    auto read_frag = [&](u32x4 (&F)[HR][2], int u, int H, int s) __attribute__((always_inline)) {
        const int blk = DUAL ? u % HR : u / 2, p = DUAL ? u / HR : u % 2;
        const int piece = MX ? 4 * H + q + 2 * p : 4 * H + 2 * q + p;
        F[blk][p] = *reinterpret_cast<const u32x4*>(lds + s * Slot::BYTES +
                                                    st128_off(blk < TM ? ra0 + 32 * blk : rb0 + 32 * (blk - TM), piece));
    };
    auto read_scale = [&](int (&S)[HR], int b, int H, int s) __attribute__((always_inline)) {
        // X: row r of block b.  Weights: the row that pair_col() gives to lane r; a block's words lie in the order of the rows
        const int j = b - TM;
        const bool single = TN % 2 && j == TN - 1;
        const uint8_t* const blk = lds + s * Slot::BYTES + Slot::ROWS + (b < TM ? wm * TM + b : NBA + block_col<TN, WN>(wn, single ? j : j & ~1) / 32) * SBB;
        const uint8_t* const sc = blk + (b < TM ? r * 4 : single ? (2 * (r & 15) + (r >> 4)) * 4 : pair_scale(r, SBB) + (j & 1) * 4);
        if constexpr (DUAL) S[b] = *reinterpret_cast<const uint16_t*>(sc + H * 128 + 2 * q);
        else S[b] = sc[2 * H + q];
    };
    const v16f zero = {};
    // fresh: the tile's first products start from zero (clearing the accumulators takes two wavefronts 512 cycles a tile: 1 to 2 %
    // of experts' tiles, 1 % of others; FEW, whose first stage may be the last, clears them)
    auto mfma = [&](auto fp4, auto fresh, const u32x4 (&F)[HR][2], const int (&S)[HR], int n) __attribute__((always_inline)) {
        if constexpr (DUAL) {
            const int p = n / (TM * TN), i = n % (TM * TN) / TN, j = n % TN;
            if constexpr (decltype(fp4)::value) {
                const v8i av = {(int)F[i][p].x, (int)F[i][p].y, (int)F[i][p].z, (int)F[i][p].w, 0, 0, 0, 0};
                const v8i bv = {(int)F[TM + j][p].x, (int)F[TM + j][p].y, (int)F[TM + j][p].z, (int)F[TM + j][p].w, 0, 0, 0, 0};
                if (p == 0) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, decltype(fresh)::value ? zero : acc[i][j], 4, 4, 0, S[i], 0, S[TM + j]);
                else acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc[i][j], 4, 4, 1, S[i], 1, S[TM + j]);
            } else {
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, F[i][p]), __builtin_bit_cast(v8bf, F[TM + j][p]),
                                                                    acc[i][j], 0, 0, 0);
            }
        } else {
            const int i = n / TN, j = n % TN;
            const v8i av = {(int)F[i][0].x, (int)F[i][0].y, (int)F[i][0].z, (int)F[i][0].w,
                            (int)F[i][1].x, (int)F[i][1].y, (int)F[i][1].z, (int)F[i][1].w};
            const v8i bv = {(int)F[TM + j][0].x, (int)F[TM + j][0].y, (int)F[TM + j][0].z, (int)F[TM + j][0].w,
                            (int)F[TM + j][1].x, (int)F[TM + j][1].y, (int)F[TM + j][1].z, (int)F[TM + j][1].w};
            if constexpr (MX) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, decltype(fresh)::value ? zero : acc[i][j], 0, 0, 0, S[i], 0, S[TM + j]);
            else acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, decltype(fresh)::value ? zero : acc[i][j], 0, 0, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f);
        }
    };
    constexpr int NSLOT = (DUAL ? 2 : 1) * TM * TN;              // MFMAs of a half stage
    constexpr int RSL = NSLOT * 5 / 8 > 0 ? NSLOT * 5 / 8 : 1;   // slots that carry fragment reads
    constexpr int RPS = (2 * HR + RSL - 1) / RSL;
    constexpr int SPS = (HR + RSL - 1) / RSL;
    // SPLIT: NL1 of a stage's requests go out behind the barrier, the others before the next one.  A CU takes a request of
    // 1 KB in 16 cycles, so the 24 to 48 of a stage are more than half a stage of FP4 products covers.  Experts of 256 rows 122 ->
    // 119.5 us (dual), 92.8 -> 91.4 (MXFP8); 64 x 128 tiles 11.3 -> 11.0, 7.2 -> 6.9.  The larger tiles of one problem are level or, with
    // operands in the second-level caches, up to 2 % slower (8192 x 1024 x 4096), as is 512 x 4096 x 768 in the form FEW (3 %).
    constexpr bool SPLIT = (LAG || GROUPED) && !FEW;
    constexpr int NL1 = SPLIT ? (NLD + 1) / 2 : NLD;
    const std::integral_constant<int, 0> none{};
    const std::integral_constant<int, NL1> part1{};
    const std::integral_constant<int, NLD - NL1> part2{};
    // requests first, first + 1, ... (count of them) are spread over the half's products
    auto half = [&](auto fp4, auto fresh, auto first, auto count, const u32x4 (&F)[HR][2], const int (&S)[HR], u32x4 (&G)[HR][2], int (&R)[HR], int H,
                    int s) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NSLOT; ++n) {
            mfma(fp4, fresh, F, S, n);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < SPS; ++u)
                if (!FP8 && n * SPS + u < HR) read_scale(R, n * SPS + u, H, s);
#pragma unroll
            for (int u = 0; u < RPS; ++u)
                if (n * RPS + u < 2 * HR) read_frag(G, n * RPS + u, H, s);
            constexpr int FIRST = decltype(first)::value, COUNT = decltype(count)::value;
#pragma unroll
            for (int l = 0; l < COUNT; ++l)
                if (l * NSLOT / (COUNT > 0 ? COUNT : 1) == n) load_one(FIRST + l);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // the branches of finish_stage() end the basic block: without a use of the results there the compiler sinks
    // every MFMA of the stage below them
    auto keep_products = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(acc[i][j]));
    };
    auto load_rest = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int l = NL1; l < NLD; ++l) load_one(l);
        finish_stage();
    };
    // load: there is a stage to ask for behind the barrier; rest: the one before it still has requests to come
    auto stage = [&](auto fp4, auto fresh, auto load, bool rest) __attribute__((always_inline)) {
        constexpr bool LOAD = decltype(load)::value;
        if constexpr (SPLIT && LOAD) {
            half(fp4, fresh, part1, part2, X, sX, Yf, sY, 1, cslot);
            keep_products();
            finish_stage();
        } else {
            if (SPLIT && rest) load_rest();
            half(fp4, fresh, none, none, X, sX, Yf, sY, 1, cslot);
        }
        if constexpr (!LAG) __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wavefront has read the whole stage
        if (LOAD || (SPLIT && rest)) wait_vmcnt<(LEAD - 2) * NLD>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        cslot = cslot + 1 == NSTG ? 0 : cslot + 1;
        if constexpr (LOAD) half(fp4, std::false_type{}, none, part1, Yf, sY, X, sX, 0, cslot);
        else half(fp4, std::false_type{}, none, none, Yf, sY, X, sX, 0, cslot);
        keep_products();
        if constexpr (!SPLIT && LOAD) finish_stage();
    };

    // first half of the stage under the compute cursor
    auto read_first = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2 * HR; ++u) read_frag(X, u, 0, cslot);
        if constexpr (!FP8) {
#pragma unroll
            for (int u = 0; u < HR; ++u) read_scale(sX, u, 0, cslot);
        }
    };

    // ---- prologue ----------------------------------------------------------------------------------------
    int ctile = ltile, cpar = 0;  // (with LEAD stages or fewer the load cursor leaves the first tile here)
    if (mapped) {
        request_map(ld);
        wait_vmcnt<0>();
    }
    enter_tile();
    if (mapped && ltile + step < last) request_map(find_tile(ltile + step));
#pragma unroll 1
    for (int s = 0; s < (FEW ? min(LEAD, left) : LEAD); ++s) {
#pragma unroll
        for (int l = 0; l < NL1; ++l) load_one(l);
        if (SPLIT && s + 1 == LEAD) break;  // the first stage asks for the rest
#pragma unroll
        for (int l = NL1; l < NLD; ++l) load_one(l);
        if (FEW && mapped && lT + 1 == nT) wait_vmcnt<0>();  // the next tile is entered before the loop's waits have covered its map entries
        finish_stage();
    }
    if (!FEW || left >= LEAD) wait_vmcnt<(LEAD - 2) * NLD + NL1>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_first();

#pragma unroll 1
    for (;;) {
        const bool more = ctile + step < last;
        // stages behind whose barrier there is still something to load, and those that have a rest to ask for (SPLIT)
        const int L = FEW ? min(nT, max(left - LEAD, 0)) : more ? nT : nT - LEAD;
        const int LR = more ? nT : nT - LEAD + 1;
        if constexpr (FEW) left -= nT;
        int T = 0;
        if (!GROUPED || cur.m0 + wm * (TM * 32) < cur.row_end) {
            if constexpr (FEW) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int k = 0; k < 16; ++k) acc[i][j][k] = 0.0f;
            }
            const std::true_type yes{};
            const std::false_type no{};
            if constexpr (!FEW) stage(yes, yes, yes, true), ++T;
            if constexpr (DUAL) {
#pragma unroll 1
                for (; T < min(nTA, L); ++T) stage(yes, no, yes, true);
#pragma unroll 1
                for (; T < L; ++T) stage(no, no, yes, true);
#pragma unroll 1
                for (; T < nTA; ++T) stage(yes, no, no, T < LR);
#pragma unroll 1
                for (; T < nT; ++T) stage(no, no, no, T < LR);
            } else {
#pragma unroll 1
                for (; T < L; ++T) stage(yes, no, yes, true);
#pragma unroll 1
                for (; T < nT; ++T) stage(yes, no, no, T < LR);
            }
            store_pairs<MODE, TM, TN, WN, WM, FP8>(a, cur, acc, tsc + cpar * (BM + BN));
        } else {
            // an expert's last tile, no rows for this wavefront: it loads for the others and keeps their barriers
#pragma unroll 1
            for (; T < nT; ++T) {
                if (SPLIT && T < LR) load_rest();
                __builtin_amdgcn_s_waitcnt(0xC07F);
                if (T < (SPLIT ? LR : L)) wait_vmcnt<(LEAD - 2) * NLD>();
                else wait_vmcnt<0>();
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_sched_barrier(0);
                cslot = cslot + 1 == NSTG ? 0 : cslot + 1;
                if (T < L) {
#pragma unroll
                    for (int l = 0; l < NL1; ++l) load_one(l);
                    if constexpr (!SPLIT) finish_stage();
                }
            }
            read_first();
        }
        if (!more) break;
        ctile += step;
        if constexpr (FEW) cur = find_tile(ctile);
        else cur = ld;
        cpar = cpar + 1 == NTSC ? 0 : cpar + 1;
    }
}

// ---- host ------------------------------------------------------------------------------------------

static size_t flow_lds(int mode, int bm, int bn, int slots, bool few, bool grouped, int E) {
    const size_t scl = mode == MODE_FP8 ? 0 : mode == MODE_DUAL ? 256 : 128;
    const size_t together = align_up((bm + bn) / 32 * scl, 1024), apart = bm / 32 * scl + align_up(bn / 32 * scl, 1024);
    return slots * ((size_t)(bm + bn) * 128 + (apart > together ? apart : together)) + (mode == MODE_FP8 ? (size_t)tile_scale_copies(few) * (bm + bn) * 4 : 0) +
           (grouped ? (size_t)(2 * E + 2) * 4 + (mode == MODE_DUAL ? 8 * 256 : 0) : 0);
}

template <int MODE, int WM, int WN, int TM, int TN, int NSTG, bool LAG, bool GROUPED, bool FEW>
static int launch_cfg(KArgs a, hipStream_t st) {
    constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN, NW = WM * WN;
    static_assert(NW == 8, "two wavefronts per SIMD");
    a.tiles_n = (a.N + BN - 1) / BN;
    const int64_t ntiles = ((int64_t)(a.M + BM - 1) / BM + (GROUPED ? a.E : 0)) * a.tiles_n;  // grouped: an upper bound
    if (ntiles <= 0) return OSC_OK;
    if (ntiles > 0x7fffffff) return fail(OSC_ERR_UNSUPPORTED, "gemm: too many tiles");
    const int ncu = cu_count();
    if (ncu <= 0) return fail(OSC_ERR_HIP, "gemm: cannot read the number of compute units");
    const size_t smem = flow_lds(MODE, BM, BN, NSTG, FEW, GROUPED, a.E);
    const int64_t grid = ntiles < ncu ? ntiles : ncu;  // one workgroup per CU, each walks its list of tiles
    auto kern = gemm_flow_kernel<MODE, WM, WN, TM, TN, NSTG, LAG, GROUPED, FEW>;
    static LdsReserved lds_reserved;
    if (int rc = reserve_lds(reinterpret_cast<const void*>(kern), smem, lds_reserved)) return rc;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * NW), smem, st, a, (int)ntiles);
    return check_launch("gemm_flow_kernel");
}

// What a launch costs, in us beyond its start: every round of tiles costs `round` plus `stage` per stage, and every
// stage of a tile `share` times the part of the CUs that has one (operands and power are shared).  Least-squares fits
// over 250 shapes (96 to 8192 rows, 1024 to 12288 columns, K 1024 to 12288) with an earlier epilogue, within 3 to 5 % on average
// then.  Every tile has become faster since, and the order between them holds: over 150 drawn shapes of these ranges that run here the
// chosen tile is 0.1 % behind the fastest of the four on average, by more than 3 % in two (3060 x 2000 x 1024 FP8 11.8 us, 64 x 128 11.3;
// 3549 x 1768 x 1024 dual 11.1, 128 x 128 10.7).
struct FlowTile {
    int bm, bn, slots, lead;
    float round, stage, share;      // dual path
    float round8, stage8, share8;   // FP8, MXFP8
};
static const FlowTile FLOW_TILES[] = {
    {128, 256, 3, 3, 3.9f, 0.52f, 0.32f, 3.2f, 0.51f, 0.21f},
    {128, 192, 3, 3, 4.0f, 0.42f, 0.25f, 3.7f, 0.42f, 0.19f},
    {128, 128, 4, 4, 2.3f, 0.35f, 0.16f, 1.7f, 0.31f, 0.15f},
    {64, 128, 5, 4, 1.0f, 0.31f, 0.06f, 1.0f, 0.25f, 0.06f},
};
constexpr int FLOW_COUNT = sizeof(FLOW_TILES) / sizeof(FLOW_TILES[0]);

bool flow_fits(int mode, int tile, int stages, bool grouped, int E) {
    if (tile < 0 || tile >= FLOW_COUNT || (grouped && tile != 0)) return false;
    const FlowTile& f = FLOW_TILES[tile];
    const bool few = stages <= f.lead;  // built for experts, and for the dual path on 64 x 128 tiles (two stages or more)
    if (few && !(grouped ? stages >= 1 : mode == MODE_DUAL && tile == 3 && stages >= 2)) return false;
    return flow_lds(mode, f.bm, f.bn, f.slots, few, grouped, E) <= 160 * 1024;
}

int flow_choose(int mode, int64_t M, int64_t N, int stages, int ncu, double* cost) {
    int best = -1;
    for (int i = 0; i < FLOW_COUNT; ++i) {
        if (!flow_fits(mode, i, stages, false, 0)) continue;
        const FlowTile& f = FLOW_TILES[i];
        const int64_t tiles = ((M + f.bm - 1) / f.bm) * ((N + f.bn - 1) / f.bn), rounds = (tiles + ncu - 1) / ncu;
        const bool dual = mode == MODE_DUAL;
        const double c = (double)rounds * ((dual ? f.round : f.round8) + (dual ? f.stage : f.stage8) * stages) +
                         (dual ? f.share : f.share8) * stages * ((double)tiles / ncu);
        if (best < 0 || c < *cost) {
            best = i;
            *cost = c;
        }
    }
    return best;
}

template <int MODE>
static int launch_mode(const KArgs& a, int tile, hipStream_t st) {
    const int stages = (MODE == MODE_DUAL ? a.K / 2 : a.K) / 128 + (MODE == MODE_DUAL ? (a.K_o * 2 + 127) / 128 : 0);
    const bool few = stages <= FLOW_TILES[tile].lead;
    if (a.off && few) return launch_cfg<MODE, 2, 4, 2, 2, 3, false, true, true>(a, st);
    if (a.off) return launch_cfg<MODE, 2, 4, 2, 2, 3, false, true, false>(a, st);
    if constexpr (MODE == MODE_DUAL)
        if (few) return launch_cfg<MODE, 2, 4, 1, 1, 5, true, false, true>(a, st);
    switch (tile) {
        case 0: return launch_cfg<MODE, 2, 4, 2, 2, 3, false, false, false>(a, st);
        case 1: return launch_cfg<MODE, 4, 2, 1, 3, 3, false, false, false>(a, st);
        case 2: return launch_cfg<MODE, 4, 2, 1, 2, 4, false, false, false>(a, st);  // (a wavefront's 64 columns: whole lines of bf16 results)
        default: return launch_cfg<MODE, 2, 4, 1, 1, 5, true, false, false>(a, st);
    }
}

int launch_flow(const KArgs& a, int mode, int tile, hipStream_t st) {
    note_gemm(GEMM_FLOW, tile);
    if (mode == MODE_DUAL) return launch_mode<MODE_DUAL>(a, tile, st);
    if (mode == MODE_FP8) return launch_mode<MODE_FP8>(a, tile, st);
    return launch_mode<MODE_MX8>(a, tile, st);
}

}  // namespace osc
