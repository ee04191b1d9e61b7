// dps_gemm.hip -- the nested linear on the matrix cores (gfx950) for every
// shape between the small-token kernels and the 256 x 256 tile.
//
// gemm4_kernel: FP16 activations, full and fast mode.  The weight tile's
// upper-byte plane (and, in full mode, its residual plane) is staged in LDS
// as bytes and merged into FP16 operands in registers right before
// v_mfma_f32_16x16x32_f16 (Sec. IV-C: reconstruction during computation);
// fast mode feeds zero residual bytes through the same merge.
// gemm3_kernel: fast mode with FP8 activations on 256 x 128 tiles.  The upper
// bytes go to v_mfma_f32_16x16x128_f8f6f4 as they are stored -- E5M2, or E4M3
// whose fast-mode value is E4M3 * 2^-8 -- against E4M3 activations, and the
// row scale (times 2^-8 for E4M3 weights) is applied to the fp32 accumulator.
//
// Both stream their tiles global -> LDS with direct-to-LDS loads through
// rings of stages, one barrier per stage.  Dense calls walk a 1-D grid
// remapped for the 8 XCDs; grouped (MoE) calls map grid.y onto (expert,
// token tile) by scanning the device offsets, so only `experts` blocks at
// most find no work.
#include <type_traits>

#include "dps_gemm_common.h"

namespace dps {

namespace {

// ------------------------------------------------------------------------------
// 256 x 128 LDS-DMA GEMM, fast mode with FP8 activations
// ------------------------------------------------------------------------------
// Block tile 256 weight rows x 128 tokens, eight compute waves (two per SIMD)
// in a 4 x 2 grid of 64 x 64 each.  A stage covers 128 K elements (one
// 16x16x128 MFMA step).  Stages stream global -> LDS by direct-to-LDS loads
// into rings of three slots (144 KiB), one barrier per stage; four more waves
// (one per SIMD) only issue those loads and wait for them: a wave that issues
// vector-memory instructions stalls on them, and the compute waves then keep
// the matrix cores busy instead.  LDS rows hold 16-byte chunks at slot
// chunk ^ swz8(row), so the 16 rows a fragment read touches land in 16
// distinct 16-byte bank groups.  Lane (i, g): A = weight row i and B = token
// row i, bytes 16g .. 16g+15 and 64+16g .. 64+16g+15 of the stage (the MFMA's
// 32-byte K slice of lane group g, permuted alike in both operands).  Reading
// chunks 2g and 2g+1 instead cost ~4 LDS bank-conflict cycles per read (rocprofv3
// SQ_LDS_BANK_CONFLICT) and 3-5% of the prefill time on MI355X.
struct G3 {
    static constexpr int BN = 256, BM = 128;          // block tile
    static constexpr int WN = 4, WM = 2;              // compute waves
    static constexpr int S = 3;                       // ring slots
    static constexpr int BK = 128;                    // bytes (K elements) per row and stage
    static constexpr int W_BYTES = BN * BK;
    static constexpr int X_BYTES = BM * BK;
    static constexpr int X_BASE = W_BYTES * S;        // weight ring, then token ring
    static constexpr int LDS = X_BASE + X_BYTES * S;
    static constexpr int NISS = 4;                    // waves that issue the DMA
    static constexpr int NW = W_BYTES / 1024 / NISS;  // their instructions per stage
    static constexpr int NX = X_BYTES / 1024 / NISS;
    // Iteration t issues tokens, then weights of stage t + S - 1; at the wait
    // for stage t the groups of the later stages may stay outstanding.
    static constexpr int OUTSTANDING = (S - 2) * (NW + NX);
    static constexpr int NT = BN / WN / 16, MT = BM / WM / 16;
    static constexpr int THREADS = (WN * WM + NISS) * 64;
    static_assert(LDS <= 160 * 1024, "LDS");
};

// TAIL (grouped calls): as in the FP16 wide-row GEMM, an expert's last token
// tile may run up to TAIL rows past 128 (block_rows); each compute wave loads the 32-byte K slices of the 16 tail tokens for
// every stage straight from memory into registers and runs them against
// two of its four weight fragments (token half 0 the first two, half 1 the
// last two): 18 MFMAs per stage instead of 16.
template <int ENC, int TAIL>
__global__ __launch_bounds__(G3::THREADS) void gemm3_kernel(GemmArgs a)
{
    using C = G3;
    constexpr int WN = C::WN, WM = C::WM, S = C::S;
    static_assert(TAIL == 0 || TAIL == 16, "one 16-token fragment");
    __shared__ __attribute__((aligned(16))) uint8_t smem[C::LDS];
    lds_u8 *const lds = (lds_u8 *)smem;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15;
    const int lg = lane >> 4;
    const bool dma_wave = wave >= WN * WM;
    const int iss = wave - WN * WM;  // index among the issuing waves

    int64_t e, mrow0, mrow1;
    int64_t mtail1 = 0;  // end of the tail rows (TAIL blocks whose range passes BM)
    int ntile, s;
    if (a.offsets) {
        // grouped: grid.y walks the experts' token tiles, grid.x the weight
        // tiles times the K ranges
        if (!block_rows(a, e, mrow0, mtail1, C::BM, TAIL))
            return;
        mrow1 = mrow0 + C::BM < mtail1 ? mrow0 + C::BM : mtail1;
        ntile = blockIdx.x / a.splits;
        s = blockIdx.x % a.splits;
    } else {
        // 1-D grid remapped for the 8 XCDs: block L runs on XCD L % 8, so XCD
        // x is given the contiguous tile range [x * per_xcd, (x+1) * per_xcd),
        // walked with the token tile fastest.  Blocks sharing a weight tile
        // then run together on one XCD and fetch it into that XCD's L2 once.
        const uint32_t mtiles = (uint32_t)((a.rows + C::BM - 1) / C::BM);
        const uint32_t ntiles = (uint32_t)((a.n + C::BN - 1) / C::BN);
        const uint32_t total = mtiles * ntiles * (uint32_t)a.splits;
        const uint32_t per_xcd = (total + 7) / 8;
        const uint32_t t0 = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
        if (t0 >= total)
            return;
        ntile = (int)((t0 / mtiles) % ntiles);
        s = (int)(t0 / (mtiles * ntiles));
        e = 0;
        mrow0 = (int64_t)(t0 % mtiles) * C::BM;
        mrow1 = mrow0 + C::BM < a.rows ? mrow0 + C::BM : a.rows;
        mtail1 = mrow1;
    }
    const int64_t n0 = (int64_t)ntile * C::BN;
    const int64_t kb0 = (int64_t)s * a.ksplit;
    const int64_t ke = kb0 + a.ksplit < a.k ? kb0 + a.ksplit : a.k;
    const int klen = (int)(ke - kb0);
    const int ntk = (klen + C::BK - 1) / C::BK;
    // stages entirely inside the K range, whose loads take 32-bit row offsets
    const int t_full = a.k <= kMaxOffsetK ? klen / C::BK : 0;

    // Tail rows: lane (i, g) of a compute wave reads bytes 16g .. 16g+15 and
    // 64+16g .. 64+16g+15 of each stage of token mrow0 + 128 + i (the slice
    // its MFMA operand takes).  K being a multiple of 16, a piece is inside
    // [kb0, ke) whenever it starts there; otherwise the lane reads the row's
    // first 16 bytes of the range and zeroes them.  Lanes past the tail read
    // its last row, whose sums they do not store.
    const bool has_tail = TAIL > 0 && mtail1 > mrow0 + C::BM;
    const uint8_t *xt = static_cast<const uint8_t *>(a.x);
    if (has_tail) {
        int64_t m = mrow0 + C::BM + li;
        m = m < mtail1 ? m : mtail1 - 1;
        xt += m * a.k + kb0;
    }

    // ---- DMA sources: buffer loads with a scalar stage offset ---------------------
    // instruction jj of an issuing wave covers rows 8j .. 8j+7 of its operand
    // tile (j = its instructions per stage times iss, plus jj): lane -> row
    // 8j + lane/8, slot lane%8.  Rows past the operand's end lie beyond its
    // resource; what they leave in LDS is never stored.
    constexpr int NW = C::NW, NX = C::NX;
    const int wr0 = dma_wave ? 8 * NW * iss : 0, xr0 = dma_wave ? 8 * NX * iss : 0;
    const int64_t wrow0 = n0 + wr0 < a.n ? n0 + wr0 : a.n - 1;
    const int64_t xrow0 = mrow0 + xr0 < mrow1 ? mrow0 + xr0 : mrow1 - 1;
    const rsrc_t wr = make_rsrc(a.hi + (e * a.n + wrow0) * a.k + kb0, (a.n - wrow0) * a.k - kb0);
    const rsrc_t xr = make_rsrc(static_cast<const uint8_t *>(a.x) + xrow0 * a.k + kb0,
                                (mrow1 - xrow0) * a.k - kb0);
    const uint32_t step = (uint32_t)(8 * a.k);  // eight rows on
    uint32_t off[2];  // instructions of even and odd j
#pragma unroll
    for (int par = 0; par < 2; ++par)
        off[par] = (uint32_t)((lane >> 3) * a.k +
                              ((lane & 7) ^ swz8(8 * par + (lane >> 3))) * 16);
    static_assert(NW % 2 == 0 && NX % 2 == 0, "instruction parity");
    auto issue_op = [&](auto n_c, const rsrc_t &r, const uint8_t *base, int64_t row0, int64_t row1,
                        int tr, lds_u8 *dst) {
        constexpr int N = decltype(n_c)::value;
        if (tr < t_full) {
#pragma unroll
            for (int jj = 0; jj < N; ++jj)
                buffer_load_lds(r, dst + jj * 1024, 16, off[jj & 1] + jj * step, tr * C::BK, 0, 0);
        } else {
            const int ln = lane_again();
#pragma unroll
            for (int jj = 0; jj < N; ++jj) {
                const int rr = 8 * jj + (ln >> 3);
                const int kk = tr * C::BK + ((ln & 7) ^ swz8(rr)) * 16;
                const bool ok = row0 + rr < row1 && kk < klen;
                const uint8_t *src = base + (row0 + rr) * a.k + kb0 + kk;
                dma16_at<AUX_CACHED>(ok ? (const void *)src : (const void *)g_zero16,
                                     dst + jj * 1024);
            }
            rare_path_end();
        }
    };
    auto issue_w = [&](int t, int slot) {
        if (t < ntk)
            issue_op(std::integral_constant<int, NW>{}, wr, a.hi + e * a.n * a.k, n0 + wr0, a.n, t,
                     lds + slot * C::W_BYTES + NW * 1024 * iss);
    };
    auto issue_x = [&](int t, int slot) {
        if (t < ntk)
            issue_op(std::integral_constant<int, NX>{}, xr, static_cast<const uint8_t *>(a.x),
                     mrow0 + xr0, mrow1, t, lds + C::X_BASE + slot * C::X_BYTES + NX * 1024 * iss);
    };
    // Iteration t fills the slots that stage t - 1 has left.
    int is = S - 1;  // the slot of stage t + S - 1
    auto issue = [&](int t) {
        issue_x(t + S - 1, is);
        issue_w(t + S - 1, is);
        is = is + 1 < S ? is + 1 : 0;
    };
    auto wait = [&](int t) {  // tokens t and weights t have landed
        if (t + S - 1 <= ntk)
            DPS_WAIT_VMCNT(C::OUTSTANDING);
        else
            DPS_WAIT_VMCNT(0);
    };

    const int wn = wave % WN;
    const int wm = wave / WN;
    f32x4 acc[C::NT][C::MT];
#pragma unroll
    for (int i = 0; i < C::NT; ++i)
#pragma unroll
        for (int j = 0; j < C::MT; ++j)
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (dma_wave) {
        // the DMA waves' own loop keeps their state out of the compute waves'
        // registers (and the accumulators out of theirs)
#pragma unroll 1
        for (int u = 0; u < S - 1; ++u) {
            issue_x(u, u);
            issue_w(u, u);
        }
        for (int t = 0; t < ntk; ++t) {
            wait(t);
            stage_barrier();
            issue(t);
        }
        DPS_WAIT_VMCNT(0);  // no DMA may still target this block's LDS when it exits
        return;
    }
    f32x4 tacc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    const int wmu = __builtin_amdgcn_readfirstlane(wm);  // token half, wave-uniform
    // one stage of a compute wave (tail_c: std::true_type in blocks with tail rows)
    // slots of the stage being multiplied (equal, but kept apart: with one counter
    // the compiler reads fragments in another order, 1-2% slower)
    int cws = 0, cxs = 0;
    auto stage = [&](int t, auto tail_c) {
        constexpr bool TL = decltype(tail_c)::value;
        stage_barrier();
        u32x4 tp = {0u, 0u, 0u, 0u}, tq = {0u, 0u, 0u, 0u};
        if constexpr (TL) {
            const int toff = t * C::BK + 16 * lg;
            const bool ok = toff < klen;
            const uint32_t msk = 0u - (uint32_t)ok;
            const uint8_t *pp = xt + (ok ? toff : 0);
            tp = load16(pp) & u32x4{msk, msk, msk, msk};
            tq = load16(pp + (ok ? 64 : 0)) & u32x4{msk, msk, msk, msk};
        }
        const uint8_t *st = smem + cws * C::W_BYTES;
        const uint8_t *xs = smem + C::X_BASE + cxs * C::X_BYTES;
        cws = cws + 1 < S ? cws + 1 : 0;
        cxs = cxs + 1 < S ? cxs + 1 : 0;
        i32x8 av[C::NT];
#pragma unroll
        for (int nt = 0; nt < C::NT; ++nt) {
            const int r = wn * 64 + nt * 16 + li;
            const uint8_t *row = st + r * C::BK;
            const int sw = swz8(r);
            const u32x4 p = *reinterpret_cast<const u32x4 *>(row + ((lg ^ sw) << 4));
            const u32x4 q = *reinterpret_cast<const u32x4 *>(row + (((4 + lg) ^ sw) << 4));
            av[nt] = i32x8{(int)p.x, (int)p.y, (int)p.z, (int)p.w,
                           (int)q.x, (int)q.y, (int)q.z, (int)q.w};
        }
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt) {
            const int r = wm * 64 + mt * 16 + li;
            const uint8_t *row = xs + r * C::BK;
            const int sw = swz8(r);
            const u32x4 p = *reinterpret_cast<const u32x4 *>(row + ((lg ^ sw) << 4));
            const u32x4 q = *reinterpret_cast<const u32x4 *>(row + (((4 + lg) ^ sw) << 4));
            const i32x8 bv = {(int)p.x, (int)p.y, (int)p.z, (int)p.w,
                              (int)q.x, (int)q.y, (int)q.z, (int)q.w};
#pragma unroll
            for (int nt = 0; nt < C::NT; ++nt)
                acc[nt][mt] = mfma16x16x128_fp8<ENC>(av[nt], bv, acc[nt][mt]);
        }
        if constexpr (TL) {
            const i32x8 tb = {(int)tp.x, (int)tp.y, (int)tp.z, (int)tp.w,
                              (int)tq.x, (int)tq.y, (int)tq.z, (int)tq.w};
            if (wmu == 0) {
                tacc[0] = mfma16x16x128_fp8<ENC>(av[0], tb, tacc[0]);
                tacc[1] = mfma16x16x128_fp8<ENC>(av[1], tb, tacc[1]);
            } else {
                tacc[0] = mfma16x16x128_fp8<ENC>(av[2], tb, tacc[0]);
                tacc[1] = mfma16x16x128_fp8<ENC>(av[3], tb, tacc[1]);
            }
        }
    };
    if (has_tail) {
        for (int t = 0; t < ntk; ++t)
            stage(t, std::integral_constant<bool, (TAIL > 0)>{});
    } else {
        for (int t = 0; t < ntk; ++t)
            stage(t, std::false_type{});
    }
    DPS_WAIT_VMCNT(0);  // no DMA may still target this block's LDS when it exits

    // E4M3 weights carry the fast-mode factor 2^-8 (exact in fp32)
    constexpr float wscale = ENC == ENC_E4M3 ? 0.00390625f : 1.f;
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) {
        const int64_t m = mrow0 + wm * 64 + mt * 16 + li;
        const float sc = m < mrow1 ? a.scale[m] * wscale : 0.f;
#pragma unroll
        for (int nt = 0; nt < C::NT; ++nt)
            store_tile_out(a, s, m, n0 + wn * 64 + nt * 16 + lg * 4, acc[nt][mt] * sc,
                           mrow1);
    }
    if (TAIL > 0 && has_tail) {
        const int64_t m = mrow0 + C::BM + li;
        const float sc = m < mtail1 ? a.scale[m] * wscale : 0.f;
#pragma unroll
        for (int j = 0; j < 2; ++j)
            store_tile_out(a, s, m, n0 + wn * 64 + (2 * wmu + j) * 16 + lg * 4,
                           tacc[j] * sc, mtail1);
    }
}

// ------------------------------------------------------------------------------
// Wide-row LDS-DMA GEMM, FP16 full/fast: 128 weight rows, 128-element stages
// ------------------------------------------------------------------------------
// On gfx950 an LDS-DMA (or plain) load instruction runs at about half speed
// when each row it touches gets 64 contiguous bytes instead of >= 128 (MI355X,
// L2-resident data: 26 vs 50 B/clk per CU; from HBM 4.4 vs 5.2-7.2 TB/s), so
// a stage here spans 128 K elements: weight planes arrive as 8 rows x 128 B
// per instruction and tokens as 4 rows x 256 B.  LDS keeps the rows, 16-byte
// chunks placed at slot chunk ^ swz(row), and fragment reads are single
// ds_read_b128 in patterns measured conflict-free:
//   weight plane, 128-byte rows, swz8(r) = (r >> 1) & 7: lane (i, g) of
//     K-half q reads chunk 4q + g of row i, K 64q+16g .. +15, which feeds two
//     MFMA steps s (bytes 8s .. 8s+7, merged into FP16 in registers);
//   tokens, 256-byte rows, swz16(r) = r & 15: step (q, s) of lane (i, g)
//     reads chunk 8q + 2g + s of token i, K 64q+16g+8s .. +7.
// Both operands of every MFMA pair the same K elements.  Eight waves: waves
// 0-3 take K-half 0 of every stage and waves 4-7 K-half 1, each over a
// 64 x BM/2 quarter of the tile (two waves per SIMD); the halves are summed
// through LDS at the end, in a fixed order.  The token tile BM (32, 64 or
// 128) follows the call's token count, so short calls stage no padding rows.
//
// SPEC adds four DMA waves (one per SIMD) that do nothing but issue the
// direct-to-LDS loads and wait for them; the eight compute waves then never
// stall on address-unit slots and keep the matrix cores fed, and a stage costs
// about max(DMA, MFMA) instead of their sum.  Both kinds of wave meet at the
// one barrier per stage.
//
// Weights and tokens stream through separate LDS rings of WS and XS slots
// (XS <= WS).  Iteration t issues tokens of stage t+XS-1, then weights of
// stage t+WS-1.  The vector-memory counter retires in issue order, so waiting
// until only the instructions issued after the later of tokens t and weights
// t are outstanding (G4::OUTSTANDING) retires exactly those two, and the later
// stages stay in flight across the barrier.
template <int MODE, int BM, int WS, int XS, int NISS>
struct G4 {
    static constexpr int PLANES = MODE == MODE_FULL ? 2 : 1;
    static constexpr int BK = 128;
    static constexpr int MT = BM / 32;              // 16-token tiles per wave
    static constexpr int W_BYTES = 128 * BK;        // one plane, 128 rows
    static constexpr int W_SLOT = W_BYTES * PLANES;
    static constexpr int X_SLOT = BM * BK * 2;      // BM tokens, FP16
    static constexpr int X_BASE = W_SLOT * WS;
    static constexpr int LDS = X_BASE + XS * X_SLOT;
    static constexpr int W_INSTR = W_BYTES / 1024 / NISS;  // per issuing wave per plane
    static constexpr int X_INSTR = X_SLOT / 1024 / NISS;
    static constexpr int NW = W_INSTR * PLANES;  // weight instructions per issuing wave per stage
    static constexpr int NX = X_INSTR;
    // Instructions that may stay outstanding at the wait for stage t: those
    // issued after the later of tokens t and weights t.  With XS < WS that is
    // tokens t, followed in its iteration by one weight group; with XS == WS
    // both go out in the same iteration and weights t come last.
    static constexpr int OUTSTANDING = (XS < WS ? NW : 0) + (XS - 2) * (NX + NW);
    static_assert(WS >= 3 && XS >= 2 && XS <= WS, "ring depths of the counter scheme");
    static_assert(OUTSTANDING <= 63, "vmcnt range");
    static_assert(BM == 32 || BM == 64 || BM == 128, "token tile");
    static_assert(X_INSTR >= 1 && W_INSTR >= 1, "DMA split over the issuing waves");
    static_assert(LDS <= 160 * 1024 && LDS >= 4 * 16384, "LDS (the K-half reduction needs 64 KiB)");
};

__device__ __forceinline__ int swz16(int r) { return r & 15; }

// TAIL (grouped calls, 128-token tiles with DMA waves): the block's token
// range may run up to TAIL rows past its 128-token tile (block_rows).  Those
// rows take no LDS: each compute wave loads its K-half of their 16-token
// fragment straight from memory into registers after the stage barrier (the
// tokens of a call are a few MiB and sit in L2) and runs it against the
// weight fragments it already holds, waves of token half 0 on the first two
// 16-row weight sub-tiles of their quarter and waves of half 1 on the other
// two, so every compute wave does 36 MFMAs per stage instead of 32.  The
// tail's K-half sums go through LDS with the others.
template <int MODE, int ENC, int BM, int WS, int XS, bool SPEC, int AUX, int TAIL = 0>
__global__ __launch_bounds__(SPEC ? 768 : 512) void gemm4_kernel(GemmArgs a)
{
    using C = G4<MODE, BM, WS, XS, SPEC ? 4 : 8>;
    static_assert(TAIL == 0 || (TAIL == 16 && SPEC && BM == 128), "tail rows: 128-token DMA-wave tile");
    __shared__ __attribute__((aligned(16))) uint8_t smem[C::LDS];
    lds_u8 *const lds = (lds_u8 *)smem;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15;
    const int lg = lane >> 4;
    const bool dma_wave = SPEC && wave >= 8;
    const int issuer = SPEC ? wave - 8 : wave;  // index among the waves that issue DMA
    const int kh = (wave >> 2) & 1;  // K-half of every stage (compute waves)
    const int wn = (wave >> 1) & 1;  // 64-row quarter
    const int wm = wave & 1;         // BM/2-token half

    int64_t e, mrow0, mrow1;
    int64_t mtail1 = 0;  // end of the tail rows (TAIL blocks whose range passes BM)
    int ntile, s;
    if (a.offsets) {
        if (!block_rows(a, e, mrow0, mtail1, BM, TAIL))
            return;
        mrow1 = mrow0 + BM < mtail1 ? mrow0 + BM : mtail1;
        ntile = blockIdx.x / a.splits;
        s = blockIdx.x % a.splits;
    } else {
        // 1-D grid remapped for the 8 XCDs (block L runs on XCD L % 8): XCD x
        // takes the tile range [x * per_xcd, (x+1) * per_xcd).  Tiles are
        // walked in groups of four weight tiles: token tile, then weight tile
        // within the group, so the ~32 blocks resident on an XCD cover about
        // 4 weight tiles x 8 token tiles and both operands are re-read from
        // that XCD's L2 rather than from HBM.
        // (Tile counts fit 32 bits: the grid does.)
        const uint32_t mtiles = (uint32_t)((a.rows + BM - 1) / BM);
        const uint32_t ntiles = (uint32_t)((a.n + 127) / 128);
        const uint32_t total = mtiles * ntiles * (uint32_t)a.splits;
        const uint32_t per_xcd = (total + 7) / 8;
        const uint32_t t = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
        if (t >= total)
            return;
        constexpr uint32_t G = 4;
        s = (int)(t / (mtiles * ntiles));
        const uint32_t r = t % (mtiles * ntiles);
        const uint32_t chunk = r / (G * mtiles);
        const uint32_t within = r % (G * mtiles);
        const uint32_t gc = ntiles - chunk * G < G ? ntiles - chunk * G : G;
        ntile = (int)(chunk * G + within % gc);
        e = 0;
        mrow0 = (int64_t)(within / gc) * BM;
        mrow1 = mrow0 + BM < a.rows ? mrow0 + BM : a.rows;
        mtail1 = mrow1;
    }
    const int64_t n0 = (int64_t)ntile * 128;
    const int64_t kb0 = (int64_t)s * a.ksplit;
    const int64_t ke = kb0 + a.ksplit < a.k ? kb0 + a.ksplit : a.k;
    const int klen = (int)(ke - kb0);
    const int ntk = (klen + C::BK - 1) / C::BK;
    // stages entirely inside the K range, whose loads take 32-bit row offsets
    const int t_full = a.k <= kMaxOffsetK ? klen / C::BK : 0;
    // Iteration t stages K range tk(t).  With rows a multiple of 4 KiB apart,
    // blocks walking their K ranges in step would all touch the same 128-byte
    // column (address bits 7-11) at once; each group of four weight tiles
    // starts at another stage instead.  Token tiles of one weight tile keep
    // the same order, so they still meet in L2.  (MI355X, gate+up 28672 x
    // 4096 in full mode: 0.78x the time at 32 tokens, 0.83x at 128, 0.91x at
    // 256; the other hidden-4096 layers within 3%.)
    const int grot = a.rotate ? (int)((uint32_t)(ntile >> 2) % (uint32_t)ntk) : 0;
    auto tk = [&](int t) { return t + grot < ntk ? t + grot : t + grot - ntk; };

    // Tail rows: lane (i, g) of a compute wave loads 32 bytes of token
    // mrow0 + BM + i per stage, K 64 kh + 16 g .. +15 (its two MFMA steps).
    // K being a multiple of 16, such a piece lies inside [kb0, ke) whenever
    // it starts there (stage offset below xtlim); otherwise the lane reads the
    // row's first 16 elements of the range and zeroes them.  Lanes past the
    // tail read its last row, whose sums they do not store.
    const bool has_tail = TAIL > 0 && mtail1 > mrow0 + BM;
    const uint16_t *xt = static_cast<const uint16_t *>(a.x);
    const int xtk = 64 * kh + 16 * lg;
    int xtlim = 0;
    if (has_tail) {
        int64_t m = mrow0 + BM + li;
        m = m < mtail1 ? m : mtail1 - 1;
        xt += m * a.k + kb0;
        xtlim = (int)(ke - kb0 - xtk);
    }
    const int wmu = __builtin_amdgcn_readfirstlane(wm);  // token half, wave-uniform

    // ---- DMA sources ---------------------------------------------------------
    // A wave that issues loads is paced by what each costs it to issue, so a
    // load takes a scalar stage offset (buffer loads of the upper bytes and
    // tokens) or one 64-bit add (residual bytes); stages cut by the K range's
    // end and rows that cross residual chunks go through branches of their own.
    // token instruction jj: rows 4j .. 4j+3 (j = X_INSTR issuer + jj), lane ->
    // row 4j + lane/16, slot lane%16
    constexpr int NP = C::W_INSTR, NX = C::X_INSTR;
    const bool issues = !SPEC || dma_wave;  // compute waves of a SPEC block keep no DMA state
    const int xr0 = 4 * NX * issuer;
    const int64_t xrow0 = issues && mrow0 + xr0 < mrow1 ? mrow0 + xr0 : mrow1 - 1;
    const rsrc_t xr = make_rsrc(static_cast<const uint16_t *>(a.x) + xrow0 * a.k + kb0,
                                ((mrow1 - xrow0) * a.k - kb0) * 2);
    uint32_t xoff[NX];
#pragma unroll
    for (int jj = 0; jj < NX; ++jj) {
        const int r = 4 * jj + (lane >> 4);
        xoff[jj] = (uint32_t)(r * a.k + ((lane & 15) ^ swz16(xr0 + r)) * 8) * 2u;
    }
    auto issue_x = [&](int tr, int slot) {
        lds_u8 *dst = lds + C::X_BASE + slot * C::X_SLOT + NX * 1024 * issuer;
        if (tr < t_full) {
#pragma unroll
            for (int jj = 0; jj < NX; ++jj)
                buffer_load_lds(xr, dst + jj * 1024, 16, xoff[jj], tr * (C::BK * 2), 0, 0);
        } else {
            const int ln = lane_again();
#pragma unroll
            for (int jj = 0; jj < NX; ++jj) {
                const int r = xr0 + 4 * jj + (ln >> 4);
                const int kk = tr * C::BK + ((ln & 15) ^ swz16(r)) * 8;
                const int64_t m = mrow0 + r;
                const bool ok = m < mrow1 && kk < klen;
                const uint16_t *src = static_cast<const uint16_t *>(a.x) + m * a.k + kb0 + kk;
                dma16_at<AUX_CACHED>(ok ? (const void *)src : (const void *)g_zero16,
                                     dst + jj * 1024);
            }
            rare_path_end();
        }
    };
    // weight instruction jj of a plane: rows 8j .. 8j+7 (j = W_INSTR issuer +
    // jj), lane -> row 8j + lane/8, slot lane%8
    auto w_row = [&](int ln, int jj, int &wel) {
        const int r = 8 * (NP * issuer + jj) + (ln >> 3);
        wel = ((ln & 7) ^ swz8(r)) * 16;
        const int64_t nr = n0 + r;
        return e * a.n + (nr < a.n ? nr : a.n - 1);
    };
    const int wr0 = issues ? 8 * NP * issuer : 0;
    const int64_t wrow0 = e * a.n + (n0 + wr0 < a.n ? n0 + wr0 : a.n - 1);
    const rsrc_t wr = make_rsrc(a.hi + wrow0 * a.k + kb0, 0xFFFFFFFFll);
    uint32_t woff[NP];
#pragma unroll
    for (int jj = 0; jj < NP; ++jj) {
        int wel;
        const int64_t nr = w_row(lane, jj, wel);
        woff[jj] = (uint32_t)((nr > wrow0 ? nr - wrow0 : 0) * a.k + wel);
    }
    // Full mode: the residual piece of instruction jj and stage t is at wp[jj] +
    // 128 t.
    //   W_ONE    for the whole K range
    //   W_TWO    before stage wb[jj]; from there on rd[jj] chunks further (rows of
    //            at most two chunks: K ranges no longer than a chunk)
    //   W_RENEW  in the stages [w_lo, w_hi); looked up anew beyond them (shorter
    //            chunks; slots outside the pool, whose pieces read zeros, stage
    //            by stage)
    // A lookup waits for the slot table and with it for every load this wave
    // has in flight, so the first one comes before all loads and rows that
    // cross chunks must not cost one per crossing (MI355X, 4096 x 4112 in 16
    // KiB chunks, 64 tokens: 26.0 us with lookups at the crossings, 16.2 with
    // both chunks' slots read once).
    enum { W_ONE, W_TWO, W_RENEW };
    const uint8_t *wp[NP];
    int32_t rd[NP];
    int wb[NP];
    int wmode = W_RENEW, w_lo = 1, w_hi = 0;
    const uint32_t cmask = (1u << a.res.log2c) - 1;
    auto w_first = [&]() __attribute__((always_inline)) {
        const int tr = tk(0);
        int64_t l0[NP];
        int32_t s0[NP], s1[NP];
        bool ok = true, two = false;
        auto slot_of = [&](int64_t c) {
            const bool in = c < a.res.n_chunks;
            ok &= in;
            return a.res.slots[in ? c : 0];
        };
#pragma unroll
        for (int jj = 0; jj < NP; ++jj) {
            int wel;
            l0[jj] = w_row(lane, jj, wel) * a.k + kb0;  // of a piece past a short K range: the row's
            l0[jj] += wel < klen ? wel : 0;
            const int b = (int)((cmask - ((uint32_t)l0[jj] & cmask) + C::BK) >> 7);
            const bool second = (int64_t)b * C::BK + wel < klen;
            wb[jj] = second ? b : ntk;
            two |= second;
            s0[jj] = s1[jj] = slot_of(l0[jj] >> a.res.log2c);
        }
        const bool any_two = __any(two);
        if (any_two) {
#pragma unroll
            for (int jj = 0; jj < NP; ++jj)
                if (wb[jj] < ntk)
                    s1[jj] = slot_of((l0[jj] >> a.res.log2c) + 1);
        }
        w_hi = ntk;
#pragma unroll
        for (int jj = 0; jj < NP; ++jj) {
            ok &= s0[jj] >= 0 && s0[jj] < a.res.n_pool_slots && s1[jj] >= 0 &&
                  s1[jj] < a.res.n_pool_slots;
            rd[jj] = s1[jj] - s0[jj] - 1;
            const bool next = wb[jj] <= tr;
            const int64_t s = s0[jj] + (next ? (int64_t)rd[jj] : 0);
            wp[jj] = a.res.pool + ((s << a.res.log2c) + ((uint32_t)l0[jj] & cmask));
            w_hi = !next && wb[jj] < w_hi ? wb[jj] : w_hi;
        }
        if (__all(ok))
            wmode = any_two ? W_TWO : W_ONE;
        else
            w_hi = 0;
    };
    auto w_renew = [&](int tr) __attribute__((always_inline)) {
        const int ln = lane_again();
        const int64_t off = (int64_t)tr * C::BK;
        w_lo = 0;
        w_hi = ntk;
#pragma unroll
        for (int jj = 0; jj < NP; ++jj) {
            int wel;
            const int64_t l0 = w_row(ln, jj, wel) * a.k + kb0 + wel;
            const bool in = off + wel < klen;
            const int64_t l = l0 + (in ? off : -wel);
            const int64_t o = residual_offset(a.res, l);
            const bool ok = in && o >= 0;
            const uint32_t at = (uint32_t)l & cmask;  // within the chunk
            const int t_in = (klen - wel + C::BK - 1) >> 7;
            const int t_out = tr + (int)((cmask - at + C::BK) >> 7);
            wp[jj] = ok ? a.res.pool + (o - off) : g_zero16 - off;
            const int t0 = ok ? tr - (int)(at >> 7) : tr;
            const int t1 = ok ? (t_out < t_in ? t_out : t_in) : tr + 1;
            w_lo = t0 > w_lo ? t0 : w_lo;
            w_hi = t1 < w_hi ? t1 : w_hi;
        }
        rare_path_end();
    };
    // W_TWO, at stage tr of a forward walk (a rotated one comes back to stage 0
    // from the last, where every piece with a second chunk lies in it)
    auto w_cross = [&](int tr) __attribute__((always_inline)) {
        w_hi = ntk;
#pragma unroll
        for (int jj = 0; jj < NP; ++jj) {
            const int64_t d = (int64_t)rd[jj] << a.res.log2c;
            if (tr == 0)
                wp[jj] -= wb[jj] < ntk ? d : 0;
            else
                wp[jj] += wb[jj] == tr ? d : 0;
            w_hi = wb[jj] > tr && wb[jj] < w_hi ? wb[jj] : w_hi;
        }
    };
    static_assert(C::BK == 128, "stage arithmetic of the residual pointers");
    auto w_update = [&](int tr) __attribute__((always_inline)) {
        if (wmode == W_RENEW) {
            if (__any(tr < w_lo || tr >= w_hi))
                w_renew(tr);
        } else {
            if (wmode == W_TWO && ((tr == 0 && grot > 0) || __any(tr >= w_hi)))
                w_cross(tr);
            if (tr >= t_full) {  // the K range ends inside this stage, the walk's last
                const int ln = lane_again();
                const int64_t off = (int64_t)tr * C::BK;
#pragma unroll
                for (int jj = 0; jj < NP; ++jj) {
                    int wel;
                    w_row(ln, jj, wel);
                    wp[jj] = off + wel < klen ? wp[jj] : g_zero16 - off;
                }
            }
        }
    };
    auto issue_w = [&](int tr, int slot) __attribute__((always_inline)) {
        lds_u8 *dst = lds + slot * C::W_SLOT + NP * 1024 * issuer;
        if (tr < t_full) {
#pragma unroll
            for (int jj = 0; jj < NP; ++jj)
                buffer_load_lds(wr, dst + jj * 1024, 16, woff[jj], tr * C::BK, 0, AUX);
        } else {
            const int ln = lane_again();
#pragma unroll
            for (int jj = 0; jj < NP; ++jj) {
                int wel;
                const int64_t nr = w_row(ln, jj, wel);
                const int kk = tr * C::BK + wel;
                const uint8_t *src = a.hi + nr * a.k + kb0 + kk;
                dma16_at<AUX>(kk < klen ? (const void *)src : (const void *)g_zero16,
                              dst + jj * 1024);
            }
            rare_path_end();
        }
        if (MODE == MODE_FULL) {
            if (wmode != W_ONE || tr >= t_full)
                w_update(tr);
#pragma unroll
            for (int jj = 0; jj < NP; ++jj)
                dma16_at<AUX>(wp[jj] + (int64_t)tr * C::BK, dst + C::W_BYTES + jj * 1024);
        }
    };
    // Iteration t issues tokens of stage t + XS - 1, then weights of stage t +
    // WS - 1, into the slots that stage t - 1 has left.
    int iws = WS - 1, ixs = XS - 1;  // their slots
    auto issue = [&](int t) {
        if (t + XS - 1 < ntk)
            issue_x(tk(t + XS - 1), ixs);
        if (t + WS - 1 < ntk)
            issue_w(tk(t + WS - 1), iws);
        iws = iws + 1 < WS ? iws + 1 : 0;
        ixs = ixs + 1 < XS ? ixs + 1 : 0;
    };
    auto wait = [&](int t) {  // tokens t and weights t have landed
        if (t + WS - 1 <= ntk)
            DPS_WAIT_VMCNT(C::OUTSTANDING);
        else
            DPS_WAIT_VMCNT(0);
    };
    f32x4 acc[4][C::MT];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < C::MT; ++j)
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // fragment read offsets (fixed across stages)
    int aoff[4], boff[C::MT][2];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const int r = wn * 64 + nt * 16 + li;
        aoff[nt] = r * 128 + (((4 * kh + lg) ^ swz8(r)) << 4);
    }
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) {
        const int r = wm * (BM / 2) + mt * 16 + li;
#pragma unroll
        for (int sidx = 0; sidx < 2; ++sidx)
            boff[mt][sidx] = r * 256 + (((8 * kh + 2 * lg + sidx) ^ swz16(r)) << 4);
    }

    f32x4 tacc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};

    // one stage of matrix work on the slots of stage t (tail_c: std::true_type
    // in blocks with tail rows)
    int cws = 0, cxs = 0;  // slots of the stage being multiplied
    auto compute = [&](int t, auto tail_c) {
        constexpr bool TL = decltype(tail_c)::value;
        const uint8_t *st = smem + cws * C::W_SLOT;
        const uint8_t *xs = smem + C::X_BASE + cxs * C::X_SLOT;
        cws = cws + 1 < WS ? cws + 1 : 0;
        cxs = cxs + 1 < XS ? cxs + 1 : 0;
        u32x4 tx0 = {0u, 0u, 0u, 0u}, tx1 = {0u, 0u, 0u, 0u};
        if constexpr (TL) {
            const int off = tk(t) * C::BK;
            const bool ok = off < xtlim;
            const uint32_t msk = 0u - (uint32_t)ok;
            const uint16_t *p = xt + (ok ? off + xtk : 0);
            tx0 = load16(p) & u32x4{msk, msk, msk, msk};
            tx1 = load16(p + 8) & u32x4{msk, msk, msk, msk};
        }
        u32x4 hv[4], lv[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            hv[nt] = *reinterpret_cast<const u32x4 *>(st + aoff[nt]);
            lv[nt] = u32x4{0u, 0u, 0u, 0u};
            if (MODE == MODE_FULL)
                lv[nt] = *reinterpret_cast<const u32x4 *>(st + C::W_BYTES + aoff[nt]);
        }
        // without DMA waves, this wave issues its share of the next stages'
        // DMA here, after its fragment reads (their latency overlaps the issue)
        if (!SPEC)
            issue(t);
        half8 a0[4], a1[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            a0[nt] = weight8<MODE, ENC>(hv[nt].x, hv[nt].y, lv[nt].x, lv[nt].y);
            a1[nt] = weight8<MODE, ENC>(hv[nt].z, hv[nt].w, lv[nt].z, lv[nt].w);
        }
#pragma unroll
        for (int sidx = 0; sidx < 2; ++sidx) {
#pragma unroll
            for (int mt = 0; mt < C::MT; ++mt) {
                const half8 bv = as_half8(*reinterpret_cast<const u32x4 *>(xs + boff[mt][sidx]));
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    acc[nt][mt] = mfma16x16x32(sidx ? a1[nt] : a0[nt], bv, acc[nt][mt]);
            }
        }
        if constexpr (TL) {
            const half8 b0 = as_half8(tx0), b1 = as_half8(tx1);
            if (wmu == 0) {
                tacc[0] = mfma16x16x32(a0[0], b0, tacc[0]);
                tacc[1] = mfma16x16x32(a0[1], b0, tacc[1]);
                tacc[0] = mfma16x16x32(a1[0], b1, tacc[0]);
                tacc[1] = mfma16x16x32(a1[1], b1, tacc[1]);
            } else {
                tacc[0] = mfma16x16x32(a0[2], b0, tacc[0]);
                tacc[1] = mfma16x16x32(a0[3], b0, tacc[1]);
                tacc[0] = mfma16x16x32(a1[2], b1, tacc[0]);
                tacc[1] = mfma16x16x32(a1[3], b1, tacc[1]);
            }
        }
    };

    // the steady-state issue of iterations -(WS-1) .. -1, keeping only stages
    // >= 0, so the counter arithmetic holds from iteration 0
    auto prologue = [&]() __attribute__((always_inline)) {
        if (MODE == MODE_FULL && a.range)
            w_first();
#pragma unroll 1
        for (int u = -(WS - 1); u < 0; ++u) {
            if (u + XS - 1 >= 0 && u + XS - 1 < ntk)
                issue_x(tk(u + XS - 1), u + XS - 1);
            if (u + WS - 1 < ntk)
                issue_w(tk(u + WS - 1), u + WS - 1);
        }
    };
    if (!SPEC) {
        prologue();
        for (int t = 0; t < ntk; ++t) {
            wait(t);
            stage_barrier();
            compute(t, std::false_type{});
        }
    } else if (dma_wave) {
        // separate loops per role keep the DMA state out of the compute waves'
        // registers and the accumulators out of the DMA waves'
        prologue();
        for (int t = 0; t < ntk; ++t) {
            wait(t);
            stage_barrier();
            issue(t);
        }
        DPS_WAIT_VMCNT(0);  // no DMA may still target this block's LDS
        __syncthreads();    // matches the compute waves' two barriers below
        __syncthreads();
        return;
    } else if (has_tail) {
        for (int t = 0; t < ntk; ++t) {
            stage_barrier();
            compute(t, std::integral_constant<bool, (TAIL > 0)>{});
        }
    } else {
        for (int t = 0; t < ntk; ++t) {
            stage_barrier();
            compute(t, std::false_type{});
        }
    }
    DPS_WAIT_VMCNT(0);  // no DMA may still target this block's LDS
    __syncthreads();    // every wave is done reading the stages

    // Each K half hands two of its four row tiles to the other through LDS (4
    // KB per tile), so both halves add and store; every sum is half 0 plus
    // half 1.  The tail's sums go to half 0.
    constexpr int RED = 4 * C::MT + (TAIL > 0 ? 2 : 0);  // 16 x 16 tiles per wave
    static_assert(4 * RED * 64 * 16 <= C::LDS, "K-half reduction area");
    f32x4 *red = reinterpret_cast<f32x4 *>(smem) + (wave & 3) * (RED * 64);
    const int khu = __builtin_amdgcn_readfirstlane(kh);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
        if ((nt >> 1) != khu)
#pragma unroll
            for (int mt = 0; mt < C::MT; ++mt)
                red[(nt * C::MT + mt) * 64 + lane] = acc[nt][mt];
    if (TAIL > 0 && has_tail && khu == 1) {
        red[(4 * C::MT) * 64 + lane] = tacc[0];
        red[(4 * C::MT + 1) * 64 + lane] = tacc[1];
    }
    __syncthreads();
    const int64_t m = mrow0 + wm * (BM / 2) + li;
    const int64_t n = n0 + wn * 64 + lg * 4;
    // a tile inside the output stores without per-element checks
    const bool whole = mrow0 + BM == mrow1 && n0 + 128 <= a.n && (a.n & 3) == 0;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        if ((nt >> 1) != khu)
            continue;
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt) {
            const f32x4 o = red[(nt * C::MT + mt) * 64 + lane];
            const f32x4 v = acc[nt][mt] + o;
            if (whole && a.splits == 1)
                store_half4(a.y + (m + 16 * mt) * a.n + n + 16 * nt, v);
            else if (whole)
                *reinterpret_cast<f32x4 *>(a.partial + ((int64_t)s * a.rows + m + 16 * mt) * a.n +
                                           n + 16 * nt) = v;
            else
                store_tile_out(a, s, m + 16 * mt, n + 16 * nt, v, mrow1);
        }
    }
    if (TAIL > 0 && has_tail && khu == 0) {
        const int64_t mt = mrow0 + BM + li;
#pragma unroll
        for (int j = 0; j < 2; ++j)
            store_tile_out(a, s, mt, n0 + wn * 64 + (2 * wmu + j) * 16 + lg * 4,
                           tacc[j] + red[(4 * C::MT + j) * 64 + lane], mtail1);
    }
}

int64_t token_tiles(int64_t rows, int64_t experts, bool grouped, int bm)
{
    return grouped ? (rows + bm - 1) / bm + experts : (rows + bm - 1) / bm;
}

}  // namespace

int gemm_rows_per_block(int variant)
{
    return (variant == GEMM_G3_256x256 || variant == GEMM_G3_256x128 ||
            variant == GEMM_G5_256x256)
               ? 256
               : 128;
}
int gemm_tokens_per_block(int variant)
{
    switch (variant) {
    case GEMM_G3_256x256: return 256;
    case GEMM_G5_256x256: return 256;
    case GEMM_G4S_128x64: return 64;
    case GEMM_G4_128x32: return 32;
    default: return 128;
    }
}

namespace {

template <int ENC>
hipError_t launch_g3(const GemmArgs &a, const LinearPlan &plan, hipStream_t stream)
{
    if (plan.variant != GEMM_G3_256x128)
        return hipErrorInvalidValue;
    const int64_t nt = (a.n + G3::BN - 1) / G3::BN;
    // grouped calls take up to 16 tail rows per expert
    if (a.offsets) {
        const dim3 grid((unsigned)(nt * plan.splits),
                        (unsigned)token_tiles(a.rows, a.experts, true, G3::BM), 1);
        hipLaunchKernelGGL((gemm3_kernel<ENC, 16>), grid, dim3(G3::THREADS), 0, stream, a);
    } else {
        const dim3 grid = dense_grid(nt * plan.splits * token_tiles(a.rows, 1, false, G3::BM));
        hipLaunchKernelGGL((gemm3_kernel<ENC, 0>), grid, dim3(G3::THREADS), 0, stream, a);
    }
    return hipGetLastError();
}

template <int MODE, int ENC, int BM, int WS, int XS, bool SPEC, int TL, int AUX>
hipError_t launch_g4_aux(const GemmArgs &a, const LinearPlan &plan, bool grouped,
                         hipStream_t stream)
{
    const int64_t nt = (a.n + 127) / 128;
    const dim3 grid = grouped ? dim3((unsigned)(nt * plan.splits),
                                     (unsigned)token_tiles(a.rows, a.experts, true, BM), 1)
                              : dense_grid(nt * plan.splits * token_tiles(a.rows, 1, false, BM));
    const dim3 block(SPEC ? 768 : 512);
    if (TL > 0 && grouped)
        hipLaunchKernelGGL((gemm4_kernel<MODE, ENC, BM, WS, XS, SPEC, AUX, TL>), grid, block, 0,
                           stream, a);
    else
        hipLaunchKernelGGL((gemm4_kernel<MODE, ENC, BM, WS, XS, SPEC, AUX>), grid, block, 0,
                           stream, a);
    return hipGetLastError();
}

// Whether a call loads its weights nontemporally.  MI355X, time with cached
// loads over time with nontemporal ones, a rotation of layers of 640 MiB in all
// / one layer called over and over:
//   - not where a row is not whole 128-byte lines: a stage's piece then shares
//     its lines with the next stage's, which fetches them again (28672 x 4112
//     0.81-0.93 / 0.54-0.76, 16 experts of 3072 x 4112 - / 0.71-0.84);
//   - not where several token tiles read the weights again a chip's round or more
//     later: 300 to 1024 tokens - / 0.81-1.00, 8 experts of 36-60 rows on 32-token
//     tiles 0.94-1.01 / 0.79-0.93.  Grouped calls count as one tile per expert up
//     to 7/8 of its rows on average (1.01-1.13 below, 0.94-1.01 at 60 of 64), with
//     tail rows up to all of them (130 of 128 + 16: 1.00-1.06).  The two tiles
//     of up to 256 dense tokens run side by side: alone 0.90-1.07 / 0.81-0.98, but a pass
//     over the hidden-4096 set at 256 tokens, 16 sets in turn, gains 1.02 full
//     and 1.01 fast, as what the smaller layers keep in the cache is not lost;
//   - from kStreamBytes on.  33-64 tokens 0.96-1.14 / 0.77-1.04.  65-128 tokens
//     0.99-1.09 / 0.85-0.98 from 80 MiB, 0.90-0.97 / 0.85-0.98 below (4096 x
//     14336 in fast mode at 128 tokens 28.3 against 26.6 us alone), where what
//     the smaller layers keep decides again: the pass at 128 tokens in fast
//     mode 95.8 us, 99.3 with a line at 80 MiB, 16 sets in turn 102.9 and 103.0.
template <int MODE, int BM, int TL>
bool streams(const GemmArgs &a, bool grouped)
{
    const bool full = MODE == MODE_FULL;
    const bool lines = a.k % 128 == 0 && (uintptr_t)a.hi % 128 == 0 &&
                       (!full || ((uintptr_t)a.res.pool % 128 == 0 && a.res.log2c >= 7));
    const bool once = grouped ? a.rows <= a.experts * (TL > 0 ? BM + TL : BM * 7 / 8)
                              : a.rows <= 256;
    return lines && once && a.experts * a.n * a.k * (full ? 2 : 1) >= kStreamBytes;
}

template <int MODE, int ENC, int BM, int WS, int XS, bool SPEC>
hipError_t launch_g4(const GemmArgs &a, const LinearPlan &plan, bool grouped, hipStream_t stream)
{
    // Grouped calls on the 128-token tile with DMA waves take up to 16 tail rows
    // per expert into its last tile (gemm4_kernel, block_rows): an expert of
    // 129-144 rows reads its weights once, not twice.  Every mode and encoding
    // fits the tail's 16 registers within the 168 that three waves per SIMD allow.
    constexpr int TL = SPEC && BM == 128 ? 16 : 0;
    return streams<MODE, BM, TL>(a, grouped)
               ? launch_g4_aux<MODE, ENC, BM, WS, XS, SPEC, TL, AUX_STREAM>(a, plan, grouped,
                                                                            stream)
               : launch_g4_aux<MODE, ENC, BM, WS, XS, SPEC, TL, AUX_CACHED>(a, plan, grouped,
                                                                            stream);
}

// (token tile, weight slots, token slots) per mode, each within 160 KiB:
// weights want depth (HBM), tokens at least a second slot ahead where it fits
template <int MODE, int ENC>
hipError_t launch_g4_variant(const GemmArgs &a, const LinearPlan &plan, bool grouped,
                             hipStream_t stream)
{
    if constexpr (MODE == MODE_FULL) {
        switch (plan.variant) {
        case GEMM_G4_128x32: return launch_g4<MODE, ENC, 32, 4, 4, false>(a, plan, grouped, stream);
        case GEMM_G4S_128x128: return launch_g4<MODE, ENC, 128, 3, 2, true>(a, plan, grouped, stream);
        case GEMM_G4S_128x64: return launch_g4<MODE, ENC, 64, 4, 2, true>(a, plan, grouped, stream);
        default: return hipErrorInvalidValue;
        }
    } else {
        switch (plan.variant) {
        case GEMM_G4_128x32: return launch_g4<MODE, ENC, 32, 8, 4, false>(a, plan, grouped, stream);
        case GEMM_G4S_128x128: return launch_g4<MODE, ENC, 128, 4, 3, true>(a, plan, grouped, stream);
        case GEMM_G4S_128x64: return launch_g4<MODE, ENC, 64, 6, 4, true>(a, plan, grouped, stream);
        default: return hipErrorInvalidValue;
        }
    }
}

}  // namespace

hipError_t launch_gemm_f16(const LinearProblem &p, const LinearPlan &plan, float *partial,
                           hipStream_t stream)
{
    GemmArgs a;
    a.x = p.x;
    a.offsets = p.offsets;
    a.rows = p.rows;
    a.experts = p.experts;
    a.hi = p.hi;
    a.res = p.res;
    a.n = p.n;
    a.k = p.k;
    a.ksplit = plan.ksplit;
    a.splits = plan.splits;
    a.y = p.y;
    a.partial = partial;
    a.scale = nullptr;
    a.cus = plan.cus;
    a.range = plan.range_addr;
    a.rotate = p.k % 4096 == 0;
    const bool grouped = p.offsets != nullptr;
    if (plan.variant == GEMM_G5_256x256)
        return grouped ? hipErrorInvalidValue : launch_gemm256_f16(p.mode, p.enc, a, stream);
    if (p.enc == ENC_E4M3)
        return p.mode == MODE_FULL ? launch_g4_variant<MODE_FULL, ENC_E4M3>(a, plan, grouped, stream)
                                   : launch_g4_variant<MODE_FAST, ENC_E4M3>(a, plan, grouped, stream);
    return p.mode == MODE_FULL ? launch_g4_variant<MODE_FULL, ENC_E5M2>(a, plan, grouped, stream)
                               : launch_g4_variant<MODE_FAST, ENC_E5M2>(a, plan, grouped, stream);
}

hipError_t launch_gemm_fp8(int enc, const uint8_t *xq, const float *scale, const int32_t *offsets,
                           int64_t m, int64_t experts, int64_t n, int64_t k, const uint8_t *hi,
                           uint16_t *y, const LinearPlan &plan, float *partial, hipStream_t stream)
{
    GemmArgs a;
    a.x = xq;
    a.offsets = offsets;
    a.rows = m;
    a.experts = experts;
    a.hi = hi;
    a.res = ResidualView{nullptr, nullptr, 0, 0, 0};
    a.n = n;
    a.k = k;
    a.ksplit = plan.ksplit;
    a.splits = plan.splits;
    a.y = y;
    a.partial = partial;
    a.scale = scale;
    a.cus = plan.cus;
    a.range = 0;
    a.rotate = 0;
    if (plan.variant == GEMM_G3_256x256)
        return offsets ? hipErrorInvalidValue : launch_gemm256_fp8(enc, a, stream);
    return enc == ENC_E4M3 ? launch_g3<ENC_E4M3>(a, plan, stream)
                           : launch_g3<ENC_E5M2>(a, plan, stream);
}

}  // namespace dps
