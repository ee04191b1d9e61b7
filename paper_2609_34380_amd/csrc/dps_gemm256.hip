// dps_gemm256.hip -- the 256 x 256 tile of the nested linear (gfx950): prefill
// on FP16 activations (full and fast mode) and on FP8 activations.
//
// Full mode merges the upper and residual bytes into FP16 operands in
// registers (Sec. IV-C: reconstruction during computation), fast mode
// converts the upper bytes alone, both for v_mfma_f32_16x16x32_f16; the FP8
// kind feeds the upper bytes as stored (E5M2, or E4M3 whose fast-mode value is
// E4M3 * 2^-8) to v_mfma_f32_16x16x128_f8f6f4 against E4M3 activations and
// applies the row scale to the fp32 sums.
//
// Bound: matrix work, 2048 MFMA cycles per SIMD and stage in every kind, and
// under sustained load the card's power (a plain library FP16 GEMM of these
// shapes reaches 1.45 PFLOP/s on random data and 2.1 on zeros).  One block of
// eight waves (4 x 2, wave tile 64 weight rows x 128 tokens) fills a CU:
// 128 fp32 accumulators per lane and 160 KiB of LDS.  What the split and the
// loop are built for:
//   - 256 x 256 reads the fewest LDS bytes per flop that fit: a stage (64 K
//     elements, FP8 128) is 32 KiB of tokens and 32 KiB of weights (fast mode
//     16), each wave reads 24 KiB of fragments for 64 MFMAs;
//   - software pipeline over the one barrier per stage: it stands before the
//     last two of a stage's eight token tiles, when every fragment of the
//     stage is in registers, so its slots can be refilled at once and the next
//     stage's first reads run beside the remaining MFMAs.  The weight operands
//     of the next stage are merged between the MFMAs of the last and the
//     first token tile;
//   - the steady state issues direct-to-LDS loads with almost no address
//     arithmetic: buffer loads with a scalar stage offset, or (full mode,
//     whose two planes share a line) one 64-bit add per load from pointers
//     that are renewed only where a lane leaves its residual chunk;
//   - output stores without per-element checks when the tile is whole, behind
//     the first loads of the block's next tile.
// MI355X, against the earlier kernels on these tiles (barrier at the head of
// a stage, all reads and merges behind it): gate+up 28672 x 4096 in full mode
// 1871 -> 1655 us at 8192 tokens and 408 -> 352 at 1531, fast mode 1578 ->
// 1455, FP8 with its quantization 972 -> 820; down 4096 x 14336 in full mode
// at 8192 tokens 917 -> 796.  Moving the loads elsewhere in the stage (all at
// the barrier, one per token tile, alternating between the two waves of a
// SIMD, one wave at a time) changed the time by -2 to +30%: each costs its
// wave 60-115 cycles wherever it stands, about 0.3 of the 1.6 us a stage
// takes at full clock.
#include "dps_gemm_common.h"

namespace dps {

namespace {

enum { T_FULL = 0, T_FAST = 1, T_FP8 = 2 };

// Rings of WS weight and XS token stages.
template <int KIND>
struct T256 {
    static constexpr int BK = KIND == T_FP8 ? 128 : 64;   // K elements per stage
    static constexpr int W_SLOT = (KIND == T_FAST ? 16 : 32) * 1024;
    static constexpr int X_SLOT = 32 * 1024;
    static constexpr int WS = KIND == T_FAST ? 4 : 3;
    static constexpr int XS = KIND == T_FAST ? 3 : 2;
    static constexpr int X_BASE = W_SLOT * WS;
    static constexpr int LDS = X_BASE + X_SLOT * XS;
    static constexpr int NW = W_SLOT / 1024 / 8;  // DMA instructions per wave per stage
    static constexpr int NX = X_SLOT / 1024 / 8;
    static constexpr int XB = KIND == T_FP8 ? 1 : 2;  // bytes per activation
    static constexpr int RAW = KIND == T_FAST ? 4 : 8;
    // group u of a wave's DMA is tokens of stage u + XS, then weights of
    // stage u + WS; at the barrier of stage t (groups up to t - 1 are out)
    // these may still be in flight without touching stage t + 1
    static constexpr int OUTSTANDING = (XS < WS ? NW : 0) + (XS - 2) * (NX + NW);
    static_assert(XS >= 2 && WS >= XS && LDS <= 160 * 1024, "rings");
};

// LDS lines of 128 bytes, 16-byte chunks at slot chunk ^ swz8(line).
// Weights: full mode line r holds row r, its 64 upper bytes in chunks 0-3 and
// its 64 residual bytes in chunks 4-7; fast mode line 16 t + i holds row
// 32 t + i in chunks 0-3 and row 32 t + 16 + i in chunks 4-7; FP8 line r holds
// 128 upper bytes of row r.  A fragment read of lane (i, g) is chunk 4q + g of
// 16 lines, conflict-free.
// Tokens: FP8 as the weights.  FP16 K chunk c (8 elements) of a row sits at
// slot sigma(c) ^ swz8(row), sigma(c) = (c >> 1) | (c & 1) << 2, so that the
// chunks 2g + q which lane group g reads in MFMA step q are four consecutive
// slots too (plain order costs bank conflicts, half of the LDS cycles);
// tok_chunk is sigma's inverse, the chunk the DMA writes into a slot.
// Either way both operands of an MFMA pair the same K elements.
__device__ __forceinline__ int tok_chunk(int slot) { return ((slot & 3) << 1) | (slot >> 2); }

template <int KIND, int ENC>
__global__ __launch_bounds__(512) void tile256_kernel(GemmArgs a)
{
    using C = T256<KIND>;
    constexpr int WS = C::WS, XS = C::XS, NW = C::NW, NX = C::NX;
    __shared__ __attribute__((aligned(16))) uint8_t smem[C::LDS];
    lds_u8 *const lds = (lds_u8 *)smem;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15;
    const int lg = lane >> 4;
    const int wn = wave & 3;   // 64-row quarter of the weight tile
    const int wm = wave >> 2;  // 128-token half of the token tile

    // 1-D grid remapped for the 8 XCDs (block L runs on XCD L % 8): XCD x
    // takes a contiguous tile range, walked in groups of four weight tiles
    // with the weight tile fastest, so the ~32 blocks resident on an XCD share
    // 4 weight tiles and 8 token tiles through its L2.
    const uint32_t mtiles = (uint32_t)((a.rows + 255) >> 8);
    const uint32_t ntiles = (uint32_t)((a.n + 255) >> 8);
    const uint32_t per_split = mtiles * ntiles;
    const uint32_t total = per_split * (uint32_t)a.splits;
    const uint32_t per_xcd = (total + 7) / 8;
    // A block takes every nloc-th tile of its XCD's range.
    const uint32_t nloc = gridDim.x / 8;
    uint32_t idx = blockIdx.x / 8;
    int s = 0, ntk = 0, klen = 0, t_full = 0;
    bool rev = false;
    int64_t mrow0 = 0, mrow1 = 0, n0 = 0, kb0 = 0;
    auto tk = [&](int t) { return rev ? ntk - 1 - t : t; };

    // ---- DMA sources ---------------------------------------------------------
    // token instruction jj: rows 8(4w+jj) .. +7, lane -> row + lane/8, slot
    // lane%8.  Rows past the tile's last token lie beyond the buffer resource.
    rsrc_t xr, wr;  // of the tile's tokens and (fast mode, FP8) upper bytes
    const uint32_t xstep = (uint32_t)(8 * a.k * C::XB);  // eight rows on
    uint32_t xoff[2];
#pragma unroll
    for (int par = 0; par < 2; ++par) {
        const int slot = (lane & 7) ^ swz8(8 * par + (lane >> 3));
        xoff[par] = (uint32_t)((lane >> 3) * a.k + (KIND == T_FP8 ? slot * 16 : tok_chunk(slot) * 8)) *
                    C::XB;
    }
    auto issue_x = [&](int tr, int slot) {
        lds_u8 *dst = lds + C::X_BASE + slot * C::X_SLOT + 4096 * wave;
        if (tr < t_full) {
#pragma unroll
            for (int jj = 0; jj < NX; ++jj)
                buffer_load_lds(xr, dst + jj * 1024, 16,
                                (uint32_t)unhoisted((int)xoff[jj & 1]) + jj * xstep,
                                tr * (C::BK * C::XB), 0, 0);
        } else {
            const int ln = lane_again();
#pragma unroll
            for (int jj = 0; jj < NX; ++jj) {
                const int sl = (ln & 7) ^ swz8(8 * jj + (ln >> 3));
                const int kk = tr * C::BK + (KIND == T_FP8 ? sl * 16 : tok_chunk(sl) * 8);
                const int64_t m = mrow0 + 32 * wave + 8 * jj + (ln >> 3);
                const bool ok = m < mrow1 && kk < klen;
                const uint8_t *src =
                    static_cast<const uint8_t *>(a.x) + (m * a.k + kb0 + kk) * C::XB;
                dma16_at<AUX_CACHED>(ok ? (const void *)src : (const void *)g_zero16, dst + jj * 1024);
            }
            rare_path_end();
        }
    };
    // weight instruction jj: lines 8j .. 8j+7 (j = NW w + jj), lane -> line
    // 8j + lane/8, slot lane%8
    auto w_row = [&](int ln, int jj, int &wel, bool &lo) {
        const int line = 8 * (NW * wave + jj) + (ln >> 3);
        const int c = (ln & 7) ^ swz8(line);
        lo = KIND == T_FULL && c >= 4;
        wel = KIND == T_FP8 ? c * 16 : (c & 3) * 16;
        const int r = KIND == T_FAST ? (2 * (line >> 4) + (c >> 2)) * 16 + (line & 15) : line;
        const int64_t nr = n0 + r;
        return nr < a.n ? nr : a.n - 1;
    };
    // Fast mode and FP8: byte offsets from wr's base (FP8: of instructions 0
    // and 1; 2 and 3 are 16 rows on).
    uint32_t woff[2];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
        const int line = 8 * jj + (lane >> 3);
        const int c = (lane & 7) ^ swz8(line);
        woff[jj] = (uint32_t)((KIND == T_FAST ? (c >> 2) * 16 + line : line) * a.k +
                              (KIND == T_FP8 ? c * 16 : (c & 3) * 16));
    }
    const uint8_t *wp[NW];  // full mode: pointer of the piece of K stage 0
    int wev = 0;            // full mode: next stage whose pieces need new pointers (-1: none)
    // Full mode, K ranges no longer than a chunk: once wknown is set, lane r (and
    // r + 32) holds how many chunks further than its first one row r of the
    // wave goes on, less one.
    bool wknown = false;
    int32_t wnext = 0;
    auto set_tile = [&]() __attribute__((always_inline)) {  // the tile of idx; false when there is none
        const uint32_t tl = (blockIdx.x % 8) * per_xcd + idx;
        if (idx >= per_xcd || tl >= total)
            return false;
        constexpr uint32_t G = 4;
        s = (int)(tl / per_split);
        const uint32_t rr = tl % per_split;
        const uint32_t chunk = rr / (G * mtiles);
        const uint32_t within = rr % (G * mtiles);
        const uint32_t gc = ntiles - chunk * G < G ? ntiles - chunk * G : G;
        const uint32_t ntile = chunk * G + within % gc;
        mrow0 = (int64_t)(within / gc) * 256;
        mrow1 = mrow0 + 256 < a.rows ? mrow0 + 256 : a.rows;
        n0 = (int64_t)ntile * 256;
        kb0 = (int64_t)s * a.ksplit;
        klen = (int)((kb0 + a.ksplit < a.k ? kb0 + a.ksplit : a.k) - kb0);
        ntk = (klen + C::BK - 1) / C::BK;
        // stages entirely inside the K range, whose loads take 32-bit row offsets
        t_full = a.k <= kMaxOffsetK ? klen / C::BK : 0;
        // Serpentine K walk (FP16): odd groups of four weight tiles walk K
        // backwards and so start on the token stages the XCD's previous group
        // read last, still in its L2 (gate+up at 2048 tokens 0.94x the time in
        // fast mode, 0.99x in full mode).
        rev = KIND != T_FP8 && ((ntile >> 2) & 1);
        const int64_t xrow0 = mrow0 + 32 * wave < mrow1 ? mrow0 + 32 * wave : mrow1 - 1;
        xr = make_rsrc(static_cast<const uint8_t *>(a.x) + (xrow0 * a.k + kb0) * C::XB,
                       ((mrow1 - xrow0) * a.k - kb0) * C::XB);
        wev = tk(0);
        wknown = false;
        if (KIND != T_FULL) {
            // (rows past n lie beyond the resource)
            const int64_t wrow0 = n0 + 32 * wave < a.n ? n0 + 32 * wave : a.n - 1;
            wr = make_rsrc(a.hi + wrow0 * a.k + kb0, (a.n - wrow0) * a.k - kb0);
        }
        return true;
    };
    // The stage from which on the residual piece at element `wel` of K stage 0
    // of row nr lies in the next chunk.
    auto two_from = [&](const GemmArgs &r, int64_t nr, int wel) __attribute__((always_inline)) {
        const uint32_t l0 = (uint32_t)nr * (uint32_t)r.k + (uint32_t)kb0 + (uint32_t)wel;
        const uint32_t c = 1u << r.res.log2c;
        return (int)((c - (l0 & (c - 1)) + C::BK - 1) >> 6);
    };
    // Full mode: the pointers of stage tr's pieces, and the next stage in walk
    // order at which any lane's piece leaves its residual chunk or passes the
    // end of the K range (pieces without a source read zeros, stage by stage).
    // A lookup waits for the slot table and with it for every load this wave
    // has in flight, so rows that cross chunks must not cost one per crossing:
    // both chunks' slots are read once where a row has two at most (MI355X,
    // 5120 x 6160 in 16 KiB chunks, 1024 tokens: 129 -> 104 us).
    auto w_pointers = [&](int tr) __attribute__((always_inline)) {
        const GemmArgs r = rare_args();
        const int ln = lane_again();
        const int64_t off = (int64_t)tr * C::BK;
        int lo_t = 0, hi_t = ntk;  // stages [lo_t, hi_t) keep these pointers
        if (wknown) {
#pragma unroll
            for (int jj = 0; jj < NW; ++jj) {
                int wel;
                bool lo;
                const int64_t nr = w_row(ln, jj, wel, lo);
                const int t1 = (klen - wel + C::BK - 1) / C::BK;
                const int b = lo ? two_from(r, nr, wel) : t1;
                const int64_t d = (int64_t)__shfl(wnext, 8 * jj + (ln >> 3), 64) << r.res.log2c;
                if (b < t1 && b == (rev ? tr + 1 : tr))
                    wp[jj] += rev ? -d : d;
                if (tr >= t1)
                    wp[jj] = g_zero16 - off;
                const int t0 = b < t1 && b <= tr ? b : 0;
                const int tn = b < t1 && b > tr ? b : (t1 > tr ? t1 : ntk);
                lo_t = t0 > lo_t ? t0 : lo_t;
                hi_t = tn < hi_t ? tn : hi_t;
            }
        } else {
            bool all_in = true;
#pragma unroll
            for (int jj = 0; jj < NW; ++jj) {
                int wel;
                bool lo;
                const int64_t nr = w_row(ln, jj, wel, lo);
                const int64_t l0 = nr * r.k + kb0 + wel;
                const bool in = off + wel < klen;
                const uint8_t *p = r.hi + l0;
                bool ok = in;
                int t0 = 0, t1 = (klen - wel + C::BK - 1) / C::BK;
                if (lo) {
                    const int64_t l = l0 + (in ? off : -wel);
                    const int64_t o = residual_offset(r.res, l);
                    ok = in && o >= 0;
                    p = r.res.pool + (o - off);
                    const uint32_t c = 1u << r.res.log2c, at = (uint32_t)l & (c - 1);
                    const int b1 = tr + (int)((c - at + C::BK - 1) >> 6);
                    t0 = tr - (int)(at >> 6);
                    t0 = t0 > 0 ? t0 : 0;
                    t1 = b1 < t1 ? b1 : t1;
                }
                wp[jj] = ok ? p : g_zero16 - off;
                all_in &= ok;
                t0 = ok ? t0 : tr;
                t1 = ok ? t1 : tr + 1;
                lo_t = t0 > lo_t ? t0 : lo_t;
                hi_t = t1 < hi_t ? t1 : hi_t;
            }
            if (r.range) {
                const int64_t row = n0 + 32 * wave + (ln & 31);
                const int64_t f = (row < r.n ? row : r.n - 1) * r.k + kb0;
                const int64_t ce = ((f >> r.res.log2c) + 1) << r.res.log2c;
                const bool two = f + klen > ce;
                if (__any(two)) {
                    const int64_t o0 = residual_offset(r.res, f);
                    const int64_t o1 = residual_offset(r.res, two ? ce : f);
                    wnext = (int32_t)((o1 >> r.res.log2c) - (o0 >> r.res.log2c) - 1);
                    all_in &= o0 >= 0 && o1 >= 0;
                }
                wknown = __all(all_in);
            }
        }
        if (__all(lo_t <= 0 && hi_t >= ntk)) {
            wev = -1;
            rare_path_end();
            return;
        }
        int v = rev ? -(lo_t - 1) : hi_t;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const int u = __shfl_xor(v, d, 64);
            v = u < v ? u : v;
        }
        v = __builtin_amdgcn_readfirstlane(v);
        wev = rev ? -v : v;
        rare_path_end();
    };
    static_assert(KIND != T_FULL || C::BK == 64, "stage arithmetic of w_pointers");
    auto issue_w = [&](int tr, int slot) __attribute__((always_inline)) {
        lds_u8 *dst = lds + slot * C::W_SLOT + NW * 1024 * wave;
        if (KIND == T_FULL) {
#pragma unroll
            for (int jj = 0; jj < NW; ++jj)
                dma16_at<AUX_CACHED>(wp[jj] + (int64_t)tr * C::BK, dst + jj * 1024);
        } else if (tr < t_full) {
#pragma unroll
            for (int jj = 0; jj < NW; ++jj)
                buffer_load_lds(wr, dst + jj * 1024, 16,
                                (uint32_t)unhoisted((int)woff[jj & 1]) + (jj >> 1) * 2 * xstep,
                                tr * C::BK, 0, 0);
        } else {
            const int ln = lane_again();
#pragma unroll
            for (int jj = 0; jj < NW; ++jj) {
                int wel;
                bool lo;
                const int64_t nr = w_row(ln, jj, wel, lo);
                const int kk = tr * C::BK + wel;
                const uint8_t *src = a.hi + nr * a.k + kb0 + kk;
                dma16_at<AUX_CACHED>(kk < klen ? (const void *)src : (const void *)g_zero16, dst + jj * 1024);
            }
            rare_path_end();
        }
    };

    f32x4 acc[4][8];

    // ---- fragment reads ---------------------------------------------------------
    // Both operands' addresses have one lane part; E4M3 in full mode has a register
    // for the tokens' only and reaches the weights by a scalar difference.
    constexpr bool ONE = KIND == T_FULL && ENC == ENC_E4M3;
    const int abase = wn * (KIND == T_FAST ? 32 : 64) * 128;
    const int bbase = C::X_BASE + wm * 128 * 128;
    const int boff0 = bbase + li * 128 + ((lg ^ swz8(li)) << 4);
    const int aoff0 = ONE ? boff0 : boff0 - bbase + abase;
    u32x4 raw[C::RAW];
    u32x4 bv[4][2];
    auto ld = [&](int off) { return *reinterpret_cast<const u32x4 *>(smem + off); };
    auto read_w = [&](int slot) {
        const int b = ONE ? scalar_part(slot * C::W_SLOT + abase - bbase) : slot * C::W_SLOT;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            if (KIND == T_FAST) {
                raw[nt] = ld(b + ((nt & 1) ? aoff0 ^ 64 : aoff0) + (nt >> 1) * 2048);
            } else {
                raw[nt] = ld(b + aoff0 + nt * 2048);
                raw[(4 + nt) % C::RAW] = ld(b + (aoff0 ^ 64) + nt * 2048);
            }
        }
    };
    auto read_b = [&](int slot, int mt) {
        const int b = slot * C::X_SLOT + mt * 2048;
        bv[mt & 3][0] = ld(b + boff0);
        bv[mt & 3][1] = ld(b + (boff0 ^ 64));
    };

    auto prologue = [&]() __attribute__((always_inline)) {  // the loads of groups -WS .. -1
#pragma unroll 1
        for (int u = -WS; u < 0; ++u) {
            if (u + XS >= 0 && u + XS < ntk)
                issue_x(tk(u + XS), u + XS);
            if (u + WS < ntk) {
                if (KIND == T_FULL && tk(u + WS) == wev)
                    w_pointers(wev);
                issue_w(tk(u + WS), u + WS);
            }
        }
    };
    if (!set_tile())
        return;
    prologue();

    // Weight operands of stage t: av[q] feeds MFMA step q.  Step 0's are formed
    // at the end of stage t - 1, after the last MFMA that reads the old ones,
    // and step 1's between the first MFMAs of stage t, so the byte merges run
    // beside matrix work.
    half8 av[2][4];
    i32x8 a8[4];
    auto form = [&](int q) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const u32x4 h = raw[nt];
            const u32x4 l = KIND == T_FULL ? raw[(4 + nt) % C::RAW] : u32x4{0u, 0u, 0u, 0u};
            constexpr int MODE = KIND == T_FULL ? MODE_FULL : MODE_FAST;
            if (KIND == T_FP8)
                a8[nt] = i32x8{(int)h.x, (int)h.y, (int)h.z, (int)h.w,
                               (int)raw[(4 + nt) % C::RAW].x, (int)raw[(4 + nt) % C::RAW].y,
                               (int)raw[(4 + nt) % C::RAW].z, (int)raw[(4 + nt) % C::RAW].w};
            else
                av[q][nt] = q ? weight8<MODE, ENC>(h.z, h.w, l.z, l.w)
                              : weight8<MODE, ENC>(h.x, h.y, l.x, l.y);
        }
    };
    auto mma_q = [&](int mt, int q) {  // F16 kinds: MFMA step q of token tile mt
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
            acc[nt][mt] = mfma16x16x32(av[q][nt], as_half8(bv[mt & 3][q]), acc[nt][mt]);
    };
    auto mma = [&](int mt) {
        if (KIND == T_FP8) {
            const u32x4 p = bv[mt & 3][0], q = bv[mt & 3][1];
            const i32x8 b8 = {(int)p.x, (int)p.y, (int)p.z, (int)p.w,
                              (int)q.x, (int)q.y, (int)q.z, (int)q.w};
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                acc[nt][mt] = mfma16x16x128_fp8<ENC>(a8[nt], b8, acc[nt][mt]);
        } else {
            mma_q(mt, 0);
            mma_q(mt, 1);
        }
    };
    int stores = 0;  // instructions of the last tile's stores, still in flight behind the prologue
    for (;;) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (WS > ntk || stores < 0)
            DPS_WAIT_VMCNT(0);
        else if (stores > 0)
            DPS_WAIT_VMCNT(C::OUTSTANDING + NX + NW + 32);
        else
            DPS_WAIT_VMCNT(C::OUTSTANDING + NX + NW);
        stage_barrier();
        read_w(0);
        read_b(0, 0);
        read_b(0, 1);
        form(0);
        int ws = 0, xs = 0;  // slots of stage t
        int wf = 0;          // weight slot that stage t - 1 left
        for (int t = 0; t < ntk; ++t) {
            const int ws1 = ws + 1 < WS ? ws + 1 : 0;
            const int xs1 = xs + 1 < XS ? xs + 1 : 0;
#pragma unroll
            for (int mt = 0; mt < 6; ++mt) {
                if (mt > 0)
                    __builtin_amdgcn_sched_barrier(0);
                read_b(xs, mt + 2);
                if (mt == 0 && KIND != T_FP8) {
                    mma_q(0, 0);
                    form(1);
                    mma_q(0, 1);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);
                    }
                } else {
                    mma(mt);
                }
                if (mt == 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (t > 0 && t - 1 + WS < ntk)
                        issue_w(tk(t - 1 + WS), wf);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (t + WS <= ntk)
                DPS_WAIT_VMCNT(C::OUTSTANDING);
            else
                DPS_WAIT_VMCNT(0);
            stage_barrier();
            if (KIND == T_FULL && t + WS < ntk && tk(t + WS) == wev)
                w_pointers(wev);
            read_w(ws1);
            read_b(xs1, 0);
            read_b(xs1, 1);
            __builtin_amdgcn_sched_barrier(0);
            if (t + XS < ntk)
                issue_x(tk(t + XS), xs);
            __builtin_amdgcn_sched_barrier(0);
            mma(6);
            if (KIND == T_FP8) {
                mma(7);
                form(0);
            } else {
                mma_q(7, 0);
                form(0);
                mma_q(7, 1);
                __builtin_amdgcn_sched_group_barrier(0x8, 12, 1);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 1);
                    __builtin_amdgcn_sched_group_barrier(0x2, 8, 1);
                }
            }
            wf = ws;
            ws = ws1;
            xs = xs1;
        }

        // Lane (i, g) holds rows 16 nt + 4g .. +3 of the wave's 64 weight rows for
        // token 16 mt + i.  A tile inside the output stores without per-element
        // checks; every lane's addresses are one pointer plus constants.
        constexpr float wscale = ENC == ENC_E4M3 ? 0.00390625f : 1.f;
        if (KIND == T_FP8) {
#pragma unroll
            for (int mt = 0; mt < 8; ++mt) {
                const int64_t m = mrow0 + wm * 128 + 16 * mt + (lane_again() & 15);
                const float sc = m < mrow1 ? a.scale[m] * wscale : 0.f;
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    acc[nt][mt] *= sc;
            }
        }
        // The next tile's first loads go out before this tile's stores: every
        // wave has read its last fragments (the last stage's barrier), so the ring
        // is free, and the loads' latency runs under the stores.
        const int64_t m1 = mrow1;
        const bool whole = mrow0 + 256 == mrow1 && n0 + 256 <= a.n && (a.n & 3) == 0;
        const int sd = s;
        const int64_t md = mrow0 + wm * 128, nd = n0 + wn * 64;
        idx += nloc;
        const bool more = set_tile();
        if (more)
            prologue();
        stores = whole ? 32 : -1;
        const int le = lane_again();
        const int64_t m = md + (le & 15), n = nd + (le >> 4) * 4;
        if (whole) {
            if (a.splits == 1) {
                uint16_t *yp = a.y + m * a.n + n;
#pragma unroll
                for (int mt = 0; mt < 8; ++mt, yp += 16 * a.n)
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt)
                        store_half4(yp + nt * 16, acc[nt][mt]);
            } else {
                float *pp = a.partial + ((int64_t)sd * a.rows + m) * a.n + n;
#pragma unroll
                for (int mt = 0; mt < 8; ++mt, pp += 16 * a.n)
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt)
                        *reinterpret_cast<f32x4 *>(pp + nt * 16) = acc[nt][mt];
            }
        } else {
#pragma unroll
            for (int mt = 0; mt < 8; ++mt)
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    store_tile_out(a, sd, m + 16 * mt, n + 16 * nt, acc[nt][mt], m1);
        }
        if (!more)
            return;
    }
}

template <int KIND, int ENC>
hipError_t launch(const GemmArgs &a, hipStream_t stream)
{
    // FP16: one block per CU (160 KiB of LDS), each taking tiles until its
    // XCD's range is done, so that a tile's first loads run under the previous
    // tile's stores (MI355X, against a block per tile: gate+up in full mode
    // 1658 -> 1627 us at 8192 tokens, 357 -> 350 at 1531, 128 -> 124 at 512).
    // FP8 is 1% slower that way (795 -> 802 at 8192) and runs a block per tile.
    const int64_t tiles = (a.n + 255) / 256 * a.splits * ((a.rows + 255) / 256);
    const dim3 grid = dense_grid(KIND == T_FP8 || tiles < a.cus ? tiles : a.cus);
    hipLaunchKernelGGL((tile256_kernel<KIND, ENC>), grid, dim3(512), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm256_f16(int mode, int enc, const GemmArgs &a, hipStream_t stream)
{
    if (mode == MODE_FULL)
        return enc == ENC_E4M3 ? launch<T_FULL, ENC_E4M3>(a, stream)
                               : launch<T_FULL, ENC_E5M2>(a, stream);
    return enc == ENC_E4M3 ? launch<T_FAST, ENC_E4M3>(a, stream)
                           : launch<T_FAST, ENC_E5M2>(a, stream);
}

hipError_t launch_gemm256_fp8(int enc, const GemmArgs &a, hipStream_t stream)
{
    return enc == ENC_E4M3 ? launch<T_FP8, ENC_E4M3>(a, stream)
                           : launch<T_FP8, ENC_E5M2>(a, stream);
}

}  // namespace dps
