// dps_gemm_common.h -- what the matrix-core GEMM kernels share: the argument
// block, the token range of a grouped block, output stores, direct-to-LDS
// loads and the stage barrier (gfx950).
#pragma once

#include <type_traits>

#include "dps_internal.h"

namespace dps {

struct GemmArgs {
    const void *x;  // FP16 [rows][k] or E4M3 [rows][k]
    const int32_t *offsets;
    int64_t rows;
    int64_t experts;
    const uint8_t *hi;
    ResidualView res;
    int64_t n, k, ksplit;
    int splits;
    uint16_t *y;
    float *partial;
    const float *scale;
    int cus;     // compute units of the device (the 256 x 256 tile's grid)
    int range;   // full mode: a row's residual bytes of one K range span at most two chunks
    int rotate;  // wide-row GEMM: start each block's K walk by weight tile (see gemm4)
};

namespace {

// Token range of a block of a grouped call: grid.y walks the experts' tile
// counts.  Returns false if no work.  With tail > 0 an expert's last tile also
// takes up to `tail` rows beyond bm, so an expert of bm + 1 .. bm + tail rows
// is one tile, not two: its weights are read once.  Such a range [m0, m1) spans
// more than bm rows; the kernel treats rows m0 + bm .. m1 - 1 as its tail.
// The tile count per expert never grows, so the host's grid bound still holds.
__device__ __forceinline__ bool block_rows(const GemmArgs &a, int64_t &e, int64_t &m0,
                                           int64_t &m1, int bm, int tail)
{
    const int64_t t = blockIdx.y;
    int64_t cum = 0;
    int64_t prev = 0;
    for (int64_t ex = 0; ex < a.experts; ++ex) {
        int64_t o1 = a.offsets[ex + 1];
        o1 = o1 < prev ? prev : (o1 > a.rows ? a.rows : o1);
        const int64_t r = o1 - prev;
        const int64_t tiles =
            r <= 0 ? 0 : (r <= bm + tail ? 1 : (r - tail + bm - 1) / bm);
        if (t < cum + tiles) {
            e = ex;
            m0 = prev + (t - cum) * bm;
            m1 = t == cum + tiles - 1 ? o1 : m0 + bm;  // the last tile takes the tail
            return true;
        }
        cum += tiles;
        prev = o1;
    }
    return false;
}

typedef _Float16 half4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void store_half4(uint16_t *p, f32x4 v)
{
    *reinterpret_cast<half4 *>(p) = half4{(_Float16)v.x, (_Float16)v.y, (_Float16)v.z,
                                          (_Float16)v.w};
}

__device__ __forceinline__ void store_tile_out(const GemmArgs &a, int s, int64_t m, int64_t n0,
                                               f32x4 v, int64_t m1)
{
    if (m >= m1 || n0 >= a.n)
        return;
    if (a.splits == 1) {
        uint16_t *yp = a.y + m * a.n + n0;
        if (n0 + 3 < a.n && (a.n & 3) == 0) {
            store_half4(yp, v);
        } else {
            const float vv[4] = {v.x, v.y, v.z, v.w};
            for (int r = 0; r < 4 && n0 + r < a.n; ++r)
                yp[r] = __builtin_bit_cast(uint16_t, (_Float16)vv[r]);
        }
    } else {
        float *pp = a.partial + ((int64_t)s * a.rows + m) * a.n + n0;
        if (n0 + 3 < a.n && (a.n & 3) == 0) {
            *reinterpret_cast<f32x4 *>(pp) = v;
        } else {
            const float vv[4] = {v.x, v.y, v.z, v.w};
            for (int r = 0; r < 4 && n0 + r < a.n; ++r)
                pp[r] = vv[r];
        }
    }
}

__device__ __attribute__((aligned(16))) const uint8_t g_zero16[16] = {0};

// Cache policies of a direct-to-LDS load: plain, and nontemporal for weights
// that are read once and do not stay cached (dps_gemm.hip, streams).
enum { AUX_CACHED = 0, AUX_STREAM = 2 };

// 16 bytes per lane from `src` into the wave's 1 KiB at LDS address `lds` (lane
// l lands at lds + 16 l), as one asm statement without outputs.  The compiler
// takes the builtin for a flat access that may retire out of
// order and then waits for lgkmcnt(0) before every use of an LDS read, where
// the reads still in flight could stay so.  Completion is the caller's own
// business (vmcnt, in issue order).
typedef __attribute__((address_space(3))) uint8_t lds_u8;

// M0 is put back, since the compiler keeps values of its own there.
template <int AUX>
__device__ __forceinline__ void dma16_at(const void *src, lds_u8 *lds)
{
    uint32_t m0;
    if (AUX == AUX_STREAM)
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, off nt\n\ts_mov_b32 m0, %0"
                     : "=&s"(m0)
                     : "s"((uint32_t)(uintptr_t)lds), "v"(src)
                     : "memory");
    else
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, off\n\ts_mov_b32 m0, %0"
                     : "=&s"(m0)
                     : "s"((uint32_t)(uintptr_t)lds), "v"(src)
                     : "memory");
}

// A raw buffer over [p, p + bytes): 48-bit base, byte count, data format 32
// (the descriptor of untyped buffers on gfx9).  Loads past the end return zero.
typedef int32_t rsrc_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ rsrc_t make_rsrc(const void *p, int64_t bytes)
{
    const uint64_t b = (uint64_t)p;
    return rsrc_t{__builtin_amdgcn_readfirstlane((int)(uint32_t)b),
                  __builtin_amdgcn_readfirstlane((int)((b >> 32) & 0xFFFFu)),
                  __builtin_amdgcn_readfirstlane((int)(bytes < 0xFFFFFFFFll ? bytes : 0xFFFFFFFFll)),
                  0x00020000};
}

// buffer_load_dwordx4 ... lds: 16 bytes per lane from buffer offset voffset +
// soffset into the wave's 1 KiB at `lds`.
__device__ void buffer_load_lds(rsrc_t rsrc, __attribute__((address_space(3))) void *lds, int size,
                                int voffset, int soffset, int offset,
                                int aux) __asm("llvm.amdgcn.raw.buffer.load.lds");

// The value, opaque to the optimizer: what the rare paths of the stage loop
// derive from it is computed there instead of being kept in registers.
__device__ __forceinline__ int unhoisted(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// The same for a wave-uniform value, which stays in a scalar register.
__device__ __forceinline__ int scalar_part(int v)
{
    asm("" : "+s"(v));
    return v;
}

// lgkmcnt(0).  Scalar loads retire out of order with LDS reads, and a rare
// path of the stage loop that leaves some pending would make the compiler
// wait for every LDS read of the common path where it needs only the oldest.
__device__ __forceinline__ void rare_path_end()
{
    __builtin_amdgcn_s_waitcnt(0xC07F);
}

// The kernel's arguments, loaded anew where a rare path needs them: what the
// stage loop does not use takes no scalar registers there.
__device__ __forceinline__ GemmArgs rare_args()
{
    auto p = (const __attribute__((address_space(4))) void *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    GemmArgs a;
    __builtin_memcpy(&a, (const void *)p, sizeof(a));
    return a;
}

// This lane's index, computed anew where it is called.
__device__ __forceinline__ int lane_again()
{
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, (uint32_t)unhoisted(0)));
}

// s_waitcnt vmcnt(n) leaving the other counters alone (gfx9 encoding).
#define DPS_WAIT_VMCNT(n) \
    __builtin_amdgcn_s_waitcnt(((n) & 0xF) | ((((n) >> 4) & 3) << 14) | (0x7 << 4) | (0xF << 8))

// Block barrier between pipeline stages.  __syncthreads() carries a
// workgroup-scope fence, which the compiler satisfies by waiting for every
// outstanding vector-memory operation (direct-to-LDS loads count as LDS
// writes): the whole DMA ring would drain at every stage.  The loops instead
// wait for exactly what they need -- their own DMA of the stage about to be
// read (vmcnt, before this call) and their own LDS reads of the slot about to
// be refilled (lgkmcnt(0), here) -- and then meet at a bare s_barrier.  The
// empty asm statements keep the compiler from moving memory accesses across.
__device__ __forceinline__ void stage_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt and expcnt at their maxima
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Swizzle of 128-byte LDS rows: 16-byte chunk c of row r sits at slot
// c ^ swz8(r).  Lane (i, g) reading chunk 4q + g of 16 such rows is the
// pattern measured conflict-free (ds_read_b128 at ~210 B/clk per CU).
__device__ __forceinline__ int swz8(int r) { return (r >> 1) & 7; }

// Rows of up to this many elements are reached by 32-bit byte offsets from the
// first row a wave loads (at most 31 rows of two bytes per element on); longer
// ones take the general path of the stage loads, with 64-bit addresses.
constexpr int64_t kMaxOffsetK = int64_t(1) << 25;

// dense calls: a 1-D grid, padded to a multiple of the 8 XCDs
inline dim3 dense_grid(int64_t tiles)
{
    return dim3((unsigned)((tiles + 7) / 8 * 8), 1, 1);
}

}  // namespace

// The 256 x 256 tile (dps_gemm256.hip): FP16 full and fast mode, and FP8
// activations.
hipError_t launch_gemm256_f16(int mode, int enc, const GemmArgs &a, hipStream_t stream);
hipError_t launch_gemm256_fp8(int enc, const GemmArgs &a, hipStream_t stream);

}  // namespace dps
