// What the bf16 dense-layer kernels share (paper section 2.1: the dense layers of an encoder layer): the layout of
// their weights, the layout of their panels in LDS, and the way a wave stores its part of the result.
//
// Weights in fragment order.  W[N, K] lies in memory as the operands of v_mfma_f32_16x16x32_bf16: blocks of 16
// columns of C by 32 of K, 1 KB each, [N / 16][K / 32][64 lanes][8]; lane l of a block holds row l % 16 of W and the K
// chunk kchunk(l / 16) of eight.  A fragment is one contiguous 1 KB access, straight into registers (no LDS) or into
// LDS, where it is read back lane by lane without bank conflicts.  ep_bf16_pack_weights makes it once, when a stage or
// an embedding is created; the bytes are the same as row by row.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "ep_device.h"
#include "ep_kernels.h"

namespace ep_tile {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int NUM_XCD = 8;
constexpr int GROUP_M = 4;                           // tile rows of a group (see tile_of)
constexpr int BK = 64;                               // K step
constexpr int CPR = BK / 8;                          // 16-byte chunks of a panel row in LDS
constexpr int NS = BK / 32;                          // 32-wide slices of a K step
constexpr int FRAG_BYTES = 1024;                     // a weight fragment
constexpr int PAST_END = 0x40000000;                 // at least the bytes of a tile's rows of C: 256 rows, N < MAX_TILE_N
constexpr int MAX_TILE_N = 1 << 20;                  // offsets inside a tile's rows of C are 32-bit: N < MAX_TILE_N
constexpr int OOB = 0x7FFFFFF0;                      // past the end of any buffer: reads as zeros

// s_waitcnt with only the vector-memory counter, or only the LDS counter, constrained (gfx9 encoding)
#define EP_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))
#define EP_WAIT_LGKMCNT0() __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4) | (0x0 << 8))
#define EP_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// a lambda that is always inlined: the register arrays it captures must not be addressed
#define EP_INLINE __attribute__((always_inline))

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>)
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Panel rows of the activations in LDS are 8 chunks of 16 bytes; chunk c of row r sits at slot c ^ swz(r): the 16-byte
// fragment reads of 16 consecutive rows spread over all banks whether the LDS serves 8 or 16 lanes a cycle.
__device__ inline int swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }

// Quarter g of a wave multiplies K chunk kchunk(g) of a slice (any order would do, as long as both operands keep it): in
// the order 0, 2, 1, 3 the quarters' reads of a panel stay off each other's banks.  Its own inverse.
__device__ inline int kchunk(int g) { return ((g & 1) << 1) | (g >> 1); }

#if defined(__HIP_DEVICE_COMPILE__)   // buffer-resource builtins exist only in the device pass
typedef __attribute__((address_space(3))) void *lds_ptr;

// Buffer resource over a dense array: loads beyond `bytes` return zero and stores beyond it are dropped, which is
// how rows past M, columns past N and K steps past the end are handled without branches.
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
#endif

// Workgroup -> (K range, tile).  Consecutive workgroup ids land on different XCDs (8 of them, each with its own L2), so
// ids are first regrouped per XCD, and inside an XCD tiles are visited in groups of GROUP_M tile rows, column by
// column, so that workgroups running at the same time share panels of A and W.  `ranges` K ranges follow each other.
struct TileOf { int range, m, n; bool live; };
__device__ inline TileOf tile_of(int tiles_m, int tiles_n, int ranges)
{
    const int tiles = tiles_m * tiles_n, total = tiles * ranges;
    const int per_xcd = (total + NUM_XCD - 1) / NUM_XCD;
    int lid = (int)(blockIdx.x % NUM_XCD) * per_xcd + (int)(blockIdx.x / NUM_XCD);
    if (lid >= total) return {0, 0, 0, false};
    const int range = ranges > 1 ? lid / tiles : 0;
    lid -= range * tiles;
    const int group_sz = GROUP_M * tiles_n;
    const int group = lid / group_sz;
    const int first_m = group * GROUP_M;
    const uint32_t rows = (uint32_t)min(GROUP_M, tiles_m - first_m), in_group = (uint32_t)(lid - group * group_sz);
    // in_group / rows, without a division (a division of two numbers is some 20 instructions one behind the other)
    static_assert(GROUP_M == 4, "one to four rows");
    const uint32_t n = rows == 3 ? (uint32_t)((uint64_t)in_group * 0x55555556u >> 32) : in_group >> (rows == 4 ? 2 : rows - 1);
    return {range, first_m + (int)(in_group - n * rows), (int)n, true};
}

// How a wave's part of the result, MI x NI accumulators of 16 x 16 (operand roles are swapped, MFMA A = weights, so
// a lane holds four consecutive columns of one row), reaches memory: a pass of rows at a time through LDS, so that
// stores and residual loads are whole row segments.  Straight from the accumulators 16 lanes in a row are 16
// rows apart, and the address pipe takes 64 cycles for an access that it takes 16 for when four lanes share 64
// bytes: 16 instead of 64 bytes a clock for a compute unit, 2 us for the 64 KB of fp32 outputs of a 128 x 128 tile and
// as much for its residual.
template <int MI, int NI, int EPI, int MAX_PASS = 32>
struct WaveOut {
    static constexpr bool RES = EPI == EPI_BIAS_RESID;
    static constexpr int ESZ = RES || EPI == EPI_PARTIAL ? 4 : 2;
    static constexpr int ROW = NI * 16 * ESZ;                          // bytes of a row of the wave's part
    static constexpr int LPR = ROW / 16;                               // lanes to a row
    static constexpr int PITCH = ROW + 16;                             // in LDS: rows shifted by four banks
    static constexpr int PASS = MI % 2 == 0 && ROW <= 128 && MAX_PASS == 32 ? 32 : 16;   // rows of a pass
    static constexpr int NPASS = MI * 16 / PASS, PP = PASS * LPR / 64; // passes; accesses of a lane and pass
    static constexpr size_t LDS_BYTES = 2 * PASS * PITCH;              // two passes take turns
    static_assert(PASS * LPR % 64 == 0, "whole accesses");

#if defined(__HIP_DEVICE_COMPILE__)
    __amdgpu_buffer_rsrc_t c_rs, r_rs;
    f32x4 bias[NI], res[RES ? NPASS : 1][RES ? PP : 1];
    int m0, n0, N, lane;                             // the wave's first row inside the tile, its first column

    // tile_m0: first row of the tile; range_base: rows in front of this K range's sums
    __device__ __forceinline__ void init(const void *Cout, const float *resid, const float *bias_, int tile_m0, int bm, int wm0, int col0,
                                         int M, int N_, size_t range_base, int lane_)
    {
        m0 = wm0; n0 = col0; N = N_; lane = lane_;
        // the tile's rows of C, and of the residual, are buffers that end behind row M - 1
        const uint32_t bytes = (uint32_t)(min(bm, M - tile_m0) * N * ESZ);
        c_rs = make_rsrc(static_cast<const char *>(Cout) + (range_base + tile_m0) * N * ESZ, bytes);
        r_rs = RES ? make_rsrc(resid + (size_t)tile_m0 * N, bytes) : c_rs;
        if (EPI != EPI_PARTIAL) {
            const __amdgpu_buffer_rsrc_t b_rs = make_rsrc(bias_, (uint32_t)N * 4);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                bias[ni] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(b_rs, (n0 + ni * 16 + (lane >> 4) * 4) * 4, 0, 0));
        }
    }
    // bytes from the tile's first row of access p of a pass; a column past N: beyond any end
    __device__ __forceinline__ int offset(int pass, int p) const
    {
        const int c = p * 64 + lane, r = m0 + pass * PASS + c / LPR, n = n0 + (c % LPR) * (16 / ESZ);
        int past = n < N ? 0 : PAST_END;
        asm volatile("" : "+v"(past));               // a value, not a reason to branch
        return (r * N + n) * ESZ + past;
    }
    __device__ __forceinline__ void fetch(int pass)
    {
#pragma unroll
        for (int p = 0; p < PP; ++p)
            res[RES ? pass : 0][RES ? p : 0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r_rs, offset(pass, p), 0, 0));
    }
    // AHEAD passes of the residual have been fetched.  stg: LDS_BYTES of LDS that nobody else uses any more
    template <int AHEAD>
    __device__ __forceinline__ void store(const f32x4 (&acc)[NI][MI], char *stg)
    {
        constexpr int LATE = 2;                      // passes under way once the residual has to be fetched here
        if constexpr (RES && AHEAD < NPASS)
            static_for<(NPASS - AHEAD < LATE ? NPASS - AHEAD : LATE)>([&](auto i) EP_INLINE { fetch(AHEAD + decltype(i)::value); });
        EP_SCHED_FENCE();
        const int l15 = lane & 15, g4 = lane >> 4;
        static_for<NPASS>([&](auto pass_c) EP_INLINE {
            constexpr int pass = decltype(pass_c)::value;
            char *sp = stg + (pass & 1) * (PASS * PITCH);
#pragma unroll
            for (int h = 0; h < PASS / 16; ++h)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    f32x4 c = acc[ni][pass * (PASS / 16) + h];
                    if (EPI != EPI_PARTIAL) c += bias[ni];
                    if (EPI == EPI_BIAS_GELU) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) c[i] = gelu_erf(c[i]);
                    }
                    char *at = sp + (h * 16 + l15) * PITCH + (ni * 16 + g4 * 4) * ESZ;
                    if (ESZ == 4)
                        *reinterpret_cast<f32x4 *>(at) = c;
                    else
                        *reinterpret_cast<uint2 *>(at) = make_uint2(pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3]));
                }
#pragma unroll
            for (int p = 0; p < PP; ++p) {
                const int c = p * 64 + lane;
                u32x4 v = *reinterpret_cast<const u32x4 *>(sp + (c / LPR) * PITCH + (c % LPR) * 16);
                if (RES) v = __builtin_bit_cast(u32x4, __builtin_bit_cast(f32x4, v) + res[RES ? pass : 0][RES ? p : 0]);
                __builtin_amdgcn_raw_buffer_store_b128(v, c_rs, offset(pass, p), 0, 0);
            }
            if constexpr (RES && AHEAD < NPASS && pass + AHEAD + LATE < NPASS) fetch(pass + AHEAD + LATE);
            EP_SCHED_FENCE();
        });
    }
#endif
};

}  // namespace ep_tile
