// Persistent bf16 MFMA GEMM for the large dense layers of an encoder layer
// (paper section 2.1; section 5.1 attributes most of a layer's time to them).
//
//   C[M, N] = A[M, K] . W[N, K]^T + bias[N]   (+ erf GELU | + fp32 residual)
//
// One workgroup per compute unit stays resident and walks a static list of
// 256 x BN output tiles (BN = 256 or 320, chosen per problem by the dispatcher's
// cost model); the K
// loop of consecutive tiles forms one continuous software pipeline, so the
// first K step of the next tile is already in LDS when a tile is stored.
//
// Pipeline (per workgroup, 8 waves, two per SIMD):
//   - K advances in steps of 64 (rows of 128 bytes = whole cache lines, which the
//     L2 -> LDS path moves ~1.6x faster than half lines).  A step's A and W
//     panels go from global memory straight into LDS with buffer_load ... lds
//     (no register staging), two stages.  The A panel has rows of 8 chunks of 16
//     bytes, chunk c of row r at slot c ^ swz(r); the W panel holds the fragments that
//     the weights are stored in (ep_gemm_bf16_tile.h), read lane by lane.
//   - The matrix instruction is v_mfma_f32_16x16x32_bf16: at the power limit
//     the chip runs the same flops about 15 % faster in this form than as
//     32 x 32 x 16.
//   - A step is multiplied in units of 32 columns of each wave.  What a unit has used is free in
//     every wave at the next unit's barrier and is refilled then, a few loads at a time, for
//     the step after next: a load has one to nearly two steps to land, where one
//     barrier a step left the last loads of a step half a step.  Waits count the
//     loads that may still be on their way (Tile::in_flight).
//   - Fragments are read again between the matrix instructions as soon as their last product is out, 8 to
//     12 instructions ahead of their use, so that one step's worth of activations and one unit's of
//     weights is all that registers hold.
// What bounds it: waiting, then the clock.  Under counters (profiles/vit_huge_b64_sq_counters.md) the matrix pipe is busy 58
// (proj and FC2), 62 (FC1) and 67 % (q|k|v) of the clocks of ViT-Huge's layers on 64 images at 1.9 GHz, and no more on 256; a
// loop of nothing but matrix instructions keeps it 97 % busy at the same clock.  The waves spend 42 to 47 % of their cycles
// in s_waitcnt, and all workgroups reach the epilogue together (the residual one moves 6.7 TB/s meanwhile).  The clock
// takes over where a K loop is long: 8192 cubed, launched as 256-wide tiles, 82 % busy at 1.65 GHz, a library kernel 92 % at
// 1.60.  Against the loop with one barrier a step (both in turn, us): 8192 cubed 747 -> 725 (1472 -> 1516 TFLOP/s), 16384 x
// 5120 x 1280 + GELU in 256-wide tiles 198 -> 185, 16384 x 1280 x 5120 + residual 174 -> 166, 16384 x 1280 x 1280 + residual
// 70.3 -> 65.6, 65792 rows 744 -> 720 and 774 -> 730.  Moving its barrier, its loads or its reads by a few instructions, wave
// priorities and wider groups of tile rows changed nothing.
//   Its waits count loads and stores in the order in which they are sent out: panel loads to LDS, the epilogue's stores, the
// next tile's loads.  Residual loads (to registers) lie between stores that use them, so none is under way when a step counts.
// Epilogue: 32 x 32 blocks of accumulators (+bias, GELU) are transposed through the
// W part of the LDS stage the tile's last step has just retired (4 KB per wave),
// so that global stores and residual loads are whole row segments; the refill of
// the stage's A part for the next tile is already under way meanwhile (issued
// before the epilogue, like after any other step), the rest follows it.  The next tile's first step does
// not wait for the stores.  The tile's bias values wait in LDS (loaded there during the K loop).
//
// Operand roles are swapped (MFMA A = W fragment, B = activation fragment) so
// that a lane owns 4 consecutive output columns of one row.
//
// Workgroup w runs on XCD w % 8 (round-robin dispatch); in every round the 32
// workgroups of an XCD take 32 consecutive tiles of an order that walks groups
// of 4 tile rows column by column, so that they share A and W panels in L2.
//
// Requirements: K % 64 == 0, K >= 128, N % 16 == 0, N < 2^20; M*K*2, N*K*2 < 2^31.  Rows
// past M and columns past N are read as zeros (per-lane buffer offsets beyond
// the end of the buffer) and never stored.  `m_rows` <= M limits the rows the
// tile walk computes.  The remaining rows are left to the caller, or, with
// `fuse_tail`, computed in the same launch: before its first tile a workgroup
// takes narrow tiles of rows [m_rows, M) (the short-M tile routine: 64, 32 or
// 16 rows by 32 columns, as narrow as it takes to give every workgroup one; K
// dealt to the 8 waves, fixed-order sum through LDS), which saves the launch and
// ramp of a second kernel when M is a few rows more than a multiple of 256.
#include "ep_gemm_bf16_tile.h"
#include "ep_gemm_bf16_skinny_tile.h"
#include "ep_launch.h"

namespace {

using namespace ep_tile;

constexpr int BM = 256, STAGES = 2;
constexpr int NW = 8;                                // waves, 4 x 2: 64 rows by half the columns each

// What a wave may have in flight.  A tile is 256 x BN, BN = 64 NU; a K step is multiplied in NU units of 32 columns of the
// wave.  Region j of a stage's W panel is what the waves read for their unit j: 8 KB, a load to a wave.
template <int BN_>
struct Tile {
    static constexpr int BN = BN_, NU = BN / 64;
    static constexpr int A_STAGE = BM * CPR, W_STAGE = BN * CPR;      // uint4 per stage and operand
    static constexpr int STAGE_U4 = A_STAGE + W_STAGE;
    static constexpr int LDA = BM / 8 / NW;                           // A loads of a wave and step, 64 rows each
    static constexpr size_t SMEM = (size_t)(STAGES * STAGE_U4 + BN / 4) * sizeof(uint4);   // stages + the tile's bias
    static_assert(BN % 64 == 0 && NU >= 4 && W_STAGE >= NW * 256, "4 KB of epilogue staging per wave in the W part of a stage");
    // A loads that go out in unit j, and in units 1 .. j - 1
    static constexpr int a_in(int j) { return j < 1 ? 0 : (LDA * j + NU - 2) / (NU - 1) - (LDA * (j - 1) + NU - 2) / (NU - 1); }
    static constexpr int a_before(int j) { return j <= 1 ? 0 : a_in(j - 1) + a_before(j - 1); }
    // Loads of step k go out while step k - 2 is multiplied (the A panel and region j - 1 of W in unit j >= 1, once every
    // wave has passed that far) and in unit 0 of step k - 1 (region NU - 1); in the last step of a tile all W regions
    // but that one wait until its epilogue, which stages through them, is over.  The number of loads that may be in flight at
    // the barrier of unit j: those behind the ones that unit reads (region j + 1, or the next step's region 0 and A
    // panel), in whichever of the two orders leaves fewer.
    static constexpr int in_flight(int j, bool last)
    {
        const int here = (j >= 1 ? 1 : 0) + a_before(j) + (last || j < 2 ? 0 : j - 1);          // of this step so far
        if (j == NU - 1) return 1 + here;
        return (j + 1 < NU - 1 ? NU - 2 - j : 0) + LDA + NU - 1 + here;
    }
};
typedef Tile<256> Tile256;
typedef Tile<320> Tile320;

}  // namespace

// Measurement: the shader-cycle counter and the constant 100 MHz counter read by workgroup 0 at the
// start ([0], [1]) and at the end ([2], [3]) of the most recent launch on this device; their ratio
// is the shader clock that launch ran at (ep_gemm_clock_sample).
static __device__ unsigned long long g_clock_sample[4];

namespace {

enum StepKind { STEP_FIRST, STEP_MIDDLE, STEP_LAST };               // of a tile's K steps

template <class T, int EPI>
__global__ __launch_bounds__(NW * 64, 1) void gemm_bf16_persistent_kernel(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ W, const float *__restrict__ bias,
    const float *resid, void *Cout, int M, int m_rows, int N, int K, int tiles_m, int tiles_n, int tail_rows, int tail_tm)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BN = T::BN, NU = T::NU, MI = 2, NI = NU;            // 32 x 32 blocks of the wave tile (epilogue)
    constexpr int A_STAGE = T::A_STAGE, STAGE_U4 = T::STAGE_U4, LDA = T::LDA;
    constexpr bool RESID = EPI == EPI_BIAS_RESID;
    constexpr int ESZ = RESID ? 4 : 2, STORES = MI * NI * (RESID ? 4 : 2);      // of a wave and tile

    extern __shared__ uint4 lds[];                   // [STAGES][A panel | W panel]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: wave-derived addressing stays scalar
    if (blockIdx.x == 0 && tid == 0) {
        g_clock_sample[0] = clock64();
        g_clock_sample[1] = wall_clock64();
    }
    const int wm0 = (wave >> 1) * 64, wn0 = (wave & 1) * (NU * 32);

    // ---- this workgroup's tile list: tile j has logical id j*G + (w%8)*(G/8) + w/8
    const int G = gridDim.x;                         // multiple of 8
    const int total = tiles_m * tiles_n;
    const int first_id = (int)(blockIdx.x % NUM_XCD) * (G / NUM_XCD) + (int)(blockIdx.x / NUM_XCD);
    if (first_id >= total && tail_rows == 0) return;
    const int n_my = first_id < total ? (total - first_id + G - 1) / G : 0;
    const int KT = K / BK;

    auto tile_origin = [&](int seq, int &m0, int &n0) {
        const int id = seq * G + first_id;
        const int group_sz = GROUP_M * tiles_n;
        const int group = id / group_sz;
        const int fm = group * GROUP_M;
        const int rows = min(GROUP_M, tiles_m - fm);
        const int in_group = id - group * group_sz;
        m0 = (fm + in_group % rows) * BM;
        n0 = (in_group / rows) * BN;
    };

    // ---- load stream: two K steps ahead of the multiply stream.  The tile's panels are buffers that end behind row M - 1
    // and column N - 1 (whole weight fragments, so that check is wave-uniform); past the last tile they are empty.
    const int row_a = wave * 8 + (lane >> 3);        // load i fills panel rows i * 64 + wave * 8 .. + 7
    const int off_a = row_a * K * 2 + ((lane & 7) ^ swz(row_a)) * 16;
    const int lane16 = lane * 16;
    const int w_col = (wave >> 2) * (32 * NU) + (wave >> 1 & 1) * 16;  // region j: the fragment of columns w_col + j * 32 .. + 15
    const int w_frag = w_col * K * 2 + (wave & 1) * FRAG_BYTES;        // .. of slice wave % 2, bytes from the tile's first
    const char *a_base = nullptr, *w_base = nullptr;
    uint32_t a_bytes = 0;
    int w_cols = 0;                                  // valid columns of the tile
    int ld_seq = 0, ld_kt = 0, ld_stage = 0;
    auto set_load_tile = [&](int seq) EP_INLINE {
        int m0 = 0, n0 = 0;
        const bool live = seq < n_my;
        if (live) tile_origin(seq, m0, n0);
        a_base = reinterpret_cast<const char *>(A) + (size_t)m0 * K * 2;
        w_base = reinterpret_cast<const char *>(W) + (size_t)n0 * K * 2;
        a_bytes = live ? (uint32_t)(M - m0) * (uint32_t)K * 2u : 0u;
        w_cols = live ? N - n0 : 0;
    };
    auto issue_a = [&](int i) EP_INLINE {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(a_base, a_bytes), (lds_ptr)(lds + ld_stage * STAGE_U4 + (i * NW + wave) * 64), 16,
                                                 off_a + i * (128 * K), ld_kt * (BK * 2), 0, 0);
    };
    auto issue_w = [&](int j, int kt, int stage) EP_INLINE {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(w_base, w_col + j * 32 < w_cols ? 0x7FFFFFFFu : 0u),
                                                 (lds_ptr)(lds + stage * STAGE_U4 + A_STAGE + (j * NW + wave) * 64), 16, lane16,
                                                 w_frag + j * (64 * K) + kt * (NS * FRAG_BYTES), 0, 0);
    };
    auto advance_load = [&]() EP_INLINE {
        ld_stage ^= 1;
        if (++ld_kt == KT) {
            ld_kt = 0;
            set_load_tile(++ld_seq);
        }
    };

    // ---- fragments and accumulators (v_mfma_f32_16x16x32_bf16).  A unit multiplies two weight fragments a slice (32
    // columns of the wave) with the four activation fragments a slice of its 64 rows, weight fragment by weight fragment:
    // each is read again, for the next unit, as soon as its four products are out, 12 matrix instructions ahead of
    // its use; in the last unit of a step the activation fragments follow each other in the same way, eight ahead.
    int p_off[NS], h_off;
    auto derive_read_offsets = [&]() EP_INLINE {     // again after every epilogue: no registers while a tile is stored
        int le = lane;
        asm volatile("" : "+v"(le));
        const int l15 = le & 15, g4 = le >> 4;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) p_off[sl] = (wm0 + l15) * CPR + ((sl * 4 + kchunk(g4)) ^ swz(l15));
        h_off = A_STAGE + (wave & 1) * 256 + le;
    };
    derive_read_offsets();
    bf16x8 fp[4][NS], fh[2][NS];
    f32x4 acc[2 * NU][4];
    auto read_p = [&](const uint4 *stage, int p, int sl) EP_INLINE {
        fp[p][sl] = __builtin_bit_cast(bf16x8, stage[p_off[sl] + p * 16 * CPR]);
    };
    auto read_h = [&](const uint4 *stage, int j, int h, int sl) EP_INLINE {
        fh[h][sl] = __builtin_bit_cast(bf16x8, stage[h_off + (j * NW + h * 2 + sl) * 64]);
    };

    // The BN bias values of a tile sit in LDS behind the stages, brought there with 4-byte
    // global -> LDS loads when the tile before it is stored (columns past N read as zeros), so the
    // epilogue gets its lane's four values with one LDS read and no select between the quarters of
    // the wave; the loads ride on the K loop's own waits.
    float *bias_lds = reinterpret_cast<float *>(lds + STAGES * STAGE_U4);
    const __amdgpu_buffer_rsrc_t b_rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(bias), 0, N * 4, 0x00020000);
    auto issue_bias = [&](int seq) {                 // wave w brings columns w*64 .. w*64+63 of tile seq
        if (wave < BN / 64 && seq < n_my) {
            int m0, n0;
            tile_origin(seq, m0, n0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rs, (lds_ptr)(bias_lds + wave * 64), 4, (n0 + wave * 64 + lane) * 4, 0,
                                                     0, 0);
        }
    };
    auto bias4 = [&](int col, int g4) {              // col: column inside the tile, a multiple of 16; g4 = lane / 16
        return *reinterpret_cast<const float4 *>(bias_lds + col + 4 * g4);
    };

    // ---- epilogue of the tile at (m0, n0); the W part of `stage` has just been retired and is free LDS.
    // It goes by 32 x 32 blocks: four accumulators (wj, aj) each.  The tile's rows of C (and of the residual) are buffers
    // that end behind row m_rows - 1; columns past N lie past any end.  No branches: the next step counts the stores.
    auto epilogue = [&](int m0, int n0, int stage) EP_INLINE {
        // the lane-dependent addressing of the epilogue is derived afresh for every tile from a lane index
        // the compiler cannot see through: otherwise it computes all of it ahead of the K loop, where the
        // values do not fit in registers next to the accumulators and come back from scratch memory
        int le = lane;
        asm volatile("" : "+v"(le));
        const int l15 = le & 15, g4 = le >> 4, lane = le;
        uint4 *stg = lds + stage * STAGE_U4 + A_STAGE + wave * 256; // 4 KB of the W panel's part
        const uint32_t tile_bytes = (uint32_t)(min(BM, m_rows - m0) * N * ESZ);
        const __amdgpu_buffer_rsrc_t c_rs = make_rsrc(reinterpret_cast<const char *>(Cout) + (size_t)m0 * N * ESZ, tile_bytes);
        const __amdgpu_buffer_rsrc_t r_rs = RESID ? make_rsrc(resid + (size_t)m0 * N, tile_bytes) : c_rs;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int nblk = n0 + wn0 + ni * 32, mblk = wm0 + mi * 32;
                float4 bq[2];
#pragma unroll
                for (int wj = 0; wj < 2; ++wj) bq[wj] = bias4(wn0 + ni * 32 + wj * 16, g4);
                if (RESID) {
                    // block [32 m][32 n] fp32: rows of 128 B = 8 chunks of 4 floats
#pragma unroll
                    for (int aj = 0; aj < 2; ++aj)
#pragma unroll
                        for (int wj = 0; wj < 2; ++wj) {
                            const f32x4 c = acc[ni * 2 + wj][mi * 2 + aj];
                            const float4 bb = bq[wj];
                            const int r = aj * 16 + l15;
                            *reinterpret_cast<float4 *>(&stg[r * 8 + ((wj * 4 + g4) ^ (r & 7))]) =
                                make_float4(c[0] + bb.x, c[1] + bb.y, c[2] + bb.z, c[3] + bb.w);
                        }
                    const int rrow = lane >> 3, rc = lane & 7;      // read-back: 8 rows x 8 chunks per pass
                    const int n = nblk + rc * 4, past = n < N ? 0 : PAST_END;
                    f32x4 v[4], x[4];
                    int off[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const int r = p * 8 + rrow;
                        off[p] = ((mblk + r) * N + n) * 4 + past;
                        x[p] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r_rs, off[p], 0, 0));
                        v[p] = *reinterpret_cast<const f32x4 *>(&stg[r * 8 + (rc ^ (r & 7))]);
                    }
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[p] + x[p]), c_rs, off[p], 0, 0);
                } else {
                    // block [32 m][32 n] bf16: rows of 64 B = 4 chunks of 8 bf16; chunk c of row r sits at slot
                    // c ^ ((r >> 2) & 3): four rows span the 64 banks, so the 8-byte writes of 32 rows meet two to
                    // a bank (the best a 64-byte row stride allows) and the 16-byte reads of 4 rows not at all
#pragma unroll
                    for (int aj = 0; aj < 2; ++aj)
#pragma unroll
                        for (int wj = 0; wj < 2; ++wj) {
                            const f32x4 c = acc[ni * 2 + wj][mi * 2 + aj];
                            const float4 bb = bq[wj];
                            float v0 = c[0] + bb.x, v1 = c[1] + bb.y, v2 = c[2] + bb.z, v3 = c[3] + bb.w;
                            if (EPI == EPI_BIAS_GELU) {
                                v0 = gelu_erf(v0); v1 = gelu_erf(v1); v2 = gelu_erf(v2); v3 = gelu_erf(v3);
                            }
                            uint2 o;
                            o.x = pack_bf16x2(v0, v1);
                            o.y = pack_bf16x2(v2, v3);
                            const int r = aj * 16 + l15;
                            reinterpret_cast<uint2 *>(&stg[r * 4 + ((wj * 2 + (g4 >> 1)) ^ ((r >> 2) & 3))])[g4 & 1] = o;
                        }
                    const int rrow = lane >> 2, rc = lane & 3;      // read-back: 16 rows x 4 chunks per pass
                    const int n = nblk + rc * 8, past = n < N ? 0 : PAST_END;
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const int r = p * 16 + rrow;
                        const u32x4 v = *reinterpret_cast<const u32x4 *>(&stg[r * 4 + (rc ^ ((r >> 2) & 3))]);
                        __builtin_amdgcn_raw_buffer_store_b128(v, c_rs, ((mblk + r) * N + n) * 2 + past, 0, 0);
                    }
                }
            }
        }
    };

    // ---- prologue: step 0 into stage 0
    set_load_tile(0);
    issue_bias(0);
#pragma unroll
    for (int i = 0; i < LDA; ++i) issue_a(i);
#pragma unroll
    for (int j = 0; j < NU; ++j) issue_w(j, 0, 0);
    advance_load();

    // ---- rows [m_rows, m_rows + tail_rows): tail_tm x 32 tiles, dealt to the workgroups from the end
    // of the tile order backwards (those are the ones with a tile less when the tiles do not divide).  They come
    // first, through the stage that is still empty, while step 0 is on its way: after the last tile their loads
    // queued behind that tile's stores (both builds in turn: three layers of ViT-Huge on 256 images, 256 such rows,
    // 7.93 -> 7.86 ms; 32 layers on 64 images, 64 rows, 21.27 -> 21.20; 3500 launches with tails of up to 511 rows 0.6 %
    // faster on average).
    if (tail_rows > 0) {
        const int tn = (N + ep_skinny::TN - 1) / ep_skinny::TN;
        const int units = tn * ((tail_rows + tail_tm - 1) / tail_tm);
        float *scratch = reinterpret_cast<float *>(lds + STAGE_U4);
        static_assert(STAGE_U4 * sizeof(uint4) >= ep_skinny::SMEM, "a stage holds the tail's partial sums");
        for (int u = G - 1 - first_id; u < units; u += G) {
            const int tm0 = m_rows + (u / tn) * tail_tm, tn0 = (u % tn) * ep_skinny::TN;
            if (tail_tm == 64)
                ep_skinny::tile<EPI, 64, true>(A, W, bias, resid, Cout, m_rows + tail_rows, N, K, tm0, tn0, scratch);
            else if (tail_tm == 32)
                ep_skinny::tile<EPI, 32, true>(A, W, bias, resid, Cout, m_rows + tail_rows, N, K, tm0, tn0, scratch);
            else
                ep_skinny::tile16<EPI>(A, W, bias, resid, Cout, m_rows + tail_rows, N, K, tm0, tn0, scratch);
            __syncthreads();
        }
    }

    // ---- step 1 into stage 1, all but the region that step 0 sends for; once step 0 is there, the first fragments
#pragma unroll
    for (int i = 0; i < LDA; ++i) issue_a(i);
#pragma unroll
    for (int j = 0; j < NU - 1; ++j) issue_w(j, ld_kt, ld_stage);
    EP_WAIT_VMCNT(NU - 1 + LDA);                     // (a tile's first step does not wait for its own panels, see below)
    EP_WAIT_LGKMCNT0();
    __builtin_amdgcn_s_barrier();
    EP_SCHED_FENCE();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) read_h(lds, 0, h, sl);
#pragma unroll
    for (int sl = 0; sl < NS; ++sl)
#pragma unroll
        for (int p = 0; p < 4; ++p) read_p(lds, p, sl);
    EP_SCHED_FENCE();

    int stage = 0;
    // One step.  The load stream stands at the step after this one when it begins (its region NU - 1 goes out first) and moves
    // on behind unit 0.
    auto step = [&](auto kind_c) EP_INLINE {
        constexpr int KIND = decltype(kind_c)::value;
        constexpr bool LAST = KIND == STEP_LAST;
        const uint4 *cur = lds + stage * STAGE_U4;
        const uint4 *nxt = lds + (stage ^ 1) * STAGE_U4;
        static_for<NU>([&](auto j_c) EP_INLINE {
            constexpr int j = decltype(j_c)::value;
            constexpr bool end = j == NU - 1;
            static_for<16>([&](auto m_c) EP_INLINE {
                constexpr int m = decltype(m_c)::value, h = m >> 3, sl = m >> 2 & 1, p = (m >> 2 & 1) ? 3 - (m & 3) : m & 3;
                f32x4 &c = acc[2 * j + h][p];
                if constexpr (KIND == STEP_FIRST && sl == 0)
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fh[h][sl], fp[p][sl], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                else
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fh[h][sl], fp[p][sl], c, 0, 0, 0);
                EP_SCHED_FENCE();
                if constexpr (m == 3) {
                    // what this unit reads has landed, in everyone's part; everyone is done with what unit j - 1
                    // multiplied.  In the first step of a tile the stores of the tile before it may still be on their way (before the first
                    // tile there are none, and step 0 has landed).
                    if constexpr (LAST && end) EP_WAIT_LGKMCNT0();         // the stage's W part becomes staging
                    EP_WAIT_VMCNT(T::in_flight(j, LAST) + (KIND == STEP_FIRST && !end ? STORES : 0));
                    __builtin_amdgcn_s_barrier();
                    EP_SCHED_FENCE();
                }
                if constexpr ((m & 3) == 3) {
                    if constexpr (end) read_h(nxt, 0, h, sl);
                    else read_h(cur, j + 1, h, sl);
                }
                if constexpr (end && h == 1) read_p(nxt, p, sl);
                if constexpr (j == 0 && m == 5) {
                    issue_w(NU - 1, ld_kt, ld_stage);
                    advance_load();
                }
                if constexpr (j > 0 && m >= 5 && (m & 1)) {
                    constexpr int q = (m - 5) / 2;
                    if constexpr (q < T::a_in(j)) issue_a(T::a_before(j) + q);
                    else if constexpr (q == T::a_in(j) && !LAST) issue_w(j - 1, ld_kt, ld_stage);
                }
                EP_SCHED_FENCE();
            });
        });
        stage ^= 1;
    };
    for (int c_seq = 0; c_seq < n_my; ++c_seq) {
        step(std::integral_constant<int, STEP_FIRST>{});
        for (int kt = 1; kt < KT - 1; ++kt) step(std::integral_constant<int, STEP_MIDDLE>{});
        step(std::integral_constant<int, STEP_LAST>{});
        int m0, n0;
        tile_origin(c_seq, m0, n0);
        epilogue(m0, n0, stage ^ 1);
        EP_WAIT_LGKMCNT0();
        __builtin_amdgcn_s_barrier();                // every wave is done with the staging area and the bias
#pragma unroll
        for (int j = 0; j < NU - 1; ++j) issue_w(j, ld_kt, ld_stage);
        issue_bias(c_seq + 1);
        derive_read_offsets();
    }
    EP_WAIT_VMCNT(0);                                // drain the last (empty) loads before LDS is released
    if (blockIdx.x == 0 && tid == 0) {
        g_clock_sample[2] = clock64();
        g_clock_sample[3] = wall_clock64();
    }
#endif
}

// one resident workgroup per compute unit of the current device, a multiple of the number of XCDs
hipError_t resident_grid(int *grid)
{
    int cus = 0;
    const hipError_t e = ep_device_cu_count(&cus);
    if (e != hipSuccess) return e;
    *grid = cus / NUM_XCD * NUM_XCD;
    if (*grid < NUM_XCD) *grid = NUM_XCD;
    return hipSuccess;
}

template <class T, int EPI>
hipError_t launch_persistent(const uint16_t *A, const uint16_t *W, const float *bias, const float *resid,
                             void *C, int M, int m_rows, int N, int K, int tail_rows, int g_grid, hipStream_t s)
{
    auto kern = gemm_bf16_persistent_kernel<T, EPI>;
    static EpSmemLimit smem_limit;
    const hipError_t e = smem_limit.ensure(reinterpret_cast<const void *>(kern), (int)T::SMEM);
    if (e != hipSuccess) return e;
    const int tiles_m = (m_rows + BM - 1) / BM, tiles_n = (N + T::BN - 1) / T::BN;
    hipLaunchKernelGGL(kern, dim3(g_grid), dim3(NW * 64), T::SMEM, s, A, W, bias, resid, C, M, m_rows, N, K,
                       tiles_m, tiles_n, tail_rows, tail_rows ? ep_bf16_gemm_tail_tile_rows(tail_rows, N, g_grid) : 0);
    return hipGetLastError();
}

template <class T>
hipError_t launch_tile(const uint16_t *A, const uint16_t *W, const float *bias, const float *resid, void *C,
                       int M, int m_rows, int N, int K, int epi, int tail_rows, hipStream_t s)
{
    int g_grid = 0;
    const hipError_t e = resident_grid(&g_grid);
    if (e != hipSuccess) return e;
    switch (epi) {
    case EPI_BIAS: return launch_persistent<T, EPI_BIAS>(A, W, bias, resid, C, M, m_rows, N, K, tail_rows, g_grid, s);
    case EPI_BIAS_GELU: return launch_persistent<T, EPI_BIAS_GELU>(A, W, bias, resid, C, M, m_rows, N, K, tail_rows, g_grid, s);
    case EPI_BIAS_RESID: return launch_persistent<T, EPI_BIAS_RESID>(A, W, bias, resid, C, M, m_rows, N, K, tail_rows, g_grid, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// Rows per tile (64, 32 or 16; all 32 columns wide) for the rows past the tile walk: the fewest rounds over the
// workgroups, then the fewest bytes a workgroup pulls per tile (rows + 32 panel rows of K elements).
int ep_bf16_gemm_tail_tile_rows(int tail_rows, int N, int wgs)
{
    const int tn = (N + 31) / 32;
    int best = 64;
    int64_t best_cost = -1;
    for (int tm : {64, 32, 16}) {
        const int units = tn * ((tail_rows + tm - 1) / tm);
        const int64_t cost = (int64_t)((units + wgs - 1) / wgs) * (tm + 32);
        if (best_cost < 0 || cost < best_cost) { best = tm; best_cost = cost; }
    }
    return best;
}

hipError_t ep_bf16_gemm_persistent_clock(double *shader_mhz, double *seconds)
{
    unsigned long long h[4] = {0, 0, 0, 0};
    const hipError_t e = hipMemcpyFromSymbol(h, HIP_SYMBOL(g_clock_sample), sizeof(h));
    if (e != hipSuccess) return e;
    const double cycles = (double)(h[2] - h[0]), ticks = (double)(h[3] - h[1]);     // ticks of 10 ns
    if (h[3] <= h[1] || h[2] <= h[0]) return hipErrorNotReady;      // no launch has finished on this device yet
    *shader_mhz = cycles / ticks * 100.0;
    *seconds = ticks * 1e-8;
    return hipSuccess;
}

bool ep_bf16_gemm_persistent_supported(int64_t M, int N, int K)
{
    // N: the epilogue addresses a tile's rows of C with 32 bits and sends columns past N beyond them (PAST_END)
    return M > 0 && N > 0 && N < MAX_TILE_N && K >= 2 * BK && K % BK == 0 && N % 16 == 0 &&
           M * (int64_t)K * 2 < 0x7FFFFFF0ll && (int64_t)N * K * 2 < 0x7FFFFFF0ll && M * (int64_t)N < (1ll << 31);
}

int ep_bf16_gemm_persistent_workgroups()
{
    int g = 0;
    return resident_grid(&g) == hipSuccess ? g : 256;
}

// tile_bn: 256 or 320.  m_rows <= M: the tile walk covers rows [0, m_rows);
// fuse_tail: rows [m_rows, M) are computed by the same launch as 64 x 32 tiles.
hipError_t ep_bf16_gemm_persistent(const uint16_t *A, const uint16_t *W, const float *bias, const float *resid,
                                   void *C, int64_t M, int64_t m_rows, int N, int K, int epi, int tile_bn,
                                   bool fuse_tail, hipStream_t s)
{
    if (!ep_bf16_gemm_persistent_supported(M, N, K) || m_rows < 0 || m_rows > M) return hipErrorInvalidValue;
    if (epi == EPI_BIAS_RESID && !resid) return hipErrorInvalidValue;
    if (m_rows == 0) return hipSuccess;
    const int tail = fuse_tail ? (int)(M - m_rows) : 0;
    if (tile_bn == 320) return launch_tile<Tile320>(A, W, bias, resid, C, (int)M, (int)m_rows, N, K, epi, tail, s);
    if (tile_bn == 256) return launch_tile<Tile256>(A, W, bias, resid, C, (int)M, (int)m_rows, N, K, epi, tail, s);
    return hipErrorInvalidValue;
}
