// fp32 path of a ViT encoder layer (paper section 2.1) for configurations where
// exactness matters more than speed: fp32 operands, products and sums everywhere.
// The matrix products run on v_mfma_f32_16x16x4_f32 (fp32 in, fp32 accumulation,
// twice the vector ALU's unpacked rate):
//   dense layers   few tiles: 16 x 16 to 32 x 32 outputs per workgroup, K dealt to its four waves, each with its own part
//                  of LDS, LayerNorm of the input rows done on the way where it comes first;
//                  many rows behind a LayerNorm, K <= 384: 64 rows per workgroup, normalised and kept in registers;
//                  many tiles: 64 x 32 outputs, K panels through LDS;
//   attention      16 queries to a wave, online softmax: 16 to a workgroup whose four waves share the keys and merge at
//                  the end while queries are few, else 64 to a workgroup whose waves each meet all keys.
// Plain vector-ALU kernels stand in where rows are not made of whole, aligned 16-byte pieces (K, D or d_head not
// a multiple of 4, d_head above 128).
#include "ep_kernels.h"
#include "ep_launch.h"

namespace {

constexpr int WAVE = 64;

__device__ inline float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, WAVE);
    return v;
}

__device__ inline float wave_max(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, WAVE));
    return v;
}

__device__ inline float gelu_erf(float u) { return 0.5f * u * (1.0f + erff(u * 0.70710678118654752440f)); }

// ---------------------------------------------------------------- LayerNorm
__global__ __launch_bounds__(256) void ln_f32_kernel(const float *__restrict__ x, int64_t ldx,
                                                     const float *__restrict__ g,
                                                     const float *__restrict__ b, float eps,
                                                     float *__restrict__ y, int64_t rows, int D)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t row = (int64_t)blockIdx.x * (256 / WAVE) + (threadIdx.x / WAVE);
    if (row >= rows) return;
    const float *xr = x + row * ldx;
    float s = 0.f;
    for (int d = lane; d < D; d += WAVE) s += xr[d];
    const float mean = wave_sum(s) / (float)D;
    float v = 0.f;
    for (int d = lane; d < D; d += WAVE) {
        const float c = xr[d] - mean;
        v += c * c;
    }
    const float inv = 1.0f / sqrtf(wave_sum(v) / (float)D + eps);
    float *yr = y + row * D;
    for (int d = lane; d < D; d += WAVE) yr[d] = (xr[d] - mean) * inv * g[d] + b[d];
}

// The same for rows of whole 16-byte pieces, the row in registers: one pass over memory.  NV float4 per lane.
template <int NV>
__global__ __launch_bounds__(256) void ln_f32_vec_kernel(const float *__restrict__ x, int64_t ldx, const float *__restrict__ g,
                                                         const float *__restrict__ b, float eps, float *__restrict__ y,
                                                         int64_t rows, int D)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t row = (int64_t)blockIdx.x * (256 / WAVE) + (threadIdx.x / WAVE);
    if (row >= rows) return;
    const float4 *xr = reinterpret_cast<const float4 *>(x + row * ldx);
    const float4 *g4 = reinterpret_cast<const float4 *>(g), *b4 = reinterpret_cast<const float4 *>(b);
    const int nvec = D >> 2;
    float4 v[NV], gg[NV], bb[NV];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = lane + i * WAVE;
        const bool in = c < nvec;
        v[i] = in ? xr[c] : make_float4(0.f, 0.f, 0.f, 0.f);
        gg[i] = in ? g4[c] : v[i];
        bb[i] = in ? b4[c] : v[i];
        s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    }
    const float mean = wave_sum(s) / (float)D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        if (lane + i * WAVE < nvec) {
            v[i].x -= mean; v[i].y -= mean; v[i].z -= mean; v[i].w -= mean;
            q += (v[i].x * v[i].x + v[i].y * v[i].y) + (v[i].z * v[i].z + v[i].w * v[i].w);
        }
    }
    const float inv = 1.0f / sqrtf(wave_sum(q) / (float)D + eps);
    float4 *yr = reinterpret_cast<float4 *>(y + row * D);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = lane + i * WAVE;
        if (c < nvec)
            yr[c] = make_float4(v[i].x * inv * gg[i].x + bb[i].x, v[i].y * inv * gg[i].y + bb[i].y,
                                v[i].z * inv * gg[i].z + bb[i].z, v[i].w * inv * gg[i].w + bb[i].w);
    }
}

// ------------------------------------------------------------- dense layers on the matrix cores
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float frag4 __attribute__((ext_vector_type(4)));   // one 16-byte piece of a row: four k, one per MFMA

// v_mfma_f32_16x16x4_f32, four of them: slot g = lane / 16 of step j holds k = 4 g + j of a 16-wide slice (any
// assignment does, as long as both operands share it), so one 16-byte piece per lane feeds four steps
__device__ inline f32x4 mfma_slice(frag4 a, frag4 b, f32x4 c)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], c, 0, 0, 0);
    return c;
}

constexpr int F32_OOB = 0x7FFFFFF0;

#if defined(__HIP_DEVICE_COMPILE__)   // buffer-resource builtins exist only in the device pass
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const float *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, bytes, 0x00020000);
}
__device__ inline frag4 load_piece(__amdgpu_buffer_rsrc_t rs, int byte)
{
    return __builtin_bit_cast(frag4, __builtin_amdgcn_raw_buffer_load_b128(rs, byte, 0, 0));
}
#endif

// bias, GELU or residual, store of four consecutive columns n .. n+3 of row m; `vec`: N % 4 == 0 and 16-byte
// aligned resid and C
template <int EPI>
__device__ inline void store_four(const float (&v)[4], const float *bias, const float *resid, float *C, int64_t m, int n, int N,
                                  bool vec)
{
    const int64_t off = m * N + n;
    if (vec) {
        const float4 bb = *reinterpret_cast<const float4 *>(bias + n);
        float4 r = make_float4(v[0] + bb.x, v[1] + bb.y, v[2] + bb.z, v[3] + bb.w);
        if (EPI == EPI_BIAS_GELU) { r.x = gelu_erf(r.x); r.y = gelu_erf(r.y); r.z = gelu_erf(r.z); r.w = gelu_erf(r.w); }
        if (EPI == EPI_BIAS_RESID) {
            const float4 x = *reinterpret_cast<const float4 *>(resid + off);
            r.x += x.x; r.y += x.y; r.z += x.z; r.w += x.w;
        }
        *reinterpret_cast<float4 *>(C + off) = r;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (n + i >= N) break;
            float r = v[i] + bias[n + i];
            if (EPI == EPI_BIAS_GELU) r = gelu_erf(r);
            if (EPI == EPI_BIAS_RESID) r += resid[off + i];
            C[off + i] = r;
        }
    }
}

// Workgroup -> tile, columns fastest: workgroup w runs on XCD w % 8 (round-robin dispatch), and each XCD takes a
// contiguous run of tiles, as long as its share of the workgroups, so that the tiles of a row panel meet in one L2.  One
// workgroup to a tile and none beside (a grid may not have 2^32 threads).
__device__ inline void f32_tile_of(int tiles_n, int tiles, int *tm, int *tn)
{
    const int xcd = blockIdx.x % 8, id = xcd * (tiles / 8) + min(xcd, tiles % 8) + (int)(blockIdx.x / 8);
    *tm = id / tiles_n;
    *tn = id - *tm * tiles_n;
}

// Few tiles: one 16 MR x 16 MC tile per workgroup.  Such a launch is a chain of latencies (a 65-row layer has 60 to
// 240 tiles of 16 x 16), so no wave waits for another on the way in: the 16-wide K slices are dealt to the four waves
// and each brings its own from memory into its own part of LDS (buffer_load ... lds, R slices ahead, four lanes to
// a 64-byte row piece; fragments loaded straight into registers would have every lane of a quarter wave on a row of its
// own, four times the cache lines per load: 17.2 against 10.9 us at 1576 x 192 x 768), and the four sums are added
// in wave order at the end.  Two layers on one 65 x 192 image: 229 us on the vector ALU, 64 x 64 tiles, before; 42 now.
// LN > 0: A is the residual stream and its rows are normalised first (all K in LDS at once: LN slices per wave,
// K <= 64 LN); every workgroup does that for its own rows, which costs two small exchanges through LDS and saves
// the launch of LayerNorm and a trip through memory.
// LDS rows are 64 bytes, four rows to all the banks: piece c of row r sits at slot c ^ (r >> 2 & 3), so that the
// 16-byte reads of 16 rows meet no bank twice.
template <int MR, int MC, int LN>
struct F32Direct {
    static constexpr int TR = 16 * MR, TC = 16 * MC, R = LN ? LN : (MR + MC == 2 ? 6 : 4), LP = TC + 4;
    static constexpr int SLICE = (TR + TC) * 4;                         // 16-byte pieces of a slice: A rows, then W rows
    static constexpr size_t ring = (size_t)4 * R * SLICE * 16, sums = (size_t)4 * TR * LP * 4;
    static constexpr size_t smem = ring > sums ? ring : sums;       // the sums reuse the ring
};

template <int MR, int MC, int EPI, int LN>
__global__ __launch_bounds__(256) void gemm_f32_direct_kernel(const float *__restrict__ A, const float *__restrict__ W, int M, int N,
                                                              int K, int tiles_n, int tiles, int vec,
                                                              const float *__restrict__ ln_g, const float *__restrict__ ln_b,
                                                              const float *__restrict__ bias, const float *resid, float *C, float eps)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using S = F32Direct<MR, MC, LN>;
    constexpr int TR = S::TR, TC = S::TC, R = S::R;
    extern __shared__ uint4 lds_raw[];
    __shared__ float stat[2][4][TR];
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l15 = lane & 15, g = lane >> 4;
    int tm, tn;
    f32_tile_of(tiles_n, tiles, &tm, &tn);
    const int64_t m0 = (int64_t)tm * TR;
    const int n0 = tn * TC;
    const int nsl = (K + 15) / 16, my = (nsl - wave + 3) / 4;       // slices of all, of this wave (wave, wave + 4, ...)
    // rows past M or N lie past the end of the panel's descriptor, pieces past K get such an offset: both read as zeros
    const int am = (int)(M - m0 < TR ? M - m0 : TR), wn = N - n0 < TC ? N - n0 : TC;
    const __amdgpu_buffer_rsrc_t a_rs = make_rsrc(A + m0 * K, am * K * 4), w_rs = make_rsrc(W + (int64_t)n0 * K, wn * K * 4);
    uint4 *ring = lds_raw + wave * R * S::SLICE;
    const int lrow = lane >> 2, lk = ((lane & 3) ^ ((lrow >> 2) & 3)) * 4;
    auto issue = [&](int t) {                                       // slice t of this wave
        uint4 *dst = ring + (t % R) * S::SLICE;
        const int k = (wave + 4 * t) * 16 + lk;
#pragma unroll
        for (int i = 0; i < MR || i < MC; ++i) {
            const int off = k < K ? ((i * 16 + lrow) * K + k) * 4 : F32_OOB;
            if (i < MR) __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rs, (lds_ptr)(dst + i * 64), 16, off, 0, 0, 0);
            if (i < MC) __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rs, (lds_ptr)(dst + TR * 4 + i * 64), 16, off, 0, 0, 0);
        }
    };
    const int rd = l15 * 4 + (g ^ ((l15 >> 2) & 3));
    auto frag = [&](int t, int part, int i) {                       // part 0: A rows, 1: W rows
        return reinterpret_cast<const frag4 *>(ring + (t % R) * S::SLICE)[part * TR * 4 + i * 64 + rd];
    };

    f32x4 acc[MC][MR];
#pragma unroll
    for (int ni = 0; ni < MC; ++ni)
#pragma unroll
        for (int mi = 0; mi < MR; ++mi) acc[ni][mi] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < R; ++t) issue(t);

    if (LN) {
        frag4 fa[R][MR], gg[R], bb[R];
        const __amdgpu_buffer_rsrc_t g_rs = make_rsrc(ln_g, K * 4), b_rs = make_rsrc(ln_b, K * 4);
        auto col = [&](int t) { return (wave + 4 * t) * 16 + 4 * g; };          // first k of this lane in slice t
#pragma unroll
        for (int t = 0; t < R; ++t) {
            gg[t] = load_piece(g_rs, col(t) < K ? col(t) * 4 : F32_OOB);
            bb[t] = load_piece(b_rs, col(t) < K ? col(t) * 4 : F32_OOB);
        }
        __builtin_amdgcn_s_waitcnt(0 | (0x7 << 4) | (0xF << 8));
#pragma unroll
        for (int t = 0; t < R; ++t)
#pragma unroll
            for (int i = 0; i < MR; ++i) fa[t][i] = frag(t, 0, i);
        float mean[MR], inv[MR];
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
            for (int i = 0; i < MR; ++i) {
                float s = 0.f;
#pragma unroll
                for (int t = 0; t < R; ++t) {
                    if (pass == 1) {                                // K % 4 == 0: a piece is inside or outside as a whole
                        const float in = col(t) < K ? 1.f : 0.f;
                        fa[t][i] = (fa[t][i] - mean[i]) * in;
                        s += (fa[t][i][0] * fa[t][i][0] + fa[t][i][1] * fa[t][i][1]) + (fa[t][i][2] * fa[t][i][2] + fa[t][i][3] * fa[t][i][3]);
                    } else {
                        s += (fa[t][i][0] + fa[t][i][1]) + (fa[t][i][2] + fa[t][i][3]);
                    }
                }
                s += __shfl_xor(s, 16, WAVE);
                s += __shfl_xor(s, 32, WAVE);
                if (g == 0) stat[pass][wave][i * 16 + l15] = s;
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < MR; ++i) {
                const int r = i * 16 + l15;
                const float s = ((stat[pass][0][r] + stat[pass][1][r]) + (stat[pass][2][r] + stat[pass][3][r])) / (float)K;
                if (pass == 0) mean[i] = s;
                else inv[i] = 1.0f / sqrtf(s + eps);
            }
        }
#pragma unroll
        for (int t = 0; t < R; ++t) {
            frag4 fw[MC];
#pragma unroll
            for (int i = 0; i < MC; ++i) fw[i] = frag(t, 1, i);
#pragma unroll
            for (int i = 0; i < MR; ++i) fa[t][i] = fa[t][i] * inv[i] * gg[t] + bb[t];     // zero beyond K: gain and shift are
#pragma unroll
            for (int ni = 0; ni < MC; ++ni)
#pragma unroll
                for (int mi = 0; mi < MR; ++mi) acc[ni][mi] = mfma_slice(fw[ni], fa[t][mi], acc[ni][mi]);
        }
    } else {
        for (int t = 0; t < my; ++t) {
            // slice t has landed once at most the loads of the R - 1 slices after it are in flight
            constexpr int V = (R - 1) * (MR + MC);
            __builtin_amdgcn_s_waitcnt((V & 0xF) | (V >> 4 << 14) | (0x7 << 4) | (0xF << 8));
            asm volatile("" ::: "memory");
            frag4 fa[MR], fw[MC];
#pragma unroll
            for (int i = 0; i < MR; ++i) fa[i] = frag(t, 0, i);
#pragma unroll
            for (int i = 0; i < MC; ++i) fw[i] = frag(t, 1, i);
#pragma unroll
            for (int ni = 0; ni < MC; ++ni)
#pragma unroll
                for (int mi = 0; mi < MR; ++mi) acc[ni][mi] = mfma_slice(fw[ni], fa[mi], acc[ni][mi]);
            __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4) | (0x0 << 8));       // lgkmcnt: the slice has been read
            asm volatile("" ::: "memory");
            issue(t + R);                                           // past the last slice: zeros, to keep the count
        }
        __builtin_amdgcn_s_waitcnt(0 | (0x7 << 4) | (0xF << 8));
    }

    // acc[ni][mi][i] <-> column ni*16 + 4 g + i, row mi*16 + l15
    __syncthreads();
    float (*part)[TR][S::LP] = reinterpret_cast<float (*)[TR][S::LP]>(lds_raw);
#pragma unroll
    for (int mi = 0; mi < MR; ++mi)
#pragma unroll
        for (int ni = 0; ni < MC; ++ni)
            *reinterpret_cast<float4 *>(&part[wave][mi * 16 + l15][ni * 16 + g * 4]) =
                make_float4(acc[ni][mi][0], acc[ni][mi][1], acc[ni][mi][2], acc[ni][mi][3]);
    __syncthreads();
    for (int id = tid; id < TR * TC / 4; id += 256) {
        const int r = id / (TC / 4), c = id % (TC / 4) * 4;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (part[0][r][c + i] + part[1][r][c + i]) + (part[2][r][c + i] + part[3][r][c + i]);
        if (m0 + r < M && n0 + c < N) store_four<EPI>(v, bias, resid, C, m0 + r, n0 + c, N, vec);
    }
#endif
}

// Many tiles: 64 x 32 outputs, four waves of 32 x 16, K in steps of 32 (rows of 128 bytes) that go from memory
// straight into LDS (buffer_load ... lds), FS - 1 steps ahead; up to six workgroups per compute unit, whose number
// hides what two stages do not (four stages and two workgroups: 257 against 228 us per layer of 256 tiny images;
// tiles of 64 columns no faster there, and 189 against 172 us with 17 deit_small images, 318 tiles of 64 on 256
// compute units).  72 to 90 TFLOP/s at K = 192 to 1536, 30 with the vector-ALU kernel it replaced.  LDS rows are
// eight 16-byte chunks, chunk c of row r at slot c ^ (r & 7) ^ (r >> 3 & 1), the chunks of a 16-wide slice dealt
// 0, 2, 1, 3 to the quarters of a wave: the bf16 kernels' layout, free of bank conflicts.
constexpr int FT = 64, FN = 32, FK = 32, FCH = FK / 4, FS = 2;
template <int EPI>
__global__ __launch_bounds__(256, 4) void gemm_f32_tile_kernel(const float *__restrict__ A, const float *__restrict__ W, int M,
                                                               int N, int K, int tiles_n, int tiles, int vec,
                                                               const float *__restrict__ bias, const float *resid, float *C)
{
#if defined(__HIP_DEVICE_COMPILE__)
    extern __shared__ uint4 lds_raw[];                              // [FS][A panel | W panel], FT rows of FCH chunks each
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l15 = lane & 15, g = lane >> 4;
    int tm, tn;
    f32_tile_of(tiles_n, tiles, &tm, &tn);
    const int64_t m0 = (int64_t)tm * FT;
    const int n0 = tn * FN;
    constexpr int NI = FN / 32, STAGE = (FT + FN) * FCH;
    const int wm0 = (wave >> 1) * 32, wn0 = (wave & 1) * (FN / 2);
    auto swz = [](int r) { return (r & 7) ^ ((r >> 3) & 1); };
    const int am = (int)(M - m0 < FT ? M - m0 : FT), wn = N - n0 < FN ? N - n0 : FN;
    const __amdgpu_buffer_rsrc_t a_rs = make_rsrc(A + m0 * K, am * K * 4);
    const __amdgpu_buffer_rsrc_t w_rs = make_rsrc(W + (int64_t)n0 * K, wn * K * 4);
    // load i of a wave fills panel rows (4 i + wave) * 8 .. + 7; lane l lands at row l / 8, slot l % 8
    int roff[2], kc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = (i * 4 + wave) * 8 + (lane >> 3);
        kc[i] = ((lane & 7) ^ swz(r)) * 4;
        roff[i] = r * K * 4;                                        // rows past the panel's end lie past the descriptor's
    }
    const int KT = (K + FK - 1) / FK;
    auto issue = [&](int kt) {
        uint4 *dst = lds_raw + (kt % FS) * STAGE;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = kt * FK + kc[i];
            const int off = k < K ? roff[i] + k * 4 : F32_OOB;          // past K: zeros
            __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rs, (lds_ptr)(dst + (i * 4 + wave) * 64), 16, off, 0, 0, 0);
            if (i < NI)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rs, (lds_ptr)(dst + FT * FCH + (i * 4 + wave) * 64), 16, off, 0, 0, 0);
        }
    };
    f32x4 acc[NI][2];
#pragma unroll
    for (int a = 0; a < NI; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int kc4 = ((g & 1) << 1) | (g >> 1);
#pragma unroll
    for (int st = 0; st < FS - 1; ++st) issue(st);
    for (int kt = 0; kt < KT; ++kt) {
        __builtin_amdgcn_s_waitcnt(((FS - 2) * (2 + NI)) | (0x7 << 4) | (0xF << 8));       // vmcnt: step kt has landed
        __builtin_amdgcn_s_barrier();
        issue(kt + FS - 1);
        const frag4 *Ab = reinterpret_cast<const frag4 *>(lds_raw + (kt % FS) * STAGE), *Wb = Ab + FT * FCH;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int c = (kk * 4 + kc4) ^ swz(l15);
            frag4 fa[2], fw[NI];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                fa[i] = Ab[(wm0 + i * 16 + l15) * FCH + c];
                if (i < NI) fw[i] = Wb[(wn0 + i * 16 + l15) * FCH + c];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int mi = 0; mi < 2; ++mi)
                        acc[ni][mi] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[ni][j], fa[mi][j], acc[ni][mi], 0, 0, 0);
        }
    }
    __builtin_amdgcn_s_waitcnt(0 | (0x7 << 4) | (0xF << 8));        // the loads past the last step, before LDS goes away
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const int64_t m = m0 + wm0 + mi * 16 + l15;
            const int n = n0 + wn0 + ni * 16 + g * 4;
            const float v[4] = {acc[ni][mi][0], acc[ni][mi][1], acc[ni][mi][2], acc[ni][mi][3]};
            if (m < M && n < N) store_four<EPI>(v, bias, resid, C, m, n, N, vec);
        }
#endif
}

// LayerNorm and the dense layer after it, many rows, K <= 16 NS (NS the next multiple of four): 64 rows to a workgroup,
// which stay in registers (each of its eight waves holds 16 of them, all K, normalised there: a row's sums need two shuffles
// and no exchange between waves) while the weights pass by in steps of 32 columns, 16 for each half of the waves.  Three steps of weights in
// LDS, two on their way: the first is fetched with the rows, the other two use the rows' place once those are in registers.
// LDS: chunks of 32 k, rows of eight 16-byte pieces, placed and dealt to the quarters of a wave as in the tile kernel.
// Every load of the loop goes to LDS; what goes to registers (gain, shift, bias) is waited for before it begins.
//   What bounds it: the matrix instructions of a step (1.3 us at full clock, 1.7 to 2.3 measured), before them the rows'
// way from memory and their sums, about a step's time.  The halves of the waves share the SIMDs and store in turns, one
// while the other multiplies.  Before: LayerNorm as a launch of its own and the 64 x 32 tiles: 1576 x 576 x 192
// 10.1 us, now 8.4; 1576 x 768 x 192 with GELU 13.1, now 11.4; 6304 x 768 x 192 32.1, now 27.3; 394 x 1536 x 384, then
// on 32 x 32 tiles, 17.8, now 13.6.  Four sums per output: against 64 bits 1.2e-7 where one long sum had 2.1e-7.
template <int NS>
struct F32Rows {
    static constexpr int T = 64, CN = 32, MAX_STEPS = 32;
    static constexpr int A_PIECES = NS / 2 * T * 8, W_PIECES = NS / 2 * CN * 8;
    static constexpr int A_LOADS = A_PIECES / 512, W_LOADS = W_PIECES / 512;      // of each wave
    static constexpr size_t smem = (size_t)(A_PIECES + W_PIECES) * 16;            // rows | step 0; later steps 1 and 2 | step 0
    static_assert(A_PIECES == 2 * W_PIECES && A_PIECES % 512 == 0 && W_PIECES % 512 == 0, "");
};

template <int NS, int EPI>
__global__ __launch_bounds__(512, NS <= 12 ? 4 : 2) void gemm_f32_rows_kernel(
    const float *__restrict__ A, const float *__restrict__ W, int M, int N, int K, int steps, int groups, int tiles,
    const float *__restrict__ ln_g, const float *__restrict__ ln_b, const float *__restrict__ bias, float *C, float eps, int vec)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using S = F32Rows<NS>;
    extern __shared__ uint4 lds_raw[];
    __shared__ __align__(16) float gs[NS * 16], bs[NS * 16], cs[S::MAX_STEPS * S::CN];
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l15 = lane & 15, g = lane >> 4;
    int tm, tg;
    f32_tile_of(groups, tiles, &tm, &tg);
    const int64_t m0 = (int64_t)tm * S::T;
    const int n0 = tg * steps * S::CN;
    auto swz = [](int r) { return (r & 7) ^ ((r >> 3) & 1); };
    // rows past M or N lie past the end of the panel's descriptor, pieces past K get such an offset: both read as zeros
    const int am = (int)(M - m0 < S::T ? M - m0 : S::T), wn = N - n0 < steps * S::CN ? N - n0 : steps * S::CN;
    const __amdgpu_buffer_rsrc_t a_rs = make_rsrc(A + m0 * K, am * K * 4), w_rs = make_rsrc(W + (int64_t)n0 * K, wn * K * 4);
    auto slot = [&](int st) { return st % 3 == 0 ? S::A_PIECES : (st % 3 - 1) * S::W_PIECES; };
    auto load = [&](__amdgpu_buffer_rsrc_t rs, int dst, int chunk, int row0, int first) {   // rows row0 .. + 7 of a panel in LDS
        const int r = row0 + (lane >> 3), k = chunk * 32 + ((lane & 7) ^ swz(r)) * 4;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(lds_raw + dst), 16, k < K ? ((first + r) * K + k) * 4 : F32_OOB, 0, 0, 0);
    };
    auto issue = [&](int st) {                                      // past the last step: zeros, to keep the count
#pragma unroll
        for (int i = 0; i < S::W_LOADS; ++i) {
            const int id = i * 8 + wave;
            load(w_rs, slot(st) + id * 64, id / 4, id % 4 * 8, st * S::CN);
        }
    };
#pragma unroll
    for (int i = 0; i < S::A_LOADS; ++i) load(a_rs, (i * 8 + wave) * 64, i, wave * 8, 0);
    issue(0);
    if (tid < NS * 16) {
        gs[tid] = tid < K ? ln_g[tid] : 0.f;
        bs[tid] = tid < K ? ln_b[tid] : 0.f;
    }
    for (int i = tid; i < steps * S::CN; i += 512) cs[i] = n0 + i < N ? bias[n0 + i] : 0.f;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    const int kc4 = ((g & 1) << 1) | (g >> 1), rg = wave & 3, half = wave >> 2;
    frag4 fa[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s)
        fa[s] = reinterpret_cast<const frag4 *>(lds_raw)[((s >> 1) * S::T + rg * 16 + l15) * 8 + (((s & 1) * 4 + kc4) ^ swz(l15))];
    __syncthreads();                                                // every wave has its rows: steps 1 and 2 may land on them
    issue(1);
    issue(2);
    float mean = 0.f, inv = 0.f;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        float p[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (pass == 1) {                                        // K % 4 == 0: a piece is inside or outside as a whole
                const float in = s * 16 + kc4 * 4 < K ? 1.f : 0.f;
                fa[s] = (fa[s] - mean) * in;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) p[j] += pass == 1 ? fa[s][j] * fa[s][j] : fa[s][j];
        }
        float sum = (p[0] + p[1]) + (p[2] + p[3]);
        sum += __shfl_xor(sum, 16, WAVE);
        sum += __shfl_xor(sum, 32, WAVE);
        if (pass == 0) mean = sum / (float)K;
        else inv = 1.0f / sqrtf(sum / (float)K + eps);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)                                    // zero beyond K: gain and shift are
        fa[s] = fa[s] * inv * *reinterpret_cast<const frag4 *>(&gs[s * 16 + kc4 * 4]) + *reinterpret_cast<const frag4 *>(&bs[s * 16 + kc4 * 4]);

    const int64_t m = m0 + rg * 16 + l15;
    f32x4 acc[4];
    auto store = [&](int st) __attribute__((always_inline)) {
        const int cl = st * S::CN + half * 16 + g * 4, n = n0 + cl;
        if (m < M && n < N) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]) + cs[cl + i];
                if (EPI == EPI_BIAS_GELU) v[i] = gelu_erf(v[i]);
            }
            float *c = C + m * N + n;
            if (vec) {
                *reinterpret_cast<float4 *>(c) = make_float4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (n + i < N) c[i] = v[i];
            }
        }
    };
    for (int st = 0; st < steps; ++st) {
        if (st > 0) {
            // this step has landed once at most the next one's loads are in flight (a store between them only makes
            // the wait longer), for all waves at the barrier; the step before it has been read by then
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(S::W_LOADS | (0x7 << 4) | (0x0 << 8));
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            issue(st + 2);
            if (half) store(st - 1);                                // while the other half multiplies
        }
        const frag4 *Wb = reinterpret_cast<const frag4 *>(lds_raw + slot(st)) + (half * 16 + l15) * 8;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; s += 2) {                           // a chunk of 32 k; four sums, so that products overlap
            const frag4 w0 = Wb[(s >> 1) * S::CN * 8 + (kc4 ^ swz(l15))], w1 = Wb[(s >> 1) * S::CN * 8 + ((4 + kc4) ^ swz(l15))];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[s & 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(w0[j], fa[s][j], acc[s & 2], 0, 0, 0);
                acc[(s & 2) + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[j], fa[s + 1][j], acc[(s & 2) + 1], 0, 0, 0);
            }
        }
        if (!half) store(st);
    }
    if (half) store(steps - 1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // the loads past the last step, before LDS goes away
#endif
}

// ---------------------------------------------- dense layers on the vector ALU: any K, any alignment
constexpr int GT = 64;  // tile edge
constexpr int GK = 64;  // k step: few, long steps (each one costs a trip to memory on the small problems this path serves)

template <int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ A,
                                                       const float *__restrict__ W,
                                                       const float *__restrict__ bias,
                                                       const float *resid, float *C, int64_t M,
                                                       int N, int K)
{
    // rows padded to a multiple of 16 bytes: a thread's four a's (and w's) of one k are one 16-byte read
    __shared__ __align__(16) float As[GK][GT + 4];
    __shared__ __align__(16) float Ws[GK][GT + 4];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int64_t m0 = (int64_t)blockIdx.y * GT;
    const int n0 = blockIdx.x * GT;
    float acc[4][4] = {};
    // 64 rows x GK k per operand, EPT elements per thread; the elements of step k0 + GK are fetched
    // into registers while step k0 is multiplied out of LDS
    constexpr int EPT = GT * GK / 256;
    float ra[EPT], rw[EPT];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int id = threadIdx.x + i * 256;
            const int r = id / GK, k = id % GK;
            const int64_t gm = m0 + r;
            const int gn = n0 + r;
            ra[i] = (gm < M && k0 + k < K) ? A[gm * K + k0 + k] : 0.f;
            rw[i] = (gn < N && k0 + k < K) ? W[(int64_t)gn * K + k0 + k] : 0.f;
        }
    };
    fetch(0);
    for (int k0 = 0; k0 < K; k0 += GK) {
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int id = threadIdx.x + i * 256;
            const int r = id / GK, k = id % GK;
            As[k][r] = ra[i];
            Ws[k][r] = rw[i];
        }
        __syncthreads();
        if (k0 + GK < K) fetch(k0 + GK);
#pragma unroll
        for (int k = 0; k < GK; ++k) {
            const float4 a4 = *reinterpret_cast<const float4 *>(&As[k][ty * 4]);
            const float4 w4 = *reinterpret_cast<const float4 *>(&Ws[k][tx * 4]);
            const float a[4] = {a4.x, a4.y, a4.z, a4.w}, w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t gm = m0 + ty * 4 + i;
        if (gm >= M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int gn = n0 + tx * 4 + j;
            if (gn >= N) continue;
            float v = acc[i][j] + bias[gn];
            if (EPI == EPI_BIAS_GELU) v = gelu_erf(v);
            if (EPI == EPI_BIAS_RESID) v += resid[gm * N + gn];
            C[gm * N + gn] = v;
        }
    }
}

// ---------------------------------------------------------------- attention
// A wave works on 16 queries of one (image, head), 16 keys at a time.  SPLIT: the four waves of a workgroup share the
// queries, the key blocks are dealt to them, each with its own running maximum, sum and output, merged through LDS at
// the end (few queries in all: latency counts); otherwise every wave has queries of its own and meets all keys.
// Keys and values arrive a block ahead.  A value piece goes straight into registers (16 lanes to a row); key fragments
// would put every lane of a quarter wave on a row of its own, so keys pass through LDS, each wave's through its own
// part (piece c of row r at slot c ^ r: the 16-byte reads of 16 rows meet no bank twice).
//   S^T = K . Q^T    lane: query l % 16, keys 4 (l/16) + i
//   O^T += V^T . P^T step i multiplies key 4 g + i of every quarter g: the probabilities are the B operand as they
//                    stand, and V's 16-byte piece 4 (l%16) .. + 3 of that key's row feeds four 16-component blocks,
//                    block j holding components 4 r + j, r = 0 .. 15 (of each 64; NT of them).
// d_head % 4 == 0, d_head <= 64 NT; pieces past it are zeros.
template <int NT, bool SPLIT>
__global__ __launch_bounds__(256) void attn_f32_mfma_kernel(const float *__restrict__ qkv, float *__restrict__ o, int T, int D,
                                                            int H, int groups, int tiles)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int LP = 64 * NT + 4, CPR = 16 * NT;                  // padded output row; 16-byte pieces of a key row
    __shared__ __align__(16) float Os[SPLIT ? 4 : 1][16][LP];
    __shared__ float ms[4][16], ls[4][16];
    __shared__ uint4 Ks[4][2][16 * CPR];
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l15 = lane & 15, g = lane >> 4;
    // the groups of a pair on one XCD: its keys and values come past that L2 once (dealt to all eight XCDs: 24 pairs of 197
    // tokens 12.2 us, so 11.1; 96 of 65 8.3, so 7.3)
    int pair, grp;
    f32_tile_of(groups, tiles, &pair, &grp);
    const int dh = D / H, q0 = (SPLIT ? grp : grp * 4 + wave) * 16, h = pair % H;
    if (q0 >= T) return;                                            // without SPLIT: a wave with no queries
    const int64_t b = pair / H;
    const float *base = qkv + b * T * 3 * D + h * dh;
    const float scale = 1.0f / sqrtf((float)dh);
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(base, ((T - 1) * 3 * D + 2 * D + dh) * 4);
    auto piece = [&](int t, int which, int e) -> frag4 {            // components e .. e+3 of q, k or v of token t
        return load_piece(rs, t < T && e < dh ? (t * 3 * D + which * D + e) * 4 : F32_OOB);
    };
    const int w = __builtin_amdgcn_readfirstlane(wave);
    frag4 qf[4 * NT], vf[4][NT], vn[4][NT];
#pragma unroll
    for (int s = 0; s < 4 * NT; ++s) qf[s] = piece(q0 + l15, 0, s * 16 + g * 4);
    auto fetch = [&](int kb, int buf, frag4 (&v)[4][NT]) {          // a block past the last one: zeros, no traffic
#pragma unroll
        for (int i = 0; i < 4 * NT; ++i) {
            const int p = i * 64 + lane, row = p / CPR, e = ((p % CPR) ^ row) * 4, t = kb * 16 + row;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(&Ks[w][buf][i * 64]), 16,
                                                     t < T && e < dh ? (t * 3 * D + D + e) * 4 : F32_OOB, 0, 0, 0);
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) v[i][t] = piece(kb * 16 + g * 4 + i, 2, t * 64 + l15 * 4);
        asm volatile("" ::: "memory");
    };
    f32x4 acc[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mx = -INFINITY, sum = 0.f;
    const int nkb = (T + 15) / 16, step = SPLIT ? 4 : 1;
    int kb = SPLIT ? wave : 0;
    fetch(kb, 0, vf);
    for (int buf = 0; kb < nkb; kb += step, buf ^= 1) {
        fetch(kb + step, buf ^ 1, vn);
        // this block's keys have landed: younger are its 4 NT value pieces and the next block's loads
        __builtin_amdgcn_s_waitcnt((12 * NT & 0xF) | (12 * NT >> 4 << 14) | (0x7 << 4) | (0xF << 8));
        asm volatile("" ::: "memory");
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 4 * NT; ++c)
            s = mfma_slice(reinterpret_cast<const frag4 *>(Ks[w][buf])[l15 * CPR + ((c * 4 + g) ^ l15)], qf[c], s);
        float p[4], m = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = kb * 16 + g * 4 + i < T ? s[i] * scale : -INFINITY;
            m = fmaxf(m, p[i]);
        }
        m = fmaxf(m, __shfl_xor(m, 16, WAVE));
        m = fmaxf(m, __shfl_xor(m, 32, WAVE));
        m = fmaxf(m, mx);
        // -inf while every score so far is (a product past the fp32 range): such keys weigh nothing next to a finite
        // score of a later block, so they are measured against zero, not against each other
        const float ref = m == -INFINITY ? 0.f : m;
        const float alpha = expf(mx - ref);
        mx = m;
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = expf(p[i] - ref);
        sum = sum * alpha + ((p[0] + p[1]) + (p[2] + p[3]));        // this lane's keys
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[t][j] *= alpha;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i][t][j], p[i], acc[t][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) vf[i][t] = vn[i][t];
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // nothing on its way to LDS when the wave ends
    sum += __shfl_xor(sum, 16, WAVE);
    sum += __shfl_xor(sum, 32, WAVE);
    float *orow = o + (b * T + q0) * D + h * dh;                    // first query's output
    // acc[t][j][i] <-> query l15, component 64 t + 16 g + 4 i + j
    if (!SPLIT) {
        const float inv = 1.0f / sum;
        if (q0 + l15 < T) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int e = 64 * t + 16 * g + 4 * i;
                    if (e < dh)
                        *reinterpret_cast<float4 *>(orow + (int64_t)l15 * D + e) =
                            make_float4(acc[t][0][i] * inv, acc[t][1][i] * inv, acc[t][2][i] * inv, acc[t][3][i] * inv);
                }
        }
        return;
    }
    if (g == 0) { ms[wave][l15] = mx; ls[wave][l15] = sum; }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<float4 *>(&Os[SPLIT ? wave : 0][l15][64 * t + 16 * g + 4 * i]) =
                make_float4(acc[t][0][i], acc[t][1][i], acc[t][2][i], acc[t][3][i]);
    __syncthreads();
    const int d4 = dh / 4;
    for (int id = tid; id < 16 * d4; id += 256) {
        const int q = id / d4, e = id % d4 * 4;
        if (q0 + q >= T) continue;
        const float m = fmaxf(fmaxf(ms[0][q], ms[1][q]), fmaxf(ms[2][q], ms[3][q]));
        float l = 0.f;
        float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float f = expf(ms[w][q] - m);                     // 0 for a wave without keys or with none above -inf
            const float4 x = *reinterpret_cast<const float4 *>(&Os[SPLIT ? w : 0][q][e]);
            l += f * ls[w][q];
            r.x += f * x.x; r.y += f * x.y; r.z += f * x.z; r.w += f * x.w;
        }
        const float inv = 1.0f / l;
        *reinterpret_cast<float4 *>(orow + (int64_t)q * D + e) = make_float4(r.x * inv, r.y * inv, r.z * inv, r.w * inv);
    }
#endif
}

// Any d_head: one workgroup (128 threads) per (image, head, query token).
__global__ __launch_bounds__(128) void attn_f32_kernel(const float *__restrict__ qkv,
                                                       float *__restrict__ o, int T, int D, int H)
{
    extern __shared__ float sm[];  // [T] scores, then [dh] query, then 2 partials
    const int dh = D / H;
    float *sc = sm;
    float *qs = sm + T;
    float *part = qs + dh;
    const int t = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const float *base = qkv + (int64_t)b * T * 3 * D;
    for (int e = tid; e < dh; e += 128) qs[e] = base[(int64_t)t * 3 * D + h * dh + e];
    __syncthreads();
    const float scale = 1.0f / sqrtf((float)dh);
    float mx = -INFINITY;
    for (int u = tid; u < T; u += 128) {
        const float *k = base + (int64_t)u * 3 * D + D + h * dh;
        float acc = 0.f;
        for (int e = 0; e < dh; ++e) acc = fmaf(qs[e], k[e], acc);
        acc *= scale;
        sc[u] = acc;
        mx = fmaxf(mx, acc);
    }
    mx = wave_max(mx);
    if (lane == 0) part[wv] = mx;
    __syncthreads();
    mx = fmaxf(part[0], part[1]);
    __syncthreads();
    float sum = 0.f;
    for (int u = tid; u < T; u += 128) {
        const float p = expf(sc[u] - mx);
        sc[u] = p;
        sum += p;
    }
    sum = wave_sum(sum);
    if (lane == 0) part[wv] = sum;
    __syncthreads();
    const float inv = 1.0f / (part[0] + part[1]);
    for (int e = tid; e < dh; e += 128) {
        float acc = 0.f;
        for (int u = 0; u < T; ++u) acc = fmaf(sc[u], base[(int64_t)u * 3 * D + 2 * D + h * dh + e], acc);
        o[((int64_t)b * T + t) * D + h * dh + e] = acc * inv;
    }
}

__global__ void fill_pattern_kernel(float *x, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t v = (uint32_t)i * 2654435761u;
    v ^= v >> 15;
    v *= 2246822519u;
    v ^= v >> 13;
    x[i] = (float)(int32_t)v * (1.0f / 2147483648.0f);
}

}  // namespace

static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

hipError_t ep_f32_layernorm(const float *x, int64_t ldx, const float *g, const float *b, float eps, float *y,
                            int64_t rows, int D, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    const int rows_per_block = 256 / WAVE;
    const dim3 grid((unsigned)((rows + rows_per_block - 1) / rows_per_block));
    if (D % 4 == 0 && ldx % 4 == 0 && D <= 4 * 256 && aligned16(x) && aligned16(y)) {
        switch ((D + 255) / 256) {
        case 1: hipLaunchKernelGGL(ln_f32_vec_kernel<1>, grid, dim3(256), 0, s, x, ldx, g, b, eps, y, rows, D); break;
        case 2: hipLaunchKernelGGL(ln_f32_vec_kernel<2>, grid, dim3(256), 0, s, x, ldx, g, b, eps, y, rows, D); break;
        case 3: hipLaunchKernelGGL(ln_f32_vec_kernel<3>, grid, dim3(256), 0, s, x, ldx, g, b, eps, y, rows, D); break;
        default: hipLaunchKernelGGL(ln_f32_vec_kernel<4>, grid, dim3(256), 0, s, x, ldx, g, b, eps, y, rows, D); break;
        }
    } else {
        hipLaunchKernelGGL(ln_f32_kernel, grid, dim3(256), 0, s, x, ldx, g, b, eps, y, rows, D);
    }
    return hipGetLastError();
}

namespace {

// tiles of t x t outputs
int64_t square_tiles(int64_t M, int N, int t) { return ((M + t - 1) / t) * ((N + t - 1) / t); }

template <int MR, int MC, int EPI, int LN>
hipError_t launch_f32_direct(const float *A, const float *g, const float *b, float eps, const float *W, const float *bias,
                             const float *resid, float *C, int64_t M, int N, int K, int vec, hipStream_t s)
{
    using S = F32Direct<MR, MC, LN>;
    auto kern = gemm_f32_direct_kernel<MR, MC, EPI, LN>;
    static EpSmemLimit smem_limit;
    const hipError_t e = smem_limit.ensure(reinterpret_cast<const void *>(kern), (int)S::smem);
    if (e != hipSuccess) return e;
    const int tiles_n = (N + S::TC - 1) / S::TC;
    const int64_t tiles = (M + S::TR - 1) / S::TR * tiles_n;
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(256), S::smem, s, A, W, (int)M, N, K, tiles_n, (int)tiles, vec, g, b, bias,
                       resid, C, eps);
    return hipGetLastError();
}

template <int EPI>
hipError_t launch_f32_gemm(const float *A, const float *W, const float *bias, const float *resid, float *C, int64_t M,
                           int N, int K, hipStream_t s)
{
    if (K % 4 == 0 && aligned16(A) && aligned16(W) && square_tiles(M, N, 32) < (1 << 24) && K < (1 << 23)) {    // 2^32 threads to a grid, 32-bit offsets in a panel
        int cus = 0;
        const hipError_t e = ep_device_cu_count(&cus);
        if (e != hipSuccess) return e;
        const int vec = N % 4 == 0 && aligned16(bias) && aligned16(C) && (EPI != EPI_BIAS_RESID || aligned16(resid));
        const int64_t t16 = square_tiles(M, N, 16), t32 = square_tiles(M, N, 32);
        // The smallest tiles up to two to a compute unit (more of them: 16 tiny images 42.6 against 39.2 us per layer,
        // one deit_small image 45.4 against 44.5), tiles of 32 up to three (four deit_small images 70.9 us per layer
        // against 89.2 with twice as many, whose K panels every workgroup brings in on its own), then the LDS tiles.
        if (t16 <= 2 * cus) {
            return launch_f32_direct<1, 1, EPI, 0>(A, nullptr, nullptr, 0.f, W, bias, resid, C, M, N, K, vec, s);
        } else if (t32 <= 3 * cus) {
            // half as tall where that leaves the fullest compute unit less to do (1576 x 192 x 768 9.9 -> 9.2 us, three
            // halves instead of two tiles to a unit; 788 x 384 x 1536 17.1 -> 16.1)
            const int64_t t16x32 = (M + 15) / 16 * ((N + 31) / 32);
            if ((t16x32 + cus - 1) / cus < 2 * ((t32 + cus - 1) / cus))
                return launch_f32_direct<1, 2, EPI, 0>(A, nullptr, nullptr, 0.f, W, bias, resid, C, M, N, K, vec, s);
            return launch_f32_direct<2, 2, EPI, 0>(A, nullptr, nullptr, 0.f, W, bias, resid, C, M, N, K, vec, s);
        } else {
            const int tiles_n = (N + FN - 1) / FN, tiles = (int)((M + FT - 1) / FT) * tiles_n;
            hipLaunchKernelGGL(gemm_f32_tile_kernel<EPI>, dim3(tiles), dim3(256), FS * (FT + FN) * FK * sizeof(float), s, A, W,
                               (int)M, N, K, tiles_n, tiles, vec, bias, resid, C);
        }
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((N + GT - 1) / GT), (unsigned)((M + GT - 1) / GT));
    if (grid.y > 65535u) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gemm_f32_kernel<EPI>, grid, dim3(256), 0, s, A, W, bias, resid, C, M, N, K);
    return hipGetLastError();
}

}  // namespace

hipError_t ep_f32_gemm(const float *A, const float *W, const float *bias, const float *resid,
                       float *C, int64_t M, int N, int K, int epi, hipStream_t s)
{
    if (M <= 0 || N <= 0) return hipSuccess;
    switch (epi) {
    case EPI_BIAS: return launch_f32_gemm<EPI_BIAS>(A, W, bias, resid, C, M, N, K, s);
    case EPI_BIAS_GELU: return launch_f32_gemm<EPI_BIAS_GELU>(A, W, bias, resid, C, M, N, K, s);
    case EPI_BIAS_RESID: return launch_f32_gemm<EPI_BIAS_RESID>(A, W, bias, resid, C, M, N, K, s);
    }
    return hipErrorInvalidValue;
}

namespace {

constexpr int F32_ROWS = 64, F32_STEP = 32, F32_MAX_STEPS = 32;     // F32Rows' panel, columns of a step and most steps

// Steps of a workgroup of the rows kernel, and those of the fullest compute unit in all: bringing the rows in and normalising
// them takes about as long as a step
struct F32RowsSteps { int steps; int64_t unit; };
F32RowsSteps f32_rows_steps(int64_t M, int N, int cus)
{
    const int64_t panels = (M + F32_ROWS - 1) / F32_ROWS;
    const int all = (N + F32_STEP - 1) / F32_STEP;
    F32RowsSteps best = {1, INT64_MAX};
    for (int n = 1; n <= F32_MAX_STEPS && n <= all; ++n) {
        const int64_t c = (panels * ((all + n - 1) / n) + cus - 1) / cus * (n + 1);
        if (c < best.unit) best = {n, c};
    }
    return best;
}

inline int f32_rows_depth(int K) { return (K + 63) / 64 * 64; }    // what the rows kernel multiplies of it: whole F32Rows<4 n>

// LayerNorm and the dense layer behind it: how
enum F32LnRoute { F32_TWO_LAUNCHES = 0, F32_TILES_16 = 1, F32_TILES_32 = 2, F32_ROWS_IN_REGISTERS = 3 };

// K % 4 == 0, K <= 384.  A row of tiles of 16 or 32 normalises its rows again and again: past two and three of them to a unit
// (K <= 192: 788 x 768 8.5 us against 8.9 with 64 rows, 1040 x 768 10.4 against 9.2) or one of 32 (394 x 1536 x 384 17.8 against
// 13.6) the rows kernel, where it pays.  It saves a launch and the rows' trip through memory, and loses to the 64 x 32 tiles
// what it multiplies past K, and beyond 192 deep, with room for one workgroup on a unit, some of their rate: its steps against
// two for the launch, 0.85 for each tile a unit would have, in the measure of the depth, and 5.5 for each panel's LayerNorm.  Over 1095
// shapes (K = 16 to 384, N = 2 to 8 K, 65 to 25216 rows) 11 % faster on average than two launches (or 32-wide tiles) and 14 %
// slower at worst (2364 x 400 x 200 12.2 -> 14.0 us).  Depths that fill it up to 192 always go there: 7 % slower at worst
// (4728 x 1536 x 192 38.8 -> 41.4), 0.6 of the time at best (12608 x 96 x 32 10.2 -> 6.3).  With no depths but 192 and 384 and no
// rule up to 192, 25216 x 256 x 32 took 36.8 us where two launches take 22.9, 25216 x 768 x 96 84.1 for 60.5.
F32LnRoute f32_ln_route(int64_t M, int N, int K, int cus)
{
    const int64_t t32 = square_tiles(M, N, 32);
    if (square_tiles(M, N, 16) <= 2 * cus) return F32_TILES_16;
    if (t32 <= (K <= 192 ? 3 : 1) * cus) return F32_TILES_32;
    const int depth = f32_rows_depth(K);
    const int64_t panels = (M + F32_ROWS - 1) / F32_ROWS, tiles = panels * ((N + F32_STEP - 1) / F32_STEP);
    const bool fills = K <= 64 || (K <= 192 && depth - K < 16);
    if (fills || f32_rows_steps(M, N, cus).unit <= 2.0 + (0.85 * tiles * K / depth + 5.5 * panels) / cus) return F32_ROWS_IN_REGISTERS;
    return t32 <= 3 * cus ? F32_TILES_32 : F32_TWO_LAUNCHES;
}

template <int NS, int EPI>
hipError_t launch_f32_rows(const float *x, const float *g, const float *b, float eps, const float *W, const float *bias, float *C,
                           int64_t M, int N, int K, int vec, int cus, hipStream_t s)
{
    using S = F32Rows<NS>;
    static_assert(S::T == F32_ROWS && S::CN == F32_STEP && S::MAX_STEPS == F32_MAX_STEPS, "as planned");
    auto kern = gemm_f32_rows_kernel<NS, EPI>;
    static EpSmemLimit smem_limit;
    const hipError_t e = smem_limit.ensure(reinterpret_cast<const void *>(kern), (int)S::smem);
    if (e != hipSuccess) return e;
    const int64_t panels = (M + S::T - 1) / S::T;
    const int all = (N + S::CN - 1) / S::CN, steps = f32_rows_steps(M, N, cus).steps;
    const int groups = (all + steps - 1) / steps;
    const int64_t tiles = panels * groups;
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(512), S::smem, s, x, W, (int)M, N, K, steps, groups, (int)tiles, g, b, bias, C,
                       eps, vec);
    return hipGetLastError();
}

template <int EPI>
hipError_t launch_f32_ln_gemm(const float *x, const float *g, const float *b, float eps, const float *W, const float *bias,
                              float *C, int64_t M, int N, int K, hipStream_t s)
{
    int cus = 0;
    const hipError_t e = ep_device_cu_count(&cus);
    if (e != hipSuccess) return e;
    const int vec = N % 4 == 0 && aligned16(bias) && aligned16(C);
    switch (f32_ln_route(M, N, K, cus)) {
    case F32_TILES_16:
        return K <= 192 ? launch_f32_direct<1, 1, EPI, 3>(x, g, b, eps, W, bias, nullptr, C, M, N, K, vec, s)
                        : launch_f32_direct<1, 1, EPI, 6>(x, g, b, eps, W, bias, nullptr, C, M, N, K, vec, s);
    case F32_TILES_32:
        return K <= 192 ? launch_f32_direct<2, 2, EPI, 3>(x, g, b, eps, W, bias, nullptr, C, M, N, K, vec, s)
                        : launch_f32_direct<2, 2, EPI, 6>(x, g, b, eps, W, bias, nullptr, C, M, N, K, vec, s);
    case F32_ROWS_IN_REGISTERS:
#define EP_F32_ROWS(NS) return launch_f32_rows<NS, EPI>(x, g, b, eps, W, bias, C, M, N, K, vec, cus, s)
        switch (f32_rows_depth(K)) {
        case 64: EP_F32_ROWS(4);
        case 128: EP_F32_ROWS(8);
        case 192: EP_F32_ROWS(12);
        case 256: EP_F32_ROWS(16);
        case 320: EP_F32_ROWS(20);
        case 384: EP_F32_ROWS(24);
        }
#undef EP_F32_ROWS
        break;
    case F32_TWO_LAUNCHES: break;
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool ep_f32_ln_gemm_supported(const float *x, const float *W, int64_t M, int N, int K)
{
    int cus = 0;
    if (ep_device_cu_count(&cus) != hipSuccess) return false;
    return K % 4 == 0 && K <= 384 && M > 0 && N > 0 && aligned16(x) && aligned16(W) && square_tiles(M, N, 32) < (1 << 24) &&
           f32_ln_route(M, N, K, cus) != F32_TWO_LAUNCHES;
}

extern "C" int32_t ep_query_f32_ln_route(int64_t M, int32_t N, int32_t K, int32_t cus) { return f32_ln_route(M, N, K, cus); }

hipError_t ep_f32_ln_gemm(const float *x, const float *g, const float *b, float eps, const float *W, const float *bias, float *C,
                          int64_t M, int N, int K, int epi, hipStream_t s)
{
    if (!ep_f32_ln_gemm_supported(x, W, M, N, K) || !aligned16(g) || !aligned16(b)) return hipErrorInvalidValue;
    switch (epi) {
    case EPI_BIAS: return launch_f32_ln_gemm<EPI_BIAS>(x, g, b, eps, W, bias, C, M, N, K, s);
    case EPI_BIAS_GELU: return launch_f32_ln_gemm<EPI_BIAS_GELU>(x, g, b, eps, W, bias, C, M, N, K, s);
    }
    return hipErrorInvalidValue;
}

hipError_t ep_f32_attention(const float *qkv, float *o, int B, int T, int D, int H, hipStream_t s)
{
    if (B <= 0) return hipSuccess;
    if (H > 65535 || B > 65535) return hipErrorInvalidValue;
    const int dh = D / H;
    if (D % 4 == 0 && dh % 4 == 0 && dh <= 128 && aligned16(qkv) && aligned16(o) &&
        (int64_t)B * H * ((T + 15) / 16) < (1 << 24) && (int64_t)T * 3 * D * 4 < F32_OOB) {
        int cus = 0;
        const hipError_t e = ep_device_cu_count(&cus);
        if (e != hipSuccess) return e;
        const int64_t pairs = (int64_t)B * H;
        const int t16 = (T + 15) / 16;
        // up to a wave and a half per SIMD the keys are split (24 deit_tiny images, 936 waves: 95.6 us per layer against
        // 103.0; 768 tiny ones, 3840 waves: 222 against 219)
        const bool split = pairs * t16 <= 6 * cus;
        const int groups = split ? t16 : (t16 + 3) / 4;
        const int64_t tiles = pairs * groups;
#define EP_LAUNCH(NT, SPLIT) \
    hipLaunchKernelGGL((attn_f32_mfma_kernel<NT, SPLIT>), dim3((unsigned)tiles), dim3(256), 0, s, qkv, o, T, D, H, groups, (int)tiles)
        if (dh <= 64) { if (split) EP_LAUNCH(1, true); else EP_LAUNCH(1, false); }
        else { if (split) EP_LAUNCH(2, true); else EP_LAUNCH(2, false); }
#undef EP_LAUNCH
        return hipGetLastError();
    }
    const size_t smem = sizeof(float) * (size_t)(T + dh + 2);
    if (smem > 64 * 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(attn_f32_kernel, dim3(T, H, B), dim3(128), smem, s, qkv, o, T, D, H);
    return hipGetLastError();
}

hipError_t ep_fill_pattern(float *x, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_pattern_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, n);
    return hipGetLastError();
}
