// Multi-head self-attention of the bf16 path (paper section 2.1:
// attention scores of the token sequence through dot products; every output
// token independent).  qkv[b*T + t, :] = [q | k | v], each block head-major.
//
// Persistent workgroups, at most one per compute unit, each walking a list of units:
// a unit is one (image, head) pair with all its queries, or with one group of them
// where pairs are few (plan_attention).  The keys and values of a pair stream through LDS in chunks of 96
// tokens, K and V both row-major as they lie in memory: two loader waves bring
// chunk after chunk in with buffer_load ... lds (no register staging, no
// transposing copy) into a ring of five chunk buffers, up to four chunks - more
// than a whole pair at T = 257 - ahead of the query waves, so the memory latency
// of a unit hides behind the arithmetic of the one before, and any number of
// tokens passes through the same buffers.  One barrier per chunk both hands a
// landed chunk to the query waves and returns the buffer they have finished to
// the loaders.
//
// A query wave owns 32 queries (two 16-query blocks; one where pairs are few) and walks a chunk in three
// steps of 32 keys with v_mfma_f32_16x16x32_bf16:
//   S^T = K . Q^T   (A = K fragment: 16 keys x 32 components, one ds_read_b128
//                    per lane; B = Q fragment, held in registers for the pair):
//                   the accumulator puts one query per lane column (l % 16) and
//                   four consecutive keys per lane, so the row maximum is an
//                   in-lane reduction plus two exchanges across the quarters of
//                   the wave;
//   P = exp2((S - reference) * scale * log2 e), fp32, keys beyond T masked to
//                   -inf; the reference follows the true maximum lazily (what
//                   has been accumulated is rescaled only when some query's
//                   maximum grew by more than 2^6: bf16 and fp32 have exponent
//                   range to spare); rounded to bf16 the probabilities of two
//                   16-key blocks are, register for register, the B operand of
//   O^T += V^T . P^T (the order of the contraction index is free as long as both
//                   operands agree: slot 8g + m of the 32-key step is key
//                   4g + m of its first block for m < 4 and of its second block
//                   for m >= 4).  The A operand, 16 components x 32 keys of V^T,
//                   comes straight out of the row-major V with two
//                   ds_read_b64_tr_b16 per lane (within 16 lanes the instruction
//                   takes four rows of 16 elements and hands lane j column j);
//                   a fragment of ones as a further A operand makes the matrix
//                   pipe deliver the softmax denominator as well (the sum of the
//                   rounded probabilities, i.e. of the weights actually applied).
// The last 32-component step of a head width that is not a multiple of 32 (80)
// reads past the row into the next row (finite data) against zeros in Q.
//
// Weights touched.  The launches behind this one walk K in step with each other, every step's weights are new to all of them at once, and where
// they come from memory each step waits a part of that trip (FC2 of ViT-Large on 16 images, 64 steps: 36 us, and 28 where its 8 MB are in the memory-side
// cache; DeiT-Small on 32, 24 steps and 1.2 MB: 15.6 and 11.8).  This kernel is bound by its vector ALU, and memory idles meanwhile, so a
// wave of each workgroup more brings weights into that cache: those of the rest of the layer and of the next q|k|v projection, those of the projection and
// the second MLP layer, or none (the stage decides: touch_weights in ep_stage.hip).  The launch itself takes 2 to 3 us longer for 25 MB (64 components
// a head).
#include "ep_kernels.h"
#include "ep_device.h"
#include "ep_launch.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int CK = 96;                               // keys per chunk
constexpr int SUBS = CK / 32;                        // 32-key steps per chunk
constexpr int NBUF = 5;                              // chunk buffers in the ring
constexpr int DEPTH = NBUF - 1;                      // chunks in flight ahead of the one being consumed
constexpr int NLOADER = 2;                           // loader waves
constexpr int MAXQW = 10;                            // query waves
constexpr uint32_t MAX_TOUCH = 1u << 30;             // offsets of touched lines are 32-bit

template <int DH>
struct StreamShape {
    static constexpr int ROWB = DH * 2;              // bytes of a K or V row in LDS
    static constexpr int PARTB = CK * ROWB;          // K part (then V part) of a chunk buffer
    static constexpr int BUFB = 2 * PARTB;
    static constexpr int LPW = PARTB / 1024;         // ... per loader wave: one takes the K parts, the other the V parts
    static constexpr int KS = (DH + 31) / 32;        // 32-component steps of the first product
    static constexpr int EB = DH / 16;               // 16-component blocks of the output
    static constexpr bool SWZ = ROWB == 128;         // 16-byte pieces of a row change places (see piece)
    static constexpr size_t smem = (size_t)NBUF * BUFB;
    static_assert(DH % 16 == 0 && PARTB % 1024 == 0 && NLOADER == 2, "chunk parts are whole loads, one loader per part");
    static_assert(DEPTH * LPW <= 63, "the loaders' counted wait fits the vmcnt field");
};

// Where piece c (16 bytes) of row r of a K or V part sits.  Rows of 128 bytes start at one of two banks and every read here goes
// across rows, so at d_head 64 the pieces of eight consecutive rows are dealt to all places of a row (without it bank conflicts
// were 20 to 27 % of the kernel's clocks); rows of 160 bytes spread by themselves.
template <int DH>
__device__ inline int piece(int r, int c)
{
    return StreamShape<DH>::SWZ ? c ^ (r & 7) ^ ((r >> 3) & 1) : c;
}

// maximum over lanes l, l ^ 16, l ^ 32, l ^ 48 (the four quarters of the wave hold the keys of one query):
// v_permlane16_swap exchanges the odd 16-lane rows of its first operand with the even rows of its
// second, v_permlane32_swap the upper half of the first with the lower half of the second; fed the
// same value twice, a maximum of the two results folds rows 0|1 and 2|3, then the two halves.
__device__ inline float quarter_max(float v)
{
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const float w = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    const unsigned x = __float_as_uint(w);
    const auto q = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

#define EP_ATTN_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))

// Q fragments of NQB 16-query blocks starting at query q0 of a pair (B operand: column = query l15 of the
// block, 8 consecutive components at 32 ks + 8 g; components past the head width read as zeros: an offset
// past the descriptor's end).  The empty assembly keeps the loads here, a whole unit ahead of their use.
template <int DH, int NQB>
__device__ __forceinline__ void issue_q(const uint16_t *__restrict__ qkv, int T, int D, int H, int pair, int q0,
                                        u32x4 (&qf)[NQB][StreamShape<DH>::KS])
{
    constexpr int KS = StreamShape<DH>::KS;
    const int lane = threadIdx.x & 63;
    const int l15 = lane & 15, g = lane >> 4;
    const int row_bytes = 3 * D * 2;
    const int seg_bytes = (T - 1) * row_bytes + DH * 2;
    const uint16_t *base = qkv + (size_t)(pair / H) * T * 3 * D + (size_t)(pair % H) * DH;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(base), 0, seg_bytes, 0x00020000);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
        const int qrow = min(q0 + qb * 16 + l15, T - 1);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bool in_row = ks * 32 + g * 8 < DH;
            const int voff = in_row ? qrow * row_bytes + ks * 64 + g * 16 : 0x7FFFFFF0;
            qf[qb][ks] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, 0, 0));
        }
    }
    asm volatile("" ::: "memory");
}

// One pass of a query wave over the keys of a pair: the NQB 16-query blocks whose Q fragments are in qf, chunk
// steps j0 .. j0 + nch - 1 of the workgroup's barrier sequence.  mid() is called once, at the start of the pass's
// second chunk (of its only one): the place for the caller's fetch of the next unit's fragments, away from the
// burst of output stores at the end of a unit.
template <int DH, int NQB, class Mid>
__device__ __forceinline__ void attn_pass(const u32x4 (&qf)[NQB][StreamShape<DH>::KS], char *lds, int T, int nch, int j0,
                                          float scale_log2e, f32x4 (&acc_o)[StreamShape<DH>::EB][NQB], f32x4 (&acc_sum)[NQB],
                                          Mid mid)
{
    using S = StreamShape<DH>;
    constexpr int ROWB = S::ROWB, PARTB = S::PARTB, BUFB = S::BUFB, KS = S::KS, EB = S::EB;
    const int lane = threadIdx.x & 63;
    const int l15 = lane & 15, g = lane >> 4;
    bf16x8 ones;
#pragma unroll
    for (int i = 0; i < 8; ++i) ones[i] = (__bf16)1.0f;
    asm volatile("" : "+v"(ones));                    // four registers, not moves in every step
    // lane's part of the V^T fragment addressing: source lane s = l % 16 of quarter g supplies row 4g + s/4,
    // elements 4 (s % 4) .. + 3 of the 16-component block
    // (blocks of 32 and of 16 rows further on keep the places of the pieces)
    int v_lane[EB], k_lane[KS];
    {
        const int r = 4 * g + (l15 >> 2);
#pragma unroll
        for (int eb = 0; eb < EB; ++eb) v_lane[eb] = r * ROWB + piece<DH>(r, eb * 2 + ((l15 >> 1) & 1)) * 16 + (l15 & 1) * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) k_lane[ks] = l15 * ROWB + piece<DH>(l15, ks * 4 + g) * 16;
    }

    float mref[NQB];                                                // reference maximum, in scaled log2 units
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
        mref[qb] = -INFINITY;
        acc_sum[qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int eb = 0; eb < EB; ++eb) acc_o[eb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    for (int c = 0; c < nch; ++c) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();              // chunk j0 + c has landed; the buffer of the chunk before goes back to the loaders
        asm volatile("" ::: "memory");
        const char *Kb = lds + ((j0 + c) % NBUF) * BUFB;
        const char *Vb = Kb + PARTB;
        if (c == (nch > 1 ? 1 : 0)) mid();
        const int nsub = min(SUBS, (T - c * CK + 31) / 32); // 32-key steps that hold a key (wave-uniform)
        // K fragments of a 32-key step, and V^T fragments.  At d_head 64 they are sent for a softmax ahead of their use, which a
        // wave that is alone on its SIMD would otherwise wait for (577 tokens, 24 pairs: 9.5 -> 8.7 us a launch); at 80 the
        // registers run out (64 images of 257 tokens 49 -> 62 us).
        bf16x8 kf[KS][2], vf[EB];
        auto read_k = [&](int sub) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
                    kf[ks][kb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(Kb + k_lane[ks] + (sub * 32 + kb * 16) * ROWB));
        };
        auto read_v = [&](int sub) {
#pragma unroll
            for (int eb = 0; eb < EB; ++eb) {
                typedef __attribute__((address_space(3))) s16x4 *tr_ptr;
                typedef short s16x8 __attribute__((ext_vector_type(8)));
                const char *vp = Vb + v_lane[eb] + (sub * 32) * ROWB;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(vp));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(vp + 16 * ROWB));
                const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                vf[eb] = __builtin_bit_cast(bf16x8, both);
            }
        };
        // S^T = K . Q^T: s[kb][qb][i] <-> key key0 + kb*16 + 4g + i, query q0 + qb*16 + l15
        auto scores = [&](f32x4 (&s)[2][NQB]) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int qb = 0; qb < NQB; ++qb) s[kb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int qb = 0; qb < NQB; ++qb)
                        s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks][kb], __builtin_bit_cast(bf16x8, qf[qb][ks]), s[kb][qb], 0, 0, 0);
        };
        // With one query block a wave is alone on its SIMD and one step after the other is a chain: there the next
        // step's scores are on the matrix pipe while this step's go through the vector ALU (577 tokens, 24 pairs:
        // twelve layers 774 -> 764 us).  With two blocks and two or three waves to a SIMD it gains nothing, and at
        // d_head 80 the registers run out (three layers of 256 images 7945 -> 7971).
        constexpr bool AHEAD = NQB == 1;
        constexpr bool EARLY = DH == 64;
        f32x4 sc[AHEAD ? 2 : 1][2][NQB];
        if (EARLY || AHEAD) read_k(0);
        if (AHEAD) {
            scores(sc[0]);
            if (EARLY && nsub > 1) read_k(1);
        }
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub) {
            if (sub >= nsub) break;                         // nothing but padding from here on
            if (!AHEAD) {
                if (!EARLY) read_k(sub);
                scores(sc[0]);
            }
            if (EARLY) read_v(sub);
            if (AHEAD && sub + 1 < SUBS && sub + 1 < nsub) {
                if (!EARLY) read_k(sub + 1);
                scores(sc[AHEAD ? (sub + 1) & 1 : 0]);
            }
            if (EARLY) {
                constexpr int next = AHEAD ? 2 : 1;         // the step whose scores come next
                if (sub + next < SUBS && sub + next < nsub) read_k(sub + next);
                __builtin_amdgcn_sched_barrier(0);
            }
            f32x4 (&s)[2][NQB] = sc[AHEAD ? sub & 1 : 0];
            const int key0 = c * CK + sub * 32;
            if (key0 + 32 > T) {                            // wave-uniform: keys to mask in the last step only
                const int lim = T - key0 - 4 * g;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (kb * 16 + i >= lim) {
#pragma unroll
                            for (int qb = 0; qb < NQB; ++qb) s[kb][qb][i] = -INFINITY;
                        }
            }
            // ---- softmax numerators of the step, as B fragments of the second product
            bf16x8 pf[NQB];
#pragma unroll
            for (int qb = 0; qb < NQB; ++qb) {
                float mx = fmaxf(fmaxf(fmaxf(s[0][qb][0], s[0][qb][1]), fmaxf(s[0][qb][2], s[0][qb][3])),
                                 fmaxf(fmaxf(s[1][qb][0], s[1][qb][1]), fmaxf(s[1][qb][2], s[1][qb][3])));
                mx = quarter_max(mx);
                const float t = mx * scale_log2e;           // finite: a step visited has a key < T
                if (__builtin_amdgcn_ballot_w64(t > mref[qb] + 6.0f) != 0) {
                    const float nref = fmaxf(mref[qb], t);
                    const float alpha = __builtin_amdgcn_exp2f(mref[qb] - nref);
                    mref[qb] = nref;
#pragma unroll
                    for (int eb = 0; eb < EB; ++eb) acc_o[eb][qb] *= alpha;
                    acc_sum[qb] *= alpha;
                }
                const float mb = mref[qb];
                float p[8];
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        p[kb * 4 + i] = __builtin_amdgcn_exp2f(fmaf(s[kb][qb][i], scale_log2e, -mb));
                u32x4 pw;
                pw[0] = pack_bf16x2(p[0], p[1]);
                pw[1] = pack_bf16x2(p[2], p[3]);
                pw[2] = pack_bf16x2(p[4], p[5]);
                pw[3] = pack_bf16x2(p[6], p[7]);
                pf[qb] = __builtin_bit_cast(bf16x8, pw);
            }
            // ---- O^T += V^T . P^T and the denominators
            if (!EARLY) read_v(sub);
#pragma unroll
            for (int eb = 0; eb < EB; ++eb)
#pragma unroll
                for (int qb = 0; qb < NQB; ++qb)
                    acc_o[eb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[eb], pf[qb], acc_o[eb][qb], 0, 0, 0);
#pragma unroll
            for (int qb = 0; qb < NQB; ++qb)
                acc_sum[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[qb], acc_sum[qb], 0, 0, 0);
        }
    }

}

// Normalise and store a pass's output: acc_o[eb][qb][i] <-> component eb*16 + 4g + i, query q0 + qb*16 + l15;
// every row of acc_sum's block holds the query's softmax denominator.  A lane's four components of a block
// are 8 bytes of bf16; for a pair of blocks (eb, eb + 1) v_permlane16_swap trades them between the even and
// odd quarters of the wave so that an even quarter ends up with components 4g .. 4g + 7 of block eb and an
// odd one with 4(g-1) .. 4(g-1) + 7 of block eb + 1: 16 contiguous bytes per lane, half the store
// instructions.  A last unpaired block goes out in 8-byte pieces.
template <int DH, int NQB>
__device__ __forceinline__ void store_pass(const f32x4 (&acc_o)[StreamShape<DH>::EB][NQB], const f32x4 (&acc_sum)[NQB],
                                           uint16_t *__restrict__ o, int T, int D, int H, int pair, int q0)
{
    constexpr int EB = StreamShape<DH>::EB;
    const int lane = threadIdx.x & 63;
    const int l15 = lane & 15, g = lane >> 4;
    const int b = pair / H, h = pair % H;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
        const int q = q0 + qb * 16 + l15;
        const float inv = 1.0f / acc_sum[qb][0];
        uint16_t *row = o + ((size_t)b * T + q) * D + (size_t)h * DH;
        auto packed = [&](int eb, int half) {
            return pack_bf16x2(acc_o[eb][qb][2 * half] * inv, acc_o[eb][qb][2 * half + 1] * inv);
        };
#pragma unroll
        for (int eb = 0; eb + 1 < EB; eb += 2) {
            // after the swaps: even quarters hold (own block eb | block eb of quarter g + 1), odd quarters
            // (block eb + 1 of quarter g - 1 | own block eb + 1)
            const auto lo = __builtin_amdgcn_permlane16_swap(packed(eb, 0), packed(eb + 1, 0), false, false);
            const auto hi = __builtin_amdgcn_permlane16_swap(packed(eb, 1), packed(eb + 1, 1), false, false);
            const uint4 w = make_uint4(lo[0], hi[0], lo[1], hi[1]);
            const int e = (eb + (g & 1)) * 16 + 4 * (g & 2);
            if (q < T) *reinterpret_cast<uint4 *>(row + e) = w;
        }
        if (EB & 1) {
            uint2 w;
            w.x = packed(EB - 1, 0);
            w.y = packed(EB - 1, 1);
            if (q < T) *reinterpret_cast<uint2 *>(row + (EB - 1) * 16 + 4 * g) = w;
        }
    }
}

// All the work of a query wave.  A unit is one pair's keys against one group of nqw query tiles (QW = 16 NQB
// queries each; ng groups to a pair).  The Q fragments of the next unit are fetched before the current one is
// worked on, so their latency hides behind it.  A wave whose tile lies past the last query of its unit's pair (the
// last group may be short) only keeps the barrier count.
template <int DH, int NQB>
__device__ __forceinline__ void attn_wave(const uint16_t *__restrict__ qkv, uint16_t *__restrict__ o, char *lds, int T, int D,
                                          int H, int ng, int nqw, int wave, int unit, int unit_step, int my_units, int nch,
                                          float scale_log2e)
{
    constexpr int KS = StreamShape<DH>::KS, QW = 16 * NQB;
    u32x4 qf[NQB][KS], qn[NQB][KS];
    int pair = unit / ng, q0 = ((unit - pair * ng) * nqw + wave) * QW;
    issue_q<DH, NQB>(qkv, T, D, H, pair, q0, qf);
    for (int ui = 0; ui < my_units; ++ui) {
        const int o_pair = pair, o_q0 = q0;
        const bool more = ui + 1 < my_units;
        unit += unit_step;
        pair = unit / ng;
        q0 = ((unit - pair * ng) * nqw + wave) * QW;
        // qf takes the next unit's fragments ahead of the output stores (a wait for them behind the stores would
        // be a wait for the stores as well)
        auto take_next = [&]() {
#pragma unroll
            for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) qf[qb][ks] = qn[qb][ks];
        };
        if (o_q0 < T) {                                             // wave-uniform
            f32x4 acc_o[StreamShape<DH>::EB][NQB], acc_sum[NQB];
            attn_pass<DH, NQB>(qf, lds, T, nch, ui * nch, scale_log2e, acc_o, acc_sum,
                               [&]() { if (more) issue_q<DH, NQB>(qkv, T, D, H, pair, q0, qn); });
            if (more) take_next();
            store_pass<DH, NQB>(acc_o, acc_sum, o, T, D, H, o_pair, o_q0);
        } else {
            for (int c = 0; c < nch; ++c) {
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            if (more) issue_q<DH, NQB>(qkv, T, D, H, pair, q0, qf);
        }
    }
}

// QW: queries of a query wave (32 or 16).  TOUCH: a last wave touches weights (a template argument: as a branch it cost a stage of
// single images, which does not, 0.9 %)
template <int DH, int QW, bool TOUCH>
__global__ __launch_bounds__((MAXQW + NLOADER) * 64) void attn_stream_kernel(const uint16_t *__restrict__ qkv,
                                                                             uint16_t *__restrict__ o, int T, int D, int H, int ng,
                                                                             int nqw, int grid, int each, int rest,
                                                                             float scale_log2e, uint32_t touch_bytes, const void *touch)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using S = StreamShape<DH>;
    constexpr int ROWB = S::ROWB, PARTB = S::PARTB, BUFB = S::BUFB, LPW = S::LPW;
    extern __shared__ uint4 smem_raw[];
    char *lds = reinterpret_cast<char *>(smem_raw);
    typedef __attribute__((address_space(3))) void *lds_ptr;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool loader = wave >= nqw;                               // wave-uniform
    const int row_bytes = 3 * D * 2;
    const int seg_bytes = (T - 1) * row_bytes + DH * 2;            // first to last byte of a head's q, k or v
    const int nch = (T + CK - 1) / CK;                             // chunks per unit

    // Workgroup w sits on XCD w % 8 (round-robin dispatch).  Each XCD gets a contiguous range of
    // units, as long as its share of the workgroups, so that the heads of an image, which
    // share cache lines of the qkv rows, meet in one L2; the workgroups of an XCD stride through it.
    // nqw query waves; grid * each + rest units in all, rest < grid: the n-th share of the grid begins at each * n + rest * n / grid.
    int unit, unit_end, unit_step;
    {
        const int x = blockIdx.x % 8, g8 = grid / 8, r8 = grid % 8;
        const int before = x * g8 + min(x, r8);                    // workgroups on the XCDs in front of this one
        unit_step = g8 + (x < r8 ? 1 : 0);                         // workgroups on this one
        auto begin = [&](int n) { return each * n + (int)((uint32_t)(rest * n) / (uint32_t)grid); };
        unit = begin(before) + blockIdx.x / 8;
        unit_end = begin(before + unit_step);
    }
    if (unit >= unit_end) return;                                  // whole workgroup
    const int my_units = (unit_end - unit + unit_step - 1) / unit_step;
    const int total = my_units * nch;                              // chunk steps = barriers, the same for every wave

    if (TOUCH && wave == nqw + NLOADER) {
        // ---- the wave that touches the weights of the launches behind this one, a line to a lane, FLIGHT lines at a time, and ends: the
        // barriers behind the first are without it
        constexpr uint32_t LINE = 128;
        constexpr int FLIGHT = 4;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(touch), 0, (int)touch_bytes, 0x00020000);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();              // behind the first chunk, which everyone waits for
        asm volatile("" ::: "memory");
        const uint32_t step = (uint32_t)grid * 64 * LINE;
        for (uint32_t at = blockIdx.x * 64 * LINE; at < touch_bytes; at += FLIGHT * step) {
            uint32_t v[FLIGHT];
#pragma unroll
            for (int i = 0; i < FLIGHT; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(at + i * step + lane * LINE), 0, 0);
#pragma unroll
            for (int i = 0; i < FLIGHT; ++i) asm volatile("" ::"v"(v[i]));
        }
        return;
    }

    if (loader) {
        // ---- loader waves: loader 0 brings the K part of every chunk, loader 1 the V part, LPW loads of
        // 1 KB each (64 lanes x 16 bytes, contiguous in LDS); lane l of load s fetches the 16 bytes at linear
        // byte s*1024 + 16 l of the part, i.e. row lin / ROWB, piece(lin % ROWB / 16) of the row.  Rows at or past T
        // lie past the end of the buffer descriptor (per-lane offset, which the bounds check covers) and read
        // as zeros.
        const int lw = wave - nqw;
        int goff[LPW];
#pragma unroll
        for (int s = 0; s < LPW; ++s) {
            const int lin = s * 1024 + lane * 16;
            goff[s] = (lin / ROWB) * row_bytes + piece<DH>(lin / ROWB, lin % ROWB / 16) * 16;      // (its own inverse)
        }
        int pf_unit = unit, pf_pair = unit / ng, pf_chunk = 0;       // the next chunk to fetch
        auto issue = [&](int buf) {
            const uint16_t *part = qkv + (size_t)(pf_pair / H) * T * 3 * D + (size_t)(pf_pair % H) * DH + (size_t)(1 + lw) * D;
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(part), 0, seg_bytes, 0x00020000);
            const int base = pf_chunk * CK * row_bytes;
            char *dst = lds + buf * BUFB + lw * PARTB;
#pragma unroll
            for (int s = 0; s < LPW; ++s)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(dst + s * 1024), 16, base + goff[s], 0, 0, 0);
            if (++pf_chunk == nch) {
                pf_chunk = 0;
                pf_unit += unit_step;
                pf_pair = pf_unit / ng;
            }
        };
        // Chunk 0 and its successor go out first, alone (everyone waits for them); from then on the loader
        // tops the ring up to DEPTH chunks ahead right after each barrier, which is where a buffer comes free.
        int issued = 0;
        for (int j = 0; j < total; ++j) {
            while (issued < total && issued < j + 2) issue(issued++ % NBUF);
            // chunk j has landed once at most the loads of the chunks issued after it are outstanding
            switch (issued - 1 - j) {
            case 0: EP_ATTN_WAIT_VMCNT(0); break;
            case 1: EP_ATTN_WAIT_VMCNT(1 * LPW); break;
            case 2: EP_ATTN_WAIT_VMCNT(2 * LPW); break;
            case 3: EP_ATTN_WAIT_VMCNT(3 * LPW); break;
            default: EP_ATTN_WAIT_VMCNT(4 * LPW); break;
            }
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();          // chunk j is there; the query waves are done with chunk j - 1
            asm volatile("" ::: "memory");
            while (issued < total && issued < j + 1 + DEPTH) issue(issued++ % NBUF);   // ... whose buffer comes free here
        }
        return;
    }

    // ---- query waves.  With one group to a pair a wave's tile is the same in every unit, and the wave that holds the
    // ragged end of T leaves out a second 16-query block with no query in it.
    if (QW == 32 && (ng > 1 || wave * 32 + 16 < T))
        attn_wave<DH, 2>(qkv, o, lds, T, D, H, ng, nqw, wave, unit, unit_step, my_units, nch, scale_log2e);
    else if (QW == 16 || ng == 1)
        attn_wave<DH, 1>(qkv, o, lds, T, D, H, ng, QW == 16 ? nqw : 0, QW == 16 ? wave : 2 * wave, unit, unit_step, my_units, nch, scale_log2e);
#endif
}

// How the queries of a pair are dealt: tiles of qw queries, ng groups of tiles, one workgroup per (pair, group).
// A unit takes as long as its keys take to stream through and its busiest SIMD to work on them, so while pairs are
// fewer than compute units the queries of a pair are spread over as many of them as there are to a pair
// (microseconds per launch, before -> after, T = 197, d_head 64: 16 pairs 8.5 -> 5.5, 80 pairs 8.8 -> 6.7, 128
// pairs 8.9 -> 7.4; T = 577: 24 pairs 35.1 -> 10.9, 96 pairs 36.3 -> 22.0; T = 257, d_head 80: 16 pairs
// 10.9 -> 6.0); a second round of units would cost more than it saves (160 pairs at T = 197: 9.4 us with one group,
// 12.0 with two).  In one round of units tiles of 16 queries, up to nine waves: a step of 32 keys is a chain (reads, scores, maximum,
// exponentials, second product) that takes a lone wave some 1100 clocks for two blocks of 16 queries and 650 for one,
// and two waves of one block to a SIMD fill each other's waits (80 pairs at T = 197, three groups of five waves: 6.4 us
// against 7.1 with three waves of 32; 48 pairs at T = 577 12.2 against 13.0; 64 pairs at T = 257, d_head 80, 8.0 against
// 9.0).  Beyond nine every wave's reading all keys and values from LDS costs more
// (60 pairs at T = 577: ten waves of 16 queries take 16.7 us, five of 32 15.8).  More than 320 queries to a group
// do not fit the query waves of a workgroup.  No more groups than hold a query: 17 tiles (T = 257) in groups of two are
// nine, and the workgroups of seven more would bring in all keys and values for nothing.
struct AttnPlan { int qw, ng; };

AttnPlan plan_attention(int64_t pairs, int T, int n_cu)
{
    const int t32 = (T + 31) / 32, t16 = (T + 15) / 16;
    const int most = (int)(n_cu / pairs);                           // groups to a pair that fit one round
    const int ng_min = (t32 + MAXQW - 1) / MAXQW;
    if (most <= ng_min) return {32, ng_min};
    const int ng = most < t16 ? most : t16;
    const int w32 = (t32 + ng - 1) / ng, w16 = (t16 + ng - 1) / ng;     // tiles to a group
    if (w16 <= 9) return {16, (t16 + w16 - 1) / w16};
    return {32, (t32 + w32 - 1) / w32};
}

int query_waves(int T, int qw, int ng) { return ((T + qw - 1) / qw + ng - 1) / ng; }

template <int DH, int QW, bool TOUCH>
hipError_t launch_as(const uint16_t *qkv, uint16_t *o, int B, int T, int D, int H, int ng, int n_cu, EpTouch touch, hipStream_t s)
{
    using S = StreamShape<DH>;
    auto kern = attn_stream_kernel<DH, QW, TOUCH>;
    static EpSmemLimit smem_limit;
    const hipError_t e = smem_limit.ensure(reinterpret_cast<const void *>(kern), (int)S::smem);
    if (e != hipSuccess) return e;
    const int nqw = query_waves(T, QW, ng);
    if (nqw + (TOUCH ? 1 : 0) > MAXQW) return hipErrorInvalidValue;
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)DH);
    const int64_t n_units = (int64_t)B * H * ng;
    if (n_units > 0x7FFFFFFF) return hipErrorInvalidValue;
    // at most one workgroup per compute unit, and no more than the rounds of units need: 272 units on 136 workgroups
    // of two take 15.3 us where 256 workgroups, 16 of them with a second unit, take 16.2
    const int64_t rounds = (n_units + n_cu - 1) / n_cu;
    const int grid = (int)((n_units + rounds - 1) / rounds);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3((nqw + NLOADER + (TOUCH ? 1 : 0)) * 64), S::smem, s, qkv, o, T, D, H, ng, nqw, grid,
                       (int)(n_units / grid), (int)(n_units % grid), scale_log2e, touch.bytes, touch.p);
    return hipGetLastError();
}

template <int DH, int QW>
hipError_t launch_stream(const uint16_t *qkv, uint16_t *o, int B, int T, int D, int H, int ng, int n_cu, EpTouch touch, hipStream_t s)
{
    // where the query waves leave room for a wave more: all do but those of 289 to 320 tokens and, of higher counts, the like
    if (touch.bytes && touch.bytes <= MAX_TOUCH && query_waves(T, QW, ng) < MAXQW)
        return launch_as<DH, QW, true>(qkv, o, B, T, D, H, ng, n_cu, touch, s);
    return launch_as<DH, QW, false>(qkv, o, B, T, D, H, ng, n_cu, touch, s);
}

template <int DH>
hipError_t launch_attention(const uint16_t *qkv, uint16_t *o, int B, int T, int D, int H, EpTouch touch, hipStream_t s)
{
    int n_cu = 0;
    const hipError_t e = ep_device_cu_count(&n_cu);
    if (e != hipSuccess) return e;
    const AttnPlan p = plan_attention((int64_t)B * H, T, n_cu);
    return p.qw == 32 ? launch_stream<DH, 32>(qkv, o, B, T, D, H, p.ng, n_cu, touch, s)
                      : launch_stream<DH, 16>(qkv, o, B, T, D, H, p.ng, n_cu, touch, s);
}

}  // namespace

extern "C" void ep_query_attention_plan(int64_t pairs, int32_t T, int32_t cus, int32_t *qw, int32_t *ng)
{
    const AttnPlan p = plan_attention(pairs, T, cus);
    *qw = p.qw;
    *ng = p.ng;
}

bool ep_bf16_attention_touches(int64_t pairs, int T)
{
    int n_cu = 0;
    if (pairs <= 0 || T <= 0) return false;
    if (ep_device_cu_count(&n_cu) != hipSuccess) n_cu = 256;       // asked without a GPU
    const AttnPlan p = plan_attention(pairs, T, n_cu);
    return query_waves(T, p.qw, p.ng) < MAXQW;
}

bool ep_bf16_attention_supported(int T, int d_head)
{
    return T >= 1 && T <= 4096 && (d_head == 64 || d_head == 80);
}

hipError_t ep_bf16_attention(const uint16_t *qkv, uint16_t *o, int B, int T, int D, int H, EpTouch touch, hipStream_t s)
{
    if (B <= 0) return hipSuccess;
    if (H <= 0 || D % H != 0 || !ep_bf16_attention_supported(T, D / H)) return hipErrorInvalidValue;
    if ((int64_t)B * H > 0x7FFFFFFF || (int64_t)T * 3 * D * 2 >= 0x7FFFFFF0ll) return hipErrorInvalidValue;
    switch (D / H) {
    case 64: return launch_attention<64>(qkv, o, B, T, D, H, touch, s);
    case 80: return launch_attention<80>(qkv, o, B, T, D, H, touch, s);
    }
    return hipErrorInvalidValue;
}
