// Prefill attention: causal attention of all prompt positions of a sequence against the K/V rows that
// the same prefill pass has just written into the cache (tiled, online softmax, f16 MFMA).
//
// Layout of the computation for gfx950 (wavefront = 64 lanes, v_mfma_f32_32x32x16_f16):
//   * workgroup = NW wavefronts = 32 NW consecutive query positions of one (sequence, query head);
//     wavefront w owns 32 of them and keeps its Q fragments in registers for the whole kernel;
//   * scores are computed TRANSPOSED, S^T = K Q^T, so that in the accumulator layout a lane holds one
//     query column and 16 key rows: the softmax statistics of a query are lane-local (one shuffle
//     joins the two half-wavefronts), and the probabilities already sit in the register layout of the
//     B operand of the second product O^T += V^T P^T -- no shuffle or LDS round trip for P;
//   * a tile of 8 NW cache rows is staged once per workgroup: the rows of tile i + 1 are in flight (registers) while
//     tile i is multiplied, are then converted and stored to the other of two LDS buffers, and one barrier ends the trip;
//   * V is stored transposed, the keys of a row in the order in which the accumulator holds the probabilities, so a V^T
//     fragment is one 16-byte LDS read.
// Softmax and accumulation are fp32; probabilities are rounded to half for the matrix cores (two terms over block-scaled rows).
//
// What bounds it: long prompts the matrix cores together with the vector work of the softmax (719-886 TFLOP/s executed at 2048 and
// 4096 positions); short ones the chain of latencies of a wavefront's tiles: of 5800 cycles per 32 keys with one wavefront per SIMD, 2200
// are the two products, 1750 the softmax, 1300 the conversion to LDS.  What keeps the rest of that chain short:
//   * consecutive rows are read through descriptors (one address register per operand and no comparison; rows of page lists, and
//     sequences beyond 32-bit offsets, by a general path: template parameter LINEAR);
//   * K and V fragments are read one product ahead; the queries are requested behind the first tile and arrive while it is staged;
//   * there is no barrier after the last tile, so the wavefronts above its diagonal store their rows while the others multiply.
//   Without these three: one prompt of 64 / 128 / 256 positions, 32 heads, block-scaled rows 12.6 / 20.4 / 33.4 us, now 10.4 / 16.7 / 28.3.
// Compared with 128 queries per workgroup, 16-bit gathers from untransposed V (128 LDS reads per 32 keys and wavefront instead of 16), a
// single buffer and every element scaled in fp32 on its way to LDS, us a launch, that -> now, block-scaled rows, 32 heads: 8 x 2048
// positions 3530 -> 1150, 32 x 512 1000 -> 440, 32 x 384 465 -> 284, 37 x 205 288 -> 174, 128 x 128 380 -> 244, 1 x 1000 118 -> 84, 1 x 128
// 17.8 -> 15.6; half rows, 32/8 heads, 16 x 1024 681 -> 411.
// Error of the two-term output against 64 bits (normal rows, scores of deviation 1.5, that -> now): 128 keys 3.05e-7 -> 2.27e-7,
// 333 keys 3.67e-7 -> 2.76e-7, 1000 keys 4.61e-7 -> 3.49e-7; scores all equal 1.82e-7 -> 1.85e-7, and all scales equal as well 1.82e-7 -> 2.02e-7.
#include <type_traits>

#include "kernels.h"

#define PA_PSHIFT 14        // probabilities over block-scaled rows are split at this power of two above their value (products
#define PA_PSCALE 16384.f   // with a scale stay below 2^15), which keeps the low term of a small one out of the subnormal halves

// Staging of block-scaled rows.  Two int16 elements n -> the two-term half split of n / 64 (both exact: hi = n / 64 rounded to
// half, lo = the rest, a multiple of 1/64).  The bits 15..6 and 5..0 become halves by placing them in the mantissa of 1024, so
// everything is packed 16-bit arithmetic and no element is ever widened; the row scales are applied to the scores (K) and to the
// probabilities (V) in fp32 instead.
__device__ __forceinline__ void pa_split_i16x2(uint32_t n, uint32_t &hi, uint32_t &lo) {
    typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
    const uint32_t top = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2_t, n) >> 6) ^ 0x66006600u;  // 1024 + (n >> 6) + 512
    const uint32_t bot = (n & 0x003f003fu) | 0x64006400u;                                                 // 1024 + (n & 63)
    const f16x2_t a = __builtin_bit_cast(f16x2_t, top) - (_Float16)1536.f;
    const f16x2_t b = __builtin_bit_cast(f16x2_t, bot) * (_Float16)0.015625f - (_Float16)16.f;
    const f16x2_t s = a + b;  // |a| >= |b| or a = 0: the rounding error of the sum is b - (s - a), exactly
    hi = __builtin_bit_cast(uint32_t, s);
    lo = __builtin_bit_cast(uint32_t, b - (s - a));
}

// 4 rows x 2 W columns of 16-bit values (W packed words per row) -> the columns, 4 rows each
template <int W>
__device__ __forceinline__ void pa_transpose4(const uint32_t (&r)[4][W], u32x2_t (&c)[2 * W]) {
#pragma unroll
    for (int p = 0; p < W; ++p) {
        c[2 * p].x = __builtin_amdgcn_perm(r[1][p], r[0][p], 0x05040100u);
        c[2 * p].y = __builtin_amdgcn_perm(r[3][p], r[2][p], 0x05040100u);
        c[2 * p + 1].x = __builtin_amdgcn_perm(r[1][p], r[0][p], 0x07060302u);
        c[2 * p + 1].y = __builtin_amdgcn_perm(r[3][p], r[2][p], 0x07060302u);
    }
}

// largest of 32 lanes, in lanes 31 and 63 (values >= 0): register-to-register moves, a tenth of the latency of shuffles through LDS
__device__ __forceinline__ float pa_max32(float v) {
    auto from = [](float x, auto ctrl) {  // the lanes that the move does not reach get 0
        return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v = fmaxf(v, from(v, std::integral_constant<int, 0x111>{}));  // lane - 1, - 2, - 4, - 8 of the same 16
    v = fmaxf(v, from(v, std::integral_constant<int, 0x112>{}));
    v = fmaxf(v, from(v, std::integral_constant<int, 0x114>{}));
    v = fmaxf(v, from(v, std::integral_constant<int, 0x118>{}));
    return fmaxf(v, from(v, std::integral_constant<int, 0x142>{}));  // lane 15 of the 16 before
}
__device__ __forceinline__ uint32_t pa_exponent(float v) { return __float_as_uint(v) & 0x7f800000u; }

// LDS of one buffer: K [terms][KT][HD + 8] and V^T [terms][HD][KT + 8] halves, then (block-scaled rows) the score factors and
// the normalised value scales [KT] and of every 32 rows the value reference and the mask of rows without a finite scale.  Both row
// strides are 4 banks modulo 16, which keeps the 16-byte fragment reads free of conflicts; the 16-byte pieces of a V^T row are permuted
// by the row's 16-row group so that the transposing 8-byte stores of a wavefront spread over all banks.
template <int HD, bool I16, int NW>
struct PaTile {
    static constexpr int KT = 8 * NW, NT = I16 ? 2 : 1;
    static constexpr int KSTR = HD + 8, VSTR = KT + 8;
    static constexpr int K_HALVES = NT * KT * KSTR, V_HALVES = NT * HD * VSTR;
    static constexpr int BYTES = (K_HALVES + V_HALVES) * 2 + (I16 ? (2 * KT + 4) * 4 : 0);
    // piece p (keys 8 p .. + 7) of row dim is kept in place p ^ (dim / 16) of the row, modulo the KT / 8 pieces
    __device__ static __forceinline__ int v_place(int piece, int dim) { return ((piece ^ (dim >> 4)) & (KT / 8 - 1)) * 8; }
};

// I16: the cache rows are 16-bit block-scaled fixed point (KvMap::kscale / vscale).  A row element has more
// significant bits than a half holds, so it enters the matrix cores as a two-term half sum hi + lo, and so do the
// probabilities and -- when q_lo is given -- the queries: each of the two products of a tile becomes three matrix
// instructions (hi x hi, lo x hi, hi x lo; lo x lo is at most 2^-24 of a product) and no operand carries a single half rounding.
// A probability is multiplied with its row's value scale before it is split; so that the product stays in the normal range of a
// half, scales are taken relative to a power of two, the one at or below the largest scale up to the 32 rows at hand (the reference,
// part of the online rescale).  The grid of the low term is 2^-25 of a probability for rows of 2^-14 of the reference and larger, the
// grid that probabilities split by themselves would have; below that a row loses one bit per factor of two.  Rows that a query does not
// see have no part in its reference: in the diagonal block every query takes its own, as a shift of its running maximum.
// A row whose value scale is not finite makes the output of the queries that see it NaN (stored as the largest half, like any NaN).
// q_lo (optional, I16 only): second half term of q, laid out like q.
// out_lo (optional): half(o - half(o)), the second term of the output for a two-term output projection.
// xcd_heads > 0: heads of all sequences, a multiple of 8; the workgroups of one head and of its neighbours run on one XCD, whose
// L2 then reads their cache rows once.
template <int HD, bool I16, int NW, bool LINEAR>
__global__ __launch_bounds__(64 * NW, 2) void prefill_attention_kernel(const f16_t *__restrict__ q, const f16_t *__restrict__ q_lo,
                                                                       const f16_t *__restrict__ kc, const f16_t *__restrict__ vc,
                                                                       f16_t *__restrict__ out, f16_t *__restrict__ out_lo, int b0,
                                                                       int T, int Hq, int Hkv, int S, KvMap map,
                                                                       const int32_t *__restrict__ d_valid, int xcd_heads) {
    using L = PaTile<HD, I16, NW>;
    constexpr int KT = L::KT, NT = L::NT, THREADS = 64 * NW, ROWS = 32 * NW;
    constexpr int KS = HD / 16;   // k16 steps of the QK product
    constexpr int ET = HD / 32;   // 32-row tiles of O^T
    constexpr int KP = HD / 64;   // 16-byte pieces of K per thread and tile: KT * HD / 8 = KP * THREADS
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), half = lane >> 5, l32 = lane & 31;
    int qt = blockIdx.x, u = blockIdx.y, bl = blockIdx.z;  // query tile, query head, sequence within the chunk
    if (xcd_heads) {
        const int id = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x, xcd = id & 7, nth = id >> 3;
        const int head = xcd * (xcd_heads >> 3) + nth / (int)gridDim.x;
        qt = nth % (int)gridDim.x;
        u = head % Hq;
        bl = head / Hq;
    }
    qt = gridDim.x - 1 - qt;  // the longest rows first
    const int kvh = u / (Hq / Hkv);
    const int q0 = qt * ROWS + w * 32;  // first query position of this wavefront
    const int qpos = q0 + l32;          // this lane's query column
    const size_t ldq = (size_t)Hq * HD;

    int n_keys = T;  // keys this sequence really has in the cache
    if (d_valid) {
        int nv = d_valid[b0 + bl];
        n_keys = nv < 1 ? 1 : (nv > T ? T : nv);
    }

    f32x16_t oacc[ET];
#pragma unroll
    for (int e = 0; e < ET; ++e)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[e][i] = 0.f;
    float mrun = -INFINITY, lrun = 0.f;  // running max (shared by both halves) and this half's partial sum, base 2
    float vref = 0.f;                    // value reference the accumulators are relative to
    const float c2 = rsqrtf((float)HD) * 1.44269504088896340736f;  // scores times this are exponents of 2

    // ---- staging: K as rows (16-byte pieces), V as groups of 4 rows x HD / 32 columns, one per thread, the scales by the first KT
    //      threads (wavefront 0)
    constexpr int VW = HD / 64;  // words of 2 columns
    const int vrow = t / 32 * 4, vcol = t % 32 * (2 * VW);
    u32x4_t kreg[KP];
    uint32_t vreg[4][VW];
    float kscr = 0.f, vscr = 0.f, vmax_run = 0.f;
    // LINEAR: the keys of a sequence are consecutive rows.  The descriptors end with its last key, so rows that it does not have read as
    // zeros, and a tile takes three address registers and no comparison.
    const size_t slab = LINEAR ? ((size_t)(b0 + bl) * Hkv + kvh) * S : 0;
    auto rsrc = [&](const void *p, int row_bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, LINEAR ? n_keys * row_bytes : 0, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t kr = rsrc(kc + slab * HD, HD * 2), vr = rsrc(vc + slab * HD, HD * 2);
    const __amdgpu_buffer_rsrc_t ksr = rsrc(I16 ? map.kscale + slab : nullptr, 4), vsr = rsrc(I16 ? map.vscale + slab : nullptr, 4);
    auto fetch = [&](int kt) {
        if constexpr (LINEAR) {
#pragma unroll
            for (int i = 0; i < KP; ++i) kreg[i] = __builtin_amdgcn_raw_buffer_load_b128(kr, t * 16 + (kt * KP + i) * THREADS * 16, 0, 0);
            const int vat = ((kt * KT + vrow) * HD + vcol) * 2;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (VW == 2) {
                    const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(vr, vat + r * HD * 2, 0, 0);
                    vreg[r][0] = v.x; vreg[r][1] = v.y;
                } else vreg[r][0] = __builtin_amdgcn_raw_buffer_load_b32(vr, vat + r * HD * 2, 0, 0);
            }
            if (I16 && w == 0) {
                const int at = lane < KT ? (kt * KT + lane) * 4 : 0x7fffff00;  // the lanes behind a tile of 32 rows: out of range
                kscr = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ksr, at, 0, 0));
                vscr = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(vsr, at, 0, 0));
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < KP; ++i) {
            const int idx = t + i * THREADS, key = kt * KT + idx / (HD / 8);
            kreg[i] = u32x4_t{0u, 0u, 0u, 0u};
            if (key < n_keys)  // rows past the prompt may hold arbitrary bits: keep them out (0 * NaN)
                kreg[i] = *reinterpret_cast<const u32x4_t *>(kc + kv_row_index(map, b0 + bl, kvh, Hkv, S, key) * HD + (idx % (HD / 8)) * 8);
        }
        const int key4 = kt * KT + vrow;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int p = 0; p < VW; ++p) vreg[r][p] = 0u;
        if (key4 < n_keys) {  // 4 aligned rows share a page (a page holds a power of two >= 16)
            const f16_t *vp = vc + kv_row_index(map, b0 + bl, kvh, Hkv, S, key4) * HD + vcol;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (key4 + r < n_keys) {
                    if constexpr (VW == 2) {
                        const u32x2_t v = *reinterpret_cast<const u32x2_t *>(vp + r * HD);
                        vreg[r][0] = v.x; vreg[r][1] = v.y;
                    } else vreg[r][0] = *reinterpret_cast<const uint32_t *>(vp + r * HD);
                }
        }
        if (I16 && w == 0) {
            const int key = kt * KT + lane;
            kscr = 0.f;
            vscr = 0.f;
            if (lane < KT && key < n_keys) {
                const size_t rowi = kv_row_index(map, b0 + bl, kvh, Hkv, S, key);
                kscr = map.kscale[rowi];
                vscr = map.vscale[rowi];
            }
        }
    };
    auto stash = [&](int buf) {
        f16_t *ks = reinterpret_cast<f16_t *>(smem + buf * L::BYTES), *vs = ks + L::K_HALVES;
#pragma unroll
        for (int i = 0; i < KP; ++i) {
            const int idx = t + i * THREADS;
            f16_t *at = ks + idx / (HD / 8) * L::KSTR + (idx % (HD / 8)) * 8;
            if (I16) {
                u32x4_t hi, lo;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t h, l;
                    pa_split_i16x2(kreg[i][j], h, l);
                    hi[j] = h;
                    lo[j] = l;
                }
                *reinterpret_cast<u32x4_t *>(at) = hi;
                *reinterpret_cast<u32x4_t *>(at + KT * L::KSTR) = lo;
            } else {
                *reinterpret_cast<u32x4_t *>(at) = kreg[i];
            }
        }
        // rows 8a + 4h + 0..3 of a 32-row block are slots 4 (a & 1) + 0..3 of the fragment (step a / 2, half-wavefront h)
        const int g = vrow / 4, piece = (g >> 3) * 4 + ((g >> 2) & 1) * 2 + (g & 1), slot = ((g >> 1) & 1) * 4;
        f16_t *at = vs + vcol * L::VSTR + L::v_place(piece, vcol) + slot;  // of the group's first column; all its columns have one place
        u32x2_t col[2 * VW];
        if (I16) {
            uint32_t hi[4][VW], low[4][VW];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int p = 0; p < VW; ++p) pa_split_i16x2(vreg[r][p], hi[r][p], low[r][p]);
            pa_transpose4(hi, col);
#pragma unroll
            for (int i = 0; i < 2 * VW; ++i) *reinterpret_cast<u32x2_t *>(at + i * L::VSTR) = col[i];
            pa_transpose4(low, col);
#pragma unroll
            for (int i = 0; i < 2 * VW; ++i) *reinterpret_cast<u32x2_t *>(at + (HD + i) * L::VSTR) = col[i];
        } else {
            pa_transpose4(vreg, col);
#pragma unroll
            for (int i = 0; i < 2 * VW; ++i) *reinterpret_cast<u32x2_t *>(at + i * L::VSTR) = col[i];
        }
        if (I16 && w == 0) {
            float *sc = reinterpret_cast<float *>(vs + L::V_HALVES);
            const bool finite = fabsf(vscr) < INFINITY;  // not for a NaN
            const float m = pa_max32(finite ? fabsf(vscr) : 0.f);
            const float top0 = fmaxf(vmax_run, __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(m), 31)));
            vmax_run = fmaxf(top0, __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(m), 63)));
            const float top = lane < 32 ? top0 : vmax_run;
            // the power of two at or below the largest scale: taking it out is exact
            const float ref = top > 0.f ? fmaxf(__uint_as_float(pa_exponent(top)), 1.17549435e-38f) : 0.f;
            const uint64_t bad = __ballot(!finite);
            if (lane < KT) {
                sc[lane] = kscr * (64.f * c2);
                sc[KT + lane] = finite && ref > 0.f ? ldexpf(vscr, PA_PSHIFT + 127 - (int)(__float_as_uint(ref) >> 23)) : 0.f;
            }
            if (lane < KT && (lane & 31) == 0) {
                float *blk = sc + 2 * KT + (lane >> 5) * 2;
                blk[0] = ref;
                reinterpret_cast<uint32_t *>(blk)[1] = (uint32_t)(bad >> lane);
            }
        }
    };

    int last_q = qt * ROWS + ROWS - 1;
    if (last_q > T - 1) last_q = T - 1;
    const int n_tiles = last_q / KT + 1;  // key tiles any wavefront of the workgroup needs
    fetch(0);
    // Q fragments (B operand of S^T = K Q^T): lane = (query column l32, hd slice half*8 + 16*s); on their way while the first tile is staged
    f16x8_t qf[KS], ql[I16 ? KS : 1];
    const bool two_q = I16 && q_lo != nullptr;  // uniform
    {
        const int qrow = qpos < T ? qpos : T - 1;
        const size_t qoff = ((size_t)bl * T + qrow) * ldq + (size_t)u * HD + half * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s) qf[s] = *reinterpret_cast<const f16x8_t *>(q + qoff + s * 16);
        if (I16) {
            const f16_t *qp = two_q ? q_lo : q;  // without a second term: not used
#pragma unroll
            for (int s = 0; s < KS; ++s) ql[s] = *reinterpret_cast<const f16x8_t *>(qp + qoff + s * 16);
        }
    }
    stash(0);
    __syncthreads();
    for (int kt = 0; kt < n_tiles; ++kt) {
        const bool more = kt + 1 < n_tiles;
        if (more) fetch(kt + 1);
        const f16_t *ks = reinterpret_cast<const f16_t *>(smem + (kt & 1) * L::BYTES), *vs = ks + L::K_HALVES;
        const float *sc = reinterpret_cast<const float *>(vs + L::V_HALVES);
#pragma unroll 1
        for (int sub = 0; sub < KT / 32; ++sub) {
            const int key0 = kt * KT + sub * 32;
            if (key0 > q0 + 31 || q0 >= T) break;  // above this wavefront's diagonal, or no query (uniform per wavefront)
            // The small products of a two-term operand are summed on their own: 8 instead of 24 roundings at the magnitude of the
            // score (with one accumulator the output error over 333 keys is a quarter larger), and two shorter chains.
            f32x16_t sacc, slow;
#pragma unroll
            for (int i = 0; i < 16; ++i) sacc[i] = slow[i] = 0.f;
            // fragments are read one k-step ahead of their products
            auto scores = [&](auto two_tag) {
                f16x8_t kf[2][NT];
                auto read_k = [&](int s) {
#pragma unroll
                    for (int tm = 0; tm < NT; ++tm)
                        kf[s & 1][tm] = *reinterpret_cast<const f16x8_t *>(ks + (tm * KT + sub * 32 + l32) * L::KSTR + half * 8 + s * 16);
                };
                read_k(0);
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    if (s + 1 < KS) read_k(s + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    sacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[s & 1][0], qf[s], sacc, 0, 0, 0);
                    if (decltype(two_tag)::value) slow = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[s & 1][0], ql[I16 ? s : 0], slow, 0, 0, 0);
                    if (I16) slow = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[s & 1][NT - 1], qf[s], slow, 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            if (I16 && two_q) scores(std::true_type{});
            else scores(std::false_type{});
            if (I16) sacc += slow;
            // register i holds key row (i/4)*8 + half*4 + (i%4) of the block, query column l32
            const float *blk = sc + 2 * KT + sub * 2;
            float rel = 1.f, vnew = 0.f;
            if (I16) vnew = blk[0];
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                f32x4_t f = {c2, c2, c2, c2};
                if (I16) f = *reinterpret_cast<const f32x4_t *>(sc + sub * 32 + i4 * 8 + half * 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) sacc[i4 * 4 + j] *= f[j];
            }
            const bool diagonal = key0 == q0;
            float seen = 0.f;  // largest normalised value scale among the rows of the block that this query sees
            if (diagonal) {    // causal mask
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    f32x4_t f = {0.f, 0.f, 0.f, 0.f};
                    if (I16) f = *reinterpret_cast<const f32x4_t *>(sc + KT + sub * 32 + i4 * 8 + half * 4);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (key0 + i4 * 8 + half * 4 + j > qpos) sacc[i4 * 4 + j] = -INFINITY;
                        else if (I16) seen = fmaxf(seen, fabsf(f[j]));
                    }
                }
            }
            float tmax = sacc[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, sacc[i]);
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
            float mnew = fmaxf(mrun, tmax);  // finite: key 0 is visible to every query
            if (I16 && vnew != vref) rel = vref / vnew;  // powers of two; the reference only grows, so it is positive here
            if (I16 && diagonal) {
                // The query's own reference, the largest of the rows that it sees, may be 2^k below the block's: its probabilities are
                // taken 2^k times larger, in numerator and denominator (this block is the query's last).
                seen = fmaxf(seen, __shfl_xor(seen, 32, 64));
                const float own = fmaxf(vref, __uint_as_float(pa_exponent(seen)) * (vnew * (1.f / PA_PSCALE)));
                const int shift = (int)(__float_as_uint(vnew) >> 23) - (int)(__float_as_uint(own) >> 23);
                if (own > 0.f) mnew -= (float)(shift < 100 ? shift : 100);
            }
            if (I16) {  // rows without a finite value scale
                const uint32_t bad = reinterpret_cast<const uint32_t *>(blk)[1];
                if (bad & (diagonal ? (2u << l32) - 1u : ~0u)) lrun = __builtin_nanf("");
            }
            if (__any(mnew != mrun) || rel != 1.f) {
                const float alpha = __builtin_amdgcn_exp2f(mrun - mnew);
                lrun *= alpha;
#pragma unroll
                for (int e = 0; e < ET; ++e)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[e][i] *= alpha * rel;
                mrun = mnew;
                vref = vnew;
            }
            f16x8_t vf[2][NT];  // V^T fragments, read one product ahead
            // place of piece 4 sub + 2 s + half of row 32 e + l32, bit by bit: what depends on the lane is one address
            auto read_v = [&](int n) {
                const int s = n / ET, e = n % ET;
                const f16_t *at = vs + l32 * L::VSTR + (half ^ (l32 >> 4)) * 8 + (KT == 64 ? (sub ^ (e >> 1)) * 32 : 0);
#pragma unroll
                for (int tm = 0; tm < NT; ++tm)
                    vf[n & 1][tm] = *reinterpret_cast<const f16x8_t *>(at + (tm * HD + e * 32) * L::VSTR + (s ^ (e & 1)) * 16);
            };
            read_v(0);
            f16x8_t pf[2], pl[I16 ? 2 : 1];
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                f32x4_t f = {1.f, 1.f, 1.f, 1.f};
                if (I16) f = *reinterpret_cast<const f32x4_t *>(sc + KT + sub * 32 + i4 * 8 + half * 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int i = i4 * 4 + j;
                    float p = __builtin_amdgcn_exp2f(sacc[i] - mnew);
                    lrun += p;
                    if (I16) {
                        p *= f[j];
                        // The product is a value of its own: contracted into the conversion, one use of ph would come from the
                        // unrounded product and the other from the rounded one, and where these fall on different halves the two
                        // terms miss p by a half's spacing (2.0e-6 instead of 3.7e-7 over 333 keys).
                        asm("" : "+v"(p));
                    }
                    const _Float16 ph = (_Float16)p;
                    pf[i >> 3][i & 7] = ph;
                    if (I16) pl[i >> 3][i & 7] = (_Float16)(p - (float)ph);
                }
            }
            // O^T += V^T P^T.  Slot j of k-step s in lane-half h stands for key (2s + j/4)*8 + h*4 + j%4 -- the
            // key that accumulator register s*8 + j already holds, so P needs no data movement.
#pragma unroll
            for (int n = 0; n < 2 * ET; ++n) {
                const int s = n / ET, e = n % ET;
                if (n + 1 < 2 * ET) read_v(n + 1);
                __builtin_amdgcn_sched_barrier(0);
                oacc[e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[n & 1][0], pf[s], oacc[e], 0, 0, 0);
                if (I16) {
                    oacc[e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[n & 1][0], pl[s], oacc[e], 0, 0, 0);
                    oacc[e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[n & 1][NT - 1], pf[s], oacc[e], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!more) break;    // the wavefronts above the diagonal of the last tile store their rows while the others multiply
        stash((kt + 1) & 1);  // the buffer of tile kt - 1: read before the last barrier
        __syncthreads();
    }

    // normalise and store: lane = query column; register i of tile e is head_dim row e*32 + (i/4)*8 + half*4 + i%4
    float ltot = lrun + __shfl_xor(lrun, 32, 64);
    if (qpos < T) {
        float inv = (I16 ? vref * (64.f / PA_PSCALE) : 1.0f) / ltot;
        f16_t *op = out + ((size_t)bl * T + qpos) * ldq + (size_t)u * HD;
#pragma unroll
        for (int e = 0; e < ET; ++e)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                u32x2_t o2;
                o2.x = pack_f16x2(oacc[e][i4 * 4 + 0] * inv, oacc[e][i4 * 4 + 1] * inv);
                o2.y = pack_f16x2(oacc[e][i4 * 4 + 2] * inv, oacc[e][i4 * 4 + 3] * inv);
                *reinterpret_cast<u32x2_t *>(op + e * 32 + i4 * 8 + half * 4) = o2;
                if (out_lo) {
                    u32x2_t l2;
                    l2.x = pack_f16x2_lo(oacc[e][i4 * 4 + 0] * inv, oacc[e][i4 * 4 + 1] * inv, o2.x);
                    l2.y = pack_f16x2_lo(oacc[e][i4 * 4 + 2] * inv, oacc[e][i4 * 4 + 3] * inv, o2.y);
                    *reinterpret_cast<u32x2_t *>(out_lo + (op - out) + e * 32 + i4 * 8 + half * 4) = l2;
                }
            }
    }
}

template <int HD, bool I16, int NW, bool LINEAR>
static void launch_pa(const f16_t *q, const f16_t *q_lo, const f16_t *kc, const f16_t *vc, f16_t *out, f16_t *out_lo, int nb, int b0,
                      int T, int Hq, int Hkv, int S, const KvMap &map, const int32_t *d_valid, hipStream_t st) {
    constexpr int lds = 2 * PaTile<HD, I16, NW>::BYTES;
    static_assert(lds <= 160 * 1024, "two buffers fit a compute unit");
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&prefill_attention_kernel<HD, I16, NW, LINEAR>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    (void)attr;
    dim3 grid(ceil_div(T, 32 * NW), Hq, nb);
    const int64_t heads = (int64_t)Hq * nb;
    const int xcd_heads = heads % 8 == 0 && heads * grid.x < (1ll << 31) ? (int)heads : 0;
    prefill_attention_kernel<HD, I16, NW, LINEAR><<<grid, 64 * NW, lds, st>>>(q, q_lo, kc, vc, out, out_lo, b0, T, Hq, Hkv, S, map, d_valid,
                                                                              xcd_heads);
}

void launch_prefill_attention(const f16_t *q, const f16_t *kc, const f16_t *vc, f16_t *out, int nb, int b0, int T,
                              int Hq, int Hkv, int hd, int S, hipStream_t st, KvMap map, const int32_t *d_valid, f16_t *out_lo,
                              const f16_t *q_lo) {
    if (nb <= 0 || T <= 0) return;
    const bool i16 = map.kscale != nullptr;
    // 256 queries per workgroup from 129 positions on; up to 128 its second half would hold no query.  128 / 256 queries, time ratio, 1-4
    // prompts, 32-64 heads of 128: up to 256 positions 0.87-0.94, 384 1.17-1.38, 512 0.95-1.20, 1024 0.97-1.22, 2048 0.96-1.21, 4096 0.98-1.07;
    // 16 prompts 0.83-1.11.
    const bool wide = T > 128;
    const bool linear = !map.table && (int64_t)T * hd * 2 < (1ll << 30);  // 32-bit offsets inside a sequence
    auto run = [&](auto kernel) { kernel(q, i16 ? q_lo : nullptr, kc, vc, out, out_lo, nb, b0, T, Hq, Hkv, S, map, d_valid, st); };
    auto rows = [&](auto hd_tag, auto i16_tag, auto nw_tag) {
        constexpr int HD = decltype(hd_tag)::value, NW = decltype(nw_tag)::value;
        constexpr bool I16 = decltype(i16_tag)::value;
        linear ? run(launch_pa<HD, I16, NW, true>) : run(launch_pa<HD, I16, NW, false>);
    };
    auto width = [&](auto hd_tag, auto i16_tag) {
        if (wide) rows(hd_tag, i16_tag, std::integral_constant<int, 8>{});
        else rows(hd_tag, i16_tag, std::integral_constant<int, 4>{});
    };
    auto type = [&](auto hd_tag) {
        if (i16) width(hd_tag, std::true_type{});
        else width(hd_tag, std::false_type{});
    };
    if (hd == 128) type(std::integral_constant<int, 128>{});
    else type(std::integral_constant<int, 64>{});
}
