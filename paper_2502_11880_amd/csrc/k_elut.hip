// Integer-weight ELUT formats (c4g2, c5g2, c3g5; Appendix "Insight", Table 3) on int8 MFMA: the group codes are expanded
// to int8 weights in registers and multiplied as a dense int8 contraction, which gives the same integer sums as the
// table lookups of Eq. 3 (the tables hold exactly these products).  One launch serves every weight of a fused group
// and up to 16 tokens per token slice (blockIdx.y); one token can be quantised inside (QX, Sec. 2.1).
//
// Work split.  A work group holds its tokens' codes in LDS for the whole launch and walks the 16-row groups
// blockIdx.x, blockIdx.x + gridDim.x, ...; its waves split K and meet through LDS once per row group.  The packed rows
// are row-major, so lane (r, q) of a wave loads the 16 bytes of row r at 64 kb + 16 q of block kb: a block is 64
// contiguous bytes of 16 rows (256 weights, or 320 for c3g5), and a wave takes U neighbouring blocks so that whole
// 128-byte lines are used by one wave.  The loads of the next step are in flight while a step is multiplied.
//
// Operands of v_mfma_i32_16x16x64_i8 (B column = weight row r, A row = token, rows past the tokens repeat token 0).
// Any order of k works as long as both operands agree, so the weights are taken in the order the codes unpack and the
// activations are put in that order once, when they are copied to LDS:
//   c4g2, c5g2: 32-bit word j of the lane's 16 bytes holds the weights 16 j + e of its 64; field f of the operand
//               holds e = 4 b + (f ^ 1) in byte b
//   c3g5:       byte i of the lane's 16 is the group of weights 5 i + d of its 80; step d takes digit d of all 16
// Codes are offset to be non-negative (w + 2, or t + 1); the offset times the token's code sum, which the first row
// group takes from an MFMA against ones, is subtracted in the epilogue.  Codes past K are zero in LDS.
//
// What bounds it: at one token the start of a launch and the weight stream, at 8 tokens the same (a lane expands 64
// weights with 28 VALU operations in c4g2, about 130 in c5g2, about 130 for 80 weights in c3g5).  The 3B-class layer set at
// 8 tokens, C4G2, 195 -> 46 us per layer
// (table lookups of 4 tokens per launch before: every work group rebuilt the tables of every block it read); one token
// 47 -> 28 us, C5G2 57 -> 40 us, C3G5 51 -> 32 us.
#include "bitnet_internal.hpp"

#include <type_traits>

namespace bitnet {
namespace {

// The formats: weights of C consecutive integers in groups of G, GW groups to a packed 32-bit word.
//   c4g2  {-2, -1, 0, 1}: 4-bit code 4 (w0 + 2) + (w1 + 2), 2 bits per weight
//   c5g2  {-2, .., 2}:    4-bit index |5 w0 + w1| and a sign plane, 2.5 bits per weight
//   c3g5  {-1, 0, 1}:     one byte per group, index |sum_j 3^(4-j) w_j| (0..121) and the sign in bit 7, 1.6 bits
template <int F>
struct ElutFmt;
template <>
struct ElutFmt<kElutC4G2> {
    static constexpr int C = 4, G = 2, GW = 8;
    static constexpr bool kMirror = false;
};
template <>
struct ElutFmt<kElutC5G2> {
    static constexpr int C = 5, G = 2, GW = 8;
    static constexpr bool kMirror = true;
};
template <>
struct ElutFmt<kElutC3G5> {
    static constexpr int C = 3, G = 5, GW = 4;
    static constexpr bool kMirror = true;
};

typedef unsigned short us2 __attribute__((ext_vector_type(2)));

template <int F>
struct MfmaFmt {                                    // c4g2, c5g2
    static constexpr int BK = 256, OFF = 2;
    static constexpr int row_div = 4;               // weights per packed byte
};
template <>
struct MfmaFmt<kElutC3G5> {
    static constexpr int BK = 320, OFF = 1;
    static constexpr int row_div = 5;
};

// Offset codes (w + 2) of the 16 weights of a c5g2 word: indices |5 w0 + w1| of 8 groups in nibbles, their signs in the
// low 8 bits of sg.  Byte arithmetic on four groups at a time; no byte over- or underflows.
__device__ __forceinline__ v4i c5_codes(uint32_t w, uint32_t sg) {
    v4i b;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t idx2 = ((w >> (4 * h)) & 0x0F0F0F0Fu) + 0x02020202u;        // |5 w0 + w1| + 2: 2..14
        // w0 of the positive group: (index + 2) / 5 = 13 (index + 2) / 64 for these; then w1 + 2 in 0..4
        const uint32_t a0 = ((idx2 * 13u) >> 6) & 0x03030303u;
        const uint32_t c1 = idx2 - 5u * a0;
        // sign bit 2 b + h of group 2 b + h to bit 8 b (masked first: the shifted copies never carry into one)
        const uint32_t m = (((sg >> h) & 0x55u) * 0x00041041u) & 0x01010101u;
        const uint32_t m3 = m * 3u;
        // negative groups: w0 + 2 = 2 - a0, w1 + 2 = 4 - c1
        const uint32_t w0 = (a0 ^ m3) + 0x02020202u - m3;                          // 3 - a0 - 1
        const uint32_t w1 = (c1 ^ (m * 7u)) - m3;                                  // 7 - c1 - 3
        if (h == 0) {
            b.x = (int)w1;
            b.y = (int)w0;
        } else {
            b.z = (int)w1;
            b.w = (int)w0;
        }
    }
    return b;
}

// The digits t + 1 of four c3g5 groups (one byte each), most significant first: d[j] holds digit j of the four.
__device__ __forceinline__ void c3_digits(uint32_t g, uint32_t (&d)[5]) {
    const uint32_t s = (g >> 7) & 0x01010101u, s7 = (s << 7) - s;
    // 121 + value: 121 + index, or 127 - index + 121 - 127 where the sign is set; 0..242
    const uint32_t u = ((g & 0x7F7F7F7Fu) ^ s7) + 0x79797979u - s7;
    us2 e = __builtin_bit_cast(us2, u & 0x00FF00FFu), o = __builtin_bit_cast(us2, (u >> 8) & 0x00FF00FFu);
#pragma unroll
    for (int j = 4; j >= 1; --j) {
        const us2 qe = (e * (unsigned short)171) >> (unsigned short)9;             // x / 3 for x < 256
        const us2 qo = (o * (unsigned short)171) >> (unsigned short)9;
        const us2 de = e - qe * (unsigned short)3, dd = o - qo * (unsigned short)3;
        d[j] = __builtin_bit_cast(uint32_t, de) | (__builtin_bit_cast(uint32_t, dd) << 8);
        e = qe;
        o = qo;
    }
    d[0] = __builtin_bit_cast(uint32_t, e) | (__builtin_bit_cast(uint32_t, o) << 8);
}

// 16 codes in the order of the c4g2 and c5g2 operands: byte b of word f is code 4 b + (f ^ 1).
__device__ __forceinline__ v4i order_pairs(v4i a) {
    // v_perm_b32(hi, lo): bytes 0..3 of the selector's numbering are lo, 4..7 hi
    const uint32_t e01 = __builtin_amdgcn_perm((uint32_t)a.y, (uint32_t)a.x, 0x06020400u);  // x0 y0 x2 y2
    const uint32_t o01 = __builtin_amdgcn_perm((uint32_t)a.y, (uint32_t)a.x, 0x07030501u);  // x1 y1 x3 y3
    const uint32_t e23 = __builtin_amdgcn_perm((uint32_t)a.w, (uint32_t)a.z, 0x06020400u);
    const uint32_t o23 = __builtin_amdgcn_perm((uint32_t)a.w, (uint32_t)a.z, 0x07030501u);
    v4i o;
    o.x = (int)__builtin_amdgcn_perm(o23, o01, 0x05040100u);                                // x1 y1 z1 w1
    o.y = (int)__builtin_amdgcn_perm(e23, e01, 0x05040100u);                                // x0 y0 z0 w0
    o.z = (int)__builtin_amdgcn_perm(o23, o01, 0x07060302u);                                // x3 y3 z3 w3
    o.w = (int)__builtin_amdgcn_perm(e23, e01, 0x07060302u);                                // x2 y2 z2 w2
    return o;
}

// Where code k of a token goes in its LDS row.
template <int F>
__device__ __forceinline__ int code_pos(int k) {
    if constexpr (F == kElutC3G5) {
        const int u = k / 80, e = k - 80 * u, i = e / 5, d = e - 5 * i;
        return 80 * u + 16 * d + i;
    } else {
        return (k & ~15) + 4 * ((k & 3) ^ 1) + ((k >> 2) & 3);
    }
}

template <int F, int WAVES, int U, bool QX>
__global__ __launch_bounds__(64 * WAVES) void elut_kernel(FusedLinears L, const float* __restrict__ x,
                                                               const int8_t* __restrict__ xq,
                                                               const float* __restrict__ x_scale, int M, int K,
                                                               int slice, int8_t* __restrict__ xq_out,
                                                               float* __restrict__ s_out, int32_t* __restrict__ rs_out) {
    using T = MfmaFmt<F>;
    constexpr int kThreads = 64 * WAVES;
    extern __shared__ __align__(16) int8_t xs[];    // token rows of nkb BK codes + 16 bytes
    __shared__ v4i part[2][WAVES][64];
    __shared__ int rs_s[WAVES][16];
    __shared__ float redf[WAVES];

    const int m0 = (int)blockIdx.y * slice;         // this work group's token slice
    M = min(M - m0, slice);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, r = lane & 15;
    const int G = gridDim.x, bid = blockIdx.x;
    const int nkb = (K + T::BK - 1) / T::BK;
    const int stride = nkb * T::BK + 16;            // an odd multiple of 16: the rows of an operand read in other banks
    const int nb = (nkb + WAVES * U - 1) / (WAVES * U);
    const int S = ((L.total - bid + G - 1) / G) * nb;
    const uint32_t row_bytes = (uint32_t)K / T::row_div;

    // step st = batch st % nb of row group bid + (st / nb) G
    auto step_gb = [&](int st, int& g, int& b) {
        const int gi = nb == 1 ? st : st / nb;
        b = st - gi * nb;
        g = bid + gi * G;
    };
    struct Batch {
        v4u w[U];
        uint32_t sg[F == kElutC5G2 ? U : 1];
        float bw;
    };
    auto issue = [&](Batch& B, int st) {
        int g, b, li, rg;
        step_gb(st, g, b);
        locate(L, g, li, rg);
        const uint8_t* base = pick(L.packed, li);
        const uint32_t n = (uint32_t)(rg * kRowsPerGroup + r);
        const int kb0 = b * (WAVES * U) + wave * U;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // chunks past the row read its last one (their activation codes are zero, or the block is not multiplied)
            const uint32_t off = min((uint32_t)(64 * (kb0 + u) + 16 * q), row_bytes - 16u);
            B.w[u] = load_stream16(base + ((size_t)n * row_bytes + off));
            if constexpr (F == kElutC5G2)
                B.sg[u] = *reinterpret_cast<const uint32_t*>(base + (size_t)pick(L.N, li) * row_bytes +
                                                             ((size_t)n * (row_bytes / 4) + off / 4));
        }
        B.bw = *pick(L.w_scale, li);
    };

    Batch A0, A1;
    float sx = 1.0f;
    const v4i zero = {0, 0, 0, 0};
    if constexpr (QX) {
        // the row in registers (up to kXV float4 per thread, longer rows read twice), its absmax, its codes
        constexpr int kXV = 4;
        const float4* x4 = reinterpret_cast<const float4*>(x);
        const int K4 = K >> 2;
        float4 xv[kXV];
        float amax = 0.0f;
        auto amax4 = [&](const float4& v) {
            amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
        };
#pragma unroll
        for (int i = 0; i < kXV; ++i) xv[i] = x4[min(tid + i * kThreads, K4 - 1)];
        __builtin_amdgcn_s_barrier();               // every wave's row loads before any weight load
        issue(A0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kXV; ++i) amax4(xv[i]);  // a repeated element changes nothing
        for (int e = tid + kXV * kThreads; e < K4; e += kThreads) amax4(x4[e]);
        amax = wave_max_all(amax);
        if (lane == 0) redf[wave] = amax;
        __syncthreads();
        amax = redf[0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) amax = fmaxf(amax, redf[w]);
        sx = 127.0f / fmaxf(amax, 1e-5f);
        auto put = [&](const float4& v, int e) {
            const uint32_t c = quant4(v, sx);
#pragma unroll
            for (int p = 0; p < 4; ++p) xs[code_pos<F>(4 * e + p)] = (int8_t)(c >> (8 * p));
            if (bid == 0) reinterpret_cast<uint32_t*>(xq_out)[e] = c;
        };
#pragma unroll
        for (int i = 0; i < kXV; ++i)
            if (tid + i * kThreads < K4) put(xv[i], tid + i * kThreads);
        for (int e = tid + kXV * kThreads; e < K4; e += kThreads) put(x4[e], e);
        for (int k = K + 16 * tid; k < nkb * T::BK; k += 16 * kThreads) *reinterpret_cast<v4i*>(xs + k) = zero;
        if (bid == 0 && tid == 0) s_out[0] = sx;
    } else {
        // Each wave copies the codes of its own blocks, every token, in the operands' order; no other wave reads them.
        // The first eight tokens' loads of the first batch go out before any weight load, and the barrier keeps the
        // last waves' codes from queueing behind the first waves' weights.
        const int8_t* src = xq + (size_t)m0 * K;
        auto start = [&]() {
            __builtin_amdgcn_s_barrier();
            issue(A0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        if constexpr (F == kElutC3G5) {
            // lane: token lane / 4, run lane % 4 (80 codes) of a block; every load in bounds, stores where it is real
            const int m = lane >> 2;
            for (int b = 0; b < nb; ++b) {
                for (int u = 0; u < U; ++u) {
                    const int k = (b * (WAVES * U) + wave * U + u) * T::BK + 80 * (lane & 3);
                    const int8_t* p = src + (size_t)min(m, M - 1) * K + min(k, K - 80);
                    uint32_t in[20];
#pragma unroll
                    for (int i = 0; i < 5; ++i) {
                        const v4u v = *reinterpret_cast<const v4u*>(p + 16 * i);
                        in[4 * i] = v.x;
                        in[4 * i + 1] = v.y;
                        in[4 * i + 2] = v.z;
                        in[4 * i + 3] = v.w;
                    }
                    if (b == 0 && u == 0) start();
                    if (m < M && k < K) {
#pragma unroll
                        for (int d = 0; d < 5; ++d) {
                            v4u o;
#pragma unroll
                            for (int f = 0; f < 4; ++f) {
                                uint32_t word = 0u;
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    const int kk = 5 * (4 * f + e) + d;
                                    word |= ((in[kk >> 2] >> (8 * (kk & 3))) & 0xFFu) << (8 * e);
                                }
                                o[f] = word;
                            }
                            *reinterpret_cast<v4u*>(xs + m * stride + k + 16 * d) = o;
                        }
                    }
                }
            }
        } else {
            // lane: token lane / 16 of four, 16-byte chunk lane % 16 of a block; eight tokens at a time
            const int end = nkb * T::BK;
            for (int b = 0; b < nb; ++b) {
                const int kw = (b * (WAVES * U) + wave * U) * T::BK + 16 * r;
                for (int mg = 0; mg < M; mg += 8) {
                    v4i in[2][U];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int u = 0; u < U; ++u)
                            in[h][u] = *reinterpret_cast<const v4i*>(src + (size_t)min(mg + 4 * h + q, M - 1) * K +
                                                                     min(kw + u * T::BK, K - 16));
                    if (b == 0 && mg == 0) start();
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int m = mg + 4 * h + q, k = kw + u * T::BK;
                            if (m < M && k < end)
                                *reinterpret_cast<v4i*>(xs + m * stride + k) = k < K ? order_pairs(in[h][u]) : zero;
                        }
                }
            }
        }
        wave_lds_handoff();
    }
    // epilogue operands of tokens m = 4 q + v
    float xs_m[4];
    int off_m[4] = {0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < 4; ++v) xs_m[v] = QX ? sx : x_scale[m0 + min(4 * q + v, M - 1)];

    v4i acc = zero, rsum = zero;
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    const int8_t* arow = xs + (r < M ? r : 0) * stride + q * (T::BK / 4);
    int par = 0;
    // FIRST: the work group's first row group, which also sums the codes
    auto compute = [&](const Batch& B, int st, auto first) {
        constexpr bool kFirst = decltype(first)::value;
        int g, b;
        step_gb(st, g, b);
        if (b == 0) acc = zero;
        const int kb0 = b * (WAVES * U) + wave * U;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (kb0 + u < nkb) {
                const int8_t* ab = arow + (kb0 + u) * T::BK;
                if constexpr (F == kElutC3G5) {
                    uint32_t d0[5], d1[5], d2[5], d3[5];
                    c3_digits(B.w[u].x, d0);
                    c3_digits(B.w[u].y, d1);
                    c3_digits(B.w[u].z, d2);
                    c3_digits(B.w[u].w, d3);
#pragma unroll
                    for (int j = 0; j < 5; ++j) {
                        const v4i a = *reinterpret_cast<const v4i*>(ab + 16 * j);
                        acc = mfma16x16x64(a, v4i{(int)d0[j], (int)d1[j], (int)d2[j], (int)d3[j]}, acc);
                        if constexpr (kFirst) rsum = mfma16x16x64(a, ones, rsum);
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const v4i a = *reinterpret_cast<const v4i*>(ab + 16 * j);
                        const uint32_t w = word_of(B.w[u], j);
                        const v4i c = F == kElutC5G2 ? c5_codes(w, (B.sg[F == kElutC5G2 ? u : 0] >> (8 * j)) & 0xFFu)
                                                     : unpack_codes(w);
                        acc = mfma16x16x64(a, c, acc);
                        if constexpr (kFirst) rsum = mfma16x16x64(a, ones, rsum);
                    }
                }
            }
        }
        if (b != nb - 1) return;
        part[par][wave][lane] = acc;
        if constexpr (kFirst) {
            if (r == 0) {
#pragma unroll
                for (int v = 0; v < 4; ++v) rs_s[wave][4 * q + v] = rsum[v];
            }
        }
        __syncthreads();
        if (wave == 0) {
            if constexpr (kFirst) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    int t = 0;
#pragma unroll
                    for (int w2 = 0; w2 < WAVES; ++w2) t += rs_s[w2][4 * q + v];
                    off_m[v] = T::OFF * t;
                    if (QX && v == 0 && bid == 0 && tid == 0) rs_out[0] = t;
                }
            }
            if (4 * q < M) {
                v4i tot = part[par][0][lane];
#pragma unroll 4
                for (int w2 = 1; w2 < WAVES; ++w2) tot += part[par][w2][lane];
                int li, rg;
                locate(L, g, li, rg);
                const int N = pick(L.N, li);
                const int n = rg * kRowsPerGroup + r;
                float* y = pick(L.y, li);
                int32_t* acc_out = pick(L.acc, li);
                // D element v of lane l is row 4 (l / 16) + v (token), column l % 16 (weight row)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int m = 4 * q + v;
                    if (m < M) {
                        const int val = tot[v] - off_m[v];
                        y[(size_t)(m0 + m) * N + n] = (float)val * (B.bw / xs_m[v]);
                        if (acc_out) acc_out[(size_t)(m0 + m) * N + n] = val;
                    }
                }
            }
        }
        par ^= 1;
    };

    const std::true_type kFirstGroup{};
    const std::false_type kLaterGroup{};
    if (S == 1) {
        if constexpr (QX) __syncthreads();          // the codes are in LDS
        compute(A0, 0, kFirstGroup);
        return;
    }
    issue(A1, 1);
    if constexpr (QX) __syncthreads();
    // steps st and st + 1 are in flight; each set is refilled right after it is multiplied (past the last step: the
    // last one again, never multiplied)
    auto step = [&](Batch& B, int st) {
        if (st < nb) compute(B, st, kFirstGroup);
        else compute(B, st, kLaterGroup);
        issue(B, min(st + 2, S - 1));
    };
    int st = 0;
    for (; st + 1 < S; st += 2) {
        step(A0, st);
        step(A1, st + 1);
    }
    if (st < S) step(A0, st);
}

constexpr size_t kElutLds = 120 * 1024;             // dynamic LDS of a launch (16 waves hold 34 KiB beside it)

template <int F, int WAVES, int U>
hipError_t launch_cfg(const FusedLinears& L, const float* x, const int8_t* xq, const float* x_scale, int M, int K,
                      int slice, int8_t* xq_out, float* s_out, int32_t* rs_out, hipStream_t stream) {
    using T = MfmaFmt<F>;
    const int nkb = (K + T::BK - 1) / T::BK;
    const int per = M < slice ? M : slice;
    const size_t lds = (size_t)per * (size_t)(nkb * T::BK + 16);
    const void* kern = x ? reinterpret_cast<const void*>(elut_kernel<F, WAVES, U, true>)
                         : reinterpret_cast<const void*>(elut_kernel<F, WAVES, U, false>);
    const int occ = resident_groups(kern, 64 * WAVES, lds);
    constexpr int kMaxSlices = 4096;                // of one launch (grid y)
    for (int s0 = 0; s0 * (int64_t)per < M; s0 += kMaxSlices) {
        const int m0 = s0 * per;
        const int mc = (int64_t)(M - m0) < (int64_t)kMaxSlices * per ? M - m0 : kMaxSlices * per;
        const int slices = (mc + per - 1) / per;
        // as many work groups as are resident at once, balanced over the row groups; with token slices the columns
        // are a multiple of 8, so that the slices of a row group run on one XCD and share its weight bytes in L2
        int64_t max_g = (int64_t)device_cus() * occ;
        if (slices > 1) max_g = max_g / slices / kNumXcd * kNumXcd;
        if (max_g < kNumXcd) max_g = kNumXcd;
        const int64_t rounds = (L.total + max_g - 1) / max_g;
        int64_t gx = (L.total + rounds - 1) / rounds;
        if (slices > 1 && gx > kNumXcd) gx = gx / kNumXcd * kNumXcd;
        FusedLinears Ls = L;
        for (int i = 0; i < L.count; ++i) {
            Ls.y[i] = L.y[i] + (size_t)m0 * L.N[i];
            Ls.acc[i] = L.acc[i] ? L.acc[i] + (size_t)m0 * L.N[i] : nullptr;
        }
        const dim3 grid((unsigned)gx, (unsigned)slices), block(64 * WAVES);
        if (x)
            hipLaunchKernelGGL((elut_kernel<F, WAVES, U, true>), grid, block, lds, stream, Ls, x, xq, x_scale, mc, K,
                               per, xq_out, s_out, rs_out);
        else
            hipLaunchKernelGGL((elut_kernel<F, WAVES, U, false>), grid, block, lds, stream, Ls, x,
                               xq + (size_t)m0 * K, x_scale + m0, mc, K, per, xq_out, s_out, rs_out);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int F>
hipError_t launch_fmt(const FusedLinears& L, const float* x, const int8_t* xq, const float* x_scale, int M, int K,
                      int8_t* xq_out, float* s_out, int32_t* rs_out, hipStream_t s) {
    using T = MfmaFmt<F>;
    const int nkb = (K + T::BK - 1) / T::BK;
    const int64_t fit = (int64_t)(kElutLds / (size_t)(nkb * T::BK + 16));
    const int slice = fit < 16 ? (int)fit : 16;
    // 4-wave groups where a row fits one batch of theirs and there are row groups for half the CUs: several groups per
    // CU do not wait on one another's barriers; and where a row has no work for a fifth wave (1024 rows of K = 960 at
    // one token: C4G2 5.6 us with 16 waves, 4.6 with 4; C3G5 5.9 and 4.8).  Otherwise 16 waves, the batches of a row group
    // balanced (up to two blocks per wave: with more the kernel spills).  Rows of K > 122000 leave LDS only for the partial sums of 8 waves.
    if (nkb <= 4 || (nkb <= 16 && L.total > device_cus() / 2)) {
        const int u = (nkb + 3) / 4;
        if (u <= 1) return launch_cfg<F, 4, 1>(L, x, xq, x_scale, M, K, slice, xq_out, s_out, rs_out, s);
        if (u <= 2) return launch_cfg<F, 4, 2>(L, x, xq, x_scale, M, K, slice, xq_out, s_out, rs_out, s);
        if (u <= 3) return launch_cfg<F, 4, 3>(L, x, xq, x_scale, M, K, slice, xq_out, s_out, rs_out, s);
        return launch_cfg<F, 4, 4>(L, x, xq, x_scale, M, K, slice, xq_out, s_out, rs_out, s);
    }
    if (fit < 1) return launch_cfg<F, 8, 2>(L, x, xq, x_scale, M, K, 1, xq_out, s_out, rs_out, s);
    const int nb = (nkb + 31) / 32, u = (nkb + 16 * nb - 1) / (16 * nb);
    if (u <= 1) return launch_cfg<F, 16, 1>(L, x, xq, x_scale, M, K, slice, xq_out, s_out, rs_out, s);
    return launch_cfg<F, 16, 2>(L, x, xq, x_scale, M, K, slice, xq_out, s_out, rs_out, s);
}

// Packing: one thread per packed word of a row (c4g2 and c5g2: 8 groups, plus their sign byte; c3g5: 4 groups).
// Values outside the set are clamped into it.
template <int F>
__global__ __launch_bounds__(256) void pack_elut_words(const int8_t* __restrict__ Wq, int N, int K,
                                                       uint8_t* __restrict__ packed) {
    using T = ElutFmt<F>;
    const size_t wpr = (size_t)K / (T::G * T::GW);       // words per row
    const size_t d = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (d >= (size_t)N * wpr) return;
    const size_t n = d / wpr;
    const int w = (int)(d - n * wpr);
    const int8_t* src = Wq + n * (size_t)K + (size_t)w * T::G * T::GW;
    const int lo = -(T::C / 2), hi = T::C - 1 - T::C / 2;
    uint32_t word = 0u, sign = 0u;
    for (int i = 0; i < T::GW; ++i) {
        int v = 0;
        for (int j = 0; j < T::G; ++j) {
            const int wj = min(max((int)src[i * T::G + j], lo), hi);
            v = v * T::C + (T::kMirror ? wj : wj - lo);
        }
        const uint32_t idx = (uint32_t)(v < 0 ? -v : v);
        const uint32_t sg = v < 0 ? 1u : 0u;
        if constexpr (F == kElutC3G5) word |= (idx | (sg << 7)) << (8 * i);
        else word |= idx << (4 * i);
        sign |= sg << i;
    }
    const size_t row_bytes = T::GW == 8 ? (size_t)K / 4 : (size_t)K / 5;
    *reinterpret_cast<uint32_t*>(packed + n * row_bytes + 4 * (size_t)w) = word;
    if constexpr (F == kElutC5G2) packed[(size_t)N * K / 4 + n * (K / 16) + w] = (uint8_t)sign;
}

template <int F>
hipError_t launch_pack_fmt(const int8_t* Wq, int N, int K, void* packed, hipStream_t stream) {
    using T = ElutFmt<F>;
    const size_t words = (size_t)N * K / (T::G * T::GW);
    hipLaunchKernelGGL((pack_elut_words<F>), dim3((unsigned)((words + 255) / 256)), dim3(256), 0, stream, Wq, N, K,
                       static_cast<uint8_t*>(packed));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_elut(int fmt, const FusedLinears& L, const float* x, const int8_t* xq, const float* x_scale, int M,
                            int K, int8_t* xq_out, float* s_out, int32_t* rs_out, hipStream_t stream) {
    switch (fmt) {
        case kElutC4G2: return launch_fmt<kElutC4G2>(L, x, xq, x_scale, M, K, xq_out, s_out, rs_out, stream);
        case kElutC5G2: return launch_fmt<kElutC5G2>(L, x, xq, x_scale, M, K, xq_out, s_out, rs_out, stream);
        default: return launch_fmt<kElutC3G5>(L, x, xq, x_scale, M, K, xq_out, s_out, rs_out, stream);
    }
}

hipError_t launch_pack_elut(int fmt, const int8_t* Wq, int N, int K, void* packed, hipStream_t stream) {
    switch (fmt) {
        case kElutC4G2: return launch_pack_fmt<kElutC4G2>(Wq, N, K, packed, stream);
        case kElutC5G2: return launch_pack_fmt<kElutC5G2>(Wq, N, K, packed, stream);
        default: return launch_pack_fmt<kElutC3G5>(Wq, N, K, packed, stream);
    }
}

}  // namespace bitnet
