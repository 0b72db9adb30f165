// The lossy layouts TL2_0 and TL1_0 (Sec. 3.2.1) for several tokens (slices of up to 16), as one-hot contractions on int8
// MFMA.
//
// Every table entry is an int8 (divided by the block's power of two and rounded), so looking an entry up is the product
// of the token's 16-entry table with a row that holds the Eq. 5 sign at the code's index and zeros elsewhere.  In
// v_mfma_i32_16x16x64_i8 (A row = token, B column = weight row) lane (r, q) gives 16 of the 64 k: as A the table of one
// group of token r, as B the one-hot of row r's code for that group.  So one MFMA looks four groups up for 16 rows and
// 16 tokens, whatever the tables hold; the integers are those of the rule.
//
// Work split.  A work group owns RG 16-row groups; its waves take the k blocks (384 k of TL2, 256 k of TL1, the TL2
// tail's units as one more block) in turn.  A wave builds the tables of a block straight into its registers, as MFMA
// operands (lane (r, q): token r, the groups that quarter q holds in the packed layout: 32 tables of 4 registers), and
// then runs the RG row groups over them, so building is shared by 16 RG rows and no table goes through LDS.  With up to
// eight (four) tokens two (four) lanes of a quarter build a share of one token's tables each and exchange them.  A
// block's sums are scaled back by its shift and added up in registers; the waves meet in LDS at the end.
//
// What bounds it: VALU, about ten operations per group and lane to make the one-hot row (a 64-bit shift and a select),
// and 26 to build a table.  The 8B-class layer set at 8 tokens: TL2_0 229 -> 90 us, TL1_0 243 -> 115 us (a table lookup
// per group, row and token before, every 16-row work group building the tables of its own; TL2_0 gate and up 129 -> 31 us,
// down 75 -> 24 us).
#include "bitnet_internal.hpp"

namespace bitnet {
namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t u32_of(h2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ h2 h2_of(uint32_t v) { return __builtin_bit_cast(h2, v); }

// The smallest s >= 0 with mx <= 127 * 2^s, for mx <= 384 (the largest |entry|).
__device__ __forceinline__ int shift_of(int mx) { return (mx > 127 ? 1 : 0) + (mx > 254 ? 1 : 0); }

// Tables are made in fp16 pairs: codes and their sums are integers of at most 384, exact.  An entry e becomes
// fp16(e 2^-s + 1536), one rounding: fp16 has units of 1 from 1024 to 2048, so that rounds e 2^-s half to even, and the
// low byte of 0x6600 + q is q in two's complement.
struct Quantiser {
    h2 scale;
    __device__ __forceinline__ explicit Quantiser(int s) {
        const uint32_t b = (uint32_t)(15 - s) << 10;           // 2^-s
        scale = h2_of(b | (b << 16));
    }
    __device__ __forceinline__ uint32_t operator()(h2 e) const {
        const h2 magic = {(_Float16)1536.0f, (_Float16)1536.0f};
        return u32_of(__builtin_elementwise_fma(e, scale, magic));
    }
};
// The low bytes of the four halves of two words.
__device__ __forceinline__ int low_bytes(uint32_t a, uint32_t b) { return (int)__builtin_amdgcn_perm(b, a, 0x06040200u); }

// Bytes of `u` (codes + 128) as an fp16 pair of codes: a byte u under 0x64 is 1024 + u; 0x6480 (selector bytes 5, 4) is 0.
template <uint32_t SEL>
__device__ __forceinline__ h2 codes_of(uint32_t u) {
    const h2 off = {(_Float16)1152.0f, (_Float16)1152.0f};
    return h2_of(__builtin_amdgcn_perm(0x00006480u, u, SEL)) - off;
}

// The 14 mirror-consolidated sums of a triple (9 d0 + 3 d1 + d2 = index, leading digit >= 0), quantised, as bytes.
// u: its three codes + 128 in the low bytes.
__device__ __forceinline__ v4i triple_bytes(uint32_t u, const Quantiser& Q) {
    const h2 xy = codes_of<0x05010500u>(u), z0 = codes_of<0x05040502u>(u);         // (a0, a1), (a2, 0)
    const h2 oz = h2_of(u32_of(z0) << 16), zm = {z0.x, -z0.x};                     // (0, a2), (a2, -a2)
    const h2 xx = {xy.x, xy.x}, yy = {xy.y, xy.y}, my = {-xy.y, xy.y};
    const h2 pt = xx + my;                                                         // a0 - a1, a0 + a1
    const h2 pp = {pt.x, pt.x}, tt = {pt.y, pt.y}, yp = {xy.y, pt.x}, xt = {xy.x, pt.y};
    return v4i{low_bytes(Q(oz), Q(yy - z0)), low_bytes(Q(yp + zm), Q(pp + oz)), low_bytes(Q(xx - z0), Q(xt + zm)),
               low_bytes(Q(tt + oz), 0u)};
}

// The 9 sums (i / 3 - 1) b0 + (i % 3 - 1) b1 of a pair, quantised, as bytes.  u: its codes + 128 in the low bytes.
__device__ __forceinline__ v4i pair_bytes(uint32_t u, const Quantiser& Q) {
    const h2 xy = codes_of<0x05010500u>(u), y0 = codes_of<0x05040501u>(u);         // (b0, b1), (b1, 0)
    const h2 xx = {xy.x, xy.x}, my = {-xy.y, xy.y};
    const h2 pt = xx + my;                                                         // b0 - b1, b0 + b1
    const h2 a = {-pt.y, -xy.x}, b = {-pt.x, -xy.y}, c = h2_of(u32_of(y0) << 16), d = {pt.x, xy.x}, e = {pt.y, pt.y};
    return v4i{low_bytes(Q(a), Q(b)), low_bytes(Q(c), Q(d)), (int)(Q(e) & 0xFFu), 0};
}

// 16 bytes with `v` (one byte) at byte idx: sh8 holds 8 (idx % 8) in its low 6 bits, hi is all ones where idx >= 8.
__device__ __forceinline__ v4i one_hot(uint32_t v, uint32_t sh8, uint32_t hi) {
    const unsigned long long b = (unsigned long long)v << (sh8 & 63u);
    const uint32_t lo32 = (uint32_t)b, hi32 = (uint32_t)(b >> 32);
    const uint32_t c = lo32 & hi, d = hi32 & hi;
    return v4i{(int)(lo32 ^ c), (int)(hi32 ^ d), (int)c, (int)d};
}
// All ones if the bit is set.  (In C the compiler turns the sign selection that uses it into an and, a compare and a
// select, one operation more.)
__device__ __forceinline__ uint32_t ones_if(uint32_t w, int bit) {
    uint32_t m;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(w), "s"(bit));
    return m;
}

// The one-hot row of the nibble at bit 4 nib of w; neg: all ones for a negative group.
__device__ __forceinline__ v4i code_row(uint32_t w, uint32_t even, uint32_t odd, int nib, uint32_t neg) {
    // 8 (index % 8) from the nibbles' low bits, every other nibble cleared so that the bits below are zero
    const uint32_t src = (nib & 1) ? odd : even;
    const int at = 8 * (nib >> 1);
    return one_hot((neg & 0xFEu) | 1u, at ? src >> (at - 3) : src << 3, ones_if(w, 4 * nib + 3));
}

// The table of the lane BY places up in the row of 16 (row_ror moves a value that many places up: 16 - BY).
template <int BY>
__device__ __forceinline__ int from_above(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x120 + 16 - BY, 0xF, 0xF, true);
}
template <int BY>
__device__ __forceinline__ v4i from_above(v4i t) {
    return v4i{from_above<BY>(t.x), from_above<BY>(t.y), from_above<BY>(t.z), from_above<BY>(t.w)};
}
// Tables 0 .. own - 1 are this lane's; the rest come from the lanes of the same token above it, own each (the lowest of
// a token's lanes, an output row, ends with all of them in order; the rows of the others are not stored).
template <int DUP, int N>
__device__ __forceinline__ void share_tables(v4i (&t)[N]) {
    constexpr int own = N / DUP;
    if constexpr (DUP >= 2) {
#pragma unroll
        for (int i = 0; i < own; ++i) t[own + i] = from_above<16 / DUP>(t[i]);
    }
    if constexpr (DUP >= 4) {
#pragma unroll
        for (int i = 0; i < own; ++i) {
            t[2 * own + i] = from_above<8>(t[i]);
            t[3 * own + i] = from_above<12>(t[i]);
        }
    }
}
// A maximum over the lanes that hold parts of one token: the four quarters, and the DUP lanes of the token in each.
template <int DUP>
__device__ __forceinline__ int token_max(int v) {
    if (DUP >= 2) v = max(v, dpp_row_step(v, 3));
    if (DUP >= 4) v = max(v, dpp_row_step(v, 2));
    v = max(v, __shfl_xor(v, 16, 64));
    return max(v, __shfl_xor(v, 32, 64));
}

// N words from src (4-byte aligned, to 16 bytes where N is a multiple of 4).
template <int N, int A>
__device__ __forceinline__ void load_words(uint32_t (&c)[A], const int8_t* src) {
    if constexpr (N % 4 == 0) {
#pragma unroll
        for (int i = 0; i < N / 4; ++i) {
            const v4u v = *reinterpret_cast<const v4u*>(src + 16 * i);
            c[4 * i] = v.x;
            c[4 * i + 1] = v.y;
            c[4 * i + 2] = v.z;
            c[4 * i + 3] = v.w;
        }
    } else if constexpr (N % 2 == 0) {
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            const uint2 v = *reinterpret_cast<const uint2*>(src + 8 * i);
            c[2 * i] = v.x;
            c[2 * i + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) c[i] = *reinterpret_cast<const uint32_t*>(src + 4 * i);
    }
}

// TL1: the packed words are TL1's (TL1_0), else TL2's (TL2_0).  At most 16 / DUP tokens (DUP 1, 2 or 4): the lanes r,
// r + 16 / DUP, ... of a quarter hold the same token and build a share of its tables each.
template <bool TL1, int DUP, int WAVES, int RG>
__global__ __attribute__((amdgpu_waves_per_eu(TL1 ? (RG <= 4 ? 4 : 2) : RG == 1 && DUP > 1 ? 4 : 2, 4)))
__launch_bounds__(64 * WAVES) void lossy_kernel(
    FusedLinears L, const int8_t* __restrict__ xq, const float* __restrict__ x_scale, int M, int K, int slice) {
    __shared__ v4i red[WAVES][RG][64];

    const int m0 = (int)blockIdx.y * slice;
    M = min(M - m0, slice);
    xq += (size_t)m0 * K;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, r = lane & 15;
    const int tok = min(r % (16 / DUP), M - 1), share = r / (16 / DUP);
    const int8_t* xrow = xq + (size_t)tok * K;

    const int three = TL1 ? 0 : (K / kTl2BlockK) * kTl2BlockK;
    const int nblk = three / kTl2BlockK;
    const int units = (K - three) / kSubK;                    // 64-k units of pairs: the TL2 tail, or all of TL1
    const int nwork = TL1 ? (units + 3) / 4 : nblk + (units ? 1 : 0);

    // this work group's row groups (past the last: the last, never stored)
    const uint8_t* base[RG];
    int rgi[RG], rli[RG];
#pragma unroll
    for (int i = 0; i < RG; ++i) {
        const int g = min((int)blockIdx.x * RG + i, L.total - 1);
        locate(L, g, rli[i], rgi[i]);
        base[i] = pick(L.packed, rli[i]);
    }

    const v4i zero = {0, 0, 0, 0};
    v4i acc[RG];
#pragma unroll
    for (int i = 0; i < RG; ++i) acc[i] = zero;

    // The shifts of the output rows' tokens 4 q + v, from lane v's own token shift.
    auto row_shifts = [&](int sh, int (&o)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = __shfl(sh, 4 * q + v, 64);
    };
    auto add_scaled = [&](v4i& a, v4i d, const int (&o)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) a[v] += d[v] << o[v];
    };

    // One 64-k unit of pairs: lane (r, q) holds pairs 8 q .. 8 q + 7 (codes k .. k + 15) of its token and its row's word
    // of every row group; pair i is nibble i (TL2 tail) or nibble 2 (i % 4) + i / 4 (TL1).
    auto pair_unit = [&](int k0, const uint32_t (&word)[RG]) {
        constexpr int kOwn = 8 / DUP;                         // pairs this lane builds
        uint32_t c[kOwn / 2];
        load_words<kOwn / 2>(c, xrow + k0 + 16 * q + 2 * kOwn * share);
        int mx = 0;
#pragma unroll
        for (int i = 0; i < kOwn / 2; ++i) c[i] ^= 0x80808080u;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            const uint32_t p = (i & 1) ? c[i >> 1] >> 16 : c[i >> 1] & 0xFFFFu;
            mx = max(mx, (int)__builtin_amdgcn_sad_u8(p, 0x8080u, 0u));
        }
        const int sh = shift_of(token_max<DUP>(mx));
        const Quantiser Q(sh);
        v4i t[8];
#pragma unroll
        for (int i = 0; i < kOwn; ++i) t[i] = pair_bytes((i & 1) ? c[i >> 1] >> 16 : c[i >> 1], Q);
        share_tables<DUP>(t);
        int o[4];
        row_shifts(sh, o);
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            const uint32_t w = word[g], ev = w & 0x07070707u, od = (w >> 4) & 0x07070707u;
            v4i d0 = zero, d1 = zero;
#pragma unroll
            for (int i = 0; i < 8; i += 2) {
                const int n0 = TL1 ? 2 * (i & 3) + (i >> 2) : i, n1 = TL1 ? 2 * ((i + 1) & 3) + ((i + 1) >> 2) : i + 1;
                d0 = mfma16x16x64(t[i], code_row(w, ev, od, n0, 0u), d0);
                d1 = mfma16x16x64(t[i + 1], code_row(w, ev, od, n1, 0u), d1);
            }
            add_scaled(acc[g], d0 + d1, o);
        }
    };

    for (int blk = wave; blk < nwork; blk += WAVES) {
        if constexpr (TL1) {
            // up to four units of a 256-k block; lane's words at 4 T lane (word j of unit j; past T: a real word)
            const int T = min(4, units - 4 * blk);
            uint32_t word[4][RG];
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    word[j][g] = *reinterpret_cast<const uint32_t*>(base[g] + (size_t)rgi[g] * 4 * K + (size_t)blk * 1024 +
                                                                    4 * (T * lane + min(j, T - 1)));
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j < T) pair_unit(blk * kI2sBlockK + kSubK * j, word[j]);
        } else if (blk == nblk) {
            for (int u = 0; u < units; ++u) {
                uint32_t word[RG];
#pragma unroll
                for (int g = 0; g < RG; ++g) {
                    const size_t N = (size_t)pick(L.N, rli[g]);
                    const uint8_t* tail = base[g] + N * (three / 6) + N * (three / 24);
                    word[g] = *reinterpret_cast<const uint32_t*>(tail + (((size_t)rgi[g] * 64 + lane) * units + u) * 4);
                }
                pair_unit(three + kSubK * u, word);
            }
        } else {
            v4u iw[RG];
            uint32_t sw[RG];
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                const size_t tile = (size_t)rgi[g] * nblk + blk;
                iw[g] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(base[g] + tile * 1024 + 16 * lane));
                sw[g] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(
                    base[g] + (size_t)pick(L.N, rli[g]) * (three / 6) + tile * 256 + 4 * lane));
            }
            // the block's shift: quarter q's 96 codes of the token, three a triple, shared by its DUP lanes
            constexpr int kOwn = 32 / DUP;
            int mx = 0;
            {
                uint32_t c[3 * kOwn / 4 + 1];
                load_words<3 * kOwn / 4>(c, xrow + blk * kTl2BlockK + 96 * q + 3 * kOwn * share);
                c[3 * kOwn / 4] = 0u;
#pragma unroll
                for (int i = 0; i < 3 * kOwn / 4; ++i) c[i] ^= 0x80808080u;
#pragma unroll
                for (int i = 0; i < kOwn; ++i) {
                    const uint32_t tr = __builtin_amdgcn_alignbyte(c[(3 * i >> 2) + 1], c[3 * i >> 2], (3 * i) & 3) & 0xFFFFFFu;
                    mx = max(mx, (int)__builtin_amdgcn_sad_u8(tr, 0x808080u, 0u));
                }
            }
            const int sh = shift_of(token_max<DUP>(mx));
            const Quantiser Q(sh);
            int o[4];
            row_shifts(sh, o);
            // two passes of 16 of the quarter's triples (all 32 tables at once leave too few registers)
#pragma unroll 1
            for (int p = 0; p < 2; ++p) {
                constexpr int kPass = 16 / DUP;               // triples this lane builds
                uint32_t c[3 * kPass / 4 + 1];
                load_words<3 * kPass / 4>(c, xrow + blk * kTl2BlockK + 96 * q + 48 * p + 3 * kPass * share);
                c[3 * kPass / 4] = 0u;
                v4i t[16];
#pragma unroll
                for (int i = 0; i < 3 * kPass / 4; ++i) c[i] ^= 0x80808080u;
#pragma unroll
                for (int i = 0; i < kPass; ++i)
                    t[i] = triple_bytes(__builtin_amdgcn_alignbyte(c[(3 * i >> 2) + 1], c[3 * i >> 2], (3 * i) & 3), Q);
                share_tables<DUP>(t);
#pragma unroll
                for (int g = 0; g < RG; ++g) {
                    const uint32_t wl = p ? iw[g].z : iw[g].x, wh = p ? iw[g].w : iw[g].y, sg = sw[g] >> (16 * p);
                    v4i d0 = zero, d1 = zero;
#pragma unroll
                    for (int i = 0; i < 16; i += 2) {
                        const uint32_t w = i < 8 ? wl : wh, ev = w & 0x07070707u, od = (w >> 4) & 0x07070707u;
                        d0 = mfma16x16x64(t[i], code_row(w, ev, od, i & 7, ones_if(sg, i)), d0);
                        d1 = mfma16x16x64(t[i + 1], code_row(w, ev, od, (i & 7) + 1, ones_if(sg, i + 1)), d1);
                    }
                    add_scaled(acc[g], d0 + d1, o);
                }
            }
        }
    }

#pragma unroll
    for (int g = 0; g < RG; ++g) red[wave][g][lane] = acc[g];
    __syncthreads();
    for (int g = wave; g < RG; g += WAVES) {
        const int gg = (int)blockIdx.x * RG + g;
        if (gg >= L.total || 4 * q >= M) continue;
        v4i tot = red[0][g][lane];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) tot += red[w][g][lane];
        int li, rg;
        locate(L, gg, li, rg);
        const int N = pick(L.N, li), n = rg * kRowsPerGroup + r;
        const float beta = *pick(L.w_scale, li);
        float* y = pick(L.y, li);
        int32_t* acc_out = pick(L.acc, li);
        // D element v of lane l is row 4 (l / 16) + v (token), column l % 16 (weight row)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int m = 4 * q + v;
            if (m < M) {
                y[(size_t)(m0 + m) * N + n] = (float)tot[v] * (beta / x_scale[m0 + m]);
                if (acc_out) acc_out[(size_t)(m0 + m) * N + n] = tot[v];
            }
        }
    }
}

constexpr int kMaxSlices = 4096;                             // token slices of one launch (grid y)

template <bool TL1, int DUP, int WAVES, int RG>
void launch_cfg(const FusedLinears& L, const int8_t* xq, const float* x_scale, int M, int K, int slice,
                hipStream_t stream) {
    const dim3 grid((unsigned)((L.total + RG - 1) / RG), (unsigned)((M + slice - 1) / slice)), block(64 * WAVES);
    hipLaunchKernelGGL((lossy_kernel<TL1, DUP, WAVES, RG>), grid, block, 0, stream, L, xq, x_scale, M, K, slice);
}

// Few row groups: 16 waves share one (the block loop is the longest chain), then 8 in two groups per CU.  Else 4-wave
// groups, two per CU (TL1, which has 8 tables at a time: four), with as few row groups each as keep the launch within one
// round, so that the tables are built as seldom as the grid allows.  (Nine tokens and more keep all of their tables in one lane each: 8 waves and 4
// row groups are what their registers allow.)
template <bool TL1, int DUP>
void launch_rg(const FusedLinears& L, const int8_t* xq, const float* x_scale, int M, int K, int slice, hipStream_t s) {
    constexpr int kOne = DUP > 1 ? 16 : 8, kMost = DUP > 1 ? 8 : 4, kPer = TL1 ? 4 : 2;
    const int64_t cus = device_cus(), work = (int64_t)L.total * ((M + slice - 1) / slice);
    if (work <= cus) launch_cfg<TL1, DUP, kOne, 1>(L, xq, x_scale, M, K, slice, s);
    else if (work <= 2 * cus) launch_cfg<TL1, DUP, 8, 1>(L, xq, x_scale, M, K, slice, s);
    else if (work <= kPer * 2 * cus) launch_cfg<TL1, DUP, 4, 2>(L, xq, x_scale, M, K, slice, s);
    else if (work <= kPer * 4 * cus) launch_cfg<TL1, DUP, 4, 4>(L, xq, x_scale, M, K, slice, s);
    else launch_cfg<TL1, DUP, 4, kMost>(L, xq, x_scale, M, K, slice, s);
}

}  // namespace

hipError_t launch_lossy(bool tl1, const FusedLinears& L, const int8_t* xq, const float* x_scale, int64_t M, int K,
                        hipStream_t stream) {
    const int slice = M <= 4 ? 4 : M <= 8 ? 8 : 16;
    for (int64_t m0 = 0; m0 < M; m0 += (int64_t)kMaxSlices * slice) {
        const int mc = (int)(M - m0 < (int64_t)kMaxSlices * slice ? M - m0 : (int64_t)kMaxSlices * slice);
        FusedLinears Ls = L;
        for (int i = 0; i < L.count; ++i) {
            Ls.y[i] = L.y[i] + m0 * L.N[i];
            Ls.acc[i] = L.acc[i] ? L.acc[i] + m0 * L.N[i] : nullptr;
        }
        const int8_t* xs = xq + m0 * K;
        const float* sc = x_scale + m0;
        if (tl1) {
            if (slice == 4) launch_rg<true, 4>(Ls, xs, sc, mc, K, slice, stream);
            else if (slice == 8) launch_rg<true, 2>(Ls, xs, sc, mc, K, slice, stream);
            else launch_rg<true, 1>(Ls, xs, sc, mc, K, slice, stream);
        } else {
            if (slice == 4) launch_rg<false, 4>(Ls, xs, sc, mc, K, slice, stream);
            else if (slice == 8) launch_rg<false, 2>(Ls, xs, sc, mc, K, slice, stream);
            else launch_rg<false, 1>(Ls, xs, sc, mc, K, slice, stream);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace bitnet
