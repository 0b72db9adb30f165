// Small batches (17 tokens up to the prefill GEMM's range) for the I2_S and TL1 layouts: ternary x int8 accumulation (Eq. 1) on
// v_mfma_i32_32x32x32_i8 with the dequantisation epilogue fused.
//
// Between decode (weight bytes) and prefill (matrix rate) a launch is bound by the stream of operands into the CUs:
// the packed weights once from HBM, the int8 codes again from L2 for every work group.  So a weight word is unpacked
// once for 32 tokens (the decode GEMV in slices of up to 16: twice or more), and an activation operand feeds up to 64
// weight rows.  64 tokens a work group measured slower (half as many groups, with more to start and to end each: 14.5
// against 8.0 us for 4096 -> 4096 rows at 64 tokens).
//
// A work group owns 32 NT weight rows x 32 tokens and the whole of K; its waves take every WAVES-th 256-k block and
// reduce through LDS once at the end, so nothing is synchronised inside the stream.  Per block a wave
//   * loads the rows' packed words straight into registers: lane (j, h) of the MFMA's B operand needs, for its row j
//     and the 32-k step s = 2 w + p, word w of the layout's lane chunk 2 p + h, so two 16-byte loads per 32 rows hold
//     the words of all eight steps;
//   * copies the tokens' 256-byte runs through LDS of its own (whole rows in, rows padded to 272 bytes, so an operand
//     read of 32 rows hits every bank once).  Operands loaded from global memory as the MFMA wants them would touch 32
//     lines per instruction, twice the cache's cycles of whole runs.
// The next block's loads are in flight while the current one multiplies.
#include "bitnet_internal.hpp"

#include <algorithm>
#include <type_traits>

namespace bitnet {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kTok = 32;                   // tokens per work group
constexpr int kARow = kI2sBlockK + 16;     // padded LDS row of one token's block

struct SmallLinears {
    FusedLinears L;
    int tile_start[kMaxFused];             // first tile of each weight; INT_MAX past the last
    int tiles;
};

template <int NT, int WAVES, int FMT>
__global__ __attribute__((amdgpu_waves_per_eu(NT == 1 ? 4 : 2, NT == 1 ? 4 : 2)))
__launch_bounds__(64 * WAVES) void smallbatch_kernel(SmallLinears P, const int8_t* __restrict__ xq,
                                                     const float* __restrict__ x_scale,
                                                     const int32_t* __restrict__ x_rowsum, int M, int K, int slices) {
    constexpr int kWaveBytes = 32 * kARow;
    static_assert(NT * 16 * 64 * 4 <= kWaveBytes, "a wave's sums fit its staging rows");
    __shared__ __align__(16) int8_t smem[WAVES * kWaveBytes];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j32 = lane & 31, h = lane >> 5;
    // the token slices of one tile are neighbours on one XCD: its L2 serves their weight bytes after the first
    const int id = xcd_logical_id(blockIdx.x, gridDim.x);
    const int tile = id / slices, m0 = (id - tile * slices) * kTok;
    int li = 0, t0 = 0;
#pragma unroll
    for (int i = 1; i < kMaxFused; ++i) {
        const int st = P.tile_start[i];
        li = tile >= st ? i : li;
        t0 = tile >= st ? st : t0;
    }
    const int N = pick(P.L.N, li);
    const int n0 = (tile - t0) * (32 * NT);
    const uint8_t* __restrict__ packed = pick(P.L.packed, li);
    const int nkb = (K + kI2sBlockK - 1) / kI2sBlockK, nfull = K / kI2sBlockK;
    const int Tl = nkb > nfull ? (K - nfull * kI2sBlockK) / kSubK : 4;      // 64-k sub-tiles of the last block

    // Weights: chunk p of lane (j, h) is layout lane chunk 16 (2 p + h) + j % 16 of row group j / 16.  The short last
    // block gives a chunk 4 Tl bytes; it is read through a 16-byte window moved back to end inside the block.  Row
    // groups past N repeat the last one (never stored).
    uint32_t w_rg[NT];
#pragma unroll
    for (int ni = 0; ni < NT; ++ni)
        w_rg[ni] = (uint32_t)min(n0 / kRowsPerGroup + 2 * ni + (j32 >> 4), N / kRowsPerGroup - 1) * (4u * (uint32_t)K);
    const int chunk0 = 16 * h + (lane & 15);
    uint32_t off_tail[2];
    int sh_tail[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int want = 4 * Tl * (chunk0 + 32 * p);
        off_tail[p] = (uint32_t)min(want, 256 * Tl - 16);
        sh_tail[p] = (want - (int)off_tail[p]) >> 2;
    }
    v4u w[2][NT];
    v4i a[8];
    auto load = [&](int kb) {
        const int c16 = lane & 15;
        // columns past K read a real column (they meet zero codes), rows past M a real row (never stored)
        const uint32_t col = min((uint32_t)(kb * kI2sBlockK + 16 * c16), (uint32_t)K - 16u);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t row = (uint32_t)min(m0 + 4 * i + (lane >> 4), M - 1);
            a[i] = *reinterpret_cast<const v4i*>(xq + (row * (uint32_t)K + col));
        }
        const uint8_t* pk = packed + (size_t)kb * 1024;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const uint32_t off = kb < nfull ? 16u * (uint32_t)(chunk0 + 32 * p) : off_tail[p];
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) w[p][ni] = load_stream16(pk + w_rg[ni] + off);
        }
    };

    int8_t* st = smem + wave * kWaveBytes;
    const int8_t* a_src = st + j32 * kARow + 16 * h;
    int8_t* a_dst = st + (lane >> 4) * kARow + 16 * (lane & 15);
    v16i acc[NT];
#pragma unroll
    for (int ni = 0; ni < NT; ++ni) acc[ni] = v16i{};

    int kb = wave;
    if (kb < nkb) load(kb);
    // the epilogue's operands, so that it waits for no load: record f = tid + 64 WAVES i (see below)
    constexpr int kRecords = NT * 4 * 64, kPer = (kRecords + 64 * WAVES - 1) / (64 * WAVES);
    const float beta = *pick(P.L.w_scale, li);
    float xs_m[kPer][4];
    int rs_m[kPer][4];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int rec = (tid + 64 * WAVES * i) >> 6;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int m = min(m0 + 8 * (rec & 3) + 4 * h + v, M - 1);
            xs_m[i][v] = x_scale[m];
            rs_m[i][v] = x_rowsum[m];
        }
    }
    while (kb < nkb) {
        wave_lds_handoff();                                       // the previous block's operand reads are done
#pragma unroll
        for (int i = 0; i < 8; ++i) *reinterpret_cast<v4i*>(a_dst + 4 * i * kARow) = order_a<FMT>(a[i]);
        // the short block's words are shifted into place (all selects) and cleared past K
        const bool full = kb < nfull;
        v4u b[2][NT];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int sh = full ? 0 : sh_tail[p];
            const bool s1 = (sh & 1) != 0, s2 = (sh & 2) != 0;
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) {
                const v4u v = w[p][ni];
                const uint32_t u0 = s1 ? v.y : v.x, u1 = s1 ? v.z : v.y, u2 = s1 ? v.w : v.z;
                b[p][ni].x = s2 ? u2 : u0;
                b[p][ni].y = full || Tl > 1 ? (s2 ? v.w : u1) : 0u;
                b[p][ni].z = full || Tl > 2 ? u2 : 0u;
                b[p][ni].w = full ? v.w : 0u;
            }
        }
        kb += WAVES;
        load(min(kb, nkb - 1));                                   // past the last block: repeats it, never used
        wave_lds_handoff();
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const v4i av = *reinterpret_cast<const v4i*>(a_src + 32 * s);
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) {
                const v4i bq = decode_b<FMT>(word_of(b[s & 1][ni], s >> 1));
                acc[ni] = __builtin_amdgcn_mfma_i32_32x32x32_i8(av, bq, acc[ni], 0, 0, 0);
            }
        }
    }

    // The waves' sums, in place of the staged rows: record (ni, q) of lane (j, h) holds the tokens
    // 8 q + 4 h + 0..3 of weight row 32 ni + j.  Then every thread sums and stores whole records.
    v4i* red = reinterpret_cast<v4i*>(st);
    wave_lds_handoff();
#pragma unroll
    for (int ni = 0; ni < NT; ++ni)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            red[(ni * 4 + q) * 64 + lane] =
                v4i{acc[ni][4 * q], acc[ni][4 * q + 1], acc[ni][4 * q + 2], acc[ni][4 * q + 3]};
    __syncthreads();
    float* y = pick(P.L.y, li);
    int32_t* acc_out = pick(P.L.acc, li);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int f = tid + 64 * WAVES * i;
        if (f >= kRecords) break;                                 // (64 WAVES divides or exceeds the records)
        v4i t = reinterpret_cast<const v4i*>(smem)[f];
#pragma unroll
        for (int wv = 1; wv < WAVES; ++wv) t += reinterpret_cast<const v4i*>(smem + wv * kWaveBytes)[f];
        const int rec = f >> 6;                                   // 4 ni + q; lane = f % 64 = this lane
        const int ni = rec >> 2, q = rec & 3;
        const int n = n0 + 32 * ni + j32, mb = m0 + 8 * q + 4 * h;
        if (n >= N) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int m = mb + v;
            if (m >= M) break;
            const int val = t[v] - rs_m[i][v];
            y[(size_t)m * N + n] = (float)val * (beta / xs_m[i][v]);
            if (acc_out) acc_out[(size_t)m * N + n] = val;
        }
    }
}

// Launches with rows for the whole chip: 128 weight rows x 32 tokens a work group.  Here the codes are the larger
// stream (a work group of 32 rows would pass M K bytes of codes through the cache and LDS for 8 K bytes of weights), so
// 8 waves share each staged 512-k run of every token: two columns of 64 rows, and four k-quarters (half blocks: chunk p
// of block b) whose sums meet in LDS at the end.  Codes and words are loaded a stage and two stages ahead into
// registers; one barrier a stage, the next stage's codes written to the other buffer while this one multiplies.
template <int FMT>
__global__ __attribute__((amdgpu_waves_per_eu(4, 4))) __launch_bounds__(512) void smallbatch_wide_kernel(
    SmallLinears P, const int8_t* __restrict__ xq, const float* __restrict__ x_scale,
    const int32_t* __restrict__ x_rowsum, int M, int K, int slices) {
    constexpr int NT = 2, kStageK = 2 * kI2sBlockK, kRow = kStageK + 16;
    constexpr int kBuf = 32 * kRow;
    constexpr int kPart = 4 * 64;                            // records of one 32-row half of a wave's sums
    constexpr int kSmem = 2 * kBuf > 4 * 2 * kPart * 16 ? 2 * kBuf : 4 * 2 * kPart * 16;
    __shared__ __align__(16) int8_t smem[kSmem];
    __shared__ float sc_s[32];
    __shared__ int rs_s[32];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, kq = wave >> 1, bl = kq >> 1, p = kq & 1;
    const int j32 = lane & 31, h = lane >> 5;
    const int id = xcd_logical_id(blockIdx.x, gridDim.x);
    const int tile = id / slices, m0 = (id - tile * slices) * kTok;
    int li = 0, t0 = 0;
#pragma unroll
    for (int i = 1; i < kMaxFused; ++i) {
        const int st = P.tile_start[i];
        li = tile >= st ? i : li;
        t0 = tile >= st ? st : t0;
    }
    const int N = pick(P.L.N, li);
    const int n0 = (tile - t0) * 128 + 64 * wn;                   // this wave's first row (may lie past N)
    const uint8_t* __restrict__ packed = pick(P.L.packed, li);
    const int nkb = (K + kI2sBlockK - 1) / kI2sBlockK, nfull = K / kI2sBlockK;
    const int nst = (nkb + 1) / 2;
    const int Tl = nkb > nfull ? (K - nfull * kI2sBlockK) / kSubK : 4;

    uint32_t w_rg[NT];
#pragma unroll
    for (int ni = 0; ni < NT; ++ni)
        w_rg[ni] = (uint32_t)min(n0 / kRowsPerGroup + 2 * ni + (j32 >> 4), N / kRowsPerGroup - 1) * (4u * (uint32_t)K);
    const int chunk = 16 * (2 * p + h) + (lane & 15);
    const int want = 4 * Tl * chunk;
    const uint32_t off_tail = (uint32_t)min(want, 256 * Tl - 16);
    const int sh_tail = (want - (int)off_tail) >> 2;
    auto load_w = [&](v4u (&w)[NT], int s) {
        const int kb = min(2 * s + bl, nkb - 1);
        const uint8_t* pk = packed + (size_t)kb * 1024;
        const uint32_t off = kb < nfull ? 16u * (uint32_t)chunk : off_tail;
#pragma unroll
        for (int ni = 0; ni < NT; ++ni) w[ni] = load_stream16(pk + w_rg[ni] + off);
    };
    // codes: chunk c = tid + 512 i of a stage is token row c / 32, bytes 16 (c % 32)
    auto load_a = [&](v4i (&a)[2], int s) {
        const uint32_t col = min((uint32_t)(s * kStageK + 16 * (tid & 31)), (uint32_t)K - 16u);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t row = (uint32_t)min(m0 + (tid >> 5) + 16 * i, M - 1);
            a[i] = *reinterpret_cast<const v4i*>(xq + (row * (uint32_t)K + col));
        }
    };
    int8_t* a_dst = smem + (tid >> 5) * kRow + 16 * (tid & 31);
    auto store_a = [&](const v4i (&a)[2], int buf) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            *reinterpret_cast<v4i*>(a_dst + buf * kBuf + 16 * i * kRow) = order_a<FMT>(a[i]);
    };
    const int8_t* a_src = smem + j32 * kRow + 256 * bl + 32 * p + 16 * h;

    v16i acc[NT];
#pragma unroll
    for (int ni = 0; ni < NT; ++ni) acc[ni] = v16i{};

    v4u wa[NT], wb[NT];
    v4i aa[2], ab[2];
    load_a(aa, 0);
    load_w(wa, 0);
    load_a(ab, min(1, nst - 1));
    load_w(wb, min(1, nst - 1));
    if (tid < 32) {
        const int m = min(m0 + tid, M - 1);
        sc_s[tid] = *pick(P.L.w_scale, li) / x_scale[m];
        rs_s[tid] = x_rowsum[m];
    }
    store_a(aa, 0);
    load_a(aa, min(2, nst - 1));
    // w: the words of stage s; a: the codes of stage s + 1
    auto stage = [&](v4u (&w)[NT], v4i (&a)[2], int s) {
        __syncthreads();                                          // stage s is in its buffer, the other one is free
        const int kb = 2 * s + bl, buf = s & 1;
        const bool full = kb < nfull, live = kb < nkb;
        const int sh = full ? 0 : sh_tail;
        const bool s1 = (sh & 1) != 0, s2 = (sh & 2) != 0;
        v4u b[NT];
#pragma unroll
        for (int ni = 0; ni < NT; ++ni) {
            const v4u v = w[ni];
            const uint32_t u0 = s1 ? v.y : v.x, u1 = s1 ? v.z : v.y, u2 = s1 ? v.w : v.z;
            b[ni].x = live ? (s2 ? u2 : u0) : 0u;
            b[ni].y = full || (live && Tl > 1) ? (s2 ? v.w : u1) : 0u;
            b[ni].z = full || (live && Tl > 2) ? u2 : 0u;
            b[ni].w = full ? v.w : 0u;
        }
        load_w(w, min(s + 2, nst - 1));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const v4i av = *reinterpret_cast<const v4i*>(a_src + buf * kBuf + 64 * j);
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) {
                const v4i bq = decode_b<FMT>(word_of(b[ni], j));
                acc[ni] = __builtin_amdgcn_mfma_i32_32x32x32_i8(av, bq, acc[ni], 0, 0, 0);
            }
            if (j == 1) {
                store_a(a, buf ^ 1);
                load_a(a, min(s + 3, nst - 1));
            }
        }
    };
    for (int s = 0;;) {
        stage(wa, ab, s);
        if (++s >= nst) break;
        stage(wb, aa, s);
        if (++s >= nst) break;
    }

    // Quarters 2 and 3 hand their sums to 0 and 1; those swap halves (32 rows each) and store one each.
    // Record q of a half, lane (j, h): tokens 8 q + 4 h + 0..3 of one weight row.
    v4i* red = reinterpret_cast<v4i*>(smem);
    auto put = [&](v4i* dst, int ni) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            dst[q * 64 + lane] = v4i{acc[ni][4 * q], acc[ni][4 * q + 1], acc[ni][4 * q + 2], acc[ni][4 * q + 3]};
    };
    auto add = [&](const v4i* src, int ni) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v4i o = src[q * 64 + lane];
            acc[ni][4 * q] += o.x;
            acc[ni][4 * q + 1] += o.y;
            acc[ni][4 * q + 2] += o.z;
            acc[ni][4 * q + 3] += o.w;
        }
    };
    v4i* slot = red + ((kq & 1) * 2 + wn) * 2 * kPart;            // one slot per wave of quarters 0 and 1
    __syncthreads();
    if (kq >= 2) {
        put(slot, 0);
        put(slot + kPart, 1);
    }
    __syncthreads();
    if (kq < 2) {
        add(slot, 0);
        add(slot + kPart, 1);
        // quarter 0 keeps half 0, quarter 1 half 1: the other half goes over in this wave's own slot
        if (kq == 0) put(slot, 1);
        else put(slot, 0);
    }
    __syncthreads();
    if (kq >= 2) return;
    float* y = pick(P.L.y, li);
    int32_t* acc_out = pick(P.L.acc, li);
    auto finish = [&](auto half) {
        constexpr int ni = decltype(half)::value;
        add(red + ((ni ^ 1) * 2 + wn) * 2 * kPart, ni);
        const int n = n0 + 32 * ni + j32;
        if (n >= N) return;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int ml = 8 * (v >> 2) + 4 * h + (v & 3), m = m0 + ml;
            if (m < M) {
                const int val = acc[ni][v] - rs_s[ml];
                y[(size_t)m * N + n] = (float)val * sc_s[ml];
                if (acc_out) acc_out[(size_t)m * N + n] = val;
            }
        }
    };
    if (kq == 0) finish(std::integral_constant<int, 0>{});
    else finish(std::integral_constant<int, 1>{});
}

SmallLinears tile_linears(const FusedLinears& L, int rows) {
    SmallLinears P{};
    P.L = L;
    for (int i = 0; i < kMaxFused; ++i) {
        P.tile_start[i] = i < L.count ? P.tiles : 0x7fffffff;
        if (i < L.count) P.tiles += (L.N[i] + rows - 1) / rows;
    }
    return P;
}

// A launch holds less than 2^32 threads: 2^28 rows at 97 tokens (eight weights of K = 64) are past it, so the token slices
// go in as many launches as that takes (one slice of every row that the entry points accept fits).
template <int FMT>
void launch_wide(const FusedLinears& L, const int8_t* xq, const float* x_scale, const int32_t* x_rowsum, int M, int K,
                 hipStream_t stream) {
    constexpr int64_t kThreads = 512, kMaxGroups = 0xffffffffLL / kThreads;
    SmallLinears P = tile_linears(L, 128);
    const int64_t most = kMaxGroups / P.tiles * kTok;             // tokens of one launch
    for (int64_t m0 = 0; m0 < M; m0 += most) {
        const int mc = (int)(M - m0 < most ? M - m0 : most), slices = (mc + kTok - 1) / kTok;
        for (int i = 0; i < L.count; ++i) {
            P.L.y[i] = L.y[i] + m0 * L.N[i];
            P.L.acc[i] = L.acc[i] ? L.acc[i] + m0 * L.N[i] : nullptr;
        }
        hipLaunchKernelGGL((smallbatch_wide_kernel<FMT>), dim3((unsigned)(P.tiles * slices)), dim3(kThreads), 0, stream, P,
                           xq + m0 * K, x_scale + m0, x_rowsum + m0, mc, K, slices);
    }
}

template <int NT, int WAVES, int FMT>
void launch_tile(const FusedLinears& L, const int8_t* xq, const float* x_scale, const int32_t* x_rowsum, int M, int K,
                 hipStream_t stream) {
    const SmallLinears P = tile_linears(L, 32 * NT);
    const int slices = (M + kTok - 1) / kTok;
    hipLaunchKernelGGL((smallbatch_kernel<NT, WAVES, FMT>), dim3((unsigned)(P.tiles * slices)), dim3(64 * WAVES), 0,
                       stream, P, xq, x_scale, x_rowsum, M, K, slices);
}

// The routes of a small batch: the shapes of the tile kernels, and the token slices of the decode GEMV.
enum Route { kGemvSlices, kTiles32x4, kTiles32x8, kTiles64x8, kTiles64x4, kTilesWide };

// The tile shape, by t = 32-row x 32-token tiles in the launch against the CUs (us, I2_S, K = 4096 unless given; the 8B-
// and 3B-class groups):
//   t <= CUs      32 rows, 8 waves: every tile on a CU of its own (down projection, K = 14336, 45 tokens: 12.0 against
//                 14.5 with 64 rows, 14.2 with 4 waves, 20.0 as token slices of the GEMV)
//   t <= 2 CUs    64 rows, 8 waves: still one round (q + k + v at 45 tokens: 7.4; 32 rows 8.6, GEMV 8.4)
//   t <= 4 CUs    64 rows, 4 waves: several groups to a CU, one's start under another's stream (gate + up at 32 tokens:
//                 12.6; 8 waves 15.0, wide 12.7, GEMV 15.5)
//   more          the wide kernel (gate + up at 45 tokens: 16.2; 64 rows 19.1, GEMV 22.7)
// Up to four blocks of K have no work for a fifth wave: 32 rows, 4 waves.
Route tile_route(const FusedLinears& L, int64_t M, int64_t K, int64_t cus) {
    int64_t t = 0;
    for (int i = 0; i < L.count; ++i) t += (L.N[i] + 31) / 32;
    t *= (M + kTok - 1) / kTok;
    if (t > 4 * cus) return kTilesWide;
    if (K <= 4 * kI2sBlockK) return kTiles32x4;
    return t <= cus ? kTiles32x8 : t <= 2 * cus ? kTiles64x8 : kTiles64x4;
}

// Estimated times in us, each a line through what its kernel spends time on: the start, the chain of 256-k blocks, the
// work groups on a CU, and their rounds.  Fitted to launches of 2200 shapes (17 to 1200 tokens, K to 43008, 16 to 66048
// rows, I2_S and TL1), one in three of which is off by more than 4 to 8%; checked on 1500 others.
double tiles_us(Route r, const FusedLinears& L, int64_t M, int64_t K, int64_t cus) {
    const double nkb = (double)((K + kI2sBlockK - 1) / kI2sBlockK);
    const int rows = r == kTilesWide ? 128 : r == kTiles64x8 || r == kTiles64x4 ? 64 : 32;
    int64_t groups = 0;
    for (int i = 0; i < L.count; ++i) groups += (L.N[i] + rows - 1) / rows;
    groups *= (M + kTok - 1) / kTok;
    const double g = (double)groups / (double)cus;                // work groups a CU; the wide kernel keeps two resident
    switch (r) {
        case kTiles32x4: return 3.56 + 0.10 * nkb + 0.16 * g * nkb + 0.17 * g;
        case kTiles32x8: return 3.65 + 0.14 * nkb + 0.03 * g * nkb + 0.52 * g;
        case kTiles64x8: return 4.25 + 0.18 * nkb + 0.05 * g * nkb + 0.46 * g;
        case kTiles64x4: return 4.50 + 0.34 * nkb + 0.04 * g * nkb + 0.59 * g;
        default: return 7.06 + 0.06 * nkb + 0.16 * g * nkb + 0.30 * nkb * (double)((int64_t)(g / 2) + (2 * (int64_t)(g / 2) < g));
    }
}

// The GEMV's token slices as launch_i2s_decode plans them; infinite where they are no candidate: up to four blocks of K
// (the tiles were ahead in all but four of 515 shapes, in those by 9% at most) and launches whose work groups walk more
// than three row groups, which stream, and read every word once a slice (98 tokens, 2048 -> 6144 + 6144 rows: 14.5 against
// 11.2).
double slices_us(const FusedLinears& L, int64_t M, int64_t K, int64_t cus) {
    const double never = __builtin_inf();
    if (!i2s_sliced_ok(M, K, true) || K <= 4 * kI2sBlockK) return never;
    const int64_t nkb = (K + kI2sBlockK - 1) / kI2sBlockK;
    const int64_t per = std::min<int64_t>(M, decode_slice_tokens(K)), slices = (M + per - 1) / per;
    const bool four = nkb <= 16 && L.total > cus / 2;             // 4-wave groups, several to a CU; else 16 waves, one
    const int64_t u = (nkb + (four ? 3 : 15)) / (four ? 4 : 16);  // blocks a wave
    constexpr int64_t kByRegisters[4] = {5, 4, 3, 3}, kLds = 160 * 1024, kSums = 8192;
    const int64_t occ = four ? std::max<int64_t>(1, std::min(kByRegisters[u - 1], kLds / (per * (K + 16) + kSums))) : 1;
    int64_t gx = std::max<int64_t>(kNumXcd, cus * occ / slices / kNumXcd * kNumXcd);
    const int64_t planned = (L.total + gx - 1) / gx;
    gx = (L.total + planned - 1) / planned;
    if (gx > kNumXcd) gx = gx / kNumXcd * kNumXcd;
    const int64_t rounds = (L.total + gx - 1) / gx;               // row groups a work group walks
    if (rounds > 3) return never;
    const double fill = (double)(gx * slices) / (double)cus, staged = (double)(per * K) / 65536.0 * fill;
    return four ? 3.87 - 0.15 * u + 0.19 * u * rounds + 0.11 * u * rounds * fill + 0.50 * staged
                : 3.18 + 0.34 * u + 0.95 * rounds + 0.23 * u * rounds + 0.62 * staged;
}

// The GEMV's slices are the finer split (16 rows a work group, 16 waves on one row of blocks), the tiles the cheaper one per
// word: few rows with long K go to the slices (us, slices / tiles: 64 rows of K = 11648 at 84 tokens 5.7 / 10.4; 512 of 10112
// at 31 6.1 / 9.9; 3 x 1536 of 1536 at 112 6.8 / 7.6; 1152 of 3392 at 41 5.1 / 6.3), the rest to the tiles (3840 of 3840 at
// 45 7.1 / 6.4; 4096 of 14336 at 45 20.0 / 12.0).  On a tie, the tiles.
Route route_of(const FusedLinears& L, int64_t M, int64_t K, int64_t cus) {
    const Route r = tile_route(L, M, K, cus);
    const double sliced = slices_us(L, M, K, cus);
    return sliced < __builtin_inf() && 1.02 * sliced < tiles_us(r, L, M, K, cus) ? kGemvSlices : r;
}

template <int FMT>
hipError_t launch_fmt(const FusedLinears& L, const int8_t* xq, const float* x_scale, const int32_t* x_rowsum, int M,
                      int K, hipStream_t stream) {
    switch (route_of(L, M, K, device_cus())) {
        case kGemvSlices: return launch_i2s_decode(L, xq, x_scale, x_rowsum, M, K, stream, FMT);
        case kTiles32x4: launch_tile<1, 4, FMT>(L, xq, x_scale, x_rowsum, M, K, stream); break;
        case kTiles32x8: launch_tile<1, 8, FMT>(L, xq, x_scale, x_rowsum, M, K, stream); break;
        case kTiles64x8: launch_tile<2, 8, FMT>(L, xq, x_scale, x_rowsum, M, K, stream); break;
        case kTiles64x4: launch_tile<2, 4, FMT>(L, xq, x_scale, x_rowsum, M, K, stream); break;
        default: launch_wide<FMT>(L, xq, x_scale, x_rowsum, M, K, stream); break;
    }
    return hipGetLastError();
}

}  // namespace

int smallbatch_route(const FusedLinears& L, int64_t M, int64_t K) { return route_of(L, M, K, device_cus()); }

double smallbatch_us(const FusedLinears& L, int64_t M, int64_t K) {
    const int64_t cus = device_cus();
    return std::min(tiles_us(tile_route(L, M, K, cus), L, M, K, cus), slices_us(L, M, K, cus));
}

hipError_t launch_smallbatch(const FusedLinears& L, const int8_t* xq, const float* x_scale, const int32_t* x_rowsum,
                             int M, int K, hipStream_t stream, int fmt) {
    return fmt == kFmtTl1 ? launch_fmt<kFmtTl1>(L, xq, x_scale, x_rowsum, M, K, stream)
                          : launch_fmt<kFmtI2s>(L, xq, x_scale, x_rowsum, M, K, stream);
}

}  // namespace bitnet
