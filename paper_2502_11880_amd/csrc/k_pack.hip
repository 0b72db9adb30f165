// Offline weight preprocessing: absmean ternarisation (Sec. 2.1) and packing into the I2_S format
// (Table 1, Sec. 3.2.2), the TL1 format, or the TL2 format (Sec. 3.1: mirror consolidation, signed-unsigned weight
// splitting, block-fitting weight splitting; codes of Table 5 and Table 6).
//
// beta is the fp32 value nearest to the exact mean of |W| (ties to even), so it is the same for any
// launch shape and summation order:
//   1. every |w| = m * 2^(e-150) (24-bit significand m, biased exponent e; subnormals use e = 1); the significands
//      are summed exactly into 256 uint64 buckets, bucket b weighing 2^(b-150) (registers, LDS, then global);
//   2. the last work group to finish folds the buckets into a 448-bit integer U (sum |w| = U * 2^-213), divides it
//      by N*K with 32-bit limbs, and rounds the quotient to 24 significant bits, ties to even.
// Both passes over W are bound by reading it (the second partly from the 256 MB last-level cache).  One 8B-class layer
// (seven weights, 872 MB of fp32) into I2_S: 915 -> 380 us; the 235 MB gate weight 51 us for its mean (4.6 TB/s) and
// 37 us for its packing (79 us before, 6.4 TB/s now), a 17 MB weight 12 and 5 us.
#include "bitnet_internal.hpp"

namespace bitnet {
namespace {

constexpr int kBuckets = 256;

__global__ __launch_bounds__(256) void fill_zero_u64(unsigned long long* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// The sum in the buckets divided by `count`, as the nearest fp32 (ties to even).  One whole wave; bucket b >= 1 weighs
// 2^(b-150) and holds less than 2^60.  Lane i gathers limb i of U = sum bucket[b] << (b - 1 + 64); the carries then run
// over scalars.  U / count needs 24 bits and a sticky bit: with t the top nonzero limb of U the quotient's top limb is
// t or t - 1 (count < 2^32), so the quotient of the four limbs t .. t - 3 holds the significand and the rounding bit
// (a subnormal result has t <= 3, and then these are all limbs); the remainder and the limbs below are sticky.
__device__ float mean_of_buckets(const unsigned long long* sb, unsigned long long count) {
    constexpr int kU = 14;
    const int lane = threadIdx.x & 63;
    unsigned long long part = 0;
#pragma unroll
    for (int g = 0; g < kBuckets / 64; ++g) {
        const unsigned long long mine = g == 0 && lane == 0 ? 0ull : sb[64 * g + lane];   // bucket 0 is no bucket
        unsigned long long live = __ballot(mine != 0);
        while (live) {
            const int l = __builtin_ctzll(live);
            live &= live - 1;
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, l);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), l);
            const int sh = 64 * g + l - 1 + 64, bi = sh & 31, d = lane - (sh >> 5);
            const unsigned long long vl = (unsigned long long)lo << bi, vh = (unsigned long long)hi << bi;
            part += d == 0 ? (vl & 0xffffffffull) : d == 1 ? (vl >> 32) + (vh & 0xffffffffull) : d == 2 ? vh >> 32 : 0ull;
        }
    }
    uint32_t U[kU];
    unsigned long long carry = 0;
    int t = -1;
#pragma unroll
    for (int i = 0; i < kU; ++i) {
        const unsigned long long p =
            ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(part >> 32), i) << 32) |
            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)part, i);
        carry += p;
        U[i] = (uint32_t)carry;
        carry >>= 32;
        t = U[i] ? i : t;
    }
    if (t < 0) return 0.0f;
    const int base = t > 3 ? t - 3 : 0;
    bool sticky = false;
    uint32_t u[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < kU; ++i) {
        if (i < base) sticky = sticky || U[i] != 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) u[j] = i == base + j ? U[i] : u[j];
    }
    unsigned __int128 Q = 0;
    unsigned long long rem = 0;
    for (int j = 3; j >= 0; --j) {
        const unsigned long long cur = (rem << 32) | u[j];
        Q = (Q << 32) | (uint32_t)(cur / count);
        rem = cur % count;
    }
    sticky = sticky || rem != 0;
    const unsigned long long qh = (unsigned long long)(Q >> 64), ql = (unsigned long long)Q;
    if (!qh && !ql) return 0.0f;                       // below 2^-213: rounds to zero
    const int p = 32 * base + (qh ? 127 - __clzll((long long)qh) : 63 - __clzll((long long)ql));   // value = Q 2^-213
    const int E = p - 213;
    const int shift = (E >= -126 ? p - 23 : 64) - 32 * base;
    uint32_t mant = (uint32_t)(Q >> shift) & 0xffffffu;
    const bool half = ((uint32_t)(Q >> (shift - 1)) & 1u) != 0u;
    const bool lower = sticky || (Q & (((unsigned __int128)1 << (shift - 1)) - 1)) != 0;
    if (half && (lower || (mant & 1u))) mant += 1u;
    // normal: mant in [2^23, 2^24]; subnormal: mant <= 2^23
    return __uint_as_float(E >= -126 ? ((uint32_t)(E + 126) << 23) + mant : mant);
}

constexpr int kMeanThreads = 1024;

// One window of 32 exponents per wave, from 24 below the largest exponent of its first loads: a value inside it adds
// its significand, shifted to the window's base, to a 64-bit register (2^55 at most, so 512 values before it is
// drained); the rare value outside it goes to its LDS bucket by itself.  (An LDS atomic per value, on the five or so
// buckets that hold nearly all of them, ran at 1.6 TB/s on a 67 MB weight.)
__global__ __launch_bounds__(kMeanThreads) void absmean_kernel(const float4* __restrict__ W4, size_t n4,
                                                               unsigned long long count,
                                                               unsigned long long* __restrict__ buckets,
                                                               float* __restrict__ beta_out) {
    __shared__ unsigned long long sb[kBuckets];
    __shared__ int last_s;
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < kBuckets) sb[tid] = 0ull;
    __syncthreads();

    const size_t step = (size_t)gridDim.x * kMeanThreads;
    size_t i = (size_t)blockIdx.x * kMeanThreads + tid;
    const uint4* __restrict__ B4 = reinterpret_cast<const uint4*>(W4);
    auto expo = [](uint32_t w) { return max((w & 0x7FFFFFFFu) >> 23, 1u); };
    const uint4 f = B4[i < n4 ? i : n4 - 1];
    uint32_t emax = max(max(expo(f.x), expo(f.y)), max(expo(f.z), expo(f.w)));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) emax = max(emax, (uint32_t)__shfl_xor((int)emax, off, 64));
    const uint32_t base = (uint32_t)__builtin_amdgcn_readfirstlane((int)min(max(emax, 25u) - 24u, 223u));

    unsigned long long acc = 0;
    auto add = [&](uint32_t w) {
        const uint32_t eb = (w & 0x7FFFFFFFu) >> 23;
        const uint32_t m = (w & 0x7FFFFFu) | (min(eb, 1u) << 23);
        const uint32_t d = max(eb, 1u) - base;
        if (d < 32u) acc += (unsigned long long)m << d;
        else if (m) atomicAdd(&sb[max(eb, 1u)], (unsigned long long)m);
    };
    auto add4 = [&](const uint4& v) {
        add(v.x);
        add(v.y);
        add(v.z);
        add(v.w);
    };
    auto drain = [&]() {
        // 64 lanes of 32-bit halves: below 2^38 each; bucket base + 32 <= 255
        unsigned long long lo = acc & 0xffffffffull, hi = acc >> 32;
        acc = 0;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            lo += __shfl_xor(lo, off, 64);
            hi += __shfl_xor(hi, off, 64);
        }
        if (lane == 0) {
            if (lo) atomicAdd(&sb[base], lo);
            if (hi) atomicAdd(&sb[base + 32], hi);
        }
    };
    constexpr int kUnroll = 8;
    int left = 128;                                     // float4s until the register may be full
    while (__any(i < n4)) {
        uint4 v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const size_t k = i + u * step;
            v[u] = B4[k < n4 ? k : n4 - 1];
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            if (i + u * step < n4) add4(v[u]);
        i += kUnroll * step;
        left -= kUnroll;
        if (left < kUnroll) {
            drain();
            left = 128;
        }
    }
    drain();
    __syncthreads();
    // The first wave adds this group's buckets to the device's; bucket 0 counts the groups that are done, and the last
    // one makes beta.  Everything handed over is an agent-scope atomic, so the count only has to follow the adds: the wave
    // waits until they have returned their old values (the memory clobber keeps the compiler from moving the count up).
    // That orders them on this chip; the memory model would want a release here, which writes back the XCD's whole L2: the
    // fences of 512 groups took 100 us.
    if (tid < 64) {
#pragma unroll
        for (int g = 0; g < kBuckets / 64; ++g) {
            const int b = 64 * g + tid;
            const unsigned long long s = b ? sb[b] : 0ull;
            unsigned long long old = s;
            if (s) old = __hip_atomic_fetch_add(&buckets[b], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("" : "+v"(old) : : "memory");   // the form that returns the value
        }
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        if (tid == 0)
            last_s = __hip_atomic_fetch_add(&buckets[0], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                     (unsigned long long)gridDim.x - 1;
    }
    __syncthreads();
    if (!last_s) return;
    if (tid < kBuckets) sb[tid] = __hip_atomic_load(&buckets[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (tid < 64) {
        const float beta = mean_of_buckets(sb, count);
        if (tid == 0) *beta_out = beta;
    }
}

// ---- packing ----
// One wave packs one (16-row group, k block) tile: it reads the tile's rows in whole runs (16 bytes per lane, rows of
// 1 or 1.5 KiB), turns every weight into its code t + 1 in a byte of LDS, and each lane then reads the bytes of its own
// layout chunk and writes that.  (Read straight from W, a lane's chunk is 64 to 384 bytes of one row, 16 rows a load:
// the TL2 form of that took 0.7 ms on a 235 MB weight.)  The tiles go from the end of W to its start: the end is what
// the mean's pass left in the last-level cache.
//
// t = clamp(rint(fp32(w / beta)), -1, 1) needs no division: t = 0 exactly where 2 |w| <= beta.  With w <= beta / 2 the
// quotient is at most 0.5, which rounds to 0.  The next fp32 above beta / 2 is at least beta / 2 (1 + 2^-24) away from
// it relatively (2^-23 significands have 24 bits), strictly more than the 0.5 + 2^-25 that still rounds to 0.5; of a
// subnormal beta of n units it is (n + 1) / 2 units or more, further off still.  2 |w| is exact (or infinite, and then
// above every finite beta).  beta = 0 gives 0.  Weights that are not finite keep what the division gives under
// clamp = fmin(fmax(., -1), 1): NaN is -1, and so is every weight where beta is NaN; where beta is infinite a finite
// weight is 0 and an infinite one (inf / inf) -1.
constexpr int kPackWaves = 4;

// code_of a weight w: 1 where scale |w| <= thr, else 2 where w > low, else 0.
struct Threshold {
    float scale, thr, low;
    __device__ __forceinline__ explicit Threshold(float beta) {
        const bool finite = beta < __builtin_inff();           // false for NaN
        scale = finite ? 2.0f : 1.0f;
        thr = beta == 0.0f ? __builtin_inff() : finite ? beta : beta == __builtin_inff() ? 0x1.fffffep127f : beta;
        low = finite ? 0.0f : __builtin_inff();
    }
};

__device__ __forceinline__ uint32_t code_of(float w, const Threshold& t) {
    return fabsf(w) * t.scale <= t.thr ? 1u : w > t.low ? 2u : 0u;
}
__device__ __forceinline__ uint32_t codes4(const float4& v, const Threshold& t) {
    return code_of(v.x, t) | (code_of(v.y, t) << 8) | (code_of(v.z, t) << 16) | (code_of(v.w, t) << 24);
}

// 4 bytes below 16 as 16 bits, byte 0 lowest
__device__ __forceinline__ uint32_t nibbles4(uint32_t c) {
    const uint32_t p = c | (c >> 4);
    return (p & 0xffu) | ((p >> 8) & 0xff00u);
}
// The Table 5 codes 3 (t0 + 1) + (t1 + 1) of the four pairs in eight code bytes, a byte each
__device__ __forceinline__ uint32_t pair_codes(uint32_t a, uint32_t b) {
    const uint32_t t0 = __builtin_amdgcn_perm(b, a, 0x06040200u), t1 = __builtin_amdgcn_perm(b, a, 0x07050301u);
    return 3u * t0 + t1;
}

// I2_S (FMT kFmtI2s) and TL1: tiles of up to 256 k; lane (r, q) owns the words j < T, k = 64 j + 16 q .. + 15.
template <int FMT>
__global__ __launch_bounds__(64 * kPackWaves) void pack_i2s_tiles(const float* __restrict__ W, int K, size_t tiles,
                                                                  const float* __restrict__ beta_p,
                                                                  uint32_t* __restrict__ out) {
    constexpr int kRow = kI2sBlockK + 16;               // LDS row: 16 rows' 16-byte chunks fall in different banks
    __shared__ __align__(16) uint8_t tile_s[kPackWaves][kRowsPerGroup * kRow];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t id = (size_t)blockIdx.x * kPackWaves + wave;
    if (id >= tiles) return;
    const size_t d = tiles - 1 - id;
    const int nblk = (K + kI2sBlockK - 1) / kI2sBlockK;
    const size_t R = d / (size_t)nblk;
    const int s = (int)(d - R * (size_t)nblk);
    const int T = min(4, K / kSubK - 4 * s);
    const Threshold thr(*beta_p);
    uint8_t* ts = tile_s[wave];
    const float* src = W + R * kRowsPerGroup * (size_t)K + (size_t)s * kI2sBlockK + 4 * min(lane, 16 * T - 1);
    float4 v[kRowsPerGroup];
#pragma unroll
    for (int r = 0; r < kRowsPerGroup; ++r) v[r] = *reinterpret_cast<const float4*>(src + (size_t)r * K);
#pragma unroll
    for (int r = 0; r < kRowsPerGroup; ++r) *reinterpret_cast<uint32_t*>(ts + r * kRow + 4 * lane) = codes4(v[r], thr);
    wave_lds_handoff();
    const int r = lane & 15, q = lane >> 4;
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const v4u c = *reinterpret_cast<const v4u*>(ts + r * kRow + kSubK * j + 16 * q);
        if constexpr (FMT == kFmtI2s) w[j] = c.x | (c.y << 2) | (c.z << 4) | (c.w << 6);
        else w[j] = pair_codes(c.x, c.y) | (pair_codes(c.z, c.w) << 4);
    }
    uint32_t* dst = out + R * (size_t)K + (size_t)s * kI2sBlockK + lane * T;
    if (T == 4) {
        *reinterpret_cast<v4u*>(dst) = v4u{w[0], w[1], w[2], w[3]};
    } else {
#pragma unroll
        for (int j = 0; j < 3; ++j)
            if (j < T) dst[j] = w[j];
    }
}

// TL1 words rewritten as I2_S words at the same positions (both formats tile a word as 16 weights of one row):
// weight e of the word is pair e / 2, code c: t + 1 = c / 3 for even e, c % 3 for odd e; it goes to byte e % 4,
// bits 2 (e / 4).  blockIdx.y is the weight.
struct Tl1Transcode {
    const uint32_t* src[kMaxFused];
    uint32_t* dst[kMaxFused];
    size_t nwords[kMaxFused];
};

__global__ __launch_bounds__(256) void tl1_to_i2s_words(Tl1Transcode T) {
    const int li = blockIdx.y;
    const size_t d = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (d >= T.nwords[li]) return;
    const uint32_t w = T.src[li][d];
    uint32_t o = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int i = e >> 1;
        const uint32_t c = (w >> (8 * (i & 3) + 4 * (i >> 2))) & 0xFu;
        const uint32_t code = (e & 1) ? c % 3u : c / 3u;
        o |= code << (8 * (e & 3) + 2 * (e >> 2));
    }
    T.dst[li][d] = o;
}

// TL2: tiles of 384 k (lane (r, q): 32 triples, 16 index bytes and 4 sign bytes), and one tile per row group for the
// TL1 tail (up to 320 k: one word of 8 pairs per 64-k unit).
__global__ __launch_bounds__(64 * kPackWaves) void pack_tl2_tiles(const float* __restrict__ W, int K, int nblk, int units,
                                                                  size_t tiles, const float* __restrict__ beta_p,
                                                                  uint32_t* __restrict__ idx_plane,
                                                                  uint32_t* __restrict__ sign_plane,
                                                                  uint32_t* __restrict__ tail) {
    constexpr int kRow = kTl2BlockK + 16;
    constexpr int kQuads = kTl2BlockK / 4;              // float4s per row of a whole tile
    __shared__ __align__(16) uint8_t tile_s[kPackWaves][kRowsPerGroup * kRow];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t id = (size_t)blockIdx.x * kPackWaves + wave;
    if (id >= tiles) return;
    const size_t d = tiles - 1 - id;
    const int per_rg = nblk + (units ? 1 : 0);
    const size_t R = d / (size_t)per_rg;
    const int blk = (int)(d - R * (size_t)per_rg);
    const Threshold thr(*beta_p);
    uint8_t* ts = tile_s[wave];
    const float* src = W + R * kRowsPerGroup * (size_t)K + (size_t)blk * kTl2BlockK;
    const int r = lane & 15, q = lane >> 4;
    if (blk == nblk) {                                  // the tail's 64-k units, 16 float4s of 16 rows each
        for (int u = 0; u < units; ++u) {
            float4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                v[i] = *reinterpret_cast<const float4*>(src + (size_t)(4 * i + q) * K + kSubK * u + 4 * r);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<uint32_t*>(ts + (4 * i + q) * kRow + kSubK * u + 4 * r) = codes4(v[i], thr);
        }
        wave_lds_handoff();
        for (int u = 0; u < units; ++u) {
            const v4u c = *reinterpret_cast<const v4u*>(ts + r * kRow + kSubK * u + 16 * q);
            tail[(R * 64 + lane) * (size_t)units + u] = nibbles4(pair_codes(c.x, c.y)) | (nibbles4(pair_codes(c.z, c.w)) << 16);
        }
        return;
    }
    constexpr int kPer = kRowsPerGroup * kQuads / 64;   // 24 float4s per lane
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        float4 v[kPer / 2];
#pragma unroll
        for (int i = 0; i < kPer / 2; ++i) {
            const int f = lane + 64 * (i + h * (kPer / 2)), row = f / kQuads, col = f - row * kQuads;
            v[i] = *reinterpret_cast<const float4*>(src + (size_t)row * K + 4 * col);
        }
#pragma unroll
        for (int i = 0; i < kPer / 2; ++i) {
            const int f = lane + 64 * (i + h * (kPer / 2)), row = f / kQuads, col = f - row * kQuads;
            *reinterpret_cast<uint32_t*>(ts + row * kRow + 4 * col) = codes4(v[i], thr);
        }
    }
    wave_lds_handoff();
    // 12 code bytes hold 4 triples: V = 9 (t0 + 1) + 3 (t1 + 1) + (t2 + 1) = 13 + value in a byte each (at most 26);
    // x = V + 115 has bit 7 where the value is not negative; |value| = x - 128 there and 128 - x elsewhere
    uint32_t idx[4] = {0u, 0u, 0u, 0u}, sign = 0u;
    const uint32_t* cw = reinterpret_cast<const uint32_t*>(ts + r * kRow + 96 * q);
#pragma unroll
    for (int g = 0; g < 8; ++g) {
        const uint32_t a = cw[3 * g], b = cw[3 * g + 1], c = cw[3 * g + 2];
        // bytes 0 3 6 9 | 1 4 7 10 | 2 5 8 11 of the twelve
        const uint32_t u0 = __builtin_amdgcn_perm(c, __builtin_amdgcn_perm(b, a, 0x00060300u), 0x05020100u);
        const uint32_t u1 = __builtin_amdgcn_perm(c, __builtin_amdgcn_perm(b, a, 0x00070401u), 0x06020100u);
        const uint32_t u2 = __builtin_amdgcn_perm(c, __builtin_amdgcn_perm(b, a, 0x00000502u), 0x07040100u);
        const uint32_t x = 9u * u0 + 3u * u1 + u2 + 0x73737373u;
        const uint32_t neg = (~x >> 7) & 0x01010101u;
        const uint32_t mag = ((x ^ (neg * 0x7Fu)) & 0x7F7F7F7Fu) + neg;
        idx[g >> 1] |= nibbles4(mag) << (16 * (g & 1));
        sign |= ((neg | (neg >> 7) | (neg >> 14) | (neg >> 21)) & 0xFu) << (4 * g);
    }
    const size_t chunk = (R * (size_t)nblk + blk) * 64 + lane;
    reinterpret_cast<v4u*>(idx_plane)[chunk] = v4u{idx[0], idx[1], idx[2], idx[3]};
    sign_plane[chunk] = sign;
}

inline unsigned grid_for(size_t n, int block) { return (unsigned)((n + block - 1) / block); }

}  // namespace

size_t pack_workspace_bytes() { return kBuckets * sizeof(unsigned long long); }

hipError_t launch_pack(int layout, const float* W, int64_t N, int64_t K, void* packed, float* w_scale,
                       void* ws, hipStream_t stream) {
    unsigned long long* buckets = static_cast<unsigned long long*>(ws);
    hipLaunchKernelGGL(fill_zero_u64, dim3(1), dim3(256), 0, stream, buckets, kBuckets);
    const size_t n = (size_t)N * (size_t)K;
    const size_t n4 = n / 4;
    // one work group of 16 waves per CU: with eight loads of each thread in flight as fast as two groups on large
    // weights, and half of the atomics on the same buckets at the end (17 MB: 12 against 17 us)
    const unsigned gb = (unsigned)std::min<size_t>((size_t)device_cus(), (n4 + kMeanThreads - 1) / kMeanThreads);
    hipLaunchKernelGGL(absmean_kernel, dim3(gb), dim3(kMeanThreads), 0, stream, reinterpret_cast<const float4*>(W), n4,
                       (unsigned long long)n, buckets, w_scale);
    const size_t rgs = (size_t)(N / kRowsPerGroup);
    const dim3 block(64 * kPackWaves);
    if (layout == 0 || layout == 2) {
        const size_t tiles = rgs * (size_t)((K + kI2sBlockK - 1) / kI2sBlockK);
        const dim3 grid(grid_for(tiles, kPackWaves));
        uint32_t* out = static_cast<uint32_t*>(packed);
        if (layout == 0)
            hipLaunchKernelGGL((pack_i2s_tiles<kFmtI2s>), grid, block, 0, stream, W, (int)K, tiles, w_scale, out);
        else
            hipLaunchKernelGGL((pack_i2s_tiles<kFmtTl1>), grid, block, 0, stream, W, (int)K, tiles, w_scale, out);
    } else {
        const int three = (int)(K / kTl2BlockK) * kTl2BlockK;
        const int nblk = three / kTl2BlockK, units = ((int)K - three) / kSubK;
        uint8_t* base = static_cast<uint8_t*>(packed);
        const size_t tiles = rgs * (size_t)(nblk + (units ? 1 : 0));
        hipLaunchKernelGGL(pack_tl2_tiles, dim3(grid_for(tiles, kPackWaves)), block, 0, stream, W, (int)K, nblk, units,
                           tiles, w_scale, reinterpret_cast<uint32_t*>(base),
                           reinterpret_cast<uint32_t*>(base + (size_t)N * three / 6),
                           reinterpret_cast<uint32_t*>(base + (size_t)N * three / 6 + (size_t)N * three / 24));
    }
    return hipGetLastError();
}

hipError_t launch_tl1_to_i2s(const void* const* packed, const int* N, void* const* i2s_out, int count, int K,
                             hipStream_t stream) {
    Tl1Transcode T{};
    size_t most = 0;
    for (int i = 0; i < count; ++i) {
        T.src[i] = static_cast<const uint32_t*>(packed[i]);
        T.dst[i] = static_cast<uint32_t*>(i2s_out[i]);
        T.nwords[i] = (size_t)N[i] * (size_t)K / 16;
        most = T.nwords[i] > most ? T.nwords[i] : most;
    }
    hipLaunchKernelGGL(tl1_to_i2s_words, dim3(grid_for(most, 256), (unsigned)count), dim3(256), 0, stream, T);
    return hipGetLastError();
}

}  // namespace bitnet
