// RaZeR block encoder for gfx950: Eq. 1 (tensor scale), Eq. 2 (block scale),
// Eq. 4 (special-value search) and Eq. 5 (final rounding) of arxiv 2501.04052.
//
// Bit-exactness contract: codes, scales and the tensor scale are those of the literal computation -- every fp32
// operation a single IEEE operation (true division), squared errors summed in fp64 over the block's elements in index
// order (also for blocks of 32, 64, 128 -- the block-size study of Sec. 5.4 -- where the lanes that share a block
// hand the running sum from one to the next), ties broken as documented in razer.h.  The block encoder reaches most
// of these results by cheaper operations that are proven to give the same bits; the proofs are stated there.
// Compile without fast-math.
#include "razer_device.hpp"
#include "razer_kernels.hpp"

namespace razer {

// ---------------------------------------------------------------- absmax (Eq. 1)
// The running maximum lives in kAbsmaxCells cells of the workspace (workgroup b updates cell
// b % kAbsmaxCells): atomics on a single address serialize at roughly 10 ns each, so a thousand
// workgroups on one cell cost more than the pass over a 32 MB tensor itself.
constexpr int kAbsmaxCells = 64;
constexpr int kAbsmaxBlocks = 256, kAbsmaxRowBlocks = 1024;     // dense; strided rows (one load in flight per lane)
constexpr int64_t kAbsmaxOnceBytes = (int64_t)96 << 20;
__global__ void absmax_init_kernel(uint32_t* ws) { ws[threadIdx.x] = 0u; }

// max over the cells, by every wavefront that needs it (64 lanes, one cell each)
__device__ __forceinline__ float absmax_from_cells(const uint32_t* __restrict__ ws)
{
    uint32_t m = ws[threadIdx.x & 63u];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
    return u2f(m);
}

// Bound by the read.  One workgroup per compute unit with eight loads in flight per lane: more workgroups only add
// atomics and a tail (encoder with this pass, 256 against 1024 workgroups of four loads: bf16 4096 x 4096 27.5 -> 24.8 us,
// fp32 4096 x 4096 49.7 -> 48.0; eight loads alone 27.0, 48.9).  ONCE: a tensor too large to stay in the last-level
// cache until the encoder reads it again is read around the caches (fp32 8192 x 8192 with its decoding 157 -> 146 us, bf16
// 14336 x 4096, 117 MB, 111 -> 101; 67 MB of bf16 would take 42.2 instead of 41.5, hence the line at 96 MiB).
template <typename T, bool ONCE>
__global__ __launch_bounds__(256) void absmax_kernel(const T* __restrict__ x, int64_t rows, int64_t cols,
                                                     int64_t ld, uint32_t* __restrict__ ws)
{
    // 16-byte vectors: 4 floats or 8 bf16.  |x| of finite non-negative floats orders like uint32.
    constexpr int VEC = 16 / sizeof(T);
    __shared__ uint32_t wmax[4];
    uint32_t m = 0;
    auto fold = [&](const uint4& v) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (sizeof(T) == 4) {
                m = max(m, w[j] & 0x7FFFFFFFu);
            } else {
                m = max(m, (w[j] << 16) & 0x7FFFFFFFu);
                m = max(m, w[j] & 0x7FFF0000u);
            }
        }
    };
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    if (ld == cols) {                                   // dense: one flat array of vectors
        const int64_t total = rows * cols / VEC;
        const uint4* p = reinterpret_cast<const uint4*>(x);
        int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
        for (; i + 7 * stride < total; i += 8 * stride) {        // eight loads in flight per lane
            uint4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if constexpr (ONCE) v[j] = load_once16(p + i + j * stride);
                else v[j] = p[i + j * stride];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) fold(v[j]);
        }
        for (; i < total; i += stride) fold(p[i]);
    } else {                                            // strided rows: workgroups stride over rows
        const int64_t vec_per_row = cols / VEC;
        for (int64_t r = blockIdx.x; r < rows; r += gridDim.x) {
            const uint4* p = reinterpret_cast<const uint4*>(x + r * ld);
            for (int64_t c = threadIdx.x; c < vec_per_row; c += blockDim.x) fold(p[c]);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(ws + (blockIdx.x % kAbsmaxCells), max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3])));
}

// ---------------------------------------------------------------- scale rounding (Eq. 2)
// Nearest value of the scale grid, ties to the even code, saturating at the top.
template <int FMT>
__device__ __forceinline__ uint32_t round_scale(float t)
{
    if (FMT == 2) {
        // the hardware's round-to-nearest-even cast to half; anything that would land on 2.0 or
        // above saturates at the largest 14-bit code
        const uint32_t h = __builtin_bit_cast(uint16_t, (_Float16)t);
        return (t >= 2.0f || h > 0x3FFFu) ? 0x3FFFu : h;
    }
    constexpr float kMinNormal = (FMT == 0) ? 0.25f : 0.015625f;          // 2^-2 / 2^-6
    constexpr float kSubScale = (FMT == 0) ? 32.0f : 512.0f;              // 1 / subnormal step
    constexpr uint32_t kBiasAdj = (FMT == 0) ? (124u << 3) : (120u << 3);
    constexpr uint32_t kMaxCode = (FMT == 0) ? 63u : 126u;
    uint32_t code;
    if (t < kMinNormal) {
        code = (uint32_t)__builtin_rintf(t * kSubScale);                  // exact product, RNE
    } else {
        uint32_t b = f2u(t);
        b += 0x7FFFFu + ((b >> 20) & 1u);                                 // RNE to 3 mantissa bits
        code = (b >> 20) - kBiasAdj;
    }
    return code > kMaxCode ? kMaxCode : code;
}

// Nearest FP4 value, ties to the even code, saturating at +-6: the hardware conversion (verified against the threshold
// form of the same rule on every boundary +- 1 ulp and 10^6 random values).  It writes the two codes into byte `i` of
// the packed dword; a negative value that rounds to zero comes out as code 0x8 and is cleared later.
__device__ __forceinline__ uint32_t encode_pair(uint32_t word, float a, float b, int i)
{
    return (i == 0)   ? __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, a, b, 1.0f, 0)
           : (i == 1) ? __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, a, b, 1.0f, 1)
           : (i == 2) ? __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, a, b, 1.0f, 2)
                      : __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, a, b, 1.0f, 3);
}
__device__ __forceinline__ v2f decode_pair_f32(uint32_t word, int i)      // the values of those two codes
{
    return (i == 0)   ? __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(word, 1.0f, 0)
           : (i == 1) ? __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(word, 1.0f, 1)
           : (i == 2) ? __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(word, 1.0f, 2)
                      : __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(word, 1.0f, 3);
}

// ---------------------------------------------------------------- block encoder
// A thread encodes runs of 16 elements; G = block / 16 consecutive lanes share a block: they
// agree on the block maximum (hence on the scale) by exchanging their run's maximum, and on the
// special value.
//
// What bounds it: written out literally (IEEE division, four fp64 error sums) an element costs about 220 clocks of
// a SIMD, twice what its bytes take from memory.  Two things make it cheaper without changing a bit:
//  * division.  y = 1 / den is one IEEE division per block; q = x y, then twice q += (x - q den) y with the residual
//    in one fma.  The first correction makes q faithful, and for a faithful q, a correctly rounded reciprocal and an
//    exact residual the second yields the correctly rounded quotient (Markstein's theorem); 5 operations instead of
//    ~12.  It needs normal operands: den below 2^-70 and tensor scales above 2^60 take the literal path (an element
//    whose residual is still subnormal is below 2^-30 after scaling and leaves no trace in a sum that decides anything).
//  * the special-value search.  Candidate v lowers an element's squared error by (v - q)(2 x - q - v) when that is
//    positive; sign and zero of that product are exact in fp32 (2 x - q is exact, and so is the difference to v where
//    it is close to it), so "no element takes v" and the elements that take it are known exactly, and the sums of the
//    gains to a relative error below (elements + 8) 2^-23.  The candidate with the largest gain has the smallest error
//    where the others are further away than that bound.  Where one other is not, the fp64 sums of Eq. 4 are formed for
//    those two alone (nearest_two): 16-bit data, with few distinct magnitudes, ties in about one block of 400, so one
//    wave in seven goes there.  Only what is left -- three candidates that close, non-finite blocks, blocks beyond 512
//    scales -- takes the literal chain.
// A thread has one run until the launch has 2^20; such launches wait for loads and for the slowest wave, the larger
// ones for vector issue with as many waves as registers allow.  Hence the next run is fetched while one is encoded
// (AHEAD) for 16-bit elements (8 registers, 3 % at 4096 x 4096) and for fp32 weights in blocks of 16 (11008 x 4096 with
// Eq. 1's pass 78.2 -> 76.0), not where the 16 registers of fp32 cost more waves (blocks of 64 and 128, 3-5 %) or launches
// seldom reach 2^20 runs (activations); scaled 16-bit elements are kept for nearest_two, fp32 ones are scaled again there.
// Measured against the kernel that formed all four fp64 sums for every block (us per dispatch, tensor scale given; in
// parentheses with ties decided by the literal chain): bf16 activations 4096 wide, 64 rows 5.0 (5.8) -> 5.0, 512 rows
// 6.1 (6.9) -> 5.6, 1024 rows 8.3 (8.8) -> 7.6, 4096 rows 20.2 (18.1) -> 15.6; bf16 weights in blocks of 128, 256 rows
// 7.1 (10.7) -> 6.9, 4096 rows 45.0 (27.4) -> 20.6; fp32 weights 11008 x 4096 in blocks of 16 62.0 (41.5) -> 39.3 (206 MB,
// 5.2 TB/s), of 128 120 (49.6) -> 42.4.

// Eq. 4 and the codes literally: fp32 division, squared errors in fp64, one chain over the block's elements in index
// order (lane j of the block continues where lane j - 1 ended).  lo / hi: the 16 codes as the hardware rounds them;
// take: bit k set if element k takes the chosen special value.  NP candidates go side by side; with more than one such
// pass the empty asm keeps the compiler from holding what does not depend on the candidate (the base errors, in fp64)
// over all of them: where this path is the rare one, its registers count against the occupancy of the other.
template <int FMT, int G, int NP>
__device__ __forceinline__ void encode_literal(const float (&xv)[kBlock], float den, float sv0, float sv1, uint32_t& lo,
                                               uint32_t& hi, uint32_t& meta, uint32_t& take)
{
    constexpr int NC = (FMT == 1) ? 2 : 4;
    float xs[kBlock];                                                     // X^Scaled
    lo = hi = 0;
#pragma unroll
    for (int k = 0; k < kBlock; k += 2) {
        xs[k] = xv[k] / den;
        xs[k + 1] = xv[k + 1] / den;
        uint32_t& word = (k < 8) ? lo : hi;
        word = encode_pair(word, xs[k], xs[k + 1], (k % 8) / 2);
    }
    const int sub = (int)(threadIdx.x & 63u) & (G - 1), base = (int)(threadIdx.x & 63u) & ~(G - 1);
    double best = 0.0;
    meta = 0;
    take = 0;
#pragma unroll 1
    for (int pass = 0; pass < NC / NP; ++pass) {
        // metadata index of candidate c of this pass: +sv0, (+sv1,) -sv0, (-sv1); two of four at once: one magnitude's signs
        auto index = [&](int c) { return NP == 2 && NC == 4 ? pass + 2 * c : NP == 1 ? pass : c; };
        double sse[NP], e2[G > 1 ? NP : 1][kBlock];
        uint32_t bits[NP];
#pragma unroll
        for (int c = 0; c < NP; ++c) { sse[c] = 0.0; bits[c] = 0u; }
#pragma unroll
        for (int k = 0; k < kBlock; k += 2) {
            float x0 = xs[k], x1 = xs[k + 1];
            uint32_t word = (k < 8) ? lo : hi;
            if constexpr (NP < NC) {
                asm volatile("" : "+v"(x0), "+v"(x1), "+v"(word));
#pragma unroll
                for (int c = 0; c < NP; ++c) asm volatile("" : "+v"(sse[c]), "+v"(bits[c]));
            }
            const v2f q = decode_pair_f32(word, (k % 8) / 2);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const double xd = (double)(j ? x1 : x0), eb = xd - (double)(j ? q.y : q.x);
#pragma unroll
                for (int c = 0; c < NP; ++c) {
                    const int m = index(c);
                    const float mag = (FMT != 1 && (m & 1)) ? sv1 : sv0;
                    const double ev = xd - (double)(m >= NC / 2 ? -mag : mag);
                    const bool sp = fabs(ev) < fabs(eb);
                    const double e = sp ? ev : eb;
                    if (G > 1) e2[c][k + j] = e * e;                      // exact in fp64
                    else sse[c] = __builtin_fma(e, e, sse[c]);            // the same as sse + e*e
                    bits[c] |= (uint32_t)sp << (k + j);
                }
            }
        }
        if constexpr (G > 1) {
            // round p is the one in which lane base + p of the block holds the right starting value (its predecessor's
            // total of round p - 1)
#pragma unroll 1
            for (int p = 0; p < G; ++p) {
#pragma unroll
                for (int c = 0; c < NP; ++c) {
                    double a = (p == 0) ? 0.0 : __shfl(sse[c], base + p - 1);
#pragma unroll
                    for (int k = 0; k < kBlock; ++k) a += e2[c][k];
                    sse[c] = (sub == p) ? a : sse[c];
                }
            }
        }
#pragma unroll
        for (int c = 0; c < NP; ++c) {                                    // Eq. 4: smallest error, ties to the smallest index
            const uint32_t m = (uint32_t)index(c);
            const double s = G > 1 ? __shfl(sse[c], base + G - 1) : sse[c];   // (every lane of the block: the block's sum)
            if (m == 0 || s < best || (s == best && m < meta)) {
                best = s;
                meta = m;
                take = bits[c];
            }
        }
    }
}

// x / den, correctly rounded, from y = 1 / den (correctly rounded)
__device__ __forceinline__ float quotient(float x, float den, float y)
{
    float q = x * y;
    q = __builtin_fmaf(__builtin_fmaf(-q, den, x), y, q);
    return __builtin_fmaf(__builtin_fmaf(-q, den, x), y, q);
}

// Eq. 4 between the two candidates a and b alone, the sums as above: the block is scaled and rounded, and which elements
// take a candidate is seen in fp32 -- xs - q is exact, and so is xs - v where v is the nearer of the two.
template <int FMT, int G, bool SCALED>
__device__ __forceinline__ uint32_t nearest_two(const float (&xv)[kBlock], float den, uint32_t lo, uint32_t hi, float sv0, float sv1,
                                                uint32_t a, uint32_t b)
{
    constexpr uint32_t NM = (FMT == 1) ? 1 : 2;
    const uint32_t m0 = a < b ? a : b, m1 = a < b ? b : a;
    auto value = [&](uint32_t m) { const float v = (NM == 2 && (m & 1u)) ? sv1 : sv0; return m >= NM ? -v : v; };
    const float v0 = value(m0), v1 = value(m1), y = SCALED ? 1.0f : 1.0f / den;
    double e0[G > 1 ? kBlock : 1], e1[G > 1 ? kBlock : 1];                // squared errors
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int k = 0; k < kBlock; k += 2) {
        float x0 = xv[k], x1 = xv[k + 1];
        uint32_t word = (k < 8) ? lo : hi;
        asm volatile("" : "+v"(x0), "+v"(x1), "+v"(word), "+v"(s0), "+v"(s1));   // (one pair after the other: registers)
        const v2f q = decode_pair_f32(word, (k % 8) / 2);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float xk = j ? x1 : x0, x = SCALED ? xk : quotient(xk, den, y), eb = x - (j ? q.y : q.x), f0 = x - v0, f1 = x - v1;
            const double t0 = (double)(fabsf(f0) < fabsf(eb) ? f0 : eb), t1 = (double)(fabsf(f1) < fabsf(eb) ? f1 : eb);
            if constexpr (G > 1) {
                e0[k + j] = t0 * t0;                                      // exact
                e1[k + j] = t1 * t1;
                asm volatile("" : "+v"(e0[k + j]), "+v"(e1[k + j]));
            } else {
                s0 = __builtin_fma(t0, t0, s0);
                s1 = __builtin_fma(t1, t1, s1);
            }
        }
    }
    if constexpr (G > 1) {
        const int sub = (int)(threadIdx.x & 63u) & (G - 1), base = (int)(threadIdx.x & 63u) & ~(G - 1);
#pragma unroll 1
        for (int p = 0; p < G; ++p) {
            double c0 = (p == 0) ? 0.0 : __shfl(s0, base + p - 1), c1 = (p == 0) ? 0.0 : __shfl(s1, base + p - 1);
#pragma unroll
            for (int k = 0; k < kBlock; ++k) {
                c0 += e0[k];
                c1 += e1[k];
            }
            s0 = (sub == p) ? c0 : s0;
            s1 = (sub == p) ? c1 : s1;
        }
        s0 = __shfl(s0, base + G - 1);
        s1 = __shfl(s1, base + G - 1);
    }
    return s1 < s0 ? m1 : m0;
}

template <typename T, int FMT, int G>
__global__ __launch_bounds__(256) void encode_kernel(const T* __restrict__ x, int64_t rows, int64_t cols,
                                                     int64_t ld, float sv0, float sv1,
                                                     const uint32_t* __restrict__ absmax_ws,
                                                     float* __restrict__ tensor_scale, int given_scale,
                                                     uint8_t* __restrict__ codes, uint8_t* __restrict__ scales)
{
    constexpr int NM = (FMT == 1) ? 1 : 2;                                // special magnitudes
    constexpr int NV = (int)sizeof(T);                                    // 16-byte vectors per run
    constexpr bool B16 = sizeof(T) == 2, AHEAD = B16 || (G == 1 && FMT == 0);
    const int64_t nb = cols / kBlock, runs = rows * nb;
    const int64_t first_run = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    auto load = [&](uint4 (&v)[NV], int64_t run) {
        // dense rows are one array of runs; only strided ones need the row number
        int64_t src = run * kBlock;
        if (ld != cols) {
            const int64_t r = run / nb;
            src = r * ld + (run - r * nb) * kBlock;
        }
        const uint4* xp = reinterpret_cast<const uint4*>(x + src);
#pragma unroll
        for (int j = 0; j < NV; ++j) v[j] = xp[j];
    };
    uint4 next[NV];
    if (first_run < runs) load(next, first_run);

    float delta32;
    if (given_scale) {
        delta32 = *tensor_scale;
    } else {
        float amax = absmax_from_cells(absmax_ws);
        constexpr float kDenom = (FMT == 0) ? 180.0f : (FMT == 1) ? 2688.0f : 11.994140625f;   // Qmax_scale * 6
        delta32 = (amax == 0.0f) ? 1.0f : amax / kDenom;
        if (first_run == 0) *tensor_scale = delta32;
    }

    // several runs per thread
#pragma unroll 1
    for (int64_t gid = first_run; gid < runs; gid += stride) {
        float xv[kBlock];
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const uint32_t w[4] = {next[j].x, next[j].y, next[j].z, next[j].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (sizeof(T) == 4) {
                    xv[4 * j + i] = u2f(w[i]);
                } else {
                    xv[8 * j + 2 * i + 0] = u2f(w[i] << 16);
                    xv[8 * j + 2 * i + 1] = u2f(w[i] & 0xFFFF0000u);
                }
            }
        }
        if (AHEAD) load(next, gid + stride < runs ? gid + stride : gid);

        float bmax = 0.0f;
#pragma unroll
        for (int k = 0; k < kBlock; ++k) bmax = fmaxf(bmax, fabsf(xv[k]));
        bool finite = true;                                                   // (fmaxf drops a NaN)
        if (given_scale) {                                                    // else Eq. 1's maximum has seen every element
            float z = 0.0f;
#pragma unroll
            for (int k = 0; k < kBlock; ++k) z = __builtin_fmaf(xv[k], 0.0f, z);
            finite = z == 0.0f;
        }
#pragma unroll
        for (int off = 1; off < G; off <<= 1) {                               // the block's maximum
            bmax = fmaxf(bmax, __shfl_xor(bmax, off));
            finite = __shfl_xor((int)finite, off) != 0 && finite;
        }

        // Eq. 2
        const float d = delta32 * 6.0f;
        const float t = bmax / d;
        const uint32_t sc = round_scale<FMT>(t);
        const float s = (FMT == 0) ? e3m3_value(sc) : (FMT == 1) ? e4m3_value(sc) : half14_value(sc);

        uint32_t lo = 0, hi = 0, meta = 0;                                    // 16 nibbles, low dword = k 0..7
        if (s != 0.0f) {
            float den = delta32 * s;
            uint32_t tlo = 0, thi = 0;                                        // bit 3 of a nibble: the element takes the special value
            uint32_t runner = 0;
            bool two = false, decided = finite && den >= 0x1p-70f && delta32 <= 0x1p60f && bmax <= 512.0f * den;
            uint32_t took[NM][2];
#pragma unroll
            for (int m = 0; m < NM; ++m) took[m][0] = took[m][1] = 0u;
            if (decided) {
                const float y = 1.0f / den;
                float all[NM], dir[NM];                                       // gains / 4096: sum, and sum with the element's sign
#pragma unroll
                for (int m = 0; m < NM; ++m) all[m] = dir[m] = 0.0f;
#pragma unroll
                for (int k = 0; k < kBlock; k += 2) {
                    const float xs[2] = {quotient(xv[k], den, y), quotient(xv[k + 1], den, y)};
                    uint32_t& word = (k < 8) ? lo : hi;
                    word = encode_pair(word, xs[0], xs[1], (k % 8) / 2);
                    if constexpr (B16) { xv[k] = xs[0]; xv[k + 1] = xs[1]; }  // (kept: the next pass needs them often)
                    const v2f q2 = decode_pair_f32(word, (k % 8) / 2);
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const float q = j ? q2.y : q2.x;
                        const float u = fabsf(__builtin_fmaf(2.0f, xs[j], -q));
#pragma unroll
                        for (int m = 0; m < NM; ++m) {
                            const float v = m ? sv1 : sv0;
                            // gain / 4096 (below 1 up to 512 scales), 0 where the special value is no better
                            const float g = __builtin_amdgcn_fmed3f(__builtin_fmaf(fabsf(q), -0x1p-12f, v * 0x1p-12f) * (u - v), 0.0f, 1.0f);
                            all[m] += g;
                            dir[m] += u2f(__builtin_amdgcn_bitop3_b32(f2u(g), f2u(xs[j]), 0x80000000u, 0xF8));
                            // sign bit of 0 - g: set where g > 0; eight elements shift it into the nibbles' top bits
                            uint32_t& b = took[m][k >= 8];
                            b = __builtin_amdgcn_bitop3_b32(b >> 4, f2u(0.0f - g), 0x80000000u, 0xF8);
                        }
                    }
                }
                float gain[2 * NM], total = 0.0f;
#pragma unroll
                for (int m = 0; m < NM; ++m) {
#pragma unroll
                    for (int off = 1; off < G; off <<= 1) { all[m] += __shfl_xor(all[m], off); dir[m] += __shfl_xor(dir[m], off); }
                    gain[m] = 0.5f * (all[m] + dir[m]);                       // metadata order: +sv0, (+sv1,) -sv0, (-sv1)
                    gain[NM + m] = 0.5f * (all[m] - dir[m]);
                    total += all[m];
                }
                float first = gain[0], second = -1.0f;
#pragma unroll
                for (int c = 1; c < 2 * NM; ++c) {
                    const bool up = gain[c] > first;
                    second = fmaxf(second, up ? first : gain[c]);
                    meta = up ? (uint32_t)c : meta;
                    first = up ? gain[c] : first;
                }
                // (the second term covers the rounding of the fp64 sums themselves: each at most 16 G xm^2)
                const float xm = bmax * y, margin = total * ((16.0f * G + 8.0f) * 0x1p-23f) + 1e-15f * xm * xm;
                decided = total == 0.0f || first - second > margin;
                if (!decided) {
                    int near = 0;
#pragma unroll
                    for (int c = 0; c < 2 * NM; ++c) {
                        const bool close = meta != (uint32_t)c && !(first - gain[c] > margin);
                        near += close;
                        runner = close ? (uint32_t)c : runner;
                    }
                    two = decided = near == 1;
                }
                if (B16) den = 1.0f;
            }
            if (!decided) {
                uint32_t bits;
                encode_literal<FMT, G, (G == 1 ? 2 : 1)>(xv, den, sv0, sv1, lo, hi, meta, bits);
                // bit k of a byte-wide mask to bit 4 k + 3
                auto spread = [](uint32_t b) {
                    b = (b | (b << 12)) & 0x000F000Fu;
                    b = (b | (b << 6)) & 0x03030303u;
                    return ((b | (b << 3)) & 0x11111111u) << 3;
                };
                tlo = spread(bits & 0xFFu);
                thi = spread((bits >> 8) & 0xFFu);
            }
            if (two) meta = nearest_two<FMT, G, B16>(xv, den, lo, hi, sv0, sv1, meta, runner);   // (here the elements are needed no more)
            if (decided) {
                const bool one = NM == 2 && (meta & 1u) != 0;
                const uint32_t mlo = one ? took[NM - 1][0] : took[0][0], mhi = one ? took[NM - 1][1] : took[0][1];
                const uint32_t flip = meta >= (uint32_t)NM ? 0u : 0xFFFFFFFFu;  // + candidates: elements with a clear sign bit
                tlo = mlo & (lo ^ flip);
                thi = mhi & (hi ^ flip);
            }
            // Eq. 5 on the packed nibbles: zero keeps code 0x0 whatever its sign, taken elements get the remapped code 0x8
            auto finish = [](uint32_t w, uint32_t taken) {
                const uint32_t nz = (w & 0x77777777u) + 0x77777777u;              // bit 3: magnitude not zero
                w &= nz | 0x77777777u;                                            // -0 -> +0
                return (w & ~(taken - (taken >> 3))) | taken;
            };
            lo = finish(lo, tlo);
            hi = finish(hi, thi);
        }
        *reinterpret_cast<uint2*>(codes + gid * 8) = make_uint2(lo, hi);
        if ((gid & (G - 1)) == 0) {                                           // (a row holds whole blocks)
            if (FMT == 2) reinterpret_cast<uint16_t*>(scales)[gid / G] = (uint16_t)((meta << 14) | sc);
            else scales[gid / G] = (uint8_t)((meta << (FMT == 0 ? 6 : 7)) | sc);
        }
        if (!AHEAD && gid + stride < runs) load(next, gid + stride);
    }
}

// ---------------------------------------------------------------- host launchers
constexpr int64_t kEncodeBlocks = 4096;    // workgroups of the encoder (1024 .. one run per thread: within 4 % of each other)
template <typename T, int FMT>
static void launch_encode(int lb, unsigned grid, unsigned threads, hipStream_t st, const T* x, int64_t rows,
                          int64_t cols, int64_t ld, SvConfig cfg, const uint32_t* ws, float* tensor_scale, int given,
                          uint8_t* codes, uint8_t* scales)
{
#define RAZER_ENC(G) launch(encode_kernel<T, FMT, G>, grid, threads, 0, st, x, rows, cols, ld, cfg.sv0, cfg.sv1, ws, tensor_scale, given, codes, scales)
    switch (lb) {
        case 4: RAZER_ENC(1); break;
        case 5: RAZER_ENC(2); break;
        case 6: RAZER_ENC(4); break;
        default: RAZER_ENC(8); break;
    }
#undef RAZER_ENC
}

template <typename T>
static hipError_t launch_quantize_t(int fmt, SvConfig cfg, const T* x, int64_t rows, int64_t cols, int64_t ld,
                                    uint8_t* codes, uint8_t* scales, float* tensor_scale, int given,
                                    uint32_t* ws, hipStream_t st)
{
    if (rows == 0 || cols == 0) {
        if (!given) {                       // an empty tensor gets the all-zero tensor's scale of 1
            launch(absmax_init_kernel, 1, kAbsmaxCells, 0, st, ws);
            if (fmt == 0) launch_encode<T, 0>(4, 1, 64, st, x, 0, 16, 16, cfg, ws, tensor_scale, 0, codes, scales);
            else launch_encode<T, 1>(4, 1, 64, st, x, 0, 16, 16, cfg, ws, tensor_scale, 0, codes, scales);
        }
        return hipGetLastError();
    }
    if (!given) {
        launch(absmax_init_kernel, 1, kAbsmaxCells, 0, st, ws);
        constexpr int VEC = 16 / sizeof(T);
        int64_t total = rows * (cols / VEC);
        int64_t blocks = (total + 255) / 256;
        const int64_t most = ld == cols ? kAbsmaxBlocks : kAbsmaxRowBlocks;
        if (blocks > most) blocks = most;
        if (rows * cols * (int64_t)sizeof(T) > kAbsmaxOnceBytes)
            launch(absmax_kernel<T, true>, (unsigned)blocks, 256, 0, st, x, rows, cols, ld, ws);
        else
            launch(absmax_kernel<T, false>, (unsigned)blocks, 256, 0, st, x, rows, cols, ld, ws);
    }
    int64_t nblk = rows * (cols / kBlock);
    unsigned grid = (unsigned)((nblk + 255) / 256 < kEncodeBlocks ? (nblk + 255) / 256 : kEncodeBlocks);
    if (fmt == 0) launch_encode<T, 0>(cfg.lb, grid, 256, st, x, rows, cols, ld, cfg, ws, tensor_scale, given, codes, scales);
    else if (fmt == 1) launch_encode<T, 1>(cfg.lb, grid, 256, st, x, rows, cols, ld, cfg, ws, tensor_scale, given, codes, scales);
    else launch(encode_kernel<T, 2, 8>, grid, 256, 0, st, x, rows, cols, ld, cfg.sv0, cfg.sv1, ws, tensor_scale, given, codes, scales);
    return hipGetLastError();
}

hipError_t launch_quantize(int fmt, SvConfig cfg, const void* x, int dtype_bf16, int64_t rows, int64_t cols,
                           int64_t ld, uint8_t* codes, uint8_t* scales, float* tensor_scale, int given,
                           void* ws, hipStream_t st)
{
    if (dtype_bf16)
        return launch_quantize_t<uint16_t>(fmt, cfg, (const uint16_t*)x, rows, cols, ld, codes, scales,
                                           tensor_scale, given, (uint32_t*)ws, st);
    return launch_quantize_t<float>(fmt, cfg, (const float*)x, rows, cols, ld, codes, scales, tensor_scale,
                                    given, (uint32_t*)ws, st);
}

}  // namespace razer
