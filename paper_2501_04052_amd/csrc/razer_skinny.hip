// Linear layer for 5..64 activation rows (long rows: from 2) on gfx950 (small-batch decode, Sec. 4.3 / App. D.2 of arxiv 2501.04052):
// every packed weight is read from HBM and decoded exactly once, in registers, straight into the operand of
// v_mfma_f32_16x16x32_bf16 it is used in.
//
// Mapping (ring_kernel).  A workgroup owns G groups of 16 weight rows, numbered through all matrices of the launch
// one after another; its W waves (8; 16 or 4 where launch_ring_t and launch_ring_w say so) take the 128-k steps of K in turn
// (wave w: steps w, w + W, ...).  What a step needs
// -- G x (1 KiB of codes, 64 scale entries) and the step's activation rows -- is copied global -> LDS by the load
// unit into memory that only this wave reads, so the K loop has no barrier: the wave waits for its own copies, takes
// the operands into registers, requests its next step into the same place and multiplies while that one is on its
// way.  Above 32 rows, and with 16 waves at 9 .. 16, the activations come in halves of 64 k (one 128-byte line per row), codes
// and scales still a step at a time, the next step's behind this step's second half.  Partial sums of the waves meet in LDS after one barrier.  One launch, no
// workspace (but for the K-slices of sliced_ring_kernel).
//
// Why through LDS although nothing is shared: the matrix instruction wants 16 rows in 16 neighbouring lanes, and a
// load whose neighbouring lanes lie in 16 different rows costs the address unit a cache-line lookup per lane.  Read
// straight into registers like that, the activations alone cost more than everything else together (22016 x 4096,
// 16 rows: 35.7 us, 24.6 us with the same bytes read contiguously, 16.5 us without activations).  The copies read
// 64 to 256 consecutive bytes per row; the order the lanes need comes from the LDS addresses, xor-swizzled so that a
// 128-bit read of 16 rows hits 16 different bank groups.
// What bounds it: the load path of a compute unit, which codes, scales and activations pass one after the other, then
// the decode.  22016 x 4096 at 16 rows (us; an empty loop 6.6): decode and matrix instructions alone 12.9, codes alone
// 11.5, with scales 13.5, with activations too 16.7, everything 18.3; 4096 x 11008 at 64 rows: activations alone 18, all
// copies and all of it 25.5.  More copies in flight per wave (two to four steps) only delay the last wave's data.
// Measured against the kernels this replaced (K cut into slices that met in a workspace; activations loaded into
// registers), 7B-shaped layer as 4 calls: 8 rows 59 -> 44 us, 16 rows 65 -> 48, 32 rows 84 -> 60, 64 rows (they took
// the 64-row tiles of the register-decode GEMM) 110 -> 89; FP16-scale format 8 rows 56 -> 41, 64 rows 215 -> 84.
#include <type_traits>

#include "razer_device.hpp"
#include "razer_kernels.hpp"

namespace razer {

typedef uint32_t v2u __attribute__((ext_vector_type(2)));

// 8 codes -> 8 bare, negated FP4 values as bf16, remapped codes patched with `patch` (the negated special
// value as a bf16 pair): the FP16-scale format, whose scale multiplies the block's partial sum instead.
template <int BYTE>
__device__ __forceinline__ uint32_t sk_cvt_bare_pair(uint32_t xflip, uint32_t patch)
{
    v2bf p = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(xflip, 1.0f, BYTE);
    return patch_zero_halves(__builtin_bit_cast(uint32_t, p), patch);
}
__device__ __forceinline__ v8bf sk_decode_dword_bare(uint32_t x, uint32_t patch)
{
    const uint32_t xf = x ^ kRemapXor;
    const uint4 r = make_uint4(sk_cvt_bare_pair<0>(xf, patch), sk_cvt_bare_pair<1>(xf, patch), sk_cvt_bare_pair<2>(xf, patch),
                               sk_cvt_bare_pair<3>(xf, patch));
    return __builtin_bit_cast(v8bf, r);
}

// ---- decode through byte tables ----------------------------------------------------------------------------
// A block's eight scaled magnitudes and its special value are 8 bf16 numbers: their high bytes fill one pair of
// registers and their low bytes another, and v_perm_b32 looks up four codes per instruction.  Table position of
// FP4 magnitude m: m ^ 4, position 4 (the magnitude 0) holds the negated special value; the selector of the true
// zero (code 0) gets bit 3 set as well: 12, which v_perm_b32 answers with 0x00.  The codes' sign bits flip the high
// bytes' signs afterwards (code 8 carries one, hence the negation).  The pairs come out in the order (0,2) (4,6)
// (1,3) (5,7) of the dword's codes: sk_permute_pairs() puts the activations in the same order.
// Per dword 8 byte permutes (4.2 clk each, measured) and 10 plain logic operations (2.3-2.5 clk): 58 clk against 89
// for convert, two multiplications, convert and patch per pair.
__device__ __forceinline__ uint4 sk_byte_table(uint32_t sb, float sv0, float sv1)
{
    float s, sv;
    decode_scale_byte<0>(sb, sv0, sv1, s, sv);
    // bf16 bits of s x {2, 3, 4, 6} and {special, .5, 1, 1.5}; a zero scale makes all of them 0
    const uint32_t b1 = f2u(s) >> 16, b15 = f2u(1.5f * s) >> 16, live = s != 0.0f ? 0xFFFFu : 0u;
    const uint32_t sp = (uint32_t)f32_to_bf16_rne(-(sv * s));
    const uint32_t v0 = (b1 + 0x80u) & live, v1 = (b15 + 0x80u) & live, v2 = (b1 + 0x100u) & live, v3 = (b15 + 0x100u) & live;
    const uint32_t v4 = sp, v5 = (b1 - 0x80u) & live, v6 = b1, v7 = b15;
    return make_uint4((v0 >> 8) | ((v1 >> 8) << 8) | ((v2 >> 8) << 16) | ((v3 >> 8) << 24),
                      (v4 >> 8) | ((v5 >> 8) << 8) | ((v6 >> 8) << 16) | ((v7 >> 8) << 24),
                      (v0 & 255u) | ((v1 & 255u) << 8) | ((v2 & 255u) << 16) | (v3 << 24),
                      (v4 & 255u) | ((v5 & 255u) << 8) | ((v6 & 255u) << 16) | (v7 << 24));
}
__device__ __forceinline__ v8bf sk_decode_dword_table(uint32_t x, v4u t)
{
    const uint32_t z = x ^ 0x44444444u, nz = (x | 0x88888888u) - 0x11111111u;          // bit 3 of nz: magnitude not 0
    const uint32_t sel = __builtin_amdgcn_bitop3_b32(nz, z, 0x77777777u, 0x89);         // low bits of z, bit 3 of ~(nz | z)
    const uint32_t se = sel & 0x0F0F0F0Fu, so = (sel >> 4) & 0x0F0F0F0Fu;
    const uint32_t he = __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_perm(t.y, t.x, se), x << 4, 0x80808080u, 0x78);
    const uint32_t ho = __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_perm(t.y, t.x, so), x, 0x80808080u, 0x78);
    const uint32_t le = __builtin_amdgcn_perm(t.w, t.z, se), lo = __builtin_amdgcn_perm(t.w, t.z, so);
    return __builtin_bit_cast(v8bf, make_uint4(__builtin_amdgcn_perm(he, le, 0x05010400u), __builtin_amdgcn_perm(he, le, 0x07030602u),
                                               __builtin_amdgcn_perm(ho, lo, 0x05010400u), __builtin_amdgcn_perm(ho, lo, 0x07030602u)));
}
// 8 bf16 activations in the pair order of sk_decode_dword_table
__device__ __forceinline__ v4u sk_permute_pairs(v4u a)
{
    return v4u{__builtin_amdgcn_perm(a.y, a.x, 0x05040100u), __builtin_amdgcn_perm(a.w, a.z, 0x05040100u),
               __builtin_amdgcn_perm(a.y, a.x, 0x07060302u), __builtin_amdgcn_perm(a.w, a.z, 0x07060302u)};
}

// ---------------------------------------------------------------------------------------------
// NA: activation KiB per step (m <= 4 NA); G: groups of 16 weight rows per workgroup.  LDS of a wave: the activations
// of its step [4 NA rows][256 B], in ring_parts() = 2 of half a step [4 NA rows][128 B], the codes [G][16 rows][64 B], the scale
// entries [G][16 rows][4] (a 1- or 2-byte copy lands zero-extended in 4 bytes); the partial sums reuse it.
// Halves: half the LDS and half the operand registers, so that all eight waves fit at 64 rows (seven did) and smaller
// workgroups share a unit; a lane then has 16 elements of each half instead of 32 of the step.  Against whole steps (us):
// {q,k,v} 3 x 4096 x 4096 at 64 rows 19.0 -> 17.0, 4096 x 4096 11.0 -> 9.5; with 16 waves (below) 4096 x 11008 at
// 9 rows 11.8 -> 10.7.  Elsewhere up to 32 rows slower (8192 x 8192 at 9 rows 13.1 -> 14.1, 2 x 11008 x 4096 with FP16
// scales at 32 rows 20.4 -> 22.2): whole steps there, and where ring_split_lines says so.
// SF = 1: the FP16-scale format (one step = one block of 128: one scale word per row).  The operands are bare FP4
// values and swap roles, so that a lane's four results of a step belong to ITS weight row (lane % 16) and activation
// rows 4 (lane / 16) + 0..3, and the step's sum is folded into the running sums with the lane's own scale in fp32.
constexpr int kRingWaves = 8;
constexpr uint32_t kRingTableBytes = 4096;
template <int NA, int W>
constexpr int ring_parts() { return NA == 16 || (NA == 4 && W == 16) ? 2 : 1; }
template <int NA, int H>
constexpr uint32_t ring_act_bytes() { return NA * 1024u / H; }
template <int NA, int G, int H, bool ST>
constexpr uint32_t ring_slot_bytes() { return ring_act_bytes<NA, H>() + G * (ST ? 1024u : 1280u); }
template <int NA, int G, int H, bool ST>
constexpr uint32_t ring_wave_bytes()
{
    const uint32_t slot = ring_slot_bytes<NA, G, H, ST>(), part = G * ((NA + 3) / 4) * 1024u;
    return slot > part ? slot : part;
}

// One argument, not the 33 values it holds: the runtime copies arguments one by one (0.5 us of host time per launch).
// e: first group of 16 rows behind each matrix; matrices past the last one repeat it.
struct RingArgs {
    const uint8_t* codes[4];
    const uint8_t* scales[4];
    const float* ts[4];
    uint16_t* y[4];
    int64_t n[4], ld_y[4];
    uint32_t e[4];
    float sv0, sv1;
    int64_t k, m;
    const uint16_t* a;
    int chunk, lb;
    uint32_t waves;                                                   // of a workgroup (a field: the hidden argument lies in a line of its own)
    float* partial;                                                   // K-slices: [slice][m][n] sums, steps per slice
    uint32_t slice_steps;
};

// Staged scales (ST): the scale entries of a group's 16 rows are one contiguous piece of memory, K bytes with 16-element
// blocks.  The workgroup copies the pieces of its groups to LDS once, 1 KiB per instruction, ahead of the first step,
// instead of 8 bytes per row and step: those copies ask for as many lines as the codes' (a third of all the lookups at 8
// rows), all waves for the same ones, and the load path waits where a line is asked for again that is still on its way.
// The LDS address of chunk c of 16 bytes is c ^ ((c >> 4) & 15): rows of 256 bytes (K = 4096) would all start in one bank.
__device__ __forceinline__ uint32_t ring_scale_swizzle(uint32_t byte) { return byte ^ ((byte >> 4) & 0xF0u); }
__host__ __device__ __forceinline__ uint32_t ring_scale_region(uint32_t scale_ld) { return (16u * scale_ld + 255u) & ~255u; }

// FORM: SF, + 2: whole steps where ring_parts() would take halves
template <int NA, int G, bool GB, int FORM, int W, bool IL, bool ST, bool KS = false>
__device__ __forceinline__ void ring_body(const RingArgs arg)
{
    constexpr int SF = FORM & 1, H = FORM & 2 ? 1 : ring_parts<NA, W>();
    constexpr bool EARLY = SF || ST;                                  // the tensor scales
    // All arguments in one wait (those of line 0x40 .. 0x7f, used at the end, into the scalar cache): the compiler loads them where
    // they are first used, one cold line after the other ahead of the first copy
    asm volatile("" ::"s"(arg.codes[0]), "s"(arg.ts[0]), "s"(arg.n[0]), "s"(arg.e[0]), "s"(arg.k), "s"(arg.m), "s"(arg.a), "s"(arg.chunk), "s"(arg.lb), "s"(arg.waves));
    const uint32_t e1 = arg.e[0], e2 = arg.e[1], e3 = arg.e[2], e4 = arg.e[3];
    const float sv0 = arg.sv0, sv1 = arg.sv1;
    const int64_t k = arg.k, m0 = (int64_t)blockIdx.y * arg.chunk, m = arg.m - m0 < arg.chunk ? arg.m - m0 : arg.chunk;
    const int lb = arg.lb;
    const uint16_t* a = arg.a + m0 * k;
    constexpr int NB = (NA + 3) / 4, J = 4 / H, AC = NA / H;
    constexpr uint32_t ACT = ring_act_bytes<NA, H>(), AROW = 256u / H;
    constexpr uint32_t WAVE = ring_wave_bytes<NA, G, H, ST>();
    static_assert(!ST || !IL, "the interleaved layout keeps scales with the codes");
    __shared__ uint4 lut[SF ? 1 : 256];
    extern __shared__ __align__(16) uint8_t dyn_smem[];               // [waves][WAVE], ST: [G][ring_scale_region]
    const uint32_t lane = threadIdx.x & 63u, nwaves = arg.waves;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t r = lane & 15u, g = lane >> 4;
    const uint32_t kk32 = (uint32_t)k;
    static_assert(!IL || (!GB && !SF), "interleaved layout: 16-element blocks, scale bytes");
    const uint32_t code_ld = IL ? (uint32_t)il_row_bytes(k) : (uint32_t)(k >> 1);
    const uint32_t scale_ld = IL ? code_ld : SF ? (uint32_t)(k >> 7) * 2u : (uint32_t)(k >> (GB ? lb : 4));
    const uint32_t all_steps = (kk32 + 127u) >> 7, step0 = KS ? blockIdx.z * arg.slice_steps : 0u;
    const uint32_t nsteps = KS && step0 + arg.slice_steps < all_steps ? step0 + arg.slice_steps : all_steps;   // (behind the last one)

    // copy lanes: codes and scale bits -- row lane / 4, 16-byte chunk / 32-element run; activations -- row 4 i + lane / 16
    const uint32_t wr = lane >> 2, wp = lane & 3u, wc = wp ^ ((wr >> 2) & 3u);
    const uint8_t* cbase[G];
    const uint8_t* sbase[G];
    uint32_t crow[G], srow[G], sleft[ST ? G : 1];
#pragma unroll
    for (int gi = 0; gi < G; ++gi) {
        uint32_t q = blockIdx.x * G + gi;
        q = q < e4 ? q : e4 - 1u;                                     // groups past the last one re-read it, never stored
        const uint8_t* codes = arg.codes[0]; const uint8_t* scales = arg.scales[0];
        int64_t n = arg.n[0];
        uint32_t first = 0;
        if (q >= e1) { codes = arg.codes[1]; scales = arg.scales[1]; n = arg.n[1]; first = e1; }
        if (q >= e2) { codes = arg.codes[2]; scales = arg.scales[2]; n = arg.n[2]; first = e2; }
        if (q >= e3) { codes = arg.codes[3]; scales = arg.scales[3]; n = arg.n[3]; first = e3; }
        const int64_t row0 = (int64_t)(q - first) * 16;
        const uint32_t left = (uint32_t)((n - 1 - row0 < 15) ? n - 1 - row0 : 15);
        const uint32_t dl = wr < left ? wr : left;                    // rows past N re-read the last row
        cbase[gi] = codes + row0 * (int64_t)code_ld;
        sbase[gi] = (IL ? codes + 1024 : scales) + row0 * (int64_t)scale_ld;
        crow[gi] = dl * code_ld;
        srow[gi] = dl * scale_ld;
        if constexpr (ST) sleft[gi] = left;
    }
    uint32_t arow[AC], achk[AC];
#pragma unroll
    for (int i = 0; i < AC; ++i) {
        const uint32_t row = 4u * H * i + (H == 2 ? lane >> 3 : lane >> 4);
        arow[i] = (row < (uint32_t)m ? row : (uint32_t)m - 1u) * (kk32 * 2u);
        achk[i] = H == 2 ? (lane & 7u) ^ ((row >> 1) & 7u) : (lane & 15u) ^ (row & 15u);   // logical 16-byte chunk this lane fetches
    }
#define RAZER_COPY(src, off, dst, bytes)                                                                           \
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)((src) + (off)),              \
                                     (__attribute__((address_space(3))) void*)(dst), bytes, 0, 0)
    uint8_t* ring = dyn_smem + wave * WAVE;
    const uint8_t* abytes = reinterpret_cast<const uint8_t*>(a);
    // the copies of a step: its codes and scales, the activations of a part of it
    auto issue = [&](uint32_t step, auto weights, auto acts, uint32_t part) {
        const bool full = 128u * step + 128u <= kk32;                 // uniform
        const uint32_t left = kk32 - 128u * step;                     // elements of this step inside K (>= 32)
        // byte of this step's codes / scale entries inside a row (interleaved layout: 16 steps per run of 2048 elements)
        const size_t cstep = IL ? (size_t)((step >> 4) * kIlRun + (step & 15u) * 64u) : (size_t)step * 64u;
        const size_t sstep = IL ? (size_t)((step >> 4) * kIlRun + (step & 15u) * 8u) : (size_t)step * 8u;
        const uint32_t wcc = full || wc * 32u < left ? wc : 0u, wpp = full || wp * 32u < left ? wp : 0u;
        if constexpr (decltype(weights)::value) {
#pragma unroll
            for (int gi = 0; gi < G; ++gi) RAZER_COPY(cbase[gi] + cstep, crow[gi] + wcc * 16u, ring + ACT + gi * 1024, 16);
#pragma unroll
            for (int gi = 0; gi < (ST ? 0 : G); ++gi) {
                if constexpr (SF != 0)
                    RAZER_COPY(sbase[gi] + (size_t)step * 2u, srow[gi], ring + ACT + G * 1024 + gi * 256, 2);
                else if constexpr (GB)
                    RAZER_COPY(sbase[gi], srow[gi] + ((128u * step + 32u * wpp) >> lb), ring + ACT + G * 1024 + gi * 256, 1);
                else
                    RAZER_COPY(sbase[gi] + sstep, srow[gi] + wpp * 2u, ring + ACT + G * 1024 + gi * 256, 2);
            }
        }
        if constexpr (decltype(acts)::value) {
            if constexpr (NA == 8) __builtin_amdgcn_sched_barrier(0); // (the first copies ahead of these addresses: 2 %)
            const uint32_t first = part * (128u / H);                 // elements past K: the step's first ones again
            if (NA >= 2 && H == 1 && full) {                          // (without the selections: 2 %, 64 rows 3-5)
#pragma unroll
                for (int i = 0; i < AC; ++i) RAZER_COPY(abytes + (size_t)step * 256u, arow[i] + achk[i] * 16u, ring + i * 1024, 16);
                return;
            }
#pragma unroll
            for (int i = 0; i < AC; ++i)
                RAZER_COPY(abytes + (size_t)step * 256u, arow[i] + (full || first + achk[i] * 8u < left ? first / 8u + achk[i] : 0u) * 16u, ring + i * 1024, 16);
        }
    };
    constexpr std::true_type yes;
    constexpr std::false_type no;
    // LDS addresses of this lane's operands inside a slot
    const uint32_t ring_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)ring;
    const uint32_t lut_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4*)lut;
    // H = 1: the lane's MFMA k-range are 32 elements of the step; H = 2: 16 elements of each half
    const uint32_t swz = (r >> 2) & 3u;
    const uint32_t code_lds0 = ring_lds + ACT + r * 64u + (H == 1 ? (g ^ swz) << 4 : (((g >> 1) ^ swz) << 4) + (g & 1u) * 8u);
    const uint32_t code_lds1 = code_lds0 ^ 32u;
    // ST: byte of the lane's first scale entry inside its group's piece at step 0
    const uint32_t scale_row = r * scale_ld + (SF ? 0u : GB ? 0u : H == 1 ? 2u * g : g), scale_k = H == 1 ? 32u * g : 16u * g;
    const uint32_t region = ST ? ring_scale_region(scale_ld) : 0u, staged = nwaves * WAVE;
    const uint32_t staged_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)dyn_smem + staged;
    const uint32_t scale_lds = ring_lds + ACT + G * 1024u + (H == 1 || SF ? (4u * r + g) * 4u : (4u * r + (g >> 1)) * 4u + (GB ? 0u : g & 1u));
    // (fewer than 16 staged rows: the lanes of the missing ones repeat staged rows, their product columns are never stored)
    const uint32_t ra = NA < 4 ? r & (4u * NA - 1u) : r;
    uint32_t a_lds[J];
#pragma unroll
    for (int j = 0; j < J; ++j) a_lds[j] = ring_lds + ra * AROW + (((J * g + j) ^ (H == 1 ? ra : (ra >> 1) & 7u)) << 4);

#define RAZER_DS128(dst, addr, imm) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(imm))
#define RAZER_DS64(dst, addr, imm) asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(imm))
#define RAZER_DS8(dst, addr, imm) asm volatile("ds_read_u8 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(imm))
#define RAZER_DS16(dst, addr, imm) asm volatile("ds_read_u16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(imm))

    uint32_t step = step0 + wave;                                     // (the host starts no more waves than there are steps)
    if constexpr (ST) {
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
            uint8_t* dst = dyn_smem + staged + gi * region;
            const uint32_t have = (sleft[gi] + 1u) * scale_ld;        // the last rows of a matrix: not a byte past them
            uint32_t p = wave + (gi & 1) * (nwaves >> 1);             // (the waves share the pieces evenly)
            for (p = p < nwaves ? p : p - nwaves; p * 1024u < region; p += nwaves) {
                const uint32_t at = p * 1024u + lane * 16u, from = ring_scale_swizzle(at);
                if (at < region && from + 16u <= have) RAZER_COPY(sbase[gi], from, dst + p * 1024u, 16);
            }
            const uint32_t i = (have & ~15u) + threadIdx.x;
            if (i < have) {
                const uint32_t v = sbase[gi][i];
                asm volatile("ds_write_b8 %0, %1" ::"v"(staged_lds + gi * region + ring_scale_swizzle(i)), "v"(v) : "memory");
            }
        }
    }
    issue(step, yes, yes, 0u);
    // The groups' tensor scales, requested behind the first step (read at the end, their way from memory, 2 us under load, is
    // the last thing a workgroup waits for).  FP16 scales: 4096 x 4096 at 8 rows 5.11 -> 4.75 us, x 11008 7.6 -> 7.4; staged: 57344 x
    // 8192 at 8 rows, seven workgroups per unit, 68.9 -> 62.  Not with a step's scale bytes at a time: the wait would stand
    // ahead of the table's barrier, which costs as much as it gains.
    float tensor_scales[EARLY ? G : 1];
    if constexpr (EARLY) {
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
            uint32_t q = blockIdx.x * G + gi;
            q = q < e4 ? q : e4 - 1u;
            const float* ts = arg.ts[0];
            if (q >= e1) ts = arg.ts[1];
            if (q >= e2) ts = arg.ts[2];
            if (q >= e3) ts = arg.ts[3];
            tensor_scales[gi] = *(const __attribute__((address_space(4))) float*)(uintptr_t)ts;
        }
    }
    if (!SF) {
        for (uint32_t sb = threadIdx.x; sb < 256u; sb += 64u * nwaves) {
            const v4u e = __builtin_bit_cast(v4u, sk_byte_table(sb, sv0, sv1));
            asm volatile("ds_write_b128 %0, %1" ::"v"(lut_lds + sb * 16u), "v"(e) : "memory");
        }
        if constexpr (!ST) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
    }
    if constexpr (ST) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    if constexpr (EARLY) {
#pragma unroll
        for (int gi = 0; gi < G; ++gi) asm volatile("" : "+s"(tensor_scales[gi]));   // (loaded here, not at its use)
    }
    v4f acc[G][NB];
#pragma unroll
    for (int gi = 0; gi < G; ++gi)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[gi][b] = v4f{0.f, 0.f, 0.f, 0.f};

    typedef typename std::conditional<H == 1, v4u, v2u>::type Codes;
    while (step < nsteps) {
        Codes cw[G][H];
        uint32_t sw[G][SF ? 1 : H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            // what this part reads has landed: in the second half the next step's codes and scales, the newest 2 G
            // copies (with staged scales G), may be under way (copies land in the order of their issue)
            if (h == 1 && step + nwaves < nsteps) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((ST ? 1 : 2) * G) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            v4u af[NB][J];
            if (h == 0) {
                uint32_t s_at[H];
                if constexpr (ST) {
#pragma unroll
                    for (int i = 0; i < H; ++i) {
                        const uint32_t off = SF ? step * 2u : GB ? (128u * step + 64u * i + scale_k) >> lb : step * 8u + 4u * i;
                        s_at[i] = staged_lds + ring_scale_swizzle(scale_row + off);
                    }
                }
#pragma unroll
                for (int gi = 0; gi < G; ++gi) {
                    if constexpr (ST) {
                        if constexpr (SF || (H == 1 && !GB)) RAZER_DS16(sw[gi][0], s_at[0] + gi * region, 0);
                        else {
                            RAZER_DS8(sw[gi][0], s_at[0] + gi * region, 0);
                            if constexpr (H == 2) RAZER_DS8(sw[gi][H - 1], s_at[H - 1] + gi * region, 0);
                        }
                    } else if constexpr (H == 1 || SF) RAZER_DS16(sw[gi][0], scale_lds, gi * 256);
                    else { RAZER_DS8(sw[gi][0], scale_lds, gi * 256); RAZER_DS8(sw[gi][H - 1], scale_lds, gi * 256 + 8); }
                    if constexpr (H == 1) RAZER_DS128(cw[gi][0], code_lds0, gi * 1024);
                    else { RAZER_DS64(cw[gi][0], code_lds0, gi * 1024); RAZER_DS64(cw[gi][H - 1], code_lds1, gi * 1024); }
                }
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int j = 0; j < J; ++j) RAZER_DS128(af[b][j], a_lds[j], b * 16 * AROW);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (h == 0) {
#pragma unroll
                for (int gi = 0; gi < G; ++gi)
#pragma unroll
                    for (int i = 0; i < H; ++i) {
                        asm volatile("" : "+v"(cw[gi][i]));
                        if (!SF || i == 0) asm volatile("" : "+v"(sw[gi][SF ? 0 : i]));
                    }
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int j = 0; j < J; ++j) asm volatile("" : "+v"(af[b][j]));
            v4u le[G][GB || H == 2 ? 1 : 2];
            if constexpr (!SF) {
#pragma unroll
                for (int gi = 0; gi < G; ++gi) {
                    RAZER_DS128(le[gi][0], lut_lds + (H == 2 ? sw[gi][h] : sw[gi][h] & 255u) * 16u, 0);
                    if constexpr (!GB && H == 1) RAZER_DS128(le[gi][1], lut_lds + (sw[gi][0] >> 8) * 16u, 0);
                }
            }
            // (everything that the copies overwrite has been read)
            const uint32_t next = step + nwaves;
            if (h + 1 < H) {
                issue(step, no, yes, 1u);
                __builtin_amdgcn_sched_barrier(0x40F);                // no memory operation crosses: the second half's wait counts on this order
            }
            if (next < nsteps) {
                if constexpr (H == 1) issue(next, yes, yes, 0u);
                else if (h == 0) issue(next, yes, no, 0u);
                else issue(next, no, yes, 0u);
            }
            if (128u * step + 128u > kk32) {                              // ragged last step: activations past K are 0 (0 x Inf is not)
                const uint32_t keep = (128u * step + 64u * h + 8u * J * g < kk32) ? 0xFFFFFFFFu : 0u;
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int j = 0; j < J; ++j) af[b][j] &= keep;
            }
            if constexpr (!SF) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int j = 0; j < J; ++j) af[b][j] = sk_permute_pairs(af[b][j]);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int gi = 0; gi < G; ++gi) {
                    asm volatile("" : "+v"(le[gi][0]));
                    if constexpr (!GB && H == 1) asm volatile("" : "+v"(le[gi][1]));
                }
            }
#pragma unroll
            for (int gi = 0; gi < G; ++gi) {
                if constexpr (SF != 0) {
                    float bs, sv;
                    decode_scale_word(sw[gi][0], sv0, sv1, bs, sv);
                    const uint32_t nsv = (uint32_t)f32_to_bf16_rne(-sv);
                    v4f blk[NB];
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        const v8bf wf = sk_decode_dword_bare(cw[gi][h][j], nsv | (nsv << 16));
#pragma unroll
                        for (int b = 0; b < NB; ++b)
                            blk[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, af[b][j]), wf,
                                                                             j == 0 ? v4f{0.f, 0.f, 0.f, 0.f} : blk[b], 0, 0, 0);
                    }
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[gi][b][i] = __builtin_fmaf(bs, blk[b][i], acc[gi][b][i]);
                } else {
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        const v8bf wf = sk_decode_dword_table(cw[gi][h][j], le[gi][(GB || H == 2 || j < 2) ? 0 : 1]);
#pragma unroll
                        for (int b = 0; b < NB; ++b)
                            acc[gi][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, __builtin_bit_cast(v8bf, af[b][j]), acc[gi][b], 0, 0, 0);
                    }
                }
            }
        }
        step += nwaves;
    }
#undef RAZER_DS128
#undef RAZER_DS64
#undef RAZER_DS16
#undef RAZER_DS8
#undef RAZER_COPY

    // partial sums in the wave's own ring (all its copies have landed and been read)
    float4* part = reinterpret_cast<float4*>(ring);
#pragma unroll
    for (int gi = 0; gi < G; ++gi)
#pragma unroll
        for (int b = 0; b < NB; ++b)
            part[(gi * NB + b) * 64 + lane] = make_float4(acc[gi][b][0], acc[gi][b][1], acc[gi][b][2], acc[gi][b][3]);
    __syncthreads();
    // unit u = (group gi, fragment b), one wave each: lane l holds rows 16 q + 4 (l / 16) + 0..3, column 16 b + l % 16
    for (uint32_t u = wave; u < (uint32_t)(G * NB); u += nwaves) {
        const uint32_t gi = u / NB, b = u % NB, q = blockIdx.x * G + gi;
        if (q >= e4) break;
        const float* ts = arg.ts[0]; uint16_t* y = arg.y[0];
        int64_t n = arg.n[0], ld_y = arg.ld_y[0];
        uint32_t first = 0;
        if (q >= e1) { ts = arg.ts[1]; y = arg.y[1]; n = arg.n[1]; ld_y = arg.ld_y[1]; first = e1; }
        if (q >= e2) { ts = arg.ts[2]; y = arg.y[2]; n = arg.n[2]; ld_y = arg.ld_y[2]; first = e2; }
        if (q >= e3) { ts = arg.ts[3]; y = arg.y[3]; n = arg.n[3]; ld_y = arg.ld_y[3]; first = e3; }
        y += m0 * ld_y;
        const int64_t row0 = (int64_t)(q - first) * 16;
        float sc = 1.0f;
        if constexpr (KS) {
        } else if constexpr (EARLY) {
            sc = tensor_scales[0];
#pragma unroll
            for (int i = 1; i < G; ++i) sc = gi == (uint32_t)i ? tensor_scales[i] : sc;
        } else {
            sc = *ts;
        }
        sc = SF ? -sc : sc;                                               // (the bare decode carries a negation)
        float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
        for (uint32_t w = 0; w < nwaves; ++w) {
            const float4 p = *reinterpret_cast<const float4*>(dyn_smem + w * WAVE + (u * 64u + lane) * 16u);
            t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
        }
        const float v[4] = {t.x, t.y, t.z, t.w};
        if constexpr (KS) {
            // (negated: slice_reduce_kernel undoes the negation of the other kernels' decode)
            const int64_t gn = row0 + 4 * g, gm = 16 * b + r;
            if (gm < m && gn < n) {
                float* dst = arg.partial + ((int64_t)blockIdx.z * m + gm) * n + gn;
                if ((n & 3) == 0) {
                    *reinterpret_cast<float4*>(dst) = make_float4(-t.x, -t.y, -t.z, -t.w);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (gn + i < n) dst[i] = -v[i];
                }
            }
        } else if constexpr (SF != 0) {
            // swapped operands: weight row 16 q + l % 16, activation rows 16 b + 4 (l / 16) + 0..3
            const int64_t wn = row0 + r;
            if (wn < n) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t am = 16 * b + 4 * g + i;
                    if (am < m) y[am * ld_y + wn] = f32_to_bf16_rne(sc * v[i]);
                }
            }
        } else {
            const int64_t gn = row0 + 4 * g, gm = 16 * b + r;
            if (gm < m && gn < n) {
                uint16_t* dst = y + gm * ld_y + gn;
                if (gn + 3 < n && ((reinterpret_cast<uintptr_t>(dst) & 7u) == 0)) {
                    const uint32_t lo = (uint32_t)f32_to_bf16_rne(sc * t.x) | ((uint32_t)f32_to_bf16_rne(sc * t.y) << 16);
                    const uint32_t hi = (uint32_t)f32_to_bf16_rne(sc * t.z) | ((uint32_t)f32_to_bf16_rne(sc * t.w) << 16);
                    *reinterpret_cast<uint2*>(dst) = make_uint2(lo, hi);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (gn + i < n) dst[i] = f32_to_bf16_rne(sc * v[i]);
                }
            }
        }
    }
}

template <int NA, int G, bool GB, int FORM, int W, bool IL = false>
__global__ __launch_bounds__(64 * W) void ring_kernel(const RingArgs arg)
{
    ring_body<NA, G, GB, FORM, W, IL, false>(arg);
}
template <int NA, int G, bool GB, int FORM, int W, bool IL = false>
__global__ __launch_bounds__(64 * W) void staged_ring_kernel(const RingArgs arg)
{
    ring_body<NA, G, GB, FORM, W, IL, true>(arg);
}
// blockIdx.z: a slice of K; its sums go to the workspace.
template <int NA, int G, bool GB, int FORM, int W, bool IL = false>
__global__ __launch_bounds__(64 * W) void sliced_ring_kernel(const RingArgs arg)
{
    ring_body<NA, G, GB, FORM, W, IL, false, true>(arg);
}

// More than 64 activation rows go in equal runs of at most 64, blockIdx.y counting them.
static int64_t ring_chunk(int64_t m)
{
    const int64_t chunks = (m + kRingMaxM - 1) / kRingMaxM;
    return (m + chunks - 1) / chunks;
}
static int64_t ring_row_groups(int count, const GemvProblem* p)
{
    int64_t groups = 0;
    for (int i = 0; i < count; ++i) groups += (p[i].n + 15) / 16;
    return groups;
}
template <int G>
static int64_t ring_wgs(int count, const GemvProblem* p, int64_t m)
{
    return (ring_row_groups(count, p) + G - 1) / G * ((m + kRingMaxM - 1) / kRingMaxM);
}

// Staged scales or a step's at a time.  Staging takes the scales out of the load path's way, which every workgroup of a unit
// gains from, and costs a start: no wave begins before all scales and every wave's first step are there.  So it pays with
// the work of a workgroup (G x steps of 128 elements) and with several workgroups per unit, which start over each other's
// work.  Time with staged scales against without at 8 / 16 / 64 rows.  Several workgroups per unit: 22016 x 1024 (G x steps =
// 24) 1.05 / 1.07 / 1.03, x 2048 (48) 0.97 / 0.97 / 1.00, x 4096 0.98 / 0.95 / 0.96, x 6144 0.91 / 0.92 / 0.95, 57344 x 8192 at 8 rows 0.88
// (68.7 -> 60.6 us); FP16 scales 22016 x 4096 (96) 1.02 / 1.02 / 0.99, 28672 x 4096 (128) 0.98 / 0.99 / 1.00, 57344 x 8192 0.86 / 0.87 / 0.95.
// One workgroup per unit: 4096 x 4096 (32) 1.11 / 1.10 / 1.04, 12288 x 4096 (96) 1.03 / 1.03 / 1.01, 12288 x 6144 (144) 1.02 / 0.99 / 0.98,
// 12288 x 8192 (192) 1.00 / 0.97 / 0.98, 12288 x 20480 0.85 / 0.83 / 0.99; with one or two groups later: 8192 x 12288 (192) 1.01 / 0.99 /
// 0.97, 5120 x 13824 (216) at 24 rows 1.08, 8192 x 20480 (320) 0.95 / 0.93 / 0.95, x 28672 at 8 rows 0.95.  Where the regions leave
// LDS for fewer workgroups than without them: two are as good as three up to 32 rows; one instead of two pays from about
// 190 (28672 x 4096 at 16 rows 1.07, x 6144 0.98, 22016 x 8192 1.01, 28672 x 8192 0.96); above 32 rows (four waves) behind: 57344 x
// 8192 1.16.  Runs of more than 64 rows gain nothing (3 x 5120 x 3840 at 571 rows 1.01, 2 x 5120 x 5120 at 320 1.00) and lose where
// outputs are stored an element at a time (3 x 5098 x 3808 at 571 1.05): launch_ring_w leaves them out.
template <int NA, int G>
static bool ring_stages(bool f16, int64_t wgs, int64_t nsteps, size_t plain, size_t staged)
{
    const int64_t per_unit = (wgs + kComputeUnits - 1) / kComputeUnits, now = kLdsBytes / plain, then = kLdsBytes / staged, work = G * nsteps;
    if (then < 1) return false;
    if (then < now && then < per_unit && (NA > 8 || (then < 2 && work < 190))) return false;
    if (per_unit > 1) return work >= (f16 ? 120 : 48);
    return work >= (G <= 2 ? 300 : NA <= 2 ? 190 : 140);
}

template <int NA, int G, bool GB, int SF, bool IL, int W, int H = ring_parts<NA, W>()>
static hipError_t launch_ring_w(SvConfig cfg, int count, const GemvProblem* p, int64_t k, const uint16_t* a, int64_t m, int asked, hipStream_t st)
{
    RingArgs arg;
    uint32_t groups = 0;
    for (int i = 0; i < 4; ++i) {
        const GemvProblem& q = p[i < count ? i : count - 1];
        arg.codes[i] = q.codes;
        arg.scales[i] = q.scales;
        arg.ts[i] = q.ts;
        arg.y[i] = q.y;
        arg.n[i] = q.n;
        arg.ld_y[i] = q.ld_y;
        if (i < count) groups += (uint32_t)((q.n + 15) / 16);
        arg.e[i] = groups;
    }
    arg.sv0 = cfg.sv0;
    arg.sv1 = cfg.sv1;
    arg.k = k;
    arg.m = m;
    arg.chunk = (int)ring_chunk(m);
    arg.a = a;
    arg.lb = cfg.lb;
    arg.waves = 0;
    arg.partial = nullptr;
    arg.slice_steps = 0;
    // as many of the W waves as their LDS leaves room for
    constexpr uint32_t fit = (kLdsBytes - kRingTableBytes) / ring_wave_bytes<NA, G, H, false>();
    constexpr int most = fit < (uint32_t)W ? (int)fit : W;
    static_assert(most >= 4, "LDS");
    const int64_t nsteps = (k + 127) / 128;
    const int64_t wgs = ring_wgs<G>(count, p, m);
    const int use = NA == 16 && wgs > kComputeUnits && asked != 8 ? 4 : most;
    const int waves = nsteps < use ? (int)nsteps : use;
    arg.waves = (uint32_t)waves;
    constexpr int FORM = SF + (H == ring_parts<NA, W>() ? 0 : 2);
    const dim3 grid((groups + G - 1) / G, (unsigned)((m + arg.chunk - 1) / arg.chunk));
    const size_t plain = (size_t)waves * ring_wave_bytes<NA, G, H, false>();
    if constexpr (!IL) {
        const int64_t scale_ld = SF ? (k >> 7) * 2 : k >> cfg.lb;
        if (scale_ld <= (int64_t)kLdsBytes / 16) {
            const size_t staged = (size_t)waves * ring_wave_bytes<NA, G, H, true>() + G * (size_t)ring_scale_region((uint32_t)scale_ld);
            if (m <= kRingMaxM && ring_stages<NA, G>(SF != 0, wgs, nsteps, plain + kRingTableBytes, staged + kRingTableBytes)) {
                auto kern = staged_ring_kernel<NA, G, GB, FORM, W, IL>;
                RAZER_RAISE_LDS_LIMIT(kern, kLdsBytes - kRingTableBytes);
                launch(kern, grid, 64 * waves, staged, st, arg);
                return hipGetLastError();
            }
        }
    }
    auto kern = ring_kernel<NA, G, GB, FORM, W, IL>;
    constexpr uint32_t lds = (uint32_t)most * ring_wave_bytes<NA, G, H, false>();
    if constexpr (lds > 64u * 1024u) RAZER_RAISE_LDS_LIMIT(kern, lds);
    launch(kern, grid, 64 * waves, plain, st, arg);
    return hipGetLastError();
}

// Rows of an odd number of 32-element runs start in the middle of a 128-byte line, and half a step of such a row (128
// bytes) lies in two lines: halves then ask for four lines where the whole step asks for three.  Whole steps (and 8 waves)
// where that shows, which is where many rows are read or many workgroups read them (us, halves -> whole): one group,
// 4096 x 3360 at 64 rows 10.3 -> 9.8, 4096 x 8224 22.1 -> 20.7; 100 x 11040 at 190 rows 26.0 -> 23.5, 500 x 16416 at 448
// 35.2 -> 31.8; two groups, 8192 x 16416 at 64 rows 52.3 -> 49.3, 5003 x 8224 at 64 25.7 -> 24.9; 4096 x 8224 at 16 rows
// 11.1 -> 10.5.  Below the lines halves stay ahead: 100 x 8224 at 64 rows 13.5, whole 14.8; 500 x 5792 at 190 13.0, 13.5; 5003 x 3360 at
// 37 rows 10.5, 10.9; 1500 x 11040 at 12 rows 9.0, 9.7.
template <int NA, int G>
static bool ring_split_lines(int count, const GemvProblem* p, int64_t k, int64_t m)
{
    const int64_t wgs = ring_wgs<G>(count, p, m), rows = ring_chunk(m);
    if (k % 64 == 0) return false;
    if (NA == 4) return m > 12 || m * k > 200000 || wgs > 160;
    if (NA != 16 || wgs > kComputeUnits) return false;
    return m * k > 1200000 || (G == 1 ? rows > 48 && wgs > 192 : rows * k > 250000);
}

// 9 .. 16 activation rows, one group of weight rows: whether the rows are long enough for 16 waves.  Sixteen start and meet
// later than eight and save steps of the longest wave; eight also take the copies of a full step without selections.
// Time of 16 waves against 8 at 12 rows, scale bytes: 4096 elements 1.05 with 64 weight rows, 1.02 with 1000 to 4096;
// 4608 1.05, 1.01; 4736 1.01, 0.97; 6656 1.02, 0.98; 6784 0.98, 0.96; 11008 0.96, 0.92 .. 0.94 (4096 x 11008 13.0 -> 12.3 us).
// FP16 scales: 4096 1.07, 1.05; 6656 1.05, 1.03; 8192 1.04, 1.01; 8832 with 2000 weight rows and more 0.98 (at 16 rows
// 1.01); 10496 1.02, 0.99; 11008 0.99, 0.95.  (A step is 128 elements.)
static bool ring_long_rows(bool f16, int count, const GemvProblem* p, int64_t k, int64_t m)
{
    const int64_t steps = (k + 127) / 128, groups = ring_row_groups(count, p);
    return f16 ? steps > 82 || (steps > 68 && groups > 120 && m <= 12) : steps > 52 || (steps > 36 && groups > 40);
}

// 8 waves; 16 for one group of rows and at most 8 activation rows, or 16 where the rows are long: such a launch has at most
// one workgroup per compute unit and little data under way, so twice the waves pay (4096 x 11008 at 4 rows 11.0 -> 8.8 us,
// at 8 rows 11.1 -> 9.8; at 24 and 32 rows within 2 %, with two groups or more 0-15 % slower); 16 again above 32 rows with
// one group and rows of 10240 elements and more (4096 x 11008 at 64 rows 25.2 -> 24.4; 4096 x 4096 9.5 -> 10.0).
// 4 above 32 rows when the workgroups outnumber the compute units: three or four of them then share a unit, each at
// another point of its steps (2 x 11008 x 4096 at 64 rows 31.4 -> 28.9; with one workgroup per unit 8 stay faster:
// {q,k,v} 3 x 4096 x 4096 17.0, with 4 waves 18.4).  The number of waves decides the order of the sum over K: asked: 8 or 16
// where a launch shape asks for them (16 only where built and, from 9 rows up, with rows of 4096 elements or more).
template <int NA, int G, bool GB, int SF, bool IL = false>
static hipError_t launch_ring_t(SvConfig cfg, int count, const GemvProblem* p, int64_t k, const uint16_t* a, int64_t m, int asked, hipStream_t st)
{
    if constexpr (G == 1 && NA == 1) {                            // (up to 4 rows no launch shape is asked for)
        return launch_ring_w<NA, G, GB, SF, IL, 16>(cfg, count, p, k, a, m, asked, st);
    } else {
        if constexpr (G == 1 && NA <= 4) {
            if (asked != 8 && (NA < 4 || ((asked == 16 ? k >= 4096 : ring_long_rows(SF != 0, count, p, k, m)) && !ring_split_lines<NA, G>(count, p, k, m))))
                return launch_ring_w<NA, G, GB, SF, IL, 16>(cfg, count, p, k, a, m, asked, st);
        }
        if constexpr (NA == 16 && G <= 2 && !SF) {
            if (ring_split_lines<NA, G>(count, p, k, m))
                return launch_ring_w<NA, G, GB, SF, IL, kRingWaves, 1>(cfg, count, p, k, a, m, asked, st);
        }
        if constexpr (G == 1 && NA == 16) {
            if (asked != 8 && k >= 10240) return launch_ring_w<NA, G, GB, SF, IL, 16>(cfg, count, p, k, a, m, asked, st);
        }
        return launch_ring_w<NA, G, GB, SF, IL, kRingWaves>(cfg, count, p, k, a, m, asked, st);
    }
}

// Groups of 16 rows per workgroup.  The busiest of the 256 compute units holds ceil(workgroups / 256) workgroups of G
// groups each; what a workgroup spends on its activations (m x K, whatever G is) grows with m / G: about 5.5 % of a
// group's time per activation row.  Six groups leave one workgroup of eight waves per unit, which overlaps less
// (15 %).  Measured over 1024 x 1024 .. 57344 x 8192 at 4..64 rows, with eight waves throughout (above 32 rows four, where
// workgroups share a unit, came later), this picks the fastest G or one within 3 % of it:
// 4096 rows 1; 8192 or 5003 rows 2; {q,k,v} 3 x 4096 or 10240 rows 3; 2 x 11008 rows 3, with 32 activation rows 6.
// More than 32 activation rows take at most 4 groups (the FP16-scale format 3): with whole steps six did not fit the registers,
// and their sums take 24 KiB of LDS per wave; with halves they have not been tried.
static int ring_groups(int64_t groups, int64_t m, bool f16)
{
    int best = 1;
    double cost = 0.0;
    const int64_t chunks = (m + kRingMaxM - 1) / kRingMaxM;
    m = ring_chunk(m);
    for (int g : {1, 2, 3, 4, 6}) {
        if (m > 32 && g > (f16 ? 3 : 4)) continue;
        const int64_t wgs = chunks * ((groups + g - 1) / g);
        const double c = (double)(g * ((wgs + kComputeUnits - 1) / kComputeUnits)) * (1.0 + 0.055 * (double)m / g) * (g == 6 ? 1.15 : 1.0);
        if (g == 1 || c < cost) { best = g; cost = c; }
    }
    return best;
}
// About how long (us) a scale-byte call above 64 activation rows takes here: per round of workgroups (above 32 rows several
// share a unit; with less than a full round more their number still counts as rounded up) K times what a group of weight
// rows and an activation row cost, rows that start inside a 128-byte line nearly twice as much; 16 waves are 10 % slower
// again from about 18000 elements; activations that the XCDs fetch each for itself and that leave the L2; and the output,
// which rows that are no multiple of 4 let a lane store only an element at a time.  Fitted to 863 calls before short launches
// got 3 to 6 % faster.  As the kernels are now, on 212 other calls on which neither kernel takes more than 1.7 times the
// other's time, the middle is 1.00 of the estimate and 90 % lie within 0.78 and 1.13; those far below it are long rows of
// few weights (114 x 104 x 8480 13.2 us, estimate 18.2), those above it many runs of few weights (1994 x 2 x 72 x 8256 30.5, 25.3).
static double ring_estimate_us(int count, const GemvProblem* p, int64_t k, int64_t m)
{
    int64_t rows = 0;
    bool by4 = true;
    for (int i = 0; i < count; ++i) {
        rows += p[i].n;
        by4 = by4 && p[i].n % 4 == 0;
    }
    const int64_t groups = ring_row_groups(count, p);
    const int g = ring_groups(groups, m, false);
    const int64_t chunks = (m + kRingMaxM - 1) / kRingMaxM, per_run = (groups + g - 1) / g, rounds = (chunks * per_run + kComputeUnits - 1) / kComputeUnits;
    double kk = 1e-3 * (double)k;
    const double fetched = kk * 1e-3 * (double)(m * (per_run < 8 ? per_run : 8)), values = 1e-6 * (double)(m * rows);
    if (k > 18000 && g == 1 && rounds == 1) kk *= 1.1;
    const double row = k % 64 == 0 ? 0.0074 : 0.0131;
    return 5.1 + (double)rounds * kk * (0.27 + row * (double)ring_chunk(m) + 0.52 * g) + (fetched > 40.0 ? 0.115 * (fetched - 40.0) : 0.0) +
           (by4 ? 2.2 : 2.5) * values;
}

template <int G, bool GB>
static hipError_t launch_ring_slices(SvConfig cfg, const GemvProblem& p, int64_t k, const uint16_t* a, int64_t m, int slices, float* workspace, hipStream_t st)
{
    constexpr int NA = 16, W = kRingWaves, H = ring_parts<NA, W>();
    const uint32_t groups = (uint32_t)((p.n + 15) / 16), steps = (uint32_t)((k + 127) / 128), per = (steps + slices - 1) / slices;
    RingArgs arg;
    for (int i = 0; i < 4; ++i) {
        arg.codes[i] = p.codes; arg.scales[i] = p.scales; arg.ts[i] = p.ts; arg.y[i] = p.y; arg.n[i] = p.n; arg.ld_y[i] = p.ld_y; arg.e[i] = groups;
    }
    arg.sv0 = cfg.sv0; arg.sv1 = cfg.sv1; arg.k = k; arg.m = m; arg.chunk = (int)m; arg.a = a; arg.lb = cfg.lb;
    arg.waves = W;
    arg.partial = workspace;
    arg.slice_steps = per;
    constexpr uint32_t lds = W * ring_wave_bytes<NA, G, H, false>();
    static_assert(lds + kRingTableBytes <= kLdsBytes, "LDS");
    auto kern = sliced_ring_kernel<NA, G, GB, 0, W>;
    RAZER_RAISE_LDS_LIMIT(kern, lds);
    launch(kern, dim3((groups + G - 1) / G, 1, (unsigned)slices), 64 * W, lds, st, arg);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_slice_reduce(workspace, p.ts, nullptr, m, p.n, slices, p.y, p.ld_y, st);
}
// K-slices of one matrix of 33 .. 64 rows (0: none) and the groups of weight rows per workgroup with them.  Where the weight rows
// are few, a workgroup of one group (16 rows) reads all the activations for them, 64 x 11008 x 2 B = 1.4 MB at what a unit's
// load path takes, 50 bytes a clock; slices of K let it own two or four groups and read half or a quarter.  They cost the
// sums' way through the workspace and a second launch, 3.5 us (four groups 5.6).  Times as ring_estimate_us has them (16 waves, rows of 10240
// elements and more: 10 % more).  us, without -> with: 4096 x 11008 at 64
// rows 21.4 -> 18.3, at 40 18.6 -> 17.0, 2048 x 8192 14.8 -> 11.8, 13.2 -> 11.3, 1024 x 8192 14.6 -> 10.8, 1000 x 11008 at 40 17.7 -> 11.9,
// 5120 x 13824 (four groups) 27.1 -> 22.5; not taken: 4096 x 5120 at 64 rows 12.0, 12.1, 2048 x 4096 9.2, 10.2, 4096 x 8192 at 40 13.7, 14.2.
// Not up to 32 rows, where callers have the promise that nothing is written to the workspace.
static double ring_sum_us(int64_t k, int64_t m, int64_t rounds, int g)
{
    const double row = k % 64 == 0 ? 0.0074 : 0.0131;
    return 1e-3 * (double)(k * rounds) * (0.27 + row * (double)m + 0.52 * g);
}
static int ring_slices(int64_t n, int64_t k, int64_t m, int g, size_t workspace_bytes, int& groups_each)
{
    const int64_t steps = (k + 127) / 128, groups = (n + 15) / 16, wgs = (groups + g - 1) / g;
    const double whole = (5.1 + ring_sum_us(k, m, (wgs + kComputeUnits - 1) / kComputeUnits, g)) * (g == 1 && k >= 10240 ? 1.1 : 1.0);
    int best = 0;
    double us = 0.98 * whole;
    for (int sg = 2; sg <= 4; sg += 2) {
        int64_t s = kComputeUnits / ((groups + sg - 1) / sg);
        for (s = s < 8 ? s : 8; s >= 2; --s) {                        // every slice has a step for each wave
            const int64_t per = (steps + s - 1) / s;
            if (per >= kRingWaves && steps - (s - 1) * per >= kRingWaves && (size_t)(s * m * n) * sizeof(float) <= workspace_bytes) break;
        }
        if (s < 2) continue;
        const double sliced = (sg == 2 ? 8.6 : 10.7) + ring_sum_us(k, m, 1, sg) / (double)s;
        if (sliced < us) { us = sliced; best = (int)s; groups_each = sg; }
    }
    return best;
}

static hipError_t launch_ring(SvConfig cfg, int count, const GemvProblem* p, int64_t k, const uint16_t* a, int64_t m, float* workspace, size_t workspace_bytes, hipStream_t st)
{
    int g = ring_groups(ring_row_groups(count, p), m, cfg.f16 != 0);
    int64_t rows = 0;
    for (int i = 0; i < count; ++i) rows += p[i].n;
    // the launch shape on record, a family of 5 rows and more; any forced shape that does not ask for 16 waves keeps 8, so
    // that it stands for one order of the sum whatever the number of rows
    TuneShape t{{0, 0, 0, 0}, 0};
    if (m > kGemvDirectMaxM) t = tuned_shape(kTuneSmallBatch, m, rows, k);
    const bool shaped = t.source && t.p[0] == 2;
    if (shaped && (t.p[1] == 1 || t.p[1] == 2 || t.p[1] == 3 || (t.p[1] == 4 && !(m > 32 && cfg.f16)) || (t.p[1] == 6 && m <= 32))) g = t.p[1];
    const int asked = shaped && t.p[2] ? (t.p[2] == 16 ? 16 : 8) : t.source == 1 ? 8 : 0;
    if (count == 1 && !cfg.f16 && !cfg.il && m > kSkinnyMaxM && m <= kRingMaxM && !t.source && workspace) {
        int sg = 0;
        const int slices = ring_slices(p[0].n, k, m, g, workspace_bytes, sg);
#define RAZER_RING_SLICES(G)                                                                                             \
    (cfg.lb == 4 ? launch_ring_slices<G, false>(cfg, p[0], k, a, m, slices, workspace, st)                              \
                 : launch_ring_slices<G, true>(cfg, p[0], k, a, m, slices, workspace, st))
        if (slices) return sg == 4 ? RAZER_RING_SLICES(4) : RAZER_RING_SLICES(2);
#undef RAZER_RING_SLICES
    }
#define RAZER_RING(NA, G)                                                                  \
    do {                                                                                   \
        if (cfg.f16) return launch_ring_t<NA, G, false, 1>(cfg, count, p, k, a, m, asked, st);    \
        if (cfg.lb == 4) return launch_ring_t<NA, G, false, 0>(cfg, count, p, k, a, m, asked, st); \
        return launch_ring_t<NA, G, true, 0>(cfg, count, p, k, a, m, asked, st);                  \
    } while (0)
#define RAZER_RING_G(NA)                   \
    do {                                   \
        if (g == 1) RAZER_RING(NA, 1);     \
        if (g == 2) RAZER_RING(NA, 2);     \
        if (g == 3) RAZER_RING(NA, 3);     \
        if (g == 4) RAZER_RING(NA, 4);     \
        RAZER_RING(NA, 6);                 \
    } while (0)
    if (m <= 4 && cfg.il) {                                       // the interleaved layout is a form of 2..4 rows
        if (g == 1) return launch_ring_t<1, 1, false, 0, true>(cfg, count, p, k, a, m, asked, st);
        if (g == 2) return launch_ring_t<1, 2, false, 0, true>(cfg, count, p, k, a, m, asked, st);
        if (g == 3) return launch_ring_t<1, 3, false, 0, true>(cfg, count, p, k, a, m, asked, st);
        if (g == 4) return launch_ring_t<1, 4, false, 0, true>(cfg, count, p, k, a, m, asked, st);
        return launch_ring_t<1, 6, false, 0, true>(cfg, count, p, k, a, m, asked, st);
    }
    if (cfg.il) return hipErrorInvalidValue;
    if (m <= 4) RAZER_RING_G(1);
    if (m <= 8) RAZER_RING_G(2);
    if (m <= 16) RAZER_RING_G(4);
    if (m <= 32) RAZER_RING_G(8);
    if (g == 1) RAZER_RING(16, 1);
    if (g == 2) RAZER_RING(16, 2);
    if (g == 3) RAZER_RING(16, 3);
    return cfg.lb == 4 ? launch_ring_t<16, 4, false, 0>(cfg, count, p, k, a, m, asked, st) : launch_ring_t<16, 4, true, 0>(cfg, count, p, k, a, m, asked, st);
#undef RAZER_RING_G
#undef RAZER_RING
}

// Where this kernel takes over from its neighbours (unless a tuner or test forces one of their launch shapes).
// 33..64 activation rows, scale-byte format, against the K-sliced register-decode GEMM: except where one group per
// workgroup makes every workgroup read more activations than it gains: one group and m x K above 600 thousand; from 161
// groups on the length of K decides, whatever the number of rows.  The lines were drawn for whole K (1500 x 12288 at 64 rows
// 21.4 us on the GEMM, 21.9 here; 2600 weight rows at 64 rows 0.95 of the GEMM's time with 12288 elements, 1.04 with 14336;
// 3200 0.91, 1.01; 4096 at 56 rows 0.90, 0.97 and with 16384 1.02) and still hold for groups of matrices.  With the K-slices of
// one matrix (ring_slices), which this rule does not ask, they lie too low: 1500 x 12288 at 64 rows 20.8 on the GEMM, 12.4
// here, 1000 x 16384 21.8, 12.6, 2600 x 14336 25.0, 17.1, 4096 x 16384 at 56 rows 33.0, 22.5.
// 2..4 activation rows, against the 4x4x4 kernel of razer_gemv.hip, whose waves cross all of K in one or two passes:
// long rows and not too many of them (1024 groups) -- at 4 rows 8192 x 28672 38.4 -> 31.0 us, {q,k,v} 10240 x 8192
// 16.5 -> 14.5, 2 x 3000 x 6144 9.8 -> 8.2; at 2 rows one group per workgroup only (4096 x 11008 9.4 -> 7.8; but
// 10240 x 8192 13.9 -> 14.4) -- and 4 rows with one group per workgroup from 2048 elements up (4096 x 4096
// 5.30 -> 4.97).  Beyond the lines, as both kernels are now: 57344 x 8192 at 4 rows 58.0, here 56.9; 2 x 11008 x 4096 at 3 and
// 4 rows 14.0, 14.6 and 14.5, 14.7; but 3 x 4096 x 4096 9.0, 8.7 and 9.7, 8.7, which is not taken yet.
// Above 64 rows, scale bytes, against the register-decode and the tiled GEMM: whichever of two estimates is the shorter.
// Where the two meet depends on how well either fills the chip -- K-slices and the width of tiles there, groups per
// workgroup and rounds of workgroups here -- so that no bound on sizes follows it: over 420 calls of 65 .. 2048 rows that
// nothing was fitted to the choice is 0.43 % (geometric mean) behind the faster kernel and at most 1.26 times its time (108 x
// 2 x 36 x 8480 16.5 us, 13.1 here); limits on units, units x K
// and K were 1.6 to 8 % behind it and up to 2.9 times.  GEMM -> this (us): 4096 x 4096 at 512 rows 40.4 -> 29.8, 2 x 5120 x
// 5120 at 320 88 -> 64, 1139 x 5376 at 1249 55.6 -> 32.8, 1000 x 28672 at 256 67.7 -> 51.1, 2865 x 8832 at 380 62.2 -> 43.9,
// 5539 x 1536 at 1390 (rows that the GEMM stores an element at a time) 83.8 -> 57.6; not taken 100 x 24576 at 128 rows 25.6
// -> 41.2, 3000 x 28672 at 128 50.0 -> 65.6, 720 x 15104 at 1445 59.8 -> 88.3, 10352 x 1216 at 438 25.4 -> 34.9, 130 x 21696
// at 1514 60.5 -> 84.7.
// FP16 scales, whose GEMM multiplies every block apart and has one launch per matrix: 8.5 million units (a group of 16
// weight rows times a run of up to 64 activation rows) x K per matrix.  28672 x 8192 at 128 rows 237 -> 114; 4096 x 4096 at
// 512 rows (8.4) 41.0 -> 34.2; 4096 x 11008 at 192 rows (8.4) 42.7 -> 41.8; 8192 x 8192 at 160 rows (12.6) 52.0 -> 53.7;
// 2 x 11008 x 4096 at 192 rows (8.5) 103 -> 69; 3 x 4096 x 4096 at 512 rows (8.4) 122 -> 90.
// This kernel scales its operands; a special value of 9.5 times a block scale does not always fit a bf16, which the
// 4x4x4 kernel (bare operands) does not need, so up to 4 rows such tensors stay there.  The layout of the weights has
// no say: canonical and interleaved tensors give the same bits.
bool ring_serves(SvConfig cfg, int count, const GemvProblem* p, int64_t k, int64_t m)
{
    if (k > kSkinnyMaxK) return false;
    int64_t rows = 0;
    for (int i = 0; i < count; ++i) rows += p[i].n;
    const int64_t groups = ring_row_groups(count, p);
    if (m >= 2 && m <= kGemvDirectMaxM) {
        if (!cfg.f16 && (cfg.sv0 == 9.5f || cfg.sv1 == 9.5f)) return false;
        if (groups <= kComputeUnits ? k < (m == 2 ? 8192 : m == 3 ? 6144 : 2048) : m == 2 || k < 6144 || groups > 1024) return false;
        return tuned_shape(kTuneGemvQuad, m, rows, k).source != 1 && tuned_shape(kTuneGemv, m, rows, k).source != 1;
    }
    if (m > kRingMaxM) {
        if (!cfg.f16 && tuned_shape(kTuneGemmSlices, m, rows, k).source == 1) return false;
        if (cfg.f16) {
            const int64_t units = (m + kRingMaxM - 1) / kRingMaxM * groups;
            return m <= 128 || (units <= 2500 * count && units * k <= (int64_t)8500000 * count);
        }
        return k <= kRbMaxK && ring_estimate_us(count, p, k, m) <= gemm_estimate_us(count, p, m, k);
    }
    if (m <= kSkinnyMaxM || cfg.f16) return false;
    if (tuned_shape(kTuneGemmSlices, m, rows, k).source == 1) return false;
    return ring_groups(groups, m, false) > 1 || m * k <= 600000 || (groups > 160 && k <= (groups > 208 ? 14336 : 12288));
}

// What razer_workspace_bytes reports for 5..32 activation rows.  The kernel above writes nothing there; callers size and pass
// what these functions have always asked for, and a smaller workspace is refused as before, so the rule stays: the
// K-slices of 512 or 1024 elements ([slices][m][rows] fp32) unless the launch shape on record keeps K inside the
// workgroup.
static bool ws_free_shape(int s, int g) { return (s == 1 && g >= 1 && g <= 4) || (s == 2 && ((g >= 1 && g <= 4) || g == 8)); }
// some G <= 4 groups of 16 rows per workgroup make one round of workgroups that covers half of the compute units
static bool ws_one_round(int64_t rows, int count, int64_t k, int64_t m)
{
    if (m > 16 || k > 16384 || (k > 8192 && m > 8)) return false;
    const int64_t groups = (rows + 15) / 16;
    for (int g = 1; g <= 4; ++g) {
        const int64_t wgs = (groups + g - 1) / g + (count - 1);
        if (wgs <= kComputeUnits) return wgs >= kComputeUnits / 2;
    }
    return false;
}
static size_t ws_bytes(int64_t rows, int64_t k, int64_t m, int count)
{
    int64_t steps = (m <= 16 && k > 8192) ? 8 : 4;
    const TuneShape t = tuned_shape(kTuneSmallBatch, m, rows, k);
    if (t.source && t.p[0] == 1 && m <= 16 && ws_free_shape(t.p[1], t.p[2])) return 0;
    if (t.source && t.p[0] == 0 && (t.p[1] == 4 || (t.p[1] == 8 && m <= 16)) && (t.p[2] == 1 || t.p[2] == 2 || t.p[2] == 4)) steps = t.p[1];
    else if (ws_one_round(rows, count, k, m)) return 0;
    const int64_t nslices = (k + 128 * steps - 1) / (128 * steps);
    return nslices > 1 ? (size_t)(nslices * m * rows) * sizeof(float) : 0;
}
size_t skinny_workspace_bytes(int64_t n, int64_t k, int64_t m)
{
    if (m <= kGemvDirectMaxM || m > kSkinnyMaxM || k == 0 || k > kSkinnyMaxK) return 0;
    return ws_bytes(n, k, m, 1);
}
size_t skinny_grouped_workspace_bytes(int count, const GemvProblem* p, int64_t k, int64_t m)
{
    if (m <= kGemvDirectMaxM || m > kSkinnyMaxM || k == 0 || k > kSkinnyMaxK) return 0;
    int64_t rows = 0;
    for (int i = 0; i < count; ++i) rows += p[i].n;
    return ws_bytes(rows, k, m, count);
}

hipError_t launch_skinny(SvConfig cfg, int count, const GemvProblem* p, int64_t k, const uint16_t* a, int64_t m, hipStream_t st,
                         float* workspace, size_t workspace_bytes)
{
    if (count < 1 || count > 4 || m < 2 || k <= 0 || k > kSkinnyMaxK) return hipErrorInvalidValue;
    for (int i = 0; i < count; ++i)
        if (p[i].n <= 0) return hipErrorInvalidValue;
    return launch_ring(cfg, count, p, k, a, m, workspace, workspace_bytes, st);
}


// ---------------------------------------------------------------------------------------------
// y[m][n] = bf16(scale * sum over slices, in slice order, of partial[slice][m][n]); scale = -ts_w
// (weight-only: the decode carries a global negation) or ts_w * ts_a (both operands decoded).
// VEC = 4: four consecutive columns per thread (n and ld_y multiples of 4).
template <int VEC>
__global__ __launch_bounds__(256) void slice_reduce_kernel(const float* __restrict__ partial,
                                                           const float* __restrict__ w_ts,
                                                           const float* __restrict__ a_ts, int64_t m, int64_t n,
                                                           int nslices, uint16_t* __restrict__ y, int64_t ld_y)
{
    asm volatile("" ::"s"(partial), "s"(w_ts), "s"(a_ts), "s"(m), "s"(n), "s"(nslices), "s"(y), "s"(ld_y));   // (all arguments in one wait)
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * VEC;
    if (i >= m * n) return;
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    if (VEC == 4) {
        for (int s = 0; s < nslices; ++s) {
            const float4 p = *reinterpret_cast<const float4*>(partial + (int64_t)s * m * n + i);
            t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
        }
    }
    const float scale = a_ts ? (*w_ts) * (*a_ts) : -(*w_ts);
    // Small sums are bound by one thread's chain: 64-bit division (32 bits hold nearly every call), arguments, tensor scale
    // ahead of the loads (4096 x 11008 at 64 rows, two slices: 18.09 -> 17.86 us with the main kernel, 2048 x 8192 11.71 -> 11.35)
    const int64_t r = m * n <= 0xFFFFFFFF ? (int64_t)((uint32_t)i / (uint32_t)n) : i / n, c = i - r * n;
    if (VEC == 4) {
        const uint32_t lo = (uint32_t)f32_to_bf16_rne(scale * t.x) | ((uint32_t)f32_to_bf16_rne(scale * t.y) << 16);
        const uint32_t hi = (uint32_t)f32_to_bf16_rne(scale * t.z) | ((uint32_t)f32_to_bf16_rne(scale * t.w) << 16);
        *reinterpret_cast<uint2*>(y + r * ld_y + c) = make_uint2(lo, hi);
    } else {
        for (int s = 0; s < nslices; ++s) t.x += partial[(int64_t)s * m * n + i];
        y[r * ld_y + c] = f32_to_bf16_rne(scale * t.x);
    }
}

hipError_t launch_slice_reduce(const float* partial, const float* w_ts, const float* a_ts, int64_t m, int64_t n,
                               int nslices, uint16_t* y, int64_t ld_y, hipStream_t st)
{
    const int64_t total = m * n;
    if (n % 4 == 0 && ld_y % 4 == 0 && (reinterpret_cast<uintptr_t>(y) & 7u) == 0)
        launch(slice_reduce_kernel<4>, (unsigned)((total / 4 + 255) / 256), 256, 0, st, partial, w_ts, a_ts, m, n, nslices, y, ld_y);
    else
        launch(slice_reduce_kernel<1>, (unsigned)((total + 255) / 256), 256, 0, st, partial, w_ts, a_ts, m, n, nslices, y, ld_y);
    return hipGetLastError();
}

// The same reduction for the matrices of a grouped launch: thread index space = the 4-column groups
// of matrix 0, then of matrix 1, ... (e1..e3 = first group of matrices 1..3; every n a multiple of 4).
__global__ __launch_bounds__(256) void slice_reduce_grouped_kernel(
    const float* __restrict__ partial, const float* f0, const float* f1, const float* f2, const float* f3,
    uint16_t* y0, uint16_t* y1, uint16_t* y2, uint16_t* y3, int64_t n0, int64_t n1, int64_t n2, int64_t n3,
    int64_t l0, int64_t l1, int64_t l2, int64_t l3, int64_t e1, int64_t e2, int64_t e3, int64_t e4, int64_t m,
    int nslices)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= e4) return;
    const float* ts = f0; uint16_t* y = y0;
    int64_t n = n0, ld = l0, first = 0, before = 0;
    if (g >= e1) { ts = f1; y = y1; n = n1; ld = l1; first = e1; before = n0; }
    if (g >= e2) { ts = f2; y = y2; n = n2; ld = l2; first = e2; before = n0 + n1; }
    if (g >= e3) { ts = f3; y = y3; n = n3; ld = l3; first = e3; before = n0 + n1 + n2; }
    const int64_t i = (g - first) * 4;
    const int64_t r = i / n, c = i - r * n;
    const float* src = partial + (int64_t)nslices * m * before + i;
    const float scale = -(*ts);
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s = 0; s < nslices; ++s) {
        const float4 p = *reinterpret_cast<const float4*>(src + (int64_t)s * m * n);
        t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
    }
    const uint32_t lo = (uint32_t)f32_to_bf16_rne(scale * t.x) | ((uint32_t)f32_to_bf16_rne(scale * t.y) << 16);
    const uint32_t hi = (uint32_t)f32_to_bf16_rne(scale * t.z) | ((uint32_t)f32_to_bf16_rne(scale * t.w) << 16);
    *reinterpret_cast<uint2*>(y + r * ld + c) = make_uint2(lo, hi);      // y 8-byte aligned, ld a multiple of 4
}

// partial: matrix i's [nslices][m][n_i] fp32 slices behind those of matrices 0 .. i-1.  Every n a
// positive multiple of 4, every y 8-byte aligned, every ld_y a multiple of 4.
hipError_t launch_slice_reduce_grouped(const float* partial, int count, const GemvProblem* p, int64_t m, int nslices,
                                       hipStream_t st)
{
    GemvProblem q[4];
    int64_t e[5] = {0, 0, 0, 0, 0};
    for (int i = 0; i < 4; ++i) {
        q[i] = p[i < count ? i : count - 1];
        e[i + 1] = e[i] + (i < count ? m * q[i].n / 4 : 0);
    }
    launch(slice_reduce_grouped_kernel, (unsigned)((e[4] + 255) / 256), 256, 0, st, partial, q[0].ts, q[1].ts, q[2].ts, q[3].ts, q[0].y, q[1].y, q[2].y, q[3].y, q[0].n, q[1].n, q[2].n, q[3].n,
        q[0].ld_y, q[1].ld_y, q[2].ld_y, q[3].ld_y, e[1], e[2], e[3], e[4], m, nslices);
    return hipGetLastError();
}

}  // namespace razer
