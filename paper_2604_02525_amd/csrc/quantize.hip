// Fused residual masking -> block Hadamard transform -> OCP-MX FP4 quantisation (gfx950).
//
// What is computed (paper Eq. 5 applied to one operand, App. F items 1-2): for every row of the
// logical [outer, K] operand, entries flagged by the masks become 0, every block of B consecutive
// K-elements is multiplied by the normalised Sylvester Hadamard matrix, and every 32 consecutive
// K-elements are quantised to E2M1 with one shared E8M0 scale.
//
// Numerics are fixed so that the packed bytes are reproducible: fp32 butterflies in ascending
// stride order (x+y to the lower index, x-y to the upper), one fp32 multiply by (float)(1/sqrt(B)),
// amax on those fp32 values, scale = biased exponent of amax minus 2, round-to-nearest-even to E2M1
// with saturation at 6; a transformed value that is exactly zero is stored as +0.  The file is
// compiled with -ffp-contract=off.
//
// One kernel per storage order of the operand (k_quant_kc16, k_quant_ks16, for every K % 32 == 0) and a variant of the
// first that also copies the extracted K-channels out; what bounds them and how the work is split stands at each.
#include "common.h"
#include "foid_topk.h"
#include "gemm_mx_common.h"

#include <type_traits>

namespace adahop {

namespace {

__device__ __forceinline__ int e8m0_of_amax(float amax)
{
    int e = (int)((__float_as_uint(amax) >> 23) & 0xffu);
    int s = e - 2;
    return s < 0 ? 0 : s; // zero and subnormal amax -> 0
}

// ---- optional stochastic rounding of the elements (the paper cites it as prior work for unbiased
// gradient quantisation).  Random bits: Philox4x32 with 10 rounds (Salmon et al., SC'11), key = the two
// halves of the caller's seed, counter = (row, K index / 8, 0, 0): one block serves the 8 consecutive
// K-elements of a group, element j taking half j (word j / 2, low half for even j).
struct sr_key_t {
    uint32_t k0, k1;
};

// One instruction each, by its truth table, where the compiler makes two: the kernel with stochastic rounding is bound by its vector
// instructions (825 -> 779 in all; the input gradient 8192 x 4096 x 11008 with rounded gradients 263.4 -> 259.4 us).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, (int)c, 0x96);
}

// The bits of a under mask, those of b elsewhere.
__device__ __forceinline__ uint32_t insert_bits(uint32_t mask, uint32_t a, uint32_t b)
{
    return (uint32_t)__builtin_amdgcn_bitop3_b32((int)mask, (int)a, (int)b, 0xCA);
}

__device__ __forceinline__ uint4 philox4x32_10(uint32_t c0, uint32_t c1, sr_key_t key)
{
    uint32_t c2 = 0, c3 = 0, k0 = key.k0, k1 = key.k1;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        // both halves of a product from one instruction (the two 32-bit multiplies cost a quarter-rate slot each)
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        c0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        c1 = (uint32_t)p1;
        c2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return make_uint4(c0, c1, c2, c3);
}

// E2M1 code of v / 2^(s-127) rounded stochastically with the 16-bit draw r: up to the next magnitude iff
// r / 65536 < (|q| - lo) / (hi - lo); |q| >= 6 saturates; the sign bit of v is kept.  The code lies in bits 16 .. 19 of the result.
//
// Code plus fraction as one number is f(a) = idx + frac = min(2 a, a + 2, a / 2 + 4, 7), the magnitudes' steps of 1/2, 1, 2 being
// a concave line, and "up iff r / 65536 < frac" is code = ceil(f(a) - r / 65536) = floor((F - r + 65535) / 65536) with
// F = ceil(65536 f(a)).  With G = ceil(2^17 a) a whole number of at most 2^20, the four lines in G are exact in fp32 (a quarter is
// the finest fraction; + 65535.75 rounds up to whole numbers under the truncating conversion), so every decision is the
// one that real arithmetic makes.  Nine instructions per element in place of about 25 (six compares, a selected
// step and draw); with the generator's products taken whole, 8192 x 11008 takes 155 -> 82 us (46 rounded to nearest even),
// K-strided 118 -> 73.  inv = 2^(127-s) (its product with 2^17 may exceed the range of fp32).
__device__ __forceinline__ uint32_t e2m1_bits16_sr(float v, float inv, uint32_t r)
{
    const float G = __builtin_ceilf(fabsf(v) * inv * 0x1p17f);
    const float f1 = G + 65535.75f, f2 = __builtin_fmaf(G, 0.5f, 131072.0f + 65535.75f), f3 = __builtin_fmaf(G, 0.25f, 262144.0f + 65535.75f);
    // (the median of three in place of a fourth minimum: an element that is no number gets code 0, for the same instructions)
    const float F = __builtin_amdgcn_fmed3f(fminf(fminf(f1, f2), f3), 65535.75f, 458752.0f + 65535.75f);
    return insert_bits(0x80000u, __float_as_uint(v) >> 12, (uint32_t)F - r);
}

// Packed codes of 8 consecutive K-elements (first in the low nibble) starting at K index kk of row `row`.
__device__ __forceinline__ uint32_t pack8_sr(const float (&w)[8], int s, sr_key_t key, int64_t row, int64_t kk)
{
    const uint4 r = philox4x32_10((uint32_t)row, (uint32_t)(kk >> 3), key);
    const uint32_t word[4] = {r.x, r.y, r.z, r.w};
    const float inv = __uint_as_float((uint32_t)(254 - s) << 23); // s <= 253 (amax finite)
    uint32_t pair[4]; // byte 2: two codes
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t lo = e2m1_bits16_sr(w[2 * i], inv, word[i] & 0xffffu), hi = e2m1_bits16_sr(w[2 * i + 1], inv, word[i] >> 16);
        pair[i] = insert_bits(0x0fffffu, lo, hi << 4); // (the other bytes go nowhere)
    }
    const uint32_t p01 = __builtin_amdgcn_perm(pair[1], pair[0], 0x0c0c0602u), p23 = __builtin_amdgcn_perm(pair[3], pair[2], 0x06020c0cu);
    return p01 | p23;
}

template <int B> __device__ __forceinline__ float hadamard_norm();
template <> __device__ __forceinline__ float hadamard_norm<0>() { return 1.0f; }
template <> __device__ __forceinline__ float hadamard_norm<32>() { return 0x1.6a09e6p-3f; }
template <> __device__ __forceinline__ float hadamard_norm<64>() { return 0.125f; }
template <> __device__ __forceinline__ float hadamard_norm<128>() { return 0x1.6a09e6p-4f; }
template <> __device__ __forceinline__ float hadamard_norm<256>() { return 0.0625f; }

// ================================================================================================
// Both quantisers are bound by vector-ALU work long before HBM unless the per-element instruction count is kept
// near 12, so these kernels
//   - let the hardware convert: v_cvt_scalef32_pk_fp4_f32 rounds two fp32 values / 2^(s-127) to E2M1
//     (nearest even, saturating, first value in the low nibble) in one instruction;
//   - do every cross-lane butterfly as ONE fused multiply-add whose first operand comes through DPP:
//     w <- partner * t + w with t = +1 on the lower lane of the pair and -1 on the upper one.  That
//     yields L+U on the lower lane and -(L-U) on the upper lane; the stray sign is not fixed up but
//     tracked (it only depends on the lane) and folded into the final 1/sqrt(B) multiply.  Negation
//     commutes with rounding, so the stored bits are exactly those of the plain butterflies.
//
// Rows are cut into units of 256 K-elements; K need only be a multiple of 32: the lanes past the end of a row's last,
// shorter unit hold zeros and store nothing (no transform block reaches across that end, because K is a multiple of
// the block).  On [5000][3040] bf16 that takes 13.7 us, against 17.6 us for a kernel of its own with eight elements per lane
// and the conversion in compares, and on K-strided [2016][11008] 17.2 against 26.2 us.
//
// Work split: 16 lanes (one DPP row) own 256 consecutive K-elements of one row; a lane holds two
// groups of 8 consecutive elements, 128 apart (chunk c of each half).  Strides 1, 2, 4 are register
// butterflies inside a group, strides 8..64 pair lanes, stride 128 pairs the lane's two groups.  A
// gfx9 DPP row offers the lane exchanges xor 1, xor 2 (quad_perm), xor 7 (row_half_mirror) and xor 8
// (row_ror:8) but not xor 4, so chunk c sits on lane (c0 ^ c2, c1 ^ c2, c2, c3): flipping chunk bit 2
// then is the xor-7 exchange.
// ================================================================================================
template <int CTRL> __device__ __forceinline__ float dpp_get(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

struct lane_plan_t {
    int chunk;     // which 8-element chunk (0..15) of each 128-element half this lane owns
    float t[4];    // multiplier of the partner value in cross-lane stage b
    float fin;     // sign left over from the stages times 1/sqrt(B)
};

template <int B> __device__ __forceinline__ lane_plan_t make_plan(int lane)
{
    constexpr int NS = B >= 128 ? 4 : (B == 64 ? 3 : (B == 32 ? 2 : 0));
    const int r = lane & 15;
    lane_plan_t p;
    p.chunk = r ^ ((r << 29 >> 31) & 3); // chunk bit 2 set: the two below it flipped
    p.fin = B > 0 ? hadamard_norm<B>() : 1.0f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        p.t[b] = b < NS ? __uint_as_float(((uint32_t)p.chunk << (31 - b) & 0x80000000u) | 0x3f800000u) : 1.0f;
        if (b < NS) p.fin *= p.t[b];
    }
    return p;
}

// One cross-lane butterfly stage on all 16 values of the lane: w <- partner(w) * t + w, the partner
// being the lane of the DPP row whose chunk index differs in bit STAGE.  Written as assembly because
// the compiler does not fold the DPP move into the multiply-add (it emits a move, wait states and a
// separate v_fmac per value, doubling the cost of the stage).  The leading s_nop covers the two wait
// states a DPP read needs after a vector write of the same register; inside the block each
// instruction reads a register last written 16 instructions earlier.
#define ADAHOP_FMAC_DPP16(CTRL)                                                                        \
    asm volatile("s_nop 1\n\t"                                                                        \
                 "v_fmac_f32_dpp %0, %0, %16 " CTRL "\n\tv_fmac_f32_dpp %1, %1, %16 " CTRL "\n\t"     \
                 "v_fmac_f32_dpp %2, %2, %16 " CTRL "\n\tv_fmac_f32_dpp %3, %3, %16 " CTRL "\n\t"     \
                 "v_fmac_f32_dpp %4, %4, %16 " CTRL "\n\tv_fmac_f32_dpp %5, %5, %16 " CTRL "\n\t"     \
                 "v_fmac_f32_dpp %6, %6, %16 " CTRL "\n\tv_fmac_f32_dpp %7, %7, %16 " CTRL "\n\t"     \
                 "v_fmac_f32_dpp %8, %8, %16 " CTRL "\n\tv_fmac_f32_dpp %9, %9, %16 " CTRL "\n\t"     \
                 "v_fmac_f32_dpp %10, %10, %16 " CTRL "\n\tv_fmac_f32_dpp %11, %11, %16 " CTRL "\n\t" \
                 "v_fmac_f32_dpp %12, %12, %16 " CTRL "\n\tv_fmac_f32_dpp %13, %13, %16 " CTRL "\n\t" \
                 "v_fmac_f32_dpp %14, %14, %16 " CTRL "\n\tv_fmac_f32_dpp %15, %15, %16 " CTRL "\n\t" \
                 "s_nop 1"                                                                            \
                 : "+v"(w0[0]), "+v"(w0[1]), "+v"(w0[2]), "+v"(w0[3]), "+v"(w0[4]), "+v"(w0[5]), "+v"(w0[6]),   \
                   "+v"(w0[7]), "+v"(w1[0]), "+v"(w1[1]), "+v"(w1[2]), "+v"(w1[3]), "+v"(w1[4]), "+v"(w1[5]),   \
                   "+v"(w1[6]), "+v"(w1[7])                                                            \
                 : "v"(t))

template <int STAGE> __device__ __forceinline__ void cross_stage(float (&w0)[8], float (&w1)[8], float t)
{
    if constexpr (STAGE == 0)
        ADAHOP_FMAC_DPP16("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf");
    else if constexpr (STAGE == 1)
        ADAHOP_FMAC_DPP16("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf");
    else if constexpr (STAGE == 2)
        ADAHOP_FMAC_DPP16("row_half_mirror row_mask:0xf bank_mask:0xf");
    else
        ADAHOP_FMAC_DPP16("row_ror:8 row_mask:0xf bank_mask:0xf");
}

// Transform (B > 0) and quantise the lane's two groups; returns the packed codes of each group and
// the scale code of the MX block each group belongs to (identical on the 4 lanes of the block).
// SR: elements rounded stochastically; the groups start at K indices kk0 and kk1 of row `row`.
template <int B, bool SR>
__device__ __forceinline__ void transform_quantize16(float (&w0)[8], float (&w1)[8], const lane_plan_t &p,
                                                     uint32_t &codes0, uint32_t &codes1, int &s0, int &s1,
                                                     sr_key_t key, int64_t row, int64_t kk0, int64_t kk1)
{
    if constexpr (B > 0) {
#pragma unroll
        for (int h = 1; h < 8; h *= 2)
#pragma unroll
            for (int i = 0; i < 8; i += 2 * h)
#pragma unroll
                for (int j = i; j < i + h; ++j) {
                    float a = w0[j], b = w0[j + h];
                    w0[j] = a + b;
                    w0[j + h] = a - b;
                    a = w1[j], b = w1[j + h];
                    w1[j] = a + b;
                    w1[j + h] = a - b;
                }
        cross_stage<0>(w0, w1, p.t[0]);                        // stride 8: chunk bit 0
        cross_stage<1>(w0, w1, p.t[1]);                        // stride 16: chunk bit 1
        if constexpr (B >= 64) cross_stage<2>(w0, w1, p.t[2]); // stride 32: chunk bit 2
        if constexpr (B >= 128) cross_stage<3>(w0, w1, p.t[3]); // stride 64: chunk bit 3
        if constexpr (B == 256) {
#pragma unroll
            for (int i = 0; i < 8; ++i) { // stride 128: the lane's two groups (same leftover sign)
                const float a = w0[i], b = w1[i];
                w0[i] = a + b;
                w1[i] = a - b;
            }
        }
        // the "+ 0" turns an exactly zero result into +0 whatever sign the lane carries (and changes
        // nothing else): transformed zeros are stored unsigned
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            w0[i] = __builtin_fmaf(w0[i], p.fin, 0.0f);
            w1[i] = __builtin_fmaf(w1[i], p.fin, 0.0f);
        }
    }
    float m0 = 0.0f, m1 = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        m0 = fmaxf(m0, fabsf(w0[i]));
        m1 = fmaxf(m1, fabsf(w1[i]));
    }
    m0 = fmaxf(m0, dpp_get<0xB1>(m0)); // the MX block = chunks 4q..4q+3 = the lane's quad
    m1 = fmaxf(m1, dpp_get<0xB1>(m1));
    m0 = fmaxf(m0, dpp_get<0x4E>(m0));
    m1 = fmaxf(m1, dpp_get<0x4E>(m1));
    s0 = e8m0_of_amax(m0);
    s1 = e8m0_of_amax(m1);
    if constexpr (SR) {
        codes0 = pack8_sr(w0, s0, key, row, kk0);
        codes1 = pack8_sr(w1, s1, key, row, kk1);
        return;
    }
    const float x0 = __uint_as_float((uint32_t)s0 << 23), x1 = __uint_as_float((uint32_t)s1 << 23);
    codes0 = __float_as_uint(w0[0]); // (every byte is written: any register that is free)
    codes1 = __float_as_uint(w1[0]);
    codes0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes0, w0[0], w0[1], x0, 0);
    codes0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes0, w0[2], w0[3], x0, 1);
    codes0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes0, w0[4], w0[5], x0, 2);
    codes0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes0, w0[6], w0[7], x0, 3);
    codes1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes1, w1[0], w1[1], x1, 0);
    codes1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes1, w1[2], w1[3], x1, 1);
    codes1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes1, w1[4], w1[5], x1, 2);
    codes1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes1, w1[6], w1[7], x1, 3);
}

__device__ __forceinline__ void apply_k_mask(float (&w)[8], uint64_t zm)
{
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if ((zm >> (8 * i)) & 0xffu) w[i] = 0.0f;
}

// Slot of MX block j (0 .. 7) of unit u in the stage-major copy of the scales: the last unit of a row holds
// t = K / 32 - 8 u blocks if K is no multiple of 256, and the tiled GEMM kernels read that stage so that it ends with the
// row (see there): its blocks then are the last t of 8, and the slots before them, which stand for blocks that the
// stage before has already used, hold scale 0.  Rotating by 8 - t puts the zeros of the missing blocks there.
__device__ __forceinline__ int tail_rotation(int64_t K, int64_t k0)
{
    const int64_t left = (K - k0) >> 5;
    return left < 8 ? 8 - (int)left : 0;
}

// k0: start of the lane group's 256 K-elements (a multiple of 256); in0 / in1: the lane's chunk of the first / second
// half lies inside the row.  sm: optional second copy of the scales in the order the tiled GEMM kernels read them,
// [ceil(K/256)][sm.rows][8].
template <bool TAIL>
__device__ __forceinline__ void store_codes_scales(uint8_t *codes, uint8_t *scales, int64_t row, int64_t K, int64_t k0,
                                                   int chunk, bool in0, bool in1, uint32_t c0, uint32_t c1, int s0, int s1,
                                                   scales_sm_t sm)
{
    uint8_t *crow = codes + row * (K >> 1) + ((k0 + chunk * 8) >> 1);
    if (!TAIL || in0) *reinterpret_cast<uint32_t *>(crow) = c0;
    if (!TAIL || in1) *reinterpret_cast<uint32_t *>(crow + 64) = c1;
    if ((chunk & 3) == 0) {
        uint8_t *srow = scales + row * (K >> 5) + ((k0 + chunk * 8) >> 5);
        if (!TAIL || in0) srow[0] = (uint8_t)s0;
        if (!TAIL || in1) srow[4] = (uint8_t)s1;
        if (sm.out) {
            uint8_t *q = sm.out + ((k0 >> 8) * sm.rows + row) * 8;
            const int j = (chunk >> 2) + (TAIL ? tail_rotation(K, k0) : 0);
            q[j & 7] = (uint8_t)s0; // (0 where the block is missing)
            q[(j + 4) & 7] = (uint8_t)s1;
        }
    }
}

__device__ __forceinline__ uint32_t row_of_unit(uint32_t u, uint32_t upr, uint32_t magic)
{
    return upr == 1 ? u : __umulhi(u, magic); // u / upr, exact for u upr < 2^32
}

// The order of the workgroups of a K-strided operand (ks_order).
struct ks_order_t {
    uint32_t run, rest; // workgroups of an XCD (of the first `rest`: one more); run = 0: the order as it is
    uint32_t groups;    // whole groups of KS_GROUP column tiles
    uint32_t per_group, narrow, narrow_magic; // workgroups of a group; column tiles of a last, narrower one, ceil(2^32 / narrow)
    uint64_t magic;                           // ceil(2^44 / per_group): v / per_group is exact for v per_group < 2^44
};

// One operand's quantisation: what is read, which entries count as zero and where the results go.
struct quant_t {
    const uint16_t *x;
    int64_t outer, K, ld;
    const uint8_t *zero_outer, *zero_k;
    uint8_t *codes, *scales;
    sr_key_t key;
    scales_sm_t sm;
    k_gather_t gk;
    row_gather_t gr;
    uint32_t upr, magic;  // 256-element units per row (K-strided: K-blocks); ceil(2^32 / upr)
    uint32_t rows_per_wg; // of the kernel that copies K-channels
    uint32_t col_tiles;   // K-strided: workgroups along the outer index
    uint32_t gather_blocks; // K-strided: workgroups that copy K-channels out (a multiple of 8)
    ks_order_t order;
};

// K-contiguous operand: 16 lanes per 256 K-elements of a row, unit `unit` of row `row`.  TAIL: K % 256 != 0 (an instance of
// its own, because the conditions of a shorter last unit cost the others 2 %).
// An outer index that is extracted (q.gr) leaves the quantiser as it came, for the bf16 product of the extracted rows, and
// counts as zero here: the copy is made where the row is in registers anyway, in place of a launch that reads it again.
template <int B, bool SR, bool TAIL>
__device__ __forceinline__ void quant_kc_unit(const quant_t &q, int64_t row, uint32_t unit, bool active)
{
    const int64_t K = q.K;
    const lane_plan_t plan = make_plan<B>(threadIdx.x & 63);
    const int64_t k0 = (int64_t)unit * 256, kk = k0 + plan.chunk * 8;
    const bool in0 = active && (!TAIL || kk < K), in1 = active && (!TAIL || kk + 128 < K);

    uint4 r0 = make_uint4(0, 0, 0, 0), r1 = make_uint4(0, 0, 0, 0);
    if (active) { // the row's mask travels with the data (1 % of the rows are read for nothing) instead of ahead of it
        const uint16_t *src = q.x + row * q.ld + kk;
        if (!TAIL || in0) r0 = load_once16(src);
        if (!TAIL || in1) r1 = load_once16(src + 128);
        if (q.gr.out) {
            const uint32_t p = q.gr.pos1[row];
            if (p) {
                uint16_t *dst = q.gr.out + (int64_t)(p - 1) * K + kk;
                if (!TAIL || in0) *reinterpret_cast<uint4 *>(dst) = r0;
                if (!TAIL || in1) *reinterpret_cast<uint4 *>(dst + 128) = r1;
                r0 = r1 = make_uint4(0, 0, 0, 0);
            }
        } else if (q.zero_outer && q.zero_outer[row]) {
            r0 = r1 = make_uint4(0, 0, 0, 0);
        }
    }
    float w0[8] = {bf16_lo(r0.x), bf16_hi(r0.x), bf16_lo(r0.y), bf16_hi(r0.y),
                   bf16_lo(r0.z), bf16_hi(r0.z), bf16_lo(r0.w), bf16_hi(r0.w)};
    float w1[8] = {bf16_lo(r1.x), bf16_hi(r1.x), bf16_lo(r1.y), bf16_hi(r1.y),
                   bf16_lo(r1.z), bf16_hi(r1.z), bf16_lo(r1.w), bf16_hi(r1.w)};
    if (q.zero_k && active) {
        uint64_t z0 = 0, z1 = 0;
        if (!TAIL || in0) z0 = *reinterpret_cast<const uint64_t *>(q.zero_k + kk);
        if (!TAIL || in1) z1 = *reinterpret_cast<const uint64_t *>(q.zero_k + kk + 128);
        apply_k_mask(w0, z0);
        apply_k_mask(w1, z1);
    }
    uint32_t c0, c1;
    int s0, s1;
    transform_quantize16<B, SR>(w0, w1, plan, c0, c1, s0, s1, q.key, row, kk, kk + 128);
    if (active) store_codes_scales<TAIL>(q.codes, q.scales, row, K, k0, plan.chunk, in0, in1, c0, c1, s0, s1, q.sm);
}

// The same for a workgroup whose units, numbered consecutively over the rows from u0 (uniform) on, all exist, K % 256 == 0: the results then lie one
// unit after the other, and so does the operand but for the gap between its rows, so that addresses are a scalar base and a small offset, and nothing has a
// condition: 235 vector instructions per wave in place of 271 at B = 256.  us: 8192 x 2048 9.7 -> 9.2, 2016 x 11008 11.5 -> 10.9, 1000 x 3072 6.4 -> 6.05;
// where the memory bounds it 1 .. 2 %, 16384 x 28672 196.9 -> 193.4.
template <int B, bool SR> __device__ __forceinline__ void quant_kc_whole(const quant_t &q, uint32_t u0)
{
    const int64_t K = q.K;
    const lane_plan_t plan = make_plan<B>(threadIdx.x & 63);
    const uint32_t n = threadIdx.x >> 4, u = u0 + n;
    const uint32_t first = row_of_unit(u0, q.upr, q.magic);
    uint32_t row = 0, unit = 0, skip = 0;
    if (q.sm.out || q.ld != K || q.gr.out || q.zero_outer || q.zero_k || SR) { // (uniform)
        row = row_of_unit(u, q.upr, q.magic);
        unit = u - row * q.upr;
        skip = (row - first) * (uint32_t)((q.ld - K) * 2);
    }
    const uint8_t *base = reinterpret_cast<const uint8_t *>(q.x) + ((int64_t)u0 * 512 + (int64_t)first * (q.ld - K) * 2);
    const uint32_t at = n * 512 + plan.chunk * 16 + skip;
    uint4 r0 = load_once16(base + at), r1 = load_once16(base + at + 256);
    if (q.gr.out) {
        const uint32_t p = q.gr.pos1[row];
        if (p) {
            uint16_t *dst = q.gr.out + (int64_t)(p - 1) * K + unit * 256 + plan.chunk * 8;
            *reinterpret_cast<uint4 *>(dst) = r0;
            *reinterpret_cast<uint4 *>(dst + 128) = r1;
            r0 = r1 = make_uint4(0, 0, 0, 0);
        }
    } else if (q.zero_outer) {
        if (q.zero_outer[row]) r0 = r1 = make_uint4(0, 0, 0, 0);
    }
    float w0[8] = {bf16_lo(r0.x), bf16_hi(r0.x), bf16_lo(r0.y), bf16_hi(r0.y),
                   bf16_lo(r0.z), bf16_hi(r0.z), bf16_lo(r0.w), bf16_hi(r0.w)};
    float w1[8] = {bf16_lo(r1.x), bf16_hi(r1.x), bf16_lo(r1.y), bf16_hi(r1.y),
                   bf16_lo(r1.z), bf16_hi(r1.z), bf16_lo(r1.w), bf16_hi(r1.w)};
    if (q.zero_k) {
        const uint8_t *zk = q.zero_k + unit * 256 + plan.chunk * 8;
        apply_k_mask(w0, *reinterpret_cast<const uint64_t *>(zk));
        apply_k_mask(w1, *reinterpret_cast<const uint64_t *>(zk + 128));
    }
    uint32_t c0, c1;
    int s0, s1;
    const int64_t kk = (int64_t)unit * 256 + plan.chunk * 8;
    transform_quantize16<B, SR>(w0, w1, plan, c0, c1, s0, s1, q.key, row, kk, kk + 128);
    uint8_t *crow = q.codes + (int64_t)u0 * 128 + (n * 128 + plan.chunk * 4);
    *reinterpret_cast<uint32_t *>(crow) = c0;
    *reinterpret_cast<uint32_t *>(crow + 64) = c1;
    if ((plan.chunk & 3) == 0) {
        uint8_t *srow = q.scales + (int64_t)u0 * 8 + (n * 8 + (plan.chunk >> 2));
        srow[0] = (uint8_t)s0;
        srow[4] = (uint8_t)s1;
        if (q.sm.out) {
            uint8_t *sm = q.sm.out + ((uint64_t)unit * (uint32_t)q.sm.rows + row) * 8 + (plan.chunk >> 2);
            sm[0] = (uint8_t)s0;
            sm[4] = (uint8_t)s1;
        }
    }
}

// FLAT = 0: blockIdx.x is the row, blockIdx.y and the thread its units, 16 to a workgroup; FLAT = 1: the units of all rows are
// numbered consecutively.  FLAT = 1 where it is free to choose: of a row that is no whole number of workgroups FLAT = 0 leaves a part of the last one idle,
// with several of them a row's parts are written far apart in time, and whole workgroups of consecutive units have fewer instructions (quant_kc_whole).
// FLAT = 0 / 1, us: 10000 rows x 4256 27.2 / 19.9, x 3072 15.4 / 15.0, x 11008 53.2 / 45.4; 28672 x 8192 113 / 99; 16384 x 28672 232 / 196; rows of
// exactly one workgroup 2016 x 4096 6.0 / 5.8, 4096 x 4096 9.5 / 9.2, 8192 x 4096 16.2 / 15.7, 32768 x 4096 54.1 / 54.1.  FLAT = 0 for counts above row_of_unit's, and where
// it is the faster one by 1 .. 2 %: such rows that are few or end inside their last unit (500 x 4096 4.7 / 4.8, 10000 x 4064 21.0 / 21.2), and,
// rounded stochastically, which has fewer vector instructions with a row that is the same for the workgroup, rows of whole workgroups (28672 x 8192 165.8 /
// 167.0, 8192 x 12288 73.5 / 73.9, 2048 x 8192 15.0 / 15.3, but x 4256 33.8 / 26.5, x 2048 16.6 / 13.6).
template <int B, bool SR, bool TAIL, int NT> __device__ __forceinline__ void quant_kc_block(const quant_t &q, uint32_t block)
{
    if constexpr (!TAIL) { // (up to 16 or 32 rows' gaps lie within 32 bits)
        const uint32_t u0 = block * (NT / 16);
        if ((uint64_t)u0 + NT / 16 <= (uint64_t)q.outer * q.upr && q.ld - q.K < 1 << 20) {
            quant_kc_whole<B, SR>(q, u0);
            return;
        }
    }
    const uint32_t u = (block * (uint32_t)NT + threadIdx.x) >> 4, r = row_of_unit(u, q.upr, q.magic);
    quant_kc_unit<B, SR, TAIL>(q, r, u - r * q.upr, r < q.outer);
}

template <int B, int FLAT, bool SR, bool TAIL> __global__ __launch_bounds__(256) void k_quant_kc16(quant_t q)
{
    if constexpr (FLAT) {
        quant_kc_block<B, SR, TAIL, 256>(q, blockIdx.x);
    } else {
        const uint32_t unit = (blockIdx.y * 256u + threadIdx.x) >> 4;
        quant_kc_unit<B, SR, TAIL>(q, blockIdx.x, unit, unit < q.upr);
    }
}

// The same with the extracted K-channels copied out on the way (Eq. 7 with S a set of K-channels).  One workgroup takes whole rows, 4096 K-elements
// per pass: one row, or as many shorter ones as fill a pass.  The 16 lanes of a unit leave its elements in LDS as they came, look up the indices that
// fall into it (the list ascends: two loads of 16 entries, one of them the same for all units, or three for a long list), take those elements out, to a copy
// in LDS and to zero, and read their own back: no barrier, since it all stays within a wave.  The copies leave for memory at the end in whole 16-byte pieces.
//
// What bounds it is the issue of vector instructions (the more so beside a large product, whose power budget it shares) and, where a workgroup has one pass, its chain of
// loads.  With a 16-bit table of positions read beside the elements, all of them scattered in LDS and cleared by it, it issued 325 per wave and 16 elements of a lane, here 244 (the plain
// kernel 235): both operands, us, 16384 + 28672 rows x 8192, 82 channels, 226.7 -> 188.7; 8192 + 8192 x 2048, 8, 25.1 -> 23.6; 8192 + 4096 x 4096, 41, 33.4 ->
// 31.1; 2016 + 11008 x 4096, 41, 32.9 -> 32.2; 1000 + 5000 x 3040, 31, 15.4 -> 15.25.  The elements taken out by the whole workgroup between two
// barriers: 203, 27.4, 37.5, 35.9, 15.5; the same with the next row's loads on their way and one .. eight rows per workgroup 196 .. 212, 21 .. 28, 32.6 .. 36,
// 32.6 .. 37, 16 .. 21.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 lds16_t __attribute__((may_alias)); // (a unit's elements are written and read in pieces and one by one)
// What a pointer kept in LDS points to: of one that does not say so the compiler makes flat loads, which are waited for together with all others.
typedef __attribute__((address_space(1))) uint16_t global_u16;
typedef __attribute__((address_space(1))) u32x4 global_u32x4;
constexpr int KC_GATHER_MAX_KPAD = 4096;
constexpr int KC_GATHER_COPY = KC_GATHER_MAX_KPAD * 2, KC_GATHER_LDS = KC_GATHER_COPY + 4096 * 2; // bytes: the copies of the rows, and a pass

template <int B, bool SR, bool TAIL>
__device__ __forceinline__ void quant_kc_gather_rows(const quant_t &q, uint32_t block, uint8_t *lds)
{
    const k_gather_t gk = q.gk;
    const int64_t K = q.K, row0 = (int64_t)block * q.rows_per_wg;
    const int tid = threadIdx.x, l16 = tid & 15, none = 0x7fffffff;
    const int nrows = (int)min((int64_t)q.rows_per_wg, q.outer - row0);
    uint16_t *const copy = reinterpret_cast<uint16_t *>(lds), *const raw = reinterpret_cast<uint16_t *>(lds + KC_GATHER_COPY) + (tid >> 4) * 256;
    const lane_plan_t plan = make_plan<B>(tid & 63);
    // The list at 16 places, and at 16 places between two of those.  Loads without a condition, at places that exist: a wait can then be for one of them.
    const int last = gk.k - 1, step = (gk.k + 15) >> 4, fine = (step + 15) >> 4;
    auto load = [&](int t) { return gk.idx[min(t, last)]; };
    auto entry = [&](int t) {
        const int at = load(t);
        return t <= last ? at : none;
    };
    auto of_unit = [&](bool hit) { return (int)__popc((uint32_t)(__ballot(hit) >> (tid & 48)) & 0xffffu); }; // of its 16 lanes, how many
    const int coarse = entry(l16 * step);
    if (tid < gk.kpad - gk.k) {
#pragma clang loop vectorize(disable) unroll(disable)
        for (int r = 0; r < nrows; ++r) copy[r * gk.kpad + gk.k + tid] = 0;
    }
    // the lane's place in the pass that begins with unit u0, its elements, and the first entries of the list that may lie in its unit
    struct part_t {
        u32x4 r0, r1;
        int64_t row;
        int from, r, t, at;
        bool active;
    };
    auto fetch = [&](uint32_t u0) {
        part_t f;
        uint32_t unit = u0 + (tid >> 4), r = 0;
        if (q.rows_per_wg > 1) { // (one pass)
            r = row_of_unit(unit, q.upr, q.magic);
            unit -= r * q.upr;
        }
        f.active = (int)r < nrows && unit < q.upr;
        r = min(r, (uint32_t)nrows - 1), unit = min(unit, q.upr - 1);
        f.r = (int)r, f.row = row0 + r, f.from = (int)unit * 256;
        const uint16_t *const src = q.x + f.row * q.ld;
        const int kk = f.from + plan.chunk * 8, end = (int)K - 8;
        f.r0 = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + (TAIL ? min(kk, end) : kk)));
        f.r1 = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + (TAIL ? min(kk + 128, end) : kk + 128)));
        const int before = of_unit(coarse < f.from);
        f.t = (before > 0 ? before - 1 : 0) * step;
        if (fine > 1) {
            const int more = of_unit(entry(f.t + l16 * fine) < f.from);
            f.t += (more > 0 ? more - 1 : 0) * fine;
        }
        f.t += l16;
        f.at = load(f.t); // (looked at when it is needed)
        return f;
    };
    part_t f = fetch(0);
    for (uint32_t u0 = 16;; u0 += 16) {
        if (!__ballot(f.active)) break; // (nothing left for this wave)
        const int kk = f.from + plan.chunk * 8;
        const bool in0 = !TAIL || kk < K, in1 = !TAIL || kk + 128 < K;
        lds16_t *const own = reinterpret_cast<lds16_t *>(raw + plan.chunk * 8);
        own[0] = in0 ? f.r0 : u32x4{0, 0, 0, 0};
        own[16] = in1 ? f.r1 : u32x4{0, 0, 0, 0};
        lds_between_lanes();
        int t = f.t, at = f.active && t <= last ? f.at : none;
        for (;;) {
            if (at >= f.from && at < f.from + 256) {
                uint16_t *const e = raw + (at - f.from);
                copy[f.r * gk.kpad + t] = *e;
                *e = 0;
            }
            const uint64_t again = __ballot(l16 == 15 && at < f.from + 256); // (few waves)
            if (!again) break;
            t += 16;
            at = again >> (tid & 48) & 0x8000 ? entry(t) : none;
        }
        lds_between_lanes();
        const u32x4 e0 = own[0], e1 = own[16];
        float w0[8] = {bf16_lo(e0.x), bf16_hi(e0.x), bf16_lo(e0.y), bf16_hi(e0.y),
                       bf16_lo(e0.z), bf16_hi(e0.z), bf16_lo(e0.w), bf16_hi(e0.w)};
        float w1[8] = {bf16_lo(e1.x), bf16_hi(e1.x), bf16_lo(e1.y), bf16_hi(e1.y),
                       bf16_lo(e1.z), bf16_hi(e1.z), bf16_lo(e1.w), bf16_hi(e1.w)};
        const int64_t row = f.row, k0 = f.from;
        const bool active = f.active, more = u0 < q.upr;
        if (more) f = fetch(u0); // the next pass's, on their way while this one's are transformed
        uint32_t c0, c1;
        int s0, s1;
        transform_quantize16<B, SR>(w0, w1, plan, c0, c1, s0, s1, q.key, row, kk, kk + 128);
        if (active) store_codes_scales<TAIL>(q.codes, q.scales, row, K, k0, plan.chunk, in0, in1, c0, c1, s0, s1, q.sm);
        if (!more) break;
    }
    __syncthreads();
    // (the rows' copies lie one after the other, here and there)
#pragma clang loop unroll(disable)
    for (int p = tid * 8; p < nrows * gk.kpad; p += 256 * 8)
        *reinterpret_cast<lds16_t *>(gk.out + row0 * gk.kpad + p) = *reinterpret_cast<const lds16_t *>(copy + p);
}

template <int B, bool SR, bool TAIL> __global__ __launch_bounds__(256) void k_quant_kc16_gather(quant_t q)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[KC_GATHER_LDS];
    quant_kc_gather_rows<B, SR, TAIL>(q, blockIdx.x, lds);
}

// ------------------------------------------------------------------------------------------------
// K-strided operand (element (o, kk) at x[kk*ld + o]).  A workgroup takes a tile of 256 K-rows (fewer in the last
// one, filled up with zeros) x 64 columns: coalesced 16-byte loads (8 columns of one K-row per lane) go to LDS as they are, and the LDS
// transposing read of gfx950 (ds_read_b64_tr_b16) hands every lane 4 consecutive K-elements of one column per
// instruction -- the transposition costs a quarter of an LDS instruction per element.
//
// The transposing read works on groups of 16 lanes: lane s supplies the address of 4 consecutive 16-bit elements
// (a piece of one K-row), and lane n of the group receives, as element j, the element n % 4 of the piece that lane
// 4 j + n / 4 supplied.  With lane s of group g pointing at K-row 64 g + 4 t + s / 4 of the columns 4 (s % 4) .. + 3 of
// the wave's 16, lane n receives K-rows 64 g + 4 t .. + 3 of column n: after 16 reads (t = 0 .. 15) it holds the 64
// consecutive K-elements [64 g, 64 g + 64) of its column.  That is also how the BF16 matrix cores want an operand of 16
// columns (v_mfma_f32_16x16x32_bf16: 8 consecutive K-elements of a column per lane, a quarter of the K-elements in each group of 16
// lanes), which the kernel that forms the outlier product on the way makes use of (k_quant_ks16_outliers).
//
// Strides 1 .. 32 of the transform are butterflies inside a lane's 64 registers.  Strides 64 and 128 are between lanes 16
// and 32 apart: v_permlane16_swap (v_permlane32_swap) exchanges the odd rows of 16 lanes (the upper half) of one register with
// the even rows (the lower half) of another.  Given the registers of K-elements 32 apart, it leaves both terms of a
// butterfly in one lane: afterwards the register's place stands for K bit 6 (7) and the lane's for bit 5 (6).  The two MX
// blocks of a lane lie entirely in its registers (no cross-lane maximum).
//
// (A variant with 128 columns per workgroup, 256-byte pieces of the operand's K-rows, runs at the same speed, and so do plain and
// write-through stores of the codes in whole 128-byte rows.  What it waits for is the memory, and that depends on the order of the workgroups:
// see ks_order.  Reads and writes alone, without the transform, take 62 of 65 us on 4096 x 32768.)
//
// LDS layout: K-row kk at kk * 128 bytes, its four pieces of 32 bytes exchanged by kk's bits 1 and 6: the eight rows that the
// half wave of a transposing read touches then lie in eight different eighths of the 64 banks.
// ------------------------------------------------------------------------------------------------
constexpr int KS_COLS = 64, KT_PITCH = 128;
constexpr uint32_t KS_GROUP = 16, KS_PLAIN = 2048; // column tiles that walk the K-blocks together; tiles up to which they need not

typedef short v4s __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint4 pieces(v4s a, v4s b)
{
    const v2u x = __builtin_bit_cast(v2u, a), y = __builtin_bit_cast(v2u, b);
    return make_uint4(x.x, x.y, y.x, y.y);
}

constexpr int KS_LDS = 256 * KT_PITCH + 256; // bytes: the tile and the K-mask of its rows

__device__ __forceinline__ int ks_swizzle(int kk) { return ((kk >> 1) & 1) | ((kk >> 5) & 2); } // of a row's 32-byte pieces

// a + b and a - b of the lanes that hold the two terms: (x of K-element e, y of e + 32) -> see above.
template <bool HALVES> __device__ __forceinline__ void swap_butterfly(float &x, float &y)
{
    v2u r;
    if constexpr (HALVES)
        r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    else
        r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    const float a = __uint_as_float(r.x), b = __uint_as_float(r.y);
    x = a + b;
    y = a - b;
}

// A tile on its way to LDS: a pass is 32 K-rows x 64 columns; lane: 8 columns (cg) of one of the wave's 8 rows.
struct ks_tile_t {
    uint4 v[8], last;
    uint8_t kz;
};

__device__ __forceinline__ bool ks_at_end(const quant_t &q, int64_t o0, int64_t k0)
{
    return (q.outer & 7) && k0 + 256 >= q.K && o0 + KS_COLS > q.outer;
}

__device__ __forceinline__ void ks_fetch_tile(const quant_t &q, int tid, int64_t o0, int64_t k0, ks_tile_t &f)
{
    const uint16_t *x = q.x;
    const int64_t outer = q.outer, K = q.K, ld = q.ld;
    const int cg = tid & 7, rw = tid >> 3;
    const int64_t oc = o0 + cg * 8;
    const bool ok = oc < outer;
    // K-mask: one byte of the tile's 256 per thread, loaded ahead of the data and handed round through LDS (eight
    // byte loads per lane, one for each of its K-rows, made the masked call 15 % slower than the plain one)
    f.kz = 0;
    if (q.zero_k && k0 + tid < K) f.kz = q.zero_k[k0 + tid];
    // The matrix ends with its last element.  Where that lies inside a piece, the workgroup takes the last pass by itself, the part
    // of a piece with the elements that exist.  (Behind any other K-row there is the next one, or what its stride leaves.)  A
    // condition more on the loads of every pass cost 8192 rows x 4096 0.7 of 20.3 us.
    const bool at_end = ks_at_end(q, o0, k0);
    const int64_t k_end = at_end ? K - 32 : K;
#pragma unroll
    for (int it = 0; it < 8; ++it) { // (a pass is one MX block of K: inside the operand or not as a whole)
        const int64_t kk = k0 + it * 32 + rw;
        f.v[it] = ok && k0 + it * 32 < k_end ? load_once16(x + kk * ld + oc) : make_uint4(0, 0, 0, 0);
    }
    f.last = make_uint4(0, 0, 0, 0);
    if (at_end && ok) {
        const uint16_t *p = x + (k_end + rw) * ld + oc;
        f.last = rw == 31 && oc + 8 > outer ? load_part16(p, (int)(outer - oc)) : load_once16(p);
    }
}

__device__ __forceinline__ void ks_put_tile(const quant_t &q, int tid, int64_t o0, int64_t k0, uint8_t *lds, const ks_tile_t &f)
{
    uint8_t *tile = lds, *kmask = lds + 256 * KT_PITCH;
    const int64_t outer = q.outer;
    const uint8_t *zero_outer = q.gr.out ? nullptr : q.zero_outer;
    const int cg = tid & 7, rw = tid >> 3;
    const int64_t oc = o0 + cg * 8;
    uint32_t cm[4] = {~0u, ~0u, ~0u, ~0u}; // keeps the columns that are not masked out
    if (zero_outer && oc < outer) {
        // the 8 mask bytes of the lane's columns in one load where that is possible (eight dependent byte loads
        // at the head of every workgroup cost the masked call a third more time)
        uint64_t z = 0;
        if ((reinterpret_cast<uintptr_t>(zero_outer) & 7) == 0 && oc + 8 <= outer) {
            z = *reinterpret_cast<const uint64_t *>(zero_outer + oc);
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c)
                if (oc + c < outer && zero_outer[oc + c]) z |= (uint64_t)1 << (8 * c);
        }
#pragma unroll
        for (int c = 0; c < 8; ++c)
            if ((z >> (8 * c)) & 0xffu) cm[c >> 1] &= (c & 1) ? 0x0000ffffu : 0xffff0000u;
    }
    uint32_t zk = 0;   // bit it: the lane's K-row of pass it is masked out
    if (q.zero_k) {    // (uniform: a kernel argument)
        kmask[tid] = f.kz;
        __syncthreads();
#pragma unroll
        for (int it = 0; it < 8; ++it) zk |= (kmask[it * 32 + rw] ? 1u : 0u) << it;
    }
    auto put = [&](int it, uint4 p) {
        const int row = it * 32 + rw; // K-row within the tile
        const uint32_t kz = ((zk >> it) & 1u) ? 0u : ~0u;
        *reinterpret_cast<uint4 *>(tile + row * KT_PITCH + ((cg * 16) ^ (ks_swizzle(row) * 32))) =
            make_uint4(p.x & cm[0] & kz, p.y & cm[1] & kz, p.z & cm[2] & kz, p.w & cm[3] & kz);
    };
#pragma unroll
    for (int it = 0; it < 8; ++it) put(it, f.v[it]);
    if (ks_at_end(q, o0, k0)) put((int)(q.K - 1 - k0) >> 5, f.last);
}

// A tile that lies inside the operand as a whole, with no column masked out (uniform), which all but those at its edges are: no condition
// on its loads and stores, whose addresses are a scalar base and one 32-bit offset per lane.  The general code spends a third of its
// vector instructions on these (846 -> 601 per wave and tile at B = 32, with the products of 64 rows 967 -> 671), which the kernels whose workgroups do more
// than wait for the memory feel: kernels with products, us, 4096 x 32768, 64 rows, 103 -> 97.5, 8192 x 4096, 41 rows, 28.9 -> 27.4, 4096 x 4096, 82 rows,
// 23.0 -> 21.5; plain ones of 2048 x 4096 9.9 -> 8.6, 8192 x 4096 24.4 -> 23.2, 4096 x 32768 74.9 -> 73.1.
__device__ __forceinline__ bool ks_whole(const quant_t &q, int64_t o0, int64_t k0)
{
    return k0 + 256 <= q.K && o0 + KS_COLS <= q.outer && q.ld <= 1 << 24 && (!q.zero_outer || q.gr.out);
}

__device__ __forceinline__ uint32_t ks_load_offset(const quant_t &q, int tid) { return ((uint32_t)(tid >> 3) * (uint32_t)q.ld + (uint32_t)(tid & 7) * 8) * 2; }

__device__ __forceinline__ void ks_fetch_whole(const quant_t &q, uint32_t voff, int64_t o0, int64_t k0, ks_tile_t &f)
{
    const uint8_t *base = reinterpret_cast<const uint8_t *>(q.x + k0 * q.ld + o0);
    const int64_t pass = 64 * q.ld;
#pragma unroll
    for (int it = 0; it < 8; ++it) f.v[it] = load_once16(base + it * pass + voff);
}

__device__ __forceinline__ void ks_put_whole(const quant_t &q, int tid, int64_t k0, uint8_t *lds, const ks_tile_t &f)
{
    const int cg = tid & 7, rw = tid >> 3;
    uint8_t *const even = lds + rw * KT_PITCH + ((cg * 16) ^ (ks_swizzle(rw) * 32)), *const odd = lds + rw * KT_PITCH + ((cg * 16) ^ (ks_swizzle(rw + 64) * 32));
    uint4 v[8];
#pragma unroll
    for (int it = 0; it < 8; ++it) v[it] = f.v[it];
    if (q.zero_k) { // (uniform: a kernel argument)
        uint8_t *kmask = lds + 256 * KT_PITCH;
        kmask[tid] = q.zero_k[k0 + tid];
        __syncthreads();
#pragma unroll
        for (int it = 0; it < 8; ++it)
            if (kmask[it * 32 + rw]) v[it] = make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int it = 0; it < 8; ++it) *reinterpret_cast<uint4 *>(((it & 2) ? odd : even) + it * 32 * KT_PITCH) = v[it];
}

// LDS -> registers, transposed: wave w takes columns [16 w, 16 w + 16); d[t]: K-elements 64 g + 4 t .. + 3 of the lane's column.
__device__ __forceinline__ void ks_read_tile(int tid, const uint8_t *lds, v4s (&d)[16])
{
    const int lane = tid & 63, w = tid >> 6, g = lane >> 4, j = (lane >> 2) & 3, c = lane & 3;
    const uint8_t *src = lds + (64 * g + j) * KT_PITCH + ((w ^ ks_swizzle(64 * g + j)) * 32) + 8 * c;
#pragma unroll
    for (int t = 0; t < 16; ++t)
        d[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)(src + t * 4 * KT_PITCH));
}

// The transform's strides from FROM on, of a lane that holds the 64 consecutive K-elements [64 g, 64 g + 64) of its column, and the factor.
template <int B, int FROM> __device__ __forceinline__ void ks_transform(float (&wv)[64])
{
    if constexpr (B > 0) {
        constexpr int HMAX = B >= 64 ? 32 : 16;
#pragma unroll
        for (int h = FROM; h <= HMAX; h *= 2)
#pragma unroll
            for (int i = 0; i < 64; i += 2 * h)
#pragma unroll
                for (int j = i; j < i + h; ++j) {
                    const float a = wv[j], b = wv[j + h];
                    wv[j] = a + b;
                    wv[j + h] = a - b;
                }
        if constexpr (B >= 128) {
#pragma unroll
            for (int i = 0; i < 32; ++i) swap_butterfly<false>(wv[i], wv[i + 32]); // stride 64
        }
        if constexpr (B == 256) {
#pragma unroll
            for (int i = 0; i < 32; ++i) swap_butterfly<true>(wv[i], wv[i + 32]); // stride 128
        }
        // "+ 0" stores exact zeros unsigned
        const float fin = hadamard_norm<B>();
#pragma unroll
        for (int i = 0; i < 64; ++i) wv[i] = __builtin_fmaf(wv[i], fin, 0.0f);
    }
}

// The lane's column, transformed: quantised and stored.  WHOLE: see ks_whole.
template <int B, bool SR, bool WHOLE> __device__ __forceinline__ void ks_pack(const quant_t &q, int tid, int64_t o0, int64_t k0, const float (&wv)[64])
{
    const int64_t outer = q.outer, K = q.K;
    const int lane = tid & 63, w = tid >> 6, g = lane >> 4, b4 = g & 1, b5 = g >> 1;
    const uint32_t col = 16 * w + (lane & 15);
    const int64_t o = o0 + col;
    const bool active = WHOLE || o < outer;
    // ---- the lane's two MX blocks; at[i]: which of the tile's eight
    const int at[2] = {B == 256 ? b4 + 2 * b5 : B == 128 ? b4 + 4 * b5 : 2 * g, B == 256 ? 4 + b4 + 2 * b5 : B == 128 ? 2 + b4 + 4 * b5 : 2 * g + 1};
    uint32_t c[8];
    uint32_t sc[2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        float amax = 0.0f;
#pragma unroll
        for (int i = 0; i < 32; ++i) amax = fmaxf(amax, fabsf(wv[32 * blk + i]));
        const int s = e8m0_of_amax(amax);
        sc[blk] = (uint32_t)s;
        if constexpr (SR) {
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                float t8[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) t8[i] = wv[32 * blk + 8 * q4 + i];
                c[4 * blk + q4] = pack8_sr(t8, s, q.key, o, k0 + 32 * at[blk] + 8 * q4);
            }
        } else {
            const float X = __uint_as_float((uint32_t)s << 23);
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const float *v8 = wv + 32 * blk + 8 * q4;
                uint32_t p = __float_as_uint(v8[0]); // (every byte is written: any register that is free)
                p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(p, v8[0], v8[1], X, 0);
                p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(p, v8[2], v8[3], X, 1);
                p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(p, v8[4], v8[5], X, 2);
                p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(p, v8[6], v8[7], X, 3);
                c[4 * blk + q4] = p;
            }
        }
    }
    if constexpr (WHOLE) {
        uint8_t *crow = q.codes + (o0 * (K >> 1) + (k0 >> 1)) + (col * (uint32_t)(K >> 1) + 16 * (uint32_t)at[0]);
        *reinterpret_cast<uint4 *>(crow) = make_uint4(c[0], c[1], c[2], c[3]);
        *reinterpret_cast<uint4 *>(crow + (B == 256 ? 64 : B == 128 ? 32 : 16)) = make_uint4(c[4], c[5], c[6], c[7]);
    } else if (active) {
        uint8_t *crow = q.codes + o * (K >> 1) + (k0 >> 1);
        if (k0 + 32 * at[0] < K) *reinterpret_cast<uint4 *>(crow + 16 * at[0]) = make_uint4(c[0], c[1], c[2], c[3]);
        if (k0 + 32 * at[1] < K) *reinterpret_cast<uint4 *>(crow + 16 * at[1]) = make_uint4(c[4], c[5], c[6], c[7]);
    }
    // The column's 8 scale bytes of this tile sit in its four lanes, two each: two exchanges give every lane all of them, and one lane
    // stores them at once, another the second copy.  Byte stores, four per lane, were three quarters of the kernel's write requests.
    const uint32_t own = sc[0] | sc[1] << 8;
    const v2u r16 = __builtin_amdgcn_permlane16_swap(own, own, false, false); // of the even and the odd row of 16 lanes
    // bytes of half a column: in the order of the blocks (B < 128), else first blocks of both lanes, then second ones
    const uint32_t four = __builtin_amdgcn_perm(r16.y, r16.x, B >= 128 ? 0x05010400u : 0x05040100u);
    const v2u r32 = __builtin_amdgcn_permlane32_swap(four, four, false, false);
    const uint32_t lower = B == 256 ? __builtin_amdgcn_perm(r32.y, r32.x, 0x05040100u) : r32.x;
    const uint32_t upper = B == 256 ? __builtin_amdgcn_perm(r32.y, r32.x, 0x07060302u) : r32.y;
    const int rot = WHOLE ? 0 : tail_rotation(K, k0);
    if (active && g == 0) {
        uint8_t *srow = q.scales + (o0 * (K >> 5) + (k0 >> 5)) + col * (uint32_t)(K >> 5);
        if (rot == 0 && (reinterpret_cast<uintptr_t>(srow) & 7) == 0) {
            *reinterpret_cast<uint2 *>(srow) = make_uint2(lower, upper);
        } else { // the canonical array has no alignment rule, and the last tile may hold fewer blocks
            const uint64_t all = (uint64_t)upper << 32 | lower;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i < 8 - rot) srow[i] = (uint8_t)(all >> (8 * i));
        }
    }
    if (q.sm.out && active && g == 1)
        *reinterpret_cast<uint64_t *>(q.sm.out + ((k0 >> 8) * q.sm.rows + o0) * 8 + col * 8) = ((uint64_t)upper << 32 | lower) << (8 * rot);
}

// The column of the lane from its raw elements on: copied out if it is extracted, transformed, quantised and stored.
template <int B, bool SR, bool WHOLE> __device__ __forceinline__ void ks_finish(const quant_t &q, int tid, int64_t o0, int64_t k0, const v4s (&d)[16])
{
    float wv[64];
#pragma unroll
    for (int t = 0; t < 16; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) wv[4 * t + j] = bf16_one((uint16_t)d[t][j]);

    // ---- an extracted column leaves as it came and counts as zero here: the lane has 64 of its K-elements in a row
    // (as a launch of its own that reads two bytes of every K-row, this copy took 31 us for 64 columns x 32768)
    if (q.gr.out) {
        const int lane = tid & 63, g = lane >> 4;
        const int64_t o = o0 + 16 * (tid >> 6) + (lane & 15);
        const uint32_t p = WHOLE || o < q.outer ? q.gr.pos1[o] : 0u;
        if (p) {
            uint16_t *dst = q.gr.out + (int64_t)(p - 1) * q.K + k0 + 64 * g;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (WHOLE || k0 + 64 * g + 8 * i < q.K) *reinterpret_cast<uint4 *>(dst + 8 * i) = pieces(d[2 * i], d[2 * i + 1]);
#pragma unroll
            for (int i = 0; i < 64; ++i) wv[i] = 0.0f;
        }
    }
    ks_transform<B, 1>(wv);
    ks_pack<B, SR, WHOLE>(q, tid, o0, k0, wv);
}

template <int B, bool SR>
__device__ __forceinline__ void quant_ks_tile(const quant_t &q, uint32_t bx, uint32_t by, uint8_t *lds)
{
    const int64_t o0 = (int64_t)bx * KS_COLS, k0 = (int64_t)by * 256;
    const int tid = threadIdx.x;
    ks_tile_t f;
    v4s d[16];
    if (ks_whole(q, o0, k0)) { // (uniform)
        ks_fetch_whole(q, ks_load_offset(q, tid), o0, k0, f);
        ks_put_whole(q, tid, k0, lds, f);
        __syncthreads();
        ks_read_tile(tid, lds, d);
        ks_finish<B, SR, true>(q, tid, o0, k0, d);
    } else {
        ks_fetch_tile(q, tid, o0, k0, f);
        ks_put_tile(q, tid, o0, k0, lds, f);
        __syncthreads();
        ks_read_tile(tid, lds, d);
        ks_finish<B, SR, false>(q, tid, o0, k0, d);
    }
}

// Workgroup L -> column tile bx, K-block by.  Consecutive workgroups go to the eight XCDs in turn; here each XCD takes a contiguous run of the
// sequence in which KS_GROUP neighbouring column tiles walk all K-blocks together.  What an XCD's workgroups in flight touch then lies together:
// reads in pieces of KS_GROUP x 128 bytes of a K-row, which share an L2 where the rows do not begin on 128-byte lines, and a few output rows,
// each written in one go (their scales too, of which 16 K-blocks share a line).  In the plain order (all column tiles of a K-block, then
// the next) eight L2s held parts of the same lines, and 128-byte pieces of thousands of output rows were written at a time.  Plain / in runs,
// us: [32768][4096] 72.7 / 64.9, [28672][8192] 129 / 119, [8192][14336] 63.8 / 56.6, [28672][9056] 181 / 148, [28672][20976] (rows off the
// lines) 482 / 360, [11008][4096] 27.1 / 25.3; groups of 8 and 32 within 2 % of that.  Workgroups that are nearly all in flight at once gain only where
// rows lie off the lines ([2048][11488] 16.8 / 14.9, [4096][1000] 5.8 / 5.1, but [4096][4096] 11.1 / 12.6, [5120][6400] 18.4 / 19.4, [8192][4096] 19.5 /
// 20.3): up to KS_PLAIN tiles take the plain order there (run = 0).
__device__ __forceinline__ void ks_order(const ks_order_t &o, uint32_t L, uint32_t &bx, uint32_t &by)
{
    const uint32_t xcd = L & 7, v = o.run ? xcd * o.run + min(xcd, o.rest) + (L >> 3) : L;
    const uint32_t g = (uint32_t)(v * o.magic >> 44), r = v - g * o.per_group;
    if (g < o.groups) {
        by = r / KS_GROUP;
        bx = g * KS_GROUP + r % KS_GROUP;
    } else { // the last group is narrower
        by = o.narrow == 1 ? r : __umulhi(r, o.narrow_magic);
        bx = g * KS_GROUP + r - by * o.narrow;
    }
}

// The extracted K-channels of a K-strided operand, copied out: 64 channels x 64 outer indices per workgroup through LDS, so that both the reads (along
// the outer indices of one channel) and the writes (along the channels of one outer index) are whole 128-byte segments, 16 bytes per lane.  These
// workgroups go ahead of the operand's tiles, in their launch, which takes no longer for it, where a launch for each operand
// took 3 .. 5 us: weight gradients 4096 x 4096 x 8192, 82 channels, 140 -> 131 us, 352 x 2048 x 2464, 25, 31 -> 24.5.
__device__ __forceinline__ void ks_gather_channels(const quant_t &q, uint32_t block, uint8_t *lds)
{
    constexpr int PITCH = 72; // elements: 144-byte rows, 16-byte aligned
    uint16_t *const tile = reinterpret_cast<uint16_t *>(lds);
    const int row = threadIdx.x >> 3, seg = threadIdx.x & 7;
    const uint32_t groups = (uint32_t)q.gk.kpad >> 6, to = block / groups;
    const int t0 = (int)(block - to * groups) * 64;
    const int64_t o0 = (int64_t)to * 64, o = o0 + seg * 8;
    if (o0 >= q.outer) return;
    uint4 v[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int t = t0 + p * 32 + row;
        v[p] = make_uint4(0u, 0u, 0u, 0u);
        if (t < q.gk.k && o < q.outer) {
            const uint16_t *src = q.x + (int64_t)q.gk.idx[t] * q.ld + o;
            if (o + 8 <= q.outer) {
                v[p] = load_once16(src);
            } else { // (the last, ragged segment of a channel)
                uint32_t e[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) e[j] = o + j < q.outer ? load_once2(src + j) : (uint16_t)0;
                v[p] = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
            }
        }
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) *reinterpret_cast<lds16_t *>(&tile[(p * 32 + row) * PITCH + seg * 8]) = u32x4{v[p].x, v[p].y, v[p].z, v[p].w};
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int ol = p * 32 + row; // one outer index, 8 channels per lane
        uint32_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = tile[(seg * 8 + j) * PITCH + ol];
        if (o0 + ol < q.outer)
            *reinterpret_cast<uint4 *>(q.gk.out + (o0 + ol) * q.gk.kpad + t0 + seg * 8) = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
    }
}

// Workgroup `block` of a K-strided operand.
template <int B, bool SR> __device__ __forceinline__ void quant_ks_block(const quant_t &q, uint32_t block, uint8_t *lds)
{
    if (block < q.gather_blocks) {
        ks_gather_channels(q, block, lds);
        return;
    }
    uint32_t bx, by;
    ks_order(q.order, block - q.gather_blocks, bx, by);
    quant_ks_tile<B, SR>(q, bx, by, lds);
}

template <int B, bool SR> __global__ __launch_bounds__(256) void k_quant_ks16(quant_t q)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[KS_LDS];
    quant_ks_block<B, SR>(q, blockIdx.x, lds);
}

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// A K-strided operand (nothing extracted from it), and on the way its bf16 products with the k <= 16 RT rows extracted from the other
// one (second term of Eq. 7 / 8): the operand's tile is in registers in the matrix cores' layout anyway, and reading it once more for these products by
// themselves is what they cost.  Quantiser and products, us in two kernels / here: 4096 x 32768 with 64 rows 73 + 50 / 92, 4096 x 11008 with 21
// 26.5 + 22.5 / 31, 8192 x 4096 with 41 20 + 19 / 27, 4096 x 4096 with 82 11.5 + 13.7 / 21.5; the partial sums are added by k_oe_reduce as before.
//
// A workgroup takes every nslice-th tile along K, so that the sums leave once per slice and not once per tile; four of them per compute unit
// hide each other's loads.  The extracted rows' 256 K-elements of the tile come with its loads and take its place in LDS once it is in
// registers (each wave reading its fragments from memory: 103 in place of 92 us in the first example; the matrix cores' own time is a tenth).
//
// The extracted rows are those that the other operand's quantiser has copied out, or (idx) lie in that operand where it is
// K-contiguous: then its quantiser need not know the selection, and a workgroup more for each extracted row sets its codes and scales
// to zero.  B = -1: an operand that is packed already or rounded stochastically, the same products by themselves (short slices; for long
// ones k_outlier_products).
template <int B, int RT> __global__ __launch_bounds__(256, RT <= 4 ? 4 : 3) void k_quant_ks16_outliers(quant_t q, outlier_job_t e)
{
    constexpr int TILE_LDS = RT * 8192 > KS_LDS ? RT * 8192 : KS_LDS;
    __shared__ __attribute__((aligned(16))) uint8_t lds[TILE_LDS + RT * 16 * 8];
    const global_u16 **const row_at = reinterpret_cast<const global_u16 **>(lds + TILE_LDS);
    const int64_t K = q.K;
    const uint32_t tiles = q.col_tiles * (uint32_t)e.nslice;
    if (blockIdx.x >= tiles) {
        clear_extracted_row(e, (int)(blockIdx.x - tiles), K);
        return;
    }
    uint32_t bx, slice;
    ks_order(q.order, blockIdx.x, bx, slice);
    const int64_t o0 = (int64_t)bx * KS_COLS;
    for (int t = threadIdx.x; t < 16 * RT; t += 256) { // (the last row stands for those behind it, whose sums are not stored)
        const int r = min(t, e.k - 1);
        row_at[t] = (const global_u16 *)(e.rows + (e.idx ? e.idx[r] : r) * e.ld);
    }
    __syncthreads();
    v4f acc[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    constexpr bool AHEAD = B < 0 && RT <= 3; // (registers that a tile's quantisation needs: with it three workgroups fit, and nothing is gained)
    const int upr = (int)q.upr, nslice = e.nslice;
    int by = (int)slice;
    ks_tile_t ahead;
    auto fetch = [&](auto whole, int tid, int64_t k0, ks_tile_t &tile) {
        if constexpr (decltype(whole)::value)
            ks_fetch_whole(q, ks_load_offset(q, tid), o0, k0, tile);
        else
            ks_fetch_tile(q, tid, o0, k0, tile);
    };
    // The tile at K-block by (AHEAD: which lies in `ahead`; the next one follows it there).
    auto take = [&](auto whole) {
        constexpr bool WHOLE = decltype(whole)::value;
        // What depends on the lane alone is formed anew for every tile: kept across the tiles it took 40 registers too many.
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int64_t k0 = (int64_t)by * 256;
        ks_tile_t tile;
        if constexpr (AHEAD)
            tile = ahead;
        else
            fetch(whole, tid, k0, tile);
        // the extracted rows' 256 K-elements: piece c (8 elements) of row r0 + 8 i
        const int c = tid & 31, r0 = tid >> 5;
        u32x4 f[2 * RT];
#pragma unroll
        for (int i = 0; i < 2 * RT; ++i) {
            f[i] = u32x4{0, 0, 0, 0};
            if (WHOLE || k0 + 8 * c < K) f[i] = *reinterpret_cast<const global_u32x4 *>(row_at[r0 + 8 * i] + (k0 + 8 * c));
        }
        if constexpr (WHOLE)
            ks_put_whole(q, tid, k0, lds, tile);
        else
            ks_put_tile(q, tid, o0, k0, lds, tile);
        __syncthreads();
        v4s d[16];
        ks_read_tile(tid, lds, d);
        if constexpr (AHEAD) {
            if (by + nslice < upr) fetch(whole, tid, k0 + 256ll * nslice, ahead);
        }
        __syncthreads(); // the tile is in registers: its place takes the extracted rows
        // A tile of 16 rows as 8 x 64 pieces: at (i, 16 g + r) the K-elements 64 g + 8 i .. + 7 of row r, what lane 16 g + r hands to
        // matrix-core instruction i.  Row r at r ^ (8 (g & 1) + i): the 16 pieces that 16 lanes write then cover the banks once.
        uint4 *const s = reinterpret_cast<uint4 *>(lds);
        {
            const int at = (c & 7) * 64 + (c >> 3) * 16, x = c & 15;
#pragma unroll
            for (int i = 0; i < 2 * RT; ++i) *reinterpret_cast<u32x4 *>(s + (i >> 1) * 512 + at + ((r0 + 8 * (i & 1)) ^ x)) = f[i];
        }
        __syncthreads();
        {
            const int lane = tid & 63, g16 = lane & 48, x = 8 * ((lane >> 4) & 1), r = lane & 15;
#pragma unroll
            for (int i = 0; i < 8; ++i) { // (the sums of different rows in turn: none waits for the one before)
                const v8bf column = __builtin_bit_cast(v8bf, pieces(d[2 * i], d[2 * i + 1]));
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, s[rt * 512 + i * 64 + g16 + (r ^ (x + i))]), column,
                                                                      acc[rt], 0, 0, 0);
                if (i & 1) __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (by + nslice < upr) __syncthreads(); // (the next tile may be written)
        if constexpr (B >= 0) ks_finish<B, false, WHOLE>(q, tid, o0, k0, d);
    };
    if constexpr (AHEAD) {
        fetch(std::false_type{}, threadIdx.x, (int64_t)by * 256, ahead);
        for (; by < upr; by += nslice) take(std::false_type{});
    } else {
        const int whole = ks_whole(q, o0, 0) ? (int)(K >> 8) : 0;
        for (; by < whole; by += nslice) take(std::true_type{});
#pragma unroll 1
        for (; by < upr; by += nslice) take(std::false_type{});
    }
    const int g = (threadIdx.x >> 4) & 3;
    const int64_t o = o0 + 16 * (threadIdx.x >> 6) + (threadIdx.x & 15);
    if (o < q.outer) {
        float *p = e.p + (int64_t)slice * e.k * q.outer + o;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = 16 * rt + 4 * g + r;
                if (t < e.k) p[(int64_t)t * q.outer] = acc[rt][r];
            }
    }
}

// The same for a K-contiguous operand.  A workgroup takes tiles of 64 rows x 256 K-elements, 16 rows to a wave: lane 16 g + r loads the eight pieces 32 i + 8 g
// .. + 7 of row r, which is what it hands to matrix-core instruction i, and after the strides 1, 2, 4 in registers and 8, 16 between lanes (each exchange
// leaves a lane with the halves of the next pair of K bits, see swap_butterfly) it holds 64 consecutive K-elements as the K-strided kernel's lanes do.
// In place of a second pass over the operand.  Quantiser and products, us in two kernels / here: 12296 x 6368 with 2 rows 40 + 45 / 52, 9152 x 16672 with 2 73
// + 56 / 105, 11008 x 4096 with 21 25 + 24 / 32, 4096 x 4096 with 82 14 + 15 / 21, 2048 x 544 with 7 4 + 7 / 5.
//
// What bounds it is how the memory takes pieces of 64 bytes of 16 rows: an operand up to KEEP_LONG is read through the caches, which fetch both halves of a line at
// once (56 / 52, 36 / 32, 11.5 / 9.3 us); a larger one past them, or the product finds the packed operands gone (9152 x 16672: 105 / 97, but the product 61 / 89; 5632 x
// 16384 71 / 71 and 193 / 208; 11008 x 8192 67 / 62 and 107 / 108).  The slices of a tile of rows are neighbours on an XCD and take every nslice-th K-block, so that what is read at a time lies
// together; each slice a run of K-blocks, its workgroups on all XCDs: 60, 109, 37.  The next tile's loads ahead: the same.
template <int B, int RT, bool KEEP> __global__ __launch_bounds__(256, RT <= 4 ? 4 : 3) void k_quant_kc16_outliers(quant_t q, outlier_job_t e)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[RT * 8192 + RT * 16 * 8];
    const global_u16 **const row_at = reinterpret_cast<const global_u16 **>(lds + RT * 8192);
    const int64_t K = q.K;
    const uint32_t tiles = q.col_tiles * (uint32_t)e.nslice;
    if (blockIdx.x >= tiles) {
        clear_extracted_row(e, (int)(blockIdx.x - tiles), K);
        return;
    }
    // Each XCD takes a run of the workgroups, the slices of a tile of rows next to each other.
    const uint32_t xcd = blockIdx.x & 7, rest = tiles & 7, at = xcd * (tiles >> 3) + min(xcd, rest) + (blockIdx.x >> 3), bx = at / (uint32_t)e.nslice;
    const int upr = (int)q.upr, nslice = e.nslice, slice = (int)(at - bx * (uint32_t)nslice);
    const int64_t o0 = (int64_t)bx * KS_COLS;
    for (int t = threadIdx.x; t < 16 * RT; t += 256) { // (the last row stands for those behind it, whose sums are not stored)
        const int r = min(t, e.k - 1);
        row_at[t] = (const global_u16 *)(e.rows + (e.idx ? e.idx[r] : r) * e.ld);
    }
    __syncthreads();
    v4f acc[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    // (rows past the end repeat the last one; what comes of them is not stored)
    const uint16_t *const src = q.x + min(o0 + 16 * (threadIdx.x >> 6) + (threadIdx.x & 15), q.outer - 1) * q.ld + ((threadIdx.x >> 4) & 3) * 8;
    auto take = [&](int by, auto whole) {
        constexpr bool WHOLE = decltype(whole)::value;
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int64_t k0 = (int64_t)by * 256;
        u32x4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = u32x4{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (WHOLE || k0 + 32 * i < K) {
                const u32x4 *p = reinterpret_cast<const u32x4 *>(src + k0 + 32 * i);
                v[i] = KEEP ? *p : __builtin_nontemporal_load(p);
            }
        // the extracted rows' 256 K-elements: piece c (8 elements) of row r0 + 8 i
        const int c = tid & 31, r0 = tid >> 5;
        u32x4 f[2 * RT];
#pragma unroll
        for (int i = 0; i < 2 * RT; ++i) {
            f[i] = u32x4{0, 0, 0, 0};
            if (WHOLE || k0 + 8 * c < K) f[i] = *reinterpret_cast<const global_u32x4 *>(row_at[r0 + 8 * i] + (k0 + 8 * c));
        }
        // A tile of 16 rows as 8 x 64 pieces: at (i, 16 g + r) piece 4 i + g of row r, at r ^ (4 i + g): the 16 pieces that 16 lanes write then cover the banks once.
        u32x4 *const s = reinterpret_cast<u32x4 *>(lds);
        {
            const int at = (c >> 2) * 64 + (c & 3) * 16, x = c & 15;
#pragma unroll
            for (int i = 0; i < 2 * RT; ++i) s[(i >> 1) * 512 + at + ((r0 + 8 * (i & 1)) ^ x)] = f[i];
        }
        __syncthreads();
        {
            const int g = (tid >> 4) & 3, r = tid & 15;
#pragma unroll
            for (int i = 0; i < 8; ++i) { // (the sums of different rows in turn: none waits for the one before)
                const v8bf row = __builtin_bit_cast(v8bf, v[i]);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, s[rt * 512 + i * 64 + g * 16 + (r ^ ((4 * i + g) & 15))]), row, acc[rt], 0, 0, 0);
                if (i & 1) __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads(); // (the next tile's rows may be written)
        if constexpr (B > 0) {
            float wv[64]; // K bits 0 .. 2, then of the piece's number i: bit 1 and bit 2 (after the exchanges K bits 3 and 4), bit 0 (K bit 5)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int at = 8 * ((i >> 1) & 1) + 16 * (i >> 2) + 32 * (i & 1);
                const uint32_t p[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) wv[at + 2 * j] = bf16_lo(p[j]), wv[at + 2 * j + 1] = bf16_hi(p[j]);
            }
#pragma unroll
            for (int h = 1; h <= 4; h *= 2)
#pragma unroll
                for (int i = 0; i < 64; i += 2 * h)
#pragma unroll
                    for (int j = i; j < i + h; ++j) {
                        const float a = wv[j], b = wv[j + h];
                        wv[j] = a + b;
                        wv[j + h] = a - b;
                    }
#pragma unroll
            for (int i = 0; i < 64; ++i)
                if (!(i & 8)) swap_butterfly<false>(wv[i], wv[i + 8]); // stride 8
#pragma unroll
            for (int i = 0; i < 64; ++i)
                if (!(i & 16)) swap_butterfly<true>(wv[i], wv[i + 16]); // stride 16
            ks_transform<B, 32>(wv);
            ks_pack<B, false, WHOLE>(q, tid, o0, k0, wv);
        }
    };
    const int whole = o0 + KS_COLS <= q.outer ? (int)(K >> 8) : 0;
    int by = slice;
#pragma unroll 1
    for (; by < whole; by += nslice) take(by, std::true_type{});
#pragma unroll 1
    for (; by < upr; by += nslice) take(by, std::false_type{});
    const int g = (threadIdx.x >> 4) & 3;
    const int64_t o = o0 + 16 * (threadIdx.x >> 6) + (threadIdx.x & 15);
    if (o < q.outer) {
        float *p = e.p + (int64_t)slice * e.k * q.outer + o;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = 16 * rt + 4 * g + r;
                if (t < e.k) p[(int64_t)t * q.outer] = acc[rt][r];
            }
    }
}

// Both operands of a product in one launch: the workgroups below `na` take the first, the others the second; a K-strided one beside a
// K-contiguous one goes first (its workgroups take longest).  A launch costs at
// least 4 us next to its neighbours (the last workgroups of one kernel run alone, and so do the first of the next), half of
// what an operand of 8 M elements takes.
enum quant_kind_t { KC, KC_GATHER, KS };
template <quant_kind_t OP> constexpr int quant_lds() { return OP == KS ? KS_LDS : OP == KC_GATHER ? KC_GATHER_LDS : 16; }

template <int B, quant_kind_t OP, bool TAIL, int NT = 256, bool SR = false>
__device__ __forceinline__ void quant_block(const quant_t &q, uint32_t block, uint8_t *lds)
{
    if constexpr (OP == KS) {
        quant_ks_block<B, SR>(q, block, lds);
    } else if constexpr (OP == KC_GATHER) {
        quant_kc_gather_rows<B, SR, TAIL>(q, block, lds);
    } else {
        quant_kc_block<B, SR, TAIL, NT>(q, block);
    }
}

// The top-k selection in workgroup 0, an operand that does not depend on it in the others.  Every workgroup of the launch gets the LDS that
// the selection needs (46 KB for 8192 keys).  Beside a K-contiguous operand, whose own kernel needs none, workgroups of 512 threads let more waves
// share it, and hold more keys than the 8192 of 256 threads; with few keys beside a large operand, which outlasts their selection anyway, the smaller ones
// are a little faster.  Whole calls with 1 % of the rows extracted, M x N x K, us with 256 / 512 threads: 8192 x 4096 x 4096 126.2 / 123.7, 4096 x 4096 x 4096 88.9 /
// 87.1, 2048 x 4096 x 4096 77.4 / 76.1 (each call waited for), 1024 rows beside a K-strided operand of 1 M elements, read in place, 35.5 / 34.3 (the same), but
// 2000 x 8192 x 8192 142.2 / 143.9, 2000 x 4096 x 11008 113.9 / 116.1, 500 x 8192 x 8192 95.3 / 97.3.
constexpr int TOPK_BESIDE_DIM = 8192, TOPK_BESIDE_DIM_KC = 16384;
bool topk_by_512(int64_t dim, const quant_t &q) { return dim > 2048 || q.outer * q.K <= 16ll << 20; } // (K-contiguous)
template <int B, quant_kind_t OP, bool TAIL, int NT> __global__ __launch_bounds__(NT) void k_topk_and_quant(topk_job_t t, quant_t q)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t dyn[];
    if (blockIdx.x == 0)
        topk_lds<NT>(t.scores, t.dim, t.k, t.idx, t.mask, t.pos1, reinterpret_cast<uint32_t *>(dyn));
    else
        quant_block<B, OP, TAIL, NT>(q, blockIdx.x - 1, dyn);
}

template <int B, quant_kind_t OPA, quant_kind_t OPB, bool TAIL>
__global__ __launch_bounds__(256) void k_quant_two(quant_t qa, quant_t qb, uint32_t na)
{
    constexpr int LDS = quant_lds<OPA>() > quant_lds<OPB>() ? quant_lds<OPA>() : quant_lds<OPB>();
    __shared__ __attribute__((aligned(16))) uint8_t lds[LDS];
    if (blockIdx.x < na)
        quant_block<B, OPA, TAIL>(qa, blockIdx.x, lds);
    else
        quant_block<B, OPB, TAIL>(qb, blockIdx.x - na, lds);
}

// A K-strided operand rounded to nearest and a stochastically rounded one in one launch, in this order: the second is bound by its vector
// instructions (8192 x 11008: 79 us, of which the memory takes 46) and starts while the first, bound by the memory, ends.  Whole calls, two
// launches / this order / the other / workgroups mixed evenly, us: dgrad 8192 x 4096 x 11008 244 / 241 / 242 / 248, 2048 x 8192 x 8192 112.8 / 107.7 / 109.8 /
// 122.6, 2048 x 11008 x 4096 87.9 / 77.6 / 78.7 / 79.9, 47 x 4096 x 28672 87.7 / 84.1 / 84.8 / 82.6, wgrad 4096 x 4096 x 8192 105.2 / 99.6 / 102.2 / 107.9.
template <int B, quant_kind_t OPA, bool TAIL> __global__ __launch_bounds__(256) void k_quant_two_sr(quant_t qa, quant_t qb, uint32_t nb)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[KS_LDS];
    if (blockIdx.x < nb)
        quant_block<B, KS, false>(qb, blockIdx.x, lds);
    else
        quant_block<B, OPA, TAIL, 256, true>(qa, blockIdx.x - nb, lds);
}

// A small product of two K-contiguous operands from which nothing is extracted, in one launch: a workgroup quantises the 32 rows of A and the
// 32 of B that its tile of C needs, 256 K-elements at a time, into LDS, and multiplies them there.  The codes and scales of a row leave
// with the first tile that has it.
// Bound by the launches: 3 us of the host and 3 of the GPU for each, and quantisers and product by themselves were two.  256 x 256 x 256, whole
// call: 10.4 us in two launches, 7.2 here, of which the host's part is 7.  A wave quantises four rows of a stage: with 256 threads, 16 rows for each wave, a
// stage took 2.6 us, now 1.2.  The loads of the next stage are on their way meanwhile, and two buffers leave one barrier for a stage.
// As in the product kernel of such shapes (tiles of 32 or 64 rows, gemm_mx_small.hip) four waves take a matrix-core step of each stage, their
// sums are added in wave order, and a last stage of K that is no multiple of 256 ends with the row: the same bits.
constexpr int TILE_THREADS = 1024;
struct tile_product_t {
    const uint16_t *x[2]; // A, B
    int64_t ld[2], rows[2], K;
    uint8_t *codes[2], *scales[2];
    int64_t ldc;
    int tiles_m;
};
__device__ __forceinline__ void put_c(float *p, float v) { *p = v; }
__device__ __forceinline__ void put_c(uint16_t *p, float v)
{
    const __bf16 b = (__bf16)v; // nearest even
    *p = __builtin_bit_cast(uint16_t, b);
}
template <int B, typename OUT> __global__ __launch_bounds__(TILE_THREADS) void k_quant_and_product(tile_product_t p, OUT *__restrict__ C)
{
    constexpr int SLAB = 64 * 128, BUF = SLAB + 64 * 8; // codes of 64 rows (rows of A, then of B), their scales
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * BUF];
    static_assert(2 * BUF >= 4 * 16 * 64 * 4, "the waves' sums take the place of the stages");
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, h = lane >> 5;
    const int bm = blockIdx.x % p.tiles_m, bn = blockIdx.x / p.tiles_m;
    const int64_t K = p.K;
    // Quantisation: 16 lanes for row r of the slab, in the first half of the waves a row of A, in the second one of B.
    const lane_plan_t plan = make_plan<B>(lane);
    const int side = w >> 3, r = tid >> 4, x = (r >> 1) & 7, in_chunk = (plan.chunk & 3) * 4;
    const int64_t row = 32ll * (side ? bn : bm) + (r & 31);
    const bool active = row < p.rows[side], leaves = active && (side ? bm : bn) == 0;
    const uint16_t *const src = p.x[side] + row * p.ld[side] + plan.chunk * 8;
    uint4 raw[2];
    auto fetch = [&](int64_t k0) {
        const int64_t kk = k0 + plan.chunk * 8;
        raw[0] = raw[1] = make_uint4(0, 0, 0, 0);
        if (active && kk < K) raw[0] = *reinterpret_cast<const uint4 *>(src + k0);
        if (active && kk + 128 < K) raw[1] = *reinterpret_cast<const uint4 *>(src + k0 + 128);
    };
    v16f acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
    fetch(0);
    int buf = 0;
    for (int64_t k0 = 0; k0 < K; k0 += 256, buf ^= 1) {
        uint8_t *const slab = lds + buf * BUF;
        const int64_t kk = k0 + plan.chunk * 8;
        const int j0 = ((plan.chunk >> 2) + tail_rotation(K, k0)) & 7, j1 = (j0 + 4) & 7; // the lane's MX blocks in the stage
        float w0[8] = {bf16_lo(raw[0].x), bf16_hi(raw[0].x), bf16_lo(raw[0].y), bf16_hi(raw[0].y),
                       bf16_lo(raw[0].z), bf16_hi(raw[0].z), bf16_lo(raw[0].w), bf16_hi(raw[0].w)};
        float w1[8] = {bf16_lo(raw[1].x), bf16_hi(raw[1].x), bf16_lo(raw[1].y), bf16_hi(raw[1].y),
                       bf16_lo(raw[1].z), bf16_hi(raw[1].z), bf16_lo(raw[1].w), bf16_hi(raw[1].w)};
        if (k0 + 256 < K) fetch(k0 + 256);
        uint32_t c0, c1;
        int s0, s1;
        transform_quantize16<B, false>(w0, w1, plan, c0, c1, s0, s1, sr_key_t{0, 0}, 0, 0, 0);
        *reinterpret_cast<uint32_t *>(slab + r * 128 + (j0 ^ x) * 16 + in_chunk) = c0;
        *reinterpret_cast<uint32_t *>(slab + r * 128 + (j1 ^ x) * 16 + in_chunk) = c1;
        if (in_chunk == 0) slab[SLAB + r * 8 + j0] = (uint8_t)s0, slab[SLAB + r * 8 + j1] = (uint8_t)s1;
        if (leaves)
            store_codes_scales<true>(p.codes[side], p.scales[side], row, K, k0, plan.chunk, kk < K, kk + 128 < K, c0, c1, s0, s1, {nullptr, 0});
        __syncthreads();
        if (w < 4) {
            const int at = ((4 * h + w) ^ ((l32 >> 1) & 7)) * 16;
            const uint4 a = *reinterpret_cast<const uint4 *>(slab + l32 * 128 + at), b = *reinterpret_cast<const uint4 *>(slab + (32 + l32) * 128 + at);
            const int sa = *reinterpret_cast<const int *>(slab + SLAB + l32 * 8 + 4 * h) >> (8 * w);
            const int sb = *reinterpret_cast<const int *>(slab + SLAB + (32 + l32) * 8 + 4 * h) >> (8 * w);
            const v8i av = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0}, bv = {(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
            acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc, 4, 4, 0, sa, 0, sb);
        }
    }
    __syncthreads(); // every wave has read its last fragments
    float *const red = reinterpret_cast<float *>(lds);
    if (w < 4) {
#pragma unroll
        for (int i = 0; i < 16; ++i) red[(w * 16 + i) * 64 + lane] = acc[i];
    }
    __syncthreads();
    // wave w: accumulator register w
    float v = red[w * 64 + lane];
#pragma unroll
    for (int q = 1; q < 4; ++q) v += red[(q * 16 + w) * 64 + lane];
    const int64_t m = 32ll * bm + (w >> 2) * 8 + h * 4 + (w & 3), n = 32ll * bn + l32;
    if (m < p.rows[0] && n < p.rows[1]) put_c(C + m * p.ldc + n, v);
}

ks_order_t order_of(uint32_t nx, uint32_t ny, uint32_t blocks, int64_t ld) // column tiles x K-blocks, or slices of `blocks` K-blocks
{
    const uint32_t n = nx * ny, per_group = KS_GROUP * ny; // n < 2^24, ny <= 2^13
    const bool plain = nx * blocks <= KS_PLAIN && ld % 64 == 0;
    const uint32_t narrow = plain ? nx : nx % KS_GROUP;
    const uint32_t narrow_magic = narrow > 1 ? (uint32_t)((((uint64_t)1 << 32) + narrow - 1) / narrow) : 0;
    if (plain) return {0, 0, 0, per_group, narrow, narrow_magic, 0};
    return {n >> 3, n & 7, nx / KS_GROUP, per_group, narrow, narrow_magic, (((uint64_t)1 << 44) + per_group - 1) / per_group};
}

// The descriptor of an operand and the kernel kind that takes it.
quant_kind_t describe(const quant_job_t &j, quant_t &q)
{
    const adahop_operand_t &x = *j.x;
    q.x = static_cast<const uint16_t *>(x.data);
    q.outer = x.outer, q.K = x.K, q.ld = x.ld;
    q.zero_outer = j.zero_outer, q.zero_k = j.zero_k;
    q.codes = j.codes, q.scales = j.scales;
    q.key = j.sr_seed ? sr_key_t{(uint32_t)*j.sr_seed, (uint32_t)(*j.sr_seed >> 32)} : sr_key_t{0, 0};
    q.sm = j.sm;
    q.gk = j.gk;
    q.gr = j.gr;
    q.upr = (uint32_t)ceil_div(x.K, 256);
    auto magic_of = [](uint32_t d) { return (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };
    q.magic = magic_of(q.upr);
    q.rows_per_wg = 1, q.gather_blocks = 0;
    q.col_tiles = (uint32_t)ceil_div(x.outer, KS_COLS);
    if (!x.k_contig) {
        q.order = order_of(q.col_tiles, q.upr, q.upr, x.ld);
        if (q.gk.out) q.gather_blocks = (q.col_tiles * (uint32_t)(q.gk.kpad / 64) + 7) & ~7u;
        return KS;
    }
    if (!q.gk.out) return KC;
    const uint32_t fit = 16 / q.upr, room = (uint32_t)(KC_GATHER_MAX_KPAD / q.gk.kpad); // rows per pass, and in LDS
    const uint32_t rows = fit < room ? fit : room;
    if (rows > 1) q.rows_per_wg = rows;
    return KC_GATHER;
}

// Whether row_of_unit is exact for all units of a K-contiguous operand that is taken without a grid of its own (and of K-strided ones: their order
// has divisors of its own).
bool counts_flat(quant_kind_t kind, const quant_t &q) { return kind != KC || (uint64_t)(q.outer * q.upr + 64) * q.upr < (uint64_t)1 << 32; }

// Workgroups of 256 threads that one launch takes (its threads are counted in 32 bits).
constexpr uint64_t MAX_BLOCKS = (1u << 24) - 1;

uint32_t blocks_of(quant_kind_t kind, const quant_t &q)
{
    if (kind == KS) return q.gather_blocks + q.col_tiles * q.upr;
    if (kind == KC_GATHER) return (uint32_t)ceil_div(q.outer, q.rows_per_wg);
    return (uint32_t)ceil_div(q.outer * q.upr, 16);
}

template <int B, bool SR> int launch_one_b(quant_kind_t kind, const quant_t &q, hipStream_t st)
{
    const bool tail = q.K % 256 != 0;
    if (kind == KS) {
        hipLaunchKernelGGL((k_quant_ks16<B, SR>), dim3(blocks_of(KS, q)), dim3(256), 0, st, q);
    } else if (kind == KC_GATHER) {
        const dim3 grid(blocks_of(KC_GATHER, q));
        if (tail)
            hipLaunchKernelGGL((k_quant_kc16_gather<B, SR, true>), grid, dim3(256), 0, st, q);
        else
            hipLaunchKernelGGL((k_quant_kc16_gather<B, SR, false>), grid, dim3(256), 0, st, q);
    } else if ((q.upr == 16 && (tail || q.outer < 1024)) || (SR && q.upr % 16 == 0) || !counts_flat(KC, q)) {
        const dim3 grid((unsigned)q.outer, (unsigned)ceil_div(q.upr, 16));
        if (tail)
            hipLaunchKernelGGL((k_quant_kc16<B, 0, SR, true>), grid, dim3(256), 0, st, q);
        else
            hipLaunchKernelGGL((k_quant_kc16<B, 0, SR, false>), grid, dim3(256), 0, st, q);
    } else {
        const dim3 grid(blocks_of(KC, q));
        if (tail)
            hipLaunchKernelGGL((k_quant_kc16<B, 1, SR, true>), grid, dim3(256), 0, st, q);
        else
            hipLaunchKernelGGL((k_quant_kc16<B, 1, SR, false>), grid, dim3(256), 0, st, q);
    }
    return check_launch();
}

// Elements of a K-contiguous operand up to which the caches keep it (see k_quant_kc16_outliers).
constexpr int64_t KEEP_LONG = 80ll << 20;

template <int B> int launch_outliers_b(quant_kind_t kind, const quant_t &q, const outlier_job_t &e, hipStream_t st)
{
    const dim3 grid(q.col_tiles * (uint32_t)e.nslice + (uint32_t)(e.codes ? e.k : 0));
    auto go = [&](auto tiles) {
        if (kind == KS)
            hipLaunchKernelGGL((k_quant_ks16_outliers<B, decltype(tiles)::value>), grid, dim3(256), 0, st, q, e);
        else if (B < 0 || q.outer * q.ld <= KEEP_LONG)
            hipLaunchKernelGGL((k_quant_kc16_outliers<B, decltype(tiles)::value, true>), grid, dim3(256), 0, st, q, e);
        else if constexpr (B >= 0)
            hipLaunchKernelGGL((k_quant_kc16_outliers<B, decltype(tiles)::value, false>), grid, dim3(256), 0, st, q, e);
        return check_launch();
    };
    switch (e.tiles) {
    case 1: return go(std::integral_constant<int, 1>());
    case 2: return go(std::integral_constant<int, 2>());
    case 3: return go(std::integral_constant<int, 3>());
    case 4: return go(std::integral_constant<int, 4>());
    case 6: return go(std::integral_constant<int, 6>());
    }
    return ADAHOP_E_INVALID_ARG;
}

template <int B> int launch_two_b(quant_kind_t ka, const quant_t &qa, quant_kind_t kb, const quant_t &qb, hipStream_t st)
{
    const uint32_t na = blocks_of(ka, qa), nb = blocks_of(kb, qb);
    auto go = [&](auto a, auto b, auto tail) {
        hipLaunchKernelGGL((k_quant_two<B, decltype(a)::value, decltype(b)::value, decltype(tail)::value>), dim3(na + nb), dim3(256),
                           0, st, qa, qb, na);
    };
    typedef std::integral_constant<quant_kind_t, KC> kc_t;
    typedef std::integral_constant<quant_kind_t, KC_GATHER> kg_t;
    typedef std::integral_constant<quant_kind_t, KS> ks_t;
    auto pick = [&](auto tail) {
        if (ka == KC && kb == KC) go(kc_t(), kc_t(), tail);
        if (ka == KS && kb == KC) go(ks_t(), kc_t(), tail);
        if (ka == KC_GATHER && kb == KC_GATHER) go(kg_t(), kg_t(), tail);
        if (ka == KS && kb == KC_GATHER) go(ks_t(), kg_t(), tail);
    };
    if (ka == KS && kb == KS)
        go(ks_t(), ks_t(), std::false_type()); // (no kernel of a K-strided operand depends on it)
    else if (qa.K % 256)
        pick(std::true_type());
    else
        pick(std::false_type());
    return check_launch();
}

template <quant_kind_t OP, int NT> size_t topk_quant_lds(int dim)
{
    const size_t topk = topk_lds_bytes<NT>(dim), own = OP == KS ? (size_t)KS_LDS : 0;
    return topk > own ? topk : own;
}

template <int B> int launch_two_sr_b(quant_kind_t ka, const quant_t &qa, const quant_t &qb, hipStream_t st)
{
    const uint32_t nb = blocks_of(KS, qb);
    const dim3 grid(blocks_of(ka, qa) + nb);
    if (ka == KS)
        hipLaunchKernelGGL((k_quant_two_sr<B, KS, false>), grid, dim3(256), 0, st, qa, qb, nb);
    else if (qa.K % 256)
        hipLaunchKernelGGL((k_quant_two_sr<B, KC, true>), grid, dim3(256), 0, st, qa, qb, nb);
    else
        hipLaunchKernelGGL((k_quant_two_sr<B, KC, false>), grid, dim3(256), 0, st, qa, qb, nb);
    return check_launch();
}

template <int B, quant_kind_t OP, bool TAIL, int NT> int allow_topk_lds()
{
    return check_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_topk_and_quant<B, OP, TAIL, NT>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)topk_quant_lds<OP, NT>(OP == KC && NT == 512 ? TOPK_BESIDE_DIM_KC : TOPK_BESIDE_DIM)));
}

template <int B> int launch_topk_b(const topk_job_t &t, quant_kind_t kind, const quant_t &q, hipStream_t st)
{
    if (kind == KS) {
        hipLaunchKernelGGL((k_topk_and_quant<B, KS, false, 256>), dim3(1 + blocks_of(kind, q)), dim3(256), (topk_quant_lds<KS, 256>(t.dim)), st, t, q);
        return check_launch();
    }
    auto go = [&](auto tail, auto threads) {
        constexpr int NT = decltype(threads)::value;
        const dim3 grid((unsigned)(1 + ceil_div(q.outer * q.upr, NT / 16)));
        hipLaunchKernelGGL((k_topk_and_quant<B, KC, decltype(tail)::value, NT>), grid, dim3(NT), (topk_quant_lds<KC, NT>(t.dim)), st, t, q);
        return check_launch();
    };
    auto pick = [&](auto tail) {
        return topk_by_512(t.dim, q) ? go(tail, std::integral_constant<int, 512>()) : go(tail, std::integral_constant<int, 256>());
    };
    return q.K % 256 ? pick(std::true_type()) : pick(std::false_type());
}

template <int B> int allow_topk_b()
{
    int rc;
    if ((rc = allow_topk_lds<B, KS, false, 256>()) != ADAHOP_OK || (rc = allow_topk_lds<B, KC, true, 256>()) != ADAHOP_OK ||
        (rc = allow_topk_lds<B, KC, false, 256>()) != ADAHOP_OK || (rc = allow_topk_lds<B, KC, true, 512>()) != ADAHOP_OK)
        return rc;
    return allow_topk_lds<B, KC, false, 512>();
}

#define ADAHOP_DISPATCH(b, CALL)            \
    switch (b) {                            \
    case 0: return CALL(0);                 \
    case 32: return CALL(32);               \
    case 64: return CALL(64);               \
    case 128: return CALL(128);             \
    case 256: return CALL(256);             \
    default: return ADAHOP_E_INVALID_ARG;   \
    }

int launch_one(int b, bool sr, quant_kind_t kind, const quant_t &q, hipStream_t st)
{
#define ADAHOP_ONE(BB) (sr ? launch_one_b<BB, true>(kind, q, st) : launch_one_b<BB, false>(kind, q, st))
    ADAHOP_DISPATCH(b, ADAHOP_ONE)
#undef ADAHOP_ONE
}

int launch_two(int b, quant_kind_t ka, const quant_t &qa, quant_kind_t kb, const quant_t &qb, hipStream_t st)
{
#define ADAHOP_TWO(BB) launch_two_b<BB>(ka, qa, kb, qb, st)
    ADAHOP_DISPATCH(b, ADAHOP_TWO)
#undef ADAHOP_TWO
}
int launch_two_sr(int b, quant_kind_t ka, const quant_t &qa, const quant_t &qb, hipStream_t st)
{
#define ADAHOP_TWO_SR(BB) launch_two_sr_b<BB>(ka, qa, qb, st)
    ADAHOP_DISPATCH(b, ADAHOP_TWO_SR)
#undef ADAHOP_TWO_SR
}
int launch_topk(int b, const topk_job_t &t, quant_kind_t kind, const quant_t &q, hipStream_t st)
{
#define ADAHOP_TOPK(BB) launch_topk_b<BB>(t, kind, q, st)
    ADAHOP_DISPATCH(b, ADAHOP_TOPK)
#undef ADAHOP_TOPK
}
template <typename OUT> int launch_tiles(int b, const tile_product_t &p, OUT *C, hipStream_t st)
{
    const dim3 grid((unsigned)(p.tiles_m * ceil_div(p.rows[1], 32)));
    auto go = [&](auto bb) {
        hipLaunchKernelGGL((k_quant_and_product<decltype(bb)::value, OUT>), grid, dim3(TILE_THREADS), 0, st, p, C);
        return check_launch();
    };
#define ADAHOP_TILES(BB) go(std::integral_constant<int, BB>())
    ADAHOP_DISPATCH(b, ADAHOP_TILES)
#undef ADAHOP_TILES
}
#undef ADAHOP_DISPATCH

} // namespace

// Up to a tile per compute unit and three stages, or two tiles and one stage.  Every tile quantises its rows once more and its stages come one after the
// other, which then costs as much as the launch.  Two launches / one, us, in a queue and (each call waited for): 256 x 512 x 512 (128 tiles)
// 10.0 / 7.0 (20.6 / 18.7), 256 x 1024 x 768 (256) 9.9 / 7.6 (20.7 / 20.6), 512 x 1024 x 256 (512) 9.9 / 7.1 (20.7 / 20.1); beyond the line
// 256 x 1024 x 1024 10.0 / 9.4 (20.7 / 22.2), 512 x 1024 x 512 9.9 / 10.1 (20.7 / 23.1), 1024 x 1024 x 256 10.8 / 12.4.
bool quant_and_product_takes(const quant_job_t &a, const quant_job_t &b)
{
    if (!a.x->k_contig || !b.x->k_contig || a.sr_seed || b.sr_seed) return false;
    const int64_t tiles = ceil_div(a.x->outer, 32) * ceil_div(b.x->outer, 32), K = a.x->K;
    return (tiles <= 256 && K <= 768) || (tiles <= 512 && K <= 256);
}

int launch_quant_and_product(int b, const quant_job_t &ja, const quant_job_t &jb, void *C, int64_t ldc, int c_bf16, hipStream_t st)
{
    const adahop_operand_t &A = *ja.x, &B = *jb.x;
    const tile_product_t p = {{static_cast<const uint16_t *>(A.data), static_cast<const uint16_t *>(B.data)}, {A.ld, B.ld}, {A.outer, B.outer}, A.K,
                              {ja.codes, jb.codes}, {ja.scales, jb.scales}, ldc, (int)ceil_div(A.outer, 32)};
    return c_bf16 ? launch_tiles(b, p, static_cast<uint16_t *>(C), st) : launch_tiles(b, p, static_cast<float *>(C), st);
}

bool iht_quantize_gathers_k(const adahop_operand_t &x, int kpad, bool ascending)
{
    if (!x.k_contig) return ceil_div(x.outer, 64) * (kpad / 64 + ceil_div(x.K, 256)) < (1 << 23); // (workgroups of one launch, both operands)
    return ascending && kpad <= KC_GATHER_MAX_KPAD;
}

bool iht_quantize_takes_outliers(int tiles) { return (tiles >= 1 && tiles <= 4) || tiles == 6; }

int launch_iht_quantize_outliers(int b, const quant_job_t &job, const outlier_job_t &e, hipStream_t st)
{
    quant_t q;
    const quant_kind_t kind = describe(job, q);
    if (kind == KC_GATHER || (b >= 0 && job.sr_seed) || !iht_quantize_takes_outliers(e.tiles)) return ADAHOP_E_INVALID_ARG;
    q.order = order_of(q.col_tiles, (uint32_t)e.nslice, q.upr, q.ld);
    switch (b) {
    case -1: return launch_outliers_b<-1>(kind, q, e, st);
    case 32: return launch_outliers_b<32>(kind, q, e, st);
    case 64: return launch_outliers_b<64>(kind, q, e, st);
    case 128: return launch_outliers_b<128>(kind, q, e, st);
    case 256: return launch_outliers_b<256>(kind, q, e, st);
    }
    return ADAHOP_E_INVALID_ARG;
}

int launch_iht_quantize(int b, const quant_job_t &job, hipStream_t st)
{
    if (job.x->outer == 0 || job.x->K == 0) return ADAHOP_OK;
    quant_t q;
    const quant_kind_t kind = describe(job, q);
    return launch_one(b, job.sr_seed != nullptr, kind, q, st);
}

// Both operands share a launch: what is gained is a launch and its gap, whatever the size.  Whole calls, two launches / one, us: forward, both
// K-contiguous, 8192 x 8192 x 4096 181 / 175.8, 16384 x 8192 x 4096 338 / 335, with 82 K-channels copied out 382 / 379; weight gradient, both
// K-strided, 4096 x 4096 x 16384 197.7 / 190.2, 11008 x 4096 x 8192 243.8 / 241.5; input gradient, one of each, 1024 x 4096 x 11008 67.3 /
// 65.0, 512 x 8192 x 8192 69.4 / 64.6, 8192 x 4096 x 4096 107.8 / 106.  The K-contiguous one of such a pair runs with the registers and the LDS of
// the other's kernel, half as many waves per compute unit, which costs more than the launch where it is large and the other one
// is not: 16384 x 2048 x 4096 111 / 114.
int launch_iht_quantize_two(int b, const quant_job_t &ja, const quant_job_t &jb, hipStream_t st)
{
    quant_t qa, qb;
    const quant_kind_t ka = describe(ja, qa), kb = describe(jb, qb);
    const bool copies_differ = ka != kb && kb != KS && ka != KS; // one K-contiguous operand with its channels copied out, one without
    const bool mixed = (ka == KS) != (kb == KS);
    const int64_t n_kc = (ka == KS ? qb.outer : qa.outer) * qa.K, n_ks = (ka == KS ? qa.outer : qb.outer) * qa.K; // (mixed)
    const bool pays = !mixed || n_kc <= 48ll << 20 || n_kc <= 2 * n_ks;
    if (qa.K == qb.K && pays && !copies_differ && !ja.sr_seed && !jb.sr_seed && counts_flat(ka, qa) && counts_flat(kb, qb) &&
        (uint64_t)blocks_of(ka, qa) + blocks_of(kb, qb) <= MAX_BLOCKS)
        return kb == KS && ka != KS ? launch_two(b, kb, qb, ka, qa, st) : launch_two(b, ka, qa, kb, qb, st);
    if (qa.K == qb.K && (ja.sr_seed != nullptr) != (jb.sr_seed != nullptr)) {
        const bool first = ja.sr_seed != nullptr;
        const quant_kind_t ks = first ? ka : kb, kn = first ? kb : ka;
        const quant_t &qs = first ? qa : qb, &qn = first ? qb : qa;
        if (kn == KS && ks != KC_GATHER && counts_flat(ks, qs) && (uint64_t)blocks_of(ka, qa) + blocks_of(kb, qb) <= MAX_BLOCKS) return launch_two_sr(b, ks, qs, qn, st);
    }
    const int rc = launch_one(b, ja.sr_seed != nullptr, ka, qa, st);
    return rc != ADAHOP_OK ? rc : launch_one(b, jb.sr_seed != nullptr, kb, qb, st);
}

// Every instance of the kernel that selects beside a quantiser, once per device (host-side calls, nothing queued).
int configure_iht_quantize()
{
    static device_once_t once;
    int dev = 0;
    int rc = check_hip(hipGetDevice(&dev));
    if (rc != ADAHOP_OK || !once.need(dev)) return rc;
    if ((rc = allow_topk_b<0>()) != ADAHOP_OK || (rc = allow_topk_b<32>()) != ADAHOP_OK || (rc = allow_topk_b<64>()) != ADAHOP_OK ||
        (rc = allow_topk_b<128>()) != ADAHOP_OK || (rc = allow_topk_b<256>()) != ADAHOP_OK)
        return rc;
    once.mark(dev);
    return ADAHOP_OK;
}

// The selection by 256 threads, the workgroup size of the quantisers, takes up to 15 us in place of the 9 us of 1024 threads (8192
// keys), but then 9 us less of everything else: 9 + 31 -> 16 + 19 us for 8192 x 4096 beside a K-strided 4096 x 4096, 9 + 44 -> 22 +
// 24 for two K-strided operands of 8192 tokens x 4096.  Not for operands that are rounded stochastically (no such instance), and
// above 64 M elements of a K-strided one only where the keys fit into the LDS that every workgroup of the launch has anyway: more of it costs waves in flight.  Whole calls with 1 % of the rows extracted (M x N x K), selection first / beside, the
// other operand K-strided | K-contiguous:
//   8192 x 4096 x 4096 (16 M)    132.8 / 128.4 | 130.4 / 128.2      8192 x  8192 x 8192 (64 M)   380.7 / 372.9 | 373.4 / 375.1
//   4096 x 11008 x 4096 (43 M)   173.6 / 163.0 | 170.6 / 164.7      8192 x 12288 x 8192 (96 M)   511.6 / 504.2 | 502.6 / 509.2
// and columns, 4096 x 4096 x 32768 (128 M, K-strided), 444.5 / 436.1.  With more than 8192 keys two workgroups of 512 threads fit, half the waves of
// the quantiser by itself: beside a K-contiguous operand up to 32 Mi elements, 12288 x 4096 x 4096 167.3 / 162.9, 16384 x 8192 x 4096 380 / 375, up to 64 Mi with rows of a
// workgroup, 16384 x 11008 x 4096 492 / 482 (16384 x 28672 x 4096 1093 / 1102), but 16384 x 4096 x 11008 481 / 512, 16384 x 8192 x 8192 634 / 676, 16384 x 12288 x
// 8192 931 / 1000.  An operand that is done before the selection gains nothing:
// 8192 x 2048 x 2048 71.1 / 69.9 | 67.1 / 69.4.
bool topk_beside_quant(int64_t dim, const quant_job_t &job)
{
    quant_t q;
    const quant_kind_t kind = describe(job, q);
    if (job.sr_seed || kind == KC_GATHER) return false;
    if (kind == KC) return (dim <= TOPK_BESIDE_DIM || (dim <= TOPK_BESIDE_DIM_KC && q.outer * q.K <= (q.K <= 4096 ? 64ll : 32ll) << 20)) && counts_flat(kind, q);
    if (dim > TOPK_BESIDE_DIM) return false;
    const bool fits = topk_lds_bytes<256>((int)dim) <= (size_t)KS_LDS;
    return q.outer * q.K <= (fits ? 1ll << 31 : 64ll << 20);
}

bool iht_quantize_beside_topk(int64_t dim, const adahop_operand_t &x)
{
    return topk_beside_quant(dim, {&x, nullptr, nullptr, nullptr, nullptr, nullptr, {nullptr, 0}, {nullptr, nullptr, 0, 0}, {nullptr, nullptr}});
}

int launch_topk_beside_quant(const topk_job_t &topk, int b, const quant_job_t &job, hipStream_t st)
{
    int rc = configure_iht_quantize();
    if (rc != ADAHOP_OK) return rc;
    quant_t q;
    const quant_kind_t kind = describe(job, q);
    return launch_topk(b, topk, kind, q, st);
}

} // namespace adahop
