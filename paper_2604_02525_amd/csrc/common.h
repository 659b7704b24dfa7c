// Shared host/device helpers of the AdaHOP HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "../../include/adahop.h"

namespace adahop {

// Records the hipError_t of a failed call for adahop_last_hip_error().
void set_last_hip_error(int e);

inline int check_hip(hipError_t e)
{
    if (e == hipSuccess) return ADAHOP_OK;
    set_last_hip_error((int)e);
    return ADAHOP_E_HIP;
}

inline int check_launch() { return check_hip(hipGetLastError()); }

inline bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Argument checks shared by the entry points; all run before any HIP call.
int validate_operand(const adahop_operand_t *x);
bool valid_iht_block(int b);

// One-time set-up per device and kernel family: function attributes (LDS sizes above the default) for every
// instance of the family, and the compute-unit count for the persistent kernels.  Host-side calls only; the
// launchers call them, adahop_prepare_device calls them all.
int configure_gemm_mx(int *ncu_out);
int configure_gemm_mx_dual(int *ncu_out);
int configure_gemm_mx_small();
int configure_oe_rowcol();
int configure_oht();
int configure_foid();
int configure_iht_quantize();

// Launchers (one per kernel family); each validates nothing and returns a status.
// Stage-major copy of the scales for the tiled GEMM kernels [ceil(K/256)][rows][8].
struct scales_sm_t {
    uint8_t *out; // stage-major copy, or nullptr
    int64_t rows; // rows of the operand
};
// The extracted K-channels of an operand, copied out by the quantiser that reads the operand anyway (Eq. 7 with
// S a set of K-channels): out[o, t] = x(o, idx[t]), out[o, k .. kpad) = 0.
// out is [outer, kpad] bf16.
struct k_gather_t {
    const int32_t *idx;
    uint16_t *out;        // nullptr: no copy
    int k, kpad;
};
// The extracted rows of an operand (outer indices), copied out in the same way: out[pos1[o] - 1, :] = x(o, :) for every o with
// pos1[o] != 0, which count as zero in the quantisation.  out is [k, K] bf16.
struct row_gather_t {
    const uint16_t *pos1; // per outer index
    uint16_t *out;        // nullptr: no copy
};
// Whether launch_iht_quantize honours a k_gather_t for this operand: up to 4096 channels of a K-contiguous one, whose list has to ascend.
bool iht_quantize_gathers_k(const adahop_operand_t &x, int kpad, bool ascending);
// One operand to quantise.
struct quant_job_t {
    const adahop_operand_t *x;
    const uint8_t *zero_outer, *zero_k; // byte masks or nullptr; gk goes with the zero_k of the same channels, gr takes the place of zero_outer
    uint8_t *codes, *scales;
    const uint64_t *sr_seed;            // nullptr = round to nearest even; else the elements are rounded stochastically under that seed
    scales_sm_t sm;                     // out = nullptr: no second copy
    k_gather_t gk;
    row_gather_t gr;
};
int launch_iht_quantize(int iht_block, const quant_job_t &job, hipStream_t st);
int launch_iht_quantize_two(int iht_block, const quant_job_t &a, const quant_job_t &b, hipStream_t st); // both of a product
// Both operands of a small product, and the product, in one launch; where quant_and_product_takes them and gemm_mx_splits_stages holds.
bool quant_and_product_takes(const quant_job_t &a, const quant_job_t &b);
int launch_quant_and_product(int iht_block, const quant_job_t &a, const quant_job_t &b, void *C, int64_t ldc, int c_bf16, hipStream_t st);
// One operand of either storage order (nothing extracted from it, rounded to nearest), and on the way its products with the k rows extracted from the
// other one (k_quant_ks16_outliers, k_quant_kc16_outliers): slice s of p is [k, outer] and holds the sums over the 256-element blocks s, s + nslice, ... of K.
struct outlier_job_t {
    const uint16_t *rows; // extracted row t begins at rows + (idx ? idx[t] : t) * ld
    int64_t ld;
    const int32_t *idx;
    float *p;
    int k, tiles, nslice; // tiles: of 16 rows
    // the rows idx[t] of the other operand's codes and scales, to be set to zero (codes = nullptr: they are)
    uint8_t *codes, *scales;
    scales_sm_t sm;
};
constexpr int OUTLIER_TILES = 6; // at most
bool iht_quantize_takes_outliers(int tiles);
// iht_block = -1: the products without the quantisation (see launch_outlier_products).
int launch_iht_quantize_outliers(int iht_block, const quant_job_t &job, const outlier_job_t &e, hipStream_t st);
// The selection from `scores` (launch_foid_scores) in the first workgroup of a launch whose others quantise an operand that does
// not depend on it; topk_beside_quant says whether that can be done.
struct topk_job_t {
    const float *scores;
    int dim, k;
    int32_t *idx;
    uint8_t *mask;
    uint16_t *pos1; // (or nullptr) not where scores lies: a caller finds the scores afterwards
};
bool topk_beside_quant(int64_t dim, const quant_job_t &job);
bool iht_quantize_beside_topk(int64_t dim, const adahop_operand_t &x); // the same for an operand rounded to nearest, no K-channels copied out
int launch_topk_beside_quant(const topk_job_t &topk, int iht_block, const quant_job_t &job, hipStream_t st);
// pos1 (may be nullptr): pos1[c] = t + 1 where c = idx[t], 0 elsewhere, for k <= 0xffff, where foid_writes_positions holds; not where
// scores lies, which a caller finds afterwards.
bool foid_writes_positions(int64_t dim);
int launch_foid_scores(const adahop_operand_t &x, int axis, float *scores, hipStream_t st);
int launch_foid_topk(const adahop_operand_t &x, int axis, int k, int32_t *idx, uint8_t *mask, float *scores,
                     hipStream_t st, uint16_t *pos1 = nullptr);
// Device address, on the current device, of the library's built-in score scratch (ADAHOP_FOID_NOALLOC_MAX_DIM floats).
int foid_static_scores(float **out);
int launch_mask_from_idx(const int32_t *idx, int k, uint8_t *mask, int64_t dim, hipStream_t st);
// OE-K operands for the fused prologue: Ag [M, kpad], Bg [N, kpad] bf16, K-contiguous, zero padded.
int launch_gemm_mx(int64_t M, int64_t N, int64_t K, const uint8_t *a_codes, const uint8_t *a_scales,
                   const uint8_t *b_codes, const uint8_t *b_scales, void *C, int64_t ldc, int c_bf16,
                   const uint16_t *Ag, const uint16_t *Bg, int kpad, void *workspace, hipStream_t st,
                   int sm_ready = 0);
size_t gemm_mx_workspace_bytes(int64_t M, int64_t N, int64_t K);
// The kernels read the scales in a stage-major copy, [ceil(K/256)][rows][8].  A caller that quantises right before the
// product lets the quantiser write that copy as well (scales_sm_t above) and says so with sm_ready (bit 0: A, bit 1: B);
// otherwise launch_gemm_mx re-orders the canonical scales itself where the chosen kernel needs that.
uint8_t *gemm_mx_scales_sm(void *workspace, int64_t M, int64_t K, int which);
// The 256 x 128 kernel with two accumulator sets (gemm_mx_dual.hip): at most 128 gathered K-channels, K > 1792; a bf16 C of whole 4-byte
// pairs (dual_takes_bf16).
bool gemm_mx_dual_eligible(int64_t M, int64_t N, int64_t K, int kpad);
int launch_gemm_mx_dual(int64_t M, int64_t N, int64_t K, const uint8_t *a_codes, const uint8_t *a_sm, const uint8_t *b_codes, const uint8_t *b_sm,
                        void *C, int64_t ldc, int c_bf16, const uint16_t *Ag, const uint16_t *Bg, int kpad, hipStream_t st);
// Rows of C of whole 64-byte pieces: the kernels with tiles of 256 rows then stream C past the caches (see store_tile in gemm_mx.hip).
inline bool c_rows_streamed(const void *C, int64_t row_bytes) { return aligned(C, 64) && row_bytes % 64 == 0; }
inline bool dual_takes_bf16(const void *C, int64_t N, int64_t ldc) { return aligned(C, 4) && ldc % 2 == 0 && N % 2 == 0; }
// Any shape, tiles of 32 .. 128 (gemm_mx_small.hip).  a_sm / b_sm: the scales are the stage-major copy, else the canonical
// array (only for K % 256 == 0 and 4-byte aligned, or where gemm_mx_small_takes_canonical holds).
bool gemm_mx_small_takes_canonical(int64_t K);
int launch_gemm_mx_small(int variant, int64_t M, int64_t N, int64_t K, const uint8_t *a_codes, const uint8_t *a_scales, int a_sm,
                         const uint8_t *b_codes, const uint8_t *b_scales, int b_sm, void *C, int64_t ldc, int c_bf16,
                         const uint16_t *Ag, const uint16_t *Bg, int kpad, hipStream_t st);
int gemm_mx_small_pick(int64_t M, int64_t N, int64_t stages, double *us, int variants = 6); // the variant for a shape and its expected time
// Whether a product of that shape (no K-channels) goes to small tiles whose four waves share the K-elements of a stage: what
// launch_quant_and_product computes has the same bits as that.
bool gemm_mx_splits_stages(int64_t M, int64_t N, int64_t K);
// Diagnostics: 0 = choose by shape, 1 = the 256 x 256 kernel and 2 = the 256 x 128 kernel, each wherever it can run,
// 3 .. 6 = by shape with a forced tile walk, 7 .. 12 = a variant of the kernel with small tiles.
void gemm_mx_force_kernel(int which);
int launch_gather_k(const adahop_operand_t &x, const int32_t *idx, int k, int kpad, uint16_t *out, hipStream_t st);
// C is float[M, ldc], or bf16[M, ldc] when c_bf16 is set (here and in launch_oe_rowcol).
// Row / column outlier product; workspace of oe_rowcol_workspace_bytes() bytes, 256-byte aligned.
size_t oe_rowcol_workspace_bytes(int64_t M, int64_t N, int64_t K, int kind, int k);
// Offset in it of the partial sums, and their size: free until launch_oe_rowcol.
size_t oe_rowcol_partials_at(int64_t M, int64_t N, int64_t K, int kind, int k, size_t *bytes);
// gathered: the extracted rows lie at the start of the workspace already, [k, K] (a quantiser has copied them out).
int launch_oe_rowcol(const adahop_operand_t &A, const adahop_operand_t &B, int kind, const int32_t *idx, int k,
                     void *C, int64_t ldc, int c_bf16, void *workspace, hipStream_t st, bool gathered = false);
// Whether the products of the k rows extracted from S are formed on tiles of L in the quantiser's layout, by L's quantiser or by
// launch_outlier_products: a rule on sizes and layouts alone, the same for every caller, so that a product has the same bits
// whichever of them forms it.  The region of the partial sums above takes outlier_job_t::p.
bool oe_rowcol_on_the_way(const adahop_operand_t &S, const adahop_operand_t &L, int k, outlier_job_t *e);
int launch_outlier_products(const adahop_operand_t &L, const outlier_job_t &e, hipStream_t st); // the products alone
int launch_gather_rows(const adahop_operand_t &x, const int32_t *idx, int k, uint16_t *out, hipStream_t st); // out[t, :] = x(idx[t], :)
// C[idx[t], l] (rows) or C[l, idx[t]] = the sum over the slices of p[slice][t][l], p being [nslice][rows_all][Lo].
int launch_oe_reduce(const float *p, int nslice, int64_t rows_all, int64_t Lo, bool rows, const int32_t *idx, int k, void *C, int64_t ldc,
                     int c_bf16, hipStream_t st);
int launch_oe_k_accumulate(int64_t M, int64_t N, const uint16_t *Ag, const uint16_t *Bg, int kpad, float *C,
                           int64_t ldc, hipStream_t st);

// Outer Hadamard Transform strategy (paper Eq. 6): operand side and the rotations of C after the product.
bool valid_oht_block(int b);
// The OHT kernels put outer / b into the second grid dimension, which may not exceed 65535.
inline bool oht_grid_ok(int64_t outer, int b) { return b > 0 && outer / b <= 65535; }
int launch_oht_quantize(const adahop_operand_t &x, int b, uint8_t *codes, uint8_t *scales, hipStream_t st);
int launch_oht_inverse(float *C, int64_t M, int64_t N, int64_t ldc, int b, hipStream_t st);

size_t pattern_workspace_bytes(const adahop_operand_t &x);
int launch_detect_pattern(const adahop_operand_t &x, double tau, double eps, int32_t *pattern_out, double *stats_out,
                          void *workspace, hipStream_t st);

// One-time set-up per device (function attributes, device properties): the only state the library keeps.
// need(dev) is true until mark(dev) has been called for that device; devices numbered 64 and above are set
// up on every call.
struct device_once_t {
    std::atomic<uint64_t> done{0};
    bool need(int dev) const { return dev < 0 || dev >= 64 || !((done.load(std::memory_order_acquire) >> dev) & 1u); }
    void mark(int dev)
    {
        if (dev >= 0 && dev < 64) done.fetch_or((uint64_t)1 << dev, std::memory_order_release);
    }
};

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

#if defined(__HIPCC__)
// Loads of operand data that a kernel reads exactly once.  They are marked non-temporal (streaming) so that they
// do not displace what the caches hold for the kernels that follow -- above all the packed codes the quantisers
// write, which the product reads next: the product's own prefetch depth (two LDS stages) covers the latency of the
// memory-side cache, not that of HBM under its C-write load.
__device__ __forceinline__ uint4 load_once16(const void *p)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = __builtin_nontemporal_load(static_cast<const u32x4 *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint16_t load_once2(const uint16_t *p) { return __builtin_nontemporal_load(p); }
// The first n of the 8 elements of a 16-byte piece, 1 <= n < 8, zeros behind them: where a matrix of at least 8 elements ends inside the
// piece.  One load of the 8 elements that end there (at 2-byte alignment), moved into place: element by element, the small
// quantisers that have such a piece took a microsecond longer.
__device__ __forceinline__ uint4 load_part16(const uint16_t *p, int n)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(2)));
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p + n - 8));
    const int by = 16 * (8 - n); // bits, 16 .. 112
    const uint64_t lo = (uint64_t)v.y << 32 | v.x, hi = (uint64_t)v.w << 32 | v.z;
    const uint64_t l = by < 64 ? lo >> by | hi << (64 - by) : hi >> (by - 64), h = by < 64 ? hi >> by : 0;
    return make_uint4((uint32_t)l, (uint32_t)(l >> 32), (uint32_t)h, (uint32_t)(h >> 32));
}

// Between what lanes of a wave write to LDS and what other lanes of the same wave read there.  A wave's LDS operations take effect in their
// order, so this is no instruction; but the compiler looks at one lane at a time: without it a lane whose own code did not change what it
// had stored may be handed that on in place of what another lane has put there since.
__device__ __forceinline__ void lds_between_lanes()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The codes and scales of the extracted row idx[t], by a workgroup of 256 threads.
__device__ __forceinline__ void clear_extracted_row(const outlier_job_t &e, int t, int64_t K)
{
    const int64_t o = e.idx[t];
    for (int64_t i = threadIdx.x; i < K / 32; i += 256) {
        *reinterpret_cast<uint4 *>(e.codes + o * (K >> 1) + i * 16) = make_uint4(0, 0, 0, 0);
        e.scales[o * (K >> 5) + i] = 0;
    }
    if (e.sm.out)
        for (int64_t i = threadIdx.x; i < (K + 255) / 256; i += 256) *reinterpret_cast<uint64_t *>(e.sm.out + (i * e.sm.rows + o) * 8) = 0;
}

__device__ __forceinline__ float bf16_lo(uint32_t pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t pair) { return __uint_as_float(pair & 0xffff0000u); }
__device__ __forceinline__ float bf16_one(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
#endif

} // namespace adahop
