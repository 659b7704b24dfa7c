// The BF16 outlier products of Outlier Extraction (second term of paper Eq. 7 and Eq. 8) and the
// gather that feeds the K-channel form.  Operands are the ORIGINAL bf16 values, accumulated in fp32
// on the BF16 matrix cores (v_mfma_f32_32x32x16_bf16).
//
//   OE-row:  C[idx[t], n] = sum_kk A(idx[t], kk) B(n, kk)      for t < k, all n
//   OE-col:  C[m, idx[t]] = sum_kk A(m, kk) B(idx[t], kk)      for all m, t < k
//
// The extracted rows / columns of the residual are zero, so the MXFP4 product left exact zeros in
// these places of C and the sum of Eq. 7 / 8 is a plain overwrite.
#include "common.h"

#include <type_traits>

namespace adahop {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// ------------------------------------------------------------------------------------------------
// Row / column form.  With S the k extracted rows of the "short" operand (A for OE-row, B for
// OE-col) and L the other, "long" operand, both products are  P[t, l] = sum_kk S(idx[t], kk) L(l, kk),
// a skinny product: a few hundred rows against a whole operand, bound by reading L once.
//
//   1. the operand's quantiser (quantize.hip), or k_gather_rows, copies the extracted rows into a K-contiguous staging
//                      matrix Sg of whole 32-row matrix-core tiles; rows past the k extracted ones may hold anything;
//   2. k_oe_skinny     workgroup = (RT x 32 rows of Sg) x (128 NCW rows of L) x (one slice of K), a wave = all the rows
//                      of Sg x 32 NCW rows of L.  Stages of 64 K-elements travel memory -> registers -> LDS; two are
//                      on their way in registers while a third is multiplied from one LDS buffer and a fourth is
//                      being written into the other (one barrier per stage).  Sg and a K-contiguous L lie in LDS
//                      as [row][64 K]; a K-strided L lies there as it lies in memory, [K][128 NCW rows], and the
//                      transposing LDS read hands the matrix cores their 8 consecutive K-elements of a row.  K
//                      is split over workgroups so that the chip is full although there are few tiles; every
//                      slice writes its own partial tile (no atomics: the result does not depend on scheduling);
//      (with at most 96 rows L's quantiser forms the products instead, k_quant_ks16_outliers and k_quant_kc16_outliers, or
//      launch_outlier_products in the same order: oe_rowcol_on_the_way);
//   3. k_oe_reduce     adds the slices in a fixed order and writes the rows / columns of C.
// ------------------------------------------------------------------------------------------------
constexpr int SK_LCOLS = 256;  // rows of L per workgroup (NCW = 2; half of them with NCW = 1)
constexpr int SK_KSTAGE = 64;  // K-elements per pipeline stage
constexpr int SK_PITCH = 72;   // LDS row pitch in bf16 of the [row][64 K] layout (144 bytes: 16-byte fragment
                               // reads of 16 consecutive rows then cover the 64 banks exactly once)
// Pitch in bf16 of the [K][128 NCW rows] layout (576 or 320 bytes: the four K-rows of one transposing read of 32 lanes start
// 16 banks apart), and the elements of a stage of L in either layout.
template <int NCW> constexpr int sk_tpitch() { return NCW == 2 ? 288 : 160; }
template <int NCW> constexpr int sk_l_elems() { return NCW == 2 ? 256 * SK_PITCH : SK_KSTAGE * 160; }
static_assert(sk_l_elems<2>() == SK_KSTAGE * sk_tpitch<2>() && sk_l_elems<1>() >= 128 * SK_PITCH, "either layout fits");

typedef short v4s __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_gather_rows(const uint16_t *__restrict__ x, int64_t ld, int64_t K,
                                                     const int32_t *__restrict__ idx, int k, uint16_t *__restrict__ out)
{ // K-contiguous source: one thread = 8 consecutive K-elements of one row
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x, per_row = K >> 3;
    if (g >= k * per_row) return;
    const int64_t t = g / per_row, c = g - t * per_row;
    *reinterpret_cast<uint4 *>(out + t * K + c * 8) = load_once16(x + (int64_t)idx[t] * ld + c * 8);
}

// K-strided source (element (o, kk) at x[kk * ld + o]): a workgroup takes 64 K-rows x 64 extracted columns.  It reads
// with the extracted column as the fast index, so that a wave's 64 two-byte reads fall into one K-row of the source
// (one DRAM page, neighbouring sectors where the indices are close) instead of 64 rows, turns the tile in LDS and
// writes 128-byte runs along K.
__global__ __launch_bounds__(256) void k_gather_rows_strided(const uint16_t *__restrict__ x, int64_t ld, int64_t K,
                                                             const int32_t *__restrict__ idx, int k,
                                                             uint16_t *__restrict__ out)
{
    __shared__ uint16_t tile[64][66]; // [t][kk], 33-word pitch: the column writes below spread over the banks
    const int64_t kk0 = (int64_t)blockIdx.x * 64;
    const int t0 = blockIdx.y * 64, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int t = t0 + lane;
    const int64_t col = t < k ? idx[t] : -1;
    uint16_t v[16]; // all 16 reads of a thread in flight at once: few workgroups, each bound by its round trips
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int64_t kk = kk0 + 4 * i + w;
        v[i] = (col >= 0 && kk < K) ? load_once2(x + kk * ld + col) : (uint16_t)0;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) tile[lane][4 * i + w] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int tt = 4 * i + w; // row of the tile; the wave's lanes run along K
        if (kk0 + lane < K) out[(int64_t)(t0 + tt) * K + kk0 + lane] = tile[tt][lane];
    }
}

// NCW: column tiles of 32 rows of L per wave.  2, and 1 where the products' workgroups then fill no more than half of the compute
// units (a short L, or a K of few slices): 82 rows x 4096 x 4096 16.4 -> 14.1 us, 82 x 2048 x 2048 13.0 -> 8.8, 41 x 2048 x 8192
// 14.5 -> 11.1, 41 columns x 320 x 4096 10.3 -> 6.9.
// EDGE (K-strided L of a number of rows that is no multiple of 8): the matrix ends inside the last 16-byte piece of its last K-row.  The
// lanes of that piece read the K-row above in its place and write the elements that exist, read one by one at the start.
template <int RT, bool LONG_KC, int NCW, bool EDGE>
__global__ __launch_bounds__(256, 1) void k_oe_skinny(const uint16_t *__restrict__ Sg, const uint16_t *__restrict__ L,
                                                      int64_t ldl, int64_t Lo, int64_t K, int stages_per_slice,
                                                      float *__restrict__ P, int64_t rows_all)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[]; // 2 x (stage of Sg, stage of L)
    constexpr int S_ELEMS = RT * 32 * SK_PITCH, BUF_ELEMS = S_ELEMS + sk_l_elems<NCW>(), SK_TPITCH = sk_tpitch<NCW>();
    constexpr int NL = 4 * NCW, KPP = NCW == 2 ? 8 : 16; // pieces of L per lane and stage; K-rows per pass of a K-strided L
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int64_t l0 = (int64_t)blockIdx.x * (128 * NCW);
    const int nstage_all = (int)((K + SK_KSTAGE - 1) / SK_KSTAGE);
    const int s0 = blockIdx.y * stages_per_slice, s1 = min(s0 + stages_per_slice, nstage_all);
    Sg += (int64_t)blockIdx.z * RT * 32 * K;
    P += ((int64_t)blockIdx.y * rows_all + (int64_t)blockIdx.z * RT * 32) * Lo;

    // loader geometry.  [row][K] sources: 16-byte chunk c8 of rows r32 + 32 i.  K-strided L: chunk c32 (8 rows of
    // L) of K-rows k8 + 8 i (16 i with NCW = 1), so that a wave reads whole pieces of K-rows.  Every address is a base that
    // is the same for the whole workgroup plus a 32-bit byte offset of the lane (the offsets stay below 2^31: at most
    // 256 rows of at most 2^21 elements).  Rows of L past the end are replaced by the last row (their results are
    // not stored); in a last stage of 32 K-elements the upper half reads the lower half again and the Sg side is
    // zero there.
    const int c8 = tid & 7, r32 = tid >> 3, c32 = tid & (16 * NCW - 1), k8 = tid / (16 * NCW);
    const int64_t last_row = Lo - 1 - l0; // >= 0
    const char *const Lb = reinterpret_cast<const char *>(L + (LONG_KC ? l0 * ldl : 0));
    const char *const Sb = reinterpret_cast<const char *>(Sg);
    const uint32_t voff_s = (uint32_t)(((int64_t)r32 * K + c8 * 8) * 2);
    uint32_t voff_l[LONG_KC ? NL : 1];
    if constexpr (LONG_KC) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int64_t r = r32 + 32 * i;
            voff_l[i] = (uint32_t)(((r < last_row ? r : last_row) * ldl + c8 * 8) * 2);
        }
    } else {
        const int64_t l = l0 + 8 * c32, l_last = (Lo - 1) / 8 * 8; // whole 16-byte pieces: ld is a multiple of 8
        voff_l[0] = (uint32_t)(((int64_t)(k8 + EDGE) * ldl) * 2) + (uint32_t)((l < l_last ? l : l_last) * 2);
    }
    static_assert(!(EDGE && LONG_KC), "rows of a K-contiguous operand are whole pieces");
    uint4 end_piece = make_uint4(0, 0, 0, 0);
    int end_row = -1; // the K-row whose piece this lane must not read (selects, no branches: see below)
    if (EDGE && l0 + 8 * c32 >= Lo / 8 * 8) {
        end_piece = load_part16(L + (K - 1) * ldl + Lo / 8 * 8, (int)(Lo & 7));
        end_row = (int)K - 1;
    }
    // whether piece i of a stage is that piece (kk0: the stage's first K-row)
    auto is_end = [&](int64_t kk0, int i) { return (int)kk0 + k8 + (kk0 + SK_KSTAGE > K ? (KPP * i) & 31 : KPP * i) == end_row; };

    // A stage past the end of the slice (the loop below works on pairs of stages) reads the slice's last stage
    // again with the Sg side cleared.  No branches: the loop body stays one block, which the interleaving of
    // memory and matrix-core instructions below relies on.
    // QUARTER = 0 .. 3: the quarter of a stage's loads / LDS writes that is slotted between the matrix-core
    // instructions of K-step QUARTER (rows of L 2 q and 2 q + 1 of the lane's eight, row tiles q and q + 4 of Sg);
    // QUARTER = -1: all of them.
    // (The clearing of the Sg side happens when the registers are written to LDS, stage_keep below: touching a
    // loaded value here would make the wave wait for the load it has just issued.)
    auto stage_keep = [&](int stage) -> uint32_t {
        const bool ghost = stage >= s1;
        const int64_t kk0 = (int64_t)(ghost ? s1 - 1 : stage) * SK_KSTAGE;
        return (ghost || (kk0 + SK_KSTAGE > K && c8 >= 4)) ? 0u : 0xffffffffu;
    };
    auto fetch = [&](int stage, uint4 (&fs)[RT], uint4 (&fl)[NL], auto quarter) {
        constexpr int Q = decltype(quarter)::value;
        const bool ghost = stage >= s1;
        const int64_t kk0 = (int64_t)(ghost ? s1 - 1 : stage) * SK_KSTAGE;
        const bool half = kk0 + SK_KSTAGE > K; // K is a multiple of 32: the last stage may hold 32 K-elements
        const uint32_t back = half && c8 >= 4 ? 64u : 0u;
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            if (Q >= 0 && (i & 3) != Q) continue;
            fs[i] = *reinterpret_cast<const uint4 *>(Sb + ((int64_t)32 * i * K + kk0) * 2 + (voff_s - back));
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            if (Q >= 0 && i / NCW != Q) continue;
            if constexpr (LONG_KC)
                fl[i] = load_once16(Lb + kk0 * 2 + (voff_l[i] - back));
            else
                fl[i] = load_once16(Lb + (kk0 - EDGE + (half ? (KPP * i) & 31 : KPP * i)) * ldl * 2 +
                                    (voff_l[0] - (EDGE && is_end(kk0, i) ? (uint32_t)(2 * ldl) : 0u)));
        }
    };
    auto stash = [&](int stage, uint16_t *buf, const uint4 (&fs)[RT], const uint4 (&fl)[NL], uint32_t keep, auto quarter) {
        constexpr int Q = decltype(quarter)::value;
        uint16_t *sS = buf, *sL = buf + S_ELEMS;
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            if (Q >= 0 && (i & 3) != Q) continue;
            *reinterpret_cast<uint4 *>(sS + (r32 + 32 * i) * SK_PITCH + c8 * 8) =
                make_uint4(fs[i].x & keep, fs[i].y & keep, fs[i].z & keep, fs[i].w & keep);
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            if (Q >= 0 && i / NCW != Q) continue;
            if constexpr (LONG_KC)
                *reinterpret_cast<uint4 *>(sL + (r32 + 32 * i) * SK_PITCH + c8 * 8) = fl[i];
            else
            {
                uint4 v = fl[i];
                if constexpr (EDGE) {
                    const bool end = is_end((int64_t)(stage >= s1 ? s1 - 1 : stage) * SK_KSTAGE, i);
                    v = make_uint4(end ? end_piece.x : v.x, end ? end_piece.y : v.y, end ? end_piece.z : v.z, end ? end_piece.w : v.w);
                }
                *reinterpret_cast<uint4 *>(sL + (k8 + KPP * i) * SK_TPITCH + 8 * c32) = v;
            }
        }
    };
    typedef std::integral_constant<int, -1> all_t;

    v16f acc[RT][NCW];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int c = 0; c < NCW; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][c][r] = 0.0f;

    // As supplier of addresses for the transposing read, lane s of a group of 16 points at 4 consecutive rows of L
    // (4 (s % 4) ..) in K-row s / 4; lane n of the group then receives K-rows 0 .. 3 of row n.  The four groups of a
    // wave are (rows 0-15 | 16-31 of the 32-row tile) x (K-half h) as the matrix cores want them.
    const int tr_elem = ((lane & 15) >> 2) * SK_TPITCH + 32 * NCW * w + 16 * ((lane >> 4) & 1) + 4 * (lane & 3) + 8 * h * SK_TPITCH;

    // One stage: multiply from `cur`; meanwhile write the stage that has arrived in (fs, fl) into `oth` (every wave
    // left that buffer before the last barrier) and refill (fs, fl) with stage `next`.  A wave issues in order and
    // is alone on its SIMD, so whatever is issued in a burst keeps it from feeding the matrix core: the fragment
    // reads of K-step ks + 1, a quarter of the LDS writes and a quarter of the loads are slotted one by one between
    // the matrix-core instructions of K-step ks (scheduling groups), and a scheduling barrier after every K-step
    // keeps the compiler from reading a whole stage's fragments (128 registers) ahead.
    // (fs, fl) hold stage next - 2 on entry.
    auto stage_body = [&](const uint16_t *cur, uint16_t *oth, uint4 (&fs)[RT], uint4 (&fl)[NL], int next) {
        const uint32_t keep = stage_keep(next - 2);
        const uint16_t *sS = cur, *sL = cur + S_ELEMS;
        uint4 a[2][RT];
        v8bf b[2][NCW];
        auto fragments = [&](int ks, uint4 (&fa)[RT], v8bf (&fb)[NCW]) {
#pragma unroll
            for (int c = 0; c < NCW; ++c) {
                if constexpr (LONG_KC) {
                    const uint4 v = *reinterpret_cast<const uint4 *>(sL + (32 * NCW * w + 32 * c + l32) * SK_PITCH + 16 * ks + 8 * h);
                    fb[c] = __builtin_bit_cast(v8bf, v);
                } else {
                    const uint16_t *q = sL + tr_elem + 16 * ks * SK_TPITCH + 32 * c;
                    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)q);
                    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (__attribute__((address_space(3))) v4s *)(q + 4 * SK_TPITCH));
                    typedef short v8s __attribute__((ext_vector_type(8)));
                    const v8s both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                    fb[c] = __builtin_bit_cast(v8bf, both);
                }
            }
#pragma unroll
            for (int i = 0; i < RT; ++i)
                fa[i] = *reinterpret_cast<const uint4 *>(sS + (32 * i + l32) * SK_PITCH + 16 * ks + 8 * h);
        };
        auto step = [&](auto ks_c) {
            constexpr int ks = decltype(ks_c)::value;
            constexpr int n_read = ks + 1 < SK_KSTAGE / 16 ? RT + (LONG_KC ? NCW : 2 * NCW) : 0;
            constexpr int n_move = NCW + (ks < RT ? 1 : 0) + (ks + 4 < RT ? 1 : 0); // LDS writes = loads of this quarter
            if constexpr (ks + 1 < SK_KSTAGE / 16) fragments(ks + 1, a[(ks + 1) & 1], b[(ks + 1) & 1]);
            stash(next - 2, oth, fs, fl, keep, ks_c);
            fetch(next, fs, fl, ks_c);
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int c = 0; c < NCW; ++c)
                    acc[i][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a[ks & 1][i]), b[ks & 1][c],
                                                                        acc[i][c], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < NCW * RT; ++j) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                 // one matrix-core instruction
                if (j < n_read) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); // one LDS read
                if (j < n_move) {
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);             // one LDS write
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);             // one load
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        fragments(0, a[0], b[0]);
        step(std::integral_constant<int, 0>());
        step(std::integral_constant<int, 1>());
        step(std::integral_constant<int, 2>());
        step(std::integral_constant<int, 3>());
    };
    static_assert(SK_KSTAGE == 64, "four K-steps per stage, one quarter of the data movement in each");

    // Register set (stage - s0) & 1 carries a stage from memory to LDS buffer (stage - s0) & 1.  While a stage is
    // multiplied, the next one is written into the other buffer and the two after that are in flight.
    uint4 ps[2][RT], pl[2][NL];
    uint16_t *buf0 = smem, *buf1 = smem + BUF_ELEMS;
    fetch(s0, ps[0], pl[0], all_t());
    fetch(s0 + 1, ps[1], pl[1], all_t());
    stash(s0, buf0, ps[0], pl[0], stage_keep(s0), all_t());
    fetch(s0 + 2, ps[0], pl[0], all_t());
    __syncthreads();
    for (int stage = s0; stage < s1; stage += 2) { // no branch around a multiply: the accumulators stay where they are
        stage_body(buf0, buf1, ps[1], pl[1], stage + 3);
        __syncthreads();
        stage_body(buf1, buf0, ps[0], pl[0], stage + 4);
        __syncthreads();
    }

#pragma unroll
    for (int c = 0; c < NCW; ++c) {
        const int64_t l = l0 + 32 * NCW * w + 32 * c + l32;
        if (l < Lo) {
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    P[(int64_t)(32 * i + (r >> 2) * 8 + h * 4 + (r & 3)) * Lo + l] = acc[i][c][r];
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The same products with a K-strided L by themselves, in the order of its quantiser (k_quant_ks16_outliers), so that a product has the same bits
// whether L is quantised in the call or not: slice s holds the 256-element blocks s, s + nslice, ... of K, and matrix-core
// instruction i of a block (v_mfma_f32_16x16x32_bf16) the K-elements 64 g + 8 i .. + 7, g = 0 .. 3 (the groups of 16 lanes).
// Bound by reading L.  Workgroup = 32 R extracted rows x 64 CT rows of L x one slice, a wave = all the extracted rows x 16 CT rows of L.
//   L travels in stages of 64 K-elements as in k_oe_skinny: two on their way in registers, one in the LDS buffer that is multiplied, one
//   being written into the other.  Stage s of a block holds what instructions 2 s and 2 s + 1 take, the K-rows 64 g + 16 s .. + 15.  K-row
//   r = 16 g + 8 u + 4 h + j of it (u: which instruction, j < 4) lies at row j + 4 (g & 1) + 8 h + 16 u + 32 (g >> 1) of the buffer, pieces of 32
//   bytes exchanged by the row's low three bits: the eight K-rows that a transposing read of 32 lanes touches lie in different eighths of the banks.
//   The extracted rows' 256 K-elements of a block lie in LDS as in the quantiser; those of the next block arrive with the four stages, a
//   quarter of the rows each, so that whole lines are read (28672 x 8192, 64 rows, whole call with 96 rows of the other operand: 142 us, with the 32 bytes
//   of a row that each stage needs 160; k_oe_skinny, which adds in another order, 137).
// With slices that do not fill the chip evenly k_oe_skinny, which splits K as suits it, is up to a quarter faster in such a call (20000 x 4096, 40 rows, 63.5 / 78.6;
// 4096 x 32768, 40 rows, 107 / 110; 12288 x 8192, 64 rows, 73 / 78); bits that do not depend on who packs an operand are worth that.
// ------------------------------------------------------------------------------------------------
template <int CT> constexpr int op_l_bytes() { return 64 * 128 * CT; }
template <int R> constexpr int op_s_bytes() { return R * 16384; }
template <int R, int CT> constexpr int op_lds_bytes() { return 2 * (op_l_bytes<CT>() + op_s_bytes<R>()); }
typedef float v4f __attribute__((ext_vector_type(4)));

template <int R, int CT, bool EDGE>
__global__ __launch_bounds__(256, CT == 4 || R == 3 ? 1 : 2) void k_outlier_products(const uint16_t *__restrict__ L, int64_t ldl, int64_t Lo, int64_t K,
                                                                                     outlier_job_t e, int col_groups)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t op_smem[]; // 2 stages of L, 2 blocks of the extracted rows
    constexpr int NL = 2 * CT, KPP = 32 / CT; // pieces of L per lane and stage, K-rows per pass of the workgroup
    constexpr int LB = op_l_bytes<CT>(), SB = op_s_bytes<R>(), PITCH = 128 * CT;
    static_assert(CT == 2 || CT == 4, "a pass lies within one group of 16 K-rows");
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int tiles = col_groups * e.nslice;
    if ((int)blockIdx.x >= tiles) {
        clear_extracted_row(e, (int)blockIdx.x - tiles, K);
        return;
    }
    const int slice = (int)blockIdx.x / col_groups;
    const int64_t l0 = (int64_t)((int)blockIdx.x - slice * col_groups) * (64 * CT);
    const int nblock = ((int)((K + 255) / 256) - slice + e.nslice - 1) / e.nslice;
    auto block_at = [&](int blk) { return (int64_t)(slice + e.nslice * (blk < nblock ? blk : nblock - 1)) * 256; }; // (behind the last one: loaded, not used)

    // Loader of the extracted rows: piece c32 (8 K-elements) of rows 8 R q + r8 + 8 i in quarter q; rows past the last by that one (not stored).
    const int c32 = tid & 31, r8 = tid >> 5;
    int row_no[4][R];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int t = min(8 * (R * q + i) + r8, e.k - 1);
            row_no[q][i] = e.idx ? e.idx[t] : t;
        }
    auto fetch_s = [&](int blk, const int (&rows)[R], uint4 (&fs)[R]) {
        const int64_t k0 = block_at(blk), k = k0 + 8 * c32;
        const uint16_t *const at = e.rows + (k < K ? k : k0);
#pragma unroll
        for (int i = 0; i < R; ++i) fs[i] = *reinterpret_cast<const uint4 *>(at + (int64_t)rows[i] * e.ld);
    };
    // tile rt of 16 rows as 8 x 64 pieces, row r of it at r ^ (8 (g & 1) + i): see k_quant_ks16_outliers
    const int s_at = (c32 & 7) * 64 + (c32 >> 3) * 16, s_x = c32 & 15;
    auto stash_s = [&](int blk, auto quarter, uint8_t *buf, const uint4 (&fs)[R]) {
        constexpr int Q = decltype(quarter)::value;
        const uint32_t keep = block_at(blk) + 8 * c32 < K ? ~0u : 0u;
        uint4 *const s = reinterpret_cast<uint4 *>(buf);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            constexpr int first = R * Q;
            const int n = first + i; // rows 8 n + r8
            s[(n >> 1) * 512 + s_at + ((r8 + 8 * (n & 1)) ^ s_x)] = make_uint4(fs[i].x & keep, fs[i].y & keep, fs[i].z & keep, fs[i].w & keep);
        }
    };

    // Loader of L: 16-byte piece cl of the K-rows kl + KPP i.  Rows of L past the end are replaced by the last piece (not stored).
    const int cl = tid & (8 * CT - 1), kl = tid / (8 * CT);
    const int64_t l = l0 + 8 * cl, l_last = (Lo - 1) / 8 * 8; // whole 16-byte pieces: ld is a multiple of 8
    const uint16_t *const lrow = L + (int64_t)kl * ldl + (l < l_last ? l : l_last);
    uint4 end_piece = make_uint4(0, 0, 0, 0);
    int end_row = -1; // the K-row whose piece this lane must not read whole
    if (EDGE && l >= Lo / 8 * 8) {
        end_piece = load_part16(L + (K - 1) * ldl + Lo / 8 * 8, (int)(Lo & 7));
        end_row = (int)K - 1;
    }
    // Pass i of stage s: K-rows pass(s, i) + ... of the block; behind the end of K the block's first ones, which exist, in their place, and zeros on
    // both sides: an infinity there must not meet one of those zeros.
    auto pass = [](int s, int i) { return 16 * s + 64 * (CT == 4 ? i >> 1 : i); };
    auto row_of = [&](int64_t k0, int s, int i) { return (k0 + pass(s, i) < K ? k0 + pass(s, i) : k0) + (CT == 4 ? 8 * (i & 1) : 0); };
    auto fetch_l = [&](int blk, int s, int half, uint4 (&fl)[NL]) {
        const int64_t k0 = block_at(blk);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            if (half >= 0 && i / CT != half) continue;
            const int64_t row = row_of(k0, s, i);
            fl[i] = load_once16(lrow + (row - (EDGE && (int)row + kl == end_row ? 1 : 0)) * ldl);
        }
    };
    const int l_unit = (cl >> 1) ^ (kl & 3);
    auto stash_l = [&](int blk, int s, int half, uint8_t *buf, const uint4 (&fl)[NL]) {
        const int64_t k0 = block_at(blk);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            if (half >= 0 && i / CT != half) continue;
            const uint32_t keep = k0 + pass(s, i) < K ? ~0u : 0u;
            uint4 v = fl[i];
            if constexpr (EDGE) {
                const bool end = (int)row_of(k0, s, i) + kl == end_row;
                v = make_uint4(end ? end_piece.x : v.x, end ? end_piece.y : v.y, end ? end_piece.z : v.z, end ? end_piece.w : v.w);
            }
            const int g4 = 4 * (CT == 4 ? (i >> 1) & 1 : i & 1); // 4 (g & 1)
            const int row = CT == 4 ? (kl & 3) + 8 * (kl >> 2) + 16 * (i & 1) + g4 + 32 * (i >> 2)
                                    : (kl & 3) + 8 * ((kl >> 2) & 1) + 16 * (kl >> 3) + g4 + 32 * (i >> 1);
            *reinterpret_cast<uint4 *>(buf + row * PITCH + (l_unit ^ g4) * 32 + 16 * (cl & 1)) = make_uint4(v.x & keep, v.y & keep, v.z & keep, v.w & keep);
        }
    };

    v4f acc[2 * R][CT];
#pragma unroll
    for (int i = 0; i < 2 * R; ++i)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[i][c] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

    // As supplier of addresses for the transposing read, lane s of a group of 16 points at 4 neighbouring rows of L (4 (s % 4) ..) in
    // K-row s / 4; lane n of the group receives K-rows 0 .. 3 of row n.
    const int x7 = (l16 >> 2) + 4 * (g & 1), tr = (x7 + 32 * (g >> 1)) * PITCH + 8 * (l16 & 3);
    int tr_unit[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) tr_unit[c] = tr + ((CT * w + c) ^ x7) * 32;
    const int s_read = 16 * g, s_row = l16 ^ (8 * (g & 1));

    uint4 ps[2][R], pl[2][NL];
    uint8_t *const lbuf = op_smem, *const sbuf = op_smem + 2 * LB;

    // Stage s of block blk: multiply; meanwhile write the next stage of L, which has arrived in set (s + 1) & 1, into the other buffer and refill
    // the set with the third one from here, and write quarter s of the next block's extracted rows, and refill its set with the quarter after the next.
    auto stage = [&](auto s_c, int blk) {
        constexpr int s = decltype(s_c)::value;
        const uint8_t *const cur = lbuf + (s & 1) * LB;
        uint8_t *const oth = lbuf + (1 - (s & 1)) * LB;
        const uint4 *const rows = reinterpret_cast<const uint4 *>(sbuf + (blk & 1) * SB);
        uint4 (&fl)[NL] = pl[(s + 1) & 1];
        uint4 (&fs)[R] = ps[s & 1];
        uint4 a[2][2 * R];
        v8bf b[2][CT];
        auto fragments = [&](int u) {
            const int i = 2 * s + u;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const uint8_t *q = cur + tr_unit[c] + 16 * u * PITCH;
                const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)q);
                const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)(q + 8 * PITCH));
                typedef short v8s __attribute__((ext_vector_type(8)));
                const v8s both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                b[u][c] = __builtin_bit_cast(v8bf, both);
            }
#pragma unroll
            for (int rt = 0; rt < 2 * R; ++rt) a[u][rt] = rows[rt * 512 + i * 64 + s_read + (s_row ^ i)];
        };
        auto step = [&](auto u_c) {
            constexpr int u = decltype(u_c)::value;
            constexpr int n_read = u == 0 ? 2 * R + 2 * CT : 0, n_move = CT + (u == 1 ? R : 0), N = 2 * R * CT;
            constexpr int reads = (n_read + N - 1) / N, moves = (n_move + N - 1) / N; // behind one instruction
            if constexpr (u == 0) fragments(1);
            stash_l(blk + (s == 3), (s + 1) & 3, u, oth, fl);
            fetch_l(blk + (s >= 1), (s + 3) & 3, u, fl);
            if constexpr (u == 1) {
                stash_s(blk + 1, s_c, sbuf + ((blk + 1) & 1) * SB, fs);
                fetch_s(blk + 1 + (s >= 2), row_no[(s + 2) & 3], fs);
            }
#pragma unroll
            for (int i = 0; i < 2 * R; ++i)
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    acc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a[u][i]), b[u][c], acc[i][c], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < N; ++j) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                             // one matrix-core instruction
                if (j * reads < n_read) __builtin_amdgcn_sched_group_barrier(0x100, reads, 0); // LDS reads
                if (j * moves < n_move) {
                    __builtin_amdgcn_sched_group_barrier(0x200, moves, 0);                     // LDS writes
                    __builtin_amdgcn_sched_group_barrier(0x020, moves, 0);                     // loads
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        fragments(0);
        step(std::integral_constant<int, 0>());
        step(std::integral_constant<int, 1>());
        __syncthreads();
    };

    fetch_l(0, 0, -1, pl[0]);
    fetch_l(0, 1, -1, pl[1]);
    {
        uint4 f[4][R];
#pragma unroll
        for (int q = 0; q < 4; ++q) fetch_s(0, row_no[q], f[q]);
        fetch_s(1, row_no[0], ps[0]);
        fetch_s(1, row_no[1], ps[1]);
        stash_l(0, 0, -1, lbuf, pl[0]);
        fetch_l(0, 2, -1, pl[0]);
        stash_s(0, std::integral_constant<int, 0>(), sbuf, f[0]);
        stash_s(0, std::integral_constant<int, 1>(), sbuf, f[1]);
        stash_s(0, std::integral_constant<int, 2>(), sbuf, f[2]);
        stash_s(0, std::integral_constant<int, 3>(), sbuf, f[3]);
    }
    __syncthreads();
    for (int blk = 0; blk < nblock; ++blk) {
        stage(std::integral_constant<int, 0>(), blk);
        stage(std::integral_constant<int, 1>(), blk);
        stage(std::integral_constant<int, 2>(), blk);
        stage(std::integral_constant<int, 3>(), blk);
    }
    float *p = e.p + (int64_t)slice * e.k * Lo;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int64_t o = l0 + 16 * CT * w + 16 * c + l16;
        if (o < Lo) {
#pragma unroll
            for (int i = 0; i < 2 * R; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int t = 16 * i + 4 * g + r;
                    if (t < e.k) p[(int64_t)t * Lo + o] = acc[i][c][r];
                }
        }
    }
}

// The same for a K-contiguous L, in the order of k_quant_kc16_outliers: slices as above, a block's K-elements in ascending chunks of 32, one instruction
// each.  Bound by reading L, and by the extracted rows beside it where they are many (12288 x 8192, 90 rows, 128 rows of L per workgroup: 66 us, 50 without its loads of L).
//   Workgroup = T tiles of 16 extracted rows x 64 CT rows of L x one slice, a wave = all the extracted rows x 16 CT rows of L.
//   L goes from memory to the matrix cores' operands without the LDS.  A load takes whole lines, 8 rows x 64 K-elements: lane 16 g + 8 u + r piece 4 u + g of
//   row r.  Of two of them, rows 0 .. 7 and 8 .. 15 of a tile, an exchange of the lanes 8 apart makes the operands of two instructions, u = 0 and 1.  Two chunks of 64
//   K-elements are on their way in registers while a third is multiplied (four: 16384 x 4096, 64 rows, 39 -> 44 us; through the LDS as in k_oe_skinny: the same,
//   9152 x 16672, 2 rows, 72 / 66).
//   The extracted rows travel in stages of 128 K-elements through two buffers, one barrier per stage; in a buffer as 4 x 64 pieces for each 16 rows, as in
//   the quantiser.
//   A tile's slices are neighbours on an XCD, as in the quantiser, and each XCD begins its run of the workgroups three tiles further than the one before: begun alike,
//   the XCDs read a power of two apart (16384 x 4096, 10 rows 35.7 -> 30.5 us, 64 rows 47 -> 40; 8192 x 8192 29.6 -> 27.7).
constexpr int OPK_STAGE = 128;

template <int T, int CT>
__global__ __launch_bounds__(256, 2) void k_outlier_products_kc(const uint16_t *__restrict__ L, int64_t ldl, int64_t Lo, int64_t K, outlier_job_t e, int row_groups)
{
    constexpr int NS = 2 * ((T + 1) / 2), SB = OPK_STAGE * 2 * 16 * NS; // pieces of the extracted rows per lane and stage; bytes of a stage
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * SB];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int tiles = row_groups * e.nslice;
    if ((int)blockIdx.x >= tiles) {
        clear_extracted_row(e, (int)blockIdx.x - tiles, K);
        return;
    }
    const int xcd = blockIdx.x & 7, rest = tiles & 7, run = (tiles >> 3) + (xcd < rest ? 1 : 0);
    const int at = xcd * (tiles >> 3) + min(xcd, rest) + (((int)blockIdx.x >> 3) + 3 * e.nslice * xcd) % run;
    const int group = at / e.nslice, slice = at - group * e.nslice;
    const int64_t l0 = (int64_t)group * (64 * CT) + 16 * CT * w;
    const int nblock = ((int)((K + 255) / 256) - slice + e.nslice - 1) / e.nslice;
    const int64_t last = (int64_t)(slice + e.nslice * (nblock - 1)) * 256;
    const int nstage = 2 * (nblock - 1) + (K - last > OPK_STAGE ? 2 : 1);
    auto k_of = [&](int chunk) { return (int64_t)(slice + e.nslice * (chunk >> 2)) * 256 + 64 * (chunk & 3); }; // (behind the slice's last block: past the end of K)

    // Rows past the last one by that one (not stored).
    const uint16_t *lrows[2 * CT];
    const int lk = 32 * (lane >> 3 & 1) + 8 * g;
#pragma unroll
    for (int i = 0; i < 2 * CT; ++i) lrows[i] = L + min(l0 + 8 * i + (lane & 7), Lo - 1) * ldl;
    // (past the end of K: the row's first piece, which exists, and zeros on both sides: an infinity there must not meet one of those zeros)
    auto fetch_l = [&](int chunk, uint4 (&f)[2 * CT]) {
        const int64_t k = k_of(chunk) + lk, there = k < K ? k : 0;
#pragma unroll
        for (int i = 0; i < 2 * CT; ++i) f[i] = load_once16(lrows[i] + there);
    };
    // Piece sc of the rows sr + 16 i.
    const int sc = tid & 15, sr = tid >> 4;
    const uint16_t *srows[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int t = min(sr + 16 * i, e.k - 1);
        srows[i] = e.rows + (e.idx ? e.idx[t] : t) * e.ld;
    }
    uint4 ps[NS];
    auto fetch_s = [&](int stage) {
        const int64_t k = k_of(2 * stage) + 8 * sc, there = k < K ? k : 0;
#pragma unroll
        for (int i = 0; i < NS; ++i) ps[i] = *reinterpret_cast<const uint4 *>(srows[i] + there);
    };
    auto stash_s = [&](int stage) {
        const uint32_t keep = k_of(2 * stage) + 8 * sc < K ? ~0u : 0u;
        uint4 *const s = reinterpret_cast<uint4 *>(lds + (stage & 1) * SB) + (sc >> 2) * 64 + (sc & 3) * 16 + (sr ^ sc);
#pragma unroll
        for (int i = 0; i < NS; ++i) s[i * 256] = make_uint4(ps[i].x & keep, ps[i].y & keep, ps[i].z & keep, ps[i].w & keep);
    };

    v4f acc[T][CT];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[i][c] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    uint4 set[2][2 * CT];
    v8bf a[2][T], b[2][CT];

    // Half h of a stage: chunk 2 stage + h, which has arrived in set h; the set is refilled with the chunk after the next one.
    auto half = [&](auto h_c, int stage) {
        constexpr int h = decltype(h_c)::value;
        const uint4 *const rows = reinterpret_cast<const uint4 *>(lds + (stage & 1) * SB) + 16 * g;
        auto fragments = [&](int i) { // instruction i of the stage
#pragma unroll
            for (int t = 0; t < T; ++t) a[i & 1][t] = __builtin_bit_cast(v8bf, rows[t * 256 + i * 64 + (l16 ^ (4 * i + g))]);
        };
        if constexpr (h == 0) fragments(0);
        const uint32_t keep = k_of(2 * stage + h) + lk < K ? ~0u : 0u;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const uint4 p = set[h][2 * c], q = set[h][2 * c + 1];
            const uint32_t lo[4] = {p.x & keep, p.y & keep, p.z & keep, p.w & keep}, hi[4] = {q.x & keep, q.y & keep, q.z & keep, q.w & keep};
            uint32_t v[2][4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { // (row_ror:8, into the lanes 8 .. 15 or 0 .. 7 of each 16)
                v[0][j] = __builtin_amdgcn_update_dpp(lo[j], hi[j], 0x128, 0xf, 0xc, false);
                v[1][j] = __builtin_amdgcn_update_dpp(hi[j], lo[j], 0x128, 0xf, 0x3, false);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) b[u][c] = __builtin_bit_cast(v8bf, make_uint4(v[u][0], v[u][1], v[u][2], v[u][3]));
        }
        fetch_l(2 * stage + h + 2, set[h]);
        if constexpr (h == 1) {
            stash_s(stage + 1);
            fetch_s(stage + 2);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = 2 * h + u;
            if (i < 3) fragments(i + 1);
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int c = 0; c < CT; ++c) acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i & 1][t], b[u][c], acc[t][c], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // (in this order, and into a loop that is entered without a condition: its waits count the loads behind the one that is needed, on either way into it)
    fetch_s(0);
    __builtin_amdgcn_sched_barrier(0);
    fetch_l(0, set[0]);
    __builtin_amdgcn_sched_barrier(0);
    fetch_l(1, set[1]);
    __builtin_amdgcn_sched_barrier(0);
    stash_s(0);
    fetch_s(1);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    int stage = 0;
    do {
        half(std::integral_constant<int, 0>(), stage);
        half(std::integral_constant<int, 1>(), stage);
        __syncthreads();
    } while (++stage < nstage);
    float *p = e.p + (int64_t)slice * e.k * Lo;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int64_t o = l0 + 16 * c + l16;
        if (o < Lo) {
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int t = 16 * i + 4 * g + r;
                    if (t < e.k) p[(int64_t)t * Lo + o] = acc[i][c][r];
                }
        }
    }
}

// C[idx[t], l] (ROWS) or C[l, idx[t]] = sum over the K slices of P[s][t][l], in slice order.
// C holds float, or bf16 as its 16 bits (rounded to nearest even from the fp32 sum).
template <bool ROWS, typename OUT>
__global__ __launch_bounds__(256) void k_oe_reduce(const float *__restrict__ P, int nslice, int64_t rows_all, int64_t Lo,
                                                   const int32_t *__restrict__ idx, int k, OUT *__restrict__ C, int64_t ldc)
{
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= (int64_t)k * Lo) return;
    const int64_t t = g / Lo, l = g - t * Lo;
    float s = 0.0f;
    for (int i = 0; i < nslice; ++i) s += P[((int64_t)i * rows_all + t) * Lo + l];
    const int64_t o = idx[t];
    OUT v;
    if constexpr (sizeof(OUT) == 4) {
        v = s;
    } else {
        const uint32_t u = __float_as_uint(s);
        v = (OUT)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
    }
    if (ROWS)
        C[o * ldc + l] = v;
    else
        C[l * ldc + o] = v;
}

// The same on 4 consecutive long-side indices per thread (Lo % 4 == 0; for ROWS also 16-byte / 8-byte aligned rows of
// C): 16-byte reads of the partials, and for ROWS one 16-byte (fp32) or 8-byte (bf16) store.
// Bound by latency: a few waves per compute unit at most.  Eight slices are in flight at a time and added in slice order: 41 columns
// x 8192 tokens (16 slices of 4096) 13.0 -> 9.6 us, 21 rows x 4096 7.6 -> 5.4, 64 columns x 4096 14.1 -> 11.0.  What is left
// for columns is the stores, one sector of C each.
__device__ __forceinline__ uint16_t bf16_rne(float s)
{
    const uint32_t u = __float_as_uint(s);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

template <bool ROWS, typename OUT>
__global__ __launch_bounds__(256) void k_oe_reduce4(const float *__restrict__ P, int nslice, int64_t rows_all, int64_t Lo,
                                                    const int32_t *__restrict__ idx, int k, OUT *__restrict__ C, int64_t ldc)
{
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x, per = Lo >> 2;
    if (g >= (int64_t)k * per) return;
    const int64_t t = g / per, l = (g - t * per) * 4;
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const int64_t o = idx[t];
    const float *p = P + t * Lo + l;
    const int64_t slice = rows_all * Lo;
    int i = 0;
    for (; i + 8 <= nslice; i += 8) {
        float4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const float4 *>(p + (i + j) * slice);
#pragma unroll
        for (int j = 0; j < 8; ++j) s.x += v[j].x, s.y += v[j].y, s.z += v[j].z, s.w += v[j].w;
    }
    for (; i < nslice; ++i) {
        const float4 v = *reinterpret_cast<const float4 *>(p + i * slice);
        s.x += v.x, s.y += v.y, s.z += v.z, s.w += v.w;
    }
    if constexpr (ROWS) {
        if constexpr (sizeof(OUT) == 4) {
            *reinterpret_cast<float4 *>(C + o * ldc + l) = s;
        } else {
            const uint32_t lo = (uint32_t)bf16_rne(s.x) | ((uint32_t)bf16_rne(s.y) << 16);
            const uint32_t hi = (uint32_t)bf16_rne(s.z) | ((uint32_t)bf16_rne(s.w) << 16);
            *reinterpret_cast<uint2 *>(C + o * ldc + l) = make_uint2(lo, hi);
        }
    } else {
        const float e[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (sizeof(OUT) == 4)
                C[(l + j) * ldc + o] = e[j];
            else
                C[(l + j) * ldc + o] = bf16_rne(e[j]);
        }
    }
}

struct skinny_plan_t {
    int rt, groups, nslice, stages_per_slice, ncw;
    int64_t rows_all;
    size_t sg_bytes, p_bytes;
};

// Row tiles per workgroup from {2, 4, 6}; K slices so that up to one workgroup per compute unit exists, each
// with at least 8 stages.
skinny_plan_t plan_skinny(int64_t Lo, int64_t K, int k)
{
    skinny_plan_t p;
    const int tiles = (k + 31) / 32;
    p.groups = (tiles + 5) / 6; // every group of row tiles reads L once: as few as possible
    p.rt = 6;
    for (int rt = 4; rt >= 2; rt -= 2)
        if ((tiles + rt - 1) / rt == p.groups) p.rt = rt; // the same passes with less padding
    p.rows_all = (int64_t)p.groups * p.rt * 32;
    const int64_t nstage = ceil_div(K, SK_KSTAGE), wgs = ceil_div(Lo, SK_LCOLS) * p.groups;
    int64_t want = 256 / wgs; // one workgroup per compute unit is resident; never more than that many: a second,
                              // partly filled round costs more than idle compute units do
    if (want > nstage / 8) want = nstage / 8;
    if (want < 1) want = 1;
    auto slice = [&](int64_t n) {
        p.stages_per_slice = (int)ceil_div(nstage, n);
        p.nslice = (int)ceil_div(nstage, p.stages_per_slice);
    };
    slice(want);
    p.sg_bytes = align_up((size_t)p.rows_all * K * 2, 256);
    p.p_bytes = align_up((size_t)p.nslice * p.rows_all * Lo * 4, 256);
    p.ncw = 2;
    if (wgs * want <= 128) { // half of L per workgroup; never more slices (and scratch) than with the whole of it
        p.ncw = 1;
        const int64_t most = 256 / (ceil_div(Lo, SK_LCOLS / 2) * p.groups);
        if (want > most) slice(most < 1 ? 1 : most);
    }
    return p;
}

template <int RT, int NCW> constexpr size_t skinny_lds_bytes() { return 2 * (RT * 32 * SK_PITCH + sk_l_elems<NCW>()) * sizeof(uint16_t); }

template <int RT, bool LONG_KC, int NCW, bool EDGE> int allow_skinny_lds()
{
    return check_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_oe_skinny<RT, LONG_KC, NCW, EDGE>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)skinny_lds_bytes<RT, NCW>()));
}

template <int RT, int NCW> int allow_skinny_lds_all()
{
    int rc;
    if ((rc = allow_skinny_lds<RT, true, NCW, false>()) != ADAHOP_OK || (rc = allow_skinny_lds<RT, false, NCW, false>()) != ADAHOP_OK) return rc;
    return allow_skinny_lds<RT, false, NCW, true>();
}

template <int RT, int NCW>
int launch_skinny_as(bool long_kc, dim3 grid, hipStream_t st, const uint16_t *Sg, const uint16_t *L, int64_t ldl, int64_t Lo, int64_t K,
                     int sps, float *P, int64_t rows_all)
{
    const int rc = configure_oe_rowcol(); // more LDS than a launch may ask for by default: allowed once per device
    if (rc != ADAHOP_OK) return rc;
    constexpr size_t lds = skinny_lds_bytes<RT, NCW>();
    if (long_kc)
        hipLaunchKernelGGL((k_oe_skinny<RT, true, NCW, false>), grid, dim3(256), lds, st, Sg, L, ldl, Lo, K, sps, P, rows_all);
    else if (Lo % 8 == 0)
        hipLaunchKernelGGL((k_oe_skinny<RT, false, NCW, false>), grid, dim3(256), lds, st, Sg, L, ldl, Lo, K, sps, P, rows_all);
    else
        hipLaunchKernelGGL((k_oe_skinny<RT, false, NCW, true>), grid, dim3(256), lds, st, Sg, L, ldl, Lo, K, sps, P, rows_all);
    return check_launch();
}

template <int RT>
int launch_skinny(bool long_kc, int ncw, dim3 grid, hipStream_t st, const uint16_t *Sg, const uint16_t *L, int64_t ldl, int64_t Lo,
                  int64_t K, int sps, float *P, int64_t rows_all)
{
    return ncw == 1 ? launch_skinny_as<RT, 1>(long_kc, grid, st, Sg, L, ldl, Lo, K, sps, P, rows_all)
                    : launch_skinny_as<RT, 2>(long_kc, grid, st, Sg, L, ldl, Lo, K, sps, P, rows_all);
}

template <int R, int CT> int allow_products_lds()
{
    const int rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_outlier_products<R, CT, false>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)op_lds_bytes<R, CT>()));
    return rc != ADAHOP_OK ? rc
                           : check_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_outlier_products<R, CT, true>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)op_lds_bytes<R, CT>()));
}

template <int R, int CT> int launch_products_as(const adahop_operand_t &x, const outlier_job_t &e, hipStream_t st)
{
    const int64_t groups = ceil_div(x.outer, 64 * CT);
    const dim3 grid((unsigned)(groups * e.nslice + (e.codes ? e.k : 0)));
    const uint16_t *l = static_cast<const uint16_t *>(x.data);
    if (x.outer % 8 == 0)
        hipLaunchKernelGGL((k_outlier_products<R, CT, false>), grid, dim3(256), (op_lds_bytes<R, CT>()), st, l, x.ld, x.outer, x.K, e, (int)groups);
    else
        hipLaunchKernelGGL((k_outlier_products<R, CT, true>), grid, dim3(256), (op_lds_bytes<R, CT>()), st, l, x.ld, x.outer, x.K, e, (int)groups);
    return check_launch();
}

template <int T, int CT> int launch_products_kc_as(const adahop_operand_t &x, const outlier_job_t &e, hipStream_t st)
{
    const int64_t groups = ceil_div(x.outer, 64 * CT);
    hipLaunchKernelGGL((k_outlier_products_kc<T, CT>), dim3((unsigned)(groups * e.nslice + (e.codes ? e.k : 0))), dim3(256), 0, st,
                       static_cast<const uint16_t *>(x.data), x.ld, x.outer, x.K, e, (int)groups);
    return check_launch();
}

constexpr int64_t LONG_SLICE = 4; // blocks of 256 K-elements
constexpr int64_t LONG_KC = 32ll << 20; // elements of a K-contiguous operand

// out[o, t] = x(o, idx[t]) for t < k, 0 for k <= t < kpad.  out is [outer, kpad] bf16.
__global__ __launch_bounds__(256) void k_gather_k(const uint16_t *__restrict__ x, int64_t ld, int k_contig,
                                                  int64_t outer, const int32_t *__restrict__ idx, int k, int kpad,
                                                  uint16_t *__restrict__ out)
{
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= outer * kpad) return;
    int64_t o, t;
    if (k_contig) { // neighbouring threads: neighbouring t of one row
        o = g / kpad;
        t = g - o * kpad;
    } else {        // neighbouring threads: neighbouring rows of one t (coalesced reads)
        t = g / outer;
        o = g - t * outer;
    }
    uint16_t v = 0;
    if (t < k) {
        const int64_t kk = idx[t];
        v = load_once2(k_contig ? x + o * ld + kk : x + kk * ld + o);
    }
    out[o * kpad + t] = v;
}

// The same for a K-strided operand (x stored [K, outer]): 64 channels x 64 rows per workgroup through
// LDS, so that both the reads (along the rows of one channel) and the writes (along the channels of
// one row) are whole 128-byte segments, 16 bytes per lane.
__global__ __launch_bounds__(256) void k_gather_k_strided(const uint16_t *__restrict__ x, int64_t ld, int64_t outer,
                                                          const int32_t *__restrict__ idx, int k, int kpad,
                                                          uint16_t *__restrict__ out)
{
    constexpr int PITCH = 72; // elements: 144-byte rows, 16-byte aligned
    __shared__ __align__(16) uint16_t tile[64 * PITCH];
    const int row = threadIdx.x >> 3, seg = threadIdx.x & 7;
    const int64_t o0 = (int64_t)blockIdx.x * 64;
    const int t0 = blockIdx.y * 64;
    uint4 v[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int t = t0 + p * 32 + row;
        const int64_t o = o0 + seg * 8;
        v[p] = make_uint4(0u, 0u, 0u, 0u);
        if (t < k) {
            const uint16_t *src = x + (int64_t)idx[t] * ld + o;
            if (o + 7 < outer) {
                v[p] = load_once16(src);
            } else { // (the last, ragged segment of a channel)
                uint16_t e[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) e[q] = o + q < outer ? load_once2(src + q) : (uint16_t)0;
                v[p] = make_uint4(e[0] | (uint32_t)e[1] << 16, e[2] | (uint32_t)e[3] << 16, e[4] | (uint32_t)e[5] << 16,
                                  e[6] | (uint32_t)e[7] << 16);
            }
        }
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) *reinterpret_cast<uint4 *>(&tile[(p * 32 + row) * PITCH + seg * 8]) = v[p];
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int ol = p * 32 + row; // row of the output: one outer index, 8 channels per lane
        uint16_t e[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) e[q] = tile[(seg * 8 + q) * PITCH + ol];
        if (o0 + ol < outer)
            *reinterpret_cast<uint4 *>(out + (o0 + ol) * kpad + t0 + seg * 8) =
                make_uint4(e[0] | (uint32_t)e[1] << 16, e[2] | (uint32_t)e[3] << 16, e[4] | (uint32_t)e[5] << 16,
                           e[6] | (uint32_t)e[7] << 16);
    }
}

} // namespace

int launch_gather_k(const adahop_operand_t &x, const int32_t *idx, int k, int kpad, uint16_t *out, hipStream_t st)
{
    const int64_t n = x.outer * kpad;
    if (n == 0) return ADAHOP_OK;
    if (!x.k_contig && kpad % 64 == 0) {
        const dim3 grid((unsigned)ceil_div(x.outer, 64), (unsigned)(kpad / 64));
        hipLaunchKernelGGL(k_gather_k_strided, grid, dim3(256), 0, st, static_cast<const uint16_t *>(x.data), x.ld,
                           x.outer, idx, k, kpad, out);
        return check_launch();
    }
    hipLaunchKernelGGL(k_gather_k, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st,
                       static_cast<const uint16_t *>(x.data), x.ld, x.k_contig, x.outer, idx, k, kpad, out);
    return check_launch();
}

// Every instance of the row / column product kernel, once per device (host-side calls, nothing queued).
int configure_oe_rowcol()
{
    static device_once_t once;
    int dev = 0;
    int rc = check_hip(hipGetDevice(&dev));
    if (rc != ADAHOP_OK || !once.need(dev)) return rc;
    if ((rc = allow_skinny_lds_all<2, 1>()) != ADAHOP_OK || (rc = allow_skinny_lds_all<4, 1>()) != ADAHOP_OK ||
        (rc = allow_skinny_lds_all<6, 1>()) != ADAHOP_OK || (rc = allow_skinny_lds_all<2, 2>()) != ADAHOP_OK ||
        (rc = allow_skinny_lds_all<4, 2>()) != ADAHOP_OK || (rc = allow_skinny_lds_all<6, 2>()) != ADAHOP_OK)
        return rc;
    if ((rc = allow_products_lds<1, 2>()) != ADAHOP_OK || (rc = allow_products_lds<2, 2>()) != ADAHOP_OK || (rc = allow_products_lds<1, 4>()) != ADAHOP_OK ||
        (rc = allow_products_lds<2, 4>()) != ADAHOP_OK || (rc = allow_products_lds<3, 4>()) != ADAHOP_OK)
        return rc;
    once.mark(dev);
    return ADAHOP_OK;
}

// K-strided, slices of up to three blocks: the quantiser's kernel without the quantisation, which takes a block at once; k_outlier_products has to fill its
// pipeline first.  Whole calls with 96 rows of the other operand, the quantiser's kernel / this, us: one block, 11008 x 2016, 16 rows 34.7 / 39.7; two, 8192 x 5024, 16
// rows 46.8 / 50.8; three, 14336 x 4096, 40 rows 57.3 / 61.0; four, 20000 x 4096, 1 row 69.6 / 67.0, 40 rows 81.0 / 78.6; seven, 11008 x 12000, 1 row 103 / 94.6;
// more, 5000 x 28672, 16 rows 153 / 133, 28672 x 8192, 64 rows 185 / 144.
// 256 columns per workgroup where these fill the chip in one round, or with more than 64 rows, where half as wide ones do not fit twice into the LDS
// either: 17000 x 10048, 64 rows (201 workgroups) 134 / 156 with 128 columns, 90 rows (268) 175 / 183; but 12288 x 8192, 16 rows (384) 80 / 73, and
// 20000 x 4096, 1 row (316) 70 / 67.
// K-contiguous, fewer than LONG_KC elements: the quantiser's kernel, which leaves the operand in the caches; a larger one takes the place of the packed operands there,
// which the next product reads.  Whole calls on operands used in turn, the quantiser's kernel / k_outlier_products_kc, us: 6144 x 4096, 10 rows 44 / 48.5;
// 8192 x 4096, 41 rows 82 / 83; 4096 x 8192, 10 rows 58.5 / 56; 2048 x 16384, 10 rows 71 / 67; 9216 x 4096, 41 rows 101 / 97; 16384 x 4096, 10 rows 98 / 87;
// 11008 x 8192, 40 rows 187 / 167; 28672 x 2048, 82 rows 246 / 199; 28672 x 8192, 41 rows 384 / 375.
// There 128 rows of L per workgroup, but 192 or 64 where the fullest compute unit then has fewer rows, 64 with up to 48 extracted rows (each workgroup moves all of
// them), and of 192 and 128 alike 192 with more than 64.  Products alone, us, 128 / 192 rows: 36000 x 2048, 70 rows 59 / 48, 40 rows 50.5 / 39.4; 35008 x 3072, 48 rows
// 68 / 53; 24000 x 4096, 60 rows 55.5 / 48; alike 12288 x 8192, 90 rows 71 / 66, 20000 x 4096, 40 rows 45.4 / 44.0, 14336 x 4096, 40 rows 36.8 / 37.7; more 16384 x
// 4096, 80 rows 42 / 49.  128 / 64 rows: 18000 x 4096, 10 rows 36.6 / 33.2, 40 rows 44.3 / 43.5; 9000 x 11008, 30 rows 56.5 / 52.7; 28672 x 8192, 10 rows 90 / 82; 20000 x 8192, 70 rows
// 84 (192) / 92; alike 9152 x 16672, 2 rows 66.6 / 68.4, 14336 x 4096, 40 rows 36.4 / 40.5.
// (k_oe_skinny, which adds in another order and splits K as suits it, is up to 6 % faster in such a call with many rows and short slices: 16384 x 4096, 64 rows 92 / 96, 12288 x
// 8192, 90 rows 127 / 135, 14336 x 4096, 40 rows 82 / 87; elsewhere as fast, or up to 20 % slower.)
int launch_outlier_products(const adahop_operand_t &L, const outlier_job_t &e, hipStream_t st)
{
    if (L.k_contig ? L.outer * L.K < LONG_KC : ceil_div(ceil_div(L.K, 256), e.nslice) < LONG_SLICE)
        return launch_iht_quantize_outliers(-1, {&L, nullptr, nullptr, nullptr, nullptr, nullptr, {nullptr, 0}, {nullptr, nullptr, 0, 0}, {nullptr, nullptr}}, e, st);
    if (L.k_contig) {
        // the rows of L, in 64, that the fullest compute unit takes
        auto most = [&](int64_t ct) { return ct * ceil_div(ceil_div(L.outer, 64 * ct) * e.nslice, 256); };
        auto go = [&](auto tiles) {
            constexpr int T = decltype(tiles)::value;
            const int64_t two = most(2), three = most(3);
            if constexpr (T <= 3) {
                if (most(1) < (two < three ? two : three)) return launch_products_kc_as<T, 1>(L, e, st);
            }
            return three < two || (T == 6 && three == two) ? launch_products_kc_as<T, 3>(L, e, st) : launch_products_kc_as<T, 2>(L, e, st);
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
    const int rc = configure_oe_rowcol();
    if (rc != ADAHOP_OK) return rc;
    if (e.k > 64) return launch_products_as<3, 4>(L, e, st);
    const int64_t workgroups = ceil_div(L.outer, 256) * e.nslice;
    if (workgroups >= 160 && workgroups <= 256) return e.k <= 32 ? launch_products_as<1, 4>(L, e, st) : launch_products_as<2, 4>(L, e, st);
    return e.k <= 32 ? launch_products_as<1, 2>(L, e, st) : launch_products_as<2, 2>(L, e, st);
}

size_t oe_rowcol_workspace_bytes(int64_t M, int64_t N, int64_t K, int kind, int k)
{
    if (k <= 0) return 0;
    const skinny_plan_t p = plan_skinny(kind == ADAHOP_IHT_OE_ROW ? N : M, K, k);
    return p.sg_bytes + p.p_bytes;
}

size_t oe_rowcol_partials_at(int64_t M, int64_t N, int64_t K, int kind, int k, size_t *bytes)
{
    const skinny_plan_t p = plan_skinny(kind == ADAHOP_IHT_OE_ROW ? N : M, K, k);
    *bytes = p.p_bytes;
    return p.sg_bytes;
}

// Whole groups of 64 rows of out are written at most.  (Rows past the k extracted ones may hold anything: row t of the product depends on
// row t alone, and the reduction reads the first k.)
int launch_gather_rows(const adahop_operand_t &S, const int32_t *idx, int k, uint16_t *out, hipStream_t st)
{
    const int64_t K = S.K;
    if (S.k_contig)
        hipLaunchKernelGGL(k_gather_rows, dim3((unsigned)ceil_div(k * (K >> 3), 256)), dim3(256), 0, st,
                           static_cast<const uint16_t *>(S.data), S.ld, K, idx, k, out);
    else
        hipLaunchKernelGGL(k_gather_rows_strided, dim3((unsigned)ceil_div(K, 64), (unsigned)ceil_div(k, 64)), dim3(256), 0, st,
                           static_cast<const uint16_t *>(S.data), S.ld, K, idx, k, out);
    return check_launch();
}

int launch_oe_reduce(const float *P, int nslice, int64_t rows_all, int64_t Lo, bool rows, const int32_t *idx, int k, void *C, int64_t ldc,
                     int c_bf16, hipStream_t st)
{
    const unsigned rblocks = (unsigned)ceil_div((int64_t)k * Lo, 256);
    auto reduce = [&](auto *c) {
        typedef typename std::remove_pointer<decltype(c)>::type out_t;
        // four long-side indices per thread where rows of the partials (and, for rows of C, of C) are 16-byte pieces
        if (Lo % 4 == 0 && (!rows || (ldc % 4 == 0 && aligned(c, 4 * sizeof(out_t))))) {
            const unsigned b4 = (unsigned)ceil_div((int64_t)k * (Lo >> 2), 256);
            if (rows)
                hipLaunchKernelGGL((k_oe_reduce4<true, out_t>), dim3(b4), dim3(256), 0, st, P, nslice, rows_all, Lo, idx, k, c,
                                   ldc);
            else
                hipLaunchKernelGGL((k_oe_reduce4<false, out_t>), dim3(b4), dim3(256), 0, st, P, nslice, rows_all, Lo, idx, k,
                                   c, ldc);
            return;
        }
        if (rows)
            hipLaunchKernelGGL((k_oe_reduce<true, out_t>), dim3(rblocks), dim3(256), 0, st, P, nslice, rows_all, Lo, idx,
                               k, c, ldc);
        else // (a variant that turns 32 x 64 blocks in LDS so that a wave's stores fall into two rows of C was measured
             // and is slower, 42 against 33 us on 123 x 8192: the k x Lo partial-sector writes cost the same either way)
            hipLaunchKernelGGL((k_oe_reduce<false, out_t>), dim3(rblocks), dim3(256), 0, st, P, nslice, rows_all, Lo, idx,
                               k, c, ldc);
    };
    if (c_bf16)
        reduce(static_cast<uint16_t *>(C));
    else
        reduce(static_cast<float *>(C));
    return check_launch();
}

// As many 256-element blocks of K per workgroup as leave four workgroups for each of the 256 compute units (4096 x 32768 with 64 rows, whole
// call: two for each 421, four 416, eight 416 us), and more where the sums would not fit otherwise.
// Not where L's quantiser would then have to wait for a selection that could stand beside it, and so does that of S: it takes some
// work for that to pay.  416 x 4096 (128 tiles), 55 columns, whole call 45 us beside, 48 on the way; 32 x 1440
// (23) 36.9 / 38.1; 96 x 8992 (141) 78.7 / 79.3; 32 x 17376 (272) 52.7 / 49.5; 32 x 20608 (322) 77.2 / 74.3.  (Extracted rows of a K-contiguous S are read
// in place, and the selection stands beside S's quantiser: on the way at any size, 4096 rows, 40 extracted, x 416 x 4096 46.0 / 40.3, x 32 x 1440 32.9 / 27.2,
// 1024 rows, 10 extracted, x 512 x 1024 41 / 34, each call waited for.)
bool oe_rowcol_on_the_way(const adahop_operand_t &S, const adahop_operand_t &L, int k, outlier_job_t *e)
{
    const int64_t Lo = L.outer, K = L.K;
    if (!S.k_contig && iht_quantize_beside_topk(S.outer, L) && ceil_div(Lo, 64) * ceil_div(K, 256) < 192) return false;
    e->tiles = (k + 15) / 16;
    while (e->tiles <= OUTLIER_TILES && !iht_quantize_takes_outliers(e->tiles)) ++e->tiles;
    if (e->tiles > OUTLIER_TILES) return false;
    const size_t room = plan_skinny(Lo, K, k).p_bytes;
    auto fits = [&](int64_t slices) { return (size_t)slices * k * Lo * 4 <= room; };
    const int64_t upr = ceil_div(K, 256), cols = ceil_div(Lo, 64);
    int64_t blocks = cols * upr / 1024;
    if (blocks < 1) blocks = 1;
    while (blocks < upr && !fits(ceil_div(upr, blocks))) ++blocks;
    int64_t n = ceil_div(upr, blocks);
    // Where that is somewhat more than four, and their slices are long, a second round is nearly empty and takes as long as the first: up to twice
    // as many, shorter slices then, if that makes the rounds together shorter.  Quantiser with the products, whole call with 96 rows of the other
    // operand / products alone, the same, us: 11008 x 12000, 8 rows, 7 -> 10 slices 129.9 -> 126.3 / 103 -> 100; 12288 x 8192, 8 rows, 6 -> 8 98.2 -> 89.4 /
    // 77 -> 71, 40 rows 104.7 -> 96 / 88 -> 84; 28672 x 8192, 8 rows, 3 -> 4 186 -> 173 / 151 -> 142.  (With slices of three blocks, 6400 x 8192, 11 -> 16 slices,
    // 53.8 / 53.8.  With more than 64 rows three workgroups fit: 12288 x 8192, 90 rows, 112 -> 115.)
    if (e->tiles <= 4 && ceil_div(upr, n) >= LONG_SLICE) {
        auto time = [&](int64_t slices) { return ceil_div(cols * slices, 1024) * ceil_div(upr, slices); };
        const int64_t most = 2 * n;
        for (int64_t s = n + 1; s <= most && fits(s); ++s)
            if (time(s) < time(n)) n = s;
    }
    e->k = k;
    e->nslice = (int)n;
    return fits(n);
}

int launch_oe_rowcol(const adahop_operand_t &A, const adahop_operand_t &B, int kind, const int32_t *idx, int k,
                     void *C, int64_t ldc, int c_bf16, void *workspace, hipStream_t st, bool gathered)
{
    const int64_t M = A.outer, N = B.outer, K = A.K;
    if (k == 0 || M == 0 || N == 0) return ADAHOP_OK;
    const bool rows = kind == ADAHOP_IHT_OE_ROW;
    const adahop_operand_t &S = rows ? A : B, &L = rows ? B : A;
    const int64_t Lo = L.outer;
    const skinny_plan_t p = plan_skinny(Lo, K, k);
    uint16_t *Sg = static_cast<uint16_t *>(workspace);
    float *P = reinterpret_cast<float *>(static_cast<char *>(workspace) + p.sg_bytes);

    outlier_job_t e = {};
    const bool as_on_the_way = oe_rowcol_on_the_way(S, L, k, &e), in_place = as_on_the_way && S.k_contig && !gathered;
    int rc = gathered || in_place ? ADAHOP_OK : launch_gather_rows(S, idx, k, Sg, st);
    if (rc != ADAHOP_OK) return rc;
    if (as_on_the_way) {
        e.rows = in_place ? static_cast<const uint16_t *>(S.data) : Sg;
        e.ld = in_place ? S.ld : K;
        e.idx = in_place ? idx : nullptr;
        e.p = P;
        rc = launch_outlier_products(L, e, st);
        return rc != ADAHOP_OK ? rc : launch_oe_reduce(P, e.nslice, k, Lo, rows, idx, k, C, ldc, c_bf16, st);
    }

    const dim3 grid((unsigned)ceil_div(Lo, SK_LCOLS / 2 * p.ncw), (unsigned)p.nslice, (unsigned)p.groups);
    const uint16_t *l = static_cast<const uint16_t *>(L.data);
    switch (p.rt) {
    case 2: rc = launch_skinny<2>(L.k_contig, p.ncw, grid, st, Sg, l, L.ld, Lo, K, p.stages_per_slice, P, p.rows_all); break;
    case 4: rc = launch_skinny<4>(L.k_contig, p.ncw, grid, st, Sg, l, L.ld, Lo, K, p.stages_per_slice, P, p.rows_all); break;
    default: rc = launch_skinny<6>(L.k_contig, p.ncw, grid, st, Sg, l, L.ld, Lo, K, p.stages_per_slice, P, p.rows_all); break;
    }
    if (rc != ADAHOP_OK) return rc;

    return launch_oe_reduce(P, p.nslice, p.rows_all, Lo, rows, idx, k, C, ldc, c_bf16, st);
}

} // namespace adahop
