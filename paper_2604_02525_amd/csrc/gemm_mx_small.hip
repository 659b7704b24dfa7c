// Block-scaled FP4 GEMM (the MXFP4 term of paper Eq. 4 / 5 / 7 / 8, with the K-channel outlier product in front of it),
// for products that the tiles of 256 rows do not fill the chip with or do not fit: few rows, few tiles, short K.  Any M, N,
// any K % 32 == 0, any alignment of C.
//
//   C[m, n] = sum_t Ag[m, t] Bg[n, t]                                   (bf16, optional, t < kpad)
//           + sum_blk 2^(sa[m,blk]-127) 2^(sb[n,blk]-127) sum_{i<32} a[m,32blk+i] b[n,32blk+i]
//
// Same instructions, operand layout and LDS slab layout as the 256 x 256 kernel (gemm_mx.hip); what differs:
//   - tiles of 32 .. 128 rows and columns, four waves.  A wave owns at most 64 x 64 of C (64 accumulators per lane), which
//     leaves registers for a second workgroup on the compute unit;
//   - WK waves share a part of C and take the four matrix-core steps of every stage between them (WK = 2: two steps
//     each, WK = 4: one); their sums are added through LDS at the end, in wave order.  A tile of 64 x 64 by four waves then reads
//     every operand byte from LDS once, and four times as many workgroups share a product of few tiles;
//   - NST stages of 256 K-elements rotate in LDS, NST - PU of them on the way: such a product is bound by the latency of
//     its operands (a tile's own share of the copy rate is 64 bytes per cycle and compute unit, reached with 64 .. 96 KiB
//     in flight), not by the matrix cores.  One barrier per PU stages, at the head of the first: they have landed (a counted
//     wait for all but the copies of the younger stages) and every wave has left the buffers that are refilled next.  PU is 1, and 2
//     for 32 x 32, where a wave has one matrix-core instruction per stage and a barrier for each would be most of its time; NST =
//     1 is for products of a single stage;
//   - rows past the end of an operand repeat its last row and are not stored.  A last stage of K that is no multiple of
//     256 starts at K - 256 as in the 256 x 256 kernel, its leading blocks with scale 0; of a K below 256 the missing
//     blocks are the first block again, with scale 0.
//   - what it replaced, a kernel that read its operands straight from global memory, took 420 us on 128 x 1248 x 28672 (now 19),
//     63 us on 128 x 11008 x 4096 (10) and 78 us on 4096 x 11008 x 512 (40); 256 rows of 4096 x 4096 took 13.4 us in tiles of
//     256 x 128 (now 7.8);
//   - the scales come from the stage-major copy or, where K % 256 == 0, straight from the canonical array (8 bytes per row
//     and stage: two 4-byte copies), which saves a product of packed operands the launch that re-orders them; up to
//     PRE_STAGES stages they may be canonical at any K: see there.
#include "common.h"
#include "gemm_mx_common.h"

#include <type_traits>

namespace adahop {

namespace {

namespace small {

constexpr int TKB = 128; // bytes of K per row and stage

// Where the scale bytes of a stage lie: row r of stage s at p + r * row + s * stage, 8 bytes, 4-byte aligned.
struct scale_src_t {
    const uint8_t *p;
    int64_t row, stage;
    uint32_t canonical; // (only for PRE) 0: stage-major, else ceil(2^20 / (K / 32)), which turns bytes of the canonical array into rows
};

// PRE: the scales of all stages lie in LDS from the start, brought through registers: at a K that is no multiple of 256 the canonical
// array cannot be copied straight into stages (no piece of it is aligned, and the last stage wants zeros in front).  The
// K / 32 bytes of a tile's rows are one run of bytes; the threads read them side by side and put each where its stage wants
// it.  For short products of packed operands, of which the launch that re-orders the scales and its gap would be the larger part:
// 1 x 16716 x 96 9.7 -> 4.1 us, 665 x 852 x 320 11.3 -> 5.5.  At more stages than PRE_STAGES the bytes to place grow and the launch is the smaller part.
constexpr int PRE_STAGES = 4;

__device__ __forceinline__ void dma4(const uint8_t *base, uint32_t voff, uint32_t lds_addr)
{ // as dma16, 4 bytes per lane
    base = uniform_ptr(base);
    lds_addr = __builtin_amdgcn_readfirstlane(lds_addr);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                 :
                 : "v"(voff), "s"(base), "s"(lds_addr)
                 : "memory", "m0");
}

template <int T, int I = 0, typename F> __device__ __forceinline__ void for_each_index(F &&f)
{
    if constexpr (I < T) {
        f(std::integral_constant<int, I>());
        for_each_index<T, I + 1>(f);
    }
}

template <int X> __device__ __forceinline__ void wait_and_meet()
{
    // my copies of the stage have landed and my LDS reads are done; then every wave's
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::"n"(X) : "memory");
}

__device__ __forceinline__ void put(float *p, float v) { *p = v; }
__device__ __forceinline__ void put(uint16_t *p, float v)
{
    const __bf16 b = (__bf16)v; // nearest even
    *p = __builtin_bit_cast(uint16_t, b);
}

template <int TMB, int TNB, int WM, int WN, int WK, int NST, int PU, bool PRE> struct shape_t {
    static constexpr int TM = 32 * TMB * WM, TN = 32 * TNB * WN;
    static constexpr int SLAB = (TM + TN) * TKB, SCALES = (TM + TN) * 8; // bytes of a stage
    static constexpr int STAGE = SLAB + (PRE ? 0 : SCALES);              // bytes of a buffer
    static constexpr int RED = WK > 1 ? 4 * TMB * TNB * 16 * 64 * 4 : 0;
    static constexpr int ALL = NST * STAGE + (PRE ? PRE_STAGES * SCALES : 0);
    static constexpr int LDS = ALL > RED ? ALL : RED;
    static constexpr int NC = (TM + TN) / 32;      // 16-byte copies per wave and stage (a copy: 8 rows; 4 waves)
    static constexpr int NS = PRE ? 0 : ((TM + TN) / 32 + 3) / 4; // 4-byte copies of scales per wave and stage (a copy: 32 rows)
};

// The order of the tiles (launch_as).  A C that the Infinity Cache holds: down the columns of tiles, in runs per XCD, so that the
// workgroups that read the same rows of B share an L2.  A larger one leaves for memory while the product runs, and what counts is that
// what lies together is written together: along the rows of tiles, in runs per XCD, which also puts the pieces of a line that two
// tiles share into one L2; without the runs where the rows of C are whole 4-KiB pages, of which the runs would write eight times as many in
// different places, but on the same memory channels (with one stage of K in fp32: of whole 64-byte pieces, 8569 x 8576 x 96 49 along, 57 in
// runs).  Where K is one stage there is little to share, and the line lies lower: 8454 x 10175 x 192 in bf16 (164 MB) 54 / 43 / 43, but 2541 x
// 13392 x 96 (130 MB) 26.6 / 27.2 / 27.3.  128 x 128 tiles, us, down in runs / along / along in runs:
//   9687 x 14001 x 64 (517 MB, ldc 14001)  203 / 185 / 133      8192 x 16384 x 64 (512 MB)     153 / 109 / 110
//   24515 x 9536 x 320 (891 MB)            234 / 249 / 214      8192 x 16384 x 1024           231 / 166 / 190
//   6000 x 9001 x 64 (206 MB, ldc 9001)     47 /  47 /  43      30000 x 4096 x 512 (468 MB)    116 / 118 / 147
//   4001 x 12001 x 512 (183 MB, ldc 12001)  47 /  53 /  49      4096 x 11008 x 512 (172 MB)     40 /  42 /  44
// Below those lines, along the rows in runs from 24 MB of C and 16 rows of tiles on, for K up to 192, off the 64-byte grid 512: as much is shared as down the columns, and the
// pieces of C's lines meet in one L2.  Down / along in runs: 10911 x 2828 x 64 (118 MB) 29.2 / 26.9, 5345 x 8125 x 384 (166 MB)
// 52.1 / 44.1, 9187 x 2427 x 320 (85 MB) 27.5 / 24.9, 4096 x 2048 x 64 (32 MB) 10.8 / 9.7, 6374 x 2200 x 64 in bf16 (27 MB) 14.8 / 11.7,
// 2743 x 11808 x 192 (124 MB) 30.0 / 28.6; fewer rows of tiles do not spread over the XCDs: 1158 x 6892 x 64 11.1 / 11.6, 1356 x 12198 x 192
// 19.8 / 20.3.  On the grid, where two tiles share no line, more K takes it back: 3378 x 10976 x 512 (141 MB) 32 / 38, and of the lines above
// 3360 x 11416 x 256 (146 MB, ldc 11424) 28 / 31.
enum walk_t { DOWN = 0, ALONG_ROWS = 1, RUNS = 2 };
constexpr int64_t C_STAYS = 192ll << 20, C_STAYS_SHORT = 136ll << 20; // bytes of C; the latter for K <= 192, off the 64-byte grid 256
constexpr int64_t C_ALONG = 24ll << 20;

template <int TMB, int TNB, int WM, int WN, int WK, int NST, int PU, bool PRE, bool OEK, typename OUT>
__global__ __launch_bounds__(256, NST == 1 ? 4 : 2) void k_gemm_mx_small(int64_t K, const uint8_t *__restrict__ a_codes, scale_src_t a_sc,
                                                          const uint8_t *__restrict__ b_codes, scale_src_t b_sc, int64_t M,
                                                          int64_t N, OUT *__restrict__ C, int64_t ldc,
                                                          const uint16_t *__restrict__ Ag, const uint16_t *__restrict__ Bg,
                                                          int kpad, int walk, int tiles_fast)
{
    typedef shape_t<TMB, TNB, WM, WN, WK, NST, PU, PRE> S;
    constexpr int TM = S::TM, TN = S::TN, NC = S::NC, NS = S::NS, CPS = NC + NS; // CPS: copies per wave and stage
    static_assert(WM * WN * WK == 4 && TM % 32 == 0 && TN % 32 == 0 && 4 % WK == 0, "four waves");
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = w % WK, wmn = w / WK, wm = wmn / WN, wn = wmn % WN;

    // Workgroup v -> tile.  Consecutive ids land on the 8 XCDs in turn; RUNS: every XCD takes a contiguous run of the tiles.
    int tix = blockIdx.x;
    if (walk & RUNS) {
        const int nt = gridDim.x, per = nt >> 3, rest = nt & 7, x = tix & 7;
        tix = x * per + min(x, rest) + (tix >> 3);
    }
    const int fast = tix % tiles_fast, slow = tix / tiles_fast;
    const int64_t m0 = (int64_t)(walk & ALONG_ROWS ? slow : fast) * TM, n0 = (int64_t)(walk & ALONG_ROWS ? fast : slow) * TN;

    // ---- copy engine.  Copy d of wave w: rows 8 (w + 4 d) .. + 7 of the tile's TM rows of A and TN rows of B; lane i writes
    // LDS row i / 8 of them, chunk position i % 8, which holds logical chunk (i % 8) ^ ((row / 2) & 7).
    const int nbf = OEK ? kpad >> 6 : 0, nfp = (int)((K + 255) >> 8), n = nbf + nfp;
    const uint32_t chunk16 = (uint32_t)(((lane & 7) ^ (4 * (w & 1) + (lane >> 4))) * 16);
    const int last_off = K >= 256 ? (int)(K >> 1) - TKB : 0;
    const int short_by = K >= 256 ? 0 : TKB - (int)(K >> 1); // bytes that a row lacks of a whole stage
    const uint32_t pitch = (uint32_t)(K >> 1), gpitch = (uint32_t)kpad * 2;
    uint32_t vo[NC]; // byte offset of the lane's chunk (OEK: its row, of which the offset is made for either pitch)
    const uint32_t chunk_fp4 = (uint32_t)max((int)chunk16 - short_by, 0);
#pragma unroll
    for (int d = 0; d < NC; ++d) {
        const int r = 8 * (w + 4 * d) + (lane >> 3);
        const int64_t left = d < TM / 32 ? M - 1 - m0 : N - 1 - n0;
        const uint32_t row = (uint32_t)min((int64_t)(d < TM / 32 ? r : r - TM), left);
        vo[d] = OEK ? row : row * pitch + chunk_fp4;
    }
    constexpr int NS1 = NS > 0 ? NS : 1;
    uint32_t so[NS1];     // scales: lane i copies half i % 2 of row i / 2 of 32
    bool s_is_a[NS1];     // (wave-uniform)
    int s_at[NS1];
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int q = (w + 4 * j) % ((TM + TN) / 32); // (a wave without a copy of its own repeats another's: same bytes)
        s_at[j] = q;
        s_is_a[j] = q < TM / 32;
        const int r = 32 * (s_is_a[j] ? q : q - TM / 32) + (lane >> 1);
        const uint32_t row = (uint32_t)min((int64_t)r, s_is_a[j] ? M - 1 - m0 : N - 1 - n0);
        so[j] = row * (uint32_t)(s_is_a[j] ? a_sc.row : b_sc.row) + (lane & 1) * 4;
    }
    const uint64_t ga = reinterpret_cast<uint64_t>(a_codes) + m0 * pitch, gb = reinterpret_cast<uint64_t>(b_codes) + n0 * pitch;
    const uint64_t gga = reinterpret_cast<uint64_t>(Ag) + m0 * gpitch, ggb = reinterpret_cast<uint64_t>(Bg) + n0 * gpitch;
    // scale copies: base and stage stride of the operand that copy j of this wave serves
    const uint8_t *sp[NS1];
    int64_t sstep[NS1];
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        sp[j] = s_is_a[j] ? a_sc.p + m0 * a_sc.row : b_sc.p + n0 * b_sc.row;
        sstep[j] = s_is_a[j] ? a_sc.stage : b_sc.stage;
    }
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));

    // Copies D0 .. D1-1 of the CPS of a stage, into LDS buffer b: NC of codes (or gathered bf16), then NS of scales.
    auto issue = [&](int stage, int b, auto d0_c, auto d1_c) {
        constexpr int D0 = decltype(d0_c)::value, D1 = decltype(d1_c)::value;
        if constexpr (D0 < D1) {
            const uint32_t buf = lds0 + (uint32_t)b * S::STAGE;
            // (The choices between a bf16 and an FP4 stage are made with a mask: written as selections of the variables that this
            // function captures, they put those into memory, and the K-channel products ran at half the speed.)
            const bool bf = OEK && stage < nbf;
            const uint64_t m = bf ? ~(uint64_t)0 : 0;
            const uint32_t rp = pitch ^ ((pitch ^ gpitch) & (uint32_t)m), ch = chunk_fp4 ^ ((chunk_fp4 ^ chunk16) & (uint32_t)m);
            const int fs = bf ? 0 : stage - nbf; // (a bf16 stage copies the scales of the first FP4 stage: the count stays the same)
            const int off = bf ? stage * TKB : min(fs * TKB, last_off);
            const uint8_t *pa = reinterpret_cast<const uint8_t *>(ga ^ ((ga ^ gga) & m)) + off;
            const uint8_t *pb = reinterpret_cast<const uint8_t *>(gb ^ ((gb ^ ggb) & m)) + off;
#pragma unroll
            for (int d = D0; d < D1; ++d) {
                if (d < NC) {
                    uint32_t v = vo[d];
                    if constexpr (OEK) v = __umul24(v, rp) + ch;
                    if (NST > 1 || (int)chunk16 >= short_by) dma16(d < TM / 32 ? pa : pb, v, buf + (uint32_t)(w + 4 * d) * 1024);
                } else {
                    const int j = d - NC;
                    dma4(sp[j] + fs * sstep[j], so[j], buf + S::SLAB + s_at[j] * 256);
                }
            }
        }
    };
    auto issue_all = [&](int stage, int b) { issue(stage, b, std::integral_constant<int, 0>(), std::integral_constant<int, CPS>()); };

    // ---- fragment reads: row l32 (+ 32 i) of the wave's part, logical chunk 4 h + s in step s
    const int rx = (l32 >> 1) & 7;
    const int a_row = (wm * TMB * 32 + l32) * TKB, b_row = (TM + wn * TNB * 32 + l32) * TKB;
    const int sa_row = (wm * TMB * 32 + l32) * 8 + 4 * h, sb_row = (TM + wn * TNB * 32 + l32) * 8 + 4 * h;
    auto scales_of = [&](int t, int b) { return smem + (PRE ? NST * S::STAGE + (t - nbf) * S::SCALES : b * S::STAGE + S::SLAB); };

    // (PRE) the last stage's first `zeros` scales of a row, which stand for blocks that it lacks, count as 0
    const int zeros = PRE ? -(int)(K >> 5) & 7 : 0, behind = min(max(zeros - 4 * h, 0), 4);
    const uint32_t keep_last = behind == 4 ? 0u : ~0u << (8 * behind);
    const uint8_t *const last_scales = smem + NST * S::STAGE + (nfp - 1) * S::SCALES;

    v16f acc[TMB][TNB];
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
        for (int j = 0; j < TNB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // One stage: its matrix-core instructions, the fragment reads of the next step ahead of those of a step, and between them
    // (ISSUE) the copies of stage `which` into buffer `wb`, spread evenly: a wave issues in order, and all copies at the head
    // of the stage kept it from the matrix cores for half of its time (0.67 us per stage of 128 x 128 where the matrix
    // cores need 0.2).
    auto stage = [&](const uint8_t *st, const uint8_t *ss, auto bf_c, auto issue_c, int which, int wb) {
        constexpr bool BF = decltype(bf_c)::value, ISSUE = decltype(issue_c)::value;
        constexpr int STEPS = 4 / WK, T = TMB * TNB * STEPS;
        int sa[TMB], sb[TNB];
        uint4 a[2][TMB], b[2][TNB];
        auto read = [&](int q) {
            const int at = ((4 * h + STEPS * wk + q) ^ rx) * 16;
#pragma unroll
            for (int i = 0; i < TMB; ++i) a[q & 1][i] = *reinterpret_cast<const uint4 *>(st + a_row + i * 32 * TKB + at);
#pragma unroll
            for (int j = 0; j < TNB; ++j) b[q & 1][j] = *reinterpret_cast<const uint4 *>(st + b_row + j * 32 * TKB + at);
        };
        if constexpr (!BF) {
#pragma unroll
            for (int i = 0; i < TMB; ++i) sa[i] = *reinterpret_cast<const int *>(ss + sa_row + i * 256);
#pragma unroll
            for (int j = 0; j < TNB; ++j) sb[j] = *reinterpret_cast<const int *>(ss + sb_row + j * 256);
        }
        const int absent = NST == 1 ? max(4 - (int)(K >> 5), 0) : 0; // steps of a stage of K < 128 that hold none of its blocks
        read(0);
        ADAHOP_PIN();
        if constexpr (!BF && PRE) {
            const int keep = ss == last_scales ? (int)keep_last : -1;
#pragma unroll
            for (int i = 0; i < TMB; ++i) sa[i] &= keep;
#pragma unroll
            for (int j = 0; j < TNB; ++j) sb[j] &= keep;
        }
        if constexpr (!BF && WK > 1) {
#pragma unroll
            for (int i = 0; i < TMB; ++i) sa[i] >>= 8 * STEPS * wk;
#pragma unroll
            for (int j = 0; j < TNB; ++j) sb[j] >>= 8 * STEPS * wk;
        }
        auto one = [&](auto k_c) { // matrix-core instruction k of the stage: step k / (TMB TNB), row-major over the wave's tiles
            constexpr int k = decltype(k_c)::value, q = k / (TMB * TNB), e = k % (TMB * TNB), i = e / TNB, j = e % TNB;
            if (NST == 1 && q < absent) return; // (only blocks of scale 0)
            if constexpr (e == 0 && NST == 1 && q > 0) {
                if (q == absent) read(q); // (the first step that is there)
            }
            if constexpr (e == 0 && q + 1 < STEPS) {
                read(q + 1);
                ADAHOP_PIN();
            }
            if constexpr (BF) {
                acc[i][j] = mfma_bf16(a[q & 1][i], b[q & 1][j], acc[i][j]);
            } else {
                const uint4 x = a[q & 1][i], y = b[q & 1][j];
                v8i av = {(int)x.x, (int)x.y, (int)x.z, (int)x.w, 0, 0, 0, 0};
                v8i bv = {(int)y.x, (int)y.y, (int)y.z, (int)y.w, 0, 0, 0, 0};
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc[i][j], 4, 4, q, sa[i], q, sb[j]);
            }
            if constexpr (ISSUE) {
                ADAHOP_PIN();
                issue(which, wb, std::integral_constant<int, CPS * k / T>(), std::integral_constant<int, CPS *(k + 1) / T>());
                ADAHOP_PIN();
            }
        };
        for_each_index<T>(one);
    };
    auto run = [&](int t, int b, auto issue_c, int which, int wb) {
        const uint8_t *st = smem + b * S::STAGE;
        if (OEK && t < nbf)
            stage(st, st, std::true_type(), issue_c, which, wb);
        else
            stage(st, scales_of(t, b), std::false_type(), issue_c, which, wb);
    };

    constexpr int AHEAD = NST > 1 ? NST - PU : 1; // stages whose copies are asked for here
    if constexpr (PRE) {
        // A run is read in aligned words (four per thread) and the bytes in front of the first and behind the
        // last of them.  The loads of both operands go ahead of the stages' copies, so that the wait for them is the wait that the
        // first stage needs anyway.
        uint8_t *const all = smem + NST * S::STAGE;
        const int KB = (int)(K >> 5);
        struct run_t {
            const uint8_t *p;
            int rows, head, words, edge; // edge: the byte in front of or behind the words that this thread takes, if it lies in the run
            uint32_t v[4], e;
        };
        auto fetch = [&](const scale_src_t &sc, int64_t first, int64_t left, int most) {
            run_t r;
            r.rows = (int)min((int64_t)most, left);
            r.p = sc.p + first * KB;
            const int total = r.rows * KB;
            r.head = min((int)(-(uint32_t)reinterpret_cast<uintptr_t>(r.p) & 3u), total);
            r.words = sc.canonical ? (total - r.head) >> 2 : 0;
            // (one buffer: one stage)
            static_assert((S::TM > S::TN ? S::TM : S::TN) * 8 * (NST == 1 ? 1 : PRE_STAGES) <= 4 * 4 * 256, "four words per thread hold an operand's run");
            r.edge = tid < r.head ? tid : 4 * r.words + tid;
            r.e = 0;
            if (sc.canonical && r.edge < total) r.e = r.p[r.edge];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                r.v[j] = 0;
                if (256 * j < r.words) r.v[j] = *reinterpret_cast<const uint32_t *>(r.p + r.head + 4 * min(tid + 256 * j, r.words - 1));
            }
            return r;
        };
        auto place = [&](const scale_src_t &sc, const run_t &r, int64_t first, int to) {
            if (!sc.canonical) { // stage-major: eight bytes per row and stage as they are
                for (int s = 0; s < nfp; ++s)
                    if (tid < r.rows)
                        *reinterpret_cast<uint64_t *>(all + s * S::SCALES + (to + tid) * 8) =
                            *reinterpret_cast<const uint64_t *>(sc.p + (first + tid) * 8 + s * sc.stage);
                return;
            }
            auto put_byte = [&](int row, int blk, uint32_t x) {
                const int s = blk >> 3;
                all[s * S::SCALES + (to + row) * 8 + (blk & 7) + (s == nfp - 1 ? zeros : 0)] = (uint8_t)x;
            };
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (256 * j < r.words) {
                    const int i = r.head + 4 * (tid + 256 * j);
                    int row = (int)((uint32_t)i * sc.canonical >> 20), blk = i - row * KB;
                    if (tid + 256 * j < r.words) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            put_byte(row, blk, r.v[j] >> (8 * q));
                            const bool over = ++blk == KB;
                            row += over, blk = over ? 0 : blk;
                        }
                    }
                }
            if (r.edge < r.rows * KB) {
                const int row = (int)((uint32_t)r.edge * sc.canonical >> 20);
                put_byte(row, r.edge - row * KB, r.e);
            }
        };
        const run_t ra = fetch(a_sc, m0, M - m0, TM), rb = fetch(b_sc, n0, N - n0, TN);
        for (int s = 0; s < AHEAD && s < n; ++s) issue_all(s, s);
        place(a_sc, ra, m0, 0);
        place(b_sc, rb, n0, TM); // (the barrier at the head of the first stage stands between these and their readers)
    } else {
        for (int s = 0; s < AHEAD && s < n; ++s) issue_all(s, s);
    }
    int t = 0, b = 0; // stage t lies in buffer b = t % NST
    auto at = [&](int x) { return x < NST ? x : x - NST; };
    // PU stages with the copies of PU more, into the buffers of stages t - PU .. t - 1, which every wave has left
    auto full = [&](auto &&body) {
        wait_and_meet<CPS *(NST - 2 * PU)>(); // stages t + PU .. t + NST - PU - 1 may still be on the way
#pragma unroll
        for (int u = 0; u < PU; ++u) body(t + u, at(b + u), t + NST - PU + u, at(b + NST - PU + u));
        t += PU;
        b = at(b + PU);
    };
    const std::true_type yes;
    const std::false_type no;
    if constexpr (OEK) { // loops of their own: a branch around the matrix-core instructions moves the accumulators at every stage
        while (t + NST <= n && t + PU <= nbf) full([&](int, int rb, int which, int wb) { stage(smem + rb * S::STAGE, smem, yes, yes, which, wb); });
        if (PU > 1 && t + NST <= n && t < nbf) full([&](int s, int rb, int which, int wb) { run(s, rb, yes, which, wb); });
    }
    while (NST > 1 && t + NST <= n) full([&](int s, int rb, int which, int wb) { stage(smem + rb * S::STAGE, scales_of(s, rb), no, yes, which, wb); });
    for (; t < n; t += PU, b = at(b + PU)) {
        wait_and_meet<0>();
#pragma unroll
        for (int u = 0; u < PU; ++u)
            if (NST > 1 && t + NST - PU + u < n) issue_all(t + NST - PU + u, at(b + NST - PU + u));
        run(t, b, std::false_type(), 0, 0);
#pragma unroll
        for (int u = 1; u < PU; ++u)
            if (t + u < n) run(t + u, at(b + u), std::false_type(), 0, 0);
    }

    // ---- the waves that share a part of C add up, each wave the sums of its share of the accumulator tile
    if constexpr (WK > 1) {
        constexpr int E = TMB * TNB * 16, SH = E / WK;
        float *red = reinterpret_cast<float *>(smem);
        wait_and_meet<0>(); // every wave has read its last fragments
#pragma unroll
        for (int i = 0; i < TMB; ++i)
#pragma unroll
            for (int j = 0; j < TNB; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) red[(w * E + (i * TNB + j) * 16 + r) * 64 + lane] = acc[i][j][r];
        wait_and_meet<0>();
#pragma unroll
        for (int e0 = 0; e0 < SH; ++e0) {
            const int e = wk * SH + e0, t = e >> 4, r = e & 15, i = t / TNB, j = t % TNB;
            float v = red[((wmn * WK) * E + e) * 64 + lane];
#pragma unroll
            for (int q = 1; q < WK; ++q) v += red[((wmn * WK + q) * E + e) * 64 + lane];
            const int64_t row = m0 + (wm * TMB + i) * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
            const int64_t col = n0 + (wn * TNB + j) * 32 + l32;
            if (row < M && col < N) put(C + row * ldc + col, v);
        }
    } else {
        // Row by row over the wave's columns: what lies together is written together, and where rows lie off the 64-byte grid the two halves of the
        // line between two accumulator tiles meet in the L2 (tile by tile / row by row, us: 2528 x 13392 x 96 43.8 / 36.6, 6000 x 9000 x 320
        // 72 / 60, 8192 x 9001 x 96 90 / 66, 4096 x 11008 x 480 58.7 / 53.9, 28672 x 8192 x 64 in bf16 103 / 91).
#pragma unroll
        for (int i = 0; i < TMB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = m0 + (wm * TMB + i) * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
#pragma unroll
                for (int j = 0; j < TNB; ++j) {
                    const int64_t col = n0 + (wn * TNB + j) * 32 + l32;
                    if (row < M && col < N) put(C + row * ldc + col, acc[i][j][r]);
                }
            }
    }
}

template <int TMB, int TNB, int WM, int WN, int WK, int NST, int PU> struct variant_t {
    template <bool PRE, bool OEK, typename OUT> static int allow()
    {
        return check_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gemm_mx_small<TMB, TNB, WM, WN, WK, NST, PU, PRE, OEK, OUT>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             shape_t<TMB, TNB, WM, WN, WK, NST, PU, PRE>::LDS));
    }
    template <bool PRE> static int configure_as()
    {
        int rc;
        if ((rc = allow<PRE, false, float>()) != ADAHOP_OK || (rc = allow<PRE, false, uint16_t>()) != ADAHOP_OK) return rc;
        if constexpr (NST > 1) { // (K-channels and a stage of K are two stages)
            if ((rc = allow<PRE, true, float>()) != ADAHOP_OK || (rc = allow<PRE, true, uint16_t>()) != ADAHOP_OK) return rc;
        }
        return ADAHOP_OK;
    }
    static int configure()
    {
        const int rc = configure_as<false>();
        return rc != ADAHOP_OK ? rc : configure_as<true>();
    }
    template <bool PRE, typename OUT>
    static int launch_as(int64_t M, int64_t N, int64_t K, const uint8_t *a, scale_src_t as, const uint8_t *b, scale_src_t bs, OUT *C,
                         int64_t ldc, const uint16_t *Ag, const uint16_t *Bg, int kpad, hipStream_t st)
    {
        typedef shape_t<TMB, TNB, WM, WN, WK, NST, PU, PRE> S;
        const int64_t tm = ceil_div(M, S::TM), tn = ceil_div(N, S::TN);
        const dim3 grid((unsigned)(tm * tn));
        const int64_t c_bytes = M * N * (int64_t)sizeof(OUT);
        const bool off = !c_rows_streamed(C, ldc * (int64_t)sizeof(OUT)); // rows off the 64-byte grid
        const bool leaves = c_bytes >= (K <= 192 || (K <= 256 && off) ? C_STAYS_SHORT : C_STAYS);
        const bool stores = c_bytes >= C_ALONG && tm >= 16 && K <= (off ? 512 : 192);
        const int64_t whole = NST == 1 && sizeof(OUT) == 4 ? 64 : 4096;
        const int walk = leaves ? (ldc * (int64_t)sizeof(OUT) % whole == 0 ? ALONG_ROWS : ALONG_ROWS | RUNS) : stores ? ALONG_ROWS | RUNS : DOWN | RUNS;
        const int fast = (int)(walk & ALONG_ROWS ? tn : tm);
        if constexpr (NST > 1) {
            if (kpad > 0) {
                hipLaunchKernelGGL((k_gemm_mx_small<TMB, TNB, WM, WN, WK, NST, PU, PRE, true, OUT>), grid, dim3(256), S::LDS, st, K, a, as, b,
                                   bs, M, N, C, ldc, Ag, Bg, kpad, walk, fast);
                return check_launch();
            }
        }
        hipLaunchKernelGGL((k_gemm_mx_small<TMB, TNB, WM, WN, WK, NST, PU, PRE, false, OUT>), grid, dim3(256), S::LDS, st, K, a, as, b, bs,
                           M, N, C, ldc, Ag, Bg, kpad, walk, fast);
        return check_launch();
    }
    template <typename OUT>
    static int launch(int64_t M, int64_t N, int64_t K, const uint8_t *a, scale_src_t as, const uint8_t *b, scale_src_t bs, OUT *C,
                      int64_t ldc, const uint16_t *Ag, const uint16_t *Bg, int kpad, hipStream_t st)
    {
        return as.canonical || bs.canonical ? launch_as<true>(M, N, K, a, as, b, bs, C, ldc, Ag, Bg, kpad, st)
                                            : launch_as<false>(M, N, K, a, as, b, bs, C, ldc, Ag, Bg, kpad, st);
    }
};

typedef variant_t<2, 2, 2, 2, 1, 2, 1> v128_t;    // 128 x 128, two workgroups per compute unit
// 128 x 128 for a K of one stage: one buffer, half the registers, four workgroups.  Such a product is its stores, which three other
// workgroups' loads then run beside: 2541 x 13392 x 96 30.4 -> 26.8 us, in bf16 26.5 -> 20.5, 16384 x 16384 x 96 217 -> 190.
// Not for more than 64 MB of fp32 off the 64-byte grid, where twice the tiles in flight cost more line pieces than they hide (9687 x
// 14001 x 64 133 / 203 us, 6000 x 9001 x 64 43 / 46; 3324 x 2547 x 32, 32 MB, 13.8 / 12.1), and not for K = 256, where it gains nothing.
typedef variant_t<2, 2, 2, 2, 1, 1, 1> v128one_t;
// The same in tiles of 64 x 256, three workgroups (50 KB of LDS), for fp32 rows on the 64-byte grid and more than 80 MB of C: the four waves store 1 KiB of a row at about the
// same time, and stores alone reach 5.9 TB/s in such tiles, 5.5 in 128 x 128.  128 x 128 / 64 x 256, us: 8192 x 12288 x 96 75.9 / 69.4, 16384 x 16384 x
// 96 194 / 166, 8192 x 14336 x 192 88.7 / 80.8, 8192 x 4096 x 192 35.5 / 33.3; below that as much as they gain is lost with the rows of B that a tile reads, 5152
// x 2912 x 64 (60 MB) 17.3 / 18.2, 2048 x 8192 x 192 (64 MB) 19.0 / 19.2; off the grid 8192 x 9001 x 96 66 (two buffers) / 70, bf16 28672 x 8192 x 64 91 / 110.
typedef variant_t<2, 2, 1, 4, 1, 1, 1> v64x256_t;
typedef variant_t<2, 2, 2, 2, 1, 3, 1> v128deep_t; // 128 x 128, one workgroup, two stages on the way
typedef variant_t<2, 2, 1, 1, 4, 4, 1> v64_t;     // 64 x 64
typedef variant_t<1, 2, 1, 1, 4, 4, 1> v32x64_t;  // 32 x 64
typedef variant_t<1, 1, 1, 1, 4, 8, 2> v32_t;     // 32 x 32
// 96 x 64 for products that it gives one tile per compute unit and the smaller tiles two or three, us, the smaller ones / this: 96 x 11008 x 4096 14.3 / 11.4,
// 384 x 4096 x 4096 14.9 / 11.9, 96 x 16384 x 8192 23.2 / 21.2 (with weights not in the Infinity Cache 18.9 / 17.3, 15.8 / 12.8 the first two).  Two
// waves share a part of C: with four, each with all of it (<3, 2, 1, 1, 4>), the sums to add fill the LDS of two workgroups, 12.5 for the first; five stages in
// place of three 11.9.  Not for products of more tiles than compute units: 261 x 15506 x 7168, 729 tiles, 40.3 / 49.1, 191 x 23746 x 9056, 744, 68.6 / 75.6.
typedef variant_t<3, 1, 1, 2, 2, 3, 1> v96x64_t;

// What a variant takes, in us: start + stages max(alone, busy L) + tile L, L = tiles on the fullest of the 256 compute units.
// Fitted on MI355X to 330 products (16 .. 4096 rows, 320 .. 20000 columns, K 512 .. 28672; mean error 8 .. 15 %).  On 240 others
// (profiles/gemm_mx_kernel_choice.txt: 16 .. 8192 rows, K 256 .. 28672, every variant's time) the estimate of the chosen variant is off by 10 % in
// the mean, and the choice is 0.9 % behind the fastest variant in the geometric mean, 19 % at worst.  On 260 more, with 96 x 64 and weights not in the
// Infinity Cache (40 .. 1100 rows, 800 .. 24000 columns, K 512 .. 14000), 1.9 %, 22 % at worst (K = 512).
struct cost_t {
    int tm, tn;
    double start, alone, busy, tile;
};
// (96 x 64: fitted to 140 products of M 72 .. 384, N 2048 .. 16384, K 1024 .. 8192.  200 products of M 40 .. 2000, N 600 .. 30000, K 512 .. 14000 that it is chosen for:
// geometric mean 1.14 over the other variants' choice, 0.984 .. 1.40.)
constexpr cost_t COST[6] = {{128, 128, 0.9, 0.743, 0.521, 3.2},
                            {128, 128, 0.2, 0.448, 0.500, 5.0},
                            {64, 64, 2.8, 0.138, 0.222, 1.4},
                            {32, 64, 3.0, 0.172, 0.153, 0.6},
                            {32, 32, 2.5, 0.135, 0.111, 0.6},
                            {96, 64, 0.4, 0.390, 0.250, 4.9}};

} // namespace small

} // namespace

int configure_gemm_mx_small()
{
    static device_once_t once;
    int dev = 0;
    int rc = check_hip(hipGetDevice(&dev));
    if (rc != ADAHOP_OK || !once.need(dev)) return rc;
    using namespace small;
    if ((rc = v128_t::configure()) != ADAHOP_OK || (rc = v128one_t::configure()) != ADAHOP_OK ||
        (rc = v64x256_t::allow<false, false, float>()) != ADAHOP_OK || (rc = v64x256_t::allow<true, false, float>()) != ADAHOP_OK ||
        (rc = v128deep_t::configure()) != ADAHOP_OK ||
        (rc = v64_t::configure()) != ADAHOP_OK || (rc = v32x64_t::configure()) != ADAHOP_OK ||
        (rc = v32_t::configure()) != ADAHOP_OK || (rc = v96x64_t::configure()) != ADAHOP_OK)
        return rc;
    once.mark(dev);
    return ADAHOP_OK;
}

template <typename OUT>
static int launch_small_t(int variant, int64_t M, int64_t N, int64_t K, const uint8_t *a, small::scale_src_t as, const uint8_t *b,
                          small::scale_src_t bs, OUT *C, int64_t ldc, const uint16_t *Ag, const uint16_t *Bg, int kpad,
                          hipStream_t st)
{
    using namespace small;
    switch (variant) {
    case 0:
        if (K <= 192 && kpad == 0) {
            const bool streamed = c_rows_streamed(C, ldc * 4);
            if constexpr (sizeof(OUT) == 4) {
                if (streamed && M * N > (20 << 20)) return v64x256_t::launch(M, N, K, a, as, b, bs, C, ldc, Ag, Bg, kpad, st);
            }
            if (sizeof(OUT) == 2 || streamed || M * N <= (16 << 20))
                return v128one_t::launch(M, N, K, a, as, b, bs, C, ldc, Ag, Bg, kpad, st);
        }
        return v128_t::launch(M, N, K, a, as, b, bs, C, ldc, Ag, Bg, kpad, st);
    case 1: return v128deep_t::launch(M, N, K, a, as, b, bs, C, ldc, Ag, Bg, kpad, st);
    case 2: return v64_t::launch(M, N, K, a, as, b, bs, C, ldc, Ag, Bg, kpad, st);
    case 3: return v32x64_t::launch(M, N, K, a, as, b, bs, C, ldc, Ag, Bg, kpad, st);
    case 4: return v32_t::launch(M, N, K, a, as, b, bs, C, ldc, Ag, Bg, kpad, st);
    case 5: return v96x64_t::launch(M, N, K, a, as, b, bs, C, ldc, Ag, Bg, kpad, st);
    }
    return ADAHOP_E_INVALID_ARG;
}

// The fastest of the first `variants` variants for a product of `stages` pipeline stages, and what it is expected to take.
int gemm_mx_small_pick(int64_t M, int64_t N, int64_t stages, double *us, int variants)
{
    int best = 0;
    for (int v = 0; v < variants; ++v) {
        const small::cost_t &c = small::COST[v];
        const double L = (double)ceil_div(ceil_div(M, c.tm) * ceil_div(N, c.tn), 256);
        if (v == 5 && L > 1.0) continue; // (see v96x64_t)
        const double each = c.alone > c.busy * L ? c.alone : c.busy * L;
        const double t = c.start + (double)stages * each + c.tile * L;
        if (v == 0 || t < *us) {
            *us = t;
            best = v;
        }
    }
    return best;
}

bool gemm_mx_small_takes_canonical(int64_t K) { return ceil_div(K, 256) <= small::PRE_STAGES; }

int launch_gemm_mx_small(int variant, int64_t M, int64_t N, int64_t K, const uint8_t *a_codes, const uint8_t *a_scales, int a_sm,
                         const uint8_t *b_codes, const uint8_t *b_scales, int b_sm, void *C, int64_t ldc, int c_bf16,
                         const uint16_t *Ag, const uint16_t *Bg, int kpad, hipStream_t st)
{
    const int rc = configure_gemm_mx_small();
    if (rc != ADAHOP_OK) return rc;
    const int64_t KB = K / 32;
    // canonical scales that cannot be copied stage by stage: 8 bytes of every row, 4-byte aligned
    const bool any = KB % 8 != 0 || !aligned(a_sm ? nullptr : a_scales, 4) || !aligned(b_sm ? nullptr : b_scales, 4);
    const uint32_t rows_of = any ? (uint32_t)(((1 << 20) + KB - 1) / KB) : 0u;
    const small::scale_src_t as = {a_scales, a_sm ? 8 : KB, a_sm ? M * 8 : 8, a_sm ? 0u : rows_of},
                             bs = {b_scales, b_sm ? 8 : KB, b_sm ? N * 8 : 8, b_sm ? 0u : rows_of};
    if (c_bf16)
        return launch_small_t(variant, M, N, K, a_codes, as, b_codes, bs, static_cast<uint16_t *>(C), ldc, Ag, Bg, kpad, st);
    return launch_small_t(variant, M, N, K, a_codes, as, b_codes, bs, static_cast<float *>(C), ldc, Ag, Bg, kpad, st);
}

} // namespace adahop
