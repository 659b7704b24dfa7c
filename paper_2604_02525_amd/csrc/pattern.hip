// Outlier-pattern detection of one tensor (paper Sec. 4.1, App. A) and the pattern-pair -> strategy
// table (Sec. 4.2).
//
// For an operand in its logical [outer, K] shape: the variance of every outer index (over its K
// elements) and of every K index (over the outer elements); the coefficient of variation of each of
// the two variance vectors, CV = std(v) / (mean(v) + eps); each CV divided by its value for IID
// data, sqrt(2 / (samples - 1)); and the class: "outer-wise" if CV^_outer / CV^_k > tau, "K-wise" if
// CV^_k / CV^_outer > tau, else none.  In the paper's notation (A is m x k, B is k x n) outer-wise is
// Row-wise for A and Column-wise for B, K-wise is Column-wise for A and Row-wise for B.
//
// All sums are kept in fp64 (the inputs are bf16, so x and x^2 are exact in fp64 and the variances
// follow from sum and sum of squares without cancellation trouble); variances are population
// variances, as are the standard deviations of the variance vectors.
//
//   k_pattern_partial  one pass over the stored matrix S[R][C]: a workgroup takes 256 rows x 512
//                      columns and writes, per row, its sum / sum of squares over the 512 columns,
//                      and per column over the 256 rows (no atomics); k_pattern_partial_small for tensors of few
//                      such blocks;
//   k_pattern_fold     adds the partials of every row and every column in a fixed order, forms the variances and
//                      sums them and their squares over 32 neighbours;
//   k_pattern_finish   one workgroup adds these and writes the class and the four CV figures.
#include "common.h"

#include <type_traits>

namespace adahop {

namespace {

constexpr int PT_ROWS = 256, PT_COLS = 512;

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_down(v, d);
    return v; // valid in lane 0
}

// x and y of the pair handed on: the lower half of the wave (MASK = 32; of a pair of rows of 16: the even one, MASK = 16) ends
// with x summed over both halves, the other with y.
template <int MASK> __device__ __forceinline__ double halve(double x, double y)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const uint64_t xb = (uint64_t)__double_as_longlong(x), yb = (uint64_t)__double_as_longlong(y);
    u32x2 lo, hi;
    if constexpr (MASK == 32) {
        lo = __builtin_amdgcn_permlane32_swap((unsigned)xb, (unsigned)yb, false, false);
        hi = __builtin_amdgcn_permlane32_swap((unsigned)(xb >> 32), (unsigned)(yb >> 32), false, false);
    } else {
        lo = __builtin_amdgcn_permlane16_swap((unsigned)xb, (unsigned)yb, false, false);
        hi = __builtin_amdgcn_permlane16_swap((unsigned)(xb >> 32), (unsigned)(yb >> 32), false, false);
    }
    return __longlong_as_double((long long)((uint64_t)hi.x << 32 | lo.x)) + __longlong_as_double((long long)((uint64_t)hi.y << 32 | lo.y));
}

template <int CTRL> __device__ __forceinline__ double dpp_double(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// rowpart[cb][r] = (sum, sumsq) of row r over column block cb; colpart[rb][c] likewise.  A lane keeps 8 columns of the block, a
// wave takes consecutive rows.
//
// Bound by the reads, beside fp64 sums (five fp64 instructions per element, and what the row sums take across the lanes: those
// of 8 rows (16 numbers per lane) are halved together: every exchange leaves a lane with half as many numbers summed over
// twice as many lanes, 63 instructions for 8 rows, where a reduction for each row by itself was 288, two thirds of them through the LDS;
// 16384 x 8192: 91 -> 64 us).
// In a whole block (256 rows x 512 columns, all in memory) a wave keeps eight rows on their way and asks for the next one as soon as one is
// read, and which rows the waves in flight are at counts as much: at a row pitch of 16 KB the waves of all blocks, reading row w + 8 i at about the
// same time, meet on the same memory channels.  Reads alone: 5.6 TB/s so, 6.5 with 32 consecutive rows per wave, 6.8 with
// these also begun an eighth of a block further from wave to wave and from block to block (4096 x 32768 6.5 / 4.9 / 6.7); the detector, 16384 x 8192
// 66.0 -> 55.5 us, 28672 x 8192 108 -> 92, 8192 x 8192 39.9 -> 32.4, 16384 x 4096 40 -> 36.
// W waves: 8 (two workgroups per compute unit), and 16 where there are fewer workgroups than compute units.
template <int W>
__global__ __launch_bounds__(64 * W, 4) void k_pattern_partial(const uint16_t *__restrict__ S, int64_t ld, int64_t R, int64_t C,
                                                            double2 *__restrict__ rowpart, double2 *__restrict__ colpart)
{
    __shared__ double2 scol[W][PT_COLS]; // column 8 l + j of the block at 64 j + l
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r0 = (int64_t)blockIdx.y * PT_ROWS, c0 = (int64_t)blockIdx.x * PT_COLS + lane * 8;
    double cs[8], cq[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) cs[j] = cq[j] = 0.0;
    const bool whole = c0 + 8 <= C; // C % 8 == 0 is not required: what lies behind a row counts as 0
    const int mine = (int)min((int64_t)PT_ROWS, R - r0); // rows of this block
    // Every 16-byte piece of the block lies inside the matrix, from its first element to its last one: all but the last rows of the
    // last columns where C % 8 != 0.
    const int64_t cb = (int64_t)blockIdx.x * PT_COLS, cend = min(cb + PT_COLS, (C + 7) / 8 * 8), end = (R - 1) * ld + C;
    const bool clean = (r0 + mine - 1) * ld + cend <= end;
    const uint16_t *const mycol = S + (c0 < C ? c0 : cb);

    const int per = ((mine + W - 1) / W + 7) & ~7, first = w * per; // the wave's rows
    // A clean block's loads have no condition (rows behind the last one read that again and are cleared at their use): of loads under a
    // lane's condition the compiler waits for some before it asks for the next.
    enum { WHOLE, CLEAN, EDGE };
    const auto row_of = [&](auto kind, int i) { // the i-th row of the wave
        if (decltype(kind)::value != WHOLE) return first + i;
        return w * (PT_ROWS / W) + ((i + 8 * (int)(blockIdx.y + w)) & (PT_ROWS / W - 1));
    };
    const auto load_row = [&](auto kind, int i) {
        const int r = row_of(kind, i);
        if constexpr (decltype(kind)::value == WHOLE) {
            return load_once16(reinterpret_cast<const uint8_t *>(S + (r0 + r) * ld + cb) + lane * 16);
        } else if constexpr (decltype(kind)::value == CLEAN) {
            return load_once16(mycol + (r0 + min(r, mine - 1)) * ld);
        } else {
            uint4 u = make_uint4(0, 0, 0, 0);
            if (r < mine) {
                const uint16_t *p = S + (r0 + r) * ld + c0;
                if (c0 < C && (r0 + r) * ld + c0 + 8 <= end) { // (behind a row there is the next one, or what its stride leaves)
                    u = load_once16(p);
                } else if (c0 < C) { // the last chunk of the last row
                    u = load_part16(p, (int)min((int64_t)8, C - c0));
                }
            }
            return u;
        }
    };
    // Eight rows of the wave from i0 on, in u; used(n) follows the last use of u[n].
    const auto eight_rows = [&](auto kind, int i0, uint4(&u)[8], auto &&used) {
        constexpr bool whole_block = decltype(kind)::value == WHOLE;
        // number 2 t of the 16: the sum of row t, 2 t + 1: its sum of squares.  Rows t and t + 4 one after the other, their numbers
        // halved at once, and no row begun before: more rows under way take more registers than two workgroups have.
        double v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            double n4[2][2];
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                uint32_t word[4] = {u[t + 4 * y].x, u[t + 4 * y].y, u[t + 4 * y].z, u[t + 4 * y].w};
                if (!whole_block && row_of(kind, i0 + t + 4 * y) >= mine) word[0] = word[1] = word[2] = word[3] = 0;
                if (!whole_block && !whole) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) word[j] &= (c0 + 2 * j < C ? 0xffffu : 0u) | (c0 + 2 * j + 1 < C ? 0xffff0000u : 0u);
                }
                asm volatile("" : "+v"(word[0]), "+v"(word[1]), "+v"(word[2]), "+v"(word[3]));
                __builtin_amdgcn_sched_barrier(0);
                used(t + 4 * y);
                __builtin_amdgcn_sched_barrier(0);
                double rs = 0.0, rq = 0.0;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const double x = (double)(j & 1 ? bf16_hi(word[j >> 1]) : bf16_lo(word[j >> 1]));
                    rs += x;
                    rq = __builtin_fma(x, x, rq); // (the square is exact: fused or not, the same sums)
                    cs[j] += x;
                    cq[j] = __builtin_fma(x, x, cq[j]);
                }
                // (here, not at the end of the loop body, where the compiler would add a whole iteration's elements, kept in registers)
                asm volatile("" : "+v"(cs[0]), "+v"(cs[1]), "+v"(cs[2]), "+v"(cs[3]), "+v"(cs[4]), "+v"(cs[5]), "+v"(cs[6]), "+v"(cs[7]));
                asm volatile("" : "+v"(cq[0]), "+v"(cq[1]), "+v"(cq[2]), "+v"(cq[3]), "+v"(cq[4]), "+v"(cq[5]), "+v"(cq[6]), "+v"(cq[7]));
                n4[y][0] = rs;
                n4[y][1] = rq;
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const double both = halve<32>(n4[0][k], n4[1][k]);
                v[2 * (t & 1) + k] = t < 2 ? both : halve<16>(v[2 * (t & 1) + k], both);
            }
        }
        const bool b3 = lane & 8, b2 = lane & 4;
#pragma unroll
        for (int k = 0; k < 2; ++k) // lane ^ 8
            v[k] = (b3 ? v[k + 2] : v[k]) + dpp_double<0x128>(b3 ? v[k] : v[k + 2]);
        double s = (b2 ? v[1] : v[0]) + dpp_double<0x141>(b2 ? v[0] : v[1]); // lane ^ 7
        s += dpp_double<0xB1>(s);                                            // lane ^ 1
        s += dpp_double<0x4E>(s);                                            // lane ^ 2
        // the quad q = lane / 4 holds number q of the 16
        const int r = row_of(kind, i0 + (lane >> 3));
        if ((lane & 3) == 0 && r < mine)
            reinterpret_cast<double *>(rowpart + (int64_t)blockIdx.x * R + r0 + r)[(lane >> 2) & 1] = s;
    };
    const auto rows_in_turn = [&](auto kind) {
        for (int i0 = 0; i0 < per; i0 += 8) {
            if (first + i0 >= mine) break;
            uint4 u[8]; // eight rows of the wave are in flight together, asked for in the order of their use
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                u[t] = load_row(kind, i0 + t);
                u[t + 4] = load_row(kind, i0 + t + 4);
            }
            eight_rows(kind, i0, u, [](int) {});
        }
    };
    if (clean && mine == PT_ROWS && cb + PT_COLS <= C) {
        const std::integral_constant<int, WHOLE> kind{};
        uint4 u[8];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            u[t] = load_row(kind, t);
            u[t + 4] = load_row(kind, t + 4);
        }
#pragma unroll
        for (int i0 = 0; i0 < PT_ROWS / W; i0 += 8)
            eight_rows(kind, i0, u, [&](int n) {
                if (i0 + 8 < PT_ROWS / W) u[n] = load_row(kind, i0 + 8 + n);
            });
    } else if (clean) {
        rows_in_turn(std::integral_constant<int, CLEAN>{});
    } else {
        rows_in_turn(std::integral_constant<int, EDGE>{});
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) scol[w][64 * j + lane] = make_double2(cs[j], cq[j]);
    __syncthreads();
    for (int k = tid; k < PT_COLS; k += 64 * W) {
        const int64_t cg = (int64_t)blockIdx.x * PT_COLS + 8 * (k & 63) + (k >> 6);
        if (cg < C) {
            double2 a = scol[0][k];
#pragma unroll
            for (int x = 1; x < W; ++x) {
                a.x += scol[x][k].x;
                a.y += scol[x][k].y;
            }
            colpart[(int64_t)blockIdx.y * C + cg] = a;
        }
    }
}

// The same for a tensor of few blocks, whose fp64 sums a few compute units would do: rows and columns by themselves, in smaller pieces that leave
// the same partials: 256 rows x 512 columns take one compute unit 6 us of vector instructions.  The first row_wgs workgroups take 32 rows x 512 columns and sum the rows (a wave: 8 rows); the others 256 rows x 64
// columns and sum the columns (a thread: 8 columns of 8 rows).  Every element is read and converted twice, over sixteen times as many
// workgroups.  Whole blocks / small pieces, the detector: 20000 x 256 20.6 / 14.3 us, 2048 x 2048 16.8 / 14.2, 344 x 19168 (76 blocks) 20.5 / 15.8, but 4096 x
// 4096 (128) 18.7 / 19.6, 512 x 25000 (98) 20.1 / 21.2, 4096 x 7168 20.1 / 27.7.
constexpr int PS_ROWS = 32, PS_COLS = 64;
__global__ __launch_bounds__(256) void k_pattern_partial_small(const uint16_t *__restrict__ S, int64_t ld, int64_t R, int64_t C, int cb,
                                                               int row_wgs, double2 *__restrict__ rowpart, double2 *__restrict__ colpart)
{
    __shared__ double2 sums[4][PS_COLS];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool rows = (int)blockIdx.x < row_wgs;
    const int b = rows ? (int)blockIdx.x : (int)blockIdx.x - row_wgs;
    const int cols = rows ? PT_COLS : PS_COLS, across = rows ? cb : (int)((C + PS_COLS - 1) / PS_COLS);
    const int by = b / across, bx = b - by * across;
    const int64_t r0 = (int64_t)by * (rows ? PS_ROWS : PT_ROWS), rend = min(r0 + (rows ? PS_ROWS : PT_ROWS), R), cb0 = (int64_t)bx * cols;
    const int64_t first = r0 + 8 * (rows ? w : tid >> 3), c0 = cb0 + 8 * (rows ? lane : tid & 7); // the thread's 8 rows and 8 columns
    // (as in k_pattern_partial: a block that the matrix holds to its last piece loads without conditions)
    const int64_t end = (R - 1) * ld + C, cend = min(cb0 + cols, (C + 7) / 8 * 8);
    uint32_t word[8][4];
    if ((rend - 1) * ld + cend <= end) {
        const uint16_t *const mycol = S + (c0 < C ? c0 : cb0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint4 u = *reinterpret_cast<const uint4 *>(mycol + min(first + i, rend - 1) * ld);
            word[i][0] = u.x, word[i][1] = u.y, word[i][2] = u.z, word[i][3] = u.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            uint4 u = make_uint4(0, 0, 0, 0);
            const int64_t at = (first + i) * ld + c0;
            if (first + i < rend && c0 < C) u = at + 8 <= end ? *reinterpret_cast<const uint4 *>(S + at) : load_part16(S + at, (int)min((int64_t)8, C - c0));
            word[i][0] = u.x, word[i][1] = u.y, word[i][2] = u.z, word[i][3] = u.w;
        }
    }
    uint32_t keep[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) keep[j] = (c0 + 2 * j < C ? 0xffffu : 0u) | (c0 + 2 * j + 1 < C ? 0xffff0000u : 0u);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) word[i][j] = first + i < rend ? word[i][j] & keep[j] : 0u;
    double v[16]; // rows: sum and sum of squares of row i at 2 i and 2 i + 1; columns: of column i at i and i + 8
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = 0.0;
    if (rows) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const double x = (double)(j & 1 ? bf16_hi(word[i][j >> 1]) : bf16_lo(word[i][j >> 1]));
                v[2 * i] += x;
                v[2 * i + 1] = __builtin_fma(x, x, v[2 * i + 1]);
            }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const double x = (double)(j & 1 ? bf16_hi(word[i][j >> 1]) : bf16_lo(word[i][j >> 1]));
                v[j] += x;
                v[8 + j] = __builtin_fma(x, x, v[8 + j]);
            }
    }
    // across the lanes 32, 16 and 8 apart: a lane keeps the numbers 8 b5 + 4 b4 + 2 b3 and the one behind it
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = halve<32>(v[k], v[k + 8]);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = halve<16>(v[k], v[k + 4]);
    const bool b3 = lane & 8;
#pragma unroll
    for (int k = 0; k < 2; ++k) v[k] = (b3 ? v[k + 2] : v[k]) + dpp_double<0x128>(b3 ? v[k] : v[k + 2]);
    if (rows) {
        const bool b2 = lane & 4;
        double s = (b2 ? v[1] : v[0]) + dpp_double<0x141>(b2 ? v[0] : v[1]); // lane ^ 7
        s += dpp_double<0xB1>(s);                                            // lane ^ 1
        s += dpp_double<0x4E>(s);                                            // lane ^ 2
        const int64_t r = first + (lane >> 3); // the quad q = lane / 4 holds number q of the 16
        if ((lane & 3) == 0 && r < rend) reinterpret_cast<double *>(rowpart + (int64_t)bx * R + r)[(lane >> 2) & 1] = s;
        return;
    }
    const int n = 8 * (lane >> 5) + 4 * ((lane >> 4) & 1) + 2 * ((lane >> 3) & 1);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        double2 &to = sums[w][8 * (lane & 7) + ((n + k) & 7)];
        (n + k < 8 ? to.x : to.y) = v[k];
    }
    __syncthreads();
    if (tid < PS_COLS && cb0 + tid < C) {
        double2 a = sums[0][tid];
#pragma unroll
        for (int x = 1; x < 4; ++x) {
            a.x += sums[x][tid].x;
            a.y += sums[x][tid].y;
        }
        colpart[(int64_t)by * C + cb0 + tid] = a;
    }
}

// The variances of FOLD_N rows or columns: their partials part[p * n + i] added in a fixed order, eight threads per index, and the
// block's sums of the variances and of their squares, which go to the place of the block's first partial (nobody else reads the
// partials of these indices).  Each variance is taken over `samples` elements.  Over the whole chip: in the one workgroup of
// k_pattern_finish these sums were most of the detector's time, and with one thread per index that walks up to 64 partials,
// 17 us (and 17 more for the statistics of 24576 sums in one workgroup; now 5 and 4).
constexpr int FOLD_N = 32;
__global__ __launch_bounds__(256) void k_pattern_fold(double2 *__restrict__ rowpart, int row_parts, double2 *__restrict__ colpart,
                                                      int col_parts, int64_t R, int64_t C, int row_blocks)
{
    __shared__ double2 sums[8][FOLD_N];
    const bool rows = (int)blockIdx.x < row_blocks;
    double2 *part = rows ? rowpart : colpart;
    const int64_t n = rows ? R : C, first = (int64_t)(rows ? blockIdx.x : blockIdx.x - row_blocks) * FOLD_N;
    const double samples = (double)(rows ? C : R);
    const int parts = rows ? row_parts : col_parts, x = threadIdx.x & (FOLD_N - 1), g = threadIdx.x / FOLD_N;
    const int64_t i = first + x;
    double s = 0.0, q = 0.0;
    if (i < n) {
#pragma unroll 4
        for (int p = g; p < parts; p += 8) {
            const double2 v = part[(int64_t)p * n + i];
            s += v.x;
            q += v.y;
        }
    }
    sums[g][x] = make_double2(s, q);
    __syncthreads();
    if (threadIdx.x >= 64) return;
    double a = 0.0, b = 0.0;
    if (threadIdx.x < FOLD_N && i < n) {
#pragma unroll
        for (int k = 1; k < 8; ++k) {
            s += sums[k][x].x;
            q += sums[k][x].y;
        }
        const double m = s / samples;
        double var = q / samples - m * m;
        if (var < 0.0) var = 0.0;
        a = var;
        b = var * var;
    }
    a = wave_sum(a);
    b = wave_sum(b);
    if (threadIdx.x == 0) part[first] = make_double2(a, b);
}

// (mean, mean of squares) of the n variances of one axis from the sums that k_pattern_fold left (block reduction through sh,
// fixed order).
__device__ void variance_stats(const double2 *__restrict__ part, int64_t n, double *sh, double &mean_v, double &mean_v2)
{
    double a = 0.0, b = 0.0;
    for (int64_t i = (int64_t)threadIdx.x * FOLD_N; i < n; i += (int64_t)blockDim.x * FOLD_N) {
        const double2 v = part[i];
        a += v.x;
        b += v.y;
    }
    a = wave_sum(a);
    b = wave_sum(b);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if (lane == 0) {
        sh[2 * w] = a;
        sh[2 * w + 1] = b;
    }
    __syncthreads();
    double ta = 0.0, tb = 0.0;
    for (int v = 0; v < nw; ++v) {
        ta += sh[2 * v];
        tb += sh[2 * v + 1];
    }
    mean_v = ta / (double)n;
    mean_v2 = tb / (double)n;
}

__device__ __forceinline__ double ratio_or_inf(double a, double b)
{
    if (b > 0.0) return a / b;
    return a > 0.0 ? __longlong_as_double(0x7ff0000000000000LL) : 0.0;
}

// stats_out: CV_outer, CV_k, CV^_outer, CV^_k.  rows_are_outer: the stored rows are the outer indices.
__global__ __launch_bounds__(512) void k_pattern_finish(const double2 *__restrict__ rowpart,
                                                         const double2 *__restrict__ colpart, int64_t R,
                                                         int64_t C, int rows_are_outer, double tau, double eps,
                                                         int32_t *__restrict__ pattern_out, double *__restrict__ stats_out)
{
    __shared__ double sh[32];
    double mr, mr2, mc, mc2;
    variance_stats(rowpart, R, sh, mr, mr2); // row variances: over the C columns
    variance_stats(colpart, C, sh, mc, mc2); // column variances: over the R rows
    if (threadIdx.x == 0) {
        double sr = mr2 - mr * mr, sc = mc2 - mc * mc;
        sr = sr > 0.0 ? sqrt(sr) : 0.0;
        sc = sc > 0.0 ? sqrt(sc) : 0.0;
        const double cv_row = sr / (mr + eps), cv_col = sc / (mc + eps);
        const double hat_row = cv_row / sqrt(2.0 / (double)(C - 1)), hat_col = cv_col / sqrt(2.0 / (double)(R - 1));
        const double cv_outer = rows_are_outer ? cv_row : cv_col, cv_k = rows_are_outer ? cv_col : cv_row;
        const double hat_outer = rows_are_outer ? hat_row : hat_col, hat_k = rows_are_outer ? hat_col : hat_row;
        int p = ADAHOP_PATTERN_NONE;
        if (ratio_or_inf(hat_outer, hat_k) > tau)
            p = ADAHOP_PATTERN_OUTER;
        else if (ratio_or_inf(hat_k, hat_outer) > tau)
            p = ADAHOP_PATTERN_K;
        *pattern_out = p;
        stats_out[0] = cv_outer;
        stats_out[1] = cv_k;
        stats_out[2] = hat_outer;
        stats_out[3] = hat_k;
    }
}

} // namespace

static void pattern_geometry(const adahop_operand_t &x, int64_t &R, int64_t &C, int64_t &rb, int64_t &cb)
{
    R = x.k_contig ? x.outer : x.K;
    C = x.k_contig ? x.K : x.outer;
    rb = ceil_div(R, PT_ROWS);
    cb = ceil_div(C, PT_COLS);
}

size_t pattern_workspace_bytes(const adahop_operand_t &x)
{
    int64_t R, C, rb, cb;
    pattern_geometry(x, R, C, rb, cb);
    return align_up((size_t)cb * R * sizeof(double2), 256) + align_up((size_t)rb * C * sizeof(double2), 256);
}

int launch_detect_pattern(const adahop_operand_t &x, double tau, double eps, int32_t *pattern_out, double *stats_out,
                          void *workspace, hipStream_t st)
{
    int64_t R, C, rb, cb;
    pattern_geometry(x, R, C, rb, cb);
    double2 *rowpart = static_cast<double2 *>(workspace);
    double2 *colpart = reinterpret_cast<double2 *>(static_cast<char *>(workspace) + align_up((size_t)cb * R * sizeof(double2), 256));
    const dim3 grid((unsigned)cb, (unsigned)rb);
    const uint16_t *d = static_cast<const uint16_t *>(x.data);
    if (cb * rb <= 80) {
        const int64_t row_wgs = cb * ceil_div(R, PS_ROWS), col_wgs = rb * ceil_div(C, PS_COLS);
        hipLaunchKernelGGL(k_pattern_partial_small, dim3((unsigned)(row_wgs + col_wgs)), dim3(256), 0, st, d, x.ld, R, C, (int)cb, (int)row_wgs, rowpart,
                           colpart);
    } else if (cb * rb < 256) {
        hipLaunchKernelGGL(k_pattern_partial<16>, grid, dim3(1024), 0, st, d, x.ld, R, C, rowpart, colpart);
    } else {
        hipLaunchKernelGGL(k_pattern_partial<8>, grid, dim3(512), 0, st, d, x.ld, R, C, rowpart, colpart);
    }
    int rc = check_launch();
    if (rc != ADAHOP_OK) return rc;
    const int row_blocks = (int)ceil_div(R, FOLD_N);
    hipLaunchKernelGGL(k_pattern_fold, dim3((unsigned)(row_blocks + ceil_div(C, FOLD_N))), dim3(256), 0, st, rowpart, (int)cb, colpart,
                       (int)rb, R, C, row_blocks);
    rc = check_launch();
    if (rc != ADAHOP_OK) return rc;
    hipLaunchKernelGGL(k_pattern_finish, dim3(1), dim3(512), 0, st, rowpart, colpart, R, C, x.k_contig ? 1 : 0, tau, eps,
                       pattern_out, stats_out);
    return check_launch();
}

} // namespace adahop
