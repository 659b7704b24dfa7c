// The top-k selection of one workgroup of NT threads with its keys in LDS (paper App. F item 1), for the kernel that
// does only this (foid.hip) and the one that quantises an operand beside it (quantize.hip).
#pragma once
#include "common.h"

namespace adahop {

namespace {

constexpr int TOPK_THREADS = 1024, TOPK_WAVES = TOPK_THREADS / 64; // of the kernel that does nothing else

// The selection for dim <= TOPK_LDS_KEYS with every key staged in LDS once: wave w owns the contiguous index
// range [w*per, (w+1)*per) throughout.
//
// One workgroup is all the parallelism there is, and it runs every instruction of the kernel once or a few times
// only: what such a kernel costs is, first, the instruction lines it has to fetch (the cache is cold at every launch;
// a version of this kernel with the keys in registers and every loop unrolled spent most of its 12-18 us there) and,
// second, the number of passes over all keys.  So every pass is a rolled loop over keys in LDS, the select and the
// compaction exist once each (they run over a list described by a few numbers), and the passes over all keys are light:
//   1. every thread takes the maximum of the keys it loads; the k-th largest of these NT maxima, cut down to its
//      upper 16 bits (two radix passes over ONE value per thread), is a threshold T0 that at least k keys reach -- so
//      the k largest keys, and every key tied with the k-th, are among the keys >= T0 -- and that few others reach
//      (about 1.2 k of them for scores without structure).  With fewer than k threads that own a key the threshold
//      comes out as 0 and step 2 finds too many candidates, which is handled there;
//   2. the keys >= T0 are counted per wave and then copied, with their indices, to a list in index order (a compare
//      per key in each of the two passes);
//   3. radix select and ordered compaction run over this list (at most TOPK_CAND / NT entries per thread).
// If k > NT, or more than TOPK_CAND keys reach T0, or there are no more keys than four per thread, the list is
// the keys themselves.
constexpr int TOPK_LDS_KEYS = 32768;
constexpr int TOPK_CAND = 2048;

// hist[bin] += 1 for every lane with valid set: one combined add for the bin of the first valid lane (the scores of
// ordinary rows share their high bytes, so that bin usually takes most of the wave), plain per-lane adds for the rest.
__device__ __forceinline__ void wave_histogram_once(uint32_t *hist, bool valid, uint32_t bin)
{
    const uint64_t todo = __ballot(valid);
    if (todo == 0) return;
    const int leader = __ffsll((long long)todo) - 1;
    const uint32_t b = __builtin_amdgcn_readlane(bin, leader);
    const uint64_t same = __ballot(valid && bin == b);
    if ((int)(threadIdx.x & 63) == leader) atomicAdd(&hist[b], (uint32_t)__popcll(same));
    if (valid && bin != b) atomicAdd(&hist[bin], 1u);
}

// Inclusive sum over the lanes of a wave (all 64 active): four shifts within the rows of 16 lanes, then the row totals
// handed on to the following rows.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false); // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false); // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false); // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false); // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false); // lane 15 of rows 0, 2 to rows 1, 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false); // lane 31 to rows 2, 3
    return v;
}

struct topk_shared_t { // behind the keys
    uint32_t hist[2][256];              // used in turn by the radix passes, each cleared again after its pass
    uint32_t cand[TOPK_CAND];           // first the 1024 thread maxima, then the keys >= T0 in index order
    uint16_t cand_i[TOPK_CAND];         // and their indices (< TOPK_LDS_KEYS)
    uint32_t prefix, remaining, whole_bin, unused;
    uint32_t wave_a[TOPK_WAVES], wave_b[TOPK_WAVES];
};
static_assert(TOPK_LDS_KEYS <= 65536, "candidate indices are kept in 16 bits");

template <int NT> constexpr int topk_per_wave(int n) { return ((n + NT / 64 - 1) / (NT / 64) + 63) / 64 * 64; }
template <int NT> constexpr size_t topk_lds_bytes(int dim) { return (size_t)topk_per_wave<NT>(dim) * (NT / 64) * 4 + sizeof(topk_shared_t); }
static_assert(topk_lds_bytes<TOPK_THREADS>(TOPK_LDS_KEYS) <= 160 * 1024, "keys, histograms and candidates share one compute unit's LDS");

// pos1 (or nullptr): the position in idx + 1 of every selected index, 0 for the others; not in the memory of the scores,
// which a caller finds there afterwards.  skeys: topk_lds_bytes<NT>(dim) of LDS, per * NW keys, then topk_shared_t.
// dim <= 2048 NT / 64 (eight 16-byte loads per lane).
template <int NT>
__device__ __forceinline__ void topk_lds(const float *scores, int dim, int k, int32_t *__restrict__ idx, uint8_t *__restrict__ mask,
                                         uint16_t *pos1, uint32_t *skeys)
{
    constexpr int NW = NT / 64, TOPK_DIRECT = 4 * NT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6); // (a scalar: loop bounds derived from it are uniform)
    const uint32_t *keys = reinterpret_cast<const uint32_t *>(scores);
    const int per = topk_per_wave<NT>(dim); // <= 2048
    const int lo = w * per, hi = min(dim, lo + per);
    const int nslice = hi > lo ? (hi - lo + 63) / 64 : 0; // 64-key slices of this wave that hold keys
    topk_shared_t &sh = *reinterpret_cast<topk_shared_t *>(skeys + per * NW);

    if (k <= 0) {
        for (int i = tid; i < dim; i += NT) mask[i] = 0;
        return;
    }

    // 0. the wave's keys into LDS (a wave reads back only what it wrote itself: no barrier), the thread's maximum,
    // and the mask cleared (the selected entries are set at the end, many barriers later)
    uint32_t tmax = 0;
    if (((reinterpret_cast<uintptr_t>(keys) & 15) | (reinterpret_cast<uintptr_t>(mask) & 3)) == 0) {
        // 16 bytes per lane, all loads of the wave in flight together (per <= 2048 = 8 x 256)
        uint4 u[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int o = 256 * q + 4 * lane, i = lo + o; // (per is a multiple of 64, not of 256)
            u[q] = make_uint4(0u, 0u, 0u, 0u);
            if (o < per) {
                if (i + 3 < hi) {
                    u[q] = *reinterpret_cast<const uint4 *>(keys + i);
                    *reinterpret_cast<uint32_t *>(mask + i) = 0u;
                } else { // (one lane of one wave at most)
                    if (i < hi) u[q].x = keys[i], mask[i] = 0;
                    if (i + 1 < hi) u[q].y = keys[i + 1], mask[i + 1] = 0;
                    if (i + 2 < hi) u[q].z = keys[i + 2], mask[i + 2] = 0;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int o = 256 * q + 4 * lane;
            if (o < per) {
                *reinterpret_cast<uint4 *>(skeys + lo + o) = u[q];
                tmax = max(max(tmax, u[q].x), max(max(u[q].y, u[q].z), u[q].w));
            }
        }
    } else {
#pragma unroll 4
        for (int i = lo + lane; i < hi; i += 64) {
            const uint32_t key = keys[i];
            mask[i] = 0;
            skeys[i] = key;
            tmax = max(tmax, key);
        }
    }

    // The list that the final select and the compaction run over: entries [c_lo, c_hi) of src are this wave's part
    // (in index order over the waves; c_n slices of 64), entry p standing for index p (the keys themselves) or
    // cand_i[p] (candidates).  Entries up to the end of the last slice may be read (and are ignored).
    const uint32_t *src = skeys;
    int c_lo = lo, c_hi = hi, c_n = nslice;
    bool direct = true;

    // 1./2. radix select, once over the thread maxima (gives T0) and once over the list: digits of 8 bits from bit 24
    // down to bit last_shift.  After a use `prefix` holds the upper bits of the k-th largest key and `remaining` how
    // many keys with exactly these upper bits are among the k largest.  Over the list it stops at the first digit at
    // which the k largest keys are exactly the keys of the found bin and of the bins above it (well separated
    // outliers: usually the first or second digit): the remaining digits cannot change the selection then; `prefix`
    // then has zeros below that digit and `remaining` is UINT32_MAX, which says "every key >= prefix is selected".
    bool maxima = dim > TOPK_DIRECT && k <= NT;
    if (maxima) sh.cand[tid] = tmax;
    for (int j = tid; j < 512; j += NT) sh.hist[0][j] = 0; // (both histograms)
    __syncthreads();
    if (pos1) // every wave has its keys
        for (int i = tid; i < (dim + 1) / 2; i += NT) reinterpret_cast<uint32_t *>(pos1)[i] = 0u;
    int pass = 0;
    uint32_t T = 0, T0 = 0, remaining = (uint32_t)k;
    const uint64_t below = ((uint64_t)1 << lane) - 1;
    for (;;) {
        const uint32_t *from = maxima ? sh.cand : src;
        const int first = maxima ? tid : c_lo + lane;
        const int end = maxima ? 64 * (w + 1) : c_hi; // (the maxima: one per thread, the wave's own 64)
        const int n = maxima ? 1 : c_n;
        const int last_shift = maxima ? 16 : 0;
        uint32_t prefix = 0, pmask = 0;
        remaining = (uint32_t)k;
        for (int shift = 24; shift >= last_shift; shift -= 8) {
            uint32_t *hist = sh.hist[pass & 1]; // (all zeros: cleared two passes ago, or before the first)
            ++pass;
            for (int j = 0; j < n; j += 2) { // (two reads in flight; what lies past the list is ignored)
                const int i0 = first + 64 * j, i1 = i0 + 64;
                const uint32_t key0 = from[i0], key1 = from[i1];
                const bool in0 = i0 < end && (key0 & pmask) == prefix, in1 = i1 < end && (key1 & pmask) == prefix;
                if (__ballot(in0)) wave_histogram_once(hist, in0, (key0 >> shift) & 255u);
                if (__ballot(in1)) wave_histogram_once(hist, in1, (key1 >> shift) & 255u);
            }
            __syncthreads();
            // The digit of the k-th largest key: the highest bin b with (keys in bins above b) + count[b] >= remaining.
            // Wave 0 scans the 256 bins in parallel: lane l owns bins 255 - 4l .. 252 - 4l.
            if (w == 0) {
                const uint4 h = *reinterpret_cast<const uint4 *>(&hist[252 - 4 * lane]);
                const uint32_t c[4] = {h.w, h.z, h.y, h.x};
                const uint32_t mine = c[0] + c[1] + c[2] + c[3];
                uint32_t cum = wave_inclusive_sum(mine) - mine; // keys in bins above this lane's (lanes = descending bins)
                int found = -1;
                uint32_t cum_at = 0, c_at = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (found < 0 && cum + c[j] >= remaining) {
                        found = 255 - 4 * lane - j;
                        cum_at = cum;
                        c_at = c[j];
                    }
                    cum += c[j];
                }
                const uint64_t hit = __ballot(found >= 0);
                if (hit && lane == __ffsll((long long)hit) - 1) {
                    sh.prefix = prefix | ((uint32_t)found << shift);
                    sh.remaining = remaining - cum_at;
                    sh.whole_bin = c_at == remaining - cum_at ? 1u : 0u;
                }
            }
            __syncthreads();
            if (tid < 256) hist[tid] = 0; // for the pass after the next (barriers in between)
            prefix = sh.prefix;
            remaining = sh.remaining;
            pmask |= 255u << shift;
            const bool stop = !maxima && shift > last_shift && sh.whole_bin; // (uniform: every thread reads the same word)
            if (stop || shift == last_shift) __syncthreads(); // what comes next must not overtake these reads
            if (stop) {
                remaining = 0xffffffffu;
                break;
            }
        }
        if (!maxima) {
            // (stopped early over the candidates, the threshold may lie below T0, where keys that are no candidates begin)
            T = max(prefix, T0);
            break;
        }
        maxima = false;
        T0 = prefix; // upper 16 bits of the k-th largest maximum, lower bits 0
        // the keys >= T0: how many in this wave's part, in the parts before it, and in all
        // (four reads in flight; what lies past the wave's part is ignored)
        uint32_t mine = 0;
        for (int j = 0; j < nslice; j += 4) {
            uint32_t key[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) key[q] = skeys[lo + 64 * (j + q) + lane];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                mine += (uint32_t)__popcll(__ballot(lo + 64 * (j + q) + lane < hi && key[q] >= T0));
        }
        if (lane == 0) sh.wave_a[w] = mine;
        __syncthreads();
        uint32_t pos = 0, count = 0;
        for (int v = 0; v < NW; ++v) {
            const uint32_t c = sh.wave_a[v];
            pos += v < w ? c : 0u;
            count += c;
        }
        pos = __builtin_amdgcn_readfirstlane(pos);
        count = __builtin_amdgcn_readfirstlane(count);
        if (count <= (uint32_t)TOPK_CAND) {
            // copied in index order, with their indices
            for (int j = 0; j < nslice; j += 4) {
                uint32_t key[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) key[q] = skeys[lo + 64 * (j + q) + lane];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = lo + 64 * (j + q) + lane;
                    const bool c = i < hi && key[q] >= T0;
                    const uint64_t m = __ballot(c);
                    if (m) { // (most slices hold no candidate)
                        if (c) {
                            const uint32_t p = pos + (uint32_t)__popcll(m & below);
                            sh.cand[p] = key[q];
                            sh.cand_i[p] = (uint16_t)i;
                        }
                        pos += (uint32_t)__popcll(m);
                    }
                }
            }
            const int per_c = topk_per_wave<NT>((int)count);
            src = sh.cand;
            direct = false;
            c_lo = w * per_c;
            c_hi = min((int)count, c_lo + per_c);
            c_n = c_hi > c_lo ? (c_hi - c_lo + 63) / 64 : 0;
        }
        __syncthreads();
    }

    // 3. ordered compaction over the list
    uint32_t gt = 0, eq = 0;
#pragma unroll 2
    for (int j = 0; j < c_n; ++j) {
        const int i = c_lo + 64 * j + lane;
        const uint32_t key = src[i];
        gt += (uint32_t)__popcll(__ballot(i < c_hi && key > T));
        eq += (uint32_t)__popcll(__ballot(i < c_hi && key == T));
    }
    if (lane == 0) {
        sh.wave_a[w] = gt;
        sh.wave_b[w] = eq;
    }
    __syncthreads();
    uint32_t gt_before = 0, eq_before = 0;
    for (int v = 0; v < w; ++v) {
        gt_before += sh.wave_a[v];
        eq_before += sh.wave_b[v];
    }
#pragma unroll 2
    for (int j = 0; j < c_n; ++j) {
        const int i = c_lo + 64 * j + lane;
        const bool in = i < c_hi;
        const uint32_t key = src[i];
        const bool is_gt = in && key > T, is_eq = in && key == T;
        const uint64_t m_gt = __ballot(is_gt), m_eq = __ballot(is_eq);
        const uint32_t my_gt = gt_before + (uint32_t)__popcll(m_gt & below);
        const uint32_t my_eq = eq_before + (uint32_t)__popcll(m_eq & below);
        // selected entries before this one: every greater key, and the equal keys that were taken
        if (is_gt || (is_eq && my_eq < remaining)) {
            const int index = direct ? i : (int)sh.cand_i[i];
            const uint32_t at = my_gt + min(my_eq, remaining);
            idx[at] = index;
            mask[index] = 1;
            if (pos1) pos1[index] = (uint16_t)(at + 1);
        }
        gt_before += (uint32_t)__popcll(m_gt);
        eq_before += (uint32_t)__popcll(m_eq);
    }
}

} // namespace

} // namespace adahop
