// The search of many fp32 queries, with fp16 copies in front: the same exact top-k as xc_mine.hip (which includes this file).
// Bound of the fp32 kernels: the matrix pipe, whose fp32 products run at a sixteenth of the 16-bit rate.  z and w rounded to 11
// bits give a score that is off by at most half_error() |z| |w| (a thousandth of it), so the sweep over all labels runs on fp16
// copies with thresholds lowered by that, and the few labels left get their score from the fp32 rows, in the order of sums of the
// other kernels.  With e(q) a query's error for the largest row so far:
//   half_queries_kernel, half_rows_kernel   the copies, padded to whole tiles and stages, and the largest |w|
//   mine_tile_kernel / mine_rows_kernel     on them, as for bf16 rows.  A label passes if its 16-bit score reaches T = B - e(q),
//                                           where B is a score that k labels are known to reach: no label of the answer is lost
//   half_select_kernel                      B = (k-th best 16-bit score) - e(q), and the list cut to what can still matter
//   half_finish_kernel                      the fp32 scores of the list, the best k of them
// What this does not settle - a list that ran over, scores or rows out of fp16's range, a warm search whose thresholds were too
// high - is flagged by query tile, and the fp32 kernels take these tiles (they return at once where there are none).
#pragma once

#include "xc_mine.h"

namespace xc {

constexpr int64_t kHalfChunkBytes = 512ll << 20;     // fp16 rows held at a time
constexpr int64_t kHalfMaxRowBytes = 8192;           // of fp32 rows
constexpr float kHalfPlain = 0.0f, kHalfZero = 1.0f, kHalfBad = 2.0f;       // kinds of queries

constexpr int64_t kHalfWaveQueries = 2048;           // from so many queries on, a wave each forms the fp32 scores

struct HalfPlan {
    int64_t pitch;                                   // bytes of an fp16 row: whole stages; 0 = not used
    int64_t chunk;                                   // label tiles at a time
    size_t off_rows, off_z, off_zpar, off_stats, off_over, bytes;      // within its part of the workspace
};

// e(q) in units of the scaled scores.  zpar: (|z| scaled, B scaled, scale, kind)
__device__ __forceinline__ float half_query_error(const float4& zpar, const uint32_t* stats, int d) {
    return zpar.x * (sqrtf(__uint_as_float(stats[0])) * 1.001f * half_error(d) + half_error_small(d));
}

__global__ __launch_bounds__(256)
void half_queries_kernel(const unsigned char* __restrict__ Z, int64_t Zq, int64_t nq, int row_bytes, int pitch,
                         unsigned char* __restrict__ out, float4* __restrict__ zpar, uint32_t* __restrict__ stats) {
    const int lane = lane_id();
    const int64_t q = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (blockIdx.x == 0 && threadIdx.x < 2) stats[threadIdx.x] = 0u;
    if (q >= nq) return;
    const float* zr = reinterpret_cast<const float*>(Z + (q < Zq ? q : 0) * row_bytes);
    const int d = q < Zq ? row_bytes / 4 : 0;
    float m = 0.0f, s2 = 0.0f;
    for (int i = lane; i < d; i += kWave) {
        const float v = zr[i];
        m = fmaxf(m, fabsf(v) <= kHalfMost ? fabsf(v) : INFINITY);       // (infinite where it is no number, too)
        s2 = fmaf(v, v, s2);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { m = fmaxf(m, __shfl_xor(m, off, kWave)); s2 += __shfl_xor(s2, off, kWave); }
    const bool bad = m > kHalfMost || (m != 0.0f && m < kHalfLeast);
    const int e = m == 0.0f || bad ? 0 : 14 - (static_cast<int>(__float_as_uint(m) >> 23) - 127);         // largest element to [2^14, 2^15)
    const float up = ldexpf(1.0f, e);
    for (int i = lane; i < pitch / 2; i += kWave)
        reinterpret_cast<_Float16*>(out + q * pitch)[i] = static_cast<_Float16>(i < d && !bad ? zr[i] * up : 0.0f);
    if (lane == 0) {
        const float scale = up * kHalfScale;
        zpar[q] = make_float4(bad ? 0.0f : sqrtf(s2) * 1.001f * scale, -INFINITY, scale, q >= Zq || m == 0.0f ? kHalfZero : bad ? kHalfBad : kHalfPlain);
    }
}

// Rows [0, n_lab) of the chunk, LG lanes (a power of two) to a row; rows up to n_rows are zeros.  Bound: HBM (6 bytes per element).
__global__ __launch_bounds__(256)
void half_rows_kernel(const unsigned char* __restrict__ W, int64_t n_lab, int64_t n_rows, int row_bytes, int pitch, int LG,
                      unsigned char* __restrict__ out, uint32_t* __restrict__ stats) {
    __shared__ float sh[4][2];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int per = kWave / LG, l = lane & (LG - 1);
    const int64_t step = static_cast<int64_t>(gridDim.x) * 4 * per;
    float most = 0.0f, top = 0.0f;
    for (int64_t r0 = (static_cast<int64_t>(blockIdx.x) * 4 + wave) * per; r0 < n_rows; r0 += step) {
        const int64_t r = r0 + lane / LG;
        float s2 = 0.0f;
        for (int c = l; c * 16 < pitch; c += LG) {       // 8 elements: two chunks in, one out
            uint4 a = make_uint4(0, 0, 0, 0), b = make_uint4(0, 0, 0, 0);
            if (r < n_lab && c * 32 < row_bytes) a = load16<true>(W + r * row_bytes + c * 32);
            if (r < n_lab && c * 32 + 16 < row_bytes) b = load16<true>(W + r * row_bytes + c * 32 + 16);
            const float f[8] = {__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z), __uint_as_float(a.w),
                                __uint_as_float(b.x), __uint_as_float(b.y), __uint_as_float(b.z), __uint_as_float(b.w)};
            f16x8 h;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                s2 = fmaf(f[i], f[i], s2);
                top = fmaxf(top, fabsf(f[i]) <= 1e15f ? fabsf(f[i]) : INFINITY);
                h[i] = static_cast<_Float16>(f[i] * kHalfScale);
            }
            if (r < n_rows) *reinterpret_cast<f16x8*>(out + r * pitch + c * 16) = h;
        }
        for (int off = LG >> 1; off > 0; off >>= 1) s2 += __shfl_xor(s2, off, kWave);
        most = fmaxf(most, s2);                          // (of a row that is no number: see top)
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { most = fmaxf(most, __shfl_xor(most, off, kWave)); top = fmaxf(top, __shfl_xor(top, off, kWave)); }
    if (lane == 0) { sh[wave][0] = most; sh[wave][1] = top; }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < 4; ++w) { most = fmaxf(most, sh[w][0]); top = fmaxf(top, sh[w][1]); }
        atomicMax(&stats[0], __float_as_uint(most));
        if (top >= 65504.0f / kHalfScale) stats[1] = 1u;         // beyond fp16: everything goes to the fp32 kernels
    }
}

// Thresholds of the first sweep.  from: 0 none yet, 1 the k-th best 16-bit scores of the dense phase, 2 those of the search before,
// lowered by rel |tau| (fp32 scores).
__global__ void half_start_kernel(int from, float rel, uint32_t* __restrict__ tau_g, int32_t* __restrict__ gcnt, float4* __restrict__ zpar,
                                  const uint32_t* __restrict__ stats, int32_t* __restrict__ over /* [1 + n / kBN] */, int64_t n, int64_t Zq, int d) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (q <= n / kBN) over[q] = 0;
    if (q >= n) return;
    gcnt[q] = 0;
    const float4 zp = zpar[q];
    const float e = half_query_error(zp, stats, d);
    float base = -INFINITY;
    if (from == 1) base = ordered_to_float(tau_g[q]) - e;
    if (from == 2) { const float t = ordered_to_float(tau_g[q]); base = (t - rel * fabsf(t)) * zp.z; }
    zpar[q].y = base;
    tau_g[q] = float_to_ordered(q >= Zq || zp.w != kHalfPlain ? INFINITY : base - e);
}

// A query's list cut to the labels that can still be among the best k; the threshold of the next sweep.  By one wave.
__device__ int half_prune(uint64_t* list, int n, int k, float e, float* base, float* thr, int* hist, uint64_t* scratch) {
    const int lane = lane_id();
    if (n >= k) {
        float t;
        if (n == k || n > kSelectRegs * kWave) {
            const uint64_t bound = n == k ? kKeySentinel : wave_bound_stream(list, n, k, hist);
            uint64_t worst = 0;
            for (int i = lane; i < n; i += kWave) { const uint64_t key = list[i]; if (key <= bound && key > worst) worst = key; }
            t = key_score(wave_max_u64(worst));
        } else {
            auto at = [list](int idx) { return list[idx]; };
            t = n <= kSelectRegs / 2 * kWave ? wave_select_k<kSelectRegs / 2>(scratch, at, n, k, hist) : wave_select_k<kSelectRegs>(scratch, at, n, k, hist);
        }
        *base = fmaxf(*base, t - e);
    }
    *thr = *base - e;
    int out = 0;
    for (int i0 = 0; i0 < n; i0 += kWave) {              // in place: a chunk is read before anything of it is overwritten
        const uint64_t key = i0 + lane < n ? list[i0 + lane] : kKeySentinel;
        const bool keep = i0 + lane < n && key_score(key) >= *thr;
        const uint64_t bal = __ballot(keep);
        if (keep) list[out + __popcll(bal & lanemask_lt())] = key;
        out += __popcll(bal);
    }
    return out;
}

__global__ __launch_bounds__(256)
void half_select_kernel(uint64_t* __restrict__ glist, int32_t* __restrict__ gcnt, uint32_t* __restrict__ tau_g, float4* __restrict__ zpar,
                        const uint32_t* __restrict__ stats, int32_t* __restrict__ over, int64_t Zq, int glist_cap, int k, int d) {
    __shared__ int hist[4][256];
    __shared__ uint64_t scratch[4][XC_MAX_K_MINE];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int64_t q = static_cast<int64_t>(blockIdx.x) * 4 + wave;
    if (q >= Zq) return;                                 // wave-uniform; no workgroup barrier below
    const float4 zp = zpar[q];
    if (zp.w != kHalfPlain) return;
    const int n = gcnt[q];
    if (n > glist_cap || __builtin_amdgcn_readfirstlane(over[1 + q / kBN]) != 0) {       // given up: nothing reaches it any more
        if (lane == 0) {
            over[0] = 1; over[1 + q / kBN] = 1;
            gcnt[q] = 0;
            tau_g[q] = float_to_ordered(INFINITY);
        }
        return;
    }
    float base = zp.y, thr;
    const int left = half_prune(glist + static_cast<size_t>(q) * glist_cap, n, k, half_query_error(zp, stats, d), &base, &thr, hist[wave], scratch[wave]);
    if (lane == 0) { gcnt[q] = left; tau_g[q] = float_to_ordered(thr); zpar[q].y = base; }
}

// The fp32 scores of what is left, 16 rows by one query as in the few-query search, and the best k.  Bound: random rows from HBM or the
// last-level cache, and where the lists are short a query's dependent steps (15 us), so that with many queries a wave each (WQ = 1)
// is better than a workgroup each (WQ = 4).  The search of 65 536 queries, k = 10, 60 000 x 128: 3.85 ms with WQ = 4, 3.43 with 1; 2100,
// k = 50, 131 072 x 256 0.712 and 0.699; 1200, k = 100, 131 072 x 768 0.742 and 0.768.
template <int WQ>
__global__ __launch_bounds__(256)
void half_finish_kernel(const unsigned char* __restrict__ Z, const unsigned char* __restrict__ W, int row_bytes,
                        uint64_t* __restrict__ glist, int32_t* __restrict__ gcnt, uint32_t* __restrict__ tau_g, const float4* __restrict__ zpar,
                        const uint32_t* __restrict__ stats, int32_t* __restrict__ over, int glist_cap, int k,
                        int64_t Zq, int32_t* __restrict__ shortlist, float* __restrict__ scores) {
    extern __shared__ uint4 zops[];                      // [4 / WQ] queries as operands, whole steps of 64 bytes
    __shared__ int hists[4 / WQ][256];
    __shared__ uint64_t srts[4 / WQ][XC_MAX_K_MINE];
    __shared__ int n_sh;
    __shared__ float base_sh;
    const int lane = lane_id();
    const int wave = WQ == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);         // of the query
    const int slot = WQ == 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const int tid = wave * kWave + lane;
    const int64_t q = static_cast<int64_t>(blockIdx.x) * (4 / WQ) + slot;
    if (q >= Zq) return;                                 // (WQ = 1: no workgroup barrier below)
    uint4* zop = zops + slot * ((row_bytes + 63) / 64 * 4);
    int* hist = hists[slot];
    uint64_t* srt = srts[slot];
    auto meet = []() {
        if (WQ > 1) __syncthreads();
        else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    };
    const float4 zp = zpar[q];
    int n = gcnt[q];
    if (stats[1] != 0u || zp.w == kHalfBad || (zp.w == kHalfPlain && n > glist_cap)) {       // uniform (nothing writes these here)
        if (tid == 0) { over[0] = 1; over[1 + q / kBN] = 1; }
        return;
    }
    if (zp.w == kHalfZero) {                             // all scores are zero: the first k labels
        for (int i = tid; i < k; i += WQ * kWave) {
            shortlist[q * k + i] = i;
            if (scores) scores[q * k + i] = 0.0f;
        }
        if (tid == 0) tau_g[q] = float_to_ordered(0.0f);
        return;
    }
    uint64_t* list = glist + static_cast<size_t>(q) * glist_cap;
    for (int c0 = wave * 4; c0 * 16 < row_bytes; c0 += 4 * WQ) {         // the query's operands: a step of 64 bytes per wave
        const int c = c0 + (lane >> 4);
        uint4 v = make_uint4(0, 0, 0, 0);
        if (c * 16 < row_bytes) v = *reinterpret_cast<const uint4*>(Z + q * row_bytes + c * 16);
        v = FewMma<float>::operand(v);
        if ((lane & 15) == 0) zop[c] = v;
    }
    float base = zp.y;
    if (wave == 0) {
        // The other queries' workgroups set the tile's word meanwhile: what one wave reads holds for all of them (two waves that read
        // for themselves could part here, one gone and one at the barrier with an n that nobody wrote).
        float thr;
        n = __builtin_amdgcn_readfirstlane(over[1 + q / kBN]) != 0
                ? 0 : half_prune(list, n, k, half_query_error(zp, stats, row_bytes / 4), &base, &thr, hist, srt);
        if (WQ > 1 && lane == 0) { n_sh = n; base_sh = base; }
    }
    meet();
    if (WQ > 1) { n = n_sh; base = base_sh; }
    base = base / zp.z;                                  // (a power of two)
    if (n < k) {                                         // uniform
        if (tid == 0) { over[0] = 1; over[1 + q / kBN] = 1; }
        return;
    }
    const int r = lane & 15, g = lane >> 4;
    for (int b = wave; b * 16 < n; b += 2 * WQ) {             // two blocks of 16 rows side by side
        int32_t id[2];
        const unsigned char* wrow[2];
        f32x4 acc[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int e = 16 * (b + WQ * u) + r;
            id[u] = key_id(list[e < n ? e : n - 1]);
            wrow[u] = W + static_cast<int64_t>(id[u]) * row_bytes;
        }
        score_rows<float, 2, 4>(wrow, zop, row_bytes, g, acc);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float v = (r & 2) ? ((r & 1) ? acc[u][3] : acc[u][2]) : ((r & 1) ? acc[u][1] : acc[u][0]);
            const int32_t lab = __shfl(id[u], 4 * g + (r & 3), kWave);
            const int e = 16 * (b + WQ * u) + 4 * g + r;
            if (r < 4 && e < n) list[e] = make_key(v + 0.0f, lab);
        }
    }
    meet();
    if (wave != 0) return;
    float t;
    auto at = [list](int idx) { return list[idx]; };
    if (n > k) {
        t = n <= kSelectRegs / 2 * kWave ? wave_select_k<kSelectRegs / 2>(list, at, n, k, hist)
            : n <= kSelectRegs * kWave   ? wave_select_k<kSelectRegs>(list, at, n, k, hist)
                                         : wave_select_stream(list, n, k, hist);
    } else {
        uint64_t worst = 0;
        for (int i = lane; i < n; i += kWave) { const uint64_t key = list[i]; worst = key > worst ? key : worst; }
        t = key_score(wave_max_u64(worst));
    }
    if (!(t >= base)) {                                  // (from thresholds: a label below them may belong to the answer)
        if (lane == 0) { over[0] = 1; over[1 + q / kBN] = 1; }
        return;
    }
    if (lane == 0) tau_g[q] = float_to_ordered(t);
    wave_write_winners(list, k, k, srt, shortlist + q * k, scores != nullptr ? scores + q * k : nullptr);
}

}  // namespace xc
