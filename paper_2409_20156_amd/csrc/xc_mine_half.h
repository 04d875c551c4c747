// The search of many fp32 queries, with fp16 copies in front: the same exact top-k as xc_mine.hip (which includes this file).
// Bound of the fp32 kernels: the matrix pipe, whose fp32 products run at a sixteenth of the 16-bit rate.  z and w rounded to 11
// bits give a score that is off by at most half_error() |z| |w| (a thousandth of it), so the sweep over all labels runs on fp16
// copies with thresholds lowered by that, and the few labels left get their score from the fp32 rows, in the order of sums of the
// other kernels.  Queries are brought to one norm, so that the error e(l) is
// that of the largest row in the label's tile of 256, whatever the query:
//   half_queries_kernel, half_rows_kernel   the copies, padded to whole tiles and stages, and the largest |w| of each tile
//   mine_tile_kernel / mine_rows_kernel     on them, as for bf16 rows.  A label passes if its 16-bit score reaches B(q) - e(l), where
//                                           B is a score that k labels are known to reach: no label of the answer is lost
//   half_select_kernel                      B = the k-th best of (16-bit score - e), and the list cut to what can still matter
//   half_finish_kernel                      the fp32 scores of the list, the best k of them
// A tile with a row that fp16 cannot hold has an infinite error: its labels always pass.  (One error for all labels let one row of
// norm 10 among a million of norm 1 double the time of a search, and one element of 2000 ran every list over.)
// What this does not settle - a list that ran over, queries out of fp16's range, a warm search whose thresholds were too
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
    size_t off_rows, off_z, off_zpar, off_err, off_range, off_skip, bytes;      // within its part of the workspace
};

// The copies: queries to a norm of kHalfNorm, W by a scale for all.  A score's error then depends on the label alone: tile_err[l / kBM] at most.
// The last workgroup finds the scale.  zpar: (scale of the query, kind)
constexpr float kHalfNorm = 16384.0f;
__global__ __launch_bounds__(256)
void half_queries_kernel(const unsigned char* __restrict__ Z, int64_t Zq, int64_t nq, int row_bytes, int pitch,
                         unsigned char* __restrict__ out, float2* __restrict__ zpar,
                         float* __restrict__ tile_err, int64_t nLT, int32_t* __restrict__ over, int32_t* __restrict__ skip, const unsigned char* __restrict__ W, int64_t L, float* __restrict__ scale, uint32_t* __restrict__ zeros /* [64] */) {
    const int lane = lane_id();
    if (blockIdx.x == gridDim.x - 1) {
        __shared__ uint32_t most[kHalfSample];
        const int i = threadIdx.x >> 4;                  // sixteen lanes to a row
        const unsigned char* wr = W + half_sample_row(i, L) * row_bytes;
        uint32_t m = 0;
        for (int c = threadIdx.x & 15; c * 16 < row_bytes; c += 16) {
            const uint32_t b = half_sample_bits(*reinterpret_cast<const uint4*>(wr + c * 16));
            m = b > m ? b : m;
        }
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) { const uint32_t o = __shfl_xor(m, off, kWave); m = o > m ? o : m; }
        if ((threadIdx.x & 15) == 0) most[i] = m;
        __syncthreads();
        const float s = half_scale(most[lane & (kHalfSample - 1)]);
        if (threadIdx.x == 0) scale[0] = s;
        if (threadIdx.x < 64) zeros[threadIdx.x] = 0u;
        return;
    }
    const int64_t q = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < nLT; i += static_cast<int64_t>(gridDim.x - 1) * 256) tile_err[i] = 0.0f;
    if (lane == 0 && (q & (kBN - 1)) == 0 && q < nq) { over[1 + q / kBN] = 0; skip[q / kBN] = 0; if (q == 0) over[0] = 0; }
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
    const float up = m == 0.0f || bad ? 0.0f : kHalfNorm / sqrtf(s2);
    for (int i = lane; i < pitch / 2; i += kWave)
        reinterpret_cast<_Float16*>(out + q * pitch)[i] = static_cast<_Float16>(i < d && !bad ? zr[i] * up : 0.0f);
    if (lane == 0) zpar[q] = make_float2(up, q >= Zq || m == 0.0f ? kHalfZero : bad ? kHalfBad : kHalfPlain);
}

// Rows [0, n_lab) of the chunk, LG lanes (a power of two) to a row; rows up to n_rows are zeros.  Bound: HBM (6 bytes per element).
__global__ __launch_bounds__(256)
void half_rows_kernel(const unsigned char* __restrict__ W, int64_t n_lab, int64_t n_rows, int row_bytes, int pitch, int LG, int unit,
                      unsigned char* __restrict__ out, float* __restrict__ tile_err /* of the chunk's first tile */, const float* __restrict__ w_scale) {
    const int wave_rows = unit / 4;                      // one after the other, of one tile
    const float scale = w_scale[0];                      // (a power of two)
    const uint32_t far = __float_as_uint(65504.0f / scale);
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int per = kWave / LG, l = lane & (LG - 1);
    constexpr float kUp = kHalfNorm * 1.002f;            // (both norms are rounded)
    const float he = half_error(row_bytes / 4) * kUp * scale, hs = half_error_small(row_bytes / 4) * kUp;
    for (int64_t u0 = static_cast<int64_t>(blockIdx.x) * unit; u0 < n_rows; u0 += static_cast<int64_t>(gridDim.x) * unit) {
        const int64_t w0 = u0 + wave * wave_rows;
        float most = 0.0f;                               // the largest |w|^2
        uint32_t top_bits = 0;                           // of the largest element
        for (int i0 = 0; i0 < wave_rows; i0 += per) {
            const int64_t r = w0 + i0 + lane / LG;
            float s2 = 0.0f;
            for (int c = l; c * 16 < pitch; c += LG) {   // 8 elements: two chunks in, one out
                uint4 a = make_uint4(0, 0, 0, 0), b = make_uint4(0, 0, 0, 0);
                if (r < n_lab && c * 32 < row_bytes) a = load16<true>(W + r * row_bytes + c * 32);
                if (r < n_lab && c * 32 + 16 < row_bytes) b = load16<true>(W + r * row_bytes + c * 32 + 16);
                const uint32_t u[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
                uint32_t m = 0;
                f16x8 h;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float f = __uint_as_float(u[i]);
                    s2 = fmaf(f, f, s2);
                    const uint32_t bits = u[i] & 0x7fffffffu;
                    m = bits > m ? bits : m;
                    h[i] = static_cast<_Float16>(f * scale);
                }
                if (m >= far) {                          // beyond fp16, or no number: such a row's score is never looked at
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if ((u[i] & 0x7fffffffu) >= far) h[i] = static_cast<_Float16>(0.0f);
                }
                top_bits = m > top_bits ? m : top_bits;
                *reinterpret_cast<f16x8*>(out + r * pitch + c * 16) = h;
            }
            for (int off = LG >> 1; off > 0; off >>= 1) s2 += __shfl_xor(s2, off, kWave);
            most = fmaxf(most, s2);                      // (of a row that is no number: see far)
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) most = fmaxf(most, __shfl_xor(most, off, kWave));
        const bool all_zero = __ballot(top_bits != 0u) == 0ull, wide = __ballot(top_bits >= far) != 0ull;
        if (lane == 0) {
            const float e = wide ? INFINITY : all_zero ? 0.0f : sqrtf(most) * he + hs;
            if (e > 0.0f) atomicMax(reinterpret_cast<uint32_t*>(tile_err) + w0 / kBM, __float_as_uint(e));
        }
    }
}

// The range of the first n tiles' errors that are not zero, see half_error_of_all.  By one workgroup of 256.  (Additions of every workgroup of
// half_rows_kernel to two words took longer than its rows: 200 000 x 128 62 us with them, 35 without.)
__device__ void half_range(const float* __restrict__ tile_err, int64_t n, uint32_t* __restrict__ range) {
    __shared__ float sh[4][2];
    float top = 0.0f, low = INFINITY;
#pragma unroll 8
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const float e = tile_err[i];
        top = fmaxf(top, e);
        low = e > 0.0f ? fminf(low, e) : low;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { top = fmaxf(top, __shfl_xor(top, off, kWave)); low = fminf(low, __shfl_xor(low, off, kWave)); }
    if (lane_id() == 0) { sh[threadIdx.x >> 6][0] = top; sh[threadIdx.x >> 6][1] = low; }
    __syncthreads();
    if (threadIdx.x == 0) {
        range[0] = __float_as_uint(fmaxf(fmaxf(sh[0][0], sh[1][0]), fmaxf(sh[2][0], sh[3][0])));
        range[1] = __float_as_uint(fminf(fminf(sh[0][1], sh[1][1]), fminf(sh[2][1], sh[3][1])));
    }
}
__global__ __launch_bounds__(256)
void half_range_kernel(const float* __restrict__ tile_err, int64_t n, uint32_t* __restrict__ range) { half_range(tile_err, n, range); }

// Thresholds of the first sweep.  from: 0 none yet, 1 the k-th best 16-bit scores of the dense phase, less their error, 2 those of the search
// before, lowered by rel |tau| (fp32 scores).  The last workgroup has the errors' range to find.
__global__ __launch_bounds__(256)
void half_start_kernel(int from, float rel, uint32_t* __restrict__ tau_g, int32_t* __restrict__ gcnt, const float2* __restrict__ zpar,
                       int32_t* __restrict__ over, int32_t* __restrict__ skip, int64_t n, int64_t Zq,
                       const float* __restrict__ tile_err, int64_t n_tiles, uint32_t* __restrict__ range, const float* __restrict__ scale) {
    if (blockIdx.x == gridDim.x - 1) { half_range(tile_err, n_tiles, range); return; }
    const int64_t q = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (q >= n) return;
    gcnt[q] = 0;
    const float2 zp = zpar[q];
    if (q < Zq && zp.y == kHalfBad) { over[0] = 1; over[1 + q / kBN] = 1; skip[q / kBN] = 1; }       // the tile is not swept at all
    if (q >= Zq || zp.y != kHalfPlain) tau_g[q] = float_to_ordered(INFINITY);
    else if (from == 0) tau_g[q] = kTauInit;
    else if (from == 2) { const float t = ordered_to_float(tau_g[q]); tau_g[q] = float_to_ordered((t - rel * fabsf(t)) * zp.x * scale[0]); }
}

// A query's list cut to the labels that can still be among the best k, `base` raised to what k of them are known to reach.  By one wave.
__device__ int half_prune(uint64_t* list, int n, int k, const float* __restrict__ tile_err, float all, float* base, int* hist, uint64_t* scratch) {
    const int lane = lane_id();
    if (n >= k) {
        float t;
        auto pick = [=](auto least) {                        // the k-th best
            if (n == k || n > kSelectRegs * kWave) {
                const uint64_t bound = n == k ? kKeySentinel : wave_bound_stream(least, n, k, hist);
                uint64_t worst = 0;
                for (int i = lane; i < n; i += kWave) { const uint64_t key = least(i); if (key <= bound && key > worst) worst = key; }
                return key_score(wave_max_u64(worst));
            }
            return n <= kSelectRegs / 2 * kWave ? wave_select_k<kSelectRegs / 2>(scratch, least, n, k, hist) : wave_select_k<kSelectRegs>(scratch, least, n, k, hist);
        };
        if (all >= 0.0f) t = pick([list](int idx) { return list[idx]; });
        else t = pick([list, tile_err](int idx) { const uint64_t key = list[idx]; return make_key(key_score(key) - tile_err[key_id(key) / kBM], key_id(key)); });
        *base = fmaxf(*base, all >= 0.0f ? t - all : t);
    }
    const float thr = *base - all;
    int out = 0;
    for (int i0 = 0; i0 < n; i0 += kWave) {              // in place: a chunk is read before anything of it is overwritten
        const uint64_t key = i0 + lane < n ? list[i0 + lane] : kKeySentinel;
        bool keep = i0 + lane < n;
        if (all >= 0.0f) keep = keep && key_score(key) >= thr;
        else if (keep) keep = key_score(key) + tile_err[key_id(key) / kBM] >= *base;
        const uint64_t bal = __ballot(keep);
        if (keep) list[out + __popcll(bal & lanemask_lt())] = key;
        out += __popcll(bal);
    }
    return out;
}

__global__ __launch_bounds__(256)
void half_select_kernel(uint64_t* __restrict__ glist, int32_t* __restrict__ gcnt, uint32_t* __restrict__ tau_g, const float2* __restrict__ zpar,
                        const float* __restrict__ tile_err, const uint32_t* __restrict__ range, int32_t* __restrict__ over, int32_t* __restrict__ skip, int64_t Zq, int glist_cap, int k) {
    __shared__ int hist[4][256];
    __shared__ uint64_t scratch[4][XC_MAX_K_MINE];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int64_t q = static_cast<int64_t>(blockIdx.x) * 4 + wave;
    if (q >= Zq) return;                                 // wave-uniform; no workgroup barrier below
    const float2 zp = zpar[q];
    if (zp.y != kHalfPlain) return;
    const int n = gcnt[q];
    if (n > glist_cap || __builtin_amdgcn_readfirstlane(over[1 + q / kBN]) != 0) {       // given up: nothing reaches it any more
        if (lane == 0) {
            over[0] = 1; over[1 + q / kBN] = 1;
            skip[q / kBN] = 1;
            gcnt[q] = 0;
            tau_g[q] = float_to_ordered(INFINITY);
        }
        return;
    }
    float base = ordered_to_float(tau_g[q]);
    const int left = half_prune(glist + static_cast<size_t>(q) * glist_cap, n, k, tile_err, half_error_of_all(range), &base, hist[wave], scratch[wave]);
    if (lane == 0) { gcnt[q] = left; tau_g[q] = float_to_ordered(base); }
}

// The fp32 scores of what is left, 16 rows by one query as in the few-query search, and the best k.  Bound: random rows from HBM or the
// last-level cache, and where the lists are short a query's dependent steps (15 us), so that with many queries a wave each (WQ = 1)
// is better than a workgroup each (WQ = 4).  The search of 65 536 queries, k = 10, 60 000 x 128: 3.85 ms with WQ = 4, 3.43 with 1; 2100,
// k = 50, 131 072 x 256 0.712 and 0.699; 1200, k = 100, 131 072 x 768 0.742 and 0.768.
template <int WQ>
__global__ __launch_bounds__(256)
void half_finish_kernel(const unsigned char* __restrict__ Z, const unsigned char* __restrict__ W, int row_bytes,
                        uint64_t* __restrict__ glist, int32_t* __restrict__ gcnt, uint32_t* __restrict__ tau_g, const float2* __restrict__ zpar,
                        const float* __restrict__ tile_err, const uint32_t* __restrict__ range, const float* __restrict__ scale,
                        int32_t* __restrict__ over, int glist_cap, int k, int64_t Zq, int32_t* __restrict__ shortlist, float* __restrict__ scores) {
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
    const float2 zp = zpar[q];
    int n = gcnt[q];
    if (zp.y == kHalfBad || (zp.y == kHalfZero && range[0] == __float_as_uint(INFINITY)) || (zp.y == kHalfPlain && n > glist_cap)) {      // uniform (nothing writes these here)
        if (tid == 0) { over[0] = 1; over[1 + q / kBN] = 1; }
        return;
    }
    if (zp.y == kHalfZero) {                             // all scores are zero: the first k labels
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
    float base = ordered_to_float(tau_g[q]);             // (wave 0's, which also writes tau_g below)
    if (wave == 0) {
        // The other queries' workgroups set the tile's word meanwhile: what one wave reads holds for all of them (two waves that read
        // for themselves could part here, one gone and one at the barrier with an n that nobody wrote).
        n = __builtin_amdgcn_readfirstlane(over[1 + q / kBN]) != 0
                ? 0 : half_prune(list, n, k, tile_err, half_error_of_all(range), &base, hist, srt);
        if (WQ > 1 && lane == 0) { n_sh = n; base_sh = base; }
    }
    meet();
    if (WQ > 1) { n = n_sh; base = base_sh; }
    base = base / zp.x / scale[0];
    base -= 1e-6f * fabsf(base);                         // (rounded; the errors have a hundredth to spare)
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
            // (a score that is no number comes last.  The label stays: another block's lanes past the list's end may read it here)
            if (r < 4 && e < n) list[e] = v == v ? make_key(v + 0.0f, lab) : (0xffffffffull << 32) | static_cast<uint32_t>(lab);
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
