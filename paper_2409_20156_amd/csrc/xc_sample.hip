// Negative sampling: the stale hard negatives of each query plus uniform draws
// from the remaining labels, with the log-proposal of every slot (Alg. 1,
// hard+random step; Sec. 3.1 Idea 2; p = 1/(L-k_h) under Eq. 2; warm-up phase
// of Alg. 1 when no shortlist is given).  Integer arithmetic only, so the ids
// are a function of (seed, query, draw, shortlist row) and of no launch shape.
#include <cmath>
#include <type_traits>

#include "xc_common.h"

namespace xc {

constexpr int kSampleThreads = 256;
constexpr uint64_t kQueryMul = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kDrawMul = 0xD1B54A32D192ED03ull;

__device__ __forceinline__ uint64_t fmix64(uint64_t x) {
    x ^= x >> 30; x *= 0xBF58476D1CE4E5B9ull;
    x ^= x >> 27; x *= 0x94D049BB133111EBull;
    x ^= x >> 31;
    return x;
}

// One workgroup per query.  The distinct in-range ids of the shortlist row, in ascending order h_0 < h_1 < ..., are
// stored as a_m = h_m - m, which is non-decreasing.  Draw r in [0, M) then maps to the r-th label of the complement:
// r + #{m : a_m <= r}.
// Rows of up to kRankRow ids find their order by counting the smaller ids, every wave a part of the row, four ids at a
// time and the same for all lanes; equal ids get equal counts, which is how repeats are found.  (Sorting took a barrier for each of
// the 28 steps of 128 ids, and one wave, the same in every workgroup, did all of it on its SIMD.)  The number of draws and the
// size of the complement are the same for every row without repeats, so their log comes from the host; a row with some
// forms its own.  Bound: the vector ALU, whose 64-bit products the mixer needs, and the launch.  2048 rows of 100 + 1024
// ids: 17.4 -> 11.5 us per call, of which the caller takes 8.6.  Rows with repeats number the distinct ids by the bits of their
// counts (counted a second time, id by id: 32 768 rows of 216 with repeats + 1 draw 302 us, now 174).
constexpr int kRankRow = 256;
constexpr int kDraws = 4;                // draws a thread makes side by side

__global__ __launch_bounds__(kSampleThreads)
void sample_kernel(const int32_t* __restrict__ shortlist, int k_h, int k_r, int64_t L,
                   uint64_t seed, int n2, float lq_distinct /* log(draws / (L - distinct)) of a row without repeats */,
                   int32_t* __restrict__ neg, float* __restrict__ logq) {
    __shared__ __align__(16) int32_t hs[XC_MAX_K_SAMPLE];
    __shared__ int32_t adj[XC_MAX_K_SAMPLE];
    __shared__ int n_unique;
    __shared__ int wave_cnt[kSampleThreads / kWave];
    __shared__ uint32_t head_bits[kRankRow / 32];
    const int64_t i = blockIdx.x;
    const int n = k_h + k_r;
    int32_t* out = neg + i * n;
    float* lq = logq + i * n;
    int u = 0, n_draw = n, first = 0;
    // (here, so that it is formed while the row is on its way)
    uint64_t state = fmix64(seed ^ (kQueryMul * static_cast<uint64_t>(i + 1))) + kDrawMul * static_cast<uint64_t>(threadIdx.x + 1);

    if (shortlist != nullptr) {
        const int32_t* row = shortlist + i * k_h;
        for (int m = threadIdx.x; m < n2; m += blockDim.x) {
            int32_t v = 0x7fffffff;
            if (m < k_h) {
                const int32_t id = row[m];
                out[m] = id;
                lq[m] = 0.0f;
                if (id >= 0 && id < L) v = id;
            }
            hs[m] = v;
            if (n2 <= kRankRow) adj[m] = 0;
        }
        if (threadIdx.x == 0) n_unique = 0;
        __syncthreads();
        if (n2 <= kRankRow) {
            // thread t counts, for id t mod n2, the smaller ids in a part of the row: all four waves have work (each
            // runs on a SIMD of its own, and all workgroups of a compute unit put the same wave on the same SIMD)
            const int m = threadIdx.x & (n2 - 1);
            int parts = kSampleThreads / n2;
            parts = parts < n2 / 4 ? parts : n2 / 4;
            const int part = threadIdx.x / n2, len = n2 / parts;
            const int32_t v = hs[m];
            if (part < parts) {
                int c = 0;
                for (int e = part * len; e < (part + 1) * len; e += 4) {
                    const int4 h = *reinterpret_cast<const int4*>(&hs[e]);
                    c += (h.x < v ? 1 : 0) + (h.y < v ? 1 : 0) + (h.z < v ? 1 : 0) + (h.w < v ? 1 : 0);
                }
                atomicAdd(&adj[m], c);
            }
            __syncthreads();
            // equal ids have equal counts: one of them stands for all
            int rank = adj[m];
            const bool valid = threadIdx.x < n2 && v != 0x7fffffff;
            __syncthreads();
            if (valid) adj[rank] = m;
            __syncthreads();
            const bool head = valid && adj[rank] == m;
            const uint64_t bal = __ballot(head);
            if (lane_id() == 0) wave_cnt[threadIdx.x >> 6] = __popcll(bal);
            __syncthreads();
#pragma unroll
            for (int w = 0; w < kSampleThreads / kWave; ++w) u += wave_cnt[w];
            if (u < k_h) {                                   // uniform: repeats or padding, count the distinct ones only
                if (threadIdx.x < kRankRow / 32) head_bits[threadIdx.x] = 0;
                __syncthreads();
                if (head) atomicOr(&head_bits[rank >> 5], 1u << (rank & 31));
                __syncthreads();
                if (head) {                                  // (waves without one pass by)
                    int below = __popc(head_bits[rank >> 5] & ((1u << (rank & 31)) - 1u));
                    for (int w = 0; w < (rank >> 5); ++w) below += __popc(head_bits[w]);
                    rank = below;
                }
            }
            if (head) adj[rank] = v - rank;
        } else {
        for (int size = 2; size <= n2; size <<= 1) {
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int t = threadIdx.x; t < n2 / 2; t += blockDim.x) {
                    const int lo = 2 * t - (t & (stride - 1));
                    const int hi = lo + stride;
                    const bool up = (lo & size) == 0;
                    const int32_t a = hs[lo], b = hs[hi];
                    if ((a > b) == up) { hs[lo] = b; hs[hi] = a; }
                }
                __syncthreads();
            }
        }
        // distinct valid ids, in order: position = number of distinct ids before m
        for (int m0 = 0; m0 < n2; m0 += blockDim.x) {
            const int m = m0 + threadIdx.x;
            bool head = false;
            int32_t v = 0;
            if (m < n2) {
                v = hs[m];
                head = v != 0x7fffffff && (m == 0 || hs[m - 1] != v);
            }
            // block-wide exclusive count of heads below m within this chunk
            const uint64_t bal = __ballot(head);
            const int w = threadIdx.x >> 6;
            if (lane_id() == 0) wave_cnt[w] = __popcll(bal);
            __syncthreads();
            int before = n_unique;
            for (int ww = 0; ww < w; ++ww) before += wave_cnt[ww];
            const int p = before + __popcll(bal & lanemask_lt());
            int chunk_total = 0;
            for (int ww = 0; ww < kSampleThreads / kWave; ++ww) chunk_total += wave_cnt[ww];
            __syncthreads();
            if (head) adj[p] = v - p;
            if (threadIdx.x == 0) n_unique += chunk_total;
            __syncthreads();
        }
        u = n_unique;
        }
        n_draw = k_r;
        first = k_h;
    }

    // the list ends in entries no draw reaches, so the search below needs no bounds
    if (shortlist != nullptr) {
        for (int m = u + static_cast<int>(threadIdx.x); m < n2; m += kSampleThreads) adj[m] = 0x7fffffff;
        __syncthreads();
    }
    if (static_cast<int>(threadIdx.x & ~(kWave - 1u)) >= n_draw) return;     // a wave without draws (no barrier below)
    const uint64_t M = static_cast<uint64_t>(L) - static_cast<uint64_t>(u);
    // log of the expected number of copies of a label among the draws
    const float lq_rand = u == (shortlist != nullptr ? k_h : 0)
                              ? lq_distinct
                              : static_cast<float>(log(static_cast<double>(n_draw) / static_cast<double>(M)));
    const uint32_t M32 = static_cast<uint32_t>(M);           // (L < 2^31)
    constexpr uint64_t kStride = kDrawMul * kSampleThreads;
    // N draws of a thread, j0 the first; the last ones of the row possibly past its end
    auto draw = [&](auto nc, int j0) {
        constexpr int N = decltype(nc)::value;
        uint32_t r[N];
        int pos[N];
#pragma unroll
        for (int d = 0; d < N; ++d) {
            const uint64_t w = fmix64(state);
            state += kStride;
            // floor(w M / 2^64) by halves of w
            const uint64_t low = (static_cast<uint64_t>(static_cast<uint32_t>(w)) * M32) >> 32;
            r[d] = static_cast<uint32_t>(((w >> 32) * M32 + low) >> 32);
            pos[d] = 0;
        }
        // count of a_m <= r over the non-decreasing a (n2 entries, a power of two)
        if (u > 0) {
            for (int s = n2 >> 1; s > 0; s >>= 1)
#pragma unroll
                for (int d = 0; d < N; ++d) pos[d] += static_cast<uint32_t>(adj[pos[d] + s - 1]) <= r[d] ? s : 0;
#pragma unroll
            for (int d = 0; d < N; ++d) pos[d] += static_cast<uint32_t>(adj[pos[d]]) <= r[d] ? 1 : 0;
        }
#pragma unroll
        for (int d = 0; d < N; ++d) {
            const int j = j0 + d * kSampleThreads;
            if (j < n_draw) {
                out[first + j] = static_cast<int32_t>(r[d] + static_cast<uint32_t>(pos[d]));
                lq[first + j] = lq_rand;
            }
        }
    };
    if (n_draw > (kDraws - 1) * kSampleThreads) {
        for (int j0 = threadIdx.x; j0 < n_draw; j0 += kDraws * kSampleThreads) draw(std::integral_constant<int, kDraws>{}, j0);
    } else {                                                 // (fewer: three of four would be made for nothing)
        for (int j0 = threadIdx.x; (j0 & ~(kWave - 1)) < n_draw; j0 += kSampleThreads) draw(std::integral_constant<int, 1>{}, j0);
    }
}

// ---------------------------------------------------------------------------
// Sampling from the mixture proposal itself (Sec. 3.1, Idea 2): k_h draws from the importance
// part, label of shortlist slot m with probability w_m / T, and k_r uniform draws from [0, L).
// ---------------------------------------------------------------------------

// Integer image of 2^32 * sigmoid(score), fixed point throughout so that the draw is a function
// of the score's bits: t = floor(clamp(score) * 2^16); y = |t| log2(e) in Q16; 2^-y in Q30 from
// a degree-5 polynomial (coefficients ln(2)^k / k! * 2^30) and a shift; sigmoid(-|x|) in Q32 by
// one integer division; mirrored for positive scores.  NaN -> 0, otherwise at least 1.
__device__ __forceinline__ uint64_t sigmoid_weight(float score) {
    if (score != score) return 0ull;
    const float x = fminf(fmaxf(score, -30.0f), 30.0f);
    const int64_t t = static_cast<int64_t>(floor(static_cast<double>(x) * 65536.0));   // exact
    const uint64_t a = static_cast<uint64_t>(t < 0 ? -t : t);
    const uint64_t y = (a * 94548ull) >> 16;
    const uint64_t ip = y >> 16, f = y & 0xffffull;
    uint64_t m = 1ull << 30;
    uint64_t shift = ip;
    if (f != 0) {
        const uint64_t u = 65536ull - f;            // 2^(-f/65536) = 2^(u/65536) / 2
        uint64_t r = 1431680ull;
        r = 10327387ull + ((r * u) >> 16);
        r = 59597083ull + ((r * u) >> 16);
        r = 257941248ull + ((r * u) >> 16);
        r = 744261118ull + ((r * u) >> 16);
        m = (1ull << 30) + ((r * u) >> 16);
        shift = ip + 1;
    }
    const uint64_t e = shift < 62 ? (m >> shift) : 0ull;
    const uint64_t sn = (e << 32) / ((1ull << 30) + e);
    const uint64_t w = t >= 0 ? (1ull << 32) - sn : sn;
    return w ? w : 1ull;
}

// One workgroup per query.  LDS holds, per shortlist slot, the id, the weight, the running sum of
// the weights in slot order (for the draw) and the slots sorted by id (for the total weight of a
// label, which may sit in several slots).
__global__ __launch_bounds__(kSampleThreads)
void sample_mixture_kernel(const int32_t* __restrict__ shortlist, const float* __restrict__ scores, int M,
                           int k_h, int k_r, int64_t L, uint64_t seed, int n2,
                           int32_t* __restrict__ neg, float* __restrict__ logq) {
    __shared__ int32_t ids[XC_MAX_K_SAMPLE];
    __shared__ uint64_t wts[XC_MAX_K_SAMPLE];
    __shared__ uint64_t cum[2][XC_MAX_K_SAMPLE];
    __shared__ uint64_t byid[XC_MAX_K_SAMPLE];
    const int64_t i = blockIdx.x;
    const int n = k_h + k_r;
    const int32_t* row = shortlist + i * M;
    const float* srow = scores + i * M;
    for (int m = threadIdx.x; m < n2; m += blockDim.x) {
        int32_t id = -1;
        uint64_t w = 0;
        if (m < M) {
            id = row[m];
            if (id >= 0 && id < L) w = sigmoid_weight(srow[m]);
        }
        ids[m] = id;
        wts[m] = w;
        cum[0][m] = w;
        byid[m] = w ? ((static_cast<uint64_t>(static_cast<uint32_t>(id)) << 32) | static_cast<uint32_t>(m)) : ~0ull;
    }
    __syncthreads();
    // inclusive running sums (doubling steps between two buffers)
    int cur = 0;
    for (int off = 1; off < n2; off <<= 1) {
        for (int m = threadIdx.x; m < n2; m += blockDim.x)
            cum[cur ^ 1][m] = cum[cur][m] + (m >= off ? cum[cur][m - off] : 0ull);
        cur ^= 1;
        __syncthreads();
    }
    const uint64_t* run = cum[cur];
    // slots ordered by label id (slots without weight last)
    for (int size = 2; size <= n2; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = threadIdx.x; t < n2 / 2; t += blockDim.x) {
                const int lo = 2 * t - (t & (stride - 1));
                const int hi = lo + stride;
                const bool up = (lo & size) == 0;
                const uint64_t a = byid[lo], b = byid[hi];
                if ((a > b) == up) { byid[lo] = b; byid[hi] = a; }
            }
            __syncthreads();
        }
    }
    const uint64_t T = run[n2 - 1];
    const int n_imp = T > 0 ? k_h : 0;
    const uint64_t qstate = fmix64(seed ^ (kQueryMul * static_cast<uint64_t>(i + 1)));
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        const uint64_t u = fmix64(qstate + kDrawMul * static_cast<uint64_t>(j + 1));
        int64_t lab;
        if (j < n_imp) {
            const uint64_t r = __umul64hi(u, T);
            int lo = 0, hi = n2 - 1;                 // first slot whose running sum exceeds r
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (run[mid] > r) hi = mid; else lo = mid + 1;
            }
            lab = ids[lo];
        } else {
            lab = static_cast<int64_t>(__umul64hi(u, static_cast<uint64_t>(L)));
        }
        double c;
        if (T > 0) {
            // total weight of the slots that hold this label
            const uint64_t key = static_cast<uint64_t>(lab) << 32;
            int lo = 0, hi = n2;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (byid[mid] < key) lo = mid + 1; else hi = mid;
            }
            uint64_t wl = 0;
            for (int p = lo; p < n2 && (byid[p] >> 32) == static_cast<uint64_t>(lab); ++p)
                wl += wts[static_cast<uint32_t>(byid[p])];
            c = static_cast<double>(k_h) * static_cast<double>(wl) / static_cast<double>(T) +
                static_cast<double>(k_r) / static_cast<double>(L);
        } else {
            c = static_cast<double>(n) / static_cast<double>(L);
        }
        neg[i * n + j] = static_cast<int32_t>(lab);
        logq[i * n + j] = static_cast<float>(log(c));
    }
}

// ---------------------------------------------------------------------------
// Hard negatives sampled WITHOUT replacement from a wider stale shortlist, slot m with probability
// proportional to w_m = sigmoid_weight(stale score) (Sec. 3.1, Observation 2, inside the mixture of
// Idea 2).  k = min(k_h, slots with weight) slots are chosen:
//   (1) slots with k' w_m >= T' (k' still to choose, T' the remaining weight) are certain; all such
//       slots are taken at once and the test is repeated with the reduced k', T';
//   (2) the rest by systematic sampling: the k' points U + j T' on the axis of the running sums of the
//       remaining weights (slot order) scaled by k', U = floor(u T' / 2^64) from the query's draw 0;
//       a slot is taken when a point falls into its interval (at most one does: k' w_m < T').
// pi_m = 1 resp. k' w_m / T' exactly.  Slots k.. of the output are uniform draws from [0, L), and
// logq = log(sum of pi over the slots holding the label + (k_h + k_r - k) / L).
// One workgroup per query; integer arithmetic for everything that decides an id.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kSampleThreads)
void sample_pps_kernel(const int32_t* __restrict__ shortlist, const float* __restrict__ scores, int M,
                       int k_h, int k_r, int64_t L, uint64_t seed, int n2,
                       int32_t* __restrict__ neg, float* __restrict__ logq) {
    __shared__ int32_t ids[XC_MAX_K_SAMPLE];
    __shared__ uint64_t wts[XC_MAX_K_SAMPLE];
    __shared__ uint64_t cum[2][XC_MAX_K_SAMPLE];
    __shared__ uint64_t byid[XC_MAX_K_SAMPLE];
    __shared__ double pi[XC_MAX_K_SAMPLE];
    __shared__ int32_t sel[XC_MAX_K_SAMPLE];          // taken slots in slot order
    __shared__ unsigned char state[XC_MAX_K_SAMPLE];  // 0 no weight, 1 remaining, 2 certain, 3 taken by a point
    __shared__ uint64_t red_w[kSampleThreads / kWave];
    __shared__ int red_c[kSampleThreads / kWave];
    const int64_t i = blockIdx.x;
    const int n = k_h + k_r;
    const int tid = threadIdx.x;
    const int32_t* row = shortlist + i * M;
    const float* srow = scores + i * M;
    // sum of (count, weight) over the workgroup, fixed order; every thread gets both
    auto block_sum2 = [&](int c, uint64_t w, int& c_out, uint64_t& w_out) {
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) { c += __shfl_xor(c, off, kWave); w += __shfl_xor(w, off, kWave); }
        if ((tid & (kWave - 1)) == 0) { red_c[tid / kWave] = c; red_w[tid / kWave] = w; }
        __syncthreads();
        c_out = 0; w_out = 0;
        for (int q = 0; q < kSampleThreads / kWave; ++q) { c_out += red_c[q]; w_out += red_w[q]; }
        __syncthreads();
    };
    int c_loc = 0;
    uint64_t w_loc = 0;
    for (int m = tid; m < n2; m += blockDim.x) {
        int32_t id = -1;
        uint64_t w = 0;
        if (m < M) {
            id = row[m];
            if (id >= 0 && id < L) w = sigmoid_weight(srow[m]);
        }
        ids[m] = id;
        wts[m] = w;
        state[m] = w ? 1 : 0;
        byid[m] = w ? ((static_cast<uint64_t>(static_cast<uint32_t>(id)) << 32) | static_cast<uint32_t>(m)) : ~0ull;
        c_loc += w ? 1 : 0;
        w_loc += w;
    }
    int nv;
    uint64_t TT;
    block_sum2(c_loc, w_loc, nv, TT);
    const int k = k_h < nv ? k_h : nv;
    int kk = k;
    // (1) certain slots, round by round (each round takes at least one slot or ends the loop)
    while (kk > 0) {
        c_loc = 0; w_loc = 0;
        for (int m = tid; m < n2; m += blockDim.x) {
            if (state[m] == 1 && static_cast<uint64_t>(kk) * wts[m] >= TT) { state[m] = 2; ++c_loc; w_loc += wts[m]; }
        }
        int c_all;
        uint64_t w_all;
        block_sum2(c_loc, w_loc, c_all, w_all);
        if (c_all == 0) break;
        kk -= c_all;
        TT -= w_all;
    }
    // running sums of the remaining weights in slot order (doubling steps between two buffers)
    for (int m = tid; m < n2; m += blockDim.x) cum[0][m] = state[m] == 1 ? wts[m] : 0ull;
    __syncthreads();
    int cur = 0;
    for (int off = 1; off < n2; off <<= 1) {
        for (int m = tid; m < n2; m += blockDim.x)
            cum[cur ^ 1][m] = cum[cur][m] + (m >= off ? cum[cur][m - off] : 0ull);
        cur ^= 1;
        __syncthreads();
    }
    // (2) systematic sampling of the remaining slots, and pi of every slot
    const uint64_t qstate = fmix64(seed ^ (kQueryMul * static_cast<uint64_t>(i + 1)));
    {
        const uint64_t U = (kk > 0 && TT > 0) ? __umul64hi(fmix64(qstate + kDrawMul), TT) : 0ull;
        auto points_below = [&](uint64_t x) -> uint64_t {        // number of j in [0, kk) with U + j TT < x
            if (x <= U) return 0ull;
            const uint64_t c = (x - U - 1) / TT + 1;
            return c < static_cast<uint64_t>(kk) ? c : static_cast<uint64_t>(kk);
        };
        for (int m = tid; m < n2; m += blockDim.x) {
            double p = state[m] == 2 ? 1.0 : 0.0;
            if (state[m] == 1) {
                p = static_cast<double>(static_cast<uint64_t>(kk) * wts[m]) / static_cast<double>(TT);
                if (kk > 0) {
                    const uint64_t hi = static_cast<uint64_t>(kk) * cum[cur][m];
                    const uint64_t lo = hi - static_cast<uint64_t>(kk) * wts[m];
                    if (points_below(hi) - points_below(lo) == 1ull) state[m] = 3;
                }
            }
            pi[m] = p;
        }
    }
    __syncthreads();
    // taken slots in slot order: positions from a running count (reuses the scan buffers)
    for (int m = tid; m < n2; m += blockDim.x) cum[0][m] = state[m] >= 2 ? 1ull : 0ull;
    __syncthreads();
    cur = 0;
    for (int off = 1; off < n2; off <<= 1) {
        for (int m = tid; m < n2; m += blockDim.x)
            cum[cur ^ 1][m] = cum[cur][m] + (m >= off ? cum[cur][m - off] : 0ull);
        cur ^= 1;
        __syncthreads();
    }
    for (int m = tid; m < n2; m += blockDim.x)
        if (state[m] >= 2) sel[cum[cur][m] - 1] = m;
    // slots ordered by label id (slots without weight last), for the expected count of a label
    for (int size = 2; size <= n2; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = tid; t < n2 / 2; t += blockDim.x) {
                const int lo = 2 * t - (t & (stride - 1));
                const int hi = lo + stride;
                const bool up = (lo & size) == 0;
                const uint64_t a = byid[lo], b = byid[hi];
                if ((a > b) == up) { byid[lo] = b; byid[hi] = a; }
            }
            __syncthreads();
        }
    }
    const double unif = static_cast<double>(n - k) / static_cast<double>(L);
    for (int j = tid; j < n; j += blockDim.x) {
        int64_t lab;
        if (j < k) lab = ids[sel[j]];
        else lab = static_cast<int64_t>(__umul64hi(fmix64(qstate + kDrawMul * static_cast<uint64_t>(j + 1)), static_cast<uint64_t>(L)));
        double c = 0.0;
        if (k > 0) {
            const uint64_t key = static_cast<uint64_t>(lab) << 32;
            int lo = 0, hi = n2;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (byid[mid] < key) lo = mid + 1; else hi = mid;
            }
            for (int p = lo; p < n2 && (byid[p] >> 32) == static_cast<uint64_t>(lab); ++p)
                c += pi[static_cast<uint32_t>(byid[p])];                   // in slot order
        }
        neg[i * n + j] = static_cast<int32_t>(lab);
        logq[i * n + j] = static_cast<float>(log(c + unif));
    }
}

}  // namespace xc

extern "C" int xc_sample_negatives(const int32_t* shortlist, int64_t B, int k_h, int k_r, int64_t L,
                                   uint64_t seed, int32_t* neg, float* logq, void* stream) {
    using namespace xc;
    if (B < 1 || k_h < 0 || k_r < 0 || k_h + k_r < 1 || k_h > XC_MAX_K_SAMPLE) return XC_ESHAPE;
    if (L < 1 || L > 0x7fffffffLL || k_h >= L) return XC_ESHAPE;
    if (B > 0x7fffffffLL) return XC_ESHAPE;
    if (!neg || !logq) return XC_EINVAL;
    int n2 = 4;                              // (the row is read four ids at a time)
    while (n2 < k_h) n2 <<= 1;
    if (k_h == 0) shortlist = nullptr;      // nothing to exclude: same as the warm-up draw
    const double draws = shortlist != nullptr ? k_r : k_h + k_r;
    const float lq_distinct = static_cast<float>(log(draws / static_cast<double>(shortlist != nullptr ? L - k_h : L)));
    hipStream_t st = static_cast<hipStream_t>(stream);
    XC_LAUNCH(K_SAMPLE, st, (sample_kernel<<<dim3(static_cast<unsigned>(B)), kSampleThreads, 0, st>>>(
        shortlist, k_h, k_r, L, seed, n2, lq_distinct, neg, logq)));
    XC_HIP_CHECK(hipGetLastError());
    return XC_OK;
}

extern "C" int xc_sample_negatives_mixture(const int32_t* shortlist, const float* scores, int64_t B, int M,
                                           int k_h, int k_r, int64_t L, uint64_t seed, int32_t* neg,
                                           float* logq, void* stream) {
    using namespace xc;
    if (B < 1 || B > 0x7fffffffLL || M < 1 || M > XC_MAX_K_SAMPLE) return XC_ESHAPE;
    if (k_h < 0 || k_r < 0 || k_h + k_r < 1 || L < 1 || L > 0x7fffffffLL) return XC_ESHAPE;
    if (!shortlist || !scores || !neg || !logq) return XC_EINVAL;
    int n2 = 2;
    while (n2 < M) n2 <<= 1;
    hipStream_t st = static_cast<hipStream_t>(stream);
    XC_LAUNCH(K_SAMPLE, st, (sample_mixture_kernel<<<dim3(static_cast<unsigned>(B)), kSampleThreads, 0, st>>>(
        shortlist, scores, M, k_h, k_r, L, seed, n2, neg, logq)));
    XC_HIP_CHECK(hipGetLastError());
    return XC_OK;
}

extern "C" int xc_sample_negatives_pps(const int32_t* shortlist, const float* scores, int64_t B, int M,
                                       int k_h, int k_r, int64_t L, uint64_t seed, int32_t* neg,
                                       float* logq, void* stream) {
    using namespace xc;
    if (B < 1 || B > 0x7fffffffLL || M < 1 || M > XC_MAX_K_SAMPLE) return XC_ESHAPE;
    if (k_h < 0 || k_h > XC_MAX_K_SAMPLE || k_r < 0 || k_h + k_r < 1 || L < 1 || L > 0x7fffffffLL) return XC_ESHAPE;
    if (!shortlist || !scores || !neg || !logq) return XC_EINVAL;
    int n2 = 2;
    while (n2 < M) n2 <<= 1;
    hipStream_t st = static_cast<hipStream_t>(stream);
    XC_LAUNCH(K_SAMPLE, st, (sample_pps_kernel<<<dim3(static_cast<unsigned>(B)), kSampleThreads, 0, st>>>(
        shortlist, scores, M, k_h, k_r, L, seed, n2, neg, logq)));
    XC_HIP_CHECK(hipGetLastError());
    return XC_OK;
}
