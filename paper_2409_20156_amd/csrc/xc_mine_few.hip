// The search for few queries: the same exact top-k as xc_mine.hip (score of Sec. 2.1) where the work is
// reading W once, not the products.  Inference over a handful of queries, small pools.
//
//   few_line_kernel    streams W once (few_max_kernel where rows are short or LDS is, see few_lines; few_half_kernel
//       more than 16 fp32 queries).  A wave multiplies 32 labels with all queries of the workgroup, whose rows
//       lie in LDS as MFMA operands, and keeps of every group of 16 << gshift labels the largest score per
//       query: the only thing written, 1 / (16 << gshift) of the score matrix.
//   few_finish_kernel  one workgroup per query: the k-th largest group maximum tau (a bound from 256 part maxima, then
//       by counting).  At least k
//       labels score tau or more, so every label of the answer does, and it lies in a group whose maximum is
//       above tau or, for scores equal to tau, in one of the first groups (in label order) whose maximum is tau:
//       of equal scores the smaller ids win, and each of these groups holds one.  So k groups in all hold the
//       answer.  Their scores are formed again, with the sums in the same order (hence the same
//       bits), what is below tau is dropped, the rest sorted.
// Bound: HBM, one read of W.  131 072 x 768 bf16, 32 queries, k = 5: 54 us in all (first kernel 41 us, 4.9 TB/s; a plain
// copy reaches 5.1), where the general kernel took 378; 4 M x 256 bf16, 32 queries: 0.47 ms against 0.55 by half lines.  In
// fp32 with more than 16 queries the matrix pipe, which is why the maxima then come from 16-bit products (few_half_kernel): 1000
// queries x 50 021 x 300, 158 us (76 and 83 the two kernels) against 364 with fp32 products (318 and 105; these alone need 195) and 782
// by the general kernel.
// No thresholds to find in phases, no lists that could overflow, two launches.  The general kernel pads the
// pool to 256 queries and sweeps the labels in four or more serial phases, of which the first have fewer work
// items than the chip has compute units.
#include <cmath>

#include "xc_mine.h"

namespace xc {

constexpr int kFewThreads = 512;
constexpr size_t kFewLds = 144u << 10;   // LDS for the query block at most
constexpr size_t kLineLds = 160u << 10;  // the same with a stage per wave beside it
constexpr int kFewWaves = kFewThreads / kWave;
constexpr int kFewRing = 8;              // 64-byte steps in flight per wave (two rows of 16 B per lane each: 16 KiB)
constexpr int kFewTile = 32;             // labels a wave multiplies at a time
// The second kernel: 1024 threads per query while there are few queries, 256 (and a quarter of the key list, so that
// eight queries are in flight per compute unit) from 512 queries on: 1000 queries x 50 021 x 300 fp32, k = 32: 118 -> 102 us.
constexpr int64_t kSmallFinishQueries = 512;
template <int NT> struct Finish {
    static constexpr int kWaves = NT / kWave;
    static constexpr int kKeys = 4 * NT;                // candidate keys of a query in LDS
};
constexpr int kRankSort = 512;           // up to so many candidates are sorted by counting
constexpr int kMaxSplit = 8;             // workgroups per query of the second kernel at most
constexpr int kPartKeys = Finish<1024>::kKeys / kMaxSplit;      // candidates one of them hands over at most
static_assert(kPartKeys >= XC_MAX_K_MINE, "a workgroup hands over at least its best k");

struct FewArgs {
    const unsigned char* Z;
    const unsigned char* W;
    int64_t Zq, L, row_bytes;
    int ks, n_qb, gshift, k;
    int64_t n_groups;
    uint32_t* gmax;              // [Zq][n_groups] ordered image of the largest score, 0 = no score that is a number
    uint32_t* tau_g;
    int32_t* flag;
    int n_flag;
    int32_t* shortlist;
    float* scores;
    int n_split;                 // workgroups that share a query in the second kernel
    uint64_t* part;              // [Zq][n_split][kPartKeys] their candidates
    int32_t* part_n;             // [Zq][n_split]
    int32_t* done;               // [Zq] how many of them are through (cleared by the first kernel)
    float* gerr;                 // 16-bit maxima: [n_groups] times |z| is the error of the group's maximum
    int32_t* redo_any;           // 16-bit maxima: 1 if any query has to be searched again in fp32 (cleared by the first kernel),
    int32_t* redo;               // [Zq] 1 if q has
    int again;                   // 1: this is that search: only queries with redo[q]
};

// ordered image of a score; 0 (below every number) for NaN.  -0 counts as +0, as in the result.
__device__ __forceinline__ uint32_t score_image(float v) { return v == v ? float_to_ordered(v + 0.0f) : 0u; }

// Whether one of the queries [q0, q0 + n) has to be searched again; workgroup 0 of such a launch goes on in any case (it clears the counters).
__device__ __forceinline__ bool few_again(const FewArgs& a, int64_t q0, int n) {
    if (a.redo_any[0] == 0) return false;
    bool any = blockIdx.x == 0;
    for (int i = 0; i < n && q0 + i < a.Zq; ++i) any = any || a.redo[q0 + i] != 0;
    return any;
}

// MFMA operands: lane (r, g) = (lane & 15, lane >> 4) loads 16 bytes of row r: chunk 4 s + g of the row in step s, for
// labels and queries alike.
template <typename T, int NB, bool KTAIL>
__global__ __launch_bounds__(kFewThreads)
void few_max_kernel(const FewArgs a) {
    extern __shared__ __align__(16) unsigned char zlds[];       // [ks][NB] operands of 1 KiB
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int KS = a.ks;
    // workgroups of one XCD (id % 8) that differ in the query block only are neighbours: they read the same rows of W
    // at about the same time, and all but the first find them in that XCD's L2
    const int id = blockIdx.x;
    const int qb = (id / 8) % a.n_qb;
    const int wg = (id % 8) + 8 * (id / (8 * a.n_qb));
    const int n_wg = gridDim.x / a.n_qb;                        // (a multiple of 8, see the launch)
    const int64_t q0 = static_cast<int64_t>(qb) * NB * 16;
    if (a.again && !few_again(a, q0, NB * 16)) return;          // uniform

    // a unit is the tiles whose maxima one wave combines: a tile of two groups (gshift 0), or 2^(gshift-1) tiles of one
    const int comb = a.gshift > 0 ? 1 << (a.gshift - 1) : 1;
    const int64_t n_tiles = (a.L + kFewTile - 1) / kFewTile;
    const int64_t n_units = (n_tiles + comb - 1) / comb;
    const int64_t u_step = static_cast<int64_t>(n_wg) * kFewWaves;
    int64_t unit = static_cast<int64_t>(wg) * kFewWaves + wave;

    // ---- the load stream: ring of kFewRing steps, running ahead across tiles and units; begun before the queries are laid out (a
    // call with few labels has one tile per wave, and would wait for memory twice: 32 x 131 072 x 768 65.2 -> 62.5 us in all)
    int64_t ld_unit = unit < n_units ? unit : n_units - 1;
    int ld_t = 0;
    int ld_off = 0;                                             // bytes into the rows
    const unsigned char *p0, *p1;
    auto set_rows = [&]() {
        const int64_t l = (ld_unit * comb + ld_t) * kFewTile + r;
        const int64_t l0 = l < a.L ? l : a.L - 1, l1 = l + 16 < a.L ? l + 16 : a.L - 1;      // rows past the end: dropped later
        p0 = a.W + l0 * a.row_bytes;
        p1 = a.W + l1 * a.row_bytes;
    };
    set_rows();
    uint4 ra[kFewRing][2];
    auto load_step = [&](int j) {
        int64_t off = ld_off + g * 16;
        if (KTAIL) off = off < a.row_bytes ? off : 0;           // (zeroed where it is used)
        ra[j][0] = *reinterpret_cast<const uint4*>(p0 + off);
        ra[j][1] = *reinterpret_cast<const uint4*>(p1 + off);
        ld_off += 64;
        if (ld_off == KS * 64) {                                // uniform
            ld_off = 0;
            ++ld_t;
            if (ld_t == comb || ld_unit * comb + ld_t >= n_tiles) { ld_t = 0; ld_unit += u_step; }
            if (ld_unit < n_units) set_rows();                  // else: the last tile again, never used
        }
    };
#pragma unroll
    for (int j = 0; j < kFewRing; ++j) load_step(j);

    // ---- the queries, four chunks of a thread at a time
    for (int e0 = tid; e0 < KS * NB * 64; e0 += 4 * kFewThreads) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * kFewThreads, l = e & 63, blk = e >> 6;
            const int64_t q = q0 + (blk % NB) * 16 + (l & 15);
            const int64_t off = static_cast<int64_t>(blk / NB) * 64 + (l >> 4) * 16;
            v[u] = make_uint4(0, 0, 0, 0);
            if (q < a.Zq && off < a.row_bytes) v[u] = *reinterpret_cast<const uint4*>(a.Z + q * a.row_bytes + off);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * kFewThreads;
            const uint4 o = FewMma<T>::operand(v[u]);           // (a wave takes whole blocks)
            if (e < KS * NB * 64) *reinterpret_cast<uint4*>(zlds + static_cast<size_t>(e) * 16) = o;
        }
    }
    if (id == 0)
        for (int64_t i = tid; i < a.Zq; i += kFewThreads) a.done[i] = 0;
    __syncthreads();
    if (unit >= n_units) return;                                // (no barrier below)

    const bool tail_chunk = static_cast<int64_t>(KS - 1) * 64 + g * 16 >= a.row_bytes;       // this lane's chunk of the last step
    f32x4 acc[2][NB];
    // maxima are taken as floats: fmaxf passes over NaN, so a group is NaN only if all its scores are
    const float nan = __builtin_nanf("");
    float run[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        run[n] = nan;
        acc[0][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        acc[1][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    int t = 0, s = 0;
    for (;;) {
#pragma unroll
        for (int j = 0; j < kFewRing; ++j) {
            uint4 a0 = ra[j][0], a1 = ra[j][1];
            if (KTAIL && s == KS - 1 && tail_chunk) { a0 = make_uint4(0, 0, 0, 0); a1 = make_uint4(0, 0, 0, 0); }
            a0 = FewMma<T>::operand(a0);
            a1 = FewMma<T>::operand(a1);
            const unsigned char* zb = zlds + static_cast<size_t>(s) * NB * 1024 + lane * 16;
            uint4 b[NB];
#pragma unroll
            for (int n = 0; n < NB; ++n) b[n] = *reinterpret_cast<const uint4*>(zb + n * 1024);
            // (an accumulator's own instructions lie 2 NB apart: one that follows the other waits for it)
#pragma unroll
            for (int m = 0; m < FewMma<T>::kSteps; ++m)
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    acc[0][n] = FewMma<T>::mma(m, a0, b[n], acc[0][n]);
                    acc[1][n] = FewMma<T>::mma(m, a1, b[n], acc[1][n]);
                }
            // (fp32 exchanges operands in the ring's registers: a load scheduled before their last use would need others, which
            // the compiler then moves at the end of the loop, awaiting the whole ring)
            if (FewMma<T>::kSteps > 1) __builtin_amdgcn_sched_barrier(0);
            load_step(j);
            if (++s == KS) {                                    // uniform: a tile is complete
                s = 0;
                const int64_t tile = unit * comb + t;
                const int64_t lab = tile * kFewTile + 4 * g;    // accumulator i of block b: label lab + 16 b + i, query r
                const bool full = (tile + 1) * kFewTile <= a.L;
                const bool unit_done = t + 1 == comb || tile + 1 >= n_tiles;
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    float m[2];
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        if (!full)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (lab + 16 * b + i >= a.L) acc[b][n][i] = nan;
                        m[b] = fmaxf(fmaxf(acc[b][n][0], acc[b][n][1]), fmaxf(acc[b][n][2], acc[b][n][3]));
                    }
                    acc[0][n] = f32x4{0.f, 0.f, 0.f, 0.f};
                    acc[1][n] = f32x4{0.f, 0.f, 0.f, 0.f};
                    const int64_t q = q0 + n * 16 + r;
                    if (a.gshift == 0) {
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            m[b] = fmaxf(m[b], __shfl_xor(m[b], 16, kWave));
                            m[b] = fmaxf(m[b], __shfl_xor(m[b], 32, kWave));
                        }
                        // lanes 0..15 store the first group's maxima, lanes 16..31 the second's
                        const int64_t grp = 2 * tile + g;
                        if (g < 2 && q < a.Zq && grp < a.n_groups) a.gmax[q * a.n_groups + grp] = score_image(g == 0 ? m[0] : m[1]);
                    } else {
                        run[n] = fmaxf(run[n], fmaxf(m[0], m[1]));
                        if (unit_done) {
                            run[n] = fmaxf(run[n], __shfl_xor(run[n], 16, kWave));
                            run[n] = fmaxf(run[n], __shfl_xor(run[n], 32, kWave));
                            if (g == 0 && q < a.Zq) a.gmax[q * a.n_groups + unit] = score_image(run[n]);
                            run[n] = nan;
                        }
                    }
                }
                ++t;
                if (unit_done) { t = 0; unit += u_step; if (unit >= n_units) return; }
            }
        }
    }
}

// The same for rows of 128 bytes and more, with W read a line at a time.  What few_max_kernel loads with one instruction, 64 bytes of
// each of 16 rows, is half a line each, and memory delivered 4.2 TB/s that way whatever was under way; here an instruction brings
// 128 bytes of 8 rows, and the wave exchanges them for operands through 4 KiB of LDS of its own (chunk c of row r at position
// c ^ (r >> 1) & 7, so that 16 lanes reading one chunk of 16 rows meet no bank twice).  Half lines and whole ones, us in all: 32 queries x
// 4 M x 200 bf16 515 and 484, 30 x 300 000 x 504 99 and 87, 500 x 60 000 x 768 126 and 94, 1000 x 50 000 x 256 130 and 105; read past the caches (see
// line_way) 32 x 1.3 M x 768 484 and 400 (5.0 TB/s), 8 x 1.3 M x 768 442 and 360 (5.5), 16 x 1 M x 256 fp32 260 and 217.
constexpr int kFewStage = kFewTile * 128;   // bytes of a wave's stage

template <typename T, int NB, bool KTAIL, bool STREAM>
__global__ __launch_bounds__(kFewThreads, 4)
void few_line_kernel(const FewArgs a) {
    extern __shared__ __align__(16) unsigned char zlds[];       // [ks][NB] operands of 1 KiB, then a stage per wave
    constexpr int kStages = NB == 1 ? 4 : NB == 2 ? 3 : 2;      // in a wave's registers, 4 KiB each (so that four waves fit a SIMD)
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int KS = (a.ks + 1) & ~1;                             // steps of 64 bytes, in pairs
    // workgroups of one XCD (id % 8) that differ in the query block only are neighbours: they read the same rows of W
    // at about the same time, and all but the first find them in that XCD's L2
    const int id = blockIdx.x;
    const int qb = (id / 8) % a.n_qb;
    const int wg = (id % 8) + 8 * (id / (8 * a.n_qb));
    const int n_wg = gridDim.x / a.n_qb;                        // (a multiple of 8, see the launch)
    const int64_t q0 = static_cast<int64_t>(qb) * NB * 16;

    // a unit is the tiles whose maxima one wave combines: a tile of two groups (gshift 0), or 2^(gshift-1) tiles of one
    const int comb = a.gshift > 0 ? 1 << (a.gshift - 1) : 1;
    const int64_t n_tiles = (a.L + kFewTile - 1) / kFewTile;
    const int64_t n_units = (n_tiles + comb - 1) / comb;
    const int64_t u_step = static_cast<int64_t>(n_wg) * kFewWaves;
    int64_t unit = static_cast<int64_t>(wg) * kFewWaves + wave;

    // ---- the load stream: ring of stages of 128 bytes of 32 rows, running ahead across tiles and units; begun before the queries are
    // laid out (a call with few labels has one tile per wave, and would wait for memory twice)
    const int srow = lane >> 3, schunk = lane & 7;              // of the 8 rows of a load instruction
    int64_t ld_unit = unit < n_units ? unit : n_units - 1;
    int ld_t = 0;
    int ld_off = schunk * 16;                                   // bytes into the rows
    const int row_bytes = static_cast<int>(a.row_bytes);
    const unsigned char* p[4];
    auto set_rows = [&]() {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t l = (ld_unit * comb + ld_t) * kFewTile + 8 * t + srow;
            p[t] = a.W + (l < a.L ? l : a.L - 1) * a.row_bytes; // rows past the end: dropped later
        }
    };
    set_rows();
    uint4 ra[kStages][4];
    auto load_stage = [&](int j) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            ra[j][t] = load16<STREAM>(p[t] + (KTAIL && ld_off >= row_bytes ? 0 : ld_off));           // (zeroed where it is used)
        }
        ld_off += 128;
        if (ld_off - schunk * 16 == KS * 64) {                  // uniform
            ld_off = schunk * 16;
            ++ld_t;
            if (ld_t == comb || ld_unit * comb + ld_t >= n_tiles) { ld_t = 0; ld_unit += u_step; }
            if (ld_unit < n_units) set_rows();                  // else: the last tile again, never used
        }
    };
#pragma unroll
    for (int j = 0; j < kStages; ++j) load_stage(j);

    // ---- the queries, four chunks of a thread at a time
    for (int e0 = tid; e0 < KS * NB * 64; e0 += 4 * kFewThreads) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * kFewThreads, l = e & 63, blk = e >> 6;
            const int64_t q = q0 + (blk % NB) * 16 + (l & 15);
            const int64_t off = static_cast<int64_t>(blk / NB) * 64 + (l >> 4) * 16;
            v[u] = make_uint4(0, 0, 0, 0);
            if (q < a.Zq && off < a.row_bytes) v[u] = *reinterpret_cast<const uint4*>(a.Z + q * a.row_bytes + off);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * kFewThreads;
            const uint4 o = FewMma<T>::operand(v[u]);           // (a wave takes whole blocks)
            if (e < KS * NB * 64) *reinterpret_cast<uint4*>(zlds + static_cast<size_t>(e) * 16) = o;
        }
    }
    if (id == 0)
        for (int64_t i = tid; i < a.Zq; i += kFewThreads) a.done[i] = 0;
    __syncthreads();
    if (unit >= n_units) return;                                // (no barrier below)

    f32x4 acc[2][NB];
    // maxima are taken as floats: fmaxf passes over NaN, so a group is NaN only if all its scores are
    const float nan = __builtin_nanf("");
    float run[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        run[n] = nan;
        acc[0][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        acc[1][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    unsigned char* stage = zlds + static_cast<size_t>(KS) * NB * 1024 + wave * kFewStage;
    const bool tail = KS * 64 - 128 + schunk * 16 >= row_bytes;
    // (the swizzle term of the 8 rows of load t is 4 (t & 1) + (lane >> 4), that of an operand's rows (lane >> 1) & 7)
    const uint32_t put[2] = {static_cast<uint32_t>(srow * 128 + ((schunk ^ (lane >> 4)) * 16)),
                             static_cast<uint32_t>(srow * 128 + ((schunk ^ ((lane >> 4) + 4)) * 16))};
    const uint32_t get = static_cast<uint32_t>(r * 128 + ((g ^ ((lane >> 1) & 7)) * 16));
    int t = 0, s = 0;
    for (;;) {
#pragma unroll
        for (int j = 0; j < kStages; ++j) {
            if (KTAIL && s + 2 == KS && tail)                   // this lane's chunks lie past the rows' end
#pragma unroll
                for (int u = 0; u < 4; ++u) ra[j][u] = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 4; ++u) *reinterpret_cast<uint4*>(stage + put[u & 1] + u * 1024) = ra[j][u];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");      // (a wave's LDS operations are done in order)
            load_stage(j);
            uint4 w[2][2], b[2][NB];                            // [half of the stage][block of 16 rows]
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int m = 0; m < 2; ++m) w[h][m] = *reinterpret_cast<const uint4*>(stage + (get ^ (h * 64)) + m * 2048);
#pragma unroll
                for (int n = 0; n < NB; ++n) b[h][n] = *reinterpret_cast<const uint4*>(zlds + (static_cast<size_t>(s + h) * NB + n) * 1024 + lane * 16);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint4 a0 = FewMma<T>::operand(w[h][0]), a1 = FewMma<T>::operand(w[h][1]);
                // (an accumulator's own instructions lie 2 NB apart: one that follows the other waits for it)
#pragma unroll
                for (int m = 0; m < FewMma<T>::kSteps; ++m)
#pragma unroll
                    for (int n = 0; n < NB; ++n) {
                        acc[0][n] = FewMma<T>::mma(m, a0, b[h][n], acc[0][n]);
                        acc[1][n] = FewMma<T>::mma(m, a1, b[h][n], acc[1][n]);
                    }
            }
            s += 2;
            if (s == KS) {                                      // uniform: a tile is complete
                s = 0;
                const int64_t tile = unit * comb + t;
                const int64_t lab = tile * kFewTile + 4 * g;    // accumulator i of block b: label lab + 16 b + i, query r
                const bool full = (tile + 1) * kFewTile <= a.L;
                const bool unit_done = t + 1 == comb || tile + 1 >= n_tiles;
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    float m[2];
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        if (!full)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (lab + 16 * b + i >= a.L) acc[b][n][i] = nan;
                        m[b] = fmaxf(fmaxf(acc[b][n][0], acc[b][n][1]), fmaxf(acc[b][n][2], acc[b][n][3]));
                    }
                    acc[0][n] = f32x4{0.f, 0.f, 0.f, 0.f};
                    acc[1][n] = f32x4{0.f, 0.f, 0.f, 0.f};
                    const int64_t q = q0 + n * 16 + r;
                    if (a.gshift == 0) {
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            m[b] = fmaxf(m[b], __shfl_xor(m[b], 16, kWave));
                            m[b] = fmaxf(m[b], __shfl_xor(m[b], 32, kWave));
                        }
                        // lanes 0..15 store the first group's maxima, lanes 16..31 the second's
                        const int64_t grp = 2 * tile + g;
                        if (g < 2 && q < a.Zq && grp < a.n_groups) a.gmax[q * a.n_groups + grp] = score_image(g == 0 ? m[0] : m[1]);
                    } else {
                        run[n] = fmaxf(run[n], fmaxf(m[0], m[1]));
                        if (unit_done) {
                            run[n] = fmaxf(run[n], __shfl_xor(run[n], 16, kWave));
                            run[n] = fmaxf(run[n], __shfl_xor(run[n], 32, kWave));
                            if (g == 0 && q < a.Zq) a.gmax[q * a.n_groups + unit] = score_image(run[n]);
                            run[n] = nan;
                        }
                    }
                }
                ++t;
                if (unit_done) { t = 0; unit += u_step; if (unit >= n_units) return; }
            }
        }
    }
}

// The same in fp32 for more than 16 queries, where the 16-bit maxima below did not settle them, with the operands of the tile kernels: lane (r, h) = (lane & 31, lane >> 5) holds
// chunks 4 s + h and 4 s + 2 + h of row r.  Nothing is exchanged.  fp32 matrix instructions run on the vector unit, which the
// exchanges of few_max_kernel and every address come out of: 600 queries x 300 000 x 768 4.55 ms with them, 3.93 without;
// 2048 x 130 000 x 64 522 and 445 us; 256 x 1 M x 128 729 and 639; 1000 x 50 021 x 300 380 and 365.  An instruction loads 32 bytes of a row
// instead of 64, which costs where loads bind: 64 queries x 500 000 x 520 368 us and 376; one block of 16 queries, 1.3 M x 256,
// 331 and 373, so that one stays there.
template <int NB, bool KTAIL>
__global__ __launch_bounds__(kFewThreads)
void few_wide_kernel(const FewArgs a) {
    constexpr int NC = NB / 2;                                  // blocks of 32 queries
    extern __shared__ __align__(16) unsigned char zlds[];       // [ks][NC][2] operands of 1 KiB
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int KS = a.ks;
    // workgroups of one XCD (id % 8) that differ in the query block only are neighbours: they read the same rows of W
    // at about the same time, and all but the first find them in that XCD's L2
    const int id = blockIdx.x;
    const int qb = (id / 8) % a.n_qb;
    const int wg = (id % 8) + 8 * (id / (8 * a.n_qb));
    const int n_wg = gridDim.x / a.n_qb;                        // (a multiple of 8, see the launch)
    const int64_t q0 = static_cast<int64_t>(qb) * NB * 16;
    if (a.again && !few_again(a, q0, NB * 16)) return;          // uniform

    for (int e = tid; e < KS * NB * 64; e += kFewThreads) {
        const int l = e & 63, blk = e >> 6;
        const int m = blk & 1, n = (blk >> 1) % NC, s = (blk >> 1) / NC;
        const int64_t q = q0 + n * 32 + (l & 31);
        const int64_t off = static_cast<int64_t>(s) * 64 + m * 32 + (l >> 5) * 16;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (q < a.Zq && off < a.row_bytes) v = *reinterpret_cast<const uint4*>(a.Z + q * a.row_bytes + off);
        *reinterpret_cast<uint4*>(zlds + static_cast<size_t>(e) * 16) = v;
    }
    if (id == 0)
        for (int64_t i = tid; i < a.Zq; i += kFewThreads) a.done[i] = 0;
    __syncthreads();

    // a unit is the tiles whose maxima one wave combines: a tile of two groups (gshift 0), or 2^(gshift-1) tiles of one
    const int comb = a.gshift > 0 ? 1 << (a.gshift - 1) : 1;
    const int64_t n_tiles = (a.L + kFewTile - 1) / kFewTile;
    const int64_t n_units = (n_tiles + comb - 1) / comb;
    const int64_t u_step = static_cast<int64_t>(n_wg) * kFewWaves;
    int64_t unit = static_cast<int64_t>(wg) * kFewWaves + wave;
    if (unit >= n_units) return;                                // (no barrier below)

    // ---- the load stream: ring of kFewRing steps, running ahead across tiles and units
    int64_t ld_unit = unit;
    int ld_t = 0;
    int ld_off = 0;                                             // bytes into the rows
    const unsigned char* p;
    auto set_rows = [&]() {
        const int64_t l = (ld_unit * comb + ld_t) * kFewTile + r;
        p = a.W + (l < a.L ? l : a.L - 1) * a.row_bytes;        // rows past the end: dropped later
    };
    set_rows();
    uint4 ra[kFewRing][2];
    auto load_step = [&](int j) {
        int64_t o0 = ld_off + h * 16, o1 = o0 + 32;
        if (KTAIL) { o0 = o0 < a.row_bytes ? o0 : 0; o1 = o1 < a.row_bytes ? o1 : 0; }      // (zeroed where it is used)
        ra[j][0] = *reinterpret_cast<const uint4*>(p + o0);
        ra[j][1] = *reinterpret_cast<const uint4*>(p + o1);
        ld_off += 64;
        if (ld_off == KS * 64) {                                // uniform
            ld_off = 0;
            ++ld_t;
            if (ld_t == comb || ld_unit * comb + ld_t >= n_tiles) { ld_t = 0; ld_unit += u_step; }
            if (ld_unit < n_units) set_rows();                  // else: the last tile again, never used
        }
    };
#pragma unroll
    for (int j = 0; j < kFewRing; ++j) load_step(j);

    // this lane's chunks of the last step that lie past the row's end
    const bool tail0 = static_cast<int64_t>(KS - 1) * 64 + h * 16 >= a.row_bytes, tail1 = static_cast<int64_t>(KS - 1) * 64 + 32 + h * 16 >= a.row_bytes;
    f32x16 acc[NC];
    const float nan = __builtin_nanf("");
    float run[NC];
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        run[n] = nan;
        acc[n] = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    }
    int t = 0, s = 0;
    for (;;) {
#pragma unroll
        for (int j = 0; j < kFewRing; ++j) {
            uint4 a0 = ra[j][0], a1 = ra[j][1];
            if (KTAIL && s == KS - 1) {                         // uniform
                if (tail0) a0 = make_uint4(0, 0, 0, 0);
                if (tail1) a1 = make_uint4(0, 0, 0, 0);
            }
            const unsigned char* zb = zlds + static_cast<size_t>(s) * NB * 1024 + lane * 16;
#pragma unroll
            for (int n = 0; n < NC; ++n) {
                RowMma<float>::mma(a0, *reinterpret_cast<const uint4*>(zb + (2 * n) * 1024), acc[n]);
                RowMma<float>::mma(a1, *reinterpret_cast<const uint4*>(zb + (2 * n + 1) * 1024), acc[n]);
            }
            load_step(j);
            if (++s == KS) {                                    // uniform: a tile is complete
                s = 0;
                const int64_t tile = unit * comb + t;
                const int64_t lab = tile * kFewTile + 4 * h;    // accumulator i: label lab + 8 (i / 4) + i % 4, query r
                const bool full = (tile + 1) * kFewTile <= a.L;
                const bool unit_done = t + 1 == comb || tile + 1 >= n_tiles;
#pragma unroll
                for (int n = 0; n < NC; ++n) {
                    if (!full)
#pragma unroll
                        for (int i = 0; i < 16; ++i)
                            if (lab + 8 * (i >> 2) + (i & 3) >= a.L) acc[n][i] = nan;
                    float m[2];                                 // labels 0..15 and 16..31 of the tile
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        m[b] = acc[n][8 * b];
#pragma unroll
                        for (int i = 1; i < 8; ++i) m[b] = fmaxf(m[b], acc[n][8 * b + i]);
                    }
                    acc[n] = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    const int64_t q = q0 + n * 32 + r;
                    if (a.gshift == 0) {
                        // the lower lanes store the first group's maxima, the upper ones the second's
                        const float v = fmaxf(h == 0 ? m[0] : m[1], __shfl_xor(h == 0 ? m[1] : m[0], 32, kWave));
                        const int64_t grp = 2 * tile + h;
                        if (q < a.Zq && grp < a.n_groups) a.gmax[q * a.n_groups + grp] = score_image(v);
                    } else {
                        run[n] = fmaxf(run[n], fmaxf(m[0], m[1]));
                        if (unit_done) {
                            run[n] = fmaxf(run[n], __shfl_xor(run[n], 32, kWave));
                            if (h == 0 && q < a.Zq) a.gmax[q * a.n_groups + unit] = score_image(run[n]);
                            run[n] = nan;
                        }
                    }
                }
                ++t;
                if (unit_done) { t = 0; unit += u_step; if (unit >= n_units) return; }
            }
        }
    }
}

// ---- fp32 rows, group maxima from 16-bit products.  fp32 matrix instructions do a sixteenth of what the 16-bit ones do, and
// which groups can hold an answer is known well enough from fp16 copies formed on the way to the matrix pipe: with z and
// w rounded to 11 bits each a score is off by at most half_error() |z| |w|, a thousandth, about a thirtieth of the scores'
// spread at 1024 elements.  The second kernel forms the scores of the k best groups in fp32 as ever, and then of every other group whose
// maximum plus its error reaches the k-th of them: the answer is that of the fp32 search, bit for bit.
// Powers of two keep fp16's range out of it: a query is scaled by its largest element, W by that of a sample (half_scale).  Elements of W
// beyond fp16 become infinite, and so does their group's error: such a group is always looked at.  Where too many groups are
// (equal rows by the thousand, odd numbers), the query is searched again by the fp32 kernels, whose launches return at once otherwise.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
constexpr int kHalfRing = 4;             // steps of 32 elements in flight per wave (two rows of 32 B per lane each: 16 KiB)
// Groups beside the k best that the second kernel looks at.  108 searches of nine shapes on rows of eleven kinds (a common part of up to three times the
// rest, clusters, long tails, few dimensions) needed 16 to 192 of them; rows that lie in hundreds of copies each settle with none, and
// what is read in vain comes on top.  1000 queries x 50 021 x 300, 100 different rows, 512 : 256 groups 1002 : 491 us (fp32 alone 370); with rows
// in 300 copies 724 (396), in 50 copies 213 (431).
constexpr int kMoreGroups = 256;
__device__ __forceinline__ f16x8 to_half8(const uint4& a, const uint4& b, float scale) {
    const float f[8] = {__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z), __uint_as_float(a.w),
                        __uint_as_float(b.x), __uint_as_float(b.y), __uint_as_float(b.z), __uint_as_float(b.w)};
    f16x8 h;
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = static_cast<_Float16>(f[i] * scale);
    return h;
}

// The structure of few_max_kernel: a step is 32 elements, lane (r, g) holds elements 4 g .. 4 g + 3 and 16 + 4 g .. of row r (labels
// and queries alike; the order of the sums does not matter here).  gshift -1: groups of 8 labels, so that the second kernel has
// half the rows to read.
template <int NB, bool KTAIL>
__global__ __launch_bounds__(kFewThreads)
void few_half_kernel(const FewArgs a) {
    extern __shared__ __align__(16) unsigned char zlds[];       // [ks][NB] operands of 1 KiB, then a factor per query, then the sample's rows
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int KS = a.ks;
    float* back = reinterpret_cast<float*>(zlds + static_cast<size_t>(KS) * NB * 1024);      // [NB * 16] from 16-bit scores to scores
    const int id = blockIdx.x;
    const int qb = (id / 8) % a.n_qb;
    const int wg = (id % 8) + 8 * (id / (8 * a.n_qb));
    const int n_wg = gridDim.x / a.n_qb;                        // (a multiple of 8, see the launch)
    const int64_t q0 = static_cast<int64_t>(qb) * NB * 16;

    // a unit is the tiles whose maxima one wave combines: a tile of its groups (gshift <= 0), or 2^(gshift-1) tiles of one
    const int comb = a.gshift > 0 ? 1 << (a.gshift - 1) : 1;
    const int64_t n_tiles = (a.L + kFewTile - 1) / kFewTile;
    const int64_t n_units = (n_tiles + comb - 1) / comb;
    const int64_t u_step = static_cast<int64_t>(n_wg) * kFewWaves;
    int64_t unit = static_cast<int64_t>(wg) * kFewWaves + wave;

    // ---- W's scale, from 32 chunks of each of the sample's rows (the same in every workgroup)
    uint32_t* most = reinterpret_cast<uint32_t*>(back + NB * 16);            // [kHalfSample]
    const uint4 sample = *reinterpret_cast<const uint4*>(a.W + half_sample_row(tid >> 5, a.L) * a.row_bytes + (tid & 31) * (a.row_bytes / 16) / 32 * 16);
    static_assert(kFewThreads == 32 * kHalfSample, "");

    // ---- the load stream, begun before the queries are laid out
    int64_t ld_unit = unit < n_units ? unit : n_units - 1;
    int ld_t = 0;
    int ld_off = 0;                                             // bytes into the rows
    const unsigned char *p0, *p1;
    auto set_rows = [&]() {
        const int64_t l = (ld_unit * comb + ld_t) * kFewTile + r;
        const int64_t l0 = l < a.L ? l : a.L - 1, l1 = l + 16 < a.L ? l + 16 : a.L - 1;      // rows past the end: dropped later
        p0 = a.W + l0 * a.row_bytes;
        p1 = a.W + l1 * a.row_bytes;
    };
    set_rows();
    uint4 ra[kHalfRing][4];
    auto load_step = [&](int j) {
        int64_t o0 = ld_off + g * 16, o1 = o0 + 64;             // (64 bytes of a row together per instruction)
        if (KTAIL) { o0 = o0 < a.row_bytes ? o0 : 0; o1 = o1 < a.row_bytes ? o1 : 0; }      // (zeroed where it is used)
        ra[j][0] = *reinterpret_cast<const uint4*>(p0 + o0);
        ra[j][1] = *reinterpret_cast<const uint4*>(p0 + o1);
        ra[j][2] = *reinterpret_cast<const uint4*>(p1 + o0);
        ra[j][3] = *reinterpret_cast<const uint4*>(p1 + o1);
        ld_off += 128;
        if (ld_off == KS * 128) {                               // uniform
            ld_off = 0;
            ++ld_t;
            if (ld_t == comb || ld_unit * comb + ld_t >= n_tiles) { ld_t = 0; ld_unit += u_step; }
            if (ld_unit < n_units) set_rows();                  // else: the last tile again, never used
        }
    };
#pragma unroll
    for (int j = 0; j < kHalfRing; ++j) load_step(j);

    {
        uint32_t m = half_sample_bits(sample);
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) { const uint32_t o = __shfl_xor(m, off, kWave); m = o > m ? o : m; }
        if ((tid & 31) == 0) most[tid >> 5] = m;
    }
    // ---- the queries, 512 / (16 NB) neighbouring lanes for each: the largest element, then the scaled row
    {
        constexpr int TQ = kFewThreads / (NB * 16);
        const int i = tid / TQ, sub = tid % TQ;
        const int64_t q = q0 + i;
        const int chunks = static_cast<int>(a.row_bytes / 16);
        const unsigned char* zr = a.Z + (q < a.Zq ? q : a.Zq - 1) * a.row_bytes;
        uint32_t m = 0;
#pragma unroll 8
        for (int c = sub; c < chunks; c += TQ) {
            const uint4 v = *reinterpret_cast<const uint4*>(zr + c * 16);
            const uint32_t x = v.x & 0x7fffffffu, y = v.y & 0x7fffffffu, z = v.z & 0x7fffffffu, w = v.w & 0x7fffffffu;
            const uint32_t xy = x > y ? x : y, zw = z > w ? z : w, all = xy > zw ? xy : zw;
            m = all > m ? all : m;
        }
#pragma unroll
        for (int off = TQ / 2; off > 0; off >>= 1) { const uint32_t o = __shfl_xor(m, off, kWave); m = o > m ? o : m; }
        const float mf = __uint_as_float(m);
        const bool ok = m == 0 || (mf >= kHalfLeast && mf <= kHalfMost);        // (else the second kernel has it searched again)
        const int e = m == 0 || !ok ? 0 : 14 - (static_cast<int>(m >> 23) - 127);            // largest element to [2^14, 2^15)
        const float up = ldexpf(1.0f, e);
        if (sub == 0) back[i] = ldexpf(1.0f, -e);
#pragma unroll 8
        for (int c = sub; c < KS * 8; c += TQ) {                // chunk c: elements 4 c .. 4 c + 3
            uint4 v = make_uint4(0, 0, 0, 0);
            if (c < chunks && ok && q < a.Zq) v = *reinterpret_cast<const uint4*>(zr + c * 16);
            typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
            f16x4 h;
            h[0] = static_cast<_Float16>(__uint_as_float(v.x) * up); h[1] = static_cast<_Float16>(__uint_as_float(v.y) * up);
            h[2] = static_cast<_Float16>(__uint_as_float(v.z) * up); h[3] = static_cast<_Float16>(__uint_as_float(v.w) * up);
            *reinterpret_cast<f16x4*>(zlds + (static_cast<size_t>(c >> 3) * NB + (i >> 4)) * 1024 + ((c & 3) * 16 + (i & 15)) * 16 + ((c >> 2) & 1) * 8) = h;
        }
    }
    if (id == 0) {
        for (int64_t i = tid; i < a.Zq; i += kFewThreads) { a.done[i] = 0; a.redo[i] = 0; }
        if (tid == 0) a.redo_any[0] = 0;
    }
    __syncthreads();
    if (unit >= n_units) return;                                // (no barrier below)
    const float scale = half_scale(most[lane & (kHalfSample - 1)]), unscale = 1.0f / scale;        // (powers of two)
    const float he = half_error(static_cast<int>(a.row_bytes / 4)) * 1.001f * unscale;             // (rounded elements are up to 2^-11 smaller)
    const float hs = half_error_small(static_cast<int>(a.row_bytes / 4)) * unscale;
    float bk[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) bk[n] = back[n * 16 + r] * unscale;

    // this lane's chunks of the last step that lie past the row's end
    const bool tail0 = static_cast<int64_t>(KS - 1) * 128 + g * 16 >= a.row_bytes, tail1 = static_cast<int64_t>(KS - 1) * 128 + g * 16 + 64 >= a.row_bytes;
    f32x4 acc[2][NB];
    const float nan = __builtin_nanf("");
    float run[NB], sq[2] = {0.0f, 0.0f}, run_sq = 0.0f;
    uint32_t any = 0;                                           // an element that is not zero
    // the norms of a unit's rows are taken by one of the query blocks
    bool norms = static_cast<int>(unit % a.n_qb) == qb;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        run[n] = nan;
        acc[0][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        acc[1][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    int t = 0, s = 0;
    for (;;) {
#pragma unroll
        for (int j = 0; j < kHalfRing; ++j) {
            // the queries' operands, all on their way before the rows are converted (one at a time, as the compiler orders them by
            // itself, every pair of products waited for its own: 81 us, with this 76, at 1000 queries x 50 021 x 300)
            const unsigned char* zb = zlds + static_cast<size_t>(s) * NB * 1024 + lane * 16;
            f16x8 b[NB];
#pragma unroll
            for (int n = 0; n < NB; ++n) b[n] = *reinterpret_cast<const f16x8*>(zb + n * 1024);
            __builtin_amdgcn_sched_barrier(0);
            if (KTAIL && s == KS - 1) {                         // uniform
                if (tail0) { ra[j][0] = make_uint4(0, 0, 0, 0); ra[j][2] = make_uint4(0, 0, 0, 0); }
                if (tail1) { ra[j][1] = make_uint4(0, 0, 0, 0); ra[j][3] = make_uint4(0, 0, 0, 0); }
            }
            const f16x8 a0 = to_half8(ra[j][0], ra[j][1], scale), a1 = to_half8(ra[j][2], ra[j][3], scale);
            if (norms) {                                        // uniform
#pragma unroll
                for (int u = 0; u < 4; ++u) any |= (ra[j][u].x | ra[j][u].y | ra[j][u].z | ra[j][u].w) << 1;
#pragma unroll
                for (int i = 0; i < 8; i += 2) {
                    sq[0] = __builtin_amdgcn_fdot2(f16x2{a0[i], a0[i + 1]}, f16x2{a0[i], a0[i + 1]}, sq[0], false);
                    sq[1] = __builtin_amdgcn_fdot2(f16x2{a1[i], a1[i + 1]}, f16x2{a1[i], a1[i + 1]}, sq[1], false);
                }
            }
            load_step(j);
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                acc[0][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, b[n], acc[0][n], 0, 0, 0);
                acc[1][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, b[n], acc[1][n], 0, 0, 0);
            }
            if (++s == KS) {                                    // uniform: a tile is complete
                s = 0;
                const int64_t tile = unit * comb + t;
                const int64_t lab = tile * kFewTile + 4 * g;    // accumulator i of block b: label lab + 16 b + i, query r
                const bool full = (tile + 1) * kFewTile <= a.L;
                const bool unit_done = t + 1 == comb || tile + 1 >= n_tiles;
                if (norms) {
                    // the largest |w|^2 of the rows of a group (rows past the end repeat the last one): zero only if every element
                    // of the tile is, infinite where something is no number
                    const float least = __ballot(any != 0u) != 0ull ? 1e-30f : 0.0f;
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        float v = sq[b];
                        v += __shfl_xor(v, 16, kWave);
                        v += __shfl_xor(v, 32, kWave);
                        v = v == v ? fmaxf(v, least) : INFINITY;
                        v = fmaxf(v, __shfl_xor(v, 1, kWave));
                        v = fmaxf(v, __shfl_xor(v, 2, kWave));
                        v = fmaxf(v, __shfl_xor(v, 4, kWave));
                        if (a.gshift >= 0) v = fmaxf(v, __shfl_xor(v, 8, kWave));
                        sq[b] = v;
                    }
                    auto error = [he, hs](float v) { return v == 0.0f ? 0.0f : sqrtf(v) * he + hs; };
                    if (a.gshift <= 0) {
                        const int per = a.gshift < 0 ? 4 : 2;   // groups of a tile: lanes 0, 8, 16, 24 of it, or 0, 16
                        const int grp = a.gshift < 0 ? (lane >> 3) : (lane >> 4);
                        const float v = (a.gshift < 0 ? grp >> 1 : grp) == 0 ? sq[0] : sq[1];
                        // (of block 1 the lanes 16.. hold the values of their r as well: rows 0..7 in lanes r < 8, 8..15 in r >= 8)
                        if (grp < per && (lane & (a.gshift < 0 ? 7 : 15)) == 0 && tile * per + grp < a.n_groups)
                            a.gerr[tile * per + grp] = error(v);
                    } else {
                        run_sq = fmaxf(run_sq, fmaxf(sq[0], sq[1]));
                        if (unit_done) {
                            if (lane == 0) a.gerr[unit] = error(run_sq);
                            run_sq = 0.0f;
                        }
                    }
                    sq[0] = 0.0f;
                    sq[1] = 0.0f;
                    any = 0;
                }
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    float m[2];
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        if (!full)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (lab + 16 * b + i >= a.L) acc[b][n][i] = nan;
                        m[b] = fmaxf(fmaxf(acc[b][n][0], acc[b][n][1]), fmaxf(acc[b][n][2], acc[b][n][3])) * bk[n];
                    }
                    acc[0][n] = f32x4{0.f, 0.f, 0.f, 0.f};
                    acc[1][n] = f32x4{0.f, 0.f, 0.f, 0.f};
                    const int64_t q = q0 + n * 16 + r;
                    if (a.gshift <= 0) {
                        m[0] = fmaxf(m[0], __shfl_xor(m[0], 16, kWave));         // lanes g = 0, 1: labels 0..7 of a block, 2, 3: 8..15
                        m[1] = fmaxf(m[1], __shfl_xor(m[1], 16, kWave));
                        if (a.gshift < 0) {
                            // lane g stores group g & 1 of ... : g = 0: block 0 first half, 2: second half, 1 and 3 those of block 1
                            const int64_t grp = 4 * tile + (g >> 1) + 2 * (g & 1);
                            if (q < a.Zq && grp < a.n_groups) a.gmax[q * a.n_groups + grp] = score_image((g & 1) == 0 ? m[0] : m[1]);
                        } else {
                            m[0] = fmaxf(m[0], __shfl_xor(m[0], 32, kWave));
                            m[1] = fmaxf(m[1], __shfl_xor(m[1], 32, kWave));
                            const int64_t grp = 2 * tile + g;
                            if (g < 2 && q < a.Zq && grp < a.n_groups) a.gmax[q * a.n_groups + grp] = score_image(g == 0 ? m[0] : m[1]);
                        }
                    } else {
                        run[n] = fmaxf(run[n], fmaxf(m[0], m[1]));
                        if (unit_done) {
                            run[n] = fmaxf(run[n], __shfl_xor(run[n], 16, kWave));
                            run[n] = fmaxf(run[n], __shfl_xor(run[n], 32, kWave));
                            if (g == 0 && q < a.Zq) a.gmax[q * a.n_groups + unit] = score_image(run[n]);
                            run[n] = nan;
                        }
                    }
                }
                ++t;
                if (unit_done) {
                    t = 0;
                    unit += u_step;
                    if (unit >= n_units) return;
                    norms = static_cast<int>(unit % a.n_qb) == qb;
                }
            }
        }
    }
}

// Bitonic sort of keys[0..n), n <= Finish<NT>::kKeys, by the whole workgroup (ascending; padded with sentinels).
template <int NT>
__device__ void block_sort(uint64_t* keys, int n) {
    int n2 = 64;
    while (n2 < n) n2 <<= 1;
    for (int e = n + static_cast<int>(threadIdx.x); e < n2; e += NT) keys[e] = kKeySentinel;
    __syncthreads();
    for (int size = 2; size <= n2; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int e = threadIdx.x; e < n2 / 2; e += NT) {
                const int lo = 2 * e - (e & (stride - 1));
                const int hi = lo + stride;
                const bool up = (lo & size) == 0;
                const uint64_t x = keys[lo], y = keys[hi];
                if ((x > y) == up) { keys[lo] = y; keys[hi] = x; }
            }
            __syncthreads();
        }
}

// Exclusive prefix sum over the workgroup; `total` gets the sum.  `sh` holds a value per wave.
template <int NT>
__device__ __forceinline__ int block_excl_scan(int v, int* sh, int* total) {
    const int incl = wave_incl_scan(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if (lane_id() == kWave - 1) sh[w] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < Finish<NT>::kWaves; ++i) { before += i < w ? sh[i] : 0; all += sh[i]; }
    *total = all;
    return before + incl - v;
}

// HALF: the maxima are those of few_half_kernel, off by up to their error.
template <typename T, int NT, bool HALF>
__global__ __launch_bounds__(NT)
void few_finish_kernel(const FewArgs a) {
    static_assert(!HALF || std::is_same<T, float>::value, "");
    __shared__ uint64_t keys[Finish<NT>::kKeys];
    __shared__ __align__(16) int hist[2048];
    __shared__ int sh[Finish<NT>::kWaves];
    __shared__ int32_t groups[HALF ? kMoreGroups : XC_MAX_K_MINE];
    __shared__ uint64_t best[HALF ? XC_MAX_K_MINE : 1];
    __shared__ uint4 zop[kFewLds / 256];                       // the query's chunks as operands (ks * 4 of them)
    __shared__ int n_sel, n_key, sel_bin, sel_need, sel_have;
    __shared__ uint32_t tau_sh;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t q = blockIdx.x / a.n_split;
    const int split = blockIdx.x % a.n_split;
    const uint32_t* gm = a.gmax + q * a.n_groups;
    if (!HALF && a.again && a.redo[q] == 0) return;        // uniform
    if (a.flag != nullptr && blockIdx.x == 0)
        for (int i = tid; i < a.n_flag; i += NT) a.flag[i] = 0;

    // ---- the k groups.  Of 256 parts of the groups the k-th largest maximum is no more than the k-th largest of all, and usually
    // close below it: the groups at or above it are ordered by counting.  Where they are too many for that (large maxima close
    // together in the label range, equal ones), digits of 11, 11, 10 bits from the top, until those at or above the digit of
    // the k-th are few enough.  (Digits alone: every maximum adds to one of a few counters, whose additions wait for each
    // other.)  The maxima are read once where the threads can hold them.
    constexpr int kHold = HALF && NT == 256 ? 32 : 8;
    const bool held = a.n_groups <= NT * kHold;                // uniform
    for (int c0 = wave * 4; c0 * 16 < a.row_bytes; c0 += Finish<NT>::kWaves * 4) {         // a step per wave
        const int c = c0 + (lane >> 4);
        uint4 v = make_uint4(0, 0, 0, 0);
        if (c * 16 < a.row_bytes) v = *reinterpret_cast<const uint4*>(a.Z + q * a.row_bytes + c * 16);
        v = FewMma<T>::operand(v);
        if ((lane & 15) == 0) zop[c] = v;
    }
    uint32_t hv[kHold];
    if (held) {
#pragma unroll
        for (int j = 0; j < kHold; ++j) hv[j] = tid + j * NT < a.n_groups ? gm[tid + j * NT] : 0u;
    }
    // f(value, group) for every group, in no order
    auto for_groups = [&](auto f) {
        if (held) {
#pragma unroll
            for (int j = 0; j < kHold; ++j) f(hv[j], static_cast<int32_t>(tid + j * NT));
        } else {
            for (int64_t i = tid; i < a.n_groups; i += NT) f(gm[i], static_cast<int32_t>(i));
        }
    };
    if (tid == 0) { n_sel = 0; n_key = 0; tau_sh = 0xffffffffu; }
    // the query's norm
    float zn = 0.0f;
    auto redo = [&]() {                                        // (every thread that gets here writes the same)
        a.redo_any[0] = 1;
        a.redo[q] = 1;
    };
    if constexpr (HALF) {
        float s2 = 0.0f, zmax = 0.0f;
        for (int64_t i = lane; i * 4 < a.row_bytes; i += kWave) {
            const float v = *reinterpret_cast<const float*>(a.Z + q * a.row_bytes + i * 4);
            s2 = fmaf(v, v, s2);
            zmax = fabsf(v) <= kHalfMost ? fmaxf(zmax, fabsf(v)) : INFINITY;       // (also where it is no number; stays, see below)
            if (!(fabsf(v) <= kHalfMost)) s2 = INFINITY;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) { s2 += __shfl_xor(s2, off, kWave); zmax = fmaxf(zmax, __shfl_xor(zmax, off, kWave)); }
        if (!(s2 < INFINITY) || (zmax != 0.0f && zmax < kHalfLeast)) { redo(); return; }      // uniform over the workgroup: every wave sees the whole row
        zn = sqrtf(s2) * 1.001f;
    }
    auto group_error = [&](int64_t i) {
        const float e = a.gerr[i];
        return e == 0.0f ? 0.0f : zn * e;
    };
    uint32_t prefix = 0;           // the digits found so far
    int bits = 32;                 // bits below them
    int need = a.k;                // groups still to take among those that share the prefix
    uint32_t bound = 0;            // the groups at or above it are ordered by counting; 0: too many with the same maximum
    {
        constexpr int kShare = NT / 256;                        // threads of a part
        uint32_t* part_max = reinterpret_cast<uint32_t*>(hist);             // [256]
        uint32_t mine = 0;
        for_groups([&](uint32_t o, int32_t) { mine = o > mine ? o : mine; });
#pragma unroll
        for (int off = kShare / 2; off > 0; off >>= 1) { const uint32_t o = __shfl_xor(mine, off, kWave); mine = o > mine ? o : mine; }
        if (tid % kShare == 0) part_max[tid / kShare] = mine;
        __syncthreads();
        if (wave == 0) {
            const uint4 v = *reinterpret_cast<const uint4*>(part_max + lane * 4);
            uint32_t t0 = 0;                                    // the k-th largest of them, bit by bit
            for (int b = 31; b >= 0; --b) {
                const uint32_t c = t0 | (1u << b);
                const int have = __popcll(__ballot(v.x >= c)) + __popcll(__ballot(v.y >= c)) + __popcll(__ballot(v.z >= c)) + __popcll(__ballot(v.w >= c));
                if (have >= a.k) t0 = c;
            }
            if (lane == 0) sel_bin = static_cast<int>(t0);      // (0: fewer parts with a score than k)
        }
        __syncthreads();
        const uint32_t t0 = static_cast<uint32_t>(sel_bin);
        if (t0 != 0) {
            for_groups([&](uint32_t o, int32_t i) {
                if (o >= t0) {
                    const int at = atomicAdd(&n_key, 1);
                    if (at < kRankSort) keys[at] = (static_cast<uint64_t>(~o) << 32) | static_cast<uint32_t>(i);
                }
            });
            __syncthreads();
            if (n_key <= kRankSort) bound = t0;
            __syncthreads();
            if (bound == 0 && tid == 0) n_key = 0;
        }
        __syncthreads();
    }
    const bool listed = bound != 0;
    for (int pass = 0; pass < 3 && bound == 0; ++pass) {
        const int width = pass < 2 ? 11 : 10;
        for (int d = tid; d < 2048; d += NT) hist[d] = 0;
        __syncthreads();
        for_groups([&](uint32_t o, int32_t) {
            if (o != 0 && (pass == 0 || (o >> bits) == prefix))
                atomicAdd(&hist[(o >> (bits - width)) & ((1u << width) - 1u)], 1);
        });
        __syncthreads();
        constexpr int kPer = 2048 / NT;                                        // digits per thread, largest first
        int c[kPer], local = 0, total;
#pragma unroll
        for (int j = 0; j < kPer; ++j) { c[j] = hist[2047 - kPer * tid - j]; local += c[j]; }
        int before = block_excl_scan<NT>(local, sh, &total);
        if (pass == 0 && total <= kRankSort) { bound = 1u; break; }            // uniform
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (before < need && need <= before + c[j]) { sel_bin = 2047 - kPer * tid - j; sel_need = need - before; sel_have = c[j]; }
            before += c[j];
        }
        __syncthreads();
        bits -= width;
        prefix = (prefix << width) | static_cast<uint32_t>(sel_bin);
        need = sel_need;
        if (a.k - need + sel_have <= kRankSort) { bound = prefix << bits; break; }      // uniform
        __syncthreads();
    }
    // (bound 0: the prefix is a whole score.  Taken are the groups above it and the first `need` in label order of those
    // that share it; adding 1 cannot wrap: the largest image is that of a NaN)
    const uint32_t least = bound != 0 ? bound : prefix + 1u;
    if (!listed) for_groups([&](uint32_t o, int32_t i) {
        if (o >= least) keys[atomicAdd(&n_key, 1)] = (static_cast<uint64_t>(~o) << 32) | static_cast<uint32_t>(i);
    });
    __syncthreads();
    const int n_cand = n_key;
    for (int m = tid; m < n_cand; m += NT) {                   // larger maxima first, of equal ones the smaller labels
        const uint64_t mine = keys[m];
        int rank = 0;
#pragma unroll 8
        for (int e = 0; e < n_cand; ++e) rank += keys[e] < mine ? 1 : 0;
        if (rank < a.k) groups[rank] = static_cast<int32_t>(mine & 0xffffffffu);
        if (rank == a.k - 1) tau_sh = ~static_cast<uint32_t>(mine >> 32);
    }
    if (tid == 0) n_sel = n_cand < a.k ? n_cand : a.k;
    if (bound == 0) {
        int got = 0;
        for (int64_t i0 = 0; got < need; i0 += NT) {           // uniform (need <= their number)
            const int64_t i = i0 + tid;
            const bool tie = i < a.n_groups && gm[i] == prefix;
            int total;
            const int at = got + block_excl_scan<NT>(tie ? 1 : 0, sh, &total);
            if (tie && at < need) groups[n_cand + at] = static_cast<int32_t>(i);
            got += total;
        }
        __syncthreads();
        if (tid == 0) { n_sel = a.k; tau_sh = prefix; }
    }
    __syncthreads();
    const uint32_t tau = n_sel < a.k ? 1u : tau_sh;            // (fewer groups with a score than k: every score counts)
    __syncthreads();
    if (tid == 0) n_key = 0;
    __syncthreads();
    const int gsh = 4 + a.gshift;                              // labels of a group: 1 << gsh
    int n_rows = n_sel << gsh;
    int n_blocks = (n_rows + 15) >> 4;                         // blocks of 16 labels
    // the first one that is not among the k best groups, as the key of its maximum and place; and the least score that can matter
    uint64_t group_key = 0xffffffffull << 32;                  // (fewer groups with a score: all that have one are)
    if constexpr (HALF) {
        if (n_sel == a.k) group_key = ((static_cast<uint64_t>(~tau) << 32) | static_cast<uint32_t>(groups[a.k - 1])) + 1;
        __syncthreads();
        if (tid == 0) tau_sh = n_sel == a.k ? 0xffffffffu : kTauInit;
        __syncthreads();
        for (int m = tid; m < n_sel; m += NT) {
            const float lo = ordered_to_float(gm[groups[m]]) - group_error(groups[m]);
            atomicMin(&tau_sh, lo == lo ? float_to_ordered(lo) : kTauInit);
        }
        __syncthreads();
    }
    const uint32_t least_score = HALF ? tau_sh : tau;

    // ---- the scores of these groups again: one query in all 16 columns of the product
    const int r = lane & 15, g = lane >> 4;
    auto row_label = [&](int j) { return (static_cast<int64_t>(groups[j >> gsh]) << gsh) + (j & ((1 << gsh) - 1)); };
    // block b: rows 16 b .. 16 b + 15 of the groups; a lane with r < 4 gets the score and label of row 4 g + r.  A wave takes kSide
    // blocks side by side, kAhead steps of each under way: it waits for memory, not for the products.
    constexpr int kSide = NT == 256 ? 2 : 1, kAhead = NT == 256 ? 4 : 16;
    const int row_bytes = static_cast<int>(a.row_bytes);
    auto score_blocks = [&](int b, int b_step, int64_t (&lab)[kSide], float (&score)[kSide]) {
        const unsigned char* wrow[kSide];
        f32x4 acc[kSide];
#pragma unroll
        for (int u = 0; u < kSide; ++u) {
            const int j0 = 16 * (b + u * b_step) + r, j = j0 < n_rows ? j0 : n_rows - 1;
            const int64_t l = row_label(j);
            wrow[u] = a.W + (l < a.L ? l : a.L - 1) * row_bytes;
        }
        score_rows<T, kSide, kAhead>(wrow, zop, row_bytes, g, acc);
#pragma unroll
        for (int u = 0; u < kSide; ++u) {
            const int jr = 16 * (b + u * b_step) + 4 * g + r;
            lab[u] = r < 4 && jr < n_rows ? row_label(jr) : a.L;
            score[u] = (r & 2) ? ((r & 1) ? acc[u][3] : acc[u][2]) : ((r & 1) ? acc[u][1] : acc[u][0]);
        }
    };
    const bool may_overflow = (n_blocks / a.n_split + 1) * 16 > Finish<NT>::kKeys;
    const int n_mine = (n_blocks - split + a.n_split - 1) / a.n_split;          // blocks split, split + n_split, ...
    for (int b0 = 0; b0 < n_mine; b0 += Finish<NT>::kWaves * kSide) {
        const int b = split + (b0 + wave) * a.n_split;
        if (b < n_blocks) {
            int64_t lab[kSide];
            float v[kSide];
            score_blocks(b, Finish<NT>::kWaves * a.n_split, lab, v);
#pragma unroll
            for (int u = 0; u < kSide; ++u)
                if (lab[u] < a.L && score_image(v[u]) >= least_score)
                    keys[atomicAdd(&n_key, 1)] = make_key(v[u] + 0.0f, static_cast<int32_t>(lab[u]));
        }
        if (may_overflow) {                                    // uniform
            __syncthreads();
            if (n_key > Finish<NT>::kKeys - Finish<NT>::kWaves * kSide * 16) {     // the next round might not fit: keep the best k
                const int n = n_key;
                block_sort<NT>(keys, n);
                if (tid == 0) n_key = n < a.k ? n : a.k;
            }
            __syncthreads();
        }
    }
    __syncthreads();
    int n = n_key;
    if (a.n_split > 1) {
        // hand the candidates over; whoever comes last has all of them and finishes the query (nobody waits)
        if (n > kPartKeys) { block_sort<NT>(keys, n); n = a.k; }
        // (stores at agent scope, acknowledged before the count goes up: no cache has to be written back for them, which
        // a fence at that scope would do for the whole XCD - with it, 64 queries of 512-byte rows took 134 us, not 33)
        uint64_t* part = a.part + (q * a.n_split + split) * kPartKeys;
        for (int e = tid; e < n; e += NT)
            __hip_atomic_store(&part[e], keys[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (tid == 0) __hip_atomic_store(&a.part_n[q * a.n_split + split], n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0);                         // this wave's stores have arrived ...
        __syncthreads();                                       // ... and everyone's
        if (tid == 0) sel_have = __hip_atomic_fetch_add(&a.done[q], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (sel_have != a.n_split - 1) return;                 // uniform
        n = 0;
        for (int sp = 0; sp < a.n_split; ++sp) {
            const int np = __hip_atomic_load(&a.part_n[q * a.n_split + sp], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint64_t* from = a.part + (q * a.n_split + sp) * kPartKeys;
            for (int e = tid; e < np; e += NT)
                keys[n + e] = __hip_atomic_load(&from[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            n += np;
        }
        __syncthreads();
    }
    if constexpr (HALF) {
        // ---- the other groups whose maximum, with its error, reaches the k-th best so far (of equal scores the smaller label)
        if (n < a.k) { redo(); return; }                       // uniform (scores that are no numbers)
        __syncthreads();                                       // every wave has read n_key, which starts again below
        if (n <= kRankSort) {
            for (int m = tid; m < n; m += NT) {
                const uint64_t mine = keys[m];
                int rank = 0;
#pragma unroll 8
                for (int e = 0; e < n; ++e) rank += keys[e] < mine ? 1 : 0;
                if (rank < a.k) best[rank] = mine;
            }
        } else {
            block_sort<NT>(keys, n);
            if (tid < a.k) best[tid] = keys[tid];
        }
        if (tid == 0) { n_sel = 0; n_key = 0; }
        __syncthreads();
        const uint64_t kth = best[a.k - 1];
        const float kth_score = key_score(kth);
        // (a maximum that is no number: some score may be one)
        for_groups([&](uint32_t o, int32_t i) {
            if (i >= a.n_groups) return;
            float most = ordered_to_float(o) + group_error(i);
            if (o != 0 && most < kth_score) return;             // nearly all of them
            if (((static_cast<uint64_t>(~o) << 32) | static_cast<uint32_t>(i)) < group_key) return;
            most = o == 0 ? INFINITY : most;
            if (most == most && make_key(most + 0.0f, static_cast<int32_t>(static_cast<int64_t>(i) << gsh)) >= kth) return;
            const int at = atomicAdd(&n_sel, 1);
            if (at < kMoreGroups) groups[at] = i;
        });
        __syncthreads();
        if (n_sel > kMoreGroups) { redo(); return; }           // uniform
        n_rows = n_sel << gsh;
        n_blocks = (n_rows + 15) >> 4;
        for (int b = wave; b < n_blocks; b += Finish<NT>::kWaves * kSide) {
            int64_t lab[kSide];
            float v[kSide];
            score_blocks(b, Finish<NT>::kWaves, lab, v);
#pragma unroll
            for (int u = 0; u < kSide; ++u) {
                const uint64_t key = make_key(v[u] + 0.0f, static_cast<int32_t>(lab[u]));
                if (lab[u] < a.L && v[u] == v[u] && key < kth) {
                    const int at = atomicAdd(&n_key, 1);
                    if (at < Finish<NT>::kKeys - XC_MAX_K_MINE) keys[at] = key;
                }
            }
        }
        __syncthreads();
        n = n_key;
        if (n > Finish<NT>::kKeys - XC_MAX_K_MINE) { redo(); return; }        // uniform
        __syncthreads();
        if (tid < a.k) keys[n + tid] = best[tid];
        n += a.k;
        __syncthreads();
    }
    int32_t* ids = a.shortlist + q * a.k;
    float* sc = a.scores != nullptr ? a.scores + q * a.k : nullptr;
    auto put = [&](int rank, uint64_t key) {
        ids[rank] = key_id(key);
        if (sc != nullptr) sc[rank] = key_score(key);
        if (rank == a.k - 1) a.tau_g[q] = float_to_ordered(key_score(key));
    };
    if (n <= kRankSort) {                                      // a key's place is the number of smaller keys
        for (int m = tid; m < n; m += NT) {
            const uint64_t mine = keys[m];
            int rank = 0;
#pragma unroll 8
            for (int e = 0; e < n; ++e) rank += keys[e] < mine ? 1 : 0;
            if (rank < a.k) put(rank, mine);
        }
    } else {
        block_sort<NT>(keys, n);
        if (tid < a.k) put(tid, keys[tid]);
    }
    if (tid < a.k && tid >= n) {
        ids[tid] = -1;
        if (sc != nullptr) sc[tid] = -INFINITY;
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
constexpr int64_t kHalfFrom = 16;            // fp32: more queries than this take 16-bit maxima
// ... and more Gflop (blocks of 16 queries padded): below, the two launches that return at once cost more than fp32 products.  us, fp32 and 16-bit
// maxima: 20 queries x 4096 x 64 19 and 27, 250 x 10 000 x 128 33 and 38, 100 x 20 000 x 256 43 and 47, 128 x 40 000 x 256 65 and 51, 250 x 20 000 x 256 70 and 48
constexpr double kHalfGflop = 2.5;
constexpr int64_t kFewAlways = 96;           // up to so many queries always
constexpr int64_t kFewQueries = 256;         // one query tile of the other kernels: up to so many usually
constexpr int64_t kFewMaxQueries = 2048;     // beyond that never

// Workgroups of the first kernel: as many label ranges per block of queries as fit the chip (two workgroups per compute unit
// where two query blocks fit its LDS), in multiples of the 8 XCDs and at least 8.
static int64_t few_slots(size_t lds) { return lds <= (80u << 10) ? 512 : 256; }
static int64_t few_ranges(size_t lds, int n_qb) {
    const int64_t n = few_slots(lds) / n_qb / 8 * 8;
    return n < 8 ? 8 : n;
}

// The share of the slots' time that such workgroups use.
static double few_used(size_t lds, int n_qb) {
    const double slots = static_cast<double>(few_slots(lds)), wgs = static_cast<double>(few_ranges(lds, n_qb) * n_qb);
    return wgs / (slots * ceil(wgs / slots));
}

// Whether W is read by whole lines (few_line_kernel) where the rows have them and the stages fit LDS beside the queries, or 64 bytes of 16 rows at a
// time (few_max_kernel).  Lines are the better way but for two things.  Short rows that end within a line share it with their neighbours, and where
// several blocks of queries read them from memory that costs more than lines gain: halves : lines, us, 127 x 8.2 M x 96 bf16 784 : 905, 459 x
// 8.1 M x 96 2062 : 2550, 328 x 3.8 M x 200 1923 : 2298; the other way 128 x 300 000 x 96 50 : 47, 256 x 300 000 x 200 120 : 112.  And a
// stage's LDS may leave one workgroup to a compute unit where two would fit, and a last round mostly empty: 1120 x 192 228 x 504 559 : 661.
// Over 2250 searches of 97 to 2048 queries this is 0.3 % off the better of both, 19 % at worst (always lines 0.6 and 26).
static bool few_lines(const FewPlan& p, int64_t L, int64_t row_bytes, bool f32) {
    if ((f32 && p.nb > 1) || row_bytes < 128 || p.line_lds > kLineLds) return false;
    if (row_bytes % 128 != 0 && row_bytes < 512 && L * row_bytes >= (192ll << 20) && p.n_qb >= (row_bytes < 256 ? 2 : 5)) return false;
    return few_used(p.line_lds, p.n_qb) >= 0.75 * few_used(p.lds, p.n_qb);
}

// Estimated time of this search, and of the other kernels' where it can be the smaller one, in us.  bf16: least squares over 2650
// searches of 97 to 2048 queries, 3000 to 30 million rows of 128 to 9216 bytes, k = 5 to 100, W from memory.  Half of the estimates are
// within an eighth, nine in ten within two fifths; choosing by them costs 1.7 % over always choosing right (beyond 256 queries 2.8 %; the line at six
// tiles of 256 x 256 per compute unit that was fitted to half lines, with all that the row kernel takes on this side of it, cost 28 %, and
// 9 of 1600 searches took a better way there, by a third at most).  fp32: 870 searches, 0.6 % with the fifth below.  This search: scores and their products per block of 16, 32 or 64 queries, with
// what the last round of workgroups leaves idle; rows read again by the second kernel; maxima (stored four bytes at a time, dearer
// where 64 MB of them are under way); W.  The others: products, W, what passes (more per query tile, and
// much more where k > 64), the phases' start-up; rows that are no multiple of a stage load slowly.
static double few_us(const FewPlan& p, int64_t Zq, int64_t L, int64_t row_bytes, int k, bool f32) {
    const double padded = static_cast<double>(p.n_qb) * p.nb * 16;
    const double gflop = 2e-9 * padded * L * (row_bytes / (f32 ? 4 : 2)) / few_used(p.lines ? p.line_lds : p.lds, p.n_qb);
    const double maxima = 1e-6 * padded * p.n_groups, rows = 1e-6 * Zq * k * (16 << p.gshift) * row_bytes;
    if (f32) return 22.0 + gflop * (p.nb == 1 ? 13.9 : p.nb == 2 ? 8.4 : 8.2) + 0.16 * rows + maxima * (maxima < 16.0 ? 5.1 : 12.0);
    const double per = p.nb == 1 ? 3.4 : p.nb == 2 ? (p.lines ? 1.5 : 3.2) : (p.lines ? 0.88 : 1.4);
    return 15.0 + 79e-9 * padded * L + gflop * per + 0.125 * rows + 4.5 * maxima + (maxima > 16.0 ? 4.3 * (maxima - 16.0) : 0.0) + 0.27e-6 * L * row_bytes;
}
static double others_us(int64_t Zq, int64_t L, int64_t row_bytes, int k, bool f32, bool row_kernel, bool warm) {
    const double mlab = 1e-6 * L, kb = 1e-3 * row_bytes, long_list = k > 64 ? 1.0 : 0.0, zk = 1e-3 * Zq * k;
    const bool tail = row_bytes % kStageBytes != 0;
    if (Zq <= kBN) {
        if (row_kernel) return 45.0 + mlab * (kb * (541.0 + long_list * 636.0) + 9.0 + 0.44 * k) + 21.0 * kb + 1.28 * zk;
        return (warm ? 37.0 + 17.0 * kb : 58.0 + 30.0 * kb) + mlab * (kb * (860.0 + (tail ? 280.0 : 0.0) + long_list * 820.0) + 90.0 + long_list * 190.0) + 0.77 * zk;
    }
    const double qt = static_cast<double>((Zq + kBN - 1) / kBN), gflop = 2e-9 * qt * kBN * L * (row_bytes / (f32 ? 4 : 2));
    if (f32) return 84.0 + gflop * (tail ? 5.2 : 2.3) + 2960.0 * mlab * kb + 19.0 * qt * mlab + 100.0 * kb + long_list * 1190.0 * mlab;
    if (row_kernel) return 245.0 + 0.99 * gflop + mlab * (102.0 + 46.0 * kb + 1.3 * qt + long_list * 279.0) + 1.09 * zk + 0.0124 * Zq;
    return 63.0 + 0.62 * gflop + mlab * ((tail ? 825.0 : 537.0) * kb + 55.0 * qt + long_list * 666.0) + 0.124 * zk + 28.0 * kb;
}

// The same where both have fp16 copies (fp32 rows, more than 256 queries): least squares over 70 searches of 128 to 2048 queries, 5000 to
// 4 million rows of 64 to 768 elements, k = 5 to 100, within a tenth for half of them; over 473 others of 257 to 2048 queries, 3000 to 10 million rows
// of 64 to 1024 elements, choosing by these costs 4 % over always choosing right (always one or the other 29 % and more).  Searches of too few products
// for 16-bit maxima are held against the copies by few_us: few queries : copies, us, 264 x 10 771 x 256, k = 20 58 : 158; 560 x 8264 x 256, k = 5 61 : 121;
// 910 x 6435 x 200, k = 20 77 : 147; 293 x 4253 x 768, k = 100 335 : 199 (of 34 such searches three take the slower, by 1.3 at most).
static double few_half_us(const FewPlan& p, int64_t Zq, int64_t L, int64_t row_bytes, int k) {
    const double slots = static_cast<double>(few_slots(p.hlds)), wgs = static_cast<double>(few_ranges(p.hlds, p.hn_qb) * p.hn_qb);
    const double gflop = 2e-9 * p.hn_qb * p.hnb * 16 * L * (row_bytes / 4) * slots * ceil(wgs / slots) / wgs;
    const double rows = static_cast<double>(Zq) * k * (1 << (4 + p.hgshift)) * row_bytes;
    return 30.0 + gflop * (p.hnb == 8 ? 1.73 : 3.04) + 0.157e-6 * rows + 9.5e-6 * Zq * p.hn_groups + 0.143e-6 * L * row_bytes;
}
static double others_half_us(int64_t Zq, int64_t L, int64_t row_bytes, int k) {
    const double nq = static_cast<double>((Zq + kBN - 1) / kBN * kBN), zk = static_cast<double>(Zq) * k;
    return 142.0 + 0.075e-9 * 2.0 * nq * L * (row_bytes / 4) + 0.70e-6 * L * row_bytes + 1.07e-3 * zk + 0.386e-6 * nq * L + 0.235e-6 * zk * row_bytes;
}

// Scratch: maxima, candidates of shared queries and the counts that go with these; with 16-bit maxima the groups' norms and a word per query.
static size_t few_bytes(size_t q, int64_t groups, int ns) { return round_up(q * groups * 4, 256) + q * ns * kPartKeys * 8 + round_up(q * ns * 4, 256) + q * 4; }
static size_t few_half_bytes(size_t q, int64_t groups) { return 256 + round_up(static_cast<size_t>(groups) * 4, 256) + q * 4; }

// Which searches come here.  Up to 96 queries (less than half of a query tile of the general kernel) all whose query block fits LDS:
// 131 072 x 768 bf16, k = 5: 54 us against 408 at 64 queries; 4 M x 256 bf16, k = 50: 0.57 ms against 1.57.  More queries
// cost this path time in proportion (it multiplies W once per block of at most 64), the others almost nothing until their tiles of
// 256 x 256 fill the chip several times over.  Up to 256 queries also all whose alternative has phases too short to fill the chip: fp32
// (256 x 1 M x 128, k = 100 639 and 4302), and bf16 from scratch, rows that leave LDS room for 64 queries (of 400 searches
// the other way was better in three, by 6 % at most).  Of the rest up to 2048 queries the estimates choose: up to 256 queries (from thresholds) with a
// seventh in favour of this path against the row kernel, beyond with a twentieth against it, and a quarter where there are more than six tiles of 256 x
// 256 per compute unit (where the estimates err by these parts); in fp32 with a fifth in favour, up to 16 tiles of
// 256 x 256 per compute unit and 1.3 GB of rows read again.  Here and there, us, bf16: 1257 x 118 938 x 256, k = 100 291 and 640;
// 276 x 652 935 x 1024, k = 20 692 and 1363; 643 x 361 318 x 128, k = 20 240 and 478; the other way 690 x 793 300 x 1024, k =
// 20 2124 and 1702; from thresholds 256 x 10 M x 128, k = 50 1293 and 1601, 256 x 4 M x 128, k = 5 866 and 643, 256 x 4 M x 64 688 and 383; fp32
// 1024 x 262 141 x 768 3480 and 3100, 1024 x 78 589 x 300 445 and 590.
bool plan_few(int64_t Zq, int64_t L, int64_t row_bytes, int k, xc_dtype t, bool warm, bool half, size_t scratch, FewPlan* p) {
    const bool f32 = t == XC_F32;
    const int64_t tiles = ((Zq + 255) / 256) * ((L + 255) / 256);
    if (Zq > kFewQueries) {
        if (Zq > kFewMaxQueries || (f32 && tiles > 16 * 256)) return false;
        if (f32 && static_cast<double>(Zq) * k * 16.0 * static_cast<double>(row_bytes) > 1.3e9) return false;
    }
    const int64_t ks = (row_bytes + 63) / 64;
    if (ks * 1024 > static_cast<int64_t>(kFewLds)) return false;
    p->ks = static_cast<int>(ks);
    int nb = 1;
    while (nb < 4 && nb * 16 < Zq && static_cast<size_t>(2 * nb * ks) * 1024 <= kFewLds) nb <<= 1;
    p->nb = nb;
    p->n_qb = static_cast<int>((Zq + nb * 16 - 1) / (nb * 16));
    p->lds = static_cast<size_t>(nb) * ks * 1024;
    p->line_lds = static_cast<size_t>(nb) * ((ks + 1) & ~1) * 1024 + kFewWaves * kFewStage;
    p->lines = few_lines(*p, L, row_bytes, f32);
    // groups of 16 labels (least to compute again) while a query has at most 2^17 of them
    int gs = 0;
    while (gs < 4 && (L >> (4 + gs)) > (1 << 17)) ++gs;
    p->gshift = gs;
    p->n_groups = (L + (16LL << gs) - 1) / (16LL << gs);
    const bool row_kernel = !f32 && row_bytes % kStageBytes == 0 && row_bytes <= kMaxRowKernelBytes;
    const bool always = Zq <= kFewAlways || (Zq <= kFewQueries && (f32 || (!warm && nb == 4)));
    const double favour = f32 ? 1.2 : Zq <= kFewQueries ? (row_kernel ? 1.15 : 1.0) : tiles <= 6 * 256 ? 0.95 : 0.75;
    // (the choice among the fp16 forms of both is made below)
    if (!always && !(f32 && half) && few_us(*p, Zq, L, row_bytes, k, f32) >= favour * others_us(Zq, L, row_bytes, k, f32, row_kernel, warm)) return false;
    // the second kernel: as many workgroups per query as give each wave one block of 16 labels, within what the chip holds
    int ns = 1;
    while (ns < kMaxSplit && Zq * ns * 2 <= 256 && (static_cast<int64_t>(k) << gs) > ns * Finish<1024>::kWaves) ns <<= 1;
    p->n_split = ns;
    const size_t q = static_cast<size_t>(Zq);
    if (few_bytes(q, p->n_groups, ns) > scratch) return false;
    p->hnb = 0;
    if (f32 && Zq > kHalfFrom && 2e-9 * p->n_qb * p->nb * 16 * L * (row_bytes / 4) > kHalfGflop) {
        p->hks = static_cast<int>((row_bytes + 127) / 128);
        int hnb = 2;
        while (hnb < 8 && hnb * 16 < Zq && static_cast<size_t>(2 * hnb * p->hks) * 1024 + 2 * hnb * 64 + kHalfSample * 4 <= kFewLds) hnb <<= 1;
        p->hlds = static_cast<size_t>(hnb) * p->hks * 1024 + hnb * 64 + kHalfSample * 4;
        p->hn_qb = static_cast<int>((Zq + hnb * 16 - 1) / (hnb * 16));
        p->hgshift = gs == 0 ? -1 : gs;
        p->hn_groups = gs == 0 ? (L + 7) / 8 : p->n_groups;
        if (p->hlds <= kFewLds && few_bytes(q, p->hn_groups, ns) + few_half_bytes(q, p->hn_groups) <= scratch) p->hnb = hnb;
    }
    if (!always && f32 && half) {
        const double here = p->hnb > 0 ? few_half_us(*p, Zq, L, row_bytes, k) : few_us(*p, Zq, L, row_bytes, k, true);
        if (here >= others_half_us(Zq, L, row_bytes, k)) return false;
    }
    return true;
}

typedef void (*FewFn)(const FewArgs);
template <typename T>
static FewFn few_kernel(int nb, bool ktail);
// way: 0 whole lines, 1 rows that end within one, 2 whole lines read past the caches
template <typename T> static FewFn line_kernel(int nb, int way);
template <> FewFn line_kernel<bf16_t>(int nb, int way) {
    static const FewFn fns[3][3] = {
        {&few_line_kernel<bf16_t, 1, false, false>, &few_line_kernel<bf16_t, 1, true, false>, &few_line_kernel<bf16_t, 1, false, true>},
        {&few_line_kernel<bf16_t, 2, false, false>, &few_line_kernel<bf16_t, 2, true, false>, &few_line_kernel<bf16_t, 2, false, true>},
        {&few_line_kernel<bf16_t, 4, false, false>, &few_line_kernel<bf16_t, 4, true, false>, &few_line_kernel<bf16_t, 4, false, true>}};
    return fns[nb >> 1][way];
}
template <> FewFn line_kernel<float>(int nb, int way) {
    static const FewFn fns[3] = {&few_line_kernel<float, 1, false, false>, &few_line_kernel<float, 1, true, false>, &few_line_kernel<float, 1, false, true>};
    return nb == 1 ? fns[way] : nullptr;
}
template <> FewFn few_kernel<bf16_t>(int nb, bool ktail) {
    return nb == 1 ? (ktail ? &few_max_kernel<bf16_t, 1, true> : &few_max_kernel<bf16_t, 1, false>)
         : nb == 2 ? (ktail ? &few_max_kernel<bf16_t, 2, true> : &few_max_kernel<bf16_t, 2, false>)
                   : (ktail ? &few_max_kernel<bf16_t, 4, true> : &few_max_kernel<bf16_t, 4, false>);
}
template <> FewFn few_kernel<float>(int nb, bool ktail) {
    return nb == 1 ? (ktail ? &few_max_kernel<float, 1, true> : &few_max_kernel<float, 1, false>)
         : nb == 2 ? (ktail ? &few_wide_kernel<2, true> : &few_wide_kernel<2, false>)
                   : (ktail ? &few_wide_kernel<4, true> : &few_wide_kernel<4, false>);
}

static FewFn half_kernel(int nb, bool ktail) {
    return nb == 2 ? (ktail ? &few_half_kernel<2, true> : &few_half_kernel<2, false>)
         : nb == 4 ? (ktail ? &few_half_kernel<4, true> : &few_half_kernel<4, false>)
                   : (ktail ? &few_half_kernel<8, true> : &few_half_kernel<8, false>);
}

int few_raise_lds() {
    for (int nb = 1; nb <= 4; nb <<= 1)
        for (int way = 0; way < 3; ++way)
            for (const FewFn fn : {line_kernel<bf16_t>(nb, way), line_kernel<float>(nb, way)})
                if (fn != nullptr)
                    XC_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     static_cast<int>(kLineLds)));
    for (int nb = 2; nb <= 8; nb <<= 1)
        for (int tail = 0; tail < 2; ++tail)
            XC_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(half_kernel(nb, tail != 0)),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kFewLds)));
    for (int nb = 1; nb <= 4; nb <<= 1)
        for (int tail = 0; tail < 2; ++tail)
            for (int f32 = 0; f32 < 2; ++f32) {
                const FewFn fn = f32 ? few_kernel<float>(nb, tail != 0) : few_kernel<bf16_t>(nb, tail != 0);
                XC_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kFewLds)));
            }
    return XC_OK;
}

// Workgroups of a first kernel: no more label ranges than there are tiles.
static dim3 few_grid(size_t lds, int n_qb, int64_t L) {
    const int64_t tiles = (L + kFewTile - 1) / kFewTile;
    const int64_t enough = ((tiles + kFewWaves - 1) / kFewWaves + 7) / 8 * 8;
    const int64_t most = few_ranges(lds, n_qb);
    return dim3(static_cast<unsigned>((most < enough ? most : enough) * n_qb));
}

template <typename T, bool HALF>
static void launch_finish(const FewArgs& a, hipStream_t st) {
    const unsigned n = static_cast<unsigned>(a.Zq * a.n_split);
    if (a.Zq >= kSmallFinishQueries) few_finish_kernel<T, 256, HALF><<<n, 256, 0, st>>>(a);
    else few_finish_kernel<T, 1024, HALF><<<n, 1024, 0, st>>>(a);
}

// Rows of whole lines that one block of queries reads once, from a W that the last-level cache does not hold, leave the caches at once.
// us without and with that: 32 queries x 1.3 M x 768 452 and 400, 64 x 3 M x 256 432 and 393, 2 x 500 000 x 384 94 and 91, 32 x 131 072 x 768 (201 MB) 52
// and 52; but rows of 400 bytes, whose lines two loads share, 483 and 640, and several blocks of queries (1000 x 50 000 x 256) 105 and 117.
static int line_way(const FewArgs& a, int n_qb) {
    if (a.row_bytes % 128 != 0) return 1;
    return n_qb == 1 && reinterpret_cast<uintptr_t>(a.W) % 128 == 0 && a.L * a.row_bytes > (256ll << 20) ? 2 : 0;
}

template <typename T>
static int launch_few(const FewPlan& p, const FewArgs& a, hipStream_t st) {
    const FewFn fn = p.lines ? line_kernel<T>(p.nb, line_way(a, p.n_qb)) : few_kernel<T>(p.nb, a.row_bytes % 64 != 0);
    const size_t lds = p.lines ? p.line_lds : p.lds;
    const dim3 grid = few_grid(lds, p.n_qb, a.L);
    XC_LAUNCH(K_MINE_TILE, st, (fn<<<grid, kFewThreads, lds, st>>>(a)));
    XC_HIP_CHECK(hipGetLastError());
    XC_LAUNCH(K_MINE_SELECT, st, (launch_finish<T, false>(a, st)));
    XC_HIP_CHECK(hipGetLastError());
    return XC_OK;
}

// 16-bit maxima; then the fp32 kernels for the queries that these did not settle (without any, they return at once).  The event timing counts
// all behind the maxima as one selection.
static int launch_half(const FewPlan& p, const FewArgs& exact, hipStream_t st) {
    FewArgs a = exact;
    a.ks = p.hks; a.n_qb = p.hn_qb; a.gshift = p.hgshift; a.n_groups = p.hn_groups;
    const FewFn fn = half_kernel(p.hnb, a.row_bytes % 128 != 0);
    const dim3 grid = few_grid(p.hlds, p.hn_qb, a.L);
    XC_LAUNCH(K_MINE_TILE, st, (fn<<<grid, kFewThreads, p.hlds, st>>>(a)));
    XC_HIP_CHECK(hipGetLastError());
    auto rest = [&]() -> int {
        launch_finish<float, true>(a, st);
        XC_HIP_CHECK(hipGetLastError());
        a = exact;
        a.again = 1;
        a.flag = nullptr;
        const FewFn again = few_kernel<float>(p.nb, a.row_bytes % 64 != 0);
        again<<<few_grid(p.lds, p.n_qb, a.L), kFewThreads, p.lds, st>>>(a);
        XC_HIP_CHECK(hipGetLastError());
        launch_finish<float, false>(a, st);
        XC_HIP_CHECK(hipGetLastError());
        return XC_OK;
    };
    int rc = XC_OK;
    XC_LAUNCH(K_MINE_SELECT, st, rc = rest());
    return rc;
}

int run_mine_few(const FewPlan& p, const void* Z, const void* W, int64_t Zq, int64_t L, int64_t row_bytes, int k,
                 xc_dtype t, unsigned char* scratch, uint32_t* tau_g, int32_t* flag, int n_flag, int32_t* redo_any,
                 int32_t* shortlist, float* scores, hipStream_t st) {
    FewArgs a;
    a.Z = static_cast<const unsigned char*>(Z);
    a.W = static_cast<const unsigned char*>(W);
    a.Zq = Zq; a.L = L; a.row_bytes = row_bytes;
    a.ks = p.ks; a.n_qb = p.n_qb; a.gshift = p.gshift; a.k = k;
    a.n_groups = p.n_groups;
    a.tau_g = tau_g; a.flag = flag; a.n_flag = n_flag;
    a.shortlist = shortlist; a.scores = scores;
    a.n_split = p.n_split;
    a.again = 0;
    a.redo_any = redo_any;
    const int64_t most_groups = p.hnb > 0 && p.hn_groups > p.n_groups ? p.hn_groups : p.n_groups;
    unsigned char* s = scratch;
    a.gmax = reinterpret_cast<uint32_t*>(s); s += round_up(static_cast<size_t>(Zq) * most_groups * 4, 256);
    a.part = reinterpret_cast<uint64_t*>(s); s += static_cast<size_t>(Zq) * p.n_split * kPartKeys * 8;
    a.part_n = reinterpret_cast<int32_t*>(s); s += round_up(static_cast<size_t>(Zq) * p.n_split * 4, 256);
    a.done = reinterpret_cast<int32_t*>(s); s += round_up(static_cast<size_t>(Zq) * 4, 256);
    a.gerr = reinterpret_cast<float*>(s); s += round_up(static_cast<size_t>(most_groups) * 4, 256);     // (these two only with 16-bit maxima)
    a.redo = reinterpret_cast<int32_t*>(s);
    if (t == XC_BF16) return launch_few<bf16_t>(p, a, st);
    return p.hnb > 0 ? launch_half(p, a, st) : launch_few<float>(p, a, st);
}

}  // namespace xc
