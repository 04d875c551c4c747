// The search of a large pool over a long range of short bf16 rows, with an 8-bit filter in front: the same exact top-k as
// xc_mine.hip.  What a search spends its time on is finding out, for nearly every label, that it does NOT reach a
// query's threshold; the matrix pipe answers that twice as fast on 8-bit integers as on bf16, with a rigorous margin:
//   z = a p + dz, w = b q + dw   (p, q integers in [-127, 127]; a per query, b per tile of 64 labels)
//   <z, w> = a b <p, q> + <a p, dw> + <dz, w>,  hence  <z, w> <= a b <p, q> + |a p| |dw| + |dz| |w|   (Cauchy-Schwarz),
// with <p, q> exact in the integer accumulators.  A label whose right side stays below the threshold is out; the few
// others (four to five times as many as a filter without error would let through, at 256 elements) get their score from
// the bf16 rows, summed in fp32 in the order of the bf16 kernels, and only these scores decide.  The result is that of
// the bf16 search, bit for bit.
//   q8_queries_kernel   p, 1 / a and the margins of a query, once per search
//   per chunk of labels (up to kQ8ChunkBytes of 8-bit rows):
//   q8_rows_kernel      q, 1 / b and the largest |dw|, |w| of every tile of 64 labels (HBM: 3 bytes per element)
//   mine_q8_kernel      the filter: mine_rows_kernel's structure (512 queries of a work item in registers, W streamed
//                       through LDS), labels that pass go to lists owned by a lane
//   q8_rescore_kernel   one wave per query: the scores of what passed; what is not a number or below the threshold goes
//   mine_rows_kernel    on the 256-query tiles that the filter gave up (a list ran over: scores that rise along the label
//                       range, rows too uneven for 8 bits, infinities); returns at once if there are none
//   mine_select_kernel  the best k so far and the next threshold
// Once the tiles that a chunk gives up take more than half as long as a search without the filter, it is not tried again in
// this search.
#include "xc_mine.h"

namespace xc {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

constexpr int kQ8Tile = 64;              // labels of a tile: one scale
constexpr int kQ8Queries = 512;          // queries of a work item
constexpr int kQ8Cap = 512;              // entries of a lane's list (2 lists per query)
constexpr int kQ8MaxTiles = 4096;        // tiles of a slice at most (their margins are kept in LDS)
constexpr float kQ8Huge = 3.0e38f;
// kinds of queries (last component of their parameters)
constexpr float kQueryPlain = 0.0f, kQueryWide = 1.0f /* infinite, or out of the margins' range */, kQueryZero = 2.0f, kQueryNan = 3.0f;

// ---------------------------------------------------------------------------
// operands
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t abs_max_bits(const uint4& v) {       // largest |element| of 8, as float bits
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t x = i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
        const uint32_t lo = (x << 16) & 0x7fff0000u, hi = x & 0x7fff0000u;
        m = lo > m ? lo : m;
        m = hi > m ? hi : m;
    }
    return m;
}
// not a finite number, or so large or small that the margins could leave the range of fp32
__device__ __forceinline__ bool unusable(uint32_t max_bits) {
    const float m = __uint_as_float(max_bits);
    return max_bits >= 0x7f800000u || m > 1e15f || (max_bits != 0 && m < 1e-15f);
}
// 8 elements -> 8 integers; adds the squares of the errors and of the rounded values' originals
__device__ __forceinline__ uint2 quantise8(const uint4& v, float inv, float step, float& err2, float& sum2, float& app2) {
    float f[8];
    unpack8(v, f);
    uint32_t o[2] = {0, 0};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float q = rintf(f[e] * inv);
        const float d = fmaf(-q, step, f[e]);
        err2 = fmaf(d, d, err2);
        sum2 = fmaf(f[e], f[e], sum2);
        app2 = fmaf(q, q, app2);
        o[e >> 2] |= (static_cast<uint32_t>(static_cast<int>(q)) & 0xffu) << (8 * (e & 3));
    }
    return make_uint2(o[0], o[1]);
}

template <int NK>
__global__ __launch_bounds__(256)
void q8_queries_kernel(const unsigned char* __restrict__ Z, int64_t Zq, unsigned char* __restrict__ out,
                       float4* __restrict__ zpar, int32_t* __restrict__ state) {
    constexpr int G = 16 * NK;                           // lanes with a chunk
    const int lane = lane_id();
    const int64_t q = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (blockIdx.x == 0 && threadIdx.x < 2) state[threadIdx.x] = 0;
    if (q >= Zq) return;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (lane < G) v = *reinterpret_cast<const uint4*>(Z + (q * G + lane) * 16);
    uint32_t m = abs_max_bits(v);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { const uint32_t o = __shfl_xor(m, off, kWave); m = o > m ? o : m; }
    const bool bad = unusable(m) || m == 0;
    const float kind = m == 0 ? kQueryZero : m > 0x7f800000u ? kQueryNan : bad ? kQueryWide : kQueryPlain;
    const float inv = bad ? 0.0f : 127.0f / __uint_as_float(m), step = __uint_as_float(m) / 127.0f;
    float e2 = 0.0f, s2 = 0.0f, a2 = 0.0f;
    const uint2 o = quantise8(v, inv, step, e2, s2, a2);
    if (lane < G) *reinterpret_cast<uint2*>(out + (q * G + lane) * 8) = bad ? make_uint2(0, 0) : o;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        e2 += __shfl_xor(e2, off, kWave); s2 += __shfl_xor(s2, off, kWave); a2 += __shfl_xor(a2, off, kWave);
    }
    if (lane == 0) {
        // in units of a: |p| multiplies a tile's |dw|, (|dz| + what summing d products in fp32 can lose, over |z|) its |w|;
        // a ten-thousandth on top covers the rounding of the norms and of the threshold itself
        constexpr float kSum = 4.0f * (128 * NK) * 5.97e-8f;
        const float p = sqrtf(a2) * 1.0001f, w = fmaxf((sqrtf(e2) + kSum * sqrtf(s2)) * inv * 1.0001f, 1e-20f);
        zpar[q] = bad ? make_float4(0.0f, 0.0f, 1e-20f, kind) : make_float4(inv, p, w, kind);
    }
}

template <int NK>
__global__ __launch_bounds__(256)
void q8_rows_kernel(const unsigned char* __restrict__ W /* first row of the chunk */, int64_t n_lab,
                    unsigned char* __restrict__ out, float4* __restrict__ tmeta, const int32_t* __restrict__ gcnt,
                    int32_t* __restrict__ gbase, int64_t nq, int32_t* __restrict__ flag /* [1 + n_qt] */, int n_qt,
                    const int32_t* __restrict__ state) {
    constexpr int G = 16 * NK;                           // lanes per row
    constexpr int kRows = 256 / G;                       // rows of one pass
    constexpr int kIter = kQ8Tile / kRows;
    __shared__ uint32_t shm[4];
    __shared__ float shf[4][2];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const bool off = state[1] != 0;                      // the filter is not tried again: every tile goes the other way
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + tid; i < nq; i += static_cast<int64_t>(gridDim.x) * 256)
        gbase[i] = gcnt[i];
    for (int i = blockIdx.x * 256 + tid; i <= n_qt; i += gridDim.x * 256) flag[i] = off ? 1 : 0;
    if (off) return;                                     // uniform
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * kQ8Tile + tid / G;
    const int c = tid % G;
    uint4 v[kIter];
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        const int64_t r = row0 + i * kRows;
        v[i] = make_uint4(0, 0, 0, 0);                   // (rows past the end: zeros, dropped by the filter)
        if (r < n_lab) v[i] = load16<true>(W + (r * G + c) * 16);
    }
#pragma unroll
    for (int i = 0; i < kIter; ++i) { const uint32_t x = abs_max_bits(v[i]); m = x > m ? x : m; }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { const uint32_t x = __shfl_xor(m, o, kWave); m = x > m ? x : m; }
    if (lane == 0) shm[wave] = m;
    __syncthreads();
    m = shm[0];
#pragma unroll
    for (int w = 1; w < 4; ++w) m = shm[w] > m ? shm[w] : m;
    const bool bad = unusable(m);
    const float inv = (bad || m == 0) ? 0.0f : 127.0f / __uint_as_float(m);
    const float step = bad ? 0.0f : __uint_as_float(m) / 127.0f;
    float emax = 0.0f, smax = 0.0f;
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        float e2 = 0.0f, s2 = 0.0f, a2 = 0.0f;
        const uint2 o = quantise8(v[i], inv, step, e2, s2, a2);
        *reinterpret_cast<uint2*>(out + ((row0 + i * kRows) * G + c) * 8) = bad ? make_uint2(0, 0) : o;
#pragma unroll
        for (int x = G / 2; x > 0; x >>= 1) { e2 += __shfl_xor(e2, x, kWave); s2 += __shfl_xor(s2, x, kWave); }
        emax = fmaxf(emax, e2);
        smax = fmaxf(smax, s2);
    }
#pragma unroll
    for (int x = 32; x >= G; x >>= 1) { emax = fmaxf(emax, __shfl_xor(emax, x, kWave)); smax = fmaxf(smax, __shfl_xor(smax, x, kWave)); }
    if (lane == 0) { shf[wave][0] = emax; shf[wave][1] = smax; }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 0; w < 4; ++w) { emax = fmaxf(emax, shf[w][0]); smax = fmaxf(smax, shf[w][1]); }
        // (1 / b, |dw| / b, |w| / b); a tile of zeros: its scores are zero, so any positive threshold is out of reach; an
        // unusable one: everything passes
        tmeta[blockIdx.x] = bad ? make_float4(0.0f, 0.0f, kQ8Huge, 0.0f)
                          : m == 0 ? make_float4(kQ8Huge, 0.0f, 0.0f, 0.0f)
                                   : make_float4(inv, sqrtf(emax) * inv * 1.0001f, sqrtf(smax) * inv * 1.0001f, 0.0f);
    }
}

// ---------------------------------------------------------------------------
// the filter.  mine_rows_kernel's work items, stages and waits (see there) with integer products: a stage is 128 elements of
// 64 rows, a wave multiplies the tile's 64 labels with its 64 queries (2 x 2 blocks of v_mfma_i32_32x32x32_i8, twice the
// products of the bf16 instruction in the same time).  Bound: the matrix pipe, with what it waits for beside it.  Measured on
// 16 384 queries x 12 M labels x 256 (search, ms): 44.0; without the looks at single scores and the pushes 38.2; also
// without the maxima 38.1, the stage loads 35.5, the stage barriers 35.1, the operand reads 32.6, which leaves the products
// (3.5 POP/s at the chip's power limit) and what goes before them.  A score is looked at on its own only in a group of eight
// whose maximum passes (all 32 of a column in turn: 47.7).  16 384 x 120 M x 256, k = 50: 371 to 389 ms on different
// boxes, of which 15 form the 8-bit rows; 685 to 707 with the bf16 kernel.
// ---------------------------------------------------------------------------
struct Q8Args {
    const unsigned char* Z;          // 8-bit queries [Zq][128 NK]
    const float4* zpar;
    const unsigned char* W;          // 8-bit rows of the chunk, whole tiles
    const float4* tmeta;
    int64_t Zq, n_lab, lab0;         // labels of the chunk, and the first one's id
    int n_items, n_tiles, tiles_per_slice, S, Qx, n_qt;
    int append_max, glist_cap;
    uint32_t* lists;                 // [kMineGrid][kQ8Queries][2][kQ8Cap] labels, offset from the chunk's first
    uint64_t* glist;
    int32_t* gcnt;
    const uint32_t* tau_g;
    int32_t* flag;
    const int32_t* state;            // [0] tiles given up so far, once per chunk; [1] 1: the filter is switched off
};
constexpr size_t kQ8Lds = static_cast<size_t>(kRing) * kQ8Tile * kStageBytes + kQ8MaxTiles * sizeof(float4) +
                          kQ8Queries * 2 * sizeof(int);

template <int NK>
__global__ __launch_bounds__(kMineThreads, 1)
void mine_q8_kernel(const Q8Args a) {
    constexpr int kStage = kQ8Tile * kStageBytes;
    constexpr int row_bytes = NK * kStageBytes;
    constexpr int kLd = 2;                               // load instructions of a wave per stage it brings in
    extern __shared__ __align__(16) unsigned char smem[];
    float4* meta = reinterpret_cast<float4*>(smem + kRing * kStage);
    int* cnt2 = reinterpret_cast<int*>(meta + kQ8MaxTiles);               // [kQ8Queries][2] list fills at the end of a slice
    if (a.state[1] != 0) return;                         // uniform (only the rescoring kernel writes it)
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) unsigned char*)smem));
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);           // which 64 queries of the work item
    const int half = lane >> 5;
    uint32_t* my_lists = a.lists + static_cast<size_t>(blockIdx.x) * kQ8Queries * 2 * kQ8Cap;

    const int xcd = blockIdx.x % kXcds, cu = blockIdx.x / kXcds;
    // (a division runs on the vector unit: back to scalar registers, with everything that follows from it)
    const int slice = __builtin_amdgcn_readfirstlane(xcd + kXcds * (cu / a.Qx));
    if (slice >= a.S) return;
    const int t_begin = slice * a.tiles_per_slice;
    const int t_end = t_begin + a.tiles_per_slice < a.n_tiles ? t_begin + a.tiles_per_slice : a.n_tiles;
    const int n_tiles = t_end - t_begin;
    if (n_tiles <= 0) return;
    const int n_stages = n_tiles * NK;

    const int swz = (lane >> 1) & 7;
    const int frag_a = (lane & 31) * kStageBytes + ((half ^ swz) * 16);
    const int drow = lane >> 3;
    const int wq = wave & 3;
    const int my_parity = wave >> 2;
    const uint32_t dcol[2] = {static_cast<uint32_t>(((lane & 7) ^ (lane >> 4)) * 16),
                              static_cast<uint32_t>(((lane & 7) ^ ((lane >> 4) + 4)) * 16)};
    const uint32_t voff[2] = {static_cast<uint32_t>(drow * row_bytes) + dcol[0],
                              static_cast<uint32_t>((drow + 8) * row_bytes) + dcol[1]};
    const uint32_t dma_dst = lds_base + wq * kLd * 1024;
    for (int i = tid; i < n_tiles; i += kMineThreads) meta[i] = a.tmeta[t_begin + i];

    for (int item = __builtin_amdgcn_readfirstlane(cu % a.Qx); item < a.n_items; item += a.Qx) {
        const int64_t q0 = static_cast<int64_t>(item) * kQ8Queries;
        uint4 zf[NK * 4][2];
        float tu[2], tv[2], tw[2];
        int cnt[2] = {0, 0};
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const int64_t q = q0 + wave * 64 + nt * 32 + (lane & 31);
            const int64_t qc = q < a.Zq ? q : a.Zq - 1;
            const float4 zp = a.zpar[qc];
            const float tau = ordered_to_float(a.tau_g[qc]);
            // Nothing in this chunk can change the result of a query that is not there, whose scores are all NaN, or whose k
            // best so far already hold the largest score it can have (+inf; zero for a zero query: labels of this chunk have
            // larger ids and lose the tie).  Other queries that 8 bits do not describe: everything passes.
            const bool settled = q >= a.Zq || zp.w == kQueryNan || tau == INFINITY || (zp.w == kQueryZero && tau >= 0.0f);
            tu[nt] = settled ? INFINITY : (zp.w != kQueryPlain ? -kQ8Huge : fminf(fmaxf(tau * zp.x, -kQ8Huge), kQ8Huge));
            tv[nt] = zp.y;
            tw[nt] = zp.z;
            const unsigned char* zr = a.Z + qc * row_bytes + half * 16;
#pragma unroll
            for (int ks = 0; ks < NK * 4; ++ks) zf[ks][nt] = *reinterpret_cast<const uint4*>(zr + ks * 32);
        }
        wait_all_vmem();                                 // from here on only stage loads and rare stores are in flight

        int ld_stage = 0, ld_kb = 0;
        uint32_t ld_dst = dma_dst;
        const unsigned char* ld_w = a.W + (static_cast<int64_t>(t_begin) * kQ8Tile + wq * 8 * kLd) * row_bytes;
        auto issue_stage = [&]() {
            if ((ld_stage & 1) == my_parity) {
                const uint64_t b64 = reinterpret_cast<uint64_t>(ld_w + ld_kb * kStageBytes);
                const uint64_t sb =
                    (static_cast<uint64_t>(static_cast<uint32_t>(
                         __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64 >> 32)))) << 32) |
                    static_cast<uint64_t>(static_cast<uint32_t>(
                        __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64))));
                const unsigned char* sp = reinterpret_cast<const unsigned char*>(sb);
                lds_dma16_sbase<0>(sp, voff[0], ld_dst);
                lds_dma16_sbase<1024>(sp, voff[1], ld_dst);
            }
            ++ld_stage;
            ld_dst += kStage;
            if ((ld_stage & (kRing - 1)) == 0) ld_dst = dma_dst;
            if (++ld_kb == NK) { ld_kb = 0; ld_w += kQ8Tile * row_bytes; }
        };
        auto wait_stage = [&](int g) {
            if (ld_stage - 1 - g >= kRing - 2) wait_vmem_at_most<kLd * ((kRing - 2) / 2)>();
            else wait_all_vmem();
        };
        i32x16 acc[2][2][2];                             // [tile parity][mt][nt]
        uint4 fa[2][2];
        auto read_frags = [&](int slot, int kk, int sel) {
            const unsigned char* buf = smem + slot * kStage;
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
                fa[sel][mt] = *reinterpret_cast<const uint4*>(buf + ((frag_a ^ (kk * 32)) + mt * 32 * kStageBytes));
        };
        auto publish = [&](int g_next) {
            wait_stage(g_next);
            lds_barrier();
            if (ld_stage < n_stages) issue_stage();
            read_frags(g_next & (kRing - 1), 0, 0);
        };
        __syncthreads();                                 // the ring and cnt2 are free, meta is there
        for (int s = 0; s < kRing - 1 && s < n_stages; ++s) issue_stage();
        publish(0);

        // the scores of one column block that reach the threshold, looked for eight at a time
        auto push_block = [&](auto parc, auto ntc, int l0, int t) __attribute__((always_inline)) {
            constexpr int par = decltype(parc)::value, nt = decltype(ntc)::value;
            const int lmax = static_cast<int>(a.n_lab);
#pragma unroll
            for (int e0 = 0; e0 < 32; e0 += 8) {
                int m = acc[par][e0 >> 4][nt][e0 & 15];
#pragma unroll
                for (int e = e0 + 1; e < e0 + 8; ++e) { const int v = acc[par][e >> 4][nt][e & 15]; m = v > m ? v : m; }
                if (__builtin_expect(__ballot(m >= t) != 0ull, 0)) {
#pragma unroll
                    for (int e = e0; e < e0 + 8; ++e) {
                        const int i = e & 15;
                        if (__builtin_expect(__ballot(acc[par][e >> 4][nt][i] >= t) != 0ull, 0)) {
                            const uint32_t l = lane_now();
                            const int lab = l0 + 4 * static_cast<int>(l >> 5) + (e >> 4) * 32 + 8 * (i >> 2) + (i & 3);
                            if (acc[par][e >> 4][nt][i] >= t && lab < lmax) {
                                const uint32_t sub = static_cast<uint32_t>((wave * 64 + nt * 32) * 2) + (l & 31u) * 2 + (l >> 5);
                                if (cnt[nt] < kQ8Cap) my_lists[sub * kQ8Cap + static_cast<uint32_t>(cnt[nt])] = static_cast<uint32_t>(lab);
                                ++cnt[nt];               // (beyond the capacity: counted, and the tile given up at the end)
                            }
                        }
                    }
                }
            }
        };

        // The maxima of a tile's scores are taken while the next tile is multiplied, a few per k-step in the shadow of its
        // MFMAs (both waves of a SIMD finish a tile together, so a filter of its own would leave the matrix pipe idle).
        int g = 0;
        int mx[2] = {0, 0};
        int tp[2] = {0x7fffffff, 0x7fffffff}, tc[2];     // thresholds of the tile before and of this one
        constexpr int kSteps = NK * 4, kPart = 32 / kSteps;              // scores of a column looked at per k-step
        auto part_max = [&](auto parc, int ks) __attribute__((always_inline)) {
            constexpr int par = decltype(parc)::value;
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int e = ks * kPart; e < (ks + 1) * kPart; ++e) {
                    const int v = acc[par][e >> 4][nt][e & 15];
                    mx[nt] = e == 0 ? v : (v > mx[nt] ? v : mx[nt]);
                }
            asm volatile("" : "+v"(mx[0]), "+v"(mx[1]));             // here, not collected at the end of the tile
        };
        auto push_tile = [&](auto parc, int tile) __attribute__((always_inline)) {
            if (__builtin_expect(__ballot(mx[0] >= tp[0] || mx[1] >= tp[1]) != 0ull, 0)) {
                const int l0 = (t_begin + tile) * kQ8Tile;
                if (__ballot(mx[0] >= tp[0]) != 0ull) push_block(parc, IC<0>{}, l0, tp[0]);
                if (__ballot(mx[1] >= tp[1]) != 0ull) push_block(parc, IC<1>{}, l0, tp[1]);
                // a list that ran over costs its tile of queries the filter whatever follows: nothing reaches it any more, from the
                // tile after next on (a query that everything passes for held up its whole work item: 16 384 x 8 M x 256, one
                // such query, 72.0 ms against 39.0; with the next tile's threshold changed too, every search took 1 % longer)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    if (cnt[nt] > kQ8Cap) tu[nt] = INFINITY;
            }
        };
        auto do_tile = [&](auto parc, int tile) __attribute__((always_inline)) {
            constexpr int par = decltype(parc)::value;
#pragma unroll
            for (int kb = 0; kb < NK; ++kb) {
                const int slot = g & (kRing - 1);
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    const int sel = kk & 1;
                    if (kk < 3) read_frags(slot, kk + 1, sel ^ 1);
                    else publish(g + 1);
                    if (kb == 0 && kk == 0) {
                        // the integer a label of this tile has to reach: (tau - margins) / (a b), rounded down with room to spare
                        const float4 m = meta[tile];
#pragma unroll
                        for (int nt = 0; nt < 2; ++nt) {
                            const float t = fmaf(tu[nt], m.x, -fmaf(tv[nt], m.y, fmaf(tw[nt], m.z, 2.0f)));
                            tc[nt] = static_cast<int>(fmaxf(fminf(t, 2.0e9f), -2.0e9f));     // (settled, or NaN where the tile is unusable: out of reach as well)
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    part_max(IC<(par ^ 1)>{}, kb * 4 + kk);
#pragma unroll
                    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                        for (int nt = 0; nt < 2; ++nt) {
                            i32x4 av, bv;
                            __builtin_memcpy(&av, &fa[sel][mt], 16);
                            __builtin_memcpy(&bv, &zf[kb * 4 + kk][nt], 16);
                            if (kb == 0 && kk == 0) {
                                const i32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                                acc[par][mt][nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(av, bv, zero, 0, 0, 0);
                            } else {
                                acc[par][mt][nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(av, bv, acc[par][mt][nt], 0, 0, 0);
                            }
                        }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {        // an MFMA, then its share of the maxima
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, kPart / 4 + 1, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                ++g;
            }
            push_tile(IC<(par ^ 1)>{}, tile - 1);
            tp[0] = tc[0];
            tp[1] = tc[1];
        };
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[1][mt][nt][i] = 0;      // "before the first tile": below every threshold
        for (int tile = 0; tile < n_tiles; tile += 2) {
            do_tile(IC<0>{}, tile);
            if (tile + 1 < n_tiles) do_tile(IC<1>{}, tile + 1);
        }
        // the last tile
        if (n_tiles & 1) {
#pragma unroll
            for (int ks = 0; ks < kSteps; ++ks) part_max(IC<0>{}, ks);
            push_tile(IC<0>{}, n_tiles - 1);
        } else {
#pragma unroll
            for (int ks = 0; ks < kSteps; ++ks) part_max(IC<1>{}, ks);
            push_tile(IC<1>{}, n_tiles - 1);
        }

        // ---- close the slice
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) cnt2[(wave * 64 + nt * 32 + (lane & 31)) * 2 + half] = cnt[nt];
        wait_all_vmem();                                 // this wave's list stores have arrived (the lists are read by this workgroup only)
        __syncthreads();
#pragma unroll 1
        for (int qr = 0; qr < kQ8Queries; qr += kMineWaves * 32) {
            const int ql = qr + wave * 32 + (lane & 31);                 // lanes l and l + 32 look after the same query
            const int64_t q = q0 + ql;
            const int c0 = q < a.Zq ? cnt2[ql * 2] : 0, c1 = q < a.Zq ? cnt2[ql * 2 + 1] : 0;
            const int n = c0 + c1;
            const bool over = c0 > kQ8Cap || c1 > kQ8Cap || n > a.append_max;
            if (over && lane < 32) {
                a.flag[0] = 1;
                a.flag[1 + q / kBN] = 1;
            }
            int base = 0;
            if (lane < 32 && n > 0 && !over) base = atomicAdd(&a.gcnt[q], n);
            base = __shfl(base, lane & 31, kWave);
            if (n > 0 && !over) {
                uint64_t* out = a.glist + static_cast<size_t>(q) * a.glist_cap;
                const uint32_t* from = my_lists + static_cast<size_t>(ql) * 2 * kQ8Cap;
                for (int e = half; e < c0; e += 2)
                    if (base + e < a.glist_cap) out[base + e] = from[e] + static_cast<uint64_t>(a.lab0);
                for (int e = half; e < c1; e += 2)
                    if (base + c0 + e < a.glist_cap) out[base + c0 + e] = from[kQ8Cap + e] + static_cast<uint64_t>(a.lab0);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// scores of the labels that passed: entries [gbase, gcnt) of a query's list are labels and become keys.  One wave per
// query; 16 rows at a time as the A operand of the matrix product, the query in all 16 columns of B.  The products are summed
// in the order of mine_rows_kernel, so a row's score has the same bits whichever kernel formed it: equal rows tie wherever
// they lie, and a search from thresholds or without the filter gives the same shortlist.  Bound: HBM, random rows (up to 32
// of a wave in flight).
// ---------------------------------------------------------------------------
template <int NK>
__global__ __launch_bounds__(256)
void q8_rescore_kernel(const unsigned char* __restrict__ Z, const unsigned char* __restrict__ W, int64_t Zq,
                       uint64_t* __restrict__ glist, int glist_cap, int32_t* __restrict__ gcnt,
                       const int32_t* __restrict__ gbase, const uint32_t* __restrict__ tau_g,
                       const int32_t* __restrict__ flag, int n_qt, int item_tiles, int64_t sweep_tiles, int sx_max,
                       int32_t* __restrict__ items, int32_t* __restrict__ state) {
    constexpr int kSteps = 4 * NK, kBlocks = 2, kRow = NK * 256;         // steps of 64 bytes; blocks of 16 rows per round
    const int lane = lane_id();
    if (blockIdx.x == 0 && threadIdx.x < kWave && flag[0] != 0) {
        // the work items that hold a tile given up, and how the search of them splits the labels: with the plan of the whole
        // pool a single item would keep one compute unit per slice busy for as long as all of them take
        int n = 0, tiles = 0;
        for (int i0 = 0; i0 * item_tiles < n_qt; i0 += kWave) {
            const int i = i0 + lane;
            int have = 0;
            for (int t = i * item_tiles; t < (i + 1) * item_tiles && t < n_qt; ++t) have += flag[1 + t] != 0 ? 1 : 0;
            const uint64_t bal = __ballot(have > 0);
            if (have > 0) items[2 + n + __popcll(bal & lanemask_lt())] = i;
            n += __popcll(bal);
            for (int u = 1; u <= item_tiles; ++u) tiles += __popcll(__ballot(have >= u));
        }
        if (lane == 0) {
            const int sx = rows_slices_per_xcd(n, sweep_tiles, sx_max);
            items[0] = n;
            items[1] = sx;
            // The filter costs about six tenths of the bf16 search.  It is not tried again in this search once the tiles that
            // one chunk gives up take more than half of the time that all of them would take without it: n items in
            // ceil(n / (32 / sx)) rounds over slices of 1 / (8 sx) of the labels.
            if (state[1] == 0) {
                const int n_all = (n_qt + item_tiles - 1) / item_tiles, sx_all = rows_slices_per_xcd(n_all, sweep_tiles, sx_max);
                const int qx = kCusPerXcd / sx, qx_all = kCusPerXcd / sx_all;
                state[0] += tiles;
                if (2 * ((n + qx - 1) / qx) * sx_all > ((n_all + qx_all - 1) / qx_all) * sx) state[1] = 1;
            }
        }
    }
    const int64_t q = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (q >= Zq) return;
    const int base = gbase[q];
    if (flag[1 + q / kBN] != 0) {                        // the tile was given up: what other slices appended is dropped
        if (lane == 0) gcnt[q] = base;
        return;
    }
    const int n = gcnt[q];
    if (n == base) return;
    const float tau = ordered_to_float(tau_g[q]);
    uint64_t* list = glist + static_cast<size_t>(q) * glist_cap;
    const int r = lane & 15, g = lane >> 4;              // operands: 16 bytes of row r, chunk 4 s + g in step s
    uint4 z[kSteps];
#pragma unroll
    for (int s = 0; s < kSteps; ++s) z[s] = *reinterpret_cast<const uint4*>(Z + q * kRow + s * 64 + g * 16);
    int out = base;
    for (int e0 = base; e0 < n; e0 += 16 * kBlocks) {
        int32_t id[kBlocks];
        uint4 w[kBlocks][kSteps];
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            const int e = e0 + 16 * b + r;
            id[b] = e < n ? static_cast<int32_t>(list[e]) : 0;           // (past the end: a row that exists, dropped below)
            if (e0 + 16 * b < n)                         // uniform
#pragma unroll
                for (int s = 0; s < kSteps; ++s)
                    w[b][s] = *reinterpret_cast<const uint4*>(W + static_cast<int64_t>(id[b]) * kRow + s * 64 + g * 16);
        }
        // accumulator i: row 4 g + i, in every column.  Lanes with r = 4 b + i, i < 4, take row 4 g + i of block b.
        float mine = 0.0f;
        int32_t my_id = 0;
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            if (e0 + 16 * b < n) {                       // uniform
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < kSteps; ++s) acc = row_mma_bf16(w[b][s], z[s], acc);
                const float v = (r & 2) ? ((r & 1) ? acc[3] : acc[2]) : ((r & 1) ? acc[1] : acc[0]);
                if ((r >> 2) == b) mine = v;
            }
            const int32_t from = __shfl(id[b], 4 * g + (r & 3), kWave);
            if ((r >> 2) == b) my_id = from;
        }
        const bool have = r < 4 * kBlocks && e0 + 16 * (r >> 2) + 4 * g + (r & 3) < n;
        const bool keep = have && mine >= tau;           // (false for NaN)
        const uint64_t bal = __ballot(keep);
        if (keep) list[out + __popcll(bal & lanemask_lt())] = make_key(mine + 0.0f /* -0 -> +0 */, my_id);
        out += __popcll(bal);
    }
    if (lane == 0) gcnt[q] = out;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Which searches take the filter: bf16 rows of 128 or 256 elements (the margins grow with the square root of the row
// length: at 768 elements the threshold sinks by half a standard deviation of the scores, and what then passes costs more
// than the products saved), from 4096 queries on (forming the 8-bit rows costs as much as the products of about 900), and from
// 2^20 labels on (the first 2^17 are searched in bf16).  Measured, bf16 : filter, 1.05 M labels: 256 elements, k = 50, 4096
// queries 2.59 : 2.23 ms, 65 536 35.3 : 27.7; k = 100, 4096 2.94 : 2.67; 128 elements, 4096 1.89 : 1.53; 4 M labels, k = 100,
// 4096 8.2 : 6.2.
bool plan_q8(int64_t Zq, int64_t L, int64_t row_bytes, xc_dtype t, Q8Plan* p) {
    p->nk = 0;
    if (t != XC_BF16 || (row_bytes != 256 && row_bytes != 512)) return false;
    if (Zq < kQ8MinQueries || L < kQ8MinLabels) return false;
    p->nk = static_cast<int>(row_bytes / 256);
    // labels of a chunk: whole label tiles of the bf16 kernel, a slice (an eighth of a chunk at least) within the margins' room in LDS
    int64_t c = kQ8ChunkBytes / (128 * p->nk);
    const int64_t most = static_cast<int64_t>(kXcds) * kQ8MaxTiles * kQ8Tile;
    c = c < most ? c : most;
    const int64_t whole = (L + kBM - 1) / kBM * kBM;
    p->chunk = (c < whole ? c : whole) / kBM * kBM;
    size_t off = 0;
    auto take = [&off](size_t bytes) { const size_t o = off; off += round_up(bytes, 256); return o; };
    p->off_rows = take(static_cast<size_t>(p->chunk) * 128 * p->nk);
    p->off_meta = take(static_cast<size_t>(p->chunk / kQ8Tile) * sizeof(float4));
    p->off_z = take(static_cast<size_t>(Zq) * 128 * p->nk);
    p->off_zpar = take(static_cast<size_t>(Zq) * sizeof(float4));
    p->off_base = take(static_cast<size_t>((Zq + kBN - 1) / kBN * kBN) * sizeof(int32_t));
    p->off_items = take(static_cast<size_t>((Zq + kBN - 1) / kBN + 2) * sizeof(int32_t));
    p->off_flag = take(static_cast<size_t>((Zq + kBN - 1) / kBN + 3) * sizeof(int32_t));
    p->bytes = off;
    return true;
}

int q8_raise_lds() {
    XC_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&mine_q8_kernel<1>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kQ8Lds)));
    XC_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&mine_q8_kernel<2>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kQ8Lds)));
    return XC_OK;
}

int q8_begin(const Q8Plan& p, unsigned char* ws, const void* Z, int64_t Zq, hipStream_t st) {
    const dim3 grid(static_cast<unsigned>((Zq + 3) / 4));
    const unsigned char* z = static_cast<const unsigned char*>(Z);
    float4* zpar = reinterpret_cast<float4*>(ws + p.off_zpar);
    int32_t* state = reinterpret_cast<int32_t*>(ws + p.off_flag);
    if (p.nk == 1) q8_queries_kernel<1><<<grid, 256, 0, st>>>(z, Zq, ws + p.off_z, zpar, state);
    else q8_queries_kernel<2><<<grid, 256, 0, st>>>(z, Zq, ws + p.off_z, zpar, state);
    XC_HIP_CHECK(hipGetLastError());
    return XC_OK;
}

const int32_t* q8_flags(const Q8Plan& p, const unsigned char* ws) { return reinterpret_cast<const int32_t*>(ws + p.off_flag) + 2; }

const int32_t* q8_items(const Q8Plan& p, const unsigned char* ws) { return reinterpret_cast<const int32_t*>(ws + p.off_items); }

template <int NK>
static int q8_chunk_impl(const Q8Plan& p, unsigned char* ws, const Q8Chunk& c, hipStream_t st) {
    const int64_t n_lab = c.lab1 - c.lab0;
    Q8Args a;
    a.Z = ws + p.off_z;
    a.zpar = reinterpret_cast<const float4*>(ws + p.off_zpar);
    a.W = ws + p.off_rows;
    a.tmeta = reinterpret_cast<const float4*>(ws + p.off_meta);
    a.Zq = c.Zq; a.n_lab = n_lab; a.lab0 = c.lab0;
    a.n_items = static_cast<int>((c.Zq + kQ8Queries - 1) / kQ8Queries);
    a.n_tiles = static_cast<int>((n_lab + kQ8Tile - 1) / kQ8Tile);
    a.n_qt = static_cast<int>((c.Zq + kBN - 1) / kBN);
    // one label slice per XCD where there are query items for its 32 compute units, else as many as keep them busy (and
    // as the global lists have room for)
    int sx = 1;
    while (sx < 8 && kXcds * sx * 2 <= c.max_slices && a.n_items * sx < kCusPerXcd) sx <<= 1;
    a.S = kXcds * sx;
    a.Qx = kCusPerXcd / sx;
    a.tiles_per_slice = (a.n_tiles + a.S - 1) / a.S;
    a.append_max = (c.glist_cap - c.kcap) / a.S;
    a.glist_cap = c.glist_cap;
    a.lists = reinterpret_cast<uint32_t*>(c.lists);
    a.glist = c.glist; a.gcnt = c.gcnt; a.tau_g = c.tau_g;
    int32_t* state = reinterpret_cast<int32_t*>(ws + p.off_flag);
    a.state = state;
    a.flag = state + 2;
    int32_t* gbase = reinterpret_cast<int32_t*>(ws + p.off_base);
    const unsigned char* w = static_cast<const unsigned char*>(c.W);
    XC_LAUNCH(K_MINE_TILE, st, (q8_rows_kernel<NK><<<static_cast<unsigned>(a.n_tiles), 256, 0, st>>>(
        w + c.lab0 * 256 * NK, n_lab, ws + p.off_rows, reinterpret_cast<float4*>(ws + p.off_meta), c.gcnt, gbase,
        static_cast<int64_t>(a.n_qt) * kBN, a.flag, a.n_qt, state)));
    XC_HIP_CHECK(hipGetLastError());
    XC_LAUNCH(K_MINE_TILE, st, (mine_q8_kernel<NK><<<kMineGrid, kMineThreads, kQ8Lds, st>>>(a)));
    XC_HIP_CHECK(hipGetLastError());
    XC_LAUNCH(K_MINE_SELECT, st, (q8_rescore_kernel<NK><<<static_cast<unsigned>((c.Zq + 3) / 4), 256, 0, st>>>(
        static_cast<const unsigned char*>(c.Z), w, c.Zq, c.glist, c.glist_cap, c.gcnt, gbase, c.tau_g, a.flag, a.n_qt,
        c.item_tiles, c.sweep_tiles, c.sx_max, reinterpret_cast<int32_t*>(ws + p.off_items), state)));
    XC_HIP_CHECK(hipGetLastError());
    return XC_OK;
}

int q8_chunk(const Q8Plan& p, unsigned char* ws, const Q8Chunk& c, hipStream_t st) {
    return p.nk == 1 ? q8_chunk_impl<1>(p, ws, c, st) : q8_chunk_impl<2>(p, ws, c, st);
}

}  // namespace xc
