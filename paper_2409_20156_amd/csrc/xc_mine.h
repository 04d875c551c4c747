// What the search files share: tile geometry, the direct global->LDS loads, and the two other searches that xc_mine.hip
// calls (few queries: xc_mine_few.hip; the 8-bit filter of long label ranges: xc_mine_q8.hip).
#pragma once

#include <type_traits>

#include "xc_common.h"

namespace xc {

constexpr int kBM = 256;            // labels per tile   (MFMA M)
constexpr int kBN = 256;            // queries per tile  (MFMA N)
constexpr int kStageBytes = 128;    // bytes of a row staged in LDS per K step (= LDS row pitch; the
                                    // 16-byte chunks of a row are stored swizzled, see lds_chunk_swizzle)
constexpr int kCandCap = 1024;      // keys per query candidate list
constexpr int kPool = 320;          // passing scores a wave parks in LDS before it empties them into the lists
constexpr int kPoolCheck = 4;       // accumulators between two looks at the pool's fill (each adds <= 64 entries)
constexpr int kPoolKeep = kPool - kPoolCheck * 64;      // entries a wave may carry from one tile to the next
constexpr int kMineThreads = 512;   // 8 waves: 2 along labels x 4 along queries
constexpr int kMineWaves = kMineThreads / kWave;
static_assert(kPoolKeep >= 0, "the pool holds what can arrive between two looks at its fill");
constexpr int kMineGrid = 256;      // persistent workgroups, one per compute unit
constexpr int kXcds = 8;            // workgroup w runs on XCD w % 8
constexpr int kCusPerXcd = kMineGrid / kXcds;
constexpr int kPhaseGrowth = 8;     // labels of a phase / labels before it
constexpr int kMaxSlices = 64;      // label slices of a phase at most (one lane per slice in the select)
constexpr int kMaxRowKernelBytes = 512;   // longest bf16 rows whose queries the row kernel holds in registers
constexpr int kSelectRegs = 16;     // keys per lane held in registers by the phase select
constexpr uint32_t kTauInit = 0x007fffffu;   // ordered image of -inf

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// One order of sums.  A label's score has the same bits in every search kernel, so that equal rows tie wherever they are
// scored and every route to a shortlist (from scratch, from thresholds, few queries, the filter) gives the same one.  The order
// is that of RowMma: from an accumulator of zero, a row's 16-byte chunks in pairs (lanes 0..31 hold the first of a pair, lanes
// 32..63 the second), each pair one v_mfma_f32_32x32x16_bf16 or four v_mfma_f32_32x32x2_f32.
// The 16x16 instructions give the same bits: v_mfma_f32_16x16x32_bf16 takes two pairs and adds their products as two of the
// former do (21 million random sums of 64 products, with exponents spread over 0 to 40 binary orders, agree bit for bit); both
// fp32 instructions are chains of fused multiply-adds over their elements in lane order (fmaf on as many sums agrees), so
// v_mfma_f32_16x16x4_f32 may take four elements of the order at a time.
template <typename T> struct RowMma;
template <> struct RowMma<bf16_t> {
    static __device__ __forceinline__ void mma(const uint4& a, const uint4& b, f32x16& c) {
        bf16x8 av, bv;
        __builtin_memcpy(&av, &a, 16);
        __builtin_memcpy(&bv, &b, 16);
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, c, 0, 0, 0);
    }
};
template <> struct RowMma<float> {
    static __device__ __forceinline__ void mma(const uint4& a, const uint4& b, f32x16& c) {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    }
};
// fp16 copies of fp32 rows (the filter of xc_mine_half.h, which forms the scores that decide from the fp32 rows)
struct half_t { uint16_t bits; };
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
template <> struct RowMma<half_t> {
    static __device__ __forceinline__ void mma(const uint4& a, const uint4& b, f32x16& c) {
        f16x8 av, bv;
        __builtin_memcpy(&av, &a, 16);
        __builtin_memcpy(&bv, &b, 16);
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, bv, c, 0, 0, 0);
    }
};
__device__ __forceinline__ f32x4 row_mma_bf16(const uint4& a /* 16 rows */, const uint4& b /* 16 columns */, f32x4 c) {
    bf16x8 av, bv;
    __builtin_memcpy(&av, &a, 16);
    __builtin_memcpy(&bv, &b, 16);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, c, 0, 0, 0);
}

// Products in the order of the other search kernels (RowMma and the text above it).  `operand` turns a lane's 16 bytes
// of a row (chunk g of a 64-byte step) into what the matrix instructions of the step take from that lane.
template <typename T> struct FewMma;
template <> struct FewMma<bf16_t> {
    static __device__ __forceinline__ uint4 operand(const uint4& v) { return v; }
    static constexpr int kSteps = 1;             // matrix instructions per step
    static __device__ __forceinline__ f32x4 mma(int, const uint4& a, const uint4& b, f32x4 c) { return row_mma_bf16(a, b, c); }
};
template <> struct FewMma<float> {
    // Lanes g = 0, 1, 2, 3 of a product stand for elements 2i of chunks 0 and 1, then 2i + 1 of them: elements 2i + 1 of
    // the lower chunk pair change places with elements 2i of the upper one.  x, z: the lower pair; y, w: the upper one.
    static __device__ __forceinline__ uint4 operand(const uint4& v) {
        const auto lo = __builtin_amdgcn_permlane32_swap(v.x, v.y, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(v.z, v.w, false, false);
        return make_uint4(lo[0], lo[1], hi[0], hi[1]);
    }
    static constexpr int kSteps = 4;
    static __device__ __forceinline__ f32x4 mma(int t, const uint4& a, const uint4& b, f32x4 c) {
        const uint32_t av = t == 0 ? a.x : t == 1 ? a.z : t == 2 ? a.y : a.w, bv = t == 0 ? b.x : t == 1 ? b.z : t == 2 ? b.y : b.w;
        return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(av), __uint_as_float(bv), c, 0, 0, 0);
    }
};

// kSide blocks of 16 rows (a lane's row of each: wrow) by one query, whose chunks lie in LDS as operands (zop, whole steps of 64 bytes);
// kAhead steps of each are under way at a time.  Accumulator i of a lane: row 4 g + i, in every column r.
template <typename T, int kSide, int kAhead>
__device__ __forceinline__ void score_rows(const unsigned char* const (&wrow)[kSide], const uint4* zop, int row_bytes, int g, f32x4 (&acc)[kSide]) {
    auto product = [&](int u, int s, const uint4& w) {
        const uint4 wo = FewMma<T>::operand(w), zo = zop[4 * s + g];
#pragma unroll
        for (int m = 0; m < FewMma<T>::kSteps; ++m) acc[u] = FewMma<T>::mma(m, wo, zo, acc[u]);
    };
#pragma unroll
    for (int u = 0; u < kSide; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    int s = 0;
    for (; s + kAhead <= row_bytes / 64; s += kAhead) {
        uint4 w[kAhead][kSide];
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
#pragma unroll
            for (int u = 0; u < kSide; ++u) w[i][u] = *reinterpret_cast<const uint4*>(wrow[u] + (s + i) * 64 + g * 16);
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
#pragma unroll
            for (int u = 0; u < kSide; ++u) product(u, s + i, w[i][u]);
    }
    if (s * 64 < row_bytes) {                               // the last steps, of which one may be a part
        uint4 w[kAhead][kSide];
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
#pragma unroll
            for (int u = 0; u < kSide; ++u) {
                w[i][u] = make_uint4(0, 0, 0, 0);
                if ((s + i) * 64 + g * 16 < row_bytes) w[i][u] = *reinterpret_cast<const uint4*>(wrow[u] + (s + i) * 64 + g * 16);
            }
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            if ((s + i) * 64 < row_bytes)                   // uniform
#pragma unroll
                for (int u = 0; u < kSide; ++u) product(u, s + i, w[i][u]);
    }
}

// ---- scores of fp32 rows from fp16 copies (few_half_kernel, xc_mine_half.h)
// Powers of two keep fp16's range out of it: a query is scaled by its own size, W by a scale S that brings the middle one of sixteen rows'
// largest elements to [8, 16).  Elements up to 4000 times that are held, and those below 2^-17 of it lose bits.
constexpr int kHalfSample = 16;
constexpr float kHalfLeast = 1e-15f, kHalfMost = 1e15f;      // largest elements of a query that scaling and norm cover (or all zero)

// |score - 16-bit score| <= half_error |z| |w| + half_error_small / S |z|: two roundings of 2^-11, what fp32 sums of d products lose on both
// sides, a hundredth of that to spare; the second term, 1.05 * 2^-14 sqrt(d), is what elements of W below fp16's normal range can lose.
__device__ __forceinline__ float half_error(int d) { return (2.0f / 2048.0f) * 1.01f + 6.0f * static_cast<float>(d) * 5.97e-8f; }
__device__ __forceinline__ float half_error_small(int d) { return 6.41e-5f * sqrtf(static_cast<float>(d)); }

// Row i of the sample, and the scale from the rows' largest elements (lane i < 16 of the wave: that of row i as bits, 0 if it has none; the
// same in all waves that ask).
__device__ __forceinline__ int64_t half_sample_row(int i, int64_t L) { return (2 * i + 1) * L / (2 * kHalfSample); }
__device__ __forceinline__ uint32_t half_sample_bits(const uint4& v) {       // of four elements; those that are no finite numbers do not count
    uint32_t m = 0;
    const uint32_t u[4] = {v.x & 0x7fffffffu, v.y & 0x7fffffffu, v.z & 0x7fffffffu, v.w & 0x7fffffffu};
#pragma unroll
    for (int i = 0; i < 4; ++i) m = u[i] < 0x7f800000u && u[i] > m ? u[i] : m;
    return m;
}
__device__ __forceinline__ float half_scale(uint32_t bits) {
    const bool have = lane_id() < kHalfSample && bits != 0u;
    int rank = 0;
#pragma unroll
    for (int j = 0; j < kHalfSample; ++j) {
        const uint32_t o = __builtin_amdgcn_readlane(bits, j);
        rank += o != 0u && (o < bits || (o == bits && j < lane_id())) ? 1 : 0;
    }
    const int n = __popcll(__ballot(have));
    const uint64_t middle = __ballot(have && rank == n / 2);
    if (middle == 0ull) return 64.0f;                // nothing but zeros
    int e = 3 - (static_cast<int>(__builtin_amdgcn_readlane(bits, __ffsll(static_cast<long long>(middle)) - 1) >> 23) - 127);
    e = e < -47 ? -47 : e > 53 ? 53 : e;
    return __uint_as_float(static_cast<uint32_t>(e + 127) << 23);
}

// The errors of the tiles' scores from fp16 copies: range holds the bits of the largest and of the smallest that is not zero (of any wave's share
// of a tile).  Within four of each other the largest stands for all: returned.  Else -1: each tile has its own.
__device__ __forceinline__ float half_error_of_all(const uint32_t* range) {
    const float most = __uint_as_float(range[0]), least = __uint_as_float(range[1]);
    return most <= 4.0f * least ? most : -1.0f;
}

// p[i], the same for the whole wave and written before this launch, by a scalar load that is awaited here (a vector load's wait would be one
// for every stage load under way).
__device__ __forceinline__ float uniform_load(const float* p, int64_t i) {
    typedef const __attribute__((address_space(4))) uint32_t* const_ptr;
    const uint64_t at = reinterpret_cast<uint64_t>(p + i);
    const uint64_t u = (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(at >> 32)))) << 32) |
                       static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(at))));
    uint32_t v = *reinterpret_cast<const_ptr>(u);
    v = __builtin_amdgcn_readfirstlane(v);
    asm volatile("" : "+s"(v));
    return __uint_as_float(v);
}

constexpr int kRing = 8;            // stages in LDS (8 or 16 KiB each)
static_assert(kRing >= 4 && (kRing & (kRing - 1)) == 0, "stage slots are indexed modulo a power of two, and the two halves of the workgroup fill them in turn");

__device__ __forceinline__ void lds_dma16(const void* gptr, uint32_t lds_addr /* wave-uniform */) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(gptr), "s"(lds_addr) : "memory");
}
// The same with a wave-uniform 64-bit base and a 32-bit lane offset: no vector arithmetic is needed
// to form the address, so issuing the load never competes with another wave's MFMAs for the VALU.
template <int V> using IC = std::integral_constant<int, V>;

template <int kLdsOffset>
__device__ __forceinline__ void lds_dma16_sbase(const void* sbase /* wave-uniform */, uint32_t voff,
                                                uint32_t lds_addr /* wave-uniform; kLdsOffset is added */) {
    asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr), "n"(kLdsOffset) : "memory", "scc");
}
__device__ __forceinline__ void wait_all_vmem() {
    __builtin_amdgcn_s_waitcnt(0x0070 | 0x0f00);      // vmcnt(0); expcnt and lgkmcnt untouched
}

// The lane number, computed where it is asked for (the compiler can neither hoist nor keep it).
__device__ __forceinline__ uint32_t lane_now() {
    uint32_t l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

template <int N>
__device__ __forceinline__ void wait_vmem_at_most() {   // until at most N vector memory operations are outstanding
    __builtin_amdgcn_s_waitcnt((N & 0xf) | ((N >> 4) << 14) | 0x0070 | 0x0f00);
}

// Stage fill of the last, ragged label tile: per-lane addresses, rows past the end repeat the last row.
__device__ __noinline__ void issue_stage_ragged(const unsigned char* W, int64_t L, int64_t row, int row_bytes, int kbyte,
                                                uint32_t dcol0, uint32_t dcol1, uint32_t dst, int n_instr) {
#pragma unroll 1
    for (int t = 0; t < n_instr; ++t) {
        int64_t r = row + 8 * t;
        r = r < L ? r : L - 1;
        lds_dma16(W + r * row_bytes + kbyte + ((t & 1) ? dcol1 : dcol0), __builtin_amdgcn_readfirstlane(dst + t * 1024));
    }
}

// Slices per XCD for the kernel that keeps the query tile in registers.  The compute units of an XCD
// that work on one slice read the same stream of W tiles, a few tiles apart, so all but the first find
// them in that XCD's L2: the fewer slices per XCD, the fewer times W comes from memory (with 8 slices
// per XCD the search of 16 384 queries over 120 M rows of 512 bytes ran at the rate the memory system
// delivered W, with one slice 19 % faster).  The other side: 32 / slices query tiles are in flight per
// XCD, and compute units without a query tile idle.  Among the counts the phase allows (<= sx_max) take
// the one that keeps the most compute units busy, and of those the smallest.
// Opening and closing an item (operands, the ring, the lists) costs about what eight tiles of a slice do, so that short
// slices are not worth a slightly fuller last round (60 items of 256 queries over 803 tiles: 2 rounds of 100 tiles are 94 %
// full, 15 rounds of 13 tiles are 100 % full and took 1.8 times as long; 205 654 x 256, 50 000 queries 13.5 -> 7.6 ms from
// scratch, 7.4 -> 5.4 from thresholds; 2 M x 128, 30 000 queries 23.3 -> 13.7).
__host__ __device__ inline int rows_slices_per_xcd(int64_t nQT, int64_t n_tiles, int sx_max) {
    int best = sx_max;
    double best_eff = -1.0;
    for (int sx = 1; sx <= sx_max; sx <<= 1) {
        const int qx = kCusPerXcd / sx;
        const int64_t rounds = (nQT + qx - 1) / qx;
        const double per = static_cast<double>(n_tiles) / (kXcds * sx);
        const double eff = static_cast<double>(nQT) / static_cast<double>(rounds * qx) * per / (per + 8.0);
        if (eff > best_eff + 1e-9) { best_eff = eff; best = sx; }
    }
    return best;
}

struct FewPlan {
    int ks;                  // 64-byte steps of a row
    int nb;                  // blocks of 16 queries per workgroup
    int n_qb;                // groups of nb blocks
    int gshift;              // labels of a group: 16 << gshift
    int64_t n_groups;
    int n_split;             // workgroups per query in the second kernel
    size_t lds;              // bytes of the query block in LDS
    bool lines;              // W read by whole lines, with a stage per wave beside the query block: line_lds bytes
    size_t line_lds;
    // fp32 with group maxima from 16-bit products (hnb 0: not used)
    int hnb, hn_qb, hks, hgshift;
    int64_t hn_groups;
    size_t hlds;
};

// Whether the search of few queries takes this shape, and how.  `scratch`: bytes for the group maxima
// and the candidates of shared queries.
// `half`: the search of many queries on fp16 copies (xc_mine_half.h) is the alternative.
bool plan_few(int64_t Zq, int64_t L, int64_t row_bytes, int k, xc_dtype t, bool warm, bool half, size_t scratch, FewPlan* p);

constexpr int kRedoWord = 32;        // redo_any among the words of the search's flags (the tiles of so few queries take nine)
int few_raise_lds();         // the dynamic LDS limit of its kernels, on the current device
int run_mine_few(const FewPlan& p, const void* Z, const void* W, int64_t Zq, int64_t L, int64_t row_bytes, int k,
                 xc_dtype t, unsigned char* scratch, uint32_t* tau_g, int32_t* flag /* null: leave alone */, int n_flag,
                 int32_t* redo_any /* 1 afterwards if 16-bit maxima left a query to the fp32 kernels, 0 if none */, int32_t* shortlist, float* scores, hipStream_t st);

// ---- the 8-bit filter (xc_mine_q8.hip)
constexpr int64_t kQ8MinQueries = 4096, kQ8MinLabels = 1 << 20;
constexpr int64_t kQ8ChunkBytes = 512ll << 20;       // 8-bit rows held at a time
constexpr int64_t kQ8FirstTile = 512;                // label tiles that the bf16 phases cover first (a threshold to filter with)
constexpr int kQ8Growth = 3;                         // labels of a chunk / labels before it, at most

struct Q8Plan {
    int nk;                                          // row bytes / 256; 0 = not used
    int64_t chunk;                                   // labels at a time
    size_t off_rows, off_meta, off_z, off_zpar, off_base, off_items, off_flag, bytes;      // within its part of the workspace
};
struct Q8Chunk {
    const void *Z, *W;
    int64_t Zq, lab0, lab1;
    int kcap, glist_cap, max_slices;
    uint64_t *lists, *glist;
    int32_t* gcnt;
    const uint32_t* tau_g;
    int item_tiles;                                  // the caller's own search of the range: query tiles per work item,
    int64_t sweep_tiles;                             // label tiles
    int sx_max;                                      // and slices per XCD at most
};

bool plan_q8(int64_t Zq, int64_t L, int64_t row_bytes, xc_dtype t, Q8Plan* p);
int q8_raise_lds();
int q8_begin(const Q8Plan& p, unsigned char* ws, const void* Z, int64_t Zq, hipStream_t st);
// Filters labels [lab0, lab1) and appends the keys of those that reach the thresholds to the queries' global lists, except
// for query tiles qt whose flag q8_flags()[1 + qt] is set afterwards (then [0] is too): for these the caller searches the range itself.
int q8_chunk(const Q8Plan& p, unsigned char* ws, const Q8Chunk& c, hipStream_t st);
const int32_t* q8_flags(const Q8Plan& p, const unsigned char* ws);
const int32_t* q8_items(const Q8Plan& p, const unsigned char* ws);       // the work items of that search, see MineArgs::items

}  // namespace xc
