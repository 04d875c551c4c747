// Hard-negative mining: exact top-k inner product of every query against all
// classifier rows (Alg. 1, "ANNS refresh" step, with exact search in place of
// the index; score of Sec. 2.1).
//
// The labels are swept in phases of geometrically growing size (256 labels,
// then 8x more each time).  Within a phase every query has a FIXED threshold
// tau: the exact k-th best score over all labels of the earlier phases, so the
// k best labels overall are never below it and only about 8k scores per query
// pass it.
//   mine_tile_kernel    persistent tiled MFMA product W_tile x Z_tile^T (256
//       labels x 256 queries per workgroup, 8 waves of 128 x 64), K staged 64
//       elements at a time through two LDS buffers that are filled by direct
//       global->LDS loads one stage ahead.  Labels run along the MFMA M axis
//       and queries along N, so one lane owns one query column and compares its
//       accumulators with that query's tau; the score matrix never leaves
//       registers.  Passing scores are parked in a per-wave pool in LDS (slot
//       from a ballot, no atomic on the path) that lives as long as the label
//       slice; the pool is emptied into a 1024-key list per query when it
//       fills, and the lists are appended to the queries' global candidate
//       lists when the workgroup finishes its slice.  The filter of a tile
//       needs no barrier: the workgroup meets only after a tile in which a
//       pool was emptied, to cut any list that could overflow to its best k
//       (radix select by one wave; tau rises locally).
//   mine_select_kernel  after each phase, one wave per query cuts the global
//       candidate list to its best k and publishes the new tau; after the last
//       phase it sorts the winners by (score descending, id ascending).
#include <cmath>
#include <cstdlib>
#include <mutex>
#include <type_traits>

#include "xc_common.h"
#include "xc_mine.h"

namespace xc {

// ---------------------------------------------------------------------------
// Reduce a candidate list of n > k keys to its k smallest keys (best scores).
// One wave; n <= 64*R keys, fetched by load(index) and held in registers.  Radix select, most significant byte first, with a
// 256-bin histogram in LDS; stops as soon as every key sharing the prefix is
// needed.  Writes the survivors to buf[0..k), returns the score of the k-th.
// ---------------------------------------------------------------------------
template <int R, typename Load>
__device__ __noinline__ float wave_select_k(uint64_t* __restrict__ buf, Load load, int n, int k, int* hist) {
    const int lane = lane_id();
    uint64_t key[R];
    bool valid[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int idx = r * kWave + lane;
        valid[r] = idx < n;
        key[r] = valid[r] ? load(idx) : kKeySentinel;
    }
    // leading bytes shared by every key (scores of one query lie close together) need no pass:
    // all keys would fall into one histogram bin, one atomic after the other
    uint64_t diff = 0;
    const uint64_t ref = __shfl(key[0], 0, kWave);          // index 0 is valid (n > k >= 1)
#pragma unroll
    for (int r = 0; r < R; ++r) diff |= valid[r] ? (key[r] ^ ref) : 0ull;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) diff |= __shfl_xor(diff, off, kWave);
    const int first_pass = diff == 0ull ? 8 : (__clzll(static_cast<long long>(diff)) >> 3);
    uint64_t pmask = first_pass == 0 ? 0ull : (~0ull << (64 - 8 * first_pass));
    uint64_t prefix = ref & pmask;
    int need = k;
    for (int pass = first_pass; pass < 8; ++pass) {
        const int shift = 56 - 8 * pass;
#pragma unroll
        for (int j = 0; j < 4; ++j) hist[lane * 4 + j] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (valid[r] && (key[r] & pmask) == prefix)
                atomicAdd(&hist[static_cast<int>((key[r] >> shift) & 255u)], 1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        int c[4];
        int s = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) { c[j] = hist[lane * 4 + j]; s += c[j]; }
        const int incl = wave_incl_scan(s);
        const int excl = incl - s;
        const bool mine = (excl < need) && (need <= incl);
        int dsel = 0, needn = 0, have = 0;
        if (mine) {
            int cum = excl;
            bool done = false;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!done && need <= cum + c[j]) {
                    dsel = lane * 4 + j; needn = need - cum; have = c[j]; done = true;
                }
                cum += c[j];
            }
        }
        const uint64_t bal = __ballot(mine);
        const int src = __ffsll(static_cast<long long>(bal)) - 1;   // exactly one lane
        dsel = __shfl(dsel, src, kWave);
        needn = __shfl(needn, src, kWave);
        have = __shfl(have, src, kWave);
        prefix |= static_cast<uint64_t>(dsel) << shift;
        pmask |= 0xffull << shift;
        need = needn;
        if (have == need) break;
    }
    const uint64_t bound = prefix | ~pmask;
    uint64_t kmax = 0;
    int base = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool sel = valid[r] && key[r] <= bound;
        const uint64_t m = __ballot(sel);
        const int p = base + __popcll(m & lanemask_lt());
        if (sel && p < k) {
            buf[p] = key[r];
            kmax = key[r] > kmax ? key[r] : kmax;
        }
        base += __popcll(m);
    }
    kmax = wave_max_u64(kmax);
    return key_score(kmax);
}

struct MineArgs {
    const unsigned char* Z;
    const unsigned char* W;
    int64_t Zq, L, row_bytes;
    int64_t z_rows, w_rows;  // rows that can be read (copies made for a search are padded to whole tiles)
    int k, kcap;
    int nkb;                 // K stages per tile
    int64_t nQT;             // query tiles
    int64_t tile_lo, tile_hi;   // label tiles of this phase
    int64_t tiles_per_slice;
    int S;                   // label slices of the phase
    int Qx;                  // > 0: query tiles in flight per XCD (slices bound to XCDs);
                             // 0: plain order, item = qtile * S + slice
    int append_max;          // keys one slice may append per query (>= kcap)
    int glist_cap;           // keys per query in the global candidate lists
    uint64_t* lists;         // [kMineGrid][kBN][kCandCap] per-workgroup lists
    uint64_t* glist;         // [nQT*kBN][glist_cap] per-query candidates across slices and phases
    int32_t* gcnt;           // [nQT*kBN] fill of glist
    const uint32_t* tau_g;   // [nQT*kBN] ordered image of the phase threshold
    const unsigned char* zeros;   // 256 zero bytes (source of the chunks past the end of a row)
    float* dense;            // first phase, all scores of its tiles: [nQT*kBN][dense_ld]
    int dense_ld;
    const int32_t* cond;     // not null: repeat of a warm search; cond[0] != 0 if any query tile needs it,
                             // cond[1 + qt] != 0 if query tile qt does
    // fp16 copies: tau_g holds scores that k labels are known to reach; a label passes if its 16-bit score is below by no more than its error
    const float* tile_err;   // [label tile] the error, for every query
    const uint32_t* err_range;   // the errors' range, see half_error_of_all
    int32_t* over;           // [0] and [1 + qt] are set when query tile qt is given up (a list ran over)
    const int32_t* skip;     // [qt]: given up before this launch
    const int32_t* items;    // not null (row kernel): only these work items, [0] their number, [1] slices per XCD, [2..] the items
};

// ---------------------------------------------------------------------------
// LDS staging.  One K stage is 512 rows (256 of W, then 256 of Z) x 128 bytes, row pitch 128.
// Chunk c (16 bytes) of row r is stored at chunk position c ^ ((r >> 1) & 7): the 16 lanes
// that read the same chunk of 16 consecutive rows for an MFMA operand then hit 16 different
// 16-byte bank groups.  The stage is filled by direct global->LDS loads: lane i of a wave
// instruction writes bytes [16 i, 16 i + 16) of a 1 KiB block (8 rows), so the swizzle is
// applied to the SOURCE address of each lane.  The loads are written as inline assembly so
// that the compiler does not serialise later LDS reads behind them; they are awaited with an
// explicit vmcnt wait followed by a workgroup barrier.
// ---------------------------------------------------------------------------
// Stage fill of a ragged tile (rows past the end repeat the last row) or of rows whose length is
// not a multiple of the stage (chunks past the end come from the zero block): lane addresses are
// formed one by one.  Kept out of line so that its registers do not burden the main loop.
template <bool KTAIL>
__device__ __noinline__ void issue_stage_slow(const unsigned char* base, int64_t last_row, int64_t row_bytes,
                                              uint32_t kb, int drow, uint32_t dcol0, uint32_t dcol1,
                                              uint32_t dst, const unsigned char* zeros) {
#pragma unroll 1
    for (int t = 0; t < 16; ++t) {
        const int64_t r = drow + 8 * t;
        const uint32_t dc = (t & 1) ? dcol1 : dcol0;
        const unsigned char* g = base + ((r < last_row ? r : last_row) * row_bytes + dc + kb);
        if (KTAIL && kb + dc >= static_cast<uint32_t>(row_bytes)) g = zeros;
        lds_dma16(g, __builtin_amdgcn_readfirstlane(dst + t * 1024));
    }
}

// The nth of the n tiles whose flag is set; their number if there are fewer.  By whole waves.
__device__ __forceinline__ int flagged_tiles(const int32_t* flag, int64_t n, int nth) {
    int seen = 0;
    for (int64_t i0 = 0; i0 < n; i0 += kWave) {
        uint64_t bal = __ballot(i0 + lane_id() < n && flag[i0 + lane_id()] != 0);
        const int c = __popcll(bal);
        if (nth < seen + c) {
            for (int j = seen; j < nth; ++j) bal &= bal - 1;
            return __builtin_amdgcn_readfirstlane(static_cast<int>(i0) + __ffsll(static_cast<long long>(bal)) - 1);
        }
        seen += c;
    }
    return seen;
}

// DENSE: the first phase, where no threshold exists yet: a work item is one tile, and all its scores are written.
template <typename T, bool KTAIL, bool DENSE>
__global__ __launch_bounds__(kMineThreads, 1)
void mine_tile_kernel(const MineArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (a.cond != nullptr && a.cond[0] == 0) return;          // uniform: a repeat that is not needed
    // two stage buffers, each: W rows then Z rows
    constexpr int kStageBuf = (kBM + kBN) * kStageBytes;
    float* tau = reinterpret_cast<float*>(smem + 2 * kStageBuf);
    int* cnt = reinterpret_cast<int*>(tau + kBN);
    int* hist = cnt + kBN;                                   // [kMineWaves][256]
    constexpr bool kHalf = std::is_same<T, half_t>::value;
    uint2* pools = reinterpret_cast<uint2*>(hist + kMineWaves * 256);       // [kMineWaves][kPool]
    int* dirty = reinterpret_cast<int*>(pools + kMineWaves * kPool);        // [2], by tile parity
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) unsigned char*)smem));

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1;          // which 128-label half
    const int wn = wave >> 1;         // which 64-query quarter
    uint64_t* my_lists = a.lists + static_cast<size_t>(blockIdx.x) * kBN * kCandCap;

    // ---- which (query tile, label slice) items this workgroup processes
    int item, item_step, item_end;     // (nQT * S fits: at most 2^23 query tiles, 64 slices)
    int slice_fixed = -1;
    if (a.Qx > 0) {                   // slices bound to XCDs: workgroup w runs on XCD w % 8
        const int xcd = blockIdx.x % kXcds;
        const int cu = blockIdx.x / kXcds;
        slice_fixed = xcd + kXcds * (cu / a.Qx);
        item = cu % a.Qx; item_step = a.Qx; item_end = static_cast<int>(a.nQT);        // items are query tiles
        if (slice_fixed >= a.S) item_end = 0;
    } else {
        item = blockIdx.x; item_step = kMineGrid; item_end = static_cast<int>(a.nQT * a.S);
    }

    // ---- fragment reads: lane reads row (lane & 31) of a 32-row block, chunk 2 kk + (lane >> 5);
    // the swizzle term of those rows is (lane >> 1) & 7, and the k-step enters as an xor of 32 kk
    const int swz = (lane >> 1) & 7;
    const int frag_a = (wm * 128 + (lane & 31)) * kStageBytes + (((lane >> 5) ^ swz) * 16);
    const int frag_b = (kBM + wn * 64 + (lane & 31)) * kStageBytes + (((lane >> 5) ^ swz) * 16);

    // ---- stage fill.  A stage is brought in by four waves, one per SIMD, while their SIMD-mates
    // (waves w and w + 4 share a SIMD) start on the MFMAs at once; the two halves of the workgroup
    // take turns from stage to stage.  The issuing waves wait in the texture unit's queue, not in
    // front of the matrix pipe.  Wave w (and w + 4) owns 128 rows: W rows 0..127 / 128..255 for
    // w & 3 = 0 / 1, Z rows likewise for 2 / 3; instruction t covers rows 8 t .. 8 t + 7 of them,
    // lane i -> row i / 8, position i % 8.  The chunk a lane fetches is position ^ swizzle(row),
    // which depends on t only through t & 1.
    const bool dma_z = (wave & 3) >= 2;
    const int drow = (wave & 1) * 128 + (lane >> 3);
    const uint32_t dcol[2] = {static_cast<uint32_t>(((lane & 7) ^ (lane >> 4)) * 16),
                              static_cast<uint32_t>(((lane & 7) ^ ((lane >> 4) + 4)) * 16)};
    const uint32_t dma_dst = lds_base + (dma_z ? kBM * kStageBytes : 0) + (wave & 1) * 128 * kStageBytes;
    const uint32_t voff[2] = {static_cast<uint32_t>(drow * a.row_bytes) + dcol[0],
                              static_cast<uint32_t>((drow + 8) * a.row_bytes) + dcol[1]};

    // a repeat in fp32: the items are those of the tiles that need it, so that a few of them keep as many compute units busy as they can
    constexpr bool kListed = std::is_same<T, float>::value;
    if (kListed && a.cond != nullptr) {
        const int n = flagged_tiles(a.cond + 1, a.nQT, 0x7fffffff);
        item_end = item_end == 0 ? 0 : a.Qx > 0 ? n : n * a.S;
    }

    for (; item < item_end; item += item_step) {
        int64_t qtile = a.Qx > 0 ? item : item / a.S;
        if (kListed && a.cond != nullptr) qtile = flagged_tiles(a.cond + 1, a.nQT, static_cast<int>(qtile));
        if (!kListed && a.cond != nullptr && a.cond[1 + qtile] == 0) continue;     // uniform: this query tile came out complete
        if (kHalf && !DENSE && a.skip[qtile] != 0) continue;           // uniform
        const int slice = a.Qx > 0 ? slice_fixed : static_cast<int>(item % a.S);
        const int64_t t_begin = a.tile_lo + static_cast<int64_t>(slice) * a.tiles_per_slice;
        // tiles of the slice are counted from t_begin in 32 bits (a slice has at most 2^31 / 256 / 8 tiles)
        int n_tiles;
        {
            int64_t t_end = t_begin + a.tiles_per_slice;
            t_end = t_end < a.tile_hi ? t_end : a.tile_hi;
            if (t_end <= t_begin) continue;                  // uniform: an empty slice
            n_tiles = static_cast<int>(t_end - t_begin);
        }
        // tiles [0, full_tiles) of the slice have all kBM rows
        int full_tiles;
        {
            const int64_t f = a.w_rows / kBM - t_begin;
            full_tiles = f < 0 ? 0 : (f < n_tiles ? static_cast<int>(f) : n_tiles);
        }
        const int64_t q0 = qtile * kBN;
        if (tid < kBN) { tau[tid] = ordered_to_float(a.tau_g[q0 + tid]); cnt[tid] = 0; }
        if (tid < 2) dirty[tid] = 0;

        // ---- the load stream runs one stage ahead of the compute stream and stops at the last stage
        const unsigned char* zbase = a.Z + q0 * a.row_bytes;
        const unsigned char* wld = a.W + t_begin * kBM * a.row_bytes;       // W rows of the tile being loaded
        const bool z_full = a.z_rows - q0 >= kBN;
        int ld_tile = 0;
        int ld_kb = 0, ld_slot = 0;
        int to_issue = n_tiles * a.nkb;
        auto issue_stage = [&]() {
            const bool full = dma_z ? z_full : ld_tile < full_tiles;
            const unsigned char* base = dma_z ? zbase : wld;
            const uint32_t kb = static_cast<uint32_t>(ld_kb) * kStageBytes;
            const uint32_t dst = dma_dst + static_cast<uint32_t>(ld_slot) * kStageBuf;
            if ((wave < 4) == (ld_slot == 0)) {              // this half's turn
                if (!KTAIL && full) {
                    // the usual case: every row of the tile exists.  Lane offsets voff[t & 1] are the
                    // same for all stages; everything else is added to the scalar base.
                    const uint64_t b64 = reinterpret_cast<uint64_t>(base + kb);     // wave-uniform
                    // (readfirstlane returns a signed int: widen each half as unsigned)
                    const uint64_t sb =
                        (static_cast<uint64_t>(static_cast<uint32_t>(
                             __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64 >> 32)))) << 32) |
                        static_cast<uint64_t>(static_cast<uint32_t>(
                            __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64))));
                    const uint64_t pair_step = 16u * static_cast<uint64_t>(a.row_bytes);     // 16 rows per two instructions
                    auto pair = [&](auto tc) {
                        constexpr int t = decltype(tc)::value;
                        const unsigned char* sp = reinterpret_cast<const unsigned char*>(sb + (t >> 1) * pair_step);
                        lds_dma16_sbase<t * 1024>(sp, voff[0], dst);
                        lds_dma16_sbase<(t + 1) * 1024>(sp, voff[1], dst);
                    };
                    pair(std::integral_constant<int, 0>{});  pair(std::integral_constant<int, 2>{});
                    pair(std::integral_constant<int, 4>{});  pair(std::integral_constant<int, 6>{});
                    pair(std::integral_constant<int, 8>{});  pair(std::integral_constant<int, 10>{});
                    pair(std::integral_constant<int, 12>{}); pair(std::integral_constant<int, 14>{});
                } else {
                    const int64_t last_row = dma_z ? a.z_rows - 1 - q0 : a.w_rows - 1 - (t_begin + ld_tile) * kBM;
                    issue_stage_slow<KTAIL>(base, last_row, a.row_bytes, kb, drow, dcol[0], dcol[1], dst, a.zeros);
                }
            }
            ld_slot ^= 1;
            --to_issue;
            if (++ld_kb == a.nkb) { ld_kb = 0; ++ld_tile; wld += kBM * a.row_bytes; }
        };

        f32x16 acc[4][2];            // (never cleared: the first k-step of a tile multiplies into zeros, see below)

        // ---- main loop.  At the top of a stage its data is visible in LDS, the next stage's loads
        // have been issued into the other buffer, and the fragments of its first k-step are already
        // in registers.  The barrier that publishes the next stage sits before the last k-step's
        // MFMAs, so the first fragment reads of the next stage (and the loads of the stage after it)
        // are under way while those MFMAs run.
        uint4 fa[2][4], fb[2][2];
        auto read_frags = [&](const unsigned char* buf, int kk, int sel) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                fa[sel][mt] = *reinterpret_cast<const uint4*>(buf + ((frag_a ^ (kk * 32)) + mt * 32 * kStageBytes));
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                fb[sel][nt] = *reinterpret_cast<const uint4*>(buf + ((frag_b ^ (kk * 32)) + nt * 32 * kStageBytes));
        };
        auto products = [&](int sel) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    RowMma<T>::mma(fa[sel][mt], fb[sel][nt], acc[mt][nt]);
        };
        // the first k-step of a tile: the accumulators start from a zero operand instead of being cleared
        // one register at a time after the filter (128 vector moves per tile and wave)
        auto products_first = [&](int sel) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    f32x16 c = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    RowMma<T>::mma(fa[sel][mt], fb[sel][nt], c);
                    acc[mt][nt] = c;
                }
        };
        int buf_sel = 0;
        auto publish_next = [&](const unsigned char* next_buf) {
            wait_all_vmem();                                 // this wave's part of the next stage has landed
            __syncthreads();                                 // everyone's has; the current buffer is free
            if (to_issue > 0) issue_stage();                 // the stage after it, into the current buffer
            read_frags(next_buf, 0, 0);
        };

        __syncthreads();                                     // tau/cnt visible; both stage buffers free
        issue_stage();
        publish_next(smem);                                  // stage 0 visible, stage 1 under way

        // ---- a passing score is first parked, with its query and label offset, in this wave's pool:
        // the slot comes from a ballot and a wave-uniform fill count, so nothing waits on an atomic.
        // The pool is emptied into the per-query lists (slots from LDS counters) when it fills up, at
        // the end of a tile if it holds more than kPoolKeep entries, and at the end of the slice.
        // No barrier is needed for any of that; what does need the whole workgroup - cutting a list
        // that could overflow, closing the slice - is done at the start of the next tile's filter,
        // when a flag says that lists have grown.
        uint2* pool = pools + wave * kPool;
        int fill = 0;
        int pool_tile = 0;                                   // labels in the pool count from this tile
        const float err_all = kHalf && !DENSE ? half_error_of_all(a.err_range) : 0.0f;
        auto flush = [&]() {
            const int64_t l0 = (t_begin + pool_tile) * kBM;
#pragma unroll 1
            for (int e0 = 0; e0 < fill; e0 += 2 * kWave) {   // two batches of 64 at a time: the slot atomics overlap
                uint2 en[2];
                int slot[2];
                bool ok[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int e = e0 + u * kWave + lane;
                    ok[u] = e < fill;
                    en[u] = ok[u] ? pool[e] : make_uint2(0u, 0u);
                    ok[u] = ok[u] && (l0 + (en[u].y & 0xffffffu) < a.L);   // rows past the end repeat the last row
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) slot[u] = ok[u] ? atomicAdd(&cnt[en[u].y >> 24], 1) : 0;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (ok[u])
                        my_lists[static_cast<size_t>(en[u].y >> 24) * kCandCap + slot[u]] =
                            make_key(__uint_as_float(en[u].x) + 0.0f /* -0 -> +0 */,
                                     static_cast<int32_t>(l0 + (en[u].y & 0xffffffu)));
                }
            }
            fill = 0;
        };

        for (int tile = 0; tile < n_tiles; ++tile) {          // counted from t_begin
            const int par = tile & 1;
            for (int kb = 0; kb < a.nkb; ++kb) {
                const unsigned char* cur = smem + buf_sel * kStageBuf;
                const unsigned char* nxt = smem + (buf_sel ^ 1) * kStageBuf;
                buf_sel ^= 1;
                read_frags(cur, 1, 1);
                __builtin_amdgcn_sched_barrier(0);
                if (kb == 0) products_first(0); else products(0);
                __builtin_amdgcn_sched_barrier(0);
                read_frags(cur, 2, 0);
                __builtin_amdgcn_sched_barrier(0);
                products(1);
                __builtin_amdgcn_sched_barrier(0);
                read_frags(cur, 3, 1);
                __builtin_amdgcn_sched_barrier(0);
                products(0);
                __builtin_amdgcn_sched_barrier(0);
                // the next stage - of this tile or of the next one - is published before the last products
                if (kb + 1 < a.nkb || tile + 1 < n_tiles) publish_next(nxt);
                __builtin_amdgcn_sched_barrier(0);
                products(1);
                __builtin_amdgcn_sched_barrier(0);
            }


            if constexpr (DENSE) {
                // accumulators 4 j .. 4 j + 3 of a block are four labels in a row of the lane's query
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    const int64_t q = q0 + wn * 64 + nt * 32 + (lane & 31);
                    float* out = a.dense + q * a.dense_ld + static_cast<int>(t_begin - a.tile_lo + tile) * kBM + wm * 128 + 4 * (lane >> 5);
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            *reinterpret_cast<float4*>(out + mt * 32 + 8 * j) =
                                make_float4(acc[mt][nt][4 * j], acc[mt][nt][4 * j + 1], acc[mt][nt][4 * j + 2], acc[mt][nt][4 * j + 3]);
                }
                continue;
            }

            // ---- threshold filter: lane owns query column (lane & 31) of each N tile
            const bool last = tile + 1 == n_tiles;
            float err = err_all;
            if (kHalf && err_all < 0.0f) {                   // uniform
                err = uniform_load(a.tile_err, t_begin + tile);
            }
            // The flag this tile may set shares its slot with the flag of two tiles back, which the waves
            // read after the previous tile's filter: a barrier has to lie between that read and this
            // tile's filter.  Every tile has one in its main loop except a one-stage last tile.
            if (last && a.nkb == 1) __syncthreads();
            bool grew = false;                               // this wave emptied its pool during the tile
            auto filter = [&](auto ntc) {
                constexpr int nt = decltype(ntc)::value;
                const int qloc = wn * 64 + nt * 32 + (lane & 31);
                float t = (q0 + qloc) < a.Zq ? tau[qloc] : INFINITY;
                if (kHalf) t -= err;
                // the largest score of each 32-label block, then of all: a block is looked through only if its own passes
                // (late phases let through about one score per four blocks: 10 M x 120 bf16, 18 834 queries 69.4 -> 65.9 ms
                // together with the smaller growth of these phases)
                float mb[4];
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    mb[mt] = acc[mt][nt][0];
#pragma unroll
                    for (int i = 1; i < 16; ++i) mb[mt] = fmaxf(mb[mt], acc[mt][nt][i]);
                }
                if (__ballot(fmaxf(fmaxf(mb[0], mb[1]), fmaxf(mb[2], mb[3])) >= t) != 0ull) {
                    // entry: score bits, query << 24 | label offset from the pool's first tile
                    auto row_word = [&]() {
                        uint32_t w = (static_cast<uint32_t>(qloc) << 24) |
                                     (static_cast<uint32_t>(tile - pool_tile) * kBM + static_cast<uint32_t>(4 * (lane >> 5)));
                        asm volatile("" : "+v"(w));          // keep the 64 row words out of registers
                        return w;
                    };
                    uint32_t qrow = row_word();
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt) {
                        if (__ballot(mb[mt] >= t) == 0ull) continue;
#pragma unroll
                        for (int i0 = 0; i0 < 16; i0 += kPoolCheck) {
#pragma unroll
                            for (int ii = 0; ii < kPoolCheck; ++ii) {
                                const int i = i0 + ii;
                                const float v = acc[mt][nt][i];
                                const bool hit = v >= t;
                                const uint64_t m = __ballot(hit);
                                if (__builtin_expect(m != 0ull, 0)) {    // out of line: a taken branch costs more
                                    if (hit) {
                                        const int pos = fill + static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                                            static_cast<uint32_t>(m >> 32),
                                            __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)));
                                        pool[pos] = make_uint2(
                                            __float_as_uint(v),
                                            qrow + static_cast<uint32_t>(wm * 128 + mt * 32 + 8 * (i >> 2) + (i & 3)));
                                    }
                                    fill += __popcll(m);
                                }
                            }
                            // kPoolCheck accumulators add at most kPool - kPoolKeep entries
                            if (__builtin_expect(fill > kPoolKeep, 0)) {
                                flush();
                                pool_tile = tile;
                                qrow = row_word();
                                grew = true;
                            }
                        }
                    }
                }
            };
            filter(IC<0>{});
            filter(IC<1>{});
            // the label offset of an entry has 24 bits
            if (fill > 0 && (tile + 1 == n_tiles || tile - pool_tile >= 60000)) {
                flush();
                pool_tile = tile;
                grew = true;
            }
            if (grew && lane == 0) dirty[par] = 1;

            // ---- lists grown during the previous tile (the flag was set before barriers that every
            // wave has passed since), or the end of the slice: wave w looks after queries 32w..32w+31.
            // A list that could overflow before the next look (two tiles add at most 2 kBM entries, the
            // two pools that feed it at most kPoolKeep each), or, at the end of the slice, exceeds what
            // a slice may append, is cut to its best k and tau rises for the rest of the slice.
            if (last || dirty[par ^ 1] != 0) {               // uniform
                __syncthreads();                             // the pools' stores to the lists are complete
                const int qloc = wave * 32 + (lane & 31);
                const bool qok = (q0 + qloc) < a.Zq;
                int n = cnt[qloc];
                const bool want = lane < 32 && qok &&
                                  (last ? n > a.append_max : n > kCandCap - 2 * kBM - 2 * kPoolKeep);
                uint64_t todo = __ballot(want);
                if (kHalf && todo != 0ull) {
                    // scores that are not exact choose nothing: the query tile is left to the fp32 kernels
                    if (want) { tau[qloc] = INFINITY; cnt[qloc] = 0; n = 0; }
                    if (lane == 0) { a.over[0] = 1; a.over[1 + qtile] = 1; }
                    todo = 0ull;
                }
                if (todo != 0ull || last) {
                    float t_new = -INFINITY;
                    while (todo) {
                        const int src = __ffsll(static_cast<long long>(todo)) - 1;
                        todo &= todo - 1;
                        const int qsel = wave * 32 + src;
                        const int nsel = __shfl(n, src, kWave);
                        uint64_t* lsel = my_lists + static_cast<size_t>(qsel) * kCandCap;
                        const float t = wave_select_k<kCandCap / kWave>(
                            lsel, [lsel](int idx) { return lsel[idx]; }, nsel, a.k, hist + wave * 256);
                        if (lane == src) { t_new = t; n = a.k; }
                    }
                    if (!kHalf && want) { tau[qloc] = fmaxf(tau[qloc], t_new); cnt[qloc] = n; }
                    if (last) {
                        // ---- close the slice: append the survivors to the global list of each query
                        int base = 0;
                        const bool have = lane < 32 && qok && n > 0;
                        if (have) base = atomicAdd(&a.gcnt[q0 + qloc], n);
                        if (__ballot(have && n > 16) == 0ull) {
                            // short lists (the usual case): lanes l and l + 32 copy the list of query l,
                            // even and odd entries, all loads issued before the stores
                            const int nq = __shfl(have ? n : 0, lane & 31, kWave);
                            const int bq = __shfl(base, lane & 31, kWave);
                            const int ql = wave * 32 + (lane & 31);
                            const uint64_t* list = my_lists + static_cast<size_t>(ql) * kCandCap;
                            uint64_t* out = a.glist + static_cast<size_t>(q0 + ql) * a.glist_cap + bq;
                            uint64_t v[8];
#pragma unroll
                            for (int j = 0; j < 8; ++j) {
                                const int e = (lane >> 5) + 2 * j;
                                v[j] = e < nq ? list[e] : 0ull;
                            }
#pragma unroll
                            for (int j = 0; j < 8; ++j) {
                                const int e = (lane >> 5) + 2 * j;
                                if (e < nq && bq + e < a.glist_cap) out[e] = v[j];
                            }
                        } else {
                            // long lists (dense early phases): 64 entries of 8 queries per round,
                            // loads before stores
                            const int nv = have ? n : 0;
                            for (int c0 = 0; __ballot(nv > c0) != 0ull; c0 += kWave) {
                                const int e = c0 + lane;
                                for (int qb = 0; qb < 32; qb += 8) {
                                    uint64_t v[8];
                                    int dst[8];
#pragma unroll
                                    for (int u = 0; u < 8; ++u) {
                                        const int nsel = __shfl(nv, qb + u, kWave);
                                        const int bsel = __shfl(base, qb + u, kWave);
                                        dst[u] = (e < nsel && bsel + e < a.glist_cap) ? bsel + e : -1;
                                        v[u] = dst[u] >= 0
                                                   ? my_lists[static_cast<size_t>(wave * 32 + qb + u) * kCandCap + e]
                                                   : 0ull;
                                    }
#pragma unroll
                                    for (int u = 0; u < 8; ++u)
                                        if (dst[u] >= 0)
                                            a.glist[static_cast<size_t>(q0 + wave * 32 + qb + u) * a.glist_cap + dst[u]] = v[u];
                                }
                            }
                        }
                    }
                }
                if (tid == 0) { dirty[par ^ 1] = 0; if (last) dirty[par] = 0; }
                __syncthreads();
            }
        }
    }
}

// ---------------------------------------------------------------------------
// The same work item (256 queries x one label slice) for bf16 rows of at most 512 bytes
// (NK = row bytes / 128 = 1..4), where a wave's share of the query tile fits its registers.
//   * The query tile never passes through LDS: wave (wm, wn) keeps the MFMA B operands of its 64
//     queries for the whole row in registers (NK * 32 of them), loaded once per work item.
//   * Only W is streamed: a label tile is 64 WM labels, staged 128 bytes of each row at a time
//     through a ring of kRing stages in LDS, filled kRing - 1 stages ahead by direct
//     global->LDS loads, issued by one wave per SIMD in turn.  2 operand reads from LDS per 4
//     MFMAs instead of 6 per 8.
//   * A wave computes 64 labels x 64 queries (2 x 2 MFMA blocks); the 8 waves are laid out WM
//     along the labels x 8 / WM along the queries.  WM = 2: 128 labels x 256 queries per tile,
//     half the bytes staged per flop of the general kernel.  WM = 1: 64 labels x 512 queries
//     (two adjacent 256-query tiles form one work item), a quarter; for pools that fill it.
//   * A lane owns two query columns and the thresholds of exactly those, which it keeps in
//     registers.  A passing score goes straight to a candidate list that belongs to the lane
//     alone (2 WM owners per query: WM waves x 2 lane halves, 256 keys each, in the workgroup's
//     part of the workspace), at a position the lane counts itself: no atomics, no LDS, no
//     barrier on the path.
//   * A lane's list that could overflow in the next tile is cut to its best k by the lane's wave
//     (every label of the overall best k that is in this list is among the list's own best k),
//     and the lane's threshold rises to the k-th of them.  Nothing of that involves other waves.
//   * At the end of the slice the lists of a query are appended to its global list, cut to
//     the best k of them all first if they hold more than a slice may append.
// ---------------------------------------------------------------------------
constexpr int kSubCap = kCandCap / 4;            // keys of a lane's own list
constexpr int kSubFull = kSubCap - 32;           // above this a tile could overflow it (a lane adds <= 32 per column)
constexpr size_t rows_lds_bytes(int wm) {     // ring, list fills at the end of a slice, select histograms
    return static_cast<size_t>(kRing) * wm * 64 * kStageBytes + kBN * 4 * sizeof(int) + kMineWaves * 256 * sizeof(int);
}

// XC_MINE_GENERAL=1 in the environment (read at every call) sends every shape through the general tile
// kernel, for A/B timing and for tests
static bool force_general_kernel() {
    const char* e = getenv("XC_MINE_GENERAL");
    return e != nullptr && e[0] == '1';
}

// fp16 copies: VARIED where each label tile has its own error, else one error for all.  Both forms are launched, and one returns at once (the
// question asked where scores pass, or two ways in one kernel, cost rows of 128 to 512 bytes 3 to 9 %).
template <typename T, int NK, int WM, bool VARIED>
__global__ __launch_bounds__(kMineThreads, 1)
void mine_rows_kernel(const MineArgs a) {
    static_assert(WM == 1 || WM == 2, "wave layouts");
    constexpr bool kHalf = std::is_same<T, half_t>::value;
    constexpr int kRowTile = 64 * WM;                   // labels per tile
    constexpr int kRowStage = kRowTile * kStageBytes;   // bytes of a stage
    constexpr int kQN = (kMineWaves / WM) * 64;         // queries per work item
    constexpr int kOwn = 2 * WM;                        // lists per query (kOwn * kQN = 4 kBN)
    constexpr int kQCap = kOwn * kSubCap;               // keys of a query's lists together
    constexpr int kLd = 2 * WM;                         // load instructions of a wave per stage it brings in
    extern __shared__ __align__(16) unsigned char smem[];
    if (a.cond != nullptr && a.cond[0] == 0) return;          // uniform: a repeat that is not needed
    if (kHalf && VARIED != (half_error_of_all(a.err_range) < 0.0f)) return;         // uniform
    int* cnt4 = reinterpret_cast<int*>(smem + kRing * kRowStage);            // [kQN][kOwn] list fills at the end of a slice
    int* hist = cnt4 + kBN * 4;                                             // [kMineWaves][256]
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) unsigned char*)smem));

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM;         // which 64 labels of the tile
    const int wn = wave / WM;         // which 64 queries of the work item
    const int half = lane >> 5;
    uint64_t* my_lists = a.lists + static_cast<size_t>(blockIdx.x) * kBN * kCandCap;
    constexpr int row_bytes = NK * kStageBytes;
    // a query takes part if it exists and, in the repeat of a warm search, if its 256-query tile needs it
    auto live = [&](int64_t q) {
        return q < a.Zq && (kHalf ? a.skip[q / kBN] == 0 : a.cond == nullptr || a.cond[1 + q / kBN] != 0);
    };

    int item, item_step, item_end;
    int slice_fixed = -1;
    int64_t tiles_per_slice = a.tiles_per_slice;
    int append_max = a.append_max;
    if (a.Qx > 0) {                   // slices bound to XCDs: workgroup w runs on XCD w % 8
        const int xcd = blockIdx.x % kXcds;
        const int cu = blockIdx.x / kXcds;
        int S = a.S, Qx = a.Qx;
        item_end = static_cast<int>(a.nQT);
        if (a.items != nullptr) {     // a plan of its own for the few items there are (see the 8-bit filter)
            item_end = __builtin_amdgcn_readfirstlane(a.items[0]);
            const int sx = __builtin_amdgcn_readfirstlane(a.items[1]);
            S = kXcds * sx;
            Qx = kCusPerXcd / sx;
            tiles_per_slice = (a.tile_hi - a.tile_lo + S - 1) / S;
            append_max = (a.glist_cap - a.kcap) / S;
        }
        slice_fixed = __builtin_amdgcn_readfirstlane(xcd + kXcds * (cu / Qx));
        item = __builtin_amdgcn_readfirstlane(cu % Qx); item_step = Qx;
        if (slice_fixed >= S) item_end = 0;
    } else {
        item = blockIdx.x; item_step = kMineGrid; item_end = static_cast<int>(a.nQT * a.S);
    }

    // fragment reads of the A operand (as in the general kernel: row pitch 128, chunks swizzled by (row >> 1) & 7)
    const int swz = (lane >> 1) & 7;
    const int frag_a = (wm * 64 + (lane & 31)) * kStageBytes + ((half ^ swz) * 16);
    // stage fill.  Waves w and w + 4 share a SIMD.  A stage is brought in by four waves, one per SIMD, while
    // their SIMD-mates start on the MFMAs at once (a wave that issues loads queues at the texture unit behind
    // the other waves' loads; if all eight issued, every SIMD's matrix pipe would idle meanwhile); waves 0..3
    // take the even stages, waves 4..7 the odd ones.  Wave w brings in rows 8 kLd (w & 3) .. + 8 kLd - 1 of the stage
    // with kLd instructions of 8 rows; lane i -> row i / 8, position i % 8, source chunk = position ^ swizzle(row)
    const int drow = lane >> 3;
    const int wq = wave & 3;
    const int my_parity = wave >> 2;
    const uint32_t dcol[2] = {static_cast<uint32_t>(((lane & 7) ^ (lane >> 4)) * 16),
                              static_cast<uint32_t>(((lane & 7) ^ ((lane >> 4) + 4)) * 16)};
    const uint32_t voff[2] = {static_cast<uint32_t>(drow * row_bytes) + dcol[0],
                              static_cast<uint32_t>((drow + 8) * row_bytes) + dcol[1]};
    const uint32_t dma_dst = lds_base + wq * kLd * 1024;

    for (; item < item_end; item += item_step) {
        const int64_t qtile = a.Qx > 0 ? (a.items != nullptr ? __builtin_amdgcn_readfirstlane(a.items[2 + item]) : item) : item / a.S;
        const int64_t q0 = qtile * kQN;
        if (a.cond != nullptr) {                             // uniform: every 256-query tile of the item came out complete
            bool any = false;
            for (int64_t qt = q0 / kBN; qt < (q0 + kQN) / kBN && qt * kBN < a.Zq; ++qt) any = any || a.cond[1 + qt] != 0;
            if (!any) continue;
        }
        if (kHalf) {                                         // the same for tiles given up
            bool any = false;
            for (int64_t qt = q0 / kBN; qt < (q0 + kQN) / kBN && qt * kBN < a.Zq; ++qt) any = any || a.skip[qt] == 0;
            if (!any) continue;
        }
        const int slice = a.Qx > 0 ? slice_fixed : static_cast<int>(item % a.S);
        const int64_t t_begin = a.tile_lo + static_cast<int64_t>(slice) * tiles_per_slice;
        int64_t lab_begin, lab_end;
        {
            int64_t t_end = t_begin + tiles_per_slice;
            t_end = t_end < a.tile_hi ? t_end : a.tile_hi;
            if (t_end <= t_begin) continue;                  // uniform: an empty slice
            lab_begin = t_begin * kBM;
            lab_end = t_end * kBM;
            lab_end = lab_end < a.L ? lab_end : a.L;
        }
        const int n_tiles = static_cast<int>((lab_end - lab_begin + kRowTile - 1) / kRowTile);
        const int n_stages = n_tiles * NK;

        // ---- this wave's queries: B operands for the whole row, thresholds of the lane's two columns
        uint4 zf[NK * 4][2];
        float tau[2];
        int cnt[2] = {0, 0};
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const int64_t q = q0 + wn * 64 + nt * 32 + (lane & 31);
            const int64_t qc = q < a.Zq ? q : a.Zq - 1;
            tau[nt] = live(q) ? ordered_to_float(a.tau_g[q]) : INFINITY;
            if (kHalf && !VARIED) tau[nt] -= half_error_of_all(a.err_range);
            const unsigned char* zr = a.Z + qc * row_bytes + half * 16;
#pragma unroll
            for (int ks = 0; ks < NK * 4; ++ks) zf[ks][nt] = *reinterpret_cast<const uint4*>(zr + ks * 32);
        }

        // every load so far has landed before the first stage load is issued: from here on the only vector memory
        // operations in flight are the stage loads (and the filter's rare stores), counted by the waits below
        wait_all_vmem();

        // ---- the load stream: stage g = (tile g / NK, bytes 128 (g % NK) .. of the rows) goes to slot g % kRing
        int ld_stage = 0, ld_kb = 0, ld_tile = 0;
        uint32_t ld_dst = dma_dst;
        const unsigned char* ld_w = a.W + (lab_begin + wq * 8 * kLd) * row_bytes;   // this wave's rows of the tile being loaded
        const int full_tiles = static_cast<int>((a.w_rows - lab_begin) / kRowTile < n_tiles ? (a.w_rows - lab_begin) / kRowTile : n_tiles);
        auto issue_stage = [&]() {
            if ((ld_stage & 1) != my_parity) {
                // the other half's turn
            } else if (ld_tile < full_tiles) {
                const uint64_t b64 = reinterpret_cast<uint64_t>(ld_w + ld_kb * kStageBytes);
                const uint64_t sb =
                    (static_cast<uint64_t>(static_cast<uint32_t>(
                         __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64 >> 32)))) << 32) |
                    static_cast<uint64_t>(static_cast<uint32_t>(
                        __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64))));
                const unsigned char* sp = reinterpret_cast<const unsigned char*>(sb);
                lds_dma16_sbase<0>(sp, voff[0], ld_dst);
                lds_dma16_sbase<1024>(sp, voff[1], ld_dst);
                if (WM == 2) {
                    const unsigned char* sp2 = sp + 16 * row_bytes;
                    lds_dma16_sbase<2048>(sp2, voff[0], ld_dst);
                    lds_dma16_sbase<3072>(sp2, voff[1], ld_dst);
                }
            } else {
                // the last tile of the label range: rows past the end repeat the last row (dropped by the filter)
                issue_stage_ragged(a.W, a.w_rows, lab_begin + static_cast<int64_t>(ld_tile) * kRowTile + wq * 8 * kLd + drow,
                                   row_bytes, ld_kb * kStageBytes, dcol[0], dcol[1], ld_dst, kLd);
            }
            ++ld_stage;
            ld_dst += kRowStage;
            if ((ld_stage & (kRing - 1)) == 0) ld_dst = dma_dst;
            if (++ld_kb == NK) { ld_kb = 0; ++ld_tile; ld_w += kRowTile * row_bytes; }
        };
        // This wave's part of stage g (if it has one) is complete once at most kLd * (its stages issued after g)
        // loads are outstanding: of the kRing - 2 stages issued after g in the steady state half are this
        // wave's, whichever half g belongs to.  Stores of the filter only make the wait stricter (loads complete
        // in order among themselves).  Near the end of the work item everything is awaited.
        auto wait_stage = [&](int g) {
            if (ld_stage - 1 - g >= kRing - 2) wait_vmem_at_most<kLd * ((kRing - 2) / 2)>();
            else wait_all_vmem();
        };

        f32x16 acc[2][2];
        uint4 fa[2][2];
        auto read_frags = [&](int slot, int kk, int sel) {
            const unsigned char* buf = smem + slot * kRowStage;
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
                fa[sel][mt] = *reinterpret_cast<const uint4*>(buf + ((frag_a ^ (kk * 32)) + mt * 32 * kStageBytes));
        };
        // stage g + 1 visible to everyone, stage g's slot free: refill it, and fetch the first operands of stage g + 1
        auto publish = [&](int g_next) {
            wait_stage(g_next);
            lds_barrier();
            if (ld_stage < n_stages) issue_stage();
            read_frags(g_next % kRing, 0, 0);
        };

        __syncthreads();                                     // the ring and cnt4 are free (previous item closed)
        for (int s = 0; s < kRing - 1 && s < n_stages; ++s) issue_stage();
        publish(0);

        // ---- threshold filter of one N block (the lane owns query column (lane & 31) of it) of the tile that
        // starts at label l0: the block's largest score per lane, and, where some lane's reaches its threshold,
        // the scores one by one
        auto block_max = [&](auto ntc) {
            constexpr int nt = decltype(ntc)::value;
            float mx = acc[0][nt][0];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc[mt][nt][i]);
            return mx;
        };
        auto push_block = [&](auto ntc, int64_t l0, float mx, float t) __attribute__((always_inline)) {
            constexpr int nt = decltype(ntc)::value;
            if (__ballot(mx >= t) != 0ull) {
                // Everything a push needs is formed here from the lane number, read afresh, and from wave-uniform
                // values: a per-lane pointer or row number kept in a register over the main loop would be
                // spilled there, and its reload would wait for every stage load in flight.
                const int32_t lmax = static_cast<int32_t>(a.L);
                const int32_t lbase = static_cast<int32_t>(l0) + wm * 64;
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float v = acc[mt][nt][i];
                        if (__builtin_expect(__ballot(v >= t) != 0ull, 0)) {
                            const uint32_t l = lane_now();
                            const int32_t lab = lbase + 4 * static_cast<int32_t>(l >> 5) + mt * 32 + 8 * (i >> 2) + (i & 3);
                            if (v >= t && lab < lmax) {             // rows past the end repeat the last row
                                const uint32_t sub = static_cast<uint32_t>(((wn * 64 + nt * 32) * kOwn + wm * 2)) + (l & 31u) * kOwn + (l >> 5);
                                my_lists[sub * kSubCap + static_cast<uint32_t>(cnt[nt])] = make_key(v + 0.0f /* -0 -> +0 */, lab);
                                ++cnt[nt];
                            }
                        }
                    }
            }
        };
        // ---- a list that the next tile could overflow: cut to its best k, by this wave alone
        auto cut_lists = [&]() {
            if (kHalf) {                                     // (not exact: the query's tile is left to the fp32 kernels)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    if (cnt[nt] > kSubFull) {
                        const int64_t q = q0 + wn * 64 + nt * 32 + (lane_now() & 31u);
                        a.over[0] = 1;
                        a.over[1 + q / kBN] = 1;
                        cnt[nt] = 0;
                        tau[nt] = INFINITY;
                    }
            } else if (__builtin_expect(__ballot(cnt[0] > kSubFull || cnt[1] > kSubFull) != 0ull, 0)) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");       // this wave's list stores are complete ...
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");       // ... and are what the loads below see
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    uint64_t todo = __ballot(cnt[nt] > kSubFull);
                    while (todo) {
                        const int src = __ffsll(static_cast<long long>(todo)) - 1;
                        todo &= todo - 1;
                        const int qsel = wn * 64 + nt * 32 + (src & 31);
                        const int nsel = __shfl(cnt[nt], src, kWave);
                        uint64_t* lsel = my_lists + static_cast<size_t>(qsel * kOwn + wm * 2 + (src >> 5)) * kSubCap;
                        const float tk = wave_select_k<kSubCap / kWave>(
                            lsel, [lsel](int idx) { return lsel[idx]; }, nsel, a.k, hist + wave * 256);
                        if (lane == src) { cnt[nt] = a.k; tau[nt] = fmaxf(tau[nt], tk); }
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            }
        };

        // ---- main loop.  (Deferring a block's filter into the next tile's first products, so that the vector
        // ALU works while the matrix pipe does, was measured and gained nothing: the kernel runs at the chip's
        // power limit, where the clock falls as the matrix pipe fills.)
        int g = 0;                                           // stage being computed
        for (int tile = 0; tile < n_tiles; ++tile) {
            const int64_t l0 = lab_begin + static_cast<int64_t>(tile) * kRowTile;
#pragma unroll
            for (int kb = 0; kb < NK; ++kb) {
                const int slot = g % kRing;
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    const int sel = kk & 1;
                    if (kk < 3) {
                        read_frags(slot, kk + 1, sel ^ 1);
                    } else {
                        // (reads into fa[0], which the products of kk = 2 have left.  Also after the last stage,
                        // where the operands read are never used: one way through the loop body, so that no wait
                        // meant for another way in holds up the products below)
                        publish(g + 1);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                        for (int nt = 0; nt < 2; ++nt) {
                            if (kb == 0 && kk == 0) {
                                f32x16 c = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                                RowMma<T>::mma(fa[sel][mt], zf[kb * 4 + kk][nt], c);
                                acc[mt][nt] = c;
                            } else {
                                RowMma<T>::mma(fa[sel][mt], zf[kb * 4 + kk][nt], acc[mt][nt]);
                            }
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
                ++g;
            }
            // one test per tile on the usual way: does any lane see a score at its threshold, or a list to cut?
            const float mx0 = block_max(IC<0>{}), mx1 = block_max(IC<1>{});
            float t0 = tau[0], t1 = tau[1];
            if (VARIED) {
                const float err = uniform_load(a.tile_err, l0 / kBM);
                t0 -= err;
                t1 -= err;
            }
            const bool look = mx0 >= t0 || mx1 >= t1 || cnt[0] > kSubFull || cnt[1] > kSubFull;
            if (__builtin_expect(__ballot(look) != 0ull, 0)) {
                push_block(IC<0>{}, l0, mx0, t0);
                push_block(IC<1>{}, l0, mx1, t1);
                cut_lists();
            }
        }

        // ---- close the slice: the lists of a query go to its global list
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) cnt4[(wn * 64 + nt * 32 + (lane & 31)) * kOwn + wm * 2 + half] = cnt[nt];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
#pragma unroll 1
        for (int qr = 0; qr < kQN; qr += kMineWaves * 32) {
            const int qw = qr + wave * 32;                   // lanes l and l + 32 look after query qw + l
            const int ql = qw + (lane & 31);
            const bool qok = live(q0 + ql);
            int c[kOwn];
            int n = 0;
#pragma unroll
            for (int s = 0; s < kOwn; ++s) { c[s] = qok ? cnt4[ql * kOwn + s] : 0; n += c[s]; }
            uint64_t* qlist = my_lists + static_cast<size_t>(ql) * kQCap;
            uint64_t todo = __ballot(lane < 32 && n > append_max);
            while (todo) {                                   // more than a slice may append: the best k of them all
                const int src = __ffsll(static_cast<long long>(todo)) - 1;
                todo &= todo - 1;
                int cs[kOwn];
                int ntot = 0;
#pragma unroll
                for (int s = 0; s < kOwn; ++s) { cs[s] = __shfl(c[s], src, kWave); ntot += cs[s]; }
                uint64_t* lsel = my_lists + static_cast<size_t>(qw + src) * kQCap;
                auto at = [lsel, &cs](int idx) {
                    int s = 0;
#pragma unroll
                    for (int u = 0; u + 1 < kOwn; ++u)
                        if (s == u && idx >= cs[u]) { idx -= cs[u]; s = u + 1; }
                    return lsel[s * kSubCap + idx];
                };
                wave_select_k<kQCap / kWave>(lsel, at, ntot, a.k, hist + wave * 256);
                if ((lane & 31) == src) {
                    c[0] = a.k;
#pragma unroll
                    for (int s = 1; s < kOwn; ++s) c[s] = 0;
                    n = a.k;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            int base = 0;
            if (lane < 32 && n > 0) base = atomicAdd(&a.gcnt[q0 + ql], n);
            base = __shfl(base, lane & 31, kWave);
            uint64_t* out = a.glist + static_cast<size_t>(q0 + ql) * a.glist_cap;
            int off = base;
#pragma unroll
            for (int s = 0; s < kOwn; ++s) {
                for (int e = half; e < c[s]; e += 2)
                    if (off + e < a.glist_cap) out[off + e] = qlist[s * kSubCap + e];
                off += c[s];
            }
        }
    }
}

// The instances of the row kernel: rows of 128..512 bytes in either wave layout.  (With four waves, one per
// SIMD and 512 registers each, the queries of rows up to 1 KiB fit as well; measured at 1 KiB rows that
// ran 15 % slower than the general kernel - no second wave covers a wave's barrier and filter time.)
typedef void (*RowsKernelFn)(const MineArgs);
struct RowsKernel { RowsKernelFn fn; int nk, wm; bool half; RowsKernelFn varied; };
#define XC_ROWS(NK, WM) {&mine_rows_kernel<bf16_t, NK, WM, false>, NK, WM, false, nullptr}
#define XC_ROWS_HALF(NK, WM) {&mine_rows_kernel<half_t, NK, WM, false>, NK, WM, true, &mine_rows_kernel<half_t, NK, WM, true>}
static const RowsKernel kRowsKernels[] = {
    XC_ROWS(1, 2), XC_ROWS(2, 2), XC_ROWS(3, 2), XC_ROWS(4, 2), XC_ROWS(1, 1), XC_ROWS(2, 1), XC_ROWS(3, 1), XC_ROWS(4, 1),
    XC_ROWS_HALF(1, 2), XC_ROWS_HALF(2, 2), XC_ROWS_HALF(3, 2), XC_ROWS_HALF(4, 2),
    XC_ROWS_HALF(1, 1), XC_ROWS_HALF(2, 1), XC_ROWS_HALF(3, 1), XC_ROWS_HALF(4, 1),
};
#undef XC_ROWS
#undef XC_ROWS_HALF
static const RowsKernel* find_rows_kernel(int nk, int wm, bool half) {
    for (const RowsKernel& k : kRowsKernels)
        if (k.nk == nk && k.wm == wm && k.half == half) return &k;
    return nullptr;
}

__global__ void mine_init_kernel(uint32_t* tau_g, int32_t* gcnt, int64_t n, uint32_t* zeros /* [64] */,
                                 const int32_t* cond) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < 64) zeros[i] = 0u;
    if (i < n && (cond == nullptr || cond[1 + i / kBN] != 0)) { tau_g[i] = kTauInit; gcnt[i] = 0; }
}

// Start of a warm search: the thresholds the previous search left behind, lowered by rel * |tau|,
// are the thresholds of one sweep over all labels.  Whatever they are, the outcome is exact: a query
// that ends the sweep with fewer than k candidates raises the flag of its query tile, and the full
// search is repeated for the flagged tiles.
__global__ void mine_warm_init_kernel(uint32_t* tau_g, int32_t* gcnt, int64_t n, uint32_t* zeros /* [64] */,
                                      int32_t* flag /* [1 + n / kBN] */, float rel) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) {
        const float t = ordered_to_float(tau_g[i]);
        tau_g[i] = float_to_ordered(t - rel * fabsf(t));
        gcnt[i] = 0;
    }
    if (i < 64) zeros[i] = 0u;
    if (i <= n / kBN) flag[i] = 0;
}

// ---------------------------------------------------------------------------
// Radix select for lists too long for registers (n > 64*kSelectRegs): the keys
// are streamed from memory in every pass.  Same result as wave_select_k.
// ---------------------------------------------------------------------------
// Bound such that exactly k of the n > k keys load(0..n-1) are at or below it.
template <typename Load>
__device__ __noinline__ uint64_t wave_bound_stream(Load load, int n, int k, int* hist) {
    const int lane = lane_id();
    uint64_t prefix = 0, pmask = 0;
    int need = k;
    for (int pass = 0; pass < 8; ++pass) {
        const int shift = 56 - 8 * pass;
#pragma unroll
        for (int j = 0; j < 4; ++j) hist[lane * 4 + j] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        for (int idx = lane; idx < n; idx += kWave) {
            const uint64_t key = load(idx);
            if ((key & pmask) == prefix) atomicAdd(&hist[static_cast<int>((key >> shift) & 255u)], 1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        int c[4];
        int s = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) { c[j] = hist[lane * 4 + j]; s += c[j]; }
        const int incl = wave_incl_scan(s);
        const int excl = incl - s;
        const bool mine = (excl < need) && (need <= incl);
        int dsel = 0, needn = 0, have = 0;
        if (mine) {
            int cum = excl;
            bool done = false;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!done && need <= cum + c[j]) {
                    dsel = lane * 4 + j; needn = need - cum; have = c[j]; done = true;
                }
                cum += c[j];
            }
        }
        const uint64_t bal = __ballot(mine);
        const int src = __ffsll(static_cast<long long>(bal)) - 1;
        dsel = __shfl(dsel, src, kWave);
        needn = __shfl(needn, src, kWave);
        have = __shfl(have, src, kWave);
        prefix |= static_cast<uint64_t>(dsel) << shift;
        pmask |= 0xffull << shift;
        need = needn;
        if (have == need) break;
    }
    return prefix | ~pmask;
}

__device__ __noinline__ float wave_select_stream(uint64_t* __restrict__ buf, int n, int k, int* hist) {
    const int lane = lane_id();
    const uint64_t bound = wave_bound_stream([buf](int idx) { return buf[idx]; }, n, k, hist);
    // compaction in place: a chunk is read into registers before anything of it is
    // overwritten, and the write position never passes the read position
    uint64_t kmax = 0;
    int base = 0;
    for (int c0 = 0; c0 < n; c0 += kWave) {
        const int idx = c0 + lane;
        const uint64_t key = idx < n ? buf[idx] : kKeySentinel;
        const bool sel = idx < n && key <= bound;
        const uint64_t m = __ballot(sel);
        const int p = base + __popcll(m & lanemask_lt());
        if (sel && p < k) {
            buf[p] = key;
            kmax = key > kmax ? key : kmax;
        }
        base += __popcll(m);
    }
    kmax = wave_max_u64(kmax);
    return key_score(kmax);
}

// ---------------------------------------------------------------------------
// After a phase: one wave per query cuts the global candidate list to its best
// k and publishes the k-th score as the threshold of the next phase.  After the
// last phase the winners are sorted and written out.
// ---------------------------------------------------------------------------
// bitonic sort of the (at most 128) winners inside the wave, and the result
__device__ __forceinline__ void wave_write_winners(const uint64_t* list, int n, int k, uint64_t* srt, int32_t* ids, float* scores) {
    const int lane = lane_id();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // the select's stores to `list` are visible
    for (int e = lane; e < XC_MAX_K_MINE; e += kWave) srt[e] = e < n ? list[e] : kKeySentinel;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    for (int size = 2; size <= XC_MAX_K_MINE; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const int t = lane;                       // 64 compare-exchanges cover 128 keys
            const int lo = 2 * t - (t & (stride - 1));
            const int hi = lo + stride;
            const bool up = (lo & size) == 0;
            const uint64_t x = srt[lo], y = srt[hi];
            if ((x > y) == up) { srt[lo] = y; srt[hi] = x; }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        }
    }
    for (int r = lane; r < k; r += kWave) {
        const uint64_t v = srt[r];
        ids[r] = key_id(v);
        if (scores) scores[r] = (v == kKeySentinel) ? -INFINITY : key_score(v);
    }
}

constexpr int kSelectWaves = 4;

__global__ __launch_bounds__(kSelectWaves * kWave)
void mine_select_kernel(uint64_t* __restrict__ glist, int32_t* __restrict__ gcnt,
                        uint32_t* __restrict__ tau_g, int64_t Zq, int glist_cap, int k, int final_phase,
                        int32_t* __restrict__ shortlist, float* __restrict__ scores,
                        const int32_t* __restrict__ cond /* not null: only query tiles qt with cond[1 + qt] != 0 */,
                        int32_t* __restrict__ short_flag /* not null: [0] and [1 + qt] are set when a query of tile qt
                                                            has fewer than k candidates */) {
    __shared__ int hist[kSelectWaves][256];
    __shared__ uint64_t sorted[kSelectWaves][XC_MAX_K_MINE];
    const int lane = lane_id();
    const int wave = threadIdx.x >> 6;
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kSelectWaves + wave;
    if (q >= Zq) return;                               // wave-uniform; no workgroup barrier below
    if (cond != nullptr && cond[1 + q / kBN] == 0) return;
    uint64_t* list = glist + static_cast<size_t>(q) * glist_cap;
    int n = gcnt[q];
    n = n < glist_cap ? n : glist_cap;
    if (short_flag != nullptr && n < k && lane == 0) { short_flag[0] = 1; short_flag[1 + q / kBN] = 1; }
    if (n > k) {
        auto at = [list](int idx) { return list[idx]; };
        const float t = (n <= kSelectRegs / 2 * kWave) ? wave_select_k<kSelectRegs / 2>(list, at, n, k, hist[wave])
                        : (n <= kSelectRegs * kWave)   ? wave_select_k<kSelectRegs>(list, at, n, k, hist[wave])
                                                       : wave_select_stream(list, n, k, hist[wave]);
        n = k;
        if (lane == 0) { gcnt[q] = k; tau_g[q] = float_to_ordered(t); }
    }
    if (!final_phase) return;
    wave_write_winners(list, n, k, sorted[wave], shortlist + q * k, scores != nullptr ? scores + q * k : nullptr);
}

// ---------------------------------------------------------------------------
// After the dense first phase: one wave per query takes the best k of its R * 256 scores (label = position) and publishes
// the threshold.  The k-th largest of the 128 maxima that the lanes hold over halves of their scores bounds the k-th score from
// below (k of the scores reach it); what passes that - about 1.3 k - goes through the radix select.  If too many pass
// (equal scores), the k-th largest score is found by bisection over all of them, ties by the smaller label.
// ---------------------------------------------------------------------------
constexpr int kDenseTiles = 16;                 // tiles of the dense phase at most (one float4 per tile and lane)
constexpr int kDenseMin = 4;                    // and at least: k <= 128 halves of the lanes' scores have a maximum
constexpr int kDenseList = 512;                 // keys of a wave's list

__device__ __forceinline__ uint32_t dense_image(float v) { return v == v ? float_to_ordered(v + 0.0f /* -0 -> +0 */) : 0u; }

template <int R>
__global__ __launch_bounds__(kSelectWaves * kWave)
void mine_dense_select_kernel(const float* __restrict__ dense, int dense_ld, uint64_t* __restrict__ glist,
                              int32_t* __restrict__ gcnt, uint32_t* __restrict__ tau_g, int64_t Zq, int glist_cap, int k,
                              const float* __restrict__ tile_err /* not null: 16-bit scores, to be lowered by their errors */,
                              const int32_t* __restrict__ cond /* not null: only query tiles qt with cond[1 + qt] != 0 */) {
    static_assert(R % 2 == 0 && R <= kDenseTiles, "");
    __shared__ int hist[kSelectWaves][256];
    __shared__ uint64_t picked[kSelectWaves][kDenseList];
    const int lane = lane_id();
    const int wave = threadIdx.x >> 6;
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kSelectWaves + wave;
    if (q >= Zq) return;                               // wave-uniform; no workgroup barrier below
    if (cond != nullptr && cond[1 + q / kBN] == 0) return;
    uint64_t* list = glist + static_cast<size_t>(q) * glist_cap;
    // label of v[r][j]: 256 r + 4 lane + j; rows past dense_ld do not exist (image 0, as a score that is no number)
    uint32_t v[R][4];
    float4 f[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        f[r] = make_float4(NAN, NAN, NAN, NAN);
        if (r * 256 < dense_ld) f[r] = *reinterpret_cast<const float4*>(dense + q * dense_ld + r * 256 + lane * 4);
    }
    if (tile_err != nullptr) {                         // uniform
        const float errs = lane * 256 < dense_ld ? tile_err[lane] : 0.0f;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float e = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(errs), r));
            f[r].x -= e; f[r].y -= e; f[r].z -= e; f[r].w -= e;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        v[r][0] = dense_image(f[r].x); v[r][1] = dense_image(f[r].y); v[r][2] = dense_image(f[r].z); v[r][3] = dense_image(f[r].w);
    }
    uint32_t m[2] = {0, 0};
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) m[r & 1] = v[r][j] > m[r & 1] ? v[r][j] : m[r & 1];
    // k-th largest of the 128 maxima, bit by bit (k <= 128)
    uint32_t t0 = 0;
    for (int b = 31; b >= 0; --b) {
        const uint32_t c = t0 | (1u << b);
        if (__popcll(__ballot(m[0] >= c)) + __popcll(__ballot(m[1] >= c)) >= k) t0 = c;
    }
    t0 = t0 > 0 ? t0 : 1u;                             // (fewer than k maxima that are numbers: everything that is one)
    uint64_t* keys = picked[wave];
    int n = 0;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool hit = v[r][j] >= t0;
            const uint64_t bal = __ballot(hit);
            if (hit) {
                const int at = n + __popcll(bal & lanemask_lt());
                if (at < kDenseList)
                    keys[at] = (static_cast<uint64_t>(~v[r][j]) << 32) | static_cast<uint32_t>(r * 256 + lane * 4 + j);
            }
            n += __popcll(bal);
        }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    if (n <= k) {                                      // all there are
        for (int e = lane; e < n; e += kWave) list[e] = keys[e];
        uint32_t lowest = 0xffffffffu;
        if (n == k) {
            for (int e = lane; e < n; e += kWave) { const uint32_t o = ~static_cast<uint32_t>(keys[e] >> 32); lowest = o < lowest ? o : lowest; }
            for (int off = 32; off > 0; off >>= 1) { const uint32_t o = __shfl_xor(lowest, off, kWave); lowest = o < lowest ? o : lowest; }
        }
        if (lane == 0) { gcnt[q] = n; tau_g[q] = n == k ? lowest : kTauInit; }
        return;
    }
    if (n <= kDenseList) {
        const float t = wave_select_k<kDenseList / kWave>(list, [keys](int idx) { return keys[idx]; }, n, k, hist[wave]);
        if (lane == 0) { gcnt[q] = k; tau_g[q] = float_to_ordered(t); }
        return;
    }
    uint32_t t = 0;                                    // the k-th largest score of all
    for (int b = 31; b >= 0; --b) {
        const uint32_t c = t | (1u << b);
        int have = 0;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) have += __popcll(__ballot(v[r][j] >= c));
        if (have >= k) t = c;
    }
    int above = 0;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) above += __popcll(__ballot(v[r][j] > t));
    int out = 0, tie = 0;                              // written, and ties seen so far (labels ascend with r, lane, j)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint64_t eq[4];
        int lower = tie;
#pragma unroll
        for (int j = 0; j < 4; ++j) { eq[j] = __ballot(v[r][j] == t); lower += __popcll(eq[j] & lanemask_lt()); }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool mine = v[r][j] == t;
            const bool take = v[r][j] > t || (mine && lower < k - above);
            lower += mine ? 1 : 0;
            const uint64_t bal = __ballot(take);
            if (take)
                list[out + __popcll(bal & lanemask_lt())] = (static_cast<uint64_t>(~v[r][j]) << 32) | static_cast<uint32_t>(r * 256 + lane * 4 + j);
            out += __popcll(bal);
            tie += __popcll(eq[j]);
        }
    }
    if (lane == 0) { gcnt[q] = out; tau_g[q] = t; }
}

}  // namespace xc

#include "xc_mine_half.h"

namespace xc {

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct MinePlan {
    int64_t nQT, nLT;
    int kcap, nkb, glist_cap;
    size_t off_flag, off_lists, off_glist, off_gcnt, off_tau, off_zero;
    size_t ws_min, ws_bytes;         // with ws_min the 8-bit filter, which needs the rest, stays out
    Q8Plan q8;
    HalfPlan half;
    size_t lds_tile;
};

static int slices_cap(int kcap) { return kcap <= 64 ? kMaxSlices : kMaxSlices / 2; }    // slices per phase at most

// Number of label tiles of the phase that starts at tile `lo`.  Phases end at powers of the growth
// factor (1, 8, 64, ... tiles seen).  A phase of fewer than 8 tiles deals its items (query tile,
// label tile) to the workgroups in plain order, so it is shortened by up to a third if the number
// of items then comes out just under a multiple of the grid.
static int64_t phase_tiles(int64_t lo, int64_t nQT) {
    if (lo == 0) return 1;
    int64_t end = kPhaseGrowth;
    while (end < 2 * lo) end *= kPhaseGrowth;           // a shortened phase still ends in this decade
    const int64_t want = end - lo;
    if (want >= kXcds) return want;
    int64_t best = want;
    double best_fill = 0.0;
    for (int64_t n = (2 * want + 2) / 3; n <= want; ++n) {
        if (n < 1) continue;
        const int64_t items = nQT * n;
        const int64_t rounds = (items + kMineGrid - 1) / kMineGrid;
        const double fill = static_cast<double>(items) / static_cast<double>(rounds * kMineGrid);
        if (fill >= best_fill) { best_fill = fill; best = n; }
    }
    return best;
}

// Label tiles of a dense first phase (0: none).  Every score of it is written and read once (kBM floats per query and tile, in
// `room` bytes), none goes through the filter, whose cost is that of the scores that pass: 0.37 us per score that every query
// of 10 240 lets through, and thresholds found in phases of 1, 7 and 56 tiles let through 256, 384 and 448 of them, from work
// items too few or too short to fill the chip.  About 48 k scores per query (the threshold costs memory traffic in proportion
// to the scores, the passes it saves go with k), of these numbers of tiles the one whose items fill their last round best.
// Measured, without : with, 131 072 x 768 bf16: k = 64, 1024 queries 435 : 279 us, 4096 1043 : 894, 10 240 2308 : 2180;
// k = 5, 4096 873 : 783, 20 000 3782 : 3781; 300 000 x 768, k = 128, 40 000 19.8 : 19.4 ms; 60 000 x 128 fp32, k = 100,
// 30 000 5.44 : 4.71.  Many queries with a short list have nothing to gain (131 072 x 392, k = 20, 20 000 3.47 : 3.55 ms).
static int dense_tiles(int64_t nQT, int64_t full_tiles, int k, size_t room, bool half) {
    if (!half && k < 32 && nQT > 64) return 0;
    int64_t most = (48 * k + kBM - 1) / kBM;
    most = most < kDenseMin ? kDenseMin : (most > kDenseTiles ? kDenseTiles : most);
    const int64_t fits = static_cast<int64_t>(room / (static_cast<size_t>(nQT) * kBN * kBM * sizeof(float)));
    most = most < fits ? most : fits;
    most = most < full_tiles / 2 ? most : full_tiles / 2;       // (and a range long enough to use the threshold on)
    if (most < kDenseMin) return 0;
    const int64_t least = 2 * most / 3 > kDenseMin ? 2 * most / 3 : kDenseMin;
    int best = 0;
    double best_fill = 0.0;
    for (int64_t n = least; n <= most; ++n) {
        const int64_t items = nQT * n;
        const int64_t rounds = (items + kMineGrid - 1) / kMineGrid;
        const double fill = static_cast<double>(items) / static_cast<double>(rounds * kMineGrid);
        if (fill >= best_fill - 0.02) { best_fill = fill > best_fill ? fill : best_fill; best = static_cast<int>(n); }
    }
    return best;
}

// Label tiles of a phase behind a dense one, which starts at tile `lo` of nLT: equal growth to the end by at most 8.5, and so
// that the candidates of a query stay within what the select holds in registers (1024), in whole multiples of the slices, so
// that every slice of the phase has the same number of tiles.  By at most 3 where the tiles so far were 512 per compute unit:
// a phase then lasts many times what the select between two of them takes, and every score that passes makes its wave look
// through a block of accumulators (45.6 M x 120 bf16, 18 834 queries, k = 50, growth 7: the last phase alone 8 ms longer
// than with a threshold that lets through 221 scores per query instead of 300).
static int64_t even_phase_tiles(int64_t lo, int64_t nLT, int64_t nQT, int k, int slices) {
    const double ratio = static_cast<double>(nLT) / static_cast<double>(lo);
    double most = 960.0 / k;
    most = most > 8.5 ? 8.5 : most;
    if (lo * nQT >= 512 * kMineGrid && most > 3.0) most = 3.0;
    const int m = static_cast<int>(ceil(log(ratio) / log(most) - 0.01));
    if (m <= 1) return nLT - lo;
    const double want = static_cast<double>(lo) * (pow(ratio, 1.0 / m) - 1.0);
    int64_t n = static_cast<int64_t>(want / slices + 0.5) * slices;
    if (n < slices) n = slices;
    return n < nLT - lo ? n : nLT - lo;
}

// End of a phase on fp16 copies that starts at tile `lo` with thresholds from `seen` tiles (the dense ones are swept again): even growth
// as above, a quarter less because more passes than by exact scores.
static int64_t half_phase_end(int64_t lo, int64_t seen, int64_t nLT, int64_t nQT, int k, int slices) {
    const double ratio = static_cast<double>(nLT) / static_cast<double>(seen);
    double most = 720.0 / k;
    most = most > 8.5 ? 8.5 : most;
    if (seen * nQT >= 512 * kMineGrid && most > 3.0) most = 3.0;
    const int m = static_cast<int>(ceil(log(ratio) / log(most + 1.0) - 0.01));
    if (m <= 1) return nLT;
    const int64_t end = static_cast<int64_t>(static_cast<double>(seen) * pow(ratio, 1.0 / m));
    while (slices > kXcds && end - lo < 2 * slices) slices /= 2;
    int64_t n = (end - lo + slices / 2) / slices * slices;
    if (n < slices) n = slices;
    return lo + n;
}

// Work items of 512 queries (the row kernel with all eight waves along the queries) stage half the
// bytes of W per flop, but there are half as many of them: they are taken where they keep the 32 compute
// units of an XCD busy with one label slice (nine in ten over all rounds), as well as items of 256 would.  Measured, 256 against 512:
// 4 M x 256, k = 50: 512 queries 1.90 : 3.43 ms, 2048 4.25 : 4.53, 8192 14.9 : 14.9, 16 384 28.8 : 28.0;
// 1.3 M x 128: 4096 queries 2.31 : 2.46 ms, 16 384 8.2 : 7.6.  XC_MINE_ROWS=narrow or wide in the
// environment (read at every call) overrides the rule, for A/B timing and for tests.
static bool force_rows_layout() {
    const char* e = getenv("XC_MINE_ROWS");
    return e != nullptr && (e[0] == 'n' || e[0] == 'w');
}
static bool rows_wide_items(int64_t Zq) {
    if (force_rows_layout()) return getenv("XC_MINE_ROWS")[0] == 'w';
    const int64_t wide = (Zq + 2 * kBN - 1) / (2 * kBN), narrow = (Zq + kBN - 1) / kBN;
    // the share of an XCD's compute units that one slice's items keep busy, over all rounds
    const int64_t rw = (wide + kCusPerXcd - 1) / kCusPerXcd, rn = (narrow + kCusPerXcd - 1) / kCusPerXcd;
    const double busy_w = static_cast<double>(wide) / static_cast<double>(rw * kCusPerXcd);
    const double busy_n = static_cast<double>(narrow) / static_cast<double>(rn * kCusPerXcd);
    return busy_w >= 0.9 && busy_w >= 0.94 * busy_n;
}

// Which fp32 searches run on fp16 copies, of those that the search of few queries does not take: by estimates of both times in us,
// least squares over 150 searches of 416 to 65 536 queries, 1100 to 300 000 rows of 16 to 972 elements, k = 5 to 128 (within a
// seventh for half of them).  What the copies save is fp32 products; what they cost is per query: thresholds, lists, scores formed
// again.  With a sixth in favour of the fp32 kernels none of the 150 is slower than with them, and 4 % are lost over always choosing right;
// rows that make most lists run over pay for both (all rows equal 1.05 to 1.1 times the fp32 kernels' time, in hundreds of copies each 1.7).
// fp32 : copies in ms, 10 240 queries x 131 072 x 768, k = 64 15.1 : 3.0, from thresholds 14.4 : 2.6; 4096 x 1.3 M x 256, k = 100
// 19.6 : 3.8; 20 000 x 300 000 x 300, k = 32 33.7 : 5.0; 2500 x 4 M x 64, k = 50 12.1 : 3.2; 60 000 x 9000 x 300, k = 8 4.0 : 2.3; the
// other way 60 000 x 4096 x 64, k = 100 0.88 : 1.84; 20 000 x 4096 x 300, k = 100 0.95 : 0.74.  Below 2048 labels there is no dense phase to find
// thresholds with (47 767 x 1292 x 972, k = 89: 1.8 : 3.1).
constexpr int64_t kBriefStages = 40000;      // 256 x 256 x 32 products in fp32: about 2 ms
static void plan_half(int64_t Zq, int64_t L, int64_t row_bytes, int k, xc_dtype t, HalfPlan* p) {
    p->pitch = 0;
    p->bytes = 0;
    if (t != XC_F32 || row_bytes > kHalfMaxRowBytes || Zq <= kBN || L < 8 * kBM) return;
    {
        const double z = 1e-3 * Zq, cells = static_cast<double>((Zq + kBN - 1) / kBN * kBN) * static_cast<double>((L + kBM - 1) / kBM * kBM);
        const double copies = 79.0 + z * (12.9 + 0.193 * k) + 0.50e-6 * cells + 0.85e-9 * 2.0 * cells * ((row_bytes + 255) / 256 * 64) +
                              1.21e-6 * L * row_bytes + 8.8e-6 * z * k * row_bytes;
        const double fp32 = 63.0 + z * (4.9 + 0.0325 * k) + 0.43e-6 * cells + 10.5e-9 * 2.0 * cells * ((row_bytes + 127) / 128 * 32) + 0.041 * row_bytes;
        if (copies > 0.85 * fp32) return;
    }
    const int64_t nLT = (L + kBM - 1) / kBM, nq = (Zq + kBN - 1) / kBN * kBN;
    p->pitch = (row_bytes / 2 + kStageBytes - 1) / kStageBytes * kStageBytes;
    const int64_t fit = kHalfChunkBytes / (p->pitch * kBM);
    p->chunk = fit < nLT ? fit : nLT;
    size_t off = 0;
    auto take = [&off](size_t bytes) { const size_t o = off; off += round_up(bytes, 256); return o; };
    p->off_rows = take(static_cast<size_t>(p->chunk) * kBM * p->pitch);
    p->off_z = take(static_cast<size_t>(nq) * p->pitch);
    p->off_zpar = take(static_cast<size_t>(nq) * sizeof(float2));
    p->off_err = take(static_cast<size_t>(nLT) * sizeof(float));
    p->off_range = take(256);
    p->off_skip = take(static_cast<size_t>(nq / kBN) * sizeof(int32_t));
    p->bytes = off;
}

static int plan_mine(int64_t Zq, int64_t L, int d, int k_h, xc_dtype t, MinePlan* p) {
    if (t != XC_F32 && t != XC_BF16) return XC_EDTYPE;
    if (Zq < 1 || L < 1 || d < 1 || k_h < 1 || k_h > XC_MAX_K_MINE || k_h > L) return XC_ESHAPE;
    const int64_t row_bytes = static_cast<int64_t>(d) * (t == XC_F32 ? 4 : 2);
    if (row_bytes % 16 != 0 || row_bytes > (1 << 20)) return XC_ESHAPE;
    if (L > 0x7fffffffLL || Zq > 0x7fffffffLL) return XC_ESHAPE;
    int kcap = 8;
    while (kcap < k_h) kcap <<= 1;
    p->kcap = kcap;
    p->nkb = static_cast<int>((row_bytes + kStageBytes - 1) / kStageBytes);
    p->nQT = (Zq + kBN - 1) / kBN;
    p->nLT = (L + kBM - 1) / kBM;
    // a phase appends at most kcap keys per slice to a list that holds at most k keys
    p->glist_cap = kcap * (slices_cap(kcap) + 1);
    size_t off = 0;
    auto take = [&off](size_t bytes) { size_t o = off; off += round_up(bytes, 256); return o; };
    const size_t nq = static_cast<size_t>(p->nQT) * kBN;
    // first word: 1 if the last warm search, or the last on fp16 copies, had to repeat the full search for some query tile; then one word per
    // tile (rounded up to 64 words: few queries have kRedoWord behind them)
    p->off_flag = take(4 * (static_cast<size_t>(p->nQT) + 1));
    p->off_lists = take(static_cast<size_t>(kMineGrid) * kBN * kCandCap * sizeof(uint64_t));
    p->off_glist = take(nq * p->glist_cap * sizeof(uint64_t));
    p->off_gcnt = take(nq * sizeof(int32_t));
    p->off_tau = take(nq * sizeof(uint32_t));
    p->off_zero = take(256);
    p->ws_min = off;
    if (plan_q8(Zq, L, row_bytes, t, &p->q8)) off += p->q8.bytes;
    plan_half(Zq, L, row_bytes, k_h, t, &p->half);
    off += p->half.bytes;
    p->ws_bytes = off;
    p->lds_tile = 2 * static_cast<size_t>(kBM + kBN) * kStageBytes + kBN * 8 + kMineWaves * 256 * 4 +
                  static_cast<size_t>(kMineWaves) * kPool * 8 + 16;
    return XC_OK;
}

}  // namespace xc

extern "C" int xc_mine_workspace(int64_t Zq, int64_t L, int d, int k_h, xc_dtype t, size_t* bytes) {
    if (!bytes) return XC_EINVAL;
    xc::MinePlan p;
    const int rc = xc::plan_mine(Zq, L, d, k_h, t, &p);
    if (rc != XC_OK) return rc;
    *bytes = p.ws_bytes;
    return XC_OK;
}

namespace xc {
// The search proper.  warm: one sweep with the thresholds found in the workspace (lowered by
// rel_margin * |tau|), then the full search if some query came out short; the kernels of the full
// search are enqueued in any case and return at once when the flag says they are not needed.
// Slices per XCD at most: every slice has a tile, and the global lists have room for what each of them appends.
static int most_slices_per_xcd(int64_t nT, int kcap) {
    int sx = 8;
    while (sx > 1 && (nT < static_cast<int64_t>(kXcds) * sx || kXcds * sx > slices_cap(kcap))) sx >>= 1;
    return sx;
}

static int run_mine(const void* Z, const void* W, int64_t Zq, int64_t L, int d, int k_h, xc_dtype t,
                    bool warm, float rel_margin, int32_t* shortlist, float* scores, void* ws,
                    size_t ws_bytes, void* stream) {
    MinePlan p;
    const int rc = plan_mine(Zq, L, d, k_h, t, &p);
    if (rc != XC_OK) return rc;
    if (!Z || !W || !shortlist || !ws) return XC_EINVAL;
    if (warm && !(rel_margin >= 0.0f)) return XC_EINVAL;
    if (!aligned16(Z) || !aligned16(W) || !aligned16(ws)) return XC_EINVAL;
    if (ws_bytes < p.ws_min) return XC_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned char* w8 = static_cast<unsigned char*>(ws);
    MineArgs a;
    a.Z = static_cast<const unsigned char*>(Z);
    a.W = static_cast<const unsigned char*>(W);
    a.Zq = Zq; a.L = L;
    a.row_bytes = static_cast<int64_t>(d) * (t == XC_F32 ? 4 : 2);
    a.k = k_h; a.kcap = p.kcap; a.nkb = p.nkb;
    a.nQT = p.nQT;
    a.glist_cap = p.glist_cap;
    a.lists = reinterpret_cast<uint64_t*>(w8 + p.off_lists);
    a.glist = reinterpret_cast<uint64_t*>(w8 + p.off_glist);
    a.gcnt = reinterpret_cast<int32_t*>(w8 + p.off_gcnt);
    uint32_t* tau_g = reinterpret_cast<uint32_t*>(w8 + p.off_tau);
    a.tau_g = tau_g;
    a.zeros = w8 + p.off_zero;
    a.cond = nullptr;
    a.dense = nullptr;
    a.dense_ld = 0;
    a.items = nullptr;
    a.over = nullptr;
    a.skip = nullptr;
    a.tile_err = nullptr;
    a.err_range = nullptr;
    a.z_rows = Zq;
    a.w_rows = L;
    int32_t* flag = reinterpret_cast<int32_t*>(w8 + p.off_flag);

    // raise the dynamic LDS limit of the tile kernels: once per device and process (the attribute
    // belongs to the device's copy of the kernel)
    static std::mutex attr_mu;
    static uint64_t attr_done_mask = 0;          // bit = device ordinal (< 64)
    {
        int dev = 0;
        XC_HIP_CHECK(hipGetDevice(&dev));
        std::lock_guard<std::mutex> lock(attr_mu);
        if (dev < 0 || dev >= 64 || !(attr_done_mask & (1ull << dev))) {
            const void* fns[10] = {reinterpret_cast<const void*>(&mine_tile_kernel<half_t, false, true>),
                                  reinterpret_cast<const void*>(&mine_tile_kernel<half_t, false, false>),
                                  reinterpret_cast<const void*>(&mine_tile_kernel<bf16_t, false, true>),
                                  reinterpret_cast<const void*>(&mine_tile_kernel<bf16_t, true, true>),
                                  reinterpret_cast<const void*>(&mine_tile_kernel<float, false, true>),
                                  reinterpret_cast<const void*>(&mine_tile_kernel<float, true, true>),
                                  reinterpret_cast<const void*>(&mine_tile_kernel<bf16_t, false, false>),
                                  reinterpret_cast<const void*>(&mine_tile_kernel<bf16_t, true, false>),
                                  reinterpret_cast<const void*>(&mine_tile_kernel<float, false, false>),
                                  reinterpret_cast<const void*>(&mine_tile_kernel<float, true, false>)};
            for (const void* fn : fns)
                XC_HIP_CHECK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 static_cast<int>(p.lds_tile)));
            for (const RowsKernel& k : kRowsKernels)
                for (const RowsKernelFn fn : {k.fn, k.varied})
                    if (fn != nullptr)
                        XC_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize,
                                                         static_cast<int>(rows_lds_bytes(k.wm))));
            int rca = few_raise_lds();
            if (rca == XC_OK) rca = q8_raise_lds();
            if (rca != XC_OK) return rca;
            if (dev >= 0 && dev < 64) attr_done_mask |= 1ull << dev;
        }
    }
    // few queries: W is read once and the group maxima take the place of thresholds and lists.  A warm search of one
    // query tile has nothing to gain there and nothing to repeat; of more, its one sweep is the better way.
    FewPlan few;
    const bool half = p.half.pitch > 0 && ws_bytes >= p.ws_bytes && !force_general_kernel() && !force_rows_layout();
    if (!(warm && Zq > kBN) && !force_general_kernel() && !force_rows_layout() &&
        plan_few(Zq, L, a.row_bytes, k_h, t, warm, half, p.off_glist - p.off_lists, &few))
        return run_mine_few(few, Z, W, Zq, L, a.row_bytes, k_h, t, w8 + p.off_lists, tau_g,
                            warm ? flag : nullptr, static_cast<int>(p.nQT) + 1, flag + kRedoWord, shortlist, scores, st);

    const int64_t nq = p.nQT * kBN;
    const dim3 init_grid(static_cast<unsigned>((nq + 255) / 256));
    const dim3 select_grid(static_cast<unsigned>((Zq + kSelectWaves - 1) / kSelectWaves));
    uint32_t* zeros32 = reinterpret_cast<uint32_t*>(w8 + p.off_zero);

    // bf16 rows of whole stages whose queries fit a wave's registers take the row kernel: work items of
    // 512 queries where the pool fills them about as well as items of 256
    const RowsKernel* rk = nullptr;
    if (t == XC_BF16 && a.row_bytes % kStageBytes == 0 && !force_general_kernel()) {
        const int nk = static_cast<int>(a.row_bytes / kStageBytes);
        rk = find_rows_kernel(nk, rows_wide_items(Zq) ? 1 : 2, false);
    }

    // the split of label tiles [lo, hi) over the compute units
    auto split = [&](int64_t lo, int64_t hi, const RowsKernel* rk) {
        const int64_t nT = hi - lo;
        const bool rows_kernel = rk != nullptr;
        a.nQT = rows_kernel ? (Zq + 2 * kBN / rk->wm - 1) / (2 * kBN / rk->wm) : p.nQT;
        if (nT >= kXcds) {
            // slices per XCD: as many as the phase supports, so that few query tiles are in
            // flight per XCD and their Z rows stay in that XCD's L2
            int Sx = most_slices_per_xcd(nT, p.kcap);
            if (rows_kernel) Sx = rows_slices_per_xcd(a.nQT, nT, Sx);
            a.S = kXcds * Sx;
            a.Qx = kCusPerXcd / Sx;
        } else {                                           // a few tiles: one slice per tile, plain order
            a.S = static_cast<int>(nT);
            a.Qx = 0;
        }
        a.tile_lo = lo; a.tile_hi = hi;
        a.tiles_per_slice = (nT + a.S - 1) / a.S;
        a.append_max = (p.glist_cap - p.kcap) / a.S;
        if (a.append_max > kCandCap) a.append_max = kCandCap;
    };
    // one phase: the tile kernel over label tiles [lo, hi), then the select
    auto sweep = [&](int64_t lo, int64_t hi, const int32_t* cond, const int32_t* items) -> int {
        const bool rows_kernel = rk != nullptr;
        split(lo, hi, rk);
        a.items = items;
        a.cond = cond;
        const bool ktail = (a.row_bytes % kStageBytes) != 0;
        if (rows_kernel) {
            // the query tile stays in registers, only W is streamed
            XC_LAUNCH(K_MINE_TILE, st, (rk->fn<<<kMineGrid, kMineThreads, rows_lds_bytes(rk->wm), st>>>(a)));
        } else if (t == XC_BF16) {
            if (ktail) XC_LAUNCH(K_MINE_TILE, st, (mine_tile_kernel<bf16_t, true, false><<<kMineGrid, kMineThreads, p.lds_tile, st>>>(a)));
            else XC_LAUNCH(K_MINE_TILE, st, (mine_tile_kernel<bf16_t, false, false><<<kMineGrid, kMineThreads, p.lds_tile, st>>>(a)));
        } else {
            if (ktail) XC_LAUNCH(K_MINE_TILE, st, (mine_tile_kernel<float, true, false><<<kMineGrid, kMineThreads, p.lds_tile, st>>>(a)));
            else XC_LAUNCH(K_MINE_TILE, st, (mine_tile_kernel<float, false, false><<<kMineGrid, kMineThreads, p.lds_tile, st>>>(a)));
        }
        XC_HIP_CHECK(hipGetLastError());
        return XC_OK;
    };
    auto select = [&](int64_t hi, const int32_t* cond, int32_t* short_flag) -> int {
        const int final_phase = hi == p.nLT ? 1 : 0;
        XC_LAUNCH(K_MINE_SELECT, st, (mine_select_kernel<<<select_grid, kSelectWaves * kWave, 0, st>>>(
            a.glist, a.gcnt, tau_g, Zq, p.glist_cap, k_h, final_phase, shortlist, scores, cond, short_flag)));
        XC_HIP_CHECK(hipGetLastError());
        return XC_OK;
    };

    auto dense_select = [&](int n0) {
        if (n0 <= kDenseMin)
            XC_LAUNCH(K_MINE_SELECT, st, (mine_dense_select_kernel<kDenseMin><<<select_grid, kSelectWaves * kWave, 0, st>>>(
                a.dense, a.dense_ld, a.glist, a.gcnt, tau_g, Zq, p.glist_cap, k_h, a.tile_err, a.cond)));
        else if (n0 <= 8)
            XC_LAUNCH(K_MINE_SELECT, st, (mine_dense_select_kernel<8><<<select_grid, kSelectWaves * kWave, 0, st>>>(
                a.dense, a.dense_ld, a.glist, a.gcnt, tau_g, Zq, p.glist_cap, k_h, a.tile_err, a.cond)));
        else
            XC_LAUNCH(K_MINE_SELECT, st, (mine_dense_select_kernel<kDenseTiles><<<select_grid, kSelectWaves * kWave, 0, st>>>(
                a.dense, a.dense_ld, a.glist, a.gcnt, tau_g, Zq, p.glist_cap, k_h, a.tile_err, a.cond)));
    };

    auto dense_phase = [&](int n0, const int32_t* cond) -> int {
        a.nQT = p.nQT;
        a.tile_lo = 0; a.tile_hi = n0; a.tiles_per_slice = 1;
        a.S = n0; a.Qx = 0;
        a.dense = reinterpret_cast<float*>(w8 + p.off_lists);
        a.dense_ld = n0 * kBM;
        a.cond = cond;
        const bool ktail = (a.row_bytes % kStageBytes) != 0;
        if (t == XC_BF16) {
            if (ktail) XC_LAUNCH(K_MINE_TILE, st, (mine_tile_kernel<bf16_t, true, true><<<kMineGrid, kMineThreads, p.lds_tile, st>>>(a)));
            else XC_LAUNCH(K_MINE_TILE, st, (mine_tile_kernel<bf16_t, false, true><<<kMineGrid, kMineThreads, p.lds_tile, st>>>(a)));
        } else {
            if (ktail) XC_LAUNCH(K_MINE_TILE, st, (mine_tile_kernel<float, true, true><<<kMineGrid, kMineThreads, p.lds_tile, st>>>(a)));
            else XC_LAUNCH(K_MINE_TILE, st, (mine_tile_kernel<float, false, true><<<kMineGrid, kMineThreads, p.lds_tile, st>>>(a)));
        }
        XC_HIP_CHECK(hipGetLastError());
        dense_select(n0);
        XC_HIP_CHECK(hipGetLastError());
        return XC_OK;
    };

    auto phase = [&](int64_t lo, int64_t hi, const int32_t* cond, int32_t* short_flag) -> int {
        const int rcs = sweep(lo, hi, cond, nullptr);
        return rcs != XC_OK ? rcs : select(hi, cond, short_flag);
    };

    // fp32 on fp16 copies; then what these did not settle, in two phases of the fp32 kernels
    if (half) {
        const HalfPlan& hp = p.half;
        unsigned char* hw = w8 + p.ws_min;
        unsigned char* rows = hw + hp.off_rows;
        float2* zpar = reinterpret_cast<float2*>(hw + hp.off_zpar);
        float* tile_err = reinterpret_cast<float*>(hw + hp.off_err);
        uint32_t* range = reinterpret_cast<uint32_t*>(hw + hp.off_range);
        float* scale = reinterpret_cast<float*>(range) + 32;         // of W's copies
        int32_t* over = flag;
        int32_t* skip = reinterpret_cast<int32_t*>(hw + hp.off_skip);
        const int row_bytes = static_cast<int>(a.row_bytes), pitch = static_cast<int>(hp.pitch);
        int LG = 8;
        while (LG < kWave && LG * 16 < pitch) LG <<= 1;
        const MineArgs exact = a;
        a.Z = hw + hp.off_z;
        a.row_bytes = pitch;
        a.nkb = pitch / kStageBytes;
        a.z_rows = nq;
        a.over = over;
        a.skip = skip;
        a.tile_err = tile_err;
        a.err_range = range;
        const RowsKernel* hk = pitch <= kMaxRowKernelBytes ? find_rows_kernel(pitch / kStageBytes, rows_wide_items(Zq) ? 1 : 2, true) : nullptr;
        int64_t chunk_end = 0;
        auto convert = [&]() -> int {                        // the next chunk's copies
            const int64_t lo = chunk_end;
            chunk_end = lo + hp.chunk < p.nLT ? lo + hp.chunk : p.nLT;
            const int64_t n_rows = (chunk_end - lo) * kBM, n_lab = (L < chunk_end * kBM ? L : chunk_end * kBM) - lo * kBM;
            // rows a workgroup converts at a time: 131 072 x 768 64 rows 111 us, 128 103, 256 154; 131 072 x 256 43, 37 and 45
            const int unit = n_rows >= (1 << 16) ? 128 : 64;
            const int64_t blocks = n_rows / unit;
            XC_LAUNCH(K_MINE_TILE, st, (half_rows_kernel<<<static_cast<unsigned>(blocks < 2048 ? blocks : 2048), 256, 0, st>>>(
                exact.W + lo * kBM * row_bytes, n_lab, n_rows, row_bytes, pitch, LG, unit, rows, tile_err + lo, scale)));
            XC_HIP_CHECK(hipGetLastError());
            a.W = reinterpret_cast<const unsigned char*>(reinterpret_cast<uintptr_t>(rows) - static_cast<uintptr_t>(lo * kBM * pitch));    // (row numbers count from 0)
            a.w_rows = chunk_end * kBM;
            return XC_OK;
        };
        XC_LAUNCH(K_MINE_TILE, st, (half_queries_kernel<<<static_cast<unsigned>(nq / 4 + 1), 256, 0, st>>>(
            exact.Z, Zq, nq, row_bytes, pitch, hw + hp.off_z, zpar, tile_err, p.nLT, over, skip, exact.W, L, scale, zeros32)));
        XC_HIP_CHECK(hipGetLastError());
        int rch = convert();
        if (rch != XC_OK) return rch;
        const int n0 = warm ? 0 : dense_tiles(p.nQT, L / kBM < chunk_end ? L / kBM : chunk_end, k_h, p.off_glist - p.off_lists, true);
        if (n0 > 0) {                                        // only for its thresholds: its labels are swept with the others
            a.nQT = p.nQT;
            a.tile_lo = 0; a.tile_hi = n0; a.tiles_per_slice = 1;
            a.S = n0; a.Qx = 0;
            a.dense = reinterpret_cast<float*>(w8 + p.off_lists);
            a.dense_ld = n0 * kBM;
            XC_LAUNCH(K_MINE_TILE, st, (mine_tile_kernel<half_t, false, true><<<kMineGrid, kMineThreads, p.lds_tile, st>>>(a)));
            XC_HIP_CHECK(hipGetLastError());
            dense_select(n0);
            XC_HIP_CHECK(hipGetLastError());
        }
        XC_LAUNCH(K_MINE_SELECT, st, (half_start_kernel<<<static_cast<unsigned>((nq + 256) / 256 + 1), 256, 0, st>>>(
            warm ? 2 : n0 > 0 ? 1 : 0, rel_margin, tau_g, a.gcnt, zpar, over, skip, nq, Zq, tile_err, chunk_end, range, scale)));
        XC_HIP_CHECK(hipGetLastError());
        const int slices = slices_cap(p.kcap);
        int64_t seen = n0;                                   // labels behind the thresholds
        for (int64_t lo = 0; lo < p.nLT;) {
            int64_t hi = p.nLT;
            if (!warm) {
                if (n0 == 0) hi = lo + phase_tiles(lo, p.nQT);
                else hi = half_phase_end(lo, seen, p.nLT, p.nQT, k_h, slices);
                if (hi > p.nLT || (p.nLT - hi) < hi / 4) hi = p.nLT;
            }
            if (hi > chunk_end) hi = chunk_end;
            split(lo, hi, hk);
            a.append_max = kCandCap;                         // (a list is never cut; one that runs over gives its query tile up)
            if (hk != nullptr) {
                XC_LAUNCH(K_MINE_TILE, st, (hk->fn<<<kMineGrid, kMineThreads, rows_lds_bytes(hk->wm), st>>>(a)));
                XC_HIP_CHECK(hipGetLastError());
                XC_LAUNCH(K_MINE_TILE, st, (hk->varied<<<kMineGrid, kMineThreads, rows_lds_bytes(hk->wm), st>>>(a)));
            } else XC_LAUNCH(K_MINE_TILE, st, (mine_tile_kernel<half_t, false, false><<<kMineGrid, kMineThreads, p.lds_tile, st>>>(a)));
            XC_HIP_CHECK(hipGetLastError());
            if (hi < p.nLT) {
                XC_LAUNCH(K_MINE_SELECT, st, (half_select_kernel<<<select_grid, 256, 0, st>>>(a.glist, a.gcnt, tau_g, zpar, tile_err, range, over, skip, Zq, p.glist_cap, k_h)));
                XC_HIP_CHECK(hipGetLastError());
            }
            if (hi == chunk_end && hi < p.nLT) {
                rch = convert();
                if (rch != XC_OK) return rch;
                XC_LAUNCH(K_MINE_SELECT, st, (half_range_kernel<<<1, 256, 0, st>>>(tile_err, chunk_end, range)));
                XC_HIP_CHECK(hipGetLastError());
            }
            lo = hi;
            seen = seen > hi ? seen : hi;
        }
        const size_t zop = static_cast<size_t>((row_bytes + 63) / 64 * 64);
        if (Zq >= kHalfWaveQueries)
            XC_LAUNCH(K_MINE_SELECT, st, (half_finish_kernel<1><<<select_grid, 256, 4 * zop, st>>>(
                exact.Z, exact.W, row_bytes, a.glist, a.gcnt, tau_g, zpar, tile_err, range, scale, over, p.glist_cap, k_h, Zq, shortlist, scores)));
        else
            XC_LAUNCH(K_MINE_SELECT, st, (half_finish_kernel<4><<<static_cast<unsigned>(Zq), 256, zop, st>>>(
                exact.Z, exact.W, row_bytes, a.glist, a.gcnt, tau_g, zpar, tile_err, range, scale, over, p.glist_cap, k_h, Zq, shortlist, scores)));
        XC_HIP_CHECK(hipGetLastError());
        // Then the fp32 search for the tiles flagged, as for a pool that takes no copies but for its phases: while it is short, one behind the
        // dense one (two launches that return at once where nothing is flagged take as long as the second saves)
        a = exact;
        const int m0 = dense_tiles(p.nQT, L / kBM, k_h, p.off_glist - p.off_lists, true);
        if (m0 == 0) {
            mine_init_kernel<<<init_grid, 256, 0, st>>>(tau_g, a.gcnt, nq, zeros32, over);
            XC_HIP_CHECK(hipGetLastError());
        } else {
            rch = dense_phase(m0, over);
            if (rch != XC_OK) return rch;
        }
        const bool brief = m0 > 0 && p.nQT * p.nLT * a.nkb <= kBriefStages;
        for (int64_t lo = m0; lo < p.nLT;) {
            int64_t hi = brief ? p.nLT : lo + (m0 > 0 ? even_phase_tiles(lo, p.nLT, p.nQT, k_h, slices) : phase_tiles(lo, p.nQT));
            if (hi > p.nLT || p.nLT - hi < hi / 4) hi = p.nLT;
            rch = phase(lo, hi, over, nullptr);
            if (rch != XC_OK) return rch;
            lo = hi;
        }
        return XC_OK;
    }

    const int32_t* cond = nullptr;
    if (warm) {
        mine_warm_init_kernel<<<init_grid, 256, 0, st>>>(tau_g, a.gcnt, nq, zeros32, flag, rel_margin);
        XC_HIP_CHECK(hipGetLastError());
        const int rcw = phase(0, p.nLT, nullptr, flag);
        if (rcw != XC_OK) return rcw;
        cond = flag;
    }
    mine_init_kernel<<<init_grid, 256, 0, st>>>(tau_g, a.gcnt, nq, zeros32, cond);
    XC_HIP_CHECK(hipGetLastError());
    int64_t lo = 0;
    const bool q8 = p.q8.nk > 0 && !warm && ws_bytes >= p.ws_bytes && !force_general_kernel() && !force_rows_layout();
    unsigned char* q8_ws = w8 + p.ws_min;
    if (cond == nullptr && rk == nullptr) {
        // the first phase dense, by the general kernel: as many tiles as one or a few full rounds of the compute units take
        const int n0 = dense_tiles(p.nQT, L / kBM, k_h, p.off_glist - p.off_lists, false);
        if (n0 > 0) {
            const int rcd = dense_phase(n0, nullptr);
            if (rcd != XC_OK) return rcd;
            lo = n0;
        }
    }
    if (q8) { const int rcq = q8_begin(p.q8, q8_ws, Z, Zq, st); if (rcq != XC_OK) return rcq; }
    while (lo < p.nLT) {
        if (q8 && lo >= kQ8FirstTile) {
            // a chunk through the 8-bit filter, what that gave up through the bf16 kernel, the select
            int64_t hi = lo + p.q8.chunk / kBM;
            if (hi > lo + kQ8Growth * lo) hi = lo + kQ8Growth * lo;
            if (hi > p.nLT) hi = p.nLT;
            Q8Chunk c;
            c.Z = Z; c.W = W; c.Zq = Zq;
            c.lab0 = lo * kBM;
            c.lab1 = hi * kBM < L ? hi * kBM : L;
            c.kcap = p.kcap; c.glist_cap = p.glist_cap; c.max_slices = slices_cap(p.kcap);
            c.lists = a.lists; c.glist = a.glist; c.gcnt = a.gcnt; c.tau_g = tau_g;
            c.item_tiles = rk->wm == 1 ? 2 : 1;
            c.sweep_tiles = hi - lo;
            c.sx_max = most_slices_per_xcd(hi - lo, p.kcap);
            int rcp = q8_chunk(p.q8, q8_ws, c, st);
            if (rcp == XC_OK) rcp = sweep(lo, hi, q8_flags(p.q8, q8_ws), hi - lo >= kXcds ? q8_items(p.q8, q8_ws) : nullptr);
            if (rcp == XC_OK) rcp = select(hi, nullptr, nullptr);
            if (rcp != XC_OK) return rcp;
            lo = hi;
            continue;
        }
        // phases end at about 1, 8, 64, ... tiles: each sees about 8x the labels seen before it
        int64_t hi = lo + (a.dense != nullptr ? even_phase_tiles(lo, p.nLT, p.nQT, k_h, slices_cap(p.kcap)) : phase_tiles(lo, p.nQT));
        if (hi > p.nLT || p.nLT - hi < hi / 4) hi = p.nLT;      // fold a short remainder into this phase
        const int rcp = phase(lo, hi, cond, nullptr);
        if (rcp != XC_OK) return rcp;
        lo = hi;
    }
    return XC_OK;
}
}  // namespace xc

extern "C" int xc_mine_negatives(const void* Z, const void* W, int64_t Zq, int64_t L, int d, int k_h,
                                 xc_dtype t, int32_t* shortlist, float* scores, void* ws,
                                 size_t ws_bytes, void* stream) {
    return xc::run_mine(Z, W, Zq, L, d, k_h, t, false, 0.0f, shortlist, scores, ws, ws_bytes, stream);
}

extern "C" int xc_mine_negatives_warm(const void* Z, const void* W, int64_t Zq, int64_t L, int d, int k_h,
                                      xc_dtype t, float rel_margin, int32_t* shortlist, float* scores,
                                      void* ws, size_t ws_bytes, void* stream) {
    return xc::run_mine(Z, W, Zq, L, d, k_h, t, true, rel_margin, shortlist, scores, ws, ws_bytes, stream);
}
