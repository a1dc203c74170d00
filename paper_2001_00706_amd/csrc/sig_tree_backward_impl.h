// Gradient of the signature with respect to the path, prefix-tree family (d = 2..8 at N = 2..9, d = 9..16 at N = 2..6,
// final and stream mode): the recurrences of sig_backward.hip with no communication between threads, so that the
// state of one path can be spread over any number of workgroups (paper section 5.3, appendix C).
//
// A thread stands for a word u of P = N - U letters and owns the subtree of the words u c and u c c'
// below it (U = 2 levels, in registers; U = 1 beyond 8 channels), exactly as in sig_tree_impl.h.
//   * "Up" (undo the increment, Horner terms T^(k)_i) needs the signature at the prefixes of u only; every
//     thread carries its own copy of them.
//   * "Down" moves cotangent from a word to its prefixes, D^(k)_{i-1}[p] = sum_c D^(k)_i[p c] z[c]/(k-i+1).
//     Inside the subtree that sum is local.  Above it, the map from the output cotangent to the gradient is
//     linear, so the cotangent of a prefix may stay split into the parts that arrived through each thread:
//     a thread keeps, for each of its prefixes, only the part that came up through its own word, and the
//     gradient of an increment is the sum of every thread's contribution.  (The cotangent a prefix has of
//     its own in the output gradient is given to the first thread below it.)
//   * That one sum, over all threads of a path and per increment, is finished by a second kernel: every
//     workgroup (for paths of at most one wavefront: every word, or every word of P-1 letters) writes its partial
//     sums to a workspace [row][group][increment][d].
//
// Horner terms and cotangents are carried with their factorials taken out, Hh^(k)_j = T^(k)_j / (k-j)! and
// Dh^(k)_j = D^(k)_j (k-j)!: then Hh^(k)_j = Hh^(k)_{j-1} z + A_j / (k-j)!, Dh^(k)_{j-1} = Dh^(k)_j z, and a word's contribution to
// its last letter is sum_k Hh^(k)_{j-1} Dh^(k)_j, with a constant factor left only in A_j / (k-j)! and in what a prefix
// receives, sum_k Dh^(k)_j / (k-j)!.
//
// Up to 8 channels (short paths: where tb_packed_rows says; long ones in fp64: where tb_wide_rows does) nothing is summed over lanes while an increment is worked on: a
// lane leaves its d + P numbers (the subtree's share of every channel, the shares of the word's own letters) in LDS, and
// after kBatch increments a lane per (increment, group) adds up the rows of a group, the d words that share their first
// P-1 letters.  There the last letter is known from the row and the others are the group's, so they are sorted into
// channels once per group and batch, not once per word and increment.  What bounds the kernel is the issue of vector
// instructions: per wavefront and increment 430 of them at d = N = 7 with the sums formed by lane exchanges, 330 this way
// (732 -> 520 us with the closing sums for 32 paths of 128 points; d = 5, N = 7: 157 -> 95; d = 6, N = 6: 163 -> 90; 128 paths of 64 points at
// d = 7, N = 5: 92 -> 46).
#ifndef SIG_TREE_BACKWARD_IMPL_H_
#define SIG_TREE_BACKWARD_IMPL_H_

#include "sig_internal.h"
#include "sig_lane_ops.h"
#include "sig_stretch_ops.h"

#include <type_traits>

namespace sig {
namespace {


constexpr int kTbTile = 32;      // increments staged in LDS at a time
constexpr int kTbMaxPaths = 16;  // paths that may share a workgroup
constexpr int kStretchRadixLog2 = 3, kStretchLevels = 6;   // 8 stretches to a node, nodes of up to 8^5 stretches
constexpr int kStretchStage = 32 * 1024;                   // bytes of them in LDS at a time, at least

__host__ __device__ constexpr int64_t tb_off(int d, int k)   // offset of level k (1-based) in a flat element
{
    int64_t off = 0, p = 1;
    for (int j = 1; j < k; ++j) {
        p *= d;
        off += p;
    }
    return off;
}

// ROWS: the lanes' numbers go through LDS; otherwise sums by lane exchanges.
template <typename T, int D, int N, bool ROWS>
struct TbShape {
    // levels kept per thread below its word: two (d + d^2 scalars) up to 8 channels, one (d scalars) beyond
    static constexpr int U = N - 1 < (D <= 8 ? 2 : 1) ? N - 1 : (D <= 8 ? 2 : 1);
    static constexpr int P = N - U;
    static constexpr int64_t kWords = tb_off(D, P + 1) - tb_off(D, P);   // threads a path needs
    static constexpr bool kMulti = kWords >= 256;   // a path spans several workgroups
    // From 65 words on, a path takes whole wavefronts (2..4, idle lanes at the end), each of which sums up an increment's
    // gradient, and the sums meet in LDS once per tile: one partial sum per path and workgroup.  Shorter paths are packed
    // one after the other, and every group or thread writes its own part.
    static constexpr bool kWide = kWords > 64;
    static constexpr bool kRows = ROWS;
    // Lanes of a wavefront in use, and the groups of d words they hold.  Packed paths get whole groups; the wavefronts
    // of a longer path take 64 words each, so that a group may be split between two (its sums are then formed in two parts).
    static constexpr int kLanes = kRows && !kWide ? 64 / D * D : 64;
    static constexpr bool kSplit = kRows && kWide && 64 % D != 0;
    static constexpr int kGroups = !kRows ? 1 : kSplit ? (64 + D - 2) / D + 1 : 64 / D;
    static constexpr int kWavesPerPath = kMulti ? 4 : int((kWords + 63) / 64);
    static constexpr int kPathsPerGroup =
        kWide ? (kMulti ? 1 : 4 / kWavesPerPath) : (4 * kLanes / kWords < kTbMaxPaths ? int(4 * kLanes / kWords) : kTbMaxPaths);
    static constexpr int64_t kGroupsPerPath = kMulti ? (kWords + 255) / 256 : 1;   // workgroups per path
    static constexpr int64_t kPartials = kWide ? kGroupsPerPath : kRows ? kWords / D : kWords;   // partial sums per path and increment
    static constexpr int64_t kPartialsRoom = kWide ? kGroupsPerPath : kWords;                    // ... that the workspace has room for
    static constexpr int64_t kS = tb_off(D, N + 1);
    // a lane's row: d channels, the last letter's share, those of the letters before it
    static constexpr int kVec = 16 / int(sizeof(T));             // scalars of a 16-byte access
    static constexpr int kRow = kRows ? (D + P + kVec - 1) / kVec * kVec : kVec;
    static constexpr int kZRow = (D + kVec - 1) / kVec * kVec;   // scalars an increment takes in LDS
    // Groups lie an odd number of 16-byte pieces apart, so that the lanes that read them side by side hit different banks
    // (d = 4 in fp64, 128 paths of 128 points at N = 5: 77 us, without this 125).
    static constexpr int kGroupPad = kRows && D * kRow / kVec % 2 == 0 ? kVec : 0;
    static constexpr int kIncSize = kLanes * kRow + kGroups * kGroupPad;   // scalars an increment of the batch takes
    // increments per batch: a lane per (increment, group), as many as leave room for three workgroups on a compute unit
    static constexpr int kOther = int(sizeof(T)) * (kPathsPerGroup * kTbTile * kZRow + (kWide ? kTbTile * 4 * D : 1) + kRow);
    static constexpr int kRoom = (53 * 1024 - kOther) / (4 * kIncSize * int(sizeof(T)));
    static constexpr int kBatch = !kRows ? 1 : kRoom < 64 / kGroups ? (kRoom < 1 ? 1 : kRoom) : 64 / kGroups;
    static constexpr int kRowsSize = kRows ? 4 * kBatch * kIncSize + kRow : 1;   // with a row of zeros
    // Stretches: the same LDS holds their signatures before the walk, where there is room for enough of them.
    static constexpr int kStage = kRowsSize > int(kStretchStage / sizeof(T)) ? kRowsSize : int(kStretchStage / sizeof(T));
    static constexpr int kStagedNodes = int(kStage / tb_off(D, N));
    static constexpr bool kNodesInLds = kStagedNodes >= 16;
};

// Orders a wavefront's own LDS writes before its reads of what other lanes wrote (LDS serves a wavefront in order; this keeps
// the compiler from moving accesses across).
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

__host__ __device__ constexpr double inv_factorial(int n)
{
    double f = 1;
    for (int i = 2; i <= n; ++i) f *= i;
    return 1 / f;
}

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// What a launch walks back over.
enum TbMode {
    kTbFinal,      // whole paths, from the gradient with respect to the signature
    kTbStream,     // whole paths, the gradient arriving at every prefix
    kTbStretches,  // final mode, every row one of the `chunks` stretches of its path (Shape::chunks): see StretchRows
    kTbStreamStretches,   // stream mode, the same; stretches of chunk_len increments counted from the end of the path
};

// A walk over stretches (the gradient of paths that leave the chip idle, cut along their length; sig_backward_chunked.hip says why
// and from what a stretch is walked).  Only the levels below the top take part in the products around it: a word of the top
// level has no room for a suffix, and what it holds itself is not read.  A thread holds every prefix of its words, and the
// cotangents of prefixes are split over the threads anyway, so each thread forms its share of the products by itself
// (sig_stretch_ops.h): no launches for rounds of products, no copies of the points, and the increments' gradients land where one walk
// over the whole path would leave them.  Before, with the products along a tree of launches | now: 256 paths of 100 points at d = 6,
// N = 4 (one piece 53 us) 53 | 29 us; 110 x 239, d = 7, N = 4 129 | 42; 1 x 65 537, d = 4, N = 6 194 | 130; 1 x 832, d = 3, N = 7 80 | 52; 5 x 1775, d = 4,
// N = 3 46 | 28; 817 shapes 0.64 of the time.  What bounds it: the walk's latency per increment, two trips to memory
// ahead of it, 0.5 us a step of products from LDS, 1 to 2 from memory.
//
// The signatures of the stretches below the top level, [rows][levels below N], and of groups of them: a node of a level is the
// product of kStretchRadix neighbours of the level below (fewer at the end of a path).  A row first forms the signature of its
// path up to its end and the gradient with respect to it: it multiplies together what comes before, the largest nodes first, and
// carries the gradient back through what comes after, the largest and last first.
template <typename T>
struct StretchRows {
    int levels;                            // of which level 0 is the stretches themselves
    int count[kStretchLevels];             // nodes of a level per path
    const T *at[kStretchLevels];
    const T *carried;                      // stream mode: [rows][P + D + D^2][words], see sig_stream_carry_kernel
};

// An address that is the same for all lanes of the wavefront, in scalar registers.
template <typename T>
__device__ __forceinline__ const T *wave_uniform(const T *p)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(a)), hi = __builtin_amdgcn_readfirstlane(uint32_t(a >> 32));
    return reinterpret_cast<const T *>(uint64_t(hi) << 32 | lo);
}

// chunk_view with 32-bit divisions (a 64-bit one takes some 0.3 us of a lone wavefront's time); less than 2^31 rows.
__device__ __forceinline__ ChunkView stretch_view(uint32_t row, const Shape &sh)
{
    const uint32_t path = row / uint32_t(sh.chunks);
    const int64_t inc0 = int64_t(row - path * uint32_t(sh.chunks)) * sh.chunk_len, left = sh.n_inc - inc0;
    return {int64_t(path), inc0, left < sh.chunk_len ? left : sh.chunk_len};
}

// Wavefronts per SIMD the walk over stretches must leave room for: what it has for whole paths.  The products ahead of it would
// otherwise take registers (addresses of every suffix) that halve what is in flight through the whole walk.  Without | with: 64 x 400
// points, d = 3, N = 8 175 | 140 us, 1 x 4000, d = 7, N = 6, fp64 535 | 415, 400 x 200, d = 7, N = 4, fp64 132 | 108, 1 x 4000, d = 4, N = 8, fp64 357 | 319,
// 400 x 200, d = 2, N = 9 105 | 92; 160 other shapes within 3 %, but for d = 8, N = 4, which waits for spills (400 x 200 70 | 78).
constexpr int tb_stretch_waves(int elem, int d, int N)
{
    if (elem == 8) return d <= 6 || (d == 7 && N >= 4 && N <= 6) ? 2 : 1;
    return d <= 3 ? 4 : (d >= 6 && N == 3) || (d == 8 && N >= 8) ? 2 : 3;
}

// The same with the stretches counted from the end of the path: the first one may begin before it (inc0 < 0).
__device__ __forceinline__ ChunkView stretch_view_from_end(uint32_t row, const Shape &sh)
{
    const uint32_t path = row / uint32_t(sh.chunks), c = row - path * uint32_t(sh.chunks);
    return {int64_t(path), sh.n_inc - int64_t(uint32_t(sh.chunks) - c) * sh.chunk_len, sh.chunk_len};
}

template <typename T, int D, int N, int MODE, bool ROWS>
__global__ void __launch_bounds__(256, (MODE == kTbStretches ? tb_stretch_waves(int(sizeof(T)), D, N) : 1))
sig_tree_backward_kernel(Shape sh, StretchRows<T> nodes, const T *__restrict__ path, const T *__restrict__ sig,
                         const T *__restrict__ gout, T *__restrict__ partial)
{
    constexpr bool STREAM = MODE == kTbStream || MODE == kTbStreamStretches;
    constexpr bool STRETCHES = MODE == kTbStretches || MODE == kTbStreamStretches, FROM_END = MODE == kTbStreamStretches;
    using TS = TbShape<T, D, N, ROWS>;
    constexpr int U = TS::U, P = TS::P, PPG = TS::kPathsPerGroup;
    constexpr int H1 = U >= 1 ? D : 1, H2 = U >= 2 ? D * D : 1;
    constexpr int ZR = TS::kZRow, LANES = TS::kLanes, ROW = TS::kRow, BATCH = TS::kBatch, GROUPS = TS::kGroups, INC = TS::kIncSize;
    constexpr int64_t kS = TS::kS;
    __shared__ __align__(16) T zt[PPG * kTbTile * ZR];
    __shared__ T part[TS::kWide ? kTbTile * 4 * D : 1];   // [increment of the tile][wavefront][channel]
    // [wavefront][increment of the batch][lane][number], and a row of zeros
    __shared__ __align__(16) T rows[MODE == kTbStretches && TS::kNodesInLds ? TS::kStage : TS::kRowsSize];

    constexpr int WPP = TS::kWavesPerPath;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int item = wave * LANES + lane;   // the thread's place among the lanes in use
    const int slot_raw = TS::kMulti ? 0 : TS::kWide ? wave / WPP : item / int(TS::kWords);
    const int slot = slot_raw < PPG ? slot_raw : PPG - 1;
    const int64_t u_raw = TS::kMulti  ? int64_t(blockIdx.x % TS::kGroupsPerPath) * (4 * LANES) + item
                          : TS::kWide ? int64_t(item - slot_raw * WPP * LANES)
                                      : int64_t(item % int(TS::kWords));
    const int64_t row = TS::kMulti ? int64_t(blockIdx.x / TS::kGroupsPerPath) : int64_t(blockIdx.x) * PPG + slot;
    const bool live = lane < LANES && u_raw < TS::kWords && slot_raw < PPG && row < sh.B;
    const int64_t u = live ? u_raw : 0;   // idle threads shadow word 0 of a valid row and contribute nothing
    const int64_t my_row = STRETCHES ? (row < sh.B ? row : 0) : live ? row : (row < sh.B ? row : 0);   // the same either way

    int cl[P + 1];        // letters of the word
    int64_t pre[P + 1];   // index of its prefix of i letters inside level i
    bool first[P + 1];    // whether this thread is the first one below that prefix
    {
        int64_t rest = u, width = 1;
#pragma unroll
        for (int i = P; i >= 1; --i) {
            pre[i] = rest;
            first[i] = live && (u % width == 0);
            cl[i] = int(rest % D);
            rest /= D;
            width *= D;
        }
    }
    T rf[N + 2];   // 1 / m!
#pragma unroll
    for (int m = 0; m <= N + 1; ++m) rf[m] = T(inv_factorial(m));

    // a row that is a stretch: its path, where it begins in it and its increments (the walk takes chunk_len for every row: the ones
    // past the end of a shorter row are zero, change nothing and leave no partial sums)
    ChunkView mine = {my_row, 0, sh.n_inc};
    if constexpr (STRETCHES) mine = FROM_END ? stretch_view_from_end(uint32_t(my_row), sh) : stretch_view(uint32_t(my_row), sh);
    const int64_t n_walk = STRETCHES ? sh.chunk_len : sh.n_inc;
    const int64_t per_row = STREAM ? sh.n_inc * kS : kS;
    const T *sg = sig + (FROM_END ? mine.path : my_row) * per_row;
    const T *go = gout + mine.path * per_row;
    const int64_t before = FROM_END ? mine.inc0 : 0, s_last = before + n_walk - 1;   // the walk's last increment

    struct Share {
        T lo[P + 1];
        T h1[H1];
        T h2[H2];
    };
    // A thread's share of one flat element.  `own_only`: a prefix's value counts for the first thread below it
    // only (cotangents); otherwise every thread takes it (the signature).
    auto load_share = [&](const T *e, bool own_only, bool with_h1, bool with_h2) {
        Share s = {};
#pragma unroll
        for (int i = 1; i <= P; ++i) s.lo[i] = (!own_only || first[i]) ? e[tb_off(D, i) + pre[i]] : T(0);
        if constexpr (U >= 1) {
            if (with_h1) {
#pragma unroll
                for (int c = 0; c < D; ++c) s.h1[c] = e[tb_off(D, P + 1) + u * D + c];
            }
        }
        if constexpr (U >= 2) {
            if (with_h2) {
#pragma unroll
                for (int c = 0; c < D * D; ++c) s.h2[c] = e[tb_off(D, P + 2) + u * (D * D) + c];
            }
        }
        return s;
    };

    Share G = load_share(FROM_END ? go + s_last * kS : STREAM ? go + (sh.n_inc - 1) * kS : go, true, true, true);
    if constexpr (!STRETCHES) {
        if (!live) G = Share{};
    }
    Share A = {};
    if constexpr (!STREAM && !STRETCHES) {
        A = load_share(sg, false, U >= 2, false);
    }
    // Stream mode reads a row of the forward output and a row of its cotangent at every increment.  In fp32 both are
    // fetched an increment ahead of their use, so that a trip to memory is not part of every step of the chain.  In
    // fp64 they are fetched where they are used: two more shares of a flat element (up to 94 registers each at d = 6)
    // take these kernels to 350 and more registers per lane, and the code generated for d = 4, N = 8; d = 5, N = 7;
    // d = 6, N = 6 and d = 8, N = 6 then lost the cotangent of the levels above a thread's word at the first
    // increment (tests/test_backward_gpu.py: test_tree_gradient_every_shape).
    constexpr bool kAhead = STREAM && sizeof(T) == 4;
    Share A_ahead = {};
    if constexpr (kAhead) {
        if (FROM_END ? s_last >= 1 : sh.n_inc >= 2) A_ahead = load_share(sg + (FROM_END ? s_last - 1 : sh.n_inc - 2) * kS, false, U >= 2, false);
    }

    // rows served by this workgroup, for the staging of their increments
    const int64_t row0 = TS::kMulti ? int64_t(blockIdx.x / TS::kGroupsPerPath) : int64_t(blockIdx.x) * PPG;
    const T *bpv = static_cast<const T *>(sh.basepoint_value);
    // where the partial sums go: [row][group][increment][D]; group = the workgroup's number inside its path (wavefront
    // sums), the word's first P-1 letters or the whole word (short paths)
    const int64_t wg_group = TS::kMulti ? int64_t(blockIdx.x % TS::kGroupsPerPath) : 0;
    // After a batch lane s of a wavefront adds up group g = s % GROUPS at increment s / GROUPS of the batch.  The rows of group g
    // begin at lane g D - skip; its letters are those of any of its lanes, and so is the place its sums go to.
    const int sum_group = lane % GROUPS, sum_inc = lane / GROUPS;
    const int skip = TS::kSplit ? __builtin_amdgcn_readfirstlane(int((u_raw - lane) % D)) : 0;
    // Lanes with a word: the rows behind them in a path's last wavefront are left out of the sums (groups that are not split are
    // whole or nobody's).  An idle lane's cotangent is zero, but what it leaves is not where the word it shadows overflows.
    const int64_t words_left = TS::kWords - (u_raw - lane);
    const int with_word = __builtin_amdgcn_readfirstlane(words_left < 0 ? 0 : words_left < LANES ? int(words_left) : LANES);
    const int first_lane = sum_group * D - skip;
    const int some_lane = first_lane < 0 ? 0 : first_lane < LANES ? first_lane : LANES - 1;
    int gl[P + 1];   // letters 1 .. P-1 of that group
#pragma unroll
    for (int j = 1; j < P; ++j) gl[j] = TS::kRows ? __shfl(cl[j], some_lane) : 0;
    int64_t sum_at = 0;   // scalar offset of its partial sums, negative: none
    int64_t sum_n = sh.n_inc, sum_from = 0;   // how many increments it has, where stretches are walked, and the first of them
    if constexpr (!TS::kWide) {
        const int64_t at = live ? ((mine.path * TS::kPartials + (TS::kRows ? u / D : u)) * sh.n_inc + mine.inc0) * D : -1;
        sum_at = TS::kRows ? __shfl(at, some_lane) : at;
        if constexpr (STRETCHES) {
            const int64_t n = live ? mine.n : 0, from = FROM_END && before < 0 ? -before : 0;
            sum_n = TS::kRows ? __shfl(n, some_lane) : n;
            sum_from = TS::kRows ? __shfl(from, some_lane) : from;
        }
    }
    T *my_rows = rows + wave * (BATCH * INC);
    const int my_row_at = lane * ROW + (lane + skip) / D * TS::kGroupPad;
    const T *zeros = rows + 4 * BATCH * INC;
    if constexpr (TS::kRows && !STRETCHES) {
        if (tid < ROW) rows[4 * BATCH * INC + tid] = T(0);   // the first tile's barriers come before its first use
    }

    // This thread's scalars of the tile at t0, the end and the start of an increment; a workgroup of many paths that is not full
    // skips the rest.  They are fetched before the tile after it is worked on (tiles are taken from the last to the first), but
    // for fp64 beyond depth 2, where the registers that hold them meanwhile are missing elsewhere (6000 paths of 100 points,
    // d = 6, N = 3: 215 us, fetched where they are needed 173; 384 paths, d = 9, N = 4: four wavefronts per SIMD, not five, 393 | 357; at
    // depth 2, a stream of 1500 paths at d = 11: 263 | 310).
    constexpr int kStaged = PPG * kTbTile * D, kPerThread = (kStaged + 255) / 256;
    constexpr bool kFetchAhead = sizeof(T) == 4 || N == 2;
    constexpr bool kSkip = PPG > 4 || !kFetchAhead;   // a branch per scalar, worth it where many may be off
    T hi[kPerThread], lo[kPerThread];
    __shared__ ChunkView served[STRETCHES ? PPG : 1];   // the rows of the workgroup, where they are stretches
    if constexpr (STRETCHES) {
        if (tid < PPG) {
            const bool there = row0 + tid < sh.B;
            const uint32_t r = uint32_t(there ? row0 + tid : row0);
            served[tid] = FROM_END ? stretch_view_from_end(r, sh) : stretch_view(r, sh);
            if (!there) served[tid].n = 0;
        }
        __syncthreads();
    }
    auto fetch = [&](int64_t t0) {
#pragma unroll
        for (int q = 0; q < kPerThread; ++q) {
            const int e = tid + 256 * q < kStaged ? tid + 256 * q : kStaged - 1;
            const int p = e / (kTbTile * D), i = (e / D) % kTbTile, c = e % D;
            if constexpr (STRETCHES) {   // unconditional loads, on indices clamped into the path
                const ChunkView r = served[p];
                const bool on = t0 + i < r.n && (!FROM_END || r.inc0 + t0 + i >= 0);
                const T *x = path + r.path * sh.L * D;
                const int64_t i_hi = (on ? r.inc0 + t0 + i : 0) + (sh.basepoint ? 0 : 1);
                hi[q] = x[i_hi * D + c];
                lo[q] = i_hi > 0 ? x[(i_hi - 1) * D + c] : bpv != nullptr ? bpv[r.path * D + c] : T(0);
                if (!on) lo[q] = hi[q];
                continue;
            }
            const bool on = row0 + p < sh.B && t0 + i < sh.n_inc;
            const int64_t i_hi = (on ? t0 + i : 0) + (sh.basepoint ? 0 : 1);
            const T *x = path + (on ? row0 + p : row0) * sh.L * D, *b = bpv != nullptr ? bpv + (on ? row0 + p : row0) * D : nullptr;
            hi[q] = lo[q] = T(0);
            if (kSkip ? on : true) {
                hi[q] = x[i_hi * D + c];
                lo[q] = i_hi > 0 ? x[(i_hi - 1) * D + c] : b != nullptr ? b[c] : T(0);
            }
            if (!kSkip && !on) lo[q] = hi[q];
        }
    };
    const int64_t last_tile = ((n_walk - 1) / kTbTile) * kTbTile;
    if constexpr (kFetchAhead) fetch(last_tile);   // in one trip to memory with the gradient above
    if constexpr (FROM_END) {
        // The gradient that the prefixes behind the stretch leave at its end: what was carried to the front of the last stretch, carried
        // back through one stretch after the other, each adding its own.
        constexpr int64_t kBelow = tb_off(D, N), kParts = P + D + D * D;
        uint32_t at[P + 1] = {};
#pragma unroll
        for (int i = 1; i <= P; ++i) at[i] = uint32_t(pre[i]);
        const int c = int(my_row - mine.path * sh.chunks);
        Share H = {};
        for (int k = sh.chunks - 1; k > c; --k) {
            const T *x = nodes.carried + (mine.path * sh.chunks + k) * kParts * TS::kWords + u;
            Share own;
#pragma unroll
            for (int i = 1; i <= P; ++i) own.lo[i] = x[(i - 1) * TS::kWords];
#pragma unroll
            for (int j = 0; j < D; ++j) own.h1[j] = x[(P + j) * TS::kWords];
#pragma unroll
            for (int j = 0; j < D * D; ++j) own.h2[j] = x[(P + D + j) * TS::kWords];
            if (k < sh.chunks - 1)
                stretch_carry_back<T, D, P>(H.lo, H.h1, H.h2, at, nodes.at[0] + (mine.path * (sh.chunks - 2) + k - 1) * kBelow);
#pragma unroll
            for (int i = 1; i <= P; ++i) H.lo[i] += own.lo[i];
#pragma unroll
            for (int j = 0; j < D; ++j) H.h1[j] += own.h1[j];
#pragma unroll
            for (int j = 0; j < D * D; ++j) H.h2[j] += own.h2[j];
        }
#pragma unroll
        for (int i = 1; i <= P; ++i) G.lo[i] += H.lo[i];
#pragma unroll
        for (int j = 0; j < D; ++j) G.h1[j] += H.h1[j];
#pragma unroll
        for (int j = 0; j < D * D; ++j) G.h2[j] += H.h2[j];
        if (!live) G = Share{};
        if (TS::kRows && tid < ROW) rows[4 * BATCH * INC + tid] = T(0);
    } else if constexpr (STRETCHES) {
        constexpr int64_t kBelow = tb_off(D, N);            // scalars below the top level
        constexpr int kStaged = TS::kStagedNodes;
        constexpr int kInFlight = 16;
        uint32_t at[P + 1] = {};
#pragma unroll
        for (int i = 1; i <= P; ++i) at[i] = uint32_t(pre[i]);
        const int64_t row1 = row0 + PPG < sh.B ? row0 + PPG - 1 : sh.B - 1;   // the workgroup's last row
        const uint32_t first_path = uint32_t(row0) / uint32_t(sh.chunks), last_path = uint32_t(row1) / uint32_t(sh.chunks);
        for (int l = nodes.levels - 1; l >= 0; --l) {
            const int shift = l * kStretchRadixLog2, count = nodes.count[l];
            const bool top = l == nodes.levels - 1;
            // a row's node is multiplied with its siblings: the nodes of the workgroup's rows and their siblings follow one another
            const auto begin_of = [&](int c) { return top ? 0 : c >> (shift + kStretchRadixLog2) << kStretchRadixLog2; };
            const auto end_of = [&](int c) {
                const int end = begin_of(c) + (1 << kStretchRadixLog2);
                return top || end > count ? count : end;
            };
            const int c = int(my_row - mine.path * sh.chunks);
            const int64_t path0 = mine.path * count, node = path0 + (c >> shift);
            const int64_t begin = path0 + begin_of(c), end = path0 + end_of(c), last = l == 0 ? node : node - 1;
            if constexpr (TS::kNodesInLds) {
                const int64_t from = first_path * count + begin_of(int(uint32_t(row0) - first_path * uint32_t(sh.chunks)));
                const int64_t to = last_path * count + end_of(int(uint32_t(row1) - last_path * uint32_t(sh.chunks)));
                const auto stage = [&](int64_t k0, int64_t k1) {
                    __syncthreads();
                    const T *src = nodes.at[l] + k0 * kBelow;
                    const int n = int(k1 - k0) * int(kBelow);
                    for (int e = tid; e < n; e += 256 * kInFlight) {   // so many reads on their way together
                        T v[kInFlight];
#pragma unroll
                        for (int q = 0; q < kInFlight; ++q) v[q] = src[e + 256 * q < n ? e + 256 * q : n - 1];
#pragma unroll
                        for (int q = 0; q < kInFlight; ++q)
                            if (e + 256 * q < n) rows[e + 256 * q] = v[q];
                    }
                    __syncthreads();
                };
                const int64_t pieces = (to - from + kStaged - 1) / kStaged;
                for (int64_t p = 0; p < pieces; ++p) {
                    const int64_t k0 = from + p * kStaged, k1 = k0 + kStaged < to ? k0 + kStaged : to;
                    stage(k0, k1);
                    for (int64_t k = begin > k0 ? begin : k0; k <= last && k < k1; ++k) {
                        StretchFactor<T, D, P> f;
                        f.read(at, rows + int(k - k0) * int(kBelow));
                        f.multiply(A.lo, A.h1);
                    }
                }
                for (int64_t p = pieces - 1; p >= 0; --p) {
                    const int64_t k0 = from + p * kStaged, k1 = k0 + kStaged < to ? k0 + kStaged : to;
                    if (p < pieces - 1) stage(k0, k1);
                    for (int64_t k = (end < k1 ? end : k1) - 1; k > node && k >= k0; --k)
                        stretch_carry_back<T, D, P>(G.lo, G.h1, G.h2, at, rows + int(k - k0) * int(kBelow));
                }
            } else {
                const auto at_node = [&](int64_t k) { return TS::kWide ? wave_uniform(nodes.at[l] + k * kBelow) : nodes.at[l] + k * kBelow; };
                for (int64_t k = begin; k <= last; ++k) {
                    StretchFactor<T, D, P> f;
                    f.read(at, at_node(k));
                    f.multiply(A.lo, A.h1);
                }
                for (int64_t k = end - 1; k > node; --k) stretch_carry_back<T, D, P>(G.lo, G.h1, G.h2, at, at_node(k));
            }
        }
        if (!live) G = Share{};
        __syncthreads();   // the rows of the walk's numbers take the place of the nodes
        if (TS::kRows && tid < ROW) rows[4 * BATCH * INC + tid] = T(0);
    }
    for (int64_t t0 = last_tile; t0 >= 0; t0 -= kTbTile) {
        const int nt = int(n_walk - t0 < kTbTile ? n_walk - t0 : kTbTile);
        if constexpr (!kFetchAhead) fetch(t0);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kPerThread; ++q) {
            const int e = tid + 256 * q;
            if (e < kStaged) zt[e / D * ZR + e % D] = hi[q] - lo[q];
        }
        __syncthreads();
        if constexpr (kFetchAhead) {
            if (t0 > 0) fetch(t0 - kTbTile);
        }

        for (int i = nt - 1; i >= 0; --i) {
            const int64_t s = FROM_END ? before + t0 + i : t0 + i;
            const T *zrow = zt + (slot * kTbTile + i) * ZR;
            T zc[P + 1];
#pragma unroll
            for (int j = 1; j <= P; ++j) zc[j] = zrow[cl[j]];
            T zu[D];
#pragma unroll
            for (int c = 0; c < D; ++c) zu[c] = zrow[c];
            __builtin_amdgcn_sched_barrier(0);   // every read is issued before the first is used

            Share G_ahead = {};
            if constexpr (kAhead) {
                // the signature after s increments is output entry s-1 (the identity for s = 0)
                A = s > 0 ? A_ahead : Share{};
                if (s >= 2) A_ahead = load_share(sg + (s - 2) * kS, false, U >= 2, false);
                if (s > 0 && live) G_ahead = load_share(go + (s - 1) * kS, true, true, true);   // added at the end of this step
            } else if constexpr (STREAM) {
                A = s > 0 ? load_share(sg + (s - 1) * kS, false, U >= 2, false) : Share{};
            }

            // ---- up: Hh[j][k] = T^(k)_j / (k-j)! at this thread's word; the signature before the increment
            T Hh[P + 1][N + 2];
            T a_lo[P + 1];
            a_lo[1] = STREAM ? A.lo[1] : A.lo[1] - zc[1];
#pragma unroll
            for (int k = 2; k <= N; ++k) Hh[1][k] = fma_t(zc[1], rf[k], a_lo[1] * rf[k - 1]);
#pragma unroll
            for (int j = 2; j <= P; ++j) {
                if (j < N) {
                    a_lo[j] = STREAM ? A.lo[j] : fma_t(-Hh[j - 1][j], zc[j], A.lo[j]);
#pragma unroll
                    for (int k = j + 1; k <= N; ++k) Hh[j][k] = fma_t(Hh[j - 1][k], zc[j], a_lo[j] * rf[k - j]);
                } else {
                    a_lo[j] = T(0);
                }
            }
            T a_h1[H1], Th1[H1];
            if constexpr (U >= 2) {
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    a_h1[c] = STREAM ? A.h1[c] : fma_t(-Hh[P][P + 1], zu[c], A.h1[c]);
                    Th1[c] = fma_t(Hh[P][N], zu[c], a_h1[c]);
                }
            }
            if constexpr (!STREAM) {
#pragma unroll
                for (int j = 1; j <= P; ++j) A.lo[j] = a_lo[j];
                if constexpr (U >= 2) {
#pragma unroll
                    for (int c = 0; c < D; ++c) A.h1[c] = a_h1[c];
                }
            }

            // ---- down
            T dz[D];
#pragma unroll
            for (int c = 0; c < D; ++c) dz[c] = T(0);
            T Dc[N + 2];   // Dc[k] = this thread's part of D^(k)_j (k-j)! at its prefix of the level j being processed
#pragma unroll
            for (int k = 0; k <= N + 1; ++k) Dc[k] = T(0);
            T Dh[H1];
            if constexpr (U >= 2) {
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    T acc = T(0);
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        acc = fma_t(G.h2[c * D + j], zu[j], acc);
                        dz[j] = fma_t(Th1[c], G.h2[c * D + j], dz[j]);
                    }
                    Dh[c] = acc;
                }
            }
            if constexpr (U >= 1) {
                T acc1 = T(0), acc2 = T(0);
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    dz[c] = fma_t(Hh[P][P + 1], G.h1[c], dz[c]);
                    acc1 = fma_t(G.h1[c], zu[c], acc1);
                    if constexpr (U >= 2) {
                        dz[c] = fma_t(Hh[P][P + 2], Dh[c], dz[c]);
                        acc2 = fma_t(Dh[c], zu[c], acc2);
                        G.h1[c] += Dh[c];
                    }
                }
                Dc[P + 1] = acc1;
                if constexpr (U >= 2) Dc[P + 2] = acc2;
            }
            // levels P .. 1 along the word: one scalar per chain, this thread's part only
            T contrib[P + 1];   // to the channels of the word's letters
#pragma unroll
            for (int j = P; j >= 1; --j) {
                contrib[j] = j >= 2 ? Hh[j >= 2 ? j - 1 : 1][j] * G.lo[j] : G.lo[j];   // T^(k)_0 = 1
                T g_add = T(0);
#pragma unroll
                for (int k = j + 1; k <= N; ++k) {
                    contrib[j] = fma_t(j >= 2 ? Hh[j >= 2 ? j - 1 : 1][k] : rf[k], Dc[k], contrib[j]);
                    g_add = k == j + 1 ? Dc[k] : fma_t(Dc[k], rf[k - j], g_add);
                }
                if (j >= 2) {
#pragma unroll
                    for (int k = N; k >= j + 1; --k) Dc[k] *= zc[j];
                    Dc[j] = G.lo[j] * zc[j];
                }
                G.lo[j] += g_add;
            }

            // ---- this thread's (wavefront's) part of the increment's gradient
            if constexpr (TS::kRows) {
                const int ib = (nt - 1 - i) % BATCH;
                if (lane < LANES) {
                    T *r = my_rows + ib * INC + my_row_at;
#pragma unroll
                    for (int c = 0; c < D; ++c) r[c] = dz[c];
                    r[D] = contrib[P];
#pragma unroll
                    for (int j = 1; j < P; ++j) r[D + j] = contrib[j];
                }
                if (ib == BATCH - 1 || i == 0) {   // increment i + ib - k of the tile lies in place k of the batch
                    wave_lds_order();
                    T sum[D];
#pragma unroll
                    for (int c = 0; c < D; ++c) sum[c] = T(0);
                    if (sum_inc <= ib) {
                        T own[P + 1];
#pragma unroll
                        for (int j = 1; j < P; ++j) own[j] = T(0);
#pragma unroll
                        for (int w = 0; w < D; ++w) {   // the group's words by their last letter
                            const T *r = my_rows + sum_inc * INC + (first_lane + w) * ROW + sum_group * TS::kGroupPad;
                            if constexpr (TS::kSplit) r = unsigned(first_lane + w) < unsigned(with_word) ? r : zeros;
#pragma unroll
                            for (int c = 0; c < D; ++c) sum[c] += r[c];
                            sum[w] += r[D];
#pragma unroll
                            for (int j = 1; j < P; ++j) own[j] += r[D + j];
                        }
#pragma unroll
                        for (int j = 1; j < P; ++j)
#pragma unroll
                            for (int c = 0; c < D; ++c) sum[c] += gl[j] == c ? own[j] : T(0);
                    }
                    if constexpr (TS::kWide) {
                        // the wavefront's groups: a lane per increment and channel (the rows have been read)
                        wave_lds_order();
                        if (sum_inc <= ib) {
#pragma unroll
                            for (int c = 0; c < D; ++c) my_rows[(sum_inc * GROUPS + sum_group) * ZR + c] = sum[c];
                        }
                        wave_lds_order();
                        const int k = lane / D, c = lane - k * D;
                        if (k <= ib) {
                            // four running sums: a gradient at a point is the difference of two of these, so their rounding
                            // shows (d = 4, N = 6, 65 537 points: one running sum of 16 groups is off by 2.0e-5, these by 1.7e-5)
                            T acc[4] = {};
#pragma unroll
                            for (int g = 0; g < GROUPS; ++g) acc[g & 3] += my_rows[(k * GROUPS + g) * ZR + c];
                            part[((i + ib - k) * 4 + wave) * D + c] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
                        }
                        wave_lds_order();   // the next batch's rows overwrite these
                    } else {
                        const int64_t t = t0 + i + ib - sum_inc;
                        if (sum_inc <= ib && (STRETCHES ? t >= sum_from && t < sum_n : sum_at >= 0)) {
                            T *pp = partial + sum_at + (t0 + i + ib - sum_inc) * D;
#pragma unroll
                            for (int c = 0; c < D; ++c) pp[c] = sum[c];
                        }
                        wave_lds_order();
                    }
                }
            } else {
#pragma unroll
                for (int j = P; j >= 1; --j)
#pragma unroll
                    for (int c = 0; c < D; ++c) dz[c] += cl[j] == c ? contrib[j] : T(0);
                if constexpr (STREAM && !kAhead && !TS::kWide && (D <= 4 || (N == 2 && D <= 8))) {
                    // Left to itself the compiler sinks the sums, and with them the wait for the rows' loads, into the branch of the
                    // lanes that store them; the next step's loads, in registers a lane outside may still have on the way,
                    // then wait for these stores too (fp64, 100 points, d = 4, N = 2, a path: 51 us, so 43; 384 paths, d = 2, N = 5: 124 | 101;
                    // with more sums and registers it is the other way round: 48 paths, d = 8, N = 3: 326 | 343, d = 11, N = 2: 152 | 162).
#pragma unroll
                    for (int c = 0; c < D; ++c) asm volatile("" : "+v"(dz[c]));
                }
                if constexpr (TS::kWide) {
                    // the wavefronts do not wait for one another inside a tile: their sums meet in LDS at its end
#pragma unroll
                    for (int c = 0; c < D; ++c) {
                        const T total = group_sum<0, 6, T>(live ? dz[c] : T(0));
                        if (lane == c) part[(i * 4 + wave) * D + c] = total;
                    }
                } else {
                    if (live && (!STRETCHES || (t0 + i >= sum_from && t0 + i < sum_n))) {
                        T *pp = partial + sum_at + (FROM_END ? t0 + i : s) * D;
#pragma unroll
                        for (int c = 0; c < D; ++c) pp[c] = dz[c];
                    }
                }
            }

            if constexpr (STREAM) {
                if (s > 0 && live) {
                    if constexpr (!kAhead) G_ahead = load_share(go + (s - 1) * kS, true, true, true);
                    const Share &add = G_ahead;
#pragma unroll
                    for (int j = 1; j <= P; ++j) G.lo[j] += add.lo[j];
                    if constexpr (U >= 1) {
#pragma unroll
                        for (int c = 0; c < D; ++c) G.h1[c] += add.h1[c];
                    }
                    if constexpr (U >= 2) {
#pragma unroll
                        for (int c = 0; c < D * D; ++c) G.h2[c] += add.h2[c];
                    }
                }
            }
        }
        if constexpr (TS::kWide) {
            __syncthreads();
            for (int e = tid; e < PPG * nt * D; e += 256) {
                const int p = e / (nt * D), i = (e / D) % nt, c = e % D;
                if (row0 + p >= sh.B) continue;
                const T *q = part + (i * 4 + p * WPP) * D + c;
                T total = q[0];
#pragma unroll
                for (int w = 1; w < WPP; ++w) total += q[w * D];
                if constexpr (STRETCHES) {
                    const ChunkView r = served[p];
                    if (t0 + i < r.n && (!FROM_END || r.inc0 + t0 + i >= 0))
                        partial[((r.path * TS::kPartials + wg_group) * sh.n_inc + r.inc0 + t0 + i) * D + c] = total;
                } else {
                    partial[(((row0 + p) * TS::kPartials + wg_group) * sh.n_inc + t0 + i) * D + c] = total;
                }
            }
        }
    }
}

// Whether paths packed into a wavefront add up their numbers through LDS (one partial sum per group of d words) or write one
// per thread.  In final mode few threads wait for the batches' trips through LDS, many for the partial sums in memory (100
// points, us, through LDS | per thread: fp32 d = 7, N = 4, 256 paths 66 | 70, 32 paths 63 | 56, 2048 paths 94 | 213; d = 3, N = 5:
// 48 | 42 and 64 | 72 at 256 and 2048; fp64 d = 4, N = 5: 66 | 55 and 141 | 258).  In fp64 from nine words and 768 paths on (6000 paths,
// d = 7, N = 3, 7 words: 287 | 173, d = 3, N = 4, 9 words: 1 | 1.4 times; 384 paths, d = 8, N = 4: 136 | 107, 1500: 1 | 1.4 times).
// In stream mode the stores also stand between
// the loads of one increment and the next (fp32 d = 5, N = 4, 64 paths: 82 | 139; d = 6, N = 4: 96 | 157); for few paths the batches
// cost more (d = 7, N = 3, 8 paths: 96 | 89; one path, d = 7, N = 4: 1 | 0.88 times, fp64 157 | 120; 48 paths 1 | 1.4, fp64 1 | 1.2), in fp64 up
// to eight words always (d = 6, N = 3: 124 | 101).
// (Two channels in final mode, where a group is two words: from 60 000 words on; 1500 paths, N = 7, 48 000 words: 70 | 65, fp64 88 | 77.)
inline bool tb_packed_rows(int d, int64_t words, int64_t rows, size_t elem, bool stream)
{
    if (stream) return elem == 4 ? rows * words >= 300 : words >= 9 && rows * words >= 400;
    if (d == 2) return words >= 9 && rows * words >= 60000;
    return elem == 4 ? rows * words >= 8000 : words >= 9 && rows >= 768 && rows * words >= 18000;
}

// Longer paths always do, except in fp64 where a thread's share leaves no registers for the sums (with them d = 8, N = 6 moves 152 of
// its registers in and out: 48 paths of 100 points 820 us, by lane exchanges 630; d = 7, N = 6: 1 | 0.78 times, d = 6, N = 7: 1 | 0.93,
// d = 5, N = 9: 1 | 0.64; on the other side of the line d = 7, N = 5: 1 | 1.58, d = 6, N = 6: 1 | 1.32; streams at d = 7, N = 7 1 | 1.14).
template <typename T, int D, int N, bool STREAM>
constexpr bool tb_wide_rows() { return sizeof(T) == 4 || (D < 8 && (D + N < 13 || (STREAM && D == 7))); }

template <typename T, int D, int N, bool STREAM, bool ROWS>
hipError_t launch_tb_mode(const Shape &sh, const T *path, const T *sig, const T *gout, T *gpath, T *gbase, T *partial, hipStream_t st)
{
    constexpr int MODE = STREAM ? kTbStream : kTbFinal;
    using TS = TbShape<T, D, N, ROWS>;
    const int64_t groups = TS::kMulti ? sh.B * TS::kGroupsPerPath : (sh.B + TS::kPathsPerGroup - 1) / TS::kPathsPerGroup;
    if (!grid_holds(groups, 256)) return hipErrorNotSupported;
    hipLaunchKernelGGL((sig_tree_backward_kernel<T, D, N, MODE, ROWS>), dim3(unsigned(groups)), dim3(256), 0, st, sh, StretchRows<T>{}, path, sig,
                       gout, partial);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    return launch_increment_sums<T>(sh, TS::kPartials, partial, gpath, gbase, st);
}

template <typename T, int D, int N>
hipError_t launch_tb_dn(const Shape &sh, const T *path, const T *sig, const T *gout, T *gpath,
                        T *gbase, T *partial, hipStream_t st)
{
    const auto launch = [&](auto stream_rows, auto final_rows) {
        return sh.stream ? launch_tb_mode<T, D, N, true, decltype(stream_rows)::value>(sh, path, sig, gout, gpath, gbase, partial, st)
                         : launch_tb_mode<T, D, N, false, decltype(final_rows)::value>(sh, path, sig, gout, gpath, gbase, partial, st);
    };
    if constexpr (D > 8) {
        return launch(std::false_type{}, std::false_type{});
    } else if constexpr (TbShape<T, D, N, false>::kWide) {
        return launch(std::bool_constant<tb_wide_rows<T, D, N, true>()>{}, std::bool_constant<tb_wide_rows<T, D, N, false>()>{});
    } else {
        const bool rows = tb_packed_rows(D, TbShape<T, D, N, false>::kWords, sh.B, sizeof(T), sh.stream != 0);
        return rows ? launch(std::true_type{}, std::true_type{}) : launch(std::false_type{}, std::false_type{});
    }
}

// Stream mode in stretches.  The signatures are at hand at every prefix, so what makes the walk a chain is the cotangent alone,
// which gathers from the end of the path on.  This kernel gathers it inside every stretch, from that stretch's rows only: X_c, the
// gradient that they leave at the front of the stretch, split over the threads like the cotangents of the walk.  The walk over a
// stretch then begins from X_{K-1} carried back through the stretches behind it, each adding its X.  It takes the walk's
// steps down but not those up, and no sums over lanes: about a third of its time per increment.
template <typename T, int D, int N>
__global__ void __launch_bounds__(256)
sig_stream_carry_kernel(Shape sh, const T *__restrict__ path, const T *__restrict__ gout, T *__restrict__ carried)
{
    constexpr int P = N - 2;
    constexpr int64_t kS = tb_off(D, N + 1), kWords = tb_off(D, P + 1) - tb_off(D, P), kParts = P + D + D * D;
    constexpr int64_t kGroupsPerRow = kWords >= 256 ? (kWords + 255) / 256 : 1;
    constexpr int R = kWords >= 256 ? 1 : int(256 / kWords < 16 ? 256 / kWords : 16);   // rows of a workgroup
    constexpr int ZR = D + 1;
    __shared__ T zt[R * kTbTile * ZR];
    const int tid = threadIdx.x;
    const int slot_raw = kWords >= 256 ? 0 : tid / int(kWords), slot = slot_raw < R ? slot_raw : R - 1;
    const int64_t u_raw = kWords >= 256 ? int64_t(blockIdx.x % kGroupsPerRow) * 256 + tid : tid - slot_raw * int(kWords);
    const int64_t row0 = kWords >= 256 ? int64_t(blockIdx.x / kGroupsPerRow) : int64_t(blockIdx.x) * R;
    const bool live = u_raw < kWords && slot_raw < R && row0 + slot < sh.B;
    const int64_t u = live ? u_raw : 0, row = row0 + slot < sh.B ? row0 + slot : row0;
    const ChunkView mine = stretch_view_from_end(uint32_t(row), sh);
    const T *go = gout + (mine.path * sh.n_inc + mine.inc0) * kS;   // the row of its first increment

    int cl[P + 1];
    int64_t pre[P + 1];
    bool first[P + 1];
    {
        int64_t rest = u, width = 1;
#pragma unroll
        for (int i = P; i >= 1; --i) {
            pre[i] = rest;
            first[i] = u % width == 0;
            cl[i] = int(rest % D);
            rest /= D;
            width *= D;
        }
    }
    struct Share {
        T lo[P + 1], h1[D], h2[D * D];
    };
    auto load = [&](const T *e) {
        Share s = {};
#pragma unroll
        for (int i = 1; i <= P; ++i) s.lo[i] = first[i] ? e[tb_off(D, i) + pre[i]] : T(0);
#pragma unroll
        for (int c = 0; c < D; ++c) s.h1[c] = e[tb_off(D, P + 1) + u * D + c];
#pragma unroll
        for (int c = 0; c < D * D; ++c) s.h2[c] = e[tb_off(D, P + 2) + u * (D * D) + c];
        return s;
    };
    auto add = [](Share &G, const Share &o) {
#pragma unroll
        for (int i = 1; i <= P; ++i) G.lo[i] += o.lo[i];
#pragma unroll
        for (int c = 0; c < D; ++c) G.h1[c] += o.h1[c];
#pragma unroll
        for (int c = 0; c < D * D; ++c) G.h2[c] += o.h2[c];
    };
    // the steps are those of increments from .. m - 1: none for the first stretch of a path, whose share no other begins from
    const int m = int(sh.chunk_len), from = mine.inc0 <= 0 ? int(sh.chunk_len) : 0;
    const T *bpv = static_cast<const T *>(sh.basepoint_value);
    Share G = load(go + int64_t(m - 1) * kS);
    const int last_tile = (m - 1) / kTbTile * kTbTile;
    for (int t0 = last_tile; t0 >= 0; t0 -= kTbTile) {
        const int nt = m - t0 < kTbTile ? m - t0 : kTbTile;
        __syncthreads();
        for (int e = tid; e < R * kTbTile * D; e += 256) {
            const int p = e / (kTbTile * D), i = (e / D) % kTbTile, c = e % D;
            const ChunkView r = stretch_view_from_end(uint32_t(row0 + p < sh.B ? row0 + p : row0), sh);
            const int64_t s = r.inc0 + t0 + i;
            const bool on = s >= 0 && t0 + i < m;
            const int64_t k = (on ? s : 0) + (sh.basepoint ? 0 : 1);
            const T *x = path + r.path * sh.L * D;
            const T end = x[k * D + c], begin = k > 0 ? x[(k - 1) * D + c] : bpv != nullptr ? bpv[r.path * D + c] : T(0);
            zt[(p * kTbTile + i) * ZR + c] = on ? end - begin : T(0);
        }
        __syncthreads();
        for (int i = nt - 1; i >= 0 && t0 + i >= from; --i) {
            const T *zrow = zt + (slot * kTbTile + i) * ZR;
            const bool more = t0 + i > from;
            Share ahead = {};
            if (more) ahead = load(go + int64_t(t0 + i - 1) * kS);   // on its way through this step
            T zc[P + 1], zu[D];
#pragma unroll
            for (int j = 1; j <= P; ++j) zc[j] = zrow[cl[j]];
#pragma unroll
            for (int c = 0; c < D; ++c) zu[c] = zrow[c];
            T Dc[N + 2] = {};   // Dc[k] = D^(k)_j (k-j)!, as in the walk
            T acc1 = T(0), acc2 = T(0);
#pragma unroll
            for (int c = 0; c < D; ++c) {
                T Dh = T(0);
#pragma unroll
                for (int j = 0; j < D; ++j) Dh = fma_t(G.h2[c * D + j], zu[j], Dh);
                acc1 = fma_t(G.h1[c], zu[c], acc1);
                acc2 = fma_t(Dh, zu[c], acc2);
                G.h1[c] += Dh;
            }
            Dc[P + 1] = acc1;
            Dc[P + 2] = acc2;
#pragma unroll
            for (int j = P; j >= 1; --j) {
                T g_add = T(0);
#pragma unroll
                for (int k = j + 1; k <= N; ++k) g_add = fma_t(Dc[k], T(inv_factorial(k - j)), g_add);
                if (j >= 2) {
#pragma unroll
                    for (int k = N; k >= j + 1; --k) Dc[k] *= zc[j];
                    Dc[j] = G.lo[j] * zc[j];
                }
                G.lo[j] += g_add;
            }
            if (more) add(G, ahead);
        }
    }
    if (live && mine.inc0 > 0) {
        T *o = carried + row * kParts * kWords + u;
#pragma unroll
        for (int i = 1; i <= P; ++i) o[(i - 1) * kWords] = G.lo[i];
#pragma unroll
        for (int c = 0; c < D; ++c) o[(P + c) * kWords] = G.h1[c];
#pragma unroll
        for (int c = 0; c < D * D; ++c) o[(P + D + c) * kWords] = G.h2[c];
    }
}

template <typename T, int D, int N, bool ROWS>
hipError_t launch_tb_stream_stretches_mode(const Shape &sh, const Shape &rows, const StretchRows<T> &nodes, const T *path, const T *sig, const T *gout,
                                           T *gpath, T *gbase, T *partial, hipStream_t st)
{
    using TS = TbShape<T, D, N, ROWS>;
    const int64_t groups = TS::kMulti ? rows.B * TS::kGroupsPerPath : (rows.B + TS::kPathsPerGroup - 1) / TS::kPathsPerGroup;
    if (!grid_holds(groups, 256)) return hipErrorNotSupported;
    hipLaunchKernelGGL((sig_tree_backward_kernel<T, D, N, kTbStreamStretches, ROWS>), dim3(unsigned(groups)), dim3(256), 0, st, rows, nodes, path,
                       sig, gout, partial);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    return launch_increment_sums<T>(sh, TS::kPartials, partial, gpath, gbase, st);
}

template <typename T, int D, int N>
hipError_t launch_tb_stream_stretches_dn(const Shape &sh, const Shape &rows, const StretchRows<T> &nodes, const T *path, const T *sig, const T *gout,
                                         T *carried, T *gpath, T *gbase, T *partial, hipStream_t st)
{
    constexpr int64_t kWords = tb_off(D, N - 1) - tb_off(D, N - 2);
    constexpr int R = kWords >= 256 ? 1 : int(256 / kWords < 16 ? 256 / kWords : 16);
    const int64_t groups = kWords >= 256 ? rows.B * ((kWords + 255) / 256) : (rows.B + R - 1) / R;
    if (groups > 0x7fffff) return hipErrorNotSupported;
    hipLaunchKernelGGL((sig_stream_carry_kernel<T, D, N>), dim3(unsigned(groups)), dim3(256), 0, st, rows, path, gout, carried);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    if constexpr (TbShape<T, D, N, false>::kWide) {
        return launch_tb_stream_stretches_mode<T, D, N, tb_wide_rows<T, D, N, true>()>(sh, rows, nodes, path, sig, gout, gpath, gbase, partial, st);
    } else {
        return tb_packed_rows(D, TbShape<T, D, N, false>::kWords, rows.B, sizeof(T), true)
                   ? launch_tb_stream_stretches_mode<T, D, N, true>(sh, rows, nodes, path, sig, gout, gpath, gbase, partial, st)
                   : launch_tb_stream_stretches_mode<T, D, N, false>(sh, rows, nodes, path, sig, gout, gpath, gbase, partial, st);
    }
}

template <typename T, int D>
hipError_t launch_tb_stream_stretches_d(const Shape &sh, const Shape &rows, const StretchRows<T> &nodes, const T *path, const T *sig, const T *gout,
                                        T *carried, T *gpath, T *gbase, T *partial, hipStream_t st)
{
    switch (sh.N) {
        case 3: return launch_tb_stream_stretches_dn<T, D, 3>(sh, rows, nodes, path, sig, gout, carried, gpath, gbase, partial, st);
        case 4: return launch_tb_stream_stretches_dn<T, D, 4>(sh, rows, nodes, path, sig, gout, carried, gpath, gbase, partial, st);
        case 5: return launch_tb_stream_stretches_dn<T, D, 5>(sh, rows, nodes, path, sig, gout, carried, gpath, gbase, partial, st);
        case 6: return launch_tb_stream_stretches_dn<T, D, 6>(sh, rows, nodes, path, sig, gout, carried, gpath, gbase, partial, st);
    }
    return hipErrorNotSupported;
}

// The walk back over stretches in stream mode; C: the signatures below the top level of all stretches of each path but
// the first and the last.
template <typename T>
hipError_t launch_tb_stream_stretches(const Shape &sh, int64_t K, int64_t m, const T *path, const T *sig, const T *gout, const T *C, T *carried,
                                      T *gpath, T *gbase, T *partial, hipStream_t st)
{
    Shape rows = sh;
    rows.B = sh.B * K;
    rows.chunks = int(K);
    rows.chunk_len = m;
    if (rows.B > 0x7fffffff) return hipErrorNotSupported;
    StretchRows<T> nodes = {};
    nodes.at[0] = C;
    nodes.carried = carried;
    switch (sh.d) {
        case 2: return launch_tb_stream_stretches_d<T, 2>(sh, rows, nodes, path, sig, gout, carried, gpath, gbase, partial, st);
        case 3: return launch_tb_stream_stretches_d<T, 3>(sh, rows, nodes, path, sig, gout, carried, gpath, gbase, partial, st);
        case 4: return launch_tb_stream_stretches_d<T, 4>(sh, rows, nodes, path, sig, gout, carried, gpath, gbase, partial, st);
        case 5: return launch_tb_stream_stretches_d<T, 5>(sh, rows, nodes, path, sig, gout, carried, gpath, gbase, partial, st);
        case 6: return launch_tb_stream_stretches_d<T, 6>(sh, rows, nodes, path, sig, gout, carried, gpath, gbase, partial, st);
        case 7: return launch_tb_stream_stretches_d<T, 7>(sh, rows, nodes, path, sig, gout, carried, gpath, gbase, partial, st);
        case 8: return launch_tb_stream_stretches_d<T, 8>(sh, rows, nodes, path, sig, gout, carried, gpath, gbase, partial, st);
    }
    return hipErrorNotSupported;
}

// Nodes of a level of the stretches' products from those of the level below, a thread per node and word of N - 2 letters.
template <typename T, int D, int N>
__global__ void __launch_bounds__(256)
sig_stretch_group_kernel(int64_t nodes, int below, int above, const T *__restrict__ from, T *__restrict__ to)
{
    constexpr int P = N - 2;
    constexpr int64_t kBelow = tb_off(D, N), kWords = tb_off(D, P + 1) - tb_off(D, P);
    const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x, node = e / kWords;
    if (node >= nodes) return;
    const uint32_t u = uint32_t(e - node * kWords);
    uint32_t at[P + 1] = {}, rest = u;
#pragma unroll
    for (int i = P; i >= 1; --i) {
        at[i] = rest;
        rest /= D;
    }
    T lo[P + 1] = {}, h1[D] = {};
    const int64_t path = node / above;
    const int i0 = int(node - path * above) << kStretchRadixLog2;
    const int end = i0 + (1 << kStretchRadixLog2) < below ? i0 + (1 << kStretchRadixLog2) : below;
    StretchFactor<T, D, P> next, f;
    const T *C = from + path * below * kBelow;
    next.read(at, C + i0 * kBelow);
    for (int k = i0; k < end; ++k) {
        f = next;
        if (k + 1 < end) next.read(at, C + (k + 1) * kBelow);
        __builtin_amdgcn_sched_barrier(0);   // the next factor is on its way while this one is multiplied on
        f.multiply(lo, h1);
    }
    T *o = to + node * kBelow;
    uint32_t width = 1;
#pragma unroll
    for (int i = P; i >= 1; --i) {   // a prefix is written by the first thread below it
        if (u % width == 0) o[tb_off(D, i) + at[i]] = lo[i];
        width *= D;
    }
#pragma unroll
    for (int c = 0; c < D; ++c) o[tb_off(D, P + 1) + u * D + c] = h1[c];
}

template <typename T, int D, int N, bool ROWS>
hipError_t launch_tb_stretches_mode(const Shape &sh, const Shape &rows, const StretchRows<T> &nodes, const T *path, const T *gout, T *gpath,
                                    T *gbase, T *partial, hipStream_t st)
{
    using TS = TbShape<T, D, N, ROWS>;
    const int64_t groups = TS::kMulti ? rows.B * TS::kGroupsPerPath : (rows.B + TS::kPathsPerGroup - 1) / TS::kPathsPerGroup;
    if (!grid_holds(groups, 256)) return hipErrorNotSupported;
    hipLaunchKernelGGL((sig_tree_backward_kernel<T, D, N, kTbStretches, ROWS>), dim3(unsigned(groups)), dim3(256), 0, st, rows, nodes, path,
                       static_cast<const T *>(nullptr), gout, partial);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    return launch_increment_sums<T>(sh, TS::kPartials, partial, gpath, gbase, st);
}

template <typename T, int D, int N>
hipError_t launch_tb_stretches_dn(const Shape &sh, const Shape &rows, StretchRows<T> nodes, T *group, const T *path, const T *gout, T *gpath,
                                  T *gbase, T *partial, hipStream_t st)
{
    constexpr int64_t kBelow = tb_off(D, N), kGroupWords = tb_off(D, N - 1) - tb_off(D, N - 2);
    // Up to so many nodes need no level above them: a step of the products takes 0.5 us from LDS, a launch 4 to 5 and from memory
    // twice that and more (16 stretches, without | with a level above: 51 x 223 points, d = 2, N = 4 19.6 | 23.9 us; 9 x 1620 in 128 at
    // d = 2, N = 4 26.9 | 30.9; from memory 12 x 723, d = 8, N = 5 191 | 152).
    constexpr int kSingle = TbShape<T, D, N, false>::kNodesInLds ? 16 : 8;
    while (nodes.count[nodes.levels - 1] > kSingle) {
        if (nodes.levels == kStretchLevels) return hipErrorNotSupported;
        const int n = nodes.count[nodes.levels - 1];
        nodes.count[nodes.levels++] = (n + (1 << kStretchRadixLog2) - 1) >> kStretchRadixLog2;
    }
    for (int l = 1; l < nodes.levels; ++l) {
        const int64_t count = sh.B * nodes.count[l], blocks = (count * kGroupWords + 255) / 256;
        if (blocks > 0x7fffff) return hipErrorNotSupported;
        hipLaunchKernelGGL((sig_stretch_group_kernel<T, D, N>), dim3(unsigned(blocks)), dim3(256), 0, st, count, nodes.count[l - 1],
                           nodes.count[l], nodes.at[l - 1], group);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
        nodes.at[l] = group;
        group += count * kBelow;
    }
    // the lanes' numbers through LDS or not as for whole paths
    if constexpr (TbShape<T, D, N, false>::kWide) {
        return launch_tb_stretches_mode<T, D, N, tb_wide_rows<T, D, N, false>()>(sh, rows, nodes, path, gout, gpath, gbase, partial, st);
    } else {
        return tb_packed_rows(D, TbShape<T, D, N, false>::kWords, rows.B, sizeof(T), false)
                   ? launch_tb_stretches_mode<T, D, N, true>(sh, rows, nodes, path, gout, gpath, gbase, partial, st)
                   : launch_tb_stretches_mode<T, D, N, false>(sh, rows, nodes, path, gout, gpath, gbase, partial, st);
    }
}

template <typename T, int D>
hipError_t launch_tb_stretches_d(const Shape &sh, const Shape &rows, const StretchRows<T> &nodes, T *group, const T *path, const T *gout,
                                 T *gpath, T *gbase, T *partial, hipStream_t st)
{
    switch (sh.N) {
        case 3: return launch_tb_stretches_dn<T, D, 3>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 4: return launch_tb_stretches_dn<T, D, 4>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 5: return launch_tb_stretches_dn<T, D, 5>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 6: return launch_tb_stretches_dn<T, D, 6>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 7: return launch_tb_stretches_dn<T, D, 7>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 8: return launch_tb_stretches_dn<T, D, 8>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 9: return launch_tb_stretches_dn<T, D, 9>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
    }
    return hipErrorNotSupported;
}

// The walk back over stretches from their signatures C below the top level (see launch_tree_stretches in sig_internal.h).
template <typename T>
hipError_t launch_tb_stretches(const Shape &sh, int64_t K, int64_t m, const T *path, const T *C, T *group, const T *gout, T *gpath, T *gbase,
                               T *partial, hipStream_t st)
{
    Shape rows = sh;
    rows.B = sh.B * K;
    rows.chunks = int(K);
    rows.chunk_len = m;
    if (rows.B > 0x7fffffff) return hipErrorNotSupported;
    StretchRows<T> nodes = {};
    nodes.levels = 1;
    nodes.count[0] = int(K);
    nodes.at[0] = C;
    switch (sh.d) {
        case 2: return launch_tb_stretches_d<T, 2>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 3: return launch_tb_stretches_d<T, 3>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 4: return launch_tb_stretches_d<T, 4>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 5: return launch_tb_stretches_d<T, 5>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 6: return launch_tb_stretches_d<T, 6>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 7: return launch_tb_stretches_d<T, 7>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
        case 8: return launch_tb_stretches_d<T, 8>(sh, rows, nodes, group, path, gout, gpath, gbase, partial, st);
    }
    return hipErrorNotSupported;
}

template <int D, int N>
int64_t tb_partials() { return TbShape<float, D, N, false>::kPartialsRoom; }   // the same for both types and modes

constexpr int kTbMaxDepth = 9;       // d = 2..8
constexpr int kTbWideMaxDepth = 6;   // d = 9..16

template <int D>
int64_t tb_partials_d(int N)
{
    switch (N) {
        case 2: return tb_partials<D, 2>();
        case 3: return tb_partials<D, 3>();
        case 4: return tb_partials<D, 4>();
        case 5: return tb_partials<D, 5>();
        case 6: return tb_partials<D, 6>();
    }
    if constexpr (D <= 8) {
        switch (N) {
            case 7: return tb_partials<D, 7>();
            case 8: return tb_partials<D, 8>();
            case 9: return tb_partials<D, 9>();
        }
    }
    return -1;
}

template <typename T, int D>
hipError_t launch_tb_d(const Shape &sh, const T *path, const T *sig, const T *gout, T *gpath, T *gbase,
                       T *partial, hipStream_t st)
{
    switch (sh.N) {
        case 2: return launch_tb_dn<T, D, 2>(sh, path, sig, gout, gpath, gbase, partial, st);
        case 3: return launch_tb_dn<T, D, 3>(sh, path, sig, gout, gpath, gbase, partial, st);
        case 4: return launch_tb_dn<T, D, 4>(sh, path, sig, gout, gpath, gbase, partial, st);
        case 5: return launch_tb_dn<T, D, 5>(sh, path, sig, gout, gpath, gbase, partial, st);
        case 6: return launch_tb_dn<T, D, 6>(sh, path, sig, gout, gpath, gbase, partial, st);
    }
    if constexpr (D <= 8) {
        switch (sh.N) {
            case 7: return launch_tb_dn<T, D, 7>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 8: return launch_tb_dn<T, D, 8>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 9: return launch_tb_dn<T, D, 9>(sh, path, sig, gout, gpath, gbase, partial, st);
        }
    }
    return hipErrorNotSupported;
}


// Bytes of partial gradients for this shape with elements of `elem` bytes; -1 if the family does not serve it.
inline int64_t tb_workspace_bytes(const Shape &sh, int64_t elem)
{
    if (sh.d < 2 || sh.d > 16 || sh.N < 2 || sh.N > (sh.d <= 8 ? kTbMaxDepth : kTbWideMaxDepth) || sh.S >= (int64_t(1) << 31))
        return -1;
    int64_t partials = -1;
    switch (sh.d) {
        case 2: partials = tb_partials_d<2>(sh.N); break;
        case 3: partials = tb_partials_d<3>(sh.N); break;
        case 4: partials = tb_partials_d<4>(sh.N); break;
        case 5: partials = tb_partials_d<5>(sh.N); break;
        case 6: partials = tb_partials_d<6>(sh.N); break;
        case 7: partials = tb_partials_d<7>(sh.N); break;
        case 8: partials = tb_partials_d<8>(sh.N); break;
        case 9: partials = tb_partials_d<9>(sh.N); break;
        case 10: partials = tb_partials_d<10>(sh.N); break;
        case 11: partials = tb_partials_d<11>(sh.N); break;
        case 12: partials = tb_partials_d<12>(sh.N); break;
        case 13: partials = tb_partials_d<13>(sh.N); break;
        case 14: partials = tb_partials_d<14>(sh.N); break;
        case 15: partials = tb_partials_d<15>(sh.N); break;
        case 16: partials = tb_partials_d<16>(sh.N); break;
    }
    if (partials < 0) return -1;
    return sh.B * partials * sh.n_inc * sh.d * elem;
}

// WIDE: the translation unit that instantiates d = 9..16; the other one instantiates d = 2..8 and hands wider calls on.
template <typename T, bool WIDE>
hipError_t launch_tb(const Shape &sh, const T *path, const T *sig, const T *gout, T *gpath, T *gbase, void *workspace,
                     int64_t workspace_bytes, hipStream_t st)
{
    const int64_t need = tb_workspace_bytes(sh, int64_t(sizeof(T)));
    if (need < 0) return hipErrorNotSupported;
    if (workspace == nullptr || workspace_bytes < need) return hipErrorInvalidValue;
    T *partial = static_cast<T *>(workspace);
    if constexpr (WIDE) {
        switch (sh.d) {
            case 9: return launch_tb_d<T, 9>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 10: return launch_tb_d<T, 10>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 11: return launch_tb_d<T, 11>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 12: return launch_tb_d<T, 12>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 13: return launch_tb_d<T, 13>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 14: return launch_tb_d<T, 14>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 15: return launch_tb_d<T, 15>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 16: return launch_tb_d<T, 16>(sh, path, sig, gout, gpath, gbase, partial, st);
        }
    } else {
        if (sh.d > 8) return launch_tree_backward_wide(sh, path, sig, gout, gpath, gbase, workspace, workspace_bytes, st);
        switch (sh.d) {
            case 2: return launch_tb_d<T, 2>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 3: return launch_tb_d<T, 3>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 4: return launch_tb_d<T, 4>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 5: return launch_tb_d<T, 5>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 6: return launch_tb_d<T, 6>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 7: return launch_tb_d<T, 7>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 8: return launch_tb_d<T, 8>(sh, path, sig, gout, gpath, gbase, partial, st);
        }
    }
    return hipErrorNotSupported;
}

}  // namespace
}  // namespace sig

#endif  // SIG_TREE_BACKWARD_IMPL_H_
