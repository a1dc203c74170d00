// Signatures in stream mode, a lane per increment (fp32, d = 2..7): sixty-four increments at a time.
//
// The other stream kernels fold one increment after the other, or cut the paths into chunks and scan them twice around a running product: three launches.
// Here a wavefront takes a word p of N - 2 letters and everything below it.  A lane forms its increment's Horner terms Hh^(k) at the
// prefixes of p as the prefix-tree kernels do; what increments add to a scalar is summed over the lanes of the wavefront (six DPP
// additions), so every lane has the scalar after its increment, and the last lane's is what the next sixty-four begin with.
// Words below a common prefix u share a workgroup, which puts the rows together in LDS and stores each level's part of a row in one run.
//
// Few paths wait for the sums: d (d + 1) of them a wavefront and sixty-four increments, 12 instructions each (1.5 us at d = 4, 4 at d = 7); many for the
// stores of partial lines.  Of two wavefronts' halves with sixteen lanes each the sums would be cheaper but the chain four times as long.
// Rows looked up one scalar at a time (a division each) took 1.3 times the time, sums one after the other 1.15.
// 32 paths of 401 points, d = 4, N = 4: 29 us in sig_mfma_d4_shard.hip, 18 here.  A scalar is a sum over a tree instead of a chain: 0.3 to 0.9 of the error.
#include "sig_internal.h"
#include "sig_tile_common.h"

namespace sig {
namespace {

constexpr int kTsRows = 64;   // increments at a time, a row of output each

template <int D, int N>
struct TileStreamShape {
    static constexpr int M = N - 2;                                            // letters of a wavefront's word
    static constexpr int kMost = D == 2 ? 3 : D == 3 ? 2 : 1;
    static constexpr int X = M < kMost ? M : kMost;                            // ... below u
    static constexpr int Y = M - X;                                            // letters of u
    static constexpr int kWaves = int(tl_pow(D, X)), kThreads = 64 * kWaves;
    static constexpr int kGroups = int(tl_pow(D, Y));                          // workgroups of a path
    static constexpr int count(int k) { return k <= Y ? 1 : int(tl_pow(D, k - Y)); }   // scalars of level k in a row of the workgroup
    static constexpr int at(int k)
    {
        int o = 0;
        for (int j = 1; j < k; ++j) o += count(j);
        return o;
    }
    static constexpr int kScalars = at(N + 1), kSlots = (kScalars + 63) / 64;  // of a row of the workgroup, and of a lane of them
    static constexpr int kTogether = kScalars <= 32 ? 64 / kScalars : 1;       // rows a wavefront stores at once
    static constexpr int kPitch = kScalars | 1;                               // lanes that write a column fall on different banks
    static constexpr int kBytes = kTsRows * kPitch * 4;
    static_assert(kBytes <= 110 * 1024);
    // wavefronts per SIMD at least: what the code behind the last row needs must not take them (d = 6, N = 5, 35 x 23 points: 24.0 us with four, 20.8 with five)
    static constexpr int kOccupancy = D == 4 ? 8 : D == 6 ? 5 : D == 7 ? 4 : 1;
};

// The sums over the lanes up to this one of several values, side by side: a step waits for the one before.
template <int COUNT>
__device__ __forceinline__ void ts_sums(float (&v)[COUNT])
{
    tl_prefixes(v);
    // Lane 15 of the row before to rows 1 and 3, then lane 31 to the upper half.  In assembly: from the builtins the compiler makes three instructions of
    // an addition whose other rows stay as they are.  (s_nop: a DPP operand has to be two instructions old.)
#pragma unroll
    for (int i = 0; i < COUNT; ++i) asm volatile("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf" : "+v"(v[i]));
#pragma unroll
    for (int i = 0; i < COUNT; ++i) asm volatile("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf" : "+v"(v[i]));
}
__device__ __forceinline__ float ts_sum(float v)
{
    float x[1] = {v};
    ts_sums(x);
    return x[0];
}
// The value one lane down, `first` in lane 0.
__device__ __forceinline__ float ts_before(float v, float first)
{
    return tl_float(__builtin_amdgcn_update_dpp(int(tl_bits(first)), int(tl_bits(v)), 0x138, 0xf, 0xf, false));   // wave_shr:1
}
__device__ __forceinline__ float ts_last(float v) { return tl_float(__builtin_amdgcn_readlane(tl_bits(v), 63)); }

template <int D, int N>
__global__ void __launch_bounds__((TileStreamShape<D, N>::kThreads), (TileStreamShape<D, N>::kOccupancy))
sig_tile_stream_kernel(Shape sh, const float *__restrict__ path, const float *__restrict__ initial, float *__restrict__ result)
{
    using TS = TileStreamShape<D, N>;
    constexpr int M = TS::M, Y = TS::Y;
    constexpr int64_t kS = tl_off(D, N + 1);
    extern __shared__ __align__(16) float rows[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // a path's workgroups, eight apart, share an L2: the lines between two runs of a row are put together there
    const unsigned block = blockIdx.x, octets = unsigned(sh.B) / 8 * 8 * TS::kGroups;
    const int64_t row = block < octets ? block / (8 * TS::kGroups) * 8 + block % 8 : block / TS::kGroups;
    const int u = int(block < octets ? block / 8 % TS::kGroups : block % TS::kGroups);
    const float *x = path + row * sh.L * D;
    float *out = result + row * sh.n_inc * kS;
    const float *points = x + (sh.basepoint ? 0 : D);   // where the increments end
    const int n_inc = int(sh.n_inc);

    // Whether the rows are formed once more (see sig_tile_common.h), and what that needs.  Kept in registers up to there it would take more than 80 scalar ones,
    // with which a SIMD holds seven wavefronts (673 x 81 points, d = 3, N = 4: 13.9 us, 12.4 with 78).
    struct Cold {
        int anew, first_word;
        const float *points, *base, *initial;
        float *out;
        int n_inc;
    };
    __shared__ Cold cold;
    if (tid == 0) {
        const float *bpv = static_cast<const float *>(sh.basepoint_value);
        cold = {0, u * TS::kWaves * D, points, !sh.basepoint ? x : bpv != nullptr ? bpv + row * D : nullptr,
                initial != nullptr ? initial + row * kS : nullptr, out, n_inc};
    }

    int letter[M + 1];
    {
        int rest = u * TS::kWaves + wave;
#pragma unroll
        for (int j = M; j >= 1; --j) {
            letter[j] = rest % D;
            rest /= D;
        }
    }
    float start[D], last[D], hi[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
        const float *bpv = static_cast<const float *>(sh.basepoint_value);
        start[c] = last[c] = !sh.basepoint ? x[c] : bpv != nullptr ? bpv[row * D + c] : 0.f;
        hi[c] = points[int64_t(lane < n_inc ? lane : n_inc - 1) * D + c];
    }
    float rf[N + 1];
#pragma unroll
    for (int k = 0; k <= N; ++k) rf[k] = tl_inv_factorial(k);
    // the signature before the current sixty-four: the word's prefixes, the word, and below
    float ca[M + 1] = {}, cb[D] = {}, cc[D][D] = {}, first1[D] = {};
    if (initial != nullptr) {   // what came before the path: the sums begin with it
        const float *from = initial + row * kS;
        int rest = u * TS::kWaves + wave;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            first1[c] = from[c];
            cb[c] = from[tl_off(D, N - 1) + rest * D + c];
#pragma unroll
            for (int k = 0; k < D; ++k) cc[c][k] = from[tl_off(D, N) + (int64_t(rest) * D + c) * D + k];
        }
#pragma unroll
        for (int j = M; j >= 2; --j) {
            ca[j] = from[tl_off(D, j) + rest];
            rest /= D;
        }
    }
    float *my = rows + lane * TS::kPitch;
    // Where the lane's scalars of a row of the workgroup are, and where they go in a row of the result, in bytes.  Lanes without one, and those of a prefix of u that
    // belongs to an earlier workgroup, store the row's last scalar once more.
    const int my_row = TS::kTogether == 1 ? 0 : lane / TS::kScalars, my_first = TS::kTogether == 1 ? lane : lane % TS::kScalars;
    unsigned from[TS::kSlots], slot[TS::kSlots];
#pragma unroll
    for (int r = 0; r < TS::kSlots; ++r) {
        const int e = my_first + 64 * r;
        from[r] = TS::kScalars - 1;
        slot[r] = unsigned(tl_off(D, N)) + unsigned(u + 1) * TS::count(N) - 1;
        bool first = true;   // a prefix of u is written by the first workgroup below it
        int prefix = u;
#pragma unroll
        for (int k = N; k >= 1; --k) {
            if (k < Y) {
                first = first && prefix % D == 0;
                prefix /= D;
            }
            const int n = TS::count(k), i = e - TS::at(k);
            if (i >= 0 && i < n && first) {
                from[r] = e;
                slot[r] = unsigned(tl_off(D, k)) + (k > Y ? unsigned(u) * n : prefix) + i;
            }
        }
        from[r] = (my_row * TS::kPitch + from[r]) * 4;
        slot[r] = (my_row * unsigned(kS) + slot[r]) * 4;
    }

    int infinite = 0;                // an increment was
    bool broken = false;             // an increment up to the current sixty-four was not finite
    float broken1[D] = {}, last1[D] = {};   // ... NaN in its channels, and level 1 before them
    for (int t0 = 0; t0 < n_inc; t0 += kTsRows) {
        const int nt = n_inc - t0 < kTsRows ? n_inc - t0 : kTsRows;
        float z[D], level1[D], before1[D];
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const float lo = ts_before(hi[c], last[c]);
            z[c] = hi[c] - lo;
            level1[c] = hi[c] - start[c] + first1[c];
            before1[c] = lo - start[c] + first1[c];
            last[c] = ts_last(hi[c]);
        }
        // Level 1 is a difference of points: what a sum of the increments would have kept of one that is not finite is put back.
        float zeros = 0.f;
#pragma unroll
        for (int c = 0; c < D; ++c) zeros = __builtin_fmaf(0.f, z[c], zeros);
        broken = broken || __builtin_amdgcn_ballot_w64(!(zeros == 0.f)) != 0;
        if (broken) {
#pragma unroll
            for (int c = 0; c < D; ++c) {
                if (__builtin_amdgcn_ballot_w64(__builtin_isinf(z[c])) != 0) infinite = 1;
                const float sum = broken1[c] + ts_sum(0.f * z[c]);
                const float first = t0 == 0 ? first1[c] : last1[c];
                level1[c] += ts_before(sum, broken1[c]);
                broken1[c] = ts_last(sum);
                before1[c] = ts_before(level1[c], first);
            }
        }
#pragma unroll
        for (int c = 0; c < D; ++c) last1[c] = ts_last(level1[c]);
        if (t0 + kTsRows < n_inc) {   // the next points are on their way meanwhile
            const int64_t i = t0 + kTsRows + lane < n_inc ? t0 + kTsRows + lane : n_inc - 1;
#pragma unroll
            for (int c = 0; c < D; ++c) hi[c] = points[i * D + c];
        }
        const auto of = [&](const float (&v)[D], int c) {   // c the same in all lanes
            float r = v[0];
#pragma unroll
            for (int k = 1; k < D; ++k) r = c == k ? v[k] : r;
            return r;
        };
        // ---- the word's prefixes
        float Hh[N + 1];
        {
            const float z1 = of(z, letter[1]), a1 = of(before1, letter[1]), l1 = of(level1, letter[1]);
#pragma unroll
            for (int k = 2; k <= N; ++k) Hh[k] = __builtin_fmaf(z1, rf[k], a1 * rf[k - 1]);
            constexpr int kBelow = int(tl_pow(D, M - 1 < TS::X ? M - 1 : TS::X));   // wavefronts with the same first letter
            if (wave % kBelow == 0) my[TS::at(1) + (Y >= 1 ? 0 : wave / kBelow)] = l1;
        }
#pragma unroll
        for (int j = 2; j <= M; ++j) {
            const float zj = of(z, letter[j]), after = ca[j] + ts_sum(Hh[j] * zj), a = ts_before(after, ca[j]);
            ca[j] = ts_last(after);
            const int below = int(tl_pow(D, M - j < TS::X ? M - j : TS::X));
            if (wave % below == 0) my[TS::at(j) + (j <= Y ? 0 : wave / below)] = after;
#pragma unroll
            for (int k = j + 1; k <= N; ++k) Hh[k] = __builtin_fmaf(Hh[k], zj, k == j + 1 ? a : a * rf[k - j]);
        }
        // ---- the two deepest levels
        float *mb = my + TS::at(N - 1) + wave * D, *mc = my + TS::at(N) + wave * D * D;
        float after[D];
#pragma unroll
        for (int b = 0; b < D; ++b) after[b] = Hh[N - 1] * z[b];
        ts_sums(after);
#pragma unroll
        for (int b = 0; b < D; ++b) {
            after[b] += cb[b];
            mb[b] = after[b];
            const float h = __builtin_fmaf(Hh[N], z[b], ts_before(after[b], cb[b]));
            cb[b] = ts_last(after[b]);
            float v[D];
#pragma unroll
            for (int c = 0; c < D; ++c) v[c] = h * z[c];
            ts_sums(v);
#pragma unroll
            for (int c = 0; c < D; ++c) {
                v[c] += cc[b][c];
                cc[b][c] = ts_last(v[c]);
                mc[b * D + c] = v[c];
            }
        }
        // A scalar that is not finite stays so to the end of the path.  Where a point is not a number that is as it should be; an infinity or an overflow
        // is summed in another order here, and may be NaN only for that.  (Ahead of the last rows' stores: behind them this would wait for them.)
        if (t0 + kTsRows >= n_inc) {
            const auto each = [&](auto look_at) {
#pragma unroll
                for (int j = 2; j <= M; ++j) look_at(0, ca[j]);
#pragma unroll
                for (int b = 0; b < D; ++b) {
                    look_at(b, cb[b]);
#pragma unroll
                    for (int c = 0; c < D; ++c) look_at(b + c, cc[b][c]);
                }
            };
            float sums[4] = {};
            each([&](int i, float v) { sums[i & 3] = __builtin_fmaf(0.f, v, sums[i & 3]); });
            if (__builtin_expect(!(sums[0] + sums[1] + sums[2] + sums[3] == 0.f) || broken, 0)) {
                each([&](int, float v) { infinite |= __builtin_isinf(v); });
                if (lane == 0 && (infinite || !broken)) cold.anew = 1;
            }
        }
        lds_barrier();   // not __syncthreads(): the next points and the rows' stores stay in flight
        // ---- the rows, a wavefront at a time
        char *to = reinterpret_cast<char *>(out + int64_t(t0) * kS);
#pragma unroll 4
        for (int t = wave * TS::kTogether; t < nt; t += TS::kWaves * TS::kTogether) {
            if (TS::kTogether > 1 && (my_row >= TS::kTogether || t + my_row >= nt)) continue;
            char *row_to = to + t * kS * 4;
            const char *row_from = reinterpret_cast<const char *>(rows + t * TS::kPitch);
            float v[TS::kSlots];
#pragma unroll
            for (int r = 0; r < TS::kSlots; ++r) v[r] = *reinterpret_cast<const float *>(row_from + from[r]);
#pragma unroll
            for (int r = 0; r < TS::kSlots; ++r) *reinterpret_cast<float *>(row_to + slot[r]) = v[r];
        }
        lds_barrier();
    }

    if (__builtin_expect(cold.anew, 0)) {
        __threadfence();   // the rows stored so far lie under those to come
        __syncthreads();
        const auto uniform = [](const float *p) {
            const uint64_t v = reinterpret_cast<uint64_t>(p);
            const unsigned high = __builtin_amdgcn_readfirstlane(unsigned(v >> 32)), low = __builtin_amdgcn_readfirstlane(unsigned(v));   // (int: would carry its sign)
            return reinterpret_cast<float *>(uint64_t(high) << 32 | low);
        };
        float *to = uniform(cold.out);
        const int n = __builtin_amdgcn_readfirstlane(cold.n_inc), thread = wave * 64 + lane, word = cold.first_word + thread;
        if (thread < TS::kWaves * D)
            tl_one_by_one<D, N>(uniform(cold.points), n, uniform(cold.base), uniform(cold.initial), word,
                                [&](int64_t s, const float(&a)[N], const float(&leaf)[D]) { tl_store_word<D, N>(to + s * kS, word, a, leaf); });
    }
}

template <int D, int N>
hipError_t launch_tile_stream_dn(const Shape &sh, const float *path, const float *initial, float *out, hipStream_t st)
{
    using TS = TileStreamShape<D, N>;
    if (!grid_holds(sh.B * TS::kGroups, TS::kThreads)) return hipErrorNotSupported;
    if (TS::kBytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(sig_tile_stream_kernel<D, N>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, TS::kBytes);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((sig_tile_stream_kernel<D, N>), dim3(unsigned(sh.B * TS::kGroups)), dim3(TS::kThreads), TS::kBytes, st, sh, path, initial,
                       out);
    return hipGetLastError();
}

template <int D>
hipError_t launch_tile_stream_d(const Shape &sh, const float *path, const float *initial, float *out, hipStream_t st)
{
    switch (sh.N) {
        case 3: return launch_tile_stream_dn<D, 3>(sh, path, initial, out, st);
        case 4: return launch_tile_stream_dn<D, 4>(sh, path, initial, out, st);
        case 5: return launch_tile_stream_dn<D, 5>(sh, path, initial, out, st);
    }
    if constexpr (D <= 4)
        if (sh.N == 6) return launch_tile_stream_dn<D, 6>(sh, path, initial, out, st);
    if constexpr (D <= 3)
        if (sh.N == 7) return launch_tile_stream_dn<D, 7>(sh, path, initial, out, st);
    if constexpr (D == 2)
        if (sh.N == 8) return launch_tile_stream_dn<D, 8>(sh, path, initial, out, st);
    return hipErrorNotSupported;
}

}  // namespace

// The longest path, in increments, up to which that is faster than what serves these calls otherwise, by the number of paths, and with more than 64
// paths the largest output, in millions of scalars.
//  - Sixty-four increments take a workgroup 1 to 6 us however long the path is.  The kernels before cut a path into chunks, the more of them the longer it
//    is and the fewer paths there are (sig_api.hip, stream_chunks: 32 for up to 64 paths of 4096 increments, 16 up to 128, 8 up to 256, 4 up to 512):
//    their time grows with the square root.  One path, us, before | now: d = 3, N = 4 1000 increments 39 | 39, 4000 73 | 145, 60 000 507 | 2124; d = 2,
//    N = 4 4000 85 | 67, 8000 97 | 130; d = 5, N = 4 4000 194 | 189, 60 000 737 | 2780; d = 6, N = 4 1000 91 | 72, 60 000 639 | 4088.
//  - Many paths of large signatures are bound by the stores, which the kernels before do in whole rows: with an output around the 256 MB of the
//    last-level cache they are ahead (400 paths, d = 2, N = 7, 700 increments, 284 MB, 0.65 of their time, 1500 1.22; 128, d = 3, N = 5, 1000
//    increments, 186 MB, 0.97, 1500 1.28).
// Timed over 1600 shapes of up to 100 000 increments.
struct LongestPath {
    int d, N, paths_8, paths_32, paths_64, paths_128, more;   // up to so many paths
    int millions;
};
constexpr int kAny = 0x7fffffff;
constexpr LongestPath kLongest[] = {
    {2, 3, 2000, 2000, 2000, kAny, kAny, kAny}, {2, 4, 4095, 4095, kAny, kAny, kAny, kAny}, {2, 5, 4095, 4095, kAny, kAny, kAny, kAny},
    {2, 6, 4095, 4095, 20000, kAny, kAny, 300}, {2, 7, 20000, 20000, 40000, kAny, kAny, 75}, {2, 8, 20000, 20000, 4000, kAny, kAny, 55},
    {3, 3, 3000, 3000, 3000, kAny, kAny, kAny}, {3, 4, 1000, 1000, 1000, 1300, kAny, kAny}, {3, 5, 1000, 1000, 1000, kAny, kAny, 50},
    {3, 6, 3500, 3500, 1500, 1000, 1000, kAny}, {3, 7, 8000, 1500, 1000, 1000, 1000, kAny}, {4, 3, 1000, 1000, 1000, 3000, kAny, kAny},
    {5, 3, 400, 400, 400, 400, 400, kAny},      {5, 4, 4000, 3500, 4000, kAny, kAny, 50},   {5, 5, 8000, 4000, 1500, 1500, 1500, kAny},
    {6, 3, 300, 300, 300, 300, 300, kAny},      {6, 4, 1500, 2000, 2000, 2000, 2000, 120}, {7, 3, 160, 160, 160, 160, 160, kAny},
    {7, 4, 1200, 2000, 1500, 1500, 1500, kAny},   // the others' kernels are not cut, or slower at any length (d = 4, N = 4..6; d = 6, 7 at N = 5)
};
static bool short_enough(const Shape &sh)
{
    for (const LongestPath &l : kLongest)
        if (l.d == sh.d && l.N == sh.N) {
            if (sh.B > 64 && sh.B * sh.n_inc * sh.S > int64_t(l.millions) * 1000000) return false;
            return sh.n_inc <= (sh.B <= 8     ? l.paths_8
                                : sh.B <= 32  ? l.paths_32
                                : sh.B <= 64  ? l.paths_64
                                : sh.B <= 128 ? l.paths_128
                                              : l.more);
        }
    return true;
}

// Where it pays otherwise, both timed over 700 shapes of up to 1100 points (rows of B S scalars side by side; us, before | now).  A full chip stores
// 2.5 to 4 TB/s:
//  - the kernels before wait 0.3 to 0.45 us for an increment or, in chunks, some 20 to 60 for three launches: 64 x 101 points, d = 5, N = 4 27 | 12;
//    25 x 165, d = 7, N = 5 763 | 101; 8 x 227, d = 4, N = 5 24 | 12.  Under 20 increments most lanes have none.
//  - with many paths they store up to 6 TB/s: 745 x 119, d = 4, N = 4 23 | 34, 1287 x 20, d = 5, N = 4 17 | 36; at d = 4, N = 5 from 30 paths on
//    (55 x 84 11.6 | 12.8).
//  - at depth 3 from 5 channels on a path is a single workgroup of d (d + 1) sums a wavefront, and from some length on the chunks are ahead:
//    11 x 469, d = 5 26 | 24, 18 x 1047 37 | 50; 1 x 507, d = 6 26 | 32; 10 x 108, d = 7 17 | 12, 9 x 342 25 | 31.
// Over 400 drawn shapes of that range the rule takes 0.60 of the time and has 0.80 of the error of before.
bool tile_stream_preferred(const Shape &sh)
{
    if (!sh.stream || sh.chunks != 1 || sh.rows_in_stream || !sh.from_identity || sh.d < 2 || sh.d > 7 || sh.N < 3 || sh.n_inc < 20 || sh.n_inc >= (1 << 30))
        return false;
    if (sh.N > (sh.d == 2 ? 8 : sh.d == 3 ? 7 : sh.d == 4 ? 6 : 5) || !short_enough(sh)) return false;
    const int64_t k = 1000;
    const int64_t most = sh.d <= 3    ? (sh.d == 3 && sh.N == 5 ? 100 * k : 120 * k)   // 300 x 21, d = 3, N = 5 10.3 | 12.5
                         : sh.d == 4  ? (sh.N == 3 ? 120 * k : sh.N == 4 ? 54 * k : sh.N == 5 ? 24 * k : 80 * k)
                         : sh.N == 3  ? (sh.d == 7 ? 40 * k : 120 * k)
                         : sh.N == 4  ? 150 * k
                         : sh.d == 5  ? 250 * k
                                      : 500 * k;
    return sh.B * sh.S <= most;
}

hipError_t launch_tile_stream_f32(const Shape &sh, const float *path, const float *initial, float *out, hipStream_t st)
{
    switch (sh.d) {
        case 2: return launch_tile_stream_d<2>(sh, path, initial, out, st);
        case 3: return launch_tile_stream_d<3>(sh, path, initial, out, st);
        case 4: return launch_tile_stream_d<4>(sh, path, initial, out, st);
        case 5: return launch_tile_stream_d<5>(sh, path, initial, out, st);
        case 6: return launch_tile_stream_d<6>(sh, path, initial, out, st);
        case 7: return launch_tile_stream_d<7>(sh, path, initial, out, st);
    }
    return hipErrorNotSupported;
}

}  // namespace sig
