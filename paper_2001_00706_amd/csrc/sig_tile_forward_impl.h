// Signatures in final mode, tile family (fp32, d = 5..16, from depth 4 to 6 on): sixteen increments at a time, the two deepest levels as a product on
// the matrix cores.
//
// The other vector kernels fold one increment after the other into the top level, a multiply-add per scalar and 0.25 to 0.3 us an increment
// where few wavefronts share a SIMD.  With p a word of N - 2 letters, z increment s, q the path's end minus the point that ends it, and U, V the Horner
// terms of sig_tile_backward_impl.h at p before the increment, Abel summation over the increments makes the two deepest levels
//     A_N[p w j] = sum_s V_s[p] z_s[w] z_s[j] + U_s[p] z_s[w] q_s[j],      A_{N-1}[p w] = sum_s U_s[p] z_s[w],
// a product of [words x 2 increments] with [2 increments x d (d + 1)] (level N - 1 is the column where q counts as one).  A tile of
// sixteen increments is one step of K = 32 of v_mfma_f32_16x16x32_bf16, six of them for the pieces of 32-bit operands (sig_tile_common.h).  The levels
// above are prefix sums over the sixteen lanes of a row, a lane per increment.
//
// Up to 8 channels a wavefront takes four prefixes of N - 3 letters and all words below them, two results of sixteen words; beyond, one prefix.
// The right operands are the same for all of a path's wavefronts: a workgroup forms them together.
//
// Bound by the vector instructions that form U and V and cut them into pieces (some 60 per tile and word); the products take a fifth of a tile.
// 32 paths of 128 points, d = N = 7: 180 us in the prefix tree, 145 here; d = 13 N = 5, 22 paths of 171 increments 123 | 54.  The error is 0.6 to 1
// of the tree's (0.86 over 50 drawn shapes, none above 1.05), whose top level has a rounding per increment where this one has one per tile.
#ifndef SIG_TILE_FORWARD_IMPL_H_
#define SIG_TILE_FORWARD_IMPL_H_

#include "sig_internal.h"
#include "sig_tile_common.h"

namespace sig {
namespace {

template <int D, int N>
struct TileForwardShape {
    static constexpr int M = N - 2;                               // letters of a word
    static constexpr int LW = D <= 8 ? 8 : 16;
    static constexpr int RB = D <= 8 ? 2 : 1;                     // results of sixteen words a wavefront has
    static constexpr int LL = D <= 8 ? D : 4;                     // words of a lane
    static constexpr int kPrefixes = int(tl_pow(D, M - 1));
    static constexpr int kUnits = D <= 8 ? (kPrefixes + 3) / 4 : kPrefixes;   // wavefronts of a path
    static constexpr int kGroups = (kUnits + 7) / 8;              // workgroups of a path
    static constexpr int kWaves = (kUnits + kGroups - 1) / kGroups;
    static constexpr int kCols = D * (D + 1), CT = (kCols + 15) / 16;   // columns w (d + 1) + j, and tiles of sixteen
    static constexpr int kTiles = CT <= 2 ? 4 : CT <= 4 ? 2 : 1;  // tiles staged at a time
    static constexpr int kSpan = 16 * kTiles;
    static constexpr int ZR = LW + 4;                             // floats of an increment's row: sixteen rows fall on different banks
    static constexpr int kTrans = 2 * 16 * 20;                    // U and V on their way from a lane per increment to a lane per word
    // LDS, in floats: increments and level 1 before them by increment, increments and rests by channel, right operands, U and V
    static constexpr int kAtPos = kSpan * ZR, kAtZt = 2 * kSpan * ZR, kAtQt = kAtZt + (D + 1) * kSpan, kAtOps = kAtQt + (D + 1) * kSpan;
    static constexpr int kAtTrans = kAtOps + kTiles * CT * 3 * 256, kLds = kAtTrans + kWaves * kTrans;
    static_assert(kLds * 4 <= 80 * 1024 && kAtOps % 4 == 0 && kAtZt % 4 == 0);
    // wavefronts per SIMD at least; four where a few registers more than 128 would leave a workgroup of eight wavefronts a compute unit for itself (d = 14,
    // N = 5, 15 x 239 points: 71 us, 98 with 129)
    static constexpr int kOccupancy = (D == 8 && N == 8) || (D == 14 && N == 5) || (D == 15 && N == 6) ? 4 : 2;
};

template <int D, int N>
__global__ void __launch_bounds__((64 * TileForwardShape<D, N>::kWaves), (TileForwardShape<D, N>::kOccupancy))
sig_tile_forward_kernel(Shape sh, const float *__restrict__ path, float *__restrict__ result)
{
    using TS = TileForwardShape<D, N>;
    constexpr int M = TS::M, LW = TS::LW, LL = TS::LL, RB = TS::RB, CT = TS::CT, ZR = TS::ZR, NT = 64 * TS::kWaves, kSpan = TS::kSpan;
    constexpr int64_t kS = tl_off(D, N + 1);
    extern __shared__ __align__(16) float lds[];
    float *zf = lds, *pf = lds + TS::kAtPos, *zt = lds + TS::kAtZt, *qt = lds + TS::kAtQt;
    TlWords *ops = reinterpret_cast<TlWords *>(lds + TS::kAtOps);   // [tile][columns' tile][high, middle, low][lane]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *trans = lds + TS::kAtTrans + wave * TS::kTrans;          // [U, V][word][20]
    const int s = lane & 15, q = lane >> 4;
    const int64_t row = blockIdx.x / unsigned(TS::kGroups);
    const int unit = int(blockIdx.x - unsigned(row) * unsigned(TS::kGroups)) * TS::kWaves + wave;
    const float *x = path + row * sh.L * D;
    const float *bpv = static_cast<const float *>(sh.basepoint_value);

    // the lane's prefix and the letters of its words: four prefixes by row of lanes, or one prefix and letters 4q .. 4q + 3
    const int prefix_raw = LW == 8 ? unit * 4 + q : unit, letter0 = LW == 8 ? 0 : 4 * q;
    const bool there = prefix_raw < TS::kPrefixes;
    const int prefix = there ? prefix_raw : 0;
    int cl[M];
    {
        int rest = prefix;
#pragma unroll
        for (int j = M - 1; j >= 1; --j) {
            cl[j] = rest % D;
            rest /= D;
        }
    }
    float wild = 0.f;   // NaN if an increment of the first letter is not finite, or a scalar
    float ca[M] = {}, cam[LL] = {};   // the signature at its prefixes of 2 .. letters and at the words, before the current tile
    f4 acc[RB][CT];
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int t = 0; t < CT; ++t) acc[b][t] = f4{0.f, 0.f, 0.f, 0.f};
    float rf[N + 1];
#pragma unroll
    for (int k = 0; k <= N; ++k) rf[k] = tl_inv_factorial(k);

    for (int64_t t0 = 0; t0 < sh.n_inc; t0 += kSpan) {
        const int nt = int(sh.n_inc - t0 < kSpan ? sh.n_inc - t0 : kSpan);
        __syncthreads();   // the last span's operands have been read
        for (int e = tid; e < kSpan * LW; e += NT) {
            const int i = e / LW, c = e % LW, cc = c < D ? c : 0;
            const bool on = c < D && i < nt;
            const int64_t i_hi = (on ? t0 + i : 0) + (sh.basepoint ? 0 : 1);
            const float *at = x + i_hi * D + cc;
            const float end = x[(sh.L - 1) * D + cc], base = !sh.basepoint ? x[cc] : bpv != nullptr ? bpv[row * D + cc] : 0.f;
            const float hi = at[0], lo = i_hi > 0 ? at[-D] : base, z = on ? hi - lo : 0.f;
            zf[i * ZR + c] = z;
            pf[i * ZR + c] = on ? lo - base : 0.f;
            if (c < D) {
                zt[c * kSpan + i] = z;
                qt[c * kSpan + i] = on ? end - hi : 0.f;
            }
        }
        for (int i = tid; i < kSpan; i += NT) {   // the column of level N - 1
            zt[D * kSpan + i] = 0.f;
            qt[D * kSpan + i] = 1.f;
        }
        __syncthreads();
        // ---- the right operands: lane (column, quarter of the increments), its four increments with U and with V
        for (int e = wave; e < TS::kTiles * CT; e += TS::kWaves) {
            const int tile = e / CT, n = (e % CT) * 16 + s, w = n / (D + 1), j = n % (D + 1), at = tile * 16 + 4 * q;
            const bool on = n < TS::kCols;
            const f4 zw = *reinterpret_cast<const f4 *>(zt + (on ? w : D) * kSpan + at);
            const f4 zj = *reinterpret_cast<const f4 *>(zt + j * kSpan + at), qj = *reinterpret_cast<const f4 *>(qt + j * kSpan + at);
            unsigned h[8], m[8], l[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const TlPieces p = tl_split(zw[k & 3] * (k < 4 ? qj[k & 3] : zj[k & 3]));
                h[k] = p.h;
                m[k] = p.m;
                l[k] = p.l;
            }
            TlWords *o = ops + e * 192 + lane;
            o[0] = TlWords{tl_pack(h[0], h[1]), tl_pack(h[2], h[3]), tl_pack(h[4], h[5]), tl_pack(h[6], h[7])};
            o[64] = TlWords{tl_pack(m[0], m[1]), tl_pack(m[2], m[3]), tl_pack(m[4], m[5]), tl_pack(m[6], m[7])};
            o[128] = TlWords{tl_pack(l[0], l[1]), tl_pack(l[2], l[3]), tl_pack(l[4], l[5]), tl_pack(l[6], l[7])};
        }
        __syncthreads();

        for (int tile = 0; tile <= (nt - 1) >> 4; ++tile) {
            // ---- the signature before every increment and the Horner terms
            const float *zrow = zf + (tile * 16 + s) * ZR;
            float zc[LL];
#pragma unroll
            for (int i = 0; i < LL; ++i) zc[i] = zrow[letter0 + i];
            const float z1 = zrow[cl[1]], a1 = pf[(tile * 16 + s) * ZR + cl[1]];
            wild = __builtin_fmaf(0.f, z1, wild);
            float Hh[N + 1];   // T^(k)_j / (k-j)! of the prefix of j letters
#pragma unroll
            for (int k = 2; k <= N; ++k) Hh[k] = __builtin_fmaf(z1, rf[k], a1 * rf[k - 1]);
#pragma unroll
            for (int j = 2; j < M; ++j) {
                const float z = zrow[cl[j]], sum = tl_prefix(Hh[j] * z), a = ca[j] + tl_down<1>(sum);
                ca[j] += tl_last(sum);
#pragma unroll
                for (int k = j + 1; k <= N; ++k) Hh[k] = __builtin_fmaf(Hh[k], z, k == j + 1 ? a : a * rf[k - j]);
            }
            float sum[LL], U[LL], V[LL];
#pragma unroll
            for (int i = 0; i < LL; ++i) sum[i] = Hh[M] * zc[i];
            tl_prefixes(sum);
#pragma unroll
            for (int i = 0; i < LL; ++i) {
                const float a = cam[i] + tl_down<1>(sum[i]);
                cam[i] += tl_last(sum[i]);
                U[i] = __builtin_fmaf(Hh[N - 1], zc[i], a);
                V[i] = __builtin_fmaf(Hh[N], zc[i], a * 0.5f);
            }
            // ---- to a lane per word, in pieces
            TlWords A[RB][3];
#pragma unroll
            for (int b = 0; b < RB; ++b) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int k = 4 * b + i;
                    trans[(4 * q + i) * 20 + s] = k < LL ? U[k < LL ? k : 0] : 0.f;
                    trans[320 + (4 * q + i) * 20 + s] = k < LL ? V[k < LL ? k : 0] : 0.f;
                }
                tl_wave_order();
                const f4 u = *reinterpret_cast<const f4 *>(trans + s * 20 + 4 * q), v = *reinterpret_cast<const f4 *>(trans + 320 + s * 20 + 4 * q);
                tl_wave_order();
                unsigned h[8], m[8], l[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const TlPieces p = tl_split(k < 4 ? u[k & 3] : v[k & 3]);
                    h[k] = p.h;
                    m[k] = p.m;
                    l[k] = p.l;
                }
                A[b][0] = TlWords{tl_pack(h[0], h[1]), tl_pack(h[2], h[3]), tl_pack(h[4], h[5]), tl_pack(h[6], h[7])};
                A[b][1] = TlWords{tl_pack(m[0], m[1]), tl_pack(m[2], m[3]), tl_pack(m[4], m[5]), tl_pack(m[6], m[7])};
                A[b][2] = TlWords{tl_pack(l[0], l[1]), tl_pack(l[2], l[3]), tl_pack(l[4], l[5]), tl_pack(l[6], l[7])};
            }
            // ---- the two deepest levels, the small products first
#pragma unroll
            for (int t = 0; t < CT; ++t) {
                const TlWords *o = ops + (tile * CT + t) * 192 + lane;
                const TlWords Bh = o[0], Bm = o[64], Bl = o[128];
#pragma unroll
                for (int b = 0; b < RB; ++b) acc[b][t] = tl_mfma(A[b][0], Bl, acc[b][t]);
#pragma unroll
                for (int b = 0; b < RB; ++b) acc[b][t] = tl_mfma(A[b][2], Bh, acc[b][t]);
#pragma unroll
                for (int b = 0; b < RB; ++b) acc[b][t] = tl_mfma(A[b][1], Bm, acc[b][t]);
#pragma unroll
                for (int b = 0; b < RB; ++b) acc[b][t] = tl_mfma(A[b][1], Bh, acc[b][t]);
#pragma unroll
                for (int b = 0; b < RB; ++b) acc[b][t] = tl_mfma(A[b][0], Bm, acc[b][t]);
#pragma unroll
                for (int b = 0; b < RB; ++b) acc[b][t] = tl_mfma(A[b][0], Bh, acc[b][t]);
            }
        }
    }

    // ---- results: a lane holds column lane % 16 of four words
    float *out = result + row * kS;
    float wilds[4] = {wild, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int t = 0; t < CT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) wilds[i] = __builtin_fmaf(0.f, acc[b][t][i], wilds[i]);
#pragma unroll
    for (int j = 2; j < M; ++j) wilds[j & 3] = __builtin_fmaf(0.f, ca[j], wilds[j & 3]);
#pragma unroll
    for (int i = 0; i < LL; ++i) wilds[i & 3] = __builtin_fmaf(0.f, cam[i], wilds[i & 3]);
    wild = wilds[0] + wilds[1] + wilds[2] + wilds[3];
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(wild == 0.f)) != 0, 0)) {   // see sig_tile_common.h
        constexpr int kBelow = (LW == 8 ? 4 : 1) * D * D;     // words of N - 1 letters below the wavefront's prefixes
        const float *base = !sh.basepoint ? x : bpv != nullptr ? bpv + row * D : nullptr;
        for (int u = unit * kBelow + lane; u < (unit + 1) * kBelow && u < TS::kPrefixes * D * D; u += 64)
            tl_one_by_one<D, N>(x + (sh.basepoint ? 0 : D), sh.n_inc, base, nullptr, u, [&](int64_t i, const float(&a)[N], const float(&leaf)[D]) {
                if (i + 1 == sh.n_inc) tl_store_word<D, N>(out, u, a, leaf);
            });
        return;
    }
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int t = 0; t < CT; ++t) {
            const int n = t * 16 + s, w = n / (D + 1), j = n % (D + 1);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int letter = LW == 8 ? 4 * b + i : 4 * q + i;
                if (there && letter < D && n < TS::kCols) {
                    const int64_t p = int64_t(prefix) * D + letter;
                    out[j < D ? tl_off(D, N) + (p * D + w) * D + j : tl_off(D, N - 1) + p * D + w] = acc[b][t][i];
                }
            }
        }
    if (there && s == 0) {
#pragma unroll
        for (int i = 0; i < LL; ++i)
            if (letter0 + i < D) out[tl_off(D, M) + int64_t(prefix) * D + letter0 + i] = cam[i];
        if (letter0 == 0) {   // a prefix of the prefix is written by the first wavefront or row below it
            int rest = prefix;
            bool first = true;
#pragma unroll
            for (int j = M - 1; j >= 1; --j) {
                if (first) {
                    if (j >= 2) {
                        out[tl_off(D, j) + rest] = ca[j];
                    } else {
                        const float base = !sh.basepoint ? x[rest] : bpv != nullptr ? bpv[row * D + rest] : 0.f;
                        out[rest] = x[(sh.L - 1) * D + rest] - base;
                    }
                }
                first = first && cl[j] == 0;
                rest /= D;
            }
        }
    }
}

template <int D, int N>
hipError_t launch_tile_forward_dn(const Shape &sh, const float *path, float *out, hipStream_t st)
{
    using TS = TileForwardShape<D, N>;
    constexpr int kBytes = TS::kLds * int(sizeof(float));
    if (!grid_holds(sh.B * TS::kGroups, 64 * TS::kWaves)) return hipErrorNotSupported;
    if (kBytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(sig_tile_forward_kernel<D, N>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((sig_tile_forward_kernel<D, N>), dim3(unsigned(sh.B * TS::kGroups)), dim3(64 * TS::kWaves), kBytes, st, sh, path, out);
    return hipGetLastError();
}

}  // namespace

// One channel count, the depths that tile_forward_preferred takes.
template <int D>
hipError_t launch_tile_forward_d(const Shape &sh, const float *path, float *out, hipStream_t st)
{
    if constexpr (D >= 8)
        if (sh.N == 4) return launch_tile_forward_dn<D, 4>(sh, path, out, st);
    if constexpr (D >= 7)
        if (sh.N == 5) return launch_tile_forward_dn<D, 5>(sh, path, out, st);
    if (sh.N == 6) return launch_tile_forward_dn<D, 6>(sh, path, out, st);
    if constexpr (D <= 8) {
        if (sh.N == 7) return launch_tile_forward_dn<D, 7>(sh, path, out, st);
        if (sh.N == 8) return launch_tile_forward_dn<D, 8>(sh, path, out, st);
    }
    return hipErrorNotSupported;
}

}  // namespace sig

#endif  // SIG_TILE_FORWARD_IMPL_H_
