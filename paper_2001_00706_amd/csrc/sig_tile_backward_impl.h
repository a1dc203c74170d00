// Gradient of the signature with respect to the path, tile family (fp32, final mode, d = 3..16 from depth 4 on): sixteen
// increments at a time, the two deepest levels on the matrix cores.
//
// The other gradient kernels walk a path back one increment after the other because each step needs the state that the one
// before left.  But in final mode the cotangent of the top level is g_N throughout, and what the top two levels contribute is a
// product of g_N with the increments.  With p a word of N - 2 letters, z the increment s, q the path's end minus the point that ends
// the increment (level 1 of what follows it), and Hh as in sig_tree_backward_impl.h, V = Hh^(N)_{N-2}[p], U = Hh^(N-1)_{N-2}[p]:
//     D[p w]  = sum_j g_N[p w j] z[j]                    (cotangent of Hh^(N)_{N-1})
//     D2[p w] = g_{N-1}[p w] + sum_j g_N[p w j] q[j]     (cotangent of the signature's level N - 1 after the increment)
//     H[p j]  = sum_w g_N[p w j] z[w]
//     dz[w]  += sum_p V[p] D[p w] + U[p] D2[p w],   dz[j] += sum_p V[p] H[p j]  +  sum over w, p of g_N[p w j] A_{N-1}[p w],
//     e1[p]   = sum_w D[p w] z[w],   e2[p] = sum_w D2[p w] z[w]        (cotangents of V and U)
// where the last sum of dz[j] is its value at the end of the path minus sum_p U[p] H[p j] of every increment from s on, since
// U[p] z[w] is what an increment adds to A_{N-1}[p w].  D, D2 and H are products of a constant matrix with the increments: sixteen words by
// sixteen increments are one result of v_mfma_f32_16x16x32_bf16, a lane per increment and four words.  What is left of a step is
// multiply-adds inside a lane, and the levels up to N - 2: their state at every increment of the tile is the state at the tile's
// end minus a suffix sum of what the increments added, four DPP additions over the sixteen lanes of a row.  So a wavefront keeps
// g_N below sixteen words in registers for the whole path and takes sixteen increments in about the time the prefix-tree kernels
// take for two or three.
//
// The operands are cut into bfloat16 pieces, of which eight products are taken up to eight channels and six beyond (sig_tile_common.h).
//
// A block of sixteen words: a prefix of N - 3 letters and all 16 last letters (9 to 16 channels), two prefixes and 8, or four and 4.  From 9
// channels on two wavefronts share a block, half of the letters w and j each: cotangents are linear, so each carries its share of e1 and
// e2 down the word by itself, and g_N in both orders takes 128 registers instead of 256.
//
// What bounds it is the issue of vector instructions, and the matrix instructions between them, which do not run in their shadow: at d = N = 7
// a tile of 14 words takes 478 and 42 (1.9 ns for a multiply-add of three registers, 1.3 for an addition, 2.1 with DPP, 7.3 for a matrix
// instruction: 1.16 us a SIMD, measured 1.16).  Neither more wavefronts per SIMD (products and chains in wavefronts of their own) nor another
// order of the instructions changed that.  From few paths on it is the walk of a lone wavefront, 0.9 to 2 us a tile.
// Before (prefix-tree kernels, sig_backward_d16.hip, sig_wide_backward.hip) | now, us: 256 paths of 1024 points, d = 16, N = 4 1268 | 748; 256 x 101,
// d = 6, N = 4 53 | 17; 128 x 128, d = 4, N = 5 52 | 16; 64 x 201, d = 8, N = 5 156 | 46; 32 x 128, d = 16, N = 4 163 | 27; 1 x 1001, d = 13, N = 4 986 | 126
// (calls queued one behind another, with the sums that end them).  The error is 0.94 of theirs over 190 drawn shapes, at most 1.37 (few short paths: 3 of 34
// points, d = 6, N = 7 5.2e-7 | 7.1e-7; 3 x 27, d = 4, N = 7 5.7e-7 | 6.9e-7).
//
// The signature handed in carries the rounding of the scan that made it; walked back by other sums it does not end at zero, and the
// first points' gradients are off by what is left.  From depth 5 on the levels up to N - 2 are therefore formed anew ahead of the walk, by the
// same sums (a tenth of the time; 8 paths of 128 points, d = 4, N = 8: off by 3.2e-6 without, 1.35e-6 with, 1.62e-6 on the prefix-tree kernels).
// Where the caller says that sig_forward made the signature (Shape::scanned), and it did so in sig_tile_forward_impl.h, these are the sums it was made by, and
// nothing is gained by forming them again: the gradients are the same bits (32 x 128 points, d = N = 7: 489 us with, 427 without; 100 x 901, d = 9, N = 5 1373 | 1193).
#ifndef SIG_TILE_BACKWARD_IMPL_H_
#define SIG_TILE_BACKWARD_IMPL_H_

#include "sig_internal.h"
#include "sig_tile_common.h"

namespace sig {
namespace {

constexpr int kTlMaxWaves = 4;      // wavefronts of a workgroup
constexpr int kTlForwardFrom = 5;   // depth from which on the signature below the words is formed anew before the walk

template <int D, int N>
struct TileShape {
    static constexpr int M = N - 2;                                  // letters of a word
    static constexpr int LW = D <= 4 ? 4 : D <= 8 ? 8 : 16;          // last letters a block has room for
    static constexpr int kPrefixes = int(tl_pow(D, M - 1));
    static constexpr int kPerBlock = 16 / LW;                        // prefixes of a block
    static constexpr int kHalves = LW == 16 ? 2 : 1;                 // wavefronts of a block
    static constexpr int HW = (D + kHalves - 1) / kHalves;           // letters w and j of a wavefront,
    static constexpr int HR = LW == 16 ? 8 : LW;                     // and the room for them
    static constexpr int kBlocks = (kPrefixes + kPerBlock - 1) / kPerBlock * kHalves;   // wavefronts of a path
    static constexpr int kGroups = (kBlocks + kTlMaxWaves - 1) / kTlMaxWaves;           // workgroups of a path
    static constexpr int kWaves = (kBlocks + kGroups - 1) / kGroups;                    // wavefronts of a workgroup
    static_assert(LW < 16 || kWaves % 2 == 0);
    static constexpr int kTiles = LW == 16 ? 4 : 8;                  // tiles staged at a time
    static constexpr int kSpan = 16 * kTiles;
    static constexpr int ZR = LW == 4 ? 4 : LW + 4;                  // floats of an increment's row: sixteen rows fall on different banks
    static constexpr int kA = LW == 4 ? 1 : 2;                       // operands of a wavefront's matrix per letter
    static constexpr int kB = LW == 4 ? 1 : LW == 8 ? 2 : 3;         // ... of the increments
    static constexpr int OR = LW == 16 ? HR + 16 : LW;               // floats a wavefront leaves per increment
    // LDS: increments, the signature's level 1 before them, operands, g_{N-1}, what the wavefronts leave
    static constexpr int kAtPos = kSpan * ZR, kAtOps = 2 * kSpan * ZR, kAtLow = kAtOps + kTiles * 2 * kB * 64 * 4;
    static constexpr int kAtOut = kAtLow + kWaves * HR * 16, kLds = kAtOut + kWaves * kSpan * OR;
    static constexpr int kOccupancy = LW == 4 ? 3 : 2;   // wavefronts per SIMD
    static_assert(kLds * 4 <= 64 * 1024);
};

// One block per wavefront, over the whole path.
template <int D, int N, bool IDENTITY>
__device__ __forceinline__ void tl_walk(const Shape &sh, int groups, int rounds, bool anew, int round, int tid, float *lds, const float *path,
                                        const float *sig, const float *gout, float *partial)
{
    using TS = TileShape<D, N>;
    constexpr int M = TS::M, LW = TS::LW, HW = TS::HW, ZR = TS::ZR, NT = 64 * TS::kWaves;
    constexpr int64_t kS = tl_off(D, N + 1);
    float *zf = lds, *pf = lds + TS::kAtPos;
    TlWords *ops = reinterpret_cast<TlWords *>(lds + TS::kAtOps);   // [tile][increment, rest][operand][lane]
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *low = lds + TS::kAtLow + wave * (TS::HR * 16);           // [w][word]
    float *out = lds + TS::kAtOut;                                  // [wavefront][increment][OR]
    float *qf = out;                                                // [increment][LW], until the operands are made
    const int s = lane & 15, q = lane >> 4;   // the lane's increment of a tile and its words 4q .. 4q + 3 of the block
    const int64_t row = blockIdx.x / unsigned(groups);
    const int group = int(blockIdx.x - unsigned(row) * unsigned(groups));

    const float *x = path + row * sh.L * D;
    const float *sg = sig + row * kS, *go = gout + row * kS;
    const float *bpv = static_cast<const float *>(sh.basepoint_value);

    // the thread's channel of the points it stages, and the points its increments are measured from
    const int my_c = tid % LW, my_cc = my_c < D ? my_c : 0;
    const float my_end = x[(sh.L - 1) * D + my_cc];
    const float my_base = !sh.basepoint ? x[my_cc] : bpv != nullptr ? bpv[row * D + my_cc] : 0.f;
    const float my_level1 = IDENTITY ? 0.f : sg[my_cc];
    const auto stage_points = [&](int64_t t0, int nt) {
        // ---- increments, the signature's level 1 before them and what follows them; zero past the end of the path
#pragma unroll
        for (int k = 0; k < TS::kSpan * LW / NT + (TS::kSpan * LW % NT != 0); ++k) {
            const int i = tid / LW + NT / LW * k;
            if (TS::kSpan * LW % NT != 0 && i >= TS::kSpan) break;
            const bool on = my_c < D && i < nt;
            const int64_t i_hi = (on ? t0 + i : 0) + (sh.basepoint ? 0 : 1);
            const float *at = x + i_hi * D + my_cc;
            const float hi = at[0], lo = i_hi > 0 ? at[-D] : my_base;
            zf[i * ZR + my_c] = on ? hi - lo : 0.f;
            pf[i * ZR + my_c] = !on ? 0.f : IDENTITY ? lo - my_base : my_level1 - (my_end - lo);
            qf[i * LW + my_c] = on ? my_end - hi : 0.f;
        }
    };
    const auto stage = [&](int64_t t0, int nt) {
        stage_points(t0, nt);
        __syncthreads();
        // ---- the right operands: lane (increment, quarter) of a tile
        for (int e = tid; e < TS::kTiles * 64; e += NT) {
            const int tile = e >> 6, ln = e & 63, i = tile * 16 + (ln & 15), c = ln >> 4;
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const float *src = v == 0 ? zf + i * ZR : qf + i * LW;
                TlWords *o = ops + (tile * 2 + v) * TS::kB * 64 + ln;
                TlWords y, y2, y3;
#pragma unroll
                for (int k = 0; k < (LW == 4 ? 2 : 4); ++k) {   // two letters at a time
                    const float *at = src + (LW == 16 ? 8 * (c & 1) : 0) + 2 * k;
                    const TlPieces p = LW == 16 ? tl_split_pair_nearest(at[0], at[1]) : tl_split_pair(at[0], at[1]);
                    if constexpr (LW == 4) {   // [h m] [l h] [m l] [h m]
                        y[k] = c == 1 ? p.l : c == 2 ? p.m : p.h;
                        y[2 + k] = c == 1 ? p.h : c == 2 ? p.l : p.m;
                    } else if constexpr (LW == 8) {   // l h l m, h m h m
                        y[k] = c == 1 ? p.h : c == 3 ? p.m : p.l;
                        y2[k] = (c & 1) ? p.m : p.h;
                    } else {   // h h l l, m m m m, h h h h
                        y[k] = c < 2 ? p.h : p.l;
                        y2[k] = p.m;
                        y3[k] = p.h;
                    }
                }
                o[0] = y;
                if constexpr (LW >= 8) o[64] = y2;
                if constexpr (LW == 16) o[128] = y3;
            }
        }
        __syncthreads();
    };

    const int64_t last_span = (sh.n_inc - 1) / TS::kSpan * TS::kSpan;
    float rf[N + 1];
#pragma unroll
    for (int k = 0; k <= N; ++k) rf[k] = tl_inv_factorial(k);

    constexpr int kMine = LW == 4 ? 1 : 2;   // channels the lane ends up with (see the end of a tile)
    const int block = (group * rounds + round) * TS::kWaves + wave;
    const int half = block % TS::kHalves, prefix0 = block / TS::kHalves * TS::kPerBlock;
    const int w0 = half * HW;   // the wavefront's first letter w and j
    // ---- the lane's prefix and words
    const int my_prefix_raw = prefix0 + (4 * q) / LW, letter0 = (4 * q) % LW;
    const bool there = my_prefix_raw < TS::kPrefixes;
    const int my_prefix = there ? my_prefix_raw : 0;
    int cl[M];        // letters of the prefix, 1 .. M - 1
    float ca[M];      // the signature at its prefixes of 2 .. letters, at the end of the current tile
    float cg[M];      // this lane's part of their cotangents (a prefix's own belongs to the first words below it)
    float cam[4], cG[4];
    {
        int rest = my_prefix;
        bool is_first = there && half == 0 && letter0 == 0;
#pragma unroll
        for (int j = M - 1; j >= 1; --j) {
            cl[j] = rest % D;
            ca[j] = j >= 2 ? sg[tl_off(D, j) + rest] : 0.f;
            cg[j] = is_first ? go[tl_off(D, j) + rest] : 0.f;
            is_first = is_first && cl[j] == 0;
            rest /= D;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool on = there && letter0 + i < D;
            const int64_t at = tl_off(D, M) + (on ? int64_t(my_prefix) * D + letter0 + i : 0);
            cam[i] = on ? sg[at] : 0.f;
            cG[i] = on && half == 0 ? go[at] : 0.f;
        }
    }

    // ---- the wavefront's matrices, in the layout of a left operand: a lane holds word lane % 16, and of its D x D numbers those
    // of its quarter of the 32 products an instruction adds up (the pieces of the increments that they meet: see stage)
    constexpr int kLow = (HW * 16 + 63) / 64;
    float low_v[kLow];   // g_{N-1}[p w]
#pragma unroll
    for (int i = 0; i < kLow; ++i) {
        const int e = lane + 64 * i, w = e / 16, r = e % 16, pre = prefix0 + r / LW, let = r % LW;
        const bool on = w < HW && w0 + w < D && pre < TS::kPrefixes && let < D;
        low_v[i] = on ? go[tl_off(D, N - 1) + (int64_t(pre) * D + let) * D + w0 + w] : 0.f;
    }
    TlWords AD[HW][TS::kA], AH[HW][TS::kA];   // g_N[p w .] for every w, g_N[p . j] for every j
    float at_end[TS::HR];                     // sum over p, w of g_N[p w j] A_{N-1}[p w] at the end of the path
#pragma unroll
    for (int j = 0; j < TS::HR; ++j) at_end[j] = 0.f;
    {
        const int r = lane & 15, c = lane >> 4, prefix = prefix0 + r / LW, letter = r % LW;
        const bool ok = prefix < TS::kPrefixes && letter < D;
        const int64_t p = ok ? int64_t(prefix) * D + letter : 0;
        const float *a = sg + tl_off(D, N - 1) + p * D;
        if constexpr (LW <= 8) {
            float a_v[LW];
#pragma unroll
            for (int w = 0; w < LW; ++w) a_v[w] = ok && c == 0 && w < D ? a[w < D ? w : 0] : 0.f;
            // the block's words follow one another in g_N: through LDS (the operands' place), so that a row of the block is not a cache line
            // per lane
            constexpr int kBlock = TS::kPerBlock * D * D * D, kRow = D * D % 2 == 0 ? D * D + 1 : D * D;
            static_assert(TS::kWaves * TS::kPerBlock * D * kRow <= TS::kAtLow - TS::kAtOps);
            float *mine = lds + TS::kAtOps + wave * (TS::kPerBlock * D * kRow);
            const int64_t from = int64_t(prefix0) * (D * D * D), left = (int64_t(TS::kPrefixes) - prefix0) * (D * D * D);
            float v[(kBlock + 63) / 64];
#pragma unroll
            for (int i = 0; i < (kBlock + 63) / 64; ++i) {
                const int e = lane + 64 * i;
                v[i] = e < left && e < kBlock ? go[tl_off(D, N) + from + e] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < (kBlock + 63) / 64; ++i) {
                const int e = lane + 64 * i;
                if (e < kBlock) mine[e / (D * D) * kRow + e % (D * D)] = v[i];
            }
            tl_wave_order();
            const float *g = mine + (ok ? ((lane & 15) / LW * D + letter) * kRow : 0);
            // pieces by quarter: 4 letters [h h] [h m] [m m] [l l]; 8 letters, small products first: h l m l, then h h m m
            unsigned first[2][LW / 2];
#pragma unroll
            for (int w = 0; w < LW; ++w) {
                unsigned one[LW / 2], two[LW / 2];   // letters j and j + 1 in a word
                const float aw = a_v[w];
#pragma unroll
                for (int j = 0; j < LW; j += 2) {
                    float v[2];
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        v[k] = ok && w < D && j + k < D ? g[w < D && j + k < D ? w * D + j + k : 0] : 0.f;
                        if (j + k < D) at_end[j + k] = __builtin_fmaf(v[k], aw, at_end[j + k]);
                    }
                    const TlPieces e = tl_split_pair(v[0], v[1]);
                    if constexpr (LW == 4) {
                        one[j / 2] = c < 2 ? e.h : c == 2 ? e.m : e.l;
                        two[j / 2] = c == 0 ? e.h : c < 3 ? e.m : e.l;
                    } else {
                        one[j / 2] = c == 0 ? e.h : c == 2 ? e.m : e.l;
                        two[j / 2] = c < 2 ? e.h : e.m;
                    }
                }
                if constexpr (LW == 4) {
                    if (w < D) AD[w < D ? w : 0][0] = TlWords{one[0], one[1], two[0], two[1]};
                } else if (w < D) {
                    AD[w < D ? w : 0][0] = TlWords{one[0], one[1], one[2], one[3]};
                    AD[w < D ? w : 0][TS::kA - 1] = TlWords{two[0], two[1], two[2], two[3]};
                }
                if (w % 2 == 0) {
#pragma unroll
                    for (int j = 0; j < LW / 2; ++j) {
                        first[0][j] = one[j];
                        first[1][j] = two[j];
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        const unsigned u = j % 2 == 0 ? tl_pack_lower(first[0][j / 2], one[j / 2]) : tl_pack(first[0][j / 2], one[j / 2]);
                        const unsigned v = j % 2 == 0 ? tl_pack_lower(first[1][j / 2], two[j / 2]) : tl_pack(first[1][j / 2], two[j / 2]);
                        if constexpr (LW == 4) {
                            AH[j][0][w / 2] = u;
                            AH[j][0][2 + w / 2] = v;
                        } else {
                            AH[j][0][w / 2] = u;
                            AH[j][TS::kA - 1][w / 2] = v;
                        }
                    }
                }
            }
        } else {
            // The same with the two wavefronts of a block side by side, in the place of the increments and the operands (256 paths, d = 16,
            // N = 4: 16 increments took 128 us with every lane reading its own rows and columns from memory).
            constexpr int kBlock = D * D * D, kRow = D * D | 1, kEach = (kBlock + 127) / 128;
            static_assert(TS::kWaves / 2 * D * kRow <= TS::kAtLow);
            float *mine = lds + wave / 2 * (D * kRow);
            const bool is_block = prefix0 < TS::kPrefixes;
            const float *from = go + tl_off(D, N) + int64_t(is_block ? prefix0 : 0) * kBlock;
            const int at = (wave & 1) * 64 + lane;
            float v[kEach];
#pragma unroll
            for (int i = 0; i < kEach; ++i) v[i] = is_block && at + 128 * i < kBlock ? from[at + 128 * i] : 0.f;
#pragma unroll
            for (int i = 0; i < kEach; ++i) {
                const int e = at + 128 * i;
                if (e < kBlock) mine[e / (D * D) * kRow + e % (D * D)] = v[i];
            }
            __syncthreads();
            const float *g = mine + (ok ? letter * kRow : 0);
            // letters 8 (c % 2) .. + 7; pieces by quarter: l l h h, then h h m m (met twice, by the middle and by the high pieces)
            const int k0 = 8 * (c & 1);
            const bool upper = c >= 2;
            float a8[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) a8[e] = ok && !upper && k0 + e < D ? a[k0 + e < D ? k0 + e : 0] : 0.f;
#pragma unroll
            for (int w = 0; w < HW; ++w) {
                const bool wok = ok && w0 + w < D;
#pragma unroll
                for (int e = 0; e < 4; ++e) {   // two letters at a time
                    float v[2], h[2];
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const int i = k0 + 2 * e + k;
                        const bool on = wok && i < D;
                        v[k] = on ? g[on ? (w0 + w) * D + i : 0] : 0.f;
                        h[k] = on ? g[on ? i * D + w0 + w : 0] : 0.f;
                        at_end[w] = __builtin_fmaf(h[k], a8[2 * e + k], at_end[w]);
                    }
                    const TlPieces pv = tl_split_pair(v[0], v[1]), ph = tl_split_pair(h[0], h[1]);
                    AD[w][0][e] = upper ? pv.h : pv.l;
                    AD[w][TS::kA - 1][e] = upper ? pv.m : pv.h;
                    AH[w][0][e] = upper ? ph.h : ph.l;
                    AH[w][TS::kA - 1][e] = upper ? ph.m : ph.h;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kLow; ++i)
            if (lane + 64 * i < HW * 16) low[lane + 64 * i] = low_v[i];
    }
#pragma unroll
    for (int j = 0; j < HW; ++j) at_end[j] = group_sum<0, 6, float>(at_end[j]);
    // the lane's channels of what the wavefront leaves (see the end of a tile)
    float cK[kMine];
    if constexpr (LW == 4) {
        const float even = q < 2 ? at_end[0] : at_end[1], odd = q < 2 ? at_end[2] : at_end[3];
        cK[0] = (q & 1) ? odd : even;
    } else {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float even = q < 2 ? at_end[2 * k] : at_end[2 * k + 1], odd = q < 2 ? at_end[4 + 2 * k] : at_end[5 + 2 * k];
            cK[k] = (q & 1) ? odd : even;
        }
    }

    if (IDENTITY && N >= kTlForwardFrom && anew) {
        // The prefixes' and words' signatures once more from the start of the path: walked back they then end where they began, at zero.
#pragma unroll
        for (int j = 2; j < M; ++j) ca[j] = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) cam[i] = 0.f;
        for (int64_t t0 = 0; t0 < sh.n_inc; t0 += TS::kSpan) {
            const int nt = int(sh.n_inc - t0 < TS::kSpan ? sh.n_inc - t0 : TS::kSpan);
            __syncthreads();
            stage_points(t0, nt);
            __syncthreads();
            for (int tile = 0; tile <= (nt - 1) >> 4; ++tile) {
                const float *zrow = zf + (tile * 16 + s) * ZR;
                const float a1 = pf[(tile * 16 + s) * ZR + cl[1]];
                const f4 zc = *reinterpret_cast<const f4 *>(zrow + letter0);
                float Hh[M][M + 1];
                const float z1 = zrow[cl[1]];
#pragma unroll
                for (int k = 2; k <= M; ++k) Hh[1][k] = __builtin_fmaf(z1, rf[k], a1 * rf[k - 1]);
#pragma unroll
                for (int j = 2; j < M; ++j) {
                    const float z = zrow[cl[j]], sum = tl_prefix(Hh[j - 1][j] * z), a = ca[j] + tl_down<1>(sum);
                    ca[j] += tl_last(sum);
#pragma unroll
                    for (int k = j + 1; k <= M; ++k) Hh[j][k] = __builtin_fmaf(Hh[j - 1][k], z, k == j + 1 ? a : a * rf[k - j]);
                }
                float sv[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) sv[i] = Hh[M - 1][M] * zc[i];
                tl_prefixes(sv);
#pragma unroll
                for (int i = 0; i < 4; ++i) cam[i] += tl_last(sv[i]);
            }
        }
    }

    for (int64_t t0 = last_span; t0 >= 0; t0 -= TS::kSpan) {
        const int nt = int(sh.n_inc - t0 < TS::kSpan ? sh.n_inc - t0 : TS::kSpan);
        __syncthreads();   // everyone has its block (the previous span's sums are closed)
        stage(t0, nt);
        for (int tile = (nt - 1) >> 4; tile >= 0; --tile) {
            const float *zrow = zf + (tile * 16 + s) * ZR;
            float zl[M];
#pragma unroll
            for (int j = 1; j < M; ++j) zl[j] = zrow[cl[j]];
            const float a1 = pf[(tile * 16 + s) * ZR + cl[1]];
            const f4 zc = *reinterpret_cast<const f4 *>(zrow + letter0);
            TlWords Bz[TS::kB], Bq[TS::kB];
#pragma unroll
            for (int o = 0; o < TS::kB; ++o) {
                Bz[o] = ops[((tile * 2) * TS::kB + o) * 64 + lane];
                Bq[o] = ops[((tile * 2 + 1) * TS::kB + o) * 64 + lane];
            }
            float zw[TS::HR];
#pragma unroll
            for (int w = 0; w < TS::HR; w += 4) {
                if constexpr (LW < 16) {
                    const f4 v = *reinterpret_cast<const f4 *>(zrow + w);
#pragma unroll
                    for (int k = 0; k < 4; ++k) zw[w + k] = v[k];
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) zw[w + k] = zrow[w0 + w + k];   // within the row's 20 floats: w0 + 7 <= 15
                }
            }

            // ---- the signature before every increment and the Horner terms, Hh[j][k] = T^(k)_j / (k-j)!
            float Hh[M][N + 1];
#pragma unroll
            for (int k = 2; k <= N; ++k) Hh[1][k] = __builtin_fmaf(zl[1], rf[k], a1 * rf[k - 1]);
#pragma unroll
            for (int j = 2; j < M; ++j) {
                const float a = ca[j] - tl_suffix(Hh[j - 1][j] * zl[j]);
                ca[j] = tl_first(a);
#pragma unroll
                for (int k = j + 1; k <= N; ++k) Hh[j][k] = __builtin_fmaf(Hh[j - 1][k], zl[j], k == j + 1 ? a : a * rf[k - j]);
            }
            float U[4], V[4], sv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) sv[i] = Hh[M - 1][M] * zc[i];
            tl_suffixes(sv);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float a = cam[i] - sv[i];
                cam[i] = tl_first(a);
                U[i] = __builtin_fmaf(Hh[M - 1][N - 1], zc[i], a);
                V[i] = __builtin_fmaf(Hh[M - 1][N], zc[i], a * 0.5f);
            }

            // ---- the top two levels
            float e1[4] = {}, e2[4] = {}, gz[TS::HR] = {}, K[TS::HR] = {};
#pragma unroll
            for (int w = 0; w < HW; ++w) {
                f4 d = {0.f, 0.f, 0.f, 0.f}, h = {0.f, 0.f, 0.f, 0.f};
                f4 d2 = *reinterpret_cast<const f4 *>(low + w * 16 + 4 * q);
#pragma unroll
                for (int o = 0; o < TS::kB; ++o) {
                    const int oa = o < TS::kA ? o : TS::kA - 1;
                    d = tl_mfma(AD[w][oa], Bz[o], d);
                    d2 = tl_mfma(AD[w][oa], Bq[o], d2);
                    h = tl_mfma(AH[w][oa], Bz[o], h);
                }
                float g0 = 0.f, k0 = 0.f;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    e1[i] = __builtin_fmaf(d[i], zw[w], e1[i]);
                    e2[i] = __builtin_fmaf(d2[i], zw[w], e2[i]);
                    g0 = __builtin_fmaf(d[i], V[i], g0);
                    g0 = __builtin_fmaf(d2[i], U[i], g0);
                    g0 = __builtin_fmaf(h[i], V[i], g0);
                    k0 = __builtin_fmaf(h[i], U[i], k0);
                }
                gz[w] = g0;
                K[w] = k0;
            }

            // ---- down the word: cotangents of the Horner terms, of the signature after every increment, and the letters' channels
            float cc[4];   // to the channels of the words' last letters
            float Dc[N + 1];
            Dc[N] = Dc[N - 1] = Dc[M] = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) sv[i] = __builtin_fmaf(e1[i], 0.5f, e2[i]);
            tl_suffixes(sv);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float S = sv[i];
                const float G = cG[i] + tl_up<1>(S);
                cG[i] += tl_first(S);
                cc[i] = __builtin_fmaf(Hh[M - 1][N], e1[i], __builtin_fmaf(Hh[M - 1][N - 1], e2[i], Hh[M - 1][M] * G));
                Dc[N] = __builtin_fmaf(e1[i], zc[i], Dc[N]);
                Dc[N - 1] = __builtin_fmaf(e2[i], zc[i], Dc[N - 1]);
                Dc[M] = __builtin_fmaf(G, zc[i], Dc[M]);
            }
            float contrib[M];
#pragma unroll
            for (int j = M - 1; j >= 1; --j) {
                float add = Dc[j + 1];
#pragma unroll
                for (int k = j + 2; k <= N; ++k) add = __builtin_fmaf(Dc[k], rf[k - j], add);
                const float S = tl_suffix(add);
                const float G = cg[j] + tl_up<1>(S);
                cg[j] += tl_first(S);
                contrib[j] = j >= 2 ? Hh[j >= 2 ? j - 1 : 1][j] * G : G;
#pragma unroll
                for (int k = j + 1; k <= N; ++k) contrib[j] = __builtin_fmaf(j >= 2 ? Hh[j >= 2 ? j - 1 : 1][k] : rf[k], Dc[k], contrib[j]);
                if (j >= 2) {
#pragma unroll
                    for (int k = N; k >= j + 1; --k) Dc[k] *= zl[j];
                    Dc[j] = G * zl[j];
                }
            }

            // ---- the wavefront's sums: a lane ends up with one or two channels of its increment
            float *o = out + (wave * TS::kSpan + tile * 16 + s) * TS::OR;
            if constexpr (LW == 4) {   // channel 2 (q % 2) + q / 2
#pragma unroll
                for (int i = 0; i < 4; ++i) gz[i] += cc[i];
#pragma unroll
                for (int j = 1; j < M; ++j)
#pragma unroll
                    for (int c = 0; c < D; ++c) gz[c] += cl[j] == c ? contrib[j] : 0.f;
                const float g = tl_rows_32(tl_rows_16(gz[0], gz[2]), tl_rows_16(gz[1], gz[3]));
                const float k = tl_suffix(tl_rows_32(tl_rows_16(K[0], K[2]), tl_rows_16(K[1], K[3])));
                o[2 * (q & 1) + (q >> 1)] = g + (cK[0] - k);
                cK[0] -= tl_first(k);
            } else {
                if constexpr (LW == 8) {   // a prefix's two rows of lanes: letter j in the first, j + 1 in the second
#pragma unroll
                    for (int j = 1; j < M; j += 2) {
                        const float v = tl_rows_16(contrib[j], j + 1 < M ? contrib[j + 1 < M ? j + 1 : j] : 0.f);
                        const int letter = (q & 1) ? (j + 1 < M ? cl[j + 1 < M ? j + 1 : j] : -1) : cl[j];
#pragma unroll
                        for (int c = 0; c < D; ++c) gz[c] += letter == c ? v : 0.f;
                    }
                }
                float g[4], k[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    g[i] = tl_rows_16(gz[i], gz[4 + i]);
                    k[i] = tl_rows_16(K[i], K[4 + i]);
                    if constexpr (LW == 8) g[i] += cc[i];
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {   // channels 4 (q % 2) + 2 i + q / 2 of the wavefront's
                    const float v = tl_rows_32(g[2 * i], g[2 * i + 1]);
                    const float S = tl_suffix(tl_rows_32(k[2 * i], k[2 * i + 1]));
                    o[4 * (q & 1) + 2 * i + (q >> 1)] = v + (cK[i] - S);
                    cK[i] -= tl_first(S);
                }
                if constexpr (LW == 16) {   // the letters of the words: channels 4 q .. 4 q + 3
#pragma unroll
                    for (int j = 1; j < M; ++j) {
                        float v = tl_rows_16(contrib[j], contrib[j]);
                        v = tl_rows_32(v, v);
#pragma unroll
                        for (int i = 0; i < 4; ++i) cc[i] += cl[j] == 4 * q + i ? v : 0.f;
                    }
                    *reinterpret_cast<f4 *>(o + TS::HR + 4 * q) = f4{cc[0], cc[1], cc[2], cc[3]};
                }
            }
        }
        __syncthreads();
        for (int e = tid; e < nt * D; e += NT) {
            const int i = e / D, c = e % D;
            float sum = 0.f;
#pragma unroll
            for (int w = 0; w < TS::kWaves; ++w) {
                const float *o = out + (w * TS::kSpan + i) * TS::OR;
                if constexpr (LW < 16) {
                    sum += o[c];
                } else {   // kWaves is even: a wavefront's half of the letters is that of its number
                    const int mine = c - w % 2 * HW;
                    sum += o[TS::HR + c];
                    if (mine >= 0 && mine < HW) sum += o[mine];
                }
            }
            float *to = partial + ((row * groups + group) * sh.n_inc + t0 + i) * D + c;
            *to = round > 0 ? *to + sum : sum;
        }
        __syncthreads();   // the next increments' rests take the place of these sums
    }
}

template <int D, int N, bool IDENTITY>
__global__ void __launch_bounds__((64 * TileShape<D, N>::kWaves), (TileShape<D, N>::kOccupancy))
sig_tile_backward_kernel(Shape sh, int groups, int rounds, bool anew, const float *__restrict__ path, const float *__restrict__ sig,
                         const float *__restrict__ gout, float *__restrict__ partial)
{
    __shared__ __align__(16) float lds[TileShape<D, N>::kLds];
    for (int round = 0; round < rounds; ++round) {
        // Nothing is carried from one round to the next: places worked out ahead of them would take registers the walk has not (d = 8, N = 5:
        // 117 moved to memory and back, 1.6 times the time).
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        tl_walk<D, N, IDENTITY>(sh, groups, rounds, anew, round, tid, lds, path, sig, gout, partial);
    }
}

// Workgroups of a path, each of which takes `rounds` times its wavefronts' number of blocks: as few as leave about four times what the
// chip holds at a time, so that few partial gradients are left to be added up (32 paths, d = N = 7: 61 a path instead of 301), and no more than
// one round in twenty without blocks.
template <int D, int N>
int tile_groups_dn(int64_t B, int &rounds)
{
    constexpr int kGroups = TileShape<D, N>::kGroups;
    const int64_t most = kGroups < 8 ? kGroups : 8, want = (B * kGroups + 2047) / 2048;
    for (rounds = int(want < 1 ? 1 : want < most ? want : most);; --rounds) {
        const int groups = (kGroups + rounds - 1) / rounds;
        if (20 * kGroups >= 19 * groups * rounds) return groups;   // one round: always
    }
}

template <int D, int N>
hipError_t launch_tile_backward_dn(const Shape &sh, const float *path, const float *sig, const float *gout, float *gpath, float *gbase,
                                   float *partial, hipStream_t st)
{
    using TS = TileShape<D, N>;
    int rounds;
    const int groups = tile_groups_dn<D, N>(sh.B, rounds);
    if (!grid_holds(sh.B * groups, 64 * TS::kWaves)) return hipErrorNotSupported;
    const dim3 grid(unsigned(sh.B * groups)), threads(64 * TS::kWaves);
    const bool anew = !sh.scanned || !tile_forward_certain(sh);
    if (sh.from_identity) {
        hipLaunchKernelGGL((sig_tile_backward_kernel<D, N, true>), grid, threads, 0, st, sh, groups, rounds, anew, path, sig, gout, partial);
    } else {   // stretches: up to eight channels they have kernels of their own (tree_stretches_supported)
        if constexpr (D > 8)
            hipLaunchKernelGGL((sig_tile_backward_kernel<D, N, false>), grid, threads, 0, st, sh, groups, rounds, anew, path, sig, gout, partial);
        else
            return hipErrorNotSupported;
    }
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    return launch_increment_sums<float>(sh, groups, partial, gpath, gbase, st);
}

}  // namespace

// One channel count, depths 4 to 8 (to 6 from 9 channels on).
template <int D>
hipError_t launch_tile_backward_d(const Shape &sh, const float *path, const float *sig, const float *gout, float *gpath, float *gbase,
                                  float *partial, hipStream_t st)
{
    switch (sh.N) {
        case 4: return launch_tile_backward_dn<D, 4>(sh, path, sig, gout, gpath, gbase, partial, st);
        case 5: return launch_tile_backward_dn<D, 5>(sh, path, sig, gout, gpath, gbase, partial, st);
        case 6: return launch_tile_backward_dn<D, 6>(sh, path, sig, gout, gpath, gbase, partial, st);
    }
    if constexpr (D <= 8) {
        switch (sh.N) {
            case 7: return launch_tile_backward_dn<D, 7>(sh, path, sig, gout, gpath, gbase, partial, st);
            case 8: return launch_tile_backward_dn<D, 8>(sh, path, sig, gout, gpath, gbase, partial, st);
        }
    }
    return hipErrorNotSupported;
}

template <int D>
int tile_groups_d(int64_t B, int N, int &rounds)   // workgroups of a path, 0 where there is no kernel
{
    switch (N) {
        case 4: return tile_groups_dn<D, 4>(B, rounds);
        case 5: return tile_groups_dn<D, 5>(B, rounds);
        case 6: return tile_groups_dn<D, 6>(B, rounds);
    }
    if constexpr (D <= 8) {
        switch (N) {
            case 7: return tile_groups_dn<D, 7>(B, rounds);
            case 8: return tile_groups_dn<D, 8>(B, rounds);
        }
    }
    return 0;
}

}  // namespace sig

#endif  // SIG_TILE_BACKWARD_IMPL_H_
