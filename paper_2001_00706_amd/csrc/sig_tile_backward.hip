// Which calls the tile gradient kernels serve (see sig_tile_backward_impl.h; instantiated per channel count in the files beside this one).
#include "sig_internal.h"

#include <cmath>
#include <type_traits>

namespace sig {

template <int D>
hipError_t launch_tile_backward_d(const Shape &sh, const float *path, const float *sig, const float *gout, float *gpath, float *gbase,
                                  float *partial, hipStream_t st);
template <int D>
int tile_groups_d(int64_t B, int N, int &rounds);

namespace {

// f of the channel count as a constant, 3 to 16
template <typename F>
auto with_channels(int d, F f)
{
    switch (d) {
        case 3: return f(std::integral_constant<int, 3>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 5: return f(std::integral_constant<int, 5>{});
        case 6: return f(std::integral_constant<int, 6>{});
        case 7: return f(std::integral_constant<int, 7>{});
        case 8: return f(std::integral_constant<int, 8>{});
        case 9: return f(std::integral_constant<int, 9>{});
        case 10: return f(std::integral_constant<int, 10>{});
        case 11: return f(std::integral_constant<int, 11>{});
        case 12: return f(std::integral_constant<int, 12>{});
        case 13: return f(std::integral_constant<int, 13>{});
        case 14: return f(std::integral_constant<int, 14>{});
        case 15: return f(std::integral_constant<int, 15>{});
        default: return f(std::integral_constant<int, 16>{});
    }
}

int groups(const Shape &sh, int &rounds)
{
    if (sh.d < 3 || sh.d > 16) return 0;
    return with_channels(sh.d, [&](auto d) { return tile_groups_d<decltype(d)::value>(sh.B, sh.N, rounds); });
}
int groups(const Shape &sh)
{
    int rounds;
    return groups(sh, rounds);
}

}  // namespace

// Microseconds of a call, fitted to 650 shapes of 1 to 4000 paths of 17 to 1100 points (off by 4 % in the mean where the chip is full): a
// tile takes a lone wavefront 0.9 to 2.0, and a SIMD that holds two or three of them c; before the first one the matrices are cut into
// pieces, s.  The products grow with the letters of a wavefront, the chains with the depth.
double tile_backward_us(const Shape &sh)
{
    const double tiles = double((sh.n_inc + 15) / 16);
    const double prefixes = double(sh.pw[sh.N - 3]), per_block = sh.d <= 4 ? 4 : sh.d <= 8 ? 2 : 0.5;   // of a wavefront
    const double waves = double(sh.B) * std::ceil(prefixes / per_block) / 1024;
    const double alone = sh.d <= 4 ? (sh.N >= 5 ? 1.15 : 1.0) : sh.d <= 8 ? (sh.N >= 5 ? 1.75 : 1.55) : (sh.N >= 5 ? 2.3 : 2.0);
    const double s = sh.d <= 4 ? 0.8 : sh.d <= 8 ? 3.0 : 2.4;
    const double c = sh.d <= 4   ? 0.75 + 0.07 * (sh.N - 6)
                     : sh.d <= 8 ? 1.2 + 0.05 * (sh.d - 6.5) + 0.05 * (sh.N - 6)
                                 : 0.48 + 0.153 * ((sh.d + 1) / 2) + 0.16 * (sh.N - 4);
    // from depth 5 on a path is gone through forward first, unless its signature was formed in the same tiles (0.87 to 0.89 of the time)
    const double way = sh.N >= 5 && tile_forward_certain(sh) ? 0.9 : 1.0;
    return 9 + std::cbrt(std::pow(tiles * alone * way, 3.0) + std::pow(waves * (s + tiles * c * way), 3.0));
}

// Where they are used: from 24 increments on (fewer leave most of a tile, or of the time to set it up, unused), and where the prefix-tree
// kernels take longer.  Those wait 0.4 us for an increment as long as the chip is not full; once it is, they take ct for an increment of 64
// words.  At 9 channels and more that is longer from 32 increments on, up to a few channels only while few paths leave the chip idle: a block of sixteen
// words has room for 10 at 5 channels, 12 at 6, and three wavefronts in four would multiply zeros (tile | before, us: 256 x 101 points, d = 6,
// N = 4: 17 | 53; 64 x 201, d = 8, N = 5: 46 | 156; 256 x 1024, d = 16, N = 4: 748 | 1268; 1 x 1001, d = 13, N = 4: 126 | 986; 32 x 128,
// d = N = 7: 427 | 504; against the rule 648 x 80, d = 5, N = 6: 320 | 187).  Over 650 shapes of 3 to 16 channels the rule is 1.3 % off the better one of the
// two, and takes 0.60 of the time without these kernels; of 240 shapes at its line the worst is 1.03 (49 x 123, d = 7, N = 6: 109 | 106; 125 where
// the caller does not say that the signature is the scan's, which stays: the tree's gradient of a signature from tiles is less exact).
bool tile_backward_preferred(const Shape &sh)
{
    if (sh.stream || sh.n_inc < 24 || sh.S >= (int64_t(1) << 31) || (!sh.from_identity && sh.d <= 8)) return false;
    const int workgroups = groups(sh);   // of up to four wavefronts
    if (workgroups == 0 || !grid_holds(sh.B * workgroups, 256)) return false;
    // (d = 16, N = 4 has sig_backward_d16.hip for short paths: 256 x 31 points 60 | 52, 64 x 17 16 | 30)
    if (sh.d == 16 && sh.N == 4) return sh.n_inc >= 48 || sh.B <= 64;
    if (sh.d > 8) return sh.n_inc >= 32 || sh.B * sh.pw[sh.N - 3] <= 512;
    // (from 641 paths of d = 4, N = 6 on a SIMD's fourth set of wavefronts is nearly empty, which the fit does not see: 640 x 80 points 53.8 | 57.1, 680 x 80
    // 61.8 | 56.7, 680 x 400 248 | 266)
    if (sh.d == 4 && sh.N == 6 && sh.B > 640 && sh.B <= 768 && sh.n_inc < 200) return false;
    // at d = 4, N = 6 many paths have a kernel of their own, sig_backward_d4n6.hip
    const double ct = sh.d <= 4 ? (sh.N == 6 && sh.d == 4 && sh.B > 768 ? 0.19 : 0.27)
                                : sh.d == 5 ? 0.33 : sh.d == 6 ? 0.37 : sh.d == 7 ? 0.47 : 0.44;
    const double n = double(sh.n_inc), tree = std::fmax(0.4 * n, double(sh.B) * double(sh.pw[sh.N - 2]) / 65536 * n * ct);
    return tile_backward_us(sh) - 9 <= tree;
}

int tile_backward_rounds(const Shape &sh)
{
    int rounds = 0;
    groups(sh, rounds);
    return rounds;
}

int64_t tile_backward_workspace_bytes(const Shape &sh)
{
    return sh.B * groups(sh) * sh.n_inc * sh.d * int64_t(sizeof(float));
}

hipError_t launch_tile_backward_f32(const Shape &sh, const float *path, const float *sig, const float *gout, float *gpath, float *gbase,
                                    void *workspace, int64_t workspace_bytes, hipStream_t st)
{
    if (workspace == nullptr || workspace_bytes < tile_backward_workspace_bytes(sh)) return hipErrorInvalidValue;
    float *partial = static_cast<float *>(workspace);
    return with_channels(sh.d, [&](auto d) {
        return launch_tile_backward_d<decltype(d)::value>(sh, path, sig, gout, gpath, gbase, partial, st);
    });
}

}  // namespace sig
