// Which calls the tile kernels serve in final mode (see sig_tile_forward_impl.h; instantiated per channel count in the files beside this one).
#include "sig_internal.h"

namespace sig {

template <int D>
hipError_t launch_tile_forward_d(const Shape &sh, const float *path, float *out, hipStream_t st);

// Where they are faster than the prefix-tree scan and no less exact, both timed over 530 shapes of d = 5..16 (us, tree | tiles):
//  - with few wavefronts the tree needs 0.14 to 0.3 us an increment, a tile 1.2 to 3 us: d = 7 N = 5, 49 paths of 927 increments 224 | 101;
//    d = 5 N = 7, 6 of 466 106 | 40; d = 9 N = 6, 18 of 219 232 | 130.
//  - depth 4 up to 7 channels and depth 5 up to 6 leave a tile too little to multiply for what it costs to form it:
//    d = 6 N = 5, 2010 paths of 186 150 | 224; d = 7 N = 4, 2399 of 73 31 | 42.
//  - the last tile is nearly empty and the rests q of the first increments weigh more where paths are short: under 32 increments the error reaches
//    1.2 times the tree's, d = 8..16 N = 4 under 96 as well, and the time 1.3 times.
//  - a full chip on 5 or 6 channels is bound by the words' Horner terms: under 64 increments d = 5 N = 6 946 paths of 30 46 | 50, and
//    from 32768 wavefronts d = 5 N = 7 366 paths of 68 156 | 176.
//  - from 12 channels on, paths with fewer than 1024 wavefronts altogether wait for each tile's operands: d = 15 N = 4, 3 of 1037 161 | 188,
//    but 84 paths of 690 on 14 channels 207 | 132.
static bool tile_forward_sizes(const Shape &sh)
{
    if (sh.stream || sh.chunks != 1 || sh.d < 5 || sh.d > 16 || sh.N > (sh.d <= 8 ? 8 : 6) || sh.S >= (int64_t(1) << 31)) return false;
    if (sh.N < (sh.d <= 6 ? 6 : sh.d == 7 ? 5 : 4) || sh.n_inc < (sh.N == 4 ? 96 : 32)) return false;
    double waves = double(sh.B);   // four prefixes of N - 3 letters to a wavefront, or one
    for (int k = 0; k < sh.N - 3; ++k) waves *= sh.d;
    if (sh.d <= 8) waves /= 4;
    if (waves >= (1 << 25)) return false;   // at most twice as many with those that round up: a grid has less than 2^32 threads
    if (sh.d <= 6 && waves > 8192 && sh.n_inc < 64) return false;
    if (sh.d == 5 && sh.N == 7 && waves > 32768) return false;
    return sh.d < 12 || waves >= 1024;
}

// Paths that the prefix-tree kernels would cut inside a workgroup stay there: that is faster and up to four times as exact.  And the gradient
// has to be taken in tiles as well.  It walks the signature back to the start of the path, and is as exact as its roundings are those of the way there:
// the prefix tree's gradient from the tiles' signature had 1.2 to 1.5 times the error (d = N = 7, 32 paths of 128 points 2.1e-6 | 1.4e-6), in tiles
// it has 0.6 to 1 of it (1.2e-6).
bool tile_forward_preferred(const Shape &sh)
{
    return tile_forward_sizes(sh) && tree_split_stretches(sh, SIG_F32) == 1 && tile_backward_preferred(sh);
}

// Whether sig_forward forms this call's signature in tiles, for certain: 8 and 16 channels have matrix kernels of their own for some calls, and
// up to 64 paths of 512 increments may be scanned in chunks.
bool tile_forward_certain(const Shape &sh)
{
    return sh.from_identity && tile_forward_sizes(sh) && sh.d != 8 && sh.d != 16 && (sh.B > 64 || sh.n_inc < 512) &&
           tree_split_stretches(sh, SIG_F32) == 1;
}

hipError_t launch_tile_forward_f32(const Shape &sh, const float *path, float *out, hipStream_t st)
{
    switch (sh.d) {
        case 5: return launch_tile_forward_d<5>(sh, path, out, st);
        case 6: return launch_tile_forward_d<6>(sh, path, out, st);
        case 7: return launch_tile_forward_d<7>(sh, path, out, st);
        case 8: return launch_tile_forward_d<8>(sh, path, out, st);
        case 9: return launch_tile_forward_d<9>(sh, path, out, st);
        case 10: return launch_tile_forward_d<10>(sh, path, out, st);
        case 11: return launch_tile_forward_d<11>(sh, path, out, st);
        case 12: return launch_tile_forward_d<12>(sh, path, out, st);
        case 13: return launch_tile_forward_d<13>(sh, path, out, st);
        case 14: return launch_tile_forward_d<14>(sh, path, out, st);
        case 15: return launch_tile_forward_d<15>(sh, path, out, st);
        case 16: return launch_tile_forward_d<16>(sh, path, out, st);
    }
    return hipErrorNotSupported;
}

}  // namespace sig
