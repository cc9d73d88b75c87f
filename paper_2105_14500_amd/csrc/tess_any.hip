// Launches of the any-shape matrix-core kernel (tess_any.h).
#include "tess_any.h"

namespace tess {

// Tile rule, by the number of 64 x 64 tiles of the output (us of one call, MI355X; the scalar
// kernel that this one replaced in brackets):
//                                      32 x 32, K over 4 waves    64 x 64
//   fp32  128 x 512,    K 256    (16)       5.8                     10.7   [17.4]
//   fp32  128 x 128,    K 1024    (4)      11.4                     26.9   [60.9]
//   fp32  515 x 515,    K 1030   (81)      18.4                     28.6
//   fp32  1024 x 2048,  K 2048  (512)      95.3                     88.9   [393]
//   bf16  515 x 333,    K 2042   (54)      10.3                     15.6   [181]
//   bf16  333 x 1021,   K 1030   (96)      14.0                     16.2   [95]
//   bf16  515 x 1021,   K 666   (144)      11.3                      9.6   [107]
//   bf16  2001 x 1999,  K 3002 (1024)     141.6                     75.4
// Below 128 tiles half of the chip would idle and each wavefront would walk the whole contraction;
// above, the smaller tile reads its operands twice as often.
//
// fp32 has 1/16 of the matrix rate: its wavefronts wait at every stage for the LDS, with nothing
// beside them as long as a compute unit holds one workgroup.  Eight wavefronts, two per 32 x 32 part
// that share a stage twice as deep, fill that up to two workgroups per compute unit; beyond, the four
// wavefronts' workgroups overlap by themselves:
//                                      32 x 32    64 x 64, 4 wavefronts    64 x 64, 8 wavefronts
//   fp32  512 x 1024,   K 256   (128)     8.9         13.0                     10.7
//   fp32  515 x 1021,   K 666   (144)    18.6         22.5                     21.1
//   fp32  1024 x 1024,  K 4096  (256)    91.6         92.1                     83.4
//   fp32  512 x 2048,   K 2048  (256)    56.0         59.9                     49.6
//   fp32  1024 x 2048,  K 2048  (512)   103.4         90.7                     85.6
//   fp32  2048 x 2048,  K 512  (1024)    55.5         45.4                     49.3
template <typename T>
static hipError_t launch_any_type(const GemmArgs& g, hipStream_t s)
{
    const int64_t tiles64 = (int64_t)((g.N + 63) / 64) * ((g.M + 63) / 64);
    constexpr bool F32 = sizeof(T) == 4;
    if (tiles64 < (F32 ? 192 : 128)) {
        if constexpr (!F32) {
            // panels shorter than a stage of 128 load element by element; us, stages of 128 / of 64 [scalar]:
            //   11 x 17 x 17 dX  8.3 / 5.4 [5.6]    3775 x 15 x 13 dX  9.1 / 6.9 [7.0]    167 x 51 x 1465 fwd  10.2 / 8.3 [7.9]
            if (g.Kp < 128) return launch_any_tile<T, 32, 32, 64, 1, 1, 4>(g, s);
        }
        return launch_any_tile<T, 32, 32, 256 / sizeof(T), 1, 1, 4>(g, s);
    }
    if constexpr (F32) {
        if (tiles64 <= 512) return launch_any_tile<T, 64, 64, 64, 2, 2, 2>(g, s);
    }
    return launch_any_tile<T, 64, 64, 128 / sizeof(T), 2, 2, 1>(g, s);
}

hipError_t launch_generic(const GemmArgs& g, hipStream_t s)
{
    return g.in_f32 ? launch_any_type<float>(g, s) : launch_any_type<__bf16>(g, s);
}

}  // namespace tess
