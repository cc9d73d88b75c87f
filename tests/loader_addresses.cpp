// Host check of the direct-to-LDS loader's address arithmetic: every request that the first, a middle
// and the last tile of a panel send for its first and last stages, by the same functions as the
// kernels.  A granule that the panel has must be read from where it lies, inside the descriptor's
// range; one past a ragged end must be outside that range; and no offset may pass 2^32 together with
// its immediate (the sum wraps in hardware).  Prints the first violation and exits with 1.
#include "tess_mfma.h"

#include <cstdio>
#include <cstdlib>

using namespace tess;

static long checked = 0;

// rows x ld panel; KC: `extent` rows of Kp contracted elements, MC: Kp rows of `extent` elements
template <int R, bool KC, int NT>
static void check(int64_t extent, int64_t Kp, int64_t ld)
{
    constexpr bool RAGGED = true;
    typedef DmaLoader<R, 64, KC, NT, RAGGED> L;
    const int64_t rows = KC ? extent : Kp, bytes = rows * ld * 2;
    const uint64_t panel = (uint64_t)1 << 40, range = L::PAST;
    const int64_t stages = (Kp + 63) / 64, tiles = (extent + R - 1) / R;
    const int ktail = (int)(Kp - (stages - 1) * 64);
    if (bytes >= DMA_PANEL_LIMIT) { printf("panel of %ld bytes is refused: not a case\n", (long)bytes); exit(1); }
    for (int64_t tile : {(int64_t)0, tiles / 2, tiles - 2, tiles - 1})
        for (int64_t ks : {(int64_t)0, stages / 2, stages - 1}) {
            if (tile < 0) continue;
            const int origin = (int)(tile * R);
            const uint32_t adv = (uint32_t)ks * (KC ? 128u : (uint32_t)(64 * ld * 2));
            const uint64_t base = L::start(panel, origin, ld, adv);
            for (int G = 0; G < R * 8; ++G) {
                const int it = G / 64 % L::ITERS, imm = it % 4 * 1024;      // wavefront w: granules from w * ITERS * 64
                int kpos;
                const uint32_t off = L::offset(it, G, origin, (int)extent, ld, kpos);
                const bool exists = ks + 1 < stages || kpos < ktail;
                const uint32_t past = kpos >= ktail && ks + 1 == stages ? 1u << it : 0u;
                const uint64_t at = (uint64_t)L::sent(it, off, past) + imm;
                // where the LDS format wants this granule from
                int64_t r, k;
                if (KC) {
                    r = origin + G / 8;
                    if (r >= extent) r = extent - 1;
                    k = (G % 8 ^ swz_kc<64>(G / 8)) * 8 + ks * 64;
                } else {
                    r = origin + 8 * (G % (R / 8) ^ swz_mc<R>(G / (R / 8)));
                    if (r + 8 > extent) r = extent - 8;
                    k = G / (R / 8) + ks * 64;
                }
                const int64_t want = (KC ? r * ld + k : k * ld + r) * 2;
                const bool ok = at < ((uint64_t)1 << 32) && exists == (k < Kp) &&
                                (exists ? at + 16 <= range && base + at == panel + want && want >= 0 && want + 16 <= bytes : at >= range);
                if (!ok) {
                    printf("%s R %d extent %ld Kp %ld ld %ld tile %ld stage %ld granule %d: offset %lu, wanted byte %ld of %ld\n",
                           KC ? "KC" : "MC", R, (long)extent, (long)Kp, (long)ld, (long)tile, (long)ks, G, (unsigned long)at,
                           (long)want, (long)bytes);
                    exit(1);
                }
                ++checked;
            }
        }
}

template <bool KC>
static void all_tiles(int64_t extent, int64_t Kp, int64_t ld)
{
    check<32, KC, 256>(extent, Kp, ld);
    check<64, KC, 256>(extent, Kp, ld);
    check<128, KC, 256>(extent, Kp, ld);
    check<256, KC, 256>(extent, Kp, ld);
}

int main()
{
    // below, at and above 2^31 bytes and up to the limit, by the rows and by the leading dimension
    for (int64_t bytes : {(int64_t)1 << 20, ((int64_t)1 << 31) - 3072, ((int64_t)1 << 31) - 2048, (int64_t)1 << 31,
                          ((int64_t)1 << 31) + 4096, (int64_t)3 << 30, DMA_PANEL_LIMIT - 1})
        for (int64_t Kp : {8, 72, 200, 1080, 4088}) {
            all_tiles<true>(bytes / (2 * Kp), Kp, Kp);                       // many short rows
            for (int64_t rows : {1, 8, 40, 250, 264})                        // few long ones
                if (bytes / (2 * rows) / 8 * 8 >= Kp) all_tiles<true>(rows, Kp, bytes / (2 * rows) / 8 * 8);
            if (Kp >= 72) all_tiles<true>(Kp, bytes / (2 * Kp) / 64 * 64 - 56, bytes / (2 * Kp) / 8 * 8);   // long contractions
        }
    for (int64_t bytes : {(int64_t)1 << 20, ((int64_t)1 << 31) - 3072, ((int64_t)1 << 31) - 2048, (int64_t)1 << 31,
                          ((int64_t)1 << 31) + 4096, (int64_t)3 << 30, DMA_PANEL_LIMIT - 1})
        for (int64_t extent : {8, 40, 264, 1024, 4104})
            for (int64_t ld : {extent, extent + 8}) {
                const int64_t Kp = bytes / (2 * ld);
                if (Kp % 64) all_tiles<false>(extent, Kp, ld);
                if (Kp > 65) all_tiles<false>(extent, Kp / 64 * 64 - 1, ld);
                for (int64_t rows : {1, 7, 63, 65, 100})                     // few long rows
                    if (bytes / (2 * rows) / 8 * 8 >= extent) all_tiles<false>(extent, rows, bytes / (2 * rows) / 8 * 8);
                for (int64_t rows : {1, 63, 65})                             // and a wide extent
                    all_tiles<false>(bytes / (2 * rows) / 8 * 8, rows, bytes / (2 * rows) / 8 * 8);
            }
    printf("%ld requests\n", checked);
    return 0;
}
