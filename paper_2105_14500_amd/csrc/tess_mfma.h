// The bf16 matrix-core path: one kernel template (v_mfma_f32_32x32x16_bf16, fp32 accumulators that
// stay in registers over all q steps, operand tiles through LDS), the reduction behind its K
// splits, and their launch.  Instantiated by tess_mfma_fwd.hip, tess_mfma_dx.hip and
// tess_mfma_dw.hip (one operand layout each, so that they compile side by side).
#pragma once

#include "tess_epilogue.h"

#include <atomic>

namespace tess {

// Build-time diagnostic (off in the product build): wavefront 0 of every workgroup writes
// 100 MHz timestamps of its phases to the workspace.
#ifdef TESS_STAMPS
#define TESS_STAMP(i)                                                                      \
    do {                                                                                   \
        if (threadIdx.x == 0)                                                              \
            g.stamps[blockIdx.x * 16 + (i)] = wall_clock64(); \
    } while (0)
#else
#define TESS_STAMP(i)
#endif

// ---------------------------------------------------------------------------
// MFMA path
// ---------------------------------------------------------------------------
// LDS tile formats, in 16-byte granules (8 bf16), for a stage of BK contracted
// elements (CH = BK/8 granules along k):
//  KC operand, R rows x BK k:  granule (r, pc) at index r*CH + pc holds k-chunk
//      c = pc ^ swz_kc(r) of row r.  A 32x32x16 fragment read (lane -> row l%32,
//      chunk 2*kk + l/32, one 128-bit read) then touches every bank once per
//      16 consecutive rows.
//  MC operand, BK k-rows x R elements: granule (kr, pg) at index kr*(R/8) + pg
//      holds elements 8g..8g+7, g = pg ^ swz_mc(kr), of k-row kr.  Fragments are
//      read with the transposing 64-bit LDS read, which hands lane s of a 16-lane
//      group the 4 k-values of column s from 4 k-rows.
// Tiles are always written linearly (granule index = it*256 + thread), so the
// swizzle is applied on the global-memory side of the copy.
template <int BK>
__host__ __device__ __forceinline__ int swz_kc(int r)
{
    constexpr int CH = BK / 8, RPL = 128 / BK;   // chunks per row, rows per 256-byte bank line
    return (r / RPL) % CH;
}
template <int R>
__host__ __device__ __forceinline__ int swz_mc(int kr)
{
    // R = 64: a k-row is half a bank line, so k-rows two apart swap its halves
    // R = 32: four k-rows are one bank line already
    return R == 32 ? 0 : R == 64 ? ((kr >> 1) & 1) << 2 : ((kr & 3) << 2) ^ (((kr >> 3) & 1) << 1);
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Workgroup barrier that orders LDS traffic only: global loads into LDS that are
// still in flight for later stages are not waited for.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Granule index -> byte offset of that granule in a stage of the operand's tile at k0 = 0, from
// the panel's first element (RELATIVE: from the tile's first one), and the k index inside the
// stage at which it starts.  Offsets of granules that a ragged stage does not have may not fit
// into 32 bits; they are not used (see DmaLoader).
template <int R, int BK, bool KC, bool RELATIVE>
__host__ __device__ __forceinline__ uint32_t granule_offset(int G, int origin, int extent, int64_t ld,
                                                            int& kpos)
{
    constexpr int CH = BK / 8, RG = R / 8;
    const int from = RELATIVE ? origin : 0;
    if (KC) {
        const int r = G / CH, pc = G % CH;
        const int c = pc ^ swz_kc<BK>(r);
        int row = origin + r;
        row = row < extent ? row : extent - 1;          // rows past the edge repeat the last row
        kpos = 8 * c;
        return (uint32_t)(((int64_t)(row - from) * ld + 8 * c) * 2);
    } else {
        const int kr = G / RG, pg = G % RG;
        const int gidx = pg ^ swz_mc<R>(kr);
        int col = origin + 8 * gidx;
        col = col + 8 <= extent ? col : extent - 8;     // granules past the edge repeat the last one
        kpos = kr;
        return (uint32_t)(((int64_t)kr * ld + (col - from)) * 2);
    }
}

// Direct global -> LDS loader.  One request is a 64-lane x 16-byte buffer load with
// the LDS modifier: lane l's 16 bytes land at M0 + imm + 16*l, its source address is
// descriptor base + per-lane offset + scalar offset + imm.  Wavefront w owns granules
// [w*ITERS*64, (w+1)*ITERS*64) of the tile and fills them 64 at a time; groups of four
// requests share one M0 value and differ in imm (1024 bytes apart in LDS), which the
// per-lane offset compensates on the global side.  Written as inline assembly on
// purpose: a wavefront can start only one such request per ~100 clocks, and the
// scalar-base form with few M0 updates is the cheapest to issue; the compiler also
// does not track these loads, so completion is enforced by the explicit vmcnt waits
// in front of the workgroup barriers and no blanket wait precedes LDS reads.  Nor does it
// keep the five wait states between a vector instruction that writes a scalar register and a
// request that reads it (it sees no memory instruction here): the descriptors have to come from
// scalar arithmetic, and the build fails where one does not (paper_2105_14500_amd/build.py).
//
// RAGGED (panels whose contraction is no multiple of BK): the requests for granules of a panel's
// last stage that lie past its end carry the offset PAST, which is outside the descriptor's range,
// and the hardware returns zeros for them: two vector instructions per request.  So that every
// granule that exists is inside the range whatever the panel's size, the descriptor starts at the
// tile's first element of the stage (less BIAS) and the scalar offset is zero.  With panels of
// rows * ld * 2 < 2^32 - 4096 bytes (refused above that on the host) the last byte of such a granule
// is at most min(R, rows) - 1 rows of ld (KC), or 63 rows and R elements (MC), from there:
//   2 ld >= 8192:  < 2^32 - 4096 - 8192 + 512, plus BIAS < PAST;   2 ld < 8192:  < 255 * 8192 + 512.
// PAST plus an immediate does not reach 2^32: the 32-bit sum would wrap to the descriptor's start,
// which lies BIAS bytes in front of the operand.
template <int R, int BK, bool KC, int NT, bool RAGGED>
struct DmaLoader {
    static constexpr int NG = R * (BK / 8);      // granules per stage
    static constexpr int ITERS = NG / NT;        // requests per wavefront per stage
    static constexpr uint32_t BIAS = 3072;       // keeps (offset - imm) non-negative
    static constexpr uint32_t PAST = 0xfffff000u;
    uint32_t off[ITERS];
    uint32_t past_end;       // RAGGED: bit it = request `it` of a panel's last stage lies past the end
    static_assert(ITERS <= 32, "a bit per request");
    static_assert((uint64_t)PAST + BIAS + 16 <= (uint64_t)1 << 32, "no wrap");
    static_assert((uint64_t)DMA_PANEL_LIMIT - 8192 + 512 + BIAS <= PAST, "every granule of a panel is in range");
    static_assert(R <= 256 && 255 * 8192 + 512 + BIAS <= PAST, "as above, short rows");

    // byte offset, before the immediate, of the request for granule G of a stage
    static __host__ __device__ __forceinline__ uint32_t offset(int it, int G, int origin, int extent, int64_t ld, int& kpos)
    {
        return granule_offset<R, BK, KC, RAGGED>(G, origin, extent, ld, kpos) + BIAS - (it % 4) * 1024;
    }
    // the offset that is sent; `past`: `past_end` in a panel's last stage, else 0
    static __host__ __device__ __forceinline__ uint32_t sent(int it, uint32_t off, uint32_t past)
    {
        if (!RAGGED) return off;
        const uint32_t mask = (uint32_t)((int32_t)(past << (31 - it)) >> 31);
        return (mask & PAST) | (~mask & off);
    }
    // where the descriptor of a stage starts: in the panel at `panel`, the tile at row or column
    // `origin`, `adv` bytes along K.  A later stage of the panel starts that many bytes on.
    static __host__ __device__ __forceinline__ uint64_t start(uint64_t panel, int origin, int64_t ld, uint32_t adv)
    {
        if (!RAGGED) return panel - BIAS;
        return (panel + (uint64_t)(KC ? origin * ld : origin) * 2 + adv - BIAS) & 0xffffffffffffull;
    }

    // ktail: contracted elements of a panel's last stage
    __device__ __forceinline__ void init(int lane, int wave_u, int origin, int extent, int64_t ld, int ktail)
    {
        past_end = 0;
        static_for<ITERS>([&](auto it) {
            const int G = (wave_u * ITERS + it) * 64 + lane;
            int kpos;
            off[it] = offset(it, G, origin, extent, ld, kpos);
            if (RAGGED && kpos >= ktail) past_end |= 1u << it;
        });
    }
    // buffer descriptor of a panel, RAGGED: of one stage (kept by the caller in scalar registers)
    static __device__ __forceinline__ u32x4 descriptor(uint64_t from)
    {
        u32x4 rsrc;
        rsrc[0] = __builtin_amdgcn_readfirstlane((uint32_t)from);
        // stride 0 (RAGGED: start() has cleared the upper half, so that a stage costs no more than two additions)
        rsrc[1] = __builtin_amdgcn_readfirstlane(RAGGED ? (uint32_t)(from >> 32) : (uint32_t)(from >> 32) & 0xffffu);
        rsrc[2] = RAGGED ? PAST : 0xffffffffu;   // else no range clamp: every offset is in bounds
        rsrc[3] = 0x00020000u;                   // raw 32-bit data format
        return rsrc;
    }
    // lds_stage: LDS byte address of this operand's tile in the destination stage;
    // soff: byte advance of the stage along K inside the panel (wave-uniform; RAGGED: zero, the
    // descriptor has it)
    template <typename IT>
    __device__ __forceinline__ void request(IT it, const u32x4& rsrc, uint32_t lds_stage, int wave_u,
                                            uint32_t soff, uint32_t past) const
    {
        // sent(it, off[it], past) in two instructions (the compiler makes a test and a select of it, five)
        uint32_t voff = off[it];
        if constexpr (RAGGED)
            asm("v_bfe_i32 %0, %1, %2, 1\n\tv_bfi_b32 %0, %0, %3, %4"
                : "=&v"(voff) : "v"(past), "n"(it()), "s"(PAST), "v"(off[it]));
        // the descriptor must sit in scalar registers whatever the optimizer did to it
        u32x4 d;
        d[0] = __builtin_amdgcn_readfirstlane(rsrc[0]);
        d[1] = __builtin_amdgcn_readfirstlane(rsrc[1]);
        d[2] = __builtin_amdgcn_readfirstlane(rsrc[2]);
        d[3] = __builtin_amdgcn_readfirstlane(rsrc[3]);
        // One M0 value serves the four requests of a group (they differ in the immediate).
        // The compiler is only told that M0 is clobbered, not that it must survive until
        // the group's last request, so the build scans the generated code and fails if
        // anything but these statements writes M0 (paper_2105_14500_amd/build.py).
        if constexpr (it % 4 == 0) {
            const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_stage + (uint32_t)(wave_u * ITERS + it) * 1024u);
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" : : "s"(m0) : "m0", "memory");
        }
        asm volatile("buffer_load_dwordx4 %0, %1, %2 offen offset:%3 lds"
                     :
                     : "v"(voff), "s"(d), "s"(__builtin_amdgcn_readfirstlane(soff)), "n"((it % 4) * 1024)
                     : "memory");
    }
};

// Fragment reader: 32 (rows along R) x 16 (k) bf16 operand fragment for
// v_mfma_f32_32x32x16_bf16: lane l gets row l%32, k = 8*(l/32) .. +7.
template <int R, int BK, bool KC>
struct FragReader {
    static constexpr int KSTEPS = BK / 16;
    uint32_t lane_off;          // per-lane byte offset, fragment 0
    uint32_t kcol[KC ? KSTEPS : 2];   // KC: byte offset of the k-chunk for each k16 step
    __device__ __forceinline__ void init(int lane, int wave_origin)
    {
        if constexpr (KC) {
            const int r = wave_origin + (lane & 31);
            lane_off = (uint32_t)r * (uint32_t)(BK * 2);
            static_for<KSTEPS>([&](auto kk) {
                kcol[kk] = (uint32_t)(((2 * kk + (lane >> 5)) ^ swz_kc<BK>(r)) * 16);
            });
        } else {
            const int s = lane & 15, bl = lane >> 4;
            const int kr = 8 * (bl >> 1) + (s >> 2);           // k-row inside a k16 step, first read
            lane_off = (uint32_t)(kr * (R / 8) * 16 + (s & 1) * 8);
            kcol[0] = (uint32_t)swz_mc<R>(kr);
            kcol[1] = (uint32_t)(wave_origin + 16 * (bl & 1) + 4 * (s & 3)) >> 3;  // granule, frag 0
        }
    }
    // f: fragment index along R inside the wave tile, kk: k16 step of the stage
    __device__ __forceinline__ bf16x8 read(const char* lds_tile, int f, int kk) const
    {
        if constexpr (KC) {
            return *(const bf16x8*)(lds_tile + lane_off + f * (32 * BK * 2) + kcol[kk]);
        } else {
            const uint32_t gsw = ((kcol[1] + 4u * f) ^ kcol[0]) * 16u;
            const char* p = lds_tile + lane_off + gsw + kk * (16 * (R / 8) * 16);
            bf16x4 lo = __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                       (LDS_PTR(short4v))(p)));
            bf16x4 hi = __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                       (LDS_PTR(short4v))(p + 4 * (R / 8) * 16)));
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    }
};

// WGM x WGN wavefronts tile the BM x BN macro tile; each owns (BM/WGM) x (BN/WGN).
// COLSUM: the wavefronts in the first tile row that hold the top wave tile also sum the
// columns of the B operand over the contraction, from the B fragments they already hold
// in registers: four 2-element bf16 dot products with (1, 1) per fragment and k16 step,
// fp32 accumulation, issued in the shadow of the MFMAs.  (An extra MFMA with an all-ones
// A fragment would need accumulator registers that the tile already uses up: the
// compiler then copies 16 registers in and out around every such MFMA.)
template <int BM, int BN, int BK, int NSTAGE, int WGM, int WGN, bool A_KC, bool B_KC, bool RAGGED,
          bool COLSUM = false>
__global__ __launch_bounds__(64 * WGM * WGN) void tess_mfma_kernel(GemmArgs g)
{
    constexpr int NT = 64 * WGM * WGN;
    constexpr int WTM = BM / WGM, WTN = BN / WGN;      // wave tile
    constexpr int FM = WTM / 32, FN = WTN / 32;        // 32x32 fragments per wave tile
    constexpr int KSTEPS = BK / 16;
    constexpr bool SNAKE = true;
    constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
    constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    extern __shared__ __attribute__((aligned(16))) char lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    TESS_STAMP(0);
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int wm = wave / WGN, wn = wave % WGN;
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    const int nb = tiles_m * tiles_n;
    const int kt_per_panel = (g.Kp + BK - 1) / BK;
    const int kt_total = g.q * kt_per_panel;

    // ---- work of this workgroup: one output tile and a range of K stages: the whole K
    // loop, or one of g.splits equal parts of it (tiles x parts workgroups, with the
    // reduction kernel behind the launch)
    int tm = 0, tn = 0, row0 = 0, col0 = 0, kt_begin = 0, nkt = 0;

    typedef DmaLoader<BM, BK, A_KC, NT, RAGGED> LA;
    typedef DmaLoader<BN, BK, B_KC, NT, RAGGED> LB;
    constexpr int LOADS = LA::ITERS + LB::ITERS;       // requests per wavefront per stage
    FragReader<BM, BK, A_KC> ra;
    FragReader<BN, BK, B_KC> rb;
    ra.init(lane, wm * WTM);
    rb.init(lane, wn * WTN);

    floatx16 acc[FM * FN];
    // column sums (COLSUM only): the wavefronts that hold the top wave tile of the first tile row
    bool cs_wave = false;
    float cs[COLSUM ? FN : 1];

    // byte advance of one stage along K for each operand
    const uint32_t a_kstep = A_KC ? (uint32_t)BK * 2 : (uint32_t)(BK * g.lda * 2);
    const uint32_t b_kstep = B_KC ? (uint32_t)BK * 2 : (uint32_t)(BK * g.ldb * 2);

    // Panel pointers are fetched from the kernel-argument segment (constant address
    // space, scalar loads) with the uniform step index; indexing the by-value copy
    // of the argument struct dynamically would move it to scratch memory.
    typedef __attribute__((address_space(4))) const GemmArgs* KernArgs;
    const KernArgs ka = (KernArgs)__builtin_amdgcn_kernarg_segment_ptr();
    // (panel, stage-in-panel) of the next stage to fetch, advanced incrementally
    int ld_t = 0, ld_ks = 0;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(LDS_PTR(char))lds;

    bf16x8 af[2][FM], bfr[2][FN];
    // Fragment u of a k16 step: the FN fragments of B first, then the FM of A (the
    // first MFMAs of a step need af[0] and every bfr[j]).
    auto load_frag = [&](auto buf, int stage, auto kk, auto u) {
        const char* sa = lds + stage * STAGE_BYTES;
        if constexpr (u < FN) bfr[buf][u] = rb.read(sa + A_BYTES, u, kk);
        else af[buf][u - FN] = ra.read(sa, u - FN, kk);
    };
    auto load_frags = [&](auto buf, int stage, auto kk) {
        static_for<FM + FN>([&](auto u) { load_frag(buf, stage, kk, u); });
    };
    // One k16 step written out in issue order: MFMA x is followed by the side work
    // side(x) (LDS reads of the next step, requests for a later tile), and a
    // scheduling fence keeps the compiler from regrouping them, so the matrix pipe
    // is fed while the reads and requests are in flight.
    auto mfma_step = [&](auto buf, auto&& side) {
        static_for<FM * FN>([&](auto x) {
            // serpentine over the fragment grid: consecutive MFMAs share one operand
            // register set (fewer operand-bus toggles; a few percent under the power cap)
            constexpr int i = x / FN, j = (SNAKE && (i & 1)) ? FN - 1 - x % FN : x % FN;
            acc[i * FN + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[buf][i], bfr[buf][j], acc[i * FN + j], 0, 0, 0);
            side(x);
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (COLSUM) {
            if (cs_wave) {
                typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
                static_for<FN>([&](auto j) {
                    const bf16x8 b = bfr[buf][j];
                    cs[j] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 0, 1), one2, cs[j], false);
                    cs[j] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 2, 3), one2, cs[j], false);
                    cs[j] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 4, 5), one2, cs[j], false);
                    cs[j] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 6, 7), one2, cs[j], false);
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    constexpr int LASTBUF = (KSTEPS - 1) & 1;
    constexpr int NSLOT = KSTEPS * FM * FN;            // MFMA slots per tile
    constexpr int FPS = (FM + FN + FM * FN - 1) / (FM * FN);   // fragment reads per MFMA slot
    // the fragments of the next k16 step that are read behind MFMA x of this one
    auto load_frags_at = [&](auto buf, int stage, auto kk, auto x) {
        static_for<FPS>([&](auto p) {
            if constexpr (x * FPS + p < FM + FN) load_frag(buf, stage, kk, std::integral_constant<int, x * FPS + p>{});
        });
    };
    // request number `it` of a tile is attached to MFMA slot it*NSLOT/LOADS of the
    // period that follows the barrier which frees the destination slot, so the
    // requests trickle out at the rate the texture path can take them
    LA la;
    LB lb;
    // State of the tile being requested (captured by aim(), so that the requests that
    // trickle out later do not see the pointers already advanced to the next tile).
    uint32_t rq_stage = 0;          // LDS address of the stage being filled
    uint32_t rq_asoff = 0, rq_bsoff = 0;   // K advance of that tile inside its panels (RAGGED: in the descriptors)
    uint32_t rq_apast = 0, rq_bpast = 0;   // RAGGED: requests of that tile that lie past the panel's end
    u32x4 rq_rsrc_a = {0u, 0u, 0u, 0u}, rq_rsrc_b = {0u, 0u, 0u, 0u};
    int rq_left = 0;                // tiles not yet aimed at
    uint64_t rg_a = 0, rg_b = 0;    // RAGGED: where the next stage's descriptors start
    auto request = [&](auto it) {
        if constexpr (it < LA::ITERS) la.request(it, rq_rsrc_a, rq_stage, wave_u, rq_asoff, rq_apast);
        else lb.request(std::integral_constant<int, it - LA::ITERS>{}, rq_rsrc_b, rq_stage + A_BYTES, wave_u, rq_bsoff, rq_bpast);
    };
    // Point the requests at LDS stage `stage` and the next tile of the K loop.  Past
    // the end of the loop the last tile is requested again (into a slot nobody reads):
    // every period then issues the same requests and the wait counts stay constant.
    auto aim = [&](int stage) {
        rq_stage = __builtin_amdgcn_readfirstlane(lds_base + stage * STAGE_BYTES);
        if constexpr (RAGGED) {
            const bool last = ld_ks + 1 == kt_per_panel;
            rq_apast = last ? la.past_end : 0u;
            rq_bpast = last ? lb.past_end : 0u;
            rq_rsrc_a = LA::descriptor(rg_a);
            rq_rsrc_b = LB::descriptor(rg_b);
        } else {
            rq_asoff = __builtin_amdgcn_readfirstlane(ld_ks * a_kstep);
            rq_bsoff = __builtin_amdgcn_readfirstlane(ld_ks * b_kstep);
#ifdef TESS_DBG_SAMEK
            rq_asoff = rq_bsoff = 0;      // diagnostic build (wrong results): every stage re-reads K slice 0, so all requests hit the L2
#endif
            const int t = ld_t < g.q ? ld_t : g.q - 1;
            rq_rsrc_a = LA::descriptor(LA::start((uint64_t)(uintptr_t)ka->a[t], row0, g.lda, 0u));
            rq_rsrc_b = LB::descriptor(LB::start((uint64_t)(uintptr_t)ka->b[t], col0, g.ldb, 0u));
        }
        if (rq_left > 1) {
            --rq_left;
            if (++ld_ks == kt_per_panel) {
                ld_ks = 0;
                ++ld_t;
                if constexpr (RAGGED) {
                    rg_a = LA::start((uint64_t)(uintptr_t)ka->a[ld_t], row0, g.lda, 0u);
                    rg_b = LB::start((uint64_t)(uintptr_t)ka->b[ld_t], col0, g.ldb, 0u);
                }
            } else if constexpr (RAGGED) {
                rg_a += a_kstep;
                rg_b += b_kstep;
            }
        }
    };
    // with three or more stages a tile has more than a period to land and its requests
    // are spread over the whole period; with two stages they go out in the first half
    constexpr int RQ_SPAN = NSTAGE >= 3 ? NSLOT : NSLOT / 2;
    constexpr int STRIDE = RQ_SPAN / LOADS;
    static_assert(STRIDE >= 1, "requests spaced evenly over the MFMA slots");
    auto request_at = [&](auto slot) {
#ifndef TESS_DBG_NOLOAD   // (a diagnostic build without the in-loop requests measures the loop on resident data)
        if constexpr (slot % STRIDE == 0 && slot / STRIDE < LOADS)
            request(std::integral_constant<int, slot / STRIDE>{});
#endif
    };
    // The k16 steps 0 .. KSTEPS-2 of the tile in `stage`: each fetches the next step's
    // fragments with its first MFMAs.  REQ: also carry requests (slots FM*FN ..).
    auto body_steps = [&](int stage) {
        static_for<KSTEPS - 1>([&](auto kk) {
            mfma_step(std::integral_constant<int, kk & 1>{}, [&](auto x) {
                load_frags_at(std::integral_constant<int, (kk + 1) & 1>{}, stage, std::integral_constant<int, kk + 1>{}, x);
                request_at(std::integral_constant<int, (kk + 1) * FM * FN + x>{});
            });
        });
    };
    // The last k16 step of a tile, carrying the first fragments of the tile in `next`
    // (FETCH) and the first requests (REQ, slots 0 .. FM*FN-1).
    auto last_step = [&](int next) {
        mfma_step(std::integral_constant<int, LASTBUF>{}, [&](auto x) {
            load_frags_at(std::integral_constant<int, (LASTBUF ^ 1)>{}, next, std::integral_constant<int, 0>{}, x);
            request_at(std::integral_constant<int, x>{});
        });
    };

    int z = 0;                      // K part of this workgroup
    {
        kt_begin = 0;
        nkt = kt_total;
        if (g.splits <= 1) {
            tile_of_block(blockIdx.x, tiles_m, tiles_n, tm, tn);
        } else {
            // One launch of tiles x parts workgroups.  In the XCD-major order of the blocks the
            // parts come one after the other, each with all its tiles: an XCD then works on a
            // run of tiles of ONE part at a time (the workgroups that share panels in its L2 are
            // at the same K offset), in patches like the launch without a split.
            const int v = xcd_major_index(blockIdx.x, gridDim.x);
            z = v / nb;
            const int per = (int)(gridDim.x >> 3);
            tile_of_index(v - z * nb, tiles_m, tiles_n, per >= 32 ? 32 : (per >= 1 ? per : 1), tm, tn);
            const int base = kt_total / g.splits, extra = kt_total % g.splits;
            kt_begin = z * base + (z < extra ? z : extra);
            nkt = base + (z < extra ? 1 : 0);
        }
        if constexpr (RAGGED) {      // in scalar registers, and with them all that goes into the descriptors (see DmaLoader)
            tm = __builtin_amdgcn_readfirstlane(tm);
            tn = __builtin_amdgcn_readfirstlane(tn);
        }
        row0 = tm * BM;
        col0 = tn * BN;
        ld_t = kt_begin / kt_per_panel;
        ld_ks = kt_begin - ld_t * kt_per_panel;
        static_for<FM * FN>([&](auto f) {
            static_for<16>([&](auto r) { acc[f][r()] = 0.0f; });
        });
        if constexpr (COLSUM) {
            cs_wave = __builtin_amdgcn_readfirstlane((int)(g.colsum != nullptr && tm == 0 && wm == 0));
            static_for<FN>([&](auto j) { cs[j] = 0.0f; });
        }

        // Ring of NSTAGE LDS slots; tile r lives in slot r % NSTAGE.  Barrier r (every
        // wave has read tile r, tile r+1 has landed) frees slot r % NSTAGE; tile
        // r+NSTAGE is then requested into it, its requests attached to the MFMAs that
        // follow (the last k16 step of tile r, then the first steps of tile r+1).  One
        // loop body serves the whole K range: see aim() for the tail.
        const int ktail = g.Kp - (kt_per_panel - 1) * BK;
        la.init(lane, wave_u, row0, g.M, g.lda, ktail);
        lb.init(lane, wave_u, col0, g.N, g.ldb, ktail);
        rq_left = nkt;
        if constexpr (RAGGED) {
            rg_a = LA::start((uint64_t)(uintptr_t)ka->a[ld_t], row0, g.lda, ld_ks * a_kstep);
            rg_b = LB::start((uint64_t)(uintptr_t)ka->b[ld_t], col0, g.ldb, ld_ks * b_kstep);
        }
        constexpr int FIRST = (FM * FN + STRIDE - 1) / STRIDE < LOADS ? (FM * FN + STRIDE - 1) / STRIDE : LOADS;
        if (nkt > 0) {
            // tiles 0 .. NSTAGE-2 in bulk, and of tile NSTAGE-1 the requests that the
            // last k16 step of a period would carry; the first body steps bring the rest
            static_for<NSTAGE - 1>([&](auto s) {
                aim(s);
                static_for<LOADS>([&](auto it) { request(it); });
            });
            aim(NSTAGE - 1);
            static_for<FIRST>([&](auto it) { request(it); });
            wait_vmcnt<(NSTAGE - 2) * LOADS + FIRST>();            // tile 0 has landed
            lds_barrier();
            TESS_STAMP(1);
            load_frags(std::integral_constant<int, 0>{}, 0, std::integral_constant<int, 0>{});
        }
        int stage = 0;
        for (int r = 0; r < nkt; ++r) {
            body_steps(stage);
            const int next = stage + 1 == NSTAGE ? 0 : stage + 1;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // my reads of tile r are done
            wait_vmcnt<(NSTAGE - 2) * LOADS>();                    // tile r+1 has landed
            lds_barrier();                                         // barrier r
            aim(stage);
            last_step(next);
            stage = next;
        }
        TESS_STAMP(2);
        // the epilogue reuses the LDS: nothing may still be landing in it
        wait_vmcnt<0>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        lds_barrier();

        // ---- finish
        const int elane = lane, ewave = wave, ewm = wm, ewn = wn;
        // column sums of this K range: lane l holds column l % 32 of each fragment for the
        // k-values 8 (l / 32) .. + 7 of every k16 step, so the two halves of the wavefront
        // add up to the column sum (valid in lanes 0..31)
        float csv[COLSUM ? FN : 1];
        if constexpr (COLSUM) {
            static_for<FN>([&](auto j) { csv[j] = cs[j] + __shfl_xor(cs[j], 32, 64); });
        }
        if (g.splits > 1) {
            // equal K parts: partial sums in accumulator order
            // [(z*nb + tile)][wave][frag][reg][lane] for the reduction kernel
            if constexpr (COLSUM) {
                if (cs_wave) {
                    float* part = g.ws + (size_t)g.splits * nb * (BM * BN) + (size_t)z * g.N;
                    static_for<FN>([&](auto j) {
                        const int col = col0 + ewn * WTN + j * 32 + elane;
                        if (elane < 32 && col < g.N) part[col] = csv[j];
                    });
                }
            }
            float* w = g.ws + ((size_t)z * nb + (size_t)(tm * tiles_n + tn)) * (BM * BN) +
                       (size_t)ewave * (FM * FN * 16 * 64) + elane;
            static_for<FM * FN>([&](auto f) {
                static_for<16>([&](auto r) { w[(f * 16 + r) * 64] = acc[f][r()]; });
                __builtin_amdgcn_sched_barrier(0);
            });
#ifdef TESS_STAMPS
            wait_vmcnt<0>(); TESS_STAMP(4);
#endif
            return;
        }
        // ---- epilogue.  The wavefront passes its accumulators through a private slice of
        // the (now idle) LDS, half of its tile at a time, to turn the MFMA fragment layout
        // into rows: a short loop then handles four adjacent columns per lane (pass `it`
        // serves rows it * RPI + lane / CPR of the half), so every output row leaves as one
        // contiguous run and the code stays small.
        constexpr int HR = WTM / 2;                    // rows per half
        constexpr int ROWB = WTN * 4;                  // fp32 bytes per row of the wave tile
        constexpr int CPR = WTN / 4;                   // 16-byte chunks per row
        constexpr int RPI = 64 / CPR;                  // rows per 64-lane pass
        constexpr int NIT = HR / RPI;                  // passes per half
        static_assert(FM % 2 == 0, "two halves of whole fragments");
        static_assert(NSTAGE * STAGE_BYTES >= WGM * WGN * HR * ROWB, "LDS holds half a tile in fp32");
        char* slice = lds + ewave * (HR * ROWB);
        const bool vec = rows_aligned(g);
        // a lane serves the same four columns in every pass
        const int c = elane % CPR, wcol0 = col0 + ewn * WTN, col = wcol0 + c * 4;
        // accumulators of one half -> the wavefront's LDS slice.  Chunk c of row r is kept at
        // chunk c ^ (8 * bit 2 of r): the two half-waves of a fragment (rows r and r+4) then
        // write to different banks (a slice row of 8 chunks has no other half to swap with)
        auto swizzle = [](int rl) { return CPR >= 16 ? ((rl >> 2) & 1) << 3 : 0; };
        auto stage_half = [&](auto half) {
            static_for<FM / 2>([&](auto ii) {
                static_for<FN>([&](auto j) {
                    constexpr int f = (half * (FM / 2) + ii) * FN + j;
                    const int cl = j * 32 + (elane & 31);
                    static_for<16>([&](auto r) {
                        const int rl = ii * 32 + 8 * (r / 4) + 4 * (elane >> 5) + (r % 4);
                        const int phys = (cl >> 2) ^ swizzle(rl);
                        *(float*)(slice + rl * ROWB + phys * 16 + (cl & 3) * 4) = acc[f][r()];
                    });
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
        };
        auto staged = [&](int it) -> floatx4* {     // the lane's four columns of pass `it`
            const int rl = it * RPI + elane / CPR;
            const int phys = c ^ swizzle(rl);
            return (floatx4*)(slice + rl * ROWB + phys * 16);
        };
        // fetch the bias of the lane's four columns once
        floatx4 bias4 = {0.f, 0.f, 0.f, 0.f};
        if (g.bias) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < g.N) bias4[e] = bf16_bits_to_f32(((const uint16_t*)g.bias)[col + e]);
        }
        if constexpr (COLSUM) {
            if (cs_wave) {
                static_for<FN>([&](auto j) {
                    const int ccol = col0 + ewn * WTN + j * 32 + elane;
                    if (elane < 32 && ccol < g.N) g.colsum[ccol] = g.accumulate ? g.colsum[ccol] + csv[j] : csv[j];
                });
            }
        }
        // dX through GELU': the pre-activations are fetched before the accumulators are staged,
        // so that their latency is hidden behind the LDS traffic instead of sitting in the loop
        const bool dgelu = drains_dgelu(g);
        static_for<2>([&](auto half) {
            const int wrow0 = row0 + ewm * WTM + half * HR;
            u32x2 zr[NIT];
            if (dgelu) {
                static_for<NIT>([&](auto it) {
                    const int row = wrow0 + it * RPI + elane / CPR;
                    zr[it] = load_z4(g, row, col, vec);
                });
            }
            stage_half(half);
            if (dgelu) {
                static_for<NIT>([&](auto it) {
                    const floatx4 v = *staged(it);
                    const int row = wrow0 + it * RPI + elane / CPR;
                    if (row < g.M && col < g.N) emit4<MODE_BF16_DGELU>(g, row, col, v, bias4, vec, zr[it]);
                });
            } else {
                with_drain_mode(g, [&](auto mode) {
                    if constexpr (mode == MODE_BF16 || mode == MODE_BF16_GELU || mode == MODE_BF16_GELU_PRE) {
                        // 2-byte outputs: eight columns per lane, so that a row leaves in 16-byte stores
                        constexpr int CPR8 = WTN / 8, RPI8 = 64 / CPR8, NIT8 = HR / RPI8;
                        const int c8 = elane % CPR8, col8 = wcol0 + c8 * 8;
                        floatx4 b0 = {0.f, 0.f, 0.f, 0.f}, b1 = {0.f, 0.f, 0.f, 0.f};
                        if (g.bias) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                if (col8 + e < g.N) b0[e] = bf16_bits_to_f32(((const uint16_t*)g.bias)[col8 + e]);
                                if (col8 + 4 + e < g.N) b1[e] = bf16_bits_to_f32(((const uint16_t*)g.bias)[col8 + 4 + e]);
                            }
                        }
#pragma unroll 4
                        for (int it = 0; it < NIT8; ++it) {
                            const int rl = it * RPI8 + elane / CPR8;
                            const int sw = swizzle(rl);
                            const floatx4 v0 = *(const floatx4*)(slice + rl * ROWB + ((2 * c8) ^ sw) * 16);
                            const floatx4 v1 = *(const floatx4*)(slice + rl * ROWB + ((2 * c8 + 1) ^ sw) * 16);
                            const int row = wrow0 + rl;
                            if (row < g.M && col8 < g.N) emit8_bf16<mode>(g, row, col8, v0, v1, b0, b1, vec);
                        }
                    } else {
#pragma unroll 4
                        for (int it = 0; it < NIT; ++it) {
                            const floatx4 v = *staged(it);
                            const int row = wrow0 + it * RPI + elane / CPR;
                            if (row < g.M && col < g.N) emit4<mode>(g, row, col, v, bias4, vec);
                        }
                    }
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        });
#ifdef TESS_STAMPS
        wait_vmcnt<0>(); TESS_STAMP(4);
#endif
    }
}

// Parts of the K-split reductions.  Column sums: the partial ones follow the tile partials
// (`partials` floats per split), one row of N per split; thread `gid` folds column `gid`.
__device__ __forceinline__ void reduce_colsum(const GemmArgs& g, int64_t gid, int64_t partials)
{
    if (!g.colsum || gid >= g.N) return;
    const float* part = g.ws + (size_t)g.splits * partials + gid;
    float cs = 0.0f;
    for (int z = 0; z < g.splits; ++z) cs += part[(size_t)z * g.N];
    g.colsum[gid] = g.accumulate ? g.colsum[gid] + cs : cs;
}
// Four adjacent columns: 16-byte reads of every split's partial (zstride granules apart), four
// splits in flight at once, and the epilogue of the single-launch path with vector stores when the
// output rows allow it.
__device__ __forceinline__ void reduce_emit4(const GemmArgs& g, int row, int col, const float* partial, size_t zstride)
{
    const floatx4* w = (const floatx4*)partial;
    floatx4 sum = {0.f, 0.f, 0.f, 0.f};
    int z = 0;
    for (; z + 4 <= g.splits; z += 4) {
        const floatx4 v0 = w[(size_t)z * zstride], v1 = w[(size_t)(z + 1) * zstride];
        const floatx4 v2 = w[(size_t)(z + 2) * zstride], v3 = w[(size_t)(z + 3) * zstride];
        sum += v0; sum += v1; sum += v2; sum += v3;
    }
    for (; z < g.splits; ++z) sum += w[(size_t)z * zstride];
    floatx4 bias4 = {0.f, 0.f, 0.f, 0.f};
    if (g.bias) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (col + e < g.N) bias4[e] = bf16_bits_to_f32(((const uint16_t*)g.bias)[col + e]);
    }
    const int esize = g.out_f32 ? 4 : 2;
    const bool vec = ((g.ldo * esize) % 16 == 0) && ((reinterpret_cast<uintptr_t>(g.out) & 15u) == 0) &&
                     (!g.preact || (reinterpret_cast<uintptr_t>(g.preact) & 15u) == 0);
    if (g.out_f32 && g.accumulate && !g.zin && !g.preact && g.act == TESS_ACT_NONE)
        emit4<MODE_F32_ACC>(g, row, col, sum, bias4, vec);
    else
        emit4<MODE_GENERIC>(g, row, col, sum, bias4, vec);
}

// Sums the K-split partials in ascending split order and applies the epilogue.
// One thread per four consecutive accumulator lanes (same row, four adjacent
// columns): 16-byte reads of every split's partial, all splits in flight at once.
template <int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(256) void tess_splitk_reduce_kernel(GemmArgs g)
{
    constexpr int WTM = BM / WGM, WTN = BN / WGN;
    constexpr int FM = WTM / 32, FN = WTN / 32;
    constexpr int PER_TILE = BM * BN / 4;
    const int tiles_n = (g.N + BN - 1) / BN, tiles_m = (g.M + BM - 1) / BM;
    const int64_t nb = (int64_t)tiles_m * tiles_n;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    reduce_colsum(g, gid, nb * (BM * BN));
    const int64_t tile = gid / PER_TILE;
    if (tile >= nb) return;
    const int idx = (int)(gid % PER_TILE) * 4;           // position in accumulator order
    const int lane = idx & 63, r = (idx >> 6) & 15, f = (idx >> 10) % (FM * FN);
    const int wave = idx / (1024 * FM * FN);
    const int wm = wave / WGN, wn = wave % WGN, i = f / FN, j = f % FN;
    const int tm = (int)(tile / tiles_n), tn = (int)(tile % tiles_n);
    const int row = tm * BM + wm * WTM + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    const int col = tn * BN + wn * WTN + j * 32 + (lane & 31);
    if (row >= g.M || col >= g.N) return;
    reduce_emit4(g, row, col, g.ws + (size_t)tile * (BM * BN) + idx, (size_t)nb * (BM * BN) / 4);
}

// The dynamic LDS limit is a per-device attribute of a kernel: set once per device (a bit per
// device id in `done`; setting it twice from two threads is harmless).
static inline hipError_t allow_dynamic_lds(const void* kern, int bytes, std::atomic<uint64_t>& done)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
    const uint64_t bit = 1ull << (dev & 63);
    if (dev > 63 || !(done.load(std::memory_order_acquire) & bit)) {
        const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
        done.fetch_or(bit, std::memory_order_release);
    }
    return hipSuccess;
}

template <int BM, int BN, int BK, int NSTAGE, int WGM, int WGN, bool A_KC, bool B_KC, bool RAGGED,
          bool COLSUM = false>
static hipError_t launch_one(const GemmArgs& g, const Plan& p, hipStream_t s)
{
    constexpr int NT = 64 * WGM * WGN;
    constexpr int lds_bytes = NSTAGE * (BM + BN) * BK * 2;
    auto kern = tess_mfma_kernel<BM, BN, BK, NSTAGE, WGM, WGN, A_KC, B_KC, RAGGED, COLSUM>;
    static std::atomic<uint64_t> attr_done{0};
    hipError_t e = allow_dynamic_lds((const void*)kern, lds_bytes, attr_done);
    if (e != hipSuccess) return e;
    const int tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
    GemmArgs a = g;
    a.splits = p.splits > 1 ? p.splits : 1;
    hipLaunchKernelGGL(kern, dim3(tiles * a.splits, 1, 1), dim3(NT), lds_bytes, s, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p.splits > 1) {
        const int64_t groups = (int64_t)tiles * (BM * BN / 4);
        hipLaunchKernelGGL((tess_splitk_reduce_kernel<BM, BN, WGM, WGN>), dim3((unsigned)((groups + 255) / 256)),
                           dim3(256), 0, s, a);
        e = hipGetLastError();
    }
    return e;
}

// The tile variants of one operand layout.
template <bool A_KC, bool B_KC, bool COLSUM>
static hipError_t launch_tiles(const GemmArgs& g, const Plan& p, hipStream_t s)
{
    if (p.bm == 256 && p.bn == 256) {
        if (!p.direct) return launch_one<256, 256, 64, 2, 2, 2, A_KC, B_KC, true, COLSUM>(g, p, s);
        return launch_one<256, 256, 64, 2, 2, 2, A_KC, B_KC, false, COLSUM>(g, p, s);
    }
    if (p.bm == 128 && p.bn == 128) {
        if (!p.direct) {
            // More workgroups than compute units: two stages, so that a compute unit holds two workgroups
            // and one's start and drain overlap with the other's loop.  Up to one each, a third stage
            // hides the loads' latency.  us a call (workgroups, stages of the contraction), 3 stages -> 2:
            //   152 x 3632 x 4952 dW (1131, 3)  60.9 -> 42.8    4 x 184 x 1568 x 4864 dW (494, 12)  37.0 -> 27.2
            //   2952 x 2152 x 72 dX  (408, 2)   12.2 ->  9.1    3 x 2520 x 2352 x 2776 fwd (440, 111)  132 -> 117
            //   4 x 928 x 2168 x 3424 fwd (216, 136)  80.2, 120 with two    2 x 2240 x 128 x 1088 fwd (162, 4)  11.2, 11.9
            const int64_t wgs = (int64_t)((g.M + 127) / 128) * ((g.N + 127) / 128) * (p.splits > 1 ? p.splits : 1);
            if (wgs > 256) return launch_one<128, 128, 64, 2, 2, 2, A_KC, B_KC, true, COLSUM>(g, p, s);
            return launch_one<128, 128, 64, 3, 2, 2, A_KC, B_KC, true, COLSUM>(g, p, s);
        }
        return launch_one<128, 128, 64, 3, 2, 2, A_KC, B_KC, false, COLSUM>(g, p, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace tess
