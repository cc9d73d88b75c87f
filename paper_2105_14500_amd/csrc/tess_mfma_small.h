// The bf16 matrix-core kernel for small outputs: 64 x 64 or 64 x 32 tiles whose four wavefronts
// share the contraction.
#pragma once

#include "tess_mfma.h"

namespace tess {

// Fragments of 32 rows x 16 contracted elements out of the tile formats of tess_mfma.h, for the one
// k16 step of every stage that is this wavefront's.
template <int R, bool KC>
struct StepReader {
    uint32_t off[R / 32];
    __device__ __forceinline__ void init(int lane, int step)
    {
        static_for<R / 32>([&](auto f) {
            if constexpr (KC) {
                const int r = 32 * f + (lane & 31);
                off[f] = (uint32_t)(r * 128 + ((2 * step + (lane >> 5)) ^ swz_kc<64>(r)) * 16);
            } else {
                const int s = lane & 15, bl = lane >> 4;
                const int kr = 8 * (bl >> 1) + (s >> 2);
                const int granule = (2 * (bl & 1) + ((s & 3) >> 1) + 4 * f) ^ swz_mc<R>(kr);
                off[f] = (uint32_t)((16 * step + kr) * (R * 2) + granule * 16 + (s & 1) * 8);
            }
        });
    }
    __device__ __forceinline__ bf16x8 read(const char* lds_tile, int f) const
    {
        const char* p = lds_tile + off[f];
        if constexpr (KC) {
            return *(const bf16x8*)p;
        } else {
            bf16x4 lo = __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(short4v))(p)));
            bf16x4 hi = __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(short4v))(p + 4 * (R * 2))));
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    }
};

// One workgroup of four wavefronts per BM x BN tile and K part, two workgroups per compute unit.
// Wavefront w holds the whole tile for k16 step w of every 64-deep stage, so every operand byte is
// read from the LDS once per workgroup (a 2 x 2 arrangement reads it twice), and the four sums meet
// in the LDS at the end.  The ring of direct-to-LDS stages and the waits are those of
// tess_mfma_kernel.
//
// Bound: operand bytes from the L2 and behind it.  A stage of 64 x 64 (16 KiB) takes 0.17-0.25 us
// with all compute units busy, 33-40 B/clk per compute unit, the same per byte as a stage of the
// 128 x 128 kernel; a ring twice as deep (10 stages, one workgroup per compute unit) changed
// nothing, so it is not latency.  Start, finish and launch take 4-5 us in all, where the
// 128 x 128 tile with its K parts and their reduction takes 9-15: the rule and what both sides
// measure are with the cost model of the plan.
template <int BM, int BN, int NSTAGE, bool A_KC, bool B_KC, bool RAGGED, bool COLSUM>
__global__ __launch_bounds__(256) void tess_mfma_small_kernel(GemmArgs g)
{
    constexpr int BK = 64, FM = BM / 32, FN = BN / 32;
    constexpr int A_BYTES = BM * BK * 2, STAGE_BYTES = A_BYTES + BN * BK * 2;
    constexpr int LDR = BN + 8;      // row of a partial tile: rows r and r + 4, which a fragment's two
                                     // halves write together, lie half a bank line apart
    extern __shared__ __attribute__((aligned(16))) char lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN, nb = tiles_m * tiles_n;
    const int kt_per_panel = (g.Kp + BK - 1) / BK, kt_total = g.q * kt_per_panel;
    int tm, tn, z = 0, kt_begin = 0, nkt = kt_total;
    if (g.splits <= 1) {
        tile_of_block(blockIdx.x, tiles_m, tiles_n, tm, tn);
    } else {
        // the parts one after the other in XCD-major order, as in tess_mfma_kernel
        const int v = xcd_major_index(blockIdx.x, gridDim.x), per = (int)(gridDim.x >> 3);
        z = v / nb;
        tile_of_index(v - z * nb, tiles_m, tiles_n, per >= 32 ? 32 : (per >= 1 ? per : 1), tm, tn);
        const int base = kt_total / g.splits, extra = kt_total % g.splits;
        kt_begin = z * base + (z < extra ? z : extra);
        nkt = base + (z < extra ? 1 : 0);
    }
    if constexpr (RAGGED) {      // in scalar registers, and with them all that goes into the descriptors (see DmaLoader)
        tm = __builtin_amdgcn_readfirstlane(tm);
        tn = __builtin_amdgcn_readfirstlane(tn);
    }
    const int row0 = tm * BM, col0 = tn * BN;

    typedef DmaLoader<BM, BK, A_KC, 256, RAGGED> LA;
    typedef DmaLoader<BN, BK, B_KC, 256, RAGGED> LB;
    constexpr int LOADS = LA::ITERS + LB::ITERS;
    static_assert(NSTAGE * LOADS <= 63, "the wait counter has six bits");
    typedef __attribute__((address_space(4))) const GemmArgs* KernArgs;
    const KernArgs ka = (KernArgs)__builtin_amdgcn_kernarg_segment_ptr();
    const uint32_t lds_base = (uint32_t)(uintptr_t)(LDS_PTR(char))lds;
    const uint32_t a_kstep = A_KC ? (uint32_t)BK * 2 : (uint32_t)(BK * g.lda * 2);
    const uint32_t b_kstep = B_KC ? (uint32_t)BK * 2 : (uint32_t)(BK * g.ldb * 2);

    // next stage to request; past the end the last one is requested again, so that the wait counts
    // stay constant.  The descriptors change with the panel (RAGGED: the stage) only.
    int ld_t = kt_begin / kt_per_panel, ld_ks = kt_begin - ld_t * kt_per_panel, ld_left = nkt;
    uint64_t from_a = LA::start((uint64_t)(uintptr_t)ka->a[ld_t], row0, g.lda, ld_ks * a_kstep);
    uint64_t from_b = LB::start((uint64_t)(uintptr_t)ka->b[ld_t], col0, g.ldb, ld_ks * b_kstep);
    u32x4 rsrc_a = LA::descriptor(from_a), rsrc_b = LB::descriptor(from_b);
    LA la;
    LB lb;
    const int ktail = g.Kp - (kt_per_panel - 1) * BK;
    la.init(lane, wave, row0, g.M, g.lda, ktail);
    lb.init(lane, wave, col0, g.N, g.ldb, ktail);
    uint32_t rq_stage = 0, rq_asoff = 0, rq_bsoff = 0, rq_apast = 0, rq_bpast = 0;
    auto aim = [&](int slot) {
        rq_stage = __builtin_amdgcn_readfirstlane(lds_base + slot * STAGE_BYTES);
        if constexpr (RAGGED) {
            const bool last = ld_ks + 1 == kt_per_panel;
            rq_apast = last ? la.past_end : 0u;
            rq_bpast = last ? lb.past_end : 0u;
        } else {
            rq_asoff = __builtin_amdgcn_readfirstlane(ld_ks * a_kstep);
            rq_bsoff = __builtin_amdgcn_readfirstlane(ld_ks * b_kstep);
        }
    };
    auto advance = [&] {        // behind the requests of the stage that was aimed at
        if (ld_left > 1) {
            --ld_left;
            bool moved = RAGGED;
            if (++ld_ks == kt_per_panel) {
                ld_ks = 0;
                ++ld_t;
                from_a = LA::start((uint64_t)(uintptr_t)ka->a[ld_t], row0, g.lda, 0u);
                from_b = LB::start((uint64_t)(uintptr_t)ka->b[ld_t], col0, g.ldb, 0u);
                moved = true;
            } else if constexpr (RAGGED) {
                from_a += a_kstep;
                from_b += b_kstep;
            }
            if (moved) {
                rsrc_a = LA::descriptor(from_a);
                rsrc_b = LB::descriptor(from_b);
            }
        }
    };
    auto request = [&](auto it) {
        if constexpr (it < LA::ITERS) la.request(it, rsrc_a, rq_stage, wave, rq_asoff, rq_apast);
        else lb.request(std::integral_constant<int, it - LA::ITERS>{}, rsrc_b, rq_stage + A_BYTES, wave, rq_bsoff, rq_bpast);
    };

    static_for<NSTAGE>([&](auto s) {
        aim(s);
        static_for<LOADS>([&](auto it) { request(it); });
        advance();
    });

    StepReader<BM, A_KC> ra;
    StepReader<BN, B_KC> rb;
    ra.init(lane, wave);
    rb.init(lane, wave);
    floatx16 acc[FM * FN];
    static_for<FM * FN>([&](auto f) { static_for<16>([&](auto r) { acc[f][r()] = 0.0f; }); });
    const bool cs_block = COLSUM && g.colsum != nullptr && tm == 0;
    float cs[COLSUM ? FN : 1];
    if constexpr (COLSUM) static_for<FN>([&](auto j) { cs[j] = 0.0f; });

    bf16x8 af[2][FM], bfr[2][FN];
    auto load_frags = [&](auto buf, int slot) {
        const char* s = lds + slot * STAGE_BYTES;
        static_for<FN>([&](auto j) { bfr[buf][j] = rb.read(s + A_BYTES, j); });
        static_for<FM>([&](auto i) { af[buf][i] = ra.read(s, i); });
    };
    wait_vmcnt<(NSTAGE - 1) * LOADS>();          // stage 0 has landed
    lds_barrier();
    load_frags(std::integral_constant<int, 0>{}, 0);

    int slot = 0;
    // stage r, whose fragments are in set `cur`: once every wavefront has its own and stage r+1 has
    // landed, the fragments of r+1 are read and stage r+NSTAGE goes into the freed slot behind the
    // MFMAs of stage r
    auto period = [&](auto cur) {
        const int next = slot + 1 == NSTAGE ? 0 : slot + 1;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_vmcnt<(NSTAGE - 2) * LOADS>();
        lds_barrier();
        load_frags(std::integral_constant<int, cur ^ 1>{}, next);
        aim(slot);
        __builtin_amdgcn_sched_barrier(0);
        static_for<FM * FN>([&](auto x) {
            constexpr int i = x / FN, j = (i & 1) ? FN - 1 - x % FN : x % FN;
            acc[i * FN + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[cur][i], bfr[cur][j], acc[i * FN + j], 0, 0, 0);
            // requests spread over the MFMAs, the rest behind the last one
            constexpr int lo = x * LOADS / (FM * FN), hi = (x + 1) * LOADS / (FM * FN);
            static_for<hi - lo>([&](auto p) { request(std::integral_constant<int, lo + p>{}); });
            __builtin_amdgcn_sched_barrier(0);
        });
        advance();
        if constexpr (COLSUM) {
            if (cs_block) {
                typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
                static_for<FN>([&](auto j) {
                    const bf16x8 b = bfr[cur][j];
                    cs[j] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 0, 1), one2, cs[j], false);
                    cs[j] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 2, 3), one2, cs[j], false);
                    cs[j] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 4, 5), one2, cs[j], false);
                    cs[j] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 6, 7), one2, cs[j], false);
                });
            }
        }
        slot = next;
    };
    for (int r = 0; r < nkt; r += 2) {
        period(std::integral_constant<int, 0>{});
        if (r + 1 < nkt) period(std::integral_constant<int, 1>{});
    }
    // nothing may still be landing in the LDS or being read from it
    wait_vmcnt<0>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    lds_barrier();

    // ---- the four partial tiles side by side in the LDS, row-major
    float* red = (float*)lds;
    static_for<FM * FN>([&](auto f) {
        const int r0 = 32 * (f / FN) + 4 * (lane >> 5), c = 32 * (f % FN) + (lane & 31);
        static_for<16>([&](auto x) { red[(wave * BM + r0 + 8 * (x / 4) + x % 4) * LDR + c] = acc[f][x()]; });
    });
    float* csum = red + 4 * BM * LDR;              // [4][BN]
    if constexpr (COLSUM) {
        if (cs_block) {
            static_for<FN>([&](auto j) {
                const float v = cs[j] + __shfl_xor(cs[j], 32, 64);   // the halves hold other k of the step
                if (lane < 32) csum[wave * BN + 32 * j + lane] = v;
            });
        }
    }
    lds_barrier();
    const bool split = g.splits > 1;
    if constexpr (COLSUM) {
        const int col = col0 + tid;
        if (cs_block && tid < BN && col < g.N) {
            const float v = csum[tid] + csum[BN + tid] + csum[2 * BN + tid] + csum[3 * BN + tid];
            if (split) (g.ws + (size_t)g.splits * nb * (BM * BN) + (size_t)z * g.N)[col] = v;
            else g.colsum[col] = g.accumulate ? g.colsum[col] + v : v;
        }
    }
    auto sum4 = [&](int row, int c) {
        const float* p = red + row * LDR + c;
        floatx4 v = *(const floatx4*)p;
        static_for<3>([&](auto w) { v += *(const floatx4*)(p + (w + 1) * (BM * LDR)); });
        return v;
    };
    constexpr int CPR = BN / 4, NIT = BM * CPR / 256;      // four columns per thread and pass
    const int c4 = tid % CPR * 4, r4 = tid / CPR, col = col0 + c4;
    if (split) {
        // partial tiles row-major: [(z*nb + tile)][BM][BN]
        float* w = g.ws + ((size_t)z * nb + (size_t)(tm * tiles_n + tn)) * (BM * BN);
        static_for<NIT>([&](auto it) {
            const int row = it * (256 / CPR) + r4;
            *(floatx4*)(w + row * BN + c4) = sum4(row, c4);
        });
        return;
    }
    const bool vec = rows_aligned(g);
    const bool dgelu = drains_dgelu(g);
    auto bias_of = [&](int cb) {
        floatx4 b = {0.f, 0.f, 0.f, 0.f};
        if (g.bias) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (cb + e < g.N) b[e] = bf16_bits_to_f32(((const uint16_t*)g.bias)[cb + e]);
        }
        return b;
    };
    if (dgelu) {
        u32x2 zr[NIT];
        static_for<NIT>([&](auto it) { zr[it] = load_z4(g, row0 + it * (256 / CPR) + r4, col, vec); });
        static_for<NIT>([&](auto it) {
            const int rl = it * (256 / CPR) + r4;
            if (row0 + rl < g.M && col < g.N) emit4<MODE_BF16_DGELU>(g, row0 + rl, col, sum4(rl, c4), floatx4{0.f, 0.f, 0.f, 0.f}, vec, zr[it]);
        });
        return;
    }
    with_drain_mode(g, [&](auto mode) {
        if constexpr (mode == MODE_BF16 || mode == MODE_BF16_GELU || mode == MODE_BF16_GELU_PRE) {
            constexpr int CPR8 = BN / 8, NIT8 = BM * CPR8 / 256;
            const int c8 = tid % CPR8 * 8, col8 = col0 + c8;
            const floatx4 b0 = bias_of(col8), b1 = bias_of(col8 + 4);
            static_for<NIT8>([&](auto it) {
                const int rl = it * (256 / CPR8) + tid / CPR8;
                if (row0 + rl < g.M && col8 < g.N) emit8_bf16<mode>(g, row0 + rl, col8, sum4(rl, c8), sum4(rl, c8 + 4), b0, b1, vec);
            });
        } else {
            const floatx4 b = bias_of(col);
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                const int rl = it * (256 / CPR) + r4;
                if (row0 + rl < g.M && col < g.N) emit4<mode>(g, row0 + rl, col, sum4(rl, c4), b, vec);
            }
        }
    });
}

// Sums the row-major K parts in ascending order and applies the epilogue: one thread per four columns.
template <int BM, int BN>
__global__ __launch_bounds__(256) void tess_small_reduce_kernel(GemmArgs g)
{
    constexpr int PER_TILE = BM * BN / 4;
    const int tiles_n = (g.N + BN - 1) / BN, tiles_m = (g.M + BM - 1) / BM;
    const int64_t nb = (int64_t)tiles_m * tiles_n;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    reduce_colsum(g, gid, nb * (BM * BN));
    const int tile = (int)(gid / PER_TILE), idx = (int)(gid % PER_TILE) * 4;
    if (tile >= nb) return;
    const int row = tile / tiles_n * BM + idx / BN, col = tile % tiles_n * BN + idx % BN;
    if (row >= g.M || col >= g.N) return;
    reduce_emit4(g, row, col, g.ws + (size_t)tile * (BM * BN) + idx, (size_t)nb * (BM * BN) / 4);
}

template <int BM, int BN, int NSTAGE, bool A_KC, bool B_KC, bool RAGGED, bool COLSUM>
static hipError_t launch_small(const GemmArgs& g, const Plan& p, hipStream_t s)
{
    constexpr int ring = NSTAGE * (BM + BN) * 128, finish = 4 * BM * (BN + 8) * 4 + 4 * BN * 4;
    constexpr int lds_bytes = ring > finish ? ring : finish;
    auto kern = tess_mfma_small_kernel<BM, BN, NSTAGE, A_KC, B_KC, RAGGED, COLSUM>;
    static std::atomic<uint64_t> attr_done{0};
    hipError_t e = allow_dynamic_lds((const void*)kern, lds_bytes, attr_done);
    if (e != hipSuccess) return e;
    const int tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
    GemmArgs a = g;
    a.splits = p.splits > 1 ? p.splits : 1;
    hipLaunchKernelGGL(kern, dim3(tiles * a.splits, 1, 1), dim3(256), lds_bytes, s, a);
    e = hipGetLastError();
    if (e != hipSuccess || a.splits == 1) return e;
    hipLaunchKernelGGL((tess_small_reduce_kernel<BM, BN>), dim3((unsigned)(((int64_t)tiles * (BM * BN / 4) + 255) / 256)),
                       dim3(256), 0, s, a);
    return hipGetLastError();
}

// All variants of one operand layout.
template <bool A_KC, bool B_KC, bool COLSUM>
static hipError_t launch_layout(const GemmArgs& g, const Plan& p, hipStream_t s)
{
    if (p.bm == 64 && p.bn == 64) {
        if (!p.direct) return launch_small<64, 64, 5, A_KC, B_KC, true, COLSUM>(g, p, s);
        return launch_small<64, 64, 5, A_KC, B_KC, false, COLSUM>(g, p, s);
    }
    if (p.bm == 64 && p.bn == 32) {
        if (!p.direct) return launch_small<64, 32, 6, A_KC, B_KC, true, COLSUM>(g, p, s);
        return launch_small<64, 32, 6, A_KC, B_KC, false, COLSUM>(g, p, s);
    }
    return launch_tiles<A_KC, B_KC, COLSUM>(g, p, s);
}

}  // namespace tess
