// The matrix-core path for fp32 blocks and for bf16 blocks whose contiguous extents are no
// multiples of 8: any shape, stride and element alignment, no workspace.
//
// Products run on v_mfma_f32_32x32x2_f32 (fp32: 256 flop/clk per compute unit, twice the unpacked
// vector rate, full fp32 operands and fp32 accumulation) or v_mfma_f32_32x32x16_bf16.  Operand tiles go through
// registers into a double-buffered LDS tile; the loads of a stage are issued two stages ahead.
//
// No edge is loaded element by element as long as the extents reach one tile and one stage: the
// last tile along M or N starts at (extent - tile) and stores only the rows and columns that no
// other tile has, and the last stage of a panel starts at (Kp - BK) with the k that came before
// zeroed in both operands (in registers, so that an infinity cannot meet a zero of the other one).
// Every load is then a full 16-byte load; the hardware takes them at any element alignment.
#pragma once

#include "tess_epilogue.h"

namespace tess {

template <typename T> struct AnyType;
template <> struct AnyType<float> {
    static constexpr int E = 4;        // elements of a 16-byte granule
    static constexpr int KG = 8;       // contracted elements of one fragment read
    static constexpr int KC_PAD = 4;   // LDS row padding in elements (bank spread of 128-bit reads)
    static constexpr int mc_pad(int) { return 8; }   // rows k and k+4 fall into different bank halves
};
template <> struct AnyType<__bf16> {
    static constexpr int E = 8;
    static constexpr int KG = 16;
    static constexpr int KC_PAD = 8;
    // transposing reads take 64 bytes from each of 4 k-rows: row strides of 64 mod 128 bytes
    static constexpr int mc_pad(int r) { return r == 32 ? 0 : 32; }
};

struct __attribute__((packed, aligned(2))) Granule2 { u32x4 v; };
struct __attribute__((packed, aligned(4))) Granule4 { u32x4 v; };

// Tile of R rows (columns of B) by BK contracted elements: granule `it * NT + tid` of the stage
// goes from global memory through `v` to the LDS tile.
template <typename T, int R, int BK, bool KC, int NT>
struct AnyLoader {
    static constexpr int E = AnyType<T>::E;
    static constexpr int ITERS = R * BK / E / NT;
    static constexpr int LD = KC ? BK + AnyType<T>::KC_PAD : R + AnyType<T>::mc_pad(R);   // LDS row, elements
    static constexpr int BYTES = (KC ? R : BK) * LD * (int)sizeof(T);
    static_assert(R * BK / E % NT == 0, "whole granules per thread");
    int64_t off[ITERS];       // element offset from the tile's first element of the stage
    __device__ static __forceinline__ int r_of(int G) { return KC ? G / (BK / E) : G % (R / E) * E; }
    __device__ static __forceinline__ int k_of(int G) { return KC ? G % (BK / E) * E : G / (R / E); }

    // rem_r: rows that exist from the tile's first one.  Whole rows past the edge repeat the last row
    // (what they contribute to is not stored).
    __device__ __forceinline__ void init(int tid, int64_t ld, int rem_r)
    {
        static_for<ITERS>([&](auto it) {
            const int G = it * NT + tid, k = k_of(G);
            int r = r_of(G);
            if (KC) r = r < rem_r ? r : rem_r - 1;
            off[it] = KC ? r * ld + k : k * ld + r;
        });
    }
    // base: the tile's first element of this stage.  All 16 bytes of every granule exist.
    __device__ __forceinline__ void fetch(const T* base, u32x4 (&v)[ITERS]) const
    {
        static_for<ITERS>([&](auto it) {
            if constexpr (sizeof(T) == 4) v[it] = ((const Granule4*)(base + off[it]))->v;
            else v[it] = ((const Granule2*)(base + off[it]))->v;
        });
    }
    // The same where granules may be cut off (fewer columns than the tile along the contiguous index,
    // or a panel shorter than a stage): elements past rem_r and rem_k read as zero.
    __device__ __forceinline__ void fetch_small(const T* base, u32x4 (&v)[ITERS], int tid, int rem_r, int rem_k) const
    {
        static_for<ITERS>([&](auto it) {
            const int G = it * NT + tid, r = r_of(G), k = k_of(G);
            static_for<4>([&](auto w) {
                uint32_t word = 0;
                if constexpr (sizeof(T) == 4) {
                    if ((KC || r + w < rem_r) && (KC ? k + w : k) < rem_k) word = ((const uint32_t*)(base + off[it]))[w];
                } else {
                    static_for<2>([&](auto h) {
                        constexpr int e = 2 * w + h;
                        if ((KC || r + e < rem_r) && (KC ? k + e : k) < rem_k)
                            word |= (uint32_t)((const uint16_t*)(base + off[it]))[e] << (16 * h);
                    });
                }
                v[it][w()] = word;
            });
        });
    }
    // kskip > 0: the first kskip contracted elements of the stage are zeroed
    __device__ __forceinline__ void commit(char* tile, u32x4 (&v)[ITERS], int tid, int kskip) const
    {
        if (kskip > 0) {
            static_for<ITERS>([&](auto it) {
                const int k = k_of(it * NT + tid);
                static_for<4>([&](auto w) {
                    if constexpr (!KC) {
                        if (k < kskip) v[it][w()] = 0;
                    } else if constexpr (sizeof(T) == 4) {
                        if (k + w < kskip) v[it][w()] = 0;
                    } else {
                        if (k + 2 * w < kskip) v[it][w()] &= 0xffff0000u;
                        if (k + 2 * w + 1 < kskip) v[it][w()] = 0;
                    }
                });
            });
        }
        static_for<ITERS>([&](auto it) {
            const int G = it * NT + tid, r = r_of(G), k = k_of(G);
            *(u32x4*)(tile + (KC ? r * LD + k : k * LD + r) * (int)sizeof(T)) = v[it];
        });
    }
};

// Fragment of 32 rows by KG contracted elements.  fp32: lane l holds row l % 32 at k = 4 (l / 32)
// .. + 3, and MFMA e of the four takes element e of every lane; both operands agree on that order.
template <typename T, int R, int BK, bool KC, typename L>
__device__ __forceinline__ auto any_frag(const char* tile, int row0, int k0, int lane)
{
    constexpr int S = L::LD * (int)sizeof(T);
    if constexpr (sizeof(T) == 4) {
        const int r = row0 + (lane & 31), k = k0 + 4 * (lane >> 5);
        if constexpr (KC) {
            return *(const floatx4*)(tile + r * S + k * 4);
        } else {
            floatx4 v;
            static_for<4>([&](auto e) { v[e()] = *(const float*)(tile + (k + e) * S + r * 4); });
            return v;
        }
    } else if constexpr (KC) {
        return *(const bf16x8*)(tile + (row0 + (lane & 31)) * S + (k0 + 8 * (lane >> 5)) * 2);
    } else {
        const int s = lane & 15, bl = lane >> 4;
        const char* p = tile + (k0 + 8 * (bl >> 1) + (s >> 2)) * S + (row0 + 16 * (bl & 1) + 4 * (s & 3)) * 2;
        bf16x4 lo = __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(short4v))(p)));
        bf16x4 hi = __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(short4v))(p + 4 * S)));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
}

// WGM x WGN wavefronts tile the BM x BN output tile; WGK such groups share the contracted elements
// of every stage and are summed in ascending order at the end (small outputs: the chain of one
// wavefront and the number of stages get shorter, and nothing leaves the compute unit).
template <typename T, int BM, int BN, int BK, int WGM, int WGN, int WGK, bool A_KC, bool B_KC>
__global__ __launch_bounds__(64 * WGM * WGN * WGK) void tess_any_kernel(GemmArgs g)
{
    constexpr int NT = 64 * WGM * WGN * WGK, KG = AnyType<T>::KG;
    constexpr int FM = BM / WGM / 32, FN = BN / WGN / 32;
    constexpr int KSTEPS = BK / KG / WGK;              // fragment reads of a group per stage
    typedef AnyLoader<T, BM, BK, A_KC, NT> LA;
    typedef AnyLoader<T, BN, BK, B_KC, NT> LB;
    constexpr int STAGE_BYTES = LA::BYTES + LB::BYTES;
    constexpr int RED_BYTES = WGK > 1 ? WGK * BM * BN * 4 : 0;
    constexpr int CS_BYTES = NT * 4;                   // column sums, at the end
    constexpr int LDS_BYTES = 2 * STAGE_BYTES > RED_BYTES + CS_BYTES ? 2 * STAGE_BYTES : RED_BYTES + CS_BYTES;
    static_assert(KSTEPS >= 1 && NT % BN == 0, "");
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wk = wave / (WGM * WGN), wm = wave / WGN % WGM, wn = wave % WGN;
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    int tm, tn;
    tile_of_block(blockIdx.x, tiles_m, tiles_n, tm, tn);
    // first row and column this tile stores, and where its operands start
    const int row_lo = tm * BM, col_lo = tn * BN;
    const int row0 = g.M - row_lo >= BM ? row_lo : (g.M >= BM ? g.M - BM : 0);
    const int col0 = g.N - col_lo >= BN ? col_lo : (g.N >= BN ? g.N - BN : 0);
    const bool small = g.Kp < BK || (!A_KC && g.M < BM) || (!B_KC && g.N < BN);
    const int kt_per_panel = (g.Kp + BK - 1) / BK;
    const int nkt = g.q * kt_per_panel;
    typedef __attribute__((address_space(4))) const GemmArgs* KernArgs;
    const KernArgs ka = (KernArgs)__builtin_amdgcn_kernarg_segment_ptr();

    LA la;
    LB lb;
    la.init(tid, g.lda, g.M - row0);
    lb.init(tid, g.ldb, g.N - col0);
    floatx16 acc[FM * FN];
    static_for<FM * FN>([&](auto f) { static_for<16>([&](auto r) { acc[f][r()] = 0.0f; }); });
    // column sums of B (the first tile row): NT / BN threads per column, each takes the k that it
    // reaches in steps of NT / BN
    const bool cs_block = g.colsum && tm == 0;
    float cs = 0.0f;

    u32x4 va[2][LA::ITERS], vb[2][LB::ITERS];
    int kskip[2] = {0, 0};
    int ld_t = 0, ld_ks = 0;
    // next stage of the K loop into register set `p`; past the end the last stage is read again
    auto fetch = [&](auto p, auto cut) {
        const T* pa = (const T*)ka->a[ld_t];
        const T* pb = (const T*)ka->b[ld_t];
        const int k0 = ld_ks * BK, over = k0 + BK - g.Kp;
        kskip[p] = over > 0 && g.Kp >= BK ? over : 0;
        const int k = k0 - kskip[p];
        pa += A_KC ? row0 * g.lda + k : k * g.lda + row0;
        pb += B_KC ? col0 * g.ldb + k : k * g.ldb + col0;
        if constexpr (cut) {
            la.fetch_small(pa, va[p], tid, g.M - row0, g.Kp - k);
            lb.fetch_small(pb, vb[p], tid, g.N - col0, g.Kp - k);
        } else {
            la.fetch(pa, va[p]);
            lb.fetch(pb, vb[p]);
        }
        if (ld_ks + 1 < kt_per_panel) ++ld_ks;
        else if (ld_t + 1 < g.q) { ld_ks = 0; ++ld_t; }
        __builtin_amdgcn_sched_barrier(0);             // the loads leave before the products of the stage
    };
    auto commit = [&](auto p) {
        char* st = lds + p * STAGE_BYTES;
        la.commit(st, va[p], tid, kskip[p]);
        lb.commit(st + LA::BYTES, vb[p], tid, kskip[p]);
    };
    auto compute = [&](auto p) {
        const char* sa = lds + p * STAGE_BYTES;
        const char* sb = sa + LA::BYTES;
        static_for<KSTEPS>([&](auto kk) {
            const int k0 = (wk * KSTEPS + kk) * KG;
            decltype(any_frag<T, BM, BK, A_KC, LA>(sa, 0, 0, 0)) a[FM];
            decltype(any_frag<T, BN, BK, B_KC, LB>(sb, 0, 0, 0)) b[FN];
            static_for<FM>([&](auto i) { a[i] = any_frag<T, BM, BK, A_KC, LA>(sa, wm * (BM / WGM) + 32 * i, k0, lane); });
            static_for<FN>([&](auto j) { b[j] = any_frag<T, BN, BK, B_KC, LB>(sb, wn * (BN / WGN) + 32 * j, k0, lane); });
            if constexpr (sizeof(T) == 4) {
                static_for<4>([&](auto e) {
                    static_for<FM * FN>([&](auto f) {
                        acc[f] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[f / FN][e()], b[f % FN][e()], acc[f], 0, 0, 0);
                    });
                });
            } else {
                static_for<FM * FN>([&](auto f) {
                    acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[f / FN], b[f % FN], acc[f], 0, 0, 0);
                });
            }
        });
        if constexpr (!A_KC && !B_KC) {
            if (cs_block) {
#pragma unroll 8
                for (int k = tid / BN; k < BK; k += NT / BN)
                    cs += (float)*(const T*)(sb + (k * LB::LD + tid % BN) * (int)sizeof(T));   // k outside the panel are zero
            }
        }
    };
    constexpr std::integral_constant<int, 0> P0{};
    constexpr std::integral_constant<int, 1> P1{};
    // stage r is in LDS buffer r % 2, stage r+1 in flight to register set (r+1) % 2
    auto k_loop = [&](auto cut) {
        fetch(P0, cut);
        fetch(P1, cut);
        commit(P0);
        __syncthreads();
        for (int r = 0; r < nkt; r += 2) {
            fetch(P0, cut);
            compute(P0);
            commit(P1);
            __syncthreads();
            if (r + 1 < nkt) {
                fetch(P1, cut);
                compute(P1);
                commit(P0);
                __syncthreads();
            }
        }
    };
    if (small) k_loop(std::true_type{});
    else k_loop(std::false_type{});

    if constexpr (!A_KC && !B_KC) {
        if (cs_block) {
            float* part = (float*)(lds + RED_BYTES);
            part[tid] = cs;
            __syncthreads();
            const int col = col0 + tid;
            if (tid < BN && col >= col_lo && col < g.N) {
                float sum = part[tid];
                for (int i = 1; i < NT / BN; ++i) sum += part[i * BN + tid];
                g.colsum[col] = g.accumulate ? g.colsum[col] + sum : sum;
            }
        }
    }
    // C output elements of a thread, all of one column: bias, pre-activation copy, activation, its
    // gradient, accumulation, store.  Each part goes over all C before the next begins, so that the
    // loads are in flight together and no store waits for another one.
    auto finish = [&](auto count, int col, auto&& row_of, auto&& value) {
        constexpr int C = decltype(count)::value;
        if (col < col_lo || col >= g.N) return;
        auto inside = [&](auto x) { return row_of(x) >= row_lo && row_of(x) < g.M; };
        float v[C];
        const float bias = g.bias ? load_in(g.bias, col, g.in_f32) : 0.0f;
        static_for<C>([&](auto x) { v[x] = value(x) + bias; });
        auto store = [&](void* dst) {
            if (g.out_f32) {
                static_for<C>([&](auto x) { if (inside(x)) ((float*)dst)[(int64_t)row_of(x) * g.ldo + col] = v[x]; });
            } else {
                static_for<C>([&](auto x) { if (inside(x)) ((__bf16*)dst)[(int64_t)row_of(x) * g.ldo + col] = (__bf16)v[x]; });
            }
        };
        if (g.preact) store(g.preact);
        if (g.act == TESS_ACT_GELU_ERF && !g.out_f32) static_for<C>([&](auto x) { v[x] = gelu_erf_fast(v[x]); });
        else if (g.act == TESS_ACT_GELU_ERF) static_for<C>([&](auto x) { v[x] = gelu_erf_f(v[x]); });
        else if (g.act == TESS_ACT_GELU_TANH) static_for<C>([&](auto x) { v[x] = gelu_tanh_f(v[x]); });
        if (g.zin) {
            float z[C];
            static_for<C>([&](auto x) { z[x] = inside(x) ? load_in(g.zin, (int64_t)row_of(x) * g.ldz + col, g.in_f32) : 0.0f; });
            if (g.dact == TESS_ACT_GELU_ERF) static_for<C>([&](auto x) { v[x] *= gelu_erf_grad_f(z[x]); });
            else static_for<C>([&](auto x) { v[x] *= gelu_tanh_grad_f(z[x]); });
        }
        if (g.accumulate) {
            float old[C];
            static_for<C>([&](auto x) { old[x] = inside(x) ? ((const float*)g.out)[(int64_t)row_of(x) * g.ldo + col] : 0.0f; });
            static_for<C>([&](auto x) { v[x] = old[x] + v[x]; });
        }
        store(g.out);
    };
    if constexpr (WGK == 1) {
        static_for<FM * FN>([&](auto f) {
            const int fr = row0 + wm * (BM / WGM) + 32 * (f / FN) + 4 * (lane >> 5);
            finish(std::integral_constant<int, 16>{}, col0 + wn * (BN / WGN) + 32 * (f % FN) + (lane & 31),
                   [&](auto x) { return fr + 8 * (x / 4) + x % 4; }, [&](auto x) { return acc[f][x()]; });
        });
    } else {
        float* red = (float*)lds;                      // [WGK][BM][BN]
        static_for<FM * FN>([&](auto f) {
            const int fr = wm * (BM / WGM) + 32 * (f / FN) + 4 * (lane >> 5);
            const int fc = wn * (BN / WGN) + 32 * (f % FN) + (lane & 31);
            static_for<16>([&](auto x) { red[(wk * BM + fr + 8 * (x / 4) + x % 4) * BN + fc] = acc[f][x()]; });
        });
        __syncthreads();
        constexpr int C = BM * BN / NT;
        static_assert(C >= 1 && NT % BN == 0, "a thread's outputs share a column");
        finish(std::integral_constant<int, C>{}, col0 + tid % BN, [&](auto x) { return row0 + (x * NT + tid) / BN; },
               [&](auto x) {
                   float sum = red[x * NT + tid];
                   static_for<WGK - 1>([&](auto w) { sum += red[(w + 1) * BM * BN + x * NT + tid]; });
                   return sum;
               });
    }
}

template <typename T, int BM, int BN, int BK, int WGM, int WGN, int WGK>
static hipError_t launch_any_tile(const GemmArgs& g, hipStream_t s)
{
    const int64_t tiles = (int64_t)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
    const dim3 grid((unsigned)tiles), block(64 * WGM * WGN * WGK);
    if (g.a_kc && g.b_kc) hipLaunchKernelGGL((tess_any_kernel<T, BM, BN, BK, WGM, WGN, WGK, true, true>), grid, block, 0, s, g);
    else if (g.a_kc) hipLaunchKernelGGL((tess_any_kernel<T, BM, BN, BK, WGM, WGN, WGK, true, false>), grid, block, 0, s, g);
    else if (!g.b_kc) hipLaunchKernelGGL((tess_any_kernel<T, BM, BN, BK, WGM, WGN, WGK, false, false>), grid, block, 0, s, g);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace tess
