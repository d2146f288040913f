// One layer of the recursion X <- a X^2 + b X + c I, A <- A + d X (Eq. mlsp2) for a symmetric X
// held as X = hi + lo / s with 16-bit hi/lo (Sec. V.A, Eq. emulated matmul), on CDNA4 MFMA.
//
// Design (gfx950):
//  * Only tiles (I, J) with I <= J are computed (X^2 is symmetric); the epilogue writes the tile
//    and its mirror, so every stored matrix stays exactly symmetric.
//  * X^2 is accumulated in FP32 from three products per K step in one accumulator,
//        s X^2 ~ (s hi_I) hi_J + hi_I lo_J + lo_I hi_J,
//    the lo*lo term being below 2^-22 relative for FP16. By symmetry the B operand of tile
//    (I, J) is the row panel J, so both operands are row panels with K contiguous.
//  * The epilogue is fused (see split_common.h): Y goes through LDS, one row-major pass applies
//    a Y + b X + c delta_ij, updates A and writes the next hi/lo (and, in the direct form, the FP32
//    master X); a transposed pass writes the mirror tile. The last layer writes D and FP64
//    traces. In the squared-affine form (FE_FORM=affine) the operand is the shifted state
//    x + b/(2a), so b = 0 and X is neither read nor written.
//  * Three schedules:
//      data-parallel: one workgroup per upper tile: 64 x 64 or 128 x 128 tiles with direct-to-LDS
//        operand loads where all tiles run at once (split_ring_tile), else 128 x 128 (four
//        64 x 64 wave tiles, register-staged);
//      stream-K over 128 x 128 tiles, two persistent workgroups per CU: the (tile, K-block) iterations
//        left after the whole-tile rounds are split evenly. A workgroup that stops inside a tile
//        publishes its FP32 partial; the workgroup that finishes the tile adds the earlier
//        workgroups' partials in a fixed order in its epilogue (accumulators stay in registers).
//        Where all tiles run at once, a workgroup per tile on the direct-to-LDS ring sums the same
//        segments instead (k_layer_ring_segments);
//      stream-K over 256 x 256 tiles (eight 128 x 64 wave tiles, two LDS stages filled by
//        direct global-to-LDS loads, fragment reads interleaved with the MFMAs), one
//        workgroup per CU: the same; its K loop holds no prefetch registers, so the 128
//        accumulators per lane also stay in registers through the wait and the epilogue.
//    A workgroup only ever waits for workgroups with smaller ids, which were dispatched earlier,
//    and every wait is bounded.
#include "resident.h"
#include "split_common.h"
#include "streamk_plan.h"

namespace fe {
namespace {

using namespace split;

using CfgDP = Cfg<128, 2, 2, 64, 128, 1>;
using CfgSK = Cfg<256, 2, 4, 32, 128, 2, 1>;   // direct-to-LDS operand staging
using CfgSK2 = Cfg<128, 2, 2, 64, 128, 1>;   // stream-K over 128 x 128 tiles, two workgroups per CU
// Three-part BF16 split: six panels of 32-deep K-blocks in one LDS stage (61 KiB), so two
// workgroups still fit per CU; data-parallel only.
using CfgDP3 = Cfg<128, 2, 2, 32, 128, 1, 0, 3>;
// One-round layers (k_layer_ring): 64 x 64 tiles of four 32 x 32 waves, two workgroups per CU, or one
// per CU with a deeper ring (lone tiles); 128 x 128 tiles of eight 32 x 64 waves, one workgroup per CU.
// 64-deep K-blocks: a panel row is one 128-byte line (32-deep blocks fetch every line twice: 4-8%
// slower); two workgroups of the three-part split's six panels only have room for 32-deep ones.
// Lone tiles wait for their loads with nothing beside them: us per density matrix (26 layers) with two
// stages / three, n = 449 267 / 249, 700 340 / 299, 1001 420 / 356, 1408 565 / 468 (four: 245, 311, 350,
// 478); three parts, 32-deep / 64-deep blocks, 700 373 / 362, 1001 484 / 414, 1400 743 / 627.
using CfgR64 = Cfg<64, 2, 2, 64, 64, 2, 1>;
using CfgR64x3 = Cfg<64, 2, 2, 32, 64, 3, 1, 3>;
using CfgL64 = Cfg<64, 2, 2, 64, 64, 3, 1>;
using CfgL64x3 = Cfg<64, 2, 2, 64, 64, 3, 1, 3>;
using CfgR128 = Cfg<128, 4, 2, 64, 128, 2, 1>;
using CfgR128x3 = Cfg<128, 4, 2, 32, 128, 3, 1, 3>;
static_assert(2 * CfgR64::LDS_BYTES <= 160 * 1024 && 2 * CfgR64x3::LDS_BYTES <= 160 * 1024, "two per CU");
// All layers in one launch (k_layer_resident): two stages hold the few blocks of a panel (n = 256 157 us
// with two, 174 with three; three parts 188 against 195 with three 32-deep ones, n = 448 272 / 308).
using CfgS64 = CfgR64;
using CfgS64x3 = Cfg<64, 2, 2, 64, 64, 2, 1, 3>;

template <bool BF, class C>
__global__ void __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_layer_dp(LayerArgs p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int T = (int)(p.np / C::BM);
    const int t = xcd_tile(blockIdx.x, gridDim.x);   // tiles [0, gridDim.x)
    int I, J;
    tile_coords(t, T, I, J);
    Acc<C> acc;
    zero(acc);
    if constexpr (C::NS == 3)
        kloop3<C>(p.hi_in, p.mid_in, p.lo_in, p.np, (int64_t)I * C::BM, (int64_t)J * C::BM, 0,
                  (int)(p.np / C::BK), acc, reinterpret_cast<uint16_t*>(smem));
    else
        kloop<BF, C>(p.hi_in, p.lo_in, p.np, (int64_t)I * C::BM, (int64_t)J * C::BM, 0,
                     (int)(p.np / C::BK), acc, reinterpret_cast<uint16_t*>(smem));
    epilogue<BF, C>(p, acc, reinterpret_cast<float*>(smem), I, J, t);
}

// Data-parallel layer whose upper tiles all run at once: one workgroup per tile, operands straight to
// LDS through the ring of stages (kloop_dma), and (64 x 64 tiles) the epilogue's X and A groups
// loaded before the K loop. Bound by latency rather than by the MFMA rate: at n = 1001 a layer takes
// 18 us, of which 2.2 are the launch, 4.3 the epilogue and 9.5 the K loop (its 64 K steps of MFMAs
// alone 4.5, its loads alone 4.8: the LDS port carries both). An element is one chain over K, in the
// order of k_layer_dp; the sizes that run stream-K sum its segments in k_layer_ring_segments (one chain
// of 2048 gave 1.45 times their error against FP64).
template <bool BF, class C, int AUX>
__device__ __attribute__((always_inline)) inline void ring_products(const LayerArgs& p, int I, int J,
                                                                    int kb0, int kb1, Acc<C>& acc,
                                                                    unsigned char* smem) {
    kloop_dma<BF, C, AUX>(p.hi_in, p.mid_in, p.lo_in, p.np, (int64_t)I * C::BM, (int64_t)J * C::BM,
                          kb0, kb1, acc, reinterpret_cast<uint16_t*>(smem));
}

template <bool BF, class C, int AUX>
__device__ __attribute__((always_inline)) inline void ring_epilogue(const LayerArgs& p, const Acc<C>& acc,
                                                                    int t, int I, int J,
                                                                    unsigned char* smem, bool poisoned,
                                                                    const EpiPre<C>& pre) {
    constexpr bool kPre = EpiPre<C>::PER <= 4;
    float* const sY = reinterpret_cast<float*>(smem);
    if (!p.last && !p.affine) {
        epilogue_mid<BF, C, AUX>(p, acc, sY, I, J, poisoned, kPre ? &pre : nullptr);
        return;
    }
    epilogue<BF, C, kPre ? 8 : 2, kPre>(p, acc, sY, I, J, t, nullptr, 0, 0, poisoned, &pre);
}

template <bool BF, class C, int AUX>
__device__ __attribute__((always_inline)) inline void ring_tile(const LayerArgs& p, int t,
                                                                unsigned char* smem, bool poisoned) {
    int I, J;
    tile_coords(t, (int)(p.np / C::BM), I, J);
    EpiPre<C> pre;
    if constexpr (EpiPre<C>::PER <= 4) pre.template load<AUX>(p, I, J);
    Acc<C> acc;
    zero(acc);
    ring_products<BF, C, AUX>(p, I, J, 0, (int)(p.np / C::BK), acc, smem);
    ring_epilogue<BF, C, AUX>(p, acc, t, I, J, smem, poisoned, pre);
}

template <bool BF, class C>
__global__ void __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_layer_ring(LayerArgs p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    ring_tile<BF, C, 0>(p, xcd_tile(blockIdx.x, gridDim.x), smem, false);
}

// A stream-K layer whose tiles all run at once (sk: the plan of launch_sk): a workgroup per tile sums the
// segments that the plan's workgroups would have handed to each other, in the order of their epilogue
// (sk_tile_segments), so the values are the plan's and nothing is published or
// waited for. us per density matrix (26 layers), stream-K / this: n = 2048 1874 / 1218, 2500 2399 / 1771,
// 2816 2629 / 1967 (one chain per element: 1086, 1640, 1895, and 1.3 times the error). With 64-bit divisions
// in the walk 2048 took 1245.
template <bool BF, class C>
__global__ void __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_layer_ring_segments(LayerArgs p, SplitPlan sk) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    SkGeometry G;
    G.T = (int)(p.np / C::BM);
    G.ntiles = gridDim.x;
    G.nk = (int)(p.np / C::BK);
    G.dp_tiles = 0;
    G.groups = sk.groups;
    G.grid = sk.grid;
    const int t = xcd_tile(blockIdx.x, G.ntiles);
    int I, J;
    tile_coords(t, G.T, I, J);
    EpiPre<C> pre;
    if constexpr (EpiPre<C>::PER <= 4) pre.template load<0>(p, I, J);
    Acc<C> sum;
    sk_tile_segments<uint32_t>(G, t, [&](int i, int kb0, int kb1) {
        Acc<C> acc;
        zero(acc);
        ring_products<BF, C, 0>(p, I, J, kb0, kb1, acc, smem);
#pragma unroll
        for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < C::NB; ++nb)
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    sum.v[mb][nb][j] = i == 0 ? acc.v[mb][nb][j] : sum.v[mb][nb][j] + acc.v[mb][nb][j];
    });
    ring_epilogue<BF, C, 0>(p, sum, t, I, J, smem, false, pre);
}

// All layers of a small matrix in one launch (resident.h), by the same tile code. us per density matrix
// (26 layers, with ~17 for the prologue's launches) against a launch per layer: n = 64 120 / 158,
// 256 157 / 189, 384 202 / 228; with more tiles than the XCD has CUs two workgroups share one and
// the gain is gone (n = 512, 36 tiles: 294 / 269).
template <bool BF, class C>
__global__ void __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_layer_resident(LayerArgs base, ResidentSplit T, ResidentArgs R) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    resident_items(R, [&](int layer, int tile, bool gave_up) {
        LayerArgs p = base;
        const int in = layer & 1;
        p.hi_in = T.hi[in];
        p.lo_in = T.lo[in];
        p.mid_in = T.mid[in];
        p.hi_out = T.hi[in ^ 1];
        p.lo_out = T.lo[in ^ 1];
        p.mid_out = T.mid[in ^ 1];
        const ResidentSplit::Coef& c = T.c[layer];
        p.a = c.a;
        p.b = c.b;
        p.c = c.c;
        p.d_old = c.d_old;
        p.d_new = c.d_new;
        p.last = layer == R.L - 1;
        ring_tile<BF, C, kCoherentLoad>(p, tile, smem, gave_up);
    });
}

// Thread 0 waits until the workgroups of group g with indices jlo .. j-1 have published their
// partials of the current tile (each publishes exactly once: a group never has more workgroups
// than iterations, so every range is non-empty). Their ids g + NG jlo, ..., w - NG are all smaller
// than w. Bounded: a wait that gives up sets *err and returns true for the whole workgroup (the
// caller's epilogue then writes NaN for the whole tile, so that no plausible value is built from
// partials that may belong to an earlier layer). Ends with a barrier.
__device__ inline bool wait_published(const SplitPlan& sk, int g, int NG, int jlo, int w) {
    __shared__ int gave_up_all;
    if (threadIdx.x == 0) {
        bool gave_up = false;
        for (int wp = g + NG * jlo; wp < w && !gave_up; wp += NG) {
            int spins = 0;
            while (__hip_atomic_load(sk.flags + wp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) !=
                   sk.wait_epoch) {
                if (++spins > sk.spin_limit) {
                    atomicOr(sk.err, 1);
                    gave_up = true;
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
            }
        }
        gave_up_all = gave_up ? 1 : 0;
    }
    // The partials are read after this barrier, i.e. after the flags were seen, with
    // device-coherent loads.
    __syncthreads();
    return gave_up_all != 0;
}

template <bool BF, class C>
__global__ void __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_layer_sk(LayerArgs p, SplitPlan sk) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // Accumulators stay in registers through the wait when the K loop leaves room for them
    // (small tiles, or the direct-to-LDS loop, which holds no prefetch registers); otherwise
    // (128 per lane next to a register-prefetch loop) they are staged to memory after the K loop.
    constexpr bool kRegEpi = C::MB * C::NB <= 4 || C::DMA;
    const int tid = threadIdx.x;
    const int w = blockIdx.x;
    const int T = (int)(p.np / C::BM);
    const int ntiles = T * (T + 1) / 2;
    const int nk = (int)(p.np / C::BK);
    constexpr size_t TILE = (size_t)C::BM * C::BM;
    float* own = sk.own + (size_t)w * TILE;
    float* pub = sk.partial + (size_t)w * TILE;
    float* sY = reinterpret_cast<float*>(smem);

    // Tiles [0, dp_tiles) were computed whole by a data-parallel launch before this one; the
    // walk over the rest is in streamk_plan.h (shared with the host-side plan checks).
    SkGeometry G;
    G.T = T;
    G.ntiles = ntiles;
    G.nk = nk;
    G.dp_tiles = sk.dp_tiles;
    G.groups = sk.groups;
    G.grid = sk.grid;
    const int NG = sk.groups, g = w % NG, j = w / NG;
    sk_walk(G, w, [&](int pass, int t, int kb0, int kb1, int jlo) {
        int I, J;
        tile_coords(t, T, I, J);
        // Earlier workgroups of the group with indices jlo .. j-1 hold the first kb0 blocks of
        // this tile; their partial slots are NG tiles apart. The epilogue adds them in a fixed
        // order, so the result does not depend on timing.
        const float* parts = sk.partial + (size_t)(g + NG * jlo) * TILE;
        Acc<C> acc;
        zero(acc);
        kloop<BF, C>(p.hi_in, p.lo_in, p.np, (int64_t)I * C::BM, (int64_t)J * C::BM, kb0, kb1, acc,
                     reinterpret_cast<uint16_t*>(smem));
        if (pass == 0) {
            // Publication: every wave waits until its device-coherent stores of the partial
            // have completed, then one flag store (device-coherent too) announces the tile.
            // No release fence: on this chip it writes back the whole L2, and the readers'
            // acquire would invalidate it; the partial needs neither (see store_coherent).
            store_tile<BF, C, true>(acc, pub);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (tid == 0)
                __hip_atomic_store(sk.flags + w, sk.epoch, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        } else if constexpr (kRegEpi) {
            const bool gave_up = wait_published(sk, g, NG, jlo, w);
            epilogue<BF, C, 1>(p, acc, sY, I, J, t, parts, (size_t)NG * TILE, j - jlo, gave_up);
        } else {
            store_tile<BF, C, false>(acc, own);
            const bool gave_up = wait_published(sk, g, NG, jlo, w);
            epilogue_mem<BF, C, 1>(p, own, parts, (size_t)NG * TILE, j - jlo, sY, I, J, t,
                                   gave_up);
        }
    });
}

template <class K>
hipError_t set_lds(K kern, size_t bytes, bool& done) {
    if (done) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) done = true;
    return e;
}

template <bool BF, class C = CfgDP>
hipError_t launch_dp(const LayerArgs& a, hipStream_t s) {
    auto kern = k_layer_dp<BF, C>;
    static bool done = false;
    hipError_t e = set_lds(kern, C::LDS_BYTES, done);
    if (e != hipSuccess) return e;
    const int T = (int)(a.np / C::BM);
    hipLaunchKernelGGL(kern, dim3(T * (T + 1) / 2), dim3(C::NT), C::LDS_BYTES, s, a);
    return hipGetLastError();
}

template <bool BF, class C>
hipError_t launch_ring(const LayerArgs& a, hipStream_t s) {
    auto kern = k_layer_ring<BF, C>;
    static bool done = false;
    hipError_t e = set_lds(kern, C::LDS_BYTES, done);
    if (e != hipSuccess) return e;
    const int T = (int)(a.np / C::BM);
    hipLaunchKernelGGL(kern, dim3(T * (T + 1) / 2), dim3(C::NT), C::LDS_BYTES, s, a);
    return hipGetLastError();
}

template <bool BF, class C>
hipError_t launch_resident(const LayerArgs& a, const ResidentSplit& T, const ResidentArgs& R,
                           hipStream_t s) {
    auto kern = k_layer_resident<BF, C>;
    static bool done = false;
    hipError_t e = set_lds(kern, C::LDS_BYTES, done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(8 * R.ntiles), dim3(C::NT), C::LDS_BYTES, s, a, T, R);
    return hipGetLastError();
}

template <bool BF, class C>
hipError_t launch_sk(const LayerArgs& a, const SplitPlan& sk, hipStream_t s) {
    auto kern = k_layer_sk<BF, C>;
    static bool done = false;
    hipError_t e = set_lds(kern, C::LDS_BYTES, done);
    if (e != hipSuccess) return e;
    // One workgroup per CU, but never more workgroups per group than the group's (tile,
    // K-block) iterations: then every range is non-empty and each tile's earlier contributors
    // all publish (sk_plan). Configurations that stage their accumulators through memory run
    // stream-K alone; the others run all but the last full round of tiles as whole tiles in a
    // data-parallel launch first (their K walks stay in step, which the L2 rewards).
    constexpr bool reg_epi = C::MB * C::NB <= 4;
    const SkGeometry G = sk_plan(a.np, C::BM, C::BK, sk.grid, reg_epi);
    SplitPlan plan = sk;
    plan.grid = G.grid;
    plan.groups = G.groups;
    plan.dp_tiles = G.dp_tiles;
    if (plan.grid < 1) return hipErrorInvalidValue;
    if constexpr (C::BM == CfgR128::BM) {
        if (!plan.hand_over && G.dp_tiles == 0 && G.ntiles <= plan.n_cu && sk_fits_32(G)) {
            auto rkern = k_layer_ring_segments<BF, CfgR128>;
            static bool rdone = false;
            e = set_lds(rkern, CfgR128::LDS_BYTES, rdone);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(rkern, dim3(G.ntiles), dim3(CfgR128::NT), CfgR128::LDS_BYTES, s, a, plan);
            return hipGetLastError();
        }
    }
    if constexpr (reg_epi) {
        if (plan.dp_tiles > 0) {
            auto dkern = k_layer_dp<BF, C>;
            static bool ddone = false;
            e = set_lds(dkern, C::LDS_BYTES, ddone);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(dkern, dim3(plan.dp_tiles), dim3(C::NT), C::LDS_BYTES, s, a);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    hipLaunchKernelGGL(kern, dim3(plan.grid), dim3(C::NT), C::LDS_BYTES, s, a, plan);
    return hipGetLastError();
}

}  // namespace

// Where the lines lie (ms per density matrix, 26 layers, random dense; 256 CUs): two 64 x 64 tiles
// fit a CU, so up to 512 of them run at once (n <= 1984; two parts take stream-K's segments from
// n = 1921): n = 1001 0.48 against 1.15 with 128 x 128 register-staged tiles (0.36 since). At n = 2048,
// 528 tiles need a second round for 16 of them: 1.58 against 1.09 for the 128 x 128 ring, which takes
// one round up to n = 2816 (1.90 against 2.63 for stream-K); at n = 2900 a second round makes it
// 3.61 on the ring and 3.32 register-staged against 2.98.
int split_ring_tile(int64_t n, int n_cu) {
    auto tiles = [n](int64_t bm) {
        const int64_t T = (n + bm - 1) / bm;
        return T * (T + 1) / 2;
    };
    if (tiles(CfgR64::BM) <= 2 * (int64_t)n_cu) return CfgR64::BM;
    if (tiles(CfgR128::BM) <= n_cu) return CfgR128::BM;
    return 0;
}

bool split_resident(int64_t n, int n_cu) {
    const int64_t T = (n + CfgR64::BM - 1) / CfgR64::BM;
    return 8 * (T * (T + 1) / 2) <= n_cu;
}

// Stream-K over 128 x 128 tiles when each of its workgroups (two per CU) gets at least eight K-blocks;
// with fewer the partial-tile traffic outweighs the balance. From eight whole rounds on (n >= 11521) the
// uneven last one costs less than the partial tiles: ms per density matrix, stream-K / data-parallel,
// dense 12000 150 / 146, banded 12000 201 / 182, 16384 463 / 441 (10000, six rounds: 106 / 111). Only the
// last two rounds were summed in segments; |dD|_F against an FP64 recursion, data-parallel over stream-K:
// dense 11600 1.001, 12800 1.000, 16384 1.000, banded 11600 and 16384 1.000, BF16x2 dense 12000 1.001. Not
// taken, though faster: 128 x 128 ring tiles in segments of 512 products (4096 6.56 / 5.95) and 256 x 256
// tiles (5500 17.8 / 12.9): their sums round otherwise, and on dense matrices at beta' ~ 100, where one
// rounding more or less shows as 1e-4 of D, the values moved by that.
int split_schedule(int64_t n, int n_cu) {
    const int64_t np = (n + 127) / 128 * 128, T = np / 128, tiles = T * (T + 1) / 2, nk = np / 64;
    const int64_t grid = 2 * (int64_t)n_cu, rounds = tiles / grid;
    if (rounds >= 8) return 0;
    const int64_t nsk = rounds >= 2 ? tiles - (rounds - 1) * grid : tiles;
    return nsk * nk >= 8 * grid ? 2 : 0;
}

int split_tile_for(int streamk) {
    static_assert(CfgDP3::BM == CfgDP::BM, "the three-part split runs the data-parallel tile");
    return streamk == 1 ? CfgSK::BM : streamk == 2 ? CfgSK2::BM : CfgDP::BM;
}

SkGeometry split_sk_geometry(int64_t np, int streamk, int grid) {
    if (streamk == 1) return sk_plan(np, CfgSK::BM, CfgSK::BK, grid, CfgSK::MB * CfgSK::NB <= 4);
    return sk_plan(np, CfgSK2::BM, CfgSK2::BK, grid, CfgSK2::MB * CfgSK2::NB <= 4);
}

hipError_t launch_layers_resident(const LayerArgs& a, int bf16, const ResidentSplit& T,
                                  ResidentArgs R, hipStream_t s) {
    const int T_ = (int)(a.np / CfgR64::BM);
    if (a.np % CfgR64::BM != 0 || R.L < 1 || R.L > kResMaxL || !R.ctl || a.affine)
        return hipErrorInvalidValue;
    R.ntiles = T_ * (T_ + 1) / 2;
    return bf16 == 2 ? launch_resident<true, CfgS64x3>(a, T, R, s)
           : bf16    ? launch_resident<true, CfgS64>(a, T, R, s)
                     : launch_resident<false, CfgS64>(a, T, R, s);
}

hipError_t launch_layer_split(const LayerArgs& a, int bf16, const SplitPlan& plan, hipStream_t s) {
    if (plan.streamk == 0 && plan.ring_tile != 0) {
        if (a.np % plan.ring_tile != 0) return hipErrorInvalidValue;
        const int64_t T = a.np / plan.ring_tile;
        if (plan.ring_tile == CfgL64::BM && T * (T + 1) / 2 <= plan.n_cu)   // at most one per CU
            return bf16 == 2 ? launch_ring<true, CfgL64x3>(a, s)
                   : bf16    ? launch_ring<true, CfgL64>(a, s)
                             : launch_ring<false, CfgL64>(a, s);
        if (plan.ring_tile == CfgR64::BM)
            return bf16 == 2 ? launch_ring<true, CfgR64x3>(a, s)
                   : bf16    ? launch_ring<true, CfgR64>(a, s)
                             : launch_ring<false, CfgR64>(a, s);
        if (plan.ring_tile == CfgR128::BM)
            return bf16 == 2 ? launch_ring<true, CfgR128x3>(a, s)
                   : bf16    ? launch_ring<true, CfgR128>(a, s)
                             : launch_ring<false, CfgR128>(a, s);
        return hipErrorInvalidValue;
    }
    if (bf16 == 2) {   // three-part BF16 split: data-parallel schedule only
        if (plan.streamk != 0) return hipErrorInvalidValue;
        return launch_dp<true, CfgDP3>(a, s);
    }
    if (plan.streamk == 1)
        return bf16 ? launch_sk<true, CfgSK>(a, plan, s) : launch_sk<false, CfgSK>(a, plan, s);
    if (plan.streamk == 2)
        return bf16 ? launch_sk<true, CfgSK2>(a, plan, s) : launch_sk<false, CfgSK2>(a, plan, s);
    return bf16 ? launch_dp<true>(a, s) : launch_dp<false>(a, s);
}

}  // namespace fe
