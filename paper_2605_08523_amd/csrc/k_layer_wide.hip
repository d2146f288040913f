// FP32 and FP64 layer kernels of the recursion X <- a X^2 + b X + c I, A <- A + d X
// (Eq. mlsp2), and the backward layer of the coefficient trainer.
//
// One workgroup of four waves per BM x BM output tile (BM = 32 or 64; a wave holds 1 or 2 x 2 blocks
// of 16 x 16), v_mfma_f32_16x16x4f32 or v_mfma_f64_16x16x4f64. The operands of tile (I, J) are the
// row panels I and J (X is symmetric, so column panel J = row panel J^T). They go straight from
// global memory to LDS (one 128-byte line of every panel row per K block) through a ring of stages.
// The layer form computes only upper tiles and writes each tile and its mirror through an
// LDS-staged epilogue, whose X and A groups are loaded before the K loop; waves whose block lies in
// the padding or strictly below the diagonal skip the products.
//
// Why 16 x 16 blocks: both types are bound by the MFMA rate, and a layer of ordinary size has few
// blocks per SIMD (n = 1500: 4656 of 16 x 16 on 1024 SIMDs), so the time follows the largest count on
// one SIMD. In FP32 the MFMA adds its products one by one in ascending k (measured: 16x16x4 and
// 32x32x2 chains and a scalar fmaf chain agree bitwise), so the block shape does not change a bit.
// Measured (us per layer; before: 64 x 64 tiles of four 32 x 32 waves, one LDS buffer): FP32 n = 256
// 5.3 (16.7), 1500 37 (81; the MFMA rate alone 23), FP64 n = 256 6.6 (25), 1000 29 (78; 14).
#include <type_traits>

#include "fe_internal.h"
#include "mfma_wide.h"
#include "resident.h"
#include "split_common.h"

namespace fe {
namespace {

using split::wave_sum;
using wide::doublex4;
using wide::floatx4;
using wide::Mfma;

constexpr int kPad = 64;      // padding unit of the matrices (a multiple of every tile)
constexpr int NT = 256;       // 4 waves, 2 x 2

// NPR: products per tile (two operand panels each).
template <typename T, int BM, int NPR = 1>
struct WCfg {
    static constexpr int BK = 128 / (int)sizeof(T);        // one line of every panel row
    static constexpr int NB = BM / 32;                     // 16 x 16 blocks per wave side
    static constexpr int S = 4;                            // ring stages
    static constexpr int PANEL = BM * 128, STAGE = 2 * NPR * PANEL;   // bytes
    static constexpr int IPP = BM / 32;                    // 1-KiB loads per wave, panel and stage
    static constexpr int IPW = 2 * NPR * IPP;              // ... per wave and stage
    static constexpr int LDY = BM + 4;                     // epilogue staging row (elements)
    static constexpr int G = BM / 4, PER = BM * G / NT;    // four-column groups: per row, per thread
    static constexpr size_t EPI = (size_t)BM * LDY * sizeof(double);
    static constexpr size_t LDS = (size_t)S * STAGE > EPI ? (size_t)S * STAGE : EPI;
};

// a y + b x + c with the roundings spelled out: the order the compiler picks for the plain expression
// varies from kernel to kernel, and in FP32 that alone moves a trained gradient by 2.5e-5.
template <typename T>
__device__ inline T layer_value(T a, T y, T b, T x, T c) {
#pragma clang fp contract(off)
    const T bx = b * x;
    return __builtin_elementwise_fma(a, y, bx) + c;
}

// Four elements at the element type's own alignment (the trainer's callers may pass such arrays).
template <typename T>
struct Unaligned;
template <>
struct Unaligned<float> {
    typedef floatx4 vec __attribute__((aligned(4)));
};
template <>
struct Unaligned<double> {
    typedef doublex4 vec __attribute__((aligned(8)));
};

// acc[p] += L_p R_p^T over nk K blocks for NPR products at once, from the BM-row panels at Lp[p] and
// Rp[p] of np-wide matrices: products per element in ascending k. work (the same for all lanes of a
// wave): this wave's blocks are wanted. ALIGNED: the panels start on 16 bytes (rows then do too);
// otherwise the operands go through registers into the same LDS places, element by element. Ends
// with a barrier. AUX: cache policy of the loads.
//
// Ring of stages: chunk c (16 bytes) of panel row r sits at chunk c ^ (r % 8) of its 128-byte LDS row,
// so the rows that a fragment read touches spread over the banks. Nothing in the loop needs vector
// arithmetic (MFMAs do not run beside it: four vector instructions per MFMA took 8 of its 15 ns
// here): a load's address is the lane's fixed offset plus a scalar one, a fragment's LDS address a
// fixed register plus the stage's constant (the stages are unrolled).
template <typename T, int BM, bool ALIGNED, int NPR, int AUX = 0>
__device__ __attribute__((always_inline)) inline void wide_products(
    const T* const (&Lp)[NPR], const T* const (&Rp)[NPR], int64_t np, int nk, bool work,
    unsigned char* smem,
    typename Mfma<T>::vec (&acc)[NPR][WCfg<T, BM>::NB][WCfg<T, BM>::NB]) {
    using M = Mfma<T>;
    using W = WCfg<T, BM, NPR>;
    typedef __attribute__((address_space(3))) void lds_void;
    constexpr int NB = W::NB, S = W::S, BK = W::BK;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t row_bytes = np * (int64_t)sizeof(T);
    const uint32_t lane_off = (uint32_t)((lane >> 3) * row_bytes + (((lane & 7) ^ (lane >> 3)) << 4));
    __amdgpu_buffer_rsrc_t rs[2 * NPR];
#pragma unroll
    for (int p = 0; p < 2 * NPR; ++p)
        rs[p] = split::make_rsrc(p & 1 ? Rp[p >> 1] : Lp[p >> 1], (uint32_t)(BM * row_bytes));
    auto issue = [&](int kb, int stage, int q0, int q1) {
#pragma unroll
        for (int q = q0; q < q1; ++q) {
            const int panel = q / W::IPP, blk = wave + 4 * (q % W::IPP);
            unsigned char* l = smem + stage * W::STAGE + panel * W::PANEL + blk * 1024;
            const uint32_t soff = (uint32_t)(blk * 8 * row_bytes) + (uint32_t)kb * 128;
            if constexpr (ALIGNED) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs[panel], (lds_void*)l, 16, (int)lane_off,
                                                         (int)soff, 0, AUX);
            } else {
                const T* g = reinterpret_cast<const T*>(
                    reinterpret_cast<const char*>(panel & 1 ? Rp[panel >> 1] : Lp[panel >> 1]) + soff +
                    lane_off);
                T v[16 / sizeof(T)];
#pragma unroll
                for (int k = 0; k < (int)(16 / sizeof(T)); ++k) v[k] = g[k];
#pragma unroll
                for (int k = 0; k < (int)(16 / sizeof(T)); ++k)
                    reinterpret_cast<T*>(l + lane * 16)[k] = v[k];
            }
        }
    };
    const int fr = lane & 15, fk = lane >> 4;
    constexpr int KS = BK / 4;
    static_assert(W::IPW <= KS, "a load of the next stage behind each K step");
    constexpr bool kAhead = AUX != 0;   // few blocks (a resident launch): all reads at once
    typedef __attribute__((address_space(3))) const unsigned char lds_char;
    lds_char* const lds0 = (lds_char*)smem;
    uint32_t oa[KS], ob[KS];   // byte offsets of element (row fr, k = 4 s + fk) of this wave's blocks
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        constexpr int PC = 16 / (int)sizeof(T);   // elements per chunk
        const int k = 4 * s + fk;
        const uint32_t o = fr * 128 + (((k / PC) ^ (fr & 7)) << 4) + (k % PC) * (int)sizeof(T);
        oa[s] = o + wm * NB * 2048;
        ob[s] = o + wn * NB * 2048 + W::PANEL;
        asm volatile("" : "+v"(oa[s]), "+v"(ob[s]));   // kept, not recomputed in the loop
    }
    struct Frag {
        T a[NPR][KS][NB], b[NPR][KS][NB];
    };
    auto read = [&](int stage, int s, Frag& f) {
#pragma unroll
        for (int p = 0; p < NPR; ++p)
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                typedef __attribute__((address_space(3))) const T lds_T;
                const int o = stage * W::STAGE + p * 2 * W::PANEL + x * 2048;
                f.a[p][s][x] = *(lds_T*)(lds0 + oa[s] + o);
                f.b[p][s][x] = *(lds_T*)(lds0 + ob[s] + o);
            }
    };
    auto multiply = [&](int s, const Frag& f) {
#pragma unroll
        for (int p = 0; p < NPR; ++p)
#pragma unroll
            for (int x = 0; x < NB; ++x)
#pragma unroll
                for (int y = 0; y < NB; ++y)
                    acc[p][x][y] = M::mma(f.a[p][s][x], f.b[p][s][y], acc[p][x][y]);
    };
    // Block i in stage u. First waits until this wave's loads of block i + 1 have landed (those of the
    // S - 2 blocks after it may be in flight) and its fragment reads of block i are done, and joins
    // the other waves: block i + 1 is whole and block i's stage is free. Then the block's products,
    // each K step's followed by the next block's fragment reads of that step and a load into the free
    // stage: the wave issues them while its MFMAs run. (us per density matrix, all of them ahead of the
    // products / spread: FP32 n = 512 210 / 189, 1000 545 / 491, 1500 1106 / 965, 2000 2168 / 2050;
    // FP64 512 301 / 277, 700 377 / 343, 1000 815 / 777, 1500 1861 / 1762.) full: the blocks up to
    // i + S exist (no conditions).
    auto step = [&](auto wk, auto full, int i, int u, const Frag& cur, Frag& nxt) {
        if (full || i + 1 < nk) {
            if (full || i + S - 1 < nk) __builtin_amdgcn_s_waitcnt(0x0070 | (W::IPW * (S - 2)));
            else __builtin_amdgcn_s_waitcnt(0x0070);   // lgkmcnt(0), vmcnt(loads of later blocks)
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if constexpr (kAhead) {
                if (full || i + S < nk) issue(i + S, u, 0, W::IPW);
                if constexpr (wk)
#pragma unroll
                    for (int s = 0; s < KS; ++s) read((u + 1) % S, s, nxt);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if constexpr (wk) multiply(s, cur);
            if constexpr (!kAhead) {
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (wk)
                    if (full || i + 1 < nk) read((u + 1) % S, s, nxt);
                if (s < W::IPW && (full || i + S < nk)) issue(i + S, u, s, s + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto loop = [&](auto wk) {
        constexpr std::true_type yes{};
        constexpr std::false_type no{};
        Frag f0, f1;
        if constexpr (wk)
#pragma unroll
            for (int s = 0; s < KS; ++s) read(0, s, f0);
        int i = 0;
        for (; i + 2 * S - 1 < nk; i += S) {
            step(wk, yes, i, 0, f0, f1);
            step(wk, yes, i + 1, 1, f1, f0);
            step(wk, yes, i + 2, 2, f0, f1);
            step(wk, yes, i + 3, 3, f1, f0);
        }
        for (; i < nk; i += S) {
            step(wk, no, i, 0, f0, f1);
            if (i + 1 < nk) step(wk, no, i + 1, 1, f1, f0);
            if (i + 2 < nk) step(wk, no, i + 2, 2, f0, f1);
            if (i + 3 < nk) step(wk, no, i + 3, 3, f1, f0);
        }
    };
#pragma unroll
    for (int b = 0; b < S; ++b)
        if (b < nk) issue(b, b, 0, W::IPW);
    static_assert(S == 4 && W::IPW * (S - 1) < 16, "four stages unrolled, four-bit wait count");
    if (S - 1 < nk) __builtin_amdgcn_s_waitcnt(0x0070 | (W::IPW * (S - 1)));
    else __builtin_amdgcn_s_waitcnt(0x0070);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (work) loop(std::true_type{});
    else loop(std::false_type{});
    asm volatile("" ::: "memory");
    __syncthreads();
}

// Upper tile t of one layer. AUX: cache policy of the loads (kCoherentLoad: a matrix of less than
// 4 GiB that other workgroups of this XCD wrote in the same launch). poisoned: outputs are NaN.
template <typename T, int BM, bool ALIGNED, int AUX>
__device__ __attribute__((always_inline)) inline void wide_tile_layer(const WideArgs& p, int t,
                                                                      unsigned char* smem,
                                                                      bool poisoned) {
    using M = Mfma<T>;
    using W = WCfg<T, BM>;
    using vec = typename M::vec;
    using gvec = typename std::conditional<ALIGNED, vec, typename Unaligned<T>::vec>::type;
    constexpr int NB = W::NB;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, fr = lane & 15;
    const int64_t np = p.np, n = p.n;
    const int T_ = (int)(np / BM);
    int I, J;
    split::tile_coords(t, T_, I, J);
    const bool diag = I == J;
    const int64_t I0 = (int64_t)I * BM, J0 = (int64_t)J * BM;
    const T* __restrict__ X = static_cast<const T*>(p.X_in);
    T* __restrict__ A = static_cast<T*>(p.A);
    const bool last = p.last != 0, ent = p.entropy != 0;
    const T dn = (T)p.d_next;
    const bool use_a = last || dn != (T)0;

    // the epilogue's groups (all inside the padded matrices)
    vec xg[W::PER], ag[W::PER];
    auto group = [&](int u) {
        const int e = tid + u * NT;
        return (I0 + e / W::G) * np + J0 + (e % W::G) * 4;
    };
    auto load = [&](const T* m, int u) -> vec {
        if constexpr (AUX == 0) {
            return *reinterpret_cast<const gvec*>(m + group(u));
        } else {
            const __amdgpu_buffer_rsrc_t rs = split::make_rsrc(m, (uint32_t)(np * np * sizeof(T)));
            const int o = (int)(group(u) * sizeof(T));
            split::u32x4 v[sizeof(T) / 4];
#pragma unroll
            for (int q = 0; q < (int)(sizeof(T) / 4); ++q)
                v[q] = __builtin_amdgcn_raw_buffer_load_b128(rs, o + 16 * q, 0, AUX);
            vec r;
            __builtin_memcpy(&r, v, sizeof(r));
            return r;
        }
    };
#pragma unroll
    for (int u = 0; u < W::PER; ++u) xg[u] = load(X, u);
    if (use_a) {
#pragma unroll
        for (int u = 0; u < W::PER; ++u) ag[u] = load(A, u);
    }
    // A block whose rows or columns are all padding, or that lies strictly below the diagonal, is
    // not stored: its wave skips the products. Beyond n both operands are zero.
    const bool work = I0 + wm * NB * 16 < n && J0 + wn * NB * 16 < n && !(diag && wm > wn);
    vec acc[1][NB][NB];
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y) acc[0][x][y] = vec{0, 0, 0, 0};
    const T* const lp[1] = {X + I0 * np};
    const T* const rp[1] = {X + J0 * np};
    wide_products<T, BM, ALIGNED, 1, AUX>(lp, rp, np, (int)((n + W::BK - 1) / W::BK), work, smem, acc);

    // the product tile goes through LDS to four-column groups in registers
    T* sY = reinterpret_cast<T*>(smem);
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                sY[((wm * NB + x) * 16 + M::crow(lane, j)) * W::LDY + (wn * NB + y) * 16 + fr] = acc[0][x][y][j];
    __syncthreads();
    vec yg[W::PER];
#pragma unroll
    for (int u = 0; u < W::PER; ++u) {
        const int e = tid + u * NT;
        yg[u] = *reinterpret_cast<const vec*>(sY + (e / W::G) * W::LDY + (e % W::G) * 4);
    }

    const T ca = poisoned ? (T)__builtin_nan("") : (T)p.a, cb = (T)p.b, cc = (T)p.c;
    if (!last) {
        T* __restrict__ Xo = static_cast<T*>(p.X_out);
#pragma unroll
        for (int u = 0; u < W::PER; ++u) {
            const int e = tid + u * NT, r = e / W::G, c = (e % W::G) * 4;
            const int64_t gr = I0 + r, gc = J0 + c, gi = gr * np + gc;
            vec xn, an;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const T v = layer_value(ca, yg[u][k], cb, xg[u][k], gr == gc + k ? cc : (T)0);
                xn[k] = gr < n && gc + k < n ? v : (T)0;   // the padding stays zero
                if (use_a) an[k] = ag[u][k] + dn * xn[k];
            }
            if (!diag || c >= r) {
                if (use_a) *reinterpret_cast<gvec*>(A + gi) = an;
                *reinterpret_cast<gvec*>(Xo + gi) = xn;
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (c + k < r) continue;
                    if (use_a) A[gi + k] = an[k];
                    Xo[gi + k] = xn[k];
                }
            }
            *reinterpret_cast<vec*>(sY + r * W::LDY + c) = xn;
        }
        __syncthreads();
        // Mirror: output row J0 + c, columns I0 + r .. r + 3 hold x(r .. r + 3, c).
#pragma unroll
        for (int u = 0; u < W::PER; ++u) {
            const int e = tid + u * NT, c = e / W::G, r = (e % W::G) * 4;
            if (diag && r >= c) continue;   // nothing strictly below the diagonal
            vec v;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = sY[(r + k) * W::LDY + c];
            T* o = Xo + (J0 + c) * np + I0 + r;
            if (!diag || r + 3 < c) {
                *reinterpret_cast<gvec*>(o) = v;
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (r + k < c) o[k] = v[k];
            }
        }
        return;
    }

    // Last layer: D = A + X' (I - D if flipped), or U = A + X' traced only (entropy). With f64_epi
    // (T = float) D = A + d_last X + (a y + b X + c delta) in FP64, not rounded.
    const int flip = !ent ? p.P->flipped : 0;
    const bool f64e = p.f64_epi != 0;
    const bool write = !(ent || p.out_mode == 2);
    double* sD = reinterpret_cast<double*>(smem);
    double tr = 0.0, sq = 0.0;
    auto put = [&](int64_t row, int64_t col, double v) {
        if (p.out_mode == 0) reinterpret_cast<float*>(p.D)[row * p.ldd + col] = (float)v;
        else reinterpret_cast<double*>(p.D)[row * p.ldd + col] = v;
    };
    __syncthreads();   // every thread's y is in registers: the staging now holds doubles
#pragma unroll
    for (int u = 0; u < W::PER; ++u) {
        const int e = tid + u * NT, r = e / W::G, c = (e % W::G) * 4;
        const int64_t gr = I0 + r;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t gc = J0 + c + k;
            const T y = yg[u][k], x = xg[u][k], a = ag[u][k];
            double v;
            if (f64e) {
                v = (double)a + p.d_last * (double)x +
                    (p.a * (double)y + p.b * (double)x + (gr == gc ? p.c : 0.0));
            } else {
                const T xn = layer_value(ca, y, cb, x, gr == gc ? cc : (T)0);
                v = (double)a + (double)xn;
            }
            if (flip) v = (gr == gc ? 1.0 : 0.0) - v;
            // FP32 mode carries FP32 values (so the tile and its mirror hold the same number)
            if (!(ent || sizeof(T) == 8 || f64e)) v = (double)(float)v;
            if ((!diag || c + k >= r) && gr < n && gc < n) {
                if (gr == gc) tr += v;
                sq += (gr == gc ? 1.0 : 2.0) * v * v;
                if (write) put(gr, gc, v);
            }
            sD[r * W::LDY + c + k] = v;
        }
    }
    __syncthreads();
    if (write) {
#pragma unroll
        for (int u = 0; u < W::PER; ++u) {
            const int e = tid + u * NT, c = e / W::G, r = (e % W::G) * 4;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (diag && !(r + k < c)) continue;
                if (J0 + c < n && I0 + r + k < n) put(J0 + c, I0 + r + k, sD[(r + k) * W::LDY + c]);
            }
        }
    }
    __syncthreads();
    tr = wave_sum(tr);
    sq = wave_sum(sq);
    if (lane == 0) {
        sD[2 * wave] = tr;
        sD[2 * wave + 1] = sq;
    }
    __syncthreads();
    if (tid == 0) {
        double tt = 0.0, ss = 0.0;
        for (int w = 0; w < 4; ++w) {
            tt += sD[2 * w];
            ss += sD[2 * w + 1];
        }
        p.partials[t].tr = tt;
        p.partials[t].sq = ss;
    }
}

template <typename T, int BM, bool ALIGNED>
__global__ void __launch_bounds__(NT) k_wide(WideArgs p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    wide_tile_layer<T, BM, ALIGNED, 0>(p, split::xcd_tile(blockIdx.x, gridDim.x), smem, false);
}

// All layers of a small matrix in one launch (resident.h), by the same tile code. us per density matrix
// (26 layers) against a launch per layer: FP64 n = 64 97 / 113, 128 117 / 137, 192 145 / 158 and, with
// more tiles than the XCD has CUs, 256 235 / 180; FP32 64 85 / 104, 192 120 / 137, 256 161 / 145.
// (One workgroup with the matrix in its LDS: n = 128 FP64 503.)
template <typename T>
__global__ void __launch_bounds__(NT) k_wide_resident(WideArgs base, ResidentWide L, ResidentArgs R) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    resident_items(R, [&](int layer, int tile, bool gave_up) {
        WideArgs p = base;
        p.X_in = L.X[layer & 1];
        p.X_out = L.X[(layer & 1) ^ 1];
        p.a = L.theta[4 * layer];
        p.b = L.theta[4 * layer + 1];
        p.c = L.theta[4 * layer + 2];
        p.last = layer + 1 == R.L;
        p.d_next = p.last ? 0.0 : L.theta[4 * layer + 7];
        wide_tile_layer<T, 32, true, kCoherentLoad>(p, tile, smem, gave_up);
    });
}

// Backward of one layer of the FP32 matrix recursion in one pass over the upper tiles (I, J): with
// M = Xb X (Xb the adjoint of this layer's output, X its input),
//   Xb_out = a (M + M^T) + b Xb + d G,
// and the tile's FP64 sums of <M, X>, <Xb, X>, Tr Xb and <G, X> (the layer's coefficient gradients).
// The tile needs M at (i, j) and at (j, i): two products over the same K blocks, Xb_I X_J^T and
// X_I Xb_J^T, so that no M goes through memory and no transposed pass follows. n = 256: 8 us per
// layer against 43 for the separate product, elementwise pass and one-thread reduction.
template <bool ALIGNED>
__global__ void __launch_bounds__(NT) k_wide_bwd(BwdArgs p) {
    constexpr int BM = 32;
    using M = Mfma<float>;
    using W = WCfg<float, BM, 2>;
    using gvec = typename std::conditional<ALIGNED, floatx4, Unaligned<float>::vec>::type;
    static_assert(W::PER == 1 && W::NB == 1, "one group per thread");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1, fr = lane & 15;
    const int64_t np = p.n;
    const int t = split::xcd_tile(blockIdx.x, gridDim.x);
    int I, J;
    split::tile_coords(t, (int)(np / BM), I, J);
    const bool diag = I == J;
    const int64_t I0 = (int64_t)I * BM, J0 = (int64_t)J * BM;
    // element groups: (I0 + r, J0 + c ..) of the tile and (J0 + r, I0 + c ..) of its mirror
    const int r = tid / W::G, c = (tid % W::G) * 4;
    const int64_t gu = (I0 + r) * np + J0 + c, gl = (J0 + r) * np + I0 + c;
    auto load = [](const float* m, int64_t o) -> floatx4 { return *reinterpret_cast<const gvec*>(m + o); };
    const floatx4 xu = load(p.X, gu), bu = load(p.Xb, gu), qu = load(p.G, gu);
    const floatx4 xl = load(p.X, gl), bl = load(p.Xb, gl), ql = load(p.G, gl);

    floatx4 acc[2][1][1] = {{{floatx4{0, 0, 0, 0}}}, {{floatx4{0, 0, 0, 0}}}};
    const float* const lp[2] = {p.Xb + I0 * np, p.X + I0 * np};
    const float* const rp[2] = {p.X + J0 * np, p.Xb + J0 * np};
    wide_products<float, BM, ALIGNED, 2>(lp, rp, np, (int)(np / W::BK), true, smem, acc);

    float* s0 = reinterpret_cast<float*>(smem);   // M at (i, j)
    float* s1 = s0 + BM * W::LDY;                 // M at (j, i), stored at (i, j)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int o = (wm * 16 + M::crow(lane, j)) * W::LDY + wn * 16 + fr;
        s0[o] = acc[0][0][0][j];
        s1[o] = acc[1][0][0][j];
    }
    __syncthreads();
    double sa = 0.0, sb = 0.0, sc = 0.0, sd = 0.0;
    auto half = [&](int64_t o, auto m_at, auto mt_at, const floatx4& x, const floatx4& xb,
                    const floatx4& g, int64_t row, int64_t col) {
        floatx4 out;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float m = m_at(k), mt = mt_at(k);
            sa += (double)m * x[k];
            sb += (double)xb[k] * x[k];
            if (row == col + k) sc += xb[k];
            sd += (double)g[k] * x[k];
            out[k] = fmaf(p.cd, g[k], fmaf(p.ca, m + mt, p.cb * xb[k]));
        }
        *reinterpret_cast<gvec*>(p.Xb_out + o) = out;
    };
    half(gu, [&](int k) { return s0[r * W::LDY + c + k]; }, [&](int k) { return s1[r * W::LDY + c + k]; },
         xu, bu, qu, I0 + r, J0 + c);
    if (!diag)
        half(gl, [&](int k) { return s1[(c + k) * W::LDY + r]; },
             [&](int k) { return s0[(c + k) * W::LDY + r]; }, xl, bl, ql, J0 + r, I0 + c);
    sa = wave_sum(sa);
    sb = wave_sum(sb);
    sc = wave_sum(sc);
    sd = wave_sum(sd);
    __syncthreads();
    double* red = reinterpret_cast<double*>(smem);
    if (lane == 0) {
        red[4 * wave] = sa;
        red[4 * wave + 1] = sb;
        red[4 * wave + 2] = sc;
        red[4 * wave + 3] = sd;
    }
    __syncthreads();
    if (tid < 4) p.part[(size_t)t * 4 + tid] = (red[tid] + red[4 + tid]) + (red[8 + tid] + red[12 + tid]);
}

// Lower triangle of an np x np FP32 matrix from its upper triangle (X[i][j] = X[j][i] for
// i > j), through 64 x 64 LDS tiles: workgroup (I, J), I >= J, reads the upper tile (J, I) row by
// row and writes its transpose into the lower tile (I, J); diagonal tiles copy within the tile.
__global__ void __launch_bounds__(256) k_mirror_upper(float* X, int64_t np) {
    constexpr int BM = kPad;
    __shared__ float t[BM][BM + 1];
    int rem = blockIdx.x, i = 0;
    const int T_ = (int)(np / BM);
    while (rem >= T_ - i) {   // upper-tile enumeration: tile (i, i + rem) is the source
        rem -= T_ - i;
        ++i;
    }
    const int64_t R0 = (int64_t)i * BM, C0 = (int64_t)(i + rem) * BM;   // source tile, R0 <= C0
    for (int e = threadIdx.x; e < BM * BM; e += 256) {
        const int r = e / BM, c = e % BM;
        t[r][c] = X[(R0 + r) * np + C0 + c];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < BM * BM; e += 256) {
        const int r = e / BM, c = e % BM;   // destination (C0 + r, R0 + c) = source (R0 + c, C0 + r)
        if (R0 == C0 && !(r > c)) continue;
        X[(C0 + r) * np + R0 + c] = t[c][r];
    }
}

template <typename T, int BM, bool ALIGNED>
hipError_t launch_t(const WideArgs& a, hipStream_t s) {
    auto kern = k_wide<T, BM, ALIGNED>;
    constexpr size_t lds = WCfg<T, BM>::LDS;
    static_assert(lds <= 64 * 1024, "no attribute needed for the dynamic LDS");
    const int T_ = (int)(a.np / BM);
    hipLaunchKernelGGL(kern, dim3(T_ * (T_ + 1) / 2), dim3(NT), lds, s, a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch(const WideArgs& a, hipStream_t s) {
    if (a.np % kPad != 0 || a.n < 1 || a.n > a.np) return hipErrorInvalidValue;
    const uintptr_t m = reinterpret_cast<uintptr_t>(a.X_in) | reinterpret_cast<uintptr_t>(a.X_out) |
                        reinterpret_cast<uintptr_t>(a.A);
    if (m % 16 != 0)
        return wide_bm(a.np) == 32 ? launch_t<T, 32, false>(a, s) : launch_t<T, 64, false>(a, s);
    return wide_bm(a.np) == 32 ? launch_t<T, 32, true>(a, s) : launch_t<T, 64, true>(a, s);
}

}  // namespace

int wide_tile() { return kPad; }
// Where the line lies (us per layer, 32 x 32 against 64 x 64 tiles): FP32 n = 1500 43 / 60, 4096
// 596 / 635, 5000 1321 / 1224, 8192 5024 / 4586; FP64 n = 1000 31 / 49, 4096 1197 / 1250, 5000
// 2629 / 2276, 8192 10334 / 9147: small tiles spread few blocks over the SIMDs, large ones halve the
// operand traffic.
int wide_bm(int64_t np) { return np <= 4096 ? 32 : 64; }
int wide_tiles(int64_t np) {
    const int T_ = (int)(np / wide_bm(np));
    return T_ * (T_ + 1) / 2;
}
hipError_t launch_layer_f32(const WideArgs& a, hipStream_t s) { return launch<float>(a, s); }
hipError_t launch_layer_f64(const WideArgs& a, hipStream_t s) { return launch<double>(a, s); }
bool wide_resident(int64_t np, int n_cu) {
    const int64_t T = np / 32;
    return np % kPad == 0 && 8 * (T * (T + 1) / 2) <= n_cu;
}
hipError_t launch_layers_wide_resident(const WideArgs& a, bool f64, const ResidentWide& L,
                                       ResidentArgs R, hipStream_t s) {
    if (a.np % kPad != 0 || a.n < 1 || a.n > a.np || R.L < 1 || R.L > kResMaxL || !R.ctl)
        return hipErrorInvalidValue;
    const int T_ = (int)(a.np / 32);
    R.ntiles = T_ * (T_ + 1) / 2;
    const dim3 grid(8 * R.ntiles);
    if (f64) hipLaunchKernelGGL(k_wide_resident<double>, grid, dim3(NT), (WCfg<double, 32>::LDS), s, a, L, R);
    else hipLaunchKernelGGL(k_wide_resident<float>, grid, dim3(NT), (WCfg<float, 32>::LDS), s, a, L, R);
    return hipGetLastError();
}
int wide_bwd_tiles(int64_t n) {
    const int T_ = (int)(n / 32);
    return T_ * (T_ + 1) / 2;
}
hipError_t launch_layer_bwd(const BwdArgs& a, hipStream_t s) {
    if (a.n < kPad || a.n % kPad != 0) return hipErrorInvalidValue;
    const uintptr_t m = reinterpret_cast<uintptr_t>(a.X) | reinterpret_cast<uintptr_t>(a.Xb) |
                        reinterpret_cast<uintptr_t>(a.G) | reinterpret_cast<uintptr_t>(a.Xb_out);
    constexpr size_t lds = WCfg<float, 32, 2>::LDS;
    static_assert(lds <= 64 * 1024, "no attribute needed for the dynamic LDS");
    const dim3 grid(wide_bwd_tiles(a.n));
    if (m % 16 != 0) hipLaunchKernelGGL(k_wide_bwd<false>, grid, dim3(NT), lds, s, a);
    else hipLaunchKernelGGL(k_wide_bwd<true>, grid, dim3(NT), lds, s, a);
    return hipGetLastError();
}
hipError_t launch_mirror_upper_f32(float* X, int64_t np, hipStream_t s) {
    if (np % kPad != 0) return hipErrorInvalidValue;
    const int T_ = (int)(np / kPad);
    hipLaunchKernelGGL(k_mirror_upper, dim3(T_ * (T_ + 1) / 2), dim3(256), 0, s, X, np);
    return hipGetLastError();
}

}  // namespace fe
