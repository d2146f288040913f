// A whole FP64 or FP32 expansion of a small matrix (n <= 64 and n <= 80) in one workgroup and one launch:
// Gershgorin bounds, rescale, all layers, D and the traces. us per density matrix with 26 layers: FP64
// n = 16 21, 48 46, 64 80 (five launches, all layers in one of 8 waves: 41, 76, 116); FP32 n = 64 38,
// 80 54 (a launch per layer: 257, 326).
//
// X lives in LDS (two buffers, one barrier per layer), padded to NB blocks of 16 x 16; each upper block
// has a wave of its own, which keeps its elements of X and of the accumulator A in registers. The
// values are those of the tiled kernels (k_layer_wide.hip): products in ascending k from one MFMA
// chain per block, the same roundings after them.
//
// What bounds it: the MFMA chains of the fullest SIMD (n = 64, FP64: 3 blocks of 16 MFMAs of 64 cycles,
// 1.3 of the 2.5 us that a layer takes); the rest is one trip through LDS and a barrier. LDS rows are
// np + 4 elements: a fragment read (16 rows x 4 k) then touches every bank once per 256 bytes.
#include <math.h>

#include "fe_internal.h"
#include "mfma_wide.h"
#include "rescale_params.h"
#include "split_common.h"

namespace fe {
namespace {

using split::wave_sum;

template <typename T, int NB>
struct SmallCfg {
    static constexpr int U = NB * (NB + 1) / 2;          // upper blocks
    static constexpr int NW = U < 4 ? 4 : U, NT = 64 * NW;
    static constexpr int NP = 16 * NB, LD = NP + 4;
    // buffer 0 of X, then H (FP64, before the first layer) over buffer 1, then the waves' sums
    static constexpr int BUF = NP * LD * (int)sizeof(T), HB = NP * LD * 8;
    static constexpr size_t LDS = BUF + HB + 4 * NW * sizeof(double);
    static constexpr int ROWS = (NP + NW - 1) / NW;      // rows of H per wave
};

template <typename T, int NB>
__global__ void __launch_bounds__((SmallCfg<T, NB>::NT)) k_small(SmallArgs p) {
    using C = SmallCfg<T, NB>;
    using M = wide::Mfma<T>;
    using vec = typename M::vec;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T* const X0 = reinterpret_cast<T*>(smem);
    double* const sH = reinterpret_cast<double*>(smem + C::BUF);
    double* const red = reinterpret_cast<double*>(smem + C::BUF + C::HB);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = (int)p.n;

    // Bounds: a wave per row, as k_gershgorin (r_i = sum_{j != i} |h_ij|), H kept in LDS.
    double h0[C::ROWS], h1[C::ROWS];
#pragma unroll
    for (int u = 0; u < C::ROWS; ++u) {
        const int i = wave + u * C::NW;
        h0[u] = i < n && lane < n ? p.H[i * p.ldh + lane] : 0.0;
        h1[u] = NB > 4 && i < n && lane + 64 < n ? p.H[i * p.ldh + lane + 64] : 0.0;
    }
    double lo = INFINITY, hi = -INFINITY;
    int bad = 0;
#pragma unroll
    for (int u = 0; u < C::ROWS; ++u) {
        const int i = wave + u * C::NW;
        if (i >= C::NP) continue;
        if (lane < C::NP) sH[i * C::LD + lane] = h0[u];
        if (NB > 4 && lane + 64 < C::NP) sH[i * C::LD + lane + 64] = h1[u];
        if (i >= n) continue;
        double a = fabs(h0[u]);
        if (NB > 4) a += fabs(h1[u]);
        const double sum = wave_sum(a);
        const double d = NB > 4 && i >= 64 ? __shfl(h1[u], i - 64, 64) : __shfl(h0[u], i, 64);
        const double r = sum - fabs(d);
        if (!isfinite(sum)) bad = 1;
        lo = fmin(lo, d - r);
        hi = fmax(hi, d + r);
    }
    if (lane == 0) {
        red[wave] = lo;
        red[C::NW + wave] = hi;
        reinterpret_cast<int*>(red + 2 * C::NW)[wave] = bad;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < C::NW; ++w) {
        lo = fmin(lo, red[w]);
        hi = fmax(hi, red[C::NW + w]);
        bad |= reinterpret_cast<int*>(red + 2 * C::NW)[w];
    }
    const Params par = rescale_params(lo, hi, bad, p.mu, p.kT, p.beta0, p.mu0);
    if (tid == 0) *p.P = par;

    // X0 = r (H' - mu' I) + mu0 I, for the entropy rescaled towards mu0 by alpha.
    auto start = [&](int i, int j) -> T {
        if (i >= n || j >= n) return (T)0;
        double v = par.scale * sH[i * C::LD + j] + (i == j ? par.shift : 0.0);
        v = p.alpha * v + (i == j ? (1.0 - p.alpha) * p.mu0 : 0.0);
        return (T)v;
    };
    for (int e = tid; e < C::NP * C::NP; e += C::NT) {
        const int i = e / C::NP, j = e % C::NP;
        X0[i * C::LD + j] = start(i, j);
    }
    // this wave's upper block
    const bool mine = wave < C::U;
    int I = 0, J = wave;
#pragma unroll
    for (int k = NB; k > 1; --k)
        if (J >= k && I == NB - k) {
            J -= k;
            ++I;
        }
    J += I;
    const int col = J * 16 + (lane & 15);
    vec x, acc_d;
    int row[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        row[k] = I * 16 + M::crow(lane, k);
        x[k] = mine ? start(row[k], col) : (T)0;
        acc_d[k] = (T)p.theta[3] * x[k];
    }
    const bool diag = I == J;
    __syncthreads();   // X0 whole, H no longer needed

    const T* const fa = X0 + (I * 16 + (lane & 15)) * C::LD + (lane >> 4);
    const T* const fb = X0 + (J * 16 + (lane & 15)) * C::LD + (lane >> 4);
    constexpr int BUFE = C::BUF / (int)sizeof(T);
    auto products = [&](int buf) {
        vec y = vec{0, 0, 0, 0};
        T a[4 * NB], b[4 * NB];
#pragma unroll
        for (int s = 0; s < 4 * NB; ++s) {
            a[s] = fa[buf * BUFE + 4 * s];
            b[s] = fb[buf * BUFE + 4 * s];
        }
#pragma unroll
        for (int s = 0; s < 4 * NB; ++s) y = M::mma(a[s], b[s], y);
        return y;
    };
    auto value = [&](const double* th, const vec& y, int k) -> T {
#pragma clang fp contract(off)
        const T bx = (T)th[1] * x[k];
        return __builtin_elementwise_fma((T)th[0], y[k], bx) +
               (row[k] == col && col < n ? (T)th[2] : (T)0);
    };
    for (int l = 0; l + 1 < p.L; ++l) {
        const double* th = p.theta + 4 * l;
        if (mine) {
            const vec y = products(l & 1);
            const T dn = (T)th[7];
            T* const o = X0 + ((l & 1) ^ 1) * BUFE;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                x[k] = value(th, y, k);
                if (dn != (T)0) acc_d[k] = __builtin_elementwise_fma(dn, x[k], acc_d[k]);
                if (!diag || row[k] <= col) {   // a diagonal block's lower half mirrors its upper one
                    o[row[k] * C::LD + col] = x[k];
                    o[col * C::LD + row[k]] = x[k];
                }
            }
        }
        __syncthreads();
    }

    // Last layer: D = A + X (I - D if flipped), or U = A + X traced only (entropy).
    const bool ent = p.entropy != 0;
    const int flip = !ent ? par.flipped : 0;
    double tr = 0.0, sq = 0.0;
    if (mine) {
        const double* th = p.theta + 4 * (p.L - 1);
        const vec y = products((p.L - 1) & 1);
        auto put = [&](int64_t i, int64_t j, double v) {
            if (p.out_mode == 0) static_cast<float*>(p.D)[i * p.ldd + j] = (float)v;
            else static_cast<double*>(p.D)[i * p.ldd + j] = v;
        };
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double v = (double)acc_d[k] + (double)value(th, y, k);
            if (flip) v = (row[k] == col ? 1.0 : 0.0) - v;
            if (sizeof(T) == 4 && !ent) v = (double)(float)v;
            if (row[k] <= col && col < n) {
                if (row[k] == col) tr += v;
                sq += (row[k] == col ? 1.0 : 2.0) * v * v;
                if (!ent && p.out_mode != 2) {
                    put(row[k], col, v);
                    if (row[k] < col) put(col, row[k], v);
                }
            }
        }
    }
    tr = wave_sum(tr);
    sq = wave_sum(sq);
    if (lane == 0) {
        red[wave] = tr;
        red[C::NW + wave] = sq;
    }
    __syncthreads();
    if (tid == 0) {
        tr = sq = 0.0;
#pragma unroll
        for (int w = 0; w < C::NW; ++w) {
            tr += red[w];
            sq += red[C::NW + w];
        }
        const double nan = par.status < 0 ? NAN : 0.0;
        if (p.trD) *p.trD = tr + nan;
        if (p.trD2) *p.trD2 = sq + nan;
        if (p.S) *p.S = 4.0 * 0.69314718055994530942 * (tr - sq) + nan;
    }
}

template <typename T, int NB>
hipError_t launch(const SmallArgs& a, hipStream_t s) {
    using C = SmallCfg<T, NB>;
    auto kern = k_small<T, NB>;
    if (C::LDS > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(1), dim3(C::NT), C::LDS, s, a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_nb(const SmallArgs& a, hipStream_t s) {
    switch ((a.n + 15) / 16) {
        case 1: return launch<T, 1>(a, s);
        case 2: return launch<T, 2>(a, s);
        case 3: return launch<T, 3>(a, s);
        case 4: return launch<T, 4>(a, s);
    }
    if constexpr (sizeof(T) == 4)
        if (a.n <= 80) return launch<T, 5>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_small(const SmallArgs& a, bool f64, hipStream_t s) {
    if (a.n < 1 || a.n > small_max_n(f64) || a.L < 1 || a.L > kSmallMaxL) return hipErrorInvalidValue;
    return f64 ? launch_nb<double>(a, s) : launch_nb<float>(a, s);
}

}  // namespace fe
