// Learned q-proposal: multilayer perceptron training and inference kernels,
// the proposal/inverse-CDF sampler and the importance-sampling weights.
//
// Network: z_l = W_l a_{l-1} + b_l, a_l = silu(z_l) for hidden layers, linear
// output; parameters packed per layer as W_l [out, in] then b_l [out].
// Two arithmetic paths: BF16 operands on v_mfma_f32_16x16x32_bf16 with FP32
// accumulation (float storage), and an FP64 path on v_mfma_f64_16x16x4f64
// (double storage) used to check gradients against the FP64 oracle.
#include <algorithm>

#include "ext.hpp"
#include "mlp.hpp"

namespace phx {

static inline int gridm(int64_t n, int block) {
    int64_t g = (n + block - 1) / block;
    if (g > 65535 * 16) g = 65535 * 16;
    if (g < 1) g = 1;
    return (int)g;
}

typedef short s8m __attribute__((ext_vector_type(8)));
typedef __bf16 bf8m __attribute__((ext_vector_type(8)));
typedef float f2m __attribute__((ext_vector_type(2)));
typedef __bf16 bf2m __attribute__((ext_vector_type(2)));

// two floats to BF16 (round to nearest even), the first in the low half
__device__ inline uint32_t pack_bf(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2m{a, b}, bf2m));
}

// ---------------------------------------------------------------------------
// BF16 products C[M, N] = A[M, K] B[K, N] of the network on
// v_mfma_f32_16x16x32_bf16 (FP32 storage, operands rounded once to BF16, FP32
// accumulation along ascending K).
//
// A work-group of four waves owns a 64 x 64 tile of C (each wave 32 x 32).  Per
// 64-wide K step both operand tiles are converted once into LDS, k contiguous (rows
// padded to 72 BF16), and read from there as 16-byte fragments; the next step's
// global loads are in registers while the current step's MFMAs run.  64 x 64 rather
// than larger tiles: a minibatch of 4,096 rows and 256 columns then makes 256
// work-groups, one per CU, and the products are bound by that latency, not by their
// flops.  An operand is k-fast (element (r, k) at r ld + k) or r-fast (k ld + r).
//
// Per job, besides C:
//   bias / act      C = A B + bias and act = silu(C) from the same pass (C may be NULL);
//   zprev           C = (A B) silu'(zprev), the step back through an activation;
//   nsplit, colsum  split z takes rows [z kchunk, ...) of K and writes its own C; colsum
//                   [nsplit, M] receives the sums of A's rows over the split (in double,
//                   from the unrounded values), the bias gradient.
// Minibatch of 4,096, width 256, depth 4: forward 136 -> 58 us for five layers, the
// backward products with their activations, bias sums and reduction 803 -> 77 us
// (32 x 128 tiles without K split made 16 work-groups for a weight gradient).
// ---------------------------------------------------------------------------
constexpr int kMT = 64, kMK = 64, kMLd = 72;

struct MlpSmem {
    __attribute__((aligned(16))) uint16_t a[kMT * kMLd];
    __attribute__((aligned(16))) uint16_t b[kMT * kMLd];
};

// four consecutive floats of which the first n are in range (16-byte load where
// the address allows it)
__device__ inline f4 load4(const float* p, int n, bool vec) {
    if (n >= 4 && vec) return *reinterpret_cast<const f4*>(p);
    f4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (i < n) v[i] = p[i];
    return v;
}

// one 64 x 64 operand tile: global -> registers (16 values a thread) -> BF16 in LDS
template <bool KFAST>
struct MlpOperand {
    const float* p;
    int64_t ld, r0, R, K;  // K: end of this work-group's k range
    bool vec;
    f4 v[4];
    __device__ MlpOperand(const float* p_, int64_t ld_, int64_t r0_, int64_t R_, int64_t K_)
        : p(p_), ld(ld_), r0(r0_), R(R_), K(K_) {
        vec = (ld & 3) == 0 && (reinterpret_cast<uintptr_t>(p) & 15) == 0;
    }
    __device__ void fetch(int64_t k0) {
        const int tid = threadIdx.x;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int64_t r, k;  // first element of the group of four (along k, or along r)
            if (KFAST) {
                const int e = tid + 256 * j;
                r = r0 + (e >> 4);
                k = k0 + (e & 15) * 4;
                const int64_t n = r < R ? K - k : 0;
                v[j] = load4(p + (n > 0 ? r * ld + k : 0), n > 4 ? 4 : (int)n, vec);
            } else {
                const int e = tid + 256 * (j >> 1);
                r = r0 + (e & 15) * 4;
                k = k0 + 2 * (e >> 4) + (j & 1);
                const int64_t n = k < K ? R - r : 0;
                v[j] = load4(p + (n > 0 ? k * ld + r : 0), n > 4 ? 4 : (int)n, vec);
            }
        }
    }
    __device__ void store(uint16_t* s) const {
        const int tid = threadIdx.x;
        if (KFAST) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int e = tid + 256 * j;
                *reinterpret_cast<uint2*>(s + (e >> 4) * kMLd + (e & 15) * 4) =
                    uint2{pack_bf(v[j][0], v[j][1]), pack_bf(v[j][2], v[j][3])};
            }
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int e = tid + 256 * j;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    *reinterpret_cast<uint32_t*>(s + ((e & 15) * 4 + t) * kMLd + 2 * (e >> 4)) =
                        pack_bf(v[2 * j][t], v[2 * j + 1][t]);
            }
        }
    }
};

template <bool KA, bool KB>
__device__ inline void mlp_tile(const MlpJob& g, int64_t tile, MlpSmem& sm) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int64_t nt = (g.N + kMT - 1) / kMT, mt = (g.M + kMT - 1) / kMT;
    const int64_t n0 = tile % nt * kMT, m0 = tile / nt % mt * kMT, z = tile / (nt * mt);
    const int64_t kb = z * g.kchunk, ke = g.K < kb + g.kchunk ? g.K : kb + g.kchunk;
    MlpOperand<KA> oa(g.A, g.lda, m0, g.M, ke);
    MlpOperand<KB> ob(g.B, g.ldb, n0, g.N, ke);
    f4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[i][t] = f4{0, 0, 0, 0};
    // r-fast A: a thread's rows are the same in every step
    const bool sums = !KA && g.colsum && n0 == 0;
    double cs[4] = {0.0, 0.0, 0.0, 0.0};
    oa.fetch(kb);
    ob.fetch(kb);
    for (int64_t k0 = kb; k0 < ke; k0 += kMK) {
        oa.store(sm.a);
        ob.store(sm.b);
        if (sums) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < 4; ++t) cs[t] += (double)oa.v[j][t];
        }
        __syncthreads();
        if (k0 + kMK < ke) {
            oa.fetch(k0 + kMK);
            ob.fetch(k0 + kMK);
        }
#pragma unroll
        for (int h = 0; h < kMK; h += 32) {
            s8m a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                a[i] = *reinterpret_cast<const s8m*>(&sm.a[(wm + 16 * i + li) * kMLd + h + 8 * lk]);
#pragma unroll
            for (int t = 0; t < 2; ++t)
                b[t] = *reinterpret_cast<const s8m*>(&sm.b[(wn + 16 * t + li) * kMLd + h + 8 * lk]);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf8m, a[i]), __builtin_bit_cast(bf8m, b[t]), acc[i][t], 0,
                        0, 0);
        }
        __syncthreads();
    }
    float* C = g.C ? g.C + z * g.M * g.N : nullptr;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t row = m0 + wm + 16 * i + 4 * lk + v, col = n0 + wn + 16 * t + li;
                if (row < g.M && col < g.N) {
                    float r = acc[i][t][v];
                    const int64_t o = row * g.N + col;
                    if (g.bias) r += g.bias[col];
                    if (g.zprev) {
                        const float x = g.zprev[o];
                        const float sg = 1.0f / (1.0f + exp(-x));
                        r = r * sg * (1.0f + x * (1.0f - sg));
                    }
                    if (C) C[o] = r;
                    if (g.act) g.act[o] = r / (1.0f + exp(-r));
                }
            }
    if (sums) {  // over the 16 threads that hold the same four rows, in thread order
        double* sr = reinterpret_cast<double*>(&sm);  // [16][64]; the tiles are done with
#pragma unroll
        for (int t = 0; t < 4; ++t) sr[(tid >> 4) * 64 + (tid & 15) * 4 + t] = cs[t];
        __syncthreads();
        if (tid < 64 && m0 + tid < g.M) {
            double s = 0.0;
            for (int i = 0; i < 16; ++i) s += sr[i * 64 + tid];
            g.colsum[z * g.M + m0 + tid] = s;
        }
    }
}

// act(X W^T + b): both operands k-fast
__global__ __launch_bounds__(256) void mlp_forward_kernel(MlpJob g) {
    __shared__ MlpSmem sm;
    mlp_tile<true, true>(g, blockIdx.x, sm);
}

// One layer back: work-groups below n_da take the input gradient dZ W (with the
// previous activation's derivative), the others the weight gradient dZ^T a_prev and
// the bias sums; the two are independent and fill the chip together.
__global__ __launch_bounds__(256) void mlp_backward_kernel(MlpJob da, MlpJob dw, int64_t n_da) {
    __shared__ MlpSmem sm;
    if ((int64_t)blockIdx.x < n_da)
        mlp_tile<true, false>(da, blockIdx.x, sm);
    else
        mlp_tile<false, false>(dw, (int64_t)blockIdx.x - n_da, sm);
}

// sums of the splits of every layer's weight and bias gradients, in split order
__global__ __launch_bounds__(256) void mlp_grad_reduce_kernel(MlpGradParts t, float* grad) {
    for (int64_t p = blockIdx.x * 256LL + threadIdx.x; p < t.total; p += (int64_t)gridDim.x * 256) {
        int l = 0;
        while (l + 1 < t.layers && p >= t.off[l + 1]) ++l;
        const int64_t j = p - t.off[l], nw = (int64_t)t.out[l] * t.in[l];
        if (j < nw) {
            if (t.split[l] == 1) continue;  // written in place
            float s = t.w[l][j];
            for (int z = 1; z < t.split[l]; ++z) s += t.w[l][z * nw + j];
            grad[p] = s;
        } else {
            double s = 0.0;
            for (int z = 0; z < t.split[l]; ++z) s += t.b[l][(int64_t)z * t.out[l] + (j - nw)];
            grad[p] = (float)s;
        }
    }
}

static int64_t mlp_tiles(const MlpJob& g) {
    return ((g.M + kMT - 1) / kMT) * ((g.N + kMT - 1) / kMT) * g.nsplit;
}

// K range of a split, a multiple of the K step, such that the splits fill the chip (one
// work-group per CU) with at least 128 rows each
int mlp_splits(int64_t M, int64_t N, int64_t K, int64_t* kchunk) {
    const int64_t tiles = ((M + kMT - 1) / kMT) * ((N + kMT - 1) / kMT);
    const int64_t want = std::max<int64_t>(1, std::min<int64_t>(256 / tiles, (K + 127) / 128));
    *kchunk = ((K + want - 1) / want + kMK - 1) / kMK * kMK;
    return (int)((K + *kchunk - 1) / *kchunk);
}

hipError_t launch_mlp_forward(const MlpJob& g, hipStream_t s) {
    if (g.M <= 0 || g.N <= 0) return hipSuccess;
    const int64_t n = mlp_tiles(g);
    if (n > 2147483647LL || g.K <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(mlp_forward_kernel, dim3((unsigned)n), dim3(256), 0, s, g);
    return hipGetLastError();
}

hipError_t launch_mlp_backward(const MlpJob* da, const MlpJob& dw, hipStream_t s) {
    const int64_t nd = da ? mlp_tiles(*da) : 0, n = nd + mlp_tiles(dw);
    if (n <= 0 || n > 2147483647LL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(mlp_backward_kernel, dim3((unsigned)n), dim3(256), 0, s, da ? *da : dw, dw, nd);
    return hipGetLastError();
}

hipError_t launch_mlp_grad_reduce(const MlpGradParts& t, float* grad, hipStream_t s) {
    hipLaunchKernelGGL(mlp_grad_reduce_kernel, dim3(gridm(t.total, 256)), dim3(256), 0, s, t, grad);
    return hipGetLastError();
}

// FP64 (gradient checks): A(i, k) = TA ? A[k lda + i] : A[i lda + k];
// B(k, j) = TB ? B[j ldb + k] : B[k ldb + j].  Work-group: 4 waves side by side along
// N, each 2 x 2 tiles of 16 x 16.
template <bool TA, bool TB>
__global__ __launch_bounds__(256) void mlp_gemm_f64(const double* __restrict__ A, int64_t lda,
                                                    const double* __restrict__ B, int64_t ldb,
                                                    double* __restrict__ C, int64_t ldc, int64_t M,
                                                    int64_t N, int64_t K,
                                                    const double* __restrict__ bias) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const int64_t m0 = (int64_t)blockIdx.y * 32;
    const int64_t n0 = ((int64_t)blockIdx.x * 4 + wave) * 32;
    if (n0 >= N) return;
    d4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[i][t] = d4{0, 0, 0, 0};
    for (int64_t k0 = 0; k0 < K; k0 += 4) {
        const int64_t k = k0 + lk;
        double a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int64_t row = m0 + 16 * i + li;
            a[i] = (row < M && k < K) ? (TA ? A[k * lda + row] : A[row * lda + k]) : 0.0;
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int64_t col = n0 + 16 * t + li;
            b[t] = (col < N && k < K) ? (TB ? B[col * ldb + k] : B[k * ldb + col]) : 0.0;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                acc[i][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[t], acc[i][t], 0, 0, 0);
    }
    // f64 MFMA result v of lane group lk is row lk + 4v
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t row = m0 + 16 * i + lk + 4 * v;
                const int64_t col = n0 + 16 * t + li;
                if (row < M && col < N) {
                    double r = acc[i][t][v];
                    if (bias) r += bias[col];
                    C[row * ldc + col] = r;
                }
            }
}

hipError_t launch_mlp_gemm_f64(bool ta, bool tb, const double* A, int64_t lda, const double* B,
                               int64_t ldb, double* C, int64_t ldc, int64_t M, int64_t N, int64_t K,
                               const double* bias, hipStream_t s) {
    if (M <= 0 || N <= 0) return hipSuccess;
    dim3 grid((unsigned)((N + 127) / 128), (unsigned)((M + 31) / 32));
    if (grid.y > 65535) return hipErrorInvalidValue;
#define PHX_GO(TAv, TBv)                                                                        \
    if (ta == TAv && tb == TBv) {                                                               \
        hipLaunchKernelGGL((mlp_gemm_f64<TAv, TBv>), grid, dim3(256), 0, s, A, lda, B, ldb, C,  \
                           ldc, M, N, K, bias);                                                 \
        return hipGetLastError();                                                               \
    }
    PHX_GO(false, false) PHX_GO(false, true) PHX_GO(true, false)
#undef PHX_GO
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// elementwise pieces
// ---------------------------------------------------------------------------
template <class T>
__global__ void silu_fwd_kernel(const T* z, T* a, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const T x = z[i];
        a[i] = x / ((T)1 + exp(-x));
    }
}
template <class T>
__global__ void silu_bwd_kernel(const T* da, const T* z, T* dz, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const T x = z[i];
        const T sg = (T)1 / ((T)1 + exp(-x));
        dz[i] = da[i] * sg * ((T)1 + x * ((T)1 - sg));
    }
}
// dY = 2 (Y - t) / B; squared errors summed per block into sums[block]
template <class T>
__global__ void mse_grad_kernel(const T* y, const T* t, T* dy, int64_t B, double* sums) {
    __shared__ double sh[256];
    double acc = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < B;
         i += (int64_t)gridDim.x * blockDim.x) {
        const T r = y[i] - t[i];
        dy[i] = (T)2 * r / (T)B;
        acc += (double)r * (double)r;
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = sh[0];
}
// db[j] = sum_b dZ[b, j]
template <class T>
__global__ __launch_bounds__(256) void colsum_kernel(const T* dz, int64_t B, int64_t N, T* db) {
    __shared__ double sh[256];
    const int64_t j = blockIdx.x;
    double acc = 0.0;
    for (int64_t b = threadIdx.x; b < B; b += 256) acc += (double)dz[b * N + j];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) db[j] = (T)sh[0];
}

template <class T>
hipError_t launch_silu_fwd(const T* z, T* a, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(silu_fwd_kernel<T>, dim3(gridm(n, 256)), dim3(256), 0, s, z, a, n);
    return hipGetLastError();
}
template <class T>
hipError_t launch_silu_bwd(const T* da, const T* z, T* dz, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(silu_bwd_kernel<T>, dim3(gridm(n, 256)), dim3(256), 0, s, da, z, dz, n);
    return hipGetLastError();
}
template <class T>
hipError_t launch_mse_grad(const T* y, const T* t, T* dy, int64_t B, double* sums, int nblk,
                           hipStream_t s) {
    hipLaunchKernelGGL(mse_grad_kernel<T>, dim3(nblk), dim3(256), 0, s, y, t, dy, B, sums);
    return hipGetLastError();
}
template <class T>
hipError_t launch_colsum(const T* dz, int64_t B, int64_t N, T* db, hipStream_t s) {
    hipLaunchKernelGGL(colsum_kernel<T>, dim3((unsigned)N), dim3(256), 0, s, dz, B, N, db);
    return hipGetLastError();
}
template hipError_t launch_silu_fwd<double>(const double*, double*, int64_t, hipStream_t);
template hipError_t launch_silu_bwd<double>(const double*, const double*, double*, int64_t,
                                            hipStream_t);
template hipError_t launch_colsum<double>(const double*, int64_t, int64_t, double*, hipStream_t);
template hipError_t launch_mse_grad<double>(const double*, const double*, double*, int64_t, double*,
                                            int, hipStream_t);
template hipError_t launch_mse_grad<float>(const float*, const float*, float*, int64_t, double*,
                                           int, hipStream_t);

// Adam on FP32 master parameters (Kingma & Ba, bias-corrected moments)
__global__ void adam_kernel(float* p, const float* g, float* m, float* v, int64_t n, double lr,
                            double b1, double b2, double eps, double c1, double c2) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double gi = g[i];
        const double mi = b1 * m[i] + (1.0 - b1) * gi;
        const double vi = b2 * v[i] + (1.0 - b2) * gi * gi;
        m[i] = (float)mi;
        v[i] = (float)vi;
        p[i] = (float)(p[i] - lr * (mi / c1) / (sqrt(vi / c2) + eps));
    }
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, int64_t n, int t, double lr,
                       double b1, double b2, double eps, hipStream_t s) {
    const double c1 = 1.0 - pow(b1, t), c2 = 1.0 - pow(b2, t);
    hipLaunchKernelGGL(adam_kernel, dim3(gridm(n, 256)), dim3(256), 0, s, p, g, m, v, n, lr, b1, b2,
                       eps, c1, c2);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Network inputs of one sample (k, band energy, q, mode nu):
//   n_harm = 0: [k (3 crystal coords), (eps - e0)/escale, q (3), one-hot(nu)]
//   n_harm > 0: [(eps - e0)/escale, one-hot(nu), then for h = 1..n_harm
//                cos, sin of 2 pi h k_d (3 + 3) and of 2 pi h q_d (3 + 3)]
// The periodic form gives the network the Fourier harmonics in which the
// Wannier-gauge coupling is band-limited; h i_d mod N_d is reduced exactly.
// ---------------------------------------------------------------------------
__host__ __device__ inline int n_features(int nm, int n_harm) {
    return n_harm == 0 ? 7 + nm : 1 + nm + 12 * n_harm;
}

template <class T>
__device__ inline void write_features(T* x, int k0, int k1, int k2, int q0, int q1, int q2, int nu,
                                      double e, Mesh mesh, int nm, int n_harm) {
    if (n_harm == 0) {
        x[0] = (T)((double)k0 / mesh.n0);
        x[1] = (T)((double)k1 / mesh.n1);
        x[2] = (T)((double)k2 / mesh.n2);
        x[3] = (T)e;
        x[4] = (T)((double)q0 / mesh.n0);
        x[5] = (T)((double)q1 / mesh.n1);
        x[6] = (T)((double)q2 / mesh.n2);
        for (int v = 0; v < nm; ++v) x[7 + v] = (T)(v == nu ? 1 : 0);
        return;
    }
    x[0] = (T)e;
    for (int v = 0; v < nm; ++v) x[1 + v] = (T)(v == nu ? 1 : 0);
    const int idx[6] = {k0, k1, k2, q0, q1, q2};
    const int Ns[6] = {mesh.n0, mesh.n1, mesh.n2, mesh.n0, mesh.n1, mesh.n2};
    T* y = x + 1 + nm;
    for (int h = 1; h <= n_harm; ++h)
        for (int d = 0; d < 6; ++d) {
            const int a = (int)(((int64_t)h * idx[d]) % Ns[d]);
            double sn, cs;
            sincospi(2.0 * (double)a / Ns[d], &sn, &cs);
            y[0] = (T)cs;
            y[1] = (T)sn;
            y += 2;
        }
}

template <class T>
__global__ void features_kernel(const int32_t* k_idx, const double* eps, const int32_t* q_idx,
                                const int32_t* nu, int64_t B, Mesh mesh, int nm, int n_harm,
                                double e0, double escale, T* X) {
    const int nin = n_features(nm, n_harm);
    for (int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < B;
         b += (int64_t)gridDim.x * blockDim.x) {
        int k0, k1, k2, q0, q1, q2;
        mesh_triple(k_idx[b], mesh, k0, k1, k2);
        mesh_triple(q_idx[b], mesh, q0, q1, q2);
        write_features<T>(X + b * nin, k0, k1, k2, q0, q1, q2, nu[b], (eps[b] - e0) / escale, mesh,
                          nm, n_harm);
    }
}

template <class T>
hipError_t launch_features(const int32_t* k_idx, const double* eps, const int32_t* q_idx,
                           const int32_t* nu, int64_t B, Mesh mesh, int nm, int n_harm, double e0,
                           double escale, T* X, hipStream_t s) {
    if (B <= 0) return hipSuccess;
    hipLaunchKernelGGL(features_kernel<T>, dim3(gridm(B, 256)), dim3(256), 0, s, k_idx, eps, q_idx,
                       nu, B, mesh, nm, n_harm, e0, escale, X);
    return hipGetLastError();
}
template hipError_t launch_features<float>(const int32_t*, const double*, const int32_t*,
                                           const int32_t*, int64_t, Mesh, int, int, double, double,
                                           float*, hipStream_t);
template hipError_t launch_features<double>(const int32_t*, const double*, const int32_t*,
                                            const int32_t*, int64_t, Mesh, int, int, double, double,
                                            double*, hipStream_t);

int feature_count(int nm, int n_harm) { return n_features(nm, n_harm); }

// p_raw[q] = sum_nu max(exp(y[q nm + nu]) - c, 0)
__global__ void proposal_raw_kernel(const float* y, int64_t nq, int nm, double c, double* p) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < nq;
         q += (int64_t)gridDim.x * blockDim.x) {
        double acc = 0.0;
        for (int v = 0; v < nm; ++v) {
            const double e = exp(fmin((double)y[q * nm + v], 80.0)) - c;
            acc += e > 0.0 ? e : 0.0;
        }
        p[q] = acc;
    }
}

hipError_t launch_proposal_raw(const float* y, int64_t nq, int nm, double c, double* p,
                               hipStream_t s) {
    hipLaunchKernelGGL(proposal_raw_kernel, dim3(gridm(nq, 256)), dim3(256), 0, s, y, nq, nm, c, p);
    return hipGetLastError();
}

// E[list[i]] = D[list[i]] exp(y[i])
__global__ void weight_list_kernel(const double* D, const int32_t* list, const float* y, int64_t n,
                                   double* E) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = list[i];
        E[r] = D[r] * exp(fmin((double)y[i], 80.0));
    }
}

// p_raw[q] = sum_nu E[q nm + nu] (fixed order)
__global__ void sum_modes_kernel(const double* E, int64_t N, int nm, double* p) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < N;
         q += (int64_t)gridDim.x * blockDim.x) {
        double acc = 0.0;
        for (int v = 0; v < nm; ++v) acc += E[q * nm + v];
        p[q] = acc;
    }
}

hipError_t launch_weight_list(const double* D, const int32_t* list, const float* y, int64_t n,
                              double* E, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(weight_list_kernel, dim3(gridm(n, 256)), dim3(256), 0, s, D, list, y, n, E);
    return hipGetLastError();
}
hipError_t launch_sum_modes(const double* E, int64_t N, int nm, double* p, hipStream_t s) {
    hipLaunchKernelGGL(sum_modes_kernel, dim3(gridm(N, 256)), dim3(256), 0, s, E, N, nm, p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The proposal for many k at once: entries f = k NR + (q nm + nu) of D [nk, NR]
// with D > thr x max over the k's row are listed in flat order (per-chunk
// counts, an exclusive scan, then the writes), so the network runs over the
// listed entries of every k in a few large batches.
// ---------------------------------------------------------------------------
constexpr int kSelChunk = 4096;

__global__ __launch_bounds__(256) void sel_count_kernel(const double* D, const double* dmax,
                                                        int64_t total, int64_t NR, double thr,
                                                        int32_t* counts) {
    __shared__ int sm[4];
    const int64_t c0 = (int64_t)blockIdx.x * kSelChunk;
    int n = 0;
    for (int i = threadIdx.x; i < kSelChunk; i += 256) {
        const int64_t f = c0 + i;
        if (f < total && D[f] > thr * dmax[f / NR]) ++n;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = sm[0] + sm[1] + sm[2] + sm[3];
}

__global__ __launch_bounds__(256) void sel_write_kernel(const double* D, const double* dmax,
                                                        int64_t total, int64_t NR, double thr,
                                                        const int32_t* offsets, int32_t* list) {
    __shared__ int wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t c0 = (int64_t)blockIdx.x * kSelChunk;
    int64_t base = offsets[blockIdx.x];
    for (int i0 = 0; i0 < kSelChunk; i0 += 256) {
        const int64_t f = c0 + i0 + tid;
        const bool keep = f < total && D[f] > thr * dmax[f / NR];
        const uint64_t bal = __ballot(keep);
        if (lane == 0) wsum[wave] = __popcll(bal);
        __syncthreads();
        int before = 0;
        for (int w = 0; w < wave; ++w) before += wsum[w];
        if (keep) list[base + before + __popcll(bal & ((1ull << lane) - 1ull))] = (int32_t)f;
        base += wsum[0] + wsum[1] + wsum[2] + wsum[3];
        __syncthreads();
    }
}

hipError_t launch_select_rows(const double* D, const double* dmax, int64_t nk, int64_t NR,
                              double thr, int32_t* counts, int64_t* total_out, int32_t* list,
                              hipStream_t s) {
    const int64_t total = nk * NR;
    const int64_t nch = (total + kSelChunk - 1) / kSelChunk;
    if (nch <= 0) return hipSuccess;
    if (nch > 2147483647LL || total > 2147483647LL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(sel_count_kernel, dim3((unsigned)nch), dim3(256), 0, s, D, dmax, total, NR,
                       thr, counts);
    hipError_t e = launch_exclusive_scan(counts, nch, total_out, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sel_write_kernel, dim3((unsigned)nch), dim3(256), 0, s, D, dmax, total, NR,
                       thr, counts, list);
    return hipGetLastError();
}
int64_t select_rows_chunks(int64_t nk, int64_t NR) { return (nk * NR + kSelChunk - 1) / kSelChunk; }

// features of listed flat entries f = k NR + q nm + nu; k's mesh index and band
// energy from per-k device arrays
__global__ void features_flat_kernel(const int32_t* kmesh, const double* epsk, const int32_t* list,
                                     int64_t n, int64_t NR, Mesh mesh, int nm, int n_harm,
                                     double e0, double escale, float* X) {
    const int nin = n_features(nm, n_harm);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t f = list[i];
        const int64_t kl = f / NR, r = f - kl * NR;
        const int64_t q = r / nm;
        const int nu = (int)(r - q * nm);
        int k0, k1, k2, a0, a1, a2;
        mesh_triple(kmesh[kl], mesh, k0, k1, k2);
        mesh_triple(q, mesh, a0, a1, a2);
        write_features<float>(X + i * nin, k0, k1, k2, a0, a1, a2, nu, (epsk[kl] - e0) / escale,
                              mesh, nm, n_harm);
    }
}

hipError_t launch_features_flat(const int32_t* kmesh, const double* epsk, const int32_t* list,
                                int64_t n, int64_t NR, Mesh mesh, int nm, int n_harm, double e0,
                                double escale, float* X, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(features_flat_kernel, dim3(gridm(n, 256)), dim3(256), 0, s, kmesh, epsk,
                       list, n, NR, mesh, nm, n_harm, e0, escale, X);
    return hipGetLastError();
}

// One work-group per k: normalise p_raw (mixed with the uniform distribution),
// build the CDF by an ordered FP64 scan, draw S points by inverse CDF of the
// given uniforms and write the importance weights 1 / (N S p(q)).
__global__ __launch_bounds__(1024) void sample_kernel(double* p, int64_t N, double mix,
                                                      const double* u, int S, int32_t* q_idx,
                                                      double* q_w) {
    // work-group j samples for the j-th k: its row of p and its S uniforms and outputs
    p += (int64_t)blockIdx.x * N;
    u += (int64_t)blockIdx.x * S;
    q_idx += (int64_t)blockIdx.x * S;
    q_w += (int64_t)blockIdx.x * S;
    __shared__ double wsum[16];
    __shared__ double base_sh;
    __shared__ double total_sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // total of p_raw
    double loc = 0.0;
    for (int64_t i = tid; i < N; i += 1024) loc += p[i];
    for (int o = 32; o > 0; o >>= 1) loc += __shfl_xor(loc, o, 64);
    if (lane == 0) wsum[wave] = loc;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int w = 0; w < 16; ++w) t += wsum[w];
        total_sh = t;
        base_sh = 0.0;
    }
    __syncthreads();
    const double tot = total_sh;
    const double a = tot > 0.0 ? (1.0 - mix) / tot : 0.0;
    const double b = tot > 0.0 ? mix / (double)N : 1.0 / (double)N;
    // p <- normalised mixture; then in-place inclusive scan (CDF)
    for (int64_t c0 = 0; c0 < N; c0 += 1024) {
        const int64_t i = c0 + tid;
        double v = i < N ? a * p[i] + b : 0.0;
        double x = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        __syncthreads();
        if (lane == 63) wsum[wave] = x;
        __syncthreads();
        double before = base_sh;
        for (int w = 0; w < wave; ++w) before += wsum[w];
        if (i < N) p[i] = before + x;
        __syncthreads();
        if (tid == 1023) base_sh = before + x;
        __syncthreads();
    }
    const double last = p[N - 1];
    for (int j = tid; j < S; j += 1024) {
        const double target = u[j] * last;
        int64_t lo = 0, hi = N - 1;
        while (lo < hi) {  // first index with CDF > target
            const int64_t mid = (lo + hi) / 2;
            if (p[mid] > target)
                hi = mid;
            else
                lo = mid + 1;
        }
        const double pq = (p[lo] - (lo > 0 ? p[lo - 1] : 0.0)) / last;
        q_idx[j] = (int32_t)lo;
        q_w[j] = 1.0 / ((double)N * (double)S * pq);
    }
}

hipError_t launch_sample(double* p, int64_t N, double mix, const double* u, int S, int32_t* q_idx,
                         double* q_w, int64_t nk, hipStream_t s) {
    if (nk <= 0) return hipSuccess;
    if (nk > 2147483647LL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(sample_kernel, dim3((unsigned)nk), dim3(1024), 0, s, p, N, mix, u, S, q_idx,
                       q_w);
    return hipGetLastError();
}

}  // namespace phx
