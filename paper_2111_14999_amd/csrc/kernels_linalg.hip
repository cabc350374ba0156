// Dense building blocks on gfx950: phase tables, complex FP64 GEMM on MFMA,
// batched Hermitian Jacobi eigensolver, phonon/electron post-processing and
// mesh bookkeeping (window, ordered compaction).
#include "kernels.hpp"

namespace phx {

// ---------------------------------------------------------------------------
// Phase table P[p, r] = e^{i 2 pi x_p . R_r}
// Mesh points use exact integer reduction: x.R = sum_d (i_d R_d mod N_d)/N_d.
// Fractional points reduce x.R by its nearest integer before sincospi.
// ---------------------------------------------------------------------------
__global__ void phase_table_kernel(const double* frac, const int32_t* idx, Mesh m, int64_t np,
                                   const int32_t* R, int nR, cd* P, int64_t ldp) {
    const int64_t total = np * (int64_t)nR;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = t / nR;
        const int r = (int)(t - p * nR);
        const int r0 = R[3 * r], r1 = R[3 * r + 1], r2 = R[3 * r + 2];
        double x;
        if (frac) {
            const double* f = frac + 3 * p;
            x = f[0] * r0 + f[1] * r1 + f[2] * r2;
            x -= rint(x);
        } else {
            const int64_t li = idx ? (int64_t)idx[p] : p;
            int i0, i1, i2;
            mesh_triple(li, m, i0, i1, i2);
            int a0 = (int)(((int64_t)i0 * r0) % m.n0);
            int a1 = (int)(((int64_t)i1 * r1) % m.n1);
            int a2 = (int)(((int64_t)i2 * r2) % m.n2);
            if (a0 < 0) a0 += m.n0;
            if (a1 < 0) a1 += m.n1;
            if (a2 < 0) a2 += m.n2;
            x = (double)a0 / m.n0 + (double)a1 / m.n1 + (double)a2 / m.n2;
            x -= rint(x);
        }
        P[p * ldp + r] = expi2pi(x);
    }
}

static inline int grid_for(int64_t n, int block) {
    int64_t g = (n + block - 1) / block;
    if (g > 65535 * 16) g = 65535 * 16;
    if (g < 1) g = 1;
    return (int)g;
}

hipError_t launch_phase_table(const double* frac, const int32_t* idx, Mesh m, int64_t np,
                              const int32_t* R, int nR, cd* P, int64_t ldp, hipStream_t s) {
    if (np <= 0 || nR <= 0) return hipSuccess;
    hipLaunchKernelGGL(phase_table_kernel, dim3(grid_for(np * nR, 256)), dim3(256), 0, s, frac,
                       idx, m, np, R, nR, P, ldp);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Complex FP64 GEMM C = A B on v_mfma_f64_16x16x4f64.
// A work-group is 4 waves side by side along N; each wave owns TM x TN tiles
// of 16 x 16.  MFMA operand layouts (16x16x4 f64): lane l holds A[l%16][l/16],
// B[l/16][l%16]; result v (0..3) of lane l is D[l/16 + 4v][l%16].
// Complex product with 4 real MFMAs: Cr += Ar Br - Ai Bi, Ci += Ar Bi + Ai Br.
// BT = double: a real B (force constants), two MFMAs and half the B bytes.
//
// Rows and columns past the matrix read a clamped address (their results are not
// stored) and a step past K reads the last one's and is never used, so that no load sits
// under a lane branch; k past K meets a zero A in a last step of its own.  40,000 points x
// 256 columns x 343 vectors: 505 us with loads under lane branches, 568 with A zeroed in
// every load, 463 so; 27 vectors 58, 61 and 53.
// ---------------------------------------------------------------------------
template <class BT>
struct ZgemmB;
template <>
struct ZgemmB<cd> {
    // STREAM: B goes past the caches, which it would only sweep
    template <bool STREAM>
    static __device__ inline cd load(const cd* p) {
        if constexpr (STREAM) return cd{__builtin_nontemporal_load(&p->x), __builtin_nontemporal_load(&p->y)};
        return *p;
    }
    static __device__ inline void step1(const cd& a, const cd& b, d4& cr, d4& ci) {
        cr = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, cr, 0, 0, 0);
        ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, ci, 0, 0, 0);
    }
    static __device__ inline void step2(const cd& a, const cd& b, d4& cr, d4& ci) {
        cr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, cr, 0, 0, 0);
        ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, ci, 0, 0, 0);
    }
};
template <>
struct ZgemmB<double> {
    template <bool STREAM>
    static __device__ inline double load(const double* p) {
        if constexpr (STREAM) return __builtin_nontemporal_load(p);
        return *p;
    }
    static __device__ inline void step1(const cd& a, const double& b, d4& cr, d4& ci) {
        cr = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b, cr, 0, 0, 0);
        ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b, ci, 0, 0, 0);
    }
    static __device__ inline void step2(const cd&, const double&, d4&, d4&) {}
};

template <int TM, int TN, int WPS, class BT>
__global__ __launch_bounds__(256, WPS) void zgemm_kernel(const cd* __restrict__ A, int64_t lda,
                                                      const BT* __restrict__ B, int64_t ldb,
                                                      cd* __restrict__ C, int64_t ldc, int64_t M,
                                                      int64_t N, int K, int64_t sb, int64_t sc) {
    using Z = ZgemmB<BT>;
    B += blockIdx.z * sb;  // product z: the same A
    C += blockIdx.z * sc;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const int64_t m0 = (int64_t)blockIdx.y * (16 * TM);
    const int64_t n0 = ((int64_t)blockIdx.x * 4 + wave) * (16 * TN);
    if (n0 >= N) return;
    d4 cr[TM][TN], ci[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            cr[i][j] = d4{0, 0, 0, 0};
            ci[i][j] = d4{0, 0, 0, 0};
        }
    const cd* A0 = A + m0 * lda;
    const BT* B0 = B + n0;
    const int mr = M - m0 < 16 * TM ? (int)(M - m0) : 16 * TM;  // rows and columns of this tile
    const int nc = N - n0 < 16 * TN ? (int)(N - n0) : 16 * TN;
    const cd* pa[TM];
    int cb[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) pa[i] = A0 + min(16 * i + li, mr - 1) * (int)lda;
#pragma unroll
    for (int j = 0; j < TN; ++j) cb[j] = min(16 * j + li, nc - 1);
    const int klast = (K - 1) & ~3;  // first k of the last step
    auto load = [&](int k0, cd* av, BT* bv) {
        const int kc = min(min(k0, klast) + lk, K - 1);
#pragma unroll
        for (int i = 0; i < TM; ++i) av[i] = pa[i][kc];
        const BT* b = B0 + (int64_t)kc * ldb;
#pragma unroll
        for (int j = 0; j < TN; ++j) bv[j] = Z::template load<TM == 1 && TN == 4>(b + cb[j]);
    };
    // operands are prefetched two k-steps ahead: one step of MFMA work is
    // shorter than the HBM latency of the streamed B operand
    cd a_cur[TM], a_n1[TM];
    BT b_cur[TN], b_n1[TN];
    load(0, a_cur, b_cur);
    load(4, a_n1, b_n1);
    // two passes over the tiles, so that dependent MFMAs on one accumulator
    // are 2 TM TN - 1 instructions apart
    auto step = [&] {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) Z::step1(a_cur[i], b_cur[j], cr[i][j], ci[i][j]);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) Z::step2(a_cur[i], b_cur[j], cr[i][j], ci[i][j]);
    };
    const int kfull = K & ~3;
    for (int k0 = 0; k0 < kfull; k0 += 4) {
        cd a_n2[TM];
        BT b_n2[TN];
        load(k0 + 8, a_n2, b_n2);
        step();
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            a_cur[i] = a_n1[i];
            a_n1[i] = a_n2[i];
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            b_cur[j] = b_n1[j];
            b_n1[j] = b_n2[j];
        }
    }
    if (kfull < K) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
            if (kfull + lk >= K) a_cur[i] = cd{0.0, 0.0};
        step();
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t row = m0 + 16 * i + lk + 4 * v;
                const int64_t col = n0 + 16 * j + li;
                if (row < M && col < N) C[row * ldc + col] = cd{cr[i][j][v], ci[i][j][v]};
            }
}

// The same product where the tiles alone leave most of the chip idle (a few hundred
// points): a work-group owns one 16 x 16 tile and its kKSplit waves take the k-steps
// in turn (wave w steps w, w + kKSplit, ...); their sums meet in LDS in wave order.
constexpr int kKSplit = 8;
template <class BT>
__global__ __launch_bounds__(64 * kKSplit) void zgemm_ksplit_kernel(
    const cd* __restrict__ A, int64_t lda, const BT* __restrict__ B, int64_t ldb,
    cd* __restrict__ C, int64_t ldc, int64_t M, int64_t N, int K, int64_t sb, int64_t sc) {
    using Z = ZgemmB<BT>;
    B += blockIdx.z * sb;
    C += blockIdx.z * sc;
    __shared__ cd sC[kKSplit][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const int64_t m0 = (int64_t)blockIdx.y * 16, n0 = (int64_t)blockIdx.x * 16;
    const int64_t row = m0 + li < M ? m0 + li : M - 1, col = n0 + li < N ? n0 + li : N - 1;
    d4 cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
#pragma unroll 4
    for (int k0 = 4 * wave; k0 < K; k0 += 4 * kKSplit) {
        const int k = k0 + lk, kc = k < K ? k : K - 1;
        cd a = A[row * lda + kc];
        const BT b = B[(int64_t)kc * ldb + col];
        if (k >= K) a = cd{0.0, 0.0};
        Z::step1(a, b, cr, ci);
        Z::step2(a, b, cr, ci);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) sC[wave][(lk + 4 * v) * 16 + li] = cd{cr[v], ci[v]};
    __syncthreads();
    for (int e = threadIdx.x; e < 256; e += 64 * kKSplit) {
        cd s = sC[0][e];
#pragma unroll
        for (int w = 1; w < kKSplit; ++w) s = cd{s.x + sC[w][e].x, s.y + sC[w][e].y};
        const int64_t r = m0 + (e >> 4), c = n0 + (e & 15);
        if (r < M && c < N) C[r * ldc + c] = s;
    }
}

template <class BT>
static hipError_t zgemm(const cd* A, int64_t lda, const BT* B, int64_t ldb, cd* C, int64_t ldc,
                        int64_t M, int64_t N, int K, hipStream_t s, int nb = 1, int64_t sb = 0,
                        int64_t sc = 0, bool in_order = false) {
    if (M <= 0 || N <= 0 || nb <= 0) return hipSuccess;
    if (K <= 0 || nb > 65535) return hipErrorInvalidValue;
    auto go = [&](auto kernel, int tm, int tn) {
        dim3 grid((unsigned)((N + 64 * tn - 1) / (64 * tn)), (unsigned)((M + 16 * tm - 1) / (16 * tm)),
                  (unsigned)nb);
        // Under four work-groups (one wave per SIMD each) per CU the tiles wait on their
        // loads, and K is split over waves: 13,824 points x 256 x 343, 864 work-groups, 243 us
        // against 187 us split; 301 points, 20 work-groups, 52 against 12 us.  (The two by two
        // tiles wait less: down to half as many, 3,000 x 1,024 x 343, 136 us, 158 split.)  Up to
        // 32 k, a step or less for each of the waves, the split has nothing to share out and one
        // tile a wave is as quick or quicker: 14,000 x 256 x 27, 32 us split, 23 so.  A real B
        // (dynamical matrices) gains nothing from a split up to 64.  in_order: no split
        // whatever K is, so that a row of C is the same bits in a call of any M (every unsplit
        // tile sums along ascending k).  (Rows too long for the tiles' 32-bit offsets are split
        // as well.)
        const bool few = (int64_t)grid.x * grid.y * nb < (tm == 2 && M > 64 ? 512 : 1024);
        const bool long_rows = lda > ((int64_t)1 << 24);
        if (few && !long_rows && M <= 16 * 65535 && (in_order || K <= (sizeof(BT) == 8 ? 64 : 32))) {
            grid = dim3((unsigned)((N + 63) / 64), (unsigned)((M + 15) / 16), (unsigned)nb);
            hipLaunchKernelGGL((zgemm_kernel<1, 1, 4, BT>), grid, dim3(256), 0, s, A, lda, B, ldb, C,
                               ldc, M, N, K, sb, sc);
        } else if (few || long_rows) {
            grid = dim3((unsigned)((N + 15) / 16), (unsigned)((M + 15) / 16), (unsigned)nb);
            hipLaunchKernelGGL(zgemm_ksplit_kernel<BT>, grid, dim3(64 * kKSplit), 0, s, A, lda, B,
                               ldb, C, ldc, M, N, K, sb, sc);
        } else {
            hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, A, lda, B, ldb, C, ldc, M, N, K, sb, sc);
        }
        return hipGetLastError();
    };
    // Short-and-wide products (stage 1, M = a batch of up to 64 k) cover all rows in one
    // work-group, so each B column is read once, with no more row tiles than the rows
    // fill: up to 32 rows the product is bound by the read of B, above by its MFMAs
    // (4 k x 343 Re x 1.3M columns, 7.2 GB: 4.05 ms with four row tiles, 1.33 ms with
    // one, 1.26 with B's loads past the caches; 40 k x 1.2M columns 3.6 -> 3.0 ms with the K
    // tail apart).  Tall-and-narrow ones (Fourier transforms over many points) use 4 row tiles
    // per wave.
    if (M <= 16) return go(zgemm_kernel<1, 4, 3, BT>, 1, 4);
    if (M <= 32) return go(zgemm_kernel<2, 2, 3, BT>, 2, 2);
    if (M <= 64) return go(zgemm_kernel<4, 2, 2, BT>, 4, 2);
    // Tall and wide: two by two tiles (4 products of 1,024 q' x 3,375 x 125: 284 us, 315
    // with four row tiles; 64,000 q x 3,840 x 343: 11.6 and 12.5 ms).
    // (Twice the grid rows: above 2.1 million rows more than a launch has.)
    if (N >= 1024 && M <= 32 * 65535) return go(zgemm_kernel<2, 2, 3, BT>, 2, 2);
    return go(zgemm_kernel<4, 1, 2, BT>, 4, 1);
}

hipError_t launch_zgemm(const cd* A, int64_t lda, const cd* B, int64_t ldb, cd* C, int64_t ldc,
                        int64_t M, int64_t N, int K, hipStream_t s) {
    return zgemm<cd>(A, lda, B, ldb, C, ldc, M, N, K, s);
}
hipError_t launch_zgemm_batch(const cd* A, int64_t lda, const cd* B, int64_t ldb, int64_t sb, cd* C,
                              int64_t ldc, int64_t sc, int nb, int64_t M, int64_t N, int K,
                              hipStream_t s) {
    return zgemm<cd>(A, lda, B, ldb, C, ldc, M, N, K, s, nb, sb, sc);
}
hipError_t launch_zgemm_real_b(const cd* A, int64_t lda, const double* B, int64_t ldb, cd* C,
                               int64_t ldc, int64_t M, int64_t N, int K, bool in_order, hipStream_t s) {
    return zgemm<double>(A, lda, B, ldb, C, ldc, M, N, K, s, 1, 0, 0, in_order);
}

// ---------------------------------------------------------------------------
// Mass weighting of the force constants: D-kernel entries Phi(R)/sqrt(M_s M_s')
// ---------------------------------------------------------------------------
__global__ void mass_weight_kernel(const double* phi, const double* mass, int nR, int nm,
                                   double* out) {
    const int64_t total = (int64_t)nR * nm * nm;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int j = (int)(t % nm);
        const int i = (int)((t / nm) % nm);
        out[t] = phi[t] / sqrt(mass[i / 3] * mass[j / 3]);
    }
}

hipError_t launch_mass_weight(const double* phi, const double* mass, int nR, int nm, double* out,
                              hipStream_t s) {
    hipLaunchKernelGGL(mass_weight_kernel, dim3(grid_for((int64_t)nR * nm * nm, 256)), dim3(256),
                       0, s, phi, mass, nR, nm, out);
    return hipGetLastError();
}

__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// ---------------------------------------------------------------------------
// Batched Hermitian eigensolver: cyclic Jacobi with the round-robin parallel
// ordering, matrix and eigenvectors in LDS.  Round r of a sweep pairs the indices
// (m, r), (r + k, r - k) mod m for k = 1 .. np/2 - 1, with np = n rounded up to even
// and m = np - 1 (for odd n, m is a zero row and column that never rotates).
// Rotation of pivot (f, g) with a = A_ff, d = A_gg, b = A_fg = |b| e^{i phi}:
//   x = |d - a| / sqrt((d - a)^2 + 4 |b|^2),  c = sqrt((1 + x) / 2),
//   s = sign(d - a) |b| / (c sqrt((d - a)^2 + 4 |b|^2))   (the smaller angle),
//   J_ff = J_gg = c, J_fg = s e^{i phi}, J_gf = -s e^{-i phi};  A <- J^H A J, V <- V J
// (two reciprocal square roots; the rotation of (g, f) is the same matrix).
//
// In a round the pairs partition the indices, so lane (I, J), I, J < H = np/2, owns the
// 2 x 2 block of rows {f_I, g_I} and columns {f_J, g_J}; it rotates that block and V's
// columns {f_J, g_J} on two of V's rows.  A wave holds as many matrices as fit (16 of
// order 4, 2 of order 10, one of order 16) and a round then needs no barrier, only LDS
// order; orders above 16 take H^2 threads and two barriers a round.
//
// The kernel is bound by LDS bandwidth, so the matrices are stored by slot: f_J at
// position J, g_J at H + (J - 1 mod H), rows and columns alike.  From one round to the next
// the indices move round the slots as on a conveyor (f_J -> f_{J-1}, f_1 -> g_0, g_J ->
// g_{J+1}, g_{H-1} -> f_{H-1}, f_0 stays), so a lane always reads the same addresses and
// writes its results where the next round expects them.  With this offset of the g slots
// and a row stride of H modulo 8 (in 16-byte units), bank conflicts add 22 % to the
// accesses' cycles (order 16, by counter); stored by index they added 76 %.  After a
// sweep every index is back at its first position.
//
// 64,000 matrices of order 16: 3.06 ms (parameters through LDS between two barriers,
// sorted pairs stored by index) -> 2.89 ms (pairs per lane, no barriers) -> 2.72 ms (by
// slot; LDS busy 0.76 of the time); 29,791 of order 20: 7.49 ms (row and column passes by
// one wave) -> 3.25 ms; 9,384 of order 9: 325 -> 178 us; 301 of order 16: 108 -> 75 us.
// ---------------------------------------------------------------------------
// orders whose lanes fit a wave: no barrier, but the accesses keep their order
template <int NW>
__device__ inline void eig_sync() {
    if constexpr (NW > 1) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

struct JacobiRot {
    double c, sx, sy;  // c and s e^{i phi}; (1, 0, 0) for a pair left alone
    double dlt;        // A'_ff = A_ff - dlt, A'_gg = A_gg + dlt
};

// 1 / sqrt(x) for x > 0: the hardware's estimate y (about 2^-23) and the series
// y (1 - e)^{-1/2} = y (1 + e/2 + 3 e^2/8 + ...) in its error e = 1 - x y^2, whose next
// term is below 2^-67
__device__ inline double rsqrt_pos(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// a pair (f, g); `swapped`: f > g (where d == a the sign is that of the sorted pair)
__device__ inline JacobiRot jacobi_rot(double a, double d, cd b, bool swapped, double eps2,
                                       double skip_abs) {
    const double bb2 = cabs2(b);
    const double dl = d - a;
    const double ir = rsqrt_pos(fma(dl, dl, 4.0 * bb2));
    const double cc = fma(0.5 * fabs(dl), ir, 0.5);
    const double ic = rsqrt_pos(cc);
    double s = ir * ic;
    if (dl < 0.0 || (dl == 0.0 && swapped)) s = -s;
    // A pair is left alone once |b|^2 is at the rounding level of its own diagonal
    // entries or of the mean squared diagonal entry, whichever is larger: with the first
    // test alone, pairs next to a zero eigenvalue keep rotating on rounding noise and the
    // off-diagonal norm never falls below the stopping level.
    const bool rot = bb2 > fmax(eps2 * fabs(a * d), skip_abs) && bb2 > 0.0;
    return rot ? JacobiRot{cc * ic, s * b.x, s * b.y, bb2 * (s * ic)} : JacobiRot{1.0, 0.0, 0.0, 0.0};
}

// The rotation of a sorted pair p < q in the form c, s = t c, e = e^{i phi} with
// t = sign(tau) / (|tau| + sqrt(1 + tau^2)), tau = (A_qq - A_pp) / (2 |A_pq|)
struct SortedRot {
    double c, s;
    cd e;
};
__device__ inline SortedRot sorted_rot(double a, double d, cd bpq, double eps2, double skip_abs) {
    const double bb2 = cabs2(bpq);
    if (!(bb2 > fmax(eps2 * fabs(a * d), skip_abs) && bb2 > 0.0)) return SortedRot{1.0, 0.0, {1.0, 0.0}};
    const double ib = rsqrt(bb2);
    const double tau = (d - a) * (0.5 * ib);
    const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(fma(tau, tau, 1.0)));
    const double c = rsqrt(fma(t, t, 1.0));
    return SortedRot{c, t * c, cd{bpq.x * ib, bpq.y * ib}};
}
__device__ inline void swap_if(bool sw, cd& a, cd& b) {
    // (by value: selecting between the two lvalues would put both in scratch memory)
    const double ax = a.x, ay = a.y, bx = b.x, by = b.y;
    a = cd{sw ? bx : ax, sw ? by : ay};
    b = cd{sw ? ax : bx, sw ? ay : by};
}

template <int N>
struct EigShape {
    static constexpr int NP = N + (N & 1), H = NP / 2, L = H * H;  // lanes of a matrix
    static constexpr int G = L <= 32 ? 64 / L : 1;                 // matrices of a work-group
    static constexpr int NW = (L + 63) / 64;                       // waves of a work-group
    // Where pivots are equal by the crystal's structure (CsCl: order 6), the direction of
    // a rotation, and with it the phases of the eigenvectors, hangs on the last bit.
    // Orders up to 8 therefore rotate each pair in index order, as eig_ordered_blk_kernel does
    // (the same operations; not always the same bits, the compiler contracts them differently).
    static constexpr bool SORTED = N <= 8;
    static constexpr int LD = H <= 2 ? NP : NP + (8 - H % 8) % 8;  // = H modulo 8
};

template <int N>
__global__ __launch_bounds__(64 * EigShape<N>::NW) void eig_herm_kernel(const cd* __restrict__ Aall,
                                                                        int64_t batch, int vt,
                                                                        double* __restrict__ w_out,
                                                                        cd* __restrict__ V_out) {
    using S = EigShape<N>;
    constexpr int NP = S::NP, H = S::H, L = S::L, G = S::G, NW = S::NW, LD = S::LD, m = NP - 1;
    constexpr int VO = NP * LD;  // V after A
    __shared__ cd sm[G][2 * VO];
    __shared__ int srank[G][NP];
    __shared__ double sred[2 * NW];
    __shared__ double sprm[NW > 1 ? H : 1][4];
    const int tid = threadIdx.x;
    const int64_t b0 = (int64_t)blockIdx.x * G;
    const int ng = batch - b0 < G ? (int)(batch - b0) : G;
    const cd* Ag = Aall + b0 * N * N;
    // position of index i at the start of a sweep
    auto pos = [](int i) { return i == m ? 0 : (i == 0 ? NP - 1 : (i < H ? i : 3 * H - 2 - i)); };
    for (int i = tid; i < G * NP * NP; i += 64 * NW) {  // (zeros in the padding)
        const int g = i / (NP * NP), e = i - g * NP * NP, r = e / NP, c = e - r * NP;
        const bool in = g < ng && r < N && c < N;
        sm[g][pos(r) * LD + pos(c)] = in ? Ag[(int64_t)g * N * N + r * N + c] : cd{0.0, 0.0};
        sm[g][VO + r * LD + pos(c)] = cd{r == c ? 1.0 : 0.0, 0.0};
    }
    eig_sync<NW>();
    const int g = G > 1 ? tid / L : 0;
    const int l = tid - g * L;
    const bool act = G > 1 ? g < ng : l < L;
    const int base = g * L;  // first lane of the matrix (G > 1 or one wave)
    const int I = act ? l / H : 0, J = act ? l - I * H : 0;
    cd* const A = sm[act ? g : 0];
    // slots f_k, g_k and where their contents go
    auto pf = [](int k) { return k; };
    auto pg = [](int k) { return H + (k + H - 1) % H; };
    auto nf = [&](int k) { return k == 0 ? pf(0) : (k == 1 ? pg(0) : pf(k - 1)); };
    auto ng_ = [&](int k) { return k == H - 1 ? (H == 1 ? pg(0) : pf(H - 1)) : pg(k + 1); };
    const cd* const r00 = A + pf(I) * LD + pf(J);
    const cd* const r01 = A + pf(I) * LD + pg(J);
    const cd* const r10 = A + pg(I) * LD + pf(J);
    const cd* const r11 = A + pg(I) * LD + pg(J);
    cd* const w00 = A + nf(I) * LD + nf(J);
    cd* const w01 = A + nf(I) * LD + ng_(J);
    cd* const w10 = A + ng_(I) * LD + nf(J);
    cd* const w11 = A + ng_(I) * LD + ng_(J);
    // V's rows f_I and g_I (V's rows never move: any pairing of them will do)
    cd* const v00 = A + VO + pf(I) * LD + nf(J);
    cd* const v01 = A + VO + pf(I) * LD + ng_(J);
    cd* const v10 = A + VO + pg(I) * LD + nf(J);
    cd* const v11 = A + VO + pg(I) * LD + ng_(J);
    const double eps2 = 4.9e-32;  // (2.2e-16)^2
    bool done = !act || N == 1;
    for (int sweep = 0; sweep < 40; ++sweep) {
        double off = 0.0, dia = 0.0, big = 0.0;  // big: the largest squared off-diagonal
        if (act) {
            const double a00 = cabs2(*r00), a01 = cabs2(*r01), a10 = cabs2(*r10), a11 = cabs2(*r11);
            off = a01 + a10 + (I == J ? 0.0 : a00 + a11);
            dia = I == J ? a00 + a11 : 0.0;
            big = fmax(a01, a10);
            if (I != J) big = fmax(big, fmax(a00, a11));
        }
        if constexpr (G > 1) {
            double o = 0.0, d = 0.0;
            const int bl = act ? base : 0;
#pragma unroll
            for (int t = 0; t < L; ++t) {
                o += __shfl(off, bl + t, 64);
                d += __shfl(dia, bl + t, 64);
            }
            off = o;
            dia = d;
        } else {
            off = wave_sum(off);
            dia = wave_sum(dia);
            if constexpr (NW > 1) {
                if ((tid & 63) == 0) {
                    sred[tid >> 6] = off;
                    sred[NW + (tid >> 6)] = dia;
                }
                __syncthreads();
                off = dia = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    off += sred[w];
                    dia += sred[NW + w];
                }
            }
        }
        const double skip_abs = eps2 * dia / N;
        // converged, or a sweep in which every pair would be left alone
        const bool more = off > 1e-32 * dia && big > skip_abs;
        if constexpr (NW > 1) {
            if (!__syncthreads_or(more)) break;
        } else if constexpr (G > 1) {
            const uint64_t mine = ((1ull << L) - 1ull) << base;
            done = done || !(__ballot(more) & mine);
            if (__all(done)) break;
        } else {
            if (!__any(more)) break;
        }
        // (a finished matrix sharing the wave rotates no more)
        const double skip = done ? __builtin_huge_val() : skip_abs;
        bool rotated = false;
        int fi = I == 0 ? m : I, gi = I == 0 ? 0 : m - I;  // the indices in slots f_I and g_I
        int fj = J == 0 ? m : J, gj = J == 0 ? 0 : m - J;
        for (int round = 0; round < m; ++round) {
            cd x00 = *r00, x01 = *r01, x10 = *r10, x11 = *r11;
            cd vf0 = r00[VO], vg0 = r01[VO], vf1 = r10[VO], vg1 = r11[VO];
            cd z00, z01, z10, z11;
            if constexpr (S::SORTED) {
                const bool swi = fi > gi, swj = fj > gj;
                swap_if(swi, x00, x10);
                swap_if(swi, x01, x11);
                swap_if(swj, x00, x01);
                swap_if(swj, x10, x11);
                swap_if(swj, vf0, vg0);
                swap_if(swj, vf1, vg1);
                const SortedRot rd = sorted_rot(x00.x, x11.x, x01, eps2, skip);
                const int si = base + I * (H + 1), sj = base + J * (H + 1);
                const double cI = __shfl(rd.c, si, 64), sI = __shfl(rd.s, si, 64);
                const double cJ = __shfl(rd.c, sj, 64), sJ = __shfl(rd.s, sj, 64);
                const cd eI = {__shfl(rd.e.x, si, 64), __shfl(rd.e.y, si, 64)};
                const cd eJ = {__shfl(rd.e.x, sj, 64), __shfl(rd.e.y, sj, 64)};
                rotated = rotated || sI != 0.0;
                if (sI != 0.0) {
                    const cd e0 = cmul(eI, x10), e1 = cmul(eI, x11);
                    const cd f0 = cmulc(eI, x00), f1 = cmulc(eI, x01);
                    x00 = cd{cI * x00.x - sI * e0.x, cI * x00.y - sI * e0.y};
                    x01 = cd{cI * x01.x - sI * e1.x, cI * x01.y - sI * e1.y};
                    x10 = cd{sI * f0.x + cI * x10.x, sI * f0.y + cI * x10.y};
                    x11 = cd{sI * f1.x + cI * x11.x, sI * f1.y + cI * x11.y};
                }
                z00 = vf0;
                z01 = vg0;
                z10 = vf1;
                z11 = vg1;
                if (sJ != 0.0) {
                    const cd e0 = cmulc(eJ, x01), e1 = cmulc(eJ, x11);
                    const cd f0 = cmul(eJ, x00), f1 = cmul(eJ, x10);
                    x00 = cd{cJ * x00.x - sJ * e0.x, cJ * x00.y - sJ * e0.y};
                    x10 = cd{cJ * x10.x - sJ * e1.x, cJ * x10.y - sJ * e1.y};
                    x01 = cd{sJ * f0.x + cJ * x01.x, sJ * f0.y + cJ * x01.y};
                    x11 = cd{sJ * f1.x + cJ * x11.x, sJ * f1.y + cJ * x11.y};
                    const cd q0 = cmulc(eJ, vg0), p0 = cmul(eJ, vf0);
                    const cd q1 = cmulc(eJ, vg1), p1 = cmul(eJ, vf1);
                    z00 = cd{cJ * vf0.x - sJ * q0.x, cJ * vf0.y - sJ * q0.y};
                    z01 = cd{sJ * p0.x + cJ * vg0.x, sJ * p0.y + cJ * vg0.y};
                    z10 = cd{cJ * vf1.x - sJ * q1.x, cJ * vf1.y - sJ * q1.y};
                    z11 = cd{sJ * p1.x + cJ * vg1.x, sJ * p1.y + cJ * vg1.y};
                }
                if (I == J && sI != 0.0) {  // the rotated pair: exact zero off the diagonal
                    x01 = x10 = cd{0.0, 0.0};
                    x00.y = x11.y = 0.0;
                }
                swap_if(swj, x00, x01);
                swap_if(swj, x10, x11);
                swap_if(swi, x00, x10);
                swap_if(swi, x01, x11);
                swap_if(swj, z00, z01);
                swap_if(swj, z10, z11);
            } else {
                // in lane (I, I) the block is the pair's own
                const JacobiRot rd = jacobi_rot(x00.x, x11.x, x01, fi > gi, eps2, skip);
                JacobiRot ri, rj;
                if constexpr (NW == 1) {
                    const int si = base + I * (H + 1), sj = base + J * (H + 1);
                    ri = JacobiRot{__shfl(rd.c, si, 64), __shfl(rd.sx, si, 64), __shfl(rd.sy, si, 64), 0.0};
                    rj = JacobiRot{__shfl(rd.c, sj, 64), __shfl(rd.sx, sj, 64), __shfl(rd.sy, sj, 64), 0.0};
                } else {
                    if (act && I == J) {
                        sprm[I][0] = rd.c;
                        sprm[I][1] = rd.sx;
                        sprm[I][2] = rd.sy;
                    }
                    __syncthreads();  // (and every block has been read)
                    ri = JacobiRot{sprm[I][0], sprm[I][1], sprm[I][2], 0.0};
                    rj = JacobiRot{sprm[J][0], sprm[J][1], sprm[J][2], 0.0};
                }
                const bool any = ri.sx != 0.0 || ri.sy != 0.0;
                rotated = rotated || any;
                // rows: A'_f = c A_f - s e A_g ; A'_g = s conj(e) A_f + c A_g
                auto rot_f = [](double c, double sx, double sy, cd u, cd w) {  // c u - s w
                    return cd{fma(c, u.x, fma(sy, w.y, -sx * w.x)), fma(c, u.y, -fma(sx, w.y, sy * w.x))};
                };
                auto rot_g = [](double c, double sx, double sy, cd u, cd w) {  // conj(s) u + c w
                    return cd{fma(c, w.x, fma(sy, u.y, sx * u.x)), fma(c, w.y, fma(sx, u.y, -sy * u.x))};
                };
                const double af = x00.x - rd.dlt, ag = x11.x + rd.dlt;
                const cd y00 = rot_f(ri.c, ri.sx, ri.sy, x00, x10), y01 = rot_f(ri.c, ri.sx, ri.sy, x01, x11);
                const cd y10 = rot_g(ri.c, ri.sx, ri.sy, x00, x10), y11 = rot_g(ri.c, ri.sx, ri.sy, x01, x11);
                // columns: A'_f = c A_f - s conj(e) A_g ; A'_g = s e A_f + c A_g ; V the same
                x00 = rot_f(rj.c, rj.sx, -rj.sy, y00, y01);
                x01 = rot_g(rj.c, rj.sx, -rj.sy, y00, y01);
                x10 = rot_f(rj.c, rj.sx, -rj.sy, y10, y11);
                x11 = rot_g(rj.c, rj.sx, -rj.sy, y10, y11);
                // the rotated pair: exact zero off the diagonal, and a diagonal changed by t |A_fg|
                // only: multiplied by c^2 and s^2 it would gather their rounding at every rotation
                if (I == J && any) {
                    x01 = x10 = cd{0.0, 0.0};
                    x00 = cd{af, 0.0};
                    x11 = cd{ag, 0.0};
                }
                z00 = rot_f(rj.c, rj.sx, -rj.sy, vf0, vg0);
                z01 = rot_g(rj.c, rj.sx, -rj.sy, vf0, vg0);
                z10 = rot_f(rj.c, rj.sx, -rj.sy, vf1, vg1);
                z11 = rot_g(rj.c, rj.sx, -rj.sy, vf1, vg1);
            }
            if constexpr (NW == 1) eig_sync<1>();  // (reads before writes)
            if (act) {
                *w00 = x00;
                *w01 = x01;
                *w10 = x10;
                *w11 = x11;
                *v00 = z00;
                *v01 = z01;
                *v10 = z10;
                *v11 = z11;
            }
            eig_sync<NW>();
            // the next round's pairs
            if (I > 0 && ++fi == m) fi = 0;
            if (++gi == m) gi = 0;
            if constexpr (S::SORTED) {
                if (J > 0 && ++fj == m) fj = 0;
                if (++gj == m) gj = 0;
            }
        }
        // a sweep with no rotation leaves the matrix unchanged
        if constexpr (NW > 1) {
            if (!__syncthreads_or(rotated)) break;
        } else if constexpr (G > 1) {
            const uint64_t mine = ((1ull << L) - 1ull) << base;
            done = done || !(__ballot(rotated) & mine);
        } else {
            if (!__any(rotated)) break;
        }
    }
    // ascending order, ties by index
    if (act) {
        for (int i = l; i < N; i += L) {
            const double wi = A[pos(i) * (LD + 1)].x;
            int rank = 0;
            for (int j = 0; j < N; ++j) {
                const double wj = A[pos(j) * (LD + 1)].x;
                rank += (wj < wi) || (wj == wi && j < i);
            }
            srank[g][i] = rank;
            w_out[(b0 + g) * N + rank] = wi;
        }
    }
    eig_sync<NW>();
    cd* Vg = V_out + b0 * N * N;
    for (int i = tid; i < ng * N * N; i += 64 * NW) {
        const int q = i / (N * N), e = i - q * N * N, r = e / N, c = e - r * N;
        const int rank = srank[q][c];
        Vg[(int64_t)q * N * N + (vt ? rank * N + r : r * N + rank)] = sm[q][VO + r * LD + pos(c)];
    }
}

template <int N>
static hipError_t go_eig(const cd* A, int64_t batch, bool vt, double* w, cd* V, hipStream_t s) {
    constexpr int G = EigShape<N>::G;
    const int64_t chunk = 1000000000LL / G * G;
    for (int64_t b = 0; b < batch; b += chunk) {
        const int64_t nb = batch - b < chunk ? batch - b : chunk;
        hipLaunchKernelGGL(eig_herm_kernel<N>, dim3((unsigned)((nb + G - 1) / G)),
                           dim3(64 * EigShape<N>::NW), 0, s, A + b * N * N, nb, vt ? 1 : 0, w + b * N,
                           V + b * N * N);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The eigensolver for modes that are handed out at any q: cyclic Jacobi on sorted pairs,
// one wavefront per matrix.  Near Gamma the acoustic modes' eigenvalues lie within 1e-8 of
// each other against the largest (a path's first q: 1e-4 eV of 0.16 eV), and another order
// of the same operations turns those modes into one another by 1e-8 and more, in amplitudes
// that a program compares with those it saved.  This form keeps the order and the rounding
// that such programs have.  Order 15, 201 matrices: 124 us, 66 us by eig_herm_kernel, which
// takes everything that sums over the modes.
// ---------------------------------------------------------------------------
__device__ inline void rr_pair(int k, int round, int np, int& p, int& q) {
    const int m = np - 1;
    int a, b;
    if (k == 0) {
        a = m;
        b = round;
    } else {
        a = (round + k) % m;
        b = (round - k + m) % m;
    }
    p = a < b ? a : b;
    q = a < b ? b : a;
}

// Without VEC the rotations of V and its store are left out: the eigenvalues are the same bits.
// Four waves share a matrix (orders 18 to 30): every element's operations are those of one
// wave, and the sums behind the stopping test are taken by one wave in its order.  A round
// waits on its passes over the rows and columns, 8 and 15 trips of one wave at order 30:
// modes of 300 q, 30 of them, 1331 us with one wave, 609 with four; 3,000 q 4038 and 2206 us.
constexpr int kOrdThreads = 256;
template <int NT, bool VEC>
__global__ __launch_bounds__(kOrdThreads) void eig_ordered_kernel(cd* __restrict__ Aall,
                                                                  double* __restrict__ w_out,
                                                                  cd* __restrict__ V_out) {
    constexpr int n = NT, NTH = kOrdThreads;
    __shared__ double norms[2];
    extern __shared__ char smem_raw[];
    cd* A = reinterpret_cast<cd*>(smem_raw);
    // odd row stride: 16 lanes walking down a column of 16-byte elements hit 16
    // distinct 4-bank groups (an even stride such as 16 would serialise them)
    const int ld = n | 1;
    cd* V = A + n * ld;  // VEC
    double* rc = reinterpret_cast<double*>(A + (VEC ? 2 : 1) * n * ld);  // [n/2+1] c
    double* rs = rc + (n / 2 + 1);                         // s
    cd* re = reinterpret_cast<cd*>(rs + (n / 2 + 1));      // e^{i phi}
    int* rp = reinterpret_cast<int*>(re + (n / 2 + 1));    // p
    int* rq = rp + (n / 2 + 1);                            // q
    const int64_t b = blockIdx.x;
    const int lane = threadIdx.x;  // (of the work-group)
    cd* Ag = Aall + b * (int64_t)n * n;
    for (int i = lane; i < n * n; i += NTH) {
        const int r = i / n, c = i % n;
        A[r * ld + c] = Ag[i];
        if constexpr (VEC) V[r * ld + c] = cd{r == c ? 1.0 : 0.0, 0.0};
    }
    __syncthreads();
    const int np = n + (n & 1);
    const int half = np / 2;
    const double eps2 = 4.9e-32;  // (2.2e-16)^2
    for (int sweep = 0; sweep < 40 && n > 1; ++sweep) {
        int rotated = 0;
        if (lane < 64) {
            double off = 0.0, dia = 0.0;
            for (int i = lane; i < n * n; i += 64) {
                const int r = i / n, c = i % n;
                const double v = cabs2(A[r * ld + c]);
                if (r == c)
                    dia += v;
                else
                    off += v;
            }
            off = wave_sum(off);
            dia = wave_sum(dia);
            if (lane == 0) {
                norms[0] = off;
                norms[1] = dia;
            }
        }
        __syncthreads();
        const double off = norms[0], dia = norms[1];
        if (!(off > 1e-32 * dia)) break;
        // A pair is left alone once |A_pq|^2 is at the rounding level of its own diagonal
        // entries or of the mean squared diagonal entry, whichever is larger: with the
        // first test alone, pairs next to a zero eigenvalue keep rotating on rounding noise
        // and the off-diagonal norm never falls below the stopping level above.
        const double skip_abs = eps2 * dia / n;
        for (int round = 0; round < np - 1; ++round) {
            if (lane < half) {
                int p, q;
                rr_pair(lane, round, np, p, q);
                double c = 1.0, s = 0.0;
                cd e = {1.0, 0.0};
                if (q < n) {
                    const double a = A[p * ld + p].x, d = A[q * ld + q].x;
                    const cd bpq = A[p * ld + q];
                    const double bb2 = cabs2(bpq);
                    if (bb2 > fmax(eps2 * fabs(a * d), skip_abs) && bb2 > 0.0) {
                        rotated = 1;
                        // (one reciprocal square root for 1/|b|, one for c: two
                        // divisions and a square root fewer on the round's critical path)
                        const double ib = rsqrt(bb2);
                        const double tau = (d - a) * (0.5 * ib);
                        const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(fma(tau, tau, 1.0)));
                        c = rsqrt(fma(t, t, 1.0));
                        s = t * c;
                        e = cd{bpq.x * ib, bpq.y * ib};
                    }
                }
                rc[lane] = c;
                rs[lane] = s;
                re[lane] = e;
                rp[lane] = p;
                rq[lane] = q < n ? q : -1;
            }
            __syncthreads();
            // rows: A'_pj = c A_pj - s e A_qj ; A'_qj = s conj(e) A_pj + c A_qj
            for (int it = lane; it < half * n; it += NTH) {
                const int k = it / n, j = it % n;
                const int q = rq[k];
                if (q < 0 || rs[k] == 0.0) continue;
                const int p = rp[k];
                const double c = rc[k], s = rs[k];
                const cd e = re[k];
                const cd apj = A[p * ld + j], aqj = A[q * ld + j];
                const cd eq = cmul(e, aqj);
                const cd ep = cmulc(e, apj);
                A[p * ld + j] = cd{c * apj.x - s * eq.x, c * apj.y - s * eq.y};
                A[q * ld + j] = cd{s * ep.x + c * aqj.x, s * ep.y + c * aqj.y};
            }
            __syncthreads();
            // columns: A'_ip = c A_ip - s conj(e) A_iq ; A'_iq = s e A_ip + c A_iq ; same for V
            for (int it = lane; it < (VEC ? 2 : 1) * half * n; it += NTH) {
                const int which = it / (half * n);
                const int r = it % (half * n);
                const int k = r / n, i = r % n;
                const int q = rq[k];
                if (q < 0 || rs[k] == 0.0) continue;
                const int p = rp[k];
                const double c = rc[k], s = rs[k];
                const cd e = re[k];
                cd* M = which ? V : A;
                const cd aip = M[i * ld + p], aiq = M[i * ld + q];
                const cd eq = cmulc(e, aiq);
                const cd ep = cmul(e, aip);
                M[i * ld + p] = cd{c * aip.x - s * eq.x, c * aip.y - s * eq.y};
                M[i * ld + q] = cd{s * ep.x + c * aiq.x, s * ep.y + c * aiq.y};
            }
            __syncthreads();
            if (lane < half) {
                const int q = rq[lane];
                if (q >= 0 && rs[lane] != 0.0) {
                    const int p = rp[lane];
                    A[p * ld + q] = cd{0.0, 0.0};
                    A[q * ld + p] = cd{0.0, 0.0};
                    A[p * ld + p].y = 0.0;
                    A[q * ld + q].y = 0.0;
                }
            }
            __syncthreads();
        }
        if (!__syncthreads_or(rotated)) break;  // a sweep with no rotation leaves A unchanged
    }
    // ascending order, ties by index
    for (int i = lane; i < n; i += NTH) {
        const double wi = A[i * ld + i].x;
        int rank = 0;
        for (int j = 0; j < n; ++j) {
            const double wj = A[j * ld + j].x;
            rank += (wj < wi) || (wj == wi && j < i);
        }
        w_out[b * n + rank] = wi;
        if constexpr (VEC) {
            cd* Vg = V_out + b * (int64_t)n * n;
            for (int r = 0; r < n; ++r) Vg[r * n + rank] = V[r * ld + i];
        }
    }
}

// The same Jacobi method for n <= 16 with the work of a round split by 2 x 2
// blocks: in a round the pairs partition the indices, so lane (I, J) (I, J <
// n/2 rounded up) owns the block of rows {p_I, q_I} and columns {p_J, q_J}.
// The two-sided rotation of that block reads only the block (rows by pair I,
// then columns by pair J), and so does the column rotation of V on rows
// {2I, 2I + 1}: every lane reads, rotates and writes its own elements, and a
// round needs one barrier after the parameters and one after the update.
// The pair order, the skip test and the stopping rule are those above.
template <int NT, bool VEC>
__global__ __launch_bounds__(64) void eig_ordered_blk_kernel(const cd* __restrict__ Aall, int vt,
                                                          double* __restrict__ w_out,
                                                          cd* __restrict__ V_out) {
    constexpr int n = NT;
    constexpr int LD = 17;  // odd row stride (see above)
    __shared__ cd A[16 * LD], V[VEC ? 16 * LD : 1];
    __shared__ double prm[8][4];  // c, s, e of every pair of the round
    const int64_t b = blockIdx.x;
    const int lane = threadIdx.x;
    const int I = lane >> 3, J = lane & 7;
    const int np = n + (n & 1), half = np / 2;
    const bool act = I < half && J < half;
    const cd* Ag = Aall + b * (int64_t)n * n;
    for (int i = lane; i < n * n; i += 64) {
        const int r = i / n, c = i - r * n;
        A[r * LD + c] = Ag[i];
        if constexpr (VEC) V[r * LD + c] = cd{r == c ? 1.0 : 0.0, 0.0};
    }
    __syncthreads();
    const double eps2 = 4.9e-32;  // (2.2e-16)^2
    for (int sweep = 0; sweep < 40 && n > 1; ++sweep) {
        double off = 0.0, dia = 0.0;
        for (int i = lane; i < n * n; i += 64) {
            const int r = i / n, c = i - r * n;
            const double v = cabs2(A[r * LD + c]);
            if (r == c)
                dia += v;
            else
                off += v;
        }
        off = wave_sum(off);
        dia = wave_sum(dia);
        if (!(off > 1e-32 * dia)) break;
        const double skip_abs = eps2 * dia / n;
        int rotated = 0;
        for (int round = 0; round < np - 1; ++round) {
            if (lane < half) {
                int p, q;
                rr_pair(lane, round, np, p, q);
                double c = 1.0, s = 0.0;
                cd e = {1.0, 0.0};
                if (q < n) {
                    const double a = A[p * LD + p].x, d = A[q * LD + q].x;
                    const cd bpq = A[p * LD + q];
                    const double bb2 = cabs2(bpq);
                    if (bb2 > fmax(eps2 * fabs(a * d), skip_abs) && bb2 > 0.0) {
                        rotated = 1;
                        // (one reciprocal square root for 1/|b|, one for c: two
                        // divisions and a square root fewer on the round's critical path)
                        const double ib = rsqrt(bb2);
                        const double tau = (d - a) * (0.5 * ib);
                        const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(fma(tau, tau, 1.0)));
                        c = rsqrt(fma(t, t, 1.0));
                        s = t * c;
                        e = cd{bpq.x * ib, bpq.y * ib};
                    }
                }
                prm[lane][0] = c;
                prm[lane][1] = s;
                prm[lane][2] = e.x;
                prm[lane][3] = e.y;
            }
            __syncthreads();
            if (act) {
                int pI, qI, pJ, qJ;
                rr_pair(I, round, np, pI, qI);
                rr_pair(J, round, np, pJ, qJ);
                const double cI = prm[I][0], sI = prm[I][1], cJ = prm[J][0], sJ = prm[J][1];
                const cd eI = {prm[I][2], prm[I][3]}, eJ = {prm[J][2], prm[J][3]};
                const bool qIok = qI < n, qJok = qJ < n;
                if (sI != 0.0 || sJ != 0.0) {
                    const cd z = {0.0, 0.0};
                    cd x00 = A[pI * LD + pJ];
                    cd x01 = qJok ? A[pI * LD + qJ] : z;
                    cd x10 = qIok ? A[qI * LD + pJ] : z;
                    cd x11 = qIok && qJok ? A[qI * LD + qJ] : z;
                    if (sI != 0.0) {  // rows: A'_p = c A_p - s e A_q ; A'_q = s conj(e) A_p + c A_q
                        const cd e0 = cmul(eI, x10), e1 = cmul(eI, x11);
                        const cd f0 = cmulc(eI, x00), f1 = cmulc(eI, x01);
                        x00 = cd{cI * x00.x - sI * e0.x, cI * x00.y - sI * e0.y};
                        x01 = cd{cI * x01.x - sI * e1.x, cI * x01.y - sI * e1.y};
                        x10 = cd{sI * f0.x + cI * x10.x, sI * f0.y + cI * x10.y};
                        x11 = cd{sI * f1.x + cI * x11.x, sI * f1.y + cI * x11.y};
                    }
                    if (sJ != 0.0) {  // columns: A'_ip = c A_ip - s conj(e) A_iq ; A'_iq = s e A_ip + c A_iq
                        const cd e0 = cmulc(eJ, x01), e1 = cmulc(eJ, x11);
                        const cd f0 = cmul(eJ, x00), f1 = cmul(eJ, x10);
                        x00 = cd{cJ * x00.x - sJ * e0.x, cJ * x00.y - sJ * e0.y};
                        x10 = cd{cJ * x10.x - sJ * e1.x, cJ * x10.y - sJ * e1.y};
                        x01 = cd{sJ * f0.x + cJ * x01.x, sJ * f0.y + cJ * x01.y};
                        x11 = cd{sJ * f1.x + cJ * x11.x, sJ * f1.y + cJ * x11.y};
                    }
                    if (I == J && sI != 0.0) {  // the rotated pair: exact zero off the diagonal
                        x01 = z;
                        x10 = z;
                        x00.y = 0.0;
                        x11.y = 0.0;
                    }
                    A[pI * LD + pJ] = x00;
                    if (qJok) A[pI * LD + qJ] = x01;
                    if (qIok) A[qI * LD + pJ] = x10;
                    if (qIok && qJok) A[qI * LD + qJ] = x11;
                }
                if (VEC && sJ != 0.0) {  // V columns p_J, q_J on rows 2I, 2I + 1
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int r = 2 * I + h;
                        if (r < n) {
                            const cd vp = V[r * LD + pJ];
                            const cd vq = qJok ? V[r * LD + qJ] : cd{0.0, 0.0};
                            const cd eq = cmulc(eJ, vq), ep = cmul(eJ, vp);
                            V[r * LD + pJ] = cd{cJ * vp.x - sJ * eq.x, cJ * vp.y - sJ * eq.y};
                            if (qJok) V[r * LD + qJ] = cd{sJ * ep.x + cJ * vq.x, sJ * ep.y + cJ * vq.y};
                        }
                    }
                }
            }
            __syncthreads();
        }
        if (!__any(rotated)) break;  // a sweep with no rotation leaves A unchanged
    }
    // ascending order, ties by index
    for (int i = lane; i < n; i += 64) {
        const double wi = A[i * LD + i].x;
        int rank = 0;
        for (int j = 0; j < n; ++j) {
            const double wj = A[j * LD + j].x;
            rank += (wj < wi) || (wj == wi && j < i);
        }
        w_out[b * n + rank] = wi;
        if constexpr (VEC) {
            cd* Vg = V_out + b * (int64_t)n * n;
            for (int r = 0; r < n; ++r) Vg[vt ? rank * n + r : r * n + rank] = V[r * LD + i];
        }
    }
}

template <bool VEC>
static hipError_t go_eig_ordered(cd* A, int n, int64_t batch, double* w, cd* V, hipStream_t s) {
    const int h = n / 2 + 1;
    const size_t shm = (size_t)(VEC ? 2 : 1) * n * (n | 1) * sizeof(cd) + 2 * h * sizeof(double) +
                       h * sizeof(cd) + 2 * h * sizeof(int);
    for (int64_t b0 = 0; b0 < batch; b0 += 2000000000LL) {
        const int64_t nb = batch - b0 < 2000000000LL ? batch - b0 : 2000000000LL;
        cd* Ab = A + b0 * n * n;
        double* wb = w + b0 * n;
        cd* Vb = VEC ? V + b0 * n * n : nullptr;
        switch (n) {
#define PHX_EIG(NV)                                                                                 \
    case NV:                                                                                        \
        hipLaunchKernelGGL((eig_ordered_kernel<NV, VEC>), dim3((unsigned)nb), dim3(kOrdThreads),    \
                           shm, s, Ab, wb, Vb);                                                     \
        break;
#define PHX_EIGB(NV)                                                                                \
    case NV:                                                                                        \
        hipLaunchKernelGGL((eig_ordered_blk_kernel<NV, VEC>), dim3((unsigned)nb), dim3(64), 0, s,   \
                           Ab, 0, wb, Vb);                                                          \
        break;
            PHX_EIGB(3) PHX_EIGB(6) PHX_EIGB(9) PHX_EIGB(12) PHX_EIGB(15)
            PHX_EIG(18) PHX_EIG(21) PHX_EIG(24) PHX_EIG(27) PHX_EIG(30)
#undef PHX_EIG
#undef PHX_EIGB
            default: return hipErrorInvalidValue;  // (three modes an atom, ten atoms)
        }
    }
    return hipGetLastError();
}

hipError_t launch_eig_herm_ordered(cd* A, int n, int64_t batch, double* w, cd* V, hipStream_t s) {
    if (batch <= 0) return hipSuccess;
    return V ? go_eig_ordered<true>(A, n, batch, w, V, s) : go_eig_ordered<false>(A, n, batch, w, V, s);
}

hipError_t launch_eig_herm(const cd* A, int n, int64_t batch, double* w, cd* V, bool vt,
                           hipStream_t s) {
    if (batch <= 0) return hipSuccess;
    // Orders 4 to 8 of no more matrices than the chip has SIMDs (1,024; odd orders, where a
    // pair is idle, a quarter of that): a wave for each, by the block kernel.  There a round's
    // latency counts, and the pair swaps of EigShape::SORTED lengthen it: 216 matrices of
    // order 4, 6, 8: 14.8, 26.0, 42.9 us, 18.9, 35.2, 49.6 several to a wave; 1,024: 17.7, 28.5,
    // 47.5 and 19.2, 35.8, 50.5; 1,280: 20.2, 34.6, 57.4 and 19.2, 36.1, 52.2.
    if (batch <= (n & 1 ? 256 : 1024)) {
        const int t = vt ? 1 : 0;
        switch (n) {
#define PHX_EIG(NV)                                                                                  \
    case NV:                                                                                         \
        hipLaunchKernelGGL((eig_ordered_blk_kernel<NV, true>), dim3((unsigned)batch), dim3(64), 0, s, A, \
                           t, w, V);                                                                 \
        return hipGetLastError();
            PHX_EIG(4) PHX_EIG(5) PHX_EIG(6) PHX_EIG(7) PHX_EIG(8)
#undef PHX_EIG
            default: break;
        }
    }
    switch (n) {
#define PHX_EIG(NV) \
    case NV: return go_eig<NV>(A, batch, vt, w, V, s);
        PHX_EIG(1) PHX_EIG(2) PHX_EIG(3) PHX_EIG(4) PHX_EIG(5) PHX_EIG(6) PHX_EIG(7) PHX_EIG(8)
        PHX_EIG(9) PHX_EIG(10) PHX_EIG(11) PHX_EIG(12) PHX_EIG(13) PHX_EIG(14) PHX_EIG(15)
        PHX_EIG(16) PHX_EIG(17) PHX_EIG(18) PHX_EIG(19) PHX_EIG(20) PHX_EIG(21) PHX_EIG(22)
        PHX_EIG(23) PHX_EIG(24) PHX_EIG(25) PHX_EIG(26) PHX_EIG(27) PHX_EIG(28) PHX_EIG(29)
        PHX_EIG(30) PHX_EIG(31) PHX_EIG(32)
#undef PHX_EIG
        default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------
// Phonon post-processing and occupations
// ---------------------------------------------------------------------------
// A wave per point, its lanes along the rows of E, which are written in whole cache lines; z
// is read down its columns, a few KB that stay in L1.  64,000 points, 15 modes: 117 us, 252 with
// a thread per (point, mode) walking a row of E.
__global__ __launch_bounds__(64) void phonon_post_kernel(const double* lam, const cd* z, const double* mass,
                                                         int nat, int64_t nq, double omega_min, double kT,
                                                         double c_om, double c_ph, double* omega, cd* e,
                                                         double* nb) {
    const int nm = 3 * nat, per_q = e ? nm * nm : nm;
    for (int64_t q = blockIdx.x; q < nq; q += gridDim.x) {
        for (int i = threadIdx.x; i < per_q; i += 64) {
            const int nu = e ? i / nm : i, sa = e ? i - nu * nm : 0;
            const int64_t t = q * nm + nu;
            const double l = lam[t];
            const double w = c_om * sqrt(l > 0.0 ? l : 0.0);
            const bool act = w >= omega_min && w > 0.0;
            if (sa == 0) {
                if (omega) omega[t] = w;
                if (nb) nb[t] = (act && kT > 0.0) ? 1.0 / expm1(w / kT) : 0.0;
            }
            if (!e) continue;
            // E[q, nu, sa] = z[q][sa][nu] l_{sa,nu}
            cd v = {0.0, 0.0};
            if (act) {
                const cd zv = z[(q * nm + sa) * nm + nu];
                const double ls = sqrt(c_ph / (2.0 * mass[sa / 3] * w));
                v = cd{zv.x * ls, zv.y * ls};
            }
            e[t * nm + sa] = v;
        }
    }
}

hipError_t launch_phonon_post(const double* lam, const cd* z, const double* mass, int nat,
                              int64_t nq, double omega_min, double kT, double* omega, cd* e,
                              double* nb, hipStream_t s) {
    if (nq <= 0) return hipSuccess;
    const unsigned groups = (unsigned)(nq < (1 << 20) ? nq : (1 << 20));
    hipLaunchKernelGGL(phonon_post_kernel, dim3(groups), dim3(64), 0, s, lam, z, mass, nat, nq, omega_min,
                       kT, c_omega(), kCPh, omega, e, nb);
    return hipGetLastError();
}

__global__ void fermi_kernel(const double* eps, int64_t n, double mu, double kT, double* f) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x) {
        const double x = (eps[t] - mu) / kT;
        if (x > 0.0) {
            const double ex = exp(-x);
            f[t] = ex / (1.0 + ex);
        } else {
            f[t] = 1.0 / (1.0 + exp(x));
        }
    }
}

hipError_t launch_fermi(const double* eps, int64_t n, double mu, double kT, double* f,
                        hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fermi_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, eps, n, mu, kT, f);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Window, ordered compaction, band extrema
// ---------------------------------------------------------------------------
__global__ void window_kernel(const double* eps, int64_t nk, int nW, double lo, double hi,
                              uint8_t* mask, int32_t* flag) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < nk;
         k += (int64_t)gridDim.x * blockDim.x) {
        int any = 0;
        for (int b = 0; b < nW; ++b) {
            const double e = eps[k * nW + b];
            const int in = (e > lo) && (e < hi);
            if (mask) mask[k * nW + b] = (uint8_t)in;
            any |= in;
        }
        if (flag) flag[k] = any;
    }
}

hipError_t launch_window(const double* eps, int64_t nk, int nW, double lo, double hi,
                         uint8_t* mask, int32_t* flag, hipStream_t s) {
    if (nk <= 0) return hipSuccess;
    hipLaunchKernelGGL(window_kernel, dim3(grid_for(nk, 256)), dim3(256), 0, s, eps, nk, nW, lo,
                       hi, mask, flag);
    return hipGetLastError();
}

// One work-group of 1024 threads scans the flags chunk by chunk in order.
__global__ __launch_bounds__(1024) void compact_kernel(const int32_t* flag, int64_t n, int32_t* out,
                                                        int32_t* count) {
    __shared__ int32_t wsum[16];
    __shared__ int32_t base_sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) base_sh = 0;
    __syncthreads();
    for (int64_t c0 = 0; c0 < n; c0 += 1024) {
        const int64_t i = c0 + tid;
        const int f = (i < n && flag[i] != 0) ? 1 : 0;
        // inclusive scan within the wave
        int v = f;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int u = __shfl_up(v, o, 64);
            if (lane >= o) v += u;
        }
        if (lane == 63) wsum[wave] = v;
        __syncthreads();
        int before = 0;
        for (int w = 0; w < wave; ++w) before += wsum[w];
        const int base = base_sh;
        if (f) out[base + before + v - 1] = (int32_t)i;
        __syncthreads();
        if (tid == 1023) base_sh = base + before + v;
        __syncthreads();
    }
    if (tid == 0) *count = base_sh;
}

hipError_t launch_compact(const int32_t* flag, int64_t n, int32_t* out, int32_t* count,
                          hipStream_t s) {
    hipLaunchKernelGGL(compact_kernel, dim3(1), dim3(1024), 0, s, flag, n, out, count);
    return hipGetLastError();
}

// min and max are exact in any order; the loads of a thread are unrolled so that
// eight are in flight at once
__global__ __launch_bounds__(1024) void extrema_kernel(const double* eps, int64_t nk, int nW,
                                                       const double* omega, int64_t nq, int nm,
                                                       double* bmin, double* bmax, double* wmax) {
    __shared__ double s1[1024], s2[1024];
    const int b = blockIdx.x;  // b < nW: band b; b == nW: phonon maximum
    double lo = 1e300, hi = -1e300;
    if (b < nW) {
#pragma unroll 8
        for (int64_t k = threadIdx.x; k < nk; k += 1024) {
            const double e = eps[k * nW + b];
            lo = fmin(lo, e);
            hi = fmax(hi, e);
        }
    } else {
#pragma unroll 8
        for (int64_t t = threadIdx.x; t < nq * nm; t += 1024) hi = fmax(hi, omega[t]);
    }
    s1[threadIdx.x] = lo;
    s2[threadIdx.x] = hi;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            s1[threadIdx.x] = fmin(s1[threadIdx.x], s1[threadIdx.x + o]);
            s2[threadIdx.x] = fmax(s2[threadIdx.x], s2[threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (b < nW) {
            bmin[b] = s1[0];
            bmax[b] = s2[0];
        } else {
            *wmax = s2[0];
        }
    }
}

hipError_t launch_band_extrema(const double* eps, int64_t nk, int nW, const double* omega,
                               int64_t nq, int nm, double* bmin, double* bmax, double* wmax,
                               hipStream_t s) {
    hipLaunchKernelGGL(extrema_kernel, dim3(nW + 1), dim3(1024), 0, s, eps, nk, nW, omega, nq, nm,
                       bmin, bmax, wmax);
    return hipGetLastError();
}

__global__ void kq_kernel(const double* k, int64_t nk, const double* q, int64_t nq, double* kq) {
    const int64_t total = nk * nq;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = t / nq, j = t % nq;
        for (int d = 0; d < 3; ++d) kq[3 * t + d] = k[3 * i + d] + q[3 * j + d];
    }
}

hipError_t launch_kq_points(const double* k, int64_t nk, const double* q, int64_t nq,
                            double* kq, hipStream_t s) {
    if (nk * nq <= 0) return hipSuccess;
    hipLaunchKernelGGL(kq_kernel, dim3(grid_for(nk * nq, 256)), dim3(256), 0, s, k, nk, q, nq, kq);
    return hipGetLastError();
}

// Bands at k + q for k and q on one mesh: the mesh's bands gathered per pair.
// Pair (i, j) of k index k_idx[i] and q index j takes mesh point
// ((k0 + q0) mod N0, (k1 + q1) mod N1, (k2 + q2) mod N2); one thread per (pair, entry).
__global__ void gather_kq_bands_kernel(const double* __restrict__ eps, const cd* __restrict__ U,
                                       int nW, Mesh m, const int32_t* __restrict__ k_idx,
                                       int64_t nk, int64_t nq, double* __restrict__ eps_kq,
                                       cd* __restrict__ Ukq) {
    const int64_t per = (int64_t)nW + (int64_t)nW * nW;
    const int64_t total = nk * nq * per;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t pair = t / per;
        const int64_t e = t - pair * per;
        const int64_t i = pair / nq, j = pair - i * nq;
        int k0, k1, k2, q0, q1, q2;
        mesh_triple(k_idx[i], m, k0, k1, k2);
        mesh_triple(j, m, q0, q1, q2);
        const int64_t kq = mesh_linear((k0 + q0) % m.n0, (k1 + q1) % m.n1, (k2 + q2) % m.n2, m);
        if (e < nW)
            eps_kq[pair * nW + e] = eps[kq * nW + e];
        else
            Ukq[pair * nW * nW + (e - nW)] = U[kq * nW * nW + (e - nW)];
    }
}

hipError_t launch_gather_kq_bands(const double* eps, const cd* U, int nW, Mesh m,
                                  const int32_t* k_idx, int64_t nk, int64_t nq, double* eps_kq,
                                  cd* Ukq, hipStream_t s) {
    if (nk * nq <= 0) return hipSuccess;
    const int64_t total = nk * nq * ((int64_t)nW + (int64_t)nW * nW);
    hipLaunchKernelGGL(gather_kq_bands_kernel, dim3(grid_for(total, 256)), dim3(256), 0, s, eps, U,
                       nW, m, k_idx, nk, nq, eps_kq, Ukq);
    return hipGetLastError();
}

// Fill with zeros by a kernel (safe under stream capture).
__global__ void zero_kernel(uint32_t* p, int64_t n, uint8_t* tail, int ntail) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x)
        p[t] = 0u;
    if (blockIdx.x == 0 && (int)threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    // buffers come from the workspace or the caller and are at least 4-byte aligned
    const int64_t n = (int64_t)(bytes / 4);
    const int ntail = (int)(bytes % 4);
    hipLaunchKernelGGL(zero_kernel, dim3(grid_for(n > 0 ? n : 1, 256)), dim3(256), 0, s,
                       (uint32_t*)p, n, (uint8_t*)p + 4 * n, ntail);
    return hipGetLastError();
}

}  // namespace phx
