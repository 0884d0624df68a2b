// HIP kernels of the learned initial guess of the local Newton solves:
// sampling of the patch features, the transfinite lifting, training
// targets, and the network's bfloat16 matrix-core forward/backward with
// FP32 accumulation and its Adam update.
//
// The paper starts each inner Newton iteration (eq. 4) from R_i u; this part
// only proposes a start, which the local Newton kernel accepts when its
// residual is below that of R_i u.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "guess_device.h"

namespace {

__device__ __forceinline__ uint16_t f2bf(float x) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float gelu(float z) {
    return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}
__device__ __forceinline__ float gelu_prime(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
           z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// ---------------------------------------------------------------- sampling
__device__ __forceinline__ double sample(const DevGuessTables& T, int i, int k, const double* f) {
    const size_t b = ((size_t)i * NLS_G_IN + k) * 3;
    return T.sw[b] * f[T.snode[b]] + T.sw[b + 1] * f[T.snode[b + 1]] +
           T.sw[b + 2] * f[T.snode[b + 2]];
}

// Side function s (0 bottom, 1 right, 2 top, 3 left) at parameter t: linear
// between the NS samples of the side; the last interval ends at the first
// sample of the next side (the corner).
template <int NS>
__device__ __forceinline__ double side(const double* tr, int sd, double t) {
    const double pos = t * NS;
    int j = (int)floor(pos);
    j = j < 0 ? 0 : (j > NS - 1 ? NS - 1 : j);
    const double w = pos - j;
    const int nx = (j < NS - 1) ? sd * NS + j + 1 : ((sd + 1) & 3) * NS;
    return (1.0 - w) * tr[sd * NS + j] + w * tr[nx];
}

// Transfinite (Coons) interpolant of the sampled perimeter (NS samples per
// side) at unit (xi, eta).
template <int NS = NLS_G_SIDE>
__device__ __forceinline__ double coons(const double* tr, double xi, double eta) {
    const double g0 = side<NS>(tr, 0, xi), g1 = side<NS>(tr, 1, eta);
    const double g2 = side<NS>(tr, 2, 1.0 - xi), g3 = side<NS>(tr, 3, 1.0 - eta);
    const double c00 = tr[0], c10 = tr[NS], c11 = tr[2 * NS], c01 = tr[3 * NS];
    return (1.0 - eta) * g0 + eta * g2 + (1.0 - xi) * g3 + xi * g1 -
           ((1.0 - xi) * (1.0 - eta) * c00 + xi * (1.0 - eta) * c10 + xi * eta * c11 +
            (1.0 - xi) * eta * c01);
}

// Bilinear interpolant of the GX x GY reference-node values c[q*GX + p].
template <int GX = NLS_G_GRID, int GY = NLS_G_GRID>
__device__ __forceinline__ double bilinear(const float* c, double xi, double eta) {
    const double px = xi * (GX - 1), py = eta * (GY - 1);
    int p0 = (int)floor(px), q0 = (int)floor(py);
    p0 = p0 < 0 ? 0 : (p0 > GX - 2 ? GX - 2 : p0);
    q0 = q0 < 0 ? 0 : (q0 > GY - 2 ? GY - 2 : q0);
    const double a = px - p0, b = py - q0;
    const float* r0 = c + q0 * GX + p0;
    const float* r1 = r0 + GX;
    return (1.0 - a) * (1.0 - b) * r0[0] + a * (1.0 - b) * r0[1] + (1.0 - a) * b * r1[0] +
           a * b * r1[1];
}

// ------------------------------------------------- elasticity (Q1, d = 2)
// Component c of the dof field f (node-major, two per node) at sample k.
__device__ __forceinline__ double sample_e(const DevGuessTables& T, int i, int k,
                                           const double* f, int c) {
    const size_t b = ((size_t)i * NLS_GE_NSAMP + k) * 4;
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) v += T.sw[b + q] * f[2 * T.snode[b + q] + c];
    return v;
}

// Features: u_x, u_y at the 32 perimeter points, then f_x, f_y (external
// nodal forces) at the 128 points on the right side of the box.
__global__ void __launch_bounds__(NLS_G_IN)
k_guess_features_e(DevGuessTables T, const double* __restrict__ u, const double* __restrict__ fload,
                   const float* __restrict__ xm, const float* __restrict__ xs,
                   float* __restrict__ xraw, uint16_t* __restrict__ xbf) {
    const int i = blockIdx.x, k = threadIdx.x;
    double v;
    if (k < 2 * NLS_GE_TRACE) {
        v = sample_e(T, i, k % NLS_GE_TRACE, u, k / NLS_GE_TRACE);
    } else {
        const int kk = k - 2 * NLS_GE_TRACE;
        v = sample_e(T, i, NLS_GE_TRACE + kk % NLS_GE_LOAD, fload, kk / NLS_GE_LOAD);
    }
    const size_t o = (size_t)i * NLS_G_IN + k;
    if (xraw) xraw[o] = (float)v;
    if (xbf) xbf[o] = f2bf((float)((v - (double)xm[k]) / (double)xs[k]));
}

// x_pred on the V dofs: per component Coons of its 32 trace samples +
// bilinear interpolant of its 128 coefficients; Dirichlet dofs exact.
__global__ void __launch_bounds__(256)
k_guess_lift_e(DevMaps P, DevGuessTables T, DevMesh M, const double* __restrict__ xy,
               const double* __restrict__ u, const float* __restrict__ coef,
               double* __restrict__ xpred) {
    __shared__ double tr[2 * NLS_GE_TRACE];
    __shared__ float cf[NLS_G_OUT];
    const int i = blockIdx.x;
    if (threadIdx.x < 2 * NLS_GE_TRACE)
        tr[threadIdx.x] = sample_e(T, i, threadIdx.x % NLS_GE_TRACE, u, threadIdx.x / NLS_GE_TRACE);
    for (int k = threadIdx.x; k < NLS_G_OUT; k += blockDim.x) cf[k] = coef[(size_t)i * NLS_G_OUT + k];
    __syncthreads();
    const double x0 = T.box[4 * i], y0 = T.box[4 * i + 1];
    const double W = T.box[4 * i + 2] - x0, H = T.box[4 * i + 3] - y0;
    const int rb = P.off_n[i], n = P.off_n[i + 1] - rb;
    for (int a = threadIdx.x; a < n; a += blockDim.x) {
        const int dof = P.l2g[rb + a], g = dof >> 1, c = dof & 1;
        double v;
        if (M.dflag[dof]) {
            v = M.dval[dof];
        } else {
            const double xi = (xy[2 * g] - x0) / W, eta = (xy[2 * g + 1] - y0) / H;
            v = coons<NLS_GE_SIDE>(tr + c * NLS_GE_TRACE, xi, eta) +
                bilinear<NLS_GE_GX, NLS_GE_GY>(cf + c * NLS_GE_NGRID, xi, eta);
        }
        xpred[rb + a] = v;
    }
}

// Training target: per component (v(x*) - Coons) at the 16 x 8 reference
// nodes, v(x*) = x* on the V dofs and u elsewhere.
__global__ void __launch_bounds__(NLS_G_OUT)
k_guess_target_e(DevGuessTables T, const double* __restrict__ u, const double* __restrict__ xstar,
                 float* __restrict__ traw) {
    __shared__ double tr[2 * NLS_GE_TRACE];
    const int i = blockIdx.x, k = threadIdx.x;
    if (k < 2 * NLS_GE_TRACE) tr[k] = sample_e(T, i, k % NLS_GE_TRACE, u, k / NLS_GE_TRACE);
    __syncthreads();
    const int c = k / NLS_GE_NGRID, q = k % NLS_GE_NGRID;
    const size_t b = ((size_t)i * NLS_GE_NSAMP + NLS_GE_TRACE + NLS_GE_LOAD + q) * 4;
    const size_t bl = ((size_t)i * NLS_GE_NGRID + q) * 4;
    double v = 0.0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int loc = T.sloc[bl + t];
        v += T.sw[b + t] * (loc >= 0 ? xstar[loc + c] : u[2 * T.snode[b + t] + c]);
    }
    const int p = q % NLS_GE_GX, qq = q / NLS_GE_GX;
    const double xi = (double)p / (NLS_GE_GX - 1), eta = (double)qq / (NLS_GE_GY - 1);
    traw[(size_t)i * NLS_G_OUT + k] =
        (float)(v - coons<NLS_GE_SIDE>(tr + c * NLS_GE_TRACE, xi, eta));
}

// f^_g = mean of the edge-midpoint load samples over the (element, edge)
// pairs through node g; 1 without samples.
__global__ void k_nodal_load(DevMesh M, const double* __restrict__ fmid, double* __restrict__ fhat) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= M.N) return;
    if (!fmid) {
        fhat[g] = 1.0;
        return;
    }
    double acc = 0.0;
    int cnt = 0;
    for (int k = M.nptr[g]; k < M.nptr[g + 1]; ++k) {
        const int e = M.nel[k] >> 2, a = M.nel[k] & 3;
        acc += fmid[3 * e + a] + fmid[3 * e + (a + 2) % 3];
        cnt += 2;
    }
    fhat[g] = cnt ? acc / cnt : 0.0;
}

// Features of subdomain i: 64 perimeter samples of u, 256 grid samples of
// the nodal load.  Raw FP32 copy and/or standardised bfloat16 copy.
__global__ void __launch_bounds__(NLS_G_IN)
k_guess_features(DevGuessTables T, const double* __restrict__ u, const double* __restrict__ fhat,
                 const float* __restrict__ xm, const float* __restrict__ xs,
                 float* __restrict__ xraw, uint16_t* __restrict__ xbf) {
    const int i = blockIdx.x, k = threadIdx.x;
    const double v = sample(T, i, k, k < NLS_G_TRACE ? u : fhat);
    const size_t o = (size_t)i * NLS_G_IN + k;
    if (xraw) xraw[o] = (float)v;
    if (xbf) xbf[o] = f2bf((float)((v - (double)xm[k]) / (double)xs[k]));
}

// x_pred on V_i: Coons(trace of u) + bilinear(coef); Dirichlet rows exact.
__global__ void __launch_bounds__(256)
k_guess_lift(DevMaps P, DevGuessTables T, DevMesh M, const double* __restrict__ xy,
             const double* __restrict__ u, const float* __restrict__ coef,
             double* __restrict__ xpred) {
    __shared__ double tr[NLS_G_TRACE];
    __shared__ float cf[NLS_G_NGRID];
    const int i = blockIdx.x;
    if (threadIdx.x < NLS_G_TRACE) tr[threadIdx.x] = sample(T, i, threadIdx.x, u);
    for (int k = threadIdx.x; k < NLS_G_NGRID; k += blockDim.x)
        cf[k] = coef[(size_t)i * NLS_G_NGRID + k];
    __syncthreads();
    const double x0 = T.box[4 * i], y0 = T.box[4 * i + 1];
    const double W = T.box[4 * i + 2] - x0, H = T.box[4 * i + 3] - y0;
    const int rb = P.off_n[i], n = P.off_n[i + 1] - rb;
    for (int a = threadIdx.x; a < n; a += blockDim.x) {
        const int g = P.l2g[rb + a];
        double v;
        if (M.dflag[g]) {
            v = M.dval[g];
        } else {
            const double xi = (xy[2 * g] - x0) / W, eta = (xy[2 * g + 1] - y0) / H;
            v = coons(tr, xi, eta) + bilinear(cf, xi, eta);
        }
        xpred[rb + a] = v;
    }
}

// Training target of subdomain i: (v(x*) - Coons) at the 256 reference
// nodes, v(x*) = x* on V_i and u elsewhere.
__global__ void __launch_bounds__(NLS_G_NGRID)
k_guess_target(DevGuessTables T, const double* __restrict__ u, const double* __restrict__ xstar,
               float* __restrict__ traw) {
    __shared__ double tr[NLS_G_TRACE];
    const int i = blockIdx.x, k = threadIdx.x;
    if (k < NLS_G_TRACE) tr[k] = sample(T, i, k, u);
    __syncthreads();
    const size_t b = ((size_t)i * NLS_G_IN + NLS_G_TRACE + k) * 3;
    const size_t bl = ((size_t)i * NLS_G_NGRID + k) * 3;
    double v = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int loc = T.sloc[bl + c];
        v += T.sw[b + c] * (loc >= 0 ? xstar[loc] : u[T.snode[b + c]]);
    }
    const int p = k % NLS_G_GRID, q = k / NLS_G_GRID;
    const double xi = (double)p / (NLS_G_GRID - 1), eta = (double)q / (NLS_G_GRID - 1);
    traw[(size_t)i * NLS_G_NGRID + k] = (float)(v - coons(tr, xi, eta));
}

// ------------------------------------------------------- bf16 matrix cores
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int GBM = 32, GBN = 64, GBK = 64, GLD = GBK + 8;

// A tile of ROWS rows by GBK values of k in registers and in LDS (k
// contiguous, pitch GLD).  KC: k is contiguous in memory (element (r, k) at
// p[r ld + k]), else r is (p[k ld + r]); 16-byte loads either way, eight
// values that the second form writes down the tile's rows.  Rows and k values
// past their ends are zeros; along the contiguous direction the sizes are
// multiples of 8 (320, 256) and the bases 16-byte aligned.
template <int ROWS, bool KC>
struct Stage {
    static constexpr int NCH = ROWS * GBK / 8 / 256;
    uint4 v[NCH];
    __device__ __forceinline__ void place(int c, int& r, int& k) const {
        const int e = threadIdx.x + 256 * c;
        if (KC) {
            r = e / (GBK / 8);
            k = 8 * (e % (GBK / 8));
        } else {
            k = e / (ROWS / 8);
            r = 8 * (e % (ROWS / 8));
        }
    }
    __device__ __forceinline__ void load(const uint16_t* __restrict__ p, int ld, int r0, int rows,
                                         int k0, int kend) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            int r, k;
            place(c, r, k);
            r += r0;
            k += k0;
            v[c] = uint4{0, 0, 0, 0};
            if (r < rows && k < kend)
                v[c] = *(const uint4*)(p + (KC ? (size_t)r * ld + k : (size_t)k * ld + r));
        }
    }
    __device__ __forceinline__ void store(uint16_t* T) const {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            int r, k;
            place(c, r, k);
            if (KC) {
                *(uint4*)(T + r * GLD + k) = v[c];
            } else {
                const uint32_t w[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    T[(r + i) * GLD + k] = (uint16_t)(w[i >> 1] >> (16 * (i & 1)));
            }
        }
    }
};

// A 32 x 64 output tile by four wavefronts of 16 x 32 (two blocks of the
// 16x16x16 bf16 matrix-core step, k ascending).  The next 64 values of k are
// fetched into registers while the current ones are multiplied.
template <bool AK, bool BK>
__device__ __forceinline__ void gemm_tile(const uint16_t* __restrict__ A, int lda, int M,
                                          const uint16_t* __restrict__ B, int ldb, int N, int m0,
                                          int n0, int kbeg, int kend, uint16_t* As, uint16_t* Bs,
                                          f32x4 (&acc)[2]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int wm = w >> 1, wn = w & 1, lr = lane & 15, lk = 4 * (lane >> 4);
    acc[0] = acc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    Stage<GBM, AK> a;
    Stage<GBN, BK> b;
    a.load(A, lda, m0, M, kbeg, kend);
    b.load(B, ldb, n0, N, kbeg, kend);
    for (int k0 = kbeg; k0 < kend; k0 += GBK) {
        a.store(As);
        b.store(Bs);
        __syncthreads();
        if (k0 + GBK < kend) {
            a.load(A, lda, m0, M, k0 + GBK, kend);
            b.load(B, ldb, n0, N, k0 + GBK, kend);
        }
#pragma unroll
        for (int kk = 0; kk < GBK; kk += 16) {
            const bf16x4 av = *(const bf16x4*)&As[(wm * 16 + lr) * GLD + kk + lk];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const bf16x4 bv = *(const bf16x4*)&Bs[(wn * 32 + t * 16 + lr) * GLD + kk + lk];
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bv, acc[t], 0, 0, 0);
            }
        }
        __syncthreads();
    }
}

// The layers' products.  Bound by launch and load latency at the sizes of a
// batch (1,280 rows: 160 tiles and 5 k-steps; 7 us per layer, 26 us with 64 x
// 64 tiles staged element by element).
template <bool AK, bool BK>
__global__ void __launch_bounds__(256) k_gemm_bf16(GemmArgs g) {
    __shared__ __align__(16) uint16_t As[GBM * GLD];
    __shared__ __align__(16) uint16_t Bs[GBN * GLD];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m0 = blockIdx.y * GBM, n0 = blockIdx.x * GBN;
    f32x4 acc[2];
    gemm_tile<AK, BK>(g.A, g.lda, g.M, g.B, g.ldb, g.N, m0, n0, 0, g.K, As, Bs, acc);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = m0 + (w >> 1) * 16 + 4 * (lane >> 4) + j;
            const int col = n0 + (w & 1) * 32 + t * 16 + (lane & 15);
            if (row >= g.M || col >= g.N) continue;
            const float v = acc[t][j];
            switch (g.epi) {
            case EPI_BIAS_GELU: {
                const float z = v + g.bias[col];
                if (g.out) g.out[(size_t)row * g.ldo + col] = z;
                g.outb[(size_t)row * g.ldob + col] = f2bf(gelu(z));
                break;
            }
            case EPI_BIAS: {
                float z = v + g.bias[col];
                if (g.oscale) z = z * g.oscale[col] + g.oshift[col];
                g.out[(size_t)row * g.ldo + col] = z;
                break;
            }
            default: {
                const float d = v * gelu_prime(g.aux[(size_t)row * g.ldaux + col]);
                g.out[(size_t)row * g.ldo + col] = d;
                g.outb[(size_t)row * g.ldob + col] = f2bf(d);
                break;
            }
            }
        }
}

// Weight and bias gradients of all layers, the rows of the batch split over
// blockIdx.y: block x forms one 32 x 64 tile of dW_l = dZ_l^T X_l, or (the last
// blocks of a layer) 64 column sums of dZ_l, of its rows, into split y of the
// partial sums; k_grad_sum adds the splits in order.  (1,280 rows: 952 blocks
// in one launch, 14 us; four products of 20 blocks and four column sums of one
// block took 4 x 147 and 4 x 293 us.)
__global__ void __launch_bounds__(256) k_grad_partial(GradArgs g) {
    __shared__ __align__(16) uint16_t As[GBM * GLD];
    __shared__ __align__(16) uint16_t Bs[GBN * GLD];
    int l = 0;
    while (l + 1 < 4 && (int)blockIdx.x >= g.first[l + 1]) ++l;
    const int q = blockIdx.x - g.first[l], in = g.in[l];
    const int r0 = blockIdx.y * g.chunk, r1 = min(g.rows, r0 + g.chunk);
    float* out = g.part + (size_t)blockIdx.y * g.nparam;
    const int nt = in / GBN, ntile = nt * (NLS_G_WIDTH / GBM);
    if (q >= ntile) {
        // column sums: a column per lane, every fourth row per wavefront, the
        // loads of eight rows at a time in flight; then the four partial sums
        // in a fixed order
        __shared__ float red[256];
        const int c = 64 * (q - ntile) + (threadIdx.x & 63), part = threadIdx.x >> 6;
        float s = 0.f;
        const float* dz = g.dz[l] + c;
        int r = r0 + part;
        for (; r + 28 < r1; r += 32) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = dz[(size_t)(r + 4 * u) * NLS_G_WIDTH];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; r < r1; r += 4) s += dz[(size_t)r * NLS_G_WIDTH];
        red[threadIdx.x] = s;
        __syncthreads();
        if (part == 0)
            out[g.off_b[l] + c] = (red[threadIdx.x] + red[threadIdx.x + 64]) +
                                  (red[threadIdx.x + 128] + red[threadIdx.x + 192]);
        return;
    }
    const int m0 = GBM * (q / nt), n0 = GBN * (q % nt);
    f32x4 acc[2];
    gemm_tile<false, false>(g.dzb[l], NLS_G_WIDTH, NLS_G_WIDTH, g.x[l], in, in, m0, n0, r0, r1, As,
                            Bs, acc);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = m0 + (w >> 1) * 16 + 4 * (lane >> 4) + j;
            const int col = n0 + (w & 1) * 32 + t * 16 + (lane & 15);
            out[g.off_w[l] + (size_t)row * in + col] = acc[t][j];
        }
}

__global__ void k_grad_sum(const float* __restrict__ part, int splits, int n, float* __restrict__ grad) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    float s = part[p];
    for (int y = 1; y < splits; ++y) s += part[(size_t)y * n + p];
    grad[p] = s;
}

// ------------------------------------------------------------- training
// Column means and deviations of X (n x cols) in FP64; deviations at or
// below 1e-6 max(max deviation, 1) are replaced by 1.
__global__ void k_fit_norm(const float* __restrict__ X, int64_t n, int cols, float* mean,
                           float* dev) {
    __shared__ double red[1024];
    const int c = threadIdx.x;
    double m = 0.0, s = 0.0;
    if (c < cols) {
        for (int64_t r = 0; r < n; ++r) m += (double)X[r * cols + c];
        m /= (double)(n > 0 ? n : 1);
        for (int64_t r = 0; r < n; ++r) {
            const double d = (double)X[r * cols + c] - m;
            s += d * d;
        }
        s = sqrt(s / (double)(n > 0 ? n : 1));
    }
    red[c] = (c < cols) ? s : 0.0;
    __syncthreads();
    for (int h = blockDim.x / 2; h > 0; h >>= 1) {
        if (c < h) red[c] = fmax(red[c], red[c + h]);
        __syncthreads();
    }
    const double smax = red[0];
    if (c < cols) {
        mean[c] = (float)m;
        dev[c] = (float)((s <= 1e-6 * fmax(smax, 1.0)) ? 1.0 : s);
    }
}

// Rows idx[r] (or r) of the raw inputs and targets, standardised: inputs to
// bfloat16, targets in FP32.  norm = [xm(320) xs(320) ym(256) ys(256)].
__global__ void __launch_bounds__(NLS_G_IN)
k_gather_batch(const float* __restrict__ X, const float* __restrict__ T, const int* __restrict__ idx,
               const float* __restrict__ norm, uint16_t* __restrict__ xb, float* __restrict__ tn) {
    const int r = blockIdx.x, k = threadIdx.x;
    const int64_t src = idx ? (int64_t)idx[r] : (int64_t)r;
    const float* xm = norm;
    const float* xs = norm + NLS_G_IN;
    const float* ym = norm + 2 * NLS_G_IN;
    const float* ys = ym + NLS_G_OUT;
    xb[(size_t)r * NLS_G_IN + k] = f2bf((X[src * NLS_G_IN + k] - xm[k]) / xs[k]);
    if (T && k < NLS_G_OUT) tn[(size_t)r * NLS_G_OUT + k] = (T[src * NLS_G_OUT + k] - ym[k]) / ys[k];
}

// dZ = 2 (Y - Tn) / (rows * 256); per-block partial sums of (Y - Tn)^2.
__global__ void __launch_bounds__(256)
k_mse_grad(const float* __restrict__ Y, const float* __restrict__ Tn, int64_t total, float scale,
           float* __restrict__ dz, uint16_t* __restrict__ dzb, double* __restrict__ partial) {
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const float d = Y[e] - Tn[e];
        s += (double)d * (double)d;
        const float v = scale * d;
        dz[e] = v;
        dzb[e] = f2bf(v);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void k_mse_final(const double* __restrict__ partial, int nb, double inv_total,
                            double* __restrict__ loss_acc) {
    // one wavefront: each lane its share, then a fixed tree
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += 64) s += partial[b];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if (threadIdx.x != 0) return;
    loss_acc[0] += s * inv_total;
    loss_acc[1] += 1.0;
}

// Adam (Kingma and Ba) with bias corrections c1 = 1/(1-b1^t),
// c2 = 1/(1-b2^t); refreshes the bfloat16 copy of the parameters.
__global__ void k_adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, uint16_t* __restrict__ wb, int64_t n, float lr,
                       float b1, float b2, float eps, float c1, float c2) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const float gp = g[p];
    const float mp = b1 * m[p] + (1.0f - b1) * gp;
    const float vp = b2 * v[p] + (1.0f - b2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    const float wn = w[p] - lr * (mp * c1) / (sqrtf(vp * c2) + eps);
    w[p] = wn;
    wb[p] = f2bf(wn);
}

__global__ void k_to_bf16(const float* __restrict__ x, uint16_t* __restrict__ y, int64_t n) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) y[p] = f2bf(x[p]);
}

// counts[0] += subdomains that started from the prediction, counts[1] +=
// those that fell back to R_i u (start codes 1 and 2).
__global__ void k_count_starts(const int* __restrict__ start, int n, int* __restrict__ counts) {
    __shared__ int c1[256], c2[256];
    int a = 0, b = 0;
    for (int i = threadIdx.x; i < n; i += 256) {
        a += start[i] == 1;
        b += start[i] == 2;
    }
    c1[threadIdx.x] = a;
    c2[threadIdx.x] = b;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            c1[threadIdx.x] += c1[threadIdx.x + h];
            c2[threadIdx.x] += c2[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        counts[0] = c1[0];
        counts[1] = c2[0];
    }
}

// flag[0] = 1 if any of idx[0..n) lies outside [0, limit).
__global__ void k_check_indices(const int* __restrict__ idx, int64_t n, int64_t limit,
                                int* __restrict__ flag) {
    int bad = 0;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * blockDim.x)
        bad |= (idx[p] < 0 || (int64_t)idx[p] >= limit);
    if (__any(bad) && (threadIdx.x & 63) == 0) flag[0] = 1;
}

}  // namespace

// ----------------------------------------------------------------- launchers
hipError_t launch_check_indices(const int* idx, int64_t n, int64_t limit, int* flag,
                                hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int nb = (int)((n + 255) / 256);
    if (nb > 1024) nb = 1024;
    k_check_indices<<<nb, 256, 0, s>>>(idx, n, limit, flag);
    return hipGetLastError();
}

hipError_t launch_gemm_bf16(const GemmArgs& g, hipStream_t s) {
    if (g.M <= 0 || g.N <= 0) return hipSuccess;
    dim3 grid((g.N + GBN - 1) / GBN, (g.M + GBM - 1) / GBM);
    if (g.bk)
        k_gemm_bf16<true, true><<<grid, 256, 0, s>>>(g);
    else
        k_gemm_bf16<true, false><<<grid, 256, 0, s>>>(g);
    return hipGetLastError();
}

hipError_t launch_grad(GradArgs g, float* grad, hipStream_t s) {
    if (g.rows <= 0) return hipSuccess;
    // whole k-steps per split, at most NLS_G_SPLITS of them
    g.chunk = (g.rows + NLS_G_SPLITS - 1) / NLS_G_SPLITS;
    g.chunk = (g.chunk + GBK - 1) / GBK * GBK;
    const int splits = (g.rows + g.chunk - 1) / g.chunk;
    int blocks = 0;
    for (int l = 0; l < 4; ++l) {
        g.first[l] = blocks;
        blocks += (g.in[l] / GBN) * (NLS_G_WIDTH / GBM) + NLS_G_WIDTH / 64;
    }
    k_grad_partial<<<dim3(blocks, splits), 256, 0, s>>>(g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_grad_sum<<<(g.nparam + 255) / 256, 256, 0, s>>>(g.part, splits, g.nparam, grad);
    return hipGetLastError();
}

hipError_t launch_nodal_load(const DevMesh& M, const double* fmid, double* fhat, hipStream_t s) {
    if (M.N <= 0) return hipSuccess;
    k_nodal_load<<<(M.N + 255) / 256, 256, 0, s>>>(M, fmid, fhat);
    return hipGetLastError();
}

hipError_t launch_guess_features(const DevGuessTables& T, int nrows, const double* u,
                                 const double* fhat, const float* xm, const float* xs,
                                 float* xraw, uint16_t* xbf, hipStream_t s) {
    if (nrows <= 0) return hipSuccess;
    if (T.elast)
        k_guess_features_e<<<nrows, NLS_G_IN, 0, s>>>(T, u, fhat, xm, xs, xraw, xbf);
    else
        k_guess_features<<<nrows, NLS_G_IN, 0, s>>>(T, u, fhat, xm, xs, xraw, xbf);
    return hipGetLastError();
}

hipError_t launch_guess_lift(const DevMaps& P, const DevGuessTables& T, const DevMesh& M,
                             const double* xy, const double* u, const float* coef,
                             double* xpred, hipStream_t s) {
    if (T.nsub <= 0) return hipSuccess;
    if (T.elast)
        k_guess_lift_e<<<T.nsub, 256, 0, s>>>(P, T, M, xy, u, coef, xpred);
    else
        k_guess_lift<<<T.nsub, 256, 0, s>>>(P, T, M, xy, u, coef, xpred);
    return hipGetLastError();
}

hipError_t launch_guess_target(const DevGuessTables& T, int nrows, const double* u,
                               const double* xstar, float* traw, hipStream_t s) {
    if (nrows <= 0) return hipSuccess;
    if (T.elast)
        k_guess_target_e<<<nrows, NLS_G_OUT, 0, s>>>(T, u, xstar, traw);
    else
        k_guess_target<<<nrows, NLS_G_NGRID, 0, s>>>(T, u, xstar, traw);
    return hipGetLastError();
}

hipError_t launch_fit_norm(const float* X, int64_t n, int cols, float* mean, float* dev,
                           hipStream_t s) {
    if (cols <= 0 || cols > 1024) return hipErrorInvalidValue;
    int bs = 1;
    while (bs < cols) bs <<= 1;
    k_fit_norm<<<1, bs, 0, s>>>(X, n, cols, mean, dev);
    return hipGetLastError();
}

hipError_t launch_gather_batch(const float* X, const float* T, const int* idx, int rows,
                               const float* norm, uint16_t* xb, float* tn, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    k_gather_batch<<<rows, NLS_G_IN, 0, s>>>(X, T, idx, norm, xb, tn);
    return hipGetLastError();
}

hipError_t launch_mse_grad(const float* Y, const float* Tn, int rows, float* dz, uint16_t* dzb,
                           double* partial, double* loss_acc, hipStream_t s) {
    const int64_t total = (int64_t)rows * NLS_G_OUT;
    if (total <= 0) return hipSuccess;
    int nb = (int)((total + 255) / 256);
    if (nb > 256) nb = 256;
    k_mse_grad<<<nb, 256, 0, s>>>(Y, Tn, total, 2.0f / (float)total, dz, dzb, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_mse_final<<<1, 64, 0, s>>>(partial, nb, 1.0 / (double)total, loss_acc);
    return hipGetLastError();
}

hipError_t launch_adam(float* w, const float* g, float* m, float* v, uint16_t* wb, int64_t n,
                       float lr, float b1, float b2, float eps, float c1, float c2,
                       hipStream_t s) {
    if (n <= 0) return hipSuccess;
    k_adam<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(w, g, m, v, wb, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_to_bf16(const float* x, uint16_t* y, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    k_to_bf16<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(x, y, n);
    return hipGetLastError();
}

hipError_t launch_count_starts(const int* start, int n, int* counts, hipStream_t s) {
    k_count_starts<<<1, 256, 0, s>>>(start, n, counts);
    return hipGetLastError();
}
