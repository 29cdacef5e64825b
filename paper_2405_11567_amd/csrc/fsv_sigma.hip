// Kernels of the sector-compressed state C[Ia][Ib] (alpha-string-first
// product basis): excitation rotations and the adjoint step over alpha x beta
// pair lists, the Hamiltonian product H C, and conversions.  Every kernel is
// templated on the stored amplitude: complex or real, FP64 or FP32.  A state
// built from the reference with real angles and real integrals is exactly
// real, which halves every byte and flop of the energy/gradient pass.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <rocblas/rocblas.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "fsv_device.h"
#include "fsv_internal.h"

namespace fsv {

namespace {

// ---- amplitude arithmetic (accumulations in FP64) ----
template <typename V> struct Vt;
template <> struct Vt<double2> { using R = double; };
template <> struct Vt<float2> { using R = float; };
template <> struct Vt<double> { using R = double; };
template <> struct Vt<float> { using R = float; };

// (a, b) <- (c a - s b, c b + s a)
__device__ __forceinline__ void rot(double &a, double &b, double c, double s) {
    const double t = a;
    a = c * a - s * b;
    b = c * b + s * t;
}
__device__ __forceinline__ void rot(float &a, float &b, float c, float s) {
    const float t = a;
    a = c * a - s * b;
    b = c * b + s * t;
}
__device__ __forceinline__ void rot(double2 &a, double2 &b, double c, double s) {
    rot(a.x, b.x, c, s);
    rot(a.y, b.y, c, s);
}
__device__ __forceinline__ void rot(float2 &a, float2 &b, float c, float s) {
    rot(a.x, b.x, c, s);
    rot(a.y, b.y, c, s);
}
// Re(conj(l) p)
__device__ __forceinline__ double dotre(double l, double p) { return l * p; }
__device__ __forceinline__ double dotre(float l, float p) { return (double)l * p; }
__device__ __forceinline__ double dotre(double2 l, double2 p) { return l.x * p.x + l.y * p.y; }
__device__ __forceinline__ double dotre(float2 l, float2 p) { return (double)l.x * p.x + (double)l.y * p.y; }
__device__ __forceinline__ double neg_if(bool n, double v) { return n ? -v : v; }

// ---- conversions ----
__device__ __forceinline__ void cvt(double a, double &b) { b = a; }
__device__ __forceinline__ void cvt(double a, float &b) { b = (float)a; }
__device__ __forceinline__ void cvt(float a, double &b) { b = a; }
__device__ __forceinline__ void cvt(double a, double2 &b) { b = make_double2(a, 0.0); }
__device__ __forceinline__ void cvt(double2 a, double2 &b) { b = a; }
__device__ __forceinline__ void cvt(double2 a, float2 &b) { b = make_float2((float)a.x, (float)a.y); }
__device__ __forceinline__ void cvt(float2 a, double2 &b) { b = make_double2(a.x, a.y); }
__device__ __forceinline__ void cvt(double2 a, double &b) { b = a.x; }

template <typename I, typename O>
__global__ void k_convert(const I *__restrict__ in, O *__restrict__ out, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        cvt(in[i], out[i]);
}

// ------------------------------------------------------------ rotations ----
struct CGrid {
    unsigned gx, gy, block;
};

inline CGrid cgrid_of(const PairOp &op, int64_t nsa, int64_t nsb) {
    const int64_t na = op.nA >= 0 ? op.nA : nsa, nb = op.nB >= 0 ? op.nB : nsb;
    CGrid g;
    g.block = nb <= 64 ? 64u : (nb <= 128 ? 128u : 256u);
    const int64_t gy = na < 1024 ? (na > 0 ? na : 1) : 1024;
    int64_t gx = (nb + g.block - 1) / g.block;
    const int64_t cap = kMaxGrid / gy > 0 ? kMaxGrid / gy : 1;
    if (gx > cap) gx = cap;
    if (gx < 1) gx = 1;
    g.gx = (unsigned)gx;
    g.gy = (unsigned)gy;
    return g;
}

// Alpha pair u of the operator (row u when it has no alpha part).
__device__ __forceinline__ void pair_row(const PairOp &op, const uint32_t *__restrict__ lists,
                                         int64_t u, int64_t &ia, int64_t &ia2, bool &neg) {
    if (op.nA >= 0) {
        const uint32_t e = lists[op.offA + u];
        ia = e & 0x7FFFu;
        ia2 = (e >> 15) & 0x7FFFu;
        neg = (op.sign0 < 0) ^ ((e >> 31) != 0);
    } else {
        ia = ia2 = u;
        neg = op.sign0 < 0;
    }
}

// Beta pair v (column v when it has no beta part).
__device__ __forceinline__ void pair_col(const PairOp &op, const uint32_t *__restrict__ lists,
                                         int64_t v, int64_t &ib, int64_t &ib2, bool &neg) {
    if (op.nB >= 0) {
        const uint32_t e = lists[op.offB + v];
        ib = e & 0x7FFFu;
        ib2 = (e >> 15) & 0x7FFFu;
        neg ^= (e >> 31) != 0;
    } else {
        ib = ib2 = v;
    }
}

template <typename V>
__global__ __launch_bounds__(256) void k_crot(V *__restrict__ psi, PairOp op,
                                              const uint32_t *__restrict__ lists,
                                              const double *__restrict__ cs, int k, int64_t nsa,
                                              int64_t nsb) {
    using R = typename Vt<V>::R;
    const R c = (R)cs[2 * k], s = (R)cs[2 * k + 1];
    const int64_t na = op.nA >= 0 ? op.nA : nsa, nb = op.nB >= 0 ? op.nB : nsb;
    for (int64_t u = blockIdx.y; u < na; u += gridDim.y) {
        int64_t ia, ia2;
        bool nrow;
        pair_row(op, lists, u, ia, ia2, nrow);
        for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nb;
             v += (int64_t)gridDim.x * blockDim.x) {
            int64_t ib, ib2;
            bool neg = nrow;
            pair_col(op, lists, v, ib, ib2, neg);
            const int64_t xs = ia * nsb + ib, xd = ia2 * nsb + ib2;
            V a = psi[xs], b = psi[xd];
            rot(a, b, c, neg ? -s : s);
            psi[xs] = a;
            psi[xd] = b;
        }
    }
}

// Partial of Re<lam|T|psi> over the operator's pairs, then psi, lam <- U^+ psi, U^+ lam.
template <typename V>
__global__ __launch_bounds__(256) void k_cadj(V *__restrict__ psi, V *__restrict__ lam, PairOp op,
                                              const uint32_t *__restrict__ lists,
                                              const double *__restrict__ cs, int k, int64_t nsa,
                                              int64_t nsb, double *__restrict__ partial) {
    using R = typename Vt<V>::R;
    const R c = (R)cs[2 * k], s = (R)cs[2 * k + 1];
    const int64_t na = op.nA >= 0 ? op.nA : nsa, nb = op.nB >= 0 ? op.nB : nsb;
    double acc = 0.0;
    for (int64_t u = blockIdx.y; u < na; u += gridDim.y) {
        int64_t ia, ia2;
        bool nrow;
        pair_row(op, lists, u, ia, ia2, nrow);
        for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nb;
             v += (int64_t)gridDim.x * blockDim.x) {
            int64_t ib, ib2;
            bool neg = nrow;
            pair_col(op, lists, v, ib, ib2, neg);
            const int64_t xs = ia * nsb + ib, xd = ia2 * nsb + ib2;
            V a = psi[xs], b = psi[xd], la = lam[xs], lb = lam[xd];
            const double o = dotre(lb, a) - dotre(la, b);
            acc += neg ? -o : o;
            const R sg = neg ? s : -s;  // U^+ = U(-theta)
            rot(a, b, c, sg);
            rot(la, lb, c, sg);
            psi[xs] = a;
            psi[xd] = b;
            lam[xs] = la;
            lam[xd] = lb;
        }
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) partial[blockIdx.y * gridDim.x + blockIdx.x] = acc;
}

// The adjoint sweep on real states keeps psi and lam of each sector amplitude
// side by side, z[i] = (psi[i], lam[i]), so that one access moves both.
template <typename R> struct Zip2;
template <> struct Zip2<double> { using P = double2; };
template <> struct Zip2<float> { using P = float2; };

template <typename R>
__global__ __launch_bounds__(256) void k_zip(const R *__restrict__ psi, const R *__restrict__ lam,
                                             typename Zip2<R>::P *__restrict__ z, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        z[i] = {psi[i], lam[i]};
}

// k_cadj on the interleaved pairs.
template <typename R>
__global__ __launch_bounds__(256) void k_cadj_zip(typename Zip2<R>::P *__restrict__ z, PairOp op,
                                                  const uint32_t *__restrict__ lists,
                                                  const double *__restrict__ cs, int k, int64_t nsa,
                                                  int64_t nsb, double *__restrict__ partial) {
    const R c = (R)cs[2 * k], s = (R)cs[2 * k + 1];
    const int64_t na = op.nA >= 0 ? op.nA : nsa, nb = op.nB >= 0 ? op.nB : nsb;
    double acc = 0.0;
    for (int64_t u = blockIdx.y; u < na; u += gridDim.y) {
        int64_t ia, ia2;
        bool nrow;
        pair_row(op, lists, u, ia, ia2, nrow);
        for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nb;
             v += (int64_t)gridDim.x * blockDim.x) {
            int64_t ib, ib2;
            bool neg = nrow;
            pair_col(op, lists, v, ib, ib2, neg);
            const int64_t xs = ia * nsb + ib, xd = ia2 * nsb + ib2;
            const auto A = z[xs], B = z[xd];
            R a = A.x, la = A.y, b = B.x, lb = B.y;
            const double o = (double)lb * (double)a - (double)la * (double)b;
            acc += neg ? -o : o;
            const R sg = neg ? s : -s;  // U^+ = U(-theta)
            rot(a, b, c, sg);
            rot(la, lb, c, sg);
            z[xs] = {a, la};
            z[xd] = {b, lb};
        }
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) partial[blockIdx.y * gridDim.x + blockIdx.x] = acc;
}

// ---------------------------------------------------------------- sigma ----
// out[I][:] = sum_k val[k] in[col[k]][:].  Blocks are dispatched row-fastest
// over one column tile at a time (blockIdx.x = row, blockIdx.y = tile), so the
// workgroups in flight share the input rows of the same tile in L2.
__global__ __launch_bounds__(256) void k_spmm(const int64_t *__restrict__ rowptr,
                                              const int32_t *__restrict__ col,
                                              const double *__restrict__ val, const double *__restrict__ in,
                                              double *__restrict__ out, int64_t ncols) {
    const int64_t I = blockIdx.x;
    const int64_t k0 = rowptr[I], k1 = rowptr[I + 1];
    const int64_t c = (int64_t)blockIdx.y * blockDim.x + threadIdx.x;
    if (c >= ncols) return;
    double acc = 0.0;
    for (int64_t k = k0; k < k1; ++k) acc += val[k] * in[(int64_t)col[k] * ncols + c];
    out[I * ncols + c] = acc;
}

// Dense copy of a CSR matrix (one workgroup per row; columns within a row are
// distinct, so the scatter needs no ordering).
__global__ __launch_bounds__(256) void k_csr_dense(const int64_t *__restrict__ rowptr,
                                                   const int32_t *__restrict__ col,
                                                   const double *__restrict__ val, double *__restrict__ out,
                                                   int64_t n) {
    const int64_t I = blockIdx.x;
    double *row = out + I * n;
    for (int64_t c = threadIdx.x; c < n; c += blockDim.x) row[c] = 0.0;
    __syncthreads();
    for (int64_t k = rowptr[I] + threadIdx.x; k < rowptr[I + 1]; k += blockDim.x) row[col[k]] = val[k];
}

typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));

// D (+)= A B for small row-major FP64 matrices (m x k times k x n), one
// wavefront per 16 x 16 tile of D.  The library's tiles leave most of the chip
// idle at these sizes: squares of 70 / 126 / 252 / 462 take it 8.0 / 11.6 / 18.6 /
// 18.3 us, here 4.4 / 5.7 / 7.7 / 13.  Bound by the chain along k.  A wavefront
// loads 16 k at a time (each lane four consecutive k of its row of A, so that a
// row's 128 bytes are used at once, and the same k of its column of B),
// kDtAhead such blocks ahead of the products (two: 16 us at 462, three: 14).
// Whole blocks are addressed by offsets that fit 32 bits; clamping every k
// instead took 27 us at 462.
constexpr int kDtAhead = 4;

template <bool ACC>
__global__ __launch_bounds__(256) void k_dtile(const double *__restrict__ A, const double *__restrict__ B,
                                               double *__restrict__ D, int m, int n, int k, int tn) {
    using f64x4 = __attribute__((ext_vector_type(4))) double;
    const int lane = threadIdx.x & (kWave - 1), c = lane & 15, q = lane >> 4;
    const int tile = (int)(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave);
    const int row0 = tile / tn * 16, col0 = tile % tn * 16;
    if (row0 >= m) return;
    // byte offsets of the lane's row of A and column of B in a block (dtile_fits bounds them)
    const uint32_t oa = 8u * (uint32_t)(min(row0 + c, m - 1) * k + 4 * q);
    const uint32_t ob = 8u * (uint32_t)(4 * q * n + min(col0 + c, n - 1));
    struct Block {
        dbl2u a0, a1;
        double b[4];
    };
    auto load = [&](int blk, Block &t) {
        const char *pa = (const char *)(A + 16 * blk) + oa;
        t.a0 = *(const dbl2u *)pa;
        t.a1 = *(const dbl2u *)(pa + 16);
#pragma unroll
        for (int j = 0; j < 4; ++j) t.b[j] = *(const double *)((const char *)(B + (int64_t)(16 * blk + j) * n) + ob);
    };
    f64x4 d{0.0, 0.0, 0.0, 0.0};
    auto product = [&](const Block &x) {
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a0.x, x.b[0], d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a0.y, x.b[1], d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a1.x, x.b[2], d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a1.y, x.b[3], d, 0, 0, 0);
    };
    const int nb = k / 16;  // whole blocks
    if (nb) {
        Block t[kDtAhead];
#pragma unroll
        for (int u = 0; u < kDtAhead; ++u) load(min(u, nb - 1), t[u]);
        for (int blk = 0; blk < nb; blk += kDtAhead) {
#pragma unroll
            for (int u = 0; u < kDtAhead; ++u) {
                const Block x = t[u];
                load(min(blk + u + kDtAhead, nb - 1), t[u]);
                if (blk + u < nb) product(x);
            }
        }
    }
    if (k & 15) {  // the rest of k; beyond it the last one again, without weight
        Block x;
        double av[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int kk = 16 * nb + 4 * q + j, kc = min(kk, k - 1);
            const double v = A[(int64_t)min(row0 + c, m - 1) * k + kc];
            av[j] = kk < k ? v : 0.0;
            x.b[j] = B[(int64_t)kc * n + min(col0 + c, n - 1)];
        }
        x.a0 = dbl2u{av[0], av[1]};
        x.a1 = dbl2u{av[2], av[3]};
        product(x);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = row0 + 4 * r + q;
        if (i < m && col0 + c < n) {
            double *p = D + (int64_t)i * n + col0 + c;
            *p = ACC ? *p + d[r] : d[r];
        }
    }
}

// At most one tile per SIMD: 924 squared (3364 tiles) takes 77 us here and the
// library 39.
bool dtile_fits(int64_t m, int64_t n, int64_t k) {
    return ((m + 15) / 16) * ((n + 15) / 16) <= 1024 && k <= 1024;
}

template <bool ACC>
hipError_t launch_dtile(const double *A, const double *B, double *D, int64_t m, int64_t n, int64_t k, hipStream_t st) {
    const int64_t tn = (n + 15) / 16, tiles = (m + 15) / 16 * tn;
    hipLaunchKernelGGL(k_dtile<ACC>, dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, st, A, B, D, (int)m, (int)n,
                       (int)k, (int)tn);
    return hipGetLastError();
}

// Same-spin product on the matrix cores: out (rows x w*ncols, row-major) =
// H (rows x rows, row-major, symmetric) * in (rows x w*ncols), as the
// column-major product in' * H of rocBLAS (in' = in viewed column-major).
// Atomics stay disallowed on the handle, so the result is deterministic and no
// memset enters a captured graph.
hipError_t dense_same_spin(void *blas, const double *H, const double *in, double *out, int64_t rows,
                           int64_t wcols, hipStream_t st) {
    if (dtile_fits(rows, wcols, rows)) return launch_dtile<false>(H, in, out, rows, wcols, rows, st);
    rocblas_handle h = (rocblas_handle)blas;
    const double one = 1.0, zero = 0.0;
    if (rocblas_set_stream(h, st) != rocblas_status_success) return hipErrorInvalidHandle;
    const rocblas_status rs = rocblas_dgemm(h, rocblas_operation_none, rocblas_operation_none, (rocblas_int)wcols,
                                            (rocblas_int)rows, (rocblas_int)rows, &one, in, (rocblas_int)wcols, H,
                                            (rocblas_int)rows, &zero, out, (rocblas_int)wcols);
    return rs == rocblas_status_success ? hipSuccess : hipErrorLaunchFailure;
}

// Same-spin beta part of a real state accumulated in place, with no
// transposes of the state: S[Ia][Ib] += sum_Jb Hb[Ib][Jb] C[Ia][Jb].  Read
// column-major, the row-major S and C are nsb x nsa matrices and the
// row-major Hb^T (HbT) is Hb, so this is S += Hb x C, one untransposed GEMM.
// (nsa: the rows of C, both planes' of a complex state.)
hipError_t dense_beta_accumulate(void *blas, const double *HbT, const double *C, double *S, int64_t nsa,
                                 int64_t nsb, hipStream_t st) {
    if (dtile_fits(nsa, nsb, nsb)) return launch_dtile<true>(C, HbT, S, nsa, nsb, nsb, st);
    rocblas_handle h = (rocblas_handle)blas;
    const double one = 1.0;
    if (rocblas_set_stream(h, st) != rocblas_status_success) return hipErrorInvalidHandle;
    const rocblas_status rs =
        rocblas_dgemm(h, rocblas_operation_none, rocblas_operation_none, (rocblas_int)nsb, (rocblas_int)nsa,
                      (rocblas_int)nsb, &one, HbT, (rocblas_int)nsb, C, (rocblas_int)nsb, &one, S, (rocblas_int)nsb);
    return rs == rocblas_status_success ? hipSuccess : hipErrorLaunchFailure;
}

// Alpha-beta two-body term, one workgroup per output row Ia:
//   S[Ia][Ib] += sum_{e in exc(Ia)} sum_{f in exc(Ib)} s_e s_f (pq_e|rs_f) C[J_e][J_f].
// The alpha excitations are taken ec at a time.  Their source rows are staged
// in LDS interleaved as Rt[Jb][e] and their weights as Wt[rs][e] = s_e (pq_e|rs),
// so each beta excitation of a thread's Ib costs one contiguous LDS read of
// the ec row values and one of the ec weights.
__global__ __launch_bounds__(512) void k_sigma_ab(const uint32_t *__restrict__ excA, int nexcA,
                                                  const uint32_t *__restrict__ excB, int nexcB,
                                                  const double *__restrict__ g, int M,
                                                  const double *__restrict__ Cin, double *__restrict__ Sin,
                                                  int64_t nsb, int64_t ld, int ec) {
    extern __shared__ double smem_d[];
    double *Rt = smem_d;                    // nsb * ec
    double *Wt = Rt + (int64_t)nsb * ec;    // M2 * ec
    const double *C = Cin + (int64_t)blockIdx.y * nsb;  // the plane's rows, ld apart
    double *S = Sin + (int64_t)blockIdx.y * nsb;
    const int64_t Ia = blockIdx.x;
    const int M2 = M * M;
    for (int e0 = 0; e0 < nexcA; e0 += ec) {
        const int ne = min(ec, nexcA - e0);
        for (int e = 0; e < ne; ++e) {
            const uint32_t w = excA[Ia * nexcA + e0 + e];
            const int64_t Ja = w & 0xFFFFu;
            const int pq = (w >> 16) & 0x1FFu;
            const double sa = (w >> 31) ? -1.0 : 1.0;
            for (int64_t jb = threadIdx.x; jb < nsb; jb += blockDim.x) Rt[jb * ec + e] = C[Ja * ld + jb];
            for (int rs = threadIdx.x; rs < M2; rs += blockDim.x) Wt[rs * ec + e] = sa * g[pq * M2 + rs];
        }
        __syncthreads();
        for (int64_t Ib = threadIdx.x; Ib < nsb; Ib += blockDim.x) {
            double acc = 0.0;
            for (int f = 0; f < nexcB; ++f) {
                const uint32_t eb = excB[Ib * nexcB + f];
                const double *r = Rt + (int64_t)(eb & 0xFFFFu) * ec;
                const double *wr = Wt + (int)((eb >> 16) & 0x1FFu) * ec;
                double t = 0.0;
                for (int e = 0; e < ne; ++e) t += wr[e] * r[e];
                acc += neg_if((eb >> 31) != 0, t);
            }
            S[Ia * ld + Ib] += acc;
        }
        __syncthreads();
    }
}

// Product with a factorised interaction, (pq|rs) = sum_l L_l[pq] L_l[rs]
// (l < R <= 8, padded to 8 with zero columns).  With A_l = sum_pq L_l[pq]
// E^alpha_pq, B_l the same on the beta strings and h'_pq = h_pq - 1/2 sum_r
// (pr|rq),
//   H = h'_alpha + h'_beta + 1/2 sum_l (A_l + B_l)^2,
// so all of H that is not purely alpha is local to a row of C once
// Y_l = A_l C + 1/2 B_l C is known there:
//   (H - H_alpha) C = h'_beta C + sum_l B_l Y_l,
// added to the purely alpha part that S holds already.  One workgroup per row
// (alpha string Ia), each thread CP pairs of neighbouring columns:
//  1. the row goes to LDS; B_l C gathers it through the partner table: for an
//     orbital pair {p, q}, a string holding exactly one of them maps to the
//     string holding the other, with one sign for E_pq and E_qp alike, so all
//     lanes work on the same pair and its factors L_l[pq] are scalars;
//  2. A_l C reads whole rows of C (row-uniform lists and factors);
//  3. B_l Y, pair by pair: every column's sum_l L_l[pq] Y_l goes to LDS (8
//     bytes instead of the 8 values of Y_l), and the partner reads it.
// Bound by FP64 vector arithmetic (FP64 MFMA sustains less here, 45 against 65 TFLOP/s):
// ~17 multiply-adds per element and orbital pair plus 8 per alpha excitation.
// The former kernels read the 8 values of Y_l and the 8 factors of each beta
// excitation from LDS per lane, and left both same-spin parts to GEMMs.  H C
// at 24 qubits (924 rows of 924): 102 us with the beta same-spin part, E and
// the (psi, lam) pairs included, where the former kernel, the beta GEMM and
// the pass over the result took 102 + 39 + 6 us; about half of the vector
// issue slots are filled (3.6 rows per CU).  Energies alone (two planes of a
// dense state) 55 us instead of ~300 us.  30 qubits (6435 rows of 6435): 13.5
// ms instead of 11.7 ms and a beta GEMM of 8.0 ms.  (The purely alpha part
// could run the same way on the rows of C^T: 9.7 ms there against the GEMM's
// 8.0 ms, ~60 against 39 us at 24 qubits, so it stays a GEMM.)  28 qubits,
// energy alone: 1.2 ms instead of 7.4 ms.
// The LDS slot after the row (2 ceil(ncols / 2)) holds zero: the partner of a
// string outside the pair's reach.
constexpr int kRowR = 8;

typedef double dbl2a __attribute__((ext_vector_type(2), aligned(16)));

struct RowArgs {
    int32_t nrows, ncols, npair, ts;  // ts: column pairs, the words of a pair's partner row
    int32_t nexc, noff;               // stride and off-diagonal length of the alpha lists
    int64_t ld, plane;                // row stride of C and S, offset of the imaginary plane
    double ecore;
    int32_t im_epoch;                 // energy of complex states: the plane counts when *im_flag equals it
    const int32_t *im_flag;
};

enum RowOut { ROW_ENERGY = 0, ROW_S = 1, ROW_ZIP = 2, ROW_ZIP32 = 3 };

__device__ __forceinline__ double flip_sign(double v, uint32_t sign_bit) {  // sign_bit: 0 or 1 << 31
    return __hiloint2double(__double2hiint(v) ^ (int)sign_bit, __double2loint(v));
}

// NB buffers of NC pairs (1: long rows, a second barrier per buffer); WV: waves
// per SIMD the registers must allow.
// PS groups of wavefronts share the orbital pairs and source rows of a row: each
// has all of its columns, and their sums meet in LDS.
template <int BS, int CP, int LH, int NC, int NB, int WV, int PS, int OUT>
__global__ __launch_bounds__(BS, WV) void k_row(const double *__restrict__ C, double *__restrict__ S,
                                            void *__restrict__ z, double *__restrict__ epart,
                                            const uint32_t *__restrict__ tp, const double *__restrict__ Lp,
                                            const double *__restrict__ hp, const double *__restrict__ db,
                                            const double *__restrict__ hd, const uint32_t *__restrict__ exc,
                                            const double *__restrict__ Lt, const double *__restrict__ da,
                                            const double *__restrict__ heff, const double *__restrict__ hda,
                                            RowArgs a) {
    static_assert(PS == 1 || (LH == kRowR && NB == 2 && BS / PS % kWave == 0), "whole wavefronts, one pass");
    extern __shared__ double buf[];
    constexpr int CB = BS / PS;  // threads of a group
    const int n = a.ncols, ncp = (n + 1) >> 1, zero = 2 * ncp, Wp = zero + 2;
    const int tid = PS == 1 ? threadIdx.x : threadIdx.x % CB;  // the thread's place in its group
    const int part = PS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / CB);
    // XCD x takes a contiguous range of rows: neighbouring strings share most
    // of their source rows, which then share that XCD's L2
    int row;
    {
        const int v = blockIdx.x, per = a.nrows >> 3, rem = a.nrows & 7, x = v & 7;
        row = x * per + min(x, rem) + (v >> 3);
    }
    if (OUT == ROW_ENERGY && blockIdx.y && *a.im_flag != a.im_epoch) {  // a zero imaginary plane
        if (threadIdx.x == 0) epart[a.nrows + row] = 0.0;
        return;
    }
    const double *Cp = C + (int64_t)blockIdx.y * a.plane;
    const double *crow = Cp + (int64_t)row * a.ld;
    // column pair of slot q (clamped): columns 2 j and 2 j + 1.  In a row of
    // odd length the last pair's second column is the value after the row
    // (inside the state's buffer or workspace); no partner names it.  Loads
    // take a uniform base and a 32-bit byte offset per lane.
    uint32_t off[CP];
#pragma unroll
    for (int q = 0; q < CP; ++q) off[q] = 16u * (uint32_t)min(tid + q * CB, ncp - 1);
    auto pair = [&](int q) { return (int)(off[q] >> 4); };
    auto on = [&](int q) { return tid + q * CB < ncp; };
    auto load2 = [&](const double *p, int q) { return *(const dbl2u *)((const char *)p + off[q]); };
    // a value and, Wp further on, its negative: partner words index either
    auto put2 = [&](double *b, int q, double x, double y) {
        *(dbl2a *)((char *)b + off[q]) = dbl2a{x, y};
        *(dbl2a *)((char *)(b + Wp) + off[q]) = dbl2a{-x, -y};
    };
    // keeps one column pair's loads from being hoisted over the others'
    // (their registers would spill)
    auto fence = [] {
        if (CP > 1) asm volatile("" ::: "memory");
    };
    constexpr int KB = CP > 2 ? 1 : 4, EB = CP > 2 ? 1 : 4 / CP;  // partner words, source rows loaded together
    auto words = [&](int k, uint32_t (&t)[CP]) {
        const char *p = (const char *)(tp + (int64_t)k * a.ts);
#pragma unroll
        for (int q = 0; q < CP; ++q) t[q] = *(const uint32_t *)(p + (off[q] >> 2));
    };
    constexpr double f = OUT == ROW_ENERGY ? 1.0 : 0.5;  // Y takes half of B_l C (exact scaling)
    double s[CP][2];
    for (int t = tid; t < (OUT == ROW_ENERGY || PS > 1 ? 2 : 2 * NB * NC); t += CB) buf[t * Wp + zero] = 0.0;
    double en = 0.0;
    const uint32_t *ex = exc + (int64_t)row * a.nexc;
    for (int l0 = 0; l0 < kRowR; l0 += LH) {
        const bool first = l0 == 0;
        __syncthreads();  // the previous pass's readers of buf are done
        double v[CP][2][LH];
        const double *dar = da + (int64_t)row * kRowR + l0;
#pragma unroll
        for (int q = 0; q < CP; ++q) {
            const dbl2u c = load2(crow, q);
            const double c0 = f * c.x, c1 = f * c.y;
            if (part == 0 && on(q)) put2(buf, q, c0, c1);
#pragma unroll
            for (int l = 0; l < LH; ++l) {
                const dbl2u w = load2(db + (l0 + l) * zero, q);
                v[q][0][l] = w.x * c0;
                v[q][1][l] = w.y * c1;
                v[q][0][l] += dar[l] * c.x;
                v[q][1][l] += dar[l] * c.y;
            }
            if (first) {
                const dbl2u w = load2(hd, q);
                s[q][0] = w.x * c.x;
                s[q][1] = w.y * c.y;
                const double e = OUT == ROW_ENERGY ? hda[row] + a.ecore : a.ecore;
                s[q][0] += e * c.x;
                s[q][1] += e * c.y;
            }
            if (PS > 1 && part) {  // the diagonal terms once
                s[q][0] = s[q][1] = 0.0;
#pragma unroll
                for (int l = 0; l < LH; ++l) v[q][0][l] = v[q][1][l] = 0.0;
            }
            fence();
        }
        __syncthreads();
        auto gather = [&](int k, const uint32_t (&t)[CP]) {
            double x[CP][2];
#pragma unroll
            for (int q = 0; q < CP; ++q) {
                x[q][0] = buf[t[q] & 0xFFFFu];
                x[q][1] = buf[t[q] >> 16];
            }
            const double *L = Lp + k * kRowR + l0;
#pragma unroll
            for (int l = 0; l < LH; ++l) {
                const double w = L[l];
#pragma unroll
                for (int q = 0; q < CP; ++q) {
                    v[q][0][l] += w * x[q][0];
                    v[q][1][l] += w * x[q][1];
                }
            }
            if (first) {
                const double w = hp[k] * (1.0 / f);
#pragma unroll
                for (int q = 0; q < CP; ++q) {
                    s[q][0] += w * x[q][0];
                    s[q][1] += w * x[q][1];
                }
            }
        };
        {
            int k = part * KB;  // whole blocks by turns, the rest of the pairs to the last group
            uint32_t t[KB][CP];
            for (; k + KB <= a.npair; k += PS * KB) {
#pragma unroll
                for (int u = 0; u < KB; ++u) words(k + u, t[u]);
#pragma unroll
                for (int u = 0; u < KB; ++u) gather(k + u, t[u]);
            }
            if (PS > 1) k = part == PS - 1 ? a.npair / KB * KB : a.npair;
            for (; k < a.npair; ++k) {
                words(k, t[0]);
                gather(k, t[0]);
            }
        }
        {
            auto arow = [&](uint32_t w, const dbl2u (&u)[CP]) {
                const int pq = (w >> 16) & 0x1FFu;
                const double *L = Lt + pq * kRowR + l0;
                const uint32_t sg = w & 0x80000000u;
                double x[CP][2];
#pragma unroll
                for (int q = 0; q < CP; ++q) {
                    x[q][0] = flip_sign(u[q].x, sg);
                    x[q][1] = flip_sign(u[q].y, sg);
                }
#pragma unroll
                for (int l = 0; l < LH; ++l) {
                    const double wl = L[l];
#pragma unroll
                    for (int q = 0; q < CP; ++q) {
                        v[q][0][l] += wl * x[q][0];
                        v[q][1][l] += wl * x[q][1];
                    }
                }
                if (OUT == ROW_ENERGY && first) {
                    const double wh = heff[pq];
#pragma unroll
                    for (int q = 0; q < CP; ++q) {
                        s[q][0] += wh * x[q][0];
                        s[q][1] += wh * x[q][1];
                    }
                }
            };
            auto source = [&](int e, dbl2u (&x)[CP]) {
                const double *p = Cp + (int64_t)(ex[e] & 0xFFFFu) * a.ld;
#pragma unroll
                for (int q = 0; q < CP; ++q) x[q] = load2(p, q);
            };
            int e = part * EB;
            dbl2u x[EB][CP];
            for (; e + EB <= a.noff; e += PS * EB) {
#pragma unroll
                for (int u = 0; u < EB; ++u) source(e + u, x[u]);
#pragma unroll
                for (int u = 0; u < EB; ++u) arow(ex[e + u], x[u]);
            }
            if (PS > 1) e = part == PS - 1 ? a.noff / EB * EB : a.noff;
            for (; e < a.noff; ++e) {
                source(e, x[0]);
                arow(ex[e], x[0]);
            }
        }
        if (PS > 1) {  // every group gets the sums over all of them
            __syncthreads();
            double *red = buf + tid;
#pragma unroll
            for (int q = 0; q < CP; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int l = 0; l < LH; ++l) red[(((q * 2 + h) * (LH + 1) + l) * PS + part) * CB] = v[q][h][l];
                    red[(((q * 2 + h) * (LH + 1) + LH) * PS + part) * CB] = s[q][h];
                }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < CP; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int l = 0; l <= LH; ++l) {
                        double x = red[((q * 2 + h) * (LH + 1) + l) * PS * CB];
#pragma unroll
                        for (int p = 1; p < PS; ++p) x += red[(((q * 2 + h) * (LH + 1) + l) * PS + p) * CB];
                        if (l < LH)
                            v[q][h][l] = x;
                        else
                            s[q][h] = part ? 0.0 : x;
                    }
                }
        }
        if (OUT == ROW_ENERGY) {
#pragma unroll
            for (int q = 0; q < CP; ++q)
                if (part == 0 && on(q)) {
                    double t0 = 0.0, t1 = 0.0;
#pragma unroll
                    for (int l = 0; l < LH; ++l) {
                        t0 += v[q][0][l] * v[q][0][l];
                        t1 += v[q][1][l] * v[q][1][l];
                    }
                    en += 0.5 * t0;
                    if (2 * pair(q) + 1 < n) en += 0.5 * t1;
                }
        } else {
            // B_l Y: the diagonal part, then pair by pair through LDS, NC pairs
            // to a buffer and two buffers in turn (one barrier per NC pairs)
#pragma unroll
            for (int q = 0; q < CP; ++q) {
#pragma unroll
                for (int l = 0; l < LH; ++l) {
                    const dbl2u w = load2(db + (l0 + l) * zero, q);
                    s[q][0] += part ? 0.0 : w.x * v[q][0][l];
                    s[q][1] += part ? 0.0 : w.y * v[q][1][l];
                }
                fence();
            }
            __syncthreads();  // readers of the row (or of the sums) in buf are done
            double *mine = buf + part * 2 * NB * NC * Wp;  // the group's buffers
            if (PS > 1) {
                for (int t = tid; t < 2 * NB * NC; t += CB) mine[t * Wp + zero] = 0.0;
            }
            int par = 0;
            for (int kb = 0; kb < a.npair; kb += PS * NC, par ^= 1) {
                const int k0 = kb + part * NC;
                double *b = mine + (NB == 2 ? par * 2 * NC * Wp : 0);
                uint32_t t[NC][CP];
#pragma unroll
                for (int u = 0; u < NC; ++u) words(min(k0 + u, a.npair - 1), t[u]);
#pragma unroll
                for (int u = 0; u < NC; ++u)
                    if (k0 + u < a.npair) {
                        const double *L = Lp + (k0 + u) * kRowR + l0;
                        double w[CP][2];
#pragma unroll
                        for (int q = 0; q < CP; ++q) {
                            w[q][0] = L[0] * v[q][0][0];
                            w[q][1] = L[0] * v[q][1][0];
                        }
#pragma unroll
                        for (int l = 1; l < LH; ++l) {
                            const double wl = L[l];
#pragma unroll
                            for (int q = 0; q < CP; ++q) {
                                w[q][0] += wl * v[q][0][l];
                                w[q][1] += wl * v[q][1][l];
                            }
                        }
#pragma unroll
                        for (int q = 0; q < CP; ++q)
                            if (on(q)) put2(b + 2 * u * Wp, q, w[q][0], w[q][1]);
                    }
                __syncthreads();
#pragma unroll
                for (int u = 0; u < NC; ++u)
                    if (k0 + u < a.npair)
#pragma unroll
                        for (int q = 0; q < CP; ++q) {
                            s[q][0] += b[2 * u * Wp + (t[u][q] & 0xFFFFu)];
                            s[q][1] += b[2 * u * Wp + (t[u][q] >> 16)];
                        }
                if (NB == 1) __syncthreads();
            }
        }
    }
    if (PS > 1 && OUT != ROW_ENERGY) {
        __syncthreads();
        double *red = buf + tid;
#pragma unroll
        for (int q = 0; q < CP; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h) red[((q * 2 + h) * PS + part) * CB] = s[q][h];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < CP; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int p = 1; p < PS; ++p) s[q][h] += part ? 0.0 : red[((q * 2 + h) * PS + p) * CB];
    }
    // results
    double *srow = OUT == ROW_ENERGY ? nullptr : S + (int64_t)blockIdx.y * a.plane + (int64_t)row * a.ld;
#pragma unroll
    for (int q = 0; q < CP; ++q)
        if (part == 0 && on(q)) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int col = 2 * pair(q) + h;
                if (col >= n) break;
                double r = s[q][h];
                if (OUT != ROW_ENERGY) r += srow[col];
                const double c = crow[col];
                en += c * r;
                if (OUT == ROW_ZIP)
                    ((double2 *)z)[(int64_t)row * a.ld + col] = make_double2(c, r);
                else if (OUT == ROW_ZIP32)
                    ((float2 *)z)[(int64_t)row * a.ld + col] = make_float2((float)c, (float)r);
                else if (OUT == ROW_S)
                    srow[col] = r;
            }
        }
    en = block_sum(en);
    if (threadIdx.x == 0) epart[(int64_t)blockIdx.y * a.nrows + row] = en;
}

// One-body tables of k_row from h' (M x M): the off-diagonal values per
// orbital pair p < q, and per string the sum over its occupied orbitals.
__global__ __launch_bounds__(256) void k_row_onebody(const double *__restrict__ heff, int M,
                                                     const uint32_t *__restrict__ sa, int64_t nsa,
                                                     const uint32_t *__restrict__ sb, int64_t nsb,
                                                     double *__restrict__ hp, double *__restrict__ hda,
                                                     double *__restrict__ hdb) {
    const int64_t npair = (int64_t)M * (M - 1) / 2, total = npair + nsa + nsb;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        if (i < npair) {
            int p = 0;
            int64_t k = i;
            while (k >= M - 1 - p) k -= M - 1 - p, ++p;
            hp[i] = heff[p * M + p + 1 + k];
            continue;
        }
        const bool alpha = i < npair + nsa;
        const int64_t I = alpha ? i - npair : i - npair - nsa;
        const uint32_t str = alpha ? sa[I] : sb[I];
        double d = 0.0;
        for (int p = 0; p < M; ++p)
            if (str >> p & 1u) d += heff[p * M + p];
        (alpha ? hda : hdb)[I] = d;
    }
}

// Alpha-beta term with a general interaction, one workgroup per row Ia:
//   S[Ia][Ib] += sum_{r<=s} (E_rs + E_sr) G_rs[Ib],  G_rs[Jb] = sum_e s_e (pq_e|rs) C[J_e][Jb]
// (the diagonal pairs r = s once).  Contracting the alpha side first leaves e_a
// M (M+1)/2 multiply-adds per element and one 8-byte LDS exchange per pair rs,
// to the strings that pair rs reaches (the partner table of k_row); taking
// every (alpha, beta) excitation pair of an element from LDS, e_a e_b reads of
// 16 bytes, took 511 us at 24 qubits with integrals of full rank.  A row's
// diagonal alpha excitations are one term with their factors summed per string
// (dg).  Rows of up to 2048 columns: k_abm; longer ones, whose accumulators it
// has no registers for: k_ab.
struct AbArgs {
    int32_t nrows, ncols, npd, ts;  // npd: orbital pairs r <= s, padded to a multiple of 4 rows in g and dg
    int32_t npp;                    // row length of g and dg (padded pairs)
    int32_t nexc, noff;
    int64_t ld, plane;
};

// On vector registers, the factors of RC consecutive pairs as scalars.
template <int BS, int CP, int RC, int NC>
__global__ __launch_bounds__(BS) void k_ab(const double *__restrict__ C, double *__restrict__ S,
                                           const uint32_t *__restrict__ tp, const double *__restrict__ g,
                                           const double *__restrict__ dg, const uint32_t *__restrict__ exc,
                                           AbArgs a) {
    static_assert(RC % NC == 0, "whole buffers per chunk");
    extern __shared__ double buf[];
    const int n = a.ncols, ncp = (n + 1) >> 1, zero = 2 * ncp, Wp = zero + 2, tid = threadIdx.x;
    int row;
    {
        const int v = blockIdx.x, per = a.nrows >> 3, rem = a.nrows & 7, x = v & 7;
        row = x * per + min(x, rem) + (v >> 3);
    }
    const double *Cp = C + (int64_t)blockIdx.y * a.plane;
    uint32_t off[CP];  // columns, offsets and buffers as in k_row
#pragma unroll
    for (int q = 0; q < CP; ++q) off[q] = 16u * (uint32_t)min(tid + q * BS, ncp - 1);
    auto pair = [&](int q) { return (int)(off[q] >> 4); };
    auto on = [&](int q) { return tid + q * BS < ncp; };
    auto load2 = [&](const double *p, int q) { return *(const dbl2u *)((const char *)p + off[q]); };
    for (int t = tid; t < 4 * NC; t += BS) buf[t * Wp + zero] = 0.0;
    const uint32_t *ex = exc + (int64_t)row * a.nexc;
    double s[CP][2];
#pragma unroll
    for (int q = 0; q < CP; ++q) s[q][0] = s[q][1] = 0.0;
    int par = 0;
    for (int c0 = 0; c0 < a.npd; c0 += RC) {
        double acc[RC][CP][2];
#pragma unroll
        for (int r = 0; r < RC; ++r)
#pragma unroll
            for (int q = 0; q < CP; ++q) acc[r][q][0] = acc[r][q][1] = 0.0;
        auto source = [&](int e) {  // e = noff: the row itself
            return Cp + (int64_t)(e < a.noff ? ex[e] & 0xFFFFu : (uint32_t)row) * a.ld;
        };
        dbl2u x[CP];
#pragma unroll
        for (int q = 0; q < CP; ++q) x[q] = load2(source(0), q);
        for (int e = 0; e <= a.noff; ++e) {
            dbl2u nx[CP];  // the next source row, in flight during this one's arithmetic
#pragma unroll
            for (int q = 0; q < CP; ++q) nx[q] = load2(source(min(e + 1, a.noff)), q);
            const uint32_t w = e < a.noff ? ex[e] : 0u;
            const double *wr = e < a.noff ? g + (int64_t)((w >> 16) & 0x1FFu) * a.npp + c0 : dg + (int64_t)row * a.npp + c0;
            const uint32_t sg = w & 0x80000000u;
            double y[CP][2];
#pragma unroll
            for (int q = 0; q < CP; ++q) {
                y[q][0] = flip_sign(x[q].x, sg);
                y[q][1] = flip_sign(x[q].y, sg);
                x[q] = nx[q];
            }
#pragma unroll
            for (int r = 0; r < RC; ++r) {
                const double wv = wr[r];
#pragma unroll
                for (int q = 0; q < CP; ++q) {
                    acc[r][q][0] += wv * y[q][0];
                    acc[r][q][1] += wv * y[q][1];
                }
            }
        }
#pragma unroll
        for (int r0 = 0; r0 < RC; r0 += NC) {
            if (c0 + r0 < a.npd) {
                // two buffers in turn: one is written again only after a
                // barrier that follows every read of it
                double *b = buf + par * 2 * NC * Wp;
#pragma unroll
                for (int u = 0; u < NC; ++u)
#pragma unroll
                    for (int q = 0; q < CP; ++q)
                        if (on(q)) {
                            char *d = (char *)(b + 2 * u * Wp) + off[q];
                            *(dbl2a *)d = dbl2a{acc[r0 + u][q][0], acc[r0 + u][q][1]};
                            *(dbl2a *)(d + 8 * Wp) = dbl2a{-acc[r0 + u][q][0], -acc[r0 + u][q][1]};
                        }
                uint32_t t[NC][CP];
#pragma unroll
                for (int u = 0; u < NC; ++u)
#pragma unroll
                    for (int q = 0; q < CP; ++q)
                        t[u][q] = *(const uint32_t *)((const char *)(tp + (int64_t)min(c0 + r0 + u, a.npd - 1) * a.ts) +
                                                      (off[q] >> 2));
                __syncthreads();
#pragma unroll
                for (int u = 0; u < NC; ++u)
                    if (c0 + r0 + u < a.npd)
#pragma unroll
                        for (int q = 0; q < CP; ++q) {
                            s[q][0] += b[2 * u * Wp + (t[u][q] & 0xFFFFu)];
                            s[q][1] += b[2 * u * Wp + (t[u][q] >> 16)];
                        }
                par ^= 1;
            }
        }
    }
    double *srow = S + (int64_t)blockIdx.y * a.plane + (int64_t)row * a.ld;
#pragma unroll
    for (int q = 0; q < CP; ++q)
        if (on(q)) {
            srow[2 * pair(q)] += s[q][0];
            if (2 * pair(q) + 1 < n) srow[2 * pair(q) + 1] += s[q][1];
        }
}

// G (orbital pairs rs x columns) on the matrix cores: the product of the row's
// factors (rs x sources, with the excitations' signs) and its gathered alpha
// sources (sources x columns).  A chunk is 16 pairs rs; each of W wavefronts
// holds NT 16 x 16 tiles of it.  Two neighbouring tiles take the even and the
// odd columns of 32, so that a lane's 16-byte load feeds both.  Result register
// r of a lane is pair 4 r + lane / 16, so G goes through LDS four pairs at a
// time, and two workgroups share a CU at 924 columns (59 KB of LDS, 113
// registers), one exchanging while the other multiplies.  Bound by the matrix
// cores: 160 us at 24 qubits (924 rows and columns, 37 terms, 78 pairs), of
// which the products take 120 us at the 45 TFLOP/s that back-to-back FP64 MFMA
// reach on this card.  With vector arithmetic (k_ab, whose factors are scalar
// loads that it waits for) the rows of 70 / 126 / 252 / 462 / 924 columns took
// 24 / 29 / 46 / 88 / 203 us, here 9.6 / 11 / 16 / 41 / 160.  Tiles without columns
// are skipped.
struct AbSource {
    const double *a;      // factors
    uint32_t off, sign;  // its row, in bytes; sign bit
};

template <int W, int NT>
__global__ __launch_bounds__(W *kWave, 4) void k_abm(
    const double *__restrict__ C, double *__restrict__ S, const uint32_t *__restrict__ tp,
    const double *__restrict__ g, const double *__restrict__ dg, const uint32_t *__restrict__ exc, AbArgs a) {
    static_assert(NT % 2 == 0 && NT <= 8, "tiles in pairs; one column pair per thread in the exchange");
    using f64x4 = __attribute__((ext_vector_type(4))) double;
    constexpr int BS = W * kWave;
    extern __shared__ double buf[];
    const int n = a.ncols, ncp = (n + 1) >> 1, zero = 2 * ncp, Wp = zero + 2, tid = threadIdx.x;
    const int lane = tid & (kWave - 1), m = lane & 15, kq = lane >> 4;
    AbSource *src = (AbSource *)(buf + 8 * Wp);
    int row;
    {
        const int v = blockIdx.x, per = a.nrows >> 3, rem = a.nrows & 7, x = v & 7;
        row = x * per + min(x, rem) + (v >> 3);
    }
    const double *Cp = C + (int64_t)blockIdx.y * a.plane;
    const uint32_t *ex = exc + (int64_t)row * a.nexc;
    const int ks = (a.noff + 4) >> 2;  // steps of four sources: the excitations, then the row itself
    for (int e = tid; e < 4 * ks; e += BS) {
        const uint32_t w = e < a.noff ? ex[e] : 0u;
        src[e] = AbSource{e < a.noff ? g + (int64_t)((w >> 16) & 0x1FFu) * a.npp : dg + (int64_t)row * a.npp,
                          (e < a.noff ? w & 0xFFFFu : (uint32_t)row) * (uint32_t)a.ld * 8u, w & 0x80000000u};
    }
    if (tid < 8) buf[tid * Wp + zero] = 0.0;
    uint32_t off[NT / 2];  // byte offset of each tile pair's column pair (kept in range; the surplus is not stored)
#pragma unroll
    for (int t = 0; t < NT / 2; ++t) off[t] = 16u * (uint32_t)min(((tid / kWave) * (NT / 2) + t) * 16 + m, ncp - 1);
    const int nt = __builtin_amdgcn_readfirstlane((ncp + 15) / 16 - (tid / kWave) * (NT / 2));  // tile pairs with columns
    auto store = [&](int t) { return ((tid / kWave) * (NT / 2) + t) * 16 + m < ncp; };
    const bool on = tid < ncp;  // the exchange: thread tid has column pair tid
    const int mine = min(tid, ncp - 1);
    double s0 = 0.0, s1 = 0.0;
    __syncthreads();
    for (int c0 = 0; c0 < a.npd; c0 += 16) {
        f64x4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
        double av;
        dbl2u x[NT / 2];
        auto load = [&](int k) {
            const AbSource e = src[4 * k + kq];
            av = flip_sign(e.a[c0 + m], e.sign);
            if (4 * k + kq > a.noff) av = 0.0;  // padding: the row itself again, without weight
#pragma unroll
            for (int t = 0; t < NT / 2; ++t) x[t] = *(const dbl2u *)((const char *)Cp + (e.off + off[t]));
        };
        load(0);
#pragma unroll 2
        for (int k = 0; k < ks; ++k) {
            const double ca = av;
            dbl2u cx[NT / 2];
#pragma unroll
            for (int t = 0; t < NT / 2; ++t) cx[t] = x[t];
            load(min(k + 1, ks - 1));  // in flight during this step's products
#pragma unroll
            for (int t = 0; t < NT / 2; ++t) {
                if (t >= nt) continue;
                acc[2 * t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ca, cx[t].x, acc[2 * t], 0, 0, 0);
                acc[2 * t + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(ca, cx[t].y, acc[2 * t + 1], 0, 0, 0);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (c0 + 4 * r < a.npd) {
                uint32_t t4[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) t4[u] = tp[(int64_t)min(c0 + 4 * r + u, a.npd - 1) * a.ts + mine];
                __syncthreads();  // the previous four pairs have been read
#pragma unroll
                for (int t = 0; t < NT / 2; ++t)
                    if (store(t)) {
                        double *d = (double *)((char *)(buf + 2 * kq * Wp) + off[t]);
                        *(dbl2a *)d = dbl2a{acc[2 * t][r], acc[2 * t + 1][r]};
                        *(dbl2a *)(d + Wp) = dbl2a{-acc[2 * t][r], -acc[2 * t + 1][r]};
                    }
                __syncthreads();
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (c0 + 4 * r + u < a.npd) {
                        s0 += buf[2 * u * Wp + (t4[u] & 0xFFFFu)];
                        s1 += buf[2 * u * Wp + (t4[u] >> 16)];
                    }
            }
        }
    }
    double *srow = S + (int64_t)blockIdx.y * a.plane + (int64_t)row * a.ld;
    if (on) {
        srow[2 * tid] += s0;
        if (2 * tid + 1 < n) srow[2 * tid + 1] += s1;
    }
}

// ------------------------------------------------------------ screening ----
// ADAPT pool screening, one launch for the whole pool: workgroup (x, t)
// accumulates, over its share of pool operator t's pairs, the real part of
// <lam| T_t |psi> = sum s (lam[x'] psi[x] - lam[x] psi[x']); psi and lam are
// only read.  partial[t * gridDim.x + x].
template <typename V>
__global__ __launch_bounds__(256) void k_pool(const V *__restrict__ psi, const V *__restrict__ lam,
                                              const PairOp *__restrict__ ops,
                                              const uint32_t *__restrict__ lists, int64_t nsa, int64_t nsb,
                                              double *__restrict__ partial) {
    const PairOp op = ops[blockIdx.y];
    const uint32_t na = (uint32_t)(op.nA >= 0 ? op.nA : nsa), nb = (uint32_t)(op.nB >= 0 ? op.nB : nsb);
    const uint32_t np = na * nb;
    double acc = 0.0;
    for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < np; t += gridDim.x * blockDim.x) {
        const uint32_t u = t / nb, v = t - u * nb;
        int64_t ia, ia2, ib, ib2;
        bool neg;
        pair_row(op, lists, u, ia, ia2, neg);
        pair_col(op, lists, v, ib, ib2, neg);
        const int64_t xs = ia * nsb + ib, xd = ia2 * nsb + ib2;
        const double o = dotre(lam[xd], psi[xs]) - dotre(lam[xs], psi[xd]);
        acc += neg ? -o : o;
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) partial[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = acc;
}

// Screening by rows: the pool's operators are grouped by their alpha part (all
// that move the same alpha electrons share their row pairs), and a workgroup
// stages U of the group's row pairs of psi and lam in LDS and takes every
// operator of the group through them, one wavefront per operator (or several,
// on interleaved pairs, where the group is small).  k_pool read the four
// amplitudes of each pair of each operator from L2: 3.6 GB for the 1818
// operators at 24 qubits, 877 us.  Here the rows are read once per group (0.8
// GB) and the pairs come from LDS (32 bytes per pair of an operator with a
// beta part): 266 us, about half in each of the two launches, bound by the
// latency of short loops (four steps of list words and LDS reads per operator
// and workgroup).  Operators without a beta part need no LDS: their term is a
// dot product of whole rows, taken while they are read.
template <typename V>
__global__ __launch_bounds__(512) void k_pool_rows(const V *__restrict__ psi, const V *__restrict__ lam,
                                                   const PairOp *__restrict__ ops,
                                                   const uint32_t *__restrict__ lists,
                                                   const PoolGroup *__restrict__ groups,
                                                   const int32_t *__restrict__ gops,
                                                   const int2 *__restrict__ tasks, int U, int nsb,
                                                   const int64_t *__restrict__ off, double *__restrict__ partial) {
    extern __shared__ double smem_d[];
    V *rows = (V *)smem_d;  // [u][psi source, psi target, lam source, lam target][nsb]
    const int2 task = tasks[blockIdx.x];
    const PoolGroup g = groups[task.x];
    const int u0 = task.y, nu = min(U, g.nA - u0), chunk = u0 / U;
    const V *p1[kPoolU], *p2[kPoolU], *l1[kPoolU], *l2[kPoolU];
#pragma unroll
    for (int u = 0; u < kPoolU; ++u) {
        int64_t ia = u0 + min(u, nu - 1), ia2 = ia;
        if (g.offA >= 0) {
            const uint32_t e = lists[g.offA + ia];
            ia = e & 0x7FFFu;
            ia2 = (e >> 15) & 0x7FFFu;
        }
        p1[u] = psi + ia * nsb;
        p2[u] = psi + ia2 * nsb;
        l1[u] = lam + ia * nsb;
        l2[u] = lam + ia2 * nsb;
    }
    auto signA = [&](const PairOp &op, int u) {  // sign0 and the row pair's sign, in bit 31
        return (op.sign0 < 0 ? 0x80000000u : 0u) ^ (op.nA >= 0 && u < nu ? lists[op.offA + u0 + u] & 0x80000000u : 0u);
    };
    // the rows to LDS, and the operators without a beta part (two at a time;
    // a qubit excitation may list its strings' signs)
    for (int i0 = 0; i0 < max(g.nplain, 1); i0 += 2) {
        uint32_t sg[2][kPoolU];
        const uint32_t *list[2] = {nullptr, nullptr};
        int t[2] = {0, 0};
        double acc[2] = {0.0, 0.0};
#pragma unroll
        for (int b = 0; b < 2; ++b)
            if (i0 + b < g.nplain) {
                t[b] = gops[g.op0 + g.ngen + i0 + b];
                const PairOp op = ops[t[b]];
                if (op.nB >= 0) list[b] = lists + op.offB;
#pragma unroll
                for (int u = 0; u < kPoolU; ++u) sg[b][u] = signA(op, u);
            }
        for (int v = threadIdx.x; v < nsb; v += blockDim.x) {
            double x[2] = {0.0, 0.0};
#pragma unroll
            for (int u = 0; u < kPoolU; ++u)
                if (u < nu) {
                    const V a = p1[u][v], b = p2[u][v], c = l1[u][v], d = l2[u][v];
                    if (g.ngen && i0 == 0) {
                        V *r = rows + u * 4 * nsb;
                        r[v] = a;
                        r[nsb + v] = b;
                        r[2 * nsb + v] = c;
                        r[3 * nsb + v] = d;
                    }
                    const double o = dotre(d, a) - dotre(c, b);
#pragma unroll
                    for (int b2 = 0; b2 < 2; ++b2)
                        if (i0 + b2 < g.nplain) x[b2] += flip_sign(o, sg[b2][u]);
                }
#pragma unroll
            for (int b = 0; b < 2; ++b)
                if (i0 + b < g.nplain) acc[b] += list[b] ? flip_sign(x[b], list[b][v] & 0x80000000u) : x[b];
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
            if (i0 + b < g.nplain) {
                const double r = block_sum(acc[b]);
                if (threadIdx.x == 0) partial[off[t[b]] + chunk] = r;
            }
    }
    if (g.ngen == 0) return;
    __syncthreads();
    // four operators per wavefront at a time: their list words load together
    // and their sums share one butterfly
    constexpr int B = 4;
    const int lane = threadIdx.x & (kWave - 1), nw = blockDim.x / kWave;
    const int wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), items = g.ngen * g.parts;
    for (int w0 = wid; w0 < items; w0 += B * nw) {
        const uint32_t *list[B];
        int nb[B], t[B], part[B], most = 0;
        uint32_t sg[B][kPoolU];  // sign0 and the row pair's sign, in bit 31
        double acc[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int w = min(w0 + b * nw, items - 1), i = w / g.parts;
            part[b] = w - i * g.parts;
            t[b] = gops[g.op0 + i];
            const PairOp op = ops[t[b]];
            nb[b] = w0 + b * nw < items ? op.nB : 0;
            list[b] = lists + op.offB;
#pragma unroll
            for (int u = 0; u < kPoolU; ++u) sg[b][u] = signA(op, u);
            acc[b] = 0.0;
            most = max(most, nb[b]);
        }
        for (int v0 = 0; v0 < most; v0 += kWave * g.parts) {
            uint32_t e[B];
            bool in[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int v = v0 + part[b] * kWave + lane;
                in[b] = v < nb[b];
                e[b] = in[b] ? list[b][v] : 0u;
            }
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int ib = (int)(e[b] & 0x7FFFu), ib2 = (int)((e[b] >> 15) & 0x7FFFu);
                double x = 0.0;
#pragma unroll
                for (int u = 0; u < kPoolU; ++u)
                    if (u < nu) {
                        const V *r = rows + u * 4 * nsb;
                        const double o = dotre(r[3 * nsb + ib2], r[ib]) - dotre(r[2 * nsb + ib], r[nsb + ib2]);
                        x += flip_sign(o, (e[b] ^ sg[b][u]) & 0x80000000u);
                    }
                acc[b] += in[b] ? x : 0.0;
            }
        }
        // lane l ends with the total of operator 2 (l & 1) + (l >> 1 & 1)
        const bool b0 = lane & 1, b1 = lane & 2;
        const double k0 = (b0 ? acc[2] : acc[0]) + __shfl_xor(b0 ? acc[0] : acc[2], 1, kWave);
        const double k1 = (b0 ? acc[3] : acc[1]) + __shfl_xor(b0 ? acc[1] : acc[3], 1, kWave);
        double r = (b1 ? k1 : k0) + __shfl_xor(b1 ? k0 : k1, 2, kWave);
#pragma unroll
        for (int m = 4; m < kWave; m <<= 1) r += __shfl_xor(r, m, kWave);
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (lane == (b >> 1 | (b & 1) << 1) && w0 + b * nw < items)
                partial[off[t[b]] + (int64_t)chunk * g.parts + part[b]] = r;
    }
}

// out[t] = 2 x the sum of operator t's partials, in order.
__global__ __launch_bounds__(256) void k_pool_reduce(const int64_t *__restrict__ off,
                                                     const double *__restrict__ partial, double *__restrict__ out) {
    const int t = blockIdx.x;
    double acc = 0.0;
    for (int64_t i = off[t] + threadIdx.x; i < off[t + 1]; i += blockDim.x) acc += partial[i];
    acc = block_sum(acc);
    if (threadIdx.x == 0) out[t] = 2.0 * acc;
}

// Alpha-beta term without LDS staging (rows too long for LDS): gathers from
// global memory.
__global__ __launch_bounds__(256) void k_sigma_ab_global(const uint32_t *__restrict__ excA, int nexcA,
                                                         const uint32_t *__restrict__ excB, int nexcB,
                                                         const double *__restrict__ g, int M,
                                                         const double *__restrict__ Cin, double *__restrict__ Sin,
                                                         int64_t nsb, int64_t ld) {
    const int64_t Ia = blockIdx.x;
    const int M2 = M * M;
    const double *C = Cin + (int64_t)blockIdx.y * nsb;
    double *S = Sin + (int64_t)blockIdx.y * nsb;
    for (int64_t Ib = threadIdx.x; Ib < nsb; Ib += blockDim.x) {
        double acc = 0.0;
        for (int e = 0; e < nexcA; ++e) {
            const uint32_t w = excA[Ia * nexcA + e];
            const int64_t Ja = w & 0xFFFFu;
            const double *gp = g + ((w >> 16) & 0x1FFu) * M2;
            double t = 0.0;
            for (int f = 0; f < nexcB; ++f) {
                const uint32_t eb = excB[Ib * nexcB + f];
                const double gv = gp[(eb >> 16) & 0x1FFu];
                t += ((eb >> 31) ? -gv : gv) * C[Ja * ld + (eb & 0xFFFFu)];
            }
            acc += neg_if((w >> 31) != 0, t);
        }
        S[Ia * ld + Ib] += acc;
    }
}

// out[c * ldo + r] = in[r * ldi + c], plane blockIdx.z pi / po elements further on.
__global__ void k_transpose(const double *__restrict__ in, double *__restrict__ out, int64_t rows, int64_t cols, int64_t ldi,
                            int64_t ldo, int64_t pi, int64_t po) {
    __shared__ double t[32][33];
    in += (int64_t)blockIdx.z * pi;
    out += (int64_t)blockIdx.z * po;
    const int64_t c0 = (int64_t)blockIdx.x * 32, r0 = (int64_t)blockIdx.y * 32;
    for (int j = threadIdx.y; j < 32; j += blockDim.y) {
        const int64_t r = r0 + j, c = c0 + threadIdx.x;
        if (r < rows && c < cols) t[j][threadIdx.x] = in[r * ldi + c];
    }
    __syncthreads();
    for (int j = threadIdx.y; j < 32; j += blockDim.y) {
        const int64_t c = c0 + j, r = r0 + threadIdx.x;
        if (r < rows && c < cols) out[c * ldo + r] = t[threadIdx.x][j];
    }
}

// S[i][k] += ST[k][i] + ecore C[i][k] for rows x cols matrices; per-block
// partials of <C|S>.  The transposed operand is read through an LDS tile.
__global__ void k_combine(double *__restrict__ S, const double *__restrict__ ST, const double *__restrict__ C,
                          double ecore, int64_t rows, int64_t cols, double *__restrict__ partial) {
    __shared__ double t[32][33];
    double acc = 0.0;
    const int64_t tiles_b = (cols + 31) / 32, tiles = ((rows + 31) / 32) * tiles_b;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t a0 = (tile / tiles_b) * 32, b0 = (tile % tiles_b) * 32;
        for (int j = threadIdx.y; j < 32; j += blockDim.y) {  // ST rows b0+j, columns a0+x
            const int64_t ib = b0 + j, ia = a0 + threadIdx.x;
            if (ib < cols && ia < rows) t[j][threadIdx.x] = ST[ib * rows + ia];
        }
        __syncthreads();
        for (int j = threadIdx.y; j < 32; j += blockDim.y) {
            const int64_t ia = a0 + j, ib = b0 + threadIdx.x;
            if (ia < rows && ib < cols) {
                const double c = C[ia * cols + ib];
                const double v = S[ia * cols + ib] + t[threadIdx.x][j] + ecore * c;
                S[ia * cols + ib] = v;
                acc += c * v;
            }
        }
        __syncthreads();
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0 && threadIdx.y == 0) partial[blockIdx.x] = acc;
}

// String Hamiltonian values from their two-body parts and the one-body
// descriptors (see launch_string_h_values).
__global__ __launch_bounds__(256) void k_string_h_values(double *__restrict__ val, const double *__restrict__ v2,
                                                         const int32_t *__restrict__ desc,
                                                         const uint32_t *__restrict__ str,
                                                         const double *__restrict__ ht, int M, int64_t n) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t d = desc[e];
        double o = 0.0;
        if (d <= -2) {
            const uint32_t s = str[-2 - d];
            for (int i = 0; i < M; ++i)
                if (s >> i & 1u) o += ht[i * M + i];
        } else if (d >= 0) {
            o = ht[d & 0x3FFFFFFF];
            if (d & (1 << 30)) o = -o;
        }
        val[e] = o + v2[e];
    }
}

// S += ecore C and this workgroup's share of <C|S> (real states whose beta
// part went straight into S).
__global__ __launch_bounds__(256) void k_ecore_dot(double *__restrict__ S, const double *__restrict__ C, double ecore,
                                                   int64_t dim, double *__restrict__ partial) {
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim; i += (int64_t)gridDim.x * blockDim.x) {
        const double c = C[i];
        double s = S[i];
        s += ecore * c;
        S[i] = s;
        acc += c * s;
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

// k_ecore_dot for a real state whose adjoint sweep follows on (psi, lam)
// pairs: the pairs z[i] = (C[i], S[i] + ecore C[i]) are written instead of
// S, so that the sweep needs no separate interleaving pass.
__global__ __launch_bounds__(256) void k_ecore_zip(const double *__restrict__ S, const double *__restrict__ C,
                                                   double ecore, int64_t dim, double2 *__restrict__ z,
                                                   double *__restrict__ partial) {
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim; i += (int64_t)gridDim.x * blockDim.x) {
        const double c = C[i];
        double s = S[i];
        s += ecore * c;
        z[i] = make_double2(c, s);
        acc += c * s;
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

// Dense complex image (O = double2 or float2) of a real compact vector, every
// amplitude written once: qubit index -> strings -> ranks (ra, rb: per string
// mask of the sector; rb with the prefix parity of the sign).  A chunk
// of 1024 amplitudes shares the high bits, whose strings are scalars; each
// thread's low bits are split once.  Bound by the writes: 0.81 ms at 28 qubits
// (4.3 GB; filling with zeros and scattering the sector took 0.70 + 0.44 ms), 40
// us at 24 qubits (35 + 16 us).  STREAM: non-temporal stores, for images larger
// than twice the 256 MB last-level cache, which otherwise push the compact
// state out of it (28 qubits 1.03 ms; at 24 qubits they cost 47 us).
constexpr int kImageBits = 10, kImageBlock = 256, kImagePer = (1 << kImageBits) / kImageBlock;

template <typename O, bool BLOCKED, bool STREAM>
__global__ __launch_bounds__(kImageBlock) void k_dense_image(O *__restrict__ out, const double *__restrict__ S,
                                                             const int32_t *__restrict__ ra,
                                                             const int2 *__restrict__ rb, int n, int na, int nb,
                                                             int64_t nsb) {
    const int M = n >> 1;
    const uint64_t total = 1ull << n;
    auto even = [](uint64_t x) {  // bits 0, 2, 4, ... packed
        x &= 0x5555555555555555ull;
        x = (x | x >> 1) & 0x3333333333333333ull;
        x = (x | x >> 2) & 0x0F0F0F0F0F0F0F0Full;
        x = (x | x >> 4) & 0x00FF00FF00FF00FFull;
        x = (x | x >> 8) & 0x0000FFFF0000FFFFull;
        return (uint32_t)(x | x >> 16);
    };
    auto alpha = [&](uint64_t x) { return BLOCKED ? (uint32_t)(x & ((1ull << M) - 1)) : even(x); };
    auto beta = [&](uint64_t x) { return BLOCKED ? (uint32_t)(x >> M) : even(x >> 1); };
    uint32_t la[kImagePer], lb[kImagePer];
#pragma unroll
    for (int u = 0; u < kImagePer; ++u) {
        la[u] = alpha(threadIdx.x + u * kImageBlock);
        lb[u] = beta(threadIdx.x + u * kImageBlock);
    }
    const uint64_t chunks = (total + (1u << kImageBits) - 1) >> kImageBits;
    for (uint64_t c = blockIdx.x; c < chunks; c += gridDim.x) {
        const uint64_t x0 = c << kImageBits;
        const uint32_t ha = alpha(x0), hb = beta(x0);
        const int ea = na - popc(ha), eb = nb - popc(hb);  // electrons left for the low bits
        double v[kImagePer] = {};
        if (ea >= 0 && eb >= 0 && ea + eb <= kImageBits) {
            // every load without a branch, so that all are in flight together
            // (amplitudes outside the sector read the first entries)
            bool ok[kImagePer];
            int32_t ia[kImagePer];
            int2 ib[kImagePer];
#pragma unroll
            for (int u = 0; u < kImagePer; ++u) {
                // a chunk past the end of a small image names no string at all
                ok[u] = x0 + threadIdx.x + u * kImageBlock < total && popc(la[u]) == ea && popc(lb[u]) == eb;
                ia[u] = ra[ok[u] ? ha | la[u] : 0u];
                ib[u] = rb[ok[u] ? hb | lb[u] : 0u];
            }
#pragma unroll
            for (int u = 0; u < kImagePer; ++u) v[u] = S[ok[u] ? ia[u] * nsb + ib[u].x : 0];
#pragma unroll
            for (int u = 0; u < kImagePer; ++u) {
                const bool neg = popc((ha | la[u]) & (uint32_t)ib[u].y) & 1;
                v[u] = ok[u] ? (neg ? -v[u] : v[u]) : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < kImagePer; ++u) {
            const uint64_t x = x0 + threadIdx.x + u * kImageBlock;
            using E = decltype(out->x);
            typedef E E2 __attribute__((ext_vector_type(2)));
            const E2 o{(E)v[u], (E)0};
            if (x >= total) continue;
            if (STREAM)
                __builtin_nontemporal_store(o, (E2 *)&out[x]);
            else
                *(E2 *)&out[x] = o;
        }
    }
}

int g_lds_max = -1;

// Launch shapes of the row kernels: threads, column pairs per thread, factor
// columns per pass (k_row) or orbital pairs per chunk (k_ab), pairs per LDS
// buffer, buffers, waves per SIMD, and groups per row (k_row), by the row's
// column pairs (n = ceil(columns / 2)).  At 924 columns 256 threads x 2 pairs
// (four rows resident per CU) took 102 us, 512 x 1 101-112 us, 128 x 4 116 us,
// two pairs per buffer 139 us.  At 6435 columns 1024 threads x 4 pairs and half of the
// factors per pass took 13.5 ms, 512 x 7 14.2 ms, a quarter of the factors per
// pass 21 ms.
// Few short rows leave most of the chip idle, and a row takes as long as its chain
// of M (M - 1) / 2 orbital pairs, however few of them reach a column: 2 of 12 to
// 15 beta electrons took longer than the former kernel, whose threads followed
// their columns' excitations (us a call: 28 qubits with 3 + 2 electrons 83
// against 77, 24 qubits with 2 + 2 72 against 67).  With the pairs shared by four
// groups (two at 257 to 384 columns) these take 68 and 61 us.  The groups run
// on two and three waves per SIMD, the registers that their sums need (with four
// they spilled).  The lines lie where the chip is full anyway: 495 rows of 66
// columns 79 -> 68 us, 1365 rows of 105 130 -> 120, 1716 rows of 78 123 -> 128;
// 364 rows of 364 columns 94 -> 89, 715 rows of 286 109 -> 113; at 15 pairs (12
// qubits) 51 -> 48, at 6 (8 qubits) the kernel alone 5.9 -> 7.8.
template <int BS, int CP, int NC, int NB, int PS, int OUT>
size_t row_lds(int Wp) {
    const size_t bufs = sizeof(double) * (OUT == ROW_ENERGY ? 2 : 2 * NB * NC * PS) * (size_t)Wp;
    return PS == 1 ? bufs : std::max(bufs, sizeof(double) * BS * CP * 2 * (kRowR + 1));  // the groups' sums take their place
}

template <int OUT>
hipError_t row_launch(int planes, const SectorTabs &T, const double *C, double *S, void *z, double *epart,
                      const int32_t *im_flag, int32_t im_epoch, hipStream_t st) {
    RowArgs a{};
    a.nrows = (int32_t)T.nsa;
    a.ncols = (int32_t)T.nsb;
    a.npair = T.M * (T.M - 1) / 2;
    a.ts = (int32_t)((T.nsb + 1) / 2);
    a.nexc = T.nexcA;
    a.noff = T.nexcA - T.ndA;
    a.ld = planes * T.nsb;
    a.plane = T.nsb;
    a.ecore = T.ecore;
    a.im_epoch = im_epoch;
    a.im_flag = im_flag;
    const int n = (a.ncols + 1) / 2, Wp = 2 * n + 2;
    const dim3 grid((unsigned)a.nrows, (unsigned)planes);
    const int64_t rows = (int64_t)planes * a.nrows;
#define FSV_ROW(BS, CP, LH, NC, NB, WV, PS)                                                                     \
    hipLaunchKernelGGL((k_row<BS, CP, LH, NC, NB, WV, PS, OUT>), grid, dim3(BS), (row_lds<BS, CP, NC, NB, PS, OUT>(Wp)), \
                       st, C, S, z, epart, T.tp, T.Lp, T.hp, T.db, T.hdb, T.excA, T.Lt, T.da, T.heff, T.hda, a)
    if (n <= 64 && rows <= 1536 && a.npair >= 15)
        FSV_ROW(256, 1, 8, 1, 2, 2, 4);
    else if (n <= 64)
        FSV_ROW(64, 1, 8, 1, 2, 4, 1);
    else if (n <= 128)
        FSV_ROW(128, 1, 8, 1, 2, 4, 1);
    else if (n <= 192 && rows <= 512)
        FSV_ROW(384, 1, 8, 1, 2, 3, 2);
    else if (n <= 192)
        FSV_ROW(192, 1, 8, 1, 2, 4, 1);
    else if (n <= 256)
        FSV_ROW(256, 1, 8, 1, 2, 4, 1);
    else if (n <= 512)
        FSV_ROW(256, 2, 8, 1, 2, 4, 1);
    else if (n <= 1024)
        FSV_ROW(512, 2, 8, 1, 2, 4, 1);
    else if (n <= 2048)
        FSV_ROW(512, 4, 8, 1, 2, 2, 1);
    else
        FSV_ROW(1024, 4, 4, 1, 1, 4, 1);
#undef FSV_ROW
    return hipGetLastError();
}

hipError_t ab_launch(const double *C, double *S, const SectorTabs &T, int planes, hipStream_t st) {
    AbArgs a{};
    a.nrows = (int32_t)T.nsa;
    a.ncols = (int32_t)T.nsb;
    a.npd = T.M * (T.M + 1) / 2;
    a.ts = (int32_t)((T.nsb + 1) / 2);
    a.npp = T.npp;
    a.nexc = T.nexcA;
    a.noff = T.nexcA - T.ndA;
    a.ld = planes * T.nsb;
    a.plane = T.nsb;
    const int n = (a.ncols + 1) / 2, Wp = 2 * n + 2;
    const dim3 grid((unsigned)a.nrows, (unsigned)planes);
#define FSV_AB(BS, CP, RC, NC)                                                                                 \
    hipLaunchKernelGGL((k_ab<BS, CP, RC, NC>), grid, dim3(BS), sizeof(double) * 4 * (size_t)NC * Wp, st, C, S, \
                       T.tp, T.gp, T.dg, T.excA, a)
#define FSV_ABM(W, NT)                                                                                            \
    hipLaunchKernelGGL((k_abm<W, NT>), grid, dim3(W * kWave),                                                     \
                       sizeof(double) * 8 * (size_t)Wp + sizeof(AbSource) * 4 * (size_t)((a.noff + 4) / 4), st, C, \
                       S, T.tp, T.gp, T.dg, T.excA, a)
    // k_abm holds a row's offset in 32 bits: at most 32768 rows (15-bit ranks) of two
    // planes of 2048 columns are 1 GiB
    if (n <= 64)
        FSV_ABM(4, 2);
    else if (n <= 128)
        FSV_ABM(4, 4);
    else if (n <= 256)
        FSV_ABM(8, 4);
    else if (n <= 512)
        FSV_ABM(8, 8);
    else if (n <= 1024)
        FSV_ABM(16, 8);
    else if (n <= 2048)
        FSV_AB(512, 4, 8, 1);
    else
        FSV_AB(512, 5, 6, 1);
#undef FSV_ABM
#undef FSV_AB
    return hipGetLastError();
}

// Same-spin alpha part (with the alpha one-body terms) into S: dense on the
// matrix cores, or sparse rows.
hipError_t alpha_same_spin(int planes, const SectorTabs &T, const double *C, double *S, hipStream_t st) {
    const int64_t cols = planes * T.nsb;
    if (T.ha_dense) return dense_same_spin(T.blas, T.ha_dense, C, S, T.nsa, cols, st);
    hipLaunchKernelGGL(k_spmm, dim3((unsigned)T.nsa, (unsigned)((cols + 255) / 256)), dim3(256), 0, st, T.ha_ptr,
                       T.ha_col, T.ha_val, C, S, cols);
    return hipGetLastError();
}

}  // namespace

bool row_kernel_fits(int64_t ncols) {
    // two LDS rows of 8 bytes a column (a row and its negative), on 1024 threads
    // of four column pairs; of the sectors of up to 17 orbitals only those with
    // rows of 11440 and more columns are left out.  With a smaller LDS limit only
    // the short rows' buffers fit.
    return ncols >= 2 && ncols <= (g_lds_max >= 163840 ? 8192 : 480);
}

bool ab_kernel_fits(int64_t ncols) {  // four rows: two buffers and their negatives
    return ncols >= 2 && ncols <= (g_lds_max >= 163840 ? 5096 : 480);
}

namespace {

hipError_t sigma_impl(int planes, const SectorTabs &T, const double *C, double *S, double *CT, double *ST,
                      double *epart, hipStream_t st, void *zout, bool zip32, bool *zipped) {
    const int64_t nsa = T.nsa, nsb = T.nsb, rows = planes * nsa;
    if (T.R > 0) {
        const hipError_t e = alpha_same_spin(planes, T, C, S, st);
        if (e != hipSuccess) return e;
        if (zout && planes == 1) {
            if (zipped) *zipped = true;
            return zip32 ? row_launch<ROW_ZIP32>(1, T, C, S, zout, epart, nullptr, 0, st)
                         : row_launch<ROW_ZIP>(1, T, C, S, zout, epart, nullptr, 0, st);
        }
        return row_launch<ROW_S>(planes, T, C, S, nullptr, epart, nullptr, 0, st);
    }
    hipError_t e = alpha_same_spin(planes, T, C, S, st);
    if (e != hipSuccess) return e;
    if (T.nexcA > 0 && T.nexcB > 0) {
        if (T.gp) {
            e = ab_launch(C, S, T, planes, st);
            if (e != hipSuccess) return e;
        } else {  // rows too long for k_ab's LDS buffers, or of a single column
            const int lds = g_lds_max > 0 ? g_lds_max : 65536;
            const int64_t per = nsb * (int64_t)sizeof(double) + (int64_t)T.M * T.M * (int64_t)sizeof(double);
            int64_t ec = lds / per;
            if (ec > T.nexcA) ec = T.nexcA;
            const dim3 grid((unsigned)nsa, (unsigned)planes);
            if (ec >= 1)
                hipLaunchKernelGGL(k_sigma_ab, grid, dim3(512), (size_t)(ec * per), st, T.excA, T.nexcA, T.excB,
                                   T.nexcB, T.g, T.M, C, S, nsb, planes * nsb, (int)ec);
            else  // a source row does not fit in LDS
                hipLaunchKernelGGL(k_sigma_ab_global, grid, dim3(256), 0, st, T.excA, T.nexcA, T.excB, T.nexcB, T.g,
                                   T.M, C, S, nsb, planes * nsb);
        }
    }
    const unsigned ng = combine_grid(nsa * nsb);
    if (T.hb_dense_t) {
        // the beta GEMM accumulates into S directly
        e = dense_beta_accumulate(T.blas, T.hb_dense_t, C, S, rows, nsb, st);
        if (e != hipSuccess) return e;
        if (zout && !zip32 && planes == 1) {
            hipLaunchKernelGGL(k_ecore_zip, dim3(ng), dim3(256), 0, st, S, C, T.ecore, rows * nsb, (double2 *)zout,
                               epart);
            if (zipped) *zipped = true;
        } else {
            hipLaunchKernelGGL(k_ecore_dot, dim3(ng), dim3(256), 0, st, S, C, T.ecore, rows * nsb, epart);
        }
        return hipGetLastError();
    }
    // same-spin beta part on the transpose, then combine
    hipLaunchKernelGGL(k_transpose, dim3((unsigned)((nsb + 31) / 32), (unsigned)((rows + 31) / 32)),
                       dim3(32, 8), 0, st, C, CT, rows, nsb, nsb, rows, (int64_t)0, (int64_t)0);
    hipLaunchKernelGGL(k_spmm, dim3((unsigned)nsb, (unsigned)((rows + 255) / 256)), dim3(256), 0, st, T.hb_ptr,
                       T.hb_col, T.hb_val, CT, ST, rows);
    hipLaunchKernelGGL(k_combine, dim3(ng), dim3(32, 8), 0, st, S, ST, C, T.ecore, rows, nsb, epart);
    return hipGetLastError();
}

template <typename V>
hipError_t crot_impl(void *psi, const PairOp &op, const uint32_t *lists, const double *cs, int k,
                     int64_t nsa, int64_t nsb, hipStream_t st) {
    const CGrid g = cgrid_of(op, nsa, nsb);
    hipLaunchKernelGGL(k_crot<V>, dim3(g.gx, g.gy), dim3(g.block), 0, st, (V *)psi, op, lists, cs, k, nsa, nsb);
    return hipGetLastError();
}

template <typename V>
hipError_t cadj_impl(void *psi, void *lam, const PairOp &op, const uint32_t *lists, const double *cs,
                     int k, int64_t nsa, int64_t nsb, double *partial, hipStream_t st) {
    const CGrid g = cgrid_of(op, nsa, nsb);
    hipLaunchKernelGGL(k_cadj<V>, dim3(g.gx, g.gy), dim3(g.block), 0, st, (V *)psi, (V *)lam, op, lists, cs,
                       k, nsa, nsb, partial);
    return hipGetLastError();
}

template <typename R>
hipError_t cadj_zip_impl(void *z, const PairOp &op, const uint32_t *lists, const double *cs, int k,
                         int64_t nsa, int64_t nsb, double *partial, hipStream_t st) {
    const CGrid g = cgrid_of(op, nsa, nsb);
    hipLaunchKernelGGL(k_cadj_zip<R>, dim3(g.gx, g.gy), dim3(g.block), 0, st, (typename Zip2<R>::P *)z, op,
                       lists, cs, k, nsa, nsb, partial);
    return hipGetLastError();
}

template <typename R>
hipError_t zip_impl(const void *psi, const void *lam, void *z, int64_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_zip<R>, dim3(blocks_for(n, 256)), dim3(256), 0, st, (const R *)psi, (const R *)lam,
                       (typename Zip2<R>::P *)z, n);
    return hipGetLastError();
}

template <typename I, typename O>
hipError_t convert_impl(const void *in, void *out, int64_t n, hipStream_t st) {
    hipLaunchKernelGGL((k_convert<I, O>), dim3(blocks_for(n, 256)), dim3(256), 0, st, (const I *)in, (O *)out, n);
    return hipGetLastError();
}

}  // namespace

void init_sigma_kernels() {
    std::vector<const void *> fns = {(const void *)k_sigma_ab};
#define FSV_ROW_FNS(BS, CP, LH, NC, NB, WV)                                   \
    fns.push_back((const void *)k_row<BS, CP, LH, NC, NB, WV, 1, ROW_ENERGY>); \
    fns.push_back((const void *)k_row<BS, CP, LH, NC, NB, WV, 1, ROW_S>);      \
    fns.push_back((const void *)k_row<BS, CP, LH, NC, NB, WV, 1, ROW_ZIP>);    \
    fns.push_back((const void *)k_row<BS, CP, LH, NC, NB, WV, 1, ROW_ZIP32>)
    FSV_ROW_FNS(512, 2, 8, 1, 2, 4);
    FSV_ROW_FNS(512, 4, 8, 1, 2, 2);
    FSV_ROW_FNS(1024, 4, 4, 1, 1, 4);
#undef FSV_ROW_FNS
    fns.push_back((const void *)k_abm<8, 8>);
    fns.push_back((const void *)k_abm<16, 8>);
    fns.push_back((const void *)k_ab<512, 4, 8, 1>);
    fns.push_back((const void *)k_ab<512, 5, 6, 1>);
    fns.push_back((const void *)k_pool_rows<double>);
    fns.push_back((const void *)k_pool_rows<float>);
    bool ok = true;
    for (const void *f : fns)
        ok = ok && hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, f == fns[0] ? 163840 : 163328) == hipSuccess;
    g_lds_max = ok ? 163840 : 65536;  // a gfx950 CU's LDS, or what any kernel may use
    (void)hipGetLastError();
}

unsigned combine_grid(int64_t dim) {
    const int64_t tiles = (dim + 1023) / 1024;  // upper bound on 32x32 tiles in use
    return (unsigned)(tiles < 1 ? 1 : (tiles > 1024 ? 1024 : tiles));
}

int cadj_blocks(const PairOp &op, int64_t nsa, int64_t nsb) {
    const CGrid g = cgrid_of(op, nsa, nsb);
    return (int)(g.gx * g.gy);
}

hipError_t launch_crot(int vt, void *psi, const PairOp &op, const uint32_t *lists, const double *cs,
                       int k, int64_t nsa, int64_t nsb, hipStream_t st) {
    switch (vt) {
    case V_C128: return crot_impl<double2>(psi, op, lists, cs, k, nsa, nsb, st);
    case V_C64: return crot_impl<float2>(psi, op, lists, cs, k, nsa, nsb, st);
    case V_F64: return crot_impl<double>(psi, op, lists, cs, k, nsa, nsb, st);
    default: return crot_impl<float>(psi, op, lists, cs, k, nsa, nsb, st);
    }
}

hipError_t launch_cadj(int vt, void *psi, void *lam, const PairOp &op, const uint32_t *lists,
                       const double *cs, int k, int64_t nsa, int64_t nsb, double *partial,
                       hipStream_t st) {
    switch (vt) {
    case V_C128: return cadj_impl<double2>(psi, lam, op, lists, cs, k, nsa, nsb, partial, st);
    case V_C64: return cadj_impl<float2>(psi, lam, op, lists, cs, k, nsa, nsb, partial, st);
    case V_F64: return cadj_impl<double>(psi, lam, op, lists, cs, k, nsa, nsb, partial, st);
    default: return cadj_impl<float>(psi, lam, op, lists, cs, k, nsa, nsb, partial, st);
    }
}

hipError_t launch_cadj_zip(int vt, void *z, const PairOp &op, const uint32_t *lists, const double *cs, int k,
                           int64_t nsa, int64_t nsb, double *partial, hipStream_t st) {
    if (vt == V_F64) return cadj_zip_impl<double>(z, op, lists, cs, k, nsa, nsb, partial, st);
    if (vt == V_F32) return cadj_zip_impl<float>(z, op, lists, cs, k, nsa, nsb, partial, st);
    return hipErrorInvalidValue;
}

hipError_t launch_zip(int vt, const void *psi, const void *lam, void *z, int64_t n, hipStream_t st) {
    if (vt == V_F64) return zip_impl<double>(psi, lam, z, n, st);
    if (vt == V_F32) return zip_impl<float>(psi, lam, z, n, st);
    return hipErrorInvalidValue;
}

hipError_t launch_convert(int vi, const void *in, int vo, void *out, int64_t n, hipStream_t st) {
    if (vi == V_F32 && vo == V_F64) return convert_impl<float, double>(in, out, n, st);
    if (vi == V_F64 && vo == V_F32) return convert_impl<double, float>(in, out, n, st);
    if (vi == V_C64 && vo == V_C128) return convert_impl<float2, double2>(in, out, n, st);
    if (vi == V_C128 && vo == V_C64) return convert_impl<double2, float2>(in, out, n, st);
    if (vi == V_F64 && vo == V_C128) return convert_impl<double, double2>(in, out, n, st);
    if (vi == V_C128 && vo == V_F64) return convert_impl<double2, double>(in, out, n, st);
    return hipErrorInvalidValue;
}

hipError_t launch_sector_sigma(int planes, const SectorTabs &T, const double *C, double *S, double *CT, double *ST,
                               double *epart, hipStream_t st, void *zout, int zvt, bool *zipped) {
    if (zipped) *zipped = false;
    return sigma_impl(planes, T, C, S, CT, ST, epart, st, zout, zvt == V_F32, zipped);
}

hipError_t launch_sector_energy(int planes, const SectorTabs &T, const double *C, double *S, double *CT, double *ST,
                                double *epart, const int32_t *im_flag, int32_t im_epoch, hipStream_t st) {
    if (T.R > 0) return row_launch<ROW_ENERGY>(planes, T, C, nullptr, nullptr, epart, im_flag, im_epoch, st);
    return sigma_impl(planes, T, C, S, CT, ST, epart, st, nullptr, false, nullptr);
}

int sigma_partials(const SectorTabs &T, int planes) {
    return T.R > 0 ? (int)(planes * T.nsa) : (int)combine_grid(T.nsa * T.nsb);
}

hipError_t launch_row_onebody(const double *heff, int M, const uint32_t *sa, int64_t nsa, const uint32_t *sb,
                              int64_t nsb, double *hp, double *hda, double *hdb, hipStream_t st) {
    hipLaunchKernelGGL(k_row_onebody, dim3(blocks_for((int64_t)M * (M - 1) / 2 + nsa + nsb, 256)), dim3(256), 0, st,
                       heff, M, sa, nsa, sb, nsb, hp, hda, hdb);
    return hipGetLastError();
}

hipError_t launch_pool(int vtype, const void *psi, const void *lam, const PairOp *ops, const uint32_t *lists,
                       int n_ops, int gx, int64_t nsa, int64_t nsb, double *partial, hipStream_t st) {
    const dim3 grid((unsigned)gx, (unsigned)n_ops), block(256);
    if (vtype == V_F64)
        hipLaunchKernelGGL(k_pool<double>, grid, block, 0, st, (const double *)psi, (const double *)lam, ops, lists,
                           nsa, nsb, partial);
    else if (vtype == V_F32)
        hipLaunchKernelGGL(k_pool<float>, grid, block, 0, st, (const float *)psi, (const float *)lam, ops, lists,
                           nsa, nsb, partial);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

int pool_rows_u(int vtype, int64_t nsa, int64_t nsb, double pairs, double rows) {
    // row pairs per workgroup: two workgroups of 512 threads per CU while the
    // rows allow it, at least one row pair in a CU's LDS (or in the 64 KiB that
    // are left where a larger block is refused)
    const int64_t per = 4 * nsb * vtype_bytes(vtype), lim = g_lds_max >= 163840 ? 163328 : 65024;
    if ((vtype != V_F64 && vtype != V_F32) || per > lim) return 0;
    // k_pool_rows reads whole rows once per group, k_pool the pairs of every
    // operator.  Times in us, bytes / 1e6 per us = TB/s, fitted to pools of 5 to
    // 1818 operators at 16 to 30 qubits.  k_pool: 10 TB/s while psi and lam fit
    // one XCD's L2 (4 MB; 22 qubits, 400 operators: 20 us, rows 28), 4.9 while
    // they fit all eight (24 qubits, 50 / 200 / 400 / 1818 operators: 13 / 85 /
    // 176 / 860, rows 49 / 87 / 104 / 233), 3.2 beyond (28 qubits with 5 + 5
    // electrons, 50 / 200 / 800 operators: 130 / 590 / 2290, rows 230 / 460 /
    // 720).  Rows: 4.5 TB/s with two workgroups per CU, 2.6 with one (28
    // qubits with 6 + 6 electrons, 200 / 800 operators: 1670 / 2780, k_pool
    // 1160 / 5230), the launches and the operators' LDS reads besides.
    const double amp = vtype_bytes(vtype), state = 2.0 * amp * (double)nsa * (double)nsb;
    const double by_op = 4.0 * amp * pairs, by_row = 4.0 * amp * rows * (double)nsb;
    const double t_op = by_op / (state <= 4e6 ? 10e6 : state <= 32e6 ? 4.9e6 : 3.2e6);
    const double t_row = 12.0 + by_row / (per <= 81664 ? 4.5e6 : 2.6e6) + by_op / 60e6;
    const char *mode = std::getenv("FSV_POOL");  // rows | pairs: whichever the sizes say
    const bool forced = mode && std::strcmp(mode, "rows") == 0;
    if ((mode && std::strcmp(mode, "pairs") == 0) || (!forced && t_op <= t_row)) return 0;
    int64_t u = std::min<int64_t>(81664, lim) / per;
    return (int)(u < 1 ? 1 : (u > kPoolU ? kPoolU : u));
}

template <typename V>
static hipError_t pool_rows_impl(const void *psi, const void *lam, const PairOp *ops, const uint32_t *lists,
                                 const PoolGroup *groups, const int32_t *gops, const int2 *tasks, int n_gen,
                                 int n_plain, int U, int64_t nsb, const int64_t *off, double *partial,
                                 hipStream_t st) {
    // groups with beta lists stage their rows in LDS; the others hold none, so
    // that more of their workgroups run at once
    if (n_gen > 0)
        hipLaunchKernelGGL(k_pool_rows<V>, dim3((unsigned)n_gen), dim3(512), (size_t)U * 4 * nsb * sizeof(V), st,
                           (const V *)psi, (const V *)lam, ops, lists, groups, gops, tasks, U, (int)nsb, off, partial);
    if (n_plain > 0)
        hipLaunchKernelGGL(k_pool_rows<V>, dim3((unsigned)n_plain), dim3(256), 0, st, (const V *)psi, (const V *)lam,
                           ops, lists, groups, gops, tasks + n_gen, kPoolU, (int)nsb, off, partial);
    return hipGetLastError();
}

hipError_t launch_pool_rows(int vtype, const void *psi, const void *lam, const PairOp *ops, const uint32_t *lists,
                            const PoolGroup *groups, const int32_t *gops, const int2 *tasks, int n_gen, int n_plain,
                            int U, int64_t nsb, const int64_t *off, double *partial, int n_ops, double *out,
                            hipStream_t st) {
    const hipError_t e =
        vtype == V_F64 ? pool_rows_impl<double>(psi, lam, ops, lists, groups, gops, tasks, n_gen, n_plain, U, nsb, off,
                                                partial, st)
                       : pool_rows_impl<float>(psi, lam, ops, lists, groups, gops, tasks, n_gen, n_plain, U, nsb, off,
                                               partial, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_pool_reduce, dim3((unsigned)n_ops), dim3(256), 0, st, off, partial, out);
    return hipGetLastError();
}

hipError_t launch_string_h_values(double *val, const double *v2, const int32_t *desc, const uint32_t *str,
                                  const double *ht, int M, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_string_h_values, dim3(blocks_for(n, 256)), dim3(256), 0, st, val, v2, desc, str, ht, M, n);
    return hipGetLastError();
}

hipError_t launch_csr_dense(const int64_t *rowptr, const int32_t *col, const double *val, double *out, int64_t n,
                            hipStream_t st) {
    hipLaunchKernelGGL(k_csr_dense, dim3((unsigned)n), dim3(256), 0, st, rowptr, col, val, out, n);
    return hipGetLastError();
}

hipError_t launch_plane_transpose(const double *in, double *out, int64_t rows, int64_t cols, int planes,
                                  hipStream_t st) {
    hipLaunchKernelGGL(k_transpose,
                       dim3((unsigned)((cols + 31) / 32), (unsigned)((rows + 31) / 32), (unsigned)planes), dim3(32, 8), 0,
                       st, in, out, rows, cols, planes * cols, planes * rows, cols, rows);
    return hipGetLastError();
}

hipError_t launch_dense_image(int precision, int ordering, void *out, const double *S, const int32_t *ra,
                              const int2 *rb, int n, int na, int nb, int64_t nsb, hipStream_t st) {
    const uint64_t chunks = ((1ull << n) + (1u << kImageBits) - 1) >> kImageBits;
    const dim3 grid((unsigned)std::min<uint64_t>(chunks, 65536)), block(kImageBlock);
    const bool stream = ((precision == 0 ? 16ull : 8ull) << n) > (512ull << 20);
#define FSV_IMAGE(O, BLOCKED, STREAM)                                                                           \
    hipLaunchKernelGGL((k_dense_image<O, BLOCKED, STREAM>), grid, block, 0, st, (O *)out, S, ra, rb, n, na, nb, nsb)
    if (precision == 0 && stream && ordering == 0)
        FSV_IMAGE(double2, false, true);
    else if (precision == 0 && stream)
        FSV_IMAGE(double2, true, true);
    else if (precision == 0 && ordering == 0)
        FSV_IMAGE(double2, false, false);
    else if (precision == 0)
        FSV_IMAGE(double2, true, false);
    else if (stream && ordering == 0)
        FSV_IMAGE(float2, false, true);
    else if (stream)
        FSV_IMAGE(float2, true, true);
    else if (ordering == 0)
        FSV_IMAGE(float2, false, false);
    else
        FSV_IMAGE(float2, true, false);
#undef FSV_IMAGE
    return hipGetLastError();
}

}  // namespace fsv
