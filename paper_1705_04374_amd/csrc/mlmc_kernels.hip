// OF-MLMC estimator kernels (Sukys et al., arXiv:1705.04374, Sec. 2.4.3-2.4.4),
// all in double on the device.  The statistics are small next to the solves
// (Appendix A.3 notes the coefficient system is never a bottleneck), so each
// call is one workgroup without scratch memory; the sums are deterministic
// (fixed-order strided partial sums, then a fixed tree).
#include "flow_kernels.h"

#include <math.h>

namespace ofm {

// Fixed-order workgroup sums of three doubles per thread: a butterfly within
// each wavefront, then the wavefronts in order.
template <int NT> __device__ __forceinline__ void block_sum3(double (&v)[3])
{
    constexpr int NW = NT / 64;
    __shared__ double sh[NW][3];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] += __shfl_xor(v[k], off, 64);
    __syncthreads();                                   // the previous sums have been read
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < 3; ++k) sh[threadIdx.x >> 6][k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        v[k] = 0.0;
        for (int w = 0; w < NW; ++w) v[k] += sh[w][k];
    }
}

// Moments of one term: (M_used, mean_f, mean_c, Var_f, Var_c, Cov), two-pass,
// by one workgroup.  Bound by the latency of its loads: each thread has those
// of eight samples in flight (of 16: half the speed, at 128 registers a
// thread), and there are 16 wavefronts where 4 would take more than four such
// groups in turn: from 8192 samples (the kernel alone, us, without and with
// coarse values: 1024 samples 3.7 and 4.2 with 4, 8.3 and 9.4 with 16; 6000,
// 6.8 and 8.0, 8.4 and 9.4; 8192, 8.1 and 10.0, 8.4 and 9.5).  65536 samples
// without coarse values: 119 us before (4 wavefronts, a sample at a time, six
// sums through LDS), 31 now; 3276 samples 10.2 and 5.4; 10^6, 5450 and 570.
template <int NT>
__global__ void __launch_bounds__(NT) moments_kernel(const double* __restrict__ qf, const double* __restrict__ qc,
                                                     const int32_t* __restrict__ ok, int64_t M,
                                                     double* __restrict__ out)
{
    constexpr int U = 8;
    // visit(f, c) of this thread's samples in use, in increasing order
    auto each = [&](auto visit) {
        for (int64_t i0 = threadIdx.x; i0 < M; i0 += (int64_t)U * NT) {
            int64_t j[U];
            double f[U], c[U];
            bool use[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int64_t i = i0 + (int64_t)k * NT;
                use[k] = i < M;
                j[k] = i < M ? i : M - 1;
                f[k] = qf[j[k]];
                c[k] = 0.0;
            }
            if (qc)
#pragma unroll
                for (int k = 0; k < U; ++k) c[k] = qc[j[k]];
            if (ok) {
                int32_t o[U];
#pragma unroll
                for (int k = 0; k < U; ++k) o[k] = ok[j[k]];
#pragma unroll
                for (int k = 0; k < U; ++k) use[k] = use[k] && o[k] != 0;
            }
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (use[k]) visit(f[k], c[k]);
        }
    };
    double s[3] = { 0.0, 0.0, 0.0 };
    each([&](double f, double c) {
        s[0] += 1.0;
        s[1] += f;
        s[2] += c;
    });
    block_sum3<NT>(s);
    const double m = s[0];
    const double mf = m > 0.0 ? s[1] / m : 0.0;
    const double mc = m > 0.0 ? s[2] / m : 0.0;
    double v[3] = { 0.0, 0.0, 0.0 };
    each([&](double f, double c) {
        const double df = f - mf, dc = c - mc;
        v[0] += df * df;
        v[1] += dc * dc;
        v[2] += df * dc;
    });
    block_sum3<NT>(v);
    if (threadIdx.x == 0) {
        out[0] = m;
        out[1] = mf;
        out[2] = mc;
        const bool two = m >= 2.0;
        out[3] = two ? v[0] / (m - 1.0) : 0.0;
        out[4] = two && qc ? v[1] / (m - 1.0) : 0.0;
        out[5] = two && qc ? v[2] / (m - 1.0) : 0.0;
    }
}

// The kernels below run a handful of operations per term, L + 1 <= 32 terms:
// one wavefront reads all it needs at once into LDS (one memory latency, not
// one per operand), takes what is independent per term with a lane each, and
// adds up in the order of the terms.  Four terms, one thread before and now
// (us): coefficients 4.6 and 2.3, errors 4.6 and 1.5, estimate 5.2 and 1.4,
// sample counts (arrays in scratch memory before) 9.1 and 1.9.
constexpr int kTerms = 32;
__device__ __forceinline__ void fetch(double* sh, const double* g, int n)
{
    for (int i = threadIdx.x; i < n; i += 64) sh[i] = g[i];
}

// Tridiagonal system of eq. (alpha-matvec), generalised to per-term
// estimates: row k is the derivative of the estimated cost
// sum_l W_l Var(alpha_l q_f,l - alpha_{l-1} q_c,l) with respect to alpha_k.
// Thomas algorithm; a non-positive pivot means the estimates are not
// positive definite -> flag OFM_ESINGULAR and alpha = 1 (classical MLMC).
__global__ void __launch_bounds__(64) coefficients_kernel(int L, const double* gmom, const double* gW, double* alpha,
                                                          int32_t* flag)
{
    __shared__ double mom[6 * kTerms], W[kTerms], cp[kTerms], dp[kTerms];
    fetch(mom, gmom, 6 * (L + 1));
    fetch(W, gW, L + 1);
    __syncthreads();
    if (threadIdx.x != 0) return;
    int bad = 0;
    for (int k = 0; k < L; ++k) {
        const double diag = mom[6 * k + 3] * W[k] + mom[6 * (k + 1) + 4] * W[k + 1];
        const double low = k >= 1 ? -mom[6 * k + 5] * W[k] : 0.0;
        const double up = k + 1 <= L - 1 ? -mom[6 * (k + 1) + 5] * W[k + 1] : 0.0;
        const double rhs = k == L - 1 ? mom[6 * L + 5] * W[L] : 0.0;
        const double piv = diag - (k >= 1 ? low * cp[k - 1] : 0.0);
        if (!(piv > 0.0) || fabs(piv) < 1e-300) { bad = 1; break; }
        cp[k] = up / piv;
        dp[k] = (rhs - (k >= 1 ? low * dp[k - 1] : 0.0)) / piv;
    }
    alpha[L] = 1.0;
    if (bad) {
        for (int k = 0; k < L; ++k) alpha[k] = 1.0;
        *flag = OFM_ESINGULAR;
        return;
    }
    double next = 1.0;
    for (int k = L - 1; k >= 0; --k) alpha[k] = next = dp[k] - (k + 1 <= L - 1 ? cp[k] * next : 0.0);
    *flag = 0;
}

// eq. (ocv-mlmc-err): per-term variances of the weighted differences and
// the squared sampling error.
__global__ void __launch_bounds__(64) errors_kernel(int L, const double* gmom, const double* galpha, double* sig,
                                                    double* eps2)
{
    __shared__ double mom[6 * kTerms], alpha[kTerms], part[kTerms];
    fetch(mom, gmom, 6 * (L + 1));
    fetch(alpha, galpha, L + 1);
    __syncthreads();
    const int l = threadIdx.x;
    if (l <= L) {
        const double* m = mom + 6 * l;
        double s = alpha[l] * alpha[l] * m[3];
        if (l >= 1) s += alpha[l - 1] * alpha[l - 1] * m[4] - 2.0 * alpha[l] * alpha[l - 1] * m[5];
        sig[l] = s;
        part[l] = s / m[0];
    }
    __syncthreads();
    if (l != 0) return;
    double e = 0.0;
    for (int k = 0; k <= L; ++k) e += part[k];
    *eps2 = e;
}

// eq. (ocv-mlmc): the estimator.
__global__ void __launch_bounds__(64) estimate_kernel(int L, const double* gmom, const double* galpha, double* E)
{
    __shared__ double mom[6 * kTerms], alpha[kTerms];
    fetch(mom, gmom, 6 * (L + 1));
    fetch(alpha, galpha, L + 1);
    __syncthreads();
    if (threadIdx.x != 0) return;
    double e = alpha[0] * mom[1];
    for (int l = 1; l <= L; ++l) e += alpha[l] * mom[6 * l + 1] - alpha[l - 1] * mom[6 * l + 2];
    *E = e;
}

// eq. (M-tol) / eq. (M-budget) with the keep-computed-samples loop of step 7.
// Lane l holds term l.
__global__ void __launch_bounds__(64) optimal_M_kernel(int L, const double* sig, const double* W, const int64_t* have,
                                                       int mode, double target, int64_t* out, int32_t* flag)
{
#pragma clang fp contract(off)
    __shared__ double spent[kTerms], root[kTerms];      // of a term: its share once fixed, sqrt(sig W)
    const int l = threadIdx.x;
    const bool mine = l <= L;
    const bool tol = mode == OFM_MODE_TOLERANCE;
    double ratio = 0.0;                                 // sqrt(sig / W)
    int64_t n = 0, M = 0;
    if (mine) {
        const double s = sig[l], w = W[l];
        n = M = have[l];
        spent[l] = tol ? s / (double)n : (double)n * w;
        root[l] = sqrt(s * w);
        ratio = sqrt(s / w);
    }
    __syncthreads();
    if (l == 0) *flag = 0;
    uint64_t fixed = 0;                                 // the same in every lane
    for (int it = 0; it <= L + 1; ++it) {
        double rest = tol ? target * target : target;
        double S = 0.0;
        for (int k = 0; k <= L; ++k) {
            if (fixed >> k & 1) rest -= spent[k];
            else S += root[k];
        }
        if (tol && !(rest > 0.0)) {
            if (l == 0) *flag = OFM_EINFEASIBLE;
            if (mine) out[l] = n;
            return;
        }
        const bool is_free = mine && !(fixed >> l & 1);
        if (is_free) {
            double m;
            if (tol) m = ceil(ratio * S / rest);
            else m = (rest > 0.0 && S > 0.0) ? ceil(rest * ratio / S) : 0.0;
            M = (int64_t)m;
        }
        const uint64_t now = __ballot(is_free && M < n);
        fixed |= now;
        if (now == 0 || __ballot(mine && !(fixed >> l & 1)) == 0) break;
    }
    if (mine) out[l] = fixed >> l & 1 ? n : M;
}

// Inferred variances of level differences (the optional part of step 3 of
// the adaptive algorithm, Sec. 2.4.4; App. A.1): a weighted least-squares
// line through ln V[q_l - q_{l-1}] against l over the terms l = first..L
// with at least two samples, weights (M_l - 1)/2 (Gaussian errors of a
// sample variance's logarithm).  Terms l >= max(first, 1) with fewer than
// two samples get their moments from the fit: the coarse member takes the
// variance of level l-1 (term l-1's fine variance Vc), the members'
// correlation rho is that of term l-1, and the fine member's deviation s
// gives the inferred difference variance s^2 + Vc - 2 rho s sqrt(Vc).  Terms
// with at least two but fewer than m_floor samples keep the inferred value as
// a floor of their difference variance (their few samples refine it, App.
// A.1): the covariance is lowered to (Vf + Vc - vhat) / 2, at least
// -sqrt(Vf Vc).  One thread: L is a handful of terms.
__global__ void fit_kernel(int L, int first, int m_floor, double* mom, double* vhat, int32_t* flag)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double S = 0.0, Sx = 0.0, Sy = 0.0, Sxx = 0.0, Sxy = 0.0;
    int np = 0;
    for (int l = first; l <= L; ++l) {
        const double* m = mom + 6 * l;
        const double V = m[3] + m[4] - 2.0 * m[5];
        if (m[0] >= 2.0 && V > 0.0) {
            const double y = log(V), w = (m[0] - 1.0) / 2.0, x = (double)l;
            S += w;
            Sx += w * x;
            Sy += w * y;
            Sxx += w * x * x;
            Sxy += w * x * y;
            ++np;
        }
    }
    for (int l = 0; l <= L; ++l) vhat[l] = 0.0;
    if (np < 2) {
        *flag = OFM_ESINGULAR;
        return;
    }
    const double b = (S * Sxy - Sx * Sy) / (S * Sxx - Sx * Sx);
    const double a = (Sy - b * Sx) / S;
    for (int l = first; l <= L; ++l) vhat[l] = exp(a + b * (double)l);
    // terms with fewer than two samples: coarse member = level l-1 (term
    // l-1's fine variance), the members' correlation that of term l-1, and
    // the fine member's deviation s >= 0 from s^2 + Vc - 2 rho s sqrt(Vc) =
    // vhat (larger root).  Where vhat is below the smallest difference
    // variance that correlation allows, s takes the minimiser max(rho
    // sqrt(Vc), 0): (1 - rho^2) Vc for rho >= 0, Vc (s = 0) for rho < 0.
    for (int l = first > 1 ? first : 1; l <= L; ++l) {
        double* m = mom + 6 * l;
        if (m[0] >= 2.0) continue;
        const double* b = mom + 6 * (l - 1);
        double rho = (b[3] > 0.0 && b[4] > 0.0) ? b[5] / sqrt(b[3] * b[4]) : 0.0;
        rho = fmin(fmax(rho, -1.0), 1.0);
        const double vc = b[3], sc = sqrt(vc);
        const double s = fmax(rho * sc + sqrt(fmax(vhat[l] - (1.0 - rho * rho) * vc, 0.0)), 0.0);
        m[4] = vc;
        m[3] = s * s;
        m[5] = rho * s * sc;
    }
    // terms with 2 <= M < m_floor: the inferred value as a floor
    for (int l = first > 1 ? first : 1; l <= L; ++l) {
        double* m = mom + 6 * l;
        if (!(m[0] >= 2.0 && m[0] < (double)m_floor)) continue;
        const double v = m[3] + m[4] - 2.0 * m[5];
        if (!(vhat[l] > v)) continue;
        m[5] = fmax(0.5 * (m[3] + m[4] - vhat[l]), -sqrt(m[3] * m[4]));
    }
    *flag = 0;
}

// Moments of each term over the union of two disjoint sample sets
// (pairwise update: the centred sums add, plus Ma Mb / M times the product of
// the differences of the means); one thread per term.  out may be a or b.
__global__ void merge_kernel(int n_terms, const double* a, const double* b, double* out)
{
    const int t = threadIdx.x;
    if (t >= n_terms) return;
    const double* x = a + 6 * t;
    const double* y = b + 6 * t;
    const double na = x[0], nb = y[0];
    double r[6];
    if (na == 0.0 || nb == 0.0) {
        for (int k = 0; k < 6; ++k) r[k] = na == 0.0 ? y[k] : x[k];
    } else {
        const double n = na + nb;
        const double df = y[1] - x[1], dc = y[2] - x[2];
        const double w = na * nb / n;
        const double sff = x[3] * (na - 1.0) + y[3] * (nb - 1.0) + df * df * w;
        const double scc = x[4] * (na - 1.0) + y[4] * (nb - 1.0) + dc * dc * w;
        const double sfc = x[5] * (na - 1.0) + y[5] * (nb - 1.0) + df * dc * w;
        r[0] = n;
        r[1] = x[1] + df * nb / n;
        r[2] = x[2] + dc * nb / n;
        r[3] = n >= 2.0 ? sff / (n - 1.0) : 0.0;
        r[4] = n >= 2.0 ? scc / (n - 1.0) : 0.0;
        r[5] = n >= 2.0 ? sfc / (n - 1.0) : 0.0;
    }
    for (int k = 0; k < 6; ++k) out[6 * t + k] = r[k];
}

hipError_t launch_merge(int n_terms, const double* a, const double* b, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(merge_kernel, dim3(1), dim3(64), 0, s, n_terms, a, b, out);
    return hipGetLastError();
}

hipError_t launch_fit(int L, int first, int m_floor, double* mom, double* vhat, int32_t* flag, hipStream_t s)
{
    hipLaunchKernelGGL(fit_kernel, dim3(1), dim3(64), 0, s, L, first, m_floor, mom, vhat, flag);
    return hipGetLastError();
}

hipError_t launch_moments(const double* qf, const double* qc, const int32_t* ok, int64_t M, double* out,
                          hipStream_t s)
{
    if (M < 8192)
        hipLaunchKernelGGL((moments_kernel<256>), dim3(1), dim3(256), 0, s, qf, qc, ok, M, out);
    else
        hipLaunchKernelGGL((moments_kernel<1024>), dim3(1), dim3(1024), 0, s, qf, qc, ok, M, out);
    return hipGetLastError();
}

hipError_t launch_coefficients(int L, const double* mom, const double* W, double* alpha, int32_t* flag, hipStream_t s)
{
    hipLaunchKernelGGL(coefficients_kernel, dim3(1), dim3(64), 0, s, L, mom, W, alpha, flag);
    return hipGetLastError();
}

hipError_t launch_errors(int L, const double* mom, const double* alpha, double* sig, double* eps2, hipStream_t s)
{
    hipLaunchKernelGGL(errors_kernel, dim3(1), dim3(64), 0, s, L, mom, alpha, sig, eps2);
    return hipGetLastError();
}

hipError_t launch_estimate(int L, const double* mom, const double* alpha, double* E, hipStream_t s)
{
    hipLaunchKernelGGL(estimate_kernel, dim3(1), dim3(64), 0, s, L, mom, alpha, E);
    return hipGetLastError();
}

hipError_t launch_optimal_M(int L, const double* sig, const double* W, const int64_t* have, int mode, double target,
                            int64_t* out, int32_t* flag, hipStream_t s)
{
    hipLaunchKernelGGL(optimal_M_kernel, dim3(1), dim3(64), 0, s, L, sig, W, have, mode, target, out, flag);
    return hipGetLastError();
}

}  // namespace ofm
