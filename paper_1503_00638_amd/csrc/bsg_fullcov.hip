// Full-covariance noise for small arrays (Masui et al., Section 3.1, Eqs.
// rad_full1-3 and Eq. noise): per (frequency, time) the covariance of the
// I^2 real degrees of freedom of the visibilities (Re of every product, Im
// of every cross product, in product order), the noise of each degree of
// freedom s_k^2 = 1 / (C^-1)_kk, and the rounding of Section 3.2 with
// G2 = 12 f s_k^2.  With Q = 2N C this is G2 = c / (Q^-1)_kk, c = (12 f)/(2N).
//
// A grid of G x G threads takes one sample and keeps its matrices in
// registers: thread (r, c) holds the elements (G a + r, G b + c), a >= b, of
// the lower triangle of Q, NT x NT tiles with G NT >= D = I^2.  A step of the
// right-looking Cholesky factorisation Q = L L^T (and then of the inverse
// M = L^-1, row by row) passes one column (and one row) through LDS and is
// otherwise NT^2 / 2 independent multiply-subtracts per thread, without an
// LDS access per element; the step's D divisions go one to a thread.
// (Q^-1)_kk = sum_i M_ik^2.  Up to 8 inputs a sample is one wavefront (G = 8,
// no barriers), above that a workgroup of four (G = 16).
//
// What bounds it: with the elements in LDS (one workgroup per sample, 256 or
// 512 threads) every multiply-subtract paid an LDS read and write and every
// column two barriers: 7.36 ms for 65,536 samples of 8 inputs (1.56 TFLOP/s)
// and 16.3 ms for 16,384 of 11.  With them in registers 1.54 and 2.92 ms
// (7.5 and 6.6 TFLOP/s): vector issue (per column and thread about 30
// multiplies and subtracts in the factorisation and 30 in the inverse, against
// a square root, two divisions and four LDS round trips), four waves per SIMD
// (128 VGPRs) hiding the chain.  The chain
// alone, 16 samples in a call: 51 us (8 inputs, 102 before), 128 us (11,
// 258 before).  The tile count follows the input count because its loops
// are unrolled: a smaller array does not carry a larger one's tiles.
//
// Every element sees its operations in the same order as a plain serial
// implementation (sums in increasing index order, products and sums rounded
// separately), so the results are reproducible bit for bit.  (Zeros may
// differ in sign on the way, which no nonzero value sees.)  A sample whose Q
// is not positive definite gets no estimate and is left unchanged.
#include <cmath>

#include "bsg_internal.hpp"
#include "bsg_round_dev.hpp"

namespace bsg {

namespace {

constexpr int kMaxInputs = 11; // D = 121 degrees of freedom

struct Cplx {
    double re, im;
};

__device__ __forceinline__ Cplx mul_conj(Cplx a, Cplx b) // a * conj(b)
{
    return Cplx{a.re * b.re + a.im * b.im, a.im * b.re - a.re * b.im};
}

// Degree of freedom k of I inputs as i | j << 8 | (Im ? 1 << 16 : 0).  The
// products (i, i), (i, i + 1), .. of row i have 2 (I - i) - 1 of them, so row
// i starts at I^2 - (I - i)^2.
__device__ __forceinline__ int dof_of(int I, int k)
{
    int n = (int)__builtin_sqrtf((float)(I * I - k));
    while (n * n < I * I - k) ++n;
    while (n > 1 && (n - 1) * (n - 1) >= I * I - k) --n;
    const int i = I - n, o = k - (I * I - n * n);
    return i | (i + ((o + 1) >> 1)) << 8 | (o > 0 && !(o & 1) ? 1 << 16 : 0);
}

struct FullcovArgs {
    const float2 *vis;
    const float *autos;
    int64_t F, T;
    int I, P, D;
    double c;
    float2 *vis_out;  // nullptr: only the inverse diagonal
    double *qdiag;    // [F][T][D] or nullptr
};

// Orders a sample's LDS accesses: a barrier, or a fence where one wavefront
// owns the sample (its LDS accesses complete in order).
template <int G> __device__ __forceinline__ void sample_sync()
{
    if constexpr (G * G == kWave)
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    else
        __syncthreads();
}

template <int G, int NT>
__global__ __launch_bounds__(G * G) void k_fullcov(FullcovArgs a)
{
    constexpr int N = G * NT;
    static_assert(N <= G * G, "a thread per row");
    __shared__ double raw[N], col[N], row[N], diag[N];
    __shared__ Cplx V[N]; // I x I
    __shared__ int dof[N];
    const int D = a.D, I = a.I, P = a.P;
    const int tid = threadIdx.x, r = tid / G, c = tid % G;
    const int64_t s = blockIdx.x; // sample (fr, t)
    const int64_t fr = s / a.T, t = s - fr * a.T;

    if (tid < N) dof[tid] = tid < D ? dof_of(I, tid) : 0;
    if (tid < D) {
        const int x = tid / I, y = tid - x * I;
        Cplx v;
        if (x == y) {
            v.re = a.autos[(fr * I + x) * a.T + t];
            v.im = 0.0;
        } else {
            const int lo = x < y ? x : y, hi = x < y ? y : x;
            const int p = lo * I - lo * (lo - 1) / 2 + (hi - lo);
            const float2 w = a.vis[(fr * P + p) * a.T + t];
            v.re = w.x;
            v.im = x < y ? (double)w.y : -(double)w.y;
        }
        V[tid] = v;
    }
    sample_sync<G>();

    // Q = 2N C (Eqs. rad_full1-3): with A = V_ig conj(V_jh) and B = V_ih
    // conj(V_jg), Re A + Re B between two real parts, Re A - Re B between two
    // imaginary parts, Im B - Im A for (Re ij, Im gh), Im B + Im A for
    // (Im ij, Re gh).
    double q[NT][NT];
    {
        int rd[NT], cd[NT];
#pragma unroll
        for (int x = 0; x < NT; ++x) {
            rd[x] = dof[G * x + r];
            cd[x] = dof[G * x + c];
        }
#pragma unroll
        for (int x = 0; x < NT; ++x) {
            const int i = rd[x] & 255, j = rd[x] >> 8 & 255, ix = rd[x] >> 16;
#pragma unroll
            for (int y = 0; y <= x; ++y) {
                const int g = cd[y] & 255, h = cd[y] >> 8 & 255, iy = cd[y] >> 16;
                const Cplx A = mul_conj(V[i * I + g], V[j * I + h]);
                const Cplx B = mul_conj(V[i * I + h], V[j * I + g]);
                const bool same = ix == iy;
                const double u = same ? A.re : B.im, w = same ? B.re : A.im;
                q[x][y] = same == (ix == 0) ? u + w : u - w;
            }
        }
    }

    // Cholesky, right-looking: step k = G kb + kc
    bool bad = false;
#pragma unroll
    for (int kb = 0; kb < NT; ++kb) {
        for (int kc = 0; kc < G && !bad; ++kc) {
            const int k = G * kb + kc;
            if (k >= D) break;
            if (c == kc) {
#pragma unroll
                for (int x = kb; x < NT; ++x) raw[G * x + r] = q[x][kb];
            }
            sample_sync<G>();
            const double d = raw[k]; // the same for every thread
            bad = !(d > 0.0) || d == __builtin_inf();
            const double lkk = sqrt(d);
            if (tid < N) {
                const double l = raw[tid] / lkk;
                col[tid] = tid == k ? lkk : (tid > k && tid < D ? l : 0.0);
            }
            if (tid == k) diag[k] = lkk;
            sample_sync<G>();
            double ri[NT], cj[NT];
#pragma unroll
            for (int x = kb; x < NT; ++x) {
                ri[x] = col[G * x + r];
                cj[x] = col[G * x + c];
            }
            // column k takes its final values, the columns before it keep theirs
            if (c <= kc) cj[kb] = 0.0;
#pragma unroll
            for (int x = kb; x < NT; ++x) {
                const double v = q[x][kb] - ri[x] * cj[kb];
                q[x][kb] = c == kc ? ri[x] : v;
#pragma unroll
                for (int y = kb + 1; y <= x; ++y) q[x][y] = q[x][y] - ri[x] * cj[y];
            }
        }
    }
    sample_sync<G>();

    // M = L^-1: step k = G kb + kc forms row k, M_kj = -(sum_{j <= m < k}
    // L_km M_mj) / L_kk in thread j, adds its squares to (Q^-1)_jj and its
    // products with column k of L to the sums of the rows below.
    double qk = 0.0;
    if (!bad) {
        double m[NT][NT];
#pragma unroll
        for (int kb = 0; kb < NT; ++kb) {
#pragma unroll
            for (int x = kb; x < NT; ++x) m[x][kb] = 0.0;
            for (int kc = 0; kc < G; ++kc) {
                const int k = G * kb + kc;
                if (k >= D) break;
                if (r == kc) {
#pragma unroll
                    for (int y = 0; y <= kb; ++y) raw[G * y + c] = m[kb][y];
                }
                if (c == kc) {
#pragma unroll
                    for (int x = kb; x < NT; ++x) col[G * x + r] = q[x][kb];
                }
                sample_sync<G>();
                double li[NT];
#pragma unroll
                for (int x = kb; x < NT; ++x) li[x] = col[G * x + r];
                if (tid < N) {
                    const double num = tid < k ? -raw[tid] : 1.0;
                    const double v = tid <= k ? num / diag[k] : 0.0;
                    row[tid] = v;
                    qk = qk + v * v;
                }
                sample_sync<G>();
#pragma unroll
                for (int y = 0; y <= kb; ++y) {
                    const double mj = row[G * y + c];
#pragma unroll
                    for (int x = kb; x < NT; ++x) m[x][y] = m[x][y] + li[x] * mj;
                }
            }
        }
    } else {
        qk = __builtin_nan("");
    }
    if (tid >= D) return;
    if (a.qdiag) a.qdiag[s * D + tid] = qk;
    if (!a.vis_out) return;
    // round degree of freedom k = tid
    const int i = dof[tid] & 255, j = dof[tid] >> 8 & 255, im = dof[tid] >> 16;
    const int p = i * I - i * (i - 1) / 2 + (j - i);
    const int64_t e = (fr * P + p) * a.T + t;
    const float x = im ? a.vis[e].y : a.vis[e].x;
    const uint32_t o = round_noise_bits(__float_as_uint(x), a.c / qk);
    float *out = reinterpret_cast<float *>(a.vis_out + e);
    out[im] = __uint_as_float(o);
    if (i == j) out[1] = a.vis[e].y; // Im of an auto is copied
}

template <int G, int NT> hipError_t fullcov_launch(const FullcovArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL((k_fullcov<G, NT>), dim3((unsigned)(a.F * a.T)), dim3(G * G), 0, s, a);
    return hipGetLastError();
}

} // namespace

int fullcov_max_inputs() { return kMaxInputs; }

hipError_t launch_fullcov(const float *vis, const float *autos, int64_t F, int64_t I, int64_t T,
                          double c, float *vis_out, double *qdiag, hipStream_t s)
{
    const int D = (int)(I * I), P = (int)(I * (I + 1) / 2);
    if (F * T == 0 || D == 0) return hipSuccess;
    FullcovArgs a{reinterpret_cast<const float2 *>(vis), autos, F, T, (int)I, P, D, c,
                  reinterpret_cast<float2 *>(vis_out), qdiag};
    switch (I) { // the fewest tiles that hold D
    case 1:
    case 2: return fullcov_launch<8, 1>(a, s);
    case 3:
    case 4: return fullcov_launch<8, 2>(a, s);
    case 5: return fullcov_launch<8, 4>(a, s);
    case 6: return fullcov_launch<8, 5>(a, s);
    case 7: return fullcov_launch<8, 7>(a, s);
    case 8: return fullcov_launch<8, 8>(a, s);
    case 9: return fullcov_launch<16, 6>(a, s);
    case 10: return fullcov_launch<16, 7>(a, s);
    default: return fullcov_launch<16, 8>(a, s);
    }
}

} // namespace bsg
