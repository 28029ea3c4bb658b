// Stage 1: noise-relative precision reduction (Masui et al., Section 3).
//
// Per visibility (freq f, product p = (i, j), time t):
//   G2 = 12 f s^2 with s from the diagonal radiometer equation (Section 3.1):
//        s^2 = V_ii V_jj / (2N) for i != j, s^2 = V_ii^2 / N for autos,
//   g  = the largest power of two with g^2 < G2 (Eq. trunc_error, strict),
//   re and im are rounded to the nearest multiple of g, ties to even (the
//   tie-breaking footnote of Section 3.2); Im of an auto carries no noise
//   and is left alone.
//
// The value is scaled by 2^-k in double, rounded half to even there and
// scaled back (both scalings exact); k comes from the exponent and mantissa
// of the double G2 (frexp): no log, sqrt or division.
#include <algorithm>

#include "bsg_internal.hpp"
#include "bsg_round_dev.hpp"

namespace bsg {

namespace {

constexpr int kComplexPerThread = 4;

// K visibilities of one or two rows (see RowRun), 16-byte aligned: values and
// autos are all loaded before the first is rounded, without a branch.
template <bool TWO>
__device__ __forceinline__ void round_run(const float2 *__restrict__ vin, float2 *__restrict__ vout,
                                          const RoundParams &rp, const VisCursor &c)
{
    constexpr int K = kComplexPerThread;
    const float4 *v4 = reinterpret_cast<const float4 *>(vin);
    float4 v[K / 2];
#pragma unroll
    for (int k = 0; k < K / 2; ++k) v[k] = v4[k];
    const RowRun<K, TWO, float> row(rp, c, rp.autos);
    float ai[K], aj[K];
    double sc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        ai[k] = row.ai(k);
        aj[k] = row.aj(k);
        sc[k] = 1.0;
    }
    if (rp.fscale) {
#pragma unroll
        for (int k = 0; k < K; ++k) sc[k] = row.factor(k);
    }
    float4 *o4 = reinterpret_cast<float4 *>(vout);
#pragma unroll
    for (int k = 0; k < K / 2; ++k) {
        uint32_t x[4] = {__float_as_uint(v[k].x), __float_as_uint(v[k].y), __float_as_uint(v[k].z),
                         __float_as_uint(v[k].w)};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = 2 * k + h;
            const bool is_auto = row.is_auto(j);
            double G2 = ((double)ai[j] * (double)aj[j]) * (is_auto ? rp.c_auto : rp.c);
            if (rp.fscale) G2 *= sc[j];
            x[2 * h] = round_noise_bits_nb(x[2 * h], G2);
            if (!is_auto) x[2 * h + 1] = round_noise_bits_nb(x[2 * h + 1], G2);
        }
        o4[k] = make_float4(__uint_as_float(x[0]), __uint_as_float(x[1]), __uint_as_float(x[2]),
                            __uint_as_float(x[3]));
    }
}

// As round_run, for int32 visibilities and autos (exact int64 products).
template <bool TWO>
__device__ __forceinline__ void round_run(const int2 *__restrict__ vin, int2 *__restrict__ vout,
                                          const RoundParams &rp, const VisCursor &c)
{
    constexpr int K = kComplexPerThread;
    const int4 *v4 = reinterpret_cast<const int4 *>(vin);
    int4 v[K / 2];
#pragma unroll
    for (int k = 0; k < K / 2; ++k) v[k] = v4[k];
    const RowRun<K, TWO, int32_t> row(rp, c, rp.autos_i32);
    int64_t ai[K], aj[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        ai[k] = row.ai(k);
        aj[k] = row.aj(k);
    }
    int4 *o4 = reinterpret_cast<int4 *>(vout);
#pragma unroll
    for (int k = 0; k < K / 2; ++k) {
        int32_t x[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = 2 * k + h;
            const bool is_auto = row.is_auto(j);
            const double G2 = (double)(ai[j] * aj[j]) * (is_auto ? rp.c_auto : rp.c);
            // (no estimate: k = 0, which changes nothing)
            const int kk = G2 > 0.0 && G2 != __builtin_inf() ? granularity_k(G2) : 0;
            x[2 * h] = round_int(x[2 * h], kk);
            x[2 * h + 1] = round_int(x[2 * h + 1], is_auto ? 0 : kk);
        }
        o4[k] = make_int4(x[0], x[1], x[2], x[3]);
    }
}

__device__ __forceinline__ float2 round_one(float2 v, const VisCursor &c, const RoundParams &rp)
{
    return round_at(v, c, rp);
}
__device__ __forceinline__ int2 round_one(int2 v, const VisCursor &c, const RoundParams &rp)
{
    return round_at_i32(v, c, rp);
}

// Lane i of the grid rounds the kComplexPerThread consecutive visibilities
// from e0 = i * kComplexPerThread: a run of one row where T is a multiple of
// 4, of two where T is at least 4; else (and at the array's end, or for
// unaligned buffers) a cursor steps through them one by one.  (In two rows
// every lane takes both bases.  Stepping was 42 us for 64 MB of integers at
// 30 times, this is 28: HBM.)
template <typename V2>
__global__ __launch_bounds__(256) void k_round(const V2 *__restrict__ vin, V2 *__restrict__ vout,
                                               RoundParams rp, int64_t n_complex, int aligned16)
{
    constexpr int K = kComplexPerThread;
    const int64_t e0 = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) * K;
    if (e0 >= n_complex) return;
    VisCursor c = cursor_at(rp, e0);
    if (aligned16 && e0 + K <= n_complex && rp.T >= K) {
        if (rp.T % K == 0)
            round_run<false>(vin + e0, vout + e0, rp, c);
        else
            round_run<true>(vin + e0, vout + e0, rp, c);
        return;
    }
    for (int k = 0; k < K && e0 + k < n_complex; ++k) {
        if (k) cursor_advance(rp, c, 1);
        vout[e0 + k] = round_one(vin[e0 + k], c, rp);
    }
}

// Compensation of the diagonal noise model (Section 3.2): per (frequency,
// time) the minimum over cross products of 1 - |V_ij|^2 / (V_ii V_jj), in
// double and in that order (products with V_ii V_jj not positive and finite
// skipped, 1 when none is left).  A workgroup of 512 threads (1024 where the
// grid leaves CUs empty: 24 inputs, 64 times 13.2 -> 10.3 us) takes Tb times
// and up to kCompPairs products, of one frequency after the other: thread k
// takes time k mod Tb and every R-th product from k / Tb (R = threads / Tb), so
// each step of the workgroup reads R runs of 8 Tb bytes (one contiguous piece
// of the [P][T] block where Tb = T).  The places of a product's two autos come
// from a table in LDS made once, the frequency's autos are in LDS too: above
// 128 inputs they bound Tb (8 at 2048 inputs: 32 times in 279 us, 1.9 TB/s).  The per-thread minima
// meet in LDS, those of several workgroups in an atomic minimum on the
// output, set to 1 before.  The minimum does not depend on the order of the
// terms (no term is -0, NaN terms are skipped).
//
// Bound by HBM reads.  A double-precision division per product and stepping
// the inputs along took 70 instructions per product and kept it from there:
// 201 us for 541 MB (256 frequencies, 128 inputs, 32 times), 541 us for 2.16
// GB; now 129 and 436 us (5.0 TB/s), and times that are no power of two or
// few frequencies no longer go to a slower kernel (2 frequencies, 512 inputs,
// 30 times: 20.8 ms -> 30 us).  So a product is first screened
// in float32 against the lowest term any thread has found for its time
// (`best`): with q = |V_ij|^2, ab = V_ii V_jj and c = ab (1 - best)(1 -
// 2^-18), all rounded to float32, a product with q <= c is left out where
// every factor of the comparison is good to a few parts in 2^24: ab a normal
// float (a subnormal one is off by up to a half), c at least 1e-30 (where
// underflow in q is far below the margin) and finite.  That puts the exact
// quotient below (1 - best)(1 - 2^-20), so the exact term, rounded, is not
// below best, and the minimum is the one of all exact terms.  Where any of it
// fails (products that lower the minimum, or without a usable ab) the exact
// path follows, which is soon rare.
constexpr int kCompThreads = 512;
constexpr int kCompTimes = 128;     // times of a workgroup (105 MB of 11 inputs, 512 times:
                                    // 31 us at 64, 27 at 128, 29 at 256, 35 at 512)
constexpr int kCompAhead = 8;       // visibilities a thread loads before it uses the first
constexpr int kCompPairs = 8192;    // products a workgroup has a table for (32 KiB)
constexpr int kCompAutos = 16384;   // autos of one frequency and Tb times (64 KiB)

// LDS: i Tb and j Tb of the workgroup's products fit 16 bits each and the
// autos their place; else (more inputs than kCompAutos) both are found again
// for each product.
template <bool LDS, int THREADS>
__global__ __launch_bounds__(THREADS) void k_noise_comp(const float2 *__restrict__ vis,
                                                        RoundParams rp, double *__restrict__ scale,
                                                        int Tb, int parts)
{
    __shared__ double part[THREADS];
    __shared__ double best[THREADS]; // per time; many threads write it, any term found will do
    extern __shared__ uint32_t dyn[];     // LDS: the products' table, then the autos
    const int k = threadIdx.x;
    const int R = THREADS / Tb, r = k / Tb, tl = k - r * Tb;
    const int64_t T = rp.T, t0 = (int64_t)blockIdx.z * Tb, t = t0 + tl;
    const int64_t per = (rp.P + parts - 1) / parts, first = per * blockIdx.y;
    const int count = (int)(rp.P - first < per ? (rp.P > first ? rp.P - first : 0) : per);
    uint32_t *pairs = dyn;
    float *la = reinterpret_cast<float *>(dyn + per);
    const bool mine = r < R && t < T;
    if constexpr (LDS) {
        for (int p = k; p < count; p += THREADS) {
            int32_t i, j;
            product_pair(rp, first + p, i, j);
            pairs[p] = (uint32_t)(i * Tb) | (uint32_t)(j * Tb) << 16;
        }
    }
    for (int64_t fr = blockIdx.x; fr < rp.F; fr += gridDim.x) {
        const float2 *vbase = vis + (fr * rp.P + first) * T;
        const float *abase = rp.autos + fr * rp.I * T;
        if constexpr (LDS) {
            for (int e = k; e < (int)rp.I * Tb; e += THREADS) {
                const int i = e / Tb;
                const int64_t ta = t0 + e - i * Tb;
                la[e] = ta < T ? abase[i * T + ta] : 0.0f;
            }
        }
        best[k] = 1.0;
        __syncthreads();
        double m = 1.0;
        // the autos of product p of the workgroup; false for an auto product
        const auto autos_of = [&](int p, float &ai, float &aj) {
            if constexpr (LDS) {
                const uint32_t x = pairs[p], a = x & 0xFFFFu, b = x >> 16;
                ai = la[a + tl];
                aj = la[b + tl];
                return a != b;
            } else {
                int32_t i, j;
                product_pair(rp, first + p, i, j);
                ai = abase[i * T + t];
                aj = abase[j * T + t];
                return i != j;
            }
        };
        const int64_t mine0 = r * T + t;
        const auto exact_term = [&](float2 v, float ai, float aj) {
            const double ab = (double)ai * (double)aj;
            const double term = 1.0 - ((double)v.x * (double)v.x + (double)v.y * (double)v.y) / ab;
            // a NaN term never wins
            if (ab > 0.0 && ab != __builtin_inf() && term < m) m = term;
        };
        if (mine) {
            int p = 0; // uniform; the thread's product is p + r
            for (; p + kCompAhead * R <= count; p += kCompAhead * R) {
                float2 v[kCompAhead];
#pragma unroll
                for (int u = 0; u < kCompAhead; ++u) v[u] = vbase[(int64_t)(p + u * R) * T + mine0];
                const double b = __hip_atomic_load(&best[tl], __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
                const float thr = (float)((1.0 - b) * (1.0 - 0x1p-18));
                float ai[kCompAhead], aj[kCompAhead];
                bool need[kCompAhead], any = false;
#pragma unroll
                for (int u = 0; u < kCompAhead; ++u) {
                    const bool cross = autos_of(p + u * R + r, ai[u], aj[u]);
                    const float q = v[u].x * v[u].x + v[u].y * v[u].y, ab = ai[u] * aj[u];
                    const float c = thr * ab;
                    need[u] = cross && !(q <= c && c >= 1e-30f && c < __builtin_inff() && ab >= 0x1p-126f);
                    any |= need[u];
                }
                if (any) {
#pragma unroll
                    for (int u = 0; u < kCompAhead; ++u)
                        if (need[u]) exact_term(v[u], ai[u], aj[u]);
                    if (m < b)
                        __hip_atomic_store(&best[tl], m, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            for (; p + r < count; p += R) {
                float ai, aj;
                if (autos_of(p + r, ai, aj)) exact_term(vbase[p * T + mine0], ai, aj);
            }
        }
        part[k] = m;
        __syncthreads();
        for (int n = R; n > 1;) { // rows r < n hold minima: fold the upper half
            const int h = (n + 1) / 2;
            if (r < n - h && part[k + h * Tb] < part[k]) part[k] = part[k + h * Tb];
            n = h;
            __syncthreads();
        }
        if (r == 0 && t < T) {
            if (parts == 1)
                scale[fr * T + t] = part[k];
            else if (part[k] < 1.0)
                atomicMin(&scale[fr * T + t], part[k]);
        }
        __syncthreads();
    }
}

// Small arrays: a thread takes one (frequency, time) and walks its products.
// A workgroup of the kernel above spends five barriers on each frequency,
// which 1 to 36 products do not fill: 1,000,000 frequencies of 2 inputs and 7
// times took 2770 us there, 42 here (280 MB: HBM and the cache before it).
__global__ __launch_bounds__(256) void k_noise_comp_small(const float2 *__restrict__ vis,
                                                          RoundParams rp,
                                                          double *__restrict__ scale, int64_t n)
{
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        int64_t fr, t;
        divmod(e, rp.T, fr, t);
        const float2 *v = vis + fr * rp.P * rp.T + t;
        const float *a = rp.autos + fr * rp.I * rp.T + t;
        const int I = (int)rp.I, P = (int)rp.P;
        double m = 1.0;
        int i = 0, j = 0;
#pragma unroll 4
        for (int p = 0; p < P; ++p) {
            if (rp.prod_map) {
                i = rp.prod_map[2 * p];
                j = rp.prod_map[2 * p + 1];
            }
            if (i != j) {
                const float2 x = v[p * rp.T];
                const double ab = (double)a[i * rp.T] * (double)a[j * rp.T];
                const double term = 1.0 - ((double)x.x * (double)x.x + (double)x.y * (double)x.y) / ab;
                // a NaN term never wins
                if (ab > 0.0 && ab != __builtin_inf() && term < m) m = term;
            }
            if (++j == I) j = ++i;
        }
        scale[e] = m;
    }
}

__global__ __launch_bounds__(256) void k_ones(double *__restrict__ out, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        out[i] = 1.0;
}

} // namespace

hipError_t launch_round(const float *vin, float *vout, const RoundParams &rp, hipStream_t s)
{
    const int64_t n_complex = rp.F * rp.P * rp.T;
    if (n_complex == 0) return hipSuccess;
    const int64_t waves = (n_complex + kWave * kComplexPerThread - 1) / (kWave * kComplexPerThread);
    const int64_t blocks = (waves * kWave + 255) / 256;
    const int aligned16 = (((uintptr_t)vin | (uintptr_t)vout) & 15) == 0;
    hipLaunchKernelGGL((k_round<float2>), dim3((unsigned)blocks), dim3(256), 0, s,
                       reinterpret_cast<const float2 *>(vin), reinterpret_cast<float2 *>(vout),
                       rp, n_complex, aligned16);
    return hipGetLastError();
}

hipError_t launch_round_i32(const int32_t *vin, int32_t *vout, const RoundParams &rp, hipStream_t s)
{
    const int64_t n_complex = rp.F * rp.P * rp.T;
    if (n_complex == 0) return hipSuccess;
    const int64_t waves = (n_complex + kWave * kComplexPerThread - 1) / (kWave * kComplexPerThread);
    const int64_t blocks = (waves * kWave + 255) / 256;
    const int aligned16 = (((uintptr_t)vin | (uintptr_t)vout) & 15) == 0;
    hipLaunchKernelGGL((k_round<int2>), dim3((unsigned)blocks), dim3(256), 0, s,
                       reinterpret_cast<const int2 *>(vin), reinterpret_cast<int2 *>(vout), rp,
                       n_complex, aligned16);
    return hipGetLastError();
}

hipError_t launch_noise_comp(const float *vis, const RoundParams &rp, double *scale, hipStream_t s)
{
    const int64_t n = rp.F * rp.T;
    if (n == 0) return hipSuccess;
    const float2 *v = reinterpret_cast<const float2 *>(vis);
    // A thread per sample up to 6 inputs, and up to 9 where the samples fill the
    // card (105 MB of 8 inputs, 1 time: 114 us there, 1077 below; 1 MB of 1 time:
    // 10 and 8).
    if (rp.P <= 21 || (rp.P <= 45 && n >= 131072)) {
        hipLaunchKernelGGL(k_noise_comp_small, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1 << 22)),
                           dim3(256), 0, s, v, rp, scale, n);
        return hipGetLastError();
    }
    const bool lds = rp.I <= kCompAutos;
    // (the times in equal tiles: 130 as 65 and 65)
    const int64_t fit = std::min<int64_t>(lds ? kCompAutos / rp.I : kCompTimes, kCompTimes);
    const int64_t tiles0 = (rp.T + fit - 1) / fit;
    const int Tb = (int)((rp.T + tiles0 - 1) / tiles0);
    const int64_t tiles = (rp.T + Tb - 1) / Tb;
    const int64_t most = lds ? kCompPairs : 1 << 28; // products of a workgroup
    // Enough parts for three workgroups per CU (as many as reside up to 40 KiB
    // of table and autos), if each keeps four steps, and for the table.
    const int64_t steps = rp.P / (kCompAhead * (kCompThreads / Tb));
    const int parts = (int)std::max<int64_t>(
        {(rp.P + most - 1) / most, 1,
         std::min<int64_t>(steps / 4, (3 * 256 + rp.F * tiles - 1) / (rp.F * tiles))});
    if (parts > 1) {
        hipLaunchKernelGGL(k_ones, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1024)), dim3(256),
                           0, s, scale, n);
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    // workgroups of the same products take further frequencies past eight per CU
    const int64_t gx = std::min<int64_t>(rp.F, std::max<int64_t>(1, 8 * 256 / (parts * tiles)));
    const dim3 grid((unsigned)gx, (unsigned)parts, (unsigned)tiles);
    const int64_t per = (rp.P + parts - 1) / parts;
    const size_t dyn = lds ? 4 * (size_t)(per + rp.I * Tb) : 0;
    if (!lds)
        hipLaunchKernelGGL((k_noise_comp<false, kCompThreads>), grid, dim3(kCompThreads), 0, s, v, rp,
                           scale, Tb, parts);
    else if (parts == 1 && rp.F * tiles <= 256) // a CU each: more threads, fewer steps
        hipLaunchKernelGGL((k_noise_comp<true, 2 * kCompThreads>), grid, dim3(2 * kCompThreads), dyn, s,
                           v, rp, scale, Tb, parts);
    else
        hipLaunchKernelGGL((k_noise_comp<true, kCompThreads>), grid, dim3(kCompThreads), dyn, s, v, rp,
                           scale, Tb, parts);
    return hipGetLastError();
}

} // namespace bsg
