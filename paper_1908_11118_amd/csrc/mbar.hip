// mbar.hip -- multistate reweighting of REGC samples (arXiv:1908.11118, Sec. II.B).
//
// Reduced potential of sample n in state s = (l, m):  u_s(n) = beta_l E_n - N_n ln z_lm
// (Eq. (8) with the paper's sign of mu N plus the 3N ln Lambda(T) term of Eq. (1)).
// Self-consistent equations (Eq. (9)) in log form, f_s = -ln c_s:
//     log D_n = logsumexp_k [ln Omega_k + f_k - u_k(n)],   f_s = -logsumexp_n [-u_s(n) - log D_n].
//
// On a T x mu product grid the state sum factorises exactly (the algebra is
// ours, not the paper's):
//     D_n = sum_l exp(-beta_l E_n) A_l(N_n),       A_l(N) = sum_m Omega_lm exp(f_lm + N ln z_lm),
//     exp(-f_lm) = sum_N z_lm^N P_l(N) / A_l(N),   P_l(N) = sum_{n: N_n = N} p_l(n),
// where p_l(n) = exp(-beta_l E_n) A_l(N_n) / D_n is the softmax over temperatures of
// x_l(n) = -beta_l E_n + log A_l(N_n).  One iteration therefore costs L exponentials
// per sample instead of 2 L M, and every partial sum lies in [0, count]: no overflow.
// Samples are sorted by N once (stable radix sort) and cut into chunks of one N
// each; each chunk writes its L partial sums and they are added in chunk order,
// so results are deterministic.
//
// Averages at a target (T', mu'): with y(n) = -beta' E_n - log D_n,
//     G(N) = logsumexp_{n: N_n = N} y(n),   P(N) proportional to exp(N ln z' + G(N)),
//     <N> = sum N P(N),  <E^k> = sum_N P(N) [sum_{N_n=N} E_n^k e^{y}] / [sum_{N_n=N} e^{y}],
//     f' = -logsumexp_N (N ln z' + G(N)),  phase = argmax_N P(N) (Eq. (10)/(11), smallest N on ties).
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <deque>
#include <mutex>
#include <type_traits>
#include <vector>

#include "host_util.h"
#include "philox_dev.h"
#include "regc_dev.h"

namespace regc {

constexpr int kChunk = 2048;
constexpr int kMbarThreads = 256;
constexpr int kMaxL = 64;

// Counts of the samples by state and by N and, per state, the sums of N and of E
// (fixed point, 2^-16: any order of the additions gives the same sum).  Every block
// keeps its own counters in LDS and writes them out; mbar_count_sum adds the blocks.
// With one set of counters in memory the additions queued at its few hundred lines
// (1.02e6 samples of 1024 states and 201 N: 1.25 ms, this 25 us).
// Counters per block: S counts | S sums of N | nN counts (32 bits) and S sums of E (64).
constexpr int kCountThreads = 256, kCountBlocks = 256;

__host__ __device__ inline size_t count_bytes(int S, int nN) { return (size_t)S * 16 + (size_t)((nN + 1) & ~1) * 4; }

__global__ void __launch_bounds__(kCountThreads) mbar_count(int64_t ns, const int32_t *n, const int32_t *st, const double *e,
                                                         int nN, int S, unsigned char *out, int *bad)
{
    extern __shared__ __align__(16) unsigned char cnt_lds[];
    unsigned long long *se = reinterpret_cast<unsigned long long *>(cnt_lds);
    uint32_t *cnt = reinterpret_cast<uint32_t *>(se + S), *sn = cnt + S, *seg = sn + S;
    const int words = (int)(count_bytes(S, nN) / 4);
    uint32_t *all = reinterpret_cast<uint32_t *>(cnt_lds);
    for (int k = threadIdx.x; k < words; k += blockDim.x) all[k] = 0u;
    __syncthreads();
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ns; i += (int64_t)gridDim.x * blockDim.x) {
        const int N = n[i], s = st[i];
        if (N < 0 || N >= nN || s < 0 || s >= S) {
            atomicOr(bad, 1);
            continue;
        }
        atomicAdd(cnt + s, 1u);
        atomicAdd(sn + s, (uint32_t)N);
        atomicAdd(se + s, (unsigned long long)__double2ll_rn(fmin(fmax(e[i], -1e9), 1e9) * 65536.0));
        atomicAdd(seg + N, 1u);
    }
    __syncthreads();
    uint32_t *dst = reinterpret_cast<uint32_t *>(out + (size_t)blockIdx.x * count_bytes(S, nN));
    for (int k = threadIdx.x; k < words; k += blockDim.x) dst[k] = all[k];
}

// totals: sums of E [S], counts [S], sums of N [S], counts by N [nN] (64 bits each)
__global__ void mbar_count_sum(int blocks, int S, int nN, const unsigned char *part, unsigned long long *total)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= 3 * S + nN) return;
    const size_t stride = count_bytes(S, nN);
    unsigned long long v = 0;
#pragma unroll 8
    for (int b = 0; b < blocks; ++b) {
        const unsigned char *p = part + b * stride;
        if (k < S) v += reinterpret_cast<const unsigned long long *>(p)[k];
        else v += reinterpret_cast<const uint32_t *>(p + (size_t)S * 8)[k - S];
    }
    total[k] = v;
}

// The same without room for the counters in LDS: one set in memory.
__global__ void mbar_count_global(int64_t ns, const int32_t *n, const int32_t *st, int nN, int S, unsigned long long *omega,
                                  unsigned long long *seg, int *bad)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ns; i += (int64_t)gridDim.x * blockDim.x) {
        const int N = n[i], s = st[i];
        if (N < 0 || N >= nN || s < 0 || s >= S) {
            atomicOr(bad, 1);
            continue;
        }
        atomicAdd(omega + s, 1ull);
        atomicAdd(seg + N, 1ull);
    }
}

__global__ void mbar_iota_gather(int64_t ns, const int32_t *n_in, uint32_t *keys, int32_t *idx)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ns; i += (int64_t)gridDim.x * blockDim.x) {
        keys[i] = (uint32_t)n_in[i];
        idx[i] = (int32_t)i;
    }
}

__global__ void mbar_gather_e(int64_t ns, const int32_t *perm, const double *e_in, double *e_out)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ns; i += (int64_t)gridDim.x * blockDim.x)
        e_out[i] = e_in[perm[i]];
}

// log A_l(N) for every l (block) and N (threads)
__global__ void mbar_loga(int M, int nN, const double *lnomega, const double *f, const double *lnz, double *logA)
{
    const int l = blockIdx.x;
    for (int N = threadIdx.x; N < nN; N += blockDim.x) {
        double mx = -INFINITY;
        for (int m = 0; m < M; ++m) {
            const int s = l * M + m;
            if (lnomega[s] == -INFINITY) continue;
            const double v = lnomega[s] + f[s] + (double)N * lnz[s];
            mx = v > mx ? v : mx;
        }
        double sum = 0.0;
        if (mx != -INFINITY)
            for (int m = 0; m < M; ++m) {
                const int s = l * M + m;
                if (lnomega[s] == -INFINITY) continue;
                sum += exp(lnomega[s] + f[s] + (double)N * lnz[s] - mx);
            }
        logA[(size_t)l * nN + N] = mx == -INFINITY ? -INFINITY : mx + log(sum);
    }
}

__device__ __forceinline__ double wsum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// One chunk (samples of a single N) per block: softmax over temperatures per
// sample, partial sums of p_l(n) per chunk; log D_n when requested.
// WEIGHTED: sample i counts wgt[i] times (bootstrap replicates; wgt in sorted order).
template <int LMAX, bool WEIGHTED>
__global__ void __launch_bounds__(kMbarThreads) mbar_chunk(int L, int nN, const double *beta_l, const double *logA,
                                                        const double *e, const int *chunk_n, const int *chunk_b,
                                                        const int *chunk_e, double *partial, double *logd_out,
                                                        const double *wgt)
{
    __shared__ double red[kMbarThreads / 64][LMAX];
    const int c = blockIdx.x;
    const int N = chunk_n[c];
    double la[LMAX], nb[LMAX], acc[LMAX];
#pragma unroll
    for (int l = 0; l < LMAX; ++l) {
        la[l] = l < L ? logA[(size_t)l * nN + N] : -INFINITY;
        nb[l] = l < L ? -beta_l[l] : 0.0;
        acc[l] = 0.0;
    }
    const int end = chunk_e[c];
    for (int i = chunk_b[c] + threadIdx.x; i < end; i += blockDim.x) {
        const double E = e[i];
        double x[LMAX];
        double mx = -INFINITY;
#pragma unroll
        for (int l = 0; l < LMAX; ++l) {
            x[l] = l < L ? nb[l] * E + la[l] : -INFINITY;
            mx = x[l] > mx ? x[l] : mx;
        }
        double sum = 0.0;
#pragma unroll
        for (int l = 0; l < LMAX; ++l) {
            x[l] = l < L ? exp(x[l] - mx) : 0.0;
            sum += x[l];
        }
        const double inv = WEIGHTED ? wgt[i] / sum : 1.0 / sum;
#pragma unroll
        for (int l = 0; l < LMAX; ++l) acc[l] += x[l] * inv;
        if (logd_out) logd_out[i] = mx + log(sum);
    }
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
#pragma unroll
    for (int l = 0; l < LMAX; ++l) {
        const double v = wsum(acc[l]);
        if (lane == 0) red[wave][l] = v;
    }
    __syncthreads();
    for (int l = threadIdx.x; l < L; l += blockDim.x) {
        double v = 0.0;
        for (int wv = 0; wv < kMbarThreads / 64; ++wv) v += red[wv][l];
        partial[(size_t)c * L + l] = v;
    }
}

// New free energies: one block per temperature l.
__global__ void mbar_fnew(int L, int M, int nN, const double *partial, const int *seg_c0, const int *seg_c1,
                          const double *logA, const double *lnz, double *fnew)
{
    extern __shared__ double logB[];
    const int l = blockIdx.x;
    for (int N = threadIdx.x; N < nN; N += blockDim.x) {
        double P = 0.0;
        for (int c = seg_c0[N]; c < seg_c1[N]; ++c) P += partial[(size_t)c * L + l];
        logB[N] = P > 0.0 ? log(P) - logA[(size_t)l * nN + N] : -INFINITY;
    }
    __syncthreads();
    for (int m = threadIdx.x; m < M; m += blockDim.x) {
        const double lz = lnz[l * M + m];
        double mx = -INFINITY;
        for (int N = 0; N < nN; ++N) {
            if (logB[N] == -INFINITY) continue;
            const double v = (double)N * lz + logB[N];
            mx = v > mx ? v : mx;
        }
        double sum = 0.0;
        for (int N = 0; N < nN; ++N) {
            if (logB[N] == -INFINITY) continue;
            sum += exp((double)N * lz + logB[N] - mx);
        }
        fnew[l * M + m] = -(mx + log(sum));
    }
}

// Gauge (f = 0 at state g) and max |delta f| over sampled states; f <- fnew.
__global__ void mbar_gauge(int S, int g, const double *lnomega, double *fnew, double *f, double *delta)
{
    __shared__ double red[16];
    const double f0 = fnew[g];
    double d = 0.0;
    for (int s = threadIdx.x; s < S; s += blockDim.x) {
        const double v = fnew[s] - f0;
        if (lnomega[s] != -INFINITY) {
            const double a = fabs(v - f[s]);
            d = (a > d || a != a) ? a : d;           // a NaN propagates: the host must see it
        }
        f[s] = v;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double t = __shfl_xor(d, o);
        d = (t > d || t != t) ? t : d;
    }
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = d;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = 0.0;
        for (int k = 0; k < (int)(blockDim.x / 64); ++k) m = (red[k] > m || red[k] != red[k]) ? red[k] : m;
        *delta = m;
    }
}

// Target temperatures: per chunk and target temperature the online (max, s0, s1, s2).
__global__ void __launch_bounds__(kMbarThreads) mbar_target_chunk(int nT, const double *tbeta, const double *e,
                                                               const double *logd, const int *chunk_b,
                                                               const int *chunk_e, double *tpart,
                                                               const double *wgt)
{
    __shared__ double red[kMbarThreads / 64][4];
    const int c = blockIdx.x;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    for (int t = 0; t < nT; ++t) {
        const double b = tbeta[t];
        double mx = -INFINITY, s0 = 0.0, s1 = 0.0, s2 = 0.0;
        for (int i = chunk_b[c] + threadIdx.x; i < chunk_e[c]; i += blockDim.x) {
            const double E = e[i];
            const double y = -b * E - logd[i];
            if (y > mx) {
                const double sc = exp(mx - y);
                s0 *= sc; s1 *= sc; s2 *= sc;
                mx = y;
            }
            const double w = wgt ? wgt[i] * exp(y - mx) : exp(y - mx);
            s0 += w; s1 += w * E; s2 += w * E * E;
        }
        // wave combine
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double om = __shfl_xor(mx, o), o0 = __shfl_xor(s0, o), o1 = __shfl_xor(s1, o),
                         o2 = __shfl_xor(s2, o);
            const double nm = om > mx ? om : mx;
            const double a = nm == -INFINITY ? 0.0 : exp(mx - nm), bb = nm == -INFINITY ? 0.0 : exp(om - nm);
            s0 = s0 * a + o0 * bb; s1 = s1 * a + o1 * bb; s2 = s2 * a + o2 * bb;
            mx = nm;
        }
        if (lane == 0) { red[wave][0] = mx; red[wave][1] = s0; red[wave][2] = s1; red[wave][3] = s2; }
        __syncthreads();
        if (threadIdx.x == 0) {
            double M = -INFINITY;
            for (int k = 0; k < kMbarThreads / 64; ++k) M = red[k][0] > M ? red[k][0] : M;
            double a0 = 0, a1 = 0, a2 = 0;
            if (M != -INFINITY)
                for (int k = 0; k < kMbarThreads / 64; ++k) {
                    if (red[k][0] == -INFINITY) continue;
                    const double sc = exp(red[k][0] - M);
                    a0 += red[k][1] * sc; a1 += red[k][2] * sc; a2 += red[k][3] * sc;
                }
            double *o = tpart + ((size_t)c * nT + t) * 4;
            o[0] = M; o[1] = a0; o[2] = a1; o[3] = a2;
        }
        __syncthreads();
    }
}

// Per target temperature (block): combine chunk partials by N, then every mu'.
__global__ void mbar_target_eval(int nT, int nMu, int nN, const double *tpart, const int *seg_c0, const int *seg_c1,
                                 const double *tlnz, double *f, double *mean_n, double *mean_e, double *mean_e2,
                                 double *p_n, int32_t *phase)
{
    extern __shared__ double sh[];
    double *G = sh, *E1 = sh + nN, *E2 = sh + 2 * nN;
    const int t = blockIdx.x;
    for (int N = threadIdx.x; N < nN; N += blockDim.x) {
        double M = -INFINITY;
        for (int c = seg_c0[N]; c < seg_c1[N]; ++c) {
            const double m = tpart[((size_t)c * nT + t) * 4];
            M = m > M ? m : M;
        }
        double a0 = 0, a1 = 0, a2 = 0;
        if (M != -INFINITY)
            for (int c = seg_c0[N]; c < seg_c1[N]; ++c) {
                const double *o = tpart + ((size_t)c * nT + t) * 4;
                if (o[0] == -INFINITY) continue;
                const double sc = exp(o[0] - M);
                a0 += o[1] * sc; a1 += o[2] * sc; a2 += o[3] * sc;
            }
        G[N] = (M == -INFINITY || a0 <= 0.0) ? -INFINITY : M + log(a0);
        E1[N] = a0 > 0.0 ? a1 / a0 : 0.0;
        E2[N] = a0 > 0.0 ? a2 / a0 : 0.0;
    }
    __syncthreads();
    for (int m = threadIdx.x; m < nMu; m += blockDim.x) {
        const int k = t * nMu + m;
        const double lz = tlnz[k];
        double mx = -INFINITY;
        int best = 0;
        for (int N = 0; N < nN; ++N) {
            if (G[N] == -INFINITY) continue;
            const double v = (double)N * lz + G[N];
            if (v > mx) { mx = v; best = N; }
        }
        double sum = 0.0;
        for (int N = 0; N < nN; ++N)
            if (G[N] != -INFINITY) sum += exp((double)N * lz + G[N] - mx);
        const double lse = mx + log(sum);
        double sn = 0, se = 0, se2 = 0;
        for (int N = 0; N < nN; ++N) {
            const double p = G[N] == -INFINITY ? 0.0 : exp((double)N * lz + G[N] - lse);
            sn += p * (double)N; se += p * E1[N]; se2 += p * E2[N];
            if (p_n) p_n[(size_t)k * nN + N] = p;
        }
        if (f) f[k] = -lse;
        mean_n[k] = sn;
        if (mean_e) mean_e[k] = se;
        if (mean_e2) mean_e2[k] = se2;
        if (phase) phase[k] = best;
    }
}

// Observables: gather into sorted order
__global__ void mbar_gather_obs(int64_t ns, int n_obs, const int32_t *perm, const uint32_t *in, uint32_t *out)
{
    const int64_t total = ns * n_obs;
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < total; q += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = q / n_obs;
        const int k = (int)(q - i * n_obs);
        out[q] = in[(int64_t)perm[i] * n_obs + k];
    }
}

// Per chunk c (one N) and target temperature t (grid y): the scale mx = max of
// y_i = -beta_t E_i - logD_i, s0 = sum exp(y_i - mx) and s_k = sum exp(y_i - mx) obs_ik,
// every sum in sample order (deterministic).  out[(c nT + t)(n_obs + 2) + {0, 1, 2 + k}].
__global__ void __launch_bounds__(kMbarThreads) mbar_obs_chunk(int nT, int n_obs, const double *tbeta, const double *e,
                                                            const double *logd, const int *chunk_b,
                                                            const int *chunk_e, const uint32_t *obs, double *out)
{
    __shared__ double w[kChunk];
    __shared__ double red[kMbarThreads / 64];
    const int c = blockIdx.x, t = blockIdx.y;
    const int b = chunk_b[c], cnt = chunk_e[c] - b;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const double bt = tbeta[t];
    double mx = -INFINITY;
    for (int i = threadIdx.x; i < cnt; i += blockDim.x) {
        const double y = -bt * e[b + i] - logd[b + i];
        w[i] = y;
        mx = y > mx ? y : mx;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double v = __shfl_xor(mx, o);
        mx = v > mx ? v : mx;
    }
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = red[0];
    for (int k = 1; k < kMbarThreads / 64; ++k) mx = red[k] > mx ? red[k] : mx;
    __syncthreads();
    for (int i = threadIdx.x; i < cnt; i += blockDim.x) w[i] = exp(w[i] - mx);
    __syncthreads();
    double *o = out + ((size_t)c * nT + t) * (n_obs + 2);
    if (threadIdx.x == 0) {
        double s0 = 0.0;
        for (int i = 0; i < cnt; ++i) s0 += w[i];
        o[0] = mx;
        o[1] = s0;
    }
    for (int k = threadIdx.x; k < n_obs; k += blockDim.x) {
        double acc = 0.0;
        for (int i = 0; i < cnt; ++i) acc += w[i] * (double)obs[(size_t)(b + i) * n_obs + k];
        o[2 + k] = acc;
    }
}

// Per target temperature t (block): the chunks of each N combined in order into the
// conditional average cond[t][N][k] and G(N) = ln sum_{N_n = N} exp(-beta_t E - logD);
// then for every target mu: p(N) = exp(N lnz + G(N) - lse) and mean = sum_N p(N) cond.
__global__ void mbar_obs_eval(int nT, int nMu, int nN, int n_obs, const double *part, const int *seg_c0,
                              const int *seg_c1, const double *tlnz, double *cond, double *mean)
{
    extern __shared__ double sh[];    // G [nN] | p(N) of one mu [nN]
    double *G = sh, *P = sh + nN;
    const int t = blockIdx.x;
    const size_t stride = (size_t)n_obs + 2;
    double *ct = cond + (size_t)t * nN * n_obs;
    // the average conditional on N: chunk partials of one N combined in chunk order
    for (int N = 0; N < nN; ++N) {
        double M = -INFINITY;
        for (int c = seg_c0[N]; c < seg_c1[N]; ++c) {
            const double m = part[((size_t)c * nT + t) * stride];
            M = m > M ? m : M;
        }
        double s0 = 0.0;
        if (M != -INFINITY)
            for (int c = seg_c0[N]; c < seg_c1[N]; ++c) {
                const double *o = part + ((size_t)c * nT + t) * stride;
                if (o[0] != -INFINITY) s0 += o[1] * exp(o[0] - M);
            }
        if (threadIdx.x == 0) G[N] = (M == -INFINITY || s0 <= 0.0) ? -INFINITY : M + log(s0);
        for (int k = threadIdx.x; k < n_obs; k += blockDim.x) {
            double a = 0.0;
            if (M != -INFINITY)
                for (int c = seg_c0[N]; c < seg_c1[N]; ++c) {
                    const double *o = part + ((size_t)c * nT + t) * stride;
                    if (o[0] != -INFINITY) a += o[2 + k] * exp(o[0] - M);
                }
            ct[(size_t)N * n_obs + k] = s0 > 0.0 ? a / s0 : 0.0;
        }
    }
    __syncthreads();
    if (!mean) return;
    // mean at every mu: sum over N of p(N) times the conditional average
    for (int m = 0; m < nMu; ++m) {
        const double lz = tlnz[t * nMu + m];
        if (threadIdx.x == 0) {
            double mx = -INFINITY;
            for (int N = 0; N < nN; ++N)
                if (G[N] != -INFINITY) mx = fmax(mx, (double)N * lz + G[N]);
            double sum = 0.0;
            for (int N = 0; N < nN; ++N)
                if (G[N] != -INFINITY) sum += exp((double)N * lz + G[N] - mx);
            const double lse = mx + log(sum);
            for (int N = 0; N < nN; ++N) P[N] = G[N] == -INFINITY ? 0.0 : exp((double)N * lz + G[N] - lse);
        }
        __syncthreads();
        for (int k = threadIdx.x; k < n_obs; k += blockDim.x) {
            double acc = 0.0;
            for (int N = 0; N < nN; ++N)
                if (P[N] != 0.0) acc += P[N] * ct[(size_t)N * n_obs + k];
            mean[((size_t)t * nMu + m) * n_obs + k] = acc;
        }
        __syncthreads();
    }
}

// ---- errors of the estimates ----
// Batch means: a sample's rank among its state's samples, in the order given, decides its
// batch: batch b of a state with c samples holds ranks [b c / B, (b + 1) c / B).  Sums of N are integers
// (exact in any order).
//
// Ranks come without a sort: blocks of consecutive samples count their states in LDS
// (bm_count), a scan over the blocks gives each block's first rank per state (bm_scan), and a
// second pass ranks 64 samples at a time by matching their states' bits (bm_sum) and adds N:
// in LDS while a state stays in the batch that it starts the block in, else in memory.  What
// bounds it is the atomic sums that leave the blocks, so blocks are few and large.  The radix sort that
// this replaces took 26 launches and 12 allocations (1.02e6 samples of 1024 states: 453 us,
// now 74).  It stays for more states than LDS holds counters of.
constexpr int kBmBlocks = 128, kBmThreads = 512;

// LDS of bm_sum with W waves: per state a sum (64 bits), its batch, the count, a counter per wave
__host__ __device__ inline size_t bm_bytes(int S, int W) { return (size_t)S * (16 + 4 * W); }

struct BmArgs {
    int64_t ns;
    const int32_t *st, *n;
    int S, B, blocks;
    uint32_t *hist;                // [blocks][S]: counts, then first ranks
    uint32_t *count;               // [S]
    unsigned long long *sum;       // [S][B]
    int *bad;                      // [blocks]
    double *mean, *se;             // [S]
    int *any_bad;
    __device__ int64_t begin(int b) const { return ns * b / blocks; }
};

// a state out of range or a negative N
__device__ __forceinline__ bool bm_bad(const BmArgs &p, int s, int n) { return (s < 0) | (s >= p.S) | (n < 0); }

// Samples [i0, i1) by `lanes` threads, eight of each with all their loads first: f(state, N)
// by every thread, state -1 without a sample and -2 for a bad one.
template <typename F>
__device__ __forceinline__ void bm_each(const BmArgs &p, int64_t i0, int64_t i1, int lanes, F f)
{
    const int lane = threadIdx.x % lanes;
    for (; i0 < i1; i0 += 8 * lanes) {
        int s[8], n[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t i = i0 + lanes * q + lane, in = i < i1 ? i : i1 - 1;
            s[q] = p.st[in];
            n[q] = p.n[in];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (i0 + lanes * q < i1) {
                const int k = bm_bad(p, s[q], n[q]) ? -2 : s[q];
                f(i0 + lanes * q + lane < i1 ? k : -1, n[q]);
            }
    }
}

// Samples sorted by state give a wave one state: its lanes' additions would take turns at one
// address (4e6 samples of 64 states, sorted: 570 us by the sort, 710 by counting; now 150).  A
// wave whose share begins with 64 samples of one state looks for that as it goes; the others
// don't, for the test costs samples in any order a tenth.  f(std::true_type or std::false_type).
template <typename F>
__device__ __forceinline__ void bm_runs(const BmArgs &p, int64_t i0, int64_t i1, F f)
{
    const int64_t i = i0 + threadIdx.x % 64;
    const int s = i < i1 ? p.st[i] : -1;
    if (__ballot(s != __builtin_amdgcn_readfirstlane(s)) == 0) f(std::true_type{});
    else f(std::false_type{});
}

// Adds one to c[s] (LDS) for each lane with a state s >= 0.
template <bool RUNS>
__device__ __forceinline__ void bm_add(uint32_t *c, int s)
{
    const int one = __builtin_amdgcn_readfirstlane(s);
    if (RUNS && one >= 0 && __ballot(s != one) == 0) {
        if (threadIdx.x % 64 == 0) atomicAdd(c + s, 64u);
    } else if (s >= 0) {
        atomicAdd(c + s, 1u);
    }
}

__global__ void __launch_bounds__(kBmThreads) bm_count(BmArgs p)
{
    extern __shared__ __align__(16) unsigned char bm_lds[];
    uint32_t *c = reinterpret_cast<uint32_t *>(bm_lds);
    const int b = blockIdx.x;
    for (int s = threadIdx.x; s < p.S; s += kBmThreads) c[s] = 0u;
    for (int64_t k = b * (int64_t)kBmThreads + threadIdx.x; k < (int64_t)p.S * p.B; k += (int64_t)p.blocks * kBmThreads)
        p.sum[k] = 0ull;
    __syncthreads();
    bool bad = false;
    bm_runs(p, p.begin(b) + threadIdx.x / 64 * 64, p.begin(b + 1), [&](auto runs) {
        bm_each(p, p.begin(b), p.begin(b + 1), kBmThreads, [&](int s, int) {
            bm_add<decltype(runs)::value>(c, s);
            bad |= s == -2;
        });
    });
    const bool any = __syncthreads_or(bad);
    if (threadIdx.x == 0) p.bad[b] = any;
    for (int s = threadIdx.x; s < p.S; s += kBmThreads) p.hist[(size_t)b * p.S + s] = c[s];
}

// 64 states per block, the blocks' counts in 16 groups of consecutive ones
__global__ void __launch_bounds__(1024) bm_scan(BmArgs p)
{
    constexpr int kEach = kBmBlocks / 16;
    __shared__ uint32_t group[16][64];
    const int c = threadIdx.x % 64, g = threadIdx.x / 64, s = blockIdx.x * 64 + c;
    uint32_t v[kEach], mine = 0;
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
        const int b = g * kEach + q;
        v[q] = s < p.S && b < p.blocks ? p.hist[(size_t)b * p.S + s] : 0u;
        mine += v[q];
    }
    group[g][c] = mine;
    __syncthreads();
    uint32_t at = 0;
    for (int q = 0; q < g; ++q) at += group[q][c];
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
        const int b = g * kEach + q;
        if (s < p.S && b < p.blocks) p.hist[(size_t)b * p.S + s] = at;
        at += v[q];
    }
    if (g == 15 && s < p.S) p.count[s] = at;
    if (blockIdx.x == 0) {
        const bool any = __syncthreads_or(threadIdx.x < p.blocks && p.bad[threadIdx.x]);
        if (threadIdx.x == 0) *p.any_bad = any;
    }
}

// floor(((rank + 1) B - 1) / c): the batch whose range holds the rank
__device__ __forceinline__ uint32_t bm_batch(uint32_t rank, int B, uint32_t c)
{
    const uint64_t x = ((uint64_t)rank + 1) * (uint64_t)B - 1;
    if (x >> 52) return (uint32_t)(x / c);
    const int64_t f = (int64_t)((double)x / (double)c);    // off by one at most
    const int64_t rest = (int64_t)x - f * (int64_t)c;
    return (uint32_t)(rest < 0 ? f - 1 : rest >= (int64_t)c ? f + 1 : f);
}

template <int W>
__global__ void __launch_bounds__(64 * W) bm_sum(BmArgs p)
{
    extern __shared__ __align__(16) unsigned char bm_lds[];
    unsigned long long *acc = reinterpret_cast<unsigned long long *>(bm_lds);
    uint32_t *first = reinterpret_cast<uint32_t *>(acc + p.S), *count = first + p.S, *all = count + p.S;
    const int b = blockIdx.x, wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    uint32_t *mine = all + (size_t)wave * p.S;
    for (int s = threadIdx.x; s < p.S * W; s += 64 * W) all[s] = 0u;
    __syncthreads();
    // the waves' consecutive shares of the block's samples
    const int64_t lo = p.begin(b), cnt = p.begin(b + 1) - lo;
    const int64_t w0 = lo + cnt * wave / W, w1 = lo + cnt * (wave + 1) / W;
    bm_runs(p, w0, w1, [&](auto runs) {
        bm_each(p, w0, w1, 64, [&](int s, int) { bm_add<decltype(runs)::value>(mine, s); });
    });
    __syncthreads();
#pragma unroll 4
    for (int s = threadIdx.x; s < p.S; s += 64 * W) {
        uint32_t at = p.hist[(size_t)b * p.S + s];
        const uint32_t total = p.count[s];
        acc[s] = 0ull;
        count[s] = total;
        first[s] = total ? bm_batch(at < total ? at : total - 1, p.B, total) : 0u;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t here = all[(size_t)w * p.S + s];
            all[(size_t)w * p.S + s] = at;
            at += here;
        }
    }
    __syncthreads();
    int bits = 0;
    while ((1 << bits) < p.S) ++bits;
    volatile uint32_t *c = mine;
    bm_runs(p, w0, w1, [&](auto runs) {
        bm_each(p, w0, w1, 64, [&](int s, int n) {
            const int one = __builtin_amdgcn_readfirstlane(s);
            if (decltype(runs)::value && one >= 0 && __ballot(s != one) == 0) {
                // one state: ranks in order, and where the batch is one too, one sum
                const uint32_t rank0 = c[s], cnt = count[s];
                const uint32_t b0 = bm_batch(rank0, p.B, cnt), b1 = bm_batch(rank0 + 63u, p.B, cnt);
                __builtin_amdgcn_wave_barrier();
                if (lane == 0) c[s] = rank0 + 64u;
                if (b0 == b1) {
                    unsigned long long sum = (unsigned long long)n;
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
                    if (lane == 0) atomicAdd(b0 == first[s] ? acc + s : p.sum + (size_t)s * p.B + b0, sum);
                } else {
                    atomicAdd(p.sum + (size_t)s * p.B + bm_batch(rank0 + lane, p.B, cnt), (unsigned long long)n);
                }
                return;
            }
            uint64_t same = __ballot(s >= 0);
            for (int q = 0; q < bits; ++q) {
                const uint64_t set = __ballot((s >> q) & 1);
                same &= (s >> q) & 1 ? set : ~set;
            }
            if (s >= 0) {
                const uint32_t before = (uint32_t)__popcll(same & ((1ull << lane) - 1));
                const uint32_t rank = c[s] + before;
                __builtin_amdgcn_wave_barrier();
                if (before == 0) c[s] = rank + (uint32_t)__popcll(same);
                const uint32_t batch = bm_batch(rank, p.B, count[s]);
                if (batch == first[s]) atomicAdd(acc + s, (unsigned long long)n);
                else atomicAdd(p.sum + (size_t)s * p.B + batch, (unsigned long long)n);
            }
        });
    });
    __syncthreads();
    for (int s = threadIdx.x; s < p.S; s += 64 * W)
        if (acc[s]) atomicAdd(p.sum + (size_t)s * p.B + first[s], acc[s]);
}

// floor(b c / B), where batch b of a state with c samples starts
__device__ __forceinline__ int64_t bm_first(int b, int64_t c, int B)
{
    const int64_t x = b * c;
    if (x >> 52) return x / B;
    int64_t f = (int64_t)((double)x / (double)B);          // off by one at most
    const int64_t rest = x - f * B;
    return rest < 0 ? f - 1 : rest >= B ? f + 1 : f;
}

// Mean and SE of each state (a wave) from its batch sums (NaN below B samples); batch b's mean
// is its sum / its count, SE = sqrt(sum (m_b - mean(m))^2 / ((B - 1) B)), batches in order.
// sum(b): the sum of batch b, by lane b % 64.
template <typename F>
__device__ __forceinline__ void bm_estimate(int B, int64_t cnt, F sum, double *mean, double *se)
{
    const int lane = threadIdx.x % 64;
    if (cnt < B) {
        if (lane == 0) *mean = *se = NAN;
        return;
    }
    auto from = [](double v, int l) {
        const long long bits = __double_as_longlong(v);
        return __longlong_as_double((long long)(uint32_t)__builtin_amdgcn_readlane((int)bits, l) |
                                    (long long)__builtin_amdgcn_readlane((int)(bits >> 32), l) << 32);
    };
    double tot = 0.0, mb = 0.0, own = 0.0;
    for (int b0 = 0; b0 < B; b0 += 64) {
        const int b = b0 + lane < B ? b0 + lane : B - 1;
        const int64_t lo = bm_first(b, cnt, B), hi = bm_first(b + 1, cnt, B);
        const double v = (double)sum(b);
        own = v / (double)(hi - lo);
        for (int l = 0; l < 64 && b0 + l < B; ++l) {
            tot += from(v, l);
            mb += from(own, l);
        }
    }
    mb /= B;
    double v = 0.0;
    for (int b0 = 0; b0 < B; b0 += 64) {
        if (B > 64) {
            const int b = b0 + lane < B ? b0 + lane : B - 1;
            const int64_t lo = bm_first(b, cnt, B), hi = bm_first(b + 1, cnt, B);
            own = (double)sum(b) / (double)(hi - lo);
        }
        const double d = own - mb;
        for (int l = 0; l < 64 && b0 + l < B; ++l) {
            const double x = from(d, l);
            v += x * x;
        }
    }
    if (lane == 0) {
        *mean = tot / (double)cnt;
        *se = sqrt(v / (double)(B - 1) / (double)B);
    }
}

__global__ void __launch_bounds__(256) bm_finish(BmArgs p)
{
    const int s = blockIdx.x * 4 + (int)threadIdx.x / 64;
    if (s < p.S)
        bm_estimate(p.B, p.count[s], [&](int b) { return p.sum[(size_t)s * p.B + b]; }, p.mean + s, p.se + s);
}

// The same from samples sorted by state.
__global__ void bm_check(int64_t ns, const int32_t *st, const int32_t *n, int S, int *bad)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ns; i += (int64_t)gridDim.x * blockDim.x) {
        const int k = st[i];
        if (k < 0 || k >= S || n[i] < 0) atomicOr(bad, 1);
    }
}

// Start and length of every state's run in the keys sorted by state (lower bounds).
__global__ void bm_bounds(int64_t ns, int S, const uint32_t *sorted_state, int64_t *state_start, int64_t *state_count)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= S) return;
    auto lower = [&](uint32_t key) {
        int64_t lo = 0, hi = ns;
        while (lo < hi) {
            const int64_t mid = lo + (hi - lo) / 2;
            if (sorted_state[mid] < key) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    };
    const int64_t a = lower((uint32_t)s), b = lower((uint32_t)s + 1u);
    state_start[s] = a;
    state_count[s] = b - a;
}

// One workgroup per (state, batch): the batch is a contiguous range of the sorted
// order, its sum of N a block reduction of integers (exact in any order).
__global__ void bm_segments(int B, const int32_t *sorted_idx, const int32_t *n_orig, const int64_t *state_start,
                            const int64_t *state_count, unsigned long long *bsum)
{
    __shared__ unsigned long long part[4];
    const int bin = blockIdx.x, s = bin / B, b = bin % B;
    const int64_t cnt = state_count[s];
    const int64_t lo = state_start[s] + (b * cnt) / B, hi = state_start[s] + ((b + 1) * cnt) / B;
    unsigned long long acc = 0;
    for (int64_t p = lo + threadIdx.x; p < hi; p += blockDim.x) acc += (unsigned long long)n_orig[sorted_idx[p]];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (threadIdx.x % 64 == 0) part[threadIdx.x / 64] = acc;
    __syncthreads();
    if (threadIdx.x == 0) bsum[bin] = part[0] + part[1] + part[2] + part[3];
}

__global__ void __launch_bounds__(256) bm_finish_sorted(int S, int B, const unsigned long long *sum, const int64_t *count,
                                                     double *mean, double *se)
{
    const int s = blockIdx.x * 4 + (int)threadIdx.x / 64;
    if (s < S) bm_estimate(B, count[s], [&](int b) { return sum[(size_t)s * B + b]; }, mean + s, se + s);
}

// Moving-block bootstrap, replicate b: block j (of ceil(R / block)) starts at record
// floor(w (R - block + 1) / 2^32), w = word 0 of Philox block (j, b, 0xFFFFFFFE, 7);
// mult[r] counts the occurrences of record r in the concatenation cut to R records.
__global__ void boot_mult(int64_t R, int64_t block, int b, uint32_t k0, uint32_t k1, int32_t *mult)
{
    const int64_t nb = (R + block - 1) / block;
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < nb; j += (int64_t)gridDim.x * blockDim.x) {
        const uint4 w = philox4x32_10(make_uint4((uint32_t)j, (uint32_t)b, 0xFFFFFFFEu, 7u), k0, k1);
        const int64_t start = (int64_t)(((uint64_t)w.x * (uint64_t)(R - block + 1)) >> 32);
        for (int64_t k = 0; k < block && j * block + k < R; ++k) atomicAdd(mult + start + k, 1);
    }
}

__global__ void fill_i32(int64_t count, int32_t v, int32_t *x)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        x[i] = v;
}

__global__ void fill_u64(int64_t count, unsigned long long *x)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        x[i] = 0ull;
}

// Sample weights of a replicate in sorted order and the weighted count of each state.
__global__ void boot_weights(int64_t ns, int64_t record_size, const int32_t *perm, const int32_t *state_orig,
                             const int32_t *mult, double *wgt, unsigned long long *omega)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ns; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t o = perm[i];
        const int32_t m = mult[o / record_size];
        wgt[i] = (double)m;
        if (m) atomicAdd(omega + state_orig[o], (unsigned long long)m);
    }
}

// Heat capacity C = beta^2 (<E^2> - <E>^2) and coverage <N> / n_sites per target
// (targets t = l n_mu + m, beta of row l).
__global__ void heat_cov(int nT, int nMu, const double *tbeta, const double *mean_n, const double *mean_e,
                         const double *mean_e2, double n_sites, double *heat, double *cov)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nT * nMu) return;
    const double b = tbeta[k / nMu];
    heat[k] = b * b * (mean_e2[k] - mean_e[k] * mean_e[k]);
    if (cov) cov[k] = mean_n[k] / n_sites;
}

// Standard deviation over B replicates of every target ([B][K] in, (B - 1) divisor).
__global__ void rep_sd(int B, int K, const double *rep, double *sd)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    double m = 0.0;
    for (int b = 0; b < B; ++b) m += rep[(size_t)b * K + k];
    m /= B;
    double v = 0.0;
    for (int b = 0; b < B; ++b) {
        const double d = rep[(size_t)b * K + k] - m;
        v += d * d;
    }
    sd[k] = sqrt(v / (double)(B - 1));
}

// ---- the iteration on bounded exponents ----
// With c = the middle of the inverse temperatures and E0(N) the middle of the energies
// sampled at N, every sample's softmax is that of
//     -(beta_l - c)(E - E0) + [log A_l(N) - beta_l E0 - shift(N)],
// the bracket at most 0 by the choice of shift(N).  When no |beta_l - c| |E - E0|
// exceeds kMaxExponent (checked once per set of samples), the exponentials
// X_l = exp(-(beta_l - c)(E - E0)) and their sum with the weights a_l = exp(bracket) stay
// in range without a maximum per sample, and
//     sum_{n at N} e^{-beta_l E_n} / D_n = e^{-beta_l E0 - shift} Q_l(N),  Q_l(N) = sum_n X_l / sum_k a_k X_k,
// is what the new free energies need.  The solve goes on to kMaxSolveExponent: there a
// Q_l may overflow, and a solve that does not converge is left to the general iteration.
// What weights samples by more than that (targets, observables, replicates) stays below kMaxExponent.
// Samples outside take mbar_chunk.
constexpr double kMaxExponent = 300.0, kMaxSolveExponent = 350.0;

// exp(x) for |x| <= 708: x = k ln 2 + r (Cody and Waite's reduction, the product fused),
// the Taylor series of exp(r) to r^13 / 13! (|r| <= 0.35: below 5e-18 relative), 2^k by
// the exponent.  Within one unit in the last place, like the library's, without its
// checks for overflow.
__device__ __forceinline__ double exp_bounded(double x)
{
    const double k = rint(x * 1.4426950408889634);
    const double r = fma(k, -2.3190468138462996e-17, fma(k, -0.6931471805599453, x));
    double p = 1.0 / 6227020800.0;
    p = fma(p, r, 1.0 / 479001600.0);
    p = fma(p, r, 1.0 / 39916800.0);
    p = fma(p, r, 1.0 / 3628800.0);
    p = fma(p, r, 1.0 / 362880.0);
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return __builtin_amdgcn_ldexp(p, (int)k);
}

// 1 / x of a normal positive x: the hardware's estimate and two Newton steps (within one
// unit in the last place).
__device__ __forceinline__ double recip(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_move(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xF, false);
    return __hiloint2double(hi, lo);
}

// sum over each quad of lanes, in every lane of the quad
__device__ __forceinline__ double quad_total(double v)
{
    v += dpp_move<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
    v += dpp_move<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
    return v;
}

// wave total (fixed order) as a wave-uniform value
__device__ __forceinline__ double wave_total(double v)
{
    v = quad_total(v);
    v += dpp_move<0x141, 0xF>(v);   // row_half_mirror
    v += dpp_move<0x140, 0xF>(v);   // row_mirror
    v += dpp_move<0x142, 0xA>(v);   // row_bcast:15 into rows 1, 3
    v += dpp_move<0x143, 0xC>(v);   // row_bcast:31 into rows 2, 3
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}

// Middle and half width of the energies sampled at each N (block).
constexpr int kRangeThreads = 1024;

__global__ void __launch_bounds__(kRangeThreads) mbar_range(const double *e, const int *chunk_b, const int *chunk_e,
                                                        const int *seg_c0, const int *seg_c1, double *mid, double *half)
{
    __shared__ double lo_s[kRangeThreads / 64], hi_s[kRangeThreads / 64];
    const int N = blockIdx.x, c0 = seg_c0[N], c1 = seg_c1[N];
    double lo = INFINITY, hi = -INFINITY, bad = 0.0;
    if (c1 > c0)
#pragma unroll 4
        for (int i = chunk_b[c0] + threadIdx.x; i < chunk_e[c1 - 1]; i += blockDim.x) {
            const double E = e[i];
            bad += E - E;             // NaN when an energy is not finite
            lo = fmin(lo, E);
            hi = fmax(hi, E);
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o));
        hi = fmax(hi, __shfl_xor(hi, o));
        bad += __shfl_xor(bad, o);
    }
    if (threadIdx.x % 64 == 0) {
        lo_s[threadIdx.x / 64] = lo + bad;
        hi_s[threadIdx.x / 64] = hi + bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        bool nan = false;
        for (int k = 0; k < kRangeThreads / 64; ++k) {
            nan |= !(lo_s[k] == lo_s[k]) || !(hi_s[k] == hi_s[k]);
            lo = fmin(lo, lo_s[k]);
            hi = fmax(hi, hi_s[k]);
        }
        mid[N] = c1 > c0 ? 0.5 * lo + 0.5 * hi : 0.0;
        half[N] = nan ? NAN : (c1 > c0 ? 0.5 * hi - 0.5 * lo : 0.0);
    }
}

// What the kernels of an iteration share; problem b of a batch has its own weights,
// iterate and state.
struct SolveState {
    int done, conv, it, plain_left;  // conv: 1 converged, 2 below tol_switch
    int hist, head;                  // differences' history: entries, slot of the oldest
    int gauge, memory;               // first sampled state; at most this many differences
    int polish;                      // iterations since the residual first came below tol
    int lost;                        // a map value was not finite
    double delta, d_prev;
    double kept;                     // the latest residual below tol
};

constexpr int kMaxMemory = 8;        // differences the device's least squares holds
constexpr int kPolish = 12;          // iterations past the tolerance at most (preconditioned: 2)
// A residual that is rounding.  It is absolute: where f is in the hundreds an iteration cannot reach
// it and takes all the kPolish ones, which is what brought a solution with |(I - J)^-1| of 1e4
// from 1e-8 of the 64-bit one to 2e-10 (a floor that grew with |f| stopped short of that).
constexpr double kFloor = 2e-14;
constexpr int kMaxStepStates = 4096; // states it holds (16 per thread of 256)

struct SolveArgs {
    int L, M, S, nN, nchunks, sub, rows;       // rows = nchunks * sub partial sums per temperature
    const double *beta_l, *lnz;
    double beta_c;
    const double *e, *mid;
    const int *chunk_n, *chunk_b, *chunk_e, *seg_c0, *seg_c1;
    const double *lnomega;                     // [B][S]
    double *f, *fnew, *good;                   // [B][S]
    double *kept;                              // [B][S] the map value with that residual (polish > 0)
    double *hist_r, *hist_g;                   // [B][kMaxMemory + 1][S]
    double *shift;                             // [B][nN]
    double *partial;                           // [B][L][rows]
    SolveState *st;                            // [B]
    int polish;                                // iterations past the tolerance at most
    int method, max_iter;
    double tol, tol_switch;                    // tol_switch > 0: stop below it too (conv = 2)
    const double *y;                           // [B][S] preconditioned residuals, or null
    double *hinv;                              // 1 / sum_k a_k X_k of every sample (with log D)
    unsigned int *arrived;                     // [0] blocks of a step launch done with it, [1] step launches done
    unsigned long long *host;                  // host memory: step launches done | problems done << 32
};

// log A_l(N) - beta_l E0(N) of every temperature into la [L] (LDS), block-wide, 256
// threads: G threads per temperature take its chemical potentials.
__device__ __forceinline__ void weights_log(const SolveArgs &p, const double *lnomega, const double *f, int N, double *la)
{
    const int G = p.L <= 8 ? 32 : (p.L <= 16 ? 16 : (p.L <= 32 ? 8 : 4));
    const int l = threadIdx.x / G, g = threadIdx.x % G;
    double mx = -INFINITY, sum = 0.0;
    if (l < p.L)
        for (int m = g; m < p.M; m += G) {
            const int s = l * p.M + m;
            const double v = lnomega[s] + f[s] + (double)N * p.lnz[s];
            if (lnomega[s] == -INFINITY) continue;
            mx = v > mx ? v : mx;
        }
    for (int o = G / 2; o > 0; o >>= 1) {
        const double t = __shfl_xor(mx, o);
        mx = t > mx ? t : mx;
    }
    if (l < p.L && mx != -INFINITY)
        for (int m = g; m < p.M; m += G) {
            const int s = l * p.M + m;
            if (lnomega[s] == -INFINITY) continue;
            sum += exp(lnomega[s] + f[s] + (double)N * p.lnz[s] - mx);
        }
    for (int o = G / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if (l < p.L && g == 0) la[l] = mx == -INFINITY ? -INFINITY : mx + log(sum) - p.beta_l[l] * p.mid[N];
    __syncthreads();
}

// One pass over the samples for one problem: the weights a_l of the chunk's N, then per
// sample its L exponentials and their sum.  Four lanes share a sample, each with every
// fourth temperature (J of them), so that their weights, exponents and sums stay in
// registers; a thread with all temperatures of a sample needed 256 registers and left
// the unit waiting (1.02e6 samples x 32 temperatures: 87 us, this 45 us).  Bound: FP64
// issue, about 22 operations per sample and temperature (18 us of it).
// Writes Q_l of its part of the chunk, or (LOGD) log D and 1 / sum_k a_k X_k of its samples.
template <int J, bool LOGD>
__global__ void __launch_bounds__(kMbarThreads) mbar_pass(SolveArgs p, double *logd)
{
    __shared__ double la[kMaxL];
    __shared__ double red[kMbarThreads / 64][4 * J];
    if (!LOGD && p.st[0].done) return;
    const int c = blockIdx.x / p.sub, part = blockIdx.x % p.sub;
    const int N = p.chunk_n[c];
    weights_log(p, p.lnomega, p.f, N, la);
    double shift = -INFINITY;
    for (int l = 0; l < p.L; ++l) shift = la[l] > shift ? la[l] : shift;
    if (part == 0 && threadIdx.x == 0) p.shift[N] = shift;
    const int q = threadIdx.x & 3;
    double a[J], db[J], acc[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int l = q + 4 * j;
        a[j] = l < p.L ? exp(la[l] - shift) : 0.0;
        db[j] = l < p.L ? p.beta_c - p.beta_l[l] : 0.0;
        acc[j] = 0.0;
    }
    const double mid = p.mid[N];
    const int step = p.sub * (kMbarThreads / 4);
    const int end = p.chunk_e[c];
    // (the next sample's energy is read before this one's exponentials)
    int i = p.chunk_b[c] + part * (kMbarThreads / 4) + (int)(threadIdx.x >> 2);
    double next = i < end ? p.e[i] : 0.0;
    for (; i < end; i += step) {
        const double t = next - mid;
        if (i + step < end) next = p.e[i + step];
        double x[J], d = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            x[j] = exp_bounded(db[j] * t);
            d = fma(a[j], x[j], d);
        }
        d = quad_total(d);
        if (LOGD) {
            if (q == 0) {
                logd[i] = shift - p.beta_c * t + log(d);
                p.hinv[i] = recip(d);
            }
        } else {
            const double inv = recip(d);
#pragma unroll
            for (int j = 0; j < J; ++j) acc[j] = fma(x[j], inv, acc[j]);
        }
    }
    if (LOGD) return;
    // the quads' sums: across the lanes of a wave that hold the same temperatures, then
    // the waves in order
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        double v = acc[j];
#pragma unroll
        for (int o = 4; o < 64; o <<= 1) v += __shfl_xor(v, o);
        if (lane < 4) red[wave][lane + 4 * j] = v;
    }
    __syncthreads();
    for (int l = threadIdx.x; l < p.L; l += blockDim.x) {
        double v = 0.0;
        for (int wv = 0; wv < kMbarThreads / 64; ++wv) v += red[wv][l];
        p.partial[(size_t)l * p.rows + blockIdx.x] = v;
    }
}

// New free energies of problem blockIdx.y, temperature blockIdx.x: the partial sums of
// each N (threads), then a wave per chemical potential sums over N.
constexpr int kFnewThreads = 512;

__global__ void __launch_bounds__(kFnewThreads) mbar_fnew_q(SolveArgs p)
{
    extern __shared__ double logB[];
    const int l = blockIdx.x, b = blockIdx.y;
    if (p.st[b].done) return;
    const double *part = p.partial + ((size_t)b * p.L + l) * p.rows;
    const double *lnomega = p.lnomega + (size_t)b * p.S + (size_t)l * p.M;
    // a temperature without samples has no weight A_l at any N: its states get no value
    int any = 0;
    for (int m = threadIdx.x; m < p.M; m += blockDim.x) any |= lnomega[m] != -INFINITY;
    any = __syncthreads_or(any);
    for (int N = threadIdx.x; N < p.nN; N += blockDim.x) {
        double Q = 0.0;
        for (int c = p.seg_c0[N] * p.sub; c < p.seg_c1[N] * p.sub; ++c) Q += part[c];
        logB[N] = any && Q > 0.0 ? log(Q) - p.beta_l[l] * p.mid[N] - p.shift[(size_t)b * p.nN + N] : -INFINITY;
    }
    __syncthreads();
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    for (int m = wave; m < p.M; m += kFnewThreads / 64) {
        const double lz = p.lnz[l * p.M + m];
        double mx = -INFINITY;
        for (int N = lane; N < p.nN; N += 64) mx = fmax(mx, fma((double)N, lz, logB[N]));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
        double sum = 0.0;
        if (mx != -INFINITY)
            for (int N = lane; N < p.nN; N += 64) sum += exp(fma((double)N, lz, logB[N]) - mx);
        sum = wave_total(sum);
        if (lane == 0) p.fnew[(size_t)b * p.S + l * p.M + m] = -(mx + log(sum));
    }
}

// Sums of the values first .. NV - 1 over a block of T threads, in every thread.
template <int T, int NV>
__device__ __forceinline__ void block_sums(double (&v)[NV], double (*red)[NV], int first)
{
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
#pragma unroll
    for (int k = first; k < NV; ++k) v[k] = wave_total(v[k]);
    if (T > 64) {
        __syncthreads();              // earlier readers of red are done
#pragma unroll
        for (int k = first; k < NV; ++k)
            if (lane == 0) red[wave][k] = v[k];
        __syncthreads();
#pragma unroll
        for (int k = first; k < NV; ++k) {
            v[k] = 0.0;
#pragma unroll
            for (int w = 0; w < T / 64; ++w) v[k] += red[w][k];
        }
    }
}

// The rest of an iteration for problem blockIdx.x: gauge, convergence, and the next
// iterate -- the map's value (method 0), or Anderson's mixture of the last map values
// (method 1; see solve_core).  One block of T threads with R states each: the least
// squares is a modified Gram-Schmidt whose columns stay in registers, one block-wide
// reduction per column.  Four waves hold them at every size: sixteen waves have a quarter of
// the registers each, and the columns of 1056 states in scratch made an iteration 295 us (33 x 32
// states to 1e-6: 7.2 -> 1.7 ms, 3.0 with the host's).  On the host it cost a copy each way, a synchronisation and the
// host's own sums every iteration (70 us of 230 at 1024 states).
template <int T, int R>
__global__ void __launch_bounds__(T) mbar_step(SolveArgs p)
{
    constexpr int K = kMaxMemory;
    __shared__ double red[T / 64][K + 1];
    __shared__ double Rs[K][K], qs[K];       // the triangular factor and Q^T r
    const int b = blockIdx.x, tid = threadIdx.x;
    SolveState &st = p.st[b];
    if (!st.done) {
        const double *lnomega = p.lnomega + (size_t)b * p.S, *fnew = p.fnew + (size_t)b * p.S;
        double *f = p.f + (size_t)b * p.S, *good = p.good + (size_t)b * p.S;
        double *hr = p.hist_r + (size_t)b * (K + 1) * p.S, *hg = p.hist_g + (size_t)b * (K + 1) * p.S;
        const double *y = p.y ? p.y + (size_t)b * p.S : nullptr;
        const double f0 = fnew[st.gauge];
        const int it = st.it + 1;
        double g[R], r[R], d = 0.0;
        bool on[R];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int s = tid + T * k;
            const bool in = s < p.S;
            on[k] = in && lnomega[s] != -INFINITY;
            g[k] = in ? fnew[s] - f0 : 0.0;
            r[k] = on[k] ? g[k] - f[s] : 0.0;
            const double a = fabs(r[k]);
            d = (a > d || a != a) ? a : d;           // a NaN propagates: the solve must see it
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double t = __shfl_xor(d, o);
            d = (t > d || t != t) ? t : d;
        }
        if (T > 64) {
            if (tid % 64 == 0) red[tid / 64][0] = d;
            __syncthreads();
            d = 0.0;
            for (int w = 0; w < T / 64; ++w) {
                const double t = red[w][0];
                d = (t > d || t != t) ? t : d;
            }
        }
        // every thread takes the same decisions from the same values
        int done = 0, conv = 0, hist = st.hist, head = st.head, plain_left = st.plain_left;
        double d_prev = st.d_prev;
        const int slots = st.memory + 1;
        const bool finite = d <= 1e300;
        const bool sw = finite && d < p.tol_switch;
        // A residual below tol leaves an error of up to tol |(I - J)^-1|: the iteration goes on
        // towards the residual's rounding, a few times at most (the preconditioned one, whose
        // steps are that error, while the residual still halves).  The residual may rise again on
        // the way: the result is the latest map value below tol, or the one below tol before it.
        int polish = st.polish;
        const bool under = p.method == 1 && !sw && finite && d < p.tol;
        const bool last = (polish > 0 && (!finite || polish >= p.polish || (y && !(d < 0.5 * d_prev)))) || (under && d < kFloor) ||
                          ((polish > 0 || under) && it >= p.max_iter) || (under && p.polish == 0);
        const bool newest = under && (!last || d <= st.kept);
        const double kept = newest ? d : st.kept;
        if (polish > 0 || under) ++polish;
        if (newest && !last)
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (tid + T * k < p.S) p.kept[(size_t)b * p.S + tid + T * k] = g[k];
        if (p.method == 0 || (!finite && it == 1) || last || sw) {
            // plain step, or the end: f is the map's value
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (tid + T * k < p.S) f[tid + T * k] = last && !newest ? p.kept[(size_t)b * p.S + tid + T * k] : g[k];
            if (last) d = kept;
            const bool check = p.method == 1 || it % 10 == 0 || it == p.max_iter;
            conv = check && (last || (finite && d < p.tol)) ? 1 : (sw ? 2 : 0);
            done = check && (conv || !finite);
        } else if (!finite) {
            // back to the last finite map value, plain steps for a while
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (tid + T * k < p.S) f[tid + T * k] = good[tid + T * k];
            hist = 0;
            plain_left = 5;
            d_prev = INFINITY;
        } else {
            if (d > 10.0 * d_prev) hist = 0;
            // the preconditioned map: x + y with y = (I - J)^-1 (g - x).  Near the end the
            // residual is the rounding of g, which (I - J)^-1 amplifies and the plain map
            // does not: where it stops falling, a few plain steps
            if (y && plain_left == 0 && polish == 0 && d < 1e-9 && d > 0.1 * d_prev) {
                hist = 0;
                plain_left = 4;
            }
            d_prev = d;
            if (y && plain_left == 0)
#pragma unroll
                for (int k = 0; k < R; ++k)
                    if (on[k]) {
                        r[k] = y[tid + T * k];
                        g[k] = f[tid + T * k] + r[k];
                    }
            // the new residual and map value take a free slot, or the oldest's
            if (hist == slots) head = (head + 1) % slots;
            else ++hist;
            const int now = (head + hist - 1) % slots;
            const int mk = hist - 1;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int s = tid + T * k;
                if (s < p.S) {
                    hr[(size_t)now * p.S + s] = r[k];
                    hg[(size_t)now * p.S + s] = g[k];
                    good[s] = g[k];
                }
            }
            double gamma[K] = {};
            const bool mix = plain_left == 0 && mk > 0;
            if (mix) {
                // columns: consecutive differences of the residuals, oldest first
                double q[K][R];
#pragma unroll
                for (int j = 0; j < K; ++j)
#pragma unroll
                    for (int k = 0; k < R; ++k) {
                        const int s = tid + T * k;
                        q[j][k] = 0.0;
                        if (j < mk && on[k]) {
                            const double lo = hr[(size_t)((head + j) % slots) * p.S + s];
                            const double hi = j + 1 == mk ? r[k] : hr[(size_t)((head + j + 1) % slots) * p.S + s];
                            q[j][k] = hi - lo;
                        }
                    }
                double norm0[K + 1] = {};
#pragma unroll
                for (int k = 0; k < R; ++k)
#pragma unroll
                    for (int i = 0; i < K; ++i) norm0[i] = fma(q[i][k], q[i][k], norm0[i]);
                block_sums<T>(norm0, red, 0);
                unsigned keep = 0;
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    if (j >= mk) break;
                    // column j against itself, the later columns and the residual
                    double v[K + 1] = {};
#pragma unroll
                    for (int k = 0; k < R; ++k) {
#pragma unroll
                        for (int i = j; i < K; ++i) v[i] = fma(q[j][k], q[i][k], v[i]);
                        v[K] = fma(q[j][k], r[k], v[K]);
                    }
                    block_sums<T>(v, red, j);
                    const double nn = v[j];
                    // a column that depends on earlier ones is left out
                    if (!(nn > 1e-24 * (norm0[j] + 1e-300))) continue;
                    keep |= 1u << j;
                    const double len = sqrt(nn);
                    if (tid == 0) {
                        qs[j] = v[K] / len;
                        Rs[j][j] = len;
                    }
#pragma unroll
                    for (int i = j + 1; i < K; ++i) {
                        if (tid == 0) Rs[j][i] = v[i] / len;
                        const double c = v[i] / nn;
#pragma unroll
                        for (int k = 0; k < R; ++k) q[i][k] = fma(-c, q[j][k], q[i][k]);
                    }
                }
                __syncthreads();
#pragma unroll
                for (int j = K - 1; j >= 0; --j) {
                    if (!((keep >> j) & 1u)) continue;
                    double v = qs[j];
#pragma unroll
                    for (int i = j + 1; i < K; ++i) v = fma(-Rs[j][i], gamma[i], v);    // (0 where left out)
                    gamma[j] = v / Rs[j][j];
                }
            }
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int s = tid + T * k;
                if (s >= p.S) continue;
                double v = g[k];
                if (mix && on[k]) {
                    double lo = hg[(size_t)head * p.S + s];
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        if (j >= mk) break;
                        const double hi = j + 1 == mk ? g[k] : hg[(size_t)((head + j + 1) % slots) * p.S + s];
                        v = fma(-gamma[j], hi - lo, v);
                        lo = hi;
                    }
                }
                f[s] = v;
            }
            if (plain_left > 0) --plain_left;
        }
        if (it >= p.max_iter) done = 1;
        __syncthreads();              // every thread has read the state
        if (tid == 0) {
            st.done = done; st.conv = conv; st.it = it; st.plain_left = plain_left;
            st.hist = hist; st.head = head; st.polish = polish;
            if (!finite) st.lost = 1;
            st.delta = d; st.d_prev = d_prev; st.kept = kept;
        }
    }
    // the last block of the launch tells the host how far the batch is, in one store
    if (tid == 0) {
        int done = p.st[b].done;
        if (gridDim.x > 1) {
            __threadfence();
            if (atomicAdd(p.arrived, 1u) != gridDim.x - 1) return;
            __threadfence();
            for (int k = 0; k < (int)gridDim.x; ++k)
                if (k != b) done += __hip_atomic_load(&p.st[k].done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *p.arrived = 0u;
        }
        const unsigned long long word = (unsigned long long)(++p.arrived[1]) | ((unsigned long long)done << 32);
        __hip_atomic_store(p.host, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// ---- the preconditioned iteration ----
// With J the Jacobian of the map f -> g(f) at the iterate, (I - J) = W^-1 H, where
// W_s = Omega_s e^{f_s - g_s} is the sum of state s's weights over the samples and
//     H = diag(W) - sum_n w_n w_n^T,  w_{n,lm} = p_l(n) q_lm(N),  q_lm(N) = Omega_lm z_lm^N e^{f_lm} / A_l(N),
// factorises like everything else over the product grid:
//     H_{lm,l'm'} = delta W_lm - sum_N q_lm(N) C_ll'(N) q_l'm'(N),   C_ll'(N) = sum_{n at N} p_l(n) p_l'(n).
// Anderson's iteration on x + H^-1 W (g(x) - x), with H taken once where max |g - x| has
// come below kSwitch, converges to 1e-12 in about ten steps where the plain one takes
// hundreds (its slowest errors shrink by a per cent or less per step).
constexpr double kSwitch = 0.1;
// More states or temperatures keep the plain iteration: the vector of mbar_newton_one and the
// products of mbar_pass_c hold so many in LDS, and larger inversions were not measured.  Fewer
// allowed iterations than kNewtonMinIter do too, as an attempt that fails takes up to 60.
constexpr int kNewtonStates = 1024, kNewtonTemps = 32, kNewtonMinIter = 64;
// Largest row sum of |(I - J)^-1| at which the solution counts as determined by the data:
// stopping at tol leaves an error of up to tol times it.  Above it the samples hardly
// connect the states, the point where an iteration stops depends on where it began, and
// the solve begins at f = 0 with the plain iteration.
constexpr double kMaxInverse = 2e4;
constexpr int kGj = 64;              // block of the inversion

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c)
{
    // lane l: a = A[l % 16][l / 16], b = B[l / 16][l % 16]; c[r] = C[l / 16 + 4 r][l % 16]
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// mbar_pass that also sums p p^T over the samples of its part of the chunk: a wave takes
// four samples at a time, lane (r, k) the temperatures r and r + 16 (G of them) of sample
// k, which is the layout of both operands of the matrix product.  C tiles (0,0), (0,1),
// (1,1) of the block go to cpart[block][tile][16][16], the log weights to lw [nN][L].
template <int G>
__global__ void __launch_bounds__(kMbarThreads) mbar_pass_c(SolveArgs p, double *cpart, double *lw)
{
    constexpr int NT = G == 1 ? 1 : 3;
    __shared__ double la[kMaxL];
    __shared__ double red[kMbarThreads / 64][16 * G];
    __shared__ double tile[NT][256];
    const int c = blockIdx.x / p.sub, part = blockIdx.x % p.sub;
    const int N = p.chunk_n[c];
    weights_log(p, p.lnomega, p.f, N, la);
    double shift = -INFINITY;
    for (int l = 0; l < p.L; ++l) shift = la[l] > shift ? la[l] : shift;
    if (part == 0) {
        if (threadIdx.x == 0) p.shift[N] = shift;
        if ((int)threadIdx.x < p.L) lw[(size_t)N * p.L + threadIdx.x] = la[threadIdx.x] + p.beta_l[threadIdx.x] * p.mid[N];
    }
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, k = lane / 16;
    double a[G], db[G], acc[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
        const int l = r + 16 * j;
        a[j] = l < p.L ? exp(la[l] - shift) : 0.0;
        db[j] = l < p.L ? p.beta_c - p.beta_l[l] : 0.0;
        acc[j] = 0.0;
    }
    f64x4 ct[NT] = {};
    const double mid = p.mid[N];
    const int end = p.chunk_e[c], step = p.sub * (kMbarThreads / 16);
    for (int i0 = p.chunk_b[c] + part * (kMbarThreads / 16) + wave * 4; i0 < end; i0 += step) {
        const int i = i0 + k;
        const double t = i < end ? p.e[i] - mid : 0.0;
        double x[G], d = 0.0;
#pragma unroll
        for (int j = 0; j < G; ++j) {
            x[j] = exp_bounded(db[j] * t);
            d = fma(a[j], x[j], d);
        }
        d = quad_total(d);
        d += dpp_move<0x141, 0xF>(d);
        d += dpp_move<0x140, 0xF>(d);       // the 16 lanes of the sample
        const double inv = i < end ? recip(d) : 0.0;
#pragma unroll
        for (int j = 0; j < G; ++j) {
            acc[j] = fma(x[j], inv, acc[j]);
            x[j] *= a[j] * inv;
        }
        ct[0] = mfma64(x[0], x[0], ct[0]);
        if constexpr (G == 2) {
            ct[1] = mfma64(x[0], x[1], ct[1]);
            ct[2] = mfma64(x[1], x[1], ct[2]);
        }
    }
#pragma unroll
    for (int j = 0; j < G; ++j) {
        double v = acc[j];
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 32);
        if (lane < 16) red[wave][lane + 16 * j] = v;
    }
    // the waves' tiles added in wave order
    for (int w = 0; w < kMbarThreads / 64; ++w) {
        if (wave == w)
#pragma unroll
            for (int q = 0; q < NT; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    double *dst = &tile[q][(k + 4 * e) * 16 + r];
                    *dst = w == 0 ? ct[q][e] : *dst + ct[q][e];
                }
        __syncthreads();
    }
    for (int l = threadIdx.x; l < p.L; l += blockDim.x) {
        double v = 0.0;
        for (int wv = 0; wv < kMbarThreads / 64; ++wv) v += red[wv][l];
        p.partial[(size_t)l * p.rows + blockIdx.x] = v;
    }
#pragma unroll
    for (int q = 0; q < NT; ++q) cpart[((size_t)blockIdx.x * NT + q) * 256 + threadIdx.x] = tile[q][threadIdx.x];
}

// Per N (block): C of its parts added, into csum[(l L + l') nK + N] (nK: nN rounded up to
// four, zero beyond), and the shares q_lm(N) into q[N][S].
__global__ void __launch_bounds__(256) mbar_csum(SolveArgs p, int nK, int tiles, const double *cpart, const double *lw,
                                              double *csum, double *q)
{
    const int N = blockIdx.x;
    const bool held = N < p.nN && p.seg_c1[N] > p.seg_c0[N];
    const int first = blockIdx.y * blockDim.x + threadIdx.x, stride = gridDim.y * blockDim.x;
    for (int t = first; t < p.L * p.L; t += stride) {
        const int l = t / p.L, l2 = t % p.L;
        double v = 0.0;
        if (held) {
            // stored tiles: rows l / 16 <= columns l' / 16
            const int lo = l < l2 ? l : l2, hi = l < l2 ? l2 : l;
            const int tl = lo / 16 == hi / 16 ? (lo / 16 == 0 ? 0 : tiles - 1) : 1;
#pragma unroll 4
            for (int c = p.seg_c0[N] * p.sub; c < p.seg_c1[N] * p.sub; ++c)
                v += cpart[((size_t)c * tiles + tl) * 256 + (lo % 16) * 16 + hi % 16];
        }
        csum[(size_t)t * nK + N] = v;
    }
    for (int s = first; s < p.S; s += stride) {
        double v = 0.0;
        if (held && p.lnomega[s] != -INFINITY)
            v = exp(p.lnomega[s] + p.f[s] + (double)N * p.lnz[s] - lw[(size_t)N * p.L + s / p.M]);
        q[(size_t)N * p.S + s] = v;
    }
}

// H in n x n storage (n: S rounded up to kGj; the identity for states without samples,
// the gauge state and the rounding) and W.  A wave per 16 x 16 tile of the chemical
// potentials of a pair l <= l' of temperatures; K = N.
__global__ void __launch_bounds__(64) mbar_hess(SolveArgs p, int nK, int n, const double *csum, const double *q, double *H,
                                             double *W)
{
    // the pair: blockIdx.x = l (2 L - l + 1) / 2 + (l' - l)
    int l = 0, rest = blockIdx.x;
    while (rest >= p.L - l) { rest -= p.L - l; ++l; }
    const int l2 = l + rest;
    const int lane = threadIdx.x, r = lane % 16, k = lane / 16;
    const int m = blockIdx.y * 16 + r, m2 = blockIdx.z * 16 + r;      // row of A, column of B
    const double *c = csum + (size_t)(l * p.L + l2) * nK;
    f64x4 acc = {};
    for (int N = k; N < nK; N += 4) {
        const double a = m < p.M ? q[(size_t)N * p.S + l * p.M + m] * c[N] : 0.0;
        const double b = m2 < p.M ? q[(size_t)N * p.S + l2 * p.M + m2] : 0.0;
        acc = mfma64(a, b, acc);
    }
    const int gauge = p.st[0].gauge;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int mi = blockIdx.y * 16 + k + 4 * e, mj = blockIdx.z * 16 + r;
        if (mi >= p.M || mj >= p.M) continue;
        const int s = l * p.M + mi, s2 = l2 * p.M + mj;
        const bool on = p.lnomega[s] != -INFINITY && p.lnomega[s2] != -INFINITY && s != gauge && s2 != gauge;
        double v = on ? -acc[e] : 0.0;
        if (s == s2) {
            const double w = on ? exp(p.lnomega[s] + p.f[s] - p.fnew[s]) : 0.0;
            W[s] = w;
            v = on ? w + v : 1.0;
        }
        H[(size_t)s * n + s2] = v;
        if (l != l2) H[(size_t)s2 * n + s] = v;      // (with l = l' the block of the other order writes it)
    }
}

// The identity in the rounding's rows and columns.
__global__ void mbar_pad(int S, int n, double *H)
{
    const int i = blockIdx.x;
    for (int j = threadIdx.x; j < n; j += blockDim.x)
        if (i >= S || j >= S) H[(size_t)i * n + j] = i == j ? 1.0 : 0.0;
}

// Block Gauss-Jordan inversion in place, step kb.  mbar_gj_row, block j: the pivot block
// inverted in LDS (every block its own copy), row block j of the pivot row times it into
// rowbuf, and column block j of the pivot column into colbuf.  mbar_gj_update, block
// (i, j): A_ij -= A_ik (P^-1 A_kj), and the pivot's row and column themselves.  H is
// symmetric and, where it is inverted at all, positive definite, so no pivoting.  Bound:
// the chain of the pivot blocks (64 steps each), about 20 us per step, 0.3 ms at 1024.
__global__ void __launch_bounds__(256) mbar_gj_row(int n, int kb, const double *A, double *rowbuf, double *colbuf)
{
    __shared__ double P[kGj][kGj + 1];
    __shared__ double prow[2][kGj], pcol[2][kGj];     // (by turns: one barrier per step)
    const int tid = threadIdx.x, j = blockIdx.x;
    const int ti = tid / 16, tj = tid % 16;           // rows ti + 16 a, columns tj + 16 b
    double v[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) v[a][b] = A[(size_t)(kb * kGj + ti + 16 * a) * n + kb * kGj + tj + 16 * b];
    for (int x = tid; x < kGj * kGj; x += 256)
        colbuf[(size_t)(j * kGj + x / kGj) * kGj + x % kGj] = A[(size_t)(j * kGj + x / kGj) * n + kb * kGj + x % kGj];
#pragma unroll
    for (int sa = 0; sa < 4; ++sa)
        for (int sr = 0; sr < 16; ++sr) {
            // row and column s = 16 sa + sr from the threads that hold them
            const int s = 16 * sa + sr;
            double *row = prow[sr & 1], *col = pcol[sr & 1];
            if (ti == sr)
#pragma unroll
                for (int b = 0; b < 4; ++b) row[tj + 16 * b] = v[sa][b];
            if (tj == sr)
#pragma unroll
                for (int b = 0; b < 4; ++b) col[ti + 16 * b] = v[b][sa];
            __syncthreads();
            const double piv = recip(row[s]);
            double rj[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) rj[b] = row[tj + 16 * b] * piv;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const bool pr = a == sa && ti == sr;
                const double ci = col[ti + 16 * a];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const bool pc = b == sa && tj == sr;
                    v[a][b] = pr ? (pc ? piv : rj[b]) : (pc ? -ci * piv : fma(-ci, rj[b], v[a][b]));
                }
            }
        }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) P[ti + 16 * a][tj + 16 * b] = v[a][b];
    __syncthreads();
    // rowbuf[., j] = P A[kb, j]; the pivot's own block gets the inverse
    const int wave = tid / 64, lane = tid % 64, r = lane % 16, k = lane / 16;
#pragma unroll
    for (int cj = 0; cj < 4; ++cj) {
        f64x4 acc = {};
        if (j != kb)
#pragma unroll
            for (int q = 0; q < kGj; q += 4)
                acc = mfma64(P[wave * 16 + r][q + k], A[(size_t)(kb * kGj + q + k) * n + j * kGj + cj * 16 + r], acc);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = wave * 16 + k + 4 * e, col = cj * 16 + r;
            rowbuf[(size_t)row * n + j * kGj + col] = j == kb ? P[row][col] : acc[e];
        }
    }
}

__global__ void __launch_bounds__(256) mbar_gj_update(int n, int kb, double *A, const double *rowbuf, const double *colbuf)
{
    const int i = blockIdx.y, j = blockIdx.x;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, k = lane / 16;
#pragma unroll
    for (int cj = 0; cj < 4; ++cj) {
        f64x4 acc = {};
        if (i != kb)
#pragma unroll
            for (int q = 0; q < kGj; q += 4)
                acc = mfma64(colbuf[(size_t)(i * kGj + wave * 16 + r) * kGj + q + k],
                             rowbuf[(size_t)(q + k) * n + j * kGj + cj * 16 + r], acc);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = wave * 16 + k + 4 * e, col = cj * 16 + r;
            double *a = A + (size_t)(i * kGj + row) * n + j * kGj + col;
            if (i == kb) *a = rowbuf[(size_t)row * n + j * kGj + col];
            else *a = (j == kb ? 0.0 : *a) - acc[e];
        }
    }
}

// Row sums of |H^-1 W|: one above kMaxInverse (or no number) ends the attempt, before its
// iterations.
__global__ void __launch_bounds__(64) mbar_inverse_norm(int S, int n, const double *Hi, const double *W, SolveState *st)
{
    double v = 0.0;
    for (int j = threadIdx.x; j < S; j += 64) v += fabs(Hi[(size_t)blockIdx.x * n + j] * W[j]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (threadIdx.x == 0 && !(v <= kMaxInverse)) st->done = 1;      // (with conv 0; every row stores the same)
}

// y = H^-1 W (fnew - f) of one problem: the vector in LDS, a wave per row.
__global__ void __launch_bounds__(256) mbar_newton_one(SolveArgs p, int n, const double *Hi, const double *W, double *y)
{
    __shared__ double v[kNewtonStates];
    if (p.st[0].done) return;
    for (int s = threadIdx.x; s < p.S; s += 256) {
        const double w = W[s];
        v[s] = w != 0.0 ? w * (p.fnew[s] - p.f[s]) : 0.0;
    }
    __syncthreads();
    const int row = blockIdx.x * 4 + threadIdx.x / 64;
    if (row >= p.S) return;
    const double *h = Hi + (size_t)row * n;
    double acc = 0.0;
#pragma unroll 4
    for (int s = threadIdx.x % 64; s < p.S; s += 64) acc = fma(h[s], v[s], acc);
    acc = wave_total(acc);
    if (threadIdx.x % 64 == 0) y[row] = acc;
}

// The same for 16 problems (columns) and 16 states (rows) per block; its waves
// split the sum over the states, their parts are added in wave order.
constexpr int kNewtonWaves = 8;

__global__ void __launch_bounds__(64 * kNewtonWaves) mbar_newton(SolveArgs p, int B, int n, const double *Hi,
                                                              const double *W, double *y)
{
    __shared__ double part[kNewtonWaves][256];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, k = lane / 16;
    const int row = blockIdx.x * 16 + r, b = blockIdx.y * 16 + r;
    const bool live = b < B && !p.st[b].done;
    const double *f = p.f + (size_t)b * p.S, *fnew = p.fnew + (size_t)b * p.S;
    f64x4 acc = {};
    for (int s0 = wave * 4; s0 < p.S; s0 += 4 * kNewtonWaves) {
        const int s = s0 + k;
        double v = 0.0;
        if (live && s < p.S) {
            const double w = W[s];
            v = w != 0.0 ? w * (fnew[s] - f[s]) : 0.0;
        }
        acc = mfma64(s < p.S ? Hi[(size_t)row * n + s] : 0.0, v, acc);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) part[wave][(k + 4 * e) * 16 + r] = acc[e];
    __syncthreads();
    if (threadIdx.x < 256) {
        double v = 0.0;
        for (int w = 0; w < kNewtonWaves; ++w) v += part[w][threadIdx.x];
        const int s = blockIdx.x * 16 + threadIdx.x / 16, c = blockIdx.y * 16 + threadIdx.x % 16;
        if (s < p.S && c < B) y[(size_t)c * p.S + s] = v;
    }
}

// ---- bootstrap replicates, all at once ----
// A replicate weights every sample by its record's multiplicity, so the exponentials X of
// a sample are the same for all of them and an iteration of B replicates is two matrix
// products around one division:
//     D[n][b] = sum_l X[n][l] a[l][b],   G = w / D,   Q[l][b] = sum_n X[n][l] G[n][b],
// on the FP64 matrix unit, 16 samples x 16 replicates per tile.  The tile of D leaves the
// first product in the layout in which the second takes G.  One after the other, 100
// replicates of 2.05e5 samples and 1024 states took 1.43 s in 15 700 passes; this takes 17
// iterations of 0.4 ms (162 us of it in the pass, about half its matrix-unit time).
// Replicates are columns b < Bp (B rounded up to 16); bb: columns per block of the pass.
constexpr int kBootTiles = 4;        // 16-column tiles per block of a pass
constexpr int kBootMax = 128;        // replicates at once
constexpr int kBootNs = 1024;        // values of N that 16 replicates keep in LDS

struct BootArgs {
    SolveArgs p;
    int B, Bp;
    const int32_t *rec;              // record of each sample, in sorted order
    const int32_t *mult;             // [record][Bp]
    double *a;                       // [nN][L][Bp] weights exp(log A_l - beta_l E0 - shift)
    double *part;                    // [rows][outputs][Bp]
    double *sum;                     // [nN][outputs][Bp]
};

// mult[r][b]: how often record r occurs in replicate b (block row y): block j (of ceil(R / block))
// starts at record floor(w (R - block + 1) / 2^32), w = word 0 of Philox block
// (j, b, 0xFFFFFFFE, 7), the concatenation cut to R records.  A thread per record of the
// concatenation: a workgroup that takes a replicate's blocks in turn needs half a microsecond
// for each (2e6 records in blocks of one, 100 replicates: 1190 -> 30 ms).
__global__ void boot_mult_all(int64_t R, int64_t block, int b0, int Bp, uint32_t k0, uint32_t k1, int32_t *mult)
{
    const int b = blockIdx.y;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < R; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t j = (int64_t)((uint32_t)i / (uint32_t)block);        // (R below 2^31)
        const uint4 w = philox4x32_10(make_uint4((uint32_t)j, (uint32_t)(b0 + b), 0xFFFFFFFEu, 7u), k0, k1);
        const int64_t start = (int64_t)(((uint64_t)w.x * (uint64_t)(R - block + 1)) >> 32);
        atomicAdd(mult + (start + i - j * block) * Bp + b, 1);
    }
}

__global__ void boot_records(int64_t ns, int64_t record_size, const int32_t *perm, int32_t *rec)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ns; i += (int64_t)gridDim.x * blockDim.x)
        rec[i] = (int32_t)(perm[i] / record_size);
}

// Weighted counts of the states: omega[s][b] += mult of the sample's record (lanes: b).
__global__ void boot_omega(int64_t ns, int64_t record_size, const int32_t *state, const int32_t *mult, int Bp, uint32_t *omega)
{
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, waves = blockDim.x / 64;
    for (int64_t i = blockIdx.x * (int64_t)waves + wave; i < ns; i += (int64_t)gridDim.x * waves) {
        const int64_t r = i / record_size;
        const int s = state[i];
        for (int b = lane; b < Bp; b += 64) {
            const int32_t m = mult[r * Bp + b];
            if (m) atomicAdd(omega + (size_t)s * Bp + b, (uint32_t)m);
        }
    }
}

// Replicate b (block): log weights of its states, start at f0, state of its solve.
__global__ void __launch_bounds__(256) boot_start(int S, int Bp, int memory, const uint32_t *omega, const double *f0,
                                               double *lnomega, double *f, double *good, SolveState *st)
{
    __shared__ int first, held;
    const int b = blockIdx.x;
    if (threadIdx.x == 0) { first = S; held = 0; }
    __syncthreads();
    for (int s = threadIdx.x; s < S; s += blockDim.x) {
        const uint32_t c = omega[(size_t)s * Bp + b];
        lnomega[(size_t)b * S + s] = c ? log((double)c) : -INFINITY;
        f[(size_t)b * S + s] = f0[s];
        good[(size_t)b * S + s] = f0[s];
        if (c) {
            atomicMin(&first, s);
            atomicAdd(&held, 1);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        SolveState z{};
        z.gauge = first < S ? first : 0;
        z.memory = min(memory, max(held - 2, 0));
        z.delta = z.d_prev = z.kept = INFINITY;
        st[b] = z;
    }
}

// Weights of replicate blockIdx.y at N = blockIdx.x.
__global__ void __launch_bounds__(kMbarThreads) boot_weights_log(BootArgs g, int all)
{
    __shared__ double la[kMaxL];
    const SolveArgs &p = g.p;
    const int N = blockIdx.x, b = blockIdx.y;
    if (p.seg_c1[N] == p.seg_c0[N] || (!all && p.st[b].done)) return;
    weights_log(p, p.lnomega + (size_t)b * p.S, p.f + (size_t)b * p.S, N, la);
    double shift = -INFINITY;
    for (int l = 0; l < p.L; ++l) shift = la[l] > shift ? la[l] : shift;
    if (threadIdx.x == 0) p.shift[(size_t)b * p.nN + N] = shift;
    if ((int)threadIdx.x < p.L)
        g.a[((size_t)N * p.L + threadIdx.x) * g.Bp + b] = exp(la[threadIdx.x] - shift);
}

// The pass: block (part of a chunk, group of kBootTiles column tiles, row tile pair).
// TARGET = false: rows are the temperatures, outputs Q_l (L <= 32: two row tiles).
// TARGET = true: rows are 16 target temperatures (tb), outputs the sums of
// exp(-(beta_t - c)(E - E0)) (E - E0)^k w / D, k = 0, 1, 2 (three row tiles).
template <bool TARGET>
__global__ void __launch_bounds__(kMbarThreads) boot_pass(BootArgs g, const double *tb, int nT)
{
    constexpr int RT = TARGET ? 3 : 2;
    extern __shared__ __align__(16) double lds[];
    const SolveArgs &p = g.p;
    const int c = blockIdx.x / p.sub, part = blockIdx.x % p.sub, N = p.chunk_n[c];
    const int b0 = blockIdx.y * kBootTiles * 16;
    const int tiles = min(kBootTiles, (g.Bp - b0) / 16);
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, k = lane / 16;
    // weights of this N: [32][kBootTiles * 16], zero beyond L
    constexpr int W = kBootTiles * 16;
    for (int x = threadIdx.x; x < 32 * W; x += blockDim.x) {
        const int l = x / W, b = b0 + x % W;
        lds[x] = l < p.L && b < g.Bp ? g.a[((size_t)N * p.L + l) * g.Bp + b] : 0.0;
    }
    __syncthreads();
    double db1[8], db2[2];
#pragma unroll
    for (int q = 0; q < 8; ++q) db1[q] = k + 4 * q < p.L ? p.beta_c - p.beta_l[k + 4 * q] : 0.0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int l = TARGET ? blockIdx.z * 16 + r : r + 16 * q;
        db2[q] = TARGET ? (l < nT ? p.beta_c - tb[l] : 0.0) : (l < p.L ? p.beta_c - p.beta_l[l] : 0.0);
    }
    f64x4 acc[kBootTiles][RT] = {};
    const double mid = p.mid[N];
    const int end = p.chunk_e[c], step = p.sub * (kMbarThreads / 64) * 16;
    for (int i0 = p.chunk_b[c] + (part * (kMbarThreads / 64) + wave) * 16; i0 < end; i0 += step) {
        // first product: sample r of the tile, temperatures k + 4 q
        const double t1 = i0 + r < end ? p.e[i0 + r] - mid : 0.0;
        double x1[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) x1[q] = exp_bounded(db1[q] * t1);
        // second: samples k + 4 e, temperature r (+ 16)
        double x2[RT][4];
        const int32_t *mu[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = i0 + k + 4 * e;
            const double t2 = i < end ? p.e[i] - mid : 0.0;
            x2[0][e] = exp_bounded(db2[0] * t2);
            if (TARGET) {
                x2[1][e] = x2[0][e] * t2;
                x2[RT - 1][e] = x2[1][e] * t2;
            } else {
                x2[1][e] = exp_bounded(db2[1] * t2);
            }
            mu[e] = i < end ? g.mult + (size_t)g.rec[i] * g.Bp + b0 + r : nullptr;
        }
#pragma unroll
        for (int t = 0; t < kBootTiles; ++t) {
            if (t >= tiles) break;
            f64x4 d = {};
#pragma unroll
            for (int q = 0; q < 8; ++q) d = mfma64(x1[q], lds[(k + 4 * q) * W + t * 16 + r], d);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double w = mu[e] ? (double)mu[e][t * 16] : 0.0;
                const double gw = w != 0.0 ? w * recip(d[e]) : 0.0;
#pragma unroll
                for (int j = 0; j < RT; ++j) acc[t][j] = mfma64(x2[j][e], gw, acc[t][j]);
            }
        }
    }
    // the waves' tiles added in wave order (LDS: [row][W]), then to memory
    __syncthreads();
    for (int w = 0; w < kMbarThreads / 64; ++w) {
        if (wave == w)
#pragma unroll
            for (int t = 0; t < kBootTiles; ++t)
#pragma unroll
                for (int j = 0; j < RT; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        double *dst = lds + (16 * j + k + 4 * e) * W + t * 16 + r;
                        *dst = w == 0 ? acc[t][j][e] : *dst + acc[t][j][e];
                    }
        __syncthreads();
    }
    // output rows: temperature l, or (target t, moment j) as t 3 + j
    const int outs = TARGET ? 3 * nT : p.L;
    for (int x = threadIdx.x; x < 16 * RT * W; x += blockDim.x) {
        const int row = x / W, b = b0 + x % W;
        const int t = blockIdx.z * 16 + row % 16;
        const int o = TARGET ? (t < nT ? t * 3 + row / 16 : -1) : (row < p.L ? row : -1);
        if (o >= 0 && b < g.Bp) g.part[((size_t)blockIdx.x * outs + o) * g.Bp + b] = lds[x];
    }
}

// Parts of each N (block x) added in order: sum[N][outputs][Bp].
__global__ void __launch_bounds__(256) boot_sum(BootArgs g, int outs)
{
    const int N = blockIdx.x;
    const size_t row = (size_t)outs * g.Bp;
    const int c0 = g.p.seg_c0[N] * g.p.sub, c1 = g.p.seg_c1[N] * g.p.sub;
    for (size_t x = blockIdx.y * (size_t)blockDim.x + threadIdx.x; x < row; x += (size_t)gridDim.y * blockDim.x) {
        double v = 0.0;
#pragma unroll 4
        for (int c = c0; c < c1; ++c) v += g.part[c * row + x];
        g.sum[N * row + x] = v;
    }
}

// New free energies of temperature blockIdx.x in 16 replicates: mbar_fnew_q of each.
__global__ void __launch_bounds__(kFnewThreads) boot_fnew(BootArgs g)
{
    extern __shared__ double logB[];          // [16][nN]
    const SolveArgs &p = g.p;
    const int l = blockIdx.x, b0 = blockIdx.y * 16;
    const double bl = p.beta_l[l];
    __shared__ int any[16];
    if (threadIdx.x < 16) any[threadIdx.x] = 0;
    __syncthreads();
    for (int x = threadIdx.x; x < 16 * p.M; x += blockDim.x) {
        const int b = b0 + x / p.M;
        if (b < g.B && p.lnomega[(size_t)b * p.S + l * p.M + x % p.M] != -INFINITY) any[x / p.M] = 1;
    }
    __syncthreads();
    for (int x = threadIdx.x; x < 16 * p.nN; x += blockDim.x) {
        const int N = x / 16, b = x % 16;
        double v = -INFINITY;
        if (b0 + b < g.B && any[b] && p.seg_c1[N] > p.seg_c0[N]) {
            const double Q = g.sum[((size_t)N * p.L + l) * g.Bp + b0 + b];
            if (Q > 0.0) v = log(Q) - bl * p.mid[N] - p.shift[(size_t)(b0 + b) * p.nN + N];
        }
        logB[b * p.nN + N] = v;
    }
    __syncthreads();
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    for (int x = wave; x < 16 * p.M; x += kFnewThreads / 64) {
        const int b = x / p.M, m = x % p.M;
        if (b0 + b >= g.B || p.st[b0 + b].done) continue;
        const double *lb = logB + b * p.nN;
        const double lz = p.lnz[l * p.M + m];
        double mx = -INFINITY;
        for (int N = lane; N < p.nN; N += 64) mx = fmax(mx, fma((double)N, lz, lb[N]));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
        double sum = 0.0;
        if (mx != -INFINITY)
            for (int N = lane; N < p.nN; N += 64) sum += exp(fma((double)N, lz, lb[N]) - mx);
        sum = wave_total(sum);
        if (lane == 0) p.fnew[(size_t)(b0 + b) * p.S + l * p.M + m] = -(mx + log(sum));
    }
}

// <N> and the heat capacity of replicate blockIdx.y at target temperature blockIdx.x: G(N)
// and the moments of E at each N from the sums, then a wave per chemical potential.  nT: the
// temperatures of this pass, nK: targets of a replicate in rep_n and rep_c.
__global__ void __launch_bounds__(256) boot_target_eval(BootArgs g, int nT, int nMu, int nK, const double *tb,
                                                     const double *tlnz, double *rep_n, double *rep_c)
{
    extern __shared__ double sh[];
    const SolveArgs &p = g.p;
    const int t = blockIdx.x, b = blockIdx.y;
    double *G = sh, *E1 = sh + p.nN, *E2 = sh + 2 * p.nN;
    for (int N = threadIdx.x; N < p.nN; N += blockDim.x) {
        double gn = -INFINITY, e1 = 0.0, e2 = 0.0;
        if (p.seg_c1[N] > p.seg_c0[N]) {
            const double *m = g.sum + ((size_t)N * 3 * nT + 3 * t) * g.Bp + b;
            const double m0 = m[0], mid = p.mid[N];
            if (m0 > 0.0) {
                const double d1 = m[g.Bp] / m0, d2 = m[2 * (size_t)g.Bp] / m0;
                gn = log(m0) - tb[t] * mid - p.shift[(size_t)b * p.nN + N];
                e1 = mid + d1;
                e2 = fma(mid, mid, fma(2.0 * mid, d1, d2));
            }
        }
        G[N] = gn;
        E1[N] = e1;
        E2[N] = e2;
    }
    __syncthreads();
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    for (int m = wave; m < nMu; m += blockDim.x / 64) {
        const double lz = tlnz[t * nMu + m];
        double mx = -INFINITY;
        for (int N = lane; N < p.nN; N += 64) mx = fmax(mx, fma((double)N, lz, G[N]));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
        double s0 = 0.0, sn = 0.0, se = 0.0, se2 = 0.0;
        for (int N = lane; N < p.nN; N += 64) {
            const double w = G[N] == -INFINITY ? 0.0 : exp(fma((double)N, lz, G[N]) - mx);
            s0 += w;
            sn = fma(w, (double)N, sn);
            se = fma(w, E1[N], se);
            se2 = fma(w, E2[N], se2);
        }
        s0 = wave_total(s0);
        sn = wave_total(sn);
        se = wave_total(se);
        se2 = wave_total(se2);
        if (lane == 0) {
            const size_t k = (size_t)b * nK + t * nMu + m;
            const double e1 = se / s0;
            rep_n[k] = sn / s0;
            rep_c[k] = tb[t] * tb[t] * (se2 / s0 - e1 * e1);
        }
    }
}

// ---- averages at target temperatures on bounded exponents ----
// With h = 1 / sum_k a_k X_k of the solution (mbar_pass) a sample's weight at a target
// temperature is e^{-beta_t E - log D} = e^{-beta_t E0 - shift} exp(-(beta_t - c)(E - E0)) h,
// so a chunk's sums need one exponential per sample and target, no running maximum, and
// the moments are those of E - E0.  Four lanes share a sample as in mbar_pass.  64
// targets x 1.02e6 samples: 540 -> 80 us.  Output [chunk][target][4] (three used).
template <int J>
__global__ void __launch_bounds__(kMbarThreads) mbar_target_pass(SolveArgs p, int nT, const double *tb, double *tpart)
{
    __shared__ double red[kMbarThreads / 64][4 * J][3];
    const int c = blockIdx.x, t0 = blockIdx.y * 4 * J, q = threadIdx.x & 3;
    double db[J], a0[J], a1[J], a2[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int t = t0 + q + 4 * j;
        db[j] = t < nT ? p.beta_c - tb[t] : 0.0;
        a0[j] = a1[j] = a2[j] = 0.0;
    }
    const double mid = p.mid[p.chunk_n[c]];
    const int end = p.chunk_e[c];
    int i = p.chunk_b[c] + (int)(threadIdx.x >> 2);
    double ne = i < end ? p.e[i] : 0.0, nh = i < end ? p.hinv[i] : 0.0;
    for (; i < end; i += kMbarThreads / 4) {
        const double d = ne - mid, h = nh;
        if (i + kMbarThreads / 4 < end) {
            ne = p.e[i + kMbarThreads / 4];
            nh = p.hinv[i + kMbarThreads / 4];
        }
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const double w = exp_bounded(db[j] * d) * h, wd = w * d;
            a0[j] += w;
            a1[j] += wd;
            a2[j] = fma(wd, d, a2[j]);
        }
    }
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        double v[3] = {a0[j], a1[j], a2[j]};
#pragma unroll
        for (int k = 0; k < 3; ++k) {
#pragma unroll
            for (int o = 4; o < 64; o <<= 1) v[k] += __shfl_xor(v[k], o);
            if (lane < 4) red[wave][lane + 4 * j][k] = v[k];
        }
    }
    __syncthreads();
    for (int x = threadIdx.x; x < 12 * J; x += blockDim.x) {
        const int t = x / 3, k = x % 3;
        if (t0 + t >= nT) continue;
        double v = 0.0;
        for (int w = 0; w < kMbarThreads / 64; ++w) v += red[w][t][k];
        tpart[((size_t)c * nT + t0 + t) * 4 + k] = v;
    }
}

// The averages at target temperature blockIdx.x from the chunks' sums: G(N) and the
// moments of E at each N (threads), then a wave per chemical potential (a thread each and
// every p(N) in turn: 90 us for 64 x 64 targets and 512 N; 46 us).  A block takes kEvalMu of the
// chemical potentials (blockIdx.y), each with its own copy of G and the moments: all 700 of one
// temperature in one block were 88 in turn for a wave (2 x 700 targets and 41 N 180 -> 345 us; now 166).
constexpr int kEvalThreads = 512, kEvalMu = 64;

__global__ void __launch_bounds__(kEvalThreads) mbar_target_eval_q(SolveArgs p, int nT, int nMu, const double *tb,
                                                                const double *tpart, const double *tlnz, double *f,
                                                                double *mean_n, double *mean_e, double *mean_e2, double *p_n,
                                                                int32_t *phase)
{
    extern __shared__ double sh[];
    double *G = sh, *E1 = sh + p.nN, *E2 = sh + 2 * p.nN;
    const int t = blockIdx.x;
    for (int N = threadIdx.x; N < p.nN; N += blockDim.x) {
        double m0 = 0.0, m1 = 0.0, m2 = 0.0;
        for (int c = p.seg_c0[N]; c < p.seg_c1[N]; ++c) {
            const double *o = tpart + ((size_t)c * nT + t) * 4;
            m0 += o[0]; m1 += o[1]; m2 += o[2];
        }
        const double mid = p.mid[N], d1 = m0 > 0.0 ? m1 / m0 : 0.0, d2 = m0 > 0.0 ? m2 / m0 : 0.0;
        G[N] = m0 > 0.0 ? log(m0) - tb[t] * mid - p.shift[N] : -INFINITY;
        E1[N] = m0 > 0.0 ? mid + d1 : 0.0;
        E2[N] = m0 > 0.0 ? fma(mid, mid, fma(2.0 * mid, d1, d2)) : 0.0;
    }
    __syncthreads();
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    // (kEvalMu is a multiple of the waves, so that a wave's next one after them is the next group's)
    for (int m = blockIdx.y * kEvalMu + wave; m < nMu;
         m += m % kEvalMu + kEvalThreads / 64 < kEvalMu ? kEvalThreads / 64 : kEvalThreads / 64 + ((int)gridDim.y - 1) * kEvalMu) {
        const int k = t * nMu + m;
        const double lz = tlnz[k];
        double mx = -INFINITY;
        int best = 0;
        for (int N = lane; N < p.nN; N += 64) {
            const double v = fma((double)N, lz, G[N]);
            if (v > mx) { mx = v; best = N; }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double v = __shfl_xor(mx, o);
            const int b = __shfl_xor(best, o);
            if (v > mx || (v == mx && b < best)) { mx = v; best = b; }     // the smallest N on ties
        }
        double s0 = 0.0, sn = 0.0, se = 0.0, se2 = 0.0;
        for (int N = lane; N < p.nN; N += 64) {
            const double w = G[N] == -INFINITY ? 0.0 : exp(fma((double)N, lz, G[N]) - mx);
            s0 += w;
            sn = fma(w, (double)N, sn);
            se = fma(w, E1[N], se);
            se2 = fma(w, E2[N], se2);
        }
        s0 = wave_total(s0);
        sn = wave_total(sn);
        se = wave_total(se);
        se2 = wave_total(se2);
        if (p_n) {
            const double inv = 1.0 / s0;
            for (int N = lane; N < p.nN; N += 64)
                p_n[(size_t)k * p.nN + N] = G[N] == -INFINITY ? 0.0 : exp(fma((double)N, lz, G[N]) - mx) * inv;
        }
        if (lane == 0) {
            if (f) f[k] = -(mx + log(s0));
            mean_n[k] = sn / s0;
            if (mean_e) mean_e[k] = se / s0;
            if (mean_e2) mean_e2[k] = se2 / s0;
            if (phase) phase[k] = best;
        }
    }
}

// Observables on bounded exponents: sums over a chunk's part (block x of rows) of
// w_t obs_k for 16 target temperatures (block z) and all observables, and of w_t (column
// n_obs), a matrix product on the FP64 matrix unit: rows t, columns k, four samples per
// step.  A wave takes four tiles of 16 columns.  The records are read once, not once per
// temperature (2.05e5 samples x 221 x 16: 360 -> 177 us).  out [row][nT][n_obs + 1].
__global__ void __launch_bounds__(kMbarThreads) mbar_obs_pass(SolveArgs p, int nT, int n_obs, const double *tb,
                                                           const uint32_t *obs, double *out)
{
    const int c = blockIdx.x / p.sub, part = blockIdx.x % p.sub;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, k = lane / 16;
    const int t = blockIdx.z * 16 + r, col0 = (blockIdx.y * (kMbarThreads / 64) + wave) * 64;
    if (col0 > n_obs) return;
    const double db = t < nT ? p.beta_c - tb[t] : 0.0;
    const double mid = p.mid[p.chunk_n[c]];
    const int b = p.chunk_b[c], cnt = p.chunk_e[c] - b;
    const int lo = b + (int)((int64_t)cnt * part / p.sub), end = b + (int)((int64_t)cnt * (part + 1) / p.sub);
    f64x4 acc[4] = {};
    // sixteen samples per round: all their loads are in flight before the first product
    for (int i0 = lo; i0 < end; i0 += 16) {
        uint32_t v[4][4];
        double d[4], h[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + 4 * u + k, ic = i < end ? i : lo;
            const uint32_t *o = obs + (size_t)ic * n_obs;
            d[u] = p.e[ic];
            h[u] = i < end ? p.hinv[ic] : 0.0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = col0 + 16 * q + r;
                v[u][q] = col < n_obs ? o[col] : 1u;      // (columns past n_obs are not written)
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double w = exp_bounded(db * (d[u] - mid)) * h[u];
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = mfma64(w, (double)v[u][q], acc[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int to = blockIdx.z * 16 + k + 4 * e, col = col0 + 16 * q + r;
            if (to < nT && col <= n_obs) out[((size_t)blockIdx.x * nT + to) * (n_obs + 1) + col] = acc[q][e];
        }
}

// cond[t][N][k] and G[t][N] from the parts, block (N, t).
__global__ void __launch_bounds__(256) mbar_obs_cond(SolveArgs p, int nT, int n_obs, const double *tb, const double *part,
                                                  double *cond, double *G)
{
    const int N = blockIdx.x, t = blockIdx.y;
    const int c0 = p.seg_c0[N] * p.sub, c1 = p.seg_c1[N] * p.sub;
    const size_t stride = (size_t)nT * (n_obs + 1);
    const double *src = part + (size_t)t * (n_obs + 1);
    double s0 = 0.0;
#pragma unroll 8
    for (int c = c0; c < c1; ++c) s0 += src[c * stride + n_obs];
    if (threadIdx.x == 0) G[(size_t)t * p.nN + N] = s0 > 0.0 ? log(s0) - tb[t] * p.mid[N] - p.shift[N] : -INFINITY;
    for (int k = threadIdx.x; k < n_obs; k += blockDim.x) {
        double a = 0.0;
#pragma unroll 8
        for (int c = c0; c < c1; ++c) a += src[c * stride + k];
        cond[((size_t)t * p.nN + N) * n_obs + k] = s0 > 0.0 ? a / s0 : 0.0;
    }
}

// mean[t][mu][k] = sum_N p(N) cond[t][N][k], block (mu, t) (a block per t with mu in turn:
// 6.4 ms for 16 temperatures x 64 mu x 221 counts; 16 x 64 blocks: 30 us).
__global__ void __launch_bounds__(256) mbar_obs_mean(int nMu, int nN, int n_obs, const double *G, const double *tlnz,
                                                  const double *cond, double *mean)
{
    extern __shared__ double P[];
    const int m = blockIdx.x, t = blockIdx.y, lane = threadIdx.x % 64;
    const double lz = tlnz[t * nMu + m];
    const double *g = G + (size_t)t * nN;
    double mx = -INFINITY, sum = 0.0;              // (every wave for itself)
    for (int N = lane; N < nN; N += 64) mx = fmax(mx, fma((double)N, lz, g[N]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
    for (int N = lane; N < nN; N += 64) sum += g[N] == -INFINITY ? 0.0 : exp(fma((double)N, lz, g[N]) - mx);
    sum = wave_total(sum);
    for (int N = threadIdx.x; N < nN; N += blockDim.x)
        P[N] = g[N] == -INFINITY ? 0.0 : exp(fma((double)N, lz, g[N]) - mx) / sum;
    __syncthreads();
    for (int k = threadIdx.x; k < n_obs; k += blockDim.x) {
        double acc = 0.0;
        const double *c = cond + (size_t)t * nN * n_obs + k;
#pragma unroll 8
        for (int N = 0; N < nN; ++N) acc = fma(P[N], c[(size_t)N * n_obs], acc);
        mean[((size_t)t * nMu + m) * n_obs + k] = acc;
    }
}

}  // namespace regc

using namespace regc;

struct regc_mbar {
    int L = 0, M = 0, S = 0, nN = 0;
    double lambda1 = 1.0;
    std::vector<double> t, mu, beta_l, lnz;
    hipStream_t stream = nullptr;
    DevBuf<double> beta_d, lnz_d, lnomega_d, f_d, fnew_d, logA_d, partial_d, delta_d, e_d, logd_d;
    DevBuf<int32_t> perm_d;           // sorted position -> original sample index
    DevBuf<uint32_t> obs_d;           // observables in sorted order [ns][n_obs]
    int n_obs = 0;
    DevBuf<int> chunk_n_d, chunk_b_d, chunk_e_d, seg_c0_d, seg_c1_d;
    int64_t ns = 0;
    int nchunks = 0;
    int gauge = -1;
    std::vector<double> lnomega;
    bool have_samples = false, solved = false;
    double ms_iter = 0.0;
    int64_t n_iter = 0;
    int method = 1, memory = 8;
    DevBuf<int32_t> n_orig_d, s_orig_d;   // N and state of the samples in the order given
    DevBuf<double> wgt_d;                 // bootstrap multiplicities in sorted order
    bool weighted = false;
    // the device-resident iteration
    double beta_c = 0.0, beta_half = 0.0; // middle and half width of the inverse temperatures
    DevBuf<double> mid_d, half_d;         // middle and half width of the energies sampled at each N
    bool bounded = false;                 // the exponents around them stay below kMaxSolveExponent
    bool tight = false;                   // and below kMaxExponent
    double half_max = 0.0;                // the largest half width
    DevBuf<double> hinv_d;                // 1 / sum of every sample at the solution
    bool hinv_valid = false;              // hinv_d and shift_d are those of the solution in f_d
    int sub = 1;                          // blocks per chunk of a pass
    DevBuf<double> shift_d, q_d, hist_r_d, hist_g_d, good_d, kept_d;
    DevBuf<SolveState> state_d;
    DevBuf<unsigned int> arrived_d;
    unsigned long long *progress = nullptr;   // host memory the step kernel writes (SolveArgs::host)
    // the preconditioned iteration
    std::vector<double> mean_n, mean_e;   // of the samples of each state (empty: not known)
    DevBuf<double> cpart_d, lw_d, csum_d, share_d, hess_d, w_d, row_d, col_d, y_d;
    bool inverse_valid = false;           // hess_d holds the inverse of the solution's solve
    // the bootstrap's batch
    DevBuf<int32_t> b_rec_d, b_mult_d;
    DevBuf<uint32_t> b_omega_d;
    DevBuf<double> b_lnomega_d, b_f_d, b_fnew_d, b_good_d, b_hr_d, b_hg_d, b_shift_d, b_a_d, b_part_d, b_sum_d;
    DevBuf<SolveState> b_state_d;
    // set_samples' intermediates
    DevBuf<double> e_in_d;
    DevBuf<uint32_t> keys_d, keys_out_d;
    DevBuf<int32_t> idx_d;
    DevBuf<unsigned char> sort_d, count_d;
    DevBuf<unsigned long long> totals_d;
    DevBuf<int> bad_d;
    ~regc_mbar()
    {
        if (progress) (void)hipHostFree(progress);
    }
};

static double lnz_of(double T, double mu, double lambda1)
{
    return mu / T - 3.0 * std::log(lambda1 / std::sqrt(T));
}

extern "C" int regc_mbar_create(const regc_grid *grid, double lambda1, int n_max, regc_mbar **out)
{
    REGC_CHECK(grid && out && grid->t && grid->mu, REGC_EINVAL, "null argument");
    REGC_CHECK(grid->n_t > 0 && grid->n_mu > 0 && n_max >= 0, REGC_EINVAL, "empty grid or negative n_max");
    REGC_CHECK(grid->n_t <= kMaxL, REGC_EUNSUPPORTED, "at most %d temperatures per reweighting grid", kMaxL);
    REGC_CHECK(n_max < 2048, REGC_EUNSUPPORTED, "n_max above 2047");
    REGC_CHECK(lambda1 > 0, REGC_EINVAL, "lambda1 must be positive");
    regc_mbar *mb = new regc_mbar();
    mb->L = grid->n_t; mb->M = grid->n_mu; mb->S = mb->L * mb->M; mb->nN = n_max + 1;
    mb->lambda1 = lambda1;
    mb->t.assign(grid->t, grid->t + mb->L);
    mb->mu.assign(grid->mu, grid->mu + mb->M);
    for (int l = 0; l < mb->L; ++l) {
        if (!(mb->t[l] > 0)) { delete mb; set_error("temperatures must be positive"); return REGC_EINVAL; }
        mb->beta_l.push_back(1.0 / mb->t[l]);
        for (int m = 0; m < mb->M; ++m) mb->lnz.push_back(lnz_of(mb->t[l], mb->mu[m], lambda1));
    }
    const auto ends = std::minmax_element(mb->beta_l.begin(), mb->beta_l.end());
    mb->beta_c = 0.5 * (*ends.first + *ends.second);
    mb->beta_half = 0.5 * (*ends.second - *ends.first);
    int rc;
    if ((rc = mb->beta_d.alloc(mb->L)) || (rc = mb->lnz_d.alloc(mb->S)) || (rc = mb->lnomega_d.alloc(mb->S)) ||
        (rc = mb->f_d.alloc(mb->S)) || (rc = mb->fnew_d.alloc(mb->S)) ||
        (rc = mb->logA_d.alloc((size_t)mb->L * mb->nN)) || (rc = mb->delta_d.alloc(1)) ||
        (rc = mb->seg_c0_d.alloc(mb->nN)) || (rc = mb->seg_c1_d.alloc(mb->nN)) || (rc = mb->mid_d.alloc(mb->nN)) ||
        (rc = mb->half_d.alloc(mb->nN))) {
        delete mb;
        return rc;
    }
    if (hipMemcpy(mb->beta_d.p, mb->beta_l.data(), sizeof(double) * mb->L, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(mb->lnz_d.p, mb->lnz.data(), sizeof(double) * mb->S, hipMemcpyHostToDevice) != hipSuccess) {
        delete mb;
        set_error("hipMemcpy failed");
        return REGC_EHIP;
    }
    *out = mb;
    return REGC_OK;
}

extern "C" int regc_mbar_set_stream(regc_mbar *mb, void *stream)
{
    REGC_CHECK(mb, REGC_EINVAL, "null handle");
    mb->stream = (hipStream_t)stream;
    return REGC_OK;
}

constexpr int64_t kKeptSamples = (int64_t)1 << 23;

extern "C" int regc_mbar_set_samples(regc_mbar *mb, int64_t ns, const double *e, const int32_t *n,
                                     const int32_t *state, int on_device)
{
    REGC_CHECK(mb, REGC_EINVAL, "null handle");
    REGC_CHECK(ns > 0 && e && n && state, REGC_EINVAL, "no samples");
    REGC_CHECK(ns < (int64_t)1 << 31, REGC_EUNSUPPORTED, "more than 2^31 - 1 samples");
    // the handle's sample buffers are replaced below: until this call succeeds the
    // handle holds no samples (a failed call leaves it empty, not half updated)
    mb->have_samples = false;
    mb->solved = false;
    mb->hinv_valid = false;
    mb->n_obs = 0;
    hipStream_t s = mb->stream;
    const hipMemcpyKind kind = on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
    DevBuf<double> &e_in = mb->e_in_d;
    DevBuf<int32_t> &n_in = mb->n_orig_d, &s_in = mb->s_orig_d, &idx = mb->idx_d, &idx_out = mb->perm_d;
    DevBuf<uint32_t> &keys = mb->keys_d, &keys_out = mb->keys_out_d;
    mb->weighted = false;
    mb->mean_n.clear();
    mb->mean_e.clear();
    int rc;
    const size_t totals = 3 * (size_t)mb->S + mb->nN;
    // the counters of a block in LDS where they fit (64 KB), else one set in memory
    const size_t cbytes = count_bytes(mb->S, mb->nN);
    const bool lds_count = cbytes <= 65536;
    const int cblocks = (int)std::min<int64_t>(kCountBlocks, (ns + 1023) / 1024);
    if ((rc = e_in.reserve(ns)) || (rc = n_in.reserve(ns)) || (rc = s_in.reserve(ns)) || (rc = keys.reserve(ns)) ||
        (rc = keys_out.reserve(ns)) || (rc = idx.reserve(ns)) || (rc = idx_out.reserve(ns)) ||
        (rc = mb->totals_d.reserve(totals)) || (rc = mb->count_d.reserve(lds_count ? cblocks * cbytes : 1)) ||
        (rc = mb->bad_d.reserve(1)) || (rc = mb->e_d.reserve(ns)) || (rc = mb->logd_d.reserve(ns)))
        return rc;
    REGC_HIP(hipMemcpyAsync(e_in.p, e, sizeof(double) * ns, kind, s));
    REGC_HIP(hipMemcpyAsync(n_in.p, n, sizeof(int32_t) * ns, kind, s));
    REGC_HIP(hipMemcpyAsync(s_in.p, state, sizeof(int32_t) * ns, kind, s));
    REGC_HIP(hipMemsetAsync(mb->bad_d.p, 0, sizeof(int), s));
    const int grid = (int)std::min<int64_t>((ns + 255) / 256, 4096);
    if (lds_count) {
        hipLaunchKernelGGL(mbar_count, dim3(cblocks), dim3(kCountThreads), cbytes, s, ns, n_in.p, s_in.p, e_in.p, mb->nN,
                           mb->S, mb->count_d.p, mb->bad_d.p);
        hipLaunchKernelGGL(mbar_count_sum, dim3((unsigned)((totals + 63) / 64)), dim3(64), 0, s, cblocks, mb->S, mb->nN,
                           mb->count_d.p, mb->totals_d.p);
    } else {
        REGC_HIP(hipMemsetAsync(mb->totals_d.p, 0, sizeof(unsigned long long) * totals, s));
        hipLaunchKernelGGL(mbar_count_global, dim3(grid), dim3(256), 0, s, ns, n_in.p, s_in.p, mb->nN, mb->S,
                           mb->totals_d.p + mb->S, mb->totals_d.p + 3 * (size_t)mb->S, mb->bad_d.p);
    }
    REGC_HIP(hipGetLastError());
    int h_bad = 0;
    std::vector<unsigned long long> h_tot(totals);
    REGC_HIP(hipMemcpyAsync(&h_bad, mb->bad_d.p, sizeof(int), hipMemcpyDeviceToHost, s));
    REGC_HIP(hipMemcpyAsync(h_tot.data(), mb->totals_d.p, sizeof(unsigned long long) * totals, hipMemcpyDeviceToHost, s));
    REGC_HIP(hipStreamSynchronize(s));
    REGC_CHECK(!h_bad, REGC_EINVAL, "sample with N outside 0..n_max or state outside the grid");
    const unsigned long long *h_omega = h_tot.data() + mb->S, *h_seg = h_tot.data() + 3 * (size_t)mb->S;
    if (lds_count) {
        mb->mean_n.assign(mb->S, 0.0);
        mb->mean_e.assign(mb->S, 0.0);
        for (int k = 0; k < mb->S; ++k)
            if (h_omega[k] > 0) {
                mb->mean_n[k] = (double)h_tot[2 * (size_t)mb->S + k] / (double)h_omega[k];
                mb->mean_e[k] = (double)(long long)h_tot[k] / 65536.0 / (double)h_omega[k];
            }
    }

    // stable sort by N
    hipLaunchKernelGGL(mbar_iota_gather, dim3(grid), dim3(256), 0, s, ns, n_in.p, keys.p, idx.p);
    REGC_HIP(hipGetLastError());
    int end_bit = 1;
    while ((1 << end_bit) < mb->nN) ++end_bit;
    size_t temp_bytes = 0;
    REGC_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, temp_bytes, keys.p, keys_out.p, idx.p, idx_out.p, (int)ns, 0,
                                                end_bit, s));
    if ((rc = mb->sort_d.reserve(temp_bytes))) return rc;
    REGC_HIP(hipcub::DeviceRadixSort::SortPairs(mb->sort_d.p, temp_bytes, keys.p, keys_out.p, idx.p, idx_out.p, (int)ns, 0,
                                                end_bit, s));
    hipLaunchKernelGGL(mbar_gather_e, dim3(grid), dim3(256), 0, s, ns, idx_out.p, e_in.p, mb->e_d.p);
    REGC_HIP(hipGetLastError());

    // chunks of one N each
    std::vector<int> cn, cb, ce, c0(mb->nN), c1(mb->nN);
    int64_t pos = 0;
    for (int N = 0; N < mb->nN; ++N) {
        c0[N] = (int)cn.size();
        const int64_t cnt = (int64_t)h_seg[N];
        for (int64_t k = 0; k < cnt; k += kChunk) {
            cn.push_back(N);
            cb.push_back((int)(pos + k));
            ce.push_back((int)(pos + std::min<int64_t>(cnt, k + kChunk)));
        }
        pos += cnt;
        c1[N] = (int)cn.size();
    }
    mb->nchunks = (int)cn.size();
    if ((rc = mb->chunk_n_d.reserve(mb->nchunks)) || (rc = mb->chunk_b_d.reserve(mb->nchunks)) ||
        (rc = mb->chunk_e_d.reserve(mb->nchunks)) || (rc = mb->partial_d.reserve((size_t)mb->nchunks * mb->L)))
        return rc;
    REGC_HIP(hipMemcpyAsync(mb->chunk_n_d.p, cn.data(), sizeof(int) * cn.size(), hipMemcpyHostToDevice, s));
    REGC_HIP(hipMemcpyAsync(mb->chunk_b_d.p, cb.data(), sizeof(int) * cb.size(), hipMemcpyHostToDevice, s));
    REGC_HIP(hipMemcpyAsync(mb->chunk_e_d.p, ce.data(), sizeof(int) * ce.size(), hipMemcpyHostToDevice, s));
    REGC_HIP(hipMemcpyAsync(mb->seg_c0_d.p, c0.data(), sizeof(int) * mb->nN, hipMemcpyHostToDevice, s));
    REGC_HIP(hipMemcpyAsync(mb->seg_c1_d.p, c1.data(), sizeof(int) * mb->nN, hipMemcpyHostToDevice, s));
    mb->lnomega.assign(mb->S, -INFINITY);
    mb->gauge = -1;
    for (int k = 0; k < mb->S; ++k)
        if (h_omega[k] > 0) {
            mb->lnomega[k] = std::log((double)h_omega[k]);
            if (mb->gauge < 0) mb->gauge = k;
        }
    REGC_HIP(hipMemcpyAsync(mb->lnomega_d.p, mb->lnomega.data(), sizeof(double) * mb->S, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(mbar_range, dim3(mb->nN), dim3(kRangeThreads), 0, s, mb->e_d.p, mb->chunk_b_d.p, mb->chunk_e_d.p,
                       mb->seg_c0_d.p, mb->seg_c1_d.p, mb->mid_d.p, mb->half_d.p);
    REGC_HIP(hipGetLastError());
    std::vector<double> half(mb->nN);
    REGC_HIP(hipMemcpyAsync(half.data(), mb->half_d.p, sizeof(double) * mb->nN, hipMemcpyDeviceToHost, s));
    REGC_HIP(hipStreamSynchronize(s));
    mb->bounded = mb->tight = true;
    mb->half_max = 0.0;
    for (double h : half) {
        mb->bounded = mb->bounded && mb->beta_half * h <= kMaxSolveExponent;    // (false on a NaN)
        mb->tight = mb->tight && mb->beta_half * h <= kMaxExponent;
        mb->half_max = std::max(mb->half_max, h);
    }
    // blocks per chunk: a few per compute unit (each carries the weights of its N, about as
    // much work as 100 samples, so never below 256 samples a block)
    mb->sub = (int)std::min<int64_t>(kChunk / 256, std::max<int64_t>(1, (1024 + mb->nchunks - 1) / mb->nchunks));
    // the intermediates of a large set are given back, those of an ordinary one stay for the next
    if (ns > kKeptSamples) {
        e_in.release();
        keys.release();
        keys_out.release();
        idx.release();
        mb->sort_d.release();
    }
    mb->ns = ns;
    mb->have_samples = true;
    return REGC_OK;
}

static hipError_t launch_chunk(regc_mbar *mb, double *logd)
{
    const int L = mb->L;
    hipStream_t s = mb->stream;
#define CHUNK_CASE(LM, WT)                                                                                     \
    hipLaunchKernelGGL((mbar_chunk<LM, WT>), dim3(mb->nchunks), dim3(kMbarThreads), 0, s, L, mb->nN, mb->beta_d.p, \
                       mb->logA_d.p, mb->e_d.p, mb->chunk_n_d.p, mb->chunk_b_d.p, mb->chunk_e_d.p,               \
                       mb->partial_d.p, logd, mb->wgt_d.p)
    if (mb->weighted) {
        if (L <= 8) CHUNK_CASE(8, true);
        else if (L <= 16) CHUNK_CASE(16, true);
        else if (L <= 32) CHUNK_CASE(32, true);
        else CHUNK_CASE(64, true);
    } else {
        if (L <= 8) CHUNK_CASE(8, false);
        else if (L <= 16) CHUNK_CASE(16, false);
        else if (L <= 32) CHUNK_CASE(32, false);
        else CHUNK_CASE(64, false);
    }
#undef CHUNK_CASE
    return hipGetLastError();
}

static hipError_t mbar_iteration(regc_mbar *mb)
{
    hipStream_t s = mb->stream;
    hipLaunchKernelGGL(mbar_loga, dim3(mb->L), dim3(256), 0, s, mb->M, mb->nN, mb->lnomega_d.p, mb->f_d.p,
                       mb->lnz_d.p, mb->logA_d.p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if ((e = launch_chunk(mb, nullptr)) != hipSuccess) return e;
    hipLaunchKernelGGL(mbar_fnew, dim3(mb->L), dim3(256), sizeof(double) * mb->nN, s, mb->L, mb->M, mb->nN,
                       mb->partial_d.p, mb->seg_c0_d.p, mb->seg_c1_d.p, mb->logA_d.p, mb->lnz_d.p, mb->fnew_d.p);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(mbar_gauge, dim3(1), dim3(1024), 0, s, mb->S, mb->gauge, mb->lnomega_d.p, mb->fnew_d.p,
                       mb->f_d.p, mb->delta_d.p);
    return hipGetLastError();
}

// ---- the device-resident solve ----
// Whether the problem fits the device's iteration: energies in range of its exponents,
// states and differences within the step kernel's registers (else the general iteration,
// driven by the host).
static bool device_solve(const regc_mbar *mb)
{
    return mb->bounded && !mb->weighted && mb->S <= kMaxStepStates && (mb->method == 0 || mb->memory <= kMaxMemory);
}

static SolveArgs solve_args(regc_mbar *mb)
{
    SolveArgs p{};
    p.L = mb->L; p.M = mb->M; p.S = mb->S; p.nN = mb->nN;
    p.nchunks = mb->nchunks; p.sub = mb->sub; p.rows = mb->nchunks * mb->sub;
    p.beta_l = mb->beta_d.p; p.lnz = mb->lnz_d.p; p.beta_c = mb->beta_c;
    p.e = mb->e_d.p; p.mid = mb->mid_d.p;
    p.chunk_n = mb->chunk_n_d.p; p.chunk_b = mb->chunk_b_d.p; p.chunk_e = mb->chunk_e_d.p;
    p.seg_c0 = mb->seg_c0_d.p; p.seg_c1 = mb->seg_c1_d.p;
    p.lnomega = mb->lnomega_d.p;
    p.f = mb->f_d.p; p.fnew = mb->fnew_d.p; p.good = mb->good_d.p; p.kept = mb->kept_d.p;
    p.hist_r = mb->hist_r_d.p; p.hist_g = mb->hist_g_d.p;
    p.shift = mb->shift_d.p; p.partial = mb->q_d.p; p.st = mb->state_d.p; p.hinv = mb->hinv_d.p;
    p.arrived = mb->arrived_d.p; p.host = mb->progress;
    p.method = mb->method;
    p.polish = kPolish;
    return p;
}

// Workspace for B problems, kept with the handle and grown when a larger one is asked for.
static int solve_workspace(regc_mbar *mb, int B)
{
    int rc;
    const size_t hist = (size_t)B * (kMaxMemory + 1) * mb->S;
    if ((rc = mb->hinv_d.reserve(mb->ns)) || (rc = mb->shift_d.reserve((size_t)B * mb->nN)) || (rc = mb->q_d.reserve((size_t)B * mb->L * mb->nchunks * mb->sub)) ||
        (rc = mb->hist_r_d.reserve(hist)) || (rc = mb->hist_g_d.reserve(hist)) ||
        (rc = mb->good_d.reserve((size_t)B * mb->S)) || (rc = mb->kept_d.reserve(mb->S)) || (rc = mb->state_d.reserve(B)) || (rc = mb->arrived_d.reserve(2)))
        return rc;
    if (!mb->progress) REGC_HIP(hipHostMalloc((void **)&mb->progress, sizeof(unsigned long long), hipHostMallocDefault));
    return REGC_OK;
}

static hipError_t launch_pass(regc_mbar *mb, const SolveArgs &p, double *logd)
{
    const dim3 grid(p.rows), block(kMbarThreads);
#define PASS_CASE(J)                                                                                          \
    do {                                                                                                      \
        if (logd) hipLaunchKernelGGL((mbar_pass<J, true>), grid, block, 0, mb->stream, p, logd);              \
        else hipLaunchKernelGGL((mbar_pass<J, false>), grid, block, 0, mb->stream, p, logd);                  \
    } while (0)
    if (p.L <= 8) PASS_CASE(2);
    else if (p.L <= 16) PASS_CASE(4);
    else if (p.L <= 32) PASS_CASE(8);
    else PASS_CASE(16);
#undef PASS_CASE
    return hipGetLastError();
}

static hipError_t launch_step(regc_mbar *mb, const SolveArgs &p, int B)
{
    if (p.S <= 64) hipLaunchKernelGGL((mbar_step<64, 1>), dim3(B), dim3(64), 0, mb->stream, p);
    else if (p.S <= 256) hipLaunchKernelGGL((mbar_step<256, 1>), dim3(B), dim3(256), 0, mb->stream, p);
    else if (p.S <= 1024) hipLaunchKernelGGL((mbar_step<256, 4>), dim3(B), dim3(256), 0, mb->stream, p);
    else if (p.method == 0) hipLaunchKernelGGL((mbar_step<1024, 4>), dim3(B), dim3(1024), 0, mb->stream, p);   // (no columns)
    else if (p.S <= 2048) hipLaunchKernelGGL((mbar_step<256, 8>), dim3(B), dim3(256), 0, mb->stream, p);
    else hipLaunchKernelGGL((mbar_step<256, 16>), dim3(B), dim3(256), 0, mb->stream, p);
    return hipGetLastError();
}

// Runs iterations (enqueued by `iteration`) until every one of B problems has set its
// state's done.  The step kernel reports to host memory; the host keeps a few iterations
// enqueued ahead of the report (those past the end return at once) and never waits for
// the stream.
template <typename F>
static int run_iterations(regc_mbar *mb, int B, int max_iter, F iteration)
{
    constexpr int kAhead = 6;
    auto report = [&]() { return __atomic_load_n(mb->progress, __ATOMIC_RELAXED); };
    int sent = 0;
    for (unsigned long long now = report(); (int)(now >> 32) < B && sent < max_iter; now = report()) {
        if (sent - (int)(uint32_t)now < kAhead) {
            REGC_HIP(iteration());
            ++sent;
            continue;
        }
        // (a stream with nothing left to do while its iterations are unreported has failed)
        for (int k = 0; k < 4096 && report() == now; ++k) __builtin_ia32_pause();
        if (report() == now) {
            const hipError_t e = hipStreamQuery(mb->stream);
            if (e == hipErrorNotReady) continue;
            REGC_HIP(e);
            REGC_CHECK(report() != now, REGC_EHIP, "the reweighting iteration stopped reporting");
        }
    }
    return REGC_OK;
}

static hipError_t launch_map(regc_mbar *mb, const SolveArgs &p)
{
    hipError_t e = launch_pass(mb, p, nullptr);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mbar_fnew_q, dim3(p.L, 1), dim3(kFnewThreads), sizeof(double) * p.nN, mb->stream, p);
    return hipGetLastError();
}

// The state and the iterate of a solve's start: f (host, S values; null: what f_d holds).
static int start_solve(regc_mbar *mb, const double *f, const SolveState &st)
{
    hipStream_t s = mb->stream;
    __atomic_store_n(mb->progress, 0ull, __ATOMIC_RELAXED);
    static const unsigned int none[2] = {0u, 0u};        // (the copies may end after this function)
    if (f) {
        REGC_HIP(hipMemcpyAsync(mb->f_d.p, f, sizeof(double) * mb->S, hipMemcpyHostToDevice, s));
        REGC_HIP(hipMemcpyAsync(mb->good_d.p, f, sizeof(double) * mb->S, hipMemcpyHostToDevice, s));
    }
    REGC_HIP(hipMemcpyAsync(mb->state_d.p, &st, sizeof st, hipMemcpyHostToDevice, s));
    REGC_HIP(hipMemcpyAsync(mb->arrived_d.p, none, sizeof none, hipMemcpyHostToDevice, s));
    return REGC_OK;
}

// A first estimate of the free energies from the states' mean E and N: along a path of
// neighbouring sampled states, df = <E> d(beta) - <N> d(ln z) with the trapezoid rule.
static std::vector<double> mean_estimate(const regc_mbar *mb)
{
    std::vector<double> f(mb->S, 0.0);
    const int M = mb->M;
    auto step = [&](int a, int b) {
        return f[a] + 0.5 * (mb->mean_e[a] + mb->mean_e[b]) * (mb->beta_l[b / M] - mb->beta_l[a / M]) -
               0.5 * (mb->mean_n[a] + mb->mean_n[b]) * (mb->lnz[b] - mb->lnz[a]);
    };
    int above = -1;                  // the first sampled state of the row before
    for (int l = 0; l < mb->L; ++l) {
        int prev = -1;
        for (int m = 0; m < M; ++m) {
            const int s = l * M + m;
            if (mb->lnomega[s] == -INFINITY) continue;
            if (prev >= 0) f[s] = step(prev, s);
            else if (above >= 0) {
                // from the row before: its sampled state nearest in mu
                int best = above;
                for (int q = above; q < (above / M + 1) * M; ++q)
                    if (mb->lnomega[q] != -INFINITY && std::abs(q % M - m) < std::abs(best % M - m)) best = q;
                f[s] = step(best, s);
            }
            if (prev < 0) above = s;
            prev = s;
        }
    }
    return f;
}

// H at the iterate f_d (whose map value is in fnew_d afterwards) and its inverse.
static int factorise(regc_mbar *mb, const SolveArgs &p)
{
    hipStream_t s = mb->stream;
    const int G = p.L <= 16 ? 1 : 2, tiles = G == 1 ? 1 : 3, nK = (p.nN + 3) & ~3, n = (p.S + kGj - 1) / kGj * kGj;
    int rc;
    if ((rc = mb->cpart_d.reserve((size_t)p.rows * tiles * 256)) || (rc = mb->lw_d.reserve((size_t)p.nN * p.L)) ||
        (rc = mb->csum_d.reserve((size_t)p.L * p.L * nK)) || (rc = mb->share_d.reserve((size_t)nK * p.S)) ||
        (rc = mb->hess_d.reserve((size_t)n * n)) || (rc = mb->w_d.reserve(n)) || (rc = mb->row_d.reserve((size_t)kGj * n)) ||
        (rc = mb->col_d.reserve((size_t)kGj * n)) || (rc = mb->y_d.reserve(p.S)))
        return rc;
    if (G == 1) hipLaunchKernelGGL((mbar_pass_c<1>), dim3(p.rows), dim3(kMbarThreads), 0, s, p, mb->cpart_d.p, mb->lw_d.p);
    else hipLaunchKernelGGL((mbar_pass_c<2>), dim3(p.rows), dim3(kMbarThreads), 0, s, p, mb->cpart_d.p, mb->lw_d.p);
    hipLaunchKernelGGL(mbar_fnew_q, dim3(p.L, 1), dim3(kFnewThreads), sizeof(double) * p.nN, s, p);
    hipLaunchKernelGGL(mbar_csum, dim3(nK, 4), dim3(256), 0, s, p, nK, tiles, mb->cpart_d.p, mb->lw_d.p, mb->csum_d.p,
                       mb->share_d.p);
    if (n > p.S) hipLaunchKernelGGL(mbar_pad, dim3(n), dim3(256), 0, s, p.S, n, mb->hess_d.p);
    const int mt = (p.M + 15) / 16;
    hipLaunchKernelGGL(mbar_hess, dim3(p.L * (p.L + 1) / 2, mt, mt), dim3(64), 0, s, p, nK, n, mb->csum_d.p, mb->share_d.p,
                       mb->hess_d.p, mb->w_d.p);
    REGC_HIP(hipGetLastError());
    for (int kb = 0; kb < n / kGj; ++kb) {
        hipLaunchKernelGGL(mbar_gj_row, dim3(n / kGj), dim3(256), 0, s, n, kb, mb->hess_d.p, mb->row_d.p, mb->col_d.p);
        hipLaunchKernelGGL(mbar_gj_update, dim3(n / kGj, n / kGj), dim3(256), 0, s, n, kb, mb->hess_d.p, mb->row_d.p,
                           mb->col_d.p);
    }
    hipLaunchKernelGGL(mbar_inverse_norm, dim3(p.S), dim3(64), 0, s, p.S, n, mb->hess_d.p, mb->w_d.p, p.st);
    REGC_HIP(hipGetLastError());
    return REGC_OK;
}

static hipError_t launch_newton(regc_mbar *mb, const SolveArgs &p, int B)
{
    const int n = (p.S + kGj - 1) / kGj * kGj;
    if (B == 1) {
        hipLaunchKernelGGL(mbar_newton_one, dim3((p.S + 3) / 4), dim3(256), 0, mb->stream, p, n, mb->hess_d.p, mb->w_d.p,
                           mb->y_d.p);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(mbar_newton, dim3((p.S + 15) / 16, (B + 15) / 16), dim3(64 * kNewtonWaves), 0, mb->stream, p, B, n,
                       mb->hess_d.p, mb->w_d.p, mb->y_d.p);
    return hipGetLastError();
}

// The preconditioned solve: the plain iteration from the states' means until it is near,
// H once, then Anderson's iteration on the preconditioned map.  `solved` is left false
// (and the caller solves from f = 0) when the plain phase takes more than kNearIter
// iterations, the second more than kPreIter, both together more than max_iter, or the data
// do not determine the solution.  iters counts every evaluation of the map, H's too.
static int solve_preconditioned(regc_mbar *mb, double tol, int max_iter, int n_sampled, bool *solved, int *iters,
                                double *delta)
{
    constexpr int kNearIter = 60, kPreIter = 60;
    *solved = false;
    mb->inverse_valid = false;
    int rc;
    SolveArgs p = solve_args(mb);
    p.tol = tol;
    SolveState st{}, near{};
    st.gauge = mb->gauge;
    st.memory = std::min(mb->memory, std::max(n_sampled - 2, 0));
    st.delta = st.d_prev = st.kept = INFINITY;
    const std::vector<double> f0 = mean_estimate(mb);
    if ((rc = start_solve(mb, f0.data(), st))) return rc;
    p.tol_switch = kSwitch;
    p.max_iter = std::min(kNearIter, max_iter);
    if ((rc = run_iterations(mb, 1, p.max_iter, [&]() {
             const hipError_t e = launch_map(mb, p);
             return e != hipSuccess ? e : launch_step(mb, p, 1);
         })))
        return rc;
    REGC_HIP(hipMemcpyAsync(&near, mb->state_d.p, sizeof near, hipMemcpyDeviceToHost, mb->stream));
    REGC_HIP(hipStreamSynchronize(mb->stream));
    *iters = near.it;
    if (near.conv == 0 || near.it + 1 >= max_iter) return REGC_OK;
    if ((rc = start_solve(mb, nullptr, st)) || (rc = factorise(mb, p))) return rc;
    p.tol_switch = 0.0;
    p.max_iter = std::min(kPreIter, max_iter - near.it - 1);
    p.polish = 2;
    p.y = mb->y_d.p;
    if ((rc = run_iterations(mb, 1, p.max_iter, [&]() {
             hipError_t e = launch_map(mb, p);
             if (e == hipSuccess) e = launch_newton(mb, p, 1);
             return e != hipSuccess ? e : launch_step(mb, p, 1);
         })))
        return rc;
    REGC_HIP(hipMemcpyAsync(&st, mb->state_d.p, sizeof st, hipMemcpyDeviceToHost, mb->stream));
    REGC_HIP(hipStreamSynchronize(mb->stream));
    *solved = st.conv == 1;
    mb->inverse_valid = *solved;
    *iters = near.it + 1 + st.it;
    *delta = st.delta;
    return REGC_OK;
}

// solve_core on the device: the preconditioned solve where it applies, else (or where it
// does not settle) the iteration and the decisions of the host's.
static int solve_on_device(regc_mbar *mb, double tol, int max_iter, const double *start, int *iters, double *delta,
                           bool *lost)
{
    hipStream_t s = mb->stream;
    int rc;
    if ((rc = solve_workspace(mb, 1))) return rc;
    int n = 0;
    for (double v : mb->lnomega) n += v != -INFINITY;
    ScopedEvent e0, e1;
    REGC_HIP(e0.create());
    REGC_HIP(e1.create());
    REGC_HIP(hipEventRecord(e0.e, s));
    SolveState st{};
    bool solved = false;
    int tried = 0;                        // the iterations of an attempt given up
    if (mb->method == 1 && !start && max_iter >= kNewtonMinIter && mb->S <= kNewtonStates && mb->L <= kNewtonTemps &&
        n >= 3 && !mb->mean_n.empty()) {
        rc = solve_preconditioned(mb, tol, max_iter, n, &solved, &st.it, &st.delta);
        st.conv = 1;
        if (!solved) tried = st.it;
    }
    SolveArgs p = solve_args(mb);
    if (!rc && !solved) {
        p.max_iter = max_iter;
        p.tol = tol;
        st = SolveState{};
        st.gauge = mb->gauge;
        st.memory = std::min(mb->memory, std::max(n - 2, 0));
        st.delta = st.d_prev = st.kept = INFINITY;
        const std::vector<double> zero(start ? 0 : mb->S, 0.0);
        if (!(rc = start_solve(mb, start ? start : zero.data(), st)))
            rc = run_iterations(mb, 1, max_iter, [&]() {
                const hipError_t e = launch_map(mb, p);
                return e != hipSuccess ? e : launch_step(mb, p, 1);
            });
    }
    if (rc) {
        (void)hipStreamSynchronize(s);      // nothing writes the progress words after a failure
        return rc;
    }
    REGC_HIP(hipEventRecord(e1.e, s));
    // f_d holds g of the last iterate; log D consistent with it
    REGC_HIP(launch_pass(mb, p, mb->logd_d.p));
    mb->hinv_valid = true;
    if (!solved) REGC_HIP(hipMemcpyAsync(&st, mb->state_d.p, sizeof st, hipMemcpyDeviceToHost, s));
    REGC_HIP(hipStreamSynchronize(s));
    float ms = 0.f;
    REGC_HIP(hipEventElapsedTime(&ms, e0.e, e1.e));
    mb->ms_iter = ms;
    mb->n_iter = tried + st.it;
    if (iters) *iters = st.it;
    if (delta) *delta = st.delta;
    mb->solved = true;
    *lost = st.lost != 0;
    if (!st.conv) {
        set_error("reweighting did not converge: max |delta f| = %g after %d iterations", st.delta, st.it);
        return REGC_ENOCONV;
    }
    return REGC_OK;
}

// Least-squares coefficients gamma minimising || r - dR gamma ||_2 (dR: n x m,
// column-major) by modified Gram-Schmidt QR; columns that are numerically
// dependent on earlier ones get gamma = 0.
static void lsq_mgs(int n, int m, const std::vector<double> &dR, const std::vector<double> &r,
                    std::vector<double> &gamma)
{
    std::vector<double> Q(dR), R((size_t)m * m, 0.0), qtr(m, 0.0);
    std::vector<bool> keep(m, true);
    for (int j = 0; j < m; ++j) {
        double *qj = &Q[(size_t)j * n];
        double norm0 = 0.0;
        for (int i = 0; i < n; ++i) norm0 += qj[i] * qj[i];
        for (int k = 0; k < j; ++k) {
            if (!keep[k]) continue;
            const double *qk = &Q[(size_t)k * n];
            double d = 0.0;
            for (int i = 0; i < n; ++i) d += qk[i] * qj[i];
            R[(size_t)k * m + j] = d;
            for (int i = 0; i < n; ++i) qj[i] -= d * qk[i];
        }
        double nn = 0.0;
        for (int i = 0; i < n; ++i) nn += qj[i] * qj[i];
        if (nn <= 1e-24 * (norm0 + 1e-300)) {
            keep[j] = false;
            continue;
        }
        nn = std::sqrt(nn);
        R[(size_t)j * m + j] = nn;
        for (int i = 0; i < n; ++i) qj[i] /= nn;
        double d = 0.0;
        for (int i = 0; i < n; ++i) d += qj[i] * r[i];
        qtr[j] = d;
    }
    gamma.assign(m, 0.0);
    for (int j = m - 1; j >= 0; --j) {
        if (!keep[j]) continue;
        double v = qtr[j];
        for (int k = j + 1; k < m; ++k)
            if (keep[k]) v -= R[(size_t)j * m + k] * gamma[k];
        gamma[j] = v / R[(size_t)j * m + j];
    }
}

extern "C" int regc_mbar_set_solver(regc_mbar *mb, int method, int memory)
{
    REGC_CHECK(mb, REGC_EINVAL, "null handle");
    REGC_CHECK(method == 0 || method == 1, REGC_EINVAL, "method must be 0 (plain) or 1 (Anderson)");
    REGC_CHECK(memory >= 1 && memory <= 32, REGC_EINVAL, "memory must be 1..32");
    mb->method = method;
    mb->memory = memory;
    return REGC_OK;
}

// Fixed point f = g(f) of the self-consistent map (one device iteration = g plus the
// gauge).  Plain: f <- g(f).  Anderson acceleration (Walker & Ni, SIAM J. Numer.
// Anal. 49 (2011) 1715, type II) on the sampled states' components:
// x_{k+1} = g_k - dG gamma, gamma = argmin || r_k - dR gamma ||, r = g(x) - x, with
// at most min(memory, n - 2) differences for n sampled states (one component is
// fixed by the gauge, and more differences than free components make the least
// squares ill-posed).  A step that raises the residual tenfold restarts the history;
// a non-finite map value returns to the last finite one and takes plain steps for a
// while.  Converged when max |g(x) - x| over sampled states < tol.
// start: NULL (f = 0) or the starting iterate [S] (host).
static int solve_core(regc_mbar *mb, double tol, int max_iter, const double *start, int *iters, double *delta)
{
    mb->inverse_valid = mb->hinv_valid = false;
    if (device_solve(mb)) {
        bool lost = false;
        const int rc = solve_on_device(mb, tol, max_iter, start, iters, delta, &lost);
        // sums of exponents past kMaxExponent may have overflowed, which a map value shows; without
        // that the general iteration would come no farther (its second run took half as long
        // again: 60 iterations of 1024 states 17.7 -> 6.5 ms)
        if (mb->tight || rc != REGC_ENOCONV || !lost) return rc;
        mb->inverse_valid = mb->hinv_valid = false;
    }
    hipStream_t s = mb->stream;
    if (start) REGC_HIP(hipMemcpyAsync(mb->f_d.p, start, sizeof(double) * mb->S, hipMemcpyHostToDevice, s));
    else REGC_HIP(hipMemsetAsync(mb->f_d.p, 0, sizeof(double) * mb->S, s));
    ScopedEvent e0, e1;
    REGC_HIP(e0.create());
    REGC_HIP(e1.create());
    REGC_HIP(hipEventRecord(e0.e, s));
    std::vector<int> idx;
    for (int k = 0; k < mb->S; ++k)
        if (mb->lnomega[k] != -INFINITY) idx.push_back(k);
    const int n = (int)idx.size();
    const int m = std::min(mb->memory, std::max(n - 2, 0));
    std::vector<double> x(mb->S, 0.0), gx(mb->S), xs(n), gs(n), r(n);
    if (start) x.assign(start, start + mb->S);
    std::deque<std::vector<double>> hist_r, hist_g;   // last residuals and map values (sampled part)
    double d = INFINITY, d_prev = INFINITY;
    int it = 0, plain_left = 0;
    bool conv = false;
    std::vector<double> good(mb->S, 0.0);            // the last finite map value
    const int check = mb->method == 0 ? 10 : 1;
    for (it = 0; it < max_iter;) {
        REGC_HIP(mbar_iteration(mb));   // f_d <- gauge(map(f_d)), delta_d <- max |new - old|
        ++it;
        if (it % check != 0 && it != max_iter) continue;
        REGC_HIP(hipMemcpyAsync(&d, mb->delta_d.p, sizeof(double), hipMemcpyDeviceToHost, s));
        if (mb->method == 1) REGC_HIP(hipMemcpyAsync(gx.data(), mb->f_d.p, sizeof(double) * mb->S, hipMemcpyDeviceToHost, s));
        REGC_HIP(hipStreamSynchronize(s));
        if (!(d <= 1e300)) {                        // NaN or inf
            if (mb->method == 0 || it == 1) break;  // nothing to return to: report it
            hist_r.clear();
            hist_g.clear();
            x = good;
            plain_left = 5;
            d_prev = INFINITY;
            REGC_HIP(hipMemcpyAsync(mb->f_d.p, x.data(), sizeof(double) * mb->S, hipMemcpyHostToDevice, s));
            continue;
        }
        if (d < tol) { conv = true; break; }
        if (mb->method == 0) continue;
        good = gx;
        for (int q = 0; q < n; ++q) {
            gs[q] = gx[idx[q]];
            r[q] = gx[idx[q]] - x[idx[q]];
        }
        if (d > 10.0 * d_prev) { hist_r.clear(); hist_g.clear(); }
        d_prev = d;
        hist_r.push_back(r);
        hist_g.push_back(gs);
        if ((int)hist_r.size() > m + 1) { hist_r.pop_front(); hist_g.pop_front(); }
        const int mk = (int)hist_r.size() - 1;
        std::vector<double> xn(gx);
        if (plain_left > 0) {
            --plain_left;
        } else if (mk > 0) {
            std::vector<double> dR((size_t)n * mk), gamma;
            for (int j = 0; j < mk; ++j)
                for (int q = 0; q < n; ++q) dR[(size_t)j * n + q] = hist_r[j + 1][q] - hist_r[j][q];
            lsq_mgs(n, mk, dR, r, gamma);
            for (int q = 0; q < n; ++q) {
                double v = gs[q];
                for (int j = 0; j < mk; ++j) v -= gamma[j] * (hist_g[j + 1][q] - hist_g[j][q]);
                xn[idx[q]] = v;
            }
        }
        x = xn;
        REGC_HIP(hipMemcpyAsync(mb->f_d.p, x.data(), sizeof(double) * mb->S, hipMemcpyHostToDevice, s));
    }
    REGC_HIP(hipEventRecord(e1.e, s));
    // f_d holds g of the last iterate; log D consistent with it
    hipLaunchKernelGGL(mbar_loga, dim3(mb->L), dim3(256), 0, s, mb->M, mb->nN, mb->lnomega_d.p, mb->f_d.p,
                       mb->lnz_d.p, mb->logA_d.p);
    REGC_HIP(hipGetLastError());
    REGC_HIP(launch_chunk(mb, mb->logd_d.p));
    REGC_HIP(hipStreamSynchronize(s));
    float ms = 0.f;
    REGC_HIP(hipEventElapsedTime(&ms, e0.e, e1.e));
    mb->ms_iter = ms;
    mb->n_iter = it;
    if (iters) *iters = it;
    if (delta) *delta = d;
    mb->solved = true;
    if (!conv) {
        set_error("reweighting did not converge: max |delta f| = %g after %d iterations", d, it);
        return REGC_ENOCONV;
    }
    return REGC_OK;
}

extern "C" int regc_mbar_solve(regc_mbar *mb, double tol, int max_iter, double *f_out, int *iters, double *delta)
{
    REGC_CHECK(mb, REGC_EINVAL, "null handle");
    REGC_CHECK(mb->have_samples, REGC_ESTATE, "no samples loaded");
    REGC_CHECK(max_iter > 0 && tol > 0, REGC_EINVAL, "max_iter and tol must be positive");
    const int rc = solve_core(mb, tol, max_iter, nullptr, iters, delta);
    if (rc != REGC_OK && rc != REGC_ENOCONV) return rc;
    if (f_out) REGC_HIP(hipMemcpy(f_out, mb->f_d.p, sizeof(double) * mb->S, hipMemcpyDeviceToHost));
    return rc;
}

// Target grid constants (beta per row, ln z per target) on the device.
struct TargetDev {
    int nT = 0, nMu = 0, nK = 0;
    std::vector<double> tb;
    DevBuf<double> tb_d, tz_d;
};

static int target_grid(regc_mbar *mb, const regc_grid *targets, TargetDev &T)
{
    T.nT = targets->n_t;
    T.nMu = targets->n_mu;
    T.nK = T.nT * T.nMu;
    REGC_CHECK(T.nT > 0 && T.nMu > 0, REGC_EINVAL, "empty target grid");
    std::vector<double> &tb = T.tb, tz(T.nK);
    tb.resize(T.nT);
    for (int l = 0; l < T.nT; ++l) {
        REGC_CHECK(targets->t[l] > 0, REGC_EINVAL, "target temperatures must be positive");
        tb[l] = 1.0 / targets->t[l];
        for (int m = 0; m < T.nMu; ++m) tz[l * T.nMu + m] = lnz_of(targets->t[l], targets->mu[m], mb->lambda1);
    }
    int rc;
    if ((rc = T.tb_d.alloc(T.nT)) || (rc = T.tz_d.alloc(T.nK))) return rc;
    REGC_HIP(hipMemcpyAsync(T.tb_d.p, tb.data(), sizeof(double) * T.nT, hipMemcpyHostToDevice, mb->stream));
    REGC_HIP(hipMemcpyAsync(T.tz_d.p, tz.data(), sizeof(double) * T.nK, hipMemcpyHostToDevice, mb->stream));
    return REGC_OK;
}

// Whether exponents around the samples' energies stay bounded at inverse temperatures tb.
static bool bounded_targets(const regc_mbar *mb, const double *tb, int nT)
{
    double far = 0.0;
    for (int t = 0; t < nT; ++t) far = std::max(far, std::fabs(tb[t] - mb->beta_c));
    return mb->tight && far * mb->half_max <= kMaxExponent;
}

// The chunks' sums and the averages at the targets on the handle's stream: on bounded
// exponents where the solution and the targets allow, else with a running maximum.  part:
// [nchunks][nT][4]; tb: the targets' inverse temperatures (host), tb_d, tz_d (device).
static hipError_t launch_targets(regc_mbar *mb, int nT, int nMu, const double *tb, const double *tb_d, const double *tz_d,
                                 double *part, double *f, double *mn, double *me, double *me2, double *pn, int32_t *ph)
{
    hipStream_t s = mb->stream;
    const size_t lds = sizeof(double) * 3 * mb->nN;
    if (mb->hinv_valid && !mb->weighted && nT <= 1 << 20 && bounded_targets(mb, tb, nT)) {
        const SolveArgs p = solve_args(mb);
        if (nT <= 8)
            hipLaunchKernelGGL((mbar_target_pass<2>), dim3(mb->nchunks, 1), dim3(kMbarThreads), 0, s, p, nT, tb_d, part);
        else if (nT <= 16)
            hipLaunchKernelGGL((mbar_target_pass<4>), dim3(mb->nchunks, 1), dim3(kMbarThreads), 0, s, p, nT, tb_d, part);
        else
            hipLaunchKernelGGL((mbar_target_pass<8>), dim3(mb->nchunks, (nT + 31) / 32), dim3(kMbarThreads), 0, s, p, nT,
                               tb_d, part);
        hipLaunchKernelGGL(mbar_target_eval_q, dim3(nT, std::min((nMu + kEvalMu - 1) / kEvalMu, 4096)), dim3(kEvalThreads), lds,
                           s, p, nT, nMu, tb_d, part, tz_d, f, mn, me, me2, pn, ph);
    } else {
        hipLaunchKernelGGL(mbar_target_chunk, dim3(mb->nchunks), dim3(kMbarThreads), 0, s, nT, tb_d, mb->e_d.p,
                           mb->logd_d.p, mb->chunk_b_d.p, mb->chunk_e_d.p, part, mb->weighted ? mb->wgt_d.p : nullptr);
        hipLaunchKernelGGL(mbar_target_eval, dim3(nT), dim3(256), lds, s, nT, nMu, mb->nN, part, mb->seg_c0_d.p,
                           mb->seg_c1_d.p, tz_d, f, mn, me, me2, pn, ph);
    }
    return hipGetLastError();
}

// Reweighted averages at the targets into device arrays (any may be NULL but mn).
static int targets_dev(regc_mbar *mb, const TargetDev &T, double *f, double *mn, double *me, double *me2,
                       double *pn, int32_t *ph)
{
    hipStream_t s = mb->stream;
    DevBuf<double> tpart;
    int rc;
    if ((rc = tpart.alloc((size_t)mb->nchunks * T.nT * 4))) return rc;
    REGC_HIP(launch_targets(mb, T.nT, T.nMu, T.tb.data(), T.tb_d.p, T.tz_d.p, tpart.p, f, mn, me, me2, pn, ph));
    REGC_HIP(hipStreamSynchronize(s));     // tpart is freed on return
    return REGC_OK;
}

extern "C" int regc_mbar_targets(regc_mbar *mb, const regc_grid *targets, double *f, double *mean_n,
                                 double *mean_e, double *mean_e2, double *p_n, int32_t *phase)
{
    REGC_CHECK(mb && targets && mean_n && targets->t && targets->mu, REGC_EINVAL, "null argument");
    REGC_CHECK(mb->solved, REGC_ESTATE, "solve first");
    TargetDev T;
    int rc;
    if ((rc = target_grid(mb, targets, T))) return rc;
    const int nK = T.nK;
    DevBuf<double> f_d, mn_d, me_d, me2_d, pn_d;
    DevBuf<int32_t> ph_d;
    if ((rc = f_d.alloc(nK)) || (rc = mn_d.alloc(nK)) || (rc = me_d.alloc(nK)) || (rc = me2_d.alloc(nK)) ||
        (rc = ph_d.alloc(nK)) || (rc = pn_d.alloc(p_n ? (size_t)nK * mb->nN : 1)))
        return rc;
    if ((rc = targets_dev(mb, T, f_d.p, mn_d.p, me_d.p, me2_d.p, p_n ? pn_d.p : nullptr, ph_d.p))) return rc;
    if (f) REGC_HIP(hipMemcpy(f, f_d.p, sizeof(double) * nK, hipMemcpyDeviceToHost));
    REGC_HIP(hipMemcpy(mean_n, mn_d.p, sizeof(double) * nK, hipMemcpyDeviceToHost));
    if (mean_e) REGC_HIP(hipMemcpy(mean_e, me_d.p, sizeof(double) * nK, hipMemcpyDeviceToHost));
    if (mean_e2) REGC_HIP(hipMemcpy(mean_e2, me2_d.p, sizeof(double) * nK, hipMemcpyDeviceToHost));
    if (phase) REGC_HIP(hipMemcpy(phase, ph_d.p, sizeof(int32_t) * nK, hipMemcpyDeviceToHost));
    if (p_n) REGC_HIP(hipMemcpy(p_n, pn_d.p, sizeof(double) * nK * mb->nN, hipMemcpyDeviceToHost));
    return REGC_OK;
}

// ---- reweighted averages without allocation ----
// Device scratch of regc_mbar_targets_static: the target constants, the per-chunk
// partial sums and the outputs before their copy to the host.  Every GPU the library
// runs on holds its own copy for the life of the process; host code reaches it only
// through the address hipGetSymbolAddress returns on that device.
constexpr size_t kStaticScratchDoubles = (size_t)1 << 19;     // 4 MiB
constexpr int kStaticMaxT = 1024, kStaticMaxK = 4096;
constexpr int kStaticMaxDevices = 64;
static __device__ __align__(256) double scratch[kStaticScratchDoubles];
static std::mutex g_static_mu;
static double *g_static_ptr[kStaticMaxDevices];

// The current device's scratch address (looked up once per device, with it current).
static int static_scratch(double **out)
{
    int dev = -1;
    REGC_HIP(hipGetDevice(&dev));
    REGC_CHECK(dev >= 0 && dev < kStaticMaxDevices, REGC_EINVAL, "device %d beyond the static scratch table", dev);
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[dev]) {
        void *p = nullptr;
        REGC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        REGC_CHECK(p != nullptr, REGC_EINVAL, "no address for the static scratch on device %d", dev);
        g_static_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_static_ptr[dev];
    return REGC_OK;
}

extern "C" int regc_mbar_targets_static(regc_mbar *mb, const regc_grid *targets, double *f, double *mean_n,
                                        double *mean_e, double *mean_e2, int32_t *phase)
{
    REGC_CHECK(mb && targets && mean_n && targets->t && targets->mu, REGC_EINVAL, "null argument");
    REGC_CHECK(mb->solved, REGC_ESTATE, "solve first");
    const int nT = targets->n_t, nMu = targets->n_mu;
    REGC_CHECK(nT > 0 && nMu > 0, REGC_EINVAL, "empty target grid");
    REGC_CHECK(nT <= kStaticMaxT && (int64_t)nT * nMu <= kStaticMaxK, REGC_EINVAL,
               "target grid %d x %d beyond the static limits (%d temperatures, %d targets)", nT, nMu, kStaticMaxT,
               kStaticMaxK);
    const int nK = nT * nMu;
    // scratch: tb [nT] | tz [nK] | partials [nchunks][nT][4] | f, mean_n, mean_e, mean_e2, phase [nK] each
    const size_t need = (size_t)nT + (size_t)nK + (size_t)mb->nchunks * nT * 4 + (size_t)5 * nK;
    REGC_CHECK(need <= kStaticScratchDoubles, REGC_EINVAL,
               "%zu doubles of scratch needed (%d sample chunks x %d temperatures), %zu available", need,
               mb->nchunks, nT, kStaticScratchDoubles);
    double tb[kStaticMaxT], tz[kStaticMaxK];
    for (int l = 0; l < nT; ++l) {
        REGC_CHECK(targets->t[l] > 0, REGC_EINVAL, "target temperatures must be positive");
        tb[l] = 1.0 / targets->t[l];
        for (int m = 0; m < nMu; ++m) tz[l * nMu + m] = lnz_of(targets->t[l], targets->mu[m], mb->lambda1);
    }
    double *sp = nullptr;
    int rc;
    if ((rc = static_scratch(&sp))) return rc;
    double *tb_d = sp, *tz_d = tb_d + nT, *part = tz_d + nK, *f_d = part + (size_t)mb->nchunks * nT * 4;
    double *mn_d = f_d + nK, *me_d = mn_d + nK, *me2_d = me_d + nK;
    int32_t *ph_d = reinterpret_cast<int32_t *>(me2_d + nK);
    hipStream_t s = mb->stream;
    REGC_HIP(hipMemcpyAsync(tb_d, tb, sizeof(double) * nT, hipMemcpyHostToDevice, s));
    REGC_HIP(hipMemcpyAsync(tz_d, tz, sizeof(double) * nK, hipMemcpyHostToDevice, s));
    // every partial and output entry read below is written by these two kernels
    REGC_HIP(launch_targets(mb, nT, nMu, tb, tb_d, tz_d, part, f_d, mn_d, me_d, me2_d, nullptr, ph_d));
    if (f) REGC_HIP(hipMemcpyAsync(f, f_d, sizeof(double) * nK, hipMemcpyDeviceToHost, s));
    REGC_HIP(hipMemcpyAsync(mean_n, mn_d, sizeof(double) * nK, hipMemcpyDeviceToHost, s));
    if (mean_e) REGC_HIP(hipMemcpyAsync(mean_e, me_d, sizeof(double) * nK, hipMemcpyDeviceToHost, s));
    if (mean_e2) REGC_HIP(hipMemcpyAsync(mean_e2, me2_d, sizeof(double) * nK, hipMemcpyDeviceToHost, s));
    if (phase) REGC_HIP(hipMemcpyAsync(phase, ph_d, sizeof(int32_t) * nK, hipMemcpyDeviceToHost, s));
    REGC_HIP(hipStreamSynchronize(s));     // the stack copies of tb, tz live until here
    return REGC_OK;
}

extern "C" int regc_mbar_set_observables(regc_mbar *mb, const uint32_t *obs, int n_obs, int on_device)
{
    REGC_CHECK(mb && obs, REGC_EINVAL, "null argument");
    REGC_CHECK(mb->have_samples, REGC_ESTATE, "set the samples first");
    REGC_CHECK(n_obs > 0 && n_obs <= 4096, REGC_EINVAL, "n_obs must be 1..4096");
    mb->n_obs = 0;     // no observables until this call succeeds
    hipStream_t s = mb->stream;
    const size_t count = (size_t)mb->ns * n_obs;
    DevBuf<uint32_t> in;
    int rc;
    if ((rc = in.alloc(count)) || (rc = mb->obs_d.alloc(count))) return rc;
    REGC_HIP(hipMemcpyAsync(in.p, obs, sizeof(uint32_t) * count,
                            on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, s));
    const int grid = (int)std::min<size_t>((count + 255) / 256, 8192);
    hipLaunchKernelGGL(mbar_gather_obs, dim3(grid), dim3(256), 0, s, (int64_t)mb->ns, n_obs, mb->perm_d.p, in.p,
                       mb->obs_d.p);
    REGC_HIP(hipGetLastError());
    REGC_HIP(hipStreamSynchronize(s));
    mb->n_obs = n_obs;
    return REGC_OK;
}

extern "C" int regc_mbar_observables(regc_mbar *mb, const regc_grid *targets, double *mean, double *cond)
{
    REGC_CHECK(mb && targets && targets->t && targets->mu, REGC_EINVAL, "null argument");
    REGC_CHECK(mb->solved, REGC_ESTATE, "solve first");
    REGC_CHECK(mb->n_obs > 0, REGC_ESTATE, "no observables loaded");
    REGC_CHECK(!mb->weighted, REGC_ESTATE, "a bootstrap is in progress");
    const int nT = targets->n_t, nMu = targets->n_mu, nK = nT * nMu, no = mb->n_obs;
    REGC_CHECK(nT > 0 && nMu > 0, REGC_EINVAL, "empty target grid");
    std::vector<double> tb(nT), tz(nK);
    for (int l = 0; l < nT; ++l) {
        REGC_CHECK(targets->t[l] > 0, REGC_EINVAL, "target temperatures must be positive");
        tb[l] = 1.0 / targets->t[l];
        for (int m = 0; m < nMu; ++m) tz[l * nMu + m] = lnz_of(targets->t[l], targets->mu[m], mb->lambda1);
    }
    hipStream_t s = mb->stream;
    const bool fast = mb->hinv_valid && bounded_targets(mb, tb.data(), nT);
    SolveArgs p{};
    if (fast) {
        p = solve_args(mb);
        // parts of chunks while they hold some 16 samples and their sums stay below 64 MiB (an
        // allocation above 2 MB costs 25 us: 200 samples, 300 observables, 20 temperatures in 8 parts
        // 147 us instead of 127)
        p.sub = (int)std::min<int64_t>(p.sub, std::max<int64_t>(1, mb->ns / ((int64_t)mb->nchunks * 16)));
        const size_t row = sizeof(double) * (size_t)nT * (no + 1) * p.nchunks;
        p.sub = (int)std::min<size_t>(p.sub, std::max<size_t>(1, ((size_t)64 << 20) / row));
        p.rows = p.nchunks * p.sub;
    }
    DevBuf<double> tb_d, tz_d, part, cond_d, mean_d, g_d;
    int rc;
    if ((rc = tb_d.alloc(nT)) || (rc = tz_d.alloc(nK)) ||
        (rc = part.alloc(fast ? (size_t)p.rows * nT * (no + 1) : (size_t)mb->nchunks * nT * (no + 2))) ||
        (rc = cond_d.alloc((size_t)nT * mb->nN * no)) || (rc = mean_d.alloc(mean ? (size_t)nK * no : 1)) ||
        (rc = g_d.alloc((size_t)nT * mb->nN)))
        return rc;
    REGC_HIP(hipMemcpyAsync(tb_d.p, tb.data(), sizeof(double) * nT, hipMemcpyHostToDevice, s));
    REGC_HIP(hipMemcpyAsync(tz_d.p, tz.data(), sizeof(double) * nK, hipMemcpyHostToDevice, s));
    if (fast) {
        const int cols = 64 * (kMbarThreads / 64);        // columns per block
        hipLaunchKernelGGL(mbar_obs_pass, dim3(p.rows, (no + cols) / cols, (nT + 15) / 16), dim3(kMbarThreads), 0, s, p, nT,
                           no, tb_d.p, mb->obs_d.p, part.p);
        hipLaunchKernelGGL(mbar_obs_cond, dim3(mb->nN, nT), dim3(256), 0, s, p, nT, no, tb_d.p, part.p, cond_d.p, g_d.p);
        if (mean)
            hipLaunchKernelGGL(mbar_obs_mean, dim3(nMu, nT), dim3(256), sizeof(double) * mb->nN, s, nMu, mb->nN, no, g_d.p,
                               tz_d.p, cond_d.p, mean_d.p);
    } else {
        hipLaunchKernelGGL(mbar_obs_chunk, dim3(mb->nchunks, nT), dim3(kMbarThreads), 0, s, nT, no, tb_d.p, mb->e_d.p,
                           mb->logd_d.p, mb->chunk_b_d.p, mb->chunk_e_d.p, mb->obs_d.p, part.p);
        hipLaunchKernelGGL(mbar_obs_eval, dim3(nT), dim3(256), 2 * sizeof(double) * mb->nN, s, nT, nMu, mb->nN, no,
                           part.p, mb->seg_c0_d.p, mb->seg_c1_d.p, tz_d.p, cond_d.p, mean ? mean_d.p : nullptr);
    }
    REGC_HIP(hipGetLastError());
    REGC_HIP(hipStreamSynchronize(s));
    if (cond) REGC_HIP(hipMemcpy(cond, cond_d.p, sizeof(double) * (size_t)nT * mb->nN * no, hipMemcpyDeviceToHost));
    if (mean) REGC_HIP(hipMemcpy(mean, mean_d.p, sizeof(double) * (size_t)nK * no, hipMemcpyDeviceToHost));
    return REGC_OK;
}

extern "C" int regc_mbar_timing(regc_mbar *mb, double *ms_iter_total, int64_t *n_iter)
{
    REGC_CHECK(mb, REGC_EINVAL, "null handle");
    if (ms_iter_total) *ms_iter_total = mb->ms_iter;
    if (n_iter) *n_iter = mb->n_iter;
    return REGC_OK;
}

extern "C" void regc_mbar_destroy(regc_mbar *mb) { delete mb; }

// ---------------------------------------------------------------------------
// The batch's workspace: replicates of a batch and target temperatures of a pass over them,
// such that it stays below kBootBytes (a chunk's partial sums are 8 max(L, 3 temperatures)
// bytes per replicate, so that 1e8 samples would take 8 GB for 64 temperatures at once).
// Fewer temperatures at once cost little (a pass reads the samples for 16 of them either way),
// fewer replicates cost whole solves: those go last.  The workspace stays with the handle up to
// kBootKept, which holds it for 1e6 samples and 64 temperatures.
constexpr size_t kBootBytes = (size_t)1 << 30, kBootKept = (size_t)256 << 20;

struct BootPlan {
    int batch = 0, temps = 0;        // multiples of 16; batch 0: nothing fits
    int sub = 1, rows = 0, outs = 0;
    size_t bytes = 0;
};

static BootPlan boot_plan(const regc_mbar *mb, int64_t R, int B, int nT)
{
    BootPlan q;
    // blocks of a pass are a part of a chunk and a group of columns
    q.sub = (int)std::min<int64_t>(kChunk / 256, std::max<int64_t>(1, (512 + mb->nchunks - 1) / mb->nchunks));
    q.rows = mb->nchunks * q.sub;
    const double fixed = (double)R * 4 + 8.0 * mb->nN * mb->L + mb->S * (4.0 + 8.0 * (6 + 2 * (kMaxMemory + 1)));
    for (int batch = std::min(kBootMax, (B + 15) & ~15); batch > 0; batch -= 16)
        for (int temps = (nT + 15) & ~15; temps > 0; temps = temps > 16 ? std::max(16, temps / 2 & ~15) : 0) {
            const int outs = std::max(mb->L, 3 * std::min(temps, nT));
            const double bytes = batch * (fixed + 8.0 * outs * ((double)q.rows + mb->nN));
            if (bytes > (double)kBootBytes) continue;
            q.batch = batch;
            q.temps = temps;
            q.outs = outs;
            q.bytes = (size_t)bytes;
            return q;
        }
    return q;
}

static void release_boot(regc_mbar *mb)
{
    mb->b_rec_d.release(); mb->b_mult_d.release(); mb->b_omega_d.release();
    mb->b_lnomega_d.release(); mb->b_f_d.release(); mb->b_fnew_d.release(); mb->b_good_d.release();
    mb->b_hr_d.release(); mb->b_hg_d.release(); mb->b_shift_d.release();
    mb->b_a_d.release(); mb->b_part_d.release(); mb->b_sum_d.release(); mb->b_state_d.release();
}

// All bootstrap replicates b0 .. b0 + B - 1 together: their solutions from the full one
// (f_d) by Anderson's iteration preconditioned with the full data's inverse Jacobian, then
// <N> and the heat capacity at the targets into rep_n, rep_c [B][targets] (device).  `ok`
// is left false where a replicate does not settle, or where memory for them lacks.
static int bootstrap_batch(regc_mbar *mb, const BootPlan &plan, const TargetDev &T, double tol, int64_t R, int64_t rs,
                           int64_t blk, uint64_t seed, int b0, int B, double *rep_n, double *rep_c, bool *ok)
{
    constexpr int kBootIter = 80;
    *ok = false;
    hipStream_t s = mb->stream;
    const int Bp = (B + 15) & ~15, S = mb->S, L = mb->L, outs = plan.outs;
    BootArgs g{};
    g.B = B;
    g.Bp = Bp;
    SolveArgs &p = g.p;
    p = solve_args(mb);
    p.polish = 0;                 // (a replicate's spread is what is asked for; and kept stays unused)
    p.sub = plan.sub;
    p.rows = plan.rows;
    int rc;
    const size_t hist = (size_t)B * (kMaxMemory + 1) * S;
    if ((rc = mb->b_rec_d.reserve(mb->ns)) || (rc = mb->b_mult_d.reserve((size_t)R * Bp)) ||
        (rc = mb->b_omega_d.reserve((size_t)S * Bp)) || (rc = mb->b_lnomega_d.reserve((size_t)B * S)) ||
        (rc = mb->b_f_d.reserve((size_t)B * S)) || (rc = mb->b_fnew_d.reserve((size_t)B * S)) ||
        (rc = mb->b_good_d.reserve((size_t)B * S)) || (rc = mb->b_hr_d.reserve(hist)) || (rc = mb->b_hg_d.reserve(hist)) ||
        (rc = mb->b_shift_d.reserve((size_t)B * mb->nN)) || (rc = mb->b_a_d.reserve((size_t)mb->nN * L * Bp)) ||
        (rc = mb->b_part_d.reserve((size_t)p.rows * outs * Bp)) || (rc = mb->b_sum_d.reserve((size_t)mb->nN * outs * Bp)) ||
        (rc = mb->b_state_d.reserve(B)) || (rc = mb->y_d.reserve((size_t)B * S))) {
        (void)hipGetLastError();
        release_boot(mb);
        return rc == REGC_ENOMEM ? REGC_OK : rc;
    }
    p.lnomega = mb->b_lnomega_d.p;
    p.f = mb->b_f_d.p; p.fnew = mb->b_fnew_d.p; p.good = mb->b_good_d.p;
    p.hist_r = mb->b_hr_d.p; p.hist_g = mb->b_hg_d.p;
    p.shift = mb->b_shift_d.p; p.st = mb->b_state_d.p;
    p.y = mb->y_d.p;
    p.tol = tol;
    p.max_iter = kBootIter;
    g.rec = mb->b_rec_d.p; g.mult = mb->b_mult_d.p; g.a = mb->b_a_d.p; g.part = mb->b_part_d.p; g.sum = mb->b_sum_d.p;
    const int grid = (int)std::min<int64_t>((mb->ns + 255) / 256, 4096);
    hipLaunchKernelGGL(fill_i32, dim3((unsigned)std::min<int64_t>((R * Bp + 255) / 256, 4096)), dim3(256), 0, s, R * Bp, 0,
                       mb->b_mult_d.p);
    hipLaunchKernelGGL(fill_i32, dim3((unsigned)((S * Bp + 255) / 256)), dim3(256), 0, s, (int64_t)S * Bp, 0,
                       (int32_t *)mb->b_omega_d.p);
    hipLaunchKernelGGL(boot_mult_all, dim3((unsigned)std::min<int64_t>((R + 255) / 256, 1024), B), dim3(256), 0, s, R, blk, b0,
                       Bp, (uint32_t)seed, (uint32_t)(seed >> 32), mb->b_mult_d.p);
    hipLaunchKernelGGL(boot_records, dim3(grid), dim3(256), 0, s, mb->ns, rs, mb->perm_d.p, mb->b_rec_d.p);
    hipLaunchKernelGGL(boot_omega, dim3(2048), dim3(256), 0, s, mb->ns, rs, mb->s_orig_d.p, mb->b_mult_d.p, Bp,
                       mb->b_omega_d.p);
    hipLaunchKernelGGL(boot_start, dim3(B), dim3(256), 0, s, S, Bp, mb->memory, mb->b_omega_d.p, mb->f_d.p,
                       mb->b_lnomega_d.p, mb->b_f_d.p, mb->b_good_d.p, mb->b_state_d.p);
    hipLaunchKernelGGL(fill_u64, dim3(1), dim3(64), 0, s, (int64_t)1, (unsigned long long *)mb->arrived_d.p);
    REGC_HIP(hipGetLastError());
    __atomic_store_n(mb->progress, 0ull, __ATOMIC_RELAXED);
    const dim3 pass_grid(p.rows, (Bp + kBootTiles * 16 - 1) / (kBootTiles * 16));
    const size_t pass_lds = sizeof(double) * 48 * kBootTiles * 16;
    rc = run_iterations(mb, B, kBootIter, [&]() {
        hipLaunchKernelGGL(boot_weights_log, dim3(p.nN, B), dim3(kMbarThreads), 0, s, g, 0);
        hipLaunchKernelGGL((boot_pass<false>), pass_grid, dim3(kMbarThreads), pass_lds, s, g, (const double *)nullptr, 0);
        hipLaunchKernelGGL(boot_sum, dim3(p.nN, 8), dim3(256), 0, s, g, L);
        hipLaunchKernelGGL(boot_fnew, dim3(L, Bp / 16), dim3(kFnewThreads), sizeof(double) * 16 * p.nN, s, g);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = launch_newton(mb, p, B);
        return e != hipSuccess ? e : launch_step(mb, p, B);
    });
    if (rc) return rc;
    std::vector<SolveState> st(B);
    REGC_HIP(hipMemcpyAsync(st.data(), mb->b_state_d.p, sizeof(SolveState) * B, hipMemcpyDeviceToHost, s));
    REGC_HIP(hipStreamSynchronize(s));
    for (const SolveState &x : st)
        if (x.conv != 1) return REGC_OK;
    // the averages at the targets, on the solutions' weights
    hipLaunchKernelGGL(boot_weights_log, dim3(p.nN, B), dim3(kMbarThreads), 0, s, g, 1);
    for (int t0 = 0; t0 < T.nT; t0 += plan.temps) {
        const int nt = std::min(plan.temps, T.nT - t0), k0 = t0 * T.nMu;
        hipLaunchKernelGGL((boot_pass<true>), dim3(pass_grid.x, pass_grid.y, (nt + 15) / 16), dim3(kMbarThreads), pass_lds, s,
                           g, T.tb_d.p + t0, nt);
        hipLaunchKernelGGL(boot_sum, dim3(p.nN, 8), dim3(256), 0, s, g, 3 * nt);
        hipLaunchKernelGGL(boot_target_eval, dim3(nt, B), dim3(256), sizeof(double) * 3 * p.nN, s, g, nt, T.nMu, T.nK,
                           T.tb_d.p + t0, T.tz_d.p + k0, rep_n + k0, rep_c + k0);
    }
    REGC_HIP(hipGetLastError());
    *ok = true;
    return REGC_OK;
}

// Estimates with their errors: the solve, the averages at the targets, batch means
// at the sampled states and a moving-block bootstrap over records (re-solving with
// the records' multiplicities as sample weights, warm-started from the full solve).
extern "C" void regc_default_reweight_opts(regc_reweight_opts *o)
{
    if (!o) return;
    o->n_batches = 20;
    o->n_boot = 100;
    o->record_size = 0;
    o->block_records = 0;
    o->seed = 1;
    o->n_sites = 0.0;
}

// Sets the handle's state counts (and gauge) from a device array of counts.
static int set_omega(regc_mbar *mb, const unsigned long long *omega_d)
{
    std::vector<unsigned long long> h(mb->S);
    REGC_HIP(hipMemcpyAsync(h.data(), omega_d, sizeof(unsigned long long) * mb->S, hipMemcpyDeviceToHost, mb->stream));
    REGC_HIP(hipStreamSynchronize(mb->stream));
    mb->lnomega.assign(mb->S, -INFINITY);
    mb->gauge = -1;
    for (int k = 0; k < mb->S; ++k)
        if (h[k] > 0) {
            mb->lnomega[k] = std::log((double)h[k]);
            if (mb->gauge < 0) mb->gauge = k;
        }
    REGC_HIP(hipMemcpyAsync(mb->lnomega_d.p, mb->lnomega.data(), sizeof(double) * mb->S, hipMemcpyHostToDevice,
                            mb->stream));
    return REGC_OK;
}

// log D of the current f (after changing the weights or restoring f)
static int refresh_logd(regc_mbar *mb)
{
    hipLaunchKernelGGL(mbar_loga, dim3(mb->L), dim3(256), 0, mb->stream, mb->M, mb->nN, mb->lnomega_d.p, mb->f_d.p,
                       mb->lnz_d.p, mb->logA_d.p);
    REGC_HIP(hipGetLastError());
    REGC_HIP(launch_chunk(mb, mb->logd_d.p));
    return REGC_OK;
}

// Per-state mean of N and its batch-means SE of ns samples (state, n) in the order
// given, device arrays; outputs host arrays [S].  EINVAL on a state outside 0..S-1
// or a negative N.
static int batch_means_sorted(hipStream_t s, int64_t ns, const int32_t *st_d, const int32_t *n_d, int S, int B, double *mean,
                              double *se)
{
    DevBuf<uint32_t> keys, keys_out;
    DevBuf<int32_t> idx, idx_out;
    DevBuf<int64_t> start_d, count_d;
    DevBuf<unsigned long long> bsum;
    DevBuf<double> out_d;
    DevBuf<int> bad;
    int rc;
    if ((rc = keys.alloc(ns)) || (rc = keys_out.alloc(ns)) || (rc = idx.alloc(ns)) || (rc = idx_out.alloc(ns)) ||
        (rc = start_d.alloc(S)) || (rc = count_d.alloc(S)) || (rc = bsum.alloc((size_t)S * B)) ||
        (rc = out_d.alloc(2 * (size_t)S)) || (rc = bad.alloc(1)))
        return rc;
    const int grid = (int)std::min<int64_t>((ns + 255) / 256, 4096);
    // the inputs are checked before they are used as sort keys
    int h_bad = 0;
    hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, (int64_t)1, 0, bad.p);
    hipLaunchKernelGGL(bm_check, dim3(grid), dim3(256), 0, s, ns, st_d, n_d, S, bad.p);
    REGC_HIP(hipGetLastError());
    REGC_HIP(hipMemcpyAsync(&h_bad, bad.p, sizeof(int), hipMemcpyDeviceToHost, s));
    REGC_HIP(hipStreamSynchronize(s));
    REGC_CHECK(!h_bad, REGC_EINVAL, "a sample's state is outside 0..%d or its N is negative", S - 1);
    // stable sort of the sample indices by state: each state's series in sample order
    hipLaunchKernelGGL(mbar_iota_gather, dim3(grid), dim3(256), 0, s, ns, st_d, keys.p, idx.p);
    REGC_HIP(hipGetLastError());
    int end_bit = 1;
    while ((1 << end_bit) < S) ++end_bit;
    size_t temp_bytes = 0;
    REGC_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, temp_bytes, keys.p, keys_out.p, idx.p, idx_out.p, (int)ns, 0,
                                                end_bit, s));
    DevBuf<unsigned char> temp;
    if ((rc = temp.alloc(temp_bytes))) return rc;
    REGC_HIP(hipcub::DeviceRadixSort::SortPairs(temp.p, temp_bytes, keys.p, keys_out.p, idx.p, idx_out.p, (int)ns, 0,
                                                end_bit, s));
    hipLaunchKernelGGL(bm_bounds, dim3((S + 255) / 256), dim3(256), 0, s, ns, S, keys_out.p, start_d.p, count_d.p);
    REGC_HIP(hipGetLastError());
    hipLaunchKernelGGL(bm_segments, dim3(S * B), dim3(256), 0, s, B, idx_out.p, n_d, start_d.p, count_d.p, bsum.p);
    REGC_HIP(hipGetLastError());
    hipLaunchKernelGGL(bm_finish_sorted, dim3((S + 3) / 4), dim3(256), 0, s, S, B, bsum.p, count_d.p, out_d.p, out_d.p + S);
    REGC_HIP(hipGetLastError());
    REGC_HIP(hipStreamSynchronize(s));
    REGC_HIP(hipMemcpy(mean, out_d.p, sizeof(double) * S, hipMemcpyDeviceToHost));
    REGC_HIP(hipMemcpy(se, out_d.p + S, sizeof(double) * S, hipMemcpyDeviceToHost));
    return REGC_OK;
}

static int batch_means_dev(hipStream_t s, int64_t ns, const int32_t *st_d, const int32_t *n_d, int S, int B, double *mean,
                           double *se)
{
    int rc;
    // waves per block: as many as there is LDS for
    constexpr size_t kLds = (size_t)64 << 10;
    const int W = bm_bytes(S, 8) <= kLds ? 8 : bm_bytes(S, 2) <= kLds ? 2 : 0;
    if (!W) {
        return batch_means_sorted(s, ns, st_d, n_d, S, B, mean, se);
    } else {
        BmArgs p{};
        p.ns = ns; p.st = st_d; p.n = n_d; p.S = S; p.B = B;
        p.blocks = (int)std::min<int64_t>((ns + 255) / 256, kBmBlocks);
        // one allocation: batch sums | mean, se, the flag | first ranks | counts | the blocks' flags
        DevBuf<unsigned long long> work;
        const size_t bins = (size_t)S * B;
        if ((rc = work.alloc(bins + 2 * (size_t)S + 1 + ((size_t)(p.blocks + 1) * S + p.blocks + 1) / 2))) return rc;
        p.sum = work.p;
        p.mean = reinterpret_cast<double *>(work.p + bins);
        p.se = p.mean + S;
        p.any_bad = reinterpret_cast<int *>(p.se + S);
        p.hist = reinterpret_cast<uint32_t *>(p.se + S + 1);
        p.count = p.hist + (size_t)p.blocks * S;
        p.bad = reinterpret_cast<int *>(p.count + S);
        hipLaunchKernelGGL(bm_count, dim3(p.blocks), dim3(kBmThreads), sizeof(uint32_t) * S, s, p);
        hipLaunchKernelGGL(bm_scan, dim3((S + 63) / 64), dim3(1024), 0, s, p);
        if (W == 8) hipLaunchKernelGGL((bm_sum<8>), dim3(p.blocks), dim3(512), bm_bytes(S, 8), s, p);
        else hipLaunchKernelGGL((bm_sum<2>), dim3(p.blocks), dim3(128), bm_bytes(S, 2), s, p);
        hipLaunchKernelGGL(bm_finish, dim3((S + 3) / 4), dim3(256), 0, s, p);
        REGC_HIP(hipGetLastError());
        std::vector<double> out(2 * (size_t)S + 1);
        REGC_HIP(hipMemcpyAsync(out.data(), p.mean, sizeof(double) * out.size(), hipMemcpyDeviceToHost, s));
        REGC_HIP(hipStreamSynchronize(s));
        int bad;
        memcpy(&bad, &out[2 * (size_t)S], sizeof bad);
        REGC_CHECK(!bad, REGC_EINVAL, "a sample's state is outside 0..%d or its N is negative", S - 1);
        std::copy(out.begin(), out.begin() + S, mean);
        std::copy(out.begin() + S, out.begin() + 2 * (size_t)S, se);
    }
    return REGC_OK;
}

extern "C" int regc_batch_means(int64_t ns, const int32_t *state, const int32_t *n, int n_states, int n_batches,
                                int on_device, double *mean, double *se, void *stream)
{
    REGC_CHECK(state && n && mean && se, REGC_EINVAL, "null argument");
    REGC_CHECK(ns > 0 && ns <= INT32_MAX, REGC_EINVAL, "sample count must be 1..2^31-1");
    REGC_CHECK(n_states > 0 && n_batches >= 2, REGC_EINVAL, "n_states must be positive and n_batches >= 2");
    hipStream_t s = static_cast<hipStream_t>(stream);
    DevBuf<int32_t> st_in, n_in;
    int rc;
    const int32_t *st_d = state, *n_d = n;
    if (!on_device) {
        if ((rc = st_in.alloc(ns)) || (rc = n_in.alloc(ns))) return rc;
        REGC_HIP(hipMemcpyAsync(st_in.p, state, sizeof(int32_t) * ns, hipMemcpyHostToDevice, s));
        REGC_HIP(hipMemcpyAsync(n_in.p, n, sizeof(int32_t) * ns, hipMemcpyHostToDevice, s));
        st_d = st_in.p;
        n_d = n_in.p;
    }
    return batch_means_dev(s, ns, st_d, n_d, n_states, n_batches, mean, se);
}

extern "C" int regc_reweight(regc_mbar *mb, const regc_grid *targets, double tol, int max_iter,
                             const regc_reweight_opts *opts, double *f_states, double *mean_state_n,
                             double *se_state_n, double *mean_n, double *se_n, int32_t *phase, double *coverage,
                             double *se_coverage, double *heat_cap, double *se_heat_cap, double *p_n)
{
    REGC_CHECK(mb && targets && targets->t && targets->mu, REGC_EINVAL, "null argument");
    REGC_CHECK(mb->have_samples, REGC_ESTATE, "no samples loaded");
    REGC_CHECK(max_iter > 0 && tol > 0, REGC_EINVAL, "max_iter and tol must be positive");
    regc_reweight_opts o;
    regc_default_reweight_opts(&o);
    if (opts) o = *opts;
    const int64_t rs = o.record_size > 0 ? o.record_size : mb->S;
    REGC_CHECK(o.n_batches >= 2 && o.n_boot >= 0 && o.n_boot != 1, REGC_EINVAL,
               "n_batches must be >= 2 and n_boot 0 or >= 2");
    REGC_CHECK(mb->ns % rs == 0, REGC_EINVAL, "%lld samples are not whole records of %lld", (long long)mb->ns,
               (long long)rs);
    const int64_t R = mb->ns / rs;
    const int64_t blk = o.block_records > 0 ? o.block_records : std::max<int64_t>(1, R / o.n_batches);
    REGC_CHECK(blk <= R, REGC_EINVAL, "bootstrap blocks of %lld records exceed the %lld records", (long long)blk,
               (long long)R);
    REGC_CHECK((coverage == nullptr && se_coverage == nullptr) || o.n_sites > 0, REGC_EINVAL,
               "coverage needs n_sites > 0");
    hipStream_t s = mb->stream;
    mb->weighted = false;
    int rc = solve_core(mb, tol, max_iter, nullptr, nullptr, nullptr);
    if (rc != REGC_OK && rc != REGC_ENOCONV) return rc;
    const int solve_rc = rc;
    std::vector<double> f0(mb->S);
    REGC_HIP(hipMemcpy(f0.data(), mb->f_d.p, sizeof(double) * mb->S, hipMemcpyDeviceToHost));
    if (f_states) std::copy(f0.begin(), f0.end(), f_states);
    TargetDev T;
    if ((rc = target_grid(mb, targets, T))) return rc;
    const int nK = T.nK;
    DevBuf<double> mn, me, me2, pn, heat, cov;
    std::vector<double> state_mean(mb->S), state_se(mb->S);
    DevBuf<int32_t> ph;
    if ((rc = mn.alloc(nK)) || (rc = me.alloc(nK)) || (rc = me2.alloc(nK)) || (rc = ph.alloc(nK)) ||
        (rc = pn.alloc(p_n ? (size_t)nK * mb->nN : 1)) || (rc = heat.alloc(nK)) || (rc = cov.alloc(nK)))
        return rc;
    if ((rc = targets_dev(mb, T, nullptr, mn.p, me.p, me2.p, p_n ? pn.p : nullptr, ph.p))) return rc;
    hipLaunchKernelGGL(heat_cov, dim3((nK + 255) / 256), dim3(256), 0, s, T.nT, T.nMu, T.tb_d.p, mn.p, me.p, me2.p,
                       o.n_sites > 0 ? o.n_sites : 1.0, heat.p, cov.p);
    REGC_HIP(hipGetLastError());
    if ((rc = batch_means_dev(s, mb->ns, mb->s_orig_d.p, mb->n_orig_d.p, mb->S, o.n_batches, state_mean.data(),
                              state_se.data())))
        return rc;
    REGC_HIP(hipStreamSynchronize(s));
    if (mean_n) REGC_HIP(hipMemcpy(mean_n, mn.p, sizeof(double) * nK, hipMemcpyDeviceToHost));
    if (phase) REGC_HIP(hipMemcpy(phase, ph.p, sizeof(int32_t) * nK, hipMemcpyDeviceToHost));
    if (p_n) REGC_HIP(hipMemcpy(p_n, pn.p, sizeof(double) * nK * mb->nN, hipMemcpyDeviceToHost));
    if (heat_cap) REGC_HIP(hipMemcpy(heat_cap, heat.p, sizeof(double) * nK, hipMemcpyDeviceToHost));
    if (coverage) REGC_HIP(hipMemcpy(coverage, cov.p, sizeof(double) * nK, hipMemcpyDeviceToHost));
    if (mean_state_n) std::copy(state_mean.begin(), state_mean.end(), mean_state_n);
    if (se_state_n) std::copy(state_se.begin(), state_se.end(), se_state_n);
    const bool want_boot = se_n || se_coverage || se_heat_cap;
    if (!want_boot || o.n_boot == 0) {
        const double nan = NAN;
        for (int k = 0; k < nK; ++k) {
            if (se_n) se_n[k] = nan;
            if (se_coverage) se_coverage[k] = nan;
            if (se_heat_cap) se_heat_cap[k] = nan;
        }
        return solve_rc;
    }
    // bootstrap replicates
    const int B = o.n_boot;
    const std::vector<double> lnomega0 = mb->lnomega;
    const int gauge0 = mb->gauge;
    DevBuf<int32_t> mult;
    DevBuf<unsigned long long> omega;
    DevBuf<double> rep_n, rep_c, sd_n, sd_c, bme, bme2;
    if ((rc = mult.alloc(R)) || (rc = omega.alloc(mb->S)) || (rc = mb->wgt_d.reserve(mb->ns)) ||
        (rc = rep_n.alloc((size_t)B * nK)) || (rc = rep_c.alloc((size_t)B * nK)) || (rc = sd_n.alloc(nK)) ||
        (rc = sd_c.alloc(nK)) || (rc = bme.alloc(nK)) || (rc = bme2.alloc(nK)))
        return rc;
    const int grid = (int)std::min<int64_t>((mb->ns + 255) / 256, 4096);
    const int64_t nblk = (R + blk - 1) / blk;
    int boot_rc = REGC_OK;
    // together where the solution came from the preconditioned iteration, else (or where
    // a replicate does not settle there) one after the other
    bool together = mb->inverse_valid && solve_rc == REGC_OK && max_iter >= kNewtonMinIter && R < INT32_MAX &&
                    mb->nN <= kBootNs &&
                    bounded_targets(mb, T.tb.data(), T.nT);
    const BootPlan plan = together ? boot_plan(mb, R, B, T.nT) : BootPlan{};
    together = together && plan.batch > 0;
    for (int b0 = 0; b0 < B && together; b0 += plan.batch) {
        rc = bootstrap_batch(mb, plan, T, tol, R, rs, blk, o.seed, b0, std::min(plan.batch, B - b0),
                             rep_n.p + (size_t)b0 * nK, rep_c.p + (size_t)b0 * nK, &together);
        if (rc) {
            (void)hipStreamSynchronize(s);
            return rc;
        }
    }
    if (plan.bytes > kBootKept) {
        REGC_HIP(hipStreamSynchronize(s));
        release_boot(mb);
    }
    for (int b = 0; b < B && boot_rc == REGC_OK && !together; ++b) {
        hipLaunchKernelGGL(fill_i32, dim3((unsigned)std::min<int64_t>((R + 255) / 256, 4096)), dim3(256), 0, s, R, 0,
                           mult.p);
        hipLaunchKernelGGL(boot_mult, dim3((unsigned)std::min<int64_t>((nblk + 255) / 256, 4096)), dim3(256), 0, s, R,
                           blk, b, (uint32_t)o.seed, (uint32_t)(o.seed >> 32), mult.p);
        hipLaunchKernelGGL(fill_u64, dim3(1), dim3(256), 0, s, (int64_t)mb->S, omega.p);
        hipLaunchKernelGGL(boot_weights, dim3(grid), dim3(256), 0, s, mb->ns, rs, mb->perm_d.p, mb->s_orig_d.p, mult.p,
                           mb->wgt_d.p, omega.p);
        REGC_HIP(hipGetLastError());
        if ((rc = set_omega(mb, omega.p))) { boot_rc = rc; break; }
        mb->weighted = true;
        rc = solve_core(mb, tol, max_iter, f0.data(), nullptr, nullptr);
        if (rc != REGC_OK && rc != REGC_ENOCONV) { boot_rc = rc; break; }
        if (rc == REGC_ENOCONV) boot_rc = REGC_ENOCONV;
        if ((rc = targets_dev(mb, T, nullptr, rep_n.p + (size_t)b * nK, bme.p, bme2.p, nullptr, ph.p))) {
            boot_rc = rc;
            break;
        }
        hipLaunchKernelGGL(heat_cov, dim3((nK + 255) / 256), dim3(256), 0, s, T.nT, T.nMu, T.tb_d.p,
                           rep_n.p + (size_t)b * nK, bme.p, bme2.p, 1.0, rep_c.p + (size_t)b * nK, nullptr);
        REGC_HIP(hipGetLastError());
    }
    if (!together) {
        // back to the full data: counts, f, log D
        mb->weighted = false;
        mb->lnomega = lnomega0;
        mb->gauge = gauge0;
        REGC_HIP(hipMemcpyAsync(mb->lnomega_d.p, lnomega0.data(), sizeof(double) * mb->S, hipMemcpyHostToDevice, s));
        REGC_HIP(hipMemcpyAsync(mb->f_d.p, f0.data(), sizeof(double) * mb->S, hipMemcpyHostToDevice, s));
        if ((rc = refresh_logd(mb))) return rc;
        REGC_HIP(hipStreamSynchronize(s));
    }
    if (boot_rc != REGC_OK && boot_rc != REGC_ENOCONV) return boot_rc;
    hipLaunchKernelGGL(rep_sd, dim3((nK + 255) / 256), dim3(256), 0, s, B, nK, rep_n.p, sd_n.p);
    hipLaunchKernelGGL(rep_sd, dim3((nK + 255) / 256), dim3(256), 0, s, B, nK, rep_c.p, sd_c.p);
    REGC_HIP(hipGetLastError());
    REGC_HIP(hipStreamSynchronize(s));
    std::vector<double> h(nK);
    REGC_HIP(hipMemcpy(h.data(), sd_n.p, sizeof(double) * nK, hipMemcpyDeviceToHost));
    if (se_n) std::copy(h.begin(), h.end(), se_n);
    if (se_coverage)
        for (int k = 0; k < nK; ++k) se_coverage[k] = h[k] / o.n_sites;
    if (se_heat_cap) REGC_HIP(hipMemcpy(se_heat_cap, sd_c.p, sizeof(double) * nK, hipMemcpyDeviceToHost));
    if (boot_rc == REGC_ENOCONV) {
        set_error("a bootstrap replicate did not converge");
        return REGC_ENOCONV;
    }
    return solve_rc;
}
