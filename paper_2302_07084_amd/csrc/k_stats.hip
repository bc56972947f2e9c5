// Graph descriptors for the hyperparameter search's surrogate (section 4.4
// searches trials per graph; which descriptors condition the surrogate is
// this library's choice): degree moments, the median degree and the Hill
// tail exponent above it, wedge-sampled clustering, and the spectral gap of
// D^-1/2 A D^-1/2 by block subspace iteration.
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "philox.hpp"

namespace lne {
namespace {

constexpr uint32_t kTagWedge = 6u << 24;   // counter tag of the wedge draws
constexpr int kStatThreads = 256;
constexpr int kStatBlocks = 256;
constexpr int kHistLds = 4096;             // degrees below this count in LDS first
constexpr int kWalkB = 16;                 // widest block of the subspace iteration

// sums: [0] degree sum, [1] sum of squared degrees, [2] vertices of degree
// >= 2, [3] maximum degree (integers, so the order of accumulation is moot)
__global__ void k_deg_moments(const int64_t *__restrict__ rp, int64_t n,
                              unsigned long long *__restrict__ sums) {
    unsigned long long s1 = 0, s2 = 0, c2 = 0, mx = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const unsigned long long d = (unsigned long long)(rp[i + 1] - rp[i]);
        s1 += d;
        s2 += d * d;
        c2 += d >= 2 ? 1 : 0;
        mx = d > mx ? d : mx;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        s1 += __shfl_xor(s1, o, 64);
        s2 += __shfl_xor(s2, o, 64);
        c2 += __shfl_xor(c2, o, 64);
        const unsigned long long y = __shfl_xor(mx, o, 64);
        mx = y > mx ? y : mx;
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&sums[0], s1);
        atomicAdd(&sums[1], s2);
        atomicAdd(&sums[2], c2);
        atomicMax(&sums[3], mx);
    }
}

// Degree histogram (hist has at least kHistLds bins): small degrees, where a
// power-law graph puts most vertices, are counted per block in LDS first.
__global__ void k_deg_hist(const int64_t *__restrict__ rp, int64_t n, uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[kHistLds];
    for (int b = threadIdx.x; b < kHistLds; b += blockDim.x) h[b] = 0;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t d = rp[i + 1] - rp[i];
        if (d < kHistLds) atomicAdd(&h[d], 1u);
        else atomicAdd(&hist[d], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kHistLds; b += blockDim.x)
        if (h[b]) atomicAdd(&hist[b], h[b]);
}

// The degrees of ranks r0 and r1 in ascending order (cum: exclusive prefix
// counts of the histogram, nb + 1 entries).
__global__ void k_order_stat(const uint64_t *__restrict__ cum, int64_t nb, uint64_t r0,
                             uint64_t r1, int64_t *__restrict__ out) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nb) return;
    const uint64_t lo = cum[b], hi = cum[b + 1];
    if (lo <= r0 && r0 < hi) out[0] = b;
    if (lo <= r1 && r1 < hi) out[1] = b;
}

// Per-block sums of log(d / (x_min - 1/2)) over degrees d >= x_min, and
// their count.
__global__ void k_hill(const int64_t *__restrict__ rp, int64_t n, double xmin,
                       double *__restrict__ part, unsigned long long *__restrict__ cnt) {
    __shared__ double ws[kStatThreads / 64];
    double s = 0.0;
    unsigned long long c = 0;
    const double den = xmin - 0.5;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double d = (double)(rp[i + 1] - rp[i]);
        if (d >= xmin) {
            s += log(d / den);
            ++c;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        s += __shfl_xor(s, o, 64);
        c += __shfl_xor(c, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        ws[threadIdx.x >> 6] = s;
        atomicAdd(cnt, c);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kStatThreads / 64; ++w) t += ws[w];
        part[blockIdx.x] = t;
    }
}

// out[0] = sum of part[0..np) in a fixed order (one wave).
__global__ void k_sum_parts(const double *__restrict__ part, int np, double *__restrict__ out) {
    double s = 0.0;
    for (int i = threadIdx.x; i < np; i += 64) s += part[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (threadIdx.x == 0) out[0] = s;
}

__global__ void k_flag_deg2(const int64_t *__restrict__ rp, int64_t n, uint32_t *__restrict__ f) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) f[i] = rp[i + 1] - rp[i] >= 2 ? 1u : 0u;
}

__global__ void k_compact_deg2(const int64_t *__restrict__ rp, int64_t n,
                               const uint64_t *__restrict__ off, int32_t *__restrict__ cand) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && rp[i + 1] - rp[i] >= 2) cand[off[i]] = (int32_t)i;
}

// Wedge t: Philox block of counter (t_lo, t_hi, 0, tag) under key seed;
// centre = cand[((z1 << 32) | z0) mod nc], ends = its neighbours at z2 mod d
// and z3 mod (d - 1) (moved past the first when not smaller); closed when
// the second end is in the first end's sorted row.
__global__ void k_wedges(const int64_t *__restrict__ rp, const int32_t *__restrict__ col,
                         const int32_t *__restrict__ cand, uint64_t nc, uint64_t seed,
                         int64_t wedges, unsigned long long *__restrict__ closed) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= wedges) return;
    const uint4 z = philox4x32_10(make_uint4((uint32_t)t, (uint32_t)((uint64_t)t >> 32), 0u,
                                             kTagWedge),
                                  (uint32_t)seed, (uint32_t)(seed >> 32));
    const int32_t c = cand[((((uint64_t)z.y) << 32) | z.x) % nc];
    const int64_t r0 = rp[c];
    const uint32_t d = (uint32_t)(rp[c + 1] - r0);
    const uint32_t ia = z.z % d;
    uint32_t ib = z.w % (d - 1);
    if (ib >= ia) ++ib;
    const int32_t a = col[r0 + ia], b = col[r0 + ib];
    int64_t lo = rp[a];
    const int64_t end = rp[a + 1];
    int64_t hi = end;
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if (col[mid] < b) lo = mid + 1; else hi = mid;
    }
    if (lo < end && col[lo] == b) atomicAdd(closed, 1ull);
}

__global__ void k_inv_sqrt_deg(const int64_t *__restrict__ rp, int64_t n, double *__restrict__ s) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t d = rp[i + 1] - rp[i];
    s[i] = d > 0 ? 1.0 / sqrt((double)d) : 0.0;
}

// Y = (X + S A S X) / 2 for n x b row-major blocks (b <= kWalkB), S =
// diag(s).  G groups of kWalkB lanes take a row: they read a neighbour and its s
// a lane, then each group gathers every G-th neighbour's row of X, lane c of it
// summing column c.  Bound by latency (a row is three dependent reads), on many
// rows by the gathered lines: with kWalkB lanes a row, one neighbour at a time,
// it took 29 us at n = 30,000 and 9 10^5 arcs, with eight in flight 25, with a
// wave a row 18 us.
constexpr int kWalkU = 4;
constexpr int64_t kWalkBlocks = 1 << 22;   // a launch has fewer than 2^32 threads: more rows are
                                           // taken in turn
// The groups of a row: a wave's four where a hub's row would outlast the others,
// two of them where there are rows enough to cover that, one on short rows of
// like length (all four on few rows, where only latency counts).  A step of
// graph_stats, us, by G:
//                          1      2      4
//      2,000 planted      21.9   21.8   21.5      (12)
//     30,000 cycle        29.8   35.1   39.5      (2 arcs a row)
//     30,000 planted      36.9   37.7   39.6      (16)    64.4   62.8   62.4 (100)
//  3,000,000 cycle         761  1,029  1,585
//  3,000,000 planted     2,047  2,023  2,058      (16)
//     30,000 power-law    96.6   66.4   50.9      (16)
//    300,000 power-law     199    132    146      (4)      378    233    185 (16)
//  3,000,000 power-law   1,231  1,157  1,624      (4)    3,117  2,542  2,800 (24)
inline int half_walk_groups(int64_t n, double mean, uint64_t max_deg) {
    if (n < 8192) return 4;
    if (max_deg <= 64) return mean <= 16.0 ? 1 : 4;
    return n >= 1 << 20 && mean <= 32.0 ? 2 : 4;
}
template <int G>
__global__ void __launch_bounds__(kStatThreads)
k_half_walk(const int64_t *__restrict__ rp, const int32_t *__restrict__ col,
            const double *__restrict__ s, const double *__restrict__ X, double *__restrict__ Y,
            int64_t n, int b) {
    constexpr int L = kWalkB * G;
    const int lane = threadIdx.x % L, grp = lane / kWalkB, c = lane % kWalkB;
    const double *xc = X + (c < b ? c : 0);   // idle lanes read column 0
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / L; i < n;
         i += (int64_t)gridDim.x * blockDim.x / L) {
        double acc = 0.0;
        const int64_t end = rp[i + 1];
        for (int64_t e0 = rp[i]; e0 < end; e0 += L) {
            const int cnt = (int)min((int64_t)L, end - e0);
            const int32_t j = col[e0 + min(lane, cnt - 1)];
            const double sj = lane < cnt ? s[j] : 0.0;
            for (int t0 = 0; t0 < cnt; t0 += G * kWalkU) {
                double x[kWalkU], f[kWalkU];
#pragma unroll
                for (int u = 0; u < kWalkU; ++u) {
                    const int t = t0 + G * u + grp;   // past cnt: the last one, weight 0
                    const int32_t jt = __shfl(j, min(t, L - 1), L);
                    f[u] = t < L ? __shfl(sj, min(t, L - 1), L) : 0.0;
                    x[u] = xc[(int64_t)jt * b];
                }
#pragma unroll
                for (int u = 0; u < kWalkU; ++u) acc += f[u] * x[u];
            }
        }
#pragma unroll
        for (int o = kWalkB; o < L; o <<= 1) acc += __shfl_xor(acc, o, 64);
        if (grp == 0 && c < b) Y[i * b + c] = 0.5 * (X[i * b + c] + s[i] * acc);
    }
}

}  // namespace

lne_status graph_stats_impl(lne_ctx *ctx, const Graph *g, uint64_t seed, int32_t wedges,
                            int32_t iters, double *out) {
    const int64_t n = g->n, arcs = g->n_arcs;
    const int64_t *rp = g->row_ptr;
    const unsigned nblk = std::min<unsigned>(grid_of(n, kStatThreads), 1024u);
    // degree moments
    Buf sums(ctx);
    LNE_TRY(alloc(ctx, sums, 4 * sizeof(unsigned long long)));
    LNE_HIP(ctx, hipMemsetAsync(sums.p, 0, 4 * sizeof(unsigned long long), ctx->stream));
    {
        Launch L(ctx, "graph_stats");
        k_deg_moments<<<nblk, kStatThreads, 0, ctx->stream>>>(rp, n, sums.as<unsigned long long>());
    }
    LNE_TRY(check_launch(ctx, "graph_stats"));
    unsigned long long hs[4];
    LNE_HIP(ctx, hipMemcpyAsync(hs, sums.p, sizeof(hs), hipMemcpyDeviceToHost, ctx->stream));
    LNE_HIP(ctx, hipStreamSynchronize(ctx->stream));
    const unsigned long long s1 = hs[0], s2 = hs[1], ncand = hs[2], maxd = hs[3];
    if (s1 != (unsigned long long)arcs)
        return fail(ctx, LNE_EINVAL, "graph_stats: row_ptr does not span n_arcs");
    const double mean = (double)s1 / (double)n;
    // population variance from exact integers: (n s2 - s1^2) / n^2
    const unsigned __int128 num = (unsigned __int128)n * s2 - (unsigned __int128)s1 * s1;
    const double var = (double)num / ((double)n * (double)n);
    out[0] = std::log((double)n);
    out[1] = std::log((double)std::max<int64_t>(arcs / 2, 1));
    out[2] = std::log(mean);
    out[3] = std::sqrt(var) / mean;
    out[4] = std::log((double)maxd);
    // median degree from the histogram's prefix counts
    const int64_t nb = std::max<int64_t>((int64_t)maxd + 1, kHistLds);
    Buf hist(ctx), cum(ctx), ost(ctx);
    LNE_TRY(alloc(ctx, hist, sizeof(uint32_t) * (size_t)nb));
    LNE_TRY(alloc(ctx, cum, sizeof(uint64_t) * (size_t)(nb + 1)));
    LNE_TRY(alloc(ctx, ost, 2 * sizeof(int64_t)));
    LNE_HIP(ctx, hipMemsetAsync(hist.p, 0, sizeof(uint32_t) * (size_t)nb, ctx->stream));
    {
        Launch L(ctx, "graph_stats");
        k_deg_hist<<<nblk, kStatThreads, 0, ctx->stream>>>(rp, n, hist.as<uint32_t>());
    }
    LNE_TRY(check_launch(ctx, "graph_stats"));
    LNE_TRY(scan_u32(ctx, hist.as<uint32_t>(), cum.as<uint64_t>(), nb));
    {
        Launch L(ctx, "graph_stats");
        k_order_stat<<<grid_of(nb, kStatThreads), kStatThreads, 0, ctx->stream>>>(
            cum.as<uint64_t>(), nb, (uint64_t)(n - 1) / 2, (uint64_t)n / 2, ost.as<int64_t>());
    }
    LNE_TRY(check_launch(ctx, "graph_stats"));
    int64_t med[2];
    LNE_HIP(ctx, hipMemcpyAsync(med, ost.p, sizeof(med), hipMemcpyDeviceToHost, ctx->stream));
    LNE_HIP(ctx, hipStreamSynchronize(ctx->stream));
    const double xmin = std::max(1.0, 0.5 * ((double)med[0] + (double)med[1]));
    // Hill tail exponent
    Buf part(ctx), hsum(ctx), hcnt(ctx);
    LNE_TRY(alloc(ctx, part, sizeof(double) * kStatBlocks));
    LNE_TRY(alloc(ctx, hsum, sizeof(double)));
    LNE_TRY(alloc(ctx, hcnt, sizeof(unsigned long long)));
    LNE_HIP(ctx, hipMemsetAsync(hcnt.p, 0, sizeof(unsigned long long), ctx->stream));
    {
        Launch L(ctx, "graph_stats");
        k_hill<<<kStatBlocks, kStatThreads, 0, ctx->stream>>>(rp, n, xmin, part.as<double>(),
                                                             hcnt.as<unsigned long long>());
        k_sum_parts<<<1, 64, 0, ctx->stream>>>(part.as<double>(), kStatBlocks, hsum.as<double>());
    }
    LNE_TRY(check_launch(ctx, "graph_stats"));
    double hl = 0.0;
    unsigned long long hc = 0;
    LNE_HIP(ctx, hipMemcpyAsync(&hl, hsum.p, sizeof(hl), hipMemcpyDeviceToHost, ctx->stream));
    LNE_HIP(ctx, hipMemcpyAsync(&hc, hcnt.p, sizeof(hc), hipMemcpyDeviceToHost, ctx->stream));
    LNE_HIP(ctx, hipStreamSynchronize(ctx->stream));
    out[5] = 1.0 + (double)hc / std::max(hl, 1e-9);
    // wedge clustering
    unsigned long long closed = 0;
    if (ncand > 0) {
        Buf flag(ctx), off(ctx), cand(ctx), cl(ctx);
        LNE_TRY(alloc(ctx, flag, sizeof(uint32_t) * (size_t)n));
        LNE_TRY(alloc(ctx, off, sizeof(uint64_t) * (size_t)(n + 1)));
        LNE_TRY(alloc(ctx, cand, sizeof(int32_t) * (size_t)ncand));
        LNE_TRY(alloc(ctx, cl, sizeof(unsigned long long)));
        LNE_HIP(ctx, hipMemsetAsync(cl.p, 0, sizeof(unsigned long long), ctx->stream));
        {
            Launch L(ctx, "graph_stats");
            k_flag_deg2<<<grid_of(n, kStatThreads), kStatThreads, 0, ctx->stream>>>(
                rp, n, flag.as<uint32_t>());
        }
        LNE_TRY(check_launch(ctx, "graph_stats"));
        LNE_TRY(scan_u32(ctx, flag.as<uint32_t>(), off.as<uint64_t>(), n));
        {
            Launch L(ctx, "graph_stats");
            k_compact_deg2<<<grid_of(n, kStatThreads), kStatThreads, 0, ctx->stream>>>(
                rp, n, off.as<uint64_t>(), cand.as<int32_t>());
            k_wedges<<<grid_of(wedges, kStatThreads), kStatThreads, 0, ctx->stream>>>(
                rp, g->col, cand.as<int32_t>(), ncand, seed, wedges,
                cl.as<unsigned long long>());
        }
        LNE_TRY(check_launch(ctx, "graph_stats"));
        LNE_HIP(ctx, hipMemcpyAsync(&closed, cl.p, sizeof(closed), hipMemcpyDeviceToHost,
                                    ctx->stream));
        LNE_HIP(ctx, hipStreamSynchronize(ctx->stream));
    }
    out[6] = (double)closed / (double)wedges;
    // spectral gap: subspace iteration on (I + S A S) / 2 from X = Omega; S_2
    // is the second singular value of the last product, the same for any
    // orthonormal basis of the span of the block before it.  So the steps
    // before the last orthonormalise by one CholeskyQR pass (8 us of
    // factorisation at b = 16 against 122 us of eigen-solve, 8.8 ms against 36 ms
    // in all at n = 30,000 and 200 steps), which keeps the span, and the block
    // before the last product takes a second: one pass is off by about cond^2 u.  A breakdown (a block that is rank deficient to
    // rounding, as on graphs of few vertices) repeats the steps with eigSVD,
    // which drops the directions that vanish.  It is looked for after the
    // second step, before the others are spent (11.4 ms in all for twelve
    // separate edges with eigSVD alone, 13.6 when looked for at the end only):
    // the operator H is positive semi-definite, so |H H y| / |H y| >= |H y| /
    // |y|, and the least singular value of a step's product can only rise from
    // the first orthonormal block on.
    const int b = (int)std::min<int64_t>(kWalkB, n);
    Buf s(ctx), X(ctx), Y(ctx), S(ctx), G(ctx), W(ctx), fl(ctx);
    LNE_TRY(alloc(ctx, s, sizeof(double) * (size_t)n));
    LNE_TRY(alloc(ctx, X, sizeof(double) * (size_t)n * b));
    LNE_TRY(alloc(ctx, Y, sizeof(double) * (size_t)n * b));
    LNE_TRY(alloc(ctx, S, sizeof(double) * (size_t)b));
    LNE_TRY(alloc(ctx, G, sizeof(double) * (size_t)b * b));
    LNE_TRY(alloc(ctx, W, sizeof(double) * (size_t)b * b));
    LNE_TRY(alloc(ctx, fl, sizeof(int32_t) * kFlagStride));
    LNE_HIP(ctx, hipMemsetAsync(fl.p, 0, fl.bytes, ctx->stream));
    {
        Launch L(ctx, "graph_stats");
        k_inv_sqrt_deg<<<grid_of(n, kStatThreads), kStatThreads, 0, ctx->stream>>>(
            rp, n, s.as<double>());
    }
    LNE_TRY(check_launch(ctx, "graph_stats"));
    const int wide = half_walk_groups(n, mean, maxd);
    double sv[2] = {0.0, 0.0};
    int32_t hf[kFlagStride];
    for (const bool eig : {false, true}) {
        bool broken = false;
        double *x = X.as<double>(), *y = Y.as<double>();
        LNE_TRY(lne_gaussian(ctx, n, b, b, seed, LNE_F64, x));
        for (int it = 0; it < iters; ++it) {
            {
                Launch L(ctx, "graph_stats");
                const unsigned grid = (unsigned)std::min<int64_t>(
                    ceil_div(n * kWalkB * wide, kStatThreads), kWalkBlocks);
#define LNE_HW(G)                                                                          \
    k_half_walk<G><<<grid, kStatThreads, 0, ctx->stream>>>(rp, g->col, s.as<double>(), x, y, n, b)
                if (wide == 1) LNE_HW(1);
                else if (wide == 2) LNE_HW(2);
                else LNE_HW(4);
#undef LNE_HW
            }
            LNE_TRY(check_launch(ctx, "graph_stats"));
            if (it + 1 == iters) {
                LNE_TRY(lne_eigsvd(ctx, y, n, b, b, LNE_F64, nullptr, b, S.as<double>(), nullptr));
            } else if (eig) {
                LNE_TRY(lne_eigsvd(ctx, y, n, b, b, LNE_F64, x, b, nullptr, nullptr));
            } else {
                int32_t *f = fl.as<int32_t>();
                for (int pass = it + 2 == iters ? 2 : 1; pass > 0; --pass) {
                    LNE_TRY(gram(ctx, y, LNE_F64, n, b, b, G.as<double>(), nullptr));
                    LNE_TRY(chol_inv(ctx, G.as<double>(), b, W.as<double>(), f, f + 1, n, nullptr,
                                     nullptr));
                    LNE_TRY(project(ctx, y, LNE_F64, b, n, b, W.as<double>(), b, y, LNE_F64, b,
                                    nullptr, 1, 0, 0, 0, nullptr, true));
                }
                std::swap(x, y);
                if (it == 1) {
                    LNE_HIP(ctx, hipMemcpyAsync(hf, fl.p, sizeof(hf), hipMemcpyDeviceToHost,
                                                ctx->stream));
                    LNE_HIP(ctx, hipStreamSynchronize(ctx->stream));
                    broken = hf[0] != 0 || hf[1] != 0;
                    if (broken) break;
                }
            }
        }
        if (broken) continue;
        LNE_HIP(ctx, hipMemcpyAsync(hf, fl.p, sizeof(hf), hipMemcpyDeviceToHost, ctx->stream));
        LNE_HIP(ctx, hipMemcpyAsync(sv, S.p, sizeof(double) * (size_t)std::min(b, 2),
                                    hipMemcpyDeviceToHost, ctx->stream));
        LNE_HIP(ctx, hipStreamSynchronize(ctx->stream));
        if (hf[0] == 0 && hf[1] == 0) break;   // no breakdown and no shift
    }
    out[7] = 1.0 - (2.0 * (b > 1 ? sv[1] : sv[0]) - 1.0);
    return LNE_OK;
}

}  // namespace lne
