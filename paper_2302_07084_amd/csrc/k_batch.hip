// Batched hyperparameter trials sharing one sampling pass (section 4.4: many
// trials of s_1..s_T, k, theta, mu on one graph).
//
// The shared pass draws the walk length r from a sampling distribution pi
// (chosen for the batch) and keeps r in the count matrix, giving per-length
// channels W_r.  Trial t then uses sum_r (s_r^(t) / pi_r) W_r in place of the
// counts, which has the expectation of its own sampler whenever pi_r > 0 for
// every r with s_r^(t) > 0; the truncated logarithm is applied per trial on
// the shared structure (dropped entries keep an explicit zero).
//
// Nothing per trial is materialised at the size of the matrix: each SpMM of
// trial t regenerates M_t's values from the channel CSR while it streams it,
// and the dense blocks of all trials (n x k' each, trial-major) go through
// one launch per step (batched Gram, Cholesky, eigen-solves and projections,
// one channel SpMM over every (trial, row) pair, one graph SpMM per
// propagation step with per-trial epilogue coefficients).
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace lne {

namespace {

// number of distinct base columns (extended column >> 4) in each row
__global__ void k_split_count(const int64_t *__restrict__ rp, const int32_t *__restrict__ col,
                              int64_t n, uint32_t *__restrict__ cnt) {
    const int64_t a = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (a >= n) return;
    const int64_t beg = rp[a], end = rp[a + 1];
    uint32_t c = 0;
    for (int64_t i = beg + lane; i < end; i += 64)
        c += (i == beg || (col[i] >> 4) != (col[i - 1] >> 4)) ? 1u : 0u;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if (lane == 0) cnt[a] = c;
}

__global__ void k_split_fill(const int64_t *__restrict__ rp, const int32_t *__restrict__ col,
                             const uint64_t *__restrict__ W, int64_t n,
                             const int64_t *__restrict__ srp, int32_t *__restrict__ scol,
                             uint64_t *__restrict__ chan, int T) {
    const int64_t a = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (a >= n) return;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const int64_t beg = rp[a], end = rp[a + 1];
    int64_t pos = srp[a];
    for (int64_t i0 = beg; i0 < end; i0 += 64) {
        const int64_t i = i0 + lane;
        const bool valid = i < end;
        int32_t c = 0;
        bool head = false;
        if (valid) {
            c = col[i];
            head = i == beg || (c >> 4) != (col[i - 1] >> 4);
        }
        const uint64_t hm = __ballot(head);
        if (valid) {
            const int64_t u = pos + (int64_t)__popcll(hm & (lt | (1ull << lane))) - 1;
            if (head) scol[u] = c >> 4;
            const int r = c & 15;
            if (r < T) chan[u * T + r] = W[i];
        }
        pos += __popcll(hm);
    }
}

// vals[i * ntr + t] = ln x if x > 1 else 0, x = scale * sum_r c_t[r] W_r /
// (d_a d_b) with c_t[r] = s_t[r] / pi_r and scale = vol^2 / (2 b M) / 2^16.
__global__ void k_trial_values(const int64_t *__restrict__ grp, const int64_t *__restrict__ srp,
                               const int32_t *__restrict__ scol, const uint64_t *__restrict__ chan,
                               int T, int64_t n, const double *__restrict__ s, int ntr,
                               double scale, float *__restrict__ vals) {
    const int64_t a = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (a >= n) return;
    const double da = (double)(grp[a + 1] - grp[a]);
    for (int64_t i = srp[a] + lane; i < srp[a + 1]; i += 64) {
        const int32_t b = scol[i];
        const double dd = da * (double)(grp[b + 1] - grp[b]);
        double w[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) w[r] = r < T ? (double)chan[i * T + r] : 0.0;
        for (int t = 0; t < ntr; ++t) {
            double acc = 0.0;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc += s[t * 16 + r] * w[r];
            const double x = acc * scale / dd;
            vals[i * ntr + t] = x > 1.0 ? (float)log(x) : 0.0f;
        }
    }
}

// Channel weights in place: W_r (fixed-point counts) -> the FP64 number
// scale W_r / (d_a d_b) (scale = vol^2 / (2 b M 2^16)), so that a trial's
// Eq. (1) argument is x = sum_r coef_t[r] w_r with coef_t[r] = s_t[r] / pi_r.
__global__ void k_norm_chan(const int64_t *__restrict__ rp, const int32_t *__restrict__ ecol,
                            const int64_t *__restrict__ grp, int64_t n, double scale,
                            uint64_t *__restrict__ W) {
    const int64_t a = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (a >= n) return;
    const double da = (double)(grp[a + 1] - grp[a]);
    double *out = reinterpret_cast<double *>(W);
    for (int64_t i = rp[a] + lane; i < rp[a + 1]; i += 64) {
        const int32_t b = ecol[i] >> 4;
        const double db = (double)(grp[b + 1] - grp[b]);
        out[i] = scale * (double)W[i] / (da * db);
    }
}

// ---- channel SpMM -------------------------------------------------------------
// Y_t = M_t X_t for trials t = 0..ntr-1 with M_t generated on the fly from
// the normalised channel CSR: every (row a, column b) structure entry is a
// run of channel entries with the same b (ascending r); a segmented scan over
// the wave sums x = sum_r coef_t[r] w_r with coef_t[r] = s_t[r] / pi_r (FP64,
// so the x > 1 decision is taken in FP64; a run crossing a 64-entry chunk
// carries its partial sum), and the lane holding the run's last entry forms
// the truncated logarithm ln x (FP32; 0 if x <= 1).  Then the wave gathers the
// X rows of the chunk's nonzero values, in column order, U rows in flight,
// lane l holding VW columns (k <= 256; padding columns of X zero).
//
// seg: the columns are cut into ranges whose X rows fit one XCD's L2 beside
// the stream of entries (chan_ranges); each launch adds range sg's entries to
// Y, and a row's range is found in a table of offsets (k_chan_segments).
// Every row still takes its entries in column order, its running sums carried
// through Y between the launches (FP32 both ways), so that the ranges do not
// change the result.
//   TB = 1: wave (trial, row), trial-major (TM: consecutive waves share a
//   trial's operand) or row-major (they share a row's entries).
//   TB > 1: wave = row, TB trials of one shared operand: an X row is gathered
//   once for all of them (a trial that drops the entry adds nothing).
// 2 10^8 entries, n = 10^5, 144 columns, eight trials: each trial's own operand
// 132 ms by whole rows with four columns a lane (bound by memory-side lines),
// 50 by ranges of 2.5 MB; one operand for all 70 ms with a gather each, 24
// with one.  Bound by instruction issue then: a lane holds the fewest columns
// that 64 lanes cover k with (48 lanes of three at k = 144, not 36 of four),
// the kept entries are found by scalar bit operations and their rows addressed
// by scalars, and the scan stops at the chunk's longest run (seen in the bits
// of the run heads).
template <int VW> struct FVec { float v[VW]; };

template <int TB, int VW, int U, bool TM>
__global__ void __launch_bounds__(256)
k_chan_seg(const int64_t *__restrict__ rp, const uint32_t *__restrict__ seg, int nseg, int sg,
           const int32_t *__restrict__ ecol, const double *__restrict__ wn, int64_t n, int ntr,
           const double *__restrict__ coef, const float *__restrict__ X, int64_t ldx, int64_t xs,
           float *__restrict__ Y, int64_t ldy, int64_t ys, int k, int first) {
    static_assert(TB == 1 || TM, "shared operands: a wave per row");
    const int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t groups = (ntr + TB - 1) / TB;
    if (w >= n * groups) return;
    const int64_t tg = TM ? w / n : w % ntr, row = TM ? w - tg * n : w / ntr;
    const int t0 = (int)tg * TB;
    const int lane = threadIdx.x & 63;
    const int c0 = lane * VW;
    const bool act = c0 < k;
    // row j at j * ldx (scalar), the lane's columns behind it (idle lanes read
    // the row's first)
    X += (int64_t)t0 * xs;
    const uint32_t ldw = (uint32_t)ldx, xo = act ? 4 * c0 : 0;
    Y += (int64_t)t0 * ys + row * ldy + c0;
    coef += 16 * t0;
    int64_t beg = rp[row], end = rp[row + 1];
    if (seg) {
        end = beg + seg[row * (nseg + 1) + sg + 1];
        beg += seg[row * (nseg + 1) + sg];
    }
    if (beg == end && !first) return;
    using V = FVec<VW>;
    V acc[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t) {
        acc[t] = V{};
        if (!first && act && t0 + t < ntr) acc[t] = *reinterpret_cast<const V *>(Y + t * ys);
    }
    const uint64_t upto = lane == 63 ? ~0ull : ((2ull << lane) - 1);   // lanes 0..lane
    int32_t prev_b = -1;      // base column of the entry before the chunk
    double carry[TB];         // partial sum of the run that reaches into the chunk
#pragma unroll
    for (int t = 0; t < TB; ++t) carry[t] = 0.0;
    // the next chunk's structure is loaded while the current one is gathered
    int32_t ec_next = beg + lane < end ? ecol[beg + lane] : -16;
    double w_next = beg + lane < end ? wn[beg + lane] : 0.0;
    for (int64_t b0 = beg; b0 < end; b0 += 64) {
        const int64_t i = b0 + lane;
        const bool valid = i < end;
        const int32_t ec = ec_next;
        const double wv = w_next;
        ec_next = i + 64 < end ? ecol[i + 64] : -16;
        w_next = i + 64 < end ? wn[i + 64] : 0.0;
        const int32_t jb = ec >> 4;
        const int32_t up_b = __shfl_up(jb, 1, 64);
        const bool head = valid && (lane == 0 ? prev_b : up_b) != jb;
        const uint64_t hm = __ballot(head);
        // longest run of the chunk: more than off entries iff off neighbouring
        // lanes are not heads
        const uint64_t nh = ~hm & __ballot(valid);
        const int32_t dn_b = __shfl_down(jb, 1, 64);
        const int32_t first_next = __builtin_amdgcn_readfirstlane(ec_next) >> 4;
        const int32_t nb = lane == 63 ? (b0 + 64 < end ? first_next : -2) : dn_b;
        const bool last = valid && (i + 1 >= end || nb != jb);
        const bool open = valid && (hm & upto) == 0;    // in the run carried into the chunk
        float v[TB];
        uint64_t any = 0, all = ~0ull;   // entries that some trial keeps, that all do
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            double sum = valid && t0 + t < ntr ? coef[16 * t + (ec & 15)] * wv : 0.0;
            // segmented inclusive scan: a lane adds the partial of lane - off
            // when no run starts in (lane - off, lane]; a run holds at most
            // one entry per length (<= 16), so four doubling steps cover it
            uint64_t more = nh;
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) {
                if (more == 0) break;
                const double o = __shfl_up(sum, off, 64);
                const int src = lane - off;
                const uint64_t below = src < 0 ? 0ull : (src == 63 ? ~0ull : ((2ull << src) - 1));
                if (src >= 0 && (hm & upto & ~below) == 0) sum += o;
                more &= more >> off;
            }
            if (open) sum += carry[t];
            v[t] = 0.f;
            if (last) v[t] = sum > 1.0 ? logf((float)sum) : 0.f;
            carry[t] = __shfl(sum, 63, 64);
            const uint64_t kept = __ballot(v[t] != 0.f);
            any |= kept;
            if (t0 + t < ntr) all &= kept;
        }
        prev_b = __builtin_amdgcn_readlane(jb, 63);
        // the kept entries in order, U rows in flight
        auto pop = [&](auto count) {
            int l[count];
            uint64_t group = 0;
#pragma unroll
            for (int q = 0; q < count; ++q) {
                l[q] = __builtin_ctzll(any);
                group |= 1ull << l[q];
                any &= ~(1ull << l[q]);
            }
            V x[count];
#pragma unroll
            for (int q = 0; q < count; ++q)
                x[q] = *reinterpret_cast<const V *>(
                    reinterpret_cast<const char *>(
                        X + (uint64_t)(uint32_t)__builtin_amdgcn_readlane(jb, l[q]) * ldw) + xo);
            auto add = [&](auto every) {
#pragma unroll
                for (int q = 0; q < count; ++q)
#pragma unroll
                    for (int t = 0; t < TB; ++t) {
                        const float f =
                            __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[t]), l[q]));
                        if (!every && f == 0.f) continue;
#pragma unroll
                        for (int i = 0; i < VW; ++i) acc[t].v[i] += f * x[q].v[i];
                    }
            };
            // an entry that only some trials keep adds 0 times its row to the
            // others, which is nothing unless the row is infinite or undefined
            bool exact = TB == 1 || (group & ~all) == 0;
            if (!exact) {
                float z = 0.f;
#pragma unroll
                for (int q = 0; q < count; ++q)
#pragma unroll
                    for (int i = 0; i < VW; ++i) z = fmaf(x[q].v[i], 0.f, z);
                exact = __ballot(z != 0.f) == 0;
            }
            if (exact) add(std::true_type{});
            else add(std::false_type{});
        };
        int left = __popcll(any);
        for (; left >= U; left -= U) pop(std::integral_constant<int, U>{});
        if constexpr (U > 4) if (left & 4) pop(std::integral_constant<int, 4>{});
        if constexpr (U > 2) if (left & 2) pop(std::integral_constant<int, 2>{});
        if (left & 1) pop(std::integral_constant<int, 1>{});
    }
    if (!act) return;
#pragma unroll
    for (int t = 0; t < TB; ++t)
        if (t0 + t < ntr) *reinterpret_cast<V *>(Y + t * ys) = acc[t];
}

// seg[row * (nseg + 1) + s] = entries of the row (from its first) with base
// column below s * width, s = 0 .. nseg.
__global__ void k_chan_segments(const int64_t *__restrict__ rp, const int32_t *__restrict__ ecol,
                                int64_t n, int nseg, int64_t width, uint32_t *__restrict__ seg) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * (nseg + 1)) return;
    const int64_t row = i / (nseg + 1), s = i - row * (nseg + 1);
    const int64_t beg = rp[row];
    int64_t lo = beg, hi = rp[row + 1];
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if ((ecol[mid] >> 4) < s * width) lo = mid + 1; else hi = mid;
    }
    seg[i] = (uint32_t)(lo - beg);
}

// Propagation step of every trial: out_t = a_t Z_t + b_t D^-1 A Z_t + c1_t E1_t
// + c2_t E2_t and accum_t += e_t out_t, coefficients coef[5 t + {0..4}].  The
// trials' n x ld blocks are zs apart.  L lanes (float4 each) per gathered row,
// 64 / L gathered rows per step of the wave, U steps in flight.
template <int L, int U, bool TM>
__global__ void __launch_bounds__(256)
k_gspmm_batch(const int64_t *__restrict__ rp, const int32_t *__restrict__ col, int64_t n,
              int ntr, int k, int64_t ld, int64_t zs, const float *__restrict__ Z,
              float *__restrict__ out, const float *__restrict__ E1, const float *__restrict__ E2,
              float *__restrict__ accum, const float *__restrict__ coef) {
    constexpr int G = 64 / L;
    const int64_t w = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (w >= n * ntr) return;
    int64_t row;
    int t;
    if (TM) {
        t = (int)(w / n);
        row = w - (int64_t)t * n;
    } else {
        row = w / ntr;
        t = (int)(w - row * ntr);
    }
    const int lane = threadIdx.x & 63;
    const int gi = lane / L, c0 = (lane % L) * 4;
    const bool act = c0 < k;
    const int64_t off = (int64_t)t * zs;
    Z += off;
    const int64_t beg = rp[row], end = rp[row + 1];
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int64_t b0 = beg; b0 < end; b0 += 64) {
        const int64_t idx = b0 + lane;
        const int32_t cj = idx < end ? col[idx] : 0;
        const int cnt = (int)min((int64_t)64, end - b0);
        for (int t0 = 0; t0 < cnt; t0 += U * G) {
            int32_t j[U];
            float4 x[U];
#pragma unroll
            for (int q = 0; q < U; ++q) j[q] = __shfl(cj, (t0 + gi + q * G) & 63, 64);
#pragma unroll
            for (int q = 0; q < U; ++q)
                x[q] = (act && t0 + gi + q * G < cnt)
                           ? *reinterpret_cast<const float4 *>(Z + (int64_t)j[q] * ld + c0)
                           : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int q = 0; q < U; ++q) {
                s.x += x[q].x;
                s.y += x[q].y;
                s.z += x[q].z;
                s.w += x[q].w;
            }
        }
    }
#pragma unroll
    for (int o = L; o < 64; o <<= 1) {
        s.x += __shfl_xor(s.x, o, 64);
        s.y += __shfl_xor(s.y, o, 64);
        s.z += __shfl_xor(s.z, o, 64);
        s.w += __shfl_xor(s.w, o, 64);
    }
    if (gi != 0 || !act) return;
    const float *cf = coef + 5 * t;
    const float a = cf[0], b = cf[1], c1 = cf[2], c2 = cf[3], e = cf[4];
    const float inv = end > beg ? 1.0f / (float)(end - beg) : 0.0f;
    const int64_t o = off + row * ld + c0;
    const float4 z = *reinterpret_cast<const float4 *>(Z + row * ld + c0);
    float4 r = make_float4(a * z.x + b * (inv * s.x), a * z.y + b * (inv * s.y),
                           a * z.z + b * (inv * s.z), a * z.w + b * (inv * s.w));
    if (E1) {
        const float4 q = *reinterpret_cast<const float4 *>(E1 + o);
        r.x += c1 * q.x; r.y += c1 * q.y; r.z += c1 * q.z; r.w += c1 * q.w;
    }
    if (E2) {
        const float4 q = *reinterpret_cast<const float4 *>(E2 + o);
        r.x += c2 * q.x; r.y += c2 * q.y; r.z += c2 * q.z; r.w += c2 * q.w;
    }
    *reinterpret_cast<float4 *>(out + o) = r;
    if (accum) {
        float4 q = *reinterpret_cast<const float4 *>(accum + o);
        q.x += e * r.x; q.y += e * r.y; q.z += e * r.z; q.w += e * r.w;
        *reinterpret_cast<float4 *>(accum + o) = q;
    }
}

// y = alpha[i / per] x over `count` floats (alpha per trial block of `per`)
__global__ void k_scale_blocks(const float *__restrict__ x, float *__restrict__ y, int64_t count,
                               int64_t per, const float *__restrict__ alpha) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) y[i] = alpha[i / per] * x[i];
}

__global__ void k_fill_u32(uint32_t *__restrict__ p, int64_t count, uint32_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

}  // namespace

lne_status split_channels(lne_ctx *ctx, const lne_csr *ext, int T, lne_csr *st, Buf &chan) {
    const int64_t n = ext->n_rows;
    Buf cnt(ctx), srp(ctx);
    LNE_TRY(alloc(ctx, cnt, sizeof(uint32_t) * (size_t)(n + 1)));
    LNE_TRY(alloc(ctx, srp, sizeof(int64_t) * (size_t)(n + 1)));
    const unsigned grid = grid_of(n * 64, 256);
    {
        Launch L(ctx, "split_channels");
        k_split_count<<<grid, 256, 0, ctx->stream>>>(ext->row_ptr, ext->col, n, cnt.as<uint32_t>());
    }
    LNE_TRY(check_launch(ctx, "split_channels"));
    LNE_TRY(scan_u32(ctx, cnt.as<uint32_t>(), srp.as<uint64_t>(), n));
    int64_t nnz = 0;
    LNE_HIP(ctx, hipMemcpyAsync(&nnz, srp.as<int64_t>() + n, 8, hipMemcpyDeviceToHost, ctx->stream));
    LNE_HIP(ctx, hipStreamSynchronize(ctx->stream));
    Buf scol(ctx);
    LNE_TRY(alloc(ctx, scol, sizeof(int32_t) * (size_t)(nnz ? nnz : 1)));
    LNE_TRY(alloc(ctx, chan, sizeof(uint64_t) * (size_t)(nnz ? nnz : 1) * T));
    LNE_HIP(ctx, hipMemsetAsync(chan.p, 0, sizeof(uint64_t) * (size_t)(nnz ? nnz : 1) * T,
                                ctx->stream));
    {
        Launch L(ctx, "split_channels");
        k_split_fill<<<grid, 256, 0, ctx->stream>>>(ext->row_ptr, ext->col,
                                                    (const uint64_t *)ext->val, n,
                                                    srp.as<int64_t>(), scol.as<int32_t>(),
                                                    chan.as<uint64_t>(), T);
    }
    LNE_TRY(check_launch(ctx, "split_channels"));
    st->n_rows = n;
    st->n_cols = n;
    st->nnz = nnz;
    st->row_ptr = (int64_t *)srp.detach();
    st->col = (int32_t *)scol.detach();
    st->val = nullptr;
    st->val_type = LNE_F32;
    return LNE_OK;
}

lne_status trial_values(lne_ctx *ctx, const Graph *g, const lne_csr *st, const uint64_t *chan,
                        int T, const double *s_dev, int ntr, double scale, float *vals) {
    if (st->n_rows > 0) {
        Launch L(ctx, "trial_values");
        k_trial_values<<<grid_of(st->n_rows * 64, 256), 256, 0, ctx->stream>>>(
            g->row_ptr, st->row_ptr, st->col, chan, T, st->n_rows, s_dev, ntr, scale, vals);
    }
    return check_launch(ctx, "trial_values");
}

lne_status norm_channels(lne_ctx *ctx, lne_csr *ext, const Graph *g, double scale) {
    if (ext->val_type != LNE_U64) return fail(ctx, LNE_EINVAL, "norm_channels: counts expected");
    if (ext->n_rows > 0) {
        Launch L(ctx, "norm_channels");
        k_norm_chan<<<grid_of(ext->n_rows * 64, 256), 256, 0, ctx->stream>>>(
            ext->row_ptr, ext->col, g->row_ptr, ext->n_rows, scale, (uint64_t *)ext->val);
    }
    LNE_TRY(check_launch(ctx, "norm_channels"));
    ext->val_type = LNE_F64;
    return LNE_OK;
}

int chan_ranges(int64_t n, int64_t nnz, int64_t ldx) {
    const int64_t bytes = n * ldx * (int64_t)sizeof(float);
    const int64_t ranges = ceil_div(bytes, kChanRangeBytes);
    if (n == 0 || ranges < 2 || ranges > 4096 || nnz >= n * (int64_t)UINT32_MAX) return 1;
    return nnz / (n * ranges) >= kChanMinRun ? (int)ranges : 1;
}

lne_status chan_segments(lne_ctx *ctx, const lne_csr *ext, int nseg, uint32_t *seg) {
    const int64_t n = ext->n_rows;
    if (n == 0) return LNE_OK;
    {
        Launch L(ctx, "chan_segments");
        k_chan_segments<<<grid_of(n * (nseg + 1), 256), 256, 0, ctx->stream>>>(
            ext->row_ptr, ext->col, n, nseg, ceil_div(n, nseg), seg);
    }
    return check_launch(ctx, "chan_segments");
}

// Whether tb trials of one operand (n rows of k floats) share its gather.  A wave
// then takes a row for all of them, which leaves too few waves on few rows, and a
// small operand is in the caches for a gather each.  Shared and not, us, by
// rows x columns (some 1,500 entries a row):
//                  2 trials       4 trials        8 trials
//    2,000 x 144    227   155     (5: 538  298)    591   448
//    4,000 x  48    236   177      320   286       527   505
//    6,000 x  48    321   279      457   464       760   843
//    8,000 x  48    401   370      617   655     1,000 1,208
//    4,000 x 144    291   279      427   500       757   904
//    6,000 x 144    419   477      658   830     1,181 1,501
//    8,000 x 144    539   647      871 1,163     1,543 2,194
//   16,000 x 144  1,083 1,502    1,696 2,786     3,144 5,279
static bool chan_shared_pays(int64_t n, int k, int tb) {
    return n >= 4096 && n * k * tb * (int64_t)sizeof(float) >= 3 << 21;
}

lne_status spmm_chan(lne_ctx *ctx, const lne_csr *ext, const uint32_t *seg, int nseg, bool shared,
                     int ntr, const double *coef, const float *X, int64_t ldx, int64_t xs,
                     float *Y, int64_t ldy, int64_t ys, int k, int variant) {
    if (ext->val_type != LNE_F64)
        return fail(ctx, LNE_EINVAL, "spmm_chan: channel weights must be normalised");
    if (k % 4 || k > 256 || ldx % 4 || ldy % 4 || xs % 4 || ys % 4 || (uintptr_t)X % 16 ||
        (uintptr_t)Y % 16)
        return fail(ctx, LNE_EINVAL, "spmm_chan: k <= 256, k %% 4 == 0 and 16-byte aligned rows");
    if (ldx >= (int64_t)1 << 32 || (shared && xs != 0) || variant < 0 ||
        variant >= kSpmmChanVariants)
        return fail(ctx, LNE_EINVAL, "spmm_chan: ldx, a shared operand's stride or variant %d",
                    variant);
    const int64_t n = ext->n_rows;
    if (n == 0 || ntr == 0) return LNE_OK;
    for (int t0 = 0; t0 < ntr;) {
        // groups of eight, four and two trials, then a single one.  An incomplete
        // group costs what a full one does: at 8,000 x 144 five trials in a group
        // of eight took 1,545 us, as four and one 1,219, but three as two and one
        // 887 against 852 in a group of four, and six as four and two 1,410
        const int left = ntr - t0;
        const int group = left >= 7 ? 8 : left >= 3 ? 4 : left;
        const int tb = shared && chan_shared_pays(n, k, group) ? group : 1;
        const int nt = tb == 1 ? left : left >= 8 ? left / 8 * 8 : std::min(tb, left);
        // a gather for eight by whole rows, where ranges are short (chan_ranges
        // has the times of both)
        const uint32_t *sg = tb == 8 && ext->nnz < kChanSharedRun * n * nseg ? nullptr : seg;
        const double *cf = coef + 16 * t0;
        const float *Xt = X + t0 * xs;
        float *Yt = Y + t0 * ys;
        for (int s = 0; s < (sg ? nseg : 1); ++s) {
            Launch L(ctx, "spmm_chan");
#define LNE_CS(TB, VW, U, TM)                                                                  \
        k_chan_seg<TB, VW, U, TM><<<grid_of(n * ceil_div(nt, TB), 4), 256, 0, ctx->stream>>>(  \
            ext->row_ptr, sg, nseg, s, ext->col, (const double *)ext->val, n, nt, cf, Xt, ldx, \
            xs, Yt, ldy, ys, k, s == 0 ? 1 : 0)
#define LNE_CV(VW)                                                                             \
        do {                                                                                   \
            if (tb == 2) LNE_CS(2, VW, 4, true);                                               \
            else if (tb == 4) LNE_CS(4, VW, 4, true);                                          \
            else if (tb == 8) LNE_CS(8, VW, 4, true);                                          \
            else if (sg || variant == 0) LNE_CS(1, VW, 4, true);                              \
            else if (variant == 1) LNE_CS(1, VW, 2, true);                                     \
            else if (variant == 2) LNE_CS(1, VW, 8, true);                                     \
            else if (variant == 3) LNE_CS(1, VW, 4, false);                                    \
            else if (variant == 4) LNE_CS(1, VW, 2, false);                                    \
            else LNE_CS(1, VW, 8, false);                                                      \
        } while (0)
            if (k <= 64) LNE_CV(1);
            else if (k <= 128) LNE_CV(2);
            else if (k <= 192 && k % 3 == 0) LNE_CV(3);
            else LNE_CV(4);
#undef LNE_CV
#undef LNE_CS
        }
        t0 += nt;
    }
    return check_launch(ctx, "spmm_chan");
}

lne_status gspmm_batch(lne_ctx *ctx, const Graph *g, int ntr, int k, int64_t ld, int64_t zs,
                       const float *Z, float *out, const float *E1, const float *E2, float *acc,
                       const float *coef, int variant) {
    if (k % 4 || k > 256 || ld % 4 || zs % 4 || (uintptr_t)Z % 16 || (uintptr_t)out % 16)
        return fail(ctx, LNE_EINVAL, "gspmm_batch: k <= 256, k %% 4 == 0 and aligned rows");
    const int64_t n = g->n;
    if (n == 0 || ntr == 0) return LNE_OK;
    const unsigned grid = grid_of(n * ntr * 64, 256);
    const bool wide = k > 128;
    {
        Launch L(ctx, "graph_spmm_batch");
#define LNE_GB(LL, UU, TMM)                                                                  \
    k_gspmm_batch<LL, UU, TMM><<<grid, 256, 0, ctx->stream>>>(g->row_ptr, g->col, n, ntr, k, \
                                                             ld, zs, Z, out, E1, E2, acc,   \
                                                             coef)
        switch (variant * 2 + (wide ? 1 : 0)) {
            case 0: LNE_GB(32, 4, true); break;
            case 1: LNE_GB(64, 4, true); break;
            case 2: LNE_GB(32, 2, true); break;
            case 3: LNE_GB(64, 2, true); break;
            case 4: LNE_GB(32, 4, false); break;
            case 5: LNE_GB(64, 4, false); break;
            case 6: LNE_GB(32, 2, false); break;
            case 7: LNE_GB(64, 2, false); break;
            default: return fail(ctx, LNE_EINVAL, "gspmm_batch: variant %d", variant);
        }
#undef LNE_GB
    }
    return check_launch(ctx, "graph_spmm_batch");
}

lne_status scale_blocks(lne_ctx *ctx, const float *x, float *y, int64_t count, int64_t per,
                        const float *alpha) {
    if (count == 0) return LNE_OK;
    {
        Launch L(ctx, "scale_blocks");
        k_scale_blocks<<<grid_of(count, 256), 256, 0, ctx->stream>>>(x, y, count, per, alpha);
    }
    return check_launch(ctx, "scale_blocks");
}

lne_status fill_u32(lne_ctx *ctx, void *p, int64_t count, uint32_t v) {
    if (count == 0) return LNE_OK;
    {
        Launch L(ctx, "fill");
        k_fill_u32<<<grid_of(count, 256), 256, 0, ctx->stream>>>((uint32_t *)p, count, v);
    }
    return check_launch(ctx, "fill");
}

}  // namespace lne
