// Dense steps of the fast randomized SVD (section 4.2): tall-skinny Gram
// products C = Y^T Y and projections Y W on MFMA, and the small FP64 solves
// (Cholesky with inverse, symmetric eigen-decomposition) of eigSVD and
// CholeskyQR2, each in one workgroup so the whole chain stays on the device.
//
// MFMA use (gfx950, 64-lane waves, 16 x 16 output tiles):
//   FP64 / FP32 data: v_mfma_f64_16x16x4f64 (FP32 inputs widened to FP64)
//   BF16 data:        v_mfma_f32_16x16x32_bf16 with FP32 accumulation
// Operand lane layout of a 16 x 16 x K step: lane l supplies A[l % 16][k-block
// l / 16] and B[k-block l / 16][l % 16].  Accumulator value i of lane l is
// column l % 16 of the output tile, row 4 (l / 16) + i for the FP32/BF16
// forms but row l / 16 + 4 i for the FP64 form (checked by a lane probe).
#include <mutex>
#include <type_traits>

#include "common.hpp"

namespace lne {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

template <class T> __device__ __forceinline__ double to_d(T x) { return (double)x; }
template <> __device__ __forceinline__ double to_d<__bf16>(__bf16 x) { return (double)(float)x; }

__device__ __forceinline__ void upper_tile(int t, int nt, int &I, int &J) {
    I = 0;
    while (t >= nt - I) { t -= nt - I; ++I; }
    J = I + t;
}

// ---------------------------------------------------------------- Gram FP64
constexpr int kGramRows = 16;
constexpr int kGramThreads = 512;

// Widest padded k whose upper 16 x 16 tiles fit SPLIT blocks of 8 waves x
// MAXT tiles.
constexpr int gram_kp_max(int maxt, int split) {
    int nt = 1;
    while ((nt + 1) * (nt + 2) / 2 <= 8 * maxt * split) ++nt;
    return 16 * nt;
}

// Two LDS tiles of kGramRows rows: the next tile's loads are issued into
// registers before the matrix-core steps of the current one and stored to
// the other buffer after them, so one block barrier per tile separates them.
// Small tiles (16 rows) keep a block's LDS small enough for three blocks per
// CU at k' <= 144 and two at k' <= 272, so that other blocks' matrix-core
// steps cover each block's barrier and tile turnaround.  SPLIT blocks
// (blockIdx.z) share a row range and split its upper output tiles, so that a
// wide k keeps its accumulators in registers.
template <class YT, int MAXT, int SPLIT>
__global__ void __launch_bounds__(kGramThreads, MAXT <= 6 ? 6 : 2)
k_gram64(const YT *__restrict__ Y, int64_t n, int k, int64_t ld, int KP, int64_t rows_per_wg,
         double *__restrict__ part, const int32_t *__restrict__ skip, int64_t ys) {
    Y += (int64_t)blockIdx.y * ys;
    part += (int64_t)blockIdx.y * gridDim.x * KP * KP;
    if (skip) skip += kFlagStride * blockIdx.y;
    if (skip && *skip == 0) return;
    constexpr int KPM = gram_kp_max(MAXT, SPLIT);
    __shared__ double tile[2][kGramRows * KPM];       // kGramRows x KP each
    // the wave index as a scalar, so that the tile indices below are too
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = KP / 16, ntu = nt * (nt + 1) / 2;
    // a block takes a contiguous run of the upper tiles in row order and each
    // wave a contiguous part of it, so that a wave's tiles mostly share their
    // tile row and its A fragment is read from LDS once per step
    const int cb = (ntu + SPLIT - 1) / SPLIT, cw = (cb + 7) / 8;
    const int t0 = (int)blockIdx.z * cb + w * cw, t1 = min(min(ntu, ((int)blockIdx.z + 1) * cb),
                                                           t0 + cw);
    int TI[MAXT], TJ[MAXT];
    v4d acc[MAXT];
#pragma unroll
    for (int s = 0; s < MAXT; ++s) {
        acc[s] = (v4d){0, 0, 0, 0};
        const int t = t0 + s;
        if (t < t1) upper_tile(t, nt, TI[s], TJ[s]); else { TI[s] = TJ[s] = -1; }
    }
    const int64_t r_begin = (int64_t)blockIdx.x * rows_per_wg;
    const int64_t r_end = min(n, r_begin + rows_per_wg);
    const int kr = lane >> 4, kc = lane & 15;
    // a tile is loaded by whole rows: wave w takes rows w, w + 8, ... and its
    // lanes the row's columns 64 apart (no index division per element)
    constexpr int RPW = kGramRows / 8, CPR = (KPM + 63) / 64, NLD = RPW * CPR;
    auto gload = [&](int64_t r0, YT v[NLD]) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int64_t row = r0 + w + 8 * i;
#pragma unroll
            for (int j = 0; j < CPR; ++j) {
                const int c = lane + 64 * j;
                v[i * CPR + j] = (row < r_end && c < k) ? Y[row * ld + c] : (YT)0;
            }
        }
    };
    auto lstore = [&](int buf, const YT v[NLD]) {
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
            for (int j = 0; j < CPR; ++j) {
                const int c = lane + 64 * j;
                if (c < KP) tile[buf][(w + 8 * i) * KP + c] = to_d(v[i * CPR + j]);
            }
    };
auto mfma_tile = [&](int cur) {
#pragma unroll
        for (int kk = 0; kk < kGramRows; kk += 4) {
            const double *trow = tile[cur] + (kk + kr) * KP + kc;
            double a = 0.0;
#pragma unroll
            for (int s = 0; s < MAXT; ++s) {
                if (TI[s] >= 0) {
                    if (s == 0 || TI[s] != TI[s - 1]) a = trow[16 * TI[s]];
                    const double b = trow[16 * TJ[s]];
                    acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[s], 0, 0, 0);
                }
            }
        }
    };
    YT v[NLD];
    if (r_begin < r_end) {
        gload(r_begin, v);
        lstore(0, v);
    }
    __syncthreads();
    int cur = 0;
    for (int64_t r0 = r_begin; r0 < r_end; r0 += kGramRows, cur ^= 1) {
        const bool more = r0 + kGramRows < r_end;
        if (more) gload(r0 + kGramRows, v);
        mfma_tile(cur);
        if (more) lstore(cur ^ 1, v);
        __syncthreads();
    }
    double *P = part + (int64_t)blockIdx.x * KP * KP;
#pragma unroll
    for (int s = 0; s < MAXT; ++s) {
        if (TI[s] < 0) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            P[(int64_t)(16 * TI[s] + kr + 4 * i) * KP + 16 * TJ[s] + kc] = acc[s][i];
    }
}

// ---------------------------------------------------------------- Gram BF16
constexpr int kTS = 40;   // LDS row stride (bf16) of the transposed tile: 80 B

constexpr int kBR = 128;           // rows per BF16 Gram tile (four MFMA k-steps)
constexpr int kTS2 = kBR + 8;      // LDS row stride (bf16) of the transposed tile: 272 B
constexpr int kGBThreads = 1024;   // BF16 Gram block: sixteen waves
constexpr int kGBWaves = kGBThreads / 64;

// Loads 8 consecutive bf16 of row `row` from column c (zero beyond k or r_end).
__device__ __forceinline__ v8bf load8(const __bf16 *__restrict__ Y, int64_t ld, int64_t row,
                                      int64_t r_end, int c, int k, bool vec) {
    v8bf v;
    if (row < r_end && vec && c + 8 <= k) {
        v = *reinterpret_cast<const v8bf *>(Y + row * ld + c);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            v[i] = (row < r_end && c + i < k) ? Y[row * ld + c + i] : (__bf16)0.0f;
    }
    return v;
}

// BF16 Gram: 128-row tiles read with 16-byte loads (consecutive lanes take
// consecutive rows of one 8-column chunk, so the transposed LDS writes do not
// conflict), four 16 x 16 x 32 MFMA steps per tile and output tile.  Sixteen
// waves share a block, so each holds few output tiles and one block per CU
// has a whole 128-row tile (68 KB at k' = 266) of loads in flight; the
// transposed tile lives in dynamic LDS (KP x kTS2 bf16).  The per-block sums
// are FP32 (the accumulators' own type).  vec: rows are 16-byte aligned
// (ld % 8 == 0, aligned base).
template <int MAXT>
__global__ void __launch_bounds__(kGBThreads)
k_gram_bf16(const __bf16 *__restrict__ Y, int64_t n, int k, int64_t ld, int KP,
            int64_t rows_per_wg, float *__restrict__ part, const int32_t *__restrict__ skip,
            int64_t ys, int vec) {
    Y += (int64_t)blockIdx.y * ys;
    part += (int64_t)blockIdx.y * gridDim.x * KP * KP;
    if (skip) skip += kFlagStride * blockIdx.y;
    if (skip && *skip == 0) return;
    extern __shared__ __attribute__((aligned(16))) __bf16 tt[];   // KP x kTS2, transposed
    // the wave index as a scalar, so that the tile indices below are too
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = KP / 16, ntu = nt * (nt + 1) / 2;
    int TI[MAXT], TJ[MAXT];
    v4f acc[MAXT];
#pragma unroll
    for (int s = 0; s < MAXT; ++s) {
        acc[s] = (v4f){0, 0, 0, 0};
        const int t = w + kGBWaves * s;
        if (t < ntu) upper_tile(t, nt, TI[s], TJ[s]); else { TI[s] = TJ[s] = -1; }
    }
    const int64_t r_begin = (int64_t)blockIdx.x * rows_per_wg;
    const int64_t r_end = min(n, r_begin + rows_per_wg);
    const int kr = lane >> 4, kc = lane & 15;
    const int nch = KP / 8;
    // the next tile's 16-byte chunks are requested into registers before the
    // matrix-core steps of the current one and written to LDS after them
    constexpr int NP = (288 / 8 * kBR + kGBThreads - 1) / kGBThreads;
    v8bf pv[NP];
    auto fetch = [&](int64_t r0) {
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int idx = tid + u * kGBThreads;
            if (idx < nch * kBR) pv[u] = load8(Y, ld, r0 + idx % kBR, r_end, (idx / kBR) * 8, k, vec != 0);
        }
    };
    if (r_begin < r_end) fetch(r_begin);
    for (int64_t r0 = r_begin; r0 < r_end; r0 += kBR) {
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int idx = tid + u * kGBThreads;
            if (idx < nch * kBR) {
                const int rr = idx % kBR, c = (idx / kBR) * 8;
#pragma unroll
                for (int i = 0; i < 8; ++i) tt[(c + i) * kTS2 + rr] = pv[u][i];
            }
        }
        __syncthreads();
        if (r0 + kBR < r_end) fetch(r0 + kBR);
#pragma unroll
        for (int ks = 0; ks < kBR; ks += 32) {
#pragma unroll
            for (int s = 0; s < MAXT; ++s) {
                if (TI[s] >= 0) {
                    const v8bf a =
                        *reinterpret_cast<const v8bf *>(tt + (16 * TI[s] + kc) * kTS2 + ks + 8 * kr);
                    const v8bf b =
                        *reinterpret_cast<const v8bf *>(tt + (16 * TJ[s] + kc) * kTS2 + ks + 8 * kr);
                    acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[s], 0, 0, 0);
                }
            }
        }
        __syncthreads();
    }
    float *P = part + (int64_t)blockIdx.x * KP * KP;
#pragma unroll
    for (int s = 0; s < MAXT; ++s) {
        if (TI[s] < 0) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            P[(int64_t)(16 * TI[s] + 4 * kr + i) * KP + 16 * TJ[s] + kc] = acc[s][i];
    }
}

// G = sum of the per-workgroup upper partial Grams, mirrored.  A block sums
// 64 consecutive entries (a, b), b >= a, of one row a: its sixteen waves take
// the workgroups w = q mod 16, eight running sums each, combined in a fixed
// order (the result does not depend on the launch).  Bound by latency: up to
// 768 strided partials an entry, so as many of them in flight as possible (four
// waves with two sums each took 32 us at k = 16 and 34 us at 138; this takes 8
// and 16).
constexpr int kRedThreads = 1024;
constexpr int kRedWaves = kRedThreads / 64;
constexpr int kRedSums = 8;
template <class PT>
__global__ void __launch_bounds__(kRedThreads)
k_gram_reduce(const PT *__restrict__ part, int nwg, int KP, int k, double *__restrict__ G,
              const int32_t *__restrict__ skip) {
    part += (int64_t)blockIdx.y * nwg * KP * KP;
    G += (int64_t)blockIdx.y * k * k;
    if (skip) skip += kFlagStride * blockIdx.y;
    if (skip && *skip == 0) return;
    const int nbc = (k + 63) / 64;
    const int a = (int)blockIdx.x / nbc, b = ((int)blockIdx.x % nbc) * 64 + (threadIdx.x & 63);
    const int q = threadIdx.x >> 6;
    __shared__ double sums[kRedWaves][64];
    double s[kRedSums];
#pragma unroll
    for (int u = 0; u < kRedSums; ++u) s[u] = 0.0;
    if (b >= a && b < k) {
        const PT *pa = part + (int64_t)a * KP + b;
        const int64_t step = (int64_t)KP * KP;
        int w = q;
        for (; w + kRedWaves * (kRedSums - 1) < nwg; w += kRedWaves * kRedSums)
#pragma unroll
            for (int u = 0; u < kRedSums; ++u) s[u] += (double)pa[(w + kRedWaves * u) * step];
#pragma unroll
        for (int u = 0; u < kRedSums; ++u)
            if (w + kRedWaves * u < nwg) s[u] += (double)pa[(w + kRedWaves * u) * step];
    }
#pragma unroll
    for (int h = kRedSums / 2; h > 0; h >>= 1)
#pragma unroll
        for (int u = 0; u < h; ++u) s[u] += s[u + h];
    sums[q][threadIdx.x & 63] = s[0];
    __syncthreads();
    if (q == 0 && b >= a && b < k) {
        const int l = threadIdx.x;
        double g = 0.0;
#pragma unroll
        for (int u = 0; u < kRedWaves; ++u) g += sums[u][l];
        G[(int64_t)a * k + b] = g;
        G[(int64_t)b * k + a] = g;
    }
}

// ---------------------------------------------------------------- projection
constexpr int kProjRows = 128;
constexpr int kProjThreads = 512;
constexpr int kKC = 16;           // K chunk (FP64 path)

// Four consecutive elements of row `row` from column c as doubles (zero
// beyond k or n); vec: 16-byte (FP32) or 2 x 16-byte (FP64) loads allowed.
template <class YT>
__device__ __forceinline__ void load4d(const YT *__restrict__ Y, int64_t ld, int64_t row,
                                       int64_t n, int c, int k, bool vec, double out[4]) {
    if (row < n && vec && c + 4 <= k) {
        if constexpr (sizeof(YT) == 4) {
            const float4 v = *reinterpret_cast<const float4 *>(Y + row * ld + c);
            out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
        } else {
            const double2 v0 = *reinterpret_cast<const double2 *>(Y + row * ld + c);
            const double2 v1 = *reinterpret_cast<const double2 *>(Y + row * ld + c + 2);
            out[0] = v0.x; out[1] = v0.y; out[2] = v1.x; out[3] = v1.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            out[i] = (row < n && c + i < k) ? to_d(Y[row * ld + c + i]) : 0.0;
    }
}

// FP64-MFMA projection out = Y W.  Each 16 x 16 x 4 step sums over four k;
// lane group kr takes k = k0 + 4 kr + t in step t, so a lane's A operands for
// a 16-wide k chunk are four consecutive elements of its row, read with one
// vector load; the chunk of W is staged in LDS.
template <class YT, class OT, int MAXJ>
__global__ void __launch_bounds__(kProjThreads, MAXJ <= 3 ? 6 : 2)
k_proj64(const YT *__restrict__ Y, int64_t ldy, int64_t n, int kin,
         const double *__restrict__ W, int kout, OT *__restrict__ out, int64_t ldo,
         const int32_t *__restrict__ skip, int64_t ys, int64_t ws, int64_t os, int vec) {
    Y += (int64_t)blockIdx.y * ys;
    W += (int64_t)blockIdx.y * ws;
    out += (int64_t)blockIdx.y * os;
    if (skip) skip += kFlagStride * blockIdx.y;
    if (skip && *skip == 0) return;
    // two W chunks in LDS: chunk i + 1 is loaded into registers before the
    // matrix-core steps of chunk i and stored to the other buffer after them,
    // so one block barrier per chunk separates the two
    constexpr int KPo = 16 * MAXJ;
    constexpr int kWn = (kKC * KPo + kProjThreads - 1) / kProjThreads;
    __shared__ double Ws[2][kKC * KPo];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // blockIdx.z takes output column tiles jz .. jz + MAXJ - 1
    const int jz = (int)blockIdx.z * MAXJ, cz = 16 * jz;
    const int ntout = min(MAXJ, (kout + 15) / 16 - jz);
    const int64_t r0 = (int64_t)blockIdx.x * kProjRows;
    const int kr = lane >> 4, kc = lane & 15;
    const int64_t arow = r0 + 16 * w + kc;
    auto wload = [&](int k0, double wr[kWn]) {
#pragma unroll
        for (int u = 0; u < kWn; ++u) {
            const int idx = tid + u * kProjThreads;
            const int rr = idx / KPo, c = idx - rr * KPo;
            const int krow = k0 + rr;
            wr[u] = (idx < kKC * KPo && krow < kin && cz + c < kout)
                        ? W[(int64_t)krow * kout + cz + c]
                        : 0.0;
        }
    };
    auto wstore = [&](int buf, const double wr[kWn]) {
#pragma unroll
        for (int u = 0; u < kWn; ++u) {
            const int idx = tid + u * kProjThreads;
            if (idx < kKC * KPo) Ws[buf][idx] = wr[u];
        }
    };
    v4d acc[MAXJ];
#pragma unroll
    for (int J = 0; J < MAXJ; ++J) acc[J] = (v4d){0, 0, 0, 0};
    double wr[kWn], a4[4];
    wload(0, wr);
    load4d<YT>(Y, ldy, arow, n, 4 * kr, kin, vec != 0, a4);
    wstore(0, wr);
    __syncthreads();
    for (int k0 = 0, cur = 0; k0 < kin; k0 += kKC, cur ^= 1) {
        const bool more = k0 + kKC < kin;
        double a4n[4];
        if (more) {
            wload(k0 + kKC, wr);
            load4d<YT>(Y, ldy, arow, n, k0 + kKC + 4 * kr, kin, vec != 0, a4n);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
            for (int J = 0; J < MAXJ; ++J) {
                if (J < ntout) {
                    const double b = Ws[cur][(4 * kr + t) * KPo + 16 * J + kc];
                    acc[J] = __builtin_amdgcn_mfma_f64_16x16x4f64(a4[t], b, acc[J], 0, 0, 0);
                }
            }
        }
        if (more) {
            wstore(cur ^ 1, wr);
#pragma unroll
            for (int i = 0; i < 4; ++i) a4[i] = a4n[i];
        }
        __syncthreads();
    }
#pragma unroll
    for (int J = 0; J < MAXJ; ++J) {
        if (J >= ntout) continue;
        const int c = cz + 16 * J + kc;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t row = r0 + 16 * w + kr + 4 * i;
            if (row < n && c < kout) out[row * ldo + c] = (OT)acc[J][i];
        }
    }
}

// FP64-MFMA projection Y <- Y W in place for an upper triangular W (the
// orthonormaliser's R^-1; k x k).  Output tile J sums the 16-column chunks up
// to J only, half the matrix steps of a full product.  A block keeps the tiles
// of W behind its MJ output column tiles in LDS for the whole launch and its
// eight waves walk 16-row strips of Y on their own, with no barrier between
// them; a strip's operands come straight from memory, ahead of their use.
// Lane group kr takes k = 4 kr + t of a chunk in step t (four consecutive
// elements of its row); W's tiles are stored in the order the lanes read them
// (two steps per 16-byte read, no bank conflicts).
// Outputs that need more tiles than fit in LDS go MJ column tiles at a time,
// the last columns first: a wave writes only rows it has read, and no group
// reads a column that an earlier one has written.  (Splitting the columns
// over blocks, as the full product does, lets one block overwrite what
// another still reads.)
// 2 10^6 x 138 FP32: 1605 us as a full product with a barrier and the waits
// for W and Y per chunk, 1566 with half its matrix steps left out, 858 so (46
// GFLOP in 16 x 16 x 4 steps: 68% of the matrix rate; 1 TB/s of operands each
// way).
constexpr int kTriThreads = 512;
constexpr int kTriWaves = kTriThreads / 64;
constexpr int kTriMaxTiles = 76;   // 2 KB tiles of W in LDS (152 of 160 KB)

// Tiles of W behind output tiles [J0, J0 + MJ), J0 >= 0.
constexpr int tri_tiles(int J0, int MJ) { return J0 * MJ + MJ * (MJ + 1) / 2; }
// Tile (chunk q, output tile J0 + j), j >= q - J0.  The first columns' group
// may start before column 0 (J0 < 0; its tiles j < -J0 are none).
template <int MJ>
__device__ __forceinline__ int tri_index(int q, int J0, int j) {
    const int d = q - J0;
    if (d <= 0) return q * MJ + j;
    return (J0 > 0 ? J0 * MJ : 0) + d * MJ - d * (d - 1) / 2 + (j - d);
}

// Elements c .. c + 3 of a row (zero from column k on); whole: all inside,
// and 16-byte aligned.
template <class T>
__device__ __forceinline__ void load4(const T *row, int c, int k, bool whole, T out[4]) {
    if (whole) {
        if constexpr (sizeof(T) == 4) {
            const float4 v = *reinterpret_cast<const float4 *>(row + c);
            out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
        } else {
            const double2 v0 = *reinterpret_cast<const double2 *>(row + c);
            const double2 v1 = *reinterpret_cast<const double2 *>(row + c + 2);
            out[0] = v0.x; out[1] = v0.y; out[2] = v1.x; out[3] = v1.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const T x = row[min(c + i, k - 1)];
            out[i] = c + i < k ? x : (T)0;
        }
    }
}

// steps(J0 + d, u[d], d) for d = 0 .. MJ - 1 with d a constant in each.
template <int MJ, int D = 0, class U, class F>
__device__ __forceinline__ void tri_steps(const U &u, int J0, F &&steps) {
    if constexpr (D < MJ) {
        if (J0 + D >= 0) steps(J0 + D, u[D], std::integral_constant<int, D>{});
        tri_steps<MJ, D + 1>(u, J0, steps);
    }
}

template <class T, int MJ>
__global__ void __launch_bounds__(kTriThreads)
k_proj_tri(T *Y, int64_t ld, int64_t n, int k, const double *__restrict__ W,
           const int32_t *__restrict__ skip, int64_t ys, int64_t ws, int vec) {
    Y += (int64_t)blockIdx.y * ys;
    W += (int64_t)blockIdx.y * ws;
    if (skip) skip += kFlagStride * blockIdx.y;
    if (skip && *skip == 0) return;
    extern __shared__ __attribute__((aligned(16))) double wl[];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kr = lane >> 4, kc = lane & 15;
    const int64_t strips = (n + 15) / 16;
    for (int J0 = (k + 15) / 16 - MJ; J0 > -MJ; J0 -= MJ) {
        __syncthreads();
        for (int e = tid; e < (J0 + MJ) * MJ * 256; e += kTriThreads) {
            const int r = (e >> 4) & 15, c = e & 15, tile = e >> 8;
            const int q = tile / MJ, j = tile - q * MJ;
            if (J0 + j < q) continue;
            const int row = 16 * q + r, col = 16 * (J0 + j) + c;
            const double x = row < k && col < k ? W[(int64_t)row * k + col] : 0.0;
            // step t = r & 3 of lane 16 (r / 4) + c, two steps side by side
            wl[tri_index<MJ>(q, J0, j) * 256 + ((r & 3) >> 1) * 128 + ((r >> 2) * 16 + c) * 2 +
               (r & 1)] = x;
        }
        __syncthreads();
        for (int64_t st = blockIdx.x + (int64_t)gridDim.x * w; st < strips;
             st += (int64_t)gridDim.x * kTriWaves) {
            const int64_t r0 = 16 * st;
            const T *yr = Y + min(r0 + kc, n - 1) * ld;
            v4d acc[MJ];
#pragma unroll
            for (int J = 0; J < MJ; ++J) acc[J] = (v4d){0, 0, 0, 0};
            auto load = [&](int q, T (&v)[4]) {
                load4<T>(yr, 16 * q + 4 * kr, k, vec && 16 * q + 16 <= k, v);
            };
            // chunk q from output tile j0 on
            auto steps = [&](int q, const T (&v)[4], auto j0) {
                const double *t0 = wl + tri_index<MJ>(q, J0, j0) * 256 + lane * 2;
#pragma unroll
                for (int J = j0; J < MJ; ++J) {
                    const double2 b01 = *reinterpret_cast<const double2 *>(t0 + (J - j0) * 256);
                    const double2 b23 = *reinterpret_cast<const double2 *>(t0 + (J - j0) * 256 + 128);
                    acc[J] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)v[0], b01.x, acc[J], 0, 0, 0);
                    acc[J] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)v[1], b01.y, acc[J], 0, 0, 0);
                    acc[J] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)v[2], b23.x, acc[J], 0, 0, 0);
                    acc[J] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)v[3], b23.y, acc[J], 0, 0, 0);
                }
                // (else the tiles of later chunks are read ahead, and spill)
                __builtin_amdgcn_sched_barrier(0);
            };
            // chunks before the group's own: every tile, two chunks at a time
            // with the next two requested first
            if (J0 > 0) {
                T v[2][4], vn[2][4];
                load(0, v[0]);
                load(min(1, J0 - 1), v[1]);
                for (int q = 0; q < J0; q += 2) {
                    load(min(q + 2, J0 - 1), vn[0]);
                    load(min(q + 3, J0 - 1), vn[1]);
                    steps(q, v[0], std::integral_constant<int, 0>{});
                    if (q + 1 < J0) steps(q + 1, v[1], std::integral_constant<int, 0>{});
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        v[0][i] = vn[0][i];
                        v[1][i] = vn[1][i];
                    }
                }
            }
            // the group's own chunks J0 + d: tiles d .. MJ - 1
            T u[MJ][4];
#pragma unroll
            for (int d = 0; d < MJ; ++d)
                if (J0 + d >= 0) load(J0 + d, u[d]);
            tri_steps<MJ>(u, J0, steps);
#pragma unroll
            for (int J = 0; J < MJ; ++J) {
                const int c = 16 * (J0 + J) + kc;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t row = r0 + kr + 4 * i;
                    if (row < n && c >= 0 && c < k) Y[row * ld + c] = (T)acc[J][i];
                }
            }
        }
    }
}

// BF16 projection: each lane reads its A operand (8 consecutive k of one
// row) straight from memory with one 16-byte load; the 32-k slice of W^T is
// staged in LDS, double-buffered: the next step's operand and W slice are
// requested into registers before the current step's matrix-core steps and
// the slice is stored to the other buffer after them, one barrier per step.
// TRI: W is upper triangular, and output tile J takes the steps up to its own
// columns only (out may be Y: a wave reads its rows before it writes them).
// The full product took 459 us at 10^6 x 266, this 390.
template <class OT, int MAXJ, bool TRI>
__global__ void __launch_bounds__(kProjThreads)
k_proj_bf16(const __bf16 *__restrict__ Y, int64_t ldy, int64_t n, int kin,
            const __bf16 *__restrict__ Wt, int ldw, int kout, OT *__restrict__ out,
            int64_t ldo, const int32_t *__restrict__ skip, int64_t ys, int64_t os, int vec) {
    Y += (int64_t)blockIdx.y * ys;
    Wt += (int64_t)blockIdx.y * kout * ldw;
    out += (int64_t)blockIdx.y * os;
    if (skip) skip += kFlagStride * blockIdx.y;
    if (skip && *skip == 0) return;
    __shared__ __attribute__((aligned(16))) __bf16 Ws[2][16 * MAXJ * kTS];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int ntout = (kout + 15) / 16;
    const int64_t r0 = (int64_t)blockIdx.x * kProjRows;
    const int kr = lane >> 4, kc = lane & 15;
    const int64_t arow = r0 + 16 * w + kc;
    // a thread's share of one W slice: 16 MAXJ columns x 4 chunks of 8 k
    constexpr int NW = (16 * MAXJ * 4 + kProjThreads - 1) / kProjThreads;
    auto wload = [&](int k0, v8bf v[NW]) {
#pragma unroll
        for (int u = 0; u < NW; ++u) {
            const int idx = tid + u * kProjThreads;
            const int c = idx >> 2, kcol = k0 + (idx & 3) * 8;
            if (idx >= 16 * MAXJ * 4) continue;
            if (c < kout && kcol + 8 <= kin) {
                v[u] = *reinterpret_cast<const v8bf *>(Wt + (int64_t)c * ldw + kcol);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    v[u][i] = (c < kout && kcol + i < kin) ? Wt[(int64_t)c * ldw + kcol + i]
                                                           : (__bf16)0.0f;
            }
        }
    };
    auto wstore = [&](int buf, const v8bf v[NW]) {
#pragma unroll
        for (int u = 0; u < NW; ++u) {
            const int idx = tid + u * kProjThreads;
            if (idx < 16 * MAXJ * 4)
                *reinterpret_cast<v8bf *>(Ws[buf] + (idx >> 2) * kTS + (idx & 3) * 8) = v[u];
        }
    };
    v4f acc[MAXJ];
#pragma unroll
    for (int J = 0; J < MAXJ; ++J) acc[J] = (v4f){0, 0, 0, 0};
    v8bf wv[NW];
    wload(0, wv);
    wstore(0, wv);
    v8bf a = load8(Y, ldy, arow, n, 8 * kr, kin, vec != 0);
    __syncthreads();
    int cur = 0;
    for (int k0 = 0; k0 < kin; k0 += 32, cur ^= 1) {
        const bool more = k0 + 32 < kin;
        v8bf an = a;
        if (more) {
            an = load8(Y, ldy, arow, n, k0 + 32 + 8 * kr, kin, vec != 0);
            wload(k0 + 32, wv);
        }
#pragma unroll
        for (int J = 0; J < MAXJ; ++J) {
            if (J < ntout && (!TRI || 16 * J + 15 >= k0)) {
                const v8bf b =
                    *reinterpret_cast<const v8bf *>(Ws[cur] + (16 * J + kc) * kTS + 8 * kr);
                acc[J] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[J], 0, 0, 0);
            }
        }
        if (more) wstore(cur ^ 1, wv);
        __syncthreads();
        a = an;
    }
#pragma unroll
    for (int J = 0; J < MAXJ; ++J) {
        if (J >= ntout) continue;
        const int c = 16 * J + kc;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t row = r0 + 16 * w + 4 * kr + i;
            if (row < n && c < kout) out[row * ldo + c] = (OT)acc[J][i];
        }
    }
}

__global__ void k_w_to_bf16t(const double *__restrict__ W, int kin, int kout,
                             __bf16 *__restrict__ Wt, int ldw, int64_t ws) {
    W += (int64_t)blockIdx.y * ws;
    Wt += (int64_t)blockIdx.y * kout * ldw;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)kin * kout) return;
    const int i = (int)(t / kout), c = (int)(t % kout);
    Wt[(int64_t)c * ldw + i] = (__bf16)(float)W[t];
}

// ---------------------------------------------------------------- Cholesky
constexpr int kSolveThreads = 1024;
constexpr int kEigMaxK = 288;   // widest k of the Cholesky and eigen-solver kernels

// A double moved between lanes by a DPP pattern (both halves).
template <int CTRL>
__device__ inline double dpp_d(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

__device__ inline double readlane_d(double x, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                            __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Bounds-checked doubles of a k x k matrix: zero outside the rows and columns,
// stores there dropped (out_if turns an index past k into an offset outside
// the buffer by arithmetic; a guard written as a condition becomes a branch
// and a wait per access).
typedef unsigned v2u __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int out_if(int i, int k) { return ((k - 1 - i) >> 31) & 0x7ffffff0; }
__device__ __forceinline__ __amdgpu_buffer_rsrc_t square_buf(double *p, int k) {
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, 8 * k * k, 0x00020000);
}
__device__ __forceinline__ double buf_d(__amdgpu_buffer_rsrc_t r, int off) {
    const v2u v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
    return __hiloint2double((int)v[1], (int)v[0]);
}
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, int off, double x) {
    const v2u v = (v2u){(unsigned)__double2loint(x), (unsigned)__double2hiint(x)};
    __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, 0);
}

// Cholesky of the Gram G = R^T R (a shifted retry if a pivot fails) and W =
// R^-1 by one workgroup, in 16 x 16 tiles on FP64 matrix instructions.
//
// Factorisation, right-looking over tile rows j.  The tiles above the diagonal
// live in the registers of waves 1..7 (accumulator layout: row l / 16 + 4 i,
// column l % 16), dealt in row order; the diagonal ones in LDS.
//   - Each tile T of row j becomes X = R_jj^-T T: M T with M the block's
//     explicit inverse, then one correction X += M (T - R_jj^T X), which
//     leaves the residual of a substitution.  X goes to LDS (the panel) and G.
//   - Every tile (I, J), I > j, takes the panel's rank-16 update in four
//     matrix steps; wave 0 updates and factors the next diagonal block first,
//     then updates the others.
// The diagonal block is factored by one wave with a column per lane (the
// multipliers by lane reads); lanes 16..31 carry the identity through the same
// row operations, so they end with M.
// Inverse: W_JJ = M^T; then each wave takes whole tile columns J and forms
// W_IJ = -W_II sum_{L > I} R_IL W_LJ for I = J-1 .. 0 with no barrier: an
// accumulator tile is the next product's B operand as it stands (term
// l / 16 + 4 t in step t).
// Bound by the 16-step chain of each diagonal block (a reciprocal square root
// and a lane read per step, with the two barriers of a panel) and, at the
// widest, by the FP64 matrix rate of one CU.  A column at a time with three
// barriers each took 3580 us at k = 266, 459 us at 138 and 76 us at 42; this
// takes 348, 77 and 17 us (the width sets the tiles a wave keeps: MAXT).
constexpr int kCholThreads = 512;
constexpr int kCholWaves = kCholThreads / 64;
constexpr int kCholGroup = 4;   // products of the inverse whose operands are loaded together
// LDS row stride of the panel: an odd number of tiles, so that two of its rows
// read by one half wave sit in different banks.
__host__ __device__ constexpr int panel_ld(int nt) { return 16 * (nt | 1); }
constexpr int kBlk = 16 * 17;   // a diagonal block in LDS, rows 17 apart
inline size_t chol_lds(int nt) {
    return sizeof(double) * (size_t)(16 * panel_ld(nt) + (nt + 1) * kBlk);
}

template <int MAXT>
__global__ void __launch_bounds__(kCholThreads)
k_chol_inv(double *Gb, int k, double *Wb, int32_t *__restrict__ status,
           int32_t *__restrict__ shifted, int64_t n_rows, const int32_t *__restrict__ skip,
           int32_t *__restrict__ run_next) {
    extern __shared__ double lds_c[];
    __shared__ double diag0[kEigMaxK];
    __shared__ int bad;
    __shared__ double sigma_s;
    double *G = Gb + (int64_t)blockIdx.x * k * k;
    double *W = Wb + (int64_t)blockIdx.x * k * k;
    {
        const int64_t b = blockIdx.x;
        status += kFlagStride * b;
        shifted += kFlagStride * b;
        if (skip) skip += kFlagStride * b;
        if (run_next) run_next += kFlagStride * b;
    }
    if (skip && *skip == 0) {
        if (run_next && threadIdx.x == 0) *run_next = 0;
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int kr = lane >> 4, kc = lane & 15;
    const int nt = (k + 15) / 16, PL = panel_ld(nt);
    double *P = lds_c, *Dg = P + 16 * PL, *M = Dg + nt * kBlk;
    const __amdgpu_buffer_rsrc_t gb = square_buf(G, k), wb = square_buf(W, k);
    for (int i = tid; i < k; i += kCholThreads) diag0[i] = G[(int64_t)i * k + i];
    if (tid == 0) bad = 0;
    // this wave's tiles: every seventh one above the diagonal, in row order
    int TI[MAXT], TJ[MAXT];
#pragma unroll
    for (int s = 0; s < MAXT; ++s) {
        int t = (w - 1) + (kCholWaves - 1) * s, I = 0;
        if (w == 0) t = nt * nt;
        while (I < nt && t >= nt - 1 - I) { t -= nt - 1 - I; ++I; }
        TI[s] = I < nt ? I : nt;   // nt: no tile
        TJ[s] = I < nt ? I + 1 + t : nt;
    }
    __syncthreads();
    // factors diagonal block j (wave 0): Dg[j] becomes R_jj (zeros below), M
    auto factor = [&](int j, bool sh) {
        double *D = Dg + j * kBlk;
        double a[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const double x = D[i * 17 + kc];
            a[i] = (lane & 16) ? (i == kc ? 1.0 : 0.0) : x;
        }
        // lane i: the least pivot i may be, whether it was
        const int gi = 16 * j + kc;
        const double least = sh || gi >= k ? 0.0 : 1e-14 * diag0[gi < k ? gi : 0];
        int good = 1;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const double piv = readlane_d(a[q], q);
            const int fine = (int)(a[q] > least) & (int)(a[q] > 0.0) & (int)(a[q] < INFINITY);
            good &= fine | (int)(lane != q);
            // 1 / sqrt by the hardware estimate and two Newton steps
            const double h = 0.5 * piv;
            double y = __builtin_amdgcn_rsq(piv);
            y = y * fma(-h * y, y, 1.5);
            y = y * fma(-h * y, y, 1.5);
            a[q] *= y;
#pragma unroll
            for (int i = q + 1; i < 16; ++i) a[i] = fma(-readlane_d(a[q], i), a[q], a[i]);
            __builtin_amdgcn_sched_barrier(0);   // (else the lane reads pile up and spill)
        }
        if (lane < 32) {
            double *o = (lane < 16 ? D : M) + kc;
#pragma unroll
            for (int i = 0; i < 16; ++i) o[i * 17] = lane >= 16 || i <= kc ? a[i] : 0.0;
        }
        if (__any(!good) && lane == 0) bad = 1;
    };
    v4d acc[MAXT];
    bool ok = false, sh = false;
    for (int attempt = 0; attempt < 2 && !ok; ++attempt) {
        // (lane and panel indices are made opaque where a loop starts, so that
        // the addresses in it are formed there instead of being kept, one per
        // tile, from outside: they would take more registers than the tiles)
        asm volatile("" : "+v"(kr), "+v"(kc));
        sh = attempt == 1;
        double sigma = 0.0;
        if (sh) {
            // shifted retry: G + sigma I, sigma = 11 (n k + k (k + 1)) u trace(G)
            if (tid == 0) {
                double t = 0.0;
                for (int i = 0; i < k; ++i) t += diag0[i];
                sigma_s = 11.0 * ((double)n_rows * k + (double)k * (k + 1)) *
                          1.1102230246251565e-16 * t;
                bad = 0;
            }
            __syncthreads();
            sigma = sigma_s;
        }
        // the retry reads G's lower triangle (R is written to the upper one)
        const int rs = sh ? 1 : k, cs = sh ? k : 1;
#pragma unroll
        for (int s = 0; s < MAXT; ++s) {
            const int c = 16 * TJ[s] + kc, out = out_if(c, k);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[s][i] = buf_d(gb, 8 * ((16 * TI[s] + kr + 4 * i) * rs + c * cs) | out);
        }
        // diagonal blocks from the lower triangle and the saved diagonal,
        // identity past k
        for (int e = tid; e < 256 * nt; e += kCholThreads) {
            const int r = (e >> 4) & 15, c = e & 15, r0 = 16 * (e >> 8) + r, c0 = 16 * (e >> 8) + c;
            const int hi = max(r0, c0), lo = min(r0, c0);
            double x = buf_d(gb, 8 * (hi * k + lo) | out_if(hi, k));
            if (r == c) x = r0 < k ? diag0[min(r0, k - 1)] + sigma : 1.0;
            Dg[(e >> 8) * kBlk + r * 17 + c] = x;
        }
        __syncthreads();
        if (w == 0) factor(0, sh);
        __syncthreads();
        int nxt = 0;   // this wave's tiles before nxt are done
        for (int jp = 0; jp < nt && !bad; ++jp) {
            int j = jp;
            asm volatile("" : "+s"(j), "+v"(kr), "+v"(kc));
            if (w == 0) {
                // diagonal block j to G (upper) and W_jj = M^T
                const double *D = Dg + j * kBlk;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = kr + 4 * i, gr = 16 * j + r, gc = 16 * j + kc;
                    const int off = 8 * (gr * k + gc) | out_if(gr, k) | out_if(gc, k);
                    buf_store(gb, off | out_if(r, kc + 1), D[r * 17 + kc]);
                    buf_store(wb, off, r <= kc ? M[kc * 17 + r] : 0.0);
                }
            } else {
                double m[4], l[4];   // A operands M and R_jj^T
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    m[t] = M[kc * 17 + kr + 4 * t];
                    l[t] = Dg[j * kBlk + (kr + 4 * t) * 17 + kc];
                }
#pragma unroll
                for (int s = 0; s < MAXT; ++s) {
                    if (TI[s] != j) continue;
                    nxt = s + 1;
                    const v4d T = acc[s];
                    v4d X = (v4d){0, 0, 0, 0}, r = T;
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        X = __builtin_amdgcn_mfma_f64_16x16x4f64(m[t], T[t], X, 0, 0, 0);
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        r = __builtin_amdgcn_mfma_f64_16x16x4f64(-l[t], X[t], r, 0, 0, 0);
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        X = __builtin_amdgcn_mfma_f64_16x16x4f64(m[t], r[t], X, 0, 0, 0);
                    const int c = 16 * TJ[s] + kc, out = out_if(c, k);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        P[(kr + 4 * i) * PL + c] = X[i];
                        buf_store(gb, 8 * ((16 * j + kr + 4 * i) * k + c) | out, X[i]);
                    }
                }
            }
            __syncthreads();
            if (j + 1 == nt) break;
            if (w == 0) {
                auto update = [&](int t) {
                    double *D = Dg + t * kBlk + kr * 17 + kc;
                    const double *row = P + kr * PL + 16 * t + kc;
                    v4d c;
                    double x[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        c[i] = D[4 * i * 17];
                        x[i] = row[4 * i * PL];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        c = __builtin_amdgcn_mfma_f64_16x16x4f64(-x[i], x[i], c, 0, 0, 0);
#pragma unroll
                    for (int i = 0; i < 4; ++i) D[4 * i * 17] = c[i];
                };
                update(j + 1);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
                __builtin_amdgcn_wave_barrier();
                factor(j + 1, sh);
                for (int t = j + 2; t < nt; ++t) update(t);
            } else {
#pragma unroll
                for (int s = 0; s < MAXT; ++s) {
                    if (s < nxt || TI[s] >= nt) continue;
                    const double *row = P + kr * PL + kc;
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            -row[4 * t * PL + 16 * TI[s]], row[4 * t * PL + 16 * TJ[s]], acc[s], 0,
                            0, 0);
                }
            }
            __syncthreads();
        }
        ok = bad == 0;
        __syncthreads();
    }
    if (tid == 0) {
        if (!ok) *status = 1;
        if (sh) atomicAdd(shifted, 1);
        if (run_next) *run_next = sh ? 1 : 0;
    }
    // zeros below the diagonal of R and W (W_JJ holds its own)
    for (int r = w; r < k; r += kCholWaves)
        for (int c = lane; c < r; c += 64) {
            G[(int64_t)r * k + c] = 0.0;
            if (c < (r & ~15)) W[(int64_t)r * k + c] = 0.0;
        }
    if (!ok) {   // no factor: W = 0, as the status says
        for (int i = tid; i < k * k; i += kCholThreads) W[i] = 0.0;
        return;
    }
    for (int q = 0; kCholWaves * q < nt; ++q) {
        const int J = nt - 1 - (kCholWaves * q + ((q & 1) ? kCholWaves - 1 - w : w));
        if (J < 1) continue;
        const int c = 16 * J + kc, co = out_if(c, k);
        v4d last;   // W_{I+1, J}
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int r = 16 * J + kr + 4 * t;
            last[t] = buf_d(wb, 8 * (r * k + c) | co | out_if(r, k));
        }
        for (int I = J - 1; I >= 0; --I) {
            v4d S = (v4d){0, 0, 0, 0};
            const int arow = (16 * I + kc) * k + kr;   // A operands: row 16 I + kc
            double al[4], d[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int l = 16 * (I + 1) + 4 * t;
                al[t] = buf_d(gb, 8 * (arow + l) | out_if(l + kr, k));
                d[t] = buf_d(wb, 8 * (arow + 16 * I + 4 * t));
            }
            for (int L0 = J; L0 > I + 1; L0 -= kCholGroup) {
                double a[kCholGroup][4], b[kCholGroup][4];
#pragma unroll
                for (int u = 0; u < kCholGroup; ++u) {
                    const int L = L0 - u, gone = out_if(I + 2, L + 1);   // L <= I + 1: zeros
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int l = 16 * L + 4 * t, out = gone | out_if(l + kr, k);
                        a[u][t] = buf_d(gb, 8 * (arow + l) | out);
                        b[u][t] = buf_d(wb, 8 * ((l + kr) * k + c) | co | out);
                    }
                }
#pragma unroll
                for (int u = 0; u < kCholGroup; ++u)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        S = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][t], b[u][t], S, 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
                S = __builtin_amdgcn_mfma_f64_16x16x4f64(al[t], last[t], S, 0, 0, 0);
            last = (v4d){0, 0, 0, 0};
#pragma unroll
            for (int t = 0; t < 4; ++t)
                last = __builtin_amdgcn_mfma_f64_16x16x4f64(-d[t], S[t], last, 0, 0, 0);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                buf_store(wb, 8 * ((16 * I + kr + 4 * t) * k + c) | co, last[t]);
        }
    }
}

// ---------------------------------------------------------------- eigen-solver
// Symmetric eigen-decomposition of a k x k matrix, in three phases: Householder
// reduction to tridiagonal form and the tridiagonal eigen-problem, by one
// workgroup each, and the reflectors applied to its eigenvectors, by a wave for
// each 16 of these:
//  1. k - 2 Householder steps on the matrix scaled to unit size.  Step j
//     reflects the entries of column j below the subdiagonal to zero by H = I -
//     tau v v^T: with x = A[j+1.., j] and beta = -sign(x0) |x|, v = (1, x1 / (x0 -
//     beta), ...) and tau = (beta - x0) / beta.  The trailing block becomes A -
//     v w^T - w v^T with p = tau A v, w = p - (tau/2)(p.v) v (k_tridiag works
//     with u = (x0 - beta) v instead).  v is left in row j (which later steps
//     never touch).
//  2. The tridiagonal matrix (d, e): implicit QL sweeps (Wilkinson's shift)
//     chase the shifted bulge from the bottom of an unreduced block to its
//     top with plane rotations.  One wave computes a sweep's rotations while
//     other waves apply the previous sweep's rotations to the eigenvector
//     rows (two rotation buffers, one block barrier per sweep); each of their
//     lanes owns one component of every eigenvector.  From kEigSplit on, the
//     matrix is first torn in two halves plus a rank-one term (Cuppen), the
//     halves are swept side by side by two waves, and a merge solves the
//     rank-one problem (its comment gives the steps).
//  3. k_eig_back multiplies the halves' eigenvectors by the rank-one
//     problem's and applies the reflectors.
// The eigenvectors of the tridiagonal matrix are kept transposed (row i =
// eigenvector i), so a rotation of eigenvectors (i, i+1) reads two rows; with
// IN_LDS the halves' are in LDS during phase 2, as the sweeps' rotations would
// wait for global memory otherwise (phase 2 at k = 128: 0.97 ms in global
// memory with the slower chain, 0.58 ms now).
constexpr int kEigMaxLds = 144;   // largest k of the LDS variant
constexpr int kZStride = kEigMaxLds / 2;   // LDS rows of a half's eigenvector components
constexpr int kEigSplit = 32;   // tear the tridiagonal matrix from this size on

// What k_sym_eig hands to k_eig_back: rows of eigenvectors of the tridiagonal
// matrix (or of its halves), the rank-one problem's eigenvectors (U, K x K,
// rows k apart), the eigenvalues (before, the diagonal), the reflectors'
// factors, the coupling, the rows of Zt the columns of the result are built
// from, and K.
struct EigWs {
    double *Zt, *U, *eig, *tau, *off;
    int32_t *kept, *K;
};
__host__ __device__ constexpr int64_t eig_ws_one(int64_t k) { return 2 * k * k + 4 * k + 1; }
__device__ __forceinline__ EigWs eig_ws(double *ws, int k, int64_t batch) {
    double *p = ws + batch * eig_ws_one(k), *q = p + 2 * (int64_t)k * k;
    return {p,     p + (int64_t)k * k,        q,
            q + k, q + 2 * k, (int32_t *)(q + 3 * k), (int32_t *)(q + 4 * k)};
}

// Sum over a fully active wave, the same bits in every lane: pairs, quads,
// half rows and rows by DPP (each step adds two equal sums in either order),
// then the four row sums read from lanes 0, 16, 32 and 48.
__device__ inline double wave_sum(double x) {
    x += dpp_d<0xB1>(x);    // quad_perm [1, 0, 3, 2]
    x += dpp_d<0x4E>(x);    // quad_perm [2, 3, 0, 1]
    x += dpp_d<0x141>(x);   // row_half_mirror
    x += dpp_d<0x140>(x);   // row_mirror
    return (readlane_d(x, 0) + readlane_d(x, 16)) + (readlane_d(x, 32) + readlane_d(x, 48));
}

// Largest of a fully active wave's values, in every lane (undefined ones passed
// over).
__device__ inline double wave_max(double x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o, 64));
    return x;
}

// The power of two that brings numbers of largest size m to unit size (or to
// normal numbers, where m is near the type's limits); 1 where none does.
__device__ inline double unit_scale(double m) {
    return m > 0.0 && isfinite(m) ? ldexp(1.0, -min(max(ilogb(m), -1000), 1000)) : 1.0;
}

// Serial QL state of the producing wave.
struct QlState {
    int l = 0;      // eigenvalues 0 .. l-1 have converged
    int iter = 0;   // sweeps spent on eigenvalue l
};

// The rotations of one QL sweep, rows m-1 up to l, by one lane: a serial chain
// that takes the (d, e) pairs from LDS a group of rows ahead of their use and
// writes the new ones and the rotations (cosine, sine, by upper row) as it
// goes.  Bound by the instructions a single wave issues (some 28 a rotation,
// five to six cycles each, 18 for the root's estimate), hence pairs in one
// access, no clamped addresses (up to 2 kChain - 1 rows above l are read and
// not used) and one refined root: 200 cycles a rotation, against 470 with the
// pairs in registers read by lane index and every lane's stores masked.  The
// matrix is scaled to unit size, so f^2 + g^2 is a normal number unless both
// are negligible (below 2^-500), which is where the sweep must deflate instead.
// CHECK = false runs the chain with no branch on that test and returns -2 if
// it failed anywhere (the stored values are then void); CHECK = true returns
// the row at which it deflated, or -1 when the sweep completed.
constexpr int kChain = 4;
template <bool CHECK>
__device__ int ql_chain(int l, int m, double g, double2 *de, double2 *rot) {
    double s = 1.0, c = 1.0, p = 0.0, dn = de[m].x, least = 1.0;
    const double dl = de[l].x;
    auto rotate = [&](int i, double2 x0) {
        const double f = s * x0.y, b = c * x0.y;
        const double x = fma(f, f, g * g);
        least = fmin(least, x);
        // 1/sqrt(x) by the hardware estimate y (to 2^-23) and one cubic step,
        // y (1 + h/2 + 3 h^2 / 8) with h = 1 - x y^2
        const double y = __builtin_amdgcn_rsq(x);
        const double h = fma(-(x * y), y, 1.0);
        const double y1 = fma(y, h * fma(0.375, h, 0.5), y);
        c = g * y1;
        s = f * y1;
        const double gp = dn - p;
        const double r2 = fma(b + b, c, (x0.x - gp) * s);
        p = s * r2;
        g = fma(c, r2, -b);
        de[i + 1] = make_double2(gp + p, x * y1);
        rot[i] = make_double2(c, s);
        dn = x0.x;
    };
    int i = m - 1;
    if constexpr (CHECK) {
        for (; i >= l; --i) {
            const double2 x0 = de[i];
            const double f = s * x0.y;
            if (!(fma(f, f, g * g) >= 0x1p-1000)) {   // both vanished: deflate at i + 1
                de[i + 1] = make_double2(dn - p, 0.0);
                de[m].y = 0.0;
                return i;
            }
            rotate(i, x0);
        }
    } else {
        double2 x0[kChain], x1[kChain];
#pragma unroll
        for (int u = 0; u < kChain; ++u) x0[u] = de[i - u];
        for (; i - 2 * kChain + 1 >= l; i -= 2 * kChain) {
#pragma unroll
            for (int u = 0; u < kChain; ++u) x1[u] = de[i - kChain - u];
#pragma unroll
            for (int u = 0; u < kChain; ++u) rotate(i - u, x0[u]);
#pragma unroll
            for (int u = 0; u < kChain; ++u) x0[u] = de[i - 2 * kChain - u];
#pragma unroll
            for (int u = 0; u < kChain; ++u) rotate(i - kChain - u, x1[u]);
        }
        if (i - kChain + 1 >= l) {
#pragma unroll
            for (int u = 0; u < kChain; ++u) x1[u] = de[i - kChain - u];
#pragma unroll
            for (int u = 0; u < kChain; ++u) rotate(i - u, x0[u]);
#pragma unroll
            for (int u = 0; u < kChain; ++u) x0[u] = x1[u];
            i -= kChain;
        }
#pragma unroll
        for (int u = 0; u < kChain - 1; ++u)
            if (i - u >= l) rotate(i - u, x0[u]);
        if (!(least >= 0x1p-1000) || g != g) return -2;
    }
    de[l] = make_double2(dl - p, g);
    de[m].y = 0.0;
    return -1;
}

// One QL sweep on the pairs de (length-k diagonal and coupling between i and
// i+1, the last 0), run by a whole wave.  Returns false once every eigenvalue
// has converged; else the sweep's rotations are in rot over [*lo, *hi).  Ends
// whatever the values: an undefined coupling or neighbour counts as negligible
// (hence the negated test), and so does the zero of a coupling given up.
template <int R>
__device__ bool ql_sweep(double2 *de, int k, QlState &st, double2 *rot, int *lo, int *hi,
                         int lane) {
    const double eps = 2.220446049250313e-16;
    for (;;) {
        double2 x[R];
        uint64_t split[R];   // couplings that are negligible
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int j = 64 * q + lane;
            x[q] = de[min(j, k - 1)];
            const double dn = de[min(j + 1, k - 1)].x;
            split[q] = __ballot(j < k - 1 && !(fabs(x[q].y) > eps * (fabs(x[q].x) + fabs(dn))));
        }
        // l: the first eigenvalue not yet converged, m: the first negligible
        // coupling at or after it
        int l = st.l, m = 0;
        for (; l < k; ++l) {
            m = k - 1;
#pragma unroll
            for (int q = R - 1; q >= 0; --q) {
                const int from = min(max(l - 64 * q, 0), 64);
                const uint64_t left = from < 64 ? split[q] >> from << from : 0;
                if (left) m = 64 * q + __builtin_ctzll(left);
            }
            if (m != l) break;
        }
        if (l != st.l) {
            st.l = l;
            st.iter = 0;
        }
        if (l >= k) return false;
        if (st.iter++ >= 64) {   // not expected: give up on this coupling
            if (lane == 0) de[l].y = 0.0;
            __builtin_amdgcn_wave_barrier();
            continue;
        }
        int at = 0;
        double g = 0.0;
        if (lane == 0) {
            // shift: the eigenvalue of the leading 2 x 2 block nearer d[l]; the
            // coupling is not negligible, so the quotient is below 2^52
            const double2 xl = de[l];
            g = (de[l + 1].x - xl.x) / (2.0 * xl.y);
            const double r = sqrt(fma(g, g, 1.0));
            g = de[m].x - xl.x + xl.y / (g + (g >= 0.0 ? r : -r));
            at = ql_chain<false>(l, m, g, de, rot);
        }
        __builtin_amdgcn_wave_barrier();
        at = __builtin_amdgcn_readfirstlane(at);
        if (at == -2) {
            // put the sweep's starting values back, then take the checked path
#pragma unroll
            for (int q = 0; q < R; ++q)
                if (64 * q + lane < k) de[64 * q + lane] = x[q];
            __builtin_amdgcn_wave_barrier();
            if (lane == 0) at = ql_chain<true>(l, m, g, de, rot);
            __builtin_amdgcn_wave_barrier();
            at = __builtin_amdgcn_readfirstlane(at);
        }
        *lo = at >= 0 ? at + 1 : l;
        *hi = m;
        if (*lo < *hi) return true;
    }
}

// The rotations hi-1 .. lo of a sweep applied to one component of the
// eigenvectors, rows ld apart at z (row 0), the operands of G rotations read
// ahead of their use.
template <int G>
__device__ void ql_apply(double *z, int ld, const double2 *rot, int lo, int hi) {
    double *p = z + hi * ld;
    double carry = *p;
    auto turn = [&](double *q, double x, double2 f) {   // q: the lower row
        *q = fma(f.x, carry, f.y * x);
        carry = fma(-f.y, carry, f.x * x);
    };
    int i = hi - 1;
    double x[G];
    double2 f[G];
    auto read = [&](int from) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int j = max(from - u, lo);
            x[u] = z[j * ld];
            f[u] = rot[j];
        }
    };
    read(i);
    for (; i - G + 1 >= lo; i -= G, p -= G * ld) {
        double x0[G];
        double2 f0[G];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            x0[u] = x[u];
            f0[u] = f[u];
        }
        read(i - G);
#pragma unroll
        for (int u = 0; u < G; ++u) turn(p - u * ld, x0[u], f0[u]);
    }
#pragma unroll
    for (int u = 0; u < G - 1; ++u)
        if (i - u >= lo) turn(p - u * ld, x[u], f[u]);
    z[lo * ld] = carry;
}

// Phase 1 for k <= 64 C: the matrix in registers, wave w of W holding the
// pairs of rows w + W q, lane l of it columns l + 64 c.  Step j: with x row j, u = x past the
// diagonal, its first entry less beta, and H = I - g u u^T, g = 1 / (beta^2 -
// beta x0), the trailing block becomes A - u w^T - w u^T, w = p - (g/2)(p.u) u,
// p = g A u.  The matrix is scaled by a power of two first (exact; taken back
// in d and e), so that no square overflows and a row whose squares vanish (u
// below 2^-500 of the largest entry) is negligible: it counts as reduced, as g
// would overflow.  The waves' parts of p meet in LDS; every wave forms the same sums
// and its own w, so a step has two block barriers.  Bound by its chain (two
// sums over a wave, a root, a reciprocal, three trips through LDS): with the
// matrix in LDS, read twice and written once a step, and three barriers, 380
// us at k = 128 and 71 at 42; this takes 199 and 46.
constexpr double kSquareLeast = 0x1p-1000;   // least sum of squares of a row not yet reduced
constexpr int kTriDiagThreads = 512;
constexpr int kTriDiagWaves = kTriDiagThreads / 64;
// A block barrier that waits for the wave's LDS accesses only (__syncthreads
// waits for its stores to global memory too, some 1500 cycles a step here).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
template <int C, int W>
__device__ __forceinline__ void tridiag(double *__restrict__ A, int k, const EigWs &out) {
    constexpr int Q = C == 3 ? kEigMaxLds / W : 64 * C / W;
    constexpr int H = Q / 4 * 2;
    __shared__ __align__(16) double row[64 * C], part[W][64 * C], own[W][64 * C];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const __amdgpu_buffer_rsrc_t ab = square_buf(A, k);
    auto held = [&](int q) { return 2 * (w + W * (q / 2)) + q % 2; };   // row of a[q]
    // (the largest entry from a read of its own: with the matrix already held,
    // its registers spill)
    double amax = 0.0;
    for (int i = tid; i < k * k; i += 8 * 64 * W)
#pragma unroll
        for (int u = 0; u < 8; ++u)
            amax = fmax(amax, fabs(buf_d(ab, 8 * (i + 64 * W * u))));   // past the end: zeros
    part[w][lane] = wave_max(amax);
    lds_barrier();
#pragma unroll
    for (int v = 0; v < W; ++v) amax = fmax(amax, part[v][lane]);
    const double unit = readlane_d(unit_scale(amax), 0), back = readlane_d(1.0 / unit, 0);
    double a[Q][C];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int i = held(q), l = lane + 64 * c;
            a[q][c] = unit * buf_d(ab, 8 * (i * k + l) | out_if(i, k) | out_if(l, k));
        }
    // row j to LDS by the wave that holds it
    auto publish = [&](int j) {
        if (w != j / 2 % W) return;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (held(q) == j)
#pragma unroll
                for (int c = 0; c < C; ++c) row[lane + 64 * c] = a[q][c];
    };
    publish(0);
    lds_barrier();
    for (int j = 0; j + 2 < k; ++j) {
        double u[C], sg = 0.0;
        const double x0 = row[j + 1];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int l = lane + 64 * c;
            u[c] = l > j + 1 && l < k ? row[l] : 0.0;
            sg = fma(u[c], u[c], sg);
        }
        sg = wave_sum(sg);
        if (tid == 0) out.eig[j] = row[j] * back;
        if (sg < kSquareLeast) {   // already reduced: H = I
            if (tid == 0) {
                out.off[j] = x0 * back;
                out.tau[j] = 0.0;
            }
            lds_barrier();
        } else {
            const double beta = -copysign(sqrt(fma(x0, x0, sg)), x0), u0 = x0 - beta;
            const double g = -1.0 / (beta * u0);
            // u by rows: zero for rows up to j and past k
            double p[C] = {}, ui[Q];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (lane + 64 * c == j + 1) u[c] = u0;
                own[w][lane + 64 * c] = u[c];
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int q = 0; q < Q; ++q) ui[q] = own[w][held(q)];
            // the first H of a wave's rows only until all waves' are reduced
#pragma unroll
            for (int half = 0; half < 2; ++half)
                if (half || j < 2 * W * (H / 2))
#pragma unroll
                    for (int q = half ? H : 0; q < (half ? Q : H); ++q)
#pragma unroll
                        for (int c = 0; c < C; ++c) p[c] = fma(a[q][c], ui[q], p[c]);
#pragma unroll
            for (int c = 0; c < C; ++c) part[w][lane + 64 * c] = p[c];
            lds_barrier();
            double pu = 0.0;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                double t[W];
#pragma unroll
                for (int v = 0; v < W; ++v) t[v] = part[v][lane + 64 * c];
#pragma unroll
                for (int o = W / 2; o > 0; o /= 2)
#pragma unroll
                    for (int v = 0; v < o; ++v) t[v] += t[v + o];
                p[c] = g * t[0];
                pu = fma(p[c], u[c], pu);
            }
            const double K = 0.5 * g * wave_sum(pu);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                p[c] = fma(-K, u[c], p[c]);
                own[w][lane + 64 * c] = p[c];
            }
            __builtin_amdgcn_wave_barrier();
            double wi[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) wi[q] = own[w][held(q)];
#pragma unroll
            for (int half = 0; half < 2; ++half)
                if (half || j < 2 * W * (H / 2))
#pragma unroll
                    for (int q = half ? H : 0; q < (half ? Q : H); ++q)
#pragma unroll
                        for (int c = 0; c < C; ++c)
                            a[q][c] = fma(-ui[q], p[c], fma(-wi[q], u[c], a[q][c]));
            // the reflector, scaled to a first entry of 1, where k_eig_back reads it
            if (w == j / 2 % W) {
                const double sc = 1.0 / u0;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const int l = lane + 64 * c;
                    if (l > j && l < k) A[(int64_t)j * k + l] = l == j + 1 ? 1.0 : u[c] * sc;
                }
                if (lane == 0) {
                    out.off[j] = beta * back;
                    out.tau[j] = -u0 / beta;
                }
            }
        }
        publish(j + 1);
        lds_barrier();
    }
    if (tid == 0) {
        const int j = max(k - 2, 0);
        out.eig[j] = row[j] * back;
        out.tau[j] = out.tau[k - 1] = 0.0;
        out.off[j] = k >= 2 ? row[k - 1] * back : 0.0;
        out.off[k - 1] = 0.0;
    }
    lds_barrier();
    if (k >= 2) publish(k - 1);
    lds_barrier();
    if (tid == 0) out.eig[k - 1] = row[k - 1] * back;
}
template <int C>
__global__ void __launch_bounds__(kTriDiagThreads)
k_tridiag(double *__restrict__ A, int k, double *__restrict__ ws) {
    tridiag<C, kTriDiagWaves>(A + (int64_t)blockIdx.x * k * k, k, eig_ws(ws, k, blockIdx.x));
}

// Phase 1 for wider matrices, worked on in place in global memory, scaled as
// above.  Per step:
// every wave forms the reflector from row j; threads (row i, part q) sum parts
// of p = tau A v; thread i < m finishes p_i and writes v_i into row j (first
// entry 1); threads (column l, row group g) apply the rank-2 update.  Three
// block barriers per step.
__global__ void __launch_bounds__(kSolveThreads)
k_tridiag_wide(double *__restrict__ A, int k, double *__restrict__ ws) {
    constexpr int MK = kEigMaxK;
    __shared__ double pq[4 * MK];   // P x MK partial sums, then p (row 0) and v (row 1)
    A += (int64_t)blockIdx.x * k * k;
    const EigWs out = eig_ws(ws, k, blockIdx.x);
    const int tid = threadIdx.x, lane = tid & 63;
    constexpr int P = kSolveThreads / MK < 4 ? kSolveThreads / MK : 4;   // parts per row sum
    constexpr int G = kSolveThreads / MK;                                 // row groups
    // (eight reads at a time; past the end: zeros, and no stores)
    const __amdgpu_buffer_rsrc_t ab = square_buf(A, k);
    double amax = 0.0;
    for (int i = tid; i < k * k; i += 8 * kSolveThreads)
#pragma unroll
        for (int u = 0; u < 8; ++u) amax = fmax(amax, fabs(buf_d(ab, 8 * (i + kSolveThreads * u))));
    amax = wave_max(amax);
    if (lane == 0) pq[tid >> 6] = amax;
    __syncthreads();
    for (int v = 0; v < kSolveThreads / 64; ++v) amax = fmax(amax, pq[v]);
    const double unit = unit_scale(amax), back = 1.0 / unit;
    for (int i = tid; i < k * k; i += 8 * kSolveThreads) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = buf_d(ab, 8 * (i + kSolveThreads * u));
#pragma unroll
        for (int u = 0; u < 8; ++u) buf_store(ab, 8 * (i + kSolveThreads * u), unit * x[u]);
    }
    __syncthreads();
    for (int j = 0; j + 2 < k; ++j) {
        const int m = k - j - 1;   // trailing indices j+1 .. k-1
        double *x = A + (int64_t)j * k + j + 1;
        double sg = 0.0;
        for (int l = 1 + lane; l < m; l += 64) sg += x[l] * x[l];
        sg = wave_sum(sg);
        const double x0 = x[0];
        if (tid == 0) out.eig[j] = A[(int64_t)j * k + j] * back;
        if (sg < kSquareLeast) {   // already reduced: H = I
            if (tid == 0) { out.off[j] = x0 * back; out.tau[j] = 0.0; }
            continue;
        }
        const double beta = -copysign(sqrt(x0 * x0 + sg), x0);
        const double tau = (beta - x0) / beta, sc = 1.0 / (x0 - beta);
        if (tid == 0) { out.off[j] = beta * back; out.tau[j] = tau; }
        {
            const int i = tid % MK, q = tid / MK, L = (m + P - 1) / P;
            if (q < P && i < m) {
                // A[j+1+l][j+1+i] = A[j+1+i][j+1+l]: lanes read along a row
                const double *col = A + (int64_t)(j + 1) * k + j + 1 + i;
                const int l1 = m < (q + 1) * L ? m : (q + 1) * L;
                double acc0 = 0.0, acc1 = 0.0;
                int l = q * L;
                if (l == 0) { acc0 = col[0]; l = 1; }
                for (; l + 1 < l1; l += 2) {
                    acc0 += col[(int64_t)l * k] * (x[l] * sc);
                    acc1 += col[(int64_t)(l + 1) * k] * (x[l + 1] * sc);
                }
                if (l < l1) acc0 += col[(int64_t)l * k] * (x[l] * sc);
                pq[q * MK + i] = acc0 + acc1;
            }
        }
        __syncthreads();
        if (tid < m) {
            double ps = 0.0;
            for (int q = 0; q < P; ++q) ps += pq[q * MK + tid];
            const double v = tid == 0 ? 1.0 : x[tid] * sc;
            pq[tid] = tau * ps;
            pq[MK + tid] = v;
            x[tid] = v;
        }
        __syncthreads();
        double pd = 0.0;
        for (int l = lane; l < m; l += 64) pd += pq[l] * pq[MK + l];
        const double K = 0.5 * tau * wave_sum(pd);
        {
            const int l = tid % MK, g = tid / MK;
            if (g < G && l < m) {
                const double vl = pq[MK + l], wl = pq[l] - K * vl;
                double *colp = A + (int64_t)(j + 1) * k + j + 1 + l;
#pragma unroll 4
                for (int i = g; i < m; i += G) {
                    const double vi = pq[MK + i], wi = pq[i] - K * vi;
                    colp[(int64_t)i * k] -= __dadd_rn(__dmul_rn(vi, wl), __dmul_rn(wi, vl));
                }
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        for (int j = k - 2; j < k; ++j) {
            out.eig[j] = A[(int64_t)j * k + j] * back;
            out.tau[j] = 0.0;
        }
        out.off[k - 2] = A[(int64_t)(k - 2) * k + k - 1] * back;
        out.off[k - 1] = 0.0;
    }
}

template <bool IN_LDS, int NT>
__device__ __forceinline__ void tridiag_eig(int k, const EigWs &out) {
    constexpr int MK = IN_LDS ? kEigMaxLds : kEigMaxK;
    extern __shared__ double lds_a[];
    __shared__ double dg[MK], eg[MK];
    __shared__ double2 rot[2 * MK];   // the rotation buffers; after, vectors
    double *buf = (double *)rot;      // of the merge
    __shared__ double2 de_pad[2 * kChain + MK];
    double2 *de = de_pad + 2 * kChain;   // the pairs (d, e) of the sweeps; then
    int *idx = (int *)de_pad;            // merge: order, kept and deflated rows
    __shared__ int s_lo[2][2], s_hi[2][2], s_more[2][2];   // [problem][buffer]
    __shared__ double s_rho, s_unit, s_tol;
    __shared__ int s_K, s_flip, s_finite;
    double *__restrict__ Zt = out.Zt;
    // the wave index as a scalar, so that code under `w == 0` branches as a
    // uniform wave
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    if constexpr (!IN_LDS)
        for (int64_t i = tid; i < (int64_t)k * k; i += NT)
            Zt[i] = (i / k == i % k) ? 1.0 : 0.0;
    for (int i = tid; i < k; i += NT) {
        dg[i] = out.eig[i];
        eg[i] = out.off[i];
    }
    if (tid == 0) s_more[0][0] = s_more[0][1] = s_more[1][0] = s_more[1][1] = 0;
    __syncthreads();

    // ---- 2. eigen-decomposition of the tridiagonal matrix T = (d, e).
    // Wave 0 scales (d, e) by a power of two to unit size (exact).  For
    // k >= kEigSplit, T is torn at h = k/2 into blockdiag(T1, T2) + rho w w^T
    // (w = e_{h-1} + e_h, rho the coupling, taken off d[h-1] and d[h]); waves
    // 0 and 1 run the QL sweeps of T1 and T2 side by side while waves 2..
    // apply each problem's previous sweep to its block of eigenvector rows
    // (component c by thread c; rotation buffer b at rot + MK b, indexed by
    // global row).  The merge below then solves the rank-one problem.  Smaller
    // k: one problem, waves 1.. apply.
    const int h = k >= kEigSplit ? k / 2 : k;
    const int np = h < k ? 2 : 1;
    if constexpr (IN_LDS) {   // the identity, row i of its half's components
        for (int i = tid; i < k * kZStride; i += NT) {
            const int r = i / kZStride, c = i % kZStride;
            lds_a[i] = c == (r >= h ? r - h : r) ? 1.0 : 0.0;
        }
    }
    if (w == 0) {
        double amax = 0.0;
        bool finite = true;
        for (int i = lane; i < k; i += 64) {
            amax = fmax(amax, fmax(fabs(dg[i]), fabs(eg[i])));
            finite &= isfinite(dg[i]) && isfinite(eg[i]);
        }
        const double unit = unit_scale(wave_max(amax));
        // the tear's rank-one term leaves d[h-1] and d[h]
        const double rho = np == 2 ? eg[h - 1] * unit : 0.0;
        for (int i = lane; i < k; i += 64) {
            const bool torn = np == 2 && (i == h - 1 || i == h);
            de[i] = make_double2(torn ? dg[i] * unit - rho : dg[i] * unit,
                                 np == 2 && i == h - 1 ? 0.0 : eg[i] * unit);
        }
        if (lane == 0) {
            s_unit = unit;
            s_rho = rho;
        }
        const bool all_finite = __all(finite);
        if (lane == 0) s_finite = all_finite ? 1 : 0;
    }
    __syncthreads();
    if (!s_finite) {   // no eigenvalues: all of the result is undefined
        for (int i = tid; i < k * k; i += NT) Zt[i] = NAN;
        for (int i = tid; i < k; i += NT) {
            out.eig[i] = NAN;
            out.kept[i] = i;
        }
        if (tid == 0) *out.K = 0;
        return;
    }
    {
        QlState st;
        if (w < np) __builtin_amdgcn_s_setprio(3);   // a chain goes before its SIMD's other waves
        for (int t = 0;; ++t) {
            const int b = t & 1;
            if (w < np) {
                const int base = w == 0 ? 0 : h, n = w == 0 ? h : k - h;
                int lo = 0, hi = 0;
                const bool more = ql_sweep<(MK / 2 + 63) / 64>(de + base, n, st,
                                                              rot + MK * b + base, &lo, &hi, lane);
                if (lane == 0) {
                    s_more[w][b] = more ? 1 : 0;
                    s_lo[w][b] = base + lo;
                    s_hi[w][b] = base + hi;
                }
            }
            const int pb = b ^ 1;
            const int pr = w - np >= (h + 63) / 64 ? 1 : 0;   // whole waves for each half
            const int kk = tid - 64 * (np + (pr ? (h + 63) / 64 : 0));
            if (t > 0 && w >= np && kk < (pr ? k - h : h) && s_more[pr][pb]) {
                const int lo = __builtin_amdgcn_readfirstlane(s_lo[pr][pb]);
                const int hi = __builtin_amdgcn_readfirstlane(s_hi[pr][pb]);
                if constexpr (IN_LDS)
                    ql_apply<4>(lds_a + kk, kZStride, rot + MK * pb, lo, hi);
                else
                    ql_apply<8>(Zt + (pr ? h : 0) + kk, k, rot + MK * pb, lo, hi);
            }
            __syncthreads();
            if (!s_more[0][b] && !s_more[1][b]) break;
        }
        __builtin_amdgcn_s_setprio(0);
        if constexpr (IN_LDS) {
            for (int i = tid; i < k * k; i += NT) {
                const int r = i / k, c = i % k;
                Zt[i] = (r >= h) == (c >= h) ? lds_a[r * kZStride + (c >= h ? c - h : c)] : 0.0;
            }
        }
        for (int i = tid; i < k; i += NT) dg[i] = de[i].x;
        __syncthreads();
    }
    if (np == 1) {
        for (int i = tid; i < k; i += NT) {
            out.eig[i] = dg[i] / s_unit;
            out.kept[i] = i;
        }
        if (tid == 0) *out.K = 0;
    } else {
        // ---- merge: eigenvalues and eigenvectors of D + rho z z^T, D the
        // eigenvalues of T1 and T2, z the rows h-1 / h of their eigenvectors.
        // Deflation (a negligible weight, or two poles whose rotation
        // leaves a negligible coupling), then each root of the secular
        // equation 1 + rho sum z_i^2 / (d_i - lambda) = 0 in its interval
        // between poles, by a bracketed iteration (its distance to the nearer
        // pole kept as (origin, tau) so that differences stay accurate), and
        // weights recomputed from the roots (Gu and Eisenstat) so that the
        // eigenvectors z_i / (d_i - lambda_j) come out orthogonal (column j of
        // U; k_eig_back multiplies).
        int *ord = idx, *kept = idx + MK;
        double *dk = buf, *zk = buf + MK, *tau = buf + 2 * MK, *zh = buf + 3 * MK;
        for (int i = tid; i < k; i += NT)
            eg[i] = i < h ? Zt[(int64_t)i * k + h - 1] : Zt[(int64_t)i * k + h];
        __syncthreads();
        if (w == 0) {
            double zz = 0.0, dmax = 0.0;
            for (int i = lane; i < k; i += 64) {
                zz += eg[i] * eg[i];
                dmax = fmax(dmax, fabs(dg[i]));
            }
            zz = wave_sum(zz);
            dmax = wave_max(dmax);
            if (lane == 0) {
                const double rt = s_rho * zz;
                s_flip = rt < 0.0 ? 1 : 0;
                s_rho = fabs(rt);
                s_tol = 8.0 * 2.220446049250313e-16 * fmax(dmax, fabs(rt));
                zh[0] = zz > 0.0 ? 1.0 / sqrt(zz) : 0.0;
            }
        }
        __syncthreads();
        {
            const double sz = zh[0];
            const bool flip = s_flip != 0;
            for (int i = tid; i < k; i += NT) {
                eg[i] *= sz;
                if (flip) dg[i] = -dg[i];
            }
        }
        __syncthreads();
        // ascending order of the poles (ties by index)
        for (int i = tid; i < k; i += NT) {
            const double di = dg[i];
            int r = 0;
            for (int j = 0; j < k; ++j) r += (dg[j] < di || (dg[j] == di && j < i)) ? 1 : 0;
            ord[r] = i;
        }
        __syncthreads();
        // deflation, in pole order, by wave 0: negligible weights at once;
        // if a pair of the others deflates, all of it one pole after the other
        // (a rotated pair changes what its successor meets)
        if (w == 0) {
            const double rho = s_rho, tol = s_tol;
            int K = 0, nd = 0, prev = -1;
            for (int s0 = 0; s0 < k; s0 += 64) {
                const int i = s0 + lane < k ? ord[s0 + lane] : 0;
                const bool small = rho * fabs(eg[i]) <= tol;
                const uint64_t in = __ballot(s0 + lane < k && !small);
                const uint64_t gone = __ballot(s0 + lane < k && small);
                const uint64_t before = (1ull << lane) - 1;
                if (in >> lane & 1) kept[K + __popcll(in & before)] = i;
                if (gone >> lane & 1) kept[k - 1 - nd - __popcll(gone & before)] = i;
                K += __popcll(in);
                nd += __popcll(gone);
            }
            __builtin_amdgcn_wave_barrier();
            bool pair = false;
            for (int q = lane; q + 1 < K; q += 64) {
                const int ip = kept[q], i = kept[q + 1];
                const double zp = eg[ip], zi = eg[i], r = hypot(zp, zi);
                pair |= fabs(zi / r * (zp / r) * (dg[i] - dg[ip])) <= tol;
            }
            const bool serial = __ballot(pair) != 0;
            if (serial) K = nd = 0;
            for (int sidx = 0; serial && sidx < k; ++sidx) {
                const int i = ord[sidx];
                const double zi = eg[i];
                if (rho * fabs(zi) <= tol) {
                    if (lane == 0) kept[k - 1 - nd] = i;
                    ++nd;
                    continue;
                }
                if (prev >= 0) {
                    const double zp = eg[prev], dp = dg[prev], di = dg[i];
                    const double r = hypot(zp, zi);
                    const double c = zi / r, sn = zp / r;
                    if (fabs(c * sn * (di - dp)) <= tol) {
                        // rotate rows prev, i so that prev's weight vanishes
                        for (int cc = lane; cc < k; cc += 64) {
                            const double a = Zt[(int64_t)prev * k + cc], bb = Zt[(int64_t)i * k + cc];
                            Zt[(int64_t)prev * k + cc] = c * a - sn * bb;
                            Zt[(int64_t)i * k + cc] = sn * a + c * bb;
                        }
                        if (lane == 0) {
                            dg[prev] = c * c * dp + sn * sn * di;
                            dg[i] = sn * sn * dp + c * c * di;
                            eg[i] = r;
                            eg[prev] = 0.0;
                            kept[k - 1 - nd] = prev;
                        }
                        __builtin_amdgcn_wave_barrier();
                        ++nd;
                        prev = i;
                        continue;
                    }
                    if (lane == 0) kept[K] = prev;
                    ++K;
                }
                prev = i;
            }
            if (prev >= 0) {
                if (lane == 0) kept[K] = prev;
                ++K;
            }
            if (lane == 0) s_K = K;
        }
        __syncthreads();
        const int K = s_K;
        const double rho = s_rho;
        for (int j = tid; j < K; j += NT) {
            dk[j] = dg[kept[j]];
            zk[j] = eg[kept[j]];
        }
        __syncthreads();
        // roots: lambda_j in (dk_j, dk_j+1), the last in (dk_K-1, dk_K-1 +
        // rho |z|^2].  Eight lanes per root (partial sums over every eighth
        // pole, summed by DPP).  A step solves the secular function with each
        // side's poles replaced by the next one, value and slopes kept (Li's
        // middle way; the last root: all poles by the last), Newton's if that
        // leaves the bracket, a bisection if that does too.  With Newton's
        // alone, four lanes a root and divisions, and the deflation one pole
        // after the other, the two took 0.26 ms at k = 128, now 0.055 ms.
        constexpr int LR = 8;
        const int sub = tid % LR;
        auto lanes_sum = [](double x) {
            x += dpp_d<0xB1>(x);
            x += dpp_d<0x4E>(x);
            return x + dpp_d<0x141>(x);
        };
        for (int i = tid; i < K; i += NT) zh[i] = rho * zk[i] * zk[i];
        __syncthreads();
        for (int j = tid / LR; j < K; j += NT / LR) {
            // 1 + rho sum z^2 / delta, delta_i = (dk_i - dk_o) - t, and its
            // derivative over the poles up to j and past j
            auto secular = [&](int oo, double tt, double &below, double &above) {
                double f = 0.0, g0 = 0.0, g1 = 0.0;
                const double dko = dk[oo];
                for (int i = sub; i < K; i += LR) {
                    const double x = (dk[i] - dko) - tt;
                    // 1 / x by the hardware estimate and two Newton steps
                    double r = __builtin_amdgcn_rcp(x);
                    r = fma(r, fma(-x, r, 1.0), r);
                    r = fma(r, fma(-x, r, 1.0), r);
                    const double a2 = zh[i] * r, g = a2 * r;
                    f += a2;
                    g0 += i <= j ? g : 0.0;
                    g1 += i <= j ? 0.0 : g;
                }
                below = lanes_sum(g0);
                above = lanes_sum(g1);
                return 1.0 + lanes_sum(f);
            };
            int o;
            double lo, hi, ps, ph;
            const double gap = j < K - 1 ? dk[j + 1] - dk[j] : 0.0;
            if (j < K - 1) {
                if (secular(j, 0.5 * gap, ps, ph) >= 0.0) { o = j; lo = 0.0; hi = 0.5 * gap; }
                else { o = j + 1; lo = -0.5 * gap; hi = 0.0; }
            } else {
                double zz = 0.0;
                for (int i = sub; i < K; i += LR) zz += zh[i];
                o = j; lo = 0.0; hi = lanes_sum(zz);
            }
            double t = 0.5 * (lo + hi);
            for (int it = 0; it < 200; ++it) {
                const double f = secular(o, t, ps, ph);
                if (f == 0.0) break;
                if (f < 0.0) lo = t; else hi = t;
                double tn;
                if (j < K - 1) {
                    const double d0 = (o == j ? 0.0 : -gap) - t, d1 = (o == j ? gap : 0.0) - t;
                    const double c = f - d0 * ps - d1 * ph, b = d0 * d1 * f;
                    const double a = (d0 + d1) * f - d0 * d1 * (ps + ph);
                    const double q = sqrt(fmax(a * a - 4.0 * b * c, 0.0));
                    tn = t + (a <= 0.0 ? (a - q) / (2.0 * c) : 2.0 * b / (a + q));
                } else {
                    tn = t - t * f / (f + t * ps);
                }
                if (!(tn > lo && tn < hi)) tn = t - f / (ps + ph);
                if (!(tn > lo && tn < hi)) tn = 0.5 * (lo + hi);
                const bool done = !(tn > lo && tn < hi) ||
                                  fabs(tn - t) <= 4.440892098500626e-16 * fabs(tn);
                if (!(tn > lo && tn < hi)) break;
                t = tn;
                if (done) break;
            }
            if (sub == 0) {
                ord[j] = o;
                tau[j] = t;
            }
        }
        __syncthreads();
        // recomputed weights: zh_i^2 = prod_j (lambda_j - dk_i) / (rho prod_l!=i (dk_l - dk_i))
        for (int i = tid / LR; i < K; i += NT / LR) {
            auto lmd = [&](int j) { return (dk[ord[j]] - dk[i]) + tau[j]; };   // lambda_j - dk_i
            double P = 1.0;
            for (int j = sub; j < K - 1; j += LR) P *= lmd(j) / (dk[j < i ? j : j + 1] - dk[i]);
            P *= dpp_d<0xB1>(P);
            P *= dpp_d<0x4E>(P);
            P *= dpp_d<0x141>(P);
            P *= lmd(K - 1) / rho;
            if (sub == 0) zh[i] = copysign(sqrt(fmax(P, 0.0)), zk[i]);
        }
        __syncthreads();
        // eigenvectors of the rank-one problem (columns of U), and the new
        // eigenvalues (unscaled, sign restored) next to the deflated ones
        {
            const double sgn = s_flip ? -1.0 : 1.0, un = s_unit;
            for (int j = tid / LR; j < K; j += NT / LR) {
                const double dj = dk[ord[j]], tj = tau[j];
                double nrm = 0.0;
                for (int i = sub; i < K; i += LR) {
                    const double u = zh[i] / ((dk[i] - dj) - tj);
                    out.U[(int64_t)i * k + j] = u;
                    nrm += u * u;
                }
                const double inv = 1.0 / sqrt(lanes_sum(nrm));
                for (int i = sub; i < K; i += LR) out.U[(int64_t)i * k + j] *= inv;
            }
            for (int j = tid; j < k; j += NT) {
                out.eig[j] = sgn * (j < K ? dk[ord[j]] + tau[j] : dg[kept[j]]) / un;
                out.kept[j] = kept[j];
            }
            if (tid == 0) *out.K = K;
        }
    }
}

// The eigenvectors from what k_sym_eig leaves: a wave takes a strip of 16 of
// them, as 16 x 16 accumulator tiles (row = component) it keeps throughout,
//   - forms them: columns c < K sum_r Zt[kept_r] U[r][c], the others Zt[kept_c];
//   - applies the reflectors in blocks of 16, last to first, in the compact
//     form of Schreiber and Van Loan: Z -= V (T (V^T Z)), V the block's
//     reflectors (rows of A, staged in LDS), T upper triangular with T_ii =
//     tau_i and column i above it -tau_i T (V^T v_i).  An accumulator tile is
//     the next product's B operand as it stands (term l / 16 + 4 t in step t);
//   - writes them to V in order of decreasing eigenvalue, and these to lam.
// Four waves share the blocks' T, which they compute first, a block each in
// turn.  Reflectors one at a time by the waves of k_sym_eig, with a sum over
// the wave each, and the sums over kept rows by its threads took 0.37 ms at k =
// 128 and 2.6 ms at 266; this takes 53 and 154 us (6 at 16, where the launch
// costs what it saves), bound by the latency of the chain of blocks.
constexpr int kBackThreads = 256;
constexpr int kBackWaves = kBackThreads / 64;
constexpr int kBackGroup = 3;   // tiles whose operands are read together
__host__ __device__ constexpr int back_ld(int nt) { return 16 * nt + 2; }
inline size_t back_lds(int maxt) {
    return sizeof(double) * (size_t)(maxt * kBlk + 2 * 16 * back_ld(maxt));
}
template <int MAXT, int WAVES>
__device__ __forceinline__ void eig_back(double *__restrict__ A, int k, const EigWs &in,
                                         double *__restrict__ V, double *__restrict__ lam,
                                         int block) {
    static_assert(MAXT % kBackGroup == 0);
    extern __shared__ double lds_a[];
    constexpr int LD = back_ld(MAXT), VB = 16 * LD;
    double *Ts = lds_a, *Vs = lds_a + MAXT * kBlk;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kr = lane >> 4, c16 = lane & 15;
    const int c = 16 * (WAVES * block + w) + c16;   // this lane's eigenvector
    const bool work = c - c16 < k;                  // the wave has a strip
    const int nblk = (k - 2 + 15) / 16;                            // blocks of reflectors
    const __amdgpu_buffer_rsrc_t ab = square_buf(A, k), zb = square_buf(in.Zt, k),
                                 ub = square_buf(in.U, k);
    // entry i of reflector j (rows 0 .. k-3 of A right of the diagonal)
    auto refl = [&](int j, int i) {
        return buf_d(ab, 8 * (j * k + i) | out_if(i, k) | out_if(j, k - 2) | out_if(j, i));
    };

    // T of each block: V^T V by matrix steps, then row c16 of T by its lane
    for (int b = w; b < nblk; b += WAVES) {
        v4d g[kBackGroup] = {};
        for (int I0 = b; I0 * 16 < k; I0 += kBackGroup) {
            double x[kBackGroup][4];
#pragma unroll
            for (int u = 0; u < kBackGroup; ++u)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    x[u][t] = refl(16 * b + c16, 16 * (I0 + u) + kr + 4 * t);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int u = 0; u < kBackGroup; ++u)
                    g[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[u][t], x[u][t], g[u], 0, 0, 0);
        }
        double *T = Ts + b * kBlk;
#pragma unroll
        for (int t = 0; t < 4; ++t) T[(kr + 4 * t) * 17 + c16] = g[0][t] + g[1][t] + g[2][t];
        __builtin_amdgcn_wave_barrier();
        double tr[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const double tau = 16 * b + i < k ? in.tau[16 * b + i] : 0.0;
            double acc = 0.0;
#pragma unroll
            for (int s = 0; s < i; ++s) acc = fma(tr[s], T[s * 17 + i], acc);
            tr[i] = i == c16 ? tau : i > c16 ? -tau * acc : 0.0;
        }
        __builtin_amdgcn_wave_barrier();
        if (kr == 0)
#pragma unroll
            for (int i = 0; i < 16; ++i) T[c16 * 17 + i] = tr[i];
    }

    // the eigenvectors of the tridiagonal matrix
    const int K = *in.K;
    v4d z[MAXT];
    if (work) {
        const int kc = c < k ? in.kept[c] : 0, copied = out_if(c, k) | out_if(K, c + 1);
#pragma unroll
        for (int I = 0; I < MAXT; ++I)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int i = 16 * I + kr + 4 * t;
                z[I][t] = buf_d(zb, 8 * (kc * k + i) | out_if(i, k) | copied);
            }
        // the operands of a step are read two steps ahead, the row indices three
        double x[2][MAXT], u[2];
        auto row = [&](int r) { return in.kept[min(r, k - 1)]; };
        auto read = [&](int h, int r, int kept) {
            const int past = out_if(r, K);
            u[h] = buf_d(ub, 8 * (r * k + c) | past | out_if(c, K));
#pragma unroll
            for (int I = 0; I < MAXT; ++I)
                x[h][I] = buf_d(zb, 8 * (kept * k + 16 * I + c16) | past | out_if(16 * I + c16, k));
        };
        read(0, kr, row(kr));
        read(1, 4 + kr, row(4 + kr));
        int next[2] = {row(8 + kr), row(12 + kr)};
        for (int r0 = 0; r0 < K; r0 += 8) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int I = 0; I < MAXT; ++I)
                    z[I] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[h][I], u[h], z[I], 0, 0, 0);
                read(h, r0 + 4 * h + 8 + kr, next[h]);
                next[h] = row(r0 + 4 * h + 16 + kr);
            }
        }
    }

    // reflectors, block nblk - 1 first
    const int sr = tid >> 4, si = tid & 15;   // staging: row, column of a tile
    const bool stages = w < 4;
    double st[MAXT];
    auto fetch = [&](int b) {
#pragma unroll
        for (int I = 0; I < MAXT; ++I) st[I] = refl(16 * b + sr, 16 * I + si);
    };
    auto store = [&](int b) {
#pragma unroll
        for (int I = 0; I < MAXT; ++I) Vs[(b & 1) * VB + sr * LD + 16 * I + si] = st[I];
    };
    if (stages) {
        fetch(nblk - 1);
        store(nblk - 1);
    }
    __syncthreads();
    for (int b = nblk - 1; b >= 0; --b) {
        if (stages && b > 0) fetch(b - 1);
        const double *v = Vs + (b & 1) * VB, *T = Ts + b * kBlk;
        if (work) {
            v4d p[kBackGroup] = {};
#pragma unroll
            for (int I0 = 0; I0 < MAXT; I0 += kBackGroup) {
                if (I0 + kBackGroup <= b || 16 * I0 >= k) continue;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int u = 0; u < kBackGroup; ++u)
                        p[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            v[c16 * LD + 16 * (I0 + u) + kr + 4 * t], z[I0 + u][t], p[u], 0, 0, 0);
            }
            v4d q = {};
#pragma unroll
            for (int t = 0; t < 4; ++t)
                q = __builtin_amdgcn_mfma_f64_16x16x4f64(T[c16 * 17 + kr + 4 * t],
                                                         -(p[0][t] + p[1][t] + p[2][t]), q, 0, 0, 0);
#pragma unroll
            for (int I0 = 0; I0 < MAXT; I0 += kBackGroup) {
                if (I0 + kBackGroup <= b || 16 * I0 >= k) continue;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int u = 0; u < kBackGroup; ++u)
                        z[I0 + u] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            v[(kr + 4 * t) * LD + 16 * (I0 + u) + c16], q[t], z[I0 + u], 0, 0, 0);
            }
        }
        if (stages && b > 0) store(b - 1);
        __syncthreads();
    }

    // rank by decreasing eigenvalue, ties (and undefined ones) by index; four
    // lanes share a column
    if (!work) return;
    const double lc = c < k ? in.eig[c] : 0.0;
    int rank = 0;
    for (int j = kr; j < k; j += 4) {
        const double lj = in.eig[j];
        rank += lj > lc || (!(lc > lj) && j < c) ? 1 : 0;
    }
    rank += __shfl_xor(rank, 16, 64);
    rank += __shfl_xor(rank, 32, 64);
    if (c >= k) return;
    if (kr == 0) lam[rank] = lc;
#pragma unroll
    for (int I = 0; I < MAXT; ++I)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int i = 16 * I + kr + 4 * t;
            if (i < k) V[(int64_t)i * k + rank] = z[I][t];
        }
}

template <bool IN_LDS>
__global__ void __launch_bounds__(kSolveThreads) k_sym_eig(int k, double *__restrict__ ws) {
    tridiag_eig<IN_LDS, kSolveThreads>(k, eig_ws(ws, k, blockIdx.x));
}

template <int MAXT>
__global__ void __launch_bounds__(kBackThreads, 1)
k_eig_back(double *__restrict__ A, int k, double *__restrict__ ws, double *__restrict__ V,
           double *__restrict__ lam) {
    const int64_t b = blockIdx.y;
    eig_back<MAXT, kBackWaves>(A + b * k * k, k, eig_ws(ws, k, b), V + b * k * k, lam + b * k,
                               (int)blockIdx.x);
}

// All three phases in one launch for matrices that are not torn, whose phases
// are as short as a launch (k = 3: 23 us in three launches, 16 in one, before the
// scaling; k = 16: 103 and 93).
__global__ void __launch_bounds__(kTriDiagThreads)
k_sym_eig_small(double *__restrict__ A, int k, double *__restrict__ ws, double *__restrict__ V,
                double *__restrict__ lam) {
    const int64_t b = blockIdx.x;
    const EigWs w = eig_ws(ws, k, b);
    A += b * k * k;
    tridiag<1, kTriDiagWaves>(A, k, w);
    __syncthreads();
    tridiag_eig<true, kTriDiagThreads>(k, w);
    __syncthreads();
    eig_back<3, kTriDiagWaves>(A, k, w, V + b * k * k, lam + b * k, 0);
}

__global__ void k_eig_weights(const double *__restrict__ V, const double *__restrict__ lam,
                              int k, int kout, double power, double *__restrict__ W,
                              double *__restrict__ S, const int32_t *__restrict__ on) {
    const int64_t b = blockIdx.y;
    V += b * k * k;
    lam += b * k;
    if (W) W += b * k * kout;
    if (S) S += b * kout;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (on && on[b] == 0) {
        // pass-through entry: identity weights
        if (W && t < (int64_t)k * kout) W[t] = (t / kout == t % kout) ? 1.0 : 0.0;
        if (S && t < kout) S[t] = 1.0;
        return;
    }
    const double lmax = lam[0] > 0.0 ? lam[0] : 0.0;
    const double floor_ = (double)k * 2.220446049250313e-16 * lmax;
    if (S && t < kout) {
        const double l = lam[t];
        S[t] = l > floor_ ? sqrt(l) : l != l ? l : 0.0;
    }
    if (W && t < (int64_t)k * kout) {
        const int i = (int)(t / kout), c = (int)(t % kout);
        const double l = lam[c];
        W[t] = l > floor_ ? V[(int64_t)i * k + c] * pow(l, power) : l != l ? l : 0.0;
    }
}

}  // namespace

// ---------------------------------------------------------------- host side
// Lets `fn` use `bytes` of dynamic LDS (above the default 64 KB), once per
// kernel and device (the attribute belongs to the current device's copy of the
// kernel); fails when the device offers less.
static lne_status lds_opt_in(lne_ctx *ctx, const void *fn, size_t bytes) {
    if (bytes <= 64 * 1024) return LNE_OK;
    int dev = 0;
    LNE_HIP(ctx, hipGetDevice(&dev));
    static std::mutex mu;
    static std::map<std::pair<int, const void *>, size_t> done;
    std::lock_guard<std::mutex> lock(mu);
    size_t &have = done[{dev, fn}];
    if (have >= bytes) return LNE_OK;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) !=
        hipSuccess) {
        (void)hipGetLastError();
        return fail(ctx, LNE_EUNSUPPORTED, "%zu bytes of LDS per block are not available", bytes);
    }
    have = bytes;
    return LNE_OK;
}

size_t project_bf16_ws_bytes(int32_t kin, int32_t kout, int32_t nb) {
    return sizeof(__bf16) * (size_t)nb * kout * (((kin + 31) / 32) * 32);
}

lne_status gram(lne_ctx *ctx, const void *Y, int32_t dtype, int64_t n, int32_t k, int64_t ld,
                double *G, const int32_t *skip, int32_t nb, int64_t ys, double *part_ws,
                size_t part_ws_bytes) {
    if (k < 1) return fail(ctx, LNE_EINVAL, "gram: k = %d", k);
    const int KP = ((k + 15) / 16) * 16;
    const int nt = KP / 16, ntu = nt * (nt + 1) / 2;
    const int per_wave = (ntu + 7) / 8;
    if (per_wave > 22) return fail(ctx, LNE_EUNSUPPORTED, "gram: k = %d above 288", k);
    if (nb < 1 || nb > 65535) return fail(ctx, LNE_EINVAL, "gram: batch of %d", nb);
    // BF16: row ranges in whole 128-row tiles, one sixteen-wave block per CU
    const bool bf = dtype == LNE_BF16;
    const int rows_unit = bf ? kBR : kGramRows;
    const int64_t blocks_rows = ceil_div(n > 0 ? n : 1, rows_unit);
    // about 768 (512 for wide k, 256 for BF16) workgroups over the whole
    // batch, one round of three (two, one) blocks per CU, or as many
    // per-workgroup partial sums as a caller's workspace holds
    int64_t target = std::max<int64_t>(1, (bf ? 256 : KP > 160 ? 512 : 768) / nb);
    // per-workgroup sums: FP32 for BF16 data (its accumulators), else FP64
    const size_t part_es = dtype == LNE_BF16 ? sizeof(float) : sizeof(double);
    const size_t part_one = part_es * (size_t)nb * KP * KP;
    if (part_ws) {
        if (part_ws_bytes < part_one)
            return fail(ctx, LNE_EUNSUPPORTED, "gram: workspace of %zu bytes below %zu",
                        part_ws_bytes, part_one);
        target = std::min<int64_t>(target, (int64_t)(part_ws_bytes / part_one));
    }
    const int nwg = (int)std::min<int64_t>(blocks_rows, target);
    const int64_t rows_per_wg = ceil_div(blocks_rows, nwg) * rows_unit;
    Buf part(ctx);
    if (part_ws) part.p = part_ws, part.ctx = nullptr;   // borrowed: never released
    else LNE_TRY(alloc(ctx, part, part_one * nwg));
    const dim3 grid((unsigned)nwg, (unsigned)nb);
    const int vec = ((uintptr_t)Y % 16 == 0 && ld % 8 == 0 && ys % 8 == 0) ? 1 : 0;
    {
        Launch L(ctx, "gram");
        if (bf) {
            const int bpw = (ntu + kGBWaves - 1) / kGBWaves;
            const size_t lds = sizeof(__bf16) * (size_t)KP * kTS2;
#define LNE_GB(MT)                                                                         \
    do {                                                                                   \
        LNE_TRY(lds_opt_in(ctx, (const void *)k_gram_bf16<MT>, lds));                      \
        k_gram_bf16<MT><<<grid, kGBThreads, lds, ctx->stream>>>(                           \
            (const __bf16 *)Y, n, k, ld, KP, rows_per_wg, part.as<float>(), skip, ys, vec); \
    } while (0)
            if (bpw <= 1) LNE_GB(1);
            else if (bpw <= 6) LNE_GB(6);
            else if (bpw <= 10) LNE_GB(10);
            else LNE_GB(12);
#undef LNE_GB
        } else {
#define LNE_G64(T, MT, SP)                                                               \
    k_gram64<T, MT, SP><<<dim3(grid.x, grid.y, SP), kGramThreads, 0, ctx->stream>>>(   \
        (const T *)Y, n, k, ld, KP, rows_per_wg, part.as<double>(), skip, ys)
            if (dtype == LNE_F64) {
                if (per_wave <= 1) LNE_G64(double, 1, 1);
                else if (per_wave <= 6) LNE_G64(double, 6, 1);
                else if (per_wave <= 12) LNE_G64(double, 12, 1);
                else LNE_G64(double, 11, 2);
            } else {
                if (per_wave <= 1) LNE_G64(float, 1, 1);
                else if (per_wave <= 6) LNE_G64(float, 6, 1);
                else if (per_wave <= 12) LNE_G64(float, 12, 1);
                else LNE_G64(float, 11, 2);
            }
#undef LNE_G64
        }
    }
    LNE_TRY(check_launch(ctx, "gram"));
    {
        Launch L(ctx, "gram_reduce");
        const dim3 rgrid((unsigned)(k * ((k + 63) / 64)), (unsigned)nb);
        if (dtype == LNE_BF16)
            k_gram_reduce<float><<<rgrid, kRedThreads, 0, ctx->stream>>>(part.as<float>(), nwg, KP,
                                                                         k, G, skip);
        else
            k_gram_reduce<double><<<rgrid, kRedThreads, 0, ctx->stream>>>(part.as<double>(), nwg,
                                                                          KP, k, G, skip);
    }
    return check_launch(ctx, "gram_reduce");
}

lne_status project(lne_ctx *ctx, const void *Y, int32_t y_t, int64_t ldy, int64_t n,
                   int32_t kin, const double *W, int32_t kout, void *out, int32_t out_t,
                   int64_t ldo, const int32_t *skip, int32_t nb, int64_t ys, int64_t ws,
                   int64_t os, void *wt_ws, bool tri) {
    if (tri && (kin != kout || out_t != y_t || out != Y || ldo != ldy))
        return fail(ctx, LNE_EINVAL, "project: a triangular W is applied in place");
    if (kout > 288 || kin > 288) return fail(ctx, LNE_EUNSUPPORTED, "project: width above 288");
    if (nb < 1 || nb > 65535) return fail(ctx, LNE_EINVAL, "project: batch of %d", nb);
    const dim3 grid(grid_of(n > 0 ? n : 1, kProjRows), (unsigned)nb);
    const int ntout = (kout + 15) / 16;
    if (y_t == LNE_BF16) {
        const int ldw = ((kin + 31) / 32) * 32;
        const int vec = ((uintptr_t)Y % 16 == 0 && ldy % 8 == 0 && ys % 8 == 0) ? 1 : 0;
        Buf wt(ctx);
        // wt_ws (if given) holds project_bf16_ws_bytes(kin, kout, nb)
        if (wt_ws) wt.p = wt_ws, wt.ctx = nullptr;
        else LNE_TRY(alloc(ctx, wt, project_bf16_ws_bytes(kin, kout, nb)));
        {
            Launch L(ctx, "w_to_bf16");
            k_w_to_bf16t<<<dim3(grid_of((int64_t)kin * kout, 256), (unsigned)nb), 256, 0,
                           ctx->stream>>>(W, kin, kout, wt.as<__bf16>(), ldw, ws);
        }
        LNE_TRY(check_launch(ctx, "w_to_bf16"));
        Launch L(ctx, "project");
#define LNE_PB(OT, MJ, TRI)                                                                \
    k_proj_bf16<OT, MJ, TRI><<<grid, kProjThreads, 0, ctx->stream>>>(                      \
        (const __bf16 *)Y, ldy, n, kin, wt.as<__bf16>(), ldw, kout, (OT *)out, ldo, skip, ys, os, \
        vec)
#define LNE_PBJ(OT, TRI)                                                                   \
    do {                                                                                   \
        if (ntout <= 3) LNE_PB(OT, 3, TRI);                                                \
        else if (ntout <= 9) LNE_PB(OT, 9, TRI);                                           \
        else LNE_PB(OT, 18, TRI);                                                          \
    } while (0)
        if (out_t == LNE_BF16 && tri) {
            LNE_PBJ(__bf16, true);
        } else if (out_t == LNE_BF16) {
            LNE_PBJ(__bf16, false);
        } else if (out_t == LNE_F32) {
            LNE_PBJ(float, false);
        } else {
            return fail(ctx, LNE_EINVAL, "project: bf16 input needs bf16/f32 output");
        }
#undef LNE_PBJ
#undef LNE_PB
    } else if (tri) {
        const int vmul = y_t == LNE_F64 ? 2 : 4;
        const int vec = ((uintptr_t)Y % 16 == 0 && ldy % vmul == 0 && ys % vmul == 0) ? 1 : 0;
        // as many column tiles at a time as keep W's tiles in LDS, in groups
        // of about one size; a block per CU over the batch (fewer strips of
        // 16 rows than that: a block each)
        int mj = std::min(ntout, 9);
        while (mj > 1 && tri_tiles(ntout - mj, mj) > kTriMaxTiles) --mj;
        mj = (int)ceil_div(ntout, ceil_div(ntout, mj));
        const size_t lds = 2048 * (size_t)tri_tiles(ntout - mj, mj);
        const int64_t strips = ceil_div(n > 0 ? n : 1, 16);
        const dim3 tgrid((unsigned)std::min<int64_t>(strips, std::max(1, 256 / nb)), (unsigned)nb);
        Launch L(ctx, "project");
#define LNE_PT(T, MJ)                                                                     \
    case MJ:                                                                              \
        LNE_TRY(lds_opt_in(ctx, (const void *)k_proj_tri<T, MJ>, lds));                   \
        k_proj_tri<T, MJ><<<tgrid, kTriThreads, lds, ctx->stream>>>((T *)out, ldy, n, kin, W, \
                                                                    skip, ys, ws, vec);   \
        break
#define LNE_PTJ(T)                                                                        \
    switch (mj) {                                                                         \
        LNE_PT(T, 1);                                                                     \
        LNE_PT(T, 2);                                                                     \
        LNE_PT(T, 3);                                                                     \
        LNE_PT(T, 4);                                                                     \
        LNE_PT(T, 5);                                                                     \
        LNE_PT(T, 6);                                                                     \
        LNE_PT(T, 7);                                                                     \
        LNE_PT(T, 8);                                                                     \
        default:                                                                          \
            LNE_PT(T, 9);                                                                 \
    }
        if (y_t == LNE_F64) LNE_PTJ(double)
        else LNE_PTJ(float)
#undef LNE_PTJ
#undef LNE_PT
    } else {
        const int vmul = y_t == LNE_F64 ? 2 : 4;
        const int vec = ((uintptr_t)Y % 16 == 0 && ldy % vmul == 0 && ys % vmul == 0) ? 1 : 0;
        Launch L(ctx, "project");
        // at most 9 output column tiles per block: a wider output is split
        // over blockIdx.z (fewer accumulators per wave, so that two blocks
        // share a CU and cover each other's barriers; at k' <= 144 a split
        // costs more in repeated Y reads and spills than it gains)
#define LNE_P64(YT, OT, MJ)                                                                \
    k_proj64<YT, OT, MJ><<<dim3(grid.x, grid.y, (unsigned)((ntout + (MJ) - 1) / (MJ))),  \
                           kProjThreads, 0, ctx->stream>>>(                                \
        (const YT *)Y, ldy, n, kin, W, kout, (OT *)out, ldo, skip, ys, ws, os, vec)
#define LNE_P64J(YT, OT)                                                                   \
    do {                                                                                   \
        if (ntout <= 3) LNE_P64(YT, OT, 3);                                                \
        else LNE_P64(YT, OT, 9);                                                           \
    } while (0)
        if (y_t == LNE_F64 && out_t == LNE_F64) LNE_P64J(double, double);
        else if (y_t == LNE_F32 && out_t == LNE_F32) LNE_P64J(float, float);
        else if (y_t == LNE_F32 && out_t == LNE_F64) LNE_P64J(float, double);
        else if (y_t == LNE_F64 && out_t == LNE_F32) LNE_P64J(double, float);
        else return fail(ctx, LNE_EINVAL, "project: unsupported types");
#undef LNE_P64J
#undef LNE_P64
    }
    return check_launch(ctx, "project");
}

lne_status chol_inv(lne_ctx *ctx, double *G, int32_t k, double *W, int32_t *status,
                    int32_t *shifted, int64_t n_rows, const int32_t *skip, int32_t *skip_next,
                    int32_t nb) {
    if (k < 1 || k > kEigMaxK) return fail(ctx, LNE_EUNSUPPORTED, "chol_inv: k = %d", k);
    const int nt = (k + 15) / 16;
    const size_t lds = chol_lds(nt);
    {
        Launch L(ctx, "chol_inv");
        // a wave holds a seventh of the nt (nt - 1) / 2 tiles above the diagonal
#define LNE_CI(MT)                                                                           \
    do {                                                                                     \
        LNE_TRY(lds_opt_in(ctx, (const void *)k_chol_inv<MT>, lds));                         \
        k_chol_inv<MT><<<nb, kCholThreads, lds, ctx->stream>>>(G, k, W, status, shifted,     \
                                                               n_rows, skip, skip_next);     \
    } while (0)
        if (nt <= 4) LNE_CI(1);
        else if (nt <= 9) LNE_CI(6);
        else if (nt <= 13) LNE_CI(12);
        else if (nt <= 17) LNE_CI(20);
        else LNE_CI(22);
#undef LNE_CI
    }
    return check_launch(ctx, "chol_inv");
}

size_t sym_eig_ws_doubles(int32_t k, int32_t nb) { return (size_t)nb * eig_ws_one(k); }

lne_status sym_eig(lne_ctx *ctx, double *C, int32_t k, double *V, double *lam, int32_t nb,
                   double *vw_ws) {
    if (k > kEigMaxK) return fail(ctx, LNE_EUNSUPPORTED, "sym_eig: k = %d above %d", k, kEigMaxK);
    Buf vw(ctx);
    // vw_ws (if given) holds sym_eig_ws_doubles(k, nb) doubles
    if (vw_ws) vw.p = vw_ws, vw.ctx = nullptr;
    else LNE_TRY(alloc(ctx, vw, sizeof(double) * sym_eig_ws_doubles(k, nb)));
    double *ws = vw.as<double>();
    if (k < kEigSplit) {
        const size_t lds = std::max(sizeof(double) * (size_t)k * kZStride, back_lds(3));
        Launch L(ctx, "sym_eig");
        k_sym_eig_small<<<nb, kTriDiagThreads, lds, ctx->stream>>>(C, k, ws, V, lam);
        return check_launch(ctx, "sym_eig");
    }
    {
        Launch L(ctx, "sym_eig");
        if (k <= 64) k_tridiag<1><<<nb, kTriDiagThreads, 0, ctx->stream>>>(C, k, ws);
        else if (k <= 128) k_tridiag<2><<<nb, kTriDiagThreads, 0, ctx->stream>>>(C, k, ws);
        else if (k <= kEigMaxLds) k_tridiag<3><<<nb, kTriDiagThreads, 0, ctx->stream>>>(C, k, ws);
        else k_tridiag_wide<<<nb, kSolveThreads, 0, ctx->stream>>>(C, k, ws);
    }
    LNE_TRY(check_launch(ctx, "sym_eig"));
    // the halves' eigenvectors in LDS where they fit
    const size_t need = sizeof(double) * (size_t)k * kZStride;
    if (k <= kEigMaxLds) LNE_TRY(lds_opt_in(ctx, (const void *)k_sym_eig<true>, need));
    {
        Launch L(ctx, "sym_eig");
        if (k <= kEigMaxLds) k_sym_eig<true><<<nb, kSolveThreads, need, ctx->stream>>>(k, ws);
        else k_sym_eig<false><<<nb, kSolveThreads, 0, ctx->stream>>>(k, ws);
    }
    LNE_TRY(check_launch(ctx, "sym_eig"));
    const int nt = (k + 15) / 16;
    const dim3 grid((unsigned)((nt + kBackWaves - 1) / kBackWaves), (unsigned)nb);
#define LNE_EB(M)                                                                              \
    do {                                                                                       \
        LNE_TRY(lds_opt_in(ctx, (const void *)k_eig_back<M>, back_lds(M)));                    \
        Launch L(ctx, "sym_eig");                                                              \
        k_eig_back<M><<<grid, kBackThreads, back_lds(M), ctx->stream>>>(C, k, ws, V, lam);     \
    } while (0)
    if (nt <= 3) LNE_EB(3);
    else if (nt <= 9) LNE_EB(9);
    else LNE_EB(18);
#undef LNE_EB
    return check_launch(ctx, "sym_eig");
}

lne_status eig_weights(lne_ctx *ctx, const double *V, const double *lam, int32_t k,
                       int32_t kout, double power, double *W, double *S, int32_t nb,
                       const int32_t *on) {
    if (on && k != kout) return fail(ctx, LNE_EINVAL, "eig_weights: pass-through needs k == kout");
    {
        Launch L(ctx, "eig_weights");
        k_eig_weights<<<dim3(grid_of((int64_t)k * kout, 256), (unsigned)nb), 256, 0,
                        ctx->stream>>>(V, lam, k, kout, power, W, S, on);
    }
    return check_launch(ctx, "eig_weights");
}

}  // namespace lne
