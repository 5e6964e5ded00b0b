// Top Block-Pair Selection: which key blocks each query block attends to.
//
// One workgroup per (query block r, slice b), all arithmetic in float64 (the matrix is K_q x K_k;
// the cost is nothing next to the attention it prunes):
//   a_j  = scale * <cq[r], ck[j]>            coarse block estimate A_bar = C_q C_k^T
//   w_j  = n_j exp(a_j - max) / Z            softmax over non-empty key blocks, weighted by size
//   rank_j = position of j in the order by descending w, equal weights by lower index (bins of the weight)
//   m    = shortest sorted prefix with cumulative weight >= tau, summed sequentially in that order
//   b    = ceil(keep * K_k) (a product within 1e-6 K_k of an integer counts as that integer);
//          kept = (keep > theta ? min(m, b) : max(m, b)) clamped to [1, #live]
#include "common.h"

#define MASK_THREADS 256
#define MASK_WAVES (MASK_THREADS / SVOO_WAVE)
#define MASK_BINS 1024      // 32 octaves of the weight, 32 bins each
#define MASK_BIN_MAX 128    // fuller bins are left to the bitonic sort
#define MASK_SUM_BATCH 16
#define EST_COLS 32         // centroid elements per step of the estimate (d is a multiple of it)

// A_bar[b, r, j] = <cq[b, r], ck[b, j]> in float64, the d products added in index order (32 x 32
// output tile per workgroup, 2 x 2 per thread), so that the selection kernel reads one coalesced
// row instead of every workgroup re-reading all key centroids.  Bound by latency: the next step's elements are
// loaded while this one's are multiplied.
__global__ void __launch_bounds__(256)
block_estimate_kernel(const float* __restrict__ cq, const float* __restrict__ ck, double* __restrict__ abar, int kq,
                      int kk, int d) {
    __shared__ double as[EST_COLS][33];
    __shared__ double bs[EST_COLS][33];
    const int b = blockIdx.z, m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    const int c_ld = threadIdx.x % EST_COLS, r_ld = threadIdx.x / EST_COLS;     // rows r_ld, r_ld + 8, ..
    const float* a = cq + (size_t)b * kq * d;
    const float* bm = ck + (size_t)b * kk * d;
    float av[4], bv[4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = r_ld + 8 * u;
            av[u] = (m0 + r < kq) ? a[(size_t)(m0 + r) * d + k0 + c_ld] : 0.f;
            bv[u] = (n0 + r < kk) ? bm[(size_t)(n0 + r) * d + k0 + c_ld] : 0.f;
        }
    };
    double acc[2][2] = {{0, 0}, {0, 0}};
    fetch(0);
    for (int k0 = 0; k0 < d; k0 += EST_COLS) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            as[c_ld][r_ld + 8 * u] = (double)av[u];
            bs[c_ld][r_ld + 8 * u] = (double)bv[u];
        }
        __syncthreads();
        if (k0 + EST_COLS < d) fetch(k0 + EST_COLS);
#pragma unroll
        for (int c = 0; c < EST_COLS; ++c) {
            const double a0 = as[c][ty * 2], a1 = as[c][ty * 2 + 1];
            const double b0 = bs[c][tx * 2], b1 = bs[c][tx * 2 + 1];
            acc[0][0] = fma(a0, b0, acc[0][0]);
            acc[0][1] = fma(a0, b1, acc[0][1]);
            acc[1][0] = fma(a1, b0, acc[1][0]);
            acc[1][1] = fma(a1, b1, acc[1][1]);
        }
        __syncthreads();
    }
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) {
            const int m = m0 + ty * 2 + i, n = n0 + tx * 2 + j;
            if (m < kq && n < kk) abar[((size_t)b * kq + m) * kk + n] = acc[i][j];
        }
}

// Bit pattern of a weight: weights are not negative, so it orders as the weight does, and unlike the weight it
// also orders a NaN, so that every row is ranked by a permutation.
__device__ __forceinline__ long long weight_key(double w) { return __builtin_bit_cast(long long, w); }

// Bin of a weight, falling as the key rises: the exponent and five bits of the mantissa, down to 2^-32.
__device__ __forceinline__ int weight_bin(double w) {
    const int bin = (0x3FF00000 - (int)(weight_key(w) >> 32)) >> 15;
    return bin < 0 ? 0 : bin >= MASK_BINS ? MASK_BINS - 1 : bin;
}

// Bound by latency: dependent LDS round trips and barriers.  The reductions therefore go through
// lane exchanges, the position in the order is the start of the weight's bin plus a look at the few others in the
// bin, and the cumulative sum fetches its terms in batches.  With the estimate, 12 x 256 query blocks, before and now:
// 256 key blocks 69 -> 34 us (threshold 0.95), 1,024 315 -> 89; 1,024 blocks that all tie, where the sort remains,
// 439 -> 210.  PT = key blocks per thread: up to 256 there is one, and a quarter of the code to fetch.
template <int PT>
__global__ void __launch_bounds__(MASK_THREADS)
block_mask_kernel(const double* __restrict__ abar, const int32_t* __restrict__ counts_q,
                  const int32_t* __restrict__ counts_k, const float* __restrict__ keep, double tau, double theta,
                  double scale, int32_t* __restrict__ block_count, int32_t* __restrict__ block_list,
                  uint8_t* __restrict__ bitmap, int kq, int kk, int d) {
    __shared__ double w_sorted[PT * MASK_THREADS + MASK_SUM_BATCH];     // also: the weights in bin order
    __shared__ int32_t ord[PT * MASK_THREADS];
    __shared__ int32_t bins[MASK_BINS];     // counts, then starts; also: position of a block (bitonic sort)
    __shared__ double red[MASK_THREADS];
    __shared__ int32_t red_i[2][MASK_WAVES];
    __shared__ int32_t kept_n[PT][MASK_WAVES];
    __shared__ int32_t n_keep_s;
    static_assert(MASK_BINS == 4 * MASK_THREADS && MASK_BINS >= PT * MASK_THREADS, "bins");

    const int b = blockIdx.y, r = blockIdx.x, t = threadIdx.x;
    const int lane = t % SVOO_WAVE, wave = t / SVOO_WAVE;
    const size_t row_off = ((size_t)b * kq + r) * kk;
    auto keep_nothing = [&]() {
        for (int j = t; j < kk; j += MASK_THREADS) {
            block_list[row_off + j] = -1;
            if (bitmap) bitmap[row_off + j] = 0;
        }
        if (t == 0) block_count[(size_t)b * kq + r] = 0;
    };
    if (counts_q[(size_t)b * kq + r] <= 0) return keep_nothing();   // empty query block

    // logits and their maximum over non-empty key blocks
    double e[PT];
    int nk[PT];
    double mx = -INFINITY;
    int n_live = 0;
#pragma unroll
    for (int u = 0; u < PT; ++u) {
        const int j = t + u * MASK_THREADS;
        e[u] = 0.0;
        nk[u] = 0;
        if (j < kk) {
            nk[u] = counts_k[(size_t)b * kk + j];
            e[u] = scale * abar[row_off + j];
            if (nk[u] > 0) {
                mx = e[u] > mx ? e[u] : mx;
                ++n_live;
            }
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) bins[4 * t + u] = 0;
    for (int s = SVOO_WAVE / 2; s > 0; s >>= 1) {
        const double o = __shfl_xor(mx, s);
        mx = o > mx ? o : mx;
        n_live += __shfl_xor(n_live, s);
    }
    if (lane == 0) {
        red[wave] = mx;
        red_i[0][wave] = n_live;
    }
    __syncthreads();
    n_live = 0;
#pragma unroll
    for (int u = 0; u < MASK_WAVES; ++u) {
        mx = red[u] > mx ? red[u] : mx;
        n_live += red_i[0][u];
    }
    if (n_live == 0) return keep_nothing();     // no key at all
    __syncthreads();

    // unnormalised weights, their sum in a fixed order (index order inside a thread, then a tree)
    double z = 0.0;
#pragma unroll
    for (int u = 0; u < PT; ++u) {
        e[u] = nk[u] > 0 ? (double)nk[u] * exp(e[u] - mx) : 0.0;
        z += e[u];
    }
    red[t] = z;
    __syncthreads();
    z = (red[lane] + red[lane + 128]) + (red[lane + 64] + red[lane + 192]);
    for (int s = SVOO_WAVE / 2; s > 0; s >>= 1) z += __shfl_xor(z, s);

    // Position in the descending order (ties: lower index first).  Blocks of a higher bin come first; within the bin
    // every block looks at the others.
    int bin[PT], rank[PT], fullest = 0;
#pragma unroll
    for (int u = 0; u < PT; ++u) {
        e[u] = e[u] / z;
        bin[u] = weight_bin(e[u]);
        rank[u] = nk[u] > 0 ? atomicAdd(&bins[bin[u]], 1) : -1;
    }
    __syncthreads();
    int count[4], before = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        count[u] = bins[4 * t + u];
        before += count[u];
        fullest = count[u] > fullest ? count[u] : fullest;
    }
    int upto = before;
    for (int s = 1; s < SVOO_WAVE; s <<= 1) {
        const int o = __shfl_up(upto, s);
        if (lane >= s) upto += o;
        const int f = __shfl_xor(fullest, s);
        fullest = f > fullest ? f : fullest;
    }
    if (lane == SVOO_WAVE - 1) {
        red_i[0][wave] = upto;
        red_i[1][wave] = fullest;
    }
    __syncthreads();
    int start = upto - before;
#pragma unroll
    for (int u = 0; u < MASK_WAVES; ++u) {
        start += u < wave ? red_i[0][u] : 0;
        fullest = red_i[1][u] > fullest ? red_i[1][u] : fullest;
    }
    // Up to 256 blocks a full bin costs what counting over every pair did (all tied: 101 us before, 100 now) and needs no
    // sort; with 1,024 blocks, 128 in a bin are 128 LDS reads per block against the 55 steps of the sort.
    if (PT == 1 || fullest <= MASK_BIN_MAX) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            bins[4 * t + u] = start;
            start += count[u];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PT; ++u)
            if (nk[u] > 0) {
                const int p = bins[bin[u]] + rank[u];
                w_sorted[p] = e[u];
                ord[p] = t + u * MASK_THREADS;
            }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PT; ++u)
            if (nk[u] > 0) {
                const int lo = bins[bin[u]], hi = bin[u] + 1 < MASK_BINS ? bins[bin[u] + 1] : n_live;
                const long long key = weight_key(e[u]);
                int rk = lo;
                for (int p = lo; p < hi; ++p) {
                    const long long o = weight_key(w_sorted[p]);
                    rk += (o > key || (o == key && ord[p] < t + u * MASK_THREADS)) ? 1 : 0;
                }
                rank[u] = rk;
            }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PT; ++u)
            if (nk[u] > 0) w_sorted[rank[u]] = e[u];
    } else {
        // many blocks of nearly the same weight: bitonic sort, empty blocks and the padding up to a power of two last
        int P = 1;
        while (P < kk) P <<= 1;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            const int j = t + u * MASK_THREADS;
            w_sorted[j] = nk[u] > 0 ? e[u] : -0.0;      // the lowest key there is
            ord[j] = j;
        }
        __syncthreads();
        for (int k2 = 2; k2 <= P; k2 <<= 1)
            for (int j2 = k2 >> 1; j2 > 0; j2 >>= 1) {
                for (int i = t; i < P; i += MASK_THREADS) {
                    const int ixj = i ^ j2;
                    if (ixj > i) {
                        const int x = ord[i], y = ord[ixj];
                        const double wx = w_sorted[i], wy = w_sorted[ixj];
                        const long long kx = weight_key(wx), ky = weight_key(wy);
                        const bool x_first = kx > ky || (kx == ky && x < y);
                        if (x_first != ((i & k2) == 0)) {
                            ord[i] = y;
                            ord[ixj] = x;
                            w_sorted[i] = wy;
                            w_sorted[ixj] = wx;
                        }
                    }
                }
                __syncthreads();
            }
        for (int i = t; i < P; i += MASK_THREADS) bins[ord[i]] = i;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PT; ++u)
            if (nk[u] > 0) rank[u] = bins[t + u * MASK_THREADS];
        __syncthreads();
    }
    if (t < MASK_SUM_BATCH) w_sorted[n_live + t] = 0.0;
    __syncthreads();

    if (t == 0) {
        int m = n_live;
        if (tau < 1.0) {
            double csum = 0.0;
            bool found = false;
            for (int i = 0; i < n_live && !found; i += MASK_SUM_BATCH) {
                double upto_w[MASK_SUM_BATCH];
#pragma unroll
                for (int u = 0; u < MASK_SUM_BATCH; ++u) upto_w[u] = w_sorted[i + u];
#pragma unroll
                for (int u = 0; u < MASK_SUM_BATCH; ++u) upto_w[u] = csum += upto_w[u];
                if (!(csum < tau)) {
#pragma unroll
                    for (int u = MASK_SUM_BATCH - 1; u >= 0; --u)
                        if (upto_w[u] >= tau) {
                            m = i + u + 1;
                            found = true;
                        }
                }
            }
            m = m < n_live ? m : n_live;
        }
        // keep arrives as a float32: a decimal ratio whose product with K_k is an integer (0.3 x 20)
        // sits a hair above it, so a product within 1e-6 K_k of an integer is that integer
        const double kp = (double)keep[b];
        const double prod = kp * (double)kk, nearest = rint(prod);
        const int budget = fabs(prod - nearest) <= 1e-6 * (double)kk ? (int)nearest : (int)ceil(prod);
        int n_keep = kp > theta ? (m < budget ? m : budget) : (m > budget ? m : budget);
        n_keep = n_keep > n_live ? n_live : n_keep;
        n_keep = n_keep < 1 ? 1 : n_keep;
        n_keep_s = n_keep;
        block_count[(size_t)b * kq + r] = n_keep;
    }
    __syncthreads();
    const int n_keep = n_keep_s;

    // compact the kept ids in ascending order: thread t owns ids t, t + 256, ...
    unsigned long long kept[PT];
#pragma unroll
    for (int u = 0; u < PT; ++u) {
        kept[u] = __ballot(rank[u] >= 0 && rank[u] < n_keep);
        if (lane == 0) kept_n[u][wave] = __popcll(kept[u]);
    }
    __syncthreads();
    int base = 0;
#pragma unroll
    for (int u = 0; u < PT; ++u) {
        const int j = t + u * MASK_THREADS;
        int at = base;
#pragma unroll
        for (int o = 0; o < MASK_WAVES; ++o) {
            at += o < wave ? kept_n[u][o] : 0;
            base += kept_n[u][o];
        }
        const bool mine = (kept[u] >> lane) & 1;
        if (mine) block_list[row_off + at + __popcll(kept[u] & ((1ull << lane) - 1))] = j;
        if (j < kk && bitmap) bitmap[row_off + j] = (uint8_t)mine;
    }
    for (int j = n_keep + t; j < kk; j += MASK_THREADS) block_list[row_off + j] = -1;
}

size_t mask_ws_bytes(const svoo_shape* s) { return align_up((size_t)s->bh * s->kq * s->kk * sizeof(double), 256); }

extern "C" int svoo_block_mask(const svoo_shape* shape, const float* cq, const float* ck, const int32_t* counts_q,
                               const int32_t* counts_k, const float* keep, float tau, float theta, float scale,
                               int32_t* block_count, int32_t* block_list, uint8_t* bitmap, void* ws, size_t ws_bytes,
                               void* hip_stream) {
    int st = check_shape(shape, true);
    if (st != SVOO_OK) return st;
    if (!cq || !ck || !counts_q || !counts_k || !keep || !block_count || !block_list) return SVOO_ERR_INVALID_ARG;
    if (!(tau > 0.0f) || !(tau <= 1.0f) || !(scale == scale) || !(theta == theta)) return SVOO_ERR_INVALID_ARG;
    if (shape->bh > 65535 || !ws || (((uintptr_t)ws) & 255u) != 0) return SVOO_ERR_INVALID_ARG;
    if (ws_bytes < mask_ws_bytes(shape)) return SVOO_ERR_WORKSPACE_TOO_SMALL;
    hipStream_t stream = (hipStream_t)hip_stream;
    double* abar = (double*)ws;
    hipLaunchKernelGGL(block_estimate_kernel, dim3((shape->kk + 31) / 32, (shape->kq + 31) / 32, shape->bh), dim3(256), 0,
                       stream, cq, ck, abar, shape->kq, shape->kk, shape->d);
    auto kern = shape->kk <= MASK_THREADS ? block_mask_kernel<1> : block_mask_kernel<SVOO_MAX_K / MASK_THREADS>;
    hipLaunchKernelGGL(kern, dim3(shape->kq, shape->bh), dim3(MASK_THREADS), 0, stream, abar, counts_q,
                       counts_k, keep, (double)tau, (double)theta, (double)scale, block_count, block_list, bitmap,
                       shape->kq, shape->kk, shape->d);
    return launch_status();
}
