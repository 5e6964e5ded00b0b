// Cluster-contiguous layout: stable counting sort of labels, row gather (permute) and row
// scatter (un-permute).  Pure integer work and data movement; HBM-bandwidth bound.
//
// Sort of one slice (n tokens, K bins) in chunks:
//   hist     K-entry histogram per chunk: written by the assignment kernel, whose workgroups own a chunk of
//            256 tokens each, or by one wave per 512 tokens where only labels are at hand
//   scan     (unless chunks and bins are few) per bin, inclusive prefix over the chunks, in place: the
//            row before a chunk is where its tokens start, the last row the bin totals.  A workgroup takes
//            64 bins, its 16 waves a sixteenth of the chunks each
//   scatter  one wave per chunk walks its tokens 64 at a time in index order; lanes with equal
//            labels find each other with one ballot per label bit and are ranked by lane, so equal
//            labels keep ascending token order.  Every workgroup scans the K bin totals for the cluster
//            offsets itself, and without a scan it sums the histograms before its own
#include "common.h"

#define SORT_WAVES 4
// With few chunks and bins every scatter wave sums the histograms itself, a batch of loads in flight per bin, instead of
// the scan's launch.  svoo_permute, 4 slices, direct / scan, us: 2,048 tokens, 512 bins (4 chunks) 28.0 / 31.3;
// 8,192, 256 (16) 29.5 / 29.4; 16,384, 128 (32) 28.5 / 29.7; but 6,000, 512 (12) 35.0 / 31.8 and 16,384, 1,024 64 / 36.
// More than 32 chunks never: 12 x 32,760 tokens in 128 chunks of the assignment 97 / 91 per half-step.
#define SORT_DIRECT_CHUNKS 32
#define SORT_DIRECT_COUNTS 4096
#define SORT_DIRECT_BATCH 8

size_t sort_scratch_ints(int bh, int n, int n_clusters, bool have_hist) {
    return (size_t)bh * sort_chunks(n, have_hist) * n_clusters;
}

__device__ __forceinline__ int clamp_label(int l, int k) { return l < 0 ? 0 : (l >= k ? k - 1 : l); }

__global__ void __launch_bounds__(SORT_WAVES* SVOO_WAVE)
sort_hist_kernel(const int32_t* __restrict__ labels, int32_t* __restrict__ chunk_hist, int n, int k, int nchunks) {
    extern __shared__ int32_t lds[];
    const int wave = threadIdx.x / SVOO_WAVE, lane = threadIdx.x % SVOO_WAVE;
    const int b = blockIdx.y;
    const int chunk = blockIdx.x * SORT_WAVES + wave;
    int32_t* hist = lds + wave * k;
    for (int j = lane; j < k; j += SVOO_WAVE) hist[j] = 0;
    __syncthreads();
    if (chunk < nchunks) {
        const int32_t* lab = labels + (size_t)b * n;
        const int start = chunk * LABEL_CHUNK;
        for (int g = 0; g < LABEL_CHUNK / SVOO_WAVE; ++g) {
            int i = start + g * SVOO_WAVE + lane;
            if (i < n) atomicAdd(&hist[clamp_label(lab[i], k)], 1);
        }
    }
    __syncthreads();
    if (chunk < nchunks) {
        int32_t* out = chunk_hist + ((size_t)b * nchunks + chunk) * k;
        for (int j = lane; j < k; j += SVOO_WAVE) out[j] = hist[j];
    }
}

__global__ void __launch_bounds__(1024)
sort_scan_kernel(int32_t* __restrict__ chunk_hist, int k, int nchunks) {
    __shared__ int32_t tot[16][64];
    const int b = blockIdx.y, g = threadIdx.x / 64, lane = threadIdx.x % 64, j = blockIdx.x * 64 + lane;
    const int cpg = (nchunks + 15) / 16;
    const int c0 = g * cpg < nchunks ? g * cpg : nchunks, c1 = c0 + cpg < nchunks ? c0 + cpg : nchunks;
    int32_t* h = chunk_hist + (size_t)b * nchunks * k;
    int sum = 0;
    if (j < k) {
#pragma unroll 8
        for (int c = c0; c < c1; ++c) sum += h[(size_t)c * k + j];
    }
    tot[g][lane] = sum;
    __syncthreads();
    if (j >= k) return;
    int running = 0;
#pragma unroll
    for (int gg = 0; gg < 16; ++gg) running += gg < g ? tot[gg][lane] : 0;
#pragma unroll 8
    for (int c = c0; c < c1; ++c) {
        running += h[(size_t)c * k + j];
        h[(size_t)c * k + j] = running;
    }
}

template <bool DIRECT, int CHUNK>
__global__ void __launch_bounds__(SORT_WAVES* SVOO_WAVE)
sort_scatter_kernel(const int32_t* __restrict__ labels, const int32_t* __restrict__ chunk_hist,
                    int32_t* __restrict__ offsets, int32_t* __restrict__ perm, int n, int k, int nchunks) {
    constexpr int NT = SORT_WAVES * SVOO_WAVE, GROUPS = CHUNK / SVOO_WAVE;
    extern __shared__ int32_t lds[];
    __shared__ int32_t wave_sum[SORT_WAVES];
    const int tid = threadIdx.x, wave = tid / SVOO_WAVE, lane = tid % SVOO_WAVE;
    const int b = blockIdx.y;
    const int chunk = blockIdx.x * SORT_WAVES + wave;
    const bool active = chunk < nchunks;
    int32_t* off = lds;                        // [k] bin totals, then first positions of the clusters
    int32_t* cnt = lds + k + wave * k;         // [k] next position of each label in this chunk
    const int32_t* h = chunk_hist + (size_t)b * nchunks * k;
    const int32_t* lab = labels + (size_t)b * n;
    const int start = chunk * CHUNK;
    int mine[GROUPS];                          // all of the lane's labels requested at once
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        const int i = start + g * SVOO_WAVE + lane;
        mine[g] = (active && i < n) ? clamp_label(lab[i], k) : -1;
    }
    if (DIRECT) {
        for (int j = lane; j < k; j += SVOO_WAVE) {
            int base = 0, total = 0;
            for (int c0 = 0; c0 < nchunks; c0 += SORT_DIRECT_BATCH) {      // a batch of loads in flight, also of the rest
                int v[SORT_DIRECT_BATCH];
#pragma unroll
                for (int u = 0; u < SORT_DIRECT_BATCH; ++u) v[u] = c0 + u < nchunks ? h[(size_t)(c0 + u) * k + j] : 0;
#pragma unroll
                for (int u = 0; u < SORT_DIRECT_BATCH; ++u) {
                    total += v[u];
                    base += c0 + u < chunk ? v[u] : 0;
                }
            }
            cnt[j] = base;
            if (wave == 0) off[j] = total;
        }
    } else {
        for (int j = tid; j < k; j += NT) off[j] = h[(size_t)(nchunks - 1) * k + j];
        if (active)
            for (int j = lane; j < k; j += SVOO_WAVE) cnt[j] = chunk > 0 ? h[(size_t)(chunk - 1) * k + j] : 0;
    }
    __syncthreads();
    // exclusive scan of the totals: thread t owns `per` adjacent bins
    const int per = (k + NT - 1) / NT, j0 = tid * per;
    int sum = 0;
    for (int u = 0; u < per; ++u) sum += j0 + u < k ? off[j0 + u] : 0;
    int incl = sum;
#pragma unroll
    for (int s = 1; s < SVOO_WAVE; s <<= 1) {
        const int v = __shfl_up(incl, s);
        incl += lane >= s ? v : 0;
    }
    if (lane == SVOO_WAVE - 1) wave_sum[wave] = incl;
    __syncthreads();
    int run = incl - sum;
    for (int w = 0; w < wave; ++w) run += wave_sum[w];
    for (int u = 0; u < per; ++u)
        if (j0 + u < k) {
            const int v = off[j0 + u];
            off[j0 + u] = run;
            if (blockIdx.x == 0) offsets[(size_t)b * (k + 1) + j0 + u] = run;
            run += v;
            if (blockIdx.x == 0 && j0 + u == k - 1) offsets[(size_t)b * (k + 1) + k] = run;
        }
    __syncthreads();
    if (!active) return;
    for (int j = lane; j < k; j += SVOO_WAVE) cnt[j] += off[j];
    __builtin_amdgcn_wave_barrier();
    int32_t* out = perm + (size_t)b * n;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    int label_bits = 0;
    while ((1 << label_bits) < k) ++label_bits;
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        const int i = start + g * SVOO_WAVE + lane;
        const int label = mine[g];
        const bool valid = label >= 0;
        // lanes with my label: one ballot per label bit, no loop over the distinct labels
        unsigned long long same = __ballot(valid);
        for (int bit = 0; bit < label_bits; ++bit) {
            const bool set = (label >> bit) & 1;
            const unsigned long long bal = __ballot(set);
            same &= set ? bal : ~bal;
        }
        int first = 0;
        if (valid) {
            first = cnt[label];
            const int pos = first + __popcll(same & lt_mask);
            if (pos >= 0 && pos < n) out[pos] = i;     // always true for the histogram of these labels
        }
        __builtin_amdgcn_wave_barrier();
        if (valid && (same & lt_mask) == 0) cnt[label] = first + __popcll(same);   // lowest lane of each label
        __builtin_amdgcn_wave_barrier();   // cnt belongs to this wave alone: no workgroup barrier needed
    }
}

template <int CHUNK>
static void launch_scatter(dim3 grid, const int32_t* labels, int32_t* chunk_hist, int32_t* offsets, int32_t* perm, int n,
                           int k, int nchunks, hipStream_t stream) {
    const size_t lds = (size_t)(SORT_WAVES + 1) * k * sizeof(int32_t);
    if (nchunks <= SORT_DIRECT_CHUNKS && nchunks * k <= SORT_DIRECT_COUNTS) {
        hipLaunchKernelGGL((sort_scatter_kernel<true, CHUNK>), grid, dim3(SORT_WAVES * SVOO_WAVE), lds, stream, labels,
                           chunk_hist, offsets, perm, n, k, nchunks);
    } else {
        hipLaunchKernelGGL(sort_scan_kernel, dim3((k + 63) / 64, grid.y), dim3(1024), 0, stream, chunk_hist, k, nchunks);
        hipLaunchKernelGGL((sort_scatter_kernel<false, CHUNK>), grid, dim3(SORT_WAVES * SVOO_WAVE), lds, stream, labels,
                           chunk_hist, offsets, perm, n, k, nchunks);
    }
}

int sort_labels(int bh, int n, int k, const int32_t* labels, int32_t* perm, int32_t* offsets, int32_t* chunk_hist,
                bool have_hist, hipStream_t stream) {
    const int nchunks = sort_chunks(n, have_hist);
    dim3 grid((nchunks + SORT_WAVES - 1) / SORT_WAVES, bh);
    if (have_hist) {
        launch_scatter<ASSIGN_CHUNK>(grid, labels, chunk_hist, offsets, perm, n, k, nchunks, stream);
    } else {
        hipLaunchKernelGGL(sort_hist_kernel, grid, dim3(SORT_WAVES * SVOO_WAVE), SORT_WAVES * k * sizeof(int32_t), stream,
                           labels, chunk_hist, n, k, nchunks);
        launch_scatter<LABEL_CHUNK>(grid, labels, chunk_hist, offsets, perm, n, k, nchunks, stream);
    }
    return launch_status();
}

// ---------------------------------------------------------------------------------------------
// Row gather / scatter: every lane moves 16 bytes; a row of d elements takes row_bytes/16 lanes.
// ---------------------------------------------------------------------------------------------
struct RowPtrs {
    const uint4* src[4];
    uint4* dst[4];
};

// dst[b, p] = src[b, perm[b, p]]   (GATHER=true)    dst[b, perm[b, p]] = src[b, p]   (GATHER=false)
template <bool GATHER>
__global__ void __launch_bounds__(256)
move_rows_kernel(RowPtrs ptrs, const int32_t* __restrict__ perm, int n, int vec_per_row, int rows_per_block) {
    const int b = blockIdx.z, t = blockIdx.y;
    const int row_in_block = threadIdx.x / vec_per_row;
    const int v = threadIdx.x % vec_per_row;
    const int p = blockIdx.x * rows_per_block + row_in_block;
    if (row_in_block >= rows_per_block || p >= n) return;
    int token = perm[(size_t)b * n + p];
    token = token < 0 ? 0 : (token >= n ? n - 1 : token);   // an entry outside [0, n) must not leave the tensor
    const uint4* src = ptrs.src[t] + (size_t)b * n * vec_per_row;
    uint4* dst = ptrs.dst[t] + (size_t)b * n * vec_per_row;
    if (GATHER)
        dst[(size_t)p * vec_per_row + v] = src[(size_t)token * vec_per_row + v];
    else
        dst[(size_t)token * vec_per_row + v] = src[(size_t)p * vec_per_row + v];
}

template <bool GATHER>
static int move_rows(const svoo_shape* s, int n_tensors, const RowPtrs& ptrs, const int32_t* perm,
                     hipStream_t stream) {
    if (n_tensors == 0) return SVOO_OK;
    const int vec_per_row = s->d * elem_size(s->dtype) / 16;  // 8, 16 or 32
    const int rows_per_block = 256 / vec_per_row;
    dim3 grid((s->n + rows_per_block - 1) / rows_per_block, n_tensors, s->bh);
    hipLaunchKernelGGL(move_rows_kernel<GATHER>, grid, dim3(256), 0, stream, ptrs, perm, s->n, vec_per_row,
                       rows_per_block);
    return launch_status();
}

extern "C" int svoo_permute(const svoo_shape* shape, const int32_t* labels, int32_t n_clusters, int32_t n_tensors,
                            const void* const* src, void* const* dst, int32_t* perm, int32_t* offsets, void* ws,
                            size_t ws_bytes, void* hip_stream) {
    int st = check_shape(shape, false);
    if (st != SVOO_OK) return st;
    if (!labels || !perm || !offsets || !ws) return SVOO_ERR_INVALID_ARG;
    if (n_clusters < 1 || n_clusters > SVOO_MAX_K) return SVOO_ERR_INVALID_ARG;
    if (n_tensors < 0 || n_tensors > 4) return SVOO_ERR_INVALID_ARG;
    if (n_tensors > 0 && (!src || !dst)) return SVOO_ERR_INVALID_ARG;
    if (shape->bh > 65535) return SVOO_ERR_INVALID_ARG;
    RowPtrs ptrs = {};
    for (int t = 0; t < n_tensors; ++t) {
        if (!src[t] || !dst[t] || !aligned16(src[t]) || !aligned16(dst[t]) || src[t] == dst[t])
            return SVOO_ERR_INVALID_ARG;
        ptrs.src[t] = (const uint4*)src[t];
        ptrs.dst[t] = (uint4*)dst[t];
    }
    if ((((uintptr_t)ws) & 255u) != 0) return SVOO_ERR_INVALID_ARG;
    const size_t need = align_up(sort_scratch_ints(shape->bh, shape->n, n_clusters, false) * sizeof(int32_t), 256);
    if (ws_bytes < need) return SVOO_ERR_WORKSPACE_TOO_SMALL;
    hipStream_t stream = (hipStream_t)hip_stream;
    st = sort_labels(shape->bh, shape->n, n_clusters, labels, perm, offsets, (int32_t*)ws, false, stream);
    if (st != SVOO_OK) return st;
    return move_rows<true>(shape, n_tensors, ptrs, perm, stream);
}

extern "C" int svoo_gather(const svoo_shape* shape, const int32_t* perm, int32_t n_tensors, const void* const* src,
                           void* const* dst, void* hip_stream) {
    int st = check_shape(shape, false);
    if (st != SVOO_OK) return st;
    if (!perm || !src || !dst || n_tensors < 1 || n_tensors > 4 || shape->bh > 65535) return SVOO_ERR_INVALID_ARG;
    RowPtrs ptrs = {};
    for (int t = 0; t < n_tensors; ++t) {
        if (!src[t] || !dst[t] || !aligned16(src[t]) || !aligned16(dst[t]) || src[t] == dst[t])
            return SVOO_ERR_INVALID_ARG;
        ptrs.src[t] = (const uint4*)src[t];
        ptrs.dst[t] = (uint4*)dst[t];
    }
    return move_rows<true>(shape, n_tensors, ptrs, perm, (hipStream_t)hip_stream);
}

extern "C" int svoo_unpermute(const svoo_shape* shape, const void* src_sorted, const int32_t* perm, void* dst,
                              void* hip_stream) {
    int st = check_shape(shape, false);
    if (st != SVOO_OK) return st;
    if (!src_sorted || !perm || !dst || src_sorted == dst) return SVOO_ERR_INVALID_ARG;
    if (!aligned16(src_sorted) || !aligned16(dst)) return SVOO_ERR_INVALID_ARG;
    if (shape->bh > 65535) return SVOO_ERR_INVALID_ARG;
    RowPtrs ptrs = {};
    ptrs.src[0] = (const uint4*)src_sorted;
    ptrs.dst[0] = (uint4*)dst;
    return move_rows<false>(shape, 1, ptrs, perm, (hipStream_t)hip_stream);
}
