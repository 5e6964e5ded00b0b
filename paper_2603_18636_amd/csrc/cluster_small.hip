// Algorithm 1 with few clusters and tokens: a half-step in two launches.
//
// The general path (cluster.hip) runs four or five dependent kernels per half-step.  With up to SMALL_MAX_K
// clusters a side and SMALL_MAX_N tokens each of them takes 4-9 us whatever it has to do, so here
//   assign   every workgroup builds the score matrix W of the slice itself, in LDS, while its tokens are on their way
//            (P = C_own C_opp^T, row norms, W = P^ C_opp: 2-7 us, as long as the launch it replaces), then decides
//            its 256 tokens: pre-filter, float64 decision of what that leaves open
//   update   the workgroup of a cluster finds its members in the labels itself (n labels, one pass; the labels
//            below its own are its offset), so there is no sort; it leaves the cluster-order layout on the way
// Same arithmetic and the same bits as the general path, however many tokens are open: the same float64 products in the
// same order in W, in the scores and in ||x C_opp^T||, and in the means the same row groups.
// Measured per half-step: 1 x 1,024 x 64 float32, 16 blocks 24.3 -> 14.8 us, 13.5 with the row-wise steps on 16 lanes a row and the
// rows of open tokens kept in LDS; 3 x 2,945 x 64 bf16, 24 / 40 blocks 28.8 -> 20.8, 17.4; 3 x 4,096 x 128, 32 blocks
// 33.5 -> 25.8.  Of the first one's assignment (9.5 us) 3.5 are the launch and the first loads, 2.5 W, 1.9 the pre-filter, 1.6 the
// open tokens.  One workgroup per slice for all iterations (no launches
// in between) was slower: 22 and 38 us for the first two, the pre-filter alone keeps a compute unit busy for 11-14.
#include <type_traits>

#include "cluster.h"

#define SMALL_MAX_N 8192
#define SMALL_MAX_K 64
#define SMALL_MAX_W 4096   // clusters of a side x d
#define SMALL_WAVES 8      // 32 tokens each
#define SMALL_MANY 24      // more open tokens of a workgroup than this are decided in tiles of 16

struct SmallAssign {
    const void* x;
    const double* c_own;
    const double* c_opp;
    int32_t* labels;
    int n, k_own, k_opp;
};

// Elements kq, 4 + kq, 8 + kq, .. of a row: what a lane feeds the float64 matrix instruction as the contraction runs on
template <int D>
__device__ __forceinline__ void load_every_4th(const uint16_t* row, int kq, double (&v)[D / 4]) {
#pragma unroll
    for (int c = 0; c < D / 8; ++c) {
        const uint4 u = ((const uint4*)row)[c];
        const uint32_t lo = kq < 2 ? u.x : u.y, hi = kq < 2 ? u.z : u.w;
        v[2 * c] = (double)__uint_as_float(kq & 1 ? lo & 0xffff0000u : lo << 16);
        v[2 * c + 1] = (double)__uint_as_float(kq & 1 ? hi & 0xffff0000u : hi << 16);
    }
}
template <int D>
__device__ __forceinline__ void load_every_4th(const float* row, int kq, double (&v)[D / 4]) {
#pragma unroll
    for (int c = 0; c < D / 4; ++c) {
        const float4 u = ((const float4*)row)[c];
        const float lo = kq & 1 ? u.y : u.x, hi = kq & 1 ? u.w : u.z;
        v[c] = (double)(kq & 2 ? hi : lo);
    }
}

// LDS layout in bytes, the same on both sides
template <typename T, int D>
struct SmallLds {
    static constexpr int CP = D + 2, WP = D + 1;       // row pitches in doubles: C_opp (pairs), W (columns)
    static constexpr int ROWB = 2 * D;                 // one term of one row of the split
    static constexpr int TERMS = 2;
    static constexpr int BLOCK = 32 * ROWB;
    static constexpr bool ROOM = sizeof(T) == 2 || D == 64;    // 128 registers hold more than the tokens
    int pitch, split, c_opp, ph, bterm, open, fixed, bytes;    // W in float64 takes C_opp's place once it is used up
    __host__ __device__ constexpr SmallLds(int k_own, int k_opp)
        : pitch(0), split(0), c_opp(0), ph(0), bterm(0), open(0), fixed(0), bytes(0) {
        const int own16 = (k_own + 15) / 16 * 16, own32 = (k_own + 31) / 32 * 32;
        pitch = (k_opp + 15) / 16 * 16 + 2;
        const int c = k_opp * CP * 8, w = own16 * WP * 8;
        split = 0;                                     // first: its swizzle wants whole rows aligned
        bterm = split + own32 / 32 * TERMS * BLOCK;
        c_opp = bterm + own16 * 8;
        ph = c_opp + (c > w ? c : w);
        fixed = ph + own16 * pitch * 8;
        open = c_opp + w;                              // rows of the open tokens, in float32, where P was
        const int end = open + (ROOM ? SMALL_MANY * D * 4 : 0);
        bytes = end > fixed ? end : fixed;
    }
};
// 16 waves of 128 registers fill a compute unit: the rows of the open tokens must not cost one of its two workgroups.  In a place of
// their own they did at 48 / 64 clusters of 64: 12 x 8,192 tokens (384 workgroups), two iterations, 153 us, now 133.
template <typename T, int D>
constexpr bool open_rows_keep_two_workgroups() {
    constexpr int HALF = 80 * 1024 - 2048;              // less the other shared variables
    for (int own = 1; own <= SMALL_MAX_W / D; ++own)
        for (int opp = 1; opp <= SMALL_MAX_W / D; ++opp) {
            const SmallLds<T, D> l(own, opp);
            if (l.fixed <= HALF && l.bytes > HALF) return false;
        }
    return true;
}
static_assert(open_rows_keep_two_workgroups<uint16_t, 64>() && open_rows_keep_two_workgroups<float, 64>() &&
              open_rows_keep_two_workgroups<uint16_t, 128>() && open_rows_keep_two_workgroups<float, 128>(), "a workgroup lost");

template <typename T, int D>
__global__ void __launch_bounds__(64 * SMALL_WAVES)
assign_small_kernel(SmallAssign a) {
    using L = SmallLds<T, D>;
    constexpr int CP = L::CP, WP = L::WP, ROWB = L::ROWB, CPR = ROWB / 16, DC = ROWB / 32, BLOCK = L::BLOCK;
    constexpr int XT = sizeof(T) == 2 ? 1 : 2;         // terms of a token
    constexpr int NW = SMALL_WAVES, NT = 64 * NW;
    constexpr bool ROOM = L::ROOM;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    __shared__ int32_t wmax_bits, degenerate_s, n_open;
    __shared__ int32_t open[32 * NW];
    const int n = a.n, k_own = a.k_own, k_opp = a.k_opp;
    const L l(k_own, k_opp);
    unsigned char* split = lds + l.split;
    double* opp_s = (double*)(lds + l.c_opp);
    double* w64 = (double*)(lds + l.c_opp);
    double* ph = (double*)(lds + l.ph);
    double* bterm = (double*)(lds + l.bterm);
    float* open_rows = (float*)(lds + l.open);
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int i16 = lane % 16, kq4 = lane / 16, j = lane % 32, h = lane / 32;
    const T* x = (const T*)a.x + (size_t)b * n * D;
    const double* c_own = a.c_own + (size_t)b * k_own * D;
    const double* c_opp = a.c_opp + (size_t)b * k_opp * D;
    const int pitch = l.pitch, rt = (k_own + 15) / 16, ct = (k_opp + 15) / 16;

    // ---- this wave's tokens, for later; C_opp into LDS
    const int tok = blockIdx.x * (32 * NW) + 32 * wave + j;
    RawChunk<T> xr[DC];
    {
        const T* src = x + (size_t)(tok < n ? tok : n - 1) * D;
#pragma unroll
        for (int c = 0; c < DC; ++c) load_raw(src + 16 * c + 8 * h, xr[c]);
    }
    for (int e = tid; e < k_opp * D / 2; e += NT) {
        const int r = e / (D / 2), t = e % (D / 2);
        *(double2*)(opp_s + r * CP + 2 * t) = ((const double2*)c_opp)[e];
    }
    // C_own's rows of the wave's first tile of P are on their way meanwhile, where there are registers for them
    double2 av[D / 8];
    auto load_own = [&](int job) {
        const int r0 = job / ct * 16;
        const double* ar = c_own + (size_t)(r0 + i16 < k_own ? r0 + i16 : k_own - 1) * D + 2 * kq4;
#pragma unroll
        for (int kb = 0; kb < D / 8; ++kb) av[kb] = *(const double2*)(ar + 8 * kb);
    };
    if (ROOM && wave < rt * ct) load_own(wave);
    if (tid == 0) {
        wmax_bits = 0;
        degenerate_s = 0;
        n_open = 0;
    }
    __syncthreads();

    // ---- P = C_own C_opp^T, one 16 x 16 tile per wave and trip; lane (i, kq) feeds row / column i and the
    // contraction indices 2 kq, 2 kq + 1 of a block of 8; accumulator v holds row kq + 4 v, column i
    for (int job = wave; job < rt * ct; job += NW) {
        const int r0 = job / ct * 16, col = job % ct * 16 + i16;
        const double* br = opp_s + (col < k_opp ? col : k_opp - 1) * CP + 2 * kq4;
        if (!ROOM || job != wave) load_own(job);
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kb = 0; kb < D / 8; ++kb) {
            const double2 bv = *(const double2*)(br + 8 * kb);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[kb].x, bv.x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[kb].y, bv.y, acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) ph[(r0 + kq4 + 4 * v) * pitch + col] = col < k_opp ? acc[v] : 0.0;
    }
    __syncthreads();
    // ---- row-wise L2 normalisation, b_j, degenerate flag: 16 lanes a row, four columns each (k_opp <= 64), added in the order
    // of the general path.  With a wave per row, 40 rows took 2.3 us, five of them in a row for a wave, each a chain of six exchanges, a
    // root and a division; now 1.
    static_assert(SMALL_MAX_K == 64, "four columns a lane");
    for (int r0 = 4 * wave; r0 < k_own; r0 += 4 * NW) {
        const int r = r0 + kq4 < k_own ? r0 + kq4 : k_own - 1;
        double p[4], q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            p[u] = i16 + 16 * u < k_opp ? ph[r * pitch + i16 + 16 * u] : 0.0;
            q[u] = fma(p[u], p[u], 0.0);               // rounded before it is added
        }
        const double nrm = sqrt(sum_of_16((q[0] + q[2]) + (q[1] + q[3])));
        const double div = nrm > NORM_FLOOR ? nrm : NORM_FLOOR;
        if (r0 + kq4 < k_own) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i16 + 16 * u < k_opp) ph[r * pitch + i16 + 16 * u] = p[u] / div;
            if (i16 == 0) {
                const bool degenerate = !(nrm >= NORM_FLOOR);
                const double t = nrm / NORM_FLOOR;
                bterm[r] = degenerate ? t * t : 1.0;
                if (degenerate) degenerate_s = 1;
            }
        }
    }
    __syncthreads();
    // ---- W = P^ C_opp, at most two 16 x 16 tiles per wave, kept in registers until C_opp's LDS is free
    {
        constexpr int JOBS = SMALL_MAX_W / (16 * 16 * NW);
        f64x4 acc[JOBS];
#pragma unroll
        for (int u = 0; u < JOBS; ++u) {
            acc[u] = f64x4{0.0, 0.0, 0.0, 0.0};
            const int job = wave + u * NW;
            if (job < rt * (D / 16)) {
                const double* ar = ph + (job / (D / 16) * 16 + i16) * pitch + 2 * kq4;
                const double* bc = opp_s + job % (D / 16) * 16 + i16;
                for (int k0 = 0; k0 < ct * 16; k0 += 16) {
#pragma unroll
                    for (int v = 0; v < 2; ++v) {
                        const double2 av = *(const double2*)(ar + k0 + 8 * v);
                        const int k = k0 + 8 * v + 2 * kq4;
                        const double b0 = k < k_opp ? bc[k * CP] : 0.0;
                        const double b1 = k + 1 < k_opp ? bc[(k + 1) * CP] : 0.0;
                        acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.x, b0, acc[u], 0, 0, 0);
                        acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.y, b1, acc[u], 0, 0, 0);
                    }
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < JOBS; ++u) {
            const int job = wave + u * NW;
            if (job < rt * (D / 16))
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    w64[(job / (D / 16) * 16 + kq4 + 4 * v) * WP + job % (D / 16) * 16 + i16] = acc[u][v];
        }
    }
    __syncthreads();
    // ---- W in the pre-filter's form, swizzled as its tiles are read, and the largest row norm: 16 lanes a row
    for (int r0 = 4 * wave; r0 < k_own; r0 += 4 * NW) {
        const int r = r0 + kq4 < k_own ? r0 + kq4 : k_own - 1;         // the last row may be written more than once
        unsigned char* blk = split + r / 32 * (L::TERMS * BLOCK);
        const int rl = r % 32;
        double sq = 0.0;
#pragma unroll
        for (int u = 0; u < D / 64; ++u) {
            const int t = 64 * u + 4 * i16, at = rl * ROWB + (((t / 8) ^ (rl % CPR)) * 16) + t % 8 * 2;
            uint16_t hi[4], lo[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double v = w64[r * WP + t + e];
                store_split(v, e, hi, lo);
                sq = fma(v, v, sq);
            }
            *(uint2*)(blk + at) = make_uint2(hi[0] | (uint32_t)hi[1] << 16, hi[2] | (uint32_t)hi[3] << 16);
            *(uint2*)(blk + BLOCK + at) = make_uint2(lo[0] | (uint32_t)lo[1] << 16, lo[2] | (uint32_t)lo[3] << 16);
        }
        sq = sum_of_16(sq);
        if (i16 == 0) atomicMax(&wmax_bits, __float_as_int(norm_rounded_up(sq)));
    }
    __syncthreads();

    // ---- pre-filter: assign_kernel's products and margin, without the places in the scores.  Tokens are split here and no
    // earlier: in two terms while W was built they took 228 registers (d = 128 float32), one workgroup of a compute unit's two,
    // and the loads were waited for first: 12 x 8,000 x 128, 32 blocks, two iterations 225 us, 193 now (207 with the float32
    // matrix instruction).
#pragma unroll
    for (int c = 0; c < DC; ++c) keep_raw(xr[c]);
    const float wmax = __int_as_float(wmax_bits);
    const bool degenerate = degenerate_s != 0;
    {
        float xn2 = 0.f;
#pragma unroll
        for (int c = 0; c < DC; ++c) xn2 = add_squares(xr[c], xn2);
        auto swap = [](float v) {
            return __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
        };
        {
            auto r = swap(xn2);
            xn2 = __int_as_float(r[0]) + __int_as_float(r[1]);
        }
        float best = -INFINITY, second = -INFINITY;
        int bidx = 0;
        for (int cb = 0; cb * 32 < k_own; ++cb) {
            const unsigned char* base = split + cb * (L::TERMS * BLOCK) + j * ROWB;
            f32x16_t acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
            for (int c = 0; c < DC; ++c) {
                const int at = ((2 * c + h) ^ (j % CPR)) * 16;
                const bf16x8_t wh = __builtin_bit_cast(bf16x8_t, *(const uint4*)(base + at));
                const bf16x8_t wl = __builtin_bit_cast(bf16x8_t, *(const uint4*)(base + BLOCK + at));
                const TokenChunk<XT> xf = split_chunk(xr[c]);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh, xf.term[0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wl, xf.term[0], acc, 0, 0, 0);
                if constexpr (XT == 2) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh, xf.term[1], acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int idx = 32 * cb + 8 * (v / 4) + 4 * h + (v % 4);
                const float val = idx < k_own ? acc[v] : -INFINITY;     // rows past the end were never written
                second = __builtin_amdgcn_fmed3f(best, second, val);
                bidx = val > best ? idx : bidx;
                best = val > best ? val : best;
            }
        }
        auto rb = swap(best), rs = swap(second);
        auto ri = __builtin_amdgcn_permlane32_swap(bidx, bidx, false, false);
        const float b0 = __int_as_float(rb[0]), b1 = __int_as_float(rb[1]);
        const float fb = fmaxf(b0, b1), fs = fmaxf(fminf(b0, b1), fmaxf(__int_as_float(rs[0]), __int_as_float(rs[1])));
        int slot = -1;
        if (h == 0 && tok < n) {
            const int fi = b0 >= b1 ? (int)ri[0] : (int)ri[1];
            const float xw = score_bound(xn2, wmax);
            const bool sure = (fb - fs) > 2.0f * fast_eps<T>() * xw && xw < SCORE_MAX;        // false for NaN as well
            if (degenerate || !sure) {
                slot = atomicAdd(&n_open, 1);
                open[slot] = tok;
            } else {
                a.labels[(size_t)b * n + tok] = fi < k_own ? fi : k_own - 1;
            }
        }
        // its row, from the two lanes that hold it: nobody has to fetch it again
        auto rs2 = __builtin_amdgcn_permlane32_swap(slot, slot, false, false);
        if (h) slot = (int)rs2[0];
        if (ROOM && slot >= 0 && slot < SMALL_MANY)
#pragma unroll
            for (int c = 0; c < DC; ++c) {
                float* dst = open_rows + slot * D + 16 * c + 8 * h;
#pragma unroll
                for (int e = 0; e < 8; ++e) dst[e] = raw_element(xr[c], e);
            }
    }
    __syncthreads();
    // ---- float64 decision of the open tokens, one per wave: lane = centroid, products added in index order
    const int count = n_open;
    // Many (a slice with a degenerate anchor, zero tokens): tiles of 16 tokens on the float64 matrix instruction, a wave
    // each (assign_kernel says why the bits are the same).  A token per thread and half of the centroids waited for its
    // loads; one iteration, in us, general path before there was this one / a token per thread / now:
    // 3 x 8,192 x 64 bf16, 64 blocks, a twentieth of zero tokens 123 / 145 / 114, one of them an anchor 462 / 236 / 235;
    // 2 x 6,000 x 128 float32, 30 blocks, zero tokens 155 / 191 / 124, an anchor 413 / 406 / 264.
    if (count > SMALL_MANY) {
        for (int p0 = 16 * wave; p0 < count; p0 += 16 * NW) {
            double av[D / 4];
            load_every_4th<D>(x + (size_t)open[p0 + i16 < count ? p0 + i16 : p0] * D, kq4, av);
            double nx[4] = {1.0, 1.0, 1.0, 1.0};       // of token kq + 4 v, as everything below
            if (degenerate) {                          // nx = ||x C_opp^T||, added in pairs of columns, then of pairs
                double s2[4] = {0.0, 0.0, 0.0, 0.0}, pair[4];
                static_assert(SMALL_MAX_K == 64, "two pairs of 16 columns");
#pragma unroll 1
                for (int c = 0; c < ct; ++c) {
                    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
                    const int col = 16 * c + i16;
                    const double* row = c_opp + (size_t)(col < k_opp ? col : k_opp - 1) * D + kq4;
#pragma unroll
                    for (int t = 0; t < D / 4; ++t) {
                        if (t % 8 == 0) __builtin_amdgcn_sched_barrier(0);     // all loads at once would not fit 128 registers
                        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[t], row[4 * t], acc, 0, 0, 0);
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        double sq = col < k_opp ? fma(acc[v], acc[v], 0.0) : 0.0;
#pragma unroll
                        for (int o = 1; o < 16; o <<= 1) sq += __shfl_xor(sq, o);
                        pair[v] = c & 1 ? pair[v] + sq : sq;
                        if (c & 1 || c + 1 == ct) s2[v] += pair[v];
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double r = sqrt(s2[v]);
                    nx[v] = r > NORM_FLOOR ? r : NORM_FLOOR;
                }
            }
            double best_v[4];
            int best_j[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                best_v[v] = -INFINITY;
                best_j[v] = NO_INDEX;
            }
            for (int c = 0; c < rt; ++c) {             // ascending per lane: ">" keeps the lowest index
                const int col = 16 * c + i16;
                const double* wr = w64 + col * WP + kq4;
                f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int t = 0; t < D / 4; ++t) {
                    if (t % 8 == 0) __builtin_amdgcn_sched_barrier(0);
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[t], wr[4 * t], acc, 0, 0, 0);
                }
                const double bj = bterm[col < k_own ? col : k_own - 1];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double val = degenerate ? general_score(acc[v], nx[v], bj) : acc[v];
                    if (col < k_own && val > best_v[v]) {
                        best_v[v] = val;
                        best_j[v] = col;
                    }
                }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
#pragma unroll
                for (int o = 8; o > 0; o >>= 1) {
                    const double ov = __shfl_xor(best_v[v], o);
                    const int oj = __shfl_xor(best_j[v], o);
                    if (wins(ov, oj, best_v[v], best_j[v])) {
                        best_v[v] = ov;
                        best_j[v] = oj;
                    }
                }
                const int p = p0 + kq4 + 4 * v;
                if (i16 == 0 && p < count) a.labels[(size_t)b * n + open[p]] = best_j[v] == NO_INDEX ? 0 : best_j[v];
            }
        }
        return;
    }
    for (int p = wave; p < count; p += NW) {
        const int t = __builtin_amdgcn_readfirstlane(open[p]);
        float x0, x1 = 0.f;
        if constexpr (ROOM) {
            x0 = open_rows[p * D + lane];
            if (D > 64) x1 = open_rows[p * D + (D > 64 ? 64 : 0) + lane];
        } else {
            x0 = (float)load_as_f64<T>(x + (size_t)t * D + lane);
            if (D > 64) x1 = (float)load_as_f64<T>(x + (size_t)t * D + (D > 64 ? 64 : 0) + lane);
        }
        auto at = [&](int c) {
            return (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(c < 64 ? x0 : x1), c % 64));
        };
        double sum = 0.0;
        const double* wr = w64 + (lane < k_own ? lane : k_own - 1) * WP;
#pragma unroll 32
        for (int c = 0; c < D; ++c) sum = fma(at(c), wr[c], sum);
        double val = sum;
        if (degenerate) {                              // nx = ||x C_opp^T||
            const double* row = c_opp + (size_t)(lane < k_opp ? lane : 0) * D;
            double s = 0.0;
#pragma unroll 16
            for (int c = 0; c < D; ++c) s = fma(at(c), row[c], s);
            double sq = lane < k_opp ? fma(s, s, 0.0) : 0.0;      // rounded before it is added
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) sq += __shfl_xor(sq, o);
            const double r = sqrt(sq);
            val = general_score(sum, r > NORM_FLOOR ? r : NORM_FLOOR, bterm[lane < k_own ? lane : k_own - 1]);
        }
        int idx = lane < k_own && val > -INFINITY ? lane : NO_INDEX;
        best_of_wave(val, idx);
        if (lane == 0) a.labels[(size_t)b * n + t] = idx == NO_INDEX ? 0 : idx;
    }
}

// One workgroup per (cluster, slice).  Wave w looks through the w-th quarter of the labels, 64 at a time (all in
// flight at once), counts its members and the labels below; the members then go into LDS in token order.
template <typename T, int D, int UNITS>
__global__ void __launch_bounds__(256)
update_small_kernel(const T* __restrict__ x, const int32_t* __restrict__ labels, double* __restrict__ c64,
                    float* __restrict__ c32, int32_t* __restrict__ counts, int32_t* __restrict__ perm,
                    int32_t* __restrict__ offsets, int n, int k) {
    constexpr int LANES = D / 8, GROUPS = 256 / LANES;
    __shared__ double part[GROUPS][D];
    __shared__ uint16_t member[UNITS * 256];
    __shared__ int32_t wave_cnt[4], wave_below[4];
    const int b = blockIdx.y, j = blockIdx.x, tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const int32_t* lab = labels + (size_t)b * n;
    const int units = (n + 255) / 256, t0 = wave * units * 64 + lane;      // tokens t0, t0 + 64, ...
    int mine[UNITS];
#pragma unroll
    for (int u = 0; u < UNITS; ++u) mine[u] = u < units && t0 + 64 * u < n ? lab[t0 + 64 * u] : 0x7fffffff;
    int cnt = 0, below = 0;
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        cnt += __popcll(__ballot(mine[u] == j));
        below += __popcll(__ballot(mine[u] < j));
    }
    if (lane == 0) {
        wave_cnt[wave] = cnt;
        wave_below[wave] = below;
    }
    __syncthreads();
    int run = 0, total = 0, beg = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        run += w < wave ? wave_cnt[w] : 0;
        total += wave_cnt[w];
        beg += wave_below[w];
    }
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        const unsigned long long bal = __ballot(mine[u] == j);
        if (mine[u] == j) member[run + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)(t0 + 64 * u);
        run += __popcll(bal);
    }
    __syncthreads();
    // the general path's sums: row group g takes the members g, g + GROUPS, ..., the groups are added in order
    const int le = tid % LANES, grp = tid / LANES;
    const T* xb = x + (size_t)b * n * D + 8 * le;
    double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    constexpr int ROWS = 8;
    for (int p = grp; p < total; p += ROWS * GROUPS) {
        double v[ROWS][8];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int q = p + r * GROUPS < total ? p + r * GROUPS : total - 1;
            load8_as_f64<T>(xb + (size_t)member[q] * D, v[r]);
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            if (p + r * GROUPS < total)
#pragma unroll
                for (int e = 0; e < 8; ++e) s[e] += v[r][e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) part[grp][8 * le + e] = s[e];
    __syncthreads();
    if (tid < D) {
        const size_t o = ((size_t)b * k + j) * D + tid;
        if (total > 0) {                               // an empty cluster keeps its centroid
            double t = part[0][tid];
            for (int g = 1; g < GROUPS; ++g) t += part[g][tid];
            c64[o] = t / (double)total;
        }
        if (c32) c32[o] = (float)c64[o];
    }
    if (tid == 0) {
        if (counts) counts[(size_t)b * k + j] = total;
        if (offsets) {
            offsets[(size_t)b * (k + 1) + j] = beg;
            if (j == k - 1) offsets[(size_t)b * (k + 1) + k] = beg + total;
        }
    }
    if (perm)
        for (int p = tid; p < total; p += 256) perm[(size_t)b * n + beg + p] = member[p];
}

template <typename T, int D>
static bool small_assign(const svoo_shape* s, const SmallAssign& a, hipStream_t stream) {
    auto kern = assign_small_kernel<T, D>;
    constexpr int k_max = SMALL_MAX_W / D;             // 64 clusters of 64, 32 of 128
    constexpr int most = SmallLds<T, D>(k_max, k_max).bytes;
    static unsigned char opted_in[SVOO_MAX_DEVICES];
    if (!opt_in_dynamic_lds((const void*)kern, most, opted_in)) return false;
    const int bytes = SmallLds<T, D>(a.k_own, a.k_opp).bytes;
    hipLaunchKernelGGL(kern, dim3((a.n + 32 * SMALL_WAVES - 1) / (32 * SMALL_WAVES), s->bh), dim3(64 * SMALL_WAVES), bytes,
                       stream, a);
    return true;
}

template <typename T, int D>
static bool small_half_step(const svoo_shape* s, const SmallStep& st, hipStream_t stream) {
    const SmallAssign a = {st.x, st.c_own, st.c_opp, st.labels, s->n, st.k_own, st.k_opp};
    if (!small_assign<T, D>(s, a, stream)) return false;
    auto update = [&](auto units) {
        auto kern = update_small_kernel<T, D, decltype(units)::value>;
        hipLaunchKernelGGL(kern, dim3(st.k_own, s->bh), dim3(256), 0, stream, (const T*)st.x, st.labels, st.c_own, st.c32,
                           st.counts, st.perm, st.offsets, s->n, st.k_own);
    };
    if (s->n <= 2048)
        update(std::integral_constant<int, 8>{});
    else if (s->n <= 4096)
        update(std::integral_constant<int, 16>{});
    else
        update(std::integral_constant<int, SMALL_MAX_N / 256>{});
    return true;
}

// What the launch saved is worth is the time W takes in every workgroup: up to 4,096 elements a side (3 x 4,096
// tokens, 64 blocks: 29.6 against 30.3 us per half-step at d = 64, but 40.9 against 36.5 at d = 128), and not more
// workgroups than the chip runs at once, fewer the larger W is (40 x 4,096 x 64, 24 blocks = 0.98 M: 33.1 against
// 37.5; 12 x 8,192 x 128, 32 blocks = 1.57 M: 42.6 against 46.0; 40 of those 92 against 64).
bool small_fits(const svoo_shape* s) {
    if (s->n > SMALL_MAX_N || s->kq > SMALL_MAX_K || s->kk > SMALL_MAX_K) return false;
    const long long w = (long long)(s->kq > s->kk ? s->kq : s->kk) * s->d;
    return w <= SMALL_MAX_W && w * s->bh * ((s->n + 255) / 256) <= 1600000;
}

int small_half_step(const svoo_shape* s, const SmallStep& st, hipStream_t stream) {
    bool ok;
    if (s->dtype == SVOO_BF16)
        ok = s->d == 128 ? small_half_step<uint16_t, 128>(s, st, stream) : small_half_step<uint16_t, 64>(s, st, stream);
    else
        ok = s->d == 128 ? small_half_step<float, 128>(s, st, stream) : small_half_step<float, 64>(s, st, stream);
    return ok ? launch_status() : SVOO_ERR_HIP;
}
