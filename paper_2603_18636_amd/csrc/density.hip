// Offline profiling: attention density of one head's attention map (paper Sec. 4.1, the offline
// profiling module; the equation defining d_{l,h}).
//
// For a query row i with logits s_t = <q_i, k_t> and p_t = softmax_t(scale * s_t) over all n keys,
// the row's prefix length is the size of the shortest descending-sorted prefix of p whose sum
// reaches tau.  Nothing is sorted: the row keeps a bracket [lo, hi) of logit values that holds the
// prefix's last key, and every pass over the keys narrows it BINS-fold (64 bins for bf16, 32 for float32, where
// a K tile takes twice the LDS):
//
//   pass 0      row maximum m and minimum of the logits, mean and variance of a sample of them
//   pass 1      histogram over all keys of the masses 2^((s_t - m) c2)  (c2 = scale * log2 e): BINS equal
//               bins around the value a normal distribution of the logits would give, the outer two
//               open-ended.  The sum of the bins is Z; the bin in which the running mass from above
//               meets tau Z is the bracket.
//   pass 2...   rows whose bracket may hold more than CAP = 2 BINS keys: the same histogram inside the
//               bracket only.  Rows with fewer: the keys in it are collected into a list, and those
//               above it counted; the row is done.
//
// and the lists are ordered at the end.  75,600 keys take four or five passes where halving the
// bracket took 29 (float32: four at 4,096 to 8,190 keys, 27-30).  Rows whose logits are all equal are done after
// pass 0.  A bracket that shrinks to one float value holds ties, taken one at a time by a division.  A bracket that
// equal bins cannot split (its width is not a usable float32) is split by the order of the float bit patterns instead.
//
// The logits are recomputed in every pass by the same instruction sequence, so they are
// bit-identical from pass to pass, and a bin's edges are the exact floats at which the bin function
// steps, so the histogram, the bracket and the list agree on every key.  Masses are rounded to a 64-bit
// fixed-point unit 2^-S and added as integers (LDS atomics): independent of the order of the additions.  The n
// roundings drop at most n 2^-(S+1); svoo_attention_density chooses S.
//
// S^T = K Q^T on the matrix cores (bf16: 32x32x16, float32: 32x32x2), one query per lane column.  A
// workgroup owns 32 RG query rows and splits the keys KS ways (wave (rg, ks) takes the tiles ks,
// ks + KS, ... for row group rg); K tiles come by direct global->LDS loads, swizzled as in the
// attention kernel.  All waves add into one histogram per row.
//
// Bound (12 x 2,048 rows x 75,600 keys, d = 128, bf16): vector issue.  A logit of a histogram pass
// costs ~60 vector cycles (exponential 16, bin index 12, fixed-point mass 20) against 16 of its
// share of the matrix instruction.  Measured there: 24.7 ms for 29 passes of halving; four passes with a branch per
// logit in the later ones 4.3 - 4.55 ms, as they are 4.0 - 4.2.  Of a lane's 16 logits two bit masks say which are inside
// the bracket, and every lane of the wave picks its next one: 1.5 % of the keys are inside in pass 2, two rounds for all
// 64 lanes, where 10 of 16 branches were taken for some lane.
#include <math.h>

#include <type_traits>

#include "common.h"

#define LOG2E_F 1.4426950408889634f
#define DEN_REFINE_N (1 << 18)   // more keys: masses in the unit of the row (svoo_attention_density says why)
// Keys inside the bracket, of a lane's 16, up to which they are picked one by one.  On normal logits up to 1 / 2 / 3 cost up to
// 20 / 9 / 2.5 % against 4, and 6 or 8 nothing either way; always picking saves 1 - 3 % there but costs 2 - 25 % where
// outliers leave most keys inside.
#define DEN_PICK 4
#define DEN_MAX_PASSES 48   // pass 0, pass 1, and far more splits than a float interval allows; a hard stop

typedef __attribute__((ext_vector_type(8))) __bf16 den_bf16x8;
typedef __attribute__((ext_vector_type(16))) float den_f32x16;
typedef unsigned long long den_u64;

struct DensityArgs {
    const void* q;
    const void* k;
    const int32_t* rows;     // nullable: query row indices shared by all slices
    int32_t* prefix_len;     // [bh, n_rows]
    int32_t* passes;         // nullable [bh]: most passes over the keys any workgroup of the slice made
    int n, n_rows, bh;
    float scale, tau;
    float z_tau;             // normal quantile of 1 - tau: where pass 1 centres its bins
    int fix_bits;            // S: masses are integers in units of 2^-S, n 2^S < 2^62
    double fix;              // 2^S
};

// next representable float above x (x finite or +inf)
__device__ __forceinline__ float next_up(float x) {
    if (!(x < INFINITY)) return x;
    uint32_t u = __float_as_uint(x);
    if ((u << 1) == 0) return __uint_as_float(1u);          // +-0 -> smallest subnormal
    return __uint_as_float((u >> 31) ? u - 1 : u + 1);
}

// float order as unsigned integer order (adding +0 turns -0 into +0), and back
__device__ __forceinline__ uint32_t float_key(float x) {
    const uint32_t u = __float_as_uint(x + 0.f);
    return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k) {
    return __uint_as_float(k ^ ((k >> 31) ? 0x80000000u : 0xffffffffu));
}

// p in units of 2^-S, rounded to nearest: p 2^S < 2^52, so adding 2^52 leaves the integer in the mantissa
__device__ __forceinline__ den_u64 to_fixed(float p, double fix) {
    const long long u = __double_as_longlong(fma((double)p, fix, 4503599627370496.0));
    return (den_u64)u & 0xfffffffffffffULL;
}

// by value: of two array elements the compiler would select the address, and keep the array in memory
__device__ __forceinline__ float pick(bool second, float b, float a) { return second ? b : a; }

// What a lane needs of its row during a pass.
struct Bracket {
    float lo, hi;            // lo <= s < hi is inside
    float inv, off;          // equal bins: floor(s inv + off), clamped
    uint32_t mode;           // DEN_EQUAL, DEN_ORDER (bits 8.. = shift), DEN_COLLECT, DEN_DONE
};
enum { DEN_EQUAL = 0, DEN_ORDER = 1, DEN_COLLECT = 2, DEN_DONE = 3 };

template <int BINS>
__device__ __forceinline__ int equal_bin(float s, float inv, float off) {
    return (int)__builtin_amdgcn_fmed3f(fmaf(s, inv, off), 0.f, (float)(BINS - 1));
}

template <int BINS>
__device__ __forceinline__ int bracket_bin(float s, const Bracket& r) {     // s >= r.lo
    if ((r.mode & 255u) == DEN_ORDER) {
        const uint32_t b = (float_key(s) - float_key(r.lo)) >> (r.mode >> 8);
        return (int)(b < BINS - 1 ? b : BINS - 1);
    }
    return equal_bin<BINS>(s, r.inv, r.off);
}

// Smallest float of [lo, hi] whose bin is at least `bin` (hi if there is none): the exact lower edge.
template <int BINS>
__device__ __forceinline__ float bin_edge(int bin, float lo, float hi, const Bracket& r) {
    uint32_t a = float_key(lo), b = float_key(hi);
    while (a < b) {
        const uint32_t mid = a + (b - a) / 2;
        if (bracket_bin<BINS>(key_float(mid), r) >= bin) b = mid; else a = mid + 1;
    }
    return key_float(a) + 0.f;
}

// no float but lo itself in [lo, hi)
__device__ __forceinline__ bool one_value(float lo, float hi) { return next_up(lo) >= hi; }

// Bins for the bracket [lo, hi): equal ones unless the last split did not narrow it or they are no use.
template <int BINS>
__device__ __forceinline__ void set_bins(Bracket& r, bool by_order) {
    r.inv = (float)BINS / (r.hi - r.lo);
    r.off = -r.lo * r.inv;
    r.mode = DEN_EQUAL;
    if (by_order || !(r.inv > 0.f && r.inv < 1e37f) || !(fabsf(r.off) < 1e7f)) {
        const uint32_t span = float_key(r.hi) - float_key(r.lo);
        uint32_t shift = 0;
        while (((span - 1) >> shift) >= (uint32_t)BINS) ++shift;
        r.mode = DEN_ORDER | (shift << 8);
    }
}

// Partial result of one pass for one row, one per key split
struct PassPartial {
    float mx, mn, sum, sq;   // pass 0
    int cnt, samples;        // keys at or above hi; logits in sum / sq
};

template <typename T, int D>
struct DenTile {
    static constexpr int ROWB = D * (int)sizeof(T);
    static constexpr int KEYS = 8192 / ROWB < 32 ? 32 : 8192 / ROWB;   // 8 KB a tile (16 KB for float32, d = 128)
    static constexpr int BYTES = KEYS * ROWB;
};

template <typename T, int D, int RG, int KS, int BINS>
struct DenLds {
    static constexpr int ROWS = 32 * RG;
    static constexpr int STAGE = KS * DenTile<T, D>::BYTES;
    static constexpr int HIST = 2 * STAGE;                             // [BINS][ROWS] u64, or a list of 2 BINS floats per row
    static constexpr int PART = HIST + BINS * ROWS * 8;                // [KS][ROWS] PassPartial
    static constexpr int STATE = PART + KS * ROWS * (int)sizeof(PassPartial);   // per row: bracket, nmb, list length, unit
    static constexpr int BYTES = STATE + 8 * ROWS * 4;
    static_assert(2 * STAGE >= 2 * BINS * ROWS * 4, "the ordered lists reuse the K tiles");
    static_assert(BYTES <= 160 * 1024, "LDS");
};

// REFINE: so many keys that pass 1 is done again in the unit that the row's own mass allows
template <typename T, int D, int RG, int KS, int BINS, bool REFINE>
__global__ void __launch_bounds__(64 * RG * KS)
density_kernel(DensityArgs a) {
    using L = DenLds<T, D, RG, KS, BINS>;
    constexpr bool BF16 = std::is_same<T, uint16_t>::value;
    constexpr int ROWB = DenTile<T, D>::ROWB, KEYS = DenTile<T, D>::KEYS, TILE = DenTile<T, D>::BYTES;
    constexpr int CPR = ROWB / 16, DC = ROWB / 32, NKB = KEYS / 32, ROWS = L::ROWS, STAGE = L::STAGE;
    constexpr int NW = RG * KS, NT = 64 * NW, CAP = 2 * BINS;
    constexpr int RPL = 1024 / ROWB;                       // tile rows covered by one wave-load (1 KB)
    constexpr int LOADS = STAGE / 1024, LPW = (LOADS + NW - 1) / NW;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    den_u64* hist = (den_u64*)(lds + L::HIST);
    float* list = (float*)(lds + L::HIST);                 // entry e of row r: word 2 ((e / 2) ROWS + r) + e % 2
    PassPartial* part = (PassPartial*)(lds + L::PART);
    float* st_lo = (float*)(lds + L::STATE);
    float* st_hi = st_lo + ROWS;
    float* st_inv = st_hi + ROWS;
    float* st_off = st_inv + ROWS;
    uint32_t* st_mode = (uint32_t*)(st_off + ROWS);
    float* st_nmb = (float*)(st_mode + ROWS);
    int* st_len = (int*)(st_nmb + ROWS);                   // keys collected
    int* st_fix = st_len + ROWS;                           // S of the row's masses

    // consecutive workgroups of one slice on one XCD: they read the same keys at the same time
    const int wps = (a.n_rows + ROWS - 1) / ROWS, total = wps * a.bh;
    const int per_xcd = (total + 7) / 8;
    const int wg = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
    if ((int)(blockIdx.x / 8) >= per_xcd || wg >= total) return;
    const int b = wg / wps, row_base = (wg % wps) * ROWS;
    const int tid = threadIdx.x, lane = tid % 64, j = lane % 32, h = lane / 32;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), rg = wave % RG, ks = wave / RG;
    const int n = a.n;
    const int row = 32 * rg + j;                           // of the workgroup
    const bool rvalid = row_base + row < a.n_rows;
    int qrow = rvalid ? (a.rows ? a.rows[row_base + row] : row_base + row) : 0;
    qrow = qrow < 0 ? 0 : (qrow >= n ? n - 1 : qrow);
    const unsigned char* kg = (const unsigned char*)a.k + (size_t)b * n * ROWB;
    const int n_tiles = (n + KEYS - 1) / KEYS;
    const int n_steps = (n_tiles + KS - 1) / KS;           // a step = KS tiles, one per key split

    auto issue = [&](int step, int buf) {
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            int l = wave + i * NW;
            l = l < LOADS ? l : LOADS - 1;                 // the last load may be issued twice, with the same bytes
            const int tile = l / (TILE / 1024), rl = (l % (TILE / 1024)) * RPL + lane / CPR;
            int key = (step * KS + tile) * KEYS + rl;
            key = key < n ? key : n - 1;                   // rows past the end are masked or unused
            const int chunk = (lane % CPR) ^ (rl % CPR);
            load_global_to_lds_16(kg + (size_t)key * ROWB + chunk * 16, lds_address(lds) + buf * STAGE + l * 1024);
        }
    };
    issue(0, 0);

    uint4 qf[DC];                                          // contraction elements of chunk 2 c + h
    {
        const uint4* src = (const uint4*)((const unsigned char*)a.q + ((size_t)b * n + qrow) * ROWB);
#pragma unroll
        for (int c = 0; c < DC; ++c) qf[c] = src[2 * c + h];
    }
    int koff[DC];
#pragma unroll
    for (int c = 0; c < DC; ++c) koff[c] = j * ROWB + (((2 * c + h) ^ (j % CPR)) * 16);
    // the compiler's wait for the Q loads must not end up inside the tile loop
#pragma unroll
    for (int c = 0; c < DC; ++c) asm volatile("" ::"v"(qf[c].x), "v"(qf[c].y), "v"(qf[c].z), "v"(qf[c].w));

    const float c2 = a.scale * LOG2E_F;
    const bool owner = ks == 0 && h == 0;                  // this thread keeps the row's state
    // owner's state: bracket, mass above it, target mass, keys above it, length if already known
    Bracket br = {0.f, 0.f, 0.f, 0.f, rvalid ? (uint32_t)DEN_EQUAL : (uint32_t)DEN_DONE};
    float row_max = 0.f, row_min = 0.f;
    den_u64 m_hi = 0, target = 0;
    double fix = a.fix;
    int c_hi = 0, known_len = -1, valid = n;               // valid: keys whose logit is a number
    int g = 0;                                             // running step number: stage g % 2

    auto of_slice = [&](int first, int v) { return first + 8 * (v / 4) + 4 * h + (v % 4) < n; };
    // One pass; body(s, ragged, first) sees every logit of this lane's row and key split, 32 keys from `first` on; of a
    // ragged block the logits past the end are -inf.
    auto over_keys = [&](auto body) {
        for (int step = 0; step < n_steps; ++step, ++g) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            issue(step + 1 < n_steps ? step + 1 : 0, (g + 1) & 1);     // wraps into the next pass
            const int kt = step * KS + ks;
            if (kt < n_tiles) {
                const unsigned char* base = lds + (g & 1) * STAGE + ks * TILE;
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) {
                    den_f32x16 s;
#pragma unroll
                    for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
                    for (int c = 0; c < DC; ++c) {
                        const uint4 kf = *(const uint4*)(base + kb * 32 * ROWB + koff[c]);
                        if constexpr (BF16) {
                            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(den_bf16x8, kf),
                                                                        __builtin_bit_cast(den_bf16x8, qf[c]), s, 0, 0, 0);
                        } else {
                            s = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(kf.x), __uint_as_float(qf[c].x), s, 0, 0, 0);
                            s = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(kf.y), __uint_as_float(qf[c].y), s, 0, 0, 0);
                            s = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(kf.z), __uint_as_float(qf[c].z), s, 0, 0, 0);
                            s = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(kf.w), __uint_as_float(qf[c].w), s, 0, 0, 0);
                        }
                    }
                    const int first = kt * KEYS + 32 * kb;
                    if (first + 32 > n) {                  // ragged end: keys past it sort below everything
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            if (!of_slice(first, v)) s[v] = -INFINITY;
                        body(s, true, first);
                    } else {
                        body(s, false, first);
                    }
                }
            }
        }
    };
    // Publish the row's bracket for the next pass and clear what that pass adds into.
    auto publish = [&]() {
        const bool off = br.mode == DEN_DONE;
        st_lo[row] = off ? INFINITY : br.lo;
        st_hi[row] = off ? INFINITY : br.hi;
        st_inv[row] = br.inv;
        st_off[row] = br.off;
        st_mode[row] = br.mode;
        if (!off) {
            st_len[row] = 0;
            if (br.mode != DEN_COLLECT)
                for (int i = 0; i < BINS; ++i) hist[i * ROWS + row] = 0;
        }
    };
    // of `count` keys of mass p below the mass m_hi: as many as reach the target
    auto ties_taken = [&](den_u64 p, int count) {
        const den_u64 take = p ? (target - m_hi + p - 1) / p : (den_u64)count;
        return take < 1 ? 1 : (take > (den_u64)count ? count : (int)take);
    };
    // Walk the bins from the top: the one in which the mass reaches the target becomes the bracket.
    auto narrow = [&](float lowest, float highest) {
        const Bracket was = br;
        den_u64 mass = 0;
        int bin = BINS - 1;
        for (; bin >= 0; --bin) {
            mass = hist[bin * ROWS + row];
            if (m_hi + mass >= target || bin == 0) break;
            m_hi += mass;
        }
        br.lo = bin == 0 ? lowest : bin_edge<BINS>(bin, lowest, highest, was);
        br.hi = bin == BINS - 1 ? highest : bin_edge<BINS>(bin + 1, lowest, highest, was);
        const den_u64 p_lo = to_fixed(__builtin_amdgcn_exp2f(fmaf(br.lo, c2, st_nmb[row])), fix);
        // at most mass / p_lo keys; collect when they surely fit, when there is nothing left to split, and
        // when the masses are too small to tell (the list's length then does)
        if (mass <= p_lo * (den_u64)(CAP - 8) || one_value(br.lo, br.hi))
            br.mode = DEN_COLLECT;
        else
            set_bins<BINS>(br, br.lo == was.lo && br.hi == was.hi);
    };

    auto other = [&](float x) {          // the half-wave's other half of the row's keys
        auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
        return __int_as_float(h == 0 ? (int)r[1] : (int)r[0]);
    };
    // Some row of the workgroup has a logit that is no finite number, which is rare: extremes without the NaNs and
    // the logits above -inf counted.  A row with an infinite logit gets that count as its length, a key whose
    // logit is NaN weighs nothing.
    auto look_again = [&]() {
        float mx = -INFINITY, mn = INFINITY;
        int cnt = 0;
        over_keys([&](const den_f32x16& s, bool ragged, int first) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                mx = fmaxf(mx, s[v]);
                mn = fminf(mn, ragged && !of_slice(first, v) ? INFINITY : s[v]);
                cnt += s[v] > -INFINITY ? 1 : 0;
            }
        });
        mx = fmaxf(mx, other(mx));
        mn = fminf(mn, other(mn));
        cnt += __float_as_int(other(__int_as_float(cnt)));
        __syncthreads();                                   // the owners have read what pass 0 left here
        if (h == 0) part[ks * ROWS + row] = PassPartial{mx, mn, 0.f, 0.f, cnt, 0};
        __syncthreads();
        if (owner) {
            row_max = -INFINITY;
            row_min = INFINITY;
            cnt = 0;
            for (int o = 0; o < KS; ++o) {
                const PassPartial u = part[o * ROWS + row];
                row_max = fmaxf(row_max, u.mx);
                row_min = fminf(row_min, u.mn);
                cnt += u.cnt;
            }
            row_min += 0.f;
            valid = cnt;
            if (!(row_max < INFINITY && row_min > -INFINITY)) {
                br.mode = DEN_DONE;
                known_len = cnt;
            }
        }
    };

    // ---- pass 0
    bool careful;
    {
        float mx = -INFINITY, mn = INFINITY, sum = 0.f, sq = 0.f;
        int samples = 0;
        over_keys([&](const den_f32x16& s, bool ragged, int first) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                mx = __builtin_elementwise_maximum(mx, s[v]);      // keeps a NaN, for the look below
                mn = fminf(mn, ragged && !of_slice(first, v) ? INFINITY : s[v]);
            }
            if ((first / (KEYS * KS) & 3) == 0 && !ragged) {       // a quarter of the keys is plenty for the first guess
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    sum += s[v];
                    sq = fmaf(s[v], s[v], sq);
                }
                samples += 16;
            }
        });
        const float omx = other(mx), omn = other(mn), osum = other(sum), osq = other(sq);
        if (h == 0)
            part[ks * ROWS + row] = PassPartial{__builtin_elementwise_maximum(mx, omx), fminf(mn, omn), sum + osum, sq + osq, 0, 2 * samples};
        __syncthreads();
        if (owner) {
            mx = -INFINITY; mn = INFINITY; sum = 0.f; sq = 0.f; samples = 0;
            for (int o = 0; o < KS; ++o) {
                const PassPartial u = part[o * ROWS + row];
                mx = __builtin_elementwise_maximum(mx, u.mx);
                mn = fminf(mn, u.mn);
                sum += u.sum;
                sq += u.sq;
                samples += u.samples;
            }
            row_max = mx;
            row_min = mn + 0.f;
        }
        careful = __syncthreads_or(owner && rvalid && !(row_max < INFINITY && row_min > -INFINITY));
        if (careful) look_again();
        if (owner) {
            mx = row_max;
            mn = row_min;
            st_nmb[row] = -mx * c2;
            // normal logits of mean mu and deviation sd: their masses are normal about mu + scale sd^2 (natural
            // units), so the prefix ends z_tau sd from there; +-1.25 sd around it, inside [min, max]
            const float mu = samples ? sum / samples : 0.5f * (mx + mn);
            const float var = samples ? sq / samples - mu * mu : 0.f;
            const float sd = sqrtf(fmaxf(var, 0.f));
            float guess = mu + a.scale * sd * sd + a.z_tau * sd;
            guess = fminf(fmaxf(guess, mn + 1.25f * sd), mx - 1.25f * sd);
            const bool usable = sd > 0.f && guess - 1.25f * sd > mn && guess + 1.25f * sd < mx;
            br.lo = usable ? guess - 1.25f * sd : row_min;
            br.hi = usable ? guess + 1.25f * sd : next_up(mx);
            if (br.mode != DEN_DONE && row_min == row_max) {
                // all logits equal (a zero query): as many as the target needs, no further pass
                const den_u64 p = to_fixed(__builtin_amdgcn_exp2f(fmaf(row_max, c2, st_nmb[row])), fix);
                const den_u64 z = p * (den_u64)valid;
                target = a.tau < 1.f ? (den_u64)ceil((double)a.tau * (double)z) : z;
                known_len = ties_taken(p, valid);
                br.mode = DEN_DONE;
            }
            if (br.mode != DEN_DONE) {
                set_bins<BINS>(br, false);
                if (br.mode != DEN_EQUAL) {                // pass 1 has equal bins only: everything in the lowest
                    br.inv = 0.f;
                    br.off = 0.f;
                    br.mode = DEN_EQUAL;
                }
            }
            publish();
        }
    }

    // ---- pass 1
    int pass = 1;
    if (!__syncthreads_and(!owner || br.mode == DEN_DONE)) {
        const float inv = st_inv[row], off = st_off[row], nmb = st_nmb[row];
        for (int round = 0;; ++round) {
            ++pass;
            over_keys([&](den_f32x16& s, bool, int) {
                if (careful)
#pragma unroll
                    for (int v = 0; v < 16; ++v) s[v] = s[v] == s[v] ? s[v] : -INFINITY;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(s[v], c2, nmb));
                    atomicAdd(&hist[equal_bin<BINS>(s[v], inv, off) * ROWS + row], to_fixed(p, fix));
                    if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);      // 16 at once would not fit the registers
                }
            });
            __syncthreads();
            den_u64 z = 0;
            if (owner && br.mode != DEN_DONE)
                for (int i = 0; i < BINS; ++i) z += hist[i * ROWS + row];
            if (round == (REFINE ? 1 : 0)) {
                if (owner) {
                    if (br.mode != DEN_DONE) {
                        target = a.tau < 1.f ? (den_u64)ceil((double)a.tau * (double)z) : z;
                        narrow(row_min, next_up(row_max));
                    }
                    publish();
                }
                break;
            }
            if (owner) {                                   // n masses of half a unit more at most
                const int octaves = 64 - __clzll((long long)(z + (den_u64)n / 2 + 1)) - a.fix_bits;
                const int s_bits = 61 - octaves < 50 ? 61 - octaves : 50;
                st_fix[row] = s_bits > a.fix_bits ? s_bits : a.fix_bits;
                publish();
            }
            __syncthreads();
            fix = ldexp(1.0, st_fix[row]);
        }
    }
    while (!__syncthreads_and(!owner || br.mode == DEN_DONE) && pass < DEN_MAX_PASSES) {
        // ---- later passes: only keys inside the bracket cost more than two comparisons
        int cnt = 0;
        {
            const Bracket r = {st_lo[row], st_hi[row], st_inv[row], st_off[row], st_mode[row]};
            const float nmb = st_nmb[row];
            auto take = [&](float x) __attribute__((always_inline)) {      // a key inside the bracket
                if (r.mode == DEN_COLLECT) {
                    const int e = atomicAdd(&st_len[row], 1);
                    if (e < CAP) list[2 * ((e / 2) * ROWS + row) + e % 2] = x;
                } else {
                    const float p = __builtin_amdgcn_exp2f(fmaf(x, c2, nmb));
                    atomicAdd(&hist[bracket_bin<BINS>(x, r) * ROWS + row], to_fixed(p, fix));
                }
            };
            over_keys([&](const den_f32x16& s, bool, int) {
                uint32_t from_lo = 0, from_hi = 0;         // bit v: s[v] is at or above the edge
#pragma unroll
                for (int v = 15; v >= 0; --v) {
                    from_lo = from_lo + from_lo + (s[v] >= r.lo ? 1u : 0u);
                    from_hi = from_hi + from_hi + (s[v] >= r.hi ? 1u : 0u);
                }
                cnt += __popc(from_hi);
                uint32_t in = from_lo & ~from_hi;
                if (__any(__popc(in) > DEN_PICK)) {        // a wide bracket: most logits have some lane's work
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        if (in >> v & 1u) take(s[v]);
                } else {
                    while (in) {                           // every lane its next key
                        const int v = __ffs(in) - 1;
                        in &= in - 1;
                        float t[8], u[4];
#pragma unroll
                        for (int i = 0; i < 8; ++i) t[i] = pick(v & 1, s[2 * i + 1], s[2 * i]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) u[i] = pick(v & 2, t[2 * i + 1], t[2 * i]);
                        take(pick(v & 8, pick(v & 4, u[3], u[2]), pick(v & 4, u[1], u[0])));
                    }
                }
            });
        }
        {
            auto r = __builtin_amdgcn_permlane32_swap(cnt, cnt, false, false);
            if (h == 0) part[ks * ROWS + row].cnt = (int)r[0] + (int)r[1];
        }
        __syncthreads();
        if (owner) {
            if (br.mode == DEN_COLLECT) {
                c_hi = 0;
                for (int o = 0; o < KS; ++o) c_hi += part[o * ROWS + row].cnt;
                const int len = st_len[row];
                if (len <= CAP) {
                    br.mode = DEN_DONE;
                } else if (one_value(br.lo, br.hi)) {     // ties: as many as the target needs
                    const den_u64 p = to_fixed(__builtin_amdgcn_exp2f(fmaf(br.lo, c2, st_nmb[row])), fix);
                    known_len = c_hi + ties_taken(p, len);
                    br.mode = DEN_DONE;
                } else {                                   // more keys than their masses suggested
                    set_bins<BINS>(br, true);
                }
            } else if (br.mode != DEN_DONE) {
                narrow(br.lo, br.hi);
            }
            publish();
        }
        ++pass;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // loads issued for the pass that never ran
    __syncthreads();
    // ---- order the lists: every entry counts the entries before it and puts its mass at that position
    float* ordered = (float*)lds;                          // [CAP][ROWS], over the K tiles
    for (int i = tid; i < CAP * ROWS; i += NT) {
        const int r = i % ROWS, e = i / ROWS;
        if (st_mode[r] != DEN_DONE) continue;              // stopped by the pass limit: no list
        const int len = st_len[r];
        if (len > CAP || e >= len) continue;
        const float v = list[2 * ((e / 2) * ROWS + r) + e % 2];
        int rank = 0;
        for (int o = 0; o < len; ++o) {
            const float u = list[2 * ((o / 2) * ROWS + r) + o % 2];
            rank += (u > v || (u == v && o < e)) ? 1 : 0;
        }
        if (rank < CAP) ordered[rank * ROWS + r] = __builtin_amdgcn_exp2f(fmaf(v, c2, st_nmb[r]));
    }
    __syncthreads();
    if (a.passes && tid == 0) atomicMax(&a.passes[b], pass + (careful ? 1 : 0));
    if (owner && rvalid) {
        int len = known_len;
        if (len < 0) {
            len = c_hi;
            if (br.mode == DEN_DONE) {
                den_u64 m = m_hi;
                for (int i = 0; i < st_len[row]; ++i) {
                    m += to_fixed(ordered[i * ROWS + row], fix);
                    ++len;
                    if (m >= target) break;
                }
            }
        }
        a.prefix_len[(size_t)b * a.n_rows + row_base + row] = len < 1 ? 1 : (len > n ? n : len);
    }
}

template <typename T, int D, int RG, int KS, int BINS, bool REFINE = false>
static int launch_density(const DensityArgs& a, hipStream_t stream) {
    static unsigned char opted_in[SVOO_MAX_DEVICES];
    constexpr int bytes = DenLds<T, D, RG, KS, BINS>::BYTES;
    auto kern = density_kernel<T, D, RG, KS, BINS, REFINE>;
    if (!opt_in_dynamic_lds((const void*)kern, bytes, opted_in)) return SVOO_ERR_HIP;
    const long long total = (long long)((a.n_rows + 32 * RG - 1) / (32 * RG)) * a.bh;
    hipLaunchKernelGGL(kern, dim3((unsigned)((total + 7) / 8 * 8)), dim3(64 * RG * KS), bytes, stream, a);
    return SVOO_OK;
}

// One workgroup fits a compute unit (its histograms and K stages fill the LDS) and runs for the whole launch,
// so the rows per workgroup are the fewest with which one round of the 256 units covers all rows, else 128.  That
// is not always the best split: 12 x 2,048 rows are 264 workgroups of 96 rows, eight too many, and run as 192
// of 128 (4.0-4.2 ms), a quarter of the chip idle; three full rounds of 32-row workgroups have not been measured.
template <typename T, int D>
static int dispatch_density(const DensityArgs& a, hipStream_t stream) {
    auto wgs = [&](int rg) { return (long long)((a.n_rows + 32 * rg - 1) / (32 * rg)) * a.bh; };
    if (a.n > DEN_REFINE_N) {
        constexpr int FEW = std::is_same<T, float>::value ? 4 : 8, BINS = std::is_same<T, float>::value ? 32 : 64;
        if (wgs(1) <= 256) return launch_density<T, D, 1, FEW, BINS, true>(a, stream);
        return launch_density<T, D, FEW / 2, 4, BINS, true>(a, stream);
    }
    if constexpr (std::is_same<T, float>::value) {
        if (wgs(1) <= 256) return launch_density<T, D, 1, 4, 32>(a, stream);
        return launch_density<T, D, 2, 4, 32>(a, stream);
    } else {
        if (wgs(1) <= 256) return launch_density<T, D, 1, 8, 64>(a, stream);
        if (wgs(2) <= 256) return launch_density<T, D, 2, 6, 64>(a, stream);
        if (wgs(3) <= 256) return launch_density<T, D, 3, 4, 64>(a, stream);
        return launch_density<T, D, 4, 4, 64>(a, stream);
    }
}

// density[b] = mean_i prefix_len[b, i] / n: integer sum in a fixed order, one division
__global__ void __launch_bounds__(1024)
density_mean_kernel(const int32_t* __restrict__ prefix_len, double* __restrict__ density, int n_rows, int n) {
    __shared__ long long red[1024];
    const int b = blockIdx.x, t = threadIdx.x;
    long long s = 0;
    for (int i = t; i < n_rows; i += 1024) s += prefix_len[(size_t)b * n_rows + i];
    red[t] = s;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (t < w) red[t] += red[t + w];
        __syncthreads();
    }
    if (t == 0) density[b] = (double)red[0] / ((double)n_rows * (double)n);
}

__global__ void density_clear_kernel(int32_t* p, int count) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = 0;
}

// x with P(N(0, 1) <= x) = p, by bisection on erfc; only a first guess hangs on it
static double normal_quantile(double p) {
    double lo = -6.0, hi = 6.0;
    for (int i = 0; i < 40; ++i) {
        const double mid = 0.5 * (lo + hi);
        if (0.5 * erfc(-mid * 0.7071067811865476) < p) lo = mid; else hi = mid;
    }
    return lo;
}

extern "C" int svoo_attention_density(const svoo_shape* shape, const void* q, const void* k, const int32_t* rows,
                                      int32_t n_rows, float tau, float scale, int32_t* prefix_len, double* density,
                                      int32_t* passes, void* hip_stream) {
    int st = check_shape(shape, false);
    if (st != SVOO_OK) return st;
    if (!q || !k || !prefix_len || !density) return SVOO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || shape->bh > 65535) return SVOO_ERR_INVALID_ARG;
    if (n_rows < 1 || n_rows > shape->n || (!rows && n_rows != shape->n)) return SVOO_ERR_INVALID_ARG;
    if (!(tau > 0.0f) || !(tau <= 1.0f) || !(scale > 0.0f) || !(scale < 1e30f)) return SVOO_ERR_INVALID_ARG;
    hipStream_t stream = (hipStream_t)hip_stream;
    // Fixed-point unit: n masses of at most 1 (and a rounding) stay below 2^62, one mass below 2^51.  The n roundings
    // of half a unit are 2^-26 of a row's mass at most up to 2^18 keys, less than float32 sums of 64 keys would
    // round; beyond that the unit that allows for rows of mass n is too coarse for rows of mass 1 (2^-14 at
    // 2^24 keys), and pass 1 is done again in the row's own (2 x 524,293 x 64, 512 rows: 10.6 -> 12.8 ms).
    int bits = 0;
    while ((1LL << bits) < shape->n) ++bits;
    const int s_bits = 61 - bits < 50 ? 61 - bits : 50;
    DensityArgs a = {q, k, rows, prefix_len, passes, shape->n, n_rows, shape->bh, scale, tau,
                     (float)normal_quantile(1.0 - (double)tau), s_bits,
                     (double)(1LL << s_bits)};
    if (passes)
        hipLaunchKernelGGL(density_clear_kernel, dim3((shape->bh + 255) / 256), dim3(256), 0, stream, passes, shape->bh);
    if (shape->dtype == SVOO_BF16)
        st = shape->d == 128 ? dispatch_density<uint16_t, 128>(a, stream) : dispatch_density<uint16_t, 64>(a, stream);
    else
        st = shape->d == 128 ? dispatch_density<float, 128>(a, stream) : dispatch_density<float, 64>(a, stream);
    if (st != SVOO_OK) return st;
    hipLaunchKernelGGL(density_mean_kernel, dim3(shape->bh), dim3(1024), 0, stream, prefix_len, density, n_rows,
                       shape->n);
    return launch_status();
}
