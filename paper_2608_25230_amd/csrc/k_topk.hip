// Top-k forced-weight evaluation of attention rows (Definition 2.1; gap via
// the first form of Lemma 2.2), any dtype and shape.
//
// Three passes, and a fourth where the keys are split over workgroups:
//   scores  z[r][j] = scale_h * <q_r, k_j> + bias_j, float32 sums in column
//           order, on the matrix cores
//   select  per row: max m, sum l of exp(z - m), and for every budget the
//           exact k-th largest logit (one histogram for all budgets, ties by
//           index), optionally the top-kmax indices in rank order
//   tiers   per row: disjoint tier sums T_t = sum p_j v_j, M_t = sum p_j over
//           ranks [0,k_0), [k_0,k_1), ..., [k_last, n) on the matrix cores,
//           then o, o_S, the gap (1 - p(S)) * ||m_{S^c} - m_S|| and the
//           dropped mass
//   combine the key splits' tier sums added in order, then the same outputs
#include "fw_internal.hpp"
#include "select.hpp"
#include "topk_fused.hpp"

namespace fw {

namespace {

// Four floats at float alignment (logit rows start anywhere when n is odd).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ f32x4 mfma_bf16(const uint4 &a, const uint4 &b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// scale * acc + bias as a product and a sum, each rounded (opaque: the backend
// would fuse them)
__device__ __forceinline__ float logit(float scale, float acc, const float *bias, float b) {
    const float v = opaque(scale * acc);
    return bias ? v + b : v;
}

// 16 bytes of row `row` (d elements) from element c, zero past the row's end;
// one vector load when `vec` (d a multiple of the chunk, base 16-byte aligned).
template <typename T>
__device__ __forceinline__ uint4 chunk16(const T *row, int c, int d, bool vec) {
    constexpr int E = 16 / (int)sizeof(T);
    if (c >= d) return make_uint4(0u, 0u, 0u, 0u);
    if (vec) return *(const uint4 *)(row + c);
    T x[E];
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = c + e < d ? row[c + e] : (T)0;
    return __builtin_bit_cast(uint4, x);
}

}  // namespace

// ---------------------------------------------------------------------------
// scores.  A wave takes tiles of 16 keys: the tile is read as whole rows (a
// wave instruction covers contiguous kilobytes), turned through LDS into the
// MFMA operand layout and multiplied with RT tiles of 16 query rows held in
// registers; the next tile's loads are in flight meanwhile.  DC: columns in
// chunks of 32.
//
// The float32 MFMA (four columns per instruction) chains one fused
// multiply-add per column in order, bit for bit what fmaf over the columns
// gives (checked on 512,000 sums, denormals among them), so the logits, and
// with them the selected sets, do not depend on the tiling.  The bf16 MFMA
// sums in another order; logits that agree to their last bits then change
// ranks.  Lane (row m, kg) feeds columns kg, 4 + kg, 8 + kg, ...: LDS holds
// [kg][row][16-byte chunk], for bf16 the chunk's columns kg and 4 + kg in one
// word.
//
// Bound by the logits' writes, the keys' reads and, with many rows, the
// float32 MFMA rate.  64 units of 4 rows of 5003 bf16 keys: 26 us (95 us as
// 32 x 64 tiles of vector products); 8 units of 128 rows of 32,768: 107 us (272).
// ---------------------------------------------------------------------------
template <typename T, int DC, int RT>
__global__ void __launch_bounds__(256)
scores_kernel(const T *__restrict__ q, const T *__restrict__ k, const float *__restrict__ scale,
              const float *__restrict__ bias, int64_t H, int64_t G, int64_t n, int d, int splits, int vec,
              float *__restrict__ z) {
    constexpr bool B16 = sizeof(T) == 2;
    constexpr int E = 16 / (int)sizeof(T);      // elements per 16-byte chunk
    constexpr int CH = DC * 32 / E;             // chunks per row
    constexpr int LD = CH / 4;                  // loads per lane and tile (16 rows x CH chunks / 64)
    constexpr int RS = CH + 4;                  // words per row and kg: no bank conflicts on the reads
    extern __shared__ __align__(16) uint32_t lds_k[];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t *tile = lds_k + w * (64 * RS);
    const uint32_t rgs = (uint32_t)((G + 16 * RT - 1) / (16 * RT));
    const uint32_t b = xcd_order(blockIdx.x, gridDim.x), tb = b / (uint32_t)splits;
    const int64_t sp = b % (uint32_t)splits, g0 = (int64_t)(tb % rgs) * (16 * RT), h = tb / rgs;
    const T *qh = q + h * G * (int64_t)d;
    const T *kh = k + h * n * (int64_t)d;
    const int m16 = lane & 15, kg = lane >> 4;
    uint4 raw[LD];
    auto load = [&](const T *base, int64_t row0, int64_t rows) {
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int id = lane + 64 * i;
            const int64_t j = row0 + id / CH;
            raw[i] = j < rows ? chunk16(base + j * d, (id % CH) * E, d, vec) : make_uint4(0u, 0u, 0u, 0u);
        }
    };
    auto stage = [&]() {  // raw to LDS; this wave's reads of it follow
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int id = lane + 64 * i;
            uint32_t *to = tile + (id / CH) * RS + id % CH;
            const uint4 x = raw[i];
            to[0] = B16 ? __builtin_amdgcn_perm(x.z, x.x, 0x05040100u) : x.x;
            to[16 * RS] = B16 ? __builtin_amdgcn_perm(x.z, x.x, 0x07060302u) : x.y;
            to[32 * RS] = B16 ? __builtin_amdgcn_perm(x.w, x.y, 0x05040100u) : x.z;
            to[48 * RS] = B16 ? __builtin_amdgcn_perm(x.w, x.y, 0x07060302u) : x.w;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    const uint4 *mine = (const uint4 *)(tile + (kg * 16 + m16) * RS);
    uint4 qf[RT][LD];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        load(qh, g0 + 16 * t, G);
        stage();
#pragma unroll
        for (int f = 0; f < LD; ++f) qf[t][f] = mine[f];
    }
    const float sc = scale ? scale[h] : (float)(1.0 / sqrt((double)d));
    const int64_t tiles = (n + 15) / 16;
    const int64_t per = (uint32_t)(tiles + splits - 1) / (uint32_t)splits;
    const int64_t t0 = sp * per, t1 = t0 + per < tiles ? t0 + per : tiles;
    if (t0 + w < t1) load(kh, 16 * (t0 + w), n);
    for (int64_t t = t0 + w; t < t1; t += 4) {
        stage();
        if (t + 4 < t1) load(kh, 16 * (t + 4), n);
        f32x4 acc[RT];
#pragma unroll
        for (int x = 0; x < RT; ++x) acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < LD; ++f) {
            const uint4 kf = mine[f];
            const uint32_t kw[4] = {kf.x, kf.y, kf.z, kf.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
#pragma unroll
                for (int x = 0; x < RT; ++x) {
                    const uint32_t qw = ((const uint32_t *)&qf[x][f])[c];
                    if constexpr (B16) {
                        acc[x] = mfma_f32(__uint_as_float(kw[c] << 16), __uint_as_float(qw << 16), acc[x]);
                    } else {
                        acc[x] = mfma_f32(__uint_as_float(kw[c]), __uint_as_float(qw), acc[x]);
                    }
                }
                if constexpr (B16) {
#pragma unroll
                    for (int x = 0; x < RT; ++x) {
                        const uint32_t qw = ((const uint32_t *)&qf[x][f])[c];
                        acc[x] = mfma_f32(__uint_as_float(kw[c] & 0xFFFF0000u), __uint_as_float(qw & 0xFFFF0000u), acc[x]);
                    }
                }
            }
        }
        // lane: query row m16 of each row tile, keys 4 kg .. 4 kg + 3
        const int64_t j = 16 * t + 4 * kg;
        float bj[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) bj[i] = (bias && j + i < n) ? bias[j + i] : 0.f;
#pragma unroll
        for (int x = 0; x < RT; ++x) {
            const int64_t g = g0 + 16 * x + m16;
            if (g >= G) continue;
            f32x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = logit(sc, acc[x][i], bias, bj[i]);
            float *zr = z + (h * G + g) * n + j;
            if (j + 4 <= n) {
                *(f32x4u *)zr = v;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (j + i < n) zr[i] = v[i];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// select: one workgroup per row.  Three passes over the row, held in registers
// (PER logits per thread) or, past 32 per thread of 1024, read again: the
// largest logit and the least above kSelFloor; the normaliser with a histogram
// of kSelBins equal bins over that range (values outside it go to the end
// bins; the map is monotone, so bins order like values); and a collection of
// the bins that hold a budget's k-th logit (every bin from the largest
// budget's up when indices are wanted), one list segment per bin.  An entry's
// rank is the count above its bin plus the larger entries of its segment,
// which gives thresholds and rank order exactly.  Rows that this does not suit
// (a NaN or infinite maximum, segments that overflow) take the radix selection
// (four passes per budget and a bitonic sort).  1024 rows of 32,768 logits with
// 1024 indices: 93 us (760 us with the radix selection for every row).
// ---------------------------------------------------------------------------
constexpr int kSelBins = 1024;
constexpr int kSelSeg = 512;       // entries of a segment that rank counting takes
constexpr int kSelList = 1536;     // list entries beyond the index list's own
constexpr float kSelFloor = -1e4f; // masked logits below stay out of the histogram's range

template <int NTH, int PER>
__global__ void __launch_bounds__(NTH)
select_kernel(const float *__restrict__ z, int64_t R, int64_t n, KsArg ks, float *__restrict__ row_m,
              float *__restrict__ row_l, uint32_t *__restrict__ thr_key, int32_t *__restrict__ thr_cut,
              int32_t *__restrict__ topk_idx, int kmax, int sort_len, int cap) {
    extern __shared__ unsigned long long sortbuf[];
    __shared__ int hist[kSelBins];
    __shared__ int abv[kSelBins];      // logits in higher bins
    __shared__ int fill[kSelBins];     // next free list entry, negative: bin not collected
    __shared__ int scan[NTH];
    __shared__ int sh[4];
    __shared__ float redf[NTH / 64];
    const int64_t r = blockIdx.x;
    if (r >= R) return;
    const int tid = threadIdx.x;
    const float *zr = z + r * n;
    // every logit of the row: f(j, z_j)
    float held[PER > 0 ? PER : 1];
    auto each = [&](auto &&f) {
        if constexpr (PER > 0) {
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int64_t j = tid + (int64_t)NTH * i;
                if (j < n) f(j, held[i]);
            }
        } else {
#pragma unroll 4
            for (int64_t j = tid; j < n; j += NTH) f(j, zr[j]);
        }
    };
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int64_t j = tid + (int64_t)NTH * i;
        held[i] = j < n ? zr[j] : 0.f;
    }

    float m = -INFINITY, lo = INFINITY;
    each([&](int64_t, float x) {
        m = fmaxf(m, x);
        lo = fminf(lo, x > kSelFloor ? x : INFINITY);
    });
    for (int i = tid; i < kSelBins; i += NTH) {
        hist[i] = 0;
        fill[i] = -1;
    }
    m = block_reduce(m, redf, OpMax());
    lo = block_reduce(lo, redf, OpMin());
    const float inv = (m > lo) ? (float)kSelBins / (m - lo) : 0.f;
    auto bin_of = [&](float x) {
        const float f = (x - lo) * inv;
        return f > 0.f ? min((int)f, kSelBins - 1) : 0;
    };
    float s = 0.f;
    each([&](int64_t, float x) {
        s += expf(x - m);
        atomicAdd(&hist[bin_of(x)], 1);
    });
    s = block_reduce(s, redf, OpSum());
    if (tid == 0) { row_m[r] = m; row_l[r] = s; }
    // counts above each bin: a thread takes kSelBins / NTH bins from the top
    {
        constexpr int PB = kSelBins / NTH;
        const int lane = tid & 63, w = tid >> 6;
        int c[PB], sum = 0;
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            c[i] = hist[kSelBins - 1 - (tid * PB + i)];
            sum += c[i];
        }
        int inc = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off);
            if (lane >= off) inc += o;
        }
        if (lane == 63) scan[w] = inc;
        if (tid == 0) { sh[0] = 1; sh[1] = 0; }
        __syncthreads();
        int base = inc - sum;
        for (int i = 0; i < w; ++i) base += scan[i];
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const int b = kSelBins - 1 - (tid * PB + i);
            abv[b] = base;
            if (topk_idx && base < kmax && c[i] > 0) {
                fill[b] = base;
                if (c[i] > kSelSeg || base + c[i] > cap) sh[0] = 0;
            }
            if (!topk_idx) {
                // the bin of some budget's k-th logit, given list space in any order
                bool hit = false;
                for (int t = 0; t < ks.n; ++t) hit = hit || (base < ks.k[t] && ks.k[t] <= base + c[i]);
                if (hit) {
                    const int at = atomicAdd(&sh[1], c[i]);
                    fill[b] = at;
                    if (c[i] > kSelSeg || at + c[i] > cap) sh[0] = 0;
                }
            }
            base += c[i];
        }
    }
    __syncthreads();
    // a NaN or +inf logit makes the sum NaN; sums are at least 1 otherwise
    if (sh[0] && s >= 1.f && lo < INFINITY) {
        each([&](int64_t j, float x) {
            const int b = bin_of(x);
            if (fill[b] >= 0)
                sortbuf[atomicAdd(&fill[b], 1)] = ((unsigned long long)ord_key(x) << 32) | (0xFFFFFFFFu - (uint32_t)j);
        });
        __syncthreads();
        // each collected bin's segment is [fill - hist, fill); the bins are walked
        // by entry: the total list length is the sum over collected bins
        int len = topk_idx ? 0 : sh[1];
        if (topk_idx) {
            // the last collected bin ends the list
            for (int b = tid; b < kSelBins; b += NTH)
                if (fill[b] >= 0 && abv[b] + hist[b] >= kmax) sh[2] = abv[b] + hist[b];
            __syncthreads();
            len = sh[2];
        }
        for (int i = tid; i < len; i += NTH) {
            const unsigned long long e = sortbuf[i];
            const int b = bin_of(key_to_float((uint32_t)(e >> 32)));
            const int e1 = fill[b], e0 = e1 - hist[b];
            int rank = abv[b];
            for (int x = e0; x < e1; ++x) rank += sortbuf[x] > e;
            const int j = (int)(0xFFFFFFFFu - (uint32_t)(e & 0xFFFFFFFFull));
            for (int t = 0; t < ks.n; ++t)
                if (rank == ks.k[t] - 1) {
                    thr_key[r * ks.n + t] = (uint32_t)(e >> 32);
                    thr_cut[r * ks.n + t] = j;
                }
            if (topk_idx && rank < kmax) topk_idx[r * kmax + rank] = j;
        }
        return;
    }

    __syncthreads();
    uint32_t kmax_key = 0;
    int64_t kmax_cut = 0;
    for (int t = 0; t < ks.n; ++t) {
        uint32_t key;
        int rem;
        radix_select_desc(zr, n, ks.k[t], hist, sh, &key, &rem);
        int64_t cut = nth_tie(zr, n, key, rem, scan, sh);
        if (tid == 0) {
            thr_key[r * ks.n + t] = key;
            thr_cut[r * ks.n + t] = (int32_t)cut;
        }
        if (ks.k[t] == kmax) { kmax_key = key; kmax_cut = cut; }
    }
    if (topk_idx == nullptr) return;

    // gather the top-kmax as 64-bit sort keys, then bitonic sort descending
    for (int i = tid; i < sort_len; i += NTH) sortbuf[i] = 0ull;
    __syncthreads();
    const int64_t chunk = (n + NTH - 1) / NTH;
    const int64_t lo_j = tid * chunk, hi_j = (lo_j + chunk < n) ? lo_j + chunk : n;
    int c = 0;
    for (int64_t j = lo_j; j < hi_j; ++j) {
        uint32_t u = ord_key(zr[j]);
        c += (u > kmax_key) || (u == kmax_key && j <= kmax_cut);
    }
    int total;
    int pos = block_exclusive_scan(c, scan, &total);
    for (int64_t j = lo_j; j < hi_j; ++j) {
        uint32_t u = ord_key(zr[j]);
        if ((u > kmax_key) || (u == kmax_key && j <= kmax_cut))
            sortbuf[pos++] = ((unsigned long long)u << 32) | (0xFFFFFFFFu - (uint32_t)j);
    }
    __syncthreads();
    for (int size = 2; size <= sort_len; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int i = tid; i < sort_len / 2; i += NTH) {
                int lo2 = 2 * stride * (i / stride) + (i % stride);
                int hi2 = lo2 + stride;
                bool desc = (lo2 & size) == 0;
                unsigned long long a = sortbuf[lo2], bb = sortbuf[hi2];
                if (desc ? (a < bb) : (a > bb)) { sortbuf[lo2] = bb; sortbuf[hi2] = a; }
            }
            __syncthreads();
        }
    }
    for (int i = tid; i < kmax; i += NTH)
        topk_idx[r * kmax + i] = (int32_t)(0xFFFFFFFFu - (uint32_t)(sortbuf[i] & 0xFFFFFFFFull));
}

// ---------------------------------------------------------------------------
// tiers
// ---------------------------------------------------------------------------
struct TierArgs {
    const void *v;
    const float *z, *row_m, *row_l;
    const uint32_t *thr_key;
    const int32_t *thr_cut;
    int64_t H, G, n;
    int d, vec, splits;
    KsArg ks;
    float *o, *o_s, *gap, *dropped;
    float *part;    // [splits][R][NT][d] tier sums, splits > 1
    float *part_m;  // [splits][R][NT] tier masses
};

// The power of two by which a row's weights exp(z - m) are scaled so that they
// sum to at most one (l >= 1 is their sum): no tier sum exceeds the largest
// value, and a quotient of tier sums keeps its bits.
__device__ __forceinline__ float weight_scale(float l) {
    return __uint_as_float((253u - (__float_as_uint(l) >> 23)) << 23);
}

// Outputs of row r for the columns c = lane + 64 x, x < NC (those below cw) of
// a slice at c0, from its tier sums T(t, x) and masses; returns through ss the
// slice's share of ||m_rest - m_S||^2 per budget, summed over the wave.
template <int NT, int NC, typename F>
__device__ __forceinline__ void tier_outputs(const KsArg &ks, int64_t R, int64_t r, int d, int c0, int cw, int lane,
                                             const float (&mass)[NT], F &&T, float *o, float *o_s,
                                             float (&ss)[NT - 1]) {
    float mtot = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t) mtot += mass[t];
    const float inv_tot = 1.0f / mtot;
    float km[NT - 1], rm[NT - 1];
#pragma unroll
    for (int t = 0; t < NT - 1; ++t) {
        km[t] = rm[t] = ss[t] = 0.f;
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            if (u <= t) km[t] += mass[u]; else rm[t] += mass[u];
        }
    }
#pragma unroll
    for (int x = 0; x < NC; ++x) {
        const int c = lane + kWave * x;
        if (c >= cw) continue;
        float a[NT], sum = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            a[t] = T(t, c);
            sum += a[t];
        }
        if (o) o[r * d + c0 + c] = sum * inv_tot;
#pragma unroll
        for (int t = 0; t < NT - 1; ++t) {
            float kt = 0.f, rt = 0.f;
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                if (u <= t) kt += a[u]; else rt += a[u];
            }
            const float oS = kt / km[t];
            if (rm[t] > 0.f) {
                const float diff = rt / rm[t] - oS;
                ss[t] = fmaf(diff, diff, ss[t]);
            }
            if (o_s) o_s[((int64_t)ks.perm[t] * R + r) * d + c0 + c] = oS;
        }
    }
#pragma unroll
    for (int t = 0; t < NT - 1; ++t) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) ss[t] += __shfl_xor(ss[t], off);
    }
}

template <int NT>
__device__ __forceinline__ void tier_gaps(const KsArg &ks, int64_t R, int64_t r, const float (&mass)[NT],
                                          const float (&ss)[NT - 1], float *gap, float *dropped) {
    float mtot = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t) mtot += mass[t];
#pragma unroll
    for (int t = 0; t < NT - 1; ++t) {
        float rm = 0.f;
#pragma unroll
        for (int u = t + 1; u < NT; ++u) rm += mass[u];
        const int64_t at = (int64_t)ks.perm[t] * R + r;
        const float f = rm * (1.0f / mtot);
        gap[at] = (rm > 0.f) ? f * sqrtf(ss[t]) : 0.f;
        dropped[at] = f;
    }
}

// One workgroup of four waves: 16 rows of a unit (the MFMA's rows) and one of
// `splits` ranges of the keys, in blocks of 32 keys dealt to the waves.  A
// lane holds row lane % 16 and eight consecutive keys (lane / 16) of a block
// as the weight operand, masked once per tier, and reads CPL consecutive
// columns (lane % 16) of the same eight keys as the value operand; column
// tile i of the products is then columns i, CPL + i, 2 CPL + i, ..., so whole value
// rows are read and no transpose through LDS is needed.
//
// bf16 values: the float32 weights are split into three bf16 parts (8 bits
// each, exact), three MFMAs per tier and column tile; the result is a float32
// weight times a bf16 value in a float32 sum, as on the vector unit.  float32
// values use the float32 MFMA.  A masked weight times an infinite or NaN value
// would put NaN into every tier, so a wave whose sums are not finite forms
// them again on the vector unit, each key into its own tier only: one infinite
// value makes the decode call below 950 us instead of 86, and 8 units of 128 rows
// of 32,768 keys 4.7 ms instead of 0.27, with it in every unit 1.3 and 4.8 ms
// (4.6 and 23.7 ms for any values with one wave per row walking the keys).
//
// Columns are taken in slices of 16 CPL: CPL = 8 up to four tiers, else 4
// (accumulators: 4 NT CPL registers; past 256 registers the weights spill, while
// each slice forms the weights again).  Four tiers at 8 spill 72 registers and
// pay only for bf16 rows of whole chunks: 64 units of 17 rows of 20,000 keys, 8
// against 4, a call: bf16 of 128 columns 508 us and 518 (few rows 83 and 78), of
// 100 1172 and 898, float32 of 102 1103 and 974.  Three tiers: float32 of 128
// columns 569 and 629.
//
// 64 units of 4 rows of 5003 keys, four tiers: 44 us (4.4 ms with one wave per
// row walking the keys); 8 units of 128 rows of 32,768 keys, two tiers: 89 us
// (23.5 ms).  Bound by the load latency of the few blocks a wave has and by the
// weights (expf and three-part splits, 600 vector instructions per block).
template <typename T, int CPL, int NT>
__global__ void __launch_bounds__(256, NT * CPL <= 32 ? 2 : 1)
tiers_kernel(TierArgs a) {
    constexpr bool B16 = sizeof(T) == 2;
    constexpr int CW = 16 * CPL;
    constexpr int LPK = CPL * (int)sizeof(T) >= 16 ? CPL * (int)sizeof(T) / 16 : 1;  // loads per key
    __shared__ f32x4 red[NT * CPL * 64];  // [tier][column tile][lane], as the products come
    __shared__ float mass_w[4][NT][16];
    __shared__ float mass_s[NT][16];
    __shared__ float ss_s[16][NT];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m16 = lane & 15, kg = lane >> 4;
    const int64_t G = a.G, n = a.n;
    const int d = a.d;
    const uint32_t rts = (uint32_t)((G + 15) / 16);
    const uint32_t b = xcd_order(blockIdx.x, gridDim.x), tb = b / (uint32_t)a.splits;
    const int64_t sp = b % (uint32_t)a.splits, g0 = (int64_t)(tb % rts) * 16, h = tb / rts;
    const int64_t R = a.H * G, r0 = h * G + g0;
    const int rows = G - g0 < 16 ? (int)(G - g0) : 16;
    const int64_t blocks = (n + 31) / 32, per = (uint32_t)(blocks + a.splits - 1) / (uint32_t)a.splits;
    const int64_t b0 = sp * per, b1 = b0 + per < blocks ? b0 + per : blocks;
    const T *vh = (const T *)a.v + h * n * (int64_t)d;
    const int64_t r = r0 + m16;
    // a row whose weights' sum is NaN takes no part: its masses start as that NaN,
    // which reaches all of its outputs
    const bool there = m16 < rows;
    const float l = there ? a.row_l[r] : 1.f, m = there ? a.row_m[r] : 0.f, wsc = weight_scale(l);
    const bool live = there && l < INFINITY;
    const float *zr = a.z + (there ? r : r0) * n;
    unsigned long long thr[NT - 1];
#pragma unroll
    for (int t = 0; t < NT - 1; ++t)
        thr[t] = there ? ((unsigned long long)a.thr_key[r * (NT - 1) + t] << 32) |
                            (0xFFFFFFFFu - (uint32_t)a.thr_cut[r * (NT - 1) + t])
                      : 0ull;
    if (tid < 16 * NT) ss_s[tid / NT][tid % NT] = 0.f;
    float mass[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) mass[t] = l < INFINITY ? 0.f : l;

#pragma nounroll
    for (int c0 = 0; c0 < d; c0 += CW) {
        const int cw = d - c0 < CW ? d - c0 : CW;
        const int col = c0 + m16 * CPL;  // this lane's columns
        // byte offsets of the lane's values and logits in a block; past the end: reads zero
        // (far past every descriptor, and no step of a block wraps it)
        const uint32_t vcol = col < d ? (uint32_t)((kg * 8 * d + col) * (int)sizeof(T)) : 0x7FFFFF00u;
        const uint32_t kstep = (uint32_t)(d * (int)sizeof(T));
        const uint32_t vrow = there ? (uint32_t)((m16 * n + kg * 8) * 4) : 0xFFFFFFC0u;
        f32x4 acc[NT][CPL];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int i = 0; i < CPL; ++i) acc[t][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        for (int64_t blk = b0 + w; blk < b1; blk += 4) {
            const int64_t j0 = blk * 32 + kg * 8;
            // values of the lane's eight keys and their logits for its row.  With
            // a.vec by buffer loads: a descriptor per block (wave-uniform), so that
            // keys past the end and lanes without columns or row read zero and no
            // per-key address is held.  The key step is part of the vector offset:
            // the range check leaves the scalar offset out.
            uint4 raw[8][LPK];
            float zz[8];
            if (a.vec) {
                const int64_t left = n - blk * 32;
                const uint32_t vo = opaque(vcol);  // eight sums per block rather than eight registers
                const rsrc_t rv = make_rsrc(vh + blk * 32 * d, (uint32_t)((left < 32 ? left : 32) * d * (int)sizeof(T)));
#pragma unroll
                for (int e = 0; e < 8; ++e) {
#pragma unroll
                    for (int l = 0; l < LPK; ++l) {
                        if (B16 && CPL == 4) {  // 8 bytes per key
                            const auto x = __builtin_amdgcn_raw_buffer_load_b64(rv, vo + e * kstep, 0, 0);
                            const uint2 y = __builtin_bit_cast(uint2, x);
                            raw[e][l] = make_uint4(y.x, y.y, 0u, 0u);
                        } else {
                            // d is a multiple of 8: a lane with its first column has all of them
                            raw[e][l] = __builtin_bit_cast(
                                uint4, __builtin_amdgcn_raw_buffer_load_b128(rv, vo + e * kstep + l * 16, 0, 0));
                        }
                    }
                }
                const rsrc_t rz = make_rsrc(a.z + r0 * n + blk * 32, (uint32_t)((rows * n - blk * 32) * 4));
                const f32x4 x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rz, vrow, 0, 0));
                const f32x4 y = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rz, vrow + 16, 0, 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) { zz[e] = x[e]; zz[4 + e] = y[e]; }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const T *row = vh + (j0 + e) * d;
                    zz[e] = (there && j0 + e < n) ? zr[j0 + e] : 0.f;
                    // one load at any alignment, not CPL: rows of 250 columns 1926 to
                    // 1640 us (64 units of 17 rows of 20,000 keys)
                    if (B16 && j0 + e < n && col + CPL <= d) {
                        __builtin_memcpy(&raw[e][0], row + col, CPL * sizeof(T));
                        continue;
                    }
                    uint32_t x[CPL];
#pragma unroll
                    for (int i = 0; i < CPL; ++i) {
                        x[i] = 0u;
                        if (j0 + e < n && col + i < d) {
                            if constexpr (B16) x[i] = (uint32_t)row[col + i];
                            else x[i] = __float_as_uint(row[col + i]);
                        }
                    }
                    uint32_t *to = (uint32_t *)&raw[e][0];
                    if constexpr (B16) {
#pragma unroll
                        for (int i = 0; i < CPL; i += 2) to[i / 2] = x[i] | x[i + 1] << 16;
                    } else {
#pragma unroll
                        for (int i = 0; i < CPL; ++i) to[i] = x[i];
                    }
                }
            }
            float p[8];
            int tier[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int64_t j = j0 + e;
                p[e] = (live && j < n) ? expf(zz[e] - m) * wsc : 0.f;
                const unsigned long long u =
                    ((unsigned long long)ord_key(zz[e]) << 32) | (0xFFFFFFFFu - (uint32_t)j);
                tier[e] = NT - 1;
#pragma unroll
                for (int t = NT - 2; t >= 0; --t)
                    if (u >= thr[t]) tier[e] = t;
            }
            if (c0 == 0) {
#pragma unroll
                for (int t = 0; t < NT; ++t) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) mass[t] += tier[e] == t ? p[e] : 0.f;
                }
            }
            if constexpr (B16) {
                uint32_t part[3][4];
                uint32_t msk[NT][4];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    float lo = p[2 * x], hi = p[2 * x + 1];
#pragma unroll
                    for (int s = 0; s < 3; ++s) {
                        const uint32_t ul = __float_as_uint(lo), uh = __float_as_uint(hi);
                        part[s][x] = __builtin_amdgcn_perm(uh, ul, 0x07060302u);
                        lo -= __uint_as_float(ul & 0xFFFF0000u);
                        hi -= __uint_as_float(uh & 0xFFFF0000u);
                    }
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        msk[t][x] = (tier[2 * x] == t ? 0xFFFFu : 0u) | (tier[2 * x + 1] == t ? 0xFFFF0000u : 0u);
                }
                // the eight keys' values column by column
                uint4 B[CPL];
#pragma unroll
                for (int i = 0; i < CPL; ++i) {
                    uint32_t bv[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const uint32_t *lo = (const uint32_t *)&raw[2 * x][0], *hi = (const uint32_t *)&raw[2 * x + 1][0];
                        bv[x] = __builtin_amdgcn_perm(hi[i / 2], lo[i / 2], i & 1 ? 0x07060302u : 0x05040100u);
                    }
                    B[i] = make_uint4(bv[0], bv[1], bv[2], bv[3]);
                }
                // one weight operand live at a time
#pragma unroll
                for (int s = 0; s < 3; ++s) {
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        __builtin_amdgcn_sched_barrier(0);
                        const uint4 A = make_uint4(part[s][0] & msk[t][0], part[s][1] & msk[t][1],
                                                   part[s][2] & msk[t][2], part[s][3] & msk[t][3]);
#pragma unroll
                        for (int i = 0; i < CPL; ++i) acc[t][i] = mfma_bf16(A, B[i], acc[t][i]);
                    }
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float *x = (const float *)&raw[e][0];
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        __builtin_amdgcn_sched_barrier(0);
                        const float A = tier[e] == t ? p[e] : 0.f;
#pragma unroll
                        for (int i = 0; i < CPL; ++i) acc[t][i] = mfma_f32(A, x[i], acc[t][i]);
                    }
                }
            }
        }
        if (c0 == 0) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                float ms = mass[t];
                ms += __shfl_xor(ms, 16);
                ms += __shfl_xor(ms, 32);
                if (kg == 0) mass_w[w][t][m16] = ms;
            }
            __syncthreads();
            if (tid < 16 * NT) {
                const int t = tid / 16, g = tid % 16;
                mass_s[t][g] = mass_w[0][t][g] + mass_w[1][t][g] + mass_w[2][t][g] + mass_w[3][t][g];
            }
        }
        // lane: rows 4 kg + i4 of acc[t][i][i4], columns m16 CPL + i of the slice
        float worst = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int i = 0; i < CPL; ++i) {
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) worst = fmaf(acc[t][i][i4], 0.f, worst);
            }
        }
        if (__ballot(!(worst == 0.f))) {
            // an infinite or NaN value (or sum) among these keys: tier by tier
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int i = 0; i < CPL; ++i) acc[t][i] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            for (int i4 = 0; i4 < 4; ++i4) {
                const int rr = 4 * kg + i4;
                if (rr >= rows) continue;
                const int64_t rw = r0 + rr;
                const float mr = a.row_m[rw], lr = a.row_l[rw], wr = weight_scale(lr);
                if (!(lr < INFINITY)) continue;
                for (int64_t blk = b0 + w; blk < b1; blk += 4) {
                    for (int64_t j = blk * 32; j < blk * 32 + 32 && j < n; ++j) {
                        const float x = a.z[rw * n + j], pj = expf(x - mr) * wr;
                        const uint32_t u = ord_key(x);
                        int tj = NT - 1;
                        for (int t = NT - 2; t >= 0; --t) {
                            const uint32_t tk = a.thr_key[rw * (NT - 1) + t];
                            if (u > tk || (u == tk && j <= a.thr_cut[rw * (NT - 1) + t])) tj = t;
                        }
#pragma unroll
                        for (int i = 0; i < CPL; ++i) {
                            const float vv = col + i < d ? Elem<T>::load(vh, j * d + col + i) : 0.f;
#pragma unroll
                            for (int t = 0; t < NT; ++t) {
#pragma unroll
                                for (int y = 0; y < 4; ++y)
                                    if (t == tj && y == i4) acc[t][i][y] = fmaf(pj, vv, acc[t][i][y]);
                            }
                        }
                    }
                }
            }
        }
        // the waves' sums added in wave order
        if (w == 0) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int i = 0; i < CPL; ++i) red[(t * CPL + i) * 64 + lane] = acc[t][i];
            }
        }
        __syncthreads();
#pragma nounroll
        for (int x = 1; x < 4; ++x) {
            if (w == x) {
#pragma unroll
                for (int t = 0; t < NT; ++t) {
#pragma unroll
                    for (int i = 0; i < CPL; ++i) red[(t * CPL + i) * 64 + lane] += acc[t][i];
                }
            }
            __syncthreads();
        }
        const auto sum_of = [&](int t, int g, int c) {
            return red[(t * CPL + c % CPL) * 64 + (g >> 2) * 16 + c / CPL][g & 3];
        };
        if (a.splits > 1) {
            for (int e = tid; e < rows * NT * CW; e += 256) {
                const int c = e % CW, t = (e / CW) % NT, g = e / (CW * NT);
                if (c < cw) a.part[((sp * R + r0 + g) * NT + t) * d + c0 + c] = sum_of(t, g, c);
            }
            if (c0 == 0 && tid < rows * NT) a.part_m[(sp * R + r0) * NT + tid] = mass_s[tid % NT][tid / NT];
        } else {
            for (int g = w; g < rows; g += 4) {
                float ms[NT], ss[NT - 1];
#pragma unroll
                for (int t = 0; t < NT; ++t) ms[t] = mass_s[t][g];
                tier_outputs<NT, CW / 64>(a.ks, R, r0 + g, d, c0, cw, lane, ms,
                                          [&](int t, int c) { return sum_of(t, g, c); }, a.o, a.o_s, ss);
                if (lane == 0) {
#pragma unroll
                    for (int t = 0; t < NT - 1; ++t) ss_s[g][t] += ss[t];
                }
                if (c0 + CW >= d && lane == 0) {
#pragma unroll
                    for (int t = 0; t < NT - 1; ++t) ss[t] = ss_s[g][t];
                    tier_gaps<NT>(a.ks, R, r0 + g, ms, ss, a.gap, a.dropped);
                }
            }
        }
        __syncthreads();
    }
}

// The splits' tier sums added and the row's outputs: one workgroup per row, wave w
// takes splits w, w + 4, ..., and the waves' sums are added in order.
template <int NT>
__global__ void __launch_bounds__(256)
tiers_combine_kernel(TierArgs a) {
    __shared__ float part_s[4][NT][kWave];
    const int64_t r = blockIdx.x, R = a.H * a.G;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), d = a.d;
    float ms[NT], sum[NT - 1], ss[NT - 1];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        // at most 64 splits: one per lane
        ms[t] = lane < a.splits ? a.part_m[(lane * R + r) * NT + t] : 0.f;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) ms[t] += __shfl_xor(ms[t], off);
    }
#pragma unroll
    for (int t = 0; t < NT - 1; ++t) sum[t] = 0.f;
    for (int c0 = 0; c0 < d; c0 += kWave) {
        float T[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) T[t] = 0.f;
        if (c0 + lane < d) {
#pragma unroll 4
            for (int s = w; s < a.splits; s += 4) {
#pragma unroll
                for (int t = 0; t < NT; ++t) T[t] += a.part[((s * R + r) * NT + t) * d + c0 + lane];
            }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t) part_s[w][t][lane] = T[t];
        __syncthreads();
        if (w != 0) continue;
        tier_outputs<NT, 1>(a.ks, R, r, d, c0, d - c0, lane, ms,
                            [&](int t, int) { return part_s[0][t][lane] + part_s[1][t][lane] + part_s[2][t][lane] + part_s[3][t][lane]; },
                            a.o, a.o_s, ss);
#pragma unroll
        for (int t = 0; t < NT - 1; ++t) sum[t] += ss[t];
    }
    if (threadIdx.x == 0) tier_gaps<NT>(a.ks, R, r, ms, sum, a.gap, a.dropped);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <typename T, int DC, int RT>
static void scores_t(const T *q, const T *k, const float *scale, const float *bias, int64_t H, int64_t G, int64_t n,
                     int d, float *z, hipStream_t st) {
    const int64_t units = H * ((G + 16 * RT - 1) / (16 * RT)), tiles = (n + 15) / 16;
    // a workgroup's four waves take one 16-key tile each per step; about eight
    // workgroups per CU, and no split shorter than one step
    int64_t splits = (2048 + units - 1) / units;
    const int64_t most = (tiles + 3) / 4;
    if (splits > most) splits = most;
    const int vec = d % (16 / (int)sizeof(T)) == 0 && ((uintptr_t)q | (uintptr_t)k) % 16 == 0;
    const size_t lds = (size_t)4 * 64 * (DC * 2 * sizeof(T) + 4) * 4;
    hipLaunchKernelGGL((scores_kernel<T, DC, RT>), dim3((unsigned)(units * splits)), dim3(256), lds, st, q, k, scale,
                       bias, H, G, n, d, (int)splits, vec, z);
}

template <typename T>
static void scores_dc(const T *q, const T *k, const float *scale, const float *bias, int64_t H, int64_t G, int64_t n,
                      int d, float *z, hipStream_t st) {
    // Row tiles per wave: two past 16 rows, so that a key tile turned through LDS
    // serves both; where they don't fit the registers (float32 past 128 columns),
    // one.  A call with one, two and four tiles, bf16 of 128 columns: 64 units of
    // 24 rows of 8192 keys 144, 144 and 179 us (four are mostly padding), 32 of 128
    // rows 258, 247 and 253; float32 of 64 columns 272, 254 and 259.  Least gain:
    // 16 units of 48 rows of 8192 bf16 keys 94, 98 and 105.
    const bool two = G > 16;
    if (d <= 64) two ? scores_t<T, 2, 2>(q, k, scale, bias, H, G, n, d, z, st) : scores_t<T, 2, 1>(q, k, scale, bias, H, G, n, d, z, st);
    else if (d <= 128) two ? scores_t<T, 4, 2>(q, k, scale, bias, H, G, n, d, z, st) : scores_t<T, 4, 1>(q, k, scale, bias, H, G, n, d, z, st);
    else if (sizeof(T) == 2 && two) scores_t<T, 8, 2>(q, k, scale, bias, H, G, n, d, z, st);
    else scores_t<T, 8, 1>(q, k, scale, bias, H, G, n, d, z, st);
}

hipError_t launch_scores(int dtype, const void *q, const void *k, const float *scale,
                         const float *bias, int64_t H, int64_t G, int64_t n, int d, float *z,
                         hipStream_t st) {
    if (dtype == FW_BF16) scores_dc((const uint16_t *)q, (const uint16_t *)k, scale, bias, H, G, n, d, z, st);
    else scores_dc((const float *)q, (const float *)k, scale, bias, H, G, n, d, z, st);
    return hipGetLastError();
}

hipError_t launch_select(const float *z, int64_t R, int64_t n, const KsArg &ks, float *row_m,
                         float *row_l, uint32_t *thr_key, int32_t *thr_cut, int32_t *topk_idx,
                         int kmax, hipStream_t st) {
    int sort_len = 1;
    while (sort_len < kmax) sort_len <<= 1;
    int cap = kSelList;
    if (topk_idx) cap = kmax + kSelList / 2 > sort_len ? kmax + kSelList / 2 : sort_len;
    const size_t lds = (size_t)cap * sizeof(unsigned long long);
    // 16 waves for up to a row per CU, where a row's passes are one chain per
    // thread, and for rows that four don't hold in registers (8192 logits); with
    // many rows, whose barriers then bound it, only from where reading them again
    // costs more, sooner when long index lists are ranked.  A call with four and 16
    // waves: 256 rows of 2500 logits 32 and 30 us, of 8192 51 and 44; 512 of 2500 38
    // and 41, of 8192 66 and 67, of 12,000 106 and 86; 8192 rows of 8200 438 and 568,
    // of 12,288 655 and 742 (3072 indices: 1056 and 927), of 16,384 893 and 920, of
    // 32,768 1779 and 1603 (8192 indices: 6637 and 2522).
    const bool list = topk_idx && kmax >= 1024;
    // (a grid's threads are counted in 32 bits)
    const bool big = n > (R <= 256 ? 2048 : R <= 768 ? 8192 : list ? 9216 : 12288) && R < ((int64_t)1 << 22);
#define FW_SELECT(NTH, PER)                                                                                        \
    hipLaunchKernelGGL((select_kernel<NTH, PER>), dim3((unsigned)R), dim3(NTH), lds, st, z, R, n, ks, row_m, row_l, \
                       thr_key, thr_cut, topk_idx, kmax, sort_len, cap)
    if (big) {
        if (n <= 8 * 1024) FW_SELECT(1024, 8);
        else if (n <= 32 * 1024) FW_SELECT(1024, 32);
        else FW_SELECT(1024, 0);
    } else {
        if (n <= 8 * 256) FW_SELECT(256, 8);
        else if (n <= 32 * 256) FW_SELECT(256, 32);
        else FW_SELECT(256, 0);
    }
#undef FW_SELECT
    return hipGetLastError();
}

// Key splits, at least eight 32-key blocks each (two per wave).  bf16: about
// 512 workgroups, the two per CU that run at once (64 units of 4 rows of 5003
// keys: a quarter less than with 1024); float32, whose products run at a
// sixteenth of the rate: about 1024 (16 units of 90 rows of 1999 keys: 35 us
// against 42 with 512).
int tiers_splits(int dtype, int64_t H, int64_t G, int64_t n) {
    const int64_t tiles = H * ((G + 15) / 16), most = (n + 255) / 256;
    const int64_t want = dtype == FW_BF16 ? 512 : 1024;
    int64_t s = (want + tiles - 1) / tiles;
    if (s > most) s = most;
    if (s > 64) s = 64;  // the combination takes one split per lane
    return (int)s;
}

template <typename T, int CPL, int NT>
static void tiers_t(const TierArgs &a, hipStream_t st) {
    const int64_t tiles = a.H * ((a.G + 15) / 16);
    hipLaunchKernelGGL((tiers_kernel<T, CPL, NT>), dim3((unsigned)(tiles * a.splits)), dim3(256), 0, st, a);
    if (a.splits > 1)
        hipLaunchKernelGGL((tiers_combine_kernel<NT>), dim3((unsigned)(a.H * a.G)), dim3(256), 0, st, a);
}

template <typename T>
static void tiers_nt(const TierArgs &a, hipStream_t st) {
    const bool wide = a.d > 64;
    switch (a.ks.n) {
        case 1: wide ? tiers_t<T, 8, 2>(a, st) : tiers_t<T, 4, 2>(a, st); break;
        case 2: wide ? tiers_t<T, 8, 3>(a, st) : tiers_t<T, 4, 3>(a, st); break;
        case 3: wide && sizeof(T) == 2 && a.vec ? tiers_t<T, 8, 4>(a, st) : tiers_t<T, 4, 4>(a, st); break;
        case 4: tiers_t<T, 4, 5>(a, st); break;
        case 5: tiers_t<T, 4, 6>(a, st); break;
        case 6: tiers_t<T, 4, 7>(a, st); break;
        case 7: tiers_t<T, 4, 8>(a, st); break;
        default: tiers_t<T, 4, 9>(a, st); break;
    }
}

hipError_t launch_tiers(int dtype, const void *v, const float *z, const float *row_m, const float *row_l,
                        const uint32_t *thr_key, const int32_t *thr_cut, int64_t H, int64_t G, int64_t n, int d,
                        const KsArg &ks, float *o, float *o_s, float *gap, float *dropped, int splits, float *part,
                        float *part_m, hipStream_t st) {
    TierArgs a{};
    a.v = v;
    a.z = z;
    a.row_m = row_m;
    a.row_l = row_l;
    a.thr_key = thr_key;
    a.thr_cut = thr_cut;
    a.H = H;
    a.G = G;
    a.n = n;
    a.d = d;
    a.splits = splits;
    a.ks = ks;
    a.o = o;
    a.o_s = o_s;
    a.gap = gap;
    a.dropped = dropped;
    a.part = part;
    a.part_m = part_m;
    // buffer loads: whole 16-byte chunks of a value row, 16 rows of logits within 4 GiB
    a.vec = d % 8 == 0 && (uintptr_t)v % 16 == 0 && n < (1ll << 25);
    if (dtype == FW_BF16) tiers_nt<uint16_t>(a, st);
    else tiers_nt<float>(a, st);
    return hipGetLastError();
}

}  // namespace fw
