// Observation-window importance and the per-unit dropped-mass curve
// (Section 4, "ContourKV"; Definition 2.1's least achievable dropped mass as
// a function of the budget).
//
//   r_j      = (1/G) sum_g softmax_j(z_g),  z_gj = scale_h <q_g, k_j> + bias_j
//   curve[k] = sum of all but the k largest r, k = 0..n (curve[n] = 0)
//
// Passes: (1) per key chunk, each window row's local max and local sum of
// exponentials; (2) combine the chunks per row in a fixed order; (3) recompute
// the logits, weights and their window mean; (4) per unit, a stable LSD radix
// sort of the scores (descending, ties by index); (5) a float64 suffix scan.
#include "fw_internal.hpp"
#include "topk_fused.hpp"

namespace fw {

namespace {
constexpr int kChunk = 512;   // keys per workgroup in the logit passes
constexpr int kRowGrp = 16;   // window rows per LDS tile
constexpr int kSortThreads = 1024;

// rows of fewer columns take a key per thread (window_thin_kernel)
template <typename T> constexpr int thin_cols() { return sizeof(T) == 2 ? 24 : 16; }

// words per row of a staged key tile of ch chunks: four times an odd number, so
// that 16 rows' reads of a chunk meet no bank twice
__host__ __device__ constexpr int window_rs(int ch) { return ch / 4 % 2 ? ch : ch + 4; }

// Per window row of the group (16 threads each): the largest of the chunk's
// logits zt and the sum of exponentials over it, into part_m and part_s.
__device__ __forceinline__ void chunk_stats(const float (*zt)[kChunk + 1], float *red, int gn, int64_t row0, int nchunks,
                                            int ch, float *part_m, float *part_s) {
    const int tid = threadIdx.x, g = tid / 16, l = tid % 16;
    float m = -INFINITY;
    for (int jl = l; jl < kChunk; jl += 16) m = fmaxf(m, zt[g][jl]);
    red[tid] = m;
    __syncthreads();
    m = red[g * 16];
    for (int t = 1; t < 16; ++t) m = fmaxf(m, red[g * 16 + t]);
    __syncthreads();
    float s = 0.f;
    for (int jl = l; jl < kChunk; jl += 16) s += (zt[g][jl] == -INFINITY) ? 0.f : expf(zt[g][jl] - m);
    red[tid] = s;
    __syncthreads();
    if (l == 0 && g < gn) {
        float st = 0.f;
        for (int t = 0; t < 16; ++t) st += red[g * 16 + t];
        part_m[(row0 + g) * nchunks + ch] = m;
        part_s[(row0 + g) * nchunks + ch] = st;
    }
}
}  // namespace

// Pass 1 (MODE 0) and pass 3 (MODE 1) share the logit computation: a
// workgroup takes kChunk keys, 16 window rows at a time; each wave a quarter of
// the keys in tiles of 16, read as whole rows, turned through LDS and
// multiplied on the float32 MFMA.  Its chain gives, bit for bit, the fused
// multiply-adds over the columns in order (see scores_kernel), and the sums
// over keys and rows below run in one fixed order, so the scores and the order
// built on them do not depend on the tiling.  Takes every window that
// k_window.hip and window_thin_kernel do not.  64 cells of 64 rows of 8192
// float32 keys of 128 columns: 0.42 ms a call, 1.90 ms with one thread per key
// reading its own row; of 20,000 keys of 129 to 192 bf16 columns (DC = 6) 2.09
// ms at 129, 2.55 padded to 256.
template <typename T, int DC, int MODE>
__global__ void __launch_bounds__(256)
window_logits_kernel(const T *__restrict__ q, const T *__restrict__ k, const float *__restrict__ scale,
                     const float *__restrict__ bias, int64_t G, int64_t n, int d, int nchunks, int vec,
                     float *__restrict__ part_m, float *__restrict__ part_s,
                     const float *__restrict__ row_m, const float *__restrict__ row_il,
                     float *__restrict__ importance) {
    constexpr bool B16 = sizeof(T) == 2;
    constexpr int E = 16 / (int)sizeof(T);  // elements per 16-byte chunk
    constexpr int CH = DC * 32 / E;         // chunks per row
    constexpr int LD = CH / 4;              // loads per lane and tile (16 rows x CH chunks / 64)
    constexpr int RS = window_rs(CH);       // words per row and kg
    extern __shared__ __align__(16) uint32_t lds_w[];  // [wave][kg][row][chunk]
    __shared__ float zt[MODE == 0 ? kRowGrp : 1][kChunk + 1];  // logits; MODE 1: the keys' sums
    __shared__ float red[256];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m16 = lane & 15, kg = lane >> 4;
    uint32_t *tile = lds_w + w * (64 * RS);
    const uint4 *mine = (const uint4 *)(tile + (kg * 16 + m16) * RS);
    const int64_t h = (uint32_t)blockIdx.x / (uint32_t)nchunks;
    const int ch = (uint32_t)blockIdx.x % (uint32_t)nchunks;
    const int64_t j0 = (int64_t)ch * kChunk;
    const T *qh = q + h * G * d;
    const T *kh = k + h * n * d;
    const float sc = scale ? scale[h] : (float)(1.0 / sqrt((double)d));
    uint4 raw[LD];
    auto load = [&](const T *base, int64_t row0, int64_t rows) {
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int id = lane + 64 * i, c = (id % CH) * E;
            const int64_t j = row0 + id / CH;
            raw[i] = make_uint4(0u, 0u, 0u, 0u);
            if (j >= rows || c >= d) continue;
            if (vec) {
                raw[i] = *(const uint4 *)(base + j * d + c);
            } else if (B16 && c + E <= d) {  // a whole chunk at any alignment, not eight loads
                __builtin_memcpy(&raw[i], base + j * d + c, 16);
            } else {
                T x[E];
#pragma unroll
                for (int e = 0; e < E; ++e) x[e] = c + e < d ? base[j * d + c + e] : (T)0;
                raw[i] = __builtin_bit_cast(uint4, x);
            }
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
    if (MODE == 1)
        for (int e = tid; e < kChunk; e += 256) zt[0][e] = 0.f;
    __syncthreads();
    for (int64_t g0 = 0; g0 < G; g0 += kRowGrp) {
        const int gn = (G - g0 < kRowGrp) ? (int)(G - g0) : kRowGrp;
        uint4 qf[LD];
        load(qh, g0, G);
        stage();
#pragma unroll
        for (int f = 0; f < LD; ++f) qf[f] = mine[f];
        // lane: key m16 of a tile, window rows 4 kg .. 4 kg + 3 of the group
        float rm[4], ril[4];
        if (MODE == 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool ok = 4 * kg + i < gn;
                rm[i] = ok ? row_m[h * G + g0 + 4 * kg + i] : 0.f;
                ril[i] = ok ? row_il[h * G + g0 + 4 * kg + i] : 0.f;
            }
        }
        constexpr int KT = kChunk / 64;  // key tiles per wave
        load(kh, j0 + w * (kChunk / 4), n);
        for (int t = 0; t < KT; ++t) {
            const int jl = w * (kChunk / 4) + 16 * t + m16;
            const int64_t j = j0 + jl;
            stage();
            if (t + 1 < KT) load(kh, j0 + w * (kChunk / 4) + 16 * (t + 1), n);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int f = 0; f < LD; ++f) {
                const uint4 kf = mine[f];
                const uint32_t kw[4] = {kf.x, kf.y, kf.z, kf.w}, qw[4] = {qf[f].x, qf[f].y, qf[f].z, qf[f].w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if constexpr (B16) {
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(qw[c] << 16),
                                                                   __uint_as_float(kw[c] << 16), acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(qw[c] & 0xFFFF0000u),
                                                                   __uint_as_float(kw[c] & 0xFFFF0000u), acc, 0, 0, 0);
                    } else {
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(qw[c]), __uint_as_float(kw[c]), acc,
                                                                   0, 0, 0);
                    }
                }
            }
            const float bj = (bias && j < n) ? bias[j] : 0.f;
            if (MODE == 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int g = 4 * kg + i;
                    zt[g][jl] = (j < n && g < gn) ? fmaf(sc, acc[i], bj) : -INFINITY;
                }
            } else {
                // the key's sum over the rows in order: lane group after lane group
                float part[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) part[i] = expf(fmaf(sc, acc[i], bj) - rm[i]);
                float r = zt[0][jl];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    float y = r;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (4 * x + i < gn) y = fmaf(part[i], ril[i], y);
                    r = __shfl(y, 16 * x + m16);
                }
                if (kg == 0) zt[0][jl] = r;
            }
        }
        if (MODE == 0) {
            __syncthreads();
            chunk_stats(zt, red, gn, h * G + g0, nchunks, ch, part_m, part_s);
        }
        __syncthreads();
    }
    if (MODE == 1) {
        const float invG = 1.0f / (float)G;
        for (int e = tid; e < kChunk; e += 256)
            if (j0 + e < n) importance[h * n + j0 + e] = zt[0][e] * invG;
    }
}

// The same passes for rows of fewer than thin_cols columns, two keys per
// thread: the matrix tiles would be mostly padding and the sums over a key's
// rows cross lanes.  Same bits.  64 cells of 64 rows of 20,000 keys, a call, here
// and on the tiles: 4 bf16 columns 278 us and 549 (padded to 64); 20 bf16 columns
// 405 and 416, 30 508 and 427; 16 float32 columns 393 and 408, 20 486 and 414.
template <typename T, int MODE>
__global__ void __launch_bounds__(256)
window_thin_kernel(const T *__restrict__ q, const T *__restrict__ k, const float *__restrict__ scale,
                   const float *__restrict__ bias, int64_t G, int64_t n, int d, int nchunks,
                   float *__restrict__ part_m, float *__restrict__ part_s, const float *__restrict__ row_m,
                   const float *__restrict__ row_il, float *__restrict__ importance) {
    __shared__ float Qs[kRowGrp][thin_cols<T>()];
    __shared__ float zt[MODE == 0 ? kRowGrp : 1][kChunk + 1];
    __shared__ float red[256];
    const int tid = threadIdx.x;
    const int64_t h = (uint32_t)blockIdx.x / (uint32_t)nchunks;
    const int ch = (uint32_t)blockIdx.x % (uint32_t)nchunks;
    const int64_t j0 = (int64_t)ch * kChunk;
    const T *qh = q + h * G * d;
    const T *kh = k + h * n * d;
    const float sc = scale ? scale[h] : (float)(1.0 / sqrt((double)d));
    float racc[2] = {0.f, 0.f};
    for (int64_t g0 = 0; g0 < G; g0 += kRowGrp) {
        const int gn = (G - g0 < kRowGrp) ? (int)(G - g0) : kRowGrp;
        for (int e = tid; e < kRowGrp * d; e += 256) {
            const int rr = e / d, cc = e % d;
            Qs[rr][cc] = (rr < gn) ? Elem<T>::load(qh, (g0 + rr) * d + cc) : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int jl = tid + 256 * u;
            const int64_t j = j0 + jl;
            float acc[kRowGrp];
#pragma unroll
            for (int g = 0; g < kRowGrp; ++g) acc[g] = 0.f;
            if (j < n) {
                for (int c = 0; c < d; ++c) {
                    const float kv = Elem<T>::load(kh, j * d + c);
#pragma unroll
                    for (int g = 0; g < kRowGrp; ++g) acc[g] = fmaf(Qs[g][c], kv, acc[g]);
                }
            }
            const float bj = (bias && j < n) ? bias[j] : 0.f;
#pragma unroll
            for (int g = 0; g < kRowGrp; ++g) {
                const float zz = fmaf(sc, acc[g], bj);
                if (MODE == 0) {
                    zt[g][jl] = (j < n && g < gn) ? zz : -INFINITY;
                } else if (j < n && g < gn) {
                    const int64_t row = h * G + g0 + g;
                    racc[u] = fmaf(expf(zz - row_m[row]), row_il[row], racc[u]);
                }
            }
        }
        if (MODE == 0) {
            __syncthreads();
            chunk_stats(zt, red, gn, h * G + g0, nchunks, ch, part_m, part_s);
        }
        __syncthreads();
    }
    if (MODE == 1) {
        const float invG = 1.0f / (float)G;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t j = j0 + tid + 256 * u;
            if (j < n) importance[h * n + j] = racc[u] * invG;
        }
    }
}

// Pass 2: combine the per-chunk statistics of every window row.
__global__ void window_combine_kernel(int64_t rows, int nchunks, const float *part_m,
                                      const float *part_s, float *row_m, float *row_il) {
    const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= rows) return;
    float m = -INFINITY;
    for (int c = 0; c < nchunks; ++c) m = fmaxf(m, part_m[row * nchunks + c]);
    double s = 0.0;
    for (int c = 0; c < nchunks; ++c) {
        const float pm = part_m[row * nchunks + c];
        if (pm != -INFINITY) s += (double)part_s[row * nchunks + c] * exp((double)pm - (double)m);
    }
    row_m[row] = m;
    row_il[row] = (float)(1.0 / s);
}

// Pass 4: stable LSD radix sort of one unit's scores, descending (keys are
// the complement of the order-preserving bits), payload = key index (only
// when the order is asked for: a separate instance, whose payload registers
// and LDS traffic are gone).  One workgroup per unit; four 8-bit passes.
// The digit histograms of all four passes come from one read.  Each pass
// takes tiles of kSortTile keys, 8 per thread in index order (wave, slot,
// lane): a key's rank among the equal digits of its wave comes from ballots
// slot by slot with running per-wave counters, the tile is placed
// digit-ordered in LDS, and then written out as contiguous runs (coalesced)
// at the digit's running global offset.  (Longer tiles, 12 or 16 keys per
// thread, run out of registers at 16 waves per workgroup.)
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortE = 8;
constexpr int kSortTile = kSortThreads * kSortE;
template <bool with_vals>
__global__ void __launch_bounds__(kSortThreads)
unit_sort_kernel(const float *__restrict__ importance, int64_t n, uint32_t *keys_a, uint32_t *keys_b,
                 int32_t *vals_a, int32_t *vals_b) {
    __shared__ int gb[4][256];             // per pass: running global offset of each digit
    __shared__ int wc[kSortWaves][256];    // per wave: digit counts, then their cross-wave prefix
    __shared__ int tdp[256], ttot[256];    // tile: digit prefix, digit totals
    __shared__ uint32_t stk[kSortTile];
    __shared__ int32_t stv[with_vals ? kSortTile : 1];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t h = blockIdx.x;
    const float *imp = importance + h * n;
    uint32_t *ka = keys_a + h * n, *kb = keys_b + h * n;
    int32_t *va = vals_a + h * n, *vb = vals_b + h * n;
    const uint64_t below_mask = (1ull << lane) - 1ull;
    for (int i = tid; i < 4 * 256; i += kSortThreads) (&gb[0][0])[i] = 0;
    __syncthreads();
    // (scores of a unit often share their top bytes: a digit common to every
    // live lane of the wave is added once)
    for (int64_t j0 = (int64_t)wv * 64; j0 < n; j0 += kSortThreads) {
        const int64_t j = j0 + lane;
        const bool live = j < n;
        const uint32_t key = live ? ~ord_key(imp[j]) : 0u;
        const uint64_t lv = __ballot(live);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const uint32_t d = (key >> (8 * p)) & 255u;
            const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
            if (__ballot(live && d == d0) == lv) {
                if (lane == 0) atomicAdd(&gb[p][d0], __popcll(lv));
            } else if (live) {
                atomicAdd(&gb[p][d], 1);
            }
        }
    }
    __syncthreads();
    if (wv < 4) {  // exclusive prefix over the digits, one wave per pass
        int v[4], sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) { v[q] = gb[wv][4 * lane + q]; sum += v[q]; }
        int incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(incl, off);
            if (lane >= off) incl += y;
        }
        int run = incl - sum;
#pragma unroll
        for (int q = 0; q < 4; ++q) { gb[wv][4 * lane + q] = run; run += v[q]; }
    }
    __syncthreads();
    for (int p = 0; p < 4; ++p) {
        const int shift = 8 * p;
        const uint32_t *sk = (p & 1) ? kb : ka;
        const int32_t *sv = (p & 1) ? vb : va;
        uint32_t *dk = (p & 1) ? ka : kb;
        int32_t *dv = (p & 1) ? va : vb;
        // the keys of tile t0 + kSortTile load while tile t0 is ranked and written
        uint32_t nkey[kSortE];
        int32_t nval[kSortE];
        auto load_tile = [&](int64_t t0) {
#pragma unroll
            for (int s = 0; s < kSortE; ++s) {
                const int64_t e = t0 + (int64_t)wv * 64 * kSortE + s * 64 + lane;
                const bool live = e < n;
                if (p == 0) {
                    nkey[s] = live ? ~ord_key(imp[e]) : 0u;
                    nval[s] = (int32_t)e;
                } else {
                    nkey[s] = live ? sk[e] : 0u;
                    nval[s] = (with_vals && live) ? sv[e] : 0;
                }
            }
        };
        load_tile(0);
        for (int64_t t0 = 0; t0 < n; t0 += kSortTile) {
            for (int i = lane; i < 256; i += 64) wc[wv][i] = 0;
            uint32_t key[kSortE];
            int32_t val[kSortE];
            int lr[kSortE];
            // the slot's digit (256: past the end), recomputed where used
            const int64_t ebase = t0 + (int64_t)wv * 64 * kSortE + lane;
            auto digit = [&](int s) -> int {
                return (ebase + s * 64 < n) ? (int)((key[s] >> shift) & 255u) : 256;
            };
#pragma unroll
            for (int s = 0; s < kSortE; ++s) {
                key[s] = nkey[s];
                val[s] = nval[s];
            }
            if (t0 + kSortTile < n) load_tile(t0 + kSortTile);
#pragma unroll
            for (int s = 0; s < kSortE; ++s) {
                // lanes of this wave holding the same digit in this slot
                const int dg = digit(s);
                uint64_t same = __ballot(dg < 256);
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const uint64_t bal = __ballot((dg >> b) & 1);
                    same &= ((dg >> b) & 1) ? bal : ~bal;
                }
                const int below = __popcll(same & below_mask);
                int pre = 0;
                if (dg < 256) pre = wc[wv][dg];
                lr[s] = pre + below;
                if (dg < 256 && below == 0) wc[wv][dg] = pre + __popcll(same);
            }
            lds_barrier();
            if (tid < 256) {
                int c[kSortWaves];
#pragma unroll
                for (int w = 0; w < kSortWaves; ++w) c[w] = wc[w][tid];
                int run = 0;
#pragma unroll
                for (int w = 0; w < kSortWaves; ++w) { wc[w][tid] = run; run += c[w]; }
                ttot[tid] = run;
            }
            lds_barrier();
            if (wv == 0) {
                int v[4], sum = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) { v[q] = ttot[4 * lane + q]; sum += v[q]; }
                int incl = sum;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const int y = __shfl_up(incl, off);
                    if (lane >= off) incl += y;
                }
                int run = incl - sum;
#pragma unroll
                for (int q = 0; q < 4; ++q) { tdp[4 * lane + q] = run; run += v[q]; }
            }
            lds_barrier();
#pragma unroll
            for (int s = 0; s < kSortE; ++s) {
                const int dg = digit(s);
                if (dg < 256) {
                    const int lp = tdp[dg] + wc[wv][dg] + lr[s];
                    stk[lp] = key[s];
                    if (with_vals) stv[lp] = val[s];
                }
            }
            lds_barrier();
            const int cnt = (int)((n - t0 < kSortTile) ? n - t0 : kSortTile);
            for (int i = tid; i < cnt; i += kSortThreads) {
                const uint32_t kk = stk[i];
                const int d = (int)((kk >> shift) & 255u);
                const int64_t gp = (int64_t)gb[p][d] + (i - tdp[d]);
                dk[gp] = kk;
                if (with_vals) dv[gp] = stv[i];
            }
            lds_barrier();
            if (tid < 256) gb[p][tid] += ttot[tid];
            lds_barrier();
        }
        __syncthreads();  // this pass's global writes are the next pass's input
    }
    // four passes: the result is back in keys_a / vals_a
}

// Pass 5: curve[k] = sum_{i >= k} sorted[i] (float64) read from the sorted
// keys themselves, and the order.  Tiles of 8192 positions from the end: a
// coalesced load into LDS, per-thread sums of 8 consecutive positions, a
// suffix scan of the thread sums (wave shuffles, then across waves), and a
// coalesced store.
constexpr int kCurveTile = 8 * kSortThreads;
__global__ void __launch_bounds__(kSortThreads)
unit_curve_kernel(const uint32_t *__restrict__ keys, int64_t n, const int32_t *__restrict__ vals,
                  float *__restrict__ curve, int32_t *__restrict__ order) {
    __shared__ float tile[kCurveTile];
    __shared__ double wsum[kSortThreads / 64];
    __shared__ double carry_s;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t h = blockIdx.x;
    const uint32_t *kh = keys + h * n;
    float *ch = curve + h * (n + 1);
    if (tid == 0) carry_s = 0.0;
    for (int64_t t0 = ((n - 1) / kCurveTile) * kCurveTile; t0 >= 0; t0 -= kCurveTile) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t e = t0 + i * kSortThreads + tid;
            tile[i * kSortThreads + tid] = e < n ? key_to_float(~kh[e]) : 0.f;
        }
        __syncthreads();
        double part = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) part += (double)tile[8 * tid + q];
        // inclusive suffix sum over the lanes of this wave
        double suf = part;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double y = __shfl_down(suf, off);
            if (lane + off < 64) suf += y;
        }
        if (lane == 0) wsum[wv] = suf;  // the wave's total
        __syncthreads();
        double after = carry_s;  // everything right of this wave
        for (int w2 = wv + 1; w2 < kSortThreads / 64; ++w2) after += wsum[w2];
        double acc = after + (suf - part);  // right of this thread's 8 positions
#pragma unroll
        for (int q = 7; q >= 0; --q) {
            acc += (double)tile[8 * tid + q];
            tile[8 * tid + q] = (float)acc;
        }
        __syncthreads();
        if (tid == 0) {
            double tot = 0.0;
            for (int w2 = 0; w2 < kSortThreads / 64; ++w2) tot += wsum[w2];
            carry_s += tot;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t e = t0 + i * kSortThreads + tid;
            if (e < n) {
                ch[e] = tile[i * kSortThreads + tid];
                if (order) order[h * n + e] = vals[h * n + e];
            }
        }
        __syncthreads();
    }
    if (tid == 0) ch[n] = 0.f;
}

// ---------------------------------------------------------------------------
namespace {
struct CurveLayout {
    float *part_m, *part_s, *row_m, *row_il;
    uint32_t *ka, *kb;
    int32_t *va, *vb;
    size_t bytes;
};

CurveLayout curve_layout(const fw_rows &rows, void *ws) {
    const size_t H = rows.H, G = rows.G, n = rows.n;
    const size_t nch = (n + kChunk - 1) / kChunk;
    CurveLayout L{};
    size_t off = 0;
    char *base = (char *)ws;
    auto take = [&](size_t bytes) -> void * {
        off = align_up(off, 256);
        void *p = base ? base + off : nullptr;
        off += bytes;
        return p;
    };
    L.part_m = (float *)take(H * G * nch * 4);
    L.part_s = (float *)take(H * G * nch * 4);
    L.row_m = (float *)take(H * G * 4);
    L.row_il = (float *)take(H * G * 4);
    L.ka = (uint32_t *)take(H * n * 4);
    L.kb = (uint32_t *)take(H * n * 4);
    L.va = (int32_t *)take(H * n * 4);
    L.vb = (int32_t *)take(H * n * 4);
    L.bytes = align_up(off, 256);
    return L;
}
}  // namespace

size_t curve_ws_bytes(const fw_rows &rows) { return curve_layout(rows, nullptr).bytes; }

// both logit passes of a window that k_window.hip does not take; DC chunks of
// 32 columns, 0: the thin kernel
template <typename T, int DC>
static void window_general(const fw_rows &rows, const CurveLayout &L, float *importance, hipStream_t st) {
    const int64_t H = rows.H, G = rows.G, n = rows.n;
    const int d = (int)rows.d, nch = (int)((n + kChunk - 1) / kChunk);
    const dim3 grid((unsigned)(H * nch));
    const T *q = (const T *)rows.q, *k = (const T *)rows.k;
    const int vec = d % (16 / (int)sizeof(T)) == 0 && ((uintptr_t)q | (uintptr_t)k) % 16 == 0;
    const size_t lds = (size_t)4 * 64 * window_rs(DC * 2 * (int)sizeof(T)) * 4;
    if constexpr (DC == 0)
        hipLaunchKernelGGL((window_thin_kernel<T, 0>), grid, dim3(256), 0, st, q, k, rows.scale, rows.bias, G, n, d,
                           nch, L.part_m, L.part_s, nullptr, nullptr, nullptr);
    else
        hipLaunchKernelGGL((window_logits_kernel<T, DC, 0>), grid, dim3(256), lds, st, q, k, rows.scale, rows.bias, G,
                           n, d, nch, vec, L.part_m, L.part_s, nullptr, nullptr, nullptr);
    hipLaunchKernelGGL(window_combine_kernel, dim3((unsigned)((H * G + 255) / 256)), dim3(256), 0, st, H * G, nch,
                       L.part_m, L.part_s, L.row_m, L.row_il);
    if constexpr (DC == 0)
        hipLaunchKernelGGL((window_thin_kernel<T, 1>), grid, dim3(256), 0, st, q, k, rows.scale, rows.bias, G, n, d,
                           nch, nullptr, nullptr, L.row_m, L.row_il, importance);
    else
        hipLaunchKernelGGL((window_logits_kernel<T, DC, 1>), grid, dim3(256), lds, st, q, k, rows.scale, rows.bias, G,
                           n, d, nch, vec, nullptr, nullptr, L.row_m, L.row_il, importance);
}

template <typename T>
static hipError_t curve_impl(const fw_rows &rows, float *importance, float *curve, int32_t *order,
                             void *ws, hipStream_t st) {
    CurveLayout L = curve_layout(rows, ws);
    const int64_t H = rows.H, n = rows.n;
    if (window_mfma_supported(rows)) {
        // bf16, d = 128, up to 64 window rows: MFMA scores (k_window.hip)
        launch_window_mfma(rows, L.part_m, L.part_s, L.row_m, L.row_il, importance, st);
    } else if (rows.d < thin_cols<T>()) {
        window_general<T, 0>(rows, L, importance, st);
    } else {  // as little padding as chunks of 32 and, past 128, 64 columns allow
        switch ((rows.d + 31) / 32) {
            case 1: window_general<T, 1>(rows, L, importance, st); break;
            case 2: window_general<T, 2>(rows, L, importance, st); break;
            case 3: window_general<T, 3>(rows, L, importance, st); break;
            case 4: window_general<T, 4>(rows, L, importance, st); break;
            case 5:
            case 6: window_general<T, 6>(rows, L, importance, st); break;
            default: window_general<T, 8>(rows, L, importance, st); break;
        }
    }
    if (order)
        hipLaunchKernelGGL((unit_sort_kernel<true>), dim3((unsigned)H), dim3(kSortThreads), 0, st,
                           importance, n, L.ka, L.kb, L.va, L.vb);
    else
        hipLaunchKernelGGL((unit_sort_kernel<false>), dim3((unsigned)H), dim3(kSortThreads), 0, st,
                           importance, n, L.ka, L.kb, L.va, L.vb);
    hipLaunchKernelGGL(unit_curve_kernel, dim3((unsigned)H), dim3(kSortThreads), 0, st,
                       (const uint32_t *)L.ka, n, (const int32_t *)L.va, curve, order);
    return hipGetLastError();
}

hipError_t launch_curve(const fw_rows &rows, float *importance, float *curve, int32_t *order,
                        void *ws, hipStream_t st) {
    if (rows.dtype == FW_BF16) return curve_impl<uint16_t>(rows, importance, curve, order, ws, st);
    return curve_impl<float>(rows, importance, curve, order, ws, st);
}

}  // namespace fw
