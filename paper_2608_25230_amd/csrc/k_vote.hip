// Group vote (Section 2.1: deployment fixes one kept set per key/value head
// and applies it to the group of query rows that share the head), float64.
//
// One workgroup per group (the rows of all query heads of a unit at one
// position).  The member rows are taken RB at a time, so that every key and
// value row read serves RB of them: logits over the unit's keys, then, each
// row on its own NT / RB threads, softmax and the row's own top-mass set
// (logit desc, index asc); the dense outputs of the RB rows; the error of each
// own set.  Then the vote: the s keys of largest summed mass (index asc on
// ties).  Finally each member's forced-weight error with the vote's set and
// the vote's dropped mass.
//
// RB is the largest of 4, 2, 1 whose rows fit LDS (float64 logits, then
// weights, of RB rows; a group of at most RB rows needs no array of summed
// masses, and the vote keys' weights are read back instead of formed again).
// Bound by the float64 multiply-adds and by the lanes' reductions of the
// logits, one workgroup per CU (four rows at a time spill 80 of 256 registers,
// two 51): 1536 groups of 4 rows, 4096 bf16 keys of 128 columns: 2.08 ms, 3.12 ms
// one row at a time.
#include "fw_internal.hpp"
#include "instance64.hpp"
#include "rowpass.hpp"

namespace fw {

namespace {

constexpr int kVoteList = 32;  // sets up to this size are picked by waves and merged

struct VoteLds {
    size_t xq, red, own, vote, rowsc, mu, pk, zz, score, total;
};

// Layout for RB rows at a time; score only when the group has more than RB.
__host__ __device__ inline VoteLds vote_lds(int64_t N, int d, int gs, int s, int RB) {
    VoteLds L{};
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 16); return at; };
    L.xq = take((size_t)RB * d * 8);
    L.red = take(4096);  // reductions; the waves' pick lists
    L.own = take((size_t)RB * s * 4);
    L.vote = take((size_t)s * 4);
    L.rowsc = take((size_t)gs * 2 * 8);  // per member: max logit, normaliser
    L.mu = take((size_t)gs * d * 8);     // per member: dense output
    // masses of a set's keys per row: beside the reductions when they are few
    L.pk = (size_t)RB * s * 8 <= 2048 ? L.red + 2048 : take((size_t)RB * s * 8);
    L.zz = take((size_t)RB * N * 8);
    L.score = gs > RB ? take((size_t)N * 8) : 0;
    L.total = o;
    return L;
}

// rows at a time: the most that fit, no more than the group has
int vote_rows(int64_t N, int d, int gs, int s) {
    for (int rb = 4; rb > 1; rb >>= 1)
        if (rb / 2 < gs && vote_lds(N, d, gs, s, rb).total <= 160 * 1024) return rb;
    return 1;
}

struct VoteArgs {
    const void *q, *k, *v;
    const float *scale, *bias;
    int64_t H, G, N;
    int d, s, gs;
    int32_t *vote_idx;
    float *es_vote, *es_top, *dropped;
};

// Reductions and picks by teams of NW waves (threads t of the workgroup's
// team `team`); red holds one entry per wave of the workgroup.  Every thread
// of the workgroup calls them.
template <typename V, typename Op>
__device__ __forceinline__ V team_reduce(V v, V *red, int NW, Op op) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, w0 = w / NW * NW;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = op(v, __shfl_xor(v, off));
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    V r = red[w0];
    for (int i = 1; i < NW; ++i) r = op(r, red[w0 + i]);
    return r;
}

// The s keys of largest get(j) (index asc on ties) of each team's row into
// out[0, s); the keys t, t + NT, .. of [0, N) are thread t's of the team.
// Up to kVoteList keys: every wave picks its own s (each pick a wave reduction
// of the lanes' best keys; the lane that held it looks for its next), and the
// waves' lists are merged by counting ranks.  More: s picks of the whole team.
// A NaN is never picked: where fewer than s keys are left, the entries without
// one are 0 (a row with a NaN has no finite weight; its list only has to hold
// keys).
template <typename F>
__device__ void team_top(F &&get, int64_t N, int s, int *out, int t, int NT, unsigned char *red) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, NW = NT >> 6, w0 = w / NW * NW;
    double pv = INFINITY, bv = 0.0;
    int pi = -1, bi = -1;
    auto next = [&]() {  // this thread's best key after (pv, pi)
        bi = -1;
        for (int64_t j = t; j < N; j += NT) {
            const double x = get(j);
            const bool after = x < pv || (x == pv && (int)j > pi);
            if (after && (bi < 0 || x > bv)) { bv = x; bi = (int)j; }
        }
    };
    auto wave_best = [&](double &mv, int &mi) {
        mv = bv;
        mi = bi;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double ov = __shfl_xor(mv, off);
            const int oi = __shfl_xor(mi, off);
            if (top_ahead(ov, oi, mv, mi)) { mv = ov; mi = oi; }
        }
    };
    next();
    __syncthreads();
    if (s <= kVoteList) {
        double *cv = (double *)red;                            // [waves][s]
        int *ci = (int *)(red + 8 * kVoteList * 8);              // [waves][s], at most eight waves
        for (int u = 0; u < s; ++u) {
            double mv;
            int mi;
            wave_best(mv, mi);
            if (lane == 0) {
                cv[w * s + u] = mv;
                ci[w * s + u] = mi;
            }
            if (mi >= 0 && bi == mi) {
                pv = mv;
                pi = mi;
                next();
            }
        }
        for (int u = t; u < s; u += NT) out[u] = 0;
        __syncthreads();
        for (int c = t; c < NW * s; c += NT) {
            const int i = ci[w0 * s + c];
            if (i < 0) continue;
            const double x = cv[w0 * s + c];
            int rank = 0;
            for (int e = 0; e < NW * s; ++e) rank += top_ahead(cv[w0 * s + e], ci[w0 * s + e], x, i);
            if (rank < s) out[rank] = i;
        }
    } else {
        double *cv = (double *)red;
        int *ci = (int *)(red + 512);
        for (int u = 0; u < s; ++u) {
            double mv;
            int mi;
            wave_best(mv, mi);
            __syncthreads();
            if (lane == 0) {
                cv[w] = mv;
                ci[w] = mi;
            }
            __syncthreads();
            mv = cv[w0];
            mi = ci[w0];
            for (int i = 1; i < NW; ++i)
                if (top_ahead(cv[w0 + i], ci[w0 + i], mv, mi)) { mv = cv[w0 + i]; mi = ci[w0 + i]; }
            if (t == 0) out[u] = mi >= 0 ? mi : 0;
            if (mi >= 0 && bi == mi) {
                pv = mv;
                pi = mi;
                next();
            }
        }
    }
    __syncthreads();
}

// es(A) = ||sum_{i in A} p_i (v_i - mu)|| / p(A) of each team's list of keys
// with their masses (d-dimensional sums, one column per thread).
template <typename T>
__device__ double es_list(const T *vh, int d, const int *keys, const double *pk, int s, const double *mu,
                          double *red, int t, int NT) {
    double g2 = 0.0;
    for (int c = t; c < d; c += NT) {
        double g = 0.0;
#pragma unroll 4
        for (int i = 0; i < s; ++i) g = fma(pk[i], (double)Elem<T>::load(vh, (int64_t)keys[i] * d + c) - mu[c], g);
        g2 = fma(g, g, g2);
    }
    g2 = team_reduce(g2, red, NT >> 6, OpSum());
    double pm = 0.0;
    for (int i = 0; i < s; ++i) pm += pk[i];
    return sqrt(g2) / pm;
}

}  // namespace

template <typename T, int RB, int VT>
__global__ void __launch_bounds__(VT, 2) vote_group_kernel(VoteArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NT = VT / RB, NW = NT / 64;  // a row's team
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), team = tid / NT, t = tid % NT;
    const int64_t N = a.N;
    const int d = a.d, s = a.s, gs = a.gs;
    const VoteLds L = vote_lds(N, d, gs, s, RB);
    double *xq = (double *)(smem + L.xq);
    double *redd = (double *)(smem + L.red);
    int *vote = (int *)(smem + L.vote);
    double *rowsc = (double *)(smem + L.rowsc);
    double *mus = (double *)(smem + L.mu);
    double *zz = (double *)(smem + L.zz);
    double *score = (double *)(smem + L.score);
    // this thread's team's row
    int *own = (int *)(smem + L.own) + team * s;
    double *pk = (double *)(smem + L.pk) + team * s;
    double *zt = zz + team * N;
    const bool resident = gs <= RB;  // every member's weights stay in LDS

    const uint32_t T_ = (uint32_t)(a.G / gs);  // positions per unit
    const uint32_t bl = (uint32_t)xcd_order(blockIdx.x, gridDim.x);  // a unit's groups on one XCD
    const int64_t h = bl / T_, pos = bl % T_;
    const T *kh = (const T *)a.k + h * N * d;
    const T *vh = (const T *)a.v + h * N * d;
    const double scale = a.scale ? (double)a.scale[h] : (double)default_scale(d);
    constexpr int VEC = RowVec<T>::VEC;
    const bool vec = d % VEC == 0;
    const int GL = vec ? group_lanes(d, VEC) : 64, gi = lane % GL, KPW = 64 / GL, gk = lane / GL;
    const bool has = vec && gi < d / VEC;
    if (!resident)
        for (int64_t j = tid; j < N; j += VT) score[j] = 0.0;

    for (int m0 = 0; m0 < gs; m0 += RB) {
        const bool mine = m0 + team < gs;  // this team has a row (absent rows work on zeros)
        for (int e = tid; e < RB * d; e += VT) {
            const int rr = e / d, c = e - rr * d;
            const int64_t r = h * a.G + (int64_t)(m0 + rr) * T_ + pos;  // query head m0 + rr, position pos
            xq[e] = m0 + rr < gs ? (double)Elem<T>::load((const T *)a.q, r * d + c) : 0.0;
        }
        __syncthreads();
        // ---- logits of the RB rows -------------------------------------------------
        auto put = [&](int64_t j, int rr, double acc) {
            zz[rr * N + j] = scale * acc + (a.bias ? (double)a.bias[j] : 0.0);
        };
        if (vec) {
            // U keys x RB rows = 16 sums per lane
            constexpr int U = 16 / RB;
            double xr[RB][VEC];
#pragma unroll
            for (int rr = 0; rr < RB; ++rr) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) xr[rr][i] = has ? xq[rr * d + gi * VEC + i] : 0.0;
            }
            const int64_t stride = (int64_t)(VT / 64) * KPW;
            uint4 raw[U];
            auto load = [&](int64_t j0) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int64_t j = j0 + u * stride + gk;
                    raw[u] = (j < N && has) ? RowVec<T>::raw(kh + j * d, gi * VEC) : make_uint4(0u, 0u, 0u, 0u);
                }
            };
            if constexpr (RB > 1) load((int64_t)w * KPW);
#pragma nounroll
            for (int64_t j0 = (int64_t)w * KPW; j0 < N; j0 += stride * U) {
                if constexpr (RB == 1) load(j0);  // both sets of 16 keys would spill
                double acc[16];  // [key][row]
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    float x[VEC];
                    RowVec<T>::unpack(raw[u], x);
#pragma unroll
                    for (int rr = 0; rr < RB; ++rr) acc[u * RB + rr] = 0.0;
#pragma unroll
                    for (int i = 0; i < VEC; ++i) {
                        const double xd = (double)x[i];
#pragma unroll
                        for (int rr = 0; rr < RB; ++rr) acc[u * RB + rr] = fma(xr[rr][i], xd, acc[u * RB + rr]);
                    }
                }
                if constexpr (RB > 1) load(j0 + stride * U);  // in flight during the reductions
                if (GL == 16) {
                    // transposed: at each exchange a lane gives away half of its
                    // sums, and lane i ends with sum i of its group
#pragma unroll
                    for (int half = 8; half > 0; half >>= 1) {
                        const bool upper = (gi & half) != 0;
#pragma unroll
                        for (int i = 0; i < half; ++i) {
                            const double give = upper ? acc[i] : acc[i + half];
                            const double keep = upper ? acc[i + half] : acc[i];
                            acc[i] = keep + __shfl_xor(give, half);
                        }
                    }
                    const int64_t j = j0 + (gi / RB) * stride + gk;
                    if (j < N) put(j, gi % RB, acc[0]);
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[i] = group_sum(acc[i], GL);
                    if (gi == 0) {
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int64_t j = j0 + u * stride + gk;
                            if (j < N) {
#pragma unroll
                                for (int rr = 0; rr < RB; ++rr) put(j, rr, acc[u * RB + rr]);
                            }
                        }
                    }
                }
            }
        } else {
            for (int64_t j = w; j < N; j += VT / 64) {
                double acc[RB];
#pragma unroll
                for (int rr = 0; rr < RB; ++rr) acc[rr] = 0.0;
                for (int c = lane; c < d; c += 64) {
                    const double xd = (double)Elem<T>::load(kh, j * d + c);
#pragma unroll
                    for (int rr = 0; rr < RB; ++rr) acc[rr] = fma(xq[rr * d + c], xd, acc[rr]);
                }
#pragma unroll
                for (int rr = 0; rr < RB; ++rr) {
                    acc[rr] = group_sum(acc[rr], 64);
                    if (lane == 0) put(j, rr, acc[rr]);
                }
            }
        }
        __syncthreads();
        // ---- each row on its team: softmax and its own top-mass set ----------------
        double zmax = -INFINITY;
        for (int64_t j = t; j < N; j += NT) zmax = fmax(zmax, zt[j]);
        zmax = team_reduce(zmax, redd, NW, OpMax());
        team_top([&](int64_t j) { return zt[j]; }, N, s, own, t, NT, smem + L.red);
        double lsum = 0.0;
        for (int64_t j = t; j < N; j += NT) {
            const double e = exp(zt[j] - zmax);
            zt[j] = e;
            lsum += e;
        }
        lsum = team_reduce(lsum, redd, NW, OpSum());
        for (int64_t j = t; j < N; j += NT) zt[j] = zt[j] / lsum;
        if (t == 0 && mine) {
            rowsc[2 * (m0 + team)] = zmax;
            rowsc[2 * (m0 + team) + 1] = lsum;
        }
        for (int e = tid; e < RB * d; e += VT)
            if (m0 + e / d < gs) mus[(size_t)m0 * d + e] = 0.0;
        __syncthreads();
        if (!resident)
            for (int64_t j = tid; j < N; j += VT) {
                double sc = score[j];
                for (int rr = 0; rr < RB && m0 + rr < gs; ++rr) sc += zz[rr * N + j];
                score[j] = sc;
            }
        // ---- dense outputs: each lane its columns over the keys it visits ----------
        {
            double part[RB][VEC > 4 ? VEC : 4];
#pragma unroll
            for (int rr = 0; rr < RB; ++rr) {
#pragma unroll
                for (int i = 0; i < (VEC > 4 ? VEC : 4); ++i) part[rr][i] = 0.0;
            }
            if (vec) {
                constexpr int U = 8;
                const int64_t stride = (int64_t)(VT / 64) * KPW;
#pragma nounroll
                for (int64_t j0 = (int64_t)w * KPW; j0 < N; j0 += stride * U) {
                    uint4 raw[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int64_t j = j0 + u * stride + gk;
                        raw[u] = (j < N && has) ? RowVec<T>::raw(vh + j * d, gi * VEC) : make_uint4(0u, 0u, 0u, 0u);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int64_t j = j0 + u * stride + gk;
                        if (j >= N) continue;
                        float x[VEC];
                        RowVec<T>::unpack(raw[u], x);
                        double pr[RB];
#pragma unroll
                        for (int rr = 0; rr < RB; ++rr) pr[rr] = zz[rr * N + j];
#pragma unroll
                        for (int i = 0; i < VEC; ++i) {
                            const double xd = (double)x[i];
#pragma unroll
                            for (int rr = 0; rr < RB; ++rr) part[rr][i] = fma(pr[rr], xd, part[rr][i]);
                        }
                    }
                }
                // the wave's groups by a butterfly, the waves in order below
#pragma nounroll
                for (int off = GL; off < 64; off <<= 1) {
#pragma unroll
                    for (int rr = 0; rr < RB; ++rr) {
#pragma unroll
                        for (int i = 0; i < VEC; ++i) part[rr][i] += __shfl_xor(part[rr][i], off);
                    }
                }
            } else {
                for (int64_t j = w; j < N; j += VT / 64) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int c = lane + 64 * i;
                        const double xd = c < d ? (double)Elem<T>::load(vh, j * d + c) : 0.0;
#pragma unroll
                        for (int rr = 0; rr < RB; ++rr) part[rr][i] = fma(zz[rr * N + j], xd, part[rr][i]);
                    }
                }
            }
#pragma nounroll
            for (int x = 0; x < VT / 64; ++x) {
                if (w == x && (vec ? has && gk == 0 : true)) {
#pragma unroll
                    for (int rr = 0; rr < RB; ++rr) {
                        if (m0 + rr >= gs) continue;
                        double *mu = mus + (size_t)(m0 + rr) * d;
#pragma unroll
                        for (int i = 0; i < (VEC > 4 ? VEC : 4); ++i) {
                            const int c = vec ? gi * VEC + i : lane + 64 * i;
                            if (c < d && (!vec || i < VEC)) mu[c] += part[rr][i];
                        }
                    }
                }
                __syncthreads();
            }
        }
        // ---- each row's own top-mass error ------------------------------------------
        for (int u = t; u < s; u += NT) pk[u] = zt[own[u]];
        __syncthreads();
        const double es = es_list<T>(vh, d, own, pk, s, mus + (size_t)(mine ? m0 + team : 0) * d, redd, t, NT);
        if (t == 0 && mine) a.es_top[h * a.G + (int64_t)(m0 + team) * T_ + pos] = (float)(s >= N ? 0.0 : es);
        __syncthreads();
    }

    // ---- the vote: s keys of largest summed mass, index asc on ties ---------------
    team_top(
        [&](int64_t j) {
            if (!resident) return score[j];
            double sc = 0.0;
#pragma unroll
            for (int rr = 0; rr < RB; ++rr)
                if (rr < gs) sc += zz[rr * N + j];
            return sc;
        },
        N, s, vote, tid, VT, smem + L.red);
    for (int u = tid; u < s; u += VT) a.vote_idx[(h * T_ + pos) * s + u] = vote[u];

    // ---- each member under the vote's set -------------------------------------------
    for (int m0 = 0; m0 < gs; m0 += RB) {
        const bool mine = m0 + team < gs;
        const int m = mine ? m0 + team : 0;
        const int64_t r = h * a.G + (int64_t)m * T_ + pos;
        if (resident) {
            for (int u = t; u < s; u += NT) pk[u] = zt[vote[u]];
        } else {
            // the weights again, from the vote keys' logits (summed in column order:
            // rounding-level differences from the row pass's grouped sums) with the
            // row's own maximum and normaliser
            const double zmax = rowsc[2 * m], lsum = rowsc[2 * m + 1];
            const T *qr = (const T *)a.q + r * d;
            for (int u = t; u < s; u += NT) {
                const int j = vote[u];
                double acc = 0.0;
#pragma unroll 8
                for (int c = 0; c < d; ++c)
                    acc = fma((double)Elem<T>::load(qr, c), (double)Elem<T>::load(kh, (int64_t)j * d + c), acc);
                const double z = scale * acc + (a.bias ? (double)a.bias[j] : 0.0);
                pk[u] = exp(z - zmax) / lsum;
            }
        }
        __syncthreads();
        const double es = es_list<T>(vh, d, vote, pk, s, mus + (size_t)m * d, redd, t, NT);
        if (t == 0 && mine) {
            double pv = 0.0;
            for (int u = 0; u < s; ++u) pv += pk[u];
            a.es_vote[r] = (float)(s >= N ? 0.0 : es);
            if (a.dropped) a.dropped[r] = (float)(s >= N ? 0.0 : 1.0 - pv);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
bool vote_supported(const fw_rows &rows, int s, int gs) {
    if (gs < 1 || rows.G % gs != 0 || s < 1 || s > rows.n || s > 256) return false;
    // one row at a time with the summed masses beside it
    const size_t score = gs > 1 ? 0 : (size_t)rows.n * 8;
    return vote_lds(rows.n, (int)rows.d, gs, s, 1).total + score <= 160 * 1024;
}

hipError_t launch_vote(const fw_rows &rows, int s, int gs, int32_t *vote_idx, float *es_vote, float *es_top,
                       float *dropped, hipStream_t st) {
    if (!vote_supported(rows, s, gs)) return hipErrorInvalidConfiguration;
    VoteArgs a{};
    a.q = rows.q;
    a.k = rows.k;
    a.v = rows.v;
    a.scale = rows.scale;
    a.bias = rows.bias;
    a.H = rows.H;
    a.G = rows.G;
    a.N = rows.n;
    a.d = (int)rows.d;
    a.s = s;
    a.gs = gs;
    a.vote_idx = vote_idx;
    a.es_vote = es_vote;
    a.es_top = es_top;
    a.dropped = dropped;
    const int rb = vote_rows(rows.n, (int)rows.d, gs, s);
    const size_t lds = vote_lds(rows.n, (int)rows.d, gs, s, rb).total;
    const dim3 g((unsigned)(rows.H * (rows.G / gs)));
    // One row at a time: four waves per group, two workgroups on a CU (one in its
    // serial picks, the other reading), where there are groups and LDS for two, and
    // for a few keys in whole chunks, whose picks eight waves' lists only lengthen;
    // else eight.  Groups of one, s = 8, bf16 rows of 128 columns, four waves
    // against eight: 1536 of 4096 keys 626 us against 835 (eight with a prefetch
    // that spilled); 256 of 4096 178 against 134, of 130 32 against 45; 4 of 130
    // keys of 100 columns 42 against 35.
    const bool chunks = rows.d % (rows.dtype == FW_BF16 ? 8 : 4) == 0;
    const bool four = (rows.n <= 256 && chunks) || (lds <= 80 * 1024 && g.x > 256);
#define FW_VOTE_K(T, RB, VT) hipLaunchKernelGGL((vote_group_kernel<T, RB, VT>), g, dim3(VT), lds, st, a)
#define FW_VOTE(T)                               \
    switch (rb) {                                \
        case 4: FW_VOTE_K(T, 4, 512); break;     \
        case 2: FW_VOTE_K(T, 2, 512); break;     \
        default:                                 \
            if (four) FW_VOTE_K(T, 1, 256);      \
            else FW_VOTE_K(T, 1, 512);           \
    }
    if (rows.dtype == FW_BF16) {
        FW_VOTE(uint16_t)
    } else {
        FW_VOTE(float)
    }
#undef FW_VOTE
#undef FW_VOTE_K
    return hipGetLastError();
}

}  // namespace fw
