// rtf_alias.hip -- the Alias Method (Sec. 2.6; Walker's table of cells that
// hold at most two intervals, Fig. alias_map), the non-monotone comparison
// mapping of the paper's quality study (Figs. results_sine64, 2d_zoom,
// convergence).  It is not on the inversion path; it exists so that the
// same uniforms can be pushed through both mappings on the GPU.
//
// Table (exact integers): item i of a distribution of n weights carries the
// mass w_i n, a cell holds W = sum w.  Record j = { thr_j, alias_j }: the part
// thr_j in [0, W] of cell j kept by item j, the rest going to alias_j.
// Construction: Vose's two-worklist method ("A linear algorithm for
// generating random numbers with a given distribution", IEEE TSE 1991) in a
// fixed order -- items of mass below W ("small") and at least W ("large") on
// two stacks in increasing index order; each step pops one of each, gives the
// small item's cell remainder to the large item, and pushes the large item
// back on the stack its remaining mass belongs to; large items left at the
// end keep their whole cell.  The setup is serial as it is written (the
// paper's remark in Sec. 2.6), but its pairing follows from two prefix sums.
// Take the small items in popping order (falling index) with deficits
// W - mass and their running sums D_i, and the large items in theirs with
// excesses mass - W and running sums X_j.  A large item whose rest falls
// below W is popped as the very next small item and hands its deficit on to
// the next large one, so after i small items the large item on top is the
// first with X_j >= D_i and what it holds beyond W is X_j - D_i.  Hence
//   small i:  alias = the first large j with X_j >= D_{i-1}, thr = its mass;
//   large j:  with i the first small with D_i > X_j, thr = W + X_j - D_i and
//             alias = large j + 1; without one (X_j is then the sum of all
//             deficits) thr = W and alias = itself.
// k_alias_build computes that with a block per distribution (the table of
// the serial form, bit for bit); batches of tiny distributions keep the
// serial form, one thread each (k_alias_serial).
//
// Sampling: xi = u 2^-64 lies in cell j = floor(u n / 2^64) at offset
// r = (u n) mod 2^64; the item is j when floor(r W / 2^64) < thr_j, else
// alias_j (exact: f < thr/W  <=>  r W < thr 2^64).
#include "rtf_internal.h"

namespace rtf {

namespace {

struct alignas(16) AliasRec {
    uint64_t thr;
    int32_t alias;
    int32_t pad;
};

// One thread per distribution: the total, the masses, the two stacks, the
// pairing.  recs, small and large cover the distribution's own range.
__global__ __launch_bounds__(64) void k_alias_serial(const uint32_t *__restrict__ w,
                                                    const int64_t *__restrict__ eoff, int32_t D,
                                                    AliasRec *__restrict__ recs,
                                                    int32_t *__restrict__ small_st,
                                                    int32_t *__restrict__ large_st,
                                                    uint64_t *__restrict__ Wd,
                                                    uint32_t *__restrict__ status) {
    const int32_t d = (int32_t)(blockIdx.x * 64 + threadIdx.x);
    if (d >= D) return;
    const int64_t e0 = eoff[d], e1 = eoff[d + 1];
    const int64_t n = e1 - e0;
    uint64_t W = 0;
    for (int64_t i = e0; i < e1; ++i) W += w[i];
    Wd[d] = W;
    if (W == 0) {
        atomicOr(status, status_bit(RTF_ERR_ZERO_TOTAL));
        return;
    }
    int32_t *sm = small_st + e0, *lg = large_st + e0;
    int64_t ns = 0, nl = 0;
    for (int64_t i = 0; i < n; ++i) {
        const uint64_t mass = (uint64_t)w[e0 + i] * (uint64_t)n;
        recs[e0 + i].thr = mass;
        recs[e0 + i].alias = (int32_t)i;
        recs[e0 + i].pad = 0;
        if (mass < W) sm[ns++] = (int32_t)i;
        else lg[nl++] = (int32_t)i;
    }
    while (ns > 0 && nl > 0) {
        const int32_t s = sm[--ns], l = lg[--nl];
        recs[e0 + s].alias = l;
        const uint64_t rest = recs[e0 + l].thr - (W - recs[e0 + s].thr);
        recs[e0 + l].thr = rest;
        if (rest < W) sm[ns++] = l;
        else lg[nl++] = l;
    }
    while (nl > 0) {  // mass exactly W: the cell is the item's own
        const int32_t l = lg[--nl];
        recs[e0 + l].thr = W;
        recs[e0 + l].alias = l;
    }
    if (ns > 0) atomicOr(status, status_bit(RTF_ERR_VALUE));  // cannot happen with exact sums
}

// The tables of distributions by whole blocks, one block each: k_alias_build
// those of at most ALDS items, whose lists stay in LDS with 64-bit running
// sums (below n W <= 2^56 there), k_alias_big larger ones, with lists and
// 128-bit sums in the workspace, in rounds of ABT items.  A block is a chain
// of scans and LDS searches, so it is sized for three blocks a CU: 41 KB, and
// 80 registers, to which it is held at the price of 44 spilled bytes a thread.
// A thread advances AQ searches together.  4097 tables of a 4096 x 4096 map
// (67 MB read, 268 MB written, 65 us at the copy rate): 4712 us by one thread
// a table, 180 us by blocks; at two blocks a CU, where nothing spills, 175 us
// with four searches together and 157 with eight, but 30,000 tables of 300
// items then take 531 us against 341; 1024 threads a block 474 us.
constexpr int ABT = 512;
constexpr int ALDS = 4096;
constexpr int AIT = ALDS / ABT;
typedef unsigned __int128 u128;

// A running (count of small items, sum of deficits, sum of excesses) and its
// exclusive scan over the block.
template <class Sum>
struct AliasAcc {
    int32_t small;
    Sum def, exc;
};

__device__ inline uint64_t shfl_up_sum(uint64_t v, int o) { return __shfl_up(v, o, 64); }
__device__ inline u128 shfl_up_sum(u128 v, int o) {
    return ((u128)__shfl_up((uint64_t)(v >> 64), o, 64) << 64) | __shfl_up((uint64_t)v, o, 64);
}

template <class Sum>
__device__ inline AliasAcc<Sum> alias_scan(AliasAcc<Sum> x, AliasAcc<Sum> *s_wave, AliasAcc<Sum> &total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const AliasAcc<Sum> own = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t c = __shfl_up(x.small, o, 64);
        const Sum d = shfl_up_sum(x.def, o), e = shfl_up_sum(x.exc, o);
        if (lane >= o) {
            x.small += c;
            x.def += d;
            x.exc += e;
        }
    }
    if (lane == 63) s_wave[w] = x;
    __syncthreads();
    AliasAcc<Sum> pre{0, 0, 0}, tot{0, 0, 0};
    for (int i = 0; i < ABT / 64; ++i) {
        const AliasAcc<Sum> t = s_wave[i];
        if (i < w) {
            pre.small += t.small;
            pre.def += t.def;
            pre.exc += t.exc;
        }
        tot.small += t.small;
        tot.def += t.def;
        tot.exc += t.exc;
    }
    __syncthreads();
    total = tot;
    pre.small += x.small - own.small;
    pre.def += x.def - own.def;
    pre.exc += x.exc - own.exc;
    return pre;
}

// One distribution's lists hold the ns small items' sums and indices from the
// front and the large ones' from the back (large j at n - 1 - j).
//
// first j in [0, nl) with sum(large j) >= v; the last large item's sum is the
// sum of all deficits, so there is one
template <class Sum>
__device__ inline int64_t first_large(const Sum *cum, int64_t n, int64_t nl, Sum v) {
    int64_t lo = 0, hi = nl - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (cum[n - 1 - mid] >= v) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// first i in [0, ns] with sum(small i) > v (ns if none)
template <class Sum>
__device__ inline int64_t first_small(const Sum *cum, int64_t ns, Sum v) {
    int64_t lo = 0, hi = ns;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (cum[mid] > v) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

__device__ inline void store_rec(AliasRec *recs, int64_t i, uint64_t thr, int32_t alias) {
    reinterpret_cast<uint4 *>(recs)[i] = make_uint4((uint32_t)thr, (uint32_t)(thr >> 32), (uint32_t)alias, 0u);
}

// Record of the item at place k of the lists (mass: the item's, used for the
// small ones).
template <class Sum>
__device__ inline void alias_record(const Sum *cum, const int32_t *item, int64_t n, int64_t ns, int64_t k,
                                    uint64_t W, const uint32_t *w, AliasRec *recs) {
    const int64_t nl = n - ns;
    const int64_t i = item[k];
    if (k < ns) {
        const int64_t j = first_large(cum, n, nl, k > 0 ? cum[k - 1] : (Sum)0);
        store_rec(recs, i, (uint64_t)w[i] * (uint64_t)n, item[n - 1 - j]);
    } else {
        const Sum X = cum[k];
        const int64_t q = first_small(cum, ns, X);
        if (q < ns) store_rec(recs, i, W - (uint64_t)(cum[q] - X), item[k - 1]);
        else store_rec(recs, i, W, (int32_t)i);
    }
}

// sum of x over the block, in every thread
__device__ inline uint64_t block_total(uint64_t x, uint64_t *s_sum) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = x;
    __syncthreads();
    x = 0;
    for (int i = 0; i < ABT / 64; ++i) x += s_sum[i];
    return x;
}

__global__ __launch_bounds__(ABT) __attribute__((amdgpu_waves_per_eu(6))) void k_alias_build(
    const uint32_t *__restrict__ w_all, const int64_t *__restrict__ eoff, AliasRec *recs_all,
    uint64_t *__restrict__ Wd, uint32_t *status) {
    __shared__ uint64_t s_cum[ALDS];
    __shared__ uint16_t s_item[ALDS];
    __shared__ AliasAcc<uint64_t> s_acc[ABT / 64];
    __shared__ uint64_t s_sum[ABT / 64];
    const int tid = threadIdx.x;
    const int32_t d = (int32_t)blockIdx.x;
    const int64_t e0 = eoff[d], n = eoff[d + 1] - e0;
    if (n > ALDS) return;  // k_alias_big's
    const uint32_t *w = w_all + e0;
    AliasRec *recs = recs_all + e0;
    // thread t holds the AIT places from t AIT on of the popping order (its
    // run, read once into registers)
    const int p0 = tid * AIT, ni = (int)n;
    uint32_t r[AIT] = {};
    uint64_t W = 0;
#pragma unroll
    for (int q = 0; q < AIT; ++q) {
        const int i = ni - 1 - (p0 + q);
        if (i >= 0) r[q] = w[i];
    }
#pragma unroll
    for (int q = 0; q < AIT; ++q) W += r[q];
    W = block_total(W, s_sum);
    if (tid == 0) {
        Wd[d] = W;
        if (W == 0) atomicOr(status, status_bit(RTF_ERR_ZERO_TOTAL));
    }
    if (W == 0) return;
    AliasAcc<uint64_t> acc{0, 0, 0}, total;
#pragma unroll
    for (int q = 0; q < AIT; ++q) {
        if (p0 + q >= ni) break;
        const uint64_t mass = (uint64_t)r[q] * (uint64_t)n;
        if (mass < W) {
            ++acc.small;
            acc.def += W - mass;
        } else {
            acc.exc += mass - W;
        }
    }
    AliasAcc<uint64_t> run = alias_scan(acc, s_acc, total);
#pragma unroll
    for (int q = 0; q < AIT; ++q) {
        if (p0 + q >= ni) break;
        const uint64_t mass = (uint64_t)r[q] * (uint64_t)n;
        int k;
        if (mass < W) {
            k = run.small++;
            run.def += W - mass;
            s_cum[k] = run.def;
        } else {
            k = ni - 1 - (p0 + q - run.small);  // large items before: places minus small ones
            run.exc += mass - W;
            s_cum[k] = run.exc;
        }
        s_item[k] = (uint16_t)(ni - 1 - (p0 + q));
    }
    __syncthreads();
    // Every item counts the sums of the other list below a bound of its
    // own: a small one the large items' X < D_{i-1}, a large one the small
    // items' D < X + 1.  AQ searches of a thread advance together, one
    // LDS read each per step.
    constexpr int AQ = 2;
    const int ns = total.small, nl = ni - ns;
    int top = 1;  // the largest power of two within the longer list
    while (2 * top <= max(ns, nl)) top *= 2;
    for (int k0 = tid; k0 < ni; k0 += AQ * ABT) {
        int pos[AQ], len[AQ], first[AQ], dir[AQ];
        uint64_t bound[AQ];
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int k = min(k0 + q * ABT, ni - 1);
            const bool small = k < ns;
            bound[q] = small ? (k > 0 ? s_cum[max(k - 1, 0)] : 0) : s_cum[k] + 1;
            len[q] = small ? nl : ns;
            first[q] = small ? ni - 1 : 0;
            dir[q] = small ? -1 : 1;
            pos[q] = 0;
        }
        for (int step = top; step >= 1; step >>= 1) {
#pragma unroll
            for (int q = 0; q < AQ; ++q) {
                const int t = pos[q] + step;
                const uint64_t v = s_cum[t <= len[q] ? first[q] + dir[q] * (t - 1) : 0];
                if (t <= len[q] && v < bound[q]) pos[q] = t;
            }
        }
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int k = k0 + q * ABT;
            if (k >= ni) break;
            const int i = s_item[k];
            if (k < ns)
                store_rec(recs, i, (uint64_t)w[i] * (uint64_t)n, s_item[ni - 1 - pos[q]]);
            else if (pos[q] < ns)
                store_rec(recs, i, W - (s_cum[pos[q]] - s_cum[k]), s_item[k - 1]);
            else
                store_rec(recs, i, W, i);
        }
    }
}

// The same for the distributions of more than ALDS items.
__global__ __launch_bounds__(ABT) void k_alias_big(const uint32_t *__restrict__ w_all,
                                                   const int64_t *__restrict__ eoff, AliasRec *recs_all,
                                                   int32_t *item_all, u128 *cum_all, uint64_t *__restrict__ Wd,
                                                   uint32_t *status) {
    __shared__ AliasAcc<u128> s_acc[ABT / 64];
    __shared__ uint64_t s_sum[ABT / 64];
    const int tid = threadIdx.x;
    const int32_t d = (int32_t)blockIdx.x;
    const int64_t e0 = eoff[d], n = eoff[d + 1] - e0;
    if (n <= ALDS) return;
    const uint32_t *w = w_all + e0;
    AliasRec *recs = recs_all + e0;
    uint64_t W = 0;
    for (int64_t i = tid; i < n; i += ABT) W += w[i];
    W = block_total(W, s_sum);
    if (tid == 0) {
        Wd[d] = W;
        if (W == 0) atomicOr(status, status_bit(RTF_ERR_ZERO_TOTAL));
    }
    if (W == 0) return;
    int32_t *item = item_all + e0;
    u128 *cum = cum_all + e0;
    AliasAcc<u128> base{0, 0, 0};
    for (int64_t p0 = 0; p0 < n; p0 += ABT) {
        const int64_t p = p0 + tid, i = n - 1 - p;
        AliasAcc<u128> acc{0, 0, 0}, total;
        bool small = false;
        if (p < n) {
            const uint64_t mass = (uint64_t)w[i] * (uint64_t)n;
            small = mass < W;
            if (small) {
                acc.small = 1;
                acc.def = W - mass;
            } else {
                acc.exc = mass - W;
            }
        }
        const AliasAcc<u128> pre = alias_scan(acc, s_acc, total);
        if (p < n) {
            const int64_t ks = (int64_t)base.small + pre.small;  // small items before this one
            const int64_t k = small ? ks : n - 1 - (p - ks);
            cum[k] = small ? base.def + pre.def + acc.def : base.exc + pre.exc + acc.exc;
            item[k] = (int32_t)i;
        }
        base.small += total.small;
        base.def += total.def;
        base.exc += total.exc;
    }
    __threadfence_block();
    __syncthreads();
    for (int64_t k = tid; k < n; k += ABT)
        alias_record<u128>(cum, item, n, base.small, k, W, w, recs);
}

__device__ inline int32_t alias_pick(const AliasRec *__restrict__ recs, int64_t e0, int64_t n,
                                     uint64_t W, uint64_t u) {
    const uint64_t j = mulhi64(u, (uint64_t)n);
    const uint64_t r = u * (uint64_t)n;
    const uint64_t t = mulhi64(r, W);
    const uint4 v = *reinterpret_cast<const uint4 *>(recs + e0 + (int64_t)j);
    const uint64_t thr = ((uint64_t)v.y << 32) | v.x;
    return t < thr ? (int32_t)j : (int32_t)v.z;
}

constexpr int AT = 256;

// Samples of one distribution each: sample s belongs to distribution d with
// sample_off[d] <= s < sample_off[d+1] (one distribution: sample_off null).
__global__ __launch_bounds__(AT) void k_alias_sample(const AliasRec *__restrict__ recs,
                                                     const int64_t *__restrict__ eoff,
                                                     const uint64_t *__restrict__ Wd, int32_t D,
                                                     const int64_t *__restrict__ soff,
                                                     const uint64_t *__restrict__ u, int64_t S,
                                                     int32_t *__restrict__ idx) {
    const int64_t s = (int64_t)blockIdx.x * AT + threadIdx.x;
    if (s >= S) return;
    int32_t d = 0;
    if (soff) {
        int32_t lo = 0, hi = D;  // last d with soff[d] <= s
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (soff[mid] <= s) lo = mid;
            else hi = mid;
        }
        d = lo;
    }
    const int64_t e0 = eoff[d], n = eoff[d + 1] - e0;
    const uint64_t W = Wd[d];
    idx[s] = W == 0 ? -1 : alias_pick(recs, e0, n, W, u[s]);
}

// Pairs: distribution 0 is the marginal over the R = D - 1 rows, row r is
// distribution r + 1; u2[2s] picks the row, u2[2s+1] the column.
__global__ __launch_bounds__(AT) void k_alias_sample_2d(const AliasRec *__restrict__ recs,
                                                        const int64_t *__restrict__ eoff,
                                                        const uint64_t *__restrict__ Wd, int32_t D,
                                                        const uint64_t *__restrict__ u2, int64_t S,
                                                        int32_t *__restrict__ rc) {
    const int64_t s = (int64_t)blockIdx.x * AT + threadIdx.x;
    if (s >= S) return;
    const uint4 uv = *reinterpret_cast<const uint4 *>(u2 + 2 * s);
    const uint64_t ua = ((uint64_t)uv.y << 32) | uv.x, ub = ((uint64_t)uv.w << 32) | uv.z;
    const uint64_t Wm = Wd[0];
    int32_t r = -1, c = -1;
    if (Wm != 0) {
        r = alias_pick(recs, 0, eoff[1], Wm, ua);
        if ((uint32_t)r < (uint32_t)(D - 1)) {  // the marginal must have one item per row table 1..D-1
            const int64_t e0 = eoff[r + 1], n = eoff[r + 2] - e0;
            const uint64_t W = Wd[r + 1];
            c = W == 0 ? -1 : alias_pick(recs, e0, n, W, ub);
        } else {
            r = -1;
        }
    }
    *reinterpret_cast<int2 *>(rc + 2 * s) = make_int2(r, c);
}

inline size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

// Blocks or threads.  A block costs about 11 ns of the GPU's time whatever it
// holds, a thread about 2.5 ns an item once the GPU is full of them and 0.45
// us an item before: 100,000 tables of 48 items 1167 us by blocks and 621 by
// threads, 30,000 of 128 items 397 and 183; 1000 of 24 items 19 and 23, one
// of 4096 items 21 and 1819.
inline bool alias_by_blocks(int32_t D, int64_t n) { return n >= 192 * (int64_t)D || (D <= 1024 && n >= 32 * (int64_t)D); }

// Whether one of the D distributions can hold more than ALDS items, whatever
// the offsets: empty ones, which break their rule, leave all n to another.
inline bool alias_may_be_big(int32_t D, int64_t n) { return alias_by_blocks(D, n) && n > ALDS; }

struct AliasLayout {
    size_t status, recs, W, eoff, small_st, large_st, cum, total;
};

AliasLayout alias_layout(int32_t D, int64_t n) {
    AliasLayout L;
    size_t o = 0;
    L.status = o;
    o = a256(o + 256);
    L.recs = o;
    o = a256(o + sizeof(AliasRec) * (size_t)n);
    L.W = o;
    o = a256(o + sizeof(uint64_t) * (size_t)D);
    L.eoff = o;
    o = a256(o + sizeof(int64_t) * (size_t)(D + 1));
    L.small_st = o;
    o = a256(o + sizeof(int32_t) * (size_t)n);
    // the second stack of the serial form, or the sums outside LDS
    L.large_st = L.cum = o;
    o = a256(o + (alias_may_be_big(D, n) ? sizeof(u128) : sizeof(int32_t)) * (size_t)n);
    L.total = o;
    return L;
}

__global__ __launch_bounds__(AT) void k_alias_offsets(const int64_t *src, int32_t D, int64_t n, int64_t *dst,
                                                      uint32_t *status) {
    const int64_t q = (int64_t)blockIdx.x * AT + threadIdx.x;
    if (q <= D) dst[q] = src ? src[q] : (q ? n : 0);
    if (q == 0) *status = 0u;
}


constexpr int64_t MAX_ALIAS_N = 2147483647;

bool alias_ok(const rtf_alias_table *t) {
    return t && t->recs && t->W && t->elem_off && t->status && t->D >= 1 && t->n_total >= t->D;
}

}  // namespace

}  // namespace rtf

using namespace rtf;

extern "C" {

size_t rtf_alias_workspace_bytes(int32_t D, int64_t n_total) {
    if (D < 1 || n_total < D || n_total > MAX_ALIAS_N) return 0;
    return alias_layout(D, n_total).total;
}

rtf_status rtf_alias_build(const uint32_t *w, const int64_t *elem_off, int32_t D, int64_t n_total,
                           void *ws, size_t ws_bytes, hipStream_t stream, rtf_alias_table *out) {
    if (!w || !ws || !out || (D > 1 && !elem_off)) return RTF_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(ws) & 255) || (reinterpret_cast<uintptr_t>(w) & 3))
        return RTF_ERR_INVALID_ARG;
    if (D < 1 || n_total < D) return RTF_ERR_INVALID_ARG;
    if (n_total > MAX_ALIAS_N) return RTF_ERR_SIZE;
    const AliasLayout L = alias_layout(D, n_total);
    if (ws_bytes < L.total) return RTF_ERR_WORKSPACE;
    char *b = static_cast<char *>(ws);
    rtf_alias_table t;
    t.D = D;
    t.n_total = n_total;
    t.recs = b + L.recs;
    t.W = reinterpret_cast<uint64_t *>(b + L.W);
    t.elem_off = reinterpret_cast<int64_t *>(b + L.eoff);
    t.status = reinterpret_cast<uint32_t *>(b + L.status);
    int32_t *small_st = reinterpret_cast<int32_t *>(b + L.small_st);
    hipLaunchKernelGGL(k_alias_offsets, dim3((unsigned)(D / AT + 1)), dim3(AT), 0, stream,
                       D > 1 ? elem_off : nullptr, D, n_total, t.elem_off, t.status);
    if (alias_by_blocks(D, n_total)) {
        hipLaunchKernelGGL(k_alias_build, dim3((unsigned)D), dim3(ABT), 0, stream, w, t.elem_off,
                           static_cast<AliasRec *>(t.recs), t.W, t.status);
        if (alias_may_be_big(D, n_total))
            hipLaunchKernelGGL(k_alias_big, dim3((unsigned)D), dim3(ABT), 0, stream, w, t.elem_off,
                               static_cast<AliasRec *>(t.recs), small_st, reinterpret_cast<u128 *>(b + L.cum),
                               t.W, t.status);
    } else
        hipLaunchKernelGGL(k_alias_serial, dim3((unsigned)((D + 63) / 64)), dim3(64), 0, stream, w,
                           t.elem_off, D, static_cast<AliasRec *>(t.recs), small_st,
                           reinterpret_cast<int32_t *>(b + L.large_st), t.W, t.status);
    if (hipGetLastError() != hipSuccess) return RTF_ERR_HIP;
    *out = t;
    return RTF_OK;
}

rtf_status rtf_alias_sample(const rtf_alias_table *t, const int64_t *sample_off, const uint64_t *u,
                            int64_t S, int32_t *out_idx, hipStream_t stream) {
    if (!alias_ok(t) || S < 0 || (t->D > 1 && !sample_off)) return RTF_ERR_INVALID_ARG;
    if (S == 0) return RTF_OK;
    if (!u || !out_idx || (reinterpret_cast<uintptr_t>(u) & 7) || (reinterpret_cast<uintptr_t>(out_idx) & 3))
        return RTF_ERR_INVALID_ARG;
    hipLaunchKernelGGL(k_alias_sample, dim3((unsigned)((S + AT - 1) / AT)), dim3(AT), 0, stream,
                       static_cast<const AliasRec *>(t->recs), t->elem_off, t->W, t->D,
                       t->D > 1 ? sample_off : nullptr, u, S, out_idx);
    return hipGetLastError() == hipSuccess ? RTF_OK : RTF_ERR_HIP;
}

rtf_status rtf_alias_sample_2d(const rtf_alias_table *t, const uint64_t *u2, int64_t S,
                               int32_t *out_rc, hipStream_t stream) {
    if (!alias_ok(t) || t->D < 2 || S < 0) return RTF_ERR_INVALID_ARG;
    if (S == 0) return RTF_OK;
    if (!u2 || !out_rc || (reinterpret_cast<uintptr_t>(u2) & 15) ||
        (reinterpret_cast<uintptr_t>(out_rc) & 7))
        return RTF_ERR_INVALID_ARG;
    hipLaunchKernelGGL(k_alias_sample_2d, dim3((unsigned)((S + AT - 1) / AT)), dim3(AT), 0, stream,
                       static_cast<const AliasRec *>(t->recs), t->elem_off, t->W, t->D, u2, S,
                       out_rc);
    return hipGetLastError() == hipSuccess ? RTF_OK : RTF_ERR_HIP;
}

rtf_status rtf_alias_export(const rtf_alias_table *t, uint64_t *h_thr, int32_t *h_alias,
                            uint64_t *h_W, hipStream_t stream) {
    if (!alias_ok(t)) return RTF_ERR_INVALID_ARG;
    if (hipStreamSynchronize(stream) != hipSuccess) return RTF_ERR_HIP;
    uint32_t st = 0;
    if (hipMemcpy(&st, t->status, sizeof st, hipMemcpyDeviceToHost) != hipSuccess) return RTF_ERR_HIP;
    if (h_thr || h_alias) {
        AliasRec *tmp = static_cast<AliasRec *>(malloc(sizeof(AliasRec) * (size_t)t->n_total));
        if (!tmp) return RTF_ERR_INVALID_ARG;
        const hipError_t e = hipMemcpy(tmp, t->recs, sizeof(AliasRec) * (size_t)t->n_total,
                                       hipMemcpyDeviceToHost);
        if (e == hipSuccess)
            for (int64_t i = 0; i < t->n_total; ++i) {
                if (h_thr) h_thr[i] = tmp[i].thr;
                if (h_alias) h_alias[i] = tmp[i].alias;
            }
        free(tmp);
        if (e != hipSuccess) return RTF_ERR_HIP;
    }
    if (h_W && hipMemcpy(h_W, t->W, sizeof(uint64_t) * (size_t)t->D, hipMemcpyDeviceToHost) !=
                   hipSuccess)
        return RTF_ERR_HIP;
    for (int c = 1; c < 32; ++c)
        if (st & (1u << c)) return static_cast<rtf_status>(c);
    return RTF_OK;
}

}  // extern "C"
