// rtf_sample.hip -- Alg. 2 (guide-table lookup plus tree descent), the
// continuous position of Sec. 5, the 2D component-by-component inversion of
// Sec. 5, and two baselines with the identical mapping (Sec. 4): binary search
// over all keys (Sec. 2.2) and the Cutpoint Method with bisection (Sec. 2.5).
#include "rtf_internal.h"

namespace rtf {

namespace {

// Index d with off[d] <= i < off[d+1] over off[0..D], found by a whole block
// of NT threads (uniform i): each round probes NT evenly spaced offsets, so
// 10^4 distributions take two dependent loads.  Every thread must call it.
template <int NT = 256>
__device__ inline int32_t block_find_segment(const int64_t *off, int32_t D, int64_t i) {
    int32_t lo = 0, hi = D;  // off[lo] <= i < off[hi]
    while (hi - lo > 1) {
        const int32_t step = (hi - lo + NT - 1) / NT;
        const int32_t p = lo + ((int32_t)threadIdx.x + 1) * step;
        const int below = (p < hi && off[p] <= i) ? 1 : 0;
        const int32_t nlo = lo + __syncthreads_count(below) * step;
        hi = nlo + step < hi ? nlo + step : hi;
        lo = nlo;
    }
    return lo;
}

constexpr int SB_T = 1024;      // threads of the kernels that stage records
constexpr int LCELLS = 1024;    // staged records, 64 KB: two blocks per CU
constexpr int STAGE_MIN = 2;    // samples per cell that make staging pay

// A staged segment's average length from which staging pays.  Measured over
// 1 to 4096 distributions of 64 to 1024 cells: at 4096 samples a distribution
// the staged kernel takes 0.6 to 1.05 times the chunk kernel's time, at 2048
// 0.8 to 1.4, at 512 2.4 to 2.7 (333 uneven tables of 16 to 2048 weights, 186K
// samples: 85 us staged, 11 us in chunks), since a block then spends its time
// finding and staging one short segment after another.  Large calls of equal
// distributions would gain from 2048 on, uneven ones lose, and their totals do
// not tell them apart (with x and without: 3000 of 250 cells and 2796 samples
// 68 and 44 us staged, 86 and 70 in chunks; 1000 of 16 to 4096 weights, 176
// cells and 2097 samples on average, 52 and 35 against 32 and 25).
constexpr int64_t STAGE_SEGMENT = 4096;

// One distribution of a batched call is staged from so many samples on, with x
// and without: 1000 cells, 2^22 samples 33.6 and 22.5 us by the plain kernel's
// quads, 24.1 and 15.4 staged; 2^24 144 and 103, 78 and 44; 2^20 7.6 and 5.8,
// 9.9 and 6.2.
constexpr int64_t STAGE_ONE_X = 1 << 22, STAGE_ONE = 1 << 21;

// Bytes of guide table up to which single-distribution sampling fetches the
// records by whole quads of lanes.  While the table fits the L2s the texture
// path's 64 lines per wave load bound the kernel (2^26 samples with x from a
// 1 MiB table: 795 us with a record per lane, 679 by quads; index only 659 and
// 516); from about 16 MiB the lines from the fabric do, and the quads'
// transposition only costs (256 MiB table: 1430 us a record per lane, 1440 by
// quads; index only 1339 and 1351).
constexpr int64_t QUAD_TABLE = 12 << 20;

// The batched kernel's blocks take chunks of 2048 samples from 2^21 samples
// on, below that 512, so that small calls reach more CUs (137K samples of 333
// distributions 14.6 us in chunks of 2048, 7.4 of 512; 2^20 of 2000 21.6 and
// 18.8; but 5.1M of 10000 144 and 152: a chunk's search for its distributions
// is paid four times as often).
constexpr int64_t CHUNK_LONG = 1 << 21;
constexpr int CHUNK_DISTS = 256;  // distributions a chunk can stage in LDS

static_assert(sizeof(Dist) == 64, "a staged record is four 16-byte words");
__device__ inline Dist lds_dist(const uint4 *s_dist, int32_t k) {
    Dist P;
    uint4 *q = reinterpret_cast<uint4 *>(&P);
#pragma unroll
    for (int w = 0; w < 4; ++w) q[w] = s_dist[4 * k + w];
    return P;
}

// index k in [lo, hi) with off[k] <= i < off[k+1], given off[lo] <= i < off[hi]
// (off may hold equal neighbours; the last k with off[k] <= i is taken)
__device__ inline int32_t find_segment_in(const int64_t *off, int32_t lo, int32_t hi, int64_t i) {
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (off[mid] <= i) lo = mid;
        else hi = mid;
    }
    return lo;
}

__device__ inline Node load_node(const Node *nodes, int64_t j) {
    uint4 v = *reinterpret_cast<const uint4 *>(nodes + j);
    Node r;
    r.key = ((uint64_t)v.y << 32) | v.x;
    r.c0 = (int32_t)v.z;
    r.c1 = (int32_t)v.w;
    return r;
}

// A record as it was loaded, its 16-byte words in flight until cell_of().
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
struct Words {
    u64x2 v[CELL_WORDS];
};

__device__ inline Words load_words(const Cell *cells, int64_t g) {
    const u64x2 *p = reinterpret_cast<const u64x2 *>(cells + g);
    Words r;
#pragma unroll
    for (int w = 0; w < CELL_WORDS; ++w) r.v[w] = p[w];  // all in flight together
    return r;
}

// Record c of a staged table: word w of every record lies in a plane of its
// own, [CELL_WORDS][LCELLS], so that a wave's 16-byte reads of one word
// spread over all banks (in record order they would fall on a quarter).
__device__ inline Words lds_words(const u64x2 *s_cell, uint32_t c) {
    Words r;
#pragma unroll
    for (int w = 0; w < CELL_WORDS; ++w) r.v[w] = s_cell[w * LCELLS + c];
    return r;
}

// The record, once its words have arrived.  Every word is marked as used here,
// whole, so that its loads complete together (one wait) and are made once:
// the compiler otherwise splits the record load along the branches that use
// each word (up to three round trips to the same line, one after another) or
// loads a half of a word a second time.
__device__ inline Cell cell_of(Words &r) {
#pragma unroll
    for (int w = 0; w < CELL_WORDS; ++w) asm volatile("" : "+v"(r.v[w]));
    Cell c;
#pragma unroll
    for (int w = 0; w < CELL_WORDS; ++w) {
        c.k[2 * w] = r.v[w].x;
        if (w + 1 < CELL_WORDS) c.k[2 * w + 1] = r.v[w].y;
    }
    c.ref = (int32_t)(uint32_t)r.v[CELL_WORDS - 1].y;
    c.aux = (int32_t)(uint32_t)(r.v[CELL_WORDS - 1].y >> 32);
    return c;
}

// Keeps the compiler from moving a wave's LDS accesses across: within a wave
// they execute in order, so lanes may hand each other data without a barrier.
__device__ inline void wave_fence() {
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// Every lane's record cells[g], fetched by whole quads of lanes: in step q the
// four lanes of a quad load the four 16-byte words of lane q's record, so that
// a wave instruction touches 16 lines instead of 64, and the words go through
// the wave's part of LDS to the lane they belong to.  A record takes five
// 16-byte slots there, which spreads both the writes and the reads over all
// banks.  (A transposition by DPP moves takes 64 vector instructions a record:
// 2^26 samples with x from a 16 KiB table 586 us against 561, indices 405
// against 387.)  All lanes of the wave must call it together; the table is at
// most 4 GiB.
constexpr int QUAD_SLOTS = 64 * (CELL_WORDS + 1);  // 16-byte slots per wave
__device__ inline Words load_words_quad(const Cell *cells, uint32_t g, u64x2 *s_wave) {
    static_assert(CELL_WORDS == 4, "one word of a record per lane of a quad");
    const uint32_t lane = threadIdx.x & 63, w = lane & 3;
    const char *base = reinterpret_cast<const char *>(cells);
    const int off = (int)(g << 6);
    u64x2 v[CELL_WORDS];
    v[0] = *reinterpret_cast<const u64x2 *>(base + ((uint32_t)__builtin_amdgcn_mov_dpp(off, 0x00, 0xf, 0xf, true) + 16 * w));
    v[1] = *reinterpret_cast<const u64x2 *>(base + ((uint32_t)__builtin_amdgcn_mov_dpp(off, 0x55, 0xf, 0xf, true) + 16 * w));
    v[2] = *reinterpret_cast<const u64x2 *>(base + ((uint32_t)__builtin_amdgcn_mov_dpp(off, 0xaa, 0xf, 0xf, true) + 16 * w));
    v[3] = *reinterpret_cast<const u64x2 *>(base + ((uint32_t)__builtin_amdgcn_mov_dpp(off, 0xff, 0xf, 0xf, true) + 16 * w));
    u64x2 *to = s_wave + (lane & ~3u) * (CELL_WORDS + 1) + w;
#pragma unroll
    for (int q = 0; q < 4; ++q) to[q * (CELL_WORDS + 1)] = v[q];
    wave_fence();
    Words r;
    const u64x2 *from = s_wave + lane * (CELL_WORDS + 1);
#pragma unroll
    for (int q = 0; q < CELL_WORDS; ++q) r.v[q] = from[q];
    wave_fence();
    return r;
}

// Whether the wave's samples are (by its first and last lane) in order within
// a few cells, as those of sorted or stratified uniforms are: their records
// share lines as they are, and the quads' transposition would only cost (2^26
// ordered indices from a 1 MiB table: 281 us by quads, 267 a record
// per lane).
__device__ inline bool narrow_wave(uint32_t g) {
    const uint32_t a = __builtin_amdgcn_readlane(g, 0), b = __builtin_amdgcn_readlane(g, 63);
    return b - a < 32u;
}

// A sampled leaf with the keys of its interval's two ends (KEY_END for the
// distribution's end); leaf -1 flags a damaged workspace.
struct Hit {
    int32_t i;
    uint64_t lo, hi;
};

// floor(u m / 2^64) for distribution P's m cells, P the same for the whole
// wave: a shift when m is a power of two (the shift is in the distribution's
// flags), else the high word of the product
__device__ inline int64_t cell_in(const Dist &P, uint64_t u) {
    const uint32_t sh = P.flags >> DIST_SHIFT_BIT;
    return sh ? (int64_t)(u >> sh) : (int64_t)mulhi64(u, (uint64_t)P.m);
}

__device__ inline int64_t cell_index(const Dist &P, uint64_t u) {
    return P.co + (int64_t)mulhi64(u, (uint64_t)P.m);
}

__device__ inline Wide load_wide(const Wide *wide, int64_t j) {
    const uint4 *p = reinterpret_cast<const uint4 *>(wide + j);
    const uint4 a = p[0], b = p[1], c = p[2];  // 48 bytes of one line, in flight together
    Wide r;
    r.k = ((uint64_t)a.y << 32) | a.x;
    r.kc[0] = ((uint64_t)a.w << 32) | a.z;
    r.kc[1] = ((uint64_t)b.y << 32) | b.x;
    r.r[0] = (int32_t)b.z;
    r.r[1] = (int32_t)b.w;
    r.r[2] = (int32_t)c.x;
    r.r[3] = (int32_t)c.y;
    return r;
}

// The three selections of a search, each under an execution mask instead of
// with v_cndmask: a masked v_mov_b64 moves a whole key in one instruction
// where a select takes two, and three or more selects on vcc in a row, which
// is what the compiler makes of the plain code, issue at 23 cycles each here
// instead of 4 (a compare between them, or the mask in another register
// pair, restores the rate).

// j = the number of k[1..5] at or below u before the first that is not, lo =
// k[j], hi = k[j + 1].
__device__ inline void count_bounds(const uint64_t *k, uint64_t u, int32_t &j, uint64_t &lo, uint64_t &hi) {
    static_assert(CELL_BOUNDS == 5, "five compares");
    uint64_t e, m2, m3, m4, m5;
    j = 0;
    lo = k[0];
    hi = k[1];
    asm("v_cmp_le_u64 vcc, %[k1], %[u]\n\t"
        "v_cmp_le_u64 %[m2], %[k2], %[u]\n\t"
        "v_cmp_le_u64 %[m3], %[k3], %[u]\n\t"
        "v_cmp_le_u64 %[m4], %[k4], %[u]\n\t"
        "v_cmp_le_u64 %[m5], %[k5], %[u]\n\t"
        "s_and_saveexec_b64 %[e], vcc\n\t"
        "v_mov_b64 %[lo], %[k1]\n\t"
        "v_mov_b64 %[hi], %[k2]\n\t"
        "v_mov_b32 %[j], 1\n\t"
        "s_and_b64 exec, exec, %[m2]\n\t"
        "v_mov_b64 %[lo], %[k2]\n\t"
        "v_mov_b64 %[hi], %[k3]\n\t"
        "v_mov_b32 %[j], 2\n\t"
        "s_and_b64 exec, exec, %[m3]\n\t"
        "v_mov_b64 %[lo], %[k3]\n\t"
        "v_mov_b64 %[hi], %[k4]\n\t"
        "v_mov_b32 %[j], 3\n\t"
        "s_and_b64 exec, exec, %[m4]\n\t"
        "v_mov_b64 %[lo], %[k4]\n\t"
        "v_mov_b64 %[hi], %[k5]\n\t"
        "v_mov_b32 %[j], 4\n\t"
        "s_and_b64 exec, exec, %[m5]\n\t"
        "v_mov_b64 %[lo], %[k5]\n\t"
        "v_mov_b64 %[hi], %[k6]\n\t"
        "v_mov_b32 %[j], 5\n\t"
        "s_mov_b64 exec, %[e]"
        : [e] "=&s"(e), [m2] "=&s"(m2), [m3] "=&s"(m3), [m4] "=&s"(m4), [m5] "=&s"(m5), [j] "+&v"(j),
          [lo] "+&v"(lo), [hi] "+&v"(hi)
        : [u] "v"(u), [k1] "v"(k[1]), [k2] "v"(k[2]), [k3] "v"(k[3]), [k4] "v"(k[4]), [k5] "v"(k[5]),
          [k6] "v"(k[6])
        : "vcc", "scc");
}

// One binary step past a node: u >= key goes right.  klo and khi keep the
// last key at or below u and the last above it.
__device__ inline void step_node(uint64_t key, int32_t c0, int32_t c1, uint64_t u, int32_t &jn,
                                 uint64_t &klo, uint64_t &khi) {
    uint64_t e;
    jn = c0;
    asm("v_cmp_le_u64 vcc, %[k], %[u]\n\t"
        "s_and_saveexec_b64 %[e], vcc\n\t"
        "v_mov_b64 %[klo], %[k]\n\t"
        "v_mov_b32 %[jn], %[c1]\n\t"
        "s_andn2_b64 exec, %[e], vcc\n\t"
        "v_mov_b64 %[khi], %[k]\n\t"
        "s_mov_b64 exec, %[e]"
        : [e] "=&s"(e), [jn] "+&v"(jn), [klo] "+&v"(klo), [khi] "+&v"(khi)
        : [u] "v"(u), [k] "v"(key), [c1] "v"(c1)
        : "vcc", "scc");
}

// Two binary steps past a collapsed node.  A leaf child repeats its reference
// (r[2s] == r[2s+1]) and ends the second step.
__device__ inline void step_wide(const Wide &w, uint64_t u, int32_t &jn, uint64_t &klo, uint64_t &khi) {
    uint64_t e, kc = w.kc[0];
    int32_t g0 = w.r[0], g1 = w.r[1];
    asm("v_cmp_le_u64 vcc, %[k], %[u]\n\t"
        "s_and_saveexec_b64 %[e], vcc\n\t"
        "v_mov_b64 %[klo], %[k]\n\t"
        "v_mov_b64 %[kc], %[kc1]\n\t"
        "v_mov_b32 %[g0], %[r2]\n\t"
        "v_mov_b32 %[g1], %[r3]\n\t"
        "s_andn2_b64 exec, %[e], vcc\n\t"
        "v_mov_b64 %[khi], %[k]\n\t"
        "s_mov_b64 exec, %[e]"
        : [e] "=&s"(e), [klo] "+&v"(klo), [khi] "+&v"(khi), [kc] "+&v"(kc), [g0] "+&v"(g0), [g1] "+&v"(g1)
        : [u] "v"(u), [k] "v"(w.k), [kc1] "v"(w.kc[1]), [r2] "v"(w.r[2]), [r3] "v"(w.r[3])
        : "vcc", "scc");
    if (g0 == g1) jn = g0;
    else step_node(kc, g0, g1, u, jn, klo, khi);
}

// Alg. 2: g = floor(xi * m); follow the reference until it names a leaf.
// The cell record c resolves the guide step and, for a cell that holds at
// most CELL_BOUNDS lower bounds (or for u below the record's last key), the
// whole sample: the leaf is a - 1 plus the number of the cell's lower bounds
// at or below u.  Otherwise the descent continues from the cell's tree root.
// A reference outside the forest, or a path longer than the forest has nodes,
// can only come from a damaged workspace.
//
// The record's answer needs no look at how many bounds it holds: the key
// after the last bound is the upper end of the cell's last interval, which
// lies above u, so the count ends there and the unused slots (0) past it are
// never reached; a covered cell counts none.  The one key that u can equal
// without reaching it is KEY_END, at u = 2^64 - 1: there the count compares
// 2^64 - 2, which every real key below KEY_END is at most (W <= 2^63).
__device__ inline Hit resolve(const Node *nodes, const Wide *wide, const Cell &c, const Dist &P,
                              uint64_t u, int64_t n_total) {
    Hit h;
    int32_t j;
    count_bounds(c.k, u - (u == ~0ull ? 1 : 0), j, h.lo, h.hi);
    const int32_t sgn = c.ref >> 31;  // covered: leaf ~ref, else the leaf before a, plus j
    h.i = (c.ref ^ sgn) + ~sgn + j;
    if ((c.ref | c.aux) >= 0 && u >= c.k[CELL_KEYS - 1]) {  // past the record: the tree
        // Both bounds adjacent to the sampled leaf i are its ancestors when
        // they lie inside the cell, so the descent meets U_i as the last key
        // at or below u and U_{i+1} as the last key above it; only when i is
        // the cell's last leaf (no key above u met: they are not 0) is
        // U_{i+1} read after the descent.
        const int32_t nt = (int32_t)n_total;
        uint64_t klo = c.k[CELL_KEYS - 1], khi = 0;
        int32_t jn = c.aux;
        uint32_t steps = 0;
        if (wide) {
            // collapsed nodes: two binary levels per record (Sec. 5)
            while (descent_goes_on(jn, steps, nt)) {
                step_wide(load_wide(wide, jn), u, jn, klo, khi);
                ++steps;
            }
        } else {
            while (descent_goes_on(jn, steps, nt)) {
                const Node nd = load_node(nodes, jn);
                step_node(nd.key, nd.c0, nd.c1, u, jn, klo, khi);
                ++steps;
            }
        }
        h.i = jn < 0 ? ~jn : (int32_t)-1;
        h.lo = klo;
        h.hi = khi;
        if (khi == 0 && (uint32_t)(h.i - (int32_t)P.eo) < (uint32_t)P.n)
            h.hi = (uint32_t)(h.i - (int32_t)P.eo) + 1 < (uint32_t)P.n ? nodes[(int64_t)h.i + 1].key : KEY_END;
    }
    if ((uint32_t)(h.i - (int32_t)P.eo) >= (uint32_t)P.n) h.i = -1;
    return h;
}

__device__ inline Hit descend(const Node *nodes, const Wide *wide, const Cell *cells, const Dist &P,
                              uint64_t u, int64_t n_total) {
    Words r = load_words(cells, cell_index(P, u));
    return resolve(nodes, wide, cell_of(r), P, u, n_total);
}

// x = (i + ((t - C_i) + lo * 2^-64) / w_i) / n with t:lo = u * W, where
// C_i = floor(U_i * W / 2^64) recovers the exact partial sum from a key.
// For the sampled i, 0 <= t - C_i < w_i = C_{i+1} - C_i < 2^32 and
// i - eo < 2^31, so those convert to FP64 from 32 bits (one instruction
// each, and the same values).  The division by n is a product with 1/n,
// computed once where the distribution is the same for a whole loop; the
// result is kept at most 1 (it could round one ulp above 1 when the offset in
// the interval rounds up to w_i in the last leaf).
__device__ inline double position(const Dist &P, const Hit &h, uint64_t u) {
    const uint64_t W = P.W;
    const uint64_t Ci = mulhi64(h.lo, W);
    const uint64_t t = mulhi64(u, W);
    const uint64_t lo = u * W;
    const double w = interval_weight(h.lo, h.hi, Ci, W, P.s);
    const double lod = __builtin_fma((double)(uint32_t)(lo >> 32), 0x1p32, (double)(uint32_t)lo);
    const double frac = div_small(__builtin_fma(lod, 0x1p-64, (double)(uint32_t)(t - Ci)), w);
    const double x = ((double)(h.i - (int32_t)P.eo) + frac) * (1.0 / (double)P.n);
    return __builtin_fmin(x, 1.0);
}

// The same, for a leaf found without its keys (the baselines).
__device__ inline double position_of(const Node *nodes, const Dist &P, int64_t i, uint64_t u) {
    Hit h;
    h.i = (int32_t)i;
    h.lo = nodes[i].key;
    h.hi = (i + 1 < P.eo + P.n) ? nodes[i + 1].key : KEY_END;
    return position(P, h, u);
}

template <bool BATCHED, bool WANT_X, bool QUAD>
__global__ __launch_bounds__(256) void k_sample(const Node *__restrict__ nodes,
                                                const Wide *__restrict__ wide,
                                                const Cell *__restrict__ cells,
                                                const Dist *__restrict__ dists,
                                                const int64_t *__restrict__ sample_off,
                                                int32_t D, int64_t n_total,
                                                const uint64_t *__restrict__ u, int64_t S,
                                                int32_t *__restrict__ idx,
                                                double *__restrict__ x, int64_t chunk) {
    if (!BATCHED) {
        __shared__ u64x2 s_quad[QUAD ? 4 * QUAD_SLOTS : 1];
        u64x2 *s_wave = s_quad + (QUAD ? (threadIdx.x >> 6) * QUAD_SLOTS : 0);
        const Dist P = dists[0];
        const int64_t stride = (int64_t)gridDim.x * blockDim.x;
        auto sample = [&](uint64_t us) {
            const int64_t g = cell_in(P, us);
            Words r;
            if (QUAD && !narrow_wave((uint32_t)g)) r = load_words_quad(cells, (uint32_t)g, s_wave);
            else r = load_words(cells, g);
            return resolve(nodes, wide, cell_of(r), P, us, n_total);
        };
        auto put = [&](int64_t s, const Hit &h, uint64_t us) {
            __builtin_nontemporal_store(h.i < 0 ? (int32_t)-1 : h.i - (int32_t)P.eo, idx + s);
            if (WANT_X) {
                const double px = position(P, h, us);
                __builtin_nontemporal_store(h.i < 0 ? (double)__builtin_nan("") : px, x + s);
            }
        };
        int64_t s0 = (int64_t)blockIdx.x * blockDim.x;
        if (P.flags & DIST_ZERO) {
            Hit none;
            none.i = -1;
            none.lo = none.hi = 0;
            for (int64_t s = s0 + threadIdx.x; s < S; s += stride) put(s, none, 0);
            return;
        }
        // Whole steps of a block, the next step's uniform loaded a step ahead.
        // Neither its address nor the stores depend on the lane's place, so
        // that no wait for the uniform waits for the stores issued after it.
        const int64_t whole = S - 255;
        if (s0 < whole) {
            uint64_t next = __builtin_nontemporal_load(u + s0 + threadIdx.x);
            for (; s0 < whole; s0 += stride) {
                const uint64_t us = next;
                next = __builtin_nontemporal_load(u + (s0 + stride < whole ? s0 + stride : s0) + threadIdx.x);
                const Hit h = sample(us);
                put(s0 + threadIdx.x, h, us);
            }
        }
        if (s0 < S) {  // the last, part of a step: lanes past the end repeat the last sample
            const int64_t s = s0 + threadIdx.x;
            const uint64_t us = u[s < S ? s : S - 1];
            const Hit h = sample(us);
            if (s < S) put(s, h, us);
        }
        return;
    }
    __shared__ int64_t s_soff[256];
    __shared__ uint4 s_dist[4 * CHUNK_DISTS];
    // batched: a block takes chunks of consecutive samples (numbered
    // per XCD, so that one XCD's L2 serves a few neighbouring distributions),
    // finds the chunk's first distribution once (block-wide), and each lane
    // steps on through the few distributions the chunk spans, two samples
    // 256 apart at a time with both samples' loads issued together.  A chunk
    // inside one distribution keeps its parameters in scalar registers.
    auto store = [&](int64_t s, const Dist &P, const Hit &h, uint64_t us) {
        if (h.i < 0) {
            idx[s] = -1;
            if (WANT_X) x[s] = __builtin_nan("");
            return;
        }
        __builtin_nontemporal_store(h.i - (int32_t)P.eo, idx + s);
        if (WANT_X) __builtin_nontemporal_store(position(P, h, us), x + s);
    };
    // two samples whose parameters are Pa and Pb, taken by value: through a
    // reference the fields would be fetched again after the stores
    auto two = [&](int64_t sa, int64_t sb, bool has_b, const Dist Pa, const Dist Pb) {
        const uint64_t ua = __builtin_nontemporal_load(u + sa);
        const uint64_t ub = __builtin_nontemporal_load(u + (has_b ? sb : sa));  // no branch
        const bool za = Pa.flags & DIST_ZERO, zb = Pb.flags & DIST_ZERO;
        Words ra = load_words(cells, za ? 0 : cell_index(Pa, ua));
        Words rb = load_words(cells, zb ? 0 : cell_index(Pb, ub));
        const Cell ca = cell_of(ra), cb = cell_of(rb);
        Hit ha, hb;
        ha.i = hb.i = -1;
        if (!za) ha = resolve(nodes, wide, ca, Pa, ua, n_total);
        if (!zb) hb = resolve(nodes, wide, cb, Pb, ub, n_total);
        store(sa, Pa, ha, ua);
        if (has_b) store(sb, Pb, hb, ub);
    };
    for (int64_t c0 = xcd_block() * chunk; c0 < S; c0 += (int64_t)gridDim.x * chunk) {
        int32_t d = __builtin_amdgcn_readfirstlane(block_find_segment(sample_off, D, c0));
        int64_t dend = sample_off[d + 1];
        const int64_t cend = c0 + chunk < S ? c0 + chunk : S;
        const int steps = (int)(chunk / 256);
        if (dend >= cend) {
            // the chunk lies in one distribution: its parameters are uniform
            const Dist P = dists[d];
#pragma unroll 1
            for (int k = 0; k < steps; k += 2) {
                const int64_t sa = c0 + threadIdx.x + 256 * k, sb = sa + 256;
                if (sa >= cend) break;
                two(sa, sb, sb < cend, P, P);
            }
            continue;
        }
        // Several distributions: thread k reads offset d + k, and those below
        // the chunk's end count the distributions starting inside it.  With
        // fewer than CHUNK_DISTS of them their offsets and parameters are
        // staged in LDS, and each sample finds its own by a search there;
        // otherwise each lane walks the offsets in global memory.
        const int64_t ok = sample_off[d + (int32_t)threadIdx.x <= D ? d + (int32_t)threadIdx.x : D];
        s_soff[threadIdx.x] = ok;
        const int nb = __syncthreads_count(threadIdx.x > 0 && d + (int32_t)threadIdx.x < D && ok < cend);
        if (nb < CHUNK_DISTS - 1) {  // offsets d .. d + nb + 1 held, the last at or past cend
            const uint4 *src = reinterpret_cast<const uint4 *>(dists + d);
            for (int q = threadIdx.x; q < 4 * (nb + 1); q += 256) s_dist[q] = src[q];
            __syncthreads();
#pragma unroll 1
            for (int k = 0; k < steps; k += 2) {
                const int64_t sa = c0 + threadIdx.x + 256 * k, sb = sa + 256;
                if (sa >= cend) break;
                const bool has_b = sb < cend;
                const int32_t ka = find_segment_in(s_soff, 0, nb + 1, sa);
                const int32_t kb = has_b ? find_segment_in(s_soff, ka, nb + 1, sb) : ka;
                two(sa, sb, has_b, lds_dist(s_dist, ka), lds_dist(s_dist, kb));
            }
            __syncthreads();  // before the next chunk restages
            continue;
        }
#pragma unroll 1
        for (int k = 0; k < steps; k += 2) {
            const int64_t sa = c0 + threadIdx.x + 256 * k, sb = sa + 256;
            if (sa >= cend) break;
            // (d stays below D even for offsets that break the rules)
            while (sa >= dend && d + 1 < D) dend = sample_off[++d + 1];
            const int32_t da = d;
            const bool has_b = sb < cend;
            if (has_b)
                while (sb >= dend && d + 1 < D) dend = sample_off[++d + 1];
            two(sa, sb, has_b, dists[da], dists[d]);
        }
        __syncthreads();  // s_soff is rewritten by the next chunk
    }
}

// Batched sampling with the guide cells staged in LDS, for batches with
// several samples per cell and distributions of at most LCELLS cells: a block
// of SB_T threads takes a contiguous share of the samples, walks it one
// distribution segment at a time, and copies a segment's cells into LDS when
// the segment has at least STAGE_MIN samples per cell, so that a sample reads
// its cell record from LDS and only the rare descents reach L2.  Copying a
// record streams 64 bytes, at most 32 per sample of the segment; a random L2
// read per sample costs more.
template <bool WANT_X>
__global__ __launch_bounds__(SB_T) __attribute__((amdgpu_waves_per_eu(8))) void k_sample_staged(
    const Node *__restrict__ nodes, const Wide *__restrict__ wide, const Cell *__restrict__ cells,
    const Dist *__restrict__ dists, const int64_t *__restrict__ sample_off, int32_t D, int64_t n_total,
    const uint64_t *__restrict__ u, int64_t S, int32_t *__restrict__ idx, double *__restrict__ x) {
    __shared__ u64x2 s_cell[LCELLS * CELL_WORDS];
    const int64_t per = (S + gridDim.x - 1) / gridDim.x;
    const int64_t r0 = xcd_block() * per;
    const int64_t r1 = r0 + per < S ? r0 + per : S;
    auto store = [&](int64_t s, const Dist &P, const Hit &h, uint64_t us) {
        if (h.i < 0) {
            idx[s] = -1;
            if (WANT_X) x[s] = __builtin_nan("");
            return;
        }
        __builtin_nontemporal_store(h.i - (int32_t)P.eo, idx + s);
        if (WANT_X) __builtin_nontemporal_store(position(P, h, us), x + s);
    };
    for (int64_t s0 = r0; s0 < r1;) {  // uniform loop over the share's segments
        const int32_t d = __builtin_amdgcn_readfirstlane(block_find_segment<SB_T>(sample_off, D, s0));
        const int64_t de = sample_off[d + 1];
        // the segment ends past s0 (offsets that break the rules still make
        // progress, one sample at a time)
        const int64_t e = de > s0 ? (de < r1 ? de : r1) : s0 + 1;
        const Dist P = dists[d];
        const bool zero = P.flags & DIST_ZERO;
        const bool staged = !zero && P.m <= LCELLS && e - s0 >= STAGE_MIN * P.m;
        if (staged) {
            const u64x2 *src = reinterpret_cast<const u64x2 *>(cells + P.co);
            for (int64_t k = threadIdx.x; k < CELL_WORDS * P.m; k += SB_T)
                s_cell[(k % CELL_WORDS) * LCELLS + k / CELL_WORDS] = src[k];
            __syncthreads();
        }
        if (staged) {
            // cells from LDS: two samples per step, both uniforms loaded
            // together (the second index clamped: no branch)
            for (int64_t sa = s0 + threadIdx.x; sa < e; sa += 2 * SB_T) {
                const int64_t sb = sa + SB_T;
                const uint64_t ua = __builtin_nontemporal_load(u + sa);
                const uint64_t ub = __builtin_nontemporal_load(u + (sb < e ? sb : sa));
                Words ra = lds_words(s_cell, (uint32_t)cell_in(P, ua));
                Words rb = lds_words(s_cell, (uint32_t)cell_in(P, ub));
                const Cell ca = cell_of(ra), cb = cell_of(rb);
                const Hit ha = resolve(nodes, wide, ca, P, ua, n_total);
                const Hit hb = resolve(nodes, wide, cb, P, ub, n_total);
                store(sa, P, ha, ua);
                if (sb < e) store(sb, P, hb, ub);
            }
        } else {
            // cells from global memory (segments too short to stage, or
            // distributions with more than LCELLS cells)
            for (int64_t sa = s0 + threadIdx.x; sa < e; sa += SB_T) {
                const uint64_t us = __builtin_nontemporal_load(u + sa);
                Hit h;
                h.i = -1;
                if (!zero) h = descend(nodes, wide, cells, P, us, n_total);
                store(sa, P, h, us);
            }
        }
        if (staged) __syncthreads();  // before the next segment overwrites the cells
        s0 = e;
    }
}

// The 2D inversion of Sec. 5, component by component: the row from the
// marginal (distribution 0), then the column from that row's distribution.
// The marginal's guide cells are staged in LDS when it has at most LCELLS
// cells, so a pair resolves its row without a global record read.  A pair is
// read with one 16-byte load and written with one 8-byte and one 16-byte
// store, so every wave access covers whole consecutive lines.  Blocks of SB_T
// threads, two per CU, one pair per lane and step.
template <bool WANT_X>
__global__ __launch_bounds__(SB_T) __attribute__((amdgpu_waves_per_eu(8))) void k_sample_2d_staged(
    const Node *__restrict__ nodes, const Wide *__restrict__ wide, const Cell *__restrict__ cells,
    const Dist *__restrict__ dists, int32_t D, int64_t n_total, const uint64_t *__restrict__ u2, int64_t S,
    int32_t *__restrict__ rc,
    double *__restrict__ xy) {
    typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    __shared__ u64x2 s_cell[LCELLS * CELL_WORDS];
    const u64x2 *up = reinterpret_cast<const u64x2 *>(u2);
    i32x2 *rcp = reinterpret_cast<i32x2 *>(rc);
    f64x2 *xyp = reinterpret_cast<f64x2 *>(xy);
    const int64_t T = (int64_t)gridDim.x * blockDim.x;
    const Dist M = dists[0];
    const int64_t s_first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (M.flags & DIST_ZERO) {  // a marginal without mass: no row, and none of its records was written
        const i32x2 none = {-1, -1};
        const f64x2 nans = {__builtin_nan(""), __builtin_nan("")};
        for (int64_t s = s_first; s < S; s += T) {
            rcp[s] = none;
            if (WANT_X) xyp[s] = nans;
        }
        return;
    }
    const bool staged = M.m <= LCELLS;
    if (staged) {
        const u64x2 *src = reinterpret_cast<const u64x2 *>(cells + M.co);
        for (int64_t k = threadIdx.x; k < CELL_WORDS * M.m; k += SB_T)
            s_cell[(k % CELL_WORDS) * LCELLS + k / CELL_WORDS] = src[k];
        __syncthreads();
    }
    for (int64_t s = s_first; s < S; s += T) {
        const u64x2 uu = __builtin_nontemporal_load(up + s);
        Words wr = staged ? lds_words(s_cell, (uint32_t)cell_in(M, uu.x)) : load_words(cells, cell_index(M, uu.x));
        const Hit hr = resolve(nodes, wide, cell_of(wr), M, uu.x, n_total);
        // the marginal must have one weight per row distribution 1..D-1
        const int32_t r = hr.i - (int32_t)M.eo;
        const bool row = hr.i >= 0 && 1 + r < D;
        const Dist R = dists[row ? 1 + r : 0];
        i32x2 out = {row ? r : -1, -1};
        f64x2 pos = {__builtin_nan(""), __builtin_nan("")};
        // the column's record is on its way before the row's position is
        // worked out, and its wait comes after.  With positions the record's
        // ref and aux are loaded once more, by themselves, past the L2's
        // retention: 2^27 pairs of the 4096 x 4096 map 4633 -> 4388 us (4485
        // by an ordinary second load), where indices alone take 3772 us
        // without it and 4126 with an ordinary one.
        const int64_t gc = cell_index(R, uu.y);
        Words wc = load_words(cells, gc);
        uint64_t ra = 0;
        if (WANT_X) ra = __builtin_nontemporal_load(reinterpret_cast<const uint64_t *>(&cells[gc].ref));
        __builtin_amdgcn_sched_barrier(0);
        if (WANT_X) {
            const double y = position(M, hr, uu.x);
            pos.x = row ? y : pos.x;
        }
        __builtin_amdgcn_sched_barrier(0);
        Cell cc = cell_of(wc);
        if (WANT_X) {
            asm volatile("" : "+v"(ra));  // kept a load of its own
            cc.ref = (int32_t)(uint32_t)ra;
            cc.aux = (int32_t)(uint32_t)(ra >> 32);
        }
        // The build writes no record for a row without mass: what the
        // workspace held there must not start a descent, whose nodes (the
        // collapsed ones are not written either) need not end.
        if (R.flags & DIST_ZERO) cc.aux = -1;
        const Hit hc = resolve(nodes, wide, cc, R, uu.y, n_total);
        if (row && hc.i >= 0 && !(R.flags & DIST_ZERO)) {
            out.y = hc.i - (int32_t)R.eo;
            if (WANT_X) pos.y = position(R, hc, uu.y);
        }
        __builtin_nontemporal_store(out, rcp + s);
        if (WANT_X) __builtin_nontemporal_store(pos, xyp + s);
    }
}

// last leaf x in [lo, hi] of the distribution with key_x <= u; keys of leaves
// past the last positive weight are all-ones and never qualify
__device__ inline int64_t bisect(const Node *nodes, int64_t lo, int64_t hi, uint64_t u) {
    // invariant: key[lo] <= u (lo qualifies), hi + 1 does not
    int64_t a = lo, b = hi + 1;
    while (b - a > 1) {
        int64_t mid = a + (b - a) / 2;
        uint64_t k = nodes[mid].key;
        if (k != ~0ull && k <= u) a = mid;
        else b = mid;
    }
    return a;
}

template <bool CUTPOINT, bool WANT_X>
__global__ __launch_bounds__(256) void k_sample_bsearch(const Node *__restrict__ nodes,
                                                        const Cell *__restrict__ cells,
                                                        const Dist *__restrict__ dists,
                                                        const uint64_t *__restrict__ u,
                                                        int64_t S, int32_t *__restrict__ idx,
                                                        double *__restrict__ x) {
    const Dist &P = dists[0];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < S; s += stride) {
        const uint64_t us = u[s];
        if (P.flags & DIST_ZERO) {
            idx[s] = -1;
            if (WANT_X) x[s] = __builtin_nan("");
            continue;
        }
        const int64_t first = P.eo, last = P.eo + P.n - 1;
        int64_t lo = first, hi = last;
        if (CUTPOINT) {
            // the cell's first overlapping interval bounds the search from
            // below, the next cell's first overlapping interval from above
            const int64_t g = (int64_t)mulhi64(us, (uint64_t)P.m);
            const int32_t r0 = cells[P.co + g].ref;
            if (r0 < 0) {
                lo = hi = ~r0;
            } else {
                lo = (r0 > P.eo) ? r0 - 1 : r0;
                if (g + 1 < P.m) {
                    const int32_t r1 = cells[P.co + g + 1].ref;
                    hi = (r1 < 0) ? ~r1 : r1;
                }
            }
        }
        lo = lo < first ? first : (lo > last ? last : lo);
        hi = hi < lo ? lo : (hi > last ? last : hi);
        const int64_t i = (lo == hi) ? lo : bisect(nodes, lo, hi, us);
        idx[s] = (int32_t)(i - P.eo);
        if (WANT_X) x[s] = position_of(nodes, P, i, us);
    }
}

inline int grid_for(int64_t S) {
    int64_t b = (S + 255) / 256;
    const int64_t cap = 256 * 64;  // 256 CUs x 64 blocks in flight at most
    return (int)(b < cap ? b : cap);
}

}  // namespace

hipError_t launch_sample(const Node *nodes, const Wide *wide, const Cell *cells, const Dist *dists,
                         const int64_t *sample_off, int32_t D, int64_t n_total, int64_t m_total,
                         const uint64_t *u, int64_t S, int32_t *idx, double *x,
                         hipStream_t st) {
    // many samples per cell and per distribution, and small distributions:
    // stage the cells in LDS (two blocks of SB_T threads per CU)
    const bool enough = D == 1 ? S >= (x ? STAGE_ONE_X : STAGE_ONE) : S >= STAGE_SEGMENT * D;
    if (sample_off && enough && S >= (int64_t)STAGE_MIN * m_total && m_total <= (int64_t)LCELLS * D) {
        int64_t nb = (S + 4 * SB_T - 1) / (4 * SB_T);
        nb = nb < 512 ? nb : 512;
        if (x)
            hipLaunchKernelGGL((k_sample_staged<true>), dim3((unsigned)nb), dim3(SB_T), 0, st, nodes, wide, cells, dists,
                               sample_off, D, n_total, u, S, idx, x);
        else
            hipLaunchKernelGGL((k_sample_staged<false>), dim3((unsigned)nb), dim3(SB_T), 0, st, nodes, wide, cells,
                               dists, sample_off, D, n_total, u, S, idx, x);
        return hipGetLastError();
    }
    const bool batched = sample_off != nullptr && D > 1;  // one distribution's samples are all its own
    const int64_t chunk = S >= CHUNK_LONG ? 2048 : 512;
    const dim3 g(batched ? grid_for((S + chunk / 256 - 1) / (chunk / 256)) : grid_for(S)), b(256);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, g, b, 0, st, nodes, wide, cells, dists, sample_off, D, n_total, u, S, idx, x, chunk);
    };
    if (batched) {
        if (x) go(k_sample<true, true, false>);
        else go(k_sample<true, false, false>);
    } else if (m_total * (int64_t)sizeof(Cell) <= QUAD_TABLE) {
        if (x) go(k_sample<false, true, true>);
        else go(k_sample<false, false, true>);
    } else {
        if (x) go(k_sample<false, true, false>);
        else go(k_sample<false, false, false>);
    }
    return hipGetLastError();
}

hipError_t launch_sample_2d(const Node *nodes, const Wide *wide, const Cell *cells, const Dist *dists,
                            int32_t D, int64_t n_total, const uint64_t *u2, int64_t S,
                            int32_t *rc, double *xy, hipStream_t st) {
    // two blocks per CU, each copying the marginal's records once
    int64_t nb = (S + SB_T - 1) / SB_T;
    nb = nb < 512 ? nb : 512;
    const dim3 g((unsigned)nb), b(SB_T);
    if (xy)
        hipLaunchKernelGGL((k_sample_2d_staged<true>), g, b, 0, st, nodes, wide, cells, dists, D, n_total, u2,
                           S, rc, xy);
    else
        hipLaunchKernelGGL((k_sample_2d_staged<false>), g, b, 0, st, nodes, wide, cells, dists, D, n_total,
                           u2, S, rc, xy);
    return hipGetLastError();
}

hipError_t launch_sample_bsearch(const Node *nodes, const Cell *cells, const Dist *dists,
                                 bool cutpoint, const uint64_t *u, int64_t S, int32_t *idx,
                                 double *x, hipStream_t st) {
    const dim3 g(grid_for(S)), b(256);
    if (cutpoint && x)
        hipLaunchKernelGGL((k_sample_bsearch<true, true>), g, b, 0, st, nodes, cells, dists, u,
                           S, idx, x);
    else if (cutpoint)
        hipLaunchKernelGGL((k_sample_bsearch<true, false>), g, b, 0, st, nodes, cells, dists, u,
                           S, idx, x);
    else if (x)
        hipLaunchKernelGGL((k_sample_bsearch<false, true>), g, b, 0, st, nodes, cells, dists, u,
                           S, idx, x);
    else
        hipLaunchKernelGGL((k_sample_bsearch<false, false>), g, b, 0, st, nodes, cells, dists,
                           u, S, idx, x);
    return hipGetLastError();
}

}  // namespace rtf
