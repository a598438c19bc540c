// amg.hip -- smoothed-aggregation AMG setup on the GPU and the V-cycle.
//
// Per level: strength graph (squared Frobenius block norms f_ij, strong iff
// f_ij^2 >= theta^4 f_ii f_jj, symmetrised by OR) -> distance-2 maximal independent set by
// synchronous rounds over seeded priorities (equal to the sequential greedy set in descending
// priority order) -> aggregates -> tentative prolongator by Gram-Schmidt of the near-null space
// on each aggregate -> P = (I - omega D^-1 A) P_tent, omega = 4/(3 lambda_hat) -> R = P^T ->
// A_c = R (A P), all products on structural patterns -> dense inverse of the coarsest level.
// The paper (Sec. 5.2) preconditions with BoomerAMG; smoothed aggregation replaces it here.
//
// Built with -ffp-contract=off: the strength predicate and the Gram-Schmidt decisions are
// evaluated as written, without fused multiply-adds.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "solver.h"

namespace scr {

// ====================================================================== helpers
__device__ __forceinline__ int32_t find_col(const int32_t* __restrict__ ci, int32_t lo, int32_t hi, int32_t c) {
    int32_t e = hi;
    while (lo < hi) {
        int32_t mid = (lo + hi) >> 1;
        if (ci[mid] < c) lo = mid + 1; else hi = mid;
    }
    return (lo < e && ci[lo] == c) ? lo : -1;
}

// first index in [lo, hi) whose column is >= c (hi if none)
__device__ __forceinline__ int32_t lower_col(const int32_t* __restrict__ ci, int32_t lo, int32_t hi, int32_t c) {
    while (lo < hi) {
        int32_t mid = (lo + hi) >> 1;
        if (ci[mid] < c) lo = mid + 1; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ uint64_t sm64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ULL;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ULL;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBULL;
    return x ^ (x >> 31);
}
// priority of node i at a level: 30 bits of splitmix64(seed, level, i) above the index
__device__ __forceinline__ uint64_t mis_key(uint64_t seed, int level, int64_t i) {
    uint64_t h = sm64(seed ^ ((uint64_t)level << 56) ^ ((uint64_t)i * 0xD1B54A32D192ED03ULL));
    return ((h >> 34) << 32) | (uint64_t)(uint32_t)i;
}

DBsr bsr_alloc(int64_t nr, int64_t nc, int br, int bc, int64_t nnzb, Arena& ar) {
    DBsr M;
    M.nr = nr; M.nc = nc; M.br = br; M.bc = bc; M.nnzb = nnzb;
    M.rp = ar.make<int32_t>(nr + 1);
    M.ci = ar.make<int32_t>(nnzb > 0 ? nnzb : 1);
    M.v = ar.make<double>((nnzb > 0 ? nnzb : 1) * br * bc);
    return M;
}
void bsr_release(DBsr& M, Arena& ar) {
    ar.free(M.rp); ar.free(M.ci); ar.free(M.v);
    M = DBsr();
}

// ====================================================================== block split and S^
__global__ void split_k(int64_t nnzb, const double* __restrict__ K, double* __restrict__ A, double* __restrict__ G,
                        double* __restrict__ D, double* __restrict__ C) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nnzb) return;
    const double* k = K + q * 16;
    for (int i = 0; i < 3; ++i) {
        for (int j = 0; j < 3; ++j) A[q * 9 + 3 * i + j] = k[4 * i + j];
        G[q * 3 + i] = k[4 * i + 3];
        D[q * 3 + i] = k[12 + i];
    }
    C[q] = k[15];
}

void split_values(const DBsr& K, DBsr& A, DBsr& G, DBsr& D, DBsr& C, hipStream_t s) {
    if (K.nnzb > 0) split_k<<<cdiv(K.nnzb, 256), 256, 0, s>>>(K.nnzb, K.v, A.v, G.v, D.v, C.v);
    check_launch("split");
}

void split_blocks(const DBsr& K, DBsr& A, DBsr& G, DBsr& D, DBsr& C, Arena& ar, hipStream_t s) {
    auto mk = [&](DBsr& M, int br, int bc) {
        M.nr = K.nr; M.nc = K.nc; M.br = br; M.bc = bc; M.nnzb = K.nnzb;
        M.rp = K.rp; M.ci = K.ci;          // index arrays shared with K
        M.v = ar.make<double>(K.nnzb * br * bc);
    };
    mk(A, 3, 3); mk(G, 3, 1); mk(D, 1, 3); mk(C, 1, 1);
    if (K.nnzb > 0) split_k<<<cdiv(K.nnzb, 256), 256, 0, s>>>(K.nnzb, K.v, A.v, G.v, D.v, C.v);
    check_launch("split");
}

// ====================================================================== generic SpGEMM
// C = X Y row by row.  A row's columns lie in a window [first, last] of Y's columns (the smallest first and
// the largest last column of the Y rows that it meets), narrow on a mesh whose numbering is local, so LDS
// holds the row's columns as flags over its window: the distinct columns of a row are its set flags,
// their number a population count, in ascending order without a sort, and the place of a column in the
// row a prefix count plus a population count within one word.  Against LDS hash tables with a rank
// sort (pattern) and serial read-add-write steps per X entry (numeric), over all products of one set-up at
// 324k rows: pattern 11.4 -> 8.3 ms, scalar products 9.1 -> 5.1, block products 6.4 -> 7.0; one host
// synchronisation per product instead of three.  Bound by the latency of the gathers of Y's rows: each
// wavefront keeps four steps of loads in flight.
// Rows whose window is wider than a map take hash tables instead, whose cost follows the candidates and not the
// numbering (SPG_WIN, SPG_SEG).
constexpr int HMAX = 4096;         // unique columns allowed per row
constexpr int SPG_WIDE = 2048;     // mean candidates per row from which a row takes four wavefronts
constexpr int SPG_LONG = 24;       // mean length of the Y rows from which one X entry takes a wavefront

// Maximum over a 256-thread workgroup, folded into *out by one atomic (every thread must call it).
// A same-address atomic per row serialises at one L2 channel: 324k of them cost about 3.5 ms.
template <typename T>
__device__ __forceinline__ void block_max_to(T v, T* out) {
    __shared__ T red[256 / WAVE];
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        T w = __shfl_xor(v, o, WAVE);
        v = w > v ? w : v;
    }
    if ((threadIdx.x & (WAVE - 1)) == 0) red[threadIdx.x / WAVE] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        T m = red[0];
        for (int w = 1; w < 256 / WAVE; ++w) m = red[w] > m ? red[w] : m;
        atomicMax(out, m);
    }
}

// largest of n counts, and of the n window sizes win[2 i + 1] (one atomic of each kind per workgroup)
__global__ void __launch_bounds__(256) spg_max_k(int64_t n, const int32_t* __restrict__ cnt, const int32_t* __restrict__ win,
                                                 int* __restrict__ wmax, int* __restrict__ maxwin) {
    int m = 0, w = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        m = cnt[i] > m ? cnt[i] : m;
        w = win[2 * i + 1] > w ? win[2 * i + 1] : w;
    }
    block_max_to(m, wmax);
    __syncthreads();
    block_max_to(w, maxwin);
}

// The candidates (X entry, Y entry) of 64 consecutive X entries as one list in (X entry, Y entry) order,
// spread over the lanes of a wavefront: lane l holds X entry q0 + l, `incl` the number of candidates of the
// entries up to its own and `off` the Y index of its first candidate minus the candidates before it.
struct SpgList {
    int st, len, incl, off, total, nq;
    __device__ __forceinline__ SpgList(int32_t q0, int32_t x1, int lane, const int32_t* __restrict__ xci,
                                       const int32_t* __restrict__ yrp) {
        st = len = 0;
        nq = x1 - q0 < WAVE ? x1 - q0 : WAVE;
        if (lane < nq) {
            const int32_t k = xci[q0 + lane];
            st = yrp[k];
            len = yrp[k + 1] - st;
        }
        incl = len;
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            const int v = __shfl_up(incl, o, WAVE);
            if (lane >= o) incl += v;
        }
        total = __builtin_amdgcn_readlane(incl, WAVE - 1);
        off = st - (incl - len);
    }
    // long Y rows: one X entry per step, its Y row over the lanes
    __device__ __forceinline__ bool is_long() const { return total >= SPG_LONG * nq; }
    // one candidate per X entry at most: the lane's own
    __device__ __forceinline__ bool single() const { return !__any(len > 1); }
    // X entry (its lane) and Y index of candidate c, the last one for c beyond the list (every lane takes
    // part; the list is not empty)
    __device__ __forceinline__ void get(int c, int& l, int32_t& t) const {
        c = c < total ? c : total - 1;
        l = 0;     // number of lanes whose inclusive count is <= c
#pragma unroll
        for (int step = WAVE / 2; step > 0; step >>= 1) {
            const int v = __shfl(incl, l + step - 1, WAVE);
            if (v <= c) l += step;
        }
        t = __shfl(off, l, WAVE) + c;
    }
};
// walks the X entries of a list in steps of up to 64 candidates of one entry
struct SpgWalk {
    const SpgList& list;
    int j = -1, o = 0, n = 0, s = 0;
    __device__ __forceinline__ explicit SpgWalk(const SpgList& l) : list(l) { entry(); }
    __device__ __forceinline__ void entry() {
        do {
            ++j;
            n = j < list.nq ? __builtin_amdgcn_readlane(list.len, j) : 0;
        } while (j < list.nq && n == 0);
        if (j < list.nq) s = __builtin_amdgcn_readlane(list.st, j);
        o = 0;
    }
    __device__ __forceinline__ bool more() const { return j < list.nq; }
    // the step's X entry, the lane's Y index (the entry's last one beyond it) and whether the lane has one
    __device__ __forceinline__ void take(int lane, int& l, int32_t& t, bool& in) {
        l = j;
        in = o + lane < n;
        t = s + (in ? o + lane : n - 1);
        o += WAVE;
        if (o >= n) entry();
    }
};
constexpr int SPG_PASS = 4;        // steps of a wavefront over the list whose loads are in flight together
// calls f(first candidate, number of steps) for a list of `total` candidates, `per` of them a step, up to
// SPG_PASS steps at a time
template <typename F>
__device__ __forceinline__ void spg_steps(int total, int per, F f) {
    int base = 0;
    for (; total - base > 2 * per; base += SPG_PASS * per) f(base, std::integral_constant<int, SPG_PASS>{});
    if (total - base > per) f(base, std::integral_constant<int, 2>{});
    else if (total > base) f(base, std::integral_constant<int, 1>{});
}

// calls f(column) for every candidate of the list, some of them more than once (beyond the list the last
// candidate again, so that no load waits behind a branch)
template <typename F>
__device__ __forceinline__ void spg_columns(const SpgList& list, int lane, const int32_t* __restrict__ yci, F f) {
    if (list.is_long()) {
        SpgWalk walk(list);
        while (walk.more()) {
            int32_t t[SPG_PASS], c[SPG_PASS];
            int l;
            bool in;
#pragma unroll
            for (int u = 0; u < SPG_PASS; ++u) {
                t[u] = u ? t[0] : 0;
                if (walk.more()) walk.take(lane, l, t[u], in);
            }
#pragma unroll
            for (int u = 0; u < SPG_PASS; ++u) c[u] = yci[t[u]];
#pragma unroll
            for (int u = 0; u < SPG_PASS; ++u) f(c[u]);
        }
    } else if (list.single()) {
        if (list.len) f(yci[list.st]);
    } else {
        spg_steps(list.total, WAVE, [&](int base, auto steps) {
            constexpr int U = decltype(steps)::value;
            int32_t t[U], c[U];
            int l;
#pragma unroll
            for (int u = 0; u < U; ++u) list.get(base + u * WAVE + lane, l, t[u]);
#pragma unroll
            for (int u = 0; u < U; ++u) c[u] = yci[t[u]];
#pragma unroll
            for (int u = 0; u < U; ++u) f(c[u]);
        });
    }
}

// Pattern of row i of X*Y: count (PHASE 0) or columns in ascending order (PHASE 1), NW wavefronts per row
// (NW = 4 where a row meets thousands of candidates; they take 64 X entries in turn) and 4 / NW rows per
// workgroup.  The candidates' columns set their flags, a byte each (the same column may be set by many
// lanes at once: plain byte stores, where bits would need atomics that neighbouring columns serialise:
// 8.8 -> 6.0 ms over the products of a 324k-row set-up).  PHASE 0 finds the row's window and leaves it in
// win; flags of masked rows stay empty, and rows whose window exceeds SPG_WIN are left to spg_hash_k.
// Dynamic LDS: 4 / NW maps of `seg` bytes.
// SPG_WIN, the columns of one map (four of them in a workgroup's LDS): against every candidate read once per
// map of the window, set-up of a 324k-row tube renumbered at random 110 -> 52 ms (in layers 41), with rows moved
// by up to 20,000 places 47.0 -> 43.7, of a Y bifurcation of 892k rows 96.9 -> 92.4; windows of up to two and four
// maps read so, the rest hashed: shuffled 53.9 and 65.3, the Y 94.3 and 95.8.
constexpr int SPG_WIN = 8192;
template <int PHASE, int NW>
__global__ void __launch_bounds__(256) spg_pattern_k(int64_t nr, int seg, const int32_t* __restrict__ xrp,
                                                     const int32_t* __restrict__ xci, const int32_t* __restrict__ yrp,
                                                     const int32_t* __restrict__ yci, const uint8_t* __restrict__ rowmask,
                                                     int32_t* __restrict__ win, int32_t* __restrict__ cnt,
                                                     const int32_t* __restrict__ crp,
                                                     int32_t* __restrict__ cci) {
    extern __shared__ uint32_t flagw[];
    __shared__ int red[2][256 / WAVE];
    constexpr int NT = NW * WAVE, ROWS = 256 / NT;
    const int row = threadIdx.x / NT, tid = threadIdx.x % NT, lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const int64_t i = (int64_t)blockIdx.x * ROWS + row;
    uint32_t* fw = flagw + row * (seg / 4);
    uint8_t* fb = reinterpret_cast<uint8_t*>(fw);
    const bool live = i < nr && (!rowmask || rowmask[i]);
    const int32_t x0 = live ? xrp[i] : 0, x1 = live ? xrp[i + 1] : 0;
    int32_t c0 = 0;
    int n = 0;
    if (PHASE == 0) {
        int lo = INT32_MAX, hi = -1;
        for (int32_t q = x0 + tid; q < x1; q += NT) {
            const int32_t k = xci[q];
            const int32_t s = yrp[k], e = yrp[k + 1];
            if (e <= s) continue;
            const int f = yci[s], l = yci[e - 1];
            lo = f < lo ? f : lo;
            hi = l > hi ? l : hi;
        }
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) {
            const int a = __shfl_xor(lo, o, WAVE), b = __shfl_xor(hi, o, WAVE);
            lo = a < lo ? a : lo;
            hi = b > hi ? b : hi;
        }
        if (lane == 0) { red[0][w] = lo; red[1][w] = hi; }
        __syncthreads();
        for (int v = row * NW; v < (row + 1) * NW; ++v) {
            lo = red[0][v] < lo ? red[0][v] : lo;
            hi = red[1][v] > hi ? red[1][v] : hi;
        }
        n = hi >= lo ? hi - lo + 1 : 0;
        c0 = n ? lo : 0;
        if (tid == 0 && i < nr) {
            win[2 * i] = c0;
            win[2 * i + 1] = n;
        }
        __syncthreads();
    } else if (i < nr) {
        c0 = win[2 * i];
        n = win[2 * i + 1];
    }
    if (n > SPG_WIN) n = 0;
    const int words = (n + 3) / 4;
    for (int t = tid; t < words; t += NT) fw[t] = 0;
    __syncthreads();
    if (n > 0)
        for (int32_t q0 = x0 + tid / WAVE * WAVE; q0 < x1; q0 += NT) {
            const SpgList list(q0, x1, lane, xci, yrp);
            spg_columns(list, lane, yci, [&](int32_t c) { fb[c - c0] = 1; });
        }
    __syncthreads();
    int count = 0;
    if (PHASE == 0) {
        for (int t = tid; t < words; t += NT) count += __popc(fw[t]);
    } else if (tid < WAVE && n > 0) {
        // one wavefront emits the columns, 16 of the map per lane: a prefix of the lanes' counts
        int32_t base = crp[i];
        for (int t0 = 0; t0 < words; t0 += 4 * WAVE) {
            uint32_t v[4];
            int own = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + 4 * lane + u;
                v[u] = t < words ? fw[t] : 0;
                own += __popc(v[u]);
            }
            int incl = own;
#pragma unroll
            for (int o = 1; o < WAVE; o <<= 1) {
                const int u = __shfl_up(incl, o, WAVE);
                if (lane >= o) incl += u;
            }
            int32_t at = base + incl - own;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                for (uint32_t m = v[u]; m; m &= m - 1) cci[at++] = c0 + (t0 + 4 * lane + u) * 4 + (__builtin_ctz(m) >> 3);
            base += __shfl(incl, WAVE - 1, WAVE);
        }
    }
    if (PHASE == 0) {
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) count += __shfl_xor(count, o, WAVE);
        if (NW > 1) {
            __syncthreads();
            if (lane == 0) red[1][w] = count;
            __syncthreads();
            count = red[1][0];
            for (int v = 1; v < NW; ++v) count += red[1][v];
        }
        if (tid == 0 && i < nr) cnt[i] = count;
    }
}

// The same for the rows whose window exceeds SPG_WIN, NW wavefronts and one workgroup per row: the columns go
// into a hash table in LDS.  PHASE 0: a table of twice the row's candidates, `hs` slots (a power of two, 512 NW
// or more) at the most; a row whose columns fill half of those gets cnt = -1 and raises *overflow, and a
// later pass (retry) with a larger table counts such rows again.  PHASE 1: a table of twice the row's
// columns, which go to their ranks.  Dynamic LDS: hs slots, in PHASE 1 the longest row's columns after them.
constexpr int HS_COUNT = 2048;     // first table of PHASE 0 (x4 on each overflow)
constexpr int HS_MAX = 2 * HMAX;
__device__ __forceinline__ unsigned hash_slot(int key, int hs) { return ((unsigned)key * 2654435761u) & (unsigned)(hs - 1); }
// true if newly inserted (a table that is never full)
__device__ __forceinline__ bool hash_insert(int* t, int hs, int key) {
    unsigned h = hash_slot(key, hs);
    for (;;) {
        const int prev = atomicCAS(&t[h], -1, key);
        if (prev == -1) return true;
        if (prev == key) return false;
        h = (h + 1) & (unsigned)(hs - 1);
    }
}
template <int PHASE, int NW>
__global__ void __launch_bounds__(NW * WAVE) spg_hash_k(int64_t nr, int hs, int retry, const int32_t* __restrict__ xrp,
                                                        const int32_t* __restrict__ xci, const int32_t* __restrict__ yrp,
                                                        const int32_t* __restrict__ yci, const int32_t* __restrict__ win,
                                                        int32_t* __restrict__ cnt, const int32_t* __restrict__ crp,
                                                        int32_t* __restrict__ cci, int* __restrict__ overflow) {
    extern __shared__ int table[];
    __shared__ unsigned long long cand;     // candidates of the row
    __shared__ int nuniq;
    constexpr int NT = NW * WAVE;
    const int64_t i = blockIdx.x;
    if (i >= nr || win[2 * i + 1] <= SPG_WIN || (PHASE == 0 && retry && cnt[i] >= 0)) return;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int32_t x0 = xrp[i], x1 = xrp[i + 1];
    if (tid == 0) { cand = 0; nuniq = 0; }
    __syncthreads();
    uint64_t want;
    if (PHASE == 0) {
        uint64_t own = 0;
        for (int32_t q = x0 + tid; q < x1; q += NT) {
            const int32_t k = xci[q];
            own += (uint64_t)(yrp[k + 1] - yrp[k]);
        }
        own = wave_sum(own);
        if (lane == 0) atomicAdd(&cand, (unsigned long long)own);
        __syncthreads();
        want = 2 * cand;
    } else {
        want = 2 * (uint64_t)(crp[i + 1] - crp[i]);
    }
    int size = WAVE;
    while (size < hs && (uint64_t)size < want) size <<= 1;
    // half a table at the most, plus what the wavefronts insert between two looks at the number
    const int limit = PHASE == 0 && (uint64_t)size < want ? size / 2 : INT32_MAX;
    int32_t* cols = table + hs;
    for (int t = tid; t < size; t += NT) table[t] = -1;
    __syncthreads();
    for (int32_t q0 = x0 + tid / WAVE * WAVE; q0 < x1; q0 += NT) {
        const SpgList list(q0, x1, lane, xci, yrp);
        spg_columns(list, lane, yci, [&](int32_t c) {
            if (*(volatile int*)&nuniq >= limit) return;
            if (!hash_insert(table, size, c)) return;
            const int at = atomicAdd(&nuniq, 1);
            if (PHASE == 1) cols[at] = c;
        });
    }
    __syncthreads();
    const int w = nuniq;
    if (PHASE == 0) {
        if (tid == 0) {
            cnt[i] = w < limit ? w : -1;
            if (w >= limit) atomicOr(overflow, 1);
        }
    } else {
        for (int a = tid; a < w; a += NT) {
            const int key = cols[a];
            int rank = 0;
            for (int b = 0; b < w; ++b) rank += cols[b] < key;
            cci[crp[i] + rank] = key;
        }
    }
}

// numeric phase of the rows too long for the forms below (more than fit_map columns, fit_hash where they span more
// than SPG_SEG): lane owns output blocks; accumulates X_iq * Y_kc over q in ascending order
constexpr int SPG_SEG = 32768;     // columns of one map of places
template <int M, int N, int P>
__global__ void __launch_bounds__(256) spg_numeric(int64_t nr, int fit_map, int fit_hash, const int32_t* __restrict__ xrp,
                                                   const int32_t* __restrict__ xci, const double* __restrict__ xv, const int32_t* __restrict__ yrp,
                                                   const int32_t* __restrict__ yci, const double* __restrict__ yv,
                                                   const int32_t* __restrict__ crp, const int32_t* __restrict__ cci,
                                                   double* __restrict__ cv) {
    int64_t i = (int64_t)blockIdx.x * 4 + threadIdx.x / WAVE;
    if (i >= nr || crp[i + 1] <= crp[i]) return;
    if (crp[i + 1] - crp[i] <= (cci[crp[i + 1] - 1] - cci[crp[i]] >= SPG_SEG ? fit_hash : fit_map)) return;
    int lane = threadIdx.x & (WAVE - 1);
    for (int32_t p = crp[i] + lane; p < crp[i + 1]; p += WAVE) {
        int32_t c = cci[p];
        double acc[M * P];
        for (int e = 0; e < M * P; ++e) acc[e] = 0.0;
        for (int32_t q = xrp[i]; q < xrp[i + 1]; ++q) {
            int32_t k = xci[q];
            int32_t t = find_col(yci, yrp[k], yrp[k + 1], c);
            if (t < 0) continue;
            const double* xb = xv + (int64_t)q * M * N;
            const double* yb = yv + (int64_t)t * N * P;
            for (int r = 0; r < M; ++r)
                for (int cc = 0; cc < P; ++cc) {
                    double sum = 0.0;
                    for (int l = 0; l < N; ++l) sum += xb[r * N + l] * yb[l * P + cc];
                    acc[r * P + cc] += sum;
                }
        }
        double* o = cv + (int64_t)p * M * P;
        for (int e = 0; e < M * P; ++e) o[e] = acc[e];
    }
}

// ---- numeric phase with the row's sums in LDS.  Every entry of C sums its products in the order of X's row
// (q ascending), as the pull kernel above, so the values are identical: the candidates are taken in list
// order, and products are added to their sums by LDS atomics without return, one X entry per instruction
// (its Y row has distinct columns; spg_add_in_order); LDS serves a wavefront's instructions in order.
// Nothing waits for a sum, so the loads of SPG_PASS passes are in flight.
// The row's columns as {bits, columns before the word} of each 32 columns of the window: a column's place is
// one 8-byte LDS read and a population count.  Rows that span more than SPG_SEG columns: a hash table.
struct SpgWord { uint32_t bits; int32_t before; };
// fills map[0 .. ceil(sn / 32)) for the columns [s0, s0 + sn) of cci[lo, hi), `before` of which come before s0
// (the NT threads of a workgroup); returns the columns up to the segment's end on the first wavefront
template <int NT = WAVE>
__device__ __forceinline__ int spg_map(SpgWord* map, int32_t s0, int sn, const int32_t* __restrict__ cci, int32_t lo,
                                        int32_t hi, int before, int tid) {
    const int sw = (sn + 31) / 32, lane = tid & (WAVE - 1);
    for (int t = tid; t < sw; t += NT) map[t].bits = 0;
    __syncthreads();
    for (int32_t p = lo + tid; p < hi; p += NT) {
        const unsigned at = (unsigned)(cci[p] - s0);
        if (at < (unsigned)sn) atomicOr(&map[at >> 5].bits, 1u << (at & 31));
    }
    __syncthreads();
    if (tid < WAVE)
        for (int t0 = 0; t0 < sw; t0 += WAVE) {
            const int own = t0 + lane < sw ? __popc(map[t0 + lane].bits) : 0;
            int incl = own;
#pragma unroll
            for (int o = 1; o < WAVE; o <<= 1) {
                const int u = __shfl_up(incl, o, WAVE);
                if (lane >= o) incl += u;
            }
            if (t0 + lane < sw) map[t0 + lane].before = before + incl - own;
            before += __shfl(incl, WAVE - 1, WAVE);
        }
    __syncthreads();
    return before;
}
// place of column c in the row, -1 if it lies outside [s0, s0 + sn) (c is one of the row's columns)
__device__ __forceinline__ int spg_place(const SpgWord* map, int32_t s0, int sn, int32_t c) {
    const unsigned at = (unsigned)(c - s0);
    const bool in = at < (unsigned)sn;
    const SpgWord w = map[in ? at >> 5 : 0];
    return in ? w.before + __popc(w.bits & ((1u << (at & 31)) - 1)) : -1;
}
// the places of the columns of cci[lo, hi) in one form or the other; table: a power of two of slots, twice the
// columns or more (its words hold {column, place})
template <bool HASH, int NT>
struct SpgPlaces {
    SpgWord* map;
    int32_t c0;
    int n;       // columns spanned, or slots
    __device__ __forceinline__ SpgPlaces(SpgWord* m, const int32_t* __restrict__ cci, int32_t lo, int32_t hi, int tid) : map(m) {
        if constexpr (HASH) {
            for (n = WAVE; n < 2 * (hi - lo); n <<= 1) {}
            for (int t = tid; t < n; t += NT) map[t].bits = ~0u;
            __syncthreads();
            for (int32_t p = lo + tid; p < hi; p += NT) {
                const int c = cci[p];
                unsigned h = hash_slot(c, n);
                while (atomicCAS(&map[h].bits, ~0u, (uint32_t)c) != ~0u) h = (h + 1) & (unsigned)(n - 1);
                map[h].before = p - lo;
            }
            __syncthreads();
        } else {
            c0 = cci[lo];
            n = cci[hi - 1] - c0 + 1;
            spg_map<NT>(map, c0, n, cci, lo, hi, 0, tid);
        }
    }
    __device__ __forceinline__ int operator()(int32_t c) const {
        if constexpr (HASH) {
            unsigned h = hash_slot(c, n);
            for (;;) {
                const SpgWord w = map[h];
                if (w.bits == (uint32_t)c) return w.before;
                if (w.bits == ~0u) return -1;      // not reached: every column met is in the pattern
                h = (h + 1) & (unsigned)(n - 1);
            }
        } else {
            return spg_place(map, c0, n, c);
        }
    }
};
__device__ __forceinline__ void spg_add(double* p, double v) {
    (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// adds v to sums[p] on the lanes with p >= 0, X entry after X entry (l ascends over the lanes)
__device__ __forceinline__ void spg_add_in_order(double* sums, int p, double v, int l) {
    uint64_t todo = __ballot(p >= 0);
    while (todo) {
        const int lead = __builtin_amdgcn_readlane(l, __builtin_ctzll(todo));
        const bool mine = p >= 0 && l == lead;
        if (mine) spg_add(sums + p, v);
        todo &= ~__ballot(mine);
    }
}

// scalar rows of C (M = P = 1, inner dimension N), one wavefront per row; of the rows of up to `fit` columns those
// that span more than SPG_SEG (HASH) or the others.  Dynamic LDS: `fit` sums, then the map or table.
template <int N, bool HASH>
__global__ void __launch_bounds__(WAVE) spg_scalar_k(int64_t nr, int fit, const int32_t* __restrict__ xrp,
                                                     const int32_t* __restrict__ xci, const double* __restrict__ xv,
                                                     const int32_t* __restrict__ yrp, const int32_t* __restrict__ yci,
                                                     const double* __restrict__ yv, const int32_t* __restrict__ crp,
                                                     const int32_t* __restrict__ cci, double* __restrict__ cv) {
    extern __shared__ double sums[];
    SpgWord* map = reinterpret_cast<SpgWord*>(sums + fit);
    const int64_t i = blockIdx.x;
    if (i >= nr) return;
    const int lane = threadIdx.x;
    const int32_t lo = crp[i], hi = crp[i + 1];
    if (hi <= lo || hi - lo > fit || (cci[hi - 1] - cci[lo] >= SPG_SEG) != HASH) return;
    for (int p = lane; p < hi - lo; p += WAVE) sums[p] = 0.0;
    const int32_t x0 = xrp[i], x1 = xrp[i + 1];
    const SpgPlaces<HASH, WAVE> place(map, cci, lo, hi, lane);
    for (int32_t q0 = x0; q0 < x1; q0 += WAVE) {
        double x[N];
#pragma unroll
        for (int k = 0; k < N; ++k) x[k] = q0 + lane < x1 ? xv[(int64_t)(q0 + lane) * N + k] : 0.0;
        const SpgList list(q0, x1, lane, xci, yrp);
        if (list.is_long()) {
            SpgWalk walk(list);
            while (walk.more()) {
                int l[SPG_PASS];
                int32_t t[SPG_PASS], c[SPG_PASS];
                bool in[SPG_PASS];
                double y[SPG_PASS][N];
#pragma unroll
                for (int u = 0; u < SPG_PASS; ++u) {
                    l[u] = 0;
                    t[u] = u ? t[0] : 0;
                    in[u] = false;
                    if (walk.more()) walk.take(lane, l[u], t[u], in[u]);
                }
#pragma unroll
                for (int u = 0; u < SPG_PASS; ++u) {
                    c[u] = yci[t[u]];
#pragma unroll
                    for (int k = 0; k < N; ++k) y[u][k] = yv[(int64_t)t[u] * N + k];
                }
#pragma unroll
                for (int u = 0; u < SPG_PASS; ++u) {
                    double sum = 0.0;
#pragma unroll
                    for (int k = 0; k < N; ++k) sum += __shfl(x[k], l[u], WAVE) * y[u][k];
                    const int p = place(c[u]);
                    if (in[u] && p >= 0) spg_add(sums + p, sum);
                    __builtin_amdgcn_wave_barrier();
                }
            }
        } else if (list.single()) {
            const bool in = list.len != 0;
            const int32_t t = in ? list.st : 0;
            const int32_t c = yci[t];
            double sum = 0.0;
#pragma unroll
            for (int k = 0; k < N; ++k) sum += x[k] * yv[(int64_t)t * N + k];
            spg_add_in_order(sums, in ? place(c) : -1, sum, lane);
        } else {
            spg_steps(list.total, WAVE, [&](int base, auto steps) {
                constexpr int U = decltype(steps)::value;
                int l[U];
                int32_t t[U], c[U];
                double y[U][N];
#pragma unroll
                for (int u = 0; u < U; ++u) list.get(base + u * WAVE + lane, l[u], t[u]);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    c[u] = yci[t[u]];
#pragma unroll
                    for (int k = 0; k < N; ++k) y[u][k] = yv[(int64_t)t[u] * N + k];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    double sum = 0.0;
#pragma unroll
                    for (int k = 0; k < N; ++k) sum += __shfl(x[k], l[u], WAVE) * y[u][k];
                    const bool in = base + u * WAVE + lane < list.total;
                    spg_add_in_order(sums, in ? place(c[u]) : -1, sum, l[u]);
                }
            });
        }
    }
    __syncthreads();
    for (int p = lane; p < hi - lo; p += WAVE) cv[lo + p] = sums[p];
}

// block rows (M x P blocks of C, inner dimension N), MP / 9 wavefronts per row: each owns 9 entries of every
// block, so that each sum has one owner and the sums in LDS (18 or 36 doubles per block
// column, which bound the rows in flight) serve 2 or 4 wavefronts; a pass takes 7 candidates, one lane
// per entry.  Rows and dynamic LDS as above (fit * M * P sums).
constexpr int SPG_E = 9;
struct SpgCand { int32_t t, lp; };     // Y index; X entry (bits 24-29) and place in the row (bits 0-23)
template <int M, int N, int P, bool HASH>
__global__ void __launch_bounds__(M* P / SPG_E* WAVE)
    spg_block_k(int64_t nr, int fit, const int32_t* __restrict__ xrp, const int32_t* __restrict__ xci,
                const double* __restrict__ xv, const int32_t* __restrict__ yrp, const int32_t* __restrict__ yci,
                const double* __restrict__ yv, const int32_t* __restrict__ crp, const int32_t* __restrict__ cci,
                double* __restrict__ cv) {
    constexpr int MP = M * P, E = SPG_E, NW = MP / E, CPP = WAVE / E, NT = NW * WAVE;
    extern __shared__ double sums[];
    __shared__ SpgCand batch[NT];
    SpgWord* map = reinterpret_cast<SpgWord*>(sums + (size_t)fit * MP);
    const int64_t i = blockIdx.x;
    if (i >= nr) return;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int32_t lo = crp[i], hi = crp[i + 1];
    if (hi <= lo || hi - lo > fit || (cci[hi - 1] - cci[lo] >= SPG_SEG) != HASH) return;
    for (int p = tid; p < (hi - lo) * MP; p += NT) sums[p] = 0.0;
    const int32_t x0 = xrp[i], x1 = xrp[i + 1];
    const int slot = lane / E;                  // lane 63 holds no candidate (slot 7)
    const int en = w * E + lane % E, r = en / P, cc = en % P;
    const SpgPlaces<HASH, NT> place(map, cci, lo, hi, tid);
    for (int32_t q0 = x0; q0 < x1; q0 += WAVE) {
        const SpgList list(q0, x1, lane, xci, yrp);
        for (int base = 0; base < list.total; base += NT) {
            // a batch: each thread finds one candidate and its place, for the wavefronts to share
            int l;
            int32_t t;
            list.get(base + tid, l, t);
            const int32_t col = yci[t];
            __syncthreads();
            batch[tid].t = t;
            batch[tid].lp = base + tid < list.total ? (l << 24 | (place(col) & 0xffffff)) : -1;
            __syncthreads();
            const int left = list.total - base < NT ? list.total - base : NT;
            spg_steps(left, CPP, [&](int b0, auto steps) {
                constexpr int U = decltype(steps)::value;
                int lu[U], p[U];
                double x[U][N], y[U][N];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int at = b0 + u * CPP + slot;
                    const bool in = slot < CPP && at < left;
                    const SpgCand c = batch[in ? at : b0];
                    lu[u] = (c.lp >> 24) & 63;
                    p[u] = in ? (c.lp << 8) >> 8 : -1;
#pragma unroll
                    for (int k = 0; k < N; ++k) {
                        x[u][k] = xv[((int64_t)(q0 + lu[u]) * M + r) * N + k];
                        y[u][k] = yv[((int64_t)c.t * N + k) * P + cc];
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    double sum = 0.0;
#pragma unroll
                    for (int k = 0; k < N; ++k) sum += x[u][k] * y[u][k];
                    spg_add_in_order(sums, p[u] >= 0 ? p[u] * MP + en : -1, sum, lu[u]);
                }
            });
        }
    }
    __syncthreads();
    for (int p = tid; p < (hi - lo) * MP; p += NT) cv[(int64_t)lo * MP + p] = sums[p];
}

// numeric phase of C = X Y into C's pattern: the rows whose sums and map or table fit into LDS (SPG_LDS: two
// workgroups a CU), and the longer ones by the pull form
constexpr int SPG_LDS = 68 * 1024;
static void spgemm_numeric(const DBsr& X, const DBsr& Y, DBsr& C, hipStream_t s) {
    if (X.nr <= 0) return;
    const int key = X.br * 100 + X.bc * 10 + Y.bc, mp = C.br * C.bc;
    const int most = SPG_LDS - (mp > 1 ? mp / SPG_E * WAVE * (int)sizeof(SpgCand) : 0), sum = mp * (int)sizeof(double);
    const int words = (std::min(C.wmax_cols, SPG_SEG) + 31) / 32 * (int)sizeof(SpgWord);
    const int fit_map = std::min(C.wmax, (most - words) / sum);
    // (the table of twice the columns is a power of two: the size that leaves room for the longest row)
    int fit_hash = 0, table = 0;
    for (int t = WAVE; C.wmax_cols > SPG_SEG && fit_hash < C.wmax && t * (int)sizeof(SpgWord) < most; t <<= 1) {
        const int f = std::min({C.wmax, t / 2, (most - t * (int)sizeof(SpgWord)) / sum});
        if (f > fit_hash) { fit_hash = f; table = t * (int)sizeof(SpgWord); }
    }
    const bool wide = fit_hash > 0, pull = fit_map < C.wmax || (wide && fit_hash < C.wmax);
    const size_t lds = (size_t)(fit_map * sum + words), ldsh = (size_t)(fit_hash * sum + table);
    const unsigned nb = (unsigned)cdiv(X.nr, 4);
#define SPG_ARGS X.rp, X.ci, X.v, Y.rp, Y.ci, Y.v, C.rp, C.ci, C.v
#define SPS(n)                                                                                                  \
    {                                                                                                           \
        spg_scalar_k<n, false><<<(unsigned)X.nr, WAVE, lds, s>>>(X.nr, fit_map, SPG_ARGS);                      \
        if (wide) spg_scalar_k<n, true><<<(unsigned)X.nr, WAVE, ldsh, s>>>(X.nr, fit_hash, SPG_ARGS);           \
        if (pull) spg_numeric<1, n, 1><<<nb, 256, 0, s>>>(X.nr, fit_map, fit_hash, SPG_ARGS);                   \
    }
#define SPB(m, n, p)                                                                                            \
    {                                                                                                           \
        constexpr int T = m * p / SPG_E * WAVE;                                                                 \
        spg_block_k<m, n, p, false><<<(unsigned)X.nr, T, lds, s>>>(X.nr, fit_map, SPG_ARGS);                    \
        if (wide) spg_block_k<m, n, p, true><<<(unsigned)X.nr, T, ldsh, s>>>(X.nr, fit_hash, SPG_ARGS);         \
        if (pull) spg_numeric<m, n, p><<<nb, 256, 0, s>>>(X.nr, fit_map, fit_hash, SPG_ARGS);                   \
    }
    switch (key) {
        case 111: SPS(1) break;
        case 131: SPS(3) break;
        case 336: SPB(3, 3, 6) break;
        case 636: SPB(6, 3, 6) break;
        case 666: SPB(6, 6, 6) break;
        default: throw Error(SCR_E_UNIMPLEMENTED, "spgemm block shape " + std::to_string(key));
    }
#undef SPS
#undef SPB
#undef SPG_ARGS
    check_launch("spg_numeric");
}

DBsr spgemm(const DBsr& X, const DBsr& Y, const uint8_t* rowmask, Arena& ar, hipStream_t s) {
    DBsr C;
    C.nr = X.nr; C.nc = Y.nc; C.br = X.br; C.bc = Y.bc;
    C.rp = ar.make<int32_t>(X.nr + 1);
    int32_t* cnt = ar.make<int32_t>(X.nr + 1);
    int32_t* win = ar.make<int32_t>(2 * X.nr + 1);
    struct Head { int maxwin, wmax, overflow; };     // widest window, longest row
    Head* head = ar.make<Head>(1);
    Head h{};
    zero_dev(head, sizeof(Head), s);
    // rows that meet SPG_WIDE candidates or more (by the mean lengths of both factors) take four wavefronts
    const bool wide = X.nr > 0 && Y.nr > 0 &&
                      (double)X.nnzb * (double)Y.nnzb >= (double)SPG_WIDE * (double)X.nr * (double)Y.nr;
    const int seg = (int)(std::min<int64_t>(Y.nc > 0 ? Y.nc : 1, SPG_WIN) + 3) / 4 * 4;
    const unsigned grid = (unsigned)cdiv(X.nr, wide ? 1 : 4);
    const size_t lds = (size_t)seg * (wide ? 1 : 4);
#define SPP(ph)                                                                                                    \
    if (X.nr > 0 && wide)                                                                                          \
        spg_pattern_k<ph, 4><<<grid, 256, lds, s>>>(X.nr, seg, X.rp, X.ci, Y.rp, Y.ci, rowmask, win, cnt,          \
                                                    C.rp, C.ci);                                    \
    else if (X.nr > 0)                                                                                             \
        spg_pattern_k<ph, 1><<<grid, 256, lds, s>>>(X.nr, seg, X.rp, X.ci, Y.rp, Y.ci, rowmask, win, cnt,          \
                                                    C.rp, C.ci)
#define SPH(ph, lds, hs, retry)                                                                                    \
    if (wide)                                                                                                      \
        spg_hash_k<ph, 4><<<(unsigned)X.nr, 4 * WAVE, lds, s>>>(X.nr, hs, retry, X.rp, X.ci, Y.rp, Y.ci, win, cnt, \
                                                               C.rp, C.ci, &head->overflow);                       \
    else                                                                                                           \
        spg_hash_k<ph, 1><<<(unsigned)X.nr, WAVE, lds, s>>>(X.nr, hs, retry, X.rp, X.ci, Y.rp, Y.ci, win, cnt,     \
                                                            C.rp, C.ci, &head->overflow)
    auto totals = [&]() {      // C.rp, C.nnzb and h from the counts
        if (X.nr > 0)
            spg_max_k<<<(unsigned)std::min<int64_t>(cdiv(X.nr, 256), 256), 256, 0, s>>>(X.nr, cnt, win, &head->wmax,
                                                                                        &head->maxwin);
        check_launch("spg_count");
        HIPCHK(hipMemcpyAsync(&h, head, sizeof(Head), hipMemcpyDeviceToHost, s));
        C.nnzb = scan_i32(cnt, C.rp, X.nr, ar, s);      // synchronises
    };
    SPP(0);
    totals();
    const bool far = h.maxwin > SPG_WIN;
    if (far) {
        // the counts of the rows that the pattern kernel left
        for (int hs = HS_COUNT, retry = 0;; hs *= 4, retry = 1) {
            SPH(0, (size_t)hs * sizeof(int), hs, retry);
            check_launch("spg_hash");
            HIPCHK(hipMemcpyAsync(&h, head, sizeof(Head), hipMemcpyDeviceToHost, s));
            HIPCHK(hipStreamSynchronize(s));
            if (!h.overflow) break;
            if (hs >= HS_MAX) throw Error(SCR_E_INVALID, "Galerkin product row wider than " + std::to_string(HMAX) + " blocks");
            zero_dev(&head->overflow, sizeof(int), s);
        }
        totals();
    }
    if (h.wmax >= HMAX) throw Error(SCR_E_INVALID, "Galerkin product row wider than " + std::to_string(HMAX) + " blocks");
    C.wmax = h.wmax;
    C.wmax_cols = h.maxwin;
    C.ci = ar.make<int32_t>(C.nnzb > 0 ? C.nnzb : 1);
    C.v = ar.make<double>((C.nnzb > 0 ? C.nnzb : 1) * C.br * C.bc);
    SPP(1);
    if (far) {
        int hs = WAVE;
        while (hs < 2 * h.wmax) hs <<= 1;
        SPH(1, (size_t)(hs + h.wmax) * sizeof(int), hs, 0);
    }
#undef SPP
#undef SPH
    check_launch("spg_fill");
    ar.free(cnt); ar.free(win); ar.free(head);
    spgemm_numeric(X, Y, C, s);
    return C;
}

__global__ void __launch_bounds__(256) rowlen_max_k(int64_t nr, const int32_t* __restrict__ rp, int* __restrict__ out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    block_max_to(i < nr ? rp[i + 1] - rp[i] : 0, out);
}

// ---------------------------------------------------------------------- S^ = C - D d^-1 G
// d per velocity dof: the diagonal of A (mode 0) or the sum of the absolute values of its row
// (mode 1, SIMPLEC), summed block by block in column order
__global__ void schur_diag_k(int64_t nr, int mode, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                             const double* __restrict__ Av, double* __restrict__ d) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    if (mode == 0) {
        int32_t dq = find_col(ci, rp[i], rp[i + 1], (int32_t)i);
        for (int c = 0; c < 3; ++c) d[3 * i + c] = Av[(int64_t)dq * 9 + 4 * c];
        return;
    }
    for (int c = 0; c < 3; ++c) {
        double sum = 0.0;
        for (int32_t q = rp[i]; q < rp[i + 1]; ++q)
            for (int k = 0; k < 3; ++k) sum += fabs(Av[(int64_t)q * 9 + 3 * c + k]);
        d[3 * i + c] = sum;
    }
}
__global__ void diag_scale_D(int64_t nr, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                             const double* __restrict__ d, const double* __restrict__ Dv, double* __restrict__ X) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    for (int32_t q = rp[i]; q < rp[i + 1]; ++q) {
        int32_t j = ci[q];
        for (int c = 0; c < 3; ++c) X[(int64_t)q * 3 + c] = Dv[(int64_t)q * 3 + c] / d[3 * (int64_t)j + c];
    }
}
// union pattern of C and DG (both sorted, a column at most once per row): count, then fill with
// C - DG.  One wavefront per row: an entry's place in the union is its index in its own row, plus
// the entries of the other row with smaller columns, minus the columns the two rows share below it
// (a prefix count of the shared flags over its own row); a column in both rows is written once, by
// its C entry.
template <int PHASE>
__global__ void __launch_bounds__(256) merge_sub_k(int64_t nr, const int32_t* __restrict__ arp, const int32_t* __restrict__ aci,
                                                   const double* __restrict__ av, const int32_t* __restrict__ brp,
                                                   const int32_t* __restrict__ bci, const double* __restrict__ bv,
                                                   int32_t* __restrict__ cnt, const int32_t* __restrict__ crp,
                                                   int32_t* __restrict__ cci, double* __restrict__ cv) {
    const int64_t i = (int64_t)blockIdx.x * (256 / WAVE) + threadIdx.x / WAVE;
    if (i >= nr) return;
    const int lane = threadIdx.x & (WAVE - 1);
    const uint64_t below = (1ull << lane) - 1;
    const int32_t a0 = arp[i], a1 = arp[i + 1], b0 = brp[i], b1 = brp[i + 1];
    const int32_t o = PHASE ? crp[i] : 0;
    int shared = 0;
    for (int32_t base = a0; base < a1; base += WAVE) {
        const int32_t a = base + lane;
        const bool in = a < a1;
        const int32_t ca = in ? aci[a] : 0;
        const int32_t lb = in ? lower_col(bci, b0, b1, ca) : b1;
        const bool m = in && lb < b1 && bci[lb] == ca;
        const uint64_t mask = __ballot(m);
        if (PHASE && in) {
            const int32_t pos = (a - a0) + (lb - b0) - (shared + __popcll(mask & below));
            cci[o + pos] = ca;
            cv[o + pos] = m ? av[a] - bv[lb] : av[a];
        }
        shared += __popcll(mask);
    }
    if (!PHASE) {
        if (lane == 0) cnt[i] = (a1 - a0) + (b1 - b0) - shared;
        return;
    }
    shared = 0;
    for (int32_t base = b0; base < b1; base += WAVE) {
        const int32_t b = base + lane;
        const bool in = b < b1;
        const int32_t cb = in ? bci[b] : 0;
        const int32_t la = in ? lower_col(aci, a0, a1, cb) : a1;
        const bool m = in && la < a1 && aci[la] == cb;
        const uint64_t mask = __ballot(m);
        if (in && !m) {
            const int32_t pos = (la - a0) + (b - b0) - (shared + __popcll(mask & below));
            cci[o + pos] = cb;
            cv[o + pos] = -bv[b];
        }
        shared += __popcll(mask);
    }
}

DBsr schur_approx(const DBsr& A, const DBsr& G, const DBsr& D, const DBsr& C, int mode, double* d, DBsr& DG, Arena& ar,
                  hipStream_t s) {
    DBsr X = D;
    X.v = ar.make<double>(D.nnzb * 3);
    if (A.nr > 0) schur_diag_k<<<cdiv(A.nr, 256), 256, 0, s>>>(A.nr, mode, A.rp, A.ci, A.v, d);
    if (D.nr > 0) diag_scale_D<<<cdiv(D.nr, 256), 256, 0, s>>>(D.nr, D.rp, D.ci, d, D.v, X.v);
    check_launch("diag_scale_D");
    DG = spgemm(X, G, nullptr, ar, s);
    ar.free(X.v);
    DBsr S;
    S.nr = C.nr; S.nc = C.nc; S.br = 1; S.bc = 1;
    S.rp = ar.make<int32_t>(C.nr + 1);
    int32_t* cnt = ar.make<int32_t>(C.nr + 1);
    int64_t nw = cdiv(C.nr, 256 / WAVE);
    if (nw) merge_sub_k<0><<<nw, 256, 0, s>>>(C.nr, C.rp, C.ci, C.v, DG.rp, DG.ci, DG.v, cnt, nullptr, nullptr, nullptr);
    S.nnzb = scan_i32(cnt, S.rp, C.nr, ar, s);
    ar.free(cnt);
    S.ci = ar.make<int32_t>(S.nnzb);
    S.v = ar.make<double>(S.nnzb);
    if (nw) merge_sub_k<1><<<nw, 256, 0, s>>>(C.nr, C.rp, C.ci, C.v, DG.rp, DG.ci, DG.v, nullptr, S.rp, S.ci, S.v);
    check_launch("merge_sub");
    ar.free(DG.v);
    DG.v = nullptr;
    return S;
}

void schur_update(const DBsr& A, const DBsr& G, const DBsr& D, const DBsr& C, int mode, double* d, DBsr& DG, DBsr& S,
                  Arena& ar, hipStream_t s) {
    DBsr X = D;
    X.v = ar.make<double>(D.nnzb * 3);
    if (A.nr > 0) schur_diag_k<<<cdiv(A.nr, 256), 256, 0, s>>>(A.nr, mode, A.rp, A.ci, A.v, d);
    if (D.nr > 0) diag_scale_D<<<cdiv(D.nr, 256), 256, 0, s>>>(D.nr, D.rp, D.ci, d, D.v, X.v);
    check_launch("diag_scale_D");
    DG.v = ar.make<double>(DG.nnzb > 0 ? DG.nnzb : 1);
    spgemm_numeric(X, G, DG, s);
    ar.free(X.v);
    int64_t nw = cdiv(C.nr, 256 / WAVE);
    if (nw) merge_sub_k<1><<<nw, 256, 0, s>>>(C.nr, C.rp, C.ci, C.v, DG.rp, DG.ci, DG.v, nullptr, S.rp, S.ci, S.v);
    check_launch("merge_sub");
    ar.free(DG.v);
    DG.v = nullptr;
}

// ---------------------------------------------------------------------- rigid-body modes
__global__ void centroid_partial(int64_t nb, const double* __restrict__ xyz, double* __restrict__ part) {
    __shared__ double red[3][256];
    double a[3] = {0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nb; i += (int64_t)gridDim.x * 256)
        for (int d = 0; d < 3; ++d) a[d] += xyz[3 * i + d];
    for (int d = 0; d < 3; ++d) red[d][threadIdx.x] = a[d];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o)
            for (int d = 0; d < 3; ++d) red[d][threadIdx.x] += red[d][threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int d = 0; d < 3; ++d) part[blockIdx.x * 3 + d] = red[d][0];
}
__global__ void rigid_k(int64_t nb, const double* __restrict__ xyz, const double* __restrict__ part, int np,
                        double* __restrict__ B) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nb) return;
    double c[3] = {0.0, 0.0, 0.0};
    for (int p = 0; p < np; ++p)
        for (int d = 0; d < 3; ++d) c[d] += part[p * 3 + d];
    double x = xyz[3 * i] - c[0] / (double)nb, y = xyz[3 * i + 1] - c[1] / (double)nb, z = xyz[3 * i + 2] - c[2] / (double)nb;
    double* r0 = B + (3 * i) * 6;
    double* r1 = r0 + 6;
    double* r2 = r1 + 6;
    for (int t = 0; t < 6; ++t) { r0[t] = 0.0; r1[t] = 0.0; r2[t] = 0.0; }
    r0[0] = 1.0; r1[1] = 1.0; r2[2] = 1.0;
    r0[3] = -y; r1[3] = x;
    r1[4] = -z; r2[4] = y;
    r0[5] = z; r2[5] = -x;
}
void rigid_modes(int64_t nb, const double* xyz, double* B, Arena& ar, hipStream_t s) {
    int np = 64;
    double* part = ar.make<double>(np * 3);
    centroid_partial<<<np, 256, 0, s>>>(nb, xyz, part);
    if (nb > 0) rigid_k<<<cdiv(nb, 256), 256, 0, s>>>(nb, xyz, part, np, B);
    check_launch("rigid_modes");
    ar.free(part);
}

// ====================================================================== strength and MIS-2
// squared Frobenius norm of every block, its entries added in order.  A workgroup takes 64 blocks: their
// values come coalesced through LDS (36 values a block read by one thread each kept 64 lines per load busy:
// the strength pass over 1.35M 6x6 blocks took 970 us)
__global__ void __launch_bounds__(256) block_f_k(int64_t nnzb, int bb, const double* __restrict__ v, double* __restrict__ f) {
    extern __shared__ double stage[];        // 64 blocks of bb values, bb + 1 apart
    const int64_t q0 = (int64_t)blockIdx.x * WAVE;
    const int n = nnzb - q0 < WAVE ? (int)(nnzb - q0) : WAVE;
    for (int t = threadIdx.x; t < n * bb; t += 256) {
        const int q = t / bb;
        stage[q * (bb + 1) + t - q * bb] = v[q0 * bb + t];
    }
    __syncthreads();
    if ((int)threadIdx.x >= n) return;
    double sum = 0.0;
    for (int e = 0; e < bb; ++e) {
        const double x = stage[threadIdx.x * (bb + 1) + e];
        sum = sum + x * x;
    }
    f[q0 + threadIdx.x] = sum;
}
__global__ void fdiag_k(int64_t nr, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci, const double* __restrict__ f,
                        double* __restrict__ fd) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    int32_t q = find_col(ci, rp[i], rp[i + 1], (int32_t)i);
    fd[i] = q >= 0 ? f[q] : 0.0;
}
// strength of the coupling at entry q = (i, j) of row i, symmetrised with (j, i), which is looked up only
// where (i, j) alone is not strong
__device__ __forceinline__ uint8_t strong_entry(int64_t i, int32_t q, const int32_t* __restrict__ rp,
                                                const int32_t* __restrict__ ci, const double* __restrict__ f,
                                                const double* __restrict__ fd, double th4) {
    const int32_t j = ci[q];
    if (j == i) return 0;
    const double fij = f[q];
    if ((fij * fij) >= ((th4 * fd[i]) * fd[j])) return 1;
    const int32_t t = find_col(ci, rp[j], rp[j + 1], (int32_t)i);
    if (t < 0) return 0;
    const double fji = f[t];
    return (fji * fji) >= ((th4 * fd[j]) * fd[i]) ? 1 : 0;
}

__global__ void strength_k(int64_t nr, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                           const double* __restrict__ f, const double* __restrict__ fd, double th4,
                           uint8_t* __restrict__ flags, uint8_t* __restrict__ iso) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    uint8_t any = 0;
    for (int32_t q = rp[i]; q < rp[i + 1]; ++q) {
        const uint8_t st = strong_entry(i, q, rp, ci, f, fd, th4);
        flags[q] = st;
        any |= st;
    }
    iso[i] = any ? 0 : 1;
}

// the same with one wavefront per row, lanes over its entries (levels with long rows)
__global__ void __launch_bounds__(256) strength_wave_k(int64_t nr, const int32_t* __restrict__ rp,
                                                       const int32_t* __restrict__ ci, const double* __restrict__ f,
                                                       const double* __restrict__ fd, double th4,
                                                       uint8_t* __restrict__ flags, uint8_t* __restrict__ iso) {
    const int64_t i = (int64_t)blockIdx.x * (256 / WAVE) + threadIdx.x / WAVE;
    const int lane = threadIdx.x & (WAVE - 1);
    if (i >= nr) return;
    int any = 0;
    for (int32_t q = rp[i] + lane; q < rp[i + 1]; q += WAVE) {
        const uint8_t st = strong_entry(i, q, rp, ci, f, fd, th4);
        flags[q] = st;
        any |= st;
    }
    const uint64_t b = __ballot(any);
    if (lane == 0) iso[i] = b ? 0 : 1;
}

// state word: top 2 bits = 0 out/isolated, 1 undecided, 2 in; low 62 bits = priority
constexpr uint64_t ST_UND = 1ULL << 62, ST_IN = 2ULL << 62, KEYMASK = (1ULL << 62) - 1;

__global__ void mis_init_k(int64_t nr, const uint8_t* __restrict__ iso, uint64_t seed, int level, uint64_t* __restrict__ st) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    st[i] = iso[i] ? 0ULL : (ST_UND | mis_key(seed, level, i));
}
__global__ void mis_max_k(int64_t nr, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                          const uint8_t* __restrict__ flags, const uint64_t* __restrict__ in, uint64_t* __restrict__ out,
                          const uint64_t* __restrict__ und_only) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    if (und_only && (und_only[i] >> 62) != 1) return;
    uint64_t m = in[i];
    for (int32_t q = rp[i]; q < rp[i + 1]; ++q)
        if (flags[q]) {
            uint64_t v = in[ci[q]];
            m = v > m ? v : m;
        }
    out[i] = m;
}
// the same with one wavefront per row (levels with long rows)
__global__ void __launch_bounds__(256) mis_max_wave_k(int64_t nr, const int32_t* __restrict__ rp,
                                                      const int32_t* __restrict__ ci, const uint8_t* __restrict__ flags,
                                                      const uint64_t* __restrict__ in, uint64_t* __restrict__ out,
                                                      const uint64_t* __restrict__ und_only) {
    const int64_t i = (int64_t)blockIdx.x * (256 / WAVE) + threadIdx.x / WAVE;
    const int lane = threadIdx.x & (WAVE - 1);
    if (i >= nr) return;
    if (und_only && (und_only[i] >> 62) != 1) return;
    uint64_t m = 0;
    for (int32_t q = rp[i] + lane; q < rp[i + 1]; q += WAVE)
        if (flags[q]) {
            uint64_t v = in[ci[q]];
            m = v > m ? v : m;
        }
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        uint64_t w = __shfl_xor(m, o, WAVE);
        m = w > m ? w : m;
    }
    if (lane == 0) {
        const uint64_t self = in[i];
        out[i] = self > m ? self : m;
    }
}
// *und becomes nonzero if a node stays undecided (one atomic per workgroup at most)
__global__ void __launch_bounds__(256) mis_decide_k(int64_t nr, uint64_t* __restrict__ st,
                                                    const uint64_t* __restrict__ m2, int* __restrict__ und) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int left = 0;
    if (i < nr) {
        uint64_t s = st[i];
        if ((s >> 62) == 1) {
            uint64_t m = m2[i];
            if ((m >> 62) == 2) st[i] = s & KEYMASK;               // an IN node within distance 2
            else if (m == s) st[i] = ST_IN | (s & KEYMASK);        // largest undecided priority within distance 2
            else left = 1;
        }
    }
    if (__syncthreads_or(left) && threadIdx.x == 0) atomicOr(und, 1);
}

__global__ void root_flag_k(int64_t nr, const uint64_t* __restrict__ st, int32_t* __restrict__ isroot) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nr) isroot[i] = (st[i] >> 62) == 2 ? 1 : 0;
}
__global__ void agg_roots_k(int64_t nr, const uint64_t* __restrict__ st, const int32_t* __restrict__ rid,
                            int32_t* __restrict__ agg) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nr) agg[i] = (st[i] >> 62) == 2 ? rid[i] : -1;
}
// (a wavefront per row; the first strong IN neighbour, and the strong neighbour of largest key, as a walk over
// the row in order finds them)
__global__ void __launch_bounds__(256) agg_dist1_k(int64_t nr, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                                   const uint8_t* __restrict__ flags, const uint8_t* __restrict__ iso,
                                                   const uint64_t* __restrict__ st, const int32_t* __restrict__ rid,
                                                   int32_t* __restrict__ agg, uint8_t* __restrict__ step1) {
    const int64_t i = (int64_t)blockIdx.x * (256 / WAVE) + threadIdx.x / WAVE;
    if (i >= nr) return;
    const int lane = threadIdx.x & (WAVE - 1);
    if (iso[i] || (st[i] >> 62) == 2) {
        if (lane == 0) step1[i] = 0;
        return;
    }
    for (int32_t q0 = rp[i]; q0 < rp[i + 1]; q0 += WAVE) {
        const int32_t q = q0 + lane;
        const bool in = q < rp[i + 1];
        const int32_t j = in ? ci[q] : 0;
        const uint64_t hit = __ballot(in && flags[q] && (st[j] >> 62) == 2);
        if (hit) {
            if (lane == __builtin_ctzll(hit)) {
                agg[i] = rid[j];
                step1[i] = 1;
            }
            return;
        }
    }
    if (lane == 0) step1[i] = 0;
}
__global__ void __launch_bounds__(256) agg_dist2_k(int64_t nr, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                                   const uint8_t* __restrict__ flags, const uint8_t* __restrict__ iso,
                                                   const uint8_t* __restrict__ step1, uint64_t seed, int level,
                                                   int32_t* __restrict__ agg, int* __restrict__ err) {
    const int64_t i = (int64_t)blockIdx.x * (256 / WAVE) + threadIdx.x / WAVE;
    if (i >= nr) return;
    const int lane = threadIdx.x & (WAVE - 1);
    if (iso[i] || agg[i] >= 0) return;
    uint64_t best = 0;       // key + 1 (keys hold the index: no two are equal)
    for (int32_t q = rp[i] + lane; q < rp[i + 1]; q += WAVE) {
        const int32_t j = ci[q];
        if (!flags[q] || !step1[j]) continue;
        const uint64_t kj = mis_key(seed, level, j) + 1;
        best = kj > best ? kj : best;
    }
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        const uint64_t k = __shfl_xor(best, o, WAVE);
        best = k > best ? k : best;
    }
    if (lane != 0) return;
    if (best == 0) { atomicOr(err, 1); return; }
    agg[i] = agg[(uint32_t)(best - 1)];   // it joined in the distance-1 step: its aggregate is final
}

// ====================================================================== tentative prolongator
__global__ void agg_count_k(int64_t nr, const int32_t* __restrict__ agg, int32_t* __restrict__ cnt) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nr && agg[i] >= 0) atomicAdd(&cnt[agg[i]], 1);
}
__global__ void agg_fill_k(int64_t nr, const int32_t* __restrict__ agg, const int32_t* __restrict__ mrp,
                           int32_t* __restrict__ fillc, int32_t* __restrict__ mem) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nr && agg[i] >= 0) mem[mrp[agg[i]] + atomicAdd(&fillc[agg[i]], 1)] = (int32_t)i;
}
// members of each aggregate in ascending order: every member goes to its rank in its aggregate's list
__global__ void agg_sort_k(int64_t nm, const int32_t* __restrict__ agg, const int32_t* __restrict__ mrp,
                           const int32_t* __restrict__ mem, int32_t* __restrict__ out) {
    int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= nm) return;
    const int32_t i = mem[m];
    const int32_t lo = mrp[agg[i]], hi = mrp[agg[i] + 1];
    int32_t rank = 0;
    for (int32_t t = lo; t < hi; ++t) rank += mem[t] < i;
    out[lo + rank] = i;
}

// Gram-Schmidt (two modified-GS passes) of B restricted to the aggregate's rows (members in
// ascending order, b rows each).  Column j is dead when its remainder is <= 1e-10 of its norm.
__global__ void tentative_k(int64_t na, int b, int k, const int32_t* __restrict__ mrp, const int32_t* __restrict__ mem,
                            const double* __restrict__ B, double* __restrict__ Q, double* __restrict__ Bc,
                            uint8_t* __restrict__ dead) {
    int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= na) return;
    int32_t lo = mrp[a], hi = mrp[a + 1];
    double* Rk = Bc + a * k * k;
    for (int e = 0; e < k * k; ++e) Rk[e] = 0.0;
    // Q rows of the members start as B rows
    for (int32_t t = lo; t < hi; ++t) {
        int64_t node = mem[t];
        for (int r = 0; r < b; ++r)
            for (int c = 0; c < k; ++c) Q[(node * b + r) * k + c] = B[(node * b + r) * k + c];
    }
    for (int j = 0; j < k; ++j) {
        double nb = 0.0;
        for (int32_t t = lo; t < hi; ++t)
            for (int r = 0; r < b; ++r) {
                double w = Q[((int64_t)mem[t] * b + r) * k + j];
                nb += w * w;
            }
        nb = sqrt(nb);
        for (int pass = 0; pass < 2; ++pass)
            for (int i = 0; i < j; ++i) {
                if (dead[a * k + i]) continue;
                double c = 0.0;
                for (int32_t t = lo; t < hi; ++t)
                    for (int r = 0; r < b; ++r) {
                        int64_t row = ((int64_t)mem[t] * b + r) * k;
                        c += Q[row + i] * Q[row + j];
                    }
                for (int32_t t = lo; t < hi; ++t)
                    for (int r = 0; r < b; ++r) {
                        int64_t row = ((int64_t)mem[t] * b + r) * k;
                        Q[row + j] -= c * Q[row + i];
                    }
                Rk[i * k + j] += c;
            }
        double nv = 0.0;
        for (int32_t t = lo; t < hi; ++t)
            for (int r = 0; r < b; ++r) {
                double w = Q[((int64_t)mem[t] * b + r) * k + j];
                nv += w * w;
            }
        nv = sqrt(nv);
        bool isdead = (nb == 0.0) || (nv <= 1e-10 * nb);
        dead[a * k + j] = isdead ? 1 : 0;
        for (int32_t t = lo; t < hi; ++t)
            for (int r = 0; r < b; ++r) {
                int64_t row = ((int64_t)mem[t] * b + r) * k;
                Q[row + j] = isdead ? 0.0 : Q[row + j] / nv;
            }
        Rk[j * k + j] = isdead ? 0.0 : nv;
    }
}

// The same factorisation with one wavefront per aggregate and the aggregate's rows of Q in LDS (rows in member
// order, k columns).  The products of a dot go to LDS from all lanes, and every lane then adds them in row
// order (the rounding is that of tentative_k, and no lane waits for another's result); the element-wise
// updates run on all lanes.  Dynamic LDS: nmax b k values of Q, then nmax b products.
__device__ __forceinline__ double ordered_sum(const double* p, int n) {
    double sum = 0.0;
    int t = 0;
    for (; t + 8 <= n; t += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = p[t + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) sum += x[u];
    }
    for (; t < n; ++t) sum += p[t];
    return sum;
}
__global__ void __launch_bounds__(WAVE) tentative_lds_k(int64_t na, int b, int k, int nmax, const int32_t* __restrict__ mrp,
                                                        const int32_t* __restrict__ mem, const double* __restrict__ B,
                                                        double* __restrict__ Q, double* __restrict__ Bc,
                                                        uint8_t* __restrict__ dead) {
    extern __shared__ double q[];
    double* prod = q + (size_t)nmax * b * k;
    const int64_t a = blockIdx.x;
    if (a >= na) return;
    const int lane = threadIdx.x;
    const int32_t lo = mrp[a], hi = mrp[a + 1];
    const int nrow = (hi - lo) * b;
    for (int e = lane; e < nrow * k; e += WAVE) {
        const int rr = e / k, c = e - rr * k;
        const int t = rr / b, r = rr - t * b;
        q[e] = B[((int64_t)mem[lo + t] * b + r) * k + c];
    }
    for (int e = lane; e < k * k; e += WAVE) Bc[a * k * k + e] = 0.0;
    __syncthreads();
    auto dot = [&](int i, int j) {
        for (int rr = lane; rr < nrow; rr += WAVE) prod[rr] = q[rr * k + i] * q[rr * k + j];
        __syncthreads();
        const double c = ordered_sum(prod, nrow);
        __syncthreads();
        return c;
    };
    unsigned gone = 0;       // dead columns (k <= 8)
    for (int j = 0; j < k; ++j) {
        const double nb = sqrt(dot(j, j));
        double rij[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) rij[i] = 0.0;
        for (int pass = 0; pass < 2; ++pass)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (i >= j || (gone >> i) & 1) continue;
                const double c = dot(i, j);
                rij[i] += c;
                for (int rr = lane; rr < nrow; rr += WAVE) q[rr * k + j] -= c * q[rr * k + i];
                __syncthreads();
            }
        const double nv = sqrt(dot(j, j));
        const bool isdead = (nb == 0.0) || (nv <= 1e-10 * nb);
        if (isdead) gone |= 1u << j;
        if (lane == 0) {
            dead[a * k + j] = isdead ? 1 : 0;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i < j) Bc[a * k * k + i * k + j] = rij[i];
            Bc[a * k * k + j * k + j] = isdead ? 0.0 : nv;
        }
        for (int rr = lane; rr < nrow; rr += WAVE) q[rr * k + j] = isdead ? 0.0 : q[rr * k + j] / nv;
        __syncthreads();
    }
    for (int e = lane; e < nrow * k; e += WAVE) {
        const int rr = e / k, c = e - rr * k;
        const int t = rr / b, r = rr - t * b;
        Q[((int64_t)mem[lo + t] * b + r) * k + c] = q[e];
    }
}

// tentative prolongator of all aggregates: the LDS form when the largest aggregate fits
static void tentative_run(int64_t na, int b, int k, const int32_t* mrp, const int32_t* mem, const double* B,
                          double* Q, double* Bc, uint8_t* dead, Arena& ar, hipStream_t s) {
    if (na <= 0) return;
    int* mx = ar.make<int>(1);
    zero_dev(mx, sizeof(int), s);
    rowlen_max_k<<<cdiv(na, 256), 256, 0, s>>>(na, mrp, mx);
    check_launch("agg_max");
    int hm = 0;
    HIPCHK(hipMemcpyAsync(&hm, mx, sizeof(int), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    ar.free(mx);
    const size_t lds = (size_t)hm * b * (k + 1) * sizeof(double);
    if (k <= 8 && lds <= 56 * 1024) tentative_lds_k<<<(unsigned)na, WAVE, lds, s>>>(na, b, k, hm, mrp, mem, B, Q, Bc, dead);
    else tentative_k<<<cdiv(na, 64), 64, 0, s>>>(na, b, k, mrp, mem, B, Q, Bc, dead);
    check_launch("tentative");
}

// P_tent as BSR: one b x k block per aggregated row
__global__ void ptent_cnt_k(int64_t nr, const int32_t* __restrict__ agg, int32_t* __restrict__ cnt) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nr) cnt[i] = agg[i] >= 0 ? 1 : 0;
}
__global__ void ptent_fill_k(int64_t nr, int bk, const int32_t* __restrict__ agg, const int32_t* __restrict__ rp,
                             const double* __restrict__ Q, int32_t* __restrict__ ci, double* __restrict__ v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr || agg[i] < 0) return;
    int32_t q = rp[i];
    ci[q] = agg[i];
    for (int e = 0; e < bk; ++e) v[(int64_t)q * bk + e] = Q[i * bk + e];
}

// ====================================================================== D^-1 and lambda_hat
template <int B>
__device__ bool invert_small(const double* __restrict__ a, double* __restrict__ out) {
    double m[B][2 * B];
    for (int r = 0; r < B; ++r)
        for (int c = 0; c < B; ++c) {
            m[r][c] = a[r * B + c];
            m[r][B + c] = r == c ? 1.0 : 0.0;
        }
    for (int k = 0; k < B; ++k) {
        int p = k;
        double best = fabs(m[k][k]);
        for (int r = k + 1; r < B; ++r)
            if (fabs(m[r][k]) > best) { best = fabs(m[r][k]); p = r; }
        if (best == 0.0) return false;
        if (p != k)
            for (int c = 0; c < 2 * B; ++c) { double t = m[k][c]; m[k][c] = m[p][c]; m[p][c] = t; }
        double piv = m[k][k];
        for (int c = 0; c < 2 * B; ++c) m[k][c] /= piv;
        for (int r = 0; r < B; ++r) {
            if (r == k) continue;
            double f = m[r][k];
            for (int c = 0; c < 2 * B; ++c) m[r][c] -= f * m[k][c];
        }
    }
    for (int r = 0; r < B; ++r)
        for (int c = 0; c < B; ++c) out[r * B + c] = m[r][B + c];
    return true;
}

template <int B>
__global__ void __launch_bounds__(256) dinv_k(int64_t nr, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                              const double* __restrict__ v, double* __restrict__ Dinv, int* __restrict__ err) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    const int32_t q = find_col(ci, rp[i], rp[i + 1], (int32_t)i);
    double Di[B * B];
    const bool ok = q >= 0 && invert_small<B>(v + (int64_t)q * B * B, Di);
    if (!ok) atomicOr(err, 1);
    for (int e = 0; e < B * B; ++e) Dinv[i * B * B + e] = ok ? Di[e] : 0.0;
}
// lam = max over the rows of the absolute row sums of D^-1 A: a wavefront per block row (grid-stride), its
// blocks over the lanes (one thread per row left rows of 50 and more blocks to one lane: 6x6 blocks at
// 24,500 rows 650 us)
constexpr int LAMBDA_BLOCKS = 2048;
template <int B>
__global__ void __launch_bounds__(256) lambda_k(int64_t nr, const int32_t* __restrict__ rp, const double* __restrict__ v,
                                                const double* __restrict__ Dinv, unsigned long long* __restrict__ lam) {
    const int lane = threadIdx.x & (WAVE - 1), w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    double m = 0.0;     // max absolute row sum of D^-1 A over the rows taken
    for (int64_t i = (int64_t)blockIdx.x * (256 / WAVE) + w; i < nr; i += (int64_t)gridDim.x * (256 / WAVE)) {
        double Di[B * B], rs[B];
#pragma unroll
        for (int e = 0; e < B * B; ++e) Di[e] = Dinv[i * B * B + e];
#pragma unroll
        for (int r = 0; r < B; ++r) rs[r] = 0.0;
        for (int32_t t = rp[i] + lane; t < rp[i + 1]; t += WAVE) {
            double blk[B * B];
#pragma unroll
            for (int e = 0; e < B * B; ++e) blk[e] = v[(int64_t)t * B * B + e];
#pragma unroll
            for (int r = 0; r < B; ++r)
#pragma unroll
                for (int c = 0; c < B; ++c) {
                    double sum = 0.0;
#pragma unroll
                    for (int l = 0; l < B; ++l) sum += Di[r * B + l] * blk[l * B + c];
                    rs[r] += fabs(sum);
                }
        }
#pragma unroll
        for (int r = 0; r < B; ++r) {
            const double sum = wave_sum(rs[r]);
            m = sum > m ? sum : m;
        }
    }
    // nonnegative doubles order as their bit patterns
    block_max_to((unsigned long long)__double_as_longlong(m), lam);
}

// P = -omega D^-1 (A P_tent) + P_tent  (rows of AP_t are those of P)
template <int B, int K>
__global__ void smooth_p_k(int64_t nr, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                           double* __restrict__ v, const double* __restrict__ Dinv, const int32_t* __restrict__ agg,
                           const double* __restrict__ Q, double omega) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr || agg[i] < 0) return;
    const double* Di = Dinv + i * B * B;
    for (int32_t q = rp[i]; q < rp[i + 1]; ++q) {
        double* blk = v + (int64_t)q * B * K;
        double t[B * K];
        for (int r = 0; r < B; ++r)
            for (int c = 0; c < K; ++c) {
                double sum = 0.0;
                for (int l = 0; l < B; ++l) sum += Di[r * B + l] * blk[l * K + c];
                t[r * K + c] = -omega * sum;
            }
        if (ci[q] == agg[i])
            for (int e = 0; e < B * K; ++e) t[e] += Q[i * B * K + e];
        for (int e = 0; e < B * K; ++e) blk[e] = t[e];
    }
}

// ====================================================================== transpose
__global__ void tr_count_k(int64_t nnz, const int32_t* __restrict__ ci, int32_t* __restrict__ cnt) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < nnz) atomicAdd(&cnt[ci[q]], 1);
}
__global__ void tr_fill_k(int64_t nr, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                          const int32_t* __restrict__ trp, int32_t* __restrict__ fillc, int32_t* __restrict__ tci,
                          int32_t* __restrict__ src) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    for (int32_t q = rp[i]; q < rp[i + 1]; ++q) {
        int32_t c = ci[q];
        int32_t pos = trp[c] + atomicAdd(&fillc[c], 1);
        tci[pos] = (int32_t)i;
        src[pos] = q;
    }
}
// the entries of each transposed row in ascending order (source rows are unique within a row): a wavefront per
// row, the place of an entry from the prefix counts of a map of the row's keys (TR_SEG keys of its window at
// a time), as in the products above; rows of a thousand entries cost no more per entry than short ones.  A short
// row of a wide window counts the smaller keys of each entry instead: its work does not depend on the numbering.
constexpr int TR_SEG = 8192;
constexpr int TR_PAIRS = 512;     // comparisons of a wavefront in about the time that a segment of the map takes
__global__ void __launch_bounds__(WAVE) tr_sort_k(int64_t ntr, const int32_t* __restrict__ trp, const int32_t* __restrict__ tci,
                                                  const int32_t* __restrict__ src, int32_t* __restrict__ oci,
                                                  int32_t* __restrict__ osrc) {
    __shared__ SpgWord map[TR_SEG / 32];
    const int64_t r = blockIdx.x;
    if (r >= ntr) return;
    const int lane = threadIdx.x;
    const int32_t lo = trp[r], hi = trp[r + 1];
    if (hi <= lo) return;
    int k0 = INT32_MAX, k1 = -1;
    for (int32_t p = lo + lane; p < hi; p += WAVE) {
        const int k = tci[p];
        k0 = k < k0 ? k : k0;
        k1 = k > k1 ? k : k1;
    }
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        const int a = __shfl_xor(k0, o, WAVE), b = __shfl_xor(k1, o, WAVE);
        k0 = a < k0 ? a : k0;
        k1 = b > k1 ? b : k1;
    }
    const int len = hi - lo;
    if (k1 - k0 >= TR_SEG && (int64_t)len * ((len + WAVE - 1) / WAVE) <= TR_PAIRS * ((int64_t)(k1 - k0) / TR_SEG + 1)) {
        for (int32_t p = lo + lane; p < hi; p += WAVE) {
            const int32_t k = tci[p];
            int rank = 0;
            for (int32_t u = lo; u < hi; ++u) rank += tci[u] < k;
            oci[lo + rank] = k;
            osrc[lo + rank] = src[p];
        }
        return;
    }
    int before = 0;
    for (int64_t s0 = k0; s0 <= k1; s0 += TR_SEG) {
        const int sn = k1 + 1 - s0 < TR_SEG ? (int)(k1 + 1 - s0) : TR_SEG;
        before = spg_map(map, (int32_t)s0, sn, tci, lo, hi, before, lane);
        for (int32_t p = lo + lane; p < hi; p += WAVE) {
            const int32_t k = tci[p];
            const int at = spg_place(map, (int32_t)s0, sn, k);
            if (at >= 0) {
                oci[lo + at] = k;
                osrc[lo + at] = src[p];
            }
        }
        __syncthreads();
    }
}
// values of the transpose from those of the matrix: thread per value, in the order they are written
__global__ void tr_values_k(int64_t nv, int br, int bc, const int32_t* __restrict__ src, const double* __restrict__ v,
                            double* __restrict__ ov) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nv) return;
    const int bb = br * bc;
    const int64_t p = t / bb;
    const int e = (int)(t - p * bb), c = e / br, r = e - c * br;
    ov[t] = v[(int64_t)src[p] * bb + r * bc + c];
}

// M^T; src (if not NULL) receives the index in M of each of its entries, for transpose_values
DBsr transpose(const DBsr& M, Arena& ar, hipStream_t s, int32_t** src_out) {
    DBsr T;
    T.nr = M.nc; T.nc = M.nr; T.br = M.bc; T.bc = M.br; T.nnzb = M.nnzb;
    int32_t* cnt = ar.make<int32_t>(M.nc + 1);
    zero_dev(cnt, (M.nc + 1) * sizeof(int32_t), s);
    if (M.nnzb) tr_count_k<<<cdiv(M.nnzb, 256), 256, 0, s>>>(M.nnzb, M.ci, cnt);
    T.rp = ar.make<int32_t>(M.nc + 1);
    scan_i32(cnt, T.rp, M.nc, ar, s);
    zero_dev(cnt, (M.nc + 1) * sizeof(int32_t), s);
    int32_t* tci = ar.make<int32_t>(M.nnzb + 1);
    int32_t* src = ar.make<int32_t>(M.nnzb + 1);
    if (M.nr) tr_fill_k<<<cdiv(M.nr, 256), 256, 0, s>>>(M.nr, M.rp, M.ci, T.rp, cnt, tci, src);
    T.ci = ar.make<int32_t>(M.nnzb + 1);
    T.v = ar.make<double>((M.nnzb + 1) * M.br * M.bc);
    int32_t* osrc = ar.make<int32_t>(M.nnzb + 1);
    if (T.nr) tr_sort_k<<<(unsigned)T.nr, WAVE, 0, s>>>(T.nr, T.rp, tci, src, T.ci, osrc);
    check_launch("transpose");
    ar.free(cnt); ar.free(tci); ar.free(src);
    transpose_values(M, T, osrc, s);
    if (src_out) *src_out = osrc;
    else ar.free(osrc);
    return T;
}
void transpose_values(const DBsr& M, DBsr& T, const int32_t* src, hipStream_t s) {
    const int64_t nv = M.nnzb * M.br * M.bc;
    if (nv) tr_values_k<<<cdiv(nv, 256), 256, 0, s>>>(nv, M.br, M.bc, src, M.v, T.v);
    check_launch("transpose values");
}

__global__ void dead_diag_k(int64_t na, int k, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                            double* __restrict__ v, const uint8_t* __restrict__ dead) {
    int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= na) return;
    int32_t q = find_col(ci, rp[a], rp[a + 1], (int32_t)a);
    if (q < 0) return;
    for (int c = 0; c < k; ++c)
        if (dead[a * k + c]) v[(int64_t)q * k * k + c * k + c] = 1.0;
}

// ====================================================================== coarsest level: dense inverse
__global__ void densify_k(int64_t nr, int b, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                          const double* __restrict__ v, double* __restrict__ M, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    for (int32_t q = rp[i]; q < rp[i + 1]; ++q)
        for (int r = 0; r < b; ++r)
            for (int c = 0; c < b; ++c) M[(i * b + r) * n + (int64_t)ci[q] * b + c] = v[((int64_t)q * b + r) * b + c];
}
// Gauss-Jordan exchange steps over all pivots in order turn A into A^-1.  This fast form takes
// the pivots in order without interchanges; the result is checked afterwards (the backward error
// of one solve with it, coarse_check_*) and recomputed with row interchanges (partial pivoting,
// gjp_*) when a small or zero leading pivot spoilt it: the coarsest operators are not SPD in
// general (the advective velocity block is nonsymmetric).
// A panel of GJ_P consecutive pivots K = [k0, k0 + np) at once, by the block form of the exchange
// step (equal in exact arithmetic to the np single steps in order): with W = M_KK^-1,
//   out_KK = W,  out_KR = W M_KR,  out_RK = -M_RK W,  out_RR = M_RR - M_RK W M_KR.
constexpr int GJ_P = 32;
// W by single exchange steps in LDS (every workgroup, redundantly), then T = M_RK W for the
// workgroup's rows (T is n x GJ_P); workgroup 0 also stores W
__global__ void __launch_bounds__(256) gj_panel_t_k(int64_t n, int64_t k0, int np, const double* __restrict__ src,
                                                    double* __restrict__ T, double* __restrict__ Wout) {
    __shared__ double W[GJ_P][GJ_P + 1];
    constexpr int PER = GJ_P * GJ_P / 256;     // entries of W per thread (compile-time: registers)
    {
        double w0[PER];     // all loads issued before the first is used (clamped, branch-free indices)
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            int e = threadIdx.x + 256 * c;
            int ee = e < np * np ? e : 0;
            w0[c] = src[(k0 + ee / np) * n + k0 + ee % np];
        }
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            int e = threadIdx.x + 256 * c;
            if (e < np * np) W[e / np][e % np] = w0[c];
        }
    }
    __syncthreads();
    for (int k = 0; k < np; ++k) {
        const double ip = 1.0 / W[k][k];
        double upd[PER];
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            int e = threadIdx.x + 256 * c;
            upd[c] = 0.0;
            if (e < np * np) {
                int i = e / np, j = e % np;
                if (i == k) upd[c] = (j == k) ? ip : W[k][j] * ip;
                else if (j == k) upd[c] = -W[i][k] * ip;
                else upd[c] = W[i][j] - W[i][k] * W[k][j] * ip;
            }
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            int e = threadIdx.x + 256 * c;
            if (e < np * np) W[e / np][e % np] = upd[c];
        }
        __syncthreads();
    }
    if (blockIdx.x == 0)
        for (int e = threadIdx.x; e < np * np; e += 256) Wout[e] = W[e / np][e % np];
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    double r[GJ_P];     // the row's panel entries, loaded once (clamped, branch-free indices)
#pragma unroll
    for (int l = 0; l < GJ_P; ++l) r[l] = src[i * n + k0 + (l < np ? l : np - 1)];
    for (int c = 0; c < np; ++c) {
        double t = 0.0;
#pragma unroll
        for (int l = 0; l < GJ_P; ++l)
            if (l < np) t += r[l] * W[l][c];
        T[i * GJ_P + c] = t;
    }
}
__global__ void gj_panel_apply_k(int64_t n, int64_t k0, int np, const double* __restrict__ src,
                                 const double* __restrict__ T, const double* __restrict__ W, double* __restrict__ dst) {
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n * n) return;
    int64_t i = idx / n, j = idx % n;
    bool iK = i >= k0 && i < k0 + np, jK = j >= k0 && j < k0 + np;
    double out;
    if (iK && jK) {
        out = W[(i - k0) * np + (j - k0)];
    } else if (iK) {
        out = 0.0;
        for (int l = 0; l < np; ++l) out += W[(i - k0) * np + l] * src[(k0 + l) * n + j];
    } else if (jK) {
        out = -T[i * GJ_P + (j - k0)];
    } else {
        out = src[idx];
        for (int l = 0; l < np; ++l) out -= T[i * GJ_P + l] * src[(k0 + l) * n + j];
    }
    dst[idx] = out;
}
__global__ void finite_k(int64_t n, const double* __restrict__ a, int* __restrict__ err) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && !isfinite(a[i])) atomicOr(err, 1);
}

// ---- accuracy check of an explicit inverse X of A: y = X v for a fixed v, then the normwise
// backward error eta = ||A y - v||_inf / (||A||_inf ||y||_inf + ||v||_inf) (about n * 1e-16 for
// a stable inverse; a spoilt pivot makes it large or non-finite)
__device__ __forceinline__ double check_vec(int64_t i) { return 1.0 + (double)((i * 7919) % 13) / 13.0; }
__global__ void __launch_bounds__(256) coarse_check_y_k(int64_t n, const double* __restrict__ X, double* __restrict__ y) {
    int64_t row = (int64_t)blockIdx.x * 4 + threadIdx.x / WAVE;
    if (row >= n) return;
    int lane = threadIdx.x & (WAVE - 1);
    double acc = 0.0;
    for (int64_t c = lane; c < n; c += WAVE) acc += X[row * n + c] * check_vec(c);
    acc = wave_sum(acc);
    if (lane == 0) y[row] = acc;
}
// per row: |(A y)_i - v_i| and the absolute row sum of A
__global__ void __launch_bounds__(256) coarse_check_r_k(int64_t n, const double* __restrict__ A, const double* __restrict__ y,
                                                        double* __restrict__ rr, double* __restrict__ ra) {
    int64_t row = (int64_t)blockIdx.x * 4 + threadIdx.x / WAVE;
    if (row >= n) return;
    int lane = threadIdx.x & (WAVE - 1);
    double acc = 0.0, abs_sum = 0.0;
    for (int64_t c = lane; c < n; c += WAVE) {
        acc += A[row * n + c] * y[c];
        abs_sum += fabs(A[row * n + c]);
    }
    acc = wave_sum(acc);
    abs_sum = wave_sum(abs_sum);
    if (lane == 0) {
        rr[row] = fabs(acc - check_vec(row));
        ra[row] = abs_sum;
    }
}
// one workgroup: eta into *eta (NaN propagates: fmax would drop it, so non-finite values are flagged)
__global__ void __launch_bounds__(256) coarse_check_eta_k(int64_t n, const double* __restrict__ rr,
                                                          const double* __restrict__ ra, const double* __restrict__ y,
                                                          double* __restrict__ eta) {
    __shared__ double red[3][256];
    __shared__ int bad;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    double m[3] = {0.0, 0.0, 0.0};
    int nf = 0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const double a = rr[i], b = ra[i], c = fabs(y[i]);
        if (!isfinite(a) || !isfinite(b) || !isfinite(c)) nf = 1;
        m[0] = a > m[0] ? a : m[0];
        m[1] = b > m[1] ? b : m[1];
        m[2] = c > m[2] ? c : m[2];
    }
    if (nf) atomicOr(&bad, 1);
    for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = m[q];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o)
            for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = fmax(red[q][threadIdx.x], red[q][threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) *eta = bad ? INFINITY : red[0][0] / (red[1][0] * red[2][0] + 2.0);
}

// ---- Gauss-Jordan with partial pivoting (the fallback): step k picks the row p >= k with the
// largest |M_pk| (the smallest such p on ties), swaps rows k and p of the current matrix and
// applies the exchange step at (k, k); at the end the column interchanges are undone in reverse
// order (the inverse of the row-permuted matrix is A^-1 P^-1).
__global__ void __launch_bounds__(256) gjp_pivot_k(int64_t n, int64_t k, double* __restrict__ M, int32_t* __restrict__ perm,
                                                   int* __restrict__ err) {
    __shared__ double bv[256];
    __shared__ int64_t bi[256];
    double best = -1.0;
    int64_t arg = n;
    for (int64_t i = k + threadIdx.x; i < n; i += 256) {
        const double v = fabs(M[i * n + k]);
        if (v > best) { best = v; arg = i; }     // ascending i per thread: the first largest
    }
    bv[threadIdx.x] = best;
    bi[threadIdx.x] = arg;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            const double v = bv[threadIdx.x + o];
            const int64_t a = bi[threadIdx.x + o];
            if (v > bv[threadIdx.x] || (v == bv[threadIdx.x] && a < bi[threadIdx.x])) {
                bv[threadIdx.x] = v;
                bi[threadIdx.x] = a;
            }
        }
        __syncthreads();
    }
    const int64_t p = bi[0];
    if (threadIdx.x == 0) {
        perm[k] = (int32_t)(p < n ? p : k);
        if (!(bv[0] > 0.0) || !isfinite(bv[0])) atomicOr(err, 1);
    }
    if (p >= n || p == k) return;
    for (int64_t j = threadIdx.x; j < n; j += 256) {
        const double a = M[k * n + j];
        M[k * n + j] = M[p * n + j];
        M[p * n + j] = a;
    }
}
__global__ void gjp_exchange_k(int64_t n, int64_t k, const double* __restrict__ src, double* __restrict__ dst) {
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n * n) return;
    const int64_t i = idx / n, j = idx % n;
    const double ip = 1.0 / src[k * n + k];
    double out;
    if (i == k) out = (j == k) ? ip : src[k * n + j] * ip;
    else if (j == k) out = -src[i * n + k] * ip;
    else out = src[idx] - src[i * n + k] * src[k * n + j] * ip;
    dst[idx] = out;
}
// undo the interchanges on the columns: row i applies swap (k, perm[k]) for k = n-1 .. 0
__global__ void gjp_unpermute_k(int64_t n, const int32_t* __restrict__ perm, double* __restrict__ M) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double* row = M + i * n;
    for (int64_t k = n - 1; k >= 0; --k) {
        const int64_t p = perm[k];
        if (p != k) {
            const double a = row[k];
            row[k] = row[p];
            row[p] = a;
        }
    }
}

// ====================================================================== hierarchy with solve-phase data in T
template <typename T>
class HierT : public Hierarchy {
   public:
    struct LS {
        DSell<T> A, P;
        DBsrT<T> R;
        T* Dinv = nullptr;
        T *b = nullptr, *x = nullptr, *w = nullptr, *t1 = nullptr, *t2 = nullptr, *d = nullptr, *r = nullptr;
        // the same vectors for three interleaved columns (scalar hierarchies built with `three`)
        T *b3 = nullptr, *x3 = nullptr, *w3 = nullptr, *t13 = nullptr, *t23 = nullptr, *d3 = nullptr, *r3 = nullptr;
        std::vector<double> c1, c2;    // smoothing-step coefficients
        bool cheb = false;
    };
    std::vector<LS> S;
    Arena* ar = nullptr;
    Profiler* prof = nullptr;

    void prepare(Arena& a, hipStream_t s) {
        ar = &a;
        S.resize(L.size());
        for (size_t l = 0; l < L.size(); ++l) {
            LevelSetup& ls = L[l];
            LS& q = S[l];
            int64_t n = ls.A.nr * ls.b;
            q.b = a.make<T>(n); q.x = a.make<T>(n);
            if (three) { q.b3 = a.make<T>(3 * n); q.x3 = a.make<T>(3 * n); }
            if (l + 1 == L.size()) continue;
            q.A = sell_from_bsr<T>(ls.A, a, s);
            q.P = sell_from_bsr<T>(ls.P, a, s);
            q.R = bsrt_from_bsr<T>(ls.R, a, s);
            q.Dinv = a.make<T>((int64_t)ls.A.nr * ls.b * ls.b);
            q.w = a.make<T>(n); q.t1 = a.make<T>(n); q.t2 = a.make<T>(n); q.d = a.make<T>(n); q.r = a.make<T>(n);
            if (three) {
                q.w3 = a.make<T>(3 * n); q.t13 = a.make<T>(3 * n); q.t23 = a.make<T>(3 * n);
                q.d3 = a.make<T>(3 * n); q.r3 = a.make<T>(3 * n);
            }
            smoother(l, s);
        }
    }
    // D^-1 in T and the smoothing coefficients of level l from its set-up data:
    // step t computes dn = c1[t] d + c2[t] Dinv (b - A x)
    void smoother(size_t l, hipStream_t s) {
        LevelSetup& ls = L[l];
        LS& q = S[l];
        const int64_t bb = (int64_t)ls.A.nr * ls.b * ls.b;
        if (std::is_same<T, double>::value) copy_d(bb, ls.Dinv, (double*)q.Dinv, s);
        else cast_d2f(ls.Dinv, (float*)q.Dinv, bb, s);
        q.c1.clear();
        q.c2.clear();
        if (opts.smoother == SCR_SMOOTH_CHEBYSHEV) {
            q.cheb = true;
            double lmax = ls.lam, lmin = ls.lam / opts.cheb_ratio;
            double theta = 0.5 * (lmax + lmin), delta = 0.5 * (lmax - lmin);
            double sigma = theta / delta, rho_prev = 1.0 / sigma;
            q.c1.push_back(0.0); q.c2.push_back(1.0 / theta);
            for (int t = 1; t < opts.cheb_degree; ++t) {
                double rho = 1.0 / (2.0 * sigma - rho_prev);
                q.c1.push_back(rho * rho_prev); q.c2.push_back(2.0 * rho / delta);
                rho_prev = rho;
            }
        } else {
            double w = 4.0 / (3.0 * ls.lam);
            for (int t = 0; t < opts.jacobi_sweeps; ++t) { q.c1.push_back(0.0); q.c2.push_back(w); }
        }
    }

    // the patterns are kept: new values into the same slices, vectors and index arrays untouched
    void refresh(Arena&, hipStream_t s) override {
        for (size_t l = 0; l + 1 < L.size(); ++l) {
            sell_refill(L[l].A, S[l].A, s);
            sell_refill(L[l].P, S[l].P, s);
            bsrt_refill(L[l].R, S[l].R, s);
            smoother(l, s);
        }
    }

    // algorithmic bytes of one smoother step with a matrix product: every stored block (values
    // and column index) once, a 4-byte row index per block row, x once, the right-hand side, the
    // output and d as used.  D^-1 is not counted: it follows from the diagonal block the step
    // streams anyway (the block-row-lane kernels solve with that block; the other smoothers read
    // the stored inverse, which this count leaves out).
    double step_bytes(const LS& q, bool rd, bool wd) const {
        const double b = q.A.br, t = sizeof(T);
        double rows = (double)q.A.nr;
        return (double)q.A.nnzb * (b * b * t + 4.0) + rows * (4.0 + b * t * (3.0 + (rd ? 1.0 : 0.0) + (wd ? 1.0 : 0.0)));
    }

    // smoothing sweeps from xin (nullptr = zero) into dst.  Passes over a level's matrix alternate in
    // direction (down), so that each starts with what the one before left in the caches; the last sweep
    // runs down, and the product with the system matrix that follows in a Krylov step runs up.
    void smooth(size_t l, LS& q, const T* b, const T* xin, T* dst, bool& down, hipStream_t s) {
        int ns = (int)q.c1.size();
        const T* cur = xin;
        for (int t = 0; t < ns; ++t) {
            T* out = (t == ns - 1) ? dst : ((t % 2 == 0) ? q.t1 : q.t2);
            bool rd = q.cheb && t > 0, wd = q.cheb && t + 1 < ns, zero = cur == nullptr;
            bool timed = prof && l == 0 && !zero;
            hipEvent_t e0 = nullptr, e1 = nullptr;
            if (timed) { e0 = prof->get(); e1 = prof->get(); }
            smooth_step<T>(q.A, q.Dinv, b, cur, q.d, out, q.c1[t], q.c2[t], rd, wd, zero, down, s, e0, e1);
            if (!zero) down = !down;
            if (timed) prof->push(e0, e1, step_bytes(q, rd, wd));
            cur = out;
        }
    }

    void cycle(size_t l, const T* b, T* x, hipStream_t s) {
        if (l + 1 == S.size()) {
            dense_mv<T>(ncoarse, cinv, b, x, s);
            return;
        }
        LS& q = S[l];
        bool down = true;
        smooth(l, q, b, nullptr, q.w, down, s);
        sell_mv<T>(q.A, q.w, b, q.r, 1, down, s);
        bsrt_mv<T>(q.R, q.r, S[l + 1].b, s);
        cycle(l + 1, S[l + 1].b, S[l + 1].x, s);
        sell_mv<T>(q.P, S[l + 1].x, nullptr, q.w, 2, s);
        down = false;
        smooth(l, q, b, q.w, x, down, s);
    }

    // the V-cycle on three interleaved columns: every kernel passes over its matrix once for all
    // three, and each column's result is bitwise the one-column V-cycle's
    void smooth3(LS& q, const T* b, const T* xin, T* dst, bool& down, hipStream_t s) {
        int ns = (int)q.c1.size();
        const T* cur = xin;
        for (int t = 0; t < ns; ++t) {
            T* out = (t == ns - 1) ? dst : ((t % 2 == 0) ? q.t13 : q.t23);
            bool rd = q.cheb && t > 0, wd = q.cheb && t + 1 < ns, zero = cur == nullptr;
            smooth_step3<T>(q.A, q.Dinv, b, cur, q.d3, out, q.c1[t], q.c2[t], rd, wd, zero, down, s);
            if (!zero) down = !down;
            cur = out;
        }
    }
    void cycle3(size_t l, const T* b, T* x, hipStream_t s) {
        if (l + 1 == S.size()) {
            dense_mv3<T>(ncoarse, cinv, b, x, s);
            return;
        }
        LS& q = S[l];
        bool down = true;
        smooth3(q, b, nullptr, q.w3, down, s);
        sell_mv3<T>(q.A, q.w3, b, q.r3, 1, down, s);
        bsrt_mv3<T>(q.R, q.r3, S[l + 1].b3, s);
        cycle3(l + 1, S[l + 1].b3, S[l + 1].x3, s);
        sell_mv3<T>(q.P, S[l + 1].x3, nullptr, q.w3, 2, s);
        down = false;
        smooth3(q, b, q.w3, x, down, s);
    }
    void vcycle3(const double* x, double* y, hipStream_t s) override {
        if (!three) throw Error(SCR_E_INVALID, "three-column V-cycle on a hierarchy built without it");
        vcycles += 3;
        int64_t n = n0();
        if (std::is_same<T, double>::value) {
            cycle3(0, (const T*)x, (T*)y, s);
        } else {
            cast_d2f(x, (float*)S[0].b3, 3 * n, s);
            cycle3(0, S[0].b3, S[0].x3, s);
            cast_f2d((const float*)S[0].x3, y, 3 * n, s);
        }
    }

    void vcycle_f(const float* x, float* y, hipStream_t s) override {
        if (!std::is_same<T, float>::value) throw Error(SCR_E_INVALID, "FP32 V-cycle on an FP64 hierarchy");
        ++vcycles;
        cycle(0, (const T*)x, (T*)y, s);
    }
    const DSell<float>* level0_f() const override {
        if (!std::is_same<T, float>::value || S.size() < 2) return nullptr;
        return (const DSell<float>*)&S[0].A;
    }
    const DSell<double>* level0_d() const override {
        if (!std::is_same<T, double>::value || S.size() < 2) return nullptr;
        return (const DSell<double>*)&S[0].A;
    }

    void vcycle(const double* x, double* y, hipStream_t s) override {
        ++vcycles;
        int64_t n = n0();
        if (std::is_same<T, double>::value) {
            cycle(0, (const T*)x, (T*)y, s);
        } else {
            cast_d2f(x, (float*)S[0].b, n, s);
            cycle(0, S[0].b, S[0].x, s);
            cast_f2d((const float*)S[0].x, y, n, s);
        }
    }
};

__global__ void rowmask_k(int64_t nr, const int32_t* __restrict__ agg, uint8_t* __restrict__ m) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nr) m[i] = agg[i] >= 0 ? 1 : 0;
}

// ====================================================================== hierarchy construction
// D^-1 (into L.Dinv) and lambda_hat = max abs row sum of D^-1 A (into L.lam)
void level_diag(LevelSetup& L, int l, int* err, unsigned long long* lamd, hipStream_t s) {
    const int64_t nr = L.A.nr;
    const int64_t g = cdiv(nr, 256);
    const int b = L.b;
    zero_dev(err, sizeof(int), s);
    zero_dev(lamd, sizeof(unsigned long long), s);
    if (g) {
        const unsigned gl = (unsigned)std::min<int64_t>(cdiv(nr, 256 / WAVE), LAMBDA_BLOCKS);
#define DL(B)                                                                     \
    {                                                                             \
        dinv_k<B><<<g, 256, 0, s>>>(nr, L.A.rp, L.A.ci, L.A.v, L.Dinv, err);      \
        lambda_k<B><<<gl, 256, 0, s>>>(nr, L.A.rp, L.A.v, L.Dinv, lamd);          \
    }
        if (b == 1) DL(1)
        else if (b == 3) DL(3)
        else if (b == 6) DL(6)
        else throw Error(SCR_E_UNIMPLEMENTED, "AMG block size");
#undef DL
    }
    check_launch("dinv_lambda");
    unsigned long long hl = 0;
    int he = 0;
    HIPCHK(hipMemcpyAsync(&hl, lamd, sizeof(hl), hipMemcpyDeviceToHost, s));
    HIPCHK(hipMemcpyAsync(&he, err, sizeof(int), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (he) throw Error(SCR_E_INVALID, "singular or missing diagonal block at AMG level " + std::to_string(l));
    double lam;
    std::memcpy(&lam, &hl, sizeof(double));
    L.lam = lam;
}

// backward error of the explicit inverse X of the dense A (one check solve; synchronises)
static double coarse_check(int64_t nc, const double* A, const double* X, Arena& ar, hipStream_t s) {
    double* y = ar.make<double>(nc);
    double* rr = ar.make<double>(nc);
    double* ra = ar.make<double>(nc);
    double* eta = ar.make<double>(1);
    coarse_check_y_k<<<cdiv(nc, 4), 256, 0, s>>>(nc, X, y);
    coarse_check_r_k<<<cdiv(nc, 4), 256, 0, s>>>(nc, A, y, rr, ra);
    coarse_check_eta_k<<<1, 256, 0, s>>>(nc, rr, ra, y, eta);
    check_launch("coarse check");
    double he = 0.0;
    HIPCHK(hipMemcpyAsync(&he, eta, sizeof(double), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    ar.free(y); ar.free(rr); ar.free(ra); ar.free(eta);
    return he;
}

// largest accepted backward error of the fast inverse (a stable inverse gives about n * 1e-16)
constexpr double COARSE_ETA_MAX = 1e-10;

// coarsest level: explicit inverse by Gauss-Jordan exchange steps, in order (fast panels), or
// with partial pivoting when the fast inverse fails its check.  H.coarse_pivoted records which.
void coarse_inverse(Hierarchy& H, int* err, Arena& ar, hipStream_t s) {
    LevelSetup& C = H.L.back();
    int64_t nc = C.A.nr * C.b;
    H.ncoarse = nc;
    if (nc > 8192) throw Error(SCR_E_INVALID, "coarsest AMG level too large for a direct solve (" + std::to_string(nc) + ")");
    if (H.cinv) { ar.free(H.cinv); H.cinv = nullptr; }
    double* A = ar.make<double>(nc * nc + 1);      // the dense coarsest matrix, kept for the check
    double* M0 = ar.make<double>(nc * nc + 1);
    double* M1 = ar.make<double>(nc * nc + 1);
    zero_dev(A, nc * nc * sizeof(double), s);
    if (C.A.nr) densify_k<<<cdiv(C.A.nr, 256), 256, 0, s>>>(C.A.nr, C.b, C.A.rp, C.A.ci, C.A.v, A, nc);
    copy_dev(M0, A, nc * nc * sizeof(double), s);
    double* T = ar.make<double>(nc * GJ_P + 1);
    double* W = ar.make<double>(GJ_P * GJ_P);
    for (int64_t k0 = 0; k0 < nc; k0 += GJ_P) {
        int np = (int)std::min<int64_t>(GJ_P, nc - k0);
        gj_panel_t_k<<<cdiv(nc, 256), 256, 0, s>>>(nc, k0, np, M0, T, W);
        gj_panel_apply_k<<<cdiv(nc * nc, 256), 256, 0, s>>>(nc, k0, np, M0, T, W, M1);
        std::swap(M0, M1);
    }
    check_launch("coarse inverse");
    ar.free(T);
    ar.free(W);
    H.coarse_eta = nc ? coarse_check(nc, A, M0, ar, s) : 0.0;
    H.coarse_pivoted = false;
    if (!(H.coarse_eta <= COARSE_ETA_MAX)) {
        // partial pivoting, one exchange step per pivot
        int32_t* perm = ar.make<int32_t>(nc);
        zero_dev(err, sizeof(int), s);
        copy_dev(M0, A, nc * nc * sizeof(double), s);
        for (int64_t k = 0; k < nc; ++k) {
            gjp_pivot_k<<<1, 256, 0, s>>>(nc, k, M0, perm, err);
            gjp_exchange_k<<<cdiv(nc * nc, 256), 256, 0, s>>>(nc, k, M0, M1);
            std::swap(M0, M1);
        }
        gjp_unpermute_k<<<cdiv(nc, 256), 256, 0, s>>>(nc, perm, M0);
        check_launch("coarse inverse (pivoted)");
        int he = 0;
        HIPCHK(hipMemcpyAsync(&he, err, sizeof(int), hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        ar.free(perm);
        if (he) throw Error(SCR_E_INVALID, "coarsest AMG matrix is singular");
        H.coarse_eta = coarse_check(nc, A, M0, ar, s);
        H.coarse_pivoted = true;
    }
    zero_dev(err, sizeof(int), s);
    if (nc) finite_k<<<cdiv(nc * nc, 256), 256, 0, s>>>(nc * nc, M0, err);
    int he = 0;
    HIPCHK(hipMemcpyAsync(&he, err, sizeof(int), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (he) throw Error(SCR_E_INVALID, "coarsest AMG matrix is singular");
    ar.free(M1);
    ar.free(A);
    H.cinv = M0;
}

std::unique_ptr<Hierarchy> build_hierarchy(const DBsr& A0, const double* B0, int k, const scr_amg_opts& o, Arena& ar,
                                           hipStream_t s, Profiler* prof, bool three) {
    if (three && A0.br != 1) throw Error(SCR_E_INVALID, "three-column V-cycles need a scalar matrix");
    if (o.amg_type == SCR_AMG_CLASSICAL) return build_classical(A0, o, ar, s, three);
    std::unique_ptr<Hierarchy> H;
    HierT<double>* hd = nullptr;
    HierT<float>* hf = nullptr;
    if (o.precision != SCR_FP64) { hf = new HierT<float>(); hf->prof = prof; H.reset(hf); }
    else { hd = new HierT<double>(); hd->prof = prof; H.reset(hd); }
    H->opts = o;
    H->three = three;
    int* err = ar.make<int>(1);
    unsigned long long* lamd = ar.make<unsigned long long>(1);
    // level 0: copy of A0 and B0
    {
        LevelSetup l0;
        l0.A = bsr_alloc(A0.nr, A0.nc, A0.br, A0.bc, A0.nnzb, ar);
        l0.A.wmax = A0.wmax;
        copy_dev(l0.A.rp, A0.rp, (A0.nr + 1) * sizeof(int32_t), s);
        copy_dev(l0.A.ci, A0.ci, A0.nnzb * sizeof(int32_t), s);
        copy_dev(l0.A.v, A0.v, A0.nnzb * A0.br * A0.bc * sizeof(double), s);
        l0.b = A0.br; l0.k = k;
        l0.B = ar.make<double>(A0.nr * A0.br * k);
        copy_dev(l0.B, B0, A0.nr * A0.br * k * sizeof(double), s);
        H->L.push_back(l0);
    }
    for (int l = 0;; ++l) {
        LevelSetup& L = H->L[l];
        const int64_t nr = L.A.nr;
        const int b = L.b, bb = b * b;
        const int64_t n = nr * b;
        const int64_t g = cdiv(nr, 256);
        // D^-1 and lambda_hat (every level but the coarsest needs them; computed here for all)
        L.Dinv = ar.make<double>(nr * bb);
        level_diag(L, l, err, lamd, s);
        int he = 0;
        if (n <= o.coarse_max || l + 1 >= o.max_levels || l + 1 >= 16) break;
        // strength
        double* fd = ar.make<double>(nr);
        L.strong = ar.make<uint8_t>(L.A.nnzb > 0 ? L.A.nnzb : 1);
        uint8_t* iso = ar.make<uint8_t>(nr);
        double* f = ar.make<double>(L.A.nnzb > 0 ? L.A.nnzb : 1);
        if (L.A.nnzb > 0)
            block_f_k<<<(unsigned)cdiv(L.A.nnzb, WAVE), 256, (size_t)WAVE * (bb + 1) * sizeof(double), s>>>(L.A.nnzb, bb, L.A.v, f);
        fdiag_k<<<g, 256, 0, s>>>(nr, L.A.rp, L.A.ci, f, fd);
        double theta = std::ldexp(o.theta, -l);
        double th4 = ((theta * theta) * theta) * theta;
        // rows of 16 or more entries on average: one wavefront per row (same flags); of 8 or more for the
        // strength (1,030 -> 430 us at 324k rows of 15.6 blocks)
        const bool wide = L.A.nnzb >= 16 * nr;
        if (L.A.nnzb >= 8 * nr)
            strength_wave_k<<<cdiv(nr, 256 / WAVE), 256, 0, s>>>(nr, L.A.rp, L.A.ci, f, fd, th4, L.strong, iso);
        else strength_k<<<g, 256, 0, s>>>(nr, L.A.rp, L.A.ci, f, fd, th4, L.strong, iso);
        check_launch("strength");
        ar.free(fd);
        ar.free(f);
        // MIS-2 rounds
        uint64_t* st = ar.make<uint64_t>(nr);
        uint64_t* m1 = ar.make<uint64_t>(nr);
        uint64_t* m2 = ar.make<uint64_t>(nr);
        int* und = ar.make<int>(1);
        mis_init_k<<<g, 256, 0, s>>>(nr, iso, o.seed, l, st);
        for (int round = 0;; ++round) {
            if (round > 100000) throw Error(SCR_E_HIP, "MIS-2 did not terminate");
            zero_dev(und, sizeof(int), s);
            // the second sweep only for the undecided nodes: the decision reads nothing else of m2
            if (wide) {
                mis_max_wave_k<<<cdiv(nr, 256 / WAVE), 256, 0, s>>>(nr, L.A.rp, L.A.ci, L.strong, st, m1, nullptr);
                mis_max_wave_k<<<cdiv(nr, 256 / WAVE), 256, 0, s>>>(nr, L.A.rp, L.A.ci, L.strong, m1, m2, st);
            } else {
                mis_max_k<<<g, 256, 0, s>>>(nr, L.A.rp, L.A.ci, L.strong, st, m1, nullptr);
                mis_max_k<<<g, 256, 0, s>>>(nr, L.A.rp, L.A.ci, L.strong, m1, m2, st);
            }
            mis_decide_k<<<g, 256, 0, s>>>(nr, st, m2, und);
            check_launch("mis2");
            int hu = 0;
            HIPCHK(hipMemcpyAsync(&hu, und, sizeof(int), hipMemcpyDeviceToHost, s));
            HIPCHK(hipStreamSynchronize(s));
            if (hu == 0) break;
        }
        ar.free(m1); ar.free(m2); ar.free(und);
        // aggregates
        int32_t* isroot = ar.make<int32_t>(nr + 1);
        int32_t* rid = ar.make<int32_t>(nr + 1);
        root_flag_k<<<g, 256, 0, s>>>(nr, st, isroot);
        int64_t na = scan_i32(isroot, rid, nr, ar, s);
        ar.free(isroot);
        L.agg = ar.make<int32_t>(nr);
        uint8_t* step1 = ar.make<uint8_t>(nr);
        agg_roots_k<<<g, 256, 0, s>>>(nr, st, rid, L.agg);
        agg_dist1_k<<<cdiv(nr, 256 / WAVE), 256, 0, s>>>(nr, L.A.rp, L.A.ci, L.strong, iso, st, rid, L.agg, step1);
        zero_dev(err, sizeof(int), s);
        agg_dist2_k<<<cdiv(nr, 256 / WAVE), 256, 0, s>>>(nr, L.A.rp, L.A.ci, L.strong, iso, step1, o.seed, l, L.agg, err);
        check_launch("aggregate");
        HIPCHK(hipMemcpyAsync(&he, err, sizeof(int), hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        ar.free(step1); ar.free(rid); ar.free(st); ar.free(iso);
        if (he) throw Error(SCR_E_HIP, "aggregation left a node unassigned");
        if (na <= 0 || (double)(na * L.k) > o.max_coarse_ratio * (double)n) {
            ar.free(L.agg); L.agg = nullptr;
            ar.free(L.strong); L.strong = nullptr;
            break;
        }
        L.nagg = na;
        const int kk = L.k;
        // members of each aggregate, ascending
        int32_t* mcnt = ar.make<int32_t>(na + 1);
        zero_dev(mcnt, (na + 1) * sizeof(int32_t), s);
        agg_count_k<<<g, 256, 0, s>>>(nr, L.agg, mcnt);
        int32_t* mrp = ar.make<int32_t>(na + 1);
        int64_t nmem = scan_i32(mcnt, mrp, na, ar, s);
        zero_dev(mcnt, (na + 1) * sizeof(int32_t), s);
        int32_t* mem = ar.make<int32_t>(nmem + 1);
        int32_t* unsorted = ar.make<int32_t>(nmem + 1);
        agg_fill_k<<<g, 256, 0, s>>>(nr, L.agg, mrp, mcnt, unsorted);
        if (nmem > 0) agg_sort_k<<<cdiv(nmem, 256), 256, 0, s>>>(nmem, L.agg, mrp, unsorted, mem);
        ar.free(unsorted);
        // tentative prolongator and coarse near-null space
        double* Q = ar.make<double>(nr * b * kk);
        zero_dev(Q, nr * b * kk * sizeof(double), s);
        LevelSetup N;
        N.b = kk; N.k = kk;
        N.B = ar.make<double>(na * kk * kk);
        L.dead = ar.make<uint8_t>(na * kk);
        zero_dev(L.dead, na * kk, s);
        tentative_run(na, b, kk, mrp, mem, L.B, Q, N.B, L.dead, ar, s);
        ar.free(mcnt);
        L.mrp = mrp;
        L.mem = mem;
        DBsr Pt;
        Pt.nr = nr; Pt.nc = na; Pt.br = b; Pt.bc = kk;
        Pt.rp = ar.make<int32_t>(nr + 1);
        int32_t* pc = ar.make<int32_t>(nr + 1);
        ptent_cnt_k<<<g, 256, 0, s>>>(nr, L.agg, pc);
        Pt.nnzb = scan_i32(pc, Pt.rp, nr, ar, s);
        ar.free(pc);
        Pt.ci = ar.make<int32_t>(Pt.nnzb + 1);
        Pt.v = ar.make<double>((Pt.nnzb + 1) * b * kk);
        ptent_fill_k<<<g, 256, 0, s>>>(nr, b * kk, L.agg, Pt.rp, Q, Pt.ci, Pt.v);
        check_launch("ptent");
        // smoothed prolongator on the pattern of A * P_tent (aggregated rows only)
        uint8_t* rowmask = ar.make<uint8_t>(nr);
        rowmask_k<<<g, 256, 0, s>>>(nr, L.agg, rowmask);
        DBsr P = spgemm(L.A, Pt, rowmask, ar, s);
        ar.free(rowmask);
        bsr_release(Pt, ar);
        double omega = 4.0 / (3.0 * L.lam);
        if (b == 1 && kk == 1) smooth_p_k<1, 1><<<g, 256, 0, s>>>(nr, P.rp, P.ci, P.v, L.Dinv, L.agg, Q, omega);
        else if (b == 3 && kk == 6) smooth_p_k<3, 6><<<g, 256, 0, s>>>(nr, P.rp, P.ci, P.v, L.Dinv, L.agg, Q, omega);
        else if (b == 6 && kk == 6) smooth_p_k<6, 6><<<g, 256, 0, s>>>(nr, P.rp, P.ci, P.v, L.Dinv, L.agg, Q, omega);
        else throw Error(SCR_E_UNIMPLEMENTED, "prolongator block shape");
        check_launch("smooth_p");
        ar.free(Q);
        L.P = P;
        L.R = transpose(L.P, ar, s, &L.rsrc);
        // Galerkin product A_c = R (A P) on structural patterns; dead coarse dofs get a unit diagonal
        DBsr AP = spgemm(L.A, L.P, nullptr, ar, s);
        N.A = spgemm(L.R, AP, nullptr, ar, s);
        ar.free(AP.v);
        AP.v = nullptr;
        L.AP = AP;
        if (na) dead_diag_k<<<cdiv(na, 256), 256, 0, s>>>(na, kk, N.A.rp, N.A.ci, N.A.v, L.dead);
        check_launch("dead_diag");
        H->L.push_back(N);   // invalidates L
    }
    coarse_inverse(*H, err, ar, s);
    ar.free(err);
    ar.free(lamd);
    if (hf) hf->prepare(ar, s);
    else hd->prepare(ar, s);
    HIPCHK(hipStreamSynchronize(s));
    return H;
}

void update_hierarchy(Hierarchy& H, const double* vals0, const double* B0, Arena& ar, hipStream_t s) {
    if (H.opts.amg_type == SCR_AMG_CLASSICAL) {
        update_classical(H, vals0, ar, s);
        return;
    }
    int* err = ar.make<int>(1);
    unsigned long long* lamd = ar.make<unsigned long long>(1);
    LevelSetup& L0 = H.L[0];
    copy_dev(L0.A.v, vals0, L0.A.nnzb * L0.b * L0.b * sizeof(double), s);
    if (B0) copy_dev(L0.B, B0, L0.A.nr * L0.b * L0.k * sizeof(double), s);
    for (size_t l = 0; l < H.L.size(); ++l) {
        LevelSetup& L = H.L[l];
        level_diag(L, (int)l, err, lamd, s);
        if (l + 1 == H.L.size()) break;
        LevelSetup& N = H.L[l + 1];
        const int64_t nr = L.A.nr, na = L.nagg;
        const int b = L.b, kk = L.k;
        const int64_t g = cdiv(nr, 256);
        // tentative prolongator, coarse near-null space and dead dofs from the kept aggregates
        double* Q = ar.make<double>(nr * b * kk);
        zero_dev(Q, nr * b * kk * sizeof(double), s);
        zero_dev(L.dead, na * kk, s);
        tentative_run(na, b, kk, L.mrp, L.mem, L.B, Q, N.B, L.dead, ar, s);
        DBsr Pt;
        Pt.nr = nr; Pt.nc = na; Pt.br = b; Pt.bc = kk;
        Pt.rp = ar.make<int32_t>(nr + 1);
        int32_t* pc = ar.make<int32_t>(nr + 1);
        ptent_cnt_k<<<g, 256, 0, s>>>(nr, L.agg, pc);
        Pt.nnzb = scan_i32(pc, Pt.rp, nr, ar, s);
        ar.free(pc);
        Pt.ci = ar.make<int32_t>(Pt.nnzb + 1);
        Pt.v = ar.make<double>((Pt.nnzb + 1) * b * kk);
        ptent_fill_k<<<g, 256, 0, s>>>(nr, b * kk, L.agg, Pt.rp, Q, Pt.ci, Pt.v);
        check_launch("ptent");
        // smoothed prolongator into its kept pattern
        spgemm_numeric(L.A, Pt, L.P, s);
        bsr_release(Pt, ar);
        double omega = 4.0 / (3.0 * L.lam);
        if (b == 1 && kk == 1) smooth_p_k<1, 1><<<g, 256, 0, s>>>(nr, L.P.rp, L.P.ci, L.P.v, L.Dinv, L.agg, Q, omega);
        else if (b == 3 && kk == 6) smooth_p_k<3, 6><<<g, 256, 0, s>>>(nr, L.P.rp, L.P.ci, L.P.v, L.Dinv, L.agg, Q, omega);
        else if (b == 6 && kk == 6) smooth_p_k<6, 6><<<g, 256, 0, s>>>(nr, L.P.rp, L.P.ci, L.P.v, L.Dinv, L.agg, Q, omega);
        else throw Error(SCR_E_UNIMPLEMENTED, "prolongator block shape");
        check_launch("smooth_p");
        ar.free(Q);
        transpose_values(L.P, L.R, L.rsrc, s);
        // Galerkin product into the kept patterns of A P and A_{l+1}
        L.AP.v = ar.make<double>((L.AP.nnzb > 0 ? L.AP.nnzb : 1) * L.AP.br * L.AP.bc);
        spgemm_numeric(L.A, L.P, L.AP, s);
        spgemm_numeric(L.R, L.AP, N.A, s);
        ar.free(L.AP.v);
        L.AP.v = nullptr;
        if (na) dead_diag_k<<<cdiv(na, 256), 256, 0, s>>>(na, kk, N.A.rp, N.A.ci, N.A.v, L.dead);
        check_launch("dead_diag");
    }
    coarse_inverse(H, err, ar, s);
    ar.free(err);
    ar.free(lamd);
    H.refresh(ar, s);
    HIPCHK(hipStreamSynchronize(s));
}

}  // namespace scr
