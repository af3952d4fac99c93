// Row analysis, binning, row-pointer scan and small utility kernels.
//
// The symbolic phase of section 2.2.1 needs each row's size before C can be
// allocated.  These kernels produce what the accumulator kernels consume:
//   - per B row: length and column range (one pass over B's structure);
//   - per A row: products (the row's FLOP count, which the paper uses to pick
//     a parallelisation method), column range of C's row, largest referenced
//     B row, and the row's accumulator class;
//   - the permutation that groups rows of one class together;
//   - C's row pointer as the exclusive prefix sum of the row counts (section
//     2.2.1), single pass with decoupled look-back, plus the numeric-phase
//     class of every row.
// Index validity is checked in the same passes that read the indices.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <climits>
#include <cstddef>

#include "spg_internal.h"

namespace spg {

namespace {

constexpr int ROW_LANES = 8;        // lanes per B row when compressing B
constexpr int AN_LANES = 4;         // lanes per row in the row analysis passes
constexpr int AN_LOADS = 8;         // independent entry loads per lane and round trip there
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;

__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_fill_u8(uint8_t* p, uint8_t v, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_zero(uint4* p, int64_t n16) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n16; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0, 0, 0, 0);
}

__global__ __launch_bounds__(256) void k_publish(const uint32_t* __restrict__ ctl, uint32_t* host, uint32_t seq) {
    constexpr int WORDS = offsetof(Control, seq) / 4;
    for (int i = threadIdx.x; i < WORDS; i += 256)
        __hip_atomic_store(&host[i], ctl[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(&host[WORDS], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Every vector memory access of this thread has completed.
__device__ inline void wait_mem() { __builtin_amdgcn_s_waitcnt(0); }

// Adds the workgroup's counters (acc, NCOUNT in LDS, complete and
// synchronised) to its shard.
__device__ inline void add_counts(const unsigned long long* acc, Shard* shards) {
    const int t = threadIdx.x, s = blockIdx.x % NSHARD;
    if (t < NCOUNT && acc[t]) {
        if (t < CNT_MAX) atomicAdd(&shards[s].f[t], acc[t]);
        else atomicMax(&shards[s].f[t], acc[t]);
    }
}

// After add_counts and this thread's other stores: true in every thread of
// the workgroup that finishes last, whose acc then holds the totals of the
// whole grid.
__device__ inline bool sum_counts(unsigned long long* acc, Shard* shards, int32_t* top, int* sh) {
    const int t = threadIdx.x, s = blockIdx.x % NSHARD;
    wait_mem();  // the counters are out before the workgroup counts as done
    __syncthreads();
    if (t == 0) {
        *sh = 0;
        const int members = ((int)gridDim.x - s + NSHARD - 1) / NSHARD;
        if (members == 1 || atomicAdd(&shards[s].done, 1) == members - 1) {
            const int used = (int)gridDim.x < NSHARD ? (int)gridDim.x : NSHARD;
            *sh = atomicAdd(top, 1) == used - 1;
        }
    }
    __syncthreads();
    if (!*sh) return false;
    if (t < NCOUNT) {
        unsigned long long v[NSHARD], r = 0;
#pragma unroll
        for (int u = 0; u < NSHARD; ++u)
            v[u] = __hip_atomic_load(&shards[u].f[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int u = 0; u < NSHARD; ++u) r = t < CNT_MAX ? r + v[u] : max(r, v[u]);
        acc[t] = r;
    }
    __syncthreads();
    return true;
}

// Grids of at most this many workgroups add straight to the control block: so
// few do not queue there, and the last workgroup's round trips are saved (3 us
// of a pass over 4096 rows).
constexpr unsigned DIRECT_GRID = 64;
__device__ inline void add_to(int32_t* p, unsigned long long v) {
    if (v) atomicAdd(p, (int32_t)v);
}
__device__ inline void add_to(int64_t* p, unsigned long long v) {
    if (v) atomicAdd((unsigned long long*)p, v);
}
__device__ inline void max_to(int64_t* p, unsigned long long v) {
    if (v) atomicMax((unsigned long long*)p, v);
}

// Rows of the two analysis passes are dealt to the workgroups CHUNK
// consecutive rows at a time, chunk c to workgroup c mod grid, and a row of
// more than long_row entries may be walked by a whole wavefront, not by its few
// lanes (by_wavefront, for A): the hub rows of a power-law matrix (low row
// indices) would otherwise sit in a few workgroups that walk them in hundreds
// of dependent round trips while the rest of the grid is done (R-MAT scale 18:
// 0.67 and 0.75 ms for the two passes, nearly all of it that).
// Lanes per row L: with at least SHORT_MIN_ROWS rows of at most SHORT_ROWS
// entries on average every row gets one lane, which takes eight of its
// entries at a time with two 16-byte loads: several lanes per row leave most
// of them idle there while every instruction is paid for (2.1M rows of 1
// entry of B: 94 us with 8 lanes, 26 with one; of 7 entries of A: 113 us with
// 4 lanes, 72 with one).  Longer rows read better coalesced with several (1M
// rows of 27 entries of B: 138 us with one lane, 102 with eight), and below
// SHORT_MIN_ROWS the chip is not full (4096 rows of A: 9 us against 16).
constexpr int SHORT_ROWS = 8;
constexpr int SHORT_MIN_ROWS = 1 << 17;
// (B rows, eight lanes each: 20 thousand rows of 200 entries took 45 us in all
// with rows of more than 128 by a wavefront, 36 so)
template <int L>
constexpr int long_row() {
    return L == 8 ? 256 : 64;
}
// Whether a row of `len` entries of A goes to a wavefront: its own lanes take
// PER of its entries a round trip, beside the other rows of their wavefront; a
// wavefront takes 512 of one row.  So the long rows go where all of them one
// after another take fewer round trips than the longest does with its own
// lanes: a hub row among short ones does, rows that are all somewhat long do
// not (20 thousand rows of 128 entries: 66 us with every one of them by a
// wavefront, 22 so).  Past ALWAYS_LONG entries they all go: their lanes read
// from as many far places a round trip, which costs several times a
// wavefront's 2 KB in a row (200 rows of 20000 entries, one behind another:
// the analysis 0.95 ms with their own lanes, 0.27 so; 2000 rows of 2000: 0.13
// and 0.07).
constexpr int ALWAYS_LONG = 512;
template <int L, int PER>
__device__ inline bool by_wavefront(int len) {
    const bool is_long = len > long_row<L>();
    if (!__any(is_long)) return false;
    int trips = is_long && threadIdx.x % L == 0 ? (len - 1) / 512 + 1 : 0, longest = is_long ? len : 0;
    for (int d = 32; d > 0; d >>= 1) {
        trips += __shfl_xor(trips, d, 64);
        longest = max(longest, __shfl_xor(longest, d, 64));
    }
    return is_long && (len > ALWAYS_LONG || trips * PER < longest);
}

// A chunk is a wavefront's rows: neighbouring rows share what they gather and
// the cache lines that they write.  One row where a single pass covers all
// (m up to 131072): everything is in cache then, and the hub rows spread best
// (R-MAT scale 13: 51 us with chunks of 16 rows, 21 so).
// The row of thread group `g` of the workgroup's 256 / L in pass `pass`:
template <int L>
__device__ inline int64_t dealt_row(int64_t pass, int64_t passes, int g) {
    const int C = passes == 1 ? 1 : 64 / L, per = 256 / L / C;
    // (rotated from one round to the next: hub rows have few index bits set,
    // and a power-of-two stride would deal them all to the same workgroups)
    const int64_t round = pass * per + g / C;
    const int64_t chunk = round * gridDim.x + (uint32_t)(blockIdx.x + round * 61) % gridDim.x;
    return chunk * C + g % C;
}

// Reductions over aligned groups of AN_LANES = 4 lanes with DPP: swaps of
// neighbours and of pairs inside each quad, after which every lane of the
// group holds the result.  No LDS.
static_assert(AN_LANES == 4, "the row reductions below cover one quad");
template <typename Op>
__device__ inline int rowq_reduce(int v, Op op) {
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0xb1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0x4e, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
    return v;
}
__device__ inline int rowq_sum(int v) { return rowq_reduce(v, [](int x, int y) { return x + y; }); }
__device__ inline int rowq_min(int v) { return rowq_reduce(v, [](int x, int y) { return min(x, y); }); }
__device__ inline int rowq_max(int v) { return rowq_reduce(v, [](int x, int y) { return max(x, y); }); }
__device__ inline int rowq_or(int v) { return rowq_reduce(v, [](int x, int y) { return x | y; }); }
template <int CTRL>
__device__ inline int64_t dpp64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)((uint64_t)v >> 32), CTRL, 0xf, 0xf, false);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ inline int64_t rowq_sum64(int64_t v) {
    v += dpp64<0xb1>(v);
    v += dpp64<0x4e>(v);
    return v;
}

__device__ inline float log2p1(int64_t v) { return log2f(1.0f + (float)v); }

// A rows: products, column range, largest B row; symbolic class from an upper
// bound on the row's occupied blocks (binning 0: its products, 2: the
// compressed-B runs it reads, 3: the exact count of a previous run) or
// features only (binning 1, learned: classified by k_mlp_classify).
struct RowSums {
    int64_t ub = 0, rs = 0;  // products; compressed-B runs (a bound on occupied blocks)
    int mx = 0, cmin = INT_MAX, cmax = -1, bad = 0, diag = 0;
};

// Indices of entries are stepped as unsigned numbers in the walks below: a
// row may end at 2^31 - 1, and the step behind its last entries then passes
// the int32 range.

// Entries q..q+7 of an index array of `total` (those past its end: the last
// one), with two 16-byte loads (dword-aligned) unless they reach past it.
struct __attribute__((packed, aligned(4))) I4 {
    int x, y, z, w;
};
__device__ inline void load8(int* c, const int32_t* __restrict__ p, uint32_t q, int64_t total) {
    if (q + (int64_t)8 <= total) {
        const I4 a = *reinterpret_cast<const I4*>(p + q), b = *reinterpret_cast<const I4*>(p + q + 4);
        c[0] = a.x, c[1] = a.y, c[2] = a.z, c[3] = a.w;
        c[4] = b.x, c[5] = b.y, c[6] = b.z, c[7] = b.w;
    } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) c[u] = p[min((int64_t)q + u, total - 1)];
    }
}

// U entries of a row at p0, p0 + step, ... per lane (STEP1: eight at p0 on): independent index loads,
// then their gathers.  Every load is unconditional (indices clamped into the
// row, and to B's first row for entries that are past the row's end or
// invalid; n > 0 whenever the row has an entry that can be valid) and its
// value is discarded afterwards where it does not count: a load under a
// condition with a default in the other branch makes the compiler wait for
// it before the next one is issued.
template <int U, bool STEP1 = false>
__device__ inline void row_entries(RowSums& r, const int32_t* __restrict__ aci, int64_t annz,
                                   const int4* __restrict__ binfo, int32_t n, int64_t row, uint32_t p0, int step,
                                   uint32_t e) {
    int jj[U];
    if constexpr (STEP1) {
        static_assert(U == 8, "load8");
        load8(jj, aci, p0, annz);
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) jj[u] = aci[min(p0 + u * step, e - 1)];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool in_row = p0 + u * step < e;
        if (in_row && (jj[u] < 0 || jj[u] >= n)) r.bad = ERR_A_COL;
        if (!in_row || jj[u] < 0 || jj[u] >= n) jj[u] = -1;
        r.diag |= jj[u] == row;  // a stored diagonal entry (square A)
    }
    if (n <= 0) return;  // every entry is invalid: nothing to gather
    int4 bb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) bb[u] = binfo[max(jj[u], 0)];
    int ub = 0, rs = 0;  // U rows of B: below 2^34 in all, so 64 bits only where a row is that long
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (jj[u] < 0) continue;
        if (bb[u].x >= 1 << 26) {
            r.ub += bb[u].x, r.rs += bb[u].w;
        } else {
            ub += bb[u].x, rs += bb[u].w;
        }
        r.mx = max(r.mx, bb[u].x);
        r.cmin = min(r.cmin, bb[u].y);
        r.cmax = max(r.cmax, bb[u].z);
    }
    r.ub += ub, r.rs += rs;
}

template <typename T, typename Op>
__device__ inline T wave_reduce(T v, Op op) {
    for (int d = 32; d > 0; d >>= 1) v = op(v, (T)__shfl_xor(v, d, 64));
    return v;
}

template <int L>
__global__ __launch_bounds__(256) void k_a_rowinfo(int32_t m, int32_t n, const int32_t* __restrict__ arp,
                                                   const int32_t* __restrict__ aci, int64_t annz,
                                                   const int4* __restrict__ binfo, RowInfo* __restrict__ rinfo,
                                                   float* __restrict__ feats, ClassCfg cfg, int binning,
                                                   uint8_t* __restrict__ sym_cls, int32_t* __restrict__ row_nnz,
                                                   int32_t* __restrict__ row_blocks, int32_t* __restrict__ lofs,
                                                   Shard* shards, Control* ctl) {
    constexpr int GROUPS = 256 / L;
    static_assert(L == 1 || L == AN_LANES, "one lane, or the quad that the reductions cover");
    __shared__ unsigned long long acc[NCOUNT];
    __shared__ int32_t longs[GROUPS];
    __shared__ int nlong[2], sh;  // by pass parity: a wavefront may be a pass ahead of another's reading
    if (threadIdx.x < NCOUNT) acc[threadIdx.x] = 0;
    if (threadIdx.x < 2) nlong[threadIdx.x] = 0;
    __syncthreads();
    // a lane's counts over its rows, added to the workgroup's counters at the
    // end (classes once per run of equal ones): an LDS atomic per row and
    // counter is sixteen lanes of a wavefront on one address each time
    int n_empty = 0, n_nodiag = 0, cur = CLS_EMPTY, n_cur = 0;
    int64_t t_prod = 0;
    int32_t t_pmax = 0, t_words = 0, t_wglob = 0;
    auto finish_row = [&](int64_t row, int len, const RowSums& r) {
        const int64_t ub = r.bad ? 0 : r.ub;
        const int32_t ubc = ub > INT_MAX ? INT_MAX : (int32_t)ub;
        const int cmin = ub == 0 ? 0 : r.cmin, cmax = ub == 0 ? 0 : r.cmax;
        if (m == n && !r.diag) ++n_nodiag;
        rinfo[row] = make_int4(cmin, cmax, ubc, r.mx);
        if (feats) {
            feats[row * 3 + 0] = log2p1(len);
            feats[row * 3 + 1] = log2p1(ub);
            feats[row * 3 + 2] = log2p1(r.mx);
        }
        if (ub == 0) {
            row_nnz[row] = 0;
            row_blocks[row] = 0;
            sym_cls[row] = CLS_EMPTY;
            ++n_empty;
            return;
        }
        const int32_t words = row_words(cmin, cmax);
        lofs[row] = list_capacity(r.rs, words);
        t_words = max(t_words, words);
        t_prod += ub;
        t_pmax = max(t_pmax, ubc);
        if (binning != 1) {
            // binning 3 (ideal estimate): the row's exact occupied blocks, left in
            // row_blocks by a previous symbolic run of the same matrices
            const int64_t est = binning == 2 ? r.rs : binning == 3 ? (int64_t)row_blocks[row] : ub;
            const int cls = sym_class(ub, cmin, cmax, est, cfg, true);
            sym_cls[row] = (uint8_t)cls;
            if (cls != cur) {
                if (n_cur) atomicAdd(&acc[CNT_HIST + cur], (unsigned long long)n_cur);
                cur = cls, n_cur = 0;
            }
            ++n_cur;
            if (cls % NTIER == TIER_GLOBAL) t_wglob = max(t_wglob, words);
        }
    };
    const int lane = (int)(threadIdx.x % L), wl = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t passes = ((int64_t)m + (int64_t)gridDim.x * GROUPS - 1) / ((int64_t)gridDim.x * GROUPS);
    for (int64_t pass = 0; pass < passes; ++pass) {
        const int64_t row = dealt_row<L>(pass, passes, threadIdx.x / L);
        RowSums r;
        int32_t s = 0, e = 0;
        if (row < m) {
            s = arp[row], e = arp[row + 1];
            if (s < 0 || e < s || (int64_t)e > annz || (row == 0 && s != 0) || (row == m - 1 && (int64_t)e != annz))
                r.bad = ERR_A_ROWPTR, s = e = 0;
        }
        const int len = e - s;
        const bool put_off = by_wavefront<L, L == 1 ? 8 : AN_LOADS * L>(len);
        if (put_off) {
            if (lane == 0) longs[atomicAdd(&nlong[pass & 1], 1)] = (int32_t)row;
            e = s;
        }
        // as many loads per round trip as the wavefront's longest row needs
        if constexpr (L == 1) {
            for (uint32_t p0 = s; p0 < (uint32_t)e; p0 += 8) row_entries<8, true>(r, aci, annz, binfo, n, row, p0, 1, e);
        } else if (!__any(e - s > 2 * L)) {
            if (s < e) row_entries<2>(r, aci, annz, binfo, n, row, (uint32_t)s + lane, L, e);
        } else {
            for (uint32_t p0 = (uint32_t)s + lane; p0 < (uint32_t)e; p0 += AN_LOADS * L)
                row_entries<AN_LOADS>(r, aci, annz, binfo, n, row, p0, L, e);
        }
        if (r.bad) atomicOr(&ctl->err, r.bad);
        if constexpr (L > 1) {
            r.ub = rowq_sum64(r.ub);
            r.rs = rowq_sum64(r.rs);
            r.mx = rowq_max(r.mx);
            r.cmin = rowq_min(r.cmin);
            r.cmax = rowq_max(r.cmax);
            r.bad = rowq_or(r.bad);
            r.diag = rowq_or(r.diag);
        }
        if (row < m && lane == 0 && !put_off) finish_row(row, len, r);
        __syncthreads();
        const int nl = nlong[pass & 1];
        if (nl > 0) {  // uniform; the pass's long rows, a wavefront each
            for (int l = wv; l < nl; l += 4) {
                const int64_t lrow = longs[l];
                const int32_t ls = arp[lrow], le = arp[lrow + 1];
                RowSums q;
                for (uint32_t p0 = (uint32_t)ls + wl; p0 < (uint32_t)le; p0 += AN_LOADS * 64)
                    row_entries<AN_LOADS>(q, aci, annz, binfo, n, lrow, p0, 64, le);
                auto add = [](auto x, auto y) { return x + y; };
                auto hi = [](auto x, auto y) { return x > y ? x : y; };
                if (q.bad) atomicOr(&ctl->err, q.bad);
                q.ub = wave_reduce((long long)q.ub, add);
                q.rs = wave_reduce((long long)q.rs, add);
                q.mx = wave_reduce(q.mx, hi);
                q.cmin = wave_reduce(q.cmin, [](auto x, auto y) { return x < y ? x : y; });
                q.cmax = wave_reduce(q.cmax, hi);
                q.bad = __any(q.bad) ? ERR_A_COL : 0;
                q.diag = __any(q.diag);
                if (wl == 0) finish_row(lrow, le - ls, q);
            }
            __syncthreads();
            if (threadIdx.x == 0) nlong[pass & 1] = 0;
            __syncthreads();
        }
    }
    if (n_cur) atomicAdd(&acc[CNT_HIST + cur], (unsigned long long)n_cur);
    if (n_empty) atomicAdd(&acc[CNT_ROWS], (unsigned long long)n_empty);
    if (n_nodiag) atomicAdd(&acc[CNT_NODIAG], (unsigned long long)n_nodiag);
    if (t_prod) {
        atomicAdd(&acc[CNT_PRODUCTS], (unsigned long long)t_prod);
        atomicMax(&acc[CNT_MAXPROD], (unsigned long long)t_pmax);
        atomicMax(&acc[CNT_WORDS], (unsigned long long)t_words);
        if (t_wglob) atomicMax(&acc[CNT_WGLOB], (unsigned long long)t_wglob);
    }
    __syncthreads();
    // (one workgroup left, or each of a few: the totals into the control block)
    if (gridDim.x > DIRECT_GRID) {
        add_counts(acc, shards);
        if (!sum_counts(acc, shards, &ctl->done[0], &sh)) return;
    }
    if (threadIdx.x < NCLS) add_to(&ctl->sym_hist[threadIdx.x], acc[CNT_HIST + threadIdx.x]);
    if (threadIdx.x == 64) {
        add_to(&ctl->empty_rows, acc[CNT_ROWS]);
        add_to(&ctl->a_missing_diag, acc[CNT_NODIAG]);
        add_to(&ctl->products, acc[CNT_PRODUCTS]);
        max_to(&ctl->max_words_all, acc[CNT_WORDS]);
        max_to(&ctl->max_products, acc[CNT_MAXPROD]);
        max_to(&ctl->max_words_sym_global, acc[CNT_WGLOB]);
    }
}

// Learned binning: the 3-32-32-1 network on each row's features (weights are
// wave-uniform, so they are read as scalars) sizes the symbolic table from
// 2^(y + margin) - 1 occupied blocks.  Consecutive rows with the same
// features (a stencil's interior) share one evaluation: per pass of 256 rows
// the first row of every run of equal features takes a slot (a block scan of
// the run starts, so slots follow row order), the slots are evaluated packed
// into as few wavefronts as possible, and every row reads its run's result.
__device__ inline float mlp_eval(const float* __restrict__ w, float x0, float x1, float x2) {
    const float* W1 = w;
    const float* b1 = w + 96;
    const float* W2 = w + 128;
    const float* b2 = w + 1152;
    const float* w3 = w + 1184;
    const float b3 = w[1216];
    float h1[32];
#pragma unroll
    for (int o = 0; o < 32; ++o) {
        float z = b1[o] + W1[o * 3] * x0 + W1[o * 3 + 1] * x1 + W1[o * 3 + 2] * x2;
        h1[o] = z > 0.f ? z : 0.f;
    }
    float y = b3;
#pragma unroll 4
    for (int o = 0; o < 32; ++o) {
        float z = b2[o];
#pragma unroll
        for (int i = 0; i < 32; ++i) z += W2[o * 32 + i] * h1[i];
        y += w3[o] * (z > 0.f ? z : 0.f);
    }
    return y;
}

__global__ __launch_bounds__(256) void k_mlp_classify(int32_t m, const float* __restrict__ feats,
                                                      const float* __restrict__ w, const RowInfo* __restrict__ rinfo,
                                                      ClassCfg cfg, float margin, uint8_t* __restrict__ sym_cls,
                                                      Control* ctl) {
    __shared__ int32_t hist[NCLS];
    __shared__ unsigned long long wmax_glob;
    __shared__ float xs[3][256];      // each row's features
    __shared__ float ys[256];         // the prediction of each run (by slot)
    __shared__ int32_t wsum[4];
    if (threadIdx.x < NCLS) hist[threadIdx.x] = 0;
    if (threadIdx.x == 0) wmax_glob = 0;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int cur = CLS_EMPTY, n_cur = 0;
    unsigned long long my_wglob = 0;
    // every thread runs the same number of passes (the barriers below)
    for (int64_t r0 = blockIdx.x * (int64_t)blockDim.x; r0 < m; r0 += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = r0 + tid;
        RowInfo ri = make_int4(0, 0, 0, 0);
        float x0 = 0.f, x1 = 0.f, x2 = 0.f;
        if (row < m) {
            ri = rinfo[row];
            x0 = feats[row * 3], x1 = feats[row * 3 + 1], x2 = feats[row * 3 + 2];
        }
        const bool valid = row < m && ri.z > 0;
        __syncthreads();  // the previous pass is done with xs and ys
        // an invalid row holds NaN, which equals nothing: the next valid row starts a run
        xs[0][tid] = valid ? x0 : __builtin_nanf(""), xs[1][tid] = x1, xs[2][tid] = x2;
        __syncthreads();
        const bool start = valid && (tid == 0 || xs[0][tid - 1] != x0 || xs[1][tid - 1] != x1 ||
                                     xs[2][tid - 1] != x2);
        // slots of the run starts in row order: block scan of the start flags
        int inc = start ? 1 : 0;
        for (int d = 1; d < 64; d <<= 1) {
            const int up = __shfl_up(inc, d, 64);
            if (lane >= d) inc += up;
        }
        if (lane == 63) wsum[wv] = inc;
        __syncthreads();  // every start test has read xs
        int before = 0, nslots = 0;
        for (int u = 0; u < 4; ++u) {
            if (u < wv) before += wsum[u];
            nslots += wsum[u];
        }
        // the run a valid row belongs to (its own start or the latest one before it)
        const int slot = before + inc - 1;
        if (start) xs[0][slot] = x0, xs[1][slot] = x1, xs[2][slot] = x2;  // slot <= tid
        __syncthreads();
        // the runs' features evaluated packed from thread 0
        if (tid < nslots) ys[tid] = mlp_eval(w, xs[0][tid], xs[1][tid], xs[2][tid]);
        __syncthreads();
        if (valid) {
            // a valid row that starts no run continues the run of a valid row before it
            const float y = ys[slot];
            float e = exp2f(fminf(y + margin, 40.f)) - 1.f;
            int64_t est = e < 1.f ? 1 : (int64_t)ceilf(e);
            int cls = sym_class(ri.z, ri.x, ri.y, est, cfg);
            sym_cls[row] = (uint8_t)cls;
            if (cls != cur) {
                if (n_cur) atomicAdd(&hist[cur], n_cur);
                cur = cls, n_cur = 0;
            }
            n_cur += 1;
            if (cls % NTIER == TIER_GLOBAL) my_wglob = max(my_wglob, (unsigned long long)row_words(ri.x, ri.y));
        }
    }
    if (n_cur) atomicAdd(&hist[cur], n_cur);
    if (my_wglob) atomicMax(&wmax_glob, my_wglob);
    __syncthreads();
    if (threadIdx.x < NCLS && hist[threadIdx.x]) atomicAdd(&ctl->sym_hist[threadIdx.x], hist[threadIdx.x]);
    if (threadIdx.x == 0 && wmax_glob) atomicMax((unsigned long long*)&ctl->max_words_sym_global, wmax_glob);
}

// Status word of a decoupled look-back: 2 flag bits over a 62-bit value.
constexpr uint64_t ST_AGG = 1ull << 62;
constexpr uint64_t ST_PRE = 2ull << 62;
constexpr uint64_t ST_VAL = (1ull << 62) - 1;

// Groups rows by class, each class in ascending row order up to the order
// inside a chunk: a workgroup takes chunks of 2048 consecutive rows by
// ticket, ranks each row inside its class with LDS atomics, and finds the
// chunk's range in every class from the counts of the chunks before it (a
// decoupled look-back per class over the chunks in ticket order), then
// writes the row ids there, with each row's descriptor {row, A start, A end,
// C start (or list offset)} beside it.  The order matters for speed: the
// row kernels take their rows in this order, so rows that share B rows run
// close together and, where row index and row size go together (R-MAT), the
// longest rows start first.  For the symbolic rows it also places the rows'
// lists: a scan of the chunk's capacities and one global atomic for the
// chunk's range.  state: the ticket, then a status word per chunk and class
// (scatter_state_bytes, all zero on entry).
constexpr int SCATTER_ITEMS = 8;
constexpr int SCATTER_CHUNK = 256 * SCATTER_ITEMS;
__global__ __launch_bounds__(256) void k_scatter(int32_t m, const uint8_t* __restrict__ cls, int merge,
                                                 const int32_t* __restrict__ hist, int32_t* __restrict__ state,
                                                 int32_t* __restrict__ perm, const int32_t* __restrict__ arp,
                                                 const int32_t* __restrict__ crp, int4* __restrict__ desc,
                                                 int32_t* __restrict__ lofs, Control* ctl, int64_t list_limit) {
    __shared__ int32_t cnt[NCLS];
    __shared__ int32_t base[NCLS];
    __shared__ int32_t off[NCLS];
    __shared__ int64_t wsum[4];
    __shared__ int64_t lbase;
    __shared__ uint8_t remap[NCLS];
    __shared__ int32_t merged[NCLS];
    __shared__ int32_t chunk_sh;
    int32_t* ticket = state;
    uint64_t* status = reinterpret_cast<uint64_t*>(state + 16);
    // the class merge, a lane per table mode
    if (threadIdx.x < 3) merge_classes_mode(hist, remap, merged, threadIdx.x, merge != 0);
    __syncthreads();
    if (threadIdx.x < 64) {
        // first slot of every class, in class order; symbolic rows tier-major
        // (a persistent launch takes a tier's three modes as one range) and
        // published by the first workgroup
        const int l = threadIdx.x;
        const int c = l < NCLS ? (lofs ? l % 3 * NTIER + l / 3 : l) : 0;
        const int32_t v = l < NCLS ? merged[c] : 0;
        int32_t x = v;
        for (int d = 1; d < 32; d <<= 1) {
            const int32_t y = __shfl_up(x, d, 64);
            if (l >= d) x += y;
        }
        if (l < NCLS) {
            off[c] = x - v;
            if (lofs && blockIdx.x == 0) ctl->sym_cnt[c] = v, ctl->sym_off[c] = x - v;
        }
    }
    const int64_t nchunks = ((int64_t)m + SCATTER_CHUNK - 1) / SCATTER_CHUNK;
    for (;;) {
        if (threadIdx.x < NCLS) cnt[threadIdx.x] = 0;
        if (threadIdx.x == 0) chunk_sh = atomicAdd(ticket, 1);
        __syncthreads();
        const int64_t chunk = chunk_sh;
        if (chunk >= nchunks) break;  // uniform
        const int64_t r0 = chunk * SCATTER_CHUNK;
        // the chunk's inputs first, as unconditional loads (a row past the end
        // reads the last row's, unused; arp has m + 1 entries): a load under a
        // condition would be waited for before the next one is issued
        uint8_t raw[SCATTER_ITEMS];
        int32_t lraw[SCATTER_ITEMS], a_lo[SCATTER_ITEMS], a_hi[SCATTER_ITEMS], cw[SCATTER_ITEMS];
#pragma unroll
        for (int t = 0; t < SCATTER_ITEMS; ++t) {
            const int64_t row = r0 + t * 256 + threadIdx.x;
            const int64_t rr = row < m ? row : m - 1;
            raw[t] = cls[rr];
            a_lo[t] = arp[rr];
            a_hi[t] = arp[rr + 1];
            lraw[t] = lofs ? lofs[rr] : 0;
            cw[t] = crp ? crp[rr] : 0;
        }
        int c[SCATTER_ITEMS], local[SCATTER_ITEMS];
#pragma unroll
        for (int t = 0; t < SCATTER_ITEMS; ++t) {
            const int64_t row = r0 + t * 256 + threadIdx.x;
            c[t] = row < m ? raw[t] : CLS_EMPTY;
            if (c[t] != CLS_EMPTY) c[t] = remap[c[t]];
            local[t] = c[t] != CLS_EMPTY ? atomicAdd(&cnt[c[t]], 1) : 0;
        }
        // list capacities of the chunk (rows of the global path get none)
        int32_t cap[SCATTER_ITEMS];
        int64_t lsum = 0;
#pragma unroll
        for (int t = 0; t < SCATTER_ITEMS; ++t) {
            cap[t] = 0;
            if (lofs && c[t] != CLS_EMPTY && c[t] % NTIER != TIER_GLOBAL) cap[t] = lraw[t];
            lsum += cap[t];
        }
        int64_t lex = 0;
        if (lofs) {
            const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
            int64_t x = lsum;
            for (int d = 1; d < 64; d <<= 1) {
                const int64_t y = __shfl_up(x, d, 64);
                if (lane >= d) x += y;
            }
            if (lane == 63) wsum[wv] = x;
            __syncthreads();
            int64_t pre = 0, tot = 0;
            for (int u = 0; u < 4; ++u) {
                if (u < wv) pre += wsum[u];
                tot += wsum[u];
            }
            lex = pre + x - lsum;
            if (threadIdx.x == 0) lbase = tot ? (int64_t)atomicAdd((unsigned long long*)&ctl->list_total,
                                                                   (unsigned long long)tot)
                                              : 0;
        }
        __syncthreads();
        if (threadIdx.x < NCLS) {
            // the chunk's start in class c: the counts of every chunk before it
            // (chunks are taken in ticket order, so each one waited for is
            // resident or finished and the wait ends)
            const int c = threadIdx.x;
            const uint64_t agg = (uint32_t)cnt[c];
            uint64_t* mine = status + chunk * NCLS + c;
            int64_t prefix = 0;
            if (chunk == 0) {
                __hip_atomic_store(mine, ST_PRE | agg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                __hip_atomic_store(mine, ST_AGG | agg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                for (int64_t t = chunk - 1; t >= 0; --t) {
                    uint64_t w;
                    do {
                        w = __hip_atomic_load(status + t * NCLS + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    } while ((w >> 62) == 0);
                    prefix += (int64_t)(w & ST_VAL);
                    if ((w >> 62) == 2) break;
                }
                __hip_atomic_store(mine, ST_PRE | (uint64_t)(prefix + (int64_t)agg), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            base[c] = (int32_t)prefix;
        }
        __syncthreads();
        int64_t lpos = lofs ? lbase + lex : 0;
#pragma unroll
        for (int t = 0; t < SCATTER_ITEMS; ++t) {
            if (c[t] == CLS_EMPTY) continue;
            const int32_t row = (int32_t)(r0 + t * 256 + threadIdx.x);
            const int32_t pos = off[c[t]] + base[c[t]] + local[t];
            int32_t w = cw[t];
            if (lofs) {
                w = cap[t] > 0 && lpos + cap[t] <= list_limit ? (int32_t)lpos : -1;
                lofs[row] = w;
                lpos += cap[t];
            }
            perm[pos] = row;
            desc[pos] = make_int4(row, a_lo[t], a_hi[t], w);
        }
        __syncthreads();
    }
}

// Row pointer = exclusive prefix sum of row_nnz, in 64-bit, single pass with
// decoupled look-back over tiles taken in launch order.  Also assigns each
// row's numeric class (its exact size is now known; rows without a list take
// the global path) and counts rows whose symbolic class differed from the
// class their true size asks for.
template <int ITEMS>
__global__ __launch_bounds__(SCAN_THREADS) void k_scan(int32_t m, const int32_t* __restrict__ row_nnz,
                                                       const int32_t* __restrict__ row_blocks,
                                                       const RowInfo* __restrict__ rinfo,
                                                       const int32_t* __restrict__ arp,
                                                       const uint8_t* __restrict__ sym_cls,
                                                       const int32_t* __restrict__ lofs,
                                                       int32_t* __restrict__ c_row_ptr, uint64_t* tile_status,
                                                       ClassCfg cfg, uint8_t* __restrict__ num_cls, Shard* shards,
                                                       Control* ctl) {
    __shared__ int32_t tile_sh;
    __shared__ int64_t wsum[SCAN_THREADS / 64];
    __shared__ int64_t tile_prefix;
    __shared__ unsigned long long acc[NCOUNT];
    __shared__ int sh;
    if (threadIdx.x == 0) tile_sh = atomicAdd(&ctl->tile_counter, 1);
    if (threadIdx.x < NCOUNT) acc[threadIdx.x] = 0;
    __syncthreads();
    const int tile = tile_sh;
    const int64_t r0 = ((int64_t)tile * SCAN_THREADS + threadIdx.x) * ITEMS;
    int64_t v[ITEMS];
    int64_t run = 0;
    // every row's inputs first, as unconditional loads (a row past the end
    // reads the last row's, unused; arp has m + 1 entries): a load under a
    // condition would be waited for before the next one is issued
    int32_t nz[ITEMS], bl[ITEMS], lo[ITEMS], ap[ITEMS + 1];
    RowInfo rf[ITEMS];
    uint8_t sc[ITEMS];
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) {
        const int64_t rr = r0 + t < m ? r0 + t : m - 1;
        nz[t] = row_nnz[rr];
        rf[t] = rinfo[rr];
        bl[t] = row_blocks[rr];
        lo[t] = lofs[rr];
        sc[t] = sym_cls[rr];
    }
#pragma unroll
    for (int t = 0; t <= ITEMS; ++t) ap[t] = arp[r0 + t < m ? r0 + t : m];
    // the thread's consecutive rows of one class are counted in registers and
    // added to the workgroup's counters once per run of equal classes
    int cur = CLS_EMPTY, n_cur = 0, miss = 0;
    unsigned long long a_cur = 0, c_cur = 0, p_cur = 0;
    auto flush = [&]() {
        if (cur == CLS_EMPTY) return;
        atomicAdd(&acc[CNT_HIST + cur], (unsigned long long)n_cur);
        atomicAdd(&acc[CNT_ANNZ + cur], a_cur);
        atomicAdd(&acc[CNT_CNNZ + cur], c_cur);
        atomicAdd(&acc[CNT_PROD + cur], p_cur);
    };
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) {
        int64_t r = r0 + t;
        int64_t c = 0;
        if (r < m) {
            c = nz[t];
            const RowInfo ri = rf[t];
            const int blocks = bl[t];
            int nc = num_class(ri.z, ri.x, ri.y, c, blocks, cfg);
            // a row kernel builds its table from the row's list: without one, the global path
            if (nc != CLS_EMPTY && nc % NTIER != TIER_GLOBAL && lo[t] < 0) nc = MODE_DIRECT * NTIER + TIER_GLOBAL;
            num_cls[r] = (uint8_t)nc;
            if (nc != CLS_EMPTY) {
                if (nc != cur) {
                    flush();
                    cur = nc, n_cur = 0, a_cur = c_cur = p_cur = 0;
                }
                n_cur += 1;
                a_cur += (unsigned long long)(ap[t + 1] - ap[t]);
                c_cur += (unsigned long long)c;
                p_cur += (unsigned long long)ri.z;
                if (nc % NTIER == TIER_GLOBAL) atomicMax(&acc[CNT_WGLOB], (unsigned long long)row_words(ri.x, ri.y));
                // the class the exact size asks for, under the same sizing rule as the estimate's
                miss += sym_class(ri.z, ri.x, ri.y, blocks, cfg, cfg.bound_est != 0) != sc[t];
            }
        }
        run += c;
        v[t] = run;
    }
    flush();
    if (miss) atomicAdd(&acc[CNT_ROWS], (unsigned long long)miss);
    // block scan of the per-thread totals
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int64_t x = run;
    for (int d = 1; d < 64; d <<= 1) {
        int64_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) wsum[wv] = x;
    __syncthreads();
    int64_t wpre = 0, agg = 0;
    for (int u = 0; u < SCAN_THREADS / 64; ++u) {
        if (u < wv) wpre += wsum[u];
        agg += wsum[u];
    }
    const int64_t thread_excl = wpre + x - run;
    if (gridDim.x > DIRECT_GRID) add_counts(acc, shards);
    // decoupled look-back: publish the aggregate, then add predecessors, 64
    // tiles of them at a time by the first wavefront (one by one, a round
    // trip each, it was most of this kernel at a few hundred tiles)
    if (threadIdx.x < 64) {
        if (threadIdx.x == 0)
            __hip_atomic_store(&tile_status[tile], (tile == 0 ? ST_PRE : ST_AGG) | (uint64_t)agg, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        int64_t prefix = 0;
        // tiles are numbered in the order they started, so every predecessor
        // is resident or finished and each wait below ends
        for (int t0 = tile - 1; t0 >= 0; t0 -= 64) {
            const int t = t0 - lane;
            uint64_t st = ST_PRE;  // past the first tile: nothing before
            if (t >= 0) {
                do {
                    st = __hip_atomic_load(&tile_status[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } while ((st >> 62) == 0);
            }
            const uint64_t pre = __ballot((st >> 62) == 2);
            const int last = pre ? __builtin_ctzll(pre) : 63;  // the nearest tile whose prefix is known
            int64_t v = lane <= last ? (int64_t)(st & ST_VAL) : 0;
            for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
            prefix += v;
            if (pre) break;
        }
        if (threadIdx.x == 0) {
            if (tile > 0)
                __hip_atomic_store(&tile_status[tile], ST_PRE | (uint64_t)(prefix + agg), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            tile_prefix = prefix;
        }
    }
    __syncthreads();
    const int64_t base = tile_prefix + thread_excl;
    bool ovf = false;
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) {
        int64_t r = r0 + t;
        if (r < m) {
            int64_t val = base + v[t];
            if (val > INT_MAX) ovf = true;
            c_row_ptr[r + 1] = (int32_t)val;
            if (r == m - 1) ctl->nnz_c = val;
        }
    }
    if (tile == 0 && threadIdx.x == 0) c_row_ptr[0] = 0;
    if (ovf) atomicOr(&ctl->err, ERR_NNZ_OVERFLOW);
    if (gridDim.x > DIRECT_GRID && !sum_counts(acc, shards, &ctl->done[1], &sh)) return;
    if (threadIdx.x < NCLS) {
        add_to(&ctl->num_hist[threadIdx.x], acc[CNT_HIST + threadIdx.x]);
        add_to(&ctl->num_a_nnz[threadIdx.x], acc[CNT_ANNZ + threadIdx.x]);
        add_to(&ctl->num_c_nnz[threadIdx.x], acc[CNT_CNNZ + threadIdx.x]);
        add_to(&ctl->num_products[threadIdx.x], acc[CNT_PROD + threadIdx.x]);
    }
    if (threadIdx.x == 64) {
        add_to(&ctl->mispredicted, acc[CNT_ROWS]);
        max_to(&ctl->max_words_num_global, acc[CNT_WGLOB]);
    }
}

__global__ void k_export_rows(int32_t m, const float* __restrict__ feats, const int32_t* __restrict__ row_blocks,
                              const int32_t* __restrict__ row_nnz_in, float* __restrict__ x, float* __restrict__ y,
                              int32_t* __restrict__ row_nnz_out) {
    const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (r >= m) return;
    x[r * 3] = feats[r * 3];
    x[r * 3 + 1] = feats[r * 3 + 1];
    x[r * 3 + 2] = feats[r * 3 + 2];
    y[r] = log2f(1.0f + (float)row_blocks[r]);
    if (row_nnz_out) row_nnz_out[r] = row_nnz_in[r];
}


// Batched products as one block-diagonal product: product p's rows are
// appended to the packed row pointer (entry offsets made global) and, for A,
// its column indices are shifted by the number of B rows before it so they
// address its own B rows.  B's columns stay local: a row of C only ever
// meets the columns of its own product's B.  Each product's local arrays are
// checked (row pointer from 0 to its nnz, columns below its own width).
__global__ __launch_bounds__(256) void k_pack(int32_t count, const int64_t* __restrict__ desc,
                                              const int32_t* __restrict__ rp_pool,
                                              const int32_t* __restrict__ col_pool, int32_t* __restrict__ rp_out,
                                              int32_t* __restrict__ col_out, int32_t* __restrict__ err) {
    // desc per product: row offset, row-pointer offset, nnz offset, rows, nnz, column shift, column limit
    for (int p = blockIdx.x; p < count; p += gridDim.x) {
        const int64_t* d = desc + 7 * (int64_t)p;
        const int64_t roff = d[0], rpoff = d[1], noff = d[2], rows = d[3], nnz = d[4], shift = d[5], lim = d[6];
        int bad = 0;
        if (threadIdx.x == 0 && (rp_pool[rpoff] != 0 || (int64_t)rp_pool[rpoff + rows] != nnz)) bad = 1;
        for (int64_t r = threadIdx.x; r < rows; r += blockDim.x) {
            const int32_t v = rp_pool[rpoff + r];
            if (v < 0 || (int64_t)v > nnz || v > rp_pool[rpoff + r + 1]) bad = 1;
            rp_out[roff + r] = (int32_t)(noff + v);
        }
        for (int64_t q = threadIdx.x; q < nnz; q += blockDim.x) {
            const int32_t c = col_pool[noff + q];
            if (c < 0 || (int64_t)c >= lim) bad = 1;
            if (col_out) col_out[noff + q] = (int32_t)(c + shift);
        }
        if (bad) atomicOr(err, 1);
    }
}

// Reduction over an aligned group of 8 lanes: quad swaps, then the half-row
// mirror (lane i with lane 7 - i), after which every lane holds the result.
template <typename Op>
__device__ inline int row8_reduce(int v, Op op) {
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0xb1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0x4e, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, false));  // row_half_mirror
    return v;
}

// B rows in one pass, ROW_LANES lanes per row reading it in coalesced chunks:
// the row pointer and the columns are checked; the row's length, smallest
// and largest column go to binfo; and the row is compressed (section 2.2.1):
// every run of consecutive entries that share a 32-column block becomes one
// {block, OR of the column bits} entry.  A row has at most as many runs as
// entries, so its runs are stored from the row's own first entry on (no scan
// places them), and the header {first entry, length, first run, run count}
// and binfo's run count follow.  An entry starts a run when its block differs
// from the previous entry's; a segmented OR across the chunk gathers each
// run's bits, and the lane holding a run's last entry writes it at the run's
// index (runs begun before it in the row).  A malformed row gets length and
// runs 0 and raises the error flag, on which every later kernel exits.
struct BRow {
    int bad = 0;
    int done = 0;          // runs begun in earlier chunks
    int mn = INT_MAX, mx = -1;
    uint32_t carry = 0;    // bits of the run still open at the end of the last chunk
    // block of the last chunk's final entry; before the first chunk what no
    // column's block is, an invalid one's included: the first entry starts a
    // run whatever it holds, so no run index is below 0
    int last_blk = INT_MIN;
};

// U chunks of the row from entry Q0 on.  Unconditional loads, indices clamped
// into the row (a load under a condition would be waited for before the next
// one is issued); entries past the row's end are not used.
template <int U>
__device__ inline void b_chunks(BRow& r, const int32_t* __restrict__ bci, int2* __restrict__ bc, int32_t k, uint32_t s,
                                uint32_t e, uint32_t Q0, int sl, int shift) {
    constexpr int L = ROW_LANES;
    static_assert(L == 8, "the DPP shifts and swizzles below assume 8-lane groups");
    int cc[U], nx[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t q = Q0 + u * L + sl;
        cc[u] = bci[min(q, e - 1)];
        nx[u] = bci[min(q + 1, e - 1)];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t q0 = Q0 + u * L;
        if (q0 >= e) break;  // uniform in the row's lanes
        const uint32_t q = q0 + sl;
        const bool v = q < e;
        const int c = cc[u];
        if (v) {
            if (c < 0 || c >= k) r.bad = ERR_B_COL;
            r.mn = min(r.mn, c);
            r.mx = max(r.mx, c);
        }
        const int blk = v ? c >> 5 : -1;
        // neighbours inside the 8-lane group: DPP row shifts (a group is an
        // aligned half of a 16-lane row; the lanes whose neighbour lies
        // outside the group take it from elsewhere)
        int prev = __builtin_amdgcn_mov_dpp(blk, 0x111, 0xf, 0xf, false);  // row_shr:1
        if (sl == 0) prev = r.last_blk;
        int next = __builtin_amdgcn_mov_dpp(blk, 0x101, 0xf, 0xf, false);  // row_shl:1
        if (sl == L - 1) next = q + 1 < e ? nx[u] >> 5 : -1;
        const int start = v && blk != prev;
        const bool last = v && (q + 1 >= e || next != blk);
        // segmented inclusive OR of the column bits, segments begin at run starts
        uint32_t m = v ? 1u << (c & 31) : 0u;
        int f = start;
        const auto seg_step = [&](uint32_t mu, int fu, int d) {
            if (sl >= d && !f) {
                m |= mu;
                f = fu;
            }
        };
        seg_step((uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x111, 0xf, 0xf, false),
                 __builtin_amdgcn_mov_dpp(f, 0x111, 0xf, 0xf, false), 1);  // row_shr:1
        seg_step((uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x112, 0xf, 0xf, false),
                 __builtin_amdgcn_mov_dpp(f, 0x112, 0xf, 0xf, false), 2);  // row_shr:2
        seg_step((uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x114, 0xf, 0xf, false),
                 __builtin_amdgcn_mov_dpp(f, 0x114, 0xf, 0xf, false), 4);  // row_shr:4
        if (!f) m |= r.carry;
        const uint64_t starts = (__ballot(start) >> shift) & ((1ull << L) - 1);
        const int idx = r.done + __popcll(starts & ((2ull << sl) - 1)) - 1;
        if (last) bc[s + idx] = make_int2(blk, (int)m);
        r.done += __popcll(starts);
        // lane 7 of each group to the whole group: swizzle lane -> (lane & 0x18) | 7
        r.carry = (uint32_t)__builtin_amdgcn_ds_swizzle((int)m, 0xF8);
        r.last_blk = __builtin_amdgcn_ds_swizzle(blk, 0xF8);
    }
}

// A row by one lane, eight entries at a time; its runs are written as they end.
__device__ inline void b_lane(BRow& r, const int32_t* __restrict__ bci, int64_t bnnz, int2* __restrict__ bc, int32_t k,
                              uint32_t s, uint32_t e) {
    int blk = -1;
    uint32_t m = 0;  // the open run
    int2* out = bc + s;
    for (uint32_t q = s; q < e; q += 8) {
        int c[8];
        load8(c, bci, q, bnnz);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (q + u >= e) break;
            if ((unsigned)c[u] >= (unsigned)k) r.bad = ERR_B_COL;
            r.mn = min(r.mn, c[u]);
            r.mx = max(r.mx, c[u]);
            const int b = c[u] >> 5;
            if (b != blk) {
                if (m) out[r.done++] = make_int2(blk, (int)m);
                blk = b, m = 0;
            }
            m |= 1u << (c[u] & 31);
        }
    }
    if (m) out[r.done++] = make_int2(blk, (int)m);
}

// 64 U entries of a row from Q0 on by a whole wavefront, as b_chunks.
template <int U>
__device__ inline void b_wave(BRow& r, const int32_t* __restrict__ bci, int2* __restrict__ bc, int32_t k, uint32_t s,
                              uint32_t e, uint32_t Q0, int wl) {
    int cc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) cc[u] = bci[min(Q0 + u * 64 + wl, e - 1)];
    const int after = bci[min(Q0 + U * 64, e - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t q = Q0 + u * 64 + wl;
        if (Q0 + u * 64 >= e) break;  // uniform
        const bool v = q < e;
        const int c = cc[u];
        if (v) {
            if (c < 0 || c >= k) r.bad = ERR_B_COL;
            r.mn = min(r.mn, c);
            r.mx = max(r.mx, c);
        }
        const int blk = v ? c >> 5 : -1;
        int prev = __shfl_up(blk, 1, 64);
        if (wl == 0) prev = r.last_blk;
        int next = __shfl_down(blk, 1, 64);
        const int nx = u + 1 < U ? __builtin_amdgcn_readlane(cc[u + 1 < U ? u + 1 : u], 0) : after;
        if (wl == 63) next = q + 1 < e ? nx >> 5 : -1;
        const bool start = v && blk != prev;
        const bool last = v && (q + 1 >= e || next != blk);
        const uint64_t starts = __ballot(start);
        // segmented inclusive OR over the wavefront: DPP shifts inside rows of
        // 16 lanes, then broadcasts of lanes 15 and 31 into the rows after
        uint32_t m = v ? 1u << (c & 31) : 0u;
        int f = start;
        const auto seg_step = [&](int mu, int fu, bool has) {
            if (has && !f) m |= (uint32_t)mu, f = fu;
        };
        const int l16 = wl & 15;
        seg_step(__builtin_amdgcn_mov_dpp((int)m, 0x111, 0xf, 0xf, false),
                 __builtin_amdgcn_mov_dpp(f, 0x111, 0xf, 0xf, false), l16 >= 1);  // row_shr:1
        seg_step(__builtin_amdgcn_mov_dpp((int)m, 0x112, 0xf, 0xf, false),
                 __builtin_amdgcn_mov_dpp(f, 0x112, 0xf, 0xf, false), l16 >= 2);  // row_shr:2
        seg_step(__builtin_amdgcn_mov_dpp((int)m, 0x114, 0xf, 0xf, false),
                 __builtin_amdgcn_mov_dpp(f, 0x114, 0xf, 0xf, false), l16 >= 4);  // row_shr:4
        seg_step(__builtin_amdgcn_mov_dpp((int)m, 0x118, 0xf, 0xf, false),
                 __builtin_amdgcn_mov_dpp(f, 0x118, 0xf, 0xf, false), l16 >= 8);  // row_shr:8
        seg_step(__builtin_amdgcn_update_dpp(0, (int)m, 0x142, 0xa, 0xf, false),
                 __builtin_amdgcn_update_dpp(0, f, 0x142, 0xa, 0xf, false), (wl & 16) != 0);  // row_bcast:15
        seg_step(__builtin_amdgcn_update_dpp(0, (int)m, 0x143, 0xc, 0xf, false),
                 __builtin_amdgcn_update_dpp(0, f, 0x143, 0xc, 0xf, false), wl >= 32);  // row_bcast:31
        if (!f) m |= r.carry;
        const int idx = r.done + __popcll(starts & ((2ull << wl) - 1)) - 1;
        if (last) bc[s + idx] = make_int2(blk, (int)m);
        r.done += __popcll(starts);
        r.carry = (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
        r.last_blk = __builtin_amdgcn_readlane(blk, 63);
    }
}

template <int L>
__global__ __launch_bounds__(256) void k_b_rows(int32_t n, int32_t k, const int32_t* __restrict__ brp,
                                                const int32_t* __restrict__ bci, int64_t bnnz, int4* __restrict__ binfo,
                                                int2* __restrict__ bc, int4* __restrict__ bhdr, Control* ctl) {
    constexpr int GROUPS = 256 / L;
    static_assert(L == 1 || L == ROW_LANES, "one lane, or the group that b_chunks covers");
    __shared__ int32_t longs[GROUPS];
    __shared__ int nlong[2];  // by pass parity: a wavefront may be a pass ahead of another's reading
    if (threadIdx.x < 2) nlong[threadIdx.x] = 0;
    __syncthreads();
    const int sl = threadIdx.x % L, wl = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int shift = wl & ~(L - 1);
    auto finish_row = [&](int64_t j, int32_t s, int32_t e, const BRow& r) {
        if (r.bad) {
            atomicOr(&ctl->err, r.bad);
            binfo[j] = make_int4(0, INT_MAX, -1, 0);
            bhdr[j] = make_int4(0, 0, 0, 0);
        } else {
            binfo[j] = make_int4(e - s, r.mn, r.mx, r.done);
            bhdr[j] = make_int4(s, e - s, s, r.done);
        }
    };
    const int64_t passes = ((int64_t)n + (int64_t)gridDim.x * GROUPS - 1) / ((int64_t)gridDim.x * GROUPS);
    for (int64_t pass = 0; pass < passes; ++pass) {
        const int64_t j = dealt_row<L>(pass, passes, threadIdx.x / L);
        BRow r;
        int32_t s = 0, e = 0;
        if (j < n) {
            s = brp[j], e = brp[j + 1];
            if (s < 0 || e < s || (int64_t)e > bnnz || (j == 0 && s != 0) || (j == n - 1 && (int64_t)e != bnnz))
                r.bad = ERR_B_ROWPTR;
        }
        const bool put_off = !r.bad && e - s > long_row<L>();
        if (put_off && sl == 0) longs[atomicAdd(&nlong[pass & 1], 1)] = (int32_t)j;
        const int32_t len = r.bad || put_off ? 0 : e - s;
        if constexpr (L == 1) {
            if (len > 0) b_lane(r, bci, bnnz, bc, k, s, e);
        } else {
            // one chunk's loads where no row of the wavefront has more
            if (!__any(len > L)) {
                if (len > 0) b_chunks<1>(r, bci, bc, k, s, e, s, sl, shift);
            } else {
                for (uint32_t Q0 = s; Q0 < (uint32_t)(s + len); Q0 += 4 * L)
                    b_chunks<4>(r, bci, bc, k, s, e, Q0, sl, shift);
            }
            r.bad = row8_reduce(r.bad, [](int x, int y) { return x | y; });
            r.mn = row8_reduce(r.mn, [](int x, int y) { return min(x, y); });
            r.mx = row8_reduce(r.mx, [](int x, int y) { return max(x, y); });
        }
        if (sl == 0 && j < n && !put_off) finish_row(j, s, e, r);
        __syncthreads();
        const int nl = nlong[pass & 1];
        if (nl > 0) {
            // uniform; the pass's long rows, a wavefront each
            for (int l = wv; l < nl; l += 4) {
                const int64_t lj = longs[l];
                const int32_t ls = brp[lj], le = brp[lj + 1];
                BRow q;
                for (uint32_t Q0 = ls; Q0 < (uint32_t)le; Q0 += 8 * 64) b_wave<8>(q, bci, bc, k, ls, le, Q0, wl);
                q.bad = __any(q.bad) ? ERR_B_COL : 0;
                q.mn = wave_reduce(q.mn, [](auto x, auto y) { return x < y ? x : y; });
                q.mx = wave_reduce(q.mx, [](auto x, auto y) { return x > y ? x : y; });
                if (wl == 0) finish_row(lj, ls, le, q);
            }
            __syncthreads();
            if (threadIdx.x == 0) nlong[pass & 1] = 0;
            __syncthreads();
        }
    }
}

inline unsigned grid_for(int64_t threads, int per_block) {
    int64_t g = (threads + per_block - 1) / per_block;
    return (unsigned)(g < 1 ? 1 : g);
}

// Workgroups of an analysis pass over `rows` rows with L lanes each.  Where
// rows are long on average, at least one workgroup per four rows: as few
// workgroups as their lanes need leave the chip idle (2000 rows of 2000
// entries of A: the analysis 141 us with 32 workgroups, 38 so; 10 thousand rows
// of 400: 55 and 47; 15 thousand rows of 256: 46 and 62).
constexpr int LONG_AVERAGE = 320;
inline unsigned analysis_grid(int64_t rows, int lanes, int64_t nnz, unsigned most) {
    int64_t g = grid_for(rows * lanes, 256);
    if (nnz > rows * LONG_AVERAGE) g = std::max(g, (rows + 3) / 4);
    return (unsigned)std::min<int64_t>(g, most);
}

}  // namespace

// Rows per thread of the scan: one for small m, where a thread's eight rows
// one after another (two class choices each) are most of the kernel's time.
constexpr int32_t SCAN_SMALL = 1 << 17;
int64_t scan_tiles(int32_t m) {
    const int64_t tile = SCAN_THREADS * (m <= SCAN_SMALL ? 1 : SCAN_ITEMS);
    return ((int64_t)m + tile - 1) / tile;
}

void launch_pack(hipStream_t s, int32_t count, const int64_t* desc, const int32_t* rp_pool, const int32_t* col_pool,
                 int32_t* rp_out, int32_t* col_out, int32_t* err) {
    if (count <= 0) return;
    hipLaunchKernelGGL(k_pack, dim3((unsigned)std::min(count, 4096)), dim3(256), 0, s, count, desc, rp_pool, col_pool,
                       rp_out, col_out, err);
}

void launch_fill_i32(hipStream_t s, int32_t* p, int32_t v, int64_t n) {
    if (n <= 0) return;
    int64_t g = (n + 255) / 256;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)g), dim3(256), 0, s, p, v, n);
}

void launch_fill_u8(hipStream_t s, void* p, uint8_t v, int64_t bytes) {
    if (bytes <= 0) return;
    int64_t g = (bytes + 255) / 256;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_fill_u8, dim3((unsigned)g), dim3(256), 0, s, (uint8_t*)p, v, bytes);
}

void launch_publish(hipStream_t s, const Control* ctl, Control* host, uint32_t seq) {
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(256), 0, s, (const uint32_t*)ctl, (uint32_t*)host, seq);
}

void launch_zero(hipStream_t s, void* p, int64_t bytes) {
    if (bytes <= 0) return;
    const int64_t n16 = bytes / 16;
    hipLaunchKernelGGL(k_zero, dim3((unsigned)std::min<int64_t>((n16 + 255) / 256, 1024)), dim3(256), 0, s,
                       (uint4*)p, n16);
}

void launch_b_rows(hipStream_t s, int32_t n, int32_t k, const int32_t* brp, const int32_t* bci, int64_t bnnz,
                   int4* binfo, int2* bc, int4* bhdr, Control* ctl) {
    if (n <= 0) return;
    if (n >= SHORT_MIN_ROWS && bnnz <= (int64_t)SHORT_ROWS * n)
        hipLaunchKernelGGL(k_b_rows<1>, dim3(std::min(grid_for(n, 256), 2048u)), dim3(256), 0, s, n, k, brp, bci, bnnz,
                           binfo, bc, bhdr, ctl);
    else
        hipLaunchKernelGGL(k_b_rows<ROW_LANES>, dim3(analysis_grid(n, ROW_LANES, bnnz, 4096)),
                           dim3(256), 0, s, n, k, brp, bci, bnnz, binfo, bc, bhdr, ctl);
}

void launch_a_rowinfo(hipStream_t s, int32_t m, int32_t n, const int32_t* arp, const int32_t* aci, int64_t annz,
                      const int4* binfo, RowInfo* rinfo, float* feats, ClassCfg cfg, int binning,
                      uint8_t* sym_cls, int32_t* row_nnz, int32_t* row_blocks, int32_t* lofs, Shard* shards,
                      Control* ctl) {
    if (m <= 0) return;
    if (m >= SHORT_MIN_ROWS && annz <= (int64_t)SHORT_ROWS * m)
        hipLaunchKernelGGL(k_a_rowinfo<1>, dim3(std::min(grid_for(m, 256), 2048u)), dim3(256), 0, s, m, n, arp, aci,
                           annz, binfo, rinfo, feats, cfg, binning, sym_cls, row_nnz, row_blocks, lofs, shards, ctl);
    else
        hipLaunchKernelGGL(k_a_rowinfo<AN_LANES>, dim3(analysis_grid(m, AN_LANES, annz, 2048)),
                           dim3(256), 0, s, m, n, arp, aci, annz, binfo, rinfo, feats, cfg, binning, sym_cls, row_nnz,
                           row_blocks, lofs, shards, ctl);
}

void launch_mlp_classify(hipStream_t s, int32_t m, const float* feats, const float* w, const RowInfo* rinfo,
                         ClassCfg cfg, float margin, uint8_t* sym_cls, Control* ctl) {
    if (m <= 0) return;
    hipLaunchKernelGGL(k_mlp_classify, dim3(std::min(grid_for(m, 256), 1024u)), dim3(256), 0, s, m, feats, w, rinfo,
                       cfg, margin,
                       sym_cls, ctl);
}

size_t scatter_state_bytes(int32_t m) {
    return 64 + (size_t)(((int64_t)std::max(m, 0) + SCATTER_CHUNK - 1) / SCATTER_CHUNK) * NCLS * 8;
}

void launch_scatter(hipStream_t s, int32_t m, const uint8_t* cls, int merge, const int32_t* hist, int32_t* state,
                    int32_t* perm, const int32_t* arp, const int32_t* crp, int4* desc, int32_t* lofs, Control* ctl,
                    int64_t list_limit) {
    if (m <= 0) return;
    hipLaunchKernelGGL(k_scatter, dim3(std::min(grid_for(m, SCATTER_CHUNK), 1024u)), dim3(256), 0, s, m, cls, merge,
                       hist, state, perm, arp, crp, desc, lofs, ctl, list_limit);
}

void launch_scan(hipStream_t s, int32_t m, const int32_t* row_nnz, const int32_t* row_blocks, const RowInfo* rinfo,
                 const int32_t* arp, const uint8_t* sym_cls, const int32_t* lofs, int32_t* c_row_ptr,
                 uint64_t* tile_status, ClassCfg cfg, uint8_t* num_cls, Shard* shards, Control* ctl) {
    if (m <= 0) return;
    const dim3 grid((unsigned)scan_tiles(m));
    if (m <= SCAN_SMALL)
        hipLaunchKernelGGL(k_scan<1>, grid, dim3(SCAN_THREADS), 0, s, m, row_nnz, row_blocks, rinfo, arp, sym_cls, lofs,
                           c_row_ptr, tile_status, cfg, num_cls, shards, ctl);
    else
        hipLaunchKernelGGL(k_scan<SCAN_ITEMS>, grid, dim3(SCAN_THREADS), 0, s, m, row_nnz, row_blocks, rinfo, arp,
                           sym_cls, lofs, c_row_ptr, tile_status, cfg, num_cls, shards, ctl);
}

void launch_export_rows(hipStream_t s, int32_t m, const float* feats, const int32_t* row_blocks,
                        const int32_t* row_nnz_in, float* x, float* y, int32_t* row_nnz_out) {
    if (m <= 0) return;
    hipLaunchKernelGGL(k_export_rows, dim3(grid_for(m, 256)), dim3(256), 0, s, m, feats, row_blocks, row_nnz_in, x,
                       y, row_nnz_out);
}

}  // namespace spg
