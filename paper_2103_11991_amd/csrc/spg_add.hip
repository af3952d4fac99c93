// Sparse matrix addition C = alpha*A + beta*B on CRS matrices (section 2.3).
//
// Two phases like the product: symbolic finds, for every row, the union of
// the columns of A(i,:) and B(i,:) (entries of one column merged), its size
// (scanned into C's row pointer) and, for every input entry, the position of
// its column inside C's row (the paper's Apos and Bpos); numeric scatters
// alpha*A(i,j) and beta*B(i,j) to those positions and writes the columns, so
// a numeric call with new values needs no search at all.
//
// A row whose entries are strictly ascending in both matrices (at most 64 in
// all) needs no sort: an entry's position is its own index plus the entries
// of the other matrix before its column (a binary search among the columns
// in LDS) less the columns before it that both hold (a popcount of the
// matches).  G lanes hold one row, 64 / G rows per wavefront (section 2.3's
// sorted merge).  Other rows order their keys (column, then the entry's index
// inside the row: A's entries first), and a key whose column differs from its
// predecessor's starts a new column of C: rows of up to 256 entries with a
// bitonic network over 32-bit keys in registers (one to four per lane, when
// column and index fit 32 bits), rows of up to 1024 with 64-bit keys in the
// wavefront's LDS, rows of up to 16384 on a 1024-lane workgroup with 128 KB
// of LDS (section 5's team-level sort); longer rows are refused
// (SPG_ERR_UNSUPPORTED).  In LDS, two sorted rows take the merge network
// alone.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <string>

#include "spg_internal.h"

namespace {

constexpr int WAVE = 64;
constexpr int MID_CAP = 1024;      // keys per wavefront in LDS
constexpr int NUM_CAP = 512;       // columns per wavefront in LDS, numeric (16 KB per workgroup: full occupancy)
constexpr int WIDE_THREADS = 256;  // lanes of a numeric row of more than NUM_CAP columns
constexpr int WIDE_CAP = 4096;     // ... and its columns in LDS at a time, at most (32 KB)
constexpr int LONG_CAP = 16384;    // keys per row on the long-row path
constexpr int LONG_THREADS = 1024;
constexpr int ROWS_PER_WG = 4;     // wavefronts (rows) per workgroup of the short/medium kernels
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;
constexpr uint64_t ST_AGG = 1ull << 62, ST_PRE = 2ull << 62, ST_VAL = (1ull << 62) - 1;

// error flags
constexpr int AE_ROWPTR = 1, AE_COL = 2, AE_LONG = 4, AE_OVERFLOW = 8;

struct AddCtl {
    int32_t err;
    int32_t long_rows;      // rows queued for the long-row kernel
    int32_t tile_counter;   // dynamic tile id of the row-pointer scan
    int32_t widest;         // longest row of C of more than NUM_CAP columns (0: no such row)
    int64_t nnz_c;
};

__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Inclusive sum over the wavefront.
__device__ inline int wave_scan(int x) {
    const int lane = threadIdx.x & 63;
    for (int d = 1; d < WAVE; d <<= 1) {
        const int y = __shfl_up(x, d, WAVE);
        if (lane >= d) x += y;
    }
    return x;
}

// Key of entry t of the row (A's la entries, then B's): column, then t, in
// 64 bits, or in 32 where columns fit the 22 bits that MID_CAP's index leaves.
constexpr int32_t KEY32_COLS = 1 << 22;
template <typename K>
constexpr int key_bits() {
    return sizeof(K) == 8 ? 32 : 10;
}
template <typename K>
__device__ inline K make_key(int32_t col, int t) {
    return ((K)(uint32_t)col << key_bits<K>()) | (K)t;
}
template <typename K>
__device__ inline int key_entry(K k) {
    return (int)(k & (((K)1 << key_bits<K>()) - 1));
}

// The row's entries: t < la are A's, the others B's.
struct RowPair {
    const int32_t* ac;
    const int32_t* bc;
    int la, lb;
    __device__ inline int32_t col(int t) const { return t < la ? ac[t] : bc[t - la]; }
};

// Slot of entry t in the bitonic arrangement of P slots: A ascending in
// [0, la), B reversed at the end (descending), so the unused slots lie between.
__device__ inline int merge_slot(int t, int la, int lb, int P) { return t < la ? t : P - 1 - (t - la); }

// Writes each entry's position in C's row from the ordered keys (slot s
// holds key[s]) and returns the row's size.  Lanes of the group own P/G
// consecutive slots each.  The row's L keys come first; the slots after them
// go by that count and not by their filling, which is a key too: column
// 2^22 - 1 and entry 1023 are 32 set bits.  (The key before kept in a register
// made rows of 140 to 1024 entries 2 to 8 % faster and short rows, by the
// kernel's three registers more, 2 % slower.)
template <int G, typename K>
__device__ inline int positions_from_sorted(const K* key, int P, int L, int la, int32_t* apos, int32_t* bpos,
                                            int* red) {
    const int lane = threadIdx.x % G;
    const int per = P / G > 0 ? P / G : 1;
    const int s0 = lane * per;
    int local = 0;
    for (int s = s0; s < s0 + per && s < P; ++s) {
        const K k = key[s];
        if (s >= L) break;
        local += s == 0 || (key[s - 1] >> key_bits<K>()) != (k >> key_bits<K>());
    }
    int total, ex;
    if constexpr (G == WAVE) {
        const int incl = wave_scan(local);
        total = __shfl(incl, WAVE - 1, WAVE);
        ex = incl - local;
    } else {
        const int wl = threadIdx.x & 63, wv = threadIdx.x >> 6;
        const int incl = wave_scan(local);
        __syncthreads();
        if (wl == 63) red[wv] = incl;
        __syncthreads();
        int pre = 0;
        total = 0;
        for (int u = 0; u < G / WAVE; ++u) {
            if (u < wv) pre += red[u];
            total += red[u];
        }
        ex = pre + incl - local;
    }
    int pos = ex - 1;
    for (int s = s0; s < s0 + per && s < P; ++s) {
        const K k = key[s];
        if (s >= L) break;
        pos += s == 0 || (key[s - 1] >> key_bits<K>()) != (k >> key_bits<K>());
        const int t = key_entry(k);
        if (t < la) apos[t] = pos;
        else bpos[t - la] = pos;
    }
    return total;
}

// Bitonic ordering of P (a power of two) keys in LDS by a group of G lanes:
// the merge network alone when the keys form a bitonic sequence, else the
// whole sort.  sync() orders the group's LDS accesses.
template <int G, typename K, typename Sync>
__device__ inline void lds_bitonic(K* key, int P, bool merge_only, Sync sync) {
    const int lane = threadIdx.x % G;
    for (int k = merge_only ? P : 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int x = lane; x < P / 2; x += G) {
                // the x-th pair of this step: lo has bit j clear
                const int lo = ((x & ~(j - 1)) << 1) | (x & (j - 1));
                const int hi = lo | j;
                const bool up = (lo & k) == 0;
                const K a = key[lo], b = key[hi];
                if ((a > b) == up) key[lo] = b, key[hi] = a;
            }
            sync();
        }
    }
}

// Lane ^ J of the wavefront (J a power of two below 64): quad permutes for 1
// and 2, a swizzle inside 32 lanes up to 16, a permute across for 32.
template <int J>
__device__ inline uint32_t lane_xor(uint32_t v) {
    if constexpr (J == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, false);
    else if constexpr (J == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4e, 0xf, 0xf, false);
    else if constexpr (J < 32) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (J << 10) | 0x1f);
    else return (uint32_t)__shfl_xor((int)v, 32, WAVE);
}

// Bitonic sort of 64 R keys in registers, slot r * 64 + lane in v[r]; strides
// of 64 and more stay inside a lane.
template <int R, int K, int J>
__device__ inline void sort_step(uint32_t* v) {
    const int lane = threadIdx.x & 63;
    if constexpr (J >= WAVE) {
        constexpr int jr = J / WAVE;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r & jr) continue;
            const bool up = ((r * WAVE) & K) == 0;  // K > J >= 64: the same for all lanes
            const uint32_t lo = min(v[r], v[r | jr]), hi = max(v[r], v[r | jr]);
            v[r] = up ? lo : hi, v[r | jr] = up ? hi : lo;
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t o = lane_xor<J>(v[r]);
            const bool up = ((r * WAVE + lane) & K) == 0, low = (lane & J) == 0;
            // the lower slot of a pair keeps the smaller key when ascending
            v[r] = low == up ? min(v[r], o) : max(v[r], o);
        }
    }
    if constexpr (J > 1) sort_step<R, K, J / 2>(v);
    else if constexpr (K < WAVE * R) sort_step<R, 2 * K, K>(v);
}

// Positions of a row of la + lb <= 64 R entries by sorting; returns its size.
template <int R>
__device__ inline int sort_positions(const RowPair& rw, int32_t* ap, int32_t* bp) {
    constexpr int TB = R == 1 ? 6 : R == 2 ? 7 : 8;  // bits of an entry's index
    const int lane = threadIdx.x & 63, L = rw.la + rw.lb;
    uint32_t v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int t = r * WAVE + lane;
        v[r] = ~0u;
        if (t < L) v[r] = ((uint32_t)rw.col(t) << TB) | (uint32_t)t;
    }
    sort_step<R, 2, 1>(v);
    int before = 0;
    uint32_t last = 0;  // key of the previous register's lane 63
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint32_t pv = (uint32_t)__shfl_up((int)v[r], 1, WAVE);
        if (lane == 0) pv = last;
        // valid keys come first: their count is L
        const bool valid = r * WAVE + lane < L;
        const bool start = valid && ((r == 0 && lane == 0) || (pv >> TB) != (v[r] >> TB));
        const uint64_t starts = __ballot(start);
        if (valid) {
            const int t = (int)(v[r] & ((1u << TB) - 1u));
            const int pos = before + __popcll(starts & ((2ull << lane) - 1)) - 1;
            if (t < rw.la) ap[t] = pos;
            else bp[t - rw.la] = pos;
        }
        before += __popcll(starts);
        last = (uint32_t)__builtin_amdgcn_readlane((int)v[r], 63);
    }
    return before;
}

// One row by a whole wavefront, of at most MID_CAP entries (longer rows are
// queued for k_add_sym_long).  Its pointers are valid.
template <typename K>
__device__ inline void wave_row(int64_t i, int32_t n, const RowPair& rw, int32_t* ap, int32_t* bp, K* key,
                                int32_t* row_nnz, int32_t* long_list, AddCtl* ctl) {
    const int lane = threadIdx.x % WAVE;
    const int L = rw.la + rw.lb;
    if (rw.la > MID_CAP - rw.lb) {  // (their sum may pass 2^31)
        if (lane == 0) {
            long_list[atomicAdd(&ctl->long_rows, 1)] = (int32_t)i;
            row_nnz[i] = 0;
        }
        return;
    }
    // columns in range, and whether each matrix row is ascending
    int bad = 0, unsorted = 0;
    for (int t = lane; t < L; t += WAVE) {
        const int32_t c = rw.col(t);
        bad |= c < 0 || c >= n;
        if (t != 0 && t != rw.la && rw.col(t - 1) > c) unsorted = 1;
    }
    if (__any(bad)) {
        if (lane == 0) atomicOr(&ctl->err, AE_COL), row_nnz[i] = 0;
        return;
    }
    int total;
    if (L <= WAVE && n <= 1 << 26) {
        total = sort_positions<1>(rw, ap, bp);
    } else if (L <= 2 * WAVE && n <= 1 << 25) {
        total = sort_positions<2>(rw, ap, bp);
    } else if (L <= 4 * WAVE && n <= 1 << 24) {
        total = sort_positions<4>(rw, ap, bp);
    } else {
        // keys in the wavefront's LDS
        const bool merge_only = !__any(unsorted);
        int P = WAVE;
        while (P < L) P <<= 1;
        for (int s = lane; s < P; s += WAVE) key[s] = (K)~(K)0;
        wave_sync();
        for (int t = lane; t < L; t += WAVE) {
            const int s = merge_only ? merge_slot(t, rw.la, rw.lb, P) : t;
            key[s] = make_key<K>(rw.col(t), t);
        }
        wave_sync();
        lds_bitonic<WAVE, K>(key, P, merge_only, wave_sync);
        total = positions_from_sorted<WAVE, K>(key, P, L, rw.la, ap, bp, nullptr);
        wave_sync();
    }
    if (lane == 0) row_nnz[i] = total;
}

// Symbolic phase.  G lanes per row: rows of at most G entries, strictly
// ascending in A and in B, are merged in place, two of them per lane group
// and step; every other row of the wavefront is then taken by the whole
// wavefront, one after another.  Bound by its instructions per row and the
// latency of a row's dependent accesses (pointers, columns, the search), hence
// the two rows together, the next ones' pointers a step ahead, and 32-bit
// keys (4 KB of LDS per wavefront, full occupancy) where columns allow (1M
// rows of 30 + 30 entries, G = 64: 0.86 ms as a bitonic merge of 64-bit keys,
// 0.48 as this search one row at a time, 0.32 now; 250k unsorted rows of 0 to
// 96 entries: 0.39 ms with 64-bit keys through LDS permutes, 0.15 now).
template <int G, typename K>
__global__ __launch_bounds__(WAVE * ROWS_PER_WG) void k_add_sym(int32_t m, int32_t n, const int32_t* __restrict__ arp,
                                                                const int32_t* __restrict__ aci, int64_t annz,
                                                                const int32_t* __restrict__ brp,
                                                                const int32_t* __restrict__ bci, int64_t bnnz,
                                                                int32_t* __restrict__ apos, int32_t* __restrict__ bpos,
                                                                int32_t* __restrict__ row_nnz,
                                                                int32_t* __restrict__ long_list, AddCtl* ctl) {
    constexpr int RPW = WAVE / G;  // lane groups per wavefront
    constexpr int R = 2;           // rows per lane group and step
    constexpr uint64_t ONES = G == WAVE ? ~0ull : (1ull << (G & 63)) - 1;
    __shared__ K keys[ROWS_PER_WG][MID_CAP];
    static_assert(sizeof(keys[0]) >= (size_t)R * 2 * WAVE * 4, "two lists of G columns per row");
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int wl = threadIdx.x % WAVE, lane = wl % G, sub = wl / G;
    K* key = keys[wv];
    const int64_t step = (int64_t)gridDim.x * ROWS_PER_WG * RPW * R;
    // rows i0 + r * RPW + sub (a row past the end: the last, unused)
    struct Ptr {
        int as, ae, bs, be;
    };
    auto ptrs = [&](int64_t i) {
        i = i < m ? i : m - 1;
        return Ptr{arp[i], arp[i + 1], brp[i], brp[i + 1]};
    };
    int64_t i0 = ((int64_t)blockIdx.x * ROWS_PER_WG + wv) * RPW * R;
    Ptr nxt[R];
#pragma unroll
    for (int r = 0; r < R; ++r) nxt[r] = ptrs(i0 + r * RPW + sub);
    for (; i0 < m; i0 += step) {
        Ptr p[R];
        int la[R], lb[R], c[R];
        bool ok[R], has[R], strict[R];
#pragma unroll
        for (int r = 0; r < R; ++r) p[r] = nxt[r], nxt[r] = ptrs(i0 + step + r * RPW + sub);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = i0 + r * RPW + sub;
            const bool valid = p[r].as >= 0 && p[r].ae >= p[r].as && (int64_t)p[r].ae <= annz && p[r].bs >= 0 &&
                               p[r].be >= p[r].bs && (int64_t)p[r].be <= bnnz &&
                               (i != 0 || (p[r].as == 0 && p[r].bs == 0)) &&
                               (i != m - 1 || ((int64_t)p[r].ae == annz && (int64_t)p[r].be == bnnz));
            ok[r] = i < m && valid;
            if (i < m && !valid && lane == 0) atomicOr(&ctl->err, AE_ROWPTR), row_nnz[i] = 0;
            la[r] = ok[r] ? p[r].ae - p[r].as : 0, lb[r] = ok[r] ? p[r].be - p[r].bs : 0;
            if (la[r] > G || lb[r] > G - la[r]) la[r] = lb[r] = 0, strict[r] = false;  // not in place
            else strict[r] = ok[r];
            has[r] = lane < la[r] + lb[r];
            c[r] = 0;
            if (has[r]) c[r] = lane < la[r] ? aci[p[r].as + lane] : bci[p[r].bs + lane - la[r]];
        }
        // the row's two lists of columns, each padded to G with a column past all
        wave_sync();  // the previous step's readers are done
        int32_t* list[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            list[r] = reinterpret_cast<int32_t*>(key) + r * 2 * WAVE + sub * 2 * G;
            list[r][lane] = INT_MAX, list[r][G + lane] = INT_MAX;
        }
        wave_sync();
        int longest = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (has[r]) list[r][lane < la[r] ? lane : G + lane - la[r]] = c[r];
            // strictly ascending, except from A's last entry to B's first
            const int prev = __shfl_up(c[r], 1, WAVE);
            const bool wrong =
                has[r] && (c[r] < 0 || c[r] >= n || (lane != 0 && lane != la[r] && prev >= c[r]));
            if (__ballot(wrong) >> (sub * G) & ONES) strict[r] = false;
            longest = max(longest, max(la[r], lb[r]));
        }
        wave_sync();
        // entries of the other list below this column: a count built bit by
        // bit (an entry's own list is not empty, so the other has less than G)
        int lo[R] = {};
        const int32_t* other[R];
#pragma unroll
        for (int r = 0; r < R; ++r) other[r] = list[r] + (lane < la[r] ? G : 0);
#pragma unroll
        for (int h = G / 2; h >= 1; h >>= 1) {
            if (!__any(longest >= h)) continue;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (other[r][lo[r] + h - 1] < c[r]) lo[r] += h;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = i0 + r * RPW + sub;
            const bool mine = has[r] && strict[r];
            const bool match = mine && other[r][lo[r]] == c[r];
            const uint64_t mt = __ballot(match) >> (sub * G) & ONES;
            const uint64_t a_lanes = la[r] >= 64 ? ~0ull : (1ull << la[r]) - 1;
            const uint64_t below = (1ull << lane) - 1;
            if (mine) {
                if (lane < la[r]) apos[p[r].as + lane] = lane + lo[r] - __popcll(mt & below);
                else bpos[p[r].bs + lane - la[r]] = lane - la[r] + lo[r] - __popcll(mt & below & ~a_lanes);
            }
            if (strict[r] && lane == 0) row_nnz[i] = la[r] + lb[r] - __popcll(mt & a_lanes);
        }
        // the wavefront's other rows
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint64_t rest = __ballot(ok[r] && !strict[r] && lane == 0);
            while (rest) {
                const int src = __builtin_ctzll(rest);
                rest &= rest - 1;
                const int64_t ri = i0 + r * RPW + src / G;
                const int ras = __builtin_amdgcn_readlane(p[r].as, src), rae = __builtin_amdgcn_readlane(p[r].ae, src);
                const int rbs = __builtin_amdgcn_readlane(p[r].bs, src), rbe = __builtin_amdgcn_readlane(p[r].be, src);
                const RowPair rw{aci + ras, bci + rbs, rae - ras, rbe - rbs};
                wave_sync();
                wave_row<K>(ri, n, rw, apos + ras, bpos + rbs, key, row_nnz, long_list, ctl);
            }
        }
    }
}

// Symbolic phase of the queued long rows (MID_CAP < entries <= LONG_CAP):
// one 1024-lane workgroup per row, keys in 128 KB of LDS.
__global__ __launch_bounds__(LONG_THREADS) void k_add_sym_long(int32_t n, const int32_t* __restrict__ arp,
                                                               const int32_t* __restrict__ aci,
                                                               const int32_t* __restrict__ brp,
                                                               const int32_t* __restrict__ bci,
                                                               int32_t* __restrict__ apos, int32_t* __restrict__ bpos,
                                                               int32_t* __restrict__ row_nnz,
                                                               const int32_t* __restrict__ long_list, AddCtl* ctl) {
    extern __shared__ uint64_t key[];
    __shared__ int red[LONG_THREADS / WAVE];
    __shared__ int flags[2];
    const int count = ctl->long_rows;
    const int tid = threadIdx.x;
    for (int r = blockIdx.x; r < count; r += gridDim.x) {
        const int i = long_list[r];
        const int as = arp[i], bs = brp[i];
        const RowPair rw{aci + as, bci + bs, arp[i + 1] - as, brp[i + 1] - bs};
        const int L = rw.la + rw.lb;
        if (tid == 0) flags[0] = flags[1] = 0;
        __syncthreads();
        if (rw.la > LONG_CAP - rw.lb) {
            if (tid == 0) atomicOr(&ctl->err, AE_LONG);
            continue;
        }
        int bad = 0, unsorted = 0;
        for (int t = tid; t < L; t += LONG_THREADS) {
            const int32_t c = rw.col(t);
            bad |= c < 0 || c >= n;
            if (t != 0 && t != rw.la && rw.col(t - 1) > c) unsorted = 1;
        }
        if (bad) atomicOr(&flags[0], 1);
        if (unsorted) atomicOr(&flags[1], 1);
        __syncthreads();
        if (flags[0]) {
            if (tid == 0) atomicOr(&ctl->err, AE_COL), row_nnz[i] = 0;
            __syncthreads();
            continue;
        }
        const bool merge_only = flags[1] == 0;
        int P = LONG_THREADS;
        while (P < L) P <<= 1;
        for (int s = tid; s < P; s += LONG_THREADS) key[s] = ~0ull;
        __syncthreads();
        for (int t = tid; t < L; t += LONG_THREADS) {
            const int s = merge_only ? merge_slot(t, rw.la, rw.lb, P) : t;
            key[s] = make_key<uint64_t>(rw.col(t), t);
        }
        __syncthreads();
        lds_bitonic<LONG_THREADS, uint64_t>(key, P, merge_only, [] { __syncthreads(); });
        const int total = positions_from_sorted<LONG_THREADS, uint64_t>(key, P, L, rw.la, apos + as, bpos + bs, red);
        if (tid == 0) row_nnz[i] = total;
        __syncthreads();
    }
}

// C's row pointer: exclusive scan of the row sizes in int64, single pass with
// decoupled look-back over tiles taken in order; flags nnz(C) >= 2^31 and finds
// the longest row.
__global__ __launch_bounds__(SCAN_THREADS) void k_add_scan(int32_t m, const int32_t* __restrict__ row_nnz,
                                                           int32_t* __restrict__ crp, uint64_t* tile_status,
                                                           AddCtl* ctl) {
    __shared__ int32_t tile_sh;
    __shared__ int64_t wsum[SCAN_THREADS / 64];
    __shared__ int64_t tile_prefix;
    if (threadIdx.x == 0) tile_sh = atomicAdd(&ctl->tile_counter, 1);
    __syncthreads();
    const int tile = tile_sh;
    const int64_t r0 = (int64_t)tile * SCAN_TILE + threadIdx.x * SCAN_ITEMS;
    int64_t v[SCAN_ITEMS];
    int64_t run = 0;
    int longest = 0;
#pragma unroll
    for (int t = 0; t < SCAN_ITEMS; ++t) {
        const int64_t r = r0 + t;
        const int size = r < m ? row_nnz[r] : 0;
        longest = max(longest, size);
        run += size;
        v[t] = run;
    }
    // (read first: atomics of many wavefronts on one address take their turns)
    if (__any(longest > NUM_CAP)) {
        for (int d = 32; d > 0; d >>= 1) longest = max(longest, __shfl_xor(longest, d, 64));
        if ((threadIdx.x & 63) == 0 &&
            __hip_atomic_load(&ctl->widest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < longest)
            atomicMax(&ctl->widest, longest);
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int64_t x = run;
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) wsum[wv] = x;
    __syncthreads();
    int64_t wpre = 0, agg = 0;
    for (int u = 0; u < SCAN_THREADS / 64; ++u) {
        if (u < wv) wpre += wsum[u];
        agg += wsum[u];
    }
    if (threadIdx.x < 64) {
        // look-back over 64 tiles at a time (tiles are numbered in the order
        // they started, so every wait ends)
        if (threadIdx.x == 0)
            __hip_atomic_store(&tile_status[tile], (tile == 0 ? ST_PRE : ST_AGG) | (uint64_t)agg, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        int64_t prefix = 0;
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
            int64_t w = lane <= last ? (int64_t)(st & ST_VAL) : 0;
            for (int d = 32; d > 0; d >>= 1) w += __shfl_xor(w, d, 64);
            prefix += w;
            if (pre) break;
        }
        if (threadIdx.x == 0) {
            if (tile > 0)
                __hip_atomic_store(&tile_status[tile], ST_PRE | (uint64_t)(prefix + agg), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            tile_prefix = prefix;
            const int64_t last_tile = ((int64_t)m + SCAN_TILE - 1) / SCAN_TILE - 1;
            if (tile == last_tile) {
                ctl->nnz_c = prefix + agg;
                if (prefix + agg > INT_MAX) atomicOr(&ctl->err, AE_OVERFLOW);
            }
        }
    }
    __syncthreads();
    const int64_t base = tile_prefix + wpre + x - run;
#pragma unroll
    for (int t = 0; t < SCAN_ITEMS; ++t) {
        const int64_t r = r0 + t;
        if (r < m) crp[r + 1] = (int32_t)(base + v[t]);
    }
    if (tile == 0 && threadIdx.x == 0) crp[0] = 0;
}

// Numeric phase: per row, every entry adds alpha*a (A's first) or beta*b at
// its position; columns written by every contributor (the same value).  The
// row's values are summed in LDS, in FP64 (an LDS add of FP32 values
// serialises its lanes, see acc_bytes), and copied out coalesced.  Entries of A
// are added before those of B, so a column with one entry of each gets
// alpha*a + beta*b, each rounded once.  Two rows of up to 64 entries per
// wavefront and step, their loads issued together and the next two rows'
// pointers a step ahead: the kernel is bound by the latency of its two
// dependent loads (1M rows of 30 + 30 entries, FP64: 0.62 ms with one row at
// a time, 0.375 now, 4.7 TB/s, about what a copy of that size reaches).  Rows
// of more entries and up to NUM_CAP columns take a wavefront's LDS whole, one
// after another; longer ones have a kernel of their own (k_add_num_wide).

// U entries per lane from t0 on of one matrix's row (which ends at q1), added
// at their positions less s0 by G lanes; positions outside [0, len) are left
// out (ALL: none is).  Only the last U-th of them may pass the row's end.
template <int G, int U, bool ALL, typename T>
__device__ inline void add_chunk(uint32_t t0, uint32_t q1, const int32_t* __restrict__ pos,
                                 const int32_t* __restrict__ ci, const T* __restrict__ v, T scale, int s0, int len,
                                 int32_t* __restrict__ cc, double* s) {
    const int lane = threadIdx.x % G;
    int p[U], c[U];
    T x[U];
    const uint32_t q = t0 + lane;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u < U - 1 || q + u * G < q1) p[u] = pos[q + u * G], c[u] = ci[q + u * G], x[u] = v[q + u * G];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = p[u] - s0;
        if ((u == U - 1 && q + u * G >= q1) || (!ALL && (unsigned)r >= (unsigned)len)) continue;
        cc[p[u]] = c[u];
        atomicAdd(&s[r], (double)(scale * x[u]));
    }
}

// All entries [q0, q1) so, up to four per lane together.
template <int G, bool ALL, typename T>
__device__ inline void add_entries(uint32_t q0, uint32_t q1, const int32_t* __restrict__ pos,
                                   const int32_t* __restrict__ ci, const T* __restrict__ v, T scale, int s0, int len,
                                   int32_t* __restrict__ cc, double* s) {
    for (uint32_t t0 = q0; t0 < q1; t0 += 4 * G) {  // (unsigned: the step behind a row's end may pass 2^31)
        const uint32_t left = q1 - t0;
        if (left > 3 * G) add_chunk<G, 4, ALL, T>(t0, q1, pos, ci, v, scale, s0, len, cc, s);
        else if (left > 2 * G) add_chunk<G, 3, ALL, T>(t0, q1, pos, ci, v, scale, s0, len, cc, s);
        else if (left > G) add_chunk<G, 2, ALL, T>(t0, q1, pos, ci, v, scale, s0, len, cc, s);
        else add_chunk<G, 1, ALL, T>(t0, q1, pos, ci, v, scale, s0, len, cc, s);
    }
}

template <typename T>
__global__ __launch_bounds__(WAVE * ROWS_PER_WG) void k_add_num(int32_t m, const int32_t* __restrict__ arp,
                                                                const int32_t* __restrict__ aci,
                                                                const T* __restrict__ av, const int32_t* __restrict__ brp,
                                                                const int32_t* __restrict__ bci,
                                                                const T* __restrict__ bv,
                                                                const int32_t* __restrict__ apos,
                                                                const int32_t* __restrict__ bpos,
                                                                const int32_t* __restrict__ crp, T alpha, T beta,
                                                                int32_t* __restrict__ ccol, T* __restrict__ cval) {
    __shared__ double acc[ROWS_PER_WG][NUM_CAP];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), lane = threadIdx.x % WAVE;
    double* s = acc[wv];
    constexpr int R = 2;
    const int64_t step = (int64_t)gridDim.x * ROWS_PER_WG * R;
    // pointers of rows i0 and i0 + 1 (a row past the end: the last, unused)
    struct Ptr {
        int as, ae, bs, be, c0, nc;
    };
    auto ptrs = [&](int64_t i) {
        i = i < m ? i : m - 1;
        Ptr p;
        p.as = arp[i], p.ae = arp[i + 1], p.bs = brp[i], p.be = brp[i + 1], p.c0 = crp[i], p.nc = crp[i + 1] - p.c0;
        return p;
    };
    int64_t i0 = ((int64_t)blockIdx.x * ROWS_PER_WG + wv) * R;
    Ptr nxt[R];
    for (int r = 0; r < R; ++r) nxt[r] = ptrs(i0 + r);
    for (; i0 < m; i0 += step) {
        Ptr p[R];
#pragma unroll
        for (int r = 0; r < R; ++r) p[r] = nxt[r], nxt[r] = ptrs(i0 + step + r);
        bool small = true;
#pragma unroll
        for (int r = 0; r < R; ++r) small &= p[r].ae - p[r].as + p[r].be - p[r].bs <= WAVE;
        if (!small) {
            for (int r = 0; r < R; ++r) {
                if (i0 + r >= m || p[r].nc > NUM_CAP) continue;
                for (int t = lane; t < p[r].nc; t += WAVE) s[t] = 0.0;
                wave_sync();
                add_entries<WAVE, true, T>(p[r].as, p[r].ae, apos, aci, av, alpha, 0, p[r].nc, ccol + p[r].c0, s);
                wave_sync();
                add_entries<WAVE, true, T>(p[r].bs, p[r].be, bpos, bci, bv, beta, 0, p[r].nc, ccol + p[r].c0, s);
                wave_sync();
                for (int t = lane; t < p[r].nc; t += WAVE) cval[p[r].c0 + t] = (T)s[t];
                wave_sync();
            }
            continue;
        }
        // one entry per lane and row: A's, then B's
        int pos[R], col[R];
        double v[R];
        bool in_a[R], has[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int la = p[r].ae - p[r].as, L = la + p[r].be - p[r].bs;
            in_a[r] = lane < la;
            has[r] = lane < L && i0 + r < m;
            pos[r] = 0, col[r] = 0, v[r] = 0.0;
            if (has[r]) {
                const int q = in_a[r] ? p[r].as + lane : p[r].bs + lane - la;
                pos[r] = (in_a[r] ? apos : bpos)[q];
                col[r] = (in_a[r] ? aci : bci)[q];
                v[r] = (double)((in_a[r] ? alpha : beta) * (in_a[r] ? av : bv)[q]);
            }
            s[r * WAVE + lane] = 0.0;
        }
        wave_sync();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (has[r] && in_a[r]) atomicAdd(&s[r * WAVE + pos[r]], v[r]);
        wave_sync();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (has[r] && !in_a[r]) atomicAdd(&s[r * WAVE + pos[r]], v[r]);
            if (has[r]) ccol[p[r].c0 + pos[r]] = col[r];
        }
        wave_sync();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (lane < p[r].nc && i0 + r < m) cval[p[r].c0 + lane] = (T)s[r * WAVE + lane];
        wave_sync();
    }
}

// Numeric rows of more than NUM_CAP columns, a workgroup each, `cap` columns at
// a time (what the longest row needs, at most WIDE_CAP, a quarter of the longest
// possible: fewer leave room for more workgroups); launched where there are
// such rows.  Every workgroup looks for them among m / grid rows, one per lane,
// spread over the matrix.  One wavefront per row walked it once per 512
// columns and, beyond 4096, summed in C's own storage; before that, beyond
// 1024.  FP64 rows of 3500 entries, 1700 of them / 11 thousand, in order and
// not, in us: 252 and 505 / 620 and 1353 so; 95 and 268 / 513 and 1862 before;
// 49 and 56 / 288 and 378 in this kernel.  Of 700 entries, 57 thousand: 351 and
// 522; 280 and 349; 262 and 327.
template <typename T>
__global__ __launch_bounds__(WIDE_THREADS) void k_add_num_wide(int32_t m, const int32_t* __restrict__ arp,
                                                               const int32_t* __restrict__ aci,
                                                               const T* __restrict__ av,
                                                               const int32_t* __restrict__ brp,
                                                               const int32_t* __restrict__ bci,
                                                               const T* __restrict__ bv,
                                                               const int32_t* __restrict__ apos,
                                                               const int32_t* __restrict__ bpos,
                                                               const int32_t* __restrict__ crp, T alpha, T beta,
                                                               int32_t* __restrict__ ccol, T* __restrict__ cval,
                                                               int cap) {
    constexpr int G = WIDE_THREADS;
    extern __shared__ double s[];
    __shared__ int32_t rows[G];
    __shared__ int count;
    const int tid = threadIdx.x;
    for (int64_t r0 = blockIdx.x; r0 < m; r0 += (int64_t)G * gridDim.x) {
        if (tid == 0) count = 0;
        __syncthreads();
        const int64_t i = r0 + (int64_t)tid * gridDim.x;
        if (i < m && crp[i + 1] - crp[i] > NUM_CAP) rows[atomicAdd(&count, 1)] = (int32_t)i;
        __syncthreads();
        for (int k = 0; k < count; ++k) {
            const int row = rows[k];
            const uint32_t as = arp[row], ae = arp[row + 1], bs = brp[row], be = brp[row + 1];
            const int c0 = crp[row], nc = crp[row + 1] - c0;
            int32_t* cc = ccol + c0;
            for (int s0 = 0; s0 < nc; s0 += cap) {
                const int len = min(cap, nc - s0);
                for (int t = tid; t < len; t += G) s[t] = 0.0;
                __syncthreads();
                if (nc <= cap) add_entries<G, true, T>(as, ae, apos, aci, av, alpha, s0, len, cc, s);
                else add_entries<G, false, T>(as, ae, apos, aci, av, alpha, s0, len, cc, s);
                __syncthreads();
                if (nc <= cap) add_entries<G, true, T>(bs, be, bpos, bci, bv, beta, s0, len, cc, s);
                else add_entries<G, false, T>(bs, be, bpos, bci, bv, beta, s0, len, cc, s);
                __syncthreads();
                for (int t = tid; t < len; t += G) cval[c0 + s0 + t] = (T)s[t];
                __syncthreads();
            }
        }
        __syncthreads();
    }
}

int64_t add_scan_tiles(int32_t m) { return ((int64_t)m + SCAN_TILE - 1) / SCAN_TILE; }

}  // namespace

struct spg_add_s {
    hipStream_t stream = nullptr;
    int n_cu = 256;
    std::string err;
    spg_dtype dt = SPG_F64;
    int32_t m = 0, n = 0;
    const int32_t *arp = nullptr, *aci = nullptr, *brp = nullptr, *bci = nullptr;
    int64_t annz = 0, bnnz = 0;
    int32_t* crp = nullptr;
    int64_t nnz_c = 0;
    bool have_sym = false;
    int32_t widest = 0;      // longest row of C of more than NUM_CAP columns (0: no such row)
    void* buf = nullptr;     // apos | bpos | row_nnz | long list | tile status | control
    size_t cap = 0;
    AddCtl* hctl = nullptr;  // pinned copy of the control block
    int32_t *apos = nullptr, *bpos = nullptr, *row_nnz = nullptr, *long_list = nullptr;
    uint64_t* tiles = nullptr;
    AddCtl* ctl = nullptr;
};

namespace {

spg_status afail(spg_add h, spg_status s, const std::string& msg) {
    if (h) h->err = msg;
    return s;
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

template <typename T>
void launch_num(spg_add h, T alpha, const void* a_vals, T beta, const void* b_vals, int32_t* c_col_idx, void* c_vals) {
    const T *av = static_cast<const T*>(a_vals), *bv = static_cast<const T*>(b_vals);
    T* cv = static_cast<T*>(c_vals);
    const int grid = (int)std::min<int64_t>(((int64_t)h->m + ROWS_PER_WG - 1) / ROWS_PER_WG, (int64_t)h->n_cu * 32);
    hipLaunchKernelGGL(k_add_num<T>, dim3(grid), dim3(WAVE * ROWS_PER_WG), 0, h->stream, h->m, h->arp, h->aci, av,
                       h->brp, h->bci, bv, h->apos, h->bpos, h->crp, alpha, beta, c_col_idx, cv);
    if (h->widest > 0) {
        int cap = 2 * NUM_CAP;
        while (cap < h->widest && cap < WIDE_CAP) cap *= 2;
        hipLaunchKernelGGL(k_add_num_wide<T>, dim3((unsigned)std::min(h->m, h->n_cu * 8)), dim3(WIDE_THREADS),
                           (size_t)cap * sizeof(double), h->stream, h->m, h->arp, h->aci, av, h->brp, h->bci, bv,
                           h->apos, h->bpos, h->crp, alpha, beta, c_col_idx, cv, cap);
    }
}

}  // namespace

extern "C" {

spg_status spg_add_create(spg_add* out, void* stream) {
    if (!out) return SPG_ERR_ARG;
    *out = nullptr;
    try {
        spg_add h = new spg_add_s();
        h->stream = static_cast<hipStream_t>(stream);
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&h->n_cu, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess) e = hipHostMalloc((void**)&h->hctl, sizeof(AddCtl), hipHostMallocDefault);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            delete h;
            return SPG_ERR_HIP;
        }
        *out = h;
        return SPG_OK;
    } catch (...) {
        return SPG_ERR_ALLOC;
    }
}

spg_status spg_add_destroy(spg_add h) {
    if (!h) return SPG_OK;
    (void)hipStreamSynchronize(h->stream);
    if (h->buf) (void)hipFree(h->buf);
    if (h->hctl) (void)hipHostFree(h->hctl);
    delete h;
    return SPG_OK;
}

const char* spg_add_last_error(spg_add h) { return h ? h->err.c_str() : "null handle"; }

spg_status spg_add_symbolic(spg_add h, int32_t m, int32_t n, const int32_t* a_row_ptr, const int32_t* a_col_idx,
                            int64_t a_nnz, const int32_t* b_row_ptr, const int32_t* b_col_idx, int64_t b_nnz,
                            int32_t* c_row_ptr, int64_t* nnz_c) {
    if (!h) return SPG_ERR_ARG;
    try {
        h->have_sym = false;
        if (m < 0 || n < 0 || a_nnz < 0 || b_nnz < 0) return afail(h, SPG_ERR_ARG, "negative dimension or nnz");
        if (a_nnz > INT32_MAX || b_nnz > INT32_MAX) return afail(h, SPG_ERR_ARG, "nnz exceeds int32 range");
        if (!a_row_ptr || !b_row_ptr || !c_row_ptr || !nnz_c) return afail(h, SPG_ERR_ARG, "null pointer");
        if ((a_nnz > 0 && !a_col_idx) || (b_nnz > 0 && !b_col_idx)) return afail(h, SPG_ERR_ARG, "null column index");
        if (n == 0 && (a_nnz > 0 || b_nnz > 0)) return afail(h, SPG_ERR_SHAPE, "entries but no columns");
        h->m = m, h->n = n;
        h->arp = a_row_ptr, h->aci = a_col_idx, h->annz = a_nnz;
        h->brp = b_row_ptr, h->bci = b_col_idx, h->bnnz = b_nnz;
        const size_t M = (size_t)std::max(m, 1);
        const size_t need = align256((size_t)std::max<int64_t>(a_nnz, 1) * 4) +
                            align256((size_t)std::max<int64_t>(b_nnz, 1) * 4) + 2 * align256(M * 4) +
                            align256((size_t)(add_scan_tiles(m) + 1) * 8) + align256(sizeof(AddCtl));
        if (need > h->cap) {
            if (h->buf) {
                if (hipStreamSynchronize(h->stream) != hipSuccess) return afail(h, SPG_ERR_HIP, "stream wait");
                (void)hipFree(h->buf);
                h->buf = nullptr, h->cap = 0;
            }
            if (hipMalloc(&h->buf, need) != hipSuccess) {
                (void)hipGetLastError();
                return afail(h, SPG_ERR_ALLOC, "device allocation of " + std::to_string(need) + " bytes failed");
            }
            h->cap = need;
        }
        uint8_t* p = static_cast<uint8_t*>(h->buf);
        h->apos = reinterpret_cast<int32_t*>(p), p += align256((size_t)std::max<int64_t>(a_nnz, 1) * 4);
        h->bpos = reinterpret_cast<int32_t*>(p), p += align256((size_t)std::max<int64_t>(b_nnz, 1) * 4);
        h->row_nnz = reinterpret_cast<int32_t*>(p), p += align256(M * 4);
        h->long_list = reinterpret_cast<int32_t*>(p), p += align256(M * 4);
        h->tiles = reinterpret_cast<uint64_t*>(p), p += align256((size_t)(add_scan_tiles(m) + 1) * 8);
        h->ctl = reinterpret_cast<AddCtl*>(p);
        hipStream_t s = h->stream;
        // the scan's tile states and the control block after them start from zero
        spg::launch_zero(s, h->tiles, (int64_t)(align256((size_t)(add_scan_tiles(m) + 1) * 8) + align256(sizeof(AddCtl))));
        if (m > 0) {
            // lanes per row: the fewest that hold most rows (up to a third
            // more entries than the average row; the others take a whole
            // wavefront each, which costs more than idle lanes)
            const int64_t total = (a_nnz + b_nnz) * 4 / 3;
            const int G = total <= (int64_t)16 * m ? 16 : total <= (int64_t)32 * m ? 32 : 64;
            const int64_t per_wg = (int64_t)ROWS_PER_WG * (WAVE / G) * 2;
            const int grid_rows = (int)std::min<int64_t>((m + per_wg - 1) / per_wg, (int64_t)h->n_cu * 32);
            const auto kernel = n <= KEY32_COLS ? (G == 16   ? k_add_sym<16, uint32_t>
                                                   : G == 32 ? k_add_sym<32, uint32_t>
                                                             : k_add_sym<64, uint32_t>)
                                                : (G == 16   ? k_add_sym<16, uint64_t>
                                                   : G == 32 ? k_add_sym<32, uint64_t>
                                                             : k_add_sym<64, uint64_t>);
            hipLaunchKernelGGL(kernel, dim3(grid_rows), dim3(WAVE * ROWS_PER_WG), 0, s, m, n, a_row_ptr, a_col_idx,
                               a_nnz, b_row_ptr, b_col_idx, b_nnz, h->apos, h->bpos, h->row_nnz, h->long_list, h->ctl);
            hipLaunchKernelGGL(k_add_sym_long, dim3((unsigned)std::min(h->n_cu, m)), dim3(LONG_THREADS),
                               (size_t)LONG_CAP * 8, s, n, a_row_ptr, a_col_idx, b_row_ptr, b_col_idx, h->apos,
                               h->bpos, h->row_nnz, h->long_list, h->ctl);
            hipLaunchKernelGGL(k_add_scan, dim3((unsigned)add_scan_tiles(m)), dim3(SCAN_THREADS), 0, s, m, h->row_nnz,
                               c_row_ptr, h->tiles, h->ctl);
        } else {
            spg::launch_fill_i32(s, c_row_ptr, 0, 1);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return afail(h, SPG_ERR_HIP, std::string("symbolic launch: ") + hipGetErrorString(e));
        if (hipMemcpyAsync(h->hctl, h->ctl, sizeof(AddCtl), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return afail(h, SPG_ERR_HIP, "control block read-back");
        const AddCtl c = *h->hctl;
        if (c.err & AE_ROWPTR) return afail(h, SPG_ERR_INDEX, "malformed row pointer in A or B");
        if (c.err & AE_COL) return afail(h, SPG_ERR_INDEX, "column index out of range in A or B");
        if (c.err & AE_LONG)
            return afail(h, SPG_ERR_UNSUPPORTED, "a row of A and B together holds more than " +
                                                     std::to_string(LONG_CAP) + " entries");
        if (c.err & AE_OVERFLOW) return afail(h, SPG_ERR_OVERFLOW, "nnz(C) exceeds the int32 range");
        h->nnz_c = m > 0 ? c.nnz_c : 0;
        h->widest = c.widest;
        h->crp = c_row_ptr;
        h->have_sym = true;
        *nnz_c = h->nnz_c;
        return SPG_OK;
    } catch (...) {
        return afail(h, SPG_ERR_HIP, "unexpected host exception");
    }
}

spg_status spg_add_numeric(spg_add h, spg_dtype dt, double alpha, const void* a_vals, double beta,
                           const void* b_vals, int32_t* c_col_idx, void* c_vals) {
    if (!h) return SPG_ERR_ARG;
    try {
        if (!h->have_sym) return afail(h, SPG_ERR_STATE, "spg_add_symbolic must come first");
        if (dt != SPG_F32 && dt != SPG_F64) return afail(h, SPG_ERR_ARG, "dtype must be SPG_F32 or SPG_F64");
        if ((h->annz > 0 && !a_vals) || (h->bnnz > 0 && !b_vals)) return afail(h, SPG_ERR_ARG, "null input values");
        if (h->nnz_c > 0 && (!c_col_idx || !c_vals)) return afail(h, SPG_ERR_ARG, "null output");
        if (h->m == 0) return SPG_OK;
        if (dt == SPG_F64) launch_num<double>(h, alpha, a_vals, beta, b_vals, c_col_idx, c_vals);
        else launch_num<float>(h, (float)alpha, a_vals, (float)beta, b_vals, c_col_idx, c_vals);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return afail(h, SPG_ERR_HIP, std::string("numeric launch: ") + hipGetErrorString(e));
        return SPG_OK;
    } catch (...) {
        return afail(h, SPG_ERR_HIP, "unexpected host exception");
    }
}

}  // extern "C"
