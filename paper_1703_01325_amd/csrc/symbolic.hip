// Symbolic phase on the device: the ILU(k) pattern P with the level of fill
// of every kept entry (Algorithm 3 with Eq 1-2) and the level sets of the
// four sweeps (Eq 4).  The results are the ones the host analysis computes.
//
// Pattern.  Eq 1-2 take the levels of row i from the finished rows p < i,
// one row after another.  The same levels have a per-row characterisation
// (the fill-path theorem of Hysom and Pothen, 2001): (i, j) is kept with
// level l exactly when the shortest path i -> ... -> j in the graph of A
// (edge u -> v for every stored block (u, v)) whose inner vertices are all
// below min(i, j) has l + 1 edges.  Every row is then independent of the
// others.  A group of lanes takes a row and runs k + 1 rounds of a
// Bellman-Ford search in the (min, max) semiring: M(v) is the smallest
// possible largest inner vertex over the paths i -> v of at most L edges
// whose inner vertices lie below i; a round extends by one edge the paths
// ending in the vertices u < i whose M dropped in the round before
// (M(v) <- min(M(v), max(M(u), u))), and v is kept with level L - 1 in the
// first round where M(v) < min(i, v).  The visited vertices live in a hash
// table in LDS, of a size for what rows of this k reach on grids; a row that
// outgrows it is searched again in a larger one, and one that reaches more
// than 3/4 kHash distinct vertices is refused.  A count pass sizes the rows, a scan gives
// the row pointers and a write pass repeats the search and emits each row in
// ascending column order (rank of each kept column among the row's).
//
// Level sets.  The level of a row is one more than the deepest row it reads
// (0 if none).  A persistent kernel takes 64 rows at a time, in sweep order,
// from a ticket; a lane polls the levels of the rows its row reads (-1 until
// published, read with device-coherent loads) and publishes its own once all
// are there.  Every row read lies earlier in sweep order, so the rows held
// by running wavefronts always include one that can finish and the launch
// drains.  The transposed sweeps read the columns of P, gathered into lists
// per column first.  level_rows is a stable radix sort of the rows by level
// (rows ascending inside a level), level_ptr the first position of each
// level.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <vector>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "bilu.h"
#include "bilu_internal.h"

namespace {

constexpr int kHash = 1024;          // hash slots of the largest row search; it may reach 3/4 as many vertices
// Up to this many rows a search is its launches and allocations: one launch with
// the largest table (7 points, one launch against small tables and lists: 15625
// rows k = 0 293 and 311 us; 8000 rows k = 1 306 and 355, k = 3 427 and 388; 4096
// rows k = 2 292 and 332, k = 4 371 and 320).
constexpr int few_rows(int k) { return 24000 / (2 * k + 1); }
constexpr unsigned short kKept = 0x8000u;
constexpr unsigned int kSpinLimit = 1u << 20;

// status bits of the symbolic kernels
constexpr int kStPattern = 1;        // unsorted / duplicate / out-of-range column
constexpr int kStDiag = 2;           // a row without its diagonal block
constexpr int kStTable = 4;          // a row search outgrew the hash table
constexpr int kStTimeout = 8;        // a level wait expired

__global__ void k_check_pattern(int nb, const int32_t* __restrict__ Ap, const int32_t* __restrict__ Aj,
                                int* status)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nb; i += gridDim.x * blockDim.x) {
        const int e0 = Ap[i], e1 = Ap[i + 1];
        if (e1 < e0) {
            atomicOr(status, kStPattern);
            continue;
        }
        bool diag = false;
        int prev = -1;
        for (int e = e0; e < e1; ++e) {
            const int j = Aj[e];
            if (j <= prev || j >= nb) {
                atomicOr(status, kStPattern);
                break;
            }
            diag |= (j == i);
            prev = j;
        }
        if (!diag) atomicOr(status, kStDiag);
    }
}

// (and the entry count, status[1])
__global__ void k_check_ptr(int nb, const int32_t* __restrict__ Ap, int* status)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) status[1] = Ap[nb];
    if (blockIdx.x == 0 && threadIdx.x == 0 && Ap[0] != 0) atomicOr(status, kStPattern);
}

template <int SLOTS>
struct RowTable {
    int key[SLOTS];              // vertex, -1 empty
    int mval[SLOTS];             // M after the last round
    int mnext[SLOTS];            // running minimum of the candidates
    unsigned short info[SLOTS];  // kKept | level
    unsigned short list[SLOTS];  // frontier slots / kept slots
    int nlist;
    int nused;
    int over;
};

// log2 of a table size
constexpr int slot_bits(int slots) { return slots <= 1 ? 0 : 1 + slot_bits(slots / 2); }

template <int SLOTS>
__device__ __forceinline__ int table_slot(RowTable<SLOTS>& t, int v)
{
    unsigned int h = (static_cast<unsigned int>(v) * 2654435761u) >> (32 - slot_bits(SLOTS));
    // (no further than this, so that the vertices in flight when a table is given up
    // do not probe all of a full one; the largest is probed to its end)
    constexpr int kProbes = SLOTS < kHash && SLOTS > 64 ? 64 : SLOTS;
    for (int probe = 0; probe < kProbes; ++probe) {
        const int old = atomicCAS(&t.key[h], -1, v);
        if (old == v) return static_cast<int>(h);
        if (old == -1) {
            if (atomicAdd(&t.nused, 1) >= SLOTS / 4 * 3) t.over = 1;
            return static_cast<int>(h);
        }
        h = (h + 1) & (SLOTS - 1);
    }
    t.over = 1;
    return -1;
}

// LANES lanes per row, 64 / LANES rows per wavefront, a table of SLOTS slots
// each.  rows == nullptr: all nb rows, else the *nrows listed ones.  WRITE =
// false: cnt[i] = kept entries of row i; WRITE = true: row i written at Pp[i]
// in ascending columns.  A row that outgrows its table goes on the list
// over_rows, or is refused if there is none.
//
// The searches wait on LDS and on the pattern's rows; what counts is how many
// are in flight, and clearing and scanning the table is most of a small one's
// work.  60x220x85, 7 points, k = 1: one row per wavefront in a table of 1024
// slots (8 wavefronts fit a compute unit's LDS) took 5170 us to count and
// 5630 us to write; four rows per wavefront in tables of 64 slots (32
// wavefronts a compute unit) take 239 and 267 us.
template <int SLOTS, int LANES, bool WRITE>
__global__ __launch_bounds__(64) void k_sym_rows(int nb, const int32_t* __restrict__ rows,
                                                 const int* __restrict__ nrows, const int32_t* __restrict__ Ap,
                                                 const int32_t* __restrict__ Aj, int k, int32_t* __restrict__ cnt,
                                                 const int32_t* __restrict__ Pp, int32_t* __restrict__ Pj,
                                                 int32_t* __restrict__ Plev, int32_t* __restrict__ over_rows,
                                                 int* __restrict__ over_count, int* status)
{
    constexpr int kRows = 64 / LANES;
    constexpr int kEdges = 4;            // lanes along the row of one frontier vertex
    __shared__ RowTable<SLOTS> table[kRows];
    const int lane = threadIdx.x % LANES;
    const int group = threadIdx.x / LANES;
    RowTable<SLOTS>& t = table[group];
    const int n = rows ? *nrows : nb;
    for (int64_t q0 = static_cast<int64_t>(blockIdx.x) * kRows; q0 < n; q0 += static_cast<int64_t>(gridDim.x) * kRows) {
        const bool live = q0 + group < n;
        const int i = !live ? 0 : rows ? rows[q0 + group] : static_cast<int>(q0) + group;
        __syncthreads();
        for (int s = lane; s < SLOTS; s += LANES) {
            t.key[s] = -1;
            t.mval[s] = INT_MAX;
            t.mnext[s] = INT_MAX;
            t.info[s] = 0;
        }
        if (lane == 0) {
            t.nlist = 0;
            t.nused = 0;
            t.over = 0;
        }
        __syncthreads();
        // row i of A: level 0, no inner vertex (M = -1)
        // (a table given up is not searched on: every vertex more would probe all
        // of a full one)
        if (live && Ap[i + 1] - Ap[i] > SLOTS / 4 * 3) {
            if (lane == 0) t.over = 1;
        } else if (live) {
            for (int e = Ap[i] + lane; e < Ap[i + 1]; e += LANES) {
                const int v = Aj[e];
                const int s = table_slot(t, v);
                if (s < 0) continue;
                t.mval[s] = -1;
                t.mnext[s] = -1;
                t.info[s] = kKept;
                if (v < i) t.list[atomicAdd(&t.nlist, 1)] = static_cast<unsigned short>(s);
            }
        }
        __syncthreads();
        for (int L = 2; L <= k + 1; ++L) {
            const int nf = t.over ? 0 : t.nlist;
            if (!__any(nf)) break;
            // extend the paths ending in the frontier by one edge of A
            for (int f = lane / kEdges; f < nf; f += LANES / kEdges) {
                if (__hip_atomic_load(&t.over, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
                const int su = t.list[f];
                const int u = t.key[su];
                const int mu = max(t.mval[su], u);
                const int e1 = Ap[u + 1];
                for (int e = Ap[u] + lane % kEdges; e < e1; e += kEdges) {
                    const int s = table_slot(t, Aj[e]);
                    if (s >= 0) atomicMin(&t.mnext[s], mu);
                }
            }
            __syncthreads();
            if (lane == 0) t.nlist = 0;
            __syncthreads();
            // fold the round in; the next frontier: vertices below i whose M dropped
            for (int s = lane; s < SLOTS; s += LANES) {
                const int v = t.key[s];
                if (v >= 0 && t.mnext[s] < t.mval[s]) {
                    const int m = t.mnext[s];
                    t.mval[s] = m;
                    if (!(t.info[s] & kKept) && m < min(i, v)) t.info[s] = static_cast<unsigned short>(kKept | (L - 1));
                    if (v < i) t.list[atomicAdd(&t.nlist, 1)] = static_cast<unsigned short>(s);
                }
            }
            __syncthreads();
        }
        const bool over = t.over != 0;
        if (over && live && lane == 0) {
            if (over_rows)
                over_rows[atomicAdd(over_count, 1)] = i;
            else
                atomicOr(status, kStTable);
        }
        __syncthreads();
        if (lane == 0) t.nlist = 0;
        __syncthreads();
        // the kept entries: columns into mnext[], levels into mval[]
        int col[SLOTS / LANES], lev[SLOTS / LANES];
#pragma unroll
        for (int u = 0; u < SLOTS / LANES; ++u) {
            const int s = u * LANES + lane;
            col[u] = (t.info[s] & kKept) ? t.key[s] : -1;
            lev[u] = t.info[s] & 0xff;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < SLOTS / LANES; ++u) {
            if (col[u] >= 0) {
                const int q = atomicAdd(&t.nlist, 1);
                t.mnext[q] = col[u];
                t.mval[q] = lev[u];
            }
        }
        __syncthreads();
        const int nk = live && !over ? t.nlist : 0;
        if (!WRITE) {
            if (live && !over && lane == 0) cnt[i] = nk;
            continue;
        }
        const int base = live ? Pp[i] : 0;
        for (int q = lane; q < nk; q += LANES) {
            const int c = t.mnext[q];
            int rank = 0;
            for (int f = 0; f < nk; ++f) rank += t.mnext[f] < c;
            Pj[base + rank] = c;
            Plev[base + rank] = t.mval[q];
        }
    }
}

__global__ void k_narrow_ptr(int n1, const int64_t* __restrict__ in, int32_t* __restrict__ out)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n1; i += gridDim.x * blockDim.x)
        out[i] = static_cast<int32_t>(in[i]);
}

__device__ __forceinline__ int coherent_load_i(const int* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void coherent_store_i(int* p, int v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Level of every row (Eq 4) for one sweep.  Row r reads the rows idx[e],
// e in [ptr[r], ptr[r+1]) that pass the filter: mode 0 below r, mode 1
// above r, mode 2 all.  forward: sweep order is ascending rows.
//
// A chain of dependent rows: what counts is the time from a level's store to
// the store of the level above it.  So a lane lists the rows it reads in LDS
// before it waits (the far ones first) and holds the next kLevelSlots of
// them in registers; a round loads the levels of all of those that are still
// pending at once; a dependency on a row of the same wavefront is read from
// LDS, and chains inside the wavefront advance there without a round trip
// through memory.  A dependency found published is never read again.  On a
// grid numbered line by line the rows held by running wavefronts are the
// window in which the chains of different lines overlap: 16 wavefronts a
// compute unit; 12 lose to the window, 32 to each other's polls.  Wavefronts
// in which nothing moved sleep between rounds.
// Level sets of L on 60x220x85, 7 points, in ms: k = 0, 1, 2 (363, 750 and
// 1305 levels) 6.5, 13.4 and 24.5 with the lists read again from memory in
// every round by 8 wavefronts a compute unit, 1.6, 2.4 and 3.6 so; with 8
// wavefronts of this kernel 2.4, 3.6 and 5.5, with 32 2.0, 3.4 and 5.5.
constexpr int kLevelSlots = 12;      // rows polled at once
constexpr int kLevelStage = 36;      // rows listed before the first wait: ILU(4) on 7 points reads 35

// Lists of columns (LISTS) come in the order in which k_col_fill's atomics hand
// out places, about ascending, and a wait for the first entries of a long list
// leaves the others to be read when it is over.  There the near rows come first
// once a list has more than one round's entries, and of the rows that do not fit
// the first kLevelStage those already published are not listed at all.  L^T, 27
// points, 10^3, k = 2 and 3 (rows that read up to 57 and 91): 1.53 and 2.43 ms
// with a cursor in the list, 3.34 and 6.74 ms far first and listed, 1.08 and
// 1.77 ms so; 7 points, 60^3, k = 4, 14.0, 18.9 and 7.5 ms.
template <bool LISTS>
__global__ __launch_bounds__(256, 4) void k_levels(int nb, const int32_t* __restrict__ ptr,
                                                   const int32_t* __restrict__ idx, int mode, int forward, int* lvl,
                                                   unsigned int* ticket, int* status)
{
    constexpr int kFetch = LISTS ? 8 : 4;
    __shared__ int wl[4][64];
    __shared__ int wstage[4][kLevelStage][64];
    const int lane = threadIdx.x & 63;
    int* mine = wl[threadIdx.x >> 6];
    int (*stage)[64] = wstage[threadIdx.x >> 6];
    for (;;) {
        unsigned int tk = 0;
        if (lane == 0) tk = atomicAdd(ticket, 1u);
        tk = __shfl(tk, 0);
        if (static_cast<int64_t>(tk) * 64 >= nb) break;
        const int pos0 = static_cast<int>(tk) * 64;
        const int pos = pos0 + lane;
        const int row = pos < nb ? (forward ? pos : nb - 1 - pos) : -1;
        bool done = row < 0;
        mine[lane] = -1;
        int e = done ? 0 : ptr[row];
        const int e1 = done ? 0 : ptr[row + 1];
        const int ends = e + e1 - 1;
        const bool turned = (forward == 0) != (LISTS && e1 - e > kLevelSlots);
        bool again = false;            // entries were listed before
        int best = -1;
        int dep[kLevelSlots];          // a row of another wavefront, or a lane of this one
        unsigned int pend = 0, local = 0, slots = 0;
        int staged = 0, taken = 0;
        // the next entries that pass, into the stage
        auto fetch = [&]() {
            staged = taken = 0;
            while (e < e1 && staged < kLevelStage) {
                int j[kFetch], lv[kFetch];
#pragma unroll
                for (int u = 0; u < kFetch; ++u) {
                    const int at = min(e + u, e1 - 1);
                    j[u] = idx[turned ? ends - at : at];
                    lv[u] = -1;
                }
                if (LISTS && again) {
#pragma unroll
                    for (int u = 0; u < kFetch; ++u) lv[u] = coherent_load_i(lvl + j[u]);
                }
#pragma unroll
                for (int u = 0; u < kFetch; ++u) {
                    if (e < e1 && staged < kLevelStage) {
                        if (LISTS && lv[u] != -1) best = max(best, lv[u]);
                        else if (LISTS || (mode == 0 ? j[u] < row : j[u] > row)) stage[staged++][lane] = j[u];
                        ++e;
                    }
                }
            }
            again = true;
        };
        // the next of the stage, into registers
        auto refill = [&]() {
            if (taken == staged && e < e1) fetch();
            const int c = min(staged - taken, kLevelSlots);
            pend = (1u << c) - 1u;
            local = 0;
#pragma unroll
            for (int u = 0; u < kLevelSlots; ++u) {
                const int j = u < c ? stage[taken + u][lane] : 0;
                const int l = (forward ? j : nb - 1 - j) - pos0;
                const bool in = u < c && l >= 0 && l < 64;
                dep[u] = in ? l : j;
                if (in) local |= 1u << u;
            }
            taken += c;
        };
        if (!done) refill();
        unsigned int spins = 0;
        bool fresh = true;
        for (;;) {
            bool moved = false;
            // rows of other wavefronts: every pending level at once
            int lv[kLevelSlots];
            const unsigned int far = pend & ~local;
#pragma unroll
            for (int u = 0; u < kLevelSlots; ++u) lv[u] = (far >> u & 1u) ? coherent_load_i(lvl + dep[u]) : -1;
#pragma unroll
            for (int u = 0; u < kLevelSlots; ++u) {
                if (lv[u] != -1) {
                    best = max(best, lv[u]);
                    pend &= ~(1u << u);
                    moved = true;
                }
            }
            // rows of this one, until nothing moves
            for (;;) {
                if (fresh) {
                    slots = 0;
#pragma unroll
                    for (int u = 0; u < kLevelSlots; ++u) slots |= __any(local >> u & 1u) ? 1u << u : 0u;
                    fresh = false;
                }
#pragma unroll
                for (int u = 0; u < kLevelSlots; ++u) {
                    if (slots >> u & 1u) {
                        const int l = (pend & local) >> u & 1u ? mine[dep[u]] : -1;
                        if (l != -1) {
                            best = max(best, l);
                            pend &= ~(1u << u);
                        }
                    }
                }
                bool step = false;
                if (!done && pend == 0) {
                    if (taken < staged || e < e1) {
                        refill();
                        fresh = true;
                    }
                    if (pend == 0) {
                        mine[lane] = best + 1;
                        coherent_store_i(lvl + row, best + 1);
                        done = true;
                    }
                    step = true;
                }
                fresh = __any(fresh);
                if (!__any(step)) break;
                moved = true;
                __builtin_amdgcn_wave_barrier();
                asm volatile("" ::: "memory");
            }
            if (__all(done)) break;
            if (!__any(moved)) {
                if (++spins > kSpinLimit) {
                    atomicOr(status, kStTimeout);
                    return;
                }
                __builtin_amdgcn_s_sleep(8);
            }
        }
    }
}

// Column lists of the transposed sweeps: entry (i, j) of P with j > i
// (upper = 1: U'^T, row j reads row i) or j < i (upper = 0: L^T, row j
// reads row i) adds i to the list of j.
__global__ void k_col_count(int nb, const int32_t* __restrict__ Pp, const int32_t* __restrict__ Pj, int upper,
                            int32_t* cnt)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nb; i += gridDim.x * blockDim.x)
        for (int e = Pp[i]; e < Pp[i + 1]; ++e) {
            const int j = Pj[e];
            if (upper ? j > i : j < i) atomicAdd(cnt + j, 1);
        }
}

__global__ void k_col_fill(int nb, const int32_t* __restrict__ Pp, const int32_t* __restrict__ Pj, int upper,
                           int32_t* cursor, int32_t* __restrict__ cidx)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nb; i += gridDim.x * blockDim.x)
        for (int e = Pp[i]; e < Pp[i + 1]; ++e) {
            const int j = Pj[e];
            if (upper ? j > i : j < i) cidx[atomicAdd(cursor + j, 1)] = i;
        }
}

__global__ void k_iota_max(int nb, const int32_t* __restrict__ lvl, int32_t* __restrict__ rows, int* nlev)
{
    int m = 0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nb; i += gridDim.x * blockDim.x) {
        rows[i] = i;
        m = max(m, lvl[i] + 1);
    }
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) atomicMax(nlev, m);
}

// level_ptr[l] = first position of the sorted keys with key >= l.
__global__ void k_level_ptr(int nb, const int32_t* __restrict__ keys, int nlev, int32_t* __restrict__ level_ptr)
{
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p <= nb; p += gridDim.x * blockDim.x) {
        const int lo = p == 0 ? -1 : keys[p - 1];
        const int hi = p == nb ? nlev : keys[p];
        for (int l = lo + 1; l <= hi && l <= nlev; ++l) level_ptr[l] = p;
    }
}

// Device scratch released on every exit path.
struct Scratch {
    std::vector<void*> ptrs;
    ~Scratch()
    {
        for (void* p : ptrs) (void)hipFree(p);
    }
    template <typename T>
    T* get(size_t n)
    {
        void* p = nullptr;
        if (hipMalloc(&p, std::max<size_t>(n, 1) * sizeof(T)) != hipSuccess) return nullptr;
        ptrs.push_back(p);
        return static_cast<T*>(p);
    }
};

int grid_for(int64_t n, int threads, int cap = 4096)
{
    return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>((n + threads - 1) / threads, cap)));
}

bilu_status status_to_error(int st)
{
    if (st & kStTimeout) return BILU_ERR_TIMEOUT;
    if (st & kStPattern) return BILU_ERR_PATTERN;
    if (st & kStDiag) return BILU_ERR_MISSING_DIAG;
    if (st & kStTable) return BILU_ERR_ALLOC;
    return BILU_OK;
}

#define CKH(call)                                       \
    do {                                                \
        if ((call) != hipSuccess) return BILU_ERR_HIP; \
    } while (0)

// Searches all rows: first in tables for what a row is expected to reach (a
// table takes 3/4 of its slots), the rows that outgrow them in larger ones.  On a
// 7-point grid a row reaches 7, 19, 43, 86 and 151 vertices for k = 0 to 4, 0.7
// times those within k + 1 steps, on a 27-point grid about 0.65 times the cube of
// that radius; a pattern is taken for the one or the other by its entries a row,
// and to spread in proportion to them.  A first guess too low costs the searches
// up to where the table is given up: 27 points, 30^3, k = 2, in tables of 256
// slots first 2152 us, in the largest at once 1447 us.
template <bool WRITE>
bilu_status search_rows(int nb, int64_t nnz, const int32_t* Ap, const int32_t* Aj, int k, int32_t* cnt,
                        const int32_t* Pp, int32_t* Pj, int32_t* Plev, int* d_status, Scratch& sc, hipStream_t s)
{
    if (nb <= few_rows(k)) {
        k_sym_rows<kHash, 64, WRITE><<<nb, 64, 0, s>>>(nb, nullptr, nullptr, Ap, Aj, k, cnt, Pp, Pj, Plev, nullptr,
                                                       nullptr, d_status);
        return BILU_OK;
    }
    const double steps = k + 1.0;
    const double side = 2.0 * steps + 1.0, mean = static_cast<double>(nnz) / nb;
    const double reach = mean <= 13.0 ? 0.1 * mean * side * (2.0 * steps * steps + 2.0 * steps + 3.0) / 3.0
                                      : 0.65 * mean * (side / 3.0) * (side / 3.0) * (side / 3.0);
    int* over = sc.get<int>(2 + 2 * static_cast<size_t>(nb));     // lengths of the two lists, and these
    if (!over) return BILU_ERR_ALLOC;
    int32_t* list1 = over + 2;
    int32_t* list2 = list1 + nb;
    CKH(hipMemsetAsync(over, 0, 2 * sizeof(int), s));
    const auto grid = [nb](int rows) { return std::min((nb + rows - 1) / rows, 65536); };
    if (reach <= 48)
        k_sym_rows<64, 16, WRITE><<<grid(4), 64, 0, s>>>(nb, nullptr, nullptr, Ap, Aj, k, cnt, Pp, Pj, Plev, list1,
                                                         over, d_status);
    else if (reach <= 96)
        k_sym_rows<128, 32, WRITE><<<grid(2), 64, 0, s>>>(nb, nullptr, nullptr, Ap, Aj, k, cnt, Pp, Pj, Plev, list1,
                                                          over, d_status);
    const bool all256 = reach > 96 && reach <= 192, all = reach > 192;
    if (!all)
        k_sym_rows<256, 64, WRITE><<<std::min(nb, all256 ? 65536 : 8192), 64, 0, s>>>(
            nb, all256 ? nullptr : list1, over, Ap, Aj, k, cnt, Pp, Pj, Plev, list2, over + 1, d_status);
    k_sym_rows<kHash, 64, WRITE><<<std::min(nb, all ? 65536 : 2048), 64, 0, s>>>(
        nb, all ? nullptr : list2, over + 1, Ap, Aj, k, cnt, Pp, Pj, Plev, nullptr, nullptr, d_status);
    return BILU_OK;
}

// Checks the pattern, sizes the rows and writes the row pointers; *nnzb
// receives the entry count, *nnzA that of A.
bilu_status sym_count(int nb, const int32_t* Ap, const int32_t* Aj, int k, int32_t* Pp, int64_t* nnzb, int32_t* nnzA,
                      hipStream_t s)
{
    Scratch sc;
    int* d_status = sc.get<int>(2);
    int32_t* cnt = sc.get<int32_t>(static_cast<size_t>(nb) + 1);
    int64_t* ptr64 = sc.get<int64_t>(static_cast<size_t>(nb) + 1);
    if (!d_status || !cnt || !ptr64) return BILU_ERR_ALLOC;
    CKH(hipMemsetAsync(d_status, 0, sizeof(int), s));
    CKH(hipMemsetAsync(cnt + nb, 0, sizeof(int32_t), s));
    k_check_ptr<<<1, 64, 0, s>>>(nb, Ap, d_status);
    k_check_pattern<<<grid_for(nb, 256), 256, 0, s>>>(nb, Ap, Aj, d_status);
    int h_small[2] = {0, 0}, h_status = 0;
    CKH(hipMemcpyAsync(h_small, d_status, 2 * sizeof(int), hipMemcpyDeviceToHost, s));
    CKH(hipStreamSynchronize(s));
    if (h_small[0]) return status_to_error(h_small[0]);
    *nnzA = h_small[1];
    const bilu_status st = search_rows<false>(nb, *nnzA, Ap, Aj, k, cnt, nullptr, nullptr, nullptr, d_status, sc, s);
    if (st != BILU_OK) return st;
    size_t tmp_bytes = 0;
    if (rocprim::exclusive_scan(nullptr, tmp_bytes, cnt, ptr64, int64_t(0), static_cast<size_t>(nb) + 1,
                                rocprim::plus<int64_t>(), s) != hipSuccess)
        return BILU_ERR_HIP;
    void* tmp = sc.get<unsigned char>(tmp_bytes);
    if (!tmp) return BILU_ERR_ALLOC;
    if (rocprim::exclusive_scan(tmp, tmp_bytes, cnt, ptr64, int64_t(0), static_cast<size_t>(nb) + 1,
                                rocprim::plus<int64_t>(), s) != hipSuccess)
        return BILU_ERR_HIP;
    int64_t total = 0;
    CKH(hipMemcpyAsync(&total, ptr64 + nb, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    CKH(hipMemcpyAsync(&h_status, d_status, sizeof(int), hipMemcpyDeviceToHost, s));
    CKH(hipStreamSynchronize(s));
    if (h_status) return status_to_error(h_status);
    if (total > INT32_MAX) return BILU_ERR_ALLOC;
    k_narrow_ptr<<<grid_for(nb + 1, 256), 256, 0, s>>>(nb + 1, ptr64, Pp);
    CKH(hipStreamSynchronize(s));
    *nnzb = total;
    return BILU_OK;
}

// Writes the rows at the pointers sym_count produced.
bilu_status sym_write(int nb, int32_t nnzA, const int32_t* Ap, const int32_t* Aj, int k, const int32_t* Pp, int32_t* Pj,
                      int32_t* Plev, hipStream_t s)
{
    Scratch sc;
    int* d_status = sc.get<int>(1);
    if (!d_status) return BILU_ERR_ALLOC;
    CKH(hipMemsetAsync(d_status, 0, sizeof(int), s));
    const bilu_status st = search_rows<true>(nb, nnzA, Ap, Aj, k, nullptr, Pp, Pj, Plev, d_status, sc, s);
    if (st != BILU_OK) return st;
    int h_status = 0;
    CKH(hipMemcpyAsync(&h_status, d_status, sizeof(int), hipMemcpyDeviceToHost, s));
    CKH(hipStreamSynchronize(s));
    return status_to_error(h_status);
}

bilu_status levels_impl(int nb, const int32_t* Pp, const int32_t* Pj, int sweep, int32_t* lvl, int32_t* level_ptr,
                        int32_t* level_rows, int* nlev, hipStream_t s)
{
    Scratch sc;
    int* d_small = sc.get<int>(4);   // status, nlev, ticket
    if (!d_small) return BILU_ERR_ALLOC;
    CKH(hipMemsetAsync(d_small, 0, 4 * sizeof(int), s));
    CKH(hipMemsetAsync(lvl, 0xff, static_cast<size_t>(nb) * sizeof(int32_t), s));
    const int32_t* ptr = Pp;
    const int32_t* idx = Pj;
    int mode = 0;
    const bool forward = (sweep == BILU_SWEEP_L || sweep == BILU_SWEEP_UT);
    if (sweep == BILU_SWEEP_U) {
        mode = 1;
    } else if (sweep == BILU_SWEEP_UT || sweep == BILU_SWEEP_LT) {
        const int upper = sweep == BILU_SWEEP_UT;
        int32_t* ccnt = sc.get<int32_t>(static_cast<size_t>(nb) + 1);
        int64_t* cptr64 = sc.get<int64_t>(static_cast<size_t>(nb) + 1);
        int32_t* cptr = sc.get<int32_t>(static_cast<size_t>(nb) + 1);
        int32_t* cursor = sc.get<int32_t>(static_cast<size_t>(nb) + 1);
        if (!ccnt || !cptr64 || !cptr || !cursor) return BILU_ERR_ALLOC;
        CKH(hipMemsetAsync(ccnt, 0, (static_cast<size_t>(nb) + 1) * sizeof(int32_t), s));
        k_col_count<<<grid_for(nb, 256), 256, 0, s>>>(nb, Pp, Pj, upper, ccnt);
        size_t tmp_bytes = 0;
        if (rocprim::exclusive_scan(nullptr, tmp_bytes, ccnt, cptr64, int64_t(0), static_cast<size_t>(nb) + 1,
                                    rocprim::plus<int64_t>(), s) != hipSuccess)
            return BILU_ERR_HIP;
        void* tmp = sc.get<unsigned char>(tmp_bytes);
        if (!tmp) return BILU_ERR_ALLOC;
        if (rocprim::exclusive_scan(tmp, tmp_bytes, ccnt, cptr64, int64_t(0), static_cast<size_t>(nb) + 1,
                                    rocprim::plus<int64_t>(), s) != hipSuccess)
            return BILU_ERR_HIP;
        int64_t total = 0;
        CKH(hipMemcpyAsync(&total, cptr64 + nb, sizeof(int64_t), hipMemcpyDeviceToHost, s));
        CKH(hipStreamSynchronize(s));
        int32_t* cidx = sc.get<int32_t>(static_cast<size_t>(total));
        if (!cidx) return BILU_ERR_ALLOC;
        k_narrow_ptr<<<grid_for(nb + 1, 256), 256, 0, s>>>(nb + 1, cptr64, cptr);
        CKH(hipMemcpyAsync(cursor, cptr, (static_cast<size_t>(nb) + 1) * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
        k_col_fill<<<grid_for(nb, 256), 256, 0, s>>>(nb, Pp, Pj, upper, cursor, cidx);
        ptr = cptr;
        idx = cidx;
        mode = 2;
    }
    // persistent: at most as many wavefronts as there are row groups
    const int groups = static_cast<int>((static_cast<int64_t>(nb) + 63) / 64);
    const int wg = std::max(1, std::min((groups + 3) / 4, 1024));
    unsigned int* ticket = reinterpret_cast<unsigned int*>(d_small + 2);
    if (mode == 2) k_levels<true><<<wg, 256, 0, s>>>(nb, ptr, idx, mode, forward ? 1 : 0, lvl, ticket, d_small);
    else k_levels<false><<<wg, 256, 0, s>>>(nb, ptr, idx, mode, forward ? 1 : 0, lvl, ticket, d_small);
    int32_t* rows_in = sc.get<int32_t>(static_cast<size_t>(nb));
    int32_t* keys_out = sc.get<int32_t>(static_cast<size_t>(nb));
    if (!rows_in || !keys_out) return BILU_ERR_ALLOC;
    k_iota_max<<<grid_for(nb, 256, 1024), 256, 0, s>>>(nb, lvl, rows_in, d_small + 1);
    int h_small[2] = {0, 0};
    CKH(hipMemcpyAsync(h_small, d_small, 2 * sizeof(int), hipMemcpyDeviceToHost, s));
    CKH(hipStreamSynchronize(s));
    if (h_small[0]) return status_to_error(h_small[0]);
    const int nl = h_small[1];
    int bits = 1;
    while (bits < 31 && (1 << bits) < nl) ++bits;
    size_t tmp_bytes = 0;
    const unsigned int* kin = reinterpret_cast<const unsigned int*>(lvl);
    unsigned int* kout = reinterpret_cast<unsigned int*>(keys_out);
    if (rocprim::radix_sort_pairs(nullptr, tmp_bytes, kin, kout, rows_in, level_rows, static_cast<unsigned int>(nb),
                                  0, bits, s) != hipSuccess)
        return BILU_ERR_HIP;
    void* tmp = sc.get<unsigned char>(tmp_bytes);
    if (!tmp) return BILU_ERR_ALLOC;
    if (rocprim::radix_sort_pairs(tmp, tmp_bytes, kin, kout, rows_in, level_rows, static_cast<unsigned int>(nb), 0,
                                  bits, s) != hipSuccess)
        return BILU_ERR_HIP;
    k_level_ptr<<<grid_for(nb + 1, 256), 256, 0, s>>>(nb, keys_out, nl, level_ptr);
    CKH(hipStreamSynchronize(s));
    *nlev = nl;
    return BILU_OK;
}

}  // namespace

namespace bilu {

// Host-vector form used by bilu_analyze with BILU_DEVICE_SYMBOLIC: copies the
// pattern to the current device, runs the symbolic phase and the requested
// level sets there and copies the results back.
int device_analysis(int nb, const int32_t* Ap, const int32_t* Aj, int k, int nsweeps, std::vector<int32_t>& Pp,
                    std::vector<int32_t>& Pj, std::vector<int32_t>& Plev, std::vector<int32_t> (&lvl)[4])
{
    Scratch sc;
    hipStream_t s = nullptr;
    const int64_t nA = Ap[nb];
    int32_t* dAp = sc.get<int32_t>(static_cast<size_t>(nb) + 1);
    int32_t* dAj = sc.get<int32_t>(static_cast<size_t>(nA));
    int32_t* dPp = sc.get<int32_t>(static_cast<size_t>(nb) + 1);
    if (!dAp || !dAj || !dPp) return BILU_ERR_ALLOC;
    CKH(hipMemcpy(dAp, Ap, (static_cast<size_t>(nb) + 1) * sizeof(int32_t), hipMemcpyHostToDevice));
    CKH(hipMemcpy(dAj, Aj, static_cast<size_t>(nA) * sizeof(int32_t), hipMemcpyHostToDevice));
    int64_t nnz = 0;
    int32_t nnzA = 0;
    bilu_status st = sym_count(nb, dAp, dAj, k, dPp, &nnz, &nnzA, s);
    if (st != BILU_OK) return st;
    int32_t* dPj = sc.get<int32_t>(static_cast<size_t>(nnz));
    int32_t* dPl = sc.get<int32_t>(static_cast<size_t>(nnz));
    if (!dPj || !dPl) return BILU_ERR_ALLOC;
    st = sym_write(nb, nnzA, dAp, dAj, k, dPp, dPj, dPl, s);
    if (st != BILU_OK) return st;
    Pp.resize(static_cast<size_t>(nb) + 1);
    Pj.resize(static_cast<size_t>(nnz));
    Plev.resize(static_cast<size_t>(nnz));
    CKH(hipMemcpy(Pp.data(), dPp, Pp.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    CKH(hipMemcpy(Pj.data(), dPj, Pj.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    CKH(hipMemcpy(Plev.data(), dPl, Plev.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    int32_t* dl = sc.get<int32_t>(static_cast<size_t>(nb));
    int32_t* dptr = sc.get<int32_t>(static_cast<size_t>(nb) + 1);
    int32_t* drows = sc.get<int32_t>(static_cast<size_t>(nb));
    if (!dl || !dptr || !drows) return BILU_ERR_ALLOC;
    for (int w = 0; w < 4; ++w) {
        lvl[w].clear();
        if (w >= nsweeps) continue;
        int nl = 0;
        st = levels_impl(nb, dPp, dPj, w, dl, dptr, drows, &nl, s);
        if (st != BILU_OK) return st;
        lvl[w].resize(static_cast<size_t>(nb));
        CKH(hipMemcpy(lvl[w].data(), dl, static_cast<size_t>(nb) * sizeof(int32_t), hipMemcpyDeviceToHost));
    }
    return BILU_OK;
}

}  // namespace bilu

extern "C" {

bilu_status bilu_symbolic_device(int nb, const int32_t* Ap, const int32_t* Aj, int k, int32_t* Pp, int32_t* Pj,
                                 int32_t* lev, int64_t cap, int64_t* nnzb, void* stream)
{
    if (nb < 1 || k < 0 || k > 250 || !Ap || !Aj || !Pp || !nnzb || cap < 0) return BILU_ERR_ARG;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    int32_t nnzA = 0;
    const bilu_status st = sym_count(nb, Ap, Aj, k, Pp, nnzb, &nnzA, s);
    if (st != BILU_OK) return st;
    if (!Pj && !lev && cap == 0) return BILU_OK;   // size query
    if (!Pj || !lev || cap < *nnzb) return BILU_ERR_ARG;
    return sym_write(nb, nnzA, Ap, Aj, k, Pp, Pj, lev, s);
}

bilu_status bilu_levels_device(int nb, const int32_t* Pp, const int32_t* Pj, int sweep, int32_t* lvl,
                               int32_t* level_ptr, int32_t* level_rows, int* nlev, void* stream)
{
    if (nb < 1 || !Pp || !Pj || !lvl || !level_ptr || !level_rows || !nlev || sweep < 0 || sweep > 3)
        return BILU_ERR_ARG;
    return levels_impl(nb, Pp, Pj, sweep, lvl, level_ptr, level_rows, nlev, static_cast<hipStream_t>(stream));
}

}  // extern "C"
