// Pencil sweep for gfx950 (CDNA4, wave64): the level-scheduled sweep of one
// unit-diagonal block triangular factor (Eq 4, Algorithm 7) on a pattern in
// natural grid order, by blocks of grid lines.  Instantiated in pencil_b.hip
// (one translation unit per block size) and, over a batch, in pencil_batch.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "sweep_kernels.h"

namespace bilu {
namespace dev {

// ---------------------------------------------------------------------------
// A tile is a block of grid lines (at most 64/B, so a level of the sweep
// holds at most one chunk of a tile) over their whole length.  A workgroup of
// four wavefronts takes one tile (times one group of CB right-hand-side
// columns) per ticket, each wavefront with one job, joined by counters in
// LDS (the LDS operations of a wavefront take effect in issue order, so a
// count that is seen covers what was written before it):
//   sweep    walks the tile's chunks in level order, lane (q, r) owning
//            component r of the chunk's q-th row; every operand but the
//            factor values, which it prefetches NR - 1 chunks ahead, comes
//            from LDS;
//   stager   writes each chunk's right-hand side (FUSE: D^{-1} times it) into
//            the chunk's slot of the ring, ahead of the sweep, which
//            overwrites it with the result; also hands the feeder its list;
//   feeder   polls the rows that other tiles hand over and puts them into
//            LDS;
//   storer   publishes the finished rows that other tiles read and stores
//            every finished row.
// What bounds a sweep is the chain of dependent levels, and a wavefront alone
// on its SIMD issues an instruction about every eight cycles, so the chain is
// kept to the instructions it cannot do without: about 0.15 us a level inside
// a tile at b = 3, ILU(0), and about 1 us more from tile to tile.  Against the
// row tiles (k_sweep_grouped, k_sweep_tiled, the faster of both), one
// application on MI355X: 60x220x85, b = 3, ILU(0) 975 -> 469 us, ILU(1) with
// FP32 factors 2374 -> 781 us; 10^3 ILU(1) 134 -> 47 us; 64^3 ILU(1), 32
// columns, 4147 -> 1487 us; 120^3 Poisson in blocks of 4, ILU(2), 9109 -> 1780.
//
// Rows that other tiles read (and only those) are published in a compact
// exchange array, one entry per such row in ticket order, which starts at
// kNotReady (see the data-carried readiness above await_value); the result
// itself is stored plainly.  Each launch resets the exchange array of the
// other sweep of the pair.  Tickets run in an order in which every tile comes
// after the tiles it reads, so the launch drains.
// ---------------------------------------------------------------------------
struct PencilArgs {
    const int32_t* tile_ptr;   // [ntiles + 1] first chunk of each tile
    const int32_t* ext_ptr;    // [ntiles + 1] first fed row of each tile
    const int2* rows;          // [(nchunks + kPencilSlack) * (64/B)] first element of the block
                               // row (-1 idle), of its exchange entry (-1 none)
    const char* recs;          // [nchunks + kPencilSlack] factor values and codes, see PencilRec
    const int4* ext;           // [next] first element of the exchange entry read, LDS byte offset
                               // of its place, chunks of the tile finished before that is free
    const double* dinv;        // FUSE: D^{-1} by block rows, column-major blocks
    const double* rhs;
    double* out;
    double* exch;              // [column groups][nexch][B][CB]
    double* reset;             // exchange array of the pair's other sweep
    int64_t nreset;
    int64_t nexch;
    unsigned long long* ticket;
    unsigned int* done;
    int* status;
    const int* gate;           // nothing runs when *gate == 0 (may be null)
    int ntiles;
    int ncg;                   // groups of CB columns
    int ring;                  // chunks of the tile kept in LDS
    int reach;                 // chunks a dependency inside a tile reaches back
    int ext_ring;              // fed rows kept in LDS
    int rhs_R, out_R;          // columns of a row of rhs / out
    int transposed;            // FUSE: multiply by the transposed blocks
    unsigned int total_waves;  // workgroups launched
    unsigned int spin_limit;
};

// A chunk's record: its factor values, value j = k*B + c of every lane, the
// lanes' pairs (FP64) or quads (FP32) of values next to each other, so that a
// lane loads 16 bytes at a time, the values left over one by one (FP32: two,
// then one); then the words of its rows: W4 planes of 64/B quads, two 16-bit
// LDS byte offsets to a word, and the fed rows the chunk needs.
template <int B, typename T, int K>
struct PencilRec {
    static constexpr int KB = K * B;
    static constexpr int RPC = 64 / B;
    static constexpr int W4 = pencil_meta_quads(K);
    static constexpr int value_bytes = KB * 64 * static_cast<int>(sizeof(T));
    static constexpr int bytes = value_bytes + W4 * RPC * 16;
    static constexpr int state = KB * static_cast<int>(sizeof(T) / 4) + 4 * W4;
    // The operands of a row are read from LDS all at once where they are few,
    // else `group` dependencies at a time, one group ahead.
    static constexpr int group(int cb)
    {
        return KB * cb <= 18 ? K : 10 / (B * cb) < 1 ? 1 : 10 / (B * cb);
    }
    // Registers decide how far ahead the sweep wavefront loads: as many chunks
    // of values and words as fit beside those operands in the 256 registers
    // that two wavefronts per SIMD leave, or, where that is less than three, in
    // the 512 of one; a divisor of the ring.
    static constexpr int chunks(int cb, int registers)
    {
        const int held = 2 * B * cb * group(cb) * (group(cb) < K ? 2 : 1) + 2 * cb + (cb == 1 ? 34 : 70) +
                         (sizeof(T) == 4 && KB > 18 ? 30 : 0);
        return (registers - held) / state;
    }
    static constexpr int waves(int cb) { return chunks(cb, 252) >= 3 ? 2 : 1; }
    static constexpr int depth(int cb)
    {
        const int fit = chunks(cb, waves(cb) == 2 ? 252 : 500);
        return fit >= 8 ? 8 : fit >= 6 ? 6 : fit >= 4 ? 4 : fit >= 3 ? 3 : 2;
    }
};

// Global memory at a scalar address, 16 (8, 4) bytes at a lane's offset.
typedef const __attribute__((address_space(1))) char* GlobalBytes;
typedef double Double2 __attribute__((ext_vector_type(2)));
typedef float Float2 __attribute__((ext_vector_type(2)));
typedef float Float4 __attribute__((ext_vector_type(4)));
typedef int Int2 __attribute__((ext_vector_type(2)));
typedef int Int4 __attribute__((ext_vector_type(4)));

template <typename V>
__device__ __forceinline__ V global_at(GlobalBytes base, uint32_t off)
{
    return *reinterpret_cast<const __attribute__((address_space(1))) V*>(base + off);
}

template <int B, typename T, int K>
struct PencilState {
    using S = PencilRec<B, T, K>;
    Int4 m[S::W4];
    T f[S::KB];
};

// Loads the record at rec (wave-uniform); a lane's byte offsets into it are
// the same for every chunk.
struct PencilLane {
    uint32_t by16, by8, by4, words;
};

template <int B, typename T, int K>
__device__ __forceinline__ void pencil_record(GlobalBytes rec, PencilLane& at, PencilState<B, T, K>& s)
{
    // the offsets are widened next to the loads, so that each load adds its
    // lane's offset to the scalar address by itself
    asm volatile("" : "+v"(at.by16), "+v"(at.by8), "+v"(at.by4), "+v"(at.words));
    using S = PencilRec<B, T, K>;
    constexpr int KB = S::KB;
    if constexpr (sizeof(T) == 8) {
#pragma unroll
        for (int p = 0; p < KB / 2; ++p) {
            const Double2 v = global_at<Double2>(rec + p * 1024, at.by16);
            s.f[2 * p] = v.x;
            s.f[2 * p + 1] = v.y;
        }
        if constexpr (KB % 2) s.f[KB - 1] = global_at<double>(rec + (KB / 2) * 1024, at.by8);
    } else {
#pragma unroll
        for (int p = 0; p < KB / 4; ++p) {
            const Float4 v = global_at<Float4>(rec + p * 1024, at.by16);
            s.f[4 * p] = v.x;
            s.f[4 * p + 1] = v.y;
            s.f[4 * p + 2] = v.z;
            s.f[4 * p + 3] = v.w;
        }
        constexpr int q = KB / 4 * 4;
        if constexpr (KB % 4 >= 2) {
            const Float2 v = global_at<Float2>(rec + q * 256, at.by8);
            s.f[q] = v.x;
            s.f[q + 1] = v.y;
        }
        if constexpr (KB % 2) s.f[KB - 1] = global_at<float>(rec + (KB - 1) * 256, at.by4);
    }
#pragma unroll
    for (int w = 0; w < S::W4; ++w) s.m[w] = global_at<Int4>(rec + S::value_bytes + w * (S::RPC * 16), at.words);
}

template <int W4>
__device__ __forceinline__ int pencil_word(const Int4 (&m)[W4], int w)
{
    const Int4& v = m[w / 4];
    return w % 4 == 0 ? v.x : w % 4 == 1 ? v.y : w % 4 == 2 ? v.z : v.w;
}

// LDS byte offset of dependency k (of one column)
template <int W4>
__device__ __forceinline__ uint32_t pencil_code(const Int4 (&m)[W4], int k)
{
    const uint32_t w = static_cast<uint32_t>(pencil_word<W4>(m, k / 2));
    return k % 2 ? w >> 16 : w & 0xffffu;
}

// LDS of a workgroup: zero row, ring, fed rows (CB values to a place), then
// where the values of each ring slot go, the feeder's list (the next rows it
// is to fetch) and the place of values that are not kept.
struct PencilLds {
    char* base;
    char* ring;
    char* ext;
    char* dest;     // [ring][64] byte offsets into out and the exchange array (kNowhere: not stored)
    int4* list;
    int* swept;     // [64] chunks swept, a copy a lane: one store without a branch
    int* listed;    // rows in the list
    int* staged;    // chunks whose right-hand side is in the ring
    int* stored;    // chunks read by the storer
    int* fed;       // rows of other tiles in LDS
};

__device__ __forceinline__ void publish_count(int* c, int v)
{
    if (lane_id() == 0) __hip_atomic_store(c, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ int read_count(const int* c)
{
    return __builtin_amdgcn_readfirstlane(__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
}

// Waits (bounded) until *c reaches need; returns the count seen.  A wait that
// expired is recorded and lets everything after it pass.
__device__ __forceinline__ int reach_count(const int* c, int need, unsigned int limit, int* status)
{
    int seen;
    for (unsigned int spins = 0; (seen = read_count(c)) < need;) {
        if (++spins > limit) {
            if (lane_id() == 0) atomicOr(status, 1);
            seen = INT_MAX;
            break;
        }
        if (spins > 64) __builtin_amdgcn_s_sleep(1);
    }
    // what the count covers is read after it
    asm volatile("" ::: "memory");
    return seen;
}

template <bool V>
struct PencilFlag {
    static constexpr bool value = V;
};

template <int B, typename T, int K, int CB>
__device__ __forceinline__ void pencil_sweep(const PencilArgs& a, int t, const PencilLds& l)
{
    using S = PencilRec<B, T, K>;
    constexpr int NR = S::depth(CB);
    constexpr int LD = NR - 1;
    const int lane = lane_id();
    const int q = lane / B;
    const uint32_t qc = static_cast<uint32_t>(q < S::RPC ? q : S::RPC - 1);
    PencilLane at{lane * 16u, lane * 8u, lane * 4u, qc * 16u};
    const int c0 = uniform_load(a.tile_ptr, t);
    const int n = uniform_load(a.tile_ptr, t + 1) - c0;
    // records past the tile's end are the next tile's (or the slack after the
    // last one): loaded, never used
    GlobalBytes rec = (GlobalBytes)(a.recs + static_cast<int64_t>(c0) * S::bytes);
    PencilState<B, T, K> st[NR];
#pragma unroll
    for (int i = 0; i < LD; ++i) {
        pencil_record<B, T, K>(rec, at, st[i]);
        rec += S::bytes;
    }
    int known = 0;                            // fed rows known to be in LDS
    int staged = 0;
    uint32_t turn = 0;                        // ring offset of the turn's first chunk
    const uint32_t end = static_cast<uint32_t>(a.ring) * (512 * CB);
    char* mine = l.ring + lane * (8 * CB);
    // one turn of the register ring from chunk i0; PART: the tile ends in it
    auto sweep_turn = [&](int i0, auto part) {
        constexpr bool PART = decltype(part)::value;
#pragma unroll
        for (int p = 0; p < NR; ++p) {
            if (PART && i0 + p >= n) return;
            PencilState<B, T, K>& s = st[p];
            // the state is taken over here: nothing formed from its words may
            // move up to where they were loaded, which would wait for the load
#pragma unroll
            for (int w = 0; w < S::W4; ++w)
                asm volatile("" : "+v"(s.m[w]));
            if (__builtin_expect(staged <= i0 + p, 0)) staged = reach_count(l.staged, i0 + p + 1, a.spin_limit, a.status);
            const int need = __builtin_amdgcn_readfirstlane(pencil_word<S::W4>(s.m, (K + 1) / 2));
            if (__builtin_expect(known < need, 0)) known = reach_count(l.fed, need, a.spin_limit, a.status);
            // dependencies, every lane and slot (padding and idle slots read
            // the zero row)
            constexpr int G = S::group(CB), NG = (K + G - 1) / G;
            double x[NG > 1 ? 2 : 1][G * B * CB], acc[CB];
            auto read_group = [&](int g0) {
                double (&to)[G * B * CB] = x[NG > 1 ? g0 % 2 : 0];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    if (g0 * G + g >= K) continue;
                    const char* xp = l.base + pencil_code<S::W4>(s.m, g0 * G + g) * CB;
#pragma unroll
                    for (int c = 0; c < B; ++c) {
                        if constexpr (CB == 1) {
                            to[g * B + c] = *reinterpret_cast<const double*>(xp + c * 8);
                        } else {
#pragma unroll
                            for (int e = 0; e < CB; e += 2) {
                                const double2 v = *reinterpret_cast<const double2*>(xp + (c * CB + e) * 8);
                                to[(g * B + c) * CB + e] = v.x;
                                to[(g * B + c) * CB + e + 1] = v.y;
                            }
                        }
                    }
                }
            };
            char* place = mine + turn + p * (512 * CB);
#pragma unroll
            for (int e = 0; e < CB; ++e) acc[e] = *reinterpret_cast<const double*>(place + e * 8);
            read_group(0);
            __builtin_amdgcn_sched_barrier(0);
            // prefetch, behind the reads just issued
            pencil_record<B, T, K>(rec, at, st[(p + LD) % NR]);
            rec += S::bytes;
            // kept a scalar: the loads then add a lane's constant offset to it
            asm volatile("" : "+s"(rec));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g0 = 0; g0 < NG; ++g0) {
                if (g0 + 1 < NG) read_group(g0 + 1);
                const double (&from)[G * B * CB] = x[NG > 1 ? g0 % 2 : 0];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    if (g0 * G + g >= K) continue;
#pragma unroll
                    for (int c = 0; c < B; ++c) {
                        const double f = widen(s.f[(g0 * G + g) * B + c]);
#pragma unroll
                        for (int e = 0; e < CB; ++e) acc[e] -= f * from[(g * B + c) * CB + e];
                    }
                }
                // (keeps the reads of later groups from being gathered here)
                if (g0 + 1 < NG) __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (CB == 1) {
                *reinterpret_cast<double*>(place) = acc[0];
            } else {
#pragma unroll
                for (int e = 0; e < CB; e += 2)
                    *reinterpret_cast<double2*>(place + e * 8) = make_double2(acc[e], acc[e + 1]);
            }
            // one wavefront: its LDS operations take effect in issue order,
            // so only the compiler must keep this chunk's writes before the
            // next chunk's reads and the count
            __builtin_amdgcn_wave_barrier();
            asm volatile("" ::: "memory");
            l.swept[lane] = i0 + p + 1;
            asm volatile("" ::: "memory");
        }
        turn = turn + NR * 512 * CB == end ? 0u : turn + NR * 512 * CB;
    };
    int i0 = 0;
    for (; i0 + NR <= n; i0 += NR) sweep_turn(i0, PencilFlag<false>{});
    if (i0 < n) sweep_turn(i0, PencilFlag<true>{});
}

constexpr uint32_t kNowhere = 0xffffffffu;

// The right-hand side of every chunk into its ring slot, and where its values
// go beside it, two chunks at a time, once the slots' previous chunks are
// stored and no longer read; loads run U chunks ahead, row numbers twice that.
template <int B, int CB, bool FUSE, bool ROUND>
__device__ __forceinline__ void pencil_stage(const PencilArgs& a, int t, int cg, const PencilLds& l)
{
    constexpr int RPC = 64 / B;
    constexpr int kList = pencil_list_rows(RPC);
    constexpr int state = FUSE ? 2 * B * (1 + CB) : 2 * CB;
    constexpr int U = 160 / state >= 8 ? 8 : 160 / state >= 4 ? 4 : 2;
    const int lane = lane_id();
    const int q = lane / B;
    const int r = lane - q * B;
    const bool lane_ok = q < RPC;
    const uint32_t qc = static_cast<uint32_t>(lane_ok ? q : RPC - 1);
    const int c0 = uniform_load(a.tile_ptr, t);
    const int n = uniform_load(a.tile_ptr, t + 1) - c0;
    const int e0 = uniform_load(a.ext_ptr, t);
    const int ne = uniform_load(a.ext_ptr, t + 1) - e0;
    const uint32_t j0 = static_cast<uint32_t>(cg) * CB;
    const uint32_t rR = static_cast<uint32_t>(a.rhs_R), oR = static_cast<uint32_t>(a.out_R);
    struct Staged {
        double h[FUSE ? B * CB : CB];
        double d[FUSE ? B : 1];
        Int2 row;
    };
    Staged st[U];
    Int2 rowr[U];
    // rows past the tile's end are the next tile's (or the slack after the
    // last one): loaded, never used
    GlobalBytes rp = (GlobalBytes)(a.rows + static_cast<int64_t>(c0) * RPC);
    auto load_row = [&]() {
        const Int2 row = global_at<Int2>(rp, qc * 8u);
        rp += RPC * 8;
        return row;
    };
    auto load_rhs = [&](Int2 row, Staged& s) {
        s.row = row;
        const uint32_t rb = static_cast<uint32_t>(row.x >= 0 ? row.x : 0);
        if constexpr (FUSE) {
            const double* dp = a.dinv + static_cast<int64_t>(rb) * B;
            if (a.transposed) {
                dp += r * B;
#pragma unroll
                for (int c = 0; c < B; ++c) s.d[c] = dp[c];
            } else {
                dp += r;
#pragma unroll
                for (int c = 0; c < B; ++c) s.d[c] = dp[c * B];
            }
            const uint32_t hb = (rb * rR + j0) * 8u;
#pragma unroll
            for (int c = 0; c < B; ++c)
#pragma unroll
                for (int e = 0; e < CB; ++e) s.h[c * CB + e] = load_at(a.rhs, hb + (c * rR + e) * 8u);
        } else {
            const uint32_t hb = ((rb + r) * rR + j0) * 8u;
#pragma unroll
            for (int e = 0; e < CB; ++e) s.h[e] = load_at(a.rhs, hb + e * 8u);
        }
    };
#pragma unroll
    for (int i = 0; i < U; ++i) rowr[i] = load_row();
#pragma unroll
    for (int i = 0; i < U; ++i) {
        load_rhs(rowr[i], st[i]);
        rowr[i] = load_row();
    }
    // the feeder's list (the feeder fills it first), half of it at a time; a
    // half is free once the feeder is past what it held
    int listed = min(ne, kList);
    auto list_some = [&]() {
        if (listed >= ne || read_count(l.fed) < listed - kList / 2) return;
        const int hi = min(ne, listed + kList / 2);
        for (int o = listed + lane; o < hi; o += 64) l.list[o & (kList - 1)] = a.ext[e0 + o];
        listed = hi;
        asm volatile("" ::: "memory");
        publish_count(l.listed, listed);
    };
    int room = a.ring;                        // chunks that may be staged
    uint32_t slot = static_cast<uint32_t>(lane) * 8;
    const uint32_t end = static_cast<uint32_t>(a.ring) * 512;
    for (int i0 = 0; i0 < n; i0 += U) {
#pragma unroll
        for (int p = 0; p < U; p += 2) {
            const int i = i0 + p;
            if (i >= n) break;
            for (unsigned int spins = 0; i + 2 > room;) {
                list_some();
                room = a.ring + min(read_count(l.stored), read_count(l.swept) - a.reach);
                if (i + 2 <= room) break;
                if (++spins > a.spin_limit) {
                    if (lane == 0) atomicOr(a.status, 1);
                    room = INT_MAX;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            asm volatile("" ::: "memory");
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                Staged& s = st[p + u];
                double v[CB];
                if constexpr (FUSE) {
#pragma unroll
                    for (int e = 0; e < CB; ++e) v[e] = 0.0;
#pragma unroll
                    for (int c = 0; c < B; ++c) {
                        const double d = ROUND ? static_cast<double>(static_cast<float>(s.d[c])) : s.d[c];
#pragma unroll
                        for (int e = 0; e < CB; ++e) v[e] += d * s.h[c * CB + e];
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < CB; ++e) v[e] = s.h[e];
                }
                const bool used = lane_ok && s.row.x >= 0;
#pragma unroll
                for (int e = 0; e < CB; ++e) *reinterpret_cast<double*>(l.ring + slot * CB + e * 8) = used ? v[e] : 0.0;
                Int2 dest;
                dest.x = used ? static_cast<int>(((static_cast<uint32_t>(s.row.x) + r) * oR + j0) * 8u)
                              : static_cast<int>(kNowhere);
                dest.y = used && s.row.y >= 0 ? static_cast<int>((static_cast<uint32_t>(s.row.y) + r) * (8u * CB))
                                              : static_cast<int>(kNowhere);
                *reinterpret_cast<Int2*>(l.dest + slot) = dest;
                slot += 512;
                if (slot >= end) slot -= end;
            }
            __builtin_amdgcn_wave_barrier();
            asm volatile("" ::: "memory");
            publish_count(l.staged, i + 2);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                load_rhs(rowr[p + u], st[p + u]);
                rowr[p + u] = load_row();
            }
        }
    }
    for (unsigned int spins = 0; listed < ne && spins <= a.spin_limit; ++spins) {
        list_some();
        __builtin_amdgcn_s_sleep(1);
    }
}

// The feeder: fetches the rows of other tiles in the order they are needed,
// 64/B of them at a time from the first one missing on (lane (q, r): component
// r of the q-th), puts those that are published into LDS and counts the ones
// before the first missing one.  The loop is bound by its instructions: wider
// windows and several windows in flight ran slower (60x220x85, b = 3, an
// application at ILU(0) / ILU(1): 460 / 880 us; two or three times the rows
// 495 / 914 and 510 / 976 us; those with two, three or four windows in flight
// 512 / 1014, 541 / 1089 and 581 / 1105 us).
template <int B, int CB>
__device__ __forceinline__ void pencil_feed(const PencilArgs& a, int t, int cg, const PencilLds& l)
{
    constexpr int RPC = 64 / B;
    constexpr int kList = pencil_list_rows(RPC);
    const int lane = lane_id();
    const bool lane_ok = lane < RPC * B;
    const int q = lane_ok ? lane / B : RPC - 1;
    const int r = lane_ok ? lane - q * B : 0;
    const int e0 = uniform_load(a.ext_ptr, t);
    const int n = uniform_load(a.ext_ptr, t + 1) - e0;
    if (n <= 0) return;
    for (int o = lane; o < min(n, kList); o += 64) l.list[o] = a.ext[e0 + o];
    asm volatile("" ::: "memory");
    publish_count(l.listed, min(n, kList));
    GlobalBytes exch = (GlobalBytes)(a.exch + static_cast<int64_t>(cg) * a.nexch * (B * CB));
    const uint32_t r8 = static_cast<uint32_t>(r) * (8 * CB);
    const uint32_t dump = static_cast<uint32_t>(reinterpret_cast<char*>(l.list + kList) - l.base) + lane * (8 * CB);
    auto value_at = [&](uint32_t off) {
        return __hip_atomic_load(reinterpret_cast<const __attribute__((address_space(1))) double*>(exch + off),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    int fed = 0;
    uint32_t off, dst;               // of the lane's value: in the exchange array, in LDS
    unsigned long long blocked;      // lanes whose row is not listed yet, or its place not free
    auto aim = [&]() {
        const int swept = __hip_atomic_load(l.swept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const int listed = __hip_atomic_load(l.listed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        asm volatile("" ::: "memory");
        const int e = fed + q, ec = min(e, n - 1);
        Int4 x = *reinterpret_cast<const Int4*>(l.list + (ec & (kList - 1)));
        asm volatile("" : "+v"(x));  // one read, then selections without branches
        const bool wait = ec >= listed || x.z > swept;
        off = wait ? 0u : static_cast<uint32_t>(x.x) * (8 * CB) + r8;
        dst = wait || e >= n || !lane_ok ? dump : static_cast<uint32_t>(x.y) * CB + r8;
        blocked = __ballot(wait ? 1 : 0);
    };
    aim();
    // a tile ahead of the sweep's front looks for its first row only, and
    // slowly
    unsigned int spins = 0;
    const uint32_t first = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(off)));
    while (is_not_ready(value_at(first)) && ++spins <= a.spin_limit) __builtin_amdgcn_s_sleep(4);
    while (fed < n && spins <= a.spin_limit) {
        double v[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c) v[c] = value_at(off + c * 8u);
        bool gap = false;
#pragma unroll
        for (int c = 0; c < CB; ++c) gap |= is_not_ready(v[c]);
        const unsigned long long gaps = __ballot(gap ? 1 : 0) | blocked;
        const int lead = gaps == 0 ? RPC : __builtin_ctzll(gaps) / B;
        if (lead > 0) {
            if (!gap) {
#pragma unroll
                for (int c = 0; c < CB; ++c) *reinterpret_cast<double*>(l.base + dst + c * 8) = v[c];
            }
            fed = min(n, fed + lead);
            __builtin_amdgcn_wave_barrier();
            asm volatile("" ::: "memory");
            publish_count(l.fed, fed);
            spins = 0;
        } else {
            ++spins;
        }
        if (lead > 0 || blocked != 0) aim();
    }
    if (fed < n) {
        if (lane == 0) atomicOr(a.status, 1);
        publish_count(l.fed, n);
    }
}

// The storer: every finished chunk's rows to the exchange array, where other
// tiles read them, and to the result.  It loads nothing from memory, so it
// never waits for its stores.
template <int B, int CB>
__device__ __forceinline__ void pencil_store(const PencilArgs& a, int t, int cg, const PencilLds& l)
{
    const int lane = lane_id();
    const int n = uniform_load(a.tile_ptr, t + 1) - uniform_load(a.tile_ptr, t);
    char* exch = reinterpret_cast<char*>(a.exch + static_cast<int64_t>(cg) * a.nexch * (B * CB));
    char* out = reinterpret_cast<char*>(a.out);
    int prog = 0;
    uint32_t slot = static_cast<uint32_t>(lane) * 8;
    const uint32_t end = static_cast<uint32_t>(a.ring) * 512;
    for (int i = 0; i < n; ++i) {
        if (prog <= i) prog = reach_count(l.swept, i + 1, a.spin_limit, a.status);
        double v[CB];
#pragma unroll
        for (int e = 0; e < CB; ++e) v[e] = *reinterpret_cast<const double*>(l.ring + slot * CB + e * 8);
        const Int2 dest = *reinterpret_cast<const Int2*>(l.dest + slot);
        slot += 512;
        if (slot >= end) slot -= end;
        // (read before the count: the slot may be reused)
        asm volatile("" ::: "memory");
        if (i % 2 == 1 || i + 1 == n) publish_count(l.stored, i + 1);
        if (static_cast<uint32_t>(dest.y) != kNowhere) {
            double* ep = reinterpret_cast<double*>(exch + static_cast<uint32_t>(dest.y));
#pragma unroll
            for (int e = 0; e < CB; ++e) coherent_store(ep + e, publishable(v[e]));
        }
        if (static_cast<uint32_t>(dest.x) != kNowhere) {
#pragma unroll
            for (int e = 0; e < CB; ++e)
                *reinterpret_cast<double*>(out + static_cast<uint32_t>(dest.x) + e * 8u) = v[e];
        }
    }
}

// LDS of a workgroup; swept, count: its counters.
template <int B, int CB>
__device__ __forceinline__ PencilLds pencil_lds_map(const PencilArgs& a, char* base, int* swept, int* count)
{
    PencilLds l;
    l.base = base;
    l.ring = l.base + kPencilZeroBytes * CB;
    l.ext = l.ring + a.ring * kPencilSlotBytes * CB;
    l.dest = l.ext + a.ext_ring * (B * 8 * CB);
    l.list = reinterpret_cast<int4*>(l.dest + a.ring * 512);
    l.swept = swept;
    l.listed = count;
    l.staged = count + 1;
    l.stored = count + 2;
    l.fed = count + 3;
    return l;
}

// no destination of a slot yet: a wait that expires lets the storer pass
// slots that were never staged
__device__ __forceinline__ void pencil_clear_dest(const PencilArgs& a, const PencilLds& l)
{
    for (int i = static_cast<int>(threadIdx.x); i < a.ring * 128; i += 256)
        reinterpret_cast<uint32_t*>(l.dest)[i] = kNowhere;
}

// Tile t for column group cg, by the four wavefronts; part / parts: its share
// of the reset of the other sweep's exchange array.
template <int B, typename T, int K, int CB, bool FUSE>
__device__ __forceinline__ void pencil_tile(const PencilArgs& a, int t, int cg, int part, int parts,
                                            const PencilLds& l, int wave)
{
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(3);
        pencil_sweep<B, T, K, CB>(a, t, l);
        __builtin_amdgcn_s_setprio(0);
    } else if (wave == 1) {
        pencil_feed<B, CB>(a, t, cg, l);
        const int64_t lo = a.nreset * part / parts, hi = a.nreset * (part + 1) / parts;
        for (int64_t i = lo + lane_id(); i < hi; i += 64) a.reset[i] = not_ready();
    } else if (wave == 2) {
        pencil_stage<B, CB, FUSE, sizeof(T) == 4>(a, t, cg, l);
    } else {
        pencil_store<B, CB>(a, t, cg, l);
    }
}

template <int B, typename T, int K, int CB, bool FUSE>
__global__ __launch_bounds__(256, (PencilRec<B, T, K>::waves(CB))) void k_sweep_pencil(PencilArgs a)
{
    extern __shared__ double2 pencil_lds[];
    __shared__ int s_swept[kWave], s_count[kPencilCounts];
    if (gated_off(a.gate)) return;
    const PencilLds l = pencil_lds_map<B, CB>(a, reinterpret_cast<char*>(pencil_lds), s_swept, s_count);
    int& s_ticket = s_count[4];
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    if (static_cast<int>(threadIdx.x) < kPencilZeroBytes / 8 * CB) reinterpret_cast<double*>(l.base)[threadIdx.x] = 0.0;
    pencil_clear_dest(a, l);
    const int nticket = a.ntiles * a.ncg;
    for (;;) {
        if (threadIdx.x < 64) s_swept[threadIdx.x] = 0;
        if (threadIdx.x == 0) {
            const unsigned long long tk = atomicAdd(a.ticket, 1ULL);
            for (int i = 0; i < 4; ++i) s_count[i] = 0;
            s_ticket = tk > 0x3fffffffULL ? 0x3fffffff : static_cast<int>(tk);
        }
        __syncthreads();
        const int tk = __builtin_amdgcn_readfirstlane(s_ticket);
        if (tk >= nticket) break;
        const int t = tk / a.ncg;
        const int cg = tk - t * a.ncg;
        pencil_tile<B, T, K, CB, FUSE>(a, t, cg, tk, nticket, l, wave);
        __syncthreads();
    }
    if (wave == 0) finish_persistent(a.ticket, a.done, a.total_waves);
}

// ---------------------------------------------------------------------------
// The same over a batch: tickets are (member, tile) pairs, each member with
// arguments of its own in device memory.  One kernel holds every block size
// at the width of ILU(0) on a grid (kPencilBatchWidth): their registers all
// allow two workgroups per compute unit, which wider rows would halve.  (The
// largest blocks set the count: 38 registers spill in FP64, 29 in FP32.)
// One application of 64 systems of 8 to 40 cells a side, blocks of 2 to 8
// (1.3 GB of factors and vectors, 280 us at the rate of a copy): 1144 us with
// a wavefront a row tile (k_sweep_batch), 467 us so.
// ---------------------------------------------------------------------------
struct PencilMember {
    PencilArgs a;              // rhs, out, ticket, done, status, gate unset
    int64_t voff;              // first unknown of the member in the batch vectors
    int bs;
    int pad;
};

struct PencilBatchArgs {
    const PencilMember* mem;
    const int2* items;         // (member, tile)
    int nitems;
    const double* rhs;
    double* out;
    const int* active;         // per member, or null: every member
    const int* gate;           // nothing runs when given and *gate == 0
    unsigned long long* ticket;
    unsigned int* done;
    int* status;
    unsigned int total_waves;  // workgroups launched
    unsigned int spin_limit;
};

template <int B, typename T, bool FUSE>
__device__ __forceinline__ void pencil_batch_tile(const PencilArgs& a, int t, char* base, int* swept, int* count,
                                                  int wave)
{
    const PencilLds l = pencil_lds_map<B, 1>(a, base, swept, count);
    // the LDS held another member's tile
    pencil_clear_dest(a, l);
    __syncthreads();
    pencil_tile<B, T, kPencilBatchWidth, 1, FUSE>(a, t, 0, t, a.ntiles, l, wave);
    __syncthreads();
}

template <typename T, bool FUSE>
__global__ __launch_bounds__(256, 2) void k_sweep_pencil_batch(PencilBatchArgs b)
{
    extern __shared__ double2 pencil_lds[];
    __shared__ int s_swept[kWave], s_count[kPencilCounts];
    if (gated_off(b.gate)) return;
    char* base = reinterpret_cast<char*>(pencil_lds);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    if (static_cast<int>(threadIdx.x) < kPencilZeroBytes / 8) reinterpret_cast<double*>(base)[threadIdx.x] = 0.0;
    for (;;) {
        if (threadIdx.x < 64) s_swept[threadIdx.x] = 0;
        if (threadIdx.x == 0) {
            const unsigned long long tk = atomicAdd(b.ticket, 1ULL);
            for (int i = 0; i < 4; ++i) s_count[i] = 0;
            s_count[4] = tk > 0x3fffffffULL ? 0x3fffffff : static_cast<int>(tk);
        }
        __syncthreads();
        const int tk = __builtin_amdgcn_readfirstlane(s_count[4]);
        // (the ticket is read by every wavefront before it is drawn again)
        __syncthreads();
        if (tk >= b.nitems) break;
        const int2 it = uniform_record(b.items, tk);
        if (b.active && !uniform_load(b.active, it.x)) continue;
        PencilMember m = uniform_record(b.mem, it.x);
        m.a.rhs = b.rhs + m.voff;
        m.a.out = b.out + m.voff;
        m.a.status = b.status;
        m.a.spin_limit = b.spin_limit;
        switch (m.bs) {
#define BILU_PENCIL_BATCH(BS) \
    case BS: pencil_batch_tile<BS, T, FUSE>(m.a, it.y, base, s_swept, s_count, wave); break;
        BILU_PENCIL_BATCH(1) BILU_PENCIL_BATCH(2) BILU_PENCIL_BATCH(3) BILU_PENCIL_BATCH(4)
        BILU_PENCIL_BATCH(5) BILU_PENCIL_BATCH(6) BILU_PENCIL_BATCH(7) BILU_PENCIL_BATCH(8)
#undef BILU_PENCIL_BATCH
        default: break;
        }
    }
    if (wave == 0) finish_persistent(b.ticket, b.done, b.total_waves);
}

}  // namespace dev
}  // namespace bilu
