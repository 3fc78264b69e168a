// Pencil layouts of the sweeps (host): blocks of grid lines with their rows in
// level order, the LDS places of every dependency and the exchange of rows
// between blocks.  See HostPencil for the layout and k_sweep_pencil for the
// kernel that reads it.
#include <algorithm>
#include <cstdint>
#include <queue>
#include <utility>
#include <vector>

#include "bilu_internal.h"

namespace bilu {

namespace {

constexpr int kLdsBytes = 65536;    // LDS places whose offsets fit 16 bits
constexpr int kFeedAhead = 6;       // in units of rpc: LDS places of fed rows beyond those in use
constexpr int kStageAhead = 12;     // ring slots beyond the reach back: chunks staged ahead of the sweep
constexpr int kSkewMax = 4;

// Grid of a sweep, in its own coordinates (mirrored for backward sweeps).
struct SweepGrid {
    int nx = 0, ny = 0, nz = 0;
    bool forward = true;
    void line(int32_t i, int& y, int& z) const
    {
        const int l = i / nx;
        y = l % ny;
        z = l / ny;
        if (!forward) {
            y = ny - 1 - y;
            z = nz - 1 - z;
        }
    }
};

int own_code(int i, int ring, int q, int bs) { return kPencilZeroBytes + (i % ring) * kPencilSlotBytes + q * bs * 8; }

int fed_code(int e, int ring, int ext_ring, int bs)
{
    return kPencilZeroBytes + ring * kPencilSlotBytes + e % ext_ring * bs * 8;
}

}  // namespace

void build_pencil(const Host& h, int which, int rpc, HostPencil& s)
{
    s = HostPencil{};
    s.tried = true;
    const int nb = h.nb, bs = h.bs;
    if (bs > kMaxKernelBs || static_cast<int64_t>(nb) * bs * 8 > INT32_MAX) return;
    if (h.Pj.size() > static_cast<size_t>(INT32_MAX)) return;
    SweepGrid g;
    int nxy = 0;
    if (!grid_lines(h, g.nx, nxy)) return;
    g.ny = nxy / g.nx;
    g.nz = nb / nxy;
    g.forward = which == BILU_SWEEP_L || which == BILU_SWEEP_UT;
    std::vector<int32_t> dptr;
    std::vector<Dep> deps;
    sweep_deps(h, which, dptr, deps);
    int width = 0;
    for (int i = 0; i < nb; ++i) width = std::max(width, dptr[i + 1] - dptr[i]);
    width = pencil_width(bs, width);
    if (!width) return;
    // the skew that makes every dependency point backwards along y too
    const int nlines = g.ny * g.nz;
    std::vector<int32_t> ly(static_cast<size_t>(nlines)), lz(static_cast<size_t>(nlines));
    for (int l = 0; l < nlines; ++l) g.line(l * g.nx, ly[l], lz[l]);
    int skew = 0;
    for (int i = 0; i < nb; ++i) {
        const int l = i / g.nx;
        for (int32_t d = dptr[i]; d < dptr[i + 1]; ++d) {
            const int m = deps[d].col / g.nx;
            const int dy = ly[m] - ly[l], dz = lz[m] - lz[l];
            if (dz > 0 || (dz == 0 && dy > 0)) return;
            if (dz < 0) skew = std::max(skew, (dy - dz - 1) / -dz);
        }
        if (skew > kSkewMax) return;
    }
    // blocks of at most rpc lines with the fewest block boundaries from one
    // corner of the grid to the other: each costs the sweep a hand-over
    // through memory
    const int ext_y = g.ny + skew * (g.nz - 1);
    int best = INT32_MAX;
    for (int wz = 1; wz <= rpc; ++wz) {
        const int wy = std::min(rpc / wz, ext_y);
        const int cost = (ext_y + wy - 1) / wy + (g.nz + wz - 1) / wz;
        if (cost < best) {
            best = cost;
            s.wy = wy;
            s.wz = wz;
        }
    }
    const int NY = (ext_y + s.wy - 1) / s.wy, NZ = (g.nz + s.wz - 1) / s.wz;
    std::vector<int32_t> block_of_line(static_cast<size_t>(nlines));
    for (int l = 0; l < nlines; ++l) block_of_line[l] = (lz[l] / s.wz) * NY + (ly[l] + skew * lz[l]) / s.wy;
    // rows of every block in level order (rows ascending inside a level)
    const HostSweep& lev = h.sweep[which];
    std::vector<int32_t> bptr(static_cast<size_t>(NY) * NZ + 1, 0);
    for (int l = 0; l < nlines; ++l) bptr[block_of_line[l] + 1] += g.nx;
    for (size_t b = 0; b + 1 < bptr.size(); ++b) bptr[b + 1] += bptr[b];
    std::vector<int32_t> brow(static_cast<size_t>(nb)), blev(static_cast<size_t>(nb));
    {
        std::vector<int32_t> fill(bptr.begin(), bptr.end() - 1);
        for (int l = 0; l < lev.nlev; ++l)
            for (int32_t p = lev.level_ptr[l]; p < lev.level_ptr[l + 1]; ++p) {
                const int32_t i = lev.level_rows[p];
                const int32_t at = fill[block_of_line[i / g.nx]]++;
                brow[at] = i;
                blev[at] = l;
            }
    }
    // ticket order: blocks after the blocks they read, those whose first row
    // has the lowest level first
    const int nblk = NY * NZ;
    std::vector<int32_t> ticket(static_cast<size_t>(nblk), -1);
    {
        // block-to-block dependencies, distinct per reader
        std::vector<int32_t> stamp(static_cast<size_t>(nblk), -1), indeg(static_cast<size_t>(nblk), 0);
        std::vector<std::vector<int32_t>> readers(static_cast<size_t>(nblk));
        for (int b = 0; b < nblk; ++b)
            for (int32_t p = bptr[b]; p < bptr[b + 1]; ++p)
                for (int32_t d = dptr[brow[p]]; d < dptr[brow[p] + 1]; ++d) {
                    const int o = block_of_line[deps[d].col / g.nx];
                    if (o == b || stamp[o] == b) continue;
                    stamp[o] = b;
                    readers[o].push_back(b);
                    ++indeg[b];
                }
        using Item = std::pair<int32_t, int32_t>;
        std::priority_queue<Item, std::vector<Item>, std::greater<>> ready;
        for (int b = 0; b < nblk; ++b)
            if (indeg[b] == 0 && bptr[b] < bptr[b + 1]) ready.emplace(blev[bptr[b]], b);
        while (!ready.empty()) {
            const int b = ready.top().second;
            ready.pop();
            ticket[b] = s.ntiles++;
            for (int o : readers[b])
                if (--indeg[o] == 0) ready.emplace(blev[bptr[o]], o);
        }
    }
    std::vector<int32_t> block(static_cast<size_t>(s.ntiles), -1);
    int64_t placed = 0;
    for (int b = 0; b < nblk; ++b)
        if (ticket[b] >= 0) {
            block[ticket[b]] = b;
            placed += bptr[b + 1] - bptr[b];
        }
    if (placed != nb) return;               // a cycle between blocks
    // rows read by other tiles
    std::vector<int32_t> entry(static_cast<size_t>(nb), -1);
    for (int i = 0; i < nb; ++i)
        for (int32_t d = dptr[i]; d < dptr[i + 1]; ++d)
            if (block_of_line[deps[d].col / g.nx] != block_of_line[i / g.nx]) entry[deps[d].col] = 0;
    // chunks, exchange entries, the longest reach back
    s.tile_ptr.assign(1, 0);
    std::vector<int32_t> at(static_cast<size_t>(nb)), slot_q(static_cast<size_t>(nb));   // chunk in the tile, row slot
    int reach = 0;
    for (int t = 0; t < s.ntiles; ++t) {
        const int b = block[t];
        int32_t p = bptr[b];
        int nch = 0;
        while (p < bptr[b + 1]) {
            int q = 0;
            for (; q < rpc && p + q < bptr[b + 1] && blev[p + q] == blev[p]; ++q) {
                const int32_t i = brow[p + q];
                s.rows.push_back(i);
                at[i] = nch;
                slot_q[i] = q;
                if (entry[i] >= 0) entry[i] = static_cast<int32_t>(s.nexch++);
                for (int32_t d = dptr[i]; d < dptr[i + 1]; ++d)
                    if (block_of_line[deps[d].col / g.nx] == b) reach = std::max(reach, nch - at[deps[d].col]);
            }
            p += q;
            for (; q < rpc; ++q) s.rows.push_back(-1);
            ++nch;
        }
        s.tile_ptr.push_back(s.tile_ptr.back() + nch);
    }
    s.nchunks = s.tile_ptr.back();
    s.reach = reach;
    s.ring = kPencilRing;
    while (s.ring < reach + kStageAhead) s.ring += kPencilRing;
    std::vector<int32_t> needed(static_cast<size_t>(s.nchunks), 0);
    // rows fed to a tile, in the order its chunks first read them
    std::vector<int32_t> seen(static_cast<size_t>(nb), -1), fed_at(static_cast<size_t>(nb));
    std::vector<int32_t> last;              // per fed row: last chunk of the tile that reads it
    s.ext_ptr.assign(1, 0);
    int live = 0;
    for (int t = 0; t < s.ntiles; ++t) {
        const int b = block[t];
        const int first = static_cast<int>(last.size());
        for (int c = s.tile_ptr[t]; c < s.tile_ptr[t + 1]; ++c) {
            for (int q = 0; q < rpc; ++q) {
                const int32_t i = s.rows[static_cast<size_t>(c) * rpc + q];
                if (i < 0) break;
                for (int32_t d = dptr[i]; d < dptr[i + 1]; ++d) {
                    const int32_t j = deps[d].col;
                    if (block_of_line[j / g.nx] == b) continue;
                    if (seen[j] != t) {
                        seen[j] = t;
                        fed_at[j] = static_cast<int32_t>(last.size()) - first;
                        s.ext_idx.push_back(entry[j]);
                        last.push_back(0);
                    }
                    last[static_cast<size_t>(first + fed_at[j])] = c - s.tile_ptr[t];
                }
            }
            needed[c] = static_cast<int32_t>(last.size()) - first;
        }
        for (size_t e = static_cast<size_t>(first); e < last.size(); ++e)
            live = std::max(live, needed[s.tile_ptr[t] + last[e]] - static_cast<int>(e) + first);
        if (last.size() > static_cast<size_t>(INT32_MAX / 2)) return;
        s.ext_ptr.push_back(static_cast<int32_t>(last.size()));
    }
    s.next = s.ext_ptr.back();
    // rows in use at once, and those handed over ahead of the sweep
    s.ext_ring = live + kFeedAhead * rpc;
    s.ext_ring += s.ext_ring % 2;           // the list behind them starts at 16 bytes
    if (kPencilZeroBytes + s.ring * kPencilSlotBytes + s.ext_ring * bs * 8 > kLdsBytes) return;
    s.ext_free.assign(static_cast<size_t>(s.next), 0);
    for (int t = 0; t < s.ntiles; ++t)
        for (int e = s.ext_ptr[t] + s.ext_ring; e < s.ext_ptr[t + 1]; ++e) s.ext_free[e] = last[e - s.ext_ring] + 1;
    // dependency codes and factor entries
    const int w4 = pencil_meta_quads(width);
    s.entry.assign(s.rows.size(), -1);
    s.meta.assign(static_cast<size_t>(s.nchunks) * w4 * rpc * 4, 0);
    s.src.assign(static_cast<size_t>(s.nchunks) * width * rpc, -1);
    std::fill(seen.begin(), seen.end(), -1);
    for (int t = 0; t < s.ntiles; ++t) {
        int next = 0;                       // fed rows, numbered as above
        const int b = block[t];
        for (int c = s.tile_ptr[t]; c < s.tile_ptr[t + 1]; ++c) {
            for (int q = 0; q < rpc; ++q) {
                const int32_t i = s.rows[static_cast<size_t>(c) * rpc + q];
                auto word = [&](int w) -> int32_t& {
                    return s.meta[((static_cast<size_t>(c) * w4 + w / 4) * rpc + q) * 4 + w % 4];
                };
                word((width + 1) / 2) = needed[c];
                if (i < 0) continue;
                s.entry[static_cast<size_t>(c) * rpc + q] = entry[i];
                for (int32_t d = dptr[i]; d < dptr[i + 1]; ++d) {
                    const int k = d - dptr[i];
                    const int32_t o = deps[d].col;
                    int code;
                    if (block_of_line[o / g.nx] == b) {
                        code = own_code(at[o], s.ring, slot_q[o], bs);
                    } else {
                        if (seen[o] != t) {
                            seen[o] = t;
                            fed_at[o] = next++;
                        }
                        code = fed_code(fed_at[o], s.ring, s.ext_ring, bs);
                    }
                    word(k / 2) |= static_cast<int32_t>(static_cast<uint32_t>(code) << (k % 2 ? 16 : 0));
                    s.src[(static_cast<size_t>(c) * width + k) * rpc + q] = static_cast<int32_t>(deps[d].src);
                }
            }
        }
    }
    s.which = which;
    s.rpc = rpc;
    s.width = width;
    s.skew = skew;
    s.built = true;
}

int validate_pencil(const Host& h, const HostPencil& s)
{
    const int nb = h.nb, bs = h.bs, rpc = s.rpc, w4 = pencil_meta_quads(s.width);
    const int64_t nP = static_cast<int64_t>(h.Pj.size());
    const size_t nslots = static_cast<size_t>(s.nchunks) * rpc;
    // the stager must be able to run ahead of the sweep
    if (rpc < 1 || rpc * bs > kWave || s.width < 1 || s.ntiles < 1 || s.ring < 1 || s.ring % kPencilRing != 0 ||
        s.reach < 0 || s.reach + kPencilRing / 3 > s.ring || s.ext_ring < 2 * rpc || s.ext_ring % 2 != 0 ||
        kPencilZeroBytes + s.ring * kPencilSlotBytes + s.ext_ring * bs * 8 > kLdsBytes || s.nexch < 0 || s.nexch > nb)
        return BILU_ERR_STATE;
    if (static_cast<int>(s.tile_ptr.size()) != s.ntiles + 1 || s.tile_ptr[0] != 0 || s.tile_ptr[s.ntiles] != s.nchunks ||
        static_cast<int>(s.ext_ptr.size()) != s.ntiles + 1 || s.ext_ptr[0] != 0 || s.ext_ptr[s.ntiles] != s.next)
        return BILU_ERR_STATE;
    if (s.rows.size() != nslots || s.entry.size() != nslots || s.meta.size() != nslots * w4 * 4 ||
        s.src.size() != nslots * s.width || s.ext_idx.size() != static_cast<size_t>(s.next) ||
        s.ext_free.size() != static_cast<size_t>(s.next))
        return BILU_ERR_STATE;
    for (int t = 0; t < s.ntiles; ++t)
        if (s.tile_ptr[t + 1] <= s.tile_ptr[t] || s.ext_ptr[t + 1] < s.ext_ptr[t]) return BILU_ERR_STATE;
    auto word = [&](int c, int q, int w) {
        return static_cast<uint32_t>(s.meta[((static_cast<size_t>(c) * w4 + w / 4) * rpc + q) * 4 + w % 4]);
    };
    auto needed = [&](int c) { return static_cast<int>(word(c, 0, (s.width + 1) / 2)); };
    // every row once, idle slots last, exchange entries distinct
    std::vector<int32_t> tile_of(static_cast<size_t>(nb), -1), of_entry(static_cast<size_t>(s.nexch), -1);
    for (int t = 0; t < s.ntiles; ++t)
        for (int c = s.tile_ptr[t]; c < s.tile_ptr[t + 1]; ++c) {
            for (int q = 0; q < rpc; ++q) {
                const int32_t i = s.rows[static_cast<size_t>(c) * rpc + q];
                const int32_t e = s.entry[static_cast<size_t>(c) * rpc + q];
                if (i >= nb || i < -1 || e < -1 || e >= s.nexch) return BILU_ERR_STATE;
                if (i >= 0 && q > 0 && s.rows[static_cast<size_t>(c) * rpc + q - 1] < 0) return BILU_ERR_STATE;
                if (needed(c) != static_cast<int>(word(c, q, (s.width + 1) / 2))) return BILU_ERR_STATE;
                if (i < 0) {
                    if (e != -1) return BILU_ERR_STATE;
                    continue;
                }
                if (tile_of[i] != -1) return BILU_ERR_STATE;
                tile_of[i] = t;
                if (e >= 0) {
                    if (of_entry[e] != -1) return BILU_ERR_STATE;
                    of_entry[e] = i;
                }
            }
        }
    std::vector<int32_t> ndep(static_cast<size_t>(nb), 0);
    const int w = s.which;
    const bool rowwise = (w == BILU_SWEEP_L || w == BILU_SWEEP_U);
    for (int32_t i = 0; i < nb; ++i) {
        if (tile_of[i] < 0) return BILU_ERR_STATE;
        for (int32_t e = h.Pp[i]; e < h.Pp[i + 1]; ++e) {
            const int32_t j = h.Pj[e];
            if (j == i) continue;
            const bool lower = j < i;
            if (lower == (w == BILU_SWEEP_L || w == BILU_SWEEP_LT)) ndep[rowwise ? i : j]++;
        }
    }
    for (int t = 0; t < s.ntiles; ++t) {
        const int c0 = s.tile_ptr[t], n = s.tile_ptr[t + 1] - c0;
        const int e0 = s.ext_ptr[t], ne = s.ext_ptr[t + 1] - e0;
        // fed rows: of earlier tiles; a place is reused only after its last
        // reader, which needs no row from the new one on
        for (int j = 0; j < ne; ++j) {
            const int f = s.ext_free[e0 + j];
            if (f < 0 || f > n) return BILU_ERR_STATE;
            if (f > 0 && needed(c0 + f - 1) > j) return BILU_ERR_STATE;
            const int32_t x = s.ext_idx[static_cast<size_t>(e0 + j)];
            if (x < 0 || x >= s.nexch || of_entry[x] < 0 || tile_of[of_entry[x]] >= t) return BILU_ERR_STATE;
        }
        int prev = 0;
        for (int i = 0; i < n; ++i) {
            const int c = c0 + i;
            const int need = needed(c);
            if (need < prev || need > ne) return BILU_ERR_STATE;
            prev = need;
            for (int q = 0; q < rpc; ++q) {
                const int32_t row = s.rows[static_cast<size_t>(c) * rpc + q];
                int found = 0;
                int32_t last = -1;
                for (int k = 0; k < s.width; ++k) {
                    const uint32_t two = word(c, q, k / 2);
                    const int code = static_cast<int>(k % 2 ? two >> 16 : two & 0xffffu);
                    const int32_t e = s.src[(static_cast<size_t>(c) * s.width + k) * rpc + q];
                    if (code == 0 && e == -1) continue;
                    if (row < 0 || code < kPencilZeroBytes || e < 0 || e >= nP) return BILU_ERR_STATE;
                    const int off = code - kPencilZeroBytes;
                    int32_t j;
                    if (off < s.ring * kPencilSlotBytes) {
                        const int slot = off / kPencilSlotBytes, in = off % kPencilSlotBytes;
                        if (in % (bs * 8) != 0 || in / (bs * 8) >= rpc) return BILU_ERR_STATE;
                        const int back = ((i - 1 - slot) % s.ring + s.ring) % s.ring;
                        const int o = i - 1 - back;        // the last chunk written there
                        if (o < 0 || i - o > s.reach) return BILU_ERR_STATE;
                        j = s.rows[static_cast<size_t>(c0 + o) * rpc + in / (bs * 8)];
                    } else {
                        const int in = off - s.ring * kPencilSlotBytes;
                        if (in % (bs * 8) != 0 || in / (bs * 8) >= s.ext_ring) return BILU_ERR_STATE;
                        const int es = in / (bs * 8);
                        const int back = ((need - 1 - es) % s.ext_ring + s.ext_ring) % s.ext_ring;
                        const int o = need - 1 - back;
                        if (o < 0) return BILU_ERR_STATE;
                        // not overwritten before this chunk has read it
                        if (o + s.ext_ring < ne && s.ext_free[e0 + o + s.ext_ring] < i + 1) return BILU_ERR_STATE;
                        j = of_entry[s.ext_idx[static_cast<size_t>(e0 + o)]];
                    }
                    if (j < 0) return BILU_ERR_STATE;
                    const int32_t pi = h.Prow[e], pj = h.Pj[e];
                    if (rowwise ? (pi != row || pj != j) : (pi != j || pj != row)) return BILU_ERR_STATE;
                    if (pi == pj || (pj < pi) != (w == BILU_SWEEP_L || w == BILU_SWEEP_LT)) return BILU_ERR_STATE;
                    // ascending columns, the order in which every sweep sums (and
                    // so none twice)
                    if (j <= last) return BILU_ERR_STATE;
                    last = j;
                    ++found;
                }
                if (row >= 0 && found != ndep[row]) return BILU_ERR_STATE;
            }
        }
    }
    return BILU_OK;
}

}  // namespace bilu
