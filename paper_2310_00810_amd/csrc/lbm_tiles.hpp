// Tiles of the time-blocked D2Q9 kernels: planning and the tile table.  Host
// code without HIP.
#pragma once

#include <stddef.h>

#include <algorithm>
#include <vector>

namespace lbm {

constexpr int MS_MAX = 6;

// Per tile: instance, first column and row, the number of the list's nodes
// within distance d of the tile, and the tile's first list entry.  The list
// holds up to two entries a node of the whole batch, whose size only memory
// bounds: 64 bits.
struct MTileDesc {
    int b, x0, y0;
    int cnt[MS_MAX + 1];
    long long list;
    int pad[4];
};
static_assert(sizeof(MTileDesc) == 64, "tiles do not straddle cache lines");

// A set of tiles: steps per launch at most (0: single-step kernels), large
// region, number of tiles.
struct Blocks {
    int ms = 0, big = 0, n_tiles = 0;
    long long n_entries = 0;  // list entries at most
    size_t off_tile = 0, off_list = 0;
    int ex() const { return big ? 64 : 32; }
    int ey() const { return big ? 32 : 16; }
    int tx() const { return ex() - 2 * ms; }
    int ty() const { return ey() - 2 * ms; }
    // nodes along one axis of n nodes within ms of the tile of t nodes at v
    int extent(int v, int n, int t, bool periodic) const {
        const int lo = v - ms, hi = std::min(v + t, n) + ms;
        return periodic ? hi - lo : std::min(hi, n) - std::max(lo, 0);
    }
    // adds an instance of nx x ny nodes
    void count(int nx, int ny, bool xper, bool yper) {
        long long lx = 0, ly = 0;     // region nodes of all tiles = (sum of widths) x (sum of heights)
        int ntx = 0, nty = 0;
        for (int x = 0; x < nx; x += tx(), ++ntx) lx += extent(x, nx, tx(), xper);
        for (int y = 0; y < ny; y += ty(), ++nty) ly += extent(y, ny, ty(), yper);
        n_tiles += ntx * nty;
        n_entries += lx * ly;
    }
};

// The table of B's tiles over the instances (members nx, ny), with the first
// list entry of each.
template <class I>
std::vector<MTileDesc> tile_table(const Blocks &B, const std::vector<I> &inst, bool xper, bool yper) {
    std::vector<MTileDesc> out;
    out.reserve(B.n_tiles);
    long long at = 0;
    for (int b = 0; b < (int)inst.size(); ++b)
        for (int y = 0; y < inst[b].ny; y += B.ty())
            for (int x = 0; x < inst[b].nx; x += B.tx()) {
                MTileDesc e{};
                e.b = b; e.x0 = x; e.y0 = y; e.list = at;
                at += (long long)B.extent(x, inst[b].nx, B.tx(), xper) * B.extent(y, inst[b].ny, B.ty(), yper);
                out.push_back(e);
            }
    return out;
}

}  // namespace lbm
