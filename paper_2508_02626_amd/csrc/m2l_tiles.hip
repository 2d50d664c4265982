// M2L target tiles: which 64 targets each M2L block takes, and in which
// order the blocks are laid out over the XCDs.  Kept apart from the tree and
// list kernels because the M2L kernels' memory traffic depends on it.
#include "tree_kernels.h"
#include "sort.h"

namespace fmm {

// ---------------- M2L target tiles ----------------
// Targets (boxes with a V list, ascending) are stably sorted by octant, then
// each octant group is placed at a multiple of 64 so that the 64 targets of
// one M2L block share one set of 189 offsets.  In a uniform tree the offsets a
// box actually has depend only on its octant and on its distance (0, 1, 2 or
// more cells) to each face of the root, so there the targets are also grouped
// by these distances (Morton order inside a group): the blocks near the faces
// then skip the offsets none of their targets has.  The tiles are then laid
// out region by region: the x-th eighth of every octant's tiles (a spatial
// region, as the tiles follow Morton order) forms the x-th eighth of the
// sequence, which the M2L launch hands to XCD x, so each XCD's L2 holds the
// multipoles of one region instead of those of the whole domain.  Inside a
// region the eight octants' tiles are dealt round-robin, so the blocks that
// run at the same time hold the children of the same parents, whose V lists
// draw on the same source boxes.
// by_level (the softened kernel's adaptive trees, whose tables depend on the
// level): every (octant, level) group starts a tile of its own, as the softened
// M2L kernels require (soft_tile_level): they run one level's tables per tile.
// Tiles across a level boundary ran the classes of both levels one after the other
// (1e6 Plummer points, 64 a leaf: 51 of 944 tiles, up to three times as long).
constexpr int kCatBits = 12;
constexpr int kTileLevels = kMaxDepth + 1;

__global__ __launch_bounds__(256) void k_oct_keys(const BoxArrays bx, const int32_t *tg, int nt, int uniform,
                                                  int by_level, uint64_t *key, int32_t *val)
{
    int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= nt) return;
    const int b = tg[i];
    uint64_t cat = by_level ? bx.level[b] : 0;
    if (uniform) {
        const int l = bx.level[b], side = 1 << l;
        int c[3];
        deinterleave(bx.morton[b], l, c);
        for (int k = 0; k < 3; ++k) {
            const int lo = c[k] < 3 ? c[k] : 3, hi = side - 1 - c[k] < 3 ? side - 1 - c[k] : 3;
            cat |= (uint64_t)(lo * 4 + hi) << (4 * k);
        }
    }
    key[i] = ((bx.morton[b] & 7) << kCatBits) | cat;
    val[i] = b;
}

// The groups (octants, or with by_level octants and levels) in the sorted keys:
// off.start[o][l] their first targets, off.tile[o][l] their first tiles within
// the octant's, off.tiles[o] the octant's tiles, off.first[x][o] the first tile
// of (region x, octant o) in the region-major sequence.
struct OctOffsets {
    int start[8][kTileLevels], tile[8][kTileLevels], tiles[8], first[8][8];
};
static_assert(sizeof(OctOffsets) <= kOctOffsetInts * sizeof(int), "octant offsets");

__global__ __launch_bounds__(256) void k_oct_offsets(const uint64_t *key, int nt, int by_level, OctOffsets *off)
{
    __shared__ int st[8 * kTileLevels + 1];
    const int nl = by_level ? kTileLevels : 1, ng = 8 * nl, g = threadIdx.x;
    static_assert(8 * kTileLevels < 256, "one group per thread");
    if (g <= ng) {
        const uint64_t k = (uint64_t)(g / nl) << kCatBits | (uint64_t)(g % nl);
        int lo = 0, hi = nt;
        while (lo < hi) {
            int mid = (lo + hi) >> 1;
            if (key[mid] < k) lo = mid + 1; else hi = mid;
        }
        st[g] = g == ng ? nt : lo;
    }
    __syncthreads();
    if (g < 8) { // the octant's tiles
        int t = 0;
        for (int l = 0; l < nl; ++l) {
            off->start[g][l] = st[g * nl + l];
            off->tile[g][l] = t;
            t += (st[g * nl + l + 1] - st[g * nl + l] + 63) / 64;
        }
        off->tiles[g] = t;
    }
    __syncthreads();
    if (g == 0) {
        int t = 0;
        for (int x = 0; x < 8; ++x)
            for (int k = 0; k < 8; ++k) {
                const int T = off->tiles[k];
                off->first[x][k] = t;
                t += (x + 1) * T / 8 - x * T / 8;
            }
    }
}

__global__ __launch_bounds__(256) void k_oct_place(const uint64_t *key, const int32_t *val, int nt,
                                                   int by_level, const OctOffsets *off, int32_t *slots)
{
    int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= nt) return;
    const int o = (int)(key[i] >> kCatBits), l = by_level ? (int)(key[i] & ((1 << kCatBits) - 1)) : 0;
    const int j = i - off->start[o][l], t = off->tile[o][l] + (j >> 6), T = off->tiles[o];
    int x = 0;
    while (x < 7 && t >= (x + 1) * T / 8) ++x;
    // within region x the octants' tiles are dealt round-robin: tile u of
    // octant o follows tile u of octants < o and precedes tile u + 1 of all
    const int u = t - x * T / 8;
    int pos = 0;
    for (int k = 0; k < 8; ++k) {
        const int n = (x + 1) * off->tiles[k] / 8 - x * off->tiles[k] / 8; // tiles of octant k in region x
        pos += min(n, u + (k < o ? 1 : 0));
    }
    const int tile = off->first[x][0] + pos;
    slots[(int64_t)tile * 64 + (j & 63)] = val[i];
}

void m2l_tiles(const BoxArrays &bx, const int32_t *tg, int nt, int uniform, int by_level, uint64_t *key, int32_t *val,
               uint64_t *tk, int32_t *tv, int32_t *sort_scratch, int *octoff, int32_t *slots,
               int64_t slot_cap, hipStream_t s)
{
    fill_i32(slots, slot_cap, -1, s);
    if (nt == 0) return;
    k_oct_keys<<<ceil_div(nt, 256), 256, 0, s>>>(bx, tg, nt, uniform, by_level, key, val);
    // (adaptive Coulomb trees have no category: the octant's digit alone)
    const int lo = uniform || by_level ? 0 : kCatBits, hi = kCatBits + 3;
    radix_sort_pairs(key, val, tk, tv, nt, lo, hi, sort_scratch, s);
    if (sort_lands_in_tmp(nt, lo, hi)) {
        key = tk;
        val = tv;
    }
    OctOffsets *off = (OctOffsets *)octoff;
    k_oct_offsets<<<1, 256, 0, s>>>(key, nt, by_level, off);
    k_oct_place<<<ceil_div(nt, 256), 256, 0, s>>>(key, val, nt, by_level, off, slots);
}

} // namespace fmm
