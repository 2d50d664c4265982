// Launchers of the evaluation kernels (see ops.hip and m2l.hip).  Every
// launcher takes the device array of plan views and the block split.
#pragma once
#include <string>
#include "common.h"

namespace fmm {
void launch_permute_q(const PlanView *V, const Bases &B, hipStream_t s);   // 256 particles/block
void launch_p2m(int p, const PlanView *V, const Bases &B, hipStream_t s);  // 1 leaf/block
void launch_p2m_fold(int p, const PlanView *V, const Bases &B, hipStream_t s); // 64 leaves/block
void launch_l2lh(int p, const PlanView *V, const Bases &B, int level, hipStream_t s); // 16 parents x 16 rows/block (harmonic rows)
void launch_lh_init(const PlanView *V, const Bases &B, hipStream_t s);        // 4 boxes/block
void launch_lh_zero(const PlanView *V, const Bases &B, hipStream_t s);        // 512 doubles/block
void launch_m2mh(int p, const PlanView *V, const Bases &B, int level, hipStream_t s); // 16 parents/block
// Row-tile groups per 16-parent M2M group: levels with few parents spread the
// mt row tiles of each group over up to mt blocks (powers of two dividing mt)
// until the level has about 512 blocks.
__host__ __device__ inline int m2m_row_split(int mt, int groups)
{
    int r = 1;
    while (2 * r <= mt && mt % (2 * r) == 0 && groups * r < 512) r *= 2;
    return r;
}
// Sign-class orders (translate.hip), a wavefront per block.  M2M: wavefronts per
// 16-parent group: one per row tile where the level's groups would leave SIMDs
// idle, else one for all mt tiles (each reads all the children).  A launch with one
// per tile | one for all: order 8, 32 groups 10 | 21 us, 104 groups 16 | 20, 256 groups
// 42 | 26; order 12, 42 groups 23 | 43; order 14, 64 groups 50 | 56, 141 groups 94 | 56,
// 714 groups 378 | 80.
void launch_m2m_sym(int p, const PlanView *V, const Bases &B, int level, hipStream_t s);
void launch_l2l_sym(int p, const PlanView *V, const Bases &B, int level, hipStream_t s);
__host__ __device__ inline int m2m_tile_waves(int mt, int groups) { return groups <= 64 ? mt : 1; }
// L2L: the row tiles of a group spread over up to mt wavefronts until the level
// has about 2048 (two per SIMD).  A launch with one wavefront per group | until
// 1024 | 2048 | 4096 | one per tile: order 8, 104 groups 25 | 17 | 21 | 20 | 21 us, 256 groups
// 43 | 52 | 57 | 57 | 57; order 12, 36 groups 85 | 27 | 27 | 26 | 27; order 14, all levels,
// beside P2P and M2P, 3.65 | 3.92 | 3.81 | 4.07 | 3.82 ms.
__host__ __device__ inline int l2l_tile_waves(int mt, int groups)
{
    const int n = groups > 0 ? 2048 / groups : 1;
    return n < 1 ? 1 : n < mt ? n : mt;
}
void launch_parent_mh(const PlanView *V, const Bases &B, int full, hipStream_t s); // 4 boxes/block
void launch_unfold(int p, const PlanView *V, const Bases &B, int leaves_only, hipStream_t s); // kRemapBoxes boxes/block
void launch_p2l(int p, const PlanView *V, const Bases &B, hipStream_t s);  // 1 X target/block
void launch_p2l_transform(const PlanView *V, const Bases &B, hipStream_t s); // 16 X targets x 16 rows/block
void launch_far(int p, int fld, const PlanView *V, const Bases &B, hipStream_t s);  // 2 leaves/block (L2P + output)
// 1 leaf with a W list/block, of four wavefronts or (one) of one
constexpr int kM2POneWave = 8192; // such leaves of a plan from which it is one
void launch_m2p(int p, int fld, int one, const PlanView *V, const Bases &B, hipStream_t s);
// P2P runs in two parts (leaves [0, split) and [split, nleaves)), each
// overlapping a latency-bound phase of the far field
__host__ __device__ inline int p2p_split(int nleaves) { return (int)((int64_t)nleaves * 5 / 8) & ~3; }
// mixed: 0 FP64, 1 FP32 terms, 2 softened kernel (FP64); fld (here, in
// launch_far and launch_m2p): 0 when no plan of the launch asks for the field
void launch_p2p(int mixed, int fld, int part, const PlanView *V, const Bases &B, hipStream_t s); // 1 leaf/block
void launch_zero(double *p, int64_t n, hipStream_t s);
void launch_zero_f32(float *p, int64_t n, hipStream_t s);
void launch_m2l(int p, int f32, const PlanView *V, const Bases &B, hipStream_t s); // 64 slots/block
constexpr int kM2LSlots = 64;
// rotation-based M2L (rotation.hip): device factors of order p (built on
// first use, kept for the process), blocks per 64-target tile, launcher
const RotTables *get_rotation_tables(int p, std::string &err);
int m2l_rot_blocks_per_tile(int p);
void launch_m2l_rot(int p, const PlanView *V, const Bases &B, hipStream_t s);
constexpr int kRemapBoxes = 16; // boxes per block of the unfold
} // namespace fmm
