// M2M and L2L at sign-class orders (from 6 on) by parity classes.
//
// The child octants of a box differ from octant 7 (all centre offsets positive)
// by the axes m they negate, and a translation matrix satisfies
//   TM_(7^m) = R_m TM_7 R_m,   R_m = +-1 by the parities of the exponents on m,
// so one matrix serves the eight octants:
//   M2M  Mh(parent)_c = sum_a TM_7[a][c] H_(pi(a)^pi(c))[a],
//        H_s = sum_m (-1)^|m & s| Mh(child 7^m)
//   L2L  Lh(child 7^m)_c += sum_pi (-1)^|m & (pi^pi(c))| z_pi[c],
//        z_pi[c] = sum_(a in class pi) GH_7[a][c] Lh(parent)_a,
// with pi(a) the parity class of component a: one (p+1)^2 square product per
// parent and an eight-point transform instead of eight products, and one matrix
// read per 16 parents instead of eight.  What bounds them is the traffic of the
// expansions (each read or written once per level) and, at levels of few
// parents, the latency of one wavefront's chain: its loads are issued together
// (the children's codes, their rows), and blocks are one wavefront, since four on
// one CU wait for each other's scattered rows (a launch of order 8, few parents:
// M2M 14 us with four, 7 with one; L2L 14 and 9; order 12: 29 and 11, 29 and 20).
// The eight-matrix kernels they replace read 8 (p+1)^4 entries per 16 parents
// (3.2 MB at p = 14) and, for the L2L, the parent's vector once per row tile and
// octant.  Launches of one evaluation, those -> these: 17,389 Plummer points, p = 8,
// M2M 88 -> 41 us, L2L 67 -> 53; 250,000, p = 12, 197 -> 111 and 411 -> 360 beside the
// P2P; 4e6, p = 14, 1.96 -> 0.42 ms and, with the pass before it, 5.5 -> 3.8 ms.
//
// Matrices are stored in operand order: TMS[ks][tile][lane], GHS[tile][ks][lane],
// lane (k, c) holding the entry of column 4 ks + k (parity-sorted) and row
// 16 tile + c (sym_tile_class order).
#include "ops.h"
#include "sym_engine.h"

namespace fmm {

namespace {

template <int P> struct TShape {
    static constexpr int RT = sym_row_tiles(P), KS = sym_ksteps(P), KSV = (KS + 1) / 2, LD = folded_ld(P);
    int rc[RT] = {}, kc[2 * KSV + 2] = {};
    uint64_t tau[3][2] = {};
    int pad[LD / 4] = {}; // bit i of pad[n]: position 4 n + i of a folded row holds no component
    constexpr TShape()
    {
        for (int r = 0; r < RT; ++r) rc[r] = sym_tile_class(P, r, true);
        int k = 0;
        for (int c = 0; c < 8; ++c)
            for (int t = 0; t < sym_class_ksteps(P, c); ++t) {
                for (int b = 0; b < 3; ++b) tau[b][k / 64] |= (uint64_t)((c >> b) & 1) << (k % 64);
                for (int g = 0; g < 4; ++g) // (column 4 k + g of the sorted order)
                    if (4 * t + g < sym_class_count(P, c)) pad[sym_pos(k, g, 2) / 4] |= 1 << sym_pos(k, g, 2) % 4;
                kc[k++] = c;
            }
        for (int n = 0; n < LD / 4; ++n) pad[n] ^= 15;
    }
};

// +-1 as a scalar: (-1)^(bit & 1)
__device__ inline double pm1(uint32_t bit) { return __longlong_as_double((long long)(0x3ff0000000000000ull | ((uint64_t)bit << 63))); }
__device__ inline uint32_t odd_parity(uint32_t x) { return __popc(x) & 1; }

// children of `parent` by negated axes: ch[m] the child in octant 7 ^ m, or -1.
// Children are in octant order, so one's place is the number of octants present
// below its own.  No branches: the eight codes are loaded at once (a wait for each
// took 5 us of a launch at levels of few parents).
__device__ inline void children_by_axes(const PlanView &v, int parent, int (&ch)[8])
{
    const int cb = gptr(v.child_begin)[max(parent, 0)], ncd = parent >= 0 ? gptr(v.nchild)[max(parent, 0)] : 0;
    uint32_t code[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) code[i] = (uint32_t)gptr(v.morton)[max(cb + min(i, ncd - 1), 0)];
    uint32_t have = 0; // octants present
#pragma unroll
    for (int i = 0; i < 8; ++i) have |= i < ncd ? 1u << (code[i] & 7) : 0u;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const uint32_t o = 7 ^ m;
        ch[m] = (have >> o) & 1 ? cb + __popc(have & ((1u << o) - 1)) : -1;
    }
}

} // namespace

// ---------------- M2M ----------------
// A wavefront takes 16 parents of a level: the children's folded vectors are
// the members of a sign class, their transform the B operands, the matrix
// streamed from L2 (each operand refilled for the next k-step after its MFMA).
// Levels of few 16-parent groups give every row tile a wavefront of its own
// (m2m_tile_waves): it needs one output of the transform per k-step, a signed sum.
template <int P>
__global__ __launch_bounds__(64) void k_m2m_sym(const PlanView *V, Bases B, int level)
{
    using TS = TShape<P>;
    static constexpr TS S{};
    constexpr int RT = TS::RT, KSV = TS::KSV, LD = TS::LD;
    const int k = find_plan(B, blockIdx.x);
    const PlanView &v = V[k];
    const int lane = threadIdx.x, col = lane & 15, kq = lane >> 4;
    const int lb = v.lvl_nonleaf_off[level], le = v.lvl_nonleaf_off[level + 1];
    const int groups = (le - lb + 15) / 16, split = m2m_tile_waves(RT, groups);
    const int item = blockIdx.x - B.b[k];
    if (item >= groups * split) return;
    const int g = item / split, mt0 = item - g * split;
    const int pidx = lb + 16 * g + col;
    const int parent = pidx < le ? gptr(v.lvl_nonleaf)[pidx] : -1;
    int ch[8];
    children_by_axes(v, parent, ch);
    uint32_t src[8]; // byte offsets of the members' rows (plans check the 4 GiB bound); absent ones read the zero row
#pragma unroll
    for (int m = 0; m < 8; ++m)
        src[m] = (uint32_t)(ch[m] >= 0 ? ch[m] : v.nboxes) * (uint32_t)(8 * LD) + 16u * (uint32_t)kq;
    const auto Mg = gptr((const char *)v.Mh);
    const auto A = gptr(v.tab->TMS) + lane;
    const auto rpos = gptr(v.tab->rpos);
    const auto out = gptr(v.Mh) + (int64_t)max(parent, 0) * LD;
    if (mt0 == 0 && parent >= 0) // padding positions of the parents' rows
#pragma unroll
        for (int n = 0; n < LD / 4; ++n)
            if (S.pad[n] && ((S.pad[n] >> kq) & 1)) out[4 * n + kq] = 0.0;
    if (split == 1) {
        double4_t acc[RT];
        double ac[RT], h[2][8], sg[2][3];
        double2v_t raw[8];
#pragma unroll
        for (int t = 0; t < RT; ++t) acc[t] = double4_t{0, 0, 0, 0};
#pragma unroll
        for (int m = 0; m < 8; ++m) raw[m] = *(gp<const double2v_t>)(Mg + src[m]);
#pragma unroll
        for (int t = 0; t < RT; ++t) ac[t] = A[t * 64];
#pragma unroll 1
        for (int j = 0; j < KSV; ++j) {
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const int ks = 2 * j + w;
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    uint64_t bits = S.tau[b][0];
                    if constexpr (TS::KS > 64) bits = ks >= 64 ? S.tau[b][1] : bits;
                    sg[w][b] = pm1((uint32_t)(bits >> (ks & 63)) & 1u);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int w = 0; w < 2; ++w) {
#pragma unroll
                for (int m = 0; m < 8; ++m) h[w][m] = raw[m][w];
                signed_butterflies<0>(h[w], sg[w]);
            }
            __builtin_amdgcn_sched_barrier(0);
            const int jn = min(j + 1, KSV - 1);
#pragma unroll
            for (int w = 0; w < 2; ++w)
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ac[t], h[w][S.rc[t]], acc[t], 0, 0, 0);
                    ac[t] = A[(int64_t)((2 * j + w + 1) * RT + t) * 64];
                    if (w == 0 && t < 8) {
                        asm volatile("" : "+v"(src[t]));
                        raw[t] = *(gp<const double2v_t>)(Mg + (uint64_t)src[t] + 64 * jn);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
        static_assert(RT >= 8, "a load after each of the first eight MFMAs");
        if (parent < 0) return;
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int pos = rpos[16 * t + 4 * r + kq];
                if (pos >= 0) out[pos] = acc[t][r];
            }
        return;
    }
    // one row tile
    constexpr int NB = 6; // vectors in flight
    const uint32_t rho = (uint32_t)S.rc[mt0];
    double srho[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) srho[m] = pm1(odd_parity((uint32_t)m & rho));
    double2v_t raw[NB][8];
    double a[NB][2];
    auto load = [&](int b, int j) {
#pragma unroll
        for (int m = 0; m < 8; ++m) raw[b][m] = *(gp<const double2v_t>)(Mg + (uint64_t)src[m] + 64 * j);
#pragma unroll
        for (int w = 0; w < 2; ++w) a[b][w] = A[(int64_t)((2 * j + w) * RT + mt0) * 64];
    };
    double4_t acc = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < NB && j < KSV; ++j) load(j, j);
#pragma unroll
    for (int j = 0; j < KSV; ++j) {
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const int tau = S.kc[2 * j + w];
            double s = 0.0;
#pragma unroll
            for (int m = 0; m < 8; ++m)
                s = fma(odd_parity((uint32_t)(m & tau)) ? -srho[m] : srho[m], raw[j % NB][m][w], s);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[j % NB][w], s, acc, 0, 0, 0);
        }
        if (j + NB < KSV) load(j % NB, j + NB);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (parent < 0) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int pos = rpos[16 * mt0 + 4 * r + kq];
        if (pos >= 0) out[pos] = acc[r];
    }
}

// ---------------- L2L ----------------
// A wavefront takes 16 parents of a level and some of the row tiles
// (l2l_tile_waves): the parents' vectors stay in registers (one k-step's operand
// per lane each), each tile accumulates the eight column classes apart, and the
// transform over them gives the eight children, their rows completed on the way
// where no pass has done so (l2l_completes).
template <int P>
__global__ __launch_bounds__(64) void k_l2l_sym(const PlanView *V, Bases B, int level)
{
    using TS = TShape<P>;
    static constexpr TS S{};
    constexpr int RT = TS::RT, KS = TS::KS, LDH = pad16(nharm(P)), NB = kGHSAhead;
    const int k = find_plan(B, blockIdx.x);
    const PlanView &v = V[k];
    const int lane = threadIdx.x, col = lane & 15, kq = lane >> 4;
    const int lb = v.lvl_nonleaf_off[level], le = v.lvl_nonleaf_off[level + 1];
    const int groups = (le - lb + 15) / 16, split = l2l_tile_waves(RT, groups);
    const int item = blockIdx.x - B.b[k];
    if (item >= groups * split) return;
    const int g = item / split, sp = item - g * split, t0 = RT * sp / split, t1 = RT * (sp + 1) / split;
    const int pidx = lb + 16 * g + col;
    const int parent = pidx < le ? gptr(v.lvl_nonleaf)[pidx] : -1;
    const auto scol = gptr(v.tab->scol), srow = gptr(v.tab->srow);
    const auto A = gptr(v.tab->GHS) + lane;
    double ar[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) ar[i] = A[(int64_t)(t0 * KS + i) * 64];
    int c[4]; // the lane's components in the row tile
#pragma unroll
    for (int r = 0; r < 4; ++r) c[r] = srow[16 * t0 + 4 * r + kq];
    double x[KS];
    {
        const auto X = gptr(v.Lh) + (int64_t)max(parent, 0) * LDH;
        int ci[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) ci[ks] = scol[4 * ks + kq];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) x[ks] = X[max(ci[ks], 0)]; // (padding columns meet zeros of the matrix)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) x[ks] = ci[ks] >= 0 && parent >= 0 ? x[ks] : 0.0;
    }
    int ch[8];
    children_by_axes(v, parent, ch);
    // which children's rows hold something (bit m), and a second part's sums
    // (bit 8 + m)
    uint32_t have = 0xffu;
    const bool completes = l2l_completes(P, v.m2l_parts), two = completes && v.m2l_parts > 1;
    if (completes) {
        have = 0;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int b = max(ch[m], 0);
            const bool hv = gptr(v.V_off)[b + 1] > gptr(v.V_off)[b], hx = gptr(v.X_off)[b + 1] > gptr(v.X_off)[b];
            have |= (uint32_t)(hv || hx) << m | (uint32_t)(hv && two) << (8 + m);
        }
    }
    const auto Lh = gptr(v.Lh), Lh2 = gptr(v.Lh2);
    for (int t = t0; t < t1; ++t) {
        // the children's rows are requested before the products, all at once (absent
        // children and padding rows read something valid that is not used)
        double old[8][4];
        auto rows = [&](double(&d)[8][4], auto L) {
#pragma unroll
            for (int m = 0; m < 8; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) d[m][r] = L[(int64_t)max(ch[m], 0) * LDH + max(c[r], 0)];
        };
        rows(old, Lh);
        int cn[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) cn[r] = srow[16 * min(t + 1, RT - 1) + 4 * r + kq];
        __builtin_amdgcn_sched_barrier(0);
        double4_t z[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) z[q] = double4_t{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            z[S.kc[ks]] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[ks % NB], x[ks], z[S.kc[ks]], 0, 0, 0);
            ar[ks % NB] = A[(int64_t)(t * KS + ks + NB) * 64]; // (the next tile's follow; padded past the last)
        }
        if constexpr (KS % NB != 0) { // the next tile's first operands back to their places
            double tmp[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) tmp[i] = ar[(KS + i) % NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) ar[i] = tmp[i];
        }
#pragma unroll
        for (int st = 1; st < 8; st <<= 1)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (!(i & st)) {
                    const double4_t u = z[i], w = z[i | st];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        z[i][r] = u[r] + w[r];
                        z[i | st][r] = u[r] - w[r];
                    }
                }
#pragma unroll
        for (int m = 0; m < 8; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) old[m][r] = (have >> m) & 1 ? old[m][r] : 0.0;
        if (two) { // (uniform) the second part's sums
            double part[8][4];
            rows(part, Lh2);
#pragma unroll
            for (int m = 0; m < 8; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) old[m][r] += (have >> (8 + m)) & 1 ? part[m][r] : 0.0;
        }
        const uint32_t rho = (uint32_t)S.rc[t];
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            if (ch[m] < 0) continue;
            const double s = pm1(odd_parity((uint32_t)m & rho));
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (c[r] >= 0) Lh[(int64_t)ch[m] * LDH + c[r]] = fma(s, z[m][r], old[m][r]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) c[r] = cn[r];
    }
}

#define DISPATCH_SYM(p, KERNEL, ...)                                                   \
    switch (p) {                                                                       \
    case 6: KERNEL<6> __VA_ARGS__; break;  case 7: KERNEL<7> __VA_ARGS__; break;     \
    case 8: KERNEL<8> __VA_ARGS__; break;  case 9: KERNEL<9> __VA_ARGS__; break;     \
    case 10: KERNEL<10> __VA_ARGS__; break; case 11: KERNEL<11> __VA_ARGS__; break;  \
    case 12: KERNEL<12> __VA_ARGS__; break; case 13: KERNEL<13> __VA_ARGS__; break;  \
    case 14: KERNEL<14> __VA_ARGS__; break; case 15: KERNEL<15> __VA_ARGS__; break;  \
    default: KERNEL<16> __VA_ARGS__; break;                                            \
    }

void launch_m2m_sym(int p, const PlanView *V, const Bases &B, int level, hipStream_t s)
{
    if (B.b[B.n]) DISPATCH_SYM(p, k_m2m_sym, <<<(unsigned)B.b[B.n], 64, 0, s>>>(V, B, level));
}
void launch_l2l_sym(int p, const PlanView *V, const Bases &B, int level, hipStream_t s)
{
    if (B.b[B.n]) DISPATCH_SYM(p, k_l2l_sym, <<<(unsigned)B.b[B.n], 64, 0, s>>>(V, B, level));
}

} // namespace fmm
