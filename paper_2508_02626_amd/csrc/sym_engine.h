// Inner loop of the sign-class M2L kernels that keep one wavefront per SIMD
// (k_m2l_symh, k_m2l_soft_sym): the products of one sign class for a
// wavefront's 16 targets, every row tile in its registers.
//
// What bounds it: instruction issue of the one wavefront.  A 16x16x4 FP64 MFMA
// holds the SIMD's vector unit for its 64 cycles: no vector instruction, of this
// wavefront or another, runs beside it, and the first one after an MFMA costs
// 12 cycles, each next one 4 (measured); LDS reads, loads and scalar
// instructions are free.  So the vector work is kept small (transforms without
// sign selection, one LDS address per pair of row tiles) and in one block per
// operand vector (two k-steps), and everything else is issued between MFMAs.
// Reading every member from 16 hot rows, or every table entry from a
// conflict-free address, changes the time by 2% at most.
// Coulomb, 4e6 Plummer points, p = 14: 22.8 ms with the reads and their
// addresses before each k-step, 26.8 with the vector work interleaved an MFMA at
// a time, 20.1 in this form, of which the MFMAs are 14.6.  Softened, p = 8:
// 1e6 Plummer points, the launch 6.5 -> 5.7 ms with this loop alone, 2.7 of it
// MFMAs (then 4.3 by its block set-up and tiles, soft.hip).
//
// A shape SH gives: RT row tiles (rc: parity class of each), KS k-steps (kc:
// column class tau of each, tau: its bits per axis as masks over the k-steps),
// KSV = ceil(KS / 2) operand vectors, RP pairs of row tiles (pr: pair of each
// row tile).  A pair is tile t of the row class (x, y, 0) and tile t of
// (x, y, 1): the rows of the second have the z exponents of the first's plus one,
// in the same order, so their table addresses differ by ZOFF bytes alone.
#pragma once
#include "common.h"

#include <type_traits>

namespace fmm {

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef double double2v_t __attribute__((ext_vector_type(2)));

template <class SH> constexpr SH kShape{}; // (evaluated once)

// For zero axes Z: the row tiles whose products with a column class of value
// GV = tau & Z exist, ordered by pair, with their pairs, and the groups of
// k-steps: gk is tau & Z of a k-step (-1 past the last), uniform_vectors(j) the
// number of vectors from j on whose k-steps and the one after them have the
// value of k-step 2j.
template <class SH, int Z, int GV> struct SymTiles {
    int n, t[SH::RT], p[SH::RT];
    bool used[SH::RP];
    constexpr SymTiles() : n(0), t(), p(), used()
    {
        constexpr const SH &S = kShape<SH>;
        for (int q = 0; q < SH::RP; ++q)
            for (int r = 0; r < SH::RT; ++r)
                if (S.pr[r] == q && (S.rc[r] & Z) == GV) {
                    used[q] = true;
                    p[n] = q;
                    t[n++] = r;
                }
    }
};
template <class SH, int Z> struct SymGroups {
    static constexpr int gk(int ks)
    {
        constexpr const SH &S = kShape<SH>;
        return ks < SH::KS ? S.kc[ks] & Z : -1;
    }
    static constexpr int uniform_vectors(int j)
    {
        const int g = gk(2 * j);
        int n = 0;
        while (gk(2 * (j + n)) == g && gk(2 * (j + n) + 1) == g && gk(2 * (j + n) + 2) == g) ++n;
        return n;
    }
};

// Walsh-Hadamard transform of o over the axes not in Z, with signs s (+-1) of the
// axes folded in: output r is that of r ^ (the axes whose sign is -1)
template <int Z> __device__ __forceinline__ void signed_butterflies(double (&o)[8], const double (&s)[3])
{
#pragma unroll
    for (int st = 0; st < 3; ++st)
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (!((1 << st) & Z) && !(i & (1 << st)) && !(i & Z)) {
                const double u = o[i], x = o[i | (1 << st)];
                o[i] = fma(s[st], x, u);
                o[i | (1 << st)] = fma(-s[st], x, u);
            }
}

// One class with zero axes Z.  D + dbase: its table in LDS; Ho: byte offsets of
// the lane's columns (KS + 4 entries readable); hb: of the lane's rows, per pair;
// raw[m]: member m's operand vector 0 (in flight; members negating a zero axis
// are not read).  load(m, j) requests vector j of member m into raw[m];
// offsets() prepares and load_next(m) requests the next class's vector 0.  Row
// tiles from F32T on run on FP32 MFMA.
//
// K-steps whose column class tau agrees on Z (a group: the same row tiles run)
// share one code path: the transform output r ^ tau of a row class r is output r
// of the transform of the members with (-1)^|m & tau| folded into the
// butterflies (u + s w, u - s w, s = +-1 a scalar; the same roundings), so tau is
// a run-time value.
template <class SH, int Z, int F32T, class Load, class Offsets, class LoadNext>
__device__ __forceinline__ void sym_run_class(const char *D, uint32_t dbase, const int *Ho, const int (&hb)[SH::RP],
                                              double4_t (&acc)[F32T],
                                              float4_t (&acc32)[SH::RT > F32T ? SH::RT - F32T : 1],
                                              double2v_t (&raw)[8], Load &&load, Offsets &&offsets, LoadNext &&load_next)
{
    typedef SymGroups<SH, Z> G;
    static constexpr SH S{};
    constexpr int RT = SH::RT, RP = SH::RP, KS = SH::KS, KSV = SH::KSV, N32 = RT - F32T;
    double h[2][8];            // transforms of the vector's k-steps
    double ac[RT];             // A operands of one k-step, in the order of its row tiles
    uint32_t ho1 = 0, ho2 = 0; // D offsets of k-steps 2j + 1 and 2j + 2
    double sg[2][3];           // signs of the vector's k-steps, by axis bit
    auto dread = [&](uint32_t a, int z) { return *(const double *)(D + (a + (z ? (uint32_t)SH::ZOFF : 0u))); };
    auto sign = [&](int ks, int bit) {
        uint64_t w = S.tau[bit][0];
        if constexpr (KS > 64) w = ks >= 64 ? S.tau[bit][1] : w;
        return __longlong_as_double((long long)(0x3ff0000000000000ull | ((w >> (ks & 63)) << 63)));
    };
    auto transform = [&](double (&o)[8], auto wc, const double (&s)[3]) {
        constexpr int w = decltype(wc)::value;
#pragma unroll
        for (int m = 0; m < 8; ++m) o[m] = (m & Z) ? 0.0 : raw[m][w];
        signed_butterflies<Z>(o, s);
    };
    // the MFMAs of one k-step (its transform hw, group value GC), back to back
    // (sched_barrier keeps what is between them there): each is followed by the
    // read that refills its A operand for the k-step of group value GN (-1:
    // none) at the addresses ad, and by side(i)
    auto products = [&](const double (&hw)[8], auto gcc, auto gnc, const uint32_t *ad, auto side) {
        constexpr SymTiles<SH, Z, decltype(gcc)::value> TC{};
        constexpr int GN = decltype(gnc)::value;
        constexpr SymTiles<SH, Z, (GN < 0 ? 0 : GN)> TN{};
        constexpr int nn = GN < 0 ? 0 : TN.n, slots = TC.n > nn ? TC.n : nn;
        static_assert(TC.n > 0, "a column class without row tiles");
        float hf[N32 > 0 ? 8 : 1], af[N32 > 0 ? RT : 1]; // FP32 tiles' operands
        if constexpr (N32 > 0) {
#pragma unroll
            for (int m = 0; m < 8; ++m) hf[m] = (float)hw[m];
#pragma unroll
            for (int i = 0; i < TC.n; ++i)
                if (TC.t[i] >= F32T) af[i] = (float)ac[i];
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < slots; ++i) {
            if (i < TC.n) {
                const int mt = TC.t[i];
                if (mt < F32T) acc[mt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ac[i], hw[S.rc[mt] & ~Z], acc[mt], 0, 0, 0);
                else if constexpr (N32 > 0)
                    acc32[mt - F32T] =
                        __builtin_amdgcn_mfma_f32_16x16x4f32(af[i], hf[S.rc[mt] & ~Z], acc32[mt - F32T], 0, 0, 0);
            }
            if (i < nn) ac[i] = dread(ad[TN.p[i]], S.rc[TN.t[i]] & 1);
            side(i);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto addresses = [&](uint32_t (&ad)[RP], uint32_t ho, auto gnc) {
        constexpr int GN = decltype(gnc)::value;
        if constexpr (GN >= 0) {
            constexpr SymTiles<SH, Z, GN> TN{};
#pragma unroll
            for (int r = 0; r < RP; ++r)
                if (TN.used[r]) {
                    ad[r] = (uint32_t)hb[r] + ho;
                    asm volatile("" : "+v"(ad[r])); // (the sum is formed here, not at its reads)
                }
        }
    };
    // vector j: groups of its k-steps (GB -1: one k-step only) and of the next
    // vector's first (-1: the class ends); LAST: the class's last vector
    auto vector = [&](int j, auto gac, auto gbc, auto gnc, auto lastc) {
        constexpr int GB = decltype(gbc)::value;
        constexpr bool LAST = decltype(lastc)::value;
        uint32_t ad1[RP], ad2[RP];
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : "+v"(ho1), "+v"(ho2)); // (waits for the reads here)
        transform(h[0], std::integral_constant<int, 0>{}, sg[0]);
        if constexpr (GB >= 0) transform(h[1], std::integral_constant<int, 1>{}, sg[1]);
        addresses(ad1, ho1 + dbase, gbc);
        addresses(ad2, ho2 + dbase, gnc);
        if constexpr (LAST) offsets();
        __builtin_amdgcn_sched_barrier(0);
        constexpr SymTiles<SH, Z, decltype(gac)::value> TA{};
        constexpr int PER = (8 + TA.n - 1) / TA.n; // loads per MFMA
        auto fetch = [&](int i) {
#pragma unroll
            for (int m = PER * i; m < PER * (i + 1); ++m) {
                if (m >= 8) continue;
                if constexpr (LAST) load_next(m);
                else if (!(m & Z)) load(m, j + 1);
            }
            if (i == 0) {
                ho1 = (uint32_t)Ho[2 * j + 3];
                ho2 = (uint32_t)Ho[2 * j + 4];
            }
        };
        constexpr SymTiles<SH, Z, (GB < 0 ? 0 : GB)> TB{};
        constexpr int PERS = (3 + TB.n - 1) / TB.n; // axes per MFMA
        auto next_signs = [&](int i) {
#pragma unroll
            for (int b = PERS * i; b < PERS * (i + 1); ++b) {
                if (b >= 3) continue;
                sg[0][b] = sign(2 * j + 2, b);
                sg[1][b] = sign(2 * j + 3, b);
            }
        };
        if constexpr (GB >= 0) {
            products(h[0], gac, gbc, ad1, fetch);
            products(h[1], gbc, gnc, ad2, next_signs);
        } else {
            products(h[0], gac, gnc, ad2, fetch);
        }
    };
    { // the first k-step's A operands
        constexpr SymTiles<SH, Z, G::gk(0)> T0{};
        uint32_t ad[RP];
        addresses(ad, (uint32_t)Ho[0] + dbase, std::integral_constant<int, G::gk(0)>{});
#pragma unroll
        for (int i = 0; i < T0.n; ++i) ac[i] = dread(ad[T0.p[i]], S.rc[T0.t[i]] & 1);
        ho1 = (uint32_t)Ho[1];
        ho2 = (uint32_t)Ho[2];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            sg[0][i] = sign(0, i);
            sg[1][i] = sign(1, i);
        }
    }
    // runs of vectors whose k-steps, and the one after, are of one group in a
    // loop, the others one by one
    auto run = [&](auto self, auto jc) {
        constexpr int J = decltype(jc)::value;
        if constexpr (J < KSV) {
            constexpr int N = G::uniform_vectors(J); // vectors J .. J + N - 1 alike, none the last
            using GA = std::integral_constant<int, G::gk(2 * J)>;
            if constexpr (N > 1) {
#pragma unroll 1
                for (int j = J; j < J + N; ++j) vector(j, GA{}, GA{}, GA{}, std::false_type{});
                self(self, std::integral_constant<int, J + N>{});
            } else {
                vector(J, GA{}, std::integral_constant<int, G::gk(2 * J + 1)>{},
                       std::integral_constant<int, G::gk(2 * J + 2)>{}, std::integral_constant<bool, J == KSV - 1>{});
                self(self, std::integral_constant<int, J + 1>{});
            }
        }
    };
    run(run, std::integral_constant<int, 0>{});
}

} // namespace fmm
