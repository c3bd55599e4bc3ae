// faces.h -- the open-boundary kernels: outlet collision with the corrected
// velocity (eqs. 22-23), alpha-corrected inlet (eqs. 13-19), column-mean
// outflow velocity and convective outflow (eqs. 20-21).
//
// One wave works on one face node in 3-D and on two in 2-D: the lanes hold
// the populations of both components, one direction per lane, and sums over
// directions are lane reductions.  The face of a domain is small (hundreds to
// some ten thousand nodes) and in the caller's layout every population of an
// x-face node lies in a memory line of its own, so nothing is lost by giving
// neighbouring lanes different directions, and the dependent chain of a node
// shrinks to: slot table -> population -> lane sums -> store.  With one
// thread per node (19 x 2 gathers, all directions unrolled, 64-bit index
// divisions, some thousand instructions run once by a lone wave) the launches
// of the 150x30x30 device took 27.6 + 10.5 + 10.3 us for 900 face nodes.
// The slot of every population comes from a table built at creation, so no
// coordinates, type words or bounce-back tests are formed here.
#pragma once

#include "lattice.h"
#include "params.h"

namespace lbm {

// Bit j: lane j's direction has component `sign` along axis a.
template <int DIM>
__host__ __device__ constexpr uint32_t lane_mask(int a, int sign)
{
    uint32_t m = 0;
    for (int j = 0; j < Lat<DIM>::Q; j++)
        if (Lat<DIM>::E[lane_dir<DIM>(j)][a] == sign) m |= 1u << j;
    return m;
}

// What a lane of a face wave stands for.
template <int DIM> struct FaceLane {
    int sub;        // node of the wave
    int k;          // component
    int j;          // lane within the component, clamped to Q - 1
    bool on;        // the lane holds a population
    bool rest, axial;
    int dir;        // its direction
    float e[3], w;

    __device__ __forceinline__ FaceLane()
    {
        constexpr int Q = Lat<DIM>::Q, GL = FaceMap<DIM>::GL;
        const int t = (int)threadIdx.x & 63;
        sub = t / (2 * GL);
        k = (t / GL) & 1;
        const int l = t % GL;
        on = l < Q;
        j = on ? l : Q - 1;
        rest = l == Q - 1;
        axial = l < 2 * DIM;
        dir = lane_dir<DIM>(j);
        const uint32_t bit = on ? 1u << l : 0u;
        static_for<3>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            e[a] = (bit & lane_mask<DIM>(a, 1)) ? 1.0f : ((bit & lane_mask<DIM>(a, -1)) ? -1.0f : 0.0f);
        });
        w = rest ? weight<DIM>(0) : (axial ? weight<DIM>(1) : 1.0f / 36.0f);
    }
};

template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

// The value of the opposite direction (the neighbouring lane; 0 for the rest
// population, whose neighbour holds none).
__device__ __forceinline__ float lane_opp(float v) { return dpp<0xB1>(v); }

// Sum over the lanes of one component (every lane gets the same bits: each
// step adds a pair of equal-sized partial sums, in either order).
template <int DIM>
__device__ __forceinline__ float lane_sum(float v)
{
    v += dpp<0xB1>(v);       // lane ^ 1
    v += dpp<0x4E>(v);       // lane ^ 2
    v += dpp<0x141>(v);      // the other four of eight
    v += dpp<0x140>(v);      // the other eight of sixteen
    if constexpr (DIM == 3) v += __shfl_xor(v, 16, 64);
    return v;
}

// The value that the other component's lane of the same direction holds.
template <int DIM>
__device__ __forceinline__ float lane_other(float v) { return __shfl_xor(v, FaceMap<DIM>::GL, 64); }

__device__ __forceinline__ float lane_pick(const float (&v)[3], int a) { return a == 0 ? v[0] : (a == 1 ? v[1] : v[2]); }

// rho and J of one component from the populations its lanes hold.  The
// momentum sums the differences of opposite populations (exact, the two are
// close); both lanes of a pair hold that difference, hence the half.
template <int DIM>
__device__ __forceinline__ void lane_moments(const FaceLane<DIM> &L, float f, float &rho, float (&J)[3])
{
    const float d = f - lane_opp(f);
    rho = lane_sum<DIM>(f);
    static_for<3>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        J[a] = a < DIM ? 0.5f * lane_sum<DIM>(L.e[a] * d) : 0.0f;
    });
}

template <int DIM>
__device__ __forceinline__ float lane_feq(const FaceLane<DIM> &L, float rho, const float (&u)[3])
{
    const float eu = L.e[0] * u[0] + L.e[1] * u[1] + L.e[2] * u[2];
    const float uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    return rho * L.w * (1.0f + 3.0f * eu + 4.5f * eu * eu - 1.5f * uu);
}

// eq. (1) for the direction of this lane.  Every even moment but e and eps
// relaxes with s_nu and every odd one but j with s_q, so the collision is a
// plain relaxation of the even and odd parts of f plus the projections on
// the rows e, eps and j with the difference of the rates:
//   f* = f - [ s_nu (f+ - feq+) - (1 - s_nu/2) F+ + T_e c_e + T_eps c_eps ]
//          - [ s_q  (f- - feq-) - (1 - s_q/2)  F- + e . c_j ]
// with F the forcing of eq. (9) and f+ / f- the half sum / difference of the
// opposite populations, relaxed apart and then added.  sa: sum of f over the axis directions, f0: the rest
// population.
template <int DIM>
__device__ __forceinline__ float lane_collide(const FaceLane<DIM> &L, float f, float rho, float sa, float f0,
                                              const float (&J)[3], const float (&u)[3], const float (&F)[3],
                                              const Rates &s)
{
    const float uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const float uF = u[0] * F[0] + u[1] * F[1] + u[2] * F[2];
    const float eu = L.e[0] * u[0] + L.e[1] * u[1] + L.e[2] * u[2];
    const float eF = L.e[0] * F[0] + L.e[1] * F[1] + L.e[2] * F[2];
    const float fo = L.rest ? f : lane_opp(f);
    const float wr = L.w * rho;
    const float even = 0.5f * (f + fo) - wr * (1.0f + 4.5f * eu * eu - 1.5f * uu);
    const float odd = 0.5f * (f - fo) - wr * (3.0f * eu);
    const float Fe = L.w * (9.0f * eu * eF - 3.0f * uF), Fo = L.w * (3.0f * eF);
    const float sd = rho - f0 - sa;
    float ne, np, t1, t2, ij;
    if constexpr (DIM == 3) {
        ne = (-30.0f * f0 - 11.0f * sa + 8.0f * sd - rho * (-11.0f + 19.0f * uu) + 19.0f * uF) * (s.se - s.snu) *
             (1.0f / tnorm<3>(1));
        np = (12.0f * f0 - 4.0f * sa + sd - rho * (3.0f - 5.5f * uu) - 5.5f * uF) * (s.seps - s.snu) *
             (1.0f / tnorm<3>(2));
        t1 = L.rest ? -30.0f : (L.axial ? -11.0f : 8.0f);
        t2 = L.rest ? 12.0f : (L.axial ? -4.0f : 1.0f);
        ij = 1.0f / tnorm<3>(3);
    } else {
        ne = (-4.0f * f0 - sa + 2.0f * sd - rho * (-2.0f + 3.0f * uu) + 3.0f * uF) * (s.se - s.snu) *
             (1.0f / tnorm<2>(1));
        np = (4.0f * f0 - 2.0f * sa + sd - rho * (1.0f - 3.0f * uu) - 3.0f * uF) * (s.seps - s.snu) *
             (1.0f / tnorm<2>(2));
        t1 = L.rest ? -4.0f : (L.axial ? -1.0f : 2.0f);
        t2 = L.rest ? 4.0f : (L.axial ? -2.0f : 1.0f);
        ij = 1.0f / tnorm<2>(3);
    }
    float ec = 0.0f;
    static_for<3>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        ec += L.e[a] * (J[a] - rho * u[a] + 0.5f * F[a]);
    });
    const float dev = s.snu * even - (1.0f - 0.5f * s.snu) * Fe + (t1 * ne + t2 * np);
    const float dod = s.sq * odd - (1.0f - 0.5f * s.sq) * Fo + (1.0f - s.sq) * ij * ec;
    const float fe = 0.5f * (f + fo) - dev, fd = 0.5f * (f - fo) - dod;
    return fe + fd;
}

// chi of eq. (23); undefined (no outflow through x_{N-1}, or flow against the
// inlets) leaves the outlet uncorrected.
__device__ __forceinline__ double chi_of(double qin, double qout)
{
    return (fabs(qout) < 1e-30 || qin * qout <= 0.0) ? 1.0 : qin / qout;
}

// ---------------------------------------------------------------------------
// eq. (23) from the sums the node update left in acc (this step's parity):
// every thread of the first face launch forms chi itself; one thread records
// Q_in, Q' and chi and clears the sums of the other parity for the next step.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double chi_from(const Boundary &bd, const unsigned long long *acc,
                                           unsigned long long *next, bool record)
{
    const double qin = flow_unfix(acc[0]), qout = flow_unfix(acc[1]);
    const double chi = (bd.has_outlet && bd.chi_on) ? chi_of(qin, qout) : 1.0;
    if (record) {
        bd.scal[SC_QIN] = qin;
        bd.scal[SC_QOUT] = qout;
        bd.scal[SC_CHI] = chi;
        next[0] = 0ull;
        next[1] = 0ull;
    }
    return chi;
}

// First record of this wave in block blk.
template <int DIM>
__device__ __forceinline__ int face_first(int blk)
{
    constexpr int WPB = FACE_NT / 64, NPW = FaceMap<DIM>::NPW;
    return (blk * WPB + ((int)threadIdx.x >> 6)) * NPW;
}

// ---------------------------------------------------------------------------
// The collision of the outlet column with eq. (22) for a given chi (eq. 23):
// outlet record r by this wave (live: the lane's node exists and is this
// block's to store).  Returns the lane's population as a reader of the stored
// value gets it.
// ---------------------------------------------------------------------------
template <int DIM, int STORE>
__device__ __forceinline__ float outlet_collide(const FaceLane<DIM> &L, int r, bool live,
                                                const typename Codec<STORE>::T *__restrict__ src,
                                                typename Codec<STORE>::T *__restrict__ dst,
                                                const float2 *__restrict__ psi, const float2 *__restrict__ ref,
                                                const Geometry &g, const Physics &ph, const Boundary &bd,
                                                int *__restrict__ flag, double chi)
{
    constexpr int Q = Lat<DIM>::Q;
    const Rates rates = {L.k == 0 ? ph.se[0] : ph.se[1], L.k == 0 ? ph.seps[0] : ph.seps[1], ph.sq,
                         L.k == 0 ? ph.snu[0] : ph.snu[1]};
    const OutletRec rec = bd.out[r];
    const int *tab = bd.out_tab + (int64_t)r * (4 * Q);
    float rr = 0.0f, rd = 0.0f;
    const int slot = tab[L.j];
    if constexpr (Codec<STORE>::REF) {
        const float2 a = ref[rec.bN], b = psi[tab[2 * Q + L.j]];
        rr = L.k == 0 ? a.x : a.y;
        rd = L.k == 0 ? b.x : b.y;
    }
    const float raw = Codec<STORE>::ld(src + (int64_t)L.k * Q * g.Ppad + slot, L.w, rr);
    const float *fF = bd.faceF + (int64_t)rec.slotN * 6 + 3 * L.k;
    const float F[3] = {fF[0], fF[1], fF[2]};
    const float up = rec.slotP >= 0 ? bd.faceU[rec.slotP] : 0.0f;
    const float f = L.on ? raw : 0.0f;
    float rho, J[3], u[3];
    lane_moments<DIM>(L, f, rho, J);
    const float sa = lane_sum<DIM>(L.axial ? f : 0.0f), f0 = lane_sum<DIM>(L.rest ? f : 0.0f);
    const float rt = rho + lane_other<DIM>(rho);
    static_for<3>([&](auto dc) {
        constexpr int d = decltype(dc)::value;
        const float m = J[d] + 0.5f * F[d];
        u[d] = (m + lane_other<DIM>(m)) / rt;
    });
    if (rec.slotP >= 0) {
        // eq. (22): the outward velocity is chi times that of x_{N-1}
        const float un = (float)(chi * (double)up) * bd.out_sign;
        static_for<3>([&](auto dc) {
            constexpr int d = decltype(dc)::value;
            u[d] = bd.out_axis == d ? un : u[d];
        });
    }
    if (live && (!(rt > 0.0f) || !isfinite(rt) || !isfinite(u[0] + u[1] + u[2]))) *flag = 1;
    float fs = lane_collide<DIM>(L, f, rho, sa, f0, J, u, F, rates);
    // the rest population is the residual of the density (see collide_pairs2)
    const float moving = lane_sum<DIM>(L.on && !L.rest ? fs : 0.0f);
    if (L.rest) fs = rho - moving;
    if (live && L.on) Codec<STORE>::st(dst + ((int64_t)L.k * Q + L.dir) * g.Ppad + rec.pN, fs, L.w, rd);
    return Codec<STORE>::held(fs, L.w, rd);
}

template <int DIM, int STORE>
__device__ __forceinline__ void outlet_body(int blk, const typename Codec<STORE>::T *__restrict__ src,
                                            typename Codec<STORE>::T *__restrict__ dst,
                                            const float2 *__restrict__ psi, const float2 *__restrict__ ref,
                                            const Geometry &g, const Physics &ph, const Boundary &bd,
                                            int *__restrict__ flag, double chi)
{
    const FaceLane<DIM> L;
    const int r0 = face_first<DIM>(blk);
    if (r0 >= bd.n_out) return;                         // uniform over the wave
    const bool live = r0 + L.sub < bd.n_out;
    (void)outlet_collide<DIM, STORE>(L, live ? r0 + L.sub : r0, live, src, dst, psi, ref, g, ph, bd, flag, chi);
}

// ---------------------------------------------------------------------------
// The entering populations of the inlet nodes (eqs. 13-19).
// ---------------------------------------------------------------------------
template <int DIM, int STORE>
__device__ __forceinline__ void inlet_body(int blk, typename Codec<STORE>::T *__restrict__ dst,
                                           const float2 *__restrict__ psi, const Geometry &g, const Boundary &bd)
{
    constexpr int Q = Lat<DIM>::Q;
    const FaceLane<DIM> L;
    typename Codec<STORE>::T *dk = dst + (int64_t)L.k * Q * g.Ppad;
    const int r0 = face_first<DIM>(blk);
    if (r0 >= bd.n_in) return;                      // uniform over the wave
    const bool live = r0 + L.sub < bd.n_in;
    const int r = live ? r0 + L.sub : r0;
    const InletRec rec = bd.in[r];
    const int *tab = bd.in_tab + (int64_t)r * (2 * Q);
    const int slot1 = tab[L.j], slot2 = tab[Q + L.j];
    const Patch pt = bd.patch[rec.patch];
    // f(t+1) is read with psi(t) as the reference density
    float rr1 = 0.0f, rr2 = 0.0f;
    if constexpr (Codec<STORE>::REF) {
        const float2 a = psi[rec.b1], b = psi[rec.b2];
        rr1 = L.k == 0 ? a.x : a.y;
        rr2 = L.k == 0 ? b.x : b.y;
    }
    const float *fF1 = bd.faceF + (int64_t)rec.slot1 * 6 + 3 * L.k;
    const float F1[3] = {fF1[0], fF1[1], fF1[2]};
    const float ea = lane_pick(L.e, pt.axis);
    const bool enter = ea * (float)pt.sign > 0.0f;
    // the populations that leave x1 (the entering ones are replaced, and
    // their slots are not read) and all those of x2
    const float raw1 = L.on && !enter ? Codec<STORE>::ld(dk + slot1, L.w, rr1) : 0.0f;
    const bool x2 = rec.x2_fluid != 0;
    const float f2 = L.on && x2 ? Codec<STORE>::ld(dk + slot2, L.w, rr2) : 0.0f;
    const float *fF2 = bd.faceF + (int64_t)rec.slot2 * 6 + 3 * L.k;
    const float F2[3] = {fF2[0], fF2[1], fF2[2]};
    float rho2, J2[3], u2[3];
    lane_moments<DIM>(L, f2, rho2, J2);
    const float rt = rho2 + lane_other<DIM>(rho2);
    static_for<3>([&](auto dc) {
        constexpr int d = decltype(dc)::value;
        const float m = J2[d] + 0.5f * F2[d];
        u2[d] = (m + lane_other<DIM>(m)) / rt;
    });
    // eq. (13)/(14) on the populations entering the domain
    const float un = (float)pt.sign * pt.u_n;
    const float up[3] = {pt.axis == 0 ? un : 0.0f, pt.axis == 1 ? un : 0.0f, pt.axis == 2 ? un : 0.0f};
    const float rho_p = L.k == 0 ? pt.rho[0] : pt.rho[1];
    const float neq = x2 ? f2 - lane_feq<DIM>(L, rho2, u2) : 0.0f;
    float f1 = enter ? lane_feq<DIM>(L, rho_p, up) + neq : raw1;
    // eqs. (15)-(19): alpha_i = w_i sum_d e_id dJ_d / D_d over the entering
    // set, dJ = rho_k^p u^p - (sum_i e_i f_i + F^k/2); D is the sum of the
    // entering weights with e_id != 0: 1/6 along the normal, 1/18 across
    float rr, J[3], a = 0.0f;
    lane_moments<DIM>(L, f1, rr, J);
    static_for<DIM>([&](auto dc) {
        constexpr int d = decltype(dc)::value;
        const float dJ = rho_p * up[d] - (J[d] + 0.5f * F1[d]);
        a += L.e[d] * dJ * (pt.axis == d ? 6.0f : 18.0f);
    });
    if (pt.alpha_on) f1 += L.w * a;
    if (live && enter) Codec<STORE>::st(dk + slot1, f1, L.w, rr1);
}

// ---------------------------------------------------------------------------
// eq. (21): the outward normal velocity at x' of record rec from the
// populations f its lanes hold.
// ---------------------------------------------------------------------------
template <int DIM>
__device__ __forceinline__ float xprime_un(const FaceLane<DIM> &L, const OutletRec &rec, float f, const Boundary &bd)
{
    const float Fn = rec.slotP >= 0 ? bd.faceF[(int64_t)rec.slotP * 6 + 3 * L.k + bd.out_axis] : 0.0f;
    const float d = f - lane_opp(f);
    const float rho = lane_sum<DIM>(f);
    const float J = 0.5f * lane_sum<DIM>(lane_pick(L.e, bd.out_axis) * d);
    const float rt = rho + lane_other<DIM>(rho);
    const float m = J + 0.5f * Fn;
    return bd.out_sign * (m + lane_other<DIM>(m)) / rt;
}

// The block's partial sum, and how many nodes it holds.  One lane per node
// carries its term.
template <int DIM>
__device__ __forceinline__ void uc_store(const FaceLane<DIM> &L, int blk, bool term, float un, const Boundary &bd)
{
    __shared__ double s_red[2 * FACE_NT / 64];
    const bool carry = term && L.k == 0 && L.on && L.j == 0;
    double su = carry ? (double)un : 0.0, cnt = carry ? 1.0 : 0.0;
    block_sum2<FACE_NT>(su, cnt, s_red);
    if (threadIdx.x == 0) {
        bd.ucpart[2 * blk] = su;
        bd.ucpart[2 * blk + 1] = cnt;
    }
}

template <int DIM, int STORE>
__device__ __forceinline__ void uc_body(int blk, const typename Codec<STORE>::T *__restrict__ dst,
                                        const float2 *__restrict__ psi, const Geometry &g, const Boundary &bd)
{
    constexpr int Q = Lat<DIM>::Q;
    const FaceLane<DIM> L;
    float un = 0.0f;
    bool term = false;
    const int r0 = face_first<DIM>(blk);
    if (r0 < bd.n_out) {                                // uniform over the wave
        const bool live = r0 + L.sub < bd.n_out;
        const int r = live ? r0 + L.sub : r0;
        const OutletRec rec = bd.out[r];
        const bool x1 = rec.slotP >= 0;
        const int slot = bd.out_tab[(int64_t)r * (4 * Q) + Q + L.j];
        float rr = 0.0f;
        if constexpr (Codec<STORE>::REF) {
            const float2 a = psi[rec.bP];
            rr = L.k == 0 ? a.x : a.y;
        }
        un = xprime_un<DIM>(L, rec, L.on && x1 ? Codec<STORE>::ld(dst + (int64_t)L.k * Q * g.Ppad + slot, L.w, rr) : 0.0f,
                            bd);
        term = live && x1;
    }
    uc_store<DIM>(L, blk, term, un, bd);
}

// ---------------------------------------------------------------------------
// Outlet collision and eq. (21) sums in one launch (2-D, see UcMap).  What x'
// takes from the outlet column comes through LDS, as the stored value reads;
// the rest was stored by the node update and is loaded with the outlet's own
// populations.  Saves the launch that summed eq. (21) (4.4 of 18.3 us of the
// 800x100 T-junction's step).
// ---------------------------------------------------------------------------
template <int STORE>
__device__ __forceinline__ void outlet_uc_body(int blk, const typename Codec<STORE>::T *__restrict__ src,
                                               typename Codec<STORE>::T *__restrict__ dst,
                                               const float2 *__restrict__ psi, const float2 *__restrict__ ref,
                                               const Geometry &g, const Physics &ph, const Boundary &bd,
                                               int *__restrict__ flag, double chi)
{
    constexpr int Q = Lat<2>::Q;
    __shared__ float s_f[UcMap::NS * 2 * Q];
    const FaceLane<2> L;
    const int s = ((int)threadIdx.x >> 6) * FaceMap<2>::NPW + L.sub;      // node of the block
    const int first = blk * UcMap::INNER - 1, want = first + s;
    const bool mine = s >= 1 && s <= UcMap::INNER && want < bd.n_out;
    const int r = min(max(want, 0), bd.n_out - 1);
    const OutletRec rec = bd.out[r];
    const bool x1 = rec.slotP >= 0;
    const int *tab = bd.out_tab + (int64_t)r * (4 * Q);
    const int from = bd.chi_on ? tab[3 * Q + L.j] : -1;
    float rr = 0.0f;
    if constexpr (Codec<STORE>::REF) {
        const float2 a = psi[rec.bP];
        rr = L.k == 0 ? a.x : a.y;
    }
    float f = 0.0f;
    if (L.on && x1 && from < 0) f = Codec<STORE>::ld(dst + (int64_t)L.k * Q * g.Ppad + tab[Q + L.j], L.w, rr);
    if (bd.chi_on) {                                    // else the node update collided the outlet column
        const float h = outlet_collide<2, STORE>(L, r, mine, src, dst, psi, ref, g, ph, bd, flag, chi);
        if (L.on) s_f[(s * 2 + L.k) * Q + L.j] = h;
        __syncthreads();
        if (L.on && x1 && from >= 0 && mine) f = s_f[((from - first) * 2 + L.k) * Q + L.j];
    }
    const float un = xprime_un<2>(L, rec, f, bd);
    uc_store<2>(L, blk, mine && x1, un, bd);
}

// ---------------------------------------------------------------------------
// eq. (20) for the populations entering through the outlet: EL lanes per
// component and node, one entering direction each.
// ---------------------------------------------------------------------------
template <int DIM, int STORE>
__device__ __forceinline__ void outlet_fill_body(int blk, typename Codec<STORE>::T *__restrict__ dst,
                                                 const float2 *__restrict__ psi, const Geometry &g,
                                                 const Boundary &bd)
{
    constexpr int Q = Lat<DIM>::Q, EL = FillMap<DIM>::EL, NE = FillMap<DIM>::NE;
    __shared__ double s_red[2 * FACE_NT / 64];
    const int t = (int)threadIdx.x, r = blk * FillMap<DIM>::NPB + t / (2 * EL);
    const int k = (t / EL) & 1, m = t % EL;
    const bool live = r < bd.n_out && m < NE;
    // everything that does not need U_c is loaded before its sum
    float prev = 0.0f, fp = 0.0f, rd = 0.0f, w = 0.0f, *h = nullptr;
    typename Codec<STORE>::T *at = nullptr;
    bool inside = false;
    if (live) {
        const int j = (int)((bd.out_enter >> (8 * m)) & 0xff);
        const int i = lane_dir<DIM>(j);
        w = j < 2 * DIM ? weight<DIM>(1) : 1.0f / 36.0f;      // an entering direction is never at rest
        const OutletRec rec = bd.out[r];
        const int *tab = bd.out_tab + (int64_t)r * (4 * Q) + j;
        typename Codec<STORE>::T *dk = dst + (int64_t)k * Q * g.Ppad;
        inside = rec.slotP >= 0;
        at = dk + tab[0];
        h = bd.hist + ((int64_t)k * Q + i) * bd.n_slots + rec.slotN;
        // f(t) of x_N from the FP32 history; f(t+1) is stored for x_N with
        // psi(t) as its reference density, and x' is read at t+1 with psi(t)
        float rp = 0.0f;
        if constexpr (Codec<STORE>::REF) {
            const float2 a = psi[rec.bN], b = psi[rec.bP];
            rd = k == 0 ? a.x : a.y;
            rp = k == 0 ? b.x : b.y;
        }
        prev = *h;
        if (inside) fp = Codec<STORE>::ld(dk + tab[Q], w, rp);
    }
    double su, cnt;
    reduce_partials<FACE_NT>(bd.ucpart, bd.n_ucpart, su, cnt, s_red);
    double Uc = cnt > 0.0 ? su / cnt : 0.0;
    const bool clamped = Uc < 0.0;
    if (clamped) Uc = 0.0;
    if (blk == 0 && t == 0) {
        bd.scal[SC_UC] = Uc;
        if (clamped) bd.scal[SC_CLAMPS] += 1.0;
    }
    if (!live) return;
    const float uc = (float)Uc;
    const float v = inside ? (prev + uc * fp) / (1.0f + uc) : prev;
    *h = v;
    Codec<STORE>::st(at, v, w, rd);
}

template <int DIM, int STORE>
__global__ __launch_bounds__(FACE_NT) void k_outlet_fill(typename Codec<STORE>::T *__restrict__ dst,
                                                         const float2 *__restrict__ psi, Geometry g, Boundary bd)
{
    outlet_fill_body<DIM, STORE>((int)blockIdx.x, dst, psi, g, bd);
}

// ---------------------------------------------------------------------------
// k_faces: the first launch after the node update.  chi from this step's
// sums; blocks [0, nb_out) collide the outlet column (and sum eq. 21 where
// bd.uc_early), blocks [nb_out, nb_out + nb_in) rebuild inlet nodes (only when no inlet node pulls from the
// outlet column, checked at creation, so the two sets are independent).
// ---------------------------------------------------------------------------
template <int DIM, int STORE>
__device__ __forceinline__ void faces_body(int blk, const typename Codec<STORE>::T *__restrict__ src,
                                           typename Codec<STORE>::T *__restrict__ dst,
                                           const float2 *__restrict__ psi, const float2 *__restrict__ ref,
                                           const Geometry &g, const Physics &ph, const Boundary &bd,
                                           int *__restrict__ flag, const unsigned long long *__restrict__ acc,
                                           unsigned long long *__restrict__ next, int nb_out, int nb_in)
{
    if (blk < nb_out || blk == 0) {
        const double chi = chi_from(bd, acc, next, blk == 0 && threadIdx.x == 0);
        if (blk < nb_out) {
            if constexpr (DIM == 2) {
                if (bd.uc_early) {
                    outlet_uc_body<STORE>(blk, src, dst, psi, ref, g, ph, bd, flag, chi);
                    return;
                }
            }
            outlet_body<DIM, STORE>(blk, src, dst, psi, ref, g, ph, bd, flag, chi);
            return;
        }
    }
    if (blk - nb_out < nb_in) inlet_body<DIM, STORE>(blk - nb_out, dst, psi, g, bd);
}

template <int DIM, int STORE>
__global__ __launch_bounds__(FACE_NT) void k_faces(const typename Codec<STORE>::T *__restrict__ src,
                                                   typename Codec<STORE>::T *__restrict__ dst,
                                                   const float2 *__restrict__ psi, const float2 *__restrict__ ref,
                                                   Geometry g, Physics ph, Boundary bd, int *__restrict__ flag,
                                                   const unsigned long long *__restrict__ acc,
                                                   unsigned long long *__restrict__ next, int nb_out, int nb_in)
{
    faces_body<DIM, STORE>((int)blockIdx.x, src, dst, psi, ref, g, ph, bd, flag, acc, next, nb_out, nb_in);
}

// ---------------------------------------------------------------------------
// k_inlet: blocks [0, nb_in) take the inlet nodes that k_faces did not,
// blocks [nb_in, ...) the partial sums of eq. (21) (neither: not launched).
// ---------------------------------------------------------------------------
template <int DIM, int STORE>
__device__ __forceinline__ void inlet_uc_body(int blk, typename Codec<STORE>::T *__restrict__ dst,
                                              const float2 *__restrict__ psi, const Geometry &g, const Boundary &bd,
                                              int nb_in)
{
    if (blk < nb_in) inlet_body<DIM, STORE>(blk, dst, psi, g, bd);
    else uc_body<DIM, STORE>(blk - nb_in, dst, psi, g, bd);
}

template <int DIM, int STORE>
__global__ __launch_bounds__(FACE_NT) void k_inlet(typename Codec<STORE>::T *__restrict__ dst,
                                                   const float2 *__restrict__ psi, Geometry g, Boundary bd,
                                                   int nb_in)
{
    inlet_uc_body<DIM, STORE>((int)blockIdx.x, dst, psi, g, bd, nb_in);
}

}  // namespace lbm
