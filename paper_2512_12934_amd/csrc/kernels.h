// kernels.h -- device kernels of one lattice step (pull scheme).
//
// Storage.  Each population plane holds, at node x, the post-collision value
// f*_i(x, t) (not yet streamed), over a box padded by one node on every
// lattice axis; the padding holds the populations the open boundaries supply.
// The post-streaming distribution of eq. (2) is obtained by a gather:
//     f_i(x, t+1) = f*_i(x - e_i, t)        (periodic axes wrap)
//     f_i(x, t+1) = f*_ibar(x, t)           if x - e_i is solid (eq. B1)
//     f_i(x, t+1) = padding slot at x - e_i if that lies beyond an open face
// Two arrays alternate between source and destination every step.
//
// The launches of one step.  A closed domain takes one (fused mode) or two
// (two-pass mode), an open one at most five; k_inlet is left out where nothing
// remains for it, so an open 2-D step in the fused mode is usually three:
//   k_psi            (two-pass mode) psi_k = rho_k of every node into an array
//   k_main           all fluid nodes, swept along the last axis: densities of
//                    each plane plus a two-node lateral halo into an LDS ring
//                    (from the psi array, or recomputed from the populations
//                    in the fused mode; mirror ghost layers at open faces,
//                    eqs. 24-25), force
//                    (eqs. 10-11), common velocity (eqs. 7-8), MRT collision
//                    (eq. 1); the mass flows rho u.n of the inlet nodes and
//                    of the x_{N-1} nodes summed exactly (eq. 23)
//   k_faces          chi = Q_in / Q' (eq. 23) and the collision of the outlet
//                    column with the corrected normal velocity (eq. 22); the
//                    inlet nodes too when none of them pulls from the outlet
//                    column; in 2-D the partial sums of eq. (21) too where the
//                    face's order allows it (UcMap)
//   k_inlet          alpha-corrected NEQ extrapolation (eqs. 13-19) into the
//                    padding slots (the inlet nodes k_faces did not take);
//                    the partial sums of eq. (21) that k_faces did not take
//   k_outlet_fill    convective outflow (eq. 20) into the padding slots
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "lattice.h"
#include "params.h"

namespace lbm {

// ---------------------------------------------------------------------------
// Storage codecs.  A population is stored less an offset:
//   FP32:     f_i - w_i                         (the rest state at unit density)
//   binary16: f_i - w_i r, rounded to nearest even, where r is the previous
//             step's density of the component at the node that reads the
//             slot (the reference density, the same at write and at read).
// Near local equilibrium the stored numbers are then small for both the
// majority and the minority phase, so an 11-bit significand keeps the
// relative error of every population small; a fixed offset w_i would leave
// about 1% at a minority density of 0.03.  ld / st take the weight w and the
// reference density r of the reading node (FP32 ignores r).
//   binary16, fixed offset (storage 2): f_i - w_i, the offset as stated for
//             the precision extension, kept as a mode of its own so that its
//             error can be reported beside the reference-density codec.
// ---------------------------------------------------------------------------
template <int STORE> struct Codec;
template <> struct Codec<0> {
    using T = float;
    static constexpr bool REF = false;
    static __device__ __forceinline__ float ld(const T *p, float w, float) { return *p + w; }
    static __device__ __forceinline__ void st(T *p, float v, float w, float) { *p = v - w; }
    // what a reader of the stored value gets
    static __device__ __forceinline__ float held(float v, float w, float) { return (v - w) + w; }
};
template <> struct Codec<1> {
    using T = __half;
    static constexpr bool REF = true;
    static __device__ __forceinline__ float ld(const T *p, float w, float r) { return __half2float(*p) + w * r; }
    static __device__ __forceinline__ void st(T *p, float v, float w, float r) { *p = __float2half_rn(v - w * r); }
    static __device__ __forceinline__ float held(float v, float w, float r)
    {
        const T h = __float2half_rn(v - w * r);
        return __half2float(h) + w * r;
    }
};
template <> struct Codec<2> {
    using T = __half;
    static constexpr bool REF = false;
    static __device__ __forceinline__ float ld(const T *p, float w, float) { return __half2float(*p) + w; }
    static __device__ __forceinline__ void st(T *p, float v, float w, float) { *p = __float2half_rn(v - w); }
    static __device__ __forceinline__ float held(float v, float w, float)
    {
        const T h = __float2half_rn(v - w);
        return __half2float(h) + w;
    }
};

// Raw buffer access for the node update: one descriptor per component array
// (range-checked by the hardware), a 32-bit per-lane byte offset and a
// wave-uniform byte offset per population plane.
constexpr int BUF_FLAGS = 0x00020000;   // dword 3 of a raw gfx9 buffer descriptor

template <int STORE> struct Buf;
// Cache policy of the buffer accesses (the instruction's aux field): bit 1 is
// the non-temporal hint.  FP32 node-update stores are non-temporal: nothing
// reads them again within the launch, and keeping them out of the way of the
// gathers' neighbour lines was measured faster (binary16 stores, and
// non-temporal loads, were measured slower).
constexpr int CPOL_NT = 2;

// ld = dec(raw(...)): raw issues the load, dec turns the stored bits into the
// population, so a caller can put independent work between the two.
template <> struct Buf<0> {
    static constexpr uint32_t SZ = 4;
    using Raw = uint32_t;
    static __device__ __forceinline__ Raw raw(__amdgpu_buffer_rsrc_t r, uint32_t vo, int so)
    {
        return __builtin_amdgcn_raw_buffer_load_b32(r, (int)vo, so, 0);
    }
    static __device__ __forceinline__ float dec(Raw h, float w, float) { return __uint_as_float(h) + w; }
    static __device__ __forceinline__ float ld(__amdgpu_buffer_rsrc_t r, uint32_t vo, int so, float w, float rr)
    {
        return dec(raw(r, vo, so), w, rr);
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t vo, int so, float v, float w,
                                              float)
    {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v - w), r, (int)vo, so, CPOL_NT);
    }
};
template <> struct Buf<1> {
    static constexpr uint32_t SZ = 2;
    using Raw = unsigned short;
    static __device__ __forceinline__ Raw raw(__amdgpu_buffer_rsrc_t r, uint32_t vo, int so)
    {
        return __builtin_amdgcn_raw_buffer_load_b16(r, (int)vo, so, 0);
    }
    static __device__ __forceinline__ float dec(Raw h, float w, float rr)
    {
        return __half2float(__ushort_as_half(h)) + w * rr;
    }
    static __device__ __forceinline__ float ld(__amdgpu_buffer_rsrc_t r, uint32_t vo, int so, float w, float rr)
    {
        return dec(raw(r, vo, so), w, rr);
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t vo, int so, float v, float w,
                                              float rr)
    {
        __builtin_amdgcn_raw_buffer_store_b16(__half_as_ushort(__float2half_rn(v - w * rr)), r, (int)vo, so, 0);
    }
};

template <> struct Buf<2> {
    static constexpr uint32_t SZ = 2;
    using Raw = unsigned short;
    static __device__ __forceinline__ Raw raw(__amdgpu_buffer_rsrc_t r, uint32_t vo, int so)
    {
        return __builtin_amdgcn_raw_buffer_load_b16(r, (int)vo, so, 0);
    }
    static __device__ __forceinline__ float dec(Raw h, float w, float) { return __half2float(__ushort_as_half(h)) + w; }
    static __device__ __forceinline__ float ld(__amdgpu_buffer_rsrc_t r, uint32_t vo, int so, float w, float rr)
    {
        return dec(raw(r, vo, so), w, rr);
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t vo, int so, float v, float w, float)
    {
        __builtin_amdgcn_raw_buffer_store_b16(__half_as_ushort(__float2half_rn(v - w)), r, (int)vo, so, 0);
    }
};

template <int STORE>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t comp_rsrc(const void *base, int comp, int Q, int64_t Ppad)
{
    const char *p = (const char *)base + (int64_t)comp * Q * Ppad * Buf<STORE>::SZ;
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, (short)0, (int)((int64_t)Q * Ppad * Buf<STORE>::SZ),
                                             BUF_FLAGS);
}

__device__ __forceinline__ float pick3(const float (&v)[3], int a) { return a == 0 ? v[0] : (a == 1 ? v[1] : v[2]); }

template <int DIM>
__device__ __forceinline__ int e_axis(int i, int a)
{
    return a == 0 ? Lat<DIM>::E[i][0] : (a == 1 ? Lat<DIM>::E[i][1] : Lat<DIM>::E[i][2]);
}

// Padded index of box node (x, y, z); x = 0 sits xoff elements into each row
// so that rows start on a 128-byte line (see Geometry).
__device__ __forceinline__ int64_t pidx(const Geometry &g, int x, int y, int z)
{
    return (int64_t)(x + g.xoff) + (int64_t)g.P[0] * ((int64_t)(y + 1) + (int64_t)g.P[1] * (int64_t)(z + 1));
}

template <int DIM>
__device__ __forceinline__ int64_t dir_off(const Geometry &g, int i)
{
    return (int64_t)Lat<DIM>::E[i][0] + (int64_t)g.P[0] * ((int64_t)Lat<DIM>::E[i][1] +
                                                          (int64_t)g.P[1] * (int64_t)Lat<DIM>::E[i][2]);
}

// Padded index of the slot that supplies population i at box node (x,y,z)
// when no bounce-back applies: x - e_i with periodic wrap.
template <int DIM>
__device__ __forceinline__ int64_t src_slot(const Geometry &g, int x, int y, int z, int i)
{
    int s0 = x - Lat<DIM>::E[i][0], s1 = y - Lat<DIM>::E[i][1], s2 = z - Lat<DIM>::E[i][2];
    if (g.periodic[0]) s0 = s0 < 0 ? s0 + g.n[0] : (s0 >= g.n[0] ? s0 - g.n[0] : s0);
    if (g.periodic[1]) s1 = s1 < 0 ? s1 + g.n[1] : (s1 >= g.n[1] ? s1 - g.n[1] : s1);
    if (DIM == 3 && g.periodic[2]) s2 = s2 < 0 ? s2 + g.n[2] : (s2 >= g.n[2] ? s2 - g.n[2] : s2);
    if (DIM == 2) s2 = -1;
    return pidx(g, s0, s1, s2);
}

// Slot index (padded, within one component array) supplying population i.
template <int DIM>
__device__ __forceinline__ int64_t slot_of(const Geometry &g, int64_t p, uint32_t tw, int x, int y, int z, int i)
{
    if ((tw >> i) & 1u) return (int64_t)Lat<DIM>::OPP[i] * g.Ppad + p;
    return (int64_t)i * g.Ppad + ((tw & T_EDGE) ? src_slot<DIM>(g, x, y, z, i) : p - dir_off<DIM>(g, i));
}

// Post-streaming populations of one component at one node (pointer access).
// rr: the node's reference density of this component (see Codec).
template <int DIM, int STORE>
__device__ __forceinline__ void gather(const typename Codec<STORE>::T *__restrict__ fk, const Geometry &g,
                                       int64_t p, uint32_t tw, int x, int y, int z,
                                       float (&f)[Lat<DIM>::Q], float rr)
{
    static_for<Lat<DIM>::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        f[i] = Codec<STORE>::ld(fk + slot_of<DIM>(g, p, tw, x, y, z, i), weight<DIM>(i), rr);
    });
}

// Byte offset of population plane i within one component array, formed at
// its point of use by one scalar multiply.  The copy through an empty asm
// statement makes the stride opaque, so the compiler cannot hoist the 19
// products out of the node loop: held there, they took 19 scalar registers,
// the kernel ran out of them, and every access then read its offset back
// from a vector-register lane (v_readlane) and waited five cycles before
// the memory instruction could use it.  (The readfirstlane states that the
// stride is uniform, which the compiler does not see in every place; it
// leaves no instruction.)
template <int STORE>
__device__ __forceinline__ int plane_bytes(const Geometry &g, int i)
{
    int s = __builtin_amdgcn_readfirstlane((int)((uint32_t)g.Ppad * Buf<STORE>::SZ));
    asm volatile("" : "+s"(s));
    return s * i;
}

// Where the populations that stream into node p (pull) are stored, as byte
// offsets within one component: a[i] per lane, plus the wave-uniform offset
// so_i that uniform_plane() gives.  The wave takes the cheaper of two address
// forms that is valid for all its nodes:
// * no bounce-back and no periodic wrap (wave_fast): population i sits at
//   plane_i + p - off_i, so a[i] is the shifted lane offset and the plane is
//   the wave-uniform offset;
// * otherwise, per lane, the streamed slot (one step back along each axis,
//   around a periodic axis' end) or the node's own slot of the opposite
//   direction (bounce-back), selected without branches, with the plane in
//   a[i].  Slots formed one direction at a time from wrapped coordinates
//   cost a wave of a periodic 64x64 box 11,000 cycles, more than the rest of
//   its step.
// Only the addresses depend on the form; the loads are then issued in one
// straight run for both components, so no load is pending across a join of
// the forms (such a join would make the loads wait for earlier ones).
template <int DIM, int STORE>
__device__ __forceinline__ void gather_addr(const Geometry &g, uint32_t p, uint32_t tw, int x, int y, int z,
                                            bool wave_fast, uint32_t (&a)[Lat<DIM>::Q])
{
    constexpr uint32_t SZ = Buf<STORE>::SZ;
    const uint32_t sy = (uint32_t)g.P[0] * SZ, sz = (uint32_t)g.P[0] * (uint32_t)g.P[1] * SZ;
    if (wave_fast) {
        const uint32_t vb = (p - 1u) * SZ;
        static_for<Lat<DIM>::Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            constexpr int ex = Lat<DIM>::E[i][0], ey = Lat<DIM>::E[i][1], ez = Lat<DIM>::E[i][2];
            uint32_t vo = vb + (uint32_t)(1 - ex) * SZ;
            if constexpr (ey == 1) vo -= sy;
            if constexpr (ey == -1) vo += sy;
            if constexpr (ez == 1) vo -= sz;
            if constexpr (ez == -1) vo += sz;
            a[i] = vo;
        });
    } else {
        // bytes from a node to its source for e = +1 and e = -1 on each axis
        auto back = [](int v, int n, int per, uint32_t st) { return per && v == 0 ? (uint32_t)(n - 1) * st : 0u - st; };
        auto fore = [](int v, int n, int per, uint32_t st) { return per && v == n - 1 ? (uint32_t)(1 - n) * st : st; };
        const uint32_t bx = back(x, g.n[0], g.periodic[0], SZ), fx = fore(x, g.n[0], g.periodic[0], SZ);
        const uint32_t by = back(y, g.n[1], g.periodic[1], sy), fy = fore(y, g.n[1], g.periodic[1], sy);
        uint32_t bz = 0u, fz = 0u;
        if constexpr (DIM == 3) {
            bz = back(z, g.n[2], g.periodic[2], sz);
            fz = fore(z, g.n[2], g.periodic[2], sz);
        }
        const uint32_t own = p * SZ, stride = (uint32_t)plane_bytes<STORE>(g, 1);
        static_for<Lat<DIM>::Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            constexpr int ex = Lat<DIM>::E[i][0], ey = Lat<DIM>::E[i][1], ez = Lat<DIM>::E[i][2];
            uint32_t vo = own;
            if constexpr (ex != 0) vo += ex == 1 ? bx : fx;
            if constexpr (ey != 0) vo += ey == 1 ? by : fy;
            if constexpr (ez != 0) vo += ez == 1 ? bz : fz;
            a[i] = ((tw >> i) & 1u) ? own + stride * (uint32_t)Lat<DIM>::OPP[i] : vo + stride * (uint32_t)i;
        });
    }
}

// The wave-uniform part of the offset of direction i (the plane in the fast form).
template <int STORE>
__device__ __forceinline__ int uniform_plane(const Geometry &g, bool wave_fast, int i)
{
    // formed unconditionally and selected, so the node loop takes no branch here
    const int so = plane_bytes<STORE>(g, i);
    return wave_fast ? so : 0;
}

// The stored bits of the populations that stream into node p, one component.
template <int DIM, int STORE>
__device__ __forceinline__ void bgather_raw(__amdgpu_buffer_rsrc_t rs, const Geometry &g, uint32_t p, uint32_t tw,
                                            int x, int y, int z, bool wave_fast,
                                            typename Buf<STORE>::Raw (&f)[Lat<DIM>::Q])
{
    uint32_t a[Lat<DIM>::Q];
    gather_addr<DIM, STORE>(g, p, tw, x, y, z, wave_fast, a);
    static_for<Lat<DIM>::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        f[i] = Buf<STORE>::raw(rs, a[i], uniform_plane<STORE>(g, wave_fast, i));
    });
}

// The same for both components (same addresses, two buffers).
template <int DIM, int STORE>
__device__ __forceinline__ void bgather2_raw(__amdgpu_buffer_rsrc_t rs0, __amdgpu_buffer_rsrc_t rs1,
                                             const Geometry &g, uint32_t p, uint32_t tw, int x, int y, int z,
                                             bool wave_fast, typename Buf<STORE>::Raw (&f1)[Lat<DIM>::Q],
                                             typename Buf<STORE>::Raw (&f2)[Lat<DIM>::Q])
{
    uint32_t a[Lat<DIM>::Q];
    gather_addr<DIM, STORE>(g, p, tw, x, y, z, wave_fast, a);
    static_for<Lat<DIM>::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        f1[i] = Buf<STORE>::raw(rs0, a[i], uniform_plane<STORE>(g, wave_fast, i));
    });
    static_for<Lat<DIM>::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        f2[i] = Buf<STORE>::raw(rs1, a[i], uniform_plane<STORE>(g, wave_fast, i));
    });
}

// Populations from the stored bits that bgather_raw loaded.
template <int DIM, int STORE>
__device__ __forceinline__ void decode(const typename Buf<STORE>::Raw (&h)[Lat<DIM>::Q], float (&f)[Lat<DIM>::Q],
                                       float rr)
{
    static_for<Lat<DIM>::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        f[i] = Buf<STORE>::dec(h[i], weight<DIM>(i), rr);
    });
}

template <int DIM, int STORE>
__device__ __forceinline__ void bgather(__amdgpu_buffer_rsrc_t rs, const Geometry &g, uint32_t p, uint32_t tw,
                                        int x, int y, int z, bool wave_fast, float (&f)[Lat<DIM>::Q], float rr)
{
    typename Buf<STORE>::Raw h[Lat<DIM>::Q];
    bgather_raw<DIM, STORE>(rs, g, p, tw, x, y, z, wave_fast, h);
    decode<DIM, STORE>(h, f, rr);
}

__device__ __forceinline__ void coords_of(const Geometry &g, int64_t b, int &x, int &y, int &z)
{
    x = (int)(b % g.n[0]);
    y = (int)((b / g.n[0]) % g.n[1]);
    z = (int)(b / ((int64_t)g.n[0] * g.n[1]));
}

// Maps a halo coordinate onto the box: periodic axes wrap; beyond a
// non-periodic face the mirror image about that face (ghost layers of
// eqs. 24-25: the first ghost copies the face node, the second its neighbour).
__device__ __forceinline__ int map_axis(int v, int n, int periodic)
{
    if (v < 0) return periodic ? v + n : -1 - v;
    if (v >= n) return periodic ? v - n : 2 * n - 1 - v;
    return v;
}

// Linear index in the caller's frame of the memory-frame node (x, y, z).
__device__ __forceinline__ int64_t caller_index(const Geometry &g, int x, int y, int z)
{
    return (int64_t)x * g.ostride[0] + (int64_t)y * g.ostride[1] + (int64_t)z * g.ostride[2];
}

// Deterministic block-wide sum of two doubles over NT threads (whole waves):
// a butterfly inside each wave, then the wave sums in a fixed pairwise order.
template <int NT>
__device__ __forceinline__ void block_sum2(double &a, double &b, double *red /*[2 * NT / 64]*/)
{
    static_assert(NT % 64 == 0 && NT <= 1024, "whole waves");
    constexpr int NW = NT / 64;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, 64);
        b += __shfl_xor(b, o, 64);
    }
    if constexpr (NW > 1) {
        const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
        __syncthreads();
        if (ln == 0) { red[2 * wv] = a; red[2 * wv + 1] = b; }
        __syncthreads();
        // every thread folds the wave sums in the same fixed pairwise order
        double ta[NW], tb[NW];
#pragma unroll
        for (int j = 0; j < NW; j++) { ta[j] = red[2 * j]; tb[j] = red[2 * j + 1]; }
#pragma unroll
        for (int w = NW / 2; w > 0; w >>= 1) {
#pragma unroll
            for (int j = 0; j < w; j++) { ta[j] += ta[j + w]; tb[j] += tb[j + w]; }
        }
        a = ta[0];
        b = tb[0];
    }
}

// Deterministic sum of a partials array [n][2] by every block (fixed order).
template <int NT>
__device__ __forceinline__ void reduce_partials(const double *__restrict__ part, int n, double &a, double &b,
                                                double *red)
{
    a = 0.0;
    b = 0.0;
    for (int j = threadIdx.x; j < n; j += NT) {
        a += part[2 * j];
        b += part[2 * j + 1];
    }
    block_sum2<NT>(a, b, red);
}

// ---------------------------------------------------------------------------
// The sums Q_in and Q' of eq. (23) as integers in units of 2^-40.  Each term
// rho u.n (the FP64 product of two floats) is rounded once to that grid; the
// integer sums are then exact, so they do not depend on which block adds
// which term or in what order (every launch shape and tile configuration
// gives the same bits).  The grid is far below FP32 resolution; the range
// holds |Q| < 2^23.
// ---------------------------------------------------------------------------
__device__ __forceinline__ long long flow_fix(double q) { return __double2ll_rn(q * 0x1p40); }
__device__ __forceinline__ double flow_unfix(unsigned long long v) { return (double)(long long)v * 0x1p-40; }

// ---------------------------------------------------------------------------
// k_main: the fused per-node update as a sweep along the last lattice axis
// (y in 2-D, z in 3-D).  A block owns a lateral tile (TX in 2-D, TX x TY in
// 3-D) and a chunk of ZC planes of the sweep axis; it advances W planes per
// iteration and keeps psi of the planes it needs (window plus two on each
// side) in an LDS ring of W + 4 planes, so psi is computed once per plane and
// only the lateral two-node halo is recomputed by neighbouring blocks.
// Work items are ordered lateral-x fastest, then lateral-y, then chunk, or in
// square blocks of tiles (see xcd_group); each of the eight XCDs takes a few
// consecutive ones per turn, so that blocks which share halo data share an L2.
// ---------------------------------------------------------------------------
//
// PSRC selects where psi comes from: 0 = recomputed here from the gathered
// populations of each plane (one fused kernel), 1 = read from the psi array
// that k_psi wrote for this step (the populations are then read only once).
//
// KEEPB = 1 holds both components' populations in registers between the
// velocity and the collision; KEEPB = 0 gathers component 2 again after
// component 1 is stored (fewer registers, one more pass through the caches).
//
// FIELDS = true stops after the velocity and writes rho_k and u of every node
// of the item, solids included, in FP64 in the caller's frame (orho [2][N],
// ou [3][N]) instead of a step.
template <int DIM, int STORE, int PSRC, int TX, int TY, int W, int ZC, int KEEPB, bool FIELDS = false>
__device__ __forceinline__ void main_item(const typename Codec<STORE>::T *__restrict__ src,
                                          typename Codec<STORE>::T *__restrict__ dst,
                                          const uint32_t *__restrict__ type, const float2 *__restrict__ psi,
                                          const float2 *__restrict__ ref, const Geometry &g, const Physics &ph,
                                          const Boundary &bd, int tiles_x, int tiles_y, int item,
                                          int *__restrict__ flag, unsigned long long *__restrict__ qacc,
                                          double *__restrict__ orho = nullptr, double *__restrict__ ou = nullptr)
{
    constexpr int Q = Lat<DIM>::Q;
    constexpr int LY = DIM == 3 ? TY : 1;          // lateral y extent of the tile
    constexpr int HX = TX + 4, HY = DIM == 3 ? TY + 4 : 1;
    constexpr int PLANE = HX * HY;                 // lateral halo positions per plane
    constexpr int R = W + 4;                       // ring planes
    constexpr int RP = DIM == 3 ? 1 : 256 / TX;    // 2-D: rows covered by one pass of the block
    constexpr int NPT = DIM == 3 ? W : W / RP;     // nodes per thread per iteration
    constexpr int NOFF = DIM == 3 ? 125 : 25;      // offsets of the 5^DIM stencil box
    static_assert(DIM == 3 ? TX * LY == 256 : (256 % TX == 0 && W % RP == 0), "256 threads per block");
    __shared__ float2 s_psi[R * PLANE];
    __shared__ uint8_t s_sol[R * PLANE];
    // 2-D fused mode, binary16: the stored bits of the populations that
    // stream into each ring node, gathered once for its psi and read back by
    // the node update (the same loads, so the same bits).  FP32 would need
    // 39 KB of LDS per block and lose more occupancy than it saves.
    constexpr bool ONE = ZC == W;              // one window: its planes and the halo's are loaded at once
    // 2-D fused mode, one window: each thread forms psi of its own nodes and
    // keeps what it gathered for their update; the halo positions follow
    // (binary16 keeps them in LDS for 32-wide tiles, see STAGE)
    constexpr bool OWN = DIM == 2 && PSRC == 0 && ONE && KEEPB && (STORE == 0 || TX > 32);
    constexpr bool STAGE = DIM == 2 && PSRC == 0 && STORE != 0 && !OWN;
    __shared__ typename Buf<STORE>::Raw s_fr[STAGE ? R * PLANE * 2 * Q : 1];

    const __amdgpu_buffer_rsrc_t rs0 = comp_rsrc<STORE>(src, 0, Q, g.Ppad);
    const __amdgpu_buffer_rsrc_t rs1 = comp_rsrc<STORE>(src, 1, Q, g.Ppad);
    // the item's share of the eq. (23) sums (fixed point, see flow_fix),
    // gathered by LDS atomics at the face nodes, so that nothing is held in
    // registers across the sweep
    __shared__ unsigned long long s_q[2];
    if (threadIdx.x == 0) s_q[0] = s_q[1] = 0ull;
    __syncthreads();                               // the ring of a previous item is free
    {
        const int ns = g.n[DIM - 1];
        const int tx = item % tiles_x;
        const int ty = (item / tiles_x) % tiles_y;
        const int ch = item / (tiles_x * tiles_y);
        const int x0 = tx * TX, y0 = DIM == 3 ? ty * TY : 0;
        const int s0 = ch * ZC, s1 = min(s0 + ZC, ns);

        // psi of NP sweep planes from plane pa on into the ring: positions
        // threadIdx.x, threadIdx.x + 256, ... of them.  The loads of U
        // positions are in flight at once (of all of them where registers
        // allow): with one position at a time a block of a small domain spent
        // most of its life in one memory round trip after another (node update
        // of a 64x64 box 11.7 -> 9.3 us, of the 600x120x120 device 593 -> 560).
        // between() runs after the first loads are issued.
        auto load_planes = [&](auto npc, int pa, auto &&between) {
            constexpr int NP = decltype(npc)::value;
            // PSRC 1 in 3-D: a thread keeps its lateral positions from plane to
            // plane (NL of them), so that a load's address is the plane's
            // (scalar) and the position's; the last 256 positions of a plane
            // are dealt like that if at least half are there, and otherwise
            // counted through all planes like every position of the other modes
            // (which form each position's coordinates anew, some 35 operations;
            // that took the binary16 node update of the 600x120x120 device from
            // 378 to 412 us and of 300x60x60 from 63 to 70, FP32 of the latter
            // from 75.6 to 78.5)
            constexpr int NL = DIM == 3 && PSRC == 1 ? (PLANE + 127) / 256 : 0;
            constexpr int LAT = NL * 256, REST = LAT < PLANE ? PLANE - LAT : 0;
            constexpr int CNT = NP * REST, ITL = NP * NL, IT = ITL + (CNT + 255) / 256;
            constexpr int UMAX = PSRC == 1 ? 8 : 2;
            constexpr int U = (IT + (IT + UMAX - 1) / UMAX - 1) / ((IT + UMAX - 1) / UMAX);
            int lat[NL ? NL : 1];
            static_for<NL>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                const int r = min((int)threadIdx.x + 256 * j, PLANE - 1);
                const int x = x0 - 2 + r % HX, y = y0 - 2 + r / HX;
                const bool in = x < g.n[0] + 2 && y < g.n[1] + 2;
                lat[j] = in ? map_axis(x, g.n[0], g.periodic[0]) + g.n[0] * map_axis(y, g.n[1], g.periodic[1]) : 0;
            });
            static_for<(IT + U - 1) / U>([&](auto cc) {
                constexpr int C = decltype(cc)::value;
                int slot[U], gx[U], gy[U], gz[U];
                bool have[U], need[U];
                static_for<U>([&](auto uc) {
                    constexpr int u = decltype(uc)::value, it = C * U + u;
                    if constexpr (it < ITL) {
                        constexpr int j = it % NL;
                        const int pl = pa + it / NL;
                        have[u] = 256 * (j + 1) <= PLANE || (int)threadIdx.x + 256 * j < PLANE;
                        need[u] = pl < g.n[2] + 2;
                        slot[u] = ((pl + 4 * R) % R) * PLANE + (int)threadIdx.x + 256 * j;
                        gx[u] = lat[j];
                        gy[u] = 0;
                        gz[u] = need[u] ? map_axis(pl, g.n[2], g.periodic[2]) : 0;
                        return;
                    }
                    const int h = (int)threadIdx.x + 256 * (it - ITL);
                    const int pl = pa + h / (REST ? REST : 1), r = LAT + h % (REST ? REST : 1);
                    const int lx = r % HX, ly = r / HX;
                    have[u] = it + 1 < IT ? true : h < CNT;
                    if (it >= IT) have[u] = false;
                    int x = x0 - 2 + lx, y = DIM == 3 ? y0 - 2 + ly : pl, z = DIM == 3 ? pl : 0;
                    need[u] = have[u] && x < g.n[0] + 2 && y < g.n[1] + 2 && (DIM == 2 || z < g.n[2] + 2);
                    slot[u] = ((pl + 4 * R) % R) * PLANE + r;
                    // positions that no node needs read the box's first node
                    gx[u] = need[u] ? map_axis(x, g.n[0], g.periodic[0]) : 0;
                    gy[u] = need[u] ? map_axis(y, g.n[1], g.periodic[1]) : 0;
                    gz[u] = DIM == 3 && need[u] ? map_axis(z, g.n[2], g.periodic[2]) : 0;
                });
                auto box = [&](int u) {
                    return (int64_t)gx[u] + (int64_t)g.n[0] * ((int64_t)gy[u] + (int64_t)g.n[1] * gz[u]);
                };
                if constexpr (PSRC == 1) {
                    // psi of this step from k_psi; solids carry -0.0 (zero in
                    // every sum, and the sign marks them for the adhesion stencil)
                    float2 v[U];
                    static_for<U>([&](auto uc) {
                        constexpr int u = decltype(uc)::value;
                        if constexpr (C * U + u < ITL)
                            v[u] = (psi + (int64_t)g.n[0] * g.n[1] * gz[u])[(uint32_t)gx[u]];
                        else
                            v[u] = psi[box(u)];
                    });
                    if constexpr (C == 0) between();
                    static_for<U>([&](auto uc) {
                        constexpr int u = decltype(uc)::value;
                        if (!have[u]) return;
                        s_psi[slot[u]] = v[u];
                        s_sol[slot[u]] = !need[u] || signbit(v[u].x) ? 1 : 0;
                    });
                } else {
                    uint32_t tw[U];
                    float2 rf[U];
                    typename Buf<STORE>::Raw h1[U][Q], h2[U][Q];
                    static_for<U>([&](auto uc) {
                        constexpr int u = decltype(uc)::value;
                        tw[u] = type[box(u)];
                        rf[u] = make_float2(0.0f, 0.0f);
                        if constexpr (Codec<STORE>::REF) rf[u] = ref[box(u)];
                    });
                    if constexpr (C == 0) between();
                    static_for<U>([&](auto uc) {
                        constexpr int u = decltype(uc)::value;
                        // lanes off the fluid gather a valid node, unused, so
                        // that no load waits at the end of a branch
                        const bool fluid = need[u] && !(tw[u] & T_SOLID);
                        tw[u] = fluid ? tw[u] : T_SOLID;
                        const uint32_t t = fluid ? tw[u] : 0u;
                        const int ax = fluid ? gx[u] : 1, ay = fluid ? gy[u] : 1, az = fluid ? gz[u] : 1;
                        const uint32_t pp = (uint32_t)pidx(g, ax, ay, DIM == 3 ? az : -1);
                        const bool wave_fast = __ballot((t & (T_BBMASK | T_EDGE)) != 0) == 0;
                        bgather2_raw<DIM, STORE>(rs0, rs1, g, pp, t, ax, ay, DIM == 3 ? az : 0, wave_fast, h1[u], h2[u]);
                    });
                    static_for<U>([&](auto uc) {
                        constexpr int u = decltype(uc)::value;
                        if (!have[u]) return;
                        const bool fluid = !(tw[u] & T_SOLID);
                        float f[Q], p1 = 0.0f, p2 = 0.0f;
                        if constexpr (STAGE) {
                            if (fluid)
                                static_for<Q>([&](auto ic) {
                                    constexpr int i = decltype(ic)::value;
                                    s_fr[slot[u] * 2 * Q + i] = h1[u][i];
                                    s_fr[slot[u] * 2 * Q + Q + i] = h2[u][i];
                                });
                        }
                        decode<DIM, STORE>(h1[u], f, rf[u].x);
                        static_for<Q>([&](auto ic) { p1 += f[decltype(ic)::value]; });
                        decode<DIM, STORE>(h2[u], f, rf[u].y);
                        static_for<Q>([&](auto ic) { p2 += f[decltype(ic)::value]; });
                        s_psi[slot[u]] = fluid ? make_float2(p1, p2) : make_float2(0.0f, 0.0f);
                        s_sol[slot[u]] = fluid ? 0 : 1;
                    });
                }
            });
        };

        // node k of this thread in the sweep window starting at plane w0
        const int lx = threadIdx.x % TX, ly = DIM == 3 ? threadIdx.x / TX : 0;
        auto sweep_of = [&](int w0, int k) { return DIM == 3 ? w0 + k : w0 + k * RP + (int)threadIdx.x / TX; };
        auto type_of = [&](int sv) -> uint32_t {
            const int x = x0 + lx, y = DIM == 3 ? y0 + ly : sv, z = DIM == 3 ? sv : 0;
            const bool valid = x < g.n[0] && sv < s1 && (DIM == 2 || y < g.n[1]);
            return valid ? type[(int64_t)x + (int64_t)g.n[0] * ((int64_t)y + (int64_t)g.n[1] * z)] : T_SOLID;
        };
        // the populations of the window's node, where a thread has one node per
        // window: gathered between the ring's loads and their use
        constexpr bool AHEAD = NPT == 1 && KEEPB && !STAGE && !OWN;
        constexpr int NQ = OWN ? NPT : 1;
        typename Buf<STORE>::Raw q1[NQ][Q], q2[NQ][Q];
        if constexpr (!ONE) load_planes(std::integral_constant<int, 4>{}, s0 - 2, [] {});
        for (int w0 = s0; w0 < s1; w0 += W) {
            if constexpr (!ONE) __syncthreads();  // ring slots of w0-6..w0-3 are free
            // the type words of the window's nodes are loaded together with
            // the psi planes, whose wait covers them: loaded node by node they
            // would each wait for the previous node's stores to complete (the
            // memory counter also counts stores)
            uint32_t twq[NPT];
            if constexpr (!OWN)
                static_for<NPT>([&](auto jc) { twq[decltype(jc)::value] = type_of(sweep_of(w0, decltype(jc)::value)); });
            auto ahead = [&] {
                if constexpr (AHEAD) {
                    // lanes off the fluid gather a valid node, unused
                    const int sv = sweep_of(w0, 0);
                    const bool fluid = !(twq[0] & T_SOLID);
                    const uint32_t t = fluid ? twq[0] : 0u;
                    const int x = fluid ? x0 + lx : 1, y = fluid ? (DIM == 3 ? y0 + ly : sv) : 1, z = DIM == 3 ? (fluid ? sv : 1) : 0;
                    const bool wave_fast = __ballot((t & (T_BBMASK | T_EDGE)) != 0) == 0;
                    bgather2_raw<DIM, STORE>(rs0, rs1, g, (uint32_t)pidx(g, x, y, DIM == 3 ? z : -1), t, x, y, z,
                                             wave_fast, q1[0], q2[0]);
                }
            };
            if constexpr (OWN) {
                // HC halo positions: the rows below and above the window, then
                // two columns on either side of its rows; thread t takes
                // t, t + 256, ... of them after its own NPT nodes
                constexpr int HC = (W + 4) * HX - 256 * NPT, HP = (HC + 255) / 256, U = NPT + HP;
                static_assert(HC == 4 * HX + 4 * W, "halo of the window");
                int col[U], row[U], gx[U], gy[U];
                bool have[U], need[U];
                static_for<U>([&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    have[u] = true;
                    if constexpr (u < NPT) {
                        col[u] = lx + 2;
                        row[u] = 2 + u * RP + (int)threadIdx.x / TX;
                    } else {
                        const int h = (int)threadIdx.x + 256 * (u - NPT), e = h - 4 * HX;
                        have[u] = h < HC;
                        const int r4 = h / HX;
                        row[u] = e < 0 ? (r4 < 2 ? r4 : r4 + W) : 2 + e / 4;
                        col[u] = e < 0 ? h % HX : (e % 4 < 2 ? e % 4 : e % 4 + TX);
                    }
                    const int x = x0 - 2 + col[u], y = w0 - 2 + row[u];
                    need[u] = have[u] && x < g.n[0] + 2 && y < g.n[1] + 2;
                    gx[u] = need[u] ? map_axis(x, g.n[0], g.periodic[0]) : 0;
                    gy[u] = need[u] ? map_axis(y, g.n[1], g.periodic[1]) : 0;
                });
                uint32_t tw[U];
                float2 rf[U];
                typename Buf<STORE>::Raw g1[HP][Q], g2[HP][Q];
                static_for<U>([&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    const uint32_t b = (uint32_t)gx[u] + (uint32_t)g.n[0] * (uint32_t)gy[u];
                    tw[u] = type[b];
                    rf[u] = make_float2(0.0f, 0.0f);
                    if constexpr (Codec<STORE>::REF) rf[u] = ref[b];
                });
                static_for<U>([&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    // lanes off the fluid gather a valid node, unused, so that
                    // no load waits at the end of a branch
                    const bool fluid = need[u] && !(tw[u] & T_SOLID);
                    tw[u] = fluid ? tw[u] : T_SOLID;
                    const uint32_t t = fluid ? tw[u] : 0u;
                    const int ax = fluid ? gx[u] : 1, ay = fluid ? gy[u] : 1;
                    const bool wave_fast = __ballot((t & (T_BBMASK | T_EDGE)) != 0) == 0;
                    const uint32_t pp = (uint32_t)pidx(g, ax, ay, -1);
                    if constexpr (u < NPT)
                        bgather2_raw<DIM, STORE>(rs0, rs1, g, pp, t, ax, ay, 0, wave_fast, q1[u], q2[u]);
                    else
                        bgather2_raw<DIM, STORE>(rs0, rs1, g, pp, t, ax, ay, 0, wave_fast, g1[u - NPT], g2[u - NPT]);
                });
                static_for<U>([&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    if (!have[u]) return;
                    const bool fluid = !(tw[u] & T_SOLID);
                    float f[Q], p1 = 0.0f, p2 = 0.0f;
                    if constexpr (u < NPT) decode<DIM, STORE>(q1[u], f, rf[u].x);
                    else decode<DIM, STORE>(g1[u - NPT], f, rf[u].x);
                    static_for<Q>([&](auto ic) { p1 += f[decltype(ic)::value]; });
                    if constexpr (u < NPT) decode<DIM, STORE>(q2[u], f, rf[u].y);
                    else decode<DIM, STORE>(g2[u - NPT], f, rf[u].y);
                    static_for<Q>([&](auto ic) { p2 += f[decltype(ic)::value]; });
                    const int slot = ((w0 - 2 + row[u] + 4 * R) % R) * PLANE + col[u];
                    s_psi[slot] = fluid ? make_float2(p1, p2) : make_float2(0.0f, 0.0f);
                    s_sol[slot] = fluid ? 0 : 1;
                });
                // own positions outside the item's nodes are halo to others
                static_for<NPT>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    const int sv = sweep_of(w0, j);
                    twq[j] = x0 + lx < g.n[0] && sv < s1 ? tw[j] : T_SOLID;
                });
            } else if constexpr (ONE) load_planes(std::integral_constant<int, W + 4>{}, w0 - 2, ahead);
            else load_planes(std::integral_constant<int, W>{}, w0 + 2, ahead);
            __syncthreads();
            // settle the type loads here, once per window: an empty statement
            // that reads them, so that the wait is not placed at the head of
            // the node loop, where it would run on every node
#pragma unroll
            for (int j = 0; j < NPT; j++) asm volatile("" ::"v"(twq[j]));
#pragma unroll 1
            for (int k = 0; k < NPT; k++) {
                const int sv = sweep_of(w0, k);
                const int x = x0 + lx;
                const int y = DIM == 3 ? y0 + ly : sv;
                const int z = DIM == 3 ? sv : 0;
                const bool valid = x < g.n[0] && sv < s1 && (DIM == 2 || y < g.n[1]);
                const int64_t b = valid ? (int64_t)x + (int64_t)g.n[0] * ((int64_t)y + (int64_t)g.n[1] * z) : 0;
                const uint32_t tw = twq[0];
                static_for<NPT - 1>([&](auto jc) { twq[decltype(jc)::value] = twq[decltype(jc)::value + 1]; });
                const bool fluid = !(tw & T_SOLID);
                const bool wave_fast = __ballot(fluid && (tw & (T_BBMASK | T_EDGE))) == 0;
                if constexpr (FIELDS) {
                    if (valid && !fluid) {
                        const int64_t bo = caller_index(g, x, y, z);
                        orho[bo] = orho[g.N + bo] = 0.0;
                        ou[bo] = ou[g.N + bo] = ou[2 * g.N + bo] = 0.0;
                    }
                }
                if (!fluid) {
                    if constexpr (OWN && NPT > 1)
                        static_for<Q>([&](auto ic) {
                            constexpr int i = decltype(ic)::value;
                            static_for<NQ - 1>([&](auto jc) {
                                constexpr int j = decltype(jc)::value;
                                q1[j][i] = q1[j + 1][i];
                                q2[j][i] = q2[j + 1][i];
                            });
                        });
                    continue;
                }
                const uint32_t p = (uint32_t)pidx(g, x, y, DIM == 3 ? z : -1);
                // base[d]: ring index of the lateral corner (-2, -2) of the
                // node's neighbourhood in sweep plane sv + d - 2, so every
                // stencil offset below is a non-negative immediate
                const int corner = (DIM == 3 ? ly * HX : 0) + lx;
                int base[5];
                static_for<5>([&](auto dc) {
                    constexpr int d = decltype(dc)::value;
                    base[d] = ((sv + d - 2 + 4 * R) % R) * PLANE + corner;
                });
                constexpr int CEN = (DIM == 3 ? 2 * HX : 0) + 2;   // the node itself
                // the populations of the node: loads issued here, before the
                // force stencil, so the LDS work below hides their latency
                typename Buf<STORE>::Raw h1[Q], h2[Q];
                if constexpr (AHEAD || OWN) {
                    static_for<Q>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
                        h1[i] = q1[0][i];
                        h2[i] = q2[0][i];
                        static_for<NQ - 1>([&](auto jc) {
                            constexpr int j = decltype(jc)::value;
                            q1[j][i] = q1[j + 1][i];
                            q2[j][i] = q2[j + 1][i];
                        });
                    });
                } else if constexpr (STAGE) {
                    // staged in the ring when psi of this node's plane was formed
                    const int sl = base[2] + CEN;
                    static_for<Q>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
                        h1[i] = s_fr[sl * 2 * Q + i];
                        h2[i] = s_fr[sl * 2 * Q + Q + i];
                    });
                } else if constexpr (KEEPB) {
                    bgather2_raw<DIM, STORE>(rs0, rs1, g, p, tw, x, y, z, wave_fast, h1, h2);
                } else {
                    bgather_raw<DIM, STORE>(rs0, g, p, tw, x, y, z, wave_fast, h1);
                }
                const float2 ps = s_psi[base[2] + CEN];
                // psi(t) of the node for the next step's reference densities
                // and the face kernels (the two-pass mode has it from k_psi)
                if constexpr (PSRC == 0) const_cast<float2 *>(psi)[b] = ps;
                float2 rf = make_float2(0.0f, 0.0f);
                if constexpr (Codec<STORE>::REF) rf = ref[b];

                // ---- wall adhesion (eq. 11): only nodes with a solid within the stencil
                float A[3] = {0.f, 0.f, 0.f};
                if (ph.adhesion && (tw & T_NEARWALL)) {
                    static_for<NOFF>([&](auto oc) {
                        constexpr int o = decltype(oc)::value;
                        constexpr int dx = o % 5 - 2, dy = (o / 5) % 5 - 2, dz = DIM == 3 ? o / 25 - 2 : 0;
                        constexpr int r2 = dx * dx + dy * dy + dz * dz;
                        constexpr float w = stencil_w<DIM>(r2);
                        if constexpr (r2 != 0 && w != 0.0f) {
                            constexpr int ddy = DIM == 3 ? dy : 0, ddz = DIM == 3 ? dz : dy;
                            const float sv1 = (float)s_sol[base[2 + ddz] + CEN + ddy * HX + dx];
                            if constexpr (dx != 0) A[0] = fmaf(w * dx, sv1, A[0]);
                            if constexpr (dy != 0) A[1] = fmaf(w * dy, sv1, A[1]);
                            if constexpr (dz != 0) A[2] = fmaf(w * dz, sv1, A[2]);
                        }
                    });
                }
                // ---- forces (eqs. 10-11): the stencil in pairs of opposite
                // offsets, one sweep-plane distance at a time (the loop bounds
                // how many LDS reads are in flight)
                float g1[3] = {0.f, 0.f, 0.f}, g2[3] = {0.f, 0.f, 0.f};
#pragma unroll 1
                for (int sd = 0; sd <= 2; sd++) {
                    const int bp = ((sv + sd + 4 * R) % R) * PLANE + corner + CEN;
                    const int bm = ((sv - sd + 4 * R) % R) * PLANE + corner + CEN;
                    auto plane = [&](auto sdc) {
                        constexpr int SD = decltype(sdc)::value;
                        static_for<25>([&](auto oc) {
                            constexpr int o = decltype(oc)::value;
                            constexpr int a = o % 5 - 2, bq = o / 5 - 2;   // lateral offsets
                            // (dx, dy, dz) of the offset and its lateral / sweep split
                            constexpr int dx = a, dy = DIM == 3 ? bq : SD, dz = DIM == 3 ? SD : 0;
                            constexpr int lat_y = DIM == 3 ? bq : 0;
                            constexpr int r2 = dx * dx + dy * dy + dz * dz;
                            constexpr float w = stencil_w<DIM>(r2);
                            // the half of the stencil with a positive first nonzero of (sweep, lateral-y, x)
                            constexpr bool half = SD > 0 || (lat_y > 0 || (lat_y == 0 && dx > 0));
                            constexpr bool in2d = DIM == 3 || bq == 0;
                            if constexpr (half && in2d && w != 0.0f) {
                                constexpr int ho = lat_y * HX + dx;
                                const float2 vp = s_psi[bp + ho];
                                const float2 vm = s_psi[bm - ho];
                                const float d1 = vp.x - vm.x, d2 = vp.y - vm.y;
                                if constexpr (dx != 0) { g1[0] = fmaf(w * dx, d1, g1[0]); g2[0] = fmaf(w * dx, d2, g2[0]); }
                                if constexpr (dy != 0) { g1[1] = fmaf(w * dy, d1, g1[1]); g2[1] = fmaf(w * dy, d2, g2[1]); }
                                if constexpr (dz != 0) { g1[2] = fmaf(w * dz, d1, g1[2]); g2[2] = fmaf(w * dz, d2, g2[2]); }
                            }
                        });
                    };
                    if (sd == 0) plane(std::integral_constant<int, 0>{});
                    else if (sd == 1) plane(std::integral_constant<int, 1>{});
                    else plane(std::integral_constant<int, 2>{});
                }
                const float r1 = ps.x, r2 = ps.y, rt = r1 + r2;
                const float w1 = r1 / rt, w2 = r2 / rt;
                float F1[3], F2[3];
                static_for<3>([&](auto dc) {
                    constexpr int d = decltype(dc)::value;
                    F1[d] = -ph.G12 * r1 * g2[d] - ph.Gw[0] * r1 * A[d] + w1 * ph.Fb[d];
                    F2[d] = -ph.G12 * r2 * g1[d] - ph.Gw[1] * r2 * A[d] + w2 * ph.Fb[d];
                });

                // ---- common velocity (eqs. 7-8)
                PairF<DIM> qa, qb;
                float J1[3], J2[3];
                {
                    float f[Q];
                    decode<DIM, STORE>(h1, f, rf.x);
                    to_pairs<DIM>(f, qa);
                    pair_momentum<DIM>(qa, J1);
                    if constexpr (!KEEPB && !STAGE) bgather_raw<DIM, STORE>(rs1, g, p, tw, x, y, z, wave_fast, h2);
                    decode<DIM, STORE>(h2, f, rf.y);
                    to_pairs<DIM>(f, qb);
                    pair_momentum<DIM>(qb, J2);
                }
                if constexpr (FIELDS) {
                    const int64_t bo = caller_index(g, x, y, z);
                    orho[bo] = r1;
                    orho[g.N + bo] = r2;
                    static_for<3>([&](auto dc) {
                        constexpr int d = decltype(dc)::value;
                        ou[g.ax[d] * g.N + bo] = d < DIM ? (J1[d] + J2[d] + 0.5f * (F1[d] + F2[d])) / rt : 0.0f;
                    });
                    continue;
                }
                float u[3];
                const float irt = 1.0f / rt;
                static_for<3>([&](auto dc) {
                    constexpr int d = decltype(dc)::value;
                    u[d] = (J1[d] + J2[d] + 0.5f * (F1[d] + F2[d])) * irt;
                });

                if (!(rt > 0.0f) || !isfinite(rt) || !isfinite(u[0] + u[1] + u[2])) *flag = 1;

                if (tw & T_ROLE) {
                    const int slot = bd.bslot[b];
                    float *fF = bd.faceF + (int64_t)slot * 6;
                    fF[0] = F1[0]; fF[1] = F1[1]; fF[2] = F1[2];
                    fF[3] = F2[0]; fF[4] = F2[1]; fF[5] = F2[2];
                    if (tw & T_XPRIME) {
                        const float un = bd.out_sign * pick3(u, bd.out_axis);
                        bd.faceU[slot] = un;
                        atomicAdd(&s_q[1], (unsigned long long)flow_fix((double)rt * (double)un));
                    }
                    if (tw & T_INLET) {
                        const Patch pt = bd.patch[(tw & T_PATCH_MASK) >> T_PATCH_SHIFT];
                        atomicAdd(&s_q[0], (unsigned long long)flow_fix((double)rt * (double)(pt.sign * pick3(u, pt.axis))));
                    }
                    if ((tw & T_OUTLET) && bd.chi_on) continue;   // collided by the face launch (k_faces)
                }

                // ---- MRT collision of each component, stored at x
                const __amdgpu_buffer_rsrc_t rd0 = comp_rsrc<STORE>(dst, 0, Q, g.Ppad);
                const __amdgpu_buffer_rsrc_t rd1 = comp_rsrc<STORE>(dst, 1, Q, g.Ppad);
                const uint32_t vo = p * Buf<STORE>::SZ;
                // reference density of the node that reads population i next
                // step: the destination x + e_i, or x itself on bounce-back
                auto dest_psi = [&](auto inc, auto ic) -> float2 {
                    constexpr int i = decltype(ic)::value;
                    constexpr int ex = Lat<DIM>::E[i][0], ey = Lat<DIM>::E[i][1], ez = Lat<DIM>::E[i][2];
                    if constexpr (!decltype(inc)::value)
                        if ((tw >> Lat<DIM>::OPP[i]) & 1u) return ps;
                    if constexpr (DIM == 3) return s_psi[base[2 + ez] + CEN + ey * HX + ex];
                    else return s_psi[base[2 + ey] + CEN + ex];
                };
                float fo[Q];
                // fo of one component to rd.  Waves without bounce-back (most) skip
                // its test, which costs binary16 three operations a population
                // (node update of the 300x60x60 device 60.5 -> 58 us, of
                // 600x120x120 363 -> 357; 2-D, less bound by VALU issue, lost
                // up to 1%)
                auto put = [&](__amdgpu_buffer_rsrc_t rd, auto &&ref_of) {
                    auto all = [&](auto inc) {
                        static_for<Q>([&](auto ic) {
                            constexpr int i = decltype(ic)::value;
                            float rp = 0.0f;
                            if constexpr (Codec<STORE>::REF) rp = ref_of(inc, ic);
                            Buf<STORE>::st(rd, vo, plane_bytes<STORE>(g, i), fo[i], weight<DIM>(i), rp);
                        });
                    };
                    if (DIM == 3 && Codec<STORE>::REF && wave_fast) all(std::true_type{});
                    else all(std::false_type{});
                };
                // a moving wall: the populations that bounce back from it take
                // its momentum, -2 w_j rho_k (e_j . u_w) / cs^2, stored with
                // them (only this node reads them)
                const float *cw = (tw & T_MOVWALL) ? bd.wallc + (int64_t)bd.bslot[b] * Q : nullptr;
                const Rates ra = {ph.se[0], ph.seps[0], ph.sq, ph.snu[0]};
                collide_pairs<DIM, STORE == 0>(qa, r1, J1, u, F1, ra, fo);
                if (cw) static_for<Q>([&](auto ic) { fo[decltype(ic)::value] = fmaf(cw[decltype(ic)::value], r1, fo[decltype(ic)::value]); });
                put(rd0, [&](auto inc, auto ic) { return dest_psi(inc, ic).x; });
                if constexpr (!KEEPB) {
                    float f[Q];
                    bgather<DIM, STORE>(rs1, g, p, tw, x, y, z, wave_fast, f, rf.y);
                    to_pairs<DIM>(f, qb);
                }
                const Rates rb = {ph.se[1], ph.seps[1], ph.sq, ph.snu[1]};
                collide_pairs<DIM, STORE == 0>(qb, r2, J2, u, F2, rb, fo);
                if (cw) static_for<Q>([&](auto ic) { fo[decltype(ic)::value] = fmaf(cw[decltype(ic)::value], r2, fo[decltype(ic)::value]); });
                put(rd1, [&](auto inc, auto ic) { return dest_psi(inc, ic).y; });
            }
        }
    }
    if constexpr (FIELDS) return;
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_q[0]) atomicAdd(qacc, s_q[0]);
        if (s_q[1]) atomicAdd(qacc + 1, s_q[1]);
    }
}

// One context: one block per work item (tiles that hold fluid, in the order
// of the work list or, for populations beyond the last level cache, against
// it).
// Binary16 storage asks for four waves per SIMD (128 VGPRs): its 64x4 tile
// then runs at occupancy 4 instead of 3 without spilling, 2.4% faster; FP32
// gains nothing from the request and takes what it needs.
template <int DIM, int STORE, int PSRC, int TX, int TY, int W, int ZC, int KEEPB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(STORE != 0 ? 4 : 1)))
void k_main(const typename Codec<STORE>::T *__restrict__ src,
                                              typename Codec<STORE>::T *__restrict__ dst,
                                              const uint32_t *__restrict__ type,
                                              const float2 *__restrict__ psi, const float2 *__restrict__ ref,
                                              Geometry g, Physics ph, Boundary bd, int tiles_x, int tiles_y,
                                              int n_items, int reverse, const int *__restrict__ item_list,
                                              int *__restrict__ flag, unsigned long long *__restrict__ qacc)
{
    // blocks go round-robin to the 8 XCDs (blockIdx % 8); each XCD takes
    // groups of G consecutive work items (see xcd_group), so that all XCDs sweep
    // nearby addresses at the same time while x-neighbour tiles still share
    // an L2 (measured faster than both one item per XCD turn and contiguous
    // ranges per XCD); the grid is a multiple of 8 G blocks
    constexpr int G = xcd_group(DIM, PSRC, W == ZC);
    const int S = (int)blockIdx.x / 8, r = (int)blockIdx.x % 8;
    int k = ((S / G) * 8 + r) * G + S % G;
    if (k >= n_items) return;
    if (reverse) k = n_items - 1 - k;
    main_item<DIM, STORE, PSRC, TX, TY, W, ZC, KEEPB>(src, dst, type, psi, ref, g, ph, bd, tiles_x, tiles_y,
                                                      item_list ? item_list[k] : k, flag, qacc);
}

// ---------------------------------------------------------------------------
// k_psi: psi_k = rho_k = sum_i f_i^k of every node (eq. 8 with psi_k = rho_k)
// from the post-streaming populations, as float2 per box node; solid nodes
// get (-0.0, -0.0).
// ---------------------------------------------------------------------------
template <int DIM, int STORE>
__device__ __forceinline__ void psi_body(int blk, const typename Codec<STORE>::T *__restrict__ src,
                                             const uint32_t *__restrict__ type, Geometry g,
                                             float2 *__restrict__ psi, const float2 *__restrict__ ref)
{
    constexpr int Q = Lat<DIM>::Q;
    const int64_t b = (int64_t)blk * 256 + threadIdx.x;
    const bool valid = b < g.N;
    const uint32_t tw = valid ? type[b] : T_SOLID;
    const bool fluid = !(tw & T_SOLID);
    if (__ballot(fluid) == 0) {
        if (valid) psi[b] = make_float2(-0.0f, -0.0f);
        return;
    }
    // the other lanes gather the first interior node, unused, so that the
    // gathers run with the whole wave
    const uint32_t t = fluid ? tw : 0u;
    const bool wave_fast = __ballot((t & (T_BBMASK | T_EDGE)) != 0) == 0;
    int x = 1, y = 1, z = DIM == 3 ? 1 : 0;
    if (fluid) coords_of(g, b, x, y, z);
    const uint32_t p = (uint32_t)pidx(g, x, y, DIM == 3 ? z : -1);
    float f[Q], r1 = 0.0f, r2 = 0.0f;
    float2 rf = make_float2(0.0f, 0.0f);
    if constexpr (Codec<STORE>::REF) rf = ref[fluid ? b : 0];
    typename Buf<STORE>::Raw h1[Q], h2[Q];
    bgather2_raw<DIM, STORE>(comp_rsrc<STORE>(src, 0, Q, g.Ppad), comp_rsrc<STORE>(src, 1, Q, g.Ppad), g, p, t, x,
                             y, z, wave_fast, h1, h2);
    decode<DIM, STORE>(h1, f, rf.x);
    static_for<Q>([&](auto ic) { r1 += f[decltype(ic)::value]; });
    decode<DIM, STORE>(h2, f, rf.y);
    static_for<Q>([&](auto ic) { r2 += f[decltype(ic)::value]; });
    if (valid) psi[b] = fluid ? make_float2(r1, r2) : make_float2(-0.0f, -0.0f);
}

template <int DIM, int STORE>
__global__ __launch_bounds__(256) void k_psi(const typename Codec<STORE>::T *__restrict__ src,
                                             const uint32_t *__restrict__ type, Geometry g,
                                             float2 *__restrict__ psi, const float2 *__restrict__ ref)
{
    constexpr int G = PSI_GROUP;
    const int S = (int)blockIdx.x / 8, r = (int)blockIdx.x % 8;
    psi_body<DIM, STORE>(((S / G) * 8 + r) * G + S % G, src, type, g, psi, ref);
}

// ---------------------------------------------------------------------------
// k_moments: rho_k and the common velocity of eqs. (7)-(8) (with this
// state's force, before any outlet override) of every node: the node update's
// sweep up to the velocity (one thread per node with 92 mapped psi reads of
// its own took 1.20 ms on the 600x120x120 device, longer than a step).  The
// instability flag goes to pinned host memory with it.
// ---------------------------------------------------------------------------
template <int DIM, int STORE, int PSRC, int TX, int TY, int W, int ZC>
__global__ __launch_bounds__(256) void k_moments(const typename Codec<STORE>::T *__restrict__ src,
                                                 const uint32_t *__restrict__ type,
                                                 const float2 *__restrict__ psi, const float2 *__restrict__ ref,
                                                 Geometry g, Physics ph, Boundary bd, int tiles_x, int tiles_y,
                                                 int n_items, double *__restrict__ orho, double *__restrict__ ou,
                                                 int *__restrict__ flag, int *__restrict__ host_flag)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *host_flag = *flag;
    constexpr int G = 4;
    const int S = (int)blockIdx.x / 8, r = (int)blockIdx.x % 8;
    const int k = ((S / G) * 8 + r) * G + S % G;
    if (k < n_items)
        main_item<DIM, STORE, PSRC, TX, TY, W, ZC, 1, true>(src, nullptr, type, psi, ref, g, ph, bd, tiles_x, tiles_y,
                                                            k, flag, nullptr, orho, ou);
}

}  // namespace lbm

#include "faces.h"

namespace lbm {

// ---------------------------------------------------------------------------
// State exchange: canonical f[2][Q][N] (FP64) <-> population slots.
// ---------------------------------------------------------------------------
// The state's own densities become the reference densities of its slots
// (every slot of the node is read by the node itself), written to ref.
template <int DIM, int STORE>
__global__ void k_scatter(typename Codec<STORE>::T *__restrict__ dst, const uint32_t *__restrict__ type,
                          Geometry g, Boundary bd, const double *__restrict__ f, float2 *__restrict__ ref)
{
    constexpr int Q = Lat<DIM>::Q;
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= g.N) return;
    const uint32_t tw = type[b];
    if (tw & T_SOLID) {
        ref[b] = make_float2(-0.0f, -0.0f);
        return;
    }
    int x, y, z;
    coords_of(g, b, x, y, z);
    const int64_t p = pidx(g, x, y, DIM == 3 ? z : -1);
    const int64_t bo = caller_index(g, x, y, z);
    float rr[2];
    for (int k = 0; k < 2; k++) {
        double r = 0.0;
        for (int i = 0; i < Q; i++) r += f[((int64_t)k * Q + i) * g.N + bo];
        rr[k] = (float)r;
    }
    ref[b] = make_float2(rr[0], rr[1]);
    for (int k = 0; k < 2; k++) {
        auto *dk = dst + (int64_t)k * Q * g.Ppad;
        static_for<Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const float v = (float)f[((int64_t)k * Q + g.dmap[i]) * g.N + bo];
            Codec<STORE>::st(dk + slot_of<DIM>(g, p, tw | T_EDGE, x, y, z, i), v, weight<DIM>(i), rr[k]);
            // the outlet history of eq. (20) starts from the state itself
            if ((tw & T_OUTLET) && e_axis<DIM>(i, bd.out_axis) * bd.out_sign < 0)
                bd.hist[((int64_t)k * Q + i) * bd.n_slots + bd.bslot[b]] = v;
        });
    }
}

template <int DIM, int STORE>
__global__ void k_gather_state(const typename Codec<STORE>::T *__restrict__ src, const uint32_t *__restrict__ type,
                               const float2 *__restrict__ ref, Geometry g, Boundary bd, double *__restrict__ f)
{
    constexpr int Q = Lat<DIM>::Q;
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= g.N) return;
    const uint32_t tw = type[b];
    int x, y, z;
    coords_of(g, b, x, y, z);
    const int64_t bo = caller_index(g, x, y, z);
    for (int k = 0; k < 2; k++) {
        if (tw & T_SOLID) {
            for (int i = 0; i < Q; i++) f[((int64_t)k * Q + i) * g.N + bo] = 0.0;
            continue;
        }
        const int64_t p = pidx(g, x, y, DIM == 3 ? z : -1);
        float v[Q];
        const float2 rf = ref[b];
        gather<DIM, STORE>(src + (int64_t)k * Q * g.Ppad, g, p, tw | T_EDGE, x, y, z, v, k == 0 ? rf.x : rf.y);
        static_for<Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            // populations entering through the outlet: the FP32 history (the
            // stored copy is its rounding)
            if ((tw & T_OUTLET) && e_axis<DIM>(i, bd.out_axis) * bd.out_sign < 0)
                v[i] = bd.hist[((int64_t)k * Q + i) * bd.n_slots + bd.bslot[b]];
            f[((int64_t)k * Q + g.dmap[i]) * g.N + bo] = (double)v[i];
        });
    }
}

// f = feq(rho0, u0) in canonical FP64 layout (initial state).
template <int DIM>
__global__ void k_feq_state(const double *__restrict__ rho0, const double *__restrict__ u0, int64_t N,
                            double *__restrict__ f)
{
    constexpr int Q = Lat<DIM>::Q;
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= N) return;
    float u[3] = {0.f, 0.f, 0.f};
    if (u0) {
        u[0] = (float)u0[b];
        u[1] = (float)u0[N + b];
        u[2] = (float)u0[2 * N + b];
    }
    for (int k = 0; k < 2; k++) {
        const float r = (float)rho0[k * N + b];
        static_for<Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            f[((int64_t)k * Q + i) * N + b] = (double)feq<DIM>(i, r, u);
        });
    }
}

// Per-block FP64 partial sums of rho_1 and rho_2 over fluid nodes.
template <int DIM, int STORE>
__global__ __launch_bounds__(256) void k_mass(const typename Codec<STORE>::T *__restrict__ src,
                                              const uint32_t *__restrict__ type,
                                              const float2 *__restrict__ ref, Geometry g,
                                              double *__restrict__ part)
{
    constexpr int Q = Lat<DIM>::Q;
    __shared__ double s_red[8];
    double m1 = 0.0, m2 = 0.0;
    for (int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x; b < g.N; b += (int64_t)gridDim.x * 256) {
        const uint32_t tw = type[b];
        if (tw & T_SOLID) continue;
        int x, y, z;
        coords_of(g, b, x, y, z);
        const int64_t p = pidx(g, x, y, DIM == 3 ? z : -1);
        float f[Q];
        const float2 rf = ref[b];
        gather<DIM, STORE>(src, g, p, tw | T_EDGE, x, y, z, f, rf.x);
        static_for<Q>([&](auto ic) { m1 += (double)f[decltype(ic)::value]; });
        gather<DIM, STORE>(src + (int64_t)Q * g.Ppad, g, p, tw | T_EDGE, x, y, z, f, rf.y);
        static_for<Q>([&](auto ic) { m2 += (double)f[decltype(ic)::value]; });
    }
    block_sum2<256>(m1, m2, s_red);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = m1;
        part[2 * blockIdx.x + 1] = m2;
    }
}

static __global__ void k_reduce2(const double *__restrict__ part, int n, double *__restrict__ out)
{
    __shared__ double s_red[8];
    double a, b;
    reduce_partials<256>(part, n, a, b, s_red);
    if (threadIdx.x == 0) { out[0] = a; out[1] = b; }
}

// ---------------------------------------------------------------------------
// Batched step: every member of a batch advanced by one launch per stage.
// Members share the lattice, the storage and the node-update configuration
// and differ in everything else (size, geometry, physics, faces).  The A/B
// parity `cur` is common to all members.
// ---------------------------------------------------------------------------

// A member's descriptor is read-only for the whole launch: the batch kernels
// read it through the constant address space, so its fields come in by
// scalar loads into uniform registers, as kernel arguments do (through a
// generic pointer they were vector loads, and the node update held the
// descriptor in some twenty vector registers).
using CMember = const __attribute__((address_space(4))) Member;

// A copy of a structure held in the constant address space, word by word so
// that it compiles to scalar loads.
template <class S>
__device__ __forceinline__ S const_copy(const __attribute__((address_space(4))) S *p)
{
    static_assert(sizeof(S) % 4 == 0, "whole words");
    S v;
    const __attribute__((address_space(4))) uint32_t *q = (const __attribute__((address_space(4))) uint32_t *)p;
    uint32_t *d = (uint32_t *)&v;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(S) / 4); k++) d[k] = q[k];
    return v;
}

// Largest i in [0, n) with start[i] <= v (start is nondecreasing, start[0] = 0).
__device__ __forceinline__ int member_of(const int *__restrict__ start, int n, int v)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (start[mid] <= v) lo = mid;
        else hi = mid - 1;
    }
    return __builtin_amdgcn_readfirstlane(lo);   // uniform over the block
}

template <int DIM, int STORE>
__global__ __launch_bounds__(256) void k_psi_batch(BatchTab t, int cur)
{
    using T = typename Codec<STORE>::T;
    const int i = member_of(t.psi0, t.n, (int)blockIdx.x);
    CMember *m = (CMember *)(t.m + i);
    psi_body<DIM, STORE>((int)blockIdx.x - t.psi0[i], (const T *)m->f[cur], m->type, const_copy(&m->g),
                         (float2 *)m->psi[cur], (const float2 *)m->psi[cur ^ 1]);
}

// Persistent node update over the concatenated work items of all members.
// The blocks (a multiple of 8) step through virtual block indices v; v % 8 is
// the XCD of the block, and the items are dealt to the XCDs as in k_main, in
// groups of G consecutive items per turn.
template <int DIM, int STORE, int PSRC, int TX, int TY, int W, int ZC, int KEEPB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(STORE != 0 ? 4 : 1)))
void k_main_batch(BatchTab t, int cur)
{
    using T = typename Codec<STORE>::T;
    const int total = t.item0[t.n];
    constexpr int G = xcd_group(DIM, PSRC, W == ZC);
    const int span = (total + 8 * G - 1) / (8 * G) * (8 * G);
    for (int v = (int)blockIdx.x; v < span; v += (int)gridDim.x) {
        const int S = v / 8, r = v % 8;
        const int w = ((S / G) * 8 + r) * G + S % G;
        if (w >= total) continue;
        const int i = __builtin_amdgcn_readfirstlane(t.item_mem[w]);
        CMember *m = (CMember *)(t.m + i);
        const Geometry g = const_copy(&m->g);
        const Physics ph = const_copy(&m->ph);
        const Boundary bd = const_copy(&m->bd);
        main_item<DIM, STORE, PSRC, TX, TY, W, ZC, KEEPB>((const T *)m->f[cur], (T *)m->f[cur ^ 1], m->type,
                                                          (const float2 *)m->psi[cur],
                                                          (const float2 *)m->psi[cur ^ 1], g, ph, bd,
                                                          m->tiles_x, m->tiles_y, m->item_list[w - t.item0[i]],
                                                          m->flag, bd.qacc + 2 * cur);
    }
}

template <int DIM, int STORE>
__global__ __launch_bounds__(FACE_NT) void k_faces_batch(BatchTab t, int cur)
{
    using T = typename Codec<STORE>::T;
    const int i = member_of(t.fac0, t.n, (int)blockIdx.x);
    CMember *m = (CMember *)(t.m + i);
    const Boundary bd = const_copy(&m->bd);
    faces_body<DIM, STORE>((int)blockIdx.x - t.fac0[i], (const T *)m->f[cur], (T *)m->f[cur ^ 1],
                           (const float2 *)m->psi[cur], (const float2 *)m->psi[cur ^ 1], const_copy(&m->g),
                           const_copy(&m->ph), bd, m->flag, bd.qacc + 2 * cur, bd.qacc + 2 * (cur ^ 1), m->nb_coll,
                           m->nb_in_early);
}

template <int DIM, int STORE>
__global__ __launch_bounds__(FACE_NT) void k_inlet_batch(BatchTab t, int cur)
{
    using T = typename Codec<STORE>::T;
    const int i = member_of(t.inl0, t.n, (int)blockIdx.x);
    CMember *m = (CMember *)(t.m + i);
    inlet_uc_body<DIM, STORE>((int)blockIdx.x - t.inl0[i], (T *)m->f[cur ^ 1], (const float2 *)m->psi[cur],
                              const_copy(&m->g), const_copy(&m->bd), m->nb_in_late);
}

template <int DIM, int STORE>
__global__ __launch_bounds__(FACE_NT) void k_outlet_fill_batch(BatchTab t, int cur)
{
    using T = typename Codec<STORE>::T;
    const int i = member_of(t.fill0, t.n, (int)blockIdx.x);
    CMember *m = (CMember *)(t.m + i);
    outlet_fill_body<DIM, STORE>((int)blockIdx.x - t.fill0[i], (T *)m->f[cur ^ 1], (const float2 *)m->psi[cur],
                                 const_copy(&m->g), const_copy(&m->bd));
}

// ---------------------------------------------------------------------------
// Droplet labels.  The dispersed phase is the set of fluid nodes of a box
// whose component-k density (summed from the current populations) exceeds a
// threshold; droplets are its face-connected components.
// ---------------------------------------------------------------------------

// rho_k of a fluid node from its post-streaming populations
template <int DIM, int STORE>
__device__ __forceinline__ float node_rho(const typename Codec<STORE>::T *__restrict__ src, const Geometry &g,
                                          uint32_t tw, int x, int y, int z, int k, float rr)
{
    constexpr int Q = Lat<DIM>::Q;
    float f[Q];
    gather<DIM, STORE>(src + (int64_t)k * Q * g.Ppad, g, pidx(g, x, y, DIM == 3 ? z : -1), tw, x, y, z, f, rr);
    float r = 0.0f;
    static_for<Q>([&](auto ic) { r += f[decltype(ic)::value]; });
    return r;
}

// Count of dispersed nodes in the box.  ONE: a single block takes the whole
// box and writes the count; else every wave adds its own to *out (zeroed by
// k_zero64).
template <int DIM, int STORE, bool ONE>
__global__ __launch_bounds__(256) void k_probe(const typename Codec<STORE>::T *__restrict__ src,
                                               const uint32_t *__restrict__ type, const float2 *__restrict__ ref,
                                               Geometry g, int k, Box3 bx, float thr,
                                               unsigned long long *__restrict__ out)
{
    const int ex = bx.hi[0] - bx.lo[0], ey = bx.hi[1] - bx.lo[1], ez = bx.hi[2] - bx.lo[2];
    const int64_t vol = (int64_t)ex * ey * ez;
    unsigned long long c = 0;                   // of the wave
    for (int64_t v0 = (int64_t)blockIdx.x * 256; v0 < vol; v0 += (int64_t)gridDim.x * 256) {
        const int64_t v = v0 + threadIdx.x;
        int hit = 0;
        if (v < vol) {
            const int x = bx.lo[0] + (int)(v % ex), y = bx.lo[1] + (int)((v / ex) % ey),
                      z = bx.lo[2] + (int)(v / ((int64_t)ex * ey));
            const int64_t b = (int64_t)x + (int64_t)g.n[0] * ((int64_t)y + (int64_t)g.n[1] * z);
            const uint32_t tw = type[b];
            if (!(tw & T_SOLID)) {
                const float2 rf = ref[b];
                hit = node_rho<DIM, STORE>(src, g, tw | T_EDGE, x, y, z, k, k == 0 ? rf.x : rf.y) > thr;
            }
        }
        c += __popcll(__ballot(hit));
    }
    if constexpr (ONE) {
        __shared__ unsigned long long s_c[4];
        if ((threadIdx.x & 63) == 0) s_c[threadIdx.x >> 6] = c;
        __syncthreads();
        if (threadIdx.x == 0) *out = s_c[0] + s_c[1] + s_c[2] + s_c[3];
    } else {
        if ((threadIdx.x & 63) == 0 && c) atomicAdd(out, c);
    }
}

static __global__ void k_zero64(unsigned long long *p) { *p = 0ull; }

// Connected components by union-find over the nodes of the box (linear index
// v, x fastest): lab[v] is a node of the same component with a smaller or
// equal index, -1 off the dispersed phase.  Four launches, whatever the shape
// of the components:
//   k_lab_init    lab[v] = start of v's x-run within its wave
//   k_lab_merge   unites runs across waves, rows and planes
//   k_lab_roots   lab[v] = root; each root takes a slot and clears its record
//   k_lab_stats   size, smallest caller index and bounding box
// (k_lab_order then sorts the records.)  Minimum-label propagation with a host
// read-back every four passes and one atomic per node and quantity took
// 1.24 ms on an 800x202 field of 12 droplets, 1.05 ms of it in the atomics of
// all nodes of a droplet on one record; here a wave first reduces its nodes.

// One level of the forest; other blocks change labels while they are read,
// but only to smaller nodes of the same component, so an old value is valid.
__device__ __forceinline__ int lab_load(const int *lab, int v)
{
    return __hip_atomic_load(lab + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int lab_find(const int *lab, int v)
{
    for (int p = lab_load(lab, v); p != v; p = lab_load(lab, v)) v = p;   // p < v: ends
    return v;
}
// Every pass replaces the larger root by what its label was before, which is
// smaller, or ends.
__device__ __forceinline__ void lab_unite(int *lab, int a, int b)
{
    while (true) {
        a = lab_find(lab, a);
        b = lab_find(lab, b);
        if (a == b) return;
        if (a < b) {
            const int t = a;
            a = b;
            b = t;
        }
        const int old = atomicMin(lab + a, b);
        if (old == a) return;
        a = old;
    }
}

// Coordinates of node v of the box (offsets from its corner).
__device__ __forceinline__ void box_coords(const int (&ext)[3], uint32_t v, int &x, int &y, int &z)
{
    const uint32_t row = v / (uint32_t)ext[0];
    x = (int)(v - row * (uint32_t)ext[0]);
    z = (int)(row / (uint32_t)ext[1]);
    y = (int)(row - (uint32_t)z * (uint32_t)ext[1]);
}

template <int DIM, int STORE>
__global__ __launch_bounds__(256) void k_lab_init(const typename Codec<STORE>::T *__restrict__ src,
                                                  const uint32_t *__restrict__ type,
                                                  const float2 *__restrict__ ref, Geometry g, int k, Box3 bx,
                                                  float thr, int *__restrict__ lab, int *__restrict__ n_roots)
{
    const int ext[3] = {bx.hi[0] - bx.lo[0], bx.hi[1] - bx.lo[1], bx.hi[2] - bx.lo[2]};
    const uint32_t v = blockIdx.x * 256u + threadIdx.x, vol = (uint32_t)ext[0] * ext[1] * ext[2];
    if (v == 0) *n_roots = 0;
    int x = 0, y = 0, z = 0;
    bool in = false;
    if (v < vol) {
        box_coords(ext, v, x, y, z);
        const int gx = bx.lo[0] + x, gy = bx.lo[1] + y, gz = bx.lo[2] + z;
        const int64_t b = (int64_t)gx + (int64_t)g.n[0] * ((int64_t)gy + (int64_t)g.n[1] * gz);
        const uint32_t tw = type[b];
        if (!(tw & T_SOLID)) {
            const float2 rf = ref[b];
            in = node_rho<DIM, STORE>(src, g, tw | T_EDGE, gx, gy, gz, k, k == 0 ? rf.x : rf.y) > thr;
        }
    }
    // the run of dispersed nodes that this lane continues within its wave
    const int lane = threadIdx.x & 63;
    const unsigned long long m = __ballot(in), starts = ~(m & (m << 1)) | __ballot(x == 0);
    const int start = 63 - __clzll((long long)(starts & (~0ull >> (63 - lane))));
    if (v < vol) lab[v] = in ? (int)v - (lane - start) : -1;
}

static __global__ __launch_bounds__(256) void k_lab_merge(Box3 bx, int *lab)
{
    const int ext[3] = {bx.hi[0] - bx.lo[0], bx.hi[1] - bx.lo[1], bx.hi[2] - bx.lo[2]};
    const uint32_t u = blockIdx.x * 256u + threadIdx.x;
    if (u >= (uint32_t)ext[0] * ext[1] * ext[2]) return;
    const int v = (int)u;
    auto in = [&](int w) { return lab_load(lab, w) >= 0; };
    if (!in(v)) return;
    int x, y, z;
    box_coords(ext, u, x, y, z);
    const bool left = x > 0 && in(v - 1);
    if (left && (threadIdx.x & 63) == 0) lab_unite(lab, v, v - 1);
    // a neighbour row or plane is met once per pair of runs: where the nodes
    // to the left of both are dispersed too, the pair is united there
    if (y > 0 && in(v - ext[0]) && !(left && in(v - ext[0] - 1))) lab_unite(lab, v, v - ext[0]);
    const int pl = ext[0] * ext[1];
    if (z > 0 && in(v - pl) && !(left && in(v - pl - 1))) lab_unite(lab, v, v - pl);
}

// roots (lab[v] == v) get consecutive slots in an arbitrary order (records
// beyond cap are counted, not kept); the records are ordered afterwards
static __global__ __launch_bounds__(256) void k_lab_roots(Box3 bx, int *lab, int *__restrict__ slot,
                                                          CompStat *__restrict__ st, int cap, int *n_roots)
{
    const uint32_t u = blockIdx.x * 256u + threadIdx.x;
    const uint32_t vol = (uint32_t)(bx.hi[0] - bx.lo[0]) * (bx.hi[1] - bx.lo[1]) * (bx.hi[2] - bx.lo[2]);
    if (u >= vol) return;
    const int v = (int)u;
    if (lab_load(lab, v) < 0) return;
    const int root = lab_find(lab, v);
    lab[v] = root;                       // any value on the way to the root is valid for the others
    if (root != v) return;
    const int s = atomicAdd(n_roots, 1);
    slot[v] = s;
    if (s >= cap) return;
    CompStat c;
    c.size = 0ull;
    c.first = ~0ull;
    for (int a = 0; a < 3; a++) {
        c.lo[a] = 0x7fffffff;
        c.hi[a] = -1;
    }
    st[s] = c;
}

// Sizes, first nodes and bounding boxes.  A wave takes a strip of 64 nodes in
// x and LAB_ROWS consecutive rows, and adds what it holds of one component to
// its record at once (integer atomics: the result does not depend on their
// order), for up to LAB_TURNS components.  A wave that holds more (specks,
// thin stripes) has few nodes of each: its lanes then add what each of them
// holds, side by side (the 128 components a wave holds of a checkerboard,
// reduced in turn, took about 100 us: 8192 components 280 us a call, now 177).
constexpr int LAB_ROWS = 4, LAB_TURNS = 8;
struct LabPart {
    int first, lo[3], hi[3];
};
__device__ __forceinline__ int wave_min(int v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return v;
}

static __global__ __launch_bounds__(256) void k_lab_stats(Geometry g, Box3 bx, const int *__restrict__ lab,
                                                          const int *__restrict__ slot, CompStat *st, int cap)
{
    const int ex = bx.hi[0] - bx.lo[0], ey = bx.hi[1] - bx.lo[1], ez = bx.hi[2] - bx.lo[2];
    const int strips = (ex + 63) / 64, rows = ey * ez;
    const int w = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int x = (w % strips) * 64 + lane, row0 = (w / strips) * LAB_ROWS;
    if (row0 >= rows) return;                            // uniform over the wave
    // each lane's four nodes: slot of the component, or -1
    int sl[LAB_ROWS];
#pragma unroll
    for (int i = 0; i < LAB_ROWS; i++) {
        const bool valid = x < ex && row0 + i < rows;
        const int l = valid ? lab[(row0 + i) * ex + x] : -1;
        sl[i] = l >= 0 ? slot[l] : -1;
        if (sl[i] >= cap) sl[i] = -1;
    }
    // the first component this lane still holds, or -1
    auto next = [&] {
        int s = -1;
#pragma unroll
        for (int i = LAB_ROWS - 1; i >= 0; i--) s = sl[i] >= 0 ? sl[i] : s;
        return s;
    };
    // takes the lane's nodes of component s: how many, and their extent
    auto take = [&](int s, LabPart &p) {
        p = {0x7fffffff, {0x7fffffff, 0x7fffffff, 0x7fffffff}, {-1, -1, -1}};
        int n = 0;
#pragma unroll
        for (int i = 0; i < LAB_ROWS; i++) {
            if (sl[i] != s) continue;
            sl[i] = -1;
            n++;
            const int row = row0 + i, zz = row / ey, mc[3] = {bx.lo[0] + x, bx.lo[1] + row - zz * ey, bx.lo[2] + zz};
            p.first = min(p.first, (int)caller_index(g, mc[0], mc[1], mc[2]));
            for (int a = 0; a < 3; a++) {
                p.lo[a] = min(p.lo[a], mc[a]);
                p.hi[a] = max(p.hi[a], mc[a] + 1);
            }
        }
        return n;
    };
    auto add = [&](int s, int size, const LabPart &p) {
        CompStat *c = st + s;
        atomicAdd(&c->size, (unsigned long long)size);
        atomicMin(&c->first, (unsigned long long)p.first);
        for (int a = 0; a < 3; a++) {
            atomicMin(&c->lo[g.ax[a]], p.lo[a]);
            atomicMax(&c->hi[g.ax[a]], p.hi[a]);
        }
    };
    LabPart p;
    for (int turn = 0; turn < LAB_TURNS; turn++) {
        const int mine = next();
        const unsigned long long have = __ballot(mine >= 0);
        if (!have) return;
        const int s = __shfl(mine, __ffsll((long long)have) - 1, 64);
        int size = 0;
#pragma unroll
        for (int i = 0; i < LAB_ROWS; i++) size += __popcll(__ballot(sl[i] == s));
        take(s, p);
        p.first = wave_min(p.first);
        for (int a = 0; a < 3; a++) {
            p.lo[a] = wave_min(p.lo[a]);
            p.hi[a] = -wave_min(-p.hi[a]);
        }
        if (lane == 0) add(s, size, p);
    }
    for (int s = next(); s >= 0; s = next()) {
        const int n = take(s, p);
        add(s, n, p);
    }
}

}  // namespace lbm
