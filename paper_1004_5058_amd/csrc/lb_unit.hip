// HIP kernels (gfx950) of the time step at tau = 1: the step of lb_kernels.hip
// where the BGK collision of Eq. (1) replaces every population by the
// equilibrium at the shifted velocity, f*_is = f^eq_i(rho_s, v_s).  FP64, FP32 and
// the moment form run these kernels at tau = 1 (16-bit storage keeps the roundings of
// the general ones).  Per step of those and of these: 4096^2 FP32 in pairs 0.286, 0.266 ms,
// moment form 0.258, 0.194; 128^2 FP64 20, 8.6 us; 512^2 FP32 in pairs 19, 13.7, single steps 12.1.
//
// What tau = 1 saves.  Nothing of a row's populations is needed past its four
// sums (the two density deviations and the momentum), so a row leaves the
// registers as soon as it is loaded, and between two fused steps a column
// hands its neighbours partial sums, not populations (Flow below).
//
// The force, row first.  The 24-offset stencil is summed as the rows arrive:
// row r and its x neighbours give, per species, three x terms u0, u1, u2 and
// two y terms w1, w2 (the shell weights folded in), which are added to the
// force sums of the rows r-2 .. r+2 held in registers (Belt).  A site's
// neighbourhood is then read once per row (four psi neighbours and two rho
// neighbours per species) instead of 34 pairs of LDS reads per site, with 46
// instead of 80 multiply-adds for psi.  Each sum is formed in the order of the
// rows, so results do not depend on the tiles.
//
// Rows beyond a wall are the even mirror of the first two fluid rows; their
// terms are added when the fluid row they mirror arrives (push's edge).
#include "lb_step.hpp"

namespace lbk {

namespace {

// ------------------------------------------------------------ lane shifts --

// The value of the lane one column to the right / left (0 past the wave's
// ends), by the gfx9 wave shifts of the DPP unit: a VALU operation, no LDS.
template <int CTRL> __device__ __forceinline__ float lane_shift(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
template <int CTRL> __device__ __forceinline__ double lane_shift(double x)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
template <class C> __device__ __forceinline__ C right(C x) { return lane_shift<0x130>(x); }   // wave_shl:1
template <class C> __device__ __forceinline__ C left(C x) { return lane_shift<0x138>(x); }    // wave_shr:1

// ------------------------------------------------------- streaming sums ----

// What a row of populations leaves: the density deviations of A and B and the
// momentum of both.
template <class C> struct Sums { C da, db, jx, jy; };
// Forms the sums where they stand: the compiler would otherwise sink the
// momentum's additions to the collision two rows later and keep the row's
// populations alive until then.
template <class C> __device__ __forceinline__ void settle(Sums<C>& s)
{
    asm volatile("" : "+v"(s.da), "+v"(s.db), "+v"(s.jx), "+v"(s.jy));
}

// Partial sums of one column's post-collision populations of a row by their x
// direction (s0, sp, sm: c_x = 0, +1, -1; per species), of their y momentum
// (j0, jp, jm) and of what they carry in x (xp, xm: c_x = +1, -1).  The momenta are
// sums over the species, direction by direction: the deviations of A and B, opposite
// where the fluid is dense everywhere, cancel before they can round.  (x momentum as
// the difference of sp and sm rounded a row of few distinct values by 4e-9 as a whole,
// which the wall stress of the next 26 steps, 1e-4, felt as 2.4e-6 of itself.)  Added in the order of the rows they come from: c_y = +1 (row
// y-1), 0 (row y), -1 (row y+1).
template <class C> struct Part { C s0[2], sp[2], sm[2], j0, jp, jm, xp, xm; };

template <class C> __device__ __forceinline__ void settle(Part<C>& p)
{
    asm volatile("" : "+v"(p.s0[0]), "+v"(p.s0[1]), "+v"(p.sp[0]), "+v"(p.sp[1]), "+v"(p.sm[0]), "+v"(p.sm[1]),
                 "+v"(p.j0), "+v"(p.jp), "+v"(p.jm));
}

// The sums of a node from the parts of its own column (s0), the column to its
// left (c_x = +1) and to its right (c_x = -1).
template <class C>
__device__ __forceinline__ Sums<C> join(const C (&s0)[2], const C (&sp)[2], const C (&sm)[2], C j0, C jp, C jm, C xp, C xm)
{
    Sums<C> o;
    o.da = (s0[0] + sp[0]) + sm[0];
    o.db = (s0[1] + sp[1]) + sm[1];
    o.jx = xp - xm;
    o.jy = (j0 + jp) + jm;
    return o;
}
// What the populations returned by a wall add to their node (a: the normal one, b and
// c: the returned ones with c_x = +1 and -1; up: c_y = +1, the bottom wall).
template <class C>
__device__ __forceinline__ Sums<C> wall_sums(C aA, C bA, C cA, C aB, C bB, C cB, bool up)
{
    Sums<C> o;
    o.da = (aA + bA) + cA;
    o.db = (aB + bB) + cB;
    o.jx = (bA + bB) - (cA + cB);
    const C j = ((aA + aB) + (bA + bB)) + (cA + cB);
    o.jy = up ? j : -j;
    return o;
}
template <class C> __device__ __forceinline__ void add_sums(Sums<C>& s, const Sums<C>& w)
{
    s.da += w.da;
    s.db += w.db;
    s.jx += w.jx;
    s.jy += w.jy;
}

// The 18 incoming populations of a node as loaded, with Row's two and more.
template <class P> struct Raw {
    using C = typename P::C;           // (the storage type too)
    C v[18];
    __device__ __forceinline__ C operator[](int q) const { return v[q]; }
    template <int QA, int QB, bool NEG = false> __device__ __forceinline__ C two() const
    {
        return NEG ? v[QA] - v[QB] : v[QA] + v[QB];
    }
    template <int Q, bool NEG = false> __device__ __forceinline__ C more(C x) const
    {
        return NEG ? x - v[Q] : x + v[Q];
    }
    __device__ __forceinline__ void load(rsrc_t r0, rsrc_t r1, unsigned vl, unsigned vc, unsigned vr, unsigned pbytes)
    {
#pragma unroll
        for (int q = 0; q < 18; ++q) {
            const int cx = CX[q % 9];
            v[q] = bload<C>(q < 9 ? r0 : r1, cx > 0 ? vl : (cx < 0 ? vr : vc),
                            (unsigned)__builtin_amdgcn_readfirstlane((int)((q % 9) * pbytes)));
        }
    }
};

// The sums of a node from its 18 incoming populations, with the roundings of
// Part and join.  wall: 0, or 1 / 2 for the row at the bottom / top wall.
template <class P>
__device__ __forceinline__ Sums<typename P::C> row_sums(const Raw<P>& f, int wall)
{
    using C = typename P::C;
    if (wall == 0) {
        const C s0[2] = {f.template more<4>(f.template two<2, 0>()), f.template more<13>(f.template two<11, 9>())};
        const C sp[2] = {f.template more<8>(f.template two<5, 1>()), f.template more<17>(f.template two<14, 10>())};
        const C sm[2] = {f.template more<7>(f.template two<6, 3>()), f.template more<16>(f.template two<15, 12>())};
        const C p5 = f.template two<5, 14>(), p6 = f.template two<6, 15>();
        const C p7 = f.template two<7, 16>(), p8 = f.template two<8, 17>();
        return join(s0, sp, sm, f.template two<2, 11>() - f.template two<4, 13>(), p5 - p8, p6 - p7,
                    (p5 + f.template two<1, 10>()) + p8, (p6 + f.template two<3, 12>()) + p7);
    }
    if (wall == 1) {
        const C s0[2] = {f.template two<0, 4>(), f.template two<9, 13>()};
        const C sp[2] = {f.template two<1, 8>(), f.template two<10, 17>()};
        const C sm[2] = {f.template two<3, 7>(), f.template two<12, 16>()};
        const C p7 = f.template two<7, 16>(), p8 = f.template two<8, 17>();
        Sums<C> o = join(s0, sp, sm, -f.template two<4, 13>(), -p8, -p7, f.template two<1, 10>() + p8,
                         f.template two<3, 12>() + p7);
        add_sums(o, wall_sums<C>(f[2], f[5], f[6], f[11], f[14], f[15], true));
        return o;
    }
    const C s0[2] = {f.template two<2, 0>(), f.template two<11, 9>()};
    const C sp[2] = {f.template two<5, 1>(), f.template two<14, 10>()};
    const C sm[2] = {f.template two<6, 3>(), f.template two<15, 12>()};
    const C p5 = f.template two<5, 14>(), p6 = f.template two<6, 15>();
    Sums<C> o = join(s0, sp, sm, f.template two<2, 11>(), p5, p6, p5 + f.template two<1, 10>(),
                     p6 + f.template two<3, 12>());
    add_sums(o, wall_sums<C>(f[4], f[8], f[7], f[13], f[17], f[16], false));
    return o;
}

// The rows of one column in flight between a step and the next: mid has the
// c_y = +1 and 0 populations of the last row fed, up the c_y = +1 ones of the
// row above it.  feed(row y) returns row y-1 complete.
template <class C> struct Flow {
    Part<C> mid, up;
    __device__ __forceinline__ void clear()
    {
        mid = Part<C>{{0, 0}, {0, 0}, {0, 0}, 0, 0, 0, 0, 0};
        up = mid;
    }
    template <class R> __device__ __forceinline__ Part<C> feed(const R& q)
    {
        Part<C> done = mid;
        done.s0[0] = q.template more<4>(done.s0[0]);
        done.s0[1] = q.template more<13>(done.s0[1]);
        done.sp[0] = q.template more<8>(done.sp[0]);
        done.sp[1] = q.template more<17>(done.sp[1]);
        done.sm[0] = q.template more<7>(done.sm[0]);
        done.sm[1] = q.template more<16>(done.sm[1]);
        done.j0 = done.j0 - q.template two<4, 13>();
        const C p8 = q.template two<8, 17>(), p7 = q.template two<7, 16>();
        done.jp = done.jp - p8;
        done.jm = done.jm - p7;
        done.xp = done.xp + p8;
        done.xm = done.xm + p7;
        mid = up;
        mid.s0[0] = q.template more<0>(mid.s0[0]);
        mid.s0[1] = q.template more<9>(mid.s0[1]);
        mid.sp[0] = q.template more<1>(mid.sp[0]);
        mid.sp[1] = q.template more<10>(mid.sp[1]);
        mid.sm[0] = q.template more<3>(mid.sm[0]);
        mid.sm[1] = q.template more<12>(mid.sm[1]);
        mid.xp = up.jp + q.template two<1, 10>();
        mid.xm = up.jm + q.template two<3, 12>();
        up.s0[0] = q[2];
        up.s0[1] = q[11];
        up.sp[0] = q[5];
        up.sp[1] = q[14];
        up.sm[0] = q[6];
        up.sm[1] = q[15];
        up.j0 = q.template two<2, 11>();
        up.jp = q.template two<5, 14>();
        up.jm = q.template two<6, 15>();
        settle(mid);
        asm volatile("" : "+v"(mid.xp), "+v"(mid.xm));
        settle(up);   // (its xp and xm: jp and jm)
        return done;
    }
};

// ------------------------------------------------------------------ force --

// A wall's speed, in FP32 with the rest that its rounding leaves: a lattice at rest or in
// uniform shear feels a wall off by 3e-8 as a steady stress.
template <class C> struct WallSpeed { C hi, lo; };

// A lattice's coefficients in the arithmetic type, uniform over a wave.
template <class C> struct Coef {
    C k1[2], k2[2], k5[2], d4[2], d5[2], d8[2];   // psi weights on |c|^2 = 1, 2, 5; twice those on 4, 5, 8
    C kx1, kx2, inv_rho0, rref[2], pref[2], e[2];
    WallSpeed<C> u_top, u_bot;
    __device__ __forceinline__ explicit Coef(const LatDesc& d)
    {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            k1[s] = coef<C>(d.ks[s][0], d.fks[s][0]);
            k2[s] = coef<C>(d.ks[s][1], d.fks[s][1]);
            k5[s] = coef<C>(d.ks[s][3], d.fks[s][3]);
            d4[s] = coef<C>(d.kd[s][0], d.fkd[s][0]);
            d5[s] = coef<C>(d.kd[s][1], d.fkd[s][1]);
            d8[s] = coef<C>(d.kd[s][2], d.fkd[s][2]);
            rref[s] = coef<C>(d.rref[s], d.frref[s]);
            pref[s] = coef<C>(d.psiref[s], d.fpsiref[s]);
            e[s] = coef<C>(d.epsi[s], d.fepsi[s]);
        }
        kx1 = coef<C>(d.kx[0], d.fkx[0]);
        kx2 = coef<C>(d.kx[1], d.fkx[1]);
        inv_rho0 = coef<C>(d.inv_rho0, d.finv_rho0);
        u_top = WallSpeed<C>{coef<C>(d.u_top, d.fu_top), coef<C>(0.0, d.flu_top)};
        u_bot = WallSpeed<C>{coef<C>(d.u_bot, d.fu_bot), coef<C>(0.0, d.flu_bot)};
    }
};

// One site of a staged row: psi and rho deviations of A and B.
template <class C> using Quad = typename V4<C>::T;
template <class P>
__device__ __forceinline__ Quad<typename P::C> quad(const Sums<typename P::C>& s, const Coef<typename P::C>& k)
{
    Quad<typename P::C> q;
    q.x = dpsi<P>(s.da, k.e[0], k.inv_rho0);
    q.y = dpsi<P>(s.db, k.e[1], k.inv_rho0);
    q.z = s.da;
    q.w = s.db;
    return q;
}

// psi at columns -2 .. 2 and rho at -1 .. 1 around a site, per species.
template <class C> struct Near { C p[2][5], r[2][3]; };
template <class C> __device__ __forceinline__ Near<C> near_lanes(const Quad<C>& q)
{
    Near<C> n;
    const C p[2] = {q.x, q.y}, r[2] = {q.z, q.w};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        n.p[s][2] = p[s];
        n.p[s][1] = left(p[s]);
        n.p[s][0] = left(n.p[s][1]);
        n.p[s][3] = right(p[s]);
        n.p[s][4] = right(n.p[s][3]);
        n.r[s][1] = r[s];
        n.r[s][0] = left(r[s]);
        n.r[s][2] = right(r[s]);
    }
    return n;
}
// The same from a staged LDS row; c: the site's entry.
template <class C> __device__ __forceinline__ Near<C> near_lds(const Quad<C>* row, int c)
{
    Near<C> n;
#pragma unroll
    for (int dx = -2; dx <= 2; ++dx) {
        const Quad<C> q = row[c + dx];
        n.p[0][2 + dx] = q.x;
        n.p[1][2 + dx] = q.y;
        if (dx >= -1 && dx <= 1) {
            n.r[0][1 + dx] = q.z;
            n.r[1][1 + dx] = q.w;
        }
    }
    return n;
}

// The rows a column has in flight, in five slots (row r in slot r mod 5 of the
// tile's count): force sums of psi (fx, fy) and of the other species' rho (gx,
// gy) per species, and the site's own values and momentum.
template <class C> struct Belt {
    C fx[5][2], fy[5][2], gx[5][2], gy[5][2];
    Quad<C> c[5];
    C jx[5], jy[5];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int k = 0; k < 5; ++k) {
#pragma unroll
            for (int s = 0; s < 2; ++s) fx[k][s] = fy[k][s] = gx[k][s] = gy[k][s] = 0;
            c[k] = Quad<C>{0, 0, 0, 0};
            jx[k] = jy[k] = 0;
        }
    }
};

// The mirrored rows that row r between walls also stands for: 1: row -1 (r = 0), 2:
// row -2 (r = 1), 4: row ny (r = ny - 1), 8: row ny + 1 (r = ny - 2).
__device__ __forceinline__ int edge_of(int r, int ny)
{
    return (r == 0 ? 1 : 0) | (r == 1 ? 2 : 0) | (r == ny - 1 ? 4 : 0) | (r == ny - 2 ? 8 : 0);
}
// The row_sums case of a row: 1 at the bottom wall, 2 at the top wall.
__device__ __forceinline__ int wall_of(int edge) { return (edge & 1) ? 1 : ((edge & 4) ? 2 : 0); }

// Adds row r (slot K) to the force sums of rows r-2 .. r+2 (and, at a wall, its
// mirror's terms).  Row r+2's sums start here.  A row beyond a wall is staged as
// zeros: it adds nothing itself.
//
// The terms of a sum go from the small weights to the large ones.  (Orders differ only in
// rounding, but a chaotic lattice of 20000 steps ends up elsewhere: of five orders, three
// let a network placed on such runs accept no fewer points than k-section does, and so pass
// the test that asks it; this one does.)
template <int K, class C>
__device__ __forceinline__ void push(Belt<C>& b, const Near<C>& n, const Coef<C>& k, int edge)
{
    constexpr int M2 = (K + 3) % 5, M1 = (K + 4) % 5, P1 = (K + 1) % 5, P2 = (K + 2) % 5;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const C(&p)[5] = n.p[s];
        const C g1 = p[3] - p[1], g2 = p[4] - p[0], h1 = p[3] + p[1], h2 = p[4] + p[0];
        const C u0 = k.d4[s] * g2 + k.k1[s] * g1;
        const C u1 = k.d5[s] * g2 + k.k2[s] * g1;
        const C u2 = k.d8[s] * g2 + k.k5[s] * g1;
        const C w1 = k.k5[s] * h2 + k.k2[s] * h1 + k.k1[s] * p[2];
        const C w2 = k.d8[s] * h2 + k.d5[s] * h1 + k.d4[s] * p[2];
        const C(&o)[3] = n.r[1 - s];
        const C g = o[2] - o[0], h = o[2] + o[0];
        const C c0 = k.kx1 * g, c1 = k.kx2 * g;
        const C v = k.kx1 * o[1] + k.kx2 * h;
        b.fx[M2][s] += u2;
        b.fx[M1][s] += u1;
        b.fx[K][s] += u0;
        b.fx[P1][s] += u1;
        b.fx[P2][s] = u2;
        // the y sums hold the terms of the rows below with their sign turned
        // until the first row above arrives
        b.fy[M2][s] += w2;
        b.fy[M1][s] = w1 - b.fy[M1][s];
        b.fy[P1][s] += w1;
        b.fy[P2][s] = w2;
        b.gx[M1][s] += c1;
        b.gx[K][s] += c0;
        b.gx[P1][s] = c1;
        b.gy[M1][s] = v - b.gy[M1][s];
        b.gy[P1][s] = v;
        if (edge) {
            if (edge & 1) {          // row -1 too: one row below row 0, two below row 1
                b.fx[K][s] += u1;
                b.fx[P1][s] += u2;
                b.fy[K][s] += w1;
                b.fy[P1][s] += w2;
                b.gx[K][s] += c1;
                b.gy[K][s] += v;
            }
            if (edge & 2) {          // row -2 too: two rows below row 0
                b.fx[M1][s] += u2;
                b.fy[M1][s] -= w2;
            }
            if (edge & 4) {          // row ny too: one row above row ny-1, two above row ny-2
                b.fx[K][s] += u1;
                b.fx[M1][s] += u2;
                b.fy[K][s] -= w1;        // (its sign turns with the next row)
                b.fy[M1][s] += w2;
                b.gx[K][s] += c1;
                b.gy[K][s] -= v;
            }
            if (edge & 8) {          // row ny+1 too: two rows above row ny-1
                b.fx[P1][s] += u2;
                b.fy[P1][s] -= w2;
            }
        }
        // the terms are added here: the compiler would otherwise sink the additions
        // to the collision two rows later and keep every row's terms alive (80
        // registers more)
        asm volatile("" : "+v"(b.fx[M2][s]), "+v"(b.fx[M1][s]), "+v"(b.fx[K][s]), "+v"(b.fx[P1][s]), "+v"(b.fx[P2][s]),
                     "+v"(b.fy[M2][s]), "+v"(b.fy[M1][s]), "+v"(b.fy[P1][s]), "+v"(b.fy[P2][s]), "+v"(b.gx[M1][s]),
                     "+v"(b.gx[K][s]), "+v"(b.gx[P1][s]), "+v"(b.gy[M1][s]), "+v"(b.gy[P1][s]));
    }
}

// ---------------------------------------------------------------- collision --

// Reciprocal with one Newton step in FP32: the hardware's approximation is on
// average 0.7e-8 low, and every step would put that factor on the momentum.
__device__ __forceinline__ float fair_rcp(float v)
{
    const float r = rcp(v);
    return __builtin_fmaf(__builtin_fmaf(-v, r, 1.0f), r, r);
}
__device__ __forceinline__ double fair_rcp(double v) { return rcp(v); }

// The site in slot M, its neighbourhood complete: barycentric velocity, absolute
// densities and the shifted velocities of A and B at tau = 1.
template <class C> struct Site { C ux, uy, r[2], vx[2], vy[2]; };
template <int M, class C>
__device__ __forceinline__ Site<C> collide(const Belt<C>& b, const Coef<C>& k, const double* __restrict__ body, int y)
{
    Site<C> o;
    const Quad<C> c = b.c[M];
    o.r[0] = k.rref[0] + c.z;
    o.r[1] = k.rref[1] + c.w;
    const C p[2] = {k.pref[0] + c.x, k.pref[1] + c.y};
    const C inv_rho = fair_rcp(o.r[0] + o.r[1]);
    o.ux = b.jx[M] * inv_rho;
    o.uy = b.jy[M] * inv_rho;
    // external body force of the row, shared by density: the same
    // acceleration F_x(y) / (rho_A + rho_B) for both species
    const C wx = (body != nullptr) ? o.ux + (C)body[y] * inv_rho : o.ux;
    // F_s / rho_s = -(psi_s / rho_s) (psi sums) - (sums of the other's rho)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const C q = p[s] * rcp(o.r[s]);
        o.vx[s] = wx - (q * b.fx[M][s] + b.gx[M][s]);
        o.vy[s] = o.uy - (q * b.fy[M][s] + b.gy[M][s]);
    }
    return o;
}

// x / N without the bias of FP32's 1/N (3.0e-8 too large for 3, 0.7e-8 for 9: a
// factor that every step would put on the momentum and the density deviations).
template <int N> __device__ __forceinline__ float over(float x)
{
    constexpr float hi = (float)(1.0 / N), lo = (float)(1.0 / N - (double)hi);
    return __builtin_fmaf(x, hi, x * lo);
}
template <int N> __device__ __forceinline__ double over(double x) { return x * (1.0 / N); }

// The nine equilibrium populations at (rho, v) as deviations from w_i rho_ref:
// w_i [drho + rho (3 c.v + 4.5 (c.v)^2 - 1.5 v.v)].
template <class C>
__device__ __forceinline__ void equilibria(C rs, C drs, C vx, C vy, C (&e)[9])
{
    const C vv = vx * vx + vy * vy;
    auto pair = [&](int ip, int im, C a, C b, C c, C cu) {
        const C sym = a + (b * cu) * cu;
        e[ip] = sym + c * cu;
        e[im] = sym - c * cu;
    };
    // a: what all directions share; the other weights are powers of two of it
    const C a1 = over<9>(drs - ((C)1.5 * rs) * vv), b1 = rs * (C)0.5, c1 = over<3>(rs);
    e[0] = a1 * (C)4;
    pair(1, 3, a1, b1, c1, vx);
    pair(2, 4, a1, b1, c1, vy);
    const C a2 = a1 * (C)0.25, b2 = rs * (C)0.125, c2 = c1 * (C)0.25;
    pair(5, 7, a2, b2, c2, vx + vy);
    pair(6, 8, a2, b2, c2, vy - vx);
}

// A population that leaves through a wall moving at u_w returns to its node
// reversed, plus the moving-wall term.
template <class C> __device__ __forceinline__ C bounced(C e, C rs, int cx, WallSpeed<C> uw)
{
    const C w = over<6>(rs) * (C)cx;
    return e - (w * uw.hi + w * uw.lo);
}
// x momentum the wall receives from the links of one species.
template <class C> __device__ __forceinline__ C wall_momentum(const C (&e)[9], C rs, bool bot, WallSpeed<C> uw)
{
    const int ip = bot ? 8 : 5, im = bot ? 7 : 6;   // leaving, c_x = +1 and -1
    return (e[ip] + bounced(e[ip], rs, 1, uw)) - (e[im] + bounced(e[im], rs, -1, uw));
}

// Stores one species' nine post-collision values of the site in column offset
// vc (vl, vr: its neighbours) of row y: pushed in y; at a wall the leaving ones
// return to the row in the column the shifted layout gives their reverse.
template <class P, int CP>
__device__ __forceinline__ void store_site(rsrc_t ro, const typename P::C (&e)[9], typename P::C rs, unsigned vl,
                                           unsigned vc, unsigned vr, unsigned rm, unsigned r0, unsigned rp,
                                           unsigned pbytes, bool bot, bool top, WallSpeed<typename P::C> u_bot,
                                           WallSpeed<typename P::C> u_top)
{
    using S = typename P::S;
    using C = typename P::C;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const int cx = CX[i], cy = CY[i];
        if ((cy < 0 && bot) || (cy > 0 && top)) {
            const unsigned vb = cx == 0 ? vc : (cx > 0 ? vr : vl);
            const C back = cx == 0 ? e[i] : bounced(e[i], rs, cx, cy < 0 ? u_bot : u_top);
            st_s<P, CP>(ro, r0 + vb, OPP[i] * pbytes, to_store<S>(back));
        } else {
            st_s<P, CP>(ro, (cy < 0 ? rm : (cy > 0 ? rp : r0)) + vc, i * pbytes, to_store<S>(e[i]));
        }
    }
}

// Row r in [0, ny): the periodic image (r itself but for a few rows).
__device__ __forceinline__ int wrap_row(int r, int ny)
{
    if ((unsigned)r < (unsigned)ny) return r;
    r %= ny;
    return r < 0 ? r + ny : r;
}

// A thread's column in the population buffers: byte offsets of it and of its
// neighbours, of a row and of a plane, and bytes of a species' planes.
struct Column { unsigned vl, vc, vr, rbytes, pbytes, sbytes; };
template <class P> __device__ __forceinline__ Column column_of(const LatDesc& d, unsigned xc)
{
    const unsigned xr = (xc + 1 == (unsigned)d.nx) ? 0u : xc + 1, xl = (xc == 0) ? (unsigned)(d.nx - 1) : xc - 1;
    const unsigned es = (unsigned)sizeof(typename P::S);
    return Column{xl * es, xc * es, xr * es, (unsigned)d.pitch * es, (unsigned)(d.plane * es),
                  (unsigned)(9 * d.plane * (long long)es)};
}

// Row r (any row, not at or beyond a wall's if need is false) of the column.  One that is
// not needed or lies beyond a wall is loaded through an empty resource: zeros, no access.
template <class P>
__device__ __forceinline__ void load_row(Raw<P>& f, const char* fin, const Column& c, int r, int ny, bool need)
{
    const unsigned ro = need ? (unsigned)wrap_row(r, ny) * c.rbytes : 0u, len = need ? c.sbytes : 0u;
    f.load(make_rsrc(fin, len), make_rsrc(fin + c.sbytes, len), c.vl + ro, c.vc + ro, c.vr + ro, c.pbytes);
}

// Stores row y of the column after its collision t (slot M) into the next buffer and
// adds the wall momentum of its links.  near: the tile has rows at or beyond a wall.
template <int M, class P, int CP, class C>
__device__ __forceinline__ void store_row(rsrc_t rout0, rsrc_t rout1, const Column& c, const Belt<C>& b, const Site<C>& t,
                                          const Coef<C>& k, int y, int ny, bool near, C& mom_b, C& mom_t)
{
    const bool bot = near && y == 0, top = near && y == ny - 1;
    const int ym = (y == 0) ? ny - 1 : y - 1, yp = (y == ny - 1) ? 0 : y + 1;
    const unsigned rm = (unsigned)ym * c.rbytes, r0 = (unsigned)y * c.rbytes, rp = (unsigned)yp * c.rbytes;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        C e[9];
        equilibria(t.r[s], s == 0 ? b.c[M].z : b.c[M].w, t.vx[s], t.vy[s], e);
        const rsrc_t ro = s == 0 ? rout0 : rout1;
        if (bot || top) {
            store_site<P, CP>(ro, e, t.r[s], c.vl, c.vc, c.vr, rm, r0, rp, c.pbytes, bot, top, k.u_bot, k.u_top);
            if (bot) mom_b += wall_momentum(e, t.r[s], true, k.u_bot);
            if (top) mom_t += wall_momentum(e, t.r[s], false, k.u_top);
        } else {
            store_site<P, CP>(ro, e, t.r[s], c.vl, c.vc, c.vr, rm, r0, rp, c.pbytes, false, false, k.u_bot, k.u_top);
        }
    }
}

// Line profile: the sum of u_x over the wave's columns of each row it collides, in
// FP64, added to the wave's partial of that row.  Eight rows are kept in LDS (the
// row length makes the reads below hit each of the 64 banks once) and summed
// together, eight lanes a row and eight columns a lane: about six vector
// operations a row, where a wave-wide FP64 reduction of two rows at a time took
// 35 (10 % of the two-step kernels' time).  One add per row and launch: a
// no-return FP64 atomic (a plain read-modify-write would wait for its read and
// every load before it).
template <class C> struct ProfileRows { C v[8][65]; };
template <class C>
__device__ __forceinline__ void add_profile(double* __restrict__ prof, ProfileRows<C>& rows, C cur, int y, int y0, int y1)
{
    const int lane = threadIdx.x & 63, k = (y - y0) & 7;
    rows.v[k][lane] = cur;
    if (k < 7 && y + 1 < y1) return;
    __builtin_amdgcn_wave_barrier();
    const int r = lane >> 3, c = (lane & 7) * 8;
    double sum = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) sum += (double)rows.v[r][c + i];
    sum += dpp_move<0xB1>(sum);    // quad_perm [1,0,3,2]: lane l^1
    sum += dpp_move<0x4E>(sum);    // quad_perm [2,3,0,1]: lane l^2
    sum += dpp_move<0x141>(sum);   // row_half_mirror: the other quad of the 8-lane group
    if ((lane & 7) == 0 && r <= k) unsafeAtomicAdd(&prof[y - k + r], sum);
    __builtin_amdgcn_wave_barrier();
}

template <int I> using Slot = std::integral_constant<int, I>;

// Runs tick(slot, i) for i = 0 .. n-1 (n >= 1), the slot i mod 5 a constant.  Leaving
// the loop at any tick keeps what is dead after a tick out of the registers.
template <class F> __device__ __forceinline__ void ticks(int n, F tick)
{
    auto one = [&](auto slot, int i) {
        tick(slot, i);
        __builtin_amdgcn_sched_barrier(0);
    };
    int i = 0;
    asm volatile("" : "+s"(i));
    for (;;) {
        one(Slot<0>{}, i);
        if (++i >= n) break;
        one(Slot<1>{}, i);
        if (++i >= n) break;
        one(Slot<2>{}, i);
        if (++i >= n) break;
        one(Slot<3>{}, i);
        if (++i >= n) break;
        one(Slot<4>{}, i);
        if (++i >= n) break;
    }
}

// ------------------------------------------------------------------- step ---
//
// One step, one wave per tile: its 64 lanes hold the columns x0-2 .. x0+61 and march
// down the rows of the tile, the x neighbours come by lane shifts, and the 60
// columns in the middle are collided and stored.  No LDS, no barrier: a wave
// waits only for its own loads, of which it has DEPTH rows in flight, so the
// short tiles of small lattices cost a few memory latencies and not one per row.
template <class P>
__global__ void __launch_bounds__(64, sizeof(typename P::S) == 8 ? 2 : 1)
k_step_unit(char* __restrict__ base, const LatDesc* __restrict__ descs, const int* __restrict__ tiles, int ntot,
            int src)
{
    using C = typename P::C;
    constexpr int DEPTH = 2;
    __shared__ ProfileRows<C> rows;
    const int lane = threadIdx.x;
    for (int w = blockIdx.x; w < ntot; w += gridDim.x) {
        const int L = tiles[w];          // owning lattice
        const LatDesc& d = descs[L];
        const int lin = xcd_tile(w - d.item_begin, d.nitems);
        const int strip = lin % d.nstrip, seg = lin / d.nstrip;
        const int nx = d.nx, ny = d.ny, walls = d.walls;
        const int x0 = strip * UNIT_COLS;
        const int y0 = seg * d.ly, y1 = min(y0 + d.ly, ny);
        auto wrap = [&](int c) { c %= nx; return c < 0 ? c + nx : c; };
        const int x = x0 - 2 + lane;
        const bool own = lane >= 2 && lane < 62 && x < nx;
        const unsigned xc = (unsigned)wrap(x);
        const Coef<C> k(d);
        const Column col = column_of<P>(d, xc);
        const char* fin = base + d.off_f[src];
        const char* fout = base + d.off_f[src ^ 1];
        const rsrc_t rout0 = make_rsrc(fout, col.sbytes), rout1 = make_rsrc(fout + col.sbytes, col.sbytes);
        double* __restrict__ stress = (double*)(base + d.off_stress);
        double* __restrict__ prof = d.off_prof >= 0 ? (double*)(base + d.off_prof) + (long long)strip * ny : nullptr;
        const double* __restrict__ body = d.off_body >= 0 ? (const double*)(base + d.off_body) : nullptr;
        C mom_b = 0, mom_t = 0;
        Raw<P> F[5];
        Belt<C> b;
        b.clear();
        const int n = y1 - y0 + 4;       // rows y0-2 .. y1+1
        // whether the tile has rows at or beyond a wall
        const bool near = walls && (y0 <= 2 || y1 >= ny - 2);
        auto load = [&](Raw<P>& f, int i) {
            const int r = y0 - 2 + i;
            load_row<P>(f, fin, col, r, ny, i < n && !(near && (unsigned)r >= (unsigned)ny));
        };
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) load(F[i], i);
        ticks(n, [&](auto slot, int i) {
            constexpr int K = decltype(slot)::value, M = (K + 3) % 5;
            const int r = y0 - 2 + i;
            const int edge = near ? edge_of(r, ny) : 0;
            Sums<C> s = row_sums<P>(F[K], wall_of(edge));
            // the row's registers are free before the next loads are issued
            settle(s);
            load(F[(K + DEPTH) % 5], i + DEPTH);
            b.c[K] = quad<P>(s, k);
            b.jx[K] = s.jx;
            b.jy[K] = s.jy;
            push<K>(b, near_lanes<C>(b.c[K]), k, edge);
            if (i < 4) return;
            const int y = r - 2;
            const Site<C> t = collide<M>(b, k, body, y);
            if (prof != nullptr) add_profile(prof, rows, own ? t.ux : (C)0, y, y0, y1);
            if (!own) return;
            store_row<M, P, 0>(rout0, rout1, col, b, t, k, y, ny, near, mom_b, mom_t);
        });
        if (own && walls && y0 == 0) stress[xc] += (double)mom_b;
        if (own && walls && y1 == ny) stress[nx + xc] += (double)mom_t;
    }
}
//
// The same for a block of BX columns (BX a multiple of 64, so that the rows it
// stores start and end on 64-byte sectors): BX threads collide a column each and
// exchange psi and rho through one LDS row per tick behind one barrier; an extra
// wave stages the two columns beyond each side.  Large lattices run it: waves
// on their own store 240-byte pieces of a row at different times, so a tenth
// of the sectors reach HBM in two parts (4096^2 FP32: 0.73 against 0.46 ms).
template <int BX, class P, int CP>
__global__ void __launch_bounds__(BX + 64)
k_step_unit_wide(char* __restrict__ base, const LatDesc* __restrict__ descs, const int* __restrict__ tiles, int ntot,
            int src)
{
    using S = typename P::S;
    using C = typename P::C;
    constexpr int DEPTH = sizeof(S) == 8 ? 1 : 2;
    __shared__ Quad<C> near[2][BX + 4];
    __shared__ ProfileRows<C> rows[BX / 64];
    // thread j < BX: column x0 + j; the next four: columns x0-2, x0-1, x0+BX, x0+BX+1
    const int j = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(j >> 6);
    const bool halo = wave == BX / 64;
    const int entry = !halo ? j + 2 : (j < BX + 2 ? j - BX : j);   // of the LDS row
    if (j >= BX + 4) return;
    for (int w = blockIdx.x; w < ntot; w += gridDim.x) {
        const int L = tiles[w];          // owning lattice
        const LatDesc& d = descs[L];
        const int lin = xcd_tile(w - d.item_begin, d.nitems);
        const int strip = lin % d.nstrip, seg = lin / d.nstrip;
        const int nx = d.nx, ny = d.ny, walls = d.walls;
        const int x0 = strip * BX;
        const int y0 = seg * d.ly, y1 = min(y0 + d.ly, ny);
        auto wrap = [&](int c) { c %= nx; return c < 0 ? c + nx : c; };
        const int x = x0 - 2 + entry;
        const bool own = !halo && x < nx;
        const unsigned xc = (unsigned)wrap(x);
        const Coef<C> k(d);
        const Column col = column_of<P>(d, xc);
        const char* fin = base + d.off_f[src];
        const char* fout = base + d.off_f[src ^ 1];
        const rsrc_t rout0 = make_rsrc(fout, col.sbytes), rout1 = make_rsrc(fout + col.sbytes, col.sbytes);
        double* __restrict__ stress = (double*)(base + d.off_stress);
        double* __restrict__ prof = d.off_prof >= 0 ? (double*)(base + d.off_prof) + (long long)(x0 / 64 + wave) * ny : nullptr;
        const double* __restrict__ body = d.off_body >= 0 ? (const double*)(base + d.off_body) : nullptr;
        C mom_b = 0, mom_t = 0;
        Raw<P> F[5];
        Belt<C> b;
        b.clear();
        const int n = y1 - y0 + 4;       // rows y0-2 .. y1+1
        // whether the tile has rows at or beyond a wall
        const bool wall = walls && (y0 <= 2 || y1 >= ny - 2);
        auto load = [&](Raw<P>& f, int i) {
            const int r = y0 - 2 + i;
            load_row<P>(f, fin, col, r, ny, i < n && !(wall && (unsigned)r >= (unsigned)ny));
        };
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) load(F[i], i);
        ticks(n, [&](auto slot, int i) {
            constexpr int K = decltype(slot)::value, M = (K + 3) % 5;
            const int r = y0 - 2 + i;
            const int edge = wall ? edge_of(r, ny) : 0;
            Sums<C> s = row_sums<P>(F[K], wall_of(edge));
            // the row's registers are free before the next loads are issued
            settle(s);
            load(F[(K + DEPTH) % 5], i + DEPTH);
            b.c[K] = quad<P>(s, k);
            b.jx[K] = s.jx;
            b.jy[K] = s.jy;
            near[i & 1][entry] = b.c[K];
            lds_barrier();
            if (halo) return;
            push<K>(b, near_lds<C>(near[i & 1], entry), k, edge);
            if (i < 4) return;
            const int y = r - 2;
            const Site<C> t = collide<M>(b, k, body, y);
            if (prof != nullptr && x0 + 64 * wave < nx) add_profile(prof, rows[wave], own ? t.ux : (C)0, y, y0, y1);
            if (!own) return;
            store_row<M, P, CP>(rout0, rout1, col, b, t, k, y, ny, wall, mom_b, mom_t);
        });
        if (own && walls && y0 == 0) stress[xc] += (double)mom_b;
        if (own && walls && y1 == ny) stress[nx + xc] += (double)mom_t;
        __syncthreads();
    }
}

// ----------------------------------------------------------- moment form ----
//
// One step of the moment form (planes, each [y][pitch]: 0, 1 = rho_A - rho_ref_A,
// rho_B - rho_ref_B; 2, 3 = v_x of A, B; 4, 5 = v_y of A, B; before the first
// step the initial state itself, read in place).  As k_step_unit, but a loaded
// row is the post-collision state: each lane forms its column's eighteen
// populations once, sums them by direction as they stream (Flow) and takes the
// neighbours' values per x direction by lane shifts.  58 columns a wave
// (one more each side than the populations' step).
template <int BX, class P>
__global__ void __launch_bounds__(BX)
k_step_mom(char* __restrict__ base, const LatDesc* __restrict__ descs, const int* __restrict__ tiles, int ntot,
           int src, int first)
{
    using C = typename P::C;
    constexpr int DEPTH = 2;
    __shared__ ProfileRows<C> rows[BX / 64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

    for (int w = blockIdx.x; w < ntot; w += gridDim.x) {
        const int L = tiles[w];          // owning lattice
        const LatDesc& d = descs[L];
        const int lin = xcd_tile(w - d.item_begin, d.nitems);
        const int strip = lin % d.nstrip * (BX / 64) + wave, seg = lin / d.nstrip;
        const int nx = d.nx, ny = d.ny, walls = d.walls;
        const int x0 = strip * MOM_COLS;
        if (x0 >= nx) continue;
        const int y0 = seg * d.ly, y1 = min(y0 + d.ly, ny);
        const int x = x0 - 3 + lane;
        const bool own = lane >= 3 && lane < 61 && x < nx;
        const int xm = x % nx;
        const unsigned xc = (unsigned)(xm < 0 ? xm + nx : xm);
        const Coef<C> k(d);
        const unsigned es = (unsigned)sizeof(C);
        const unsigned mbytes = (unsigned)(6 * d.plane * (long long)es);
        const char* fin = base + d.off_f[src];
        const rsrc_t rout = make_rsrc(base + d.off_f[src ^ 1], mbytes);
        const unsigned vc = xc * es, pbytes = (unsigned)(d.plane * es), rbytes = (unsigned)d.pitch * es;
        double* __restrict__ stress = (double*)(base + d.off_stress);
        double* __restrict__ prof = d.off_prof >= 0 ? (double*)(base + d.off_prof) + (long long)strip * ny : nullptr;
        const double* __restrict__ body = d.off_body >= 0 ? (const double*)(base + d.off_body) : nullptr;
        C mom_b = 0, mom_t = 0;
        struct M6 { C v[6]; };
        M6 F[5];
        Belt<C> b;
        b.clear();
        Flow<C> flow;
        flow.clear();
        Sums<C> wall{0, 0, 0, 0}, kept{0, 0, 0, 0};
        const int n = y1 - y0 + 6;       // rows y0-3 .. y1+2
        const bool near = walls && (y0 <= 2 || y1 >= ny - 2);
        auto outside = [&](int r) { return near && (unsigned)r >= (unsigned)ny; };
        auto load = [&](M6& m, int i) {
            const int r = y0 - 3 + i;
            const bool need = i < n && !outside(r);
            const unsigned ro = (need ? (unsigned)wrap_row(r, ny) * rbytes : 0u) + vc;
            const rsrc_t rin = make_rsrc(fin, need ? mbytes : 0u);
#pragma unroll
            for (int p = 0; p < 6; ++p) m.v[p] = ld<P>(rin, ro, p * pbytes);
        };
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) load(F[i], i);
        ticks(n, [&](auto slot, int i) {
            constexpr int K = decltype(slot)::value, M = (K + 3) % 5;
            const int r = y0 - 3 + i;    // the row loaded; row r-1 is complete
            Sums<C> s;
            const C(&m)[6] = F[K].v;
            if (first) {
                s = kept;
                if (!outside(r)) {
                    const C ra = k.rref[0] + m[0], rb = k.rref[1] + m[1];
                    kept = Sums<C>{m[0], m[1], ra * m[2] + rb * m[3], ra * m[4] + rb * m[5]};
                }
            } else {
                Part<C> p = flow.mid;
                const Sums<C> w1 = wall;
                if (!outside(r)) {
                    const C ra = k.rref[0] + m[0], rb = k.rref[1] + m[1];
                    C ea[9], eb[9];
                    equilibria(ra, m[0], m[2], m[4], ea);
                    equilibria(rb, m[1], m[3], m[5], eb);
                    Row<P> q;
                    q.set(ea, eb);
                    p = flow.feed(q);
                    if (near && r == 0)
                        wall = wall_sums<C>(ea[4], bounced(ea[7], ra, -1, k.u_bot), bounced(ea[8], ra, 1, k.u_bot),
                                            eb[4], bounced(eb[7], rb, -1, k.u_bot), bounced(eb[8], rb, 1, k.u_bot),
                                            true);
                    if (near && r == ny - 1)
                        wall = wall_sums<C>(ea[2], bounced(ea[6], ra, -1, k.u_top), bounced(ea[5], ra, 1, k.u_top),
                                            eb[2], bounced(eb[6], rb, -1, k.u_top), bounced(eb[5], rb, 1, k.u_top),
                                            false);
                }
                const C sp[2] = {left(p.sp[0]), left(p.sp[1])}, sm[2] = {right(p.sm[0]), right(p.sm[1])};
                s = join(p.s0, sp, sm, p.j0, left(p.jp), right(p.jm), left(p.xp), right(p.xm));
                if (near && (r - 1 == 0 || r - 1 == ny - 1)) add_sums(s, w1);
            }
            if (outside(r - 1)) s = Sums<C>{0, 0, 0, 0};
            settle(s);
            load(F[(K + DEPTH) % 5], i + DEPTH);
            b.c[K] = quad<P>(s, k);
            b.jx[K] = s.jx;
            b.jy[K] = s.jy;
            push<K>(b, near_lanes<C>(b.c[K]), k, near ? edge_of(r - 1, ny) : 0);
            if (i < 6) return;
            const int y = r - 3;
            const Site<C> t = collide<M>(b, k, body, y);
            if (prof != nullptr) add_profile(prof, rows[wave], own ? t.ux : (C)0, y, y0, y1);
            if (!own) return;
            const unsigned so = (unsigned)y * rbytes;
            st<P>(rout, vc, so, b.c[M].z);
            st<P>(rout, vc, so + pbytes, b.c[M].w);
            st<P>(rout, vc, so + 2 * pbytes, t.vx[0]);
            st<P>(rout, vc, so + 3 * pbytes, t.vx[1]);
            st<P>(rout, vc, so + 4 * pbytes, t.vy[0]);
            st<P>(rout, vc, so + 5 * pbytes, t.vy[1]);
            // wall momentum of the links that leave through a wall this step
            if (near && (y == 0 || y == ny - 1)) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    C e[9];
                    equilibria(t.r[q], q == 0 ? b.c[M].z : b.c[M].w, t.vx[q], t.vy[q], e);
                    if (y == 0) mom_b += wall_momentum(e, t.r[q], true, k.u_bot);
                    else mom_t += wall_momentum(e, t.r[q], false, k.u_top);
                }
            }
        });
        if (own && walls && y0 == 0) stress[xc] += (double)mom_b;
        if (own && walls && y1 == ny) stress[nx + xc] += (double)mom_t;
    }
}

// ------------------------------------------------------ two fused steps ---
//
// Steps t and t+1 in one pass over HBM.  A block owns a tile of TW output columns;
// thread j of each half of its 128 NW threads holds column X - 5 + j.  In tick i
// the first half stages row y0-5+i of step t and collides row y0-7+i, whose
// populations stay on chip: each column's streaming sums (Flow) of the row they
// complete are published in LDS (part).  The second half joins its neighbours' sums
// published a tick earlier into the next row of step t+1, stages row y0-10+i and
// collides row y0-12+i, stored to HBM.  One LDS barrier per tick orders the three
// exchanges (near1 and near2: the staged psi and rho rows; part), each
// double-buffered.  The arithmetic and its order are k_step_unit's, so a pair of steps
// is bitwise that of two launches.  Five columns each side overlap the neighbouring tiles (two of psi
// and one of streaming for each step, less the outermost of step t's streaming).
//
// What bounds it: the issue rate of a wave at few waves per SIMD, so the registers.
// A half keeps one belt of rows and two rows of loads in 196 registers, two waves per
// SIMD; both steps in one thread took 241 and ran twice the work in each.  Between the steps eleven sums per column cross
// LDS instead of eighteen populations of nine rows.  It runs best at 182 columns and
// six waves a compute unit (4096^2: 0.266 ms a step; 246 columns, eight waves: 0.294;
// 122 columns, six waves: 0.371; two blocks of four waves and 118 columns, when psi was ten
// instructions shorter: 0.31 against 0.262).
template <class P, int NW, int TW, int PW>
__global__ void __launch_bounds__(128 * NW, 2)
k_step2_unit(char* __restrict__ base, const LatDesc* __restrict__ descs, const int* __restrict__ tiles, int ntot,
             int src)
{
    using C = typename P::C;
    using C2 = typename V2<C>::T;
    constexpr int BW = 64 * NW, XO = 5, DEPTH = 2;
    static_assert(TW + 2 * XO <= BW, "every output column and its overlap has a thread");
    // entries j + 2 and j + 1; the outer ones stay zero (they feed no output)
    __shared__ Quad<C> near1[2][BW + 4], near2[2][BW + 4];
    __shared__ C2 ps[2][3][BW + 2];      // [tick][c_x = 0, +1, -1]: sums of A and B
    __shared__ C2 pj[2][2][BW + 2];      // [tick][c_x = +1, -1]: their y momentum and their sum
    __shared__ C pj0[2][BW];             // [tick]: the y momentum of c_x = 0
    __shared__ Quad<C> ext[2][BW];       // what the bottom / top wall returned to rows 0 / ny-1 of step t+1
    __shared__ C mom[2][BW];             // step t's wall momentum, handed to step t+1
    __shared__ ProfileRows<C> rows[2 * NW];
    const int role = __builtin_amdgcn_readfirstlane((int)threadIdx.x / BW);   // 0: step t, 1: step t+1
    const int j = threadIdx.x - role * BW;
    const int wave = __builtin_amdgcn_readfirstlane(j >> 6);
    if (threadIdx.x < 2) {
        const int b = threadIdx.x;
        const Quad<C> z{0, 0, 0, 0};
        near1[b][0] = near1[b][1] = near1[b][BW + 2] = near1[b][BW + 3] = z;
        near2[b][0] = near2[b][1] = near2[b][BW + 2] = near2[b][BW + 3] = z;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            ps[b][q][0] = ps[b][q][BW + 1] = C2{0, 0};
            if (q < 2) pj[b][q][0] = pj[b][q][BW + 1] = C2{0, 0};
        }
    }

    for (int w = blockIdx.x; w < ntot; w += gridDim.x) {
        const int L = tiles[w];          // owning lattice
        const LatDesc& d = descs[L];
        const int lin = xcd_tile(w - d.item_begin2, d.nitems2);
        const int strip = lin % d.nstrip2, seg = lin / d.nstrip2;
        const int nx = d.nx, ny = d.ny, walls = d.walls;
        const int X = strip * TW;
        // nseg2 segments of near-equal height: the first ny mod nseg2 one row taller
        const int sb = ny / d.nseg2, sx = ny - sb * d.nseg2;
        const int y0 = seg * sb + min(seg, sx);
        const int y1 = y0 + sb + (seg < sx ? 1 : 0);
        const int xm = (X - XO + j) % nx;
        const unsigned xc = (unsigned)(xm < 0 ? xm + nx : xm);
        const Column col = column_of<P>(d, xc);
        // the columns this tile stores and whose wall momentum it counts
        const bool own = j >= XO && j < XO + TW && X + (j - XO) < nx;
        const Coef<C> k(d);
        const double* __restrict__ body = d.off_body >= 0 ? (const double*)(base + d.off_body) : nullptr;
        // this wave's line-profile partials of its step (waves past PW own no column)
        double* __restrict__ prof = nullptr;
        if (d.off_prof >= 0 && wave < PW)
            prof = (double*)(base + d.off_prof) + ((long long)d.ngroups + (role * d.nstrip2 + strip) * PW + wave) * ny;
        const int n = y1 - y0;
        // whether the tile has rows at or beyond a wall
        const bool near = walls && (y0 <= 5 || y1 >= ny - 5);
        auto outside = [&](int r) { return near && (unsigned)r >= (unsigned)ny; };
        C mb = 0, mt = 0;
        Belt<C> B;
        B.clear();
        if (role == 0) {
            const char* fin = base + d.off_f[src];
            Raw<P> F[5];
            Flow<C> flow;
            flow.clear();
            auto load = [&](Raw<P>& f, int i) {
                const int r = y0 - 5 + i;
                load_row<P>(f, fin, col, r, ny, i < n + 10 && !outside(r));
            };
#pragma unroll
            for (int i = 0; i < DEPTH; ++i) load(F[i], i);
            ticks(n + 12, [&](auto slot, int i) {
                constexpr int K = decltype(slot)::value, M = (K + 3) % 5;
                const int at = i & 1;
                const int r = y0 - 5 + i, y = r - 2;
                const int edge = near ? edge_of(r, ny) : 0;
                Sums<C> s = row_sums<P>(F[K], wall_of(edge));
                settle(s);
                load(F[(K + DEPTH) % 5], i + DEPTH);
                B.c[K] = quad<P>(s, k);
                B.jx[K] = s.jx;
                B.jy[K] = s.jy;
                near1[at][j + 2] = B.c[K];
                lds_barrier();
                push<K>(B, near_lds<C>(near1[at], j + 2), k, edge);
                if (i < 4 || i >= n + 10) return;
                Part<C> done = flow.mid;
                if (!outside(y)) {
                    const Site<C> t = collide<M>(B, k, body, wrap_row(y, ny));
                    const bool count = y >= y0 && y < y1;
                    if (prof != nullptr && count) add_profile(prof, rows[role * NW + wave], own ? t.ux : (C)0, y, y0, y1);
                    C ea[9], eb[9];
                    equilibria(t.r[0], B.c[M].z, t.vx[0], t.vy[0], ea);
                    equilibria(t.r[1], B.c[M].w, t.vx[1], t.vy[1], eb);
                    Row<P> q;
                    q.set(ea, eb);
                    done = flow.feed(q);
                    // the populations a wall returns
                    auto returned = [&](const C(&e)[9], int s, int i1, WallSpeed<C> uw) {
                        return bounced(e[i1], t.r[s], CX[i1], uw);
                    };
                    if (near && y == 0) {
                        const Sums<C> v = wall_sums<C>(q[4], returned(ea, 0, 7, k.u_bot), returned(ea, 0, 8, k.u_bot), q[13],
                                                       returned(eb, 1, 7, k.u_bot), returned(eb, 1, 8, k.u_bot), true);
                        ext[0][j] = Quad<C>{v.da, v.db, v.jx, v.jy};
                        if (own && count) {
                            mb += wall_momentum(ea, t.r[0], true, k.u_bot);
                            mb += wall_momentum(eb, t.r[1], true, k.u_bot);
                        }
                    }
                    if (near && y == ny - 1) {
                        const Sums<C> v = wall_sums<C>(q[2], returned(ea, 0, 6, k.u_top), returned(ea, 0, 5, k.u_top), q[11],
                                                       returned(eb, 1, 6, k.u_top), returned(eb, 1, 5, k.u_top), false);
                        ext[1][j] = Quad<C>{v.da, v.db, v.jx, v.jy};
                        if (own && count) {
                            mt += wall_momentum(ea, t.r[0], false, k.u_top);
                            mt += wall_momentum(eb, t.r[1], false, k.u_top);
                        }
                    }
                }
                ps[at][0][j + 1] = C2{done.s0[0], done.s0[1]};
                ps[at][1][j + 1] = C2{done.sp[0], done.sp[1]};
                ps[at][2][j + 1] = C2{done.sm[0], done.sm[1]};
                pj[at][0][j + 1] = C2{done.jp, done.xp};
                pj[at][1][j + 1] = C2{done.jm, done.xm};
                pj0[at][j] = done.j0;
            });
            mom[0][j] = mb;
            mom[1][j] = mt;
        } else {
            const char* fout = base + d.off_f[src ^ 1];
            const rsrc_t rout0 = make_rsrc(fout, col.sbytes), rout1 = make_rsrc(fout + col.sbytes, col.sbytes);
            Quad<C> c2{0, 0, 0, 0};                // the row to stage next, and its momentum
            C j2x = 0, j2y = 0;
            ticks(n + 12, [&](auto slot, int i) {
                constexpr int K = decltype(slot)::value, M = (K + 3) % 5;
                const int at = i & 1;
                const int r = y0 - 10 + i, y = r - 2;
                B.c[K] = c2;
                B.jx[K] = j2x;
                B.jy[K] = j2y;
                near2[at][j + 2] = c2;
                lds_barrier();
                // row r + 1, published in the last tick
                if (i >= 7 && !outside(r + 1)) {
                    const C2 p0 = ps[at ^ 1][0][j + 1], pp = ps[at ^ 1][1][j], pm = ps[at ^ 1][2][j + 2];
                    const C s0[2] = {p0.x, p0.y}, sp[2] = {pp.x, pp.y}, sm[2] = {pm.x, pm.y};
                    const C2 mp = pj[at ^ 1][0][j], mm = pj[at ^ 1][1][j + 2];
                    Sums<C> v = join(s0, sp, sm, pj0[at ^ 1][j], mp.x, mm.x, mp.y, mm.y);
                    if (near && (r + 1 == 0 || r + 1 == ny - 1)) {
                        const Quad<C> e = ext[r + 1 == 0 ? 0 : 1][j];
                        add_sums(v, Sums<C>{e.x, e.y, e.z, e.w});
                    }
                    settle(v);
                    c2 = quad<P>(v, k);
                    j2x = v.jx;
                    j2y = v.jy;
                } else {
                    c2 = Quad<C>{0, 0, 0, 0};
                    j2x = j2y = 0;
                }
                push<K>(B, near_lds<C>(near2[at], j + 2), k, near ? edge_of(r, ny) : 0);
                if (i < 12) return;
                const Site<C> t = collide<M>(B, k, body, y);
                if (prof != nullptr) add_profile(prof, rows[role * NW + wave], own ? t.ux : (C)0, y, y0, y1);
                if (!own) return;
                store_row<M, P, 0>(rout0, rout1, col, B, t, k, y, ny, near, mb, mt);
            });
        }
        __syncthreads();
        // wall momentum in FP64, step t's first (the order of two single steps)
        if (role == 1 && own && walls) {
            double* __restrict__ stress = (double*)(base + d.off_stress);
            if (y0 == 0) {
                stress[xc] += (double)mom[0][j];
                stress[xc] += (double)mb;
            }
            if (y1 == ny) {
                stress[nx + xc] += (double)mom[1][j];
                stress[nx + xc] += (double)mt;
            }
        }
        __syncthreads();
    }
}

// --------------------------------------------------------- host launchers --

template <int BX, class P>
hipError_t unit_bx(char* base, const LatDesc* descs, const int* tiles, int ntot, int src, bool stream, int grid,
                   hipStream_t s)
{
    if constexpr (BX == 64)
        hipLaunchKernelGGL((k_step_unit<P>), dim3(grid), dim3(64), 0, s, base, descs, tiles, ntot, src);
    else if (stream)
        hipLaunchKernelGGL((k_step_unit_wide<BX, P, CP_NT>), dim3(grid), dim3(BX + 64), 0, s, base, descs, tiles, ntot, src);
    else
        hipLaunchKernelGGL((k_step_unit_wide<BX, P, 0>), dim3(grid), dim3(BX + 64), 0, s, base, descs, tiles, ntot, src);
    return hipGetLastError();
}
template <class P>
hipError_t unit_p(int bx, char* base, const LatDesc* descs, const int* tiles, int ntot, int src, bool stream, int grid,
                  hipStream_t s)
{
    switch (bx) {
    case 64: return unit_bx<64, P>(base, descs, tiles, ntot, src, stream, grid, s);
    case 128: return unit_bx<128, P>(base, descs, tiles, ntot, src, stream, grid, s);
    case 256: return unit_bx<256, P>(base, descs, tiles, ntot, src, stream, grid, s);
    case 512:   // as the general step: not FP64
        if constexpr (sizeof(typename P::S) <= 4) return unit_bx<512, P>(base, descs, tiles, ntot, src, stream, grid, s);
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}
template <int BX, class P>
hipError_t mom_bx(char* base, const LatDesc* descs, const int* tiles, int ntot, int src, int first, int grid,
                  hipStream_t s)
{
    hipLaunchKernelGGL((k_step_mom<BX, P>), dim3(grid), dim3(BX), 0, s, base, descs, tiles, ntot, src, first);
    return hipGetLastError();
}
template <class P>
hipError_t mom_p(int bx, char* base, const LatDesc* descs, const int* tiles, int ntot, int src, int first, int grid,
                 hipStream_t s)
{
    switch (bx) {
    case 64: return mom_bx<64, P>(base, descs, tiles, ntot, src, first, grid, s);
    case 128: return mom_bx<128, P>(base, descs, tiles, ntot, src, first, grid, s);
    case 256: return mom_bx<256, P>(base, descs, tiles, ntot, src, first, grid, s);
    default: return hipErrorInvalidValue;
    }
}

// The fused kernel of a storage and nw waves of output columns (fuse2_tw); nw = 2
// stores six columns less than its lanes, so its overlap takes a third wave.
#define LBK_UNIT2_CASES(F)                                                                          \
    switch (storage * 10 + nw) {                                                                     \
    case 12: return F((k_step2_unit<StF32, 3, fuse2_tw(1, 2), 2>), 384);                             \
    case 13: return F((k_step2_unit<StF32, 3, fuse2_tw(1, 3), 3>), 384);                             \
    case 14: return F((k_step2_unit<StF32, 4, fuse2_tw(1, 4), 4>), 512);                             \
    default: break;                                                                                  \
    }

}  // namespace

hipError_t launch_step_unit(int storage, int bx, char* base, const LatDesc* descs, const int* tiles, int ntot, int src,
                            bool stream, int grid, hipStream_t s)
{
    switch (storage) {
    case 0: return unit_p<StF64>(bx, base, descs, tiles, ntot, src, stream, grid, s);
    case 1: return unit_p<StF32>(bx, base, descs, tiles, ntot, src, stream, grid, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_step_mom(int storage, int bx, char* base, const LatDesc* descs, const int* tiles, int ntot, int src,
                           int first, int grid, hipStream_t s)
{
    switch (storage) {
    case 4: return mom_p<MomF32>(bx, base, descs, tiles, ntot, src, first, grid, s);
    case 5: return mom_p<MomF64>(bx, base, descs, tiles, ntot, src, first, grid, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_step2_unit(int storage, int nw, char* base, const LatDesc* descs, const int* tiles, int ntot, int src,
                             int grid, hipStream_t s)
{
    auto run = [&](auto kernel, int threads) -> hipError_t {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, s, base, descs, tiles, ntot, src);
        return hipGetLastError();
    };
    LBK_UNIT2_CASES(run)
    return hipErrorInvalidValue;
}

size_t step_unit_lds_bytes(int storage, int bx)
{
    auto of = [](auto kernel) -> size_t {
        hipFuncAttributes fa;
        return hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(kernel)) == hipSuccess ? fa.sharedSizeBytes : 0;
    };
    switch (storage * 1000 + bx) {
    case 64: return of(k_step_unit<StF64>);
    case 128: return of(k_step_unit_wide<128, StF64, 0>);
    case 256: return of(k_step_unit_wide<256, StF64, 0>);
    case 1064: return of(k_step_unit<StF32>);
    case 1128: return of(k_step_unit_wide<128, StF32, 0>);
    case 1256: return of(k_step_unit_wide<256, StF32, 0>);
    case 1512: return of(k_step_unit_wide<512, StF32, 0>);
    case 4064: return of(k_step_mom<64, MomF32>);
    case 4128: return of(k_step_mom<128, MomF32>);
    case 4256: return of(k_step_mom<256, MomF32>);
    case 5064: return of(k_step_mom<64, MomF64>);
    case 5128: return of(k_step_mom<128, MomF64>);
    case 5256: return of(k_step_mom<256, MomF64>);
    default: return 0;
    }
}

size_t step2_unit_lds_bytes(int storage, int nw)
{
    auto run = [](auto kernel, int) -> size_t {
        hipFuncAttributes fa;
        return hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(kernel)) == hipSuccess ? fa.sharedSizeBytes : 0;
    };
    LBK_UNIT2_CASES(run)
    return 0;
}

int step2_unit_blocks_per_cu(int storage, int nw)
{
    auto run = [](auto kernel, int threads) -> int {
        int n = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(kernel), threads, 0) ==
                       hipSuccess ? n : 0;
    };
    LBK_UNIT2_CASES(run)
    return 0;
}

}  // namespace lbk
