// The update of one node (Section 3): zeroth moments of its scalar populations, flow
// moments and forces, and the collision of f, g, h^A, h^B (, h^C).  Shared by the kernels
// that march columns of nodes through memory and by the one that keeps a window of nodes
// on chip over several steps: the arithmetic of a step is the same in both.
#pragma once

#include "storage.hpp"

namespace lbm {

// index of the pair (k, opp(k)), k < opp(k), among the moving directions of lattice L
template <class L, int K>
constexpr int pair_index() {
    int n = 0;
    for (int j = 1; j < K; ++j)
        if (j < L::opp(j)) ++n;
    return n;
}

// MRT relaxation of one field (the multiple-relaxation-time alternative to BGK):
// n_k = X_k - eqs(k) to the moment basis, moment i times rate(i) / <M_i, M_i>, back
// with M^-1_{k i} = w_k M_ik / <M_i, M_i>, then out(k, X_k - w_k (M^T m)_k + src(k)).
template <class L>
inline constexpr MomentBasis<L::Q> kBasis = make_moment_basis<L>();

template <class L, class C, class EQ, class SRC, class RATE, class OUT>
__device__ __forceinline__ void mrt_relax(const C (&X)[L::Q], EQ&& eqs, SRC&& src, RATE&& rate, OUT&& out) {
    constexpr int Q = L::Q;
    C n[Q], m[Q];
    static_for<0, Q>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        n[k] = X[k] - eqs(kc);
    });
    static_for<0, Q>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        C a = C(0);
        static_for<0, Q>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            constexpr double mik = kBasis<L>.M[i][k];
            if constexpr (mik != 0.0) a += C(mik) * n[k];
        });
        m[i] = a * (rate(ic) * C(kBasis<L>.invD[i]));
    });
    static_for<0, Q>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        C a = C(0);
        static_for<0, Q>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            constexpr double mik = kBasis<L>.M[i][k];
            if constexpr (mik != 0.0) a += C(mik) * m[i];
        });
        out(kc, X[k] - C(L::w(k)) * a + src(kc));
    });
}

// order of row i of the basis, and whether it is the trace of the second order
template <class L, int I>
constexpr int basis_order() { return kBasis<L>.order[I]; }
template <class L, int I>
constexpr bool basis_trace() { return kBasis<L>.order[I] == 2 && (I == 0 || kBasis<L>.order[I - 1] != 2); }

template <class SL, class FL, int PREC, int COLL = COLL_BGK, int NC = 2>
struct Node {
    using C = typename Stor<PREC>::C;
    using SLOTS = Slots<FL::Q, SL::Q, NC>;
    using STL = typename std::conditional<SL::DIM == 2, D2Q9K, D3Q19K>::type;  // lattice of the phi stencil
    using SLT = std::common_type<SL>;  // type tags of the lattices
    using FLT = std::common_type<FL>;
    static constexpr int QS = SL::Q, QF = FL::Q, QFN = QF > 0 ? QF : 1;
    static constexpr int G0 = SLOTS::G0, A0 = SLOTS::A0, B0 = SLOTS::B0, HC0 = SLOTS::C0;
    static constexpr bool FLOW = QF > 0;
    static constexpr bool NC3 = NC == 3;
    static constexpr int QC = NC3 ? QS : 1;
    static constexpr bool TRTC = (COLL & COLL_TRT) != 0;
    static constexpr bool MRTC = (COLL & COLL_MRT) != 0;
    static constexpr bool VD = FLOW && (COLL & COLL_VD) != 0;
    static constexpr bool GK = (COLL & COLL_GK) != 0;
    static constexpr bool S16 = PREC == P16 || PREC == PB16;
    // 16-bit reference w_k ref_field of slot S (direction k of lattice L): zero for the
    // compositions (their moving equilibria w_k mu are near zero) and for f in BF16 (its
    // deviations need no scale, and f ~ w_k p_h is centred on zero)
    static constexpr bool NOREF_F = PREC == PB16;

    template <class S_, class K_, class LT>
    static __device__ __forceinline__ float wref(const KParams& P, S_, K_, LT) {
        using L = typename LT::type;
        constexpr int F = SLOTS::field(S_::value);
        if constexpr (F >= 2 || (F == 0 && NOREF_F)) return 0.0f;
        else return float(L::w(K_::value)) * P.fref[F];
    }
    // the reference a decode adds: a zero reference as -0.0, since x + (-0.0) = x folds away
    // (x + 0.0 does not: it maps -0.0 to +0.0) and the encode's x - 0.0 folds as well
    template <class S_, class K_, class LT>
    static __device__ __forceinline__ float wref_dec(const KParams& P, S_ s_, K_ k_, LT lat_) {
        constexpr int F = SLOTS::field(S_::value);
        if constexpr (F >= 2 || (F == 0 && NOREF_F)) return -0.0f;
        else return wref(P, s_, k_, lat_);
    }
    // a model constant in the compute type (the FP32 copy for FP32 arithmetic)
    static __device__ __forceinline__ C KC(double d, float f) {
        if constexpr (std::is_same<C, float>::value) return f;
        else return C(d);
    }
    // The kernels that update nodes must round alike (a state does not depend on how its
    // steps were cut into calls), but the compiler contracts a * b + c * d by use counts,
    // which differ between kernels.  In FP64, where nothing separates the closure from the
    // collision, sums of two products are therefore written with their fused operation,
    // and a product that several sums share is pinned (an empty asm, no instruction).  In
    // FP32 the conversions from the FP64 closure separate them: every expression but the
    // rest population of g contracts alike as written (tested bit for bit).
    static __device__ __forceinline__ C sum2(C x, C y, C z, C w) {  // x y + z w
        if constexpr (PREC == P64) return __builtin_fma(x, y, z * w);
        else return x * y + z * w;
    }
    static __device__ __forceinline__ C diff2(C x, C y, C z, C w) {  // x y - z w
        if constexpr (PREC == P64) return __builtin_fma(x, y, -(z * w));
        else return x * y - z * w;
    }
    static __device__ __forceinline__ C dot3(const C (&v)[3], const C (&w)[3]) {
        if constexpr (PREC == P64) return __builtin_fma(v[2], w[2], __builtin_fma(v[1], w[1], v[0] * w[0]));
        else return v[0] * w[0] + v[1] * w[1] + v[2] * w[2];
    }
    // e_k . (hs F) with Fh = hs F.  Variable density in 3D: fused by hand as in `flow`
    template <int ex, int ey, int ez>
    static __device__ __forceinline__ C edot_scaled(C hs, const C (&F)[3], const C (&Fh)[3]) {
        if constexpr (VD && SL::DIM == 3 && PREC != P64 && ex * ex + ey * ey + ez * ez == 2) {
            constexpr int i = ex != 0 ? 0 : 1, j = ez != 0 ? 2 : 1;
            constexpr int si = i == 0 ? ex : ey, sj = j == 2 ? ez : ey;
            return __builtin_elementwise_fma(si > 0 ? hs : -hs, F[i], sj > 0 ? Fh[j] : -Fh[j]);
        } else {
            return edot<ex, ey, ez>(Fh[0], Fh[1], Fh[2]);
        }
    }
    static __device__ __forceinline__ void pin1(C& x) { asm("" : "+v"(x)); }
    template <class... T>
    static __device__ __forceinline__ void pin(T&... x) {
        if constexpr (PREC == P64) (pin1(x), ...);
    }
    // a rounding residue of field F, from the encoded domain to values
    template <class F_>
    static __device__ __forceinline__ C fb(const KParams& P, F_, C res) {
        if constexpr (PREC == P16) return res * P.finv[F_::value];
        else return res;
    }
    // sum of the stored moving populations of field F on lattice L, from the sum of their
    // stored deviations: sum_{k != 0} w_k ref_F + dev 2^-s
    template <class F_, class LT>
    static __device__ __forceinline__ C stored_sum(const KParams& P, F_ f_, LT, C dev) {
        using L = typename LT::type;
        constexpr int F = F_::value;
        if constexpr (F >= 2 || (F == 0 && NOREF_F)) return fb(P, f_, dev);
        else return fb(P, f_, dev) + C(1.0 - L::w(0)) * P.fref[F];
    }
    // FP32 sum of the moving populations of one field, in the order k1, opp(k1), k2,
    // opp(k2), ... over k < opp(k) (16-bit storage; the packed LDS fill sums in this order)
    static __device__ __forceinline__ C moving_sum(const C (&x)[QS]) {
        C m = C(0);
        static_for<1, QS>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value, o = SL::opp(k);
            if constexpr (k < o) {
                if constexpr (pair_index<SL, k>() == 0) m = x[k] + x[o];
                else m = (m + x[k]) + x[o];
            }
        });
        return m;
    }
    static __device__ __forceinline__ void pop_sums(const C (&gg)[QS], const C (&aa)[QS], const C (&bb)[QS],
                                                    const C (&qq)[QC], double& phis, double& cA, double& cB,
                                                    double& cC) {
        // zeroth moments.  mu = c - c^eq(phi) cancels c ~ 0.3 down to ~1e-3, so FP32
        // partial sums over all populations (several roundings of c and phi each) would
        // enter mu with a relative error near 1e-4 per step: FP32 / FP64 storage sums in
        // FP64.  16-bit storage sums its moving populations in FP32 and adds the FP32
        // rest population in FP64: the moving h are ~w_k mu (their FP32 sum is near
        // exact) and the moving g carry 16-bit storage noise far above FP32 rounding
        if constexpr (S16) {
            phis = double(gg[0]) + double(moving_sum(gg));
            cA = double(aa[0]) + double(moving_sum(aa));
            cB = double(bb[0]) + double(moving_sum(bb));
            if constexpr (NC3) cC = double(qq[0]) + double(moving_sum(qq));
            else cC = 0.0;
        } else {
            double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
            for (int k = 0; k < QS; ++k) {
                s0 += double(gg[k]);
                s1 += double(aa[k]);
                s2 += double(bb[k]);
                if constexpr (NC3) s3 += double(qq[k]);
            }
            phis = s0;
            cA = s1;
            cB = s2;
            cC = s3;
        }
    }
    // phi, the potentials and the source of a node from its population sums (Eqs.
    // Moment0_Phi, PotChem, SourceTerm_Phi); muC of a third composition
    static __device__ __forceinline__ Scalars scalars(double ps, double sA, double sB, double sC, const KParams& P,
                                                      double& muC) {
        if constexpr (NC3) {
            const Scalars3 m3 = node_scalars3(ps, sA, sB, sC, P);
            muC = m3.muC;
            return Scalars{m3.phi, m3.muA, m3.muB, m3.S};
        } else {
            muC = 0.0;
            return node_scalars<GK>(ps, sA, sB, P);
        }
    }
    // isotropic gradient and Laplacian, Eqs. Grad and Laplacian (fluid lattice);
    // at(ex, ey, ez): phi of the neighbour, pc: phi of the node as its neighbours see it
    template <class AT>
    static __device__ __forceinline__ void stencil(AT&& at, C pc, C (&grad)[3], C& lap) {
        C nsum = C(0);  // 3 sum_{k != 0} w_k phi(x + e_k)
        static_for<1, STL::Q>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            constexpr int ex = STL::ex(k), ey = STL::ey(k), ez = STL::ez(k);
            const C v = at(IC<ex>{}, IC<ey>{}, IC<ez>{});
            const C wv = C(3.0 * STL::w(k)) * v;
            if constexpr (ex != 0) grad[0] += ex > 0 ? wv : -wv;
            if constexpr (ey != 0) grad[1] += ey > 0 ? wv : -wv;
            if constexpr (ez != 0) grad[2] += ez > 0 ? wv : -wv;
            nsum += wv;
        });
        lap = C(2) * (nsum - C(3.0 * (1.0 - STL::w(0))) * pc);
    }

    // force, pressure variable p_h (p* with variable density) and velocity of a node;
    // irho = 1 / rho(phi) with variable density
    static __device__ __forceinline__ void flow(const KParams& P, const C (&fpop)[QFN], double phi_d, C phi,
                                                double phi_ref, const C (&grad)[3], C lap, C (&F)[3], C (&u)[3],
                                                C& p_h, C& irho) {
        // Eq. SurfaceTension_Force plus buoyancy (phi - phi_ref) drho g
        C well = C(dwell_d(phi_d));
        pin(well, lap);
        const C bracket = KC(P.cap, P.f32.cap) * (well * KC(P.inv_W2, P.f32.inv_W2) - lap);
        const C buoy = C(phi_d - phi_ref) * KC(P.drho, P.f32.drho);
        F[0] = sum2(buoy, KC(P.gx, P.f32.gx), bracket, grad[0]);
        F[1] = sum2(buoy, KC(P.gy, P.f32.gy), bracket, grad[1]);
        F[2] = sum2(buoy, KC(P.gz, P.f32.gz), bracket, grad[2]);
        // Eqs. HydroPressure and Velocity
        C j0 = C(0), j1 = C(0), j2 = C(0);
        static_for<0, QF>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            p_h += fpop[k];
            if constexpr (FL::ex(k) != 0) j0 += FL::ex(k) > 0 ? fpop[k] : -fpop[k];
            if constexpr (FL::ey(k) != 0) j1 += FL::ey(k) > 0 ? fpop[k] : -fpop[k];
            if constexpr (FL::ez(k) != 0) j2 += FL::ez(k) > 0 ? fpop[k] : -fpop[k];
        });
        if constexpr (!VD) {
            const C inv_rho0 = KC(1.0 / P.rho0, P.f32.inv_rho0);
            u[0] = sum2(C(3), j0, C(0.5), F[0]) * inv_rho0;
            u[1] = sum2(C(3), j1, C(0.5), F[1]) * inv_rho0;
            u[2] = sum2(C(3), j2, C(0.5), F[2]) * inv_rho0;
        } else {
            // variable density: f is dimensionless, p_h holds p* = sum f; rho(phi)
            // interpolated; pressure force -p* c_s^2 grad rho; predictor velocity;
            // viscous force -(nu w+ / c_s^2) Pi . grad rho from the non-equilibrium
            // second moment at the predictor; final velocity
            const C drho = KC(P.drho, P.f32.drho);
            irho = rcp<C>(KC(P.rho0, P.f32.rho0) + drho * phi);
            const C fp = -p_h * C(1.0 / 3.0) * drho;
            C us[3];
            us[0] = j0 + C(0.5) * (F[0] + fp * grad[0]) * irho;
            us[1] = j1 + C(0.5) * (F[1] + fp * grad[1]) * irho;
            us[2] = j2 + C(0.5) * (F[2] + fp * grad[2]) * irho;
            const C uus = dot3(us, us);
            const C e0s = p_h - C(1.5) * uus;
            C pxx = C(0), pyy = C(0), pzz = C(0), pxy = C(0), pxz = C(0), pyz = C(0);
            static_for<0, QF>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                constexpr int ex = FL::ex(k), ey = FL::ey(k), ez = FL::ez(k);
                const C eu = edot<ex, ey, ez>(us[0], us[1], us[2]);
                const C n = fpop[k] - C(FL::w(k)) * (e0s + eu * (C(3) + C(4.5) * eu));
                if constexpr (ex != 0) pxx += n;
                if constexpr (ey != 0) pyy += n;
                if constexpr (ez != 0) pzz += n;
                if constexpr (ex != 0 && ey != 0) pxy += ex * ey > 0 ? n : -n;
                if constexpr (ex != 0 && ez != 0) pxz += ex * ez > 0 ? n : -n;
                if constexpr (ey != 0 && ez != 0) pyz += ey * ez > 0 ? n : -n;
            });
            const C nuv = sum2(KC(P.nu0, P.f32.nu0), C(1) - phi, KC(P.nu1, P.f32.nu1), phi);
            const C coef = -C(3) * nuv * rcp<C>(C(3) * nuv + C(0.5)) * drho;
            const C px[3] = {pxx, pxy, pxz}, py[3] = {pxy, pyy, pyz}, pz[3] = {pxz, pyz, pzz};
            const C dots[3] = {dot3(px, grad), dot3(py, grad), dot3(pz, grad)};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                C Fm = coef * dots[a];
                pin(Fm);
                u[a] = us[a] + C(0.5) * Fm * irho;
                // fused by hand, as the compiler does or does not by the order in which it
                // meets the two products; 16-bit states show the difference
                F[a] += __builtin_elementwise_fma(coef, dots[a], fp * grad[a]);
            }
        }
        pin(u[0], u[1], u[2], F[0], F[1], F[2], p_h);
    }

    // Collision of every field.  Post-collision populations go to sink(IC<slot>, stored
    // form): the 16 bits of a moving population with 16-bit storage, else the value.
    // 16-bit storage: the rounding residue of a field's moving populations is added to its
    // FP32 rest population, so the stored state keeps each node's post-collision mass of
    // every field (the rest population is stored last)
    template <class SINK>
    static __device__ __forceinline__ void collide(const KParams& P, const C (&fpop)[QFN], const C (&g)[QS],
                                                   const C (&a)[QS], const C (&b)[QS], const C (&cq)[QC], double c_ps,
                                                   double sA, double sB, double sC, const Scalars& m, double muC,
                                                   C phi, const C (&F)[3], const C (&u)[3], C p_h, C irho,
                                                   SINK&& sink) {
        constexpr bool FEEDBACK = S16;
        constexpr C inv_cs2s = C(1.0 / SL::cs2);
        auto push = [&](auto s_, auto, auto, C v) __attribute__((always_inline)) {
            static_assert(!S16 || SLOTS::rest(decltype(s_)::value), "16-bit moving populations carry a residue");
            sink(s_, v);
        };
        auto push_r = [&](auto s_, auto k_, auto lat_, C v, C& res) __attribute__((always_inline)) {
            if constexpr (FEEDBACK) {
                unsigned short bits;
                res += enc_res<PREC>(wref(P, s_, k_, lat_), P.fscale[SLOTS::field(decltype(s_)::value)], v, bits);
                sink(s_, bits);
            } else {
                sink(s_, v);
            }
        };
        // BGK steps: the moving populations of directions k and opp(k) of one field
        // (with 16-bit storage: one packed conversion; their stored deviations add to
        // dev, and the rest population is stored last as the field's post-collision
        // zeroth moment, conserved by the collision, minus the stored moving
        // populations, stored_sum)
        auto push_d2 = [&](auto sk_, auto so_, auto k_, auto, auto lat_, C vk, C vo, C& dev)
                           __attribute__((always_inline)) {
            if constexpr (FEEDBACK) {
                constexpr int F_ = SLOTS::field(decltype(sk_)::value);
                static_assert(F_ == SLOTS::field(decltype(so_)::value), "one field");
                float back;
                const unsigned bits = enc2_dev<PREC>(wref(P, sk_, k_, lat_), P.fscale[F_], vk, vo, back);
                sink(sk_, (unsigned short)(bits & 0xffffu));
                sink(so_, (unsigned short)(bits >> 16));
                dev += back;
            } else {
                sink(sk_, vk);
                sink(so_, vo);
            }
        };
        // ---- f: Eqs. LBE_FluidFlow, ForcingTerm, GammaFunction, Feq ----
        // f* = (1 - w) f + w w_k [p + rho0 (eu + 3/2 eu^2 - uu/2)] + (1 - w/2) F_k,
        // F_k = w_k [1 + 3 eu + 9/2 eu^2 - 3/2 uu] (e_k . F - u . F)
        if constexpr (FLOW) {
            const C uu = dot3(u, u);
            const C uF = dot3(u, F);
            const C nu = sum2(KC(P.nu0, P.f32.nu0), C(1) - phi, KC(P.nu1, P.f32.nu1), phi);
            const C wf = rcp<C>(C(3) * nu + C(0.5));
            const C keep = C(1) - wf, half = C(1) - C(0.5) * wf;
            // inertia of the equilibrium: rho0 (Eq. Feq), or 1 / c_s^2 for the
            // dimensionless populations of the variable-density model, whose
            // forcing populations are divided by rho c_s^2
            const C rho0 = VD ? C(3) : KC(P.rho0, P.f32.rho0);
            const C g0 = C(1) - C(1.5) * uu, e0 = p_h - C(0.5) * rho0 * uu;
            const C fsc = VD ? C(3) * irho : C(1);
            if constexpr (MRTC) {
                // MRT: the traceless second order at the viscous rate wf, the trace,
                // third and fourth orders at the given rates; orders 0 and 1 are
                // conserved (rate 1)
                auto feqs = [&](auto kc, C& Fk) __attribute__((always_inline)) -> C {
                    constexpr int k = decltype(kc)::value;
                    constexpr int ex = FL::ex(k), ey = FL::ey(k), ez = FL::ez(k);
                    const C wk = C(FL::w(k));
                    const C eu = edot<ex, ey, ez>(u[0], u[1], u[2]);
                    const C eF = edot<ex, ey, ez>(F[0], F[1], F[2]);
                    Fk = wk * (g0 + eu * (C(3) + C(4.5) * eu)) * (eF - uF);
                    if constexpr (VD) Fk *= fsc;
                    pin(Fk);
                    return diff2(wk, e0 + rho0 * eu * (C(1) + C(1.5) * eu), C(0.5), Fk);
                };
                C Fks[QF];
                C resm = C(0), restm = C(0);
                mrt_relax<FL>(fpop,
                    [&](auto kc) __attribute__((always_inline)) -> C {
                        return feqs(kc, Fks[decltype(kc)::value]);
                    },
                    [&](auto kc) __attribute__((always_inline)) -> C { return Fks[decltype(kc)::value]; },
                    [&](auto ic) __attribute__((always_inline)) -> C {
                        constexpr int i = decltype(ic)::value;
                        constexpr int o = basis_order<FL, i>();
                        if constexpr (o <= 1) return C(1);
                        else if constexpr (basis_trace<FL, i>()) return KC(P.mrt_f[0], P.f32.mrt_f[0]);
                        else if constexpr (o == 2) return wf;
                        else if constexpr (o == 3) return KC(P.mrt_f[1], P.f32.mrt_f[1]);
                        else return KC(P.mrt_f[2], P.f32.mrt_f[2]);
                    },
                    [&](auto kc, C v) __attribute__((always_inline)) {
                        if constexpr (decltype(kc)::value == 0 && FEEDBACK) restm = v;
                        else push_r(kc, kc, FLT{}, v, resm);
                    });
                if constexpr (FEEDBACK) push(IC<0>{}, IC<0>{}, FLT{}, restm + fb(P, IC<0>{}, resm));
            } else if constexpr (!TRTC) {
            // f*_k = keep f_k + w_k [a_k + gam_k (e_k . Fh - u . Fh)] with
            // a_k = wf (e0 + rho0 (eu + 3/2 eu^2)), gam_k = 1 + 3 eu + 9/2 eu^2 - 3/2 uu
            // and Fh = (1 - wf/2) F (times 1 / (rho c_s^2) with variable density):
            // k and opp(k) share eu^2 and differ in the signs of eu, e_k . Fh
            C A = wf * e0, B = wf * rho0;
            const C hs = half * fsc;
            C Fh[3] = {hs * F[0], hs * F[1], hs * F[2]};
            C uFh = hs * uF;
            pin(A, B, Fh[0], Fh[1], Fh[2], uFh);
            C dev = C(0);
            static_for<1, QF>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                constexpr int o = FL::opp(k);
                if constexpr (k < o) {
                    constexpr int ex = FL::ex(k), ey = FL::ey(k), ez = FL::ez(k);
                    const C wk = C(FL::w(k));  // w_opp(k) = w_k
                    const C eu = edot<ex, ey, ez>(u[0], u[1], u[2]);
                    const C eF = edot_scaled<ex, ey, ez>(hs, F, Fh);
                    const C e2 = eu * eu;
                    const C q = C(1.5) * e2;
                    const C r = g0 + C(4.5) * e2;
                    const C ak = A + B * (q + eu), ao = A + B * (q - eu);
                    const C gk = r + C(3) * eu, go = r - C(3) * eu;
                    const C vk = sum2(keep, fpop[k], wk, ak + gk * (eF - uFh));
                    const C vo = sum2(keep, fpop[o], wk, ao - go * (eF + uFh));
                    push_d2(kc, IC<o>{}, kc, IC<o>{}, FLT{}, vk, vo, dev);
                }
            });
            // rest: Sum_k f*_k = p_h (the equilibrium keeps p_h, the forcing sums to 0)
            if constexpr (FEEDBACK) push(IC<0>{}, IC<0>{}, FLT{}, p_h - stored_sum(P, IC<0>{}, FLT{}, dev));
            else push(IC<0>{}, IC<0>{}, FLT{}, sum2(keep, fpop[0], C(FL::w(0)), A - g0 * uFh));
            } else {
                // TRT: the viscosity sets the symmetric rate w+ = wf; w- from the
                // magic parameter, 1/w- - 1/2 = Lambda_f / (1/wf - 1/2) = Lambda_f / (3 nu)
                const C wm = rcp<C>(C(0.5) + KC(P.trt_lf, P.f32.trt_lf) * rcp<C>(C(3) * nu));
                // shifted equilibrium (feq - F_k/2) and source F_k of direction k
                auto eqsrc = [&](auto kc, C& eqs, C& Fk) __attribute__((always_inline)) {
                    constexpr int k = decltype(kc)::value;
                    constexpr int ex = FL::ex(k), ey = FL::ey(k), ez = FL::ez(k);
                    const C wk = C(FL::w(k));
                    const C eu = edot<ex, ey, ez>(u[0], u[1], u[2]);
                    const C eF = edot<ex, ey, ez>(F[0], F[1], F[2]);
                    Fk = wk * (g0 + eu * (C(3) + C(4.5) * eu)) * (eF - uF);
                    if constexpr (VD) Fk *= fsc;
                    pin(Fk);
                    eqs = diff2(wk, e0 + rho0 * eu * (C(1) + C(1.5) * eu), C(0.5), Fk);
                };
                C res = C(0), rest = C(0);
                static_for<0, QF>([&](auto kc) __attribute__((always_inline)) {
                    constexpr int k = decltype(kc)::value;
                    constexpr int o = FL::opp(k);
                    if constexpr (k == 0) {
                        C eqs, Fk;
                        eqsrc(kc, eqs, Fk);
                        rest = fpop[0] - wf * (fpop[0] - eqs) + Fk;
                        if constexpr (!FEEDBACK) push(kc, kc, FLT{}, rest);
                    } else if constexpr (k < o) {
                        C eqk, Fk, eqo, Fo;
                        eqsrc(kc, eqk, Fk);
                        eqsrc(IC<o>{}, eqo, Fo);
                        const C nk = fpop[k] - eqk, no = fpop[o] - eqo;
                        const C sp = wf * C(0.5) * (nk + no), sm = wm * C(0.5) * (nk - no);
                        push_r(kc, kc, FLT{}, fpop[k] - sp - sm + Fk, res);
                        push_r(IC<o>{}, IC<o>{}, FLT{}, fpop[o] - sp + sm + Fo, res);
                    }
                });
                if constexpr (FEEDBACK) push(IC<0>{}, IC<0>{}, FLT{}, rest + fb(P, IC<0>{}, res));
            }
        }
        // ---- g: Eqs. LBE_Phi, Geq, Source_LBE_Phi ----
        // g* = (1 - w) g + w w_k phi (1 + eu / c_s^2) + (1 - w/2) w_k S
        {
            const C wg = KC(P.omega_g, P.f32.omega_g);
            const C keep = C(1) - wg;
            const C wphi = wg * phi;
            const C srcS = (C(1) - C(0.5) * wg) * C(m.S);
            if constexpr (MRTC) {
                // MRT: the first order (diffusive flux) at the M_phi rate, orders 0
                // and 2 at the given even rate, third and fourth at theirs
                const C S = C(m.S), hS = C(0.5) * C(m.S);
                C resm = C(0), restm = C(0);
                mrt_relax<SL>(g,
                    [&](auto kc) __attribute__((always_inline)) -> C {
                        constexpr int k = decltype(kc)::value;
                        constexpr int ex = SL::ex(k), ey = SL::ey(k), ez = SL::ez(k);
                        const C wk = C(SL::w(k));
                        if constexpr (ex != 0 || ey != 0 || ez != 0)
                            return wk * diff2(phi, C(1) + edot<ex, ey, ez>(u[0], u[1], u[2]) * inv_cs2s, C(0.5), S);
                        else
                            return wk * (phi - hS);
                    },
                    [&](auto kc) __attribute__((always_inline)) -> C { return C(SL::w(decltype(kc)::value)) * S; },
                    [&](auto ic) __attribute__((always_inline)) -> C {
                        constexpr int o = basis_order<SL, decltype(ic)::value>();
                        if constexpr (o == 1) return wg;
                        else if constexpr (o == 3) return KC(P.mrt_s[1], P.f32.mrt_s[1]);
                        else if constexpr (o == 4) return KC(P.mrt_s[2], P.f32.mrt_s[2]);
                        else return KC(P.mrt_s[0], P.f32.mrt_s[0]);
                    },
                    [&](auto kc, C v) __attribute__((always_inline)) {
                        if constexpr (decltype(kc)::value == 0 && FEEDBACK) restm = v;
                        else push_r(IC<G0 + decltype(kc)::value>{}, kc, SLT{}, v, resm);
                    });
                if constexpr (FEEDBACK) push(IC<G0>{}, IC<0>{}, SLT{}, restm + fb(P, IC<1>{}, resm));
            } else if constexpr (!TRTC) {
            // g*_k = keep g_k + w_k (t + c eu), t = w phi + (1 - w/2) S, c = w phi / c_s^2
            C t = wphi + srcS, cu = wphi * inv_cs2s;
            pin(t, cu);
            C dev = C(0);
            static_for<1, QS>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                constexpr int o = SL::opp(k);
                if constexpr (k < o) {
                    constexpr int ex = SL::ex(k), ey = SL::ey(k), ez = SL::ez(k);
                    const C wk = C(SL::w(k));
                    const C ceu = cu * edot<ex, ey, ez>(u[0], u[1], u[2]);
                    push_d2(IC<G0 + k>{}, IC<G0 + o>{}, kc, IC<o>{}, SLT{}, sum2(keep, g[k], wk, t + ceu),
                            sum2(keep, g[o], wk, t - ceu), dev);
                }
            });
            // rest: Sum_k g*_k = (1 - w) phi* + w phi + (1 - w/2) S with phi* = Sum_k g_k
            // (phi = phi* + S*/2 takes the predictor's S*, the source the corrected S)
            if constexpr (FEEDBACK) {
                const double wgd = double(wg);
                const double mg = c_ps + wgd * (m.phi - c_ps) + (1.0 - 0.5 * wgd) * m.S;
                push(IC<G0>{}, IC<0>{}, SLT{}, C(mg) - stored_sum(P, IC<1>{}, SLT{}, dev));
            }
            else
                push(IC<G0>{}, IC<0>{}, SLT{}, fma(keep, g[0], C(SL::w(0)) * t));
            } else {
                // TRT: M_phi sets the antisymmetric rate w- = wg; w+ (uniform) from
                // the magic parameter on the host.  Shifted equilibrium
                // w_k phi (1 + eu / c_s^2) - w_k S / 2, source w_k S.
                const C wp = KC(P.omega_gp, P.f32.omega_gp);
                const C S = C(m.S), hS = C(0.5) * C(m.S);
                auto eqs = [&](auto kc) __attribute__((always_inline)) -> C {
                    constexpr int k = decltype(kc)::value;
                    constexpr int ex = SL::ex(k), ey = SL::ey(k), ez = SL::ez(k);
                    const C wk = C(SL::w(k));
                    if constexpr (ex != 0 || ey != 0 || ez != 0)
                        return wk * diff2(phi, C(1) + edot<ex, ey, ez>(u[0], u[1], u[2]) * inv_cs2s, C(0.5), S);
                    else
                        return wk * (phi - hS);
                };
                C res = C(0), rest = C(0);
                static_for<0, QS>([&](auto kc) __attribute__((always_inline)) {
                    constexpr int k = decltype(kc)::value;
                    constexpr int o = SL::opp(k);
                    if constexpr (k == 0) {
                        rest = g[0] - wp * (g[0] - eqs(kc)) + C(SL::w(0)) * S;
                        if constexpr (!FEEDBACK) push(IC<G0>{}, kc, SLT{}, rest);
                    } else if constexpr (k < o) {
                        const C nk = g[k] - eqs(kc), no = g[o] - eqs(IC<o>{});
                        const C sp = wp * C(0.5) * (nk + no), sm = wg * C(0.5) * (nk - no);
                        push_r(IC<G0 + k>{}, kc, SLT{}, g[k] - sp - sm + C(SL::w(k)) * S, res);
                        push_r(IC<G0 + o>{}, IC<o>{}, SLT{}, g[o] - sp + sm + C(SL::w(o)) * S, res);
                    }
                });
                if constexpr (FEEDBACK) push(IC<G0>{}, IC<0>{}, SLT{}, rest + fb(P, IC<1>{}, res));
            }
        }
        // ---- h^A, h^B: Eqs. LBE_c_alpha, Heq; mobility interpolated in phi ----
        {
            const C MA = sum2(KC(P.MA0, P.f32.MA0), C(1) - phi, KC(P.MA1, P.f32.MA1), phi);
            const C MB = sum2(KC(P.MB0, P.f32.MB0), C(1) - phi, KC(P.MB1, P.f32.MB1), phi);
            const C wA = rcp<C>(MA * inv_cs2s + C(0.5));
            const C wB = rcp<C>(MB * inv_cs2s + C(0.5));
            if constexpr (MRTC) {
                // MRT: the first order at the mobility rate, the others at the given
                // rates (order 0 with the even rate: c is conserved exactly)
                auto rates = [&](C wflux) __attribute__((always_inline)) {
                    return [&, wflux](auto ic) __attribute__((always_inline)) -> C {
                        constexpr int o = basis_order<SL, decltype(ic)::value>();
                        if constexpr (o == 1) return wflux;
                        else if constexpr (o == 3) return KC(P.mrt_s[1], P.f32.mrt_s[1]);
                        else if constexpr (o == 4) return KC(P.mrt_s[2], P.f32.mrt_s[2]);
                        else return KC(P.mrt_s[0], P.f32.mrt_s[0]);
                    };
                };
                auto heq = [&](double c, double mu) __attribute__((always_inline)) {
                    return [&, c, mu](auto kc) __attribute__((always_inline)) -> C {
                        constexpr int k = decltype(kc)::value;
                        constexpr int ex = SL::ex(k), ey = SL::ey(k), ez = SL::ez(k);
                        if constexpr (k == 0) return C(c - (1.0 - SL::w(0)) * mu);
                        else return C(SL::w(k)) * (C(mu) + C(c) * edot<ex, ey, ez>(u[0], u[1], u[2]) * inv_cs2s);
                    };
                };
                auto zero = [&](auto) __attribute__((always_inline)) -> C { return C(0); };
                C resA = C(0), restA = C(0), resB = C(0), restB = C(0);
                mrt_relax<SL>(a, heq(sA, m.muA), zero, rates(wA),
                              [&](auto kc, C v) __attribute__((always_inline)) {
                                  if constexpr (decltype(kc)::value == 0 && FEEDBACK) restA = v;
                                  else push_r(IC<A0 + decltype(kc)::value>{}, kc, SLT{}, v, resA);
                              });
                mrt_relax<SL>(b, heq(sB, m.muB), zero, rates(wB),
                              [&](auto kc, C v) __attribute__((always_inline)) {
                                  if constexpr (decltype(kc)::value == 0 && FEEDBACK) restB = v;
                                  else push_r(IC<B0 + decltype(kc)::value>{}, kc, SLT{}, v, resB);
                              });
                if constexpr (FEEDBACK) {
                    push(IC<A0>{}, IC<0>{}, SLT{}, restA + fb(P, IC<2>{}, resA));
                    push(IC<B0>{}, IC<0>{}, SLT{}, restB + fb(P, IC<3>{}, resB));
                }
            } else if constexpr (TRTC) {
                // TRT: the mobility sets the antisymmetric rate w- = wA (wB); w+ from
                // the magic parameter, 1/w+ - 1/2 = Lambda_s / (M / c_s^2)
                const C ls = KC(P.trt_ls, P.f32.trt_ls);
                const C wpA = rcp<C>(C(0.5) + ls * rcp<C>(MA * inv_cs2s));
                const C wpB = rcp<C>(C(0.5) + ls * rcp<C>(MB * inv_cs2s));
                // rest populations (symmetric) in double, as in BGK, stored last with
                // the rounding residues of 16-bit storage
                const double pa = double(a[0]) - double(wpA) * (double(a[0]) - (sA - (1.0 - SL::w(0)) * m.muA));
                const double pb = double(b[0]) - double(wpB) * (double(b[0]) - (sB - (1.0 - SL::w(0)) * m.muB));
                C resA = C(0), resB = C(0);
                const C muA = C(m.muA), muB = C(m.muB);
                const C cuA = C(sA) * inv_cs2s, cuB = C(sB) * inv_cs2s;
                static_for<1, QS>([&](auto kc) __attribute__((always_inline)) {
                    constexpr int k = decltype(kc)::value;
                    constexpr int o = SL::opp(k);
                    if constexpr (k < o) {
                        constexpr int ex = SL::ex(k), ey = SL::ey(k), ez = SL::ez(k);
                        const C wk = C(SL::w(k));  // w_opp(k) = w_k
                        const C eu = edot<ex, ey, ez>(u[0], u[1], u[2]);  // e_opp . u = -eu
                        // h^eq_k = w_k (mu + c eu / c_s^2): symmetric part w_k mu, antisymmetric w_k c eu / c_s^2
                        const C npA = diff2(C(0.5), a[k] + a[o], wk, muA), nmA = diff2(C(0.5), a[k] - a[o], wk * cuA, eu);
                        const C npB = diff2(C(0.5), b[k] + b[o], wk, muB), nmB = diff2(C(0.5), b[k] - b[o], wk * cuB, eu);
                        push_r(IC<A0 + k>{}, kc, SLT{}, a[k] - wpA * npA - wA * nmA, resA);
                        push_r(IC<A0 + o>{}, IC<o>{}, SLT{}, a[o] - wpA * npA + wA * nmA, resA);
                        push_r(IC<B0 + k>{}, kc, SLT{}, b[k] - wpB * npB - wB * nmB, resB);
                        push_r(IC<B0 + o>{}, IC<o>{}, SLT{}, b[o] - wpB * npB + wB * nmB, resB);
                    }
                });
                push(IC<A0>{}, IC<0>{}, SLT{}, C(pa + double(fb(P, IC<2>{}, resA))));
                push(IC<B0>{}, IC<0>{}, SLT{}, C(pb + double(fb(P, IC<3>{}, resB))));
            } else {
            // BGK: h*_k = keep h_k + w_k (w mu + w c eu / c_s^2); k and opp(k) share w mu.
            // Rest populations in double (they carry the conserved composition): from
            // the collision with FP32 / FP64 storage, as c minus the stored moving
            // populations with 16-bit storage
            const C keepA = C(1) - wA, keepB = C(1) - wB;
            C wmuA = wA * C(m.muA), wmuB = wB * C(m.muB);
            C wcA = wA * C(sA) * inv_cs2s, wcB = wB * C(sB) * inv_cs2s;
            pin(wmuA, wmuB, wcA, wcB);
            C devA = C(0), devB = C(0);
            // a third composition: the same BGK relaxation with its own mobility
            C wC = C(0), keepC = C(0), wmuC = C(0), wcC = C(0), devC = C(0);
            if constexpr (NC3) {
                const C MC = sum2(KC(P.MC0, P.f32.MC0), C(1) - phi, KC(P.MC1, P.f32.MC1), phi);
                wC = rcp<C>(MC * inv_cs2s + C(0.5));
                keepC = C(1) - wC;
                wmuC = wC * C(muC);
                wcC = wC * C(sC) * inv_cs2s;
                pin(wmuC, wcC);
            }
            static_for<1, QS>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                constexpr int o = SL::opp(k);
                if constexpr (k < o) {
                    constexpr int ex = SL::ex(k), ey = SL::ey(k), ez = SL::ez(k);
                    const C wk = C(SL::w(k));  // w_opp(k) = w_k
                    const C eu = edot<ex, ey, ez>(u[0], u[1], u[2]);
                    push_d2(IC<A0 + k>{}, IC<A0 + o>{}, kc, IC<o>{}, SLT{}, sum2(keepA, a[k], wk, wmuA + wcA * eu),
                            sum2(keepA, a[o], wk, wmuA - wcA * eu), devA);
                    push_d2(IC<B0 + k>{}, IC<B0 + o>{}, kc, IC<o>{}, SLT{}, sum2(keepB, b[k], wk, wmuB + wcB * eu),
                            sum2(keepB, b[o], wk, wmuB - wcB * eu), devB);
                    if constexpr (NC3)
                        push_d2(IC<HC0 + k>{}, IC<HC0 + o>{}, kc, IC<o>{}, SLT{},
                                sum2(keepC, cq[k], wk, wmuC + wcC * eu), sum2(keepC, cq[o], wk, wmuC - wcC * eu),
                                devC);
                }
            });
            if constexpr (FEEDBACK) {
                push(IC<A0>{}, IC<0>{}, SLT{}, C(sA - double(stored_sum(P, IC<2>{}, SLT{}, devA))));
                push(IC<B0>{}, IC<0>{}, SLT{}, C(sB - double(stored_sum(P, IC<3>{}, SLT{}, devB))));
                if constexpr (NC3)
                    push(IC<HC0>{}, IC<0>{}, SLT{}, C(sC - double(stored_sum(P, IC<4>{}, SLT{}, devC))));
            } else {
                const double w1 = 1.0 - SL::w(0);
                auto rest = [&](C h0, C w, double sc, double mu) __attribute__((always_inline)) -> C {
                    return C(double(h0) - double(w) * (double(h0) - (sc - w1 * mu)));
                };
                push(IC<A0>{}, IC<0>{}, SLT{}, rest(a[0], wA, sA, m.muA));
                push(IC<B0>{}, IC<0>{}, SLT{}, rest(b[0], wB, sB, m.muB));
                if constexpr (NC3) push(IC<HC0>{}, IC<0>{}, SLT{}, rest(cq[0], wC, sC, muC));
            }
            }
        }
    }
};

}  // namespace lbm
