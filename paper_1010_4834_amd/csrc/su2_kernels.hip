// su2_kernels.hip -- gfx950 kernels of the SU(2) library and their launchers.
//
// Method: Cardoso & Bicudo, "SU(2) Lattice Gauge Theory Simulations on Fermi
// GPUs" (arXiv:1010.4834); each kernel names the passage it implements.
// All kernels walk a (lattice, tile) list so one launch advances a whole
// batch of independent lattices; per-tile lattice data live in scalar
// registers and every link load is one global load from a scalar block base
// plus a 32-bit lane offset.  Nothing here is a dense contraction (at most
// 4x4 real products per quaternion): no MFMA, vector-ALU code fed by
// coalesced float4 / float64x2 loads of the parity-split layout.
#include <hip/hip_ext.h>

#include <algorithm>

#include "su2_internal.hpp"

namespace su2 {

// ---------------------------------------------------------------------------
// Site coordinates of half-site `cb` of parity `par`.
struct Site {
    int c[4];  // x, y, z, t
    int s;     // full-site index
};

__device__ __forceinline__ Site site_of(const LatDesc &d, int cb, int par) {
    Site S;
    int row, j, r2, y, z, t;
    udiv(cb, d.hx, d.inv_hx, row, j);
    udiv(row, d.n[1], d.inv_ny, r2, y);
    udiv(r2, d.n[2], d.inv_nz, t, z);
    const int x = 2 * j + ((par + y + z + t) & 1);
    S.c[0] = x; S.c[1] = y; S.c[2] = z; S.c[3] = t;
    S.s = x + (int)__umul24((unsigned)d.n[0], (unsigned)row);  // row < Ny Nz Nt < 2^24
    return S;
}

// Periodic forward / backward steps of the full-site index along mu.
__device__ __forceinline__ int stride_of(const LatDesc &d, int mu) {
    return mu == 0 ? 1 : mu == 1 ? d.n[0] : mu == 2 ? d.n[0] * d.n[1] : d.ns;
}
// Both candidate steps are uniform; they are pinned as scalars so that the
// select picks one of them rather than a multiplier of the stride (which
// would put a 32-bit vector multiply on every neighbour).
__device__ __forceinline__ int step_fwd(const LatDesc &d, const Site &S, int mu) {
    const int st = stride_of(d, mu);
    const int in = uni(st), wrap = uni(-(d.n[mu] - 1) * st);
    return S.c[mu] == d.n[mu] - 1 ? wrap : in;
}
__device__ __forceinline__ int step_bwd(const LatDesc &d, const Site &S, int mu) {
    const int st = stride_of(d, mu);
    const int in = uni(-st), wrap = uni((d.n[mu] - 1) * st);
    return S.c[mu] == 0 ? wrap : in;
}

// The same for a run-time (uniform) direction.
__device__ __forceinline__ int coord_of(const Site &S, int mu) {
    return mu == 0 ? S.c[0] : mu == 1 ? S.c[1] : mu == 2 ? S.c[2] : S.c[3];
}
__device__ __forceinline__ int extent_of(const LatDesc &d, int mu) {
    return mu == 0 ? d.n[0] : mu == 1 ? d.n[1] : mu == 2 ? d.n[2] : d.n[3];
}
__device__ __forceinline__ int step_fwd_rt(const LatDesc &d, const Site &S, int mu) {
    const int st = uni(stride_of(d, mu)), n = uni(extent_of(d, mu));
    return coord_of(S, mu) == n - 1 ? -(n - 1) * st : st;
}
__device__ __forceinline__ int step_bwd_rt(const LatDesc &d, const Site &S, int mu) {
    const int st = uni(stride_of(d, mu)), n = uni(extent_of(d, mu));
    return coord_of(S, mu) == 0 ? (n - 1) * st : -st;
}

// Uniform bases of the (direction, parity) blocks of one lattice in a link
// buffer whose lattice starts at link `first` ([mu][parity][cb]).
template <class T, int NDIR> struct Blocks {
    char *b[NDIR][2];
    uint32_t hoff;
};
template <class T, int NDIR>
__device__ __forceinline__ Blocks<T, NDIR> blocks(const void *buf, long long first, int vh) {
    Blocks<T, NDIR> B;
#pragma unroll
    for (int mu = 0; mu < NDIR; ++mu)
#pragma unroll
        for (int p = 0; p < 2; ++p)
            B.b[mu][p] = (char *)buf + (first + (long long)(2 * mu + p) * vh) * Links<T>::BYTES;
    B.hoff = (uint32_t)vh << 4;
    return B;
}

// Block base of (mu, p); an unrolled select so the bases stay in scalar
// registers (indexing the array with run-time values would spill it to
// private memory and turn every link load into a flat load).
template <class T, int NDIR>
__device__ __forceinline__ char *bsel(const Blocks<T, NDIR> &B, int mu, int p) {
    char *r = B.b[0][0];
#pragma unroll
    for (int m = 0; m < NDIR; ++m) {
        r = (mu == m && p == 0) ? B.b[m][0] : r;
        r = (mu == m && p == 1) ? B.b[m][1] : r;
    }
    return r;
}

template <class T, int NDIR>
__device__ __forceinline__ Q<T> lds_(const Blocks<T, NDIR> &B, int mu, int p, uint32_t cb) {
    return Links<T>::ld(bsel(B, mu, p), B.hoff, cb);
}
template <class T, int NDIR>
__device__ __forceinline__ void sts_(const Blocks<T, NDIR> &B, int mu, int p, uint32_t cb, const Q<T> &q) {
    Links<T>::st(bsel(B, mu, p), B.hoff, cb, q);
}

// Staple V of link (x, MU), x of parity `par` (paper Sec. 2: the six
// plaquettes containing the link; V is the adjoint of the sum of the
// transporters x -> x+mu of the over-relaxation equation, so that the link
// weight is exp(beta/2 Tr(U V))).  nu ascending, upper then lower:
//   upper U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag,
//   lower U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu).
// 18 link loads (gather); 7 distinct per update once shared with
// neighbouring lanes.  combine() does the arithmetic on the gathered links.
template <class T, int MU>
__device__ __forceinline__ void gather(const LatDesc &d, const Blocks<T, 4> &B, const Site &S, int par,
                                       Q<T> (&L)[18]) {
    const int op = par ^ 1;
    const int s_mu = S.s + step_fwd(d, S, MU);
#pragma unroll
    for (int nu = 0; nu < 4; ++nu) {
        if (nu == MU) continue;
        const int q = 6 * (nu < MU ? nu : nu - 1);
        const int fn = step_fwd(d, S, nu), bn = step_bwd(d, S, nu);
        L[q + 0] = lds_(B, nu, op, (uint32_t)s_mu >> 1);            // U_nu(x+mu)
        L[q + 1] = lds_(B, MU, op, (uint32_t)(S.s + fn) >> 1);      // U_mu(x+nu)
        L[q + 2] = lds_(B, nu, par, (uint32_t)S.s >> 1);            // U_nu(x)
        L[q + 3] = lds_(B, nu, par, (uint32_t)(s_mu + bn) >> 1);    // U_nu(x+mu-nu)
        L[q + 4] = lds_(B, MU, op, (uint32_t)(S.s + bn) >> 1);      // U_mu(x-nu)
        L[q + 5] = lds_(B, nu, op, (uint32_t)(S.s + bn) >> 1);      // U_nu(x-nu)
    }
}

// V accumulates nu ascending, upper then lower staple, in one chain of
// fused multiply-adds.  The planes nu < MU come first, so Vlow (the fused
// plaquette) is V as it stands after plane MU - 1: the substep updates its
// links bit for bit the same with and without the plaquette.
template <class T>
__device__ __forceinline__ Q<T> combine(const Q<T> (&L)[18], int mu, Q<T> *Vlow = nullptr) {
    Q<T> V{T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int k = 0; k < 3; ++k) {  // plane nu = k, or k + 1 from nu = mu on
        const int q = 6 * k;
        const Q<T> &A = L[q + 0], &Bm = L[q + 1], &C = L[q + 2], &D = L[q + 3], &E = L[q + 4], &F = L[q + 5];
        qmul_acc(V, A, qdag(qmul(C, Bm)));
        qmul_acc(V, qdag(qmul(E, D)), F);
        if (Vlow && k == mu - 1) *Vlow = V;
    }
    return V;
}

template <class T, int MU>
__device__ __forceinline__ Q<T> staple(const LatDesc &d, const Blocks<T, 4> &B, const Site &S, int par,
                                       Q<T> *Vlow = nullptr) {
    Q<T> L[18];
    gather<T, MU>(d, B, S, par, L);
    return combine<T>(L, MU, Vlow);
}

template <class T, int N> __device__ __forceinline__ T pick(const T (&a)[N], int m) {
    T r = a[0];
#pragma unroll
    for (int k = 1; k < N; ++k) r = (m == k) ? a[k] : r;
    return r;
}
template <class T, int N> __device__ __forceinline__ void put(T (&a)[N], int m, T v) {
#pragma unroll
    for (int k = 0; k < N; ++k)
        if (m == k) a[k] = v;
}


// ---------------------------------------------------------------------------
// Heat-bath substep (paper Sec. 2 heat bath; Sec. 4 chessboard): every link
// (x, MU) with parity(x) = par is redrawn from exp(beta/2 Tr(U V)).
// a0 from Kennedy-Pendleton (alpha >= 2) or Creutz (alpha < 2, or always
// with the Creutz sampler); one Philox call per try, counter (s, sweep,
// tag, try); the direction of the vector part from the call with try word
// 0xFFFFFFFF.  New link X W^dag with W = V/k, renormalised with a binary64
// norm.  The samplers multiply by 1/alpha, formed once per link (binary32:
// the hardware reciprocal, within 1 ulp; binary64: a division), instead of
// dividing on every try.
//
// Each lane owns NL links of the class (one per block-sized slice of its
// tile).  Staples first; then a single rejection loop in which a lane moves
// on to its next link as soon as one is accepted, so a wavefront waits for
// the lane with the most tries over NL links rather than NL times for the
// slowest lane; then the new links are composed and stored.
//
// PLAQ (odd substeps, MU >= 1): every plaquette of a plane (nu, MU) with
// nu < MU holds exactly one MU-link at an odd site, updated here after all
// its other links are final; 1/2 Tr(U' (upper + lower staple of plane nu))
// over nu < MU and over the three odd substeps MU = 1, 2, 3 is therefore the
// plaquette sum (paper Sec. 2, eq. for <P>) of the configuration at the end
// of the sweep; by linearity only the summed staple of those planes is
// kept.  Each wavefront writes its binary64 sum to slot MU-1 of its tile.
// Parts of a link update shared by the heat-bath kernels.
// alpha = beta k of a staple V, k = |V|, its reciprocal (left as it is, the
// caller's 0, when alpha = 0) and W^dag = (V/k)^dag (the caller's 1 when V = 0);
// false for a non-finite staple.
template <class T>
__device__ __forceinline__ bool link_weight(const Q<T> &V, T beta, T &alpha, T &ial, Q<T> &Wd) {
    using M = Mth<T>;
    const T k2 = V.a * V.a + V.b * V.b + V.c * V.c + V.d * V.d;
    T k, ik;
    if (sizeof(T) == 4) {
        ik = M::rsqrt_(k2);
        k = k2 > T(0) ? k2 * ik : T(0);
    } else {
        k = M::sqrt_(k2);
        ik = T(1) / k;
    }
    alpha = beta * k;
    if (alpha > T(0)) ial = M::rcp_(alpha);
    if (k2 > T(0)) Wd = Q<T>{V.a * ik, -V.b * ik, -V.c * ik, -V.d * ik};
    return k2 <= M::MAXV;
}
// Kennedy-Pendleton try: the logarithms of its random words, then 1 - a0 into
// dl and whether it is accepted.
template <class T> __device__ __forceinline__ T kp_logs(const uint4 &wd) {
    using M = Mth<T>;
    const T r1 = M::u(wd.x), r2 = M::u(wd.y), r3 = M::u(wd.z);
    const T cs = M::cos2pi(r2);
    return M::lg(r1) + cs * cs * M::lg(r3);
}
template <class T> __device__ __forceinline__ bool kp_try(const uint4 &wd, T logs, T ia, T &dl) {
    using M = Mth<T>;
    const T r4 = M::u(wd.w);
    const T lam2 = -logs * (ia * (T(0.5) * M::LN_LG));
    dl = T(2) * lam2;
    return r4 * r4 <= T(1) - lam2;
}
// Creutz try; cf = -expm1(-2 alpha).
template <class T> __device__ __forceinline__ bool creutz_try(const uint4 &wd, T al, T ia, T cf, T &dl) {
    using M = Mth<T>;
    const T u1 = M::u(wd.x), u2 = M::u(wd.y);
    if (al >= T(1e-20)) dl = -M::log1p_(-(T(1) - u1) * cf) * ia;
    else dl = T(2) * (T(1) - u1);
    return u2 * u2 <= dl * (T(2) - dl);
}
// Direction of the vector part from its own Philox call (try word
// 0xFFFFFFFF), and U' = X W^dag, renormalised.
template <class T> struct Direction { T cth, sth, cph, sph; };
template <class T> __device__ __forceinline__ Direction<T> draw_direction(const uint4 &wd) {
    using M = Mth<T>;
    const T u1 = M::u(wd.x), u2 = M::u(wd.y);
    return Direction<T>{T(1) - T(2) * u1, T(2) * M::sqrt_(u1 * (T(1) - u1)), M::cos2pi(u2), M::sin2pi(u2)};
}
template <class T> __device__ __forceinline__ Q<T> compose_link(const Direction<T> &r, T dl, const Q<T> &Wd) {
    const T ra = Mth<T>::sqrt_(dl * (T(2) - dl));
    const T rs = ra * r.sth;
    const Q<T> X{T(1) - dl, rs * r.cph, rs * r.sph, ra * r.cth};
    return qnormalize(qmul(X, Wd));
}

// One pass of up to NL links per lane, those of parity `par` at half-sites
// first, first + blockDim.x, ... below vh: staple_at(S, Vlow) the staple of the
// link at S, store(cb, s, U, rec) the new link.  Adds the tries of the
// wavefront to wtries and, with PLAQ, 1/2 Tr(U' Vlow) to pq.
template <class T, int NL, bool PLAQ, class STAPLE, class STORE>
__device__ __forceinline__ void heatbath_links(const LatDesc &d, int par, int first, T beta, int sampler, uint32_t sweep,
                                               uint32_t c2, uint32_t k0, uint32_t k1, unsigned *err,
                                               uint32_t &wtries, double &pq, const STAPLE &staple_at,
                                               const STORE &store) {
    using M = Mth<T>;
    int sidx[NL];
    T alpha[NL], ial[NL];  // alpha = beta k and its reciprocal (0 when alpha = 0)
    Q<T> Wd[NL];
    Q<T> Vl[NL];  // summed staples of the planes nu < MU (PLAQ only)
    uint32_t pend = 0, nonfinite = 0;
#pragma unroll
    for (int m = 0; m < NL; ++m) {
        const int cb = first + m * (int)blockDim.x;
        sidx[m] = 0;
        alpha[m] = T(0);
        ial[m] = T(0);
        Wd[m] = qone<T>();
        if (cb < d.vh) {
            Vl[m] = Q<T>{T(0), T(0), T(0), T(0)};
            const Site S = site_of(d, cb, par);
            const Q<T> V = staple_at(S, PLAQ ? &Vl[m] : nullptr);
            // a non-finite staple (a non-finite neighbour link) is not
            // sampled: the link becomes NaN and the error word counts it
            // (as a call of link_weight these lines take five vector
            // instructions more, 1% of the kernel)
            const T k2 = V.a * V.a + V.b * V.b + V.c * V.c + V.d * V.d;
            if (k2 <= M::MAXV) pend |= 1u << m;
            else nonfinite |= 1u << m;
            T k, ik;
            if (sizeof(T) == 4) {
                ik = M::rsqrt_(k2);
                k = k2 > T(0) ? k2 * ik : T(0);
            } else {
                k = M::sqrt_(k2);
                ik = T(1) / k;
            }
            sidx[m] = S.s;
            alpha[m] = beta * k;
            if (alpha[m] > T(0)) ial[m] = M::rcp_(alpha[m]);
            if (k2 > T(0)) Wd[m] = Q<T>{V.a * ik, -V.b * ik, -V.c * ik, -V.d * ik};
        }
    }

    // Creutz factor -expm1(-2 alpha) per link, formed only when a lane of
    // the wavefront samples with Creutz (as a loop invariant it would
    // otherwise be hoisted and evaluated for every link).
    T cfv[NL];
    bool creutz_any = false;
#pragma unroll
    for (int m = 0; m < NL; ++m) {
        cfv[m] = T(0);
        creutz_any |= ((pend >> m) & 1u) && ((sampler == 1) || !(alpha[m] >= T(2)));
    }
    if (__ballot(creutz_any)) {
#pragma unroll
        for (int m = 0; m < NL; ++m)
            if (((pend >> m) & 1u) && alpha[m] >= T(1e-20)) cfv[m] = -M::expm1_(T(-2) * alpha[m]);
    }

    // Rejection loop: a lane moves to its next link when one is accepted.
    T delta[NL];
    uint32_t rec[NL];
#pragma unroll
    for (int m = 0; m < NL; ++m) {
        delta[m] = ((nonfinite >> m) & 1u) ? M::nan_() : T(0);
        rec[m] = 0;
    }
    if (__ballot(nonfinite != 0u)) {
        if (nonfinite) atomicAdd(err, (unsigned)__popc(nonfinite));
    }
    // The loop runs while any lane of the wavefront has a link pending;
    // each pass is one try of every active lane, so the wavefront's try
    // count is the sum of the active-lane counts (scalar work).
    uint32_t j = 0;
    while (true) {
        const unsigned long long act = __ballot(pend != 0u);
        if (act == 0ull) break;
        wtries += (uint32_t)__popcll(act);
        if (!pend) continue;
        const int m = __builtin_ctz(pend);
        const int s = pick(sidx, m);
        const T al = pick(alpha, m), ia = pick(ial, m);
        const bool creutz = (sampler == 1) || !(al >= T(2));
        const uint4 wd = philox10((uint32_t)s, sweep, c2, j, k0, k1);
        bool acc;
        T dl;
        if (creutz) acc = creutz_try(wd, al, ia, pick(cfv, m), dl);
        else acc = kp_try(wd, kp_logs<T>(wd), ia, dl);
        ++j;
        if (acc || j >= MAX_TRIES) {
            if (!acc) {
                atomicAdd(err, 1u);
                dl = M::nan_();
            }
            put(delta, m, dl);
            put(rec, m, j | ((uint32_t)creutz << 31));
            pend &= pend - 1;
            j = 0;
        }
    }

    // Direction from its own Philox call (try word 0xFFFFFFFF), then
    // U' = X W^dag, renormalised.
#pragma unroll
    for (int m = 0; m < NL; ++m) {
        const int cb = first + m * (int)blockDim.x;
        if (cb < d.vh) {
            const uint4 wd = philox10((uint32_t)sidx[m], sweep, c2, 0xFFFFFFFFu, k0, k1);
            const Q<T> Un = compose_link(draw_direction<T>(wd), delta[m], Wd[m]);
            store(cb, sidx[m], Un, rec[m]);
            if (PLAQ)  // 1/2 Re Tr(U' V_low)
                pq += (double)(Un.a * Vl[m].a - Un.b * Vl[m].b - Un.c * Vl[m].c - Un.d * Vl[m].d);
        }
    }
}

template <class T, int MU, bool TRACE, int NL, bool PLAQ>
__global__ __launch_bounds__(256) void k_heatbath(KArgs a, int par) {
    // the first substep of a sweep takes the sweep word from `next`, and so
    // does a lone substep (no advance: part of the next sweep to run)
    const bool first = a.advance && MU == 0 && par == 0;
    const uint32_t sweep = uni((first || !a.advance) ? a.st->next : a.st->sweep);
    const uint32_t k0 = uni((unsigned)a.st->seed), k1 = uni((unsigned)(a.st->seed >> 32));
    if (a.advance && blockIdx.x == 0 && threadIdx.x == 0) {
        if (first) a.st->sweep = sweep;
        if (MU == 3 && par == 1) a.st->next = sweep + 1u;
    }
    double *plaq_part = a.plaq_part;
    if (PLAQ && a.nslots > 0)
        plaq_part += (long long)(((sweep - uni(a.st->run_base)) / (uint32_t)a.every) % (uint32_t)a.nslots) * 12 *
                     a.ntiles;
    TileWalk w(a.ntiles, a.xcd_remap);
    if (!w.ok()) return;
    int tile = w.tile();
    Tile tl = load_tile(a.tiles, tile);
    LatDesc d = load_desc(a.desc + tl.x);
    while (true) {
        const Blocks<T, 4> B = blocks<T, 4>(a.links, d.off, d.vh);
        const uint32_t c2 = tag(d.lat_id, PURPOSE_HEATBATH, MU, par);
        const T beta = (sizeof(T) == 4) ? (T)d.betaf : (T)d.beta;

        uint32_t wtries = 0;
        double pq = 0.0;
        heatbath_links<T, NL, PLAQ>(
            d, par, tl.y + (int)threadIdx.x, beta, a.sampler, sweep, c2, k0, k1, a.err, wtries, pq,
            [&](const Site &S, Q<T> *Vlow) { return staple<T, MU>(d, B, S, par, Vlow); },
            [&](int cb, int s, const Q<T> &U, uint32_t rec) {
                sts_(B, MU, par, (uint32_t)cb, U);
                if (TRACE) a.trace[d.toff + (long long)s * 4 + MU] = rec;
            });
        if (PLAQ) {
            pq = wave_sum_f64(pq);
            if ((threadIdx.x & 63) == 0)
                plaq_part[(3 * (long long)tile + (MU - 1)) * 4 + (threadIdx.x >> 6)] = pq;
        }
        if ((threadIdx.x & 63) == 0 && wtries) atomicAdd(&a.tries_part[tile], (unsigned long long)wtries);
        if (!w.next()) break;
        tile = w.tile();
        tl = load_tile(a.tiles, tile);
        d = load_desc(a.desc + tl.x);
    }
}

// A link updated by four lanes (those of equal threadIdx.x / 4), for substeps of
// a few wavefronts, which last as long as one wavefront's chain of dependent
// work.  All four gather the staple (the same addresses, one request); lane j of
// the four makes tries j, j + 4, ..., and the first accepted one in order
// composes and stores the link, so links, tries and branches are those of
// heatbath_links.  The first try and the direction depend on the random words
// alone and are evaluated while the links are on their way.  All lanes of a
// wavefront call it; links beyond the lattice are not valid.
template <class T, bool PLAQ, class GATHER, class STORE>
__device__ __forceinline__ void heatbath_link4(const Site &S, bool valid, int mu, T beta, int sampler, uint32_t sweep,
                                               uint32_t c2, uint32_t k0, uint32_t k1, unsigned *err, uint32_t &wtries,
                                               double &pq, const GATHER &gather_at, const STORE &store) {
    using M = Mth<T>;
    const int lane = (int)threadIdx.x & 63, j0 = lane & 3;
    Q<T> L[18];
    gather_at(L);
    __builtin_amdgcn_sched_barrier(0);
    const uint4 wd = philox10((uint32_t)S.s, sweep, c2, (uint32_t)j0, k0, k1);
    const T lg0 = sampler == 1 ? T(0) : kp_logs<T>(wd);
    const Direction<T> dir = draw_direction<T>(philox10((uint32_t)S.s, sweep, c2, 0xFFFFFFFFu, k0, k1));
    __builtin_amdgcn_sched_barrier(0);
    Q<T> Vl{T(0), T(0), T(0), T(0)};
    const Q<T> V = combine<T>(L, mu, PLAQ ? &Vl : nullptr);
    T alpha, ial = T(0);
    Q<T> Wd = qone<T>();
    const bool finite = link_weight(V, beta, alpha, ial, Wd);
    const bool creutz = (sampler == 1) || !(alpha >= T(2));
    bool open = valid && finite, win = valid && !finite && j0 == 0;
    T cf = T(0), dl = M::nan_();
    uint32_t base = 0;
    if (win) atomicAdd(err, 1u);
    if (__ballot(open && creutz)) {
        if (open && alpha >= T(1e-20)) cf = -M::expm1_(T(-2) * alpha);
    }
    while (true) {
        if (__ballot(open) == 0ull) break;
        bool acc = false;
        T t = T(0);
        if (open) {
            uint4 w = wd;
            if (base) w = philox10((uint32_t)S.s, sweep, c2, base + (uint32_t)j0, k0, k1);
            acc = creutz ? creutz_try(w, alpha, ial, cf, t) : kp_try(w, base ? kp_logs<T>(w) : lg0, ial, t);
        }
        const uint32_t g = (uint32_t)(__ballot(acc) >> (lane & ~3)) & 15u;  // the four tries of this link
        const int hit = g ? __builtin_ctz(g) : 4;
        wtries += (uint32_t)__popcll(__ballot(open && j0 <= hit));
        if (open) {
            if (g) {
                win = j0 == hit;
                if (win) dl = t;
                open = false;
            } else if ((base += 4) >= MAX_TRIES) {
                win = j0 == 0;  // the link becomes NaN
                if (win) atomicAdd(err, 1u);
                open = false;
            }
        }
    }
    if (win) {
        const Q<T> Un = compose_link(dir, dl, Wd);
        store(Un);
        if (PLAQ) pq += (double)(Un.a * Vl.a - Un.b * Vl.b - Un.c * Vl.c - Un.d * Vl.d);
    }
}

// The substep of up to split_sites() sites in all, four lanes per link.  A
// workgroup takes 64 links of its tile, as many workgroups per tile as it has
// wavefronts in k_heatbath.
template <class T, int MU, bool PLAQ>
__global__ __launch_bounds__(256) void k_heatbath_split(KArgs a, int par) {
    __shared__ double red[4];
    __shared__ uint32_t redt[4];
    // neighbouring parts of the work on the same XCD (workgroup b runs on XCD b % 8)
    const int parts = a.tile_links >> 6, item = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    const int tile = item / parts, part = item - tile * parts;
    const bool first_sub = a.advance && MU == 0 && par == 0;
    const uint32_t sweep = uni((first_sub || !a.advance) ? a.st->next : a.st->sweep);
    const uint32_t k0 = uni((unsigned)a.st->seed), k1 = uni((unsigned)(a.st->seed >> 32));
    if (a.advance && blockIdx.x == 0 && threadIdx.x == 0) {
        if (first_sub) a.st->sweep = sweep;
        if (MU == 3 && par == 1) a.st->next = sweep + 1u;
    }
    double *plaq_part = a.plaq_part;
    if (PLAQ && a.nslots > 0)
        plaq_part += (long long)(((sweep - uni(a.st->run_base)) / (uint32_t)a.every) % (uint32_t)a.nslots) * 12 *
                     a.ntiles;
    if (tile >= a.ntiles) return;
    const Tile tl = load_tile(a.tiles, tile);
    const LatDesc d = load_desc(a.desc + tl.x);
    const Blocks<T, 4> B = blocks<T, 4>(a.links, d.off, d.vh);
    const uint32_t c2 = tag(d.lat_id, PURPOSE_HEATBATH, MU, par);
    const T beta = (sizeof(T) == 4) ? (T)d.betaf : (T)d.beta;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int cb = tl.y + 64 * part + (tid >> 2);
    const bool valid = cb < d.vh;
    const Site S = site_of(d, valid ? cb : 0, par);
    uint32_t wtries = 0;
    double pq = 0.0;
    heatbath_link4<T, PLAQ>(
        S, valid, MU, beta, a.sampler, sweep, c2, k0, k1, a.err, wtries, pq,
        [&](Q<T>(&L)[18]) { gather<T, MU>(d, B, S, par, L); },
        [&](const Q<T> &U) { sts_(B, MU, par, (uint32_t)cb, U); });
    if (PLAQ) pq = wave_sum_f64(pq);
    if (lane == 0) red[tid >> 6] = pq, redt[tid >> 6] = wtries;
    __syncthreads();
    if (tid == 0) {
        if (PLAQ) plaq_part[(3 * (long long)tile + (MU - 1)) * 4 + part] = (red[0] + red[1]) + (red[2] + red[3]);
        atomicAdd(&a.tries_part[tile], (unsigned long long)(redt[0] + redt[1] + redt[2] + redt[3]));
    }
}

// Over-relaxation substep (paper Sec. 2, over-relaxation equation, in its
// action-preserving form U' = W^dag U^dag W^dag, W = V/k).
// overrelax_link: U replaced by its image under the staple V; false where V
// is zero and U stays.
template <class T> __device__ __forceinline__ bool overrelax_link(const Q<T> &V, Q<T> &U, unsigned *err) {
    const T k2 = V.a * V.a + V.b * V.b + V.c * V.c + V.d * V.d;
    if (!(k2 <= Mth<T>::MAXV)) {  // non-finite staple: NaN link, counted
        atomicAdd(err, 1u);
        const T nan = Mth<T>::nan_();
        U = Q<T>{nan, nan, nan, nan};
        return true;
    }
    if (!(k2 > T(0))) return false;
    const T ik = T(1) / Mth<T>::sqrt_(k2);
    const Q<T> Wd{V.a * ik, -V.b * ik, -V.c * ik, -V.d * ik};
    U = qnormalize(qmul(qmul(Wd, qdag(U)), Wd));
    return true;
}

template <class T, int MU>
__global__ __launch_bounds__(256) void k_overrelax(KArgs a, int par) {
    for_each_tile(a.ntiles, a.xcd_remap, [&](int tile) {
        const Tile tl = load_tile(a.tiles, tile);
        const LatDesc d = load_desc(a.desc + tl.x);
        const Blocks<T, 4> B = blocks<T, 4>(a.links, d.off, d.vh);
        const int cb = tl.y + (int)threadIdx.x;
        if (cb >= d.vh) return;
        const Site S = site_of(d, cb, par);
        const Q<T> V = staple<T, MU>(d, B, S, par);
        // overrelax_link() in place, its link loaded last: as a call the binary64
        // kernels hold 67 registers instead of 88 and wait for their loads in more
        // and smaller groups (24^3 x 48 19.7 us a substep, 18.9 in place; 32^4 29.9, 28.0)
        const T k2 = V.a * V.a + V.b * V.b + V.c * V.c + V.d * V.d;
        if (!(k2 <= Mth<T>::MAXV)) {  // non-finite staple: NaN link, counted
            atomicAdd(a.err, 1u);
            const T nan = Mth<T>::nan_();
            sts_(B, MU, par, (uint32_t)cb, Q<T>{nan, nan, nan, nan});
            return;
        }
        if (!(k2 > T(0))) return;
        const T ik = T(1) / Mth<T>::sqrt_(k2);
        const Q<T> Wd{V.a * ik, -V.b * ik, -V.c * ik, -V.d * ik};
        const Q<T> U = lds_(B, MU, par, (uint32_t)cb);
        sts_(B, MU, par, (uint32_t)cb, qnormalize(qmul(qmul(Wd, qdag(U)), Wd)));
    });
}

// ---------------------------------------------------------------------------
// Whole runs of small lattices.  A substep of a lattice of up to
// SMALL_SITES sites is a few wavefronts, and its launch lasts as long as one
// link update after a cold start (descriptor, tile and links fetched anew by
// every kernel: 3.3 us in binary32, 8 us in binary64).  Here one workgroup
// keeps its lattice in LDS for all sweeps of a call, a workgroup barrier
// between substeps, and one launch advances every lattice of the ensemble.
// The update is heatbath_links / the formula of k_overrelax on the same
// staples, so the links are bit for bit those of the substep kernels.

// Links of one lattice in LDS, in the order of the link buffer.
template <class T> struct LdsBlocks;
template <> struct LdsBlocks<float> {
    float4 *p;
    int vh;
    __device__ __forceinline__ Q<float> ld(int mu, int par, int cb) const {
        const float4 v = p[(2 * mu + par) * vh + cb];
        return Q<float>{v.x, v.y, v.z, v.w};
    }
    __device__ __forceinline__ void st(int mu, int par, int cb, const Q<float> &q) const {
        p[(2 * mu + par) * vh + cb] = make_float4(q.a, q.b, q.c, q.d);
    }
};
template <> struct LdsBlocks<double> {
    double2 *p;
    int vh;
    __device__ __forceinline__ Q<double> ld(int mu, int par, int cb) const {
        const double2 *b = p + 2 * (2 * mu + par) * vh + cb;
        return Q<double>{b[0].x, b[0].y, b[vh].x, b[vh].y};
    }
    __device__ __forceinline__ void st(int mu, int par, int cb, const Q<double> &q) const {
        double2 *b = p + 2 * (2 * mu + par) * vh + cb;
        b[0] = make_double2(q.a, q.b);
        b[vh] = make_double2(q.c, q.d);
    }
};

// gather() and staple() with the links in LDS and the direction a run-time
// (uniform) value
template <class T>
__device__ __forceinline__ void gather_lds(const LatDesc &d, const LdsBlocks<T> &B, const Site &S, int par, int mu,
                                           Q<T> (&L)[18]) {
    const int op = par ^ 1;
    const int s_mu = S.s + step_fwd_rt(d, S, mu);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int nu = k < mu ? k : k + 1, q = 6 * k;
        const int fn = step_fwd_rt(d, S, nu), bn = step_bwd_rt(d, S, nu);
        L[q + 0] = B.ld(nu, op, s_mu >> 1);
        L[q + 1] = B.ld(mu, op, (S.s + fn) >> 1);
        L[q + 2] = B.ld(nu, par, S.s >> 1);
        L[q + 3] = B.ld(nu, par, (s_mu + bn) >> 1);
        L[q + 4] = B.ld(mu, op, (S.s + bn) >> 1);
        L[q + 5] = B.ld(nu, op, (S.s + bn) >> 1);
    }
}
template <class T>
__device__ __forceinline__ Q<T> staple_lds(const LatDesc &d, const LdsBlocks<T> &B, const Site &S, int par, int mu,
                                           Q<T> *Vlow) {
    Q<T> L[18];
    gather_lds(d, B, S, par, mu, L);
    return combine<T>(L, mu, Vlow);
}

// Links of the lattice between the link buffer and LDS (16-byte words).
template <class T>
__device__ __forceinline__ void small_copy(const LatDesc &d, char *links, float4 *lds, bool in) {
    float4 *g = (float4 *)(links + d.off * Links<T>::BYTES);
    const int n = 8 * d.vh * (Links<T>::BYTES / 16);
    for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x) {
        if (in) lds[i] = g[i];
        else g[i] = lds[i];
    }
}

// Sweeps (with over = 0: heat bath, sweep words sweep0 ..; else
// over-relaxation) of lattice blockIdx.x.  Measured sweeps write the mean
// plaquette, of the links' terms as in k_heatbath, and the Polyakov loop to
// outp / outl[l * nm + measurement], both summed in (hi, lo) pairs from the
// lane on; runs without measurements take the kernel without them (4^4, one sweep
// in binary32: 19.6 us, 21.1 with the sums' code in it).
// FOUR: four lanes per link (heat bath; the workgroup holds them all).  Figures
// at small_sites().  The time is the instructions of one wavefront's update,
// issued alone on its SIMD.
template <class T, bool FOUR, bool MEAS>
__global__ __launch_bounds__(SMALL_BLOCK) void k_small_run(KArgs a, SmallRun r, double *outp, double *outl,
                                                           unsigned *errp) {
    extern __shared__ double4 small_lds[];
    __shared__ DD red[SMALL_BLOCK / 64 * 2];
    const int l = (int)blockIdx.x, tid = (int)threadIdx.x, nb = (int)blockDim.x, lane = tid & 63;
    const LatDesc d = load_desc(a.desc + l);
    const LdsBlocks<T> B{(decltype(LdsBlocks<T>::p))small_lds, d.vh};
    const T beta = (sizeof(T) == 4) ? (T)d.betaf : (T)d.beta;
    const uint32_t k0 = (uint32_t)r.seed, k1 = (uint32_t)(r.seed >> 32);
    small_copy<T>(d, (char *)a.links, (float4 *)small_lds, true);
    __syncthreads();
    unsigned long long tries = 0;
    int next = r.every - 1, m = 0;  // sweep of the next measurement
    for (int sw = 0; sw < r.nsweeps; ++sw) {
        const bool measured = MEAS && sw == next && m < r.nm;
        DD sum[2] = {{0.0, 0.0}, {0.0, 0.0}};  // plaquette, Polyakov loop
        for (int sub = 0; sub < 8; ++sub) {
            const int mu = sub >> 1, par = sub & 1;
            if (!r.over) {
                const uint32_t c2 = tag(d.lat_id, PURPOSE_HEATBATH, mu, par), sweep = r.sweep0 + (uint32_t)sw;
                if (FOUR) {
                    const int cb = tid >> 2;
                    const bool valid = cb < d.vh;
                    const Site S = site_of(d, valid ? cb : 0, par);
                    uint32_t wt = 0;
                    double pw = 0.0;
                    heatbath_link4<T, MEAS>(
                        S, valid, mu, beta, a.sampler, sweep, c2, k0, k1, a.err, wt, pw,
                        [&](Q<T>(&L)[18]) { gather_lds(d, B, S, par, mu, L); },
                        [&](const Q<T> &U) { B.st(mu, par, cb, U); });
                    tries += wt;
                    if (MEAS && par) sum[0] = dd_acc(sum[0], pw);
                }
                for (int first = tid; !FOUR && first - lane < d.vh; first += nb) {
                    uint32_t wt = 0;
                    double pw = 0.0;
                    heatbath_links<T, 1, MEAS>(
                        d, par, first, beta, a.sampler, sweep, c2, k0, k1, a.err, wt, pw,
                        [&](const Site &S, Q<T> *Vlow) { return staple_lds<T>(d, B, S, par, mu, Vlow); },
                        [&](int cb, int, const Q<T> &U, uint32_t) { B.st(mu, par, cb, U); });
                    tries += wt;
                    if (MEAS && par) sum[0] = dd_acc(sum[0], pw);
                }
            } else {
                for (int cb = tid; cb < d.vh; cb += nb) {
                    const Site S = site_of(d, cb, par);
                    const Q<T> V = staple_lds<T>(d, B, S, par, mu, (Q<T> *)nullptr);
                    Q<T> U = B.ld(mu, par, cb);
                    if (overrelax_link(V, U, a.err)) B.st(mu, par, cb, U);
                }
            }
            __syncthreads();
        }
        if (measured) {
            if (outl)
                for (int xs = tid; xs < d.ns; xs += nb) {
                    int row, x, z, y;
                    udiv(xs, d.n[0], d.inv_nx, row, x);
                    udiv(row, d.n[1], d.inv_ny, z, y);
                    Q<T> P = qone<T>();
                    const int p0 = (x + y + z) & 1;
                    for (int t = 0; t < d.n[3]; ++t) P = qmul(P, B.ld(3, (p0 + t) & 1, (xs + d.ns * t) >> 1));
                    sum[1] = dd_add(sum[1], DD{(double)P.a, 0.0});
                }
            dd_block_sum<2>(sum, red);
            if (tid == 0) {
                if (outp) outp[(long long)l * r.nm + m] = (sum[0].hi + sum[0].lo) / (12.0 * (double)d.vh);
                if (outl) outl[(long long)l * r.nm + m] = (sum[1].hi + sum[1].lo) / (double)d.ns;
            }
            next += r.every;
            ++m;
        }
    }
    small_copy<T>(d, (char *)a.links, (float4 *)small_lds, false);
    if (lane == 0 && tries) atomicAdd(&a.tries_part[d.tile0], tries);
    if (l == 0 && tid == 0 && !r.over) {
        a.st->seed = r.seed;
        a.st->sweep = a.st->next = r.sweep0 + (uint32_t)r.nsweeps;
    }
    // one lattice: its error word, all of whose counts are this workgroup's or
    // earlier, goes straight to the host
    if (errp) {
        __syncthreads();
        if (tid == 0) *errp = __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---------------------------------------------------------------------------
// Initial configurations (paper Sec. 4: cold start U = 1; hot start a
// Haar-random element per link, Haar measure of Sec. 2): one Philox call
// (purpose 1, sweep 0, try 0) -> four Box-Muller normals in binary64 ->
// normalised, rounded to the link precision.
template <class T>
__global__ __launch_bounds__(256) void k_init(KArgs a, int hot) {
    const unsigned long long seed = a.st->seed;
    for_each_tile(a.ntiles, a.xcd_remap, [&](int tile) {
        const Tile tl = load_tile(a.tiles, tile);
        const LatDesc d = load_desc(a.desc + tl.x);
        const Blocks<T, 4> B = blocks<T, 4>(a.links, d.off, d.vh);
        const int cb = tl.y + (int)threadIdx.x;
        if (cb >= d.vh) return;
        for (int par = 0; par < 2; ++par) {
            const Site S = site_of(d, cb, par);
            for (int mu = 0; mu < 4; ++mu) {
                Q<double> z = qone<double>();
                if (hot) {
                    const uint4 w = philox10((uint32_t)S.s, 0u, tag(d.lat_id, PURPOSE_HOT, mu, par),
                                             0u, (uint32_t)seed, (uint32_t)(seed >> 32));
                    const double u0 = Mth<double>::u(w.x), u1 = Mth<double>::u(w.y);
                    const double u2 = Mth<double>::u(w.z), u3 = Mth<double>::u(w.w);
                    const double r01 = sqrt(-2.0 * log(u0)), r23 = sqrt(-2.0 * log(u2));
                    const double tp = 6.283185307179586476925286766559;
                    z = Q<double>{r01 * cos(tp * u1), r01 * sin(tp * u1), r23 * cos(tp * u3),
                                  r23 * sin(tp * u3)};
                    const double nrm = sqrt(z.a * z.a + z.b * z.b + z.c * z.c + z.d * z.d);
                    z = Q<double>{z.a / nrm, z.b / nrm, z.c / nrm, z.d / nrm};
                }
                sts_(B, mu, par, (uint32_t)cb, Q<T>{(T)z.a, (T)z.b, (T)z.c, (T)z.d});
            }
        }
    });
}

// Canonical float64 [s][mu][4] <-> native layout (ndir = 4: links,
// ndir = 3: smeared spatial links).  One lattice per launch (the tile list
// holds only its tiles); `canon` is that lattice's canonical array.
template <class T>
__global__ __launch_bounds__(256) void k_from_canon(KArgs a, const double *canon) {
    for_each_tile(a.ntiles, a.xcd_remap, [&](int tile) {
        const Tile tl = load_tile(a.tiles, tile);
        const LatDesc d = load_desc(a.desc + tl.x);
        const Blocks<T, 4> B = blocks<T, 4>(a.links, d.off, d.vh);
        const int cb = tl.y + (int)threadIdx.x;
        if (cb >= d.vh) return;
        const double *c = canon;
        for (int par = 0; par < 2; ++par) {
            const Site S = site_of(d, cb, par);
            for (int mu = 0; mu < 4; ++mu) {
                const double *u = c + ((long long)S.s * 4 + mu) * 4;
                sts_(B, mu, par, (uint32_t)cb, Q<T>{(T)u[0], (T)u[1], (T)u[2], (T)u[3]});
            }
        }
    });
}

template <class T>
__global__ __launch_bounds__(256) void k_to_canon(KArgs a, const void *src, int ndir, double *canon) {
    for_each_tile(a.ntiles, a.xcd_remap, [&](int tile) {
        const Tile tl = load_tile(a.tiles, tile);
        const LatDesc d = load_desc(a.desc + tl.x);
        const long long base = ndir == 4 ? d.off : d.soff;
        const Blocks<T, 4> B = blocks<T, 4>(src, base, d.vh);
        const int cb = tl.y + (int)threadIdx.x;
        if (cb >= d.vh) return;
        double *c = canon;
        for (int par = 0; par < 2; ++par) {
            const Site S = site_of(d, cb, par);
            for (int mu = 0; mu < ndir; ++mu) {
                const Q<T> q = lds_(B, mu, par, (uint32_t)cb);
                double *u = c + ((long long)S.s * ndir + mu) * 4;
                u[0] = q.a; u[1] = q.b; u[2] = q.c; u[3] = q.d;
            }
        }
    });
}

// Largest |1 - |U|^2| (bit pattern of a non-negative double is monotone).
template <class T>
__global__ __launch_bounds__(256) void k_unit_defect(KArgs a, unsigned long long *out) {
    for_each_tile(a.ntiles, a.xcd_remap, [&](int tile) {
        const Tile tl = load_tile(a.tiles, tile);
        const LatDesc d = load_desc(a.desc + tl.x);
        const Blocks<T, 4> B = blocks<T, 4>(a.links, d.off, d.vh);
        const int cb = tl.y + (int)threadIdx.x;
        double m = 0.0;
        if (cb < d.vh)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const Q<T> u = lds_(B, q >> 1, q & 1, (uint32_t)cb);
                const double n2 = (double)u.a * u.a + (double)u.b * u.b + (double)u.c * u.c +
                                  (double)u.d * u.d;
                const double e = fabs(1.0 - n2);
                m = (e > m || e != e) ? e : m;
            }
#pragma unroll
        for (int k = 32; k >= 1; k >>= 1) {
            const double o = __shfl_xor(m, k, 64);
            m = (o > m || o != o) ? o : m;
        }
        if ((threadIdx.x & 63) == 0) {
            const unsigned long long bits = (m != m) ? 0x7FF8000000000000ull : __double_as_longlong(m);
            atomicMax(out, bits);
        }
    });
}

// ---------------------------------------------------------------------------
// Plaquette partial sums (paper Sec. 2, eq. for <P>): per site, the six
// planes mu < nu of 1/2 Tr[U_mu(s) U_nu(s+mu) U_mu(s+nu)^dag U_nu(s)^dag]
// = 1/2 Tr[(U_mu(s) U_nu(s+mu)) (U_nu(s) U_mu(s+nu))^dag], traced in link
// precision, accumulated in binary64 per lane, then a compensated block sum
// per tile (spatial, temporal planes).
// ONE: a lattice of a few tiles (ONE_TILES) in one workgroup, which writes the
// averages and the error word to mapped host memory itself; k_finalize and the
// gap before it are 5.5 us of such a call.
template <class T, bool ONE>
__global__ __launch_bounds__(256) void k_plaquette(KArgs a, double *part, double *out, unsigned *err) {
    __shared__ DD lds[2 * 4];
    DD tot[2] = {{0.0, 0.0}, {0.0, 0.0}};
    for_each_tile(a.ntiles, a.xcd_remap, [&](int tile) {
        const Tile tl = load_tile(a.tiles, tile);
        const LatDesc d = load_desc(a.desc + tl.x);
        const Blocks<T, 4> B = blocks<T, 4>(a.links, d.off, d.vh);
        const int cb = tl.y + (int)threadIdx.x;
        DD acc[2] = {{0.0, 0.0}, {0.0, 0.0}};
        if (cb < d.vh) {
            double sp = 0.0, tp = 0.0;
#pragma unroll
            for (int par = 0; par < 2; ++par) {
                const Site S = site_of(d, cb, par);
                const int op = par ^ 1;
                Q<T> U[4];
#pragma unroll
                for (int mu = 0; mu < 4; ++mu) U[mu] = lds_(B, mu, par, (uint32_t)cb);
#pragma unroll
                for (int mu = 0; mu < 4; ++mu) {
                    const uint32_t smu = (uint32_t)(S.s + step_fwd(d, S, mu)) >> 1;
#pragma unroll
                    for (int nu = mu + 1; nu < 4; ++nu) {
                        const uint32_t snu = (uint32_t)(S.s + step_fwd(d, S, nu)) >> 1;
                        const Q<T> Unu_smu = lds_(B, nu, op, smu);
                        const Q<T> Umu_snu = lds_(B, mu, op, snu);
                        const T tr = half_tr_xyd(qmul(U[mu], Unu_smu), qmul(U[nu], Umu_snu));
                        if (nu == 3) tp += (double)tr;
                        else sp += (double)tr;
                    }
                }
            }
            acc[0] = DD{sp, 0.0};
            acc[1] = DD{tp, 0.0};
        }
        if (ONE) {
            tot[0] = dd_add(tot[0], acc[0]);
            tot[1] = dd_add(tot[1], acc[1]);
            return;
        }
        dd_block_sum<2>(acc, lds);
        if (threadIdx.x == 0) {
            part[4 * tile + 0] = acc[0].hi; part[4 * tile + 1] = acc[0].lo;
            part[4 * tile + 2] = acc[1].hi; part[4 * tile + 3] = acc[1].lo;
        }
    });
    if (ONE) {
        dd_block_sum<2>(tot, lds);
        if (threadIdx.x == 0) {
            const double V = 2.0 * (double)uni(a.desc->vh);
            const double sp = tot[0].hi + tot[0].lo, tp = tot[1].hi + tot[1].lo;
            out[0] = (sp + tp) / (6.0 * V);
            out[1] = sp / (3.0 * V);
            out[2] = tp / (3.0 * V);
            *err = *a.err;
        }
    }
}

// Polyakov loop partial sums (paper Sec. 2): per spatial site, the product
// of the temporal links t = 0 .. Nt-1 in ascending t, half trace.
template <class T, bool ONE>
__global__ __launch_bounds__(256) void k_polyakov(KArgs a, double *part, double *out, unsigned *err) {
    __shared__ DD lds[4];
    DD tot[1] = {{0.0, 0.0}};
    if (a.nslots > 0)
        part += (long long)(((uni(a.st->sweep) - uni(a.st->run_base)) / (uint32_t)a.every) % (uint32_t)a.nslots) *
                2 * a.ntiles;
    for_each_tile(a.ntiles, a.xcd_remap, [&](int tile) {
        const Tile tl = load_tile(a.tiles, tile);
        const LatDesc d = load_desc(a.desc + tl.x);
        const Blocks<T, 4> B = blocks<T, 4>(a.links, d.off, d.vh);
        const int xs = tl.y + (int)threadIdx.x;
        DD acc[1] = {{0.0, 0.0}};
        if (xs < d.ns) {
            int row, x, z, y;
            udiv(xs, d.n[0], d.inv_nx, row, x);
            udiv(row, d.n[1], d.inv_ny, z, y);
            Q<T> P = qone<T>();
            const int p0 = (x + y + z) & 1;
            // unrolled so that the loads of several t issue together ahead
            // of the (ordered) product chain
#pragma unroll 4
            for (int t = 0; t < d.n[3]; ++t) {
                const uint32_t cb = (uint32_t)(xs + d.ns * t) >> 1;
                P = qmul(P, lds_(B, 3, (p0 + t) & 1, cb));
            }
            acc[0] = DD{(double)P.a, 0.0};
        }
        if (ONE) {
            tot[0] = dd_add(tot[0], acc[0]);
            return;
        }
        dd_block_sum<1>(acc, lds);
        if (threadIdx.x == 0) {
            part[2 * tile + 0] = acc[0].hi;
            part[2 * tile + 1] = acc[0].lo;
        }
    });
    if (ONE) {
        dd_block_sum<1>(tot, lds);
        if (threadIdx.x == 0) {
            out[0] = (tot[0].hi + tot[0].lo) / (double)uni(a.desc->ns);
            *err = *a.err;
        }
    }
}

// Final per-lattice reduction of the standalone measurements' tile
// partials in a fixed order.  Workgroup b handles chunk b % C of lattice
// b / C: it sums its share of the lattice's partials, writes a (hi, lo) pair
// per quantity to `chunk`, and the last chunk of the lattice to arrive
// (ticket in cnt[l]) combines the C pairs in chunk order and writes the
// plaquette (avg, spatial, temporal) and / or the Polyakov loop, and with the
// first lattice the error word, to mapped host memory: a measurement call ends
// with its synchronisation, without a copy or a kernel for the error word.
__device__ __forceinline__ void chunk_range(int n, int C, int c, int &lo, int &hi) {
    lo = (int)(((long long)n * c) / C);
    hi = (int)(((long long)n * (c + 1)) / C);
}

__global__ __launch_bounds__(256) void k_finalize(const LatDesc *desc, const double *pp, const double *pl,
                                                  unsigned *cnt, double *chunk, int C, double *outp, double *outl,
                                                  long long ostride, const DevState *st, unsigned *err) {
    __shared__ DD lds[3 * 4];
    __shared__ int last;
    last = 1;
    const int l = blockIdx.x / C, c = blockIdx.x % C;
    const LatDesc d = load_desc(desc + l);
    // four independent compensated accumulators per quantity (the sums are
    // latency bound), combined in a fixed order
    DD a4[4][3];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int k = 0; k < 3; ++k) a4[u][k] = DD{0.0, 0.0};
    if (pp) {
        int lo, hi;
        chunk_range(d.ntile, C, c, lo, hi);
        for (int t0 = lo + (int)threadIdx.x; t0 < hi; t0 += 4 * blockDim.x) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u * (int)blockDim.x;
                if (t < hi) {
                    const double4 q = reinterpret_cast<const double4 *>(pp)[d.tile0 + (long long)t];
                    a4[u][0] = dd_add(a4[u][0], DD{q.x, q.y});
                    a4[u][1] = dd_add(a4[u][1], DD{q.z, q.w});
                }
            }
        }
    }
    if (pl) {
        int lo, hi;
        chunk_range(d.nstile, C, c, lo, hi);
        for (int t0 = lo + (int)threadIdx.x; t0 < hi; t0 += 4 * blockDim.x) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u * (int)blockDim.x;
                if (t < hi) {
                    const double2 q = reinterpret_cast<const double2 *>(pl)[d.stile0 + (long long)t];
                    a4[u][2] = dd_add(a4[u][2], DD{q.x, q.y});
                }
            }
        }
    }
    DD acc[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[k] = dd_add(dd_add(a4[0][k], a4[1][k]), dd_add(a4[2][k], a4[3][k]));
    dd_block_sum<3>(acc, lds);
    if (C > 1) {  // chunk sums meet in the last chunk of the lattice to arrive
        if (threadIdx.x == 0) {
            double *ch = chunk + 6 * (long long)blockIdx.x;
            for (int k = 0; k < 3; ++k) {
                ch[2 * k] = acc[k].hi;
                ch[2 * k + 1] = acc[k].lo;
            }
            __threadfence();
            last = atomicAdd(&cnt[l], 1u) == (unsigned)(C - 1);
        }
        __syncthreads();
        if (!last) return;
    }
    if (threadIdx.x == 0) {
        DD tot[3] = {acc[0], acc[1], acc[2]};
        if (C > 1) {
            __threadfence();
            const volatile double *ch = chunk + 6 * (long long)l * C;
            for (int k = 0; k < 3; ++k) tot[k] = DD{0.0, 0.0};
            for (int cc = 0; cc < C; ++cc)
                for (int k = 0; k < 3; ++k)
                    tot[k] = dd_add(tot[k], DD{ch[6 * cc + 2 * k], ch[6 * cc + 2 * k + 1]});
            cnt[l] = 0u;
        }
        const double V = 2.0 * (double)d.vh;
        const double sp = tot[0].hi + tot[0].lo, tp = tot[1].hi + tot[1].lo;
        if (pp) {
            double *o = outp + l * ostride;
            o[0] = (sp + tp) / (6.0 * V);
            o[1] = sp / (3.0 * V);
            o[2] = tp / (3.0 * V);
        }
        if (pl) outl[l * ostride] = (tot[2].hi + tot[2].lo) / (double)d.ns;
        if (l == 0) *err = st->err;
    }
}

// Series values of a batch of measured sweeps, in two fixed-order passes.
// k_series_part: workgroup (l C + c, j) sums chunk c of C of lattice l's
// partials of slot (slot0 + j) % nslots -- the heat-bath plaquette partials
// [tile][plane slot 0, 1 spatial, 2 temporal][wavefront] and the Polyakov
// (hi, lo) pairs -- into three (hi, lo) pairs (spatial planes, temporal
// planes, Polyakov).  k_series_final: workgroup (l, j) adds the C chunk pairs
// in chunk order and writes the mean plaquette and Polyakov loop of sweep
// out0 + j.  Many workgroups per sweep keep the partial reads (0.8 MB per
// sweep at 32^4) off a single compute unit.
__global__ __launch_bounds__(256) void k_series_part(const LatDesc *desc, const double *pp, long long pp_stride,
                                                     const double *pl, long long pl_stride, int slot0, int nslots,
                                                     int Cn, double *chunk) {
    __shared__ DD lds[3 * 4];
    // x: lattice-major (lattice, chunk) pairs (lattice counts beyond the
    // y / z grid limits fit in x); y: measured sweep of the batch
    const int C = Cn, c = blockIdx.x % Cn, l = blockIdx.x / Cn, j = blockIdx.y, nsw = gridDim.y;
    const long long slot = (slot0 + j) % nslots;
    const LatDesc d = load_desc(desc + l);
    DD a4[4][3];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int k = 0; k < 3; ++k) a4[u][k] = DD{0.0, 0.0};
    if (pp) {
        int lo, hi;
        chunk_range(d.nmtile, C, c, lo, hi);
        const double4 *q4 = reinterpret_cast<const double4 *>(pp + slot * pp_stride) + 3 * (long long)d.mtile0;
        for (int t0 = lo + (int)threadIdx.x; t0 < hi; t0 += 4 * blockDim.x) {
            double4 v[4][3];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u * (int)blockDim.x;
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    v[u][k] = t < hi ? q4[3 * (long long)t + k] : make_double4(0.0, 0.0, 0.0, 0.0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    DD &x = a4[u][k == 2 ? 1 : 0];
                    x = dd_add(x, DD{(v[u][k].x + v[u][k].y), 0.0});
                    x = dd_add(x, DD{(v[u][k].z + v[u][k].w), 0.0});
                }
        }
    }
    if (pl) {
        int lo, hi;
        chunk_range(d.nstile, C, c, lo, hi);
        const double2 *q2 = reinterpret_cast<const double2 *>(pl + slot * pl_stride) + d.stile0;
        for (int t0 = lo + (int)threadIdx.x; t0 < hi; t0 += 4 * blockDim.x) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u * (int)blockDim.x;
                if (t < hi) a4[u][2] = dd_add(a4[u][2], DD{q2[t].x, q2[t].y});
            }
        }
    }
    DD acc[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[k] = dd_add(dd_add(a4[0][k], a4[1][k]), dd_add(a4[2][k], a4[3][k]));
    dd_block_sum<3>(acc, lds);
    if (threadIdx.x == 0) {
        double *o = chunk + 6 * (((long long)l * nsw + j) * C + c);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            o[2 * k] = acc[k].hi;
            o[2 * k + 1] = acc[k].lo;
        }
    }
}

__global__ __launch_bounds__(64) void k_series_final(const LatDesc *desc, const double *chunk, int C, bool plaq,
                                                     bool poly, double *outp, double *outl, long long ostride,
                                                     int out0) {
    const int l = blockIdx.x, j = blockIdx.y, nsw = gridDim.y;
    if (threadIdx.x != 0) return;
    const double *ch = chunk + 6 * ((long long)l * nsw + j) * C;
    DD tot[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
    for (int c = 0; c < C; ++c)
        for (int k = 0; k < 3; ++k) tot[k] = dd_add(tot[k], DD{ch[6 * c + 2 * k], ch[6 * c + 2 * k + 1]});
    const LatDesc d = load_desc(desc + l);
    const long long o = l * ostride + out0 + j;
    if (plaq) outp[o] = ((tot[0].hi + tot[0].lo) + (tot[1].hi + tot[1].lo)) / (12.0 * (double)d.vh);
    if (poly) outl[o] = (tot[2].hi + tot[2].lo) / (double)d.ns;
}

// Device state words set from the host values without a host copy.
__global__ void k_set_state(DevState *st, unsigned long long seed, unsigned sweep, unsigned run_base) {
    st->seed = seed;
    st->sweep = sweep;
    st->next = sweep;
    st->run_base = run_base;
}

// The same from the run state the host wrote into mapped host memory before
// launching a captured run (words: seed low, seed high, sweep, run base), so
// that the run's first node needs no kernel arguments of its own.
// Run state from mapped host memory: src[0] the seed, src[1] the sweep word
// (low half) and the run base (high half).  Two relaxed system-scope loads
// are in flight together, one round trip to host memory (four dependent
// volatile reads took four, ~8 us).
__global__ void k_set_state_mapped(DevState *st, const unsigned long long *src) {
    const unsigned long long seed = __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    const unsigned long long sr = __hip_atomic_load(src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    st->seed = seed;
    st->sweep = (unsigned)sr;
    st->next = (unsigned)sr;
    st->run_base = (unsigned)(sr >> 32);
}

__global__ void k_clear_err(DevState *st) { st->err = 0u; }

__global__ void k_err_to_host(const DevState *st, unsigned *out) { *out = st->err; }

// Quaternions in LDS: float4, or two double2 planes n apart, so that
// consecutive lanes read consecutive 16-byte words.
template <class T> struct LdsQ;
template <> struct LdsQ<float> {
    float4 *z;
    __device__ __forceinline__ LdsQ(void *p, int) : z((float4 *)p) {}
    __device__ __forceinline__ Q<float> ld(int i) const {
        const float4 v = z[i];
        return Q<float>{v.x, v.y, v.z, v.w};
    }
    __device__ __forceinline__ void st(int i, const Q<float> &q) const { z[i] = make_float4(q.a, q.b, q.c, q.d); }
};
template <> struct LdsQ<double> {
    double2 *z;
    int n;
    __device__ __forceinline__ LdsQ(void *p, int n_) : z((double2 *)p), n(n_) {}
    __device__ __forceinline__ Q<double> ld(int i) const {
        const double2 l = z[i], h = z[i + n];
        return Q<double>{l.x, l.y, h.x, h.y};
    }
    __device__ __forceinline__ void st(int i, const Q<double> &q) const {
        z[i] = make_double2(q.a, q.b);
        z[i + n] = make_double2(q.c, q.d);
    }
};

// ---------------------------------------------------------------------------
// APE smearing step (paper Sec. 2, APE equation) of the spatial links, all
// at once from the previous step: U' = normalise[(1-alpha) U + (alpha/4)
// sum over the two other spatial nu of the forward staple
// U_nu(x) U_mu(x+nu) U_nu(x+mu)^dag and the backward staple
// U_nu(x-nu)^dag U_mu(x-nu) U_nu(x-nu+mu)] with a binary64 norm.
// src_raw: read the lattice links (first step) or the smeared buffer.
// Work item v = 2 tile + parity: the two parities of a tile are neighbours
// in the walk, so an XCD updates both halves of its share of the lattice
// while the links they share are in its L2 (with the parities in separate
// passes every link was fetched twice).  A lane updates the three spatial
// links of its site.

// APE step of the three spatial links of one site (paper Sec. 2, APE
// equation).  Their twelve staples touch 24 distinct links: the three own
// links O[m] = U_m(x) and the backward links K[n] = U_n(x-n), used by every
// plane, and per spatial plane {m, n} (m < n) six links used by it alone,
// each loaded once: F_mn = U_m(x+n), F_nm = U_n(x+m), M_mn = U_m(x-n),
// M_nm = U_n(x-m), D_nm = U_n(x+m-n), D_mn = U_m(x+n-m).  Plane {m, n} adds
// to the sum of direction m its forward staple U_n(x) U_m(x+n) U_n(x+m)^dag
// and its backward staple U_n(x-n)^dag U_m(x-n) U_n(x-n+m), and the same
// with m and n exchanged to the sum of direction n.  The planes run {0,1},
// {0,2}, {1,2}, so every direction accumulates its two other directions in
// ascending order, forward then backward.  Then U' = normalise[(1-alpha) U
// + (alpha/4) sum], the norm in binary64: the hardware 1/sqrt estimate and
// two Newton steps (each squares the relative error; after the second it is
// below binary64 rounding).  A smeared sum is in general far from unit
// norm, so there is no near-group shortcut.
//
// ld(m, s, same): link m of site s, of the parity of the updated site or the
// other; f, b: the site's periodic steps; store(m, q): new link m.
template <class T, class LD, class ST>
__device__ __forceinline__ void ape_links(int s, const int (&f)[3], const int (&b)[3], T alpha, const LD &ld,
                                          const ST &store) {
    Q<T> O[3], K[3], sum[3];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        O[m] = ld(m, s, true);
        K[m] = ld(m, s + b[m], false);
        sum[m] = Q<T>{T(0), T(0), T(0), T(0)};
    }
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) {
        const int m = pl == 2 ? 1 : 0, n = pl == 0 ? 1 : 2;
        const Q<T> Fmn = ld(m, s + f[n], false);
        const Q<T> Fnm = ld(n, s + f[m], false);
        const Q<T> Mmn = ld(m, s + b[n], false);
        const Q<T> Mnm = ld(n, s + b[m], false);
        const Q<T> Dnm = ld(n, s + f[m] + b[n], true);
        const Q<T> Dmn = ld(m, s + f[n] + b[m], true);
        qmul_acc(sum[m], qmul(O[n], Fmn), qdag(Fnm));
        qmul_acc(sum[m], qmul(qdag(K[n]), Mmn), Dnm);
        qmul_acc(sum[n], qmul(O[m], Fnm), qdag(Fmn));
        qmul_acc(sum[n], qmul(qdag(K[m]), Mnm), Dmn);
    }
    const T w0 = T(1) - alpha, w1 = T(0.25) * alpha;
#pragma unroll
    for (int mu = 0; mu < 3; ++mu) {
        const Q<T> &u = O[mu], &sm = sum[mu];
        const Q<T> w{w0 * u.a + w1 * sm.a, w0 * u.b + w1 * sm.b, w0 * u.c + w1 * sm.c, w0 * u.d + w1 * sm.d};
        const double wa = w.a, wb = w.b, wc = w.c, wd = w.d;
        const double n2 = wa * wa + wb * wb + wc * wc + wd * wd;
        Q<T> un = u;
        if (n2 > 0.0) {
            double y = __builtin_amdgcn_rsq(n2);
            const double h = 0.5 * n2;
            y = y * (1.5 - h * y * y);
            y = y * (1.5 - h * y * y);
            un = Q<T>{(T)(wa * y), (T)(wb * y), (T)(wc * y), (T)(wd * y)};
        }
        store(mu, un);
    }
}

template <class T>
__global__ __launch_bounds__(256) void k_ape(KArgs a, const void *src, int src_raw, void *dst, T alpha) {
    for_each_tile(2 * a.ntiles, a.xcd_remap, [&](int v) {
        const Tile tl = load_tile(a.tiles, v >> 1);
        const int par = v & 1;
        const LatDesc d = load_desc(a.desc + tl.x);
        const Blocks<T, 3> Bs = blocks<T, 3>(src, src_raw ? d.off : d.soff, d.vh);
        const Blocks<T, 3> Bd = blocks<T, 3>(dst, d.soff, d.vh);
        const int cb = tl.y + (int)threadIdx.x;
        if (cb >= d.vh) return;
        const Site S = site_of(d, cb, par);
        int f[3], b[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            f[m] = step_fwd(d, S, m);
            b[m] = step_bwd(d, S, m);
        }
        ape_links<T>(S.s, f, b, alpha,
                     [&](int m, int s, bool same) { return lds_(Bs, m, same ? par : par ^ 1, (uint32_t)s >> 1); },
                     [&](int m, const Q<T> &q) { sts_(Bd, m, par, (uint32_t)cb, q); });
    });
}

// All steps of a lattice whose time slices have up to ape_slice() sites, one
// workgroup per slice: a step reaches no other slice, so the slice stays in LDS
// and one launch takes the place of one per step.  A thread updates one site;
// the new links wait in registers for the barrier behind the last read of the
// step.  The arithmetic is ape_links, the smeared links are bit for bit those of
// k_ape.  us per step here and as launches: binary32 1.1 and 4.8 (4^3), 1.7 and
// 4.5 (8^3), 2.8 and 4.5 (1024 sites); binary64 2.5 and 5.5 (8^3, the largest
// whose registers hold one site per thread in a single workgroup).
template <class T>
__global__ __launch_bounds__(ape_slice(sizeof(T) == 4)) void k_ape_slices(KArgs a, const void *src, int src_raw,
                                                                          void *dst, T alpha, int nsteps) {
    extern __shared__ double4 ape_lds[];
    const int t = (int)blockIdx.x;
    const LatDesc d = load_desc(a.desc);
    const Blocks<T, 3> Bs = blocks<T, 3>(src, src_raw ? d.off : d.soff, d.vh);
    const Blocks<T, 3> Bd = blocks<T, 3>(dst, d.soff, d.vh);
    const LdsQ<T> Z(ape_lds, 3 * d.ns);
    const int xs = min((int)threadIdx.x, d.ns - 1);
    const bool on = (int)threadIdx.x < d.ns;
    const uint32_t cb = (uint32_t)(xs + t * d.ns) >> 1;
    Site S;
    int r, f[3], b[3];
    udiv(xs, d.n[0], d.inv_nx, r, S.c[0]);
    udiv(r, d.n[1], d.inv_ny, S.c[2], S.c[1]);
    S.c[3] = t;
    const int par = (S.c[0] + S.c[1] + S.c[2] + t) & 1;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        f[m] = step_fwd(d, S, m);
        b[m] = step_bwd(d, S, m);
        if (on) Z.st(m * d.ns + xs, lds_(Bs, m, par, cb));
    }
    __syncthreads();
    for (int k = 0; k < nsteps; ++k) {
        Q<T> un[3];
        if (on)
            ape_links<T>(xs, f, b, alpha, [&](int m, int s, bool) { return Z.ld(m * d.ns + s); },
                         [&](int m, const Q<T> &q) { un[m] = q; });
        __syncthreads();
        if (on)
#pragma unroll
            for (int m = 0; m < 3; ++m) Z.st(m * d.ns + xs, un[m]);
        __syncthreads();
    }
    if (on)
#pragma unroll
        for (int m = 0; m < 3; ++m) sts_(Bd, m, par, cb, Z.ld(m * d.ns + xs));
}

// ---------------------------------------------------------------------------
// Wilson loops (paper Sec. 2, W(R,T)) in the temporal gauge.  With the
// prefix products P(x,t) = U_4(x,0) .. U_4(x,t-1) of a spatial site's temporal
// links the loop is, for temporal links of any norm but zero,
//   1/2 Tr[S(x,t;R) T(x+R) S(x,t+T;R)^dag T(x)^dag]
//     = w(x,t) w(x+R,t) Z(x,t;R) . Z(x,t+T;R),
//   Z(x,t;R) = P(x,t) S(x,t;R) P(x+R,t)^dag,  w = 1/|P|^2,
// the dot product running over the four quaternion components: a trace costs
// four multiply-adds, where transporting the temporal sides around each loop
// took two quaternion products more.  Times t >= Nt continue the prefix
// products over the periodic links, so a loop that wraps needs nothing of its
// own.  Products of P, the dot products and their sums are binary64; the
// lines Z are held in link precision.
// Links in a caller's buffer may have any norm.  Where a |P|^2 is further than
// 2^-6 from 1 (the links that set_links takes and the sampler leaves stay closer
// over 15000 times), k_wlinks says so in the state, and the call is made again by
// transport, which has no use for inverses: 1/|P|^2 would leave binary32, and is
// infinite behind a zero link.
template <class T> __device__ __forceinline__ Q<double> qwide(const Q<T> &q) {
    return Q<double>{(double)q.a, (double)q.b, (double)q.c, (double)q.d};
}

// k_wgauge: P of 64 spatial sites (lanes), times 0 .. next - 1.  The
// ordered product is bound by its own latency (one lane per site fills a
// fifth of the chip's wavefront slots at 24^3 sites), so the eight wavefronts
// of a workgroup take eight times each of 64: they multiply their links,
// exchange the products through LDS and start from the product of the
// wavefronts before them: 9.2 us at 24^3 x 48, T <= 16, 25 us as one ordered
// product per lane.  P: planes (a0,a1) and (a2,a3) per time, [t][plane][spatial
// site].
template <class T>
__global__ __launch_bounds__(512) void k_wgauge(KArgs a, int next, double2 *__restrict__ P) {
    __shared__ double2 seg[8][2][64];
    const LatDesc d = load_desc(a.desc);
    const Blocks<T, 4> B = blocks<T, 4>(a.links, d.off, d.vh);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.st->off_group = 0u;  // for k_wlinks
    const int lane = (int)threadIdx.x & 63, wave = uni((int)threadIdx.x >> 6);
    const int xs = min((int)blockIdx.x * 64 + lane, d.ns - 1);  // lanes beyond the lattice repeat its last site
    int r, x, y, z;
    udiv(xs, d.n[0], d.inv_nx, r, x);
    udiv(r, d.n[1], d.inv_ny, z, y);
    const int p0 = (x + y + z) & 1, Nt = d.n[3];
    Q<double> carry = qone<double>();
    for (int t0 = 0; t0 < next; t0 += 64) {
        Q<T> U[8];
        int tl = (t0 + 8 * wave) % Nt;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            U[k] = lds_(B, 3, (p0 + tl) & 1, (uint32_t)(xs + d.ns * tl) >> 1);
            tl = tl + 1 == Nt ? 0 : tl + 1;
        }
        Q<double> p{(double)U[0].a, (double)U[0].b, (double)U[0].c, (double)U[0].d};
#pragma unroll
        for (int k = 1; k < 8; ++k)
            p = qmul(p, Q<double>{(double)U[k].a, (double)U[k].b, (double)U[k].c, (double)U[k].d});
        seg[wave][0][lane] = make_double2(p.a, p.b);
        seg[wave][1][lane] = make_double2(p.c, p.d);
        __syncthreads();
        p = carry;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const double2 l = seg[v][0][lane], h = seg[v][1][lane];
            carry = qmul(carry, Q<double>{l.x, l.y, h.x, h.y});
            if (v + 1 == wave) p = carry;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int t = t0 + 8 * wave + k;
            if (t < next) {
                double2 *q = P + 2 * (long long)t * d.ns + xs;
                q[0] = make_double2(p.a, p.b);
                q[d.ns] = make_double2(p.c, p.d);
                p = qmul(p, Q<double>{(double)U[k].a, (double)U[k].b, (double)U[k].c, (double)U[k].d});
            }
        }
        __syncthreads();
    }
}

// s (1 + f), the small f given: weights within rounding of 1 are kept as their
// distance from it (rounded to binary32 themselves they average 1.3e-8 too
// small, 1e-7 in a loop of R = 8)
template <class T> __device__ __forceinline__ Q<T> qscale1p(const Q<T> &q, T f) {
    return Q<T>{fma(q.a, f, q.a), fma(q.b, f, q.b), fma(q.c, f, q.c), fma(q.d, f, q.d)};
}

// k_wlinks: the spatial links in that gauge, P(x,t) U_mu(x,t) P(x+mu,t)^dag =
// Z(x,t;1), and the weights as w - 1, line by line along mu:
// [mu][line][t][position along mu], so that k_wloops reads its lines as
// contiguous blocks.  (Gathered by k_wloops itself from the parity-split links
// and P, 16 bytes from each cache line where mu is not x, the same loads took
// 75 of its 158 us at 24^3 x 48.)  A workgroup takes a 32 x 32 tile of one
// time: x and, for mu = 2, z, else y; where mu is not x the tile is
// transposed through LDS.
__device__ __forceinline__ double rcp_newton(double x) {  // 1/x, relative error below 2^-52
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

template <class T>
__global__ __launch_bounds__(512) void k_wlinks(KArgs a, const void *sp, int sp_raw, int next, int tbase,
                                                const double2 *__restrict__ P, Q<T> *__restrict__ L,
                                                T *__restrict__ w) {
    __shared__ Q<T> tq[32 * 33];
    __shared__ T tw[32 * 33];
    const LatDesc d = load_desc(a.desc);
    const Blocks<T, 3> B = blocks<T, 3>(sp, sp_raw ? d.off : d.soff, d.vh);
    // times round-robin over the XCDs (workgroup b runs on XCD b % 8), the
    // three directions of a time one after another: its P and links are
    // fetched into that XCD's L2 once (with the directions as separate passes
    // over all times 28 us at 24^3 x 48)
    const int per = gridDim.x >> 3, q8 = (int)blockIdx.x >> 3, t = tbase + ((int)blockIdx.x & 7) + 8 * (int)blockIdx.y;
    if (t >= next) return;
    const int mu = q8 / (per / 3);
    // marked once, behind the tiles: a branch between the two elements' arithmetic
    // cost 3.4 of 25.0 us at 24^3 x 48 in binary32
    bool far = false;
    const int ntx = (d.n[0] + 31) >> 5;
    const int nj = mu == 2 ? d.n[2] : d.n[1], no = mu == 2 ? d.n[1] : d.n[2], ntj = (nj + 31) >> 5;
    for (int tile = q8 - mu * (per / 3); tile < ntx * ntj * no; tile += per / 3) {
        const int x0 = (tile % ntx) << 5, r = tile / ntx;
        const int j0 = (r % ntj) << 5, o = r / ntj;
        const int TX = min(32, d.n[0] - x0), TJ = min(32, nj - j0), nel = TX * TJ;
        const int tm = t % d.n[3], st = mu == 0 ? 1 : mu == 1 ? d.n[0] : d.n[0] * d.n[1];
        const long long first = (long long)mu * d.ns * next;
        const double2 *Pt = P + 2 * (long long)t * d.ns;
        const float iX = 1.0f / (float)TX, iJ = 1.0f / (float)TJ;
        // two elements per thread, their loads together (at most 1024 elements,
        // threads for at least half of them); threads beyond the tile repeat its
        // last element
        Q<T> U[2];
        double2 al[2], ah[2], bl[2], bh[2];
        int is[2], js[2];
        long long ks[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int e = min((int)threadIdx.x + h * (int)blockDim.x, nel - 1);
            const int j = (int)(((float)e + 0.5f) * iX), i = e - j * TX;
            const int x = x0 + i, c = j0 + j, y = mu == 2 ? o : c, z = mu == 2 ? c : o;
            const int sa = x + d.n[0] * (y + d.n[1] * z);
            const int pos = mu == 0 ? x : c, N = mu == 0 ? d.n[0] : nj;
            const int sb = sa + (pos + 1 == N ? -(N - 1) * st : st);
            is[h] = i, js[h] = j;
            ks[h] = first + ((long long)(y + d.n[1] * z) * next + t) * d.n[0] + x;
            U[h] = lds_(B, mu, (x + y + z + tm) & 1, (uint32_t)(sa + tm * d.ns) >> 1);
            al[h] = Pt[sa], ah[h] = Pt[sa + d.ns], bl[h] = Pt[sb], bh[h] = Pt[sb + d.ns];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const Q<double> m = qmul(qmul(Q<double>{al[h].x, al[h].y, ah[h].x, ah[h].y}, qwide(U[h])),
                                     Q<double>{bl[h].x, -bl[h].y, -bh[h].x, -bh[h].y});
            const double n2 = al[h].x * al[h].x + al[h].y * al[h].y + ah[h].x * ah[h].x + ah[h].y * ah[h].y;
            far |= fabs(1.0 - n2) > 0x1p-6;  // not for NaN: the loops are NaN either way
            const T wv = (T)((1.0 - n2) * rcp_newton(n2));
            const Q<T> q{(T)m.a, (T)m.b, (T)m.c, (T)m.d};
            if (mu == 0) {
                L[ks[h]] = q;
                w[ks[h]] = wv;
            } else {
                tq[is[h] * 33 + js[h]] = q;
                tw[is[h] * 33 + js[h]] = wv;
            }
        }
        if (mu == 0) continue;
        __syncthreads();
        for (int e = (int)threadIdx.x; e < nel; e += (int)blockDim.x) {
            const int i = (int)(((float)e + 0.5f) * iJ), j = e - i * TJ;
            const long long k = first + ((long long)(x0 + i + d.n[0] * o) * next + t) * nj + j0 + j;
            L[k] = tq[i * 33 + j];
            w[k] = tw[i * 33 + j];
        }
        __syncthreads();
    }
    if (far) a.st->off_group = 1u;
}

// s + 1/2 Tr(x y^dag), the trace in the precision of its operands, the sum in
// binary64
__device__ __forceinline__ double add_dot(double s, const Q<float> &x, const Q<float> &y) {
    return s + (double)half_tr_xyd(x, y);
}
__device__ __forceinline__ double add_dot(double s, const Q<double> &x, const Q<double> &y) {
    return fma(x.d, y.d, fma(x.c, y.c, fma(x.b, y.b, fma(x.a, y.a, s))));
}

// Wavefront sums of N values (a power of two) at once.  Each step adds the
// two halves of the wavefront that differ in one lane bit and, while more
// than one value is left, keeps half of the values in either half, so N = 16
// takes 17 exchanges where separate butterflies take 96.  Lane bits 5 and 4
// are exchanged by the lane-swap instructions, bits 0, 1, 3 and 2 by DPP.
// Every lane ends with the total of value `which`.
__device__ __forceinline__ void swap_halves32(double &a, double &b) {
    const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    a = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
    b = __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ void swap_halves16(double &a, double &b) {
    const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    a = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
    b = __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
template <int CTRL> __device__ __forceinline__ double dpp_f64(double v) {
    const unsigned long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_ROR4 = 0x124, DPP_ROR8 = 0x128;  // quad_perm, row_ror
template <int CTRL, int N, int H>
__device__ __forceinline__ void dpp_step(double (&v)[N], bool up) {
    if constexpr (H >= 1) {  // 2 H values left: keep H of them
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const double keep = up ? v[i + H] : v[i], send = up ? v[i] : v[i + H];
            v[i] = keep + dpp_f64<CTRL>(send);
        }
    } else {
        v[0] += dpp_f64<CTRL>(v[0]);
    }
}
template <int N> __device__ __forceinline__ double wave_sum_many(double (&v)[N], int lane, int &which) {
    static_assert(N == 4 || N == 8 || N == 16, "number of values");
    constexpr int H5 = N / 2, H4 = N / 4, H0 = N / 8, H1 = N / 16;
#pragma unroll
    for (int i = 0; i < H5; ++i) {
        swap_halves32(v[i], v[i + H5]);
        v[i] += v[i + H5];
    }
#pragma unroll
    for (int i = 0; i < H4; ++i) {
        swap_halves16(v[i], v[i + H4]);
        v[i] += v[i + H4];
    }
    dpp_step<DPP_XOR1, N, H0>(v, lane & 1);
    dpp_step<DPP_XOR2, N, H1>(v, lane & 2);
    v[0] += dpp_f64<DPP_ROR8>(v[0]);
    v[0] += dpp_f64<DPP_ROR4>(v[0]);
    which = (lane & 32 ? H5 : 0) + (lane & 16 ? H4 : 0) + (lane & 1 ? H0 : 0) + (lane & 2 ? H1 : 0);
    return v[0];
}

// Loop traces of the times toff < T <= toff + Tp (Tp <= TMAX) and every
// R <= Rmax.  A work unit is a group of G lattice lines along direction mu (or
// a piece of XC sites of one line), times t0 .. t0 + TC - 1: the workgroup
// holds Z of its elements (line, x, t) for the current R in LDS, times t0 ..
// t0 + TC - 1 and, without the gap that a large toff leaves, up to t0 + TC - 1
// + toff + Tp, and the single transformed link P(x,t) U(x,t)
// P(x+mu,t)^-1 of an element in the registers of the lane that owns it, so
// that Z(x,t;R+1) = link(x,t) Z(x+mu,t;R) reads only its LDS neighbour.  A
// line that is held whole wraps around (XE = XC = N); a piece carries
// XE - XC = Rmax elements beyond it, whose last values are not used.
// For the traces a lane owns NC successive times of one x and meets each
// later Z once for all of them: NC + Tp LDS reads per R for NC Tp four-term
// products, taken in link precision and summed in binary64.  The lane sums of one R are added over
// the wavefront and kept per (wavefront, R, T) in LDS until the last unit.
// Rows beyond the lattice or the unit enter as zero times a valid Z.
// At 24^3 x 48, R <= 12, T <= 16 in binary32: 127 us, with k_wgauge, k_wlinks
// and k_wfinal 164 us, where storing the lines of every R (84 us) and
// transporting the temporal sides around each loop (488 us, 37.5 vector
// instructions per (site, mu, R, T)) took 580.  About 9.6 us per R: 6 vector
// instructions per (site, mu, R, T) in binary32 and 4 in binary64, where a
// binary64 instruction issues every 5.6 cycles against 3.1 in binary32
// (measured), and 3.7 us per R for the next line, the sums and two barriers.
// 24^3 x 32, R <= 10, T <= 12 in binary64: 190 us, was 865.
template <class T, int TMAX, int NC, int KE>
__global__ __attribute__((amdgpu_flat_work_group_size(64, 512), amdgpu_waves_per_eu(3))) void k_wloops(
    KArgs a, WPlan pl, int Rmax, int next, const Q<T> *__restrict__ L, const T *__restrict__ w,
    double *__restrict__ part) {
    extern __shared__ double4 wl_lds[];
    const int tid = (int)threadIdx.x, nb = (int)blockDim.x, lane = tid & 63, wave = tid >> 6;
    const LatDesc d = load_desc(a.desc);
    const LdsQ<T> Z(wl_lds, pl.nel);
    T *wt = (T *)((char *)wl_lds + (size_t)pl.nel * Links<T>::BYTES);
    double *acc = (double *)(wt + pl.nel);
    for (int i = tid; i < (nb >> 6) * Rmax * TMAX; i += nb) acc[i] = 0.0;
    acc += wave * Rmax * TMAX;
    for (TileWalk u(pl.nunits, 1); u.ok(); u.next()) {
        const int unit = u.tile();
        const int mu = unit >= pl.d[2].unit0 ? 2 : unit >= pl.d[1].unit0 ? 1 : 0;
        const WDir D = mu == 2 ? pl.d[2] : mu == 1 ? pl.d[1] : pl.d[0];
        int v = unit - D.unit0;
        const int tc = v % D.ntc;
        v /= D.ntc;
        const int xc = v % D.nxc, grp = v / D.nxc;
        const int t0 = tc * D.TC, x0 = xc * D.XC, rows = min(D.TC, d.n[3] - t0), W = D.G * D.XE;
        const int nrow = D.NB * NC, off = min(pl.toff, nrow - 1), nel = W * (nrow + off + TMAX), ke = (nel + nb - 1) / nb;
        const float iW = 1.0f / (float)W, iX = 1.0f / (float)D.XE;
        const long long first = (long long)mu * d.ns * next;
        const Q<T> *Lm = L + first;
        const T *wm = w + first;

        // elements tid + k nb of this lane: Z and the LDS neighbour along mu.
        // Lanes beyond the last element repeat it into the padding.
        Q<T> Ue[KE];
        uint32_t nbr[KE / 2];  // two 16-bit indices each
#pragma unroll
        for (int k = 0; k < KE; ++k) Ue[k] = Q<T>{T(0), T(0), T(0), T(0)}, nbr[k >> 1] = 0;
#pragma unroll
        for (int k = 0; k < KE; ++k) {
            if (k < ke) {
                const int e = min(tid + k * nb, nel - 1);
                const int te = (int)(((float)e + 0.5f) * iW), gx = e - te * W;
                const int g = (int)(((float)gx + 0.5f) * iX), xi = gx - g * D.XE;
                const uint32_t up = (uint32_t)(xi + 1 < D.XE ? e + 1 : D.XE == D.XC ? e - (D.XE - 1) : e);
                nbr[k >> 1] = k & 1 ? nbr[k >> 1] | up << 16 : up;
                const int line = min(grp * D.G + g, D.lines - 1);
                const int t = min(t0 + te + (te < nrow ? 0 : pl.toff - off), next - 1);
                int xa = x0 + xi;
                while (xa >= D.N) xa -= D.N;
                const long long o = ((long long)line * next + t) * D.N + xa;
                Ue[k] = Lm[o];
                wt[tid + k * nb] = wm[o];
            }
        }
#pragma unroll
        for (int k = 0; k < KE; ++k)
            if (k < ke) Z.st(tid + k * nb, Ue[k]);
        __syncthreads();
        // P(x) U P(x+mu)^-1
#pragma unroll
        for (int k = 0; k < KE; ++k) {
            const T f = wt[k & 1 ? nbr[k >> 1] >> 16 : nbr[k >> 1] & 0xFFFFu];
            Ue[k] = qscale1p(Ue[k], f);
        }
        // rows of this lane
        const int per = D.G * D.XC, tb = (int)(((float)tid + 0.5f) * (1.0f / (float)per));
        const int gi = tid - tb * per, g = (int)(((float)gi + 0.5f) * (1.0f / (float)D.XC)), xi = gi - g * D.XC;
        const bool on = tb < D.NB && grp * D.G + g < D.lines && x0 + xi < D.N;
        const int gx = g * D.XE + xi, r0 = tb * NC;
        int gR = gx, xR = xi;  // x + R
        for (int R = 1; R <= Rmax; ++R) {
            double sum[TMAX];
#pragma unroll
            for (int k = 0; k < TMAX; ++k) sum[k] = 0.0;
            ++gR, ++xR;
            if (xR == D.XE) xR = 0, gR -= D.XE;
            if (on) {
                // opaque per R: addresses formed as they are used, not kept
                // in registers across the loop
                int o = r0 * W;
                __asm__ volatile("" : "+v"(o));
                Q<T> A[NC];
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    const Q<T> q = Z.ld(o + gx);
                    const T f = wt[o + gx], h = wt[o + gR];
                    A[j] = r0 + j < rows ? qscale1p(q, fma(f, h, f + h)) : Q<T>{T(0), T(0), T(0), T(0)};
                    o += W;
                }
                o = (r0 + off) * W + gx;
                __asm__ volatile("" : "+v"(o));
#pragma unroll
                for (int m = 1; m < NC + TMAX; ++m) {
                    o += W;
                    const Q<T> q = Z.ld(o);
#pragma unroll
                    for (int j = 0; j < NC; ++j) {
                        const int k = m - j - 1;
                        if (k >= 0 && k < TMAX) sum[k] = add_dot(sum[k], A[j], q);
                    }
                }
            }
            int which;
            const double tot = wave_sum_many<TMAX>(sum, lane, which);
            if ((lane & 12) == 0 && (TMAX > 4 || (lane & 1) == 0) && (TMAX > 8 || (lane & 2) == 0))
                acc[(R - 1) * TMAX + which] += tot;
            if (R < Rmax) {
                Q<T> n[KE];
#pragma unroll
                for (int k = 0; k < KE; ++k)
                    n[k] = Z.ld((int)(k & 1 ? nbr[k >> 1] >> 16 : nbr[k >> 1] & 0xFFFFu));
                __syncthreads();
                int e = tid;
                __asm__ volatile("" : "+v"(e));
#pragma unroll
                for (int k = 0; k < KE; ++k)
                    if (k < ke) Z.st(e + k * nb, qmul(Ue[k], n[k]));
            }
            __syncthreads();
        }
    }
    __syncthreads();
    acc -= wave * Rmax * TMAX;
    for (int i = tid; i < Rmax * pl.Tp; i += nb) {
        const int r = i / pl.Tp, k = i - r * pl.Tp;
        DD s{0.0, 0.0};
        for (int wv = 0; wv < (nb >> 6); ++wv) s = dd_add(s, DD{acc[(wv * Rmax + r) * TMAX + k], 0.0});
        double *o = part + 2 * (((long long)r * pl.Tall + pl.toff + k) * gridDim.x + blockIdx.x);
        o[0] = s.hi;
        o[1] = s.lo;
    }
}

// ---------------------------------------------------------------------------
// Wilson loops by transport: the temporal sides carried around each loop.
// Nothing is prepared but the spatial lines of the R asked for, so it is the
// shorter way for few (R, T) and for small time slices over many times
// (wloops_transport has the line between the two and figures), and its lines
// are the smaller buffer where the other is not to be had.  Spatial lines first:
// S_mu(x;R) = U_mu(x) .. U_mu(x+(R-1)mu), stored per site as Q<T> arrays
// sl[(mu*Rmax + R-1)*V + s].  `sp` / `sp_raw`: the spatial links (smeared
// buffer or raw links).  Temporal lines are not stored: the trace kernel
// builds them by transport from the raw temporal links.
template <class T>
__global__ __launch_bounds__(256) void k_wlines(KArgs a, const void *sp, int sp_raw, int Rmax, Q<T> *sl) {
    const LatDesc d = load_desc(a.desc);
    const Blocks<T, 3> Bs = blocks<T, 3>(sp, sp_raw ? d.off : d.soff, d.vh);
    const int V = 2 * d.vh;
    for_each_tile(a.ntiles, a.xcd_remap, [&](int tile) {
        const int s = tile * (int)blockDim.x + (int)threadIdx.x;
        if (s >= V) return;
        int c[4], r = s;
        udiv(r, d.n[0], d.inv_nx, r, c[0]);
        udiv(r, d.n[1], d.inv_ny, r, c[1]);
        udiv(r, d.n[2], d.inv_nz, c[3], c[2]);
#pragma unroll
        for (int mu = 0; mu < 3; ++mu) {
            const int st = mu == 0 ? 1 : mu == 1 ? d.n[0] : d.n[0] * d.n[1];
            Q<T> P = qone<T>();
            int cm = c[mu];
            for (int R = 1; R <= Rmax; ++R) {
                const int y = s + (cm - c[mu]) * st;
                const int par = (c[0] + c[1] + c[2] + c[3] - c[mu] + cm) & 1;
                P = qmul(P, lds_(Bs, mu, par, (uint32_t)y >> 1));
                sl[((long long)mu * Rmax + R - 1) * V + s] = P;
                cm = (cm + 1 == d.n[mu]) ? 0 : cm + 1;
            }
        }
    });
}

// W(R,T) partials: blockIdx.y = R-1; per site x and spatial mu the loop
// 1/2 Tr[S(x;R) T(x+R mu;T) S(x+T t;R)^dag T(x;T)^dag] = 1/2 Tr[A_T S(x+T t;R)^dag]
// with A_T = T(x;T)^dag S(x;R) T(x+R mu;T), built by transport up the two
// temporal sides: A_0 = S(x;R), A_T = U_t(x+(T-1)t)^dag A_{T-1} U_t(x+R mu+(T-1)t).
// Temporal links come from the raw link buffer, the spatial lines from sl.
//
// A lane owns a column of NC sites x_j = x_0 + j t (j < NC; NC divides Nt)
// of lattice 0 and takes the three directions mu one after another: at
// temporal offset m from x_0 every column site with step k = m - j < Tmax
// applies the same two temporal links and meets the same spatial line at
// x_0 + (m+1) t, so each is loaded once per column instead of once per site
// (NC + Tmax - 1 offsets of three loads per mu).  Column q = (spatial site
// q % Ns, t block q / Ns); column tile i is columns [i B, (i+1) B) for block
// size B.  A workgroup walks its share of the column tiles (a fixed
// assignment), each lane summing in binary64, then one compensated block sum
// per (R, workgroup, T).
template <class T, int TMAX, int NC>
__device__ __forceinline__ void wtrace_body(const KArgs &a, int Rmax, int Tmax, int ncols, int nctiles,
                                            const Q<T> *sl, double *part) {
    __shared__ DD lds[TMAX * 4];
    const int R = blockIdx.y + 1;
    double sum[TMAX];
#pragma unroll
    for (int k = 0; k < TMAX; ++k) sum[k] = 0.0;
    const LatDesc d = load_desc(a.desc);
    const Blocks<T, 4> B = blocks<T, 4>(a.links, d.off, d.vh);
    const long long V = 2LL * d.vh;
    const Q<T> *slR = sl + (long long)(R - 1) * V;
    const long long mstride = (long long)Rmax * V;
    for (TileWalk w(nctiles, a.xcd_remap); w.ok(); w.next()) {
        const int q = w.tile() * (int)blockDim.x + (int)threadIdx.x;
        if (q >= ncols) continue;
        // q = sp + Ns tb: spatial site sp = x + Nx (y + Ny z), t0 = NC tb
        int c[3], r, tb, sp;
        udiv(q, d.n[0], d.inv_nx, r, c[0]);
        udiv(r, d.n[1], d.inv_ny, r, c[1]);
        udiv(r, d.n[2], d.inv_nz, tb, c[2]);
        sp = q - tb * d.ns;
        const int t0 = NC * tb;
        const int s0 = sp + t0 * d.ns;  // site of x_0
#pragma unroll
        for (int mu = 0; mu < 3; ++mu) {
            const int st = mu == 0 ? 1 : mu == 1 ? d.n[0] : d.n[0] * d.n[1];
            int cm = c[mu] + R;
            if (cm >= d.n[mu]) cm -= d.n[mu];
            const int sR = s0 + (cm - c[mu]) * st;  // x_0 + R mu
            Q<T> A[NC];
#pragma unroll
            for (int j = 0; j < NC; ++j) A[j] = slR[mu * mstride + s0 + j * d.ns];
            // parity of x_0 + m t and of x_0 + R mu + m t (R flips it when odd)
            const int p0 = (c[0] + c[1] + c[2] + t0) & 1, pR = p0 ^ (R & 1);
            int tm = t0;  // t of x_0 + m t
#pragma unroll
            for (int m = 0; m < NC + TMAX - 1; ++m) {
                if (m < NC + Tmax - 1) {
                    const int dt = (tm - t0) * d.ns;  // x_0 + m t = s0 + dt
                    const int pm = (p0 + m) & 1, pRm = (pR + m) & 1;
                    const Q<T> ua = qdag(lds_(B, 3, pm, (uint32_t)(s0 + dt) >> 1));
                    const Q<T> ub = lds_(B, 3, pRm, (uint32_t)(sR + dt) >> 1);
                    tm = (tm + 1 == d.n[3]) ? 0 : tm + 1;
                    const Q<T> top = slR[mu * mstride + s0 + (tm - t0) * d.ns];  // S(x_0 + (m+1) t; R)
#pragma unroll
                    for (int j = 0; j < NC; ++j) {
                        const int k = m - j;
                        if (k >= 0 && k < TMAX && k < Tmax) {
                            A[j] = qmul(qmul(ua, A[j]), ub);
                            sum[k] += (double)half_tr_xyd(A[j], top);
                        }
                    }
                }
            }
        }
    }
    // Wavefront sums by binary64 butterflies in a fixed order (each lane holds
    // a plain binary64 sum; a compensated butterfly cost as much as a tenth of
    // the kernel's instructions), then the workgroup's wavefronts combined by
    // compensated sums in thread 0.
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6, nw = (int)blockDim.x >> 6;
#pragma unroll
    for (int k = 0; k < TMAX; ++k) {
        const double ws = wave_sum_f64(sum[k]);
        if (lane == 0) lds[wave * TMAX + k] = DD{ws, 0.0};
    }
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < TMAX; ++k)
            if (k < Tmax) {
                DD acc = lds[k];
                for (int w = 1; w < nw; ++w) acc = dd_add(acc, lds[w * TMAX + k]);
                double *p = part + 2 * (((long long)(R - 1) * Tmax + k) * gridDim.x + blockIdx.x);
                p[0] = acc.hi;
                p[1] = acc.lo;
            }
}

// Binary32 traces are held to 128 registers (4 waves per SIMD): under that
// bound the compiler also schedules the unrolled offsets without copying the
// binary64 sums around their run-time bounds, 10% faster at 24^3 x 48 than
// the same code unbounded (122 registers, also 4 waves).  Binary64 traces
// need more registers and run unbounded (the bound would spill).
template <int TMAX, int NC>
__global__ __launch_bounds__(256, 4) void k_wtrace(KArgs a, int Rmax, int Tmax, int ncols, int nctiles,
                                                   const Q<float> *sl, double *part) {
    wtrace_body<float, TMAX, NC>(a, Rmax, Tmax, ncols, nctiles, sl, part);
}
template <int TMAX, int NC>
__global__ __launch_bounds__(256) void k_wtrace64(KArgs a, int Rmax, int Tmax, int ncols, int nctiles,
                                                  const Q<double> *sl, double *part) {
    wtrace_body<double, TMAX, NC>(a, Rmax, Tmax, ncols, nctiles, sl, part);
}

// One block per (R, T): fixed-order sum over the workgroups'
// partials (nparts per (R, T)), written straight into mapped host memory, the
// error word and off_group with them.
__global__ __launch_bounds__(256) void k_wfinal(const LatDesc *desc, int nparts, const double *part, double *out,
                                                const DevState *st, unsigned *err) {
    __shared__ DD lds[4];
    const double2 *p = reinterpret_cast<const double2 *>(part) + (long long)blockIdx.x * nparts;
    const double vh = (double)uni(desc->vh);
    DD acc[1] = {{0.0, 0.0}};
    for (int t = threadIdx.x; t < nparts; t += blockDim.x) acc[0] = dd_add(acc[0], DD{p[t].x, p[t].y});
    dd_block_sum<1>(acc, lds);
    if (threadIdx.x == 0) {
        out[blockIdx.x] = (acc[0].hi + acc[0].lo) / (6.0 * vh);
        if (blockIdx.x == 0) {
            err[0] = st->err;
            err[1] = st->off_group;
        }
    }
}

// ---------------------------------------------------------------------------
// Launchers
static inline dim3 grid_of(const KArgs &a, int grid) {
    int g = grid > 0 ? grid : ((a.ntiles + 7) / 8) * 8;
    if (g < 8) g = 8;
    return dim3((unsigned)g);
}

// With timing events the launch itself stamps them with the kernel's own
// start and end (the dispatch's timestamps), so nothing is queued between
// the events and the kernel.
template <class K>
static void launch_ev(K kern, dim3 g, dim3 b, hipStream_t s, const Ev &ev, const KArgs &a, int par) {
    if (ev.a && ev.b) hipExtLaunchKernelGGL(kern, g, b, 0, s, ev.a, ev.b, 0, a, par);
    else hipLaunchKernelGGL(kern, g, b, 0, s, a, par);
}

template <class T, int MU, int NL>
static void launch_hb_nl(const KArgs &a, int par, int block, int grid, hipStream_t s, bool trace, bool plaq,
                         const Ev &ev) {
    const dim3 g = grid_of(a, grid), b(block);
    if (plaq) {
        if constexpr (MU >= 1) {
            if (trace) launch_ev(k_heatbath<T, MU, true, NL, true>, g, b, s, ev, a, par);
            else launch_ev(k_heatbath<T, MU, false, NL, true>, g, b, s, ev, a, par);
        }
    } else {
        if (trace) launch_ev(k_heatbath<T, MU, true, NL, false>, g, b, s, ev, a, par);
        else launch_ev(k_heatbath<T, MU, false, NL, false>, g, b, s, ev, a, par);
    }
}

template <class T, int MU>
static void launch_hb_mu(const KArgs &a, int par, int nl, int block, int grid, hipStream_t s, bool trace,
                         bool plaq, const Ev &ev) {
    switch (nl) {
    case 1: launch_hb_nl<T, MU, 1>(a, par, block, grid, s, trace, plaq, ev); break;
    case 2: launch_hb_nl<T, MU, 2>(a, par, block, grid, s, trace, plaq, ev); break;
    default: launch_hb_nl<T, MU, 4>(a, par, block, grid, s, trace, plaq, ev); break;
    }
}

template <class T, int MU>
static void launch_hb_split_mu(const KArgs &a, int par, hipStream_t s, bool plaq, const Ev &ev) {
    const dim3 g((unsigned)((a.ntiles * (a.tile_links >> 6) + 7) / 8 * 8)), b(256);
    if constexpr (MU >= 1) {
        if (plaq) return launch_ev(k_heatbath_split<T, MU, true>, g, b, s, ev, a, par);
    }
    launch_ev(k_heatbath_split<T, MU, false>, g, b, s, ev, a, par);
}

template <class T> static void launch_hb_split(const KArgs &a, int mu, int par, hipStream_t s, bool plaq, const Ev &ev) {
    switch (mu) {
    case 0: launch_hb_split_mu<T, 0>(a, par, s, false, ev); break;
    case 1: launch_hb_split_mu<T, 1>(a, par, s, plaq, ev); break;
    case 2: launch_hb_split_mu<T, 2>(a, par, s, plaq, ev); break;
    default: launch_hb_split_mu<T, 3>(a, par, s, plaq, ev); break;
    }
}

template <class T>
static void launch_hb_t(const KArgs &a, int mu, int par, int nl, int block, int grid, hipStream_t s,
                        bool trace, bool plaq, const Ev &ev) {
    switch (mu) {
    case 0: launch_hb_mu<T, 0>(a, par, nl, block, grid, s, trace, false, ev); break;
    case 1: launch_hb_mu<T, 1>(a, par, nl, block, grid, s, trace, plaq, ev); break;
    case 2: launch_hb_mu<T, 2>(a, par, nl, block, grid, s, trace, plaq, ev); break;
    default: launch_hb_mu<T, 3>(a, par, nl, block, grid, s, trace, plaq, ev); break;
    }
}

void launch_heatbath(const KArgs &a, bool f32, int mu, int par, int nl, int block, int grid, hipStream_t s,
                     bool trace, bool plaq, const Ev &ev) {
    if (a.tile_links && !trace) {
        if (f32) launch_hb_split<float>(a, mu, par, s, plaq, ev);
        else launch_hb_split<double>(a, mu, par, s, plaq, ev);
        return;
    }
    if (f32) launch_hb_t<float>(a, mu, par, nl, block, grid, s, trace, plaq, ev);
    else launch_hb_t<double>(a, mu, par, nl, block, grid, s, trace, plaq, ev);
}

template <class T, int NL> static int hb_occ(int block) {
    int best = 1 << 30;
    const void *k[4] = {(const void *)k_heatbath<T, 0, false, NL, false>, (const void *)k_heatbath<T, 1, false, NL, false>,
                        (const void *)k_heatbath<T, 2, false, NL, false>, (const void *)k_heatbath<T, 3, false, NL, false>};
    for (const void *f : k) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, block, 0) != hipSuccess) {
            (void)hipGetLastError();
            return 0;
        }
        best = n < best ? n : best;
    }
    return best;
}

int heatbath_blocks_per_cu(bool f32, int nl, int block) {
    if (f32) return nl == 1 ? hb_occ<float, 1>(block) : nl == 2 ? hb_occ<float, 2>(block) : hb_occ<float, 4>(block);
    return nl == 1 ? hb_occ<double, 1>(block) : nl == 2 ? hb_occ<double, 2>(block) : hb_occ<double, 4>(block);
}

template <class T>
static void launch_or_t(const KArgs &a, int mu, int par, int block, int grid, hipStream_t s, const Ev &ev) {
    const dim3 g = grid_of(a, grid), b((unsigned)block);
    switch (mu) {
    case 0: launch_ev(k_overrelax<T, 0>, g, b, s, ev, a, par); break;
    case 1: launch_ev(k_overrelax<T, 1>, g, b, s, ev, a, par); break;
    case 2: launch_ev(k_overrelax<T, 2>, g, b, s, ev, a, par); break;
    default: launch_ev(k_overrelax<T, 3>, g, b, s, ev, a, par); break;
    }
}

void launch_overrelax(const KArgs &a, bool f32, int mu, int par, int block, int grid, hipStream_t s, const Ev &ev) {
    if (f32) launch_or_t<float>(a, mu, par, block, grid, s, ev);
    else launch_or_t<double>(a, mu, par, block, grid, s, ev);
}

size_t small_lds_bytes(bool f32, int sites) { return (size_t)sites * (f32 ? 64 : 128); }

// Workgroups of the largest lattice's size; every one of them is resident at
// once (the caller's rule), so a run lasts as long as its slowest lattice.
bool launch_small_run(const KArgs &a, bool f32, int nlat, int sites, const SmallRun &r, double *outp, double *outl,
                      unsigned *errp, hipStream_t s) {
    const size_t lds = small_lds_bytes(f32, sites);
    const bool four = small_four(a.sampler == 1, r.over != 0);
    const int block = std::min(SMALL_BLOCK, ((four ? 4 : 1) * sites / 2 + 63) / 64 * 64);
    const bool meas = r.nm > 0;
    const auto k = f32 ? (four ? (meas ? k_small_run<float, true, true> : k_small_run<float, true, false>)
                               : (meas ? k_small_run<float, false, true> : k_small_run<float, false, false>))
                       : (four ? (meas ? k_small_run<double, true, true> : k_small_run<double, true, false>)
                               : (meas ? k_small_run<double, false, true> : k_small_run<double, false, false>));
    // the same limit from every call: it belongs to the kernel, and another
    // thread's launch may come between this one and its own
    if (lds > (48 << 10) &&
        hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)small_lds_bytes(f32, SMALL_SITES)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)nlat), dim3((unsigned)block), lds, s, a, r, outp, outl, errp);
    return true;
}

void launch_init(const KArgs &a, bool f32, int hot, int block, int grid, hipStream_t s) {
    if (f32) hipLaunchKernelGGL((k_init<float>), grid_of(a, grid), dim3(block), 0, s, a, hot);
    else hipLaunchKernelGGL((k_init<double>), grid_of(a, grid), dim3(block), 0, s, a, hot);
}

void launch_from_canon(const KArgs &a, bool f32, const double *canon, int block, hipStream_t s) {
    if (f32) hipLaunchKernelGGL((k_from_canon<float>), grid_of(a, 0), dim3(block), 0, s, a, canon);
    else hipLaunchKernelGGL((k_from_canon<double>), grid_of(a, 0), dim3(block), 0, s, a, canon);
}

void launch_to_canon(const KArgs &a, bool f32, const void *src, int ndir, double *canon, int block,
                     hipStream_t s) {
    if (f32) hipLaunchKernelGGL((k_to_canon<float>), grid_of(a, 0), dim3(block), 0, s, a, src, ndir, canon);
    else hipLaunchKernelGGL((k_to_canon<double>), grid_of(a, 0), dim3(block), 0, s, a, src, ndir, canon);
}

void launch_unit_defect(const KArgs &a, bool f32, unsigned long long *out, int block, hipStream_t s) {
    if (f32) hipLaunchKernelGGL((k_unit_defect<float>), grid_of(a, 0), dim3(block), 0, s, a, out);
    else hipLaunchKernelGGL((k_unit_defect<double>), grid_of(a, 0), dim3(block), 0, s, a, out);
}

void launch_plaquette(const KArgs &a, bool f32, double *part, int block, int grid, hipStream_t s) {
    if (f32) hipLaunchKernelGGL((k_plaquette<float, false>), grid_of(a, grid), dim3(block), 0, s, a, part, nullptr, nullptr);
    else hipLaunchKernelGGL((k_plaquette<double, false>), grid_of(a, grid), dim3(block), 0, s, a, part, nullptr, nullptr);
}

void launch_polyakov(const KArgs &a, bool f32, double *part, int block, int grid, hipStream_t s) {
    if (f32) hipLaunchKernelGGL((k_polyakov<float, false>), grid_of(a, grid), dim3(block), 0, s, a, part, nullptr, nullptr);
    else hipLaunchKernelGGL((k_polyakov<double, false>), grid_of(a, grid), dim3(block), 0, s, a, part, nullptr, nullptr);
}

void launch_plaquette_one(const KArgs &a, bool f32, int block, double *out, unsigned *err, hipStream_t s) {
    if (f32) hipLaunchKernelGGL((k_plaquette<float, true>), dim3(1), dim3(block), 0, s, a, nullptr, out, err);
    else hipLaunchKernelGGL((k_plaquette<double, true>), dim3(1), dim3(block), 0, s, a, nullptr, out, err);
}

void launch_polyakov_one(const KArgs &a, bool f32, int block, double *out, unsigned *err, hipStream_t s) {
    if (f32) hipLaunchKernelGGL((k_polyakov<float, true>), dim3(1), dim3(block), 0, s, a, nullptr, out, err);
    else hipLaunchKernelGGL((k_polyakov<double, true>), dim3(1), dim3(block), 0, s, a, nullptr, out, err);
}

void launch_finalize(const LatDesc *desc, int nlat, int chunks, const double *pp, const double *pl,
                     unsigned *cnt, double *chunk, double *outp, double *outl, long long ostride, const DevState *st,
                     unsigned *err, hipStream_t s) {
    hipLaunchKernelGGL(k_finalize, dim3((unsigned)(nlat * chunks)), dim3(256), 0, s, desc, pp, pl, cnt, chunk,
                       chunks, outp, outl, ostride, st, err);
}

void launch_series(const LatDesc *desc, int nlat, const double *pp, long long pp_stride, const double *pl,
                   long long pl_stride, int slot0, int nslots, int nsw, int C, double *chunk, double *outp,
                   double *outl, long long ostride, int out0, hipStream_t s) {
    hipLaunchKernelGGL(k_series_part, dim3((unsigned)(C * nlat), (unsigned)nsw), dim3(256), 0, s, desc, pp,
                       pp_stride, pl, pl_stride, slot0, nslots, C, chunk);
    hipLaunchKernelGGL(k_series_final, dim3((unsigned)nlat, (unsigned)nsw), dim3(64), 0, s, desc, chunk, C,
                       pp != nullptr, pl != nullptr, outp, outl, ostride, out0);
}

void launch_set_state(DevState *st, unsigned long long seed, unsigned sweep, unsigned run_base, hipStream_t s) {
    hipLaunchKernelGGL(k_set_state, dim3(1), dim3(1), 0, s, st, seed, sweep, run_base);
}

void launch_set_state_mapped(DevState *st, const unsigned *src, hipStream_t s) {
    hipLaunchKernelGGL(k_set_state_mapped, dim3(1), dim3(1), 0, s, st, (const unsigned long long *)src);
}

void launch_clear_err(DevState *st, hipStream_t s) { hipLaunchKernelGGL(k_clear_err, dim3(1), dim3(1), 0, s, st); }

void launch_err_to_host(const DevState *st, unsigned *out, hipStream_t s) {
    hipLaunchKernelGGL(k_err_to_host, dim3(1), dim3(1), 0, s, st, out);
}


void launch_ape(const KArgs &a, bool f32, const void *src, int src_raw, void *dst, double alpha, int block,
                int grid, hipStream_t s) {
    KArgs w = a;
    w.ntiles = 2 * a.ntiles;  // work items (tile, parity)
    const dim3 g = grid_of(w, grid);
    if (f32) hipLaunchKernelGGL((k_ape<float>), g, dim3(block), 0, s, a, src, src_raw, dst, (float)alpha);
    else hipLaunchKernelGGL((k_ape<double>), g, dim3(block), 0, s, a, src, src_raw, dst, alpha);
}

void launch_ape_slices(const KArgs &a, bool f32, int ns, int nt, const void *src, int src_raw, void *dst, double alpha,
                       int nsteps, hipStream_t s) {
    const size_t lds = (size_t)3 * ns * (f32 ? 16 : 32);  // 48 KiB at most
    const dim3 g((unsigned)nt), b((unsigned)((ns + 63) / 64 * 64));
    if (f32) hipLaunchKernelGGL((k_ape_slices<float>), g, b, lds, s, a, src, src_raw, dst, (float)alpha, nsteps);
    else hipLaunchKernelGGL((k_ape_slices<double>), g, b, lds, s, a, src, src_raw, dst, alpha, nsteps);
}

void launch_wgauge(const KArgs &a, bool f32, int ns, int next, void *P, hipStream_t s) {
    const dim3 g((unsigned)((ns + 63) / 64)), b(512);
    if (f32) hipLaunchKernelGGL((k_wgauge<float>), g, b, 0, s, a, next, (double2 *)P);
    else hipLaunchKernelGGL((k_wgauge<double>), g, b, 0, s, a, next, (double2 *)P);
}

void launch_wlinks(const KArgs &a, bool f32, const int *n, const void *sp, int sp_raw, int next, const void *P, void *L,
                   void *w, hipStream_t s) {
    const auto tiles = [](int k) { return (k + 31) / 32; };
    const int gx = std::min(1 << 16, tiles(n[0]) * std::max(tiles(n[1]) * n[2], tiles(n[2]) * n[1]));
    const int most = std::min(32, n[0]) * std::min(32, std::max(n[1], n[2]));
    const dim3 b((unsigned)((most + 127) / 128 * 64));  // two elements per thread
    const double2 *p = (const double2 *)P;
    // 4096 rows of the grid at most (its limit is 65535): 32768 times a launch
    for (int t = 0; t < next; t += 8 * 4096) {
        const dim3 g((unsigned)(8 * 3 * gx), (unsigned)std::min(4096, (next - t + 7) / 8));
        if (f32)
            hipLaunchKernelGGL((k_wlinks<float>), g, b, 0, s, a, sp, sp_raw, next, t, p, (Q<float> *)L, (float *)w);
        else
            hipLaunchKernelGGL((k_wlinks<double>), g, b, 0, s, a, sp, sp_raw, next, t, p, (Q<double> *)L, (double *)w);
    }
}

static int wlines_tiles(long long V, int block) { return (int)((V + block - 1) / block); }

void launch_wlines(const KArgs &arg, bool f32, long long V, const void *sp, int sp_raw, int Rmax, void *sl, int block,
                   hipStream_t s) {
    KArgs a = arg;
    a.ntiles = wlines_tiles(V, block);
    if (f32)
        hipLaunchKernelGGL((k_wlines<float>), grid_of(a, 0), dim3(block), 0, s, a, sp, sp_raw, Rmax,
                           (Q<float> *)sl);
    else
        hipLaunchKernelGGL((k_wlines<double>), grid_of(a, 0), dim3(block), 0, s, a, sp, sp_raw, Rmax,
                           (Q<double> *)sl);
}

// Workgroups per R of the Wilson trace: enough to fill the chip a few times
// over, each taking several column tiles (a multiple of 8, one share per XCD).
int wtrace_groups(long long V, int block) {
    const int g = ((wlines_tiles(V, block) + 7) / 8) * 8;
    return g < 1024 ? (g < 8 ? 8 : g) : 1024;
}

// Column height of the Wilson trace: in binary32 with up to 16 time steps,
// 6 or else 4 when it divides Nt (the same four waves per SIMD; 8 would
// spill registers); otherwise 2 (extents are even).
template <class T> static int wtrace_nc(int Nt, int Tmax) {
    if (sizeof(T) == 4 && Tmax <= 16) return Nt % 6 == 0 ? 6 : Nt % 4 == 0 ? 4 : 2;
    return 2;
}

template <class T, int NC>
static void launch_wtrace_nc(const KArgs &a, int Rmax, int Tmax, long long V, const void *sl, double *part,
                             int block, hipStream_t s) {
    const dim3 g((unsigned)wtrace_groups(V, block), (unsigned)Rmax), b((unsigned)block);
    const int ncols = (int)(V / NC), nct = (ncols + block - 1) / block;
    const Q<T> *l = (const Q<T> *)sl;
    if constexpr (sizeof(T) == 4) {
        if (Tmax <= 4) hipLaunchKernelGGL((k_wtrace<4, NC>), g, b, 0, s, a, Rmax, Tmax, ncols, nct, l, part);
        else if (Tmax <= 8) hipLaunchKernelGGL((k_wtrace<8, NC>), g, b, 0, s, a, Rmax, Tmax, ncols, nct, l, part);
        else if (Tmax <= 16) hipLaunchKernelGGL((k_wtrace<16, NC>), g, b, 0, s, a, Rmax, Tmax, ncols, nct, l, part);
        else if constexpr (NC == 2) hipLaunchKernelGGL((k_wtrace<32, NC>), g, b, 0, s, a, Rmax, Tmax, ncols, nct, l, part);
    } else {
        if (Tmax <= 4) hipLaunchKernelGGL((k_wtrace64<4, NC>), g, b, 0, s, a, Rmax, Tmax, ncols, nct, l, part);
        else if (Tmax <= 8) hipLaunchKernelGGL((k_wtrace64<8, NC>), g, b, 0, s, a, Rmax, Tmax, ncols, nct, l, part);
        else if (Tmax <= 16) hipLaunchKernelGGL((k_wtrace64<16, NC>), g, b, 0, s, a, Rmax, Tmax, ncols, nct, l, part);
        else if constexpr (NC == 2) hipLaunchKernelGGL((k_wtrace64<32, NC>), g, b, 0, s, a, Rmax, Tmax, ncols, nct, l, part);
    }
}

template <class T>
static void launch_wtrace_t(const KArgs &a, int Rmax, int Tmax, long long V, int Nt, const void *sl, double *part,
                            int block, hipStream_t s) {
    const int nc = wtrace_nc<T>(Nt, Tmax);
    if constexpr (sizeof(T) == 4) {
        if (nc == 6) return launch_wtrace_nc<T, 6>(a, Rmax, Tmax, V, sl, part, block, s);
        if (nc == 4) return launch_wtrace_nc<T, 4>(a, Rmax, Tmax, V, sl, part, block, s);
    }
    launch_wtrace_nc<T, 2>(a, Rmax, Tmax, V, sl, part, block, s);
}

void launch_wtrace(const KArgs &a, bool f32, int Rmax, int Tmax, long long V, int Nt, const void *sl, double *part,
                   int block, hipStream_t s) {
    if (f32) launch_wtrace_t<float>(a, Rmax, Tmax, V, Nt, sl, part, block, s);
    else launch_wtrace_t<double>(a, Rmax, Tmax, V, Nt, sl, part, block, s);
}

// Work split of the Wilson loops of times toff < T <= toff + Tp.  Among the
// splits that fit (elements in WL_KE per lane, rows in one per lane, LDS) it
// takes the least modelled time: wavefront instructions per R of a unit times
// its wavefronts, over the whole chip, but at least one unit's own length.
// The weights are the instruction counts of k_wloops.  A line is held whole
// unless the smallest unit of it does not fit, which takes lines of several
// hundred sites.
namespace {
constexpr int WL_LDS = 160 << 10;  // of one workgroup at most
struct WChoice {
    WPlan p;
    double cost;
    size_t lds;
};
size_t wl_bytes(bool f32, int nel, int block, int Rmax, int TM) {
    return (size_t)(nel + block - 1) / block * block * (f32 ? 20 : 40) + 8 * (size_t)(block / 64) * Rmax * TM;
}
bool wl_plan_at(bool f32, const int *n, int Rmax, int toff, int Tp, int TM, int nc, int block, size_t lds_max,
                WChoice &best) {
    WPlan p{};
    p.block = block, p.nc = nc, p.toff = toff, p.Tp = Tp;
    const int ns = n[0] * n[1] * n[2], Nt = n[3];
    const size_t sums = wl_bytes(f32, 0, block, Rmax, TM);
    if (sums >= lds_max) return false;
    // LDS elements of a unit at most
    const int cap = (int)std::min<size_t>(wl_ke(f32), (lds_max - sums) / (f32 ? 20 : 40) / block) * block;
    const auto rows = [&](int NB) { return NB * nc + std::min(toff, NB * nc - 1) + TM; };
    const double wv = block / 64, fixed = (f32 ? 6.0 : 3.0) * (nc + TM) + 4.0 * nc * TM + 8.0 * nc + 120.0;
    double cost[3], total = 0;
    for (int mu = 0; mu < 3; ++mu) {
        WDir &D = p.d[mu];
        D.N = n[mu];
        D.lines = ns / D.N;
        double dbest = 1e300;
        WDir pick{};
        const int like = n[mu] == n[0] ? 0 : n[mu] == n[1] ? 1 : 2;  // a direction with the same split
        if (like < mu) pick = p.d[like], dbest = cost[like];
        // whole lines, or for lines too long for any unit pieces of one with
        // Rmax sites beyond it
        const bool whole = D.N <= block && (long long)D.N * rows(1) <= cap;
        for (int NB = std::min(block, (Nt + nc - 1) / nc), last = 0; like == mu && NB >= 1; --NB) {
            if (whole && (D.N * NB > block || D.N * rows(NB) > cap)) continue;
            const int ntc = (Nt + NB * nc - 1) / (NB * nc);
            if (ntc == last) continue;  // the same times per unit
            last = ntc;
            const int TC = (Nt + ntc - 1) / ntc, nb = (TC + nc - 1) / nc, TE = rows(nb);
            const int XC = whole ? D.N : std::min({block / nb, cap / TE - Rmax, D.N}), XE = whole ? D.N : XC + Rmax;
            if (XC < 1) continue;
            const double per = (D.N + XC - 1) / XC * ((Nt + TC - 1) / TC);  // units per line
            for (int G = 1, ngrp = 0; G <= (whole ? std::min(D.lines, 64) : 1); ++G) {
                if (G * XC * nb > block || G * XE * TE > cap) break;
                if ((D.lines + G - 1) / G == ngrp) continue;  // as many groups of fewer lines
                ngrp = (D.lines + G - 1) / G;
                const double ke = (G * XE * TE + block - 1) / block;
                const double len = 30.0 * ke + fixed;
                const double c = std::max(ngrp * per * wv * len / 1024.0, 1.5 * len);
                if (c < dbest) {
                    dbest = c;
                    pick = D;
                    pick.XC = XC, pick.XE = XE, pick.G = G, pick.TC = TC, pick.NB = nb;
                    pick.ngrp = ngrp, pick.nxc = (D.N + XC - 1) / XC, pick.ntc = (Nt + TC - 1) / TC;
                }
            }
        }
        if (dbest >= 1e300) return false;
        pick.unit0 = p.nunits;
        D = pick;
        p.nunits += D.ngrp * D.nxc * D.ntc;
        const int e = D.G * D.XE * rows(D.NB);
        p.nel = std::max(p.nel, (e + block - 1) / block * block);
        total += cost[mu] = dbest;
    }
    if (total < best.cost) best = WChoice{p, total, wl_bytes(f32, p.nel, block, Rmax, TM)};
    return true;
}
}  // namespace

// Which way a call of the Wilson loops takes: the shorter of two estimates in us
// (V in millions of sites), fitted to 732 calls of both, in both precisions, on
// 24 lattices of 4^4 to 64^3 x 16 and 2^3 x 4096 sites, R from 1 to 12, T from 1 to
// 32.  By transport: the lines and traces of every R, cheaper where the lines of
// a few time slices stay in an L2, and a chain of Tmax steps.  In the gauge: the
// rotation of Nt + Tmax times, its bytes, its chain of 64 times at a time and its
// 32 x 32 tiles (few sites each where x and y are short), then the traces.
// us by transport and in the gauge, binary32: 64^3 x 16 156 and 343 (R = T = 1);
// 24^3 x 48 45 and 64 (R = T = 1), 59 and 68 (2), 101 and 74 (4); 8^3 x 12 32 and 31
// (2), 49 and 35 (R = 4, T = 8); 4^3 x 2048 92 and 173 (R = 4, T = 16).  Calls that
// the estimates hardly tell apart (1.04) go by transport.
bool wloops_transport(bool f32, const int *n, int Rmax, int Tmax) {
    const auto tiles = [](int k) { return (k + 31) / 32; };
    const long long slice = (long long)n[0] * n[1] * n[2];
    const double ns = 1e-6 * slice, V = ns * n[3], R = Rmax, T = Tmax, next = n[3] + Tmax;
    const double chain = (n[3] + Tmax + 63) / 64;
    const double wg = 1e-4 * next * tiles(n[0]) * std::max(tiles(n[1]) * n[2], tiles(n[2]) * n[1]);
    const bool near = slice <= 2048;
    if (f32)
        return 25.2 + R * V * (20.5 + (near ? 2.02 : 3.10) * T) + 1.84 * T <
               1.04 * (27.0 + 35.0 * ns * next + (2.77 + 234.0 * ns) * chain + R * V * (3.46 + 0.443 * T) + 1.22 * R + 25.7 * wg);
    return 24.5 + R * V * (46.9 + (near ? 5.81 : 10.3) * T) + 1.90 * T <
           1.04 * (25.4 + 61.1 * ns * next + (3.57 + 333.0 * ns) * chain + R * V * (6.63 + 0.815 * T) + 1.27 * R + 52.4 * wg);
}

bool wloops_plan(bool f32, const int *n, int Rmax, int Tmax, int toff, int step, WPlan &out) {
    const int Tp = std::min(step, Tmax - toff), TM = Tp <= 4 ? 4 : Tp <= 8 ? 8 : 16;
    WChoice best{};
    best.cost = 1e300;
    for (int block : {64, 128, 192, 256})
        for (int nc : {4, 5, 6}) wl_plan_at(f32, n, Rmax, toff, Tp, TM, nc, block, 48 << 10, best);
    if (best.cost >= 1e300) wl_plan_at(f32, n, Rmax, toff, Tp, TM, 4, 512, WL_LDS, best);
    if (best.cost >= 1e300) return false;
    out = best.p;
    out.lds = (int)best.lds;
    out.Tall = Tmax;
    // one unit per workgroup, so that the hardware evens out the last round
    // (24^3 x 48: 1728 units on 1024 resident workgroups), unless the partial
    // sums would be many
    out.grid = std::min(4096, (out.nunits + 7) / 8 * 8);
    return true;
}

template <class T, int TM, int NC>
static void launch_wloops_k(const KArgs &a, const WPlan &p, int Rmax, int next, const void *L, const void *w, double *part,
                            hipStream_t s) {
    const auto kern = k_wloops<T, TM, NC, wl_ke(sizeof(T) == 4)>;
    // the same limit from every call, as in launch_small_run; an error stays
    // for the check at the end of the call
    if (p.lds > (64 << 10))
        (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, WL_LDS);
    hipLaunchKernelGGL(kern, dim3((unsigned)p.grid), dim3((unsigned)p.block), (size_t)p.lds, s, a, p, Rmax, next,
                       (const Q<T> *)L, (const T *)w, part);
}

template <class T, int NC>
static void launch_wloops_nc(const KArgs &a, const WPlan &p, int Rmax, int next, const void *L, const void *w,
                             double *part, hipStream_t s) {
    if (p.Tp <= 4) launch_wloops_k<T, 4, NC>(a, p, Rmax, next, L, w, part, s);
    else if (p.Tp <= 8) launch_wloops_k<T, 8, NC>(a, p, Rmax, next, L, w, part, s);
    else launch_wloops_k<T, 16, NC>(a, p, Rmax, next, L, w, part, s);
}

template <class T>
static void launch_wloops_t(const KArgs &a, const WPlan &p, int Rmax, int next, const void *L, const void *w,
                            double *part, hipStream_t s) {
    if (p.nc == 6) launch_wloops_nc<T, 6>(a, p, Rmax, next, L, w, part, s);
    else if (p.nc == 5) launch_wloops_nc<T, 5>(a, p, Rmax, next, L, w, part, s);
    else launch_wloops_nc<T, 4>(a, p, Rmax, next, L, w, part, s);
}

void launch_wloops(const KArgs &a, bool f32, const WPlan &p, int Rmax, int next, const void *L, const void *w,
                   double *part, hipStream_t s) {
    if (f32) launch_wloops_t<float>(a, p, Rmax, next, L, w, part, s);
    else launch_wloops_t<double>(a, p, Rmax, next, L, w, part, s);
}

void launch_wfinal(const LatDesc *desc, int nparts, int Rmax, int Tmax, const double *part, double *out,
                   const DevState *st, unsigned *err, hipStream_t s) {
    hipLaunchKernelGGL(k_wfinal, dim3((unsigned)(Rmax * Tmax)), dim3(256), 0, s, desc, nparts, part, out, st, err);
}

}  // namespace su2
