// rr_adjoint.hip -- Gaussian log-likelihood of the population light curves
// and its hand-written adjoint: gradients with respect to every parameter
// of each row and to the shared LD profile samples.
//
//   logL_pv = -1/2 sum_t ((d_t - F_t)/sigma)^2,   psi_t = (d_t - F_t)/sigma^2
//   dlogL/dtheta = sum_t psi_t dF_t/dtheta,       F_t = 1 - mean_s delta_s
//   delta = ip(g, k) a(z, k) / I_star                               (Eq. 5)
//
//   k_adj_prep    the per-row constants, and for every block of 64 exposures
//               its time bounds and the sum of its exposures' terms with
//               F = 1, in one launch.
//   k_adjoint     one or a few workgroups of two wave64 per parameter vector,
//               each wave taking its share of the vector's in-transit
//               exposures (found through the blocks' bounds, packed 64 at a
//               time); to logL it also adds its share of the blocks outside
//               the row's windows (their sums with F = 1).  The subsample
//               loop evaluates delta together with d delta/dz and
//               d delta/dk, and z's derivatives through the transit-centred
//               Kepler solution (dE/dM = 1/(1 - e cos E),
//               dE/de = sin E/(1 - e cos E)); the lens area gives
//               da/dz = -chord and da/dk = 2 k kappa_0.  Per-lane sums are
//               FP64 and reduced in a fixed order (butterfly within the wave,
//               then waves in order) to one partial per workgroup.  With the
//               profile gradient psi-weighted lerp weights are scattered
//               into the wave's own LDS copy of d logL / d ldw (no two waves
//               share an address, and one wave's LDS additions complete in
//               program order); the copies are added in wave order and
//               stored once per workgroup, and k_adjoint_sums adds a
//               vector's workgroups in order.  Every sum therefore has an
//               order fixed by the inputs alone: the gradient is bitwise
//               reproducible.
//               Measured against the earlier form (every workgroup testing
//               a tile of 2048 exposures and evaluating the flagged ones
//               where they stood), 1024 walkers x 50 000 times x 5: float
//               132 -> 61 us, FP64 with the profile gradient 414 -> 148 us.
//   k_adjoint_sums   per parameter vector, the workgroup partials in a fixed
//               order (lanes, then a butterfly) -> logL and the gradient
//               row; the profile gradient's sums per vector, and its k-rows,
//               in the same launch.
//   k_table_grad d logL / d T[pb][i][m] from the per-vector d logL / d ldw
//               through the k-interpolation weights: chunks of vectors in
//               parallel, each in order, then the chunks in order.
//   k_ldp_grad   d logL / d ldp = sum_{i,m} W[i][j][m] dT[i][m] (fixed tree).
//   k_prof_grad  back through the profile interpolation and I_star (both
//               linear in the samples) to d logL / d I_s.
#include <algorithm>

#include "rr_device.h"

namespace rr {
namespace {

constexpr int kNq = 7;   // logL + 6 orbit parameters (k gradients follow)

// Lens area and its partial derivatives for the unit star (R = 1).
template <typename R>
__device__ inline R lens_area_grad(R k, R z, R* Az, R* Ak) {
    using N = Num<R>;
    if (z >= R(1) + k) { *Az = R(0); *Ak = R(0); return R(0); }
    if (z <= R(1) - k) { *Az = R(0); *Ak = R(2) * N::pi * k; return N::pi * k * k; }
    if (z <= k - R(1)) { *Az = R(0); *Ak = R(0); return N::pi; }
    R a = R(1), b = k, s = z, tmp;
    if (a < b) { tmp = a; a = b; b = tmp; }
    if (b < s) { tmp = b; b = s; s = tmp; }
    if (a < b) { tmp = a; a = b; b = tmp; }
    R prod = (a + (b + s)) * (s - (a - b)) * (s + (a - b)) * (a + (b - s));
    prod = prod > R(0) ? prod : R(0);
    const R area2 = R(0.5) * N::sqrt_(prod);
    const R invz = N::rcp_(z);
    const R h = area2 * invz;
    const R x1 = (z * z + (R(1) - k) * (R(1) + k)) * (R(0.5) * invz);
    const R x0 = z - x1;
    const R k1 = N::atan2_(h, x1);
    const R k0 = N::atan2_(h, x0);
    *Az = R(-2) * h;
    *Ak = R(2) * k * k0;
    return k1 + k * k * k0 - area2;
}

// Per-vector derivative constants (FP64, from the row and its PvConst).
struct PvDeriv {
    double dMtr_de, dMtr_dw, dci_da, dci_db, dci_de, dci_dw, dq_de;
};

__device__ inline PvDeriv make_pv_deriv(const PvConst& p, double b) {
    PvDeriv d;
    const double e = p.e, sw = p.sinw, cw = p.cosw, q = p.q, a = p.a;
    const double den = 1.0 + e * sw, ome2 = 1.0 - e * e;
    const double dEtr_dw = -(1.0 - e * p.cE) / q;
    const double dEtr_de = -cw / (den * q);
    d.dMtr_dw = (1.0 - e * p.cE) * dEtr_dw;
    d.dMtr_de = (1.0 - e * p.cE) * dEtr_de - p.sE;
    d.dci_da = -p.cosi / a;
    d.dci_db = den / (a * ome2);
    d.dci_de = b / a * (sw * ome2 + 2.0 * e * den) / (ome2 * ome2);
    d.dci_dw = b * e * cw / (a * ome2);
    d.dq_de = -e / q;
    return d;
}

template <typename R>
struct DerivR {
    R dMtr_de, dMtr_dw, dci_da, dci_db, dci_de, dci_dw, dq_de;
    __device__ explicit DerivR(const PvDeriv& d)
        : dMtr_de(R(d.dMtr_de)), dMtr_dw(R(d.dMtr_dw)), dci_da(R(d.dci_da)),
          dci_db(R(d.dci_db)), dci_de(R(d.dci_de)), dci_dw(R(d.dci_dw)),
          dq_de(R(d.dq_de)) {}
};

// Separation and dz/d(t0, P, a, b, e, w) for one subsample.  x = t_s - t0
// (for dM/dP = -n x / P).  Same transit-centred solve as the forward path.
template <typename R>
__device__ inline R separation_grad(R dt, R x, const OrbitR<R>& o,
                                    const DerivR<R>& dv, R invP, bool* front,
                                    R dz[6]) {
    using N = Num<R>;
    const R dM = o.n * dt;
    R s2, c2;
    if (o.e > R(0)) kepler_offset<R>(dM, o.e, o.sE, o.cE, &s2, &c2);
    else sincos_small(R(0.5) * dM, &s2, &c2);
    const R sd = R(2) * s2 * c2;
    const R cm1 = R(-2) * s2 * s2;
    const R dc = o.cE * cm1 - o.sE * sd;
    const R ds = o.sE * cm1 + o.cE * sd;
    const R X = -o.a * (dc * o.cosw - o.q * ds * o.sinw);
    const R rho = o.rtr + o.a * (dc * o.sinw + o.q * ds * o.cosw);
    const R Y = -rho * o.cosi;
    *front = rho > R(0);
    const R z = N::sqrt_(X * X + Y * Y);
    // derivatives (absolute cos E, sin E are fine here)
    const R cE = o.cE + dc, sE = o.sE + ds;
    const R iE = N::rcp_(R(1) - o.e * cE);
    const R XE = o.a * (sE * o.cosw + o.q * cE * o.sinw);
    const R rE = o.a * (o.q * cE * o.cosw - sE * o.sinw);
    const R Xe = o.a * (o.cosw + dv.dq_de * sE * o.sinw);
    const R re = o.a * (dv.dq_de * sE * o.cosw - o.sinw);
    const R inva = N::rcp_(o.a);
    const R iz = z > R(0) ? N::rcp_(z) : R(0);
    // dE/dtheta for t0, P, e, w
    const R dE_t0 = -o.n * iE;
    const R dE_P = -o.n * (x * invP) * iE;
    const R dE_e = (dv.dMtr_de + sE) * iE;
    const R dE_w = dv.dMtr_dw * iE;
    auto dzdt = [&](R dX, R drho, R dci) {
        const R dY = -o.cosi * drho - rho * dci;
        return (X * dX + Y * dY) * iz;
    };
    dz[0] = dzdt(XE * dE_t0, rE * dE_t0, R(0));
    dz[1] = dzdt(XE * dE_P, rE * dE_P, R(0));
    dz[2] = dzdt(X * inva, rho * inva, dv.dci_da);
    dz[3] = dzdt(R(0), R(0), dv.dci_db);
    dz[4] = dzdt(XE * dE_e + Xe, rE * dE_e + re, dv.dci_de);
    dz[5] = dzdt(XE * dE_w + rho, rE * dE_w - X, dv.dci_dw);
    return z;
}

template <typename T>
__device__ inline T wave_sum(T v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// sum over c = 0 .. n-1, in order, of (flag(c) ? val(c) : 0), with eight
// flags and then eight values loaded at a time (their loads are independent,
// so a flagged sum over many parts costs n/8 memory round trips, not n)
template <typename F, typename V>
__device__ inline double flagged_sum(int n, F flag, V val, bool* any = nullptr) {
    double s = 0.0;
    bool a = false;
    for (int c0 = 0; c0 < n; c0 += 8) {
        bool f[8];
        double v[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) f[b] = c0 + b < n && flag(c0 + b);
#pragma unroll
        for (int b = 0; b < 8; ++b) v[b] = f[b] ? val(c0 + b) : 0.0;
#pragma unroll
        for (int b = 0; b < 8; ++b) { s += v[b]; a = a || f[b]; }
    }
    if (any) *any = a;
    return s;
}

// Arguments of the sums after the main kernel (k_adjoint_sums).
struct AdjointSums {
    int64_t n_reduce, n_seg;                // workgroups of the first two parts
    const double* partials;
    double *logl, *grad;
    const double *seg_gw, *seg_gi;
    const int32_t* seg_flag;
    double *gldw_pv, *gist_pv;
    const double* pv;
    const PvConst* pvc;
    int32_t* kidx;
    double* kfrac;
    int32_t npv, nparts, npb, nw, npar;
};

// What every row needs before the main kernel, in one launch.  Workgroups
// [0, nrow_blocks): the per-row constants, one thread per row.  The others:
// one wave per block of kTimeBlock exposures, its bounds (block_in_window)
// and the log-likelihood of its exposures with F = 1, which the main kernel
// adds for the blocks that miss a row's windows.  A light-curve id out of
// range makes the block's sum NaN.
template <bool kF32, typename R>
__global__ __launch_bounds__(kBlock) void k_adj_prep(
    const double* __restrict__ pv, int32_t npv, int32_t npar, double k_lo, double k_hi,
    double k_small, PvConst* __restrict__ pvc, int32_t nrow_blocks,
    const double* __restrict__ times, const int32_t* __restrict__ lcids, int32_t npt, LcInfo lc,
    const R* __restrict__ obs, double inv_sig2, int32_t nblk, double* __restrict__ blk_lo,
    double* __restrict__ blk_hi, double* __restrict__ blk_ll) {
    if (int(blockIdx.x) < nrow_blocks) {
        const int ipv = int(blockIdx.x) * kBlock + int(threadIdx.x);
        if (ipv < npv)
            pvc[ipv] = make_pv_const<kF32>(pv + int64_t(ipv) * npar, npar - 6, k_lo, k_hi, k_small);
        return;
    }
    const int lane = threadIdx.x & 63;
    const int b = (int(blockIdx.x) - nrow_blocks) * (kBlock / 64) + int(threadIdx.x >> 6);
    if (b >= nblk) return;                                  // whole waves leave together
    const int it = b * kTimeBlock + lane;
    double lo = INFINITY, hi = -INFINITY, ll = 0.0;
    if (it < npt) {
        const int l = lcids ? lcids[it] : 0;
        if (l < 0 || l >= lc.nlc) {
            ll = NAN;
        } else {
            const double t = times[it], hw = 0.5 * lc.exptime[l];
            if (is_finite(t)) { lo = t - hw; hi = t + hw; }
            const double r = double(obs[it]) - 1.0;
            ll = -0.5 * r * r * inv_sig2;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, off, 64));
        hi = fmax(hi, __shfl_xor(hi, off, 64));
    }
    ll = wave_sum(ll);
    if (lane == 0) { blk_lo[b] = lo; blk_hi[b] = hi; blk_ll[b] = ll; }
}

// Workgroup ipv nparts + c: part c of row ipv's in-window exposures.  Each of
// its waves works on its own: it finds the row's blocks of exposures that
// may be in a transit from the blocks' bounds, takes every (nparts waves)-th
// of them, tests their exposures and packs the flagged ones in a ring in
// LDS, from which it evaluates 64 at a time, one per lane (all lanes busy
// until the wave's last batch).  The kernel is bound by that arithmetic, so
// full batches and no work on exposures outside a transit are what count:
// with a tile of 2048 exposures per workgroup, flagged exposures evaluated
// where they stood, the transit filled 70 % of the lanes and three quarters
// of the workgroups only added residuals.
//   logL is a sum of the exposures' own terms only: the sums of the blocks
// that miss the row's windows (64 blocks at a time, dealt to its waves in
// turn) and, in the others, each exposure's residual.  Starting from the sum
// of all blocks with F = 1 and adding what the transits change would cancel
// as (depth / sigma)^2: a relative error of 6.6e-12 for 2 % deep transits in
// 5 ppm noise, 3e-14 this way.
//   The LDS tables (ldw and its k-derivative) are built once per workgroup.
// With the profile gradient the FP64 subsample loop keeps each overlapping
// subsample's separation and area in LDS (sub_lds of them per thread;
// exposures with more, and float, where it gained only 6 %, evaluate them a
// second time), and the weighted lerp weights go to the wave's own copy of
// d logL / d ldw once the exposure's residual is known; the copies are stored
// to slot (ipv, c) of seg_gw / seg_gi with flag 1 (flag 0 and nothing else if
// no exposure was in the window), or, with seg_flag NULL (one part per vector),
// as the final per-vector sums.
//   use_ring 0 (tables that leave no LDS for the ring): a block's flagged
// exposures are evaluated where they stand.
//   Registers: with several passbands the sums of d logL / dk and d logL /
// d I_star, of which an exposure adds to one passband's, are kept per wave in
// LDS (as lane sums they took 64 vector registers for up to 16 passbands).
// FP64 then fits twice into a SIMD's registers (264 registers, once, before;
// us per call with the profile gradient, ng 96, 1024 x 50 000: five passbands
// nss 5 358 -> 271, eight 407 -> 318), and float four times, held to 128
// (four passbands spilled ten before: ng 512 nss 10 345 -> 343 with two
// passbands, 560 -> 520 with four; five at ng 96, nss 5, 303 -> 220; not held,
// 1024 x 50 000 x 5 with a profile per row and its gradient took 207 instead
// of 165).  Where the tables leave LDS for two workgroups a CU only, FP64 was
// faster with one wave per SIMD (eight passbands, ng 192, nss 5: 469 -> 526).
constexpr int kRing = 128;                    // exposures; at most 127 are held
template <typename R, bool kOne, bool kProf>
__global__ __launch_bounds__(kAdjBlock, sizeof(R) == 4 ? 4 : 2) void k_adjoint(
    const double* __restrict__ times, const int32_t* __restrict__ lcids,
    int32_t npt, LcInfo lc, const double* __restrict__ pv, int32_t npar,
    const PvConst* __restrict__ pvc, GridDev g, const R* __restrict__ T,
    const double* __restrict__ inv_istar, const R* __restrict__ obs,
    double inv_sig2, int32_t nblk, const double* __restrict__ blk_lo,
    const double* __restrict__ blk_hi, const double* __restrict__ blk_ll, int32_t nparts,
    int32_t want_grad, const double* __restrict__ wprof, double* __restrict__ partials,
    double* __restrict__ seg_gw, double* __restrict__ seg_gi, int32_t* __restrict__ seg_flag,
    int32_t rows_per_vector, int32_t use_ring, int32_t sub_lds) {
    extern __shared__ unsigned char smem_raw[];
    constexpr int kWaves = kAdjBlock / 64;
    const int npb = g.npb, ng = g.ng;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    R* ldw = reinterpret_cast<R*>(smem_raw);                    // [npb][ng]
    R* dTk = ldw + npb * ng;                                    // [npb][ng]
    // per-wave d logL / d ldw [kWaves][npb][ng] and d logL / d I_star
    // [kWaves][npb] (profile instantiation only), then each thread's
    // subsamples [sub_lds][2][kAdjBlock] and the waves' rings
    double* gw_all = reinterpret_cast<double*>(
        smem_raw + ((2 * sizeof(R) * npb * ng + 7) / 8) * 8);
    double* gw = gw_all + wave * npb * ng;                      // this wave's copy
    double* gi_all = gw_all + kWaves * npb * ng;                // [kWaves][npb]
    unsigned char* rest = reinterpret_cast<unsigned char*>(
        kProf ? gi_all + kWaves * npb : gw_all);
    R* sub = reinterpret_cast<R*>(rest) + tid;
    int32_t* ring = reinterpret_cast<int32_t*>(rest + (kProf ? 2 * sizeof(R) * sub_lds * kAdjBlock : 0)) +
                    wave * kRing;
    __shared__ double red[kWaves][kNq + (kOne ? 1 : RR_MAX_PB)];
    __shared__ int wave_any[kWaves];
    static_assert(sizeof(red) + sizeof(wave_any) <= kAdjStaticLds,
                  "static LDS must fit the reserve the host budget assumes");

    const int64_t slot = blockIdx.x;
    const int ipv = int(slot / nparts);
    const int c = int(slot - int64_t(ipv) * nparts);
    const int nq = kNq + npb;
    double* part = partials + slot * nq;
    const PvConst p = pvc[ipv];

    if (!(p.flags & kValid)) {
        if (tid < nq) part[tid] = NAN;
        if (kProf) {
            if (seg_flag) {
                if (tid == 0) seg_flag[slot] = 0;
            } else {
                for (int idx = tid; idx < npb * ng; idx += kAdjBlock)
                    seg_gw[slot * npb * ng + idx] = 0.0;
                if (tid < npb) seg_gi[slot * npb + tid] = 0.0;
            }
        }
        return;
    }

    double ll = 0.0;
    double ga[6] = {0, 0, 0, 0, 0, 0};
    double gk = 0.0, gi = 0.0;           // kOne; else red[wave] and gi_all
    if (!kOne && lane < npb) {
        red[wave][kNq + lane] = 0.0;
        if (kProf) gi_all[wave * npb + lane] = 0.0;
    }

    for (int idx = tid; idx < npb * ng; idx += kAdjBlock) {
        const int pb = idx / ng, m = idx - pb * ng;
        const double u = (pv[int64_t(ipv) * npar + 6 + pb] - g.k0) / g.dk;
        int ik = int(floor(u));
        ik = ik < 0 ? 0 : (ik > g.nk - 2 ? g.nk - 2 : ik);
        const R ak = R(u - ik);
        // the shared table's two rows, or the vector's own copies
        const R* t0r = rows_per_vector ? T + (int64_t(ipv) * npb + pb) * 2 * ng
                                       : T + (int64_t(pb) * g.nk + ik) * ng;
        ldw[idx] = (R(1) - ak) * t0r[m] + ak * t0r[ng + m];
        dTk[idx] = (t0r[ng + m] - t0r[m]) * R(g.inv_dk);
    }
    if (kProf)
        for (int idx = tid; idx < kWaves * npb * ng; idx += kAdjBlock) gw_all[idx] = 0.0;
    __syncthreads();

    const OrbitR<R> orb(p);
    const DerivR<R> dv(make_pv_deriv(p, pv[int64_t(ipv) * npar + 3]));
    const R gscale = R(g.gscale);
    const R invP = R(p.invP);

    // The wave's blocks: of the row's hit blocks, in block order, numbers
    // skip, skip + nw, skip + 2 nw, ... (wave-uniform); and of every 64 blocks
    // looked through, in turn with the other waves, the sums of those not hit.
    const int nw = nparts * kWaves;
    int skip = __builtin_amdgcn_readfirstlane(c * kWaves + wave), turn = skip, scan = 0, at = 0;
    uint64_t hits = 0;
    auto next_block = [&]() -> int {
        for (;;) {
            while (hits == 0) {
                if (scan >= nblk) return -1;
                const int b = scan + lane;
                const bool hit = b < nblk && block_in_window(blk_lo[b < nblk ? b : 0],
                                                             blk_hi[b < nblk ? b : 0], p);
                hits = __ballot(hit);
                if (turn == 0 && b < nblk && !hit) ll += blk_ll[b];
                turn = turn == 0 ? nw - 1 : turn - 1;
                at = scan;
                scan += 64;
            }
            const int bit = __builtin_ctzll(hits);
            hits &= hits - 1;
            if (skip == 0) {
                skip = nw - 1;
                return at + bit;
            }
            --skip;
        }
    };

    bool any = false;                    // an exposure was in the window (uniform)
    int head = 0, cnt = 0;
    int blk = next_block();
    double tn = 0.0;                     // the next block's times, ids and data, loaded ahead
    int ln = 0;
    R on = R(0);
    auto load_block = [&]() {
        const int it = blk * kTimeBlock + lane;
        const bool in = blk >= 0 && it < npt;
        tn = in ? times[it] : 0.0;
        ln = in && lcids ? lcids[it] : 0;
        on = in ? obs[it] : R(0);
    };
    load_block();
    for (;;) {
        int it = -1;                     // this lane's exposure
        while (blk >= 0 && cnt < 64) {
            const int cand = blk * kTimeBlock + lane;
            const double t = tn;
            const int l = ln;
            const double r0 = double(on) - 1.0;
            blk = next_block();
            load_block();
            const bool lok = l >= 0 && l < lc.nlc;
            const bool in = cand < npt && lok &&
                            in_phase_window((t - p.t0) * p.invP, p,
                                            0.5 * lc.exptime[lok ? l : 0] * p.invP);
            if (cand < npt && !in) ll += lok ? -0.5 * r0 * r0 * inv_sig2 : double(NAN);
            const uint64_t m = __ballot(in);
            if (!use_ring) {
                if (m == 0) continue;
                it = in ? cand : -1;
                any = true;
                break;
            }
            if (in) ring[(head + cnt + __popcll(m & __lanemask_lt())) & (kRing - 1)] = cand;
            cnt += __popcll(m);
        }
        if (use_ring) {
            if (cnt == 0) break;
            any = true;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int n = cnt < 64 ? cnt : 64;
            it = lane < n ? ring[(head + lane) & (kRing - 1)] : -1;
            head += n;
            cnt -= n;
            __builtin_amdgcn_wave_barrier();
        } else if (!__any(it >= 0)) {
            break;
        }
        if (it >= 0) {
            const int l = lcids ? lcids[it] : 0;
            const int pb = lc.pb[l];
            const int nss = lc.nss[l];
            const double ex = lc.exptime[l];
            const double t = times[it];
            const R k = R(pv[int64_t(ipv) * npar + 6 + pb]);
            const R onepk = R(1) + k;
            const R inv1pk = R(1) / onepk;
            const R istar_inv =
                R(inv_istar[rows_per_vector ? int64_t(ipv) * npb + pb : int64_t(pb)]);
            const R* lw = ldw + pb * ng;
            const R* dk_ = dTk + pb * ng;
            R acc = R(0);
            R gt[6] = {0, 0, 0, 0, 0, 0};
            R gkt = R(0);
            const double inv_nss = 1.0 / nss;
            const bool keep = kProf && sizeof(R) == 8 && nss <= sub_lds;
            for (int s = 0; s < nss; ++s) {
                if (keep) sub[(2 * s + 1) * kAdjBlock] = R(0);     // no overlap
                const double x = (t + ex * ((s + 0.5) * inv_nss - 0.5)) - p.t0;
                const double u = x * p.invP;
                if (!in_phase_window(u, p, 0.0)) continue;
                const double dt = x - p.P * rint(u);
                bool front;
                R dz[6];
                const R z = separation_grad<R>(R(dt), R(x), orb, dv, invP, &front, dz);
                if (!front || !(z < onepk)) continue;
                const R v = z * inv1pk * gscale;
                int m = int(v);
                m = m > ng - 2 ? ng - 2 : m;
                const R al = v - R(m);
                const R ip = (R(1) - al) * lw[m] + al * lw[m + 1];
                R Az, Ak;
                const R A = lens_area_grad<R>(k, z, &Az, &Ak);
                if (keep) {
                    sub[2 * s * kAdjBlock] = z;
                    sub[(2 * s + 1) * kAdjBlock] = A;
                }
                acc += ip * A * istar_inv;
                if (want_grad) {
                    const R slope = (lw[m + 1] - lw[m]) * gscale;
                    const R ddz = (slope * inv1pk * A + ip * Az) * istar_inv;
                    const R ipk = slope * (-z * inv1pk * inv1pk) +
                                  (R(1) - al) * dk_[m] + al * dk_[m + 1];
                    gkt += (ipk * A + ip * Ak) * istar_inv;
#pragma unroll
                    for (int q = 0; q < 6; ++q) gt[q] += ddz * dz[q];
                }
            }
            // residual in FP64: d - F = (d - 1) + mean delta
            const double mean_delta = double(acc) / nss;
            const double r = (double(obs[it]) - 1.0) + mean_delta;
            ll -= 0.5 * r * r * inv_sig2;
            const double wgt = -(r * inv_sig2) / nss;       // dlogL / d delta_s
            if (want_grad) {
#pragma unroll
                for (int q = 0; q < 6; ++q) ga[q] += wgt * double(gt[q]);
                if (kOne) gk += wgt * double(gkt);
                else atomicAdd(&red[wave][kNq + pb], wgt * double(gkt));
            }
            if (kProf) {
                // psi-weighted lerp weights of each overlapping subsample
                const double cw = wgt * (wprof ? wprof[ipv] : 1.0);
                double git = 0.0;
                for (int s = 0; s < nss; ++s) {
                    R z, area;
                    if (keep) {
                        area = sub[(2 * s + 1) * kAdjBlock];
                        if (area == R(0)) continue;
                        z = sub[2 * s * kAdjBlock];
                    } else {
                        const double x = (t + ex * ((s + 0.5) * inv_nss - 0.5)) - p.t0;
                        const double u = x * p.invP;
                        if (!in_phase_window(u, p, 0.0)) continue;
                        const double dt = x - p.P * rint(u);
                        bool front;
                        z = separation<R>(R(dt), orb, &front);
                        if (!front || !(z < onepk)) continue;
                        area = lens_area<R>(R(1), k, z);
                    }
                    const R v = z * inv1pk * gscale;
                    int m = int(v);
                    m = m > ng - 2 ? ng - 2 : m;
                    const double al = double(v - R(m));
                    const double A = double(area) * double(istar_inv);
                    const double cc = cw * A;
                    atomicAdd(&gw[pb * ng + m], (1.0 - al) * cc);
                    atomicAdd(&gw[pb * ng + m + 1], al * cc);
                    const double ip = (1.0 - al) * double(lw[m]) + al * double(lw[m + 1]);
                    git -= cw * ip * A * double(istar_inv);
                }
                if (kOne) gi += git;
                else atomicAdd(&gi_all[wave * npb + pb], git);
            }
        }
    }

    // fixed-order reduction of the per-lane sums: butterfly within the wave,
    // then the waves in order
    if (lane == 0) wave_any[wave] = any;
    double vals[kNq + 1];
    vals[0] = ll;
#pragma unroll
    for (int q = 0; q < 6; ++q) vals[1 + q] = ga[q];
    vals[kNq] = gk;
#pragma unroll
    for (int q = 0; q < (kOne ? kNq + 1 : kNq); ++q) {
        const double v = wave_sum(vals[q]);
        if (lane == 0) red[wave][q] = v;
    }
    if (kProf && kOne) {
        const double v = wave_sum(gi);
        if (lane == 0) gi_all[wave] = v;
    }
    __syncthreads();                     // also: every wave's LDS additions done
    if (tid < nq) {
        double sum = 0.0;
        for (int w = 0; w < kWaves; ++w) sum += red[w][tid];
        part[tid] = sum;
    }
    if (kProf) {
        bool ready = false;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) ready = ready || wave_any[w] != 0;
        if (seg_flag && tid == 0) seg_flag[slot] = ready ? 1 : 0;
        if (seg_flag && !ready) return;
        // the waves' copies added in wave order
        auto wsum = [&](const double* base, int stride, int idx) {
            double v = base[idx];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) v += base[w * stride + idx];
            return v;
        };
        double* out = seg_gw + slot * npb * ng;
        for (int idx = tid; idx < npb * ng; idx += kAdjBlock) out[idx] = wsum(gw_all, npb * ng, idx);
        if (tid < npb) seg_gi[slot * npb + tid] = wsum(gi_all, npb, tid);
    }
}

// d logL / d ldw_row and d logL / d I_star per vector: the flagged parts of
// k_adjoint added in part order.  idx < npv nw sums one ldw entry, the next
// npv npb one I_star entry each.
__device__ inline void prof_seg_sum(int64_t idx, const AdjointSums& a) {
    const int64_t n1 = int64_t(a.npv) * a.nw;
    const int nseg = a.nparts;
    if (idx < n1) {
        const int64_t ipv = idx / a.nw, e = idx - ipv * a.nw;
        a.gldw_pv[idx] = flagged_sum(
            nseg, [&](int sg) { return a.seg_flag[ipv * nseg + sg] != 0; },
            [&](int sg) { return a.seg_gw[(ipv * nseg + sg) * a.nw + e]; });
    } else if (idx < n1 + int64_t(a.npv) * a.npb) {
        const int64_t j = idx - n1, ipv = j / a.npb, pb = j - ipv * a.npb;
        a.gist_pv[j] = flagged_sum(
            nseg, [&](int sg) { return a.seg_flag[ipv * nseg + sg] != 0; },
            [&](int sg) { return a.seg_gi[(ipv * nseg + sg) * a.npb + pb]; });
    }
}

__global__ void k_fill(double* __restrict__ p, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

// One wave per (row, quantity): lane l sums the partials of parts l, l + 64,
// ... in order, then a fixed butterfly across the lanes.
__device__ inline void adjoint_reduce(int64_t wv, const AdjointSums& a) {
    const int nq = kNq + a.npb;
    const int lane = threadIdx.x & 63;
    if (wv >= int64_t(a.npv) * nq) return;               // whole waves leave together
    const int ipv = int(wv / nq), q = int(wv - int64_t(ipv) * nq);
    double s = 0.0;
    for (int c = lane; c < a.nparts; c += 64)
        s += a.partials[(int64_t(ipv) * a.nparts + c) * nq + q];
    s = wave_sum(s);
    if (lane != 0) return;
    if (q == 0) {
        if (a.logl) a.logl[ipv] = s;
    } else if (a.grad) {
        a.grad[int64_t(ipv) * (6 + a.npb) + (q - 1)] = s;
    }
}

// k-row index and lerp weight of every (row, passband) for the table
// gradient: kidx = ik (kNoRow for an invalid row, so that neither ik nor
// ik + 1 matches any k-row), kfrac = ak.
constexpr int kNoRow = -2;
__device__ inline void row_kidx(int64_t idx, const AdjointSums& a, const GridDev& g) {
    if (idx >= int64_t(a.npv) * a.npb) return;
    const int ipv = int(idx / a.npb), pb = int(idx - int64_t(ipv) * a.npb);
    if (!(a.pvc[ipv].flags & kValid)) {
        a.kidx[idx] = kNoRow;
        a.kfrac[idx] = 0.0;
        return;
    }
    const double u = (a.pv[int64_t(ipv) * a.npar + 6 + pb] - g.k0) / g.dk;
    int ik = int(floor(u));
    ik = ik < 0 ? 0 : (ik > g.nk - 2 ? g.nk - 2 : ik);
    a.kidx[idx] = ik;
    a.kfrac[idx] = u - ik;
}

// The sums that follow k_adjoint, in one launch (each costs about 5 us of
// launch and memory latency by itself, whatever it sums): workgroups
// [0, n_reduce) adjoint_reduce, the next n_seg prof_seg_sum, the rest row_kidx.
__global__ void k_adjoint_sums(AdjointSums a, GridDev g) {
    int64_t b = blockIdx.x;
    if (b < a.n_reduce) {
        adjoint_reduce((b * blockDim.x + threadIdx.x) >> 6, a);
        return;
    }
    b -= a.n_reduce;
    if (b < a.n_seg) {
        prof_seg_sum(b * blockDim.x + threadIdx.x, a);
        return;
    }
    row_kidx((b - a.n_seg) * blockDim.x + threadIdx.x, a, g);
}

// dlogL/dT[pb][i][m] = sum over rows of [(ik == i)(1 - ak) + (ik + 1 == i) ak]
// dlogL/dldw_row[pb][m], in two fixed-order stages.  Workgroup (x, i, c npb +
// pb), x a block of m, sums the rows of chunk c in row order; each wave reads
// the k-rows of 64 rows at a time and visits only those touching k-row i (a
// ballot), with eight loads in flight.  A chunk with no such row writes only
// its flag.  k_table_grad_sum then adds the flagged chunks in order.
__global__ void k_table_grad(const double* __restrict__ gldw_pv,
                             const int32_t* __restrict__ kidx, const double* __restrict__ kfrac,
                             int32_t npv, int32_t rows_per_chunk, GridDev g,
                             double* __restrict__ part, int32_t* __restrict__ flags) {
    const int c = int(blockIdx.z) / g.npb, pb = int(blockIdx.z) - c * g.npb, i = int(blockIdx.y);
    const int m = int(blockIdx.x) * kBlock + int(threadIdx.x);
    const int lane = threadIdx.x & 63;
    const int r0 = c * rows_per_chunk;
    const int r1 = min(npv, r0 + rows_per_chunk);
    double s = 0.0;
    bool touched = false;
    for (int base = r0; base < r1; base += 64) {
        const int r = base + lane;
        const int ik = r < r1 ? kidx[int64_t(r) * g.npb + pb] : kNoRow;
        const double ak = r < r1 ? kfrac[int64_t(r) * g.npb + pb] : 0.0;
        uint64_t hit = __ballot(ik == i || ik + 1 == i);
        touched = touched || hit != 0;
        while (hit) {
            // up to 8 hits at a time: their loads are issued together, the
            // sum still runs in row order
            constexpr int kB = 8;
            int qs[kB];
            int n = 0;
#pragma unroll
            for (int b = 0; b < kB; ++b) {
                qs[b] = hit ? __builtin_ctzll(hit) : 0;
                n += hit ? 1 : 0;
                hit &= hit - 1;
            }
            double wv[kB], gv[kB];
#pragma unroll
            for (int b = 0; b < kB; ++b) {
                const int ikq = __shfl(ik, qs[b]);
                const double akq = __shfl(ak, qs[b]);
                wv[b] = (ikq == i) ? 1.0 - akq : akq;
                gv[b] = (b < n && m < g.ng)
                            ? gldw_pv[(int64_t(base + qs[b]) * g.npb + pb) * g.ng + m] : 0.0;
            }
#pragma unroll
            for (int b = 0; b < kB; ++b)
                if (b < n) s += wv[b] * gv[b];
        }
    }
    const int64_t slot = (int64_t(c) * g.npb + pb) * g.nk + i;
    if (blockIdx.x == 0 && threadIdx.x == 0) flags[slot] = touched ? 1 : 0;
    if (touched && m < g.ng) part[slot * g.ng + m] = s;
}

// GT = the flagged chunk partials in chunk order; rowflag[pb nk + i] = 1 if
// any chunk touched k-row i (k_ldp_grad skips the other rows).
__global__ void k_table_grad_sum(const double* __restrict__ part,
                                 const int32_t* __restrict__ flags, int32_t nchunks, GridDev g,
                                 double* __restrict__ GT, int32_t* __restrict__ rowflag) {
    const int64_t per = int64_t(g.npb) * g.nk * g.ng;
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= per) return;
    const int64_t row = idx / g.ng;                       // pb nk + i
    bool any;
    GT[idx] = flagged_sum(
        nchunks, [&](int c) { return flags[int64_t(c) * g.npb * g.nk + row] != 0; },
        [&](int c) { return part[int64_t(c) * per + idx]; }, &any);
    if (idx - row * g.ng == 0) rowflag[row] = any ? 1 : 0;
}

// dlogL/dldp[pb][j] = sum_{i,m} W[i][j][m] dlogL/dT[pb][i][m], in two fixed-
// order stages: workgroup (c, j, pb) sums the k-rows of chunk c with a
// fixed-shape tree, then k_prof_grad adds the chunks in order.
constexpr int kLdpChunks = 16;
__global__ void k_ldp_grad(const double* __restrict__ W, const double* __restrict__ GT,
                           const int32_t* __restrict__ rowflag, GridDev g,
                           double* __restrict__ part_out) {
    __shared__ double part[kBlock];
    const int c = blockIdx.x;
    const int j = int(blockIdx.y), pb = int(blockIdx.z);
    const int per_chunk = (g.nk + kLdpChunks - 1) / kLdpChunks;
    const int i0 = c * per_chunk, i1 = min(g.nk, i0 + per_chunk);
    const int64_t per = int64_t(g.nk) * g.ng;
    double s = 0.0;
    for (int i = i0; i < i1; ++i) {
        if (!rowflag[pb * g.nk + i]) continue;          // GT row i is zero
        for (int m = threadIdx.x; m < g.ng; m += kBlock)
            s += W[(int64_t(i) * g.nz + j) * g.ng + m] * GT[pb * per + int64_t(i) * g.ng + m];
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part_out[(int64_t(pb) * g.nz + j) * kLdpChunks + c] = part[0];
}

// Profile gradient: chain dlogL/dldp (profile at the bin means, linear in
// the samples with the weights of the piecewise-linear interpolant) and
// dlogL/dI_star (I_star linear in the samples, Eq. 2 / Eq. 4) back to the
// samples prof[pb][s].  Workgroup (x, pb) handles samples x 256 .. + 255 of
// passband pb.  It walks the bins in chunks of kJChunk: for every bin j of
// the chunk it tabulates in LDS the interpolation segment of mu_j (a binary
// search over the samples, staged in LDS when there are at most kMuLds of
// them) and dlogL/dldp[pb][j]; then each thread adds its sample's weights
// times dlogL/dldp over the chunk's bins in order (only the run of bins that
// interpolate from its sample).
//   kShared (one profile for all rows): dlogL/dldp is the sum of k_ldp_grad's
// chunks in order and dlogL/dI_star the sum over the valid rows, in a fixed
// tree that every workgroup of a passband repeats, which costs less than the
// two launches it replaces; grad_istar, if given, gets the latter.
constexpr int kJChunk = 1024;
constexpr int kMuLds = 1024;
template <bool kShared>
__global__ __launch_bounds__(kBlock) void k_prof_grad(
    const double* __restrict__ gldp, const double* __restrict__ gist_pv, int32_t npv,
    const PvConst* __restrict__ pvc, const double* __restrict__ mu_s, int32_t nmu,
    const double* __restrict__ zm, int32_t nz, int32_t npb, int32_t istar_fixed,
    double* __restrict__ grad_istar, double* __restrict__ out) {
    __shared__ int seg_lo[kJChunk];
    __shared__ double seg_tau[kJChunk];
    __shared__ double gl[kJChunk];
    __shared__ double mu_l[kMuLds];
    const int pb = blockIdx.y;
    double gist = kShared ? 0.0 : gist_pv[pb];
    if (kShared) {
        __shared__ double part[kBlock];
        for (int ipv = threadIdx.x; ipv < npv; ipv += kBlock)
            if (pvc[ipv].flags & kValid) gist += gist_pv[int64_t(ipv) * npb + pb];
        part[threadIdx.x] = gist;
        __syncthreads();
        for (int w = kBlock / 2; w > 0; w >>= 1) {
            if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
            __syncthreads();
        }
        gist = part[0];
        if (grad_istar && blockIdx.x == 0 && threadIdx.x == 0) grad_istar[pb] = gist;
        if (!out) return;
    }
    const int s = int(blockIdx.x) * kBlock + int(threadIdx.x);
    const bool staged = nmu <= kMuLds;
    if (staged)
        for (int i = threadIdx.x; i < nmu; i += kBlock) mu_l[i] = mu_s[i];
    __syncthreads();
    const double* ms = staged ? mu_l : mu_s;
    double acc = 0.0;
    for (int j0 = 0; j0 < nz; j0 += kJChunk) {
        const int jn = min(kJChunk, nz - j0);
        for (int jj = threadIdx.x; jj < jn; jj += kBlock) {
            const double z = zm[j0 + jj];
            const double mu = sqrt(1.0 - z * z);
            int lo;
            double tau;
            if (mu <= ms[0]) {
                lo = -1; tau = 0.0;                     // weight 1 on sample 0
            } else if (mu >= ms[nmu - 1]) {
                lo = nmu - 1; tau = 1.0;                // weight 1 on sample nmu - 1
            } else {
                int a = 0, b = nmu - 1;
                while (b - a > 1) {
                    const int mid = (a + b) >> 1;
                    if (ms[mid] <= mu) a = mid; else b = mid;
                }
                lo = a;
                tau = (mu - ms[a]) / (ms[a + 1] - ms[a]);
            }
            seg_lo[jj] = lo;
            seg_tau[jj] = tau;
            const int64_t j = int64_t(pb) * nz + j0 + jj;
            double sum = kShared ? 0.0 : gldp[j];
            if (kShared)
                for (int c = 0; c < kLdpChunks; ++c) sum += gldp[j * kLdpChunks + c];
            gl[jj] = sum;
        }
        __syncthreads();
        if (s < nmu) {
            // mu_j decreases with j, so seg_lo is non-increasing in j and
            // the bins with a nonzero weight for sample s (seg_lo in
            // {s - 1, s}) are one contiguous run: two binary searches find
            // it, and the run is added in bin order
            int lo_i = 0, hi_i = jn;
            while (lo_i < hi_i) {                       // first bin with seg_lo <= s
                const int mid = (lo_i + hi_i) >> 1;
                if (seg_lo[mid] <= s) hi_i = mid; else lo_i = mid + 1;
            }
            const int ja = lo_i;
            hi_i = jn;
            while (lo_i < hi_i) {                       // first bin with seg_lo < s - 1
                const int mid = (lo_i + hi_i) >> 1;
                if (seg_lo[mid] < s - 1) hi_i = mid; else lo_i = mid + 1;
            }
            for (int jj = ja; jj < lo_i; ++jj) {
                const int lo = seg_lo[jj];
                // lo == s: 1 - tau (1 for the last sample); lo == s - 1: tau
                // (1 for sample 0, whose run holds the bins below mu_s[0])
                const double w = lo == s ? (s == nmu - 1 ? 1.0 : 1.0 - seg_tau[jj])
                                         : (s == 0 ? 1.0 : seg_tau[jj]);
                if (w != 0.0) acc += w * gl[jj];
            }
        }
        __syncthreads();
    }
    if (s >= nmu) return;
    // I_star weight of sample s
    double qs = 0.0;
    if (s < nmu - 1) {
        const double ma = ms[s], mb = ms[s + 1];
        qs += (mb - ma) / 6.0 * (2.0 * ma + mb);
    }
    if (s > 0) {
        const double ma = ms[s - 1], mb = ms[s];
        qs += (mb - ma) / 6.0 * (ma + 2.0 * mb);
    }
    if (s == 0) qs += 0.5 * ms[0] * ms[0];
    if (s == nmu - 1) qs += 0.5 * (1.0 - ms[nmu - 1] * ms[nmu - 1]);
    qs *= 2.0 * Num<double>::pi;
    // a normaliser set by the caller does not depend on the samples
    out[int64_t(pb) * nmu + s] = istar_fixed ? acc : acc + qs * gist;
}

inline unsigned nblocks(int64_t n) { return unsigned((n + kBlock - 1) / kBlock); }

template <typename R, bool kOne, bool kProf>
void launch_adjoint_t(const AdjointArgs& A, size_t lds, hipStream_t s, const KernelEvents& ev) {
    // one part per vector: the profile sums are final and go to gldw_pv
    const bool one = A.nparts == 1;
    launch_timed(k_adjoint<R, kOne, kProf>, dim3(unsigned(int64_t(A.nparts) * A.npv)),
                 dim3(kAdjBlock), lds, s, ev.before, ev.after, A.times, A.lcids, A.npt, *A.lc,
                 A.pv, A.npar, A.pvc, A.g, static_cast<const R*>(A.T), A.inv_istar,
                 static_cast<const R*>(A.obs), A.inv_sig2, A.nblk, A.blk_lo, A.blk_hi, A.blk_ll, A.nparts,
                 A.want_grad, A.wprof, A.partials, one ? A.gldw_pv : A.seg_gw,
                 one ? A.gist_pv : A.seg_gi, one ? nullptr : A.seg_flag, A.rows_per_vector,
                 A.use_ring, A.sub_lds);
}

template <typename R>
void launch_adjoint_r(const AdjointArgs& A, size_t lds, hipStream_t s, const KernelEvents& ev) {
    const bool one = A.g.npb == 1;
    if (A.want_prof) {
        if (one) launch_adjoint_t<R, true, true>(A, lds, s, ev);
        else launch_adjoint_t<R, false, true>(A, lds, s, ev);
    } else {
        if (one) launch_adjoint_t<R, true, false>(A, lds, s, ev);
        else launch_adjoint_t<R, false, false>(A, lds, s, ev);
    }
}

}  // namespace

hipError_t launch_fill(double* p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3(nblocks(n)), dim3(kBlock), 0, s, p, n);
    return hipGetLastError();
}

size_t adjoint_lds_bytes(int32_t precision, int32_t npb, int32_t ng, bool prof) {
    const size_t elt = precision == RR_FP64 ? sizeof(double) : sizeof(float);
    const size_t tables = ((2 * elt * size_t(npb) * ng + 7) / 8) * 8;
    if (!prof) return tables;
    return tables + sizeof(double) * (kAdjBlock / 64) * (size_t(npb) * ng + npb);
}

size_t adjoint_plan_lds(int32_t precision, size_t lds_max, AdjointArgs* A) {
    const size_t elt = precision == RR_FP64 ? sizeof(double) : sizeof(float);
    size_t lds = adjoint_lds_bytes(precision, A->g.npb, A->g.ng, A->want_prof != 0);
    const size_t ring = sizeof(int32_t) * kRing * (kAdjBlock / 64);
    A->use_ring = lds + ring + kAdjStaticLds <= lds_max ? 1 : 0;
    lds += A->use_ring ? ring : 0;
    A->sub_lds = 0;
    if (A->want_prof && precision == RR_FP64) {
        // As many subsamples as the largest exposure with at most kSubLds has,
        // unless that halves the workgroups a CU holds (its registers allow
        // four).  us per call, FP64, 1024 x 50 000 at nss 10, kept and evaluated
        // again: two passbands, ng 512 (four workgroups or two) 613, 500; four,
        // ng 512 (two, one) 1022, 1008, and 326, 272 for 100 rows; four, ng 192
        // (four, three) 534, 522, 172 and 197; eight, ng 192 (three, two) 756, 893.
        const size_t per = 2 * elt * kAdjBlock;             // one subsample of every thread
        auto resident = [&](int32_t n) {
            return std::min<size_t>(4, lds_max / (lds + kAdjStaticLds + size_t(n) * per));
        };
        for (int l = 0; l < A->lc->nlc; ++l) {
            const int32_t n = A->lc->nss[l];
            if (n <= kSubLds && 2 * resident(n) > resident(0)) A->sub_lds = std::max(A->sub_lds, n);
        }
        lds += size_t(A->sub_lds) * per;
    }
    return lds;
}

template <typename R>
void launch_prep_r(const AdjointArgs& A, double k_lo, double k_hi, double k_small, hipStream_t s) {
    const unsigned rows = nblocks(A.npv);
    const unsigned tb = unsigned((A.nblk + kBlock / 64 - 1) / (kBlock / 64));
    hipLaunchKernelGGL((k_adj_prep<sizeof(R) == 4, R>), dim3(rows + tb), dim3(kBlock), 0, s, A.pv,
                       A.npv, A.npar, k_lo, k_hi, k_small, const_cast<PvConst*>(A.pvc),
                       int32_t(rows), A.times, A.lcids, A.npt, *A.lc,
                       static_cast<const R*>(A.obs), A.inv_sig2, A.nblk, A.blk_lo, A.blk_hi,
                       A.blk_ll);
}

hipError_t launch_adjoint_prep(const AdjointArgs& A, int32_t precision, double k_lo, double k_hi,
                               double k_small, hipStream_t s) {
    if (precision == RR_FP64) launch_prep_r<double>(A, k_lo, k_hi, k_small, s);
    else launch_prep_r<float>(A, k_lo, k_hi, k_small, s);
    return hipGetLastError();
}

hipError_t launch_adjoint(const AdjointArgs& A, size_t lds, int32_t precision, hipStream_t s) {
    const KernelEvents ev = kernel_events();
    if (precision == RR_FP64) launch_adjoint_r<double>(A, lds, s, ev);
    else launch_adjoint_r<float>(A, lds, s, ev);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    AdjointSums u = {};
    u.npv = A.npv; u.nparts = A.nparts; u.npb = A.g.npb; u.nw = A.g.npb * A.g.ng;
    u.npar = A.npar;
    u.partials = A.partials; u.logl = A.logl; u.grad = A.grad;
    u.seg_gw = A.seg_gw; u.seg_gi = A.seg_gi; u.seg_flag = A.seg_flag;
    u.gldw_pv = A.gldw_pv; u.gist_pv = A.gist_pv;
    u.pv = A.pv; u.pvc = A.pvc; u.kidx = A.kidx; u.kfrac = A.kfrac;
    u.n_reduce = nblocks(int64_t(A.npv) * (kNq + A.g.npb) * 64);
    u.n_seg = A.want_prof && A.nparts > 1 ? nblocks(int64_t(A.npv) * (u.nw + A.g.npb)) : 0;
    const int64_t n_kidx = A.kidx ? nblocks(int64_t(A.npv) * A.g.npb) : 0;
    hipLaunchKernelGGL(k_adjoint_sums, dim3(unsigned(u.n_reduce + u.n_seg + n_kidx)),
                       dim3(kBlock), 0, s, u, A.g);
    return hipGetLastError();
}

// Per-vector LD: dlogL/dldp_r[j] = sum_m (W[ik][j][m] (1 - ak) +
// W[ik+1][j][m] ak) dlogL/dldw_r[m] for row r = (vector, passband): the
// transpose of the row's k-interpolated T = W . l, in the same two parts as
// k_pv_tables (matrix cores for tiles of 16 sorted rows on few k-rows, else
// row by row) and for the same reason bound by its loads of W: 16-byte loads,
// the nodes split over a workgroup's waves, nodes below every row's
// lowest_node (whose gradient is zero) left out.  1024 walkers, default grid,
// float: 66 us for the matrix cores with 4-byte loads that touched 16 rows
// of W each and one wave per 16 bins, and 7 us for a second launch of rows
// that found nothing to do; now 10 us together.
typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kLdpWaves = kBlock / 64;
constexpr int kLdpTileBins = 16;              // bins per matrix-core workgroup
constexpr int kLdpRowBins = 48;               // bins per single-row workgroup
// The k-weight of row r on its k-row; 0 where k is not finite (an invalid
// row: zero gradient).
__device__ inline double row_ak(const double* __restrict__ pv, int32_t npar, int64_t r, int ik,
                                const GridDev& g) {
    const int64_t ipv = r / g.npb;
    const double ak = (pv[ipv * npar + 6 + int(r - ipv * g.npb)] - g.k0) / g.dk - ik;
    return is_finite(ak) ? ak : 0.0;
}

// Tile rt, bins j0 .. j0 + 15: D[j][q] = sum_m W[ik][j][m] (1 - ak_q) g_q[m] +
// W[ik+1][j][m] ak_q g_q[m] (g_q = dlogL/dldw of row q, zero for rows on
// another k-row: selected, not multiplied, since row 0, which such a column
// loads, may hold NaN), v_mfma_f64_16x16x4f64 chains into one accumulator.  Lane l
// holds A row / B column l & 15; the k index of step u is node
// m + 4 (l >> 4) + u, so a lane's 16-byte load feeds four steps.
template <bool kVec, typename WT>
__device__ inline void pv_ldp_grad_mfma(const WT* __restrict__ W, const double* __restrict__ gldw,
                                        const double* __restrict__ pv, int32_t npar,
                                        const PvOrder& ord, int64_t nr, int32_t nz,
                                        const GridDev& g, double* __restrict__ gldp, int64_t rt,
                                        int j0, double* __restrict__ lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ka = lane >> 4, col = lane & 15;
    const int64_t pos = rt * kTileRows + col;
    const int64_t r = pos < nr ? ord.perm[pos] : -1;
    const int ik = pos < nr ? ord.key[pos] : 0x7fffffff;
    const double ak = r >= 0 ? row_ak(pv, npar, r, ik, g) : 0.0;
    const int first = wave_min(r >= 0 ? ord.mlo[r] : g.ng) / 16 * 16;
    const int jj = j0 + col < nz ? j0 + col : nz - 1;           // A row of this lane
    v4d d = {0.0, 0.0, 0.0, 0.0};
    int cur = wave_min(ik);
    while (cur != 0x7fffffff) {
        const bool take = ik == cur;
        const WT* w0 = W + (int64_t(cur) * nz + jj) * g.ng;
        const WT* w1 = w0 + int64_t(nz) * g.ng;
        const double* gr = gldw + (take ? r : 0) * g.ng;
        const double f0 = 1.0 - ak, f1 = ak;
        constexpr int kStep = 2;
        for (int m0 = first + 16 * wave; m0 < g.ng; m0 += 16 * kLdpWaves * kStep) {
            WT a0[kStep][4], a1[kStep][4];
            double b[kStep][4];
#pragma unroll
            for (int u = 0; u < kStep; ++u) {
                const int m = m0 + 16 * kLdpWaves * u + 4 * ka;
                load4<kVec>(w0, m, g.ng, a0[u]);
                load4<kVec>(w1, m, g.ng, a1[u]);
                load4<kVec>(gr, m, g.ng, b[u]);
            }
#pragma unroll
            for (int u = 0; u < kStep; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double gq = take ? b[u][q] : 0.0;
                    d = __builtin_amdgcn_mfma_f64_16x16x4f64(double(a0[u][q]), f0 * gq, d, 0, 0, 0);
                    d = __builtin_amdgcn_mfma_f64_16x16x4f64(double(a1[u][q]), f1 * gq, d, 0, 0, 0);
                }
        }
        cur = wave_min(ik > cur ? ik : 0x7fffffff);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) lds[(wave * 4 + i) * 64 + lane] = d[i];
    __syncthreads();
    static_assert(kLdpWaves == 4, "wave w finishes element w");
    double v = lds[wave * 64 + lane];
#pragma unroll
    for (int w = 1; w < kLdpWaves; ++w) v += lds[(w * 4 + wave) * 64 + lane];
    const int j = j0 + 4 * wave + ka;
    if (r >= 0 && j < nz) gldp[r * nz + j] = v;
}

// Sorted row pos, bins j0 .. j0 + kLdpRowBins - 1: one wave per bin in turn,
// lane l over nodes 4 l .. 4 l + 3 of every 256, then a fixed butterfly.
template <bool kVec, typename WT>
__device__ inline void pv_ldp_grad_row(const WT* __restrict__ W, const double* __restrict__ gldw,
                                       const double* __restrict__ pv, int32_t npar,
                                       const PvOrder& ord, int64_t pos, int32_t nz,
                                       const GridDev& g, double* __restrict__ gldp, int j0) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t r = ord.perm[pos];
    const int ik = ord.key[pos];
    const double ak = row_ak(pv, npar, r, ik, g);
    const int first = ord.mlo[r] / 4 * 4;
    const double* gr = gldw + r * g.ng;
    constexpr int kBins = 3;                  // bins of a wave in flight
    const int j1 = min(nz, j0 + kLdpRowBins);
    for (int ja = j0 + wave; ja < j1; ja += kLdpWaves * kBins) {
        double s[kBins];
#pragma unroll
        for (int u = 0; u < kBins; ++u) s[u] = 0.0;
        for (int m = first + 4 * lane; m < g.ng; m += 256) {
            double gv[4];
            WT x0[kBins][4], x1[kBins][4];
            load4<kVec>(gr, m, g.ng, gv);
#pragma unroll
            for (int u = 0; u < kBins; ++u) {
                const int j = min(ja + kLdpWaves * u, nz - 1);
                const WT* w0 = W + (int64_t(ik) * nz + j) * g.ng;
                load4<kVec>(w0, m, g.ng, x0[u]);
                load4<kVec>(w0 + int64_t(nz) * g.ng, m, g.ng, x1[u]);
            }
#pragma unroll
            for (int u = 0; u < kBins; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    s[u] += ((1.0 - ak) * double(x0[u][q]) + ak * double(x1[u][q])) * gv[q];
        }
#pragma unroll
        for (int u = 0; u < kBins; ++u) {
            const double v = wave_sum(s[u]);
            const int j = ja + kLdpWaves * u;
            if (lane == 0 && j < j1) gldp[r * nz + j] = v;
        }
    }
}

template <bool kVec, typename WT>
__global__ __launch_bounds__(kBlock) void k_pv_ldp_grad(
    const WT* __restrict__ W, const double* __restrict__ gldw, const double* __restrict__ pv,
    int32_t npar, PvOrder ord, int64_t nr, int32_t nz, GridDev g, int64_t n_mfma,
    int64_t blocks, double* __restrict__ gldp) {
    __shared__ double lds[kLdpWaves * 4 * 64];
    const int64_t b = flat_block();
    if (b >= blocks) return;
    if (b < n_mfma) {
        const int njb = (nz + kLdpTileBins - 1) / kLdpTileBins;
        const int64_t rt = b / njb;
        if (!ord.mfma[rt]) return;
        pv_ldp_grad_mfma<kVec, WT>(W, gldw, pv, npar, ord, nr, nz, g, gldp, rt,
                             int(b - rt * njb) * kLdpTileBins, lds);
        return;
    }
    const int njb = (nz + kLdpRowBins - 1) / kLdpRowBins;
    const int64_t p = b - n_mfma, pos = p / njb;
    if (ord.mfma[pos / kTileRows]) return;
    pv_ldp_grad_row<kVec, WT>(W, gldw, pv, npar, ord, pos, nz, g, gldp,
                        int(p - pos * njb) * kLdpRowBins);
}

hipError_t launch_pv_prof_grad(const rr_tables* t, const AdjointArgs& A, const PvOrder& ord,
                               double* gldp, double* out, hipStream_t s, bool w32) {
    const GridDev g = A.g;
    const int64_t nr = int64_t(A.npv) * g.npb;
    const int64_t n_mfma =
        (nr + kTileRows - 1) / kTileRows * ((t->nz + kLdpTileBins - 1) / kLdpTileBins);
    const int64_t blocks = n_mfma + nr * ((t->nz + kLdpRowBins - 1) / kLdpRowBins);
    // the transpose of the contraction that built the rows, with its weights
    auto launch = [&](auto kernel, const auto* W) {
        hipLaunchKernelGGL(kernel, flat_grid(blocks), dim3(kBlock), 0, s, W, A.gldw_pv, A.pv,
                           A.npar, ord, nr, t->nz, g, n_mfma, blocks, gldp);
    };
    const bool vec = g.ng % 4 == 0;              // 16-byte loads, as launch_pv_ld
    if (w32) launch(vec ? k_pv_ldp_grad<true, float> : k_pv_ldp_grad<false, float>, t->W32);
    else launch(vec ? k_pv_ldp_grad<true, double> : k_pv_ldp_grad<false, double>, t->W);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // the shared profile's last step with every (vector, passband) as one
    // profile: its own dlogL/dldp and dlogL/dI_star
    for (int64_t r0 = 0; r0 < nr; r0 += 65535) {
        const int32_t n = int32_t(std::min<int64_t>(65535, nr - r0));
        hipLaunchKernelGGL(k_prof_grad<false>, dim3(nblocks(t->nmu), unsigned(n)), dim3(kBlock),
                           0, s, gldp + r0 * t->nz, A.gist_pv + r0, 0, A.pvc, t->mu_s, t->nmu,
                           t->zm, t->nz, n, 0, nullptr, out + r0 * t->nmu);
    }
    return hipGetLastError();
}

hipError_t launch_profile_grad(const rr_tables* t, const AdjointArgs& A,
                               const ProfGradScratch& w, double* out, hipStream_t s) {
    const GridDev g = A.g;
    const int32_t rpc = (A.npv + w.nchunks - 1) / w.nchunks;
    hipLaunchKernelGGL(k_table_grad,
                       dim3(unsigned((g.ng + kBlock - 1) / kBlock), unsigned(g.nk),
                            unsigned(w.nchunks * g.npb)),
                       dim3(kBlock), 0, s, A.gldw_pv, A.kidx, A.kfrac, A.npv, rpc, g,
                       w.gt_part, w.gt_flags);
    hipLaunchKernelGGL(k_table_grad_sum, dim3(nblocks(int64_t(g.npb) * g.nk * g.ng)),
                       dim3(kBlock), 0, s, w.gt_part, w.gt_flags, w.nchunks, g, w.GT,
                       w.gt_rowflag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ldp_grad, dim3(unsigned(kLdpChunks), unsigned(g.nz), unsigned(g.npb)),
                       dim3(kBlock), 0, s, t->W, w.GT, w.gt_rowflag, g, w.ldp_part);
    hipLaunchKernelGGL(k_prof_grad<true>, dim3(out ? nblocks(t->nmu) : 1, unsigned(g.npb)),
                       dim3(kBlock), 0, s, w.ldp_part, A.gist_pv, A.npv, A.pvc, t->mu_s, t->nmu,
                       t->zm, t->nz, g.npb, w.istar_fixed, w.grad_istar, out);
    return hipGetLastError();
}

}  // namespace rr
