// rr_prep.hip -- table construction on the device (Sect. 2, Sect. 3.1.1,
// Sect. 3.1.2, Sect. 3.2.2).
//
//   k_zgrid     annulus edges ze[nz+1] and means zm[nz]: constant dz on
//               [0, zcut] and constant dmu on [zcut, 1] (Sect. 3.1.1);
//   k_weights   W[nk][nz][ng]: area of annulus j occluded by a planet of
//               radius k_i at separation c = g_m (1 + k_i), over the total
//               occluded area (Sect. 2); g = 1 gets the zero-overlap limit,
//               all weight in the limb annulus; g runs fastest so that the
//               table contraction below reads W coalesced;
//   k_profile   profile at the bin means, mu_m = sqrt(1 - zm^2): the
//               piecewise-linear interpolant of the samples (Sect. 3.2.2);
//   k_istar     I_star = 2 pi int_0^1 mu I(mu) dmu of that interpolant,
//               exact per segment (Eq. 2, Eq. 4), fixed-order reduction;
//   k_tables    T[pb][i][m] = sum_j W[i][j][m] ldp[pb][j] (Sect. 3.1.2), in
//               FP64 and rounded to FP32 for the mixed path.
#include <algorithm>

#include "rr_device.h"

namespace rr {
namespace {

__global__ void k_zgrid(int32_t nzin, int32_t nzlimb, double zcut,
                        double* __restrict__ ze, double* __restrict__ zm) {
    const int nz = nzin + nzlimb;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j > nz) return;
    auto edge = [&](int jj) -> double {
        if (jj < nzin) return jj * (zcut / nzin);
        if (jj == nzin) return zcut;
        if (jj == nz) return 1.0;
        const double mucut = sqrt(1.0 - zcut * zcut);
        const double mu = mucut + (jj - nzin) * ((0.0 - mucut) / nzlimb);
        return sqrt(1.0 - mu * mu);
    };
    const double e0 = edge(j);
    ze[j] = e0;
    if (j < nz) zm[j] = 0.5 * (e0 + edge(j + 1));
}

// Weight of annulus j for radius ratio k with the planet centre at c
// (Sect. 2): occluded area of the annulus over the total occluded area tot;
// at zero overlap its limit, all weight in the limb annulus.
__device__ inline double annulus_weight(const double* __restrict__ ze, int nz, int j,
                                        double k, double c, double tot) {
    if (!(tot > 0.0)) return j == nz - 1 ? 1.0 : 0.0;
    return (lens_area<double>(ze[j + 1], k, c) - lens_area<double>(ze[j], k, c)) / tot;
}

__global__ void k_weights(const double* __restrict__ ze, GridDev g,
                          double* __restrict__ W) {
    const int64_t total = int64_t(g.nk) * g.nz * g.ng;
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int m = int(idx % g.ng);
    const int64_t r = idx / g.ng;
    const int j = int(r % g.nz);
    const int i = int(r / g.nz);
    const double k = g.k0 + i * g.dk;
    const double gv = double(m) / double(g.ng - 1);
    const double c = gv * (1.0 + k);
    W[idx] = annulus_weight(ze, g.nz, j, k, c, lens_area<double>(1.0, k, c));
}

// The profile's piecewise-linear interpolant at the mean of bin j.
__device__ inline double profile_at_bin(const double* __restrict__ mu_s,
                                        const double* __restrict__ f, int32_t nmu,
                                        double z) {
    const double mu = sqrt(1.0 - z * z);
    if (mu <= mu_s[0]) return f[0];
    if (mu >= mu_s[nmu - 1]) return f[nmu - 1];
    int lo = 0, hi = nmu - 1;          // mu_s[lo] <= mu < mu_s[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (mu_s[mid] <= mu) lo = mid; else hi = mid;
    }
    const double slope = (f[lo + 1] - f[lo]) / (mu_s[lo + 1] - mu_s[lo]);
    return slope * (mu - mu_s[lo]) + f[lo];
}

__global__ void k_profile(const double* __restrict__ mu_s,
                          const double* __restrict__ prof, int32_t nmu,
                          const double* __restrict__ zm, int32_t nz,
                          int32_t npb, double* __restrict__ ldp) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= nz * npb) return;
    const int pb = idx / nz, j = idx - pb * nz;
    ldp[idx] = profile_at_bin(mu_s, prof + int64_t(pb) * nmu, nmu, zm[j]);
}

// I_star of one profile by one workgroup of kBlock threads: per-thread
// partial sums over a fixed stride, then a fixed-shape tree in LDS
// (deterministic).  Thread 0 stores I_star and 1/I_star.
__device__ inline void istar_block(const double* __restrict__ mu_s,
                                   const double* __restrict__ f, int32_t nmu,
                                   double* __restrict__ istar,
                                   double* __restrict__ inv_istar) {
    __shared__ double part[kBlock];
    double acc = 0.0;
    for (int s = threadIdx.x; s < nmu - 1; s += kBlock) {
        const double ma = mu_s[s], mb = mu_s[s + 1];
        acc += (mb - ma) / 6.0 * (f[s] * (2.0 * ma + mb) + f[s + 1] * (ma + 2.0 * mb));
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double m0 = mu_s[0], m1 = mu_s[nmu - 1];
        const double tot = part[0] + f[0] * 0.5 * m0 * m0 +
                           f[nmu - 1] * 0.5 * (1.0 - m1 * m1);
        const double is = 2.0 * Num<double>::pi * tot;
        *istar = is;
        *inv_istar = 1.0 / is;
    }
}

// One workgroup (kBlock threads) per passband.
__global__ __launch_bounds__(kBlock) void k_istar(const double* __restrict__ mu_s,
                                                  const double* __restrict__ prof, int32_t nmu,
                                                  double* __restrict__ istar,
                                                  double* __restrict__ inv_istar) {
    const int pb = blockIdx.x;
    istar_block(mu_s, prof + int64_t(pb) * nmu, nmu, istar + pb, inv_istar + pb);
}

// T = W . l for every passband, one node per thread: bound by its one read of
// W (189 MB on the default grid).  The bins are summed in order, kTableLoads of
// them loaded ahead of the sum, since a CU has only two workgroups of work here:
// 54 -> 38 us, 5.0 TB/s (6 and 20 loads ahead 37 and 38, 36 ahead 41).
constexpr int kTableLoads = 12;
__global__ __launch_bounds__(kBlock) void k_tables(const double* __restrict__ W,
                                                   const double* __restrict__ ldp, GridDev g,
                                                   double* __restrict__ T64,
                                                   float* __restrict__ T32) {
    const int64_t per = int64_t(g.nk) * g.ng;
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= per * g.npb) return;
    const int pb = int(idx / per);
    const int64_t r = idx - pb * per;
    const int i = int(r / g.ng), m = int(r - int64_t(i) * g.ng);
    const double* wrow = W + int64_t(i) * g.nz * g.ng + m;
    const double* l = ldp + int64_t(pb) * g.nz;
    double w[2][kTableLoads];
    auto load = [&](int j0, double* to) {
#pragma unroll
        for (int u = 0; u < kTableLoads; ++u)
            to[u] = wrow[int64_t(min(j0 + u, g.nz - 1)) * g.ng];
    };
    double acc = 0.0;
    auto add = [&](int j0, const double* from) {
#pragma unroll
        for (int u = 0; u < kTableLoads; ++u)
            if (j0 + u < g.nz) acc += from[u] * l[j0 + u];
    };
    load(0, w[0]);
    for (int j0 = 0; j0 < g.nz; j0 += 2 * kTableLoads) {
        load(j0 + kTableLoads, w[1]);
        add(j0, w[0]);
        load(j0 + 2 * kTableLoads, w[0]);
        add(j0 + kTableLoads, w[1]);
    }
    T64[idx] = acc;
    T32[idx] = float(acc);
}

inline unsigned nblocks(int64_t n) { return unsigned((n + kBlock - 1) / kBlock); }

}  // namespace

GridDev grid_dev(const rr_tables* t) {
    GridDev g;
    g.nz = t->nz;
    g.ng = t->grid.ng;
    g.nk = t->grid.nk;
    g.npb = t->npb;
    g.k0 = t->grid.k0;
    g.dk = t->dk;
    g.inv_dk = 1.0 / t->dk;
    g.gscale = double(t->grid.ng - 1);
    return g;
}

// FP32 copy of the weights for the mixed-precision per-vector tables.
__global__ void k_weights_f32(const double* __restrict__ W, int64_t n, float* __restrict__ W32) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) W32[i] = float(W[i]);
}

hipError_t launch_prepare_grid_weights(rr_tables* t, hipStream_t s) {
    const GridDev g = grid_dev(t);
    hipLaunchKernelGGL(k_zgrid, dim3(nblocks(t->nz + 1)), dim3(kBlock), 0, s,
                       t->grid.nzin, t->grid.nzlimb, t->grid.zcut, t->ze, t->zm);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nw = int64_t(g.nk) * g.nz * g.ng;
    hipLaunchKernelGGL(k_weights, dim3(nblocks(nw)), dim3(kBlock), 0, s, t->ze, g, t->W);
    hipLaunchKernelGGL(k_weights_f32, dim3(nblocks(nw)), dim3(kBlock), 0, s, t->W, nw, t->W32);
    return hipGetLastError();
}

// Per-vector LD rows.  Row r = (vector, passband) needs the two table rows
// T_r[s][m] = sum_j W[ik_r + s][j][m] ldp[r][j], s = 0, 1, around its k
// (Sect. 3.1.2: T = W . l, then the k-interpolation in the forward kernel).
// k_pv_prep sorts the rows by ik, so that rows with equal ik share the W
// reads of one matrix-core tile (the two parts of k_pv_tables below).
// Stable counting sort of the rows by ik, by one workgroup of kBlock
// threads: the waves (four, or as many as have a counter per key in LDS) take
// consecutive runs of the rows; each counts its keys, a scan over (key, wave)
// gives every wave its offsets, and each places its rows in row order, 64 at
// a time -- a lane's rank among the lanes with its key comes from a ballot
// per key bit -- so equal keys keep their row order and the tiles (and which
// part takes each) depend on the inputs only.  It is the launch's longest
// serial chain: for 1024 rows the launch took 13.2 us with one placing wave
// and 9.4 us with four.
// The keys of the first kSortLds rows are kept in LDS (as 16-bit values,
// nk <= 4096) for the placing loop.
constexpr int kSortLds = 8192;
constexpr int kSortCounters = 4096;
__device__ inline void sort_rows(const double* __restrict__ pv, int32_t npv, int32_t npar,
                                 const GridDev& g, const PvOrder& ord) {
    constexpr int kPer = kSortCounters / kBlock;
    __shared__ int cnt[kSortCounters];                 // [key][wave]
    __shared__ uint16_t keys[kSortLds];
    __shared__ int wsum[kBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n = int64_t(npv) * g.npb;
    int sh = 2;                                        // log2 of the waves that place
    while (sh > 0 && (g.nk << sh) > kSortCounters) --sh;
    const int nw = 1 << sh, ncnt = g.nk << sh;
    const int64_t per = ((n + nw - 1) / nw + 63) / 64 * 64;    // rows per wave
    auto key_of = [&](int64_t r) {
        const int64_t ipv = r / g.npb;
        const int pb = int(r - ipv * g.npb);
        const double u = (pv[ipv * npar + 6 + pb] - g.k0) / g.dk;
        double uf = floor(u);
        if (!(uf >= 0.0)) uf = 0.0;              // also a non-finite k (NaN row anyway)
        if (uf > g.nk - 2) uf = g.nk - 2;
        return int(uf);
    };
    for (int b = tid; b < ncnt; b += kBlock) cnt[b] = 0;
    __syncthreads();
    for (int64_t r = tid; r < n; r += kBlock) {
        const int ik = key_of(r);
        if (r < kSortLds) keys[r] = uint16_t(ik);
        atomicAdd(&cnt[(ik << sh) + int(r / per)], 1);
    }
    __syncthreads();
    int v[kPer], local = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int b = kPer * tid + q;
        v[q] = b < ncnt ? cnt[b] : 0;
        local += v[q];
    }
    int x = local;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int excl = x - local;
    for (int w = 0; w < wave; ++w) excl += wsum[w];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int b = kPer * tid + q;
        if (b < ncnt) cnt[b] = excl;
        excl += v[q];
    }
    __syncthreads();
    const int bits = 32 - __builtin_clz(g.nk);
    const int64_t r_end = min(n, per * (wave + 1));
    for (int64_t r0 = per * wave; wave < nw && r0 < r_end; r0 += 64) {
        const int64_t r = r0 + lane;
        const bool in = r < r_end;
        const int key = in ? (r < kSortLds ? int(keys[r]) : key_of(r)) : 0;
        uint64_t same = __ballot(in);            // lanes with this lane's key
        for (int b = 0; b < bits; ++b) {
            const bool bit = (key >> b) & 1;
            const uint64_t ones = __ballot(in && bit);
            same &= bit ? ones : ~ones;
        }
        const int slot = (key << sh) + wave;
        const int base = in ? cnt[slot] : 0;
        if (in) {
            const int at = base + __popcll(same & __lanemask_lt());
            ord.perm[at] = int32_t(r);
            ord.key[at] = key;
        }
        // every lane has read its key's offset before the first lane of each
        // key group (the only writer of that counter) advances it
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (in && (same & __lanemask_lt()) == 0) cnt[slot] = base + __popcll(same);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // which part takes each tile: its distinct keys (sorted, so its runs)
    __threadfence_block();
    __syncthreads();
    const int64_t ntile = (n + kTileRows - 1) / kTileRows;
    for (int64_t t = tid; t < ntile; t += kBlock) {
        int runs = 0, prev = -1;
        const int64_t p1 = min(n, (t + 1) * kTileRows);
        for (int64_t p = t * kTileRows; p < p1; ++p) {
            const int k = ord.key[p];
            runs += k != prev;
            prev = k;
        }
        ord.mfma[t] = runs <= kMfmaMaxRuns ? 1 : 0;
    }
}

// One launch for the per-vector preparation: workgroup 0 sorts the rows by
// ik (the longest serial chain, so it is dispatched first), and workgroup
// r + 1 interpolates row r's profile to the bin means, integrates its
// I_star (the table kernels' arithmetic) and finds its lowest node.  With pvc
// one thread of a vector's first row also derives the vector's constants (as
// k_pv_setup, whose launch of 4-5 us this saves).
template <bool kF32>
__global__ __launch_bounds__(kBlock) void k_pv_prep(const double* __restrict__ mu_s,
                                                    const double* __restrict__ prof,
                                                    int32_t nmu, const double* __restrict__ zm,
                                                    int32_t nz, const double* __restrict__ pv,
                                                    int32_t npv, int32_t npar, GridDev g,
                                                    double* __restrict__ ldp,
                                                    double* __restrict__ istar,
                                                    double* __restrict__ inv_istar,
                                                    PvOrder ord, double k1,
                                                    PvConst* __restrict__ pvc) {
    const int64_t nr = int64_t(npv) * g.npb;
    if (blockIdx.x == 0) {
        sort_rows(pv, npv, npar, g, ord);
        return;
    }
    const int64_t r = int64_t(blockIdx.x) - 1;
    if (r >= nr) return;
    const double* f = prof + r * nmu;
    const int64_t ipv = r / g.npb;
    const int pb = int(r - ipv * g.npb);
    const double* row = pv + ipv * npar;
    if (threadIdx.x == kBlock - 1 && pvc && pb == 0)
        pvc[ipv] = make_pv_const<kF32>(row, g.npb, g.k0, k1);
    if (threadIdx.x == kBlock - 65) ord.mlo[r] = lowest_node(row, row[6 + pb], g);
    for (int j = threadIdx.x; j < nz; j += kBlock) ldp[r * nz + j] = profile_at_bin(mu_s, f, nmu, zm[j]);
    istar_block(mu_s, f, nmu, istar + r, inv_istar + r);
}

// The per-vector table rows T_r[s][m] = sum_j W[ik_r + s][j][m] ldp_r[j],
// s = 0, 1.  Rows of a sorted 16-row tile with at most two distinct k-rows go
// to the matrix cores (each W value read once for up to 16 rows); the rows of
// the other tiles (k spread over many k-rows, where a tile would need a pass
// per k-row) one by one.  The two parts share one launch; nodes below
// lowest_node are left out.  Matrix cores: the part waits on its loads of W
// (from the L2 for the most part), so it needs many of them in flight: with
// one wave over all bins and 4-byte loads it took 32 us for 1024 walkers
// (default grid, float), with the bins split over four waves and 16-byte loads
// 15 us.
// FP32 weights, workgroups of 64 nodes and four waves that split the bins:
// lane l takes the nodes m0 + 4 (l & 15) .. + 3 of bins 4 i + (l >> 4), in
// v_mfma_f64_16x16x4f64 chains D = A B with A[m][j] = W[ik + s][j][m] and
// B[j][q] = ldp of row q when the row's k-row is ik, else 0, over the distinct
// ik of the tile (FP64 products and sums).  Lane l holds
// A[l & 15][l >> 4], B[l >> 4][l & 15] and D[4 i + (l >> 4)][l & 15] (checked
// on the device); row a of chain q is node m0 + 4 a + q.
typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kPvWaves = kBlock / 64;
constexpr int kPvNodes = 64;
constexpr int kPvLds = kPvWaves * 8 * 64;             // doubles
template <bool kVec, typename R, typename WT>
__device__ inline void pv_tables_mfma(const WT* __restrict__ W, const double* __restrict__ ldp,
                                      const PvOrder& ord, int64_t nr, int32_t nz,
                                      const GridDev& g, R* __restrict__ out, int64_t rt, int m0,
                                      double* __restrict__ lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ka = lane >> 4, col = lane & 15;
    const int64_t pos = rt * kTileRows + col;
    const int64_t r = pos < nr ? ord.perm[pos] : -1;
    const int ik = pos < nr ? ord.key[pos] : 0x7fffffff;
    if (wave_min(r >= 0 ? ord.mlo[r] : g.ng) >= m0 + kPvNodes) return;   // no row reads these
    const int mm = m0 + 4 * col;
    v4d d[2][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) d[0][q] = d[1][q] = v4d{0.0, 0.0, 0.0, 0.0};
    // distinct k-rows of the tile, smallest first (wave-uniform loop)
    int cur = wave_min(ik);
    while (cur != 0x7fffffff) {
        const bool take = ik == cur;
        const WT* w0 = W + int64_t(cur) * nz * g.ng;
        const WT* w1 = w0 + int64_t(nz) * g.ng;
        const double* lr = ldp + (take ? r : 0) * nz;
        constexpr int kStep = sizeof(WT) == 4 ? 4 : 2;     // bins in flight per lane
        for (int j0 = 4 * wave; j0 < nz; j0 += 4 * kPvWaves * kStep) {
            WT a0[kStep][4], a1[kStep][4];
            double b[kStep];
#pragma unroll
            for (int u = 0; u < kStep; ++u) {
                const int j = j0 + 4 * kPvWaves * u + ka;
                const int64_t row = int64_t(j < nz ? j : nz - 1) * g.ng;
                load4<kVec>(w0 + row, mm, g.ng, a0[u]);
                load4<kVec>(w1 + row, mm, g.ng, a1[u]);
                const double bj = lr[j < nz ? j : nz - 1];
                b[u] = j < nz && take ? bj : 0.0;
            }
#pragma unroll
            for (int u = 0; u < kStep; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    d[0][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(double(a0[u][q]), b[u], d[0][q], 0, 0, 0);
                    d[1][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(double(a1[u][q]), b[u], d[1][q], 0, 0, 0);
                }
        }
        cur = wave_min(ik > cur ? ik : 0x7fffffff);
    }
    // Add the waves' sums in wave order, half a table row at a time
    // (h: elements i = 2 h, 2 h + 1): wave w finishes element 2 h + (w & 1) of
    // chains 2 (w >> 1) and 2 (w >> 1) + 1, two consecutive nodes.
    static_assert(kPvWaves == 4, "the split of the finishing work");
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (s + h) __syncthreads();
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    lds[((wave * 2 + i) * 4 + q) * 64 + lane] = d[s][q][2 * h + i];
            __syncthreads();
            const int i = wave & 1, q0 = wave >> 1 << 1;
            const int m = m0 + 4 * (4 * (2 * h + i) + ka) + q0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                double v = lds[(i * 4 + q0 + q) * 64 + lane];
#pragma unroll
                for (int w = 1; w < kPvWaves; ++w) v += lds[((w * 2 + i) * 4 + q0 + q) * 64 + lane];
                if (r >= 0 && m + q < g.ng) out[r * 2 * g.ng + s * g.ng + m + q] = R(v);
            }
        }
}

// The same for FP64 weights with the bins in order, so that a row given the
// tables' own profile has k_tables' bits (the matrix core adds its products in
// order, as a chain of FMAs): wave w takes table row s = w & 1 of the nodes
// m0 + 32 (w >> 1) .. + 31, lane l nodes 2 (l & 15) and the next, and two
// chains run over all bins.  Calls of 1024 x 20 000 walkers 64 us (62 with the
// bins split as above, 66 with one node per lane and 8-byte loads), of 4096 x
// 1000 88 (96, 96).
template <bool kVec, typename R>
__device__ inline void pv_tables_mfma_ordered(const double* __restrict__ W,
                                              const double* __restrict__ ldp, const PvOrder& ord,
                                              int64_t nr, int32_t nz, const GridDev& g,
                                              R* __restrict__ out, int64_t rt, int m0) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int ka = lane >> 4, col = lane & 15, s = wave & 1;
    const int64_t pos = rt * kTileRows + col;
    const int64_t r = pos < nr ? ord.perm[pos] : -1;
    const int ik = pos < nr ? ord.key[pos] : 0x7fffffff;
    const int mw = m0 + 32 * (wave >> 1);
    if (mw >= g.ng || wave_min(r >= 0 ? ord.mlo[r] : g.ng) >= mw + 32) return;   // uniform
    const int mm = mw + 2 * col;
    v4d d0 = {0.0, 0.0, 0.0, 0.0}, d1 = {0.0, 0.0, 0.0, 0.0};
    int cur = wave_min(ik);
    while (cur != 0x7fffffff) {
        const bool take = ik == cur;
        const double* w = W + int64_t(cur + s) * nz * g.ng;
        const double* lr = ldp + (take ? r : 0) * nz;
        constexpr int kStep = 8;                    // steps of four bins in flight
        for (int j0 = ka; j0 - ka < nz; j0 += 4 * kStep) {
            double a[kStep][2], b[kStep];
#pragma unroll
            for (int u = 0; u < kStep; ++u) {
                const int j = j0 + 4 * u, jc = j < nz ? j : nz - 1;
                load_pair<kVec>(w + int64_t(jc) * g.ng, mm, g.ng, a[u]);
                const double bj = lr[jc];
                b[u] = j < nz && take ? bj : 0.0;
            }
#pragma unroll
            for (int u = 0; u < kStep; ++u) {
                d0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][0], b[u], d0, 0, 0, 0);
                d1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][1], b[u], d1, 0, 0, 0);
            }
        }
        cur = wave_min(ik > cur ? ik : 0x7fffffff);
    }
    if (r < 0) return;
    R* o = out + (r * 2 + s) * g.ng;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = mw + 2 * (4 * i + ka);
        if (m < g.ng) o[m] = R(d0[i]);
        if (m + 1 < g.ng) o[m + 1] = R(d1[i]);
    }
}

// One sorted row, one node per lane, the bins in order (k_tables' bits, as
// above).  What bounds it is the traffic of the distinct W rows into the eight
// L2s (53 MB in float, 106 MB in FP64 for a population of 512): the loads in
// flight only have to keep that busy (float 18.2 us with 40 of them).  In FP64
// a wave takes one of the two table rows, so that few rows still keep enough
// loads in flight (a call of 37 rows x 5000 32 us with both, 26 with one; 512 x
// 20 000 78 and 76; with the bins split over four waves, whose order is another,
// 25 and 73, and 1024 x 1000 103 instead of 112).
template <typename WT>
constexpr int kRowTabs = sizeof(WT) == 4 ? 2 : 1;                 // table rows per wave
template <typename WT>
constexpr int kRowNodes = kPvNodes * kPvWaves * kRowTabs<WT> / 2; // per workgroup
template <typename R, typename WT>
__device__ inline void pv_tables_row(const WT* __restrict__ W, const double* __restrict__ ldp,
                                     const PvOrder& ord, int64_t pos, int32_t nz,
                                     const GridDev& g, R* __restrict__ out, int m0) {
    constexpr int kTabs = kRowTabs<WT>;
    const int64_t r = ord.perm[pos];
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int mw = m0 + wave * kTabs / 2 * kPvNodes, m = mw + int(threadIdx.x & 63);
    if (mw >= g.ng || ord.mlo[r] >= mw + kPvNodes) return;     // uniform
    const int s0 = kTabs == 2 ? 0 : wave & 1;                  // first table row
    const WT* w = W + int64_t(ord.key[pos] + s0) * nz * g.ng + (m < g.ng ? m : 0);
    const int64_t next = int64_t(nz) * g.ng;                   // the k-row above
    const double* lr = ldp + r * nz;                           // uniform
    double acc[kTabs] = {};
    constexpr int kStep = 20;               // bins in flight
    int j = 0;
    for (; j + kStep <= nz; j += kStep) {
        WT x[kTabs][kStep];
#pragma unroll
        for (int b = 0; b < kStep; ++b)
#pragma unroll
            for (int s = 0; s < kTabs; ++s) x[s][b] = w[s * next + int64_t(j + b) * g.ng];
#pragma unroll
        for (int b = 0; b < kStep; ++b)
#pragma unroll
            for (int s = 0; s < kTabs; ++s) acc[s] += double(x[s][b]) * lr[j + b];
    }
    for (; j < nz; ++j)
#pragma unroll
        for (int s = 0; s < kTabs; ++s) acc[s] += double(w[s * next + int64_t(j) * g.ng]) * lr[j];
    if (m < g.ng)
#pragma unroll
        for (int s = 0; s < kTabs; ++s) out[(r * 2 + s0 + s) * g.ng + m] = R(acc[s]);
}

// Workgroups [0, n_mfma) take (tile, 64 nodes) on the matrix cores, the
// others (sorted row, kRowNodes nodes): those in an XCD-aware order -- blocks go
// round-robin to the eight XCDs, so block p works on item (p mod 8) *
// (blocks / 8) + p / 8 (rounded for a remainder; n_mfma is a multiple of 8)
// and each XCD walks a contiguous stretch of the sorted rows, whose W rows
// its L2 then serves to the following rows of equal ik.
constexpr int kXcds = 8;
template <bool kVec, typename R, typename WT>
__global__ __launch_bounds__(kBlock, 3) void k_pv_tables(const WT* __restrict__ W,
                                                      const double* __restrict__ ldp,
                                                      PvOrder ord, int64_t nr, int32_t nz,
                                                      GridDev g, int64_t n_mfma,
                                                      int64_t blocks, R* __restrict__ out) {
    const int64_t b = flat_block();
    if (b >= blocks) return;
    const int nmb = (g.ng + kPvNodes - 1) / kPvNodes;
    if (b < n_mfma) {
        const int64_t rt = b / nmb;
        if (rt * kTileRows >= nr || !ord.mfma[rt]) return;
        const int m0 = int(b - rt * nmb) * kPvNodes;
        if constexpr (sizeof(WT) == 8) {
            pv_tables_mfma_ordered<kVec, R>(W, ldp, ord, nr, nz, g, out, rt, m0);
        } else {
            __shared__ double lds[kPvLds];
            pv_tables_mfma<kVec, R, WT>(W, ldp, ord, nr, nz, g, out, rt, m0, lds);
        }
        return;
    }
    const int64_t nb = blocks - n_mfma, p = b - n_mfma;
    const int64_t q = nb / kXcds, rem = nb % kXcds, x = p % kXcds;
    const int64_t L = (x < rem ? x * (q + 1) : rem * (q + 1) + (x - rem) * q) + p / kXcds;
    const int nrb = (g.ng + kRowNodes<WT> - 1) / kRowNodes<WT>;
    const int64_t pos = L / nrb;
    if (ord.mfma[pos / kTileRows]) return;
    pv_tables_row<R, WT>(W, ldp, ord, pos, nz, g, out, int(L - pos * nrb) * kRowNodes<WT>);
}

// Direct model (Sect. 3.1.1): the LD-weighted vector of row r = (vector,
// passband) from weights built for the row's own k -- no k-grid, no
// k-interpolation, any k in (0, 1] -- with the tables' profile at the bin
// means: ldw_r[m] = sum_j (A_{j+1} - A_j) l_j / A_nz, with A_j the lens area
// of the disk of edge j and l = ldp[pb], FP64.  Stored twice ([2][ng]) in the
// evaluation precision for the forward kernel, which reads it with zero
// k-weight.
//   The kernel is bound by FP64 arithmetic, so it evaluates only the lens
// areas that need it.  Summed by parts, ldw = (A_J l_{J-1} -
// sum_{1 <= j < J} A_j (l_j - l_{j-1})) / A_nz with J the first edge that
// encloses the planet (nz if none does): edges below |c - k| have area zero
// (or pi R^2 inside the planet's disk), those from J on drop out, and only
// the edges the planet's limb crosses -- 40 of 181 on average over the
// grazing nodes, k = 0.05-0.2 on the default grid -- are evaluated, each lane
// (one node m) over its own range.  For a fixed c the half chord comes from
// its own distance x to the centre, h^2 = (R - x)(R + x): the area is
// stationary in h, so the cancellation in R - x near a contact does not reach
// it.  Workgroup: 64 nodes of one row, one per lane, whose edges its waves
// share in turn (with one wave per 64 nodes the limb's nodes, which cross up
// to 120 edges, ran on alone: 86 us), the limb's nodes first; nodes below the
// row's lowest_node are left out.
// 512 rows, default grid, FP64: 182 us with every edge evaluated, 59 without
// those that need not be, 55 without the nodes no exposure reads either (a third
// of them, but the cheap ones near the centre).
constexpr int kDirectWaves = 4;            // 66 / 59 / 63 us with 2 / 4 / 8
// sqrt of a normal x > 0 by Goldschmidt's iteration: s -> sqrt x and h ->
// 1 / (2 sqrt x) from the hardware's reciprocal square root, refined once
// together, then s once more by its residual; within an ulp or two.
__device__ inline double sqrt_nr(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double s = x * y, h = 0.5 * y;
    const double e = fma(-h, s, 0.5);
    s = fma(s, e, s);
    h = fma(h, e, h);
    return fma(fma(-s, s, x), h, s);
}
template <typename R>
__global__ __launch_bounds__(64 * kDirectWaves) void k_direct_rows(
    const double* __restrict__ ze, const double* __restrict__ ldp, const double* __restrict__ pv,
    PvConst* __restrict__ pvc, int32_t npar, int64_t nr, int32_t nz, GridDev g,
    R* __restrict__ out) {
    extern __shared__ double direct_lds[];
    double* edge = direct_lds;                     // edges 1 .. nz - 1, at j - 1
    double* dl = direct_lds + (nz - 1);            // l_j - l_{j-1}, at j - 1
    const int nmb = (g.ng + 63) / 64;
    const int64_t b = flat_block();
    if (b >= nr * nmb) return;
    const int64_t r = b % nr;
    const int mb = nmb - 1 - int(b / nr);
    const int64_t ipv = r / g.npb;
    const int pb = int(r - ipv * g.npb);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double* l = ldp + int64_t(pb) * nz;
    bool finite = is_finite(l[0]);
    for (int j = 1 + threadIdx.x; j < nz; j += 64 * kDirectWaves) {
        edge[j - 1] = ze[j];
        dl[j - 1] = l[j] - l[j - 1];
        finite = finite && is_finite(l[j]);
    }
    // the sum over all bins that this stands for is not finite wherever a bin
    // is not, also in nodes whose planet does not reach that bin
    __shared__ int prof_ok[kDirectWaves];
    const int wave_ok = __all(finite);
    if (lane == 0) prof_ok[wave] = wave_ok;
    const double k = pv[ipv * npar + 6 + pb];
    __shared__ int low;
    if (threadIdx.x == 64 * kDirectWaves - 1)
        low = lowest_node(pv + ipv * npar, k, g);
    // any k in (0, 1]: the smallest positive double as the lower bound
    if (threadIdx.x == 64 * kDirectWaves - 65 && mb == nmb - 1 && pb == 0)
        pvc[ipv] = make_pv_const<sizeof(R) == 4>(pv + ipv * npar, g.npb, 4.9406564584124654e-324,
                                                 1.0);
    __syncthreads();
    if (mb * 64 + 63 < low) return;                // no exposure reads these nodes
    const int m = mb * 64 + lane;
    const bool valid = k > 0.0 && k <= 1.0;        // uniform
    using N = Num<double>;
    const double c = (double(m) / double(g.ng - 1)) * (1.0 + k);
    double s = 0.0;
    int J = nz;
    if (valid && m < g.ng && c < 1.0 + k) {
        // first edge at or above x among 1 .. nz - 1 (nz if none)
        auto first = [&](double x, bool above) {
            int lo = 1, hi = nz;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                const double e = edge[mid - 1];
                if (above ? e > x : e >= x) hi = mid; else lo = mid + 1;
            }
            return lo;
        };
        J = first(c + k, false);
        int j = first(fabs(c - k), true);
        j = j < J ? j : J;
        if (c < k && wave == 0)
            for (int i = 1; i < j; ++i) s += N::pi * edge[i - 1] * edge[i - 1] * dl[i - 1];
        const double hic = 0.5 * N::rcp_(c > 0.0 ? c : 1.0);
        const double x1c = (c - k) * (c + k) * hic, k2 = k * k;
        for (j += wave; j < J; j += kDirectWaves) {
            const double Re = edge[j - 1], R2 = Re * Re;
            const double x1 = fma(R2, hic, x1c), x0 = c - x1;
            const double h2 = (Re - x1) * (Re + x1);
            const double h = sqrt_nr(fmax(h2, 1e-290));
            const double area = R2 * atan2_pos<HwOps, true>(h, x1) +
                                k2 * atan2_pos<HwOps, true>(h, x0) - c * h;
            s += area * dl[j - 1];
        }
    }
    // the waves' sums in wave order, in the space of the edges
    __syncthreads();
    double* part = direct_lds;
    if (wave > 0) part[(wave - 1) * 64 + lane] = s;
    __syncthreads();
    if (wave > 0 || m >= g.ng) return;
    R* o = out + r * 2 * g.ng;
    double acc = 0.0;                       // invalid row: the forward writes NaN
    if (valid) {
#pragma unroll
        for (int w = 1; w < kDirectWaves; ++w) s += part[(w - 1) * 64 + lane];
        // no overlap: the limb annulus; J < nz: the disk of edge J encloses
        // the planet, A_J = tot = pi k^2
        const double tot = lens_area<double>(1.0, k, c);
        acc = tot > 0.0 ? l[J - 1] - s / tot : l[nz - 1];
#pragma unroll
        for (int w = 0; w < kDirectWaves; ++w) acc = prof_ok[w] ? acc : double(NAN);
    }
    o[m] = R(acc);
    o[g.ng + m] = R(acc);
}

// Small-planet approximation (Sect. 3.4.2) as rows of the per-vector path:
// for a row whose k is below k_small, the LD-weighted mean over the planet's
// disk at each g node is replaced by the profile at the planet's centre,
// c = g_m (1 + k) clamped to the limb (mu = sqrt(1 - c^2) on the tables'
// piecewise-linear profile); any other row gets the shared table's two
// k-rows around its k combined with its k-weight, in the evaluation
// precision and in the order the forward kernel combines them.  Workgroup
// (row, kBlock nodes): a small-planet row stages the mu samples and its
// passband's profile in LDS (when they fit) for the binary searches.
// Stored twice ([2][ng]), read with zero k-weight.  One thread of each row also
// derives the row's constants pvc for the forward kernel, which took a launch
// of their own (about 4 us).
constexpr int kSpLds = 1024;
template <typename R>
__global__ __launch_bounds__(kBlock) void k_small_planet_rows(
    const double* __restrict__ mu_s, const double* __restrict__ prof, int32_t nmu,
    const R* __restrict__ T, const double* __restrict__ pv, int32_t npar, double k_small,
    double k1, GridDev g, PvConst* __restrict__ pvc, R* __restrict__ out) {
    __shared__ double smu[kSpLds], sf[kSpLds];
    const int64_t r = blockIdx.x;
    const int m = int(blockIdx.y) * kBlock + int(threadIdx.x);
    const int64_t ipv = r / g.npb;
    const int pb = int(r - ipv * g.npb);
    if (threadIdx.x == kBlock - 1 && blockIdx.y == 0 && pb == 0)
        pvc[ipv] = make_pv_const<sizeof(R) == 4>(pv + ipv * npar, g.npb, g.k0, k1, k_small);
    const double k = pv[ipv * npar + 6 + pb];          // uniform in the workgroup
    R* o = out + r * 2 * g.ng;
    R v = R(0);                                        // invalid rows: the forward writes NaN
    if (k < k_small) {
        if (k > 0.0) {
            const double* f = prof + int64_t(pb) * nmu;
            const bool staged = nmu <= kSpLds;
            if (staged) {
                for (int j = threadIdx.x; j < nmu; j += kBlock) {
                    smu[j] = mu_s[j];
                    sf[j] = f[j];
                }
                __syncthreads();
            }
            if (m >= g.ng) return;
            double c = (double(m) / double(g.ng - 1)) * (1.0 + k);
            c = c < 1.0 ? c : 1.0;
            v = R(staged ? profile_at_bin(smu, sf, nmu, c) : profile_at_bin(mu_s, f, nmu, c));
        }
    } else if (k >= g.k0 && k <= k1) {
        if (m >= g.ng) return;
        const double u = (k - g.k0) / g.dk;
        int ik = int(floor(u));
        ik = ik < 0 ? 0 : (ik > g.nk - 2 ? g.nk - 2 : ik);
        const R ak = R(u - ik);
        const R* t0r = T + (int64_t(pb) * g.nk + ik) * g.ng;
        v = (R(1) - ak) * t0r[m] + ak * t0r[g.ng + m];
    }
    if (m >= g.ng) return;
    o[m] = v;
    o[g.ng + m] = v;
}

hipError_t launch_direct_rows(const rr_tables* t, const double* pv, PvConst* pvc,
                              int32_t npv, int32_t npar, int32_t precision, void* rows,
                              hipStream_t s) {
    const GridDev g = grid_dev(t);
    const int64_t nr = int64_t(npv) * t->npb;
    const int64_t blocks = nr * ((g.ng + 63) / 64);
    const dim3 grid = flat_grid(blocks);
    // the edges and profile steps (65 520 B at the largest nz), then the waves' sums
    const size_t lds = sizeof(double) * std::max<size_t>(2 * size_t(t->nz - 1),
                                                         64 * (kDirectWaves - 1));
    if (precision == RR_FP64)
        hipLaunchKernelGGL(k_direct_rows<double>, grid, dim3(64 * kDirectWaves), lds, s, t->ze,
                           t->ldp, pv, pvc, npar, nr, t->nz, g, static_cast<double*>(rows));
    else
        hipLaunchKernelGGL(k_direct_rows<float>, grid, dim3(64 * kDirectWaves), lds, s, t->ze,
                           t->ldp, pv, pvc, npar, nr, t->nz, g, static_cast<float*>(rows));
    return hipGetLastError();
}

// The small-planet rows for the log-likelihood's adjoint, which reads a
// row pair (row0, row1) per (vector, passband) with the k-weight ak of the
// row's k on the tables' k-grid: ldw = (1 - ak) row0 + ak row1 and
// dldw/dk = (row1 - row0) / dk.  Below k_small the pair is built so that
// these give the centre values v[m] = I(mu(c_m)), c_m = g_m (1 + k), and
// their k-derivative D[m] = I'(mu) (-c_m / mu) g_m (zero where c_m is
// clamped to the limb or the profile is constant beyond its samples):
// row0 = v - ak dk D, row1 = row0 + dk D.  Other rows copy the shared
// table's two k-rows.  Also writes 1/I_star per row (the tables' value).
template <typename R>
__global__ __launch_bounds__(kBlock) void k_small_planet_adj_rows(
    const double* __restrict__ mu_s, const double* __restrict__ prof, int32_t nmu,
    const R* __restrict__ T, const double* __restrict__ inv_istar, const double* __restrict__ pv,
    int32_t npar, double k_small, GridDev g, R* __restrict__ out,
    double* __restrict__ inv_istar_rows) {
    __shared__ double smu[kSpLds], sf[kSpLds];
    const int64_t r = blockIdx.x;
    const int m = int(blockIdx.y) * kBlock + int(threadIdx.x);
    const int64_t ipv = r / g.npb;
    const int pb = int(r - ipv * g.npb);
    const double k = pv[ipv * npar + 6 + pb];          // uniform in the workgroup
    R* o = out + r * 2 * g.ng;
    const double u = (k - g.k0) / g.dk;
    int ik = int(floor(u));
    ik = ik < 0 ? 0 : (ik > g.nk - 2 ? g.nk - 2 : ik);
    R r0 = R(0), r1 = R(0);                           // invalid rows: NaN from the setup
    if (k < k_small) {
        if (k > 0.0) {
            const double* f = prof + int64_t(pb) * nmu;
            const bool staged = nmu <= kSpLds;
            if (staged) {
                for (int j = threadIdx.x; j < nmu; j += kBlock) {
                    smu[j] = mu_s[j];
                    sf[j] = f[j];
                }
                __syncthreads();
            }
            if (m >= g.ng) return;
            const double* ms = staged ? smu : mu_s;
            const double* fs = staged ? sf : f;
            const double gm = double(m) / double(g.ng - 1);
            const double craw = gm * (1.0 + k);
            const double c = craw < 1.0 ? craw : 1.0;
            const double v = profile_at_bin(ms, fs, nmu, c);
            double D = 0.0;
            const double mu = sqrt(1.0 - c * c);
            if (craw < 1.0 && mu > ms[0] && mu < ms[nmu - 1]) {
                int lo = 0, hi = nmu - 1;                  // ms[lo] <= mu < ms[hi]
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (ms[mid] <= mu) lo = mid; else hi = mid;
                }
                const double slope = (fs[lo + 1] - fs[lo]) / (ms[lo + 1] - ms[lo]);
                D = slope * (-c / mu) * gm;
            }
            const double ak = u - ik;
            const double b0 = v - ak * g.dk * D;
            r0 = R(b0);
            r1 = R(b0 + g.dk * D);
        }
    } else {
        if (m >= g.ng) return;
        const R* t0r = T + (int64_t(pb) * g.nk + ik) * g.ng;
        r0 = t0r[m];
        r1 = t0r[g.ng + m];
    }
    if (m >= g.ng) return;
    o[m] = r0;
    o[g.ng + m] = r1;
    if (m == 0) inv_istar_rows[r] = inv_istar[pb];
}

hipError_t launch_small_planet_adj_rows(const rr_tables* t, const double* pv, int32_t npv,
                                        int32_t npar, double k_small, int32_t precision,
                                        void* rows, double* inv_istar_rows, hipStream_t s) {
    const GridDev g = grid_dev(t);
    const int64_t nr = int64_t(npv) * t->npb;
    const dim3 grid(unsigned(nr), unsigned((g.ng + kBlock - 1) / kBlock));
    if (precision == RR_FP64)
        hipLaunchKernelGGL(k_small_planet_adj_rows<double>, grid, dim3(kBlock), 0, s, t->mu_s,
                           t->prof, t->nmu, t->T64, t->inv_istar, pv, npar, k_small, g,
                           static_cast<double*>(rows), inv_istar_rows);
    else
        hipLaunchKernelGGL(k_small_planet_adj_rows<float>, grid, dim3(kBlock), 0, s, t->mu_s,
                           t->prof, t->nmu, t->T32, t->inv_istar, pv, npar, k_small, g,
                           static_cast<float*>(rows), inv_istar_rows);
    return hipGetLastError();
}

hipError_t launch_small_planet_rows(const rr_tables* t, const double* pv, int32_t npv,
                                    int32_t npar, double k_small, int32_t precision,
                                    PvConst* pvc, void* rows, hipStream_t s) {
    const GridDev g = grid_dev(t);
    const int64_t nr = int64_t(npv) * t->npb;
    const dim3 grid(unsigned(nr), unsigned((g.ng + kBlock - 1) / kBlock));
    if (precision == RR_FP64)
        hipLaunchKernelGGL(k_small_planet_rows<double>, grid, dim3(kBlock), 0, s, t->mu_s,
                           t->prof, t->nmu, t->T64, pv, npar, k_small, t->grid.k1, g, pvc,
                           static_cast<double*>(rows));
    else
        hipLaunchKernelGGL(k_small_planet_rows<float>, grid, dim3(kBlock), 0, s, t->mu_s,
                           t->prof, t->nmu, t->T32, pv, npar, k_small, t->grid.k1, g, pvc,
                           static_cast<float*>(rows));
    return hipGetLastError();
}

hipError_t launch_pv_ld(const rr_tables* t, const double* prof, const double* pv,
                        int32_t npv, int32_t npar, int32_t precision, double* ldp,
                        double* istar, double* inv_istar, const PvOrder& ord,
                        void* rows, hipStream_t s, bool w32, PvConst* pvc) {
    const GridDev g = grid_dev(t);
    const int64_t nr = int64_t(npv) * t->npb;     // (vector, passband) rows
    hipLaunchKernelGGL(precision == RR_FP64 ? k_pv_prep<false> : k_pv_prep<true>,
                       dim3(unsigned(nr + 1)), dim3(kBlock), 0, s, t->mu_s, prof, t->nmu, t->zm,
                       t->nz, pv, npv, npar, g, ldp, istar, inv_istar, ord, t->grid.k1, pvc);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // both parts read the same weights (FP64, or the FP32 copy with w32)
    const int64_t nmb = (g.ng + kPvNodes - 1) / kPvNodes;
    const int64_t n_mfma =
        ((nr + kTileRows - 1) / kTileRows * nmb + kXcds - 1) / kXcds * kXcds;
    const int64_t row_nodes = precision != RR_FP64 && w32 ? kRowNodes<float> : kRowNodes<double>;
    const int64_t blocks = n_mfma + nr * ((g.ng + row_nodes - 1) / row_nodes);
    const dim3 grid = flat_grid(blocks);
    // 16-byte loads of W need rows of a multiple of 4 nodes
    auto launch = [&](auto kernel, const auto* W, auto* out) {
        hipLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, s, W, ldp, ord, nr, t->nz, g, n_mfma,
                           blocks, out);
    };
    const bool vec = g.ng % 4 == 0;
    if (precision == RR_FP64)
        launch(vec ? k_pv_tables<true, double, double> : k_pv_tables<false, double, double>, t->W,
               static_cast<double*>(rows));
    else if (w32)
        launch(vec ? k_pv_tables<true, float, float> : k_pv_tables<false, float, float>, t->W32,
               static_cast<float*>(rows));
    else
        launch(vec ? k_pv_tables<true, float, double> : k_pv_tables<false, float, double>, t->W,
               static_cast<float*>(rows));
    return hipGetLastError();
}

__global__ void k_istar_set(const double* __restrict__ src, int32_t npb,
                            double* __restrict__ user, double* __restrict__ istar,
                            double* __restrict__ inv_istar) {
    const int pb = blockIdx.x * blockDim.x + threadIdx.x;
    if (pb >= npb) return;
    const double v = src[pb];
    if (user) user[pb] = v;
    istar[pb] = v;
    inv_istar[pb] = (v > 0.0 && is_finite(v)) ? 1.0 / v : NAN;
}

hipError_t launch_istar_set(rr_tables* t, const double* src, hipStream_t s) {
    hipLaunchKernelGGL(k_istar_set, dim3(1), dim3(kBlock), 0, s, src, t->npb,
                       src == t->istar_user ? nullptr : t->istar_user, t->istar, t->inv_istar);
    return hipGetLastError();
}

hipError_t launch_istar_from_profile(rr_tables* t, hipStream_t s) {
    hipLaunchKernelGGL(k_istar, dim3(t->npb), dim3(kBlock), 0, s, t->mu_s, t->prof,
                       t->nmu, t->istar, t->inv_istar);
    return hipGetLastError();
}

hipError_t launch_prepare_profile(rr_tables* t, hipStream_t s) {
    const GridDev g = grid_dev(t);
    hipLaunchKernelGGL(k_profile, dim3(nblocks(int64_t(t->nz) * t->npb)), dim3(kBlock), 0, s,
                       t->mu_s, t->prof, t->nmu, t->zm, t->nz, t->npb, t->ldp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // the caller's normalisers, if set, stay in force over a new profile
    e = t->istar_fixed ? launch_istar_set(t, t->istar_user, s) : launch_istar_from_profile(t, s);
    if (e != hipSuccess) return e;
    const int64_t nt = int64_t(g.npb) * g.nk * g.ng;
    hipLaunchKernelGGL(k_tables, dim3(nblocks(nt)), dim3(kBlock), 0, s, t->W, t->ldp, g,
                       t->T64, t->T32);
    return hipGetLastError();
}

}  // namespace rr
