// Discrete adjoint of the 1D AT stepper (reverse mode): k_adj1d, one launch per
// step, and k_adj1d_wave, several steps per launch.
//
// The forward step at level n is u'_i = u_i + dt*(nu*D2_i - a_i*D1_i) with
// the central stencils of section 3.2 and, at a tile edge, halo values
// extrapolated in time from the neighbour edge's levels n-k-j (section 2,
// Eqs. (1)-(2)).  Its transpose, given lambda^{n+1} = dJ/du^{n+1}:
//   * centre:     lambda_i * (1 + dt*(nu*dD2/du - D1))     (Burgers; linear: no -D1)
//   * neighbour:  lambda_i * dt*(nu*dD2/dnb_s - a_i*dD1/dnb_s) flows to the
//     point at stencil slot s when it lies in the same tile, otherwise to the
//     halo's source edge point at the levels n-k-j with the extrapolation
//     weights dH/dv_j ((k+1, -k) for two levels; ((k+1)(k+2)/2, -k(k+2),
//     k(k+1)/2) for three; 1 for the stale halo or k = 0);
//   * dJ/dnu += lambda_i * dt * D2_i.
// The halo contributions ("mu") of step n are needed by earlier levels of the
// neighbour's edge, so they are kept in a small ring over the last L+m
// steps and GATHERED by the owner of each edge point (no atomics): at
// reverse step n an edge point adds, for n' = n .. n+L+m-1, the weight for
// j = n' - k[n'] - n of every mu^{n'} of the face it feeds.  mu^n itself is
// recomputed in place from lambda^{n+1} and u^n, which the workgroup holds.
// Each workgroup keeps one compensated dJ/dnu accumulator across launches.
#include <type_traits>

#include "at_internal.h"
#include "at_stencil1d.h"
#include "at_wave.h"

namespace atk {

namespace {

constexpr int kPPA = 4;                       // points per thread
constexpr int kCHA = kThreads * kPPA;         // points per workgroup

template <int ORDER>
struct Partials {
    double g1[ORDER], g2[ORDER], g2u;
};

template <int ORDER>
__device__ __forceinline__ Partials<ORDER> partials(double c1, double c2)
{
    Partials<ORDER> p;
    if constexpr (ORDER == 2) {
        p.g1[0] = -c1; p.g1[1] = c1;
        p.g2[0] = c2;  p.g2[1] = c2;
        p.g2u = -2.0 * c2;
    } else {
        p.g1[0] = c1;  p.g1[1] = -8.0 * c1; p.g1[2] = 8.0 * c1; p.g1[3] = -c1;
        p.g2[0] = -c2; p.g2[1] = 16.0 * c2; p.g2[2] = 16.0 * c2; p.g2[3] = -c2;
        p.g2u = -30.0 * c2;
    }
    return p;
}

// dH/dv_j
__device__ __forceinline__ double hweight(int kk, bool stale, int j, int M)
{
    if (kk == 0 || stale) return j == 0 ? 1.0 : 0.0;
    const double dk = (double)kk;
    if (M == 2) return j == 0 ? 1.0 + dk : -dk;
    const double w2 = 0.5 * dk * (dk + 1.0);
    if (j == 0) return (1.0 + dk) + w2;
    if (j == 1) return -dk - 2.0 * w2;
    return w2;
}

template <int ORDER, bool LINEAR>
__global__ __launch_bounds__(kThreads) void k_adj1d(Adj1D a)
{
    constexpr int H = ORDER / 2;
    constexpr int M = (ORDER == 2) ? 2 : 3;
    constexpr int NS = 2 * H;                 // stencil slots: offsets -H..-1, 1..H
    __shared__ double sl[kCHA + 2 * H], su[kCHA + 2 * H];
    __shared__ double red[kThreads / 64][2];

    const int tid = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x * kCHA;
    const int64_t owned = (a.N - c0 < kCHA) ? (a.N - c0) : kCHA;
    const int64_t F = 2 * a.P;
    const Partials<ORDER> pd = partials<ORDER>(a.c1, a.c2);
    const bool stale = a.stale != 0;

    // all loads issued before the first use (one round trip, not one per pass)
    double vl[kPPA + 1], vu[kPPA + 1];
#pragma unroll
    for (int it = 0; it <= kPPA; ++it) {
        const int r = it * kThreads + tid;
        vl[it] = vu[it] = 0.0;
        if (r < owned + 2 * H) {
            int64_t g = c0 - H + r;
            if (g < 0) g += a.N;
            if (g >= a.N) g -= a.N;
            vl[it] = a.lam_in[g];
            vu[it] = a.u[g];
        }
    }
#pragma unroll
    for (int it = 0; it <= kPPA; ++it) {
        const int r = it * kThreads + tid;
        if (r < owned + 2 * H) { sl[r] = vl[it]; su[r] = vu[it]; }
    }
    __syncthreads();

    // P_s(u) = dt*(nu*g2[s] - a*g1[s]): sensitivity of u'_i to its slot-s neighbour
    auto Ps = [&](int s, double u) -> double {
        const double adv = LINEAR ? a.cadv : u;
        double g1 = pd.g1[0], g2 = pd.g2[0];     // select without indexing a register array
#pragma unroll
        for (int i = 1; i < NS; ++i) {
            g1 = (s == i) ? pd.g1[i] : g1;
            g2 = (s == i) ? pd.g2[i] : g2;
        }
        return a.dt * (a.nu * g2 - adv * g1);
    };
    // mu^n of face (tile tf, side sd), halo index q, from the LDS copy whose
    // index ri is the first point of the tile behind the face (side 0) or the
    // last one (side 1).
    auto mu_now = [&](int sd, int q, int ri) -> double {
        double m = 0.0;
#pragma unroll
        for (int e = 0; e < H; ++e) {
            if (sd == 0 && e <= q) m += sl[ri + e] * Ps(q - e, su[ri + e]);
            if (sd == 1 && e <= H - 1 - q) m += sl[ri - e] * Ps(H + q + e, su[ri - e]);
        }
        return m;
    };

    Acc gacc{0.0, 0.0};
    const int W32 = (int)a.W;
    // tile index and offset of this thread's first point; later points step by kThreads
    const int64_t g0 = c0 + tid;
    int64_t t = g0 / a.W;
    int o_ = (int)(g0 - t * a.W);
#pragma unroll
    for (int it = 0; it < kPPA; ++it) {
        const int l = it * kThreads + tid;
        if (it > 0) {                       // advance by kThreads points without dividing
            o_ += kThreads;
            while (o_ >= W32) { o_ -= W32; ++t; }
        }
        if (l >= owned) break;
        const int64_t g = c0 + l;
        const int64_t o = o_;
        const int r = l + H;
        const double u = su[r];
        // neighbours at level n, AT halo where the stencil leaves the tile
        double nb[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int d = (s < H) ? -(H - s) : (s - H + 1);
            double v = su[r + d];
            const int64_t od = o + d;
            if (od < 0 || od >= a.W) {
                const int side = od < 0 ? 0 : 1;
                const int kk = a.delays[a.n * F + 2 * t + side];
                if (kk > 0) {
                    const int q = side == 0 ? (int)(od + H) : (int)(od - a.W);
                    int64_t stp = t + (side ? 1 : -1);
                    if (stp < 0) stp += a.P;
                    if (stp >= a.P) stp -= a.P;
                    double vv[3] = {0.0, 0.0, 0.0};
#pragma unroll
                    for (int j = 0; j < M; ++j) {
                        if (j == 0 || !stale) {
                            const int64_t lev = a.n - kk - j;
                            // record mode keeps every level: slot = level
                            vv[j] = a.ring[((lev * a.P + stp) * 2 + (1 - side)) * H + q];
                        }
                    }
                    v = extrap<false>(kk, stale, vv[0], vv[1], vv[2], M);
                }
            }
            nb[s] = v;
        }
        double D1, D2;
        if constexpr (ORDER == 2) {
            D1 = (nb[1] - nb[0]) * a.c1;
            D2 = ((nb[1] - 2.0 * u) + nb[0]) * a.c2;
        } else {
            D1 = (8.0 * (nb[2] - nb[1]) - (nb[3] - nb[0])) * a.c1;
            D2 = ((16.0 * (nb[2] + nb[1]) - 30.0 * u) - (nb[3] + nb[0])) * a.c2;
        }
        const double lam = sl[r];
        const double du = 1.0 + a.dt * (a.nu * pd.g2u - (LINEAR ? 0.0 : D1));
        double acc = lam * du;
        // same-tile points i = g - d that see g at their slot for offset d
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int d = (s < H) ? -(H - s) : (s - H + 1);
            const int64_t oi = o - d;
            if (oi >= 0 && oi < a.W) acc += sl[r - d] * Ps(s, su[r - d]);
        }
        // delayed halo contributions gathered over steps n .. n+L+m-1
        for (int side = 0; side < 2; ++side) {
            // side 0: g is in the tile's last h points, feeding face (t+1, low side);
            // side 1: g is in the first h points, feeding face (t-1, high side)
            const bool feeds = side == 0 ? (o >= a.W - H) : (o < H);
            if (!feeds) continue;
            int64_t tf = t + (side == 0 ? 1 : -1);
            if (tf < 0) tf += a.P;
            if (tf >= a.P) tf -= a.P;
            const int fs = side == 0 ? 0 : 1;                 // side of that face
            const int q = side == 0 ? (int)(o - (a.W - H)) : (int)o;
            // LDS index of the first (fs 0) / last (fs 1) point of tile tf
            const int ri = side == 0 ? r + (H - q) : r - (q + 1);
            // summed newest level first (the order in which the fused reverse
            // launches accumulate them), then added to acc as one term
            double gsum = 0.0;
            for (int dn = a.L + M - 1; dn >= 0; --dn) {
                const int64_t n2 = a.n + dn;
                if (n2 >= a.nsteps_total) continue;
                const int kk = a.delays[n2 * F + 2 * tf + fs];
                const int j = dn - kk;
                const int need = (kk == 0 || stale) ? 1 : M;
                if (j < 0 || j >= need) continue;
                int64_t ms = a.mslot0 + dn;
                if (ms >= a.Rmu) ms -= a.Rmu;
                const double m = dn == 0 ? mu_now(fs, q, ri)
                                         : a.mu[((ms * a.P + tf) * 2 + fs) * H + q];
                gsum += hweight(kk, stale, j, M) * m;
            }
            acc += gsum;
        }
        a.lam_out[g] = acc;
        acc_add(gacc, lam * (a.dt * D2));
        // publish mu^n of this tile's faces (owners: first and last point of the tile)
        if (o == 0)
            for (int q = 0; q < H; ++q)
                a.mu[(((int64_t)a.mslot0 * a.P + t) * 2 + 0) * H + q] = mu_now(0, q, r);
        if (o == a.W - 1)
            for (int q = 0; q < H; ++q)
                a.mu[(((int64_t)a.mslot0 * a.P + t) * 2 + 1) * H + q] = mu_now(1, q, r);
    }
    gacc = wave_acc(gacc);
    const int lane = tid & 63, wv = tid >> 6;
    if (lane == 0) { red[wv][0] = gacc.s; red[wv][1] = gacc.c; }
    __syncthreads();
    if (tid == 0) {
        Acc S{a.gnu[blockIdx.x * 2], a.gnu[blockIdx.x * 2 + 1]};
        for (int q = 0; q < kThreads / 64; ++q) acc_merge(S, Acc{red[q][0], red[q][1]});
        a.gnu[blockIdx.x * 2] = S.s;
        a.gnu[blockIdx.x * 2 + 1] = S.c;
    }
}

// a + x with the rounding error of the sum collected as in acc_add, by six
// additions instead of a comparison and selections
__device__ __forceinline__ void acc_add_nobranch(Acc &a, double x)
{
    const double t = a.s + x;
    const double y = t - a.s;
    a.c += (a.s - (t - y)) + (x - y);
    a.s = t;
}

// S reverse steps in one launch, one wave per region: RT rim lanes, CT owned
// lanes, RT rim lanes of PPT points each (RAGGED: the first nf lanes of a tile
// PPT, the others PPT - 1, so that any tile width has its lanes).  Every reverse step reads lambda and
// u within h points (across a tile face: the mu of that face, computed from
// points within h of it), so the rims go stale by h points per step, as in the
// forward fused launches (at_wave1d.h); lambda and the levels of u stay in
// registers and neighbours' values move by DPP, so no step has a barrier.
//   * The levels of u are recomputed here, K at a time: a group's lowest level
//     comes from the segment store (every K-th level of the segment), the other
//     K - 1 by forward steps with the recorded delays and edge levels, then the
//     K reverse steps run on them.  The recomputed levels go stale by at most
//     (K - 1) h points from the region's ends, hence rims of (S + K) h points.
//     What bounds this is instruction issue (29 FP64 instructions per
//     point for the reverse step of order 2, 10 for the recomputed one); with
//     every level stored and read back, by 256-thread regions with a barrier per
//     step, a gradient moved 16 bytes per point and step for u alone and the
//     reverse step waited on its latencies.  2^20 points, order 2, 1000 steps (us
//     per step): rebuild 1.7 and reverse 3.0 that way, 0.9 and 2.9 this way
//     (500 tiles of 1003 points, until then one step per launch, reverse: 2.0).
//   * In LDS: the delay rows of the launch's gather window, the record-mode ring
//     levels that the halos of these steps read, and the mu of every face of the
//     region for levels nt .. nt+L+m-2 (from the mu ring), gathered into sums for
//     the levels computed here; their own mu is added as it is computed.
// Each point's lambda^n is summed in the same order as the one-step kernel.
template <int ORDER, bool LINEAR, bool FMA, int PPT, bool RAGGED>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(PPT >= 6 ? 2 : 3)))
void k_adj1d_wave(AdjF a)
{
    constexpr int H = ORDER / 2;
    constexpr int M = (ORDER == 2) ? 2 : 3;
    constexpr int NS = 2 * H;
    constexpr int K = kAdjGroup;
    extern __shared__ double lds[];
    const int S = a.S, NT = a.NT;
    const int DW = a.L + M - 1;               // gather window beyond the step, in levels
    const int LV = S + DW;                    // levels held per history table
    double *eh = lds;                                         // [LV][NT][2][H]: u edges, levels nt-S-DW ..
    double *muh = eh + (size_t)LV * NT * 2 * H;               // [LV][NT][2][H]: mu, levels nt-S ..
    double *gt = muh + (size_t)LV * NT * 2 * H;               // [S][NT][2][H]: gathered mu, levels nt-S ..
    int8_t *kd = reinterpret_cast<int8_t *>(gt + (size_t)S * NT * 2 * H);     // [LV][NT][2]: rows nt-S ..

    const int lane = threadIdx.x;
    const int tpt = a.tpt, P = (int)a.P, NTH = P * tpt;       // threads of a tile, of the grid
    const int c0 = blockIdx.x * a.CT;
    const int owned = NTH - c0 < a.CT ? NTH - c0 : a.CT;
    const int gA = c0 - a.RT;                                 // unwrapped
    const int E = a.RT + owned + a.RT;                        // lanes in use
    int tA = gA / tpt;                                        // tile of lane 0 (unwrapped, floor)
    if (gA < tA * tpt) --tA;
    const int iA = gA - tA * tpt;                             // its index in that tile
    const int tl0 = (iA + lane) / tpt;                        // region-local tile
    const int ti = iA + lane - tl0 * tpt;
    int tb = tA % P;
    if (tb < 0) tb += P;
    const int tp0 = (tb + tl0) % P;
    const bool in_region = lane < E;
    const bool shrt = RAGGED && ti >= a.nf;                   // PPT - 1 points
    const bool lo_edge = ti == 0 && in_region;
    const bool hi_edge = ti == tpt - 1 && in_region;          // (RAGGED: always a short one)
    const bool owns = lane >= a.RT && lane < a.RT + owned;
    const int64_t gb = (int64_t)tp0 * a.W + ti * PPT - (RAGGED && ti > a.nf ? ti - a.nf : 0);
    constexpr int LAST = PPT - (RAGGED ? 1 : 0);              // points of a lane with a right face
    // a lane's points of a field; a short lane's last place holds 0 until its
    // right neighbour's point takes it
    auto load = [&](const double *src, double (&to)[PPT]) {
#pragma unroll
        for (int j = 0; j < PPT; ++j) to[j] = !RAGGED || j < PPT - 1 || !shrt ? src[gb + j] : 0.0;
    };
    const Partials<ORDER> pd = partials<ORDER>(a.coef.c1, a.coef.c2);
    const bool stale = a.stale != 0;
    const int64_t F = 2 * a.P;
    const int64_t nlo = a.nt - S;                             // lowest level computed here
    const double dt = a.coef.dt, nu = a.coef.nu;

    // ---- lambda^{nt} of the lane's points; LDS tables
    double lam[PPT];
    load(a.lam_in, lam);
    {
        const int nk = LV * NT * 2;
#pragma unroll 4
        for (int e = lane; e < nk; e += 64) {
            const int side = e & 1;
            const int tl = (e >> 1) % NT;
            const int r = (e >> 1) / NT;
            const int64_t n2 = nlo + r;
            const int tp = (tb + tl) % P;
            kd[e] = n2 < a.nsteps_total ? a.delays[n2 * F + 2 * tp + side] : (int8_t)0;
        }
        const int nh = LV * NT * 2 * H;
#pragma unroll 2
        for (int e = lane; e < nh; e += 64) {
            const int q = e % H;
            const int side = (e / H) & 1;
            const int tl = (e / (2 * H)) % NT;
            const int r = (e / (2 * H)) / NT;
            const int tp = (tb + tl) % P;
            const int64_t lev = nlo - DW + r;                 // u edge level
            double x = 0.0, y = 0.0;
            if (lev >= 0) x = a.ring[((lev * a.P + tp) * 2 + side) * H + q];
            const int64_t n2 = nlo + r;                       // mu level
            if (n2 >= a.nt && n2 < a.nsteps_total)
                y = a.mu[((n2 % a.Rmu * a.P + tp) * 2 + side) * H + q];
            eh[e] = x;
            muh[e] = y;
        }
    }
    wave_sync();
    // delayed contributions to the levels of this launch from mu levels
    // written by earlier launches (nt ..), newest first; the launch's own mu
    // levels are added by their producers as they are computed
    {
        const int ng = S * NT * 2 * H;
        for (int e = lane; e < ng; e += 64) {
            const int q = e % H;
            const int side = (e / H) & 1;
            const int tl = (e / (2 * H)) % NT;
            const int r = (e / (2 * H)) / NT;
            const int64_t n = nlo + r;
            double g = 0.0;
            int64_t top = n + DW;
            if (top > a.nsteps_total - 1) top = a.nsteps_total - 1;
            for (int64_t n2 = top; n2 >= a.nt && n2 > n; --n2) {
                const int r2 = (int)(n2 - nlo);
                const int kk = kd[(r2 * NT + tl) * 2 + side];
                const int jw = (int)(n2 - n) - kk;
                const int need = (kk == 0 || stale) ? 1 : M;
                if (jw < 0 || jw >= need) continue;
                g += hweight(kk, stale, jw, M) * muh[((r2 * NT + tl) * 2 + side) * H + q];
            }
            gt[e] = g;
        }
    }
    wave_sync();

    // P_s(u) = dt*(nu*g2[s] - a*g1[s]) for a compile-time slot s
    auto Ps = [&](int s, double u) -> double {
        const double adv = LINEAR ? a.coef.cadv : u;
        return dt * (nu * pd.g2[s] - adv * pd.g1[s]);
    };
    // region ends: no source tile in the tables
    const bool lo_src = lo_edge && lane > 0;
    const bool hi_src = hi_edge && lane < 63;
    // the AT halo across this lane's faces at row `krow` (level nlo + krow) into
    // the window's ends; contracted: the rounding of the contracted forward step
    auto halo = [&](auto contracted, int krow, double *w) {
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            if (side == 0 ? !lo_src : !hi_src) continue;
            const int kk = kd[(krow * NT + tl0) * 2 + side];
            if (kk > 0) {
                const int stl = side == 0 ? tl0 - 1 : tl0 + 1;
#pragma unroll
                for (int q = 0; q < H; ++q) {
                    double vv[3] = {0.0, 0.0, 0.0};
#pragma unroll
                    for (int jj = 0; jj < M; ++jj)
                        if (jj == 0 || !stale)
                            vv[jj] = eh[((krow + DW - kk - jj) * NT + stl) * 2 * H + (1 - side) * H + q];
                    const double hv = extrap<decltype(contracted)::value>(kk, stale, vv[0], vv[1],
                                                                          vv[2], M);
                    if (side == 0) w[q] = hv;
                    else w[LAST + H + q] = hv;
                }
            }
        }
    };
    // first and last points of the neighbouring lanes: into the places to the
    // left and right of the lane's own points (a short lane: its last place and
    // the one after)
    auto around = [&](double (&w)[PPT + 2 * H]) {
        double l[H], r[H];
#pragma unroll
        for (int q = 0; q < H; ++q) {
            const double end = RAGGED ? (shrt ? w[PPT - 1 + q] : w[PPT + q]) : w[PPT + q];
            l[q] = from_left<false>(0.0, end);
            r[q] = from_right<false>(0.0, w[H + q]);
        }
#pragma unroll
        for (int q = 0; q < H; ++q) w[q] = l[q];
        if constexpr (RAGGED) {
            w[H + PPT - 1] = shrt ? r[0] : w[H + PPT - 1];
#pragma unroll
            for (int q = 0; q < H; ++q)
                w[H + PPT + q] = shrt ? r[q + 1 < H ? q + 1 : q] : r[q];
        } else {
#pragma unroll
            for (int q = 0; q < H; ++q) w[H + PPT + q] = r[q];
        }
    };
    using exact = std::integral_constant<bool, false>;

    const int mslot0 = (int)(nlo % a.Rmu);
    Acc gacc{0.0, 0.0};                           // of all lanes; the rims' are dropped below
    // one reverse step: level nlo + krow from lambda of the level above (lam) and
    // its own u (uc)
    auto rstep = [&](int krow, const double (&uc)[PPT]) {
        // lambda and raw u of the points -H .. PPT+H-1
        double lw[PPT + 2 * H], rw[PPT + 2 * H];
#pragma unroll
        for (int j = 0; j < PPT; ++j) { lw[H + j] = lam[j]; rw[H + j] = uc[j]; }
        around(lw);
        around(rw);
        // the delays and gathered sums at this level of the neighbours' faces
        // that this lane's edge points feed
        int kown[2] = {0, 0}, knb[2] = {1, 1};
        double gth[2][H];
#pragma unroll
        for (int q = 0; q < H; ++q) { gth[0][q] = 0.0; gth[1][q] = 0.0; }
        if (lo_edge) kown[0] = kd[(krow * NT + tl0) * 2 + 0];
        if (hi_edge) kown[1] = kd[(krow * NT + tl0) * 2 + 1];
        if (hi_src) {                             // feeds the next tile's low face
            knb[0] = kd[(krow * NT + tl0 + 1) * 2 + 0];
#pragma unroll
            for (int q = 0; q < H; ++q) gth[0][q] = gt[((krow * NT + tl0 + 1) * 2 + 0) * H + q];
        }
        if (lo_src) {                             // feeds the previous tile's high face
            knb[1] = kd[(krow * NT + tl0 - 1) * 2 + 1];
#pragma unroll
            for (int q = 0; q < H; ++q) gth[1][q] = gt[((krow * NT + tl0 - 1) * 2 + 1) * H + q];
        }
        // ---- u window with the forward AT halo across the tile faces
        double uw[PPT + 2 * H];
#pragma unroll
        for (int i = 0; i < PPT + 2 * H; ++i) uw[i] = rw[i];
        if (lo_edge || hi_edge) halo(exact{}, krow, uw);
        // lambda and raw u at window index i (-H .. PPT+H-1), compile-time i
        auto lat = [&](int i) -> double { return lw[H + i]; };
        auto uat = [&](int i) -> double { return rw[H + i]; };
        // mu^n of this step for the face a point feeds, from the raw window
        auto mu_lo = [&](int q) -> double {         // face of the next tile, low side: its first h points
            double m = 0.0;
#pragma unroll
            for (int e = 0; e < H; ++e)
                if (e <= q) m += lat(LAST + e) * Ps(q - e, uat(LAST + e));
            return m;
        };
        auto mu_hi = [&](int q) -> double {         // face of the previous tile, high side: its last h points
            double m = 0.0;
#pragma unroll
            for (int e = 0; e < H; ++e)
                if (e <= H - 1 - q) m += lat(-1 - e) * Ps(H + q + e, uat(-1 - e));
            return m;
        };
        double res[PPT];
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            const double u = uc[j];
            double nb[NS];
#pragma unroll
            for (int q = 0; q < H; ++q) { nb[q] = uw[j + q]; nb[H + q] = uw[j + H + 1 + q]; }
            double D1, D2;
            if constexpr (ORDER == 2) {
                D1 = (nb[1] - nb[0]) * a.coef.c1;
                D2 = ((nb[1] - 2.0 * u) + nb[0]) * a.coef.c2;
            } else {
                D1 = (8.0 * (nb[2] - nb[1]) - (nb[3] - nb[0])) * a.coef.c1;
                D2 = ((16.0 * (nb[2] + nb[1]) - 30.0 * u) - (nb[3] + nb[0])) * a.coef.c2;
            }
            const double lg = lam[j];
            const double du = 1.0 + dt * (nu * pd.g2u - (LINEAR ? 0.0 : D1));
            double acc = lg * du;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int d = (s < H) ? -(H - s) : (s - H + 1);
                const int i = j - d;
                // (a neighbour in another tile: a product that is not added)
                const bool same = (i >= 0 || !lo_edge) && (i < LAST || !hi_edge);
                if (i >= 0 && i < LAST) acc += lat(i) * Ps(s, uat(i));
                else if (same) acc += lat(i) * Ps(s, uat(i));
            }
            // delayed halo contributions gathered over steps n .. n+L+m-1
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const bool feeds = side == 0 ? (hi_src && j >= LAST - H && j < LAST)
                                             : (lo_src && j < H);
                if (!feeds) continue;
                const int q = side == 0 ? j - (LAST - H) : j;
                // later levels' contributions, accumulated newest first by their
                // producers; then this level's own (k = 0: the raw neighbour)
                double g = gth[side][q];
                if (knb[side] == 0)
                    g += hweight(0, stale, 0, M) * (side == 0 ? mu_lo(q) : mu_hi(q));
                acc += g;
            }
            res[j] = acc;
            const double x = lg * (dt * D2);
            acc_add_nobranch(gacc, !RAGGED || j < PPT - 1 || !shrt ? x : 0.0);
        }
        // ---- mu^n of this tile's faces: added to the gathered sums of the
        // earlier levels of this launch that it feeds (n-k-j, weight dH/dv_j),
        // and to the ring for later launches
        auto scatter = [&](int side, int q, double m) {
            const int kk = kown[side];
            const int need = (kk == 0 || stale) ? 1 : M;
            for (int jw = 0; jw < need; ++jw) {
                const int row = krow - kk - jw;       // row of the level it belongs to
                if (row == krow || row < 0) continue; // own level: gathered directly
                gt[((row * NT + tl0) * 2 + side) * H + q] += hweight(kk, stale, jw, M) * m;
            }
        };
        if (lo_edge || hi_edge) {
            int ms = mslot0 + krow;
            while (ms >= a.Rmu) ms -= a.Rmu;
#pragma unroll
            for (int q = 0; q < H; ++q) {
                if (lo_edge) {                        // own first h points feed the low face
                    double m = 0.0;
#pragma unroll
                    for (int e = 0; e < H; ++e)
                        if (e <= q) m += lam[e] * Ps(q - e, uc[e]);
                    scatter(0, q, m);
                    if (owns) a.mu[(((int64_t)ms * a.P + tp0) * 2 + 0) * H + q] = m;
                }
                if (hi_edge) {                        // own last h points feed the high face
                    double m = 0.0;
#pragma unroll
                    for (int e = 0; e < H; ++e)
                        if (e <= H - 1 - q) m += lam[LAST - 1 - e] * Ps(H + q + e, uc[LAST - 1 - e]);
                    scatter(1, q, m);
                    if (owns) a.mu[(((int64_t)ms * a.P + tp0) * 2 + 1) * H + q] = m;
                }
            }
        }
        wave_sync();
#pragma unroll
        for (int j = 0; j < PPT; ++j) lam[j] = res[j];
    };
    // one forward step: level nlo + krow (u) to the one above (to)
    auto fstep = [&](int krow, const double (&u)[PPT], double (&to)[PPT]) {
        double w[PPT + 2 * H];
#pragma unroll
        for (int j = 0; j < PPT; ++j) w[H + j] = u[j];
        around(w);
        if (lo_edge || hi_edge) halo(std::integral_constant<bool, FMA>{}, krow, w);
        step_window<ORDER, LINEAR, FMA, PPT>(w, a.coef);
#pragma unroll
        for (int j = 0; j < PPT; ++j) to[j] = w[H + j];
    };

    // ---- groups of levels, from the top: base .. base + K - 1 (the first one
    // may stop below; nt - S is the base of the last one)
    double U[K][PPT], next[PPT];
    int64_t base = a.seg_n0 + (a.nt - 1 - a.seg_n0) / K * K;
    const auto level = [&](int64_t lev) { return a.seg + (lev - a.seg_n0) * a.N; };
    load(level(base), next);
    for (int count = (int)(a.nt - base); base >= nlo; base -= K, count = K) {
        const int b = (int)(base - nlo);
#pragma unroll
        for (int j = 0; j < PPT; ++j) U[0][j] = next[j];
        if (base - K >= nlo) load(level(base - K), next);        // the next group's, in flight meanwhile
#pragma unroll
        for (int i = 0; i + 1 < K; ++i)
            if (i + 1 < count) fstep(b + i, U[i], U[i + 1]);
#pragma unroll
        for (int i = K - 1; i >= 0; --i)
            if (i < count) rstep(b + i, U[i]);
    }

    if (owns) {
#pragma unroll
        for (int j = 0; j < PPT; ++j)
            if (!RAGGED || j < PPT - 1 || !shrt) a.lam_out[gb + j] = lam[j];
    }
    if (!owns) gacc = Acc{0.0, 0.0};
    gacc = wave_acc(gacc);
    if (lane == 0) {
        Acc Sg{a.gnu[blockIdx.x * 2], a.gnu[blockIdx.x * 2 + 1]};
        acc_merge(Sg, gacc);
        a.gnu[blockIdx.x * 2] = Sg.s;
        a.gnu[blockIdx.x * 2 + 1] = Sg.c;
    }
}

}  // namespace

int adj1d_points_per_block() { return kCHA; }

hipError_t launch_adj1d_fused(const AdjF &a, int order, bool linear, bool fma, int ppt,
                              int64_t nblocks, size_t lds, hipStream_t st)
{
    const dim3 grid((unsigned)nblocks), block(64);
#define AT_AF(O, LI, F, P, R) hipLaunchKernelGGL((k_adj1d_wave<O, LI, F, P, R>), grid, block, lds, st, a)
#define AT_AFP(O, LI, F) do { \
        if (a.nf == a.tpt) { if (ppt == 8) AT_AF(O, LI, F, 8, false); else AT_AF(O, LI, F, 4, false); } \
        else if (ppt == 10) AT_AF(O, LI, F, 10, true); \
        else if (ppt == 8) AT_AF(O, LI, F, 8, true); \
        else if (ppt == 6) AT_AF(O, LI, F, 6, true); \
        else AT_AF(O, LI, F, 4, true); \
    } while (0)
    if (ppt != 4 && ppt != 8 && (a.nf == a.tpt || (ppt != 6 && ppt != 10))) return hipErrorInvalidValue;
    if (order == 2) {
        if (linear) { if (fma) AT_AFP(2, true, true); else AT_AFP(2, true, false); }
        else { if (fma) AT_AFP(2, false, true); else AT_AFP(2, false, false); }
    } else {
        if (linear) { if (fma) AT_AFP(4, true, true); else AT_AFP(4, true, false); }
        else { if (fma) AT_AFP(4, false, true); else AT_AFP(4, false, false); }
    }
#undef AT_AFP
#undef AT_AF
    return hipGetLastError();
}

size_t adj1d_fused_lds_bytes(int order, int S, int NT, int L)
{
    const int H = order / 2, M = order == 2 ? 2 : 3;
    const size_t LV = (size_t)S + L + M - 1;
    const size_t dbl = 2 * LV * NT * 2 * H + (size_t)S * NT * 2 * H;
    return 8 * dbl + ((LV * NT * 2 + 7) / 8) * 8;
}

hipError_t launch_adj1d(const Adj1D &a, int order, bool linear, int64_t nblocks, hipStream_t st)
{
    dim3 grid((unsigned)nblocks), block(kThreads);
    if (order == 2) {
        if (linear) hipLaunchKernelGGL((k_adj1d<2, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_adj1d<2, false>), grid, block, 0, st, a);
    } else {
        if (linear) hipLaunchKernelGGL((k_adj1d<4, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_adj1d<4, false>), grid, block, 0, st, a);
    }
    return hipGetLastError();
}

}  // namespace atk
