// Fused 1D stepper kernels of libat.so for gfx950 (k_wave1d, k_wave1d_batch;
// instantiated per order in at_wave1d_o2.hip and at_wave1d_o4.hip).
//
// Method and evaluation order as in at_step1d.hip (paper section 3.2 stencils
// with forward Euler; AT halos of section 2, Eqs. (1)-(2), at tile edges), so
// the bits are those of one launch per step.
//
// Decomposition.  The grid is cut into threads of PPT consecutive points; a
// tile of W points is tpt = ceil(W / PPT) threads, the first nf of them with
// PPT points and the others with PPT - 1 (RAGGED; nf = tpt when PPT divides
// W), so that every thread lies in one tile whatever the width.  A workgroup
// of NW waves holds a region of RT rim threads, CT owned threads and RT rim
// threads and advances it S levels; the rims go stale by h points per step
// (overlapped trapezoids), and the tile edges inside the region are recomputed
// with the same operations as their owner's.
//   * What bounds it is FP64 issue (15 instructions per 4th-order update in
//     the exact order, 10 contracted) on large grids, the latency of a step's
//     dependent instructions on small ones.  A thread's neighbours are one lane
//     away, so the exchange is a DPP wavefront shift; with one wave per region
//     (NW = 1) no step has a barrier, and a region advances at the pace of its
//     own instructions.  NW = 4 (16 points per thread) has smaller rims for its
//     size and trades the waves' end values through LDS with a barrier per
//     step: better only where the chip is full many times over.
//   * Points per thread: more points share the exchange and the AT work of a
//     step and make the rims a smaller part of the region; fewer make more
//     waves, which a small grid needs.  Between those the number of waves per
//     SIMD decides, which is a whole number: hence kinds at 6, 10, 12, 20 and 24
//     points too (built for ragged threads only, which any width can have).
//   * AT halos.  What a lane at a tile face needs across it, the raw
//     neighbour values of the levels n-1 .. n-D (D = L + m - 1), is what the
//     exchange handed it in earlier steps; it keeps them in an LDS ring of its
//     own.  A step's delayed halos (k >= 1) read only levels below it, so they
//     are formed during the step before, next to its stencil and off the chain
//     from step to step.  Waves without a tile face run a loop without this.
//   * The ring rows are stored twice, HR = D + 1 rows apart, so that a read
//     never wraps.  The delays of the S steps are an LDS table: no step waits
//     on a global load.
//   * Measured against 256-thread regions that traded every thread's edges
//     through LDS (us per step, autotuned): order 2, N = 1024: 0.74 -> 0.26,
//     2^18: 0.70 -> 0.34, 2^20: 0.99 -> 0.65; order 4, N = 2^22: 3.45 -> 2.9,
//     contracted 2.79 -> 2.2.  Widths that 16, 8 and 4 points do not divide
//     had one step per launch: 999 tiles of 1001 points 20.6 -> 0.92.
#pragma once

#include <type_traits>

#include "at_internal.h"
#include "at_stencil1d.h"
#include "at_wave.h"

namespace atk {

namespace {

constexpr int kWave = 64;

// the field passes through the LDS stage in parts of at most 640 points per
// wave, so that LDS does not cap the waves per CU
__host__ __device__ constexpr int wave_parts(int ppt)
{
    return ppt <= 10 ? 1 : (ppt <= 20 ? 2 : 4);
}

// region points of a part
__host__ __device__ constexpr int wave_stage_pts(int ppt, int nw)
{
    return nw * ppt * kWave / wave_parts(ppt);
}

// the stage (one pad per PPT points), then the waves' end values [2][NW][2][2]
__host__ __device__ constexpr int wave_stage_doubles(int ppt, int nw)
{
    return wave_stage_pts(ppt, nw) + wave_stage_pts(ppt, nw) / ppt + (nw > 1 ? 8 * nw : 0);
}

template <int NW>
__device__ __forceinline__ void region_sync()
{
    if constexpr (NW == 1) wave_sync();
    else __syncthreads();
}

template <int ORDER, bool LINEAR, bool FMA, int PPT, bool RAGGED, int NW>
__device__ __forceinline__ void wave1d_body(const Step1D &a, const int chunk)
{
    constexpr int H = ORDER / 2;
    constexpr int M = (ORDER == 2) ? 2 : 3;
    constexpr int NL = NW * kWave;                    // threads of the region
    constexpr int SP = wave_stage_pts(PPT, NW);       // points per stage part
    constexpr int PARTS = PPT * NL / SP;
    constexpr int IT = PPT / PARTS;                   // loads per thread in one part
    constexpr int LP = NL / PARTS;                    // threads whose points a part holds
    // a tile of one thread, whose lane has both faces: only for the narrowest
    // regions (the host picks fewer points per thread otherwise)
    constexpr bool BOTH = PPT == 4 && !RAGGED;
    extern __shared__ double lds[];
    const int lane = threadIdx.x;
    const int S = a.s, D = a.D, HR = D + 1, NF = 2 * a.NT;
    const int tpt = a.tpt, P = (int)a.P;
    const int RS = (NF + 1) * H;                      // doubles of a history row: the faces, and one
                                                      // place for the lanes without a face
    double *stage = lds;
    double *eh = lds + wave_stage_doubles(PPT, NW);   // [2 HR][NT][2][H], twice the rows of level
                                                      // n0 + x: (x + D) mod HR
    int8_t *kd = reinterpret_cast<int8_t *>(eh + 2 * HR * RS);       // [S + 2][NT][2]

    // ---- threads of the region: global thread gA + lane, tile and index in it
    const int NTH = P * tpt;                          // threads of the grid
    const int c0 = chunk * a.CT;
    const int owned = NTH - c0 < a.CT ? NTH - c0 : a.CT;
    const int gA = c0 - a.RT;                         // unwrapped
    const int E = a.RT + owned + a.RT;                // lanes in use
    int tA = gA / tpt;                                // tile of lane 0 (unwrapped, floor)
    if (gA < tA * tpt) --tA;
    const int iA = gA - tA * tpt;                     // its index in that tile
    const int tl = (iA + lane) / tpt;                 // region-local tile
    const int ti = iA + lane - tl * tpt;
    int tb = tA % P;
    if (tb < 0) tb += P;                              // physical tile of lane 0
    const bool shrt = RAGGED && ti >= a.nf;           // PPT - 1 points
    // first point of the lane, relative to lane 0's
    const auto in_tile = [&](int i) { return i * PPT - (RAGGED && i > a.nf ? i - a.nf : 0); };
    const int W = (int)a.W;
    const int sA = in_tile(iA);
    // first point of thread x of the region, relative to thread 0's
    const auto first = [&](int x) {
        const int q = (iA + x) / tpt;
        return q * W + in_tile(iA + x - q * tpt) - sA;
    };
    const int r0 = tl * W + in_tile(ti) - sA;
    const int64_t G0 = (int64_t)tb * W + sA;          // periodic index of the region's first point
    const bool lo_edge = ti == 0 && lane < E;
    const bool hi_edge = ti == tpt - 1 && lane < E;
    const bool owns = lane >= a.RT && lane < a.RT + owned;

    // ---- sources of the delay table and of the history of the levels below
    // n0: a pass of the wave covers kr (er) whole rows; the first passes' loads
    // go out before the field's, so that all their latencies overlap
    const auto wrap = [&](int t) { while (t >= P) t -= P; return t; };
    constexpr int KP = 4, EP = 2;
    const int kt = lane / NF, kx = lane - kt * NF, kr = NL / NF;
    const int NE = NF * H, et = lane / NE, ex = lane - et * NE, er_ = NL / NE;
    const bool kfast = NF <= NL, efast = NE <= NL;
    const int8_t *ksrc = a.delays + a.n0 * (2 * a.P) + 2 * wrap(tb + (kx >> 1)) + (kx & 1);
    // face x / H of the region: the tile across it and that tile's facing side
    const auto across = [&](int x) -> const double * {
        const int f = x / H, side = f & 1, t = tb + (f >> 1) + (side ? 1 : P - 1);
        return a.ring + (2 * wrap(t) + 1 - side) * H + x % H;
    };
    const int64_t lev_doubles = a.P * 2 * H;
    const auto old_level = [&](const double *src, int d) -> double {   // level n0 - D + d
        if (a.n0 - D + d < 0) return 0.0;
        int slot = a.slot0 - D + d;
        if (slot < 0) slot += a.R;
        return src[slot * lev_doubles];
    };
    int8_t kv[KP];
    double ev[EP];
    const double *esrc = a.ring;
    if (kfast && kt < kr) {
#pragma unroll
        for (int i = 0; i < KP; ++i)
            if (kt + i * kr < S) kv[i] = ksrc[(int64_t)(kt + i * kr) * (2 * a.P)];
    }
    if (efast && et < er_) {
        esrc = across(ex);
#pragma unroll
        for (int i = 0; i < EP; ++i)
            if (et + i * er_ < D) ev[i] = old_level(esrc, et + i * er_);
    }

    // place of a part's point in the stage: one pad after every PPT, so that
    // neither the coalesced accesses nor the per-lane ones conflict on banks
    const auto place = [](int rr) { return rr + (int)((unsigned)rr / PPT); };
    double w[PPT + 2 * H];
    {
        // two parts of the stage in flight: their latencies overlap, and the
        // window does not share the registers with more
        double v[2][IT];
        const bool inside = G0 + PPT * NL <= a.N;
        const auto load = [&](int h, double (&to)[IT]) {
            const int rp = RAGGED ? first(h * LP) : h * SP;
            if (inside) {
                const double *src = a.uin + G0 + rp;
#pragma unroll
                for (int i = 0; i < IT; ++i) to[i] = src[i * NL + lane];
            } else if (a.N >= (int64_t)PPT * NL) { // the region wraps once
#pragma unroll
                for (int i = 0; i < IT; ++i) {
                    const int64_t g = G0 + rp + i * NL + lane;
                    to[i] = a.uin[g >= a.N ? g - a.N : g];
                }
            } else {                                  // a grid shorter than a region
#pragma unroll
                for (int i = 0; i < IT; ++i)
                    to[i] = a.uin[((unsigned)G0 + (unsigned)(rp + i * NL + lane)) % (unsigned)a.N];
            }
        };
        load(0, v[0]);
        if constexpr (PARTS > 1) load(1, v[1]);
        // delays (two rows of zeros follow the last) and history into LDS
        if (kfast) {
            if (kt < kr) {
#pragma unroll
                for (int i = 0; i < KP; ++i)
                    if (kt + i * kr < S) kd[(kt + i * kr) * NF + kx] = kv[i];
#pragma unroll 4
                for (int t = kt + KP * kr; t < S; t += kr) kd[t * NF + kx] = ksrc[(int64_t)t * (2 * a.P)];
            }
        } else {
            for (int e = lane; e < S * NF; e += NL) {
                const int t = e / NF, x = e - t * NF;
                kd[e] = a.delays[(a.n0 + t) * (2 * a.P) + 2 * wrap(tb + (x >> 1)) + (x & 1)];
            }
        }
        for (int e = lane; e < 2 * NF; e += NL) kd[S * NF + e] = 0;
        const auto old_to_lds = [&](int d, int x, double v1) {
            eh[d * RS + x] = v1;
            eh[(d + HR) * RS + x] = v1;
        };
        if (efast) {
            if (et < er_) {
#pragma unroll
                for (int i = 0; i < EP; ++i)
                    if (et + i * er_ < D) old_to_lds(et + i * er_, ex, ev[i]);
#pragma unroll 4
                for (int d = et + EP * er_; d < D; d += er_) old_to_lds(d, ex, old_level(esrc, d));
            }
        } else {
            for (int e = lane; e < D * NE; e += NL) {
                const int d = e / NE, x = e - d * NE;
                old_to_lds(d, x, old_level(across(x), d));
            }
        }
#pragma unroll
        for (int h = 0; h < PARTS; ++h) {
            const int rp = RAGGED ? first(h * LP) : h * SP;
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                stage[place(i * NL + lane)] = v[h & 1][i];
            }
            if (h + 2 < PARTS) load(h + 2, v[h & 1]);
            region_sync<NW>();
            if (lane / LP == h) {
#pragma unroll
                for (int j = 0; j < PPT; ++j) {
                    // (a short lane's last place reads the next lane's first point, unused)
                    w[H + j] = stage[RAGGED ? place(r0 - rp + j) : (lane % LP) * (PPT + 1) + j];
                }
            }
            region_sync<NW>();
        }
    }
#pragma unroll
    for (int q = 0; q < H; ++q) { w[q] = 0.0; w[PPT + H + q] = 0.0; }

    // ---- a lane's face: its left one where it starts a tile, else its right
    // one where it ends a tile (BOTH: the right one of a one-thread tile apart).
    // The other lanes run along on the spare place, with no delay.
    const bool edge = lo_edge || hi_edge;
    const int face = edge ? 2 * tl + (lo_edge ? 0 : 1) : NF;
    const int face2 = edge ? 2 * tl + 1 : NF;
    // halo of a face at delay kk for the step whose level has history row
    // `row`: levels kk, kk+1, (kk+2) below it
    const auto at_halo = [&](int kk, int row, int f, double (&out)[H]) {
        const double *p0 = eh + (row + HR) * RS + f * H - __umul24(kk, RS);
        double v[3][H];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int q = 0; q < H; ++q) v[j][q] = j < M ? p0[q - j * RS] : 0.0;
#pragma unroll
        for (int q = 0; q < H; ++q)
            out[q] = extrap<FMA>(kk, a.stale != 0, v[0][q], v[1][q], v[2][q], M);
    };
    int tphys = tb + tl;
    while (tphys >= P) tphys -= P;

    // ---- the S steps: steps t < plain with nothing to write, the rest with
    // ring or level stores (a loop of their own, so that the first has no
    // instruction for them).  row: history row of level n; kc, hv: this step's
    // delay and delayed halo (kc2, hv2: of the second face); kn: the next
    // step's delay, kp its place in the table.
    double *ends = lds + SP + SP / PPT;               // NW > 1: [2][NW][2][H]
    const int wl = lane % kWave;
    const int wv = NW > 1 ? __builtin_amdgcn_readfirstlane(lane / kWave) : 0;
    const int wprev = wv > 0 ? wv - 1 : 0, wnext = wv + 1 < NW ? wv + 1 : wv;
    int plain = S;
    if (a.levels || a.publish == 1) plain = 0;
    else if (a.publish == 2) plain = S > D ? S - D : 0;
    int t = 0, row = D;
    int kc = 0, kn = 0, kc2 = 0, kn2 = 0;
    double hv[H], hv2[H];
#pragma unroll
    for (int q = 0; q < H; ++q) hv[q] = hv2[q] = 0.0;
    const int8_t *kp = edge ? kd + face : kd + S * NF, *kp2 = edge ? kd + face2 : kd + S * NF;
    const int kstep = edge ? NF : 0;
    const auto steps = [&](auto at_, auto two_, auto stores_, const int end) {
        constexpr bool AT = decltype(at_)::value, TWO = decltype(two_)::value;
        constexpr bool STORES = decltype(stores_)::value;
        for (; t < end; ++t) {
            // ---- first and last points to the neighbouring lanes
            double el[H], er[H], hl[H], hr[H];
#pragma unroll
            for (int q = 0; q < H; ++q) {
                el[q] = w[H + q];
                er[q] = RAGGED ? (shrt ? w[PPT - 1 + q] : w[PPT + q]) : w[PPT + q];
                hl[q] = hr[q] = 0.0;
            }
            if constexpr (NW > 1) {
                // the waves' ends through LDS: a wave reads the right end of the
                // one before it and the left end of the one after it (the first
                // and last their own: rims).  Every wave takes one barrier a step.
                double *x = ends + (t & 1) * (NW * 2 * H);
                if (wl == 0) {
#pragma unroll
                    for (int q = 0; q < H; ++q) x[wv * 2 * H + q] = el[q];
                }
                if (wl == kWave - 1) {
#pragma unroll
                    for (int q = 0; q < H; ++q) x[wv * 2 * H + H + q] = er[q];
                }
                __syncthreads();
#pragma unroll
                for (int q = 0; q < H; ++q) {
                    hl[q] = x[wprev * 2 * H + H + q];
                    hr[q] = x[wnext * 2 * H + q];
                }
            }
#pragma unroll
            for (int q = 0; q < H; ++q) {
                hl[q] = from_left<(NW > 1)>(hl[q], er[q]);
                hr[q] = from_right<(NW > 1)>(hr[q], el[q]);
            }
            if constexpr (AT) {
                // ---- own tile edges to the global ring, for the levels a later
                // launch reads (every level with the edge tape)
                if (STORES && a.publish && owns && edge) {
                    int slot = a.slot0 + t;
                    if (slot >= a.R) slot -= a.R;
                    double *dst = a.ring + slot * lev_doubles + (int64_t)tphys * (2 * H);
#pragma unroll
                    for (int q = 0; q < H; ++q) {
                        if (lo_edge) dst[q] = el[q];
                        if (hi_edge) dst[H + q] = er[q];
                    }
                }
                // ---- the raw values across the face join its history; the delayed
                // halo replaces them where this step's delay is positive
                {
                    double *h0 = eh + row * RS + face * H, *h1 = h0 + HR * RS;
#pragma unroll
                    for (int q = 0; q < H; ++q) h0[q] = h1[q] = lo_edge ? hl[q] : hr[q];
                    if constexpr (TWO) {
                        double *g0 = eh + row * RS + face2 * H, *g1 = g0 + HR * RS;
#pragma unroll
                        for (int q = 0; q < H; ++q) g0[q] = g1[q] = hr[q];
                    }
                }
                const bool dl = kc > 0 && lo_edge, dr = kc > 0 && !lo_edge;
#pragma unroll
                for (int q = 0; q < H; ++q) {
                    hl[q] = dl ? hv[q] : hl[q];
                    hr[q] = dr ? hv[q] : hr[q];
                    if constexpr (TWO) hr[q] = kc2 > 0 ? hv2[q] : hr[q];
                }
                row = row + 1 == HR ? 0 : row + 1;
                kc = kn;
                // (many points per thread: issue is what counts, so only where a
                // delay asks for it)
                if (PPT < 16 || __any(kc > 0)) at_halo(kc, row, face, hv);
                kn = *kp;
                kp += kstep;
                if constexpr (TWO) {
                    kc2 = kn2;
                    at_halo(kc2, row, face2, hv2);
                    kn2 = *kp2;
                    kp2 += kstep;
                }
            }
            // ---- the window with its halos, then the standard stencil on every point
#pragma unroll
            for (int q = 0; q < H; ++q) w[q] = hl[q];
            if constexpr (RAGGED) {
                w[H + PPT - 1] = shrt ? hr[0] : w[H + PPT - 1];
#pragma unroll
                for (int q = 0; q < H; ++q)
                    w[H + PPT + q] = shrt ? hr[q + 1 < H ? q + 1 : q] : hr[q];
            } else {
#pragma unroll
                for (int q = 0; q < H; ++q) w[H + PPT + q] = hr[q];
            }
            step_window<ORDER, LINEAR, FMA, PPT>(w, a);
            // every levels_every-th intermediate level of the owned points, straight
            // from registers (used to rebuild a checkpoint segment for the adjoint)
            if (STORES && a.levels && owns && t + 1 < S && (t + 1) % a.levels_every == 0) {
                double *dst = a.levels + (int64_t)(t + 1) * a.N + (int64_t)tphys * W + in_tile(ti);
#pragma unroll
                for (int j = 0; j < PPT; ++j)
                    if (!RAGGED || j < PPT - 1 || !shrt) dst[j] = w[H + j];
            }
        }
    };
    using yes = std::integral_constant<bool, true>;
    using no = std::integral_constant<bool, false>;
    const auto run = [&](auto at_, auto two_) {
        if constexpr (decltype(at_)::value) {
            kc = kp[0];
            kn = kp[kstep];
            kp += 2 * kstep;
            at_halo(kc, row, face, hv);
            if constexpr (decltype(two_)::value) {
                kc2 = kp2[0];
                kn2 = kp2[kstep];
                kp2 += 2 * kstep;
                at_halo(kc2, row, face2, hv2);
            }
        }
        steps(at_, two_, no{}, plain);
        steps(at_, two_, yes{}, S);
    };
    if (!__any(edge)) run(no{}, no{});
    else if (!BOTH || tpt != 1) run(yes{}, no{});
    else run(yes{}, std::integral_constant<bool, BOTH>{});

    // ---- level n0 + S of the owned points through the stage, coalesced
    const int lo = first(a.RT), hi = first(a.RT + owned);             // region points to store
    const int64_t o0 = (int64_t)(c0 / tpt) * W + in_tile(c0 % tpt);   // the first owned point
#pragma unroll
    for (int h = 0; h < PARTS; ++h) {
        const int rp = RAGGED ? first(h * LP) : h * SP;
        const int re = RAGGED ? first((h + 1) * LP) : (h + 1) * SP;    // the next part's first point
        if (lane / LP == h) {
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                if (!RAGGED || j < PPT - 1 || !shrt)
                    stage[RAGGED ? place(r0 - rp + j) : (lane % LP) * (PPT + 1) + j] = w[H + j];
            }
        }
        region_sync<NW>();
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int r = rp + i * NL + lane;
            if (r >= lo && r < hi && r < re) a.uout[o0 + (r - lo)] = stage[place(r - rp)];
        }
        region_sync<NW>();
    }
}

// Waves per SIMD the registers are held to: three at 24 and 32 points (at 32,
// 128 VGPRs spilled around the loops: 10.0 against 9.6 us per step at 2^24
// points; two, without any spill, 5.58 against 5.43 ms for a batch), four from 10
// points (four-wave regions held to five spilled 36 VGPRs around the loops, 117 MB
// of scratch written per launch of 2^24 points: 9.26 against 9.03 us per step),
// five below
constexpr int wave_occupancy(int ppt) { return ppt >= 24 ? 3 : (ppt >= 10 ? 4 : 5); }

template <int ORDER, bool LINEAR, bool FMA, int PPT, bool RAGGED, int NW>
__global__ __launch_bounds__(kWave * NW)
__attribute__((amdgpu_waves_per_eu(wave_occupancy(PPT))))
void k_wave1d(Step1D a)
{
    wave1d_body<ORDER, LINEAR, FMA, PPT, RAGGED, NW>(a, blockIdx.x);
}

// Batched form: workgroup b advances chunk tbl[b].y of instance tbl[b].x;
// instance descriptors carry each instance's grid, ring, delays and
// coefficients; flip = 1 swaps the field pointers (ping-pong launches).
template <int ORDER, bool LINEAR, bool FMA, int PPT>
__global__ __launch_bounds__(kWave)
__attribute__((amdgpu_waves_per_eu(wave_occupancy(PPT))))
void k_wave1d_batch(const Step1D *descs, const int2 *tbl, int64_t n0, int flip)
{
    const int2 e = tbl[blockIdx.x];
    Step1D a = descs[e.x];
    a.n0 = n0;
    a.slot0 = (int32_t)(n0 % a.R);    // once per workgroup (uniform)
    if (flip) {
        const double *t = a.uin;
        a.uin = a.uout;
        a.uout = const_cast<double *>(t);
    }
    wave1d_body<ORDER, LINEAR, FMA, PPT, false, 1>(a, e.y);
}

template <int ORDER>
hipError_t launch_wave1d_order(const Step1D &a, bool linear, bool fma, int ppt, int nw,
                               int64_t nblocks, size_t lds, hipStream_t st)
{
    const dim3 grid((unsigned)nblocks), block(kWave * nw);
    const bool ragged = a.nf != a.tpt;
#define AT_WV(LI, F, P, RG, NW) hipLaunchKernelGGL((k_wave1d<ORDER, LI, F, P, RG, NW>), grid, block, lds, st, a)
#define AT_WR(LI, F, P, NW) do { if (ragged) AT_WV(LI, F, P, true, NW); else AT_WV(LI, F, P, false, NW); } while (0)
#define AT_WP(LI, F)                                                                     \
    do {                                                                                 \
        if (nw == 4 && ppt == 16 && !ragged) AT_WV(LI, F, 16, false, 4);                 \
        else if (nw != 1) return hipErrorInvalidValue;                                   \
        else if (ppt == 32) AT_WR(LI, F, 32, 1);                                         \
        else if (ppt == 24) AT_WV(LI, F, 24, true, 1);                                   \
        else if (ppt == 20) AT_WV(LI, F, 20, true, 1);                                   \
        else if (ppt == 12) AT_WV(LI, F, 12, true, 1);                                   \
        else if (ppt == 10) AT_WV(LI, F, 10, true, 1);                                   \
        else if (ppt == 6) AT_WV(LI, F, 6, true, 1);                                     \
        else if (ppt == 16) AT_WR(LI, F, 16, 1);                                         \
        else if (ppt == 8) AT_WR(LI, F, 8, 1);                                           \
        else if (ppt == 4) AT_WR(LI, F, 4, 1);                                           \
        else return hipErrorInvalidValue;                                                \
    } while (0)
    if (linear) { if (fma) AT_WP(true, true); else AT_WP(true, false); }
    else { if (fma) AT_WP(false, true); else AT_WP(false, false); }
#undef AT_WP
#undef AT_WR
#undef AT_WV
    return hipGetLastError();
}

template <int ORDER>
hipError_t launch_wave1d_batch_order(const Step1D *descs, const int2 *tbl, int64_t nblocks,
                                     bool linear, bool fma, int ppt, int64_t n0, int flip,
                                     size_t lds, hipStream_t st)
{
    const dim3 grid((unsigned)nblocks), block(kWave);
#define AT_WB(LI, F, P) hipLaunchKernelGGL((k_wave1d_batch<ORDER, LI, F, P>), grid, block, lds, st, descs, tbl, n0, flip)
#define AT_WBP(LI, F)                                                                    \
    do {                                                                                 \
        if (ppt == 32) AT_WB(LI, F, 32);                                                 \
        else if (ppt == 16) AT_WB(LI, F, 16);                                            \
        else if (ppt == 8) AT_WB(LI, F, 8);                                              \
        else if (ppt == 4) AT_WB(LI, F, 4);                                              \
        else return hipErrorInvalidValue;                                                \
    } while (0)
    if (linear) { if (fma) AT_WBP(true, true); else AT_WBP(true, false); }
    else { if (fma) AT_WBP(false, true); else AT_WBP(false, false); }
#undef AT_WBP
#undef AT_WB
    return hipGetLastError();
}

}  // namespace

}  // namespace atk
