// 1D stepper kernels of libat.so for gfx950: one step per launch
// (k_step1d_plain), and the general form for the tile widths that the fused
// kernels of at_wave1d.h do not take (k_step1d).
//
// Method: viscous Burgers u_t + u u_x = nu u_xx (or linear advection c u_x),
// central differences and forward Euler (paper section 3.2) on P tiles of a
// periodic grid.  A point whose stencil crosses its tile's edge reads a halo
// value extrapolated in time from the neighbour edge's levels n-k, n-k-1, ...
// (section 2, Eqs. (1)-(2); three levels for the 4th-order scheme), with the
// delay k prescribed per directed face and step.  As in section 5.2, the halo
// approximation is separate from the stencil, which is the same everywhere.
//
// Arithmetic is binary64 with contraction disabled (-ffp-contract=off); the
// evaluation order of every formula is fixed:
//   order 2: D1 = (r1 - l1)*c1,                 D2 = ((r1 - 2u) + l1)*c2
//   order 4: D1 = (8(r1 - l1) - (r2 - l2))*c1,  D2 = ((16(r1 + l1) - 30u) - (r2 + l2))*c2
//   F = nu*D2 - a*D1 (a = u, or c for linear advection),  u' = u + dt*F
//   halo, two levels:   H = v0 + k*(v0 - v1)
//   halo, three levels: H = (v0 + k*d1) + w2*(d1 - (v1 - v2)), d1 = v0 - v1, w2 = 0.5*k*(k+1)
//
// Work decomposition of k_step1d (s steps per launch):
//   * a workgroup of 256 threads owns CH consecutive points and loads the
//     region [c0 - s*h, c0 + CH + s*h) of level n0 (coalesced, through LDS);
//   * each thread keeps PPT consecutive region points in registers and trades
//     h values per side with its neighbours through LDS once per step;
//   * the valid part of the region shrinks by h per step (overlapped
//     trapezoids); neighbouring tiles' edges inside the region are recomputed
//     redundantly with the same operations, so the result is bit-identical to
//     one launch per step;
//   * edge values of in-launch levels are kept in an LDS edge history for
//     delayed halo reads; levels before n0 come from the ring in HBM;
//   * owned tile-edge points are published to ring slot n mod R: those of every
//     level when the run keeps the edge tape for the adjoint, else those of the
//     last L + m - 1 levels of a launch, the only ones a later launch reads.
#include <algorithm>

#include "at_internal.h"
#include "at_stencil1d.h"

namespace atk {

namespace {

constexpr int kPPT = 16;      // region points per thread (general kernel)

__device__ __forceinline__ int64_t floordiv(int64_t a, int64_t b)
{
    int64_t q = a / b;
    return (a % b != 0 && ((a < 0) != (b < 0))) ? q - 1 : q;
}

// ring slot of level n0 + d for d in [-(R-1), R-1] (the levels a launch
// touches lie within one ring length of n0)
__device__ __forceinline__ int64_t ring_slot(const Step1D &a, int64_t d)
{
    int64_t x = a.slot0 + d;
    if (x < 0) x += a.R;
    if (x >= a.R) x -= a.R;
    return x;
}

// whether step t of a launch of S steps writes its level's tile edges to the
// ring: every level (publish 1), or only the last D levels of the launch
// (publish 2), the only ones a later launch reads when no edge tape is kept
__device__ __forceinline__ bool publish_level(const Step1D &a, int t, int S)
{
    return a.publish == 1 || (a.publish == 2 && t + a.D >= S);
}

// The region's field passes through a padded LDS stage (point r of a part at
// r + r/PPT, so that neither the coalesced accesses nor the per-thread ones
// conflict on banks) in stage_parts(PPT) parts: at 16 points per thread in two
// halves of 2048 points, which keeps the stage at 17 KB instead of 34 KB so
// that LDS does not cap the workgroups per CU below what registers allow.
__host__ __device__ constexpr int stage_parts(int ppt) { return ppt >= 16 ? 2 : 1; }

// doubles of one stage part at ppt points per thread
__host__ __device__ constexpr int stage_doubles(int ppt)
{
    return (kThreads * ppt + kThreads) / stage_parts(ppt);
}

// Level n0 of a region of E points that starts at periodic index G0w (in
// [0, N)) into wp[0 .. PPT) of every thread (thread tid holds region points
// tid*PPT ..), 0 past E.  Every thread issues all of its PPT loads before its
// first LDS write, so their latencies overlap.  Indices are wrapped into
// [0, N) (one subtraction when the grid is at least one region wide), so
// every load is in bounds; the values past E are loaded and dropped.
// Ends with a barrier: the stage may be reused at once.
template <int PPT>
__device__ __forceinline__ void load_window(const double *__restrict__ uin, int64_t N,
                                            int64_t G0w, int E, int tid, double *stage,
                                            double *wp)
{
    constexpr int PARTS = stage_parts(PPT);
    constexpr int IT = PPT / PARTS;                 // loads per thread in one part
    constexpr int TP = kThreads / PARTS;            // threads whose points a part holds
    double v[PPT];
    if (N >= (int64_t)kThreads * PPT) {
#pragma unroll
        for (int it = 0; it < PPT; ++it) {
            int64_t g = G0w + it * kThreads + tid;
            if (g >= N) g -= N;
            v[it] = uin[g];
        }
    } else {
#pragma unroll
        for (int it = 0; it < PPT; ++it) v[it] = uin[(G0w + it * kThreads + tid) % N];
    }
#pragma unroll
    for (int h = 0; h < PARTS; ++h) {
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int rr = i * kThreads + tid;      // point h*IT*kThreads + rr of the region
            stage[rr + rr / PPT] = h * IT * kThreads + rr < E ? v[h * IT + i] : 0.0;
        }
        __syncthreads();
        if (tid / TP == h) {
#pragma unroll
            for (int j = 0; j < PPT; ++j) wp[j] = stage[(tid - h * TP) * (PPT + 1) + j];
        }
        __syncthreads();
    }
}

// The inverse: the points wp[0 .. PPT) of every thread through the stage to
// out[r - lo] for the region points r in [lo, hi), coalesced
template <int PPT>
__device__ __forceinline__ void store_window(const double *wp, int tid, double *stage, int lo,
                                             int hi, double *__restrict__ out)
{
    constexpr int PARTS = stage_parts(PPT);
    constexpr int IT = PPT / PARTS;
    constexpr int TP = kThreads / PARTS;
#pragma unroll
    for (int h = 0; h < PARTS; ++h) {
        __syncthreads();
        if (tid / TP == h) {
#pragma unroll
            for (int j = 0; j < PPT; ++j) stage[(tid - h * TP) * (PPT + 1) + j] = wp[j];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int rr = i * kThreads + tid;
            const int r = h * IT * kThreads + rr;
            if (r >= lo && r < hi) out[r - lo] = stage[rr + rr / PPT];
        }
    }
}

template <int ORDER, bool LINEAR, bool FMA>
__global__ __launch_bounds__(kThreads) void k_step1d(Step1D a)
{
    constexpr int H = ORDER / 2;
    constexpr int M = (ORDER == 2) ? 2 : 3;
    constexpr int PPT = kPPT;
    extern __shared__ double lds[];
    double *stage = lds;                                  // one part of the stage (load_window)
    double *xch = lds;                                    // [2][kThreads][2H]  (aliases stage)
    double *eh = lds + 2 * kThreads * 2 * H;              // [s-1][NT][2][H]  (aliases stage)

    const int tid = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x * a.CH;
    const int64_t owned = (a.N - c0 < a.CH) ? (a.N - c0) : a.CH;
    const int sh = a.s * H;
    const int E = (int)owned + 2 * sh;                    // region length (<= kThreads*PPT)
    const int64_t G0 = c0 - sh;                           // unwrapped start (may be < 0)
    int64_t G0w = G0 % a.N;
    if (G0w < 0) G0w += a.N;

    // ---- level n0 of the region: coalesced loads -> LDS -> registers
    double w[PPT + 2 * H];
    load_window<PPT>(a.uin, a.N, G0w, E, tid, stage, w + H);
#pragma unroll
    for (int q = 0; q < H; ++q) { w[q] = 0.0; w[PPT + H + q] = 0.0; }

    // ---- tile bookkeeping of this thread's first point
    const int rp0 = tid * PPT;                            // region position of point 0
    const int64_t Gt = G0 + rp0;
    const int64_t tdiv = floordiv(Gt, a.W);
    const int64_t o0 = Gt - tdiv * a.W;                   // offset in its tile, [0, W)
    const int tl0 = (int)(tdiv - floordiv(G0, a.W));      // region-local tile index
    int64_t tp0 = tdiv % a.P;
    if (tp0 < 0) tp0 += a.P;                              // physical tile index
    const bool has_edge = (rp0 < E) && ((o0 < H) || (o0 + PPT - 1 + H >= a.W));
    const int64_t F = 2 * a.P;

    for (int t = 0; t < a.s; ++t) {
        const int64_t n = a.n0 + t;
        // ---- edge points of level n: LDS history for later steps, ring for later launches
        if (has_edge) {
            const int64_t slot = ring_slot(a, t);
            const bool pub = publish_level(a, t, a.s);
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                const int rp = rp0 + j;
                int64_t oj = o0 + j;
                int e = 0;
                while (oj >= a.W) { oj -= a.W; ++e; }
                const bool lo = oj < H, hi = oj >= a.W - H;
                if (rp < E && (lo || hi)) {
                    const int side = lo ? 0 : 1;
                    const int q = lo ? (int)oj : (int)(oj - (a.W - H));
                    if (t < a.s - 1)
                        eh[((t * a.NT + (tl0 + e)) * 2 + side) * H + q] = w[H + j];
                    if (pub && rp >= sh && rp < sh + owned) {
                        int64_t tp = tp0 + e;
                        while (tp >= a.P) tp -= a.P;
                        a.ring[((slot * a.P + tp) * 2 + side) * H + q] = w[H + j];
                    }
                }
            }
        }
        // ---- neighbour exchange: first and last H values of every thread
        double *buf = xch + (t & 1) * kThreads * 2 * H;
#pragma unroll
        for (int q = 0; q < H; ++q) {
            buf[tid * 2 * H + q] = w[H + q];
            buf[tid * 2 * H + H + q] = w[PPT + q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < H; ++q) {
            w[q] = (tid > 0) ? buf[(tid - 1) * 2 * H + H + q] : 0.0;
            w[PPT + H + q] = (tid < kThreads - 1) ? buf[(tid + 1) * 2 * H + q] : 0.0;
        }
        // ---- standard stencil on every point
        double res[PPT];
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            double nb[2 * H];
#pragma unroll
            for (int q = 0; q < H; ++q) { nb[q] = w[j + q]; nb[H + q] = w[j + H + 1 + q]; }
            res[j] = update<ORDER, LINEAR, FMA>(nb, w[H + j], a);
        }
        // ---- points next to a tile edge: stencil again with AT halo values
        if (has_edge) {
            const int8_t *krow = a.delays + n * F;
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                const int rp = rp0 + j;
                int64_t oj = o0 + j;
                int e = 0;
                while (oj >= a.W) { oj -= a.W; ++e; }
                const bool valid = rp >= (t + 1) * H && rp < E - (t + 1) * H;   // inside the cone
                if (valid && (oj < H || oj >= a.W - H)) {
                    int64_t tp = tp0 + e;
                    while (tp >= a.P) tp -= a.P;
                    const int tl = tl0 + e;
                    double nb[2 * H];
#pragma unroll
                    for (int sl = 0; sl < 2 * H; ++sl) {
                        const int d = (sl < H) ? -(H - sl) : (sl - H + 1);
                        double v = w[H + j + d];
                        const int64_t od = oj + d;
                        if (od < 0 || od >= a.W) {
                            const int side = (od < 0) ? 0 : 1;
                            const int kk = krow[2 * tp + side];
                            if (kk > 0) {
                                const int q = (side == 0) ? (int)(od + H) : (int)(od - a.W);
                                const int stl = tl + (side ? 1 : -1);
                                int64_t stp = tp + (side ? 1 : -1);
                                if (stp < 0) stp += a.P;
                                if (stp >= a.P) stp -= a.P;
                                const int sside = 1 - side;
                                double vv[3] = {0.0, 0.0, 0.0};
#pragma unroll
                                for (int jj = 0; jj < M; ++jj) {
                                    if (jj == 0 || !a.stale) {
                                        const int64_t lev = n - kk - jj;
                                        if (lev >= a.n0)
                                            vv[jj] = eh[(((int)(lev - a.n0) * a.NT + stl) * 2 + sside) * H + q];
                                        else
                                            vv[jj] = a.ring[((ring_slot(a, lev - a.n0) * a.P + stp) * 2 + sside) * H + q];
                                    }
                                }
                                v = extrap<FMA>(kk, a.stale != 0, vv[0], vv[1], vv[2], M);
                            }
                        }
                        nb[sl] = v;
                    }
                    res[j] = update<ORDER, LINEAR, FMA>(nb, w[H + j], a);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < PPT; ++j) w[H + j] = res[j];
    }

    // ---- level n0+s of the owned points: registers -> LDS -> coalesced stores
    store_window<PPT>(w + H, tid, stage, sh, sh + (int)owned, a.uout + c0);
}


// One step per launch (the plain form), for tile widths that are multiples of
// PPT (8, else 4): every thread's points lie in one tile.  A thread that starts
// a tile writes its left AT halo values into the left part of its register
// window, a thread that ends a tile its right ones, and then every point runs
// the same stencil (the split of section 5.2).  HBM-bound: 6.2 TB/s of 16 bytes
// per point at 2^24 points; 8 points per thread keep the workgroup small and
// more of them in flight than 16.  Grids that the caches hold are bound by the
// trips to memory of a wave with a face: field, delay, ring, the ring once for
// both sides (order 4, 2^22 points, us per step, one side after the other and
// together: tiles of 4096 14.2 and 12.8, of 64 18.5 and 16.3).  100000 tiles of 12
// points: 14.2 as a launch of the fused kernels with all their history, 7.7 here.
template <int ORDER, bool LINEAR, bool FMA, int PPT>
__global__ __launch_bounds__(kThreads) void k_step1d_plain(Step1D a)
{
    constexpr int H = ORDER / 2;
    constexpr int M = (ORDER == 2) ? 2 : 3;
    extern __shared__ double lds[];
    double *stage = lds;                                  // one part of the stage (load_window)
    double *xch = lds;                                    // [kThreads][2H]  (aliases stage)

    const int tid = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x * a.CH;
    const int owned = (int)((a.N - c0 < a.CH) ? (a.N - c0) : a.CH);
    const int E = a.RL + owned + H;                       // region length (<= kThreads*PPT)
    const int64_t G0 = c0 - a.RL;                         // unwrapped start, multiple of PPT
    int64_t G0w = G0 % a.N;
    if (G0w < 0) G0w += a.N;

    double w[PPT + 2 * H];
    load_window<PPT>(a.uin, a.N, G0w, E, tid, stage, w + H);

    const int rp0 = tid * PPT;
    const int64_t Gt = G0 + rp0;
    const int64_t tdiv = floordiv(Gt, a.W);
    const int64_t o0 = Gt - tdiv * a.W;                   // multiple of PPT
    int64_t tp0 = tdiv % a.P;
    if (tp0 < 0) tp0 += a.P;
    const bool lo_edge = o0 == 0 && rp0 < E;
    const bool hi_edge = o0 + PPT == a.W && rp0 < E;
    const bool owns = rp0 >= a.RL && rp0 < a.RL + owned;

    // ---- this level's tile edges to the ring
    if ((lo_edge || hi_edge) && owns && a.publish) {
        double *dst = a.ring + (a.slot0 * a.P + tp0) * 2 * H;
#pragma unroll
        for (int q = 0; q < H; ++q) {
            if (lo_edge) dst[q] = w[H + q];
            if (hi_edge) dst[H + q] = w[PPT + q];
        }
    }
    // ---- neighbour exchange
#pragma unroll
    for (int q = 0; q < H; ++q) {
        xch[tid * 2 * H + q] = w[H + q];
        xch[tid * 2 * H + H + q] = w[PPT + q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < H; ++q) {
        w[q] = (tid > 0) ? xch[(tid - 1) * 2 * H + H + q] : 0.0;
        w[PPT + H + q] = (tid < kThreads - 1) ? xch[(tid + 1) * 2 * H + q] : 0.0;
    }
    // ---- AT halo approximation at tile edges (k = 0: the raw neighbour stays)
    if (lo_edge || hi_edge) {
        const int8_t *krow = a.delays + a.n0 * (2 * a.P) + 2 * tp0;
        const int kl = lo_edge && tid > 0 ? krow[0] : 0, kr = hi_edge ? krow[1] : 0;
        // the lanes that start a tile and those that end one in the same pass, one
        // trip to the ring for both; a lane that does both (a tile of PPT points)
        // takes its right halo in a second one
        const bool both = lo_edge && hi_edge;
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            const bool left = pass == 0 && lo_edge;
            const int kk = pass == 0 ? (lo_edge ? kl : kr) : (both ? kr : 0);
            if (kk == 0) continue;
            const int64_t src = left ? 2 * (tp0 == 0 ? a.P - 1 : tp0 - 1) + 1
                                     : 2 * (tp0 == a.P - 1 ? 0 : tp0 + 1);
#pragma unroll
            for (int q = 0; q < H; ++q) {
                double vv[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int jj = 0; jj < M; ++jj)
                    if (jj == 0 || !a.stale)
                        vv[jj] = a.ring[(ring_slot(a, -kk - jj) * a.P * 2 + src) * H + q];
                const double hv = extrap<FMA>(kk, a.stale != 0, vv[0], vv[1], vv[2], M);
                w[q] = left ? hv : w[q];
                w[PPT + H + q] = left ? w[PPT + H + q] : hv;
            }
        }
    }
    step_window<ORDER, LINEAR, FMA, PPT>(w, a);
    store_window<PPT>(w + H, tid, stage, a.RL, a.RL + owned, a.uout + c0);
}

}  // namespace

int step1d_points_per_thread() { return kPPT; }

// points per thread of k_step1d_plain at tile width W, 0: it does not take it
int step1d_plain_ppt(int64_t W) { return W % 8 == 0 ? 8 : (W % 4 == 0 ? 4 : 0); }

// LDS of k_step1d: the stage part, or the exchange buffers and behind them the
// edges of the levels that later steps of the launch read (none in a launch of
// one step: the levels below n0 and the delays are read from memory)
static size_t step1d_lds_bytes(int order, int s, int NT)
{
    const size_t stage = (size_t)stage_doubles(kPPT);
    const size_t xch = (size_t)2 * kThreads * order, hist = (size_t)(s - 1) * NT * order;
    return 8 * std::max(stage, xch + hist);
}

// k_step1d_plain of plain_ppt points per thread (one step), or (0) the general k_step1d
hipError_t launch_step1d(const Step1D &a, int order, bool linear, int plain_ppt, bool fma,
                         int64_t nblocks, hipStream_t st)
{
    size_t lds = step1d_lds_bytes(order, a.s, a.NT);
    if (plain_ppt) {
        const size_t stage = (size_t)stage_doubles(plain_ppt), xch = (size_t)kThreads * order;
        lds = 8 * std::max(stage, xch);
    }
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    dim3 grid((unsigned)nblocks), block(kThreads);
#define AT_L(O, LI, F)                                                                    \
    do {                                                                                  \
        if (plain_ppt == 8) hipLaunchKernelGGL((k_step1d_plain<O, LI, F, 8>), grid, block, lds, st, a); \
        else if (plain_ppt == 4) hipLaunchKernelGGL((k_step1d_plain<O, LI, F, 4>), grid, block, lds, st, a); \
        else hipLaunchKernelGGL((k_step1d<O, LI, F>), grid, block, lds, st, a);           \
    } while (0)
    if (order == 2) {
        if (linear) { if (fma) AT_L(2, true, true); else AT_L(2, true, false); }
        else { if (fma) AT_L(2, false, true); else AT_L(2, false, false); }
    } else {
        if (linear) { if (fma) AT_L(4, true, true); else AT_L(4, true, false); }
        else { if (fma) AT_L(4, false, true); else AT_L(4, false, false); }
    }
#undef AT_L
    return hipGetLastError();
}

}  // namespace atk
