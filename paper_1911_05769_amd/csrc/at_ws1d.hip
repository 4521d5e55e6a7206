// Weakly-synchronous 1D stepper of libat.so for gfx950: the delays EMERGE from
// the progress of the tiles instead of being prescribed.
//
// Method (paper section 5.2, Algorithm 2): every tile advances on its own.
// After computing level n+1 it writes its two edges into the circular buffer
// ("ring") slot (n+1) mod R.  Before step n a tile looks for the newest level t
// of each neighbour edge that has arrived; the delay is k = n - min(t, n).  A
// tile waits only while k would exceed the bound the method allows,
// min(L, max(0, n - m + 1)) (the blocking receive of Algorithm 2, including its
// start-up synchrony); otherwise it proceeds at once with the AT halo of
// section 2, Eqs. (1)-(2), built from levels n-k, n-k-1(, n-k-2) of the
// neighbour's edge.  The delay actually used is stored as k[n][f], so a run can
// be replayed exactly with prescribed delays.
//
// Arrival is told by the value itself: a slot whose level has not been written
// holds kUnset, one bit pattern of a signalling NaN that no arithmetic produces
// (a value with exactly these bits is sent as a quiet NaN).  What bounds a step
// is the trip of an edge value from one XCD to another, so it is made once: the
// writer stores, the reader's poll returns the value.  With a counter per edge
// the writer waited for its stores before it announced them and the reader
// loaded the values after it had seen the counter: 2.6 us per step (2^20 points,
// 1024 tiles, L = 3) against 1.5.  A poll looks at all the levels a step can
// use at once, one lane per level.
//   * Order: a tile waits for its stores of the step before (long done) before
//     it stores the next level, so levels become visible in order.
//   * Reuse: with level n goes the reset of the slot of level n + L + 2 to
//     kUnset.  A reader looks for level x from its step x on, when it has seen
//     level x - 1 - L, stored after that reset was complete; and the level the
//     slot held, n + L + 2 - R, is below n - 1 - 2L - (m - 1), the oldest one a
//     neighbour up to L steps behind can still read (R >= L + m + 63, L <= 15).
//
// Work decomposition: one workgroup of NT threads (256, or one wave of 64
// for narrow tiles) per tile of width W = NT * PPT, PPT consecutive points
// per thread held in registers for the whole run; h values per side are
// traded with the neighbouring threads through LDS each step.  The first wave
// receives the left halo, the last wave the right one (a single wave: its
// halves); thread 0 sends the tile's left edge, thread NT-1 its right one, as
// soon as those points are updated.  All tiles must be resident at once
// (cooperative launch), and every wait is bounded: past the spin limit a
// workgroup sets the error flag and leaves, and a waiting workgroup that sees
// the flag leaves too, so every wave reaches the end of the kernel.
#include "at_internal.h"
#include "at_stencil1d.h"
#include "at_ws.h"

namespace atk {

namespace {

// a ring slot whose level has not arrived (signalling NaN)
constexpr unsigned long long kUnset = 0x7FF4A55E7ED0DEADull;

__device__ __forceinline__ bool is_set(double v)
{
    return (unsigned long long)__double_as_longlong(v) != kUnset;
}

__device__ __forceinline__ double sendable(double v)
{
    return is_set(v) ? v : __longlong_as_double(0x7FF8000000000000ll);
}

template <int ORDER, bool LINEAR, int PPT, int NT>
__global__ __launch_bounds__(NT) void k_ws1d(Ws1D A)
{
    constexpr int H = ORDER / 2;
    constexpr int M = ORDER == 2 ? 2 : 3;
    constexpr int NWV = NT / 64;
    static_assert(PPT >= H, "a thread holds at least h points");
    __shared__ double lo[2][NT][H], hi[2][NT][H];
    __shared__ int s_stop;
    const int t = threadIdx.x, lane = t % 64;
    const int wave = NWV > 1 ? __builtin_amdgcn_readfirstlane(t / 64) : 0;
    const int64_t P = A.P, b = blockIdx.x;
    const int64_t bl = b == 0 ? P - 1 : b - 1, br = b + 1 == P ? 0 : b + 1;
    const int64_t base = b * A.W + (int64_t)t * PPT;
    const bool stale = A.stale != 0;
    const int64_t lev = P * 2 * H;                    // doubles of a ring level
    double v[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) v[j] = A.u[base + j];
    if (t == 0) s_stop = 0;

    // ---- receiving lanes: lane j of a side looks at level n - j of the
    // neighbour's facing edge (one wave: the left side in lanes 0 .. 31, the
    // right one in lanes 32 .. 63)
    const bool receives = wave == 0 || wave == NWV - 1;
    const int side = NWV > 1 ? (wave == 0 ? 0 : 1) : lane / 32;
    const int j = lane % 32, first_lane = NWV > 1 ? 0 : side * 32;
    const bool looks = receives && (NWV == 1 || lane < 32) && j < A.L + M;
    const double *src = A.ring + (side == 0 ? bl * 2 + 1 : br * 2) * H;
    const bool sends = t == 0 || t == NT - 1;
    double *own = A.ring + (b * 2 + (t == 0 ? 0 : 1)) * H;

    // send level n (ring slot sl) of the tile's edge e[0 .. h)
    auto send = [&](int sl, const double *e) {
        int sr = sl + A.L + 2;                        // the slot to come: unset (L + 2 < R)
        if (sr >= A.R) sr -= A.R;
        __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < H; ++i) {
            st_coherent(own + sl * lev + i, sendable(e[i]));
            st_coherent(own + sr * lev + i, __longlong_as_double((long long)kUnset));
        }
    };

    __syncthreads();                                  // s_stop initialised before any wait
    int slot = (int)(A.n0 % A.R);                     // of level n
    if (sends) send(slot, t == 0 ? v : v + PPT - H);
    for (int64_t n = A.n0; n < A.n0 + A.nsteps; ++n) {
        const int buf = (int)(n & 1);
        ws_idle(A.jitter, A.seed, b, n);
        // thread edges for the neighbouring threads
#pragma unroll
        for (int i = 0; i < H; ++i) {
            lo[buf][t][i] = v[i];
            hi[buf][t][i] = v[PPT - H + i];
        }
        // receive: the newest arrived level of the neighbour edge, waiting only
        // while the delay would pass its bound
        double halo[H];
#pragma unroll
        for (int i = 0; i < H; ++i) halo[i] = 0.0;
        int k = 0;
        if (receives) {
            const int kmax = (int)min((int64_t)A.L, max((int64_t)0, n - M + 1));
            int sl = slot - j;
            if (sl < 0) sl += A.R;
            const double *p = src + sl * lev;
            const bool look = looks && n - j >= 0;
            double x[H];
            bool stop = false;
            for (int64_t spins = 0;; ++spins) {
                bool there = look;
#pragma unroll
                for (int i = 0; i < H; ++i) {
                    x[i] = look ? ld_coherent(p + i) : 0.0;
                    there = there && is_set(x[i]);
                }
                // the newest level with the ones its halo needs behind it
                const unsigned long long all = __ballot(there);
                const unsigned mine = (unsigned)(all >> first_lane);
                k = -1;
                if (mine & 1u) k = 0;
                else {
                    unsigned ok = mine;
                    if (!stale) ok &= M == 3 ? (mine >> 1) & (mine >> 2) : mine >> 1;
                    ok &= (2u << kmax) - 2u;          // delays 1 .. kmax
                    if (ok) k = __ffs((int)ok) - 1;
                }
                if (!__any(k < 0)) break;
                if (spins >= A.spin_limit ||
                    ((spins & 63) == 63 && load_relaxed(A.err) != 0)) {
                    stop = true;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            if (stop) {
                if (lane == 0) {
                    __hip_atomic_store(A.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    s_stop = 1;
                }
            } else {
                // halo value i (left to right along x) from lanes k, k+1(, k+2)
#pragma unroll
                for (int i = 0; i < H; ++i) {
                    const double v0 = __shfl(x[i], first_lane + k, 64);
                    const double v1 = __shfl(x[i], first_lane + k + 1, 64);
                    const double v2 = M == 3 ? __shfl(x[i], first_lane + k + 2, 64) : v1;
                    halo[i] = k == 0 ? v0 : extrap<false>(k, stale, v0, v1, v2, M);
                }
            }
        }
        __syncthreads();
        if (s_stop) break;
        // stencil: ext = [left h][own PPT][right h]
        double ext[PPT + 2 * H];
#pragma unroll
        for (int i = 0; i < H; ++i) {
            ext[i] = t == 0 ? halo[i] : hi[buf][t - 1][i];
            ext[H + PPT + i] = t == NT - 1 ? halo[i] : lo[buf][t + 1][i];
        }
#pragma unroll
        for (int q = 0; q < PPT; ++q) ext[H + q] = v[q];
        auto point = [&](int q) {
            double nb[4];
            if constexpr (ORDER == 2) {
                nb[0] = ext[q];
                nb[1] = ext[q + 2];
            } else {
                nb[0] = ext[q];
                nb[1] = ext[q + 1];
                nb[2] = ext[q + 3];
                nb[3] = ext[q + 4];
            }
            return update<ORDER, LINEAR, false>(nb, ext[H + q], A.coef);
        };
        // the edge points first, so that they are on their way during the others
#pragma unroll
        for (int q = 0; q < H; ++q) v[q] = point(q);
#pragma unroll
        for (int q = PPT - H; q < PPT; ++q)
            if (q >= H) v[q] = point(q);
        slot = slot + 1 == A.R ? 0 : slot + 1;
        if (sends) {
            send(slot, t == 0 ? v : v + PPT - H);
            A.delays[n * 2 * P + 2 * b + (t == 0 ? 0 : 1)] = (int8_t)k;
        }
#pragma unroll
        for (int q = H; q < PPT - H; ++q) v[q] = point(q);
    }
#pragma unroll
    for (int q = 0; q < PPT; ++q) A.u[base + q] = v[q];
}

__global__ __launch_bounds__(256) void k_ws_init(int32_t *cnt, int64_t n, int32_t v, int32_t *err)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) cnt[i] = v;
    if (i == 0) *err = 0;
}

// every ring slot unset
__global__ __launch_bounds__(256) void k_ws_unset(unsigned long long *ring, int64_t n, int32_t *err)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        ring[i] = kUnset;
    if (blockIdx.x == 0 && threadIdx.x == 0) *err = 0;
}

}  // namespace

// Threads per workgroup and points per thread for tile width W: 256 threads
// when W = 256 q, else one wave when W = 64 q, with q in {1, 2, 4, 8, 16} and
// q >= h; false when W fits neither.
bool ws1d_shape(int64_t W, int h, int *nt, int *ppt)
{
    for (const int t : {256, 64}) {
        if (W % t != 0) continue;
        const int64_t q = W / t;
        if ((q == 1 || q == 2 || q == 4 || q == 8 || q == 16) && q >= h) {
            *nt = t;
            *ppt = (int)q;
            return true;
        }
    }
    return false;
}

// the kernel for (order, advection mode, points per thread, threads), or null
static const void *ws1d_kernel(int order, bool linear, int ppt, int nt)
{
#define WS_PICK(O, PP, T)                                                                      \
    if (order == O && ppt == PP && nt == T)                                                    \
        return linear ? (const void *)k_ws1d<O, true, PP, T> : (const void *)k_ws1d<O, false, PP, T>;
#define WS_PICK_T(T) WS_PICK(2, 1, T) WS_PICK(2, 2, T) WS_PICK(2, 4, T) WS_PICK(2, 8, T)          \
    WS_PICK(2, 16, T) WS_PICK(4, 2, T) WS_PICK(4, 4, T) WS_PICK(4, 8, T) WS_PICK(4, 16, T)
    WS_PICK_T(256)
    WS_PICK_T(64)
#undef WS_PICK_T
#undef WS_PICK
    return nullptr;
}

// Largest number of k_ws1d workgroups that can be resident at once for this
// order, advection mode and tile width (0 if the shape is not supported)
int64_t ws1d_max_tiles(int order, bool linear, int64_t W)
{
    int nt = 0, ppt = 0;
    if (!ws1d_shape(W, order / 2, &nt, &ppt)) return 0;
    const void *f = ws1d_kernel(order, linear, ppt, nt);
    if (!f) return 0;
    int per_cu = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, nt, 0) != hipSuccess) return 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    return (int64_t)per_cu * cus;
}

hipError_t launch_ws_init(int32_t *cnt, int64_t n, int32_t v, int32_t *err, hipStream_t st)
{
    const int64_t g = (n + 255) / 256;
    hipLaunchKernelGGL(k_ws_init, dim3((unsigned)(g > 0 ? g : 1)), dim3(256), 0, st, cnt, n, v,
                       err);
    return hipGetLastError();
}

hipError_t launch_ws1d(const Ws1D &a, int order, bool linear, hipStream_t st)
{
    const int64_t words = (int64_t)a.R * a.P * order;
    const int64_t g = (words + 255) / 256 < 2048 ? (words + 255) / 256 : 2048;
    hipLaunchKernelGGL(k_ws_unset, dim3((unsigned)g), dim3(256), 0, st,
                       reinterpret_cast<unsigned long long *>(a.ring), words, a.err);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int nt = 0, ppt = 0;
    if (!ws1d_shape(a.W, order / 2, &nt, &ppt)) return hipErrorInvalidValue;
    const void *f = ws1d_kernel(order, linear, ppt, nt);
    if (!f) return hipErrorInvalidValue;
    void *args[] = {(void *)&a};
    return hipLaunchCooperativeKernel(f, dim3((unsigned)a.P), dim3(nt), args, 0, st);
}

}  // namespace atk
