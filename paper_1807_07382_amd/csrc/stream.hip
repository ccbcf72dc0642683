// stream.hip -- the sweeps of Sec. 2.4 as one stream down the rows of each
// tile of systems (stream.h): f read once, x written once, nothing exchanged
// through memory and nothing to clear before the launch.
#include "stream.h"

namespace pent {
namespace {

using namespace st;

// Tiles of cw <= 64 systems, tile t's first column at t * tsf (f) and t * tsx
// (x).  HBM-bound: a wave's 32-row block lives 23 us of which its four sweeps
// take 1.5; 10 are spent waiting for the blocks below to load and 12 issuing
// loads and stores into a memory pipeline that is full (trace by the 100 MHz
// counter, N = 4096 x 65536).  That solve takes 800 us, 5.4 TB/s, as does a
// bare copy through the same persistent blocks (770 to 830 us for any block
// shape on this layout); the look-back single pass took 950.
template <int K, int NW, int EU, bool NT, typename TI>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(EU, EU))) void k_stream(
    const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg, const double *trunc, int D, int64_t n, int nblk,
    const TI *F, int64_t ldf, int64_t tsf, double *X, int64_t ldx, int64_t tsx, int64_t batch, int cw, int ntiles,
    unsigned int *err)
{
    __shared__ StreamLds<NW> sh;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
    const int lane = threadIdx.x & 63;
    stream_init(sh);
    const Tiles mine = my_tiles(ntiles);
    int t = mine.t0, b = w, par = 0;
    unsigned int turn = 0;
    auto skip = [&]() {  // block index into tile and block
        while (b >= nblk) {
            b -= nblk;
            t += mine.step;
            turn++;
        }
    };
    skip();
    for (unsigned int q = w; t < mine.end; q += NW, par ^= 1) {
        const bool act = lane < cw && (int64_t)t * cw + lane < batch;
        const int64_t r0 = (int64_t)b * K;
        const int L = (int)(n - r0 < K ? n - r0 : K);
        double v[K];
        Rec<K> rc;
        load_forward<K>(rc, fwd, r0);
        load_backward<K>(rc, bwd, r0);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_sched_barrier(0);  // the records first: the first sweep needs them with its first row
        // idle lanes repeat the tile's first column
        load_block<K, NT, TI>(v, F + (int64_t)t * tsf + r0 * ldf, act ? lane : 0, ldf, L);
        stream_phases<K, NW, true, Plain>(v, rc, bwd, (CSeg)seg, (CTrunc)trunc, b, nblk, D, q, w, par, turn, sh, err, Plain());
        if (act) store_block<K, NT>(v, X + (int64_t)t * tsx + r0 * ldx, lane, ldx, L);
        b += NW;
        skip();
    }
    store_fence();  // every wave's x is in memory before the repair reads it
    __syncthreads();
    turn = 0;
    for (t = mine.t0; t < mine.end; t += mine.step, turn++)
        if (sh.last[turn % 32] >= 0) {
            const bool act = lane < cw && (int64_t)t * cw + lane < batch;
            stream_repair<K, NW>(X + (int64_t)t * tsx + (act ? lane : 0), ldx, act, n, nblk, D, (CSeg)seg, (CBwd)bwd,
                                 (CTrunc)trunc, sh, w, turn % 32, [](int64_t) { return 0.0; });
        }
}

// r = f - A x over a block (v: f on entry, r on exit; x the block's rows, h
// the two rows above it and the two below), compensated (dot2_row); rows k >=
// L zero.  The five diagonals come as the records do, one row per lane.
template <int K>
__device__ __forceinline__ void stream_residual(double (&v)[K], const double (&x)[K], const double (&h)[4],
                                                const double *__restrict__ diag, int64_t n, int64_t r0, int L)
{
    double cl[5];
    const int64_t row = r0 + (threadIdx.x & (K - 1));
#pragma unroll
    for (int d = 0; d < 5; d++) cl[d] = diag[d * n + (row < n ? row : n - 1)];  // rows past the matrix: dropped
    unroll<K>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        if constexpr (k % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        const double cf[5] = {lane_double(cl[0], k), lane_double(cl[1], k), lane_double(cl[2], k), lane_double(cl[3], k),
                              lane_double(cl[4], k)};
        const double xv[5] = {k >= 2 ? x[k >= 2 ? k - 2 : 0] : h[k < 2 ? k : 0],
                              k >= 1 ? x[k >= 1 ? k - 1 : 0] : h[1], x[k],
                              k + 1 < K ? x[k + 1 < K ? k + 1 : 0] : h[2],
                              k + 2 < K ? x[k + 2 < K ? k + 2 : 0] : h[k + 2 - K >= 0 ? 2 + k + 2 - K : 2]};
        const double r = dot2_row(v[k], cf, xv);
        v[k] = k < L ? r : 0.0;
    });
}

// One refinement correction, x += A^{-1}(f - A x) in place, as a stream: each
// block keeps its x beside the residual it turns into the correction, so x is
// read once and written once (20 bytes per unknown with FP32 f; the look-back
// form, k_onepass_fix, holds one array and reads x again: 28).  A block's halo
// rows are read before its neighbours can have stored theirs: block b + 1
// links its forward state after block b has swept its own rows, and block b -
// 1 waits for block b's backward state.  The correction is itself of the size
// of the error it takes away, so its backward chain stops where it would
// change that by kTruncFix, and nothing is checked (a system with a value that
// is not finite has none left after its first solve).  The chain's depth sets
// the time: of 12 waves D wait (N = 8192 x 16384 FP32, sigma = 100: D = 7,
// for kTruncTarget, 910 us; D = 4, for kTruncFix, 673; the look-back form 1099).
template <int K, int NW, int EU, bool NT, typename TI>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(EU, EU))) void k_stream_fix(
    const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg, const double *diag, int D, int64_t n, int nblk,
    const TI *F, int64_t ldf, double *X, int64_t ldx, int64_t batch, int cw, int ntiles, unsigned int *err)
{
    __shared__ StreamLds<NW, false> sh;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
    const int lane = threadIdx.x & 63;
    stream_init(sh);
    const Tiles mine = my_tiles(ntiles);
    int t = mine.t0, b = w;
    auto skip = [&]() {
        while (b >= nblk) {
            b -= nblk;
            t += mine.step;
        }
    };
    skip();
    for (unsigned int q = w; t < mine.end; q += NW) {
        const bool act = lane < cw && (int64_t)t * cw + lane < batch;
        const unsigned int lo = act ? lane : 0;  // idle lanes repeat the tile's first column
        const int64_t r0 = (int64_t)b * K;
        const int L = (int)(n - r0 < K ? n - r0 : K);
        double *xt = X + (int64_t)t * cw;
        double v[K], x[K], h[4];
        // halo rows outside the matrix meet a zero diagonal entry
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int64_t r = i < 2 ? r0 - 2 + i : r0 + K + i - 2;
            h[i] = xt[(r < 0 ? 0 : r >= n ? n - 1 : r) * ldx + lo];
        }
        load_block<K, false, double>(x, xt + r0 * ldx, lo, ldx, L);
        load_block<K, NT, TI>(v, F + (int64_t)t * cw + r0 * ldf, lo, ldf, L);
        stream_residual<K>(v, x, h, diag, n, r0, L);
        __builtin_amdgcn_sched_barrier(0);
        Rec<K> rc;
        load_forward<K>(rc, fwd, r0);
        load_backward<K>(rc, bwd, r0);
        stream_phases<K, NW, false, Plain>(v, rc, bwd, (CSeg)seg, nullptr, b, nblk, D, q, w, 0, 0, sh, err, Plain());
#pragma unroll
        for (int k = 0; k < K; k++) v[k] = x[k] + v[k];
        if (act) store_block<K, NT>(v, xt + r0 * ldx, lane, ldx, L);
        b += NW;
        skip();
    }
}

// Whole rows on 128-byte lines.
inline bool on_lines(const void *p, int64_t pitch) { return (uintptr_t)p % 128 == 0 && pitch % 128 == 0; }

template <int K, int NW, int EU, bool NT, typename TI>
hipError_t launch_k(const StreamPlan &p, int64_t n, const void *F, int64_t ldf, int64_t tsf, double *X, int64_t ldx,
                    int64_t tsx, int64_t batch, int cw, unsigned int *err, hipStream_t s)
{
    const int64_t ntiles = (batch + cw - 1) / cw, nblk = (n + K - 1) / K;
    const int64_t grid = (ntiles < p.cus ? ntiles + 7 : p.cus) / 8 * 8;
    hipLaunchKernelGGL((k_stream<K, NW, EU, NT, TI>), dim3((unsigned)grid), dim3(64 * NW), 0, s, p.fwd, p.bwd, p.seg,
                       p.trunc, p.depth, n, (int)nblk, (const TI *)F, ldf, tsf, X, ldx, tsx, batch, cw, (int)ntiles, err);
    return hipGetLastError();
}

}  // namespace

// Systems per tile: the width with the least work in a compute unit's turns
// (tiles are dealt whole; the rate of a compute unit, not of the memory,
// bounds one that has a tile more than the others).  Narrow tiles use lanes
// and lines less well, a tenth for every 16 systems given up (n = 4096 x
// 20000: 266 us at 48, 302 at 64, 316 at 32; x 8192 110 at 32, 133 at 64;
// system-major 300 x 40000 43 at 64, 50 at 32).  Multiples of 16 keep tiles on
// 128-byte lines of an aligned row.
int stream_tile_width(int64_t batch, int cus)
{
    int best = 64;
    int64_t cost = 0;
    for (int cw = 64; cw >= 32; cw -= 16) {
        const int64_t tiles = (batch + cw - 1) / cw, turns = (tiles + cus - 1) / cus;
        const int64_t c = turns * cw * (160 + 64 - cw);
        if (cw == 64 || c < cost) {
            best = cw;
            cost = c;
        }
    }
    return best;
}

hipError_t launch_stream_fix(const StreamPlan &p, int depth, int64_t n, const double *diag, const void *F, bool f32,
                             int64_t ldf, double *X, int64_t ldx, int64_t batch, int cw, unsigned int *err, hipStream_t s)
{
    constexpr int K = 32, NW = 12, EU = 3;
    const int64_t ntiles = (batch + cw - 1) / cw, nblk = (n + K - 1) / K;
    const dim3 grid((unsigned)((ntiles < p.cus ? ntiles + 7 : p.cus) / 8 * 8)), block(64 * NW);
    const size_t ef = f32 ? sizeof(float) : sizeof(double);
    const bool nt = on_lines(F, ldf * ef) && on_lines(X, ldx * 8);
#define PENT_FIX_GO(NT, T)                                                                                              \
    hipLaunchKernelGGL((k_stream_fix<K, NW, EU, NT, T>), grid, block, 0, s, p.fwd, p.bwd, p.seg, diag, depth, n,          \
                       (int)nblk, (const T *)F, ldf, X, ldx, batch, cw, (int)ntiles, err)
    if (f32 && nt) PENT_FIX_GO(true, float);
    else if (f32) PENT_FIX_GO(false, float);
    else if (nt) PENT_FIX_GO(true, double);
    else PENT_FIX_GO(false, double);
#undef PENT_FIX_GO
    return hipGetLastError();
}

hipError_t launch_stream(const StreamPlan &p, int64_t n, const void *F, bool f32, int64_t ldf, int64_t tsf, double *X,
                         int64_t ldx, int64_t tsx, int64_t batch, int cw, unsigned int *err, hipStream_t s)
{
    const size_t ef = f32 ? sizeof(float) : sizeof(double);
    const bool nt = on_lines(F, ldf * ef) && on_lines(X, ldx * 8) && tsf * ef % 64 == 0 && tsx * 8 % 128 == 0;
#define PENT_STREAM_GO(K, NW, EU)                                                                                       \
    return f32 ? (nt ? launch_k<K, NW, EU, true, float>(p, n, F, ldf, tsf, X, ldx, tsx, batch, cw, err, s)                \
                     : launch_k<K, NW, EU, false, float>(p, n, F, ldf, tsf, X, ldx, tsx, batch, cw, err, s))              \
               : (nt ? launch_k<K, NW, EU, true, double>(p, n, F, ldf, tsf, X, ldx, tsx, batch, cw, err, s)               \
                     : launch_k<K, NW, EU, false, double>(p, n, F, ldf, tsf, X, ldx, tsx, batch, cw, err, s))
    if (p.rows == 32) PENT_STREAM_GO(32, 16, 4);
    PENT_STREAM_GO(64, 12, 3);
#undef PENT_STREAM_GO
}

}  // namespace pent
