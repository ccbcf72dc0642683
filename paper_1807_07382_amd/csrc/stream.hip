// stream.hip -- the sweeps of Sec. 2.4 as one stream down the rows of each
// tile of systems (stream.h): f read once, x written once, nothing exchanged
// through memory and nothing to clear before the launch.
#include <algorithm>

#include "stream.h"

namespace pent {
namespace {

using namespace st;

// Tiles of cw <= 64 systems, tile t's first column at t * tsf (f) and t * tsx
// (x).  HBM-bound: a wave's 32-row block lives 23 us of which its four sweeps
// take 1.5; 10 are spent waiting for the blocks below to load and 12 issuing
// loads and stores into a memory pipeline that is full (trace by the 100 MHz
// counter, N = 4096 x 65536).  That solve takes 817 to 833 us, 5.2 TB/s,
// and a bare copy through the same persistent blocks 770 to 830 for any block
// shape on this layout; the look-back single pass takes 950.
// GATED: after k_gate, which may leave the call to a look-back launch (10 us).
template <int K, int NW, int EU, bool NT, bool GATED, typename TI>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(EU, EU))) void k_stream(
    const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg, const double *trunc, int D, int64_t n, int nblk,
    const TI *F, int64_t ldf, int64_t tsf, double *X, int64_t ldx, int64_t tsx, int64_t batch, int cw, int ntiles,
    unsigned int *err, const unsigned int *gate)
{
    if (GATED && *gate != 0) return;  // left to the look-back launch after this one
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

// Growth from two samples to the next that shows a tail.  In a tail it
// is at least 2^18 (a correction's chain, kTruncFix) or 2^36 (a solve's) from
// one sample to the next, while of 64 systems of random values one in 2^16 has
// such a place.
constexpr double kSteep = 0x1p-14;

// Whether a call whose tails would cost streaming sweeps more than they save
// runs by look-back as a whole: where in two of eight tiles of 64 systems, at
// equal distances through the batch, one of 16 systems grows so between samples
// or is zero in all of them (a source between two); up to 66 samples of each, rows
// `stride` apart and the last one, tile t at F + t * ts.  One workgroup does, ahead of
// the streaming launch: that one may work in place, so that its own workgroups
// could not all look at the same right-hand sides.  The other workgroups clear
// the rest of the look-back launch's status words.
constexpr int kGateTiles = 8, kGateParts = 8, kGatePart = 9;
template <typename TI>
__global__ __launch_bounds__(16 * kGateParts * kGateTiles) void k_gate(const TI *F, int64_t ld, int64_t ts, int64_t n,
                                                                      int64_t batch, int stride, unsigned int *words, int64_t nwords)
{
    if (blockIdx.x > 0) {
        unsigned int *p = words + (int64_t)(blockIdx.x - 1) * blockDim.x + threadIdx.x;
        if (p < words + nwords && p != gate_word(words)) *p = 0;
        return;
    }
    __shared__ unsigned int grows, some[kGateTiles];  // tiles with growth; a tile's systems with a value
    if (threadIdx.x == 0) grows = 0;
    if (threadIdx.x < kGateTiles) some[threadIdx.x] = 0;
    __syncthreads();
    const int p = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / (16 * kGateParts)));
    const int cnt = (int)((n - 2) / stride) + 2, s0 = (int)(threadIdx.x / 16 % kGateParts) * kGatePart;
    const int64_t t = (batch + 63) / 64 * p / kGateTiles;
    int64_t col = p % 4 * 16 + (threadIdx.x & 15);
    col = t * 64 + col < batch ? col : batch - 1 - t * 64;
    const TI *c = F + t * ts + col;
    double a[kGatePart + 2];
#pragma unroll
    for (int i = 0; i < kGatePart + 2; i++)
        a[i] = fabs((double)c[(s0 + i < cnt - 1 ? (int64_t)(s0 + i) * stride : n - 1) * ld]);
    bool here = false, value = false;
#pragma unroll
    for (int i = 0; i < kGatePart + 2; i++) value = value || a[i] != 0.0;
#pragma unroll
    for (int i = 0; i < kGatePart; i++)
        here = here || (s0 + i + 2 < cnt && fmax(a[i], a[i + 1]) <= kSteep * a[i + 2] && a[i + 2] > 0.0 && a[i + 2] <= __DBL_MAX__);
    unsigned long long m = __ballot(value);
    m |= m >> 32;
    m |= m >> 16;
    const bool any = __ballot(here) != 0;
    if ((threadIdx.x & 63) == 0) {
        atomicOr(&some[p], (unsigned int)m & 0xFFFF);
        if (any) atomicOr(&grows, 1u << p);
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    int votes = 0;
    for (int i = 0; i < kGateTiles; i++) votes += (grows >> i & 1) != 0 || some[i] != 0xFFFF;
    *gate_word(words) = votes >= 2;
}

constexpr int kSampleParts = 4, kSamplePart = 17;

// Finds and marks the tiles that streaming sweeps had better leave to the
// look-back form: those where some system's values grow by more than 1 / kSteep
// from two samples to the next one below.  A system like that has long tails
// above its sources, in which the truncated chain leaves out what counts, and
// making up for that costs as much again as the sweeps, or more.  Up to 66
// samples of every system: rows left.stride apart and the last one.  This
// decides about time only.  Also clears the look-back form's words.
// A workgroup takes every gridDim.x-th tile, its waves a quarter of the samples
// each.  A launch of its own, 7 us of latency: inside the streaming kernels it
// takes scalar registers that their sweeps then lack (a correction of 8192 x
// 16384 took 40 us more).
template <typename TI>
__global__ __launch_bounds__(64 * kSampleParts) void k_find_left(const TI *F, int64_t ldf, int64_t tsf, int64_t n, int64_t batch,
                                                                int cw, int ntiles, Left left)
{
    __shared__ int sus[2][kSampleParts];
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64)), lane = threadIdx.x & 63;
    const int cnt = (int)((n - 2) / left.stride) + 2, per = (cnt + kSampleParts - 1) / kSampleParts, s0 = w * per;
    unsigned int any = 0;
    for (int t = blockIdx.x, turn = 0; t < ntiles; t += gridDim.x, turn ^= 1) {
        const int64_t j = (int64_t)t * cw + lane;
        const bool act = lane < cw && j < batch;
        const TI *c = F + (int64_t)t * tsf + (act ? lane : 0);
        double a[kSamplePart + 2];
#pragma unroll
        for (int i = 0; i < kSamplePart + 2; i++)
            a[i] = fabs((double)c[(s0 + i < cnt - 1 ? (int64_t)(s0 + i) * left.stride : n - 1) * ldf]);
        bool here = false;
#pragma unroll
        for (int i = 0; i < kSamplePart; i++)
            here = here || (i < per && s0 + i + 2 < cnt && fmax(a[i], a[i + 1]) <= kSteep * a[i + 2] && a[i + 2] > 0.0 && a[i + 2] <= __DBL_MAX__);
        const bool one = __ballot(here) != 0;
        if (lane == 0) sus[turn][w] = one;
        __syncthreads();
        unsigned int mark = 0;
        for (int i = 0; i < kSampleParts; i++) mark |= (unsigned int)sus[turn][i];
        if (w == 0 && act) *left_mark(left.ex, left.groups, j) = mark;
        any |= mark;
    }
    if (threadIdx.x == 0) *left_word(left.words, blockIdx.x) = any;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < left.nwords; i += (int64_t)gridDim.x * blockDim.x)
        if (i >= kTicketWords || i % kTicketStride == 0) left.words[i] = 0u;
}

// What a correction's block leaves out, P z, is held against x in the two rows
// that it would be added to first, as block b - D left them in LDS before its
// forward state went on.  A slot is filled again three rounds later, by when
// its readers, fewer than NW blocks below, are done.  Where even twice the
// largest entry that P may have makes no difference, P is not looked at.
template <int NW>
struct FixLds {
    double x[3][NW][2][64];              // in the two rows below a wave's block, by its round
    LeaveBits leave;
    unsigned long long marks[kLeftTiles];  // a tile's systems in which something counts
    Left left;  // (its values would take scalar registers all through the walk)
};

template <int NW>
struct FixExtra : Plain {
    FixLds<NW> &f;
    CTrunc trunc;
    int b, D, w, par, k;
    __device__ __forceinline__ void took(double z0, double z1)
    {
        if (b < D) return;
        const int lane = threadIdx.x & 63, ww = w >= D ? w - D : w - D + NW, pp = w >= D ? par : par == 0 ? 2 : par - 1;
        const double most = kNegligible * fmax(fabs(f.x[pp][ww][0][lane]), fabs(f.x[pp][ww][1][lane]));
        if (__ballot(!(2 * kTruncFix * fmax(fabs(z0), fabs(z1)) <= most) || z0 != z0 || z1 != z1) == 0) return;
        const CTrunc P = trunc + 4 * (int64_t)(b - D);
        const double c0 = fma(P[2], z1, P[0] * z0), c1 = fma(P[3], z1, P[1] * z0);
        const unsigned long long m = __ballot(!(fmax(fabs(c0), fabs(c1)) <= most) || c0 != c0 || c1 != c1);
        if (m != 0 && lane == 0) atomicOr(&f.marks[k], m);
    }
};

// One refinement correction, x += A^{-1}(f - A x) in place, as a stream: each
// block keeps its x beside the residual it turns into the correction, so x is
// read once and written once (20 bytes per unknown with FP32 f; the look-back
// form, k_onepass_fix, holds one array and reads x again: 28).  A block's halo
// rows are read before its neighbours can have stored theirs: block b + 1
// links its forward state after block b has swept its own rows, and block b -
// 1 waits for block b's backward state.  The correction is itself of the size
// of the error it takes away, so its backward chain stops where it would
// change that by kTruncFix: what is left out is not seen in x, as long as x
// does not fall by as much from one block to the one D above.  In the tails
// above a source it does, and there a correction comes from the blocks far
// below; so each tile with a system whose x falls is left to the look-back form
// (k_find_left), and what a block leaves out is looked at against x: a system in which it
// counts anywhere gets one more correction by that form.
// The chain's depth sets the time: of 12 waves D wait (N = 8192 x 16384 FP32,
// sigma = 100: D = 7, for kTruncTarget, 910 us; D = 4, for kTruncFix, 673; the
// look-back form 1099).
template <int K, int NW, int EU, bool NT, typename TI>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(EU, EU))) void k_stream_fix(
    const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg, const double *trunc, const double *diag, int D, int64_t n, int nblk,
    const TI *F, int64_t ldf, double *X, int64_t ldx, int64_t batch, int cw, int ntiles, Left left, unsigned int *err)
{
    __shared__ StreamLds<NW, false> sh;
    __shared__ FixLds<NW> fl;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
    const int lane = threadIdx.x & 63;
    stream_init(sh);
    Walk walk{my_tiles(ntiles), fl.leave};
    if (threadIdx.x == 0) fl.left = left;
    for (int i = threadIdx.x; i < kLeftTiles; i += 64 * NW) fl.marks[i] = 0;
    read_left<NW>(left, walk.mine, cw, fl.leave);
    walk.start();
    int b = w, par = 0;
    auto skip = [&]() {
        while (b >= nblk) {
            b -= nblk;
            walk.next();
        }
    };
    skip();
    for (unsigned int q = w; walk.t < walk.mine.end; q += NW, par = par == 2 ? 0 : par + 1) {
        const int64_t c0 = (int64_t)walk.t * cw;
        const bool act = lane < cw && c0 + lane < batch;
        const unsigned int lo = act ? lane : 0;  // idle lanes repeat the tile's first column
        const int64_t r0 = (int64_t)b * K;
        const int L = (int)(n - r0 < K ? n - r0 : K);
        double *xt = X + c0;
        double v[K], x[K], h[4];
        // halo rows outside the matrix meet a zero diagonal entry
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int64_t r = i < 2 ? r0 - 2 + i : r0 + K + i - 2;
            h[i] = xt[(r < 0 ? 0 : r >= n ? n - 1 : r) * ldx + lo];
        }
        load_block<K, false, double>(x, xt + r0 * ldx, lo, ldx, L);
        load_block<K, NT, TI>(v, F + c0 + r0 * ldf, lo, ldf, L);
        stream_residual<K>(v, x, h, diag, n, r0, L);
        fl.x[par][w][0][lane] = h[2];
        fl.x[par][w][1][lane] = h[3];
        __builtin_amdgcn_sched_barrier(0);
        Rec<K> rc;
        load_forward<K>(rc, fwd, r0);
        load_backward<K>(rc, bwd, r0);
        const FixExtra<NW> ex{{}, fl, (CTrunc)trunc, b, D, w, par, walk.k};
        stream_phases<K, NW, false, FixExtra<NW>>(v, rc, bwd, (CSeg)seg, nullptr, b, nblk, D, q, w, 0, 0, sh, err, ex);
#pragma unroll
        for (int k = 0; k < K; k++) v[k] = x[k] + v[k];
        if (act) store_block<K, NT>(v, xt + r0 * ldx, lane, ldx, L);
        b += NW;
        skip();
    }
    __syncthreads();
    for (int k = w; walk.mine.t0 + k * walk.mine.step < walk.mine.end; k += NW) {
        const int64_t j = (int64_t)(walk.mine.t0 + k * walk.mine.step) * cw + lane;
        if ((fl.marks[k] >> lane & 1) && lane < cw && j < batch) {
            *left_mark(fl.left.ex, fl.left.groups, j) = 1;
            *left_word(fl.left.words, 0) = 1;
        }
    }
}

template <typename TI>
hipError_t find_left(const TI *F, int64_t ldf, int64_t tsf, int64_t n, int64_t batch, int cw, const Left &left, hipStream_t s)
{
    const int64_t ntiles = (batch + cw - 1) / cw;
    hipLaunchKernelGGL(k_find_left<TI>, dim3((unsigned)std::min<int64_t>(ntiles, kLeftWgs)), dim3(64 * kSampleParts), 0, s, F, ldf,
                       tsf, n, batch, cw, (int)ntiles, left);
    return hipGetLastError();
}

// Whole rows on 128-byte lines.
inline bool on_lines(const void *p, int64_t pitch) { return (uintptr_t)p % 128 == 0 && pitch % 128 == 0; }

template <int K, int NW, int EU, bool NT, typename TI>
hipError_t launch_k(const StreamPlan &p, int64_t n, const void *F, int64_t ldf, int64_t tsf, double *X, int64_t ldx,
                    int64_t tsx, int64_t batch, int cw, unsigned int *words, int64_t nwords, unsigned int *err, hipStream_t s)
{
    const int64_t ntiles = (batch + cw - 1) / cw, nblk = (n + K - 1) / K;
    const int64_t grid = stream_workgroups(batch, cw, p.cus);
    if (words) {
        const hipError_t e = launch_gate(F, sizeof(TI) == sizeof(float), ldf, tsf == cw ? 64 : tsf, n, batch, K / 32 * p.depth,
                                         words, nwords, s);
        if (e != hipSuccess) return e;
    }
    const auto fn = words ? k_stream<K, NW, EU, NT, true, TI> : k_stream<K, NW, EU, NT, false, TI>;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(64 * NW), 0, s, p.fwd, p.bwd, p.seg,
                       p.trunc, p.depth, n, (int)nblk, (const TI *)F, ldf, tsf, X, ldx, tsx, batch, cw, (int)ntiles, err,
                       words ? gate_word(words) : nullptr);
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

hipError_t launch_gate(const void *F, bool f32, int64_t ld, int64_t ts, int64_t n, int64_t batch, int depth, unsigned int *words,
                       int64_t nwords, hipStream_t s)
{
    const int64_t wgs = 1 + (nwords + 16 * kGateParts * kGateTiles - 1) / (16 * kGateParts * kGateTiles);
    const dim3 block(16 * kGateParts * kGateTiles);
    const int stride = (int)sample_stride(n, depth);
    if (f32)
        hipLaunchKernelGGL(k_gate<float>, dim3((unsigned)wgs), block, 0, s, (const float *)F, ld, ts, n, batch, stride, words, nwords);
    else
        hipLaunchKernelGGL(k_gate<double>, dim3((unsigned)wgs), block, 0, s, (const double *)F, ld, ts, n, batch, stride, words, nwords);
    return hipGetLastError();
}

hipError_t launch_stream_fix(const StreamPlan &p, int64_t n, const double *diag, const void *F, bool f32,
                             int64_t ldf, double *X, int64_t ldx, int64_t batch, int cw, const Left &left_,
                             unsigned int *err, hipStream_t s)
{
    constexpr int K = 32, NW = 12, EU = 3;
    const int64_t ntiles = (batch + cw - 1) / cw, nblk = (n + K - 1) / K;
    const dim3 grid((unsigned)stream_workgroups(batch, cw, p.cus)), block(64 * NW);
    Left left = left_;
    left.stride = (int)sample_stride(n, p.depth);
    if (!left.words || ntiles > (int64_t)kLeftTiles * grid.x) return hipErrorInvalidValue;
    const hipError_t e = find_left<double>(X, ldx, cw, n, batch, cw, left, s);
    if (e != hipSuccess) return e;
    const size_t ef = f32 ? sizeof(float) : sizeof(double);
    const bool nt = on_lines(F, ldf * ef) && on_lines(X, ldx * 8);
#define PENT_FIX_GO(NT, T)                                                                                              \
    hipLaunchKernelGGL((k_stream_fix<K, NW, EU, NT, T>), grid, block, 0, s, p.fwd, p.bwd, p.seg, p.trunc, diag, p.depth, n, \
                       (int)nblk, (const T *)F, ldf, X, ldx, batch, cw, (int)ntiles, left, err)
    if (f32 && nt) PENT_FIX_GO(true, float);
    else if (f32) PENT_FIX_GO(false, float);
    else if (nt) PENT_FIX_GO(true, double);
    else PENT_FIX_GO(false, double);
#undef PENT_FIX_GO
    return hipGetLastError();
}

hipError_t launch_stream(const StreamPlan &p, int64_t n, const void *F, bool f32, int64_t ldf, int64_t tsf, double *X,
                         int64_t ldx, int64_t tsx, int64_t batch, int cw, unsigned int *err, hipStream_t s,
                         unsigned int *words, int64_t nwords)
{
    const size_t ef = f32 ? sizeof(float) : sizeof(double);
    const bool nt = on_lines(F, ldf * ef) && on_lines(X, ldx * 8) && tsf * ef % 64 == 0 && tsx * 8 % 128 == 0;
#define PENT_STREAM_GO(K, NW, EU)                                                                                       \
    return f32 ? (nt ? launch_k<K, NW, EU, true, float>(p, n, F, ldf, tsf, X, ldx, tsx, batch, cw, words, nwords, err, s)                \
                     : launch_k<K, NW, EU, false, float>(p, n, F, ldf, tsf, X, ldx, tsx, batch, cw, words, nwords, err, s))              \
               : (nt ? launch_k<K, NW, EU, true, double>(p, n, F, ldf, tsf, X, ldx, tsx, batch, cw, words, nwords, err, s)               \
                     : launch_k<K, NW, EU, false, double>(p, n, F, ldf, tsf, X, ldx, tsx, batch, cw, words, nwords, err, s))
    if (p.rows == 32) PENT_STREAM_GO(32, 16, 4);
    PENT_STREAM_GO(64, 12, 3);
#undef PENT_STREAM_GO
}

}  // namespace pent
