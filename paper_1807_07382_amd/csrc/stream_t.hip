// stream_t.hip -- streaming sweeps (stream.h) over system-major storage of a few
// blocks of rows: the second direction of an alternating-direction step, also
// with the 2-D Cahn-Hilliard explicit term formed on the way in.
#include "stream.h"

namespace pent {
namespace {

using namespace st;

constexpr int kTK = 32, kTNW = 16, kTEU = 4;
typedef double Dbl2u __attribute__((ext_vector_type(2), aligned(8)));  // 16 bytes at any double

// Systems i = 0 .. per - 1 of group k at F + k * kst + i * sst, n values each; a
// tile is up to cw <= 64 consecutive systems of one group.  A wave moves its
// cw systems x 32 rows as whole 128-byte runs (8 lanes per system, two rows a
// lane, at any alignment of the runs) and turns them in place through LDS, 8
// rows of one parity at a time (row stride 66 doubles: no bank conflict), so
// that each lane holds one system's rows as in k_stream.
//
// ST (cw = 64): C comes in at src and R = C + dt_k Lap_h(C^3 - C) is formed
// over it (a group is an instance k, its systems the grid rows y).  The y
// neighbours' terms are wave shifts of the row's own, with the tile's two
// neighbour systems held one row per lane (of the system above in lanes 0..31,
// of the one below in 32..63); along x the block above leaves its last row in
// LDS, and the row below the block is read from memory.  Whatever stands
// outside the grid is zero before the terms are formed, so the stencil has no
// selects (with them it kept 32 row masks and spilled 71 registers, and the
// sweep took 230 us).
//
// D = nblk - 1: a block takes the states of all blocks below it, and nothing is
// left out.  Where the chain is cut short, what it leaves out has to be added to
// finished tiles, in runs of 16 rows of 64 systems, and that costs more than
// the form saves (n = 2048 x 32768 225 us, but 700 with sources in the bottom
// rows only; 260 by look-back).
template <bool ST, bool NT>
__global__ __launch_bounds__(64 * kTNW) __attribute__((amdgpu_waves_per_eu(kTEU, kTEU))) void k_stream_t(
    const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg, int64_t n, int nblk,
    const double *src, double *F, int64_t per, int64_t sst, int64_t kst, int tpk, int cw, int ntiles, unsigned int *err,
    const double *dt, double inv_h2)
{
    constexpr int K = kTK, NW = kTNW;
    __shared__ StreamLds<NW, false> sh;
    __shared__ double tb[NW][8][66];
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
    const int lane = threadIdx.x & 63;
    const int sub = lane & 7, grp = lane >> 3;  // row pair in a 16-row chunk, system in a slice of 8
    __shared__ double hx[ST ? 2 : 1][ST ? NW : 1][64];  // ST: last row of C of a block, slots as those of z
    __shared__ unsigned int hflag[NW];
    double(*tw)[66] = tb[w];
    if (threadIdx.x < NW) hflag[threadIdx.x] = 0;
    stream_init(sh);
    const Tiles mine = my_tiles(ntiles);
    int t = mine.t0, b = w, par = 0;
    auto skip = [&]() {
        while (b >= nblk) {
            b -= nblk;
            t += mine.step;
        }
    };
    skip();
    for (unsigned int q = w; t < mine.end; q += NW, par ^= 1) {
        const int g = ST ? t / tpk : 0;
        const int64_t s0 = (int64_t)(t - g * tpk) * cw, base = g * kst + s0 * sst;
        const int cnt = (int)(per - s0 < cw ? per - s0 : cw);
        const int64_t r0 = (int64_t)b * K;
        const int L = (int)(n - r0 < K ? n - r0 : K);
        double v[K], hv = 0.0, xr = 0.0;
        Rec<K> rc;
        if constexpr (ST) {
            // the values around the block, ahead of it (from clamped addresses)
            const bool below = lane >= 32, in = below ? s0 + cnt < per : s0 > 0;
            const int64_t i = below ? (in ? cnt : cnt - 1) : in ? -1 : 0, row = r0 + (lane & 31);
            hv = src[base + i * sst + (row < n ? row : n - 1)];
            xr = src[base + (int64_t)(lane < cnt ? lane : cnt - 1) * sst + (r0 + K < n ? r0 + K : n - 1)];
            hv = in ? hv : 0.0;
            xr = r0 + K < n ? xr : 0.0;
        } else {
            load_forward<K>(rc, fwd, r0);
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_sched_barrier(0);
        // raw runs: rows 16 c + 2 sub + e of system 8 q + grp into v[16 c + 2 q + e];
        // systems past the tile repeat its last one
        typedef __attribute__((address_space(1))) const Dbl2u *G2;
        typedef __attribute__((address_space(1))) Dbl2u *W2;
        const int64_t s8 = 8 * sst;
        auto next = [&](auto &p, int i) {  // to this lane's system of slice i + 1, if the tile has it
            p += 8 * (i + 1) + grp < cnt ? s8 : 0;
            asm volatile("" : "+v"(p));
        };
        {
            const double *p = src + base + (grp < cnt ? grp : cnt - 1) * sst;
            if (L == K) {
                p += r0 + 2 * sub;
#pragma unroll
                for (int i = 0; i < 8; i++) {
#pragma unroll
                    for (int c = 0; c < K / 16; c++) {
                        const Dbl2u u = NT ? __builtin_nontemporal_load((G2)(p + 16 * c)) : *(G2)(p + 16 * c);
                        v[16 * c + 2 * i] = u.x;
                        v[16 * c + 2 * i + 1] = u.y;
                    }
                    next(p, i);
                }
            } else {
                typedef __attribute__((address_space(1))) const double *G1;
#pragma unroll
                for (int i = 0; i < 8; i++) {
#pragma unroll
                    for (int c = 0; c < K / 16; c++)
#pragma unroll
                        for (int e = 0; e < 2; e++) {
                            const int64_t row = r0 + 16 * c + 2 * sub + e;
                            v[16 * c + 2 * i + e] = ((G1)p)[row < n ? row : n - 1];
                        }
                    next(p, i);
                }
            }
        }
        // turned: v[k] = (row r0 + k, system lane)
#pragma unroll
        for (int c = 0; c < K / 16; c++)
#pragma unroll
            for (int e = 0; e < 2; e++) {
#pragma unroll
                for (int i = 0; i < 8; i++) tw[sub][8 * i + grp] = v[16 * c + 2 * i + e];
#pragma unroll
                for (int i = 0; i < 8; i++) v[16 * c + 2 * i + e] = tw[i][lane];
            }
        auto clear = [&]() {  // rows past the matrix
            if (L < K)
#pragma unroll
                for (int k = 0; k < K; k++) v[k] = k < L ? v[k] : 0.0;
        };
        clear();
        if constexpr (ST) {
            if (cnt < 64)
#pragma unroll
                for (int k = 0; k < K; k++) v[k] = lane < cnt ? v[k] : 0.0;
            hx[par][w][lane] = v[K - 1];
            lds_post(&hflag[w], q + 1);
            load_forward<K>(rc, fwd, r0);  // (with the block's loads it would not fit the registers)
            const double dtk = dt[g];
            double hw = ch_wterm(hv), wprev = 0.0;
            if (b > 0) {
                const int pw = w == 0 ? NW - 1 : w - 1, pp = w == 0 ? par ^ 1 : par;
                if (!lds_wait(&hflag[pw], q) && lane == 0) atomicOr(err, 1u);
                wprev = ch_wterm(hx[pp][pw][lane]);
            }
            double wcur = ch_wterm(v[0]);
            unroll<K>([&](auto kk) {
                constexpr int row = decltype(kk)::value;
                if constexpr (row % 4 == 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    pin(hw);
                }
                const double ws = lane_shift<true>(wcur, lane_double(hw, row));
                const double wn = lane_shift<false>(wcur, lane_double(hw, 32 + row));
                const double wnext = ch_wterm(row + 1 < K ? v[row + 1 < K ? row + 1 : 0] : xr);
                v[row] = ch_point(v[row], wcur, wnext, wprev, wn, ws, dtk, inv_h2);
                wprev = wcur;
                wcur = wnext;
            });
            clear();
        }
        stream_phases<K, NW, false, PlainLate>(v, rc, bwd, (CSeg)seg, nullptr, b, nblk, nblk - 1, q, w, 0, 0, sh, err, PlainLate());
        // turned back and stored as runs
#pragma unroll
        for (int c = 0; c < K / 16; c++)
#pragma unroll
            for (int e = 0; e < 2; e++) {
#pragma unroll
                for (int i = 0; i < 8; i++) tw[i][lane] = v[16 * c + 2 * i + e];
#pragma unroll
                for (int i = 0; i < 8; i++) v[16 * c + 2 * i + e] = tw[sub][8 * i + grp];
            }
        double *p = F + base + grp * sst + r0 + 2 * sub;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            if (8 * i + grp < cnt) {
#pragma unroll
                for (int c = 0; c < K / 16; c++) {
                    const Dbl2u u = {v[16 * c + 2 * i], v[16 * c + 2 * i + 1]};
                    if (L == K) {
                        if (NT) __builtin_nontemporal_store(u, (W2)(p + 16 * c));
                        else *(W2)(p + 16 * c) = u;
                    } else {
                        if (16 * c + 2 * sub < L) p[16 * c] = u.x;
                        if (16 * c + 2 * sub + 1 < L) p[16 * c + 1] = u.y;
                    }
                }
            }
            next(p, i);
        }
        b += NW;
        skip();
    }
}

template <bool ST>
hipError_t launch_t(const StreamPlan &p, int64_t n, const double *src, double *F, int64_t per, int64_t sst, int64_t kst,
                    int64_t groups, int cw, unsigned int *err, const double *dt, double inv_h2, hipStream_t s)
{
    const int64_t tpk = (per + cw - 1) / cw, ntiles = tpk * groups, nblk = (n + kTK - 1) / kTK;
    if (n > kStreamTRows) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((ntiles < p.cus ? ntiles + 7 : p.cus) / 8 * 8)), block(64 * kTNW);
    if ((uintptr_t)src % 128 == 0 && (uintptr_t)F % 128 == 0 && sst % 16 == 0 && kst % 16 == 0)
        hipLaunchKernelGGL((k_stream_t<ST, true>), grid, block, 0, s, p.fwd, p.bwd, p.seg, n, (int)nblk,
                           src, F, per, sst, kst, (int)tpk, cw, (int)ntiles, err, dt, inv_h2);
    else
        hipLaunchKernelGGL((k_stream_t<ST, false>), grid, block, 0, s, p.fwd, p.bwd, p.seg, n, (int)nblk,
                           src, F, per, sst, kst, (int)tpk, cw, (int)ntiles, err, dt, inv_h2);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_stream_t(const StreamPlan &p, int64_t n, double *F, int64_t ld, int64_t batch, unsigned int *err,
                           hipStream_t s)
{
    return launch_t<false>(p, n, F, F, batch, ld, 0, 1, stream_tile_width(batch, p.cus), err, nullptr, 0.0, s);
}

hipError_t launch_stream_ch2d(const StreamPlan &p, int64_t n, const double *C, double *R, int64_t ny, int64_t ninst,
                              const double *dt, double h, unsigned int *err, hipStream_t s)
{
    return launch_t<true>(p, n, C, R, ny, ninst * n, n, ninst, 64, err, dt, 1.0 / (h * h), s);
}

}  // namespace pent
