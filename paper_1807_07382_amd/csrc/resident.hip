// resident.hip -- whole systems resident in one workgroup, for batches too small
// to fill the device with walking tiles and up to 2048 rows (32 or 16 systems to
// the workgroup), 4096 (four systems, as the resident-tile schedule at any batch)
// or, for a few hundred systems, 6656.
//
// A workgroup holds all rows of a tile of S systems (S = 4, 16 or 32): lane
// l of wave w has rows [32 b, 32 b + 32) of system l % S in registers, b = w *
// 64/S + l / S.  Each row is read once and written once in pieces of S
// consecutive systems.  The sweeps are those of the streaming form (stream.h:
// zero-start sweep of every block at once, then the true one), but the
// states between the blocks come from a scan over all of them: within a wave
// lane to lane, between waves through LDS after one barrier per direction.
// Nothing is truncated, nothing goes through memory, and no wave waits for
// another workgroup: the latency of a solve is that of one load, four sweeps
// of 32 rows, two barriers and one store (us, before / now: N = 256 x 256, tiles
// of eight systems with their records in LDS, 8.5 / 7.4, of which a launch is 7;
// N = 3384 x 154, the same, 37 / 16; N = 1000 x 5003 as walking tiles 26.7 / 20.5,
// 3.9 TB/s; N = 1537 x 2500 by partitions 47 / 25; N = 4313 x 67 by look-back 33 / 24).
// Full tiles of 16 waves are bound by the four sweeps, 32 rows x 4 waves x 9
// operations of a SIMD each.
//
// The periodic solve and Crank-Nicolson step (cyclic.hip) end with
// x_tail = Minv ((f_{n-2}, f_{n-1}) - h^T y) from y = E^{-1} f^, whose four
// rows next to the border pass through LDS, and y - Z x_tail in registers (N =
// 1537 x 3001: look-back 38.6 us and 5 to clear its flags, 49.5 with the gaps;
// now 24.5).
#include "stream.h"

namespace pent {
namespace {

using namespace st;

constexpr int kResK = 32;      // rows of a block
constexpr int kResWaves = 16;  // most waves of a workgroup

// What is between the waves of a tile of S systems.
template <int S, int NW>
struct ResLds {
    double e[NW][2][S];  // state leaving a wave's rows downward, from zero
    double a[NW][2][S];  // ... and upward
    double te[S < 16 ? NW : 1][4], ta[S < 16 ? NW : 1][4];  // narrow tiles: the waves' transfer matrices
    double ft[2][S], xe[4][S];  // periodic: f_{n-2}, f_{n-1}; y at rows 0, 1, m-2, m-1
};

// (x0, x1) of the lane d before (d > 0) or after (d < 0) this one.
__device__ __forceinline__ void from_lane(int d, double x0, double x1, double &r0, double &r1)
{
    const int l = (int)(threadIdx.x & 63) - d;
    r0 = __shfl(x0, l, 64);
    r1 = __shfl(x1, l, 64);
}

// The state through all rows of wave u: y = e + T y, the wave's T from the
// table of 64-row segments (one for S = 32, two for S = 16).
template <int S, bool FWD>
__device__ __forceinline__ void through_wave(CSeg seg, int u, double e0, double e1, double &y0, double &y1)
{
    if constexpr (S == 16) {
        const int first = FWD ? 2 * u : 2 * u + 1, then = FWD ? 2 * u + 1 : 2 * u;
        if constexpr (FWD) {
            link(0.0, 0.0, seg[first].tf[0], seg[first].tf[1], seg[first].tf[2], seg[first].tf[3], y0, y1);
            link(e0, e1, seg[then].tf[0], seg[then].tf[1], seg[then].tf[2], seg[then].tf[3], y0, y1);
        } else {
            link(0.0, 0.0, seg[first].tb[0], seg[first].tb[1], seg[first].tb[2], seg[first].tb[3], y0, y1);
            link(e0, e1, seg[then].tb[0], seg[then].tb[1], seg[then].tb[2], seg[then].tb[3], y0, y1);
        }
    } else {
        if constexpr (FWD) link(e0, e1, seg[u].tf[0], seg[u].tf[1], seg[u].tf[2], seg[u].tf[3], y0, y1);
        else link(e0, e1, seg[u].tb[0], seg[u].tb[1], seg[u].tb[2], seg[u].tb[3], y0, y1);
    }
}

// The forward recurrence of every block, with the state that enters it.
template <int S, typename Lds>
__device__ __forceinline__ void res_forward(double (&v)[kResK], Rec<kResK> &rc, const SegRec *seg32, CSeg segw, int w, int sub,
                                            int64_t blk, Lds &sh)
{
    constexpr int G = 64 / S;
    const int s = threadIdx.x & (S - 1);
    const double t0 = seg32[blk].tf[0], t1 = seg32[blk].tf[1], t2 = seg32[blk].tf[2], t3 = seg32[blk].tf[3];
    double e0 = 0.0, e1 = 0.0;
    sweep_forward<kResK, false>(v, rc, e0, e1);
    pin(e0);
    pin(e1);
    double c0 = e0, c1 = e1;
#pragma unroll
    for (int j = 1; j < G; j++) {
        double p0, p1;
        from_lane(S, c0, c1, p0, p1);
        double n0 = p0, n1 = p1;
        link(e0, e1, t0, t1, t2, t3, n0, n1);
        c0 = sub == j ? n0 : c0;
        c1 = sub == j ? n1 : c1;
    }
    if (sub == G - 1) {
        sh.e[w][0][s] = c0;
        sh.e[w][1][s] = c1;
    }
    __syncthreads();
    double y0 = 0.0, y1 = 0.0;
    for (int u = 0; u < w; u++) through_wave<S, true>(segw, u, sh.e[u][0][s], sh.e[u][1][s], y0, y1);
#pragma unroll
    for (int j = 1; j < G; j++) {
        double n0 = y0, n1 = y1, p0, p1;
        link(e0, e1, t0, t1, t2, t3, n0, n1);
        from_lane(S, n0, n1, p0, p1);
        y0 = sub == j ? p0 : y0;
        y1 = sub == j ? p1 : y1;
    }
    sweep_forward<kResK, true>(v, rc, y0, y1);
}

// Back substitution of every block, with the state that enters it from below.
template <int S, typename Lds, typename Extra>
__device__ __forceinline__ void res_backward(double (&v)[kResK], Rec<kResK> &rc, const SegRec *seg32, CSeg segw, int w, int waves,
                                             int sub, int64_t blk, bool rows, Lds &sh, Extra ex)
{
    constexpr int G = 64 / S;
    const int s = threadIdx.x & (S - 1);
    const double t0 = seg32[blk].tb[0], t1 = seg32[blk].tb[1], t2 = seg32[blk].tb[2], t3 = seg32[blk].tb[3];
    double a0 = 0.0, a1 = 0.0;
    sweep_backward<kResK, false>(v, rc, a0, a1, ex);
    a0 = rows ? a0 : 0.0;  // blocks past the last row
    a1 = rows ? a1 : 0.0;
    pin(a0);
    pin(a1);
    double c0 = a0, c1 = a1;
#pragma unroll
    for (int j = G - 2; j >= 0; j--) {
        double p0, p1;
        from_lane(-S, c0, c1, p0, p1);
        double n0 = p0, n1 = p1;
        link(a0, a1, t0, t1, t2, t3, n0, n1);
        c0 = sub == j ? n0 : c0;
        c1 = sub == j ? n1 : c1;
    }
    if (sub == 0) {
        sh.a[w][0][s] = c0;
        sh.a[w][1][s] = c1;
    }
    __syncthreads();
    double z0 = 0.0, z1 = 0.0;
    for (int u = waves - 1; u > w; u--) through_wave<S, false>(segw, u, sh.a[u][0][s], sh.a[u][1][s], z0, z1);
#pragma unroll
    for (int j = G - 2; j >= 0; j--) {
        double n0 = z0, n1 = z1, p0, p1;
        link(a0, a1, t0, t1, t2, t3, n0, n1);
        from_lane(-S, n0, n1, p0, p1);
        z0 = sub == j ? p0 : z0;
        z1 = sub == j ? p1 : z1;
    }
    sweep_backward<kResK, true>(v, rc, z0, z1, ex);
#pragma unroll
    for (int k = 0; k < kResK; k++) pin(v[k]);
}

// Coefficients of tiles of four systems, where a row of 16 lanes holds
// more than one block: rows 4 i + l of the block in lane l of every four,
// broadcast within them.
struct QuadCoef {
    double c[kResK / 4];
    template <int k>
    __device__ __forceinline__ double get() const
    {
        constexpr int ctrl = k % 4 * 0x55;  // quad_perm: the same lane four times
        const long long x = __double_as_longlong(c[k / 4]);
        const int lo = __builtin_amdgcn_update_dpp(0, (int)x, ctrl, 0xF, 0xF, true);
        const int hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), ctrl, 0xF, 0xF, true);
        return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
    }
    __device__ __forceinline__ void hold()
    {
#pragma unroll
        for (int i = 0; i < kResK / 4; i++) pin(c[i]);
    }
};
struct QuadRec {
    QuadCoef ra, ap, bp, gm, dl;
};

__device__ __forceinline__ void load_quads_forward(QuadRec &r, const FwdRec *f, int64_t r0)
{
#pragma unroll
    for (int i = 0; i < kResK / 4; i++) {
        const Dbl2 *p = (const Dbl2 *)(f + r0 + 4 * i + (threadIdx.x & 3));
        const Dbl2 u = p[0];
        r.ra.c[i] = u.x;
        r.ap.c[i] = u.y;
        r.bp.c[i] = p[1].x;
    }
}

__device__ __forceinline__ void load_quads_backward(QuadRec &r, const BwdRec *b, int64_t r0)
{
#pragma unroll
    for (int i = 0; i < kResK / 4; i++) {
        const Dbl2 q = *(const Dbl2 *)(b + r0 + 4 * i + (threadIdx.x & 3));
        r.gm.c[i] = q.x;
        r.dl.c[i] = q.y;
    }
}

// The affine map y -> c + m y (m column-major) of the G blocks of a wave up to
// and including each (FWD: from the first, else from the last), by doubling;
// the wave's goes to LDS, and (c, m) become those of the blocks before.
template <int S, bool FWD>
__device__ __forceinline__ void scan_maps(double (&c)[2], double (&m)[4], int sub, double (*wc)[S], double *wm)
{
    constexpr int G = 64 / S;
    const int at = FWD ? sub : G - 1 - sub;
#pragma unroll
    for (int d = 1; d < G; d *= 2) {
        double p0, p1, q0, q1, q2, q3;
        from_lane(FWD ? S * d : -S * d, c[0], c[1], p0, p1);
        from_lane(FWD ? S * d : -S * d, m[0], m[1], q0, q1);
        from_lane(FWD ? S * d : -S * d, m[2], m[3], q2, q3);
        link(c[0], c[1], m[0], m[1], m[2], m[3], p0, p1);
        const double n0 = fma(m[2], q1, m[0] * q0), n1 = fma(m[3], q1, m[1] * q0), n2 = fma(m[2], q3, m[0] * q2),
                     n3 = fma(m[3], q3, m[1] * q2);
        if (at >= d) {
            c[0] = p0;
            c[1] = p1;
            m[0] = n0;
            m[1] = n1;
            m[2] = n2;
            m[3] = n3;
        }
    }
    if (at == G - 1) {
        const int s = threadIdx.x & (S - 1);
        wc[0][s] = c[0];
        wc[1][s] = c[1];
        if (s < 4) wm[s] = s == 0 ? m[0] : s == 1 ? m[1] : s == 2 ? m[2] : m[3];
    }
    from_lane(FWD ? S : -S, c[0], c[1], c[0], c[1]);
    from_lane(FWD ? S : -S, m[0], m[1], m[0], m[1]);
    from_lane(FWD ? S : -S, m[2], m[3], m[2], m[3]);
    if (at == 0) {
        c[0] = c[1] = m[1] = m[2] = 0.0;
        m[0] = m[3] = 1.0;
    }
}

// Both sweeps of tiles of four systems: as above, with the states between the 16
// blocks of a wave by doubling.
template <int S, typename Lds>
__device__ __forceinline__ void narrow_sweeps(double (&v)[kResK], const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg32, int w,
                                              int waves, int sub, int64_t blk, bool rows, Lds &sh)
{
    const int s = threadIdx.x & (S - 1);
    Plain ex;
    QuadRec rc;
    load_quads_forward(rc, fwd, blk * kResK);
    double c[2] = {0.0, 0.0}, m[4];
#pragma unroll
    for (int k = 0; k < 4; k++) m[k] = seg32[blk].tf[k];
    sweep_forward<kResK, false>(v, rc, c[0], c[1]);
    pin(c[0]);
    pin(c[1]);
    scan_maps<S, true>(c, m, sub, sh.e[w], sh.te[w]);
    __syncthreads();
    double y0 = 0.0, y1 = 0.0;
    for (int u = 0; u < w; u++)
        link(sh.e[u][0][s], sh.e[u][1][s], sh.te[u][0], sh.te[u][1], sh.te[u][2], sh.te[u][3], y0, y1);
    link(c[0], c[1], m[0], m[1], m[2], m[3], y0, y1);
    sweep_forward<kResK, true>(v, rc, y0, y1);
    load_quads_backward(rc, bwd, blk * kResK);
#pragma unroll
    for (int k = 0; k < 4; k++) m[k] = seg32[blk].tb[k];
    c[0] = c[1] = 0.0;
    sweep_backward<kResK, false>(v, rc, c[0], c[1], ex);
    c[0] = rows ? c[0] : 0.0;  // blocks past the last row
    c[1] = rows ? c[1] : 0.0;
    pin(c[0]);
    pin(c[1]);
    scan_maps<S, false>(c, m, sub, sh.a[w], sh.ta[w]);
    __syncthreads();
    double z0 = 0.0, z1 = 0.0;
    for (int u = waves - 1; u > w; u--)
        link(sh.a[u][0][s], sh.a[u][1][s], sh.ta[u][0], sh.ta[u][1], sh.ta[u][2], sh.ta[u][3], z0, z1);
    link(c[0], c[1], m[0], m[1], m[2], m[3], z0, z1);
    sweep_backward<kResK, true>(v, rc, z0, z1, ex);
#pragma unroll
    for (int k = 0; k < kResK; k++) pin(v[k]);
}

typedef __attribute__((address_space(1))) const char *GBytes;
typedef __attribute__((address_space(1))) char *GBytesOut;
typedef __attribute__((address_space(1))) double *GDblOut;

// Where a lane's rows are: 32 from row r0 of its column, `off` bytes past the
// uniform address of the wave's first row.
struct Place {
    int64_t rw, r0;  // first row of the wave, of the lane
    int sub, s;      // the lane's block in the wave, its system in the tile
};

// Pitches up to which a lane's rows are within 32 bits of the wave's first.
template <int S>
constexpr int64_t kFullLd = ((int64_t)1 << 24) / (64 / S);

// The lane's rows from column s of the tile F; rows from n on give zero.  full:
// no lane of the wave has such rows, and the pitch is at most kFullLd.
template <typename TI>
__device__ __forceinline__ void res_load(double (&v)[kResK], const TI *F, int64_t ld, int64_t s, const Place &at, int64_t n,
                                         bool full)
{
    typedef __attribute__((address_space(1))) const TI *G;
    if (full) {
        const unsigned int off = (unsigned int)(sizeof(TI) * (at.sub * kResK * ld + s));
        GBytes q = (GBytes)(F + at.rw * ld);
#pragma unroll
        for (int k = 0; k < kResK; k++) {
            v[k] = (double)*(G)(q + off);
            q = fresh(q + sizeof(TI) * ld);
        }
    } else {
        const int L = n - at.r0 < kResK ? (int)(n - at.r0) : kResK;
        G q = (G)F + (L > 0 ? at.r0 : n - 1) * ld + s;
#pragma unroll
        for (int k = 0; k < kResK; k++) {
            v[k] = (double)*q;
            q += k + 1 < L ? ld : 0;
            asm volatile("" : "+v"(q));
        }
#pragma unroll
        for (int k = 0; k < kResK; k++) v[k] = k < L ? v[k] : 0.0;
    }
}

__device__ __forceinline__ void res_store(const double (&v)[kResK], double *X, int64_t ld, const Place &at, int64_t n, bool full)
{
    if (full) {
        const unsigned int off = (unsigned int)(8 * (at.sub * kResK * ld + at.s));
        GBytesOut q = (GBytesOut)(X + at.rw * ld);
#pragma unroll
        for (int k = 0; k < kResK; k++) {
            *(GDblOut)(q + off) = v[k];
            q = fresh(q + 8 * ld);
        }
    } else {
        const int L = n - at.r0 < kResK ? (int)(n - at.r0) : kResK;
        GDblOut q = (GDblOut)X + at.r0 * ld + at.s;
#pragma unroll
        for (int k = 0; k < kResK; k++) {
            if (k < L) *q = v[k];
            q += ld;
            asm volatile("" : "+v"(q));
        }
    }
}

// Tiles in the order that gives each XCD a contiguous eighth of them; < 0:
// this workgroup has none.
__device__ __forceinline__ int64_t res_tile(int64_t ntiles)
{
    const int x = blockIdx.x % 8;
    const int64_t t = ntiles * x / 8 + blockIdx.x / 8;
    return t < ntiles * (x + 1) / 8 ? t : -1;
}

template <int S>
__device__ __forceinline__ Place res_place(int w)
{
    const int lane = threadIdx.x & 63;
    Place at;
    at.sub = lane / S;
    at.s = lane & (S - 1);
    at.rw = (int64_t)w * (64 / S) * kResK;
    at.r0 = at.rw + at.sub * kResK;
    return at;
}

template <int S, int NW, typename TI>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4))) void k_resident(
    const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg32, const SegRec *segw, int64_t n, const TI *F, int64_t ldf,
    double *X, int64_t ldx, int64_t batch, int64_t ntiles, int64_t ts)
{
    __shared__ ResLds<S, kResWaves> sh;
    const int64_t tile = res_tile(ntiles);
    if (tile < 0) return;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64)), waves = (int)(blockDim.x / 64);
    const Place at = res_place<S>(w);
    const int64_t c0 = tile * S, blk = at.r0 / kResK;
    const bool act = c0 + at.s < batch, full = at.rw + 64 / S * kResK <= n && ldf <= kFullLd<S> && ldx <= kFullLd<S>;
    const int64_t col = c0 / 64 * ts + c0 % 64;  // tiles of 64 systems ts apart (64: one array)
    double v[kResK];
    res_load(v, F + col, ldf, act ? at.s : batch - 1 - c0, at, n, full);  // idle lanes repeat the last column
    if constexpr (S < 16) {
        narrow_sweeps<S>(v, fwd, bwd, seg32, w, waves, at.sub, blk, at.r0 < n, sh);
    } else {
        Rec<kResK> rc;
        load_forward<kResK>(rc, fwd, at.r0);
        load_backward<kResK>(rc, bwd, at.r0);
        res_forward<S>(v, rc, seg32, (CSeg)segw, w, at.sub, blk, sh);
        res_backward<S>(v, rc, seg32, (CSeg)segw, w, waves, at.sub, blk, at.r0 < n, sh, Plain());
    }
    if (act) res_store(v, X + col, ldx, at, n, full);
}

// As above for E (m rows) and the border of a periodic matrix of m + 2 rows.
// CN: F holds C, and f_i = 2 C_i - (A C)_i is formed in registers; UNI: with
// the same five coefficients in every row, else those of cd.
template <int S, int NW, bool CN, bool UNI>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4))) void k_resident_cyclic(
    const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg32, const SegRec *segw, int64_t m, const double *F, int64_t ldf,
    double *X, int64_t ldx, int64_t batch, int64_t ntiles, const double *cd, const double *Z,
    const CycAux *__restrict__ aux, CycUni uc)
{
    constexpr int K = kResK;
    __shared__ ResLds<S, kResWaves> sh;
    const int64_t tile = res_tile(ntiles), n = m + 2, ldc = cyc_ld(n);
    if (tile < 0) return;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64)), waves = (int)(blockDim.x / 64);
    const Place at = res_place<S>(w);
    const int64_t c0 = tile * S, blk = at.r0 / K;
    const bool act = c0 + at.s < batch, full = at.rw + 64 / S * K <= m && ldf <= kFullLd<S> && ldx <= kFullLd<S>;
    const int64_t sc = act ? at.s : batch - 1 - c0;
    const double *col = F + c0 + sc;
    const int L = m - at.r0 < K ? (int)(m - at.r0) : K;
    typedef std::conditional_t<(S < 16), QuadCoef, Coef<K>> C;
    constexpr int CR = sizeof(C) / sizeof(double);
    auto crow = [&](int i) { return at.r0 + (S < 16 ? 4 * i + (int)(threadIdx.x & 3) : coef_row<K>(i)); };
    double v[K];
    if (w == 0) {  // the right-hand side's last two entries
        double f0, f1;
        if constexpr (CN) {
            const double g0 = col[(m - 2) * ldf], g1 = col[(m - 1) * ldf], g2 = col[m * ldf], g3 = col[(m + 1) * ldf], g4 = col[0],
                         g5 = col[ldf];
            CycUni u0 = uc, u1 = uc;
            if constexpr (!UNI)
#pragma unroll
                for (int d = 0; d < 5; d++) {
                    u0.c[d] = cd[d * ldc + m];
                    u1.c[d] = cd[d * ldc + m + 1];
                }
            f0 = cn_row_u(u0, g0, g1, g2, g3, g4);
            f1 = cn_row_u(u1, g1, g2, g3, g4, g5);
        } else {
            f0 = col[m * ldf];
            f1 = col[(m + 1) * ldf];
        }
        sh.ft[0][at.s] = f0;
        sh.ft[1][at.s] = f1;
    }
    if constexpr (CN) {
        // C rows r0-2 .. r0+K+1, periodic (past row n-1 nothing is used)
        double h[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int64_t r = i < 2 ? at.r0 - 2 + i : at.r0 + K + i - 2;
            h[i] = col[(r < 0 ? r + n : r >= n ? n - 1 : r) * ldf];
        }
        res_load(v, F + c0, ldf, sc, at, n, full);
        C g[5];
        if constexpr (!UNI) {
#pragma unroll
            for (int d = 0; d < 5; d++)
#pragma unroll
                for (int i = 0; i < CR; i++) g[d].c[i] = cd[d * ldc + (crow(i) < n ? crow(i) : n - 1)];
        }
        double p2 = h[0], p1 = h[1];
        unroll<K>([&](auto kk) {
            constexpr int k = decltype(kk)::value;
            if constexpr (!UNI && k % 8 == 0) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int d = 0; d < 5; d++) g[d].hold();
            }
            const double ck = v[k];
            const double n1 = k + 1 < K ? v[k + 1 < K ? k + 1 : 0] : h[2];
            const double n2 = k + 2 < K ? v[k + 2 < K ? k + 2 : 0] : (k + 2 == K ? h[2] : h[3]);
            CycUni u = uc;
            if constexpr (!UNI) u = CycUni{{g[0].template get<k>(), g[1].template get<k>(), g[2].template get<k>(),
                                            g[3].template get<k>(), g[4].template get<k>()}};
            v[k] = cn_row_u(u, p2, p1, ck, n1, n2);
            p2 = p1;
            p1 = ck;
        });
        if (!full) {
#pragma unroll
            for (int k = 0; k < K; k++) v[k] = k < L ? v[k] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < K; k++) pin(v[k]);
    } else {
        res_load(v, F + c0, ldf, sc, at, m, full);
    }
    if constexpr (S < 16) {
        narrow_sweeps<S>(v, fwd, bwd, seg32, w, waves, at.sub, blk, at.r0 < m, sh);
    } else {
        Rec<K> rc;
        load_forward<K>(rc, fwd, at.r0);
        load_backward<K>(rc, bwd, at.r0);
        res_forward<S>(v, rc, seg32, (CSeg)segw, w, at.sub, blk, sh);
        res_backward<S>(v, rc, seg32, (CSeg)segw, w, waves, at.sub, blk, at.r0 < m, sh, Plain());
    }
    // y at the rows that the border meets, x_tail, and x = y - Z x_tail
    if (at.r0 == 0) {
        sh.xe[0][at.s] = v[0];
        sh.xe[1][at.s] = v[1];
    }
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const int64_t r = m - 2 + i;
        double y = v[0];
#pragma unroll
        for (int k = 1; k < K; k++) y = k == (int)(r % K) ? v[k] : y;
        if (blk == r / K) sh.xe[2 + i][at.s] = y;
    }
    C z0, z1;
#pragma unroll
    for (int i = 0; i < CR; i++) {
        const Dbl2 u = ((const Dbl2 *)Z)[crow(i)];
        z0.c[i] = u.x;
        z1.c[i] = u.y;
    }
    __syncthreads();
    double t0 = sh.ft[0][at.s], t1 = sh.ft[1][at.s];
    const int nh = aux->nh;
    for (int k = 0; k < nh; k++) {
        const int64_t c = aux->hcol[k];
        const double y = aux->hv[k] * sh.xe[c < 2 ? (int)c : (int)(c - m) + 4][at.s];
        if (aux->hq[k] == 0) t0 -= y;
        else t1 -= y;
    }
    const double x0 = fma(aux->minv[1], t1, aux->minv[0] * t0), x1 = fma(aux->minv[3], t1, aux->minv[2] * t0);
    unroll<K>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        if constexpr (k % 8 == 0) {
            __builtin_amdgcn_sched_barrier(0);
            z0.hold();
            z1.hold();
        }
        v[k] = fma(-z1.template get<k>(), x1, fma(-z0.template get<k>(), x0, v[k]));
        pin(v[k]);  // here, not in the stores' branch
    });
    if (!act) return;
    res_store(v, X + c0, ldx, at, m, full);
    if (at.r0 == 0) {
        X[c0 + at.s + m * ldx] = x0;
        X[c0 + at.s + (m + 1) * ldx] = x1;
    }
}

// System-major storage (system i = 0 .. per - 1 of group g at src + g * kst + i *
// sst, n values each; a tile is up to S systems of one group), as k_stream_t
// (stream_t.hip) has it: runs of 16 rows are loaded as pairs and turned in
// place through LDS, 64 (system, block) combinations to the wave.
//
// ST: C comes in at src and R = C + dt_g Lap_h(C^3 - C) is formed over it.  The y
// neighbours' terms are the next lanes' own, and at the tile's ends those of
// two more systems, from LDS; the rows above and below a block are the lanes'
// of the blocks around it, and those around the wave's 128 rows come from
// memory, 16 values a side (one from a line of its own for every lane were as
// many lines again as the block: the 2-D step on 1024 x 1024 x 32 226 us, 215 so).
//
// A workgroup of 16 systems has as many waves as the rows take, and as many
// workgroups share a compute unit as its 16 waves allow, each in a phase of
// its own: HBM-bound (n = 1024 x 32768 100 us, 5.4 TB/s, from 118 streaming; with
// 32 systems, one workgroup to the unit, 126).
template <int S, int NW, bool ST, bool NT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_resident_t(
    const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg32, const SegRec *segw, int64_t n, const double *src, double *F,
    int64_t per, int64_t sst, int64_t kst, int64_t tpk, int64_t ntiles, const double *dt, double inv_h2)
{
    constexpr int K = kResK, G = 64 / S;
    __shared__ ResLds<S, NW> sh;
    __shared__ double tb[NW][8][66];
    const int64_t tile = res_tile(ntiles);
    if (tile < 0) return;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64)), waves = (int)(blockDim.x / 64);
    const Place at = res_place<S>(w);
    const int lane = threadIdx.x & 63, pair = lane & 7, grp = lane >> 3;
    const int64_t g = ST ? tile / tpk : 0, s0 = (tile - g * tpk) * S, base = g * kst + s0 * sst, blk = at.r0 / K;
    const int cnt = (int)(per - s0 < S ? per - s0 : S);
    const bool full = at.rw + G * K <= n;
    const int L = n - at.r0 < K ? (int)(n - at.r0) : K;
    double(*tw)[66] = tb[w];
    typedef Dbl2 Dbl2u __attribute__((aligned(8)));  // 16 bytes at any double
    typedef __attribute__((address_space(1))) const Dbl2u *G2;
    typedef __attribute__((address_space(1))) Dbl2u *W2;
    typedef __attribute__((address_space(1))) const double *G1;
    double v[K], up = 0.0, low = 0.0, hv[G] = {};
    if constexpr (ST) {
        // the rows around the wave's (a lane's own come from its neighbours), and
        // the tile's neighbour systems: rows rw + 64 i + lane of the system above
        // in hv[i], of the one below in hv[G / 2 + i]
        const double *c = src + base + (int64_t)(at.s < cnt ? at.s : cnt - 1) * sst;
        const int64_t ru = at.rw - 1, rl = at.rw + G * K;
        up = c[ru < 0 ? 0 : ru];
        low = c[rl < n ? rl : n - 1];
        up = ru >= 0 ? up : 0.0;
        low = rl < n ? low : 0.0;
#pragma unroll
        for (int i = 0; i < G; i++) {
            const bool below = i >= G / 2, in = below ? s0 + cnt < per : s0 > 0;
            const int64_t row = at.rw + 64 * (i % (G / 2)) + lane, y = below ? (in ? cnt : cnt - 1) : in ? -1 : 0;
            hv[i] = src[base + y * sst + (row < n ? row : n - 1)];
            hv[i] = in && row < n ? hv[i] : 0.0;
        }
    }
    // rows 16 c + 2 pair + e of combination 8 q + grp into v[16 c + 2 q + e];
    // systems past the tile repeat its last one.  Rows past the last one are
    // read all the same, and cleared, where a further system lies behind the
    // tile's (so that they are inside the array: at most 127 of them).
    const bool whole = full || (s0 + S < per && sst >= 128);
#pragma unroll
    for (int j = 0; j < S / 8; j++) {
        const int sj = 8 * j + grp;
        const double *p = src + base + (int64_t)(sj < cnt ? sj : cnt - 1) * sst;
        if (whole) {
            p += at.rw + 2 * pair;
#pragma unroll
            for (int b = 0; b < G; b++)
#pragma unroll
                for (int c = 0; c < K / 16; c++) {
                    const G2 a = (G2)(p + K * b + 16 * c);
                    const Dbl2u u = NT ? __builtin_nontemporal_load(a) : *a;
                    v[16 * c + 2 * (b * (S / 8) + j)] = u.x;
                    v[16 * c + 2 * (b * (S / 8) + j) + 1] = u.y;
                }
        } else {
#pragma unroll
            for (int b = 0; b < G; b++)
#pragma unroll
                for (int c = 0; c < K / 16; c++)
#pragma unroll
                    for (int e = 0; e < 2; e++) {
                        const int64_t row = at.rw + K * b + 16 * c + 2 * pair + e;
                        v[16 * c + 2 * (b * (S / 8) + j) + e] = ((G1)p)[row < n ? row : n - 1];
                    }
        }
    }
    // turned: v[k] = row r0 + k of the lane's system
#pragma unroll
    for (int c = 0; c < K / 16; c++)
#pragma unroll
        for (int e = 0; e < 2; e++) {
#pragma unroll
            for (int i = 0; i < 8; i++) tw[pair][8 * i + grp] = v[16 * c + 2 * i + e];
#pragma unroll
            for (int i = 0; i < 8; i++) v[16 * c + 2 * i + e] = tw[i][lane];
        }
    if (!full) {
#pragma unroll
        for (int k = 0; k < K; k++) v[k] = k < L ? v[k] : 0.0;
    }
    Rec<K> rc;
    if constexpr (ST) {
        if (cnt < S) {
#pragma unroll
            for (int k = 0; k < K; k++) v[k] = at.s < cnt ? v[k] : 0.0;
        }
        double *nb = tw[0];  // terms of the neighbour systems, above then below
#pragma unroll
        for (int i = 0; i < G; i++) nb[64 * i + lane] = ch_wterm(hv[i]);
        const bool first = at.s == 0, last = at.s == S - 1;
        const double *mine = nb + (first ? 0 : 32 * G) + 32 * at.sub;
        const double dtk = dt[g];
        const double above = __shfl(v[K - 1], lane - S, 64), next = __shfl(v[0], lane + S, 64);
        up = at.sub > 0 ? above : up;
        low = at.sub < G - 1 ? next : low;
        double wprev = ch_wterm(up), wcur = ch_wterm(v[0]);
        unroll<K>([&](auto kk) {
            constexpr int row = decltype(kk)::value;
            if constexpr (row % 4 == 0) __builtin_amdgcn_sched_barrier(0);
            const double e = mine[row];
            const double a = lane_shift<true>(wcur, e), b = lane_shift<false>(wcur, e);
            const double ws = first ? e : a, wn = last ? e : b;
            const double wnext = ch_wterm(row + 1 < K ? v[row + 1 < K ? row + 1 : 0] : low);
            v[row] = ch_point(v[row], wcur, wnext, wprev, wn, ws, dtk, inv_h2);
            wprev = wcur;
            wcur = wnext;
        });
        if (!full) {
#pragma unroll
            for (int k = 0; k < K; k++) v[k] = k < L ? v[k] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < K; k++) pin(v[k]);
    }
    load_forward<K>(rc, fwd, at.r0);
    load_backward<K>(rc, bwd, at.r0);
    res_forward<S>(v, rc, seg32, (CSeg)segw, w, at.sub, blk, sh);
    res_backward<S>(v, rc, seg32, (CSeg)segw, w, waves, at.sub, blk, at.r0 < n, sh, Plain());
    // turned back and stored as runs
#pragma unroll
    for (int c = 0; c < K / 16; c++)
#pragma unroll
        for (int e = 0; e < 2; e++) {
#pragma unroll
            for (int i = 0; i < 8; i++) tw[i][lane] = v[16 * c + 2 * i + e];
#pragma unroll
            for (int i = 0; i < 8; i++) v[16 * c + 2 * i + e] = tw[pair][8 * i + grp];
        }
#pragma unroll
    for (int j = 0; j < S / 8; j++) {
        const int sj = 8 * j + grp;
        if (sj >= cnt) continue;
        double *p = F + base + (int64_t)sj * sst + at.rw + 2 * pair;
        const int left = (int)(n - at.rw < G * K ? n - at.rw : G * K) - 2 * pair;
#pragma unroll
        for (int b = 0; b < G; b++)
#pragma unroll
            for (int c = 0; c < K / 16; c++) {
                const int i = b * (S / 8) + j;
                const Dbl2u u = {v[16 * c + 2 * i], v[16 * c + 2 * i + 1]};
                if (full) {
                    if (NT) __builtin_nontemporal_store(u, (W2)(p + K * b + 16 * c));
                    else *(W2)(p + K * b + 16 * c) = u;
                } else {
                    if (K * b + 16 * c + 1 < left) *(W2)(p + K * b + 16 * c) = u;
                    else if (K * b + 16 * c < left) p[K * b + 16 * c] = u.x;
                }
            }
    }
}

struct ResLaunch {
    dim3 grid, block;
    int64_t ntiles;
};

ResLaunch res_launch(int64_t n, int width, int64_t batch)
{
    const int64_t ntiles = (batch + width - 1) / width, rows = 64 / width * kResK;
    return ResLaunch{dim3((unsigned)((ntiles + 7) / 8 * 8)), dim3((unsigned)(64 * ((n + rows - 1) / rows))), ntiles};
}

template <bool ST>
hipError_t launch_t(const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg32, const SegRec *seg64, int64_t n,
                    const double *src, double *F, int64_t per, int64_t sst, int64_t kst, int64_t groups, const double *dt,
                    double inv_h2, hipStream_t s)
{
    const int64_t tpk = (per + 15) / 16, ntiles = tpk * groups;
    const ResLaunch g = res_launch(n, 16, ntiles * 16);
    const bool lines = (uintptr_t)src % 128 == 0 && (uintptr_t)F % 128 == 0 && sst % 16 == 0 && kst % 16 == 0;
    // (LDS for the waves there are, so that it does not limit the workgroups)
    auto fn = lines ? k_resident_t<16, 16, ST, true> : k_resident_t<16, 16, ST, false>;
    if (g.block.x <= 64) fn = lines ? k_resident_t<16, 1, ST, true> : k_resident_t<16, 1, ST, false>;
    else if (g.block.x <= 128) fn = lines ? k_resident_t<16, 2, ST, true> : k_resident_t<16, 2, ST, false>;
    else if (g.block.x <= 256) fn = lines ? k_resident_t<16, 4, ST, true> : k_resident_t<16, 4, ST, false>;
    else if (g.block.x <= 512) fn = lines ? k_resident_t<16, 8, ST, true> : k_resident_t<16, 8, ST, false>;
    hipLaunchKernelGGL(fn, g.grid, g.block, 0, s, fwd, bwd, seg32, seg64, n, src, F, per, sst, kst, tpk, ntiles, dt, inv_h2);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_resident_t(const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg32, const SegRec *seg64, int64_t n,
                             double *F, int64_t ld, int64_t batch, hipStream_t s)
{
    return launch_t<false>(fwd, bwd, seg32, seg64, n, F, F, batch, ld, 0, 1, nullptr, 0.0, s);
}

hipError_t launch_resident_ch2d(const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg32, const SegRec *seg64, int64_t n,
                                const double *C, double *R, int64_t ny, int64_t ninst, const double *dt, double h, hipStream_t s)
{
    return launch_t<true>(fwd, bwd, seg32, seg64, n, C, R, ny, ninst * n, n, ninst, dt, 1.0 / (h * h), s);
}

hipError_t launch_resident(const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg32, const SegRec *seg64, int64_t n, int width,
                           const void *F, bool f32, int64_t ldf, double *X, int64_t ldx, int64_t batch, hipStream_t s, int64_t ts)
{
    const ResLaunch g = res_launch(n, width, batch);
    auto go = [&](auto f) {
        typedef decltype(f) TI;
        auto fn = width == 32 ? k_resident<32, 16, TI> : k_resident<16, 16, TI>;
        // (eight waves of four systems have 256 registers each; sixteen spill
        // 59 of theirs: 4096 x 154 23 us, with eight 18)
        if (width == 4) fn = g.block.x <= 512 ? k_resident<4, 8, TI> : k_resident<4, 16, TI>;
        hipLaunchKernelGGL(fn, g.grid, g.block, 0, s, fwd, bwd, seg32, seg64, n, (const TI *)F, ldf, X, ldx, batch, g.ntiles, ts);
        return hipGetLastError();
    };
    return f32 ? go(float()) : go(double());
}

hipError_t launch_resident_cyclic(const FwdRec *fwd, const BwdRec *bwd, const SegRec *seg32, const SegRec *seg64,
                                  const double *cd, const double *Z, const CycAux *aux, int64_t n, int width, bool cn,
                                  const double *F, int64_t ldf, double *X, int64_t ldx, int64_t batch, hipStream_t s,
                                  const double *uni)
{
    CycUni uc = {{0.0, 0.0, 0.0, 0.0, 0.0}};
    if (uni)
        for (int k = 0; k < 5; k++) uc.c[k] = uni[k];
    auto pick = [&](auto cn_, auto uni_) {
        constexpr bool C = decltype(cn_)::value, U = decltype(uni_)::value;
        return width == 4 ? k_resident_cyclic<4, 8, C, U> : width == 16 ? k_resident_cyclic<16, 16, C, U> : k_resident_cyclic<32, 16, C, U>;
    };
    const std::true_type yes;
    const std::false_type no;
    const auto fn = !cn ? pick(no, yes) : uni ? pick(yes, yes) : pick(yes, no);
    const ResLaunch g = res_launch(n, width, batch);
    hipLaunchKernelGGL(fn, g.grid, g.block, 0, s, fwd, bwd, seg32, seg64, n, F, ldf, X, ldx, batch, g.ntiles, cd, Z, aux, uc);
    return hipGetLastError();
}

}  // namespace pent
