// stream.h -- device pieces of the streaming sweeps (stream.hip): one
// workgroup takes whole 64-system tiles and moves down their rows, its waves
// holding consecutive K-row blocks in registers, so that no value leaves the
// compute unit between the load of a block and the store of its solution.
//
// Forward (Sec. 2.4) the blocks follow one another exactly: a block starts
// from the state its predecessor left in LDS.  Backward, a block's incoming
// state depends on every row below it, but the matrices this is built for
// carry little of it far: with Tb_j the backward transfer matrix of block j
// (SegRec) and a_j the top state of a back substitution over block j from
// zero,
//     z_b = a_{b+1} + Tb_{b+1} (a_{b+2} + Tb_{b+2} (... + Tb_{b+D} z_{b+D})),
// and for the D of the plan the product P_b = Tb_{b+1} ... Tb_{b+D} is below
// kTruncTarget.  So a block waits for the next D blocks only, and takes
// z_{b+D} as zero.  What was left out, P_b z_{b+D}, is looked at as soon as
// z_{b+D} is known: where it is not below half a unit of rounding of z_b
// (kNegligible), or not a number, the workgroup adds it after its last block
// (stream_repair), exactly as the recurrence would have carried it.  The
// results are those of the untruncated chain for every right-hand side; D
// decides only how often the repair runs.
#pragma once

#include <climits>
#include <type_traits>
#include <utility>

#include "lookback.h"

namespace pent {
namespace st {

using namespace lb;

constexpr double kNegligible = 0x1p-54;  // a neglected state against the state it is left out of
constexpr double kRepair = 0x1p-53;      // ... and from where the repair adds it: a system that
                                         // passed above is never touched for a neighbour's sake

// Lane L of every row of 16 lanes, to the whole row (one 64-bit DPP move).
template <int L>
__device__ __forceinline__ double row_get(double v)
{
    return __longlong_as_double(
        __builtin_amdgcn_update_dpp((long long)0, __double_as_longlong(v), 0x150 + L, 0xF, 0xF, true));
}

// The same value, opaque to the optimiser: lane reads of it are not merged
// with those of an earlier sweep (kept, they would fill the registers).
__device__ __forceinline__ void pin(double &x) { asm volatile("" : "+v"(x)); }

// f(integral constant 0), f(1), ... f(N - 1)
template <int... I, typename F>
__device__ __forceinline__ void unroll_seq(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unroll(F f)
{
    unroll_seq(std::make_integer_sequence<int, N>{}, f);
}

// One coefficient of a block's K rows.  32-row blocks keep rows 16 s + l in
// lane l of every row of 16 lanes of register s, and broadcast by DPP; 64-row
// ones, short of registers, one row per lane, and broadcast through scalar
// registers (two v_readlane).  Neither has a memory latency between rows: a
// scalar load per batch of rows, or an LDS broadcast per row, made the
// sweeps two to five times longer.
template <int K>
struct Coef {
    static constexpr int S = K == 32 ? 2 : 1;
    double c[S];
    template <int k>
    __device__ __forceinline__ double get() const
    {
        if constexpr (K == 32) return row_get<k % 16>(c[k / 16]);
        else return lane_double(c[0], k);
    }
    __device__ __forceinline__ void hold()
    {
#pragma unroll
        for (int s = 0; s < S; s++) pin(c[s]);
    }
};

template <int K>
struct Rec {
    Coef<K> ra, ap, bp, gm, dl;
};

// Row of the block that this lane's register s holds.
template <int K>
__device__ __forceinline__ int coef_row(int s)
{
    return K == 32 ? 16 * s + (int)(threadIdx.x & 15) : (int)(threadIdx.x & 63);
}

typedef double Dbl2 __attribute__((ext_vector_type(2)));

template <int K>
__device__ __forceinline__ void load_forward(Rec<K> &r, const FwdRec *f, int64_t r0)
{
#pragma unroll
    for (int s = 0; s < Coef<K>::S; s++) {
        const Dbl2 *p = (const Dbl2 *)(f + r0 + coef_row<K>(s));
        const Dbl2 u = p[0];
        r.ra.c[s] = u.x;
        r.ap.c[s] = u.y;
        r.bp.c[s] = p[1].x;
    }
}

template <int K>
__device__ __forceinline__ void load_backward(Rec<K> &r, const BwdRec *b, int64_t r0)
{
#pragma unroll
    for (int s = 0; s < Coef<K>::S; s++) {
        const Dbl2 q = *(const Dbl2 *)(b + r0 + coef_row<K>(s));
        r.gm.c[s] = q.x;
        r.dl.c[s] = q.y;
    }
}

// Rows p, p + ld, ... at lane offset lo into v; rows k >= L give zero (the
// last row is read again in their place: no load stands under a condition).
// NT: loads and stores that pass the caches by, for rows on whole 128-byte
// lines; where a line holds the columns of two tiles the L2 has to keep it
// for the other (N = 256 x 20011 with an odd row stride: 17 us cached, 23 us
// past the caches; N = 4096 x 65536, aligned: 7% less past them).
template <int K, bool NT, typename TI>
__device__ __forceinline__ void load_block(double (&v)[K], const TI *src, unsigned int lo, int64_t ld, int L)
{
    typedef __attribute__((address_space(1))) const TI *G;
    G p = (G)src;
    if (L == K) {
#pragma unroll
        for (int k = 0; k < K; k++) {
            v[k] = (double)(NT ? __builtin_nontemporal_load(p + lo) : p[lo]);
            p = fresh(p + ld);  // one uniform pointer moved along, not K of them
        }
    } else {
#pragma unroll
        for (int k = 0; k < K; k++) {
            v[k] = (double)p[lo];
            p = fresh(k + 1 < L ? p + ld : p);
        }
#pragma unroll
        for (int k = 0; k < K; k++) v[k] = k < L ? v[k] : 0.0;
    }
}

template <int K, bool NT>
__device__ __forceinline__ void store_block(const double (&v)[K], double *dst, unsigned int lo, int64_t ld, int L)
{
    typedef __attribute__((address_space(1))) double *G;
    G p = (G)dst;
    if (L == K) {
#pragma unroll
        for (int k = 0; k < K; k++) {
            if (NT) __builtin_nontemporal_store(v[k], p + lo);
            else p[lo] = v[k];
            p = fresh(p + ld);
        }
    } else {
#pragma unroll
        for (int k = 0; k < K; k++) {
            if (k < L) p[lo] = v[k];
            p = fresh(k + 1 < L ? p + ld : p);
        }
    }
}

// The tiles of a workgroup: t0, t0 + step, ... below end.  Workgroups go
// round the eight XCDs, and each XCD takes a contiguous eighth of the tiles,
// so that lines shared by neighbouring tiles meet in one L2 (N = 4096 x 20011:
// 425 us with tiles dealt round, 398 us so).  The grid is a multiple of 8.
struct Tiles {
    int t0, step, end;
};
__device__ __forceinline__ Tiles my_tiles(int ntiles)
{
    const int x = blockIdx.x % 8;
    Tiles t;
    t.t0 = (int)((int64_t)ntiles * x / 8) + blockIdx.x / 8;
    t.step = gridDim.x / 8;
    t.end = (int)((int64_t)ntiles * (x + 1) / 8);
    return t;
}

// The walk of a workgroup over its tiles.  leave: a bit for each, in their
// order, of those that it passes by (null: none).
typedef unsigned long long LeaveBits[kLeftTiles / 64];
struct Walk {
    Tiles mine;
    const unsigned long long *leave;
    int t, k;           // the tile, and its number among the workgroup's
    unsigned int turn;  // tiles walked before it
    __device__ __forceinline__ void settle()
    {
        while (leave && t < mine.end && __builtin_amdgcn_readfirstlane((int)(leave[k / 64] >> (k % 64)) & 1)) {
            t += mine.step;
            k++;
        }
    }
    __device__ __forceinline__ void start()
    {
        t = mine.t0;
        k = 0;
        turn = 0;
        settle();
    }
    __device__ __forceinline__ void next()
    {
        t += mine.step;
        k++;
        turn++;
        settle();
    }
};

// The tiles of this workgroup that k_find_left marked (stream.hip).
template <int NW>
__device__ __forceinline__ void read_left(const Left &left, const Tiles &mine, int cw, LeaveBits &leave)
{
    for (int k = threadIdx.x; k < kLeftTiles; k += 64 * NW) {
        const int64_t t = mine.t0 + (int64_t)k * mine.step;
        const unsigned long long m = __ballot(t < mine.end && *left_mark(left.ex, left.groups, t * cw) != 0);
        if ((threadIdx.x & 63) == 0) leave[k / 64] = m;
    }
    __syncthreads();
}

// Forward recurrence over the block from (p2, p1).  STORE writes g over v.
template <int K, bool STORE, typename R>
__device__ __forceinline__ void sweep_forward(double (&v)[K], R &r, double &p2, double &p1)
{
    unroll<K>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        if constexpr (k % 8 == 0) {
            __builtin_amdgcn_sched_barrier(0);
            r.ra.hold();
            r.ap.hold();
            r.bp.hold();
        }
        const double g = fma(-r.bp.template get<k>(), p1, fma(-r.ap.template get<k>(), p2, r.ra.template get<k>() * v[k]));
        if (STORE) v[k] = g;
        p2 = p1;
        p1 = g;
    });
}

// What a plain solve adds to the phases: nothing.
struct Plain {
    static constexpr bool late = false;              // whether the backward records wait for the second sweep
    __device__ __forceinline__ void fetch() {}       // with the backward records, ahead of the second sweep
    __device__ __forceinline__ void ordered(int) {}  // in the tile's order, with the forward state
    __device__ __forceinline__ void took(double, double) {}  // with the state taken from below
    __device__ __forceinline__ void ready() {}       // before the last sweep
    template <int k>
    __device__ __forceinline__ double out(double x) const  // what is stored for row k
    {
        return x;
    }
    __device__ __forceinline__ void hold() {}
};

struct PlainLate : Plain {
    static constexpr bool late = true;
};

// Back substitution over the block from (q1, q2) = (x_{r0+K}, x_{r0+K+1}); on
// exit (q1, q2) = (x_{r0}, x_{r0+1}).  STORE writes x (ex.out of it) over v.
template <int K, bool STORE, typename R, typename Extra>
__device__ __forceinline__ void sweep_backward(double (&v)[K], R &r, double &q1, double &q2, Extra &ex)
{
    unroll<K>([&](auto kk) {
        constexpr int k = K - 1 - decltype(kk)::value;
        if constexpr (k % 8 == 7) {
            __builtin_amdgcn_sched_barrier(0);
            r.gm.hold();
            r.dl.hold();
            if (STORE) ex.hold();
        }
        const double x = fma(-r.gm.template get<k>(), q1, fma(-r.dl.template get<k>(), q2, v[k]));
        if (STORE) v[k] = ex.template out<k>(x);
        q2 = q1;
        q1 = x;
    });
}

// LDS of a workgroup of NW waves.  Block q of the workgroup's sequence (tile
// after tile, down the rows) belongs to wave q % NW and uses that wave's
// slots; a flag holds q + 1 once block q has filled its slot.  A slot is
// filled again by block q + NW at the earliest, whose forward sweep comes
// after every block up to q + NW - 1 has been swept forward, that is, after
// every wave but this one has finished its block before q + NW: the readers
// of y (block q + 1) and a (blocks before q) are done by then.  z is read by
// block q + D, which may be later, so its slots alternate.
template <int NW, bool CHECK = true>
struct StreamLds {
    double y[NW][2][64];                 // state leaving the block downward
    double a[NW][2][64];                 // top state of the zero-start back substitution
    double z[CHECK ? 2 : 1][CHECK ? NW : 1][2][64];  // state taken to enter the block from below
    unsigned int fdone;                  // blocks swept forward
    unsigned int aflag[NW], zflag[2][NW];
    int last[32], first[32];             // by turn % 32: the tile's blocks that left out something not negligible
};

template <int NW, bool CHECK>
__device__ __forceinline__ void stream_init(StreamLds<NW, CHECK> &sh)
{
    if (threadIdx.x < NW) {
        sh.aflag[threadIdx.x] = 0;
        sh.zflag[0][threadIdx.x] = 0;
        sh.zflag[1][threadIdx.x] = 0;
    }
    if (threadIdx.x < 32) {
        sh.last[threadIdx.x] = -1;
        sh.first[threadIdx.x] = INT_MAX;
    }
    if (threadIdx.x == 0) sh.fdone = 0;
    __syncthreads();
}

// Waits until the flag has reached v; false when the bounded wait ran out.
__device__ __forceinline__ bool lds_wait(unsigned int *p, unsigned int v)
{
    bool ok = true;
    for (int spin = 0;; spin++) {
        const unsigned int x = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if ((int)((unsigned int)__builtin_amdgcn_readfirstlane((int)x) - v) >= 0) break;
        if (spin >= kSpin) {
            ok = false;
            break;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    return ok;
}

// The wave's LDS writes are complete before the flag is.
__device__ __forceinline__ void lds_post(unsigned int *p, unsigned int v)
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

typedef __attribute__((address_space(4))) const double *CTrunc;  // P_b, four doubles each, column-major

// Both sweeps of block q of the workgroup (block b of nblk of its tile, wave
// w's par-th round): v holds the right-hand side on entry and x on exit.
// CHECK false: nothing is left out, or Extra looks at it (took).
template <int K, int NW, bool CHECK, typename Extra>
__device__ __forceinline__ void stream_phases(double (&v)[K], Rec<K> &rc, const BwdRec *bwd, CSeg seg, CTrunc trunc, int b, int nblk,
                                              int D, unsigned int q, int w, int par, unsigned int turn,
                                              StreamLds<NW, CHECK> &sh,
                                              unsigned int *err, Extra ex)
{
    const int lane = threadIdx.x & 63;
    // forward: the block's outgoing state for a zero incoming one, while the
    // rows arrive; then, in the tile's order, the state it enters with from
    // the block above and, one link further, the one it leaves with.  Raised
    // priority there: every later block of the tile waits for it.
    double e0 = 0.0, e1 = 0.0;
    sweep_forward<K, false>(v, rc, e0, e1);
    pin(e0);
    pin(e1);
    const double t0 = seg[b].tf[0], t1 = seg[b].tf[1], t2 = seg[b].tf[2], t3 = seg[b].tf[3];
    bool ok = lds_wait(&sh.fdone, q);
    __builtin_amdgcn_s_setprio(3);
    double y0 = 0.0, y1 = 0.0;
    if (b > 0) {
        const int pw = w == 0 ? NW - 1 : w - 1;
        y0 = sh.y[pw][0][lane];
        y1 = sh.y[pw][1][lane];
    }
    double n0 = y0, n1 = y1;
    link(e0, e1, t0, t1, t2, t3, n0, n1);
    sh.y[w][0][lane] = n0;
    sh.y[w][1][lane] = n1;
    ex.ordered(lane);
    lds_post(&sh.fdone, q + 1);
    __builtin_amdgcn_s_setprio(0);
    if constexpr (std::remove_reference_t<Extra>::late) {
        load_backward<K>(rc, bwd, (int64_t)b * K);
        ex.fetch();
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_sched_barrier(0);
    }
    sweep_forward<K, true>(v, rc, y0, y1);
    double a0 = 0.0, a1 = 0.0;
    sweep_backward<K, false>(v, rc, a0, a1, ex);
    pin(a0);
    pin(a1);
    sh.a[w][0][lane] = a0;
    sh.a[w][1][lane] = a1;
    lds_post(&sh.aflag[w], q + 1);
    // the state from below, over the next D blocks
    const int m = D < nblk - 1 - b ? D : nblk - 1 - b;
    double z0 = 0.0, z1 = 0.0;
    for (int i = m; i >= 1; i--) {
        const int ww = w + i >= NW ? w + i - NW : w + i;
        const double u0 = seg[b + i].tb[0], u1 = seg[b + i].tb[1], u2 = seg[b + i].tb[2], u3 = seg[b + i].tb[3];
        ok = lds_wait(&sh.aflag[ww], q + i + 1) && ok;
        link(sh.a[ww][0][lane], sh.a[ww][1][lane], u0, u1, u2, u3, z0, z1);
    }
    if (!ok) {  // never seen: a wait inside a workgroup that ran out
        if (lane == 0) atomicOr(err, 1u);
        z0 = __builtin_nan("");
        z1 = __builtin_nan("");
    }
    if constexpr (CHECK) {
        sh.z[par][w][0][lane] = z0;
        sh.z[par][w][1][lane] = z1;
        lds_post(&sh.zflag[par][w], q + 1);
    }
    if (CHECK && b >= D) {
        // what block b - D left out, P z, against the state it took
        const int ww = w >= D ? w - D : w - D + NW, pp = w >= D ? par : par ^ 1;
        const CTrunc P = trunc + 4 * (int64_t)(b - D);
        const double p0 = P[0], p1 = P[1], p2 = P[2], p3 = P[3];
        if (!lds_wait(&sh.zflag[pp][ww], q - D + 1) && lane == 0) atomicOr(err, 1u);
        const double c0 = fma(p2, z1, p0 * z0), c1 = fma(p3, z1, p1 * z0);
        const double o0 = sh.z[pp][ww][0][lane], o1 = sh.z[pp][ww][1][lane];
        const bool fine = fmax(fabs(c0), fabs(c1)) <= kNegligible * fmax(fabs(o0), fabs(o1)) && c0 == c0 && c1 == c1;
        if (__ballot(!fine) != 0 && lane == 0) {
            atomicMax(&sh.last[turn % 32], b - D);
            atomicMin(&sh.first[turn % 32], b - D);
        }
    }
    ex.took(z0, z1);
    ex.ready();
    sweep_backward<K, true>(v, rc, z0, z1, ex);
    // x is complete here: keep the sweep from sinking into the stores
#pragma unroll
    for (int k = 0; k < K; k++) pin(v[k]);
}

// f(k, row r + k of this lane) for 16 rows, one pointer moved along.
template <typename F>
__device__ __forceinline__ void repair_rows(double *x, int64_t rs, int64_t r, F f)
{
    double *p = x + r * rs;
#pragma unroll
    for (int k = 0; k < 16; k++) {
        f(k, p);
        p += rs;
        asm volatile("" : "+v"(p));
    }
}

// Adds to a finished tile what its blocks left out (see above), by the whole
// workgroup: element (i, this lane's system) of x at x[i * rs]; off(i) is what
// the stored value lacks to the recurrence's.  From the bottom, sixteen
// blocks at a time: every wave brings one block's incoming state from memory,
// wave 0 carries the states of the chain through them,
//     z_b = (top of block b+1 as stored) + Tb_{b+1} delta_{b+1},
//     delta_b = P_b z_{b+D} (where it counts),
// and every wave adds its block's response to delta.
// Values are read past the caches of the compute unit, in which lines loaded
// earlier may still stand.  As much again is read and written as there are
// rows with something to add, and that bounds it: 4096 x 65536 with a top-hat
// in every system took 1069 us at sigma = 1 and 1276 at 50, against 831 and 855
// for random ones, and with a pulse in one system of each tile 968 and 1139 (3%
// more with every system's rows read for it).  Bringing the states two turns
// ahead and 32 rows at once changed neither.  So the largest calls look for such
// data first, and leave it to look-back (k_gate).
template <int K, int NW, typename Off>
__device__ __forceinline__ void stream_repair(double *x, int64_t rs, bool act, int64_t n, int nblk, int D,
                                              CSeg seg, CBwd bwd, CTrunc trunc, StreamLds<NW> &sh, int w, int slot, Off off)
{
    static_assert(NW >= kStreamMaxDepth + 1, "a.slots hold the last D + 1 states");
    const int lane = threadIdx.x & 63;
    double(*zs)[2][64] = sh.z[0], (*dl)[2][64] = sh.z[1], (*ring)[2][64] = sh.a, (*mat)[2][64] = sh.y;
    // nothing is to be added below the last block that noted something, nor
    // once past the first of them no block of a chunk has anything
    const int top = sh.first[slot], low = sh.last[slot] + D;
    bool any = true;
    // sixteens counted from the bottom, whatever the tile's other systems need:
    // across their edges a state comes from memory, rounded otherwise
    for (int b1 = nblk - 2 - (low < nblk - 2 ? (nblk - 2 - low) / NW * NW : 0); b1 >= 0 && (any || b1 >= top); b1 -= NW) {
        const int b = b1 - w;
        __syncthreads();
        if (b >= 0) {
            const int64_t r = (int64_t)(b + 1) * K;
            zs[w][0][lane] = xload(x + r * rs) + off(r);
            zs[w][1][lane] = r + 1 < n ? xload(x + (r + 1) * rs) + off(r + 1) : 0.0;
            // Tb_{b+1} and P_b beside it
            if (lane < 8) mat[w][0][lane] = lane < 4 ? seg[b + 1].tb[lane & 3] : trunc[4 * (int64_t)b + (lane & 3)];
        }
        __syncthreads();
        if (w == 0) {
            double d0 = 0.0, d1 = 0.0;  // delta of the block below (its own response is in memory across chunks)
            for (int i = 0; i < NW && b1 - i >= 0; i++) {
                const int bb = b1 - i;
                double z0 = zs[i][0][lane], z1 = zs[i][1][lane];
                const double *M = mat[i][0];
                link(z0, z1, M[0], M[1], M[2], M[3], d0, d1);
                z0 = d0;
                z1 = d1;
                d0 = d1 = 0.0;
                if (bb + D <= low && bb + D <= nblk - 2) {
                    const double e0 = ring[(bb + D) % NW][0][lane], e1 = ring[(bb + D) % NW][1][lane];
                    const double c0 = fma(M[6], e1, M[4] * e0), c1 = fma(M[7], e1, M[5] * e0);
                    const bool fine = fmax(fabs(c0), fabs(c1)) <= kRepair * fmax(fabs(z0), fabs(z1)) && c0 == c0 && c1 == c1;
                    if (act && !fine) {
                        d0 = c0;
                        d1 = c1;
                    }
                }
                ring[bb % NW][0][lane] = z0;
                ring[bb % NW][1][lane] = z1;
                dl[i][0][lane] = d0;
                dl[i][1][lane] = d1;
            }
        }
        __syncthreads();
        any = false;
        for (int i = 0; i < NW && b1 - i >= 0; i++)
            any = any || __ballot(!(dl[i][0][lane] == 0.0 && dl[i][1][lane] == 0.0)) != 0;
        if (b >= 0) {
            double d1 = dl[w][0][lane], d2 = dl[w][1][lane];
            if (!(d1 == 0.0 && d2 == 0.0)) {  // in the systems that have something: the others' lines stay untouched
                for (int64_t r = (int64_t)(b + 1) * K - 16; r >= (int64_t)b * K; r -= 16) {
                    double o[16];
                    repair_rows(x, rs, r, [&](int k, const double *p) { o[k] = xload(p); });
#pragma unroll
                    for (int k = 15; k >= 0; k--) {
                        const double d = fma(-bwd[r + k].gm, d1, -bwd[r + k].dl * d2);
                        d2 = d1;
                        d1 = d;
                        o[k] += d;
                    }
                    repair_rows(x, rs, r, [&](int k, double *p) { xstore(p, o[k]); });
                }
            }
        }
        store_fence();  // in memory before the next chunk's states are read
    }
    __syncthreads();
}

}  // namespace st
}  // namespace pent
