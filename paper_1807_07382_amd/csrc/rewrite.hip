// rewrite.hip -- every system with its own matrix, factored and solved in
// one call: the paper's refactor-every-step mode (Sec. 3), in which the
// matrix may change between time steps, measured against a general batched
// pentadiagonal solver.
//
// One lane per system (the factorisation recurrence is not linear in its
// carried values, so the segment decomposition of the constant-matrix
// schedules does not apply), one workgroup per tile of 64 systems.
// Downward pass: the Sec. 2.4 factorisation and forward sweep of row i
// together (beta, alpha, gamma, delta, then g); upward pass: back
// substitution.  The rows go round the workgroup's waves in blocks, each
// wave taking the carried values from its predecessor through LDS, so that
// the chain of divisions of one block runs while the next blocks' 48 B per
// row and lane are on their way: a wave on its own can have only 63 loads
// outstanding, less than a row's latency needs.  gamma, delta and g go to
// memory (gamma and delta to the workspace, g over f) and come back to the
// same wave, except those of each wave's last block, which stay in its
// registers, and gamma and delta of the one before, which stay in LDS: 104 B of
// HBM per unknown, 48 less for the last 112 rows and 32 less for the 112 above.
#include "stream.h"

namespace pent {
namespace {

// 14 rows of six values fit the 256 registers of two waves per SIMD; with 16
// a few spill, and 12 waves of 8 rows spend more on the handovers
// (before the blocks in LDS, n = 1024, us, 14 x 8 / 16 x 8 / 8 x 12: 500 systems
// 136 / 140 / 138, 16384 245 / 249 / 252, 65536 1134 / 1128 / 1154; n = 8192 x 2000
// 1069 / 1143 / 1079).
constexpr int kRows = 14;  // rows of a block
constexpr int kWaves = 8;  // waves of a workgroup

typedef __attribute__((address_space(1))) const double *GIn;
typedef __attribute__((address_space(1))) double *GOut;

// A row's element of this lane: a uniform base and a 32-bit byte offset, so
// that the addresses take no vector registers.
__device__ __forceinline__ GIn at(GIn p, unsigned int off)
{
    return (GIn)((__attribute__((address_space(1))) const char *)p + off);
}
__device__ __forceinline__ GOut at(GOut p, unsigned int off)
{
    return (GOut)((__attribute__((address_space(1))) char *)p + off);
}

// The offset, made anew where it is used: its extension to 64 bits is not
// shared between blocks of code, and stays out of the registers.
__device__ __forceinline__ unsigned int local(unsigned int off)
{
    asm volatile("" : "+v"(off));
    return off;
}

// A block of one system: its five diagonals and right-hand side before the
// downward pass; gamma (in a), delta (in b) and g (in f) after it.
struct Block {
    double a[kRows], b[kRows], c[kRows], d[kRows], e[kRows], f[kRows];
};

// What the rows below need of the two above: the carried values of Sec. 2.4.
struct Carry {
    double gm2, gm1, dl2, dl1, g2, g1;
};

constexpr int kBadPivot = 0x267;  // v_cmp_class: a NaN, an infinity or a zero

// Factorisation and forward sweep of the block of rows i0 ..; badrow: the
// first row met so far whose pivot is zero or not finite.
__device__ __forceinline__ void down(Block &q, Carry &s, unsigned int i0, unsigned int &badrow)
{
#pragma unroll
    for (int k = 0; k < kRows; k++) {
        const double beta = fma(-q.a[k], s.gm2, q.b[k]);
        const double alpha = fma(-beta, s.gm1, fma(-q.a[k], s.dl2, q.c[k]));
        const unsigned int row = i0 + k < badrow ? i0 + k : badrow;
        badrow = __builtin_amdgcn_class(alpha, kBadPivot) ? row : badrow;
        const double r = 1.0 / alpha;
        const double gam = fma(-beta, s.dl1, q.d[k]) * r;
        const double del = q.e[k] * r;
        const double g = fma(-beta, s.g1, fma(-q.a[k], s.g2, q.f[k])) * r;
        s.gm2 = s.gm1;
        s.gm1 = gam;
        s.dl2 = s.dl1;
        s.dl1 = del;
        s.g2 = s.g1;
        s.g1 = g;
        q.a[k] = gam;
        q.b[k] = del;
        q.f[k] = g;
    }
}

// A wait of one wave for an earlier block of its own workgroup.  It ends: the
// waves of a workgroup run together, the blocks of a tile (downward, then
// upward) follow one another in one order, and every wave takes its own in
// that order.
__device__ __forceinline__ void wait_for(unsigned int *p, unsigned int v)
{
    for (;;) {
        const unsigned int x = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if ((int)((unsigned int)__builtin_amdgcn_readfirstlane((int)x) - v) >= 0) break;
        __builtin_amdgcn_s_sleep(1);
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// A workgroup takes the tiles blockIdx.x, blockIdx.x + gridDim.x .. in turn,
// the waves in reversed order every other time: the wave that is through with
// one tile first loads the first block of the next.  Two tiles at most are in
// work together, and the carried values and counters are kept twice: the wave
// of block 0 of a tile had block 0 of the last but one, which is the last to
// be finished there.
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_rewrite(
    GIn A_, GIn B_, GIn C_, GIn D_, GIn E_, int64_t ldm, int n, GOut F_, int64_t batch, int64_t ld, GOut W_,
    unsigned long long *__restrict__ bad)
{
    __shared__ double carries[2][6][64];  // the carried values of the last finished block
    __shared__ unsigned int dones[2];     // blocks finished
    __shared__ double held[kWaves][kRows][2][64];  // gamma and delta of a wave's last block but one
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t tiles = (batch + 63) / 64;
    const int nblk = (n + kRows - 1) / kRows;
    if (threadIdx.x < 2) dones[threadIdx.x] = 0;
    __syncthreads();
    Block q;
    unsigned int turn = 0;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x, turn++) {
        const int first = turn & 1 ? kWaves - 1 - w : w;  // this wave's blocks: first, first + kWaves ..
        if (first >= nblk) continue;
        const int mine = (nblk - 1 - first) / kWaves;
        const int64_t j0 = tile * 64;
        const bool active = j0 + lane < batch;
        // lanes past the batch work on the last system again and store nothing
        const unsigned int off = 8u * (unsigned int)(active ? lane : batch - 1 - j0);
        GIn A = A_ + j0, B = B_ + j0, C = C_ + j0, D = D_ + j0, E = E_ + j0;
        GOut F = F_ + j0;
        // gamma and delta of a tile lie together, a row of each in turn (rows
        // as far apart as F's cost 131072 systems 3%)
        const int64_t lw = batch - j0 < 64 ? batch - j0 : 64;
        GOut W = W_ + 2 * (int64_t)n * j0;
        double(&carry)[6][64] = carries[turn & 1];
        unsigned int &done = dones[turn & 1];
        const unsigned int base = (turn >> 1) * 2u * (unsigned int)nblk;  // finished for earlier tiles
        unsigned int badrow = UINT_MAX;
        for (int t = 0; t <= mine; t++) {
            const int b = first + t * kWaves, i0 = b * kRows, last = n - 1 - i0;
            {
                const int64_t om = (int64_t)i0 * ldm;
                const unsigned int lo = local(off);
                GIn pa = A + om, pb = B + om, pc = C + om, pd = D + om, pe = E + om, pf = F + (int64_t)i0 * ld;
#pragma unroll
                for (int k = 0; k < kRows; k++) {
                    q.a[k] = __builtin_nontemporal_load(at(pa, lo));
                    q.b[k] = __builtin_nontemporal_load(at(pb, lo));
                    q.c[k] = __builtin_nontemporal_load(at(pc, lo));
                    q.d[k] = __builtin_nontemporal_load(at(pd, lo));
                    q.e[k] = __builtin_nontemporal_load(at(pe, lo));
                    q.f[k] = *at(pf, lo);
                    // rows past the end: the last one again
                    const int64_t sm = k < last ? ldm : 0, sf = k < last ? ld : 0;
                    pa = fresh(pa + sm);
                    pb = fresh(pb + sm);
                    pc = fresh(pc + sm);
                    pd = fresh(pd + sm);
                    pe = fresh(pe + sm);
                    pf = fresh(pf + sf);
                }
            }
            // entries outside the matrix are ignored (read as zero)
            if (b == 0) q.a[0] = q.b[0] = q.a[1] = 0.0;
            if (last <= kRows) {
#pragma unroll
                for (int k = 0; k < kRows; k++) {
                    if (k + 1 > last) q.d[k] = 0.0;
                    if (k + 2 > last) q.e[k] = 0.0;
                }
            }
            wait_for(&done, base + (unsigned int)b);
            Carry s = {};
            if (b > 0)
                s = {carry[0][lane], carry[1][lane], carry[2][lane], carry[3][lane], carry[4][lane], carry[5][lane]};
            down(q, s, (unsigned int)i0, badrow);
            carry[0][lane] = s.gm2;
            carry[1][lane] = s.gm1;
            carry[2][lane] = s.dl2;
            carry[3][lane] = s.dl1;
            carry[4][lane] = s.g2;
            carry[5][lane] = s.g1;
            st::lds_post(&done, base + (unsigned int)b + 1);
            if (t < mine) {  // the last block stays in the registers, the one before in LDS
                if (t == mine - 1) {
#pragma unroll
                    for (int k = 0; k < kRows; k++) {
                        held[w][k][0][lane] = q.a[k];
                        held[w][k][1][lane] = q.b[k];
                    }
                }
                if (active) {
                    const unsigned int lo = local(off);
                    GOut pf = F + (int64_t)i0 * ld;
#pragma unroll
                    for (int k = 0; k < kRows; k++) {
                        *at(pf, lo) = q.f[k];
                        pf = fresh(pf + ld);
                    }
                    if (t < mine - 1) {
                        GOut pw = W + (int64_t)i0 * 2 * lw;
#pragma unroll
                        for (int k = 0; k < kRows; k++) {
                            __builtin_nontemporal_store(q.a[k], at(pw, lo));
                            pw = fresh(pw + lw);
                            __builtin_nontemporal_store(q.b[k], at(pw, lo));
                            pw = fresh(pw + lw);
                        }
                    }
                }
            } else if (last < kRows - 1) {  // rows past the end
#pragma unroll
                for (int k = 0; k < kRows; k++)
                    if (k > last) q.a[k] = q.b[k] = q.f[k] = 0.0;
            }
        }
        if (active && badrow < (unsigned int)n)  // not one of the rows past the end
            atomicMin(bad, (unsigned long long)(j0 + lane) * (unsigned long long)n + (unsigned long long)badrow);
        // upward: back substitution x_i = g_i - gamma_i x_{i+1} - delta_i x_{i+2}
        for (int t = mine; t >= 0; t--) {
            const int b = first + t * kWaves, i0 = b * kRows, last = n - 1 - i0, after = nblk - 1 - b;
            if (t < mine) {
                const unsigned int lo = local(off);
                GIn pf = F + (int64_t)i0 * ld;
#pragma unroll
                for (int k = 0; k < kRows; k++) {
                    q.f[k] = *at(pf, lo);
                    pf = fresh(pf + ld);
                }
                if (t < mine - 1) {
                    GIn pw = W + (int64_t)i0 * 2 * lw;
#pragma unroll
                    for (int k = 0; k < kRows; k++) {
                        q.a[k] = __builtin_nontemporal_load(at(pw, lo));
                        pw = fresh(pw + lw);
                        q.b[k] = __builtin_nontemporal_load(at(pw, lo));
                        pw = fresh(pw + lw);
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < kRows; k++) {
                        q.a[k] = held[w][k][0][lane];
                        q.b[k] = held[w][k][1][lane];
                    }
                }
            }
            const unsigned int up = base + (unsigned int)(nblk + after);
            wait_for(&done, up);
            double x1 = 0.0, x2 = 0.0;
            if (after > 0) {
                x1 = carry[0][lane];
                x2 = carry[1][lane];
            }
#pragma unroll
            for (int k = kRows - 1; k >= 0; k--) {
                const double x = fma(-q.b[k], x2, fma(-q.a[k], x1, q.f[k]));
                q.f[k] = x;
                x2 = x1;
                x1 = x;
            }
            carry[0][lane] = x1;
            carry[1][lane] = x2;
            st::lds_post(&done, up + 1);
            if (active) {
                const unsigned int lo = local(off);
                GOut pf = F + (int64_t)i0 * ld;
#pragma unroll
                for (int k = 0; k < kRows; k++) {
                    if (k <= last) *at(pf, lo) = q.f[k];
                    pf = fresh(pf + ld);
                }
            }
        }
    }
}

__global__ void k_rewrite_init(unsigned long long *bad)
{
    if (threadIdx.x == 0) *bad = ~0ull;
}

}  // namespace

size_t rewrite_workspace_bytes(int64_t n, int64_t batch)
{
    return 256 + sizeof(double) * 2 * (size_t)n * (size_t)batch;
}

hipError_t launch_rewrite(const double *a, const double *b, const double *c, const double *d,
                          const double *e, int64_t ldm, int64_t n, double *F, int64_t batch,
                          int64_t ld, void *work, hipStream_t s)
{
    unsigned long long *bad = (unsigned long long *)work;
    double *G = (double *)((char *)work + 256);
    hipLaunchKernelGGL(k_rewrite_init, dim3(1), dim3(64), 0, s, bad);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    // one workgroup per compute unit: its waves take all the registers
    // (n = 1024, us, one lane per system in workgroups of four waves / this
    // without the blocks in LDS / now: 500 systems 604 / 136 / 132, 16384 687 / 245 /
    // 237, 65536 1178 / 1132 / 1096, 131072 2659 / 2277 / 2180, 5.9 TB/s; n = 8192 x
    // 2000 4671 / 1072 / 1062, n = 203 x 131072 450 / 338 / 290, n = 64 x 100000 115 / 77 /
    // 77)
    int dev = 0, cus = 0;
    if ((err = hipGetDevice(&dev)) != hipSuccess) return err;
    if ((err = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return err;
    const int64_t tiles = (batch + 63) / 64;
    hipLaunchKernelGGL(k_rewrite, dim3((unsigned)(tiles < cus ? tiles : cus)), dim3(64 * kWaves), 0, s, (GIn)a,
                       (GIn)b, (GIn)c, (GIn)d, (GIn)e, ldm, (int)n, (GOut)F, batch, ld, (GOut)G, bad);
    return hipGetLastError();
}

}  // namespace pent
