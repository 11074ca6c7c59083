// Resident PCG iteration on wavefront strips, for gfx950, FP64: Table 1 with ASSOR II of Neumann
// order 1 (Eq 3.4-3.6) or Jacobi (Eq 2.8), the whole iteration loop in one launch, for joint
// systems whose vectors fit the registers and LDS of the chip.
//
// What bounds small and middle grids with one launch per iteration is not the arithmetic: each
// launch pays its start, a chain of dependent loads of the request record, the partial sums of
// the previous launch read back from memory, and a row march whose first loads miss every cache,
// about 20 us per iteration whatever the grid.  Here every wavefront keeps one tile (a strip of
// ring columns x a chunk of rows) for the whole solve: r, p, 1/D and, up to 24 rows, the
// conductances in registers, z and u in LDS.  An iteration is
//   1. the sums of the previous pass, exchanged by every workgroup (below), and alpha and beta;
//   2. the halo of z: two rows below the tile, three above, four columns on either side;
//   3. one march over the rows of the tile: u = z + beta u, A u, r = r - alpha A u, both ASSOR
//      sweeps, z, p = p + alpha u, and the five sums of the scheme of gap_pcgw.hpp;
//   4. the boundary cells of z written for the neighbours, and the tile's sums.
// Only z crosses tiles.  The halo of u follows from it (u is formed cell by cell), and r on the
// halo follows from u: every tile carries its own copy of both, computed with the same operations
// on the same values, so the copies agree to the bit.
//
// Exchange between workgroups.  Stores and loads of exchanged values are relaxed agent-scope
// accesses (they go past the L2 of the XCD), in buffers that nothing else touches during the
// launch.  A sum travels as two 8-byte words, each a half of the double beside the number of its
// pass, so a reader knows by the word itself that it is the one it waits for; no flag, no counter.
// A workgroup publishes its sums only after its boundary stores of z have been acknowledged, so a
// reader that has seen the sums of a neighbour may read its halo.  Words and z alternate
// between two buffers by pass parity: a workgroup writes pass e + 2 only after it has seen the
// sums of pass e + 1 of all others, which they publish after reading pass e.  Every workgroup adds
// the sums in the same order, so all derive the same alpha, beta and stopping decision to the bit.
// A condition that the sums of pass e freeze is waited for once more: each of its workgroups publishes empty words of
// pass e + 1 when it has seen all of pass e, or a late one would find pass e overwritten by the others' pass e + 2.
// The words of one value lie side by side over the workgroups (a look at 64 of them touches 8 cache
// lines, not 64: 9 % of an iteration of 128 x 64 x 9), and a wavefront first waits for the one
// word of each neighbour: looking at all words from the start fills the fabric and costs 9 % as well.
//
// Every wait is bounded by the clock: a workgroup that waits longer than wait_ticks sets the
// abort word and leaves, all others follow, and the host solves again with the strip kernel.
// The launch is cooperative, so all workgroups are resident.
//
// Measured per iteration of whole solves, launches of k_pcg_w and this kernel: 64 x 32 x 1 15.8 and 4.2 us, 128 x 64 x 9
// 16.6 and 4.1, 256 x 128 x 9 17.0 and 4.8, 512 x 256 x 9 21.9 and 8.4, 400 x 360 x 9 23.0 and 9.1.
// Clocks of one wavefront around the parts of a pass (a build with clock reads, 2.36 GHz), 128 x 64 x 9 and 512 x 256 x 9,
// us: wait for the neighbours' word 0.9 and 1.2 (one store to one load across the fabric takes 0.9 at
// least), all words 0.6 and 0.9, sums over lanes 0.5 and 0.7, alpha and beta 0.6 (two dependent divisions), halo 0.2 and
// 0.3, the march over 4 and 24 rows 0.8 and 3.5 (62 instructions a row, issued one each 4 cycles: FP64
// rate), boundary cells 0.2 and 0.7, this workgroup's sums and the acknowledgement of its stores 0.5 and 0.7.
#pragma once

#include <type_traits>

#include "gap_pcgw.hpp"

constexpr int kLoopWaves = 4;                        // tiles (wavefronts) per workgroup, one per SIMD
constexpr int kLoopThreads = 64 * kLoopWaves;
constexpr int kLoopHalo = 4;                         // halo columns of z on either side of a strip
// Columns of a tile row kept in LDS; lanes that hold none share one more.
constexpr int kLoopCols = 64 - 2 * (strip_halo(1) - kLoopHalo);
constexpr int kLoopWidth = kLoopCols + 1;
constexpr int kLoopWords = 2 * 6 * 2 * kLoopThreads;    // words of the exchange: two passes, six values, two halves
constexpr int kLoopSlotsAll = kLoopThreads;          // slots (workgroups) in all, at most: one a thread
constexpr double kLoopClock = 1e8;                   // ticks of the wall clock per second
constexpr double kLoopWait = 2.0;                    // seconds a workgroup waits at most, unless the caller sets it

// Where a tile of R rows keeps what it reads every iteration.  r, p and 1/D always stay in registers, u and
// the conductances where they fit beside them (a SIMD holds one wavefront: 512 registers a lane), z
// always in LDS, from which its boundary cells are read by other lanes than those that form them.
__host__ __device__ constexpr bool loop_u_regs(int R) { return R <= 8; }
__host__ __device__ constexpr bool loop_k_regs(int R) { return R <= 24; }
__host__ __device__ constexpr int loop_tile_rows(int R) { return R + (loop_u_regs(R) ? 0 : R + 5); }
__host__ __device__ constexpr size_t loop_tile_bytes(int R) { return (size_t)loop_tile_rows(R) * kLoopWidth * sizeof(double); }
// The tile heights built.
#define GAP_LOOP_ROWS(X) X(4) X(6) X(8) X(10) X(12) X(14) X(16) X(20) X(24) X(28) X(32)

// What one launch leaves for the next, by launch parity.
struct LoopState {
    int iter, done, act, pad;
    double rz, ss, ss_c[GAP_MAXC];                   // r.z of the pass before, ||S||^2 in all and by condition
    double sums[6 * GAP_MAXC];                       // asynchronized: six values a condition, of the pass before
};

struct LoopDev {
    LoopState* state;                                // [2]
    unsigned long long* words;                       // [2][6 values][kLoopSlotsAll][2 halves]
    int* abort_word;
    long long wait_ticks;
    int slots;                                       // workgroups per condition
    int strips, chunks;                              // tiles per ring and along the axis
};

typedef unsigned long long loop_word;

__device__ __forceinline__ void loop_store(loop_word* p, loop_word v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ loop_word loop_load(const loop_word* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void loop_store_d(GAP_AS1 double* p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double loop_load_d(const GAP_AS1 double* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Orders the LDS accesses of one wavefront, which may come from different lanes.
__device__ __forceinline__ void loop_wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Half h of x beside the pass number.
__device__ __forceinline__ loop_word loop_pack(double x, int h, unsigned pass)
{
    const loop_word b = (loop_word)__double_as_longlong(x);
    return ((loop_word)pass << 32) | (h ? (b >> 32) : (b & 0xffffffffull));
}
__device__ __forceinline__ double loop_unpack(loop_word lo, loop_word hi)
{
    return __longlong_as_double((long long)((hi << 32) | (lo & 0xffffffffull)));
}

// Whether a wait that has looked in vain `spin` times before this one is given up (a limit of 0: at the first look).
__device__ __forceinline__ bool loop_give_up(int spin, long long t0, const LoopDev& lp)
{
    return ((spin & 63) == 63 || lp.wait_ticks == 0) &&
           (wall_clock64() - t0 >= lp.wait_ticks || __hip_atomic_load(lp.abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Waits until the six pairs of words at p, p + stride, ... of every lane with `on` carry the pass number (each
// word does, so a load of two need not be atomic), and gives their values (0 elsewhere).  False if the
// wait was given up.
__device__ __forceinline__ bool loop_wait_slots(const loop_word* p, size_t stride, bool on, unsigned pass, double (&v)[6], const LoopDev& lp)
{
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    v4u x0 = {0, 0, 0, 0}, x1 = x0, x2 = x0, x3 = x0, x4 = x0, x5 = x0;
    const loop_word *p1 = p + stride, *p2 = p1 + stride, *p3 = p2 + stride, *p4 = p3 + stride, *p5 = p4 + stride;
    const long long t0 = wall_clock64();
    bool given = false;
    for (int spin = 0;; ++spin) {
        bool ok = true;
        if (on) {
            asm volatile(
                "global_load_dwordx4 %0, %6, off sc1\n\t"
                "global_load_dwordx4 %1, %7, off sc1\n\t"
                "global_load_dwordx4 %2, %8, off sc1\n\t"
                "global_load_dwordx4 %3, %9, off sc1\n\t"
                "global_load_dwordx4 %4, %10, off sc1\n\t"
                "global_load_dwordx4 %5, %11, off sc1\n\t"
                "s_waitcnt vmcnt(0)"
                : "=&v"(x0), "=&v"(x1), "=&v"(x2), "=&v"(x3), "=&v"(x4), "=&v"(x5)
                : "v"(p), "v"(p1), "v"(p2), "v"(p3), "v"(p4), "v"(p5)
                : "memory");
            auto here = [&](v4u x) { return x.y == pass && x.w == pass; };
            ok = here(x0) && here(x1) && here(x2) && here(x3) && here(x4) && here(x5);
        }
        if (__all(ok)) break;
        given = loop_give_up(spin, t0, lp);
        if (given) break;
    }
    auto value = [](v4u x) { return __longlong_as_double((long long)(((loop_word)x.z << 32) | x.x)); };
    v[0] = value(x0);
    v[1] = value(x1);
    v[2] = value(x2);
    v[3] = value(x3);
    v[4] = value(x4);
    v[5] = value(x5);
    return !given;
}
// Waits until the word at p of every lane with `on` carries the pass number.
__device__ __forceinline__ bool loop_wait_word(const loop_word* p, bool on, unsigned pass, const LoopDev& lp)
{
    const long long t0 = wall_clock64();
    for (int spin = 0;; ++spin) {
        if (__all(!on || (unsigned)(loop_load(p) >> 32) == pass)) return true;
        if (loop_give_up(spin, t0, lp)) return false;
    }
}

// fn(integral_constant<int, I>) for I = A .. B - 1.
template <int A, int B, class Fn>
__device__ __forceinline__ void static_for(Fn&& fn)
{
    if constexpr (A < B) {
        fn(std::integral_constant<int, A>{});
        static_for<A + 1, B>(fn);
    }
}

// One 32-bit half of each lane's value exchanged by DPP; both halves of a double.
template <int CTRL>
__device__ __forceinline__ double dpp_perm(double x)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b & 0xffffffffull), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
// Sums over lanes whose numbers differ in the named bits, in every one of them.  Each step adds pairs
// that hold each other's partner, so all lanes get the same bits.
__device__ __forceinline__ double lane_sum_2(double x) { return x + dpp_perm<0x4E>(x); }      // quad_perm 2,3,0,1
__device__ __forceinline__ double quad_sum(double x)         // the four quads of a row of 16: row_ror:8, row_ror:4
{
    x += dpp_perm<0x128>(x);
    return x + dpp_perm<0x124>(x);
}
__device__ __forceinline__ double lane_sum_16_32(double x)
{
    x += __shfl_xor(x, 16, 64);
    return x + __shfl_xor(x, 32, 64);
}

// PK: the preconditioner, 0 Jacobi or 2 ASSOR II.  R: rows of a tile.  init: start a solve with the pass that
// forms r_0 and z_0.  n_pass: iterations at most in this launch, 2 or more.  base:
// number of the pass before the solve's first.
template <int PK, int R>
__global__ __launch_bounds__(kLoopThreads, 1) void k_pcg_p(const PcgDev* __restrict__ reqs, LoopDev lp,
                                                          const int* __restrict__ work, int init, int n_pass, int par,
                                                          unsigned base)
{
    extern __shared__ double lds_all[];
    __shared__ double wsum[kLoopWaves][6];
    __shared__ double stage[kLoopSlotsAll][6];       // the sums of every workgroup
    __shared__ double tot[2][kLoopWaves][6];         // totals of a wavefront's slots, by pass parity
    __shared__ double sums[2][6 * GAP_MAXC];         // asynchronized: six values a condition, by pass parity
    __shared__ int gave_up;

    int req, c, kc;
    if (!pcg_work(work, blockIdx.x, req, c, kc)) return;
    const PcgDev& a = reqs[req];
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const LoopState* st_in = lp.state + par;
    LoopState* st_out = lp.state + (par ^ 1);
    const int n_cond = a.n_cond, max_iter = a.max_iter, async = a.async, warm = a.warm;
    const double eps = a.eps;
    const double eps_mine = a.eps_c[lane < n_cond ? lane : 0];
    double* const hist = a.hist;
    const int hist_cap = a.hist_cap;
    PcgScalars* const sc = a.sc;
    int j = 0;
    unsigned act = (1u << n_cond) - 1u;
    double rz_prev = 0.0, ss_all = 0.0, ss_mine = 0.0;
    if (!init) {
        if (__builtin_amdgcn_readfirstlane(st_in->done)) {
            if (c == 0 && kc == 0 && t == 0) st_out->done = 1;
            return;
        }
        j = __builtin_amdgcn_readfirstlane(st_in->iter);
        act = (unsigned)__builtin_amdgcn_readfirstlane(st_in->act) & 0xffffu;
        if (!((act >> c) & 1)) return;               // frozen in an earlier launch
        rz_prev = st_in->rz;
        ss_all = st_in->ss;
        ss_mine = st_in->ss_c[lane < n_cond ? lane : 0];
        if (async && lane < 6 * GAP_MAXC) sums[(base + (unsigned)j) & 1][lane] = st_in->sums[lane];
    }
    if (t == 0) gave_up = 0;

    // ---- the tile of this wavefront ---------------------------------------------------------
    constexpr int H = strip_halo(1), HS = H - kLoopHalo;
    constexpr int W = kLoopWidth;
    constexpr bool UREG = loop_u_regs(R), KREG = loop_k_regs(R);
    const int nt = a.nt, nz = a.nz;
    const int tile = kc * kLoopWaves + wv;
    const bool has_tile = tile < lp.strips * lp.chunks;
    const int chunk = tile / lp.strips, strip = tile - chunk * lp.strips;
    // Rows j0 .. j0 + R - 1; those past the grid (last chunk) hold zeros and 1/D = 0, like the halo rows
    // outside it, which zeroes every term they would feed.
    const int j0 = chunk * R, rows = has_tile ? min(R, nz - j0) : 0;
    const int oc0 = (int)(((long long)strip * nt) / lp.strips), oc1 = (int)(((long long)(strip + 1) * nt) / lp.strips);
    const int wid = oc1 - oc0;
    auto ring_col = [&](int m) {                     // ring column of strip column m
        int g = (oc0 - H + m) % nt;
        return g < 0 ? g + nt : g;
    };
    const int gcol = ring_col(lane);
    const bool own = has_tile && lane >= H && lane < H + wid;
    const bool live = lane >= HS && lane < H + wid + kLoopHalo;
    double* zt = lds_all + (size_t)wv * loop_tile_rows(R) * W;   // rows 0 .. R - 1 of the tile
    double* zl = zt + (live ? lane - HS : kLoopCols);            // this lane's column of it
    double* ul = zl + R * W;                                     // rows -2 .. R + 2 of u, unless in registers
    // halo and edge columns of the strip, eight rows a load or store
    const int hr = lane >> 3, hc = lane & 7;
    const int hm = hc < 4 ? HS + hc : H + wid + hc - 4;          // halo: four columns on either side
    const int em = hc < 4 ? H + hc : H + wid - 8 + hc;           // edge: the four outermost owned ones
    const bool e_on = has_tile && em >= H && em < H + wid;
    const unsigned hg = (unsigned)ring_col(hm), eg = (unsigned)ring_col(e_on ? em : H);
    const size_t n = (size_t)nt * nz, co = (size_t)c * n;
    const int op = a.op[c];
    const GAP_AS1 double* kxz = as_global(a.kxz + (size_t)op * 2 * (n + nt));
    GAP_AS1 double* const pp = as_global(a.p + co);
    GAP_AS1 double* const z0 = as_global(a.zf[0] + co);
    GAP_AS1 double* const z1 = as_global(a.zf[1] + co);
    // lanes 0 .. 8: the slot of one of the tiles around, whose z this one reads
    const int dr = lane / 3 - 1, ds = lane % 3 - 1;
    const bool near_on = lane < 9 && chunk + dr >= 0 && chunk + dr < lp.chunks;
    const int nstrip = strip + ds < 0 ? lp.strips - 1 : (strip + ds >= lp.strips ? 0 : strip + ds);
    const int near_slot = c * lp.slots + (near_on ? ((chunk + dr) * lp.strips + nstrip) / kLoopWaves : kc);
    const int n_slots = n_cond * lp.slots;
    constexpr size_t pair_stride = 2 * kLoopSlotsAll;   // words between the pairs of one slot
    const int slot_cond = t / lp.slots;              // the condition of slot t
    auto zbuf = [&](int q) { return (q & 1) ? z1 : z0; };
    double zh[5];                                    // z on the halo rows -2, -1, R, R + 1, R + 2
    double zb[5];                                    // z' on the rows 0, 1, 2, R - 2, R - 1, for the neighbours
    double ss0;                                      // ||S||^2 of this lane's cells (first pass)
    double rr_[R + 3];                               // r on rows -1 .. R + 1
    double pr[R];                                    // p on rows 0 .. R - 1
    double ur[UREG ? R + 5 : 1];                     // u on rows -2 .. R + 2
    double DI[R + 3];                                // 1/D on rows -1 .. R + 1
    double KXr[KREG ? R + 4 : 1], Fr[KREG ? R + 4 : 1];   // east faces and the axial faces above, rows -2 .. R + 1

    // pair of conductances of row i of the tile: east faces and the faces above; rows outside the grid
    // repeat a row of it
    auto load_k = [&](int jt, int i, double& kx, double& f) {
        const GAP_AS1 double* row = kxz + 2 * (size_t)((unsigned)min(max(jt + i + 1, 0), nz) * (unsigned)nt);
        kx = row[2 * (unsigned)gcol];
        f = row[2 * (unsigned)gcol + 1];
    };
    // j0 hidden from the compiler, which would otherwise keep every row's address across the iterations
    auto tile_row = [&]() {
        int q = j0;
        asm volatile("" : "+s"(q));
        return q;
    };
    auto west = [](double x) { return dpp_shift0<0x138>(x); };
    auto east = [](double x) { return dpp_shift0<0x130>(x); };
    // ---- state of the launch before (r and u in the buffers 0: no launch ends before all its workgroups have read
    // theirs, and the buffers 1 keep the initial guess for the host), or the start: z = p_0, u = 0, r = S, so that the first pass
    // with alpha = 1 and beta = 0 forms r_0 = S - A p_0 and z_0
    {
        const GAP_AS1 double* rs = as_global((init ? a.S : a.r[0]) + co);
        const GAP_AS1 double* us = as_global(a.u[0] + co);
        const GAP_AS1 double* zs = init ? (const GAP_AS1 double*)pp : zbuf(j);
        const bool zz = !init || warm;
        double fs = 0.0;                             // face below
        ss0 = 0.0;
#pragma unroll
        for (int i = -2; i < R + 3; ++i) {
            const int s = j0 + i;
            const bool in = has_tile && live && s >= 0 && s < nz;
            const unsigned g = (unsigned)s * nt + gcol;
            const double zv = (in && zz) ? loop_load_d(zs + g) : 0.0;
            const double uv = (in && !init) ? us[g] : 0.0;
            if (i < 0) zh[i + 2] = zv;
            else if (i >= R) zh[i - R + 2] = zv;
            else zl[i * W] = zv;
            if (UREG) ur[UREG ? i + 2 : 0] = uv;
            else ul[(i + 2) * W] = uv;
            if (i >= -1 && i < R + 2) rr_[i + 1] = in ? rs[g] : 0.0;
            if (i >= 0 && i < R) ss0 += rr_[i + 1] * rr_[i + 1];
            if (i >= 0 && i < R) pr[i >= 0 && i < R ? i : 0] = (own && i < rows && zz) ? pp[g] : 0.0;
            if (i < R + 2) {
                double kx, f;
                load_k(j0, i, kx, f);
                if (i >= -1) {
                    const double D = ((kx + west(kx)) + fs) + f;
                    DI[i + 1] = (has_tile && s >= 0 && s < nz) ? 1.0 / D : 0.0;
                }
                if (KREG) {
                    KXr[KREG ? i + 2 : 0] = kx;
                    Fr[KREG ? i + 2 : 0] = f;
                }
                fs = f;
            }
            if (i % 4 == 0) __builtin_amdgcn_sched_barrier(0);   // a few rows in flight, not all
        }
    }
    __syncthreads();

    // ---- one pass over the tile -------------------------------------------------------------
    const double omega = a.omega, scale = omega * (2.0 - omega);
    // couplings of the sweeps across the periodic seam: west of column 0 is in L^T, east of the last
    // column in L (Eq 3.5, 3.6)
    const double w_l = gcol > 0 ? 1.0 : 0.0, w_lt = gcol == 0 ? 1.0 : 0.0;
    const double e_l = gcol == nt - 1 ? 1.0 : 0.0, e_lt = gcol < nt - 1 ? 1.0 : 0.0;
    const double inlet = j0 == 0 ? 1.0 : 0.0;        // the face below row 0 belongs to the tile below, if there is one
    double acc[5];
    // Step s: u on row s; A u, r and D^-1 r on row s - LA; the first sweep on row s - LC; the second sweep, z and
    // the faces of z^T A z on row s - LD.  The lags are one row longer than the data needs, so the
    // stages of one step depend on earlier steps only and a SIMD with a single wavefront has
    // independent work to issue.  The rows are unrolled: no branch, every value in its register.
    constexpr int LA = 2, LC = 3, LD = PK == 2 ? 5 : 3;
    constexpr int AH = KREG ? 2 : 8;                            // conductances are loaded AH rows ahead of u
    constexpr int P = LD + AH + 2;                   // slots of the register rings: rows s + AH .. s - LD - 1
    auto pass = [&](double alpha, double beta, bool first) {
        double KX[P], F[P], KW[P], U[P], RQ[P], AU[P], Y[P], V[P];
#pragma unroll
        for (int d = 0; d < P; ++d) KX[d] = F[d] = KW[d] = U[d] = RQ[d] = AU[d] = Y[d] = V[d] = 0.0;
#pragma unroll
        for (int q = 0; q < 5; ++q) acc[q] = 0.0;
        double zbelow = 0.0;
        const double al_p = first ? 0.0 : alpha;     // the first pass forms r_0 from p_0
        // hidden likewise: products with every row's 1/D and conductances
        double om = omega, w_in_l = w_l, w_in_lt = w_lt, e_in_l = e_l, e_in_lt = e_lt;
        const int jt = tile_row();
        asm volatile("" : "+v"(om), "+v"(w_in_l), "+v"(w_in_lt), "+v"(e_in_l), "+v"(e_in_lt));
        auto slot = [](int row) constexpr { return ((row % P) + P) % P; };
        auto kload = [&](auto Ic) {
            constexpr int i = decltype(Ic)::value;
            if constexpr (i >= -2 && i <= R + 1) {
                if constexpr (KREG) {
                    KX[slot(i)] = KXr[i + 2];
                    F[slot(i)] = Fr[i + 2];
                } else {
                    load_k(jt, i, KX[slot(i)], F[slot(i)]);
                }
            }
        };
        double zv, uv;
        auto fetch = [&](auto Ic) {
            constexpr int i = decltype(Ic)::value;
            if constexpr (i < 0) zv = zh[i + 2];
            else if constexpr (i >= R) zv = zh[i - R + 2];
            else zv = zl[i * W];
            if constexpr (UREG) uv = ur[i + 2];
            else uv = ul[(i + 2) * W];
        };
        static_for<-2, -2 + AH>(kload);
        fetch(std::integral_constant<int, -2>{});
        static_for<-2, R + LD + 1>([&](auto Sc) {
            constexpr int s = decltype(Sc)::value;
            constexpr int ra = s - LA, rc = s - LC, rd = s - LD;
            kload(std::integral_constant<int, s + AH>{});
            const double zn = zv, un_ = uv;          // z and u of row s, read from LDS in the step before
            if constexpr (s + 1 <= R + 2) fetch(std::integral_constant<int, s + 1>{});
            if constexpr (rd >= 0) {                 // rows 0 .. R
                double z;
                if constexpr (PK == 2) {
                    double hi = F[slot(rd)] * V[slot(rd + 1)];
                    hi += (KX[slot(rd)] * e_in_lt) * east(V[slot(rd)]);
                    hi += (KW[slot(rd)] * w_in_lt) * west(V[slot(rd)]);
                    z = scale * (V[slot(rd)] + om * DI[rd + 1] * hi);
                } else {
                    z = Y[slot(rd)];
                }
                const double db = zbelow - z;        // the face below: an end face where z is zero beyond it
                if constexpr (rd == 0) acc[2] += inlet * (F[slot(rd - 1)] * db * db);
                else acc[2] += F[slot(rd - 1)] * db * db;
                if constexpr (rd < R) {
                    zl[rd * W] = z;
                    if constexpr (rd < 3) zb[rd] = z;
                    if constexpr (rd >= R - 2) zb[rd - R + 5] = z;
                    const double de = z - east(z);
                    acc[2] += KX[slot(rd)] * de * de;
                    acc[0] += RQ[slot(rd)] * z;
                    acc[3] += z * AU[slot(rd)];
                }
                zbelow = z;
            }
            if constexpr (PK == 2 && rc >= 0 && rc <= R + 1) {
                double lo = (KW[slot(rc)] * w_in_l) * west(Y[slot(rc)]);
                lo += (KX[slot(rc)] * e_in_l) * east(Y[slot(rc)]);
                lo += F[slot(rc - 1)] * Y[slot(rc - 1)];
                V[slot(rc)] = Y[slot(rc)] + om * DI[rc + 1] * lo;
            }
            if constexpr (ra >= -1 && ra <= R + 1) {
                const double u = U[slot(ra)];
                const double kx = KX[slot(ra)], kw = west(kx), fs = F[slot(ra - 1)], fn = F[slot(ra)];
                const double D = ((kx + kw) + fs) + fn;
                double v = D * u - kx * east(u) - kw * west(u);
                v -= fs * U[slot(ra - 1)];
                v -= fn * U[slot(ra + 1)];
                const double ro = rr_[ra + 1];
                const double al = (ra < 0 ? jt > 0 : jt + ra < nz) ? alpha : 0.0;   // rows outside the grid stay zero
                const double rn = ro - al * v;
                KW[slot(ra)] = kw;
                AU[slot(ra)] = v;
                RQ[slot(ra)] = rn;
                rr_[ra + 1] = rn;
                Y[slot(ra)] = rn * DI[ra + 1];
                if constexpr (ra >= 0 && ra < R) {
                    acc[1] += rn * rn;
                    acc[4] += u * v;
                }
            }
            if constexpr (s <= R + 2) {
                const double un = zn + beta * un_;
                if constexpr (UREG) ur[s + 2] = un;
                else ul[(s + 2) * W] = un;
                U[slot(s)] = un;
                if constexpr (s >= 0 && s < R) pr[s] += al_p * un;
            }
            __builtin_amdgcn_sched_barrier(0);       // loads stay in the step that issues them
        });
        // the sums are formed here (not where they are used, with every row's terms kept until then), and z
        // and u are read back from LDS, not kept beside it
        asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4])::"memory");
    };

    // the halo of z after a pass, from the buffer of iteration parity q: rows into registers, columns
    // into LDS once they are here
    constexpr int HN = (R + 7) / 8;
    double hv[HN];
    auto halo_load = [&](int q) {
        const GAP_AS1 double* zs = zbuf(q);
        const unsigned lc = live ? (unsigned)gcol : 0u;
        const int jt = tile_row();
#pragma unroll
        for (int k = 0; k < HN; ++k) hv[k] = loop_load_d(zs + (unsigned)(jt + min(8 * k + hr, rows - 1)) * nt + hg);
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const int s = jt + (k < 2 ? k - 2 : R + k - 2);
            zh[k] = loop_load_d(zs + (size_t)min(max(s, 0), nz - 1) * nt + lc);
        }
    };
    auto halo_keep = [&]() {
        const int jt = tile_row();
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const int s = jt + (k < 2 ? k - 2 : R + k - 2);
            zh[k] = (s >= 0 && s < nz) ? zh[k] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < HN; ++k)
            if (8 * k + hr < rows) zt[(8 * k + hr) * W + hm - HS] = hv[k];
        loop_wave_fence();
    };
    // the boundary cells of z for the neighbours, into the buffer of iteration parity q: the rows
    // within three of the tile below and two of the one above, the edge columns of the others
    auto publish_z = [&](int q) {
        GAP_AS1 double* zd = zbuf(q);
        const int jt = tile_row();
        loop_wave_fence();
        if (own) {
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                const int r = k < 3 ? k : R + k - 5;
                if ((k < 3 || r > 2) && r < rows) loop_store_d(zd + (size_t)(jt + r) * nt + (unsigned)gcol, zb[k]);
            }
        }
#pragma unroll
        for (int r0 = 3; r0 < R - 2; r0 += 8) {
            const int r = r0 + hr;
            if (e_on && r < min(rows, R - 2)) loop_store_d(zd + (unsigned)(jt + r) * nt + eg, zt[r * W + em - HS]);
        }
    };
    // Sums of six values over the lanes of a wavefront: value q in lane q (q < 4) of v, value 4 + q in lane q
    // (q < 2) of w.  Two rounds of halving leave lane l the sum of value l & 3 (and 4 + (l & 1)) over its quad.
    auto wave_sums = [&](const double (&x)[6], double& v, double& w) {
        const bool b0 = lane & 1, b1 = lane & 2;
        double p = b0 ? x[1] : x[0], q = b0 ? x[3] : x[2];
        w = b0 ? x[5] : x[4];
        p += dpp_perm<0xB1>(b0 ? x[0] : x[1]);
        q += dpp_perm<0xB1>(b0 ? x[2] : x[3]);
        w += dpp_perm<0xB1>(b0 ? x[4] : x[5]);
        v = b1 ? q : p;
        v += dpp_perm<0x4E>(b1 ? p : q);
        w += dpp_perm<0x4E>(w);
        v = lane_sum_16_32(quad_sum(v));
        w = lane_sum_16_32(quad_sum(w));
    };
    // word t & 1 of this workgroup's value t >> 1 of a pass, threads 0 .. 11
    auto put_word = [&](unsigned pass_no, double v) {
        loop_store(lp.words + ((size_t)(pass_no & 1) * 6 + (t >> 1)) * pair_stride + 2 * (c * lp.slots + kc) + (t & 1),
                   loop_pack(v, t & 1, pass_no));
    };
    // sums of this workgroup's pass: lanes of each wavefront, then the wavefronts in order
    auto publish_sums = [&](unsigned pass_no, bool first) {
        double x[6], v, w;
#pragma unroll
        for (int q = 0; q < 5; ++q) x[q] = own ? acc[q] : 0.0;
        x[5] = own && first ? ss0 : 0.0;
        wave_sums(x, v, w);
        if (lane < 4) wsum[wv][lane] = v;
        if (lane < 2) wsum[wv][4 + lane] = w;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the stores of z have been acknowledged
        __syncthreads();
        if (t < 12) {
            double s = wsum[0][t >> 1];
            for (int k = 1; k < kLoopWaves; ++k) s += wsum[k][t >> 1];
            put_word(pass_no, s);
        }
    };
    auto save_p = [&]() {
        if (!own) return;
        const int jt = tile_row();
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (i < rows) pp[(size_t)(jt + i) * nt + (unsigned)gcol] = pr[i];
    };

    // the state of the tile for the next launch, which starts with iteration q
    auto save = [&](int q) {
        save_p();
        if (!own) return;
        GAP_AS1 double* rd = as_global(a.r[0] + co);
        GAP_AS1 double* ud = as_global(a.u[0] + co);
        GAP_AS1 double* zd = zbuf(q);
        const int jt = tile_row();
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (i < rows) {
                const size_t g = (size_t)(jt + i) * nt + (unsigned)gcol;
                rd[g] = rr_[i + 1];
                ud[g] = UREG ? ur[UREG ? i + 2 : 0] : ul[(i + 2) * W];
                loop_store_d(zd + g, zl[i * W]);
            }
    };
    // ---- iterations ---------------------------------------------------------------------------
    const int n_pass_all = n_pass + (init ? 1 : 0);  // passes at most in this launch
    bool first = init != 0;                          // the next pass forms r_0
    // in the upper half of act: the conditions whose workgroups publish the next pass (a register of its own that
    // lives through the passes costs 2 %: 251 x 97 x 9 5.08 us a pass against 4.98)
    static_assert(GAP_MAXC <= 16, "two masks of conditions in a word");
    act |= act << 16;
    for (int it = 0;; ++it) {
        double alpha = 1.0, beta = 0.0;
        if (!first) {
            const unsigned pass_no = base + (unsigned)j + 1u;   // the pass whose sums are needed
            const int pb = pass_no & 1;
            // The halo as soon as the neighbours have published the pass (a light wait, which leaves the memory to
            // the last stores), then the slots of all conditions, one a lane (those frozen before the last
            // pass are not waited for).  State in memory is complete at the start of a launch: no halo is
            // needed before its first pass.
            const bool need_halo = it > 0 && has_tile;
            const bool on = t < n_slots && ((act >> (16 + slot_cond)) & 1);
            const loop_word* words = lp.words + (size_t)pb * 6 * pair_stride;
            unsigned my_word = 2 * (on ? t : 0);
            asm volatile("" : "+v"(my_word));        // as j0: no addresses kept across the iterations
            double x[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            bool ok = true;
            if (need_halo) {
                ok = loop_wait_word(words + 2 * near_slot, near_on, pass_no, lp);
                if (ok) halo_load(j);
            }
            if (ok && wv * 64 < n_slots) ok = loop_wait_slots(words + my_word, pair_stride, on, pass_no, x, lp);
            if (!ok && lane == 0) gave_up = 1;

            // ---- scalars (as in the strip kernel), by every wavefront alike ----------------------
            unsigned active = act;
            bool bad_ab, all_done = false;
            double rr, ss;
            if (!async) {
                // totals over the conditions: lanes of each wavefront, then the wavefronts
                double v, w;
                wave_sums(x, v, w);
                if (lane < 4) tot[pb][wv][lane] = v;
                if (lane < 2) tot[pb][wv][4 + lane] = w;
                __syncthreads();
                double s6[6];
#pragma unroll
                for (int q = 0; q < 6; ++q) s6[q] = (tot[pb][0][q] + tot[pb][1][q]) + (tot[pb][2][q] + tot[pb][3][q]);
                rr = s6[1];
                if (j == 0) ss_all = s6[5];
                ss = ss_all;
                beta = j > 0 ? s6[0] / rz_prev : 0.0;
                alpha = s6[0] / (j > 0 ? s6[2] + 2.0 * beta * s6[3] + beta * beta * s6[4] : s6[2]);
                bad_ab = !finite_d(beta) || !finite_d(alpha);
                rz_prev = s6[0];
            } else {
                // a stopping test for each condition.  Its sums: every slot's values in LDS, then for value q of condition k (lane 6 k + q)
                // the slots in order.
                if (t < n_cond * lp.slots)
#pragma unroll
                    for (int q = 0; q < 6; ++q) stage[t][q] = x[q];
                __syncthreads();
                if (lane < 6 * n_cond) {
                    const int k = lane / 6, q = lane - 6 * k;
                    double v = sums[pb ^ 1][lane];   // frozen: as it was
                    if ((act >> k) & 1) {
                        v = 0.0;
                        for (int k0 = 0; k0 < lp.slots; k0 += 8) {
                            double y[8];
#pragma unroll
                            for (int i = 0; i < 8; ++i) y[i] = k0 + i < lp.slots ? stage[k * lp.slots + min(k0 + i, lp.slots - 1)][q] : 0.0;
                            v += ((y[0] + y[1]) + (y[2] + y[3])) + ((y[4] + y[5]) + (y[6] + y[7]));
                        }
                        if (q == 5 && j > 0) v = sums[pb ^ 1][lane];   // ||S||^2 comes with the first pass
                    }
                    sums[pb][lane] = v;
                }
                loop_wave_fence();
                const int lc = 6 * (lane < n_cond ? lane : 0);
                const double s_rz = sums[pb][lc], s_rr = sums[pb][lc + 1], s_zaz = sums[pb][lc + 2], s_zau = sums[pb][lc + 3],
                             s_uau = sums[pb][lc + 4], s_ss = sums[pb][lc + 5], s_gp = sums[pb ^ 1][lc];
                const bool mine = lane < n_cond && ((act >> lane) & 1) && sqrt(s_rr / (s_ss > 0.0 ? s_ss : 1.0)) > eps_mine;
                active = (unsigned)__builtin_amdgcn_readfirstlane((int)__ballot(mine));
                all_done = active == 0;
                // frozen: every wavefront has met the barrier behind its look at the words
                if (__builtin_expect(!((active >> c) & 1), 0) && t < 12) put_word(pass_no + 1u, 0.0);
                auto over_conds = [&](double y, bool on) {   // conditions fill at most one row of 16 lanes
                    y = on ? y : 0.0;
                    y += dpp_perm<0x128>(y);
                    y += dpp_perm<0x124>(y);
                    y += dpp_perm<0x122>(y);
                    y += dpp_perm<0x121>(y);
                    return wave_uniform(y);
                };
                rr = over_conds(s_rr, lane < n_cond);
                ss = over_conds(s_ss, lane < n_cond);
                const double dn = over_conds(s_rz, mine), dp = over_conds(s_gp, mine);
                const double zaz = over_conds(s_zaz, mine), zau = over_conds(s_zau, mine), uau = over_conds(s_uau, mine);
                beta = j > 0 ? dn / dp : 0.0;
                alpha = dn / (j > 0 ? zaz + 2.0 * beta * zau + beta * beta * uau : zaz);
                bad_ab = !finite_d(beta) || !finite_d(alpha);
            }
            if (__builtin_amdgcn_readfirstlane(gave_up)) {
                if (t == 0) __hip_atomic_store(lp.abort_word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return;
            }
            // The square root is taken only where it can decide: a finite ||r||^2 clearly above the bound goes on.
            const bool far = !async && eps > 1e-150 && finite_d(rr) && rr > 1.000001 * eps * eps * ss && ss > 0.0;
            double rel = 1.0;
            bool converged = all_done, bad = false;
            if (__builtin_amdgcn_readfirstlane(!far)) {
                rel = sqrt(rr / (ss > 0.0 ? ss : 1.0));
                if (!async) converged = rel <= eps;
                bad = !finite_d(rel);
            }
            bad = bad || (!converged && j < max_iter && bad_ab);
            alpha = wave_uniform(alpha);
            beta = wave_uniform(beta);
            const bool stop = __builtin_amdgcn_readfirstlane(bad || converged || j >= max_iter) != 0;
            const bool quit = stop || !((active >> c) & 1);
            const bool last = stop || it + 1 == n_pass_all;
            // The first workgroup of the first condition that was iterating keeps the records.  Which that is
            // changes as conditions freeze, so a launch writes the result only here, in its last pass.
            if (kc == 0 && c == __ffs((int)act) - 1 && wv == 0) {
                // the totals leave out the conditions: lane k adds value q of condition k over its slots
                auto cond_value = [&](int q) {
                    const loop_word* src = words + q * pair_stride + 2 * (lane < n_cond ? lane : 0) * lp.slots;
                    double v = 0.0;
                    for (int k = 0; k < lp.slots; ++k) v += loop_unpack(loop_load(src + 2 * k), loop_load(src + 2 * k + 1));
                    return v;
                };
                if (!async && j == 0) ss_mine = cond_value(5);
                if (last) {                          // the record the host reads, and the next launch
                    rel = sqrt(rr / (ss > 0.0 ? ss : 1.0));
                    if (lane == 0) {
                        sc->iterations = j;
                        sc->rel = rel;
                        sc->status = bad ? -4 : (converged ? 0 : (j >= max_iter ? -3 : 0));
                        sc->done = stop ? 1 : 0;
                        st_out->iter = j + 1;
                        st_out->done = stop ? 1 : 0;
                        st_out->act = (int)active;
                        st_out->rz = rz_prev;
                        st_out->ss = ss_all;
                    }
                    if (async) {
                        if (lane < 6 * n_cond) st_out->sums[lane] = sums[pb][lane];
                        if (lane < n_cond) sc->rel_cond[lane] = sqrt(sums[pb][6 * lane + 1] / (sums[pb][6 * lane + 5] > 0.0 ? sums[pb][6 * lane + 5] : 1.0));
                    } else if (lane < n_cond) {
                        const double v = cond_value(1);   // r.r
                        st_out->ss_c[lane] = ss_mine;
                        sc->rel_cond[lane] = sqrt(v / (ss_mine > 0.0 ? ss_mine : 1.0));
                    }
                }
                if (hist && !stop && j < hist_cap && lane == 0) {
                    hist[2 * j] = alpha;
                    hist[2 * j + 1] = beta;
                }
            }
            if (quit) {                              // the solve or this condition (frozen from here on) ends
                save_p();
                return;
            }
            act = (active & 0xffffu) | (act << 16);
            if (need_halo) halo_keep();
        }
        if (has_tile) {
            pass(alpha, beta, first);
            publish_z(first ? 0 : j + 1);
        }
        publish_sums(base + (first ? 1u : (unsigned)j + 2u), first);
        if (!first) ++j;
        first = false;
        if (it + 1 == n_pass_all) {
            save(j);
            return;
        }
    }
}
