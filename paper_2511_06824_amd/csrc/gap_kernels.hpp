// HIP kernels of the joint piston-gap solve (gfx950, FP64, no MFMA: bandwidth-bound sparse work).
//
// Work decomposition shared by the solve kernels: the rows of every condition are cut into
// `per_cond` chunks of `rows` consecutive rows; block b works on chunk b (condition
// b / per_cond).  Every chunk writes one partial sum per reduced quantity to a fixed slot,
// and a one-block finalize kernel adds the slots of each condition in a fixed order, so
// all reductions are deterministic and independent of scheduling.
#pragma once

#include "gap_device.hpp"

struct ChunkMap {
    int per_cond;   // chunks per condition
    int rows;       // rows per chunk (the last chunk of a condition may hold fewer)
    int total;      // per_cond * n_cond
};

__device__ __forceinline__ void chunk_rows(const ChunkMap& cm, int nz, int b, int& c, int& j0, int& j1)
{
    c = b / cm.per_cond;
    j0 = (b - c * cm.per_cond) * cm.rows;
    j1 = min(j0 + cm.rows, nz);
}

// ---------------------------------------------------------------------------------------
// Texture: spherical caps scattered over their footprint boxes, overlaps combined by max.
// Depths are >= 0, so their IEEE bit patterns order like unsigned integers.
// plane 0: cell centres, plane 1: east faces, plane 2: axial faces (nz + 1 rows).
__global__ __launch_bounds__(GAP_BLOCK) void k_texture(GeomDev g, int count, const double* __restrict__ th_c,
                          const double* __restrict__ z_c, const double* __restrict__ rad,
                          const double* __restrict__ dep, double* tex_c, double* tex_e, double* tex_f)
{
    const int k = blockIdx.x;
    const int plane = blockIdx.y;
    if (k >= count) return;
    const double tc = th_c[k], zc = z_c[k], a = rad[k], d = dep[k];
    const double rho = (a * a + d * d) / (2.0 * d);
    const double half_ang = a / g.R;
    const int span_i = (int)ceil(half_ang / g.dth) + 2;
    int ncol = 2 * span_i + 1;
    if (ncol > g.nt) ncol = g.nt;
    const int ic0 = (int)floor(tc / g.dth) - span_i;
    const int nrows = (plane == 2) ? g.nz + 1 : g.nz;
    int jlo = (int)floor((zc - a) / g.dz) - 2;
    int jhi = (int)ceil((zc + a) / g.dz) + 2;
    if (jlo < 0) jlo = 0;
    if (jhi > nrows - 1) jhi = nrows - 1;
    if (jhi < jlo) return;
    double* dst = plane == 0 ? tex_c : (plane == 1 ? tex_e : tex_f);
    const double two_pi = 2.0 * 3.14159265358979323846;
    const long long cells = (long long)ncol * (jhi - jlo + 1);
    for (long long q = threadIdx.x; q < cells; q += blockDim.x) {
        const int jr = jlo + (int)(q / ncol);
        int i = (ic0 + (int)(q % ncol)) % g.nt;
        if (i < 0) i += g.nt;
        const double th = (plane == 1) ? (i + 1.0) * g.dth : (i + 0.5) * g.dth;
        const double z = (plane == 2) ? jr * g.dz : (jr + 0.5) * g.dz;
        double dt = th - tc + 0.5 * two_pi;
        dt = dt - two_pi * floor(dt / two_pi) - 0.5 * two_pi;
        const double ds = g.R * dt, dzz = z - zc;
        const double r2 = ds * ds + dzz * dzz;
        if (r2 < a * a) {
            const double v = sqrt(fmax(rho * rho - r2, 0.0)) - (rho - d);
            if (v > 0.0)
                atomicMax((unsigned long long*)&dst[(size_t)jr * g.nt + i],
                          (unsigned long long)__double_as_longlong(v));
        }
    }
}

// ---------------------------------------------------------------------------------------
// Assembly (step I): the face conductances of every operator and the source of every condition.
// kxz repeats the conductances as the pairs the strip iteration reads: pair (r + 1, i) holds the east
// face of cell (r, i) and the axial face above it, (kx(r, i), kz(r + 1, i)), for rows
// r = -1 .. n_axial - 1 (row -1: (0, the inlet face kz(0, i))), so that a row step reads its conductances
// with one 16-byte load per lane.
//
// A wavefront marches `rows` rows of 64 columns of one operator and forms the sources of all conditions
// that use it (their gaps are the operator's; only the squeeze term differs).  The north face of a row is
// the south face of the next, the west face of a column the east face of its neighbour lane, and what
// depends on z alone is formed once, row j0 + l on lane l, with the west faces of the first column: two
// films (a square root and two divisions each) per cell and operator, where one thread per cell and
// condition needs four.  With one thread per cell and condition and the pairs in a pass of their own,
// 2048 x 1024 with 9 conditions took 252 + 62 us, bound by those square roots and divisions; this form
// takes 113 us for the 540 MB it writes and reads (4.8 TB/s).  1024 x 512: 64 + 14 -> 31 us.
constexpr int kAssembleRows = 8;        // at most: 2048 x 1024 took 139 us in chunks of 32 rows, 113 in 10, 110 in 5
__global__ __launch_bounds__(GAP_BLOCK) void k_assemble(GeomDev g, CondDev cd, TablesDev tb, int rows,
                                                        double* __restrict__ kx, double* __restrict__ kz,
                                                        double* __restrict__ kxz, double* __restrict__ S)
{
    const int nt = g.nt, nz = g.nz, o = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int unit = blockIdx.x * (GAP_BLOCK / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int strips = (nt + 63) / 64;
    const int j0 = unit / strips * rows, j1 = min(j0 + rows, nz), i0 = unit % strips * 64;
    if (j0 >= nz) return;
    const size_t n = (size_t)nt * nz;
    const bool on = i0 + lane < nt;
    const int i = min(i0 + lane, nt - 1);                   // lanes past the ring repeat its last column
    const double* e = cd.e[o];
    // row j0 + lane: its axial position and eccentricity, those of its south face, its west face
    const int jl = j0 + min(lane, j1 - j0);                 // one more face than rows
    const int jr = min(jl, j1 - 1), iw = i0 ? i0 - 1 : nt - 1;
    const double t_row = (jr + 0.5) * g.dz / g.L;
    double ex_row, ey_row, ex_face, ey_face;
    film_axis(e, t_row, ex_row, ey_row);
    film_axis(e, jl * g.dz / g.L, ex_face, ey_face);
    const double h_row = film_at(g, ex_row, ey_row, tb.cos_e[iw], tb.sin_e[iw], tb.tex_e[jr * nt + iw]);

    const double cos_c = tb.cos_c[i], sin_c = tb.sin_c[i], cos_e = tb.cos_e[i], sin_e = tb.sin_e[i];
    const double kfx = g.dz / g.dx / (12.0 * g.mu), kfz = g.dx / g.dz / (12.0 * g.mu);
    double* kxo = kx + (size_t)o * n;
    double* kzo = kz + (size_t)o * (n + nt);
    double2* kxzo = (double2*)kxz + (size_t)o * (n + nt);
    double h_s = film_at(g, read_lane(ex_face, 0), read_lane(ey_face, 0), cos_c, sin_c, tb.tex_f[j0 * nt + i]);
    double k_s = (j0 == 0 ? 2.0 : 1.0) * (h_s * h_s * h_s) * kfz;
    if (on && j0 == 0) kxzo[i] = make_double2(0.0, k_s);
    for (int j = j0; j < j1; ++j) {
        const int r = j - j0, gidx = j * nt + i;
        const double ex = read_lane(ex_row, r), ey = read_lane(ey_row, r), t = read_lane(t_row, r);
        const double h_n = film_at(g, read_lane(ex_face, r + 1), read_lane(ey_face, r + 1), cos_c, sin_c, tb.tex_f[gidx + nt]);
        const double h_e = film_at(g, ex, ey, cos_e, sin_e, tb.tex_e[gidx]);
        const double h_w = dpp_shift<0x138>(h_e, read_lane(h_row, r));
        const double k_e = (h_e * h_e * h_e) * kfx;
        const double k_n = (j == nz - 1 ? 2.0 : 1.0) * (h_n * h_n * h_n) * kfz;
        if (on) {
            kxo[gidx] = k_e;
            kzo[gidx] = k_s;
            if (j == nz - 1) kzo[gidx + nt] = k_n;
            kxzo[gidx + nt] = make_double2(k_e, k_n);
        }
        // the squeeze rate at the cell centre, with the parts that depend on the gap alone formed once
        const double ax = fma(g.Rc, cos_c, -ex), ay = fma(g.Rc, sin_c, -ey);
        const double dist = sqrt(fma(ax, ax, ay * ay));
        const double slide = fma(g.dz, -0.5 * g.U * (h_e - h_w), g.dx * (-0.5 * g.V * (h_n - h_s)));
        for (int c = o; c < cd.n_cond; c = max(c + 1, cd.n_op)) {
            if (cd.op[c] != o) continue;
            const double* ed = cd.ed[c];
            double exd, eyd;
            film_axis(ed, t, exd, eyd);
            const double rate = fma(ax, exd, ay * eyd) / dist;      // -dh/dt
            // -U/2 (h_e - h_w) dz - V/2 (h_n - h_s) dx - dh/dt dx dz, fused explicitly (as in film_at)
            double s = fma(g.dz, g.dx * rate, slide);
            if (j == 0) s = fma(g.p_in, k_s, s);
            if (j == nz - 1) s = fma(g.p_out, k_n, s);
            if (on) S[(size_t)c * n + gidx] = s;
        }
        h_s = h_n;
        k_s = k_n;
    }
}

// Diagonal A_PP = kx(i) + kx(i-1) + kz(j) + kz(j+1) (Dirichlet faces included).
__device__ __forceinline__ double diag_at(const double* kx, const double* kz, int i, int j, int nt)
{
    const int iw = i ? i - 1 : nt - 1;
    return ((kx[j * nt + i] + kx[j * nt + iw]) + kz[j * nt + i]) + kz[(j + 1) * nt + i];
}

// (A x)(i, j) with x given by a functor of (i, j).
template <class X>
__device__ __forceinline__ double apply_A(const double* kx, const double* kz, int i, int j, int nt,
                                          int nz, X x)
{
    const int iw = i ? i - 1 : nt - 1;
    const int ie = (i + 1 < nt) ? i + 1 : 0;
    const double kE = kx[j * nt + i], kW = kx[j * nt + iw];
    const double kS = kz[j * nt + i], kN = kz[(j + 1) * nt + i];
    double a = (((kE + kW) + kS) + kN) * x(i, j) - kE * x(ie, j) - kW * x(iw, j);
    if (j > 0) a -= kS * x(i, j - 1);
    if (j < nz - 1) a -= kN * x(i, j + 1);
    return a;
}

// Diagonal preconditioners: Jacobi (Eq 2.8) and ASSOR I (Eq 3.2), stored as M^{-1}_ii per
// operator.  ASSOR I: w(2-w) / (D_ii + w^2 sum_k L_ik^2 / D_kk), L the strict lower
// triangle in the natural order (west, south, and the east wrap of the last column).
__global__ __launch_bounds__(GAP_BLOCK) void k_diag_precond(GeomDev g, int kind, double omega, const double* __restrict__ kx_all,
                               const double* __restrict__ kz_all, double* __restrict__ minv, int n_op)
{
    const int o = blockIdx.y;
    const int n = g.nt * g.nz;
    const int gidx = blockIdx.x * blockDim.x + threadIdx.x;
    if (gidx >= n || o >= n_op) return;
    const double* kx = kx_all + (size_t)o * n;
    const double* kz = kz_all + (size_t)o * (n + g.nt);
    const int nt = g.nt, j = gidx / nt, i = gidx - j * nt;
    const double D = diag_at(kx, kz, i, j, nt);
    double val;
    if (kind == 0) {
        val = 1.0 / D;
    } else {
        double s = 0.0;
        if (i > 0) { const double l = kx[j * nt + i - 1]; s += l * l / diag_at(kx, kz, i - 1, j, nt); }
        if (i == nt - 1) { const double l = kx[j * nt + i]; s += l * l / diag_at(kx, kz, 0, j, nt); }
        if (j > 0) { const double l = kz[j * nt + i]; s += l * l / diag_at(kx, kz, i, j - 1, nt); }
        val = omega * (2.0 - omega) / (D + omega * omega * s);
    }
    minv[(size_t)o * n + gidx] = val;
}

// ---------------------------------------------------------------------------------------
// Force and moment integration (step III) with the cavitation rule; partials 0..3 are
// Fx, Fy, Mx, My per chunk before the factor dA.
__device__ __forceinline__ double peff(double p, int cav, double pc) { return (cav && p < pc) ? pc : p; }

// NV = 4: (Fx, Fy, Mx, My) of pressure and shear together.  NV = 10: the pressure part
// (Fx, Fy, Mx, My), then the shear part (Fx, Fy, Mx, My, Fz, Mz) with the axial force and the
// torque of the wall shear.
//
// A workgroup takes the whole rings of a chunk of rows, ring by ring, thread t the columns t, t + 256, ...: what
// cancels around a ring, the mean pressure and every harmonic but the first, cancels while the terms are
// added.  (Columns marched down the rows, two groups of 256 to a workgroup, take 94 us where this takes 105, but
// cancel only in the final sum: up to 30 times the error of the ring order where a third harmonic is strong.)
//
// LDS: the pressures of a row and of the row below it are kept there (rings up to kForceRing columns), so that each is
// read from memory once per chunk; three rows of every resident workgroup do not fit an L2.  The loads of a thread's
// next two cells are in flight during the arithmetic of the present two (with one, a pass over assembly, forces, split
// and field at 2048 x 1024 took 408 us, with two 393, with four, whose registers leave fewer wavefronts, 407), what
// depends on z alone is formed once per chunk, and one reciprocal of the gap serves both shear stresses.  A call at
// 2048 x 1024 with 9 conditions (168 MB read), 4 and 10 values: 156 and 184 us with loads where they are used, six
// divisions per cell and a single workgroup for the final sums, 123 and 117 us without the rows in the LDS, 105 and 101
// us so, about half of it the arithmetic of some 115 instructions per cell.  3072 x 600: 138 and 168, 111 and 108, 97
// and 95 us.  Longer rings would leave one or two workgroups per CU.
constexpr int kForceRows = 64;          // rows of z-dependent data held at once
constexpr int kForceRing = 3072;        // columns of a ring kept in the LDS
constexpr int kForceAhead = 2;          // cells whose loads a thread has in flight
template <int NV, bool LDS>
__global__ __launch_bounds__(GAP_BLOCK) void k_forces(GeomDev g, CondDev cd, ChunkMap cm, TablesDev tb,
                                                      const double* __restrict__ p_all, int cav, double p_cav,
                                                      double* __restrict__ partial)
{
    extern __shared__ double ring[];    // two rows of nt pressures
    int c, j0, j1;
    chunk_rows(cm, g.nz, blockIdx.x, c, j0, j1);
    const int nt = g.nt, nz = g.nz, t = threadIdx.x;
    const double* p = p_all + (size_t)c * nt * nz;
    const double* e = cd.e[c];
    double acc[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) acc[q] = 0.0;
    // -1/2 over the pressure differences' distances: 2 dx, 2 dz, and 3/2 dz at the end rows
    const double fx = -0.25 / g.dx, fz = -0.25 / g.dz, fz_end = -0.5 / (1.5 * g.dz);
    const double mu_u = g.mu * g.U, mu_v = g.mu * g.V;
    __shared__ double row_ex[kForceRows], row_ey[kForceRows], row_z[kForceRows];
    if (LDS)
        for (int i = t; i < nt; i += GAP_BLOCK) {
            ring[i] = j0 > 0 ? peff(p[(j0 - 1) * nt + i], cav, p_cav) : 0.0;
            ring[nt + i] = peff(p[j0 * nt + i], cav, p_cav);
        }
    // what a cell loads: its pressure to the north, texture depth and angle; kForceAhead columns at a time
    struct Cell {
        double pn, tx, cs, sn;
    };
    auto load = [&](int j, int i) {
        Cell x;
        x.pn = p[min(j + 1, nz - 1) * nt + i];
        x.tx = tb.tex_c ? tb.tex_c[j * nt + i] : 0.0;
        x.cs = tb.cos_c[i];
        x.sn = tb.sin_c[i];
        return x;
    };
    for (int jb = j0; jb < j1; jb += kForceRows) {
        const int je = min(jb + kForceRows, j1);
        __syncthreads();
        if (t < je - jb) {
            const double z = (jb + t + 0.5) * g.dz;
            film_axis(e, z / g.L, row_ex[t], row_ey[t]);
            row_z[t] = z - 0.5 * g.L;
        }
        __syncthreads();
        Cell next[kForceAhead];
        auto load_ahead = [&](int j, int i0) {
#pragma unroll
            for (int b = 0; b < kForceAhead; ++b) next[b] = load(j, min(i0 + b * GAP_BLOCK, nt - 1));
        };
        load_ahead(jb, t);
        for (int j = jb; j < je; ++j) {
            double* const below = ring + ((j - j0) & 1 ? nt : 0);
            const double* const here = ring + ((j - j0) & 1 ? 0 : nt);
            const double ex = row_ex[j - jb], ey = row_ey[j - jb], zr = row_z[j - jb];
            const double f_z = j == 0 || j == nz - 1 ? fz_end : fz;
            auto cell = [&](int i, const Cell& x) {
                const int iw = i ? i - 1 : nt - 1, ie = i + 1 < nt ? i + 1 : 0;
                const double pn = peff(x.pn, cav, p_cav);
                double pc, pw, pe, ps;
                if (LDS) {
                    pc = here[i];
                    pw = here[iw];
                    pe = here[ie];
                    ps = below[i];
                    below[i] = pn;                      // the row above takes its place
                } else {
                    const double* row = p + j * nt;
                    pc = peff(row[i], cav, p_cav);
                    pw = peff(row[iw], cav, p_cav);
                    pe = peff(row[ie], cav, p_cav);
                    ps = j > 0 ? peff(row[i - nt], cav, p_cav) : 0.0;
                }
                const double dpx = pe - pw, dpz = (j == nz - 1 ? g.p_out : pn) - (j == 0 ? g.p_in : ps);
                const double cs = x.cs, sn = x.sn, h = film_at(g, ex, ey, cs, sn, x.tx), inv = 1.0 / h;
                const double tt = h * (dpx * fx) + mu_u * inv;
                const double tz = h * (dpz * f_z) + mu_v * inv;
                if (NV == 4) {
                    acc[0] += -pc * cs - tt * sn;
                    acc[1] += -pc * sn + tt * cs;
                    acc[2] += zr * (pc * sn - tt * cs) + tz * g.R * sn;
                    acc[3] += -zr * (pc * cs + tt * sn) - tz * g.R * cs;
                } else {
                    acc[0] += -pc * cs;
                    acc[1] += -pc * sn;
                    acc[2] += zr * pc * sn;
                    acc[3] += -zr * pc * cs;
                    acc[4 % NV] += -tt * sn;
                    acc[5 % NV] += tt * cs;
                    acc[6 % NV] += -zr * tt * cs + tz * g.R * sn;
                    acc[7 % NV] += -zr * tt * sn - tz * g.R * cs;
                    acc[8 % NV] += tz;
                    acc[9 % NV] += g.R * tt;
                }
            };
            for (int i0 = t; i0 < nt; i0 += kForceAhead * GAP_BLOCK) {
                Cell now[kForceAhead];
#pragma unroll
                for (int b = 0; b < kForceAhead; ++b) now[b] = next[b];
                const bool more = i0 + kForceAhead * GAP_BLOCK < nt;
                load_ahead(more ? j : min(j + 1, je - 1), more ? i0 + kForceAhead * GAP_BLOCK : t);
#pragma unroll
                for (int b = 0; b < kForceAhead; ++b)
                    if (i0 + b * GAP_BLOCK < nt) cell(i0 + b * GAP_BLOCK, now[b]);
            }
            if (LDS) __syncthreads();                   // the row above is complete
        }
    }
    block_sum<NV>(acc);
    if (t == 0)
        for (int q = 0; q < NV; ++q) partial[q * cm.total + blockIdx.x] = acc[q];
}

// cos and sin of the cell-centre angles theta_i = (i + 1/2) dtheta, i < nt, formed on the
// device (the handle-free force integration has no host-built table).
__global__ __launch_bounds__(GAP_BLOCK) void k_trig_centres(int nt, double dth, double* __restrict__ cs,
                                                            double* __restrict__ sn)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nt) return;
    const double th = (i + 0.5) * dth;
    cs[i] = cos(th);
    sn[i] = sin(th);
}

__device__ __forceinline__ double cond_sum(const double* part, const ChunkMap& cm, int c)
{
    double v[1] = {0.0};
    for (int b = threadIdx.x; b < cm.per_cond; b += blockDim.x) v[0] += part[c * cm.per_cond + b];
    block_sum<1>(v);
    return v[0];   // valid in thread 0
}

// One workgroup per condition and value (a single one took 14 us for 9 conditions of 4 values).
__global__ __launch_bounds__(GAP_BLOCK) void k_forces_finalize(ChunkMap cm, int nv, double dA,
                                                               const double* __restrict__ part, double* __restrict__ F)
{
    const int c = blockIdx.x / nv, q = blockIdx.x - c * nv;
    const double s = cond_sum(part + q * cm.total, cm, c);
    if (threadIdx.x == 0) F[c * nv + q] = s * dA;
}

// ||S - A p||^2 and ||S||^2 per chunk of rows, the true residual of a returned solution.
__global__ __launch_bounds__(GAP_BLOCK) void k_true_residual(GeomDev g, CondDev cd, ChunkMap cm,
                                                             const double* __restrict__ kx_all,
                                                             const double* __restrict__ kz_all,
                                                             const double* __restrict__ S_all,
                                                             const double* __restrict__ p_all, double* __restrict__ partial)
{
    int c, j0, j1;
    chunk_rows(cm, g.nz, blockIdx.x, c, j0, j1);
    const int nt = g.nt, nz = g.nz;
    const size_t n = (size_t)nt * nz;
    const int op = cd.op[c];
    const double* kx = kx_all + (size_t)op * n;
    const double* kz = kz_all + (size_t)op * (n + nt);
    const double* S = S_all + (size_t)c * n;
    const double* p = p_all + (size_t)c * n;
    double acc[2] = {0.0, 0.0};
    for (int j = j0; j < j1; ++j) {
        for (int i = threadIdx.x; i < nt; i += blockDim.x) {
            const size_t gi = (size_t)j * nt + i;
            const int iw = i ? i - 1 : nt - 1;
            const int ie = (i + 1 < nt) ? i + 1 : 0;
            const double kE = kx[gi], kW = kx[(size_t)j * nt + iw];
            const double kS = kz[gi], kN = kz[gi + nt];
            double Ap = (((kE + kW) + kS) + kN) * p[gi] - kE * p[(size_t)j * nt + ie] - kW * p[(size_t)j * nt + iw];
            if (j > 0) Ap -= kS * p[gi - nt];
            if (j < nz - 1) Ap -= kN * p[gi + nt];
            const double r = S[gi] - Ap;
            acc[0] += r * r;
            acc[1] += S[gi] * S[gi];
        }
    }
    block_sum<2>(acc);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = acc[0];
        partial[cm.total + blockIdx.x] = acc[1];
    }
}

// GMAF step II: the full field with its boundary rows, out[c][j][i] for j = 0 .. n_axial + 1
// (row 0: p_in at z = 0, rows 1 .. n_axial: the cell centres after the cavitation rule, last
// row: p_out at z = L).
__global__ __launch_bounds__(GAP_BLOCK) void k_rebuild(GeomDev g, int n_cond, const double* __restrict__ p_all, int cav,
                                                       double p_cav, double* __restrict__ out)
{
    const size_t nt = g.nt, nz = g.nz;
    const size_t per = (nz + 2) * nt;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= per * (size_t)n_cond) return;
    const size_t c = idx / per, r = idx - c * per;
    const size_t j = r / nt, i = r - j * nt;
    double v;
    if (j == 0) v = g.p_in;
    else if (j == nz + 1) v = g.p_out;
    else v = peff(p_all[c * nz * nt + (j - 1) * nt + i], cav, p_cav);
    out[idx] = v;
}

// Eq 2.13-2.14: J[i][k] = (F_{k+1,i} - F_{0,i}) / delta_k.
struct Delta8 { double d[8]; };
__global__ void k_jacobian_fd(const double* __restrict__ F, Delta8 dl, double* __restrict__ J)
{
    const int t = threadIdx.x;
    if (t >= 32) return;
    const int i = t / 8, k = t % 8;
    J[t] = (F[(k + 1) * 4 + i] - F[i]) / dl.d[k];
}
