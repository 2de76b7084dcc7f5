// gfx950 kernels of the 2D electrostatic PIC step (arXiv:1610.03918, Sec. II).
//
// Every kernel serves a batch of independent instances: per-instance state
// is read from a device array of Inst descriptors, and a launch covers the
// blocks of several units (instances, or instance x species pairs) listed in
// a Tab.  Grid kernels work on node grids (NX x NY, row-major in x) with
// 64x4 thread blocks; floating-point reductions are float64 block partials
// summed in block order by a one-block-per-unit finalize kernel, so every
// result is reproducible bit for bit.  The particle kernel processes one tile
// of cells per block, accumulating the area-weighting moments of its
// particles in LDS as integers and flushing them to the int64 node charge
// with atomics (exact, order-free).
//
// Compiled with -ffp-contract=off: every float operation of the push is
// rounded in the order written.
#include "pic_internal.h"
#include "wave_ops.h"

#include <algorithm>
#include <atomic>

namespace pic {

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ int wrap_lo(int a, int n) { return a < 0 ? a + n : a; }
__device__ __forceinline__ int wrap_hi(int a, int n) { return a >= n ? a - n : a; }

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return v;
}

// Unit of a launch that owns block b (uniform per block).
__device__ __forceinline__ int unit_of(const Tab &t, int b)
{
    int k = 0;
    while (k + 1 < t.n && b >= t.boff[k + 1]) k++;
    return k;
}

static inline int tab_blocks(const Tab &t) { return t.boff[t.n]; }

// Grid kernels: node (i, j) of the unit that owns this block.
#define GRID_BEGIN(t)                                                        \
    const int ku = unit_of(t, (int)blockIdx.x);                              \
    const int lb = (int)blockIdx.x - t.boff[ku];                             \
    const int byb = lb / t.bx[ku], bxb = lb - byb * t.bx[ku];                \
    const int j = bxb * kGridBX + (int)threadIdx.x;                          \
    const int i = byb * kGridBY + (int)threadIdx.y;                          \
    const Inst &I = insts[t.id[ku]];

#define NODE_IDX(NX_, NY_)                                                   \
    const int NX = (NX_), NY = (NY_);                                        \
    const bool inb = (i < NX) && (j < NY);                                   \
    const long long n = (long long)i * NY + j;

static inline dim3 gblock() { return dim3(kGridBX, kGridBY); }

// Writes this block's sums of NQ per-thread values (fixed tree order) to
// pt.p[q * stride + block].  k_finalize adds a unit's partials in block order.
template <int NQ>
__device__ void block_partials(const double (&val)[NQ], const Part &pt)
{
    __shared__ double sh[NQ][16];
    const int tid = threadIdx.x + threadIdx.y * blockDim.x;
    const int nt = blockDim.x * blockDim.y;
    const int lane = tid & 63, wid = tid >> 6, nw = (nt + 63) >> 6;
#pragma unroll
    for (int q = 0; q < NQ; q++) {
        double v = wave_sum(val[q]);
        if (lane == 0) sh[q][wid] = v;
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int q = 0; q < NQ; q++) {
            double s = 0.0;
            for (int w = 0; w < nw; w++) s += sh[q][w];
            pt.p[q * pt.stride + blockIdx.x] = s;
        }
    }
}

// Scalar logic of operation op on one instance, from the totals t0, t1 of
// its partials (one thread).
__device__ void apply_op(const Inst &I, int op, double t0, double t1)
{
    double *S = I.S;
    int *F = I.F;
    if ((op == OP_PQ || op == OP_UPDATE || op == OP_RZ) && F[F_DONE]) return;
    if (op == OP_RR64_PASS && (F[F_SKIP] || F[F_CGABORT])) return;
    if (op == OP_INIT && F[F_CONV]) {
        F[F_SKIP] = 1;
        F[F_DONE] = 1;
        return;
    }
    const double bb = S[S_BB] > 0.0 ? S[S_BB] : 1.0;
    const double tol2 = I.rtol * I.rtol;
    switch (op) {
    case OP_ASM:
        if (I.g.px && I.g.py) S[S_SUM] = t1;
        else S[S_BB] = t0;
        break;
    case OP_BB_PER: S[S_BB] = t0; break;
    case OP_SUM: S[S_SUM] = t0; break;
    case OP_RR64_START:
        // ||b||^2 of the right-hand side being solved (b may have been written
        // by the caller since the last assembly)
        S[S_BB] = t1;
        S[S_RR64] = t0;
        S[S_RELRES0] = t0;
        F[F_CONV] = (t0 <= tol2 * (t1 > 0.0 ? t1 : 1.0)) ? 1 : 0;
        F[F_ITER_TOT] = 0;
        F[F_PASSES] = 0;
        F[F_ITER1] = 0;
        F[F_DONE] = 0;
        F[F_SKIP] = 0;
        break;
    case OP_RR64_PASS:
        S[S_RR64] = t0;
        F[F_CONV] = (t0 <= tol2 * bb) ? 1 : 0;
        break;
    case OP_INIT: {
        // inner stop ratio: 0.3 rtol / relres, kept within [eta_min, 0.5]
        double eta2 = 0.09 * tol2 * bb / (S[S_RR64] > 0.0 ? S[S_RR64] : 1.0);
        const double lo = I.eta_min * I.eta_min;
        eta2 = eta2 < lo ? lo : (eta2 > 0.25 ? 0.25 : eta2);
        F[F_SKIP] = 0;
        S[S_ETA2] = eta2;
        S[S_RR0] = t0;
        S[S_RR] = t0;
        F[F_DONE] = (t0 == 0.0) ? 1 : 0;
        F[F_ITER] = 0;
        F[F_PASSES] += 1;
        if (!I.mg) { S[S_RZOLD] = S[S_RZ]; S[S_RZ] = t1; }
        break;
    }
    case OP_PQ: S[S_PQ] = t0; break;
    case OP_UPDATE:
        if (I.mg && !(S[S_CG_NALPHA] > 0.0 && S[S_CG_NALPHA] < INFINITY && S[S_CG_NBETA] < INFINITY)) {
            // the step had no usable length (the level-0 down kernel skipped it)
            F[F_DONE] = 1;
            break;
        }
        S[S_RR] = t0;
        F[F_ITER] += 1;
        F[F_ITER_TOT] += 1;
        if (F[F_PASSES] == 1) F[F_ITER1] = F[F_ITER];
        if (t0 <= S[S_ETA2] * S[S_RR0]) F[F_DONE] = 1;
        if (!I.mg) { S[S_RZOLD] = S[S_RZ]; S[S_RZ] = t1; }
        else {
            // the step's alpha, beta and r.z, computed by the level-0 down kernel
            S[S_CG_ALPHA] = S[S_CG_NALPHA];
            S[S_CG_BETA] = S[S_CG_NBETA];
            S[S_CG_GAMMA] = S[S_CG_NGAMMA];
        }
        break;
    case OP_RZ: S[S_RZOLD] = S[S_RZ]; S[S_RZ] = t0; break;
    }
}

// Sums of the partials b0 .. b1-1 of nq quantities by threads 0 .. 255 of a
// block (others pass through): per-thread sums in a fixed order, then one
// per wavefront into sh[q][0 .. 3].  The caller synchronises and adds the
// four, so every kernel that reduces the same partials gets the same totals.
// RND loads a thread and quantity are in flight.
template <int RND = 8> struct PartialSums {
    double v[2][RND];

    // the first round's loads
    __device__ __forceinline__ void load(const Part &pt, int b0, int b1, int nq, int tid)
    {
#pragma unroll
        for (int r = 0; r < RND; r++) {
            const int k = b0 + r * 256 + tid;
            v[0][r] = tid < 256 && k < b1 ? pt.p[k] : 0.0;
            v[1][r] = tid < 256 && nq > 1 && k < b1 ? pt.p[pt.stride + k] : 0.0;
        }
    }
    __device__ __forceinline__ void sum(const Part &pt, int b0, int b1, int nq, double (*sh)[4], int tid)
    {
        if (tid >= 256) return;
        const int lane = tid & 63, wid = tid >> 6;
        double s[2] = {0.0, 0.0};
        for (int k0 = b0;;) {
#pragma unroll
            for (int r = 0; r < RND; r++) {
                s[0] += v[0][r];
                s[1] += v[1][r];
            }
            k0 += RND * 256;
            if (k0 >= b1) break;
            load(pt, k0, b1, nq, tid);
        }
        for (int q = 0; q < 2; q++) {
            const double w = wave_sum(s[q]);
            if (lane == 0) sh[q][wid] = w;
        }
    }
};
__device__ __forceinline__ void partial_sums_256(const Part &pt, int b0, int b1, int nq, double (*sh)[4], int tid)
{
    PartialSums<> p;
    p.load(pt, b0, b1, nq, tid);
    p.sum(pt, b0, b1, nq, sh, tid);
}

// x, of which the compiler does not know that it has not changed: what
// follows from it is computed where it is used and not carried around a loop.
template <class X> __device__ __forceinline__ X opaque(X x)
{
    asm volatile("" : "+v"(x));
    return x;
}
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
// Ends the program where the flag is set, by an instruction beside the test: a
// jump to the kernel's end fetches code from another page.
__device__ __forceinline__ void end_if(int flag)
{
    if (__builtin_expect(uniform(flag), 1)) __builtin_amdgcn_endpgm();
}
// a[k] by a vector load: a wait for a scalar load is one for all of them, those
// for the addresses of the loads to come included.
template <class T> __device__ __forceinline__ T vload(const T *a, int k)
{
    asm("" : "+v"(k));
    return a[k];
}

// Chronopoulos-Gear recurrences of the multigrid-preconditioned CG from
// gamma = r.z and delta = (A z).z of the last V-cycle: beta = gamma /
// gamma_old, alpha = gamma / (delta - beta gamma / alpha_old) (= r.z / p.Ap);
// on the first step alpha = gamma / delta, beta = 0.  False when the step
// length is not positive and finite (the inner solve ends there; the float64
// refinement carries on).
__device__ __forceinline__ bool cg_coefficients(int iter, double gamma, double delta, double gamma_old,
                                                double alpha_old, double &alpha, double &beta)
{
    beta = 0.0;
    if (iter == 0) {
        alpha = gamma / delta;
    } else {
        beta = gamma / gamma_old;
        alpha = gamma / (delta - beta * gamma / alpha_old);
    }
    return alpha > 0.0 && alpha < INFINITY && beta < INFINITY;
}

// One block per unit: totals of the unit's partials in block order, then the
// scalar logic of the operation on that instance.
__global__ __launch_bounds__(256) void k_finalize(const Inst *insts, Tab t, Part pt, int op)
{
    const Inst &I = insts[t.id[blockIdx.x]];
    const int *F = I.F;
    const bool inner = op == OP_PQ || op == OP_UPDATE || op == OP_RZ;
    if (inner && F[F_DONE]) return;
    if (op == OP_RR64_PASS && (F[F_SKIP] || F[F_CGABORT])) return;
    if (op == OP_INIT && F[F_CONV]) {
        if (threadIdx.x == 0) apply_op(I, op, 0.0, 0.0);
        return;
    }
    __shared__ double sh[2][4];
    const int tid = threadIdx.x;
    const int nq = (op == OP_ASM || op == OP_INIT || op == OP_UPDATE || op == OP_RR64_START) ? 2 : 1;
    partial_sums_256(pt, t.boff[blockIdx.x], t.boff[blockIdx.x + 1], nq, sh, tid);
    __syncthreads();
    if (tid != 0) return;
    apply_op(I, op, sh[0][0] + sh[0][1] + sh[0][2] + sh[0][3], sh[1][0] + sh[1][1] + sh[1][2] + sh[1][3]);
}

static void finalize(const Inst *I, const Tab &t, Part pt, int op, hipStream_t s)
{
    if (t.n > 0) hipLaunchKernelGGL(k_finalize, dim3(t.n), dim3(256), 0, s, I, t, pt, op);
}

__global__ void k_zero_u64(unsigned long long *p, long long n)
{
    long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long st = (long long)gridDim.x * blockDim.x;
    for (; k < n; k += st) p[k] = 0ull;
}

void launch_zero_u64(unsigned long long *p, long long n, hipStream_t s)
{
    if (n <= 0) return;
    long long nb = (n + 255) / 256;
    if (nb > 4096) nb = 4096;
    hipLaunchKernelGGL(k_zero_u64, dim3((unsigned)nb), dim3(256), 0, s, p, n);
}

__global__ void k_tick(long long *step) { *step += 1; }

void launch_tick(long long *step, hipStream_t s)
{
    hipLaunchKernelGGL(k_tick, dim3(1), dim3(1), 0, s, step);
}

// ---------------------------------------------------------------------------
// field: E = -grad(phi) at the four corners of every cell (Sec. II)
// ---------------------------------------------------------------------------

// One axis of -grad(phi) at a node.  Inside: central difference.  At a
// Dirichlet node: two-point difference toward the only free neighbour if
// exactly one neighbour is free; central if both neighbours exist (zero along
// an equipotential wall); two-point with the only neighbour at a domain edge.
__device__ __forceinline__ double axis_field(double pm, double pc, double pp, bool hm, bool hp,
                                             bool fm, bool fp, bool fixed)
{
    if (!fixed) return -(pp - pm) * 0.5;
    if (hm && hp) {
        if (fp && !fm) return -(pp - pc);
        if (fm && !fp) return -(pc - pm);
        return -(pp - pm) * 0.5;
    }
    if (hp) return -(pp - pc);
    if (hm) return -(pc - pm);
    return 0.0;
}

__device__ __forceinline__ float2 node_field(const Geom g, const uint8_t *nc, const double *phi,
                                             int i, int j)
{
    const int NX = g.NX, NY = g.NY;
    const long long n = (long long)i * NY + j;
    // all loads at once: a neighbour that is not there is the wrapped one, not used
    const int im = wrap_lo(i - 1, NX), ip = wrap_hi(i + 1, NX), jm = wrap_lo(j - 1, NY), jp = wrap_hi(j + 1, NY);
    const long long a = (long long)im * NY + j, c = (long long)ip * NY + j;
    const long long d = (long long)i * NY + jm, e = (long long)i * NY + jp;
    const uint8_t cn = nc[n], ca = nc[a], cc = nc[c], cd = nc[d], ce = nc[e];
    const double pc = phi[n], pa = phi[a], pp_ = phi[c], pd = phi[d], pe = phi[e];
    const bool fixed = cn != 0;
    const bool hm = g.px || i > 0, hp = g.px || i < NX - 1;
    const double pm = hm ? pa : 0.0, pp = hp ? pp_ : 0.0;
    const bool fm = hm && ca == 0, fp = hp && cc == 0;
    double ex = axis_field(pm, pc, pp, hm, hp, fm, fp, fixed);
    const bool gm = g.py || j > 0, gp = g.py || j < NY - 1;
    const double qm = gm ? pd : 0.0, qp = gp ? pe : 0.0;
    const bool em = gm && cd == 0, ep = gp && ce == 0;
    double ey = axis_field(qm, pc, qp, gm, gp, em, ep, fixed);
    return make_float2((float)ex, (float)ey);
}

// One thread per cell; writes the cell's four corner fields (float32, each
// node's computed once per block) and,
// when requested (the field of a push), clears both species' node charge for
// the coming deposit.  The field of a push also counts, in F_UNCONV, a
// potential whose last residual test failed, and keeps the largest such
// relative residual in S_WORST (one thread per instance).
__global__ void k_field(const Inst *insts, Tab t, int zero_rho)
{
    GRID_BEGIN(t)
    const Geom g = I.g;
    if (zero_rho && i == 0 && j == 0 && !I.F[F_CONV]) {
        I.F[F_UNCONV] += 1;
        const double bb = I.S[S_BB] > 0.0 ? I.S[S_BB] : 1.0;
        const double rel = sqrt(I.S[S_RR64] / bb);
        if (!(rel <= I.S[S_WORST])) I.S[S_WORST] = rel;
    }
    if (zero_rho && i < g.NX && j < g.NY) {
        const long long n = (long long)i * g.NY + j;
        I.rho[0][n] = 0ull;
        I.rho[1][n] = 0ull;
    }
    // the field of each node of the block's (kGridBY + 1) x (kGridBX + 1)
    // corner set, once, in LDS; a periodic axis wraps the far row / column
    const uint8_t *nc = I.node_cond;
    const double *phi = I.phi;
    __shared__ float2 sn[kGridBY + 1][kGridBX + 1];
    const int ti = (int)threadIdx.y, tj = (int)threadIdx.x;
    auto node_at = [&](int a, int b) {
        if (g.px && a >= g.NX) a %= g.NX;
        if (g.py && b >= g.NY) b %= g.NY;
        return (a < g.NX && b < g.NY) ? node_field(g, nc, phi, a, b) : make_float2(0.f, 0.f);
    };
    sn[ti][tj] = node_at(i, j);
    if (ti == 0) sn[kGridBY][tj] = node_at(i - ti + kGridBY, j);
    if (ti == 1 && tj <= kGridBY) sn[tj][kGridBX] = node_at(i - ti + tj, j - tj + kGridBX);
    __syncthreads();
    if (i >= g.nx || j >= g.ny) return;
    const float2 e00 = sn[ti][tj], e10 = sn[ti + 1][tj], e01 = sn[ti][tj + 1], e11 = sn[ti + 1][tj + 1];
    const long long c = (long long)i * g.ny + j;
    I.E4[2 * c] = make_float4(e00.x, e00.y, e10.x, e10.y);
    I.E4[2 * c + 1] = make_float4(e01.x, e01.y, e11.x, e11.y);
}

void launch_field(const Inst *I, const Tab &t, int zero_rho, hipStream_t s)
{
    if (t.n) hipLaunchKernelGGL(k_field, dim3(tab_blocks(t)), gblock(), 0, s, I, t, zero_rho);
}

// ---------------------------------------------------------------------------
// assemble: b = (N_i - N_e) w 2^-32 + Dirichlet lifts (eq. 5, unit spacing)
// V: conductor potentials, 8 per instance (indexed by instance id)
// ---------------------------------------------------------------------------

// V: conductor potentials of every step of the table window, indexed
// ((step - base) * ninst + instance) * 8 with the device step counter.
// A window row outside [0, vwin) (the runtime never launches one) sets the
// instance's kErrVWindow error bit, which the host reports as PIC_ERR_STATE
// at its next look at the flags; the read itself stays inside the table.
__global__ void k_assemble(const Inst *insts, Tab t, const double *Vtab, const long long *ctl,
                           int ninst, int vwin, Part pt)
{
    GRID_BEGIN(t)
    const Geom g = I.g;
    NODE_IDX(g.NX, g.NY)
    long long row = ctl[0] - ctl[1];
    if (row < 0 || row >= vwin) {
        if (i == 0 && j == 0) I.F[F_ERR] |= kErrVWindow;
        row = 0;
    }
    const double *V = Vtab + (row * ninst + t.id[ku]) * 8;
    double bb = 0.0, sm = 0.0;
    if (inb) {
        // all loads at once; a bounded edge's nodes are conductors, so that the
        // wrapped neighbours there are not used
        const uint8_t *nc = I.node_cond;
        const int im = wrap_lo(i - 1, NX), ip = wrap_hi(i + 1, NX);
        const int jm = wrap_lo(j - 1, NY), jp = wrap_hi(j + 1, NY);
        const int c = nc[n], c0 = nc[(long long)im * NY + j], c1 = nc[(long long)ip * NY + j];
        const int c2 = nc[(long long)i * NY + jm], c3 = nc[(long long)i * NY + jp];
        const unsigned long long n0 = I.rho[0][n], n1 = I.rho[1][n];
        const uint8_t fixed = I.lev[0].fix[n];
        const double v0 = V[c0], v1 = V[c1], v2 = V[c2], v3 = V[c3];
        if (c) {
            I.b[n] = V[c];
            I.phi[n] = V[c];
        } else {
            long long Ni = (long long)n1;
            if (I.charge_mode == 2 && i == I.charge_row) {
                const int jl = g.py ? wrap_lo(j - 1, g.ny) : j - 1;
                if (j < g.ny) Ni += (long long)I.surf[j] << 31;
                if (jl >= 0) Ni += (long long)I.surf[jl] << 31;
            }
            double r = (double)(Ni - (long long)n0) * I.qcharge;
            if (I.charge_mode == 1 && i == I.charge_row && j >= I.sjl && j <= I.sjh) r += I.sden;
            r = c0 ? r + v0 : r;
            r = c1 ? r + v1 : r;
            r = c2 ? r + v2 : r;
            r = c3 ? r + v3 : r;
            I.b[n] = r;
            if (!fixed) bb = r * r;
            sm = r;
        }
    }
    double v[2] = {bb, sm};
    block_partials<2>(v, pt);
}

void launch_assemble(const Inst *I, const Tab &t, const double *Vtab, const long long *ctl,
                     int ninst, int vwin, Part pt, hipStream_t s)
{
    if (!t.n) return;
    hipLaunchKernelGGL(k_assemble, dim3(tab_blocks(t)), gblock(), 0, s, I, t, Vtab, ctl, ninst, vwin,
                       pt);
    finalize(I, t, pt, OP_ASM, s);
}

// Fully periodic grid: the source must have zero mean (gauge); subtract it
// and form ||b||^2 over the unknowns (the pinned node excluded).
__global__ void k_project_mean(const Inst *insts, Tab t, Part pt)
{
    GRID_BEGIN(t)
    NODE_IDX(I.g.NX, I.g.NY)
    const double mean = I.S[S_SUM] / ((double)NX * (double)NY);
    double bb = 0.0;
    if (inb) {
        const double r = I.b[n] - mean;
        I.b[n] = r;
        if (!I.lev[0].fix[n]) bb = r * r;
    }
    double v[1] = {bb};
    block_partials<1>(v, pt);
}

void launch_project_mean(const Inst *I, const Tab &t, Part pt, hipStream_t s)
{
    if (!t.n) return;
    hipLaunchKernelGGL(k_project_mean, dim3(tab_blocks(t)), gblock(), 0, s, I, t, pt);
    finalize(I, t, pt, OP_BB_PER, s);
}

__global__ void k_sum_phi(const Inst *insts, Tab t, Part pt)
{
    GRID_BEGIN(t)
    NODE_IDX(I.g.NX, I.g.NY)
    double v[1] = {inb ? I.phi[n] : 0.0};
    block_partials<1>(v, pt);
}

// phi -= S[slot] * (mean ? 1 / (NX NY) : 1) on every node
__global__ void k_shift_phi(const Inst *insts, Tab t, int slot, int mean)
{
    GRID_BEGIN(t)
    NODE_IDX(I.g.NX, I.g.NY)
    const double sc = mean ? 1.0 / ((double)NX * (double)NY) : 1.0;
    if (inb) I.phi[n] -= I.S[slot] * sc;
}

__global__ void k_read_node0(const Inst *insts, Tab t)
{
    const Inst &I = insts[t.id[blockIdx.x]];
    I.S[S_PIN] = I.phi[0];
}

void launch_shift_mean(const Inst *I, const Tab &t, Part pt, hipStream_t s)
{
    if (!t.n) return;
    hipLaunchKernelGGL(k_sum_phi, dim3(tab_blocks(t)), gblock(), 0, s, I, t, pt);
    finalize(I, t, pt, OP_SUM, s);
    hipLaunchKernelGGL(k_shift_phi, dim3(tab_blocks(t)), gblock(), 0, s, I, t, (int)S_SUM, 1);
}

// Fully periodic grid: node 0 is held at 0 during the solve (gauge); shift a
// start so that it already satisfies that.
void launch_pin_shift(const Inst *I, const Tab &t, hipStream_t s)
{
    if (!t.n) return;
    hipLaunchKernelGGL(k_read_node0, dim3(t.n), dim3(1), 0, s, I, t);
    hipLaunchKernelGGL(k_shift_phi, dim3(tab_blocks(t)), gblock(), 0, s, I, t, (int)S_PIN, 0);
}

// Start of the solve on the unknowns; on a fully periodic grid also on the
// pinned node (the gauge shift that follows moves it back to 0).  kind 0:
// zero; kind 2: copy from guess (single-unit launches only).
__global__ void k_set_guess(const Inst *insts, Tab t, int kind, const double *guess)
{
    GRID_BEGIN(t)
    NODE_IDX(I.g.NX, I.g.NY)
    if (!inb || (I.lev[0].fix[n] && !(I.g.px && I.g.py))) return;
    I.phi[n] = (kind == 0) ? 0.0 : guess[n];
}

void launch_set_guess(const Inst *I, const Tab &t, int kind, const double *guess, hipStream_t s)
{
    if (t.n) hipLaunchKernelGGL(k_set_guess, dim3(tab_blocks(t)), gblock(), 0, s, I, t, kind, guess);
}

// Linear extrapolation in time of the unknowns: phi <- 2 phi - prev and
// prev <- phi (the previous step's solution); with have_prev = 0 only the
// copy is made.
__global__ void k_extrapolate(const Inst *insts, Tab t, int have_prev)
{
    GRID_BEGIN(t)
    NODE_IDX(I.g.NX, I.g.NY)
    if (!inb) return;
    const uint8_t fixed = I.lev[0].fix[n];
    const double v = I.phi[n], u = have_prev ? I.phi_prev[n] : 0.0;
    if (fixed && !(I.g.px && I.g.py)) return;
    if (have_prev) I.phi[n] = 2.0 * v - u;
    I.phi_prev[n] = v;
}

void launch_extrapolate(const Inst *I, const Tab &t, int have_prev, hipStream_t s)
{
    if (t.n) hipLaunchKernelGGL(k_extrapolate, dim3(tab_blocks(t)), gblock(), 0, s, I, t, have_prev);
}

// ---------------------------------------------------------------------------
// float64 outer residual: r = b - A phi on the unknowns, ||r||^2 (float64),
// r rounded to float32 for the inner preconditioned CG; at the start of a
// solve also ||b||^2 over the unknowns (the reference of the tolerance).
// A = 4 - (sum of free neighbours); fixed neighbours sit in b already.
// ---------------------------------------------------------------------------

__global__ void k_resid64(const Inst *insts, Tab t, int after_pass, Part pt)
{
    GRID_BEGIN(t)
    if (after_pass && (I.F[F_SKIP] || I.F[F_CGABORT])) return;
    NODE_IDX(I.g.NX, I.g.NY)
    const uint8_t *fix = I.lev[0].fix;
    const double *phi = I.phi;
    double rr = 0.0, bsq = 0.0;
    if (inb) {
        // all loads at once (a neighbour's potential behind the test of its mask, four in turn: 5.7 us at 257 x 257)
        const int im = wrap_lo(i - 1, NX), ip = wrap_hi(i + 1, NX);
        const int jm = wrap_lo(j - 1, NY), jp = wrap_hi(j + 1, NY);
        const long long a = (long long)im * NY + j, c = (long long)ip * NY + j;
        const long long d = (long long)i * NY + jm, e = (long long)i * NY + jp;
        const uint8_t fn = fix[n], fa = fix[a], fc = fix[c], fd = fix[d], fe = fix[e];
        const double pn = phi[n], pa = phi[a], pc = phi[c], pd = phi[d], pe = phi[e], b = I.b[n];
        double s = 4.0 * pn;
        s = fa ? s : s - pa;
        s = fc ? s : s - pc;
        s = fd ? s : s - pd;
        s = fe ? s : s - pe;
        const double r = fn ? 0.0 : b - s;
        I.lev[0].g[n] = (float)r;
        bsq = fn ? 0.0 : b * b;
        rr = r * r;
    }
    double v[2] = {rr, bsq};
    block_partials<2>(v, pt);
}

void launch_resid64(const Inst *I, const Tab &t, int after_pass, Part pt, hipStream_t s)
{
    if (!t.n) return;
    hipLaunchKernelGGL(k_resid64, dim3(tab_blocks(t)), gblock(), 0, s, I, t, after_pass, pt);
    finalize(I, t, pt, after_pass ? OP_RR64_PASS : OP_RR64_START, s);
}

// ---------------------------------------------------------------------------
// the paper's own iterations for eq. (5) (Sec. II): Jacobi and Gauss-Seidel
// sweeps of the masked 5-point system in float64.  A free node takes
// (b + sum of its free neighbours) / 4 with the neighbours added in the order
// x-1, x+1, y-1, y+1 (fixed neighbours' potentials sit in b); Gauss-Seidel
// visits the red nodes (i + j even), then the black ones.  An instance whose
// float64 residual already met rtol is left alone.
// ---------------------------------------------------------------------------

__device__ __forceinline__ double sweep_value(const double *src, const double *b, const uint8_t *fix, int i,
                                              int j, int NX, int NY, long long n)
{
    const int im = wrap_lo(i - 1, NX), ip = wrap_hi(i + 1, NX);
    const int jm = wrap_lo(j - 1, NY), jp = wrap_hi(j + 1, NY);
    const long long a = (long long)im * NY + j, c = (long long)ip * NY + j;
    const long long d = (long long)i * NY + jm, e = (long long)i * NY + jp;
    double s = b[n];
    if (!fix[a]) s += src[a];
    if (!fix[c]) s += src[c];
    if (!fix[d]) s += src[d];
    if (!fix[e]) s += src[e];
    return s * 0.25;
}

// One Jacobi sweep: dir 0 reads phi and writes phi2, dir 1 the reverse.
__global__ void k_jacobi64(const Inst *insts, Tab t, int dir)
{
    GRID_BEGIN(t)
    if (I.F[F_CONV]) return;
    NODE_IDX(I.g.NX, I.g.NY)
    if (!inb) return;
    const double *src = dir ? I.phi2 : I.phi;
    double *dst = dir ? I.phi : I.phi2;
    const uint8_t *fix = I.lev[0].fix;
    dst[n] = fix[n] ? src[n] : sweep_value(src, I.b, fix, i, j, NX, NY, n);
}

// One colour of a red-black Gauss-Seidel sweep, in place.
__global__ void k_gs64(const Inst *insts, Tab t, int col)
{
    GRID_BEGIN(t)
    if (I.F[F_CONV]) return;
    NODE_IDX(I.g.NX, I.g.NY)
    if (!inb || ((i + j) & 1) != col) return;
    const uint8_t *fix = I.lev[0].fix;
    if (!fix[n]) I.phi[n] = sweep_value(I.phi, I.b, fix, i, j, NX, NY, n);
}

void launch_sweeps(const Inst *I, const Tab &t, int jacobi, int sweeps, hipStream_t s)
{
    if (!t.n) return;
    for (int k = 0; k < sweeps; k++) {
        if (jacobi) {
            hipLaunchKernelGGL(k_jacobi64, dim3(tab_blocks(t)), gblock(), 0, s, I, t, k & 1);
        } else {
            hipLaunchKernelGGL(k_gs64, dim3(tab_blocks(t)), gblock(), 0, s, I, t, 0);
            hipLaunchKernelGGL(k_gs64, dim3(tab_blocks(t)), gblock(), 0, s, I, t, 1);
        }
    }
}

__global__ void k_phi_update(const Inst *insts, Tab t)
{
    GRID_BEGIN(t)
    if (I.F[F_SKIP] || I.F[F_CGABORT]) return;
    NODE_IDX(I.g.NX, I.g.NY)
    if (!inb) return;
    const uint8_t fixed = I.lev[0].fix[n];
    const double sum = I.phi[n] + (double)I.e[n];
    if (!fixed) I.phi[n] = sum;
}

void launch_phi_update(const Inst *I, const Tab &t, hipStream_t s)
{
    if (t.n) hipLaunchKernelGGL(k_phi_update, dim3(tab_blocks(t)), gblock(), 0, s, I, t);
}

// ---------------------------------------------------------------------------
// multigrid pieces on any level (generic pointers: global or LDS)
//   stencil per level: 4u - sum(free neighbours) = g   (h^2 folded into g)
//   restriction g_c = P^T r (weights 1, 1/2, 1/4), prolongation bilinear P,
//   red-black Gauss-Seidel: pre red->black, post black->red (symmetric)
// ---------------------------------------------------------------------------

struct Nb {
    int im, ip, jm, jp;
};

__device__ __forceinline__ Nb nbs(int i, int j, int NX, int NY)
{
    Nb r;
    r.im = wrap_lo(i - 1, NX);
    r.ip = wrap_hi(i + 1, NX);
    r.jm = wrap_lo(j - 1, NY);
    r.jp = wrap_hi(j + 1, NY);
    return r;
}

// Bilinear prolongation of the coarse correction e at a red fine node
// (both indices even: coincident node; both odd: cell centre).
__device__ __forceinline__ float prolong_red(const float *e, int NXc, int NYc, int a, int c)
{
    int I = a >> 1, J = c >> 1;
    if (((a | c) & 1) == 0) return e[(long long)I * NYc + J];
    int I1 = wrap_hi(I + 1, NXc), J1 = wrap_hi(J + 1, NYc);
    return 0.25f * (e[(long long)I * NYc + J] + e[(long long)I1 * NYc + J] +
                    e[(long long)I * NYc + J1] + e[(long long)I1 * NYc + J1]);
}

// ---------------------------------------------------------------------------
// preconditioned CG on level 0 (float32 vectors, float64 dot products)
// ---------------------------------------------------------------------------

// Inner start: e = 0, z = red-from-zero of M r (or z = r/4 without MG),
// ||r||^2 and r.z partials.  Skipped once the float64 residual converged.
__global__ void k_init_red0(const Inst *insts, Tab t, Part pt)
{
    GRID_BEGIN(t)
    if (I.F[F_CONV]) return;
    const LevelDev L = I.lev[0];
    NODE_IDX(L.NX, L.NY)
    const int mg = I.mg;
    double rr = 0.0, rz = 0.0;
    if (inb) {
        const float r = L.g[n];
        I.e[n] = 0.0f;
        float z = 0.0f;
        if (!L.fix[n]) {
            rr = (double)r * (double)r;
            if (!mg || (((i + j) & 1) == 0)) z = r * 0.25f;
            rz = (double)r * (double)z;
        }
        L.u[n] = z;
    }
    double v[2] = {rr, rz};
    block_partials<2>(v, pt);
}

void launch_init_red0(const Inst *I, const Tab &t, Part pt, hipStream_t s)
{
    if (!t.n) return;
    hipLaunchKernelGGL(k_init_red0, dim3(tab_blocks(t)), gblock(), 0, s, I, t, pt);
    finalize(I, t, pt, OP_INIT, s);
}

// p_new = z + beta p_old, q = A p_new, p.q  (beta = rz / rz_old; 0 on the first)
__global__ void k_pupdate_Ap(const Inst *insts, Tab t, int kold, int first, Part pt)
{
    GRID_BEGIN(t)
    if (I.F[F_DONE]) return;
    const LevelDev L = I.lev[0];
    NODE_IDX(L.NX, L.NY)
    const float *p_old = I.p[kold];
    float *p_new = I.p[1 - kold];
    float *q = I.q;
    const float beta = first ? 0.0f : (float)(I.S[S_RZ] / I.S[S_RZOLD]);
    double pq = 0.0;
    if (inb) {
        if (L.fix[n]) {
            p_new[n] = 0.0f;
            q[n] = 0.0f;
        } else {
            Nb b = nbs(i, j, NX, NY);
            const long long m[4] = {(long long)b.im * NY + j, (long long)b.ip * NY + j,
                                    (long long)i * NY + b.jm, (long long)i * NY + b.jp};
            const float *z = I.z;
            const float pc = first ? z[n] : z[n] + beta * p_old[n];
            float s = 4.0f * pc;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                if (L.fix[m[k]]) continue;
                const float pn = first ? z[m[k]] : z[m[k]] + beta * p_old[m[k]];
                s -= pn;
            }
            p_new[n] = pc;
            q[n] = s;
            pq = (double)pc * (double)s;
        }
    }
    double v[1] = {pq};
    block_partials<1>(v, pt);
}

void launch_pupdate_Ap(const Inst *I, const Tab &t, int kold, int first, Part pt, hipStream_t s)
{
    if (!t.n) return;
    hipLaunchKernelGGL(k_pupdate_Ap, dim3(tab_blocks(t)), gblock(), 0, s, I, t, kold, first, pt);
    finalize(I, t, pt, OP_PQ, s);
}

// alpha = rz / pq; e += alpha p; r -= alpha q; ||r||^2; z = red-from-zero of
// M r (or r/4 without MG, with r.z).  The finalize marks the inner solve
// done when ||r||^2 <= eta^2 ||r0||^2 and counts the iteration.
__global__ void k_update_red0(const Inst *insts, Tab t, int knew, Part pt)
{
    GRID_BEGIN(t)
    if (I.F[F_DONE]) return;
    const LevelDev L = I.lev[0];
    NODE_IDX(L.NX, L.NY)
    const int mg = I.mg;
    const float *p = I.p[knew];
    const float alpha = (float)(I.S[S_RZ] / I.S[S_PQ]);
    double rr = 0.0, rz = 0.0;
    if (inb) {
        float z = 0.0f;
        if (!L.fix[n]) {
            I.e[n] = I.e[n] + alpha * p[n];
            const float r = L.g[n] - alpha * I.q[n];
            L.g[n] = r;
            rr = (double)r * (double)r;
            if (!mg || (((i + j) & 1) == 0)) z = r * 0.25f;
            rz = (double)r * (double)z;
        }
        L.u[n] = z;
    }
    double v[2] = {rr, rz};
    block_partials<2>(v, pt);
}

void launch_update_red0(const Inst *I, const Tab &t, int knew, Part pt, hipStream_t s)
{
    if (!t.n) return;
    hipLaunchKernelGGL(k_update_red0, dim3(tab_blocks(t)), gblock(), 0, s, I, t, knew, pt);
    finalize(I, t, pt, OP_UPDATE, s);
}

// ---------------------------------------------------------------------------
// fused V-cycle kernels for the fine levels, one block per 32 x 32 tile of the
// fine level (launch table: tiles, bx = tiles across y).  Each block stages a
// window of u, g and the mask around its tile in LDS (periodic axes wrap, nodes
// outside a bounded axis enter as fixed), recomputes in the window what it
// needs, and writes only its own tile (or its own coarse nodes).  Each
// launch reads one buffer of the level and writes the other, so no block sees
// another block's writes:
//   down: u (red-from-zero start) -> pre-smoothing (black, then red + black
//         NU - 1 times) -> uo, and the restricted residual to level l + 1
//   up:   uo -> black update with the prolonged coarse correction, then red,
//         then black + red NU - 1 times -> u (on level 0 the CG's z, with
//         the r.z partials)
// The post-smoothing is the pre-smoothing's colour sequence reversed, which
// keeps the V-cycle symmetric.
// Arithmetic per node: Gauss-Seidel value (g + neighbours) / 4 with the
// neighbours added in the order x-1, x+1, y-1, y+1; restriction = sum over
// the red fine nodes of the 3 x 3 stencil of weight x residual (centre 1,
// diagonals 1/4; the black residuals vanish after a black half-sweep);
// bilinear prolongation of the coarse correction onto the red nodes.
// ---------------------------------------------------------------------------

constexpr int kMgTile = 32;
constexpr int kMgThreads = 512;

// x modulo n.  A window reaches past a periodic axis once at most unless the
// level is smaller than the window: the two divisions (of run-time numbers,
// 80 instructions a node) are for those levels only.
__device__ __forceinline__ int wrap_any(int x, int n)
{
    x += x < 0 ? n : 0;
    x -= x >= n ? n : 0;
    if ((unsigned)x >= (unsigned)n) x = ((x % n) + n) % n;
    return x;
}

// Window index (wi0 + a, wj0 + c) -> global node of level (NX, NY), or -1
// outside a bounded axis.
__device__ __forceinline__ long long win_node(int NX, int NY, int px, int py, int gi, int gj)
{
    if (px) gi = wrap_any(gi, NX);
    else if (gi < 0 || gi >= NX) return -1;
    if (py) gj = wrap_any(gj, NY);
    else if (gj < 0 || gj >= NY) return -1;
    return (long long)gi * NY + gj;
}

// u (from src), g, fix of the W x W window with origin (wi0, wj0) on level L,
// to LDS.  Fixed nodes hold u = 0 on every level (no update ever writes them),
// so the stencils below add neighbours without testing their mask.  A launch
// of these kernels is a chain of trips to memory (what it reads was written by
// other kernels, mostly on other dies), so a kernel issues every load before it
// waits for any, the flag that may end it included (257 x 257 nodes, with each
// part's loads after the one before: 10.3, 5.8, 5.9 and 7.2 us for the level-0
// and level-1 down and the level-1 and level-0 up kernels; now 8.0, 5.0, 4.6
// and 6.2).  In a context of several instances (many), of which some have
// finished, the flag comes first: loading for nothing cost a batch of six more
// (8.5 -> 13.1 us for the level-0 down kernel) than the trip it saves, and a
// batch of one multigrid instance beside plain-CG ones 10 % of its solve.
// (many comes before the tables in a launch's arguments: behind them it is a
// trip for another line, 1 % of a step at 257 x 257 nodes.)
template <int W, int NT = kMgThreads> struct Window {
    static constexpr int R = (W * W + NT - 1) / NT;
    float uv[R], gv[R];
    uint8_t fv[R];

    __device__ __forceinline__ void load(const LevelDev &L, const float *src, const float *gsrc, int px, int py,
                                         int wi0, int wj0)
    {
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int k = (int)threadIdx.x + r * NT;
            const int a = k / W, c = k - a * W;
            const long long n = k < W * W ? win_node(L.NX, L.NY, px, py, wi0 + a, wj0 + c) : -1;
            uv[r] = 0.0f;
            gv[r] = 0.0f;
            fv[r] = 1;
            if (n >= 0) {
                fv[r] = L.fix[n];
                uv[r] = src[n];
                gv[r] = gsrc[n];
            }
        }
    }
    __device__ __forceinline__ void store(float *su, float *sg, uint8_t *sf) const
    {
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int k = (int)threadIdx.x + r * NT;
            if (k < W * W) {
                su[k] = uv[r];
                sg[k] = gv[r];
                sf[k] = fv[r];
            }
        }
    }
};

// The prolonged coarse correction e at the window's red nodes (their mask is
// tested where it is used).
template <int W, int NT = kMgThreads> struct Prolonged {
    static constexpr int R = (W * W + NT - 1) / NT;
    float e[R][4];
    unsigned one;                      // bit r: a red node of both even indices, which lies on a coarse node

    __device__ __forceinline__ void load(const LevelDev &L, const LevelDev &C, int px, int py, int wi0, int wj0)
    {
        const float *u = C.u;
        one = 0;
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int k = (int)threadIdx.x + r * NT;
            const int a = k / W, c = k - a * W;
            int gi = wi0 + a, gj = wj0 + c;
            if (px) gi = wrap_any(gi, L.NX);
            if (py) gj = wrap_any(gj, L.NY);
            const bool in = k < W * W && ((a + c) & 1) == 0 && gi >= 0 && gi < L.NX && gj >= 0 && gj < L.NY;
            const int I = in ? gi >> 1 : 0, J = in ? gj >> 1 : 0;
            const int I1 = wrap_hi(I + 1, C.NX), J1 = wrap_hi(J + 1, C.NY);
            e[r][0] = u[(long long)I * C.NY + J];
            e[r][1] = u[(long long)I1 * C.NY + J];
            e[r][2] = u[(long long)I * C.NY + J1];
            e[r][3] = u[(long long)I1 * C.NY + J1];
            if (((gi | gj) & 1) == 0) one |= 1u << r;
        }
    }
    // sc = su + the correction at the red nodes that are not fixed, else 0
    __device__ __forceinline__ void add(const float *su, const uint8_t *sf, float *sc) const
    {
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int k = (int)threadIdx.x + r * NT;
            const int a = k / W, c = k - a * W;
            const float m = 0.25f * (e[r][0] + e[r][1] + e[r][2] + e[r][3]);
            if (k < W * W) sc[k] = ((a + c) & 1) == 0 && !sf[k] ? su[k] + ((one >> r) & 1 ? e[r][0] : m) : 0.0f;
        }
    }
};

// Level 0 of the inner CG (Chronopoulos-Gear form): the residual after this
// iteration's update, r - alpha (w + beta s), as g and its red-from-zero start
// as u.  With `update` false the residual is r itself (start of a pass).
// Every block evaluates the same float32 expression for a node, so window
// copies agree with the owner's stored values.  load() also reads the own
// nodes' w, s, z, p and e.
template <int W> struct Window0 {
    static constexpr int R = (W * W + kMgThreads - 1) / kMgThreads, O = kMgTile * kMgTile / kMgThreads;
    float rv[R], s_[R], w_[R], ow[O], os[O], oz[O], op[O], oe[O];
    uint8_t fv[R];

    __device__ __forceinline__ void load(const Inst &I, int update, const float *r, const float *sv, int i0, int j0,
                                         int HD)
    {
        const LevelDev &L = I.lev[0];
        const float *wv = I.cg_w, *z = I.z, *p = I.p[0], *e = I.e;
#pragma unroll
        for (int q = 0; q < R; q++) {
            const int k = (int)threadIdx.x + q * kMgThreads;
            const int a = k / W, c = k - a * W;
            const long long n =
                k < W * W ? win_node(L.NX, L.NY, I.g.px, I.g.py, i0 - HD + a, j0 - HD + c) : -1;
            rv[q] = 0.0f;
            s_[q] = 0.0f;
            w_[q] = 0.0f;
            fv[q] = 1;
            if (n >= 0) {
                fv[q] = L.fix[n];
                rv[q] = r[n];
                if (update) {
                    w_[q] = wv[n];
                    s_[q] = sv[n];
                }
            }
        }
        if (!update) return;
#pragma unroll
        for (int q = 0; q < O; q++) {
            const int k = (int)threadIdx.x + q * kMgThreads;
            const int gi = i0 + k / kMgTile, gj = j0 + k % kMgTile;
            if (gi < L.NX && gj < L.NY) {
                const long long n = (long long)gi * L.NY + gj;
                ow[q] = wv[n];
                os[q] = sv[n];
                oz[q] = z[n];
                op[q] = p[n];
                oe[q] = e[n];
            }
        }
    }
    // first: beta = 0, s holds an earlier pass
    __device__ __forceinline__ void store(int update, int first, float alpha, float beta, float *su, float *sg,
                                          uint8_t *sf) const
    {
#pragma unroll
        for (int q = 0; q < R; q++) {
            const int k = (int)threadIdx.x + q * kMgThreads;
            if (k >= W * W) continue;
            const int a = k / W, c = k - a * W;
            float rn = 0.0f;
            if (!fv[q]) {
                rn = rv[q];
                if (update) {
                    const float sn = first ? w_[q] : w_[q] + beta * s_[q];
                    rn = rn - alpha * sn;
                }
            }
            sg[k] = rn;
            su[k] = (((a + c) & 1) == 0) ? rn * 0.25f : 0.0f;
            sf[k] = fv[q];
        }
    }
};

// Gauss-Seidel value at window node k (neighbours in the window; fixed
// neighbours contribute their zero).
template <int W>
__device__ __forceinline__ float win_gs(const float *su, const float *sg, int k)
{
    float s = sg[k];
    s += su[k - W];
    s += su[k + W];
    s += su[k - 1];
    s += su[k + 1];
    return s * 0.25f;
}

// One colour of Gauss-Seidel over window rows/cols m .. W-1-m.  The window
// origin is an even offset from an even tile corner, so (a + c) & 1 is the
// colour of the global node.
template <int W, int NT = kMgThreads>
__device__ __forceinline__ void win_sweep(float *su, const float *sg, const uint8_t *sf, int m, int col)
{
    for (int k = threadIdx.x; k < W * W; k += NT) {
        const int a = k / W, c = k - a * W;
        if (a < m || a > W - 1 - m || c < m || c > W - 1 - m || sf[k]) continue;
        if (((a + c) & 1) != col) continue;
        su[k] = win_gs<W>(su, sg, k);
    }
}

__host__ __device__ constexpr int pad16(int b) { return (b + 15) & ~15; }
__host__ __device__ constexpr int win_lds(int W) { return pad16(3 * W * W * 4) + pad16(W * W); }
// Window arrays at byte offset off: u, g, scratch (float) and the mask.
struct WinLds {
    float *u, *g, *r;
    uint8_t *f;
};
__device__ __forceinline__ WinLds win_at(unsigned char *lds, int off, int W)
{
    WinLds w;
    w.u = (float *)(lds + off);
    w.g = w.u + W * W;
    w.r = w.g + W * W;
    w.f = (uint8_t *)(lds + off + pad16(3 * W * W * 4));
    return w;
}

constexpr int kMgSmooth = 1;     // pre- and post-smoothing steps on the fine levels

// Pre-smoothing of a window from its red-from-zero start.
template <int NU, int W, int NT>
__device__ __forceinline__ void pre_smooth(float *su, const float *sg, const uint8_t *sf)
{
#pragma unroll
    for (int m = 1; m < 2 * NU; m++) {
        win_sweep<W, NT>(su, sg, sf, m, m & 1);           // odd m: black, even m: red
        __syncthreads();
    }
}

// Own nodes (both colours) to uo; residuals at the red nodes the restriction
// reads (window rows/cols 2NU .. W-1-2NU).
template <int NU, int W, int NT>
__device__ __forceinline__ void down_residuals(const LevelDev &F, int i0, int j0, const float *su, const float *sg,
                                               const uint8_t *sf, float *sr)
{
    constexpr int HD = 2 * NU + 1;
    float *uo = F.uo;
    for (int k = threadIdx.x; k < kMgTile * kMgTile; k += NT) {
        const int a = k / kMgTile, c = k - a * kMgTile;
        const int gi = i0 + a, gj = j0 + c;
        if (gi >= F.NX || gj >= F.NY) continue;
        uo[(long long)gi * F.NY + gj] = su[(a + HD) * W + (c + HD)];
    }
    for (int k = threadIdx.x; k < W * W; k += NT) {
        const int a = k / W, c = k - a * W;
        if (a < 2 * NU || a > W - 1 - 2 * NU || c < 2 * NU || c > W - 1 - 2 * NU) continue;
        if (((a + c) & 1) != 0) continue;
        float r = 0.0f;
        if (!sf[k]) {
            float q = 4.0f * su[k];
            q -= su[k - W];
            q -= su[k + W];
            q -= su[k - 1];
            q -= su[k + 1];
            r = sg[k] - q;
        }
        sr[k] = r;
    }
}

// Restriction to coarse node (CI, CJ), which lies on window node k.
template <int W>
__device__ __forceinline__ void restrict_node(const LevelDev &C, int CI, int CJ, int fixed, const float *sr, int k)
{
    const long long n = (long long)CI * C.NY + CJ;
    float gv = 0.0f, uv = 0.0f;
    if (!fixed) {
        float acc = 0.0f;
        acc += 0.25f * sr[k - W - 1];
        acc += 0.25f * sr[k - W + 1];
        acc += 1.0f * sr[k];
        acc += 0.25f * sr[k + W - 1];
        acc += 0.25f * sr[k + W + 1];
        gv = acc;
        if (((CI + CJ) & 1) == 0) uv = gv * 0.25f;
    }
    C.g[n] = gv;
    C.u[n] = uv;
}

// Down half-cycle of level l >= 1 (start staged from u) on its 32 x 32 tile
// (ti, tj) with NU pre-smoothing steps: from the red-from-zero start, black,
// then (red, black) x (NU - 1); the pre-smoothed level goes to uo, the
// restricted residual to level l + 1 (g, and u = its red-from-zero start).
template <int NU, int NT>
__device__ __forceinline__ void mg_down_fine(const Inst &I, int level, int ti, int tj, int done, unsigned char *lds)
{
    constexpr int HD = 2 * NU + 1, W = kMgTile + 2 * HD - 1;
    const LevelDev F = I.lev[level], C = I.lev[level + 1];
    const int i0 = ti * kMgTile, j0 = tj * kMgTile;
    const WinLds f = win_at(lds, 0, W);
    const int rci = (int)threadIdx.x >> 4, rcj = threadIdx.x & 15;   // coarse node of the restriction
    const int CI = (i0 >> 1) + rci, CJ = (j0 >> 1) + rcj;
    const bool coarse = threadIdx.x < 256 && CI < C.NX && CJ < C.NY;
    const uint8_t cfix = C.fix[coarse ? (long long)CI * C.NY + CJ : 0];
    Window<W, NT> win;
    win.load(F, F.u, F.g, I.g.px, I.g.py, i0 - HD, j0 - HD);
    if (uniform(done)) return;
    win.store(f.u, f.g, f.f);
    __syncthreads();
    pre_smooth<NU, W, NT>(f.u, f.g, f.f);
    down_residuals<NU, W, NT>(F, i0, j0, f.u, f.g, f.f, f.r);
    __syncthreads();
    if (coarse) restrict_node<W>(C, CI, CJ, cfix, f.r, (2 * rci + HD) * W + (2 * rcj + HD));
}

// The same of level 0.
// MODE 1: at the start of an inner pass: r = R[0], e = 0, ||r||^2 partials (pt;
//         k_finalize makes the inner stop ratio and clears the counters).
// MODE 2: a CG step: alpha and beta from the last V-cycle's dot products
//         (partials pq), s' = w + beta s, r' = r - alpha s', p = z + beta p,
//         e += alpha p (beta = 0 on the first step), r' and s' to the other
//         buffers of the pair, ||r'||^2 partials (pt), which k_coarse adds for
//         the inner stop test.  par: buffer of the pair holding r and s.
template <int NU, int MODE>
__global__ __launch_bounds__(kMgThreads, 8) void k_mg_down(const Inst *insts, int many, Tab t, int par, Part pt, Part pq)
{
    constexpr int HD = 2 * NU + 1, W = kMgTile + 2 * HD - 1;
    const int ku = unit_of(t, (int)blockIdx.x);
    const Inst &I = insts[t.id[ku]];
    int *F = I.F;
    double *S = I.S;
    const int lb = (int)blockIdx.x - t.boff[ku];
    const int ti = lb / t.bx[ku], tj = lb - ti * t.bx[ku];
    const LevelDev F0 = I.lev[0], Cc = I.lev[1];
    const int i0 = ti * kMgTile, j0 = tj * kMgTile;
    __shared__ float su[W * W], sg[W * W], sr[W * W];
    __shared__ uint8_t sf[W * W];
    double rr = 0.0;
    Window0<W> win0;
    const float *r = par ? I.cg_r1 : F0.g;
    if (MODE == 2 && many && F[F_DONE]) return;
    const int stop = vload(F, MODE == 1 ? F_CONV : F_DONE);
    PartialSums<3> ps;
    if (MODE == 2) ps.load(pq, t.boff[ku], t.boff[ku + 1], 2, (int)threadIdx.x);
    const int iter = MODE == 2 ? vload(F, F_ITER) : 0;
    const double g_old = MODE == 2 ? vload(S, S_CG_GAMMA) : 0.0, a_old = MODE == 2 ? vload(S, S_CG_ALPHA) : 0.0;
    const int rci = (int)threadIdx.x >> 4, rcj = threadIdx.x & 15;   // coarse node of the restriction
    const int CI = (i0 >> 1) + rci, CJ = (j0 >> 1) + rcj;
    const bool coarse = threadIdx.x < 256 && CI < Cc.NX && CJ < Cc.NY;
    const uint8_t cfix = Cc.fix[coarse ? (long long)CI * Cc.NY + CJ : 0];
    win0.load(I, MODE == 2, r, I.cg_s[par], i0, j0, HD);
    float alpha = 0.0f, beta = 0.0f;
    int first = 1;
    if (MODE == 2) {
        // this step's alpha and beta from the last V-cycle's r.z and (A z).z
        // partials (pq): every block adds them in the same order, so all
        // blocks agree.  Block 0 records them for the step's update, which
        // also ends the inner solve when they are not usable (no block of
        // this launch writes a flag the others read).
        __shared__ double shq[2][4];
        if (uniform(stop)) return;
        ps.sum(pq, t.boff[ku], t.boff[ku + 1], 2, shq, (int)threadIdx.x);
        __syncthreads();
        const double gamma = shq[0][0] + shq[0][1] + shq[0][2] + shq[0][3];
        const double delta = shq[1][0] + shq[1][1] + shq[1][2] + shq[1][3];
        double a, b;
        const bool ok = cg_coefficients(iter, gamma, delta, g_old, a_old, a, b);
        if (lb == 0 && threadIdx.x == 0) {
            S[S_CG_NALPHA] = a;
            S[S_CG_NBETA] = b;
            S[S_CG_NGAMMA] = gamma;
        }
        if (!ok) return;
        alpha = (float)a;
        beta = (float)b;
        first = iter == 0;
    }
    if (MODE != 1 || !uniform(stop)) {
        win0.store(MODE == 2, first, alpha, beta, su, sg, sf);
        __syncthreads();
        // own tile: the vector updates and ||r'||^2 (reads the window only)
        float *rn_out = par ? F0.g : I.cg_r1;
        float *sn_out = I.cg_s[1 - par], *p_out = I.p[0], *e_out = I.e;
#pragma unroll
        for (int q = 0; q < kMgTile * kMgTile / kMgThreads; q++) {
            const int k = (int)threadIdx.x + q * kMgThreads;
            const int a = k / kMgTile, c = k - a * kMgTile;
            const int gi = i0 + a, gj = j0 + c;
            if (gi >= F0.NX || gj >= F0.NY) continue;
            const long long n = (long long)gi * F0.NY + gj;
            const int w = (a + HD) * W + (c + HD);
            if (MODE == 1) {
                e_out[n] = 0.0f;
            } else if (!sf[w]) {
                const float pn = first ? win0.oz[q] : win0.oz[q] + beta * win0.op[q];
                const float sn = first ? win0.ow[q] : win0.ow[q] + beta * win0.os[q];
                p_out[n] = pn;
                e_out[n] = win0.oe[q] + alpha * pn;
                sn_out[n] = sn;
                rn_out[n] = sg[w];
            } else {
                p_out[n] = 0.0f;
                sn_out[n] = 0.0f;
                rn_out[n] = 0.0f;
            }
            if (!sf[w]) rr += (double)sg[w] * (double)sg[w];
        }
        pre_smooth<NU, W, kMgThreads>(su, sg, sf);
        down_residuals<NU, W, kMgThreads>(F0, i0, j0, su, sg, sf, sr);
        __syncthreads();
        if (coarse) restrict_node<W>(Cc, CI, CJ, cfix, sr, (2 * rci + HD) * W + (2 * rcj + HD));
    }
    double v[1] = {rr};
    block_partials<1>(v, pt);
}

// Post-smoothing of a window: black from the corrected reds sc, then red, then
// (black, red) x (NU - 1), without the last red half-sweep unless it covers
// the tile's ring (L0).
template <int NU, int L0, int W, int NT>
__device__ __forceinline__ void post_smooth(float *su, const float *sg, const float *sc, const uint8_t *sf)
{
    // black update over window rows/cols 1 .. W-2 from the corrected reds
    for (int k = threadIdx.x; k < W * W; k += NT) {
        const int a = k / W, c = k - a * W;
        if (a < 1 || a > W - 2 || c < 1 || c > W - 2 || sf[k]) continue;
        if (((a + c) & 1) != 1) continue;
        float s = sg[k];
        s += sc[k - W];
        s += sc[k + W];
        s += sc[k - 1];
        s += sc[k + 1];
        su[k] = s * 0.25f;
    }
    __syncthreads();
    constexpr int MEND = L0 ? 2 * NU + 1 : 2 * NU;
#pragma unroll
    for (int m = 2; m < MEND; m++) {
        win_sweep<W, NT>(su, sg, sf, m, m & 1);           // even m: red, odd m: black
        __syncthreads();
    }
}

// Up half-cycle of level l >= 1 with NU post-smoothing steps on its tile
// (ti, tj): the corrected reds (pre-smoothed value + bilinear prolongation of
// level l+1's result u), then the post-smoothing; result to u.
template <int NU, int NT>
__device__ __forceinline__ void mg_up_fine(const Inst &I, int level, int ti, int tj, int done, unsigned char *lds)
{
    constexpr int HU = 2 * NU, W = kMgTile + 2 * HU;
    const LevelDev F = I.lev[level];
    const int i0 = ti * kMgTile, j0 = tj * kMgTile;
    const WinLds f = win_at(lds, 0, W);
    Window<W, NT> win;
    Prolonged<W, NT> pro;
    win.load(F, F.uo, F.g, I.g.px, I.g.py, i0 - HU, j0 - HU);
    pro.load(F, I.lev[level + 1], I.g.px, I.g.py, i0 - HU, j0 - HU);
    if (uniform(done)) return;
    win.store(f.u, f.g, f.f);
    __syncthreads();
    pro.add(f.u, f.f, f.r);
    __syncthreads();
    post_smooth<NU, 0, W, NT>(f.u, f.g, f.r, f.f);
    // last red half-sweep on the own tile; write both colours to u
    float *u = F.u;
    for (int k = threadIdx.x; k < kMgTile * kMgTile; k += NT) {
        const int a = k / kMgTile, c = k - a * kMgTile;
        const int gi = i0 + a, gj = j0 + c;
        if (gi >= F.NX || gj >= F.NY) continue;
        const int w = (a + HU) * W + (c + HU);
        float z = 0.0f;                                   // fixed nodes carry no correction
        if (!f.f[w]) {
            z = f.u[w];
            if (((gi + gj) & 1) == 0) z = win_gs<W>(f.u, f.g, w);
        }
        u[(long long)gi * F.NY + gj] = z;
    }
}

// The same of level 0: z = the V-cycle result on the tile and a one-node ring
// around it, z to u (the CG's z), w = A z to cg_w, r.z and w.z partials.  par:
// buffer of the pair holding the current residual.
template <int NU>
__global__ __launch_bounds__(kMgThreads) void k_mg_up(const Inst *insts, int many, Tab t, int par, Part pt)
{
    constexpr int HU = 2 * NU + 1, W = kMgTile + 2 * HU;
    const int ku = unit_of(t, (int)blockIdx.x);
    const Inst &I = insts[t.id[ku]];
    if (many) end_if(I.F[F_DONE]);
    const int done = vload((const int *)I.F, F_DONE);
    const int lb = (int)blockIdx.x - t.boff[ku];
    const int ti = lb / t.bx[ku], tj = lb - ti * t.bx[ku];
    const LevelDev F = I.lev[0];
    const int i0 = ti * kMgTile, j0 = tj * kMgTile;
    __shared__ float su[W * W], sg[W * W], sc[W * W];
    __shared__ uint8_t sf[W * W];
    const float *gsrc = par ? I.cg_r1 : F.g;
    Window<W> win;
    Prolonged<W> pro;
    win.load(F, F.uo, gsrc, I.g.px, I.g.py, i0 - HU, j0 - HU);
    pro.load(F, I.lev[1], I.g.px, I.g.py, i0 - HU, j0 - HU);
    if (uniform(done)) return;
    win.store(su, sg, sf);
    __syncthreads();
    pro.add(su, sf, sc);
    __syncthreads();
    post_smooth<NU, 1, W, kMgThreads>(su, sg, sc, sf);
    // the last red sweep covered the tile and its ring; z = su
    // (0 on fixed nodes), w = A z with the neighbours in the order x-1, x+1,
    // y-1, y+1
    double rz = 0.0, wz = 0.0;
    float *z_out = F.u, *w_out = I.cg_w;
    for (int k = threadIdx.x; k < kMgTile * kMgTile; k += kMgThreads) {
        const int a = k / kMgTile, c = k - a * kMgTile;
        const int gi = i0 + a, gj = j0 + c;
        if (gi >= F.NX || gj >= F.NY) continue;
        const long long n = (long long)gi * F.NY + gj;
        const int w = (a + HU) * W + (c + HU);
        float z = 0.0f, wv = 0.0f;
        if (!sf[w]) {
            z = su[w];
            float q = 4.0f * z;
            q -= su[w - W];
            q -= su[w + W];
            q -= su[w - 1];
            q -= su[w + 1];
            wv = q;
            rz += (double)sg[w] * (double)z;
            wz += (double)wv * (double)z;
        }
        z_out[n] = z;
        w_out[n] = wv;
    }
    double v[2] = {rz, wz};
    block_partials<2>(v, pt);
}

// The level-0 up kernel's r.z and (A z).z partials: a range of their own
// after the two the other reductions use, so that they survive until the
// next level-0 down kernel reads them (plain-CG instances of a batch reduce
// in between).
static Part cg_dot_part(Part pt) { return Part{pt.p + 2 * (size_t)pt.stride, pt.stride}; }

void launch_mg_down(const Inst *I, const Tab &t, bool many, bool step, int par, Part pt, hipStream_t s)
{
    if (!t.n) return;
    const dim3 g(tab_blocks(t)), b(kMgThreads);
    const Part pq = cg_dot_part(pt);
    if (step) {
        hipLaunchKernelGGL((k_mg_down<kMgSmooth, 2>), g, b, 0, s, I, many, t, par, pt, pq);
    } else {
        hipLaunchKernelGGL((k_mg_down<kMgSmooth, 1>), g, b, 0, s, I, many, t, par, pt, pq);
        finalize(I, t, pt, OP_INIT, s);
    }
}

void launch_mg_up(const Inst *I, const Tab &t, bool many, int par, Part pt, hipStream_t s)
{
    if (!t.n) return;
    // the next level-0 down kernel turns the partials into alpha and beta
    hipLaunchKernelGGL((k_mg_up<kMgSmooth>), dim3(tab_blocks(t)), dim3(kMgThreads), 0, s, I, many, t, par,
                       cg_dot_part(pt));
}

// ---------------------------------------------------------------------------
// two fine levels l and l + 1 in one launch (one pre- / post-smoothing step):
// one 1024-thread block per 32 x 32 tile of level l + 1.  The block
// recomputes level l on the wider window its level-(l+1) window needs, so no
// block depends on another between the two levels.  Level l + 1's final
// correction is consumed inside the up kernel and never stored.
// ---------------------------------------------------------------------------

constexpr int kPairThreads = 1024;
constexpr int kPairDnF = 79;      // down, level l:     rows 2 I0 - 9 .. 2 I0 + 69
constexpr int kPairDnC = 37;      // down, level l + 1: rows I0 - 3 .. I0 + 33
constexpr int kPairUpC = 39;      // up, level l + 1:   rows I0 - 3 .. I0 + 35
constexpr int kPairUpF = 68;      // up, level l:       rows 2 I0 - 2 .. 2 I0 + 65

constexpr int kPairDnLds = win_lds(kPairDnF) + win_lds(kPairDnC);
constexpr int kPairUpLds = win_lds(kPairUpC) + win_lds(kPairUpF);

// Down half-cycles of levels l and l + 1: black half-sweep of level l from
// its red-from-zero start, level l's pre-smoothed tile nodes to uo, the
// restriction of its red residuals to the level-(l+1) window (g of the own
// tile stored), black half-sweep there, level l+1's tile to uo, and the
// restriction to level l + 2 (g and its red-from-zero start u).
__device__ __forceinline__ void mg_down_pair(const Inst &I, int level, int ti, int tj, int done, unsigned char *lds)
{
    constexpr int WF = kPairDnF, WC = kPairDnC, NT = kPairThreads;
    const LevelDev F = I.lev[level], C = I.lev[level + 1], N = I.lev[level + 2];
    const int px = I.g.px, py = I.g.py;
    const int I0 = ti * kMgTile, J0 = tj * kMgTile;
    const WinLds f = win_at(lds, 0, WF), c = win_at(lds, win_lds(WF), WC);
    const int tid = threadIdx.x;
    constexpr int RC = (WC * WC + NT - 1) / NT;
    uint8_t fc[RC];
#pragma unroll
    for (int r = 0; r < RC; r++) {
        const int k = tid + r * NT, a = k / WC, b = k - a * WC;
        const long long n = k < WC * WC ? win_node(C.NX, C.NY, px, py, I0 - 3 + a, J0 - 3 + b) : -1;
        fc[r] = 1;
        if (n >= 0) fc[r] = C.fix[n];
    }
    const int ci = tid >> 4, cj = tid & 15, CI = (I0 >> 1) + ci, CJ = (J0 >> 1) + cj;   // node of level l + 2
    const bool coarse = tid < 256 && CI < N.NX && CJ < N.NY;
    const uint8_t cfix = N.fix[coarse ? (long long)CI * N.NY + CJ : 0];
    Window<WF, NT> win;
    win.load(F, F.u, F.g, px, py, 2 * I0 - 9, 2 * J0 - 9);
    if (uniform(done)) return;
    win.store(f.u, f.g, f.f);
#pragma unroll
    for (int r = 0; r < RC; r++)
        if (tid + r * NT < WC * WC) c.f[tid + r * NT] = fc[r];
    __syncthreads();
    win_sweep<WF, NT>(f.u, f.g, f.f, 1, 1);               // black, rows 1 .. WF-2
    __syncthreads();
    for (int k = tid; k < 64 * 64; k += NT) {             // own level-l nodes
        const int a = k >> 6, b = k & 63;
        const int gi = 2 * I0 + a, gj = 2 * J0 + b;
        if (gi < F.NX && gj < F.NY) F.uo[(long long)gi * F.NY + gj] = f.u[(a + 9) * WF + (b + 9)];
    }
    for (int k = tid; k < WF * WF; k += NT) {             // red residuals, rows 2 .. WF-3
        const int a = k / WF, b = k - a * WF;
        if (a < 2 || a > WF - 3 || b < 2 || b > WF - 3 || ((a + b) & 1)) continue;
        float r = 0.0f;
        if (!f.f[k]) {
            float q = 4.0f * f.u[k];
            q -= f.u[k - WF];
            q -= f.u[k + WF];
            q -= f.u[k - 1];
            q -= f.u[k + 1];
            r = f.g[k] - q;
        }
        f.r[k] = r;
    }
    __syncthreads();
    for (int k = tid; k < WC * WC; k += NT) {             // restriction to the level-(l+1) window
        const int a = k / WC, b = k - a * WC;
        float gv = 0.0f, uv = 0.0f;
        if (!c.f[k]) {
            const int m = (3 + 2 * a) * WF + (3 + 2 * b);
            float acc = 0.0f;
            acc += 0.25f * f.r[m - WF - 1];
            acc += 0.25f * f.r[m - WF + 1];
            acc += 1.0f * f.r[m];
            acc += 0.25f * f.r[m + WF - 1];
            acc += 0.25f * f.r[m + WF + 1];
            gv = acc;
            if (((a + b) & 1) == 0) uv = gv * 0.25f;
        }
        c.g[k] = gv;
        c.u[k] = uv;
        const int gi = I0 - 3 + a, gj = J0 - 3 + b;
        if (a >= 3 && a < 35 && b >= 3 && b < 35 && gi < C.NX && gj < C.NY) C.g[(long long)gi * C.NY + gj] = gv;
    }
    __syncthreads();
    win_sweep<WC, NT>(c.u, c.g, c.f, 1, 1);               // black, rows 1 .. WC-2
    __syncthreads();
    for (int k = tid; k < kMgTile * kMgTile; k += NT) {   // own level-(l+1) nodes
        const int a = k / kMgTile, b = k - a * kMgTile;
        const int gi = I0 + a, gj = J0 + b;
        if (gi < C.NX && gj < C.NY) C.uo[(long long)gi * C.NY + gj] = c.u[(a + 3) * WC + (b + 3)];
    }
    for (int k = tid; k < WC * WC; k += NT) {             // red residuals, rows 2 .. WC-3
        const int a = k / WC, b = k - a * WC;
        if (a < 2 || a > WC - 3 || b < 2 || b > WC - 3 || ((a + b) & 1)) continue;
        float r = 0.0f;
        if (!c.f[k]) {
            float q = 4.0f * c.u[k];
            q -= c.u[k - WC];
            q -= c.u[k + WC];
            q -= c.u[k - 1];
            q -= c.u[k + 1];
            r = c.g[k] - q;
        }
        c.r[k] = r;
    }
    __syncthreads();
    if (coarse) {                                         // restriction to level l + 2
        const long long n = (long long)CI * N.NY + CJ;
        float gv = 0.0f, uv = 0.0f;
        if (!cfix) {
            const int m = (3 + 2 * ci) * WC + (3 + 2 * cj);
            float acc = 0.0f;
            acc += 0.25f * c.r[m - WC - 1];
            acc += 0.25f * c.r[m - WC + 1];
            acc += 1.0f * c.r[m];
            acc += 0.25f * c.r[m + WC - 1];
            acc += 0.25f * c.r[m + WC + 1];
            gv = acc;
            if (((CI + CJ) & 1) == 0) uv = gv * 0.25f;
        }
        N.g[n] = gv;
        N.u[n] = uv;
    }
}

// Up half-cycles of levels l + 1 and l: level l+1's pre-smoothed window plus
// the prolonged level-(l+2) correction at its reds, black update, red
// half-sweep (its final correction, in LDS); then level l likewise with the
// prolongation read from that LDS result; level l's tile to u.
__device__ __forceinline__ void mg_up_pair(const Inst &I, int level, int ti, int tj, int done, unsigned char *lds)
{
    constexpr int WC = kPairUpC, WF = kPairUpF, NT = kPairThreads;
    const LevelDev F = I.lev[level], C = I.lev[level + 1], N = I.lev[level + 2];
    const int px = I.g.px, py = I.g.py;
    const int I0 = ti * kMgTile, J0 = tj * kMgTile;
    const WinLds c = win_at(lds, 0, WC), f = win_at(lds, win_lds(WC), WF);
    const int tid = threadIdx.x;
    Window<WC, NT> wc;
    Window<WF, NT> wf;
    Prolonged<WC, NT> pro;
    wc.load(C, C.uo, C.g, px, py, I0 - 3, J0 - 3);
    pro.load(C, N, px, py, I0 - 3, J0 - 3);
    wf.load(F, F.uo, F.g, px, py, 2 * I0 - 2, 2 * J0 - 2);
    if (uniform(done)) return;
    wc.store(c.u, c.g, c.f);
    wf.store(f.u, f.g, f.f);
    __syncthreads();
    pro.add(c.u, c.f, c.r);                               // corrected reds of level l + 1
    __syncthreads();
    for (int k = tid; k < WC * WC; k += NT) {             // black update, rows 1 .. WC-2
        const int a = k / WC, b = k - a * WC;
        if (a < 1 || a > WC - 2 || b < 1 || b > WC - 2 || c.f[k] || ((a + b) & 1) != 1) continue;
        float s = c.g[k];
        s += c.r[k - WC];
        s += c.r[k + WC];
        s += c.r[k - 1];
        s += c.r[k + 1];
        c.u[k] = s * 0.25f;
    }
    __syncthreads();
    win_sweep<WC, NT>(c.u, c.g, c.f, 2, 0);               // red, rows 2 .. WC-3
    __syncthreads();
    for (int k = tid; k < WF * WF; k += NT) {             // corrected reds of level l
        const int a = k / WF, b = k - a * WF;
        float v = 0.0f;
        if (((a + b) & 1) == 0 && !f.f[k]) {
            // level-(l+1) window row of fine row 2 I0 - 2 + a is 2 + (a >> 1)
            const int m = (2 + (a >> 1)) * WC + (2 + (b >> 1));
            float e;
            if (((a | b) & 1) == 0) e = c.u[m];
            else e = 0.25f * (c.u[m] + c.u[m + WC] + c.u[m + 1] + c.u[m + WC + 1]);
            v = f.u[k] + e;
        }
        f.r[k] = v;
    }
    __syncthreads();
    for (int k = tid; k < WF * WF; k += NT) {             // black update, rows 1 .. WF-2
        const int a = k / WF, b = k - a * WF;
        if (a < 1 || a > WF - 2 || b < 1 || b > WF - 2 || f.f[k] || ((a + b) & 1) != 1) continue;
        float s = f.g[k];
        s += f.r[k - WF];
        s += f.r[k + WF];
        s += f.r[k - 1];
        s += f.r[k + 1];
        f.u[k] = s * 0.25f;
    }
    __syncthreads();
    for (int k = tid; k < 64 * 64; k += NT) {             // red half-sweep of the own tile; tile to u
        const int a = k >> 6, b = k & 63;
        const int gi = 2 * I0 + a, gj = 2 * J0 + b;
        if (gi >= F.NX || gj >= F.NY) continue;
        const int w = (a + 2) * WF + (b + 2);
        float z = 0.0f;
        if (!f.f[w]) {
            z = f.u[w];
            if (((gi + gj) & 1) == 0) z = win_gs<WF>(f.u, f.g, w);
        }
        F.u[(long long)gi * F.NY + gj] = z;
    }
}

// The half-cycle of level l of a V-cycle's instances: the pairs (l, l + 1) of tp
// (tiles of level l + 1) and the single levels l of tf.  A batch of grids of
// several sizes has both; in a launch of each they took 6.2 + 13.0 us down and
// 7.1 + 11.6 us up, of which the single levels' is all latency, and 4 us each
// where the instances have finished.  PAIRS false: no pairs, half the threads
// (a 32 x 32 tile is two nodes a thread, and the halo of a level's window then
// takes three rounds of loads instead of two: 4.6 us up at 129 x 129 nodes).
template <bool PAIRS, bool DOWN>
__global__ __launch_bounds__(PAIRS ? kPairThreads : kMgThreads) void k_mg_mid(const Inst *insts, int many, Tab t,
                                                                             int npair, int level)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int ku = unit_of(t, (int)blockIdx.x);
    const bool pair = PAIRS && ku < npair;
    const Inst &I = insts[t.id[ku]];
    if (many) end_if(I.F[F_DONE]);
    const int done = vload((const int *)I.F, F_DONE);
    const int lb = (int)blockIdx.x - t.boff[ku];
    const int ti = lb / t.bx[ku], tj = lb - ti * t.bx[ku];
    if (pair) {
        if constexpr (DOWN) mg_down_pair(I, level, ti, tj, done, lds);
        else mg_up_pair(I, level, ti, tj, done, lds);
    } else {
        if constexpr (DOWN) mg_down_fine<kMgSmooth, PAIRS ? kPairThreads : kMgThreads>(I, level, ti, tj, done, lds);
        else mg_up_fine<kMgSmooth, PAIRS ? kPairThreads : kMgThreads>(I, level, ti, tj, done, lds);
    }
}

void launch_mg_mid(const Inst *I, const Tab &tp, const Tab &tf, bool many, int level, bool down, hipStream_t s)
{
    Tab t = tp;
    for (int k = 0; k < tf.n; k++) {
        t.id[t.n] = tf.id[k];
        t.bx[t.n] = tf.bx[k];
        t.boff[t.n + 1] = t.boff[t.n] + tf.boff[k + 1] - tf.boff[k];
        t.n++;
    }
    if (!t.n) return;
    static std::atomic<bool> attr{false};
    if (!attr) {
        (void)hipFuncSetAttribute((const void *)k_mg_mid<true, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  kPairDnLds);
        (void)hipFuncSetAttribute((const void *)k_mg_mid<true, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  kPairUpLds);
        attr = true;
    }
    const dim3 g(tab_blocks(t)), bp(kPairThreads), bf(kMgThreads);
    constexpr int fine = win_lds(kMgTile + 2 * (2 * kMgSmooth + 1) - 1);   // the down window, the larger one
    if (tp.n && down) hipLaunchKernelGGL((k_mg_mid<true, true>), g, bp, kPairDnLds, s, I, many, t, tp.n, level);
    else if (tp.n) hipLaunchKernelGGL((k_mg_mid<true, false>), g, bp, kPairUpLds, s, I, many, t, tp.n, level);
    else if (down) hipLaunchKernelGGL((k_mg_mid<false, true>), g, bf, fine, s, I, many, t, tp.n, level);
    else hipLaunchKernelGGL((k_mg_mid<false, false>), g, bf, fine, s, I, many, t, tp.n, level);
}

// ---------------------------------------------------------------------------
// coarse levels: the rest of the V-cycle in one work-group per instance,
// all in LDS
// ---------------------------------------------------------------------------

// Gauss-Seidel value from the four neighbours without mask tests: fixed
// nodes hold u = 0 on the LDS levels (staged as 0, never updated).  A free
// node never lies on a bounded edge, so only periodic axes wrap.
__device__ __forceinline__ float gs_nofix(const float *u, const float *gg, int i, int j, int NX, int NY)
{
    Nb b = nbs(i, j, NX, NY);
    float s = gg[i * NY + j];
    s += u[b.im * NY + j];
    s += u[b.ip * NY + j];
    s += u[i * NY + b.jm];
    s += u[i * NY + b.jp];
    return s * 0.25f;
}

// q / d for 0 <= q < 2^22 and d >= 1 from rcp = 1/d in float32: the exact
// quotient (q + 1/2) / d lies at least 1/(2d) from an integer, more than
// the rounding error of the product.
__device__ __forceinline__ int div_rcp(int q, float rcp) { return (int)(((float)q + 0.5f) * rcp); }

// Phases of the LDS levels.  Each is run by a group of threads (first,
// step): the whole work-group, or one wavefront for the small levels, with
// the group's barrier between phases.  Half-sweeps and the red-node passes
// visit the nodes of their colour only (j = 2 jj + ((i + colour) & 1)).
struct CLev {
    float *u, *g;
    const uint8_t *f;
    int NX, NY;
};

// Gauss-Seidel half-sweep of one colour (1 black, 0 red).
__device__ __forceinline__ void c_sweep(const CLev &L, int col, int first, int step)
{
    const int HW = (L.NY + 1) >> 1;
    const float rcp = 1.0f / (float)HW;
    for (int q = first; q < L.NX * HW; q += step) {
        const int i = div_rcp(q, rcp), j = 2 * (q - i * HW) + ((i + col) & 1);
        if (j < L.NY && !L.f[i * L.NY + j]) L.u[i * L.NY + j] = gs_nofix(L.u, L.g, i, j, L.NX, L.NY);
    }
}

// The same of a coarsest level with an odd number of nodes along a periodic
// axis (ox, oy).  The two sides of its wrap are neighbours of one colour: each
// reads the other's value from before the half-sweep, or it would depend on
// the wavefronts which of the two is updated first.  rd holds those values
// (rows 0 and NX - 1, then columns 0 and NY - 1), wr takes the new ones for the
// next sweep.  A solve with c_sweep's race / so, us: periodic 62 x 62 (31 x 31
// nodes) 850 / 700, 376 x 376 (47 x 47) 2790 / 2396 (23 iterations instead of 23 to
// 29), trench 416 x 488 (53 x 61) 2000 / 1877; k_coarse there 71.6 / 72.3.  (The last
// row and column after the others, with a barrier more: 1360, 3100, 2775.)
template <int ox, int oy>
__device__ __forceinline__ void c_sweep_odd(const CLev &L, const float *rd, float *wr, int col, int first, int step)
{
    const int NX = L.NX, NY = L.NY, HW = (NY + 1) >> 1, D = (int)(rd - L.u);
    const float rcp = 1.0f / (float)HW;
    // positions across the wrap: above row 0, below the last one (+ j), left of column 0, right of the last one (+ i si)
    const int up0 = ox ? D + NY : (NX - 1) * NY, dn0 = ox ? D : 0;
    const int lf0 = oy ? D + 2 * NY + NX : NY - 1, rt0 = oy ? D + 2 * NY : 0, si = oy ? 1 : NY;
    for (int q = first; q < NX * HW; q += step) {
        const int i = div_rcp(q, rcp), j = 2 * (q - i * HW) + ((i + col) & 1), k = i * NY + j;
        const bool x0 = i == 0, x1 = i == NX - 1, y0 = j == 0, y1 = j == NY - 1;
        const bool live = !L.f[k] && j < NY;      // (the other loads do not wait for it)
        float s = L.g[k];
        s += L.u[x0 ? up0 + j : k - NY];
        s += L.u[x1 ? dn0 + j : k + NY];
        s += L.u[y0 ? lf0 + i * si : k - 1];
        s += L.u[y1 ? rt0 + i * si : k + 1];
        if (!live) continue;
        s *= 0.25f;
        L.u[k] = s;
        if (ox && (x0 || x1)) wr[(x0 ? 0 : NY) + j] = s;
        if (oy && (y0 || y1)) wr[2 * NY + (y0 ? 0 : NX) + i] = s;
    }
}

// Values of the edges of a level as c_sweep_odd reads them.
__device__ __forceinline__ void c_edges(const CLev &L, float *e, int first, int step)
{
    const int NX = L.NX, NY = L.NY;
    for (int q = first; q < edge_floats(NX, NY); q += step) {
        const int r = q - 2 * NY;
        e[q] = r < 0 ? L.u[q < NY ? q : (NX - 2) * NY + q] : L.u[(r < NX ? r : r - NX) * NY + (r < NX ? 0 : NY - 1)];
    }
}

// Residual g - A u at the red nodes into sr (0 at fixed nodes).
__device__ __forceinline__ void c_resid_red(const CLev &L, float *sr, int first, int step)
{
    const int HW = (L.NY + 1) >> 1, NY = L.NY;
    const float rcp = 1.0f / (float)HW;
    for (int q = first; q < L.NX * HW; q += step) {
        const int i = div_rcp(q, rcp), j = 2 * (q - i * HW) + (i & 1);
        if (j >= NY) continue;
        const int k = i * NY + j;
        float r = 0.0f;
        if (!L.f[k]) {
            Nb b = nbs(i, j, L.NX, NY);
            float v = 4.0f * L.u[k];
            v -= L.u[b.im * NY + j];
            v -= L.u[b.ip * NY + j];
            v -= L.u[i * NY + b.jm];
            v -= L.u[i * NY + b.jp];
            r = L.g[k] - v;
        }
        sr[k] = r;
    }
}

// Restriction of the red residuals sr of level L to level C (g), with C's
// red-from-zero start (u).
__device__ __forceinline__ void c_restrict(const CLev &L, const float *sr, const CLev &C, int px, int py,
                                           int first, int step)
{
    const int NX = L.NX, NY = L.NY;
    const float rcp = 1.0f / (float)C.NY;
    for (int k = first; k < C.NX * C.NY; k += step) {
        const int Ic = div_rcp(k, rcp), Jc = k - Ic * C.NY;
        float gv = 0.0f, uv = 0.0f;
        if (!C.f[k]) {
            float acc = 0.0f;
#pragma unroll
            for (int di = -1; di <= 1; di++) {
#pragma unroll
                for (int dj = -1; dj <= 1; dj++) {
                    if ((di + dj) & 1) continue;
                    int ai = 2 * Ic + di, cj = 2 * Jc + dj;
                    if (px) ai = wrap_hi(wrap_lo(ai, NX), NX);
                    else if (ai < 0 || ai >= NX) continue;
                    if (py) cj = wrap_hi(wrap_lo(cj, NY), NY);
                    else if (cj < 0 || cj >= NY) continue;
                    const float w = (di == 0) ? 1.0f : 0.25f;
                    acc += w * sr[ai * NY + cj];
                }
            }
            gv = acc;
            if (((Ic + Jc) & 1) == 0) uv = gv * 0.25f;
        }
        C.g[k] = gv;
        C.u[k] = uv;
    }
}

// Red nodes of level L plus the prolonged correction of level C into sr (0
// at fixed nodes).
__device__ __forceinline__ void c_correct_red(const CLev &L, const CLev &C, float *sr, int first, int step)
{
    const int HW = (L.NY + 1) >> 1, NY = L.NY;
    const float rcp = 1.0f / (float)HW;
    for (int q = first; q < L.NX * HW; q += step) {
        const int i = div_rcp(q, rcp), j = 2 * (q - i * HW) + (i & 1);
        if (j >= NY) continue;
        const int k = i * NY + j;
        sr[k] = L.f[k] ? 0.0f : L.u[k] + prolong_red(C.u, C.NX, C.NY, i, j);
    }
}

// Black update of level L from the corrected reds in sr.
__device__ __forceinline__ void c_black_from(const CLev &L, const float *sr, int first, int step)
{
    const int HW = (L.NY + 1) >> 1, NY = L.NY;
    const float rcp = 1.0f / (float)HW;
    for (int q = first; q < L.NX * HW; q += step) {
        const int i = div_rcp(q, rcp), j = 2 * (q - i * HW) + ((i + 1) & 1);
        if (j >= NY || L.f[i * NY + j]) continue;
        Nb b = nbs(i, j, L.NX, NY);
        float v = L.g[i * NY + j];
        v += sr[b.im * NY + j];
        v += sr[b.ip * NY + j];
        v += sr[i * NY + b.jm];
        v += sr[i * NY + b.jp];
        L.u[i * NY + j] = v * 0.25f;
    }
}

// One wavefront's barrier: its lanes run in lockstep and LDS serves one
// wavefront's accesses in order, so fences around a wave barrier order the
// phases.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kCoarseWaveNodes = 200;   // LDS levels at most this size are run by one wavefront

// Sums of four floats over the 64 lanes of a wavefront (all lanes active),
// returned in lane 63: row-local butterflies (quad permutes, row mirrors)
// give every lane its row sum, then two row broadcasts carry the sums of
// rows 0-2 up to row 3.  A fixed order of additions.
#define DPPF_STEP(ctrl, rmask)                                                                          \
    a += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), ctrl, rmask, 0xF, false));    \
    b += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(b), ctrl, rmask, 0xF, false));    \
    c += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(c), ctrl, rmask, 0xF, false));    \
    d += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(d), ctrl, rmask, 0xF, false));
__device__ __forceinline__ void wave_sum4_f32(float &a, float &b, float &c, float &d)
{
    DPPF_STEP(0xB1, 0xF)   // quad_perm [1,0,3,2]
    DPPF_STEP(0x4E, 0xF)   // quad_perm [2,3,0,1]
    DPPF_STEP(0x141, 0xF)  // row_half_mirror
    DPPF_STEP(0x140, 0xF)  // row_mirror
    DPPF_STEP(0x142, 0xA)  // row_bcast:15 into rows 1, 3
    DPPF_STEP(0x143, 0xC)  // row_bcast:31 into rows 2, 3
}
#undef DPPF_STEP

// Exact solve of the coarsest level, u = A^-1 g, from the packed lower
// triangle T of the inverse the host factorised (row r: columns 0 .. r padded
// to a multiple of 4, diagonal halved, zero rows and columns at fixed nodes).
// Part w of 16 takes rows w, w + 16, ... (a wavefront's; where there are NW = 8,
// two parts in turn); the lanes read 16-byte pieces of the row (Q pieces per
// lane and row), R rows per pass with every load of a pass issued before any
// is used.  Each stored entry serves twice: its row's dot
// product with g (the lower part of u[r] and half its diagonal term, summed
// across the wave) and T[r][c] g[r] added to the lane's partial sum for
// column c (the upper part and the other half).  The column partials of the
// 16 parts meet in LDS (part, 16 x n floats) and are summed in a fixed
// order.  Every stored float is read once.  Small levels (n <= 256: one piece
// per lane and row, 8 rows of a wave per pass) pay one or two memory latencies.
template <int Q, int R, int NW = kCoarseWaves>
__device__ __forceinline__ void c_dense(const CLev &L, const float *__restrict__ T, int n, float *part, int tid)
{
    static_assert(R == 2 || R % 4 == 0, "rows per pass: 2 or a multiple of 4 (four-way wave sums)");
    const int lane = tid & 63;
    const int npc = (n + 3) >> 2;                 // 16-byte pieces of the longest row
    // g is read in 16-byte pieces: its padding up to a multiple of 4 (inside
    // the level's 16-byte rounded array) is cleared first
    if (tid < 4 && n + tid < 4 * npc) L.g[n + tid] = 0.0f;
    __syncthreads();
    const float4 *g4 = (const float4 *)L.g;
    // (the row addresses in scalar registers)
    for (int w = uniform(tid >> 6); w < kCoarseWaves; w += NW) {
        float4 acc[Q];
#pragma unroll
        for (int q = 0; q < Q; q++) acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int r0 = w; r0 < n; r0 += R * kCoarseWaves) {
            float4 t[R][Q];
#pragma unroll
            for (int i = 0; i < R; i++) {
                const int r = r0 + i * kCoarseWaves;
                const int len = r < n ? (r >> 2) + 1 : 0;      // pieces of row r
                const float4 *row = (const float4 *)(T + tri_off(r < n ? r : 0));
#pragma unroll
                for (int q = 0; q < Q; q++) {
                    const int k = lane + 64 * q;
                    t[i][q] = k < len ? row[k] : make_float4(0.f, 0.f, 0.f, 0.f);
                }
            }
            float4 gq[Q];
#pragma unroll
            for (int q = 0; q < Q; q++) {
                const int k = lane + 64 * q;
                gq[q] = k < npc ? g4[k] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
            float dot[R];
#pragma unroll
            for (int i = 0; i < R; i++) {
                const int r = r0 + i * kCoarseWaves;
                const float gr = r < n ? L.g[r] : 0.0f;
                dot[i] = 0.0f;
#pragma unroll
                for (int q = 0; q < Q; q++) {
                    dot[i] += t[i][q].x * gq[q].x + t[i][q].y * gq[q].y + t[i][q].z * gq[q].z + t[i][q].w * gq[q].w;
                    acc[q].x += t[i][q].x * gr;
                    acc[q].y += t[i][q].y * gr;
                    acc[q].z += t[i][q].z * gr;
                    acc[q].w += t[i][q].w * gr;
                }
            }
            if constexpr (R == 2) {
                float d2 = 0.0f, d3 = 0.0f;
                wave_sum4_f32(dot[0], dot[1], d2, d3);
            } else {
#pragma unroll
                for (int i = 0; i < R; i += 4) wave_sum4_f32(dot[i], dot[i + 1], dot[i + 2], dot[i + 3]);
            }
            if (lane == 63) {
#pragma unroll
                for (int i = 0; i < R; i++) {
                    const int r = r0 + i * kCoarseWaves;
                    if (r < n) L.u[r] = dot[i];
                }
            }
        }
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const int k = lane + 64 * q, c = 4 * k;
            if (k < npc) {
                float *pw = part + (size_t)w * n;
                if (c < n) pw[c] = acc[q].x;
                if (c + 1 < n) pw[c + 1] = acc[q].y;
                if (c + 2 < n) pw[c + 2] = acc[q].z;
                if (c + 3 < n) pw[c + 3] = acc[q].w;
            }
        }
    }
    __syncthreads();
    for (int c = tid; c < n; c += 64 * NW) {
        float v = L.u[c];
#pragma unroll
        for (int q = 0; q < kCoarseWaves; q++) v += part[(size_t)q * n + c];
        L.u[c] = v;
    }
}

constexpr int kDenseOnePass = 256;   // coarsest levels up to this size: one piece per lane, 8 rows per pass

__device__ __forceinline__ void c_dense_any(const CLev &L, const float *__restrict__ T, int n, float *part, int tid)
{
    if (n <= kDenseOnePass) c_dense<1, 8>(L, T, n, part, tid);
    else c_dense<(kDenseMaxNodes + 255) / 256, 2>(L, T, n, part, tid);
}

constexpr int kCoarsePre = 4;   // 16-byte pieces per thread loaded before the level-0 reduction (fetch calls)

// The V-cycle of LDS levels lev(0 .. nlev-1), level 0 holding its right-hand
// side and red-from-zero start, by a whole work-group.  The levels of at most
// kCoarseWaveNodes nodes, from the first such level to the coarsest and back,
// are run by the first wavefront alone.  dense(): solves the coarsest level
// exactly (called by every thread) and returns true, or returns false.
// ODD: the coarsest level may be a swept one with an odd wrap.
template <bool ODD, class Lev, class Dense>
__device__ __forceinline__ void c_cycle(Lev lev, int nlev, float *sr, int px, int py, int sweeps, Dense dense, int tid,
                                        int nt)
{
    int ls = 0;
    while (ls < nlev) {
        const CLev L = lev(ls);
        if (L.NX * L.NY <= kCoarseWaveNodes) break;
        ls++;
    }
    const int lb = ls < nlev - 1 ? ls : nlev - 1;           // levels below lb descend with the work-group
    for (int l = 0; l < lb; l++) {
        const CLev L = lev(l), C = lev(l + 1);
        c_sweep(L, 1, tid, nt);
        __syncthreads();
        c_resid_red(L, sr, tid, nt);
        __syncthreads();
        c_restrict(L, sr, C, px, py, tid, nt);
        __syncthreads();
    }
    if (ls < nlev) {
        if (tid < 64) {
            for (int l = ls; l < nlev - 1; l++) {
                const CLev L = lev(l), C = lev(l + 1);
                c_sweep(L, 1, tid, 64);
                wave_sync();
                c_resid_red(L, sr, tid, 64);
                wave_sync();
                c_restrict(L, sr, C, px, py, tid, 64);
                wave_sync();
            }
        }
        __syncthreads();
        const bool solved = dense();
        __syncthreads();
        if (tid < 64) {
            if (!solved) {
                // coarsest: red-black sweeps (the first black completes the pre-smoothing)
                const CLev L = lev(nlev - 1);
                for (int sw = 0; sw < sweeps; sw++) {
                    c_sweep(L, 1, tid, 64);
                    wave_sync();
                    c_sweep(L, 0, tid, 64);
                    wave_sync();
                }
            }
            for (int l = nlev - 2; l >= ls; l--) {
                const CLev F = lev(l), C = lev(l + 1);
                c_correct_red(F, C, sr, tid, 64);
                wave_sync();
                c_black_from(F, sr, tid, 64);
                wave_sync();
                c_sweep(F, 0, tid, 64);
                wave_sync();
            }
        }
        __syncthreads();
    } else if (dense()) {
        __syncthreads();
    } else {
        const CLev L = lev(nlev - 1);
        auto solve = [&](auto x_, auto y_) __attribute__((always_inline)) {
            constexpr int X = decltype(x_)::value, Y = decltype(y_)::value;
            float *const e0 = sr, *const e1 = sr + edge_floats(L.NX, L.NY);
            if constexpr (X || Y) {
                c_edges(L, e0, tid, nt);
                c_edges(L, e1, tid, nt);
                __syncthreads();
            }
            for (int sw = 0; sw < sweeps; sw++) {
                for (int col = 1; col >= 0; col--) {
                    if constexpr (X || Y) c_sweep_odd<X, Y>(L, sw & 1 ? e1 : e0, sw & 1 ? e0 : e1, col, tid, nt);
                    else c_sweep(L, col, tid, nt);
                    __syncthreads();
                }
            }
        };
        const bool ox = ODD && (px & L.NX & 1), oy = ODD && (py & L.NY & 1);
        if (ox && oy) solve(Int<1>{}, Int<1>{});
        else if (ox) solve(Int<1>{}, Int<0>{});
        else if (oy) solve(Int<0>{}, Int<1>{});
        else solve(Int<0>{}, Int<0>{});
    }
    for (int l = lb - 1; l >= 0; l--) {
        const CLev F = lev(l), C = lev(l + 1);
        c_correct_red(F, C, sr, tid, nt);
        __syncthreads();
        c_black_from(F, sr, tid, nt);
        __syncthreads();
        c_sweep(F, 0, tid, nt);
        __syncthreads();
    }
}

// Positions in a level's LDS arrays that one thread smooths, looked up once: NP
// pairs of neighbours (i, 2j) and (i, 2j + 1), one red and one black.  The
// phases compute them anew otherwise, 70 of 85 instructions a node.  Five words
// a pair: the first node (16 bits), whether its row is odd, which of the two
// are free and which exist; the nodes above and below the first; those left
// and right of the pair; the four coarse nodes the red one's prolongation
// reads.  A position past a row's end is read but never used.  Positions are
// unpacked where they are used: kept unpacked they would not fit.
template <int NP> struct Pairs {
    unsigned p[NP], v[NP], h[NP], ca[NP], cb[NP];
    int last;                          // this wavefront has pairs of the last round

    __device__ __forceinline__ void find(int NX, int NY, int NXc, int NYc, int tid, int nt)
    {
        const int HW = (NY + 1) >> 1, n = NX * HW;
        const float rcp = 1.0f / (float)HW;
        last = uniform(tid) + (NP - 1) * nt < n;
#pragma unroll
        for (int k = 0; k < NP; k++) {
            const int q = tid + k * nt, i = q < n ? div_rcp(q, rcp) : 0, j = q < n ? 2 * (q - i * HW) : 0;
            const int I = i >> 1, J = j >> 1, I1 = wrap_hi(I + 1, NXc), J1 = wrap_hi(J + 1, NYc);
            p[k] = (i * NY + j) | (unsigned)(i & 1) << 16 | (q < n ? 1u << 19 : 0u) | (q < n && j + 1 < NY ? 1u << 20 : 0u);
            v[k] = (wrap_lo(i - 1, NX) * NY + j) | (unsigned)(wrap_hi(i + 1, NX) * NY + j) << 16;
            h[k] = (i * NY + wrap_lo(j - 1, NY)) | (unsigned)(i * NY + (j + 2 < NY ? j + 2 : 0)) << 16;
            ca[k] = (I * NYc + J) | (unsigned)(I1 * NYc + J) << 16;
            cb[k] = (I * NYc + J1) | (unsigned)(I1 * NYc + J1) << 16;
        }
    }
    // which nodes are free, once the level's mask is in LDS
    __device__ __forceinline__ void mark(const uint8_t *f)
    {
        unsigned f0[NP], f1[NP];
#pragma unroll
        for (int k = 0; k < NP; k++) {
            const int o = p[k] & 0xFFFFu;
            f0[k] = f[o];
            f1[k] = f[o + 1];
        }
#pragma unroll
        for (int k = 0; k < NP; k++)
            p[k] |= (p[k] >> 2) & ((f0[k] ? 0u : 1u << 17) | (f1[k] ? 0u : 1u << 18));   // of those that exist
    }
    struct At {
        int o, up, dn, lf, rt;         // the node of the colour and its neighbours
        bool free, in;
    };
    template <int COL> __device__ __forceinline__ At at(int k) const
    {
        const unsigned w = opaque(p[k]), t = ((w >> 16) & 1) ^ COL;   // 1: the pair's second node
        const unsigned x = opaque(v[k]) + t * 0x10001u, y = opaque(h[k]);
        At r;
        r.o = (int)((w & 0xFFFFu) + t);
        r.up = (int)(x & 0xFFFFu);
        r.dn = (int)(x >> 16);
        r.lf = t ? r.o - 1 : (int)(y & 0xFFFFu);
        r.rt = t ? (int)(y >> 16) : r.o + 1;
        r.free = (w >> (17 + t)) & 1;
        r.in = (w >> (19 + t)) & 1;
        return r;
    }
    // u = (g + four of src) / 4 at the free nodes of a colour (0 red)
    template <int COL> __device__ __forceinline__ void sweep(const float *src, const float *g, float *u) const
    {
        float s[NP];
#pragma unroll
        for (int k = 0; k < NP; k++) {
            if (NP > 1 && k == NP - 1 && !last) continue;
            const At n = at<COL>(k);
            s[k] = g[n.o];
            s[k] += src[n.up];
            s[k] += src[n.dn];
            s[k] += src[n.lf];
            s[k] += src[n.rt];
        }
#pragma unroll
        for (int k = 0; k < NP; k++) {
            if (NP > 1 && k == NP - 1 && !last) continue;
            const unsigned w = opaque(p[k]), t = ((w >> 16) & 1) ^ COL;
            if ((w >> (17 + t)) & 1) u[(w & 0xFFFFu) + t] = s[k] * 0.25f;
        }
    }
    // red-from-zero start
    __device__ __forceinline__ void start(const float *g, float *u) const
    {
#pragma unroll
        for (int k = 0; k < NP; k++) {
            const At r = at<0>(k), b = at<1>(k);
            const float x = g[r.o] * 0.25f;
            if (r.in) u[r.o] = r.free ? x : 0.0f;
            if (b.in) u[b.o] = 0.0f;
        }
    }
    // residual at the red nodes, 0 at fixed ones
    __device__ __forceinline__ void resid_red(const float *u, const float *g, float *sr) const
    {
#pragma unroll
        for (int k = 0; k < NP; k++) {
            if (NP > 1 && k == NP - 1 && !last) continue;
            const At n = at<0>(k);
            float v = 4.0f * u[n.o];
            v -= u[n.up];
            v -= u[n.dn];
            v -= u[n.lf];
            v -= u[n.rt];
            v = g[n.o] - v;
            if (n.in) sr[n.o] = n.free ? v : 0.0f;
        }
    }
    // red nodes with the prolonged coarse correction e, 0 at fixed ones
    __device__ __forceinline__ void correct_red(const float *u, const float *e, float *sr) const
    {
#pragma unroll
        for (int k = 0; k < NP; k++) {
            if (NP > 1 && k == NP - 1 && !last) continue;
            const unsigned w = opaque(p[k]), odd = (w >> 16) & 1, o = (w & 0xFFFFu) + odd;
            const unsigned x = opaque(ca[k]), y = opaque(cb[k]);
            const float c = e[x & 0xFFFFu];
            const float m = 0.25f * (c + e[x >> 16] + e[y & 0xFFFFu] + e[y >> 16]);
            const float v = u[o] + (odd ? m : c);
            if ((w >> (19 + odd)) & 1) sr[o] = (w >> (17 + odd)) & 1 ? v : 0.0f;
        }
    }
};

// Positions of the red residuals that up to NC coarse nodes tid, tid + nt, ...
// of a thread restrict: the centre (16 bits), whether the coarse node is red,
// free, and exists; (-,-) and (-,+); (+,-) and (+,+).  Those outside a bounded
// axis read node 0, which is red and lies on that axis' edge: a fixed node's
// residual, 0.
template <int NC> struct Restrict {
    unsigned c[NC], a[NC], b[NC];

    __device__ __forceinline__ void find(int NX, int NY, int NXc, int NYc, int px, int py, int tid, int nt)
    {
        const float rcp = 1.0f / (float)NYc;
#pragma unroll
        for (int k = 0; k < NC; k++) {
            const bool in = tid + k * nt < NXc * NYc;
            const int q = in ? tid + k * nt : 0, I = div_rcp(q, rcp), J = q - I * NYc, i = 2 * I, j = 2 * J;
            const bool um = px || i > 0, up = px || i + 1 < NX, lm = py || j > 0, lp = py || j + 1 < NY;
            const int rm = wrap_lo(i - 1, NX) * NY, rp = wrap_hi(i + 1, NX) * NY;
            const int cm = wrap_lo(j - 1, NY), cp = wrap_hi(j + 1, NY);
            c[k] = (i * NY + j) | (((I + J) & 1) == 0 ? 1u << 16 : 0u) | (in ? 1u << 18 : 0u);
            a[k] = (unsigned)(um && lm ? rm + cm : 0) | (unsigned)(um && lp ? rm + cp : 0) << 16;
            b[k] = (unsigned)(up && lm ? rp + cm : 0) | (unsigned)(up && lp ? rp + cp : 0) << 16;
        }
    }
    __device__ __forceinline__ void mark(const uint8_t *fc, int tid, int nt)
    {
#pragma unroll
        for (int k = 0; k < NC; k++) {
            const bool in = (c[k] >> 18) & 1;
            const int f = fc[in ? tid + k * nt : 0];
            if (in && !f) c[k] |= 1u << 17;
        }
    }
    __device__ __forceinline__ void run(const float *sr, float *g, float *u, int tid, int nt) const
    {
#pragma unroll
        for (int k = 0; k < NC; k++) {
            const unsigned z = opaque(c[k]), x = opaque(a[k]), y = opaque(b[k]);
            float acc = 0.0f;
            acc += 0.25f * sr[x & 0xFFFFu];
            acc += 0.25f * sr[x >> 16];
            acc += sr[z & 0xFFFFu];
            acc += 0.25f * sr[y & 0xFFFFu];
            acc += 0.25f * sr[y >> 16];
            if ((z >> 17) & 1) {
                g[tid + k * nt] = acc;
                u[tid + k * nt] = (z >> 16) & 1 ? acc * 0.25f : 0.0f;
            } else if ((z >> 18) & 1) {
                g[tid + k * nt] = 0.0f;
                u[tid + k * nt] = 0.0f;
            }
        }
    }
};

// The levels from lg on: one 1024-thread work-group per instance, every level
// in LDS.  Per level on the way down a black half-sweep, the red residuals,
// their restriction to the next level with its red-from-zero start; on the
// coarsest level red-black sweeps; per level on the way up the corrected
// reds, the black update from them, then a red half-sweep.  The levels of at
// most kCoarseWaveNodes nodes, from the first such level to the coarsest and
// back, are run by the first wavefront alone (no work-group barriers).
// With fuse set it first does what k_finalize(OP_UPDATE) does after the
// level-0 CG step (t0: that launch's units, in the same order as t): the
// totals of its partials in the same order, the iteration count and the
// inner stop test; one launch fewer per iteration.  The paired or single
// fine levels between the two run on regardless (their output is then
// unused).
// NP > 0: the first two levels by positions looked up once (Pairs, Restrict),
// NP pairs of the first a thread: a phase of a 65 x 65 level takes 1500 cycles
// instead of 3000.  What is left is spread over the chain: loads and the
// step's totals 9000 cycles, masks and start 5000, the first two levels 15000,
// the levels below 8000, the exact solve 7000, each piece of code fetched for
// one pass through it.  257 x 257 nodes (first level 65 x 65): 17.7 -> 15.8 us,
// 1024 x 513 (128 x 65): 26.2 -> 24.0 us.
template <int NP, bool ODD>
__global__ __launch_bounds__(1024) void k_coarse(const Inst *insts, int many, int fuse, Tab t, Tab t0, Part pt)
{
    const Inst &I = insts[t.id[blockIdx.x]];
    const int tid = threadIdx.x, nt = blockDim.x;
    if (!fuse || many) end_if(I.F[F_DONE]);
    const CoarseArgs &a = I.coarse;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ int tab[3][kMaxLev];
    __shared__ int dims[2][kMaxLev];
    // 16-byte pieces to stage: the masks of every level, then the first
    // level's g (the global arrays are 256-byte aligned and padded, the LDS
    // ones 16-byte rounded, so whole pieces stay inside both)
    __shared__ Dev<const uint4> src[kMaxLev + 1];
    __shared__ int dst[kMaxLev + 1], cum[kMaxLev + 2];
    if (tid == 0) {
        int c = 0;
        for (int l = 0; l < a.nlev; l++) {
            tab[0][l] = a.off_u[l];
            tab[1][l] = a.off_g[l];
            tab[2][l] = a.off_f[l];
            dims[0][l] = a.NX[l];
            dims[1][l] = a.NY[l];
            src[l] = (const uint4 *)(const uint8_t *)a.fix[l];
            dst[l] = a.off_f[l];
            cum[l] = c;
            c += (a.NX[l] * a.NY[l] + 15) >> 4;
        }
        src[a.nlev] = (const uint4 *)(const float *)a.g_top;
        dst[a.nlev] = a.off_g[0];
        cum[a.nlev] = c;
        cum[a.nlev + 1] = c + ((a.NX[0] * a.NY[0] + 3) >> 2);
    }
    __syncthreads();
    const int nlev = a.nlev, px = a.px, py = a.py, npieces = cum[nlev + 1];
    // every thread issues its first pieces' loads before the level-0
    // reduction below, so their latencies overlap
    auto fetch = [&](int m, uint4 &v, int &d) {
        const int p = tid + m * nt;
        d = -1;
        if (p < npieces) {
            int k = 0;
            while (p >= cum[k + 1]) k++;
            const int q = p - cum[k];
            v = src[k][q];
            d = dst[k] + 16 * q;
        }
    };
    uint4 pv0, pv1, pv2, pv3;
    int pd0, pd1, pd2, pd3;
    fetch(0, pv0, pd0);
    fetch(1, pv1, pd1);
    fetch(2, pv2, pd2);
    fetch(3, pv3, pd3);
    // the coarsest level's inverse on its way to this die's cache: a word of
    // every line (from other kernels' launches it is not there any more)
    constexpr int kWarm = 5;
    float warm_inv[kWarm];
    const int lines = a.dense_n ? (int)((tri_off(a.dense_n) + 31) >> 5) : 0;
    if (NP) {
        const float *inv = a.ainv;
#pragma unroll
        for (int k = 0; k < kWarm; k++) warm_inv[k] = tid + k * 1024 < lines ? inv[(tid + k * 1024) * 32] : 0.0f;
    }
    // positions of the first two levels, looked up while the loads are under way
    constexpr int NPA = NP ? NP : 1, NPB = NP > 3 ? 2 : 1, NCA = NP > 3 ? 3 : 2;
    Pairs<NPA> P0;
    Pairs<NPB> P1;
    Restrict<NCA> R0;
    Restrict<1> R1;
    if (NP) {
        P0.find(dims[0][0], dims[1][0], dims[0][1], dims[1][1], tid, 1024);
        R0.find(dims[0][0], dims[1][0], dims[0][1], dims[1][1], px, py, tid, 1024);
        P1.find(dims[0][1], dims[1][1], dims[0][2], dims[1][2], tid, 1024);
        R1.find(dims[0][1], dims[1][1], dims[0][2], dims[1][2], px, py, tid, 1024);
    }
    if (fuse) {
        // what k_finalize(OP_UPDATE) does after the level-0 CG step (t0: that
        // launch's units, in the same order as t): the totals of its partials
        // in the same order, the iteration count and the inner stop test
        __shared__ double fsh[2][4];
        __shared__ int fdone;
        if (tid == 256) {
            // a wavefront outside the sums reads the scalars and flags the
            // update uses (just written by other kernels, on other XCDs), so
            // that thread 0 finds them in the caches after the barrier (the
            // empty asm keeps the loads)
            const double *ws = I.S;
            const int *wf = I.F;
            const double warm = ws[S_ETA2] + ws[S_RR0] + ws[S_CG_NALPHA] + ws[S_CG_NBETA] + ws[S_CG_NGAMMA] +
                                (double)(wf[F_ITER] + wf[F_ITER_TOT] + wf[F_PASSES]);
            asm volatile("" ::"v"(warm));
        }
        PartialSums<4> ps;
        ps.load(pt, t0.boff[blockIdx.x], t0.boff[blockIdx.x + 1], 2, tid);
        ps.sum(pt, t0.boff[blockIdx.x], t0.boff[blockIdx.x + 1], 2, fsh, tid);
        __syncthreads();
        if (tid == 0) {
            apply_op(I, OP_UPDATE, fsh[0][0] + fsh[0][1] + fsh[0][2] + fsh[0][3],
                     fsh[1][0] + fsh[1][1] + fsh[1][2] + fsh[1][3]);
            fdone = I.F[F_DONE];
        }
        __syncthreads();
        if (fdone) return;
    }
    if (pd0 >= 0) *(uint4 *)(lds + pd0) = pv0;
    if (pd1 >= 0) *(uint4 *)(lds + pd1) = pv1;
    if (pd2 >= 0) *(uint4 *)(lds + pd2) = pv2;
    if (pd3 >= 0) *(uint4 *)(lds + pd3) = pv3;
    for (int p = tid + kCoarsePre * nt; p < npieces; p += nt) {
        int k = 0;
        while (p >= cum[k + 1]) k++;
        const int q = p - cum[k];
        *(uint4 *)(lds + dst[k] + 16 * q) = src[k][q];
    }
    auto lev = [&](int l) {
        CLev L;
        L.u = (float *)(lds + tab[0][l]);
        L.g = (float *)(lds + tab[1][l]);
        L.f = (const uint8_t *)(lds + tab[2][l]);
        L.NX = dims[0][l];
        L.NY = dims[1][l];
        return L;
    };
    float *sr = (float *)(lds + a.off_s);
    __syncthreads();
    auto dense = [&]() __attribute__((always_inline)) {
        if (a.dense_n) c_dense_any(lev(nlev - 1), a.ainv, a.dense_n, (float *)(lds + a.off_p), tid);
        return a.dense_n != 0;
    };
    const CLev A = lev(0);
    if constexpr (NP > 0) {
        const CLev B = lev(1), C = lev(2);
#pragma unroll
        for (int k = 0; k < kWarm; k++) asm volatile("" ::"v"(warm_inv[k]));
        P0.mark(A.f);
        R0.mark(B.f, tid, 1024);
        P1.mark(B.f);
        R1.mark(C.f, tid, 1024);
        P0.start(A.g, A.u);
        __syncthreads();
        P0.template sweep<1>(A.u, A.g, A.u);
        __syncthreads();
        P0.resid_red(A.u, A.g, sr);
        __syncthreads();
        R0.run(sr, B.g, B.u, tid, 1024);
        __syncthreads();
        P1.template sweep<1>(B.u, B.g, B.u);
        __syncthreads();
        P1.resid_red(B.u, B.g, sr);
        __syncthreads();
        R1.run(sr, C.g, C.u, tid, 1024);
        __syncthreads();
        c_cycle<ODD>([&](int l) __attribute__((always_inline)) { return lev(l + 2); }, nlev - 2, sr, px, py, a.sweeps, dense,
                tid, nt);
        P1.correct_red(B.u, C.u, sr);
        __syncthreads();
        P1.template sweep<1>(sr, B.g, B.u);
        __syncthreads();
        P1.template sweep<0>(B.u, B.g, B.u);
        __syncthreads();
        P0.correct_red(A.u, B.u, sr);
        __syncthreads();
        P0.template sweep<1>(sr, A.g, A.u);
        __syncthreads();
        P0.template sweep<0>(A.u, A.g, A.u);
        __syncthreads();
    } else {
        const int N = A.NX * A.NY;
        const float rcp = 1.0f / (float)A.NY;
        for (int k = tid; k < N; k += nt) {
            const int i = div_rcp(k, rcp), j = k - i * A.NY;
            A.u[k] = (!A.f[k] && ((i + j) & 1) == 0) ? A.g[k] * 0.25f : 0.0f;
        }
        __syncthreads();
        c_cycle<ODD>(lev, nlev, sr, px, py, a.sweeps, dense, tid, nt);
    }
    {
        const int N = A.NX * A.NY;
        float *u = a.u_top;
        for (int k = tid; k < N; k += nt) u[k] = A.u[k];
    }
}

// The coarsest level is swept by a work-group and an odd number of its nodes
// lie along a periodic axis.
static bool odd_sweeps(const CoarseArgs &c)
{
    const int NX = c.NX[c.nlev - 1], NY = c.NY[c.nlev - 1];
    return !c.dense_n && NX * NY > kCoarseWaveNodes && ((c.px & NX & 1) || (c.py & NY & 1));
}

// The form of k_coarse for one instance: pairs of the first level a thread, 0
// where the first two levels are not there, do not fit the registers, or wrap
// an odd number of columns, 1 (ODD) where the coarsest level's sweeps cross an
// odd wrap (a kernel of its own: that code within the others' cost them up to
// 4 % on their grids).
int coarse_form(const CoarseArgs &c)
{
    if (odd_sweeps(c)) return 1;
    if (c.nlev < 3 || (c.py && ((c.NY[0] | c.NY[1]) & 1))) return 0;
    const int p0 = c.NX[0] * ((c.NY[0] + 1) / 2), p1 = c.NX[1] * ((c.NY[1] + 1) / 2);
    const int n1 = c.NX[1] * c.NY[1], n2 = c.NX[2] * c.NY[2];
    if (c.NX[0] * c.NY[0] > 65000 || n2 > 1024) return 0;
    if (p0 <= 3 * 1024 && p1 <= 1024 && n1 <= 2 * 1024) return 3;
    if (p0 <= 5 * 1024 && p1 <= 2 * 1024 && n1 <= 3 * 1024) return 5;
    return 0;
}

// The form that serves instances of both.
int coarse_form(int a, int b)
{
    if (a == 1 || b == 1) return 1;
    return a && b ? std::max(a, b) : 0;
}

void launch_coarse(const Inst *I, const Tab &t, bool many, int form, int lds_bytes, const Tab &t0, Part pt,
                   bool fuse, hipStream_t s)
{
    if (!t.n) return;
    const int f = form == 3 ? 1 : form == 5 ? 2 : form == 1 ? 3 : 0;
    static void (*const kernel[4])(const Inst *, int, int, Tab, Tab, Part) = {k_coarse<0, false>, k_coarse<3, false>,
                                                                         k_coarse<5, false>, k_coarse<0, true>};
    // a kernel's limit is the process's: always the largest that any context asks for
    static std::atomic<bool> allowed[4];
    if (lds_bytes > 64 * 1024 && !allowed[f]) {
        (void)hipFuncSetAttribute((const void *)kernel[f], hipFuncAttributeMaxDynamicSharedMemorySize, kCoarseMaxLds);
        allowed[f] = true;
    }
    hipLaunchKernelGGL(kernel[f], dim3(t.n), dim3(1024), lds_bytes, s, I, many, fuse, t, t0, pt);
}

// ---------------------------------------------------------------------------
// a whole solve of a small grid in one launch: every refinement pass of the
// multigrid-preconditioned CG by one work-group, all levels and the CG's
// vectors in LDS
//
// Launched kernel by kernel a V-cycle of a small grid is three launches and a
// pass several more, bound by the launches and by k_coarse on one CU (42 us a
// V-cycle at 81 x 30 nodes, 34 us at 64 x 64; here 17.9 and 19.2).  Arithmetic
// and the order of every addition are those of k_mg_down, k_coarse, k_mg_up,
// k_phi_update, k_resid64 and k_finalize, and the iterations a pass may take
// follow the host's rule, so the potential is the same bit for bit.
//
// A thread owns the nodes it owns in the tile kernels for the CG's vectors and
// dot products (512 threads a 32 x 32 tile, two nodes each, NT tiles in turn),
// and for the smoothing of levels 0 and 1 up to NT (level 1: a quarter) pairs
// of a red and a black node, whose LDS positions and neighbours it looks up
// once: computed anew in every phase, as k_coarse does, they cost 70 of 85
// instructions a node (64 x 64 nodes: 24 us a V-cycle so).  512 threads, as
// those positions take more than the 128 registers that 1024 would have.
// More than 4 tiles (positions in registers no longer, 35 us at 96 x 56, as
// much as launched) stay with the launched kernels.
//
// Of a V-cycle's 40000 cycles at 64 x 64 nodes the coarsest level's solve takes
// 15000 (a packed inverse of 131 KB through one CU), a smoothing phase of
// level 0 1400, the CG step with its sums 10000.  A coarsest level of more than
// kDenseOnePass nodes (41 x 15 for the paper's 80 x 30 trench, 0.76 MB) took
// one CU 19 us an iteration.  There 16 more work-groups each keep the rows of
// one part of c_dense in LDS, receive the right-hand side and return their
// share of the dot products and their column sums, in c_dense's order (7 us);
// words are exchanged as in the one-launch CG pass, with the same bounded
// waits.  At 256 nodes both ways take the same.
// ---------------------------------------------------------------------------

typedef float vf4 __attribute__((ext_vector_type(4)));

// Sums of R floats over the 64 lanes of a wavefront (all lanes active), the
// sum of v[k] returned in lane k: partners 1, 2, 4, 8, 16, 32 lanes apart, the
// narrow steps folding two values into one register (28 instructions for eight
// values; a full tree for each takes 48).
template <int CTRL> __device__ __forceinline__ float dpp_f32(float x)
{
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
template <int R> __device__ __forceinline__ float wave_sum_f32(float (&v)[R])
{
    static_assert(R == 2 || R == 4 || R == 8, "");
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < R; k++) v[k] = dpp_f32<0xB1>(v[k]);            // quad_perm [1,0,3,2]
#pragma unroll
    for (int k = 0; k < R / 2; k++) {
        const float e = v[2 * k], o = v[2 * k + 1];
        v[k] = dpp_f32<0x4E>(lane & 1 ? o : e);                        // quad_perm [2,3,0,1]
    }
    const float p0 = v[0], p1 = v[R > 2 ? 1 : 0], p2 = v[R > 4 ? 2 : 0], p3 = v[R > 4 ? 3 : 0];
    float x;
    if constexpr (R == 8) {
        const float e = lane & 2 ? p1 : p0, o = lane & 2 ? p3 : p2;
        const float e4 = dpp_f32<0x12C>(e), o4 = dpp_f32<0x124>(o);    // row_ror:12 (from 4 lanes up), row_ror:4
        x = lane & 4 ? o4 : e4;
    } else {
        x = dpp_f32<0x12C>(R == 4 && (lane & 2) ? p1 : p0);
    }
    x = dpp_f32<0x128>(x);                                             // row_ror:8
    const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(w[0]) + __uint_as_float(w[1]);
}

// Words of the exchange: the right-hand side, then each work-group's dot
// products (row r by work-group r % 16), then its column sums; whole 128-byte
// lines each.
__host__ __device__ inline int dense_line(int n) { return (n + 15) & ~15; }
constexpr int kDenseDots = 48;
__host__ __device__ inline int dense_dot_word(int n, int r) { return dense_line(n) + (r & 15) * kDenseDots + (r >> 4); }
__host__ __device__ inline int dense_col_word(int n, int h) { return dense_line(n) * (1 + h) + 16 * kDenseDots; }
__host__ __device__ inline int mg_words(int n) { return dense_col_word(n, kCoarseWaves); }
int mg_solve_words(int n) { return mg_words(n); }

// Two tagged words at an even place in one 16-byte store (a reader takes a
// word at a time, and each carries its tag).
__device__ __forceinline__ void st_pair(const __amdgpu_buffer_rsrc_t words, int at, float x, float y, unsigned epoch)
{
    typedef unsigned vu4 __attribute__((ext_vector_type(4)));
    constexpr int SC1 = 16;            // written through to where other dies read it
    __builtin_amdgcn_raw_buffer_store_b128(vu4{__float_as_uint(x), epoch, __float_as_uint(y), epoch}, words, 8 * at, 0, SC1);
}


constexpr int kDenseCols = (kDenseMaxNodes + kMgThreads - 1) / kMgThreads;   // columns a thread
constexpr int kDenseRows = (kDenseMaxNodes + kCoarseWaves - 1) / kCoarseWaves;

// Rows of work-group h of the dense solve in LDS, zero beyond each row's
// length; then one answer per right-hand side until the solve ends.
__device__ void mg_dense_helper(const Inst &I, const MgSolveArgs &m, int h, unsigned epoch, unsigned char *lds)
{
    const CoarseArgs &a = I.coarse;
    const int n = a.dense_n, np = 4 * ((n + 3) >> 2), tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = (n - h + kCoarseWaves - 1) / kCoarseWaves;
    float *T = (float *)lds, *g = T + rows * np;
    const auto words = __builtin_amdgcn_make_buffer_rsrc(m.words, 0, 8 * mg_words(n), 0x00027000);
    __shared__ float dots[kDenseDots];
    __shared__ int state;              // 0 go on, 1 finished, 2 gave up
    for (int k = tid; k < rows * np; k += blockDim.x) {
        const int i = k / np, c = k - i * np, r = h + i * kCoarseWaves;
        T[k] = c < 4 * ((r >> 2) + 1) ? a.ainv[tri_off(r) + c] : 0.f;
    }
    if (tid == 0) state = 0;
    for (int k = n + tid; k < np; k += blockDim.x) g[k] = 0.f;
    for (;; epoch++) {
        __syncthreads();
        // one lane watches one line, another one in each work-group, so that
        // no line is polled by all of them while its stores arrive
        if (tid == 0) {
            const int k = min(16 * h, n - 1);
            Patience pat;
            while (((unsigned)(ld_agent(m.words + k) >> 32) & 0x7FFFFFFFu) != epoch) {
                __builtin_amdgcn_s_sleep(2);
                if (!pat.more(m.abort_word, m.wait)) break;
            }
        }
        __syncthreads();
        int mine = 0;
        for (int k = tid; k < n; k += blockDim.x) {
            Patience pat;
            for (;;) {
                const u64 w = ld_agent(m.words + k);
                const unsigned t = (unsigned)(w >> 32);
                g[k] = __uint_as_float((unsigned)w);
                if (t == epoch) break;
                if (t == (epoch | 0x80000000u)) { mine = 1; break; }
                __builtin_amdgcn_s_sleep(4);
                if (!pat.more(m.abort_word, m.wait)) { mine = 2; break; }
            }
        }
        if (mine) atomicMax(&state, mine);
        __syncthreads();
        if (state) return;
        // dot products: rows wv, wv + 8, ... of this wavefront, pieces of 16 bytes a lane
        constexpr int RW = 8, Q = (kDenseMaxNodes + 255) / 256;
        static_assert(kDenseRows <= RW * (kMgThreads / 64) && kDenseRows <= 64, "");
        const vf4 *g4 = (const vf4 *)g;
        float dot[RW];
#pragma unroll
        for (int i = 0; i < RW; i++) dot[i] = 0.f;
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const int k = lane + 64 * q;
            const bool in = k < np / 4;
            vf4 x = g4[in ? k : 0];
            x = in ? x : vf4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < RW; i++) {
                const int ri = wv + i * (kMgThreads / 64);
                if (ri >= rows) continue;
                vf4 t = ((const vf4 *)(T + ri * np))[in ? k : 0];
                t = in ? t : vf4{0.f, 0.f, 0.f, 0.f};
                dot[i] += t.x * x.x + t.y * x.y + t.z * x.z + t.w * x.w;
            }
        }
        const float d = wave_sum_f32(dot);
        const int mr = wv + lane * (kMgThreads / 64);
        if (lane < RW && mr < rows) dots[mr] = d;
        // sums of columns 2 tid and 2 tid + 1: rows in order
        const float gl = lane < rows ? g[h + lane * kCoarseWaves] : 0.f;
        const int c2 = min(2 * tid, np - 2);
        float a0 = 0.f, a1 = 0.f;
        if (2 * (tid & ~63) < n) {
            for (int i0 = 0; i0 < rows; i0 += 8) {
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    // past the last row a zero times the last row
                    const float gr = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(gl), i0 + k));
                    const float2 t = *(const float2 *)(T + min(i0 + k, rows - 1) * np + c2);
                    a0 += t.x * gr;
                    a1 += t.y * gr;
                }
            }
        }
        if (2 * tid < n) st_pair(words, dense_col_word(n, h) + 2 * tid, a0, a1, epoch);
        __syncthreads();
        if (tid >= kMgThreads - 64 && 2 * lane < rows)
            st_pair(words, dense_dot_word(n, h) + 2 * lane, dots[2 * lane], dots[2 * lane + 1], epoch);
        // the answer leaves before the polls for the next right-hand side begin
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // nothing comes before the rest of the V-cycle is done
        __builtin_amdgcn_s_sleep(127);
    }
}

template <int NT, bool HELP, bool ODD>
__global__ __launch_bounds__(kMgThreads, 2) void k_mg_solve(const Inst *insts, MgSolveArgs m)
{
    const Inst &I = insts[0];
    extern __shared__ __align__(16) unsigned char lds[];
    unsigned epoch = m.epoch;
    int *F = I.F;
    double *S = I.S;
    if (F[F_CONV]) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            F[F_SKIP] = 1;
            F[F_DONE] = 1;
        }
        return;
    }
    if (HELP && blockIdx.x > 0) {
        mg_dense_helper(I, m, (int)blockIdx.x - 1, epoch, lds);
        return;
    }
    constexpr int NT1 = NT / 4 + 1, NC = (NT + 1) / 2 + 1;   // level 1: pairs and nodes a thread
    const CoarseArgs &a = I.coarse;
    const LevelDev L0 = I.lev[0];
    const int NX = L0.NX, NY = L0.NY, N0 = NX * NY, N1 = a.NX[0] * a.NY[0];
    const int tid = threadIdx.x, nt = kMgThreads, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __shared__ int tab[5][kMaxLev];              // levels 1 ..: LDS offsets of u, g, mask; nodes along x and y
    __shared__ double red[2][2][NT][8];          // [turn][quantity][tile][wavefront]
    __shared__ double redv[256];
    __shared__ int give_up;
    // kept: after a word exchange they would be read from memory again
    const int nlev = a.nlev, px = a.px, py = a.py, sweeps = a.sweeps, dense_n = a.dense_n;
    const float *const ainv = a.ainv;
    float *const part = (float *)(lds + a.off_p);
    if (tid == 0) {
        give_up = 0;
        for (int l = 0; l < nlev; l++) {
            tab[0][l] = a.off_u[l];
            tab[1][l] = a.off_g[l];
            tab[2][l] = a.off_f[l];
            tab[3][l] = a.NX[l];
            tab[4][l] = a.NY[l];
        }
    }
    auto lev = [&](int l) __attribute__((always_inline)) {
        CLev L;
        L.u = (float *)(lds + tab[0][l]);
        L.g = (float *)(lds + tab[1][l]);
        L.f = (const uint8_t *)(lds + tab[2][l]);
        L.NX = tab[3][l];
        L.NY = tab[4][l];
        return L;
    };
    float *const u0 = (float *)(lds + m.off_u), *const g0 = (float *)(lds + m.off_g);
    float *const sr0 = (float *)(lds + m.off_s), *const sr1 = (float *)(lds + a.off_s);
    uint8_t *const f0 = lds + m.off_f;
    __syncthreads();
    float *const u1 = (float *)(lds + tab[0][0]), *const g1 = (float *)(lds + tab[1][0]);
    for (int k = tid; k < N0; k += nt) {
        f0[k] = L0.fix[k];
        u0[k] = g0[k] = sr0[k] = 0.0f;
    }
    if (tid == 0) sr0[N0] = 0.0f;
    for (int k = tid; k < N1; k += nt) u1[k] = g1[k] = sr1[k] = 0.0f;
    for (int l = 0; l < nlev; l++)
        for (int k = tid; k < tab[3][l] * tab[4][l]; k += nt) lds[tab[2][l] + k] = a.fix[l][k];
    __syncthreads();
    Pairs<NT> P0;
    Pairs<NT1> P1;
    Restrict<NC> R0;
    Restrict<1> R1;
    P0.find(NX, NY, tab[3][0], tab[4][0], tid, nt);
    P0.mark(f0);
    R0.find(NX, NY, tab[3][0], tab[4][0], px, py, tid, nt);
    R0.mark(lds + tab[2][0], tid, nt);
    if (nlev > 1) {
        P1.find(tab[3][0], tab[4][0], tab[3][1], tab[4][1], tid, nt);
        P1.mark(lds + tab[2][0]);
        R1.find(tab[3][0], tab[4][0], tab[3][1], tab[4][1], px, py, tid, nt);
        R1.mark(lds + tab[2][1], tid, nt);
    }
    // own nodes: row and column of slot q (0, 0 where the thread has none there)
    unsigned freeb = 0, redb = 0, inb = 0;
    auto own = [&](int q, int &i, int &j) __attribute__((always_inline)) {
        const int tile = q >> 1, ti = tile / m.tiles_y, tj = tile - ti * m.tiles_y, t = opaque(tid);
        i = ti * kMgTile + (t >> 5) + (kMgThreads / kMgTile) * (q & 1);
        j = tj * kMgTile + (t & (kMgTile - 1));
    };
#pragma unroll
    for (int q = 0; q < 2 * NT; q++) {
        int i, j;
        own(q, i, j);
        const bool in = (q >> 1) < m.tiles && i < NX && j < NY;
        if (in) inb |= 1u << q;
        if (in && !f0[i * NY + j]) freeb |= 1u << q;
        if (((i + j) & 1) == 0) redb |= 1u << q;
    }
    auto node = [&](int q) __attribute__((always_inline)) {
        int i, j;
        own(q, i, j);
        return (inb >> q) & 1 ? i * NY + j : 0;
    };
    // the CG's p, s and e of slot q
    auto vec = [&](int w, int q) __attribute__((always_inline)) -> float & {
        return ((float *)(lds + m.off_v))[(w * 2 * NT + q) * kMgThreads + tid];
    };
    // the coarsest level exactly: false where it has no inverse
    auto dense = [&]() __attribute__((always_inline)) -> bool {
        const int n = dense_n;
        if (!n) return false;
        const CLev L = lev(nlev - 1);
        if constexpr (!HELP) {
            c_dense<1, 8, kMgThreads / 64>(L, ainv, n, part, tid);
            return true;
        }
        const auto words = __builtin_amdgcn_make_buffer_rsrc(m.words, 0, 8 * mg_words(n), 0x00027000);
        if (2 * tid < n) st_pair(words, 2 * tid, L.g[2 * tid], L.g[min(2 * tid + 1, n - 1)], epoch);
        // an answer takes two trips through memory and the sums between them; 17 words a thread polled
        // without a pause kept the answers from getting through (0.7 ms a V-cycle at 615 nodes)
        __builtin_amdgcn_s_sleep(64);
        auto collect = [&](auto cols_) __attribute__((always_inline)) {
            constexpr int C = decltype(cols_)::value;
            Patience pat;
            float x[C][kCoarseWaves + 1];
            for (;;) {
                bool here = true;
#pragma unroll
                for (int k = 0; k < C; k++) {
                    const int c = min(tid + k * nt, n - 1);
#pragma unroll
                    for (int q = 0; q <= kCoarseWaves; q++) {
                        const u64 w = ld_agent(m.words + (q == 0 ? dense_dot_word(n, c) : dense_col_word(n, q - 1) + c));
                        here = here && (unsigned)(w >> 32) == epoch;
                        x[k][q] = __uint_as_float((unsigned)w);
                    }
                }
                if (here) break;
                __builtin_amdgcn_s_sleep(8);
                if (!pat.more(m.abort_word, m.wait)) {
                    give_up = 1;
                    break;
                }
            }
#pragma unroll
            for (int k = 0; k < C; k++) {
                float v = x[k][0];
#pragma unroll
                for (int q = 1; q <= kCoarseWaves; q++) v += x[k][q];
                if (tid + k * nt < n) L.u[tid + k * nt] = v;
            }
        };
        if (64 * wave + (kDenseCols - 1) * nt < n) collect(Int<kDenseCols>{});
        else collect(Int<1>{});
        return true;
    };
    // levels 2 and below, or the coarsest level alone
    auto deeper = [&](int l) __attribute__((always_inline)) {
        auto sub = [&](int k) __attribute__((always_inline)) { return lev(l + k); };
        c_cycle<ODD>(sub, nlev - l, l == 0 ? sr1 : (float *)(lds + m.off_s2), px, py, sweeps, dense, tid, nt);
    };
    // V-cycle of the right-hand side g0 from the red-from-zero start in u0
    auto cycle = [&]() __attribute__((always_inline)) {
        P0.template sweep<1>(u0, g0, u0);
        __syncthreads();
        P0.resid_red(u0, g0, sr0);
        __syncthreads();
        R0.run(sr0, g1, u1, tid, nt);
        __syncthreads();
        const int deep = nlev > 1;
        if (deep) {
            P1.template sweep<1>(u1, g1, u1);
            __syncthreads();
            P1.resid_red(u1, g1, sr1);
            __syncthreads();
            const CLev C = lev(1);
            R1.run(sr1, C.g, C.u, tid, nt);
            __syncthreads();
        }
        deeper(deep);
        if (deep) {
            P1.correct_red(u1, lev(1).u, sr1);
            __syncthreads();
            P1.template sweep<1>(sr1, g1, u1);
            __syncthreads();
            P1.template sweep<0>(u1, g1, u1);
            __syncthreads();
        }
        P0.correct_red(u0, u1, sr0);
        __syncthreads();
        P0.template sweep<1>(sr0, g0, u0);
        __syncthreads();
        P0.template sweep<0>(u0, g0, u0);
        __syncthreads();
    };
    int turn = 0;
    // totals of NQ quantities from the tile threads' sums v[quantity][tile]
    auto totals = [&](double (&v)[2][NT], auto nq_, double (&out)[2]) {
        constexpr int NQ = decltype(nq_)::value, TS = NQ == 2 ? 2 : 4;
#pragma unroll
        for (int r = 0; r < NT; r += TS) {
            double x[4];
#pragma unroll
            for (int k = 0; k < 4; k++) x[k] = r + k % TS < NT ? v[k / TS][r + k % TS < NT ? r + k % TS : 0] : 0.0;
            wave_sum4(x);
            if (lane == 0) {
#pragma unroll
                for (int k = 0; k < 4; k++)
                    if (r + k % TS < NT) red[turn][k / TS][r + k % TS][wave] = x[k];
            }
        }
        __syncthreads();
        double y[4] = {0.0, 0.0, 0.0, 0.0};
        if (lane < m.tiles) {
#pragma unroll
            for (int w = 0; w < 8; w++)
#pragma unroll
                for (int q = 0; q < NQ; q++) y[q] += red[turn][q][lane][w];
        }
        wave_sum4(y);
        // the other three groups of 64 partials are empty
#pragma unroll
        for (int q = 0; q < NQ; q++) out[q] = y[q] + 0.0 + 0.0 + 0.0;
        turn ^= 1;
    };
    // float64 residual r = b - A phi into lev[0].g, ||r||^2 (virtual blocks of 4 rows x 64 columns)
    const int vbx = (NY + kGridBX - 1) / kGridBX, nvb = vbx * ((NX + kGridBY - 1) / kGridBY);
    auto residual = [&]() __attribute__((always_inline)) -> double {
        for (int vb = wave; vb < nvb; vb += nt / 64) {
            const int byb = vb / vbx, j = (vb - byb * vbx) * kGridBX + lane;
            double x[4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int i = byb * kGridBY + r, n = i * NY + j;
                x[r] = 0.0;
                if (i >= NX || j >= NY) continue;
                const int im = wrap_lo(i - 1, NX), ip = wrap_hi(i + 1, NX);
                const int jm = wrap_lo(j - 1, NY), jp = wrap_hi(j + 1, NY);
                const int a = im * NY + j, c = ip * NY + j, d = i * NY + jm, e = i * NY + jp;
                const double *phi = I.phi;
                const double pn = phi[n], pa = phi[a], pc = phi[c], pd = phi[d], pe = phi[e], b = I.b[n];
                double s = 4.0 * pn;
                s = f0[a] ? s : s - pa;
                s = f0[c] ? s : s - pc;
                s = f0[d] ? s : s - pd;
                s = f0[e] ? s : s - pe;
                const double res = f0[n] ? 0.0 : b - s;
                L0.g[n] = (float)res;
                x[r] = res * res;
            }
            wave_sum4(x);
            if (lane == 0) redv[vb] = 0.0 + x[0] + x[1] + x[2] + x[3];
        }
        __syncthreads();
        double y[4];
#pragma unroll
        for (int k = 0; k < 4; k++) y[k] = lane + 64 * k < nvb ? redv[lane + 64 * k] : 0.0;
        wave_sum4(y);
        return y[0] + y[1] + y[2] + y[3];
    };

    int total_it = F[F_ITER_TOT], passes = F[F_PASSES], iter1 = F[F_ITER1];
    int chunk0 = m.chunk0, chunk1 = m.chunk1;
    double rr64 = S[S_RR64];
    const double bb = S[S_BB] > 0.0 ? S[S_BB] : 1.0, tol2 = I.rtol * I.rtol;
    const double lo = I.eta_min * I.eta_min;
    for (int pass = 0; pass < 64; pass++) {
        if (pass > 0 && (!(rr64 < INFINITY) || total_it >= m.max_iter)) break;
        const int K = max(1, min(min(pass > 0 ? chunk1 : chunk0, 128), m.max_iter - total_it));
        // inner start: r, ||r||^2, the inner stop ratio (e, p and s start with the first step)
        float r_[2 * NT];
        double v[2][NT], t2[2];
#pragma unroll
        for (int q = 0; q < 2 * NT; q++) {
            const float x = L0.g[node(q)];
            r_[q] = (freeb >> q) & 1 ? x : 0.f;
        }
        auto sum_rr = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < NT; r++) {
                double x = 0.0;
                x += (double)r_[2 * r] * (double)r_[2 * r];
                x += (double)r_[2 * r + 1] * (double)r_[2 * r + 1];
                v[0][r] = x;
                v[1][r] = 0.0;
            }
            totals(v, Int<1>{}, t2);
        };
        sum_rr();
        double eta2 = 0.09 * tol2 * bb / (rr64 > 0.0 ? rr64 : 1.0);
        eta2 = eta2 < lo ? lo : (eta2 > 0.25 ? 0.25 : eta2);
        const double rr0 = t2[0];
        double rr = rr0, a_old = 0.0, g_old = 0.0, b_old = 0.0;
        bool done = rr0 == 0.0;
        int iter = 0;
        passes++;
        while (!done && iter < K) {
            // one V-cycle of r: z (level 0's u)
#pragma unroll
            for (int q = 0; q < 2 * NT; q++) {
                const int n = node(q);
                if ((freeb >> q) & 1) {
                    g0[n] = r_[q];
                    u0[n] = (redb >> q) & 1 ? r_[q] * 0.25f : 0.0f;
                }
            }
            __syncthreads();
            cycle();
            if (HELP) {
                epoch++;
                if (give_up) {
                    // the passes before this one stand; the host goes on from there
                    if (tid == 0) __hip_atomic_store(m.abort_word, (int)kAbortGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    return;
                }
            }
            // w = A z, r.z and w.z; the step's vectors are on their way meanwhile
            float p_[2 * NT], s_[2 * NT], e_[2 * NT], w_[2 * NT], z_[2 * NT];
#pragma unroll
            for (int q = 0; q < 2 * NT; q++) {
                const int n = node(q);
                p_[q] = vec(0, q);
                s_[q] = vec(1, q);
                e_[q] = vec(2, q);
                r_[q] = g0[n];
            }
#pragma unroll
            for (int q = 0; q < 2 * NT; q++) {
                int i, j;
                own(q, i, j);
                const bool f = (freeb >> q) & 1;
                i = f ? i : 0;
                j = f ? j : 0;
                const Nb nb = nbs(i, j, NX, NY);
                const float z = u0[i * NY + j];
                float t = 4.0f * z;
                t -= u0[nb.im * NY + j];
                t -= u0[nb.ip * NY + j];
                t -= u0[i * NY + nb.jm];
                t -= u0[i * NY + nb.jp];
                z_[q] = f ? z : 0.f;
                w_[q] = f ? t : 0.f;
                r_[q] = f ? r_[q] : 0.f;
                // before the first step the vectors hold an earlier pass
                e_[q] = iter > 0 ? e_[q] : 0.f;
            }
#pragma unroll
            for (int r = 0; r < NT; r++) {
                double x = 0.0, y = 0.0;
#pragma unroll
                for (int q = 2 * r; q < 2 * r + 2; q++) {
                    x += (double)r_[q] * (double)z_[q];
                    y += (double)w_[q] * (double)z_[q];
                }
                v[0][r] = x;
                v[1][r] = y;
            }
            totals(v, Int<2>{}, t2);
            // one CG step
            const double gamma = t2[0], delta = t2[1];
            const bool first = iter == 0;
            double al, be = 0.0;
            if (first) {
                al = gamma / delta;
            } else {
                be = gamma / g_old;
                al = gamma / (delta - be * gamma / a_old);
            }
            if (!(al > 0.0 && al < INFINITY && be < INFINITY)) {
                done = true;
                break;
            }
            const float alpha = (float)al, beta = (float)be;
#pragma unroll
            for (int q = 0; q < 2 * NT; q++) {
                const float pn = first ? z_[q] : z_[q] + beta * p_[q];
                const float sn = first ? w_[q] : w_[q] + beta * s_[q];
                const bool f = (freeb >> q) & 1;
                vec(0, q) = pn;
                vec(1, q) = sn;
                vec(2, q) = e_[q] + alpha * pn;
                r_[q] = f ? r_[q] - alpha * sn : 0.f;
            }
            sum_rr();
            rr = t2[0];
            iter++;
            total_it++;
            if (passes == 1) iter1 = iter;
            if (rr <= eta2 * rr0) done = true;
            a_old = al;
            b_old = be;
            g_old = gamma;
        }
        // end of the pass: phi += e, float64 residual and convergence test
#pragma unroll
        for (int q = 0; q < 2 * NT; q++) {
            const int n = node(q);
            if (((freeb >> q) & 1) && iter > 0) I.phi[n] += (double)vec(2, q);
        }
        __syncthreads();
        rr64 = residual();
        const bool conv = rr64 <= tol2 * bb;
        const int next = !done ? min(2 * K, 128) : max(1, iter);
        if (pass > 0) chunk1 = next;
        else chunk0 = next;
        if (tid == 0) {
            S[S_ETA2] = eta2;
            S[S_RR0] = rr0;
            S[S_RR] = rr;
            S[S_CG_ALPHA] = a_old;
            S[S_CG_BETA] = b_old;
            S[S_CG_GAMMA] = g_old;
            S[S_RR64] = rr64;
            F[F_SKIP] = 0;
            F[F_DONE] = done ? 1 : 0;
            F[F_ITER] = iter;
            F[F_ITER_TOT] = total_it;
            F[F_PASSES] = passes;
            F[F_ITER1] = iter1;
            F[F_CONV] = conv ? 1 : 0;
            F[F_CHUNK0] = chunk0;
            F[F_CHUNK1] = chunk1;
        }
        __syncthreads();
        if (conv) break;
    }
    // the helpers' last word
    if (HELP)
        for (int c = tid; c < dense_n; c += nt) st_agent(m.words + c, tagged(0u, epoch | 0x80000000u));
}

constexpr int kMgSolveMaxLds = 150 * 1024;

static const void *mg_solve_kernel(const MgPlan &p)
{
    if (p.help) return p.R == 2 ? (const void *)k_mg_solve<2, true, false> : (const void *)k_mg_solve<4, true, false>;
    if (p.odd) return p.R == 2 ? (const void *)k_mg_solve<2, false, true> : (const void *)k_mg_solve<4, false, true>;
    return p.R == 2 ? (const void *)k_mg_solve<2, false, false> : (const void *)k_mg_solve<4, false, false>;
}

MgPlan mg_solve_plan(int NX, int NY, const CoarseArgs &c, int lg)
{
    MgPlan p{};
    p.tiles_y = (NY + kMgTile - 1) / kMgTile;
    p.tiles = p.tiles_y * ((NX + kMgTile - 1) / kMgTile);
    const int nvb = ((NY + kGridBX - 1) / kGridBX) * ((NX + kGridBY - 1) / kGridBY);
    if (lg != 1 || p.tiles > 4 || nvb > 256) return p;
    if (c.py && ((NY | (c.nlev > 1 ? c.NY[0] : 0)) & 1)) return p;      // the pairs of Pairs wrap whole
    p.R = p.tiles <= 2 ? 2 : 4;
    // what a thread's registers hold of levels 0 and 1
    if (NX * ((NY + 1) / 2) > p.R * kMgThreads || c.NX[0] * ((c.NY[0] + 1) / 2) > (p.R / 4 + 1) * kMgThreads ||
        c.NX[0] * c.NY[0] > ((p.R + 1) / 2 + 1) * kMgThreads || (c.nlev > 1 && c.NX[1] * c.NY[1] > kMgThreads))
        return p;
    const int N0 = NX * NY;
    int off = (c.lds_bytes + 15) & ~15;
    p.off_u = off;
    off += (N0 * 4 + 15) & ~15;
    p.off_g = off;
    off += (N0 * 4 + 15) & ~15;
    p.off_s = off;
    off += ((N0 + 1) * 4 + 15) & ~15;
    p.off_s2 = off;
    if (c.nlev > 1) off += (scratch_floats(c.NX[1], c.NY[1]) * 4 + 15) & ~15;
    p.off_f = off;
    off += (N0 + 15) & ~15;
    p.off_v = off;
    off += 3 * 2 * p.R * kMgThreads * 4;
    p.help = c.dense_n > kDenseOnePass ? kCoarseWaves : 0;
    p.odd = odd_sweeps(c);
    if (p.help) {
        const int np = 4 * ((c.dense_n + 3) >> 2);
        off = std::max(off, (kDenseRows + 1) * np * 4);
    }
    p.lds = off;
    if (off > kMgSolveMaxLds) return p;
    const void *f = mg_solve_kernel(p);
    // (the same limit for every context: it is the process's, and one of a smaller grid would lower it under a live one)
    if (off > 64 * 1024 &&
        hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMgSolveMaxLds) != hipSuccess) {
        (void)hipGetLastError();
        return p;
    }
    int dev = 0, cus = 0, per = 0;
    p.ok = hipGetDevice(&dev) == hipSuccess &&
           hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
           hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, kMgThreads, off) == hipSuccess && per * cus > p.help;
    return p;
}

hipError_t launch_mg_solve(const Inst *I, const MgPlan &p, MgSolveArgs m, hipStream_t s)
{
    m.tiles = p.tiles;
    m.tiles_y = p.tiles_y;
    m.off_u = p.off_u;
    m.off_g = p.off_g;
    m.off_s = p.off_s;
    m.off_f = p.off_f;
    m.off_s2 = p.off_s2;
    m.off_v = p.off_v;
    const void *f = mg_solve_kernel(p);
    void *args[] = {&I, &m};
    if (p.help) return hipLaunchCooperativeKernel(f, dim3(1 + p.help), dim3(kMgThreads), args, p.lds, s);
    return hipLaunchKernel(f, dim3(1), dim3(kMgThreads), args, p.lds, s);
}

// ---------------------------------------------------------------------------
// particles: gather, leapfrog push, wall test, deposit (eqs. 1-4)
// ---------------------------------------------------------------------------

// Sums of four 32-bit values over the 64 lanes (all lanes active), returned
// as wave-uniform values.  Row-local butterflies (quad permutes, row
// mirrors) give every lane its row sum, then two row broadcasts carry the
// sums of rows 0-2 upward to lane 63.  The four chains are interleaved so
// the DPP read-after-write wait states are filled with useful work.
#define DPP_STEP(ctrl, rmask)                                                                  \
    a += (unsigned)__builtin_amdgcn_update_dpp(0, (int)a, ctrl, rmask, 0xF, false);            \
    b += (unsigned)__builtin_amdgcn_update_dpp(0, (int)b, ctrl, rmask, 0xF, false);            \
    c += (unsigned)__builtin_amdgcn_update_dpp(0, (int)c, ctrl, rmask, 0xF, false);            \
    d += (unsigned)__builtin_amdgcn_update_dpp(0, (int)d, ctrl, rmask, 0xF, false);
__device__ __forceinline__ void wave_sum4_u32(unsigned &a, unsigned &b, unsigned &c, unsigned &d)
{
    DPP_STEP(0xB1, 0xF)   // quad_perm [1,0,3,2]
    DPP_STEP(0x4E, 0xF)   // quad_perm [2,3,0,1]
    DPP_STEP(0x141, 0xF)  // row_half_mirror
    DPP_STEP(0x140, 0xF)  // row_mirror
    DPP_STEP(0x142, 0xA)  // row_bcast:15 into rows 1, 3
    DPP_STEP(0x143, 0xC)  // row_bcast:31 into rows 2, 3
    a = (unsigned)__builtin_amdgcn_readlane((int)a, 63);
    b = (unsigned)__builtin_amdgcn_readlane((int)b, 63);
    c = (unsigned)__builtin_amdgcn_readlane((int)c, 63);
    d = (unsigned)__builtin_amdgcn_readlane((int)d, 63);
}
#undef DPP_STEP

// Arguments of the particle kernels resolved once per block into plain
// scalars and pointers (the storage set in use is device info[7], flipped
// by every re-binning), so particle stores cannot force them to be reloaded.
// Global-memory (address space 1) pointers: loads, stores and atomics on
// them compile to global_* instructions, which do not share the LDS wait
// counter the way flat accesses do, so the deposit's LDS atomics never wait
// for outstanding particle loads.
#define GLOBAL __attribute__((address_space(1)))
template <class T> __device__ __forceinline__ GLOBAL T *to_global(T *p) { return (GLOBAL T *)p; }
template <class T> __device__ __forceinline__ GLOBAL T *to_global(const Dev<T> &p) { return (GLOBAL T *)p.at; }
typedef int nt_i4 __attribute__((ext_vector_type(4)));
typedef float nt_f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ld_f4(GLOBAL const float4 *p)
{
    const nt_f4 v = *(GLOBAL const nt_f4 *)p;
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ void gatomic_add(GLOBAL unsigned long long *p, unsigned long long v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct PK {
    Geom g;
    int TX, TY, H, WX, WY, tiles_y;
    GLOBAL const uint8_t *cell_cond;
    GLOBAL const float4 *E4;
    GLOBAL int32_t *cell;
    GLOBAL float *ox, *oy, *vx, *vy;
    GLOBAL unsigned long long *rho;
    float qdt, dtf, hq;
    int box_i_top, box_j_lo, box_j_hi, species;
    GLOBAL unsigned long long *surf;
    GLOBAL unsigned long long *iad;
    HitLog log;
    const long long *step;
    // LDS copy of the conductor map of cells c0i .. c0i+CW-1, c0j .. c0j+CH-1
    // (the block's deposit window and a one-cell frame; CW = 0: none)
    const uint8_t *scc;
    int c0i, c0j, CW, CH;
    // the same origin taken into [0, n) on a periodic axis, and the wrap
    // length of each axis (n when periodic, 0 when bounded)
    int c0wi, c0wj, nwx, nwy;
};

__device__ __forceinline__ PK resolve(const PushArgs &a)
{
    PK k;
    k.scc = nullptr;
    k.c0i = k.c0j = k.CW = k.CH = 0;
    k.c0wi = k.c0wj = k.nwx = k.nwy = 0;
    const int set = (int)a.info[7];
    k.g = a.g;
    k.TX = a.TX;
    k.TY = a.TY;
    k.H = a.H;
    k.WX = a.WX;
    k.WY = a.WY;
    k.tiles_y = a.tiles_y;
    k.cell_cond = to_global(a.cell_cond);
    k.E4 = to_global(a.E4);
    k.cell = to_global(set ? a.cell[1] : a.cell[0]);
    k.ox = to_global(set ? a.ox[1] : a.ox[0]);
    k.oy = to_global(set ? a.oy[1] : a.oy[0]);
    k.vx = to_global(set ? a.vx[1] : a.vx[0]);
    k.vy = to_global(set ? a.vy[1] : a.vy[0]);
    k.rho = to_global(a.rho);
    k.qdt = a.qdt;
    k.dtf = a.dtf;
    k.hq = a.hq;
    k.box_i_top = a.box_i_top;
    k.box_j_lo = a.box_j_lo;
    k.box_j_hi = a.box_j_hi;
    k.species = a.species;
    k.surf = to_global(a.surf);
    k.iad = to_global(a.iad);
    k.log = a.log;
    k.step = a.step;
    return k;
}

// Cell-by-cell walk of the straight segment (Dx, Dy) from offsets (x0, y0)
// in cell (ci, cj) across sx, sy faces (not both 0): the earlier face first,
// compared as (fx + kx)|Dy| <= (fy + ky)|Dx| (ties cross x).  Stops at the
// first cell outside a bounded axis or inside a conductor: dead = direction
// (0 +x, 1 -x, 2 +y, 3 -y) + 4 when the last cell occupied (ei, ej) lies in the
// trench box; else dead stays -1 and (ei, ej) is the final cell.
__device__ __forceinline__ void walk_cells(const PK &a, float x0, float y0, float Dx, float Dy, int sx, int sy,
                                           int &dead, int &ei, int &ej)
{
    const Geom &g = a.g;
    const float ax = fabsf(Dx), ay = fabsf(Dy);
    const float fx = sx > 0 ? 1.0f - x0 : x0, fy = sy > 0 ? 1.0f - y0 : y0;
    const int nxs = abs(sx), nys = abs(sy);
    const int di = sx > 0 ? 1 : -1, dj = sy > 0 ? 1 : -1;
    int kx = 0, ky = 0;
    while (kx < nxs || ky < nys) {
        bool gox;
        if (ky >= nys) gox = true;
        else if (kx >= nxs) gox = false;
        else gox = ((fx + (float)kx) * ay <= (fy + (float)ky) * ax);
        int ni = ei, nj = ej, dir;
        if (gox) { ni = ei + di; kx++; dir = di > 0 ? 0 : 1; }
        else { nj = ej + dj; ky++; dir = dj > 0 ? 2 : 3; }
        bool out = false;
        if (g.px) ni = wrap_hi(wrap_lo(ni, g.nx), g.nx);
        else if (ni < 0 || ni >= g.nx) out = true;
        if (g.py) nj = wrap_hi(wrap_lo(nj, g.ny), g.ny);
        else if (nj < 0 || nj >= g.ny) out = true;
        if (!out) {
            // conductor test from the block's LDS map when the cell lies in it
            int li = ni - a.c0i, lj = nj - a.c0j;
            if (g.px) { if (li < 0) li += g.nx; else if (li >= g.nx) li -= g.nx; }
            if (g.py) { if (lj < 0) lj += g.ny; else if (lj >= g.ny) lj -= g.ny; }
            const bool loc = li >= 0 && li < a.CW && lj >= 0 && lj < a.CH;
            if (loc ? a.scc[li * a.CH + lj] : a.cell_cond[(long long)ni * g.ny + nj]) out = true;
        }
        if (out) {
            const bool inbox = ei >= a.box_i_top && ej >= a.box_j_lo && ej < a.box_j_hi;
            dead = dir + (inbox ? 4 : 0);
            break;
        }
        ei = ni;
        ej = nj;
    }
}

// Leapfrog push of one particle with the bilinear gather of its cell's
// corner fields and the cell-by-cell wall test (eqs. 1-4).  Computes the new
// velocity (ux, uy), offsets (nxo, nyo) and cell (ei, ej); returns false when
// the particle was removed (class in dead, last cell occupied in ei, ej).
__device__ __forceinline__ bool push_core(const PK &a, float x0, float y0, float vx0, float vy0,
                                          float4 ea, float4 eb, int ci, int cj, int &dead, int &ei,
                                          int &ej, float &ux, float &uy, float &nxo, float &nyo)
{
    const float wx0 = 1.0f - x0, wy0 = 1.0f - y0;
    const float w00 = wx0 * wy0, w10 = x0 * wy0, w01 = wx0 * y0, w11 = x0 * y0;
    float ex = w00 * ea.x;
    ex = ex + w10 * ea.z;
    ex = ex + w01 * eb.x;
    ex = ex + w11 * eb.z;
    float ey = w00 * ea.y;
    ey = ey + w10 * ea.w;
    ey = ey + w01 * eb.y;
    ey = ey + w11 * eb.w;
    ux = vx0 + a.qdt * ex;
    uy = vy0 + a.qdt * ey;
    const float Dx = ux * a.dtf, Dy = uy * a.dtf;
    const float x1 = x0 + Dx, y1 = y0 + Dy;
    const float fsx = floorf(x1), fsy = floorf(y1);
    dead = -1;
    ei = ci;
    ej = cj;
    int sx = 0, sy = 0;
    if (!(fabsf(fsx) < 1.0e6f && fabsf(fsy) < 1.0e6f)) {
        dead = 8;
    } else {
        sx = (int)fsx;
        sy = (int)fsy;
        if (sx != 0 || sy != 0) walk_cells(a, x0, y0, Dx, Dy, sx, sy, dead, ei, ej);
    }
    nxo = x0;
    nyo = y0;
    if (dead >= 0) return false;
    nxo = x1 - (float)sx;
    nyo = y1 - (float)sy;
    if (nxo >= 1.0f) nxo = 0x1.fffffep-1f;
    if (nyo >= 1.0f) nyo = 0x1.fffffep-1f;
    return true;
}

// ---- ion recycling (Sec. III.A, III.C) --------------------------------------
// A lost ion is replaced by a thermal ion in the bulk rows 0 .. rows-1, the
// ionisation of the ambient gas.  Counter-based generator Philox4x32-10
// (Salmon, Moraes, Dror and Shaw, SC 2011): ten rounds of two 32 x 32-bit
// products (multipliers 0xD2511F53, 0xCD9E8D57), the key bumped by the Weyl
// constants 0x9E3779B9, 0xBB67AE85 between rounds.  Counter (step, bits of
// the lost ion's v_x after the kick, bits of its offsets before the move),
// keys (k0, k1) and (k0, k1 + 1):
//   cell (r0 >> 8) * rows >> 24, (r1 >> 8) * ny >> 24; offsets (r2 >> 8), (r3 >> 8) * 2^-24;
//   velocity vth sqrt(-2 ln u) (cos, sin)(2 pi v), u = ((q0 >> 8) + 1) 2^-24,
//   v = (q1 >> 8) 2^-24, in double, rounded to float.
struct Philox4 {
    unsigned x, y, z, w;
};

__device__ __forceinline__ Philox4 philox4x32_10(unsigned c0, unsigned c1, unsigned c2, unsigned c3, unsigned k0,
                                                 unsigned k1)
{
#pragma unroll
    for (int r = 0; r < 10; r++) {
        if (r > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const unsigned lo0 = 0xD2511F53u * c0, hi0 = __umulhi(0xD2511F53u, c0);
        const unsigned lo1 = 0xCD9E8D57u * c2, hi1 = __umulhi(0xCD9E8D57u, c2);
        const unsigned n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
    return Philox4{c0, c1, c2, c3};
}

struct NewIon {
    int ci, cj;
    float ox, oy, vx, vy;
};

__device__ __forceinline__ NewIon recycled_ion(unsigned long long step, float ux, float x0, float y0, unsigned k0,
                                               unsigned k1, int rows, int ny, double vth)
{
    const unsigned c0 = (unsigned)step, c1 = __float_as_uint(ux);
    const unsigned c2 = __float_as_uint(x0), c3 = __float_as_uint(y0);
    const Philox4 r = philox4x32_10(c0, c1, c2, c3, k0, k1);
    const Philox4 q = philox4x32_10(c0, c1, c2, c3, k0, k1 + 1u);
    NewIon n;
    n.ci = (int)(((unsigned long long)(r.x >> 8) * (unsigned)rows) >> 24);
    n.cj = (int)(((unsigned long long)(r.y >> 8) * (unsigned)ny) >> 24);
    n.ox = (float)(r.z >> 8) * 0x1p-24f;
    n.oy = (float)(r.w >> 8) * 0x1p-24f;
    const double u = (double)((q.x >> 8) + 1u) * 0x1p-24, v = (double)(q.y >> 8) * 0x1p-24;
    const double rad = sqrt(-2.0 * log(u)), ang = 6.283185307179586 * v;
    n.vx = (float)(vth * rad * cos(ang));
    n.vy = (float)(vth * rad * sin(ang));
    return n;
}

// push_core plus the particle's stores (velocity always; offsets if it
// stays; the cell code when it changes or the particle is removed).
__device__ __forceinline__ bool push_particle(const PK &a, int p, int c, float &x0, float &y0,
                                              float vx0, float vy0, float4 ea, float4 eb, int &ci,
                                              int &cj, int &dead, int &ei, int &ej, float &ux,
                                              float &uy)
{
    float nxo, nyo;
    const bool alive = push_core(a, x0, y0, vx0, vy0, ea, eb, ci, cj, dead, ei, ej, ux, uy, nxo, nyo);
    a.vx[p] = ux;
    a.vy[p] = uy;
    if (!alive) {
        a.cell[p] = -1 - dead;
        return false;
    }
    a.ox[p] = nxo;
    a.oy[p] = nyo;
    const int nc = (int)(((unsigned)ei << 16) | (unsigned)ej);
    if (nc != c) a.cell[p] = nc;
    x0 = nxo;
    y0 = nyo;
    ci = ei;
    cj = ej;
    return true;
}

// Records a removal: class counter in LDS, trench-bottom charge, hit ring.
__device__ __forceinline__ void record_hit(const PK &a, unsigned *tl, int dead, int ei, int ej,
                                           float ux, float uy)
{
    atomicAdd(&tl[dead], 1u);
    if (a.surf && dead == 4) gatomic_add(&a.surf[ej], 1ull);
    if (a.iad && dead == 4) {
        // impact angle to the plate normal (+x), 2-degree bins over [-90, 90)
        const float ang = atan2f(uy, ux);
        int bin = (int)floorf((ang + 1.57079632679f) * (float)(kIadBins / 3.14159265359));
        bin = bin < 0 ? 0 : (bin >= kIadBins ? kIadBins - 1 : bin);
        gatomic_add(&a.iad[bin], 1ull);
    }
    if (a.log.rec && ((a.log.species_mask >> a.species) & 1)) {
        unsigned long long k = atomicAdd(a.log.count, 1ull);
        long long slot = (long long)(k % (unsigned long long)a.log.capacity);
        int32_t *r = a.log.rec + 6 * slot;
        r[0] = (a.species << 8) | dead;
        r[1] = (int)(((unsigned)ei << 16) | (unsigned)ej);
        r[2] = __float_as_int(ux);
        r[3] = __float_as_int(uy);
        r[4] = (int)a.step[0];
        r[5] = 0;
    }
}

// Streaming (non-temporal) 16-byte particle loads and stores: each slot is
// read and written once per step, so they need not displace the field and
// charge arrays from the caches.
__device__ __forceinline__ nt_i4 ld_nt_i4(GLOBAL const int32_t *p)
{
    return __builtin_nontemporal_load((GLOBAL const nt_i4 *)p);
}
__device__ __forceinline__ nt_f4 ld_nt_f4(GLOBAL const float *p)
{
    return __builtin_nontemporal_load((GLOBAL const nt_f4 *)p);
}
__device__ __forceinline__ void st_nt_f4(GLOBAL float *p, float a, float b, float c, float d)
{
    nt_f4 v = {a, b, c, d};
    __builtin_nontemporal_store(v, (GLOBAL nt_f4 *)p);
}
__device__ __forceinline__ void st_nt_i4(GLOBAL int32_t *p, int a, int b, int c, int d)
{
    nt_i4 v = {a, b, c, d};
    __builtin_nontemporal_store(v, (GLOBAL nt_i4 *)p);
}

// Corner fields of the particle's cell (packed code c >= 0): from the
// block's LDS copy of the tile + 1-cell frame (origin e0i, e0j; EW x EH
// cells), or from global memory for a particle that left the frame.
__device__ __forceinline__ void cell_fields(const PK &a, const float4 *sE, int e0i, int e0j, int EW,
                                            int EH, int c, float4 &ea, float4 &eb)
{
    const Geom &g = a.g;
    const int ci = (int)((unsigned)c >> 16), cj = c & 0xFFFF;
    int li = ci - e0i, lj = cj - e0j;
    if (g.px) { if (li < 0) li += g.nx; else if (li >= g.nx) li -= g.nx; }
    if (g.py) { if (lj < 0) lj += g.ny; else if (lj >= g.ny) lj -= g.ny; }
    if (li >= 0 && li < EW && lj >= 0 && lj < EH) {
        const int m = 2 * (li * EH + lj);
        ea = sE[m];
        eb = sE[m + 1];
    } else {
        const long long cc = (long long)ci * g.ny + cj;
        ea = ld_f4(a.E4 + 2 * cc);
        eb = ld_f4(a.E4 + 2 * cc + 1);
    }
}

// Area weighting of one lane's particle (alive, in cell (ci, cj) at offsets
// (x0, y0)) into the block's LDS window of cell moments, or straight into the
// node charge when it lies outside the window.  Called by every lane of the
// wavefront (the merge of equal cells is wavefront-wide).
// Area weighting of one particle straight into the global charge (integer
// weights as in the LDS window path).
__device__ __forceinline__ void deposit_global(GLOBAL unsigned long long *rho, const Geom &g, int ci, int cj,
                                               unsigned ux, unsigned uy)
{
    const unsigned long long S = 65536ull;
    const int i1 = g.px ? wrap_hi(ci + 1, g.nx) : ci + 1;
    const int j1 = g.py ? wrap_hi(cj + 1, g.ny) : cj + 1;
    const unsigned long long X = ux, Y = uy;
    gatomic_add(&rho[(long long)ci * g.NY + cj], (S - X) * (S - Y));
    gatomic_add(&rho[(long long)i1 * g.NY + cj], X * (S - Y));
    gatomic_add(&rho[(long long)ci * g.NY + j1], (S - X) * Y);
    gatomic_add(&rho[(long long)i1 * g.NY + j1], X * Y);
}

template <int MERGE>
__device__ __forceinline__ void deposit_lane(const PK &a, unsigned long long *mA, unsigned long long *mB,
                                             int lane, bool alive, int ci, int cj, float x0, float y0,
                                             int i0, int j0, int WX, int WY, unsigned long long &nfb)
{
    const Geom &g = a.g;
    int key = -1;
    unsigned ux = 0, uy = 0;
    if (alive) {
        ux = (unsigned)floorf(x0 * 65536.0f);
        uy = (unsigned)floorf(y0 * 65536.0f);
        int wi = ci - i0, wj = cj - j0;
        if (g.px) { if (wi < 0) wi += g.nx; else if (wi >= g.nx) wi -= g.nx; }
        if (g.py) { if (wj < 0) wj += g.ny; else if (wj >= g.ny) wj -= g.ny; }
        if (wi >= 0 && wi < WX && wj >= 0 && wj < WY) {
            key = wi * WY + wj;
        } else {
            deposit_global(a.rho, g, ci, cj, ux, uy);
            nfb++;
        }
    }
    // wavefront merge of equal cells (all lanes take part)
    const unsigned m3 = ux * uy;
    if (MERGE > 0) {
        unsigned long long pend = __ballot(key >= 0);
        for (int it = 0; it < MERGE && pend; it++) {
            const int leader = __builtin_ctzll(pend);
            const int lk = __builtin_amdgcn_readlane(key, leader);
            const bool m = key == lk;
            const unsigned long long mask = __ballot(m);
            unsigned sx = m ? ux : 0u, sy = m ? uy : 0u;
            unsigned sh = m ? (m3 >> 16) : 0u, sl = m ? (m3 & 0xFFFFu) : 0u;
            wave_sum4_u32(sx, sy, sh, sl);
            if (lane == leader) {
                const unsigned long long cnt = (unsigned long long)__popcll(mask);
                const unsigned long long s3 = ((unsigned long long)sh << 16) + sl;
                atomicAdd(&mA[lk], (cnt << 45) + s3);
                atomicAdd(&mB[lk], (unsigned long long)sx | ((unsigned long long)sy << 29));
            }
            if (m) key = -1;
            pend &= ~mask;
        }
    }
    if (key >= 0) {
        atomicAdd(&mA[key], (1ull << 45) + (unsigned long long)m3);
        atomicAdd(&mB[key], (unsigned long long)ux | ((unsigned long long)uy << 29));
    }
}

// ---- block-local cell coordinates -------------------------------------------
// A particle's cell relative to the origin of the block's conductor map,
// taken into [0, n) on a periodic axis (c0w: the origin already in [0, n)
// there, nw = n; on a bounded axis c0w is the origin and nw = 0).  The field
// frame and the deposit window are fixed shifts of the same origin, so one
// wrapped coordinate serves all three LDS copies, and a step of the walk is
// one add.  An LDS copy holds the cell (origin + l) mod n at index l, so any
// representative of the cell modulo n that lands inside a copy reads the
// right entry.  Selects, not branches: the wrap costs the same on every lane.
__device__ __forceinline__ int map_rel(int c, int c0w, int nw)
{
    int l = c - c0w;
    l += l < 0 ? nw : 0;
    return l;
}

// A cell index one step from a valid one, back into [0, n) on a periodic
// axis (nw = n; nw = 0 leaves a bounded axis's index as it is).
__device__ __forceinline__ int wrap_step(int c, int n, int nw)
{
    c += c < 0 ? nw : 0;
    c -= c >= n ? nw : 0;
    return c;
}

// Whether the cell a step of the walk enters stops the particle (a conductor
// cell, or outside a bounded axis).  (lx, ly): its conductor-map coordinates;
// (gi, gj): its global ones, one cell from a valid cell, not yet wrapped.  The
// LDS map holds 1 for cells outside a bounded axis, so both tests agree.
__device__ __forceinline__ bool step_blocked(const PK &a, int lx, int ly, int gi, int gj)
{
    if ((unsigned)lx < (unsigned)a.CW && (unsigned)ly < (unsigned)a.CH)
        return a.scc[__umul24((unsigned)lx, (unsigned)a.CH) + ly] != 0;
    const Geom &g = a.g;
    if (g.px) gi = wrap_step(gi, g.nx, g.nx);
    else if (gi < 0 || gi >= g.nx) return true;
    if (g.py) gj = wrap_step(gj, g.ny, g.ny);
    else if (gj < 0 || gj >= g.ny) return true;
    return a.cell_cond[(long long)gi * g.ny + gj] != 0;
}

// push_core with the particle's cell also in conductor-map coordinates
// (lx, ly; moved with the particle).  The same arithmetic in the same order;
// a move of at most one face per axis (all but a few particles per million)
// is walked in straight-line code: for a diagonal move the earlier face first,
// compared as fx |Dy| <= fy |Dx| (ties cross x), then the other one.  Longer
// moves take the cell-by-cell walk of push_core.
__device__ __forceinline__ bool push_core_l(const PK &a, float x0, float y0, float vx0, float vy0,
                                            float4 ea, float4 eb, int ci, int cj, int &lx, int &ly,
                                            int &dead, int &ei, int &ej, float &ux, float &uy,
                                            float &nxo, float &nyo)
{
    const Geom &g = a.g;
    const float wx0 = 1.0f - x0, wy0 = 1.0f - y0;
    const float w00 = wx0 * wy0, w10 = x0 * wy0, w01 = wx0 * y0, w11 = x0 * y0;
    float ex = w00 * ea.x;
    ex = ex + w10 * ea.z;
    ex = ex + w01 * eb.x;
    ex = ex + w11 * eb.z;
    float ey = w00 * ea.y;
    ey = ey + w10 * ea.w;
    ey = ey + w01 * eb.y;
    ey = ey + w11 * eb.w;
    ux = vx0 + a.qdt * ex;
    uy = vy0 + a.qdt * ey;
    const float Dx = ux * a.dtf, Dy = uy * a.dtf;
    const float x1 = x0 + Dx, y1 = y0 + Dy;
    const float fsx = floorf(x1), fsy = floorf(y1);
    dead = -1;
    ei = ci;
    ej = cj;
    nxo = x0;
    nyo = y0;
    if (!(fabsf(fsx) < 1.0e6f && fabsf(fsy) < 1.0e6f)) {
        dead = 8;
        return false;
    }
    const int sx = (int)fsx, sy = (int)fsy;
    if (sx != 0 || sy != 0) {
        if ((unsigned)(sx + 1) <= 2u && (unsigned)(sy + 1) <= 2u) {
            const bool both = sx != 0 && sy != 0;
            bool gox = sy == 0;
            if (both) {
                const float fx = sx > 0 ? 1.0f - x0 : x0, fy = sy > 0 ? 1.0f - y0 : y0;
                gox = fx * fabsf(Dy) <= fy * fabsf(Dx);
            }
            const int d1x = gox ? sx : 0, d1y = gox ? 0 : sy;
            if (step_blocked(a, lx + d1x, ly + d1y, ci + d1x, cj + d1y)) {
                dead = gox ? (sx > 0 ? 0 : 1) : (sy > 0 ? 2 : 3);
            } else if (both && step_blocked(a, lx + sx, ly + sy, ci + sx, cj + sy)) {
                dead = gox ? (sy > 0 ? 2 : 3) : (sx > 0 ? 0 : 1);
                ei = wrap_step(ci + d1x, g.nx, a.nwx);
                ej = wrap_step(cj + d1y, g.ny, a.nwy);
            }
            if (dead >= 0) {
                const bool inbox = ei >= a.box_i_top && ej >= a.box_j_lo && ej < a.box_j_hi;
                dead += inbox ? 4 : 0;
                return false;
            }
            ei = wrap_step(ci + sx, g.nx, a.nwx);
            ej = wrap_step(cj + sy, g.ny, a.nwy);
        } else {
            walk_cells(a, x0, y0, Dx, Dy, sx, sy, dead, ei, ej);
            if (dead >= 0) return false;
        }
        lx += sx;
        ly += sy;
    }
    nxo = x1 - (float)sx;
    nyo = y1 - (float)sy;
    if (nxo >= 1.0f) nxo = 0x1.fffffep-1f;
    if (nyo >= 1.0f) nyo = 0x1.fffffep-1f;
    return true;
}

// Corner fields from conductor-map coordinates (lx, ly): the field frame's
// origin is the map's shifted by halo + 1 - kFieldFrame cells.
__device__ __forceinline__ void cell_fields_l(const PK &a, const float4 *sE, int sh, int EW, int EH, int lx,
                                              int ly, int ci, int cj, float4 &ea, float4 &eb)
{
    const int li = lx - sh, lj = ly - sh;
    if ((unsigned)li < (unsigned)EW && (unsigned)lj < (unsigned)EH) {
        const int m = 2 * (int)(__umul24((unsigned)li, (unsigned)EH) + lj);
        ea = sE[m];
        eb = sE[m + 1];
    } else {
        const long long cc = (long long)ci * a.g.ny + cj;
        ea = ld_f4(a.E4 + 2 * cc);
        eb = ld_f4(a.E4 + 2 * cc + 1);
    }
}

// deposit_lane with the deposit-window coordinates given (wi, wj: the
// conductor-map ones less 1).
template <int MERGE>
__device__ __forceinline__ void deposit_lane_l(const PK &a, unsigned long long *mA, unsigned long long *mB,
                                               int lane, bool alive, int ci, int cj, float x0, float y0,
                                               int wi, int wj, int WX, int WY, unsigned long long &nfb)
{
    int key = -1;
    unsigned ux = 0, uy = 0;
    if (alive) {
        // offsets lie in [0, 1): truncation is the floor
        ux = (unsigned)(x0 * 65536.0f);
        uy = (unsigned)(y0 * 65536.0f);
        if ((unsigned)wi < (unsigned)WX && (unsigned)wj < (unsigned)WY) {
            key = (int)__umul24((unsigned)wi, (unsigned)WY) + wj;
        } else {
            deposit_global(a.rho, a.g, ci, cj, ux, uy);
            nfb++;
        }
    }
    // both factors below 2^16: the 24-bit product is exact
    const unsigned m3 = __umul24(ux, uy);
    if (MERGE > 0) {
        unsigned long long pend = __ballot(key >= 0);
        for (int it = 0; it < MERGE && pend; it++) {
            const int leader = __builtin_ctzll(pend);
            const int lk = __builtin_amdgcn_readlane(key, leader);
            const bool m = key == lk;
            const unsigned long long mask = __ballot(m);
            unsigned sx = m ? ux : 0u, sy = m ? uy : 0u;
            unsigned sh = m ? (m3 >> 16) : 0u, sl = m ? (m3 & 0xFFFFu) : 0u;
            wave_sum4_u32(sx, sy, sh, sl);
            if (lane == leader) {
                const unsigned long long cnt = (unsigned long long)__popcll(mask);
                const unsigned long long s3 = ((unsigned long long)sh << 16) + sl;
                atomicAdd(&mA[lk], (cnt << 45) + s3);
                atomicAdd(&mB[lk], (unsigned long long)sx | ((unsigned long long)sy << 29));
            }
            if (m) key = -1;
            pend &= ~mask;
        }
    }
    if (key >= 0) {
        atomicAdd(&mA[key], (1ull << 45) + (unsigned long long)m3);
        atomicAdd(&mB[key], (unsigned long long)ux | ((unsigned long long)uy << 29));
    }
}

// One tile of particles per block (table entry): gather + push + wall test,
// then area weighting of the new positions into the block's LDS window of
// cell moments (count, sum ux, sum uy, sum ux*uy with ux, uy the 16-bit
// quantised offsets).  Lanes of a wavefront that land in the same cell are
// summed first when MERGE > 0 (up to MERGE distinct cells per wavefront),
// so runs of particles in one cell cost one LDS atomic per cell.
// Particles that drifted beyond the window add their four corner weights to
// global memory directly.  The window is flushed to the node charge at the end.
// The dispatcher hands blocks to the 8 XCDs in turn (block b to XCD b mod 8),
// each with its own L2.  In every group of 8 K blocks this gives XCD x the K
// consecutive table entries x K .. x K + K - 1 (a bijection on [0, G); a last,
// partial group is split the same way), so the blocks of one tile, which read
// the same field frame and conductor map, mostly share an L2, while every XCD
// still gets an equal share of each group.
__device__ __forceinline__ int xcd_swizzle(int b, int G)
{
    constexpr int K = 16;
    const int base = b / (8 * K) * (8 * K);
    const int n = min(8 * K, G - base);
    const int o = b - base, x = o & 7, q = n >> 3, r = n & 7;
    return base + (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + (o >> 3);
}

template <bool PUSH, int U, int MERGE>
__global__ __launch_bounds__(kPushThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_push(const PushArgs *A, Tab t)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int bid = xcd_swizzle((int)blockIdx.x, (int)gridDim.x);
    const int ku = unit_of(t, bid);
    const PushArgs &aa = A[t.id[ku]];
    const int lb = bid - t.boff[ku];
    if ((long long)lb >= aa.info[1]) return;
    const int4 ent = aa.table[lb];
    PK a = resolve(aa);
    unsigned long long *const tally = aa.tally;
    unsigned long long *const fallbacks = aa.fallbacks;
    const int tile = ent.x, start = ent.y, end = ent.z;
    const int ti = tile / a.tiles_y, tj = tile - ti * a.tiles_y;
    const int i0 = ti * a.TX - a.H, j0 = tj * a.TY - a.H;
    const int WX = a.WX, WY = a.WY, WC = WX * WY;
    // per window cell: mA = count << 45 | sum(ux*uy), mB = sum(ux) | sum(uy) << 29
    // (at most 8192 particles per block keep every field free of carries)
    unsigned long long *mA = (unsigned long long *)smem;
    unsigned long long *mB = mA + WC;
    unsigned *tl = (unsigned *)(mB + WC);
    // corner fields of the tile + 1-cell frame
    float4 *sE = (float4 *)(smem + (((size_t)WC * 16 + kNClass * 4 + 15) & ~(size_t)15));
    const int EW = a.TX + 2 * kFieldFrame, EH = a.TY + 2 * kFieldFrame;
    const int e0i = ti * a.TX - kFieldFrame, e0j = tj * a.TY - kFieldFrame;
    // conductor map of the window and a one-cell frame, after the fields
    uint8_t *scc = (uint8_t *)(sE + 2 * EW * EH);
    a.scc = scc;
    a.c0i = i0 - 1;
    a.c0j = j0 - 1;
    a.nwx = aa.g.px ? aa.g.nx : 0;
    a.nwy = aa.g.py ? aa.g.ny : 0;
    a.c0wi = a.nwx ? ((a.c0i % a.nwx) + a.nwx) % a.nwx : a.c0i;
    a.c0wj = a.nwy ? ((a.c0j % a.nwy) + a.nwy) % a.nwy : a.c0j;
    a.CW = PUSH ? WX + 2 : 0;
    a.CH = WY + 2;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const Geom g = a.g;
    for (int k = tid; k < WC; k += kPushThreads) {
        mA[k] = 0ull;
        mB[k] = 0ull;
    }
    if (tid < kNClass) tl[tid] = 0u;
    if (PUSH) {
        for (int k = tid; k < 2 * EW * EH; k += kPushThreads) {
            const int m = k >> 1, li = m / EH, lj = m - li * EH;
            int ci = e0i + li, cj = e0j + lj;
            if (g.px) ci = wrap_hi(wrap_lo(ci, g.nx), g.nx);
            if (g.py) cj = wrap_hi(wrap_lo(cj, g.ny), g.ny);
            if (ci >= 0 && ci < g.nx && cj >= 0 && cj < g.ny)
                sE[k] = ld_f4(a.E4 + 2 * ((long long)ci * g.ny + cj) + (k & 1));
        }
        for (int k = tid; k < a.CW * a.CH; k += kPushThreads) {
            const int li = k / a.CH, lj = k - li * a.CH;
            int ci = a.c0i + li, cj = a.c0j + lj;
            if (g.px) ci = ((ci % g.nx) + g.nx) % g.nx;
            if (g.py) cj = ((cj % g.ny) + g.ny) % g.ny;
            // cells outside a bounded axis are never looked up (the walk
            // tests the domain first)
            scc[k] = (ci >= 0 && ci < g.nx && cj >= 0 && cj < g.ny) ? a.cell_cond[(long long)ci * g.ny + cj] : 1;
        }
    }
    __syncthreads();

    unsigned long long nfb = 0;
    if constexpr (U == 4) {
        // 4 consecutive particles per thread per pass, moved with 16-byte
        // loads and stores where the 4 slots lie inside [start, end) (the
        // head and tail of the range go element by element).  Slots of
        // removed particles in a full vector are written back unchanged.
        // A pass's full vectors are loaded at the end of the pass before it,
        // ahead of that pass's stores: the wait at the top of a pass is then
        // for the loads alone, and their registers are not those of the
        // stores still in flight.  The wave issues them at raised priority,
        // so that they leave before other waves' arithmetic.
        nt_i4 c4 = {-1, -1, -1, -1};
        nt_f4 x4 = {0.f, 0.f, 0.f, 0.f}, y4 = x4, u4 = x4, w4 = x4;
        auto no_pass = [&]() {
            c4 = nt_i4{-1, -1, -1, -1};
            x4 = y4 = u4 = w4 = nt_f4{0.f, 0.f, 0.f, 0.f};
        };
        auto load_pass = [&](int v) {
            __builtin_amdgcn_s_setprio(3);
            c4 = ld_nt_i4(a.cell + v);
            x4 = ld_nt_f4(a.ox + v);
            y4 = ld_nt_f4(a.oy + v);
            if (PUSH) {
                u4 = ld_nt_f4(a.vx + v);
                w4 = ld_nt_f4(a.vy + v);
            }
            __builtin_amdgcn_s_setprio(0);
        };
        {
            const int v = (start & ~3) + 4 * tid;
            if (v >= start && v + 4 <= end) load_pass(v);
            else no_pass();
        }
        for (int vb = start & ~3; vb < end; vb += 4 * kPushThreads) {
            const int v = vb + 4 * tid;
            const bool full = v >= start && v + 4 <= end;
            int cv[4];
            float xv[4], yv[4], uxv[4], uyv[4];
            if (full) {
                cv[0] = c4.x; cv[1] = c4.y; cv[2] = c4.z; cv[3] = c4.w;
                xv[0] = x4.x; xv[1] = x4.y; xv[2] = x4.z; xv[3] = x4.w;
                yv[0] = y4.x; yv[1] = y4.y; yv[2] = y4.z; yv[3] = y4.w;
                uxv[0] = u4.x; uxv[1] = u4.y; uxv[2] = u4.z; uxv[3] = u4.w;
                uyv[0] = w4.x; uyv[1] = w4.y; uyv[2] = w4.z; uyv[3] = w4.w;
            } else {
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int p = v + k;
                    const bool in = p >= start && p < end;
                    cv[k] = in ? a.cell[p] : -1;
                    xv[k] = in ? a.ox[p] : 0.f;
                    yv[k] = in ? a.oy[p] : 0.f;
                    uxv[k] = (PUSH && in) ? a.vx[p] : 0.f;
                    uyv[k] = (PUSH && in) ? a.vy[p] : 0.f;
                }
            }
            bool alv[4];
            // slots holding a live particle on entry (cv[k] becomes its new code)
            unsigned live0 = 0u;
            // the field frame's origin relative to the conductor map's
            const int fsh = a.H + 1 - kFieldFrame;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int c = cv[k];
                bool alive = false;
                int ci = 0, cj = 0, lx = -1, ly = -1;
                if (c >= 0) {
                    ci = (int)((unsigned)c >> 16);
                    cj = c & 0xFFFF;
                    lx = map_rel(ci, a.c0wi, a.nwx);
                    ly = map_rel(cj, a.c0wj, a.nwy);
                    alive = true;
                    live0 |= 1u << k;
                    if (PUSH) {
                        // the corner fields of this particle's cell only (fewer
                        // live registers than gathering all four first)
                        float4 ea, eb;
                        cell_fields_l(a, sE, fsh, EW, EH, lx, ly, ci, cj, ea, eb);
                        int dead, ei, ej;
                        float ux, uy, nxo, nyo;
                        alive = push_core_l(a, xv[k], yv[k], uxv[k], uyv[k], ea, eb, ci, cj, lx, ly,
                                            dead, ei, ej, ux, uy, nxo, nyo);
                        uxv[k] = ux;
                        uyv[k] = uy;
                        if (!alive) {
                            cv[k] = -1 - dead;
                            record_hit(a, tl, dead, ei, ej, ux, uy);
                        } else {
                            cv[k] = (int)(((unsigned)ei << 16) | (unsigned)ej);
                            xv[k] = nxo;
                            yv[k] = nyo;
                            ci = ei;
                            cj = ej;
                        }
                    }
                }
                alv[k] = alive;
                deposit_lane_l<MERGE>(a, mA, mB, lane, alive, ci, cj, xv[k], yv[k], lx - 1, ly - 1, WX, WY,
                                      nfb);
            }
            {
                // the next pass's vectors (slots v + 1024 .. v + 1027 lie at or
                // after start, so full means inside [start, end))
                const int vn = v + 4 * kPushThreads;
                if (vn + 4 <= end) load_pass(vn);
                else no_pass();
            }
            if (PUSH) {
                if (full) {
                    // every code of the vector (unchanged ones rewritten as read)
                    st_nt_i4(a.cell + v, cv[0], cv[1], cv[2], cv[3]);
                    st_nt_f4(a.vx + v, uxv[0], uxv[1], uxv[2], uxv[3]);
                    st_nt_f4(a.vy + v, uyv[0], uyv[1], uyv[2], uyv[3]);
                    st_nt_f4(a.ox + v, xv[0], xv[1], xv[2], xv[3]);
                    st_nt_f4(a.oy + v, yv[0], yv[1], yv[2], yv[3]);
                } else {
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        if (!((live0 >> k) & 1u)) continue;   // outside the range, or removed earlier
                        a.cell[v + k] = cv[k];
                        a.vx[v + k] = uxv[k];
                        a.vy[v + k] = uyv[k];
                        if (alv[k]) {
                            a.ox[v + k] = xv[k];
                            a.oy[v + k] = yv[k];
                        }
                    }
                }
            }
        }
    } else
    // U particles per thread per pass: all their loads are issued
    // before any is used, so each wave keeps several requests in flight.
    // The loop bound is uniform per block so whole wavefronts stay active.
    for (int base = start; base < end; base += U * kPushThreads) {
        int cu[U];
        float xu[U], yu[U], vxu[U], vyu[U];
        float4 eau[U], ebu[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int p = base + u * kPushThreads + tid;
            cu[u] = (p < end) ? a.cell[p] : -1;
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int p = base + u * kPushThreads + tid;
            if (p < end) {
                xu[u] = a.ox[p];
                yu[u] = a.oy[p];
                if (PUSH) {
                    vxu[u] = a.vx[p];
                    vyu[u] = a.vy[p];
                }
            }
        }
        if (PUSH) {
#pragma unroll
            for (int u = 0; u < U; u++) {
                eau[u] = ebu[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (cu[u] >= 0) cell_fields(a, sE, e0i, e0j, EW, EH, cu[u], eau[u], ebu[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int p = base + u * kPushThreads + tid;
            int c = cu[u];
            bool alive = false;
            float x0 = 0.f, y0 = 0.f;
            int ci = 0, cj = 0;
            if (c >= 0) {
                x0 = xu[u];
                y0 = yu[u];
                ci = (int)((unsigned)c >> 16);
                cj = c & 0xFFFF;
                alive = true;
                if (PUSH) {
                    int dead, ei, ej;
                    float vnx, vny;
                    alive = push_particle(a, p, c, x0, y0, vxu[u], vyu[u], eau[u], ebu[u], ci, cj,
                                          dead, ei, ej, vnx, vny);
                    if (!alive) record_hit(a, tl, dead, ei, ej, vnx, vny);
                }
            }
            deposit_lane<MERGE>(a, mA, mB, lane, alive, ci, cj, x0, y0, i0, j0, WX, WY, nfb);
        }
    }
    if (nfb) atomicAdd(fallbacks, nfb);
    __syncthreads();
    // flush: node (wa, wb) of the window collects the four cells around it
    const unsigned long long S = 65536ull;
    const int WN = (WX + 1) * (WY + 1);
    for (int k = tid; k < WN; k += kPushThreads) {
        const int wa = k / (WY + 1), wb = k - wa * (WY + 1);
        unsigned long long v = 0ull;
        bool any = false;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int ca = wa - (q & 1), cb = wb - (q >> 1);
            if (ca < 0 || ca >= WX || cb < 0 || cb >= WY) continue;
            const int m = ca * WY + cb;
            const unsigned long long A = mA[m];
            if (A == 0ull) continue;
            any = true;
            const unsigned long long B = mB[m];
            const unsigned long long M0 = A >> 45, M3 = A & ((1ull << 45) - 1ull);
            const unsigned long long M1 = B & ((1ull << 29) - 1ull), M2 = B >> 29;
            if (q == 0) v += S * S * M0 - S * M1 - S * M2 + M3;  // node is the cell's 00 corner
            else if (q == 1) v += S * M1 - M3;                    // 10 corner of cell (wa-1, wb)
            else if (q == 2) v += S * M2 - M3;                    // 01 corner of cell (wa, wb-1)
            else v += M3;                                         // 11 corner of cell (wa-1, wb-1)
        }
        if (!any || v == 0ull) continue;
        int gi = i0 + wa, gj = j0 + wb;
        if (g.px) { gi = ((gi % g.NX) + g.NX) % g.NX; }
        else if (gi < 0 || gi >= g.NX) continue;
        if (g.py) { gj = ((gj % g.NY) + g.NY) % g.NY; }
        else if (gj < 0 || gj >= g.NY) continue;
        gatomic_add(&a.rho[(long long)gi * g.NY + gj], v);
    }
    if (PUSH && tid < kNClass && tl[tid]) atomicAdd(&tally[tid], (unsigned long long)tl[tid]);
}

template <bool PUSH>
static void launch_push_t(const PushArgs *A, const Tab &t, int unroll, int merge, size_t lds,
                          hipStream_t s)
{
    const dim3 gr(tab_blocks(t)), bl(kPushThreads);
#define PUSH_CASE(U, M)                                                                   \
    if (unroll == U && merge == M) {                                                      \
        hipLaunchKernelGGL((k_push<PUSH, U, M>), gr, bl, lds, s, A, t);                   \
        return;                                                                           \
    }
    PUSH_CASE(1, 0) PUSH_CASE(2, 0) PUSH_CASE(4, 0)
    PUSH_CASE(1, 2) PUSH_CASE(2, 2) PUSH_CASE(4, 2)
    PUSH_CASE(1, 4) PUSH_CASE(2, 4) PUSH_CASE(4, 4)
#undef PUSH_CASE
    hipLaunchKernelGGL((k_push<PUSH, 2, 0>), gr, bl, lds, s, A, t);
}

void launch_push(const PushArgs *A, const Tab &t, bool push, int unroll, int merge, size_t lds,
                 hipStream_t s)
{
    if (!t.n) return;
    if (push) launch_push_t<true>(A, t, unroll, merge, lds, s);
    else launch_push_t<false>(A, t, unroll, merge, lds, s);
}

// Leapfrog start: v -= (alpha dt / 2) E(x), same gather as the push.
__global__ void k_rewind(const PushArgs *A, Tab t)
{
    const int ku = unit_of(t, (int)blockIdx.x);
    const PushArgs &aa = A[t.id[ku]];
    const long long p = (long long)((int)blockIdx.x - t.boff[ku]) * blockDim.x + threadIdx.x;
    if (p >= aa.info[2 + aa.info[7]]) return;
    const PK a = resolve(aa);
    const int c = a.cell[p];
    if (c < 0) return;
    const int ci = (int)((unsigned)c >> 16), cj = c & 0xFFFF;
    const long long cc = (long long)ci * a.g.ny + cj;
    const float4 ea = ld_f4(a.E4 + 2 * cc), eb = ld_f4(a.E4 + 2 * cc + 1);
    const float x0 = a.ox[p], y0 = a.oy[p];
    const float wx0 = 1.0f - x0, wy0 = 1.0f - y0;
    const float w00 = wx0 * wy0, w10 = x0 * wy0, w01 = wx0 * y0, w11 = x0 * y0;
    float ex = w00 * ea.x;
    ex = ex + w10 * ea.z;
    ex = ex + w01 * eb.x;
    ex = ex + w11 * eb.z;
    float ey = w00 * ea.y;
    ey = ey + w10 * ea.w;
    ey = ey + w01 * eb.y;
    ey = ey + w11 * eb.w;
    a.vx[p] = a.vx[p] - a.hq * ex;
    a.vy[p] = a.vy[p] - a.hq * ey;
}

void launch_rewind(const PushArgs *A, const Tab &t, hipStream_t s)
{
    if (t.n) hipLaunchKernelGGL(k_rewind, dim3(tab_blocks(t)), dim3(256), 0, s, A, t);
}

// ---------------------------------------------------------------------------
// diagnostics (not on the stepping path): float64 sums in a fixed order
// ---------------------------------------------------------------------------

__device__ __forceinline__ void diag_block_sum(double v, double *part)
{
    __shared__ double sh[256];
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// Ion recycling after a push: every slot whose ion that push removed at a
// wall or conductor (code -1 - class, class 0..7) takes a thermal ion in the
// bulk rows, and the new ion's charge goes straight into rho.  The push
// leaves the lost ion's kicked v_x and its offsets before the move in the
// slot; with the step they form the generator's counter.  One thread per
// slot of the storage set in use.
__global__ __launch_bounds__(256) void k_recycle(const PushArgs *A, Tab t)
{
    const int ku = unit_of(t, (int)blockIdx.x);
    const PushArgs &a = A[t.id[ku]];
    const int set = (int)a.info[7];
    const long long p = (long long)((int)blockIdx.x - t.boff[ku]) * 256 + threadIdx.x;
    if (p >= a.info[2 + set]) return;
    GLOBAL int32_t *cell = to_global(a.cell[set]);
    const int c = cell[p];
    if (c >= 0 || c < -8) return;
    GLOBAL float *ox = to_global(a.ox[set]), *oy = to_global(a.oy[set]);
    GLOBAL float *vx = to_global(a.vx[set]), *vy = to_global(a.vy[set]);
    const NewIon n = recycled_ion((unsigned long long)*a.step, vx[p], ox[p], oy[p], a.recycle_key[0],
                                  a.recycle_key[1], a.recycle_rows, a.g.ny, a.recycle_vth);
    cell[p] = (int)(((unsigned)n.ci << 16) | (unsigned)n.cj);
    ox[p] = n.ox;
    oy[p] = n.oy;
    vx[p] = n.vx;
    vy[p] = n.vy;
    deposit_global(to_global(a.rho), a.g, n.ci, n.cj, (unsigned)floorf(n.ox * 65536.0f),
                   (unsigned)floorf(n.oy * 65536.0f));
}

void launch_recycle(const PushArgs *A, const Tab &t, hipStream_t s)
{
    if (!t.n) return;
    hipLaunchKernelGGL(k_recycle, dim3(tab_blocks(t)), dim3(256), 0, s, A, t);
}

// Bound by reading cells and velocities (12 bytes a slot).  A load behind a
// test of the slot's cell, and one slot a round, ran at 1.7 TB/s (92M slots:
// 657 us); all loads of eight slots at once: 190 us.
__global__ __launch_bounds__(256) void k_kinetic(const PushArgs *A, int unit, double *part)
{
    const PushArgs &aa = A[unit];
    const int set = (int)aa.info[7];
    const long long n = aa.info[2 + set];
    const int32_t *cell = aa.cell[set];
    const float *vx = aa.vx[set], *vy = aa.vy[set];
    double s = 0.0;
    constexpr int U = 8;
    const long long step = (long long)gridDim.x * 256;
    for (long long p0 = (long long)blockIdx.x * 256 + threadIdx.x; p0 < n; p0 += U * step) {
        int c[U];
        float x[U], y[U];
#pragma unroll
        for (int k = 0; k < U; k++) {
            const long long p = p0 + k * step < n ? p0 + k * step : p0;
            c[k] = cell[p];
            x[k] = vx[p];
            y[k] = vy[p];
        }
#pragma unroll
        for (int k = 0; k < U; k++) {
            const double e = (double)x[k] * x[k] + (double)y[k] * y[k];
            s += p0 + k * step < n && c[k] >= 0 ? e : 0.0;
        }
    }
    diag_block_sum(s, part);
}

__global__ __launch_bounds__(256) void k_field_energy(const Inst *insts, int inst, double *part)
{
    const Inst &I = insts[inst];
    const Geom g = I.g;
    const long long n = (long long)g.NX * g.NY;
    double s = 0.0;
    for (long long k = (long long)blockIdx.x * 256 + threadIdx.x; k < n; k += (long long)gridDim.x * 256) {
        const int i = (int)(k / g.NY), j = (int)(k % g.NY);
        const float2 e = node_field(g, I.node_cond, I.phi, i, j);
        s += (double)e.x * e.x + (double)e.y * e.y;
    }
    diag_block_sum(0.5 * s, part);
}

// The kDiagBlocks partials in block order: one thread adds, from LDS (from
// memory, a trip at a time, 31 us; 5.2 so).
__global__ __launch_bounds__(256) void k_sum_partials(const double *part, double *out)
{
    __shared__ double sh[kDiagBlocks];
    for (int k = threadIdx.x; k < kDiagBlocks; k += 256) sh[k] = part[k];
    __syncthreads();
    if (threadIdx.x != 0) return;
    double s = 0.0;
#pragma unroll 16
    for (int k = 0; k < kDiagBlocks; k++) s += sh[k];
    *out = s;
}

void launch_kinetic(const PushArgs *A, int unit, double *part, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_kinetic, dim3(kDiagBlocks), dim3(256), 0, s, A, unit, part);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, s, part, out);
}

void launch_field_energy(const Inst *I, int inst, double *part, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_field_energy, dim3(kDiagBlocks), dim3(256), 0, s, I, inst, part);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, s, part, out);
}

// ---------------------------------------------------------------------------
// re-binning: counting sort of live particles by tile (order inside a tile
// is arbitrary; results never depend on particle order)
// ---------------------------------------------------------------------------

__device__ __forceinline__ int tile_of(int c, int lx, int ly, int tiles_y)
{
    const int i = (int)((unsigned)c >> 16), j = c & 0xFFFF;
    return (i >> lx) * tiles_y + (j >> ly);
}

// Adds 1 per active lane to counters[key], one atomic per distinct key in
// the wavefront; returns the lane's slot (previous value + rank).
__device__ __forceinline__ unsigned wave_add(unsigned *counters, int key, bool active)
{
    unsigned mine = 0;
    const int lane = __lane_id();
    unsigned long long pend = __ballot(active);
    while (pend) {
        const int leader = __builtin_ctzll(pend);
        const int lk = __shfl(key, leader, 64);
        const unsigned long long m = __ballot(active && key == lk) & pend;
        unsigned base = 0;
        if (lane == leader) base = atomicAdd(&counters[lk], (unsigned)__popcll(m));
        base = __shfl(base, leader, 64);
        if ((m >> lane) & 1ull) mine = base + (unsigned)__popcll(m & ((1ull << lane) - 1ull));
        pend &= ~m;
    }
    return mine;
}

// A slot is binned when its code is non-negative and names a cell of the
// grid; a non-negative code outside the grid is counted in bad[0] and dropped.
__device__ __forceinline__ bool live_code(int c, int nx, int ny)
{
    return c >= 0 && (int)((unsigned)c >> 16) < nx && (c & 0xFFFF) < ny;
}

// Count and scatter work in blocks of kBinPer consecutive slots.  Between
// re-binnings particles drift less than a tile, so a block's particles lie
// in a 5 x 5 box of tiles centred on its home tile (the tile of the first
// live particle among thread 0's slots, which may itself have moved a tile;
// tile indices taken modulo the tile grid, so the box is an index map
// whatever the boundaries).  The scatter counts its particles per box tile
// in LDS (one LDS atomic per distinct tile per wavefront), reserves that
// many consecutive destination slots with one global atomic per tile and
// hands them out in LDS; particles outside the box use global
// wavefront-aggregated atomics.
constexpr int kBinPer = 2048;
constexpr int kBox = 5;
constexpr int kBoxN = kBox * kBox;

// Source (info[7]) and destination sets of a re-binning.
struct BView {
    const int32_t *cell;
    const float *ox, *oy, *vx, *vy;
    int32_t *cell2;
    float *ox2, *oy2, *vx2, *vy2;
    long long slots;
    int src, dst;
};

__device__ __forceinline__ BView bview(const BinArgs &a)
{
    BView v;
    v.src = (int)a.info[7];
    v.dst = 1 - v.src;
    v.cell = a.cell[v.src];
    v.ox = a.ox[v.src];
    v.oy = a.oy[v.src];
    v.vx = a.vx[v.src];
    v.vy = a.vy[v.src];
    v.cell2 = a.cell[v.dst];
    v.ox2 = a.ox[v.dst];
    v.oy2 = a.oy[v.dst];
    v.vx2 = a.vx[v.dst];
    v.vy2 = a.vy[v.dst];
    v.slots = a.info[2 + v.src];
    return v;
}

// A block's box: tile rows ti .. ti+kBox-1 and columns tj .. tj+kBox-1 (modulo tx, ty).
struct TileBox {
    int ti, tj, tx, ty;
    bool on;
};

// Local index of the tile of live code c in the box, or -1.
__device__ __forceinline__ int box_index(const TileBox &b, int c, int lx, int ly)
{
    if (!b.on) return -1;
    int di = (int)(((unsigned)c >> 16) >> lx) - b.ti, dj = (int)((unsigned)(c & 0xFFFF) >> ly) - b.tj;
    if (di < 0) di += b.tx;
    else if (di >= b.tx) di -= b.tx;
    if (dj < 0) dj += b.ty;
    else if (dj >= b.ty) dj -= b.ty;
    return (di < kBox && dj < kBox) ? di * kBox + dj : -1;
}

// Global tile of local index k of the box.
__device__ __forceinline__ int box_tile(const TileBox &b, int k)
{
    int ti = b.ti + k / kBox, tj = b.tj + k % kBox;
    if (ti < 0) ti += b.tx;
    else if (ti >= b.tx) ti -= b.tx;
    if (tj < 0) tj += b.ty;
    else if (tj >= b.ty) tj -= b.ty;
    return ti * b.ty + tj;
}

// Scatter pass: loads the block's cell codes (all loads issued before
// use), sets up its box (shared home) and counts the live ones per box tile
// in hist (zeroed here).
constexpr int kBinRP = kBinPer / 256;
__device__ __forceinline__ TileBox bin_local_count(const BinArgs &a, const BView &v, long long lo, long long hi,
                                                   unsigned *hist, int *home, int (&cv)[kBinRP])
{
#pragma unroll
    for (int r8 = 0; r8 < kBinRP; r8++) {
        const long long p = lo + r8 * 256 + threadIdx.x;
        cv[r8] = p < hi ? v.cell[p] : -1;
    }
    if (threadIdx.x < kBoxN) hist[threadIdx.x] = 0u;
    if (threadIdx.x == 0) {
        int h = -1;
#pragma unroll
        for (int r8 = 0; r8 < kBinRP; r8++)
            if (h < 0 && live_code(cv[r8], a.nx, a.ny)) h = cv[r8];
        *home = h;
    }
    __syncthreads();
    TileBox b;
    const int h = *home;
    b.on = h >= 0;
    b.ty = a.tiles_y;
    b.tx = a.ntiles / a.tiles_y;
    b.ti = b.on ? (int)(((unsigned)h >> 16) >> a.lx) - kBox / 2 : 0;
    b.tj = b.on ? (int)((unsigned)(h & 0xFFFF) >> a.ly) - kBox / 2 : 0;
#pragma unroll
    for (int r8 = 0; r8 < kBinRP; r8++) {
        const int c = cv[r8];
        const bool act = live_code(c, a.nx, a.ny);
        const int k = act ? box_index(b, c, a.lx, a.ly) : -1;
        wave_add(hist, k < 0 ? 0 : k, act && k >= 0);
    }
    __syncthreads();
    return b;
}

// Count pass: the block's live particles per tile in an LDS histogram over
// the whole tile grid (tiles beyond kCountLds in global counts), added to
// the global counts once per non-zero tile; codes outside the grid in bad.
// (No box here: the count has no home tile to wait for, and the scatter
// places every particle counted for a tile in that tile's range whichever
// path counted it.)
constexpr int kCountLds = 2048;

__global__ __launch_bounds__(256) void k_bin_count(const BinArgs *B, Tab t)
{
    __shared__ unsigned hist[kCountLds];
    const int ku = unit_of(t, (int)blockIdx.x);
    const BinArgs &a = B[t.id[ku]];
    const BView v = bview(a);
    const long long n = v.slots;
    const long long lo = (long long)((int)blockIdx.x - t.boff[ku]) * kBinPer;
    if (lo >= n) return;
    const long long hi = lo + kBinPer < n ? lo + kBinPer : n;
    const int nl = a.ntiles < kCountLds ? a.ntiles : kCountLds;
    int cv[kBinRP];
#pragma unroll
    for (int r8 = 0; r8 < kBinRP; r8++) {
        const long long p = lo + r8 * 256 + threadIdx.x;
        cv[r8] = p < hi ? v.cell[p] : -1;
    }
    for (int k = threadIdx.x; k < nl; k += 256) hist[k] = 0u;
    __syncthreads();
#pragma unroll
    for (int r8 = 0; r8 < kBinRP; r8++) {
        const int c = cv[r8];
        const bool act = live_code(c, a.nx, a.ny);
        if (c >= 0 && !act) atomicAdd(a.bad, 1ull);
        const int key = act ? tile_of(c, a.lx, a.ly, a.tiles_y) : 0;
        wave_add(hist, key, act && key < kCountLds);
        wave_add(a.counts, key, act && key >= kCountLds);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nl; k += 256)
        if (hist[k]) atomicAdd(&a.counts[k], hist[k]);
}

// Single work-group: exclusive scans of the tile counts and of the blocks
// per tile; writes the cursor for the scatter and the totals.
__global__ __launch_bounds__(1024) void k_bin_scan(const BinArgs *B, Tab t)
{
    const BinArgs &a = B[t.id[blockIdx.x]];
    __shared__ unsigned long long sp[1024], sb[1024];
    const int tid = threadIdx.x, nt = blockDim.x;
    const int per = (a.ntiles + nt - 1) / nt;
    const int lo = tid * per, hi = min(a.ntiles, lo + per);
    unsigned long long s = 0, sbk = 0;
    for (int t = lo; t < hi; t++) {
        unsigned c = a.counts[t];
        s += c;
        sbk += (c + a.chunk - 1) / a.chunk;
    }
    sp[tid] = s;
    sb[tid] = sbk;
    __syncthreads();
    for (int o = 1; o < nt; o <<= 1) {
        unsigned long long x = tid >= o ? sp[tid - o] : 0, y = tid >= o ? sb[tid - o] : 0;
        __syncthreads();
        sp[tid] += x;
        sb[tid] += y;
        __syncthreads();
    }
    unsigned long long off = sp[tid] - s, boff = sb[tid] - sbk;
    for (int t = lo; t < hi; t++) {
        unsigned c = a.counts[t];
        a.offsets[t] = (unsigned)off;
        a.cursor[t] = (unsigned)off;
        a.boff[t] = (unsigned)boff;
        off += c;
        boff += (c + a.chunk - 1) / a.chunk;
    }
    if (tid == nt - 1) {
        a.info[0] = (long long)sp[tid];
        a.info[1] = (long long)sb[tid];
        a.info[2 + (1 - (int)a.info[7])] = (long long)sp[tid];
        // the binned slots and their push blocks: particles appended later
        // (secondary emission) get push blocks after these
        a.info[4] = (long long)sp[tid];
        a.info[5] = (long long)sb[tid];
    }
}

// Push-block table of the new set; clears the tile counts for the next
// re-binning.
__global__ void k_bin_table(const BinArgs *B, Tab tb)
{
    const int ku = unit_of(tb, (int)blockIdx.x);
    const BinArgs &a = B[tb.id[ku]];
    const int t = ((int)blockIdx.x - tb.boff[ku]) * blockDim.x + threadIdx.x;
    if (t >= a.ntiles) return;
    const unsigned c = a.counts[t], o = a.offsets[t], b0 = a.boff[t];
    const unsigned nb = (c + a.chunk - 1) / a.chunk;
    for (unsigned k = 0; k < nb; k++) {
        unsigned s = o + k * a.chunk;
        unsigned e = min(o + c, s + (unsigned)a.chunk);
        a.table[b0 + k] = make_int4(t, (int)s, (int)e, 0);
    }
    a.counts[t] = 0u;
}

__device__ __forceinline__ unsigned gcd_u(unsigned x, unsigned y)
{
    while (y) {
        unsigned t = x % y;
        x = y;
        y = t;
    }
    return x;
}

// Scatter: the m particles a block sends to tile t take its reserved slots
// base..base+m-1, in the order r -> (r * stride) mod m (r = arrival rank,
// stride near 0.618 m and coprime to m), so runs of particles from one cell
// are spread over the tile's range (the lanes of a wavefront in the push then
// mostly deposit into different cells).  Each of the five arrays passes
// through LDS: coalesced loads of the block's slots, stores into LDS at the
// staging position, then coalesced stores of the staged runs to their
// consecutive destination slots.
// One array of the block through LDS: values (in registers, slot order) to
// their staging positions, then the staged runs to their destination slots.
// Staged moves of two arrays at a time (the cell codes travel as float
// bits): each thread puts its particles' values at their staging positions,
// then consecutive threads write consecutive destinations (the tile ranges
// are contiguous).  c0: the first array holds cell codes.  d1 null: one array.
__device__ __forceinline__ void bin_move2(const float (&v0)[kBinRP], float *d0, int32_t *c0, const float (&v1)[kBinRP],
                                          float *d1, const int (&qv)[kBinRP], const unsigned *dst, float *buf0,
                                          float *buf1, unsigned total)
{
#pragma unroll
    for (int r8 = 0; r8 < kBinRP; r8++)
        if (qv[r8] >= 0) {
            buf0[qv[r8]] = v0[r8];
            if (d1) buf1[qv[r8]] = v1[r8];
        }
    __syncthreads();
    for (unsigned q = threadIdx.x; q < total; q += 256) {
        const unsigned d = dst[q];
        if (c0) c0[d] = __float_as_int(buf0[q]);
        else d0[d] = buf0[q];
        if (d1) d1[d] = buf1[q];
    }
    __syncthreads();
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k_bin_scatter(const BinArgs *B, Tab tb)
{
    constexpr int RP = kBinPer / 256;
    __shared__ float buf0[kBinPer], buf1[kBinPer];       // staging of two arrays
    __shared__ unsigned dst[kBinPer];                    // destination slot per staging position
    __shared__ unsigned hist[kBoxN], base[kBoxN], loff[kBoxN], mstr[kBoxN];
    __shared__ unsigned total;
    __shared__ int home;
    const int ku = unit_of(tb, (int)blockIdx.x);
    const BinArgs &a = B[tb.id[ku]];
    const BView v = bview(a);
    const long long n = v.slots;
    const long long lo = (long long)((int)blockIdx.x - tb.boff[ku]) * kBinPer;
    if (lo >= n) return;
    const long long hi = lo + kBinPer < n ? lo + kBinPer : n;
    // every load of the block's slots issued up front
    float fv[4][RP];
    const float *fsrc[4] = {v.ox, v.oy, v.vx, v.vy};
#pragma unroll
    for (int f = 0; f < 4; f++)
#pragma unroll
        for (int r8 = 0; r8 < RP; r8++) {
            const long long p = lo + r8 * 256 + threadIdx.x;
            fv[f][r8] = p < hi ? fsrc[f][p] : 0.0f;
        }
    int cv[RP];
    const TileBox bx = bin_local_count(a, v, lo, hi, hist, &home, cv);
    // per box tile: a destination range, the staging offset, and a stride
    // coprime to the count that spreads runs of particles from one cell over
    // the tile's range (runs would serialise a wavefront's LDS atomics in the
    // push)
    if (threadIdx.x < kBoxN) {
        const int k = threadIdx.x;
        const unsigned m = hist[k];
        if (m) {
            base[k] = atomicAdd(&a.cursor[box_tile(bx, k)], m);
            unsigned st = (unsigned)(0.618034f * (float)m) | 1u;
            while (gcd_u(st, m) != 1u) st++;
            mstr[k] = (m << 16) | (st % m);
        }
    }
    if (threadIdx.x == 0) {
        unsigned off = 0;
        for (int k = 0; k < kBoxN; k++) {
            loff[k] = off;
            off += hist[k];
        }
        total = off;
    }
    __syncthreads();
    if (threadIdx.x < kBoxN) hist[threadIdx.x] = 0u;     // the rank counters of the pass below
    __syncthreads();
    int qv[RP];                                           // staging position of each own slot, or -1
#pragma unroll
    for (int r8 = 0; r8 < RP; r8++) {
        const int c = cv[r8];
        const bool act = live_code(c, a.nx, a.ny);
        const int k = act ? box_index(bx, c, a.lx, a.ly) : -1;
        const bool loc = act && k >= 0;
        const unsigned r = wave_add(hist, loc ? k : 0, loc);
        const unsigned d1 = wave_add(a.cursor, act ? tile_of(c, a.lx, a.ly, a.tiles_y) : 0, act && !loc);
        int qp = -1;
        if (loc) {
            const unsigned ms = mstr[k];
            const unsigned q = loff[k] + (r * (ms & 0xFFFFu)) % (ms >> 16);
            qp = (int)q;
            dst[q] = base[k] + (q - loff[k]);
        } else if (act) {
            v.cell2[d1] = c;
            v.ox2[d1] = fv[0][r8];
            v.oy2[d1] = fv[1][r8];
            v.vx2[d1] = fv[2][r8];
            v.vy2[d1] = fv[3][r8];
        }
        qv[r8] = qp;
    }
    __syncthreads();
    const unsigned nq = total;
    float cf[RP];
#pragma unroll
    for (int r8 = 0; r8 < RP; r8++) cf[r8] = __int_as_float(cv[r8]);
    bin_move2(cf, nullptr, v.cell2, fv[0], v.ox2, qv, dst, buf0, buf1, nq);
    bin_move2(fv[1], v.oy2, nullptr, fv[2], v.vx2, qv, dst, buf0, buf1, nq);
    bin_move2(fv[3], v.vy2, nullptr, fv[3], nullptr, qv, dst, buf0, buf1, nq);
}

// The destination set becomes the set in use.
__global__ void k_bin_flip(const BinArgs *B, Tab t)
{
    const BinArgs &a = B[t.id[blockIdx.x]];
    a.info[7] = 1 - a.info[7];
}

// Tabs: tcount/tscatter cover ceil(slots / kBinPer) blocks per unit, tscan
// one block per unit, ttable ceil(ntiles / 256) blocks per unit.
void launch_bin(const BinArgs *B, const Tab &tcount, const Tab &tscan, const Tab &ttable,
                hipStream_t s)
{
    if (!tscan.n) return;
    if (tab_blocks(tcount)) hipLaunchKernelGGL(k_bin_count, dim3(tab_blocks(tcount)), dim3(256), 0, s, B, tcount);
    hipLaunchKernelGGL(k_bin_scan, dim3(tscan.n), dim3(1024), 0, s, B, tscan);
    hipLaunchKernelGGL(k_bin_table, dim3(tab_blocks(ttable)), dim3(256), 0, s, B, ttable);
    if (tab_blocks(tcount)) hipLaunchKernelGGL(k_bin_scatter, dim3(tab_blocks(tcount)), dim3(256), 0, s, B, tcount);
    hipLaunchKernelGGL(k_bin_flip, dim3(tscan.n), dim3(1), 0, s, B, tscan);
}

int bin_per_block() { return kBinPer; }

// Sum of a node charge array (exact integer sum).
__global__ void k_rho_sum(const unsigned long long *rho, long long n, unsigned long long *out)
{
    __shared__ unsigned long long sh[4];
    long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long st = (long long)gridDim.x * blockDim.x;
    unsigned long long s = 0;
    for (; k < n; k += st) s += rho[k];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(out, sh[0] + sh[1] + sh[2] + sh[3]);
}

void launch_rho_sum(const unsigned long long *rho, long long n, unsigned long long *out,
                    hipStream_t s)
{
    long long nb = (n + 255) / 256;
    if (nb > 1024) nb = 1024;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_rho_sum, dim3((unsigned)nb), dim3(256), 0, s, rho, n, out);
}

// ---------------------------------------------------------------------------
// secondary electron emission at the trench surfaces (Sec. IV; constant
// yield per impact, see pic_config.see_yield)
// ---------------------------------------------------------------------------

// The removals logged since the last call (grid-stride over the ring):
// every trench-surface removal (classes 4, 6, 7) of a species with a yield
// draws from Philox4x32-10, counter (step, packed cell, bits of the kicked
// velocity), key (k0, k1), and with (r0 >> 8) < thresh frees an electron:
// on the struck face of the cell (normal offset the largest float below 1
// on the cell's high side, 0 on its low side; along it (r1 >> 8) 2^-24),
// normal speed vth sqrt(-2 ln u) away from the wall and tangential velocity
// vth sqrt(-2 ln u') cos(2 pi u'') from the draw with key (k0, k1 + 1)
// (u = ((q0 >> 8) + 1) 2^-24, u' = ((q1 >> 8) + 1) 2^-24, u'' = (q2 >> 8)
// 2^-24, in double, rounded to float).  Each takes a slot after species 0's
// slots (a counter; beyond the capacity it is dropped and counted) and adds
// its charge to rho.  Records overwritten before this call are counted as
// dropped.
__global__ __launch_bounds__(256) void k_emit(const SeeArgs *A, Tab t)
{
    const int ku = unit_of(t, (int)blockIdx.x);
    const SeeArgs &a = A[t.id[ku]];
    const int lb = (int)blockIdx.x - t.boff[ku];
    const unsigned long long total = *a.log_count, done = a.misc[0];
    const unsigned long long cap = (unsigned long long)a.log_capacity;
    const unsigned long long first = total - done > cap ? total - cap : done;
    if (lb == 0 && threadIdx.x == 0 && first > done) atomicAdd(&a.misc[3], first - done);
    const int set = (int)a.info[7];
    const long long slots0 = a.info[2 + set];
    GLOBAL int32_t *cell = to_global(a.cell[set]);
    GLOBAL float *ox = to_global(a.ox[set]), *oy = to_global(a.oy[set]);
    GLOBAL float *vx = to_global(a.vx[set]), *vy = to_global(a.vy[set]);
    const float below1 = 0x1.fffffep-1f;
    for (unsigned long long k = first + (unsigned long long)lb * 256 + threadIdx.x; k < total;
         k += (unsigned long long)kEmitBlocks * 256) {
        const int32_t *r = a.rec + 6 * (long long)(k % cap);
        const int sc = r[0], cls = sc & 0xFF, sp = sc >> 8;
        if ((cls != 4 && cls != 6 && cls != 7) || sp < 0 || sp > 1 || a.thresh[sp] == 0u) continue;
        const unsigned c0 = (unsigned)r[4], c1 = (unsigned)r[1], c2 = (unsigned)r[2], c3 = (unsigned)r[3];
        const Philox4 d = philox4x32_10(c0, c1, c2, c3, a.key[0], a.key[1]);
        if ((d.x >> 8) >= a.thresh[sp]) continue;
        const Philox4 q = philox4x32_10(c0, c1, c2, c3, a.key[0], a.key[1] + 1u);
        const float along = (float)(d.y >> 8) * 0x1p-24f;
        const double u1 = (double)((q.x >> 8) + 1u) * 0x1p-24, u2 = (double)((q.y >> 8) + 1u) * 0x1p-24;
        const double u3 = (double)(q.z >> 8) * 0x1p-24;
        const double vn = a.vth * sqrt(-2.0 * log(u1));
        const double vt = a.vth * sqrt(-2.0 * log(u2)) * cos(6.283185307179586 * u3);
        float nox, noy, nvx, nvy;
        if (cls == 4) {             // +x face (the bottom): back along -x
            nox = below1; noy = along; nvx = (float)(-vn); nvy = (float)vt;
        } else if (cls == 6) {      // +y face: back along -y
            nox = along; noy = below1; nvx = (float)vt; nvy = (float)(-vn);
        } else {                    // -y face: back along +y
            nox = along; noy = 0.0f; nvx = (float)vt; nvy = (float)vn;
        }
        const long long slot = slots0 + (long long)atomicAdd(&a.misc[1], 1ull);
        if (slot >= a.capacity) {
            atomicAdd(&a.misc[3], 1ull);
            continue;
        }
        cell[slot] = r[1];
        ox[slot] = nox;
        oy[slot] = noy;
        vx[slot] = nvx;
        vy[slot] = nvy;
        const int ci = (int)((unsigned)r[1] >> 16), cj = r[1] & 0xFFFF;
        deposit_global(to_global(a.rho), a.g, ci, cj, (unsigned)floorf(nox * 65536.0f),
                       (unsigned)floorf(noy * 65536.0f));
    }
}

// After k_emit: the slots of species 0 grow by the electrons that found
// room, the push table gets blocks of `chunk` slots over everything past the
// binned slots (on tile 0's window; the push reads other cells' fields and
// deposits their charge through its global paths), and the ring position
// and counters move on.
__global__ void k_emit_finish(const SeeArgs *A, Tab t)
{
    const SeeArgs &a = A[t.id[unit_of(t, (int)blockIdx.x)]];
    const int set = (int)a.info[7];
    const long long slots0 = a.info[2 + set];
    const long long want = (long long)a.misc[1];
    const long long room = a.capacity > slots0 ? a.capacity - slots0 : 0;
    const long long got = want < room ? want : room;
    const long long slots = slots0 + got;
    const long long t0 = a.info[4], nb0 = a.info[5];
    const long long nb = slots > t0 ? (slots - t0 + a.chunk - 1) / a.chunk : 0;
    for (long long k = threadIdx.x; k < nb; k += blockDim.x) {
        const long long s0 = t0 + k * a.chunk;
        const long long s1 = s0 + a.chunk < slots ? s0 + a.chunk : slots;
        a.table[nb0 + k] = make_int4(0, (int)s0, (int)s1, 0);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a.info[2 + set] = slots;
        a.info[1] = nb0 + nb;
        a.misc[0] = *a.log_count;
        a.misc[1] = 0ull;
        a.misc[2] += (unsigned long long)got;
    }
}

void launch_emit(const SeeArgs *A, const Tab &t, const Tab &t1, hipStream_t s)
{
    if (!t.n) return;
    hipLaunchKernelGGL(k_emit, dim3(tab_blocks(t)), dim3(256), 0, s, A, t);
    hipLaunchKernelGGL(k_emit_finish, dim3(tab_blocks(t1)), dim3(64), 0, s, A, t1);
}

} // namespace pic
