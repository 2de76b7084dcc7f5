// Plain CG of one instance as ONE launch per refinement pass (gfx950).
//
// Launched kernel by kernel an iteration of plain CG is four launches (p and
// A p, the total of p.Ap, the update, the totals of ||r||^2 and r.z), each
// bound by its launch: at 1025 x 512 nodes 21 us per iteration, of which the
// vectors' traffic (all of it in the caches) is a fraction.  Here every vector
// stays in registers for the whole pass: a wavefront owns one virtual block
// (4 rows x 64 columns of nodes, the block of the grid kernels), a node's p,
// r and e live in its lane, and an iteration exchanges only
//   - the rims of r (each virtual block's outer rows and columns; the
//     receiver keeps its own copy of the neighbours' p there and applies the
//     same update, so one exchange per iteration suffices), and
//   - two totals (p.Ap, then ||r||^2 with r.z).
// Arithmetic and the order of every addition are those of the launched
// kernels (k_init_red0, k_pupdate_Ap, k_update_red0, k_finalize), so the
// potential is the same bit for bit.
//
// Totals: k_finalize gives thread t of 256 the partials t, t + 256, ... in
// order and adds the threads in a fixed tree.  Work-group t therefore owns the
// virtual blocks t, t + 256, ... (one wavefront each), sums its own chain, and
// publishes one number; every work-group then reads all (at most 256) chain
// sums and adds the same tree.  One trip through memory per total.
//
// Published words are 64 bits, 32 of data and the 32-bit epoch of the
// exchange, written and read with agent-scope atomics (coherent between the
// XCDs' L2 caches): a reader polls the word itself, so data and signal arrive
// together and no fence is needed.  Chain sums use two buffers in turn (a
// work-group that publishes epoch e + 2 has seen every epoch e + 1, hence
// everyone has read e); a rim is rewritten only after the p.Ap total that
// follows its readers.
//
// Every wait is bounded in time: a work-group that gives up sets the abort
// word and leaves, the others follow, and the host runs the pass with the
// launched kernels (nothing the pass reads has been overwritten by then).
//
// Grids of at most kCgSingleVb virtual blocks run in one work-group with both
// exchanges in LDS.
#include "pic_internal.h"

namespace pic {

namespace {

typedef unsigned long long u64;

constexpr int kVbRows = kGridBY;       // rows of a virtual block

__device__ __forceinline__ double dpp_add(double v, const int ctrl_kind)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    int l2, h2;
    switch (ctrl_kind) {
    case 0:                            // row_ror:8
        l2 = __builtin_amdgcn_update_dpp(0, lo, 0x128, 0xF, 0xF, false);
        h2 = __builtin_amdgcn_update_dpp(0, hi, 0x128, 0xF, 0xF, false);
        break;
    case 1:                            // row_ror:4
        l2 = __builtin_amdgcn_update_dpp(0, lo, 0x124, 0xF, 0xF, false);
        h2 = __builtin_amdgcn_update_dpp(0, hi, 0x124, 0xF, 0xF, false);
        break;
    case 2:                            // quad_perm [2,3,0,1]
        l2 = __builtin_amdgcn_update_dpp(0, lo, 0x4E, 0xF, 0xF, false);
        h2 = __builtin_amdgcn_update_dpp(0, hi, 0x4E, 0xF, 0xF, false);
        break;
    default:                           // quad_perm [1,0,3,2]
        l2 = __builtin_amdgcn_update_dpp(0, lo, 0xB1, 0xF, 0xF, false);
        h2 = __builtin_amdgcn_update_dpp(0, hi, 0xB1, 0xF, 0xF, false);
        break;
    }
    return v + __hiloint2double(h2, l2);
}

// a: lanes 0..31 of a and of b;  b: lanes 32..63 of a and of b.
__device__ __forceinline__ void swap32(double &a, double &b)
{
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    a = __hiloint2double((int)hi[0], (int)lo[0]);
    b = __hiloint2double((int)hi[1], (int)lo[1]);
}

// The same with 16-lane rows: a gets rows 0, 2 of a and of b, b rows 1, 3.
__device__ __forceinline__ void swap16(double &a, double &b)
{
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    a = __hiloint2double((int)hi[0], (int)lo[0]);
    b = __hiloint2double((int)hi[1], (int)lo[1]);
}

__device__ __forceinline__ double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The wave_sum tree (partners 32, 16, 8, 4, 2, 1 lanes apart) of four values
// at once, without LDS: the two widest steps fold two values into one register.
// Uniform results.
__device__ __forceinline__ void wave_sum4(double (&v)[4])
{
    swap32(v[0], v[1]);
    double x = v[0] + v[1];            // lanes 0-31: value 0, 32-63: value 1
    swap32(v[2], v[3]);
    double y = v[2] + v[3];
    swap16(x, y);
    x = x + y;                         // rows 0, 2: values 0, 1; rows 1, 3: values 2, 3
    x = dpp_add(x, 0);
    x = dpp_add(x, 1);
    x = dpp_add(x, 2);
    x = dpp_add(x, 3);
    v[0] = lane_value(x, 0);
    v[1] = lane_value(x, 32);
    v[2] = lane_value(x, 16);
    v[3] = lane_value(x, 48);
}

__device__ __forceinline__ u64 ld_agent(const u64 *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(u64 *p, u64 v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 tagged(unsigned data, unsigned epoch) { return ((u64)epoch << 32) | data; }

// True while a poll may go on; false once its time is up or another
// work-group gave up.
struct Patience {
    long long start;
    int spins;
    __device__ __forceinline__ Patience() : start(0), spins(0) {}
    __device__ __forceinline__ bool more(const int *abort_word, long long wait)
    {
        if (wait < 0) return false;
        __builtin_amdgcn_s_sleep(1);
        if ((++spins & 1023) != 0) return true;
        const long long now = wall_clock64();
        if (start == 0) start = now;
        if (now - start > wait) return false;
        return __hip_atomic_load(abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
    }
};

// One wavefront's virtual block.
struct Vb {
    int i0, j, nr;                     // first row, this lane's column, rows inside the grid
    unsigned free_;                    // bit r: node (i0 + r, j) is an unknown
    float p[kVbRows], r[kVbRows], e[kVbRows];
    // the neighbours' nodes: the rows above and below (this lane's column),
    // and on lanes 0-3 / 4-7 the column left / right of the block, rows 0-3
    int nu, nd, ns;                    // node indices (-1: not needed)
    unsigned hfree;                    // bits 0, 1, 2: those nodes are unknowns
    float pu, pd, ps;
    int jl, jr;                        // lanes of the left and right neighbours (-1: in ps)
};

} // namespace

// V virtual blocks per wavefront; SINGLE: the whole grid in one work-group.
template <int V, bool SINGLE>
__global__ __launch_bounds__(1024) void k_cg_pass(const Inst *insts, int bx, int nvb, unsigned epoch, int cap,
                                                  u64 *rim, u64 *slots, int *abort_word, long long wait)
{
    const Inst &I = insts[0];
    const LevelDev L0 = I.lev[0];
    const int NX = L0.NX, NY = L0.NY;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
    const bool lead = blockIdx.x == 0 && tid == 0;
    if (I.F[F_CONV]) {
        if (lead) {
            I.F[F_SKIP] = 1;
            I.F[F_DONE] = 1;
        }
        return;
    }
    extern __shared__ float rlds[];    // SINGLE: r of every node
    __shared__ double red[2][2][SINGLE ? 16 * V : 16];
    __shared__ double tot[2];
    __shared__ int give_up;
    if (tid == 0) give_up = 0;

    Vb B[V];
    bool act[V];
#pragma unroll
    for (int v = 0; v < V; v++) {
        const int vb = SINGLE ? wave * V + v : (int)blockIdx.x + 256 * wave;
        act[v] = vb < nvb;
        Vb &b = B[v];
        const int q = act[v] ? vb : 0;
        const int byb = q / bx, bxb = q - byb * bx;
        b.i0 = byb * kVbRows;
        b.j = bxb * kGridBX + lane;
        b.nr = min(kVbRows, NX - b.i0);
        const int w = min(kGridBX, NY - bxb * kGridBX);     // columns inside the grid
        const bool in = act[v] && lane < w;
        b.free_ = 0;
#pragma unroll
        for (int r = 0; r < kVbRows; r++) {
            b.r[r] = 0.f;
            b.p[r] = 0.f;
            b.e[r] = 0.f;
            if (in && r < b.nr) {
                const int n = (b.i0 + r) * NY + b.j;
                if (!L0.fix[n]) b.free_ |= 1u << r;
                b.r[r] = L0.g[n];
            }
        }
        const int iu = b.i0 == 0 ? NX - 1 : b.i0 - 1;
        const int id = b.i0 + b.nr >= NX ? 0 : b.i0 + b.nr;
        b.nu = in ? iu * NY + b.j : -1;
        b.nd = in ? id * NY + b.j : -1;
        const int c0 = bxb * kGridBX, cl = c0 == 0 ? NY - 1 : c0 - 1, cr = c0 + w >= NY ? 0 : c0 + w;
        const bool lin = (cl >> 6) == bxb, rin = (cr >> 6) == bxb;   // the wrap stays in this block
        b.ns = -1;
        if (act[v] && lane < 8) {
            const int r = lane & 3;
            if (r < b.nr && !(lane < 4 ? lin : rin)) b.ns = (b.i0 + r) * NY + (lane < 4 ? cl : cr);
        }
        b.jl = lane > 0 ? lane - 1 : (lin ? cl - c0 : -1);
        b.jr = lane < w - 1 ? lane + 1 : (lane == w - 1 ? (rin ? cr - c0 : -1) : 0);
        b.hfree = 0;
        if (b.nu >= 0 && !L0.fix[b.nu]) b.hfree |= 1;
        if (b.nd >= 0 && !L0.fix[b.nd]) b.hfree |= 2;
        if (b.ns >= 0 && !L0.fix[b.ns]) b.hfree |= 4;
        b.pu = b.pd = b.ps = 0.f;
    }
    const double *S = I.S;
    double rz = S[S_RZ], rzold = S[S_RZOLD], pq = S[S_PQ];
    const double bb = S[S_BB] > 0.0 ? S[S_BB] : 1.0;
    const double rr64 = S[S_RR64];
    const int passes = I.F[F_PASSES] + 1, tot0 = I.F[F_ITER_TOT], iter1 = I.F[F_ITER1];
    int phase = 0;

    // rim values of the current r to the neighbours
    auto publish_rim = [&]() {
#pragma unroll
        for (int v = 0; v < V; v++) {
            const Vb &b = B[v];
            if (!act[v] || b.nu < 0) continue;
#pragma unroll
            for (int r = 0; r < kVbRows; r++) {
                if (r >= b.nr) continue;
                const int n = (b.i0 + r) * NY + b.j;
                if (SINGLE) {
                    rlds[n] = b.r[r];
                } else if (r == 0 || r == b.nr - 1 || lane == 0 || b.j == NY - 1 || lane == 63) {
                    st_agent(rim + n, tagged(__float_as_uint(b.r[r]), epoch));
                }
            }
        }
    };
    // the neighbours' r of this epoch into hr (0 where not needed)
    float hr[V][3];
    auto fetch_rim = [&]() -> bool {
        bool ok = true;
#pragma unroll
        for (int v = 0; v < V; v++) {
            const Vb &b = B[v];
            if (SINGLE) {
                hr[v][0] = b.nu >= 0 ? rlds[b.nu] : 0.f;
                hr[v][1] = b.nd >= 0 ? rlds[b.nd] : 0.f;
                hr[v][2] = b.ns >= 0 ? rlds[b.ns] : 0.f;
            } else {
                Patience pat;
                for (;;) {
                    const u64 none = tagged(0u, epoch);
                    const u64 a = b.nu >= 0 ? ld_agent(rim + b.nu) : none;
                    const u64 c = b.nd >= 0 ? ld_agent(rim + b.nd) : none;
                    const u64 d = b.ns >= 0 ? ld_agent(rim + b.ns) : none;
                    const bool here = (unsigned)(a >> 32) == epoch && (unsigned)(c >> 32) == epoch &&
                                      (unsigned)(d >> 32) == epoch;
                    hr[v][0] = __uint_as_float((unsigned)a);
                    hr[v][1] = __uint_as_float((unsigned)c);
                    hr[v][2] = __uint_as_float((unsigned)d);
                    if (__all(here)) break;
                    if (!pat.more(abort_word, wait)) {
                        ok = false;
                        break;
                    }
                }
            }
        }
        return ok;
    };
    // totals of NQ quantities over the grid (val: per row of each virtual block); rims: the rims of this
    // epoch are fetched while the totals travel.  False: given up.
    auto total = [&](double (&val)[2][V][kVbRows], int nq, bool rims, double (&out)[2]) -> bool {
#pragma unroll
        for (int q = 0; q < 2; q++) {
            if (q >= nq) continue;
#pragma unroll
            for (int v = 0; v < V; v++) {
                wave_sum4(val[q][v]);
                double s = 0.0;
#pragma unroll
                for (int r = 0; r < kVbRows; r++) s += val[q][v][r];
                if (lane == 0) red[phase][q][wave * V + v] = act[v] ? s : 0.0;
            }
        }
        __syncthreads();
        if (SINGLE) {
            if (rims) (void)fetch_rim();
#pragma unroll
            for (int q = 0; q < 2; q++) {
                if (q >= nq) continue;
                double x[4] = {lane < nw * V ? red[phase][q][lane] : 0.0, 0.0, 0.0, 0.0};
                wave_sum4(x);
                out[q] = x[0] + x[1] + x[2] + x[3];
            }
            phase ^= 1;
            // r in LDS is rewritten only after the next total's barrier
            return true;
        }
        bool ok = true;
        if (wave == 0) {
            u64 *buf = slots + (size_t)(epoch & 1) * 1024;
#pragma unroll
            for (int q = 0; q < 2; q++) {
                if (q >= nq) continue;
                double s = 0.0;
                for (int k = 0; k < nw; k++) s += red[phase][q][k];
                if (lane < 2)
                    st_agent(buf + 512 * q + 2 * blockIdx.x + lane,
                             tagged((unsigned)(lane ? __double2hiint(s) : __double2loint(s)), epoch));
            }
            const int nchain = gridDim.x;
            Patience pat;
            double x[2][4];
            for (;;) {
                bool here = true;
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    if (q >= nq) continue;
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        const int c = lane + 64 * k;
                        x[q][k] = 0.0;
                        if (c < nchain) {
                            const u64 lo = ld_agent(buf + 512 * q + 2 * c), hi = ld_agent(buf + 512 * q + 2 * c + 1);
                            here = here && (unsigned)(lo >> 32) == epoch && (unsigned)(hi >> 32) == epoch;
                            x[q][k] = __hiloint2double((int)(unsigned)hi, (int)(unsigned)lo);
                        }
                    }
                }
                if (__all(here)) break;
                if (!pat.more(abort_word, wait)) {
                    ok = false;
                    break;
                }
            }
#pragma unroll
            for (int q = 0; q < 2; q++) {
                if (q >= nq) continue;
                wave_sum4(x[q]);
                if (lane == 0) tot[q] = x[q][0] + x[q][1] + x[q][2] + x[q][3];
            }
        }
        if (rims && ok) ok = fetch_rim();
        if (!ok) give_up = 1;
        __syncthreads();
        for (int q = 0; q < nq; q++) out[q] = tot[q];
        phase ^= 1;
        epoch++;
        if (give_up) {
            if (tid == 0) __hip_atomic_store(abort_word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        return true;
    };

    // inner start: e = 0, z = r / 4, ||r||^2 and r.z
    double val[2][V][kVbRows], t2[2];
    auto rr_rz = [&]() {
#pragma unroll
        for (int v = 0; v < V; v++)
#pragma unroll
            for (int r = 0; r < kVbRows; r++) {
                const bool f = (B[v].free_ >> r) & 1;
                const float x = B[v].r[r], z = x * 0.25f;
                val[0][v][r] = f ? (double)x * (double)x : 0.0;
                val[1][v][r] = f ? (double)x * (double)z : 0.0;
            }
    };
    __syncthreads();
    publish_rim();
    rr_rz();
    if (!total(val, 2, true, t2)) return;
    const double tol2 = I.rtol * I.rtol;
    double eta2 = 0.09 * tol2 * bb / (rr64 > 0.0 ? rr64 : 1.0);
    const double lo = I.eta_min * I.eta_min;
    eta2 = eta2 < lo ? lo : (eta2 > 0.25 ? 0.25 : eta2);
    const double rr0 = t2[0];
    double rr = rr0;
    bool done = rr0 == 0.0;
    rzold = rz;
    rz = t2[1];
    int iter = 0;
    while (!done && iter < cap) {
        const bool first = iter == 0;
        const float beta = first ? 0.f : (float)(rz / rzold);
#pragma unroll
        for (int v = 0; v < V; v++) {
            Vb &b = B[v];
#pragma unroll
            for (int r = 0; r < kVbRows; r++) {
                const float z = b.r[r] * 0.25f;
                const float pn = first ? z : z + beta * b.p[r];
                b.p[r] = ((b.free_ >> r) & 1) ? pn : 0.f;
            }
            const float zu = hr[v][0] * 0.25f, zd = hr[v][1] * 0.25f, zs = hr[v][2] * 0.25f;
            const float u = first ? zu : zu + beta * b.pu, d = first ? zd : zd + beta * b.pd;
            const float s = first ? zs : zs + beta * b.ps;
            b.pu = (b.hfree & 1) ? u : 0.f;
            b.pd = (b.hfree & 2) ? d : 0.f;
            b.ps = (b.hfree & 4) ? s : 0.f;
        }
        float q[V][kVbRows];
#pragma unroll
        for (int v = 0; v < V; v++) {
            const Vb &b = B[v];
#pragma unroll
            for (int r = 0; r < kVbRows; r++) {
                // neighbours in the order x-1, x+1, y-1, y+1; a fixed one holds 0
                const float up = r == 0 ? b.pu : b.p[r > 0 ? r - 1 : 0];
                const float dn = r == b.nr - 1 ? b.pd : b.p[r < kVbRows - 1 ? r + 1 : 0];
                float lf = __shfl(b.p[r], b.jl < 0 ? 0 : b.jl, 64), rt = __shfl(b.p[r], b.jr < 0 ? 0 : b.jr, 64);
                const float el = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b.ps), r));
                const float er = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b.ps), 4 + r));
                if (b.jl < 0) lf = el;
                if (b.jr < 0) rt = er;
                float s = 4.0f * b.p[r];
                s -= up;
                s -= dn;
                s -= lf;
                s -= rt;
                const bool f = (b.free_ >> r) & 1;
                q[v][r] = f ? s : 0.f;
                val[0][v][r] = f ? (double)b.p[r] * (double)s : 0.0;
            }
        }
        if (!total(val, 1, false, t2)) return;
        pq = t2[0];
        const float alpha = (float)(rz / pq);
#pragma unroll
        for (int v = 0; v < V; v++) {
            Vb &b = B[v];
#pragma unroll
            for (int r = 0; r < kVbRows; r++) {
                if (!((b.free_ >> r) & 1)) continue;
                b.e[r] = b.e[r] + alpha * b.p[r];
                b.r[r] = b.r[r] - alpha * q[v][r];
            }
        }
        publish_rim();
        rr_rz();
        if (!total(val, 2, true, t2)) return;
        rr = t2[0];
        rzold = rz;
        rz = t2[1];
        iter++;
        if (rr <= eta2 * rr0) done = true;
    }
#pragma unroll
    for (int v = 0; v < V; v++) {
        const Vb &b = B[v];
        if (!act[v] || b.nu < 0) continue;
#pragma unroll
        for (int r = 0; r < kVbRows; r++)
            if (r < b.nr) I.e[(b.i0 + r) * NY + b.j] = b.e[r];
    }
    if (lead) {
        double *So = I.S;
        int *F = I.F;
        So[S_ETA2] = eta2;
        So[S_RR0] = rr0;
        So[S_RR] = rr;
        So[S_RZ] = rz;
        So[S_RZOLD] = rzold;
        So[S_PQ] = pq;
        F[F_SKIP] = 0;
        F[F_DONE] = done ? 1 : 0;
        F[F_ITER] = iter;
        F[F_ITER_TOT] = tot0 + iter;
        F[F_PASSES] = passes;
        F[F_ITER1] = passes == 1 && iter > 0 ? iter : iter1;
    }
}

namespace {

int vb_count(int NX, int NY) { return ((NY + kGridBX - 1) / kGridBX) * ((NX + kGridBY - 1) / kGridBY); }

template <int V, bool SINGLE> int fits(int blocks, int threads, size_t lds)
{
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return false;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, (const void *)k_cg_pass<V, SINGLE>, threads, lds) !=
        hipSuccess)
        return false;
    return (long long)per * cus >= blocks;
}

} // namespace

bool cg_needs_rim(int NX, int NY) { return vb_count(NX, NY) > kCgSingleVb; }

CgPlan cg_plan(int NX, int NY)
{
    CgPlan p{};
    const int nvb = vb_count(NX, NY);
    p.nvb = nvb;
    p.bx = (NY + kGridBX - 1) / kGridBX;
    if (nvb <= kCgSingleVb) {
        p.V = nvb <= 16 ? 1 : 2;
        p.single = 1;
        p.blocks = 1;
        p.threads = 64 * ((nvb + p.V - 1) / p.V);
        p.lds = (size_t)NX * NY * sizeof(float);
        p.ok = p.V == 1 ? fits<1, true>(1, p.threads, p.lds) : fits<2, true>(1, p.threads, p.lds);
    } else {
        // one chain of the totals per work-group, one wavefront per virtual block
        p.V = 1;
        p.blocks = nvb < 256 ? nvb : 256;
        const int waves = (nvb + 255) / 256;
        p.threads = 64 * waves;
        p.ok = waves <= 16 && fits<1, false>(p.blocks, p.threads, 0);
    }
    return p;
}

hipError_t launch_cg_pass(const Inst *I, const CgPlan &p, unsigned epoch, int cap, unsigned long long *rim,
                          unsigned long long *slots, int *abort_word, long long wait, hipStream_t s)
{
    const Inst *insts = I;
    int bx = p.bx, nvb = p.nvb;
    void *args[] = {&insts, &bx, &nvb, &epoch, &cap, &rim, &slots, &abort_word, &wait};
    if (p.single) {
        if (p.V == 1)
            hipLaunchKernelGGL((k_cg_pass<1, true>), dim3(1), dim3(p.threads), p.lds, s, I, bx, nvb, epoch, cap, rim,
                               slots, abort_word, wait);
        else
            hipLaunchKernelGGL((k_cg_pass<2, true>), dim3(1), dim3(p.threads), p.lds, s, I, bx, nvb, epoch, cap, rim,
                               slots, abort_word, wait);
        return hipGetLastError();
    }
    // cooperative: the runtime keeps two such launches of one process from
    // sharing the chip half and half
    return hipLaunchCooperativeKernel((const void *)k_cg_pass<1, false>, dim3(p.blocks), dim3(p.threads), args, 0, s);
}

} // namespace pic
