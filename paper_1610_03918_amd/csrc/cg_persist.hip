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
// sums and adds the same tree.  One trip through memory per total.  r.z is
// ||r||^2 / 4 exactly (z = r / 4, powers of two scale every rounding) unless a
// z underflows, so a wavefront adds it up on its own only where one may.
//
// Published words are 64 bits, written and read with agent-scope atomics
// (coherent between the XCDs' L2 caches).  A reader polls the word itself, so
// data and signal arrive together and no fence is needed: a rim word carries
// the exchange's epoch in its upper half, a chain sum replaces an all-ones
// word (no sum has that bit pattern).  Chain sums use three buffers in turn:
// whoever has all sums of epoch e knows that everyone has read those of e - 1,
// and clears its word there, for epoch e + 2, before it publishes e + 1.  A
// rim is rewritten only after the p.Ap total that follows its readers.
//
// Every wait is bounded in time: a work-group that gives up sets the abort
// word and leaves, the others follow, and the host runs the pass with the
// launched kernels (nothing the pass reads has been overwritten by then).  So
// it does where a step length is not finite: the fixed nodes, which here take
// part in the updates with zeros, would then differ.
//
// Grids of at most kCgSingleVb virtual blocks run in one work-group with both
// exchanges in LDS: 3.0 us per iteration at 41 x 48 nodes (11 virtual blocks)
// against 4.3 through device memory; at 17 the wavefronts of one CU share its
// issue slots and the two are equal.
//
// Measured, us per iteration (launched -> here): 97 x 56 nodes 16.5 -> 4.3,
// 1025 x 512 21.4 -> 6.8.  What is left is the two trips through memory (1.1
// to 1.7 us each) and, at 1025 x 512, nine wavefronts per CU.  On the way:
// every work-group polling one copy of the sums, whose few memory channels
// then serve 256 readers, and the rims stored before the sum (a rim store
// stalls its wavefront for about 1000 cycles) 8.9 us; two copies 7.0, four
// 6.9, eight 6.8, sixteen 7.8 (before the side columns were gathered into one
// store).
#include "pic_internal.h"
#include "wave_ops.h"

namespace pic {

namespace {

constexpr int kVbRows = kGridBY;       // rows of a virtual block

constexpr u64 kNoSum = ~0ull;          // a chain sum not yet published
// Chain sums: [copy][buffer][quantity][256]; work-group b reads copy b % kCopies, so that no few memory channels
// serve every poll.  After them the buffer of the next total (cleared, all ones, it is 0 mod 3).
constexpr int kCopies = kCgCopies, kCopyWords = kCgCopyWords;
constexpr int kTurnWord = kCopies * kCopyWords;

// One wavefront's virtual block.
struct Vb {
    int n0;                            // this lane's node in the first row
    int nr, w;                         // rows and columns inside the grid
    bool in;                           // this lane holds a column
    bool fr[kVbRows];                  // node of row r is an unknown
    float p[kVbRows], r[kVbRows], e[kVbRows];
    // the neighbours' nodes: the rows above and below (this lane's column) and
    // the columns beside the block: lane 0 the left one, lane w - 1 the right one
    // (pe; in a block of one column pe is the left one and pr the right one)
    int nu, nd, ns;                    // nodes to fetch (-1: none); ns: lanes 0-3 left, 4-7 right, rows 0-3
    float pu, pd, pe[kVbRows], pr[kVbRows];
    bool wrap;                         // the columns wrap inside the block
};

// p, shifted by one lane; lane 0 (63) keeps old's.
__device__ __forceinline__ float from_left(float old, float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), 0x138, 0xF, 0xF, false));
}
__device__ __forceinline__ float from_right(float old, float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), 0x130, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_f(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

} // namespace

// SINGLE: the whole grid in one work-group.
// slots[kTurnWord]: the chain sum buffer of the next total.
template <bool SINGLE>
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
    __shared__ double red[2][2][16];
    __shared__ double tot[2];
    __shared__ int give_up;
    if (tid == 0) give_up = 0;

    Vb b;
    const int vb = SINGLE ? wave : (int)blockIdx.x + 256 * wave;
    const bool act = vb < nvb;
    const int byb = act ? vb / bx : 0, bxb = act ? vb - byb * bx : 0;
    const int i0 = byb * kVbRows, c0 = bxb * kGridBX;
    b.n0 = i0 * NY + c0 + lane;
    b.nr = min(kVbRows, NX - i0);
    b.w = min(kGridBX, NY - c0);
    b.in = act && lane < b.w;
#pragma unroll
    for (int r = 0; r < kVbRows; r++) {
        b.r[r] = b.p[r] = b.e[r] = b.pe[r] = b.pr[r] = 0.f;
        b.fr[r] = false;
        if (b.in && r < b.nr) {
            const int n = b.n0 + r * NY;
            b.fr[r] = !L0.fix[n];
            b.r[r] = L0.g[n];          // 0 at fixed nodes, and stays so
        }
    }
    {
        const int iu = i0 == 0 ? NX - 1 : i0 - 1, id = i0 + b.nr >= NX ? 0 : i0 + b.nr;
        b.nu = b.in ? iu * NY + c0 + lane : -1;
        b.nd = b.in ? id * NY + c0 + lane : -1;
        b.wrap = b.w == NY;
        b.ns = -1;
        const int row = lane & 3;
        if (act && !b.wrap && lane < 8 && row < b.nr) {
            const int cb = lane < 4 ? (bxb == 0 ? bx - 1 : bxb - 1) : (bxb == bx - 1 ? 0 : bxb + 1);
            if (SINGLE) b.ns = (i0 + row) * NY + (lane < 4 ? (bxb == 0 ? NY : c0) - 1 : cb * kGridBX);
            else b.ns = (byb * bx + cb) * 8 + (lane < 4 ? 4 : 0) + row;
        }
    }
    b.pu = b.pd = 0.f;
    u64 *const side = rim + (size_t)NX * NY;           // 8 words a virtual block: its left, then its right column
    const int edge = lane < 4 ? 0 : b.w - 1;
    const double *S = I.S;
    double rz = S[S_RZ], rzold = S[S_RZOLD], pq = S[S_PQ];
    const double bb = S[S_BB] > 0.0 ? S[S_BB] : 1.0;
    const double rr64 = S[S_RR64];
    const int passes = I.F[F_PASSES] + 1, tot0 = I.F[F_ITER_TOT], iter1 = I.F[F_ITER1];
    unsigned turn = SINGLE ? 0u : (unsigned)(slots[kTurnWord] % 3);
    int phase = 0;

    // rim values of the current r to the neighbours
    auto publish_rim = [&]() {
        if (SINGLE) {
            if (!b.in) return;
#pragma unroll
            for (int r = 0; r < kVbRows; r++)
                if (r < b.nr) rlds[b.n0 + r * NY] = b.r[r];
            return;
        }
        if (!act) return;
        float x = 0.f;
#pragma unroll
        for (int r = 0; r < kVbRows; r++) {
            const float v = __shfl(b.r[r], edge, 64);
            x = (lane & 3) == r ? v : x;
        }
        if (b.in) {
            float last = b.r[kVbRows - 1];
            if (b.nr < kVbRows) last = b.nr == 1 ? b.r[0] : b.nr == 2 ? b.r[1] : b.r[2];
            st_agent(rim + b.n0, tagged(__float_as_uint(b.r[0]), epoch));
            if (b.nr > 1) st_agent(rim + b.n0 + (b.nr - 1) * NY, tagged(__float_as_uint(last), epoch));
        }
        if (!b.wrap && lane < 8) st_agent(side + 8 * vb + lane, tagged(__float_as_uint(x), epoch));
    };
    // one try at the neighbours' r of this epoch (0 where none is needed)
    float hu = 0.f, hd = 0.f, hs = 0.f;
    auto try_rim = [&]() -> bool {
        if (SINGLE) {
            hu = b.nu >= 0 ? rlds[b.nu] : 0.f;
            hd = b.nd >= 0 ? rlds[b.nd] : 0.f;
            hs = b.ns >= 0 ? rlds[b.ns] : 0.f;
            return true;
        }
        u64 x = tagged(0u, epoch), y = x, z = x;
        if (b.nu >= 0) {
            x = ld_agent(rim + b.nu);
            y = ld_agent(rim + b.nd);
        }
        if (b.ns >= 0) z = ld_agent(side + b.ns);
        hu = __uint_as_float((unsigned)x);
        hd = __uint_as_float((unsigned)y);
        hs = __uint_as_float((unsigned)z);
        return (unsigned)(x >> 32) == epoch && (unsigned)(y >> 32) == epoch && (unsigned)(z >> 32) == epoch;
    };
    // Totals of the grid from this wavefront's partial sums; with NQ == 2 (||r||^2, r.z) the rims of this
    // epoch are fetched while the totals travel.  False: given up.
    auto total = [&](const double (&part)[2], auto nq_, double (&out)[2]) -> bool {
        constexpr int NQ = decltype(nq_)::value;
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < NQ; q++) red[phase][q][wave] = act ? part[q] : 0.0;
        }
        __syncthreads();
        if (SINGLE) {
            if (NQ == 2) (void)try_rim();
#pragma unroll
            for (int q = 0; q < NQ; q++) {
                out[q] = wave_sum1(lane < nw ? red[phase][q][lane] : 0.0) + 0.0;
            }
            phase ^= 1;
            // r in LDS is rewritten only after the next total's barrier
            return true;
        }
        bool ok = true;
        Patience pat;
        if (wave == 0) {
            if (lane < NQ * kCopies) {
                const int q = NQ == 2 ? lane & 1 : 0, c = NQ == 2 ? lane >> 1 : lane;
                double s = 0.0;
                for (int k = 0; k < nw; k++) s += red[phase][q][k];
                const u64 word = (u64)__double_as_longlong(s);
                // the next buffer's word is clear everywhere before this sum is seen
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                st_agent(slots + c * kCopyWords + turn * 512 + 256 * q + blockIdx.x,
                         word == kNoSum ? 0x7FF8000000000000ull : word);
            }
            // the rims follow the sum, which everyone waits for: their stores stall the wavefront
            if (NQ == 2) publish_rim();
            const u64 *buf = slots + (blockIdx.x % kCopies) * kCopyWords + turn * 512;
            const int nchain = gridDim.x;
            double x[2][4];
            bool rims = NQ == 1;
            for (;;) {
                bool here = true;
                u64 y[NQ][4];
#pragma unroll
                for (int q = 0; q < NQ; q++)
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        y[q][k] = 0;
                        if (lane + 64 * k < nchain) y[q][k] = ld_agent(buf + 256 * q + lane + 64 * k);
                    }
                if (!rims) rims = __all(try_rim());
#pragma unroll
                for (int q = 0; q < NQ; q++)
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        here = here && y[q][k] != kNoSum;
                        x[q][k] = __longlong_as_double((long long)y[q][k]);
                    }
                if (__all(here) && rims) break;
                if (!pat.more(abort_word, wait)) {
                    ok = false;
                    break;
                }
            }
#pragma unroll
            for (int q = 0; q < NQ; q++) {
                wave_sum4(x[q]);
                if (lane == 0) tot[q] = x[q][0] + x[q][1] + x[q][2] + x[q][3];
            }
            // everyone has published this total, hence read the one before: its buffer is the next but one
            const unsigned clear = turn == 0 ? 2u : turn - 1;
            if (lane < 2 * kCopies)
                st_agent(slots + (lane >> 1) * kCopyWords + clear * 512 + 256 * (lane & 1) + blockIdx.x, kNoSum);
        } else if (NQ == 2) {
            publish_rim();
            while (!__all(try_rim()))
                if (!pat.more(abort_word, wait)) {
                    ok = false;
                    break;
                }
        }
        if (!ok) give_up = 1;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NQ; q++) out[q] = tot[q];
        phase ^= 1;
        epoch++;
        turn = turn == 2 ? 0u : turn + 1;
        if (give_up) {
            if (tid == 0) __hip_atomic_store(abort_word, (int)kAbortGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        return true;
    };
    // the wavefront's ||r||^2 and r.z
    double part[2], t2[2];
    auto rr_rz = [&]() {
        double x[4];
        bool small = false;
#pragma unroll
        for (int r = 0; r < kVbRows; r++) {
            const float a = b.r[r];
            x[r] = (double)a * (double)a;
            small = small || (fabsf(a) < 0x1p-120f && a != 0.f);
        }
        wave_sum4(x);
        part[0] = 0.0 + x[0] + x[1] + x[2] + x[3];
        part[1] = 0.25 * part[0];
        if (__any(small)) {
#pragma unroll
            for (int r = 0; r < kVbRows; r++) {
                const float a = b.r[r], z = a * 0.25f;
                x[r] = (double)a * (double)z;
            }
            wave_sum4(x);
            part[1] = 0.0 + x[0] + x[1] + x[2] + x[3];
        }
    };

    // inner start: e = 0, z = r / 4, ||r||^2 and r.z
    __syncthreads();
    if (SINGLE) publish_rim();
    rr_rz();
    if (!total(part, Int<2>{}, t2)) return;
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
        // p = z + beta p; the first step's beta is 0 (and p 0)
        const float beta = iter == 0 ? 0.f : (float)(rz / rzold);
#pragma unroll
        for (int r = 0; r < kVbRows; r++) b.p[r] = b.r[r] * 0.25f + beta * b.p[r];
        b.pu = hu * 0.25f + beta * b.pu;
        b.pd = hd * 0.25f + beta * b.pd;
#pragma unroll
        for (int r = 0; r < kVbRows; r++) {
            if (b.wrap) {
                b.pe[r] = lane == 0 ? lane_f(b.p[r], b.w - 1) : lane_f(b.p[r], 0);
                b.pr[r] = b.pe[r];
            } else {
                const float left = lane_f(hs, r), right = lane_f(hs, 4 + r);
                b.pe[r] = (lane == 0 ? left : right) * 0.25f + beta * b.pe[r];
                b.pr[r] = right * 0.25f + beta * b.pr[r];
            }
        }
        float q[kVbRows];
        double x[4];
#pragma unroll
        for (int r = 0; r < kVbRows; r++) {
            // neighbours in the order x-1, x+1, y-1, y+1; a fixed one holds 0
            const float up = r == 0 ? b.pu : b.p[r > 0 ? r - 1 : 0];
            const float dn = r == kVbRows - 1 || r == b.nr - 1 ? b.pd : b.p[r < kVbRows - 1 ? r + 1 : 0];
            const float lf = from_left(b.pe[r], b.p[r]);
            float rt = from_right(b.pe[r], b.p[r]);
            if (b.w < 64) rt = lane == b.w - 1 ? (b.w == 1 ? b.pr[r] : b.pe[r]) : rt;
            float s = 4.0f * b.p[r];
            s -= up;
            s -= dn;
            s -= lf;
            s -= rt;
            q[r] = b.fr[r] ? s : 0.f;
            x[r] = (double)b.p[r] * (double)q[r];
        }
        wave_sum4(x);
        part[0] = 0.0 + x[0] + x[1] + x[2] + x[3];
        if (!total(part, Int<1>{}, t2)) return;
        pq = t2[0];
        const float alpha = (float)(rz / pq);
        if (!(fabsf(alpha) < INFINITY && fabsf(beta) < INFINITY)) {
            if (lead) {
                *abort_word = kAbortNotFinite;
                if (!SINGLE) slots[kTurnWord] = turn;
            }
            return;
        }
#pragma unroll
        for (int r = 0; r < kVbRows; r++) {
            b.e[r] = b.e[r] + alpha * b.p[r];
            b.r[r] = b.r[r] - alpha * q[r];
        }
        if (SINGLE) publish_rim();
        rr_rz();
        if (!total(part, Int<2>{}, t2)) return;
        rr = t2[0];
        rzold = rz;
        rz = t2[1];
        iter++;
        if (rr <= eta2 * rr0) done = true;
    }
    if (b.in) {
#pragma unroll
        for (int r = 0; r < kVbRows; r++)
            if (r < b.nr) I.e[b.n0 + r * NY] = b.e[r];
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
        if (!SINGLE) slots[kTurnWord] = turn;
    }
}

namespace {

int vb_count(int NX, int NY) { return ((NY + kGridBX - 1) / kGridBX) * ((NX + kGridBY - 1) / kGridBY); }

template <bool SINGLE> int fits(int blocks, int threads, size_t lds)
{
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return false;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, (const void *)k_cg_pass<SINGLE>, threads, lds) != hipSuccess)
        return false;
    return (long long)per * cus >= blocks;
}

} // namespace

size_t cg_rim_words(int NX, int NY)
{
    const int nvb = vb_count(NX, NY);
    return nvb > kCgSingleVb ? (size_t)NX * NY + 8 * (size_t)nvb : 0;
}

CgPlan cg_plan(int NX, int NY)
{
    CgPlan p{};
    const int nvb = vb_count(NX, NY);
    p.nvb = nvb;
    p.bx = (NY + kGridBX - 1) / kGridBX;
    p.single = nvb <= kCgSingleVb;
    if (p.single) {
        p.blocks = 1;
        p.threads = 64 * nvb;
        p.lds = (size_t)NX * NY * sizeof(float);
        p.ok = fits<true>(1, p.threads, p.lds);
    } else {
        // one chain of the totals per work-group, one wavefront per virtual block
        const int waves = (nvb + 255) / 256;
        p.blocks = nvb < 256 ? nvb : 256;
        p.threads = 64 * waves;
        p.ok = waves <= 16 && fits<false>(p.blocks, p.threads, 0);
    }
    return p;
}

hipError_t launch_cg_pass(const Inst *I, const CgPlan &p, unsigned epoch, int cap, unsigned long long *rim,
                          unsigned long long *slots, int *abort_word, long long wait, hipStream_t s)
{
    int bx = p.bx, nvb = p.nvb;
    if (p.single) {
        hipLaunchKernelGGL(k_cg_pass<true>, dim3(1), dim3(p.threads), p.lds, s, I, bx, nvb, epoch, cap, rim, slots,
                           abort_word, wait);
        return hipGetLastError();
    }
    // cooperative: the runtime keeps two such launches of one process from
    // sharing the chip half and half
    void *args[] = {&I, &bx, &nvb, &epoch, &cap, &rim, &slots, &abort_word, &wait};
    return hipLaunchCooperativeKernel((const void *)k_cg_pass<false>, dim3(p.blocks), dim3(p.threads), args, 0, s);
}

} // namespace pic
