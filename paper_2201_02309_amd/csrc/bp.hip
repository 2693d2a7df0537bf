// Backprojection over the PI interval (Sec. II backprojection step) for gfx950.
//
// f(x) = dlambda/(2 pi) sum_n c_n(x) / v*_n(x) g^F(lambda_n, alpha*_n(x), w*_n(x)),
// v* = R - x cos(b) - y sin(b), alpha* = atan(u / v*), u = -x sin(b) + y cos(b),
// w* = D cos(alpha*) / v* (z - z0 - P lambda / 2 pi) = D (z - z0 - P lambda / 2 pi) / sqrt(u^2+v*^2),
// with b = lambda + lambda0 and c_n the overlap of view cell [n-1/2, n+1/2] with the PI
// interval [l_i, l_o] (view units); c_n differs from 0 and 1 only at the first and last
// view of the interval.
//
// Every pitch k reuses the first pitch's tables (Sec. II periodicity): slice j of pitch k
// sees view n = n_lo + k Nv + m exactly as slice j of pitch 0 sees view n_lo + m, so the
// per-view table (cos b, sin b, e_m = z_first - z0 - h lambda_{n_lo+m}), the PI table
// (l_i, l_o, n_first, n_last relative to n_lo) and the footprint boxes are indexed by the
// pitch-relative view m and slice j only: the geometry is bit-identical for every pitch.
#include "bp_common.hpp"

#include <type_traits>
#include <vector>

namespace kats {

namespace {

using namespace bpdev;

// ---------------------------------------------------------------------------------
// Forward backprojection.  Workgroup = 256 lanes = a 16 x 16 (x, y) tile (4 waves of
// 8 x 8) x a run of KZ consecutive slices of one pitch; every lane keeps KZ accumulators.
// The workgroup walks the hull of its voxels' PI windows view by view.  For each view the
// plan gives the tile's detector footprint box (float64 bound); the box of view m+1 is
// loaded from HBM into registers while view m is backprojected from LDS, then stored into
// the other LDS buffer (one barrier per view).  Per (lane, view): v*, 1/v*, 1/rho and the
// column coordinate (atan); per (lane, view, slice): the row coordinate (one FMA: rows
// advance by dz D / (rho dw) per slice), two ds_read2 of the 2 x 2 taps, three lerps and
// one FMA into the accumulator.  Slices are handled in groups of kKG; one comparison of the view
// with sixteen limits held across a wave's lanes says which groups have an active voxel and
// which are wholly inside their voxels' PI windows: inactive groups are skipped by a wave-uniform
// branch and covered ones skip the coverage arithmetic.  When the plan has boxes larger than
// every LDS shape, the kernel instance with the fallback reads those views' taps from the
// zero-padded g^F in HBM instead.
//
// Bound by VALU issue and LDS reads together (without half of the reads the clinical workload took
// 1.25 ms less, without two of twelve VALU operations per slice 0.35 ms less), so registers and LDS
// are kept to five workgroups per CU.  512 x 512 x 128 from 2826 views, whole reconstruction:
// 10.99 -> 10.84 ms (bit-identical); 256 x 256 x 96 with 38 x 79 boxes, backprojection 3.1 -> 2.6 ms.
// ---------------------------------------------------------------------------------
// Box tile of a kernel instance: rows of kPitch floats in LDS, boxes of up to kCols columns and
// kRows rows staged by kLanes lanes a row (one float4 each) in kPass passes.  The pitch moves each
// row by eight banks, so lanes reading one column at different rows meet fewer conflicts (9.11 ms
// against 9.15 ms on the clinical workload with 64-float rows).  The dynamic LDS holds the plan's
// own largest box; a plan takes the first shape that its boxes fit (bp_shape), and only if none
// does the instance that reads larger boxes' taps from HBM.
template <int COLS, int ROWS>
struct Shape {
    static constexpr int kCols = COLS, kRows = ROWS, kPitch = COLS + 8;
    static constexpr int kLanes = COLS / 4, kStep = kNT / kLanes, kPass = (ROWS + kStep - 1) / kStep;
    static_assert(kPass >= 2, "staging passes");
    // passes that LDS always holds whole, so that they store without a mask
    static constexpr int kFree = kStep >= 32 ? 1 : 2;
};

// 16-byte store to LDS
__device__ inline void store4(__attribute__((address_space(3))) float *p, const float4 &v) {
    typedef float V __attribute__((ext_vector_type(4)));
    *(__attribute__((address_space(3))) V *)p = (V){v.x, v.y, v.z, v.w};
}

// One workgroup task: tile (bx, by) of the grid, slice run / pitch bz = pitch * runs + run.
// Shared by the one-plan kernel (task = block index) and the packed multi-plan kernel.
// FB: some box of the plan may exceed the LDS tile (those views read their taps from HBM);
// without it the view loop has a single path, which keeps the accumulators in place.
// P4: the plan's atan polynomial has degree <= 4 in t^2 (otherwise degree 8, or atan2f).
// SUB, TEAMS (small grids): the run is split over SUB tasks of KZ slices each, and the hull's views
// over TEAMS groups of 256 lanes with box buffers of their own, whose sums are added in order.
template <int KZ, class SH, bool FB, bool P4, int SUB, int TEAMS>
__device__ void bp_tile(const BpArgs p, const float *__restrict__ gF, float *__restrict__ vol,
                        const float4 *__restrict__ view_tab, const uint2 *__restrict__ box_tab,
                        int bxi, int byi, int bz, int lds_rows, unsigned char *smem, int *red) {
    static_assert(KZ % kKG == 0 && KZ / kKG <= 8, "groups use 8-bit masks");
    constexpr int NP = SH::kPass, kRowF = SH::kPitch, kStep = SH::kStep;
    constexpr int NG = KZ / kKG;
    const int cells = kRowF * lds_rows;                      // of one box buffer
    typedef __attribute__((address_space(3))) float LdsF;
    const int tid = threadIdx.x & (kNT - 1);
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int team = TEAMS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kNT) : 0;
    LdsF *lds = (LdsF *)smem + team * 2 * cells;
    const int ix = bxi * kT + (wave & 1) * 8 + (lane & 7);     // a wave: 8 x 8 voxel columns
    const int iy = byi * kT + (wave >> 1) * 8 + (lane >> 3);
    const int sub = SUB > 1 ? bz % SUB : 0;
    const int pitch = bz / SUB / p.runs;
    const int run = bz / SUB % p.runs;
    const int j0 = run * KZ * SUB + sub * KZ;                // first slice
    const int slices = min(p.ns, p.nz - pitch * p.ns);
    const int nrun = min(KZ, slices - j0);
    if (nrun <= 0) return;                                   // uniform over the workgroup
    const bool inxy = ix < p.nx && iy < p.ny;
    const long long base = (long long)p.n_lo + (long long)pitch * p.Nv;   // view of m = 0

    // Coverage c_n = clamp(min(m - A, B - m), 0, 1), A = l_i - 1/2, B = l_o + 1/2.  A lane keeps one
    // limit per slice: -A until its group's voxels are all past their first view, B from the group's
    // first view in which one of them may end (reloaded then).
    float E[KZ], acc[KZ];
    unsigned valid = 0;
    int wlo = INT_MAX, whi = INT_MIN;
    int g_alo[NG], g_ahi[NG], g_flo[NG], g_fhi[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        int alo = INT_MAX, ahi = INT_MIN, flo = INT_MIN, fhi = INT_MAX;
#pragma unroll
        for (int s = 0; s < kKG; ++s) {
            const int jj = g * kKG + s;
            E[jj] = -3.0e38f;
            acc[jj] = 0.0f;
            if (inxy && jj < nrun) {
                const PiEntry e = ldg(p.pi + ((size_t)(j0 + jj) * p.ny + iy) * p.nx + ix);
                const long long nf = base + e.nf, nl = base + e.nl;
                if (e.nf <= e.nl && nf - 1 >= 0 && nl + 1 <= p.n_views - 1) {
                    const float A = e.li - 0.5f, B = e.lo + 0.5f;
                    E[jj] = -A;
                    valid |= 1u << jj;
                    alo = min(alo, e.nf);
                    ahi = max(ahi, e.nl);
                    // views with c_n = 1 for certain (one view of margin against rounding)
                    flo = max(flo, (int)ceilf(A + 1.0f) + 1);
                    fhi = min(fhi, (int)floorf(B - 1.0f) - 1);
                }
            }
        }
        // a group is active at m if one of its voxels is; full if every valid voxel of the
        // group has c_n = 1 at m
        g_alo[g] = wave_min(alo);
        g_ahi[g] = wave_max(ahi);
        g_flo[g] = wave_max(flo);
        g_fhi[g] = wave_min(fhi);
        wlo = min(wlo, g_alo[g]);
        whi = max(whi, g_ahi[g]);
    }
    if (lane == 0 && team == 0) {
        red[wave] = wlo;
        red[4 + wave] = whi;
    }
    __syncthreads();
    // wave-uniform (scalar) so that the per-view box and view-table reads are scalar loads
    int mlo = __builtin_amdgcn_readfirstlane(min(min(red[0], red[1]), min(red[2], red[3])));
    int mhi = __builtin_amdgcn_readfirstlane(max(max(red[4], red[5]), max(red[6], red[7])));
    // this team's share of the hull; every team walks `steps` views, the last ones' idle
    const int steps = mlo <= mhi ? (mhi - mlo) / TEAMS + 1 : 0;
    if (TEAMS > 1 && mlo <= mhi) {
        mlo += team * steps;
        mhi = min(mhi, mlo + steps - 1);
    }
    // Per-view group classification of this wave: lane kind NG + g holds the first view at which
    // group g has started (kind 0), has ended (1), is past every voxel's first view (2), has a
    // voxel near its last view (3), so that one comparison with the view and a ballot give the
    // sixteen answers in a scalar register.
    int bound = INT_MAX;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        bound = lane == g ? g_alo[g] : bound;
        bound = lane == NG + g ? g_ahi[g] + 1 : bound;
        bound = lane == 2 * NG + g ? g_flo[g] : bound;
        bound = lane == 3 * NG + g ? min(g_fhi[g], INT_MAX - 1) + 1 : bound;
    }
    constexpr unsigned kG = (1u << NG) - 1u;
    const unsigned column = (unsigned)(iy * p.nx + ix);      // of the PI table's planes
    unsigned ending = 0;                                     // groups whose E holds B

    const float x = fmaf((float)ix, p.dx, p.x_first);
    const float y = fmaf((float)iy, p.dy, p.y_first);
    const float zoff = (float)(run * KZ * SUB) * p.dz;
    const int cpitch = p.gf_cols;
    const size_t vstride = (size_t)p.gf_rows * cpitch;
    // boxes read as two dwords (scalar loads) and unpacked: {r0 | nr << 16, c0 | nc << 16}
    const uint2 *__restrict__ boxes =
        box_tab + ((size_t)(run * p.tiles_y + byi) * p.tiles_x + bxi) * p.W;
    // g^F of pitch-relative view 0; element (0, 0) of a view is detector cell (-kPad, -kPad)
    const float *gF0 = gF + (size_t)(base - p.first_view) * vstride;
    auto fits = [](const BpBox &b) { return !FB || (b.nr <= SH::kRows && b.nc <= SH::kCols); };

    // Box staging: one aligned float4 per lane and pass (the plan starts every box on a 16-byte
    // boundary of the padded row).  Lanes past the box repeat its last row or first column into
    // LDS cells that nothing reads: no lane is masked off, so the loads of a view stay in flight
    // together (masked ones each waited for the one before).
    // Passes that the box does not reach are left out from the third on, in whole tasks of 8 slices from
    // the second: 356 x 356 x 5, 16 x 27 boxes, 358 -> 349 us; 512 x 512 x 128 in runs of 8 slices 9.23 ->
    // 8.78 ms.  In halves, which mostly have more rows, that cost 512 x 512 x 10 3 % (450 -> 462 us).
    constexpr int kAlways = KZ == 8 && SUB == 1 ? 1 : 2;
    const int srow = tid / SH::kLanes, scol = (tid % SH::kLanes) * 4;
    auto fetch = [&](int m, const BpBox &b, float4 *v) {
        const float *src = gF0 + (size_t)m * vstride + (b.r0 + kPad) * cpitch + (b.c0 + kPad);
        const int col = scol < b.nc ? scol : 0;
#pragma unroll
        for (int k = 0; k < NP; ++k)
            if (k < kAlways || kStep * k < b.nr)
                v[k] = ldg(reinterpret_cast<const float4 *>(src + min(srow + kStep * k, b.nr - 1) * cpitch + col));
    };
    auto put = [&](int buf, const BpBox &b, const float4 *v) {
        LdsF *dst = lds + buf * cells + srow * kRowF + scol;
#pragma unroll
        for (int k = 0; k < NP; ++k)
            if ((k < kAlways || kStep * k < b.nr) && (k < SH::kFree || srow + kStep * k < lds_rows) &&
                (kNT % SH::kLanes == 0 || srow < kStep))
                store4(dst + kStep * k * kRowF, v[k]);
    };
    uint2 bw_next = make_uint2(0u, 0u);   // box of the view after the current one
    if (mlo <= mhi) {
        const BpBox b = unpack_box(ldg(boxes + mlo));
        bw_next = ldg(boxes + min(mlo + 1, mhi));
        if (fits(b)) {
            float4 v[NP];
            fetch(mlo, b, v);
            put(0, b, v);
        }
    }
    __syncthreads();
    BpBox b = unpack_box(ldg(boxes + (mlo <= mhi ? mlo : 0)));
    for (int step = 0; step < steps; ++step) {
        const int m = mlo + step, buf = step & 1;
        if (TEAMS > 1 && m > mhi) {                          // (uniform over the team's waves)
            __syncthreads();
            continue;
        }
        // box of view m+2, loaded one iteration ahead of its use
        const uint2 bw_after = ldg(boxes + min(m + 2, mhi));
        // prefetch the next view's box into registers (the last view's once more at the end)
        const BpBox bn = unpack_box(bw_next);
        const bool next_fits = fits(bn);
        float4 pf[NP];
        if (next_fits) fetch(min(m + 1, mhi), bn, pf);
        // per (lane, view) geometry; coordinates relative to the box origin, clamped into
        // the box (only voxels projecting outside the zero-padded detector are clamped)
        const float4 vt = ldg(view_tab + m);
        const float u = fmaf(-x, vt.y, y * vt.x);
        const float v = p.R - fmaf(x, vt.x, y * vt.y);
        const float vinv = __builtin_amdgcn_rcpf(v);
        const float rinv = __builtin_amdgcn_rsqf(fmaf(u, u, v * v));
        float acol;                                          // alpha* / dalpha
        if (P4 || p.atan_deg >= 0) {
            const float t = u * vinv;                        // tan(alpha*)
            const float s2 = t * t;
            constexpr int deg = P4 ? 4 : 8;
            float qa = p.atan_coef[deg];
#pragma unroll
            for (int k = deg - 1; k >= 0; --k) qa = fmaf(qa, s2, p.atan_coef[k]);
            acol = t * qa;
        } else {
            acol = atan2f(u, v) * p.inv_dalpha;
        }
        const float cc = med3(acol + (p.col_c - (float)b.c0), 0.0f, (float)(b.nc - 2));
        const int c0 = (int)cc;
        const float tc = cc - (float)c0;
        const float q = p.q_scale * rinv;                   // detector rows per mm of z
        float rb = fmaf(q, vt.z + zoff, p.row_c - (float)b.r0);
        const float st = q * p.dz;
        if (SUB > 1) rb = fmaf((float)(sub * KZ), st, rb);
        const float rmax = (float)(b.nr - 2);
        const float mf = (float)m;
        const unsigned word = (unsigned)__ballot(m >= bound);
        const unsigned active = word & ~(word >> NG) & kG;
        const unsigned before = ~(word >> (2 * NG)) & kG, after = (word >> (3 * NG)) & kG;
        // one group of kKG slices: the taps of all its slices, then their interpolation
        struct Taps {
            float v00[kKG], v01[kKG], v10[kKG], v11[kKG], tr[kKG];
        };
        auto take = [&](auto T, int tp, int g, Taps &x) {   // T: LDS or global taps
#pragma unroll
            for (int s = 0; s < kKG; ++s) {
                const float rr = med3(fmaf((float)(g * kKG + s), st, rb), 0.0f, rmax);
                const int r0 = (int)rr;               // rr >= 0: truncation = floor
                x.tr[s] = __builtin_amdgcn_fractf(rr);
                const auto t = T + __mul24(r0, tp);
                x.v00[s] = t[0];
                x.v01[s] = t[1];
                x.v10[s] = t[tp];
                x.v11[s] = t[tp + 1];
            }
        };
        auto add = [&](int g, const Taps &x) {
            float val[kKG];
#pragma unroll
            for (int s = 0; s < kKG; ++s) {
                const float top = fmaf(tc, x.v01[s] - x.v00[s], x.v00[s]);
                const float bot = fmaf(tc, x.v11[s] - x.v10[s], x.v10[s]);
                val[s] = fmaf(x.tr[s], bot - top, top);
            }
            // the coverage weight scales the values in place, so that both paths end in
            // the same FMA on the accumulators
            if ((before | after) & (1u << g)) {
                // uniform base of the group's first slice, 32-bit lane offset
                const size_t plane = (size_t)p.ny * p.nx;
                const PiEntry *pi = p.pi + (size_t)(j0 + g * kKG) * plane;
                // (hidden from the compiler, which would keep every slice's address and flag in
                // registers over the whole view loop)
                unsigned col = column, ok = valid >> (g * kKG);
                asm volatile("" : "+v"(col), "+v"(ok));
                float c[kKG];
                if (before & after & (1u << g)) {            // a short or steep group: both limits
#pragma unroll
                    for (int s = 0; s < kKG; ++s) {
                        c[s] = 0.0f;
                        if ((ok >> s) & 1u) {
                            const float2 l = ldg(reinterpret_cast<const float2 *>(pi + s * plane + col));
                            c[s] = med3(fminf(mf - (l.x - 0.5f), l.y + 0.5f - mf), 0.0f, 1.0f);
                        }
                    }
                } else {
                    if (after & ~ending & (1u << g)) {
                        ending |= 1u << g;
#pragma unroll
                        for (int s = 0; s < kKG; ++s)
                            if ((ok >> s) & 1u)
                                E[g * kKG + s] = ldg(reinterpret_cast<const float2 *>(pi + s * plane + col)).y + 0.5f;
                    }
                    const float sm = (after >> g) & 1u ? -mf : mf;
#pragma unroll
                    for (int s = 0; s < kKG; ++s) c[s] = med3(E[g * kKG + s] + sm, 0.0f, 1.0f);
                }
#pragma unroll
                for (int s = 0; s < kKG; ++s) val[s] *= c[s];
            }
#pragma unroll
            for (int s = 0; s < kKG; ++s) acc[g * kKG + s] = fmaf(vinv, val[s], acc[g * kKG + s]);
        };
        if (fits(b)) {
            const LdsF *T = lds + buf * cells + c0;
#pragma unroll
            for (int g = 0; g < NG; ++g)
                if (active & (1u << g)) {
                    Taps x;
                    take(T, kRowF, g, x);
                    add(g, x);
                }
        } else {
            const auto T = glb(gF0 + (size_t)m * vstride + (b.r0 + kPad) * cpitch + (b.c0 + kPad) + c0);
#pragma unroll
            for (int g = 0; g < NG; ++g)
                if (active & (1u << g)) {
                    Taps x;
                    take(T, cpitch, g, x);
                    add(g, x);
                }
        }
        if (next_fits) put(buf ^ 1, bn, pf);
        b = bn;
        bw_next = bw_after;
        __syncthreads();
    }
    if (TEAMS > 1) {
        // the other teams' sums through LDS (their boxes are done with)
        LdsF *sums = (LdsF *)smem + tid;
        if (team > 0)
#pragma unroll
            for (int jj = 0; jj < KZ; ++jj) sums[((team - 1) * KZ + jj) * kNT] = acc[jj];
        __syncthreads();
        if (team > 0) return;
#pragma unroll
        for (int t = 1; t < TEAMS; ++t)
#pragma unroll
            for (int jj = 0; jj < KZ; ++jj) acc[jj] += sums[((t - 1) * KZ + jj) * kNT];
    }
    if (!inxy) return;
    const int iz0 = pitch * p.ns + j0;
#pragma unroll
    for (int jj = 0; jj < KZ; ++jj) {
        if (jj < nrun)
            glb(vol)[((size_t)(iz0 + jj) * p.ny + iy) * p.nx + ix] =
                ((valid >> jj) & 1u) ? acc[jj] * p.scale : 0.0f;
    }
}

// Waves per SIMD that the registers are kept to: 5 where the 16-slice kernels fit 96 registers without
// spilling (6, with spills, measured within 1 % of it on the clinical workload and slower elsewhere).
constexpr int bp_waves(int kz, bool fb, int passes) { return kz >= 32 ? 2 : (fb || passes > 4 ? 4 : 5); }

template <int KZ, class SH, bool FB, bool P4, int SUB, int TEAMS>
__global__ __launch_bounds__(kNT * TEAMS, TEAMS > 1 ? 1 : bp_waves(KZ, FB, SH::kPass)) void k_bp_lds(BpArgs p, const float *__restrict__ gF,
                                                float *__restrict__ vol,
                                                const float4 *__restrict__ view_tab,
                                                const uint2 *__restrict__ box_tab, int lds_rows) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int red[8];
    const unsigned tiles = gridDim.x * gridDim.y;
    const TileAt t = xcd_tile(kXcdForward, gridDim.x, gridDim.y, blockIdx.x + gridDim.x * blockIdx.y, blockIdx.z, tiles * blockIdx.z);
    bp_tile<KZ, SH, FB, P4, SUB, TEAMS>(p, gF, vol, view_tab, box_tab, t.x, t.y, blockIdx.z, lds_rows, smem, red);
}

// ---------------------------------------------------------------------------------
// Grouped backprojection of several plans in one launch (serving): the grid enumerates
// the (pitch, slice run, tile) tasks of up to kGroupMax requests back to back; a block
// finds its request from the task prefix held in the kernel argument (a wave-uniform scan)
// and runs that request's tile exactly as the one-plan kernel does.  Descriptors travel as
// kernel arguments, so the compiler sees them as constant memory (scalar loads, global
// pointers), as for the one-plan kernel.
// ---------------------------------------------------------------------------------
struct BpRequest {
    BpArgs a;
    const float *gF;
    float *vol;
    const float4 *view;
    const uint2 *boxes;
    long long first_task;          // prefix of the task counts of earlier requests
};

constexpr int kGroupMax = 16;
struct BpGroup {
    BpRequest r[kGroupMax];
    int n;
};
static_assert(sizeof(BpGroup) <= 4000, "kernel argument segment");

template <int KZ, class SH, bool FB, bool P4, int SUB, int TEAMS>
__global__ __launch_bounds__(kNT * TEAMS, TEAMS > 1 ? 1 : bp_waves(KZ, FB, SH::kPass)) void k_bp_group(const BpGroup g, int lds_rows) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int red[8];
    const long long task = blockIdx.x;
    int r = 0;
    while (r + 1 < g.n && g.r[r + 1].first_task <= task) ++r;
    const BpRequest &q = g.r[r];
    const unsigned local = (unsigned)(task - q.first_task), tiles = (unsigned)q.a.tiles_x * (unsigned)q.a.tiles_y;
    const unsigned bz = local / tiles, l = local - bz * tiles;
    const TileAt t = xcd_tile(kXcdForward, q.a.tiles_x, q.a.tiles_y, l, bz, (unsigned)task - l);
    bp_tile<KZ, SH, FB, P4, SUB, TEAMS>(q.a, q.gF, q.vol, q.view, q.boxes, t.x, t.y, (int)bz, lds_rows, smem, red);
}

}  // namespace

// The box shapes, in the order of kShapeRows and kShapeCols.
using S32x64 = Shape<64, 32>;      // 16-slice runs of full detectors (clinical: 32 x 44)
using S64x32 = Shape<32, 64>;      // sparse detectors: few columns, steep slices (49 x 25)
using S64x64 = Shape<64, 64>;
using S48x80 = Shape<80, 48>;      // coarse grids under fine detectors (40 x 79): rows of 88 floats, five
                                   // workgroups per CU (five requests 21.5 -> 20.2 ms against S48x96)
using S64x80 = Shape<80, 64>;
using S48x96 = Shape<96, 48>;
using S48x128 = Shape<128, 48>;
// f(instance tag) for the class's template arguments
template <int KZ_, class SH_, bool FB_, bool P4_, int SUB_, int TEAMS_>
struct BpInst {
    using SH = SH_;
    static constexpr int KZ = KZ_, SUB = SUB_, TEAMS = TEAMS_;
    static constexpr bool FB = FB_, P4 = P4_;
};

template <class SH, bool FB, class F>
static void with_split(const BpClass &c, F f) {
    if (c.split == kHalves) f(BpInst<8, SH, FB, false, 2, 1>{});
    else if (c.split == kHalvesTeams) f(BpInst<8, SH, FB, false, 2, 4>{});
    else if (c.split == kQuartersTeams) f(BpInst<4, SH, FB, false, 4, 4>{});
    else if (c.split == kThin) {
        if constexpr (std::is_same<SH, S32x64>::value && !FB)
            c.poly4 ? f(BpInst<8, SH, FB, true, 1, 1>{}) : f(BpInst<8, SH, FB, false, 1, 1>{});
    }
    else if (c.poly4) f(BpInst<16, SH, FB, true, 1, 1>{});
    else f(BpInst<16, SH, FB, false, 1, 1>{});
}

template <int KZ, class F>
static void with_instance(const BpClass &c, F f) {
    if constexpr (KZ == 16) {
        switch (c.shape) {
            case 0: return with_split<S32x64, false>(c, f);
            case 1: return with_split<S64x32, false>(c, f);
            case 2: return with_split<S64x64, false>(c, f);
            case 3: return with_split<S48x80, false>(c, f);
            case 4: return with_split<S64x80, false>(c, f);
            case 5: return with_split<S48x96, false>(c, f);
            case 6: return with_split<S48x128, false>(c, f);
            default: return with_split<S32x64, true>(c, f);
        }
    } else {
        using S = typename std::conditional<(KZ < 16), S32x64, S64x64>::type;
        if (c.shape == kFallback) c.poly4 ? f(BpInst<KZ, S, true, true, 1, 1>{}) : f(BpInst<KZ, S, true, false, 1, 1>{});
        else c.poly4 ? f(BpInst<KZ, S, false, true, 1, 1>{}) : f(BpInst<KZ, S, false, false, 1, 1>{});
    }
}

template <class F>
static void with_instance(int kz, const BpClass &c, F f) {
    switch (kz) {
        case 8: return with_instance<8>(c, f);
        case 32: return with_instance<32>(c, f);
        default: return with_instance<16>(c, f);
    }
}

// LDS rows of a launch whose largest box has `rows` (the whole tile with the HBM path)
template <class I>
static int lds_rows(int rows) {
    const int least = I::SH::kFree * I::SH::kStep;
    return I::FB ? I::SH::kRows : (rows < least ? least : rows);
}

hipError_t launch_backproject(const KParams &k, const float *gF, float *vol, hipStream_t s) {
    const BpArgs a = bp_args(k);
    const uint2 *boxes = reinterpret_cast<const uint2 *>(k.boxes);
    with_instance(k.bp_kz, kernel_class(k), [&](auto inst) {
        using I = decltype(inst);
        const int rows = lds_rows<I>(k.bp_box_rows);
        const dim3 grid((unsigned)k.bp_tiles_x, (unsigned)k.bp_tiles_y, (unsigned)(k.n_pitches * k.bp_runs * I::SUB));
        hipLaunchKernelGGL((k_bp_lds<I::KZ, typename I::SH, I::FB, I::P4, I::SUB, I::TEAMS>), grid,
                           dim3(kNT * I::TEAMS), bp_bytes(I::TEAMS, I::SH::kPitch, rows, I::KZ), s, a, gF, vol, k.view,
                           boxes, rows);
    });
    return hipGetLastError();
}

// Requests are grouped by kernel instance (box shape, split, polynomial degree); each launch takes
// up to kGroupMax requests of one class.
hipError_t launch_backproject_batch(const KParams *ks, const float *const *gF, float *const *vol,
                                    int n, int kz, hipStream_t s) {
    const std::vector<BpClass> classes = batch_classes(ks, n);
    for (int shape = 0; shape <= kShapes; ++shape)
        for (int split = 0; split < kSplits; ++split)
            for (int poly4 = 0; poly4 < 2; ++poly4) {
                const BpClass cls{shape, split, poly4};
                BpGroup grp{};
                long long total = 0;
                int rows = 0;
                auto flush = [&]() {
                    if (grp.n == 0) return;
                    with_instance(kz, cls, [&](auto inst) {
                        using I = decltype(inst);
                        const int r = lds_rows<I>(rows);
                        hipLaunchKernelGGL((k_bp_group<I::KZ, typename I::SH, I::FB, I::P4, I::SUB, I::TEAMS>),
                                           dim3((unsigned)total), dim3(kNT * I::TEAMS),
                                           bp_bytes(I::TEAMS, I::SH::kPitch, r, I::KZ), s, grp, r);
                    });
                    grp = BpGroup{};
                    total = 0;
                    rows = 0;
                };
                for (int i = 0; i < n; ++i) {
                    const KParams &k = ks[i];
                    if (!(classes[i] == cls)) continue;
                    const long long tasks = (long long)k.bp_tiles_x * k.bp_tiles_y * k.n_pitches * k.bp_runs * kSubs[split];
                    if (tasks == 0) continue;
                    if (grp.n == kGroupMax || total + tasks > kMostThreads / (kNT * kTeams[split])) flush();
                    BpRequest &q = grp.r[grp.n++];
                    q.a = bp_args(k);
                    q.gF = gF[i];
                    q.vol = vol[i];
                    q.view = k.view;
                    q.boxes = reinterpret_cast<const uint2 *>(k.boxes);
                    q.first_task = total;
                    total += tasks;
                    rows = rows < k.bp_box_rows ? k.bp_box_rows : rows;
                }
                flush();
            }
    return hipGetLastError();
}

}  // namespace kats
