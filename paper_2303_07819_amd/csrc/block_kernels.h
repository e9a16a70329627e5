// K fine steps of a cell per launch (temporal blocking of the plain path).
//
// With the coarse step equal to the fine step the continuum never feeds back
// into the cell DEMs (Algorithm 1 with N0 = 1 takes no coarse-to-fine update),
// so a cell's floes stay on chip for K consecutive steps: the floe state and
// candidate lists are read once, every step's statistics go to their own slot
// of a K-slot ring for the continuum updates that follow the launch, and the
// state is written back once.  One workgroup per cell, one floe per lane: the
// launch takes as many wavefronts as its largest cell needs (up to 16, cells of
// up to 1024 floes).  A lane keeps its floe's state and inverse masses in
// registers; position, radius and velocity are in LDS beside them for the floes
// that touch it.  Per step the work is the per-step kernel's: list rebuild when
// the displacement bound passes half the skin (binned or all-pairs search), the
// exact contact decision, FP64 drag, contact forces in ascending partner order,
// the update, the FP64 statistics of the pre-step state, of which only the five
// that the continuum reads are formed (R_UBAR .. R_SW).
//
// What bounds it: VALU issue (486 VALU instructions per wavefront and step on
// 64 x 64 cells of 256 floes with 8 ocean modes, 98 % of the issue slots by
// SQ_ACTIVE_INST_VALU / SQ_BUSY_CU_CYCLES), so each choice below removes
// instructions or LDS traffic.  Measured there, us per step of a 32-step launch,
// 23.7 before: state in registers instead of LDS, five statistics instead of
// eight, arguments read where they are used instead of spilled scalar registers
// 18.1; only near candidates decided (kNearFrac) 17.2; mode constants through
// the scalar cache instead of LDS (LDS active 59 % -> 25 % of the time) 15.9;
// one workgroup per cell and one wavefront per 64 floes instead of 2^k (no
// change there; 128 x 128 cells of 0 to 700 floes 86 -> 83, 4096 cells of 64
// floes 6.7 -> 5.8).  Five wavefronts per SIMD with 24 B of spills: 15.9 against
// 17.0 with four and 17.8 with six.
//
// Contacts and candidates (list entries standing for decision, for the VALU
// accounting of the step) are counted per lane over the block and reduced once.
// TSP: the tangential spring (SP_TANGENTIAL_SPRING); each floe's contact
// history (partners and displacements, the per-step kernel's table) is staged
// in LDS at the end of the cell's memory for the block, read before the floe's
// contacts of a step and rewritten with them exactly as the per-step kernel
// does, and written back once.  LDS then holds three 256-floe cells per compute
// unit, so its wavefronts take the registers of three per SIMD (34.5 -> 22 us
// per step).
#pragma once

namespace spdem {

// Coarse-to-fine update at the end of a block (two-way coupling, Sec. 3.3):
// every cell of the launch is re-synchronised to X0 + frac (Q - X0) exactly as
// resync_kernel does (radii scaled by one factor up to r_lim, then uniform
// velocity and spin shifts), its floes still in LDS.  Inactive: x0m == null.
struct BlockNudge {
    const double* x0m;                 // [ncells][kMomStride] statistics at the coarse-step start
    const double* Q;                   // [4][ncells] coarse state
    double frac;
    double area;
    float r_lim;
    float* r;                          // radii (the launch's floes are rescaled in place)
    unsigned long long* counters;      // clamped, invalid cell updates
};

// Sum of one value per lane over the workgroup's nw wavefronts: DPP row sums,
// then the 4 nw row totals in a fixed order (every lane gets the same value).
// Every thread calls it.
__device__ __forceinline__ double group_sum_rows(double x, double* rows_g, int gt, int nw)
{
    x = row_sum(x);
    if ((gt & 15) == 15) rows_g[gt >> 4] = x;
    __syncthreads();
    double t = 0.0;
    for (int q = 0; q < 4 * nw; ++q) t += rows_g[q];
    __syncthreads();
    return t;
}

__device__ __forceinline__ float group_max(float x, float* wmax_g, int gt, int nw)
{
    x = wave_max_f32(x);
    if ((gt & 63) == 0) wmax_g[gt >> 6] = x;
    __syncthreads();
    float t = 0.0f;
    for (int q = 0; q < nw; ++q) t = fmaxf(t, wmax_g[q]);
    __syncthreads();
    return t;
}

// What a blocked launch reads.  The kernel takes it from the kernel argument
// segment again wherever it is needed rarely (block_args), so that only what
// every step uses stays in scalar registers.
struct BlockArgs {
    uint32_t* xi;
    uint32_t* yi;
    float* u;
    float* v;
    float* w;
    float* th;
    float* r;                  // written by a coarse-to-fine update only
    const float* h;
    const ModeC* modes;        // [ncells][nmodes]: every cell's mode constants
    uint4* tsp_j;
    double* tsp_x;
    uint16_t* vlist;
    uint8_t* vcount;
    float* vdisp;
    unsigned long long* contacts;
    unsigned long long* cands;
    uint32_t* err;
    const int4* work;
    double* ring;              // [K][kRing][ncells]: statistics of step t in slot t
    double* alt;               // [kRing][ncells]: where the statistics of work entries with w = 1 go instead
    int32_t cell_bytes, cap, ncells, K, nmodes, nbx, nby;
    uint32_t flags;
    float skin, qx, qy;
    float inv_qx, ratio;       // radii in units of qx, qy / qx (candidate tests)
    double qxd, qyd, inv_qxd, inv_qyd, dtd, Ed, Gd, mud;
    double cdpi;               // cd rho_o pi
    double rho_ice_d, u0, v0;
    int direct;                // as Modes
    BlockNudge nd;
};

// near_skin in units of the list skin: at 65 m of 389 m (25 km cells of 256
// floes) the near candidates last 3-8 steps of 4-9 m and are 0.3 of the 1.9
// listed ones, so that three of four steps test none of the others.  us per step
// with 1/12, 1/6, 1/3 and 1 of the skin: plain64 17.3, 17.0, 17.6, 19.1 (after 3000
// steps 24.0, 24.0, 24.6, 27.6); 64 floes per cell 7.7, 7.8, 8.1, 10.5; 512 floes
// per cell on 32 x 32 cells 9.5, 9.6, 9.9, 11.4; 32 floes in 50 km cells 5.9, 6.0,
// 6.0, 6.4.
constexpr float kNearFrac = 1.0f / 6.0f;

typedef const BlockArgs __attribute__((address_space(4)))* BlockArgsPtr;

// The launch's arguments read afresh (an opaque pointer to the kernel argument
// segment, whose first entry they are): scalar loads at the place of use.
__device__ __forceinline__ BlockArgsPtr block_args()
{
    BlockArgsPtr p = (BlockArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// Row totals (16 lanes) of five values per lane by a transposing exchange:
// while two values are left for a lane, it keeps one of them and adds its
// partner's copy of it (partners: lane i ^ 8 by row_ror:8, i ^ 7 by
// row_half_mirror, i ^ 2 and i ^ 1 by quad permutes).  Lane i of a row ends with
// the total of value 4 if i & 2, else of value 2 [i & 4] + [i & 8].  Every lane
// of the wavefront must be active.
__device__ __forceinline__ double row_sum5(const double (&v)[5], int lane)
{
    const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
    const double p = (b3 ? v[1] : v[0]) + dpp_perm<0x128>(b3 ? v[0] : v[1]);
    const double q = (b3 ? v[3] : v[2]) + dpp_perm<0x128>(b3 ? v[2] : v[3]);
    const double r = v[4] + dpp_perm<0x128>(v[4]);
    const double s = (b2 ? q : p) + dpp_perm<0x141>(b2 ? p : q);
    const double t = r + dpp_perm<0x141>(r);
    const double x = (b1 ? t : s) + dpp_perm<0x4e>(b1 ? s : t);
    return x + dpp_perm<0xb1>(x);
}

// Static LDS of dem_block_kernel<., W, .>: its arrays wsum, wdisp and rows.  A
// launch's dynamic LDS has to leave room for it.
constexpr size_t block_static_lds(int W)
{
    return (size_t)W * sizeof(int) + 2 * (size_t)W * sizeof(float) + 2 * (kRing + 1) * 4 * (size_t)W * sizeof(double);
}

// W: the most wavefronts of a launch (4, 8 or 16); a.work, a.cap and the
// launch's threads belong to one run of cells.
template <int SCHED, int W, bool TSP = false>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(TSP ? (W == 4 ? 3 : W == 8 ? 2 : 4) : 5)))
void dem_block_kernel(BlockArgs a)
{
    const int G = blockDim.x, nw = G >> 6;     // threads and wavefronts of the cell

    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int wsum[W];
    __shared__ __align__(16) float wdisp[2][W];           // largest squared displacement of each wavefront, by step parity
    __shared__ __align__(16) double rows[2][kRing + 1][4 * W];   // row totals of every statistic, by step parity

    const int gt = threadIdx.x;
    const int cap = a.cap;

    uint4* const P = reinterpret_cast<uint4*>(smem);       // xi, yi, padded r in units of qx (bits), r bits
    float4* const V = reinterpret_cast<float4*>(P + cap); // u, v, w, -
    uint4* const S = reinterpret_cast<uint4*>(V);         // sorted copy during a binned search (V is written again after it)
    uint16_t* const lst = reinterpret_cast<uint16_t*>(V + cap);
    int* const cnt = reinterpret_cast<int*>(lst + (size_t)cap * kListCap);
    // contact history (TSP): displacements [cap][SP_SPRING_CAP], then partners [cap]
    double* const HX = TSP ? reinterpret_cast<double*>(smem + a.cell_bytes - (size_t)cap * kSpringBytes) : nullptr;
    uint4* const HJ = TSP ? reinterpret_cast<uint4*>(HX + (size_t)cap * SP_SPRING_CAP) : nullptr;

    int4 wk = a.work[blockIdx.x];              // the same for every thread: scalar registers
    wk.x = __builtin_amdgcn_readfirstlane(wk.x);
    wk.y = __builtin_amdgcn_readfirstlane(wk.y);
    wk.z = __builtin_amdgcn_readfirstlane(wk.z);
    wk.w = __builtin_amdgcn_readfirstlane(wk.w);
    const int c = wk.x, s = wk.y, n = wk.z;
    const bool has = gt < n;                   // this lane's floe
    const float half_skin = 0.5f * a.skin;
    uint16_t* const my = lst + (size_t)gt * kListCap;

    const ModeTable modes = (ModeTable)(uintptr_t)(a.modes + (size_t)c * a.nmodes);
    float vd = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(a.vdisp[c])));
    // the floe
    uint32_t px = 0, py = 0;
    float rf = 1.0f, rs = 0.0f, th = 0.0f, uf = 0.0f, vf = 0.0f, wf = 0.0f;
    double inv_m = 0.0, inv_i = 0.0;
    int k = 0;                                 // its listed candidates
    if (has) {
        px = a.xi[s + gt];
        py = a.yi[s + gt];
        rf = a.r[s + gt];
        th = a.th[s + gt];
        uf = a.u[s + gt];
        vf = a.v[s + gt];
        wf = a.w[s + gt];
        const double rld = (double)rf;
        const double md = a.rho_ice_d * (double)a.h[s + gt] * kPi * rld * rld;
        inv_m = 1.0 / md;
        inv_i = 1.0 / (md * (rld * rld));
        rs = rf * a.inv_qx * kTestPad;
        P[gt] = make_uint4(px, py, __float_as_uint(rs), __float_as_uint(rf));
        V[gt] = make_float4(uf, vf, wf, 0.0f);
        if (TSP) {
            HJ[gt] = a.tsp_j[s + gt];
#pragma unroll
            for (int q = 0; q < SP_SPRING_CAP; ++q) HX[gt * SP_SPRING_CAP + q] = a.tsp_x[(size_t)(s + gt) * SP_SPRING_CAP + q];
        }
        if (vd <= half_skin) {   // the kept lists are valid for the first step
            const uint16_t* const vlst = a.vlist + (size_t)s * kListCap;
            k = a.vcount[s + gt];
            for (int q = 0; q < k; q += 8)
                *reinterpret_cast<uint4*>(my + q) = *reinterpret_cast<const uint4*>(vlst + (size_t)q * n + (size_t)gt * 8);
        }
    }
    bool rebuilt = false;
    const float near_skin = kNearFrac * a.skin, near_pad = near_skin * a.inv_qx * kTestPad;
    float vd_near = -__builtin_inff();         // the bound when `near` was made
    uint32_t near = 0;
    uint32_t my_contacts = 0, my_tests = 0;    // this lane's counts over the block
    __syncthreads();                           // the staged state is in place

    const int K = a.K;
    int turn = 0;                              // the wavefront that writes this step's statistics
    for (int step = 0; step < K; ++step) {
        const int par = step & 1;
        const bool build = !(vd <= half_skin); // the same for every thread
        const float vnow = build ? 0.0f : vd;  // displacement bound since the lists were (or are now) built
        if (build) {   // ---- candidate lists
            rebuilt = true;
            const BlockArgsPtr b = block_args();
            const float skin = b->skin, qx = b->qx, qy = b->qy;
            if (SCHED == 2) {
                const int nbx = b->nbx, nby = b->nby, nb = nbx * nby;
                int* const binof = reinterpret_cast<int*>(lst);   // sort scratch inside the lists
                int* const rank = binof + cap;
                int* const bcnt = cnt + cap;
                int* const bstart = bcnt + nb;
                if (has) cnt[gt] = 0;
                for (int q = gt; q < nb; q += G) bcnt[q] = 0;
                __syncthreads();
                int bn = 0;
                if (has) {
                    bn = (int)__umulhi(py, (uint32_t)nby) * nbx + (int)__umulhi(px, (uint32_t)nbx);
                    binof[gt] = bn;
                    rank[gt] = atomicAdd(&bcnt[bn], 1);
                }
                __syncthreads();
                group_exclusive_scan(bcnt, bstart, nb, gt, G, wsum);
                if (has)
                    S[bstart[bn] + rank[gt]] = make_uint4(px, py, __float_as_uint(rf), (uint32_t)gt | ((uint32_t)bn << 16));
                __syncthreads();
                if (has) {
                    // half shell over the sorted copy: the own sub-bin's tail and the
                    // east one, then the three of the row above, as runs of the order
                    const uint4 own = S[gt];
                    const int o = (int)(own.w & 0xffffu), ob = (int)(own.w >> 16);
                    const int by = ob / nbx, bx = ob - by * nbx;
                    const float rl = __uint_as_float(own.z) + skin;
                    const bool ex = nbx >= 3 && bx + 1 < nbx;     // the east sub-bin follows in the order
                    const int row = (by + 1 == nby ? 0 : by + 1) * nbx;
                    const int x0 = nbx < 3 || bx == 0 ? 0 : bx - 1, x1 = nbx < 3 ? nbx : min(bx + 2, nbx);
#pragma unroll 1
                    for (int q = 0; q < 4; ++q) {
                        int q0 = 0, q1 = 0;
                        if (q == 0) {
                            q0 = gt + 1;
                            q1 = bstart[ob + (ex ? 2 : 1)];
                        } else if (q == 1) {
                            if (nbx >= 3 && !ex) {                // east neighbour across the seam
                                q0 = bstart[by * nbx];
                                q1 = bstart[by * nbx + 1];
                            }
                        } else if (nby >= 3) {
                            if (q == 2) {
                                q0 = bstart[row + x0];
                                q1 = bstart[row + x1];
                            } else if (nbx >= 3 && bx == 0) {     // north-west and north-east across the seam
                                q0 = bstart[row + nbx - 1];
                                q1 = bstart[row + nbx];
                            } else if (nbx >= 3 && bx == nbx - 1) {
                                q0 = bstart[row];
                                q1 = bstart[row + 1];
                            }
                        }
                        sweep(S, q0, q1, own.x, own.y, rl, o, lst, cnt, qx, qy);
                    }
                }
                __syncthreads();   // lists complete (sweeps append to partners' lists), the sorted copy free
                if (has) V[gt] = make_float4(uf, vf, wf, 0.0f);
            } else if (has) {
                const float rl = rf + skin;
                int m = 0;
                for (int j = 0; j < n; ++j) {
                    const uint4 pj = P[j];
                    float diff, R2;
                    screen((int)(pj.x - px), (int)(pj.y - py), rl, __uint_as_float(pj.w), qx, qy, diff, R2);
                    if (diff < kGuard * R2) {
                        if (m < kListCap) my[m] = (uint16_t)j;
                        ++m;
                    }
                }
                cnt[gt] = m;
            }
            if (has) {
                k = cnt[gt];
                if (k > kListCap) {
                    atomicOr(b->err, kErrCapacity);
                    k = kListCap;
                }
                if (SCHED == 2) {   // ascending partner order
                    for (int i = 1; i < k; ++i) {
                        const uint16_t key = my[i];
                        int j = i - 1;
                        while (j >= 0 && my[j] > key) {
                            my[j + 1] = my[j];
                            --j;
                        }
                        my[j + 1] = key;
                    }
                }
            }
            if (SCHED == 2) __syncthreads();   // velocities in place again
        }

        // ---- near candidates: those within near_skin of touching, as a bit mask
        // over the ascending list.  Only they are decided until some floe of the
        // cell may have moved by half of near_skin; then every candidate is tested
        // again, four at a time (their positions loaded together; an index past
        // the list reads the floe itself and is skipped), in FP32 on padded radii
        if (build || !(vnow - vd_near <= 0.5f * near_skin)) {
            vd_near = vnow;
            near = 0;
            for (int q0 = 0; q0 < k; q0 += 4) {
                const uint2 ix = *reinterpret_cast<const uint2*>(my + q0);
                int jv[4];
                jv[0] = (int)(ix.x & 0xffffu);
                jv[1] = (int)(ix.x >> 16);
                jv[2] = (int)(ix.y & 0xffffu);
                jv[3] = (int)(ix.y >> 16);
                uint3 pj[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    jv[t] = q0 + t < k ? jv[t] : gt;
                    pj[t] = *reinterpret_cast<const uint3*>(P + jv[t]);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float fx = (float)(int)(pj[t].x - px), fy = (float)(int)(pj[t].y - py) * a.ratio;
                    const float R = rs + near_pad + __uint_as_float(pj[t].z);
                    if (fx * fx + fy * fy <= R * R && jv[t] != gt) near |= 1u << (q0 + t);
                }
            }
        }

        double acc[kRing] = {0.0, 0.0, 0.0, 0.0, 0.0};
        float disp2 = 0.0f;
        uint32_t pxn = px, pyn = py;
        float ufn = uf, vfn = vf, wfn = wf;
        if (has) {
            const double rld = (double)rf, uld = (double)uf, vld = (double)vf, wld = (double)wf;
            double Fx = 0.0, Fy = 0.0, T = 0.0;
            // ---- ocean drag and drag torque
            if (!(a.flags & SP_OCEAN_OFF)) {
                const float fx = (float)(int)(px - 0x80000000u) * 2.3283064365386963e-10f;
                const float fy = (float)(int)(py - 0x80000000u) * 2.3283064365386963e-10f;
                double uo = a.u0, vo = a.v0, zeta = 0.0;
                ocean_modes(fx, fy, modes, a.nmodes, a.direct != 0, uo, vo, zeta);
                drag_terms(uo - uld, vo - vld, zeta, wld, rld, a.cdpi, Fx, Fy, T);
            }
            acc[0] = uld;
            acc[1] = vld;
            acc[2] = Fx;
            acc[3] = Fy;
            acc[4] = T;
            my_tests += (uint32_t)k;
            // ---- contact forces and torques in ascending partner order (FP64)
            uint4 hj = make_uint4(0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu);   // the floe's contact history (TSP)
            double hx[SP_SPRING_CAP];
            uint16_t* const tj = TSP ? reinterpret_cast<uint16_t*>(HJ + gt) : nullptr;
            double* const tx = TSP ? HX + (size_t)gt * SP_SPRING_CAP : nullptr;
            bool had = false;   // the floe was in contact after the previous step
            if (TSP) {
                hj = HJ[gt];
                had = (hj.x & hj.y & hj.z & hj.w) != 0xffffffffu;
#pragma unroll
                for (int q = 0; q < SP_SPRING_CAP; ++q) hx[q] = had ? tx[q] : 0.0;
            }
            int nh = 0;
            for (uint32_t m = near; m; m &= m - 1u) {
                const int j = my[__builtin_ctz(m)];
                const uint4 pj = P[j];
                const int dxi = (int)(pj.x - px), dyi = (int)(pj.y - py);
                if (!exact_contact_inline(dxi, dyi, rld, __uint_as_float(pj.w), a.qxd, a.qyd)) continue;
                double cx, cy, ct, xi = 0.0, xi_old = 0.0;
                if (TSP) {
#pragma unroll
                    for (int e = 0; e < SP_SPRING_CAP; ++e) {
                        const uint32_t wv = e < 2 ? hj.x : e < 4 ? hj.y : e < 6 ? hj.z : hj.w;
                        if ((int)((wv >> (16 * (e & 1))) & 0xffffu) == j) xi_old = hx[e];
                    }
                }
                if (!contact_terms<TSP>(dxi, dyi, rld, uld, vld, wld, __uint_as_float(pj.w), V[j], gt < j, a, cx, cy,
                                        ct, xi_old, &xi)) {
                    atomicOr(block_args()->err, kErrOverlap);
                    continue;
                }
                if (TSP) {
                    if (nh < SP_SPRING_CAP) {
                        tj[nh] = (uint16_t)j;
                        tx[nh] = xi;
                    } else {
                        atomicOr(block_args()->err, kErrCapacity);
                    }
                    ++nh;
                }
                add_terms(Fx, Fy, T, cx, cy, ct);
                my_contacts += (gt < j) ? 1u : 0u;
            }
            if (TSP && (had || nh > 0))   // a floe out of contact before and now keeps its empty table
                for (int e = nh; e < SP_SPRING_CAP; ++e) {
                    tj[e] = 0xffffu;
                    tx[e] = 0.0;
                }
            // ---- update
            const double dt = a.dtd;
            const double und = uld + dt * (Fx * inv_m);
            const double vnd = vld + dt * (Fy * inv_m);
            const double wnd = wld + dt * (T * inv_i);
            int sx, sy;
            if (a.flags & SP_FORWARD_EULER) {
                sx = __double2int_rn(dt * uld * a.inv_qxd);
                sy = __double2int_rn(dt * vld * a.inv_qyd);
                th = (float)((double)th + dt * wld);
            } else {
                sx = __double2int_rn(dt * und * a.inv_qxd);
                sy = __double2int_rn(dt * vnd * a.inv_qyd);
                th = (float)((double)th + dt * wnd);
            }
            const float ddx = (float)sx * a.qx, ddy = (float)sy * a.qy;
            disp2 = ddx * ddx + ddy * ddy;   // squared: one root per cell below
            ufn = (float)und;
            vfn = (float)vnd;
            wfn = (float)wnd;
            pxn = px + (uint32_t)sx;
            pyn = py + (uint32_t)sy;
            if (!(isfinite(ufn) && isfinite(vfn) && isfinite(wfn))) atomicOr(block_args()->err, kErrNaN);
        }
        // ---- group reductions: row totals and displacement maxima into LDS
        {
            const double x = row_sum5(acc, gt & 15);
            const int l = gt & 15;
            if ((l & 1) == 0 && (l < 4 || l == 8 || l == 12 || l == 4))
                rows[par][l & 2 ? 4 : 2 * ((l >> 2) & 1) + (l >> 3)][gt >> 4] = x;
            const float wd = wave_max_nonneg(disp2);
            if ((gt & 63) == 0) wdisp[par][gt >> 6] = wd;
        }
        __syncthreads();                       // every lane is done with the floes' old state
        px = pxn;
        py = pyn;
        uf = ufn;
        vf = vfn;
        wf = wfn;
        if (has) {
            *reinterpret_cast<uint2*>(P + gt) = make_uint2(px, py);
            V[gt] = make_float4(uf, vf, wf, 0.0f);
        }
        __syncthreads();                       // the new state, the row totals and the maxima are in place
        {
            const float m = row_max_nonneg((gt & 63) < nw ? wdisp[par][gt & 63] : 0.0f);   // a scalar: nw <= 16
            vd = vnow + __builtin_amdgcn_sqrtf(m) * 1.0001f + 1e-3f;
        }
        // the step's statistics, by one wavefront of the group (in turn) while
        // the others go on: the row totals of each in order
        if ((gt >> 6) == turn && (gt & 63) < kRing) {
            const int st = gt & 63;
            const double2* const rt = reinterpret_cast<const double2*>(rows[par][st]);
            double x = 0.0;
#pragma unroll 2
            for (int q = 0; q < 2 * nw; ++q) {
                const double2 t = rt[q];
                x += t.x;
                x += t.y;
            }
            const BlockArgsPtr b = block_args();
            double* const mo = wk.w ? b->alt : b->ring + (size_t)step * kRing * b->ncells;
            mo[(size_t)st * b->ncells + c] = st < R_SVX ? x / (double)n : x;
        }
        turn = turn + 1 == nw ? 0 : turn + 1;
    }
    __syncthreads();                           // rows are scratch again

    unsigned long long* const totals = reinterpret_cast<unsigned long long*>(&rows[0][0][0]);   // [2][W]
    {
        const unsigned long long cs = wave_sum_u64(my_contacts);
        const unsigned long long ts = wave_sum_u64(my_tests);
        if ((gt & 63) == 0) {
            totals[gt >> 6] = cs;
            totals[W + (gt >> 6)] = ts;
        }
        __syncthreads();
        if (gt == 0) {
            const BlockArgsPtr b = block_args();
            unsigned long long ctot = 0, ttot = 0;
            for (int q = 0; q < nw; ++q) {
                ctot += totals[q];
                ttot += totals[W + q];
            }
            b->contacts[c] += ctot;
            b->cands[c] += ttot;
        }
        __syncthreads();
    }

    // ---- coarse-to-fine update of the cell (coupled cadence)
    if (block_args()->nd.x0m) {
        const BlockArgsPtr b = block_args();
        const double area = b->nd.area;
        const float r_lim = b->nd.r_lim;
        unsigned long long* const counters = b->nd.counters;
        double tg[4];
        {
            const double* st = b->nd.x0m + (size_t)c * kMomStride;
            const double inv_area = 1.0 / area;
            const double x0[4] = {st[M_MASS] * inv_area, st[M_PX] * inv_area, st[M_PY] * inv_area,
                                  st[M_L] * inv_area};
#pragma unroll
            for (int f = 0; f < 4; ++f) tg[f] = x0[f] + b->nd.frac * (b->nd.Q[(size_t)f * b->ncells + c] - x0[f]);
        }
        const bool ok = n > 0 && isfinite(tg[0]) && isfinite(tg[1]) && isfinite(tg[2]) &&
                        isfinite(tg[3]) && tg[0] > 0.0;
        if (!ok && gt == 0 && counters) atomicAdd(&counters[1], 1ull);
        const double hd = has ? (double)b->h[s + gt] : 0.0, rho = b->rho_ice_d;
        double (*const rw)[4 * W] = rows[0];
        const float ro = has ? rf : 0.0f;
        const double rod = ro;
        const double mass = group_sum_rows(has ? rho * hd * kPi * rod * rod : 0.0, rw[0], gt, nw);
        const float rmax = group_max(ro, wdisp[0], gt, nw);
        double sc = ok ? sqrt(tg[0] * area / mass) : 1.0;
        const bool clamped = ok && sc > (double)r_lim / (double)rmax;
        if (clamped) sc = (double)r_lim / (double)rmax;
        const float rn = (ok && has) ? fminf((float)(rod * sc), r_lim) : ro;
        const double rnd = rn;
        const double m = has ? rho * hd * kPi * rnd * rnd : 0.0;
        const double M = group_sum_rows(m, rw[1], gt, nw);
        const double Px = group_sum_rows(m * (double)uf, rw[2], gt, nw);
        const double Py = group_sum_rows(m * (double)vf, rw[3], gt, nw);
        const double L = group_sum_rows(m * rnd * rnd * (double)wf, rw[4], gt, nw);
        const double I = group_sum_rows(m * rnd * rnd, rw[5], gt, nw);
        const float gmax = group_max(has ? rn - ro : 0.0f, wdisp[0], gt, nw);
        if (ok && has) {
            const double dvx = (tg[1] * area - Px) / M;
            const double dvy = (tg[2] * area - Py) / M;
            const double dw = (tg[3] * area - L) / I;
            uf = (float)((double)uf + dvx);
            vf = (float)((double)vf + dvy);
            wf = (float)((double)wf + dw);
            b->r[s + gt] = rn;
        }
        if (ok && gt == 0) {
            if (gmax > 0.0f) vd = (vd + gmax * (1.0f + 0x1p-22f)) * (1.0f + 0x1p-22f);
            if (clamped && counters) atomicAdd(&counters[0], 1ull);
        }
    }

    // ---- state, lists and bound back to HBM
    const BlockArgsPtr b = block_args();
    if (has) {
        const int fi = s + gt;
        b->xi[fi] = px;
        b->yi[fi] = py;
        b->th[fi] = th;
        b->u[fi] = uf;
        b->v[fi] = vf;
        b->w[fi] = wf;
        if (TSP) {
            b->tsp_j[fi] = HJ[gt];
#pragma unroll
            for (int q = 0; q < SP_SPRING_CAP; ++q) b->tsp_x[(size_t)fi * SP_SPRING_CAP + q] = HX[gt * SP_SPRING_CAP + q];
        }
        if (rebuilt) {
            uint16_t* const vlst = b->vlist + (size_t)s * kListCap;
            for (int q = 0; q < k; ++q) vlst[(size_t)(q & ~7) * n + (size_t)gt * 8 + (q & 7)] = my[q];
            b->vcount[fi] = (uint8_t)k;
        }
    }
    if (gt == 0) b->vdisp[c] = vd;
}

}  // namespace spdem
