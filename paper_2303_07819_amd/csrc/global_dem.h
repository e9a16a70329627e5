// The global DEM of the paper's error study (Sec. 4): one DEM over the whole
// periodic domain, floes free to cross coarse cells, every pair a potential
// contact.  It is the reference ("truth") the superparameterised model is
// compared with; its coarse-grid statistics are read for that comparison.
// Included at the end of spdem.hip.
//
// Per fine step, two launches.  The re-binning (gpull_kernel) is a stable
// counting sort of the floes by sub-bin (side >= 2 r_max, so contacts only
// join neighbouring sub-bins): the counts per sub-bin and per sub-bin row are
// kept by the step's atomics, every row's wavefronts take their start from the
// row counts and their sub-bin starts by a scan, and every sub-bin gathers its
// floes in their current order from the 3 x 3 sub-bins around it (the state is
// grouped by the previous sub-bins and a floe moves far less than a sub-bin per
// step; a sub-bin that finds fewer floes than its count scans all floes
// instead).  The result is the order a stable sort by sub-bin gives.  Then one
// thread per floe (gstep_kernel) sweeps the 3 x 3 neighbouring sub-bins, decides
// contacts exactly as the cell kernel does (FP32 screen, FP64 in the guard
// band), sums drag and contact forces in FP64, writes the updated floe in the
// same order, and keeps the counts of the sub-bin of its new position for the
// next re-binning.  A floe's state is two 16-byte records and its angle.
#pragma once

namespace spdem {
struct GMode;
}

struct sp_gdem {
    sp_gdem_params p;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    std::string err;

    double u0 = 0, v0 = 0;
    int nmodes = 0;
    double kx[SP_MAX_MODES], ky[SP_MAX_MODES], au[SP_MAX_MODES], av[SP_MAX_MODES], ph[SP_MAX_MODES];
    bool phase_dirty = true;

    int64_t n = 0;
    bool have_floes = false;
    int nbx = 1, nby = 1;
    float rmax = 0.0f;
    // floe state, two buffers; cur holds the state in sub-bin order
    uint4* P[2] = {nullptr, nullptr};      // xi, yi, r, id
    float4* V[2] = {nullptr, nullptr};     // u, v, w, h
    float* th[2] = {nullptr, nullptr};
    int cur = 0;
    // re-binning: the sub-bin of every floe's position (order of buffer cur),
    // floes per sub-bin and per sub-bin row of those, sub-bin starts
    int32_t* key = nullptr;            // [n]
    int32_t* bcount = nullptr;         // [nb]
    int32_t* rcount = nullptr;         // [nby]
    int32_t* starts[2] = {nullptr, nullptr};   // [nb + 1]
    int sb = 0;                        // starts[sb] groups buffer cur
    unsigned long long* fallbacks_d = nullptr;  // sub-bins (and coarse cells) gathered by a full scan
    // coarse read-out: coarse cell of every floe, counts, starts, floes in cell order
    int32_t* ckey = nullptr;           // [n]
    int32_t* perm = nullptr;           // [n]
    int32_t* ccount = nullptr;         // [ncoarse]
    int32_t* crow = nullptr;           // [nyc]
    size_t ccount_cap = 0, crow_cap = 0;
    int32_t* cstart = nullptr;         // coarse-cell starts (read-out)
    size_t cstart_cap = 0;
    double* cmom = nullptr;            // coarse statistics (read-out)
    size_t cmom_cap = 0;
    spdem::GMode* modes = nullptr;     // [SP_MAX_MODES]
    double2* phase = nullptr;          // (sin, cos) of every mode's phase at each sub-bin centre
    uint32_t* err_d = nullptr;
    unsigned long long* contacts_d = nullptr;   // [kContactSlots x kContactStride], their sum counts
    int64_t steps = 0;
    Staging staging;                   // read-outs
    std::mutex reads;                  // held by the read-outs that use the other buffer or the coarse arrays as scratch
};

namespace spdem {

// Contact counters: workgroup i adds to slot i modulo kContactSlots, a cache
// line each (adds to one address from all over the chip take 8 ns apiece).
constexpr int kContactSlots = 64;
constexpr int kContactStride = 16;
constexpr size_t kContactBytes = (size_t)kContactSlots * kContactStride * sizeof(unsigned long long);

// Constants of a mode, read through the scalar cache (kernel arguments lie in
// host memory: their cache lines cost a trip over the bus each).
struct GMode {
    float kxL, kyL;                    // phase per sub-bin side
    double au, av, cz;                 // amplitudes and curl coefficient av kx - au ky
};
typedef double GModeWords __attribute__((ext_vector_type(4)));
typedef const GModeWords __attribute__((address_space(4)))* GModeTable;
static_assert(sizeof(GMode) == sizeof(GModeWords), "a mode's constants are one vector of the table");

struct GArgs {
    // pre-step state in sub-bin order
    const uint4* P;                    // xi, yi, r, id
    const float4* V;                   // u, v, w, h
    const float* th;
    // updated state, same order
    uint4* Po;
    float4* Vo;
    float* tho;
    const int32_t* bstart;
    const double2* phase;
    const GMode* modes;                // [nmodes]
    int n, nbx, nby, nmodes;
    int direct;                        // every phase offset is <= 1.6
    uint32_t flags;
    float qx, qy;
    double u0, v0;
    double lxd;                        // domain length in x (position of the far wall with SP_WALL_X)
    double qxd, qyd, inv_qxd, inv_qyd;
    double dtd, Ed, Gd, mud, cdrho, rho_ice_d;
    uint32_t* err;
    unsigned long long* contacts;
    // the sub-bin of every updated position; floes per sub-bin and per row,
    // corrected for the floes that changed theirs
    int32_t* key_out;
    int32_t* count;
    int32_t* rows;
};

constexpr uint32_t kErrRebin = 32u;    // a re-binning gathered another number of floes than it counted

__device__ __forceinline__ uint32_t gbin_axis(uint32_t x, int nb)
{
    return (uint32_t)(((uint64_t)x * (uint64_t)nb) >> 32);
}

// Offset of a fixed-point coordinate from its sub-bin centre, in sub-bin sides.
__device__ __forceinline__ float gbin_offset(uint32_t x, int nb)
{
    const uint32_t lo = (uint32_t)((uint64_t)x * (uint64_t)nb);
    return (float)(int)(lo - 0x80000000u) * 2.3283064365386963e-10f;
}

// The axis indices lo - 1 .. hi + 1 modulo n as at most two ascending,
// disjoint segments [a0, a1] and [b0, b1] (b0 > b1: none), the first below
// the second; all of 0 .. n - 1 when they cover the axis.
struct Segs {
    int a0, a1, b0, b1;
};

__device__ __forceinline__ Segs wrap_segments(int lo, int hi, int n)
{
    if (hi - lo + 3 >= n) return Segs{0, n - 1, 1, 0};
    const int s = lo - 1, e = hi + 1;
    if (s < 0) return Segs{0, e, s + n, n - 1};
    if (e >= n) return Segs{0, e - n, s, n - 1};
    return Segs{s, e, 1, 0};
}

// Sum over the wavefront (every lane gets it) and exclusive prefix over its lanes.
__device__ __forceinline__ int wave_sum_i32(int x)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

__device__ __forceinline__ int wave_exclusive_i32(int x)
{
    const int lane = threadIdx.x & 63;
    int incl = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    return incl - x;
}

// Up to six position ranges [lo, hi) as one sequence: element t of it is
// position t + (the offset of its range).
struct Ranges {
    int o0, o1, o2, o3, o4, o5;   // offsets
    int e0, e1, e2, e3, e4;       // elements up to the end of each range
    int total;
};

__device__ __forceinline__ Ranges make_ranges(int l0, int h0, int l1, int h1, int l2, int h2, int l3, int h3, int l4,
                                              int h4, int l5, int h5)
{
    Ranges r;
    r.e0 = h0 - l0;
    r.e1 = r.e0 + (h1 - l1);
    r.e2 = r.e1 + (h2 - l2);
    r.e3 = r.e2 + (h3 - l3);
    r.e4 = r.e3 + (h4 - l4);
    r.total = r.e4 + (h5 - l5);
    r.o0 = l0;
    r.o1 = l1 - r.e0;
    r.o2 = l2 - r.e1;
    r.o3 = l3 - r.e2;
    r.o4 = l4 - r.e3;
    r.o5 = l5 - r.e4;
    return r;
}

__device__ __forceinline__ int range_position(const Ranges& r, int t)
{
    // every field read first: a read under a condition would keep r in memory
    const int o1 = r.o1, o2 = r.o2, o3 = r.o3, o4 = r.o4, o5 = r.o5;
    const int e0 = r.e0, e1 = r.e1, e2 = r.e2, e3 = r.e3, e4 = r.e4;
    int at = r.o0;
    at = t >= e0 ? o1 : at;
    at = t >= e1 ? o2 : at;
    at = t >= e2 ? o3 : at;
    at = t >= e3 ? o4 : at;
    at = t >= e4 ? o5 : at;
    return t + at;
}

struct GPull {
    // buffer cur, grouped by ostart -> buffer out, grouped by nstart
    const uint4* P;
    const float4* V;
    const float* th;
    uint4* Po;
    float4* Vo;
    float* tho;
    const int32_t* key;        // [n] sub-bin of every floe of buffer cur
    const int32_t* ostart;     // [nb + 1]
    int32_t* nstart;           // [nb + 1]
    const int32_t* count;      // [nb] floes per sub-bin of key
    const int32_t* rows;       // [nby] floes per sub-bin row of key
    int n, nbx, nby;
    uint32_t* err;
    unsigned long long* fallbacks;
};

// Sum of v[lane], v[lane + 64], ... below n, 4 loads in flight.
__device__ __forceinline__ int strided_sum(const int32_t* v, int n, int lane)
{
    int part = 0;
    for (int i = lane; i < n; i += 256) {
        int x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = i + 64 * e < n ? v[i + 64 * e] : 0;
        part += (x[0] + x[1]) + (x[2] + x[3]);
    }
    return part;
}

// Neighbours read together per round (a floe has 9 in its 3 x 3 sub-bins on
// average in the error study's scenarios: one round for most wavefronts).
constexpr int kGBatch = 12;

// Re-binning: one wavefront per run of 64 sub-bins of a row, one lane per
// sub-bin.  A run starts after the floes of the rows before it and of its
// row's earlier sub-bins.  A chain of dependent reads bounds it (115,200 floes
// are two wavefronts per SIMD), so reads that do not depend on each other are
// made together: the bounds of all neighbour ranges, the keys of a round of
// neighbours, and the state of the floes found (a sub-bin holds one or two)
// after the search instead of at each find; 32-byte packed state.  115,200
// floes: 13.9 us before, 9.5 now.
__global__ __launch_bounds__(256) void gpull_kernel(GPull g)
{
    const int lane = threadIdx.x & 63;
    const int wid = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    const int runs = (g.nbx + 63) >> 6;
    if (wid >= g.nby * runs) return;          // whole wavefronts
    const int by = wid / runs, c0 = (wid % runs) * 64;
    const int bx = c0 + lane;
    const bool in = bx < g.nbx;
    const int b = by * g.nbx + bx;
    // the (at most 3 x 2) position ranges of the neighbouring sub-bins in
    // ascending order: rows y0 < y1 < y2, each one or two ranges
    const int nrow = min(g.nby, 3);
    const int y0 = g.nby <= 3 || by == 0 || by == g.nby - 1 ? 0 : by - 1;
    const int y1 = g.nby <= 3 || by == 0 ? 1 : by == g.nby - 1 ? g.nby - 2 : by;
    const int y2 = g.nby <= 3 ? 2 : by == 0 ? g.nby - 1 : by == g.nby - 1 ? by : by + 1;
    const Segs rx = wrap_segments(in ? bx : 0, in ? bx : 0, g.nbx);
    const bool two = rx.b0 <= rx.b1;
    const int32_t *s0 = g.ostart + y0 * g.nbx, *s1 = g.ostart + y1 * g.nbx, *s2 = g.ostart + y2 * g.nbx;
    const bool u1 = nrow > 1, u2 = nrow > 2;
    const int xa = rx.a0, xb = rx.a1 + 1, xc = two ? rx.b0 : xa, xd = two ? rx.b1 + 1 : xa;
    const Ranges rg = make_ranges(s0[xa], s0[xb], s0[xc], s0[xd], u1 ? s1[xa] : 0, u1 ? s1[xb] : 0, u1 ? s1[xc] : 0,
                                  u1 ? s1[xd] : 0, u2 ? s2[xa] : 0, u2 ? s2[xb] : 0, u2 ? s2[xc] : 0, u2 ? s2[xd] : 0);
    const int cnt = in ? g.count[b] : 0;
    const int base = wave_sum_i32(strided_sum(g.rows, by, lane) + strided_sum(g.count + by * g.nbx, c0, lane));
    const int q0 = base + wave_exclusive_i32(cnt);
    if (wid == g.nby * runs - 1 && lane == 63) g.nstart[g.nbx * g.nby] = g.n;
    if (!in) return;
    g.nstart[b] = q0;
    int i = 0;
    int m0 = 0, m1 = 0, m2 = 0, m3 = 0;   // the first four floes found
    auto take = [&](int p) {
        if (i == 0) m0 = p;
        if (i == 1) m1 = p;
        if (i == 2) m2 = p;
        if (i == 3) m3 = p;
        if (i >= 4 && i < cnt) {
            const int q = q0 + i;
            g.Po[q] = g.P[p];
            g.Vo[q] = g.V[p];
            g.tho[q] = g.th[p];
        }
        ++i;
    };
    for (int t0 = 0; t0 < rg.total; t0 += kGBatch) {
        uint32_t mine = 0;
#pragma unroll
        for (int e = 0; e < kGBatch; ++e) {
            const bool is = t0 + e < rg.total && g.key[range_position(rg, t0 + e)] == b;
            mine |= (is ? 1u : 0u) << e;
        }
        for (; mine; mine &= mine - 1) take(range_position(rg, t0 + __builtin_ctz(mine)));
    }
    if (i != cnt) {   // a floe came from further away: every floe, in order
        atomicAdd(g.fallbacks, 1ull);
        i = 0;
#pragma unroll 1
        for (int p = 0; p < g.n; ++p)
            if (g.key[p] == b) take(p);
        if (i != cnt) atomicOr(g.err, kErrRebin);
    }
    const int got = min(i, cnt);
    const bool h0 = got > 0, h1 = got > 1, h2 = got > 2, h3 = got > 3;
    uint4 P0, P1, P2, P3;
    float4 V0, V1, V2, V3;
    float t0, t1, t2, t3;
#define GPULL_GET(e) \
    if (h##e) {      \
        P##e = g.P[m##e]; \
        V##e = g.V[m##e]; \
        t##e = g.th[m##e]; \
    }
#define GPULL_PUT(e) \
    if (h##e) {      \
        g.Po[q0 + e] = P##e; \
        g.Vo[q0 + e] = V##e; \
        g.tho[q0 + e] = t##e; \
    }
    GPULL_GET(0) GPULL_GET(1) GPULL_GET(2) GPULL_GET(3)
    GPULL_PUT(0) GPULL_PUT(1) GPULL_PUT(2) GPULL_PUT(3)
#undef GPULL_GET
#undef GPULL_PUT
}

// Ocean current and curl at a floe from the phase table of its sub-bin: the
// offset's sin and cos in FP32, the angle addition and the sum over modes in
// FP64 (as the cell kernels).
__device__ __forceinline__ void gocean(const GArgs& a, uint32_t x, uint32_t y, double& uo, double& vo, double& zeta)
{
    uo = a.u0;
    vo = a.v0;
    zeta = 0.0;
    if (a.nmodes == 0) return;
    const int b = (int)(gbin_axis(y, a.nby) * (uint32_t)a.nbx + gbin_axis(x, a.nbx));
    const float fx = gbin_offset(x, a.nbx), fy = gbin_offset(y, a.nby);
    const double2* ph = a.phase + (size_t)b * a.nmodes;
    GModeTable table = (GModeTable)a.modes;
    double2 next = ph[0];
    for (int m = 0; m < a.nmodes; ++m) {
        const double2 q = next;
        if (m + 1 < a.nmodes) next = ph[m + 1];
        const GModeWords c = table[m];
        const float kxL = __int_as_float(__double2loint(c[0])), kyL = __int_as_float(__double2hiint(c[0]));
        const float d = kxL * fx + kyL * fy;
        float sdf, cdf;
        if (a.direct)
            sincos_direct(d, sdf, cdf);
        else
            sincos_small(d, sdf, cdf);
        const double sd = sdf, cd = cdf;
        const double sn = fma(q.x, cd, q.y * sd);
        const double cn = fma(q.y, cd, -(q.x * sd));
        uo = fma(c[1], sn, uo);
        vo = fma(c[2], sn, vo);
        zeta = fma(c[3], cn, zeta);
    }
}

// Drag force and drag torque of a floe (FP64), as in the cell kernel.
__device__ __forceinline__ void gdrag(const GArgs& a, uint32_t x, uint32_t y, double rld, double uld, double vld,
                                      double wld, double& fdx, double& fdy, double& tdr)
{
    fdx = fdy = tdr = 0.0;
    if (a.flags & SP_OCEAN_OFF) return;
    double uo, vo, zeta;
    gocean(a, x, y, uo, vo, zeta);
    const double du = uo - uld, dv = vo - vld;
    const double sp = sqrt(du * du + dv * dv);
    const double alpha = a.cdrho * kPi * rld * rld;
    fdx = alpha * du * sp;
    fdy = alpha * dv * sp;
    const double dW = 0.5 * zeta - wld;
    const double r2 = rld * rld;
    const double beta = a.cdrho * kPi * r2 * r2 * rld;
    tdr = beta * dW * fabs(dW);
}

// One thread per floe.  Bound by its chain of dependent reads (115,200 floes
// are two wavefronts per SIMD): own state, bounds of the candidate ranges (the
// three sub-bins of a row are consecutive, two ranges where they wrap), the
// candidates' positions and radii as one 16-byte read each and a round at a
// time, then the velocity of those in contact, the next one's read before the
// current one's force.  Candidates are decided and their forces summed in the
// order sub-bin row, sub-bin, position.  Sub-bin and row counts are corrected
// only for floes that changed theirs: adding every floe to its counter, and
// every wavefront to one contact counter, cost as much as the contacts.  115,200
// floes and two modes: 29.5 us before, 10.2 now.
__global__ __launch_bounds__(256) void gstep_kernel(GArgs a)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long ncontact = 0;
    if (k < a.n) {
        const uint4 own = a.P[k];
        const float4 vo = a.V[k];
        const float thl = a.th[k];
        const uint32_t xl = own.x, yl = own.y;
        const float rl = __uint_as_float(own.z);
        const int idl = (int)own.w;
        const double rld = rl, uld = vo.x, vld = vo.y, wld = vo.z;
        const int bx = (int)gbin_axis(xl, a.nbx), by = (int)gbin_axis(yl, a.nby);
        const bool wall = (a.flags & SP_WALL_X) != 0;
        // columns of the neighbouring sub-bins in visiting order: [ca, cb) and,
        // across the domain's edge, [0, cc1)
        int ca = bx - 1, cb = bx + 2, cc1 = 0;
        if (a.nbx < 3) {
            ca = bx;
            cb = bx + 1;
        } else if (bx == 0) {
            if (wall) {
                ca = 0;
            } else {
                ca = a.nbx - 1;
                cb = a.nbx;
                cc1 = 2;
            }
        } else if (bx == a.nbx - 1) {
            cb = a.nbx;
            cc1 = wall ? 0 : 1;
        }
        const int y0 = by == 0 ? a.nby - 1 : by - 1, y2 = by == a.nby - 1 ? 0 : by + 1;
        const bool rows3 = a.nby >= 3;
        const int32_t *s0 = a.bstart + (rows3 ? y0 : by) * a.nbx, *s1 = a.bstart + by * a.nbx,
                      *s2 = a.bstart + (rows3 ? y2 : by) * a.nbx;
        const int l0 = s0[ca], h0 = s0[cb], l1 = s1[ca], h1 = s1[cb], l2 = s2[ca], h2 = s2[cb];
        int m0 = 0, n0 = 0, m1 = 0, n1 = 0, m2 = 0, n2 = 0;
        if (cc1 > 0) {
            m0 = s0[0];
            n0 = s0[cc1];
            m1 = s1[0];
            n1 = s1[cc1];
            m2 = s2[0];
            n2 = s2[cc1];
        }
        const Ranges rg = make_ranges(l0, rows3 ? h0 : l0, m0, rows3 ? n0 : m0, l1, h1, m1, n1, l2, rows3 ? h2 : l2, m2,
                                      rows3 ? n2 : m2);
        double Fx, Fy, T;
        gdrag(a, xl, yl, rld, uld, vld, wld, Fx, Fy, T);
        const double md = a.rho_ice_d * (double)vo.w * kPi * rld * rld;
        for (int t0 = 0; t0 < rg.total; t0 += kGBatch) {
            uint4 c[kGBatch];
            int jj[kGBatch];
#pragma unroll
            for (int e = 0; e < kGBatch; ++e) {
                jj[e] = t0 + e < rg.total ? range_position(rg, t0 + e) : k;   // the floe itself stands for none
                c[e] = a.P[jj[e]];
            }
            uint32_t hits = 0;
#pragma unroll
            for (int e = 0; e < kGBatch; ++e) {
                // between walls the x difference is the plain one (pairs
                // more than half the domain apart are far from contact)
                const long long ddx = (long long)c[e].x - (long long)xl;
                const bool apart = wall && (ddx >= 0x80000000ll || ddx < -0x80000000ll);
                const int dxi = (int)(c[e].x - xl), dyi = (int)(c[e].y - yl);
                const float rj = __uint_as_float(c[e].z);
                float diff, R2;
                screen(dxi, dyi, rl, rj, a.qx, a.qy, diff, R2);
                if (!(diff > kGuard * R2) && !apart && jj[e] != k) hits |= 1u << e;
            }
            uint4 nxt;
            float4 nv;
            if (hits) {
                const int j = range_position(rg, t0 + __builtin_ctz(hits));
                nxt = a.P[j];
                nv = a.V[j];
            }
            while (hits) {
                const uint4 cur = nxt;
                const float4 vj = nv;
                hits &= hits - 1;
                if (hits) {
                    const int j = range_position(rg, t0 + __builtin_ctz(hits));
                    nxt = a.P[j];
                    nv = a.V[j];
                }
                const int dxi = (int)(cur.x - xl), dyi = (int)(cur.y - yl);
                const float rj = __uint_as_float(cur.z);
                float diff, R2;
                screen(dxi, dyi, rl, rj, a.qx, a.qy, diff, R2);
                if (fabsf(diff) <= kGuard * R2 && !exact_contact(dxi, dyi, rl, rj, a.qxd, a.qyd)) continue;
                const double dx = (double)dxi * a.qxd, dy = (double)dyi * a.qyd;
                const double d2 = dx * dx + dy * dy;
                if (!(d2 > 0.0)) {
                    atomicOr(a.err, kErrOverlap);
                    continue;
                }
                const int idj = (int)cur.w;
                const double rjd = (double)rj;
                const double d = sqrt(d2);
                const double inv_d = 1.0 / d;
                const double nx = dx * inv_d, ny = dy * inv_d;
                const double tx = -ny, ty = nx;
                const double R = rld + rjd;
                const double delta = d - R;
                const double dr = fabs(rld - rjd);
                double cc;
                if (d <= dr) {
                    cc = 2.0 * fmin(rld, rjd);
                } else {
                    const double p = (((-delta) * (d + R)) * (d - dr)) * (d + dr);
                    cc = sqrt(fmax(p, 0.0)) * inv_d;
                }
                const double Fn = cc * a.Ed * delta;
                const double wjd = (double)vj.z;
                // spin sum with the lower floe id first: exactly antisymmetric pair forces
                const double spin = (idl < idj) ? (wld * rld + wjd * rjd) : (wjd * rjd + wld * rld);
                const double vt = (((double)vj.x - uld) * tx + ((double)vj.y - vld) * ty) - spin;
                const double capf = a.mud * fabs(Fn);
                const double Ft = fmin(fmax(cc * a.Gd * vt, -capf), capf);
                Fx += Fn * nx + Ft * tx;
                Fy += Fn * ny + Ft * ty;
                T += rld * Ft;
                ncontact += (idl < idj) ? 1ull : 0ull;
            }
        }
        if (wall) {
            // the walls at x = 0 and x = lx, after the floe contacts: the
            // contact law with a fixed body, in contact iff the centre's
            // distance d to the wall is below r
            const double dw[2] = {(double)xl * a.qxd, (double)(0x100000000ull - (unsigned long long)xl) * a.qxd};
            const double sgn[2] = {-1.0, 1.0};
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const double d = dw[q];
                if (!(d < rld)) continue;
                const double cc = 2.0 * sqrt(fmax(rld * rld - d * d, 0.0));
                const double Fn = cc * a.Ed * (d - rld);
                const double vt = -(vld * sgn[q]) - wld * rld;     // t = (0, sgn): -v.t - w r
                const double capf = a.mud * fabs(Fn);
                const double Ft = fmin(fmax(cc * a.Gd * vt, -capf), capf);
                Fx += Fn * sgn[q];
                Fy += Ft * sgn[q];
                T += rld * Ft;
                ncontact += 1ull;
            }
        }
        // semi-implicit Euler (positions with the new velocities) unless forward Euler
        const double inv_m = 1.0 / md;
        const double dt = a.dtd;
        const double und = uld + dt * (Fx * inv_m);
        const double vnd = vld + dt * (Fy * inv_m);
        const double wnd = wld + dt * (T * inv_m / (rld * rld));
        const bool fe = (a.flags & SP_FORWARD_EULER) != 0;
        const double ux = fe ? uld : und, vx = fe ? vld : vnd, wx = fe ? wld : wnd;
        const int sx = __double2int_rn(dt * ux * a.inv_qxd);
        const int sy = __double2int_rn(dt * vx * a.inv_qyd);
        const float un = (float)und, vn = (float)vnd, wn = (float)wnd;
        if (wall) {
            const long long xn = (long long)xl + sx;
            if (xn < 0 || xn >= 0x100000000ll) atomicOr(a.err, kErrWall);
        }
        const uint32_t xn = xl + (uint32_t)sx, yn = yl + (uint32_t)sy;
        a.Po[k] = make_uint4(xn, yn, own.z, own.w);
        a.Vo[k] = make_float4(un, vn, wn, vo.w);
        a.tho[k] = (float)((double)thl + dt * wx);
        {
            const int row = (int)gbin_axis(yn, a.nby);
            const int b = row * a.nbx + (int)gbin_axis(xn, a.nbx), b0 = by * a.nbx + bx;
            a.key_out[k] = b;
            if (b != b0) {
                atomicAdd(&a.count[b], 1);
                atomicSub(&a.count[b0], 1);
            }
            if (row != by) {
                atomicAdd(&a.rows[row], 1);
                atomicSub(&a.rows[by], 1);
            }
        }
        if (!(isfinite(un) && isfinite(vn) && isfinite(wn))) atomicOr(a.err, kErrNaN);
    }
    const unsigned long long cs = wave_sum_u64(ncontact);
    if ((threadIdx.x & 63) == 0 && cs)
        atomicAdd(&a.contacts[(blockIdx.x % kContactSlots) * kContactStride], cs);
}

// Coarse cell of every floe of buffer cur (read-out), counted per cell and per
// row: consecutive floes mostly share both (the order is by sub-bin), so a run
// of lanes with one cell or row is one atomic.  115,200 floes onto 48 x 24
// cells: 16 us; every floe adding to its cell's and row's counters took 932.
__device__ __forceinline__ void count_runs(int32_t* counts, int c, bool valid)
{
    const int lane = threadIdx.x & 63;
    const int prev = __shfl_up(c, 1, 64);
    const unsigned long long live = __ballot(valid);                   // lanes 0 .. l - 1
    const unsigned long long heads = __ballot(valid && (lane == 0 || c != prev));
    if (!((heads >> lane) & 1ull)) return;
    const unsigned long long after = lane == 63 ? 0ull : heads >> (lane + 1);
    const int next = after ? lane + 1 + __builtin_ctzll(after) : __popcll(live);
    atomicAdd(&counts[c], next - lane);
}

__global__ __launch_bounds__(256) void ckey_kernel(const uint4* P, int n, int nxc, int nyc, int32_t* ckey,
                                                   int32_t* ccount, int32_t* crow)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = k < n;
    int c = -1, cy = -1;
    if (valid) {
        const uint4 p = P[k];
        cy = (int)gbin_axis(p.y, nyc);
        c = cy * nxc + (int)gbin_axis(p.x, nxc);
        ckey[k] = c;
    }
    count_runs(ccount, c, valid);
    count_runs(crow, cy, valid);
}

// The floes of every coarse cell in the current order (perm, from cstart): a
// stable counting sort as the re-binning, one workgroup per `run` cells of a
// coarse row.  A run starts after the floes of the rows before it and of its
// row's earlier cells; each wavefront gathers its cells' floes in order (ballot
// and prefix count) from the sub-bins a cell overlaps, one more on every side
// (the grouping is that of the last re-binning, the positions a step later); a
// cell that finds fewer floes than its count scans all floes instead.  Runs of
// 4, a cell per wavefront, while the grid is small enough for the sums before a
// run to cost nothing (48 x 24 cells: 15.5 us, a workgroup per row 89), of 64
// above.  A whole read-out of 100,000 floes with runs of 4 and of 64: 128 x 128
// cells 197 and 223 us, 256 x 128 326 and 346, 256 x 256 631 and 624, 512 x 256
// 1153 and 1133.
constexpr int kCoarseRun = 4, kCoarseRunLarge = 64, kCoarseSmall = 1 << 16;

__global__ __launch_bounds__(256) void cpull_kernel(const int32_t* ckey, const int32_t* ccount, const int32_t* crow,
                                                    const int32_t* ostart, int n, int nbx, int nby, int nxc,
                                                    int nyc, int run, int32_t* cstart, int32_t* perm, uint32_t* err,
                                                    unsigned long long* fallbacks)
{
    const int runs = (nxc + run - 1) / run;
    const int cy = blockIdx.x / runs, c0 = (blockIdx.x % runs) * run;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int here = min(run, nxc - c0);   // cells of the run, at most one per lane
    const int own = lane < here ? ccount[cy * nxc + c0 + lane] : 0;
    const int base = wave_sum_i32(strided_sum(crow, cy, lane) + strided_sum(ccount + cy * nxc, c0, lane));
    const int first = base + wave_exclusive_i32(own);   // start of the lane's cell
    if (wave == 0 && lane < here) cstart[cy * nxc + c0 + lane] = first;
    if (threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) cstart[nxc * nyc] = n;
    // sub-bin rows and columns a coarse cell overlaps
    const int ylo = (int)(((long long)cy * nby) / nyc), yhi = (int)(((long long)(cy + 1) * nby - 1) / nyc);
    for (int l = wave; l < here; l += 4) {
        const int cx = c0 + l, c = cy * nxc + cx;
        const int q0 = __shfl(first, l), cnt = __shfl(own, l);
        const int xlo = (int)(((long long)cx * nbx) / nxc), xhi = (int)(((long long)(cx + 1) * nbx - 1) / nxc);
        int i = 0;   // floes of c gathered so far (the same in every lane)
        auto chunk = [&](int p0, int p1) {   // positions [p0, p1), 64 at a time, in order
            for (int b = p0; b < p1; b += 64) {
                const int p = b + lane;
                const bool hit = p < p1 && ckey[p] == c;
                const unsigned long long m = __ballot(hit);
                const int before = __popcll(m & ((1ull << lane) - 1ull));
                if (hit && i + before < cnt) perm[q0 + i + before] = p;
                i += __popcll(m);
            }
        };
        const Segs ry = wrap_segments(ylo, yhi, nby), rx = wrap_segments(xlo, xhi, nbx);
        const int ys[4] = {ry.a0, ry.a1, ry.b0, ry.b1};
        const int xs[4] = {rx.a0, rx.a1, rx.b0, rx.b1};
        for (int sy = 0; sy < 2; ++sy)
            for (int yy = ys[2 * sy]; yy <= ys[2 * sy + 1]; ++yy)
                for (int sx = 0; sx < 2; ++sx)
                    if (xs[2 * sx] <= xs[2 * sx + 1])
                        chunk(ostart[yy * nbx + xs[2 * sx]], ostart[yy * nbx + xs[2 * sx + 1] + 1]);
        if (i != cnt) {
            if (lane == 0) atomicAdd(fallbacks, 1ull);
            i = 0;
            chunk(0, n);
            if (i != cnt && lane == 0) atomicOr(err, kErrRebin);
        }
    }
}

// The 11 statistics of every coarse cell, one wavefront per cell over its
// floes in sorted order (fixed summation order).
__global__ __launch_bounds__(64) void cmom_kernel(GArgs a, const int32_t* perm, const int32_t* cstart, int ncoarse,
                                                  double* out)
{
    const int c = blockIdx.x;
    if (c >= ncoarse) return;
    const int lane = threadIdx.x;
    double acc[SP_NMOM];
#pragma unroll
    for (int q = 0; q < SP_NMOM; ++q) acc[q] = 0.0;
    for (int i = cstart[c] + lane; i < cstart[c + 1]; i += 64) {
        const int k = perm[i];
        const uint4 p = a.P[k];
        const float4 f = a.V[k];
        const uint32_t x = p.x, y = p.y;
        const double rl = __uint_as_float(p.z), ul = f.x, vl = f.y, wl = f.z;
        const double m = a.rho_ice_d * (double)f.w * kPi * rl * rl;
        double fdx, fdy, tdr;
        gdrag(a, x, y, rl, ul, vl, wl, fdx, fdy, tdr);
        acc[M_N] += 1.0;
        acc[M_MASS] += m;
        acc[M_PX] += m * ul;
        acc[M_PY] += m * vl;
        acc[M_L] += m * rl * rl * wl;
        acc[M_UX] += ul;
        acc[M_UY] += vl;
        acc[M_SVX] += fdx;
        acc[M_SVY] += fdy;
        acc[M_SW] += tdr;
        acc[M_AICE] += kPi * rl * rl;
    }
#pragma unroll
    for (int q = 0; q < SP_NMOM; ++q) {
        double x = acc[q];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
        if (lane == 0) out[(size_t)c * SP_NMOM + q] = x;
    }
}

// Scatter the state back into input order (read-out).
__global__ __launch_bounds__(256) void gscatter_kernel(int n, const uint4* P, const float4* V, const float* th,
                                                       uint32_t* xo, uint32_t* yo, float* uo, float* vo, float* wo,
                                                       float* tho, float* ro)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const uint4 q = P[k];
    const float4 f = V[k];
    const int p = (int)q.w;
    xo[p] = q.x;
    yo[p] = q.y;
    uo[p] = f.x;
    vo[p] = f.y;
    wo[p] = f.z;
    tho[p] = th[k];
    ro[p] = __uint_as_float(q.z);
}

// The floe ids in the current order (read-out).
__global__ __launch_bounds__(256) void gids_kernel(int n, const uint4* P, int32_t* id)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) id[k] = (int)P[k].w;
}

}  // namespace spdem

namespace {

sp_status gfail(sp_gdem* g, sp_status st, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (g) g->err = buf;
    return st;
}

#define GD_TRY(g, expr)                                                                        \
    do {                                                                                       \
        hipError_t e_ = (expr);                                                                \
        if (e_ != hipSuccess) {                                                                \
            (void)hipGetLastError();                                                           \
            return gfail((g), SP_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_));             \
        }                                                                                      \
    } while (0)

template <class T>
sp_status galloc(sp_gdem* g, T** p, size_t count)
{
    if (*p) (void)hipFree(*p);
    *p = nullptr;
    if (hipMalloc((void**)p, std::max<size_t>(1, count) * sizeof(T)) != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        return gfail(g, SP_ENOMEM, "device allocation of %zu bytes failed", count * sizeof(T));
    }
    return SP_OK;
}

void gdem_free(sp_gdem* g)
{
    for (int b = 0; b < 2; ++b) {
        void* ps[] = {g->P[b], g->V[b], g->th[b], g->starts[b]};
        for (void* p : ps)
            if (p) (void)hipFree(p);
        g->P[b] = nullptr;
        g->V[b] = nullptr;
        g->th[b] = nullptr;
        g->starts[b] = nullptr;
    }
    void* ps[] = {g->key, g->bcount, g->rcount, g->ckey, g->perm, g->ccount, g->crow, g->cstart, g->cmom, g->modes, g->phase, g->err_d,
                  g->contacts_d, g->fallbacks_d};
    for (void* p : ps)
        if (p) (void)hipFree(p);
    g->key = g->bcount = g->rcount = g->ckey = g->perm = g->ccount = g->crow = g->cstart = nullptr;
    g->cmom = nullptr;
    g->modes = nullptr;
    g->phase = nullptr;
    g->err_d = nullptr;
    g->contacts_d = nullptr;
    g->fallbacks_d = nullptr;
    g->ccount_cap = g->crow_cap = g->cstart_cap = g->cmom_cap = 0;
}

GArgs gargs(const sp_gdem* g, double dt, int from, int to)
{
    GArgs a;
    memset(&a, 0, sizeof a);
    a.P = g->P[from];
    a.V = g->V[from];
    a.th = g->th[from];
    a.Po = g->P[to];
    a.Vo = g->V[to];
    a.tho = g->th[to];
    a.bstart = g->starts[g->sb ^ 1];   // the starts the re-binning before the step makes
    a.key_out = g->key;
    a.count = g->bcount;
    a.rows = g->rcount;
    a.phase = g->phase;
    a.n = (int)g->n;
    a.nbx = g->nbx;
    a.nby = g->nby;
    a.nmodes = g->nmodes;
    a.flags = g->p.flags;
    a.qxd = g->p.lx / 4294967296.0;
    a.qyd = g->p.ly / 4294967296.0;
    a.qx = (float)a.qxd;
    a.qy = (float)a.qyd;
    a.inv_qxd = 1.0 / a.qxd;
    a.inv_qyd = 1.0 / a.qyd;
    a.dtd = dt;
    a.Ed = g->p.E;
    a.Gd = g->p.G;
    a.mud = g->p.mu;
    a.cdrho = g->p.cd * g->p.rho_ocean;
    a.rho_ice_d = g->p.rho_ice;
    a.u0 = g->u0;
    a.v0 = g->v0;
    a.lxd = g->p.lx;
    const double bx = g->p.lx / g->nbx, by = g->p.ly / g->nby;
    float reach = 0.0f;
    for (int m = 0; m < g->nmodes; ++m)
        reach = std::max(reach, 0.5f * (fabsf((float)(g->kx[m] * bx)) + fabsf((float)(g->ky[m] * by))));
    a.modes = g->modes;
    a.direct = reach <= 1.6f ? 1 : 0;
    a.err = g->err_d;
    a.contacts = g->contacts_d;
    return a;
}

sp_status gupload_phase(sp_gdem* g)
{
    if (!g->phase_dirty || !g->have_floes) return SP_OK;
    const int nm = std::max(1, g->nmodes);
    const size_t nb = (size_t)g->nbx * g->nby;
    std::vector<double2> tab(nb * nm, make_double2(0.0, 1.0));
    for (size_t b = 0; b < nb; ++b) {
        const double Xc = ((double)(b % g->nbx) + 0.5) * g->p.lx / g->nbx;
        const double Yc = ((double)(b / g->nbx) + 0.5) * g->p.ly / g->nby;
        for (int m = 0; m < g->nmodes; ++m) {
            const double t = g->kx[m] * Xc + g->ky[m] * Yc + g->ph[m];
            tab[b * nm + m] = make_double2(sin(t), cos(t));
        }
    }
    GMode mode[SP_MAX_MODES];
    for (int m = 0; m < g->nmodes; ++m) {
        mode[m].kxL = (float)(g->kx[m] * (g->p.lx / g->nbx));
        mode[m].kyL = (float)(g->ky[m] * (g->p.ly / g->nby));
        mode[m].au = g->au[m];
        mode[m].av = g->av[m];
        mode[m].cz = g->av[m] * g->kx[m] - g->au[m] * g->ky[m];
    }
    if (!g->modes) SP_TRY(galloc(g, &g->modes, SP_MAX_MODES));
    GD_TRY(g, hipMemcpyAsync(g->modes, mode, (size_t)g->nmodes * sizeof(GMode), hipMemcpyHostToDevice, g->stream));
    SP_TRY(galloc(g, &g->phase, tab.size()));
    GD_TRY(g, hipMemcpyAsync(g->phase, tab.data(), tab.size() * sizeof(double2), hipMemcpyHostToDevice, g->stream));
    GD_TRY(g, hipStreamSynchronize(g->stream));
    g->phase_dirty = false;
    return SP_OK;
}

sp_status gerr(sp_gdem* g, uint32_t e)
{
    if (e & kErrOverlap) return gfail(g, SP_EOVERLAP, "two floe centres coincide");
    if (e & kErrNaN) return gfail(g, SP_ENAN, "non-finite floe state");
    if (e & kErrWall) return gfail(g, SP_EWALL, "a floe crossed a wall");
    if (e & kErrRebin) return gfail(g, SP_EDEVICE, "re-binning gathered another number of floes than it counted");
    return SP_OK;
}

// Waits for the stream.
sp_status gcheck(sp_gdem* g)
{
    uint32_t e = 0;
    hipError_t he;
    Readout rd;
    rd.add(&e, g->err_d, 1, false);
    (void)rd.run(g->staging, g->stream, he);
    GD_TRY(g, he);
    return gerr(g, e);
}

}  // namespace

extern "C" {

sp_status sp_gdem_create(const sp_gdem_params* p, void* stream, sp_gdem** out)
{
    if (!p || !out) return SP_EINVAL;
    *out = nullptr;
    if (!(p->lx > 0) || !(p->ly > 0) || !(p->rho_ice > 0) || !(p->rho_ocean > 0) || !(p->cd >= 0) ||
        !(p->E >= 0) || !(p->G >= 0) || !(p->mu >= 0))
        return SP_EINVAL;
    sp_gdem* g = new sp_gdem();
    g->p = *p;
    if (stream) {
        g->stream = (hipStream_t)stream;
    } else {
        if (hipStreamCreate(&g->stream) != hipSuccess) {
            delete g;
            return SP_EDEVICE;
        }
        g->own_stream = true;
    }
    sp_status st = galloc(g, &g->err_d, 1);
    if (!st) st = galloc(g, &g->contacts_d, kContactSlots * kContactStride);
    if (!st && (hipMemsetAsync(g->err_d, 0, 4, g->stream) != hipSuccess ||
                hipMemsetAsync(g->contacts_d, 0, kContactBytes, g->stream) != hipSuccess))
        st = SP_EDEVICE;
    if (st) {
        gdem_free(g);
        if (g->own_stream) (void)hipStreamDestroy(g->stream);
        delete g;
        return st;
    }
    (void)g->staging.reserve(2 * kStagingStep);
    *out = g;
    return SP_OK;
}

void sp_gdem_destroy(sp_gdem* g)
{
    if (!g) return;
    (void)hipStreamSynchronize(g->stream);
    gdem_free(g);
    g->staging.release();
    if (g->own_stream) (void)hipStreamDestroy(g->stream);
    delete g;
}

const char* sp_gdem_last_error(const sp_gdem* g) { return g ? g->err.c_str() : "null context"; }

sp_status sp_gdem_set_ocean(sp_gdem* g, double u0, double v0, int32_t nmodes, const double* kx, const double* ky,
                            const double* au, const double* av, const double* phase)
{
    if (!g) return SP_EINVAL;
    if (nmodes < 0 || nmodes > SP_MAX_MODES) return gfail(g, SP_EINVAL, "nmodes %d out of range", nmodes);
    if (nmodes > 0 && (!kx || !ky || !au || !av || !phase)) return gfail(g, SP_EINVAL, "null mode array");
    g->u0 = u0;
    g->v0 = v0;
    g->nmodes = nmodes;
    for (int m = 0; m < nmodes; ++m) {
        g->kx[m] = kx[m];
        g->ky[m] = ky[m];
        g->au[m] = au[m];
        g->av[m] = av[m];
        g->ph[m] = phase[m];
    }
    g->phase_dirty = true;
    return SP_OK;
}

sp_status sp_gdem_set_floes(sp_gdem* g, int64_t n, const uint32_t* xi, const uint32_t* yi, const float* u,
                            const float* v, const float* omega, const float* theta, const float* r, const float* h)
{
    if (!g) return SP_EINVAL;
    if (n < 1 || n > INT32_MAX / 2) return gfail(g, SP_EINVAL, "floe count %lld out of range", (long long)n);
    if (!xi || !yi || !u || !v || !r || !h) return gfail(g, SP_EINVAL, "null floe array");
    GD_TRY(g, hipStreamSynchronize(g->stream));
    g->have_floes = false;
    float rmax = 0.0f;
    for (int64_t i = 0; i < n; ++i) {
        if (!(r[i] > 0.0f) || !std::isfinite(r[i])) return gfail(g, SP_EINVAL, "radius %lld not positive", (long long)i);
        if (!(h[i] > 0.0f) || !std::isfinite(h[i])) return gfail(g, SP_EINVAL, "thickness %lld not positive", (long long)i);
        rmax = std::max(rmax, r[i]);
    }
    const double lmin = std::min(g->p.lx, g->p.ly);
    if (!((double)rmax < 0.25 * lmin))
        return gfail(g, SP_EINVAL, "r_max %g must stay below a quarter of the domain (%g)", rmax, 0.25 * lmin);
    // sub-bins of side >= 2 r_max: contacts only join neighbouring sub-bins;
    // fewer than 3 along an axis: one sub-bin spans it
    int bx = (int)std::min(4096.0, floor(g->p.lx / (2.0 * (double)rmax)));
    int by = (int)std::min(4096.0, floor(g->p.ly / (2.0 * (double)rmax)));
    if (bx < 3) bx = 1;
    if (by < 3) by = 1;
    g->nbx = bx;
    g->nby = by;
    g->rmax = rmax;
    g->n = n;
    const size_t N = (size_t)n;
    const size_t nb = (size_t)bx * by;
    for (int b = 0; b < 2; ++b) {
        SP_TRY(galloc(g, &g->P[b], N));
        SP_TRY(galloc(g, &g->V[b], N));
        SP_TRY(galloc(g, &g->th[b], N));
        SP_TRY(galloc(g, &g->starts[b], nb + 1));
    }
    SP_TRY(galloc(g, &g->rcount, (size_t)by));
    SP_TRY(galloc(g, &g->bcount, nb));
    SP_TRY(galloc(g, &g->key, N));
    SP_TRY(galloc(g, &g->ckey, N));
    SP_TRY(galloc(g, &g->perm, N));
    if (!g->fallbacks_d) SP_TRY(galloc(g, &g->fallbacks_d, 1));
    // the first grouping: a stable counting sort by sub-bin on the host, the
    // counts and starts the first re-binning reads
    std::vector<int32_t> key(N), count(nb, 0), rows((size_t)by, 0), start(nb + 1, 0), order(N);
    for (size_t i = 0; i < N; ++i) {
        const uint32_t ky = (uint32_t)(((uint64_t)yi[i] * (uint64_t)by) >> 32);
        const uint32_t kx = (uint32_t)(((uint64_t)xi[i] * (uint64_t)bx) >> 32);
        key[i] = (int32_t)(ky * (uint32_t)bx + kx);
        ++count[key[i]];
        ++rows[ky];
    }
    for (size_t b = 0; b < nb; ++b) start[b + 1] = start[b] + count[b];
    {
        std::vector<int32_t> fill(start.begin(), start.end() - 1);
        for (size_t i = 0; i < N; ++i) order[fill[key[i]]++] = (int32_t)i;
    }
    std::vector<int32_t> skey(N);
    for (size_t q = 0; q < N; ++q) skey[q] = key[order[q]];
    {
        std::unique_ptr<char[]> buf(new char[N * 16]);   // one array after the other
        uint32_t* P = reinterpret_cast<uint32_t*>(buf.get());
        float* V = reinterpret_cast<float*>(buf.get());
        for (size_t q = 0; q < N; ++q) {
            const int32_t i = order[q];
            P[4 * q] = xi[i];
            P[4 * q + 1] = yi[i];
            memcpy(&P[4 * q + 2], &r[i], 4);
            P[4 * q + 3] = (uint32_t)i;
        }
        GD_TRY(g, hipMemcpy(g->P[0], P, N * 16, hipMemcpyHostToDevice));
        for (size_t q = 0; q < N; ++q) {
            const int32_t i = order[q];
            V[4 * q] = u[i];
            V[4 * q + 1] = v[i];
            V[4 * q + 2] = omega ? omega[i] : 0.0f;
            V[4 * q + 3] = h[i];
        }
        GD_TRY(g, hipMemcpy(g->V[0], V, N * 16, hipMemcpyHostToDevice));
        for (size_t q = 0; q < N; ++q) V[q] = theta ? theta[order[q]] : 0.0f;
        GD_TRY(g, hipMemcpy(g->th[0], V, N * 4, hipMemcpyHostToDevice));
    }
    GD_TRY(g, hipMemcpy(g->key, skey.data(), N * 4, hipMemcpyHostToDevice));
    GD_TRY(g, hipMemcpy(g->bcount, count.data(), nb * 4, hipMemcpyHostToDevice));
    GD_TRY(g, hipMemcpy(g->rcount, rows.data(), (size_t)by * 4, hipMemcpyHostToDevice));
    GD_TRY(g, hipMemcpy(g->starts[0], start.data(), (nb + 1) * 4, hipMemcpyHostToDevice));
    GD_TRY(g, hipMemsetAsync(g->err_d, 0, 4, g->stream));
    GD_TRY(g, hipMemsetAsync(g->contacts_d, 0, kContactBytes, g->stream));
    GD_TRY(g, hipMemsetAsync(g->fallbacks_d, 0, 8, g->stream));
    GD_TRY(g, hipStreamSynchronize(g->stream));
    g->cur = 0;
    g->sb = 0;
    g->steps = 0;
    g->phase_dirty = true;
    g->have_floes = true;
    return SP_OK;
}

sp_status sp_gdem_step(sp_gdem* g, double dt, int64_t nsteps)
{
    if (!g) return SP_EINVAL;
    if (!g->have_floes) return gfail(g, SP_ESTATE, "sp_gdem_step before sp_gdem_set_floes");
    if (!(dt > 0.0) || !std::isfinite(dt) || nsteps < 0) return gfail(g, SP_EINVAL, "dt must be positive");
    SP_TRY(gupload_phase(g));
    const int n = (int)g->n;
    const dim3 grid((n + 255) / 256), blk(256);
    for (int64_t it = 0; it < nsteps; ++it) {
        const int c = g->cur, o = c ^ 1;
        GPull pl;
        pl.P = g->P[c];
        pl.V = g->V[c];
        pl.th = g->th[c];
        pl.Po = g->P[o];
        pl.Vo = g->V[o];
        pl.tho = g->th[o];
        pl.key = g->key;
        pl.ostart = g->starts[g->sb];
        pl.nstart = g->starts[g->sb ^ 1];
        pl.count = g->bcount;
        pl.rows = g->rcount;
        pl.n = n;
        pl.nbx = g->nbx;
        pl.nby = g->nby;
        pl.err = g->err_d;
        pl.fallbacks = g->fallbacks_d;
        const int64_t waves = (int64_t)g->nby * ((g->nbx + 63) / 64);
        hipLaunchKernelGGL(gpull_kernel, dim3((unsigned)((waves + 3) / 4)), blk, 0, g->stream, pl);
        GD_TRY(g, hipGetLastError());
        hipLaunchKernelGGL(gstep_kernel, grid, blk, 0, g->stream, gargs(g, dt, o, c));
        GD_TRY(g, hipGetLastError());
        g->sb ^= 1;
        g->steps++;
    }
    return SP_OK;
}

sp_status sp_gdem_read_floes(sp_gdem* g, uint32_t* xi, uint32_t* yi, float* u, float* v, float* omega,
                             float* theta, float* r)
{
    if (!g) return SP_EINVAL;
    if (!g->have_floes) return gfail(g, SP_ESTATE, "no floes");
    std::lock_guard<std::mutex> lock(g->reads);
    const int n = (int)g->n, c = g->cur, o = c ^ 1;
    // into the arrays of the other buffer, one after the other
    uint32_t* s0 = reinterpret_cast<uint32_t*>(g->P[o]);
    float* s1 = reinterpret_cast<float*>(g->V[o]);
    const size_t N = (size_t)n;
    uint32_t e = 0;
    hipError_t he;
    Readout rd;
    hipLaunchKernelGGL(gscatter_kernel, dim3((n + 255) / 256), dim3(256), 0, g->stream, n, g->P[c], g->V[c], g->th[c],
                       s0, s0 + N, s1, s1 + N, s1 + 2 * N, s1 + 3 * N, g->th[o]);
    GD_TRY(g, hipGetLastError());
    void* dst[7] = {xi, yi, u, v, omega, theta, r};
    const void* src[7] = {s0, s0 + N, s1, s1 + N, s1 + 2 * N, s1 + 3 * N, g->th[o]};
    for (int k = 0; k < 7; ++k)
        if (dst[k]) rd.add(dst[k], src[k], N, false);
    rd.add(&e, g->err_d, 1, false);
    (void)rd.run(g->staging, g->stream, he);
    GD_TRY(g, he);
    return gerr(g, e);
}

sp_status sp_gdem_coarse_moments(sp_gdem* g, int32_t nxc, int32_t nyc, double* out)
{
    if (!g) return SP_EINVAL;
    if (!g->have_floes) return gfail(g, SP_ESTATE, "no floes");
    if (nxc < 1 || nyc < 1 || (int64_t)nxc * nyc > (1 << 26) || !out)
        return gfail(g, SP_EINVAL, "coarse grid %d x %d out of range or null output", nxc, nyc);
    std::lock_guard<std::mutex> lock(g->reads);
    SP_TRY(gupload_phase(g));
    const int n = (int)g->n, c = g->cur;
    const int ncoarse = nxc * nyc;
    if ((size_t)ncoarse + 1 > g->cstart_cap) {
        SP_TRY(galloc(g, &g->cstart, (size_t)ncoarse + 1));
        g->cstart_cap = (size_t)ncoarse + 1;
    }
    if ((size_t)ncoarse * SP_NMOM > g->cmom_cap) {
        SP_TRY(galloc(g, &g->cmom, (size_t)ncoarse * SP_NMOM));
        g->cmom_cap = (size_t)ncoarse * SP_NMOM;
    }
    if ((size_t)ncoarse > g->ccount_cap) {
        SP_TRY(galloc(g, &g->ccount, (size_t)ncoarse));
        g->ccount_cap = (size_t)ncoarse;
    }
    if ((size_t)nyc > g->crow_cap) {
        SP_TRY(galloc(g, &g->crow, (size_t)nyc));
        g->crow_cap = (size_t)nyc;
    }
    GD_TRY(g, hipMemsetAsync(g->ccount, 0, (size_t)ncoarse * 4, g->stream));
    GD_TRY(g, hipMemsetAsync(g->crow, 0, (size_t)nyc * 4, g->stream));
    hipLaunchKernelGGL(ckey_kernel, dim3((n + 255) / 256), dim3(256), 0, g->stream, g->P[c], n, nxc, nyc, g->ckey, g->ccount, g->crow);
    GD_TRY(g, hipGetLastError());
    const int run = ncoarse <= kCoarseSmall ? kCoarseRun : kCoarseRunLarge;
    const int64_t runs = (int64_t)nyc * ((nxc + run - 1) / run);
    hipLaunchKernelGGL(cpull_kernel, dim3((unsigned)runs), dim3(256), 0, g->stream, g->ckey, g->ccount, g->crow,
                       g->starts[g->sb], n, g->nbx, g->nby, nxc, nyc, run, g->cstart, g->perm, g->err_d,
                       g->fallbacks_d);
    GD_TRY(g, hipGetLastError());
    hipLaunchKernelGGL(cmom_kernel, dim3(ncoarse), dim3(64), 0, g->stream, gargs(g, 0.0, c, c ^ 1), g->perm,
                       g->cstart, ncoarse, g->cmom);
    GD_TRY(g, hipGetLastError());
    uint32_t e = 0;
    hipError_t he;
    Readout rd;
    rd.add(out, g->cmom, (size_t)ncoarse * SP_NMOM, true);
    rd.add(&e, g->err_d, 1, false);
    (void)rd.run(g->staging, g->stream, he);
    GD_TRY(g, he);
    return gerr(g, e);
}

sp_status sp_gdem_read_order(sp_gdem* g, int32_t* ids, int32_t* starts, int64_t* fallbacks)
{
    if (!g) return SP_EINVAL;
    if (!g->have_floes) return gfail(g, SP_ESTATE, "no floes");
    std::lock_guard<std::mutex> lock(g->reads);
    const size_t N = (size_t)g->n, nb = (size_t)g->nbx * g->nby;
    if (ids) {
        int32_t* s = reinterpret_cast<int32_t*>(g->P[g->cur ^ 1]);
        hipLaunchKernelGGL(gids_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, g->stream, (int)N, g->P[g->cur], s);
        GD_TRY(g, hipGetLastError());
        GD_TRY(g, hipMemcpyAsync(ids, s, N * 4, hipMemcpyDeviceToHost, g->stream));
    }
    if (starts) GD_TRY(g, hipMemcpyAsync(starts, g->starts[g->sb], (nb + 1) * 4, hipMemcpyDeviceToHost, g->stream));
    unsigned long long fb = 0;
    GD_TRY(g, hipMemcpyAsync(&fb, g->fallbacks_d, 8, hipMemcpyDeviceToHost, g->stream));
    GD_TRY(g, hipStreamSynchronize(g->stream));
    if (fallbacks) *fallbacks = (int64_t)fb;
    return gcheck(g);
}

sp_status sp_gdem_get_stats(sp_gdem* g, int64_t* contacts, int64_t* steps, int32_t* bins_x, int32_t* bins_y)
{
    if (!g) return SP_EINVAL;
    unsigned long long slots[kContactSlots * kContactStride], cnt = 0;
    uint32_t e = 0;
    hipError_t he;
    Readout rd;
    rd.add(slots, g->contacts_d, kContactSlots * kContactStride, true);
    rd.add(&e, g->err_d, 1, false);
    (void)rd.run(g->staging, g->stream, he);
    GD_TRY(g, he);
    for (int i = 0; i < kContactSlots; ++i) cnt += slots[i * kContactStride];
    if (contacts) *contacts = (int64_t)cnt;
    if (steps) *steps = g->steps;
    if (bins_x) *bins_x = g->nbx;
    if (bins_y) *bins_y = g->nby;
    return gerr(g, e);
}

}  // extern "C"
