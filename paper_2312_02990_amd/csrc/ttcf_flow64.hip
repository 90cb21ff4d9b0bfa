// ttcf_flow64.hip -- daughters with FP64 pair forces on gfx950: shear (Lees-Edwards), planar
// elongation, and mixed flow, isokinetic or Nose-Hoover; and mothers (FP64 or FP32 forces) over
// the same neighbour lists.
//
// The Introduction names elongational and mixed flows among the fields TTCF extends to, and
// Section Mathematical Framework notes that a field other than shear needs mappings of its
// own. The paper prints no equations for them; the dynamics is SLLOD (Eq. system1 with the
// velocity gradient u_x = e x + s y, u_y = -e y in place of the shear; e = 0 is Eq. system1
// itself), dr/dt = p + A r, dp/dt = F - A p - alpha p, A = [[e, s, 0], [0, -e, 0], [0, 0, 0]],
// in the cell the flow carries:
//   elongation  diag(L_x e^{et}, L_y e^{-et}, L_z);
//   mixed       H(t) = exp(A t) diag(L): H_xx = L e^{et}, H_xy = L s t sinhc(e t), H_yy = L e^{-et};
//   shear       the sliding brick, offset fmod(s L_y t, L_x).
// Daughters are short transients, so the carried cells need no reproducible lattice (the host
// refuses a daughter whose cell would become narrower than 3 r_c).
//
// One step of h = dt, tau = h/2, is E(tau) K(tau) D(h) [forces] K(tau) E(tau): E the flow part
// p -> exp(-A tau) p scaled back to the old p.p, K the exact constrained kick under fixed
// forces (Zhang, J. Chem. Phys. 106, 6102 (1997)), D the exact streaming r -> exp(A h)(r + N p),
// N = int_0^h exp(-A u) du; Nose-Hoover daughters run Z T E K D K E T Z without the scalings.
// Every scalar of both halves follows in closed form from moments of (p, F) summed once after
// the force pass, so a step needs one workgroup reduction and two barriers.
//
// Layout: one workgroup per daughter at a time, one, two or four atoms per thread, momenta and
// forces in registers, FP64 positions in LDS (fractions of the carried cell, or the brick's
// coordinates). The atoms go to the threads in the cell order of the call's start, which atoms
// leave slowly, so a wave's lanes work on neighbours: their list builds read the same cells.
// Each atom has the list of every atom within r_c + skin of it, built from a cell grid and kept
// until the atoms may have moved too far (f64_fresh). The first 24 entries lie in LDS; clustered
// systems have more, the rest in global scratch, up to 128 in all; an atom with more still looks its
// partners up in the build's grid every step. (64 FP64 daughters of N = 600 in a dense slab, r_c =
// 1.75, density 0.45, over 50 steps: 1.1 ms so; 3.6 in the cell form; 9.5 with the atoms past 24
// entries tried against every other atom.) A list holds both sides of a pair, so each
// force is one thread's sum in list order: results are deterministic (they follow the rebuilds,
// so splitting a run over calls changes roundings).
//
// What bounds it: FP64 issue. Rebuilding the grid and scanning the 27-cell stencil in FP64 every
// step spends most of its lanes on candidates out of range; a list of about 8 entries per atom of
// which 5 are in range leaves the pair arithmetic (32 FP64 instructions a pair). Measured on one
// MI355X against the kernels that scanned the stencil every step: 1024 daughters of N = 2048 over
// 50 steps, shear 13.4 ms -> 3.74 (2.8e10 atom-steps/s), elongation 13.6 -> 3.61; 256 mixed-flow
// Nose-Hoover daughters of N = 864 over 100 steps 4.41 -> 1.09. Of a step's time about half is
// the force pass, a fifth the list builds, the rest the step's scalars and the two barriers.

#include <math.h>

#include <type_traits>

#include "ttcf_device.h"

namespace ttcf {
namespace {

constexpr int kF64Cap = 24;        // list entries per atom in LDS
constexpr int kF64Ext = 104;       // and further ones in global scratch
constexpr double kF64Skin = 0.15;   // list skin, in units of r_c (0.12: +5%, 0.2: +1%)
constexpr int kF64Red = 16;        // doubles per wave in the reduction scratch
constexpr int kF64Side = 4;        // atoms of a thread whose pairs are evaluated side by side
constexpr int kScan = 3;           // candidates per lane per trip of the list build

enum Flow64 { kFlowShear = 0, kFlowElong = 1, kFlowMixed = 2 };

__host__ __device__ inline size_t f64_align(size_t v) { return (v + 15) & ~(size_t)15; }

struct F64Plan {
    size_t xy, z, start, cnt, sid, list, red, wmax, scan, misc, total;
};

__host__ __device__ inline F64Plan f64_plan(int nmax, int cmax, int threads, int apt) {
    F64Plan p;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = f64_align(o + bytes);
        return at;
    };
    p.xy = take(2 * sizeof(double) * (size_t)nmax);
    p.z = take(sizeof(double) * (size_t)nmax);
    p.start = take(sizeof(uint16_t) * (size_t)(cmax + 1));
    p.sid = take(sizeof(uint16_t) * (size_t)nmax);
    // the build's counts live in the list's bytes until the list is written
    const size_t cnt = sizeof(int32_t) * (size_t)cmax;
    const size_t list = sizeof(uint16_t) * (size_t)kF64Cap * threads * apt;
    p.list = take(list > cnt ? list : cnt);
    p.cnt = p.list;
    p.red = take(sizeof(double) * kF64Red * kMaxWaves);
    p.wmax = take(sizeof(float) * kMaxWaves);
    p.scan = take(sizeof(int32_t) * kMaxWaves);
    p.misc = take(sizeof(int32_t) * 4);
    p.total = o;
    return p;
}

typedef __attribute__((address_space(1))) double GlobalF64;
typedef __attribute__((address_space(1))) uint16_t GlobalU16;

struct F64Lds {
    double2* xy;       // [nmax] positions; during a build the same bytes hold
    double* z;         //        float4 sorted[nmax]
    uint16_t* start;   // [cells + 1] first sorted slot of each cell of the last build
    uint16_t* sid;     // [nmax] its atoms by cell
    int32_t* cnt;      // [cells] counts (build only)
    uint16_t* list;    // [kF64Cap][threads][APT]
    double* red;       // [waves][kF64Red]
    float* wmax;       // [waves]
    int32_t* scan;     // [waves]
    int32_t* misc;     // [0]: the job
    GlobalU16* ext;    // [kF64Ext][threads][APT]: list entries from kF64Cap on
};

__device__ __forceinline__ F64Lds f64_carve(char* base, uint16_t* ext, int nmax, int cmax, int threads,
                                            int apt) {
    const F64Plan p = f64_plan(nmax, cmax, threads, apt);
    F64Lds S;
    S.xy = (double2*)(base + p.xy);
    S.z = (double*)(base + p.z);
    S.start = (uint16_t*)(base + p.start);
    S.cnt = (int32_t*)(base + p.cnt);
    S.sid = (uint16_t*)(base + p.sid);
    S.list = (uint16_t*)(base + p.list);
    S.red = (double*)(base + p.red);
    S.wmax = (float*)(base + p.wmax);
    S.scan = (int32_t*)(base + p.scan);
    S.misc = (int32_t*)(base + p.misc);
    S.ext = (GlobalU16*)ext + (size_t)blockIdx.x * kF64Ext * threads * apt;
    return S;
}

// A value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ double uniform(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sum of K <= P doubles over the workgroup (P = 4, 8 or 16), the same total in every thread.
// Inside a wave a transposed reduction splits the P values over the lane bits (P - 1 exchanges
// and adds in place of P log2 64), the remaining lane bits add in place; then the waves in
// sequence. Fixed order; one barrier, and `red` may be written again only after a later one.
template <int K, int P>
__device__ __forceinline__ void f64_sum(double (&v)[K], double* red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    double a[P];
#pragma unroll
    for (int k = 0; k < P; ++k) a[k] = k < K ? v[k] : 0.0;
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4, b3 = lane & 8;
    int idx = 0;
    xstage<P / 2, 0xB1>(a, b0);  // quad_perm [1, 0, 3, 2]
    xstage<P / 4, 0x4E>(a, b1);  // quad_perm [2, 3, 0, 1]
    if constexpr (P >= 8)
        xstage<P / 8, 0x124>(a, b2);  // row_ror:4
    else
        a[0] += dpp_move<0x124>(a[0]);
    if constexpr (P >= 16)
        xstage<P / 16, 0x128>(a, b3);  // row_ror:8
    else
        a[0] += dpp_move<0x128>(a[0]);
    a[0] += swap_partner<16>(a[0]);
    a[0] += swap_partner<32>(a[0]);
    idx = (P / 2) * (int)b0 + (P / 4) * (int)b1 + (P >= 8 ? (P / 8) * (int)b2 : 0) +
          (P >= 16 ? (int)b3 : 0);
    if (lane < 16 && (P >= 8 || !b2) && (P >= 16 || !b3)) red[wave * kF64Red + idx] = a[0];
    __syncthreads();
    double s = 0.0;
    if (lane < K)
        for (int w = 0; w < nw; ++w) s += red[w * kF64Red + lane];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = lane_value(s, k);
}

// The cell of one moment: how a separation is formed from two stored positions.
struct Cell64 {
    double hxx, hxy, hyy, hzz;  // carried cell; shear: the brick's edges, hxy the offset
    double ixx, iyy, izz;       // shear: reciprocal edges
};

// 1/x: the hardware estimate (relative error e below 2^-22) and one third-order step, which leaves
// e^3.
__device__ __forceinline__ double f64_recip(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    const double e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, __builtin_fma(e, e, e), r);
}

// Separation of positions (dx, dy, dz apart, as stored), through the image that holds every pair
// within r_c: the cell's perpendicular widths are 3 r_c or more, so that pair's fractional
// separations stay below 1/3 and rounding finds its image.
template <int F>
__device__ __forceinline__ void f64_sep(const Cell64& H, double dx, double dy, double dz,
                                        double (&d)[3]) {
    if constexpr (F == kFlowShear) {
        const double ny = rint(dy * H.iyy);
        dx = __builtin_fma(-ny, H.hxy, dx);
        d[1] = __builtin_fma(-ny, H.hyy, dy);
        d[0] = __builtin_fma(-rint(dx * H.ixx), H.hxx, dx);
        d[2] = __builtin_fma(-rint(dz * H.izz), H.hzz, dz);
    } else {
        dx -= rint(dx);
        dy -= rint(dy);
        dz -= rint(dz);
        d[0] = dx * H.hxx;
        if constexpr (F == kFlowMixed) d[0] = __builtin_fma(dy, H.hxy, d[0]);
        d[1] = dy * H.hyy;
        d[2] = dz * H.hzz;
    }
}

__device__ __forceinline__ double f64_frac(double s) {
    s -= floor(s);
    return s >= 1.0 ? 0.0 : s;
}

__device__ __forceinline__ int f64_cell(double s, int nc) {
    const int c = (int)(s * (double)nc);
    return c < 0 ? 0 : (c > nc - 1 ? nc - 1 : c);
}

// Grid of a build: the tilted cell (shear: the offset reduced to half an edge) and cells at least
// the list radius wide in its perpendicular widths, 3 or more a side, split in half along x (a
// row's members lie consecutively, so the scan takes 5 half cells of it in place of 3 cells: a
// sixth fewer candidates), at most cmax half cells in all.
struct Grid64 {
    double hxy;
    int nx, ny, nz;  // nx counts half cells: twice as many along x
};

// What a list was built for.
struct List64 {
    double rl;       // list radius: every pair closer than this at the build is listed
    int64_t k;       // strain counter at the build
    int nx, ny, nz;  // the grid
};

// From this list length on it names the atom's cell instead, in whose stencil its partners are looked
// up.
constexpr int kF64Over = kF64Cap + kF64Ext + 1;

template <int F>
__device__ __forceinline__ double f64_tilt(const Cell64& H) {
    if constexpr (F == kFlowShear) return H.hxy - H.hxx * rint(H.hxy * H.ixx);
    return F == kFlowMixed ? H.hxy : 0.0;
}

__device__ __forceinline__ Grid64 f64_grid(const Cell64& H, double hxy, double wx, double reach,
                                           int cmax) {
    Grid64 g;
    g.hxy = hxy;
    int nx = max(3, (int)fmin(wx / reach, 1000.0)), ny = max(3, (int)fmin(H.hyy / reach, 1000.0)),
        nz = max(3, (int)fmin(H.hzz / reach, 1000.0));
    while (2 * nx * ny * nz > cmax) {  // coarser cells, widest direction first (cmax >= 54)
        if (nx >= ny && nx >= nz)
            --nx;
        else if (ny >= nz)
            --ny;
        else
            --nz;
    }
    g.nx = __builtin_amdgcn_readfirstlane(2 * nx);
    g.ny = __builtin_amdgcn_readfirstlane(ny);
    g.nz = __builtin_amdgcn_readfirstlane(nz);
    return g;
}

// Sorted slots of the stencil's row (dy, dz) of an atom's half cell (cx, cy, cz): slot(v) for v below
// len. Half cells cx - 2 .. cx + 2 of the row; where they wrap in x a second range follows from v =
// len0 on (nx is 6 or more). yy and zz wrap too.
struct Row64 {
    int lo0, len0, off1, len;
    __device__ __forceinline__ int slot(int v) const { return v + (v < len0 ? lo0 : off1); }
};

__device__ __forceinline__ Row64 f64_row(const uint16_t* start, int nx, int ny, int nz, int cx, int yy,
                                         int zz, bool own) {
    zz += zz < 0 ? nz : (zz >= nz ? -nz : 0);
    yy += yy < 0 ? ny : (yy >= ny ? -ny : 0);
    const int row = nx * (yy + ny * zz);
    const int m0 = max(cx - 2, 0), m1 = min(cx + 3, nx);
    const int w0 = cx < 2 ? nx + cx - 2 : 0, w1 = cx < 2 ? nx : max(cx + 3 - nx, 0);
    Row64 r;
    r.lo0 = start[row + m0];
    r.len0 = own ? start[row + m1] - r.lo0 : 0;
    const int lo1 = start[row + w0];
    r.len = r.len0 + (own ? start[row + w1] - lo1 : 0);
    r.off1 = lo1 - r.len0;
    return r;
}

// Counting sort of the atoms into the grid's cells, members of a cell in index order (an atom's
// place is the number of smaller indexes in its cell, so the order does not depend on the
// placement atomics). place[j]: the sorted slot of atom t + j T; cell[j] its cell (-1: no atom);
// cart: its position in the tilted cell. Begins with nothing of the previous list in use; ends without
// a barrier (S.start and S.sid are complete).
template <int F, int APT>
__device__ __forceinline__ void f64_sort(const F64Lds& S, const Cell64& H, const Grid64& g, int n,
                                         const double (&x)[APT], const double (&y)[APT],
                                         const double (&z)[APT], int (&place)[APT],
                                         int (&cell)[APT], float (&cart)[APT][3]) {
    const int T = blockDim.x, t = threadIdx.x;
    const int C = g.nx * g.ny * g.nz;
    for (int c = t; c < C; c += T) S.cnt[c] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        const int a = t + j * T;
        cell[j] = -1;
        place[j] = 0;
        double fx = x[j], fy = y[j], fz = z[j];
        if constexpr (F == kFlowShear) {
            fy = f64_frac(y[j] * H.iyy);
            fx = f64_frac((x[j] - g.hxy * fy) * H.ixx);
            fz = f64_frac(z[j] * H.izz);
        }
        cart[j][0] = (float)(fx * H.hxx + fy * g.hxy);
        cart[j][1] = (float)(fy * H.hyy);
        cart[j][2] = (float)(fz * H.hzz);
        if (a < n) {
            cell[j] = f64_cell(fx, g.nx) + g.nx * (f64_cell(fy, g.ny) + g.ny * f64_cell(fz, g.nz));
            place[j] = atomicAdd(&S.cnt[cell[j]], 1);
        }
    }
    __syncthreads();
    scan_cells(S.cnt, S.start, C, S.scan);
    if (t == 0) S.start[C] = (uint16_t)n;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < APT; ++j)
        if (cell[j] >= 0) S.sid[S.start[cell[j]] + place[j]] = (uint16_t)(t + j * T);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        if (cell[j] >= 0) {
            const int a = t + j * T;
            const int b = S.start[cell[j]], e = S.start[cell[j] + 1];
            int q = b;
            for (int i = b; i < e; ++i) q += S.sid[i] < a ? 1 : 0;
            place[j] = q;
        }
    }
}

// Builds the lists of the positions x, y, z (wrapped into the cell here) and publishes them in
// S.xy, S.z; without STATE they are taken as they are (in the cell) and not published. nh: the own
// atoms' list lengths (kF64Over + cell: longer than any list); returns the wave's longest. The scan
// runs in FP32 over nine rows of five half cells, kScan candidates per lane per trip; the FP32 test
// has a margin for its own rounding, so a list misses no pair of its radius.
template <int F, int APT, bool STATE = true>
__device__ __forceinline__ int f64_build(const F64Lds& S, const Cell64& H, int n, int cmax, double rc,
                         double (&x)[APT], double (&y)[APT], double (&z)[APT], List64& L,
                         int (&nh)[APT]) {
    const int T = blockDim.x, t = threadIdx.x;
    float4* sorted = (float4*)S.xy;
    const double hxy = f64_tilt<F>(H);
    const double wx = H.hxx * H.hyy / sqrt(hxy * hxy + H.hyy * H.hyy);
    const double wmin = fmin(wx, fmin(H.hyy, H.hzz));
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        if constexpr (!STATE) {
        } else if constexpr (F == kFlowShear) {
            const double ny = floor(y[j] * H.iyy);
            y[j] = __builtin_fma(-ny, H.hyy, y[j]);
            x[j] = __builtin_fma(-ny, H.hxy, x[j]);
            if (y[j] < 0.0 || y[j] >= H.hyy) y[j] = 0.0;  // a quotient rounded to a whole edge
            x[j] = wrap1(x[j], H.hxx);
            z[j] = wrap1(z[j], H.hzz);
        } else {
            x[j] = f64_frac(x[j]);
            y[j] = f64_frac(y[j]);
            z[j] = f64_frac(z[j]);
        }
    }
    double skin = fmin(kF64Skin * rc, wmin * (1.0 / 3.0) - rc);
    if (skin < 0.05 * rc) skin = 0.0;
    L.rl = rc + skin;
    // FP32 positions and images are off by less than 2^-23 edges, separations by 2^-21
    const double pad = L.rl + 5e-7 * (H.hxx + fabs(hxy) + H.hyy + H.hzz);
    const Grid64 g = f64_grid(H, hxy, wx, pad, cmax);
    int place[APT], cell[APT];
    float cart[APT][3];
    f64_sort<F, APT>(S, H, g, n, x, y, z, place, cell, cart);
#pragma unroll
    for (int j = 0; j < APT; ++j)
        if (cell[j] >= 0)
            sorted[place[j]] =
                make_float4(cart[j][0], cart[j][1], cart[j][2], __int_as_float(t + j * T));
    __syncthreads();
    const float fxx = (float)H.hxx, fxy = (float)hxy, fyy = (float)H.hyy, fzz = (float)H.hzz;
    const float rl2 = (float)(pad * pad) * (1.0f + 1e-6f);
    // found(id) for each partner of an atom of cell c0 at (px, py, pz)
    auto scan = [&](int self, bool own, int c0, float px, float py, float pz, auto found) {
        const int cx = c0 % g.nx, cy = (c0 / g.nx) % g.ny, cz = c0 / (g.nx * g.ny);
        const float wrap = cx < 2 ? fxx : -fxx;
#pragma unroll 1
        for (int r = 0; r < 9; ++r) {
            const int zz = cz + r / 3 - 1, yy = cy + r % 3 - 1;
            const float uz = pz + (zz < 0 ? fzz : (zz >= g.nz ? -fzz : 0.0f));
            const float uy = py + (yy < 0 ? fyy : (yy >= g.ny ? -fyy : 0.0f));
            float ux = px;
            if constexpr (F != kFlowElong) ux += yy < 0 ? fxy : (yy >= g.ny ? -fxy : 0.0f);
            const float uw = ux + wrap;
            const Row64 row = f64_row(S.start, g.nx, g.ny, g.nz, cx, yy, zz, own);
            for (int v = 0; __builtin_amdgcn_ballot_w64(v < row.len) != 0; v += kScan) {
                float4 m[kScan];
#pragma unroll
                for (int i = 0; i < kScan; ++i) {
                    const int vv = v + i;
                    m[i] = sorted[vv < row.len ? row.slot(vv) : 0];
                }
#pragma unroll
                for (int i = 0; i < kScan; ++i) {
                    const int vv = v + i;
                    const float d0 = (vv < row.len0 ? ux : uw) - m[i].x;
                    const float d1 = uy - m[i].y, d2 = uz - m[i].z;
                    const float r2 = d0 * d0 + d1 * d1 + d2 * d2;
                    const int id = __float_as_int(m[i].w);
                    if ((vv < row.len) & (id != self) & (r2 < rl2)) found(id);
                }
            }
        }
    };
    int most = 0;
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        const bool own = cell[j] >= 0;
        if (own) S.sid[place[j]] = (uint16_t)(t + j * T);  // (each thread has read its cell's ids)
        uint16_t* list = S.list + (t * APT + j);
        int got = 0;
        scan(t + j * T, own, own ? cell[j] : 0, cart[j][0], cart[j][1], cart[j][2], [&](int id) {
            if (got < kF64Cap) list[got * (T * APT)] = (uint16_t)id;
            ++got;
        });
        nh[j] = got;
        most = max(most, got);
    }
    most = __builtin_amdgcn_readlane((int)wave_max_dpp((float)most), 63);
    if (__builtin_expect(most > kF64Cap, 0)) {
        // the entries that found no room in LDS (a second scan, so that the first one, which most
        // builds end with, is no longer)
#pragma unroll 1
        for (int j = 0; j < APT; ++j) {
            int c0 = cell[0], count = nh[0];
            float px = cart[0][0], py = cart[0][1], pz = cart[0][2];
#pragma unroll
            for (int q = 1; q < APT; ++q)
                if (q == j) {
                    c0 = cell[q];
                    count = nh[q];
                    px = cart[q][0];
                    py = cart[q][1];
                    pz = cart[q][2];
                }
            const bool own = count > kF64Cap;
            GlobalU16* ext = S.ext + (t * APT + j);
            int got = 0;
            scan(t + j * T, own, own ? c0 : 0, px, py, pz, [&](int id) {
                if (got >= kF64Cap && got < kF64Cap + kF64Ext)
                    ext[(got - kF64Cap) * (T * APT)] = (uint16_t)id;
                ++got;
            });
            count = count >= kF64Over ? kF64Over + c0 : count;
#pragma unroll
            for (int q = 0; q < APT; ++q)
                if (q == j) nh[q] = count;
        }
    }
    L.nx = g.nx;
    L.ny = g.ny;
    L.nz = g.nz;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        const int a = t + j * T;
        if (STATE && a < n) {
            S.xy[a] = make_double2(x[j], y[j]);
            S.z[a] = z[j];
        }
    }
    __syncthreads();
    return most;
}

// What lies beyond the LDS lists of a wave's lanes (nh: their list lengths): calls see(atom, whether
// it counts) for the further entries of a lane's list, kMore at a time, or for every atom of its
// stencil in the last build's grid if no list holds its partners. ext: the lane's row, its entries
// `stride` apart. One call of see in the code: with two, the two-atom builds spill ten more registers.
constexpr int kMore = 2;
template <typename See>
__device__ __forceinline__ void f64_more(const F64Lds& S, const List64& L, int nh, const GlobalU16* ext,
                                         int stride, See see) {
    const bool over = nh >= kF64Over;
    const int rows = __builtin_amdgcn_ballot_w64(over) != 0 ? 9 : 0;
    const int cell = over ? nh - kF64Over : 0;
    const int cx = cell % L.nx, cy = (cell / L.nx) % L.ny, cz = cell / (L.nx * L.ny);
#pragma unroll 1
    for (int r = -1; r < rows; ++r) {
        Row64 row{0, 0, 0, over ? 0 : nh - kF64Cap};
        if (r >= 0)
            row = f64_row(S.start, L.nx, L.ny, L.nz, cx, cy + r % 3 - 1, cz + r / 3 - 1, over);
#pragma unroll 1
        for (int v = 0; __builtin_amdgcn_ballot_w64(v < row.len) != 0; v += kMore) {
            int m[kMore];
#pragma unroll
            for (int i = 0; i < kMore; ++i) {
                m[i] = 0;
                if (v + i < row.len) m[i] = r < 0 ? ext[(v + i) * stride] : S.sid[row.slot(v + i)];
            }
#pragma unroll
            for (int i = 0; i < kMore; ++i) see(m[i], v + i < row.len);
        }
    }
}

// Forces of the own atoms over their lists, and the thread's share of the pair virials: shear
// w0 = W_xy; elongation w0 = W_xx - W_yy; mixed both (w0 = W_xx - W_yy, w1 = W_xy). Every pair is
// seen from both sides, so each side adds half. The thread's atoms run side by side (up to four
// independent chains), the next list word and positions loaded a trip ahead.
template <int F, int APT>
__device__ __forceinline__ void f64_forces(const F64Lds& S, const Cell64& H, const List64& L,
                                           int n, double rc2, double ca, const int (&nh)[APT], int longest,
                                           double (&fx)[APT], double (&fy)[APT],
                                           double (&fz)[APT], double& w0, double& w1) {
    const int T = blockDim.x, t = threadIdx.x;
    double a0 = 0.0, a1 = 0.0;
    constexpr int P = APT < kF64Side ? APT : kF64Side;  // atoms side by side
    const int trips = min(longest, kF64Cap);
    // force over separation of a pair d apart
    auto factor = [&](const double (&d)[3], bool listed) {
        const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
        const double inv = f64_recip(r2);
        const double s3 = inv * inv * inv;
        const double fs = s3 * (48.0 * s3 - 24.0 * ca) * inv;
        return (listed && r2 < rc2) ? fs : 0.0;
    };
    auto virial = [&](const double (&d)[3], double fs) {
        if constexpr (F == kFlowShear) {
            a0 += d[0] * (fs * d[1]);
        } else {
            a0 += fs * (d[0] * d[0] - d[1] * d[1]);
            if constexpr (F == kFlowMixed) a1 += fs * (d[0] * d[1]);
        }
    };
#pragma unroll
    for (int q = 0; q < APT; q += P) {
        double xi[P], yi[P], zi[P], gx[P], gy[P], gz[P];
        int own[P];
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const int a = t + (q + j) * T;
            own[j] = a < n ? a : 0;
            const double2 p = S.xy[own[j]];
            xi[j] = p.x;
            yi[j] = p.y;
            zi[j] = S.z[own[j]];
            gx[j] = gy[j] = gz[j] = 0.0;
        }
        int len[P];
#pragma unroll
        for (int j = 0; j < P; ++j) len[j] = nh[q + j] >= kF64Over ? 0 : min(nh[q + j], kF64Cap);
        // entries k of the P atoms (clamped: nothing past the longest list is read)
        struct Word {
            uint16_t id[P];
        };
        auto word = [&](int k) -> Word {
            k = k < trips ? k : trips - 1;
            Word w;
            __builtin_memcpy(&w, __builtin_assume_aligned(S.list + (k * T + t) * APT + q, 2 * P), 2 * P);
            return w;
        };
        double2 pj[P];
        double zj[P];
        auto load = [&](const Word& w, int k) {
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const int m = k < len[j] ? (int)w.id[j] : own[j];
                pj[j] = S.xy[m];
                zj[j] = S.z[m];
            }
        };
        auto pair = [&](int j, const double2& p, double z, bool listed) {
            double d[3];
            f64_sep<F>(H, xi[j] - p.x, yi[j] - p.y, zi[j] - z, d);
            const double fs = factor(d, listed);
            gx[j] += fs * d[0];
            gy[j] += fs * d[1];
            gz[j] += fs * d[2];
            virial(d, fs);
        };
        Word next{};
        if (trips > 0) {
            load(word(0), 0);
            next = word(1);
        }
#pragma unroll 1
        for (int k = 0; k < trips; ++k) {
            double2 pc[P];
            double zc[P];
#pragma unroll
            for (int j = 0; j < P; ++j) {
                pc[j] = pj[j];
                zc[j] = zj[j];
            }
            load(next, k + 1);
            next = word(k + 2);
#pragma unroll
            for (int j = 0; j < P; ++j)
                pair(j, pc[j], zc[j], k < len[j]);
        }
#pragma unroll
        for (int j = 0; j < P; ++j) {
            fx[q + j] = gx[j];
            fy[q + j] = gy[j];
            fz[q + j] = gz[j];
        }
    }
    // entries beyond LDS, an atom at a time (most waves have none)
    if (__builtin_expect(longest > kF64Cap, 0)) {
#pragma unroll 1
        for (int j = 0; j < APT; ++j) {
            int count = nh[0];
#pragma unroll
            for (int q = 1; q < APT; ++q) count = q == j ? nh[q] : count;
            const int a = t + j * T, own = a < n ? a : 0;
            const double2 pi = S.xy[own];
            const double zi = S.z[own];
            const GlobalU16* ext = S.ext + (t * APT + j);
            double gx = 0.0, gy = 0.0, gz = 0.0;
            int near = 0;  // partners in range
            auto separation = [&](int m, double (&d)[3]) {
                const double2 pm = S.xy[m];
                f64_sep<F>(H, pi.x - pm.x, pi.y - pm.y, zi - S.z[m], d);
                return d[0] * d[0] + d[1] * d[1] + d[2] * d[2] < rc2;
            };
            f64_more(S, L, count, ext, T * APT, [&](int m, bool live) {
                double d[3];
                live = live && m != own;
                near += separation(m, d) && live ? 1 : 0;
                const double fs = factor(d, live);
                gx += fs * d[0];
                gy += fs * d[1];
                gz += fs * d[2];
                virial(d, fs);
            });
            if constexpr (F != kFlowShear) {
                // a carried-flow daughter this dense fails its health check
                if (count > kF64Cap && count < kF64Over)
                    for (int k = 0; k < kF64Cap; ++k) {
                        double d[3];
                        near += separation(S.list[(k * T + t) * APT + j], d) ? 1 : 0;
                    }
                if (near > kF64Cap) gx = __builtin_nan("");
            }
#pragma unroll
            for (int q = 0; q < APT; ++q)
                if (q == j) {
                    fx[q] += gx;
                    fy[q] += gy;
                    fz[q] += gz;
                }
        }
    }
    w0 = 0.5 * a0;
    w1 = 0.5 * a1;
}

// Moments of (p, F) from which both half steps follow.
struct Mom64 {
    double pp, xx, yy, xy;        // sum p.p, p_x^2, p_y^2, p_x p_y
    double fp, gxx, gyy, gxy, gyx;  // sum F.p, F_x p_x, F_y p_y, F_x p_y, F_y p_x
    double ff, qxx, qyy, qxy;     // sum F.F, F_x^2, F_y^2, F_x F_y
};

// Moments summed over the workgroup, with the pair virials and (shear) the positions' sum, which
// carries a non-finite coordinate to the health check.
template <int F, int APT>
__device__ __forceinline__ Mom64 f64_moments(const double (&px)[APT], const double (&py)[APT],
                                             const double (&pz)[APT], const double (&fx)[APT],
                                             const double (&fy)[APT], const double (&fz)[APT],
                                             double& w0, double& w1, double& pos, double* red) {
    Mom64 m{};
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        m.pp += px[j] * px[j] + py[j] * py[j] + pz[j] * pz[j];
        m.xx += px[j] * px[j];
        m.yy += py[j] * py[j];
        m.xy += px[j] * py[j];
        m.fp += fx[j] * px[j] + fy[j] * py[j] + fz[j] * pz[j];
        m.gxx += fx[j] * px[j];
        m.gyy += fy[j] * py[j];
        m.gxy += fx[j] * py[j];
        m.gyx += fy[j] * px[j];
        m.ff += fx[j] * fx[j] + fy[j] * fy[j] + fz[j] * fz[j];
        m.qxx += fx[j] * fx[j];
        m.qyy += fy[j] * fy[j];
        m.qxy += fx[j] * fy[j];
    }
    if constexpr (F == kFlowShear) {
        double v[12] = {m.pp, m.xy, m.yy, m.fp, m.gxy, m.gyx, m.qxy, m.gyy, m.qyy, m.ff, w0, pos};
        f64_sum<12, 16>(v, red);
        m = Mom64{v[0], 0, v[2], v[1], v[3], 0, v[7], v[4], v[5], v[9], 0, v[8], v[6]};
        w0 = v[10];
        pos = v[11];
    } else if constexpr (F == kFlowElong) {
        double v[10] = {m.pp, m.xx, m.yy, m.fp, m.gxx, m.gyy, m.ff, m.qxx, m.qyy, w0};
        f64_sum<10, 16>(v, red);
        m = Mom64{v[0], v[1], v[2], 0, v[3], v[4], v[5], 0, 0, v[6], v[7], v[8], 0};
        w0 = v[9];
    } else {
        double v[15] = {m.pp,  m.xx, m.yy,  m.xy,  m.fp,  m.gxx, m.gyy, m.gxy,
                        m.gyx, m.ff, m.qxx, m.qyy, m.qxy, w0,    w1};
        f64_sum<15, 16>(v, red);
        m = Mom64{v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10], v[11], v[12]};
        w0 = v[13];
        w1 = v[14];
    }
    return m;
}

// The flow part E, p -> (fa p_x + fc p_y, fd p_y, p_z), on the moments (not rescaled).
template <int F>
__device__ __forceinline__ void f64_flow(Mom64& m, double fa, double fc, double fd) {
    if constexpr (F == kFlowShear) {
        m.pp += 2.0 * fc * m.xy + fc * fc * m.yy;
        m.fp += fc * m.gxy;
        m.xy += fc * m.yy;
    } else {
        const double zz = m.pp - m.xx - m.yy, gzz = m.fp - m.gxx - m.gyy;
        m.xx = fa * fa * m.xx;
        m.gxx = fa * m.gxx;
        if constexpr (F == kFlowMixed) {
            m.xx += 2.0 * fa * fc * m.xy + fc * fc * m.yy;
            m.gxx += fc * m.gxy;
            m.xy = fd * (fa * m.xy + fc * m.yy);
            m.gxy = fd * m.gxy;
            m.gyx = fa * m.gyx + fc * m.gyy;
        }
        m.yy = fd * fd * m.yy;
        m.gyy = fd * m.gyy;
        m.pp = m.xx + m.yy + zz;
        m.fp = m.gxx + m.gyy + gzz;
    }
}

// The kick K, p -> (p + F s) / sd, on the moments.
__device__ __forceinline__ void f64_kick(Mom64& m, double s, double isd) {
    const double i2 = isd * isd;
    m.pp = (m.pp + 2.0 * s * m.fp + s * s * m.ff) * i2;
    m.xx = (m.xx + 2.0 * s * m.gxx + s * s * m.qxx) * i2;
    m.yy = (m.yy + 2.0 * s * m.gyy + s * s * m.qyy) * i2;
    m.xy = (m.xy + s * (m.gxy + m.gyx) + s * s * m.qxy) * i2;
    m.fp = (m.fp + s * m.ff) * isd;
    m.gxx = (m.gxx + s * m.qxx) * isd;
    m.gyy = (m.gyy + s * m.qyy) * isd;
    m.gxy = (m.gxy + s * m.qxy) * isd;
    m.gyx = (m.gyx + s * m.qxy) * isd;
}

__device__ __forceinline__ void f64_scale(Mom64& m, double c) {
    const double c2 = c * c;
    m.pp *= c2;
    m.xx *= c2;
    m.yy *= c2;
    m.xy *= c2;
    m.fp *= c;
    m.gxx *= c;
    m.gyy *= c;
    m.gxy *= c;
    m.gyx *= c;
}

__device__ __forceinline__ double f64_phi(double u) { return u == 0.0 ? 1.0 : -expm1(-u) / u; }

// sinh(x) / x from e^x and e^-x; the power series where their difference would cancel (the first
// omitted term is below 1e-16 for |x| < 0.5)
__device__ __forceinline__ double f64_sinhc(double x, double ep, double em) {
    const double u = x * x;
    double c = 1.0 + u * (1.0 / 156.0);
    c = 1.0 + u * (1.0 / 110.0) * c;
    c = 1.0 + u * (1.0 / 72.0) * c;
    c = 1.0 + u * (1.0 / 42.0) * c;
    c = 1.0 + u * (1.0 / 20.0) * c;
    c = 1.0 + u * (1.0 / 6.0) * c;
    return u < 0.25 ? c : 0.5 * (ep - em) / x;
}

// What a step reads besides the moments; LDS keeps it out of the force loop's registers.
struct Const64 {
    double l0x, l0y, lz, il0x, il0y, ilz;  // edges at strain 0 and their reciprocals
    double er, sr, irn;      // flow rates (shear: sr; elongation: er), 1 / the response's divisor
    double fa, fc, fd;       // exp(-A tau)
    double nxx, nxy, nyy;    // N = int_0^h exp(-A u) du
    double h, k0, root2k0, nh_iq, nh_target, inv_v, rc, rc2, ca;
    double mu, drift;        // growth rate bound of separations; |N p| <= drift h |p|
};

// The carried cell at strain counter k, and e^{-zeta tau} (Nose-Hoover): one exp evaluation for
// all three values, a lane each.
template <int F, bool NH>
__device__ __forceinline__ void f64_cell_at(const Const64& Q, const SysDev& sys, int64_t k,
                                            double zeta, Cell64& H, double& damp) {
    const int lane = threadIdx.x & 63;
    const double tau = 0.5 * Q.h;
    damp = 1.0;
    if constexpr (F == kFlowShear) {
        H.hxy = uniform(le_offset_nb(sys, Q.sr, k, Q.il0x));
        if constexpr (NH) damp = uniform(exp(-zeta * tau));
    } else {
        const double x = Q.er * ((double)k * Q.h);
        const double v = exp(lane == 0 ? x : (lane == 1 ? -x : (NH ? -zeta * tau : 0.0)));
        const double ep = lane_value(v, 0), em = lane_value(v, 1);
        H.hxx = uniform(Q.l0x * ep);
        H.hyy = uniform(Q.l0y * em);
        H.ixx = uniform(Q.il0x * em);
        H.iyy = uniform(Q.il0y * ep);
        if constexpr (F == kFlowMixed)
            H.hxy = uniform(Q.l0y * Q.sr * ((double)k * Q.h) * f64_sinhc(x, ep, em));
        if constexpr (NH) damp = lane_value(v, 2);
    }
}

// Whether lists built at strain counter L.k still hold every pair within r_c: a pair now closer
// than r_c was closer than sigma (r_c + 2 path) at the build, sigma >= |exp(-A t)| over the time
// since (exp(mu t), mu the largest eigenvalue of the symmetric part of -A) and path the longest
// |N p| path of an atom. e^v <= 1 + v + v^2 for v <= 1.
__device__ __forceinline__ bool f64_fresh(const Const64& Q, const List64& L, int64_t k, float path) {
    const double v = Q.mu * ((double)(k - L.k) * Q.h);
    const double sigma = 1.0 + v + v * v;
    return v <= 1.0 && sigma * (Q.rc + 2.0 * Q.drift * (double)path) <= L.rl;
}

template <int F, bool NH, int APT>
__device__ __forceinline__ void flow64_job(DaughterDesc* dp, const PefLaunch& B, const F64Lds& S,
                                           Const64& Q, SysDev& sys) {
    const int T = blockDim.x, t = threadIdx.x;
    const int n = dp->sys.n;
    const int32_t done0 = dp->done;
    int health = dp->health;
    int todo = min(B.max_steps, dp->n_steps - done0);
    if (health != 0) todo = 0;
    if (todo <= 0) return;  // uniform over the workgroup
    if (t == 0) {
        sys = dp->sys;
        Q.h = dp->sys.dt;
        Q.er = F == kFlowShear ? 0.0 : (F == kFlowElong ? dp->gamma_dot : dp->erate);
        Q.sr = F == kFlowShear ? dp->gamma_dot : (F == kFlowElong ? 0.0 : dp->srate);
        Q.irn = 1.0 / dp->gamma_dot;
        const double h = Q.h, tau = 0.5 * h, x = Q.er * tau, hh = Q.er * h;
        Q.fa = exp(-x);
        Q.fd = exp(x);
        const double hs = f64_sinhc(x, Q.fd, Q.fa);
        Q.fc = -Q.sr * tau * hs;
        Q.nxx = h * f64_phi(hh);
        Q.nyy = h * f64_phi(-hh);
        Q.nxy = -0.5 * Q.sr * h * h * hs * hs;
        Q.l0x = dp->sys.box[0];
        Q.l0y = dp->sys.box[1];
        Q.lz = dp->sys.box[2];
        Q.il0x = 1.0 / Q.l0x;
        Q.il0y = 1.0 / Q.l0y;
        Q.ilz = 1.0 / Q.lz;
        Q.k0 = dp->k0;
        Q.root2k0 = sqrt(2.0 * dp->k0);
        Q.nh_iq = NH ? 1.0 / dp->nh_q : 0.0;
        Q.nh_target = dp->nh_target;
        Q.inv_v = 1.0 / dp->sys.volume;
        Q.rc = dp->sys.rc;
        Q.rc2 = dp->sys.rc2;
        Q.ca = dp->sys.c_attr;
        Q.mu = sqrt(Q.er * Q.er + 0.25 * Q.sr * Q.sr);
        const double a = fabs(hh) + fabs(Q.sr * h);
        Q.drift = (1.0 + a + a * a) * (1.0 + 1e-5);  // |N p| <= h |p| e^{|A| h}; FP32 paths
    }
    __syncthreads();
    if (n > T * APT || n > B.nmax || (F == kFlowMixed && !(dp->gamma_dot > 0.0)))
        health = kHealthNonFinite;
    int64_t k = dp->k;
    double zeta = dp->zeta, damp;
    Cell64 H;
    H.hxx = uniform(Q.l0x);
    H.hyy = uniform(Q.l0y);
    H.hzz = uniform(Q.lz);
    H.hxy = 0.0;
    H.ixx = uniform(Q.il0x);
    H.iyy = uniform(Q.il0y);
    H.izz = uniform(Q.ilz);
    f64_cell_at<F, false>(Q, sys, k, 0.0, H, damp);
    auto narrow = [&]() {  // the host refuses such runs; every lane agrees
        if constexpr (F == kFlowShear) {
            return false;
        } else {
            const double w3 = 3.0 * Q.rc * (1.0 - 1e-12);
            const double wx = F == kFlowMixed ? H.hxx * H.hyy * rsq_nr(H.hxy * H.hxy + H.hyy * H.hyy)
                                              : H.hxx;
            return !(wx >= w3) || !(H.hyy >= w3) || !(H.hzz >= w3);
        }
    };
    if (narrow()) health = kHealthNonFinite;
    if (health) {
        if (t == 0) dp->health = health;
        return;
    }
    double* st = dp->state;
    GlobalF64* series = (GlobalF64*)dp->series;
    GlobalF64* xs = F == kFlowMixed ? (GlobalF64*)dp->xseries : nullptr;
    const bool components = F == kFlowMixed && dp->xseries != nullptr;

    double px[APT], py[APT], pz[APT], fx[APT], fy[APT], fz[APT];
    float path[APT];
    int nh[APT], longest = 0;
    uint16_t atom[APT];  // the state's atom behind the thread's atom j
    List64 L{};
    double w0, w1 = 0.0;
    // a coordinate of the state as the kernel holds it
    auto stored = [&](double& x, double& y, double& z) {
        if constexpr (F == kFlowElong) {
            x /= H.hxx;
            y /= H.hyy;
            z /= H.hzz;
        } else if constexpr (F == kFlowMixed) {
            y /= H.hyy;
            x = (x - H.hxy * y) / H.hxx;
            z /= H.hzz;
        }
    };
    {
        // deal the atoms to the threads in cell order
        double x[APT], y[APT], z[APT];
#pragma unroll
        for (int j = 0; j < APT; ++j) {
            const int a = t + j * T;
            const bool v = a < n;
            x[j] = v ? st[a] : 0.0;
            y[j] = v ? st[n + a] : 0.0;
            z[j] = v ? st[2 * n + a] : 0.0;
            stored(x[j], y[j], z[j]);
            if constexpr (F != kFlowShear) {
                x[j] = f64_frac(x[j]);
                y[j] = f64_frac(y[j]);
                z[j] = f64_frac(z[j]);
            }
        }
        const double hxy = f64_tilt<F>(H);
        const double wx = H.hxx * H.hyy / sqrt(hxy * hxy + H.hyy * H.hyy);
        const Grid64 g = f64_grid(H, hxy, wx, Q.rc, B.cmax);
        int place[APT], cell[APT];
        float cart[APT][3];
        f64_sort<F, APT>(S, H, g, n, x, y, z, place, cell, cart);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < APT; ++j)
            if (cell[j] >= 0) S.sid[place[j]] = (uint16_t)(t + j * T);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < APT; ++j) {
            const int a = t + j * T;
            atom[j] = a < n ? S.sid[a] : 0;
        }
        __syncthreads();  // the build reuses these bytes
    }
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        const int a = t + j * T;
        const bool v = a < n;
        const double* q = st + atom[j];
        px[j] = v ? q[3 * (size_t)n] : 0.0;
        py[j] = v ? q[4 * (size_t)n] : 0.0;
        pz[j] = v ? q[5 * (size_t)n] : 0.0;
        path[j] = 0.0f;
        if (v) {
            double x = q[0], y = q[n], z = q[2 * (size_t)n];
            stored(x, y, z);
            S.xy[a] = make_double2(x, y);
            S.z[a] = z;
        }
    }
    // the recorded series, and for mixed flow its components
    auto record = [&](int at, const Mom64& q) {
        double b;
        if constexpr (F == kFlowShear) {
            b = q.xy + w0;
        } else if constexpr (F == kFlowElong) {
            b = q.xx - q.yy + w0;
        } else {
            const double cn = q.xx - q.yy + w0, cxy = q.xy + w1;
            b = (Q.er * cn + Q.sr * cxy) * Q.irn;
            if (t == 0 && components) {
                GlobalF64* row = xs + (size_t)at * kObsCols;
                row[0] = cn * Q.inv_v;
                row[1] = cxy * Q.inv_v;
                for (int c = 2; c < kObsCols; ++c) row[c] = 0.0;
            }
        }
        if (t == 0) series[at] = b;
        return b;
    };
    Mom64 m{};
    bool fresh = false;
    int it = -1;  // steps done; -1: the forces and moments of the start state come first
    for (;;) {
        const double h = Q.h, tau = 0.5 * h;
        if (it >= 0) {
            // ---- first half
            double s1 = 0.0, isd1 = 1.0, g1 = 1.0;
            if constexpr (NH) {
                zeta += tau * (m.pp - Q.nh_target) * Q.nh_iq;
            } else {
                const double ipp = rcp_nr(m.pp);
                f64_flow<F>(m, Q.fa, Q.fc, Q.fd);
                g1 = rsq_nr(m.pp * ipp);
                double sd;
                iso_kick_coeffs(g1 * m.fp * ipp, m.ff * ipp, tau, s1, sd);
                isd1 = rcp_nr(sd);
            }
            // ---- streaming in the cell of step k, then the cell of step k + 1
            const double ax = H.ixx, ay = H.iyy, az = h * H.izz, axy = H.hxy;
            f64_cell_at<F, NH>(Q, sys, k + 1, zeta, H, damp);
            float most = 0.0f;
#pragma unroll
            for (int j = 0; j < APT; ++j) {
                const int a = t + j * T;
                if constexpr (NH) {
                    const double qx = px[j] * damp, qy = py[j] * damp;
                    px[j] = (Q.fa * qx + Q.fc * qy) + tau * fx[j];
                    py[j] = Q.fd * qy + tau * fy[j];
                    pz[j] = pz[j] * damp + tau * fz[j];
                } else {
                    const double qx = g1 * (Q.fa * px[j] + Q.fc * py[j]);
                    const double qy = g1 * (Q.fd * py[j]);
                    const double qz = g1 * pz[j];
                    px[j] = (qx + fx[j] * s1) * isd1;
                    py[j] = (qy + fy[j] * s1) * isd1;
                    pz[j] = (qz + fz[j] * s1) * isd1;
                }
                const float ux = (float)px[j], uy = (float)py[j], uz = (float)pz[j];
                path[j] += (float)h * __builtin_sqrtf(ux * ux + uy * uy + uz * uz);
                most = fmaxf(most, path[j]);
                if (a < n) {
                    double2 r = S.xy[a];
                    if constexpr (F == kFlowShear) {
                        r.x += h * px[j] + h * Q.sr * (r.y + tau * py[j]);
                        r.y += h * py[j];
                        S.z[a] += h * pz[j];
                    } else if constexpr (F == kFlowElong) {
                        r.x += Q.nxx * px[j] * ax;
                        r.y += Q.nyy * py[j] * ay;
                        S.z[a] += az * pz[j];
                    } else {
                        const double dsy = Q.nyy * py[j] * ay;
                        r.x += ((Q.nxx * px[j] + Q.nxy * py[j]) - axy * dsy) * ax;
                        r.y += dsy;
                        S.z[a] += az * pz[j];
                    }
                    S.xy[a] = r;
                }
            }
            k += 1;
            if (narrow()) {
                health = kHealthNonFinite;  // uniform: every thread stops here
                break;
            }
            most = wave_max_dpp(most);
            if ((t & 63) == 63) S.wmax[t >> 6] = most;
            __syncthreads();
            most = 0.0f;
            for (int w = 0; w < (T >> 6); ++w) most = fmaxf(most, S.wmax[w]);
            fresh = f64_fresh(Q, L, k, most);
        }
        if (!fresh) {
            double x[APT], y[APT], z[APT];
#pragma unroll
            for (int j = 0; j < APT; ++j) {
                const int a = t + j * T;
                const double2 r = S.xy[a < n ? a : 0];
                x[j] = r.x;
                y[j] = r.y;
                z[j] = S.z[a < n ? a : 0];
                path[j] = 0.0f;
            }
            L.k = k;
            longest = f64_build<F, APT>(S, H, n, B.cmax, Q.rc, x, y, z, L, nh);
        }
        f64_forces<F, APT>(S, H, L, n, Q.rc2, Q.ca, nh, longest, fx, fy, fz, w0, w1);
        ++it;
        double pos = 0.0;
        if constexpr (F == kFlowShear) {  // carries a non-finite coordinate to the health check
#pragma unroll
            for (int j = 0; j < APT; ++j) {
                const int a = t + j * T;
                if (a < n) pos += S.xy[a].x + S.xy[a].y + S.z[a];
            }
        }
        bool bad = false, drift = false;
        if constexpr (NH) {
            // ---- second half: K E T, then Z on the new sum p.p
            double v[6] = {0.0, 0.0, 0.0, w0, w1, pos};
#pragma unroll
            for (int j = 0; j < APT; ++j) {
                if (it > 0) {
                    const double qx = px[j] + tau * fx[j], qy = py[j] + tau * fy[j];
                    px[j] = (Q.fa * qx + Q.fc * qy) * damp;
                    py[j] = (Q.fd * qy) * damp;
                    pz[j] = (pz[j] + tau * fz[j]) * damp;
                }
                v[0] += px[j] * px[j] + py[j] * py[j] + pz[j] * pz[j];
                if constexpr (F != kFlowShear) v[1] += px[j] * px[j] - py[j] * py[j];
                if constexpr (F != kFlowElong) v[2] += px[j] * py[j];
            }
            f64_sum<6, 8>(v, S.red);
            m.pp = v[0];
            m.xx = v[1];
            m.xy = v[2];
            w0 = v[3];
            w1 = v[4];
            pos = v[5];
            if (it > 0) zeta += tau * (m.pp - Q.nh_target) * Q.nh_iq;
            bad = !isfinite(zeta);
        } else {
            m = f64_moments<F, APT>(px, py, pz, fx, fy, fz, w0, w1, pos, S.red);
            if (it > 0) {
                // ---- second half: K E, then the exact K0 rescale
                const double ipp = rcp_nr(m.pp);
                double s2, sd;
                iso_kick_coeffs(m.fp * ipp, m.ff * ipp, tau, s2, sd);
                const double isd2 = rcp_nr(sd);
                f64_kick(m, s2, isd2);
                drift = fabs(m.pp * ipp - 1.0) > 1e-10;
                f64_flow<F>(m, Q.fa, Q.fc, Q.fd);
                const double c = Q.root2k0 * rsq_nr(m.pp);
                f64_scale(m, c);
#pragma unroll
                for (int j = 0; j < APT; ++j) {
                    const double qx = (px[j] + fx[j] * s2) * isd2;
                    const double qy = (py[j] + fy[j] * s2) * isd2;
                    const double qz = (pz[j] + fz[j] * s2) * isd2;
                    px[j] = c * (Q.fa * qx + Q.fc * qy);
                    py[j] = c * (Q.fd * qy);
                    pz[j] = c * qz;
                }
                bad = !isfinite(c);
            }
        }
        if (it == 0) {
            if (done0 == 0) {
                (void)record(0, m);
                if (t == 0 && (F != kFlowShear || Q.k0 <= 0.0)) {
                    Q.k0 = 0.5 * m.pp;  // read after the barriers of the first step
                    Q.root2k0 = sqrt(m.pp);
                }
            }
        } else {
            const double b = record(done0 + it, m);
            // uniform: every thread holds the same sums
            if (!isfinite(b) || (F == kFlowShear && (bad || !isfinite(pos)))) {
                health |= kHealthNonFinite;
            } else if (F == kFlowShear && drift) {
                health |= kHealthDrift;
            }
        }
        if (health != 0 || it == todo) break;
    }
    // the state, wrapped, in the coordinates of the current cell
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        const int a = t + j * T;
        if (a < n) {
            double2 r = S.xy[a];
            double z = S.z[a];
            if constexpr (F == kFlowShear) {
                const double ny = floor(r.y * H.iyy);
                r.y = __builtin_fma(-ny, H.hyy, r.y);
                r.x = wrap1(__builtin_fma(-ny, H.hxy, r.x), H.hxx);
                if (r.y < 0.0 || r.y >= H.hyy) r.y = 0.0;
                z = wrap1(z, H.hzz);
            } else {
                r.y = f64_frac(r.y);
                r.x = f64_frac(r.x) * H.hxx;
                if constexpr (F == kFlowMixed) r.x += H.hxy * r.y;
                r.y *= H.hyy;
                z = f64_frac(z) * H.hzz;
            }
            double* q = st + atom[j];
            q[0] = r.x;
            q[n] = r.y;
            q[2 * (size_t)n] = z;
            q[3 * (size_t)n] = px[j];
            q[4 * (size_t)n] = py[j];
            q[5 * (size_t)n] = pz[j];
        }
    }
    if (t == 0) {
        dp->k = k;
        dp->done = done0 + it;
        dp->k0 = Q.k0;
        if (NH) dp->zeta = zeta;
        dp->health = health;
    }
}

// A persistent grid: workgroups take daughters from a queue, largest systems first.
template <int F, bool NH, int APT>
__global__ void __launch_bounds__(APT == 4 ? 512 : 1024, APT == 4 ? 2 : 4) k_flow64(PefLaunch B) {
    extern __shared__ __align__(16) char smem[];
    __shared__ Const64 Q;
    __shared__ SysDev sys;
    const F64Lds S = f64_carve(smem, B.ext, B.nmax, B.cmax, blockDim.x, APT);
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) S.misc[0] = atomicAdd(B.queue, 1);
        __syncthreads();
        const int job = __builtin_amdgcn_readfirstlane(S.misc[0]);
        if (job >= B.n_jobs) return;
        flow64_job<F, NH, APT>(&B.descs[B.order[job]], B, S, Q, sys);
    }
}

// ---- mothers -----------------------------------------------------------------------------
// Nose-Hoover equilibrium dynamics (the step of k_mother) over the same lists, one workgroup per
// mother, atoms dealt to the threads as for daughters. Both force forms give what the cell form
// gives:
//   FP64  f64_forces (another order of the sums);
//   FP32  the cell form's bits, for atoms whose list fits LDS (the others' forces are summed in FP64
//         and rounded). Its separations come from FP32 coordinates relative to the atoms'
//         cells, and its sums run over the stencil's cells in turn, so every step each atom's cell
//         and relative coordinates go to LDS, and an atom's listed partners are taken in the
//         order (dz, dy, dx of the cells, index). The list is kept in that order; a lane that meets
//         a partner in range out of its turn (one in a hundred, each step) has its list sorted
//         and summed by its wave.
// What bounds a step is a CU's vector issue in the pair sums, of which the longest list of a wave
// sets the number of trips (13 for a mean of 8), then the builds (a fifth) and the waves that wait
// for one with several lanes out of turn. Measured on one MI355X, a step of one mother, cell form
// -> lists: N = 2048 43.8 -> 23.1 us (FP64 59.7 -> 15.6), N = 1000 22.3 -> 12.8 (30.3 -> 7.6); 256
// copies of N = 500 sampled over 150 steps 9.6 -> 2.0 ms with their export.

constexpr int kSort32 = 16;  // longest list that is sorted in registers
constexpr int kMotherAtoms = 2048;  // indexes of 11 bits

typedef uint16_t ushort2v __attribute__((ext_vector_type(2)));

// Neighbouring cells of an atom, x and y in one word, z beside the atom's index in another (packed
// 16-bit arithmetic): c - own + 1 on each axis, wrapped, 0..2 for the stencil. A pair whose cells
// are further apart is out of range by its separation (a cell is wider than r_c).
struct Near32 {
    ushort2v nc_xy, nc_z;
    ushort2v before_xy, before_z;  // own cell - 1
    float w[3];
};

__device__ __forceinline__ ushort2v f32_near(uint32_t cells, ushort2v before, ushort2v nc) {
    ushort2v d = __builtin_bit_cast(ushort2v, cells) - before;
    d = __builtin_elementwise_min(d, (ushort2v)(d + nc));
    return __builtin_elementwise_min(d, (ushort2v)(d - nc));
}

__device__ __forceinline__ void f32_own(Near32& N, uint32_t xy, uint32_t z) {
    N.before_xy = __builtin_bit_cast(ushort2v, xy) - ushort2v{1, 1};
    N.before_z = ushort2v{(uint16_t)((z & 0xFFFFu) - 1u), 0};
}

// Where a partner's turn comes: (9 tz + 3 ty + tx) 2^11 + its index.
__device__ __forceinline__ uint32_t f32_turn(ushort2v xy, ushort2v z) {
    return __builtin_amdgcn_udot2(xy, ushort2v{2048, 6144},
                                  __builtin_amdgcn_udot2(z, ushort2v{18432, 1}, 0u, false), false);
}

template <int APT>
__device__ __forceinline__ void f32_publish(const F64Lds& S, const SysDev& sys, int n,
                                            const uint16_t (&atom)[APT], const double (&x)[APT],
                                            const double (&y)[APT], const double (&z)[APT]) {
    float4* u = (float4*)S.xy;
    uint32_t* uz = (uint32_t*)S.z;
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        const int a = threadIdx.x + j * blockDim.x;
        if (a < n) {
            const int cx = cell_coord(x[j], sys.inv_w[0], sys.nc[0]);
            const int cy = cell_coord(y[j], sys.inv_w[1], sys.nc[1]);
            const int cz = cell_coord(z[j], sys.inv_w[2], sys.nc[2]);
            u[a] = make_float4((float)(x[j] - (double)cx * sys.w[0]),
                               (float)(y[j] - (double)cy * sys.w[1]),
                               (float)(z[j] - (double)cz * sys.w[2]),
                               __int_as_float(cx | (cy << 16)));
            uz[a] = (uint32_t)cz | ((uint32_t)atom[j] << 16);
        }
    }
}

struct Sum32 {
    float x, y, z, w;
};

struct Pair32 {
    float x, y, z, fs;
};

// One pair's separation and force over it; whether it is in range (the force is 0 if not).
__device__ __forceinline__ bool f32_separation(Pair32& d, const Near32& N, const float4& ui,
                                               const float4& uj, ushort2v xy, ushort2v z, bool live,
                                               float rc2, float ca) {
    d.x = (ui.x - uj.x) + N.w[0] * (1.0f - (float)xy.x);
    d.y = (ui.y - uj.y) + N.w[1] * (1.0f - (float)xy.y);
    d.z = (ui.z - uj.z) + N.w[2] * (1.0f - (float)z.x);
    const float r2 = d.x * d.x + d.y * d.y + d.z * d.z;
    const bool in = live & (r2 < rc2);
    const float inv = recip(r2);
    const float s3 = inv * inv * inv;
    d.fs = in ? s3 * (48.0f * s3 - 24.0f * ca) * inv : 0.0f;
    return in;
}

__device__ __forceinline__ void f32_add(Sum32& g, const Pair32& d) {
    g.x += d.fs * d.x;
    g.y += d.fs * d.y;
    g.z += d.fs * d.z;
    g.w += d.x * (d.fs * d.y);
}

__device__ __forceinline__ bool f32_pair(Sum32& g, const Near32& N, const float4& ui, const float4& uj,
                                         ushort2v xy, ushort2v z, bool live, float rc2, float ca) {
    Pair32 d;
    const bool in = f32_separation(d, N, ui, uj, xy, z, live, rc2, ca);
    f32_add(g, d);
    return in;
}

template <int APT>
__device__ __forceinline__ void f32_forces(const F64Lds& S, const SysDev& sys, const List64& L, int n,
                                           const int (&nh)[APT], bool rebuilt, float (&fx)[APT],
                                           float (&fy)[APT], float (&fz)[APT], double& w0) {
    const int t = threadIdx.x, T = blockDim.x;
    const float4* u = (const float4*)S.xy;
    const uint32_t* uz = (const uint32_t*)S.z;
    const float rc2 = (float)sys.rc2, ca = (float)sys.c_attr;
    const int stride = T * APT;
    double wacc = 0.0;
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        const int a = t + j * T;
        const bool own = a < n;
        const int me = own ? a : 0;
        const float4 ui = u[me];
        Near32 N;
        N.nc_xy = ushort2v{(uint16_t)sys.nc[0], (uint16_t)sys.nc[1]};
        N.nc_z = ushort2v{(uint16_t)sys.nc[2], 0};
#pragma unroll
        for (int q = 0; q < 3; ++q) N.w[q] = (float)sys.w[q];
        f32_own(N, __float_as_uint(ui.w), uz[me]);
        uint16_t* list = S.list + (t * APT + j);
        const bool over = own && nh[j] > kF64Cap;
        const int len = over || !own ? 0 : nh[j];
        auto turn_of = [&](int id) {
            return f32_turn(f32_near(__float_as_uint(u[id].w), N.before_xy, N.nc_xy),
                            f32_near(uz[id], N.before_z, N.nc_z));
        };
        Sum32 g{0.f, 0.f, 0.f, 0.f};
        // the list in order; true if a partner in range came after one whose turn is later
        auto pass = [&](int count) {
            bool late = false;
            uint32_t last = 0;
            const int first = 0 < count ? list[0] : me;
            float4 v = u[first];
            uint32_t vz = uz[first];
            int idn = 1 < count ? list[stride] : me;
            for (int k = 0; __builtin_amdgcn_ballot_w64(k < count) != 0; ++k) {
                const float4 uj = v;
                const uint32_t ujz = vz;
                v = u[idn];
                vz = uz[idn];
                const int ahead = list[min(k + 2, kF64Cap - 1) * stride];
                idn = k + 2 < count ? ahead : me;
                const ushort2v xy = f32_near(__float_as_uint(uj.w), N.before_xy, N.nc_xy);
                const ushort2v z = f32_near(ujz, N.before_z, N.nc_z);
                const bool in = f32_pair(g, N, ui, uj, xy, z, k < count, rc2, ca);
                const uint32_t at = f32_turn(xy, z);
                late = late | (in & (at < last));
                last = in ? at : last;
            }
            return late;
        };
        if (rebuilt) {  // the list by turns, for the first time
            if (__builtin_amdgcn_ballot_w64(len > kSort32) == 0) {
                uint32_t key[kSort32];
#pragma unroll
                for (int k = 0; k < kSort32; ++k) {
                    const int id = k < len ? list[k * stride] : me;
                    key[k] = k < len ? (turn_of(id) << 11) | (uint32_t)id : 0xFFFFFFFFu;
                }
                // Batcher's odd-even merge sort
#pragma unroll
                for (int p = 1; p < kSort32; p *= 2)
#pragma unroll
                    for (int k = p; k >= 1; k /= 2)
#pragma unroll
                        for (int i = k % p; i + k < kSort32; i += 2 * k)
#pragma unroll
                            for (int q = 0; q < k; ++q)
                                if (i + q + k < kSort32 && (i + q) / (2 * p) == (i + q + k) / (2 * p)) {
                                    const uint32_t lo = min(key[i + q], key[i + q + k]);
                                    key[i + q + k] = max(key[i + q], key[i + q + k]);
                                    key[i + q] = lo;
                                }
#pragma unroll
                for (int k = 0; k < kSort32; ++k)
                    if (k < len) list[k * stride] = (uint16_t)(key[k] & 2047u);
            } else {
                uint32_t top = len > 0 ? turn_of(list[0]) : 0u;
                for (int k = 1; k < len; ++k) {
                    const int id = list[k * stride];
                    const uint32_t at = turn_of(id);
                    if (at >= top) {
                        top = at;
                        continue;
                    }
                    int m = k - 1;
                    for (; m >= 0; --m) {
                        const int before = list[m * stride];
                        if (turn_of(before) <= at) break;
                        list[(m + 1) * stride] = (uint16_t)before;
                    }
                    list[(m + 1) * stride] = (uint16_t)id;
                }
            }
        }
        const bool late = pass(len);
        // a lane whose partners came out of turn: the wave takes its list, an entry a lane, sorts
        // it by rank and adds up its pairs in turn
        for (uint64_t todo = __builtin_amdgcn_ballot_w64(late); todo != 0; todo &= todo - 1) {
            const int b = __builtin_ctzll(todo), lane = t & 63;
            const int count = __builtin_amdgcn_readlane(len, b), it = __builtin_amdgcn_readlane(me, b);
            uint16_t* row = S.list + ((t - lane + b) * APT + j);
            const float4 ub = u[it];
            Near32 B = N;
            f32_own(B, __float_as_uint(ub.w), uz[it]);
            const bool live = lane < count;
            const int id = live ? row[lane * stride] : it;
            const uint32_t at = f32_turn(f32_near(__float_as_uint(u[id].w), B.before_xy, B.nc_xy),
                                         f32_near(uz[id], B.before_z, B.nc_z));
            int rank = 0;
            for (int q = 0; q < count; ++q)
                rank += (uint32_t)__builtin_amdgcn_readlane((int)at, q) < at ? 1 : 0;
            if (live) row[rank * stride] = (uint16_t)id;
            // (one wave's LDS operations complete in order; the other lanes' stores are news to
            // the compiler)
            __builtin_amdgcn_wave_barrier();
            asm volatile("" ::: "memory");
            const int mine = live ? row[lane * stride] : it;
            const float4 uj = u[mine];
            Pair32 d;
            const bool in = f32_separation(d, B, ub, uj, f32_near(__float_as_uint(uj.w), B.before_xy, B.nc_xy),
                                           f32_near(uz[mine], B.before_z, B.nc_z), live, rc2, ca);
            Sum32 sum{0.f, 0.f, 0.f, 0.f};
            for (uint64_t hits = __builtin_amdgcn_ballot_w64(in); hits != 0; hits &= hits - 1) {
                const int w = __builtin_ctzll(hits);
                auto of = [&](float v) {
                    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), w));
                };
                f32_add(sum, Pair32{of(d.x), of(d.y), of(d.z), of(d.fs)});
            }
            if (lane == b) g = sum;
        }
        // an atom whose list goes beyond LDS: its partners in the list's order, summed in FP64 (any
        // order gives the same FP32 force to a rounding)
        if (__builtin_amdgcn_ballot_w64(over) != 0) {
            double sx = 0.0, sy = 0.0, sz = 0.0, sw = 0.0;
            auto see = [&](int m, bool live) {
                const float4 uj = u[m];
                Pair32 d;
                (void)f32_separation(d, N, ui, uj, f32_near(__float_as_uint(uj.w), N.before_xy, N.nc_xy),
                                     f32_near(uz[m], N.before_z, N.nc_z), live & (m != me), rc2, ca);
                sx += (double)d.fs * (double)d.x;
                sy += (double)d.fs * (double)d.y;
                sz += (double)d.fs * (double)d.z;
                sw += (double)d.x * ((double)d.fs * (double)d.y);
            };
            const bool listed = over && nh[j] < kF64Over;
            for (int k = 0; k < kF64Cap; ++k) {
                const int m = list[k * stride];
                see(listed ? m : me, listed);
            }
            f64_more(S, L, over ? nh[j] : 0, S.ext + (t * APT + j), stride, see);
            if (over) g = Sum32{(float)sx, (float)sy, (float)sz, (float)sw};
        }
        fx[j] = own ? g.x : 0.0f;
        fy[j] = own ? g.y : 0.0f;
        fz[j] = own ? g.z : 0.0f;
        wacc += own ? (double)g.w : 0.0;
    }
    w0 = 0.5 * wacc;  // every unordered pair was visited from both sides
}

template <bool F32, int APT>
__global__ void __launch_bounds__(APT == 4 ? 512 : 1024, APT == 4 ? 2 : 4)
    k_mother_lists(const MotherLaunch* ms, uint16_t* ext, int nmax, int cmax) {
    extern __shared__ __align__(16) char smem[];
    __shared__ SysDev sys;
    const MotherLaunch& m = ms[blockIdx.x];
    const F64Lds S = f64_carve(smem, ext, nmax, cmax, blockDim.x, APT);
    if (threadIdx.x == 0) sys = m.sys;
    __syncthreads();
    const int T = blockDim.x, t = threadIdx.x, n = sys.n;
    if (n > nmax || n > T * APT || n > kMotherAtoms) return;
    Cell64 H;
    H.hxx = uniform(sys.box[0]);
    H.hyy = uniform(sys.box[1]);
    H.hzz = uniform(sys.box[2]);
    H.hxy = 0.0;
    H.ixx = uniform(1.0 / sys.box[0]);
    H.iyy = uniform(1.0 / sys.box[1]);
    H.izz = uniform(1.0 / sys.box[2]);
    double x[APT], y[APT], z[APT], px[APT], py[APT], pz[APT];
    std::conditional_t<F32, float, double> fx[APT], fy[APT], fz[APT];
    float path[APT];
    int nh[APT], longest = 0;
    List64 L{};
    double* st = m.state;
    uint16_t atom[APT];  // the state's atom behind the thread's atom j
    {
        // deal the atoms to the threads in cell order
#pragma unroll
        for (int j = 0; j < APT; ++j) {
            const int a = t + j * T;
            const bool v = a < n;
            x[j] = v ? st[a] : 0.0;
            y[j] = v ? st[n + a] : 0.0;
            z[j] = v ? st[2 * n + a] : 0.0;
        }
        const Grid64 g = f64_grid(H, 0.0, H.hxx, sys.rc, cmax);
        int place[APT], cell[APT];
        float cart[APT][3];
        f64_sort<kFlowShear, APT>(S, H, g, n, x, y, z, place, cell, cart);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < APT; ++j)
            if (cell[j] >= 0) S.sid[place[j]] = (uint16_t)(t + j * T);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < APT; ++j) {
            const int a = t + j * T;
            atom[j] = a < n ? S.sid[a] : 0;
        }
        __syncthreads();  // the build reuses these bytes
    }
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        const bool v = t + j * T < n;
        const double* q = st + atom[j];
        x[j] = v ? q[0] : 0.0;
        y[j] = v ? q[n] : 0.0;
        z[j] = v ? q[2 * (size_t)n] : 0.0;
        px[j] = v ? q[3 * (size_t)n] : 0.0;
        py[j] = v ? q[4 * (size_t)n] : 0.0;
        pz[j] = v ? q[5 * (size_t)n] : 0.0;
        path[j] = 0.0f;
        nh[j] = 0;
    }
    double zeta = *m.zeta, pp = 0.0;
    const double h = sys.dt, tau = 0.5 * h, gT = m.nf * m.temperature, iq = 1.0 / m.q;
    const int64_t chunks = m.n_chunks > 0 ? m.n_chunks : 1, each = m.steps_per_chunk;
    const int64_t total = chunks * each;
    int64_t in_chunk = 0, ch = 0;
    auto put = [&](double* q, int j) {
        q[0] = x[j];
        q[n] = y[j];
        q[2 * (size_t)n] = z[j];
        q[3 * (size_t)n] = px[j];
        q[4 * (size_t)n] = py[j];
        q[5 * (size_t)n] = pz[j];
    };
    auto snapshot = [&]() {
        if (m.snap_zeta != nullptr && t == 0) m.snap_zeta[ch] = zeta;
        if (m.snapshots != nullptr) {
            double* dst = m.snapshots + (size_t)ch * 6 * (size_t)n;
#pragma unroll
            for (int j = 0; j < APT; ++j) {
                if (t + j * T < n) put(dst + atom[j], j);
            }
        }
        ++ch;
    };
    // step -1: the forces and the momentum sum of the start state
    for (int64_t s = -1; s < total; ++s) {
        const bool start = s < 0;
        double c = 1.0;
        float most = 0.0f;
        if (!start) {
            zeta += tau * (pp - gT) * iq;
            c = exp(-zeta * tau);
#pragma unroll
            for (int j = 0; j < APT; ++j) {
                px[j] = c * px[j] + tau * (double)fx[j];
                py[j] = c * py[j] + tau * (double)fy[j];
                pz[j] = c * pz[j] + tau * (double)fz[j];
                x[j] += h * px[j];
                y[j] += h * py[j];
                z[j] += h * pz[j];
                wrap_le(sys, 0.0, x[j], y[j], z[j]);
                const float ux = (float)px[j], uy = (float)py[j], uz = (float)pz[j];
                path[j] += (float)h * __builtin_sqrtf(ux * ux + uy * uy + uz * uz);
                most = fmaxf(most, path[j]);
            }
        }
        auto publish = [&]() {
            if constexpr (F32) {
                f32_publish<APT>(S, sys, n, atom, x, y, z);
            } else {
#pragma unroll
                for (int j = 0; j < APT; ++j) {
                    const int a = t + j * T;
                    if (a < n) {
                        S.xy[a] = make_double2(x[j], y[j]);
                        S.z[a] = z[j];
                    }
                }
            }
        };
        publish();
        most = wave_max_dpp(most);
        if ((t & 63) == 63) S.wmax[t >> 6] = most;
        __syncthreads();
        most = 0.0f;
        for (int w = 0; w < (T >> 6); ++w) most = fmaxf(most, S.wmax[w]);
        // (margins: FP32 paths, and FP32 separations that pass the cutoff test beyond r_c)
        const bool stale = !(sys.rc * (1.0 + 1e-6) + 2.0 * (1.0 + 1e-5) * (double)most <= L.rl);
        if (stale) {
#pragma unroll
            for (int j = 0; j < APT; ++j) path[j] = 0.0f;
            longest = f64_build<kFlowShear, APT, false>(S, H, n, cmax, sys.rc, x, y, z, L, nh);
            publish();
            __syncthreads();
        }
        double w0, w1 = 0.0;
        if constexpr (F32)
            f32_forces<APT>(S, sys, L, n, nh, stale, fx, fy, fz, w0);
        else
            f64_forces<kFlowShear, APT>(S, H, L, n, sys.rc2, sys.c_attr, nh, longest, fx, fy, fz, w0, w1);
        double mm[3] = {0.0, 0.0, w0};
#pragma unroll
        for (int j = 0; j < APT; ++j) {
            const bool own = t + j * T < n;
            if (!start) {
                px[j] += tau * (own ? (double)fx[j] : 0.0);
                py[j] += tau * (own ? (double)fy[j] : 0.0);
                pz[j] += tau * (own ? (double)fz[j] : 0.0);
            }
            mm[0] += px[j] * px[j] + py[j] * py[j] + pz[j] * pz[j];
            mm[1] += px[j] * py[j];
        }
        f64_sum<3, 4>(mm, S.red);
        if (start) {
            pp = mm[0];
        } else {
#pragma unroll
            for (int j = 0; j < APT; ++j) {
                px[j] *= c;
                py[j] *= c;
                pz[j] *= c;
            }
            pp = c * c * mm[0];
            zeta += tau * (pp - gT) * iq;
            if (m.series != nullptr && t == 0) m.series[s] = c * c * mm[1] + mm[2];
        }
        if (start ? each <= 0 : ++in_chunk == each) {
            in_chunk = 0;
            do {
                snapshot();
            } while (each <= 0 && ch < chunks);
        }
    }
#pragma unroll
    for (int j = 0; j < APT; ++j) {
        if (t + j * T < n) put(st + atom[j], j);
    }
    if (t == 0) *m.zeta = zeta;
}

// Start states of planar-elongation daughters under their mappings: bit 1 of map exchanges
// the x and y axes of positions and momenta (the box is cubic), bit 0 reverses the momenta.
// Mixed-flow daughters (mix): bit 1 exchanges the axes, then bit 0 reflects x
// (x -> L_x - x, p_x -> -p_x).
__global__ void k_spawn_pef(const double* states, int32_t n, const int32_t* state_of,
                            const int32_t* map_of, double* const* dst, int32_t mix, double lx) {
    const int d = blockIdx.x;
    const double* src = states + (size_t)state_of[d] * 6 * (size_t)n;
    double* out = dst[d];
    const int m = map_of[d];
    const bool sw = (m & 2) != 0;
    const bool rev = !mix && (m & 1) != 0;
    const bool refl = mix && (m & 1) != 0;
    const double sg = rev ? -1.0 : 1.0;
    for (int a = threadIdx.x; a < n; a += blockDim.x) {
        const double x = src[a], y = src[n + a], z = src[2 * n + a];
        const double px = src[3 * n + a], py = src[4 * n + a], pz = src[5 * n + a];
        const double xs = sw ? y : x;
        out[a] = refl ? (xs == 0.0 ? 0.0 : lx - xs) : xs;
        out[n + a] = sw ? x : y;
        out[2 * n + a] = z;
        out[3 * n + a] = (refl ? -1.0 : sg) * (sw ? py : px);
        out[4 * n + a] = sg * (sw ? px : py);
        out[5 * n + a] = sg * pz;
    }
}


}  // namespace

size_t flow64_ext_bytes(int threads, int apt, int grid) {
    return sizeof(uint16_t) * (size_t)kF64Ext * threads * apt * grid;
}

namespace {
// Neighbours an atom of a uniform fluid has within the list radius.
double flow64_neighbours(const SysDev& S) {
    const double rl = S.rc * (1.0 + kF64Skin);
    return 4.18879020478639 * rl * rl * rl * (S.n / S.volume);
}
}  // namespace

// Shape of a launch. Atoms per thread: the fewest with which every daughter of the batch is on a
// CU at once (registers: 16 waves of 128, or 8 of 256 with four atoms; and the LDS): the steps
// of a daughter are a latency chain that more waves shorten. A batch that fills the chip either
// way takes four: every wave repeats the step's scalars, so half the waves do it half as often
// (N = 2048, 1024 daughters x 50 steps, two and four: shear 3.99 and 3.69 ms, elongation 4.35 and
// 3.60, mixed flow 4.88 and 3.81). So does a small batch of more than 1536 atoms, whose two-atom build
// would keep 13 to 16 waves waiting for its spills (256 daughters x 50 steps, shear, elongation, mixed:
// N = 2048 1.09, 1.17, 1.31 and 0.99, 0.98, 1.06 ms; N = 1600 1.03, 1.06, 1.21 and 0.99, 0.97, 1.01; but
// N = 1500 0.90, 0.92, 1.06 and 0.98, 0.98, 1.04), except elongation with Nose-Hoover, whose spills are
// fewest (N = 1600 0.83 and 0.87 ms, N = 2048 0.88 and 0.89).
bool flow64_shape(int flow, int thermo, int nmax, int cells, int n_jobs, int num_cu, size_t max_lds,
                  Flow64Shape* out) {
    if (nmax > kPefMaxAtoms) return false;
    bool found = false;
    for (int apt = nmax > 1536 && !(flow == kFlowElong && thermo) ? 4 : 1; apt <= 4; apt *= 2) {
        Flow64Shape f{};
        f.apt = apt;
        f.threads = ((nmax + apt - 1) / apt + 63) / 64 * 64;
        if (f.threads > (apt == 4 ? 512 : kMaxThreads)) continue;
        // half cells beyond the atoms' number gain nothing
        f.cmax = 2 * cells < nmax + 64 ? (cells < 27 ? 54 : 2 * cells) : nmax + 64;
        const size_t lds = f64_plan(nmax, f.cmax, f.threads, apt).total + 1024;
        if (lds > max_lds) continue;
        const int waves = (apt == 4 ? 8 : 16) / (f.threads / 64), held = (int)(max_lds / lds);
        int fit = waves < held ? waves : held;
        if (fit < 1) fit = 1;
        f.grid = n_jobs < fit * num_cu ? n_jobs : fit * num_cu;
        *out = f;
        found = true;
        if (fit * num_cu >= n_jobs) break;
    }
    return found;
}

// Lists wherever a workgroup holds them (the cell form rebuilds its grid and scans 27 cells in FP64
// every step: N = 2048, 1024 daughters x 50 steps 13.4 ms, lists 3.74) and has room in LDS for half as
// many neighbours again as the list radius holds on average, so that few atoms of a uniform fluid need
// the global part. Whatever other daughters share the call.
bool flow64_takes(const SysDev& S, size_t max_lds) {
    Flow64Shape f{};
    return 1.5 * flow64_neighbours(S) <= kF64Cap && flow64_shape(kFlowShear, 0, S.n, 1 << 28, 1, 1, max_lds, &f);
}

// The carried-flow batches taken: a cell grid at r_c fits one workgroup's LDS beside the state. Sparser
// systems are refused, as they always were (k_flow64 itself would hold them).
size_t pef_grid_bytes(int nmax, int cmax) {
    return 3 * f64_align(sizeof(double) * (size_t)nmax) + f64_align(sizeof(int32_t) * ((size_t)cmax + 1)) +
           f64_align(sizeof(int32_t) * (size_t)cmax) + f64_align(sizeof(uint16_t) * (size_t)nmax) +
           sizeof(double) * (kMaxWaves * kRedSlots + kRedSlots) + 64 +
           sizeof(uint16_t) * kF64Cap * kMaxThreads;
}

int pef_max_cells(double volume, double rc) {
    return (int)floor(volume / (rc * rc * rc));
}

namespace {
template <int F, bool NH, int APT>
hipError_t launch_flow64_t(const PefLaunch& L, hipStream_t s) {
    const size_t lds = f64_plan(L.nmax, L.cmax, L.threads, APT).total;
    (void)hipFuncSetAttribute((const void*)k_flow64<F, NH, APT>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((k_flow64<F, NH, APT>), dim3(L.grid), dim3(L.threads), lds, s, L);
    return hipGetLastError();
}

template <int F, bool NH>
hipError_t launch_flow64_a(const PefLaunch& L, hipStream_t s) {
    switch (L.apt) {
        case 1: return launch_flow64_t<F, NH, 1>(L, s);
        case 2: return launch_flow64_t<F, NH, 2>(L, s);
        case 4: return launch_flow64_t<F, NH, 4>(L, s);
    }
    return hipErrorInvalidValue;
}

template <int F>
hipError_t launch_flow64_f(const PefLaunch& L, hipStream_t s) {
    return L.thermo ? launch_flow64_a<F, true>(L, s) : launch_flow64_a<F, false>(L, s);
}
}  // namespace

hipError_t launch_flow64(const PefLaunch& L, hipStream_t s) {
    if (L.n_jobs <= 0) return hipSuccess;
    if (L.threads < 64 || L.threads > (L.apt == 4 ? 512 : kMaxThreads) || L.threads % 64 != 0 ||
        L.nmax > L.threads * L.apt || L.nmax > kPefMaxAtoms || L.cmax < 54 || L.grid < 1)
        return hipErrorInvalidValue;
    const hipError_t e = launch_zero_int(L.queue, s);
    if (e != hipSuccess) return e;
    switch (L.flow) {
        case 0: return launch_flow64_f<kFlowShear>(L, s);
        case 1: return launch_flow64_f<kFlowElong>(L, s);
        case 2: return launch_flow64_f<kFlowMixed>(L, s);
    }
    return hipErrorInvalidValue;
}

// Mothers over lists: where an atom's neighbours leave its list room (as for daughters), the lists
// and a grid fit one workgroup's LDS, and (FP32 form) the stencil is three cells a side and a cell
// and an index fit one word. Otherwise (long cutoffs, more than 2048 atoms) the cell form. One atom
// a thread as far as 1024 threads go, as the steps are a latency chain; two beyond, and four with FP64
// forces of more than 1536 atoms, whose two-atom build spills 57 registers and the four-atom one two
// (100 steps, two and four: N = 1025 1.19 and 1.49 ms, N = 1500 1.34 and 1.58, N = 1800 1.68 and 1.64,
// N = 2048 1.64 and 1.61; FP32 forces spill 117 and 111: N = 1025 1.69 and 2.20, N = 1500 1.96 and 2.45,
// N = 1800 2.35 and 2.46, N = 2048 2.33 and 2.56).
bool mother_lists(const SysDev& S, size_t max_lds, MotherLaunch* L) {
    L->list_lds = 0;
    if (S.n > kMotherAtoms || 1.5 * flow64_neighbours(S) > kF64Cap) return false;
    for (int a = 0; a < 3; ++a)
        if (S.nc[a] < 3 || S.nc[a] > 63 || !(S.w[a] > S.rc * (1.0 + 2e-6))) return false;
    const int cells = pef_max_cells(S.volume, S.rc);
    L->list_cells = 2 * cells < S.n + 64 ? (cells < 27 ? 54 : 2 * cells) : S.n + 64;
    L->list_apt = S.n <= kMaxThreads ? 1 : (L->precision == 0 && S.n > 1536 ? 4 : 2);
    L->list_threads = ((S.n + L->list_apt - 1) / L->list_apt + 63) / 64 * 64;
    const size_t lds = f64_plan(S.n, L->list_cells, L->list_threads, L->list_apt).total;
    if (lds + sizeof(SysDev) + 256 > max_lds) return false;
    L->list_lds = lds;
    return true;
}

namespace {
// Mothers of a launch: as many whole rounds of the chip's CUs as have their list scratch in 512 MB
// (1024 of N = 2048); more follow in further launches over the same scratch.
int mothers_at_once(const MotherLaunch& m) {
    const size_t most = ((size_t)512 << 20) / flow64_ext_bytes(m.list_threads, m.list_apt, 1);
    return (int)(most / 256 * 256);
}

template <bool F32, int APT>
hipError_t launch_mother_lists_t(const MotherLaunch* dev_ms, int count, const MotherLaunch& m,
                                 hipStream_t s) {
    (void)hipFuncSetAttribute((const void*)k_mother_lists<F32, APT>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)m.list_lds);
    const int held = mothers_at_once(m);
    for (int b = 0; b < count; b += held) {
        const int part = count - b < held ? count - b : held;
        hipLaunchKernelGGL((k_mother_lists<F32, APT>), dim3(part), dim3(m.list_threads), m.list_lds, s,
                           dev_ms + b, m.ext, m.sys.n, m.list_cells);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
}  // namespace

size_t mother_ext_bytes(const MotherLaunch& m, int count) {
    const int held = mothers_at_once(m);
    return flow64_ext_bytes(m.list_threads, m.list_apt, count < held ? count : held);
}

hipError_t launch_mother_lists(const MotherLaunch* dev_ms, int count, const MotherLaunch& m,
                               hipStream_t s) {
    switch (m.list_apt * 2 + (m.precision == 0 ? 0 : 1)) {
        case 2: return launch_mother_lists_t<false, 1>(dev_ms, count, m, s);
        case 3: return launch_mother_lists_t<true, 1>(dev_ms, count, m, s);
        case 4: return launch_mother_lists_t<false, 2>(dev_ms, count, m, s);
        case 5: return launch_mother_lists_t<true, 2>(dev_ms, count, m, s);
        case 8: return launch_mother_lists_t<false, 4>(dev_ms, count, m, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_spawn_pef(const double* states, int32_t n, const int32_t* state_of,
                            const int32_t* map_of, double* const* dst, int32_t n_daughters,
                            int32_t mix, double lx, hipStream_t s) {
    if (n_daughters <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_spawn_pef, dim3(n_daughters), dim3(256), 0, s, states, n, state_of,
                       map_of, dst, mix, lx);
    return hipGetLastError();
}

}  // namespace ttcf
