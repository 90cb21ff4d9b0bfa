// ttcf_channel.hip -- gfx950 kernels of the confined-channel example (Eq. system2,
// Eq. TTCF2): a Lennard-Jones liquid between two walls whose atoms are tethered to lattice
// sites moving at +-v/2 along x, with a Nose-Hoover thermostat on the wall atoms.
//
// One workgroup integrates one trajectory at a time. The state (FP64 r and p, FP32 forces)
// stays in global memory: 18000 atoms do not fit in LDS. A step is a few coalesced passes
// over the atoms. Pair separations come from 32-bit fixed-point coordinates (periodic in x
// and z, so wrapped integer differences are minimum images; plain in y). Verlet lists of
// radius r_c + skin live in global scratch, rebuilt through an LDS counting sort when the
// largest path length since the last build reaches skin / 2. All reductions have a fixed
// order, and the momentum profile is summed as 64-bit fixed point: results are
// deterministic.
//
// What bounds a step is vector arithmetic: the list build (one step in eight or so), then the
// force pass. Both walk the atoms in list-grid order with the slots around them in an LDS window
// (ch_walk), so that no candidate or neighbour is gathered from global memory; a system whose
// layers do not fit the window takes the gathering form of both (ch_rebuild_scan,
// ch_forces_global), in the same order and with the same bits. Measured on one MI355X, cycles of
// an 18000-atom trajectory on its CU, gathering form -> window: build 8.1M -> 2.9M, force pass
// 1.41M -> 1.00M (1024 lanes, 245 vector instructions and 8 quarter-rate reciprocals for 8 pairs);
// 256 daughters of 20 steps, 17 of them with a build: 77.0 -> 32.3 ms. The rest of a step is two
// passes over momenta and forces at the rate of HBM (0.31M cycles).
#include <hip/hip_runtime.h>

#include "ttcf_channel.h"

namespace ttcf {

namespace {

constexpr double kProfileScale = 1099511627776.0;  // 2^40: fixed point of the profile sums
constexpr int kChUnroll = 8;                         // list entries per trip of the force loop
constexpr int kChScanUnroll = 8;                     // candidates per trip of the list build
constexpr int kChWin = 8192;                         // window slots (entries: 8 * place, 16 bits)
constexpr int kChTail = 32;                          // of the list build, repeated past its end
constexpr uint32_t kChWinXy = 4 * kChWin, kChWinType = 12 * kChWin;
constexpr size_t kChWinBytes = 13 * (size_t)kChWin;

// LDS by its address. The kernels hold no other LDS than the block that they are launched with
// (ch_window_at_zero), so it starts at 0 and a window place is an address (through the block's symbol every access
// adds its base, two instructions a pair of the force loop).
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
template <typename V>
using ChShared = const __attribute__((address_space(3))) V;

constexpr uint16_t kChNearWall = 0x8000;             // in ncnt: a wall atom, or one is listed

__device__ __forceinline__ uint32_t fixp(double v, double scale) {
    return (uint32_t)(int64_t)rint(v * scale);
}

__device__ __forceinline__ int cell_of(uint32_t q, int nc) {
    return (int)(((uint64_t)q * (uint64_t)nc) >> 32);
}

__device__ __forceinline__ double min_image(double d, double l) { return d - l * rint(d / l); }

template <int K>
__device__ __forceinline__ void ch_block_sum(double (&v)[K], double* red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double x = v[k];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        v[k] = x;
    }
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) red[wave * K + k] = v[k];
    __syncthreads();
    if (threadIdx.x < K) {
        double s = 0.0;
        for (int w = 0; w < nw; ++w) s += red[w * K + threadIdx.x];
        red[kChMaxWaves * K + threadIdx.x] = s;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = red[kChMaxWaves * K + k];
    __syncthreads();
}

__device__ __forceinline__ float ch_block_max(float v, float* wmax) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = v;
    __syncthreads();
    float m = 0.f;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) m = fmaxf(m, wmax[w]);
    __syncthreads();
    return m;
}

// Exclusive scan of cnt[0..C) into start[0..C) and into cnt (placement cursors).
__device__ void ch_scan(int32_t* cnt, int32_t* start, int C, int32_t* ws) {
    const int T = blockDim.x, t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6, nw = T >> 6;
    const int chunk = (C + T - 1) / T;
    const int b = min(t * chunk, C), e = min(b + chunk, C);
    int local = 0;
    for (int c = b; c < e; ++c) local += cnt[c];
    int x = local;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) ws[wave] = x;
    __syncthreads();
    if (t == 0) {
        int run = 0;
        for (int w = 0; w < nw; ++w) {
            const int v = ws[w];
            ws[w] = run;
            run += v;
        }
    }
    __syncthreads();
    int run = ws[wave] + x - local;
    for (int c = b; c < e; ++c) {
        const int v = cnt[c];
        start[c] = run;
        cnt[c] = run;
        run += v;
    }
    __syncthreads();
}

struct ChLds {
    int32_t* cnt;      // [cmax]
    int32_t* start;    // [cmax + 1]
    uint16_t* sid;     // [nmax + 4]
    double* red;       // block reductions
    int32_t* ws;       // [kChMaxWaves]
    float* wmax;       // [kChMaxWaves]
    unsigned long long* bins;  // [kChMaxBins] profile sums (fixed point)
    int32_t* misc;     // [8]: job, list overflow, out of range, window of two chunks and of one,
                       // highest bottom wall atom, lowest top wall atom (fixed-point y / 2)
    // the window, if there is one (at fixed places, so that its addresses are the entries' own):
    // positions of the force pass, or in the same bytes the 16-bit ones of the list build
    uint32_t* wz;      // [kChWin] Z
    uint2* wxy;        // [kChWin] X, Y
    uint8_t* wtype;    // [kChWin] atom type
    uint2* w16;        // [kChWin + kChTail] 16-bit x, y | z, 0
    uint32_t* wall;    // [n / 32 + 2] wall atoms by slot, the first slot of a word in its top bit
    bool win;
};

__host__ __device__ inline size_t ch_align(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct ChPlan {
    size_t cnt, start, sid, red, ws, wmax, bins, misc, wall, total;
};

__host__ __device__ inline ChPlan ch_plan(int nmax, int cmax, bool win) {
    ChPlan p;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        off = ch_align(off, 16);
        const size_t at = off;
        off += bytes;
        return at;
    };
    take(win ? kChWinBytes : 0);
    p.cnt = take(4 * (size_t)cmax);
    p.start = take(4 * ((size_t)cmax + 1));
    p.sid = take(2 * ((size_t)nmax + 4));
    p.red = take(sizeof(double) * (kChMaxWaves + 1) * kChRed);
    p.ws = take(4 * kChMaxWaves);
    p.wmax = take(4 * kChMaxWaves);
    p.bins = take(8 * kChMaxBins);
    p.misc = take(32);
    p.wall = take(win ? 4 * ((size_t)nmax / 32 + 2) : 0);
    p.total = ch_align(off, 128);
    return p;
}

__device__ inline ChLds ch_carve(char* base, int nmax, int cmax, bool win) {
    const ChPlan p = ch_plan(nmax, cmax, win);
    ChLds L;
    L.cnt = (int32_t*)(base + p.cnt);
    L.start = (int32_t*)(base + p.start);
    L.sid = (uint16_t*)(base + p.sid);
    L.red = (double*)(base + p.red);
    L.ws = (int32_t*)(base + p.ws);
    L.wmax = (float*)(base + p.wmax);
    L.bins = (unsigned long long*)(base + p.bins);
    L.misc = (int32_t*)(base + p.misc);
    L.wz = (uint32_t*)base;
    L.wxy = (uint2*)(base + kChWinXy);
    L.wtype = (uint8_t*)(base + kChWinType);
    L.wall = (uint32_t*)(base + p.wall);
    L.w16 = (uint2*)base;
    L.win = win;
    return L;
}

// Per-workgroup global scratch: fixed-point positions in atom order and in list-grid order,
// lists, list lengths, path lengths. Lists and list lengths are indexed by list-grid slot
// (the position of the atom in the counting sort) and hold slots, or window places times eight
// where the window is in use, so that the force pass walks the atoms cell by cell and a wave's
// gathers stay in a few neighbouring cells.
struct ChScratch {
    uint4* posq;       // [n] by atom  (X, Y, Z, type: 0 fluid, 1 bottom wall, 2 top wall)
    uint4* posq_s;     // [n] by slot: posq_s[i] = posq[sid[i]]
    uint16_t* nbr;     // [ch_rows(kmax)][n] by slot
    uint16_t* ncnt;    // [n] by slot: list length, and kChNearWall
    float* path;       // [n] by atom
};

// list rows: the capacity, the force pass's whole trips, and a sink for rejected candidates
__host__ __device__ inline int ch_rows(int kmax) { return (kmax + kChUnroll) / kChUnroll * kChUnroll; }

__host__ __device__ inline size_t ch_scratch_bytes(int nmax, int kmax) {
    return 2 * ch_align(16 * (size_t)nmax, 256) + ch_align(2 * (size_t)ch_rows(kmax) * nmax, 256) +
           ch_align(2 * (size_t)nmax, 256) + ch_align(4 * (size_t)nmax, 256);
}

__device__ inline ChScratch ch_scratch(char* base, int nmax, int kmax) {
    ChScratch s;
    size_t off = 0;
    s.posq = (uint4*)(base + off);
    off += ch_align(16 * (size_t)nmax, 256);
    s.posq_s = (uint4*)(base + off);
    off += ch_align(16 * (size_t)nmax, 256);
    s.nbr = (uint16_t*)(base + off);
    off += ch_align(2 * (size_t)ch_rows(kmax) * nmax, 256);
    s.ncnt = (uint16_t*)(base + off);
    off += ch_align(2 * (size_t)nmax, 256);
    s.path = (float*)(base + off);
    return s;
}

__device__ __forceinline__ uint32_t atom_type(const ChannelDev& S, int a) {
    return a < S.n_fluid ? 0u : (a < S.n_fluid + S.n_wall / 2 ? 1u : 2u);
}

// fixed-point position of one atom; flags an atom that left [0, y_extent)
__device__ __forceinline__ void ch_publish_atom(const ChannelDev& S, int a, double x, double y,
                                                double z, const ChScratch& G, const ChLds& L) {
    if (!(y >= 0.0) || !(y < S.y_extent)) L.misc[2] = 1;
    const double yc = fmin(fmax(y, 0.0), S.y_extent * (1.0 - 1e-15));
    G.posq[a] = make_uint4(fixp(x, S.fix_scale[0]), fixp(yc, S.fix_scale[1]),
                           fixp(z, S.fix_scale[2]), atom_type(S, a));
}

__device__ void ch_publish(const ChannelDev& S, const double* r, const ChScratch& G,
                           const ChLds& L) {
    const int n = S.n;
    for (int a = threadIdx.x; a < n; a += blockDim.x)
        ch_publish_atom(S, a, r[a], r[n + a], r[2 * n + a], G, L);
}

// positions in list-grid order for the slots of the last list build (sid stays in LDS)
__device__ __forceinline__ void ch_gather_sorted(const ChannelDev& S, const ChScratch& G,
                                                 const ChLds& L) {
    for (int i = threadIdx.x; i < S.n; i += blockDim.x) G.posq_s[i] = G.posq[L.sid[i]];
}

__device__ __forceinline__ void ch_sep(const uint4& qa, const uint4& qb, const ChannelDev& S,
                                       float& dx, float& dy, float& dz) {
    dx = (float)(int32_t)(qa.x - qb.x) * S.fix_unit[0];
    dy = (float)(int32_t)(qa.y - qb.y) * S.fix_unit[1];
    dz = (float)(int32_t)(qa.z - qb.z) * S.fix_unit[2];
}

// Window place of slot j, `image` slots further on.
__device__ __forceinline__ int ch_place(int j, int image) { return (j + image) & (kChWin - 1); }

// Place of list entry k of slot i in nbr.
__device__ __forceinline__ size_t ch_entry(int k, int n, int i) { return (size_t)k * n + i; }

// Entries past a list's end, up to a whole trip of the force pass, name the atom itself (they add
// nothing there).
__device__ __forceinline__ void ch_pad(const ChScratch& G, int count, int n, int i, uint16_t self) {
    for (int k = count; k % kChUnroll != 0; ++k) G.nbr[ch_entry(k, n, i)] = self;
}

// Slots that atoms of cell row w (the cells of one y and z; rows and slots ascend with z, then
// with y) see: from the first one of the row below in the layer before to the last one of the row
// above in the layer after. The layers across the z edge lie n slots before or after.
__device__ __forceinline__ int ch_need_first(const ChannelDev& S, const ChLds& L, int w) {
    const int nc0 = S.lc[0], nc1 = S.lc[1], z = w / nc1, y = max(w - z * nc1 - 1, 0);
    return z > 0 ? L.start[((z - 1) * nc1 + y) * nc0] : L.start[((S.lc[2] - 1) * nc1 + y) * nc0] - S.n;
}

__device__ __forceinline__ int ch_need_end(const ChannelDev& S, const ChLds& L, int w) {
    const int nc0 = S.lc[0], nc1 = S.lc[1], z = w / nc1, y = min(w - z * nc1 + 1, nc1 - 1) + 1;
    return z + 1 < S.lc[2] ? L.start[((z + 1) * nc1 + y) * nc0] : L.start[y * nc0] + S.n;
}

// Counting sort into the list grid (LDS): the atoms of a cell in ascending id order, so that list
// order, and every force sum, does not depend on the order in which the placement atomics ran.
__device__ void ch_sort(const ChannelDev& S, const ChScratch& G, const ChLds& L) {
    const int n = S.n, T = blockDim.x, t = threadIdx.x;
    const int nc0 = S.lc[0], nc1 = S.lc[1], nc2 = S.lc[2];
    const int C = nc0 * nc1 * nc2;
    for (int c = t; c < C; c += T) L.cnt[c] = 0;
    if (t == 0) {
        L.misc[1] = 0;
        L.misc[3] = 0;
        L.misc[4] = 0;
        L.misc[5] = -1;
        L.misc[6] = 0x7FFFFFFF;
    }
    __syncthreads();
    for (int a = t; a < n; a += T) {
        const uint4 q = G.posq[a];
        const int c = cell_of(q.x, nc0) + nc0 * (cell_of(q.y, nc1) + nc1 * cell_of(q.z, nc2));
        atomicAdd(&L.cnt[c], 1);
        if (q.w == 1u) atomicMax(&L.misc[5], (int)(q.y >> 1));
        if (q.w == 2u) atomicMin(&L.misc[6], (int)(q.y >> 1));
    }
    __syncthreads();
    ch_scan(L.cnt, L.start, C, L.ws);
    if (t == 0) L.start[C] = n;
    for (int a = t; a < n; a += T) {
        const uint4 q = G.posq[a];
        const int c = cell_of(q.x, nc0) + nc0 * (cell_of(q.y, nc1) + nc1 * cell_of(q.z, nc2));
        const int idx = atomicAdd(&L.cnt[c], 1);
        L.sid[idx] = (uint16_t)a;
    }
    __syncthreads();
    for (int c = t; c < C; c += T) {
        const int b = L.start[c], e = L.start[c + 1];
        for (int i = b + 1; i < e; ++i) {
            const uint16_t v = L.sid[i];
            int q = i - 1;
            while (q >= b && L.sid[q] > v) {
                L.sid[q + 1] = L.sid[q];
                --q;
            }
            L.sid[q + 1] = v;
        }
    }
    // slots that the window has to hold for a chunk of T atoms, and for a chunk and its successor,
    // which is loaded meanwhile
    if (L.win)
        for (int c = t; c * T < n; c += T) {
            int w0 = 0;
            while (L.start[(w0 + 1) * nc0] <= c * T) ++w0;
            int w1 = w0;
            while (L.start[(w1 + 1) * nc0] < min(n, (c + 1) * T)) ++w1;
            int w2 = w1;
            while (L.start[(w2 + 1) * nc0] < min(n, (c + 2) * T)) ++w2;
            const int first = c > 0 ? ch_need_first(S, L, w0) : ch_need_first(S, L, 0);
            atomicMax(&L.misc[4], ch_need_end(S, L, w1) - first);
            atomicMax(&L.misc[3], ch_need_end(S, L, w2) - first);
        }
    for (int a = t; a < n; a += T) G.path[a] = 0.f;
    __syncthreads();
    if (L.win) {
        for (int w = t; w < n / 32 + 2; w += T) {
            uint32_t bits = 0;
            for (int u = 0; u < 32; ++u)
                bits |= (32 * w + u < n && L.sid[32 * w + u] >= S.n_fluid) ? 0x80000000u >> u : 0u;
            L.wall[w] = bits;
        }
    }
    __syncthreads();
}

__device__ __forceinline__ bool ch_windowed(const ChLds& L) { return L.win && L.misc[4] <= kChWin; }

// Lists from the sorted positions in global memory: every slot collects the atoms within
// r_c + skin over its 27-cell neighbourhood (no images in y; wall-wall pairs are left out).
// PLACES: entries are window places, as the windowed force pass reads them.
template <bool PLACES>
__device__ void ch_rebuild_scan(const ChannelDev& S, const ChScratch& G, const ChLds& L) {
    const int n = S.n, T = blockDim.x, t = threadIdx.x;
    const int nc0 = S.lc[0], nc1 = S.lc[1], nc2 = S.lc[2];
    ch_gather_sorted(S, G, L);
    __syncthreads();
    const float rl2 = S.rl2_f;
    const int kmax = S.kmax;
    const int sink = ch_rows(kmax) - 1;
    bool over = false;
    for (int i = t; i < n; i += T) {
        const uint4 qa = G.posq_s[i];
        const int cx = cell_of(qa.x, nc0), cy = cell_of(qa.y, nc1), cz = cell_of(qa.z, nc2);
        const bool wall_a = qa.w != 0u;
        bool near = wall_a;
        int count = 0;
        auto scan = [&](int lo, int hi, int image) {
            for (int tt = lo; tt < hi; tt += kChScanUnroll) {
                int jn[kChScanUnroll];
                uint4 q[kChScanUnroll];
#pragma unroll
                for (int u = 0; u < kChScanUnroll; ++u) jn[u] = tt + u < hi ? tt + u : i;
#pragma unroll
                for (int u = 0; u < kChScanUnroll; ++u) q[u] = G.posq_s[jn[u]];
#pragma unroll
                for (int u = 0; u < kChScanUnroll; ++u) {
                    float dx, dy, dz;
                    ch_sep(qa, q[u], S, dx, dy, dz);
                    const bool both_wall = wall_a & (q[u].w != 0u);
                    const bool hit = (jn[u] != i) & !both_wall &
                                     (dx * dx + dy * dy + dz * dz < rl2);
                    const bool room = hit & (count < kmax);
                    const int place = PLACES ? ch_place(jn[u], image) << 3 : jn[u];
                    G.nbr[ch_entry(room ? count : sink, n, i)] = (uint16_t)place;
                    count += hit ? 1 : 0;
                    near = near | (hit & (q[u].w != 0u));
                }
            }
        };
        for (int dy = -1; dy <= 1; ++dy) {
            const int yy = cy + dy;
            if (yy < 0 || yy >= nc1) continue;
            for (int dz = -1; dz <= 1; ++dz) {
                int zz = cz + dz;
                const int image = zz < 0 ? -n : (zz >= nc2 ? n : 0);
                zz = zz < 0 ? zz + nc2 : (zz >= nc2 ? zz - nc2 : zz);
                const int base = nc0 * (yy + nc1 * zz);
                int x0 = cx - 1;
                if (x0 < 0) x0 += nc0;
                const int xe = x0 + 3;
                scan(L.start[base + x0], L.start[base + (xe < nc0 ? xe : nc0)], image);
                if (xe > nc0) scan(L.start[base], L.start[base + xe - nc0], image);
            }
        }
        if (count > kmax) {
            over = true;
            count = kmax;
        }
        ch_pad(G, count, n, i, (uint16_t)(PLACES ? ch_place(i, 0) << 3 : i));
        G.ncnt[i] = (uint16_t)(count | (near ? kChNearWall : 0));
    }
    if (over) L.misc[1] = 1;
    __syncthreads();
}

// Walks the slots in chunks of the workgroup's size: load(j, place) brings slot j to a place of
// the window, work(i) runs once the slots that the chunk's atoms see are in place. (Layer by layer
// instead, 1800 atoms on 1024 threads leave an eighth of the lanes idle.)
template <typename Load, typename Work>
__device__ __forceinline__ void ch_walk(const ChannelDev& S, const ChLds& L, Load load, Work work) {
    const int n = S.n, T = blockDim.x, t = threadIdx.x, nc0 = S.lc[0];
    const bool wide = L.misc[3] <= kChWin;  // the next chunk's slots displace none of this one's
    int w = 0, next = ch_need_first(S, L, 0);
    for (int c0 = 0; c0 < n; c0 += T) {
        const int c1 = min(n, c0 + T);
        while (L.start[(w + 1) * nc0] < c1) ++w;
        const int end = ch_need_end(S, L, w);
        if (!wide && c0 > 0) __syncthreads();
        for (int e = next + t; e < end; e += T)
            load(e < 0 ? e + n : (e >= n ? e - n : e), e & (kChWin - 1));
        next = max(next, end);
        __syncthreads();
        if (c0 + t < c1) work(c0 + t);
    }
}

typedef short short2v __attribute__((ext_vector_type(2)));

// 16-bit coordinates of the list build in units of about `unit` on every axis.
struct ChShort {
    int ext[3];  // units per edge
    int limit;   // squared list radius, widened by what rounding can hide
    int bottom, top;  // y at which a fluid atom may list an atom of the bottom, of the top wall
};

__device__ __forceinline__ ChShort ch_short(const ChannelDev& S, const ChLds& L) {
    ChShort c;
    const double reach = S.rc + S.skin;
    const double most = fmax(S.lx, fmax(S.y_extent, S.lz));
    const double unit = fmax(most / 30000.0, reach / 6000.0);
    c.ext[0] = (int)rint(S.lx / unit);
    c.ext[1] = (int)rint(S.y_extent / unit);
    c.ext[2] = (int)rint(S.lz / unit);
    // truncated coordinates: a separation is off by less than one unit per axis, and by the
    // edges' rounding (half a unit per edge)
    const double r = reach / unit * (1.0 + 1e-4) + 3.5;
    c.limit = (int)ceil(r * r);
    const int ir = (int)r + 2;
    c.bottom = (int)__umulhi((uint32_t)(L.misc[5] + 1) << 1, (uint32_t)c.ext[1]) + ir;
    c.top = (int)__umulhi((uint32_t)L.misc[6] << 1, (uint32_t)c.ext[1]) - ir;
    if (L.misc[5] < 0) c.bottom = -1;
    if (L.misc[6] == 0x7FFFFFFF) c.top = 0x7FFFFFFF;
    return c;
}

__device__ __forceinline__ void ch_load_short(const ChShort& c, const ChScratch& G, const ChLds& L,
                                              int j, int p) {
    const uint4 q = G.posq[L.sid[j]];
    const uint32_t x = __umulhi(q.x, (uint32_t)c.ext[0]), y = __umulhi(q.y, (uint32_t)c.ext[1]),
                   z = __umulhi(q.z, (uint32_t)c.ext[2]);
    const uint2 v = make_uint2(x | (y << 16), z);
    L.w16[p] = v;
    if (p < kChTail) L.w16[kChWin + p] = v;
}

// The list of slot i through the window.
__device__ __forceinline__ int ch_list_atom(const ChannelDev& S, const ChShort& c, const ChScratch& G,
                                            const ChLds& L, int i, bool wall, uint2 q, int cx, int cy,
                                            int cz) {
    const int n = S.n, nc0 = S.lc[0], nc1 = S.lc[1], nc2 = S.lc[2];
    const int x16 = q.x & 0xFFFF, y16 = q.x >> 16, z16 = q.y;
    constexpr uint32_t places = (uint32_t)(kChWin - 1) << 3;
    const uint32_t stride = 2u * (uint32_t)n;
    uint32_t off = 2u * (uint32_t)i;  // of the next entry
    int count = 0;
    for (int dy = -1; dy <= 1; ++dy) {
        const int yy = cy + dy;
        if (yy < 0 || yy >= nc1) continue;
        for (int dz = -1; dz <= 1; ++dz) {
            int zz = cz + dz;
            const int image = zz < 0 ? -n : (zz >= nc2 ? n : 0);
            // the layer across the edge is an edge away from its own coordinates
            const int uz = z16 + (zz < 0 ? c.ext[2] : (zz >= nc2 ? -c.ext[2] : 0));
            zz = zz < 0 ? zz + nc2 : (zz >= nc2 ? zz - nc2 : zz);
            const int base = nc0 * (yy + nc1 * zz);
            const short2v b = __builtin_bit_cast(short2v, (uint32_t)uz & 0xFFFFu);
            auto shifted = [&](int x) {
                return __builtin_bit_cast(short2v, ((uint32_t)x & 0xFFFFu) | ((uint32_t)y16 << 16));
            };
            // x cells cx - 1 .. cx + 1: from the first one on, then what lies across the edge
            const int x0 = cx > 0 ? cx - 1 : nc0 - 1, xe = x0 + 3;
            short2v a = shifted(x16 + (cx > 0 ? 0 : c.ext[0]));
            int tt = L.start[base + x0], hi = L.start[base + min(xe, nc0)];
            bool second = xe > nc0;
            if (second && tt >= hi) {
                second = false;
                tt = L.start[base];
                hi = L.start[base + xe - nc0];
                a = shifted(x16 - (cx > 0 ? c.ext[0] : 0));
            }
            while (tt < hi) {
                const int p0 = ch_place(tt, image);
                const uint2* w = L.w16 + p0;
                uint32_t mask = 0;
                auto trip = [&](int u0) {
                    // stage by stage over eight candidates: a product needs three other
                    // instructions between it and the use of its result
#pragma unroll
                    for (int h = 0; h < 16; h += 8) {
                        uint2 v[8];
                        int r2[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) v[u] = w[u0 + h + u];
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const short2v e = b - __builtin_bit_cast(short2v, v[u].y);
                            // (clamped, which changes nothing, for the form with a free result)
                            r2[u] = __builtin_amdgcn_sdot2(e, e, -c.limit, true);
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const short2v d = a - __builtin_bit_cast(short2v, v[u].x);
                            r2[u] = __builtin_amdgcn_sdot2(d, d, r2[u], true);
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            mask = __builtin_amdgcn_alignbit(mask, (uint32_t)r2[u], 31);  // the sign
                    }
                };
                trip(0);
                if (tt + 16 < hi)
                    trip(16);
                else
                    mask <<= 16;
                const int left = hi - tt;  // first candidate in the highest bit
                if (left < 32) mask &= 0xFFFFFFFFu << (32 - left);
                if (image == 0 && (uint32_t)(i - tt) < 32u) mask &= ~(0x80000000u >> (i - tt));
                if (wall) {  // no wall-wall pairs
                    const uint32_t* m = L.wall + (tt >> 5);
                    mask &= ~__funnelshift_l(m[1], m[0], tt & 31);
                }
                const uint32_t p8 = (uint32_t)p0 << 3;
                count += __builtin_popcount(mask);
                if (count > S.kmax) mask = 0u;
                while (mask != 0u) {
                    const uint32_t b0 = (uint32_t)__builtin_clz(mask);
                    mask ^= 0x80000000u >> b0;
                    *(uint16_t*)((char*)G.nbr + off) = (uint16_t)((p8 + (b0 << 3)) & places);
                    off += stride;
                }
                tt += 32;
                if (tt >= hi && second) {
                    second = false;
                    tt = L.start[base];
                    hi = L.start[base + xe - nc0];
                    a = shifted(x16 - (cx > 0 ? c.ext[0] : 0));
                }
            }
        }
    }
    return count;
}

// The lists through the window, the same entries in the same order as ch_rebuild_scan's and a few
// beyond the radius (they lie outside r_c until the next build and add nothing). Distances come
// from 16-bit coordinates with packed differences and integer dot products: a conservative
// test of five instructions a candidate, 32 candidates of a row collected in a bit mask whose
// set bits are then written out. A list that outgrows its capacity here is left to
// ch_rebuild_scan, which decides exactly.
__device__ void ch_rebuild_window(const ChannelDev& S, const ChScratch& G, const ChLds& L) {
    const int n = S.n, t = threadIdx.x;
    const ChShort c = ch_short(S, L);
    const int kmax = S.kmax;
    bool over = false;
    ch_walk(S, L, [&](int j, int p) { ch_load_short(c, G, L, j, p); }, [&](int i) {
        const int own = ch_place(i, 0);
        const uint2 q = L.w16[own];
        const uint4 qa = G.posq[L.sid[i]];
        const int cx = cell_of(qa.x, S.lc[0]), cy = cell_of(qa.y, S.lc[1]), cz = cell_of(qa.z, S.lc[2]);
        const bool wall = qa.w != 0u;
        int count = ch_list_atom(S, c, G, L, i, wall, q, cx, cy, cz);
        const int y = q.x >> 16;
        const bool near = wall || y <= c.bottom || y >= c.top;
        if (count > kmax) {
            over = true;
            count = kmax;
        }
        ch_pad(G, count, n, i, (uint16_t)(own << 3));
        G.ncnt[i] = (uint16_t)(count | (near ? kChNearWall : 0));
    });
    if (over) L.misc[1] = 1;
    __syncthreads();
    if (L.misc[1] != 0) {
        __syncthreads();
        if (t == 0) L.misc[1] = 0;
        __syncthreads();
        ch_rebuild_scan<true>(S, G, L);
    }
}

__device__ void ch_rebuild(const ChannelDev& S, const ChScratch& G, const ChLds& L) {
    ch_sort(S, G, L);
    if (ch_windowed(L))
        ch_rebuild_window(S, G, L);
    else
        ch_rebuild_scan<false>(S, G, L);
}

// 1 / x for normal x, to a rounding: the hardware estimate (an ulp) and one Newton step.
__device__ __forceinline__ float ch_recip(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return __builtin_fmaf(r, __builtin_fmaf(-x, r, 1.0f), r);
}

// Pair sums of one atom.
struct ChSums {
    float gx = 0.f, gy = 0.f, gz = 0.f;  // force
    float wt = 0.f, wb = 0.f;            // x force from the top and the bottom wall (fluid atoms)
};

// One listed pair: c24 = 24 c of the pair; in: the entry counts; from: the partner's type, or 0
// where no wall partner is listed.
template <bool WALLS>
__device__ __forceinline__ void ch_pair(ChSums& g, float dx, float dy, float dz, float c24, float rc2,
                                        bool live, bool fluid_a, uint32_t from) {
    const float r2 = dx * dx + dy * dy + dz * dz;
    const float inv = ch_recip(r2);
    const float s3 = inv * inv * inv;
    const bool in = live & (r2 < rc2);
    const float fs = in ? s3 * (48.f * s3 - c24) * inv : 0.f;
    g.gx += fs * dx;
    g.gy += fs * dy;
    g.gz += fs * dz;
    if constexpr (WALLS) {
        const float fx = fs * dx;
        g.wt += (fluid_a & (from == 2u)) ? fx : 0.f;
        g.wb += (fluid_a & (from == 1u)) ? fx : 0.f;
    }
}

// Writes atom a's force: the pair sums, and for a wall atom its tether in FP64 (the sum rounded
// once to FP32). Partial sums of this thread: [0] x force on fluid from the top wall, [1] from
// the bottom wall, [2] S = sum_top dx - sum_bottom dx of the tether extensions.
__device__ __forceinline__ void ch_write_force(const ChannelDev& S, const double* r, float* f,
                                               const double* latx, const double* laty,
                                               const double* latz, double shift, int a,
                                               uint32_t type, const ChSums& g, double (&part)[3]) {
    const int n = S.n;
    if (type == 0u) {
        f[a] = g.gx;
        f[n + a] = g.gy;
        f[2 * n + a] = g.gz;
        part[0] += (double)g.wt;
        part[1] += (double)g.wb;
    } else {
        const int q = a - S.n_fluid;
        const bool top = type == 2u;
        const double xl = latx[q] + (top ? shift : -shift);
        const double ex = min_image(r[a] - xl, S.lx);
        const double ey = r[n + a] - laty[q];
        const double ez = min_image(r[2 * n + a] - latz[q], S.lz);
        f[a] = (float)((double)g.gx - S.k_spring * ex);
        f[n + a] = (float)((double)g.gy - S.k_spring * ey);
        f[2 * n + a] = (float)((double)g.gz - S.k_spring * ez);
        part[2] += top ? ex : -ex;
    }
}

// Forces (LJ through the lists in FP32), walked in list-grid order from posq_s (filled for this
// step).
__device__ void ch_forces_global(const ChannelDev& S, const double* r, float* f, const double* latx,
                                 const double* laty, const double* latz, double shift,
                                 const ChScratch& G, const ChLds& L, double (&part)[3]) {
    const int n = S.n;
    const float rc2 = S.rc2_f;
    const float cff = 24.f * (float)S.c_ff, cwf = 24.f * (float)S.c_wf;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const uint4 qa = G.posq_s[i];
        const bool fluid_a = qa.w == 0u;
        const int cnt = G.ncnt[i] & ~kChNearWall;
        ChSums g;
        // kChUnroll list entries per trip: their index loads, then their position gathers, are
        // issued together
        for (int kk = 0; kk < cnt; kk += kChUnroll) {
            int j[kChUnroll];
            uint4 qb[kChUnroll];
#pragma unroll
            for (int u = 0; u < kChUnroll; ++u) j[u] = G.nbr[ch_entry(kk + u, n, i)];
#pragma unroll
            for (int u = 0; u < kChUnroll; ++u) qb[u] = G.posq_s[j[u]];
#pragma unroll
            for (int u = 0; u < kChUnroll; ++u) {
                float dx, dy, dz;
                ch_sep(qa, qb[u], S, dx, dy, dz);
                ch_pair<true>(g, dx, dy, dz, (fluid_a & (qb[u].w == 0u)) ? cff : cwf, rc2, kk + u < cnt,
                              fluid_a, qb[u].w);
            }
        }
        ch_write_force(S, r, f, latx, laty, latz, shift, L.sid[i], qa.w, g, part);
    }
}

__device__ __forceinline__ void ch_load_position(const ChScratch& G, const ChLds& L, int j, int p) {
    const uint4 q = G.posq[L.sid[j]];
    L.wxy[p] = make_uint2(q.x, q.y);
    L.wz[p] = q.z;
    L.wtype[p] = (uint8_t)q.w;
}

// The list of slot i over window positions. WALLS: some lane of the wave has a wall partner or is
// a wall atom; the others need no types and no wall sums.
template <bool WALLS>
__device__ __forceinline__ void ch_list_sums(const ChannelDev& S, const ChScratch& G, const ChLds& L,
                                             int i, int cnt, uint2 axy, uint32_t az, bool fluid_a,
                                             float cff, float cwf, ChSums& g) {
    const int n = S.n;
    const float ux = S.fix_unit[0], uy = S.fix_unit[1], uz = S.fix_unit[2], rc2 = S.rc2_f;
    const uint16_t* row = G.nbr + i;
    const uint32_t un = (uint32_t)n;
    uint32_t e[kChUnroll], f[kChUnroll];
#pragma unroll
    for (int u = 0; u < kChUnroll; ++u) e[u] = row[u * un];
    for (int kk = 0; kk < cnt; kk += kChUnroll) {
        // the next trip's entries
        if (kk + kChUnroll < cnt) row += kChUnroll * (size_t)un;
#pragma unroll
        for (int u = 0; u < kChUnroll; ++u) f[u] = row[u * un];
        uint2v bxy[kChUnroll];
        uint32_t bz[kChUnroll], type[kChUnroll];
#pragma unroll
        for (int u = 0; u < kChUnroll; ++u) {
            const uint32_t at = e[u];  // place * 8
            bxy[u] = *(ChShared<uint2v>*)(at + kChWinXy);
            bz[u] = *(ChShared<uint32_t>*)(at >> 1);
            if constexpr (WALLS) type[u] = *(ChShared<uint8_t>*)((at >> 3) + kChWinType);
        }
#pragma unroll
        for (int u = 0; u < kChUnroll; ++u) {
            const float dx = (float)(int32_t)(axy.x - bxy[u].x) * ux;
            const float dy = (float)(int32_t)(axy.y - bxy[u].y) * uy;
            const float dz = (float)(int32_t)(az - bz[u]) * uz;
            float c24 = cff;
            if constexpr (WALLS) c24 = (fluid_a & (type[u] == 0u)) ? cff : cwf;
            ch_pair<WALLS>(g, dx, dy, dz, c24, rc2, kk + u < cnt, fluid_a, WALLS ? type[u] : 0u);
        }
        // (keeps the loads where they are: they were sunk to their use in the next trip)
#pragma unroll
        for (int u = 0; u < kChUnroll; ++u) {
            asm volatile("" : "+v"(f[u]));
            e[u] = f[u];
        }
    }
}

__device__ void ch_forces_window(const ChannelDev& S, const double* r, float* f, const double* latx,
                                 const double* laty, const double* latz, double shift,
                                 const ChScratch& G, const ChLds& L, double (&part)[3]) {
    const float cff = 24.f * (float)S.c_ff, cwf = 24.f * (float)S.c_wf;
    ch_walk(S, L, [&](int j, int p) { ch_load_position(G, L, j, p); }, [&](int i) {
        const int own = ch_place(i, 0);
        const uint2 axy = L.wxy[own];
        const uint32_t az = L.wz[own], type = L.wtype[own];
        const uint32_t packed = G.ncnt[i];
        const int cnt = (int)(packed & ~(uint32_t)kChNearWall);
        ChSums g;
        if (__builtin_amdgcn_ballot_w64((packed & kChNearWall) != 0u) != 0)
            ch_list_sums<true>(S, G, L, i, cnt, axy, az, type == 0u, cff, cwf, g);
        else
            ch_list_sums<false>(S, G, L, i, cnt, axy, az, true, cff, cwf, g);
        ch_write_force(S, r, f, latx, laty, latz, shift, L.sid[i], type, g, part);
    });
}

__device__ void ch_forces(const ChannelDev& S, const double* r, float* f, const double* latx,
                          const double* laty, const double* latz, double v, int64_t k,
                          const ChScratch& G, const ChLds& L, double (&part)[3]) {
    const double shift = 0.5 * v * ((double)k * S.dt);
    part[0] = part[1] = part[2] = 0.0;
    if (ch_windowed(L))
        ch_forces_window(S, r, f, latx, laty, latz, shift, G, L, part);
    else
        ch_forces_global(S, r, f, latx, laty, latz, shift, G, L, part);
}

__device__ void ch_write_observables(const ChannelDev& S, double fxt, double fxb, const ChLds& L,
                                     double* row) {
    const double area = S.lx * S.lz;
    for (int b = threadIdx.x; b <= S.n_bins; b += blockDim.x) {
        if (b == 0)
            row[0] = (fxt - fxb) / (2.0 * area);
        else
            row[b] = ((double)(long long)L.bins[b - 1] / kProfileScale) / (area * S.bin_w);
    }
}

__device__ __forceinline__ void ch_bin(const ChannelDev& S, double y, double px, const ChLds& L) {
    if (!(y >= S.bin_lo) || !(y < S.bin_hi)) return;
    int b = (int)floor((y - S.bin_lo) / S.bin_w);
    if (b > S.n_bins - 1) b = S.n_bins - 1;
    atomicAdd(&L.bins[b], (unsigned long long)llrint(px * kProfileScale));
}

// The system's constants, which lead the kernel arguments of both kernels that use them. Each
// phase of a step takes them anew: read once for the whole kernel they outgrow the scalar
// registers, and the force loop spends two lane reads a pair to fetch them back.
__device__ __forceinline__ const ChannelDev& ch_system() {
    auto* p = (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const ChannelDev*)p;
}

__device__ void run_channel(ChannelDesc* d, int steps_cap, const ChScratch& G, const ChLds& L) {
    const int n = ch_system().n, nf = ch_system().n_fluid, T = blockDim.x, t = threadIdx.x;
    double* r = d->r;
    double* p = d->p;
    float* f = d->f;
    const double v = d->v;
    int64_t k = d->k;
    int done = d->done;
    int health = d->health;
    double zeta = d->zeta;
    double pw2 = d->pw2;
    const int todo = health != 0 ? 0 : min(steps_cap, d->n_steps - done);
    if (todo <= 0 && done > 0) return;
    const double h = ch_system().dt, tau = 0.5 * h;
    if (t == 0) L.misc[2] = 0;
    __syncthreads();
    // step -1 is the state as it stands: its lists, and if no step was taken yet its forces, S(0),
    // sum of wall p^2 and observables (one copy of the build and the force pass in the code: two
    // took 99 registers to scratch)
    for (int step = -1; step < todo; ++step) {
        const bool start = step < 0;
        bool build = true;
        const ChannelDev& S = ch_system();
        if (start) {
            ch_publish(S, r, G, L);
            __syncthreads();
        } else {
            // thermostat half step (walls), half kick, drift, periodic wrap in x and z
            zeta += tau * (pw2 - S.nf_w * S.temperature) / S.q;
            const double c1 = exp(-zeta * tau);
            float pmax = 0.f;
            for (int a = t; a < n; a += T) {
                double px = p[a], py = p[n + a], pz = p[2 * n + a];
                if (a >= nf) {
                    px *= c1;
                    py *= c1;
                    pz *= c1;
                }
                px += tau * (double)f[a];
                py += tau * (double)f[n + a];
                pz += tau * (double)f[2 * n + a];
                double x = r[a] + h * px, y = r[n + a] + h * py, z = r[2 * n + a] + h * pz;
                // (inside the edges the quotients' floors are zero)
                if (!(x >= 0.0 && x < S.lx)) {
                    x -= S.lx * floor(x / S.lx);
                    if (x >= S.lx) x = 0.0;
                }
                if (!(z >= 0.0 && z < S.lz)) {
                    z -= S.lz * floor(z / S.lz);
                    if (z >= S.lz) z = 0.0;
                }
                ch_publish_atom(S, a, x, y, z, G, L);
                r[a] = x;
                r[n + a] = y;
                r[2 * n + a] = z;
                p[a] = px;
                p[n + a] = py;
                p[2 * n + a] = pz;
                const float pl = G.path[a] + (float)(h * sqrt(px * px + py * py + pz * pz));
                G.path[a] = pl;
                pmax = fmaxf(pmax, pl);
            }
            k += 1;
            build = 2.f * ch_block_max(pmax, L.wmax) * 1.0001f >= (float)S.skin;
        }
        if (build) {
            ch_rebuild(ch_system(), G, L);
            if (L.misc[1] != 0) {
                health |= kHealthListOverflow;
                if (!start) break;
            }
            if (start && done > 0) {
                if (health != 0) break;
                continue;
            }
        } else if (!ch_windowed(L)) {
            ch_gather_sorted(S, G, L);
            __syncthreads();
        }
        double part[3];
        ch_forces(ch_system(), r, f, d->latx, d->laty, d->latz, v, k, G, L, part);
        const ChannelDev& E = ch_system();
        for (int b = t; b < E.n_bins; b += T) L.bins[b] = 0ull;
        __syncthreads();
        // half kick, thermostat half step, observables
        const double c2 = exp(-zeta * tau);
        double w2 = 0.0;
        for (int a = t; a < n; a += T) {
            double px = p[a], py = p[n + a], pz = p[2 * n + a];
            if (!start) {
                px += tau * (double)f[a];
                py += tau * (double)f[n + a];
                pz += tau * (double)f[2 * n + a];
                if (a >= nf) {
                    px *= c2;
                    py *= c2;
                    pz *= c2;
                }
                p[a] = px;
                p[n + a] = py;
                p[2 * n + a] = pz;
            }
            if (a >= nf)
                w2 += px * px + py * py + pz * pz;
            else
                ch_bin(E, r[n + a], px, L);
        }
        double red4[4] = {part[0], part[1], part[2], w2};
        ch_block_sum<4>(red4, L.red);
        pw2 = red4[3];
        if (start) {
            if (t == 0) d->s0 = red4[2];
        } else {
            zeta += tau * (pw2 - E.nf_w * E.temperature) / E.q;
            done += 1;
        }
        if (d->series) ch_write_observables(E, red4[0], red4[1], L,
                                            d->series + (size_t)done * (1 + E.n_bins));
        if (!start && (!isfinite(pw2) || !isfinite(zeta) || L.misc[2] != 0))
            health |= kHealthNonFinite;
        if (health != 0) break;
        __syncthreads();
    }
    __syncthreads();
    if (t == 0) {
        d->k = k;
        d->done = done;
        d->health = health;
        d->zeta = zeta;
        d->pw2 = pw2;
    }
    __syncthreads();
}

// One workgroup of 16 waves per CU (128 VGPRs): the window takes the LDS.
static_assert(offsetof(ChannelLaunch, sys) == 0, "ch_system");
__global__ __launch_bounds__(kChThreads, kChWavesPerSimd) void k_channel(ChannelLaunch b) {
    extern __shared__ __align__(16) char smem[];
    const ChLds L = ch_carve(smem, b.sys.n, b.cmax, b.win);
    const ChScratch G = ch_scratch(b.scratch + (size_t)blockIdx.x * b.scratch_stride, b.sys.n,
                                   b.sys.kmax);
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) L.misc[0] = atomicAdd(b.queue, 1);
        __syncthreads();
        const int j = __builtin_amdgcn_readfirstlane(L.misc[0]);
        if (j >= b.n_jobs) break;
        run_channel(&b.descs[b.order ? b.order[j] : j], b.max_steps, G, L);
    }
}

// ---- spawn: mapped copies of stored start states -----------------------------------------
// states: per state [r (3n) | p (3n) | zeta]; mapping 1 reverses p and zeta, 2 reflects x of
// atoms and lattice sites and reverses p_x, 3 does both (p_x unchanged).
__global__ void k_channel_spawn(const double* states, int32_t n, int32_t n_wall, double lx,
                                const double* latx0, ChannelDesc* descs, int32_t count) {
    const int d = blockIdx.x;
    if (d >= count) return;
    ChannelDesc& D = descs[d];
    const double* st = states + (size_t)D.state * ((size_t)6 * n + 1);
    const int m = D.map;
    const bool rev = m == 1 || m == 3, refl = m == 2 || m == 3;
    for (int i = threadIdx.x; i < 3 * n; i += blockDim.x) {
        double x = st[i];
        double pv = st[3 * n + i];
        const bool is_x = i < n;
        if (refl && is_x) x = x == 0.0 ? 0.0 : lx - x;
        if (rev) pv = -pv;
        if (refl && is_x) pv = -pv;
        D.r[i] = x;
        D.p[i] = pv;
    }
    for (int q = threadIdx.x; q < n_wall; q += blockDim.x) {
        const double x = latx0[q];
        D.latx[q] = refl ? (x == 0.0 ? 0.0 : lx - x) : x;
    }
    if (threadIdx.x == 0) {
        const double z = st[6 * (size_t)n];
        D.zeta = rev ? -z : z;
    }
}

// Replica q of the mother: its positions, and its momenta plus kick q (kicks may be null).
__global__ void k_channel_replicate(const double* r, const double* p, const double* kicks,
                                    int32_t n, ChannelDesc* descs, int32_t count) {
    const int q = blockIdx.x;
    if (q >= count) return;
    ChannelDesc& D = descs[q];
    const double* kq = kicks ? kicks + (size_t)q * 3 * n : nullptr;
    for (int i = threadIdx.x; i < 3 * n; i += blockDim.x) {
        D.r[i] = r[i];
        D.p[i] = kq ? p[i] + kq[i] : p[i];
    }
}

// Stored start state q * per + s: replica q's positions, momenta and thermostat variable.
__global__ void k_channel_snapshot(const ChannelDesc* descs, int32_t count, int32_t n,
                                   double* states, int32_t per, int32_t s) {
    const int q = blockIdx.x;
    if (q >= count) return;
    const ChannelDesc& D = descs[q];
    double* dst = states + ((size_t)q * per + s) * ((size_t)6 * n + 1);
    for (int i = threadIdx.x; i < 3 * n; i += blockDim.x) {
        dst[i] = D.r[i];
        dst[3 * n + i] = D.p[i];
    }
    if (threadIdx.x == 0) dst[6 * (size_t)n] = D.zeta;
}

// ---- accumulate and response (several observables per time point) ------------------------
// One thread per (group, observable): D(t) = mean_m B_m(t); I(t) = mean_m int_0^t S_m(0)
// B_m(s) ds (trapezoid, compensated); the start state's TTCF series is D(0) - coef I(t).
__global__ void k_channel_accumulate(ChannelAccum a) {
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= a.n_groups * a.n_obs) return;
    const int g = id / a.n_obs, o = id % a.n_obs;
    const int b = a.first_of[g], e = a.first_of[g + 1];
    const int nm = min(e - b, 4);
    double s0[4], sum[4], comp[4], prev[4];
    const double* ser[4];
    for (int m = 0; m < nm; ++m) {
        const ChannelDesc& d = a.descs[b + m];
        ser[m] = d.series;
        s0[m] = d.s0;
        prev[m] = d.series[o];
        sum[m] = 0.0;
        comp[m] = 0.0;
    }
    const double inm = 1.0 / (double)nm;
    double* dout = a.d_out + (size_t)g * a.row_stride;
    double* iout = a.i_out + (size_t)g * a.row_stride;
    double d0 = 0.0;
    for (int m = 0; m < nm; ++m) d0 += prev[m];
    dout[o] = d0 * inm;
    iout[o] = 0.0;
    for (int k = 1; k < a.n_t; ++k) {
        double dsum = 0.0, isum = 0.0;
        for (int m = 0; m < nm; ++m) {
            const double cur = ser[m][(size_t)k * a.n_obs + o];
            const double add = 0.5 * a.dt * (s0[m] * prev[m] + s0[m] * cur);
            const double ts = sum[m] + add;
            comp[m] += fabs(sum[m]) >= fabs(add) ? (sum[m] - ts) + add : (add - ts) + sum[m];
            sum[m] = ts;
            prev[m] = cur;
            dsum += cur;
            isum += sum[m] + comp[m];
        }
        dout[(size_t)k * a.n_obs + o] = dsum * inm;
        iout[(size_t)k * a.n_obs + o] = isum * inm;
    }
}

// One thread per (t, observable column): mean and block standard error over the rows.
__global__ void k_channel_response(ChannelResponse r) {
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= r.n_t * r.n_cols) return;
    const int k = id / r.n_cols, o = r.col0 + id % r.n_cols;
    auto neu = [](double& s, double& c, double v) {
        const double ts = s + v;
        c += fabs(s) >= fabs(v) ? (s - ts) + v : (v - ts) + s;
        s = ts;
    };
    double gs = 0, gc = 0, ds = 0, dc = 0;
    for (int i = 0; i < r.n_rows; ++i) {
        const int row = r.rows[i];
        const double* dd = r.d_all + (size_t)row * r.row_stride;
        const double* ii = r.i_all + (size_t)row * r.row_stride;
        neu(gs, gc, dd[o] - r.coef[row] * ii[(size_t)k * r.n_obs + o]);
        neu(ds, dc, dd[(size_t)k * r.n_obs + o]);
    }
    const double gm = (gs + gc) / r.n_rows, dm = (ds + dc) / r.n_rows;
    double gv = 0, gvc = 0, dv = 0, dvc = 0;
    for (int i = 0; i < r.n_rows; ++i) {
        const int row = r.rows[i];
        const double* dd = r.d_all + (size_t)row * r.row_stride;
        const double* ii = r.i_all + (size_t)row * r.row_stride;
        const double g = dd[o] - r.coef[row] * ii[(size_t)k * r.n_obs + o] - gm;
        const double x = dd[(size_t)k * r.n_obs + o] - dm;
        neu(gv, gvc, g * g);
        neu(dv, dvc, x * x);
    }
    const double denom = r.n_rows > 1 ? (double)(r.n_rows - 1) * (double)r.n_rows : 1.0;
    const size_t out = (size_t)k * r.n_cols + (o - r.col0);
    const size_t plane = (size_t)r.n_t * r.n_cols;
    r.out[out] = gm;
    r.out[plane + out] = r.n_rows > 1 ? sqrt((gv + gvc) / denom) : 0.0;
    r.out[2 * plane + out] = dm;
    r.out[3 * plane + out] = r.n_rows > 1 ? sqrt((dv + dvc) / denom) : 0.0;
}

// Forces of one configuration (tests): the list build and force passes of the step kernel.
__global__ __launch_bounds__(kChThreads) void k_channel_debug_forces(ChannelLaunch b,
                                                                     double* out) {
    extern __shared__ __align__(16) char smem[];
    const ChLds L = ch_carve(smem, b.sys.n, b.cmax, b.win);
    if (threadIdx.x == 0) L.misc[2] = 0;
    __syncthreads();
    const ChannelDev& S = ch_system();
    const ChScratch G = ch_scratch(b.scratch, S.n, S.kmax);
    ChannelDesc& d = b.descs[0];
    ch_publish(S, d.r, G, L);
    __syncthreads();
    ch_rebuild(S, G, L);
    double part[3];
    ch_forces(S, d.r, d.f, d.latx, d.laty, d.latz, d.v, d.k, G, L, part);
    ch_block_sum<3>(part, L.red);
    if (threadIdx.x == 0) {
        out[0] = part[0];
        out[1] = part[1];
        out[2] = part[2];
        out[3] = (double)L.misc[1];
        out[4] = (double)L.misc[2];
    }
}

}  // namespace

size_t channel_lds_bytes(int nmax, int cmax, bool win) { return ch_plan(nmax, cmax, win).total; }
size_t channel_scratch_bytes(int nmax, int kmax) { return ch_scratch_bytes(nmax, kmax); }

// The window's addresses start at 0, so the kernel must have no LDS of a fixed size.
static bool ch_window_at_zero(const void* kernel) {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, kernel) == hipSuccess && a.sharedSizeBytes == 0;
}

hipError_t launch_channel(const ChannelLaunch& b, hipStream_t s) {
    const size_t lds = ch_plan(b.sys.n, b.cmax, b.win).total;
    if (!ch_window_at_zero((const void*)k_channel)) return hipErrorInvalidConfiguration;
    (void)hipFuncSetAttribute((const void*)k_channel, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    hipLaunchKernelGGL(k_channel, dim3(b.grid), dim3(kChThreads), lds, s, b);
    return hipGetLastError();
}

hipError_t launch_channel_debug_forces(const ChannelLaunch& b, double* out, hipStream_t s) {
    const size_t lds = ch_plan(b.sys.n, b.cmax, b.win).total;
    if (!ch_window_at_zero((const void*)k_channel_debug_forces)) return hipErrorInvalidConfiguration;
    (void)hipFuncSetAttribute((const void*)k_channel_debug_forces,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_channel_debug_forces, dim3(1), dim3(kChThreads), lds, s, b, out);
    return hipGetLastError();
}

hipError_t launch_channel_spawn(const double* states, int32_t n, int32_t n_wall, double lx,
                                const double* latx0, ChannelDesc* descs, int32_t count,
                                hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_channel_spawn, dim3(count), dim3(256), 0, s, states, n, n_wall, lx, latx0,
                       descs, count);
    return hipGetLastError();
}

hipError_t launch_channel_replicate(const double* r, const double* p, const double* kicks,
                                    int32_t n, ChannelDesc* descs, int32_t count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_channel_replicate, dim3(count), dim3(256), 0, s, r, p, kicks, n, descs,
                       count);
    return hipGetLastError();
}

hipError_t launch_channel_snapshot(const ChannelDesc* descs, int32_t count, int32_t n,
                                   double* states, int32_t per, int32_t slot, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_channel_snapshot, dim3(count), dim3(256), 0, s, descs, count, n, states,
                       per, slot);
    return hipGetLastError();
}

hipError_t launch_channel_accumulate(const ChannelAccum& a, hipStream_t s) {
    const int total = a.n_groups * a.n_obs;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_channel_accumulate, dim3((total + 63) / 64), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_channel_response(const ChannelResponse& r, hipStream_t s) {
    const int total = r.n_t * r.n_cols;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_channel_response, dim3((total + 63) / 64), dim3(64), 0, s, r);
    return hipGetLastError();
}

}  // namespace ttcf
