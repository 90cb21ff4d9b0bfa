// ttcf_mlp.hip -- gfx950 kernels of the learned control variate: start-state features, a
// bfloat16 matrix-core GEMM with FP32 accumulation (forward and backward passes of the MLP),
// Adam, and the integral h = Omega(0) int g ds of the predicted response.
#include <hip/hip_runtime.h>

#include "ttcf_internal.h"

namespace ttcf {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bfloat16 bits, round to nearest even
__device__ __forceinline__ short f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (short)(u >> 16);
}

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
           z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// ---------------------------------------------------------------------------------------
// GEMM: C(m, n) = sum_k A(m, k) B(k, n), A(m, k) = A[m sam + k sak], B(k, n) = B[k sbk + n sbn]
// Operands are rounded to bfloat16 as they are staged into LDS; gfx950's
// v_mfma_f32_16x16x32_bf16 accumulates in FP32. Workgroup tile B x B (four waves of B/2 x B/2),
// one matrix instruction per 16 x 16 tile and K step of 32.
// Operand layout of the 16x16x32 instruction: lane l holds A[l % 16][8 (l / 16) + i] and
// B[8 (l / 16) + i][l % 16] (i = 0..7); the result D[4 (l / 16) + i][l % 16]. Both operands lie
// k-fastest in LDS, so a fragment is one 16-byte read.
// Epilogues: 0 C = acc + bias; 1 Z = acc + bias, C = gelu(Z); 2 C = acc * gelu'(Zin);
// 3 C = acc + bias, dY = scale (C - T). The K loop runs in a fixed order: results are
// deterministic, and the same for both tile sizes.
//
// What bounds it at the network's sizes (a training step: rows = 256, 64-256-256-K): the latency
// of a block's loads and the launches. A block keeps a whole K chunk of loads in flight
// (coalesced along whichever index is contiguous) and loads the next chunk while it multiplies;
// 32 x 32 tiles give 64 blocks where 64 x 64 ones give 16; and up to three independent products
// and a column sum go in one launch. Training step of batch 256: 324 us with one product per
// launch, a K step of 32 and 64 x 64 tiles; 63 us now.
// ---------------------------------------------------------------------------------------

// Bias gradient: out[n] = sum over the M rows of X(m, n), 64 columns per workgroup. Sixteen
// partial sums of every 16th row (four per wave) added in order: a fixed order.
__device__ __forceinline__ void colsum_block(const GemmArgs& g, int block, float* part) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int n = block * 64 + lane;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    if (n < g.N)
        for (int m = w; m < g.M; m += 128) {
            float v[32];  // the loads of eight rows of each partial sum together
#pragma unroll
            for (int i = 0; i < 32; ++i)
                v[i] = m + 4 * i < g.M ? g.A[(int64_t)(m + 4 * i) * g.sam + n] : 0.f;
#pragma unroll
            for (int i = 0; i < 32; ++i) s[i % 4] += v[i];
        }
#pragma unroll
    for (int q = 0; q < 4; ++q) part[(w + 4 * q) * 64 + lane] = s[q];
    __syncthreads();
    if (w == 0 && n < g.N) {
        float t = 0.f;
        for (int v = 0; v < 16; ++v) t += part[v * 64 + lane];
        g.C[n] = t;
    }
}

// A tile of one operand on its way to LDS: B rows (m or n) of KC values of k as floats, four
// consecutive ones per load where the strides and the base allow it.
template <int B, int KC>
struct Strip {
    static constexpr int N4 = B * KC / 1024;  // quads per thread
    f32x4 v[N4];
    // place of quad i: (row, k) of its first value; along k if the strip's k index is contiguous
    static __device__ __forceinline__ int row(bool along_k, int i) {
        const int q = threadIdx.x + 256 * i;
        return along_k ? q / (KC / 4) : q % (B / 4) * 4;
    }
    static __device__ __forceinline__ int col(bool along_k, int i) {
        const int q = threadIdx.x + 256 * i;
        return along_k ? q % (KC / 4) * 4 : q / (B / 4);
    }
    // rows r0.. of P (stride sr), values k0.. (stride sk); one of the strides is 1
    __device__ __forceinline__ void load(const float* P, int64_t sr, int64_t sk, int r0, int rows,
                                         int k0, int K, bool along_k, bool quads) {
#pragma unroll
        for (int i = 0; i < N4; ++i) {
            const int r = r0 + row(along_k, i), k = k0 + col(along_k, i);
            v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            const float* p = P + (r * sr + k * sk);
            if (quads) {
                if (r < rows && k < K) v[i] = *(const f32x4*)p;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (r + (along_k ? 0 : e) < rows && k + (along_k ? e : 0) < K) v[i][e] = p[e];
            }
        }
    }
    template <int LD>
    __device__ __forceinline__ void store(short* S, bool along_k) const {
#pragma unroll
        for (int i = 0; i < N4; ++i) {
            short* s = S + row(along_k, i) * LD + col(along_k, i);
            if (along_k) {
                typedef short short4v __attribute__((ext_vector_type(4)));
                *(short4v*)s = short4v{f2bf(v[i][0]), f2bf(v[i][1]), f2bf(v[i][2]), f2bf(v[i][3])};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e * LD] = f2bf(v[i][e]);
            }
        }
    }
};

template <int B>
__global__ __launch_bounds__(256) void k_gemm_bf16(GemmTasks tasks) {
    constexpr int KC = B == 32 ? 256 : 64;  // K chunk
    constexpr int LD = KC + 8;
    constexpr int NT = B / 32;
    __shared__ __align__(16) short As[B * LD];
    __shared__ __align__(16) short Bs[B * LD];
    const GemmArgs& g = tasks.t[blockIdx.y];
    const int block = blockIdx.x;
    if (block >= g.blocks) return;
    if (g.epi == kEpiColsum) {
        colsum_block(g, block, (float*)As);
        return;
    }
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int nbn = (g.N + B - 1) / B;
    const int m0 = (block / nbn) * B, n0 = (block % nbn) * B;
    const int wm = (wave >> 1) * (B / 2), wn = (wave & 1) * (B / 2);
    f32x4 acc[NT][NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bool ak = g.sak == 1, bk = g.sbk == 1;
    Strip<B, KC> a, b;
    a.load(g.A, g.sam, g.sak, m0, g.M, 0, g.K, ak, g.quads & 1);
    b.load(g.B, g.sbn, g.sbk, n0, g.N, 0, g.K, bk, g.quads & 2);
    for (int k0 = 0; k0 < g.K; k0 += KC) {
        a.template store<LD>(As, ak);
        b.template store<LD>(Bs, bk);
        __syncthreads();
        if (k0 + KC < g.K) {
            a.load(g.A, g.sam, g.sak, m0, g.M, k0 + KC, g.K, ak, g.quads & 1);
            b.load(g.B, g.sbn, g.sbk, n0, g.N, k0 + KC, g.K, bk, g.quads & 2);
        }
        const int steps = min(KC, g.K - k0 + 31) / 32;
#pragma unroll 1
        for (int s = 0; s < steps; ++s) {
            const int kb = s * 32 + (lane >> 4) * 8;
            bf16x8 fa[NT], fb[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                fa[i] = *(const bf16x8*)&As[(wm + i * 16 + (lane & 15)) * LD + kb];
                fb[i] = *(const bf16x8*)&Bs[(wn + i * 16 + (lane & 15)) * LD + kb];
            }
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm + i * 16 + (lane >> 4) * 4 + r;
                const int n = n0 + wn + j * 16 + (lane & 15);
                if (m >= g.M || n >= g.N) continue;
                float v = acc[i][j][r];
                const int64_t o = (int64_t)m * g.ldc + n;
                if (g.epi == 2) {
                    g.C[o] = v * gelu_grad_f(g.Zin[o]);
                    continue;
                }
                if (g.bias) v += g.bias[n];
                if (g.epi == 1) {
                    g.Z[o] = v;
                    g.C[o] = gelu_f(v);
                } else {
                    g.C[o] = v;
                    if (g.epi == 3) g.Z[o] = g.scale * (v - g.Zin[o]);
                }
            }
}

hipError_t launch_gemms(const GemmArgs* g, int count, hipStream_t s) {
    if (count < 1 || count > kMaxGemmTasks) return hipErrorInvalidValue;
    GemmTasks tasks{};
    // whether the four consecutive values of an operand's load are aligned and all in range or none
    auto quads = [](const float* p, int64_t stride, int extent) {
        return (uintptr_t)p % 16 == 0 && stride % 4 == 0 && extent % 4 == 0;
    };
    for (int i = 0; i < count; ++i) {
        GemmArgs& a = tasks.t[i] = g[i];
        if (a.epi == kEpiColsum) continue;
        if ((a.sak != 1 && a.sam != 1) || (a.sbk != 1 && a.sbn != 1)) return hipErrorInvalidValue;
        a.quads = (quads(a.A, a.sak == 1 ? a.sam : a.sak, a.sak == 1 ? a.K : a.M) ? 1 : 0) |
                  (quads(a.B, a.sbk == 1 ? a.sbn : a.sbk, a.sbk == 1 ? a.K : a.N) ? 2 : 0);
    }
    int total = 0, most = 0;
    auto fill = [&](int tile) {
        total = most = 0;
        for (int i = 0; i < count; ++i) {
            GemmArgs& a = tasks.t[i];
            const bool none = a.M <= 0 || a.N <= 0 || (a.epi != kEpiColsum && a.K <= 0);
            a.blocks = none ? 0
                       : a.epi == kEpiColsum ? (a.N + 63) / 64
                                             : ((a.M + tile - 1) / tile) * ((a.N + tile - 1) / tile);
            total += a.blocks;
            most = a.blocks > most ? a.blocks : most;
        }
    };
    // 64 x 64 tiles read each operand half as often; below a block per CU the smaller tiles'
    // parallelism is worth more
    fill(64);
    if (total == 0) return hipSuccess;
    if (total >= 256) {
        hipLaunchKernelGGL(k_gemm_bf16<64>, dim3(most, count), dim3(256), 0, s, tasks);
    } else {
        fill(32);
        hipLaunchKernelGGL(k_gemm_bf16<32>, dim3(most, count), dim3(256), 0, s, tasks);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// small element-wise and reduction kernels (fixed-order sums)
// ---------------------------------------------------------------------------------------

__global__ void k_mse_loss(const float* Y, const float* Tg, int64_t count, double* loss) {
    __shared__ double part[256];
    double s = 0.0;
#pragma unroll 8
    for (int64_t i = threadIdx.x; i < count; i += 256) {
        const double d = (double)Y[i] - (double)Tg[i];
        s += d * d;
    }
    part[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int i = 0; i < 256; ++i) tot += part[i];
        *loss = tot / (double)count;
    }
}

__global__ void k_adam(float* P, const float* G, float* Mo, float* Vo, int64_t n, float lr,
                       float b1, float b2, float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g = G[i];
    const float m = b1 * Mo[i] + (1.f - b1) * g;
    const float v = b2 * Vo[i] + (1.f - b2) * g * g;
    Mo[i] = m;
    Vo[i] = v;
    P[i] -= lr * (m / c1) / (sqrtf(v / c2) + eps);
}

// dst[r][c] = (src[idx[r]][c] - mu[c]) * inv[c], for up to two arrays of the same rows (idx null:
// the rows in order)
__global__ void k_gather_norm(GatherArgs x, GatherArgs y, const int32_t* idx, int rows) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool second = e >= (int64_t)rows * x.cols;
    if (second) e -= (int64_t)rows * x.cols;
    const GatherArgs& g = second ? y : x;
    if (e >= (int64_t)rows * g.cols) return;
    const int r = (int)(e / g.cols), c = (int)(e % g.cols);
    const int64_t sr = idx ? idx[r] : r;
    g.dst[e] = (g.src[sr * g.cols + c] - g.mu[c]) * g.inv[c];
}

// mean and 1/std of every column (two passes in FP64; std floor 1e-12): 16 columns per workgroup,
// 64 threads on each column's rows, partial sums added in thread order (a fixed order). With one
// thread per column the 1024 rows of each pass were one chain of loads (0.33 ms).
constexpr int kStatCols = 16, kStatRows = 64;
__global__ __launch_bounds__(kStatCols * kStatRows) void k_col_stats(const float* X, int64_t rows,
                                                                     int cols, float* mu, float* inv) {
    __shared__ double part[kStatRows][kStatCols + 1];
    const int cl = threadIdx.x % kStatCols, w = threadIdx.x / kStatCols;
    const int c = blockIdx.x * kStatCols + cl;
    auto total = [&](double v) {
        __syncthreads();
        part[w][cl] = v;
        __syncthreads();
        double s = 0.0;
        for (int q = 0; q < kStatRows; ++q) s += part[q][cl];
        return s;
    };
    double s = 0.0;
    if (c < cols)
        for (int64_t r = w; r < rows; r += kStatRows) s += X[r * cols + c];
    const double m = total(s) / (double)rows;
    double q = 0.0;
    if (c < cols)
        for (int64_t r = w; r < rows; r += kStatRows) {
            const double d = X[r * cols + c] - m;
            q += d * d;
        }
    q = total(q);
    if (w != 0 || c >= cols) return;
    const double sd = sqrt(q / (double)(rows > 1 ? rows - 1 : 1));
    mu[c] = (float)m;
    inv[c] = (float)(1.0 / (sd > 1e-12 ? sd : 1e-12));
}

hipError_t launch_mse_loss(const float* Y, const float* Tg, int64_t count, double* loss,
                           hipStream_t s) {
    hipLaunchKernelGGL(k_mse_loss, dim3(1), dim3(256), 0, s, Y, Tg, count, loss);
    return hipGetLastError();
}
hipError_t launch_adam(float* P, const float* G, float* Mo, float* Vo, int64_t n, float lr,
                       int64_t step, hipStream_t s) {
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, P, G, Mo, Vo, n,
                       lr, b1, b2, 1e-8f, c1, c2);
    return hipGetLastError();
}
hipError_t launch_gather_norm(const GatherArgs& x, const GatherArgs& y, const int32_t* idx, int rows,
                              hipStream_t s) {
    const int64_t n = (int64_t)rows * (x.cols + y.cols);
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_norm, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, y, idx, rows);
    return hipGetLastError();
}
hipError_t launch_col_stats(const float* X, int64_t rows, int cols, float* mu, float* inv,
                            hipStream_t s) {
    hipLaunchKernelGGL(k_col_stats, dim3((cols + kStatCols - 1) / kStatCols), dim3(kStatCols * kStatRows), 0,
                       s, X, rows, cols, mu, inv);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// features of mapped start states
// ---------------------------------------------------------------------------------------
// Pair sums of atom i: the force, half the pair virials x_ij F_y,ij and half of (p_x,i - p_x,j)
// F_y,ij. First 64 distances at a time make a bit mask of the partners in range, then its bits, in
// order: evaluated where they are found, some lane of the wave had a partner in nearly every trip
// and all of them paid for its division.
struct CvPairs {
    double fx, fy, vir, d2;
};

__device__ __forceinline__ CvPairs cv_pairs(int i, int n, const double* X, const double* Y,
                                            const double* Z, const double* PX, double lx, double ly,
                                            double lz, double ilx, double ily, double ilz, double rc2,
                                            double c_attr) {
    const double xi = X[i], yi = Y[i], zi = Z[i], pxi = PX[i];
    CvPairs c{0.0, 0.0, 0.0, 0.0};
    auto separation = [&](int j, double& dx, double& dy, double& dz) {
        dx = xi - X[j], dy = yi - Y[j], dz = zi - Z[j];
        dx -= lx * rint(dx * ilx);
        dy -= ly * rint(dy * ily);
        dz -= lz * rint(dz * ilz);
        return dx * dx + dy * dy + dz * dz;
    };
    for (int j0 = 0; j0 < n; j0 += 64) {
        const int count = min(64, n - j0);
        uint64_t near = 0;
        double dx, dy, dz;
#pragma unroll 4
        for (int k = 0; k < count; ++k)
            near |= (uint64_t)(separation(j0 + k, dx, dy, dz) < rc2 ? 1 : 0) << k;
        if ((unsigned)(i - j0) < 64u) near &= ~(1ull << (i - j0));
        for (; near != 0; near &= near - 1) {
            const int j = j0 + __builtin_ctzll(near);
            const double r2 = separation(j, dx, dy, dz);
            const double inv2 = 1.0 / r2;
            const double inv6 = inv2 * inv2 * inv2;
            const double fs = 24.0 * inv6 * (2.0 * inv6 - c_attr) * inv2;
            c.fx += fs * dx;
            c.fy += fs * dy;
            c.vir += 0.5 * dx * (fs * dy);
            c.d2 += 0.5 * (pxi - PX[j]) * (fs * dy);
        }
    }
    return c;
}

// The row's sums, each by one thread in atom order: slab sums of p_x, p_x p_y and the virial in
// wave 0, the two force-momentum sums in waves 1 and 2. Every atom's slab goes to LDS first (over
// the z positions, which the pair sums are done with; D2 is read by its sum alone).
template <typename Put>
__device__ __forceinline__ void cv_sums(int q, int n, double ly, const double* Y, double* Z,
                                        const double* PX, const double* PY, const double* FX,
                                        const double* FY, const double* VIR, const double* D2, Put put) {
    int* slab = (int*)Z;
    const double inv = (double)kCvSlabs / ly;
    for (int a = q; a < n; a += blockDim.x) {
        const int k = (int)floor(Y[a] * inv);
        slab[a] = k < 0 ? 0 : (k > kCvSlabs - 1 ? kCvSlabs - 1 : k);
    }
    __syncthreads();
    if (q < 3 * kCvSlabs) {
        const int own = q % kCvSlabs;
        const int kind = q / kCvSlabs;  // 0 p_x, 1 p_x p_y, 2 virial
        const double* u = kind == 2 ? VIR : PX;
        double acc = 0.0;
#pragma unroll 8
        for (int a = 0; a < n; ++a) {
            const double v = kind == 1 ? u[a] * PY[a] : u[a];
            acc = slab[a] == own ? acc + v : acc;
        }
        put(q, acc);
    } else if (q == 64) {
        double acc = 0.0;
#pragma unroll 8
        for (int a = 0; a < n; ++a) acc += FX[a] * PY[a] + PX[a] * FY[a];
        put(3 * kCvSlabs, acc);
    } else if (q == 128) {
        double acc = 0.0;
#pragma unroll 8
        for (int a = 0; a < n; ++a) acc += D2[a];
        put(3 * kCvSlabs + 1, acc);
    }
}

// Row layout (kCvIn = 64): [P_xy(0), Omega(0); per slab k of kCvSlabs = 20 in y (k = floor(y
// 20 / Ly) clamped): sum p_x, sum p_x p_y, and half the pair virial x_ij F_y,ij of each of the
// slab's atoms; then sum_i (F_x,i p_y,i + p_x,i F_y,i) and sum_{i<j} (p_x,i - p_x,j) F_y,ij],
// all of the mapped start state (Eq. (mappings): x -> -x for mappings 2 and 3, p_x and p_y
// signs as below). One workgroup of 256 threads per row: the mapped state is staged in LDS,
// thread q computes the pair terms of atoms q, q + 256, ... against every other atom (each
// pair seen from both sides, so no atomics), then one thread a sum forms the 62 sums in atom order
// (deterministic). FP64 throughout; LDS 9 n doubles. 1024 rows of N = 256: one wave a row 222 us, four
// waves 140, partners found before they are evaluated 113, sums over stored slab numbers on
// three waves 84.
__global__ __launch_bounds__(256) void k_cv_features(
    const double* states, int32_t n, const int32_t* state_of, const int32_t* map_of,
    const double* vpxy0, const double* vsign, int32_t rows, double lx, double ly, double lz,
    double rc2, double c_attr, double volume, double temperature, double gamma_dot, float* out,
    double* b0_out, double* om_out) {
    extern __shared__ double cvs[];
    double* X = cvs;
    double* Y = X + n;
    double* Z = Y + n;
    double* PX = Z + n;
    double* PY = PX + n;
    double* FX = PY + n;
    double* FY = FX + n;
    double* VIR = FY + n;
    double* D2 = VIR + n;
    const int row = blockIdx.x;
    if (row >= rows) return;
    const double* st = states + (size_t)state_of[row] * 6 * (size_t)n;
    const int m = map_of[row];
    // mapping signs: p -> -p (m=1); (x, px) -> (-x, -px) (m=2); (x, py, pz) -> -(...) (m=3)
    const double sx = (m == 1 || m == 2) ? -1.0 : 1.0;
    const double sy = (m == 1 || m == 3) ? -1.0 : 1.0;
    const double sr = (m == 2 || m == 3) ? -1.0 : 1.0;  // x of the positions
    const int q = threadIdx.x;
    for (int a = q; a < n; a += blockDim.x) {
        X[a] = sr * st[a];
        Y[a] = st[n + a];
        Z[a] = st[2 * n + a];
        PX[a] = sx * st[3 * n + a];
        PY[a] = sy * st[4 * n + a];
    }
    __syncthreads();
    // minimum image with the reciprocal edges (the image chosen differs from a division's
    // only for separations within rounding of half a box, far beyond r_c)
    const double ilx = 1.0 / lx, ily = 1.0 / ly, ilz = 1.0 / lz;
    for (int i = q; i < n; i += blockDim.x) {
        const CvPairs c = cv_pairs(i, n, X, Y, Z, PX, lx, ly, lz, ilx, ily, ilz, rc2, c_attr);
        FX[i] = c.fx;
        FY[i] = c.fy;
        VIR[i] = c.vir;
        D2[i] = c.d2;
    }
    __syncthreads();
    float* o = out + (size_t)row * kCvIn;
    cv_sums(q, n, ly, Y, Z, PX, PY, FX, FY, VIR, D2, [&](int f, double v) { o[2 + f] = (float)v; });
    if (q == 0) {
        // vpxy0 indexed by row (vsign null) or by state with the mapping's sign of P_xy
        const double vp = vsign ? vpxy0[state_of[row]] * vsign[m] : vpxy0[row];
        const double pxy = vp / volume;
        const double om = -(volume / temperature) * gamma_dot * pxy;
        o[0] = (float)pxy;
        o[1] = (float)om;
        if (b0_out) b0_out[row] = pxy;
        if (om_out) om_out[row] = om;
    }
}

// The same features for the four mapped rows of each of n_states start states (row
// 4 s + m), the pair sums done once per state: every feature of mapping m is the unmapped one
// times a sign (p_x sums and the two force-momentum sums by s_x, p_x p_y by s_x s_y, the virial
// by s_r, the sign of x), and the per-row kernel's operations give exactly those negations,
// so both kernels write the same bits.
__global__ __launch_bounds__(256) void k_cv_features_maps(
    const double* states, int32_t n, int32_t n_states, const double* vpxy0, const double* vsign,
    double lx, double ly, double lz, double rc2, double c_attr, double volume,
    double temperature, double gamma_dot, float* out, double* b0_out, double* om_out) {
    extern __shared__ double cvs[];
    double* X = cvs;
    double* Y = X + n;
    double* Z = Y + n;
    double* PX = Z + n;
    double* PY = PX + n;
    double* FX = PY + n;
    double* FY = FX + n;
    double* VIR = FY + n;
    double* D2 = VIR + n;
    double* feat = D2 + n;  // [3 kCvSlabs + 2] the unmapped features
    const int st_i = blockIdx.x;
    if (st_i >= n_states) return;
    const double* st = states + (size_t)st_i * 6 * (size_t)n;
    const int q = threadIdx.x;
    for (int a = q; a < n; a += blockDim.x) {
        X[a] = st[a];
        Y[a] = st[n + a];
        Z[a] = st[2 * n + a];
        PX[a] = st[3 * n + a];
        PY[a] = st[4 * n + a];
    }
    __syncthreads();
    const double ilx = 1.0 / lx, ily = 1.0 / ly, ilz = 1.0 / lz;
    for (int i = q; i < n; i += blockDim.x) {
        const CvPairs c = cv_pairs(i, n, X, Y, Z, PX, lx, ly, lz, ilx, ily, ilz, rc2, c_attr);
        FX[i] = c.fx;
        FY[i] = c.fy;
        VIR[i] = c.vir;
        D2[i] = c.d2;
    }
    __syncthreads();
    cv_sums(q, n, ly, Y, Z, PX, PY, FX, FY, VIR, D2, [&](int f, double v) { feat[f] = v; });
    __syncthreads();
    // row 4 st_i + m: mapping signs p -> -p (m=1); (x, px) -> (-x, -px) (m=2);
    // (x, py, pz) -> -(...) (m=3)
    for (int e = q; e < 4 * (3 * kCvSlabs + 2); e += blockDim.x) {
        const int m = e / (3 * kCvSlabs + 2), f = e % (3 * kCvSlabs + 2);
        const double sx = (m == 1 || m == 2) ? -1.0 : 1.0;
        const double sy = (m == 1 || m == 3) ? -1.0 : 1.0;
        const double sr = (m == 2 || m == 3) ? -1.0 : 1.0;
        const int kind = f < 3 * kCvSlabs ? f / kCvSlabs : 3;
        const double sg = kind == 0 ? sx : (kind == 1 ? sx * sy : (kind == 2 ? sr : sx));
        out[(size_t)(4 * st_i + m) * kCvIn + 2 + f] = (float)(sg * feat[f]);
    }
    if (q < 4) {
        const int row = 4 * st_i + q;
        const double vp = vpxy0[st_i] * vsign[q];
        const double pxy = vp / volume;
        const double om = -(volume / temperature) * gamma_dot * pxy;
        out[(size_t)row * kCvIn] = (float)pxy;
        out[(size_t)row * kCvIn + 1] = (float)om;
        if (b0_out) b0_out[row] = pxy;
        if (om_out) om_out[row] = om;
    }
}

size_t lds_bytes_cv_features(int32_t n) { return sizeof(double) * 9 * (size_t)n; }
size_t lds_bytes_cv_features_maps(int32_t n) {
    return lds_bytes_cv_features(n) + sizeof(double) * (3 * kCvSlabs + 2);
}

hipError_t launch_cv_features(const double* states, int32_t n, const int32_t* state_of,
                              const int32_t* map_of, const double* vpxy0, const double* vsign,
                              int32_t rows, const double* box, double rc2, double c_attr,
                              double volume, double temperature, double gamma_dot, float* out,
                              double* b0_out, double* om_out, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const size_t lds = lds_bytes_cv_features(n);
    (void)hipFuncSetAttribute((const void*)k_cv_features,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_cv_features, dim3(rows), dim3(256), lds, s, states, n, state_of, map_of,
                       vpxy0, vsign, rows, box[0], box[1], box[2], rc2, c_attr, volume,
                       temperature, gamma_dot, out, b0_out, om_out);
    return hipGetLastError();
}

hipError_t launch_cv_features_maps(const double* states, int32_t n, int32_t n_states,
                                   const double* vpxy0, const double* vsign, const double* box,
                                   double rc2, double c_attr, double volume, double temperature,
                                   double gamma_dot, float* out, double* b0_out, double* om_out,
                                   hipStream_t s) {
    if (n_states <= 0) return hipSuccess;
    const size_t lds = lds_bytes_cv_features_maps(n);
    (void)hipFuncSetAttribute((const void*)k_cv_features_maps,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_cv_features_maps, dim3(n_states), dim3(256), lds, s, states, n, n_states,
                       vpxy0, vsign, box[0], box[1], box[2], rc2, c_attr, volume, temperature,
                       gamma_dot, out, b0_out, om_out);
    return hipGetLastError();
}

// P_xy(0) (as V P_xy) and, when targets != null, B(t_1..t_nout) = P_xy of each daughter's
// recorded series, one workgroup per daughter.
__global__ void k_cv_gather_series(const double* const* series, int32_t count, int32_t n_out,
                                   double inv_volume, float* targets, double* vpxy0) {
    const int row = blockIdx.x;
    if (row >= count) return;
    const double* s = series[row];
    if (targets)
        for (int k = threadIdx.x; k < n_out; k += blockDim.x)
            targets[(size_t)row * n_out + k] = (float)(s[k + 1] * inv_volume);
    if (threadIdx.x == 0) vpxy0[row] = s[0];
}

hipError_t launch_cv_gather_series(const double* const* series, int32_t count, int32_t n_out,
                                   double inv_volume, float* targets, double* vpxy0, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cv_gather_series, dim3(count), dim3(64), 0, s, series, count, n_out,
                       inv_volume, targets, vpxy0);
    return hipGetLastError();
}

// h rows (stride values apart) into each daughter's own h series, the first lens[r] values
__global__ void k_cv_scatter_h(const double* h, int32_t stride, int32_t count, double* const* dst,
                               const int32_t* lens) {
    const int row = blockIdx.x;
    if (row >= count) return;
    double* d = dst[row];
    for (int k = threadIdx.x; k < lens[row]; k += blockDim.x) d[k] = h[(size_t)row * stride + k];
}

hipError_t launch_cv_scatter_h(const double* h, int32_t stride, int32_t count, double* const* dst,
                               const int32_t* lens, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cv_scatter_h, dim3(count), dim3(64), 0, s, h, stride, count, dst, lens);
    return hipGetLastError();
}

__global__ void k_fill_f64(double* p, double v, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

hipError_t launch_fill_f64(double* p, double v, int64_t count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_f64, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, p, v, count);
    return hipGetLastError();
}

// h(t_k) = Omega(0) int_0^{t_k} g ds (trapezoid, g(0) = B(0)) of each row, FP64; pred holds
// the standardised predictions, B(t_k) = pred / yinv[k] + ymu[k]. out rows (n_out + 1 values)
// are out_stride apart.
__global__ void k_cv_h(const float* pred, int rows, int n_out, const float* ymu, const float* yinv,
                       const double* b0, const double* omega, double dt, double* out,
                       int64_t out_stride) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= rows) return;
    const float* p = pred + (size_t)r * n_out;
    double* h = out + (size_t)r * out_stride;
    double prev = b0[r], acc = 0.0;
    const double om = omega[r];
    h[0] = 0.0;
    for (int k = 0; k < n_out; ++k) {
        const double cur = (double)p[k] / (double)yinv[k] + (double)ymu[k];
        acc += 0.5 * dt * (prev + cur);
        prev = cur;
        h[k + 1] = om * acc;
    }
}

hipError_t launch_cv_h(const float* pred, int rows, int n_out, const float* ymu, const float* yinv,
                       const double* b0, const double* omega, double dt, double* out,
                       int64_t out_stride, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cv_h, dim3((rows + 63) / 64), dim3(64), 0, s, pred, rows, n_out, ymu, yinv,
                       b0, omega, dt, out, out_stride);
    return hipGetLastError();
}

// mean-term accumulation: for every t, add the mapping means of h over the groups of this
// chunk (group = `maps` consecutive rows) into compensated sums of H and H^2. First pass:
// workgroup (t block, partition p) takes the groups of partition p (contiguous ranges), its
// wave w every kMuWaves-th of them, and writes the wave's compensated partial sums; second
// pass: per t, the partials are added to the running sums in (p, w) order. The result does not
// depend on timing.
constexpr int kMuParts = 32;
constexpr int kMuWaves = 8;

__device__ __forceinline__ void mu_neumaier(double& sum, double& comp, double v) {
    const double t = sum + v;
    comp += fabs(sum) >= fabs(v) ? (sum - t) + v : (v - t) + sum;
    sum = t;
}

__global__ __launch_bounds__(64 * kMuWaves) void k_cv_mu_partial(const double* h, int groups,
                                                                  int maps, int nt,
                                                                  double* part) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int k = blockIdx.x * 64 + lane, p = blockIdx.y;
    if (k >= nt) return;
    const int per = (groups + kMuParts - 1) / kMuParts;
    const int g0 = p * per, g1 = min(groups, g0 + per);
    double s = 0.0, c = 0.0, s2 = 0.0, c2 = 0.0;
    for (int g = g0 + w; g < g1; g += kMuWaves) {
        double v = 0.0;
        for (int m = 0; m < maps; ++m) v += h[((size_t)g * maps + m) * nt + k];
        v /= (double)maps;
        mu_neumaier(s, c, v);
        mu_neumaier(s2, c2, v * v);
    }
    double* out = part + (size_t)(p * kMuWaves + w) * 4 * nt;
    out[k] = s;
    out[nt + k] = c;
    out[2 * nt + k] = s2;
    out[3 * nt + k] = c2;
}

__global__ void k_cv_mu_combine(const double* part, int nt, double* sum, double* comp,
                                double* sumsq, double* compsq) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nt) return;
    double s = sum[k], c = comp[k], s2 = sumsq[k], c2 = compsq[k];
    for (int i = 0; i < kMuParts * kMuWaves; ++i) {
        const double* q = part + (size_t)i * 4 * nt;
        mu_neumaier(s, c, q[k]);
        mu_neumaier(s, c, q[nt + k]);
        mu_neumaier(s2, c2, q[2 * nt + k]);
        mu_neumaier(s2, c2, q[3 * nt + k]);
    }
    sum[k] = s;
    comp[k] = c;
    sumsq[k] = s2;
    compsq[k] = c2;
}

size_t cv_mu_scratch_doubles(int nt) { return (size_t)kMuParts * kMuWaves * 4 * (size_t)nt; }

hipError_t launch_cv_mu_accum(const double* h, int groups, int maps, int nt, double* sum,
                              double* comp, double* sumsq, double* compsq, double* part,
                              hipStream_t s) {
    if (groups <= 0 || nt <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cv_mu_partial, dim3((nt + 63) / 64, kMuParts), dim3(64 * kMuWaves), 0, s,
                       h, groups, maps, nt, part);
    hipLaunchKernelGGL(k_cv_mu_combine, dim3((nt + 63) / 64), dim3(64), 0, s, part, nt, sum, comp,
                       sumsq, compsq);
    return hipGetLastError();
}

}  // namespace ttcf
