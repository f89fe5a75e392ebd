// Data-free fitting of the codec projections (Encoder-Decoder based on Low-Rank
// Compression, Eq. 8 with lambda = 0) for gfx950: the kernels that the matrix-core GEMM
// does not cover. The fit is subspace iteration on the Gram matrices of the calibration
// slices (the products run on the GEMM); every iterate is orthonormalised by a Cholesky QR
// (Yamamoto et al., 2015): G = Y^T Y, G = R^T R, Q = Y R^-1. The Gram matrix, its factor and the
// triangular solve are float64, so the factorisation holds for condition numbers of Y up to
// about 1e7 (float32 would fail near 4e3) and Q is rounded to float32 once; the last iterate
// takes a second pass (CholeskyQR2), which leaves it orthonormal to float32 at any of those
// condition numbers. The iterates before it need only span their subspace, and R from one pass
// does that as well as from two.
//
// The three kernels work on 16 x 16 blocks on the float64 matrix cores. A block in their result
// layout (lane l: rows 4 v + l / 16 of column l % 16 in register v) is at once the B operand of a
// product over its rows and, read as the A operand, its own transpose, so no block is ever
// transposed in memory.
#include "device_common.h"
#include "internal.h"

#include <algorithm>

namespace ec2moe {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// A block's registers in memory: two planes of [64 lanes][2 doubles] (16-byte accesses of
// consecutive lanes are contiguous).
struct Block64 {
    f64x2 v[2][64];
};

__device__ __forceinline__ f64x4 block_get(const Block64& b, int lane) {
    const f64x2 lo = b.v[0][lane], hi = b.v[1][lane];
    return f64x4{lo[0], lo[1], hi[0], hi[1]};
}
__device__ __forceinline__ void block_put(Block64& b, int lane, f64x4 x) {
    b.v[0][lane] = f64x2{x[0], x[1]};
    b.v[1][lane] = f64x2{x[2], x[3]};
}

// c + A^T B over 16 rows, both blocks in the result layout
__device__ __forceinline__ f64x4 block_update(f64x4 c, f64x4 at, f64x4 b) {
#pragma unroll
    for (int v = 0; v < 4; ++v) c = mfma64(at[v], b[v], c);
    return c;
}

// ------------------------------------------------------------------ Gram matrix
//
// part[z][i][j] = sum over the rows t of chunk z of y[t][i] * y[t][j] in float64, for the 64 x 64
// tiles on and above the diagonal (the factorisation reads no others). One workgroup per (tile,
// chunk of tc rows, side); wave w owns rows 16 w .. of the tile, four blocks. The operands of a
// step of four rows are one float32 per lane straight from global memory (a row's 16 columns are
// one 64-byte piece; the waves of a tile share them through the caches), with kGramU steps of
// loads in flight: the products, 64 cycles each, leave the loads ample time. 4096 x 256: 55 us
// with float64 FMAs on staged rows.
constexpr int kGramB = 64;  // tile
constexpr int kGramU = 8;   // row steps (of 4) whose loads are in flight together

struct GramArgs {
    GramSide s[2];
    int tc[2], chunks[2], tiles[2];  // rows per chunk, chunks, 64-column tiles
    int32_t* zero_status;
};

__global__ __launch_bounds__(256) void gram64_kernel(GramArgs a) {
    if (a.zero_status && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0) *a.zero_status = 0;
    const int q = blockIdx.z, tiles = a.tiles[q], r = a.s[q].r;
    if (static_cast<int>(blockIdx.x) >= tiles * (tiles + 1) / 2 || static_cast<int>(blockIdx.y) >= a.chunks[q]) return;
    int tj = 0;
    while ((tj + 1) * (tj + 2) / 2 <= static_cast<int>(blockIdx.x)) ++tj;
    const int ti = blockIdx.x - tj * (tj + 1) / 2;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, g = lane >> 4;
    const int i0 = ti * kGramB + 16 * wave, j0 = tj * kGramB;
    if (i0 >= r) return;  // r is a multiple of 16
    const int tb = blockIdx.y * a.tc[q], te = min(a.s[q].n, tb + a.tc[q]);
    const float* __restrict__ y = a.s[q].y;
    int cj[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) cj[c] = min(j0 + 16 * c, r - 16) + l16;  // blocks past r repeat the last (not stored)
    f64x4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = f64x4{0.0, 0.0, 0.0, 0.0};
    for (int t0 = tb; t0 < te; t0 += 4 * kGramU) {
        float fi[kGramU], fj[kGramU][4];
#pragma unroll
        for (int u = 0; u < kGramU; ++u) {
            const int t = t0 + 4 * u + g;
            const float* row = y + static_cast<int64_t>(min(t, te - 1)) * r;
            const float x = row[i0 + l16];
            fi[u] = t < te ? x : 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float z = row[cj[c]];
                fj[u][c] = t < te ? z : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < kGramU; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = mfma64(static_cast<double>(fi[u]), static_cast<double>(fj[u][c]), acc[c]);
    }
    double* out = a.s[q].part + static_cast<int64_t>(blockIdx.y) * r * r;
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (j0 + 16 * c < r) {
#pragma unroll
            for (int v = 0; v < 4; ++v) out[static_cast<int64_t>(i0 + 4 * v + g) * r + j0 + 16 * c + l16] = acc[c][v];
        }
}

// g[i][j] = sum over chunks z in order of part[z][i][j], for the tiles the products fill
__global__ __launch_bounds__(256) void gram_reduce_kernel(GramArgs a) {
    const int q = blockIdx.y, r = a.s[q].r;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= r * r || (e / r) / kGramB > (e % r) / kGramB) return;
    const double* src = a.s[q].part + e;
    const int64_t rr = static_cast<int64_t>(r) * r;
    const int chunks = a.chunks[q];
    double sum = 0.0;
    for (int z = 0; z < chunks; z += 16) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = z + u < chunks ? src[(z + u) * rr] : 0.0;
#pragma unroll
        for (int u = 0; u < 16; ++u) sum += v[u];
    }
    a.s[q].g[e] = sum;
}

// ------------------------------------------------------------------ Cholesky factor
//
// G = R^T R for one r x r float64 Gram matrix (r <= 256, a multiple of 16) per workgroup. The
// output is what the solve reads: block (k, i) of the upper triangle at f[i (i + 1) / 2 + k],
// -R_ki in the result layout for k < i, and R_kk^-T as an A operand on the diagonal.
//
// What bounds it is the chain of eliminations, so it runs on blocks and the chain has r / 16
// links instead of r. Per block row k, with Linv = R_kk^-T:
//   P: row k (in LDS) is multiplied by Linv: R_ki for i > k, which is final and goes out;
//   U: every block below takes its rank-16 update, G_ji -= R_kj^T R_ki, and the blocks of row
//      k + 1 go to LDS, while a wave of its own updates the next diagonal block, factors it and
//      inverts the factor.
// The blocks of the triangle live in registers, 4 doubles a lane: 11 workers of at most 13,
// dealt round robin so that those below any k are spread evenly. Everything but R_kk^-T is held
// negated, so that the updates add. The diagonal wave holds one column of [G_kk | I] per lane
// and broadcasts the multipliers by lane reads. A pivot that is not positive sets the status and
// is replaced by 1.
constexpr int kCholB = 16;
constexpr int kCholWorkers = 11;
constexpr int kCholThreads = 64 * (kCholWorkers + 1);
constexpr int kCholMaxB = 16;  // blocks per side at r = 256
constexpr int kCholSlots = (kCholMaxB * (kCholMaxB + 1) / 2 + kCholWorkers - 1) / kCholWorkers;

// 1 / sqrt(d) for d > 0 (the pivots): the hardware estimate y (relative error below 2^-20) with
// one third-order step, y (1 + e / 2 + 3 e^2 / 8) for e = 1 - d y^2, to within a few units in the
// last place of float64
__device__ __forceinline__ double rsqrt64(double d) {
    const double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-d * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

__device__ __forceinline__ double lane_read(double v, int lane) {
    const int2 b = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(b.x, lane), __builtin_amdgcn_readlane(b.y, lane)));
}

struct CholLds {
    Block64 row[kCholMaxB];    // row k before step P
    Block64 panel[kCholMaxB];  // row k after it: R_ki for i > k
    Block64 linv;              // R_kk^-T as the A operand
    Block64 diag[2];           // the diagonal blocks k + 1 and k + 2, by parity
    double tmp[kCholB][kCholB + 2];
    int bad;
};

// Factors the block x (result layout, symmetric) and publishes R^-T.
__device__ __forceinline__ void chol_diag(CholLds& sh, f64x4 x, int lane) {
    asm volatile("" : "+v"(lane));  // keeps the columns of I and the lane tests from being hoisted out of the step loop
    const int l16 = lane & 15, g = lane >> 4;
#pragma unroll
    for (int v = 0; v < 4; ++v) sh.tmp[4 * v + g][l16] = x[v];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // lanes 0..15: column l16 of the block (its row, by symmetry); the others: column l16 of I
    double c[kCholB];
#pragma unroll
    for (int i = 0; i < kCholB; ++i) c[i] = lane < 16 ? sh.tmp[l16][i] : (i == l16 ? 1.0 : 0.0);
    bool bad = false;
#pragma unroll
    for (int p = 0; p < kCholB; ++p) {
        const double d = lane_read(c[p], p);
        const bool pos = d > 0.0;
        bad |= !pos;
        const double s = rsqrt64(d);
        c[p] *= pos ? s : 1.0;
#pragma unroll
        for (int i = p + 1; i < kCholB; ++i) c[i] = fma(-lane_read(c[p], i), c[p], c[i]);
    }
    // lane 16 + j: column j of R^-T, in the A operand at lane 16 (j % 4) + row, register j / 4
    if (g == 1) {
#pragma unroll
        for (int i = 0; i < kCholB; ++i) sh.linv.v[l16 >> 3][16 * (l16 & 3) + i][(l16 >> 2) & 1] = c[i];
        if (bad && l16 == 0) sh.bad = 1;
    }
}

__global__ __launch_bounds__(kCholThreads) void chol_kernel(CholArgs args) {
    __shared__ CholLds sh;
    const CholSide& side = args.s[blockIdx.x];
    const int r = side.r, nb = r / kCholB;
    const double* __restrict__ g64 = side.g;
    Block64* f = static_cast<Block64*>(side.f);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const bool worker = wave < kCholWorkers;
    if (threadIdx.x == 0) sh.bad = 0;

    // slot n of a worker: block (j, i), j <= i, number kCholWorkers n + wave of the column order;
    // it takes part in the steps k < j (k < j - 1 on the diagonal, whose last update and factor
    // are the diagonal wave's)
    int ij[kCholSlots];  // i << 8 | j
    int lim[kCholSlots];
    f64x4 m[kCholSlots];
#pragma unroll
    for (int n = 0; n < kCholSlots; ++n) {
        const int t = kCholWorkers * n + wave;
        int i = 0;
        while ((i + 1) * (i + 2) / 2 <= t) ++i;
        const int j = t - i * (i + 1) / 2;
        const bool used = worker && i < nb;
        ij[n] = __builtin_amdgcn_readfirstlane(used ? i << 8 | j : 0);
        lim[n] = __builtin_amdgcn_readfirstlane(used ? (i == j ? j - 1 : j) : -1);
        m[n] = f64x4{0.0, 0.0, 0.0, 0.0};
        if (used) {
#pragma unroll
            for (int v = 0; v < 4; ++v) m[n][v] = -g64[static_cast<int64_t>(16 * j + 4 * v + g) * r + 16 * i + l16];
            if (i == j && i < 2) block_put(sh.diag[i], lane, m[n]);
            else if (j == 0) block_put(sh.row[i], lane, m[n]);
        }
    }
    __syncthreads();
    if (!worker) chol_diag(sh, -block_get(sh.diag[0], lane), lane);
    __syncthreads();

    for (int k = 0; k < nb; ++k) {
        const f64x4 la = block_get(sh.linv, lane);
        for (int b = k + wave; b < nb; b += kCholWorkers + 1) {
            f64x4 x = la;
            if (b > k) {
                const f64x4 y = block_get(sh.row[b], lane);
                x = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int v = 0; v < 4; ++v) x = mfma64(la[v], y[v], x);
                block_put(sh.panel[b], lane, x);
            }
            block_put(f[b * (b + 1) / 2 + k], lane, x);
        }
        if (k + 1 == nb) break;
        __syncthreads();
        if (worker) {
#pragma unroll
            for (int n = 0; n < kCholSlots; ++n) {
                if (k >= lim[n]) continue;
                const int i = ij[n] >> 8, j = ij[n] & 255;
                m[n] = block_update(m[n], block_get(sh.panel[j], lane), block_get(sh.panel[i], lane));
                if (i == j) {
                    if (j == k + 2) block_put(sh.diag[k & 1], lane, m[n]);
                } else if (j == k + 1) {
                    block_put(sh.row[i], lane, m[n]);
                }
            }
        } else {
            const f64x4 x = block_get(sh.panel[k + 1], lane);
            chol_diag(sh, -block_update(block_get(sh.diag[(k + 1) & 1], lane), x, x), lane);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0 && args.status && sh.bad) atomicOr(args.status, 1);
}

// ------------------------------------------------------------------ Q = Y R^-1
//
// Forward substitution on Q^T = R^-T Y^T without ever forming the inverse: a wave holds 16 rows of
// Y as the 16 x 16 blocks of Y^T in float64 registers; per block row k, Q^T_k = R_kk^-T Y^T_k and
// Y^T_j -= R_kj^T Q^T_k for j > k (as many products as a multiplication by the triangular
// inverse, which would cost the factorisation twice its products). The factor's row k + 1 is
// loaded while row k is applied from LDS. Out: float32 [n][r], or [r][ldt] with zeros past n.
constexpr int kSolveWaves = 4;

__global__ __launch_bounds__(64 * kSolveWaves, 1) void solve_kernel(SolveArgs args) {
    __shared__ Block64 fr[2][kCholMaxB];
    const SolveSide& side = args.s[blockIdx.y];
    const int n = side.n, r = side.r, nb = r / kCholB;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, g = lane >> 4;
    if (static_cast<int>(blockIdx.x) * 16 * kSolveWaves >= n) return;
    const Block64* f = static_cast<const Block64*>(side.f);
    const int t = (blockIdx.x * kSolveWaves + wave) * 16 + l16;
    const bool live = t < (side.ldt ? side.ldt : n);  // n <= ldt <= n + 3, inside the last workgroup's 64 rows
    const float* __restrict__ yrow = side.y + static_cast<int64_t>(min(t, n - 1)) * r + g;
    f64x4 m[kCholMaxB];
#pragma unroll
    for (int j = 0; j < kCholMaxB; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) m[j][v] = j < nb ? static_cast<double>(yrow[16 * j + 4 * v]) : 0.0;

    // row k of the factor: blocks (k, j), j >= k; thread t moves 16-byte piece t % 128 of blocks
    // t / 128 + 2 q past k
    constexpr int Q = kCholMaxB * 128 / (64 * kSolveWaves);
    const int piece = tid & 127, b0 = tid >> 7;
    f64x2 st[Q];
    auto load = [&](int k) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int j = k + b0 + 2 * q;
            if (j < nb) st[q] = (&f[j * (j + 1) / 2 + k].v[0][0])[piece];
        }
    };
    load(0);
#pragma unroll
    for (int k = 0; k < kCholMaxB; ++k) {
        if (k < nb) {
            Block64* cur = fr[k & 1];
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (k + b0 + 2 * q < nb) (&cur[k + b0 + 2 * q].v[0][0])[piece] = st[q];
            __syncthreads();
            if (k + 1 < nb) load(k + 1);
            const f64x4 la = block_get(cur[k], lane);
            f64x4 x = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int v = 0; v < 4; ++v) x = mfma64(la[v], m[k][v], x);
#pragma unroll
            for (int j = k + 1; j < kCholMaxB; ++j)
                if (j < nb) m[j] = block_update(m[j], block_get(cur[j], lane), x);  // the factor's blocks are -R_kj
            if (live) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * k + 4 * v + g;
                    const int64_t at = side.ldt ? static_cast<int64_t>(i) * side.ldt + t : static_cast<int64_t>(t) * r + i;
                    side.out[at] = t < n ? static_cast<float>(x[v]) : 0.f;
                }
            }
        }
    }
}

// xu[t][s*w + j] = x[s][t][j]: the mode-1 unfolding of c slices [c][h][w] (16-byte chunks)
template <typename T>
__global__ __launch_bounds__(256) void unfold_kernel(const T* __restrict__ x, int c, int h, int w, T* __restrict__ xu) {
    constexpr int EPC = 16 / static_cast<int>(sizeof(T));
    const int64_t chunks = static_cast<int64_t>(c) * h * (w / EPC);
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; e < chunks;
         e += static_cast<int64_t>(gridDim.x) * 256) {
        const int64_t row = e / (w / EPC);  // s * h + t
        const int j = static_cast<int>(e % (w / EPC)) * EPC;
        const int s = static_cast<int>(row / h), t = static_cast<int>(row % h);
        *reinterpret_cast<uint4*>(xu + static_cast<int64_t>(t) * c * w + static_cast<int64_t>(s) * w + j) =
            *reinterpret_cast<const uint4*>(x + row * w + j);
    }
}

}  // namespace

int gram64_chunks(int n, int r) {
    const int tiles = (r + kGramB - 1) / kGramB;
    const int want = std::max(1, 256 / (tiles * (tiles + 1) / 2));  // about one workgroup per CU and side
    const int tc = std::max(4 * kGramU, (n + want - 1) / want);
    return (n + tc - 1) / tc;
}

hipError_t launch_gram64(const GramSide (&sides)[2], int32_t* zero_status, hipStream_t s) {
    GramArgs a{};
    a.zero_status = zero_status;
    int pairs = 0, chunks = 0, rr = 0;
    for (int q = 0; q < 2; ++q) {
        a.s[q] = sides[q];
        a.chunks[q] = gram64_chunks(sides[q].n, sides[q].r);
        a.tc[q] = (sides[q].n + a.chunks[q] - 1) / a.chunks[q];
        a.tiles[q] = (sides[q].r + kGramB - 1) / kGramB;
        pairs = std::max(pairs, a.tiles[q] * (a.tiles[q] + 1) / 2);
        chunks = std::max(chunks, a.chunks[q]);
        rr = std::max(rr, sides[q].r * sides[q].r);
    }
    {
        ProfileScope prof("fit_gram", s);
        hipLaunchKernelGGL(gram64_kernel, dim3(pairs, chunks, 2), dim3(256), 0, s, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    ProfileScope prof("fit_gram_reduce", s);
    hipLaunchKernelGGL(gram_reduce_kernel, dim3((rr + 255) / 256, 2), dim3(256), 0, s, a);
    return hipGetLastError();
}

size_t chol_factor_bytes(int r) {
    const size_t nb = static_cast<size_t>(r) / kCholB;
    return nb * (nb + 1) / 2 * sizeof(Block64);
}

hipError_t launch_chol(const CholArgs& a, hipStream_t s) {
    ProfileScope prof("fit_chol", s);
    hipLaunchKernelGGL(chol_kernel, dim3(2), dim3(kCholThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_solve(const SolveArgs& a, hipStream_t s) {
    const int rows = std::max(a.s[0].n, a.s[1].n);
    ProfileScope prof("fit_qr", s);
    hipLaunchKernelGGL(solve_kernel, dim3((rows + 16 * kSolveWaves - 1) / (16 * kSolveWaves), 2), dim3(64 * kSolveWaves), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_unfold(DType dt, const void* x, int c, int h, int w, void* xu, hipStream_t s) {
    const int64_t chunks = static_cast<int64_t>(c) * h * w * static_cast<int64_t>(elem_bytes(dt)) / 16;
    const int grid = static_cast<int>(std::min<int64_t>((chunks + 255) / 256, 4096));
    ProfileScope prof("fit_unfold", s);
    if (dt == DType::BF16)
        hipLaunchKernelGGL(unfold_kernel<bf16_t>, dim3(grid), dim3(256), 0, s, static_cast<const bf16_t*>(x), c, h, w,
                           static_cast<bf16_t*>(xu));
    else
        hipLaunchKernelGGL(unfold_kernel<float>, dim3(grid), dim3(256), 0, s, static_cast<const float*>(x), c, h, w,
                           static_cast<float*>(xu));
    return hipGetLastError();
}

}  // namespace ec2moe
