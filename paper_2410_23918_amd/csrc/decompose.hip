// The compression half of the method on the device: activation-aware scaling (Eq. 3-4) and the
// iterative absolute value decomposition (Section 2.1.2, Eq. 5-7; the decomposition loop of the
// overall algorithm in the appendix).  Per block i:
//
//     S_i = sign(R_i)  (sign(0) = +1),   |R_i| ~ U_i V_i^T  (top k = 16 singular triplets, sqrt(sigma)
//     split of Eq. 2, factors rounded to fp16),   R_{i+1} = R_i - S_i (.) (U_i V_i^T)   (Eq. 6)
//
// "SVD" is a block power (subspace) iteration with k + 16 columns followed by a Rayleigh-Ritz
// step; any method that returns the leading triplets is a valid reading.  The two tall products
// per round, |R| X and |R|^T Y, run on the bf16 matrix cores from bf16 copies of |R| (written once
// per block, as it lies and transposed); the product of the Rayleigh-Ritz step, which fixes U and V,
// reads the fp32 residual (|.| applied as it is loaded); sums are fp32, the 32 x 32 Gram /
// Cholesky / eigenvalue problems fp64.  The sign matrix is never materialised.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <type_traits>

#include "kernels.h"
#include "kparams.h"
#include "layout.h"

namespace bitstack {

typedef float v16f __attribute__((ext_vector_type(16)));

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef double v4d __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

constexpr int kL = 32;        // subspace width: rank 16 + 16 columns of oversampling
constexpr int kDcTile = 128;  // output indices per workgroup of the fp32 product
constexpr int kDcChunk = 32;  // its reduction indices per LDS stage

// Fragment order: a bf16 matrix A (M x K) as the matrix cores take it, [M / 32][K / 16][half][row % 32][8 values of K], so that
// a wavefront's operand for 32 rows and 16 reduction indices is 1 KiB in the order of its lanes.  M is a multiple of 32, K of 16.
__device__ __forceinline__ size_t frag_piece(int row, int k8, int K) {   // index of the 16-byte piece with A[row][8 k8 ..]
    return (size_t(row >> 5) * (K >> 4) + (k8 >> 1)) * 64 + (k8 & 1) * 32 + (row & 31);
}

// start vectors: any full-rank matrix will do; a counter-based hash keeps it reproducible.  X (in x kL) in fragment order
// of its transpose: thread = 8 rows of one column.
__device__ __forceinline__ float start_value(unsigned i, unsigned seed) {
    unsigned h = i * 2654435761u ^ seed;
    h ^= h >> 16; h *= 0x85ebca6bu; h ^= h >> 13; h *= 0xc2b2ae35u; h ^= h >> 16;
    return float(int(h >> 8) - (1 << 23)) * (1.0f / float(1 << 23));
}

// fp32 -> bf16, round to nearest even (the residual is finite)
__device__ __forceinline__ unsigned bf16_of(float x) {
    const unsigned u = __float_as_uint(x);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__global__ __launch_bounds__(256) void k_dc_random(uint4* Xf, int in, unsigned seed) {
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= in / 8 * kL) return;
    const int c = idx % kL, k8 = idx / kL;
    unsigned w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
        w[e] = bf16_of(start_value(unsigned((8 * k8 + 2 * e) * kL + c), seed)) |
               bf16_of(start_value(unsigned((8 * k8 + 2 * e + 1) * kL + c), seed)) << 16;
    Xf[frag_piece(c, k8, in)] = make_uint4(w[0], w[1], w[2], w[3]);
}

// One pass over the residual per block: the first block's residual R = W diag(s), every later one's R <- R - sign(R) (.) (U V^T)
// with the previous block's factors as stored (fp16); from it the canonical sign words of the block (bit b of word w of a row =
// (R[row][32 w + b] >= 0), -0.0 and 0.0 both count as +1) and |R| as bf16, as it lies (Rh) and transposed (RhT), both in fragment
// order.  128 rows x 64 columns per workgroup; a thread owns 8 consecutive columns of 4 rows.  Bound by memory: 12 bytes per
// element.  4096 x 4096: 37 us for the first block and 47 us for a later one, where scaling, packing of the signs, conversion
// and update as kernels of their own took about 90 and 120.
constexpr int kResRows = 128, kResCols = 64, kResLd = kResCols + 8;
template <bool FIRST>
__global__ __launch_bounds__(256) void k_dc_residual(const float* W, const float* s, float* R, const __half* U, const __half* V,
                                                     uint32_t* words, uint4* Rh, uint4* RhT, int out, int in) {
    __shared__ float Us[FIRST ? 1 : kResRows][kRank + 4];
    __shared__ float Vs[FIRST ? 1 : kResCols][kRank + 4];
    __shared__ __attribute__((aligned(16))) unsigned short Ts[kResRows][kResLd];
    const int tid = threadIdx.x;
    const int o0 = blockIdx.y * kResRows, j0 = blockIdx.x * kResCols;   // in is a multiple of 64, out of 32
    const int oct = tid & 7, r0 = tid >> 3;   // rows r0 + 32 i
    const float* const src = FIRST ? W : R;
    float x[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const size_t at = size_t(min(o0 + r0 + 32 * i, out - 1)) * in + j0 + 8 * oct;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float4 v = *reinterpret_cast<const float4*>(src + at + 4 * q);
            x[i][4 * q] = v.x; x[i][4 * q + 1] = v.y; x[i][4 * q + 2] = v.z; x[i][4 * q + 3] = v.w;
        }
    }
    if constexpr (FIRST) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float sc = s[j0 + 8 * oct + e];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i][e] *= sc;
        }
    } else {
        for (int idx = tid; idx < kResRows * kRank; idx += 256) {
            const int r = idx / kRank, c = idx % kRank;
            Us[r][c] = __half2float(U[size_t(min(o0 + r, out - 1)) * kRank + c]);
        }
        for (int idx = tid; idx < kResCols * kRank; idx += 256) {   // column 8 o + e in row 8 e + o: a wavefront's reads are spread over the banks
            const int j = idx / kRank, c = idx % kRank;
            Vs[(j & 7) * 8 + (j >> 3)][c] = __half2float(V[size_t(j0 + j) * kRank + c]);
        }
        __syncthreads();
        float m[4][8];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) m[i][e] = 0.f;
#pragma unroll
        for (int c = 0; c < kRank; c += 4) {
            float4 u[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) u[i] = *reinterpret_cast<const float4*>(&Us[r0 + 32 * i][c]);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float4 v = *reinterpret_cast<const float4*>(&Vs[e * 8 + oct][c]);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    m[i][e] = fmaf(u[i].w, v.w, fmaf(u[i].z, v.z, fmaf(u[i].y, v.y, fmaf(u[i].x, v.x, m[i][e]))));
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) x[i][e] = (x[i][e] < 0.0f) ? x[i][e] + m[i][e] : x[i][e] - m[i][e];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int o = o0 + r0 + 32 * i;
        unsigned h[4], bits = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) bits |= (x[i][e] < 0.0f) ? 0u : 1u << e;
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = bf16_of(fabsf(x[i][2 * e])) | bf16_of(fabsf(x[i][2 * e + 1])) << 16;
        *reinterpret_cast<uint4*>(&Ts[r0 + 32 * i][8 * oct]) = make_uint4(h[0], h[1], h[2], h[3]);
        bits <<= 8 * (oct & 3);   // the four lanes of a word are neighbours
        bits |= __shfl_xor(bits, 1);
        bits |= __shfl_xor(bits, 2);
        if (o < out) {
            float* const dst = R + size_t(o) * in + j0 + 8 * oct;
            *reinterpret_cast<float4*>(dst) = make_float4(x[i][0], x[i][1], x[i][2], x[i][3]);
            *reinterpret_cast<float4*>(dst + 4) = make_float4(x[i][4], x[i][5], x[i][6], x[i][7]);
            if ((oct & 3) == 0) words[size_t(o) * (in / 32) + j0 / 32 + oct / 4] = bits;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {   // pieces of Rh: consecutive lanes take consecutive rows
        const int idx = tid + 256 * i, r = idx % kResRows, k8 = idx / kResRows;
        if (o0 + r < out) Rh[frag_piece(o0 + r, j0 / 8 + k8, in)] = *reinterpret_cast<const uint4*>(&Ts[r][8 * k8]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {   // pieces of RhT: consecutive lanes take consecutive columns
        const int idx = tid + 256 * i, c = idx % kResCols, k8 = idx / kResCols;
        unsigned w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = unsigned(Ts[8 * k8 + 2 * e][c]) | unsigned(Ts[8 * k8 + 2 * e + 1][c]) << 16;
        if (o0 + 8 * k8 < out) RhT[frag_piece(j0 + c, o0 / 8 + k8, out)] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// The product of the Rayleigh-Ritz step, from the fp32 residual on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: 32 output
// indices x 32 columns, two reduction indices per instruction):
//   P[slice][j][c] = sum_{o in slice} |R[o][j]| X[o][c]     (M = in, K = out)
// A workgroup (4 wavefronts) owns 128 output indices and one slice of the reduction range; the residual chunk goes to LDS
// as As[reduction index][output index] (|.| applied on the way), the next chunk's loads in flight during the products (4096 x 4096: 22
// -> 17 us).  The slices are added up by the kernel that reads the product.
__global__ __launch_bounds__(256) void k_dc_mul(const float* R, const float* X, float* P, int out, int in, int chunks_per_slice) {
    __shared__ float As[kDcChunk][kDcTile + 4];
    __shared__ float Xs[kDcChunk][kL];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hl = lane >> 5, ln = lane & 31;
    const int m0 = blockIdx.x * kDcTile;
    const int chunks = out / kDcChunk;
    const int c_begin = blockIdx.y * chunks_per_slice;
    const int c_end = min(chunks, c_begin + chunks_per_slice);
    v16f acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    float4 a[4], x;
    auto request = [&](int ch) {
        const int k0 = ch * kDcChunk;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int idx = tid + 256 * i, kk = idx >> 5, q = idx & 31;   // row k0 + kk, columns m0 + 4 q ..
            a[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (m0 + 4 * q < in) a[i] = *reinterpret_cast<const float4*>(R + size_t(k0 + kk) * in + m0 + 4 * q);
        }
        x = *reinterpret_cast<const float4*>(X + size_t(k0 + (tid >> 3)) * kL + 4 * (tid & 7));
    };
    if (c_begin < c_end) request(c_begin);
    for (int ch = c_begin; ch < c_end; ++ch) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int idx = tid + 256 * i, kk = idx >> 5, q = idx & 31;
            *reinterpret_cast<float4*>(&As[kk][4 * q]) = make_float4(fabsf(a[i].x), fabsf(a[i].y), fabsf(a[i].z), fabsf(a[i].w));
        }
        *reinterpret_cast<float4*>(&Xs[tid >> 3][4 * (tid & 7)]) = x;
        lds_barrier();
        if (ch + 1 < c_end) request(ch + 1);
#pragma unroll
        for (int kk = 0; kk < kDcChunk; kk += 2)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(As[kk + hl][wave * 32 + ln], Xs[kk + hl][ln], acc, 0, 0, 0);
        lds_barrier();
    }
    // D[i = output index][n = column]: lane (column ln), register v holds index 8*(v/4) + 4*hl + v%4
    float* Ps = P + size_t(blockIdx.y) * in * kL;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int m = m0 + wave * 32 + 8 * (v >> 2) + 4 * hl + (v & 3);
        if (m < in) Ps[size_t(m) * kL + ln] = acc[v];
    }
}

// The power rounds' tall products on the bf16 matrix cores: P[slice][m][c] = sum_{k in slice} A[m][k] X[k][c] with A = Rh (M =
// out, K = in) or RhT (M = in, K = out) and the transpose of X (K x kL, rounded to bf16 by the kernel that made it), both in
// fragment order: an operand is one coalesced load of 1 KiB, and nothing goes through LDS or waits at a barrier.  A
// perturbation of |R| and of the iterate of 2^-9 relative per element turns the subspace the rounds converge to by far less
// than the oversampling and the Rayleigh-Ritz step, which works on the fp32 residual, absorb.  A workgroup owns TILES x 32
// output indices (two tiles, so that an operand of X serves two, where the grid fills the chip with them) and four slices of
// the reduction range, one for each of its wavefronts; they add up in LDS.  Bound by the loads of A, of which every wavefront
// keeps 16 KiB in flight: 4096 x 4096 8.4 us a product (8.9 with 8 KiB; through LDS, from row-major copies: 11.5), 14336 x 4096 20 us
// (24-49).
template <int TILES, int AHEAD>
__global__ __launch_bounds__(256) void k_dc_mulh(const uint4* A, const uint4* X, float* P, int M, int K, int steps_per_wave) {
    __shared__ float red[4][TILES][16][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int steps = K >> 4, tile0 = blockIdx.x * TILES;
    const int s_begin = min(steps, (int(blockIdx.y) * 4 + wave) * steps_per_wave), s_end = min(steps, s_begin + steps_per_wave);
    const uint4* const x0 = X + lane;
    const uint4* a0[TILES];
    v16f acc[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        a0[t] = A + size_t(min(tile0 + t, (M >> 5) - 1)) * steps * 64 + lane;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
    }
    auto products = [&](auto count, int st) __attribute__((always_inline)) {
        constexpr int N = decltype(count)::value;
        uint4 a[N][TILES], x[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
#pragma unroll
            for (int t = 0; t < TILES; ++t) a[u][t] = a0[t][size_t(st + u) * 64];
            x[u] = x0[size_t(st + u) * 64];
        }
        __builtin_amdgcn_sched_barrier(0);   // all requests before the first product
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int t = 0; t < TILES; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a[u][t]), __builtin_bit_cast(v8bf, x[u]), acc[t], 0, 0, 0);
    };
    int st = s_begin;
    for (; st + AHEAD <= s_end; st += AHEAD) products(std::integral_constant<int, AHEAD>{}, st);
    for (; st + 2 <= s_end; st += 2) products(std::integral_constant<int, 2>{}, st);   // K is a multiple of 32
#pragma unroll
    for (int t = 0; t < TILES; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) red[wave][t][v][lane] = acc[t][v];
    __syncthreads();
    // D[i = output index][n = column]: lane (column l % 32), register v holds index 8*(v/4) + 4*(l/32) + v%4
    float* Ps = P + size_t(blockIdx.y) * M * kL;
#pragma unroll
    for (int i = 0; i < TILES * 32 * kL / 256; ++i) {
        const int o = tid + 256 * i, l = o & 63, v = (o >> 6) & 15, t = o >> 10;
        const int m = (tile0 + t) * 32 + 8 * (v >> 2) + 4 * (l >> 5) + (v & 3);
        if (m < M) Ps[size_t(m) * kL + (l & 31)] = (red[0][t][v][l] + red[1][t][v][l]) + (red[2][t][v][l] + red[3][t][v][l]);
    }
}

// four columns of one row of a product, its slices added up: in groups of four as they lie (the fp32 product's slices), or one
// by one (slices that are such groups already); the order of the additions is that of four slices to a group either way
__device__ __forceinline__ float4 slice_sum(const float* src, int slices, size_t n, bool grouped) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int sl = 0; sl < slices; sl += 4) {
        float4 a[4];   // in flight together
#pragma unroll
        for (int u = 0; u < 4; ++u)
            a[u] = sl + u < slices ? *reinterpret_cast<const float4*>(src + size_t(sl + u) * n) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (grouped || sl + 4 > slices) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                v.x += a[u].x; v.y += a[u].y; v.z += a[u].z; v.w += a[u].w;
            }
        } else {
            v.x += (a[0].x + a[1].x) + (a[2].x + a[3].x); v.y += (a[0].y + a[1].y) + (a[2].y + a[3].y);
            v.z += (a[0].z + a[1].z) + (a[2].z + a[3].z); v.w += (a[0].w + a[1].w) + (a[2].w + a[3].w);
        }
    }
    return v;
}

// 8 rows k8 of column c of a matrix in LDS (rows ld floats apart) as one piece of its transpose's fragment order
__device__ __forceinline__ uint4 bf16_piece(const float* col, int ld) {
    unsigned w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = bf16_of(col[2 * e * ld]) | bf16_of(col[(2 * e + 1) * ld]) << 16;
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// a product's slices added up and rounded to bf16 in fragment order, as the next product takes it; 32 rows per workgroup
__global__ __launch_bounds__(256) void k_dc_sum(const float* P, int slices, uint4* Xf, int m) {
    __shared__ float Ys[32][kL + 1];
    const int tid = threadIdx.x, r = tid >> 3, cq = tid & 7, row0 = blockIdx.x * 32;   // m is a multiple of 32
    const float4 v = slice_sum(P + size_t(row0 + r) * kL + 4 * cq, slices, size_t(m) * kL, true);
    Ys[r][4 * cq] = v.x; Ys[r][4 * cq + 1] = v.y; Ys[r][4 * cq + 2] = v.z; Ys[r][4 * cq + 3] = v.w;
    __syncthreads();
    if (tid < 4 * kL) {
        const int c = tid % kL, k8 = tid / kL;
        Xf[frag_piece(c, row0 / 8 + k8, m)] = bf16_piece(&Ys[8 * k8][c], kL + 1);
    }
}

// Y = sum of the product's slices (written out) and this workgroup's part of Y^T Y in fp64: stages of 128 rows of Y (m x kL),
// 16 wavefronts.  Wavefront w multiplies, on the fp64 matrix cores (v_mfma_f64_16x16x4_f64), a quarter of a stage's rows into
// one of the four 16 x 16 tiles of the part; the quarters are added up in LDS.  The parts (at most kGramParts) are added up
// in a fixed order by the kernel that consumes the Gram matrix (no atomics: the decomposition is reproducible bit for
// bit).  4096 rows: 4.4 us (12 with 256 threads to 128 rows and fp64 vector arithmetic).
constexpr int kGramRows = 128, kGramParts = 64;
__host__ __device__ inline int gram_stages(int m) { return (m + kGramRows * kGramParts - 1) / (kGramRows * kGramParts); }
inline int gram_parts(int m) { return (m + kGramRows * gram_stages(m) - 1) / (kGramRows * gram_stages(m)); }
__global__ __launch_bounds__(1024) void k_dc_gram(const float* P, int slices, bool grouped, float* Y, int m, double* Gpart) {
    __shared__ float Ys[kGramRows][kL + 1];
    __shared__ double Gq[4][kL * kL];
    const int tid = threadIdx.x, lane = tid & 63, r = tid >> 3, cq = tid & 7;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ti = (wave >> 1) & 1, tj = wave & 1, quarter = wave >> 2;
    const int stages = gram_stages(m);
    v4d acc = {0.0, 0.0, 0.0, 0.0};
    for (int st = 0; st < stages; ++st) {
        const int row = (blockIdx.x * stages + st) * kGramRows + r;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row < m) {
            v = slice_sum(P + size_t(row) * kL + 4 * cq, slices, size_t(m) * kL, grouped);
            *reinterpret_cast<float4*>(Y + size_t(row) * kL + 4 * cq) = v;
        }
        if (st) __syncthreads();
        Ys[r][4 * cq] = v.x; Ys[r][4 * cq + 1] = v.y; Ys[r][4 * cq + 2] = v.z; Ys[r][4 * cq + 3] = v.w;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 8; ++q) {   // operands: lane l holds index l % 16 of row 4 q + l / 16
            const float* const y = Ys[quarter * 32 + 4 * q + (lane >> 4)];
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(double(y[ti * 16 + (lane & 15)]), double(y[tj * 16 + (lane & 15)]), acc, 0, 0, 0);
        }
    }
    // D[i][j]: lane l, register v holds i = 4 v + l / 16, j = l % 16
#pragma unroll
    for (int v = 0; v < 4; ++v) Gq[quarter][(ti * 16 + 4 * v + (lane >> 4)) * kL + tj * 16 + (lane & 15)] = acc[v];
    __syncthreads();
    Gpart[size_t(blockIdx.x) * (kL * kL) + tid] = (Gq[0][tid] + Gq[1][tid]) + (Gq[2][tid] + Gq[3][tid]);
}

// the Gram matrix from its parts, in a fixed order, into LDS: THREADS threads, the loads of 32 values in flight together.  Buffer
// loads: past the last part, in the rest of the array of kGramParts, they bring zeros (the bounds take in the scalar offset;
// tests/test_gpu_decompose_workspace.py fills the array with NaN).  LOWER: without the tile above the diagonal (columns 16 on of rows 0-15), by the first
// 768 of 1024 threads: what a compute unit can take in (256 KiB from 32 parts) is half of the time.
template <int THREADS, bool LOWER>
__device__ __forceinline__ void gram_sum(const double* Gpart, int parts, double (*Gs)[kL + 1]) {
    static_assert(!LOWER || THREADS == kL * kL, "");
    constexpr int N = kL * kL / THREADS, kAhead = 32 / N;
    __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(Gpart), 0, parts * (kL * kL * 8), 0x00020000);
    const int t = int(threadIdx.x);
    int at = t;
    if constexpr (LOWER) {
        if (t >= 768) return;
        at = (t < 256 ? t >> 4 : 16 + ((t >> 4) & 15)) * kL + (t < 512 ? 0 : 16) + (t & 15);
    }
    double acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.0;
#pragma unroll 1
    for (int p0 = 0; p0 < parts; p0 += kAhead) {
        v2u v[kAhead][N];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int i = 0; i < N; ++i)
                v[u][i] = __builtin_amdgcn_raw_buffer_load_b64(src, at * 8, (p0 + u) * (kL * kL * 8) + i * THREADS * 8, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] += __builtin_bit_cast(double, v[u][i]);   // the order of the additions is fixed
    }
#pragma unroll
    for (int i = 0; i < N; ++i) Gs[(i * THREADS + at) / kL][(i * THREADS + at) % kL] = acc[i];
}

// G = Y^T Y = L D L^T (fp64), by one wavefront, G in LDS: in lds.pivoted the columns of L D below (and on) the diagonal, in lds.over the
// reciprocal pivots.  False for an all-zero Y (no direction to normalise).
// The matrix stays in the accumulators of the fp64 matrix cores and is eliminated four columns at a time: every lane takes the four
// columns of its row (lanes 32 on: the same rows again) and the 4 x 4 diagonal block from LDS, eliminates within them by itself, and
// one 16x16x4 product per tile (its four terms one after the other) takes the four columns off what is left.  Each entry meets the same operations in the same order as
// column by column; but there are eight trips through LDS instead of 32, and a loop's code instead of that of 32 steps.
struct FactorLds {
    double panel[kL][4], scaled[kL][4];   // [row][column of the four]: as they are, eliminated and over their pivots
    double pivoted[kL / 4][kL][4];        // [four columns][row][column]: eliminated
    double over[kL];
};
__device__ __forceinline__ bool gram_factor(const double (*Gs)[kL + 1], FactorLds& lds) {
    auto order = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); };   // LDS operations of a wavefront execute in order
    const int lane = threadIdx.x & 63, row = lane >> 4, col = lane & 15, r = lane & 31;
    double tr = 0.0;
#pragma unroll
    for (int k = 0; k < kL; ++k) tr += Gs[k][k];
    if (!(tr > 0.0)) return false;   // uniform over the wavefront
    const double ridge = tr * 1e-13;   // a tiny ridge keeps the factorisation defined if the columns are (numerically) dependent
    // tiles (0, 0), (1, 0), (1, 1), register v: row 16 rt + 4 v + row, column 16 ct + col
    v4d acc[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = (k ? 16 : 0) + 4 * v + row, j = (k == 2 ? 16 : 0) + col;
            acc[k][v] = Gs[i][j] + (i == j ? ridge : 0.0);
        }
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll 1
        for (int q = 0; q < 4; ++q) {
            const int jb = 4 * ct + q;
            order();
            if ((col >> 2) == q) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (ct == 0) lds.panel[4 * v + row][col & 3] = acc[0][v];
                    lds.panel[16 + 4 * v + row][col & 3] = acc[ct ? 2 : 1][v];
                }
            }
            order();
            double d[4][4], p[4];   // the diagonal block's lower half, the lane's row
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                p[a] = lds.panel[r][a];
#pragma unroll
                for (int b = 0; b <= a; ++b) d[a][b] = lds.panel[4 * jb + a][b];
            }
            double w[4], t[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                w[k] = 1.0 / (d[k][k] > 0.0 ? d[k][k] : ridge);
                t[k] = p[k] * w[k];
#pragma unroll
                for (int b = k + 1; b < 4; ++b) {
                    p[b] = fma(-t[k], d[b][k], p[b]);
#pragma unroll
                    for (int a = b; a < 4; ++a) d[a][b] = fma(-(d[a][k] * w[k]), d[b][k], d[a][b]);
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                lds.scaled[r][k] = t[k];
                lds.pivoted[jb][r][k] = p[k];
            }
            if (lane == 0) {
#pragma unroll
                for (int k = 0; k < 4; ++k) lds.over[4 * jb + k] = w[k];
            }
            order();
            // operands: lane l holds index l % 16 of column l / 16
            const double s1 = -lds.scaled[16 + col][row], p1 = lds.pivoted[jb][16 + col][row];
            if (ct == 0) {
                const double s0 = -lds.scaled[col][row], p0 = lds.pivoted[jb][col][row];
                acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(s0, p0, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(s1, p0, acc[1], 0, 0, 0);
            }
            acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(s1, p1, acc[2], 0, 0, 0);
        }
    return true;
}

// q_I += l_I minus for I = C + 1 .. 31, l_I in lane I % 16 of every row of sixteen lanes (lo: I < 16, hi).  The compiler does not fold
// the row operation into the multiply-add, and it does not know that the statement is a vector instruction: lo and hi come from LDS, and
// the values of q are read two instructions behind at the earliest (tests/test_asm_distances_more.py).
template <int I>
__device__ __forceinline__ void fma_row_lane(float& q, float l, float minus) {
    asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(q) : "v"(l), "v"(minus), "n"(I % 16));
}
template <int C, int I = C + 1>
__device__ __forceinline__ void take_off(float (&q)[kL], float lo, float hi, float minus) {
    if constexpr (I < kL) {
        fma_row_lane<I>(q[I], I < 16 ? lo : hi, minus);
        take_off<C, I + 1>(q, lo, hi, minus);
    }
}
// columns C to END - 1; their rows of L are requested together
template <int C, int END>
__device__ __forceinline__ void substitute(float (&q)[kL], const float (&lo)[8], const float (&hi)[8], const float (&diagonal)[8]) {
    if constexpr (C < END) {
        q[C] *= diagonal[C % 8];
        take_off<C>(q, lo[C % 8], hi[C % 8], -q[C]);
        substitute<C + 1, END>(q, lo, hi, diagonal);
    }
}
template <int C>
__device__ __forceinline__ void read_columns(const float (*Lt)[kL], int i, float (&lo)[8], float (&hi)[8], float (&diagonal)[8]) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        lo[k] = Lt[C + k][i];
        hi[k] = Lt[C + k][16 + i];
        diagonal[k] = Lt[C + k][C + k];
    }
}

// Columns made orthonormal: G = Y^T Y = L L^T, Q L^T = Y for every row of Y (m x kL), so that Q = Y L^-T.  Every workgroup factors G by
// itself (parts from cache, summed by 768 threads with 32 loads each in flight) and solves kOrthRows rows, one per thread.  4096 rows:
// 12.3 us, of which the parts take 3.9, the factorisation 4.9 and the substitution 2.0 (16.3 with the factorisation by columns, 4.9 and
// more for its code, and L broadcast from LDS).  Bound by those three chains.
//
// The substitution q_c = (y_c - sum_{i < c} q_i L[c][i]) / L[c][c] runs by columns: once q_c is known it is taken off all later
// entries, which do not depend on each other (the same operations on each entry in the same order as row by row).  A row of sixteen
// lanes keeps a column of L in two registers and the multiply-adds take it from there: read from LDS as every lane needs it, the 528
// broadcast values took 3.7 us.
// Q goes out as fp32 (Q, if not null) and as bf16 in fragment order (Xf).  Q and Y may be the same array.
constexpr int kOrthThreads = 1024, kOrthRows = 128;
__global__ __launch_bounds__(kOrthThreads) void k_dc_orth(const double* Gpart, int parts, const float* Y, float* Q, uint4* Xf, int m) {
    __shared__ double Gs[kL][kL + 1];
    __shared__ FactorLds lds;
    __shared__ __attribute__((aligned(16))) float Lt[kL][kL];   // Lt[c][r] = L[r][c] for c < r, 1 / L[r][r] on the diagonal
    __shared__ float Qs[kOrthRows][kL + 1];
    __shared__ int nonzero;
    const int tid = threadIdx.x, row = blockIdx.x * kOrthRows + tid;
    const bool mine = tid < kOrthRows && row < m;
    float q[kL];
    if (tid < kOrthRows) {
#pragma unroll
        for (int g = 0; g < kL / 4; ++g) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (mine) v = *reinterpret_cast<const float4*>(Y + size_t(row) * kL + 4 * g);
            q[4 * g] = v.x; q[4 * g + 1] = v.y; q[4 * g + 2] = v.z; q[4 * g + 3] = v.w;
        }
    }
    gram_sum<kOrthThreads, true>(Gpart, parts, Gs);
    __syncthreads();
    if (tid < 64) {
        const bool ok = gram_factor(Gs, lds);
        if (tid == 0) nonzero = ok;
    }
    __syncthreads();
    {
        const int c = tid / kL, r = tid % kL;
        const double root = nonzero ? sqrt(lds.over[c]) : 0.0;   // 1 / L[c][c]
        Lt[c][r] = !nonzero ? 0.f : r > c ? float(lds.pivoted[c / 4][r][c % 4] * root) : r == c ? float(root) : 0.f;
    }
    __syncthreads();
    if (tid < kOrthRows) {
        const int i = tid & 15;
        float lo[2][8], hi[2][8], diagonal[2][8];
        read_columns<0>(Lt, i, lo[0], hi[0], diagonal[0]);
        read_columns<8>(Lt, i, lo[1], hi[1], diagonal[1]);
        substitute<0, 8>(q, lo[0], hi[0], diagonal[0]);
        read_columns<16>(Lt, i, lo[0], hi[0], diagonal[0]);
        substitute<8, 16>(q, lo[1], hi[1], diagonal[1]);
        read_columns<24>(Lt, i, lo[1], hi[1], diagonal[1]);
        substitute<16, 24>(q, lo[0], hi[0], diagonal[0]);
        substitute<24, 32>(q, lo[1], hi[1], diagonal[1]);
#pragma unroll
        for (int c = 0; c < kL; ++c) Qs[tid][c] = q[c];
    }
    __syncthreads();
    const int c = tid % kL, k8 = tid / kL;
    if (k8 < kOrthRows / 8 && int(blockIdx.x) * kOrthRows + 8 * k8 < m)
        Xf[frag_piece(c, blockIdx.x * (kOrthRows / 8) + k8, m)] = bf16_piece(&Qs[8 * k8][c], kL + 1);
    if (Q) {
        const int r = tid >> 3, g = tid & 7, at = int(blockIdx.x) * kOrthRows + r;
        if (at < m) *reinterpret_cast<float4*>(Q + size_t(at) * kL + 4 * g) = make_float4(Qs[r][4 * g], Qs[r][4 * g + 1], Qs[r][4 * g + 2], Qs[r][4 * g + 3]);
    }
}

// 1 / sqrt(x) for x > 0 in fp64: the hardware's estimate and two Newton steps
__device__ __forceinline__ double rsqrt64(double x) {
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(y * 0.5, fma(-x * y, y, 1.0), y);
    return y;
}

// U = Q Tu, V = Z Tv (kRank columns), rounded to fp16 (nearest even); 64 rows per workgroup, the out side's first, thread = four
// columns of a row.  One launch for both, 4.5 us at 4096 x 4096; a launch each with a row per thread took 6.3 twice.
__global__ __launch_bounds__(256) void k_dc_apply(const float* Q, const float* Tu, __half* U, int out, const float* Z, const float* Tv,
                                                  __half* V, int in) {
    __shared__ __attribute__((aligned(16))) float Ts[kL][kRank];
    __shared__ float Ys[64][kL + 1];
    const int tid = threadIdx.x, wgs = (out + 63) / 64;
    const bool first = int(blockIdx.x) < wgs;
    const float* const Y = first ? Q : Z;
    const int m = first ? out : in, row0 = (int(blockIdx.x) - (first ? 0 : wgs)) * 64;
    for (int idx = tid; idx < kL * kRank; idx += 256) Ts[idx / kRank][idx % kRank] = (first ? Tu : Tv)[idx];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int idx = tid + 256 * i, r = idx >> 3, q = idx & 7;
        const float4 v = *reinterpret_cast<const float4*>(Y + size_t(min(row0 + r, m - 1)) * kL + 4 * q);
        Ys[r][4 * q] = v.x; Ys[r][4 * q + 1] = v.y; Ys[r][4 * q + 2] = v.z; Ys[r][4 * q + 3] = v.w;
    }
    __syncthreads();
    const int r = tid >> 2, c = 4 * (tid & 3);
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (int i = 0; i < kL; ++i) {
        const float y = Ys[r][i];
        const float4 w = *reinterpret_cast<const float4*>(&Ts[i][c]);
        o.x = fmaf(y, w.x, o.x); o.y = fmaf(y, w.y, o.y); o.z = fmaf(y, w.z, o.z); o.w = fmaf(y, w.w, o.w);
    }
    if (row0 + r >= m) return;
    __half* const dst = (first ? U : V) + size_t(row0 + r) * kRank + c;   // the caller's arrays: two-byte alignment
    dst[0] = __float2half_rn(o.x); dst[1] = __float2half_rn(o.y); dst[2] = __float2half_rn(o.z); dst[3] = __float2half_rn(o.w);
}

// Rayleigh-Ritz step.  With Q orthonormal (out x kL) and Z = |R|^T Q (in x kL), G = Z^T Z =
// H diag(sigma^2) H^T gives the leading triplets of |R|: left vectors Q H, right vectors
// Z H diag(1/sigma).  Tu = H_k diag(sqrt(sigma)), Tv = H_k diag(1/sqrt(sigma)) (Eq. 2's split):
// U = Q Tu, V = Z Tv.  Jacobi rotations in fp64 in the round-robin ordering: 31 rounds of 16
// disjoint pairs per sweep.  The rotations of a round act on A from both sides, so A falls into 16 x 16 independent blocks of
// 2 x 2 (rows of one pair, columns of another): 256 threads take one each and A goes from one buffer to another; the other 256
// take two lines of H each, one round behind, with the rotations that the first left in LDS.  A thread makes its column pair's
// rotation by itself and has its row pair's from the lane that makes that one, so a round needs one barrier.  One launch of one
// workgroup, bound by the rounds' chain (rotation, update, barrier) and their LDS traffic: 100 us (107 with 16 threads making the
// rotations and two barriers a round; 122 with every thread making both of its rotations).
constexpr int kRitzThreads = 512;
__global__ __launch_bounds__(kRitzThreads) void k_dc_ritz(const double* Gpart, int parts, float* Tu, float* Tv, int k) {
    __shared__ double A2[2][kL][kL + 1];
    __shared__ double H[kL][kL + 1];
    __shared__ double cs[2][kL / 2][2];
    __shared__ int order[kL];
    __shared__ double sums[kRitzThreads / 64][2];
    const int t = threadIdx.x;
    gram_sum<kRitzThreads, false>(Gpart, parts, A2[0]);
#pragma unroll
    for (int i = t; i < kL * kL; i += kRitzThreads) H[i / kL][i % kL] = (i / kL == i % kL) ? 1.0 : 0.0;
    if (t < kL) order[t] = t;
    __syncthreads();
    const int e = t & (kL / 2 - 1), f = (t >> 4) & (kL / 2 - 1);   // pair of the columns, pair of the rows (or line of H)
    // pair i of a round: (kL - 1, round) and ((round + i) mod 31, (round - i) mod 31), the smaller index first
    auto pair = [](int round, int i, int& p, int& q) {
        const int a = i == 0 ? kL - 1 : round + i < kL - 1 ? round + i : round + i - (kL - 1);
        const int b = round >= i ? round - i : round - i + (kL - 1);
        p = min(a, b);
        q = max(a, b);
    };
    auto rotation = [](double app, double aqq, double apq, double& c, double& s) {
        // tan(2 theta) = b / d; the smaller angle: cos^2 = (1 + |d| / h) / 2, sin = b sign(d) / (2 h cos)
        const double d = aqq - app, b = 2.0 * apq;
        const double rh = rsqrt64(fma(d, d, b * b));
        const double c2 = fma(0.5 * fabs(d), rh, 0.5), rc = rsqrt64(c2);
        const bool turn = fabs(apq) > 1e-300 && apq * apq > 1e-36 * fabs(app * aqq);
        c = turn ? c2 * rc : 1.0;
        s = turn ? (d >= 0.0 ? 0.5 : -0.5) * b * rh * rc : 0.0;
    };
    int cur = 0;
    for (int sweep = 0; sweep < 10; ++sweep) {
        // converged?  (off-diagonal mass against the trace; falls quadratically once small)
        double off = 0.0, tr = 0.0;
#pragma unroll
        for (int i = t; i < kL * kL; i += kRitzThreads) {
            const double v = A2[cur][i / kL][i % kL];
            if (i / kL == i % kL) tr += fabs(v);
            else off += v * v;
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            off += __shfl_xor(off, d);
            tr += __shfl_xor(tr, d);
        }
        if ((t & 63) == 0) {
            sums[t >> 6][0] = off;
            sums[t >> 6][1] = tr;
        }
        __syncthreads();
        off = tr = 0.0;
#pragma unroll
        for (int w = 0; w < kRitzThreads / 64; ++w) {
            off += sums[w][0];
            tr += sums[w][1];
        }
        if (off <= 1e-26 * tr * tr) break;   // same for every thread
        for (int round = 0; round < kL; ++round) {   // H is a round behind
            int p, q;
            if (t < 256) {
                if (round < kL - 1) {
                    double(*const A)[kL + 1] = A2[cur];
                    double(*const next)[kL + 1] = A2[cur ^ 1];
                    int g, h;
                    pair(round, e, p, q);
                    pair(round, f, g, h);
                    const double gp = A[g][p], gq = A[g][q], hp = A[h][p], hq = A[h][q];
                    double c, sn;
                    rotation(A[p][p], A[q][q], A[p][q], c, sn);
                    if (t < kL / 2) {
                        cs[round & 1][t][0] = c;
                        cs[round & 1][t][1] = sn;
                    }
                    const double cr = __shfl(c, f, 16), sr = __shfl(sn, f, 16);   // lane e = f of the same row of sixteen lanes
                    const double gp1 = c * gp - sn * gq, gq1 = sn * gp + c * gq, hp1 = c * hp - sn * hq, hq1 = sn * hp + c * hq;
                    next[g][p] = cr * gp1 - sr * hp1;
                    next[g][q] = cr * gq1 - sr * hq1;
                    next[h][p] = sr * gp1 + cr * hp1;
                    next[h][q] = sr * gq1 + cr * hq1;
                }
            } else if (round > 0) {
                pair(round - 1, e, p, q);
                const double c = cs[(round - 1) & 1][e][0], sn = cs[(round - 1) & 1][e][1];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int r = f + 16 * i;
                    const double hp = H[r][p], hq = H[r][q];
                    H[r][p] = c * hp - sn * hq;
                    H[r][q] = sn * hp + c * hq;
                }
            }
            __syncthreads();
            if (round < kL - 1) cur ^= 1;
        }
    }
    double(*const A)[kL + 1] = A2[cur];
    if (t < kL) {   // eigenvalues in descending order (equal ones by their index)
        const double mine = A[t][t];
        int rank = 0;
        for (int i = 0; i < kL; ++i) rank += (A[i][i] > mine || (A[i][i] == mine && i < t)) ? 1 : 0;
        order[rank] = t;
    }
    __syncthreads();
    for (int i = t; i < kL * k; i += kRitzThreads) {
        const int r = i % k, line = i / k, o = order[r];
        const double lam = A[o][o] > 0.0 ? A[o][o] : 0.0;
        const double sig = sqrt(lam);
        const double rt = sqrt(sig);
        Tu[line * k + r] = float(H[line][o] * rt);
        Tv[line * k + r] = rt > 0.0 ? float(H[line][o] / rt) : 0.f;
    }
}

size_t decompose_workspace_bytes(int out, int in, int slices) {
    const size_t mx = size_t(out > in ? out : in);
    size_t b = align256(size_t(out) * in * 4);               // R
    b += 2 * align256(size_t(out) * in * 2);                 // |R| as bf16 and its transpose
    b += 2 * align256(size_t(out) * kL * 4);                 // Y, Q (out side)
    b += align256(size_t(in) * kL * 4);                      // Z (in side)
    b += align256(mx * kL * 2);                              // the iterate as bf16
    b += align256(size_t(slices) * mx * kL * 4);             // partial products
    b += align256(size_t(kGramParts) * (kL * kL * 8)) + 2 * align256(kL * kL * 4);  // Gram parts, Tu, Tv
    return b;
}

int decompose_slices(int out, int in) {
    // enough workgroups of the fp32 product for 256 compute units: 128 output indices x one slice each
    const int tiles = ((out < in ? out : in) + kDcTile - 1) / kDcTile;
    int s = 1;
    while (tiles * s < 512 && s < 16) s *= 2;
    return s;
}

hipError_t launch_decompose(const float* W, const float* s, int out, int in, int n, int iters, uint32_t* sign_words,
                            __half* U, __half* V, unsigned char* ws, hipStream_t st) {
    const int slices = decompose_slices(out, in);
    const size_t mx = size_t(out > in ? out : in);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        unsigned char* p = ws + off;
        off += align256(bytes);
        return p;
    };
    float* R = reinterpret_cast<float*>(take(size_t(out) * in * 4));
    uint4* Rh = reinterpret_cast<uint4*>(take(size_t(out) * in * 2));
    uint4* RhT = reinterpret_cast<uint4*>(take(size_t(out) * in * 2));
    float* Y = reinterpret_cast<float*>(take(size_t(out) * kL * 4));
    float* Q = reinterpret_cast<float*>(take(size_t(out) * kL * 4));
    float* Z = reinterpret_cast<float*>(take(size_t(in) * kL * 4));
    uint4* X = reinterpret_cast<uint4*>(take(mx * kL * 2));   // of either side: a product has read it before the next one is made
    float* P = reinterpret_cast<float*>(take(size_t(slices) * mx * kL * 4));
    double* G = reinterpret_cast<double*>(take(size_t(kGramParts) * (kL * kL * 8)));
    float* Tu = reinterpret_cast<float*>(take(kL * kL * 4));
    float* Tv = reinterpret_cast<float*>(take(kL * kL * 4));

    // P = slices of |R| X  (X: in x kL)  or of  |R|^T X  (X: out x kL), from the bf16 copies; four of `slices` to a workgroup.
    // Two tiles to a wavefront from two workgroups per compute unit on.
    const int groups = (slices + 3) / 4;
    auto mul = [&](bool trans) {
        const int M = trans ? in : out, K = trans ? out : in;
        const int per = 4 * (((K + 63) / 64 + 4 * groups - 1) / (4 * groups));
        if ((M + 63) / 64 * groups >= 512)
            hipLaunchKernelGGL((k_dc_mulh<2, 8>), dim3((M + 63) / 64, groups), dim3(256), 0, st, trans ? RhT : Rh, X, P, M, K, per);
        else
            hipLaunchKernelGGL((k_dc_mulh<1, 16>), dim3(M / 32, groups), dim3(256), 0, st, trans ? RhT : Rh, X, P, M, K, per);
    };
    auto gram = [&](const float* src, int sl, bool grouped, float* dst, int m) {
        hipLaunchKernelGGL(k_dc_gram, dim3(gram_parts(m)), dim3(1024), 0, st, src, sl, grouped, dst, m, G);
    };
    // the product in P, added up, its columns made orthonormal into X (and Q): Cholesky QR with the Gram matrix in fp64; a
    // second pass (twice = orthonormal to rounding) where asked
    auto orth = [&](bool twice) {
        gram(P, groups, true, Y, out);
        hipLaunchKernelGGL(k_dc_orth, dim3((out + kOrthRows - 1) / kOrthRows), dim3(kOrthThreads), 0, st, G, gram_parts(out), Y, twice ? Q : nullptr, X, out);
        if (twice) {
            gram(Q, 1, true, Y, out);
            hipLaunchKernelGGL(k_dc_orth, dim3((out + kOrthRows - 1) / kOrthRows), dim3(kOrthThreads), 0, st, G, gram_parts(out), Y, Q, X, out);
        }
    };

    const dim3 tiles(in / kResCols, (out + kResRows - 1) / kResRows);
    for (int i = 0; i < n; ++i) {
        uint32_t* sw = sign_words + size_t(i) * out * (in / 32);
        __half* Ui = U + size_t(i) * out * kRank;
        __half* Vi = V + size_t(i) * in * kRank;
        if (i == 0)
            hipLaunchKernelGGL(k_dc_residual<true>, tiles, dim3(256), 0, st, W, s, R, Ui, Vi, sw, Rh, RhT, out, in);
        else
            hipLaunchKernelGGL(k_dc_residual<false>, tiles, dim3(256), 0, st, W, s, R, Ui - size_t(out) * kRank,
                               Vi - size_t(in) * kRank, sw, Rh, RhT, out, in);
        // start: random X (in x kL) -> Y = |R| X -> Q
        hipLaunchKernelGGL(k_dc_random, dim3(unsigned((size_t(in) / 8 * kL + 255) / 256)), dim3(256), 0, st, X, in,
                           0x9e3779b9u * unsigned(i + 1));
        mul(false);
        orth(false);
        // one round = |R| |R|^T applied to Q; only Q is made orthonormal again (the product in
        // between spreads the columns' lengths by sigma_0 / sigma_31 ~ 30, far inside fp32)
        for (int it = 0; it < iters; ++it) {
            mul(true);
            hipLaunchKernelGGL(k_dc_sum, dim3(in / 32), dim3(256), 0, st, P, groups, X, in);
            mul(false);
            orth(it == iters - 1);
        }
        // the Rayleigh-Ritz step sees the fp32 residual
        const int chunks = out / kDcChunk;
        hipLaunchKernelGGL(k_dc_mul, dim3((in + kDcTile - 1) / kDcTile, slices), dim3(256), 0, st, R, Q, P, out, in,
                           (chunks + slices - 1) / slices);
        gram(P, slices, false, Z, in);
        hipLaunchKernelGGL(k_dc_ritz, dim3(1), dim3(kRitzThreads), 0, st, G, gram_parts(in), Tu, Tv, kRank);
        hipLaunchKernelGGL(k_dc_apply, dim3((out + 63) / 64 + (in + 63) / 64), dim3(256), 0, st, Q, Tu, Ui, out, Z, Tv, Vi, in);
    }
    return hipGetLastError();
}

// One block from canonical device arrays (what launch_decompose writes) into its slot of a packed
// image: sign words re-tiled, V into panel order, U copied, and the per-channel maxima of V.
// The same index functions as the host-side packer; the result is byte for byte the same.
__global__ __launch_bounds__(256) void k_pack_signs(const uint32_t* csw, uint32_t* dsw, int out, int in) {
    const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
    const int wpr = in / 32;
    if (i >= size_t(out) * wpr) return;
    const int o = int(i / wpr), w = int(i % wpr);
    dsw[sign_word_index(in, o, w)] = csw[i];
}

__global__ __launch_bounds__(256) void k_pack_factors(const uint16_t* cu, const uint16_t* cv, uint16_t* du, uint16_t* dv,
                                                      uint16_t* vm, int out, int in) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < in) {
        uint16_t m = 0;
#pragma unroll
        for (int r = 0; r < kRank; ++r) {
            const uint16_t h = cv[size_t(i) * kRank + r];
            dv[v_index(i, r)] = h;
            uint16_t a = h & 0x7FFFu;
            if (a > 0x7C00u) a = 0x7C00u;   // NaN payloads: treat as infinity
            if (a > m) m = a;
        }
        vm[panel_index(i)] = m;
    }
    if (i < out) {
        const uint4* src = reinterpret_cast<const uint4*>(cu + size_t(i) * kRank);
        uint4* dst = reinterpret_cast<uint4*>(du + size_t(i) * kRank);
        dst[0] = src[0];
        dst[1] = src[1];
    }
}

hipError_t launch_pack_block_device(const Geometry& g, unsigned char* image, int slot, const uint32_t* csw,
                                    const uint16_t* cu, const uint16_t* cv, hipStream_t st) {
    unsigned char* blk = image + g.off_blocks + size_t(slot) * g.block_stride;
    uint16_t* vm = reinterpret_cast<uint16_t*>(image + g.off_vmax) + size_t(slot) * g.in;
    const size_t words = size_t(g.out) * (g.in / 32);
    hipLaunchKernelGGL(k_pack_signs, dim3(unsigned((words + 255) / 256)), dim3(256), 0, st, csw,
                       reinterpret_cast<uint32_t*>(blk), g.out, g.in);
    const int mx = g.out > g.in ? g.out : g.in;
    hipLaunchKernelGGL(k_pack_factors, dim3((mx + 255) / 256), dim3(256), 0, st, cu, cv,
                       reinterpret_cast<uint16_t*>(blk + g.off_u), reinterpret_cast<uint16_t*>(blk + g.off_v), vm, g.out,
                       g.in);
    return hipGetLastError();
}

}  // namespace bitstack
