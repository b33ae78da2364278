// The materialising path (the appendix on inference throughput, "level 2"): the weight of the
// loaded prefix is restored once per call to a dense fp16 matrix
//
//     Wd[o][j] = ( sum_i S_i[o][j] * (U_i V_i^T)[o][j] ) / s[j]        (Eq. 8, Eq. 4 folded into the columns)
//
// in caller-owned memory (restore.hip), and the batch then meets it in one dense
// product Y = X Wd^T on the matrix cores (k_gemm below).  Restoring costs the same per weight
// element whatever the batch, so for prefill-sized batches this beats rebuilding weight tiles per
// token tile; the price is out x in x 2 bytes of scratch, shared by all stacks of a model.
//
// k_gemm: one workgroup (8 wavefronts, two per SIMD) owns 256 output rows x 256 tokens and walks
// the input columns in chunks of 64.  Both operand chunks (256 x 64 each, rows of the dense weight
// and rows of x as they lie in memory) go through LDS, double buffered; every thread requests its
// eight 16-byte pieces of a chunk two chunks before they are written to LDS, so all global loads
// of a wavefront have the same, long time to arrive (loads return in order: one late load would
// hold up every younger one).  A wavefront owns 128 rows x 64 tokens: per step of 16 columns it
// reads four weight and two activation fragments from LDS (rows padded by 16 bytes, conflict-free
// 128-bit reads) and issues eight v_mfma_f32_32x32x16_f16; the other wavefront of the SIMD covers
// the read latency.  One LDS-only barrier per chunk.  The fp16 output tile is turned in LDS and
// leaves in 16-byte pieces.  Workgroup ids map to tiles so that all token tiles of a row tile run
// on one XCD (one L2 pulls that part of the weight).  Two more instantiations, with tiles of 128
// rows x 256 tokens and of 128 x 128, fill the chip for shapes with few tiles (row slabs, small
// batches; chosen per launch on the host); k_gemm_split takes the 128 x 128 tiles of long rows, k_gemm_64 (64 x 64) the products that
// larger tiles leave most of the chip idle on.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "kparams.h"
#include "layout.h"
#include "rebuild.h"

namespace bitstack {

constexpr int kGemmRows = 256;              // output rows per workgroup (128 in the narrow variant)
constexpr int kGemmTokens = 256;            // tokens per workgroup
constexpr int kGemmKc = 64;                 // input columns per chunk
constexpr int kGemmLd = kGemmKc + 8;        // fp16 per LDS row (+8: bank spread for 128-bit reads)
constexpr int kGemmTile = 256 * kGemmLd;    // fp16 per operand tile
constexpr int kGemmLds = 2 * 2 * kGemmTile * 2;   // bytes: two buffers x {weight tile, activation tile}
constexpr int kGemmYLd = 256 + 8;           // fp16 per LDS row of the output tile
static_assert(256 * kGemmYLd * 2 <= kGemmLds, "the output tile reuses the operand buffers");
constexpr int kGemmLdsSmall = kGemmLds / 2;       // the 128 x 128 variant: half-height tiles
static_assert(128 * kGemmYLd * 2 <= kGemmLdsSmall && 4 * 64 * 64 * 4 <= kGemmLdsSmall,
              "its output tile and the exchange of the column halves reuse the operand buffers");

__global__ __launch_bounds__(256) void k_dense_zero(uint4* w, size_t n16) {
    const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < n16) w[i] = make_uint4(0, 0, 0, 0);
}

// RJ: 32-row fragments per wavefront.  4: the 256-row tile described above.  2: a 128-row tile
// (wavefront tile 64 rows x 64 tokens, four matrix instructions per step), for shapes whose
// 256-row tiles would leave half of the compute units without a workgroup.
// KSPLIT (with RJ = 2): a tile of 128 rows x 128 tokens for products too small to fill the chip
// with the wider tiles (a slab of 2048 rows x 2048 tokens is 256 of these).  The wavefront tile
// stays 64 x 64 (one LDS fragment per matrix instruction, as in the 128-row variant): wavefronts
// 0-3 take the first 32 columns of every chunk, wavefronts 4-7 the other 32, and the two halves
// are added through LDS after the loop.
template <int RJ, bool KSPLIT>
__global__ __launch_bounds__(512, KSPLIT ? 4 : 1) void k_gemm(KParams p) {
    static_assert(!KSPLIT || RJ == 2, "the 128 x 128 tile is built from 64 x 64 wavefront tiles");
    constexpr int ROWS = KSPLIT ? 128 : 64 * RJ;
    constexpr int TOKS = KSPLIT ? 128 : kGemmTokens;
    constexpr int STEPS = KSPLIT ? 2 : 4;   // 16-column steps of a chunk per wavefront
    // fp16 per operand tile in LDS: 128 rows in the 128 x 128 variant, so that two of its workgroups
    // (74 KB each, at most 128 registers per lane) fit a compute unit
    constexpr int TILE = (KSPLIT ? 128 : 256) * kGemmLd;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    _Float16* const wl = reinterpret_cast<_Float16*>(smem);   // [buffer][256 rows][kGemmLd]
    _Float16* const xl = wl + 2 * TILE;                        // [buffer][256 tokens][kGemmLd]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hl = lane >> 5, ln = lane & 31;
    // my 64 tokens and 32 RJ rows inside the workgroup's tile (and, KSPLIT, my half of every chunk)
    const int tg = KSPLIT ? (wave & 1) : (wave & 3), rg = KSPLIT ? ((wave >> 1) & 1) : (wave >> 2);
    const int kh = KSPLIT ? (wave >> 2) : 0;

    // Workgroup ids are dealt round-robin to the 8 XCDs: all token tiles of a row tile go to one
    // XCD, so that a weight tile is pulled into one L2 only.
    const int ntt = (p.batch + TOKS - 1) / TOKS, nrt = (p.out + ROWS - 1) / ROWS;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int rt = xcd + 8 * (slot / ntt), tt = slot % ntt;
    if (rt >= nrt) return;
    const int row0 = rt * ROWS, tok0 = tt * TOKS;
    const int nkc = p.in / kGemmKc;   // a multiple of 4

    // both tiles of a chunk: thread (row tid/8 + 64 i, 16-byte piece tid%8), i = 0..3 (weight
    // rows: i < RJ; tokens: i < 2 in the 128-token tile); rows and tokens past the end repeat the
    // last one (computed, never stored)
    const unsigned char* const wbase = reinterpret_cast<const unsigned char*>(p.wdense);
    const unsigned char* const xbase = reinterpret_cast<const unsigned char*>(p.x);
    // (scalar variables and macros on purpose: arrays or structs of 128 bytes of load results
    // are left in scratch memory by the compiler here)
    auto off_of = [&](int first, int i, int limit) -> unsigned {
        return unsigned((size_t(min(first + (tid >> 3) + 64 * i, limit - 1)) * p.in + (tid & 7) * 8) * 2);
    };
    const unsigned wo0 = off_of(row0, 0, p.out), wo1 = off_of(row0, 1, p.out), wo2 = off_of(row0, 2, p.out),
                   wo3 = off_of(row0, 3, p.out);
    const unsigned xo0 = off_of(tok0, 0, p.batch), xo1 = off_of(tok0, 1, p.batch), xo2 = off_of(tok0, 2, p.batch),
                   xo3 = off_of(tok0, 3, p.batch);
    const int dst = (tid >> 3) * kGemmLd + (tid & 7) * 8;
    auto ld16 = [&](const unsigned char* base, unsigned off) -> uint4 {
        return *reinterpret_cast<const uint4*>(base + off);
    };
    auto st16 = [&](_Float16* tile, int buf, int i, uint4 v) {
        *reinterpret_cast<uint4*>(tile + buf * TILE + dst + 64 * i * kGemmLd) = v;
    };
#define BS_GEMM_LOAD(S, KC)                                                                \
    {                                                                                      \
        const unsigned c = unsigned(min((KC), nkc - 1)) * (kGemmKc * 2);                   \
        w##S##0 = ld16(wbase, wo0 + c);                                                    \
        w##S##1 = ld16(wbase, wo1 + c);                                                    \
        if constexpr (RJ == 4) {                                                           \
            w##S##2 = ld16(wbase, wo2 + c);                                                \
            w##S##3 = ld16(wbase, wo3 + c);                                                \
        }                                                                                  \
        x##S##0 = ld16(xbase, xo0 + c);                                                    \
        x##S##1 = ld16(xbase, xo1 + c);                                                    \
        if constexpr (!KSPLIT) {                                                           \
            x##S##2 = ld16(xbase, xo2 + c);                                                \
            x##S##3 = ld16(xbase, xo3 + c);                                                \
        }                                                                                  \
    }
#define BS_GEMM_WRITE(S, BUF)                                                              \
    {                                                                                      \
        st16(wl, BUF, 0, w##S##0);                                                         \
        st16(wl, BUF, 1, w##S##1);                                                         \
        if constexpr (RJ == 4) {                                                           \
            st16(wl, BUF, 2, w##S##2);                                                     \
            st16(wl, BUF, 3, w##S##3);                                                     \
        }                                                                                  \
        st16(xl, BUF, 0, x##S##0);                                                         \
        st16(xl, BUF, 1, x##S##1);                                                         \
        if constexpr (!KSPLIT) {                                                           \
            st16(xl, BUF, 2, x##S##2);                                                     \
            st16(xl, BUF, 3, x##S##3);                                                     \
        }                                                                                  \
    }
    // fragments of step s (16 columns) of the chunk in buffer buf: weight rows j*32.., tokens t*32..
    const _Float16* const wfr = wl + (rg * (32 * RJ) + ln) * kGemmLd + 8 * hl + kh * 32;
    const _Float16* const xfr = xl + (tg * 64 + ln) * kGemmLd + 8 * hl + kh * 32;
    auto wfrag = [&](int buf, int s, int j) -> v8h {
        return *reinterpret_cast<const v8h*>(wfr + buf * TILE + j * 32 * kGemmLd + s * 16);
    };
    auto xfrag = [&](int buf, int s, int t) -> v8h {
        return *reinterpret_cast<const v8h*>(xfr + buf * TILE + t * 32 * kGemmLd + s * 16);
    };

    v16f acc[RJ][2];   // [row fragment][token group]
#pragma unroll
    for (int j = 0; j < RJ; ++j)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][t][v] = 0.0f;

    uint4 wA0, wA1, wA2 = {}, wA3 = {}, xA0, xA1, xA2 = {}, xA3 = {}, wB0, wB1, wB2 = {}, wB3 = {}, xB0, xB1, xB2 = {}, xB3 = {};
    BS_GEMM_LOAD(A, 0)
    BS_GEMM_LOAD(B, 1)
    BS_GEMM_WRITE(A, 0)
    BS_GEMM_LOAD(A, 2)
    lds_barrier();

    // The 128 x 256 tile has registers to spare (165 of 256): its fragments are read one step ahead of
    // their use.  The other two tiles would spill with that (256 / 128 registers, 56 / 76 bytes of
    // scratch: 8 % and 2x slower), so they read a step's fragments at its start.
    constexpr bool kAhead = RJ == 2 && !KSPLIT;
    // One chunk from buffer BUF: at step 1 the chunk after it (already in registers T) goes to the
    // other buffer and the chunk two further on is requested, so every global load has two chunks
    // to arrive.  The barrier at the end makes the other buffer readable and protects this one
    // from the writes of the chunk after next.  Fragments are read at the start of their step;
    // the second wavefront of the SIMD covers that latency.
#define BS_GEMM_CHUNK(KC, BUF, S)                                                          \
    {                                                                                      \
        v8h bn[RJ], an[2];                                                                 \
        if constexpr (kAhead) {                                                            \
            _Pragma("unroll") for (int j = 0; j < RJ; ++j) bn[j] = wfrag(BUF, 0, j);       \
            _Pragma("unroll") for (int t = 0; t < 2; ++t) an[t] = xfrag(BUF, 0, t);        \
        }                                                                                  \
        _Pragma("unroll") for (int s = 0; s < STEPS; ++s) {                                \
            if (s == 1) {                                                                  \
                BS_GEMM_WRITE(S, (BUF) ^ 1)                                                \
                BS_GEMM_LOAD(S, (KC) + 3)                                                  \
            }                                                                              \
            v8h b[RJ], a[2];                                                               \
            if constexpr (kAhead) {                                                        \
                _Pragma("unroll") for (int j = 0; j < RJ; ++j) b[j] = bn[j];               \
                _Pragma("unroll") for (int t = 0; t < 2; ++t) a[t] = an[t];                \
                if (s + 1 < STEPS) {                                                       \
                    _Pragma("unroll") for (int j = 0; j < RJ; ++j) bn[j] = wfrag(BUF, s + 1, j); \
                    _Pragma("unroll") for (int t = 0; t < 2; ++t) an[t] = xfrag(BUF, s + 1, t);  \
                }                                                                          \
            } else {                                                                       \
                _Pragma("unroll") for (int j = 0; j < RJ; ++j) b[j] = wfrag(BUF, s, j);    \
                _Pragma("unroll") for (int t = 0; t < 2; ++t) a[t] = xfrag(BUF, s, t);     \
            }                                                                              \
            __builtin_amdgcn_sched_barrier(0); /* requests before the step's arithmetic */ \
            _Pragma("unroll") for (int j = 0; j < RJ; ++j) {                               \
                acc[j][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[j], acc[j][0], 0, 0, 0); \
                acc[j][1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], b[j], acc[j][1], 0, 0, 0); \
            }                                                                              \
            __builtin_amdgcn_sched_barrier(0);                                             \
        }                                                                                  \
        lds_barrier();                                                                     \
    }
    for (int kc = 0; kc < nkc; kc += 2) {
        BS_GEMM_CHUNK(kc, 0, B)
        BS_GEMM_CHUNK(kc + 1, 1, A)
    }
#undef BS_GEMM_CHUNK
#undef BS_GEMM_LOAD
#undef BS_GEMM_WRITE

    if constexpr (KSPLIT) {
        // the two column halves meet: wavefronts 4-7 park their tiles in LDS (the operand buffers are
        // free: the loop's last barrier has passed), wavefronts 0-3 add them to theirs
        float* const red = reinterpret_cast<float*>(smem) + (wave & 3) * (64 * 64) + lane;   // [4][64 registers][64 lanes]
        if (kh == 1) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) red[((j * 2 + t) * 16 + v) * 64] = acc[j][t][v];
        }
        lds_barrier();
        if (kh == 0) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[j][t][v] += red[((j * 2 + t) * 16 + v) * 64];
        }
        lds_barrier();   // read before the output tile below overwrites it
    }
    const bool owner = kh == 0;   // wavefronts that hold finished sums
    // C[i = token][n = row]: lane (row ln), register v holds token 8*(v/4) + 4*hl + v%4 of the group
    if (p.y_f32) {
        if (!owner) return;
#pragma unroll
        for (int j = 0; j < RJ; ++j)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int tok = tok0 + tg * 64 + t * 32 + 8 * (v >> 2) + 4 * hl + (v & 3);
                    const int row = row0 + rg * (32 * RJ) + j * 32 + ln;
                    if (tok < p.batch && row < p.out) static_cast<float*>(p.y)[size_t(tok) * p.y_ld + row] = acc[j][t][v];
                }
        return;
    }
    // fp16 output: the tile is turned in LDS (the operand buffers are free now; the loop's last
    // barrier has passed) so that it leaves in 16-byte pieces, 2 ROWS contiguous bytes per token,
    // instead of 2-byte pieces
    _Float16* const yl = reinterpret_cast<_Float16*>(smem);   // [TOKS tokens][kGemmYLd]
    if (owner) {
#pragma unroll
        for (int j = 0; j < RJ; ++j)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    yl[(tg * 64 + t * 32 + 8 * (v >> 2) + 4 * hl + (v & 3)) * kGemmYLd + rg * (32 * RJ) + j * 32 + ln] =
                        _Float16(acc[j][t][v]);
    }
    lds_barrier();
    __half* const y = static_cast<__half*>(p.y);
    constexpr int PIECES = ROWS / 8;   // 16-byte pieces per token
#pragma unroll 4
    for (int k = 0; k < TOKS * PIECES / 512; ++k) {
        const int idx = tid + 512 * k, tok = idx / PIECES, piece = idx % PIECES;
        const uint4 v = *reinterpret_cast<const uint4*>(yl + tok * kGemmYLd + piece * 8);
        if (tok0 + tok < p.batch && row0 + piece * 8 < p.out)
            *reinterpret_cast<uint4*>(y + size_t(tok0 + tok) * p.y_ld + row0 + piece * 8) = v;
    }
}

// The 128 x 128 tile where k_gemm's is bound by the arrival of its operands: long rows, and no more tiles for an XCD than it has compute
// units (a slab of 2048 rows x 2048 tokens is 256 of them).  2048 x 8192, 2048 tokens: 82 -> 71 us; 4096 x 14336, 1024 tokens: 134 -> 114.
// Without its loads it takes 52 us there, without its products 49: streams and products overlap in part.
// k_gemm<2, true> stays for short rows, where the exchange of four column quarters costs more than is gained (1024 x 1024, 1024 tokens:
// 11.5 us, this kernel 13.5), and for more tiles than compute units, where two of its workgroups share one (6144 x 2048, 1500
// tokens: 53 and 63).
// Eight wavefronts = two token halves x four column quarters: a wavefront multiplies 128 rows x 64 tokens over 32 columns at a time,
// so that twelve fragments read from LDS feed 32 products (64 x 64 tiles over two column halves: eight feed 16, and the
// LDS, whose reads and writes both count, would be the bound by half as much again).
//   Steps of 64 columns (32 KiB of both operands) through a ring of five in LDS, loaded there directly.  Wavefronts 0-3 take the even
//   steps, 4-7 (the other ones of each SIMD) the odd ones, one half of the columns each; a step's products last two steps.  Its
//   fragments are read two steps ahead, into a second set of registers, which frees its buffer: a step is requested five steps ahead
//   and has three to arrive, 96-128 KiB in flight per compute unit.  One barrier per step.
//   LDS: row r of a step in 128 bytes, its 16-byte piece q at position q ^ (r / 2 % 8): a fragment read of sixteen rows touches every
//   bank once, and a load's 1 KiB are eight rows.
// 16x16x32 products: with random operands the chip holds 1.96 PFLOP/s of them and 1.69 of 32x32x16 ones (registers only).
constexpr unsigned kSplitTile = 128 * 128, kSplitStep = 2 * kSplitTile;   // bytes of an operand's step, of both
constexpr int kSplitRing = 5, kSplitLds = kSplitRing * kSplitStep;
constexpr int kSplitYLd = 128 + 8;
static_assert(4 * 128 * 64 * 4 <= kSplitLds && 128 * kSplitYLd * 2 <= kSplitLds, "the exchange and the output tile reuse the ring");
__global__ __launch_bounds__(512, 2) void k_gemm_split(KParams p) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int th = wave & 1, cq = wave >> 1;   // token half, column quarter
    const int ln = lane & 15, kg = lane >> 4;
    // ids are dealt round-robin to the 8 XCDs, whose L2s each fetch what their tiles read: every fourth row tile x every second token tile
    // to one of them
    const int ntt = (p.batch + 127) / 128, nrt = (p.out + 127) / 128, per_row = (ntt + 1) / 2;
    const int xcd = blockIdx.x & 7, place = blockIdx.x >> 3;
    const int rt = (xcd >> 1) + 4 * (place / per_row), tt = (xcd & 1) + 2 * (place % per_row);
    if (rt >= nrt || tt >= ntt) return;
    const int row0 = rt * 128, tok0 = tt * 128;
    const int steps = p.in / 64;   // a multiple of 4
    const v4i w_rsrc = buffer_over(p.wdense, unsigned(size_t(p.out) * p.in * 2));
    const v4i x_rsrc = buffer_over(p.x, unsigned(size_t(p.batch) * p.in * 2));
    const unsigned lds0 = lds_address(smem);
    // this wavefront brings rows / tokens 16 wave .. + 15 of a step, eight per load; past the end the last one is repeated (computed,
    // never stored)
    unsigned w_off[2], x_off[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = 8 * i + (lane >> 3), piece = (lane & 7) ^ (r >> 1);
        w_off[i] = unsigned(size_t(min(row0 + 16 * wave + r, p.out - 1)) * p.in * 2) + unsigned(piece) * 16u;
        x_off[i] = unsigned(size_t(min(tok0 + 16 * wave + r, p.batch - 1)) * p.in * 2) + unsigned(piece) * 16u;
    }
    int q = 0;                                   // next step to request; past the last one the last one again, harmlessly
    unsigned q_dst = lds0 + unsigned(wave) * 2048u;
    auto after = [&](unsigned at, unsigned base) { return at == base + (kSplitRing - 1) * kSplitStep ? base : at + kSplitStep; };
    auto request = [&]() __attribute__((always_inline)) {
        const unsigned col = unsigned(min(q, steps - 1)) * 128u;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            load_to_lds(w_rsrc, q_dst + unsigned(i) * 1024u, w_off[i], col);
            load_to_lds(x_rsrc, q_dst + kSplitTile + unsigned(i) * 1024u, x_off[i], col);
        }
        ++q;
        q_dst = after(q_dst, lds0 + unsigned(wave) * 2048u);
    };
    const unsigned frag = lds0 + unsigned(ln) * 128u + (unsigned(4 * (cq & 1) + kg) ^ unsigned(ln >> 1)) * 16u;
    unsigned r_src = frag;                       // fragments of the step to be read next
    struct Frags {
        v8h w[8], x[4];
    };
    auto read = [&](Frags& f) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t) f.x[t] = __builtin_bit_cast(v8h, read_lds<v4i>(r_src + kSplitTile + unsigned(th * 4 + t) * 2048u));
#pragma unroll
        for (int j = 0; j < 8; ++j) f.w[j] = __builtin_bit_cast(v8h, read_lds<v4i>(r_src + unsigned(j) * 2048u));
    };
    v4f acc[8][4];   // [16 rows][16 tokens]
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[j][t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    auto products = [&](const Frags& f, int j0) __attribute__((always_inline)) {
#pragma unroll
        for (int j = j0; j < j0 + 4; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[j][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(f.x[t], f.w[j], acc[j][t], 0, 0, 0);
    };
    // the first half of a step's products, its successor's fragments read meanwhile (at step h: of step h + 2)
    auto first = [&](const Frags& now, Frags& next) __attribute__((always_inline)) {
        loads_barrier<8>();   // step h + 2 has arrived; step h is in its wavefronts' registers
        request();            // step h + 5, into step h's place
        r_src = after(after(r_src, frag), frag);
        read(next);
        products(now, 0);
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one matrix-core instruction
        }
    };
    auto second = [&](const Frags& now) __attribute__((always_inline)) {
        loads_barrier<8>();
        request();
        products(now, 4);
        __builtin_amdgcn_sched_barrier(0);
    };
    Frags fa, fb;
#pragma unroll
    for (int i = 0; i < kSplitRing; ++i) request();
    loads_barrier<12>();   // steps 0 and 1
    // (both sides meet the same barriers)
    if (cq < 2) {
        read(fa);
        for (int h = 0; h < steps; h += 4) {
            first(fa, fb);
            second(fa);
            first(fb, fa);
            second(fb);
        }
    } else {
        r_src += kSplitStep;
        read(fa);
#pragma unroll
        for (int t = 0; t < 4; ++t) fb.x[t] = v8h{};   // no step before the first
#pragma unroll
        for (int j = 0; j < 8; ++j) fb.w[j] = v8h{};
        for (int h = 0; h < steps; h += 4) {
            second(fb);
            first(fa, fb);
            second(fa);
            first(fb, fa);
        }
        products(fb, 4);
    }
    loads_barrier<0>();   // nothing may land in LDS any more

    // the column quarters meet: 2 and 3 park their sums, 0 and 1 add them, then 1 parks and 0 adds
    float* const red = reinterpret_cast<float*>(smem) + (wave & 3) * (128 * 64) + lane;   // [4][128 registers][64 lanes]
    auto park = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[((j * 4 + t) * 4 + v) * 64] = acc[j][t][v];
    };
    auto add = [&](const float* from) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[j][t][v] += from[((j * 4 + t) * 4 + v) * 64];
    };
    if (cq >= 2) park();
    lds_barrier();
    if (cq < 2) add(red);
    lds_barrier();
    if (cq == 1) park();
    lds_barrier();
    if (cq == 0) add(red + 2 * (128 * 64));
    lds_barrier();
    // D[i = token][n = row]: lane (row ln), register v holds token 4 kg + v of the group
    if (p.y_f32) {
        if (cq != 0) return;
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int tok = tok0 + th * 64 + t * 16 + 4 * kg + v, row = row0 + j * 16 + ln;
                    if (tok < p.batch && row < p.out) static_cast<float*>(p.y)[size_t(tok) * p.y_ld + row] = acc[j][t][v];
                }
        return;
    }
    _Float16* const yl = reinterpret_cast<_Float16*>(smem);   // [128 tokens][kSplitYLd]: leaves in 16-byte pieces
    if (cq == 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) yl[(th * 64 + t * 16 + 4 * kg + v) * kSplitYLd + j * 16 + ln] = _Float16(acc[j][t][v]);
    }
    lds_barrier();
    __half* const y = static_cast<__half*>(p.y);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int idx = tid + 512 * k, tok = idx / 16, piece = idx % 16;
        const uint4 v = *reinterpret_cast<const uint4*>(yl + tok * kSplitYLd + piece * 8);
        if (tok0 + tok < p.batch && row0 + piece * 8 < p.out)
            *reinterpret_cast<uint4*>(y + size_t(tok0 + tok) * p.y_ld + row0 + piece * 8) = v;
    }
}

// The 64 x 64 tile, wherever these leave no XCD with more tiles than it has compute units: a product that small is bound by the arrival of a
// tile's operands, which are half as many as a 128 x 128 tile's, and takes 0.43 (long rows, few tiles) to 0.64 (rows of 512-1024 columns,
// 32 tiles per XCD) of the time of the larger tiles (4143 products of 512 x 512 to 28672 x 14336, 20 to 2048 tokens; 0.82 at most, one
// of 1.09 apart; 512 x 4096, 256 tokens: 28 us, 12 now).  Beyond 32 tiles per XCD it is 0.91 to 1.04 in the mean and up to 1.4.
// A step is 128 columns (32 KiB of both operands) in a ring of five in LDS, loaded there directly; its fragments are read one step ahead
// into a second set of registers, which frees its buffer: a step is requested five steps ahead and has four to arrive.  One barrier per step.
// Eight wavefronts, and the order of the sums of the larger tile that would be taken instead (the same bits):
//   QUARTERS: two token halves x four column quarters with 16x16x32 products, as k_gemm_split; a wavefront multiplies 64 rows x 32 tokens
//     over its quarter of every step, six fragments feeding 8 products;
//   else: two row halves x two token halves x the two halves of every 64 columns with 32x32x16 products, as k_gemm<2, true>; 32 rows x 32
//     tokens, eight fragments feeding 4 products.
// LDS: row r of a step in 256 bytes, its 16-byte piece q at position q ^ (r % 16); a load's 1 KiB are four rows.
constexpr unsigned k64Tile = 64 * 256, k64Step = 2 * k64Tile;
constexpr int k64Ld = 64 + 4;
static_assert(kSplitRing * k64Step == kSplitLds && 4 * 64 * k64Ld * 4 <= kSplitLds, "the partial tiles reuse the ring");
template <bool QUARTERS>
__global__ __launch_bounds__(512, 2) void k_gemm_64(KParams p) {
    constexpr int kSlices = QUARTERS ? 4 : 2;   // of the columns
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int th = wave & 1, rh = QUARTERS ? 0 : (wave >> 1) & 1, slice = QUARTERS ? wave >> 1 : wave >> 2;   // token half, row half, columns
    constexpr int kSide = QUARTERS ? 16 : 32;   // rows and tokens of a fragment
    const int ln = lane & (kSide - 1), kg = lane / kSide;
    // the 8 XCDs, to which ids are dealt round-robin, share the tiles as (8 / n_ks) x n_ks: every (8 / n_ks)-th row tile x every n_ks-th token
    // tile to one of them
    const int ntt = (p.batch + 63) / 64, nrt = (p.out + 63) / 64, per_row = (ntt + p.n_ks - 1) / p.n_ks;
    const int xcd = blockIdx.x & 7, place = blockIdx.x >> 3;
    const int rt = xcd / p.n_ks + 8 / p.n_ks * (place / per_row), tt = xcd % p.n_ks + p.n_ks * (place % per_row);
    if (rt >= nrt || tt >= ntt) return;
    const int row0 = rt * 64, tok0 = tt * 64;
    const int steps = p.in / 128;   // even
    const v4i w_rsrc = buffer_over(p.wdense, unsigned(size_t(p.out) * p.in * 2));
    const v4i x_rsrc = buffer_over(p.x, unsigned(size_t(p.batch) * p.in * 2));
    const unsigned lds0 = lds_address(smem);
    // this wavefront brings rows / tokens 8 wave .. + 7 of a step, four per load; past the end the last one is repeated (computed, never
    // stored)
    unsigned w_off[2], x_off[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = 8 * wave + 4 * i + (lane >> 4), piece = (lane & 15) ^ (r & 15);
        w_off[i] = unsigned(size_t(min(row0 + r, p.out - 1)) * p.in * 2) + unsigned(piece) * 16u;
        x_off[i] = unsigned(size_t(min(tok0 + r, p.batch - 1)) * p.in * 2) + unsigned(piece) * 16u;
    }
    int q = 0;                                   // next step to request; past the last one the last one again, harmlessly
    unsigned q_dst = lds0 + unsigned(wave) * 2048u;
    auto after = [&](unsigned at, unsigned base) { return at == base + (kSplitRing - 1) * k64Step ? base : at + k64Step; };
    auto request = [&]() __attribute__((always_inline)) {
        const unsigned col = unsigned(min(q, steps - 1)) * 256u;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            load_to_lds(w_rsrc, q_dst + unsigned(i) * 1024u, w_off[i], col);
            load_to_lds(x_rsrc, q_dst + k64Tile + unsigned(i) * 1024u, x_off[i], col);
        }
        ++q;
        q_dst = after(q_dst, lds0 + unsigned(wave) * 2048u);
    };
    // fragment f of a step: pieces kg on of 32 columns (quarters) or 16 columns (halves: two of each 64)
    constexpr int kCols = QUARTERS ? 1 : 4, kRowFrags = QUARTERS ? 4 : 1, kTokFrags = QUARTERS ? 2 : 1;
    unsigned from[kCols];
#pragma unroll
    for (int c = 0; c < kCols; ++c) {
        const int piece = QUARTERS ? 4 * slice + kg : 8 * (c >> 1) + 4 * slice + 2 * (c & 1) + kg;
        from[c] = unsigned(ln) * 256u + unsigned(piece ^ (ln & 15)) * 16u;
    }
    unsigned r_src = lds0;                       // the step to be read next
    struct Frags {
        v8h w[kCols][kRowFrags], x[kCols][kTokFrags];
    };
    auto read = [&](Frags& f) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < kCols; ++c) {
#pragma unroll
            for (int t = 0; t < kTokFrags; ++t)
                f.x[c][t] = __builtin_bit_cast(v8h, read_lds<v4i>(r_src + from[c] + k64Tile + unsigned(th * 32 + t * kSide) * 256u));
#pragma unroll
            for (int j = 0; j < kRowFrags; ++j)
                f.w[c][j] = __builtin_bit_cast(v8h, read_lds<v4i>(r_src + from[c] + unsigned(rh * 32 + j * kSide) * 256u));
        }
        r_src = after(r_src, lds0);
    };
    v4f acc[QUARTERS ? 4 : 1][2];   // [16 rows][16 tokens]
    v16f acc32;                     // 32 x 32
    if constexpr (QUARTERS) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[j][t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    } else {
        acc32 = zero16();
    }
    auto step = [&](const Frags& now, Frags& next) __attribute__((always_inline)) {   // step h
        loads_barrier<12>();   // step h + 1 has arrived; step h is in the wavefronts' registers
        request();             // step h + 5, into step h's place
        read(next);            // past the last step: the last one again, not used
        if constexpr (QUARTERS) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < 2; ++t) acc[j][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(now.x[0][t], now.w[0][j], acc[j][t], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one matrix-core instruction
            }
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) acc32 = __builtin_amdgcn_mfma_f32_32x32x16_f16(now.x[c][0], now.w[c][0], acc32, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    Frags fa, fb;
#pragma unroll
    for (int i = 0; i < kSplitRing; ++i) request();
    loads_barrier<16>();   // step 0
    read(fa);
    for (int h = 0; h < steps; h += 2) {
        step(fa, fb);
        step(fb, fa);
    }
    loads_barrier<0>();   // nothing may land in LDS any more

    // the column slices meet.  D[i = token][n = row]: lane (row ln), register v holds token 4 kg + v of 16, or 8 (v / 4) + 4 kg + v % 4 of 32
    float* const red = reinterpret_cast<float*>(smem) + slice * 64 * k64Ld;   // [kSlices][64 tokens][k64Ld]
    if constexpr (QUARTERS) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[(th * 32 + t * 16 + 4 * kg + v) * k64Ld + j * 16 + ln] = acc[j][t][v];
    } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) red[(th * 32 + 8 * (v >> 2) + 4 * kg + (v & 3)) * k64Ld + rh * 32 + ln] = acc32[v];
    }
    lds_barrier();
    const int tok = tid >> 3, row = 8 * (tid & 7);   // eight rows of a token; out is a multiple of 32
    float sum[8];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        v4f part[kSlices];
#pragma unroll
        for (int c = 0; c < kSlices; ++c) part[c] = *reinterpret_cast<const v4f*>(reinterpret_cast<const float*>(smem) + (c * 64 + tok) * k64Ld + row + 4 * k);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (QUARTERS) sum[4 * k + e] = (part[0][e] + part[2][e]) + (part[1][e] + part[3][e]);
            else sum[4 * k + e] = part[0][e] + part[1][e];
        }
    }
    if (tok0 + tok >= p.batch || row0 + row >= p.out) return;
    const size_t at = size_t(tok0 + tok) * p.y_ld + row0 + row;
    if (p.y_f32) {
        v4f* const y = reinterpret_cast<v4f*>(static_cast<float*>(p.y) + at);
        y[0] = v4f{sum[0], sum[1], sum[2], sum[3]};
        y[1] = v4f{sum[4], sum[5], sum[6], sum[7]};
    } else {
        v8h o;
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] = _Float16(sum[k]);
        *reinterpret_cast<v8h*>(static_cast<__half*>(p.y) + at) = o;
    }
}

hipError_t launch_dense_zero(const LaunchArgs& a, hipStream_t st) {
    const size_t n16 = size_t(a.geo.out) * size_t(a.geo.in) * 2 / 16;
    hipLaunchKernelGGL(k_dense_zero, dim3(unsigned((n16 + 255) / 256)), dim3(256), 0, st,
                       static_cast<uint4*>(a.wdense), n16);
    return hipGetLastError();
}

// Cost model of the product (microseconds, fitted to measurements): a round of workgroups takes
// in x (a + b x the fraction of the 256 compute units that have a workgroup) - a partly filled
// chip runs each tile faster (clock, shared caches) - with (a, b) = (0.0196, 0.0148) for 256-row
// tiles, (0.0111, 0.0089) for 128-row tiles and (0.0068, 0.0032) for 128 x 128 tiles.  The
// launcher takes the cheapest tile (dense_time_us below prices it more closely).
enum GemmTile { kTile256 = 1, kTile128 = 2, kTile128x128 = 3, kTileSplit = 4, kTile64 = 5, kTile64Split = 6 };
static std::atomic<int> g_forced_tile{0};   // measurement hook: 0 = the estimate's choice
void dense_force_tile(int tile) { g_forced_tile = tile; }

static double tile_rounds_time_us(int out, int in, int batch, int tile) {
    if (tile == kTileSplit) tile = kTile128x128;   // what the crossovers between the paths are stated in
    const int rows = tile == kTile256 ? 256 : 128, toks = tile == kTile128x128 ? 128 : kGemmTokens;
    const int tiles = ((out + rows - 1) / rows) * ((batch + toks - 1) / toks);
    const double a = tile == kTile256 ? 0.0196 : tile == kTile128 ? 0.0111 : 0.0068;
    const double b = tile == kTile256 ? 0.0148 : tile == kTile128 ? 0.0089 : 0.0032;
    const int full = tiles / 256, rest = tiles % 256;
    return in * (full * (a + b) + (rest ? a + b * rest / 256.0 : 0.0));
}
// The most 64 x 64 tiles that an XCD gets, and how many ways the token tiles are shared among the XCDs for that (2: what an L2 fetches is
// least; 1 and 4 where 2 would leave XCDs with fewer tiles than others)
static int tiles64_of_xcd(int out, int batch, int* ways) {
    const int nrt = (out + 63) / 64, ntt = (batch + 63) / 64;
    int best = 0;
    for (int w : {2, 1, 4}) {
        const int n = (nrt + 8 / w - 1) / (8 / w) * ((ntt + w - 1) / w);
        if (best == 0 || n < best) {
            best = n;
            *ways = w;
        }
    }
    return best;
}
static int dense_tile(int out, int in, int batch) {
    const int forced = g_forced_tile.load();
    if (forced >= kTile256 && forced <= kTile64Split) return forced;
    int ways;
    if (tiles64_of_xcd(out, batch, &ways) <= 32) return in >= 4096 ? kTile64Split : kTile64;
    int best = kTile256;
    for (int t = kTile128; t <= kTile128x128; ++t)
        if (tile_rounds_time_us(out, in, batch, t) < tile_rounds_time_us(out, in, batch, best)) best = t;
    // 333 random shapes with rows of 4096 columns and more: 0.90 of k_gemm<2, true>'s time in the mean, none above 1.013 of it.  An XCD
    // has 32 compute units and takes every fourth row tile x every second token tile: where that is more than 32 tiles (odd numbers of
    // token tiles) it takes two rounds, 5376 x 5888, 580 tokens: 82 us against 52.
    const int per_xcd = ((out + 127) / 128 + 3) / 4 * (((batch + 127) / 128 + 1) / 2);
    if (best == kTile128x128 && in >= 4096 && per_xcd <= 32) return kTileSplit;
    return best;
}
// Duration (microseconds) of the tile taken, for the choice between the paths: rounds of 256 workgroups as above, one pass over both
// operands, the outputs.  Fitted to 7053 cases of 65 to 2048 tokens (512 x 512 to 28672 x 8192), 9.1, 7.2, 7.3 and 4.6 % root mean square
// for the first four tiles, the 64 x 64 ones to 4143 of 20 to 2048 tokens, 4.3 and 8.3 %.
double dense_time_us(int out, int in, int batch) {
    const int tile = dense_tile(out, in, batch);
    const int rows = tile == kTile256 ? 256 : tile >= kTile64 ? 64 : 128, toks = tile <= kTile128 ? kGemmTokens : tile >= kTile64 ? 64 : 128;
    const int tiles = ((out + rows - 1) / rows) * ((batch + toks - 1) / toks), full = tiles / 256, rest = tiles % 256;
    struct Fit {
        double fixed, a, b, operands, outputs;
    };
    static constexpr Fit kFits[] = {{2.14, 0.0011, 0.0304, 0.0097, 0.544},   {3.26, 0.00705, 0.00908, 0.0174, 0.437},
                                    {4.53, 0.00613, 0.00224, 0.0024, 0.356}, {7.74, 0.00522, 0.00112, 0.0386, 0.0437},
                                    {4.02, 0.00203, 0.00118, 0.0109, 0.0},   {3.31, 0.00211, 0.00081, 0.0194, 2.78}};
    const Fit& f = kFits[tile - kTile256];
    return f.fixed + in * (full * (f.a + f.b) + (rest ? f.a + f.b * rest / 256.0 : 0.0)) +
           1e-6 * (f.operands * 2.0 * (double(out) + batch) * in + f.outputs * double(out) * batch);
}

hipError_t launch_dense(const LaunchArgs& a, hipStream_t st) {
    KParams p = make_params(a);
    if (a.batch < 1 || p.wdense == nullptr) return hipErrorInvalidValue;
    if (a.rows) {
        // a slab of rows: the dense matrix holds rows [row_begin, row_begin + rows) of the weight, the
        // outputs go to the same columns of y (whose token rows stay the stack's full width apart)
        if (a.row_begin % 256 || a.row_begin < 0 || a.row_begin >= a.geo.out) return hipErrorInvalidValue;
        p.out = a.rows < a.geo.out - a.row_begin ? a.rows : a.geo.out - a.row_begin;
        p.y = static_cast<unsigned char*>(p.y) + size_t(a.row_begin) * (a.y_f32 ? 4 : 2);
    }
    if (size_t(p.batch) * p.in * 2 > 0xffffffffull || size_t(p.out) * p.in * 2 > 0xffffffffull)
        return hipErrorInvalidValue;   // 32-bit byte offsets into x and the dense weight
    static std::atomic<bool> attr_set{false};   // setting the attribute twice is harmless
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm<4, false>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm<2, false>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm<2, true>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLdsSmall);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_split), hipFuncAttributeMaxDynamicSharedMemorySize, kSplitLds);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_64<false>), hipFuncAttributeMaxDynamicSharedMemorySize, kSplitLds);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_64<true>), hipFuncAttributeMaxDynamicSharedMemorySize, kSplitLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int tile = dense_tile(p.out, p.in, p.batch);
    if (tile == kTile64 || tile == kTile64Split) {
        const unsigned tiles = unsigned(8 * tiles64_of_xcd(p.out, p.batch, &p.n_ks));
        if (tile == kTile64) hipLaunchKernelGGL(k_gemm_64<false>, dim3(tiles), dim3(512), kSplitLds, st, p);
        else hipLaunchKernelGGL(k_gemm_64<true>, dim3(tiles), dim3(512), kSplitLds, st, p);
        return hipGetLastError();
    }
    const int rows = tile == kTile256 ? 256 : 128, toks = tile >= kTile128x128 ? 128 : kGemmTokens;
    const int ntt = (p.batch + toks - 1) / toks, nrt = (p.out + rows - 1) / rows;
    const unsigned wgs = unsigned(8 * ((nrt + 7) / 8) * ntt);
    if (tile == kTileSplit)
        hipLaunchKernelGGL(k_gemm_split, dim3(unsigned(8 * ((nrt + 3) / 4) * ((ntt + 1) / 2))), dim3(512), kSplitLds, st, p);
    else if (tile == kTile128x128)
        hipLaunchKernelGGL((k_gemm<2, true>), dim3(wgs), dim3(512), kGemmLdsSmall, st, p);
    else if (tile == kTile128)
        hipLaunchKernelGGL((k_gemm<2, false>), dim3(wgs), dim3(512), kGemmLds, st, p);
    else
        hipLaunchKernelGGL((k_gemm<4, false>), dim3(wgs), dim3(512), kGemmLds, st, p);
    return hipGetLastError();
}

}  // namespace bitstack
