// Batches through matrices of few rows (up to 256 or 512 workgroups of 32 rows x 64 tokens): k_batch's arithmetic, one row tile per workgroup and the blocks shared out.
//
// k_batch's workgroups are 64 or 128 rows high, and a column split needs partial rows that a small image has no room for: 704 x 1024, 15
// blocks, 32 tokens ran on eleven of 256 compute units, each walking all blocks.  Here a workgroup is 32 rows: eight wavefronts = C column
// chunks x G groups of blocks (C G = 8), each of which rebuilds its chunk's unit (rebuild.h) over every G-th block.  The groups' sums meet
// in LDS in fp32, before the weight is scaled and rounded, so the results differ from k_batch's by the order of fp32 sums only.
//
// Nothing is shared between wavefronts before that: every one has its own two buffers in LDS (V of the chunk, signs, U: 10 KiB a step) and
// the loop has no barrier; a step's inputs are requested when the step before begins.  Bound by the chain of a wavefront's steps.  (Four
// wavefronts with rings of four buffers: a lone wavefront per SIMD takes 1.1 us a step, as long as two.)
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"
#include "kparams.h"
#include "layout.h"
#include "rebuild.h"

namespace bitstack {

namespace {

constexpr int kRowsWaves = 8, kRowsRing = 2;
typedef StepLayout<1> RowsStep;
constexpr unsigned kRowsWaveLds = kRowsRing * RowsStep::kBytes, kRowsLds = kRowsWaves * kRowsWaveLds;
constexpr unsigned kUnitSums = 128 * 64 * 4;   // a unit's fp32 sums
static_assert(kRowsLds <= 160 * 1024 && kRowsWaves / 2 * kUnitSums <= kRowsLds, "half of the wavefronts park their sums in the idle rings");

// GROUPS of 32 tokens to a workgroup; p.n_ks: column chunks at a time (C)
template <int GROUPS>
__global__ __launch_bounds__(kRowsWaves * 64, 2) void k_rows(KParams p) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    constexpr unsigned kFlagLds = kRowsWaves * 4096;   // behind the partial tiles, in the rings when they are idle
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hl = lane >> 5, ln = lane & 31;
    const int nch = p.in / kChunkCols, n = p.n_loaded, rt = blockIdx.x;
    const int tok0 = int(blockIdx.y) * (GROUPS * 32);   // this workgroup's tokens
    const int C = p.n_ks, G = kRowsWaves / C, c = wave % C, g = wave / C;
    const int iters = (nch + C - 1) / C, nb = (n - g + G - 1) / G;   // G <= n

    const unsigned stride = unsigned(p.block_stride);
    const v4i rsrc = buffer_over(p.blocks, unsigned(n) * stride);
    const unsigned s_lane = unsigned(size_t(rt) * nch * kUnitBytes) + unsigned(lane) * 16u;
    const unsigned v_lane = v_lane_offset<1>(unsigned(p.off_v), 0u, unsigned(lane));
    const unsigned u_lane = u_lane_offset<1>(unsigned(p.off_u), unsigned(rt), unsigned(lane));
    const unsigned lds0 = lds_address(smem), ring = lds0 + unsigned(wave) * kRowsWaveLds;
    const unsigned v_rd = ring + v_read_offset(unsigned(lane)), s_rd = ring + unsigned(lane) * 16u;
    constexpr unsigned kRsAt = 16384;   // behind a group's activations
    static_assert(kRsAt + kChunkCols * 4 <= kRowsWaveLds, "");
    const v4i x_rsrc = buffer_over(p.x, unsigned(p.batch) * unsigned(p.in) * 2u);
    const v4i rs_rsrc = buffer_over(p.rs, unsigned(p.in) * 4u);

    v16f yacc[GROUPS];
    auto accumulate = [&](auto on_x) __attribute__((always_inline)) {
        constexpr bool kScaleX = decltype(on_x)::value;
#pragma unroll
        for (int k = 0; k < GROUPS; ++k) yacc[k] = zero16();
        for (int it = 0; it < iters; ++it) {
            const bool valid = it * C + c < nch;   // uniform over the wavefront
            const int ch = min(it * C + c, nch - 1);
            // the wavefront's steps: its blocks of this chunk; past the last one the last one again, harmlessly
            unsigned q_off = unsigned(g) * stride, buf = 0;
            auto request = [&](unsigned to) {
                load_step<1>(rsrc, ring + to, s_lane, v_lane, u_lane, q_off + unsigned(ch) * kUnitBytes, q_off + unsigned(ch) * kVChunkBytes, q_off);
                q_off += unsigned(G) * stride;
            };
            UnitAcc acc;
            StepInputs in;
            request(0);
            loads_wait<0>();
            auto step = [&](int t, auto first) __attribute__((always_inline)) {
                begin_reads<1>(in, v_rd + buf, s_rd + buf);
                if (decltype(first)::value) in.last = in.s;
                const unsigned other = RowsStep::kBytes - buf;
                if (t + 1 < nb) request(other);
                add_block<decltype(first)::value, 1, false>(acc, in, v_rd + buf, 0u, 0u);
                loads_wait<0>();   // the next step has arrived, this one's buffer has been read
                buf = other;
            };
            step(0, std::true_type{});
            for (int t = 1; t < nb; ++t) step(t, std::false_type{});
            const bool owner = g == 0 && valid;
            // what the product takes, to the idle ring: a group's activations, a token's 32 16-byte pieces in a row, piece j of token t at
            // position j ^ (t % 16), and 1/s of the chunk
            auto request_x = [&](int k) {
                int own = lane;   // made anew: sixteen offsets kept from outside the loop would cost it registers it does not have
                asm volatile("" : "+v"(own));
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int t = 2 * i + (own >> 5), piece = (own & 31) ^ (t & 15);
                    load_to_lds(x_rsrc, ring + unsigned(i) * 1024u, unsigned(min(tok0 + k * 32 + t, p.batch - 1)) * unsigned(p.in) * 2u + unsigned(piece) * 16u,
                                unsigned(ch) * (kChunkCols * 2));
                }
            };
            auto request_product = [&]() {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    load4_to_lds(rs_rsrc, ring + kRsAt + unsigned(k) * 256u, unsigned(lane) * 4u, unsigned(ch) * (kChunkCols * 4) + unsigned(k) * 256u);
                request_x(0);
            };
            if (G == 1 && owner) request_product();
            finish_unit(acc, in);
            if (G > 1) {
                // the groups of blocks meet, half of them parking their sums for the other half at a time
                lds_barrier();   // all rings are idle
                for (int half = G / 2; half >= 1; half /= 2) {
                    if (g >= half && g < 2 * half) {
                        const unsigned to = lds0 + unsigned((g - half) * C + c) * kUnitSums + unsigned(lane) * 16u;
#pragma unroll
                        for (int k = 0; k < 32; ++k)
                            write_lds(to + unsigned(k) * 1024u,
                                      v4f{acc[k >> 2][4 * (k & 3)], acc[k >> 2][4 * (k & 3) + 1], acc[k >> 2][4 * (k & 3) + 2], acc[k >> 2][4 * (k & 3) + 3]});
                    }
                    lds_barrier();
                    if (g < half) {
                        const unsigned from = lds0 + unsigned(g * C + c) * kUnitSums + unsigned(lane) * 16u;
#pragma unroll
                        for (int k = 0; k < 32; ++k) {
                            const v4f v = read_lds<v4f>(from + unsigned(k) * 1024u);
#pragma unroll
                            for (int j = 0; j < 4; ++j) acc[k >> 2][4 * (k & 3) + j] += v[j];
                        }
                    }
                    lds_barrier();   // read before anything else lands there
                }
                if (owner) request_product();
            }
            if (owner) {
                loads_wait<0>();
                v4i b[16];   // W' diag(1/s) of the unit as B operands: step e = columns 8 e .. 8 e + 7 of both halves
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    v4f r[2];
                    read_scales(r, ring + kRsAt + unsigned(hl) * 512u, e);
#pragma unroll
                    for (int t = 0; t < 8; t += 2)
                        b[e][t >> 1] = scaled_pair(acc[t][e], acc[t + 1][e], kScaleX ? 1.0f : r[t >> 2][t & 3], kScaleX ? 1.0f : r[t >> 2][(t & 3) + 1]);
                    asm volatile("" : "+v"(b[e]));   // made here, not put off to the products
                }
#pragma unroll
                for (int k = 0; k < GROUPS; ++k) {
                    if (k > 0) loads_wait<0>();
                    v4i a[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        a[e] = read_lds<v4i>(ring + unsigned(ln) * 512u + (unsigned(hl * 16 + e) ^ unsigned(ln & 15)) * 16u);
                        if constexpr (kScaleX) {
                            v4f r[2];
                            read_scales(r, ring + kRsAt + unsigned(hl) * 512u, e);
                            const v8h h = __builtin_bit_cast(v8h, a[e]);
#pragma unroll
                            for (int t = 0; t < 8; t += 2)
                                a[e][t >> 1] = scaled_pair(float(h[t]), float(h[t + 1]), r[t >> 2][t & 3], r[t >> 2][(t & 3) + 1]);
                        }
                    }
                    loads_wait<0>();   // read before the next group, or the next chunk's steps, land there
                    if (k + 1 < GROUPS) request_x(k + 1);
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        yacc[k] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a[e]), __builtin_bit_cast(v8h, b[e]), yacc[k], 0, 0, 0);
                }
            }
        }
    };

    // the wavefronts' partial tiles meet in LDS; D[i = token][n = row]: lane (row ln), register v holds token 8 (v / 4) + 4 hl + v % 4 of 32
    float* const red = reinterpret_cast<float*>(smem);   // [wave][16][64]
    auto store = [&]() __attribute__((always_inline)) {
        float rest = 0.0f;   // 0 * y: NaN for infinities and NaN
#pragma unroll
        for (int k = 0; k < GROUPS; ++k) {
            __syncthreads();
            if (k == 0 && tid == 0) write_lds(lds0 + kFlagLds, 0u);
#pragma unroll
            for (int v = 0; v < 16; ++v) red[(wave * 16 + v) * 64 + lane] = yacc[k][v];
            __syncthreads();
#pragma unroll
            for (int o = tid; o < 32 * 32; o += kRowsWaves * 64) {   // thread = (row, token): consecutive lanes take consecutive rows
                const int row = o & 31, t = o >> 5, v = (t >> 3) * 4 + (t & 3), l = ((t >> 2) & 1) * 32 + row;
                float sum = 0.0f;
#pragma unroll
                for (int w = 0; w < kRowsWaves; ++w) sum += red[(w * 16 + v) * 64 + l];
                const int tok = tok0 + k * 32 + t;
                if (tok < p.batch) {
                    rest = __builtin_fmaf(sum, 0.0f, rest);
                    store_y(p, size_t(tok) * p.out + rt * kTileRows + row, sum);
                }
            }
        }
        if (rest != 0.0f) write_lds(lds0 + kFlagLds, 1u);
        __syncthreads();
    };
    accumulate(std::false_type{});
    store();
    // sums that are not finite: once more with 1/s on the activations, as in k_batch
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(int(read_lds<unsigned>(lds0 + kFlagLds))), 0)) {
        __syncthreads();   // everybody has seen it
        accumulate(std::true_type{});
        store();
    }
}

template <int GROUPS>
hipError_t launch_rows_t(KParams p, int chunks_at_a_time, hipStream_t st) {
    static std::atomic<bool> attr_set{false};   // setting the attribute twice is harmless
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_rows<GROUPS>), hipFuncAttributeMaxDynamicSharedMemorySize, int(kRowsLds));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    p.n_ks = chunks_at_a_time;
    hipLaunchKernelGGL((k_rows<GROUPS>), dim3(p.out / kTileRows, (p.batch + GROUPS * 32 - 1) / (GROUPS * 32)), dim3(kRowsWaves * 64), kRowsLds, st, p);
    return hipGetLastError();
}

}  // namespace

// Column chunks at a time, and the estimated duration (microseconds), fitted to 3727 cases of 2 to 64 tokens (64 x 256 to 16384 x 14336, 1 to
// 24 blocks; each timed with every share; 4.1 % root mean square) and 1377 of 65 to 1024 (4.5 %).  Where the workgroups fit the chip at once, against
// k_batch, k_fused and k_tile, it is the faster one in 57-90 % (up to 64 tokens, worth 13 to 21 % in the mean of all by number of
// workgroups) and 90-100 % (beyond, 34 to 40 %); with a second round of workgroups in 5 and 24 %, worth 1 %.
static double rows_plan(int out, int in, int batch, int n_loaded, int* chunks_at_a_time) {
    const int nch = in / kChunkCols, wgs = out / kTileRows * ((batch + 63) / 64), more = batch > 32 ? 1 : 0, rounds = (wgs + 255) / 256;
    const double fill = wgs < 256 ? wgs / 256.0 : 1.0;
    double best = 0.0;
    for (int c = kRowsWaves; c >= 1; c /= 2) {
        const int g = kRowsWaves / c;
        if (g > n_loaded) break;
        const double us = 1.52 + 0.53 * more + rounds * (1.54 + (nch + c - 1) / c * ((n_loaded + g - 1) / g * (0.957 + 0.137 * fill) + 2.04 + 0.75 * more +
                                                                                  (batch > 64 ? 0.4 : 0.0) + (g > 1 ? 1.0 + 0.34 * g : 0.0)));
        if (best == 0.0 || us < best) {
            best = us;
            *chunks_at_a_time = c;
        }
    }
    return best;
}
// What the launch takes, and what the estimate prices: up to 1024 tokens, one 32-bit buffer descriptor each over the loaded blocks and the
// activations.  (Priced without these conditions, few rows and 1025 to 2048 tokens went to the panel path for k_rows' estimate, where k_tile
// ran: 544 x 14336, 2 blocks, 1800 tokens 245 us, 99 restored; 60 such calls take 0.52 of the time restored, 0.81 at most.)
bool rows_fits(int out, int in, int batch, int n_loaded) {
    return batch <= 1024 && size_t(n_loaded) * make_geometry(out, in, 1, 1).block_stride < (size_t(1) << 32) && size_t(batch) * in * 2 < (size_t(1) << 32);
}
// For comparison with the other kernels' estimates: 4 % on top, so that an error of either leaves the call where it was (without, 40 of 2585
// cases are 3 to 15 % slower than with the others), and 20 % with a second round, where the estimates are worth less (2720 x 5888, 6 blocks, 351
// tokens: 123 us, 69 with k_rows; 7168 x 2048, 5 blocks, 249 tokens: 40, 49)
double rows_time_us(int out, int in, int batch, int n_loaded) {
    if (!rows_fits(out, in, batch, n_loaded)) return 1e30;
    int c;
    const int wgs = out / kTileRows * ((batch + 63) / 64);
    if (wgs > 512) return 1e30;
    return (wgs > 256 ? 1.2 : 1.04) * rows_plan(out, in, batch, n_loaded, &c);
}
static std::atomic<int> g_forced_chunks{0};   // measurement hook: 0 = the estimate's choice, 16 = never
void rows_force_chunks(int chunks) { g_forced_chunks = chunks == 1 || chunks == 2 || chunks == 4 || chunks == 8 || chunks == 16 ? chunks : 0; }
int rows_forced_chunks() { return g_forced_chunks.load(); }
hipError_t launch_rows(const KParams& p, hipStream_t st) {
    int c = kRowsWaves;
    rows_plan(p.out, p.in, p.batch, p.n_loaded, &c);
    const int forced = g_forced_chunks.load();
    if (forced && forced <= kRowsWaves && kRowsWaves / forced <= p.n_loaded) c = forced;
    return p.batch > 32 ? launch_rows_t<2>(p, c, st) : launch_rows_t<1>(p, c, st);
}

}  // namespace bitstack
