// Batch kernel for 2 to 64 tokens, and for up to 1024 in groups of 64, on rebuilt weight units (rebuild.h):
// Y += X (W' diag(1/s))^T, W' of a unit summed over its blocks in registers, multiplied with the activations from there and
// never stored.
//
// One workgroup = RT row tiles of 32 rows x up to 64 tokens; 8 wavefronts = 8 / RT teams (column chunks) x RT row tiles.  A wavefront
// rebuilds its unit of 32 rows x 256 columns block by block; a lane then holds 128 columns of one row, which, scaled by 1/s and
// rounded to fp16, are the B operands of 16 products over 16 columns each, and the activations as they lie in memory (8
// columns of a token: 16 bytes) the A operands.  So the weight costs the same for one token as for 64, and a block costs
// three matrix-core products' worth less than where every block's signed tile meets the activations itself (k_fused in
// panel.hip).  The activations of a chunk come through the same ring of LDS buffers as the blocks' inputs, as one to four
// further steps after the last block.  The teams' partial tiles meet in LDS.
//
// 14336 x 4096, 16 blocks: 78 us for 4 tokens (k_fused 102); 4096 x 14336, 16 tokens: 79 us.  Beyond 64 tokens every group of 64 (a
// grid dimension) rebuilds the weight again, on compute units that are idle otherwise.
// Groups of 128 would need more than the 256 registers that two wavefronts per SIMD leave.
//
// Bound by the issue of vector and matrix instructions (0.79 us a step of 8 tiles per wavefront and two wavefronts per SIMD, registers
// only) and by the arrival of the next steps' inputs: a step takes 1.17 us with RT = 2 and a ring of three, 1.0 us with RT = 4 and a ring
// of four (1.05-1.25 before, when the rebuild took 0.92).
//
// The weight over its scale is rounded to fp16 where k_fused rounds the activation over the scale; the error against fp64 is the same
// to 1.5 % (2.97e-4 of y against 2.93e-4 over 49 shapes).  For weights beyond fp16's range see the end of the accumulation.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"
#include "kparams.h"
#include "layout.h"
#include "rebuild.h"

namespace bitstack {

namespace {

// TOK tokens (16 or 32) per group of activations, GROUPS of them; RT row tiles per workgroup (2 or 4)
template <int TOK, int GROUPS, int RT>
__global__ __launch_bounds__(512, 2) void k_batch(KParams p) {
    constexpr int TEAMS = 8 / RT, kRows = RT * kTileRows;
    constexpr int kRing = RT == 4 ? 4 : 3, kInFlight = RT == 4 ? kStepLoads<RT> : 0;   // every request is four loads then
    typedef StepLayout<RT> L;
    constexpr unsigned kStep = TEAMS * L::kBytes;
    // an activation step brings TOK tokens x kPieces columns of eight per half, at most 4 RT KiB per team
    constexpr int kPieces = RT * 128 / TOK < 16 ? RT * 128 / TOK : 16, kPerGroup = 16 / kPieces, kXSteps = GROUPS * kPerGroup, kXRowBytes = kPieces * 32;
    constexpr unsigned kRsLds = kRing * kStep;   // [2][TEAMS][256] floats
    constexpr unsigned kFlagLds = 8 * 4096;   // two words behind the partial tiles, in the ring when it is idle
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = wave / RT, tile = wave % RT;
    const int hl = lane >> 5, ln = lane & 31;
    const int nch = p.in / kChunkCols, n = p.n_loaded, nrt = p.out / kTileRows;
    const int ksplit = p.n_ks;
    const int c_lo = int(blockIdx.y) * nch / ksplit, c_hi = (int(blockIdx.y) + 1) * nch / ksplit;
    const int iters = (c_hi - c_lo + TEAMS - 1) / TEAMS;
    const int rt = int(blockIdx.x) * RT + tile, rtc = min(rt, nrt - 1);
    const int tok0 = int(blockIdx.z) * (TOK * GROUPS);   // this workgroup's tokens: tok0 .. tok_end - 1
    const int tok_end = min(p.batch, tok0 + TOK * GROUPS);

    const unsigned stride = unsigned(p.block_stride);
    const v4i rsrc = buffer_over(p.blocks, unsigned(n) * stride);
    const v4i x_rsrc = buffer_over(p.x, unsigned(p.batch) * unsigned(p.in) * 2u);
    const v4i rs_rsrc = buffer_over(p.rs, unsigned(p.in) * 4u);
    const unsigned s_lane = unsigned(size_t(rtc) * nch * kUnitBytes) + unsigned(lane) * 16u;
    const unsigned v_lane = v_lane_offset<RT>(unsigned(p.off_v), unsigned(tile), unsigned(lane));
    const unsigned u_lane = u_lane_offset<RT>(unsigned(p.off_u), unsigned(rtc), unsigned(lane));
    const unsigned lds0 = lds_address(smem);
    const unsigned v_rd = lds0 + unsigned(team) * L::kBytes + v_read_offset(unsigned(lane));
    const unsigned s_rd = lds0 + unsigned(wave) * L::kWaveBytes + unsigned(lane) * 16u;
    // x in LDS: a token's 2 kPieces 16-byte pieces in a row, piece j of token t at position j ^ (t & 15)
    const unsigned x_rd = lds0 + unsigned(team) * L::kBytes + unsigned(ln % TOK) * unsigned(kXRowBytes);

    // steps of a chunk: its n blocks, then kXSteps steps of activations
    int qi = 0, qit = 0;
    unsigned qbuf = 0, qoff = 0;
    auto next_buf = [](unsigned q) { return q == (kRing - 1) * kStep ? 0u : q + kStep; };
    auto request = [&]() {
        const int ch = min(c_lo + qit * TEAMS + team, c_hi - 1);
        if (qi < n) {
            load_step<RT>(rsrc, lds0 + qbuf + unsigned(wave) * L::kWaveBytes, s_lane, v_lane, u_lane, qoff + unsigned(ch) * kUnitBytes,
                          qoff + unsigned(ch) * kVChunkBytes, qoff);
            qoff += stride;
        } else {
            // four loads of 1 KiB per wavefront
            const int xs = qi - n, g = xs / kPerGroup, e0 = xs % kPerGroup * kPieces;
            const unsigned mine = lds0 + qbuf + unsigned(team) * L::kBytes + unsigned(tile) * 4096u;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int lin = k * 64 + lane, t = (tile * (4096 / kXRowBytes) + lin / (2 * kPieces)) % TOK;   // token of the group (some twice)
                const int j = (lin % (2 * kPieces)) ^ (t & 15);   // piece: [half][kPieces]
                const int tok = min(tok0 + g * TOK + t, p.batch - 1);
                const unsigned off = unsigned(tok) * unsigned(p.in) * 2u + unsigned(j / kPieces) * 256u + unsigned(j % kPieces + e0) * 16u;
                load_to_lds(x_rsrc, mine + unsigned(k) * 1024u, off, unsigned(ch) * 512u);
            }
        }
        if (++qi == n + kXSteps) {
            qi = 0;
            qoff = 0;
            qit = min(qit + 1, iters - 1);   // past the last step the last chunks are read again, harmlessly
        }
        qbuf = next_buf(qbuf);
    };

    auto request_rs = [&](int it) {   // 1/s of the team's chunk of iteration it, 1 KiB by the team's wavefronts
        const int ch = min(c_lo + it * TEAMS + team, c_hi - 1);
#pragma unroll
        for (int k = 0; k < 4 / RT; ++k) {
            const unsigned part = unsigned(tile * (4 / RT) + k) * 256u;
            load4_to_lds(rs_rsrc, lds0 + kRsLds + unsigned(it & 1) * (TEAMS * 1024) + unsigned(team) * 1024u + part, unsigned(lane) * 4u,
                         unsigned(ch) * (kChunkCols * 4) + part);
        }
    };

    // the thread's number, made anew: what is derived from it outside the loop would cost the loop registers it does not have
    auto own_id = [&]() {
        int t = tid;
        asm volatile("" : "+v"(t));
        return t;
    };

    v16f yacc[GROUPS];
    UnitAcc acc;
    StepInputs in;
    unsigned buf = 0;

    auto accumulate = [&](auto on_x) __attribute__((always_inline)) {
        constexpr bool kScaleX = decltype(on_x)::value;
        const int hl = (own_id() >> 5) & 1;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) yacc[g] = zero16();
        request_rs(0);
        // a step's inputs are requested kRing - 1 steps ahead and have kRing - 2 steps to arrive
        request();
        if constexpr (kRing == 4) request();
        loads_barrier<kInFlight>();
        request();
        begin_reads<RT>(in, v_rd, s_rd);
        in.last = in.s;
        for (int it = 0; it < iters; ++it) {
            auto step = [&](auto first) __attribute__((always_inline)) {
                loads_barrier<kInFlight>();
                request();
                const unsigned nb = next_buf(buf);
                add_block<decltype(first)::value, RT>(acc, in, v_rd + buf, v_rd + nb, s_rd + nb);
                buf = nb;
            };
            step(std::true_type{});
            for (int i = 1; i < n; ++i) step(std::false_type{});
            finish_unit(acc, in);
            // (what the last step read ahead was activations: read again below)
            const bool valid = c_lo + it * TEAMS + team < c_hi;   // uniform over the wavefront
            const unsigned rs_rd = lds0 + kRsLds + unsigned(it & 1) * (TEAMS * 1024) + unsigned(team) * 1024u + unsigned(hl) * 512u;
            v4i b[16];   // W' diag(1/s) of the unit as B operands: step e = columns 8 e .. 8 e + 7 of both halves
            v4f r[2][2];
            auto scale = [&](auto e) __attribute__((always_inline)) {
                constexpr int E = decltype(e)::value;
                v4f(&q)[2] = r[E & 1];
                if constexpr (kScaleX) q[0] = q[1] = v4f{1.0f, 1.0f, 1.0f, 1.0f};
                else if constexpr (E < 15) read_scales(r[(E + 1) & 1], rs_rd, E + 1);
#pragma unroll
                for (int t = 0; t < 8; t += 2)
                    b[E][t >> 1] = scaled_pair(acc[t][E], acc[t + 1][E], q[t >> 2][t & 3], q[t >> 2][(t & 3) + 1]);
                asm volatile("" : "+v"(b[E]));   // made here: put off to the products, it would keep the scales in registers until then
                __builtin_amdgcn_sched_barrier(0);
            };
            if constexpr (!kScaleX) read_scales(r[0], rs_rd, 0);
#define BS_SCALE(E) scale(std::integral_constant<int, E>{});
            BS_SCALE(0) BS_SCALE(1) BS_SCALE(2) BS_SCALE(3) BS_SCALE(4) BS_SCALE(5) BS_SCALE(6) BS_SCALE(7)
            BS_SCALE(8) BS_SCALE(9) BS_SCALE(10) BS_SCALE(11) BS_SCALE(12) BS_SCALE(13) BS_SCALE(14) BS_SCALE(15)
#undef BS_SCALE
#pragma unroll
            for (int xs = 0; xs < kXSteps; ++xs) {
                const int g = xs / kPerGroup, e0 = xs % kPerGroup * kPieces;
                loads_barrier<kInFlight>();
                if (xs == 0) request_rs(it + 1);
                request();
                const unsigned nb = next_buf(buf);
                if (xs == kXSteps - 1) begin_reads<RT>(in, v_rd + nb, s_rd + nb);   // the next chunk's first step
#pragma unroll
                for (int eq = 0; eq < kPieces / 4; ++eq) {
                    v4i a[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const unsigned pos = unsigned(hl * kPieces + eq * 4 + k) ^ unsigned(ln & 15);
                        a[k] = read_lds<v4i>(x_rd + buf + pos * 16u);
                    }
                    if constexpr (kScaleX) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            v4f q[2];
                            read_scales(q, rs_rd, e0 + eq * 4 + k);
                            const v8h h = __builtin_bit_cast(v8h, a[k]);
#pragma unroll
                            for (int t = 0; t < 8; t += 2)
                                a[k][t >> 1] = scaled_pair(float(h[t]), float(h[t + 1]), q[t >> 2][t & 3], q[t >> 2][(t & 3) + 1]);
                        }
                    }
                    if (valid) {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            yacc[g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a[k]),
                                                                             __builtin_bit_cast(v8h, b[e0 + eq * 4 + k]), yacc[g], 0, 0, 0);
                    }
                }
                buf = nb;
            }
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    };

    // the teams' partial tiles meet in LDS; D[i = token][n = row]: lane (row ln), register v holds token
    // 8 (v / 4) + 4 hl + v % 4 of the group
    float* const red = reinterpret_cast<float*>(smem);   // [wave][16][64]
    float* const mine = p.part + size_t(blockIdx.y) * p.batch * p.out;
    auto store = [&]() __attribute__((always_inline)) {
        const int tid = own_id(), lane = tid & 63;
        float rest = 0.0f;   // 0 * y: NaN for infinities and NaN
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            __syncthreads();
            if (g == 0 && tid == 0) write_lds(lds0 + kFlagLds, 0u);
#pragma unroll
            for (int v = 0; v < 16; ++v) red[(wave * 16 + v) * 64 + lane] = yacc[g][v];
            __syncthreads();
            // thread = (row, token): consecutive lanes take consecutive rows
            for (int o = tid; o < kRows * TOK; o += 512) {
                const int row = o & (kRows - 1), t = o / kRows;   // token of the group
                const int v = (t >> 3) * 4 + (t & 3), l = ((t >> 2) & 1) * 32 + (row & 31);
                float sum = 0.0f;
#pragma unroll
                for (int w = 0; w < TEAMS; ++w) sum += red[((w * RT + (row >> 5)) * 16 + v) * 64 + l];
                const int tok = tok0 + g * TOK + t, r = int(blockIdx.x) * kRows + row;
                if (tok < tok_end && r < p.out) {
                    rest = __builtin_fmaf(sum, 0.0f, rest);
                    if (ksplit == 1)
                        store_y(p, size_t(tok) * p.out + r, sum);
                    else   // write-through: the reader may sit on another XCD
                        __hip_atomic_store(mine + size_t(tok) * p.out + r, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        if (rest != 0.0f) write_lds(lds0 + kFlagLds, 1u);
        if (ksplit > 1) __builtin_amdgcn_s_waitcnt(0x0F70);   // each wavefront's stores are acknowledged before it reaches the barrier
        __syncthreads();
    };

    accumulate(std::false_type{});
    store();
    // A weight over its scale need not be an fp16 number where the weight and the activation over the scale are (a channel
    // scaled far down whose activations are tiny, or zero): then y is not finite, and the workgroup starts over with 1/s on the
    // activations, its stores replaced by the same threads.  Not so in the first place: large scales would take the activations out
    // of fp16's range.  The question costs 0.2-0.3 us a call (448 x 256, 1 block, 4 tokens: 5.9 -> 6.2).
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(int(read_lds<unsigned>(lds0 + kFlagLds))), 0)) {
        __syncthreads();   // everybody has seen it
        qi = qit = 0;
        qbuf = qoff = buf = 0u;
        accumulate(std::true_type{});
        store();
    }
    if (ksplit == 1) return;

    // column split: the last workgroup of this row group adds the ksplit partial tiles in a fixed order and stores y (same
    // protocol as the decode kernel: write-through stores, one relaxed agent-scope counter after a barrier, agent-scope
    // loads by the last one)
    unsigned* const flag = reinterpret_cast<unsigned*>(smem + kFlagLds + 4);
    unsigned* const ctr = p.ctr + blockIdx.z * gridDim.x + blockIdx.x;
    if (tid == 0) {
        const unsigned old = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag = (old + 1u == unsigned(ksplit)) ? 1u : 0u;
    }
    __syncthreads();
    if (*flag) {
        const unsigned span = unsigned(size_t(ksplit) * p.batch * p.out * 4);
        __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc(p.part, 0, span, 0x00020000);
        constexpr int kAgentScope = 16;   // sc1
        // thread = (token, 4 consecutive rows)
        for (int o = tid; o < (tok_end - tok0) * (kRows / 4); o += 512) {
            const int tok = tok0 + o / (kRows / 4), row = int(blockIdx.x) * kRows + 4 * (o & (kRows / 4 - 1));
            if (row >= p.out) continue;   // out is a multiple of 32: a quad is inside or outside as a whole
            v4i v[8];
#pragma unroll
            for (int z = 0; z < 8; ++z)
                v[z] = __builtin_amdgcn_raw_buffer_load_b128(
                    prs, z < ksplit ? unsigned(((size_t(z) * p.batch + tok) * p.out + row) * 4) : span, 0, kAgentScope);
            float o4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int z = 0; z < 8; ++z)
#pragma unroll
                for (int k = 0; k < 4; ++k) o4[k] += __int_as_float(v[z][k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) store_y(p, size_t(tok) * p.out + row + k, o4[k]);
        }
        if (tid == 0) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace

constexpr int kBatchMaxSplit = 8;

// Row tiles of a workgroup (RT) and column split, with the estimated duration (microseconds).
//
// Four row tiles share a column chunk's V panel and leave LDS for a ring of four steps: a step's inputs have two steps' time to
// arrive instead of one, which is what a step of two row tiles waits for (14336 x 4096, 16 blocks, 4 tokens: 87 us with two
// row tiles, 78 with four; 4096 x 14336, 16 tokens: 91, 79).  Two row tiles with twice the column chunks per workgroup need no or half
// the column split for the same number of workgroups, so they stay where the workspace allows no split (it holds a partial row per
// split and token) and for calls of a few microseconds (8608 x 768, 3 blocks, 4 tokens: 10.0 us with two, 11.4 with four).
//
// Too few row groups to fill the chip share their column chunks among several workgroups: the split with the fewest rounds x chunk
// iterations, the smallest of equals.  The estimates of the two forms, per round, chunk iteration and block, are fitted to 6120 cases
// (64 x 256 to 28672 x 8192, 1 to 24 blocks, 2 to 300 tokens, each timed with both; 1.9 and 2.5 % root mean square): the form
// taken is 0.01 % slower than the faster one in the mean, one of them by more than 3 %.
struct BatchPlan {
    int rt, split;
    double us;
};
static std::atomic<int> g_forced_tiles{0};
void batch_force_tiles(int tiles) { g_forced_tiles = tiles == 2 || tiles == 4 ? tiles : 0; }
int batch_forced_tiles() { return g_forced_tiles.load(); }

static BatchPlan batch_plan(int out, int in, int batch, int n_loaded, int part_slots) {
    const int nch = in / kChunkCols, forced = g_forced_tiles.load();
    const bool many = batch > 64;
    BatchPlan best = {0, 1, 0.0};
    for (int rt = 4; rt >= 2; rt -= 2) {
        if (forced && forced != rt) continue;
        const int groups = (out + 32 * rt - 1) / (32 * rt) * ((batch + 63) / 64), teams = 8 / rt;
        int split = 1;
        long cost = 0;
        for (int k = 1; k <= kBatchMaxSplit && k <= nch && (k == 1 || k * batch <= part_slots); ++k) {
            if (k > 1 && size_t(k) * batch * out * 4 >= (size_t(1) << 32)) break;   // 32-bit offsets into the partial rows
            const long c = long((groups * k + 255) / 256) * (((nch + k - 1) / k + teams - 1) / teams);
            if (k == 1 || c < cost) {
                split = k;
                cost = c;
            }
        }
        const int wgs = groups * split, its = ((nch + split - 1) / split + teams - 1) / teams;
        const double fill = wgs < 256 ? wgs / 256.0 : 1.0, rounds = (wgs + 255) / 256;
        const int halves = batch > 32 ? 2 : 1;   // groups of up to 32 tokens
        const double tokens = batch > 32 ? 1.0 : batch > 16 ? 0.33 : 0.0, apart = split > 1 ? 1.73 + 0.36 * split * fill : 0.0;
        const double us = rt == 4 ? (many ? 0.3 : 1.6) + 2.2 * tokens + apart +
                                        rounds * ((many ? 4.45 : 2.5) + its * (n_loaded * (0.928 + 0.073 * fill) + 1.16 + 0.74 * halves))
                                  : (many ? 1.2 : 1.5) + 1.1 * tokens + apart +
                                        rounds * ((many ? 3.55 : 2.85) +
                                                  its * (n_loaded * (1.025 + 0.141 * fill) + 1.33 + 0.54 * (batch > 16 ? 2 * halves : 1)));
        if (best.rt == 0 || us < best.us) best = {rt, split, us};
    }
    return best;
}

template <int TOK, int GROUPS, int RT>
static hipError_t launch_batch_t(KParams p, int split, hipStream_t st) {
    const size_t smem = size_t(RT == 4 ? 4 : 3) * (8 / RT) * StepLayout<RT>::kBytes + 2 * (8 / RT) * kChunkCols * 4;
    static std::atomic<bool> attr_set{false};   // setting the attribute twice is harmless
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_batch<TOK, GROUPS, RT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, int(smem));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    p.n_ks = split;
    const dim3 grid((p.out + 32 * RT - 1) / (32 * RT), split, (p.batch + TOK * GROUPS - 1) / (TOK * GROUPS));
    hipLaunchKernelGGL((k_batch<TOK, GROUPS, RT>), grid, dim3(512), smem, st, p);
    return hipGetLastError();
}

// Beyond 64 tokens the crossover to the weight-tile kernel stays where it was when both kernels summed fp16 magnitudes and k_batch had
// two row tiles only (tests/test_gpu_small_batch.py states which kernel is taken): both became faster by about the same, 13 and
// 15-20 %.  In 3690 cases of 33 to 1024 tokens estimates of the present kernels would choose 0.4 % better in the mean.
double batch_time_us(int out, int in, int batch, int n_loaded, int part_slots) {
    if (batch <= 64) return batch_plan(out, in, batch, n_loaded, part_slots).us;
    const int groups = (out + 63) / 64 * ((batch + 63) / 64), nch = in / kChunkCols;
    int split = 1;
    long best = 0;
    for (int k = 1; k <= kBatchMaxSplit && k <= nch && (k == 1 || k * batch <= part_slots); ++k) {
        const long cost = long((groups * k + 255) / 256) * (((nch + k - 1) / k + 3) / 4);
        if (k == 1 || cost < best) {
            split = k;
            best = cost;
        }
    }
    const int wgs = groups * split, its = ((nch + split - 1) / split + 3) / 4;
    const double fill = wgs < 256 ? wgs / 256.0 : 1.0;
    return 3.3 + (wgs + 255) / 256 * (3.5 + its * (n_loaded * (1.02 + 0.17 * fill) + 3.89)) + (split > 1 ? 3.2 : 0.0);
}

// what the launch takes, beyond 64 tokens too
double batch_plan_time_us(int out, int in, int batch, int n_loaded, int part_slots) { return batch_plan(out, in, batch, n_loaded, part_slots).us; }

// one 32-bit buffer descriptor each over the loaded blocks and the activations, one counter per row group and 64 tokens
bool batch_fits(const KParams& p) {
    return size_t(p.n_loaded) * p.block_stride < (size_t(1) << 32) && size_t(p.batch) * p.in * 2 < (size_t(1) << 32) &&
           (size_t(p.out) + 63) / 64 * ((size_t(p.batch) + 63) / 64) <= size_t(kCounterSlots);
}

template <int RT>
static hipError_t launch_batch_rt(const KParams& p, int split, hipStream_t st) {
    return p.batch > 32   ? launch_batch_t<32, 2, RT>(p, split, st)
           : p.batch > 16 ? launch_batch_t<32, 1, RT>(p, split, st)
                          : launch_batch_t<16, 1, RT>(p, split, st);
}

hipError_t launch_batch(const KParams& p, hipStream_t st) {
    const BatchPlan pl = batch_plan(p.out, p.in, p.batch, p.n_loaded, p.part_slots);
    return pl.rt == 4 ? launch_batch_rt<4>(p, pl.split, st) : launch_batch_rt<2>(p, pl.split, st);
}

}  // namespace bitstack
