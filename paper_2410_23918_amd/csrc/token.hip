// One token through a small stack: the decode path (y = (sum_i S_i (.) (U_i V_i^T)) diag(1/s) x, Eq. 4 + Eq. 8) where launch and
// latency are all there is.
//
// k_decode (decode.hip) needs three barriers before its first product (x/s table, exact maxima, quantised panel) because an
// integer panel wants one scale per column range.  Here the activation goes onto V as an fp16 factor, which needs a scale only to
// stay in range, and a wavefront takes one sign unit (32 rows x 256 columns of one block) from its loads to its row sums alone:
//   * every load is issued at entry: V of the chunk to LDS, signs, U, x and 1/s of the lane's columns to registers;
//   * per column class t: A = V (8 ranks of one column, turned by the transposing LDS read) times x/s of that column, which is the
//     lane's own (the columns that a lane holds for the eight classes are eight neighbours); B = U of the row; the product is the
//     contribution of the class's 32 columns to 32 rows, before the sign;
//   * sign and sum as in rebuild.h: the accumulator holds the sum times the sign of the class added last, so a class flips the
//     signs that differ and its product adds in place.  Two accumulators take turns, so that one's product covers the other's flips.
// A workgroup is eight units of one row tile; more than eight meet in the workspace (k_decode's protocol: write-through stores, one
// relaxed agent-scope counter, the last arriver adds the partial rows in a fixed order).
//
// 512 x 512, 4 blocks: 9.3 -> 4.5 us; 1024 x 4096, 3 blocks: 10.9 -> 6.2 (k_decode, this kernel; graph replay).  Bound by launch, one
// memory latency and, with partial rows, the protocol's two more; on larger stacks by V, which every row tile loads again (1024 x
// 4096, 16 blocks: 12.1 and 12.5).
//
// Error: V and x/s are multiplied in fp16 (x/s rounded, the product rounded), as in k_decode's quantiser, whose fixed point comes on
// top there: 3.6e-4 of y where k_decode has 4.0e-4 (41 drawn stacks against fp64); sums are fp32.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "kparams.h"
#include "layout.h"
#include "rebuild.h"

namespace bitstack {

namespace {

constexpr int kTokenWaves = 8;

// largest of the non-negative floats of a wavefront's lanes (as integers), in all lanes
__device__ __forceinline__ int wave_max(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, false));   // row_ror:8
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x124, 0xF, 0xF, false));   // row_ror:4
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x122, 0xF, 0xF, false));   // row_ror:2
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x121, 0xF, 0xF, false));   // row_ror:1
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// one workgroup: part `part` of p.n_ks of row tile rt
__device__ __forceinline__ void token_part(const KParams& p, int rt, int part) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kTokenWaves * kVChunkBytes];
    __shared__ float red[kTokenWaves * 2][kTileRows];
    __shared__ unsigned last_one;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hl = lane >> 5, m = lane & 31;
    const int nch = p.in / kChunkCols, units = p.n_loaded * nch;
    const int parts = p.n_ks;
    const int unit = part * kTokenWaves + wave;
    float sum = 0.0f;   // of row m, both lane halves
    if (unit < units) {   // uniform over the wavefront
        const int blk = unit / nch, ch = unit - blk * nch;
        const unsigned char* const block = p.blocks + size_t(blk) * p.block_stride;
        const unsigned lds = lds_address(smem) + unsigned(wave) * kVChunkBytes;
        const v4i rsrc = buffer_over(block + p.off_v, unsigned(p.in) * 32u);
#pragma unroll
        for (int t = 0; t < kClasses; ++t)
            load_to_lds(rsrc, lds + unsigned(t) * kVClassBytes, v_piece_offset(unsigned(lane)), unsigned(ch) * kVChunkBytes + unsigned(t) * kVClassBytes);
        // column of row m of the A operand in class t: the first of the eight + t
        const int col = ch * kChunkCols + ((m >> 2) & 1) * 128 + (m >> 3) * 32 + (m & 3) * 8;
        const v4i xw = *reinterpret_cast<const v4i*>(p.x + col);
        const v4f r0 = *reinterpret_cast<const v4f*>(p.rs + col), r1 = *reinterpret_cast<const v4f*>(p.rs + col + 4);
        const v2u vm = *reinterpret_cast<const v2u*>(p.vmax + size_t(blk) * p.in + ch * kChunkCols + lane * 4);
        const v4i sw = *reinterpret_cast<const v4i*>(block + (size_t(rt) * nch + ch) * kUnitBytes + lane * 16);
        const v4i u = *reinterpret_cast<const v4i*>(block + p.off_u + size_t(rt * kTileRows + m) * 32 + hl * 16);

        float xs[8];
        int xm = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int two = xw[k];   // (a copy: a cast of a vector's element takes element 0)
            const v2h h = __builtin_bit_cast(v2h, two);
            xs[2 * k] = float(h[0]) * (k < 2 ? r0[2 * k] : r1[2 * k - 4]);
            xs[2 * k + 1] = float(h[1]) * (k < 2 ? r0[2 * k + 1] : r1[2 * k - 3]);
            xm = max(xm, max(__float_as_int(fabsf(xs[2 * k])), __float_as_int(fabsf(xs[2 * k + 1]))));
        }
        // max_r |V| of the chunk's channels: fp16 magnitudes compare like their bits
        const int vb = wave_max(int(max(max(vm[0] & 0xFFFFu, vm[0] >> 16), max(vm[1] & 0xFFFFu, vm[1] >> 16))));
        const float vmax = fmaxf(float(__builtin_bit_cast(_Float16, (unsigned short)vb)), 1.0f);
        // x/s times 2^k below 2^14, and times V too: products of 2^-28 of the largest are still normal numbers
        const int bound = __float_as_int(__int_as_float(wave_max(xm)) * vmax);
        const int k = min(13 - ((bound >> 23) - 127), 126);
        const float f = __int_as_float((k + 127) << 23);
        v2h xh[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) xh[t][0] = xh[t][1] = _Float16(xs[t] * f);

        // bit t of a byte: does the sign of class t differ from that of class t + 2 (t < 6), the class before it on its accumulator
        SignWords w, d;
        w.w[0] = v2u{unsigned(sw[0]), unsigned(sw[1])};
        w.w[1] = v2u{unsigned(sw[2]), unsigned(sw[3])};
#pragma unroll
        for (int q = 0; q < 2; ++q) d.w[q] = (w.w[q] ^ (w.w[q] >> 2)) << 2;   // class 5 at bit 7
        const unsigned rd = lds + v_read_offset(unsigned(lane));
        auto factor = [&](int t) __attribute__((always_inline)) -> VFrag {
            VFrag a{read_lds_turned(rd + unsigned(t) * kVClassBytes), read_lds_turned(rd + unsigned(t) * kVClassBytes + 512u)};
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const unsigned v0 = a.q0[q], v1 = a.q1[q];
                a.q0[q] = __builtin_bit_cast(unsigned, __builtin_bit_cast(v2h, v0) * xh[t]);
                a.q1[q] = __builtin_bit_cast(unsigned, __builtin_bit_cast(v2h, v1) * xh[t]);
            }
            return a;
        };
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // V is in LDS (this wavefront's own loads)
        VFrag a[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) a[t] = factor(t);
        __builtin_amdgcn_sched_barrier(0);
        v16f acc[2];   // [t & 1]
        acc[1] = magnitude(a[7], u, zero16());
        acc[0] = magnitude(a[6], u, zero16());
        asm volatile("s_nop 15");   // the first product (the compiler does not look into the flips)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 5; t >= 0; --t) {
            const FlipMasks mk = flip_masks(d);
            next_class(d);
            flip_class(acc[t & 1], mk);
            asm volatile("s_nop 3");
            __builtin_amdgcn_sched_barrier(0);
            acc[t & 1] = magnitude(a[t], u, acc[t & 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the signs of classes 1 and 0 off the sums; a cleared bit marks a negative sign
        SignWords s0, s1;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            s0.w[q] = ~w.w[q] << 7;
            s1.w[q] = ~w.w[q] << 6;
        }
        const FlipMasks m0 = flip_masks(s0), m1 = flip_masks(s1);
        asm volatile("s_nop 15");
        __builtin_amdgcn_sched_barrier(0);
        flip_class(acc[1], m1);
        __builtin_amdgcn_sched_barrier(0);
        flip_class(acc[0], m0);
        __builtin_amdgcn_sched_barrier(0);
        float s4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int v = 0; v < 16; ++v) s4[v & 3] += acc[0][v] + acc[1][v];
        sum = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        sum += __shfl_xor(sum, 32);
        sum *= __int_as_float((127 - k) << 23);
    }
    if (hl == 0) red[wave][m] = sum;
    __syncthreads();
    const int row = rt * kTileRows + tid;
    float tot = 0.0f;
    if (tid < kTileRows) {
#pragma unroll
        for (int w = 0; w < kTokenWaves; ++w) tot += red[w][tid];
        if (parts == 1) store_y(p, size_t(row), tot);
        else __hip_atomic_store(&p.part[size_t(part) * p.out + row], tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (parts == 1) return;
    if (wave == 0) {
        __builtin_amdgcn_s_waitcnt(0x0F70);   // the write-through stores are acknowledged before the counter is bumped
        if (lane == 0) {
            const unsigned old = __hip_atomic_fetch_add(&p.ctr[rt * kCounterStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last_one = old + 1u == unsigned(parts) ? 1u : 0u;
        }
    }
    __syncthreads();
    if (!last_one) return;
    // thread = (row, every 16th part), all loads of a round in flight together
    const unsigned span = unsigned(size_t(parts) * p.out * 4);
    __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc(p.part, 0, span, 0x00020000);
    constexpr int kAgentScope = 16;   // sc1
    const int g = tid >> 5, r = tid & 31;
    float mine = 0.0f;
    for (int p0 = g; p0 < parts; p0 += 64) {
        int v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int s = p0 + 16 * q;
            v[q] = __builtin_amdgcn_raw_buffer_load_b32(prs, s < parts ? unsigned((size_t(s) * p.out + rt * kTileRows + r) * 4) : span, 0, kAgentScope);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) mine += __int_as_float(v[q]);   // parts past the end read as zero
    }
    red[g][r] = mine;
    __syncthreads();
    if (tid < kTileRows) {
        float y = 0.0f;
#pragma unroll
        for (int q = 0; q < 16; ++q) y += red[q][tid];
        store_y(p, size_t(row), y);
    }
    if (tid == 0) __hip_atomic_store(&p.ctr[rt * kCounterStride], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(kTokenWaves * 64) void k_token(KParams p) { token_part(p, blockIdx.x, blockIdx.y); }

// several stacks that read the same vector: workgroups base[i] .. base[i + 1] - 1 are stack i's, the same as in a launch of its own
__global__ __launch_bounds__(kTokenWaves * 64) void k_token_group(KGroup grp) {
    int i = 0;
    while (i + 1 < grp.count && blockIdx.x >= grp.base[i + 1]) ++i;
    const int local = int(blockIdx.x - grp.base[i]), tiles = grp.s[i].out / kTileRows;
    token_part(grp.s[i], local % tiles, local / tiles);
}

}  // namespace

// Workgroups per row tile; 0: this kernel does not serve the stack
static int token_parts(int out, int in, int n_loaded, int part_slots) {
    const long units = long(n_loaded) * (in / kChunkCols), parts = (units + kTokenWaves - 1) / kTokenWaves;
    const int tiles = out / kTileRows;
    if (parts > 1 && (parts > part_slots || parts > 1024 || long(tiles) * kCounterStride > kCounterSlots)) return 0;
    return int(parts);
}

// Estimated duration (microseconds; fitted to 900 stacks of 32 x 256 to 16384 x 14336 with up to 24 blocks): one workgroup per row tile
// 4.4, with partial rows 6.1; two workgroups to a compute unit 1.2-2.1 more; from 512 workgroups on their number counts, V being
// loaded anew for every row tile.
double token_time_us(const LaunchArgs* a, int count) {
    long wgs = 0;
    int most = 1;
    for (int i = 0; i < count; ++i) {
        const int parts = token_parts(a[i].geo.out, a[i].geo.in, a[i].n_loaded, a[i].ws_part ? a[i].ws_part_slots : a[i].geo.part_slots);
        if (parts == 0) return 0.0;
        for (int j = 0; j < i; ++j)
            if (a[j].image == a[i].image) return 0.0;   // members that share a workspace
        wgs += long(a[i].geo.out / kTileRows) * parts;
        most = parts > most ? parts : most;
    }
    if (wgs > 512) return 5.2 + 0.0088 * wgs + 0.015 * most;
    return (most == 1 ? 4.4 : 6.1) + (wgs > 256 ? 1.2 + 0.9 * (wgs - 256) / 256 : 0.0);
}

void prepare_token(const LaunchArgs* a, int count, DecodeLaunch* d) {
    d->token = true;
    d->tiles = d->early = 0;
    d->grp.count = count;
    unsigned next = 0;
    for (int i = 0; i < count; ++i) {
        KParams& p = d->grp.s[i];
        p = make_params(a[i]);
        p.n_ks = token_parts(p.out, p.in, p.n_loaded, p.part_slots);
        d->grp.base[i] = next;
        next += unsigned(p.out / kTileRows) * unsigned(p.n_ks);
    }
    for (int i = count; i < kMaxGroup; ++i) d->grp.s[i] = d->grp.s[0];
    for (int i = count; i <= kMaxGroup; ++i) d->grp.base[i] = next;
    d->wgs = next;
}

hipError_t launch_token(const DecodeLaunch& d, hipStream_t st) {
    const KParams& p = d.grp.s[0];
    if (d.grp.count == 1)
        hipLaunchKernelGGL(k_token, dim3(p.out / kTileRows, p.n_ks), dim3(kTokenWaves * 64), 0, st, p);
    else
        hipLaunchKernelGGL(k_token_group, dim3(d.wgs), dim3(kTokenWaves * 64), 0, st, d.grp);
    return hipGetLastError();
}

}  // namespace bitstack
