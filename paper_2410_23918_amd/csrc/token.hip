// One token through a small stack: the decode path (y = (sum_i S_i (.) (U_i V_i^T)) diag(1/s) x, Eq. 4 + Eq. 8) where launch and
// latency are all there is.
//
// k_decode (decode.hip) needs three barriers before its first product (x/s table, exact maxima, quantised panel) because an
// integer panel wants one scale per column range.  Here nothing is quantised, and a wavefront takes one sign unit (32 rows x 256
// columns of one block) from its loads to its row sums alone:
//   * every load is issued at entry: V of the chunk to LDS, signs, U, x and 1/s of eight columns per lane to registers;
//   * per column class t the magnitudes of its 32 columns x 32 rows by one matrix product, V (8 ranks of one column, turned by the
//     transposing LDS read) times U, exactly as they are stored;
//   * a lane then holds sixteen columns of its row: their signs are flipped by the bytes of its sign words (rebuild.h), and
//     sum += magnitude * x/s in fp32.  x/s of the sixteen columns is the same for all rows; each row of sixteen lanes keeps it with one
//     column per lane and class, and the multiply-add takes it from there (row_newbcast).
// A workgroup is eight units of one row tile; more than eight meet in the workspace (k_decode's protocol: write-through stores, one
// relaxed agent-scope counter, the last arriver adds the partial rows in a fixed order).
//
// 512 x 512, 4 blocks: 9.1 and 4.4 us; 1024 x 4096, 3 blocks: 10.8 and 5.9 (k_decode, this kernel; graph replay).  Bound by launch, one
// memory latency and, with partial rows, the protocol's two more; on larger stacks by V, which every row tile loads again (1024 x
// 4096, 12 blocks: 11.9 and 10.1).  Putting x/s onto V as an fp16 factor before the product, so that signs and sums stay in the
// accumulator (rebuild.h), takes 4 % longer and needs a scale: one from separate maxima of |x/s| and |V| loses every column where the
// loudest channel has no weight.
//
// Error: sums and products in fp32 and nothing rounded before y: 1.5e-7 of y where k_decode's fixed point has 3.4e-4 (41 drawn stacks
// against fp64, fp32 outputs).
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "kparams.h"
#include "layout.h"
#include "rebuild.h"

namespace bitstack {

namespace {

constexpr int kTokenWaves = 8;

// s += sum of a x/s over the sixteen columns of one class, a the magnitudes of the lane's row with their signs taken from m: the class's
// bits stand at bit 7 of the bytes (set: negative; the other bits of bytes 0 to 2 cleared).  Lane e of a row of sixteen has register e's x/s.
// The compiler places the wait states behind a matrix product where an instruction of its own reads the result, but does not look into
// assembly.  So the first flip is its own, and the others take that one as an operand; the rest is one statement that keeps its own
// distances (one instruction between a sub-dword operation and a reader, two between a vector instruction and a row operation).
__device__ __forceinline__ void add_class(float (&s)[4], v16f a, const FlipMasks& m, float xs) {
    const unsigned top = 0x80000000u;
    a[3] = __int_as_float(__float_as_int(a[3]) ^ int(m.w[0] & top));
    asm("v_xor_b32_sdwa %4, %4, %[m0] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_0\n\t"
        "v_xor_b32_sdwa %5, %5, %[m0] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_1\n\t"
        "v_xor_b32_sdwa %6, %6, %[m0] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_2\n\t"
        "v_xor_b32_sdwa %7, %7, %[m1] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_0\n\t"
        "v_xor_b32_sdwa %8, %8, %[m1] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_1\n\t"
        "v_xor_b32_sdwa %9, %9, %[m1] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_2\n\t"
        "v_xor_b32_sdwa %11, %11, %[m2] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_0\n\t"
        "v_xor_b32_sdwa %12, %12, %[m2] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_1\n\t"
        "v_xor_b32_sdwa %13, %13, %[m2] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_2\n\t"
        "v_xor_b32_sdwa %15, %15, %[m3] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_0\n\t"
        "v_xor_b32_sdwa %16, %16, %[m3] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_1\n\t"
        "v_xor_b32_sdwa %17, %17, %[m3] dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_2\n\t"
        "v_bitop3_b32 %10, %10, %[m1], %[top] bitop3:0x78\n\t"   // a ^ (m & top)
        "v_bitop3_b32 %14, %14, %[m2], %[top] bitop3:0x78\n\t"
        "v_bitop3_b32 %18, %18, %[m3], %[top] bitop3:0x78\n\t"
        "v_fmac_f32_dpp %0, %[xs], %4 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %[xs], %5 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %[xs], %6 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %[xs], %[a3] row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %[xs], %7 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %[xs], %8 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %[xs], %9 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %[xs], %10 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %[xs], %11 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %[xs], %12 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %[xs], %13 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %[xs], %14 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %[xs], %15 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %[xs], %16 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %[xs], %17 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %[xs], %18 row_newbcast:15 row_mask:0xf bank_mask:0xf"
        : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3]),
          "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(a[8]), "+v"(a[9]), "+v"(a[10]),
          "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15])
        : [m0] "v"(m.w[0]), [m1] "v"(m.w[1]), [m2] "v"(m.w[2]), [m3] "v"(m.w[3]), [a3] "v"(a[3]), [top] "v"(top), [xs] "v"(xs));
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
        // the eight columns, one per class, that this lane keeps x/s of for its row of sixteen lanes: lane e has register e's
        const int col = ch * kChunkCols + hl * 128 + (lane & 15) * 8;
        const v4i xw = *reinterpret_cast<const v4i*>(p.x + col);
        const v4f r0 = *reinterpret_cast<const v4f*>(p.rs + col), r1 = *reinterpret_cast<const v4f*>(p.rs + col + 4);
        const v4i sw = *reinterpret_cast<const v4i*>(block + (size_t(rt) * nch + ch) * kUnitBytes + lane * 16);
        const v4i u = *reinterpret_cast<const v4i*>(block + p.off_u + size_t(rt * kTileRows + m) * 32 + hl * 16);

        float xs[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int two = xw[k];   // (a copy: a cast of a vector's element takes element 0)
            const v2h h = __builtin_bit_cast(v2h, two);
            xs[2 * k] = float(h[0]) * (k < 2 ? r0[2 * k] : r1[2 * k - 4]);
            xs[2 * k + 1] = float(h[1]) * (k < 2 ? r0[2 * k + 1] : r1[2 * k - 3]);
        }
        SignWords d;   // negative signs; class 7 at bit 7 of the bytes
        d.w[0] = v2u{~unsigned(sw[0]), ~unsigned(sw[1])};
        d.w[1] = v2u{~unsigned(sw[2]), ~unsigned(sw[3])};
        const unsigned rd = lds + v_read_offset(unsigned(lane));
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // V is in LDS (this wavefront's own loads)
        VFrag a[kClasses];
#pragma unroll
        for (int t = 0; t < kClasses; ++t) a[t] = VFrag{read_lds_turned(rd + unsigned(t) * kVClassBytes), read_lds_turned(rd + unsigned(t) * kVClassBytes + 512u)};
        __builtin_amdgcn_sched_barrier(0);
        float s4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        v16f w[2];   // a class's product is under way while the one before it is added up
        w[1] = magnitude(a[7], u, zero16());
#pragma unroll
        for (int t = kClasses - 1; t >= 0; --t) {
            if (t > 0) w[(t - 1) & 1] = magnitude(a[t - 1], u, zero16());
            __builtin_amdgcn_sched_barrier(0);
            const FlipMasks mk = flip_masks(d);
            next_class(d);
            add_class(s4, w[t & 1], mk, xs[t]);
            __builtin_amdgcn_sched_barrier(0);
        }
        sum = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        sum += __shfl_xor(sum, 32);
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
// loaded anew for every row tile.  Merged launches (184 of 2 to 4 stacks) take 3 % longer than that, up to 17 % beyond 512 workgroups, and
// what k_decode takes for the same is estimated too high: of 38 whose estimates were less than 3 us apart one was 24 % slower than
// through k_decode and the mean 3 % faster, so these go there.
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
    if (wgs > 512) return 5.2 + 0.0088 * wgs + 0.015 * most + (count > 1 ? 2.0 : 0.0);
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
