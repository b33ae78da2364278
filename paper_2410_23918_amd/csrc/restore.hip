// Restoring the dense weight of the loaded prefix (the restoring step of the appendix on inference throughput, "level 2"):
//
//     Wd[o][j] = ( sum_i S_i[o][j] * (U_i V_i^T)[o][j] ) / s[j]        (Eq. 8, Eq. 4 folded into the columns)
//
// as fp16, row-major, in caller-owned memory (dense.hip multiplies it).  One wavefront rebuilds units of 32 rows x 256
// columns (rebuild.h); a workgroup is four of them, 128 rows x one column chunk, and two workgroups share a compute
// unit, so that one's barrier or turn through LDS is covered by the other's arithmetic.
//
// 14336 x 4096, 16 blocks: 76-81 us; 28672 x 8192: 312-350; 2048 x 8192: 25-28 (with magnitudes rounded to fp16 and added by products of
// their own 78-82, 329-368, 26-28).  What bounds it: on whole matrices the issue of vector instructions (half of all cycles) and
// the traffic of signs, U, V and dense rows, which overlap in part; in slabs the first loads and last stores of 512 workgroups at once.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"
#include "kparams.h"
#include "layout.h"
#include "rebuild.h"

namespace bitstack {

constexpr int kRestoreMaxBlocks = 29;
constexpr int kRebuildWaves = 4;                          // wavefronts of a workgroup
constexpr int kRestoreRows = kRebuildWaves * kTileRows;   // a row group: 32 rows per wavefront
typedef StepLayout<kRebuildWaves> Step;
constexpr unsigned kStepBytes = Step::kBytes, kRing = 4;
constexpr unsigned kRsLds = kRing * kStepBytes, kTurnLds = kRsLds + kChunkCols * 4;
constexpr unsigned kTurnBytes = 32 * 64;

// A workgroup restores one column chunk of `groups_per_wg` row groups.  Chunks are the fastest index of the grid: ids are
// dealt round-robin to the XCDs, so an XCD sees few chunks of a wide matrix (an eighth, where the number of chunks is a
// multiple of eight) and keeps their V panels in its L2 while all row groups pass.
__global__ __launch_bounds__(kRebuildWaves * 64, 2) void k_restore(KParams p, int row_groups, int groups_per_wg) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kTurnLds + kRebuildWaves * kTurnBytes];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hl = lane >> 5, ln = lane & 31;
    const int nch = p.in / kChunkCols, n = p.n_loaded;
    const int ch = blockIdx.x;
    const int rg0 = int(blockIdx.y) * groups_per_wg, rg1 = min(row_groups, rg0 + groups_per_wg);
    if (rg0 >= rg1) return;
    const int nrt = p.out / kTileRows, rt_first = p.row_begin / kTileRows + wave;

    const unsigned stride = unsigned(p.block_stride);
    const v4i rsrc = buffer_over(p.blocks, unsigned(n) * stride);
    const v4i rs_rsrc = buffer_over(p.rs, unsigned(p.in) * 4u);
    const unsigned s_lane = unsigned(ch) * kUnitBytes + unsigned(lane) * 16u;
    const unsigned v_lane = v_lane_offset<kRebuildWaves>(unsigned(p.off_v), unsigned(wave), unsigned(lane)) + unsigned(ch) * kVChunkBytes;
    const unsigned u_lane = u_lane_offset<kRebuildWaves>(unsigned(p.off_u), 0u, unsigned(lane));
    const unsigned lds0 = lds_address(smem);
    const unsigned v_rd = lds0 + v_read_offset(unsigned(lane));
    const unsigned s_rd = lds0 + unsigned(wave) * Step::kWaveBytes + unsigned(lane) * 16u;

    // a step = (row group, block), row groups outermost; its inputs are requested three steps ahead, into a ring of
    // four buffers in LDS.  Rows past the end of the matrix repeat its last tile: computed, never stored.
    auto row_tile = [&](int rg) { return min(rt_first + rg * kRebuildWaves, nrt - 1); };
    int qi = 0, qrg = rg0;
    unsigned qv = 0, qs = unsigned(row_tile(rg0)) * unsigned(nch) * kUnitBytes, qu = unsigned(row_tile(rg0)) * 1024u;
    unsigned qbuf = 0;
    auto request = [&]() {
        load_step<kRebuildWaves>(rsrc, lds0 + qbuf + unsigned(wave) * Step::kWaveBytes, s_lane, v_lane, u_lane, qs, qv, qu);
        qv += stride;
        qs += stride;
        qu += stride;
        if (++qi == n) {
            qi = 0;
            qv = 0;
            qrg = min(qrg + 1, rg1 - 1);   // past the last step the last row group is read again, harmlessly
            qs = unsigned(row_tile(qrg)) * unsigned(nch) * kUnitBytes;
            qu = unsigned(row_tile(qrg)) * 1024u;
        }
        qbuf = (qbuf + kStepBytes) & (kRing * kStepBytes - 1);
    };
    constexpr int kInFlight = kStepLoads<kRebuildWaves>;   // loads of one step and wavefront

    UnitAcc acc;
    StepInputs in;
    unsigned buf = 0;
    load4_to_lds(rs_rsrc, lds0 + kRsLds + unsigned(wave) * 256u, unsigned(lane) * 4u, unsigned(ch) * (kChunkCols * 4) + unsigned(wave) * 256u);
    request();
    request();
    loads_barrier<kInFlight>();
    request();
    begin_reads<kRebuildWaves>(in, v_rd, s_rd);
    in.last = in.s;
    auto step = [&](auto first) __attribute__((always_inline)) {
        // the next step's inputs have landed (this wavefront's loads, then everybody's), and nobody reads the previous
        // step's any more
        loads_barrier<kInFlight>();
        request();
        const unsigned nb = (buf + kStepBytes) & (kRing * kStepBytes - 1);
        add_block<decltype(first)::value, kRebuildWaves>(acc, in, v_rd + buf, v_rd + nb, s_rd + nb);
        buf = nb;
    };
    // The unit times 1/s (Eq. 4 folded into the columns), as fp16 to the dense matrix.  A lane holds 256
    // consecutive bytes of one row; it is turned through LDS (private to the wavefront, no barrier), 64 bytes per row
    // of a half at a time, so that four lanes store 64 consecutive bytes.  Stored as the lanes hold them, 16 bytes each
    // at 64 places, the stores took as long as everything else together.
    const unsigned rs_rd = lds0 + kRsLds + unsigned(hl) * 512u;
    const unsigned turn = lds0 + kTurnLds + unsigned(wave) * kTurnBytes;
    const unsigned wr = turn + unsigned(ln) * 64u, swz = (unsigned(ln) >> 2) & 3u;
    const unsigned rd = turn + (unsigned(lane) >> 2) * 64u + (((unsigned(lane) & 3u) ^ (unsigned(lane) >> 4)) * 16u);
    auto flush = [&](int rt) {
        unsigned char* const dst = static_cast<unsigned char*>(p.wdense) +
                                   (size_t(rt * kTileRows + (lane >> 2) - p.row_begin) * p.in + ch * kChunkCols) * 2 + (lane & 3) * 16;
        unsigned char* const dst16 = dst + size_t(p.in) * 32;   // 16 rows further down
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            v4i o[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                v4f r[2];
                read_scales(r, rs_rd, w * 4 + b);
#pragma unroll
                for (int t = 0; t < 8; t += 2)
                    o[b][t >> 1] = scaled_pair(acc[t][4 * w + b], acc[t + 1][4 * w + b], r[t >> 2][t & 3], r[t >> 2][(t & 3) + 1]);
            }
            v4i q[4];
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (hl == half) {
#pragma unroll
                    for (int b = 0; b < 4; ++b) write_lds(wr + ((unsigned(b) ^ swz) * 16u), o[b]);
                }
                wavefront_lds_order();
                q[2 * half] = read_lds<v4i>(rd);
                q[2 * half + 1] = read_lds<v4i>(rd + 1024u);
                wavefront_lds_order();
            }
            *reinterpret_cast<v4i*>(dst + w * 64) = q[0];
            *reinterpret_cast<v4i*>(dst16 + w * 64) = q[1];
            *reinterpret_cast<v4i*>(dst + 256 + w * 64) = q[2];
            *reinterpret_cast<v4i*>(dst16 + 256 + w * 64) = q[3];
        }
    };
    for (int rg = rg0; rg < rg1; ++rg) {
        step(std::true_type{});
        for (int i = 1; i < n; ++i) step(std::false_type{});
        finish_unit(acc, in);
        const int rt = rt_first + rg * kRebuildWaves;
        if (rt < nrt) flush(rt);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // no load may land in LDS after the workgroup has given it back
}

// Row groups per workgroup: one, until the workgroups are many more than the 512 that run at a time; then a few, whose
// first loads are paid once (28672 x 8192: 7168 workgroups of one group 386 us, 1792 of four 346 us; 14336 x 4096: 1792 of
// one 78 us, 448 of four, whose last round is three quarters empty, 96 us).
static int restore_groups_per_wg(int groups, int chunks) {
    const int per = groups * chunks / 1536;
    return per < 1 ? 1 : per > 4 ? 4 : per;
}

// Duration (microseconds), for the choice of kernel: rounds of 512 workgroups, part of each shared with the next, and the traffic of the
// dense rows.  Fitted to 7053 cases (512 x 512 to 28672 x 8192, 1 to 24 blocks; 6.7 % root mean square).
double restore_time_us(int rows, int in, int n_loaded) {
    const int groups = (rows + kRestoreRows - 1) / kRestoreRows, chunks = in / kChunkCols, per = restore_groups_per_wg(groups, chunks);
    const int wgs = chunks * ((groups + per - 1) / per);
    const double fill = wgs < 512 ? wgs / 512.0 : 1.0, rounds = 0.36 * ((wgs + 511) / 512) + 0.64 * (wgs < 512 ? 1.0 : wgs / 512.0);
    return 3.27 + rounds * (per * (n_loaded * (0.496 + 0.558 * fill) + 3.49) - 2.78) + 0.267e-6 * rows * in;
}

// The block count is what bitstack_restore_max_blocks has always answered (the kernel before k_restore kept every block's U in LDS);
// k_restore has no such limit.  It reaches the loaded blocks through one buffer descriptor with 32-bit offsets.
int restore_max_blocks() { return kRestoreMaxBlocks; }
bool restore_fits(size_t block_stride, int n_loaded) {
    return n_loaded <= kRestoreMaxBlocks && size_t(n_loaded) * block_stride < (size_t(1) << 32);
}

hipError_t launch_restore(const LaunchArgs& a, hipStream_t st) {
    KParams p = make_params(a);
    if (a.n_loaded < 1 || !restore_fits(p.block_stride, a.n_loaded) || p.wdense == nullptr) return hipErrorInvalidValue;
    const int slab_rows = a.rows ? a.rows : p.out;
    if (a.row_begin % 256 || a.row_begin < 0 || a.row_begin >= p.out || slab_rows < 1) return hipErrorInvalidValue;
    const int rows = min(slab_rows, p.out - a.row_begin);
    const int groups = (rows + kRestoreRows - 1) / kRestoreRows;
    const int chunks = p.in / kChunkCols, per = restore_groups_per_wg(groups, chunks);
    hipLaunchKernelGGL(k_restore, dim3(chunks, (groups + per - 1) / per), dim3(kRebuildWaves * 64), 0, st, p, groups, per);
    return hipGetLastError();
}

}  // namespace bitstack
