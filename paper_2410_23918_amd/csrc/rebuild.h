// Rebuilding weight tiles on chip (gfx950): the part that the restore kernel and the batch kernels share.
//
//     W'[o][j] = sum_i S_i[o][j] * (U_i V_i^T)[o][j]              (Eq. 8)
//
// A wavefront owns one sign unit's worth of the weight, 32 rows x 256 columns, as 128 fp32 accumulators
// per lane, and adds one block per step:
//   * signs: one 128-bit load per lane, exactly the unit as it lies in memory.  Lane (half g, row j) holds
//     the 128 sign bits of row j in column half g;
//   * magnitudes: per column class t (the 32 columns whose bit in the lane's sixteen bytes is bit t: one
//     per byte e and half) one v_mfma_f32_32x32x16_f16 over the 16 ranks.  The A operand's rows are the class's
//     columns, ordered so that lane (g, j) receives, in register e, column (g, e, t) of row j: the columns of its own
//     sign words, in the order of their bytes;
//   * sign: registers e and e + 2 of a word sit 16 bits apart in it.  They are packed to a pair of fp16
//     (convert-pack), and one three-input bit operation flips the pair's signs by bits 15 and 31 of a copy
//     of the word that moves up by one bit per class (two words per instruction: v_lshl_add_u64; the bit that
//     crosses from one word into the other stays below bit 8);
//   * sum: v_mfma_f32_4x4x4_16b_f16 with a permutation matrix as A adds the four fp16 values a lane holds to
//     four of its own fp32 accumulators: 256 elements in 8 cycles, where a 32x32x16 product with an identity
//     takes 32 cycles for 512.
// Registers only, that is 56 ns per 32 x 32 tile, block and SIMD (the former scheme with a shift per pair and two
// 32x32x16 identity products: 77).
//
// V needs its 16 x 16 pieces (16 ranks x 16 columns of one half and class) turned from rank rows, as they lie in
// memory, into "8 ranks of one column".  The V panel goes to LDS without passing through registers
// (128-bit buffer loads to LDS, one KiB per class) and is turned by the transposing LDS read
// ds_read_b64_tr_b16.  The 16-byte pieces of a class are ordered in LDS so that one such read of a
// wavefront covers 512 consecutive bytes: no bank conflicts.
#pragma once
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "layout.h"

namespace bitstack {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

constexpr int kClasses = 8;                 // column classes of a unit (bit positions in a byte)
constexpr int kVClassBytes = 1024;          // V of one class: 2 halves x 16 ranks x 16 columns fp16
constexpr int kVChunkBytes = kClasses * kVClassBytes;

// The RT wavefronts (4 or 2 row tiles) that work on the same column chunk share its V panel; each loads its own signs and U
// and 8 / RT classes of V.  One step's inputs in LDS, per wavefront: [signs 1 KiB][V of its classes][U 1 KiB].
template <int RT>
struct StepLayout {
    static constexpr int kClassesPerWave = kClasses / RT;
    static constexpr int kVOffset = 1024, kUOffset = kVOffset + kClassesPerWave * kVClassBytes, kWaveBytes = kUOffset + 1024;
    static constexpr int kBytes = RT * kWaveBytes;
    static constexpr int frag(int t) { return t / kClassesPerWave * kWaveBytes + kVOffset + t % kClassesPerWave * kVClassBytes; }
};

typedef __attribute__((address_space(3))) void lds_void;

// All but the last N vector memory operations of this wavefront are complete, then the workgroup's barrier.  (The
// fences of lds_barrier() would wait for every load to LDS in flight.)  The LDS reads before it must have been
// consumed: it does not wait for them.
template <int N>
__device__ __forceinline__ void loads_barrier() {
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
}

// 16 (4) bytes per lane from the buffer to LDS, lane after lane (asynchronous, counted by vmcnt).  OFF is added to
// both addresses.
template <int OFF>
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t rsrc, void* lds, unsigned lane_off, unsigned soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)lds, 16, lane_off, soff, OFF, 0);
}
__device__ __forceinline__ void load4_to_lds(__amdgpu_buffer_rsrc_t rsrc, void* lds, unsigned lane_off, unsigned soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)lds, 4, lane_off, soff, 0, 0);
}

// byte offset inside a class's KiB in memory of the 16-byte piece that lane u of a load to LDS fetches.  In LDS
// the pieces are ordered [rank quad of a rank half][rank half][rank][column half][columns 0-7 / 8-15].
__device__ __forceinline__ unsigned v_piece_offset(unsigned u) {
    const unsigned q = u >> 5, kg = (u >> 4) & 1, rr = (u >> 2) & 3, g = (u >> 1) & 1, eh = u & 1;
    return (g * 16 + kg * 8 + q * 4 + rr) * 32 + eh * 16;
}
// byte offset inside a class's KiB in LDS that a lane reads from (rank quad 0; quad 1 is 512 bytes on)
__device__ __forceinline__ unsigned v_read_offset(unsigned lane) {
    const unsigned kg = lane >> 5, grp = (lane >> 4) & 1, rr = (lane >> 2) & 3, pc = lane & 3;
    return kg * 256 + rr * 64 + (pc & 1) * 32 + (grp * 2 + (pc >> 1)) * 8;
}

// The LDS reads of the pipeline below are inline assembly: for an ordinary LDS read the compiler would first wait for
// every load to LDS that is in flight, and those are requested several steps ahead.  Their results are valid only after
// a wait on them (wait_lds<N>: at most N reads requested since may be outstanding; LDS reads return in order).
struct VFrag {
    v2u q0, q1;
};
// A operand of the magnitude product of class T: two reads
template <int T, int RT>
__device__ __forceinline__ void read_frag(VFrag& f, unsigned addr) {
    asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                 : "=&v"(f.q0), "=&v"(f.q1)
                 : "v"(addr), "n"(StepLayout<RT>::frag(T)), "n"(StepLayout<RT>::frag(T) + 512));
}
template <int OFF>
__device__ __forceinline__ void read16(v4i& d, unsigned addr) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF));
}
template <int N>
__device__ __forceinline__ void wait_lds(VFrag& f) {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(f.q0), "+v"(f.q1) : "n"(N));
}
template <int N>
__device__ __forceinline__ void wait_lds(v4i& d) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(d) : "n"(N));
}

// One wavefront's part of a step's inputs: signs at s_off, V of its classes at v_off (class 0 of the chunk + the wavefront's
// share), U at u_off.  (A load's constant offset counts in memory and in LDS: v_lane and u_lane have it taken off.)
template <int RT>
__device__ __forceinline__ void load_step(__amdgpu_buffer_rsrc_t rsrc, unsigned char* mine, unsigned s_lane, unsigned v_lane,
                                          unsigned u_lane, unsigned s_off, unsigned v_off, unsigned u_off) {
    typedef StepLayout<RT> L;
    load_to_lds<0>(rsrc, mine, s_lane, s_off);
    load_to_lds<L::kVOffset>(rsrc, mine, v_lane, v_off);
    load_to_lds<L::kVOffset + kVClassBytes>(rsrc, mine, v_lane, v_off);
    if constexpr (RT == 4) {
        load_to_lds<L::kUOffset>(rsrc, mine, u_lane, u_off);
    } else {   // (constant offsets reach 4095)
        static_assert(RT == 4 || RT == 2, "");
        load_to_lds<L::kVOffset + 2 * kVClassBytes>(rsrc, mine, v_lane, v_off);
        load_to_lds<0>(rsrc, mine + 4096, v_lane, v_off + 4096u);
        load_to_lds<L::kUOffset - 4096>(rsrc, mine + 4096, u_lane, u_off);
    }
}
template <int RT>
constexpr int kStepLoads = kClasses / RT + 2;
template <int RT>
__device__ __forceinline__ unsigned v_lane_offset(unsigned off_v, unsigned wave_of_team, unsigned lane) {
    return off_v + wave_of_team * unsigned(kClasses / RT * kVClassBytes) + v_piece_offset(lane) - unsigned(StepLayout<RT>::kVOffset);
}
template <int RT>
__device__ __forceinline__ unsigned u_lane_offset(unsigned off_u, unsigned row_tile, unsigned lane) {
    return off_u + (row_tile * kTileRows + (lane & 31)) * 32u + (lane >> 5) * 16u - unsigned(StepLayout<RT>::kUOffset % 4096);
}

// A operand of the accumulating product: output row i of a lane's group takes slot 0, 2, 1, 3 (the pairs hold
// bytes (0, 2) and (1, 3) of a word)
__device__ __forceinline__ v4h accumulate_matrix(unsigned lane) {
    const unsigned i = lane & 3, slot = i == 1 ? 2u : i == 2 ? 1u : i;
    v4h a;
#pragma unroll
    for (unsigned s = 0; s < 4; ++s) a[s] = _Float16(s == slot ? 1.0f : 0.0f);
    return a;
}

__device__ __forceinline__ unsigned signed_pair(float a, float b, unsigned bits) {
    v2h c;
    c[0] = _Float16(a);
    c[1] = _Float16(b);
    return __builtin_bit_cast(unsigned, c) ^ (~bits & 0x80008000u);   // a cleared bit marks a negative sign
}

__device__ __forceinline__ v16f zero16() {
    v16f z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.0f;
    return z;
}

// 1/s of the eight columns of byte E: addr = LDS byte address of the lane's half of a chunk's 256 scales
template <int E>
__device__ __forceinline__ void read_scales(v4f (&d)[2], unsigned addr) {
    asm volatile("ds_read_b128 %0, %2 offset:%3\n\tds_read_b128 %1, %2 offset:%4"
                 : "=&v"(d[0]), "=&v"(d[1])
                 : "v"(addr), "n"(E * 32), "n"(E * 32 + 16));
}
template <int N>
__device__ __forceinline__ void wait_scales(v4f (&d)[2]) {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(d[0]), "+v"(d[1]) : "n"(N));
}
// fp16 pair (a ra, b rb), product and conversion in one instruction each
__device__ __forceinline__ int scaled_pair(float a, float b, float ra, float rb) {
    int d;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(d) : "v"(a), "v"(ra));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(d) : "v"(b), "v"(rb));
    return d;
}

// acc[t][w][b]: column 128 g + 32 w + 8 b + t of row lane % 32, g = lane / 32
typedef v4f UnitAcc[kClasses][4];

// What one step hands to the next: its inputs come from LDS, and the first reads and the first magnitude product of a
// step are issued inside the step before, so that no step starts with an empty pipeline.
struct StepInputs {
    v4i u;          // U: row lane % 32, ranks 8 (lane / 32) on
    v2u s[2];       // sign words
    VFrag f;        // fragment of class 6
    v16f m;         // magnitudes of class 7
};

__device__ __forceinline__ v16f magnitude(const VFrag& f, const v4i& u) {
    struct {
        v2u a, b;
    } both = {f.q0, f.q1};
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, both), __builtin_bit_cast(v8h, u), zero16(), 0, 0, 0);
}

// wait for all of a step's first reads; nothing that is still under way crosses a loop's back edge, where the compiler
// may move values between registers
__device__ __forceinline__ void wait_inputs(StepInputs& in, VFrag& f7, v4i& signs) {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(in.u), "+v"(in.f.q0), "+v"(in.f.q1), "+v"(f7.q0), "+v"(f7.q1), "+v"(signs));
    in.m = magnitude(f7, in.u);
    // (a real copy: merged with the registers the reads fill, it would have to be made before they are filled)
    const v2u lo = {unsigned(signs[0]), unsigned(signs[1])}, hi = {unsigned(signs[2]), unsigned(signs[3])};
    asm("v_mov_b64 %0, %1" : "=v"(in.s[0]) : "v"(lo));
    asm("v_mov_b64 %0, %1" : "=v"(in.s[1]) : "v"(hi));
}

// The first reads of a step that no step precedes: requested by begin_reads, taken over by wait_inputs.  vaddr: LDS byte
// address of its V panel + v_read_offset; saddr: of the lane's 16 bytes of signs (its 16 bytes of U are kUOffset further on)
struct FirstReads {
    VFrag f7;
    v4i signs;
};
template <int RT>
__device__ __forceinline__ void begin_reads(StepInputs& in, FirstReads& r, unsigned vaddr, unsigned saddr) {
    read_frag<7, RT>(r.f7, vaddr);
    read16<StepLayout<RT>::kUOffset>(in.u, saddr);
    read16<0>(r.signs, saddr);
    read_frag<6, RT>(in.f, vaddr);
}

// One block onto the wavefront's unit.  vnext, snext: addresses of the next step.  FIRST: the accumulators start
// from zero.  A SIMD issues one vector or matrix instruction per four cycles, and with two wavefronts to it a
// wavefront issues one instruction of any kind per eight: what counts is the number of instructions.
template <bool FIRST, int RT>
__device__ __forceinline__ void add_block(UnitAcc& acc, StepInputs& in, unsigned vaddr, unsigned vnext, unsigned snext, v4h ident) {
    typedef unsigned long long u64;
    // per pair of words, for the class at hand: bytes 1, 3 (hi) and 0, 2 (lo) of each word at its bits 15, 31
    u64 hi[2], lo[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        hi[k] = __builtin_bit_cast(u64, in.s[k]);
        asm("v_lshlrev_b64 %0, 8, %1" : "=v"(lo[k]) : "v"(hi[k]));
    }
    auto apply = [&](v4f (&a)[4], const v16f& mg, bool more) __attribute__((always_inline)) {
        v2u p[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int sh = (w & 1) * 32;
            p[w][0] = signed_pair(mg[4 * w], mg[4 * w + 2], unsigned(lo[w >> 1] >> sh));
            p[w][1] = signed_pair(mg[4 * w + 1], mg[4 * w + 3], unsigned(hi[w >> 1] >> sh));
        }
        __builtin_amdgcn_sched_barrier(0);   // (products behind all of this: no wait states between a pair and its product)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const v4f z = {0.0f, 0.0f, 0.0f, 0.0f};
            a[w] = __builtin_amdgcn_mfma_f32_4x4x4f16(ident, __builtin_bit_cast(v4h, p[w]), FIRST ? z : a[w], 0, 0, 0);
        }
        if (more) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                u64 h = hi[k], l = lo[k];
                asm("v_lshl_add_u64 %0, %0, 1, 0" : "+v"(h));
                asm("v_lshl_add_u64 %0, %0, 1, 0" : "+v"(l));
                hi[k] = h;
                lo[k] = l;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // the magnitudes of the next class are under way while this one's signs are applied, its fragment was requested one
    // class earlier still
    VFrag f;
    v16f n;
#define BS_CLASS(T, CUR, NXT, F0, F1)                     \
    {                                                     \
        read_frag<T - 2, RT>(F0, vaddr);                  \
        wait_lds<2>(F1);                                  \
        NXT = magnitude(F1, in.u);                        \
        __builtin_amdgcn_sched_barrier(0);                \
        apply(acc[T], CUR, true);                         \
    }
    read_frag<5, RT>(f, vaddr);
    n = magnitude(in.f, in.u);
    __builtin_amdgcn_sched_barrier(0);
    apply(acc[7], in.m, true);
    BS_CLASS(6, n, in.m, in.f, f)
    BS_CLASS(5, in.m, n, f, in.f)
    BS_CLASS(4, n, in.m, in.f, f)
    BS_CLASS(3, in.m, n, f, in.f)
    BS_CLASS(2, n, in.m, in.f, f)
#undef BS_CLASS
    wait_lds<0>(in.f);
    n = magnitude(in.f, in.u);
    __builtin_amdgcn_sched_barrier(0);
    apply(acc[1], in.m, true);
    v4i signs;
    read_frag<7, RT>(f, vnext);
    read16<StepLayout<RT>::kUOffset>(in.u, snext);
    read16<0>(signs, snext);
    read_frag<6, RT>(in.f, vnext);
    apply(acc[0], n, false);
    wait_inputs(in, f, signs);
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace bitstack
