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

// LDS by its byte address
template <class T>
__device__ __forceinline__ T read_lds(unsigned addr) {
    return *reinterpret_cast<const __attribute__((address_space(3))) T*>(addr);
}
template <class T>
__device__ __forceinline__ void write_lds(unsigned addr, T v) {
    *reinterpret_cast<__attribute__((address_space(3))) T*>(addr) = v;
}
// What the lanes of a wavefront wrote before is what they read after, lane to lane: LDS operations of a wavefront execute in
// order, so this only keeps the compiler from reordering them
__device__ __forceinline__ void wavefront_lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); }
__device__ __forceinline__ unsigned lds_address(const void* p) {
    return unsigned(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void*)p));
}

// Loads to LDS are asynchronous and several steps ahead of the reads of what they bring.  They are inline assembly because
// the compiler knows of its own ones only that they write LDS somewhere, and waits for all of them at every LDS read.
// They write no register, so nothing of theirs can be taken for ready before it is: the reads are ordinary loads, whose
// waits the compiler places, and no read passes loads_barrier() or a request ("memory").  The other way round -- reads
// in assembly with a wait further down -- left it to chance that the compiler neither spilled nor copied a register between.
//
// All but the last N vector memory operations of this wavefront are complete, and its LDS reads; then the workgroup's
// barrier.  (The fences of lds_barrier() in kparams.h are the compiler's: they do not know of these loads.)
template <int N>
__device__ __forceinline__ void loads_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// raw buffer descriptor
__device__ __forceinline__ v4i buffer_over(const void* p, unsigned bytes) {
    const unsigned long long a = reinterpret_cast<uintptr_t>(p);
    return v4i{int(unsigned(a)), int(unsigned(a >> 32)), int(bytes), 0x00020000};
}

// 16 (4) bytes per lane from the buffer to LDS at the wavefront's byte address lds, lane after lane (counted by vmcnt).
// s_nop 4: a memory instruction reads a scalar register five wait states after a vector instruction has written it at the
// earliest, and M0 one after the scalar unit has; the compiler does not look into assembly for either.
__device__ __forceinline__ void load_to_lds(v4i rsrc, unsigned lds, unsigned lane_off, unsigned soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(lane_off), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
}
__device__ __forceinline__ void load4_to_lds(v4i rsrc, unsigned lds, unsigned lane_off, unsigned soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(lds), "v"(lane_off), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
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

// A operand of the magnitude product of class T: two transposing reads
struct VFrag {
    v2u q0, q1;
};
__device__ __forceinline__ v2u read_lds_turned(unsigned addr) {
    typedef __fp16 v4f16 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(v2u, __builtin_amdgcn_ds_read_tr16_b64_v4f16(reinterpret_cast<__attribute__((address_space(3))) v4f16*>(addr)));
}
template <int T, int RT>
__device__ __forceinline__ VFrag read_frag(unsigned addr) {
    constexpr unsigned off = StepLayout<RT>::frag(T);
    return VFrag{read_lds_turned(addr + off), read_lds_turned(addr + off + 512)};
}

// One wavefront's part of a step's inputs, to its LDS byte address mine: signs at s_off, V of its classes at v_off (class 0 of
// the chunk + the wavefront's share), U at u_off.  (A load's constant offset, at most 4095, counts in memory and in LDS: v_lane
// and u_lane have it taken off.)
template <int RT>
__device__ __forceinline__ void load_step(v4i rsrc, unsigned mine, unsigned s_lane, unsigned v_lane, unsigned u_lane, unsigned s_off,
                                          unsigned v_off, unsigned u_off) {
    typedef StepLayout<RT> L;
    static_assert(RT == 4 || RT == 2, "");
    static_assert(L::kVOffset == 1024 && L::kUOffset == (RT == 4 ? 3072 : 4096 + 1024), "");
    if constexpr (RT == 4)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
                     "buffer_load_dwordx4 %1, %4, %5 offen lds\n\t"
                     "buffer_load_dwordx4 %2, %4, %6 offen offset:1024 lds\n\t"
                     "buffer_load_dwordx4 %2, %4, %6 offen offset:2048 lds\n\t"
                     "buffer_load_dwordx4 %3, %4, %7 offen offset:3072 lds" ::"s"(mine),
                     "v"(s_lane), "v"(v_lane), "v"(u_lane), "s"(rsrc), "s"(s_off), "s"(v_off), "s"(u_off)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
                     "buffer_load_dwordx4 %2, %5, %6 offen lds\n\t"
                     "buffer_load_dwordx4 %3, %5, %7 offen offset:1024 lds\n\t"
                     "buffer_load_dwordx4 %3, %5, %7 offen offset:2048 lds\n\t"
                     "buffer_load_dwordx4 %3, %5, %7 offen offset:3072 lds\n\t"
                     "s_mov_b32 m0, %1\n\ts_nop 0\n\t"
                     "buffer_load_dwordx4 %3, %5, %8 offen lds\n\t"
                     "buffer_load_dwordx4 %4, %5, %9 offen offset:1024 lds" ::"s"(mine),
                     "s"(mine + 4096u), "v"(s_lane), "v"(v_lane), "v"(u_lane), "s"(rsrc), "s"(s_off), "s"(v_off), "s"(v_off + 4096u), "s"(u_off)
                     : "memory", "m0");
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

// 1/s of the eight columns of byte e: addr = LDS byte address of the lane's half of a chunk's 256 scales
__device__ __forceinline__ void read_scales(v4f (&d)[2], unsigned addr, int e) {
    d[0] = read_lds<v4f>(addr + unsigned(e) * 32u);
    d[1] = read_lds<v4f>(addr + unsigned(e) * 32u + 16u);
}
// fp16 pair (a ra, b rb)
__device__ __forceinline__ int scaled_pair(float a, float b, float ra, float rb) {
    v2h c;
    c[0] = _Float16(__builtin_fmaf(a, ra, 0.0f));
    c[1] = _Float16(__builtin_fmaf(b, rb, 0.0f));
    return __builtin_bit_cast(int, c);
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

// The first reads of a step that no step precedes.  vaddr: LDS byte address of its V panel + v_read_offset; saddr: of the
// lane's 16 bytes of signs (its 16 bytes of U are kUOffset further on)
struct FirstReads {
    VFrag f7;
    v4i signs;
};
template <int RT>
__device__ __forceinline__ void begin_reads(StepInputs& in, FirstReads& r, unsigned vaddr, unsigned saddr) {
    r.f7 = read_frag<7, RT>(vaddr);
    in.u = read_lds<v4i>(saddr + StepLayout<RT>::kUOffset);
    r.signs = read_lds<v4i>(saddr);
    in.f = read_frag<6, RT>(vaddr);
}
// the first magnitude product from them
__device__ __forceinline__ void take_reads(StepInputs& in, const FirstReads& r) {
    in.m = magnitude(r.f7, in.u);
    in.s[0] = v2u{unsigned(r.signs[0]), unsigned(r.signs[1])};
    in.s[1] = v2u{unsigned(r.signs[2]), unsigned(r.signs[3])};
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
        F0 = read_frag<T - 2, RT>(vaddr);                 \
        NXT = magnitude(F1, in.u);                        \
        __builtin_amdgcn_sched_barrier(0);                \
        apply(acc[T], CUR, true);                         \
    }
    f = read_frag<5, RT>(vaddr);
    n = magnitude(in.f, in.u);
    __builtin_amdgcn_sched_barrier(0);
    apply(acc[7], in.m, true);
    BS_CLASS(6, n, in.m, in.f, f)
    BS_CLASS(5, in.m, n, f, in.f)
    BS_CLASS(4, n, in.m, in.f, f)
    BS_CLASS(3, in.m, n, f, in.f)
    BS_CLASS(2, n, in.m, in.f, f)
#undef BS_CLASS
    n = magnitude(in.f, in.u);
    __builtin_amdgcn_sched_barrier(0);
    apply(acc[1], in.m, true);
    FirstReads next;
    begin_reads<RT>(in, next, vnext, snext);
    __builtin_amdgcn_sched_barrier(0);
    apply(acc[0], n, false);
    take_reads(in, next);
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace bitstack
