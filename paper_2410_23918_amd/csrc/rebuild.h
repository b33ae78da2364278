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
//   * sign and sum: s_i W_i = s_i W_{i-1} + M_i with M_i the magnitudes and s_i s_i = 1, so the accumulator holds s_i times the sum.
//     Before a block's product its sign bits are flipped where s_i and s_{i-1} differ, and the product adds M_i to it as its third
//     operand: one vector instruction per element and block, no conversion, fp32 throughout.  A flip is an exclusive-or of the
//     register's top byte with a byte of a copy of the word in which the class's bits stand at bit 7 of the bytes and the others are
//     cleared (v_xor_b32_sdwa); the copy moves up by one bit per class, two words per instruction (v_lshl_add_u64: the bit that
//     crosses from one word into the other stays below bit 7).  After the last block s_n is taken off.
// Registers only, that is 48 ns per 32 x 32 tile, block and SIMD, bound by the issue of vector instructions (22 per tile, most of them
// four cycles; the matrix product takes one slot more).  Rounding the signed magnitudes to fp16 pairs, flipping two signs at
// a time and summing by v_mfma_f32_4x4x4_16b_f16 takes as many slots, 50 ns, but 24 registers more; a shift per pair and two 32x32x16
// identity products 77.
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
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

constexpr int kClasses = 8;                 // column classes of a unit (bit positions in a byte)
constexpr int kVClassBytes = 1024;          // V of one class: 2 halves x 16 ranks x 16 columns fp16
constexpr int kVChunkBytes = kClasses * kVClassBytes;

// The RT wavefronts (4, 2 or 1 row tiles) that work on the same column chunk share its V panel; each loads its own signs and U
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

// the same for inputs that no other wavefront reads: no barrier
template <int N>
__device__ __forceinline__ void loads_wait() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
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
    static_assert(RT == 4 || RT == 2 || RT == 1, "");
    static_assert(L::kVOffset == 1024 && L::kUOffset == (RT == 4 ? 3072 : RT == 2 ? 4096 + 1024 : 8192 + 1024), "");
    if constexpr (RT == 4)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
                     "buffer_load_dwordx4 %1, %4, %5 offen lds\n\t"
                     "buffer_load_dwordx4 %2, %4, %6 offen offset:1024 lds\n\t"
                     "buffer_load_dwordx4 %2, %4, %6 offen offset:2048 lds\n\t"
                     "buffer_load_dwordx4 %3, %4, %7 offen offset:3072 lds" ::"s"(mine),
                     "v"(s_lane), "v"(v_lane), "v"(u_lane), "s"(rsrc), "s"(s_off), "s"(v_off), "s"(u_off)
                     : "memory", "m0");
    else if constexpr (RT == 1)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
                     "buffer_load_dwordx4 %3, %6, %7 offen lds\n\t"
                     "buffer_load_dwordx4 %4, %6, %8 offen offset:1024 lds\n\t"
                     "buffer_load_dwordx4 %4, %6, %8 offen offset:2048 lds\n\t"
                     "buffer_load_dwordx4 %4, %6, %8 offen offset:3072 lds\n\t"
                     "s_mov_b32 m0, %1\n\ts_nop 0\n\t"
                     "buffer_load_dwordx4 %4, %6, %9 offen lds\n\t"
                     "buffer_load_dwordx4 %4, %6, %9 offen offset:1024 lds\n\t"
                     "buffer_load_dwordx4 %4, %6, %9 offen offset:2048 lds\n\t"
                     "buffer_load_dwordx4 %4, %6, %9 offen offset:3072 lds\n\t"
                     "s_mov_b32 m0, %2\n\ts_nop 0\n\t"
                     "buffer_load_dwordx4 %4, %6, %10 offen lds\n\t"
                     "buffer_load_dwordx4 %5, %6, %11 offen offset:1024 lds" ::"s"(mine),
                     "s"(mine + 4096u), "s"(mine + 8192u), "v"(s_lane), "v"(v_lane), "v"(u_lane), "s"(rsrc), "s"(s_off), "s"(v_off), "s"(v_off + 4096u),
                     "s"(v_off + 8192u), "s"(u_off)
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

// acc[t][4 w + b]: column 128 g + 32 w + 8 b + t of row lane % 32, g = lane / 32; between blocks times the sign of the block
// added last (finish_unit takes it off)
typedef v16f UnitAcc[kClasses];

// Sign words of a lane: 128 columns of its row
struct SignWords {
    v2u w[2];
};

// What one step hands to the next: its inputs come from LDS, and the first reads of a step are issued inside the step
// before, so that no step starts with an empty pipeline.
struct StepInputs {
    v4i u;             // U: row lane % 32, ranks 8 (lane / 32) on
    SignWords s;       // signs of the step's block
    SignWords last;    // signs of the block before it
    VFrag f7, f6;      // fragments of the first two classes
};

__device__ __forceinline__ v16f magnitude(const VFrag& f, const v4i& u, const v16f& c) {
    struct {
        v2u a, b;
    } both = {f.q0, f.q1};
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, both), __builtin_bit_cast(v8h, u), c, 0, 0, 0);
}

// The first reads of a step.  vaddr: LDS byte address of its V panel + v_read_offset; saddr: of the lane's 16 bytes of signs (its
// 16 bytes of U are kUOffset further on)
template <int RT>
__device__ __forceinline__ void begin_reads(StepInputs& in, unsigned vaddr, unsigned saddr) {
    in.f7 = read_frag<7, RT>(vaddr);
    in.u = read_lds<v4i>(saddr + StepLayout<RT>::kUOffset);
    const v4i signs = read_lds<v4i>(saddr);
    in.f6 = read_frag<6, RT>(vaddr);
    in.s.w[0] = v2u{unsigned(signs[0]), unsigned(signs[1])};
    in.s.w[1] = v2u{unsigned(signs[2]), unsigned(signs[3])};
}

// a's sign bit flipped where bit 7 of byte B of m is set (B < 3: the other bits of the byte are clear): the top byte of the
// register, exclusive-or with that byte; byte 3 is where it has to be already (a three-input operation with vector operands
// takes two thirds of the time).  The compiler does not know that these are vector instructions: whoever uses them keeps them
// sixteen instructions from a matrix product that writes a and two from one that reads it (tests/test_asm_distances.py searches the
// compiled kernels for one that is too close).
template <int B>
__device__ __forceinline__ float flip_sign(float a, unsigned m, unsigned top_bit) {
    static_assert(B >= 0 && B < 4, "");
    if constexpr (B == 0)
        asm("v_xor_b32_sdwa %0, %0, %1 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_0" : "+v"(a) : "v"(m));
    else if constexpr (B == 1)
        asm("v_xor_b32_sdwa %0, %0, %1 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_1" : "+v"(a) : "v"(m));
    else if constexpr (B == 2)
        asm("v_xor_b32_sdwa %0, %0, %1 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_2" : "+v"(a) : "v"(m));
    else
        asm("v_bitop3_b32 %0, %0, %1, %2 bitop3:0x78" : "+v"(a) : "v"(m), "v"(top_bit));   // a ^ (m & top_bit)
    return a;
}

// The sixteen values of the class whose bits stand at bit 7 of the bytes of d
struct FlipMasks {
    unsigned w[4];
};
__device__ __forceinline__ FlipMasks flip_masks(const SignWords& d) {
    return FlipMasks{{d.w[0][0] & 0x80808080u, d.w[0][1] & 0x80808080u, d.w[1][0] & 0x80808080u, d.w[1][1] & 0x80808080u}};
}
__device__ __forceinline__ void flip_class(v16f& a, const FlipMasks& m) {
    unsigned top = 0x80000000u;
    asm("" : "+v"(top));   // a vector register
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        a[4 * w + 0] = flip_sign<0>(a[4 * w + 0], m.w[w], top);
        a[4 * w + 1] = flip_sign<1>(a[4 * w + 1], m.w[w], top);
        a[4 * w + 2] = flip_sign<2>(a[4 * w + 2], m.w[w], top);
        a[4 * w + 3] = flip_sign<3>(a[4 * w + 3], m.w[w], top);
    }
}
// the next lower class to bit 7 (the bit that crosses from one word into the other stays below it)
__device__ __forceinline__ void next_class(SignWords& d) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        unsigned long long v = __builtin_bit_cast(unsigned long long, d.w[k]);
        asm("v_lshl_add_u64 %0, %0, 1, 0" : "+v"(v));
        d.w[k] = __builtin_bit_cast(v2u, v);
    }
}

// One block onto the wavefront's unit.  vnext, snext: addresses of the next step (AHEAD: its first reads are issued here).  FIRST: the
// accumulators start from zero.  A SIMD issues one vector or matrix instruction per four cycles: what counts is the number of instructions, 22
// vector ones and a product per class.
template <bool FIRST, int RT, bool AHEAD = true>
__device__ __forceinline__ void add_block(UnitAcc& acc, StepInputs& in, unsigned vaddr, unsigned vnext, unsigned snext) {
    SignWords d;
#pragma unroll
    for (int k = 0; k < 2; ++k) d.w[k] = in.s.w[k] ^ in.last.w[k];
    in.last = in.s;
    const v4i u = in.u;
    // a class's fragment is requested two classes ahead; its product is issued after the signs of the next class have been
    // made ready, six instructions after its last flip
    VFrag f[kClasses];
    f[7] = in.f7;
    f[6] = in.f6;
    if constexpr (FIRST) {   // nothing but products: all fragments at once (two classes ahead is less than an LDS read takes then)
        f[5] = read_frag<5, RT>(vaddr);
        f[4] = read_frag<4, RT>(vaddr);
        f[3] = read_frag<3, RT>(vaddr);
        f[2] = read_frag<2, RT>(vaddr);
        f[1] = read_frag<1, RT>(vaddr);
        f[0] = read_frag<0, RT>(vaddr);
        __builtin_amdgcn_sched_barrier(0);
    }
#define BS_CLASS(T)                                                                        \
    {                                                                                      \
        if constexpr (T >= 2 && !FIRST) f[T >= 2 ? T - 2 : 0] = read_frag<(T >= 2 ? T - 2 : 0), RT>(vaddr); \
        if constexpr (T < 2) {                                                             \
            if constexpr (T == 1 && AHEAD) begin_reads<RT>(in, vnext, snext);              \
        }                                                                                  \
        if constexpr (FIRST) {                                                             \
            acc[T] = magnitude(f[T], u, zero16());                                         \
        } else {                                                                           \
            const FlipMasks m = flip_masks(d);                                             \
            if constexpr (T > 0) next_class(d);                                            \
            __builtin_amdgcn_sched_barrier(0);                                             \
            if constexpr (T < 7) acc[T < 7 ? T + 1 : 7] = magnitude(f[T < 7 ? T + 1 : 7], u, acc[T < 7 ? T + 1 : 7]); \
            flip_class(acc[T], m);                                                         \
        }                                                                                  \
        __builtin_amdgcn_sched_barrier(0);                                                 \
    }
    BS_CLASS(7)
    BS_CLASS(6)
    BS_CLASS(5)
    BS_CLASS(4)
    BS_CLASS(3)
    BS_CLASS(2)
    BS_CLASS(1)
    BS_CLASS(0)
#undef BS_CLASS
    if constexpr (!FIRST) {
        asm volatile("s_nop 3");
        __builtin_amdgcn_sched_barrier(0);
        acc[0] = magnitude(f[0], u, acc[0]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// After the last block: the sign of that block off the sums
__device__ __forceinline__ void finish_unit(UnitAcc& acc, const StepInputs& in) {
    SignWords d;
#pragma unroll
    for (int k = 0; k < 2; ++k) d.w[k] = ~in.last.w[k];   // a cleared bit marks a negative sign
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = kClasses - 1; t >= 0; --t) {
        const FlipMasks m = flip_masks(d);
        if (t > 0) next_class(d);
        flip_class(acc[t], m);
        __builtin_amdgcn_sched_barrier(0);
    }
}

}  // namespace bitstack
