// Pieces shared by the matrix-core products over packed weights (fp16 activations): vector types, the
// 32x32x16 instruction, and the unpacking of 8 codes into its weight operand.
#ifndef FQ_MFMA_H
#define FQ_MFMA_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#define FQ_GLOBAL __attribute__((address_space(1)))
#define FQ_LDS __attribute__((address_space(3)))

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// (a + b) * s, each operation rounded to half; a + b is the exact integer q - z
__device__ __forceinline__ uint32_t deq(uint32_t a, uint32_t b, half2_t s)
{
    return __builtin_bit_cast(uint32_t, (__builtin_bit_cast(half2_t, a) + __builtin_bit_cast(half2_t, b)) * s);
}

__device__ __forceinline__ float16_t mfma32(const u32x4 a, const uint32_t (&b)[4], float16_t c)
{
    const u32x4 bv = {b[0], b[1], b[2], b[3]};
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, a),
                                                  __builtin_bit_cast(half8_t, bv), c, 0, 0, 0);
}

// A quantization group's scale (rounded to half, for both halves of a register) and the constants
// -(offset + z) of the unpacking for one weight row.
struct DeqConst {
    half2_t s;
    uint32_t nz, nz2;
};

// Masks and exponents of the unpacking.  `pin` hides their values: (v & mask) | magic is one instruction
// only with both in registers (two 32-bit literals do not fit one; the mask may be scalar).
template <int BITS>
struct DeqMagic {
    uint32_t m0 = BITS == 2 ? 0x000C0003u : 0x00F0000Fu, m1 = 0x00C00030u;
    uint32_t e0 = BITS == 2 ? 0x5C006400u : BITS == 4 ? 0x54006400u : 0x64646464u, e1 = 0x4C005400u;
    __device__ __forceinline__ void pin()
    {
        if (BITS == 2)
            asm volatile("" : "+s"(m0), "+s"(m1), "+v"(e0), "+v"(e1));
        if (BITS == 4)
            asm volatile("" : "+s"(m0), "+v"(e0));
    }
};

template <int BITS>
__device__ __forceinline__ DeqConst deq_const(float s, uint32_t z)
{
    DeqConst c;
    c.s = half2_t{(_Float16)s, (_Float16)s};
    c.nz = BITS == 8 ? ((z | (z << 16)) | 0xE400E400u)               // -(1024 + z) twice
         : BITS == 4 ? ((z | 0xE400u) | (((z << 4) | 0xD400u) << 16)) // -(1024 + z), -(64 + z)
                     : ((z | 0xE400u) | (((z << 2) | 0xDC00u) << 16)); // -(1024 + z), -(256 + z)
    c.nz2 = ((z << 4) | 0xD400u) | (((z << 6) | 0xCC00u) << 16);     // 2 bits: -(64 + z), -(16 + z)
    return c;
}

// 8 consecutive codes of a row -> the weight operand half((q - z) * half(s)), in their own order.
// 2 bits: the 16 low (i even) or high (i odd) bits of v; 4 bits: the word v; 8 bits: the words v, v2.
template <int BITS>
__device__ __forceinline__ void deq8(uint32_t v, uint32_t v2, int i, const DeqConst &c, const DeqMagic<BITS> &mg, uint32_t (&b)[4])
{
    if (BITS == 2) {
        // fields q0 .. q7, byte t holds q(4t) .. q(4t+3).  The byte is copied under both halves; fields
        // 0 and 1 (or 2 and 3) of it stay where they are, one per half, each under the exponent that
        // makes it offset + q
        const uint32_t lo = __builtin_amdgcn_perm(0u, v, (i & 1) ? 0x0c020c02u : 0x0c000c00u);
        const uint32_t hi = __builtin_amdgcn_perm(0u, v, (i & 1) ? 0x0c030c03u : 0x0c010c01u);
        b[0] = deq((lo & mg.m0) | mg.e0, c.nz, c.s);  // q0, q1
        b[1] = deq((lo & mg.m1) | mg.e1, c.nz2, c.s); // q2, q3
        b[2] = deq((hi & mg.m0) | mg.e0, c.nz, c.s);  // q4, q5
        b[3] = deq((hi & mg.m1) | mg.e1, c.nz2, c.s); // q6, q7
    } else if (BITS == 4) {
        // byte t holds (q(2t+1) q(2t)): copied under both halves, the low nibble kept in the low half
        // (exponent 0x64: 1024 + q) and the high nibble in the high half (0x54: 64 + q)
        b[0] = deq((__builtin_amdgcn_perm(0u, v, 0x0c000c00u) & mg.m0) | mg.e0, c.nz, c.s);
        b[1] = deq((__builtin_amdgcn_perm(0u, v, 0x0c010c01u) & mg.m0) | mg.e0, c.nz, c.s);
        b[2] = deq((__builtin_amdgcn_perm(0u, v, 0x0c020c02u) & mg.m0) | mg.e0, c.nz, c.s);
        b[3] = deq((__builtin_amdgcn_perm(0u, v, 0x0c030c03u) & mg.m0) | mg.e0, c.nz, c.s);
    } else {
        b[0] = deq(__builtin_amdgcn_perm(mg.e0, v, 0x04010400u), c.nz, c.s);
        b[1] = deq(__builtin_amdgcn_perm(mg.e0, v, 0x04030402u), c.nz, c.s);
        b[2] = deq(__builtin_amdgcn_perm(mg.e0, v2, 0x04010400u), c.nz, c.s);
        b[3] = deq(__builtin_amdgcn_perm(mg.e0, v2, 0x04030402u), c.nz, c.s);
    }
}

// Direct-to-LDS loads go through buffer instructions: a lane's address is a descriptor (scalar) plus a
// 32-bit offset of its own plus a scalar one, so a request costs no address arithmetic; and the reads
// of LDS between them keep counted waits.  Issued as global_load_lds the compiler took them for accesses
// that may retire among the LDS reads and put lgkmcnt(0) -- every read in flight -- before each use of
// one.  Same kernels otherwise: 2048 x 8192 x 28672 at 4 bits 894 -> 855 us, 515 x 4096 x 11008 at 8 bits
// 90 -> 82 us, W8A8 300 x 13824 x 5120 184 -> 176 us, with one scale per row 2048 x 28672 x 8192 523 -> 508 us.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00027000);
}

template <int SIZE>
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, void *lds, uint32_t lane_off, uint32_t off)
{
    static_assert(SIZE == 16 || SIZE == 4 || SIZE == 1, "bytes per lane"); // (the builtin wants a plain literal)
    if constexpr (SIZE == 16)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (FQ_LDS void *)lds, 16, (int)lane_off, (int)off, 0, 0);
    else if constexpr (SIZE == 4)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (FQ_LDS void *)lds, 4, (int)lane_off, (int)off, 0, 0);
    else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (FQ_LDS void *)lds, 1, (int)lane_off, (int)off, 0, 0);
}

// Byte offset of 16-byte piece `ch` of row `r` of a slab with RB bytes per row.  The pieces of a 256-byte line
// are permuted so that a read of one piece of 16 consecutive rows touches every bank once, rows 0 .. 7 in one half
// of the bank row and rows 8 .. 15 in the other.
template <int RB>
__device__ __forceinline__ int w_offset(int r, int ch)
{
    const int blk = r >> 4, q = r & 15;
    if (RB == 256)
        return r * 256 + ((ch ^ q) << 4);
    if (RB == 128)
        return blk * 2048 + (q & 7) * 256 + (((q >> 3) * 8 + (ch ^ (q & 7))) << 4);
    if (RB == 64)
        return blk * 1024 + ((q >> 1) & 3) * 256 + ((((q >> 3) * 2 + (q & 1)) * 4 + (ch ^ ((q >> 1) & 3))) << 4);
    return (r >> 3) * 256 + (((r & 7) * 2 + (ch ^ ((r >> 3) & 1))) << 4); // 32
}

// The inverse: the row and the byte inside the row that lane `lane` of the load fetches that fills bytes ld * 1024
// .. + 1023 of the slab, 16 per lane.
template <int RB>
__device__ __forceinline__ void w_piece(int ld, int lane, int &row, int &byte)
{
    const int line = lane >> 4, slot = lane & 15;
    if (RB == 256) {
        row = ld * 4 + line;
        byte = (slot ^ (row & 15)) << 4;
    } else if (RB == 128) {
        const int l = (ld & 1) * 4 + line;
        row = (ld >> 1) * 16 + (slot >> 3) * 8 + l;
        byte = ((slot & 7) ^ l) << 4;
    } else if (RB == 64) {
        const int q = slot >> 2;
        row = ld * 16 + (q >> 1) * 8 + line * 2 + (q & 1);
        byte = ((slot & 3) ^ line) << 4;
    } else {
        const int l8 = ld * 4 + line;
        row = l8 * 8 + (slot >> 1);
        byte = ((slot & 1) ^ (l8 & 1)) << 4;
    }
}

#endif
