// Decode-phase weight-only quantized linear for small batches (2 <= M <= 32): single calls and plans of the
// size a decoder's stages have (q/k/v, o, gate/up, down of one layer; up to 64 entries), 2, 3, 4, 8 and 16 bits; y[M][N] =
// x[M][K] . dequant(W[N][K])^T, dequant = Sec. 2.2 Eq. (3).  Bound by the weight stream (Sec. 4.1) on paper; a launch of
// 10 to 90 MB lasts 8 to 25 us, so that its start, its end and an even division count as much.
//
// Work split.  One workgroup (8 wavefronts) per compute unit.  The launch's tiles of 16 weight rows are divided
// among them by cost (batch_tile_cost), a contiguous run each; every workgroup works the division out from the
// entries' shapes and the bit-widths it finds in device memory, one entry per lane.  Within a tile the wavefronts
// split K: wavefront w takes the 128-byte lines w, w + 8, ... of all 16 rows, so that a step of the workgroup reads
// 1 KiB of each row, and their sums meet in LDS at the end, added in the wavefronts' order.
//
// x sits in LDS, 128 KiB of it at a time (4096 inputs of 16 batch rows, 2048 of 32), brought by direct-to-LDS loads
// in slabs of 64 inputs whose 16-byte pieces are permuted (w_offset) so that operand reads are conflict free; projections of
// 4096 inputs are one panel, and entries that share x (q, k, v) do not fetch it again: then the sums of a run
// stay out of x's place.  Scales and zero points of the run's tiles are laid beside it.  Weights go straight to
// registers: lane (n, c) takes 16 bytes of each half line of row n, the operand layout of v_mfma_f32_16x16x32_f16 up to a permutation of the inputs that x
// shares, RD lines ahead.
//
// Measured (us a plan launch at 4 / 8 / 16 bits, cold weights; in brackets the register-fed kernel): 16 batch rows, 4096 x 4096
// 7.3 / 9.3 / 10.7 (9.1 / 11.3 / 14.0), 3 x 4096 x 4096 12.2 / 16.0 / 23.3, 4096 rows x 11008 14.3 / 19.5 / 26.3 (17.7 / 23.9 / 30.7),
// 2 x 11008 x 4096 16.8 / 23.3 / 39.0 (23.8 / 34.8 / 46.9); 32 batch rows 9.7 / 12.2 / 13.4, 19.5 / 24.5 / 31.7, 21.1 / 27.3 / 33.0,
// 22.4 / 29.0 / 42.2; the 7B-shaped layers at 16 rows, 4 and 8 bits, 512 for 32 launches.  Where the register-fed kernel is the faster
// one: fq_batch_serves below.  Why it is as it is:
//   - requests past a run's end ask beyond the buffer's end: as re-reads of the last line, 8 ahead, they made 4096 x 4096 cost
//     12 us (the loads' line accesses, not HBM, were the limit);
//   - two lines ahead are as fast as eight (19.6 against 23.8 us at 22016 rows), sixteen wavefronts the same as eight;
//   - scales and zero points of a run are requested together (a loop that stored each before it asked for the next made up to
//     six trips to memory), but no more of them than the run has tiles: six tiles' for every run cost runs of one 0.3 us a panel;
//   - the sums meet in one round (six tiles 1.0 us, two blocks at a time 1.9), the two at a time of a run that keeps x in rounds
//     fixed at compile time (as a run-time choice, plans of many short runs took up to 1.14 times as long);
//   - an x that all entries read is requested ahead of the table, and nothing where there is none (out of range it cost 1 us);
//   - 2 and 3 bits, register-fed kernel before and this one now (us a plan launch, 16 batch rows, {2, 4, 8} resident, all at 2 bits):
//     4096 x 4096 13.6 and 7.1, 3 x 4096 x 4096 14.3 and 11.8, 2 x 11008 x 4096 21.2 and 14.2, 4096 rows x 11008 33.9 and 13.2; {3, 4, 8}, all at 3: 9.2
//     and 7.7, 18.7 and 13.1, 26.7 and 17.1, 19.2 and 15.2;
//   - the division has no integer divisions: they were half of the 0.9 us between table and first request.
// What bounds it: launch, table and first request 4 us of a launch, instructions (137 vector ones per 4-bit line of 16 rows, 11 lines a
// wavefront at 22016 rows), three panels one after the other at K = 11008.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "fq_batch_at.h"
#include "fq_internal.h"
#include "fq_mfma.h"

namespace {

constexpr int THREADS = 512;
constexpr int WAVES = 8;
constexpr int XBYTES = BATCH_X_BYTES; // x of a panel
constexpr int NB = 6;              // tiles of 16 rows a workgroup takes at a time
constexpr int RD = 2;              // 128-byte lines of each row a wavefront has in flight
constexpr int MAX_ENTRIES = 64;

__device__ __forceinline__ float4_t mfma16(const u32x4 a, const uint32_t (&b)[4], float4_t c)
{
    const u32x4 bv = {b[0], b[1], b[2], b[3]};
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, bv), c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pk_add(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, a) + __builtin_bit_cast(half2_t, b));
}

// What a request brings of a row: a lane's 32 codes of a group at 2, 3 and 4 bits, 16 bytes at 8 and 16.
template <int BITS>
__device__ __forceinline__ u32x4 load_piece(__amdgpu_buffer_rsrc_t buf, uint32_t at)
{
    if constexpr (BITS == 2) {
        const u32x2 q = __builtin_amdgcn_raw_buffer_load_b64(buf, (int)at, 0, 0);
        return u32x4{q.x, q.y, 0, 0};
    } else if constexpr (BITS == 3) {
        const auto q = __builtin_amdgcn_raw_buffer_load_b96(buf, (int)at, 0, 0);
        return u32x4{(uint32_t)q[0], (uint32_t)q[1], (uint32_t)q[2], 0};
    } else {
        return __builtin_amdgcn_raw_buffer_load_b128(buf, (int)at, 0, 0);
    }
}

// A lane's 32 codes of a group -> q - z as four operands of eight halves, in the order of the inputs.
template <int BITS>
struct Unpack : DeqMagic<BITS> {
    __device__ __forceinline__ void group(const u32x4 &v, uint32_t z, uint32_t (&b)[4][4]) const
    {
        if constexpr (BITS == 4) {
            const uint32_t nz = (z | 0xE400u) | (((z << 4) | 0xD400u) << 16); // -(1024 + z), -(64 + z)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint32_t q = v[i];
                b[i][0] = pk_add((__builtin_amdgcn_perm(0u, q, 0x0c000c00u) & this->m0) | this->e0, nz);
                b[i][1] = pk_add((__builtin_amdgcn_perm(0u, q, 0x0c010c01u) & this->m0) | this->e0, nz);
                b[i][2] = pk_add((__builtin_amdgcn_perm(0u, q, 0x0c020c02u) & this->m0) | this->e0, nz);
                b[i][3] = pk_add((__builtin_amdgcn_perm(0u, q, 0x0c030c03u) & this->m0) | this->e0, nz);
            }
        } else if constexpr (BITS == 2) {
            // A byte holds four consecutive codes: copied under both halves, fields 0 and 1, then 2 and 3, stay where they are,
            // each under the exponent that makes it offset + q.
            const uint32_t nz = (z | 0xE400u) | (((z << 2) | 0xDC00u) << 16);         // -(1024 + z), -(256 + z)
            const uint32_t nz2 = ((z << 4) | 0xD400u) | (((z << 6) | 0xCC00u) << 16); // -(64 + z), -(16 + z)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint32_t q = v[i >> 1];
                const uint32_t lo = __builtin_amdgcn_perm(0u, q, (i & 1) ? 0x0c020c02u : 0x0c000c00u);
                const uint32_t hi = __builtin_amdgcn_perm(0u, q, (i & 1) ? 0x0c030c03u : 0x0c010c01u);
                b[i][0] = pk_add((lo & this->m0) | this->e0, nz);
                b[i][1] = pk_add((lo & this->m1) | this->e1, nz2);
                b[i][2] = pk_add((hi & this->m0) | this->e0, nz);
                b[i][3] = pk_add((hi & this->m1) | this->e1, nz2);
            }
        }
    }
};

// 3 bits: a word holds ten codes, five to a half from bit 0 on (code 5 h + p of them at bit 16 h + 3 p), and in bits 15 and 31
// one bit of the codes 30 and 31.  Pairs of consecutive codes are put together from either half copied under
// both, as it is and shifted by nine: a field at bits 0 / 3 / 6 of a half reads 1024 / 128 / 16 + q.
template <>
struct Unpack<3> {
    uint32_t ea, eb, ec, ed, ef, m1, m2, m3, m5;
    __device__ __forceinline__ void pin()
    {
        ea = 0x58006400u, eb = 0x64004C00u, ec = 0x64005800u, ed = 0x4C005800u, ef = 0x64006400u;
        m1 = 0x00380007u, m2 = 0x000001C0u, m3 = 0x00070000u, m5 = 0x01C00038u;
        asm volatile("" : "+v"(ea), "+v"(eb), "+v"(ec), "+v"(ed), "+v"(ef), "+s"(m1), "+s"(m2), "+s"(m3), "+s"(m5));
    }
    __device__ __forceinline__ void group(const u32x4 &v, uint32_t z, uint32_t (&b)[4][4]) const
    {
        const uint32_t z0 = z | 0xE400u, z3 = (z << 3) | 0xD800u, z6 = (z << 6) | 0xCC00u; // -(1024 + z), -(128 + z), -(16 + z)
        const uint32_t na = z0 | z3 << 16, nb = z6 | z0 << 16, nc = z3 | z0 << 16, nd = z3 | z6 << 16, nf = z0 | z0 << 16;
        uint32_t t[16];
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const uint32_t w = v[j];
            const uint32_t lo = __builtin_amdgcn_perm(0u, w, 0x01000100u), hi = __builtin_amdgcn_perm(0u, w, 0x03020302u);
            const uint32_t lo9 = lo >> 9, hi9 = hi >> 9;
            t[5 * j] = pk_add((lo & m1) | ea, na);                      // codes 0, 1 of the word
            t[5 * j + 1] = pk_add((lo9 & m3) | ((lo & m2) | eb), nb);   // 2, 3
            t[5 * j + 2] = pk_add((w & m3) | ((lo9 & 0x38u) | ec), nc); // 4, 5
            t[5 * j + 3] = pk_add((hi & m5) | ed, nd);                  // 6, 7
            t[5 * j + 4] = pk_add((hi9 & m1) | ea, na);                 // 8, 9
        }
        const uint32_t last = ((v[0] >> 15) & 0x00010001u) | ((v[1] >> 14) & 0x00020002u) | ((v[2] >> 13) & 0x00040004u);
        t[15] = pk_add(last | ef, nf);
#pragma unroll
        for (int i = 0; i < 16; i++)
            b[i >> 2][i & 3] = t[i];
    }
};

struct Lds {
    __attribute__((aligned(1024))) uint8_t x[XBYTES];
    float s[NB * 16 * 33];
    uint8_t z[NB * 16 * 33];
    float4_t red[2 * WAVES * 64];
};

// Inputs of a panel; its quantization groups; their stride in LDS.
template <int MB>
struct Panel {
    static constexpr int KP = batch_panel(MB), GP = KP / 128, GS = GP + 1;
};

// Up to NB consecutive tiles of an entry at its selected width.
struct Run {
    const uint8_t *codes, *zeros;
    const float *scales;
    const uint16_t *x;
    uint16_t *y;
    int bits, N, K, t0, nt;
};

// Panel 0 of x, before the launch's widths are known.  (Every workgroup reads this x: each
// starts somewhere else in it, or they would all ask the same L2 channel at the same time.)  Slabs past K repeat the
// row's last, so that the number of requests does not depend on it.
template <int MB>
__device__ __forceinline__ void fetch_first_x(Lds &L, const uint16_t *x, int K, int M)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const __amdgpu_buffer_rsrc_t xbuf = buffer_of(x, (uint32_t)M * (uint32_t)K * 2);
    // (request j fills KiB j of the panel; a wavefront's have j % 8 in common, and with it the rows and pieces they take)
    const int first = (int)((blockIdx.x >> 3) * 37u % 32u) / 2 * 8, last = K - 64;
    int r, byte;
    w_piece<128>(wave & 1, lane, r, byte);
    const int mb = MB == 2 ? (wave >> 1) & 1 : 0;
    const uint32_t at = (uint32_t)min(mb * 16 + r, M - 1) * (uint32_t)K * 2 + byte;
#pragma unroll
    for (int i = 0; i < XBYTES / 1024 / WAVES; i++) {
        const int j = (i * WAVES + first) % (XBYTES / 1024) + wave, k = j / (2 * MB) * 64;
        load_to_lds<16>(xbuf, L.x + j * 1024, at, (uint32_t)min(k, last) * 2);
    }
}

// The tiles [t0, t0 + nt) of one entry.
template <int BITS, int MB>
__device__ __forceinline__ void run_batch(Lds &L, const uint8_t *codes, const float *scales, const uint8_t *zeros,
                                          const uint16_t *x, uint16_t *y, int N, int K, int M, int t0, int nt, bool x_there,
                                          bool keep_x)
{
    constexpr int KP = batch_panel(MB);   // inputs of a panel: 4096 or 2048
    constexpr int GP = KP / 128, GS = GP + 1; // groups of a panel; their stride in LDS
    constexpr int KL = batch_line_inputs(BITS), LB = batch_line_bytes(BITS); // inputs and bytes of a line
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = lane & 15, c = lane >> 4;
    const uint32_t row_bytes = (uint32_t)K / 8 * BITS;
    const int G = K >> 7;
    const int n0 = t0 * 16;
    float4_t sum[NB][MB];
#pragma unroll
    for (int t = 0; t < NB; t++)
#pragma unroll
        for (int mb = 0; mb < MB; mb++)
            sum[t][mb] = float4_t{0.f, 0.f, 0.f, 0.f};
    const __amdgpu_buffer_rsrc_t xbuf = buffer_of(x, (uint32_t)M * (uint32_t)K * 2);
    const __amdgpu_buffer_rsrc_t wbuf = buffer_of(codes + (size_t)n0 * row_bytes, batch_run_bytes(row_bytes, nt, N - n0));
    const uint32_t lane_off = batch_lane_offset(row_bytes, n, c, LB);
    // x operand reads: piece p of batch row n in a slab of 64 inputs
    uint32_t xat[8];
#pragma unroll
    for (int i = 0; i < 8; i++)
        xat[i] = BITS <= 4   ? (uint32_t)((c >> 1) * 2048 * MB + w_offset<128>(n, 4 * (c & 1) + (i & 3)))
                 : BITS == 8 ? (uint32_t)w_offset<128>(n, 2 * c + (i & 1))
                             : (uint32_t)w_offset<128>(n, 4 * (i & 1) + c);
    Unpack<BITS> mg;
    mg.pin();

    for (int k0 = 0; k0 < K; k0 += KP) {
        const int kp = min(KP, K - k0), gp = kp >> 7, g0 = k0 >> 7;
        if (k0 > 0 || !x_there) {
            if (k0 > 0)
                __syncthreads(); // every wavefront is done with the panel before
            const int loads = kp / 64 * 2 * MB;
            // (every workgroup reads this x: each starts somewhere else in it, or they would all ask the same
            // L2 channel at the same time)
            const int first = (int)((blockIdx.x >> 3) * 37u % 32u) * (loads >> 5);
            for (int j0 = wave; j0 < loads; j0 += WAVES) {
                const int j = j0 + first < loads ? j0 + first : j0 + first - loads;
                int r, b;
                w_piece<128>(j & 1, lane, r, b);
                const int mb = MB == 2 ? (j >> 1) & 1 : 0, slab = j / (2 * MB);
                load_to_lds<16>(xbuf, L.x + j * 1024, (uint32_t)min(mb * 16 + r, M - 1) * (uint32_t)K * 2 + b,
                                (uint32_t)(k0 + slab * 64) * 2);
            }
        }
        // lines of this panel; a wavefront takes every eighth, tile after tile
        const int lines = (kp + KL - 1) / KL, mine = (lines - wave + WAVES - 1) / WAVES;
        const int items = max(mine, 0) * nt;
        u32x4 w[RD][2];
        int it = 0, il = wave; // the next request: tile and line
        const uint32_t line0 = (uint32_t)k0 / 8 * BITS;
        auto issue = [&](u32x4 (&to)[2]) {
            // Past the last line the lanes ask beyond the buffer's end, which costs no access (fq_batch_at.h).  An odd
            // number of groups at 2, 3 and 4 bits: the second half of a row's last line is the next row's, and not used.
            const uint32_t at = batch_request(row_bytes, lane_off, it, line0, il, LB);
            to[0] = load_piece<BITS>(wbuf, at);
            to[1] = load_piece<BITS>(wbuf, at + LB / 2);
            il += WAVES;
            if (il >= lines) {
                il = wave;
                it++;
            }
        };
        if (items > 0) {
#pragma unroll
            for (int j = 0; j < RD; j++)
                issue(w[j]);
        }
        if (BITS != 16) {
            // Scales and zero points of the batch's tiles for the panel's groups, [tile][row][group]: all requested together (a
            // loop that stored each before it asked for the next made up to six trips to memory).  A thread's rows are THREADS /
            // GP apart; rows past the run are beyond both buffers, groups past K are put there.
            constexpr int ML = NB * 16 * GP / THREADS;
            const int rows = min(nt * 16, N - n0), r0 = threadIdx.x / GP, g = threadIdx.x % GP;
            const __amdgpu_buffer_rsrc_t sbuf = buffer_of(scales + (size_t)n0 * G, (uint32_t)rows * G * 4);
            const __amdgpu_buffer_rsrc_t zbuf = buffer_of(zeros + (size_t)n0 * G, (uint32_t)rows * G);
            auto fetch = [&](auto n) __attribute__((always_inline)) {
                uint32_t at = g0 + g < G ? (uint32_t)(r0 * G + g0 + g) : 0x1f000000u;
                float s[n];
                uint8_t z[n];
#pragma unroll
                for (int i = 0; i < n; i++) {
                    s[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(sbuf, (int)(at * 4), 0, 0));
                    z[i] = __builtin_amdgcn_raw_buffer_load_b8(zbuf, (int)at, 0, 0);
                    at += (uint32_t)(THREADS / GP) * (uint32_t)G;
                }
#pragma unroll
                for (int i = 0; i < n; i++) {
                    L.s[(r0 + i * (THREADS / GP)) * GS + g] = s[i];
                    L.z[(r0 + i * (THREADS / GP)) * GS + g] = z[i];
                }
            };
            if (nt * 16 <= THREADS / GP)
                fetch(std::integral_constant<int, 1>{});
            else if (ML > 3 && nt * 16 <= 3 * (THREADS / GP))
                fetch(std::integral_constant<int, 3>{});
            else
                fetch(std::integral_constant<int, ML>{});
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();

        float4_t out[MB];
#pragma unroll
        for (int mb = 0; mb < MB; mb++)
            out[mb] = float4_t{0.f, 0.f, 0.f, 0.f};
        int ct = 0, cl = wave;
        auto compute = [&](const u32x4 (&v)[2]) {
            if constexpr (BITS <= 4) {
                const int g = cl * 2;
                const uint8_t *xs = L.x + (size_t)g * 4096 * MB;
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    if (h == 1 && g + 1 >= gp)
                        break;
                    const float s = L.s[(ct * 16 + n) * GS + g + h];
                    const uint32_t z = L.z[(ct * 16 + n) * GS + g + h];
                    float4_t acc[MB];
#pragma unroll
                    for (int mb = 0; mb < MB; mb++)
                        acc[mb] = float4_t{0.f, 0.f, 0.f, 0.f};
                    uint32_t b[4][4];
                    mg.group(v[h], z, b);
#pragma unroll
                    for (int i = 0; i < 4; i++)
#pragma unroll
                        for (int mb = 0; mb < MB; mb++)
                            acc[mb] = mfma16(*reinterpret_cast<const u32x4 *>(xs + h * 4096 * MB + mb * 2048 + xat[i]), b[i], acc[mb]);
#pragma unroll
                    for (int mb = 0; mb < MB; mb++)
                        out[mb] += s * acc[mb];
                }
            } else if constexpr (BITS == 8) {
                const uint8_t *xs = L.x + (size_t)cl * 4096 * MB;
                const float s = L.s[(ct * 16 + n) * GS + cl];
                const uint32_t z = L.z[(ct * 16 + n) * GS + cl], nz = (z | (z << 16)) | 0xE400E400u;
                float4_t acc[MB];
#pragma unroll
                for (int mb = 0; mb < MB; mb++)
                    acc[mb] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const uint32_t q0 = v[i >> 1][2 * (i & 1)], q1 = v[i >> 1][2 * (i & 1) + 1];
                    uint32_t b[4];
                    b[0] = pk_add(__builtin_amdgcn_perm(mg.e0, q0, 0x04010400u), nz);
                    b[1] = pk_add(__builtin_amdgcn_perm(mg.e0, q0, 0x04030402u), nz);
                    b[2] = pk_add(__builtin_amdgcn_perm(mg.e0, q1, 0x04010400u), nz);
                    b[3] = pk_add(__builtin_amdgcn_perm(mg.e0, q1, 0x04030402u), nz);
#pragma unroll
                    for (int mb = 0; mb < MB; mb++)
                        acc[mb] = mfma16(*reinterpret_cast<const u32x4 *>(xs + ((i >> 1) * MB + mb) * 2048 + xat[i & 1]), b, acc[mb]);
                }
#pragma unroll
                for (int mb = 0; mb < MB; mb++)
                    out[mb] += s * acc[mb];
            } else {
                const uint8_t *xs = L.x + (size_t)cl * 2048 * MB;
#pragma unroll
                for (int i = 0; i < 2; i++) {
                    const uint32_t b[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
                    for (int mb = 0; mb < MB; mb++)
                        out[mb] = mfma16(*reinterpret_cast<const u32x4 *>(xs + mb * 2048 + xat[i]), b, out[mb]);
                }
            }
            cl += WAVES;
            if (cl >= lines) { // the tile's last line in this panel
                cl = wave;
#pragma unroll
                for (int t = 0; t < NB; t++)
                    if (t == ct) {
#pragma unroll
                        for (int mb = 0; mb < MB; mb++)
                            sum[t][mb] += out[mb];
                    }
#pragma unroll
                for (int mb = 0; mb < MB; mb++)
                    out[mb] = float4_t{0.f, 0.f, 0.f, 0.f};
                ct++;
            }
        };
        for (int i = 0; i < items; i += RD) {
#pragma unroll
            for (int j = 0; j < RD; j++) {
                if (i + j < items)
                    compute(w[j]);
                issue(w[j]);
            }
        }
    }
    // The wavefronts' sums, added in their order: all blocks of 16 x 16 outputs at once through the panel's place, or, if the
    // next run reads the panel, two at a time (six tiles 1.9 us instead of 1.0).
    static_assert(NB * MB * WAVES * 1024 <= XBYTES, "the sums of a run fit a panel");
    auto leave = [&](float4_t *red, int u, int at) __attribute__((always_inline)) {
        red[(at * WAVES + wave) * 64 + lane] = sum[u / MB][u % MB];
    };
    auto add_up = [&](const float4_t *red, int b0, int b1) __attribute__((always_inline)) {
        for (int u = b0 + (int)(threadIdx.x >> 8); u < b1; u += 2) {
            // D layout of the 16x16 MFMA: lane holds column n (weight row), rows (batch) 4 * c + r
            const int m16 = (threadIdx.x >> 4) & 15, nn = threadIdx.x & 15;
            const float *p = reinterpret_cast<const float *>(red + (u - b0) * WAVES * 64) + ((m16 >> 2) * 16 + nn) * 4 + (m16 & 3);
            float v = p[0];
#pragma unroll
            for (int q = 1; q < WAVES; q++)
                v += p[q * 256];
            const int tile = u / MB, row = n0 + tile * 16 + nn, m = u % MB * 16 + m16;
            if (m < M && row < N)
                ((FQ_GLOBAL uint16_t *)y)[(size_t)m * N + row] = __builtin_bit_cast(uint16_t, (_Float16)v);
        }
    };
    const int blocks = nt * MB;
    if (keep_x) {
#pragma unroll
        for (int t = 0; t < NB * MB; t += 2) {
            if (t >= blocks)
                break;
            __syncthreads();
            leave(L.red, t, 0);
            leave(L.red, t + 1, 1);
            __syncthreads();
            add_up(L.red, t, min(t + 2, blocks));
        }
    } else {
        float4_t *red = reinterpret_cast<float4_t *>(L.x);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NB * MB; u++)
            if (u < blocks)
                leave(red, u, u);
        __syncthreads();
        add_up(red, 0, blocks);
    }
}

// A wavefront's view of the launch: lane e holds entry e, all of it, so that one trip to memory serves the whole table;
// every wavefront works out the same division of the launch's cost.
template <bool SINGLE, int MB, bool NARROW>
struct Division {
    int bits, N, K, lo, hi; // lo, hi: the entry's tiles that fall to this workgroup
    const void *codes, *scales, *zeros, *x;
    void *y;
    const void *c4, *c8, *c16, *s4, *s8, *z4, *z8;
    const void *c2, *c3, *s2, *s3, *z2, *z3; // NARROW
    unsigned long long todo;
    int t, te;

    // Request lane e's entry (lanes past the last repeat it).
    __device__ __forceinline__ void request_table(const FqLinearDesc &single, int bits_host, const FqLinearDesc *table,
                                                  const int32_t *bits_dev, int count)
    {
        const int e = min((int)(threadIdx.x & 63), count - 1);
        const FqLinearDesc *d = SINGLE ? &single : &table[e];
        bits = SINGLE ? bits_host : bits_dev[e];
        c4 = d->codes4, c8 = d->codes8, c16 = d->w16, s4 = d->scales4, s8 = d->scales8, z4 = d->zeros4, z8 = d->zeros8;
        x = d->x, y = d->y, N = d->N, K = d->K;
        if (NARROW)
            c2 = d->codes2, c3 = d->codes3, s2 = d->scales2, s3 = d->scales3, z2 = d->zeros2, z3 = d->zeros3;
        __builtin_amdgcn_sched_barrier(0); // ahead of what is requested next
    }
    __device__ __forceinline__ void settle(int count, uint32_t step, int *flags)
    {
        const int lane = threadIdx.x & 63;
        if (!SINGLE) // (all of it has been asked for, whatever the width: chosen pointers alone would be a second trip)
            asm volatile("" : "+v"(c4), "+v"(c8), "+v"(c16), "+v"(s4), "+v"(s8), "+v"(z4), "+v"(z8), "+v"(bits), "+v"(N), "+v"(K),
                              "+v"(x), "+v"(y));
        if (!SINGLE && NARROW)
            asm volatile("" : "+v"(c2), "+v"(c3), "+v"(s2), "+v"(s3), "+v"(z2), "+v"(z3));
        codes = bits == 4 ? c4 : bits == 8 ? c8 : bits == 16 ? c16 : nullptr;
        scales = bits == 4 ? s4 : s8;
        zeros = bits == 4 ? z4 : z8;
        if (NARROW && (bits == 2 || bits == 3))
            codes = bits == 2 ? c2 : c3, scales = bits == 2 ? s2 : s3, zeros = bits == 2 ? z2 : z3;
        int tiles = 0, cost = 0;
        if (lane < count) {
            if (codes) {
                tiles = (N + 15) >> 4;
                cost = batch_tile_cost(MB, K, bits);
            } else if (flags && blockIdx.x == 0 && threadIdx.x < 64) {
                *flags = 1; // no such width here, or no copy of it: nobody runs this entry
            }
        }
        const uint32_t mine = tiles > 0 ? (uint32_t)tiles * cost + BATCH_START_COST : 0u;
        uint32_t upto = mine; // inclusive prefix
        if (!SINGLE)
            for (int off = 1; off < count; off <<= 1) {
                const uint32_t o = __shfl_up(upto, off, 64);
                if (lane >= off)
                    upto += o;
            }
        const uint32_t all = __builtin_amdgcn_readlane(upto, count - 1);
        // this workgroup's share of the cost; a tile belongs to the share its first unit lies in
        lo = hi = 0;
        if (tiles > 0) {
            lo = batch_first_tile(batch_share_at(all, blockIdx.x, gridDim.x, step), upto - mine, cost, tiles);
            hi = batch_first_tile(batch_share_at(all, blockIdx.x + 1, gridDim.x, step), upto - mine, cost, tiles);
        }
        todo = __ballot(hi > lo);
        t = te = 0;
    }
    __device__ __forceinline__ static const void *of(const void *p, int e) // lane e's pointer
    {
        const uint64_t v = reinterpret_cast<uint64_t>(p);
        const uint32_t lo32 = __builtin_amdgcn_readlane((uint32_t)v, e), hi32 = __builtin_amdgcn_readlane((uint32_t)(v >> 32), e);
        return reinterpret_cast<const void *>((uint64_t)hi32 << 32 | lo32);
    }
    // The run after `r`; nt = 0: there is none.
    __device__ __forceinline__ Run next_run(Run r)
    {
        if (t >= te) {
            if (!todo) {
                r.nt = 0;
                return r;
            }
            const int e = __builtin_ctzll(todo);
            todo &= todo - 1;
            r.bits = __builtin_amdgcn_readlane(bits, e);
            t = __builtin_amdgcn_readlane(lo, e), te = __builtin_amdgcn_readlane(hi, e);
            r.N = __builtin_amdgcn_readlane(N, e), r.K = __builtin_amdgcn_readlane(K, e);
            r.codes = (const uint8_t *)of(codes, e), r.zeros = (const uint8_t *)of(zeros, e);
            r.scales = (const float *)of(scales, e);
            r.x = (const uint16_t *)of(x, e);
            r.y = (uint16_t *)const_cast<void *>(of(y, e));
        }
        r.t0 = t;
        r.nt = min(NB, te - t);
        t += r.nt;
        return r;
    }
};

// x0, K0: what every entry reads, if they all read one x (else null): requested before anything else is known.  `step`:
// batch_step of the grid.
// NARROW: entries may hold 2- and 3-bit copies (the other instances are without their code and pointers); a single call's
// instance with them meets nothing else.
template <bool SINGLE, int MB, bool NARROW>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void decode_batch_kernel(
    const FqLinearDesc single, int bits_host, const FqLinearDesc *__restrict__ table, const int32_t *__restrict__ bits_dev,
    int count, int M, int *flags, const uint16_t *x0, int K0, uint32_t step)
{
    constexpr bool WIDE = !SINGLE || !NARROW;
    __shared__ Lds L;
    Division<SINGLE, MB, NARROW> dv;
    dv.request_table(single, bits_host, table, bits_dev, count);
    if (x0)
        fetch_first_x<MB>(L, x0, K0, M);
    dv.settle(count, step, flags);
    Run r = {};
    r = dv.next_run(r);
    bool there = x0 && r.nt > 0; // the run's first panel is in LDS, or on its way
    if (x0 && !there) // (no run: what was asked for arrives while the workgroup still has its LDS)
        __builtin_amdgcn_s_waitcnt(0);
    while (r.nt > 0) {
        const Run next = dv.next_run(r);
        const bool keep = next.nt > 0 && next.x == r.x && next.K == r.K && r.K <= Panel<MB>::KP;
        if (NARROW && r.bits == 2)
            run_batch<2, MB>(L, r.codes, r.scales, r.zeros, r.x, r.y, r.N, r.K, M, r.t0, r.nt, there, keep);
        else if (NARROW && r.bits == 3)
            run_batch<3, MB>(L, r.codes, r.scales, r.zeros, r.x, r.y, r.N, r.K, M, r.t0, r.nt, there, keep);
        else if (WIDE && r.bits == 4)
            run_batch<4, MB>(L, r.codes, r.scales, r.zeros, r.x, r.y, r.N, r.K, M, r.t0, r.nt, there, keep);
        else if (WIDE && r.bits == 8)
            run_batch<8, MB>(L, r.codes, r.scales, r.zeros, r.x, r.y, r.N, r.K, M, r.t0, r.nt, there, keep);
        else if (WIDE)
            run_batch<16, MB>(L, r.codes, nullptr, nullptr, r.x, r.y, r.N, r.K, M, r.t0, r.nt, there, keep);
        there = keep;
        r = next;
        if (r.nt > 0)
            __syncthreads(); // LDS is free again
    }
}

} // namespace

// Plans.  Up to 24 tiles per compute unit (two 7B-shaped layers): there the plans of mixed widths of the 7B, 13B and
// 70B shapes take 0.58 to 0.90 of the time on the register-fed kernel's round-robin tiles; at four layers {4, 8} 195 against
// 216 us, but {4, 8, 16} 296 against 265 and all widths at 32 batch rows slower, since each run of NB tiles starts anew.
// Below that as for single calls, over 3740 plans: with more than two tiles per compute unit rows must not be short, the
// mean over a plan's rows and copies (without: 4 x 16384 x 512 at {4, 8} 1.7, 3 x 24576 x 1024 at 4 bits 1.6), counted by the panels
// of x they take (K = 5120 takes two and fills one and a quarter), and where the register-fed kernel's 64-row tiles fill
// their rounds it keeps plans of 4-bit copies alone over more than 16 batch rows or over part panels (65536 x 5120: 1.15).
// Under this rule 0.85 of its time on average; one plan in a hundred is 1.06 to 1.19, where a workgroup's tiles are
// one more than full runs or a round of the other kernel is just full.
// 2- and 3-bit copies: the register-fed kernel loses more on them (over 800 timings of the 7B, 13B and 70B shapes' stages and of short rows, with
// {2}, {3}, {2, 4, 8} and {3, 4, 8} resident, 0.70 of its time; 7B stages of {2, 4, 8} 0.54, of {3, 4, 8} 0.72), so that shorter rows come here.
// No more rows than above: at 27 x 8192 x 8192 3 bits took 1.1 of its time here, 35 x 6000 x 5120 1.2.  What stays (times here over
// times there, each width for all entries and mixed):
//   - rows of two part panels with a 2- or 3-bit copy alone (5120 inputs: 1.1, 1.05; it is why 3 bits count 13 and not 14 below);
//   - several entries of part panels over up to 16 batch rows whose 64-row tiles fill their rounds: 5 x 6000 x 5120 {2, 4, 8} 1.08 / 1.04 /
//     0.92 / 0.83, 8 x 6000 x 5120 {3, 4, 8} 1.02 / 1.03 / 0.96 / 1.12, 24 x 2048 x 6144 (full rounds) {2, 4, 8} 1.09 / 1.05 / 0.95 / 1.07; not
//     60 x 512 x 6144, 0.98 / 0.93 / 0.82 / 0.82;
//   - short entries of more than three panels over more than 16, each with an x of its own, which every workgroup reads again
//     for each of its runs: 30 x 1000 x 8192 {3, 4, 8} 1.13 / 1.14 / 1.01 / 1.01, {2} 1.11 (one x for all 0.78 to 0.89; 60 x 512 x 6144, 24 x 1200 x
//     11008 and 50 x 1000 x 8192, whose 64-row tiles leave a round unfilled, 0.95, 0.96 and 0.78 on average).
// Behind the other kernel here: the 13B q/k/v stage of {2, 4, 8} when all three run at 2 bits, 18.9 us against 17.0 (all at 4 bits 20.9 against
// 22.5, at 8 26.7 against 33.3, mixed 19.7 against 30.9), and up to 1.04 60 x 512 x 6144 and 24 x 1200 x 11008 at one narrow width over 32 rows.
bool fq_batch_serves(const FqLinearDesc *table, int count, int M)
{
    const int cus = fq_device_cus(), panel = batch_panel(M <= 16 ? 1 : 2);
    long long rows = 0, tiles = 0;
    double weight = 0, inputs = 0, padded = 0; // summed over the rows
    bool four_alone = true, narrow = false, own_x = false;
    for (int i = 0; i < count; i++) {
        const FqLinearDesc &d = table[i];
        const int copies = (d.codes2 != nullptr) + (d.codes3 != nullptr) + (d.codes4 != nullptr) + (d.codes8 != nullptr) + (d.w16 != nullptr);
        const int per_group = (d.codes2 ? 11 : 0) + (d.codes3 ? 13 : 0) + (d.codes4 ? 17 : 0) + (d.codes8 ? 29 : 0) + (d.w16 ? 53 : 0); // about 3 * bits + 5
        narrow = narrow || d.codes2 || d.codes3;
        own_x = own_x || d.x != table[0].x;
        four_alone = four_alone && !d.codes2 && !d.codes3 && !d.codes8 && !d.w16;
        rows += d.N;
        tiles += ((long long)d.N + 15) / 16;
        weight += (double)d.N * (d.K >> 7) * per_group / (copies > 0 ? copies : 1);
        inputs += (double)d.N * d.K;
        padded += (double)d.N * ((d.K + panel - 1) / panel) * panel;
    }
    if (count > MAX_ENTRIES || rows > 384LL * cus)
        return false;
    if (tiles <= 2 * cus)
        return true;
    if (weight / rows * inputs / padded < (narrow ? 340 : 400))
        return false;
    const int rest = (int)(rows % (64 * cus));
    const bool filled = rows > 96 * cus && (rest == 0 || rest > 48 * cus);
    const bool parts = inputs < (rest == 0 || rest > 60 * cus ? 0.8 : 0.7) * padded; // rows are mostly part panels
    if (filled && narrow && (M <= 16 ? count > 1 && parts : own_x && rows <= 1024LL * count && inputs > 3.0 * panel * rows))
        return false;
    return !(filled && four_alone && (M > 16 || padded > inputs));
}

// Single calls, both kernels measured at 128 to 11008 inputs, 1024 to 200000 rows, 2, 16, 17 and 32 batch rows (ratios of
// times, this kernel's first).  Short rows give most of a workgroup's wavefronts nothing to do: 32768 x 512 at 4
// bits 1.5 to 1.7; from 3072 inputs at 4 bits, 1792 at 8 and 1024 at 16 on 0.7 to 1.0 -- unless there are at most three tiles
// per compute unit, where the launch is what counts (0.85 to 1.03 at any K).  The register-fed kernel's 64-row tiles
// come in rounds of one per compute unit; where they fill the last round (32768 rows: two full rounds) it wins
// back 10 to 20 %: at 4 bits it then keeps the calls over more than 16 batch rows (1.02 to 1.16; with that round three
// quarters full, 28672 x 8192: 0.92 to 0.99) or over a K that leaves part of a panel of x (5120: 1.08; 4096: 0.93,
// 8192: 0.95), up to six rounds (beyond: 0.75 to 1.0).  With 512 rows per compute unit it goes over to larger tiles and is as good or better (131072 rows at 4 bits: 1.1 to 2.9).  Under this rule
// 0.86 of the register-fed kernel's time on average over 5900 calls; one shape stays behind it (29696 x 5120 at 16 bits, 1.14).
bool fq_batch_serves_linear(int N, int K, int bits, int M)
{
    const int cus = fq_device_cus();
    if (fq_skinny_tile_rows(N, M) > 64)
        return false;
    if ((N + 15) / 16 <= 3 * cus)
        return true;
    const int weight = (K >> 7) * (3 * bits + 5); // what a tile's bytes and arithmetic grow with
    const int rest = N % (64 * cus);              // rows of the last round of 64-row tiles (0: a full one)
    const bool half = N > 96 * cus && (rest == 0 || rest > (M > 16 ? 35 : 48) * cus); // it is half or more full
    const bool filled = half && (rest == 0 || rest > 48 * cus);
    if (!half)
        return weight >= 400;
    return weight >= 470 && (!filled || bits != 4 || N > 384 * cus || (M <= 16 && K % 4096 == 0));
}

// Single calls at 2 and 3 bits: as a plan of that entry alone, which has the copy's width alone.  Over 512 to 28672 rows and as many
// inputs, 2 to 32 batch rows, 0.42 (28672 inputs, 2 bits) to 0.86 (1024, 3 bits) of the register-fed kernel's time on average, none more than 1.02.
bool fq_batch_serves_narrow(int N, int K, int bits, int M)
{
    FqLinearDesc d = {};
    d.N = N, d.K = K;
    (bits == 2 ? d.codes2 : d.codes3) = reinterpret_cast<const uint8_t *>(16); // (that there is one)
    return fq_batch_serves(&d, 1, M);
}

// (A slab finds the weights in the caches, where the register-fed kernel's 64-row tiles gain more: 28672 x 5120 over 100 batch rows
// took 1.07 of its time here, 8192 x 512 1.04; 4096 x 4096 over 100: 113 us there, 35 here.)
bool fq_batch_serves_slab(int N, int K, int M)
{
    return K >= 1024 && (K % batch_panel(2) == 0 || N <= 64 * fq_device_cus()) && fq_batch_serves_narrow(N, K, 3, M);
}

hipError_t fq_launch_batch(const FqLinearDesc *single, int bits_host, const FqLinearDesc *descs_dev, const int32_t *bits_dev,
                           int count, long long tiles, int M, bool narrow, int *flags, const uint16_t *x0, int K0, hipStream_t stream)
{
    const int cus = fq_device_cus();
    const unsigned grid = (unsigned)(tiles < cus ? tiles : cus);
    const uint32_t step = batch_step(grid);
    // The request ahead is of a whole panel.  Times with it over those without: 128 inputs 1.11 to 1.15, 512 1.03 to 1.12, 1024 0.96 (above
    // 16 rows) to 1.10 (plans), 1920 0.90 to 0.98 for single calls, 0.94 to 1.04 for plans.
    if (K0 < 2048)
        x0 = nullptr;
    FqLinearDesc none = {};
    auto go = [&](auto mb, auto narrow) {
        constexpr int MB = decltype(mb)::value;
        constexpr bool NARROW = decltype(narrow)::value;
        if (single)
            decode_batch_kernel<true, MB, NARROW><<<grid, THREADS, 0, stream>>>(*single, bits_host, nullptr, nullptr, 1, M, nullptr, x0, K0, step);
        else
            decode_batch_kernel<false, MB, NARROW><<<grid, THREADS, 0, stream>>>(none, 0, descs_dev, bits_dev, count, M, flags, x0, K0, step);
    };
    typedef std::integral_constant<int, 1> One;
    typedef std::integral_constant<int, 2> Two;
    if (narrow)
        M <= 16 ? go(One(), std::true_type()) : go(Two(), std::true_type());
    else
        M <= 16 ? go(One(), std::false_type()) : go(Two(), std::false_type());
    return hipGetLastError();
}
