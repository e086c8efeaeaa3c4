// Weight-only quantized linear for prompts of some tens to some hundreds of tokens: y[M][N] =
// x[M][K] . dequant(W[N][K])^T (Sec. 2.2 Eq. (3)), M > 32 -- the same product as the prefill GEMM
// (fq_prefill.hip, whose operand rounding it shares), for the shapes that do not give that kernel's
// 256 x 256 tiles a compute unit each: 4096 rows are 16 of them, walked by 16 of 256 compute units while the
// rest idle (100 x 11008 x 4096 at 4 bits: 174 us, of which the weights' 24 MB take 4).
//
// Split.  A workgroup (8 wavefronts) takes 64, 96 or 128 tokens x 128 weight rows and one of up to 16
// segments of K; the segments' sums meet, in binary32, in a static device array and a second launch
// adds them in order (23 us for the call above, four segments).  In a workgroup four wavefronts stand along the rows, 32
// each, and two along K: one takes the first 64 inputs of every group, one the last 64, so that a weight
// is unpacked by one wavefront only and eight wavefronts share one slab of x; the two halves meet in
// LDS at the end.  Tokens and segments are chosen by a cost model (prompt_cost below).
//
// A step is one quantization group, 128 inputs.  Slabs come in by direct-to-LDS loads, three stages; scales and
// zero points eight groups at a time.  Rows of x (256 bytes a step) are stored with their 16 pieces XOR-ed
// by row % 16, weight rows by the rules of w_offset: 16 consecutive rows of one operand read touch every
// bank once, and the first eight stay in one half of the bank row.  A wavefront takes the packed weights
// and constants of step t + 1 out of LDS during step t and unpacks the first operand ahead of the
// barrier, so that only reads of x stand between the barrier and the first MFMA (100 x 11008 x 4096 in one
// segment: 73 -> 67 us).
//
// What bounds it: a step of 128 tokens costs 0.65 to 0.8 us, of which the MFMAs are 0.45 (1024 clocks a
// SIMD) and the unpacking, 16 vector instructions per operand, most of the rest -- the two wavefronts of a
// SIMD leave the barrier together and overlap the two only in part; without the fetches the step takes
// 0.06 less, without reading x the same.  With few steps per segment the launch, the first fetch
// (cold weights) and the hand-over of the partial sums are half of the call.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "fq_internal.h"
#include "fq_mfma.h"

namespace {

constexpr int THREADS = 512;
constexpr int WAVES = 8;
constexpr int BN = 128;   // weight rows of a tile: 32 per wavefront, four wavefronts along the rows
constexpr int BK = 128;   // inputs of a step: one quantization group, 64 per half of the workgroup
constexpr int XRB = 2 * BK;
constexpr int MB = 8;     // groups per block of scales and zero points
constexpr int MAX_SEGMENTS = 16;
// Partial sums of the segments: one copy for each of the first FQ_PART_BANKS streams of a device (calls on
// different streams may overlap); any other call -- a further stream, one being captured, whose graph may
// be replayed beside anything -- walks its segments inside one workgroup, adding them in the same order:
// slower, the same bits, no array.
constexpr size_t PART_FLOATS = FQ_PART_FLOATS;
__device__ __attribute__((aligned(256))) float g_part[FQ_PART_BANKS][PART_FLOATS];

// Which 8 k of its 64-k half lane (row, c) supplies in k16-step i, as the index of a 16-byte piece of x.  A lane
// reads 16 bytes of codes at a time: 32 codes at 4 bits (8 bytes at 2 bits), words i = 0 .. 3 holding k = 32 c +
// 8 i ..; at 8 bits 16 codes, k = 32 (i / 2) + 16 c + 8 (i % 2) ..; fp16: k = 16 i + 8 c ..
template <int BITS>
__device__ __forceinline__ int x_chunk(int i, int c)
{
    return BITS == 4 || BITS == 2 ? 4 * c + i : BITS == 8 ? 4 * (i >> 1) + 2 * c + (i & 1) : 2 * i + c;
}

// MT: blocks of 32 tokens of a tile.
template <int BITS, int MT>
struct Tile {
    static constexpr int BM = 32 * MT;
    static constexpr int XST = BM * XRB;            // bytes of x per stage
    static constexpr int WRB = BK * BITS / 8;
    static constexpr int WST = BN * WRB;
    static constexpr int XL = XST / 16 / THREADS;   // loads of a thread per step
    static constexpr int WL = WST / 16 / THREADS > 0 ? WST / 16 / THREADS : 1;
    static constexpr int NST = BITS == 16 ? 2 : 3;  // stages (fp16 weights: 64 KiB each)
    static constexpr int OPS = XL + WL;
};

// `units` workgroups' work: tiles x segments, or with `serial` tiles, each with all its segments.  (K order
// of the units: all tiles of a segment are neighbours, and an XCD gets a run of them, so that the x of a
// segment is read into few L2s.)
template <int BITS, int MT>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void prompt_kernel(
    const FqLinearDesc d, int M, int m_tiles, int n_tiles, int units, int per_xcd, int segments, int serial, float *part)
{
    typedef Tile<BITS, MT> T;
    __shared__ __attribute__((aligned(1024))) uint8_t xs0[T::XST], xs1[T::XST], xs2[T::NST > 2 ? T::XST : 16];
    __shared__ __attribute__((aligned(1024))) uint8_t ws0[T::WST], ws1[T::WST], ws2[T::NST > 2 ? T::WST : 16];
    __shared__ __attribute__((aligned(1024))) float ms[BITS == 16 ? 1 : 2 * BN * MB];    // [block parity][row][group]
    __shared__ __attribute__((aligned(1024))) uint32_t mz[BITS == 16 ? 1 : 2 * BN * MB];

    const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || unit >= units)
        return;
    const int tiles = m_tiles * n_tiles;
    const int tile = serial ? unit : unit % tiles;
    const int seg0 = serial ? 0 : unit / tiles, seg1 = serial ? segments : seg0 + 1;
    const int m0 = (tile % m_tiles) * T::BM, n0 = (tile / m_tiles) * BN;

    const uint8_t *codes = BITS == 2 ? d.codes2 : BITS == 4 ? d.codes4 : BITS == 8 ? d.codes8 : (const uint8_t *)d.w16;
    const float *scales = BITS == 2 ? d.scales2 : BITS == 4 ? d.scales4 : d.scales8;
    const uint8_t *zeros = BITS == 2 ? d.zeros2 : BITS == 4 ? d.zeros4 : d.zeros8;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int l32 = lane & 31, c = lane >> 5;
    const int wn = wave & 3, wk = wave >> 2;
    const uint32_t K = (uint32_t)d.K, G = K >> 7;
    const uint32_t w_pitch = K * BITS / 8;
    const int x_last = M - 1 - m0, w_last = d.N - 1 - n0;
    const uint8_t *x_tile = (const uint8_t *)d.x + (size_t)m0 * K * 2;
    const uint8_t *w_tile = codes + (size_t)n0 * w_pitch;
    const float *scales_tile = BITS == 16 ? nullptr : scales + (size_t)n0 * G;
    const uint8_t *zeros_tile = BITS == 16 ? nullptr : zeros + (size_t)n0 * G;

    const __amdgpu_buffer_rsrc_t xbuf = buffer_of(x_tile, (uint32_t)(min(x_last, T::BM - 1) + 1) * K * 2);
    const __amdgpu_buffer_rsrc_t wbuf = buffer_of(w_tile, (uint32_t)(min(w_last, BN - 1) + 1) * w_pitch);
    const __amdgpu_buffer_rsrc_t sbuf = buffer_of(scales_tile, (uint32_t)(min(w_last, BN - 1) + 1) * G * 4);
    const __amdgpu_buffer_rsrc_t zbuf = buffer_of(zeros_tile, (uint32_t)(min(w_last, BN - 1) + 1) * G);

    // Operand reads: this lane's offset of k16-step i in a stage.
    const int row = wn * 32 + l32; // weight row
    int aofs[4], bofs[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        aofs[i] = l32 * XRB + (((wk * 8 + x_chunk<BITS>(i, c)) ^ (l32 & 15)) << 4);
        bofs[i] = BITS == 2   ? w_offset<T::WRB>(row, wk) + 8 * c
                  : BITS == 4 ? w_offset<T::WRB>(row, wk * 2 + c)
                  : BITS == 8 ? w_offset<T::WRB>(row, wk * 4 + 2 * (i & 1) + c)
                              : w_offset<T::WRB>(row, wk * 8 + 2 * i + c);
    }
    // Fetches: this thread's piece of each load, as an offset from the tile.
    uint32_t xoff[T::XL], woff[T::WL];
#pragma unroll
    for (int i = 0; i < T::XL; i++) {
        const int r = i * 32 + wave * 4 + (lane >> 4);
        xoff[i] = (uint32_t)min(r, x_last) * (K * 2) + (((lane & 15) ^ (r & 15)) << 4);
    }
    const int wwave = BITS == 2 ? wave & 3 : wave; // a 2-bit slab is half a load of the workgroup: fetched twice
#pragma unroll
    for (int i = 0; i < T::WL; i++) {
        int r, b;
        w_piece<T::WRB>(i * WAVES + wwave, lane, r, b);
        woff[i] = (uint32_t)min(r, w_last) * w_pitch + b;
    }
    // Scales and zero points, MB groups at a time: load i of wavefront w covers rows (i * 8 + w) * 8 .. + 7,
    // slot j of row r holding group j ^ (r >> 3 & 7).
    const uint32_t mgrp = (uint32_t)((lane & 7) ^ (wave & 7));
    uint32_t mrow[2];
#pragma unroll
    for (int i = 0; i < 2; i++)
        mrow[i] = (uint32_t)min((i * 8 + wave) * 8 + (lane >> 3), w_last) * G;
    auto fetch_meta = [&](uint32_t gb, int buf) {
        if (BITS == 16)
            return;
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const uint32_t at = mrow[i] + min(gb + mgrp, G - 1);
            load_to_lds<4>(sbuf, ms + buf * BN * MB + (i * 8 + wave) * 64, at * 4, 0);
            load_to_lds<1>(zbuf, mz + buf * BN * MB + (i * 8 + wave) * 64, at, 0);
        }
    };
    auto wait_vm = [](auto n) {
        constexpr int N = decltype(n)::value;
        __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
    };
    auto barrier = [] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto stage_x = [&](auto st) -> uint8_t * {
        constexpr int ST = decltype(st)::value;
        return ST == 0 ? xs0 : ST == 1 ? xs1 : xs2;
    };
    auto stage_w = [&](auto st) -> uint8_t * {
        constexpr int ST = decltype(st)::value;
        return ST == 0 ? ws0 : ST == 1 ? ws1 : ws2;
    };

    // a power of two per weight row that brings its scales to where a half holds them exactly
    int ex = 0;
    if (BITS != 16) {
        const float *srow = scales_tile + (size_t)min(row, w_last) * G;
        const float m = fmaxf(*(const FQ_GLOBAL float *)srow, *(const FQ_GLOBAL float *)(srow + (G >> 1)));
        ex = -3 - __builtin_amdgcn_frexp_expf(m);
    }

    constexpr int H = (MT + 1) / 2; // 32-token blocks that the first half of the workgroup finishes; the rest: the second
    float16_t acc[MT], total[H];
    for (int seg = seg0; seg < seg1; seg++) {
        const int g0 = (int)((long long)seg * G / segments), g1 = (int)((long long)(seg + 1) * G / segments);
        const int ng = g1 - g0;
#pragma unroll
        for (int t = 0; t < MT; t++)
#pragma unroll
            for (int v = 0; v < 16; v++)
                acc[t][v] = 0.f;
        // Loads [P0, P1) of the XL + WL that bring one step's x and one step's weights: a step issues those
        // of x two steps ahead and of the weights three ahead (fp16: both one ahead).  Steps past the end
        // are clamped: always issued, the waits count them.
        auto fetch = [&](int tx, auto sx, int tw, auto sw, auto p0, auto p1) {
            const uint32_t gx = (uint32_t)(g0 + min(tx, ng - 1)), gw = (uint32_t)(g0 + min(tw, ng - 1));
#pragma unroll
            for (int i = 0; i < T::OPS; i++) {
                if (i < decltype(p0)::value || i >= decltype(p1)::value)
                    continue;
                if (i < T::XL)
                    load_to_lds<16>(xbuf, stage_x(sx) + (i * WAVES + wave) * 1024, xoff[i < T::XL ? i : 0], gx * XRB);
                else
                    load_to_lds<16>(wbuf, stage_w(sw) + ((i - T::XL) * WAVES + wwave) * 1024, woff[i < T::XL ? 0 : i - T::XL],
                                    gw * T::WRB);
            }
        };
        typedef std::integral_constant<int, 0> I0;
        typedef std::integral_constant<int, 1> I1;
        typedef std::integral_constant<int, T::NST - 1> I2;
        typedef std::integral_constant<int, T::XL> IX;
        typedef std::integral_constant<int, T::OPS> IN;
        // What a wavefront knows of the step it is about to run: its weights (all four k16-steps, packed),
        // the group's constants, the first weight operand.  Taken from LDS during the step before, so that
        // behind the barrier only reads of x stand before the first MFMA.
        u32x4 w4 = {0, 0, 0, 0}, w5 = {0, 0, 0, 0};
        float sc = 0.f;
        uint32_t zp = 0;
        DeqConst dc;
        DeqMagic<BITS> mg;
        mg.pin();
        uint32_t b[2][4];
        auto read_w = [&](int t, auto st) {
            if (BITS == 16)
                return;
            const uint8_t *wc = stage_w(st);
            if (BITS == 2) {
                const u32x2 q = *reinterpret_cast<const u32x2 *>(wc + bofs[0]);
                w4.x = q.x, w4.y = q.y;
            } else {
                w4 = *reinterpret_cast<const u32x4 *>(wc + bofs[0]);
            }
            if (BITS == 8)
                w5 = *reinterpret_cast<const u32x4 *>(wc + bofs[1]);
            const int at = ((t >> 3) & 1) * BN * MB + row * MB + ((t & 7) ^ ((row >> 3) & 7));
            sc = ms[at];
            zp = mz[at];
        };
        auto operand = [&](int i, const u32x4 &q4, const u32x4 &q5) {
            if constexpr (BITS == 2)
                deq8<2>(i < 2 ? q4.x : q4.y, 0u, i, dc, mg, b[i & 1]);
            else if constexpr (BITS == 4)
                deq8<4>(q4[i], 0u, 0, dc, mg, b[i & 1]);
            else if constexpr (BITS == 8)
                deq8<8>(i == 0 ? q4.x : i == 1 ? q4.z : i == 2 ? q5.x : q5.z,
                        i == 0 ? q4.y : i == 1 ? q4.w : i == 2 ? q5.y : q5.w, 0, dc, mg, b[i & 1]);
        };

        fetch_meta(g0, 0);
        if (BITS == 16) {
            fetch(0, I0(), 0, I0(), I0(), IN());
            wait_vm(std::integral_constant<int, 0>());
            barrier();
        } else {
            fetch(0, I0(), 0, I0(), I0(), IN());
            fetch(0, I0(), 1, I1(), IX(), IN());
            fetch(1, I1(), 2, I2(), I0(), IN());
            wait_vm(std::integral_constant<int, T::OPS>());
            barrier();
            read_w(0, I0());
            dc = deq_const<BITS>(__builtin_ldexpf(sc, ex), zp);
            operand(0, w4, w5);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            barrier(); // step 0 refills the slab that was just read
        }

        auto step = [&](int t, auto st) {
            constexpr int ST = decltype(st)::value;
            typedef std::integral_constant<int, (ST + 1) % T::NST> NEXT1; // stage of step t + 1
            typedef std::integral_constant<int, (ST + 2) % T::NST> NEXT2; // of t + 2 (three stages)
            const uint8_t *xc = stage_x(st), *wc = stage_w(st);
            u32x4 a[2][MT];
            auto read_x = [&](int i) {
#pragma unroll
                for (int mt = 0; mt < MT; mt++)
                    a[i & 1][mt] = *reinterpret_cast<const u32x4 *>(xc + mt * 32 * XRB + aofs[i]);
                if (BITS == 16) {
                    const u32x4 q = *reinterpret_cast<const u32x4 *>(wc + bofs[i]);
                    b[i & 1][0] = q.x, b[i & 1][1] = q.y, b[i & 1][2] = q.z, b[i & 1][3] = q.w;
                }
            };
            read_x(0);
            const u32x4 c4 = w4, c5 = w5;
            // (past the end: read and not used.  Ahead of fetch_meta: behind it the compiler would wait for
            // those requests, which fill the other half of the same arrays)
            read_w(t + 1, NEXT1());
            __builtin_amdgcn_sched_barrier(0);
            if (BITS == 16)
                fetch(t + 1, NEXT1(), t + 1, NEXT1(), I0(), IN());
            else if ((t & 7) == 0 && t + MB < ng)
                fetch_meta(g0 + t + MB, ((t >> 3) + 1) & 1); // the oldest requests of the step
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; i++)
                asm volatile("" : "+v"(aofs[i]), "+v"(bofs[i]));
#pragma unroll
            for (int i = 0; i < 4; i++) {
                if (i < 3)
                    read_x(i + 1);
                if (T::NST > 2) {
                    // a quarter of the step's requests ahead of every quarter of its MFMAs
                    constexpr int O = T::OPS;
                    if (i == 0)
                        fetch(t + 2, NEXT2(), t + 3, st, I0(), std::integral_constant<int, O / 4>());
                    if (i == 1)
                        fetch(t + 2, NEXT2(), t + 3, st, std::integral_constant<int, O / 4>(), std::integral_constant<int, O / 2>());
                    if (i == 2)
                        fetch(t + 2, NEXT2(), t + 3, st, std::integral_constant<int, O / 2>(), std::integral_constant<int, O * 3 / 4>());
                    if (i == 3)
                        fetch(t + 2, NEXT2(), t + 3, st, std::integral_constant<int, O * 3 / 4>(), IN());
                }
                if (i < 3) {
                    operand(i + 1, c4, c5);
                } else if (BITS != 16) {
                    dc = deq_const<BITS>(__builtin_ldexpf(sc, ex), zp);
                    operand(0, w4, w5); // of step t + 1
                }
#pragma unroll
                for (int mt = 0; mt < MT; mt++)
                    acc[mt] = mfma32(a[i & 1][mt], b[i & 1], acc[mt]);
                // vector memory instructions stay on their side of the line, everything else may cross it
                __builtin_amdgcn_sched_barrier(0x38F);
            }
            wait_vm(std::integral_constant<int, T::NST == 3 ? T::OPS : 0>());
            barrier();
        };
        int t = 0;
        for (; t + T::NST <= ng; t += T::NST) {
            step(t, I0());
            step(t + 1, I1());
            if (T::NST > 2)
                step(t + 2, I2());
        }
        if (t < ng)
            step(t, I0());
        if (T::NST > 2 && t + 1 < ng)
            step(t + 1, I1());
        // The two halves of the workgroup meet in LDS (two of the x slabs hold a tile exactly): each leaves
        // the sums of the 32-token blocks that the other finishes and adds the other's to its own.
        __builtin_amdgcn_s_waitcnt(0);
        barrier();
        float4_t *xch = reinterpret_cast<float4_t *>(wn < 2 ? xs0 : xs1) + (wn & 1) * MT * 256 + lane;
        auto leave = [&](auto first, auto last) {
#pragma unroll
            for (int mt = decltype(first)::value; mt < decltype(last)::value; mt++)
#pragma unroll
                for (int q = 0; q < 4; q++)
                    xch[(mt * 4 + q) * 64] = float4_t{acc[mt][4 * q], acc[mt][4 * q + 1], acc[mt][4 * q + 2], acc[mt][4 * q + 3]};
        };
        auto take = [&](auto first, auto last) {
#pragma unroll
            for (int mt = decltype(first)::value; mt < decltype(last)::value; mt++)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const float4_t o = xch[(mt * 4 + q) * 64];
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const float v = acc[mt][4 * q + r] + o[r];
                        const float w = BITS == 16 ? v : __builtin_ldexpf(v, -ex);
                        total[mt - decltype(first)::value][4 * q + r] =
                            seg == seg0 ? w : total[mt - decltype(first)::value][4 * q + r] + w;
                    }
                }
        };
        typedef std::integral_constant<int, H> IH;
        typedef std::integral_constant<int, MT> IM;
        if (wk == 0)
            leave(IH(), IM());
        else
            leave(I0(), IH());
        __syncthreads();
        if (wk == 0)
            take(I0(), IH());
        else
            take(IH(), IM());
        if (seg + 1 < seg1)
            __syncthreads(); // the slabs are free again
    }
    // D layout of the 32x32 MFMA: lane holds column l32, rows 8 * (v / 4) + 4 * (lane / 32) + v % 4.
    const int mt0 = wk == 0 ? 0 : H, blocks = wk == 0 ? H : MT - H;
    if (!serial && segments > 1) {
        // partial sums as the wavefronts hold them, a lane's 16 bytes beside its neighbour's
        float *out = part + ((size_t)(seg0 * tiles + tile) * 4 * MT + wn * MT + mt0) * 1024 + lane * 4;
#pragma unroll
        for (int j = 0; j < H; j++)
            if (j < blocks)
#pragma unroll
                for (int q = 0; q < 4; q++)
                    *(FQ_GLOBAL float4_t *)(out + j * 1024 + q * 256) =
                        float4_t{total[j][4 * q], total[j][4 * q + 1], total[j][4 * q + 2], total[j][4 * q + 3]};
        return;
    }
    const int n = n0 + row;
#pragma unroll
    for (int j = 0; j < H; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) {
            const int m = m0 + (mt0 + j) * 32 + 8 * (v >> 2) + 4 * c + (v & 3);
            if (j < blocks && m < M && n < d.N)
                ((FQ_GLOBAL uint16_t *)d.y)[(size_t)m * d.N + n] = __builtin_bit_cast(uint16_t, (_Float16)total[j][v]);
        }
}

// Adds the segments' partial sums in the order of the segments.  A workgroup takes one block of 32 tokens x
// 32 weight rows (four wavefronts, a float4 per lane, as the tile's wavefront left it).
template <int MT>
__global__ __launch_bounds__(256) void prompt_reduce_kernel(const float *part, uint16_t *y, int M, int N, int m_tiles,
                                                            size_t seg_floats, int segments)
{
    const int block = blockIdx.x, tile = block / (4 * MT), wn = block / MT % 4, mt = block % MT;
    const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const float *p = part + (size_t)block * 1024 + threadIdx.x * 4;
    float4_t v = *(const FQ_GLOBAL float4_t *)p;
#pragma unroll 4
    for (int s = 1; s < segments; s++)
        v += *(const FQ_GLOBAL float4_t *)(p + s * seg_floats);
    const int n = tile / m_tiles * BN + wn * 32 + (lane & 31);
    const int m = tile % m_tiles * 32 * MT + mt * 32 + 8 * q + 4 * (lane >> 5);
#pragma unroll
    for (int r = 0; r < 4; r++)
        if (m + r < M && n < N)
            ((FQ_GLOBAL uint16_t *)y)[(size_t)(m + r) * N + n] = __builtin_bit_cast(uint16_t, (_Float16)v[r]);
}

template <int BITS, int MT>
hipError_t launch(const FqLinearDesc &d, int M, int segments, float *part, hipStream_t stream)
{
    typedef Tile<BITS, MT> T;
    const int m_tiles = (M + T::BM - 1) / T::BM, n_tiles = (d.N + BN - 1) / BN, tiles = m_tiles * n_tiles;
    const int serial = segments > 1 && !part;
    const int units = tiles * (serial ? 1 : segments);
    const int per_xcd = (units + 7) / 8;
    prompt_kernel<BITS, MT><<<(unsigned)per_xcd * 8, THREADS, 0, stream>>>(d, M, m_tiles, n_tiles, units, per_xcd, segments,
                                                                            serial, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || segments == 1 || serial)
        return e;
    prompt_reduce_kernel<MT><<<(unsigned)tiles * 4 * MT, 256, 0, stream>>>(part, d.y, M, d.N, m_tiles,
                                                                           (size_t)tiles * T::BM * BN, segments);
    return hipGetLastError();
}

// Microseconds a call is expected to take, fitted to 17000 timings of forced plans (33 to 2048 tokens, 512 to 28672
// rows, K 128 to 28672; 7 to 9 % off on average, fp16 weights 16, large tiles 6 to 10): launch and first fetch, then rounds of
// one workgroup per compute unit, each with an end that grows with its outputs, a step costing more the more tokens it has
// and the fuller the chip is; with segments the hand-over (0.8 more than fitted, for the host: a second launch).  The choice made from it is within 1 to 2 % of the best choice
// on average.  (Fitted without the rounds' ends and from K = 1024 on, it sent calls over few inputs the wrong way:
// 33 x 512 x 512 at fp16, four segments of one group, 1.28 of the large tiles' time.)
struct Cost {
    float call, round, out, step, step_mt, step_full, split, split_unit;
    float old_call, old_round, old_out, old_step, old_full, old_half; // the 256 x 256 tiles, per step of 64 inputs; a round of half tiles
};
const Cost &cost_of(int bits)
{
    static const Cost w2 = {3.45f, 2.65f, 0.207f, 0.147f, 0.110f, 0.090f, 3.5f, 4.76f / 1024, 2.f, 5.88f, 2.60f, 1.166f, 0.389f, 0.586f};
    static const Cost w4 = {3.40f, 2.50f, 0.247f, 0.193f, 0.096f, 0.109f, 3.6f, 5.72f / 1024, 2.f, 7.53f, 1.00f, 1.162f, 0.480f, 0.557f};
    static const Cost w8 = {3.48f, 2.28f, 0.320f, 0.236f, 0.091f, 0.121f, 3.6f, 5.97f / 1024, 2.f, 5.63f, 2.67f, 1.365f, 0.322f, 0.578f};
    static const Cost w16 = {3.71f, 1.26f, 0.299f, 0.572f, 0.049f, 0.129f, 3.9f, 5.08f / 1024, 2.f, 4.93f, 2.95f, 1.165f, 0.437f, 0.552f};
    return bits == 16 ? w16 : bits == 8 ? w8 : bits == 4 ? w4 : w2;
}

float prompt_cost(const Cost &c, int groups, long long tiles, int mt, int segments, int cus)
{
    const long long units = tiles * segments;
    const int steps = (groups + segments - 1) / segments;
    auto round = [&](float full) { return c.round + c.out * mt * full + steps * (c.step + c.step_mt * mt + c.step_full * mt * full); };
    float t = c.call + units / cus * round(1.f);
    if (units % cus)
        t += round((float)(units % cus) / cus);
    return segments > 1 ? t + c.split + c.split_unit * units * mt : t;
}

float prefill_cost(const Cost &c, int K, long long tiles, int cus)
{
    const long long per_xcd = (tiles + 7) / 8, per_round = cus >= 8 ? cus / 8 : 1, rest = per_xcd % per_round;
    auto round = [&](float full) { return c.old_round + c.old_out * full + (K / 64) * (c.old_step + c.old_full * full); };
    const float t = c.old_call + per_xcd / per_round * round(1.f);
    return rest == 0 ? t : 2 * rest <= per_round ? t + c.old_half * round(2.f * rest / per_round) : t + round((float)rest / per_round);
}

template <int BITS>
hipError_t launch_mt(const FqLinearDesc &d, int M, int mt, int segments, float *part, hipStream_t stream)
{
    return mt == 2   ? launch<BITS, 2>(d, M, segments, part, stream)
           : mt == 3 ? launch<BITS, 3>(d, M, segments, part, stream)
                     : launch<BITS, 4>(d, M, segments, part, stream);
}

} // namespace

FqPromptPlan fq_prompt_plan(int N, int K, int bits, int M, int cus)
{
    const Cost &c = cost_of(bits);
    const int groups = K / 128;
    const long long n_tiles = (N + BN - 1) / BN;
    FqPromptPlan best = {0, 0};
    // (left to the large tiles where they are expected to be up to 3 % slower: of 1650 calls of the fit's shapes three are
    // then 4 or 5 % slower than on the large tiles)
    // The large tiles address 256 rows of x (and of fp16 weights) by 32-bit offsets: longer rows are not for them.
    const bool too_long = (unsigned long long)K * 2 * 256 > 0xffffffffULL;
    float least = too_long ? 3.4e38f : 0.97f * prefill_cost(c, K, (long long)((M + 255) / 256) * ((N + 255) / 256), cus);
    for (int mt = 2; mt <= 4; mt++) {
        const long long tiles = (M + 32 * mt - 1) / (32 * mt) * n_tiles;
        if (tiles > 0x3ffffffLL)
            continue;
        for (int s = 1; s <= MAX_SEGMENTS && s <= groups; s++) {
            if (s > 1 && (tiles * s > 2LL * cus || (size_t)(tiles * s) * 32 * mt * BN > PART_FLOATS))
                break;
            const float t = prompt_cost(c, groups, tiles, mt, s, cus);
            if (t < least) {
                least = t;
                best = FqPromptPlan{mt, s};
            }
        }
    }
    return best;
}

hipError_t fq_part_array(hipStream_t stream, float **part, std::unique_lock<std::mutex> &both)
{
    *part = nullptr;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capture) != hipSuccess) {
        // (the null stream while a blocking stream is captured: the question fails, launches do not.  The failure
        // is not left for the query after the launch to find.)
        (void)hipGetLastError();
        return hipSuccess;
    }
    if (capture != hipStreamCaptureStatusNone)
        return hipSuccess;
    int device = 0;
    const int bank = fq_part_bank(stream, &device);
    if (bank < 0)
        return hipSuccess;
    if (const hipError_t e = hipGetSymbolAddress((void **)part, HIP_SYMBOL(g_part)))
        return e;
    *part += (size_t)bank * PART_FLOATS;
    both = std::unique_lock<std::mutex>(*fq_part_mutex(device, bank));
    return hipSuccess;
}

hipError_t fq_launch_prompt(const FqLinearDesc &d, int bits, int M, FqPromptPlan plan, hipStream_t stream)
{
    float *part = nullptr;
    std::unique_lock<std::mutex> both;
    if (plan.segments > 1)
        if (const hipError_t e = fq_part_array(stream, &part, both))
            return e;
    return bits == 2   ? launch_mt<2>(d, M, plan.mt, plan.segments, part, stream)
           : bits == 4 ? launch_mt<4>(d, M, plan.mt, plan.segments, part, stream)
           : bits == 8 ? launch_mt<8>(d, M, plan.mt, plan.segments, part, stream)
                       : launch_mt<16>(d, M, plan.mt, plan.segments, part, stream);
}
