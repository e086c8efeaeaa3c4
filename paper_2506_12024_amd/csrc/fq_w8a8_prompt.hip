// W8A8 linear for prompts of some tens to some hundreds of tokens (Sec. 4.1, 4.3): the products of
// fq_w8a8.hip -- groups of 128, or one scale per weight row -- for shapes that do not give that kernel's
// tiles of 192 or 256 tokens x 256 rows a compute unit each (300 x 13824 -> 5120: 40 tiles, 176 us).
//
// Split.  A workgroup (8 wavefronts, four along the rows, two along the tokens) takes 64, 128 or 192 tokens x
// 128 weight rows and one of up to 16 segments of K; the segments' sums -- binary32 for groups of 128, exact
// int32 with one scale per row -- meet in the stream's array and a second launch adds them in order
// (fq_prompt.hip, whose slab layout, block-wise metadata and cost model this kernel shares).  300 x 13824 -> 5120:
// 128 tokens, two segments, 56 us; one scale per row 160 -> 43 us.
//
// Groups of 128: a step is one group; a tile's chain of four v_mfma_i32_32x32x32_i8 is interleaved with the fold
// of the tile before it, out += s * float(sum), eight vector instructions to an MFMA; the last tile of a step
// is folded under the first chain of the next one, so that with one block of tokens per wavefront the two pipes
// still overlap.  The zero points' part runs on v_mfma_f32_32x32x2_f32, two groups at a time.
//
// What bounds it: a step of 128 tokens takes about 0.75 us, and no pipe is busy for most of it (MFMAs 0.21, the
// fold's 128 vector instructions a SIMD 0.24, side by side): the operand reads, scales, zero points and group sums all
// stand between the step's barrier and its first MFMA.  With one scale per row the LDS reads and the fetch (0.45 us);
// with few steps the launch, the first fetch and the hand-over of the partial sums.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "fq_internal.h"
#include "fq_mfma.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int THREADS = 512;
constexpr int WAVES = 8;
constexpr int BN = 128;  // weight rows of a tile: 32 per wavefront
constexpr int BK = 128;  // bytes of a row per step: one quantization group
constexpr int MB = 8;    // groups per block of scales, zero points and group sums
constexpr int WL = BN * BK / 16 / THREADS;
constexpr int MAX_SEGMENTS = 16;

struct Args {
    const uint8_t *codes;
    const float *scales;
    const uint8_t *zeros;
    const int8_t *xq;
    const float *sx;
    const int32_t *xsum;
    uint16_t *y;
    int M, N, K;
};

// TM: 32-token blocks per wavefront; a tile is 64 * TM tokens x 128 rows.  ROW: one scale per weight row.
template <int TM, bool ROW>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void w8a8_prompt_kernel(
    const Args d, int m_tiles, int n_tiles, int units, int per_xcd, int segments, int serial, float *part)
{
    constexpr int BM = 64 * TM;
    constexpr int XST = BM * BK, WST = BN * BK;
    constexpr int XL = XST / 16 / THREADS; // = TM
    constexpr int OPS = XL + WL;
    typedef typename std::conditional<ROW, int, float>::type sum_t; // what a tile's sums are kept in
    __shared__ __attribute__((aligned(1024))) uint8_t xs0[XST], xs1[XST], xs2[XST], ws0[WST], ws1[WST], ws2[WST];
    __shared__ __attribute__((aligned(1024))) float ms[ROW ? 1 : 2 * BN * MB];    // [block parity][row][group]
    __shared__ __attribute__((aligned(1024))) uint32_t mz[ROW ? 1 : 2 * BN * MB];
    __shared__ __attribute__((aligned(1024))) int32_t mx[2 * MB * BM];            // [block parity][group][token]
    __shared__ int32_t xtot[ROW ? BM : 1];

    const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || unit >= units)
        return;
    const int tiles = m_tiles * n_tiles;
    const int tile = serial ? unit : unit % tiles;
    const int seg0 = serial ? 0 : unit / tiles, seg1 = serial ? segments : seg0 + 1;
    const int m0 = (tile % m_tiles) * BM, n0 = (tile / m_tiles) * BN;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int l32 = lane & 31, c = lane >> 5;
    const int wn = wave & 3, wm = wave >> 2;
    const uint32_t K = (uint32_t)d.K, G = K >> 7;
    const int x_last = d.M - 1 - m0, w_last = d.N - 1 - n0;
    const uint32_t x_rows = (uint32_t)(min(x_last, BM - 1) + 1), w_rows = (uint32_t)(min(w_last, BN - 1) + 1);
    const __amdgpu_buffer_rsrc_t xbuf = buffer_of(d.xq + (size_t)m0 * K, x_rows * K);
    const __amdgpu_buffer_rsrc_t wbuf = buffer_of(d.codes + (size_t)n0 * K, w_rows * K);
    const __amdgpu_buffer_rsrc_t sbuf = buffer_of(d.scales + (size_t)n0 * G, w_rows * G * 4);
    const __amdgpu_buffer_rsrc_t zbuf = buffer_of(d.zeros + (size_t)n0 * G, w_rows * G);
    const __amdgpu_buffer_rsrc_t gbuf = buffer_of(d.xsum + m0, (G * (uint32_t)d.M - (uint32_t)m0) * 4);

    const int row = wn * 32 + l32; // weight row
    int aofs[4], bofs[4];          // piece 2 i + c of a row: k = 32 i + 16 c .. of the step
#pragma unroll
    for (int i = 0; i < 4; i++) {
        aofs[i] = wm * TM * 32 * BK + w_offset<BK>(l32, 2 * i + c);
        bofs[i] = w_offset<BK>(row, 2 * i + c);
    }
    uint32_t xoff[XL], woff[WL];
#pragma unroll
    for (int i = 0; i < XL; i++) {
        int r, b;
        w_piece<BK>(i * WAVES + wave, lane, r, b);
        xoff[i] = (uint32_t)min(r, x_last) * K + b;
    }
#pragma unroll
    for (int i = 0; i < WL; i++) {
        int r, b;
        w_piece<BK>(i * WAVES + wave, lane, r, b);
        woff[i] = (uint32_t)min(r, w_last) * K + b;
    }
    // Scales and zero points as in the fp16 kernel (slot j of row r holds group j ^ (r >> 3 & 7)); the tokens'
    // group sums: wavefront w fetches group w of the block.
    const uint32_t mgrp = (uint32_t)((lane & 7) ^ (wave & 7));
    uint32_t mrow[2], mtok[TM];
#pragma unroll
    for (int i = 0; i < 2; i++)
        mrow[i] = (uint32_t)min((i * 8 + wave) * 8 + (lane >> 3), w_last) * G;
#pragma unroll
    for (int i = 0; i < TM; i++)
        mtok[i] = (uint32_t)min(i * 64 + lane, x_last) * 4;
    auto fetch_meta = [&](uint32_t gb, int buf) {
        if (!ROW) {
#pragma unroll
            for (int i = 0; i < 2; i++) {
                const uint32_t at = mrow[i] + min(gb + mgrp, G - 1);
                load_to_lds<4>(sbuf, ms + buf * BN * MB + (i * 8 + wave) * 64, at * 4, 0);
                load_to_lds<1>(zbuf, mz + buf * BN * MB + (i * 8 + wave) * 64, at, 0);
            }
        }
        const uint32_t g = min(gb + wave, G - 1);
#pragma unroll
        for (int i = 0; i < TM; i++)
            load_to_lds<4>(gbuf, mx + buf * MB * BM + wave * BM + i * 64, mtok[i], g * (uint32_t)d.M * 4);
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
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    typedef std::integral_constant<int, 2> I2;
    typedef std::integral_constant<int, OPS> IN;

    sum_t total[TM][16];
    for (int seg = seg0; seg < seg1; seg++) {
        const int g0 = (int)((long long)seg * G / segments), g1 = (int)((long long)(seg + 1) * G / segments);
        const int ng = g1 - g0;
        // groups of 128: the folded groups and the zero points' part, in one sum.  (In sums of their own, added up at the end,
        // they are both large where zero points lie off the middle, as in groups with an outlier, and cancel: 300 x 13824 ->
        // 5120, one weight in a thousand 20 times larger, results up to 4.6e-6 of their rms beyond the rounding to fp16
        // instead of 1.1e-6; the same 56 us.)
        float16_t out[TM];
        v16i acc[ROW ? TM : 2];
#pragma unroll
        for (int t = 0; t < TM; t++)
#pragma unroll
            for (int v = 0; v < 16; v++)
                out[t][v] = 0.f;
#pragma unroll
        for (int t = 0; t < (ROW ? TM : 2); t++)
#pragma unroll
            for (int v = 0; v < 16; v++)
                acc[t][v] = 0;
        auto fetch = [&](int t, auto st) {
            const uint32_t g = (uint32_t)(g0 + min(t, ng - 1)) * BK; // (clamped: always issued, the waits count them)
#pragma unroll
            for (int i = 0; i < XL; i++)
                load_to_lds<16>(xbuf, stage_x(st) + (i * WAVES + wave) * 1024, xoff[i], g);
#pragma unroll
            for (int i = 0; i < WL; i++)
                load_to_lds<16>(wbuf, stage_w(st) + (i * WAVES + wave) * 1024, woff[i], g);
        };
        fetch_meta(g0, 0);
        fetch(0, I0());
        fetch(1, I1());
        wait_vm(IN());
        barrier();

        // The fold of a group's last tile runs under the first MFMAs of the next step: `prev_s` is its scale (0
        // ahead of the first step).  A pair of groups' zero-point terms is one v_mfma_f32_32x32x2_f32 per tile: A =
        // the tokens' group sums (k = lane / 32), B = s * (128 - z) of the weight row.
        float prev_s = 0.f, az_first[TM], bz_first = 0.f;
        int xt = 0; // ROW: thread t < BM sums the group sums of token t
#pragma unroll
        for (int t = 0; t < TM; t++)
            az_first[t] = 0.f;
        auto step = [&](int t, auto st, auto odd) {
            constexpr int ST = decltype(st)::value;
            constexpr bool ODD = decltype(odd)::value;
            typedef std::integral_constant<int, (ST + 2) % 3> NEXT2;
            const uint8_t *xc = stage_x(st), *wc = stage_w(st);
            v4i a[2][4], b[4];
            auto read_a = [&](int tt) {
#pragma unroll
                for (int i = 0; i < 4; i++)
                    a[tt & 1][i] = *reinterpret_cast<const v4i *>(xc + tt * 32 * BK + aofs[i]);
            };
#pragma unroll
            for (int i = 0; i < 4; i++)
                b[i] = *reinterpret_cast<const v4i *>(wc + bofs[i]);
            read_a(0);
            float s = 0.f, az[TM], bz = 0.f;
            const int buf = (t >> 3) & 1;
            if (!ROW) {
                const int at = buf * BN * MB + row * MB + ((t & 7) ^ ((row >> 3) & 7));
                s = ms[at];
                bz = s * (float)(128 - (int)mz[at]);
#pragma unroll
                for (int tt = 0; tt < TM; tt++)
                    az[tt] = (float)mx[buf * MB * BM + (t & 7) * BM + (wm * TM + tt) * 32 + l32]; // |.| <= 128 * 127: exact
            } else if ((t & 7) == 0 && threadIdx.x < BM) {
#pragma unroll
                for (int j = 0; j < MB; j++)
                    xt += t + j < ng ? mx[buf * MB * BM + j * BM + threadIdx.x] : 0;
            }
            __builtin_amdgcn_sched_barrier(0);
            if ((t & 7) == 0 && t + MB < ng)
                fetch_meta(g0 + t + MB, buf ^ 1);
            fetch(t + 2, NEXT2());
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; i++) // stored code q -> signed byte q - 128
                b[i] = b[i] ^ (int)0x80808080;
#pragma unroll
            for (int tt = 0; tt < TM; tt++) {
                if (tt + 1 < TM)
                    read_a(tt + 1);
                if (ROW) {
#pragma unroll
                    for (int i = 0; i < 4; i++)
                        acc[tt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[tt & 1][i], b[i], acc[tt], 0, 0, 0);
                    continue;
                }
                constexpr int FLIP = ODD && (TM & 1) ? 1 : 0;
                v16i &mine = acc[ROW ? 0 : (tt + FLIP) & 1], &last = acc[ROW ? 0 : (tt + FLIP + 1) & 1];
                v16i r = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                for (int i = 0; i < 4; i++)
                    r = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[tt & 1][i], b[i], r, 0, 0, 0);
                const float fs = tt == 0 ? prev_s : s;
#pragma unroll
                for (int v = 0; v < 16; v++)
                    out[tt == 0 ? TM - 1 : tt - 1][v] += fs * (float)last[v];
                mine = r;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); // one MFMA
                    __builtin_amdgcn_sched_group_barrier(0x002, 8, 0); // eight vector instructions
                }
                if (ODD)
                    out[tt] = __builtin_amdgcn_mfma_f32_32x32x2f32(c ? az[tt] : az_first[tt], c ? bz : bz_first, out[tt], 0, 0, 0);
                else
                    az_first[tt] = az[tt];
                asm volatile("" : "+v"(out[tt == 0 ? TM - 1 : tt - 1]), "+v"(a[0][0]), "+v"(a[1][0]));
            }
            prev_s = s;
            bz_first = bz;
            wait_vm(IN());
            barrier();
        };
        int t = 0;
        for (; t + 6 <= ng; t += 6) {
            step(t, I0(), std::false_type());
            step(t + 1, I1(), std::true_type());
            step(t + 2, I2(), std::false_type());
            step(t + 3, I0(), std::true_type());
            step(t + 4, I1(), std::false_type());
            step(t + 5, I2(), std::true_type());
        }
        if (t < ng)
            step(t, I0(), std::false_type());
        if (t + 1 < ng)
            step(t + 1, I1(), std::true_type());
        if (t + 2 < ng)
            step(t + 2, I2(), std::false_type());
        if (t + 3 < ng)
            step(t + 3, I0(), std::true_type());
        if (t + 4 < ng)
            step(t + 4, I1(), std::false_type());
        __builtin_amdgcn_s_waitcnt(0);
        if (!ROW) {
            // the last step's last tile, and the zero points of an unpaired last group
            const bool last = !((ng & 1) && (TM & 1)); // which accumulator holds it
#pragma unroll
            for (int v = 0; v < 16; v++)
                out[TM - 1][v] += prev_s * (float)(last ? acc[1][v] : acc[0][v]);
            if (ng & 1)
#pragma unroll
                for (int tt = 0; tt < TM; tt++)
                    out[tt] = __builtin_amdgcn_mfma_f32_32x32x2f32(c ? 0.f : az_first[tt], c ? 0.f : bz_first, out[tt], 0, 0, 0);
#pragma unroll
            for (int tt = 0; tt < TM; tt++)
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    const sum_t w = (sum_t)out[tt][v];
                    total[tt][v] = seg == seg0 ? w : total[tt][v] + w;
                }
        } else {
            if (threadIdx.x < BM)
                xtot[threadIdx.x] = xt;
            __syncthreads();
            const int zn = (int)d.zeros[min(n0 + row, d.N - 1)] - 128;
#pragma unroll
            for (int tt = 0; tt < TM; tt++)
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    const sum_t w = (sum_t)(acc[tt][v] - zn * xtot[(wm * TM + tt) * 32 + 8 * (v >> 2) + 4 * c + (v & 3)]);
                    total[tt][v] = seg == seg0 ? w : total[tt][v] + w;
                }
        }
        if (seg + 1 < seg1)
            __syncthreads(); // slabs, sums and blocks are free again
    }
    // D layout of the 32x32 MFMA: lane holds column l32 (weight row), rows (tokens) 8 * (v / 4) + 4 * (lane / 32) + v % 4.
    if (!serial && segments > 1) {
        sum_t *o = (sum_t *)part + ((size_t)(seg0 * tiles + tile) * WAVES + wave) * TM * 1024 + lane * 4;
        typedef sum_t sum4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int tt = 0; tt < TM; tt++)
#pragma unroll
            for (int q = 0; q < 4; q++)
                *(FQ_GLOBAL sum4 *)(o + tt * 1024 + q * 256) =
                    sum4{total[tt][4 * q], total[tt][4 * q + 1], total[tt][4 * q + 2], total[tt][4 * q + 3]};
        return;
    }
    const int n = n0 + row;
    const float sn = ROW ? d.scales[min(n, d.N - 1)] : 1.f;
    // The tokens' scales, all requested ahead of the first store: a load among the stores waits for the stores ahead of it, and
    // the next stores for the load (1455 x 512 -> 22912 with one scale per row 79 -> 53 us).  Rows past M are beyond the buffer's end.
    const __amdgpu_buffer_rsrc_t sxbuf = buffer_of(d.sx, (uint32_t)d.M * 4);
    uint32_t sx[TM][16];
#pragma unroll
    for (int tt = 0; tt < TM; tt++)
#pragma unroll
        for (int v = 0; v < 16; v++)
            sx[tt][v] = __builtin_amdgcn_raw_buffer_load_b32(sxbuf, (m0 + (wm * TM + tt) * 32 + 8 * (v >> 2) + 4 * c + (v & 3)) * 4, 0, 0);
#pragma unroll
    for (int tt = 0; tt < TM; tt++)
#pragma unroll
        for (int v = 0; v < 16; v++) {
            const int m = m0 + (wm * TM + tt) * 32 + 8 * (v >> 2) + 4 * c + (v & 3);
            const float sxm = __builtin_bit_cast(float, sx[tt][v]);
            if (m < d.M && n < d.N)
                ((FQ_GLOBAL uint16_t *)d.y)[(size_t)m * d.N + n] = __builtin_bit_cast(
                    uint16_t, (_Float16)(ROW ? sxm * (sn * (float)total[tt][v]) : sxm * (float)total[tt][v]));
        }
}

// Adds the segments' sums in the order of the segments.  A workgroup takes one wavefront's block of 32 tokens x 32
// weight rows.
template <int TM, bool ROW>
__global__ __launch_bounds__(256) void w8a8_prompt_reduce_kernel(const float *part, const float *sx, const float *scales,
                                                                 uint16_t *y, int M, int N, int m_tiles, size_t seg_words,
                                                                 int segments)
{
    typedef typename std::conditional<ROW, int, float>::type sum_t;
    typedef sum_t sum4 __attribute__((ext_vector_type(4)));
    const int tt = blockIdx.x % TM, wave = blockIdx.x / TM % WAVES, tile = blockIdx.x / (TM * WAVES);
    const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const sum_t *p = (const sum_t *)part + (size_t)blockIdx.x * 1024 + threadIdx.x * 4;
    sum4 v = *(const FQ_GLOBAL sum4 *)p;
#pragma unroll 4
    for (int s = 1; s < segments; s++)
        v += *(const FQ_GLOBAL sum4 *)(p + s * seg_words);
    const int n = tile / m_tiles * BN + (wave & 3) * 32 + (lane & 31);
    const int m = tile % m_tiles * 64 * TM + ((wave >> 2) * TM + tt) * 32 + 8 * q + 4 * (lane >> 5);
    if (n >= N)
        return;
    const float sn = ROW ? scales[n] : 1.f;
    float sxm[4];
#pragma unroll
    for (int r = 0; r < 4; r++)
        sxm[r] = sx[min(m + r, M - 1)];
#pragma unroll
    for (int r = 0; r < 4; r++)
        if (m + r < M)
            ((FQ_GLOBAL uint16_t *)y)[(size_t)(m + r) * N + n] = __builtin_bit_cast(
                uint16_t, (_Float16)(ROW ? sxm[r] * (sn * (float)v[r]) : sxm[r] * (float)v[r]));
}

template <int TM, bool ROW>
hipError_t launch(const Args &d, int segments, float *part, hipStream_t stream)
{
    const int m_tiles = (d.M + 64 * TM - 1) / (64 * TM), n_tiles = (d.N + BN - 1) / BN, tiles = m_tiles * n_tiles;
    const int serial = segments > 1 && !part;
    const int units = tiles * (serial ? 1 : segments), per_xcd = (units + 7) / 8;
    w8a8_prompt_kernel<TM, ROW><<<(unsigned)per_xcd * 8, THREADS, 0, stream>>>(d, m_tiles, n_tiles, units, per_xcd, segments,
                                                                               serial, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || segments == 1 || serial)
        return e;
    w8a8_prompt_reduce_kernel<TM, ROW><<<(unsigned)tiles * WAVES * TM, 256, 0, stream>>>(
        part, d.sx, d.scales, d.y, d.M, d.N, m_tiles, (size_t)tiles * 64 * TM * BN, segments);
    return hipGetLastError();
}

// Microseconds a call is expected to take, fitted to 9000 timings of forced plans (16 to 2048 tokens, 512 to 28672 rows, K
// 128 to 28672; 10 and 12 % off on average, large tiles 9 and 11; a hand-over 1.2 more than fitted, for the host: a second
// launch).  The ends of the tiles of either size have become shorter since, and the constants are from before: over 246 calls of
// those ranges, each under every plan, the choice takes 1.3 (groups) and 1.4 % (per row) more than the best one on average,
// 86 % of them within 3 %, one in ten over 4 and the worst 13; few inputs are the worst of all, 1455 x 512 -> 22912 with one
// scale per row 54.5 us in small tiles and 46.3 in the large ones.  A
// round's end grows with its outputs: without that, and fitted from K = 1024 on, the model took three rounds of 192 x 128
// tiles for two of 128 x 256 over few inputs (2048 x 128 .. 1536 -> 8192: 1.09 to 1.19 of the large tiles' time).
struct Cost {
    float call, round, out, step, step_tm, step_full, split, split_unit;
};
constexpr Cost GROUP_COST = {4.66f, 1.99f, 2.22f, 0.188f, 0.225f, 0.068f, 3.0f, 5.45f / 1024};
constexpr Cost ROW_COST = {4.80f, 1.52f, 2.36f, 0.272f, 0.101f, 0.075f, 3.5f, 4.93f / 1024};

float prompt_cost(const Cost &c, int groups, long long tiles, int tm, int segments, int cus)
{
    const long long units = tiles * segments;
    const int steps = (groups + segments - 1) / segments;
    auto round = [&](float full) { return c.round + c.out * tm * full + steps * (c.step + c.step_tm * tm + c.step_full * tm * full); };
    float t = c.call + units / cus * round(1.f);
    if (units % cus)
        t += round((float)(units % cus) / cus);
    return segments > 1 ? t + c.split + c.split_unit * units * tm : t;
}

// The large tiles: mt as the launcher chooses it (groups of 128), 256 tokens with the last rounds halved (per row).
float large_cost(int N, int K, int M, bool per_row, int mt, int cus)
{
    const long long n_tiles = (N + 255) / 256, bm = per_row ? 256 : 64 * mt, tiles = (M + bm - 1) / bm * n_tiles;
    const int groups = K / 128;
    if (!per_row) {
        auto round = [&](float full) { return 8.58f + 2.74f * mt * full + groups * (0.136f + 0.639f * mt + 0.009f * mt * full); };
        const float t = 2.75f + tiles / cus * round(1.f);
        return tiles % cus ? t + round((float)(tiles % cus) / cus) : t;
    }
    const long long per_xcd = (tiles + 7) / 8, per_round = cus >= 8 ? cus / 8 : 1, rest = per_xcd % per_round;
    auto round = [&](float full) { return 14.f + 9.16f * full + groups * (1.704f + 0.046f * full); };
    const float t = 3.07f + per_xcd / per_round * round(1.f);
    return rest == 0 ? t : 2 * rest <= per_round ? t + 0.552f * round(2.f * rest / per_round) : t + round((float)rest / per_round);
}

} // namespace

FqPromptPlan fq_w8a8_prompt_plan(int N, int K, int M, bool per_row, int large_mt, int cus)
{
    const Cost &c = per_row ? ROW_COST : GROUP_COST;
    const int groups = K / 128;
    const long long n_tiles = (N + BN - 1) / BN;
    FqPromptPlan best = {0, 0};
    const bool too_long = fq_w8a8_too_long(K);
    if ((unsigned long long)groups * (unsigned long long)M * 4 > 0x7fffffffULL) // the group sums' 32-bit offsets
        return best;
    // (left to the large tiles where they are expected to be up to 5 or 12 % slower: of 1050 calls of the fit's shapes two,
    // over 128 and 256 inputs, are then 6 and 9 % slower than on the large tiles)
    float least = too_long ? 3.4e38f : (per_row ? 0.95f : 0.88f) * large_cost(N, K, M, per_row, large_mt, cus);
    for (int tm = 1; tm <= 3; tm++) {
        const long long tiles = ((long long)M + 64 * tm - 1) / (64 * tm) * n_tiles;
        if (tiles > 0x3ffffffLL)
            continue;
        for (int s = 1; s <= MAX_SEGMENTS && s <= groups; s++) {
            if (s > 1 && (tiles * s > 2LL * cus || (size_t)(tiles * s) * 64 * tm * BN > FQ_PART_FLOATS))
                break;
            const float t = prompt_cost(c, groups, tiles, tm, s, cus);
            if (t < least) {
                least = t;
                best = FqPromptPlan{tm, s};
            }
        }
    }
    return best;
}

hipError_t fq_launch_w8a8_prompt(const FqLinearDesc &l, const void *xq, const float *sx, const int32_t *xsum, int M,
                                 bool per_row, FqPromptPlan plan, hipStream_t stream)
{
    float *part = nullptr;
    std::unique_lock<std::mutex> both;
    if (plan.segments > 1)
        if (const hipError_t e = fq_part_array(stream, &part, both))
            return e;
    const Args d = {l.codes8, l.scales8, l.zeros8, (const int8_t *)xq, sx, xsum, l.y, M, l.N, l.K};
    if (per_row)
        return plan.mt == 1   ? launch<1, true>(d, plan.segments, part, stream)
               : plan.mt == 2 ? launch<2, true>(d, plan.segments, part, stream)
                              : launch<3, true>(d, plan.segments, part, stream);
    return plan.mt == 1   ? launch<1, false>(d, plan.segments, part, stream)
           : plan.mt == 2 ? launch<2, false>(d, plan.segments, part, stream)
                          : launch<3, false>(d, plan.segments, part, stream);
}
