// Output layer fused with what Alg. 1 takes from its logits in every decode step: the next
// token (argmax) and the entropy behind PPLE (Sec. 4.2 Eq. 5, softmax as in Sec. 2.3).
// logits[m][v] = sum_k x[m][k] * W[v][k] for the fp16 output-layer weight W[V][K] and 1 <= M <= 4
// rows of x, accumulated in binary32; the logits never have to travel through HBM (they are
// written only if the caller asks for them).  HBM bound: the weight is read once, 2 bytes per
// entry.
//
// A wavefront takes four vocabulary rows at a time; lane l reads 16 bytes (8 halves) of each at
// k = 512 j + 8 l, j = 0 .. K / 512 - 1 -- one non-temporal 128-bit load per row and j, a
// wavefront load is 1 KiB contiguous -- with the loads of the next DEPTH steps in flight while step j is
// multiplied (v_dot2_f32_f16) against the matching x blocks, which sit in LDS for the whole
// kernel ([j][m][lane], conflict free).  The steps run on from one four rows to the next: begun anew for every four
// rows, with one step in flight and the sums through LDS, short rows and several rows of x waited for memory most (us;
// before and now: 4 x 8192 -> 32000 123 and 109, 1 x 1024 -> 32000 19.9 and 16.8, 2 x 2048 -> 9001 19.2 and 18.1; 1 x 4096 ->
// 32000 47.5 and 46.8, -> 128256 163 and 162, where it is HBM: 6.4 TB/s and the second launch; against it 1 x 512 -> 9001 10.0 and 11.0,
// where most that is in flight lies past the last block: leaving the loop there instead makes 1 x 4096 -> 1000 1.09 times as long).  With 2 and 3 steps the
// last but one takes 1.6 and 0.6 more; with one, three, four workgroups per compute unit instead of two 0, 1.4 and 2.2 more;
// with the requests past a wavefront's last block repeating its last steps instead of one line of x 0.6 more.  The four sums are reduced across the wavefront and
// handed to lanes 0 .. 3, each of which keeps an online softmax state per row of x: running
// maximum and its index, S = sum exp(a - max), U = sum (a - max) exp(a - max).  States meet per
// wavefront, per workgroup (LDS) and per call: every workgroup leaves its partial in a static
// device array and a second, one-workgroup launch combines them, H = ln S - U / S (1 x 4096 -> 32000 46.3 -> 45.1 us with a
// wavefront to a row of x there, 4 x 1024 -> 8000 20.4 -> 12.8).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "fq_internal.h"

namespace {

#define FQ_GLOBAL __attribute__((address_space(1)))

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int THREADS = 256;
constexpr int WAVES = THREADS / 64;
constexpr int RPW = 4;                 // vocabulary rows per wavefront and iteration
constexpr int ROWS_PER_WG = WAVES * RPW;
constexpr int DEPTH = 4;               // steps in flight per wavefront
constexpr int MAX_M = 4;
constexpr int MAX_WGS = 1024;

// Partials [row of x][workgroup]: (max, S, U), index of the max; one bank per stream (the two
// launches of a call follow one another on their stream; calls on different streams use different
// banks).
__device__ __attribute__((aligned(16))) u32x4 g_part[FQ_BANKS][MAX_M][MAX_WGS];

__device__ __forceinline__ float dot8(const u32x4 w, const u32x4 x, float acc)
{
    // whole-vector casts: a bit cast of a single element of an ext_vector loses the other elements
    const half8_t wh = __builtin_bit_cast(half8_t, w), xh = __builtin_bit_cast(half8_t, x);
    acc = __builtin_amdgcn_fdot2(__builtin_shufflevector(wh, wh, 0, 1), __builtin_shufflevector(xh, xh, 0, 1), acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_shufflevector(wh, wh, 2, 3), __builtin_shufflevector(xh, xh, 2, 3), acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_shufflevector(wh, wh, 4, 5), __builtin_shufflevector(xh, xh, 4, 5), acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_shufflevector(wh, wh, 6, 7), __builtin_shufflevector(xh, xh, 6, 7), acc, false);
    return acc;
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp(float v) // (0 in the rows that are masked out)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xF, false));
}

// Sum over the wavefront in vector instructions alone, in every lane: neighbours, quads, halves and rows of 16, then
// (rows 0 + 1) + (rows 2 + 3).
__device__ __forceinline__ float wave_sum(float v)
{
    v += dpp<0xB1, 0xF>(v);  // quad_perm [1,0,3,2]
    v += dpp<0x4E, 0xF>(v);  // quad_perm [2,3,0,1]
    v += dpp<0x141, 0xF>(v); // row_half_mirror
    v += dpp<0x140, 0xF>(v); // row_mirror
    v += dpp<0x142, 0xA>(v); // row_bcast15 into rows 1 and 3
    v += dpp<0x143, 0xC>(v); // row_bcast31 into rows 2 and 3
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// Online softmax state of one row of x.
struct State {
    float mx, S, U;
    int idx;
    __device__ __forceinline__ void init()
    {
        mx = -INFINITY;
        S = 0.f;
        U = 0.f;
        idx = 0x7fffffff;
    }
    __device__ __forceinline__ void add(float a, int v)
    {
        if (a > mx) { // a new maximum: rebase what was summed so far (first element: S = U = 0)
            const float d = mx - a, f = mx == -INFINITY ? 0.f : __expf(d);
            U = mx == -INFINITY ? 0.f : f * (U + d * S);
            S = f * S + 1.f;
            mx = a;
            idx = v;
        } else {
            const float d = a - mx, e = __expf(d);
            S += e;
            U += d * e;
        }
    }
    // Another state's elements join this one's; (larger maximum, then smaller index) decides the
    // maximum.  An empty state has S = 0.
    __device__ __forceinline__ void merge(float omx, float oS, float oU, int oidx)
    {
        if (oS <= 0.f)
            return;
        if (S <= 0.f) {
            mx = omx, S = oS, U = oU, idx = oidx;
            return;
        }
        if (omx > mx || (omx == mx && oidx < idx)) {
            const float d = mx - omx, f = __expf(d);
            U = f * (U + d * S) + oU;
            S = f * S + oS;
            mx = omx;
            idx = oidx;
        } else {
            const float d = omx - mx, f = __expf(d);
            S += f * oS;
            U += f * (oU + d * oS);
        }
    }
    // Butterfly over the lanes whose index differs in the bits of `mask`.
    __device__ __forceinline__ void merge_lanes(int mask)
    {
        for (int off = 1; off <= mask; off <<= 1) {
            if (!(mask & off))
                continue;
            const float omx = __shfl_xor(mx, off, 64), oS = __shfl_xor(S, off, 64), oU = __shfl_xor(U, off, 64);
            const int oidx = __shfl_xor(idx, off, 64);
            merge(omx, oS, oU, oidx);
        }
    }
};

template <int M>
__global__ __launch_bounds__(THREADS) void lm_head_entropy_kernel(const uint16_t *__restrict__ x,
                                                                  const uint16_t *__restrict__ w, int V, int K,
                                                                  int bank, float *__restrict__ logits,
                                                                  float *__restrict__ H, int32_t *__restrict__ argmax)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[]; // x: [K / 512][M][64] blocks of 16 bytes
    __shared__ float s_part[WAVES][M][3];
    __shared__ int s_idx[WAVES][M];
    u32x4 *xs = reinterpret_cast<u32x4 *>(lds_raw);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int J = K >> 9;

    for (int i = threadIdx.x; i < J * M * 64; i += THREADS) {
        const int l = i & 63, m = (i >> 6) % M, j = (i >> 6) / M;
        xs[i] = *(const FQ_GLOBAL u32x4 *)(x + (size_t)m * K + (size_t)j * 512 + l * 8);
    }
    __syncthreads();

    State st[M];
#pragma unroll
    for (int m = 0; m < M; m++)
        st[m].init();

    // Items (row block, step), DEPTH of them in flight in registers, run through the row blocks: while a block's sums are
    // reduced, the next block's first steps are on their way.
    const int nblocks = (V + ROWS_PER_WG - 1) / ROWS_PER_WG;
    u32x4 in[DEPTH][RPW];
    const FQ_GLOBAL u32x4 *wp[RPW];
    int ib = blockIdx.x, ij = 0; // the next item to request
    auto rows_of = [&](int rb) {
#pragma unroll
        for (int r = 0; r < RPW; r++) // rows past V repeat row V - 1 and are dropped below
            wp[r] = (const FQ_GLOBAL u32x4 *)(w + (size_t)min((long long)rb * ROWS_PER_WG + wave * RPW + r, (long long)V - 1) * K) + lane;
    };
    auto request = [&](u32x4 (&to)[RPW]) {
#pragma unroll
        for (int r = 0; r < RPW; r++)
            to[r] = __builtin_nontemporal_load(wp[r] + ij * 64);
        asm volatile("" ::: "memory"); // (where it is issued, not where it is used)
        if (++ij == J) {
            ij = 0;
            ib += gridDim.x;
            if (ib < nblocks) {
                rows_of(ib);
            } else { // past the last block: one line of x, so that every path has the same requests in flight
#pragma unroll
                for (int r = 0; r < RPW; r++)
                    wp[r] = (const FQ_GLOBAL u32x4 *)x;
            }
        }
    };
    rows_of(ib);
#pragma unroll
    for (int d = 0; d < DEPTH; d++)
        request(in[d]);
    float acc[RPW][M];
#pragma unroll
    for (int r = 0; r < RPW; r++)
#pragma unroll
        for (int m = 0; m < M; m++)
            acc[r][m] = 0.f;
    int rb = blockIdx.x, j = 0; // the item being multiplied
    while (rb < nblocks) {
#pragma unroll
        for (int d = 0; d < DEPTH; d++) {
            if (rb < nblocks) {
#pragma unroll
                for (int m = 0; m < M; m++) {
                    const u32x4 xv = xs[(j * M + m) * 64 + lane];
#pragma unroll
                    for (int r = 0; r < RPW; r++)
                        acc[r][m] = dot8(in[d][r], xv, acc[r][m]);
                }
            }
            request(in[d]);
            if (++j < J || rb >= nblocks)
                continue;
#pragma unroll
            for (int m = 0; m < M; m++) {
                float mine = 0.f;
#pragma unroll
                for (int r = 0; r < RPW; r++) {
                    const float s = wave_sum(acc[r][m]);
                    if (lane == r)
                        mine = s;
                    acc[r][m] = 0.f;
                }
                const int v = rb * ROWS_PER_WG + wave * RPW + lane;
                if (lane < RPW && v < V) {
                    st[m].add(mine, v);
                    if (logits)
                        logits[(size_t)m * V + v] = mine;
                }
            }
            j = 0;
            rb += gridDim.x;
        }
    }

    // lanes 0 .. RPW - 1 of every wavefront -> lane 0 -> LDS -> the first wavefront -> the
    // workgroup's partial in the static array; binary32 throughout (v_exp_f32 for the rescaling)
#pragma unroll
    for (int m = 0; m < M; m++) {
        if (lane >= RPW)
            st[m].init();
        st[m].merge_lanes(RPW - 1);
        if (lane == 0) {
            s_part[wave][m][0] = st[m].mx;
            s_part[wave][m][1] = st[m].S;
            s_part[wave][m][2] = st[m].U;
            s_idx[wave][m] = st[m].idx;
        }
    }
    __syncthreads();
    if (wave != 0)
        return;
    State wg[M];
#pragma unroll
    for (int m = 0; m < M; m++) {
        wg[m].init();
        if (lane < WAVES) {
            wg[m].mx = s_part[lane][m][0];
            wg[m].S = s_part[lane][m][1];
            wg[m].U = s_part[lane][m][2];
            wg[m].idx = s_idx[lane][m];
        }
        wg[m].merge_lanes(WAVES - 1);
        if (lane == 0 && bank < 0) { // the call's only workgroup
            H[m] = (float)(log((double)wg[m].S) - (double)wg[m].U / (double)wg[m].S);
            if (argmax)
                argmax[m] = wg[m].idx;
        } else if (lane == 0) {
            g_part[bank][m][blockIdx.x] = u32x4{__builtin_bit_cast(uint32_t, wg[m].mx), __builtin_bit_cast(uint32_t, wg[m].S),
                                                __builtin_bit_cast(uint32_t, wg[m].U), (uint32_t)wg[m].idx};
        }
    }
}

// Second launch (one workgroup): merges the workgroups' partials.  Measured against a ticket that lets the last
// workgroup do it behind a fence, which writes back an L2 per workgroup: 50 us for 1024 workgroups, more than the whole
// weight stream.  A ticket without one (partials stored past the caches and acknowledged, as fq_entropy.hip hands its own
// over) has not been measured here; what it could save is this launch, 3.8 to 4.6 us of a call.
// One wavefront to a row of x, PER partials to a lane, all requested together; the maximum first, then the sums, in double
// (4 x 1024 -> 8000: 3.8 us of a call of 12.8; 10.4 of 20.4 with one partial to each of 1024 threads, states merged pair by
// pair through the wavefront, LDS and once more).
template <int PER>
__global__ __launch_bounds__(64 * MAX_M) void lm_head_combine_kernel(int parts, int bank, float *__restrict__ H,
                                                                     int32_t *__restrict__ argmax)
{
    const int lane = threadIdx.x & 63, m = threadIdx.x >> 6;
    u32x4 p[PER];
#pragma unroll
    for (int i = 0; i < PER; i++)
        p[i] = g_part[bank][m][min(i * 64 + lane, parts - 1)];
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < PER; i++)
        mx = fmaxf(mx, __builtin_bit_cast(float, (uint32_t)p[i].x));
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
        mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    double S = 0.0, U = 0.0;
    int idx = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const float pm = __builtin_bit_cast(float, (uint32_t)p[i].x), pS = __builtin_bit_cast(float, (uint32_t)p[i].y),
                    pU = __builtin_bit_cast(float, (uint32_t)p[i].z);
        if (i * 64 + lane >= parts)
            continue;
        const float d = pm - mx;
        const double f = (double)expf(d);
        S += f * (double)pS;
        U += f > 0.0 ? f * ((double)pU + (double)d * (double)pS) : 0.0;
        if (pm == mx)
            idx = min(idx, (int)p[i].w);
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        S += __shfl_xor(S, off, 64);
        U += __shfl_xor(U, off, 64);
        idx = min(idx, __shfl_xor(idx, off, 64));
    }
    if (lane == 0) {
        H[m] = (float)(log(S) - U / S);
        if (argmax)
            argmax[m] = idx;
    }
}

int device_cus() { return fq_device_cus(); }

template <int M>
hipError_t launch(const uint16_t *x, const uint16_t *w, int V, int K, float *logits, float *H, int32_t *argmax,
                  hipStream_t stream)
{
    const size_t lds = (size_t)M * K * 2;
    if (lds > 48 * 1024) {
        hipError_t e = fq_raise_dynamic_lds((const void *)lm_head_entropy_kernel<M>, 64 * 1024);
        if (e != hipSuccess)
            return e;
    }
    const int nblocks = (V + ROWS_PER_WG - 1) / ROWS_PER_WG;
    int grid = 2 * device_cus();
    if (grid > MAX_WGS)
        grid = MAX_WGS;
    if (grid > nblocks)
        grid = nblocks;
    const int bank = fq_stream_bank(stream);
    if (bank < 0 && stream == hipStreamPerThread) { // more threads than banks: one workgroup, which needs none
        lm_head_entropy_kernel<M><<<1, THREADS, lds, stream>>>(x, w, V, K, bank, logits, H, argmax);
        return hipGetLastError();
    }
    if (bank < 0) // more streams than banks of partial results have used this call on this device
        return hipErrorOutOfMemory;
    lm_head_entropy_kernel<M><<<grid, THREADS, lds, stream>>>(x, w, V, K, bank, logits, nullptr, nullptr);
    static_assert(MAX_WGS == 16 * 64, "partials of a lane");
    if (grid <= 512)
        lm_head_combine_kernel<8><<<1, 64 * M, 0, stream>>>(grid, bank, H, argmax);
    else
        lm_head_combine_kernel<16><<<1, 64 * M, 0, stream>>>(grid, bank, H, argmax);
    return hipGetLastError();
}

} // namespace

hipError_t fq_launch_lm_head_entropy(const void *x, const void *w, int M, int V, int K, float *logits, float *H,
                                     int32_t *argmax, hipStream_t stream)
{
    const uint16_t *xp = (const uint16_t *)x, *wp = (const uint16_t *)w;
    switch (M) {
    case 1:
        return launch<1>(xp, wp, V, K, logits, H, argmax, stream);
    case 2:
        return launch<2>(xp, wp, V, K, logits, H, argmax, stream);
    case 3:
        return launch<3>(xp, wp, V, K, logits, H, argmax, stream);
    default:
        return launch<4>(xp, wp, V, K, logits, H, argmax, stream);
    }
}
