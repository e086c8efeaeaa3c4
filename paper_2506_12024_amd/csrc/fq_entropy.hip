// Entropy of softmax(a) and KL(softmax(a) || softmax(b)) per row, one pass.
// Softmax: Sec. 2.3; the entropy is the exponent's argument of the perplexity
// entropy, Sec. 4.2 Eq. (5); the KL divergence is the layer-ranking signal of
// Sec. 3.1 / 4.3, taken between two next-token distributions.
//
// One workgroup per row -- or, for up to 512 long rows (the decode step has one), up to 32
// workgroups per row whose partials meet in a small static device array and are combined
// by whichever workgroup arrives last (one launch either way; a single workgroup needs
// 11 us for one 32000-entry pair, 32 of them 5.9).  Bound by HBM for many rows, by launch and
// latency for few: 5 x 32000 6.1 us, 52 x 32000 8.2 (36 with a fence per partial and a ticket line shared by the rows).
// Every lane keeps an online (running-max) partial
//   m  = max a_i            S  = sum e^(a_i - m)
//   U  = sum e^(a_i - m) (a_i - m)          D = sum e^(a_i - m) (a_i - b_i)
//   mb = max b_i            Sb = sum e^(b_i - mb)
// over the 128-bit vectors it streams (coalesced, four in flight to the end of the row), in binary32.
// Partials are then rescaled to the row maximum and summed across the
// workgroup in double, and one lane finishes in double:
//   H  = ln S - U / S
//   KL = D / S + (mb - m) + ln(Sb / S)
// so the difference of the two log-sum-exps, which is where binary32 would lose
// the small KL of two nearly equal distributions, never passes through binary32.
#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>
#include <stdint.h>
#include <type_traits>

#include "fq_internal.h"

namespace {

// e^x as one v_exp_f32 of x * log2(e).  The product's rounding moves a term by at most
// |x| * 2^-24 relative; terms that carry weight have |x| < 20 or so, which leaves the sums three
// orders of magnitude inside the 1e-4 the results are held to, and the library routine's
// range handling costs more instructions per element than HBM delivers them.  (So does putting the rounding
// back by two multiply-adds: 800 x 128256 in half 98 -> 141 us, and the KL's error hardly moves.)
#define EXPF(x) __expf(x)

typedef float f32x4 __attribute__((ext_vector_type(4)));
// Streaming load: each logit is read once, so it should not displace anything in the caches.
__device__ __forceinline__ float4 ld4_nt(const float4 *p)
{
    const f32x4 v = __builtin_nontemporal_load((const __attribute__((address_space(1))) f32x4 *)p);
    return make_float4(v.x, v.y, v.z, v.w);
}
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
// Vector i of a row: four consecutive logits widened to binary32 (binary16 widens exactly).
__device__ __forceinline__ float4 load4(const float *row, unsigned i)
{
    return ld4_nt(reinterpret_cast<const float4 *>(row) + i);
}
__device__ __forceinline__ float4 load4(const _Float16 *row, unsigned i)
{
    const half4_t v = __builtin_nontemporal_load((const __attribute__((address_space(1))) half4_t *)row + i);
    return make_float4((float)v.x, (float)v.y, (float)v.z, (float)v.w);
}

// FINE: S and Sb in double.  In binary32 the small terms beside a lane's maximum, whose term is 1, are rounded at 2^-24, most of the
// KL's error once a lane takes more than a vector.  For up to 64 rows, where a call waits for memory and not for
// arithmetic (800 x 128256 in half would).
template <bool FINE>
struct Partial {
    typedef std::conditional_t<FINE, double, float> Sum;
    float m, U, D, mb;
    Sum S, Sb;
};

template <bool FINE>
__device__ __forceinline__ void part_init(Partial<FINE> &p)
{
    p.m = -FLT_MAX;
    p.mb = -FLT_MAX;
    p.U = p.D = 0.0f;
    p.S = p.Sb = 0;
}

template <bool FINE>
__device__ __forceinline__ void raise_max_a(Partial<FINE> &p, float cm)
{
    if (cm > p.m) {
        if (p.S > 0) {
            const float d = p.m - cm;
            const float c = EXPF(d);
            // (c = 0: nothing is left of what was summed.  Logits masked with the type's lowest value get here with d * S
            // and D beyond binary32.)
            p.U = c > 0.0f ? c * (p.U + d * (float)p.S) : 0.0f;
            p.S *= c;
            p.D = c > 0.0f ? c * p.D : 0.0f;
        }
        p.m = cm;
    }
}

template <bool FINE>
__device__ __forceinline__ void raise_max_b(Partial<FINE> &p, float cm)
{
    if (cm > p.mb) {
        if (p.Sb > 0)
            p.Sb *= EXPF(p.mb - cm);
        p.mb = cm;
    }
}

// The eight terms of each sum meet first and join the lane's sum as one: an eighth of the roundings at the sum's size.  KL of near
// distributions against 64 bits, term by term in pieces of 1024 entries / now: 2048 x 128256 (whole rows) 1.6e-5 / 6.7e-6, 300 x
// 128256 7.7e-6 / 5.2e-6; with FINE 52 x 32000 in half 1.9e-6 / 2.2e-6 (in binary32 3.8e-6), 60 x 8000 3.2e-6 / 2.8e-6 (7.2e-6).
template <bool HAS_B, bool FINE>
__device__ __forceinline__ void add_pair(Partial<FINE> &p, const float4 a0, const float4 a1, const float4 b0, const float4 b1)
{
    const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
    const float b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
    auto greatest = [](const float(&v)[8]) {
        return fmaxf(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])), fmaxf(fmaxf(v[4], v[5]), fmaxf(v[6], v[7])));
    };
    auto sum = [](const auto(&v)[8]) { return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7])); };
    raise_max_a(p, greatest(a));
    if (HAS_B)
        raise_max_b(p, greatest(b));
    typename Partial<FINE>::Sum e[8], f[8];
    float u[8], d[8];
#pragma unroll
    for (int i = 0; i < 8; i++) {
        const float t = a[i] - p.m, w = EXPF(t);
        const bool live = w > 0.0f; // 0 (a = -inf or far below the maximum) adds nothing
        e[i] = w;
        u[i] = live ? w * t : 0.0f;
        d[i] = HAS_B && live ? w * (a[i] - b[i]) : 0.0f;
        f[i] = HAS_B ? EXPF(b[i] - p.mb) : 0.0f;
    }
    p.S += sum(e);
    p.U += sum(u);
    if (HAS_B) {
        p.D += sum(d);
        p.Sb += sum(f);
    }
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_xor(v, off, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v = fmaxf(v, __shfl_xor(v, off, 64));
    return v;
}

// Scratch of the split mode: partials [row][split][S, U, D, Sb, m, mb] and arrival tickets, one
// bank per stream (calls on one stream follow one another; calls on different streams use different
// banks): FQ_BANKS for up to 64 rows, then FQ_ROWS_BANKS for more, which are given to fewer streams.  Tickets are zero at load and the combining workgroup resets its row's ticket, so every
// launch finds them zero; each has a cache line of its own, because adds to one line are served one
// after the other where the line lives.
constexpr int FINE_ROWS = 64, MAX_SPLIT_ROWS = 512, MAX_SPLITS = 32, MAX_PARTS = 2048, LINE_WORDS = 32;
static_assert(FINE_ROWS * MAX_SPLITS <= MAX_PARTS && 160 * 12 <= MAX_PARTS && 256 * 8 <= MAX_PARTS && MAX_SPLIT_ROWS * 4 <= MAX_PARTS,
              "what dispatch() gives a call");
__device__ double g_part[FQ_BANKS + FQ_ROWS_BANKS][MAX_PARTS][6];
__device__ __attribute__((aligned(128))) unsigned int g_ticket[FQ_BANKS + FQ_ROWS_BANKS][MAX_SPLIT_ROWS][LINE_WORDS];

template <int THREADS, bool HAS_B, bool VEC, bool FINE, typename T>
__global__ __launch_bounds__(THREADS) void entropy_kl_kernel(const T *__restrict__ a,
                                                             const T *__restrict__ b, int V,
                                                             int splits, int bank, float *__restrict__ H,
                                                             float *__restrict__ KL)
{
    constexpr int WAVES = THREADS / 64;
    __shared__ float s_max[2][WAVES];
    __shared__ double s_sum[4][WAVES];

    const int r = blockIdx.x / splits;
    const unsigned sidx = blockIdx.x % splits; // (unsigned, and what follows: a row of nearly 2^31 entries ends within a round of them)
    const unsigned t = threadIdx.x;
    const T *ar = a + (size_t)r * V;
    const T *br = HAS_B ? b + (size_t)r * V : ar;

    Partial<FINE> p;
    part_init(p);
    const float4 none4 = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY); // entries that carry no mass
    if (VEC) { // V % 4 == 0 and rows aligned to four entries
        const unsigned nvec = (unsigned)V >> 2;
        const unsigned per = (nvec + splits - 1) / splits;
        const unsigned end = min(nvec, (sidx + 1) * per);
        // Four vectors of a row in flight, the last round too: its requests past the end repeat the last vector and
        // are not added (one after the other, the up to three vectors of a last round cost a trip to memory each,
        // as much as everything else where a row is split).
        for (unsigned i = sidx * per + t; i < end; i += 4 * THREADS) {
            float4 av[4], bv[4];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const unsigned at = min(i + j * THREADS, end - 1);
                av[j] = load4(ar, at);
                bv[j] = HAS_B ? load4(br, at) : none4;
            }
#pragma unroll
            for (int j = 0; j < 4; j += 2) {
                if (i + (j + 1) * THREADS >= end)
                    av[j + 1] = bv[j + 1] = none4;
                if (i + j * THREADS < end)
                    add_pair<HAS_B, FINE>(p, av[j], av[j + 1], bv[j], bv[j + 1]);
            }
        }
    } else {
        // Rows that 128-bit loads do not fit: eight entries in flight.
        const unsigned per = ((unsigned)V + splits - 1) / splits;
        const unsigned end = min((unsigned)V, (sidx + 1) * per);
        for (unsigned i = sidx * per + t; i < end; i += 8 * THREADS) {
            float av[8], bv[8];
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const unsigned at = min(i + j * THREADS, end - 1);
                av[j] = (float)ar[at];
                bv[j] = HAS_B ? (float)br[at] : -INFINITY;
            }
#pragma unroll
            for (int j = 1; j < 8; j++)
                if (i + j * THREADS >= end)
                    av[j] = bv[j] = -INFINITY;
            add_pair<HAS_B, FINE>(p, make_float4(av[0], av[1], av[2], av[3]), make_float4(av[4], av[5], av[6], av[7]),
                            make_float4(bv[0], bv[1], bv[2], bv[3]), make_float4(bv[4], bv[5], bv[6], bv[7]));
        }
    }

    // Maxima over the workgroup.
    const int wave = t >> 6, lane = t & 63;
    float gm = wave_max(p.m), gmb = wave_max(p.mb);
    if (lane == 0) {
        s_max[0][wave] = gm;
        s_max[1][wave] = gmb;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; w++) {
        gm = fmaxf(gm, s_max[0][w]);
        gmb = fmaxf(gmb, s_max[1][w]);
    }
    // Rescale this lane's partial to the maxima, then sum in double.
    double S = 0.0, U = 0.0, D = 0.0, Sb = 0.0;
    if (p.S > 0) {
        const float d = p.m - gm;
        const double c = (double)expf(d);
        S = c * (double)p.S;
        U = c * ((double)p.U + (double)d * (double)p.S);
        D = c > 0.0 ? c * (double)p.D : 0.0;
    }
    if (HAS_B && p.Sb > 0)
        Sb = (double)expf(p.mb - gmb) * (double)p.Sb;
    S = wave_sum(S);
    U = wave_sum(U);
    if (HAS_B) {
        D = wave_sum(D);
        Sb = wave_sum(Sb);
    }
    if (lane == 0) {
        s_sum[0][wave] = S;
        s_sum[1][wave] = U;
        s_sum[2][wave] = D;
        s_sum[3][wave] = Sb;
    }
    __syncthreads();
    S = U = D = Sb = 0.0;
#pragma unroll
    for (int w = 0; w < WAVES; w++) {
        S += s_sum[0][w];
        U += s_sum[1][w];
        D += s_sum[2][w];
        Sb += s_sum[3][w];
    }
    if (splits > 1) {
        // Publish this workgroup's partial, then see whether it is the last to arrive: one store past the
        // caches, acknowledged before the ticket is taken.  (A fence instead writes back the XCD's whole L2,
        // once per workgroup.)
        if (wave != 0)
            return;
        if (lane < 6)
            __hip_atomic_store(&g_part[bank][r * splits + sidx][lane],
                               lane == 0   ? S
                               : lane == 1 ? U
                               : lane == 2 ? D
                               : lane == 3 ? Sb
                               : lane == 4 ? (double)gm
                                           : (double)gmb,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        unsigned int arrived = 0;
        if (lane == 0)
            arrived = __hip_atomic_fetch_add(&g_ticket[bank][r][0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_readfirstlane((int)arrived) != splits - 1)
            return;
        asm volatile("" ::: "memory");
        // first wavefront of the last workgroup: lane i takes partial i
        double pm = -INFINITY, pmb = -INFINITY;
        S = U = D = Sb = 0.0;
        if (lane < splits) {
            const double *slot = g_part[bank][r * splits + lane];
            S = __hip_atomic_load(&slot[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            U = __hip_atomic_load(&slot[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            D = __hip_atomic_load(&slot[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            Sb = __hip_atomic_load(&slot[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            pm = __hip_atomic_load(&slot[4], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            pmb = __hip_atomic_load(&slot[5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        gm = wave_max((float)pm);
        gmb = wave_max((float)pmb);
        if (S > 0.0) {
            const float d = (float)pm - gm;
            const double c = (double)expf(d);
            U = c * (U + (double)d * S);
            S *= c;
            D = c > 0.0 ? c * D : 0.0;
        }
        if (Sb > 0.0)
            Sb *= (double)expf((float)pmb - gmb);
        S = wave_sum(S);
        U = wave_sum(U);
        D = wave_sum(D);
        Sb = wave_sum(Sb);
        if (lane == 0)
            g_ticket[bank][r][0] = 0u; // ready for the next launch
    }
    if (t == 0) {
        H[r] = (float)(log(S) - U / S);
        if (HAS_B)
            KL[r] = (float)(D / S + ((double)gmb - (double)gm) + log(Sb / S));
    }
}

template <int THREADS, typename T>
hipError_t launch(const T *a, const T *b, int R, int V, int splits, int bank, float *H, float *KL,
                  hipStream_t stream)
{
    const uintptr_t mask = 4 * sizeof(T) - 1;
    const bool vec = (V % 4 == 0) && (((uintptr_t)a & mask) == 0) && (!b || ((uintptr_t)b & mask) == 0);
    const dim3 grid((unsigned)R * (unsigned)splits), block(THREADS);
    auto go = [&](auto has_b, auto is_vec, auto fine) {
        entropy_kl_kernel<THREADS, decltype(has_b)::value, decltype(is_vec)::value, decltype(fine)::value, T>
            <<<grid, block, 0, stream>>>(a, b, V, splits, bank, H, KL);
        return hipGetLastError();
    };
    typedef std::true_type Yes;
    typedef std::false_type No;
    if (R <= FINE_ROWS)
        return b ? vec ? go(Yes(), Yes(), Yes()) : go(Yes(), No(), Yes()) : vec ? go(No(), Yes(), Yes()) : go(No(), No(), Yes());
    return b ? vec ? go(Yes(), Yes(), No()) : go(Yes(), No(), No()) : vec ? go(No(), Yes(), No()) : go(No(), No(), No());
}

template <typename T>
hipError_t dispatch(const T *a, const T *b, int R, int V, float *H, float *KL, hipStream_t stream)
{
    if (R == 0)
        return hipSuccess;
    // Rows are split until the chip is full, in pieces that are whole rounds of a workgroup's four vectors a lane where that
    // can be had; what a further piece costs is its merge.  us of a call, f32 with KL unless said, whole row / split:
    //   one round (4096 entries): whole, 1 x 4000 5.1 / 5.7, 64 x 4000 5.3 / 6.1;
    //   up to two and a half (10240): 1 x 8000 5.3 / 5.9 (4 pieces), 64 x 8000 6.3 / 6.3 -- in pieces all the same up to 64
    //     rows, for the KL's error, which grows with the terms a lane takes (512 threads for more rows, 100 x 8000 6.3 and with 256
    //     6.4);
    //   R <= 64, by the pieces 8 / 16 / 32: 4 x 32000 6.3 / 6.1 / 5.9, 15 x 32000 6.6 / 6.2 / 6.7, 52 x 32000 8.2 / 9.2 / 11.5, and
    //     52 x 128256 14.2 / 14.7 / 13.4; 1 x 32000 whole 11.0;
    //   R <= 160: 100 x 32000 14.9 / 10.1 (4 pieces; 8: 10.4), 100 x 128256 48.0 / 21.9 (12);
    //   one row a compute unit: 256 x 32000 with 512 threads 13.5, in 4 pieces 15.6; 200 x 128256 in half 34 / 17.0 (8);
    //   R <= 512: 300 x 32000 19.5 / 18.8 (4), 400 x 32000 with 512 threads 21.1 / 22.8; 300 x 128256 62.6 / 52.8 (4), 512 x
    //     128256 82.6 / 82.0, in half 37 / 31.2.
    // (A stream without a bank: whole rows.)
    const bool many = V >= 65536;
    int splits = 1;
    if (V > 4096 && (V > 10240 || R <= FINE_ROWS)) {
        if (V <= 10240)
            splits = V / 2048;
        else if (R <= FINE_ROWS)
            splits = R <= 8 || many ? MAX_SPLITS : R <= 20 ? 16 : 8;
        else if (R <= 160)
            splits = many ? 12 : 4;
        else if (R <= 256)
            splits = many ? 8 : 1;
        else if (R <= MAX_SPLIT_ROWS)
            splits = many || R <= 350 ? 4 : 1;
        if (splits > V / 1024)
            splits = V / 1024;
    }
    if (splits > 1) {
        const bool few = R <= FINE_ROWS;
        const int bank = few ? fq_stream_bank(stream) : fq_rows_bank(stream);
        if (bank >= 0)
            return launch<256, T>(a, b, R, V, splits, few ? bank : FQ_BANKS + bank, H, KL, stream);
    }
    // Whole rows: 256 threads (several rows on a compute unit), 512 where there are few long ones -- up to 512 rows (200 x
    // 32000: 256 threads 15.8, 512 12.5, 1024 13.8), in half up to 1536 (600 x 128256 46.7 and 41.7 us, 2048 x 128256
    // 97.1 and 96.7; f32 with KL 100.3 and 105.4).
    if (V > 4096 && R <= (sizeof(T) == 2 && V > 10240 ? 1536 : 512))
        return launch<512, T>(a, b, R, V, 1, 0, H, KL, stream);
    return launch<256, T>(a, b, R, V, 1, 0, H, KL, stream);
}

} // namespace

hipError_t fq_launch_entropy_kl(const float *a, const float *b, int R, int V, float *H, float *KL,
                                hipStream_t stream)
{
    return dispatch<float>(a, b, R, V, H, KL, stream);
}

hipError_t fq_launch_entropy_kl_f16(const uint16_t *a, const uint16_t *b, int R, int V, float *H,
                                    float *KL, hipStream_t stream)
{
    return dispatch<_Float16>(reinterpret_cast<const _Float16 *>(a), reinterpret_cast<const _Float16 *>(b),
                              R, V, H, KL, stream);
}
