// Entropy of softmax(a) and KL(softmax(a) || softmax(b)) per row, one pass.
// Softmax: Sec. 2.3; the entropy is the exponent's argument of the perplexity
// entropy, Sec. 4.2 Eq. (5); the KL divergence is the layer-ranking signal of
// Sec. 3.1 / 4.3, taken between two next-token distributions.
//
// One workgroup per row -- or, for up to 512 long rows (the decode step has one), up to 32
// workgroups per row, one to a piece of it, whose partials meet in a small static device array and are combined
// by whichever workgroup arrives last (one launch either way; a single workgroup needs
// 11 us for one 32000-entry pair, 32 of them 5.9).  Bound by HBM for many rows, by launch and
// latency for few: 5 x 32000 6.1 us, 52 x 32000 in half 8.1 (36 with a fence per partial and a ticket line shared by the rows).
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
__device__ __forceinline__ float4 load4(const float *row, size_t i)
{
    return ld4_nt(reinterpret_cast<const float4 *>(row) + i);
}
__device__ __forceinline__ float4 load4(const _Float16 *row, size_t i)
{
    const half4_t v = __builtin_nontemporal_load((const __attribute__((address_space(1))) half4_t *)row + i);
    return make_float4((float)v.x, (float)v.y, (float)v.z, (float)v.w);
}

// FINE: S and Sb in double.  In binary32 the small terms beside a lane's maximum, whose term is 1, are rounded at 2^-24, most of the
// KL's error once a lane takes more than a vector (relative, 100 x 4096 with 256 threads 6.1e-6, with 1024 4.4e-6, FINE 1.1e-6).  For up to
// 64 rows and for short ones, where a call waits for memory and not for arithmetic (800 x 128256 in half would).
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

// Entries of a row's piece [from, end) (in vectors of four if VEC) that fall to thread t of THREADS: four vectors or, where
// 128-bit loads do not fit the rows, eight entries of a row in flight, in the last round too: its requests past the end repeat the
// piece's last vector and are not added (one after the other, the up to three vectors of a last
// round cost a trip to memory each, as much as everything else where a row is split).
template <int THREADS, bool HAS_B, bool VEC, bool FINE, typename T>
__device__ __forceinline__ void add_entries(Partial<FINE> &p, const T *ar, const T *br, unsigned from, unsigned end, unsigned t)
{
    const float4 none4 = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY); // entries that carry no mass
    unsigned i = from + t;
    if (VEC) {
        auto round = [&](auto full) {
            constexpr bool FULL = decltype(full)::value;
            float4 av[4], bv[4];
#pragma unroll
            for (unsigned j = 0; j < 4; j++) {
                const unsigned at = FULL ? i + j * THREADS : min(i + j * THREADS, end - 1);
                av[j] = load4(ar, at);
                bv[j] = HAS_B ? load4(br, at) : none4;
            }
            if (FULL)
                __builtin_amdgcn_sched_barrier(0); // (else the first sums' waits come ahead of the last requests)
#pragma unroll
            for (unsigned j = 0; j < 4; j += 2) {
                if (!FULL && i + (j + 1) * THREADS >= end)
                    av[j + 1] = bv[j + 1] = none4;
                if (FULL || i + j * THREADS < end)
                    add_pair<HAS_B, FINE>(p, av[j], av[j + 1], bv[j], bv[j + 1]);
            }
        };
        // Whole rounds without a look at the end where arithmetic counts, in half with b (450 x 128256 55.6 -> 51.8 us in four pieces, 256 x
        // 100000 28.9 -> 27.1 in eight; in f32 no gain, without b 200 x 50000 in half 10.4 -> 11.6).
        if (HAS_B && sizeof(T) == 2)
            for (; from + 4 * THREADS <= end; from += 4 * THREADS, i += 4 * THREADS)
                round(std::true_type());
        for (; i < end; i += 4 * THREADS)
            round(std::false_type());
    } else {
        for (; i < end; i += 8 * THREADS) {
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

// Scratch of rows in pieces: partials [row][piece][S, U, D, Sb, m, mb] and arrival tickets, one
// bank per stream (calls on one stream follow one another; calls on different streams use different
// banks): FQ_BANKS for up to 64 rows, then FQ_ROWS_BANKS for more, which are given to fewer streams.  Tickets are
// zero at load and the combining workgroup resets its row's ticket, so every
// launch finds them zero; each has a cache line of its own, because adds to one line are served one
// after the other where the line lives.
constexpr int FINE_ROWS = 64, MAX_SPLIT_ROWS = 512, MAX_SPLITS = 32, MAX_PARTS = 2048, LINE_WORDS = 32;
static_assert(FINE_ROWS * MAX_SPLITS <= MAX_PARTS && MAX_SPLIT_ROWS * 4 <= MAX_PARTS, "what fq_entropy_route gives a call");
__device__ double g_part[FQ_BANKS + FQ_ROWS_BANKS][MAX_PARTS][6];
__device__ __attribute__((aligned(128))) unsigned int g_ticket[FQ_BANKS + FQ_ROWS_BANKS][MAX_SPLIT_ROWS][LINE_WORDS];

// What lane i of a wavefront has of a row's piece i comes together: the row's sums and maxima, in every lane.  More than 64 rows:
// the factors in double, which takes a fifth off the KL's error (with FINE more, but 0.1 us of 6 with it).
template <bool FINE>
__device__ __forceinline__ void merge_pieces(double &S, double &U, double &D, double &Sb, float &gm, float &gmb)
{
    const float pm = gm, pmb = gmb;
    gm = wave_max(pm);
    gmb = wave_max(pmb);
    if (S > 0.0) {
        const float d = pm - gm;
        const double c = FINE ? (double)expf(d) : exp((double)d);
        U = c * (U + (double)d * S);
        S *= c;
        D = c > 0.0 ? c * D : 0.0;
    }
    if (Sb > 0.0)
        Sb *= FINE ? (double)expf(pmb - gmb) : exp((double)(pmb - gmb));
    S = wave_sum(S);
    U = wave_sum(U);
    D = wave_sum(D);
    Sb = wave_sum(Sb);
}

// A row is `pieces` pieces, each summed by a team of THREADS threads.  TEAMS = 1: a workgroup takes one piece, and those of a row
// meet in `bank`.  TEAMS > 1: a workgroup takes a row of TEAMS * PER pieces, PER to a team, which meet in LDS: the same sums in the
// same order, so that a call has the same bits with and without a bank.
template <int THREADS, int TEAMS, int PER, bool HAS_B, bool VEC, bool FINE, typename T>
__global__ __launch_bounds__(THREADS *TEAMS) void entropy_kl_kernel(const T *__restrict__ a, const T *__restrict__ b, int V,
                                                                    int pieces, int bank, float *__restrict__ H,
                                                                    float *__restrict__ KL)
{
    constexpr int WAVES = THREADS / 64;
    __shared__ float s_max[TEAMS][PER][2][WAVES];
    __shared__ double s_sum[TEAMS][PER][4][WAVES];
    __shared__ double s_piece[TEAMS > 1 ? TEAMS * PER : 1][6];

    const int r = TEAMS > 1 ? blockIdx.x : blockIdx.x / pieces;
    const int team = TEAMS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / THREADS) : 0;
    const unsigned first = TEAMS > 1 ? team : blockIdx.x % pieces; // and each TEAMS-th from there
    const unsigned t = threadIdx.x % THREADS;
    const T *ar = a + (size_t)r * V;
    const T *br = HAS_B ? b + (size_t)r * V : ar;

    // (VEC: V % 4 == 0 and rows aligned to four entries; unsigned: a row of nearly 2^31 entries ends within a round of them)
    const unsigned n = VEC ? (unsigned)V >> 2 : (unsigned)V, per = (n + pieces - 1) / pieces;
    Partial<FINE> p[PER];
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const unsigned from = (first + k * TEAMS) * per;
        part_init(p[k]);
        add_entries<THREADS, HAS_B, VEC, FINE>(p[k], ar, br, from, min(n, from + per), t);
    }

    // Maxima over each piece.
    const int wave = t >> 6, lane = t & 63;
    float gm[PER], gmb[PER];
#pragma unroll
    for (int k = 0; k < PER; k++) {
        gm[k] = wave_max(p[k].m), gmb[k] = wave_max(p[k].mb);
        if (lane == 0) {
            s_max[team][k][0][wave] = gm[k];
            s_max[team][k][1][wave] = gmb[k];
        }
    }
    __syncthreads();
    double S[PER], U[PER], D[PER], Sb[PER];
#pragma unroll
    for (int k = 0; k < PER; k++) {
#pragma unroll
        for (int w = 0; w < WAVES; w++) {
            gm[k] = fmaxf(gm[k], s_max[team][k][0][w]);
            gmb[k] = fmaxf(gmb[k], s_max[team][k][1][w]);
        }
        // Rescale this lane's partial to the maxima, then sum in double.
        S[k] = U[k] = D[k] = Sb[k] = 0.0;
        if (p[k].S > 0) {
            const float d = p[k].m - gm[k];
            const double c = (double)expf(d);
            S[k] = c * (double)p[k].S;
            U[k] = c * ((double)p[k].U + (double)d * (double)p[k].S);
            D[k] = c > 0.0 ? c * (double)p[k].D : 0.0;
        }
        if (HAS_B && p[k].Sb > 0)
            Sb[k] = (double)expf(p[k].mb - gmb[k]) * (double)p[k].Sb;
        S[k] = wave_sum(S[k]);
        U[k] = wave_sum(U[k]);
        if (HAS_B) {
            D[k] = wave_sum(D[k]);
            Sb[k] = wave_sum(Sb[k]);
        }
        if (lane == 0) {
            s_sum[team][k][0][wave] = S[k];
            s_sum[team][k][1][wave] = U[k];
            s_sum[team][k][2][wave] = D[k];
            s_sum[team][k][3][wave] = Sb[k];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; k++) {
        S[k] = U[k] = D[k] = Sb[k] = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; w++) {
            S[k] += s_sum[team][k][0][w];
            U[k] += s_sum[team][k][1][w];
            D[k] += s_sum[team][k][2][w];
            Sb[k] += s_sum[team][k][3][w];
        }
    }
    if (TEAMS > 1) {
#pragma unroll
        for (int k = 0; k < PER; k++)
            if (t == 0) {
                double *slot = s_piece[first + k * TEAMS];
                slot[0] = S[k], slot[1] = U[k], slot[2] = D[k], slot[3] = Sb[k], slot[4] = (double)gm[k], slot[5] = (double)gmb[k];
            }
        __syncthreads();
        if (threadIdx.x >= 64)
            return;
        S[0] = U[0] = D[0] = Sb[0] = 0.0;
        gm[0] = gmb[0] = -INFINITY;
        if (lane < pieces) {
            const double *slot = s_piece[lane];
            S[0] = slot[0], U[0] = slot[1], D[0] = slot[2], Sb[0] = slot[3], gm[0] = (float)slot[4], gmb[0] = (float)slot[5];
        }
        merge_pieces<FINE>(S[0], U[0], D[0], Sb[0], gm[0], gmb[0]);
    } else if (pieces > 1) {
        // Publish this workgroup's piece, then see whether it is the last to arrive: one store past the
        // caches, acknowledged before the ticket is taken.  (A fence instead writes back the XCD's whole L2,
        // once per workgroup.)
        if (wave != 0)
            return;
        if (lane < 6)
            __hip_atomic_store(&g_part[bank][r * pieces + first][lane],
                               lane == 0   ? S[0]
                               : lane == 1 ? U[0]
                               : lane == 2 ? D[0]
                               : lane == 3 ? Sb[0]
                               : lane == 4 ? (double)gm[0]
                                           : (double)gmb[0],
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        unsigned int arrived = 0;
        if (lane == 0)
            arrived = __hip_atomic_fetch_add(&g_ticket[bank][r][0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_readfirstlane((int)arrived) != pieces - 1)
            return;
        asm volatile("" ::: "memory");
        // first wavefront of the last workgroup: lane i takes piece i
        S[0] = U[0] = D[0] = Sb[0] = 0.0;
        gm[0] = gmb[0] = -INFINITY;
        if (lane < pieces) {
            const double *slot = g_part[bank][r * pieces + lane];
            S[0] = __hip_atomic_load(&slot[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            U[0] = __hip_atomic_load(&slot[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            D[0] = __hip_atomic_load(&slot[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            Sb[0] = __hip_atomic_load(&slot[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            gm[0] = (float)__hip_atomic_load(&slot[4], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            gmb[0] = (float)__hip_atomic_load(&slot[5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        merge_pieces<FINE>(S[0], U[0], D[0], Sb[0], gm[0], gmb[0]);
        if (lane == 0)
            g_ticket[bank][r][0] = 0u; // ready for the next launch
    }
    if (threadIdx.x == 0) {
        H[r] = (float)(log(S[0]) - U[0] / S[0]);
        if (HAS_B)
            KL[r] = (float)(D[0] / S[0] + ((double)gmb[0] - (double)gm[0]) + log(Sb[0] / S[0]));
    }
}

template <int THREADS, int TEAMS, int PER, bool FINE, typename T>
hipError_t launch(const T *a, const T *b, int R, int V, bool vec, int pieces, int bank, float *H, float *KL, hipStream_t stream)
{
    const dim3 grid((unsigned)R * (TEAMS > 1 ? 1u : (unsigned)pieces)), block(THREADS * TEAMS);
    auto go = [&](auto has_b, auto is_vec) {
        entropy_kl_kernel<THREADS, TEAMS, PER, decltype(has_b)::value, decltype(is_vec)::value, FINE, T>
            <<<grid, block, 0, stream>>>(a, b, V, pieces, bank, H, KL);
        return hipGetLastError();
    };
    typedef std::true_type Yes;
    typedef std::false_type No;
    return b ? vec ? go(Yes(), Yes()) : go(Yes(), No()) : vec ? go(No(), Yes()) : go(No(), No());
}

template <typename T>
hipError_t dispatch(const T *a, const T *b, int R, int V, float *H, float *KL, hipStream_t stream)
{
    if (R == 0)
        return hipSuccess;
    const uintptr_t mask = 4 * sizeof(T) - 1;
    const bool vec = (V % 4 == 0) && (((uintptr_t)a & mask) == 0) && (!b || ((uintptr_t)b & mask) == 0);
    const FqEntropyRoute route = fq_entropy_route(R, V, b != nullptr, sizeof(T) == 2, vec, fq_device_cus());
    const int pieces = route.pieces;
    if (pieces > 1 && R <= FINE_ROWS) {
        const int bank = fq_stream_bank(stream);
        if (bank >= 0)
            return launch<256, 1, 1, true>(a, b, R, V, vec, pieces, bank, H, KL, stream);
        return launch<512, 1, 1, true>(a, b, R, V, vec, 1, 0, H, KL, stream); // (more streams than banks: whole rows)
    }
    if (pieces > 1) { // (without a bank: the same pieces, all of a row in one workgroup)
        const int bank = fq_rows_bank(stream);
        if (bank >= 0)
            return launch<256, 1, 1, false>(a, b, R, V, vec, pieces, FQ_BANKS + bank, H, KL, stream);
        return pieces == 4 ? launch<256, 4, 1, false>(a, b, R, V, vec, 4, 0, H, KL, stream)
                           : launch<256, 4, 2, false>(a, b, R, V, vec, 8, 0, H, KL, stream);
    }
    if (route.threads == 512)
        return route.fine ? launch<512, 1, 1, true>(a, b, R, V, vec, 1, 0, H, KL, stream)
                          : launch<512, 1, 1, false>(a, b, R, V, vec, 1, 0, H, KL, stream);
    return route.fine ? launch<256, 1, 1, true>(a, b, R, V, vec, 1, 0, H, KL, stream)
                      : launch<256, 1, 1, false>(a, b, R, V, vec, 1, 0, H, KL, stream);
}

} // namespace

FqEntropyRoute fq_entropy_route(int R, int V, bool kl, bool half, bool vec, int cus)
{
    const bool many = V >= 65536;
    // One round (4096 entries): whole, 1 x 4000 5.1 us (split 5.7), 64 x 4000 5.3 (6.1).
    if (V <= 4096)
        return {256, 1, R <= MAX_SPLIT_ROWS};
    // R <= 64, by the pieces 8 / 16 / 32: 4 x 32000 6.3 / 6.1 / 5.9, 15 x 32000 6.6 / 6.2 / 6.7, 52 x 32000 8.2 / 9.2 / 11.5, 52 x
    // 128256 14.2 / 14.7 / 13.4; 1 x 32000 whole 11.0; up to 10240 entries 1 x 8000 whole 5.3, in 4 pieces 5.9, 64 x 8000 6.3 and 6.3.
    if (R <= FINE_ROWS) {
        const int pieces = V <= 10240 ? V / 2048 : R <= 8 || many ? MAX_SPLITS : R <= 20 ? 16 : 8;
        return {256, pieces < V / 1024 ? pieces : V / 1024, 1};
    }
    // (With 256 and 512 threads: 300 x 5000 7.2 and 8.0, 512 x 10240 9.9 and 11.2, 128 x 10240 without KL 5.8 and 5.3.)
    if (V <= 10240)
        return {!kl && R <= cus ? 512 : 256, 1, R <= MAX_SPLIT_ROWS};
    // In half 600 x 128256 46.7 with 256 threads and 41.7 with 512, 2048 x 128256 97.1 and 96.7; f32 with KL 100.3 and 105.4.
    if (R > MAX_SPLIT_ROWS)
        return {half && R <= 1536 ? 512 : 256, 1, 0};
    // Rows are split until the chip is full.  us of a call in f32 with KL unless said, whole with 256 / with 512 threads / in 4 / in 8
    // pieces; under 65536 entries:
    //   128 x 32000 14.6 / 11.8 / 10.3 / 11.0, 200 x 32000 15.2 / 12.4 / 14.6 / 14.9, 300 x 32000 18.4 / 20.5 / 17.6, 350 x 12000 9.7 / 10.7 /
    //   12.8, 350 x 50000 27.6 / 30.2 / 29.1, 450 x 32000 20.7 / 22.1 / 23.7 and in half 20.9 / 20.6 / 21.0;
    // from there on:
    //   65 x 128256 45 / 30 / 20.1 / 18.8, 100 x 128256 46 / 32 / 22.2 / 24.1, 160 x 128256 47 / 32 / 33.4 / 31.5, 300 x 128256 57 / 67 / 54, in
    //   half 100 x 128256 45 / 35 / 21.3 / 19.7, 224 x 128256 46 / 36 / 32.2 / 29.7, 480 x 100000 47.5 / 46.0 / 43.8;
    // the same with the whole rows' sums in double, which costs nothing where the chip waits for memory:
    //   200 x 100000 39.5 / 29.5 / 34.6 / 32.7, 256 x 100000 41.0 / 35.1 / 37.9 / 38.4, 400 x 100000 52.6 / 58.3 / 59.6, 512 x 128256 81.4 / 83.5 /
    //   83.9, and where 128-bit loads do not fit the rows 400 x 90001 62.6 / 54.7 / 52.0.
    if (!many)
        return R <= cus * 5 / 8 || (R > cus && R * 256 <= (V >= 24576 ? 350 : 320) * cus) ? FqEntropyRoute{256, 4, 0} : FqEntropyRoute{512, 1, 0};
    if (kl && !half && R > cus * 3 / 4 && R <= cus)
        return {512, 1, 1};
    if (kl && !half && vec && R > cus * 3 / 2)
        return {256, 1, 1};
    return {256, R <= cus && R * 8 <= MAX_PARTS ? 8 : 4, 0};
}

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
