// A decode step in the order a decoder must issue it, in ONE launch (batch 1).
//
// A token's linears are not independent: the output projection needs the attention's result, the
// down projection needs gate and up (Alg. 1's decode loop walks them in order).  Issued as one
// launch per dependent group, a 7B-shaped step is 128 launches of 2 to 14 microseconds of weight
// streaming each (Sec. 4.1: the decode phase is bound by loading the weights), and the gaps, ramps
// and tails between them cost more than the streaming.  This kernel keeps one persistent grid
// resident for the whole step: the plan's entries carry a stage number, stages run in order, and
// between two stages the workgroups wait for each other's rows instead of for a kernel boundary.  The weights do not
// depend on x: a wavefront requests the first of the next stage's while it waits.
//
// Roles.  A workgroup (one per compute unit) has CW compute wavefronts and one service wavefront.
//   compute   walks its items -- (4 rows, one slice of K), as in the one-launch kernel -- of a stage with P items of
//             weights in flight, of which PRE are requested before x is there.  Finished rows go to LDS, not to
//             memory, and are announced in a counter there.
//   service   per stage: sums and writes the workgroup's finished rows to y with write-through stores.
// x is staged into LDS by all wavefronts together (one 16-byte block or a few per thread, read at agent scope so that
// no cache of this XCD can answer with an older use of the buffer).
//
// Shares.  In a stage every workgroup serves exactly one entry: the workgroups are dealt to the
// stage's entries in proportion to their cost (rows x K x bit-width, from the device-side
// bit-width array), and an entry's 4-row chunks are dealt evenly to its workgroups.  So a stage
// needs one x per workgroup, staged once.
//
// Between two stages, where every x of the next is the y of one entry of the last (a decoder's chain; the host finds
// out, fq_staged_src.h): the data is the signal.  When the launch begins, every workgroup fills its rows of such ys with a
// half that no finished row holds (UNWRITTEN), and a workgroup that wants an x reads it until no half of it is
// unwritten.  Rows stored -> rows seen is then one way to memory and one read, instead of the store's acknowledgement, an
// arrival, a poll and a read of x one after the other.  The launch's first boundary is always the barrier below: it
// is also what has everyone's rows cleared before anyone polls.
//
// Otherwise, a grid barrier: 128 arrival counters, each on a cache line of its own, count up through the launch:
// after its rows of stage s are acknowledged workgroup b adds one to counter b % 128 (adds to one
// counter are served one after the other where the counter lives, 80 ns each: with a single counter
// the last of 256 arrivals is 20 us late, with two workgroups per counter it does not show; an
// arrival word per workgroup, stored or added, made the polls four times as large and the stage
// slower), and a poll reads all the counters, two per lane, against what they must have reached
// by then.  One more word is the abort flag.
//
// Either wait is bounded: a wavefront that has polled `wait_limit` times raises the abort flag and, if it is the first,
// adds one to a sticky count; every waiter looks at the flag and every workgroup leaves the
// kernel, all of it ahead of one stage: what a wavefront that gives up leaves in LDS is the stage it was to enter (as a plain
// flag it could be read by the service wavefront still in the stage before, which then counted its workgroup out
// while the others were waiting yet, to raise the abort flag behind its being put back).  The last workgroup out (one more counter) puts the counters and the flag back to zero,
// so that the next launch, and a replayed HIP graph, find them clean.  All workgroups must be
// resident together (the host launches at most as many as fit).
//
// Measured (7B-shaped stack in a chain, us per step, bits from {4, 8} / all 4 / all 8): 1170 / 975 / 1348; with the grid barrier at
// every stage 1310 / 1117 / 1501.  The bytes alone take 762 at the best read rate.  x polled, rows announced
// ahead of the next request and the places of their sums worked out in advance are worth a tenth (1488 -> 1344 at {4, 8} when
// requests ran on through the stages), the requests of a stage held back until the one before is done another (1344 -> 1161 in that
// run): requested as items were consumed, all of a stage's bytes had to be asked for in its compute part (6.1 us at memory speed) and
// none while the boundary was crossed (4).  Without the arithmetic (results invalid) 1076 / 848 / 1292.  A stage of 9.1 us: 4.9
// until the last wavefront is done (mean 4.1), 3.3 from the last workgroup's last row to the next x in LDS, the rest spread.
//
// Arithmetic: the item code of the one-launch kernel (fq_gemv.h).  A row whose slices are shared
// by two wavefronts is the sum, in wavefront order, of their partial sums: deterministic, the same
// whether the stage runs alone or after others, but not the one-launch kernel's order of additions.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/flexq.h"
#include "fq_internal.h"
#include "fq_gemv.h"
#include "fq_mfma.h"
#include "fq_staged_src.h"

namespace {

constexpr int CW = 8;                  // compute wavefronts per workgroup
constexpr int THREADS = (CW + 1) * 64; // + the service wavefront: up to three wavefronts per SIMD, 168 registers each
constexpr int P = 3;                   // items in flight per compute wavefront (register sets) ...
constexpr int PRE = 2;                 // ... of which so many are requested ahead of a stage's x.  7B-shaped step, us, for
                                       // P / PRE: 2/2 1180, 2/1 1178, 3/2 1161, 3/1 1217, 4/2 1225 (3/3 1230 and 4/4 1276
                                       // where 2/2 took 1207); 11 compute wavefronts, 2/2: 1192.  x returns behind all that
                                       // the compute unit has outstanding, so requests beyond what memory serves
                                       // while the boundary is crossed anyway only delay it
constexpr int XU = 3;                  // 16-byte blocks of x a thread fetches before it places them

// What a workgroup does in one stage.  64 bytes, kept in LDS for every stage of the plan.
struct Share {
    const uint8_t *codes; // the copy selected by the entry's bit-width (fp16 weights for 16)
    const float *scales;
    const uint8_t *zeros;
    const uint16_t *x;
    uint16_t *y;
    int N, K;
    int c0, c1; // this workgroup's 4-row chunks of the entry
    int mode;   // bit-width (0: nothing to do in this stage), POLL_ bits
    uint32_t inv; // ceil(2^32 / slices of K), 0 for one slice: dividing an item's number by them is a multiplication (i x slices < 2^32)
};
constexpr int POLL_X = 256;      // x is polled
constexpr int POLL_Y = 512;      // y will be polled by the next stage
constexpr int POLL_STAGE = 1024; // no grid barrier ahead of this stage (set for workgroups without a share of it too)
static_assert(sizeof(Share) == 64, "Share is read from LDS as four 16-byte pieces");
static_assert(CW <= 15, "a wavefront's number fits four bits");

// Relative cost of one row of one quantization group of an entry; 0: no such width, or no copy of it.
__device__ __forceinline__ long long group_cost(const FqLinearDesc &d, int bits)
{
    const void *copy = bits == 2    ? (const void *)d.codes2
                       : bits == 3  ? (const void *)d.codes3
                       : bits == 4  ? (const void *)d.codes4
                       : bits == 8  ? (const void *)d.codes8
                       : bits == 16 ? (const void *)d.w16
                                    : nullptr;
    return copy ? staged_group_cost(bits) : 0;
}

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Workgroup barrier that leaves vector memory loads in flight: LDS traffic of this wavefront done,
// then s_barrier (no fence: __syncthreads() would wait for vmcnt(0)).
__device__ __forceinline__ void wg_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xc07f); // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Waits until every compute wavefront has left its rows of stages 0 .. s in LDS (`rows` counts them).
__device__ __forceinline__ void wait_rows(int *rows, int s)
{
    while (uni(__hip_atomic_load(rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < CW * (s + 1))
        __builtin_amdgcn_s_sleep(0);
    asm volatile("" ::: "memory");
}

// A share out of a register: lane l holds word l & 15 of it, so that one LDS read, far ahead, serves the entry into a stage.
struct ShareReg {
    uint32_t v;
    __device__ __forceinline__ explicit ShareReg(const Share *sh) { v = reinterpret_cast<const uint32_t *>(sh)[threadIdx.x & 15]; }
    __device__ __forceinline__ int word(int i) const { return __builtin_amdgcn_readlane((int)v, i); }
    template <class T>
    __device__ __forceinline__ T *ptr(int i) const { return (T *)((uint64_t)(uint32_t)word(i + 1) << 32 | (uint32_t)word(i)); }
    __device__ __forceinline__ const uint8_t *codes() const { return ptr<const uint8_t>(0); }
    __device__ __forceinline__ const float *scales() const { return ptr<const float>(2); }
    __device__ __forceinline__ const uint8_t *zeros() const { return ptr<const uint8_t>(4); }
    __device__ __forceinline__ const uint16_t *x() const { return ptr<const uint16_t>(6); }
    __device__ __forceinline__ uint16_t *y() const { return ptr<uint16_t>(8); }
    __device__ __forceinline__ int N() const { return word(10); }
    __device__ __forceinline__ int K() const { return word(11); }
    __device__ __forceinline__ int c0() const { return word(12); }
    __device__ __forceinline__ int c1() const { return word(13); }
    __device__ __forceinline__ int bits() const { return word(14) & 255; }
    __device__ __forceinline__ bool has(int poll) const { return (word(14) & poll) != 0; }
    __device__ __forceinline__ int over_slices(int i) const { return word(15) ? (int)__umulhi((uint32_t)i, (uint32_t)word(15)) : i; }
};

// What one lane holds for one item in flight: 16 bytes of codes (12 at 3 bits) of each of the 4 rows, and its part
// of the item's scales and zero points, which are fetched TRANSPOSED: a slice touches GS = 32 / 16 /
// 8 groups of a row (2 / 3 and 4 / 8 bits), so (4 rows x GS groups) fit one or two loads of the wavefront
// -- lane l fetches row l / GS, group l % GS -- instead of one load per row and lane; the lanes pick their rows'
// values out of the other lanes (ds_bpermute) when the item is computed.
template <int BITS>
struct Item {
    uint4 w[ROWS_PER_WAVE];
    float s[BITS == 2 ? 2 : 1];
    uint8_t z[BITS == 2 ? 2 : 1]; // kept as bytes: widened where used, so that nothing touches a register while its load is in flight
};

// A compute wavefront's part of a stage.  The workgroup's items -- its chunks of 4 rows in order, inside a chunk
// the slices of K in order -- are cut into CW equal runs, one per compute wavefront, so a chunk's slices may be
// shared by neighbouring wavefronts (a stage often gives a workgroup fewer chunks than it has wavefronts).  The share is
// read through buffer descriptors that end with it: a request past the run, or past the matrix's last row, asks beyond
// the descriptor's end and costs no access, so that every step issues the same loads and the compiler's count of the loads
// in flight holds.  Uniform over the wavefront.
constexpr uint32_t BEYOND = 0xF0000000u; // an offset past every descriptor's end, and not past 2^32 with what is added to it
static_assert(FQ_STAGED_CHUNKS * 4ull * FQ_MAX_DECODE_K * 2 < BEYOND && BEYOND + 5ull * FQ_MAX_DECODE_K * 2 < 1ull << 32,
              "a share at 16 bits is below BEYOND, a row's offset beside it in range");
constexpr int MAX_SLICES = FQ_MAX_DECODE_K / (64 * 8); // of K in a row: 64 at 16 bits, fewer at the others
static_assert((long long)FQ_STAGED_CHUNKS * MAX_SLICES * (CW + 1) < 1 << 30, "a share's items times wavefronts are an int");
template <int BITS>
struct Run {
    __amdgpu_buffer_rsrc_t codes, scales, zeros;
    int K, nslice, end; // items of the run: up to `end`, counted from the share's first
    uint32_t row_bytes, G;

    __device__ __forceinline__ Run(const ShareReg &sh, int rows, int nslice_, int end_) : K(sh.K()), nslice(nslice_), end(end_)
    {
        row_bytes = BITS == 3 ? ((uint32_t)K >> 3) * 3u : (uint32_t)K * BITS / 8;
        G = (uint32_t)K >> 7;
        const size_t row0 = (size_t)sh.c0() * ROWS_PER_WAVE;
        codes = buffer_of(sh.codes() + row0 * row_bytes, (uint32_t)rows * row_bytes);
        scales = buffer_of(sh.scales() + (BITS == 16 ? 0 : row0 * G), BITS == 16 ? 0 : (uint32_t)rows * G * 4);
        zeros = buffer_of(sh.zeros() + (BITS == 16 ? 0 : row0 * G), BITS == 16 ? 0 : (uint32_t)rows * G);
    }

    // First k of this lane in slice j: a lane past the row's end repeats its last block (the lane's x is zero there).
    __device__ __forceinline__ uint32_t lane_k(int j) const
    {
        constexpr int CODES = BITS == 3 ? 32 : 128 / BITS;
        return min((uint32_t)(j * 64 + (int)(threadIdx.x & 63)) * CODES, (uint32_t)K - CODES);
    }
    static constexpr int GSH = BITS == 2 ? 5 : BITS == 8 ? 3 : 4; // log2(groups per slice)

    // The loads of slice j of chunk c (relative to the share's first); item: its number.
    __device__ __forceinline__ void issue(int item, int c, int j, Item<BITS> &L) const
    {
        const int lane = threadIdx.x & 63;
        const uint32_t row0 = (uint32_t)c * ROWS_PER_WAVE;
        const uint32_t k0 = lane_k(j);
        const uint32_t at = (item < end ? row0 * row_bytes : BEYOND) + (BITS == 3 ? (k0 >> 5) * 12u : k0 * BITS / 8);
#pragma unroll
        for (int r = 0; r < ROWS_PER_WAVE; r++) {
            if (BITS == 3) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b96(codes, (int)(at + (uint32_t)r * row_bytes), 0, 2);
                L.w[r] = make_uint4(v[0], v[1], v[2], 0u);
            } else {
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(codes, (int)(at + (uint32_t)r * row_bytes), 0, 2);
                L.w[r] = make_uint4(v.x, v.y, v.z, v.w);
            }
        }
        if (BITS != 16) {
            // lane l -> (row l >> GSH, group l & (GS - 1)) of the slice; at 2 bits the second load takes rows 2 and 3
            const uint32_t g = min(((uint32_t)j << GSH) + (uint32_t)(lane & ((1 << GSH) - 1)), G - 1);
            const uint32_t i0 = (row0 + (uint32_t)(lane >> GSH)) * G + g;
#pragma unroll
            for (int h = 0; h < (BITS == 2 ? 2 : 1); h++) {
                const uint32_t i = i0 + (uint32_t)(2 * h) * G;
                const bool ask = item < end && (BITS != 8 || lane < 32);
                L.s[h] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(scales, (int)(ask ? 4 * i : BEYOND), 0, 0));
                L.z[h] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(zeros, (int)(ask ? i : BEYOND), 0, 0);
            }
        }
        // the loads stay here: the compiler would otherwise sink some of them towards their first use,
        // steps later, where their latency is no longer hidden
        asm volatile("" ::: "memory");
    }

    // The item as the shared arithmetic takes it: every lane gets the scale and zero point of its own
    // group for each of the four rows from the lane that fetched them.
    __device__ __forceinline__ void expand(const Item<BITS> &I, int j, Loaded &L) const
    {
        const int gi = (int)(lane_k(j) >> 7) - (j << GSH); // my group's place among the slice's groups
#pragma unroll
        for (int r = 0; r < ROWS_PER_WAVE; r++) {
            L.w[r] = I.w[r];
            if (BITS == 16)
                continue;
            const int src = (((BITS == 2 ? r & 1 : r) << GSH) + gi) << 2, h = BITS == 2 ? r >> 1 : 0;
            L.s[r] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src, __builtin_bit_cast(int, I.s[h])));
            L.z[r] = (uint8_t)__builtin_amdgcn_ds_bpermute(src, (int)I.z[h]);
        }
    }
};

// Layout of the plan's sync words (ints): the abort flag, the sticky count of launches that gave
// up, flags (bit 0: an entry's bit-width is not attached to its layer, its y was left untouched;
// bit 1: a share too large for the results buffer), on the next line the count of finished
// workgroups, and from SY_COUNTERS on the NC arrival counters, CSTRIDE ints apart.
constexpr int NC = 128;     // arrival counters (workgroup b adds to counter b % NC)
constexpr int CSTRIDE = 32; // ints between two counters: a line each
constexpr int CPL = (NC + 63) / 64;  // counters a polling lane watches
static_assert(NC >= 1 && CPL <= 4, "a lane polls up to four counters");
constexpr int SY_ABORT = 0, SY_GAVE_UP = 1, SY_FLAGS = 2, SY_DONE = 32, SY_COUNTERS = 64;
static_assert((SY_COUNTERS + NC * CSTRIDE) * 4 <= FQ_STAGED_SYNC_BYTES, "the sync words fit the plan's workspace");

// What a wavefront that waits for data needs to know about the launch.
struct Wait {
    int *sync;
    long long limit;
    int *leave; // LDS: the stage ahead of which the workgroup leaves the kernel
    int stage;  // the one whose x is waited for
};
constexpr int NEVER = 0x7fffffff;

// A half that no finished row holds: what a polled y is filled with when a launch begins.  (A NaN whose bits are
// all ones is stored as another NaN.)
constexpr uint32_t UNWRITTEN = 0xFFFFu;

__device__ __forceinline__ bool unwritten(const u32x4 v)
{
    typedef uint16_t ushort2_t __attribute__((ext_vector_type(2)));
    auto h = [](uint32_t w) { return __builtin_bit_cast(ushort2_t, w); };
    const uint32_t m = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_elementwise_max(h(v.x), h(v.y)),
                                                                              __builtin_elementwise_max(h(v.z), h(v.w))));
    return (m & 0xFFFFu) == UNWRITTEN || m >> 16 == UNWRITTEN;
}

// Four blocks of 16 bytes of x per lane, at agent scope: served where the other XCDs' write-through stores have
// arrived, whatever this XCD's caches still hold of an earlier use of the buffer.  The wait is part of the block, so
// that the compiler, which counts the loads in flight, knows of no load here: with loads of its own in the
// loops below it waits for everything ahead of every item.
__device__ __forceinline__ void load_blocks(const uint16_t *x, const uint32_t (&at)[4], u32x4 (&v)[4])
{
    asm volatile("global_load_dwordx4 %0, %4, %8 sc1\n\t"
                 "global_load_dwordx4 %1, %5, %8 sc1\n\t"
                 "global_load_dwordx4 %2, %6, %8 sc1\n\t"
                 "global_load_dwordx4 %3, %7, %8 sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
                 : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "s"(x)
                 : "memory");
}
__device__ __forceinline__ void load_blocks(const uint16_t *x, const uint32_t (&at)[3], u32x4 (&v)[3])
{
    asm volatile("global_load_dwordx4 %0, %3, %6 sc1\n\t"
                 "global_load_dwordx4 %1, %4, %6 sc1\n\t"
                 "global_load_dwordx4 %2, %5, %6 sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2])
                 : "v"(at[0]), "v"(at[1]), "v"(at[2]), "s"(x)
                 : "memory");
}

// True: the wait is over, the launch is aborted.  After `limit` rounds the first to give up raises the abort
// flag and counts the launch; everyone who waits looks at the flag from time to time.
__device__ __forceinline__ bool give_up(const Wait &w, long long round)
{
    int up = 0;
    const uint32_t zero = 0;
    if (round >= w.limit) {
        if ((threadIdx.x & 63) == 0)
            asm volatile("global_atomic_swap %0, %1, %2, %3 offset:%4 sc0 sc1\n\ts_waitcnt vmcnt(0)"
                         : "=&v"(up) : "v"(zero), "v"(1), "s"(w.sync), "n"(SY_ABORT * 4) : "memory");
        if ((threadIdx.x & 63) == 0 && up == 0)
            asm volatile("global_atomic_add %0, %1, %2 offset:%3 sc1\n\ts_waitcnt vmcnt(0)"
                         : : "v"(zero), "v"(1), "s"(w.sync), "n"(SY_GAVE_UP * 4) : "memory");
        up = 1;
    } else if ((round & 63) == 63) {
        asm volatile("global_load_dword %0, %1, %2 offset:%3 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(up) : "v"(zero), "s"(w.sync), "n"(SY_ABORT * 4) : "memory");
    }
    if (uni(up)) {
        *w.leave = w.stage;
        return true;
    }
    return false;
}

// NB blocks of x per lane (block numbers b[]; zeros from block `end` on).  poll: they are being written; read again
// until no half is unwritten.
template <int NB>
__device__ __forceinline__ void fetch_blocks(const uint16_t *x, const int (&b)[NB], int end, uint4 (&out)[NB], bool poll, const Wait &w)
{
    uint32_t at[NB];
    u32x4 v[NB];
#pragma unroll
    for (int u = 0; u < NB; u++)
        at[u] = b[u] < end ? 16u * (uint32_t)b[u] : 0u; // (past the end: the first block once more)
    for (long long round = 0;; round++) {
        load_blocks(x, at, v);
        bool bad = false;
#pragma unroll
        for (int u = 0; u < NB; u++)
            bad = bad || unwritten(v[u]);
        if (!poll || __builtin_amdgcn_ballot_w64(bad) == 0 || give_up(w, round))
            break;
    }
#pragma unroll
    for (int u = 0; u < NB; u++)
        out[u] = b[u] < end ? make_uint4(v[u].x, v[u].y, v[u].z, v[u].w) : make_uint4(0, 0, 0, 0);
}

// x of one entry into LDS in the layout of its bit-width, by all THREADS threads of the workgroup:
// XU blocks per thread are requested before the first is placed, so a row of up to 12288 inputs
// costs one memory round trip and three blocks' worth of placing per thread.  poll: x is being written.
template <int BITS>
__device__ __forceinline__ void stage_x_all(const uint16_t *x, int K, uint4 *lds, bool poll, const Wait &w)
{
    const int tid = threadIdx.x;
    const int Kp = padded_k(K, BITS);
    if (BITS == 3) {
        const int nls = Kp >> 5; // lane slices of 32 k, one per thread and trip
        float2 *sums = reinterpret_cast<float2 *>(lds + (Kp >> 3));
        for (int ls = tid; ls < nls; ls += THREADS) {
            uint4 v[4];
            const int b[4] = {4 * ls, 4 * ls + 1, 4 * ls + 2, 4 * ls + 3};
            fetch_blocks(x, b, K >> 3, v, poll, w);
            place_slice3(ls, v, lds, sums);
        }
        return;
    }
    if (BITS == 2) {
        const int npair = Kp >> 4; // a multiple of 256
        float2 *sums = reinterpret_cast<float2 *>(lds + (Kp >> 3));
        for (int base = 0; base < npair; base += THREADS * 2) {
            const int pb = base + tid, pc = pb + THREADS;
            const int b[4] = {2 * pb, 2 * pb + 1, 2 * pc, 2 * pc + 1};
            uint4 v[4];
            fetch_blocks(x, b, K >> 3, v, poll, w);
            if ((pb & ~63) < npair) // uniform over the wavefront: npair is a multiple of 64
                place_pair2(pb, v[0], v[1], lds, sums);
            if ((pc & ~63) < npair)
                place_pair2(pc, v[2], v[3], lds, sums);
        }
        return;
    }
    const int nblk = Kp >> 3; // a multiple of 64
    float *sums = reinterpret_cast<float *>(lds + nblk);
    for (int base = 0; base < nblk; base += THREADS * XU) {
        uint4 v[XU];
        int at[XU];
#pragma unroll
        for (int u = 0; u < XU; u++)
            at[u] = base + u * THREADS + tid;
        fetch_blocks(x, at, K >> 3, v, poll, w);
#pragma unroll
        for (int u = 0; u < XU; u++) {
            const int b = base + u * THREADS + tid;
            if ((b & ~63) < nblk) // uniform over the wavefront
                place_block<BITS>(b, v[u], lds, sums);
        }
    }
}

__device__ __forceinline__ void stage_share_x(const ShareReg &sh, uint4 *xbuf, const Wait &w)
{
    const int bits = sh.bits();
    if (bits == 0)
        return;
    const uint16_t *x = sh.x();
    const int K = sh.K();
    const bool poll = sh.has(POLL_X);
    if (bits == 2)
        stage_x_all<2>(x, K, xbuf, poll, w);
    else if (bits == 3)
        stage_x_all<3>(x, K, xbuf, poll, w);
    else if (bits == 4)
        stage_x_all<4>(x, K, xbuf, poll, w);
    else if (bits == 8)
        stage_x_all<8>(x, K, xbuf, poll, w);
    else
        stage_x_all<16>(x, K, xbuf, poll, w);
}

// Rows finished in a stage, LDS -> y.  A row's value is the sum, in wavefront order, of the partial sums of the
// wavefronts that shared its chunk (mostly one).  Where they lie is worked out ahead of the stage's end (plan_rows),
// while the service wavefront has nothing else to do: worked out afterwards it kept the rows back for 1.2 us.
struct Rows {
    int first[2]; // the row's first partial sum, for the lane's first two rows (lane, 64 + lane)
    int more[2];  // wavefronts (w << 4 | w_last) that add to it, none if w > w_last
    int rows, n, nslice; // rows (0: nothing to do) and items of the share
    uint16_t *y;         // its first row
};

// Item i of a share of n belongs to the wavefront whose run [n w / CW, n (w + 1) / CW) holds it.
__device__ __forceinline__ int wave_of(int i, int n) { return min((int)(((uint32_t)i * CW + (CW - 1)) / (uint32_t)n), CW - 1); }

__device__ __forceinline__ int row_first(int i, int n, int nslice, int PK, int &more)
{
    const int c = i / ROWS_PER_WAVE, r = i % ROWS_PER_WAVE; // chunk relative to the share's first
    const int w = wave_of(c * nslice, n), w_last = wave_of((c + 1) * nslice - 1, n);
    more = (w + 1) << 4 | w_last;
    return (w * PK + (c - n * w / CW / nslice)) * ROWS_PER_WAVE + r; // its run begins in chunk (n w / CW) / nslice
}

__device__ __forceinline__ void plan_rows(const ShareReg &sh, int PK, Rows &R)
{
    const int bits = sh.bits(), c0 = sh.c0(), c1 = sh.c1();
    R.rows = 0;
    if (bits == 0)
        return;
    R.y = sh.y() + c0 * ROWS_PER_WAVE;
    R.rows = min(c1 * ROWS_PER_WAVE, sh.N()) - c0 * ROWS_PER_WAVE;
    R.nslice = (sh.K() + slice_span(bits) - 1) / slice_span(bits);
    R.n = (c1 - c0) * R.nslice; // (at most FQ_STAGED_CHUNKS x MAX_SLICES)
#pragma unroll
    for (int u = 0; u < 2; u++)
        R.first[u] = row_first(min(64 * u + (int)(threadIdx.x & 63), R.rows - 1), R.n, R.nslice, PK, R.more[u]);
}

// The stores write through to memory (visible to the other XCDs' caches once acknowledged).
__device__ __forceinline__ void store_rows(const float *part, int PK, const Rows &R)
{
    auto put = [&](int i, int first, int more) {
        float v = part[first];
        for (int w = more >> 4; w <= (more & 15); w++)
            if (R.n * (w + 1) / CW > R.n * w / CW) // (fewer items than wavefronts: some runs are empty)
                v += part[w * PK * ROWS_PER_WAVE + i % ROWS_PER_WAVE]; // a run that goes on with a chunk begins in it
        uint32_t h = to_half_bits(v);
        h = h == UNWRITTEN ? 0xFE00u : h; // a NaN either way
        asm volatile("global_store_short %0, %1, off sc0 sc1" ::"v"(R.y + i), "v"(h) : "memory");
    };
    const int lane = threadIdx.x & 63;
    if (lane < R.rows)
        put(lane, R.first[0], R.more[0]);
    if (lane + 64 < R.rows)
        put(lane + 64, R.first[1], R.more[1]);
    for (int i = lane + 128; i < R.rows; i += 64) {
        int more;
        const int first = row_first(i, R.n, R.nslice, PK, more);
        put(i, first, more);
    }
}

// What a launch does first about a y that the next stage polls: no row of it is written yet.
__device__ __forceinline__ void clear_share_y(const ShareReg &sh)
{
    const int lane = threadIdx.x & 63;
    if (sh.bits() == 0 || !sh.has(POLL_Y))
        return;
    uint16_t *y = sh.y();
    const int row1 = min(sh.c1() * ROWS_PER_WAVE, sh.N());
    for (int i = sh.c0() * ROWS_PER_WAVE + lane; i < row1; i += 64)
        asm volatile("global_store_short %0, %1, off sc0 sc1" ::"v"(y + i), "v"(UNWRITTEN) : "memory");
}


struct Polled {
    int c[CPL];
    int flag;
};

// Waits until every workgroup has arrived at the end of stage s.  False: the launch is aborted.
// Lane l watches counter l (and l + 64), lane 0 the abort flag besides.  A poll is a round trip to
// memory of a microsecond or more, so two are kept in flight: the arrival of the last workgroup is
// seen about one round trip after it happened, not up to two.  (A poll is 129 requests of the
// workgroup, and the polls of 256 workgroups compete with the arrivals they wait for: 7B-shaped
// step with 8 / 6 / 4 / 3 / 2 polls in flight: 1.58 / 1.56 / 1.51 / 1.50 / 1.50 ms.)
__device__ __forceinline__ bool wait_stage(int *sync, int s, int G, long long wait_limit)
{
    const int lane = threadIdx.x & 63;
    int mine[CPL];
#pragma unroll
    for (int i = 0; i < CPL; i++)
        mine[i] = lane + 64 * i < NC ? (s + 1) * ((G - (lane + 64 * i) + NC - 1) / NC) : 0; // workgroups b with b % NC = lane + 64 i
    auto poll = [&]() -> Polled {
        Polled p;
#pragma unroll
        for (int i = 0; i < CPL; i++)
            p.c[i] = lane + 64 * i < NC ? __hip_atomic_load(&sync[SY_COUNTERS + CSTRIDE * (lane + 64 * i)], __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT)
                                        : 0;
        p.flag = 0;
        if (lane == 0)
            p.flag = __hip_atomic_load(&sync[SY_ABORT], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return p;
    };
    constexpr int Q = 2;
    Polled v[Q];
#pragma unroll
    for (int q = 0; q + 1 < Q; q++) {
        v[q] = poll();
        __builtin_amdgcn_s_sleep(1);
    }
    for (long long it = 0;; it += Q) {
#pragma unroll
        for (int q = 0; q < Q; q++) {
            v[(q + Q - 1) % Q] = poll();
            const Polled got = v[q]; // the oldest of the polls in flight
            if (__builtin_amdgcn_readfirstlane(got.flag))
                return false;
            bool ok = true;
#pragma unroll
            for (int i = 0; i < CPL; i++)
                ok = ok && got.c[i] >= mine[i];
            if (__builtin_amdgcn_ballot_w64(ok) == ~0ull)
                return true;
            __builtin_amdgcn_s_sleep(1);
        }
        if (it >= wait_limit) {
            // the first to give up in this launch raises the flag and counts the launch
            if (lane == 0 &&
                __hip_atomic_exchange(&sync[SY_ABORT], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
                __hip_atomic_fetch_add(&sync[SY_GAVE_UP], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
    }
}


// Into stage s: x in LDS, by all wavefronts of the workgroup.  False: the launch is aborted.
template <int BITS>
__device__ __forceinline__ bool cross(const ShareReg &sh, int s, int *flags, uint4 *xbuf, const Wait &w)
{
    if (s > 0) {
        if (!sh.has(POLL_STAGE)) {
            wg_barrier(); // every workgroup has arrived (or the abort flag is up)
            if (uni(flags[0]) <= s)
                return false;
        }
        wait_rows(&flags[1], s - 1); // nobody reads the present x any more
    }
    if constexpr (BITS != 0)
        stage_x_all<BITS>(sh.x(), sh.K(), xbuf, sh.has(POLL_X), w);
    wg_barrier(); // x of stage s is in LDS
    return uni(flags[0]) > s;
}

// One stage of a compute wavefront (BITS = 0: no share of it).
template <int BITS>
__device__ __forceinline__ bool run_stage(const ShareReg &sh, int s, int wave, float *part, int PK, int *flags, uint4 *xbuf,
                                          const Wait &w)
{
    const int lane = threadIdx.x & 63;
    // The rows are announced as soon as they are in LDS (which serves a wavefront's accesses in order).
    auto arrive = [&]() __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        if (lane == 0)
            __hip_atomic_fetch_add(&flags[1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    if constexpr (BITS == 0) {
        if (!cross<0>(sh, s, flags, xbuf, w))
            return false;
        arrive();
        return true;
    } else {
        const int K = sh.K(), c0 = sh.c0(), c1 = sh.c1();
        const int nslice = (K + slice_span(BITS) - 1) / slice_span(BITS);
        const int n = (c1 - c0) * nslice; // (at most FQ_STAGED_CHUNKS x MAX_SLICES)
        const int i0 = n * wave / CW, i1 = n * (wave + 1) / CW, first = sh.over_slices(i0);
        const Run<BITS> run(sh, min(c1 * ROWS_PER_WAVE, sh.N()) - c0 * ROWS_PER_WAVE, nslice, i1);
        // the next item to request and the next to compute: number, chunk and slice
        int ri = i0, rc = first, rj = i0 - first * nslice;
        int ci = ri, cc = rc, cj = rj;
        auto step = [&](int &i, int &c, int &j) __attribute__((always_inline)) {
            i++;
            if (++j == nslice) {
                j = 0;
                c++;
            }
        };
        Item<BITS> L[P];
#pragma unroll
        for (int p = 0; p < PRE; p++) {
            run.issue(ri, rc, rj, L[p]);
            step(ri, rc, rj);
        }
        if (!cross<BITS>(sh, s, flags, xbuf, w))
            return false;
        if (i0 == i1) {
            arrive();
            return true;
        }
#pragma unroll
        for (int p = PRE; p < P; p++) {
            run.issue(ri, rc, rj, L[p]);
            step(ri, rc, rj);
        }
        float acc[ROWS_PER_WAVE] = {0.f, 0.f, 0.f, 0.f};
        do {
#pragma unroll
            for (int p = 0; p < P; p++) {
                if (ci < i1) {
                    Loaded T;
                    run.expand(L[p], cj, T);
                    compute<BITS>(K, cj, T, xbuf, acc);
                    if (cj + 1 == nslice || ci + 1 == i1) {
                        // this wavefront's part of the chunk's four rows: reduce over the lanes, lane 63
                        // leaves the sums in LDS
                        float v[ROWS_PER_WAVE];
#pragma unroll
                        for (int r = 0; r < ROWS_PER_WAVE; r++) {
                            v[r] = wave_sum_lane63(acc[r]);
                            acc[r] = 0.0f;
                        }
                        if (lane == 63)
                            *reinterpret_cast<float4 *>(part + ((size_t)wave * PK + (cc - first)) * ROWS_PER_WAVE) =
                                make_float4(v[0], v[1], v[2], v[3]);
                        if (ci + 1 == i1)
                            arrive();
                    }
                    step(ci, cc, cj);
                }
                run.issue(ri, rc, rj, L[p]);
                step(ri, rc, rj);
            }
        } while (ci < i1);
        return true;
    }
}

__global__ __launch_bounds__(THREADS) void decode_staged_kernel(const FqLinearDesc *__restrict__ table,
                                                                const int32_t *__restrict__ bits_dev,
                                                                const int32_t *__restrict__ stage_begin,
                                                                int n_stages, int *sync, long long wait_limit,
                                                                int res_chunks)
{
    extern __shared__ uint4 lds[];
    const int PK = res_chunks / CW + 2; // chunks one wavefront can have a hand in per stage
    Share *shares = reinterpret_cast<Share *>(lds);                  // [n_stages]
    float *part = reinterpret_cast<float *>(lds + 4 * n_stages);     // [CW][PK][4] partial rows
    int *flags = reinterpret_cast<int *>(lds + 4 * n_stages + CW * PK); // [0]: the stage ahead of which to leave; [1]: rows left in LDS, by compute wavefronts and stages
    uint4 *xbuf = lds + 4 * n_stages + CW * PK + 4;
    const int wave = uni(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int G = gridDim.x, b = blockIdx.x;

    // ---- every workgroup's share of every stage -------------------------------------------
    bool too_large = false, unattached = false;
    for (int s = threadIdx.x; s < n_stages; s += THREADS) {
        const int e0 = stage_begin[s], e1 = stage_begin[s + 1];
        long long C = 0;
        for (int e = e0; e < e1; e++) {
            const long long gc = group_cost(table[e], bits_dev[e]);
            unattached = unattached || gc == 0;
            C += gc * (table[e].K >> 7) * ((table[e].N + 3) >> 2);
        }
        Share sh = {};
        if (C > 0) {
            const long long avail = G - (e1 - e0);
            long long prefix = 0;
            for (int e = e0; e < e1; e++) {
                const FqLinearDesc d = table[e];
                const int bits = bits_dev[e];
                const int chunks = (d.N + 3) >> 2;
                const long long cost = group_cost(d, bits) * (d.K >> 7) * chunks;
                const int g_lo = (e - e0) + (int)(avail * prefix / C);
                prefix += cost;
                const int g_hi = (e - e0 + 1) + (int)(avail * prefix / C);
                if (b >= g_lo && b < g_hi && cost > 0) {
                    const long long idx = b - g_lo, n = g_hi - g_lo;
                    sh.codes = bits == 2   ? d.codes2
                               : bits == 3 ? d.codes3
                               : bits == 4 ? d.codes4
                               : bits == 8 ? d.codes8
                                           : (const uint8_t *)d.w16;
                    sh.scales = bits == 2   ? d.scales2
                                : bits == 3 ? d.scales3
                                : bits == 4 ? d.scales4
                                : bits == 8 ? d.scales8
                                            : (const float *)d.w16;
                    sh.zeros = bits == 2   ? d.zeros2
                               : bits == 3 ? d.zeros3
                               : bits == 4 ? d.zeros4
                               : bits == 8 ? d.zeros8
                                           : (const uint8_t *)d.w16;
                    sh.x = d.x;
                    sh.y = d.y;
                    sh.N = d.N;
                    sh.K = d.K;
                    sh.c0 = (int)(chunks * idx / n);
                    sh.c1 = (int)(chunks * (idx + 1) / n);
                    const int nslice = (d.K + slice_span(bits) - 1) / slice_span(bits);
                    sh.inv = nslice > 1 ? 0xffffffffu / (uint32_t)nslice + 1 : 0;
                    sh.mode = sh.c1 > sh.c0 ? bits : 0;
                    // (an entry that polls: its producer's rows come only if the producer runs)
                    if (d.src > 0 && group_cost(table[d.src - 1], bits_dev[d.src - 1]) > 0)
                        sh.mode |= POLL_X;
                    if (s + 1 < n_stages && table[e1].src > 0)
                        sh.mode |= POLL_Y;
                    if (sh.c1 - sh.c0 > res_chunks) { // more rows than the results buffer holds: refuse
                        too_large = true;
                        sh.mode = 0;
                    }
                }
            }
        }
        if (table[e0].src > 0)
            sh.mode |= POLL_STAGE;
        shares[s] = sh;
    }
    if (threadIdx.x == 0) {
        flags[0] = NEVER;
        flags[1] = 0;
    }
    if (unattached && b == 0)
        __hip_atomic_fetch_or(&sync[SY_FLAGS], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (too_large)
        __hip_atomic_fetch_or(&sync[SY_FLAGS], 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();

    Wait w = {sync, wait_limit, flags, 0};

    if (wave == CW) {
        // ---- service wavefront ------------------------------------------------------------
        __builtin_amdgcn_s_setprio(3); // it has little to do, and everyone waits for it
        ShareReg sh(&shares[0]);
        stage_share_x(sh, xbuf, w); // with the compute wavefronts
        wg_barrier(); // x of stage 0 is in LDS
        for (int s = 1; s < n_stages; s++)
            clear_share_y(ShareReg(&shares[s]));
        int met = 0; // grid barriers so far
        for (int s = 0; s < n_stages; s++) {
            Rows R = {};
            plan_rows(sh, PK, R);
            sh = ShareReg(&shares[min(s + 1, n_stages - 1)]); // the next stage's, from here on
            wait_rows(&flags[1], s); // the compute wavefronts' rows of stage s are in LDS
            store_rows(part, PK, R);
            if (s + 1 == n_stages)
                break;
            if (!sh.has(POLL_STAGE)) {
                __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0): the stores are acknowledged
                if (lane == 0)
                    __hip_atomic_fetch_add(&sync[SY_COUNTERS + CSTRIDE * (b % NC)], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const bool aborted = !wait_stage(sync, met, G, wait_limit);
                met++;
                if (aborted && lane == 0)
                    flags[0] = s + 1;
                wg_barrier(); // every workgroup has arrived (or the abort flag is up)
                if (aborted)
                    break;
            }
            w.stage = s + 1;
            stage_share_x(sh, xbuf, w); // with the compute wavefronts
            __builtin_amdgcn_s_waitcnt(0xc07f);
            wg_barrier(); // x of stage s + 1 is in LDS
            if (uni(flags[0]) <= s + 1)
                break;
        }
        // last workgroup out puts the counters back
        if (lane == 0) {
            const int done = __hip_atomic_fetch_add(&sync[SY_DONE], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (done == G - 1) {
                for (int l = 0; l < NC; l++)
                    __hip_atomic_store(&sync[SY_COUNTERS + CSTRIDE * l], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&sync[SY_ABORT], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&sync[SY_DONE], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        return;
    }

    // ---- compute wavefronts ---------------------------------------------------------------
    ShareReg next(&shares[0]);
    for (int s = 0; s < n_stages; s++) {
        const ShareReg sh = next;
        next = ShareReg(&shares[min(s + 1, n_stages - 1)]);
        const int bits = sh.bits();
        w.stage = s;
        const bool go = bits == 2    ? run_stage<2>(sh, s, wave, part, PK, flags, xbuf, w)
                        : bits == 3  ? run_stage<3>(sh, s, wave, part, PK, flags, xbuf, w)
                        : bits == 4  ? run_stage<4>(sh, s, wave, part, PK, flags, xbuf, w)
                        : bits == 8  ? run_stage<8>(sh, s, wave, part, PK, flags, xbuf, w)
                        : bits == 16 ? run_stage<16>(sh, s, wave, part, PK, flags, xbuf, w)
                                     : run_stage<0>(sh, s, wave, part, PK, flags, xbuf, w);
        if (!go)
            return;
    }
}

} // namespace


size_t fq_staged_lds_bytes(int n_stages, int max_K, int res_chunks)
{
    const size_t kp4 = ((size_t)max_K + 2047) / 2048 * 2048, kp2 = ((size_t)max_K + 4095) / 4096 * 4096;
    const size_t b4 = kp4 * 2 + kp4 / 32 * 8, b2 = kp2 * 2 + kp2 / 64 * 8;
    return (size_t)n_stages * sizeof(Share) + (size_t)CW * (res_chunks / CW + 2) * 16 + 64 + (b4 > b2 ? b4 : b2) + 64;
}

// Workgroups of the staged kernel: one per compute unit, and never more than fit at once (they
// wait for each other).  0: the kernel does not fit with this much LDS.
int fq_staged_grid(size_t lds_bytes)
{
    if (lds_bytes > 48 * 1024 &&
        fq_raise_dynamic_lds((const void *)decode_staged_kernel, 160 * 1024) != hipSuccess)
        return 0;
    const int per_cu = fq_workgroups_per_cu((const void *)decode_staged_kernel, THREADS, lds_bytes, 0);
    return per_cu < 1 ? 0 : fq_device_cus();
}

hipError_t fq_launch_decode_staged(const FqLinearDesc *table_dev, const int32_t *bits_dev,
                                   const int32_t *stage_begin_dev, int n_stages, int max_K, int res_chunks,
                                   int *sync_dev, long long wait_limit, hipStream_t stream)
{
    const size_t lds = fq_staged_lds_bytes(n_stages, max_K, res_chunks);
    const int grid = fq_staged_grid(lds);
    if (grid < 1)
        return hipErrorInvalidConfiguration;
    decode_staged_kernel<<<grid, THREADS, lds, stream>>>(table_dev, bits_dev, stage_begin_dev, n_stages, sync_dev,
                                                         wait_limit, res_chunks);
    return hipGetLastError();
}
