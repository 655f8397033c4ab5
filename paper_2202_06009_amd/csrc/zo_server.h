// zo_server.h -- the lookup-table server of Algorithm 2 (template code) and its
// launch: zo_server.hip instantiates it for up to 128 workers on aligned
// chunks, zo_server_many.hip for more workers, zo_server_ua.hip for chunk
// lengths that are not a multiple of 4.
#pragma once

#include "zo_device.h"

namespace zo {

// The arguments of one server launch (see launch_srv).
struct SrvArgs {
    const uint64_t *packed;
    const float *scales;
    int W;
    int64_t wstride, cstride;
    Chunks ch;
    int64_t c0, nch, word0, elem0;
    float *srv_err;
    uint64_t *srv_packed;
    float *srv_scales, *avg;
    uint8_t *flags;
};

hipError_t launch_srv_many(int ld, bool al, const SrvArgs &a, hipStream_t st);
hipError_t launch_srv_ua(int ld, const SrvArgs &a, hipStream_t st);

// Exact-sum condition for one chunk's scales (see zo_unpack_average): every
// partial sum of +-S_w is a multiple of the smallest ulp among the nonzero
// scales and below W * 2^(largest exponent + 1), so it is exact in binary64
// when that span fits 53 bits.  Evaluated by the first min(L, 64) lanes of the
// chunk (0 in its other waves, which have no part in it); returns 1 when
// violated (or a scale is not finite).  scale(w): worker w's scale.
template <int L, class Scale>
__device__ __forceinline__ uint32_t inexact_flag(Scale scale, int W, int lc)
{
    constexpr int LW = L < 64 ? L : 64;
    if (L > 64 && lc >= LW) return 0;
    int lo = 1 << 20, hi = -(1 << 20), bad = 0;
    {
        for (int w = lc; w < W; w += LW) {
            uint32_t b = __float_as_uint(scale(w)) & 0x7FFFFFFFu;
            if (b == 0) continue;
            int f = (int)(b >> 23);
            if (f == 255) { bad = 1; continue; }
            int l, h;
            if (f == 0) {
                l = -149;
                h = (31 - __clz((int)b)) - 149;
            } else {
                l = f - 150;
                h = f - 127;
            }
            lo = min(lo, l);
            hi = max(hi, h);
        }
    }
    lo = (int)lanes_reduce<LW>((uint32_t)lo, [](uint32_t a, uint32_t b) {
        return (uint32_t)min((int)a, (int)b);
    });
    hi = (int)lanes_reduce<LW>((uint32_t)hi, [](uint32_t a, uint32_t b) {
        return (uint32_t)max((int)a, (int)b);
    });
    bad = (int)lanes_reduce<LW>((uint32_t)bad, [](uint32_t a, uint32_t b) { return a | b; });
    int lg = 0;
    while ((1 << lg) < W) ++lg;
    if (hi < lo) return (uint32_t)bad;  // every scale is zero
    return (uint32_t)(bad || (hi + 1 + lg - lo > 53));
}

// The same condition in two parts, for workers in batches: the span of a batch's
// scales and the test of the whole.
struct Span {
    int lo, hi, bad;  // exponents of the smallest ulp and the largest bit; a scale not finite
};

// The span of scale(0) .. scale(n - 1), by the first min(L, 64) lanes of the chunk.
template <int L, class Scale>
__device__ __forceinline__ Span scale_span(Scale scale, int n, int lc)
{
    constexpr int LW = L < 64 ? L : 64;
    Span s{1 << 20, -(1 << 20), 0};
    for (int w = lc; w < n; w += LW) {
        const uint32_t b = __float_as_uint(scale(w)) & 0x7FFFFFFFu;
        const int f = (int)(b >> 23);
        if (f == 255) s.bad = 1;
        if (b == 0 || f == 255) continue;
        s.lo = min(s.lo, f == 0 ? -149 : f - 150);
        s.hi = max(s.hi, f == 0 ? (31 - __clz((int)b)) - 149 : f - 127);
    }
    s.lo = (int)lanes_reduce<LW>((uint32_t)s.lo, [](uint32_t a, uint32_t b) {
        return (uint32_t)min((int)a, (int)b);
    });
    s.hi = (int)lanes_reduce<LW>((uint32_t)s.hi, [](uint32_t a, uint32_t b) {
        return (uint32_t)max((int)a, (int)b);
    });
    s.bad = (int)lanes_reduce<LW>((uint32_t)s.bad, [](uint32_t a, uint32_t b) { return a | b; });
    return s;
}

// 1 when the condition is violated for W workers whose scales have this span.
__device__ __forceinline__ uint32_t span_inexact(const Span &s, int W)
{
    int lg = 0;
    while ((1 << lg) < W) ++lg;
    if (s.hi < s.lo) return (uint32_t)s.bad;  // every scale is zero
    return (uint32_t)(s.bad || (s.hi + 1 + lg - s.lo > 53));
}

// Adds the span of a batch's scales to the chunk's: by the chunk's first wave.
template <int L>
__device__ __forceinline__ void add_span(Span *all, const float *scales, int n, bool first, int lc)
{
    if (L > 64 && lc >= 64) return;
    Span s = scale_span<L>([&](int w) { return scales[w]; }, n, lc);
    if (lc != 0) return;
    if (!first) {
        s.lo = min(s.lo, all->lo);
        s.hi = max(s.hi, all->hi);
        s.bad |= all->bad;
    }
    *all = s;
}

// Server with a lookup table per group of 8 workers ("four Russians"): for a
// chunk, T_g[b] = sum_{k<8} (bit k of b ? +S_{8g+k} : -S_{8g+k}) in binary64
// for all 256 bytes b; an element's sum over W workers is then the sum over
// groups of T_g[byte of its 8 workers' bits].  Under the exact-sum condition
// every partial sum is exact, so any grouping gives the bits of the
// sequential sum (chunks that break it: see kWorkerOrder).  Lane mapping: one
// lane owns the 32 elements of one packed dword (lane lc, dword lc of the chunk); the
// 8 x 32 bit block of a worker group is transposed in registers so that byte c
// of register k holds element 8c+k's 8 worker bits.

// Swap the bits selected by m << s in x with the bits selected by m in y
// (a delta swap written as two bit-field inserts).
__device__ __forceinline__ void swap_bits(uint32_t &x, uint32_t &y, int s, uint32_t m)
{
    const uint32_t xs = x >> s, ys = y << s;
    y = (xs & m) | (y & ~m);
    x = (ys & (m << s)) | (x & ~(m << s));
}

__device__ __forceinline__ void transpose8x32(uint32_t (&x)[8])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) swap_bits(x[k], x[k + 4], 4, 0x0F0F0F0Fu);
    swap_bits(x[0], x[2], 2, 0x33333333u);
    swap_bits(x[1], x[3], 2, 0x33333333u);
    swap_bits(x[4], x[6], 2, 0x33333333u);
    swap_bits(x[5], x[7], 2, 0x33333333u);
#pragma unroll
    for (int k = 0; k < 8; k += 2) swap_bits(x[k], x[k + 1], 1, 0x55555555u);
}

// Byte C of x times 8 (a table offset in bytes) in one SDWA instruction.
template <int C>
__device__ __forceinline__ uint32_t byte_x8(uint32_t x)
{
    uint32_t r;
    if constexpr (C == 0)
        asm("v_lshlrev_b32_sdwa %0, 3, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
            "src1_sel:BYTE_0" : "=v"(r) : "v"(x));
    else if constexpr (C == 1)
        asm("v_lshlrev_b32_sdwa %0, 3, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
            "src1_sel:BYTE_1" : "=v"(r) : "v"(x));
    else if constexpr (C == 2)
        asm("v_lshlrev_b32_sdwa %0, 3, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
            "src1_sel:BYTE_2" : "=v"(r) : "v"(x));
    else
        asm("v_lshlrev_b32_sdwa %0, 3, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
            "src1_sel:BYTE_3" : "=v"(r) : "v"(x));
    __builtin_assume(r < 2048u);  // lets the table base fold into the LDS offset
    return r;
}

// Workgroups are dealt to the GPU's 8 XCDs round-robin (workgroup i to XCD
// i % 8), and each XCD has its own L2.  With the grid padded to a multiple
// of 8 workgroups, block i takes block number (i % 8) * (grid / 8) + i / 8:
// every XCD walks a contiguous run of blocks in order, so neighbouring
// chunks share its L2 (in every worker's row the cache line that straddles
// two chunks' words, and each line holding 32 chunks' scales).
constexpr int kXcds = 8;

__device__ __forceinline__ int64_t xcd_block()
{
    const int64_t per = gridDim.x / kXcds;
    return (int64_t)(blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
}

static inline unsigned xcd_grid(unsigned blocks)
{
    return (blocks + kXcds - 1) / kXcds * kXcds;
}

// Load the 8 dwords of worker group g (workers beyond W read as 0).  Plain
// loads: the nontemporal hint measured no faster for these dword accesses.
// a value the whole wave agrees on, moved to scalar registers: a load at
// p + wave_uniform(off) + lane is then addressed as scalar base + lane offset
__device__ __forceinline__ int64_t wave_uniform(int64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Dword lc of the chunk for the 8 workers of group g: worker w's words start
// at dword off + ws*w.  UNIFORM: the whole wave is on one chunk, so the row
// offsets are scalars and each load costs one address add.
template <bool UNIFORM>
__device__ __forceinline__ void load_group(uint32_t (&x)[8], const uint32_t *packed32, int64_t off,
                                           int64_t ws, int g, int W, uint32_t lc)
{
    int64_t r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
        r[k] = UNIFORM ? wave_uniform(off + ws * (8 * g + k)) : off + ws * (8 * g + k);
    if (8 * g + 8 <= W) {
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = packed32[r[k] + lc];
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = 8 * g + k < W ? packed32[r[k] + lc] : 0u;
    }
}

// Worker groups whose packed words are loaded ahead of the one being summed
// (HBM latency is hidden by bytes in flight, and the table lookups leave
// registers for only a few groups).
constexpr int kSrvPrefetch = 2;

// Chunks of fewer than 64 dwords (several chunks per wave) look up the two
// 16-entry half tables of each group directly instead of building the
// 256-entry table from them: the build would cost as much as the lookups, and
// the smaller tables leave LDS for more waves per CU.
constexpr bool srv_nibble(int LD) { return LD < 64; }

// Chunks per workgroup of the LUT server: enough chunks to fill a wave when a
// chunk has fewer than 64 dwords, as long as their tables fit in 64 KB.
constexpr int srv_chunks_per_block(int LD, int G)
{
    const int fill = LD >= 64 ? 1 : 64 / LD;
    const int per = srv_nibble(LD) ? 256 : 32;  // chunks of G groups' tables in 64 KB, times G
    const int fit = per / G > 1 ? per / G : 1;
    int c = fill < fit ? fill : fit;
    while (c & (c - 1)) c &= c - 1;  // a power of two (G need not be one)
    return c;
}

// Eight table lookups (byte C of the eight transposed registers) added to
// their accumulators.  The empty asm consumes the eight sums: the adds, and so
// the table reads, of one batch complete before the next batch's reads are
// issued (otherwise the scheduler hoists every read of the unrolled groups and
// their results, two registers each, spill).
template <int C>
__device__ __forceinline__ void lookup8(double (&acc)[32], const uint32_t (&x)[8], const char *tg)
{
#pragma unroll
    for (int k = 0; k < 8; ++k)
        acc[8 * C + k] += *reinterpret_cast<const double *>(tg + byte_x8<C>(x[k]));
    asm volatile(""
                 : "+v"(acc[8 * C + 0]), "+v"(acc[8 * C + 1]), "+v"(acc[8 * C + 2]),
                   "+v"(acc[8 * C + 3]), "+v"(acc[8 * C + 4]), "+v"(acc[8 * C + 5]),
                   "+v"(acc[8 * C + 6]), "+v"(acc[8 * C + 7])
                 :
                 : "memory");
}

// The same for the half tables at hg (16 entries for the low nibble of a
// worker byte, workers 8g..8g+3, then 16 for the high nibble): two lookups per
// element; every partial sum is exact, so the order of the adds does not
// matter.
template <int C>
__device__ __forceinline__ void lookup8_nib(double (&acc)[32], const uint32_t (&x)[8],
                                            const char *hg)
{
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        // nibble times 8 (a byte offset into its 128-byte table)
        const uint32_t lo = C == 0 ? (x[k] << 3) & 0x78u : (x[k] >> (8 * C - 3)) & 0x78u;
        const uint32_t hi = (x[k] >> (8 * C + 1)) & 0x78u;
        acc[8 * C + k] += *reinterpret_cast<const double *>(hg + lo);
        acc[8 * C + k] += *reinterpret_cast<const double *>(hg + 128 + hi);
    }
    asm volatile(""
                 : "+v"(acc[8 * C + 0]), "+v"(acc[8 * C + 1]), "+v"(acc[8 * C + 2]),
                   "+v"(acc[8 * C + 3]), "+v"(acc[8 * C + 4]), "+v"(acc[8 * C + 5]),
                   "+v"(acc[8 * C + 6]), "+v"(acc[8 * C + 7])
                 :
                 : "memory");
}

// Float4 slot of the transpose buffer that holds float4 t of a chunk (t = e/4).
// Lane j writes the slots 8j..8j+7 of its dword; lanes then read slots in
// coalesced order.  XOR-ing the slot's low three bits with bits 1..3 of j makes
// both the writes and the reads of 16 consecutive lanes hit 16 distinct
// 16-byte bank groups.
__device__ __forceinline__ int xpose_slot(int t)
{
    return 8 * (t >> 3) + ((t & 7) ^ ((t >> 4) & 7));
}

// LD lanes per chunk (one packed dword each), G groups of 8 workers (a
// compile-time count; groups past the last worker hold zero tables), CPW
// chunks per workgroup.  The tables of chunk q of the workgroup start at byte
// q*G*2048 of `tab` (with half tables, q*G*256 of `half`); with one chunk per
// workgroup the offset of every lookup is an immediate.  With half tables the
// register budget is held to the waves per SIMD that the workgroups' LDS
// allows, at most four (at 1024-element chunks and W = 32: four, with a
// 20-byte spill; 74 instead of 81 us on the ResNet-50 shape).
constexpr int srv_lut_waves(int LD, int G, bool many)
{
    if (!srv_nibble(LD)) return many && LD >= 256 ? 4 : 1;
    const int cpw = srv_chunks_per_block(LD, G);
    const int lds = cpw * LD * 128 + cpw * G * (256 + 32) + 256;  // transpose, tables, scales, tree
    const int per_cu = 160 * 1024 / lds;                         // one-wave workgroups per CU
    const int per_simd = (per_cu + 3) / 4;
    return per_simd < 1 ? 1 : (per_simd > 4 ? 4 : per_simd);
}

template <int LD, int G, bool MANY, bool AL>
__device__ __forceinline__ void srv_lut_body(
    const uint32_t *__restrict__ packed32, const float *__restrict__ scales, int W,
    int64_t wstride, int64_t cstride, const Chunks &ch, int64_t c0, int64_t nch, int64_t word0,
    int64_t elem0, float *__restrict__ srv_err, uint32_t *__restrict__ srv_packed32,
    float *__restrict__ srv_scales, float *__restrict__ avg_out, uint8_t *__restrict__ flags,
    double inv_w, int w_pow2)
{
    constexpr int CPW = srv_chunks_per_block(LD, G);
    constexpr bool kNib = srv_nibble(LD);
    // static arrays: their LDS addresses are link-time constants, so the group
    // offset of every lookup is an instruction immediate.  The tables are dead
    // once the sums are formed; the same memory then transposes the averages.
    constexpr int kTabBytes = kNib ? 0 : CPW * G * 256 * 8;
    constexpr int kXposeBytes = CPW * LD * 32 * 4;
    __shared__ double uni[(kTabBytes > kXposeBytes ? kTabBytes : kXposeBytes) / 8];
    __shared__ float sc[CPW * G * 8];  // W <= 8G
    __shared__ double half[CPW * G * 32];  // per group: 16 sums of workers 0-3, 16 of 4-7
    __shared__ float tree[64];
    // more than 128 workers and unaligned chunks: inexact sums worker by worker
    // (see launch_srv)
    constexpr bool kWorkerOrder = MANY || !AL;
    __shared__ uint32_t inexact;
    // Batches of aligned chunks of up to 256 dwords: the exact-sum check batch by
    // batch while the scales are staged and the tables built.  Reading them all again
    // at the end costs a round trip per chunk: 110M, chunk 8192, W = 130 611 -> 582
    // us, W = 192 770 -> 762, W = 256 973 -> 937; chunk 1024, W = 192 1666 -> 1637.
    // Wider and unaligned forms spill more with it (chunk 16384, W = 192 869 -> 885;
    // chunk 4099 1157 -> 1233).
    constexpr bool kBatchCheck = MANY && AL && LD <= 256;
    __shared__ Span spans[kBatchCheck ? CPW : 1];
    double *tab = uni;

    const int q = CPW == 1 ? 0 : (int)threadIdx.x / LD;
    const int lc = CPW == 1 ? (int)threadIdx.x : (int)threadIdx.x % LD;
    const int64_t cbase = xcd_block() * CPW;
    const int64_t cr = cbase + q;
    const bool active = cr < nch;
    const int64_t c = c0 + (active ? cr : 0);
    const int len = active ? ch.len[c] : 0;
    const int64_t el = active ? ch.start[c] - elem0 : 0;
    const int64_t wd = active ? ch.word[c] - word0 : 0;

    // lane lc sums the 32 elements of dword lc of the chunk, if the chunk has it
    const int ndw_data = (len + 31) >> 5;
    const bool has_dw = lc < ndw_data;
    const int64_t ws = 2 * wstride;
    const int64_t off = 2 * wd;
    constexpr bool kUni = LD >= 64;  // a wave never spans two chunks
    uint32_t ring[kSrvPrefetch + 1][8];
    // the server error of the lane's elements in the compress layout (lane lc
    // holds the float4s lc + LD*k, k < 8, of its chunk); loaded while the last
    // group's lookups run
    f4v serr[8];
    auto load_serr = [&]() {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int e = 4 * LD * k + 4 * lc;
            serr[k] = f4v{0.f, 0.f, 0.f, 0.f};
            if (e < len) at<AL>(el + e, len - e, [&](auto p) { serr[k] = ld(srv_err, p); });
        }
    };
    // the sum over workers of the lane's 32 elements
    double acc[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) acc[i] = 0.0;

    // MANY: the workers in batches of 8G, whose tables take each other's place
    const int nb = MANY ? (W + 8 * G - 1) / (8 * G) : 1;
    const auto batch = [&](int bt) {
        const int w0 = MANY ? 8 * G * bt : 0, g0 = MANY ? G * bt : 0;
        const int nw = MANY ? min(W - w0, 8 * G) : W;
        // the first groups' packed words are in flight while the tables are built
        if (has_dw) {
#pragma unroll
            for (int g = 0; g < kSrvPrefetch && g < G; ++g)
                load_group<kUni>(ring[g], packed32, off, ws, g0 + g, W, lc);
        }

        // stage the scales of the workgroup's chunks, then build the tables
        // (strides by the workgroup's size as a constant: read from the dispatch it
        // is a vector load here, 10 us of the 110M-element server's 180)
        for (int i = threadIdx.x; i < CPW * nw; i += LD * CPW) {
            const int qq = i / nw, w = i - qq * nw;
            sc[i] = (cbase + qq < nch) ? scales[cstride * (w0 + w) + cbase + qq] : 0.0f;
        }
        __syncthreads();  // (MANY: and every lookup in the last batch's tables is done)
        // T_g[b] = H_g,0[b & 15] + H_g,1[b >> 4], with H_g,h[n] the signed sum of
        // workers 8g+4h .. 8g+4h+3 (every partial sum is exact, so the split is
        // too)
        for (int i = threadIdx.x; i < CPW * G * 32; i += LD * CPW) {
            const int qq = i / (G * 32), g = (i >> 5) % G, h = (i >> 4) & 1, nb = i & 15;
            double t = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int w = 8 * g + 4 * h + k;
                if (w < nw) {
                    const double sw = (double)sc[qq * nw + w];
                    t += ((nb >> k) & 1) ? sw : -sw;
                }
            }
            half[i] = t;
        }
        if constexpr (kBatchCheck && kNib) add_span<LD>(spans + q, sc + q * nw, nw, bt == 0, lc);
        __syncthreads();
        if constexpr (!kNib) {
            // CPW * G * 256 entries over LD * CPW threads, kPer = the ceiling of
            // their ratio each (a thread past the last entry repeats one from the
            // start: the same value written twice), in batches
            // of at most 8 whose reads are all issued before the first add (a
            // narrow workgroup has thousands of entries per thread: one batch at
            // a time keeps them out of scratch memory)
            constexpr int kTotal = CPW * G * 256, kThreads = LD * CPW;
            constexpr int kPer = (kTotal + kThreads - 1) / kThreads;
            constexpr int kBatch = kPer < 8 ? kPer : 8;
#pragma unroll 1
            for (int k0 = 0; k0 < kPer; k0 += kBatch) {
                double lo[kBatch], hi[kBatch];
#pragma unroll
                for (int k = 0; k < kBatch; ++k) {
                    const int i = ((int)threadIdx.x + (k0 + k) * kThreads) % kTotal;
                    const int qg = i >> 8, b = i & 255;  // qg = chunk * G + group
                    lo[k] = half[32 * qg + (b & 15)];
                    hi[k] = half[32 * qg + 16 + (b >> 4)];
                }
#pragma unroll
                for (int k = 0; k < kBatch; ++k)
                    tab[((int)threadIdx.x + (k0 + k) * kThreads) % kTotal] = lo[k] + hi[k];
            }
            if constexpr (kBatchCheck) add_span<LD>(spans + q, sc + q * nw, nw, bt == 0, lc);
            __syncthreads();
        }
        const char *mytab = kNib ? reinterpret_cast<const char *>(half) + (size_t)q * G * 256
                                 : reinterpret_cast<const char *>(tab) + (size_t)q * G * 2048;


        if (has_dw) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (g + kSrvPrefetch < G)
                    load_group<kUni>(ring[(g + kSrvPrefetch) % (kSrvPrefetch + 1)], packed32, off,
                                     ws, g0 + g + kSrvPrefetch, W, lc);
                uint32_t (&cur)[8] = ring[g % (kSrvPrefetch + 1)];
                transpose8x32(cur);
                if constexpr (kNib) {
                    const char *hg = mytab + g * 256;
                    lookup8_nib<0>(acc, cur, hg);
                    lookup8_nib<1>(acc, cur, hg);
                    lookup8_nib<2>(acc, cur, hg);
                    if (!MANY && g == G - 1) load_serr();
                    lookup8_nib<3>(acc, cur, hg);
                } else {
                    const char *tg = mytab + g * 2048;
                    lookup8<0>(acc, cur, tg);
                    lookup8<1>(acc, cur, tg);
                    lookup8<2>(acc, cur, tg);
                    if (!MANY && g == G - 1) load_serr();
                    lookup8<3>(acc, cur, tg);
                }
            }
        } else if (!MANY) {
            load_serr();
        }
    };
    if constexpr (MANY) {
#pragma unroll 1
        for (int bt = 0; bt < nb; ++bt) batch(bt);
        load_serr();
    } else {
        batch(0);
    }
    // sticky: a flag once set stays set until the handle is recreated
    uint32_t f;
    if constexpr (kBatchCheck)
        f = span_inexact(spans[q], W);
    else
        f = inexact_flag<LD>(
            [&](int w) { return MANY ? scales[cstride * w + (active ? cr : 0)] : sc[q * W + w]; },
            W, lc);
    if (active && lc == 0 && f) flags[cr] = 1;
    constexpr bool kShare = kWorkerOrder && !kBatchCheck && LD > 64;  // f in one wave only
    if (kShare && lc == 0) inexact = f;

    // averages -> LDS, then back in the coalesced layout of the compress step
    __syncthreads();  // every lookup is done: the tables may be overwritten
    f4v *xp = reinterpret_cast<f4v *>(uni) + (size_t)q * LD * 8;
    const auto mean = [&](double sum) {
        return w_pow2 ? (float)(sum * inv_w) : (float)(sum / (double)W);
    };
    if (kShare) f = inexact;
    if (kWorkerOrder && f && has_dw) {
        // a chunk whose sums are not exact: formed again worker by worker, four
        // elements at a time (a rare path that takes no registers from the other)
#pragma unroll 1
        for (int p = 0; p < 8; ++p) {
            double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
            for (int w = 0; w < W; ++w) {
                const uint32_t bits = packed32[off + ws * w + lc] >> (4 * p);
                const double sw = (double)scales[cstride * w + cr];
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) sum[qq] += ((bits >> qq) & 1u) ? sw : -sw;
            }
            xp[xpose_slot(8 * lc + p)] =
                f4v{mean(sum[0]), mean(sum[1]), mean(sum[2]), mean(sum[3])};
        }
    } else {
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            f4v av;
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) av[qq] = mean(acc[4 * p + qq]);
            xp[xpose_slot(8 * lc + p)] = av;
        }
    }
    __syncthreads();
    f4v bv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int e = 4 * LD * k + 4 * lc;
        bv[k] = f4v{0.f, 0.f, 0.f, 0.f};
        if (e < len) {
            const f4v av = xp[xpose_slot(LD * k + lc)];
            f4v bk;
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) bk[qq] = av[qq] + serr[k][qq];
            at<AL>(el + e, len - e, [&](auto p) {
                if (avg_out) st(avg_out, p, av);
                bv[k] = inside(bk, p);
            });
        }
    }
    // Equation 3 with the server error
    compress_chunk<LD, 8, AL>(bv, lc, len, active, srv_err, el,
                                srv_packed32 + 2 * (active ? ch.word[c] : 0), srv_scales + c,
                                tree);
}

#define ZO_SRV_LUT_KERNEL(name, MANY, AL)                                                       \
    template <int LD, int G>                                                                    \
    __global__ __launch_bounds__(LD > 64 ? LD : 64)                                             \
    __attribute__((amdgpu_waves_per_eu(srv_lut_waves(LD, G, MANY)))) void name(                 \
        const uint32_t *__restrict__ packed32, const float *__restrict__ scales, int W,         \
        int64_t wstride, int64_t cstride, Chunks ch, int64_t c0, int64_t nch, int64_t word0,    \
        int64_t elem0, float *__restrict__ srv_err, uint32_t *__restrict__ srv_packed32,        \
        float *__restrict__ srv_scales, float *__restrict__ avg_out, uint8_t *__restrict__ flags, \
        double inv_w, int w_pow2)                                                               \
    {                                                                                           \
        srv_lut_body<LD, G, MANY, AL>(packed32, scales, W, wstride, cstride, ch, c0, nch, word0, \
                                      elem0, srv_err, srv_packed32, srv_scales, avg_out, flags, \
                                      inv_w, w_pow2);                                           \
    }

// One launch of a server kernel of LD lanes per chunk and G groups.
template <int LD, int G, class K>
static hipError_t go_srv_lut(K kernel, const SrvArgs &a, hipStream_t st)
{
    constexpr int CPW = srv_chunks_per_block(LD, G);
    hipLaunchKernelGGL(kernel, dim3(xcd_grid(grid_for(a.nch, CPW))), dim3(LD * CPW), 0, st,
                       reinterpret_cast<const uint32_t *>(a.packed), a.scales, a.W, a.wstride,
                       a.cstride, a.ch, a.c0, a.nch, a.word0, a.elem0, a.srv_err,
                       reinterpret_cast<uint32_t *>(a.srv_packed), a.srv_scales, a.avg, a.flags,
                       1.0 / (double)a.W, (a.W & (a.W - 1)) == 0 ? 1 : 0);
    return hipGetLastError();
}

// Calls f(integral_constant<LD>) for a run-time lane count of at least MIN (1,
// 16 or 64).
template <int MIN, class F>
static hipError_t with_lanes(int ld, F &&f)
{
    using std::integral_constant;
    if constexpr (MIN <= 1) {
        switch (ld) {
        case 1: return f(integral_constant<int, 1>{});
        case 2: return f(integral_constant<int, 2>{});
        case 4: return f(integral_constant<int, 4>{});
        case 8: return f(integral_constant<int, 8>{});
        default: break;
        }
    }
    if constexpr (MIN <= 16) {
        switch (ld) {
        case 16: return f(integral_constant<int, 16>{});
        case 32: return f(integral_constant<int, 32>{});
        default: break;
        }
    }
    switch (ld) {
    case 64: return f(integral_constant<int, 64>{});
    case 128: return f(integral_constant<int, 128>{});
    case 256: return f(integral_constant<int, 256>{});
    case 512: return f(integral_constant<int, 512>{});
    default: return hipErrorInvalidValue;
    }
}

}  // namespace zo
