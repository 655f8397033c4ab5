// zo_server.hip -- the server half of Algorithm 2 on gfx950: unpack the W
// workers' packed signs, average them exactly, add the server error, compress
// the result with Equation 3 per chunk and pack it (k_srv_lut with subset-sum
// lookup tables; the kernel is in zo_server.h), plus the diagnostic of the
// server's memory accesses.
#include "zo_server.h"

namespace zo {

// Plain server: per element, per worker, add +-S_w in binary64 (the sign bit
// of the worker's scale flipped by its packed bit), workers in batches of 8
// whose words and scales are all loaded before the first is used.  No tables
// to build and nothing staged in LDS: the shortest chain of memory accesses,
// and the better form where a table would serve few lookups (see launch_srv).
// L lanes per chunk, V blocks of four elements each (chunks of at most 4LV; V > 1
// only for unaligned chunks, see srv_takes_plain).  AL: aligned
// chunks (see At4 / At4u / At1).  GROUPED: the sums in the lookup tables' order
// (see launch_srv): the signed sums of workers 8g .. 8g+3 and 8g+4 .. 8g+7, one
// after the other (chunks of fewer than 64 dwords) or added to each other first.
template <int L, int V, bool AL, bool GROUPED>
__device__ __forceinline__ void srv_plain_body(
    const uint32_t *__restrict__ packed32, const float *__restrict__ scales, int W,
    int64_t wstride, int64_t cstride, const Chunks &ch, int64_t c0, int64_t nch, int64_t word0,
    int64_t elem0, float *__restrict__ srv_err, uint32_t *__restrict__ srv_packed32,
    float *__restrict__ srv_scales, float *__restrict__ avg_out, uint8_t *__restrict__ flags,
    double inv_w, int w_pow2, float *lds)
{
    constexpr int CPW = L >= 256 ? 1 : 256 / L;
    const int lc = threadIdx.x % L;
    const int in_block = L >= 64 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / L)
                                 : (int)threadIdx.x / L;
    const int64_t cr = (int64_t)blockIdx.x * CPW + in_block;  // chunk within range
    const bool active = cr < nch;
    const int64_t c = c0 + (active ? cr : 0);
    const int len = active ? ch.len[c] : 0;
    const int64_t el = active ? ch.start[c] - elem0 : 0;  // element offset in range
    const int64_t wd = active ? ch.word[c] - word0 : 0;   // word offset in range
    const float *chunk_scales = scales + (active ? cr : 0);
    // The scale this lane checks, then the error and the first workers' words and
    // scales: no branch on W before them, which the compiler would wait behind.
    const float checked = chunk_scales[cstride * min(lc, W - 1)];
    f4v b[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int e = 4 * L * k + 4 * lc;
        b[k] = f4v{0.f, 0.f, 0.f, 0.f};
        if (e >= len) continue;
        at<AL, (L > 1 && L <= 64)>(el + e, len - e, [&](auto p) { b[k] = ld(srv_err, p); });
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        const uint32_t *words = packed32 + 2 * wd + (e >> 5);
        const int sh = 31 - (e & 31);  // element q's bit to the sign's place: sh - q
        // adds workers w0 .. w0 + N - 1; past the last worker (TAIL) a load repeats
        // the last one's and its scale counts as 0
        const auto add = [&](int w0, auto n, auto tail) {
            constexpr int N = decltype(n)::value;
            constexpr bool TAIL = decltype(tail)::value;
            uint32_t bits[N];
            float sw[N];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const int w = TAIL ? min(w0 + j, W - 1) : w0 + j;
                bits[j] = words[2 * wstride * w];
                sw[j] = chunk_scales[cstride * w];
            }
            double half[2][4] = {};
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const float sj = TAIL && w0 + j >= W ? 0.0f : sw[j];
                const uint64_t neg = (uint64_t)__double_as_longlong(-(double)sj);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // -S_w, its sign flipped where the bit is set (a zero past the
                    // last worker, which leaves any sum as it is)
                    const uint32_t flip = (bits[j] << (sh - q)) & 0x80000000u;
                    const double term =
                        __longlong_as_double((int64_t)(neg ^ ((uint64_t)flip << 32)));
                    if (GROUPED) half[j >> 2][q] += term;
                    else acc[q] += term;
                }
            }
            if (GROUPED) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (srv_nibble(L / 8)) acc[q] = (acc[q] + half[0][q]) + half[1][q];
                    else acc[q] += half[0][q] + half[1][q];
                }
            }
        };
        int w0 = 0;
        for (; w0 + 8 <= W; w0 += 8)
            add(w0, std::integral_constant<int, 8>{}, std::false_type{});
        if (w0 + 4 < W)
            add(w0, std::integral_constant<int, 8>{}, std::true_type{});
        else if (w0 < W)
            add(w0, std::integral_constant<int, 4>{}, std::true_type{});
        f4v av;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            av[q] = w_pow2 ? (float)(acc[q] * inv_w) : (float)(acc[q] / (double)W);
        at<AL, (L > 1 && L <= 64)>(el + e, len - e, [&](auto p) {
            if (avg_out) st(avg_out, p, av);
            // formed in a local vector: masking b in place after writing its elements
            // made this compiler drop the loads and adds
            f4v bk;
#pragma unroll
            for (int q = 0; q < 4; ++q) bk[q] = av[q] + b[k][q];
            b[k] = inside(bk, p);
        });
    }
    // sticky: a flag once set stays set until the handle is recreated
    const uint32_t f = inexact_flag<L>(
        [&](int w) { return w == lc ? checked : chunk_scales[cstride * w]; }, W, lc);
    if (active && lc == 0 && f) flags[cr] = 1;
    compress_chunk<L, V, AL>(b, lc, len, active, srv_err, el,
                             srv_packed32 + 2 * (active ? ch.word[c] : 0), srv_scales + c, lds);
}

#define ZO_SRV_PLAIN_KERNEL(name, AL, GROUPED)                                                  \
    template <int L, int V>                                                                     \
    __global__ __launch_bounds__(L > 256 ? L : 256) void name(                                  \
        const uint32_t *__restrict__ packed32, const float *__restrict__ scales, int W,         \
        int64_t wstride, int64_t cstride, Chunks ch, int64_t c0, int64_t nch, int64_t word0,    \
        int64_t elem0, float *__restrict__ srv_err, uint32_t *__restrict__ srv_packed32,        \
        float *__restrict__ srv_scales, float *__restrict__ avg_out, uint8_t *__restrict__ flags, \
        double inv_w, int w_pow2)                                                               \
    {                                                                                           \
        __shared__ float lds[64];                                                               \
        srv_plain_body<L, V, AL, GROUPED>(packed32, scales, W, wstride, cstride, ch, c0, nch,   \
                                       word0, elem0, srv_err, srv_packed32, srv_scales,         \
                                       avg_out, flags, inv_w, w_pow2, lds);                     \
    }
ZO_SRV_PLAIN_KERNEL(k_srv_plain, true, false)
ZO_SRV_PLAIN_KERNEL(k_srv_plain_grouped, true, true)
ZO_SRV_PLAIN_KERNEL(k_srv_plain_ua, false, false)

ZO_SRV_LUT_KERNEL(k_srv_lut, false, true)

// The memory accesses of k_srv_lut without its arithmetic: per chunk of the
// server range one workgroup of LD lanes in the same XCD-aware order, each lane
// reading its dword of the chunk from all W workers' rows, then the chunk's
// server error loaded and stored back unchanged with the kernel's nontemporal
// accesses and float4 layout.  The error keeps its bits; timing it measures
// the rate the server's access pattern can reach.
template <int LD>
__global__ __launch_bounds__(LD) void k_srv_pattern(const uint32_t *__restrict__ packed32, int W,
                                                    int64_t wstride, Chunks ch, int64_t c0,
                                                    int64_t nch, int64_t word0, int64_t elem0,
                                                    float *__restrict__ srv_err)
{
    const int lc = (int)threadIdx.x;
    const int64_t cr = xcd_block();
    if (cr >= nch) return;
    const int64_t c = c0 + cr;
    const int len = ch.len[c];
    const int64_t el = ch.start[c] - elem0;
    const int64_t wd = ch.word[c] - word0;
    uint32_t x = 0;
    if (lc < (len + 31) >> 5) {
        const uint32_t *p = packed32 + 2 * wd + lc;
        const int64_t ws = 2 * wstride;
#pragma unroll 8
        for (int w = 0; w < W; ++w) x ^= p[ws * w];
    }
    asm volatile("" ::"v"(x));  // the loads are not dead
    f4v v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int e = 4 * LD * k + 4 * lc;
        if (e < len) v[k] = ldnt(srv_err, (el + e) >> 2);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int e = 4 * LD * k + 4 * lc;
        if (e < len) stnt(srv_err, (el + e) >> 2, v[k]);
    }
}


// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

// Lanes per chunk of the server: one lane per packed dword, at most 512.
static inline int srv_lanes(int chunk) { return next_pow2((chunk + 31) / 32); }

template <int G>
static hipError_t srv_lut_g(int ld, const SrvArgs &a, hipStream_t st)
{
    // chunks of fewer than 64 dwords: powers of two only (see launch_srv)
    return with_lanes<(G & (G - 1)) == 0 ? 1 : 64>(ld, [&](auto Lc) {
        constexpr int LD = decltype(Lc)::value;
        return go_srv_lut<LD, G>(k_srv_lut<LD, G>, a, st);
    });
}

static hipError_t launch_srv_plain(Geometry geo, bool al, const SrvArgs &a, hipStream_t st)
{
    return with_geometry(geo, [&](auto Lc, auto Vc) {
        constexpr int L = decltype(Lc)::value, V = decltype(Vc)::value;
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(grid_for(a.nch, chunks_per_block<L>())),
                               dim3(chunk_block<L>()), 0, st,
                               reinterpret_cast<const uint32_t *>(a.packed), a.scales, a.W,
                               a.wstride, a.cstride, a.ch, a.c0, a.nch, a.word0, a.elem0,
                               a.srv_err, reinterpret_cast<uint32_t *>(a.srv_packed),
                               a.srv_scales, a.avg, a.flags, 1.0 / (double)a.W,
                               (a.W & (a.W - 1)) == 0 ? 1 : 0);
            return hipGetLastError();
        };
        if (!al) return go(k_srv_plain_ua<L, V>);
        if constexpr (V > 1) return hipErrorInvalidValue;  // longer chunks: the tables
        else return a.W > 128 ? go(k_srv_plain<L, V>) : go(k_srv_plain_grouped<L, V>);
    });
}

// Whether a launch takes the plain server.  Times: the server alone, plain :
// tables in us, device time with about 5 us of launch and event.
static bool srv_takes_plain(Geometry geo, int W, int chunk, bool al, int64_t nch)
{
    const int64_t elems = nch * chunk;
    // lanes in flight, in elements: every lane carries four, those past a chunk's
    // end too; 2M of them are on the GPU at once
    const int64_t lanes4 = nch * 4 * geo.L * geo.V;
    // Chunks of more than 4096 elements: small launches of few workers, unaligned
    // only.  100K to 1M elements: chunk 4099, W = 2 7.7 : 10.6 to 8.4 : 11.0, W = 8
    // 7.9 : 10.4 to 8.6 : 10.8 (2M 12.8 : 11.6); chunk 8191, W = 8 9.4 : 11.1, W = 16
    // 11.6 : 11.6; chunk 12345, W = 4 10.4 : 11.5, W = 8 11.5 : 11.3; chunk 16383,
    // W = 4 11.7 : 12.1, W = 8 13.0 : 12.0.
    if (geo.V > 1) return !al && W * geo.V <= 16 && lanes4 <= (4 << 19);
    if (al && W <= 128) {
        // Small launches (every workgroup resident at once) are bound by the chain
        // of memory accesses and barriers, which is the plain server's advantage.
        // 100K elements, chunk 1000, W = 8 6.3 : 9.8; 1M, chunk 2048, W = 4
        // 7.6 : 10.3, W = 16 8.6 : 11.0; the tables' bound on 2M: chunk 2048,
        // W = 16 12.2 : 11.4.  Larger launches: the tables at every length.
        return W <= 16 && elems <= (3 << 19) && elems * W <= (16 << 20);
    }
    // More than 128 workers (tables in batches) and unaligned chunks.
    // Narrow chunks: a chunk's tables serve too few lookups.  W = 192, 4M elements:
    // chunk 32 134 : 5661, chunk 256 122 : 258.
    if (chunk <= 256) return true;
    // Batches of 128 workers that are filled by less than two thirds, at chunks of
    // up to 16 dwords: the half tables are summed for workers that are not there.
    // Chunk 512, W = 129: 1M elements 33 : 65, 4M 91 : 138, 16M 307 : 384; W = 192
    // 4M 122 : 146, 8M 220 : 220.
    const bool unfilled = W > 128 && 3 * W <= 2 * 128 * ((W + 127) / 128);
    if (chunk <= 512 && unfilled) return true;
    // Small launches, as above.  Few workers keep the advantage up to a full GPU
    // (unaligned, chunk 1023, 2M elements: W = 4 11.3 : 12.2, W = 16 13.0 : 13.0,
    // W = 64 27 : 22; chunk 2047, W = 16 12.7 : 13.4; chunk 4095, W = 12 14.2 : 15.0,
    // W = 16 14.4 : 13.0, 1.3M 13.7 : 12.9), as do unfilled batches (chunk 1024,
    // W = 129: 2M 50 : 67, 4M 87 : 82).
    const bool few = W <= (chunk <= 2048 ? 16 : 12);
    const int64_t most = few || unfilled ? 4 << 19 : chunk <= 2048 ? 3 << 19 : 2 << 19;
    if (lanes4 > most) return false;
    // Up to 32 dwords to a chunk nothing else counts (unaligned, chunk 1023, 1M
    // elements: W = 8 8.0 : 11.4, W = 64 17 : 22, W = 128 30 : 34; W = 256, chunk
    // 1024 54 : 61).  Longer chunks have the 256-entry tables, worth their build
    // with enough workers: chunk 2047, W = 64, 1M 16.5 : 16.7; W = 128, 300K
    // 16.5 : 22.6, 1M 26.9 : 23.6; W = 256, 300K 27.8 : 39; chunk 4095, W = 32, 1M
    // 11.6 : 12.6, W = 128, 300K 24.7 : 21.0; chunk 4096, W = 256, 30K 40 : 33.
    if (chunk <= 1024) return true;
    if (chunk <= 2048) return lanes4 * W <= (120 << 20);
    return W <= 128 && lanes4 * W <= (40 << 20);
}

hipError_t launch_srv(Geometry geo, const uint64_t *packed, const float *scales, int W,
                      int64_t wstride, int64_t cstride, const Chunks &ch, int64_t c0,
                      int64_t nch, int64_t word0, int64_t elem0, float *srv_err,
                      uint64_t *srv_packed, float *srv_scales, float *avg, uint8_t *flags,
                      int chunk, bool al, hipStream_t st)
{
    if (nch == 0) return hipSuccess;
    // The order of a chunk's binary64 sums.  Under the exact-sum condition it
    // changes no bit; without it it does, so it hangs on the chunk length and the
    // worker count alone, never on which form serves the chunk or on the size of
    // the server range (one GPU's share and the single server agree): aligned
    // chunks and at most 128 workers in groups as the lookup tables hold them
    // (srv_plain_body's GROUPED), all others worker by worker (kWorkerOrder in
    // srv_lut_body).
    const int ld = srv_lanes(chunk);
    const SrvArgs a{packed, scales, W, wstride, cstride, ch, c0, nch, word0, elem0,
                    srv_err, srv_packed, srv_scales, avg, flags};
    if (srv_takes_plain(geo, W, chunk, al, nch)) return launch_srv_plain(geo, al, a, st);
    if (W > 128) return launch_srv_many(ld, al, a, st);
    if (!al) return launch_srv_ua(ld, a, st);
    // worker groups of 8 (the last one may be partial); chunks of fewer than
    // 64 dwords round the count up to a power of two (fewer instantiations,
    // the extra groups' tables are zero)
    const int G = ld >= 64 ? (W + 7) / 8 : next_pow2((W + 7) / 8);
    switch (G) {
    case 1: return srv_lut_g<1>(ld, a, st);
    case 2: return srv_lut_g<2>(ld, a, st);
    case 3: return srv_lut_g<3>(ld, a, st);
    case 4: return srv_lut_g<4>(ld, a, st);
    case 5: return srv_lut_g<5>(ld, a, st);
    case 6: return srv_lut_g<6>(ld, a, st);
    case 7: return srv_lut_g<7>(ld, a, st);
    case 8: return srv_lut_g<8>(ld, a, st);
    case 9: return srv_lut_g<9>(ld, a, st);
    case 10: return srv_lut_g<10>(ld, a, st);
    case 11: return srv_lut_g<11>(ld, a, st);
    case 12: return srv_lut_g<12>(ld, a, st);
    case 13: return srv_lut_g<13>(ld, a, st);
    case 14: return srv_lut_g<14>(ld, a, st);
    case 15: return srv_lut_g<15>(ld, a, st);
    case 16: return srv_lut_g<16>(ld, a, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_srv_pattern(int chunk, const uint64_t *packed, int W, int64_t wstride,
                              const Chunks &ch, int64_t c0, int64_t nch, int64_t word0,
                              int64_t elem0, float *srv_err, hipStream_t st)
{
    const int ld = srv_lanes(chunk);
    if (ld < 64) return hipErrorInvalidValue;
    if (nch == 0) return hipSuccess;
    const dim3 grid(xcd_grid(grid_for(nch, 1)));
    const uint32_t *p = reinterpret_cast<const uint32_t *>(packed);
    switch (ld) {
    case 64: hipLaunchKernelGGL(k_srv_pattern<64>, grid, dim3(64), 0, st, p, W, wstride, ch, c0, nch, word0, elem0, srv_err); break;
    case 128: hipLaunchKernelGGL(k_srv_pattern<128>, grid, dim3(128), 0, st, p, W, wstride, ch, c0, nch, word0, elem0, srv_err); break;
    case 256: hipLaunchKernelGGL(k_srv_pattern<256>, grid, dim3(256), 0, st, p, W, wstride, ch, c0, nch, word0, elem0, srv_err); break;
    case 512: hipLaunchKernelGGL(k_srv_pattern<512>, grid, dim3(512), 0, st, p, W, wstride, ch, c0, nch, word0, elem0, srv_err); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace zo
