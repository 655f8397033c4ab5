// zo_server_many.hip -- the lookup-table server for more than 128 workers: the
// workers in batches of at most 128, each batch's tables in the same LDS (the
// sums stay in registers; every partial sum is exact, so the split changes no
// bit, and a chunk whose sums are not is summed again worker by worker).
// Select-and-add per worker is bound by the vector ALU: BERT-Base-shaped shard
// (110M), W = 192, chunk 8192: 4916 us; in batches 762 us, 4.7 TB/s (the loads of
// a batch wait for its tables' barriers, so two batches take more than one of
// twice the groups would).  The register budget is held to four waves per SIMD
// (six spilled dwords at 12 groups of 256 lanes; without the bound three waves).
#include "zo_server.h"

namespace zo {

ZO_SRV_LUT_KERNEL(k_srv_lut_many, true, true)
ZO_SRV_LUT_KERNEL(k_srv_lut_many_ua, true, false)

template <int G>
static hipError_t srv_many_g(int ld, bool al, const SrvArgs &a, hipStream_t st)
{
    return with_lanes<G == 16 ? 16 : 64>(ld, [&](auto Lc) {
        constexpr int LD = decltype(Lc)::value;
        return al ? go_srv_lut<LD, G>(k_srv_lut_many<LD, G>, a, st)
                  : go_srv_lut<LD, G>(k_srv_lut_many_ua<LD, G>, a, st);
    });
}

// The fewest batches of at most 16 groups, of the smallest even group count
// that covers them (W = 192: two batches of 12); chunks of fewer than 64
// dwords take 16.
hipError_t launch_srv_many(int ld, bool al, const SrvArgs &a, hipStream_t st)
{
    const int groups = (a.W + 7) / 8, batches = (groups + 15) / 16;
    const int G = ld >= 64 ? (groups + batches - 1) / batches : 16;
    if (G <= 10) return srv_many_g<10>(ld, al, a, st);
    if (G <= 12) return srv_many_g<12>(ld, al, a, st);
    if (G <= 14) return srv_many_g<14>(ld, al, a, st);
    return srv_many_g<16>(ld, al, a, st);
}

}  // namespace zo
