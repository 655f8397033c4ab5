// zo_server_ua.hip -- the lookup-table server for chunk lengths that are not a
// multiple of 4.  A chunk's packed words start on a word boundary whatever its
// length; only the server error's elements do not (see At4u, At1), so the
// tables, the lookups and the transpose are those of the aligned chunks.
// BERT-Base-shaped shard (110M), W = 16, chunk 4099: 879 us by select-and-add
// per worker, 269 us by tables.
#include "zo_server.h"

namespace zo {

ZO_SRV_LUT_KERNEL(k_srv_lut_ua, false, false)

template <int G>
static hipError_t srv_ua_g(int ld, const SrvArgs &a, hipStream_t st)
{
    return with_lanes<(G & (G - 1)) == 0 ? 16 : 64>(ld, [&](auto Lc) {
        constexpr int LD = decltype(Lc)::value;
        return go_srv_lut<LD, G>(k_srv_lut_ua<LD, G>, a, st);
    });
}

// Worker groups of 8, rounded up to a count that is instantiated (the extra
// groups' tables are zero): chunks of fewer than 64 dwords to a power of two.
hipError_t launch_srv_ua(int ld, const SrvArgs &a, hipStream_t st)
{
    const int g = (a.W + 7) / 8, G = ld >= 64 ? g : next_pow2(g);
    if (G <= 1) return srv_ua_g<1>(ld, a, st);
    if (G <= 2) return srv_ua_g<2>(ld, a, st);
    if (G <= 3) return srv_ua_g<3>(ld, a, st);
    if (G <= 4) return srv_ua_g<4>(ld, a, st);
    if (G <= 6) return srv_ua_g<6>(ld, a, st);
    if (G <= 8) return srv_ua_g<8>(ld, a, st);
    if (G <= 12) return srv_ua_g<12>(ld, a, st);
    return srv_ua_g<16>(ld, a, st);
}

}  // namespace zo
