// omc_decompress / omc_decompress_set: packed codes + (s, b) -> fp32.
#include "omc_codec_impl.h"

namespace omc {

static int launch_full(uint32_t bits, const CodecArgs &ca, hipStream_t st) {
    switch (bits) {
#define X(BITS)                                                                       \
    case BITS:                                                                        \
        launch_codec<BITS, kDecompress, 0>(ca, st);                                   \
        break;
        OMC_FOR_EACH_BITS(X)
#undef X
        default:
            return static_cast<int>(hipErrorInvalidValue);
    }
    return static_cast<int>(hipGetLastError());
}

int launch_decompress(const void *codes, const VarArgs &va, const float *sb, float *out, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t tiles = single_tiles_per_item(va.fp.bits, va.n);
    const uint32_t nchunks = static_cast<uint32_t>((va.n / kTileElems + tiles - 1) / tiles);
    const bool has_tail = (va.n % kTileElems) != 0;
    CodecArgs ca{};
    ca.arena = static_cast<uint8_t *>(const_cast<void *>(codes));   // never written in this mode
    ca.single.n = va.n;
    ca.single.total_dwords = va.total_dwords;
    ca.single.fp = va.fp;
    ca.single_tiles = tiles;
    ca.tail_first = nchunks;                               // the ragged tail is the launch's first workgroup
    ca.tail_nitems = has_tail ? 1u : 0u;
    ca.sb_in = sb;
    ca.vout = out;
    ca.nitems = nchunks;
    return launch_full(va.fp.bits, ca, st);
}

int launch_decompress_set(const void *arena, const PlanHeader *ph, const void *plan_dev, const float *sb_table,
                          float *out, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint8_t *ph_bytes = reinterpret_cast<const uint8_t *>(ph);
    const PlanGroup *groups = reinterpret_cast<const PlanGroup *>(ph_bytes + ph->group_off);
    CodecArgs ca{};
    ca.arena = static_cast<uint8_t *>(const_cast<void *>(arena));
    ca.plan = static_cast<const uint8_t *>(plan_dev);
    ca.var_off = ph->var_off;
    ca.item_off = ph->item_off;
    ca.sb_in = sb_table;
    ca.vout = out;
    // the copies of fp32 variables and the ragged tails ride along with the first full-tile launch
    SetGroups rest = set_groups(groups, ph->ngroups);
    for (uint32_t gi = 0; gi < ph->ngroups; ++gi) {
        const PlanGroup &g = groups[gi];
        if (g.nitems == 0 || g.kind != kGroupFull) continue;
        ca.first_item = g.first_item;
        ca.nitems = g.nitems;
        take_copies(rest, ca);
        take_tails(rest, ca);
        const int rc = launch_full(g.bits, ca, st);
        if (rc != 0) return rc;
    }
    ca.first_item = ca.nitems = 0;                     // what no full tile's launch took
    while (rest.fp32_nitems > 0) {
        take_copies(rest, ca);
        ca.tail_nitems = 0;
        launch_codec<8, kDecompress, 0>(ca, st);
        const int rc = static_cast<int>(hipGetLastError());
        if (rc != 0) return rc;
    }
    if (rest.tail_nitems > 0) {
        take_tails(rest, ca);
        codec_tail_kernel<kDecompress><<<dim3(ca.tail_nitems), dim3(64), 0, st>>>(ca);
        const int rc = static_cast<int>(hipGetLastError());
        if (rc != 0) return rc;
    }
    return 0;
}

}  // namespace omc
