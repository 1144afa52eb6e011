// attn_bf16_g4.hip -- the attention kernels for bf16 and groups of up to 4
// query heads (one translation unit per pair: they build in parallel).
#include "attn.h"

namespace mosaic {

hipError_t launch_attn_bf16_g4(const Geom &g, const WsGeom &w, float scale, const uint16_t *q, bool fixed, bool small,
                              hipStream_t s) {
    return attn_dt<1, 4>(g, w, scale, q, fixed, small, s);
}

}  // namespace mosaic
