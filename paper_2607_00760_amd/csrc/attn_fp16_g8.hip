// attn_fp16_g8.hip -- the attention kernels for fp16 and groups of up to 8
// query heads (one translation unit per pair: they build in parallel).
#include "attn.h"

namespace mosaic {

hipError_t launch_attn_fp16_g8(const Geom &g, const WsGeom &w, float scale, const uint16_t *q, bool fixed, bool small,
                              hipStream_t s) {
    return attn_dt<0, 8>(g, w, scale, q, fixed, small, s);
}

}  // namespace mosaic
