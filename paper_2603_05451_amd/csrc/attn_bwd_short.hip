// The backward pass of short key sequences in one kernel (gfx950): attn_bwd_short_kernel.inc.
#include "common.h"
#include "launch.h"

namespace attn {

#define ATTN_ELEM bf16
#define ATTN_ELEM8 bf16x8
#define ATTN_ELEM4 bf16x4
#include "elem.inc"
#undef ATTN_ELEM
#undef ATTN_ELEM8
#undef ATTN_ELEM4
#include "attn_bwd_short_kernel.inc"
#include "attn_bwd_short_launch.inc"

namespace f16k {
#define ATTN_ELEM f16
#define ATTN_ELEM8 f16x8
#define ATTN_ELEM4 f16x4
#include "elem.inc"
#undef ATTN_ELEM
#undef ATTN_ELEM8
#undef ATTN_ELEM4
#include "attn_bwd_short_kernel.inc"
#include "attn_bwd_short_launch.inc"
}  // namespace f16k

int launch_bwd_short(const BwdArgs& a) { return a.f16 ? f16k::launch_bwd_short_dims(a) : launch_bwd_short_dims(a); }

}  // namespace attn
