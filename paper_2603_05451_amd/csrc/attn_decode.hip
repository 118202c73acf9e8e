// Forward attention for few queries per sequence against many keys (decode steps, speculative tokens), and
// the merge of forward results that were computed in parts of the keys (gfx950).  What is computed is that of
// attn_fwd.hip; how, at the top of attn_decode_kernel.inc.
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
#include "attn_decode_kernel.inc"

namespace f16k {
#define ATTN_ELEM f16
#define ATTN_ELEM8 f16x8
#define ATTN_ELEM4 f16x4
#include "elem.inc"
#undef ATTN_ELEM
#undef ATTN_ELEM8
#undef ATTN_ELEM4
#include "attn_decode_kernel.inc"
}  // namespace f16k

int launch_decode(const FwdArgs& a) { return a.f16 ? f16k::launch_decode_dims(a) : launch_decode_dims(a); }
int launch_combine(const FwdArgs& a) { return a.f16 ? f16k::launch_combine_dims(a) : launch_combine_dims(a); }

}  // namespace attn
