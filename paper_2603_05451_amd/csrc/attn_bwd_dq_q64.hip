// The backward kernels with one wave per SIMD (gfx950), each for fixed-length and for variable-length batches:
//   attn_bwd_dq_q64_kernel    dQ with 64 queries per wave, head dims 128 and 64, with or without the causal
//                             mask (attn_bwd_dq_q64_kernel.inc);
//   attn_bwd_dq_t32_kernel    dQ with 32 queries per wave, head dims (192, 128) and 256
//                             (attn_bwd_dq_t32_kernel.inc);
//   attn_bwd_dkdv_t32_kernel  dK / dV, its dual: K_w / V_w stationary, 32-query tiles of Q / dO streamed;
//                             head dims 128, (192, 128), 256 (dV and dK as two launches) with 32 keys per wave
//                             and 64 with 64 keys per wave (attn_bwd_dkdv_t32_kernel.inc).
// What is computed is described in attn_bwd.hip; how, at the top of the three kernel files; which calls they take, in
// dispatch.h.  A translation
// unit of its own, like attn_fwd_q64.hip, whose techniques it shares; compiled four times
// (ATTN_F16: 0 bf16, 1 fp16; ATTN_VARLEN: 0 fixed, 1 variable length), because the compiler takes minutes over
// these schedules.
#include "common.h"
#include "launch.h"

namespace attn {

#if ATTN_F16
namespace f16k {
#define ATTN_ELEM f16
#define ATTN_ELEM8 f16x8
#define ATTN_ELEM4 f16x4
#define ATTN_MFMA "v_mfma_f32_32x32x16_f16"
typedef __attribute__((ext_vector_type(2))) _Float16 elem2;
#else
#define ATTN_ELEM bf16
#define ATTN_ELEM8 bf16x8
#define ATTN_ELEM4 bf16x4
#define ATTN_MFMA "v_mfma_f32_32x32x16_bf16"
typedef bf16x2 elem2;
#endif
#include "elem.inc"
#include "attn_bwd_dq_q64_kernel.inc"
#include "attn_bwd_dkdv_t32_kernel.inc"
#include "attn_bwd_dq_t32_kernel.inc"
#include "attn_bwd_dq_q64_launch.inc"

#if ATTN_VARLEN
int run_bwd_dq_q64_varlen(const BwdArgs& a) { return launch_bwd_dq_q64_t(a); }
int run_bwd_dq_t32_varlen(const BwdArgs& a) { return launch_bwd_dq_t32_t(a); }
int run_bwd_dkdv_t32_varlen(const BwdArgs& a) { return launch_bwd_dkdv_t32_t(a); }
#else
int run_bwd_dq_q64(const BwdArgs& a) { return launch_bwd_dq_q64_t(a); }
int run_bwd_dq_t32(const BwdArgs& a) { return launch_bwd_dq_t32_t(a); }
int run_bwd_dkdv_t32(const BwdArgs& a) { return launch_bwd_dkdv_t32_t(a); }
#endif
#if ATTN_F16
}  // namespace f16k
#endif

}  // namespace attn
