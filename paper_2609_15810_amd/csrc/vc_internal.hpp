// Internal launch arguments and launchers (not part of the public ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vc_attn.h"

namespace vc {

struct PrepArgs {
  const uint16_t *Q, *K, *V;
  const int32_t *perm, *q_perm;
  const float *rope_cos, *rope_sin;
  int8_t* q;
  float* q_scale;
  int8_t* k;
  float* k_scale;
  float* k_mean;
  uint8_t* v;
  float* v_scale;
  uint16_t* v_mean;
  uint8_t *q_mxs, *k_mxs;  // E8M0 scale bytes (MXFP4 only)
  float* ws_ksum;   // [B*H][T][128] per-block key channel sums
  float* ws_vamax;  // [B*H][T][128] per-block residual maxima
  float* ws_vinv;   // [B*H][128]    448 / amax (0 for an all-zero channel)
  int N, T, F, Ht, Wd;
  float inv_w, inv_hw;  // 1/Wd and 1/(Ht*Wd) in fp32: estimates for the token-position divisions
  int rope, hadamard, smooth_k, smooth_v;
  int qk_fmt;
};

struct FwdArgs {
  const int8_t* q;
  const float* q_scale;
  const int8_t* k;
  const float* k_scale;
  const uint8_t* v;
  const float* v_scale;
  const uint16_t* v_mean;
  const uint8_t *q_mxs, *k_mxs;  // E8M0 scale bytes (MXFP4 only)
  const int32_t* q_perm;
  uint16_t* O;
  uint8_t* p_codes;  // debugging: the probability codes of every tile [B*H][N][128 T], or null
  int N, T;
  float kappa;      // sm_scale * log2(e) (/ 128 with the Hadamard rotation), rounded once to fp32
  float cbias;      // fl(120 + beta)
  int p_mode, smooth_v;
  int qk_fmt;
  int first;        // a launch's first workgroup (in order of head and query)
};

// How a call's rows are dealt to the attention kernels: n8 workgroups of 256 queries, n4 of 128 and n1 of
// 32, each counted in order of head and query (a head's last workgroup may be ragged); first4 and first1 are
// the positions of the first ones behind those before them.
struct ForwardPlan {
  int n8, first4, n4, first1, n1;
};

struct GroupArgs {
  const uint16_t* V;
  float* centroids;
  int32_t *labels, *perm, *inv_perm;
  // workspace (k-means)
  int8_t* codes;      // [B*H][N][128] INT8 codes of V
  float* scale;       // [B*H] max |V|
  float* amax_part;   // [B*H][nblk] its partial maxima
  int8_t* cent8;      // [2][B*H][k][128] the centroids of a round and the one before
  int32_t* sums;      // [3][B*H][sums_head] member sums [k][128] and counts [k] of three rounds in turn
  int32_t* hist;      // [B*H][nsort][k] final label counts per 1024 tokens
  int BH, N, F, Ht, Wd, k, iters, warm_start, mode, cube_t, cube_h, cube_w;
  int nblk;           // 256-token blocks per head
  int sums_head;      // k * 129 rounded up to 16 bytes
  int nsort;          // 1024-token blocks per head
  int atok;           // tokens per assignment workgroup (a multiple of 256)
};

hipError_t launch_prep(const PrepArgs& a, int BH, hipStream_t s);
ForwardPlan forward_plan(int N, int BH, int qk_fmt, int p_mode);
hipError_t launch_forward(FwdArgs a, int BH, hipStream_t s);
hipError_t launch_group(const GroupArgs& a, int BH, hipStream_t s);
hipError_t launch_fp8_score_product(const uint8_t* a, const uint8_t* b, const float* c_in, float* out, int n,
                                    hipStream_t s);

}  // namespace vc

// The plan of a call, for tests on the host (not part of the public ABI): n8, first4, n4, first1, n1.
extern "C" void vc_internal_forward_plan(int32_t N, int32_t BH, int32_t qk_fmt, int32_t p_mode, int32_t plan[5]);
