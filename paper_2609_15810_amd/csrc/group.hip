// Value-guided grouping (Sec. 3.2 "Value-guided permutation"): per (batch, head) the value tokens
// are clustered and the keys/values are later gathered in cluster order.
//
// KMEANS: Lloyd rounds on per-head INT8 codes of V (scale amax/127 over the head). Centroid =
// round-half-even integer mean of its members (exact integer division), label = argmin of
// |C|^2 - 2 x.C in exact int32 (ties to the smallest cluster). Two routes with the same results:
//   N <= 1024      grp_head: one workgroup per head does everything, the codes in registers
//   N > 1024       grp_amax    per-head max |V|, one partial maximum per 256 tokens
//                  grp_assign  once per round: the centroids from the previous round's member sums
//                              (the first round: the initial centroids, and V to INT8 codes), labels
//                              and member sums on the matrix cores, sums added to the head's
//                              accumulators with integer atomics
//                  grp_scatter stable counting sort of the final labels, final centroids
// Integer arithmetic throughout makes labels, centroids and the permutation reproducible bit for
// bit regardless of the order in which partial sums are combined.
// CUBE: static cube order in closed form; IDENTITY: perm = 0..N-1.
#include "vc_common.hpp"
#include "vc_internal.hpp"

namespace vc {

constexpr int STOK = 1024;           // tokens per workgroup of the sort
constexpr int KMAX = 64;             // clusters supported by the kernels
constexpr int NORM_PAD = 8388000;    // |C|^2 of a padding cluster: above every real distance
constexpr int C8 = D + 16;           // LDS row of a centroid's int8 channels (16-byte rows, no bank conflicts)
constexpr int XW = D / 4 + 4;        // LDS row of a token's codes in words (144 bytes, likewise)
constexpr int XROWS = 32 * XW + 32;  // a wave's 32 rows; rows 16 .. 31 start half the banks further on

__device__ __forceinline__ float wave_fmax(float m) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  return m;
}

__device__ __forceinline__ float chunk_amax(const u4& w) {
  float m = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) m = fmaxf(m, fmaxf(fabsf(bf16_lo(w[q])), fabsf(bf16_hi(w[q]))));
  return m;
}

// 1.5 * 2^23 + the INT8 code rint(x * (127 / amax)) clamped to +-127 (amax = 0: inv = 0): the add
// rounds to the nearest integer, ties to even, and the low byte of the bits is its two's complement
__device__ __forceinline__ uint32_t code_bits(float x, float inv) {
  return __float_as_uint(__builtin_amdgcn_fmed3f(x * inv, -127.f, 127.f) + 12582912.f);   // NaN: -127
}
__device__ __forceinline__ uint32_t pack4(uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3) {
  return __builtin_amdgcn_perm(b1, b0, 0x0c0c0400u) | __builtin_amdgcn_perm(b3, b2, 0x04000c0cu);
}

// the codes of 8 channels (one 16-byte chunk of bf16)
__device__ __forceinline__ uint2 code_chunk(const u4& w, float inv) {
  uint32_t b[8];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    b[2 * e] = code_bits(bf16_lo(w[e]), inv);
    b[2 * e + 1] = code_bits(bf16_hi(w[e]), inv);
  }
  return make_uint2(pack4(b[0], b[1], b[2], b[3]), pack4(b[4], b[5], b[6], b[7]));
}

// num / den rounded to nearest, ties to even; den >= 1, |num| <= 127 den < 2^31. The estimate is off
// by less than 1e-4, so its nearest integer is right except next to a half, where the exact
// remainder corrects it by one.
__device__ __forceinline__ int32_t div_rne(int32_t num, int32_t den, float inv_den) {
  int32_t q = (int32_t)__builtin_rintf((float)num * inv_den);
  const int32_t rem2 = 2 * (num - q * den), odd = q & 1;
  q += rem2 + odd > den ? 1 : 0;    // rem2 > den, or = den with q odd
  q -= odd - rem2 > den ? 1 : 0;
  return q;
}

// A centroid is handled by 32 threads, thread col holding channels 4 col .. 4 col + 3 as one word of
// int8: the next round's from the members' sums and count.
__device__ __forceinline__ uint32_t next_centroid(const v4i& sum, int32_t cnt, uint32_t old) {
  const int32_t den = max(cnt, 1);
  const float inv = __builtin_amdgcn_rcpf((float)den);
  const uint32_t v = pack4(div_rne(sum[0], den, inv), div_rne(sum[1], den, inv), div_rne(sum[2], den, inv), div_rne(sum[3], den, inv));
  return cnt > 0 ? v : old;   // an empty cluster keeps its centroid
}

// initial centroid of cluster k, channels 4 col ..: the codes of token floor((2k+1) N / (2K)), or the
// caller's fp32 centroid requantized
__device__ __forceinline__ uint32_t initial_centroid(const GroupArgs& a, int bh, int k, int col, float inv) {
  float x[4];
  if (a.warm_start) {
    const float4 f = *reinterpret_cast<const float4*>(a.centroids + ((size_t)bh * a.k + k) * D + 4 * col);
    x[0] = f.x, x[1] = f.y, x[2] = f.z, x[3] = f.w;
  } else {
    const long long n0 = ((long long)(2 * k + 1) * a.N) / (2LL * a.k);
    const uint2 w = *reinterpret_cast<const uint2*>(a.V + ((size_t)bh * a.N + n0) * D + 4 * col);
    x[0] = bf16_lo(w.x), x[1] = bf16_hi(w.x), x[2] = bf16_lo(w.y), x[3] = bf16_hi(w.y);
  }
  return pack4(code_bits(x[0], inv), code_bits(x[1], inv), code_bits(x[2], inv), code_bits(x[3], inv));
}

template <int CTRL>
__device__ __forceinline__ int dpp_add(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}

// Centroid k's word v of thread col into the labels' operands: the negated channels in LDS (so that
// the product is -x.C) and the part of the argmin's key that does not depend on the token,
// (|C|^2 + 2^23) << 7 | k (rows K.. of the padding: NORM_PAD). v: channels within +-127.
__device__ __forceinline__ void publish_centroid(uint8_t (*c8)[C8], int32_t* base, int k, int col, uint32_t v, int K) {
  const uint32_t neg = 0x80808080u - (v & 0x7f7f7f7fu);   // per byte: 128 - low 7 bits ...
  const uint32_t w = neg ^ (v & 0x80808080u) ^ 0x80808080u;   // ... = -v in two's complement
  *reinterpret_cast<uint32_t*>(&c8[k][4 * col]) = w;
  int sq = __builtin_amdgcn_sdot4((int)v, (int)v, 0, false);
  sq = dpp_add<0xb1>(sq);    // quad lanes ^1
  sq = dpp_add<0x4e>(sq);    // quad lanes ^2
  sq = dpp_add<0x141>(sq);   // mirrored in 8
  sq = dpp_add<0x140>(sq);   // mirrored in 16
  sq += __shfl_xor(sq, 16);
  if (col == 0) base[k] = (((k < K ? sq : NORM_PAD) + (1 << 23)) << 7) | k;
}

// The wave's own LDS stores are in place for its other lanes' loads.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int NO_LABEL = 127;   // tokens past the head's end

// lanes of the wave whose label (7 bits) equals this lane's
__device__ __forceinline__ uint64_t same_label(int label) {
  uint64_t m = ~0ull;
#pragma unroll
  for (int b = 0; b < 7; ++b) {
    const uint64_t set = __builtin_amdgcn_ballot_w64((label >> b) & 1);
    m &= ((label >> b) & 1) ? set : ~set;
  }
  return m;
}
__device__ __forceinline__ int lanes_below(uint64_t m) {   // members of m below this lane
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// The labels' operands of a lane: centroid rows, and the keys' bases.
template <int KB>
struct Centroids {
  v4i row[KB][4], base[KB][4];
  __device__ __forceinline__ void load(const uint8_t (*c8)[C8], const int32_t* b, int lane) {
    const int kh = lane >> 5, col = lane & 31;
#pragma unroll
    for (int cb = 0; cb < KB; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        row[cb][i] = *reinterpret_cast<const v4i*>(&c8[32 * cb + col][32 * i + 16 * kh]);
        base[cb][i] = *reinterpret_cast<const v4i*>(b + 32 * cb + 8 * i + 4 * kh);
      }
  }
};

// Label of the lane's token (lane % 32 of the wave's 32 tokens, both halves get it):
//   S^T = -C X^T    INT8 MFMA 32x32x32, A = negated centroid rows, B = the tokens' codes; lane (token
//                   l%32, half l/32) holds 16 clusters' -x.C of each 32, the other 16 in lane l^32
//   key  = (|C|^2 - 2 x.C + 2^23) << 7 | cluster = base + (S << 8), argmin = integer min of the keys
//          (the distance fits 24 bits, the cluster 7; equal distances resolve to the smaller cluster)
template <int KB>
__device__ __forceinline__ int nearest(const v4i (&xb)[4], const Centroids<KB>& c) {
  int best = 0x7fffffff;
#pragma unroll
  for (int cb = 0; cb < KB; ++cb) {
    v16i S = {};
#pragma unroll
    for (int dc = 0; dc < 4; ++dc) S = __builtin_amdgcn_mfma_i32_32x32x32_i8(c.row[cb][dc], xb[dc], S, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 16; r += 2)
      best = min(min(best, (S[r] << 8) + c.base[cb][r >> 2][r & 3]), (S[r + 1] << 8) + c.base[cb][r >> 2][(r & 3) + 1]);
  }
  const auto o = __builtin_amdgcn_permlane32_swap((unsigned)best, (unsigned)best, false, false);
  return min(min(best, (int)o[0]), (int)o[1]) & 127;
}

// byte b of row r of a wave's 32 rows of codes
__device__ __forceinline__ int row_byte(int r, int b) { return 4 * (r * XW + ((r & 16) << 1)) + b; }

// B operands of the member sums: tokens (rows) 16 kh .. + 15 of channels 32 db + col, db = 0..3, byte
// i = token i. The LDS reads transpose: of the 16 lanes of a group, lane i brings bytes
// 8 (i % 2) .. + 7 of row i / 2 and receives byte i of all eight rows.
__device__ __forceinline__ void transposed(v4i (&x)[4], const uint8_t* rows, int lane) {
  typedef int v2i __attribute__((ext_vector_type(2)));
  const uint8_t* p = rows + row_byte(16 * (lane >> 5) + ((lane & 15) >> 1), (lane & 16) + 8 * (lane & 1));
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const v2i v = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
          (__attribute__((address_space(3))) v2i*)(p + 8 * h * XW * 4 + 32 * db));
      x[db][2 * h] = v[0];
      x[db][2 * h + 1] = v[1];
    }
}

// B operand of the labels: channels 32 dc + 16 kh .. of row col
__device__ __forceinline__ void token_rows(v4i (&x)[4], const uint8_t* rows, int lane) {
#pragma unroll
  for (int dc = 0; dc < 4; ++dc) x[dc] = *reinterpret_cast<const v4i*>(rows + row_byte(lane & 31, 32 * dc + 16 * (lane >> 5)));
}

// A operand of the member sums: -128 where the label of one of 16 tokens is the cluster (labels and
// clusters have 7 bits, so 128 - (label ^ cluster) keeps its top bit only where they are equal)
__device__ __forceinline__ v4i one_hot(const u4& labels, int cluster) {
  const uint32_t rep = (uint32_t)cluster * 0x01010101u;
  v4i oh;
#pragma unroll
  for (int q = 0; q < 4; ++q) oh[q] = (int32_t)((0x80808080u - (labels[q] ^ rep)) & 0x80808080u);
  return oh;
}
// ... and how many there are, times -128
__device__ __forceinline__ int32_t count_hot(const v4i& oh, int32_t n) {
#pragma unroll
  for (int q = 0; q < 4; ++q) n = __builtin_amdgcn_sdot4(oh[q], 0x01010101, n, false);
  return n;
}

// A wave's member sums of cluster block cb (times -128) added to the workgroup's in LDS
__device__ __forceinline__ void add_sums(int32_t (*acc)[D], int cb, int db, const v16i& sums, int lane) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
    atomicAdd(&acc[32 * cb + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)][32 * db + (lane & 31)], sums[r]);
}

// ------------------------------------------------------------------------------------------
// N > 1024
// ------------------------------------------------------------------------------------------

// Each workgroup reduces 64 KB of the head (16 chunks of 16 bytes per thread, all loads issued
// before the first use; chunks past the head's end re-read its last chunk) to one partial maximum.
// The member sums and counts of the first round and the label counts are cleared on the way.
__global__ __launch_bounds__(256) void grp_amax(GroupArgs a) {
  __shared__ float red[4];
  const int bh = blockIdx.y;
  const size_t words = (size_t)a.N * D / 8;  // 16-byte chunks of the head
  const u4* src = reinterpret_cast<const u4*>(a.V + (size_t)bh * a.N * D);
  u4 w[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) w[u] = src[min(((size_t)blockIdx.x * 16 + u) * 256 + threadIdx.x, words - 1)];
  for (int i = blockIdx.x * 256 + threadIdx.x; i < a.k * (D + 1); i += gridDim.x * 256) a.sums[(size_t)bh * a.sums_head + i] = 0;
  if (blockIdx.x % (STOK / 256) == 0 && (int)threadIdx.x < a.k) a.hist[((size_t)bh * a.nsort + blockIdx.x / (STOK / 256)) * a.k + threadIdx.x] = 0;
  float m = 0.f;
#pragma unroll
  for (int u = 0; u < 16; ++u) m = fmaxf(m, chunk_amax(w[u]));
  m = wave_fmax(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0)   // one partial per workgroup (gridDim.x = nblk), reduced by the first grp_assign
    a.amax_part[(size_t)bh * gridDim.x + blockIdx.x] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// The head's member sums [k][128] and, behind them, counts [k] of round r: three buffers in turn,
// so that round r adds to one, reads the previous round's and clears the next round's.
__device__ __forceinline__ int32_t* round_sums(const GroupArgs& a, int r, int bh) {
  return a.sums + ((size_t)(r % 3) * a.BH + bh) * a.sums_head;
}
// The head's int8 centroids [k][128] of round r (two buffers in turn; an empty cluster keeps its
// centroid)
__device__ __forceinline__ uint32_t* round_cent(const GroupArgs& a, int r, int bh) {
  return reinterpret_cast<uint32_t*>(a.cent8) + ((size_t)(r & 1) * a.BH + bh) * a.k * (D / 4);
}

constexpr int AW = 8;            // waves per assignment workgroup
constexpr int ACH = 32 * AW;     // tokens per step of the workgroup: 32 per wave

// One Lloyd round of a head's tokens wg * atok .. + atok - 1 (KB = clusters / 32, rounded up). Each
// wave takes 32 tokens at a time, on its own: it brings their codes into its LDS rows with coalesced
// loads issued one step ahead (the first round makes them from V and stores them), labels them, and
// adds them to its member sums, sums[db] += O X, an INT8 product with A = one-hot labels (cluster
// rows x 32 tokens) and B = the transposed codes of channels 4 col + db. At the end the waves' sums
// meet in LDS and go to the head's accumulators. The centroids are formed in every workgroup from
// the previous round's accumulators, which saves a launch per round.
// Bound by instruction issue (products and vector work of a SIMD hardly overlap: 8 products and about
// 70 vector instructions per 32 tokens) and, for few tokens per workgroup, by the latency of its
// start and end, hence one operand load for the four sum products and the transposition by the LDS
// read itself. A round of 12 heads of 32760 tokens takes 11.9 us (first round 29.1, which also moves
// 150 MB); with 256-token chunks shared by waves that took one channel byte each (two barriers per
// chunk, 16 byte permutes and four times the LDS reads per product) it took 15.5 us, and with a
// launch of its own for the centroids and the sums in per-workgroup partials 17.4 + 8.2 us.
template <int KB, bool FIRST>
__global__ __launch_bounds__(AW * 64, 2) void grp_assign(GroupArgs a, int round, int last) {
  constexpr int NT = AW * 64;
  __shared__ __attribute__((aligned(16))) uint8_t c8[KB * 32][C8];
  __shared__ __attribute__((aligned(16))) int32_t base[KB * 32];
  __shared__ __attribute__((aligned(16))) uint8_t lab[AW][32];
  __shared__ __attribute__((aligned(16))) uint8_t xs[AW][4 * XROWS];
  __shared__ __attribute__((aligned(16))) int32_t acc[KB * 32][D];
  __shared__ int32_t cnts[KB * 32];
  __shared__ float red[AW];
  // the first round walks the heads backwards: the last ones, just read by grp_amax, may be cached
  const int bh = FIRST ? gridDim.y - 1 - blockIdx.y : blockIdx.y;
  const int wg = FIRST ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kh = lane >> 5, col = lane & 31, K = a.k, N = a.N;
  const int wbase = wg * a.atok, wend = min(wbase + a.atok, N);
  constexpr int NLD = FIRST ? 8 : 4;   // 16-byte chunks per lane of the wave's 32 rows
  const char* src = FIRST ? reinterpret_cast<const char*>(a.V + (size_t)bh * N * D)
                          : reinterpret_cast<const char*>(a.codes + (size_t)bh * N * D);
  uint2* cdst = reinterpret_cast<uint2*>(a.codes + (size_t)bh * N * D);
  // rows n0 .. n0 + 31, those past N re-reading the last one (a head's bytes fit 32 bits)
  auto load = [&](int n0, u4 (&w)[NLD]) __attribute__((always_inline)) {
    constexpr int ROW = 32 * NLD;   // bytes of a row
    if (n0 + 32 <= N) {
      const uint32_t o = (uint32_t)n0 * ROW + 16 * lane;
#pragma unroll
      for (int u = 0; u < NLD; ++u) w[u] = *reinterpret_cast<const u4*>(src + o + 1024 * u);
    } else {
#pragma unroll
      for (int u = 0; u < NLD; ++u) {
        const uint32_t q = 1024 * u + 16 * lane;
        w[u] = *reinterpret_cast<const u4*>(src + (uint32_t)min(n0 + (int)(q / ROW), N - 1) * ROW + q % ROW);
      }
    }
  };

  // this round's centroids, and the next round's sums cleared
  constexpr int KS = NT / 32, NC = KB * 32 / KS;   // clusters of this thread: tid / 32 + KS i
  u4 w[NLD];
  float inv = 0.f;
  if constexpr (FIRST) {
    float m = 0.f;
    for (int i = tid; i < a.nblk; i += NT) m = fmaxf(m, a.amax_part[(size_t)bh * a.nblk + i]);
    m = wave_fmax(m);
    if (lane == 0) red[wave] = m;
    __syncthreads();
    m = red[0];
#pragma unroll
    for (int i = 1; i < AW; ++i) m = fmaxf(m, red[i]);
    inv = m > 0.f ? 127.f / m : 0.f;
    if (wg == 0 && tid == 0) a.scale[bh] = m;   // for the centroids' values
  }
  {
    uint32_t v[NC];
    if constexpr (FIRST) {
#pragma unroll
      for (int i = 0; i < NC; ++i) v[i] = initial_centroid(a, bh, min((tid >> 5) + KS * i, K - 1), col, inv);
    } else {
      const int32_t* ps = round_sums(a, round + 2, bh);   // round - 1
      const uint32_t* pc = round_cent(a, round + 1, bh);
      v4i sv[NC];
      int32_t nv[NC];
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int k = min((tid >> 5) + KS * i, K - 1);
        sv[i] = *reinterpret_cast<const v4i*>(ps + k * D + 4 * col);
        nv[i] = ps[K * D + k];
        v[i] = pc[k * (D / 4) + col];
      }
      load(wbase + 32 * wave, w);
#pragma unroll
      for (int i = 0; i < NC; ++i) v[i] = next_centroid(sv[i], nv[i], v[i]);
    }
    uint32_t* oc = round_cent(a, round, bh);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int k = (tid >> 5) + KS * i;
      if (k < K && wg == 0) oc[k * (D / 4) + col] = v[i];
      publish_centroid(c8, base, k, col, k < K ? v[i] : 0u, K);
    }
    int32_t* ns = round_sums(a, round + 1, bh);
    for (int i = wg * NT + tid; i < K * (D + 1); i += gridDim.x * NT) ns[i] = 0;
    for (int i = tid; i < KB * 32 * D / 4; i += NT) reinterpret_cast<v4i*>(&acc[0][0])[i] = v4i{0, 0, 0, 0};
    if (tid < KB * 32) cnts[tid] = 0;
  }
  __syncthreads();

  v16i sums[KB][4];
  int32_t cnt[KB];
#pragma unroll
  for (int cb = 0; cb < KB; ++cb) {
    cnt[cb] = 0;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) sums[cb][db][r] = 0;
  }
  uint8_t* rows = xs[wave];
  Centroids<KB> cent;
  if constexpr (KB == 1) cent.load(c8, base, lane);
#pragma unroll 1
  for (int n0 = wbase + 32 * wave; n0 < wend; n0 += ACH) {
    if constexpr (FIRST) load(n0, w);
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int q = u * 64 + lane;
      if constexpr (FIRST) {
        const uint2 v = code_chunk(w[u], inv);
        *reinterpret_cast<uint2*>(rows + row_byte(q >> 4, 8 * (q & 15))) = v;
        if (n0 + (q >> 4) < N) cdst[(size_t)n0 * 16 + q] = v;
      } else {
        *reinterpret_cast<u4*>(rows + row_byte(q >> 3, 16 * (q & 7))) = w[u];
      }
    }
    if constexpr (!FIRST) load(min(n0 + ACH, N - 1), w);   // the next step's rows in flight
    wave_sync();
    v4i x[4];
    token_rows(x, rows, lane);
    if constexpr (KB > 1) cent.load(c8, base, lane);   // 64 registers that two cluster blocks can't keep
    int label = nearest<KB>(x, cent);
    label = n0 + col < N ? label : NO_LABEL;
    if (kh == 0) lab[wave][col] = (uint8_t)label;
    wave_sync();
    transposed(x, rows, lane);
    const u4 l4 = *reinterpret_cast<const u4*>(&lab[wave][16 * kh]);
#pragma unroll
    for (int cb = 0; cb < KB; ++cb) {
      const v4i oh = one_hot(l4, 32 * cb + col);
#pragma unroll
      for (int db = 0; db < 4; ++db) sums[cb][db] = __builtin_amdgcn_mfma_i32_32x32x32_i8(oh, x[db], sums[cb][db], 0, 0, 0);
      cnt[cb] = count_hot(oh, cnt[cb]);
    }
    if (last) {   // labels, and their counts per STOK tokens for the sort
      const uint64_t same = same_label(label) & 0xffffffffull;
      if (kh == 0 && label != NO_LABEL) {
        a.labels[(size_t)bh * N + n0 + col] = label;
        if (lanes_below(same) == 0) atomicAdd(&a.hist[((size_t)bh * a.nsort + n0 / STOK) * K + label], __builtin_popcountll(same));
      }
    }
    wave_sync();   // the rows and labels are overwritten next
  }
#pragma unroll
  for (int cb = 0; cb < KB; ++cb) {
#pragma unroll
    for (int db = 0; db < 4; ++db) add_sums(acc, cb, db, sums[cb][db], lane);
    atomicAdd(&cnts[32 * cb + col], cnt[cb]);
  }
  __syncthreads();
  int32_t* out = round_sums(a, round, bh);
  for (int i = tid; i < K * D; i += NT) {
    const int32_t v = (&acc[0][0])[i];
    if (v) atomicAdd(out + i, -(v >> 7));
  }
  if (tid < K && cnts[tid]) atomicAdd(out + K * D + tid, -(cnts[tid] >> 7));
}

// word i of the head's centroids in value units
__device__ __forceinline__ void store_centroid(const GroupArgs& a, int bh, int i, uint32_t v, float scale) {
  const float4 f = {(float)(int8_t)v * scale, (float)(int8_t)(v >> 8) * scale, (float)(int8_t)(v >> 16) * scale,
                    (float)(int8_t)(v >> 24) * scale};
  reinterpret_cast<float4*>(a.centroids + (size_t)bh * a.k * D)[i] = f;
}

// Stable counting sort of the final labels, 1024 tokens per workgroup: a token's row is the number of
// tokens with smaller labels, plus those with its label in earlier workgroups (both from the label
// counts), plus its rank in its own workgroup. The workgroups also write the centroids in value units.
__global__ __launch_bounds__(256) void grp_scatter(GroupArgs a, int rounds) {
  __shared__ int32_t tot[4][KMAX], before[4][KMAX];
  __shared__ int32_t first[STOK / 64][KMAX];   // row of the first token of each label in each 64-token group
  const int bh = blockIdx.y, wg = blockIdx.x, t = threadIdx.x, wave = t >> 6, lane = t & 63, K = a.k, N = a.N;
  int label[STOK / 256], rank[STOK / 256];   // 64-token groups wave, wave + 4, ...
#pragma unroll
  for (int i = 0; i < STOK / 256; ++i) {
    const int n = wg * STOK + 64 * (wave + 4 * i) + lane;
    label[i] = n < N ? a.labels[(size_t)bh * N + n] : NO_LABEL;
  }
  // label l = lane: sums over the workgroups' counts, a quarter of them per wave
  {
    const int32_t* h = a.hist + (size_t)bh * a.nsort * K;
    int32_t s = 0, b = 0;
    if (lane < K) {
#pragma unroll 8
      for (int p = wave; p < a.nsort; p += 4) {
        const int32_t v = h[(size_t)p * K + lane];
        s += v;
        b += p < wg ? v : 0;
      }
    }
    tot[wave][lane] = s;
    before[wave][lane] = b;
  }
#pragma unroll
  for (int i = 0; i < STOK / 256; ++i) {
    first[wave + 4 * i][lane] = 0;
    wave_sync();
    const uint64_t same = same_label(label[i]);
    rank[i] = lanes_below(same);
    if (rank[i] == 0 && label[i] < KMAX) first[wave + 4 * i][label[i]] = __builtin_popcountll(same);
  }
  __syncthreads();
  if (t < KMAX) {   // one wave: exclusive scan of the labels' totals, then the groups' counts in turn
    int32_t all = tot[0][t] + tot[1][t] + tot[2][t] + tot[3][t];
    int32_t run = all;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t v = __shfl_up(run, o);
      run += t >= o ? v : 0;
    }
    run += before[0][t] + before[1][t] + before[2][t] + before[3][t] - all;
#pragma unroll
    for (int g = 0; g < STOK / 64; ++g) {
      const int32_t n = first[g][t];
      first[g][t] = run;
      run += n;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < STOK / 256; ++i) {
    if (label[i] < KMAX) {
      const int n = wg * STOK + 64 * (wave + 4 * i) + lane;
      const int pos = first[wave + 4 * i][label[i]] + rank[i];
      a.perm[(size_t)bh * N + pos] = n;
      if (a.inv_perm) a.inv_perm[(size_t)bh * N + n] = pos;
    }
  }
  // centroids: after the last round's update (none with iters = 0)
  const float amax = a.scale[bh];
  const float scale = amax > 0.f ? amax / 127.f : 1.f;
  const int32_t* ls = round_sums(a, rounds - 1, bh);
  const uint32_t* lc = round_cent(a, rounds - 1, bh);
  for (int i = wg * 256 + t; i < K * 32; i += gridDim.x * 256) {
    const int k = i >> 5, col = i & 31;
    const v4i sum = *reinterpret_cast<const v4i*>(ls + k * D + 4 * col);
    store_centroid(a, bh, i, a.iters > 0 ? next_centroid(sum, ls[K * D + k], lc[i]) : lc[i], scale);
  }
}

// ------------------------------------------------------------------------------------------
// N <= 1024: one workgroup per head, 8 waves. The codes of a wave's tokens (4 x 32) stay in registers
// in both operand orders, so a round touches only centroids, labels and sums in LDS. Launches and
// their latency were the whole cost of such heads: two heads of 1024 tokens take 37 us, with 22
// launches they took 140 us, and on the other route (10 launches) 58 us. 1024 tokens are what one
// workgroup's registers hold in both orders.
// ------------------------------------------------------------------------------------------
constexpr int HTOK = 1024;
constexpr int HW = AW;

template <int KB>
__global__ __launch_bounds__(HW * 64, 2) void grp_head(GroupArgs a) {
  constexpr int NT = HW * 64, NS = HTOK / ACH;   // 32-token label steps per wave
  constexpr int NC = KB * 32 * 32 / NT;          // clusters of this thread: tid / 32 + 16 i
  __shared__ __attribute__((aligned(16))) uint8_t c8[KB * 32][C8];
  __shared__ __attribute__((aligned(16))) int32_t base[KB * 32];
  __shared__ __attribute__((aligned(16))) uint8_t lab[HTOK];
  __shared__ int32_t first[HTOK / 64][KMAX];
  __shared__ float red[HW];
  __shared__ __attribute__((aligned(16))) uint8_t xs[HW][4 * XROWS];
  __shared__ __attribute__((aligned(16))) int32_t acc[KB * 32][D];
  __shared__ int32_t cnts[KB * 32];
  const int bh = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kh = lane >> 5, col = lane & 31, K = a.k, N = a.N;
  const u4* src = reinterpret_cast<const u4*>(a.V + (size_t)bh * N * D);

  // chunk i (tokens 256 i ..): 8 16-byte chunks per lane of the wave's 32 rows
  auto load = [&](int i, u4 (&w)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 8; ++u) w[u] = src[min((ACH * i + 32 * wave) * 16 + u * 64 + lane, N * 16 - 1)];
  };
  float m = 0.f;
  {
    u4 w[NS][8];
#pragma unroll
    for (int i = 0; i < NS; ++i) load(i, w[i]);
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
      for (int u = 0; u < 8; ++u) m = fmaxf(m, chunk_amax(w[i][u]));
  }
  m = wave_fmax(m);
  if (lane == 0) red[wave] = m;
  __syncthreads();
  float amax = red[0];
#pragma unroll
  for (int i = 1; i < HW; ++i) amax = fmaxf(amax, red[i]);
  const float inv = amax > 0.f ? 127.f / amax : 0.f;

  // the thread's words of the centroids
  uint32_t cw[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) cw[i] = initial_centroid(a, bh, min((tid >> 5) + 16 * i, K - 1), col, inv);

  // both operands of tokens 256 i + 32 wave ..
  uint8_t* rows = xs[wave];
  v4i xb[NS][4], xt[NS][4];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    if (ACH * i + 32 * wave >= N) break;
    u4 w[8];
    load(i, w);   // again: holding all of V beside the operands would spill, and it is in the cache now
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int q = u * 64 + lane;
      *reinterpret_cast<uint2*>(rows + row_byte(q >> 4, 8 * (q & 15))) = code_chunk(w[u], inv);
    }
    wave_sync();
    token_rows(xb[i], rows, lane);
    transposed(xt[i], rows, lane);
    wave_sync();
  }
#pragma unroll
  for (int i = 0; i < KB * 32 * D / NT; ++i) (&acc[0][0])[i * NT + tid] = 0;
  if (tid < KB * 32) cnts[tid] = 0;
  if (tid < HTOK / 16) reinterpret_cast<u4*>(lab)[tid] = u4{1, 1, 1, 1} * (NO_LABEL * 0x01010101u);

  const int rounds = a.iters > 0 ? a.iters : 1;
#pragma unroll 1
  for (int round = 0; round < rounds; ++round) {
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int k = (tid >> 5) + 16 * i;
      publish_centroid(c8, base, k, col, k < K ? cw[i] : 0u, K);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int n0 = ACH * i + 32 * wave;
      if (n0 >= N) break;
      Centroids<KB> cent;
      cent.load(c8, base, lane);
      const int label = nearest<KB>(xb[i], cent);
      if (kh == 0 && n0 + col < N) lab[n0 + col] = (uint8_t)label;
    }
    if (a.iters == 0) break;
    wave_sync();
#pragma unroll
    for (int cb = 0; cb < KB; ++cb) {
      v16i sums[4] = {};
      int32_t cnt = 0;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const int n0 = ACH * i + 32 * wave;
        if (n0 >= N) break;
        const v4i oh = one_hot(*reinterpret_cast<const u4*>(&lab[n0 + 16 * kh]), 32 * cb + col);
#pragma unroll
        for (int db = 0; db < 4; ++db) sums[db] = __builtin_amdgcn_mfma_i32_32x32x32_i8(oh, xt[i][db], sums[db], 0, 0, 0);
        cnt = count_hot(oh, cnt);
      }
#pragma unroll
      for (int db = 0; db < 4; ++db) add_sums(acc, cb, db, sums[db], lane);
      atomicAdd(&cnts[32 * cb + col], cnt);
    }
    __syncthreads();
    int32_t n[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) n[i] = cnts[(tid >> 5) + 16 * i];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int k = (tid >> 5) + 16 * i;
      v4i* p = reinterpret_cast<v4i*>(&acc[k][4 * col]);
      const v4i sum = -(*p >> 7);
      *p = v4i{0, 0, 0, 0};
      cw[i] = next_centroid(sum, -(n[i] >> 7), cw[i]);
      if (col == 0) cnts[k] = 0;   // read by this half wave alone, above
    }
  }
  __syncthreads();

  // centroids in value units; the stable counting sort of the labels
  const float scale = amax > 0.f ? amax / 127.f : 1.f;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int k = (tid >> 5) + 16 * i;
    if (k < K) store_centroid(a, bh, k * (D / 4) + col, cw[i], scale);
  }
  int label[2], rank[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int g = 2 * wave + i, n = 64 * g + lane;
    label[i] = n < N ? lab[n] : NO_LABEL;
    first[g][lane] = 0;
    wave_sync();
    const uint64_t same = same_label(label[i]);
    rank[i] = lanes_below(same);
    if (rank[i] == 0 && label[i] < KMAX) first[g][label[i]] = __builtin_popcountll(same);
  }
  __syncthreads();
  if (tid < KMAX) {
    int32_t all = 0;
#pragma unroll
    for (int g = 0; g < HTOK / 64; ++g) all += first[g][tid];
    int32_t run = all;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t v = __shfl_up(run, o);
      run += tid >= o ? v : 0;
    }
    run -= all;
#pragma unroll
    for (int g = 0; g < HTOK / 64; ++g) {
      const int32_t n = first[g][tid];
      first[g][tid] = run;
      run += n;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int g = 2 * wave + i, n = 64 * g + lane;
    if (n < N) {
      const int pos = first[g][label[i]] + rank[i];
      a.labels[(size_t)bh * N + n] = label[i];
      a.perm[(size_t)bh * N + pos] = n;
      if (a.inv_perm) a.inv_perm[(size_t)bh * N + n] = pos;
    }
  }
}

// Static cube order in closed form: the tokens of all cubes before cube (ca, cb, cc) in raster
// order, plus the token's raster rank inside its (possibly clipped) cube.
__global__ __launch_bounds__(256) void grp_cube(GroupArgs a) {
  const int bh = blockIdx.y;
  const int n = blockIdx.x * 256 + threadIdx.x;
  if (n >= a.N) return;
  const int x = n % a.Wd, y = (n / a.Wd) % a.Ht, f = n / (a.Wd * a.Ht);
  const int ca = f / a.cube_t, cb = y / a.cube_h, cc = x / a.cube_w;
  const int ft = min(a.cube_t, a.F - ca * a.cube_t), ht = min(a.cube_h, a.Ht - cb * a.cube_h);
  const int wt = min(a.cube_w, a.Wd - cc * a.cube_w);
  const long long pos = (long long)ca * a.cube_t * a.Ht * a.Wd +
                        (long long)ft * ((long long)cb * a.cube_h * a.Wd + (long long)ht * cc * a.cube_w) +
                        (long long)(f - ca * a.cube_t) * ht * wt + (long long)(y - cb * a.cube_h) * wt + (x - cc * a.cube_w);
  const int ny = (a.Ht + a.cube_h - 1) / a.cube_h, nx = (a.Wd + a.cube_w - 1) / a.cube_w;
  a.labels[(size_t)bh * a.N + n] = (ca * ny + cb) * nx + cc;
  a.perm[(size_t)bh * a.N + pos] = n;
  if (a.inv_perm) a.inv_perm[(size_t)bh * a.N + n] = (int32_t)pos;
}

__global__ __launch_bounds__(256) void grp_identity(GroupArgs a) {
  const int bh = blockIdx.y;
  const int n = blockIdx.x * 256 + threadIdx.x;
  if (n >= a.N) return;
  a.labels[(size_t)bh * a.N + n] = 0;
  a.perm[(size_t)bh * a.N + n] = n;
  if (a.inv_perm) a.inv_perm[(size_t)bh * a.N + n] = n;
}

hipError_t launch_group(const GroupArgs& a, int BH, hipStream_t s) {
  const dim3 tok((a.N + 255) / 256, BH);
  if (a.mode == 0) {
    grp_identity<<<tok, 256, 0, s>>>(a);
    return hipGetLastError();
  }
  if (a.mode == 1) {
    grp_cube<<<tok, 256, 0, s>>>(a);
    return hipGetLastError();
  }
  if (a.N <= HTOK) {
    if (a.k <= 32) grp_head<1><<<BH, HW * 64, 0, s>>>(a);
    else grp_head<2><<<BH, HW * 64, 0, s>>>(a);
    return hipGetLastError();
  }
  const int rounds = a.iters > 0 ? a.iters : 1;
  const dim3 grid((a.N + a.atok - 1) / a.atok, BH);
  grp_amax<<<tok, 256, 0, s>>>(a);
  if (a.k <= 32) grp_assign<1, true><<<grid, AW * 64, 0, s>>>(a, 0, rounds == 1);
  else grp_assign<2, true><<<grid, AW * 64, 0, s>>>(a, 0, rounds == 1);
  for (int r = 1; r < rounds; ++r) {
    if (a.k <= 32) grp_assign<1, false><<<grid, AW * 64, 0, s>>>(a, r, r == rounds - 1);
    else grp_assign<2, false><<<grid, AW * 64, 0, s>>>(a, r, r == rounds - 1);
  }
  grp_scatter<<<dim3(a.nsort, BH), 256, 0, s>>>(a, rounds);
  return hipGetLastError();
}

}  // namespace vc
