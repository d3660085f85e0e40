// Block-INT8 QKV records (Sec. 3.2, "Quantized communication"): the wire
// format of the sequence-parallel QKV exchange, one 400-byte record per
// (token, head).  The encoder is the sender's producer: it normalises and
// rotates q and k (Sec. 3.5, fusion group 2) and quantises q, k and v in one
// pass, so the bf16 q^, k^ never reach HBM.  The decoder writes the bf16
// tensors back (for consumers other than this library's attention, which
// decodes records in its own tile loads).  Both kernels stream: 768 bytes read
// and 400 written per record (encoder), the reverse (decoder).
// The quantisation rule (scale choice, rounding) lives in sol_device.h, shared
// with the attention kernel's block-INT8 output epilogue.
#include "sol_device.h"

namespace sol {
namespace {

constexpr int kRecPerWg = 4;                 // records per workgroup (decoder)
constexpr int kRecThreads = 48 * kRecPerWg;  // one thread per 16-byte chunk of q, k and v
constexpr int kEncTokens = 16;               // tokens per workgroup (encoder)
constexpr int kEncThreads = kEncTokens * kChunks;

// Scale code of a group of bf16 values with largest magnitude amax:
// ue5m3_scale_for without its two exact comparisons.  amax = X 2^j with X an
// 8-bit integer, so amax / 127 is a scale value only where 127 divides X --
// X = 127 or 254, where t below is exact -- and otherwise lies at least 2^-10
// of itself from every scale value (multiples of 1/8 2^k, 2^-17 among the
// subnormal codes) while t carries an error of 2^-23: rounding t up to a scale
// value gives the definition's code for every bf16 (all of them are checked by
// a test).
__device__ __forceinline__ uint32_t ue5m3_scale_for_bf16(float amax) {
  const float t = amax * (1.0f / 127.0f);
  const uint32_t u = __float_as_uint(t);  // compared as bits, for NaN's sake
  const int normal = (int)((u + 0xFFFFFu) >> 20) - (112 << 3);
  const int subnormal = (int)__builtin_ceilf(t * 0x1p17f);
  const int c = u < 0x38800000u ? subnormal : normal;  // 2^-14
  // a group of NaN gets 0xF6, as from ue5m3_scale_for
  return (uint32_t)(u > 0x7F800000u ? 0xF6 : min(max(c, 1), 0xF7));
}

// 1 / s of a scale value as two floats, hi the nearest and lo the rest (the
// hardware reciprocal is within an ulp; one Newton step makes it the nearest),
// and the largest magnitude it codes, 127 s (exact).
struct ScaleInv {
  float hi, lo, top;
};
__device__ __forceinline__ ScaleInv scale_inv(float s) {
  const float r = __builtin_amdgcn_rcpf(s);
  ScaleInv v;
  v.hi = __builtin_fmaf(__builtin_fmaf(-s, r, 1.0f), r, r);
  v.lo = __builtin_fmaf(-s, v.hi, 1.0f) * v.hi;
  v.top = 127.0f * s;
  return v;
}
// A quad's lane (kCtrl) hands its own to the other three.
template <int kCtrl>
__device__ __forceinline__ ScaleInv from_lane(ScaleInv v) {
  return ScaleInv{dpp<kCtrl>(v.hi), dpp<kCtrl>(v.lo), dpp<kCtrl>(v.top)};
}

// Eight bf16 values -> eight int8 codes of scale s, x / s rounded to nearest,
// ties to even (one 8-byte word).  x (hi + lo) rounded once to fp32 is exact
// where x / s is a tie; where it is not, x / s -- an 8-bit over a 4-bit
// integer, times a power of two -- lies at least 2^-13 from one, far over the
// product's error.  Adding 1.5 2^23 rounds it to an integer in the low byte
// (checked for every bf16 against every scale by a test).  5 instructions a
// value, against 13 for a quotient settled by its exact residual (int8_code,
// which takes any fp32).
__device__ __forceinline__ uint2 encode_chunk(const float (&f)[8], ScaleInv inv) {
  uint32_t c[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    // past 127 s only where no scale is large enough, and for infinities
    const float x = __builtin_amdgcn_fmed3f(f[e], -inv.top, inv.top);
    c[e] = __float_as_uint(__builtin_fmaf(x, inv.hi, x * inv.lo) + 12582912.0f);
  }
  uint32_t w[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const uint32_t lo = __builtin_amdgcn_perm(c[4 * u + 1], c[4 * u], 0x0C0C0400);
    const uint32_t hi = __builtin_amdgcn_perm(c[4 * u + 3], c[4 * u + 2], 0x0C0C0400);
    w[u] = __builtin_amdgcn_perm(hi, lo, 0x05040100);
  }
  return make_uint2(w[0], w[1]);
}

// Largest magnitude over the 4 lanes that hold a scale group's chunks.
__device__ __forceinline__ float group_amax(const float (&f)[8]) {
  float a = fabsf(f[0]);
#pragma unroll
  for (int e = 1; e < 8; ++e) a = fmaxf(a, fabsf(f[e]));
  a = fmaxf(a, dpp<kDppXor1>(a));
  return fmaxf(a, dpp<kDppXor2>(a));
}

// 16 lanes per token, one 16-byte chunk of q, k and v each (a row in 16
// aligned lanes, as the normalisation's row sums need; a scale group in 4),
// through `per_wg` heads of the token (grid.y walks the groups of heads).
//
// The floor is q, k and v read and the records written (1168 bytes a record);
// the kernel is bound by its VALU instructions, so what a thread's three
// chunks or the heads of its token share is done once: the position, cosines
// and sines once a token, 1 / rms of q in the even lanes and of k in the odd
// ones, the scale of q, k and v in lanes 0, 1 and 2 of a quad, each handed to
// the others by DPP.  The next head's chunks are loaded ahead of this one's
// arithmetic.  14,400 tokens of 40 heads, normalised and rotated: 146 us = 4.6
// TB/s, where a plain copy of those bytes runs at 5.4 (296 us with a workgroup
// per four records).
//
// Rows are read through element strides (sb, sh, sn) shared by q, k and v,
// so a packed QKV buffer (e.g. [B][N][3][H][D]) is encoded where it lies, as
// the paper's stride-aware pack kernels do; each row's D values contiguous.
template <bool kRope, bool kNorm>
__global__ __launch_bounds__(kEncThreads) void qkv_encode_kernel(
    const uint4* __restrict__ q, const uint4* __restrict__ k, const uint4* __restrict__ v,
    uint8_t* __restrict__ rec, int64_t n_tokens, int H, int per_wg, SeqGrid g,
    const float2* __restrict__ tab, const float* __restrict__ q_gamma,
    const float* __restrict__ k_gamma, float eps, int64_t sb, int64_t sh, int64_t sn) {
  const int t = threadIdx.x;
  const int cc = t & 15, part = t & 3;
  const int64_t bn = (int64_t)blockIdx.x * kEncTokens + (t >> 4);
  if (bn >= n_tokens) return;  // the 16 lanes of a token leave together
  const int64_t b = bn / g.n;
  const int n = (int)(bn - b * g.n);
  Pos pos{0, 0, 0, false};
  RopeCS cs{};
  float gq[8], gk[8];
  if (kRope) {
    pos = token_pos(n, g);
    cs = load_rope_cs(tab, tab_lo_plane(tab, g), tab_pair(cc, pos, g));
  }
  if (kNorm) {  // one of the two may be missing: weights 1 and 1 / rms 1 leave a row as it is
#pragma unroll
    for (int e = 0; e < 8; ++e) gq[e] = gk[e] = 1.0f;
    if (q_gamma) load_gamma(q_gamma, cc, gq);
    if (k_gamma) load_gamma(k_gamma, cc, gk);
  }
  const int64_t row = (b * sb + n * sn) / 8 + cc;  // strides are multiples of 8 elements
  const int64_t step_h = sh / 8;
  for (int h0 = (int)blockIdx.y * per_wg; h0 < H; h0 += (int)gridDim.y * per_wg) {
    const int h1 = min(h0 + per_wg, H);
    struct In {
      uint4 q, k, v;
    };
    auto load = [&](int h) __attribute__((always_inline)) {
      const int64_t at = row + h * step_h;
      return In{q[at], k[at], v[at]};
    };
    auto step = [&](int h, const In& in) __attribute__((always_inline)) {
      float inv_q = 1.0f, inv_k = 1.0f;
      if (kNorm) {
        const float sq = row_sumsq_lanes16(chunk_sumsq(in.q)), sk = row_sumsq_lanes16(chunk_sumsq(in.k));
        const float inv = rms_inv((t & 1) ? sk : sq, eps);
        inv_q = q_gamma ? dpp<kDppEven>(inv) : 1.0f;
        inv_k = k_gamma ? dpp<kDppOdd>(inv) : 1.0f;
      }
      float fq[8], fk[8], fv[8];
      unpack_bf16x8(qk_chunk<kRope, kNorm>(in.q, gq, inv_q, pos.rot, cs), fq);
      unpack_bf16x8(qk_chunk<kRope, kNorm>(in.k, gk, inv_k, pos.rot, cs), fk);
      unpack_bf16x8(in.v, fv);
      const float aq = group_amax(fq), ak = group_amax(fk), av = group_amax(fv);
      const uint32_t sc = ue5m3_scale_for_bf16(part == 0 ? aq : part == 1 ? ak : av);
      const ScaleInv inv = scale_inv(ue5m3_value(sc));
      uint8_t* r = rec + (bn * H + h) * kRecBytes;
      *reinterpret_cast<uint2*>(r + 8 * cc) = encode_chunk(fq, from_lane<kDppQuad0>(inv));
      *reinterpret_cast<uint2*>(r + 128 + 8 * cc) = encode_chunk(fk, from_lane<kDppQuad1>(inv));
      *reinterpret_cast<uint2*>(r + 256 + 8 * cc) = encode_chunk(fv, from_lane<kDppQuad2>(inv));
      // the record's last 16 bytes: twelve scale codes and four zero bytes
      r[kRecScales + 4 * part + (cc >> 2)] = part < 3 ? (uint8_t)sc : (uint8_t)0;
    };
    // two a trip: no load in flight moves between registers (past the last
    // head it reads that one again)
    In in0 = load(h0);
    for (int h = h0; h < h1; h += 2) {
      const In in1 = load(min(h + 1, h1 - 1));
      step(h, in0);
      in0 = load(min(h + 2, h1 - 1));
      if (h + 1 < h1) step(h + 1, in1);
    }
  }
}

// One thread per 16-byte chunk written, four records a workgroup.  Runs at a
// copy's rate as it is: 14,400 tokens of 40 heads in 124 us, 5.4 TB/s (the
// encoder's walk over a token's heads took 134 us: little to share here, and
// fewer independent loads in flight).
__global__ __launch_bounds__(kRecThreads) void qkv_decode_kernel(
    const uint8_t* __restrict__ rec, uint4* __restrict__ q, uint4* __restrict__ k,
    uint4* __restrict__ v, int64_t n_rec, int H, int N) {
  const int t = threadIdx.x;
  const int j = t / 48, p = (t / 16) % 3, cc = t & 15;
  const int64_t ri = (int64_t)blockIdx.x * kRecPerWg + j;
  if (ri >= n_rec) return;
  const int64_t bn = ri / H;
  const int h = (int)(ri - bn * H);
  const int64_t b = bn / N;
  const int n = (int)(bn - b * N);
  const size_t row = ((size_t)b * H + h) * N + n;
  uint4* dst = p == 0 ? q : (p == 1 ? k : v);
  dst[row * kChunks + cc] = rec_chunk(rec + ri * kRecBytes, p, cc);
}

}  // namespace

hipError_t launch_qkv_encode(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint8_t* rec,
                             int B, int H, const SeqGrid& g, const float2* tab,
                             const float* q_gamma, const float* k_gamma, float eps,
                             int64_t sb, int64_t sh, int64_t sn, hipStream_t stream) {
  const int64_t n_tokens = (int64_t)B * g.n;
  const int64_t gx = (n_tokens + kEncTokens - 1) / kEncTokens;
  const int per_wg = slabs_per_workgroup(gx, H, kStreamWgs);
  const int64_t groups = ((int64_t)H + per_wg - 1) / per_wg;
  const dim3 grid((unsigned)gx, (unsigned)(groups < 65535 ? groups : 65535));
  const bool norm = q_gamma != nullptr || k_gamma != nullptr;
  auto* kernel = tab ? (norm ? qkv_encode_kernel<true, true> : qkv_encode_kernel<true, false>)
                     : (norm ? qkv_encode_kernel<false, true> : qkv_encode_kernel<false, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(kEncThreads), 0, stream, reinterpret_cast<const uint4*>(q),
                     reinterpret_cast<const uint4*>(k), reinterpret_cast<const uint4*>(v), rec, n_tokens, H,
                     per_wg, g, tab, q_gamma, k_gamma, eps, sb, sh, sn);
  return hipGetLastError();
}

hipError_t launch_qkv_decode(const uint8_t* rec, uint16_t* q, uint16_t* k, uint16_t* v, int B, int H,
                             int N, hipStream_t stream) {
  const int64_t n_rec = (int64_t)B * N * H;
  const dim3 grid((unsigned)((n_rec + kRecPerWg - 1) / kRecPerWg));
  hipLaunchKernelGGL(qkv_decode_kernel, grid, dim3(kRecThreads), 0, stream, rec,
                     reinterpret_cast<uint4*>(q), reinterpret_cast<uint4*>(k),
                     reinterpret_cast<uint4*>(v), n_rec, H, N);
  return hipGetLastError();
}

}  // namespace sol
