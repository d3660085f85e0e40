// Block routing of the block-sparse attention (Sec. 3.4, "Per-step dynamic
// sparsity" and "Safety rails and the exact prefix KV sink"), for gfx950.
//
// For the self-attention of each (b, h) slab of N tokens, with query blocks of
// 256 rows (the attention kernel's workgroup tile) and key blocks of 128 keys
// (four prepared tiles), both counted from token 0:
//   qbar_I = mean of q^ over block I's rows   (q^ as the attention kernel's
//            query load makes it: normalised, rotated, rounded to bf16),
//   kbar_J = mean of k^ over block J's keys   (read from the prepared tiles),
//   s_IJ   = <qbar_I, kbar_J> / sqrt(D),
//   mu_I, sigma_I = mean and population standard deviation over all J,
//   J is kept for I iff s_IJ > mu_I + tau sigma_I, or J holds a prefix key
//   (the exact prefix sink), or J is I's first best block (no block attends
//   to nothing); a query block holding a prefix row keeps every J.
// The kept blocks of I are written in ascending order, with their count, for
// the block-sparse attention kernel to walk.
//
// Three launches, all small next to the attention: pool_q_kernel (reads q
// once), pool_k_kernel (reads the prepared K once), route_kernel (four query
// blocks per workgroup: the scores go to LDS, then one wave per query block
// finds mean and spread in fixed-order trees and compacts the kept blocks with
// ballots).
#include <type_traits>

#include "sol_device.h"

namespace sol {
namespace {

constexpr int kQB = kSparseQueryBlock;
constexpr int kKB = kSparseKeyBlock;
constexpr int kMaxKeyBlocks = kMaxSparseBlocks;

// Mean of q^ over each query block.  Grid (nqb, groups of kSlabs slabs); 256
// threads = 16 rows x 16 chunks per step, 16 steps over the block's rows: each
// thread sums its chunk's 8 entries over its 16 rows in row order, then the 16
// row groups are summed in LDS in group order.  Its floor is reading q; the
// rotation's instructions are what it is bound by, so a workgroup takes kSlabs
// slabs through each step with one row's position, cosines and sines: 272 us
// for 111,600 tokens of 40 heads (383 us with one slab, 441 us with the
// rotation's rounding to odd besides).
template <bool kRope, bool kNorm, int kSlabs>
__global__ __launch_bounds__(256) void pool_q_kernel(const uint4* __restrict__ q,
                                                     float* __restrict__ qbar, int64_t bh_count,
                                                     SeqGrid g, const float2* __restrict__ tab,
                                                     const float* __restrict__ gamma, float eps,
                                                     int nqb) {
  __shared__ float part[16][D + 4];
  lds_poison(&part[0][0], sizeof(part));
  lds_poison_done();
  const int N = g.n;
  const int I = blockIdx.x;
  const int t = threadIdx.x, cc = t & 15, rg = t >> 4;
  const int r0 = I * kQB;
  const int rows = min(kQB, N - r0);
  float gm[8] = {};
  if (kNorm) load_gamma(gamma, cc, gm);
  for (int64_t bh0 = (int64_t)blockIdx.y * kSlabs; bh0 < bh_count; bh0 += (int64_t)gridDim.y * kSlabs) {
    float acc[kSlabs][8];
#pragma unroll
    for (int s = 0; s < kSlabs; ++s)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[s][e] = 0.0f;
    // slabs past the last read that one again; rows past the block add nothing
    auto load = [&](int step, uint4 (&x)[kSlabs]) __attribute__((always_inline)) {
      const int n = min(r0 + 16 * step + rg, N - 1);
#pragma unroll
      for (int s = 0; s < kSlabs; ++s) x[s] = q[((size_t)min(bh0 + s, bh_count - 1) * N + n) * kChunks + cc];
    };
    uint4 next[kSlabs];
    load(0, next);
    for (int step = 0; step < kQB / 16; ++step) {
      const int n = r0 + 16 * step + rg;
      const bool valid = n < N;  // the 16 lanes of a row agree
      uint4 x[kSlabs];
#pragma unroll
      for (int s = 0; s < kSlabs; ++s) x[s] = next[s];
      load(min(step + 1, kQB / 16 - 1), next);
      Pos p{0, 0, 0, false};
      RopeCS cs{};
      if (kRope) {
        p = token_pos(min(n, N - 1), g);
        cs = load_rope_cs(tab, tab_lo_plane(tab, g), tab_pair(cc, p, g));
      }
#pragma unroll
      for (int s = 0; s < kSlabs; ++s) {
        const float inv = kNorm ? rms_inv(row_sumsq_lanes16(chunk_sumsq(x[s])), eps) : 1.0f;
        float f[8];
        unpack_bf16x8(qk_chunk<kRope, kNorm>(x[s], gm, inv, p.rot, cs), f);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[s][e] += valid ? f[e] : 0.0f;
      }
    }
#pragma unroll
    for (int s = 0; s < kSlabs; ++s) {
      if (bh0 + s >= bh_count) break;  // uniform
#pragma unroll
      for (int e = 0; e < 8; ++e) part[rg][8 * cc + e] = acc[s][e];
      __syncthreads();
      if (t < D) {
        float sum = 0.0f;
        for (int r = 0; r < 16; ++r) sum += part[r][t];
        qbar[((size_t)(bh0 + s) * nqb + I) * D + t] = sum / (float)rows;
      }
      __syncthreads();
    }
  }
}

// Mean of k^ over each key block, from the prepared K tiles (fp16 k^, exact;
// keys past N are zero there and add nothing).  Grid (nkb, slabs); thread t
// reads the 16-byte fragment slots t and t + 256 of each of the block's four
// tiles -- always key r = t & 31 of a tile, chunks 2(t >> 6) + hh and that +
// 8, hh = (t >> 5) & 1 -- and the 32 keys of a wave half are summed by a
// butterfly over lane bits 0..4.  kbar is laid out [D / 4][nkb][4], so that
// route_kernel's lanes, one key block each, read side by side.
__global__ __launch_bounds__(256) void pool_k_kernel(const uint4* __restrict__ kp,
                                                     float* __restrict__ kbar, int64_t bh_count,
                                                     int N, int nkb) {
  const int J = blockIdx.x;
  const int t = threadIdx.x;
  const int n_tiles = (N + kPrepTile - 1) / kPrepTile;
  const int keys = min(kKB, N - J * kKB);
  const int kk = t >> 6, hh = (t >> 5) & 1;
  for (int64_t bh = blockIdx.y; bh < bh_count; bh += gridDim.y) {
    float acc[2][8];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[u][e] = 0.0f;
    for (int tt = 0; tt < 4; ++tt) {
      const int tile = 4 * J + tt;
      if (tile >= n_tiles) break;  // uniform
      const uint4* src = kp + ((size_t)bh * n_tiles + tile) * (kPrepTileElems / 8);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint4 w = src[t + 256 * u];
        const uint32_t h[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f16x2 pr = __builtin_bit_cast(f16x2, h[e]);
          acc[u][2 * e] += (float)pr[0];
          acc[u][2 * e + 1] += (float)pr[1];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float x = acc[u][e];
        x += __shfl_xor(x, 1);
        x += __shfl_xor(x, 2);
        x += __shfl_xor(x, 4);
        x += __shfl_xor(x, 8);
        x += __shfl_xor(x, 16);
        acc[u][e] = x;
      }
    if ((t & 31) == 0) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int dim0 = 16 * (kk + 4 * u) + 8 * hh;
        float4* dst = reinterpret_cast<float4*>(kbar + (size_t)bh * nkb * D) + (size_t)(dim0 / 4) * nkb + J;
        const float n = (float)keys;
        dst[0] = make_float4(acc[u][0] / n, acc[u][1] / n, acc[u][2] / n, acc[u][3] / n);
        dst[nkb] = make_float4(acc[u][4] / n, acc[u][5] / n, acc[u][6] / n, acc[u][7] / n);
      }
    }
  }
}

// Routing of kRouteQB consecutive query blocks per workgroup.  Grid
// (ceil(nqb / kRouteQB), slabs).  All 256 threads score: a thread holds four
// key blocks (256 apart) against the four query blocks at once, so one pooled
// key read from L2 serves four products and one pooled query read from LDS
// another four.  Scores go to LDS; then wave u routes query block I0 + u by
// itself, without a barrier: mean and spread are sums over the 256 residues of
// J mod 256 in ascending J, then a binary tree pairing residue r with r + 128,
// r + 64, .. r + 1; the best block is a (score, lowest index) reduction; and
// the kept blocks are compacted in ascending order with ballots.  kCap: key
// blocks the score rows hold in LDS.  The usual case (up to 131,072 tokens)
// takes 18 KB, so that five workgroups share a CU (their registers' limit; LDS
// holds eight) and hide each other's latency; the rows for the longest sequence
// leave room for one.
// 111,600 tokens of 40 heads: 130 us, against 579 us with one reduction after
// another over the whole workgroup and rows for the longest sequence.
constexpr int kRouteQB = 4;
constexpr int kRouteCap = 1024;

// Sum over the wave (the tree's last six levels), in every lane.
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) x += __shfl_xor(x, s);
  return x;
}

template <int kCap>
__global__ __launch_bounds__(256) void route_kernel(const float* __restrict__ qbar,
                                                    const float* __restrict__ kbar,
                                                    uint16_t* __restrict__ blocks,
                                                    int* __restrict__ counts, int64_t bh_count,
                                                    int nqb, int nkb, int n_prefix, float tau,
                                                    float scale) {
  __shared__ __attribute__((aligned(16))) float qs[kRouteQB][D];
  __shared__ float sc[kRouteQB][kCap];
  lds_poison(&qs[0][0], sizeof(qs));
  lds_poison(&sc[0][0], sizeof(sc));
  lds_poison_done();
  const int I0 = blockIdx.x * kRouteQB;
  const int nq = min(kRouteQB, nqb - I0);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  for (int64_t bh = blockIdx.y; bh < bh_count; bh += gridDim.y) {
    for (int e = t; e < kRouteQB * D; e += 256) {
      const int u = e / D, d = e % D;
      qs[u][d] = u < nq ? qbar[((size_t)bh * nqb + I0 + u) * D + d] : 0.0f;
    }
    __syncthreads();
    const float4* kr = reinterpret_cast<const float4*>(kbar + (size_t)bh * nkb * D);
    for (int J0 = t; J0 < nkb; J0 += 1024) {
      float dot[kRouteQB][4];
#pragma unroll
      for (int u = 0; u < kRouteQB; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c) dot[u][c] = 0.0f;
#pragma unroll 2
      for (int d4 = 0; d4 < D / 4; ++d4) {
        float4 kv[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) kv[c] = kr[(size_t)d4 * nkb + min(J0 + 256 * c, nkb - 1)];
#pragma unroll
        for (int u = 0; u < kRouteQB; ++u) {
          const float4 qv = *reinterpret_cast<const float4*>(&qs[u][4 * d4]);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            dot[u][c] = __builtin_fmaf(qv.x, kv[c].x, dot[u][c]);
            dot[u][c] = __builtin_fmaf(qv.y, kv[c].y, dot[u][c]);
            dot[u][c] = __builtin_fmaf(qv.z, kv[c].z, dot[u][c]);
            dot[u][c] = __builtin_fmaf(qv.w, kv[c].w, dot[u][c]);
          }
        }
      }
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (J0 + 256 * c < nkb)
#pragma unroll
          for (int u = 0; u < kRouteQB; ++u) sc[u][J0 + 256 * c] = dot[u][c] * scale;
    }
    __syncthreads();
    if (wave < nq) {  // one wave per query block
      const float* s = sc[wave];
      const int I = I0 + wave;
      const size_t qi = (size_t)bh * nqb + I;
      const bool dense = I * kQB < n_prefix;  // the block holds a prefix row
      // four residues a lane: J = lane + 64 r + 256 i
      float psum[4], best_v = -__builtin_inff();
      int best_j = nkb;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        psum[r] = 0.0f;
        for (int J = lane + 64 * r; J < nkb; J += 256) {
          const float sv = s[J];
          psum[r] += sv;
          if (sv > best_v || (sv == best_v && J < best_j)) {
            best_v = sv;
            best_j = J;
          }
        }
      }
      const float mu = wave_sum((psum[0] + psum[2]) + (psum[1] + psum[3])) / (float)nkb;
      float pvar[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pvar[r] = 0.0f;
        for (int J = lane + 64 * r; J < nkb; J += 256) {
          const float d = s[J] - mu;
          pvar[r] = __builtin_fmaf(d, d, pvar[r]);
        }
      }
      const float var = wave_sum((pvar[0] + pvar[2]) + (pvar[1] + pvar[3])) / (float)nkb;
      const float thr = mu + tau * __builtin_sqrtf(var);
      // first best block: largest score, lowest index among equals
#pragma unroll
      for (int m = 32; m > 0; m >>= 1) {
        const float ov = __shfl_xor(best_v, m);
        const int oi = __shfl_xor(best_j, m);
        if (ov > best_v || (ov == best_v && oi < best_j)) {
          best_v = ov;
          best_j = oi;
        }
      }
      // kept blocks, compacted in ascending order
      int base = 0;
      uint16_t* out = blocks + qi * nkb;
      for (int c0 = 0; c0 < nkb; c0 += 64) {
        const int J = c0 + lane;
        const bool keep = J < nkb && (dense || J * kKB < n_prefix || J == best_j || s[J] > thr);
        const uint64_t m = __ballot(keep);
        if (keep) out[base + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)J;
        base += __popcll(m);
      }
      if (lane == 0) counts[qi] = base;
    }
    __syncthreads();  // the next slab overwrites the pooled queries and the scores
  }
}

}  // namespace

hipError_t launch_sparse_route(const uint16_t* q, const uint16_t* k_prep, int BH, const SeqGrid& g,
                               const float2* tab, const float* q_gamma, float eps, float tau,
                               void* workspace, hipStream_t stream) {
  const int N = g.n;
  const int nqb = (N + kQB - 1) / kQB, nkb = (N + kKB - 1) / kKB;
  size_t off[4];
  sparse_workspace_offsets(BH, N, off);
  char* ws = static_cast<char*>(workspace);
  int* counts = reinterpret_cast<int*>(ws + off[0]);
  uint16_t* blocks = reinterpret_cast<uint16_t*>(ws + off[1]);
  float* qbar = reinterpret_cast<float*>(ws + off[2]);
  float* kbar = reinterpret_cast<float*>(ws + off[3]);
  const unsigned gy = (unsigned)(BH < 65535 ? BH : 65535);
  // four slabs per workgroup of the query pooling where that leaves eight
  // workgroups a CU, else one
  const bool grouped = (int64_t)nqb * BH >= 4 * kStreamWgs;
  const int64_t groups = grouped ? ((int64_t)BH + 3) / 4 : BH;
  auto pool_q = [&](auto rope, auto norm) {
    return grouped ? pool_q_kernel<decltype(rope)::value, decltype(norm)::value, 4>
                   : pool_q_kernel<decltype(rope)::value, decltype(norm)::value, 1>;
  };
  using Yes = std::true_type;
  using No = std::false_type;
  auto* pool_q_fn = tab ? (q_gamma ? pool_q(Yes(), Yes()) : pool_q(Yes(), No()))
                        : (q_gamma ? pool_q(No(), Yes()) : pool_q(No(), No()));
  hipLaunchKernelGGL(pool_q_fn, dim3(nqb, (unsigned)(groups < 65535 ? groups : 65535)), dim3(256), 0, stream,
                     reinterpret_cast<const uint4*>(q), qbar, (int64_t)BH, g, tab, q_gamma, eps, nqb);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pool_k_kernel, dim3(nkb, gy), dim3(256), 0, stream,
                     reinterpret_cast<const uint4*>(k_prep), kbar, (int64_t)BH, N, nkb);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto* route_fn = nkb <= kRouteCap ? route_kernel<kRouteCap> : route_kernel<kMaxKeyBlocks>;
  hipLaunchKernelGGL(route_fn, dim3((nqb + kRouteQB - 1) / kRouteQB, gy), dim3(256), 0, stream, qbar, kbar,
                     blocks, counts, (int64_t)BH, nqb, nkb, g.nt, tau, (float)(1.0 / 11.313708498984761));
  return hipGetLastError();
}

}  // namespace sol
