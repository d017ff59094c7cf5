// Split-KV log-sum-exp merge of the partial results of the decode kernel.
//
// Each KV piece p of a sequence delivered a normalized partial output o_p and its
// log-sum-exp LSE_p (Algorithm 1 returns both per query row).  Per row:
//   LSE = log sum_p exp(LSE_p),   o = sum_p exp(LSE_p - LSE) * o_p.
// When the decode was given the output (ctrl[0] == 1) it has written the rows of
// every sequence that at most one piece covers; those are left as they are.
//
// Two kernels, one per slot layout (part_tile_offset), each in a few shapes that spread
// a row over more waves when there are few rows (launch_combine):
// - one row group (plain rows): G waves per row; lane l owns output dimensions
//   8l..8l+7.  The pieces' log-sum-exps are read lane-parallel, and a piece whose
//   weight underflows to zero is not read at all (the row's partial sits in its own
//   cache lines).
// - several row groups (tile order): one wave per 32-row x 32-dimension tile or per
//   chunk pair of it, lane n + 32h on row n of the tile, dimensions 8q + 4h .. +3; every
//   partial load of a wave reads 1 KiB of consecutive bytes.  Each lane merges its row
//   with a running maximum, J pieces per round so that their loads overlap.

#include "piece_end.h"
#include "snapmla_device.h"
#include "snapmla_internal.h"

namespace snapmla {

// The pieces of sequence b: candidates first..last; exists(i) rejects an empty part
// (only possible with fewer virtual positions than parts), pid(i) is the piece's slot.
// Balanced plan: part w covers the real blocks of virtual positions [w*TV/W,
// (w+1)*TV/W) (kPlanPad) and writes piece id w + b for every sequence b it touches;
// fixed chunks: piece id b*W + chunk.  (The parts that meet sequence b's real blocks
// are exactly those whose virtual range meets [prefix[b] + pad*(b+1), prefix[b+1] +
// pad*(b+1)); each of them has a non-empty range, so last - first + 1 counts its pieces.)
struct Pieces {
  int first = 0, last = -1, b = 0, W = 1;
  bool balanced = true;
  int64_t TV = 0;
  __device__ bool exists(int i) const {
    return !balanced || TV >= W || (int64_t)i * TV / W < (int64_t)(i + 1) * TV / W;
  }
  __device__ int64_t pid(int i) const { return balanced ? (int64_t)i + b : (int64_t)b * W + i; }
};

__device__ Pieces pieces_of(const CombineArgs& a, int b) {
  Pieces P;
  P.b = b;
  P.W = a.num_splits;
  P.balanced = a.chunk_blocks == 0;
  P.TV = a.prefix[a.B] + (int64_t)a.pad * a.B;
  const int p0 = a.prefix[b], p1 = a.prefix[b + 1];
  const int nb = p1 - p0;
  if (nb > 0) {
    if (P.balanced) {
      const int64_t v0 = p0 + (int64_t)a.pad * (b + 1);    // virtual position of the first block
      P.first = (int)(((v0 + 1) * P.W - 1) / P.TV);
      P.last = (int)(((v0 + nb) * P.W - 1) / P.TV);
    } else {
      P.first = 0;
      P.last = (nb + a.chunk_blocks - 1) / a.chunk_blocks - 1;
    }
  }
  return P;
}

// The bf16 or float32 results of 8 consecutive output dimensions (elements 8i .. 8i+7 of a row).
__device__ __forceinline__ void store_row8(const CombineArgs& a, int64_t orow, int i, const float (&o)[8]) {
  if (a.out_dtype == 1) {
    v4f* dst = reinterpret_cast<v4f*>(reinterpret_cast<float*>(a.out) + orow * kDc + 8 * i);
    dst[0] = v4f{o[0], o[1], o[2], o[3]};
    dst[1] = v4f{o[4], o[5], o[6], o[7]};
  } else {
    uint4 pk;
    pk.x = f32_to_bf16_bits(o[0]) | (f32_to_bf16_bits(o[1]) << 16);
    pk.y = f32_to_bf16_bits(o[2]) | (f32_to_bf16_bits(o[3]) << 16);
    pk.z = f32_to_bf16_bits(o[4]) | (f32_to_bf16_bits(o[5]) << 16);
    pk.w = f32_to_bf16_bits(o[6]) | (f32_to_bf16_bits(o[7]) << 16);
    reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(a.out) + orow * kDc)[i] = pk;
  }
}

// G waves per row (G <= 4: a workgroup holds 4 / G rows; above: one row): wave g of a
// row takes the pieces g, g + G, ... and the waves' weighted sums meet in LDS.
template <int G>
__global__ __launch_bounds__(G <= 4 ? 256 : 64 * G) void combine_rows_kernel(CombineArgs a) {
  constexpr int kRows = G <= 4 ? 4 / G : 1;           // rows of a workgroup
  constexpr int kFly = 4;                             // partial rows in flight per wave
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int g = w % G, wr = w / G;
  const int64_t wv = (int64_t)blockIdx.x * kRows + wr;
  const bool live = wv < (int64_t)a.B * a.R;          // (kRows == 1: always)
  if (G == 1 && !live) return;
  const int b = live ? (int)(wv / a.R) : 0, r = live ? (int)(wv % a.R) : 0;

  const Pieces P = pieces_of(a, b);
  const int first = P.first, last = P.last;
  const bool work = live && !(a.ctrl[0] == 1 && last <= first);
  if (G == 1 && !work) return;
  auto exists = [&](int i) { return P.exists(i); };
  auto pid = [&](int i) { return P.pid(i); };

  // pass 1: lane i reads the log-sum-exp of candidate piece first + i (64 at a
  // time), the wave reduces the maximum and NaN flag; the first 64 stay in x0 for
  // pass 2 (every wave of a row reads them all)
  float M = -INFINITY;
  bool anynan = false;
  float x0 = -INFINITY;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  float S = 0.0f;
  if (work) {
    for (int i0 = first; i0 <= last; i0 += 64) {
      const int i = i0 + lane;
      float x = -INFINITY;
      if (i <= last && exists(i)) x = a.part_lse[pid(i) * a.rows_pad + r];
      if (i0 == first) x0 = x;
      anynan |= x != x;
      M = fmaxf(M, x);
    }
    M = wave_max(M);
    anynan = __builtin_amdgcn_ballot_w64(anynan) != 0;
    // pass 2: weights exp(LSE_i - M) (lane-parallel), then this wave's weighted rows,
    // kFly pieces per round so that their loads overlap
    if (M > -INFINITY && !anynan) {
      for (int i0 = first; i0 <= last; i0 += 64) {
        const int i = i0 + lane;
        float wi = 0.0f;
        if (i <= last && exists(i)) {
          const float x = i0 == first ? x0 : a.part_lse[pid(i) * a.rows_pad + r];
          wi = x > -INFINITY ? expf(x - M) : 0.0f;
        }
        S += wi;
        const int cnt = min(64, last - i0 + 1);
        for (int j = g; j < cnt; j += kFly * G) {
          v4f u[kFly][2];
          float wj[kFly];
#pragma unroll
          for (int t = 0; t < kFly; ++t) {
            const int jt = j + t * G;
            wj[t] = jt < cnt ? __shfl(wi, jt & 63, 64) : 0.0f;   // zero for missing / empty pieces
            const bool use = wj[t] != 0.0f;
            const int ij = min(i0 + jt, last);       // in range even when unused
            const v4f* src = reinterpret_cast<const v4f*>(a.part_o + (pid(ij) * a.rows_pad + r) * kDc + 8 * lane);
            u[t][0] = use ? src[0] : v4f{0.f, 0.f, 0.f, 0.f};
            u[t][1] = use ? src[1] : v4f{0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
          for (int t = 0; t < kFly; ++t) {
            acc[0] += wj[t] * u[t][0][0]; acc[1] += wj[t] * u[t][0][1];
            acc[2] += wj[t] * u[t][0][2]; acc[3] += wj[t] * u[t][0][3];
            acc[4] += wj[t] * u[t][1][0]; acc[5] += wj[t] * u[t][1][1];
            acc[6] += wj[t] * u[t][1][2]; acc[7] += wj[t] * u[t][1][3];
          }
        }
      }
      // wave sum of the weights
      for (int o = 32; o > 0; o >>= 1) S += __shfl_xor(S, o, 64);
    }
  }
  if constexpr (G > 1) {
    __shared__ v4f sums[kRows][G][kDc / 4];
    sums[wr][g][2 * lane] = v4f{acc[0], acc[1], acc[2], acc[3]};
    sums[wr][g][2 * lane + 1] = v4f{acc[4], acc[5], acc[6], acc[7]};
    __syncthreads();
    if (!work || g != 0) return;
    for (int o = 1; o < G; ++o) {
      const v4f p = sums[wr][o][2 * lane], q = sums[wr][o][2 * lane + 1];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[j] += p[j];
        acc[4 + j] += q[j];
      }
    }
  }
  const bool bad = a.flags[b] != 0 || anynan;
  float o[8];
  float lse;
  if (bad) {
    const float nanv = __builtin_nanf("");
    for (int j = 0; j < 8; ++j) o[j] = nanv;
    lse = nanv;
  } else if (!(M > -INFINITY)) {
    for (int j = 0; j < 8; ++j) o[j] = 0.0f;
    lse = -INFINITY;
  } else {
    const float inv = 1.0f / S;
    for (int j = 0; j < 8; ++j) o[j] = acc[j] * inv;
    lse = M + logf(S);
  }
  const int64_t orow = (int64_t)b * a.R + r;
  store_row8(a, orow, lane, o);
  if (a.lse != nullptr && lane == 0) a.lse[orow] = lse;
}

// A wave merges Q of the four chunk pairs (8 dimensions each) of a 32 x 32 tile, J
// pieces per round; with G > 1 the four waves of a workgroup share one such part and
// wave g takes the pieces g, g + G, ...
template <int Q, int G, int J>
__global__ __launch_bounds__(256) void combine_tiles_kernel(CombineArgs a) {
  static_assert(G == 1 || G == 4, "waves of a part");
  constexpr int kParts = 16 / Q;                     // parts of a (sequence, row tile, dimension quarter)
  constexpr int kPerWg = 4 / G;                      // parts of a workgroup
  const int lane = threadIdx.x & 63;
  const int n = lane & 31, h = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = w % G;
  const int tiles = (a.R + 31) / 32;                 // 32-row tiles per sequence
  const int part = (int)(blockIdx.x % (kParts / kPerWg)) * kPerWg + w / G;
  const int64_t rest = blockIdx.x / (kParts / kPerWg);
  const int T = part / (4 / Q), q0 = (part % (4 / Q)) * Q;
  const int dq = (int)(rest & 3);
  const int64_t bt = rest >> 2;
  const int b = (int)(bt / tiles), t = (int)(bt % tiles);
  const int row = 32 * t + n;                        // query row of this lane (< rows_pad)

  const Pieces P = pieces_of(a, b);
  const int first = P.first, last = P.last;
  if (a.ctrl[0] == 1 && last <= first) return;
  auto exists = [&](int i) { return P.exists(i); };
  auto pid = [&](int i) { return P.pid(i); };
  const int64_t tile = part_tile_offset(t >> 1, dq, t & 1, T, q0, lane);

  // this wave's pieces, merged with a running maximum M: S = sum exp(LSE_i - M),
  // acc = sum exp(LSE_i - M) o_i.  Every row of an existing piece's slot was written
  // (0 for a row without tokens, NaN for a rejected piece).
  float M = -INFINITY, S = 0.0f;
  bool anynan = false;
  v4f acc[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) acc[q] = v4f{0.f, 0.f, 0.f, 0.f};
  for (int i0 = first + g; i0 <= last; i0 += J * G) {
    float x[J];
    v4f u[J][Q];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int i = i0 + j * G;
      const bool live = i <= last && exists(i);
      const int64_t p = pid(live ? i : first);       // in range even when unused
      x[j] = live ? a.part_lse[p * a.rows_pad + row] : -INFINITY;
      const v4f* src = reinterpret_cast<const v4f*>(a.part_o + p * a.rows_pad * kDc + tile);
#pragma unroll
      for (int q = 0; q < Q; ++q) u[j][q] = live ? src[64 * q] : v4f{0.f, 0.f, 0.f, 0.f};
    }
    float mr = M;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      anynan |= x[j] != x[j];
      mr = fmaxf(mr, x[j]);
    }
    if (mr > -INFINITY) {
      const float sc = expf(M - mr);                 // 0 while M is -inf
      S *= sc;
#pragma unroll
      for (int q = 0; q < Q; ++q) acc[q] *= sc;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const float wj = x[j] > -INFINITY ? expf(x[j] - mr) : 0.0f;
        S += wj;
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[q] += wj * u[j][q];
      }
      M = mr;
    }
  }
  if constexpr (G > 1) {
    // the waves' sums meet in LDS, relative to the largest of their maxima
    __shared__ v4f sacc[G][Q][64];
    __shared__ float sm[G][64], ss[G][64];
#pragma unroll
    for (int q = 0; q < Q; ++q) sacc[g][q][lane] = acc[q];
    sm[g][lane] = anynan ? __builtin_nanf("") : M;
    ss[g][lane] = S;
    __syncthreads();
    if (g != 0) return;
    float top = M;
#pragma unroll
    for (int o = 1; o < G; ++o) {
      const float x = sm[o][lane];
      anynan |= x != x;
      top = fmaxf(top, x);
    }
    if (top > -INFINITY) {
      const float sc = expf(M - top);                // 0 where this wave had no piece
      S *= sc;
#pragma unroll
      for (int q = 0; q < Q; ++q) acc[q] *= sc;
#pragma unroll
      for (int o = 1; o < G; ++o) {
        const float x = sm[o][lane];
        const float wo = x > -INFINITY ? expf(x - top) : 0.0f;
        S += wo * ss[o][lane];
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[q] += wo * sacc[o][q][lane];
      }
    }
    M = top;
  }
  if (row >= a.R) return;
  const bool bad = a.flags[b] != 0 || anynan;
  v4f o[Q];
  float lse;
  if (bad) {
    const float nanv = __builtin_nanf("");
    for (int q = 0; q < Q; ++q) o[q] = v4f{nanv, nanv, nanv, nanv};
    lse = nanv;
  } else if (!(M > -INFINITY)) {
    for (int q = 0; q < Q; ++q) o[q] = v4f{0.f, 0.f, 0.f, 0.f};
    lse = -INFINITY;
  } else {
    const float inv = 1.0f / S;
    for (int q = 0; q < Q; ++q) o[q] = acc[q] * inv;
    lse = M + logf(S);
  }
  const int64_t orow = (int64_t)b * a.R + row;
  const int64_t col = 128 * dq + 32 * T + 8 * q0 + 4 * h;
  for (int q = 0; q < Q; ++q) {
    if (a.out_dtype == 1) {
      *reinterpret_cast<v4f*>(reinterpret_cast<float*>(a.out) + orow * kDc + col + 8 * q) = o[q];
    } else {
      const uint32_t lo = f32_to_bf16_bits(o[q][0]) | (f32_to_bf16_bits(o[q][1]) << 16);
      const uint32_t hi = f32_to_bf16_bits(o[q][2]) | (f32_to_bf16_bits(o[q][3]) << 16);
      *reinterpret_cast<v2i*>(reinterpret_cast<uint16_t*>(a.out) + orow * kDc + col + 8 * q) = v2i{(int)lo, (int)hi};
    }
  }
  if (a.lse != nullptr && dq == 0 && T == 0 && q0 == 0 && h == 0) a.lse[orow] = lse;
}

template <int G>
static hipError_t launch_rows(const CombineArgs& a, hipStream_t stream) {
  constexpr int kRows = G <= 4 ? 4 / G : 1;
  const int64_t blocks = ((int64_t)a.B * a.R + kRows - 1) / kRows;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(combine_rows_kernel<G>, dim3((unsigned)blocks), dim3(G <= 4 ? 256 : 64 * G), 0, stream, a);
  return hipGetLastError();
}

template <int Q, int G, int J>
static hipError_t launch_tiles(const CombineArgs& a, hipStream_t stream) {
  const int64_t blocks = (int64_t)a.B * ((a.R + 31) / 32) * 4 * (4 * G / Q);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL((combine_tiles_kernel<Q, G, J>), dim3((unsigned)blocks), dim3(256), 0, stream, a);
  return hipGetLastError();
}

// How a row is spread over waves.  A merge of few rows is bound by the chain of loads of
// one wave (a memory round trip per round of pieces) and leaves the chip idle; a merge of
// many rows is bound by the partials' bytes, and there the LDS exchange and the smaller
// parts only cost.  Measured, us per call back to back (about 8 of them the host's launch):
//   plain rows  192 rows x 86 pieces: G = 1 19.3, 4 9.8, 8 8.5;  64 x 257: 39.0, 17.2, 12.7 (16: 15.0);
//               1024 x 17: G = 1 10.0, 4 8.2, 8 9.1;  2048 x 9: G = 1 9.2, 2 9.8, 4 11.1;  4096 x 5: 10.8, 13.8, 15.3
//   tile order  512 rows x 33 pieces: <4,1,4> 21.7, <1,1,8> 13.5, <1,4,8> 8.5;  256 x 65: 34.4, 20.9, 8.7;
//               32768 x 1.5: <4,1,4> 25.5, <2,1,8> 33.4, <1,4,8> 109.8
//   (in a graph, without the launch) 1024 x 6: <4,1,4> 6.1, <2,1,4> 5.3, <1,4,8> 9.5;  1536 x 9: 8.5, 7.4, 11.5;
//               768 x 17: 11.9, 9.2, 7.8
hipError_t launch_combine(const CombineArgs& a, hipStream_t stream) {
  const int64_t rows = (int64_t)a.B * a.R;
  if (rows <= 0) return hipSuccess;
  // pieces of an average sequence (fixed chunks: of the longest)
  const int mean = a.chunk_blocks == 0 ? a.num_splits / a.B + 1 : a.num_splits;
  if (a.rows_pad > 64) {
    if (rows <= 1024 && mean >= 16) return launch_tiles<1, 4, 8>(a, stream);
    if (rows <= 4096) return launch_tiles<2, 1, 4>(a, stream);
    return launch_tiles<4, 1, 4>(a, stream);
  }
  if (rows > 1024 || mean < 8) return launch_rows<1>(a, stream);
  if (mean < 16) return launch_rows<2>(a, stream);
  if (mean < 32 || rows > 256) return launch_rows<4>(a, stream);
  return launch_rows<8>(a, stream);
}

}  // namespace snapmla
