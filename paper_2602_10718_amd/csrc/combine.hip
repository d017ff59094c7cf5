// Split-KV log-sum-exp merge of the partial results of the decode kernel.
//
// Each KV piece p of a sequence delivered a normalized partial output o_p and its
// log-sum-exp LSE_p (Algorithm 1 returns both per query row).  Per row:
//   LSE = log sum_p exp(LSE_p),   o = sum_p exp(LSE_p - LSE) * o_p.
// When the decode was given the output (ctrl[0] == 1) it has written the rows of
// every sequence that at most one piece covers; those are left as they are.
//
// The partials are in accumulator tile order (part_tile_offset): one wave per 32-row x
// 32-dimension tile or per half or quarter of it, lane n + 32h on row n of the tile,
// dimensions 8q + 4h .. +3; every partial load of a wave reads 1 KiB of consecutive
// bytes.  Each lane merges its row with a running maximum, J pieces per round so that
// their loads overlap.

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
  P.balanced = a.chunk_blocks == 0;
  P.W = P.balanced ? a.ctrl[1] : a.num_splits;
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

// A wave merges Q of the four chunk pairs (8 dimensions each) of a 32 x 32 tile, J
// pieces per round; with G > 1 the G waves of a workgroup share one such part and
// wave g takes the pieces g, g + G, ...
template <int Q, int G, int J>
__global__ __launch_bounds__(G <= 4 ? 256 : 64 * G) void combine_kernel(CombineArgs a) {
  static_assert(G == 1 || G >= 4, "waves of a part");
  constexpr int kParts = 16 / Q;                     // parts of a (sequence, row tile, dimension quarter)
  constexpr int kPerWg = G == 1 ? 4 : 1;             // parts of a workgroup
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

template <int Q, int G, int J>
static hipError_t launch_shape(const CombineArgs& a, hipStream_t stream) {
  const int64_t blocks = (int64_t)a.B * ((a.R + 31) / 32) * 4 * (16 / Q) / (G == 1 ? 4 : 1);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL((combine_kernel<Q, G, J>), dim3((unsigned)blocks), dim3(G <= 4 ? 256 : 64 * G), 0, stream, a);
  return hipGetLastError();
}

// How a row is spread over waves.  A merge of few rows is bound by the chain of loads of
// one wave (a memory round trip per round of pieces) and leaves the chip idle; a merge of
// many rows is bound by the partials' bytes, and there the LDS exchange and the smaller
// parts only cost.  Measured, us per call in a graph (rows x mean pieces; shapes <Q, G, J>):
//   64 x 257  <4,1,4> 85  <2,4,4> 20.0  <1,4,8> 15.8   192 x 86  38  10.6  9.4
//   512 x 33  21.7  8.5  8.4     256 x 17  13.0  6.5  6.8     1024 x 17  16.6  8.0  10.2
//   1024 x 9  8.7  6.1  9.1      512 x 9  8.5  6.1  8.9      512 x 32  14.1  6.6  6.8
//   2048 x 9  <4,1,4> 11.7  <2,1,4> 10.0  <2,4,4> 9.6        4096 x 5  11.1  10.9  13.6
//   32768 x 1.5  <4,1,4> 24.6  <2,1,4> 25.2  <2,4,4> 56
hipError_t launch_combine(const CombineArgs& a, hipStream_t stream) {
  const int64_t rows = (int64_t)a.B * a.R;
  if (rows <= 0) return hipSuccess;
  // pieces of an average sequence (fixed chunks: of the longest)
  const int mean = a.chunk_blocks == 0 ? a.num_splits / a.B + 1 : a.num_splits;
  if (rows <= 256 && mean >= 64) return launch_shape<1, 8, 8>(a, stream);
  if (rows <= 1024 || (rows <= 2048 && mean >= 8)) return launch_shape<2, 4, 4>(a, stream);
  if (rows <= 4096) return launch_shape<2, 1, 4>(a, stream);
  return launch_shape<4, 1, 4>(a, stream);
}

}  // namespace snapmla
