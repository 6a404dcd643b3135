// Batched clustered neighbour search (paper, Sec. "AutoFocusFormer": equal-size
// clusters, fixed-size neighbourhoods by nearest-neighbour search over 2-D token
// coordinates).  Four kernels:
//   members  (only with an explicit cluster_id): token lists per cluster
//   centroid : double-precision mean of each cluster's coordinates -> fp32
//   near     : per cluster the M clusters with nearest centroids (up to 256 clusters
//              per image: by the search kernel itself)
//   knn      : per token the K nearest among the members of those M clusters
//              (staged in LDS, selected by a counted distance threshold and one sort)
// Selection is exact and unique: 64-bit keys (fp32 distance bits, index) compared
// as integers; distances are evaluated without fused multiply-add.  This file is
// compiled with -ffp-contract=off.
#include "cluster_common.h"
#include "device_util.h"
#include "launch.h"
#include "select_util.h"
#include "timing.h"

#include <algorithm>

namespace affmae {
namespace {

// Clusters hold S tokens, except that the last one (cluster G - 1, G = ceil(N / S)) holds what is left.
__device__ __forceinline__ int cluster_size(int c, int N, int S, int G) { return c == G - 1 ? N - (G - 1) * S : S; }

// members[b, c*S + r] = r-th token (ascending) whose cluster id is c.  One
// workgroup per image; a thread owns a cluster and scans the id array, which is
// staged through LDS in chunks.  Slots that an invalid assignment leaves unset
// keep the in-range default c*S + r.
constexpr int kMemChunk = 2048;
__global__ __launch_bounds__(256) void members_kernel(const int32_t* __restrict__ cluster_id, int N, int S, int G,
                                                     int32_t* __restrict__ members) {
  __shared__ int32_t ids[kMemChunk];
  const int b = blockIdx.x;
  const int32_t* cid = cluster_id + (size_t)b * N;
  int32_t* mem = members + (size_t)b * N;
  for (int i = threadIdx.x; i < N; i += blockDim.x) mem[i] = i;
  __syncthreads();
  for (int c0 = 0; c0 < G; c0 += blockDim.x) {
    const int c = c0 + threadIdx.x;
    int count = 0;
    for (int base = 0; base < N; base += kMemChunk) {
      const int n = min(kMemChunk, N - base);
      __syncthreads();
      for (int t = threadIdx.x; t < n; t += blockDim.x) ids[t] = cid[base + t];
      __syncthreads();
      if (c < G) {
        for (int t = 0; t < n; ++t) {
          if (ids[t] == c && count < cluster_size(c, N, S, G)) {
            mem[(size_t)c * S + count] = base + t;
            ++count;
          }
        }
      }
    }
  }
}

// A wave per kCentroids clusters: the lanes fetch the members' coordinates, 64 of a cluster at a time, into LDS, and then a
// lane per cluster and axis adds them up in double precision, in member order.  Bound by the latency of the reads and of
// the chain of 64 additions.  (A wave per cluster, every lane forming both sums from lane broadcasts, was bound by their
// issue: 16 images of 16384 tokens in clusters of 64 7.3 us, now 4.8; of 4096 5.3, now 3.9.)
constexpr int kCentroids = 8, kCentroidRow = 2 * kWave + 2;  // words; the lanes' words lie in banks of their own
__global__ __launch_bounds__(kWave) void centroid_kernel(const float* __restrict__ coords,
                                                        const int32_t* __restrict__ members, int B, int N, int S,
                                                        int G, float* __restrict__ centroid) {
  __shared__ __align__(8) float xy[kCentroids][kCentroidRow];
  const int lane = threadIdx.x, first = blockIdx.x * kCentroids;
  const int mine = lane >> 1, axis = lane & 1, gc = min(first + min(mine, kCentroids - 1), B * G - 1);
  const int size = cluster_size(gc % G, N, S, G);
  double sum = 0.0;
  for (int base = 0; base < S; base += kWave) {
    float2 v[kCentroids];
#pragma unroll
    for (int i = 0, b = first / G, c = first - b * G; i < kCentroids; ++i) {
      int tok = c * S + min(base + lane, cluster_size(c, N, S, G) - 1);
      if (members) tok = min(max(members[(size_t)b * N + tok], 0), N - 1);
      const float* at = coords + 2 * ((size_t)b * N + tok);
      v[i] = make_float2(at[0], at[1]);
      const bool wraps = c + 1 == G, more = first + i + 1 < B * G;  // (behind the last cluster: that one again)
      b += more && wraps ? 1 : 0;
      c = !more ? c : wraps ? 0 : c + 1;
    }
#pragma unroll
    for (int i = 0; i < kCentroids; ++i) *reinterpret_cast<float2*>(&xy[i][2 * lane]) = v[i];
    __syncthreads();
    const float* row = &xy[min(mine, kCentroids - 1)][axis];
    const int n = min(kWave, size - base);
    if (S % kWave == 0 && n == kWave) {
#pragma unroll
      for (int r = 0; r < kWave; ++r) sum += (double)row[2 * r];
    } else {
      for (int r = 0; r < n; ++r) sum += (double)row[2 * r];
    }
    __syncthreads();
  }
  if (mine < kCentroids && first + mine < B * G) centroid[2 * (size_t)gc + axis] = (float)(sum / (double)size);
}

// One wave per cluster: the M nearest centroids of the image, ascending.
__global__ __launch_bounds__(256) void near_kernel(const float* __restrict__ centroid, int B, int G, int M,
                                                  int32_t* __restrict__ near) {
  const int lane = threadIdx.x & (kWave - 1);
  const int gc = blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave);
  if (gc >= B * G) return;  // wave-uniform
  const int b = gc / G;
  const float* cen = centroid + (size_t)b * G * 2;
  const float cx = centroid[2 * (size_t)gc], cy = centroid[2 * (size_t)gc + 1];
  key_t best = kKeyMax;
  for (int base = 0; base < G; base += kWave) {
    const int e = base + lane;
    key_t key = kKeyMax;
    if (e < G) key = make_key(dist2(cx, cy, cen[2 * e], cen[2 * e + 1]), e);
    best = topk_push(best, key, lane, M - 1);
  }
  if (lane < M) near[(size_t)gc * M + lane] = (int32_t)(uint32_t)best;
}

// The K nearest among the members of a cluster's M near clusters, for the cluster's tokens; a wave serves every
// (4 parts)-th of them.  Coordinates and token ids of the candidates are staged in LDS once per workgroup, in rows of
// 64; up to 1024 candidates a wave then holds all its tokens long, a lane one candidate of every row (ROWS > 0), more
// are read from LDS as they are needed (ROWS = 0): a count of 4096 of them costs several times what is left of a query,
// so there it may be up to 128 and the steps interpolate (2 images of 4096 tokens, 64 clusters of 64 near, K = 64: 282 us
// with the steps of the other forms, 85 us as here; 8 images, 4 clusters of 512 near, K = 48: 104 and 91 us).
// Per token the wave looks for a distance threshold T with K <= #{candidates with d2 <= T} <= 64 by counting
// (ballots), starting from the previous token's threshold, and sorts the counted candidates once by (d2, index): see
// select_nearest.  The near clusters are taken in index order, so that candidates are queued in token order
// (contiguous clusters) and the sort of the queue nearly always succeeds on its short words (sort_queued).
// Bound by instruction issue, vector and scalar.  (Leaving out the rows whose bounding box is too far - a token's
// neighbours lie in 3.3 of its 8 rows - saved a third of the vector instructions and was no faster, in four forms: the
// tests and branches per row are scalar instructions, of which a SIMD issues no more than of the others.)
// `parts` workgroups share a cluster's tokens: with one per cluster a batch of few or large clusters leaves most of
// the chip idle (one cluster of 256 tokens: 85 us with one workgroup, 5 us with 64).
// Up to kNearInSearch clusters per image (a row of 64 centroids for each wave) the workgroup finds the near clusters itself:
// a launch less, 4 - 9 us.  More are searched by near_kernel, once per cluster: here every workgroup would sort several
// rows per wave in turn, with `parts` workgroups per cluster each for itself.
constexpr int kKnnWaves = 4;
constexpr int kNearInSearch = kKnnWaves * kWave;
constexpr int kFullChipWaves = 8192;  // 256 CUs x 4 SIMDs x 8 waves
constexpr int pend_keys(int ROWS) { return ROWS ? kWave : 2 * kWave; }  // queue of a wave: see select_nearest
size_t knn_lds_bytes(int ROWS, int rows) {
  return kKnnWaves * pend_keys(ROWS) * sizeof(key_t) + (size_t)rows * kWave * (sizeof(float2) + sizeof(int32_t));
}
template <int ROWS, bool MEMBERS>
__global__ __launch_bounds__(kKnnWaves* kWave) void knn_kernel(const float* __restrict__ coords,
                                                              const int32_t* __restrict__ members,
                                                              const float* __restrict__ centroid,
                                                              int32_t* __restrict__ near, int N, int S, int M, int K,
                                                              int G, int rows, int parts, uint32_t s_magic,
                                                              int32_t* __restrict__ nbr_idx) {
  extern __shared__ key_t lds[];
  __shared__ int32_t near_lds[kWave];
  __shared__ int32_t odd_lds[kKnnWaves];
  constexpr int kPend = pend_keys(ROWS);
  float2* cxy = reinterpret_cast<float2*>(lds + kKnnWaves * kPend);        // [rows][64]
  int32_t* ctok = reinterpret_cast<int32_t*>(cxy + (size_t)rows * kWave);  // [rows][64]
  const int gc = blockIdx.x / parts, part = blockIdx.x - gc * parts;
  const int b = gc / G, c = gc - b * G;
  const int Cn = M * S;
  const float* xy = coords + (size_t)b * N * 2;
  const int32_t* mem = MEMBERS ? members + (size_t)b * N : nullptr;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  key_t* pend = lds + wave * kPend;
  // lane m: the m-th of the near clusters in index order (M <= 64; they are distinct)
  int near_sorted;
  auto index_order = [&](int id) -> int {  // lane m < M: the m-th of the ids that lanes 0 .. M - 1 give
    int rank = 0;
    for (int m = 0; m < M; ++m) rank += __builtin_amdgcn_readlane(id, m) < id ? 1 : 0;
    return __builtin_amdgcn_ds_permute((lane < M ? rank : lane) * 4, id);
  };
  float2 own = make_float2(0.f, 0.f);  // this cluster's centroid
  if (G > 1) own = make_float2(centroid[2 * (size_t)gc], centroid[2 * (size_t)gc + 1]);
  if (G <= kNearInSearch) {
    // the near clusters themselves, a row of 64 centroids per wave (G == 1: there is one cluster, no centroid is needed)
    const int e = wave * kWave + lane;
    if (G > 1) {
      const float* cen = centroid + (size_t)b * G * 2;
      key_t key = kKeyMax;
      if (e < G) key = make_key(dist2(own.x, own.y, cen[2 * e], cen[2 * e + 1]), e);
      if (wave * kWave < G) pend[lane] = wave_sort(key, lane);
      __syncthreads();
    }
    if (wave == 0) {
      key_t best = 0ull;
      if (G > 1) {
        best = pend[lane];
        for (int row = 1; row * kWave < G; ++row) {  // the 64 smallest of two sorted rows are bitonic
          const key_t rev = lds[row * kPend + kWave - 1 - lane];
          best = wave_bitonic_merge(best < rev ? best : rev, lane);
        }
      }
      if (lane < M && part == 0) near[(size_t)gc * M + lane] = (int32_t)(uint32_t)best;
      near_lds[lane] = index_order(lane < M ? (int)(uint32_t)best : 0x7fffffff);
    }
    __syncthreads();
    near_sorted = near_lds[lane];
  } else {
    near_sorted = index_order(lane < M ? min(max(near[(size_t)gc * M + lane], 0), G - 1) : 0x7fffffff);
  }
  // a coordinate that is not finite among the candidates or in this cluster (whose centroid is not finite either then)
  bool odd = G > 1 && !finite_point(own.x, own.y);
  for (int p = threadIdx.x; p < rows * kWave; p += kKnnWaves * kWave) {  // (whole waves: all lanes take part)
    const int pp = p < Cn ? p : 0;
    const int m = fast_div(pp, s_magic), r = pp - m * S;
    const int e = __shfl(near_sorted, m);
    int tok = min(e * S + r, N - 1);
    if (MEMBERS) tok = min(max(mem[tok], 0), N - 1);
    const bool real = p < Cn && r < cluster_size(e, N, S, G);  // a short last cluster fills only part of its places
    // an empty place: its distance to any point is a NaN, whose bits lie above those of every distance
    const float x = xy[2 * (size_t)tok], y = xy[2 * (size_t)tok + 1];
    cxy[p] = make_float2(real ? x : __uint_as_float(0x7fc00000u), y);
    ctok[p] = real ? tok : -1;
    if (!MEMBERS) odd |= real && !finite_point(x, y);
  }
  if (!MEMBERS) {
    const bool any = __ballot(odd) != 0ull;
    if (lane == 0) odd_lds[wave] = any ? 1 : 0;
  }
  __syncthreads();
  auto key_at = [&](float qx, float qy, int row, int l) -> key_t {
    const float2 v = cxy[row * kWave + l];
    const int tok = ctok[row * kWave + l];
    return tok >= 0 ? make_key(dist2(qx, qy, v.x, v.y), MEMBERS ? tok : row * kWave + l) : kKeyMax;
  };
  const int my_size = cluster_size(c, N, S, G);
  const int step = parts * kKnnWaves, first = part * kKnnWaves + wave;
  const int served = first < my_size ? (my_size - 1 - first) / step + 1 : 0;  // tokens of this wave
  if (!MEMBERS) {
    // (distances may be NaN; "expect" puts the loop behind the others': 0.3 % of the search's time)
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(odd_lds[0] | odd_lds[1] | odd_lds[2] | odd_lds[3]) != 0, 0)) {
      for (int i = first; i < my_size; i += step) {
        const int qtok = c * S + i;
        const float qx = xy[2 * (size_t)qtok], qy = xy[2 * (size_t)qtok + 1];
        const uint32_t place = nearest_by_key(rows, K, lane, [&](int row, int l) { return key_at(qx, qy, row, l); });
        if (lane < K) nbr_idx[((size_t)b * N + qtok) * K + lane] = ctok[place];
      }
      return;
    }
  }
  float cx[ROWS ? ROWS : 1], cy[ROWS ? ROWS : 1];
#pragma unroll
  for (int row = 0; row < ROWS; ++row) {
    const float2 v = cxy[min(row, rows - 1) * kWave + lane];  // (ROWS is rounded up: the surplus rows are empty)
    cx[row] = row < rows ? v.x : __uint_as_float(0x7fc00000u);
    cy[row] = v.y;
  }
  uint32_t guess = 0u;  // threshold that worked for the previous token (0: none yet)
  for (int base = 0; base < served; base += kWave) {
    // lane i: token and coordinates of the i-th of the next 64
    int my_tok = c * S + first + min(base + lane, served - 1) * step;
    if (MEMBERS) my_tok = min(max(mem[my_tok], 0), N - 1);
    float my_x = xy[2 * (size_t)my_tok], my_y = xy[2 * (size_t)my_tok + 1];
    // a use of them here, so that the wait for the loads sits here: inside the loop it would also wait for the previous
    // token's store to reach memory
    asm volatile("" : "+v"(my_tok), "+v"(my_x), "+v"(my_y));
    for (int at = 0; at < min(kWave, served - base); ++at) {
      const int qtok = __builtin_amdgcn_readlane(my_tok, at);
      const float qx = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_x), at));
      const float qy = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_y), at));
      auto row_d2 = [&](int row) -> uint32_t {
        const float2 v = cxy[row * kWave + lane];
        return __float_as_uint(dist2(qx, qy, v.x, v.y));
      };
      auto row_low = [&](int row) -> uint32_t {  // contiguous clusters: the place stands for the token, ordered alike
        return MEMBERS ? (uint32_t)ctok[row * kWave + lane] : (uint32_t)(row * kWave + lane);
      };
      uint32_t d2[ROWS ? ROWS : 1];
#pragma unroll
      for (int row = 0; row < ROWS; ++row) d2[row] = __float_as_uint(dist2(qx, qy, cx[row], cy[row]));
      if (guess == 0u)  // no estimate: one of the distances, so that the count is not 0
        guess = min((uint32_t)__builtin_amdgcn_readlane(row_d2(0), kWave / 2), 0x7f800000u);
      const uint32_t best = select_nearest<!MEMBERS, ROWS ? kOneRow : kTwoSearched, ROWS == 0>(
          rows, K, guess, pend, lane,
          [&](auto f) {
#pragma unroll
            for (int row = 0; row < ROWS; ++row) f(d2[row], row_low(MEMBERS ? min(row, rows - 1) : row));
            if (ROWS == 0)
              for (int row = 0; row < rows; ++row) f(row_d2(row), row_low(row));
          },
          [&](int row, int l) { return key_at(qx, qy, row, l); });
      int tok = (int)best;
      if (!MEMBERS) tok = ctok[lane < K ? tok : 0];
      if (lane < K) nbr_idx[((size_t)b * N + qtok) * K + lane] = tok;
    }
  }
}

}  // namespace

hipError_t launch_knn(const KnnArgs& a, hipStream_t stream) {
  const int32_t* members = nullptr;
  if (a.cluster_id) {
    AFFMAE_LAUNCH("members_kernel", stream, members_kernel, dim3(a.B), dim3(256), 0, stream, a.cluster_id, a.N, a.S, a.G, a.members);
    members = a.members;
  }
  const int BG = a.B * a.G;
  if (a.G > 1)
    AFFMAE_LAUNCH("centroid_kernel", stream, centroid_kernel, dim3((BG + kCentroids - 1) / kCentroids), dim3(kWave), 0, stream, a.coords, members, a.B, a.N,
                  a.S, a.G, a.centroid);
  if (a.G > kNearInSearch)
    AFFMAE_LAUNCH("near_kernel", stream, near_kernel, dim3((BG + 3) / 4), dim3(256), 0, stream, a.centroid, a.B, a.G, a.M,
                  a.near_clusters);
  const int rows = (a.M * a.S + kWave - 1) / kWave;  // at most 64
  // enough workgroups for eight waves on every SIMD, while a wave still has a token to serve
  const int parts = std::max(1, std::min((kFullChipWaves / kKnnWaves + BG - 1) / BG, (std::min(a.S, a.N) + kKnnWaves - 1) / kKnnWaves));
  const dim3 grid((unsigned)BG * parts), block(kKnnWaves * kWave);
#define AFFMAE_KNN(R)                                                                                               \
  do {                                                                                                              \
    if (members)                                                                                                    \
      AFFMAE_LAUNCH("knn_kernel", stream, (knn_kernel<R, true>), grid, block, knn_lds_bytes(R, rows), stream, a.coords, members, \
                    a.centroid, a.near_clusters, a.N, a.S, a.M, a.K, a.G, rows, parts, div_magic(a.S), a.nbr_idx);              \
    else                                                                                                            \
      AFFMAE_LAUNCH("knn_kernel", stream, (knn_kernel<R, false>), grid, block, knn_lds_bytes(R, rows), stream, a.coords, members, \
                    a.centroid, a.near_clusters, a.N, a.S, a.M, a.K, a.G, rows, parts, div_magic(a.S), a.nbr_idx);              \
  } while (0)
  if (rows <= 2) AFFMAE_KNN(2);
  else if (rows <= 4) AFFMAE_KNN(4);
  else if (rows <= 6) AFFMAE_KNN(6);
  else if (rows <= 8) AFFMAE_KNN(8);
  else if (rows <= 12) AFFMAE_KNN(12);
  else if (rows <= 16) AFFMAE_KNN(16);
  else AFFMAE_KNN(0);
#undef AFFMAE_KNN
  return hipGetLastError();
}

}  // namespace affmae
