// Balanced clustering along a Z-order curve (paper, Sec. "AutoFocusFormer":
// tokens are grouped into equal-size clusters by a space-filling-curve procedure;
// the curve is not named there - this library takes the Z-order (Morton) curve
// over coordinates quantised to 16 bits per axis of a caller-given frame).
//
// Per image the tokens are sorted by the 64-bit word (curve key << 32 | token
// index): unique words, so the order is exact and ties go to the lower index.
// Chunks of 512, 1024 or 2048 words are sorted by one workgroup each (a bitonic network
// whose words stay in registers, or in LDS where there are very many chunks).  Up
// to 16 chunks an image's order then follows in one more launch: a word's place is
// its place in its chunk plus the number of smaller words in every other chunk (binary
// searches).  Larger images are merged by the network's remaining steps over the
// words padded to a power of two (pads are all ones and end up last): steps whose
// partner lies in another chunk run over global memory, up to three per pass, the
// others in LDS, and a last kernel writes the order and each token's cluster
// (place along the curve / S).
#include "cluster_common.h"
#include "device_util.h"
#include "launch.h"
#include "select_util.h"
#include "timing.h"

#include <algorithm>

namespace affmae {
namespace {

typedef unsigned long long word_t;
constexpr int kChunk = 2048;       // words sorted in LDS by one workgroup (16 KB): many workgroups per image
constexpr int kSortThreads = 256;

struct ClusterParams {
  const float* coords;  // [B,N,2]
  int N, npad, S;
  uint32_t s_magic;  // reciprocal of S
  double x0, y0, w, h;  // frame
  word_t* words;  // [B][npad]
  int32_t* order;
  int32_t* cluster_id;
};

// floor((x - x0) / w * 65536) clamped to 0..65535, in double precision.
__device__ __forceinline__ uint32_t quantise16(float x, double x0, double w) {
  double q = floor(((double)x - x0) / w * 65536.0);
  q = q < 0.0 ? 0.0 : q;
  q = q > 65535.0 ? 65535.0 : q;
  return (uint32_t)q;
}

// bit i of v -> bit 2i
__device__ __forceinline__ uint32_t spread16(uint32_t v) {
  v = (v | (v << 8)) & 0x00ff00ffu;
  v = (v | (v << 4)) & 0x0f0f0f0fu;
  v = (v | (v << 2)) & 0x33333333u;
  v = (v | (v << 1)) & 0x55555555u;
  return v;
}

__device__ __forceinline__ word_t token_word(const ClusterParams& p, int b, int i) {
  if (i >= p.N) return ~0ull;
  const float* xy = p.coords + ((size_t)b * p.N + i) * 2;
  const uint32_t key = spread16(quantise16(xy[0], p.x0, p.w)) | (spread16(quantise16(xy[1], p.y0, p.h)) << 1);
  return ((word_t)key << 32) | (word_t)(uint32_t)i;
}

// R consecutive compare-exchange steps (k, J), (k, J/2), ... of the bitonic network on a chunk held in LDS, in one
// trip through LDS: a thread takes the 2^R words that these steps connect (strides J .. J >> (R-1)), exchanges
// them in registers and writes them back.  `first` is the global position of the chunk's first word (it
// decides the direction, which is the same for all words of a group because k > J).
// Place of word w in the LDS chunk: the XOR spreads every access pattern of the passes below over all
// banks (a thread's 2^R words with stride 1, 2 or 4 would otherwise fall on a few banks).
__device__ __forceinline__ int lds_place(int w) { return w ^ ((w >> 3) & 31); }

template <int R>
__device__ __forceinline__ void lds_pass(word_t* buf, int n, int first, int k, int J) {
  const int low = J >> (R - 1);
  for (int t = threadIdx.x; t < (n >> R); t += blockDim.x) {
    const int i0 = ((t & ~(low - 1)) << R) | (t & (low - 1));
    word_t v[1 << R];
#pragma unroll
    for (int m = 0; m < (1 << R); ++m) v[m] = buf[lds_place(i0 + m * low)];
    const bool ascending = ((first + i0) & k) == 0;
#pragma unroll
    for (int bit = R - 1; bit >= 0; --bit) {
#pragma unroll
      for (int m = 0; m < (1 << R); ++m) {
        if (!((m >> bit) & 1)) {
          const word_t a = v[m], c = v[m | (1 << bit)];
          const bool swap = (a > c) == ascending;
          v[m] = swap ? c : a;
          v[m | (1 << bit)] = swap ? a : c;
        }
      }
    }
#pragma unroll
    for (int m = 0; m < (1 << R); ++m) buf[lds_place(i0 + m * low)] = v[m];
  }
  __syncthreads();
}

// The steps j = J, J/2, ..., 1 of stage k, three at a time.
__device__ __forceinline__ void lds_steps(word_t* buf, int n, int first, int k, int J) {
  int j = J;
  while (j >= 4) {
    lds_pass<3>(buf, n, first, k, j);
    j >>= 3;
  }
  if (j == 2) lds_pass<2>(buf, n, first, k, 2);
  else if (j == 1) lds_pass<1>(buf, n, first, k, 1);
}

// Place along the curve of a token of the image: its entry of `order`, and its cluster.
__device__ __forceinline__ void emit(const ClusterParams& p, int b, word_t word, int place) {
  const int tok = (int)(uint32_t)word;
  p.order[(size_t)b * p.N + place] = tok;
  if (p.cluster_id) p.cluster_id[(size_t)b * p.N + tok] = exact_div(place, p.S, p.s_magic);
}

// One step of the bitonic network, words W t .. W t + W - 1 of the chunk in the registers of thread t: partners W J
// words apart are J threads apart.  Within a thread the partners are registers, within a wave the words move on the
// vector ALU (lane_xor_key), across waves through LDS.  `k`: size of the sorted blocks that the stage makes.
template <int W>
__device__ __forceinline__ void keep(word_t& mine, word_t other, bool keep_min) {
  mine = ((mine < other) == keep_min) ? mine : other;
}
template <int W, int J>
__device__ __forceinline__ void lane_step(word_t (&v)[W], int t, int k) {
  const bool keep_min = ((t * W & k) == 0) == ((t & J) == 0);  // (k > W here: all words of a thread alike)
#pragma unroll
  for (int m = 0; m < W; ++m) keep<W>(v[m], lane_xor_key<J>(v[m], t & (kWave - 1)), keep_min);
}
// (all threads of the workgroup call it, in groups of `threads` with a t and a `buf` of their own)
template <int W>
__device__ __forceinline__ void sort_in_registers(word_t (&v)[W], word_t* buf, int threads, int t) {
  const int n = threads * W;
#pragma unroll 1
  for (int k = 2; k <= n; k <<= 1) {
#pragma unroll 1
    for (int j = k >> 1; j >= W * kWave; j >>= 1) {  // across waves
      __syncthreads();
#pragma unroll
      for (int m = 0; m < W; ++m) buf[m * threads + t] = v[m];
      __syncthreads();
      const bool keep_min = ((t * W & k) == 0) == ((t * W & j) == 0);
#pragma unroll
      for (int m = 0; m < W; ++m) keep<W>(v[m], buf[m * threads + (t ^ (j / W))], keep_min);
    }
    const int top = k >> 1;  // first step of the stage
    if (top >= W * 32) lane_step<W, 32>(v, t, k);
    if (top >= W * 16) lane_step<W, 16>(v, t, k);
    if (top >= W * 8) lane_step<W, 8>(v, t, k);
    if (top >= W * 4) lane_step<W, 4>(v, t, k);
    if (top >= W * 2) lane_step<W, 2>(v, t, k);
    if (top >= W) lane_step<W, 1>(v, t, k);
#pragma unroll
    for (int j = W / 2; j >= 1; j >>= 1) {
      if (top >= j) {
#pragma unroll
        for (int m = 0; m < W; ++m) {
          if (m & j) continue;
          const bool ascending = ((t * W + m) & k) == 0;
          const word_t a = v[m], c = v[m | j];
          const bool swap = (a > c) == ascending;
          v[m] = swap ? c : a;
          v[m | j] = swap ? a : c;
        }
      }
    }
  }
}

// Number of words of the sorted run[0 .. n - 1] (n a power of two) that are smaller than `word` (or equal, if asked for).
__device__ __forceinline__ int count_below(const word_t* run, int n, word_t word, bool or_equal) {
  auto below = [&](word_t x) { return x < word || (or_equal && x == word); };
  int s = 0;
  for (int step = n >> 1; step >= 1; step >>= 1) s += below(run[s + step - 1]) ? step : 0;
  return s + (below(run[s]) ? 1 : 0);  // (s <= n - 1 here)
}

// Builds the words of one chunk and sorts it: RUNS groups of THREADS threads sort THREADS W words each in registers, then a
// word's place is its place in its run plus the counts of smaller words in the others.  WHOLE: the chunk is the image,
// its order is written at once; otherwise the sorted words.  Bound by a chain of dependent steps with few waves per SIMD:
// 2048 words by 256 threads with 8 words each, the whole network in registers or through LDS, 18 - 19 us for 128 chunks,
// as four runs of 512 by 1024 threads 12.6 us.  Images of 513 to 1024 tokens take two runs (2048 images of 600: 57 us
// with four, half of whose words are pads; 38 as one network over 1024 words; 29 with two), images of up to 64 a wave
// (THREADS; 100 000 images of 16: 192 us with 256 threads each, 40 with 64).
template <int W, int RUNS, bool WHOLE, int THREADS = kSortThreads>
__global__ __launch_bounds__(THREADS* RUNS) void cluster_sort_chunk_kernel(ClusterParams p, int chunks, bool network) {
  constexpr int kRun = W * THREADS, kWords = kRun * RUNS;
  __shared__ word_t buf[kWords];
  const int b = blockIdx.x / chunks, c = blockIdx.x - b * chunks, first = c * kWords;
  const int g = threadIdx.x / THREADS, t = threadIdx.x % THREADS;
  const word_t flip = network && (c & 1) ? ~0ull : 0ull;  // the network goes on from chunks in alternating order
  word_t v[W];
#pragma unroll
  for (int m = 0; m < W; ++m) v[m] = token_word(p, b, first + m * THREADS * RUNS + threadIdx.x) ^ flip;  // (any order will do)
  sort_in_registers<W>(v, buf + g * kRun, THREADS, t);
  __syncthreads();
#pragma unroll
  for (int m = 0; m < W; ++m) buf[g * kRun + t * W + m] = v[m];
  __syncthreads();
  int place[W];
#pragma unroll
  for (int m = 0; m < W; ++m) {
    place[m] = t * W + m;
    if (RUNS > 1) {
#pragma unroll
      for (int o = 1; o < RUNS; ++o) {
        // equal words (pads, or complemented pads, only): those of the lower run come first
        const int other = (g + o) % RUNS;
        place[m] += count_below(buf + other * kRun, kRun, v[m], other < g);
      }
    }
  }
  if (WHOLE) {
#pragma unroll
    for (int m = 0; m < W; ++m)
      if (v[m] != ~0ull) emit(p, b, v[m], place[m]);
    return;
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < W; ++m) buf[place[m]] = v[m];
  __syncthreads();
#pragma unroll
  for (int m = 0; m < W; ++m) {
    const int at = m * THREADS * RUNS + threadIdx.x;
    p.words[(size_t)b * p.npad + first + at] = buf[at] ^ flip;
  }
}

// The same for chunks of larger images in a launch of kManyChunks or more: the whole network through LDS by 256 threads, a
// longer chain but half the work.  1000 images of 4096 tokens (2000 chunks), whole clustering: 106 us, 120 with four runs;
// 512 / 900 / 1024 chunks 44 / 69 / 68 us against 41 / 71 / 70.
constexpr int kManyChunks = 1024;
__global__ __launch_bounds__(kSortThreads) void cluster_sort_chunk_lds_kernel(ClusterParams p, int chunks, bool network) {
  __shared__ word_t buf[kChunk];
  const int b = blockIdx.x / chunks, c = blockIdx.x - b * chunks, first = c * kChunk;
  const word_t flip = network && (c & 1) ? ~0ull : 0ull;
  for (int t = threadIdx.x; t < kChunk; t += kSortThreads) buf[lds_place(t)] = token_word(p, b, first + t) ^ flip;
  __syncthreads();
  for (int k = 2; k <= kChunk; k <<= 1) lds_steps(buf, kChunk, 0, k, k >> 1);
  word_t* out = p.words + (size_t)b * p.npad + first;
  for (int t = threadIdx.x; t < kChunk; t += kSortThreads) out[t] = buf[lds_place(t)] ^ flip;
}

// Number of words below `word` in each of the chunks first .. first + U - 1 behind chunk `own` (cyclically; those from
// `others` + 1 on are not counted), added up: by binary search, 6 steps on every 32nd word of a chunk (in LDS), 5 on the
// words between (the lanes of a wave hold neighbouring words, so they read neighbouring places).  The steps of the U
// searches alternate: each is a chain of reads.
constexpr int kMaxRankChunks = 16;
template <int CH, int U>
__device__ __forceinline__ int count_in_chunks(const word_t (&split)[kMaxRankChunks][64], const word_t* w, int chunks, int own,
                                               int first, word_t word) {
  int c[U], s[U], n[U];
  const word_t* from[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    c[u] = own + min(first + u, chunks - 1);
    c[u] -= c[u] >= chunks ? chunks : 0;
    s[u] = n[u] = 0;
  }
#pragma unroll
  for (int step = 32; step >= 1; step >>= 1)
#pragma unroll
    for (int u = 0; u < U; ++u) s[u] += split[c[u]][s[u] + step - 1] < word ? step : 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    s[u] += split[c[u]][s[u]] < word ? 1 : 0;  // (s <= 63 here)
    from[u] = w + (size_t)c[u] * CH + max(s[u] - 1, 0) * (CH / 64) + 1;
  }
  // words below it among those after the last such
#pragma unroll
  for (int step = CH / 128; step >= 1; step >>= 1)
#pragma unroll
    for (int u = 0; u < U; ++u) n[u] += from[u][n[u] + step - 1] < word ? step : 0;
  int count = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) count += s[u] == 0 || first + u >= chunks ? 0 : (s[u] - 1) * (CH / 64) + 1 + n[u];
  return count;
}

// Order of an image whose `chunks` (2 .. 16) chunks are sorted: a word's place is its place in its chunk plus, for
// every other chunk, the number of smaller words there.
// Replaces the seven further launches of the network at 8 chunks (16 images of 16384 tokens: 23 us with both kernels, 49 us
// with the network; one image of 32768 tokens, 16 chunks, 21 us against 53; of 32769 by the network 80).  The line at 16
// keeps the workgroup's samples at 8 KB of LDS; the ranks would still be the faster way a little beyond.
// Bound by the chains of reads and by the scattered writes of the order and the clusters: 16 images of 8 chunks 13.8 us with
// one search after the other, 11.9 with seven at a time, 10.0 with an image's workgroups on one XCD, whose L2 then joins the
// writes to a line (and reads the words once).  (Comparing 32-bit keys, as earlier chunks have the lower numbers: 10 - 10.6.)
// CH: words of a chunk.  Small batches leave most CUs without a chunk of 2048, and a chunk's sort is a chain that shorter
// chunks shorten: a run of 512 words to a workgroup as long as that makes no more than 8 chunks an image (whole clustering
// with chunks of 2048 / 1024 / 512: 16 images of 4096 tokens 15.7 / 14.4 / 13.8 us, 64 17.7 / 15.0 / 15.4, 256 35.6 / 38.3 /
// 40.4), two runs beyond (4 images of 8192 16.0 / 14.0 / 13.8, 16 17.3 / 14.3 / 14.6, 64 25.1 / 26.6 / 30.4; 4 images of
// 16384 17.3 / 15.3, 16 22.4 / 23.5; 14 us are the host's share of two launches).
constexpr int kFewChunks512 = 512, kFewChunks1024 = 192;
template <int CH>
__global__ __launch_bounds__(256) void cluster_rank_kernel(ClusterParams p, int chunks) {
  __shared__ word_t split[kMaxRankChunks][64];
  unsigned block = blockIdx.y * gridDim.x + blockIdx.x;
  if (gridDim.x * gridDim.y % 8 == 0) block = (unsigned)xcd_contiguous_block(block, gridDim.x * gridDim.y);
  const int b = block / gridDim.x, part = block - b * gridDim.x;
  const word_t* w = p.words + (size_t)b * p.npad;
  const int at = part * 256 + threadIdx.x;  // place among the chunks' words (a workgroup stays inside one chunk)
  const int own = part / (CH / 256);
  const word_t word = w[at];
  for (int i = threadIdx.x; i < chunks * 64; i += 256) split[i >> 6][i & 63] = w[(size_t)i * (CH / 64)];
  __syncthreads();
  int place = at - own * CH;
  if (chunks == 2) place += count_in_chunks<CH, 1>(split, w, chunks, own, 1, word);
  else if (chunks <= 5) place += count_in_chunks<CH, 4>(split, w, chunks, own, 1, word);
  else if (chunks <= 8) place += count_in_chunks<CH, 7>(split, w, chunks, own, 1, word);
  else
    for (int o = 1; o < chunks; o += 8) place += count_in_chunks<CH, 8>(split, w, chunks, own, o, word);
  if (word != ~0ull) emit(p, b, word, place);
}

// R consecutive steps (k, J), (k, J/2), ... whose strides are all at least the chunk size: partners sit in
// different chunks, so the 2^R words a thread connects come from and go back to global memory.
template <int R>
__global__ __launch_bounds__(256) void cluster_global_pass_kernel(ClusterParams p, int k, int J) {
  const int groups = p.npad >> R;
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (t >= groups) return;
  const int low = J >> (R - 1);
  const int i0 = ((t & ~(low - 1)) << R) | (t & (low - 1));
  word_t* w = p.words + (size_t)b * p.npad;
  word_t v[1 << R];
#pragma unroll
  for (int m = 0; m < (1 << R); ++m) v[m] = w[i0 + m * low];
  const bool ascending = (i0 & k) == 0;
#pragma unroll
  for (int bit = R - 1; bit >= 0; --bit) {
#pragma unroll
    for (int m = 0; m < (1 << R); ++m) {
      if (!((m >> bit) & 1)) {
        const word_t a = v[m], c = v[m | (1 << bit)];
        const bool swap = (a > c) == ascending;
        v[m] = swap ? c : a;
        v[m | (1 << bit)] = swap ? a : c;
      }
    }
  }
#pragma unroll
  for (int m = 0; m < (1 << R); ++m) w[i0 + m * low] = v[m];
}

// The steps j = chunk/2 .. 1 of stage k (k > chunk size), in LDS.
__global__ __launch_bounds__(kSortThreads) void cluster_merge_chunk_kernel(ClusterParams p, int chunk, int k) {
  extern __shared__ word_t buf[];
  const int chunks_per_image = p.npad / chunk;
  const int b = blockIdx.x / chunks_per_image, c = blockIdx.x % chunks_per_image;
  const int first = c * chunk;
  word_t* io = p.words + (size_t)b * p.npad + first;
  for (int t = threadIdx.x; t < chunk; t += blockDim.x) buf[lds_place(t)] = io[t];
  __syncthreads();
  lds_steps(buf, chunk, first, k, chunk >> 1);
  for (int t = threadIdx.x; t < chunk; t += blockDim.x) io[t] = buf[lds_place(t)];
}

__global__ __launch_bounds__(256) void cluster_emit_kernel(ClusterParams p) {
  const int place = blockIdx.x * blockDim.x + threadIdx.x;
  if (place < p.N) emit(p, blockIdx.y, p.words[(size_t)blockIdx.y * p.npad + place], place);  // pads sort last
}

int next_pow2(int n) {
  int v = 2;
  while (v < n) v <<= 1;
  return v;
}

}  // namespace

size_t cluster_workspace_bytes(int B, int N) { return (size_t)B * next_pow2(N) * sizeof(word_t); }

static hipError_t launch_images(const ClusterParams& p, int B, hipStream_t stream) {
  const int N = p.N;
#define AFFMAE_SORT(W, RUNS, WHOLE, CHUNKS, NETWORK)                                                               \
  AFFMAE_LAUNCH("cluster_sort_chunk_kernel", stream, (cluster_sort_chunk_kernel<W, RUNS, WHOLE>),                  \
                dim3((unsigned)B * (CHUNKS)), dim3(kSortThreads * (RUNS)), 0, stream, p, CHUNKS, NETWORK)
#define AFFMAE_SORT_CHUNKS(CHUNKS, NETWORK)                                                                        \
  do {                                                                                                             \
    if ((long long)B * (CHUNKS) < kManyChunks) AFFMAE_SORT(2, 4, false, CHUNKS, NETWORK);                          \
    else                                                                                                           \
      AFFMAE_LAUNCH("cluster_sort_chunk_kernel", stream, cluster_sort_chunk_lds_kernel,                            \
                    dim3((unsigned)B * (CHUNKS)), dim3(kSortThreads), 0, stream, p, CHUNKS, NETWORK);              \
  } while (0)
  if (N <= kChunk) {  // one chunk per image
    if (N <= kWave)
      AFFMAE_LAUNCH("cluster_sort_chunk_kernel", stream, (cluster_sort_chunk_kernel<1, 1, true, kWave>), dim3((unsigned)B), dim3(kWave),
                    0, stream, p, 1, false);
    else if (N <= kSortThreads) AFFMAE_SORT(1, 1, true, 1, false);
    else if (N <= 2 * kSortThreads) AFFMAE_SORT(2, 1, true, 1, false);
    else if (N <= 4 * kSortThreads) AFFMAE_SORT(2, 2, true, 1, false);
    else AFFMAE_SORT(2, 4, true, 1, false);
    return hipGetLastError();
  }
  const int chunks = (N + kChunk - 1) / kChunk;
#define AFFMAE_RANK(CH)                                                                                            \
  AFFMAE_LAUNCH("cluster_rank_kernel", stream, cluster_rank_kernel<CH>, dim3((N + CH - 1) / CH * (CH / 256), B), dim3(256), 0, stream, \
                p, (N + CH - 1) / CH)
  const long long few = (long long)B * ((N + 511) / 512), mid = (long long)B * ((N + 1023) / 1024);
  if (N <= 8 * 512 && few <= kFewChunks512) {
    AFFMAE_SORT(2, 1, false, (N + 511) / 512, false);
    AFFMAE_RANK(512);
    return hipGetLastError();
  }
  if (N <= kMaxRankChunks * 1024 && mid <= kFewChunks1024) {
    AFFMAE_SORT(2, 2, false, (N + 1023) / 1024, false);
    AFFMAE_RANK(1024);
    return hipGetLastError();
  }
  if (chunks <= kMaxRankChunks) {
    AFFMAE_SORT_CHUNKS(chunks, false);
    AFFMAE_RANK(kChunk);
    return hipGetLastError();
  }
  const int chunk = kChunk;
  const size_t lds = (size_t)chunk * sizeof(word_t);
  const int threads = kSortThreads;
  const dim3 per_chunk(B * (p.npad / chunk));
  AFFMAE_SORT_CHUNKS(p.npad / chunk, true);
#undef AFFMAE_SORT_CHUNKS
#undef AFFMAE_SORT
#undef AFFMAE_RANK
  for (int k = chunk * 2; k <= p.npad; k <<= 1) {
    int j = k >> 1;
    while (j >= chunk) {  // up to three steps per pass over global memory
      int steps = 0;
      for (int jj = j; jj >= chunk && steps < 3; jj >>= 1) ++steps;
      const dim3 grid(((p.npad >> steps) + 255) / 256, B);
      if (steps == 3)
        AFFMAE_LAUNCH("cluster_global_pass_kernel", stream, cluster_global_pass_kernel<3>, grid, dim3(256), 0, stream, p, k, j);
      else if (steps == 2)
        AFFMAE_LAUNCH("cluster_global_pass_kernel", stream, cluster_global_pass_kernel<2>, grid, dim3(256), 0, stream, p, k, j);
      else
        AFFMAE_LAUNCH("cluster_global_pass_kernel", stream, cluster_global_pass_kernel<1>, grid, dim3(256), 0, stream, p, k, j);
      j >>= steps;
    }
    AFFMAE_LAUNCH("cluster_merge_chunk_kernel", stream, cluster_merge_chunk_kernel, per_chunk, dim3(threads), lds, stream,
                  p, chunk, k);
  }
  AFFMAE_LAUNCH("cluster_emit_kernel", stream, cluster_emit_kernel, dim3((N + 255) / 256, B), dim3(256), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_cluster(const float* coords, int B, int N, int S, double x0, double y0, double w, double h,
                          int32_t* order, int32_t* cluster_id, void* workspace, hipStream_t stream) {
  ClusterParams p;
  p.N = N; p.npad = next_pow2(N); p.S = S;
  p.x0 = x0; p.y0 = y0; p.w = w; p.h = h;
  p.s_magic = div_magic(S);
  // A launch has fewer than 2^32 threads: the chunk sort gives an image at most 256 or, beyond 512 tokens, one for every
  // two of its padded words.  (The batch is cut only where it would not be accepted: 2^24 images, 2^33 tokens.)
  const long long threads = N <= 2 * kSortThreads ? kSortThreads : std::max(kChunk, p.npad) / 2;
  const int most = (int)std::min((long long)B, 0xffffffffll / threads);
  for (int b0 = 0; b0 < B; b0 += most) {
    p.coords = coords + (size_t)b0 * N * 2;
    p.words = static_cast<word_t*>(workspace) + (size_t)b0 * p.npad;
    p.order = order + (size_t)b0 * N;
    p.cluster_id = cluster_id ? cluster_id + (size_t)b0 * N : nullptr;
    const hipError_t e = launch_images(p, std::min(most, B - b0), stream);
    if (e != hipSuccess) return e;
    if (B - b0 <= most) break;  // (b0 + most may pass the largest int)
  }
  return hipSuccess;
}

}  // namespace affmae
