// Layout of the split (many workgroups per sequence) summary path's
// workspace, shared by the Max-IDF (maxidf_split.hip) and scorer
// (scorers.hip) kernels.  Per sequence: N presence bitmaps of
// W = ceil(V / 32) words (padded to 32 bytes), then the df table of 32 W
// bytes (a byte per id, or the nibble df - 1 per id for N <= 16).
#pragma once

#include "summary.hpp"

constexpr int kSplitThreads = 1024;

__host__ __device__ inline int64_t split_words(int vocab) { return ((int64_t)vocab + 31) / 32; }
__host__ __device__ inline int64_t split_df_bytes(int vocab) { return split_words(vocab) * 32; }
// the bitmaps, padded to 32 bytes so that the df table (and the next
// sequence) stays 32-byte aligned
__host__ __device__ inline int64_t split_bits_bytes(int num_blocks, int vocab) {
  return ((int64_t)num_blocks * split_words(vocab) * 4 + 31) & ~int64_t(31);
}
__host__ __device__ inline int64_t split_seq_bytes(int num_blocks, int vocab) {
  return split_bits_bytes(num_blocks, vocab) + split_df_bytes(vocab);
}

// Whether the split path is the faster one for a batch that it takes (1 to 16
// sequences), by the time on the device.  A workgroup that counts df over the
// whole sequence pays for its ids and its blocks, whatever the batch; the split
// path pays for three launches, and per (sequence, block) for the vocabulary's
// tables.  Measured over 3300 shapes of 1K to 256K ids, 2 to 16 blocks,
// vocabularies of 2000 to 128256 and every scorer, by the slots of 4096 ids that
// a sequence takes (summary.hpp):
//   up to 8: one launch takes 0.42 to 1.02 times the split path's time;
//   above 16: 0.96 to 2.6 times (its ids are packed, or streamed twice): BM25, 16
//     x 8 x 10240 ids 43.6 against 38.7 us, Max-IDF 16 x 12 x 8192 20.2, 13.4;
//   between: 0.58 to 1.5 times.  The difference, one launch less split, is linear
//     in the tables' bytes, the ids, the blocks and their length, and in the
//     rounds of 4096 ids that a workgroup scores: the split path's come in twos,
//     and a round of BM25 or Entropy compares each id with its whole chunk.  One
//     launch is chosen up to 1 us above the split path's time (the estimate is
//     within 1.3 us over 3979 shapes, chunks of 16 to 256): a loop of calls, bound
//     by two launches more, is then 2 to 3 us a call faster with it, a call by
//     itself at most 1 us slower (1 x 10 x 4096 ids, in a loop 10.6 against 12.9 us,
//     by itself 24.8 and 23.7, on the device 10.7 and 9.3).
enum SplitKind { kSplitMaxidf, kSplitScorer };
inline bool split_pays(SplitKind kind, int scorer, int batch, int64_t L, int num_blocks, int chunk,
                       int vocab) {
  const int64_t rounds = (L / num_blocks + 4095) / 4096, slots = num_blocks * rounds;
  if (slots <= 8 || slots > 16) return slots > 16;
  // us; per 1024 ids of a sequence, block, 1024 ids of a block, odd round, 64 ids of
  // a chunk in it
  struct { double c, ids, blocks, len, odd, cmp; } k;
  if (kind == kSplitMaxidf) k = {-3.25, 0.064, 0.20, -0.065, -0.55, 0.0};
  else if (scorer == PULSAR_SCORE_MAXIDF) k = {-3.55, 0.065, 0.17, 0.05, -0.55, 0.0};
  else if (scorer == PULSAR_SCORE_TFIDF) k = {-4.6, 0.058, 0.28, 0.0, -1.0, 0.14};
  else if (scorer == PULSAR_SCORE_BM25) k = {-3.85, 0.075, 0.154, -0.237, -0.57, -4.24};
  else k = {-4.35, 0.069, 0.175, -0.10, 0.0, -4.57};
  const double kL = (double)L / 1024.0;
  double d = k.c + k.ids * kL + k.blocks * num_blocks + k.len * kL / num_blocks;
  if (rounds & 1) d += k.odd + k.cmp * chunk / 64.0;
  return d > 0.165e-6 * batch * num_blocks * vocab;
}

// Copy of n 16-byte units (K rounds of kSplitThreads, n > (K - 1) *
// kSplitThreads) from global memory into LDS: all K loads are issued before
// the first store.  Lanes past the end copy the last unit onto itself, so no
// lane branches on its own load or store.
template <int K>
__device__ __forceinline__ void copy_rounds(const uint4* __restrict__ src, uint4* dst, int n,
                                            int tid) {
  uint4 r[K];
#pragma unroll
  for (int k = 0; k < K; ++k) r[k] = src[min(k * kSplitThreads + tid, n - 1)];
#pragma unroll
  for (int k = 0; k < K; ++k) dst[min(k * kSplitThreads + tid, n - 1)] = r[k];
}

// The same for any n up to PULSAR_LDS_BYTES / 16 units (10 rounds).
__device__ __forceinline__ void copy_to_lds(const uint4* __restrict__ src, uint4* dst, int n,
                                            int tid) {
  static_assert(PULSAR_LDS_BYTES / 16 / kSplitThreads == 10, "copy rounds below");
  switch ((n + kSplitThreads - 1) / kSplitThreads) {
    case 1: copy_rounds<1>(src, dst, n, tid); break;
    case 2: copy_rounds<2>(src, dst, n, tid); break;
    case 3: copy_rounds<3>(src, dst, n, tid); break;
    case 4: copy_rounds<4>(src, dst, n, tid); break;
    case 5: copy_rounds<5>(src, dst, n, tid); break;
    case 6: copy_rounds<6>(src, dst, n, tid); break;
    case 7: copy_rounds<7>(src, dst, n, tid); break;
    case 8: copy_rounds<8>(src, dst, n, tid); break;
    case 9: copy_rounds<9>(src, dst, n, tid); break;
    default: copy_rounds<10>(src, dst, n, tid); break;
  }
}

// The presence and df kernels of the split path for a batch that
// maxidf_split_workspace admits: the workspace's df table of every sequence
// (nibbles for N <= 16, else bytes), and the IDF table if idf is given.
int launch_split_df(const int32_t* ids, int batch, int64_t L, int num_blocks, int vocab,
                    float* idf, void* workspace, hipStream_t stream);
