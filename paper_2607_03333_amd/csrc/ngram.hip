// gfx950 kernels of the n-gram (prompt-lookup) draft proposer, the draft
// source of the engine's n-gram speculative decoding that D3's proposer
// wraps (Sections 4.3 and 6.1).
//
// The key is the last n tokens of a sequence of L tokens, n from n_max down
// to n_min; the latest earlier occurrence (with a token after it) of the
// longest key that occurs gives up to k drafts: the tokens that follow it.
// For a position p <= L - 2, m(p) is the length of the common suffix of
// tokens[0..p] and tokens[0..L-1]; an occurrence of the n-token key ends at p
// exactly when m(p) >= n. With m capped at n_max, the longest key that
// occurs is the largest capped m (if it reaches n_min), and its latest
// occurrence the largest p with that value, so one maximum over the 64-bit
// key (capped m << 32) | p decides both.
//
//  * ngram_scan: workgroup (sequence, chunk) reads its chunk of positions and
//    the n_max - 1 tokens before it once, all loads in flight together with
//    those of the key, keeps them in LDS and computes m(p) there, eight
//    positions of a thread side by side. It writes the chunk's largest key;
//    the last chunk of a sequence runs to its end, whatever its length. The
//    drafts of a batch of one chunk per sequence are written here too.
//  * ngram_drafts: one wave per sequence takes the largest key over the
//    chunks and writes the drafts, -1 past the end of the sequence.
#include "device_common.h"
#include "ngram_kernels.h"

namespace spork {
namespace {

// The drafts of sequence s from the largest key `best` over its positions,
// written by `threads` threads of which the caller is `tx`.
__device__ __forceinline__ void write_drafts(const NgramArgs& a, int s, uint64_t best, int tx, int threads) {
  const int64_t base = a.seq_off[s];
  const int64_t L = a.seq_off[s + 1] - base;
  const int64_t p = static_cast<int64_t>(best & 0xFFFFFFFFu);
  // drafts available after the occurrence: tokens p+1 .. L-1
  const int64_t avail = best == 0 ? 0 : L - 1 - p;
  const int cnt = static_cast<int>(avail < a.k ? avail : a.k);
  for (int i = tx; i < a.k; i += threads)
    a.drafts[static_cast<size_t>(s) * a.k + i] = i < cnt ? a.tokens[base + p + 1 + i] : -1;
  if (tx == 0) a.n_drafts[s] = cnt;
}

__global__ void __launch_bounds__(256) ngram_scan(NgramArgs a) {
  constexpr int PER = kNgramChunk / 256;  // positions of a thread: tx, tx + 256, ...
  const int s = blockIdx.x / a.n_chunks, c = blockIdx.x % a.n_chunks;
  const int64_t base = a.seq_off[s];
  const int64_t L = a.seq_off[s + 1] - base;
  const int32_t* t = a.tokens + base;
  __shared__ int32_t tail[kNgramMaxN];
  __shared__ int32_t buf[kNgramMaxN + kNgramChunk];  // tokens lo - kNgramMaxN .. lo + kNgramChunk - 1
  const int tx = static_cast<int>(threadIdx.x);
  uint64_t best = 0;
  const int64_t end = c == a.n_chunks - 1 || (c + 1LL) * kNgramChunk > L - 1 ? L - 1 : (c + 1LL) * kNgramChunk;
  for (int64_t lo = static_cast<int64_t>(c) * kNgramChunk; lo < end; lo += kNgramChunk) {
    int32_t x[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) x[j] = lo + j * 256 + tx < end ? t[lo + j * 256 + tx] : 0;
    const int64_t before = lo - kNgramMaxN + tx;
    const int32_t halo = tx < kNgramMaxN && before >= 0 ? t[before] : 0;
    const int32_t key = tx < a.n_max && tx < L ? t[L - 1 - tx] : 0;
    __syncthreads();  // the chunk before has been read
    if (tx < kNgramMaxN) {
      buf[tx] = halo;
      tail[tx] = key;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) buf[kNgramMaxN + j * 256 + tx] = x[j];
    __syncthreads();
    int m[PER];  // matched so far; `alive`: bit j while position j still matches
    uint32_t alive = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const bool hit = lo + j * 256 + tx < end && x[j] == tail[0];
      m[j] = hit ? 1 : 0;
      alive |= hit ? 1u << j : 0u;
    }
    for (int d = 1; d < a.n_max && __any(alive != 0); ++d) {
      const int32_t want = tail[d];
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const bool hit = lo + j * 256 + tx >= d && buf[kNgramMaxN + j * 256 + tx - d] == want;
        if (!hit) alive &= ~(1u << j);
        m[j] += (alive >> j) & 1;
      }
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const uint64_t k = (static_cast<uint64_t>(m[j]) << 32) | static_cast<uint64_t>(lo + j * 256 + tx);
      if (m[j] >= a.n_min && k > best) best = k;
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const uint64_t other = __shfl_xor(best, o);
    best = other > best ? other : best;
  }
  __shared__ uint64_t wk[4];
  if ((threadIdx.x & 63) == 0) wk[threadIdx.x >> 6] = best;
  __syncthreads();
  best = wk[0];
  for (int i = 1; i < 4; ++i) best = wk[i] > best ? wk[i] : best;
  if (a.n_chunks == 1)
    write_drafts(a, s, best, tx, 256);
  else if (tx == 0)
    a.keys[static_cast<size_t>(s) * a.n_chunks + c] = best;
}

__global__ void __launch_bounds__(64) ngram_drafts(NgramArgs a) {
  const int s = blockIdx.x, lane = threadIdx.x;
  uint64_t best = 0;
  for (int c = lane; c < a.n_chunks; c += 64) {
    const uint64_t k = a.keys[static_cast<size_t>(s) * a.n_chunks + c];
    best = k > best ? k : best;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const uint64_t other = __shfl_xor(best, o);
    best = other > best ? other : best;
  }
  write_drafts(a, s, best, lane, 64);
}

}  // namespace

hipError_t launch_ngram_scan(const NgramArgs& a, hipStream_t stream) {
  if (a.n_seqs == 0) return hipSuccess;
  hipLaunchKernelGGL(ngram_scan, dim3(a.n_seqs * a.n_chunks), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_ngram_drafts(const NgramArgs& a, hipStream_t stream) {
  if (a.n_seqs == 0) return hipSuccess;
  hipLaunchKernelGGL(ngram_drafts, dim3(a.n_seqs), dim3(64), 0, stream, a);
  return hipGetLastError();
}

}  // namespace spork
