// gfx950 kernels around a step: token scatter into the paged KV pools, the
// block copy of copy-on-write (Section 4.1) and the patch of a plan's image.
#include "device_common.h"

namespace spork {
namespace {

// Fewest (token, KV head) pairs of a call that goes a block at a time. Below,
// the scatter by token has more threads to hide the stores' latency with; above,
// its 2- and 4-byte stores bound it. By token against by blocks, calls back to
// back, 8 heads of 128 channels (us): bf16, 16-token blocks, 2,048 tokens in runs
// of 9 21.9 and 8.3, in a row 18.3 and 8.2, each in a block of its own 31.2 and
// 18.0; fp32 35.9 and 10.1, 25.1 and 8.3, 36.5 and 30.8. At the line itself (576
// tokens) the two are level in 16-token blocks (8.0 and 8.1 in runs of 9); in
// 32-token blocks tokens that each have a block to themselves pay for the line
// being there: bf16 10.2 and 10.8, fp32 9.9 and 10.9, and 1,024 of 64 bf16
// channels 8.6 and 9.7, where runs of 9 gain (2,048: 23.3 and 8.6).
constexpr int64_t kBlocksMin = 4608;
// Most waves of a launch with several waves per block: while there is room for
// them, they store what one wave would store alone, in a row. 576 single bf16
// tokens in 32-token blocks, one wave and four: 14.4 and 10.8 us; 576 in runs of
// 9 on cold caches 13.2 and 9.7. Past it the chip is full either way, and more
// waves only make its last round longer (15,001 tokens in a row, 4 heads, one
// wave of 3,752 and two: 10.6 and 13.2 us).
constexpr int64_t kSharedWaves = 2048;

// Scatter by token: a thread per 16-byte chunk of a token and head.
template <typename T>
__global__ void __launch_bounds__(256) kv_write_kernel(int hkv, int D, int BS, int64_t num_slots, T* kc,
                                                       T* vc, const int64_t* slots, const T* kn,
                                                       const T* vn, int n, int* bad) {
  constexpr int VEC = 16 / sizeof(T);
  const int per_tok = hkv * (D / VEC);
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= static_cast<int64_t>(n) * per_tok) return;
  const int i = static_cast<int>(idx / per_tok);
  const int rem = static_cast<int>(idx % per_tok);
  const int h = rem / (D / VEC), cchunk = rem % (D / VEC);
  const int64_t slot = slots[i];
  if (slot < 0 || slot >= num_slots) {
    if (rem == 0 && bad != nullptr) atomicAdd(bad, 1);
    return;
  }
  const int64_t b = slot / BS, off = slot % BS;
  const size_t src = (static_cast<size_t>(i) * hkv + h) * D + static_cast<size_t>(cchunk) * VEC;
  *reinterpret_cast<uint4*>(kc + ((static_cast<size_t>(b) * hkv + h) * BS + off) * D + cchunk * VEC) =
      *reinterpret_cast<const uint4*>(kn + src);
  const T* vs = vn + src;
  T* vd = vc + (static_cast<size_t>(b) * hkv + h) * static_cast<size_t>(D) * BS + off;
#pragma unroll
  for (int e = 0; e < VEC; ++e) vd[static_cast<size_t>(cchunk * VEC + e) * BS] = vs[e];
}

// --------------------------------------------------------------------------
// The scatter of many tokens, a block at a time: a workgroup of one wave, or of
// several (kSharedWaves), per (window of BS tokens, KV head). The V pool holds a block transposed ([D][BS]), so a token's
// channels lie BS elements apart and the kernel above stores them one by one;
// here the workgroup transposes its window through LDS, and a window whose tokens
// fill one block in order (all but the ends of an appended run) goes out as
// contiguous 16-byte stores. The windows are laid out from the offset of the
// first token in its block. Any other window stores V by element, tokens
// fastest.
// LDS: dword rows of D channels; a bf16 row holds a pair of tokens (packed in
// registers), an fp32 row one. A 16-byte piece of the pool is the same channel
// of four rows; the padding puts the pieces that a wave reads at once into
// different banks (fp32 with 32-token blocks: two lanes per bank).
// Bound by the stream from and to HBM: 15,001 tokens of 8 heads of 128 bf16
// channels 149 us by element stores, 38.8 us by blocks, 23.6 us with
// non-temporal loads (calls over three pools in turn, whose 123 MB each the
// last-level cache partly holds; cold 25.9 us, 4.7 TB/s).
// Whole blocks are stored non-temporally too. With ordinary stores the
// last-level cache is left full of lines still to be written back, and the next
// step pays for them: the first step over new prompts, ordinary and
// non-temporal stores, 390 and 318 us (96 unforked sequences of up to 8,191
// tokens), 278 and 232 (forked decode), 831 and 749 (mixed verify and decode).
// The write itself, ordinary and non-temporal: bf16, 16-token blocks, 15,001
// tokens 23.6 and 23.7, 62,500 tokens 103 and 100 (its first call over a new
// pool 103 and 120); fp32 15,001 48.3 and 46.4; 32-token blocks, bf16
// 15,001 20.9 and 22.9, fp32 4,000 12.4 and 10.5. A prompt's write and the first
// decode over it, cold: 8,000 tokens 40.5 and 41.2, 60,000 160 and 147.
// --------------------------------------------------------------------------
template <typename T, int D, int BS, int NT>
__global__ void __launch_bounds__(NT) kv_write_blocks(int hkv, int64_t num_slots, T* kc, T* vc, const int64_t* slots,
                                                      const T* kn, const T* vn, int n, int* bad) {
  constexpr int VEC = 16 / sizeof(T), CH = D / VEC;  // 16-byte chunks of a token
  constexpr int PACK = 4 / sizeof(T);                // tokens of an LDS row
  constexpr int R = BS / PACK, QN = R / 4;           // rows; pieces per channel
  constexpr int STRIDE = D + (QN == 2 ? 8 : 4);
  constexpr int KIT = BS * CH / NT, VIT = R * CH / NT, OIT = D * QN / NT;
  __shared__ __align__(16) uint32_t tile[R * STRIDE];
  const int tid = threadIdx.x;
  const int h = static_cast<int>(blockIdx.x % static_cast<unsigned>(hkv));
  const int64_t s0 = slots[0];
  const int shift = s0 < 0 ? 0 : static_cast<int>(s0 % BS);
  const int64_t i0 = static_cast<int64_t>(blockIdx.x / static_cast<unsigned>(hkv)) * BS - shift;
  if (i0 >= n) return;
  const auto has = [&](int t) { return i0 + t >= 0 && i0 + t < n; };
  const auto src = [&](const T* x, int t, int c) {
    return reinterpret_cast<const uint4*>(x + (static_cast<size_t>(i0 + t) * hkv + h) * D + c * VEC);
  };
  const uint4 zero = make_uint4(0, 0, 0, 0);
  uint4 vr[VIT][PACK], kr[KIT];
#pragma unroll
  for (int it = 0; it < VIT; ++it) {
    const int r = (it * NT + tid) / CH, c = tid % CH;
#pragma unroll
    for (int p = 0; p < PACK; ++p) vr[it][p] = has(r * PACK + p) ? load_stream(src(vn, r * PACK + p, c)) : zero;
  }
#pragma unroll
  for (int it = 0; it < KIT; ++it) {
    const int t = (it * NT + tid) / CH;
    kr[it] = has(t) ? load_stream(src(kn, t, tid % CH)) : zero;
  }
  // lane t of each wave (and t + BS, ...): the slot of token t
  const int tt = tid % BS;
  const int64_t slot = has(tt) ? slots[i0 + tt] : -1;
  const bool ok = slot >= 0 && slot < num_slots;
  if (bad != nullptr && h == 0 && tid < BS && has(tt) && !ok) atomicAdd(bad, 1);
#pragma unroll
  for (int it = 0; it < VIT; ++it) {
    const int r = (it * NT + tid) / CH, c = tid % CH;
    uint32_t* row = tile + r * STRIDE + c * VEC;
    if constexpr (PACK == 1) {
      *reinterpret_cast<uint4*>(row) = vr[it][0];
    } else {
      const uint4 a = vr[it][0], b = vr[it][1];
      const auto lo2 = [](uint32_t x, uint32_t y) { return (x & 0xFFFFu) | (y << 16); };
      const auto hi2 = [](uint32_t x, uint32_t y) { return (x >> 16) | (y & 0xFFFF0000u); };
      *reinterpret_cast<uint4*>(row) = make_uint4(lo2(a.x, b.x), hi2(a.x, b.x), lo2(a.y, b.y), hi2(a.y, b.y));
      *reinterpret_cast<uint4*>(row + 4) = make_uint4(lo2(a.z, b.z), hi2(a.z, b.z), lo2(a.w, b.w), hi2(a.w, b.w));
    }
  }
  __syncthreads();
  const int64_t first = __shfl(slot, 0);
  const bool whole = __all(ok && slot == first + tt) && first % BS == 0;
  if (whole) {
    const size_t base = (static_cast<size_t>(first / BS) * hkv + h) * (D * BS);
    uint4* kd = reinterpret_cast<uint4*>(kc + base);
    uint4* vd = reinterpret_cast<uint4*>(vc + base);
#pragma unroll
    for (int it = 0; it < KIT; ++it) store_stream(kd + it * NT + tid, kr[it]);
#pragma unroll
    for (int it = 0; it < OIT; ++it) {
      const int d = (it * NT + tid) / QN, q = tid % QN;
      const uint32_t* col = tile + 4 * q * STRIDE + d;
      store_stream(vd + it * NT + tid, make_uint4(col[0], col[STRIDE], col[2 * STRIDE], col[3 * STRIDE]));
    }
    return;
  }
#pragma unroll
  for (int it = 0; it < KIT; ++it) {
    const int64_t ks = __shfl(slot, (it * NT + tid) / CH);
    if (ks >= 0 && ks < num_slots)
      *reinterpret_cast<uint4*>(kc + ((static_cast<size_t>(ks / BS) * hkv + h) * BS + ks % BS) * D + tid % CH * VEC) =
          kr[it];
  }
  if (!ok) return;
  T* vd = vc + (static_cast<size_t>(slot / BS) * hkv + h) * (D * BS) + slot % BS;
  const T* col = reinterpret_cast<const T*>(tile + tt / PACK * STRIDE) + tt % PACK;
#pragma unroll 8
  for (int d = tid / BS; d < D; d += NT / BS) vd[static_cast<size_t>(d) * BS] = col[d * PACK];
}

template <typename T>
__global__ void __launch_bounds__(256) kv_copy_kernel(int hkv, int D, int BS, T* kc, T* vc, int src, int dst,
                                                      int nv) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= static_cast<int64_t>(hkv) * nv * D) return;
  const int h = static_cast<int>(idx / (static_cast<int64_t>(nv) * D));
  const int rem = static_cast<int>(idx % (static_cast<int64_t>(nv) * D));
  const int off = rem / D, d = rem % D;
  const size_t ks = ((static_cast<size_t>(src) * hkv + h) * BS + off) * D + d;
  const size_t kd = ((static_cast<size_t>(dst) * hkv + h) * BS + off) * D + d;
  kc[kd] = kc[ks];
  const size_t vs = ((static_cast<size_t>(src) * hkv + h) * D + d) * BS + off;
  const size_t vd = ((static_cast<size_t>(dst) * hkv + h) * D + d) * BS + off;
  vc[vd] = vc[vs];
}

// Word writes into a plan's device image (spork_plan_advance): the patch
// travels as the kernel's argument, so nothing is copied from the host.
__global__ void __launch_bounds__(256) image_patch_kernel(int32_t* image, ImagePatch patch) {
  for (int i = threadIdx.x; i < patch.n; i += 256) image[patch.off[i]] = patch.val[i];
}

template <typename T, int D, int BS>
void write_blocks(int hkv, int64_t num_slots, T* kc, T* vc, const int64_t* slots, const T* kn, const T* vn, int n, int* bad,
                  hipStream_t stream) {
  constexpr int kPieces = D * BS * sizeof(T) / 16 * sizeof(T) / 4;  // of the window's LDS rows, one loaded by a thread at a time
  constexpr int kShared = kPieces < 256 ? kPieces : 256;
  // one window more than n / BS rounded up: the first may hold a single token
  const unsigned units = static_cast<unsigned>((static_cast<int64_t>(n) + 2 * BS - 2) / BS * hkv);
  if (static_cast<int64_t>(units) * (kShared / 64) <= kSharedWaves)
    hipLaunchKernelGGL((kv_write_blocks<T, D, BS, kShared>), dim3(units), dim3(kShared), 0, stream, hkv, num_slots, kc, vc,
                       slots, kn, vn, n, bad);
  else
    hipLaunchKernelGGL((kv_write_blocks<T, D, BS, 64>), dim3(units), dim3(64), 0, stream, hkv, num_slots, kc, vc, slots, kn,
                       vn, n, bad);
}

template <typename T>
void write_blocks(int hkv, int d, int bs, int64_t num_slots, void* kc, void* vc, const int64_t* slots, const void* kn,
                  const void* vn, int n, int* bad, hipStream_t stream) {
  const auto f = d == 128 ? (bs == 16 ? write_blocks<T, 128, 16> : write_blocks<T, 128, 32>)
                          : (bs == 16 ? write_blocks<T, 64, 16> : write_blocks<T, 64, 32>);
  f(hkv, num_slots, static_cast<T*>(kc), static_cast<T*>(vc), slots, static_cast<const T*>(kn), static_cast<const T*>(vn),
    n, bad, stream);
}

}  // namespace

hipError_t launch_image_patch(int32_t* image, const ImagePatch& patch, hipStream_t stream) {
  if (patch.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(image_patch_kernel, dim3(1), dim3(256), 0, stream, image, patch);
  return hipGetLastError();
}

hipError_t launch_kv_write(int32_t dtype, int32_t hkv, int32_t head_dim, int32_t block_size,
                           int64_t num_slots, void* k_cache, void* v_cache, const int64_t* slots,
                           const void* k_new, const void* v_new, int32_t n, int32_t* bad_slots,
                           hipStream_t stream) {
  if (n == 0) return hipSuccess;
  if (static_cast<int64_t>(n) * hkv >= kBlocksMin && (head_dim == 64 || head_dim == 128) && (block_size == 16 || block_size == 32)) {
    const auto f = dtype == 1 ? write_blocks<uint16_t> : write_blocks<float>;
    f(hkv, head_dim, block_size, num_slots, k_cache, v_cache, slots, k_new, v_new, n, bad_slots, stream);
    return hipGetLastError();
  }
  const int vec = dtype == 1 ? 8 : 4;
  const int64_t total = static_cast<int64_t>(n) * hkv * (head_dim / vec);
  const dim3 grid(static_cast<unsigned>((total + 255) / 256));
  if (dtype == 1)
    hipLaunchKernelGGL(kv_write_kernel<uint16_t>, grid, dim3(256), 0, stream, hkv, head_dim, block_size, num_slots,
                       static_cast<uint16_t*>(k_cache), static_cast<uint16_t*>(v_cache), slots,
                       static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new), n, bad_slots);
  else
    hipLaunchKernelGGL(kv_write_kernel<float>, grid, dim3(256), 0, stream, hkv, head_dim, block_size, num_slots,
                       static_cast<float*>(k_cache), static_cast<float*>(v_cache), slots,
                       static_cast<const float*>(k_new), static_cast<const float*>(v_new), n, bad_slots);
  return hipGetLastError();
}

hipError_t launch_kv_copy(int32_t dtype, int32_t hkv, int32_t head_dim, int32_t block_size,
                          void* k_cache, void* v_cache, int32_t src, int32_t dst, int32_t n_valid,
                          hipStream_t stream) {
  if (n_valid == 0) return hipSuccess;
  const int64_t total = static_cast<int64_t>(hkv) * n_valid * head_dim;
  const dim3 grid(static_cast<unsigned>((total + 255) / 256));
  if (dtype == 1)
    hipLaunchKernelGGL(kv_copy_kernel<uint16_t>, grid, dim3(256), 0, stream, hkv, head_dim, block_size,
                       static_cast<uint16_t*>(k_cache), static_cast<uint16_t*>(v_cache), src, dst, n_valid);
  else
    hipLaunchKernelGGL(kv_copy_kernel<float>, grid, dim3(256), 0, stream, hkv, head_dim, block_size,
                       static_cast<float*>(k_cache), static_cast<float*>(v_cache), src, dst, n_valid);
  return hipGetLastError();
}

}  // namespace spork
