// gfx950 (MI355X, CDNA4) attention kernels of the forked-decode hot path.
//
//  * attn_bf16 / attn_f32: partial attention of one work item's token range
//    for up to RT 16-row tiles of query rows (split-K). A work item is either
//    a fork group's shared prefix, read once for every member's rows
//    (Section 4.1: probes reuse the main thread's prefix KV), or one
//    thread's private range, where verify rows apply the causal rule over
//    the drafts (Section 4.3). Q.K^T and P.V run on MFMA with fp32
//    accumulation. bf16: K and V stream from HBM with 16-byte direct-to-LDS
//    loads (non-temporal) into a ring of LDS stages that the waves of a
//    workgroup share; fp32: 16-byte loads straight into registers.
//  * merge: log-sum-exp merge of an output row's partials (the batch's
//    maximum and weighted sum by DPP reductions over eight lanes), written
//    in the input dtype, plus the row's lse; the same launch runs the accept
//    of a verify step (Section 4.3, steps 2-3) and clears the persistent
//    launch's cursors for the next call.
#include "device_common.h"

namespace spork {
namespace {

// --------------------------------------------------------------------------
// Online softmax step shared by both attention kernels. `sv` holds this
// lane's 8 base-2 scores (query row = lane % 16, tokens chosen by the caller;
// the 4 lanes with the same lane % 16 together hold 32 tokens). Updates the
// lane's running max / partial sum and returns the probabilities and the
// rescale factor for the accumulator.
// --------------------------------------------------------------------------
__device__ __forceinline__ float softmax_step(float (&sv)[8], float& m, float& l) {
  float mx = sv[0];
#pragma unroll
  for (int j = 1; j < 8; ++j) mx = fmaxf(mx, sv[j]);
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  const float mn = fmaxf(m, mx);
  const float mu = mn == kNegInf ? 0.0f : mn;  // rows with nothing visible yet stay at zero
  const float alpha = exp2_fast(m - mu);
  float ps = 0.0f;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    sv[j] = exp2_fast(sv[j] - mu);
    ps += sv[j];
  }
  l = l * alpha + ps;
  m = mn;
  return alpha;
}

// --------------------------------------------------------------------------
// bf16 partial attention. Persistent workgroups of 4 or 8 waves work through
// lists of units; a unit is a token range of one work item and a slice of its query
// rows. The range streams through a ring of LDS slots, one 32-token K/V tile
// ("stage", 16 KB) each, filled by direct global-to-LDS 16-byte loads
// (global_load_lds_dwordx4: lane i of an instruction lands at the
// instruction's LDS base + 16*i), so the stages in flight hold no registers.
// Each wave issues 4 such loads per stage, or 2 of 8 waves (the lower half of
// the waves the K half, the upper one the V half); a barrier publishes the next two stages to all waves and frees
// the slots read before it. Two kernels share that stream:
//   narrow (attn_bf16): two workgroups per compute unit, up to 8 16-row tiles
//     each, 16x16x32 products; decode and short verify rows, bound by HBM.
//     With 8 waves: one workgroup per compute unit, up to 16 tiles; the
//     multi-row shapes (long verify, prefill) unless all their units suit
//     the wide kernel.
//   wide (attn_bf16_wide): one workgroup per compute unit, up to 8 32-row
//     tiles, 32x32x16 products; multi-row shapes whose slices are full, 13 to
//     16 tiles, and whose units are long enough (kWideStages) to pay for
//     filling and draining its pipeline. The plan chooses one kernel for all
//     units.
//
// LDS slot layout (1024 chunks of 16 bytes). Bank model (measured on
// gfx950): 64 banks of 4 bytes, so a 16-byte slot s sits in bank group
// s mod 16; a ds_read_b128 serves a wave in four groups of 16 lanes (half
// lane >> 5, phase = parity of lane bits 2-4: lanes 0-3, 12-15, 20-27 |
// 4-11, 16-19, 28-31 of each half), and inside a group distinct addresses
// in one bank group serialise. The operand reads of both kernels are
// conflict-free:
//   K: chunk t*16 + (c ^ k_swz(t)) holds channels 8c..8c+7 of tile token t;
//   V: 16-token blocks: chunk 512 + 256*h + 2*d + (q ^ v_swz(d)) holds tokens
//      16h + 8q .. + 7 of channel d, so that every load instruction reads one
//      block and its address is a scalar base plus a fixed lane offset (the
//      bench workload 3% faster than with a per-lane choice between the
//      stage's two blocks); 32-token blocks: chunk 512 + 4*d + (q ^ v_swz(d))
//      holds tokens 8q .. 8q + 7.
//
// The narrow kernel per stage and row tile (r16 = lane % 16, g = lane / 16):
//   S^T = K Q^T via v_mfma_f32_16x16x32_bf16; A-row r16 of half hh is tile
//   token 8*(r16/4) + 4*hh + r16%4, so the lane receives scores of query row
//   r16 for tokens 8g + j (j = 0..7, halves concatenated); the contraction
//   slot of channel d is (k-step d/32, lane group (d%32)/8, element d%8) on
//   both operands.
//   O^T += V^T P^T: A = V^T (channel 16*dt + r16, tokens 8g..8g+7), B = the
//   lane's own 8 probabilities; the accumulator holds query row r16 at
//   channels 16*dt + 4g + i, so the rescale by the row's factor is lane-local.
// The wide kernel's layout stands at its head.
// --------------------------------------------------------------------------
constexpr int kStageChunks = 1024;  // 32 tokens x (K + V) x 128 channels x 2 bytes / 16
// LDS stages per workgroup: 4 for two workgroups on a compute unit (4 waves),
// 8 for one (8 waves). A barrier publishes two stages (4 waves: 2 in flight, 8:
// 6). Against one stage per barrier this halves the barriers, and the waves
// drift apart inside a pair instead of all reading the same operands right
// after every barrier: on the narrow loop (with a stage fewer in flight) the
// Qwen3-4B batch 3.6% and the bench workload 1.6% faster (the fork tree 0.8%
// slower); four per barrier: slower.
constexpr int kPer = 2;  // stages a barrier publishes

// Cache-policy bits of the K/V loads: non-temporal. Every KV byte is read
// once per launch, and streaming loads marked this way reach 7.2 TB/s on
// MI355X against 5.9 TB/s with the default policy (measured with the
// direct-to-LDS read-ceiling kernel in the same ring shape).
constexpr int kNonTemporal = 2;
constexpr int kUnitBlocks = kUnitTableEntries;   // block-table entries a unit may span (see kMaxUnitTokens)
constexpr float kRescaleSlack = 8.0f;  // base-2 headroom before the reference max moves
constexpr float kRescaleSum = 256.0f;  // 2^kRescaleSlack: bound on a lane's 8 probabilities of a row

typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef __attribute__((address_space(1))) void* global_void_ptr;

// XOR swizzles of the LDS slot layout (above) that keep the operand reads of
// the narrow (16x16 products) and the wide (32x32) kernel free of bank
// conflicts: of a K token's channel groups, and of a V channel's token octets.
template <bool WIDE>
__device__ __forceinline__ int k_swz(int t) {
  return WIDE ? (t & 3) | (t & 4) | ((t >> 1) & 8) : (t & 3) | ((t >> 1) & 12);
}
template <int BS, bool WIDE>
__device__ __forceinline__ int v_swz(int d) {
  return BS == 16 ? (WIDE ? (d >> 3) & 1 : 0) : (d >> (WIDE ? 3 : 1)) & 3;
}

// Zero the bf16 lanes of an 8-token chunk starting at position `first` whose
// position is at or past `end` (two tokens per 32-bit word).
__device__ __forceinline__ uint4 zero_past(uint4 v, int first, int end) {
  uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t lo = first + 2 * i < end ? 0x0000FFFFu : 0u;
    const uint32_t hi = first + 2 * i + 1 < end ? 0xFFFF0000u : 0u;
    w[i] &= lo | hi;
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, bf16x2{static_cast<__bf16>(a), static_cast<__bf16>(b)});
}

// LDS operand reads outside the compiler's view. The compiler cannot tell the
// direct-to-LDS loads of later stages from these reads of the current stage
// and would otherwise wait for every load in flight before each read. The
// waits are explicit: lds_wait() takes the destination registers as in-out
// operands, so no consumer can be scheduled before it.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_ptr)(const_cast<void*>(p))));
}

template <int OFF = 0>
__device__ __forceinline__ u32x4 lds_read_b128(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset field");
  u32x4 r;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(OFF) : "memory");
  return r;
}

// A block-table entry, read from LDS at a wave-uniform address without a
// wait. tab_wait() waits for the read and takes the register as in-out
// operand, so no use moves above it (a copy of a register that the read has
// not yet written would copy stale contents, since the compiler does not know
// the read is still in flight).
__device__ __forceinline__ uint32_t tab_read(uint32_t addr) {
  uint32_t r;
  asm volatile("ds_read_b32 %0, %1" : "=v"(r) : "v"(addr) : "memory");
  return r;
}
__device__ __forceinline__ void tab_wait(uint32_t& r) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(r) : : "memory"); }
template <int N>
__device__ __forceinline__ void tab_wait_all(uint32_t (&r)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) tab_wait(r[i]);
}

// Wait for all LDS reads but the KEEP issued last (LDS reads complete in
// order), with the read registers as in-out operands.
template <int KEEP>
__device__ __forceinline__ void lds_wait(u32x4 (&r)[8]) {
  asm volatile("s_waitcnt lgkmcnt(%8)"
               : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]), "+v"(r[4]), "+v"(r[5]), "+v"(r[6]), "+v"(r[7])
               : "i"(KEEP)
               : "memory");
}

// The same for one register and a count that is a constant once inlined.
__device__ __forceinline__ void lds_wait_one(u32x4& r, int keep) {
  asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(r) : "i"(keep) : "memory");
}

// Workgroup-uniform reads of a unit's descriptors from the plan image (which
// no kernel writes while the attention launch runs) as scalar loads, on the
// scalar cache and its own counter, instead of vector loads that queue behind
// the stream's loads. Exactly the descriptor's bytes are read.
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ WaveDesc load_wave_desc(const WaveDesc* p) {
  static_assert(sizeof(WaveDesc) == 24, "WaveDesc layout");
  i32x4 x;
  i32x2 y;
  asm volatile("s_load_dwordx4 %0, %2, 0x0\n\ts_load_dwordx2 %1, %2, 0x10\n\ts_waitcnt lgkmcnt(0)"
               : "=s"(x), "=s"(y)
               : "s"(p)
               : "memory");
  return WaveDesc{x[0], x[1], x[2], x[3], y[0], y[1]};
}
__device__ __forceinline__ ItemDesc load_item_desc(const ItemDesc* p) {
  static_assert(sizeof(ItemDesc) == 32, "ItemDesc layout");
  i32x8 x;
  asm volatile("s_load_dwordx8 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(x) : "s"(p) : "memory");
  ItemDesc it;
  static_assert(sizeof(it) == sizeof(x), "ItemDesc layout");
  __builtin_memcpy(&it, &x, sizeof(it));
  return it;
}
__device__ __forceinline__ int load_int_uniform(const int32_t* p) {
  int x;
  asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(x) : "s"(p) : "memory");
  return x;
}

// Workgroup barrier that publishes this wave's LDS writes (and no global
// memory operation: no fence).
__device__ __forceinline__ void barrier_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Workgroup barrier without the memory fence of __syncthreads(): callers make
// their own direct-to-LDS loads complete first (wait_vmcnt). The memory
// clobber keeps loads, stores and LDS operations on their side of it.
__device__ __forceinline__ void barrier_nofence() { asm volatile("s_barrier" ::: "memory"); }

// s_waitcnt on the vector-memory counter only (expcnt and lgkmcnt left open).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Wait until at most `after` (0..7) stages of this wave's direct-to-LDS loads
// (LPW per stage), and no older vector load, are still in flight.
template <int LPW>
__device__ __forceinline__ void wait_stage(int after) {
  static_assert(7 * LPW < 64, "vmcnt range");
  switch (after) {
    case 7: wait_vmcnt<7 * LPW>(); break;
    case 6: wait_vmcnt<6 * LPW>(); break;
    case 5: wait_vmcnt<5 * LPW>(); break;
    case 4: wait_vmcnt<4 * LPW>(); break;
    case 3: wait_vmcnt<3 * LPW>(); break;
    case 2: wait_vmcnt<2 * LPW>(); break;
    case 1: wait_vmcnt<LPW>(); break;
    default: wait_vmcnt<0>(); break;
  }
}

// The workgroup's take of a unit and what both kernels read at its start.
struct UnitStart {
  WaveDesc w;
  ItemDesc it;
  int tok_hi, nb;   // end of the range, blocks of its table: with the growth since the plan
  int tb0, nstage;  // first tile token and 32-token stages
};
template <int BS>
__device__ __forceinline__ UnitStart unit_start(const AttnArgs& a, const WaveDesc& w) {
  UnitStart u;
  u.w = w;
  u.it = load_item_desc(a.items + w.item);
  // Tokens appended to a private range's thread since the plan was made: the
  // range's last unit, its rows' horizons and its table grow by them.
  u.tok_hi = w.tok_hi == u.it.hi ? w.tok_hi + u.it.grow : w.tok_hi;
  u.nb = u.it.grow != 0 ? (u.it.hi + u.it.grow + BS - 1) / BS : u.it.n_blocks;
  u.tb0 = w.tok_lo & ~(kTileTokens - 1);
  u.nstage = (u.tok_hi - u.tb0 + kTileTokens - 1) / kTileTokens;
  return u;
}

// The unit's slice of the block table, staged in LDS before the ring starts
// and read per stage outside the compiler's view (a vector load of the table
// inside the loop would make its wait also wait for every direct-to-LDS load
// issued before it), ahead of its use: tab[i] = table entry tb0/BS + i
// (clamped to the table).
template <int BS, int THREADS>
__device__ __forceinline__ void stage_table(const AttnArgs& a, const UnitStart& u, int tid, int* tab) {
  const int32_t* __restrict__ table = a.tables + u.it.table_off;
  const int tab0 = u.tb0 / BS;
  const int ntab = min((u.tb0 + u.nstage * kTileTokens + 16) / BS - tab0 + 1, kUnitBlocks);  // planner keeps it below
  for (int i = tid; i < ntab; i += THREADS) {
    const int bi = tab0 + i;
    tab[i] = table[bi < u.nb ? bi : u.nb - 1];
  }
}

// A wave's direct-to-LDS loads of a stage, kLoads = 16 / NW of them:
// instruction k of wave w fills chunks (kLoads*w + k)*64 + lane. All lanes of
// a wave read one block of the stage (16-token blocks: the second and fourth
// quarter of the waves read its second), at a scalar base plus the lane's
// fixed byte offset.
template <int BS, int NW, bool WIDE>
struct StageLoader {
  static constexpr int kLoads = 16 / NW;
  const uint16_t* pool;
  size_t head, hkv;
  uint32_t off[kLoads];
  uint32_t tab_base;  // LDS address of stage 0's table entry
  int wave, last;     // last stage of the unit
  __device__ __forceinline__ void init(const AttnArgs& a, const UnitStart& u, int wave_, int lane, const int* tab) {
    wave = wave_;
    last = u.nstage - 1;
    head = static_cast<size_t>(u.it.kv_head);
    hkv = static_cast<size_t>(a.hkv);
    pool = static_cast<const uint16_t*>(wave < NW / 2 ? a.k_cache : a.v_cache);
    tab_base = lds_addr(tab) + (BS == 16 && (wave & (NW / 4)) != 0 ? 4u : 0u);
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const int chunk = (kLoads * wave + k) * 64 + lane;
      if (wave < NW / 2) {
        const int t = chunk >> 4;
        off[k] = 2u * ((t % BS) * 128 + 8 * ((chunk & 15) ^ k_swz<WIDE>(t)));
      } else if (BS == 16) {
        const int d = (chunk & 255) >> 1;
        off[k] = 2u * (d * BS + 8 * ((chunk & 1) ^ v_swz<BS, WIDE>(d)));
      } else {
        const int d = (chunk - 512) >> 2;
        off[k] = 2u * (d * BS + 8 * ((chunk & 3) ^ v_swz<BS, WIDE>(d)));
      }
    }
  }
  // Table entry of this wave's block of stage `st` (clamped to the unit's
  // last stage), read without a wait.
  __device__ __forceinline__ uint32_t entry(int st) const {
    return tab_read(tab_base + (128u / BS) * static_cast<uint32_t>(min(st, last)));
  }
  __device__ __forceinline__ const char* base(uint32_t ent) const {
    const int e = __builtin_amdgcn_readfirstlane(static_cast<int>(ent));
    return reinterpret_cast<const char*>(pool + (static_cast<size_t>(e) * hkv + head) * (static_cast<size_t>(BS) * 128));
  }
  // As a buffer load over the one block: a scalar base and a 32-bit lane
  // offset, where a global load takes a 64-bit address per lane.
  __device__ __forceinline__ void load(const char* src, uint4* slot, int k) const {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src), 0, BS * 128 * 2, 0x00027000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(slot + (kLoads * wave + k) * 64), 16, off[k], 0, 0,
                                             kNonTemporal);
  }
  __device__ __forceinline__ void issue(uint32_t ent, uint4* slot) const {
    const char* src = base(ent);
#pragma unroll
    for (int k = 0; k < kLoads; ++k) load(src, slot, k);
  }
};

// Argmax unit u (row x vocabulary chunk) of a verify step.
template <int NT>
__device__ __forceinline__ void verify_argmax_unit(const AcceptArgs& acc, int u) {
  const int row = u / acc.chunks, c = u % acc.chunks;
  uint64_t* key = acc.keys + static_cast<size_t>(row) * acc.chunks + c;
  const size_t roff = static_cast<size_t>(row) * acc.vocab;
  if (acc.logits_dtype == 1)
    argmax_unit<uint16_t, NT, false>(static_cast<const uint16_t*>(acc.logits) + roff, acc.vocab, acc.chunks, c, key,
                                     nullptr);
  else
    argmax_unit<float, NT, false>(static_cast<const float*>(acc.logits) + roff, acc.vocab, acc.chunks, c, key, nullptr);
}

// Verify step: the greedy argmax over the logits fills the tail of the
// launch. Workgroups whose lists are done take (row, chunk) units from one
// shared cursor, so the compute units that finish early stream the logits
// while the last attention units drain.
template <int NT>
__device__ __forceinline__ void argmax_tail(const AttnArgs& a, int tid, int& next_unit) {
  if (a.tail_units <= 0) return;
  __syncthreads();  // every wave has read the last list take
  for (;;) {
    if (tid == 0) next_unit = atomicAdd(a.cursors + a.n_lists * kCursorStride, 1);
    __syncthreads();
    const int u = __builtin_amdgcn_readfirstlane(next_unit);
    if (u < 0 || u >= a.tail_units) break;
    verify_argmax_unit<NT>(a.acc, u);
    // The unit ends with thread 0 storing the key and the next take starts
    // with thread 0 taking a unit: this barrier keeps the two thread-0
    // regions apart, so the compiler cannot join them across the loop's
    // back edge into a loop whose waves run different barrier counts.
    __syncthreads();
  }
}

// Softmax in base 2 with a lazily moved reference max: scores enter as
// p = 2^(s*c - m) with m the row's reference; m (and the accumulator, by
// 2^(m_old - m_new)) moves only when a lane's probabilities of the row sum
// past 2^kRescaleSlack, so p <= 2^kRescaleSlack and most stages skip the
// rescale. The merge only needs (m, l, o) to be consistent, not m to be the
// exact maximum. rescale() is the uncommon case, some lane of the wave past
// that bound or a row without a reference (m = -inf: its sum is inf or NaN):
// the row maxima are reduced over the row's lanes (those that differ in the
// bits of XOR0 and above), the reference moved where it lags by more than
// kRescaleSlack (rows that did not trigger keep theirs) and the probabilities
// recomputed.
template <int XOR0, int N, int NA, typename Acc, typename Pop>
__device__ __forceinline__ void rescale(const float (&sv)[N], float c, float& m, float& l, Acc (&o)[NA], float& ps,
                                        Pop& pop) {
  float mx = sv[0] * c;
#pragma unroll
  for (int e = 1; e < N; ++e) mx = fmaxf(mx, sv[e] * c);
#pragma unroll
  for (int x = XOR0; x < 64; x *= 2) mx = fmaxf(mx, __shfl_xor(mx, x));
  if (mx > m + kRescaleSlack) {  // row-uniform: all lanes of the row agree
    const float alpha = exp2_fast(m - mx);  // 0 for a row's first visible tile
    l *= alpha;
#pragma unroll
    for (int i = 0; i < NA; ++i) o[i] *= alpha;
    m = mx;
  }
  const float mu = m == kNegInf ? 0.0f : m;
  ps = 0.0f;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const float pv = exp2_fast(__builtin_fmaf(sv[e], c, -mu));
    ps += pv;
    pop.set(e, pv);
  }
}

// The score of a masked position: -inf once times the scores' factor (which is
// not zero, but may be below it).
__device__ __forceinline__ float masked_score(float c) { return c < 0.0f ? -kNegInf : kNegInf; }

// Probabilities as packed bf16 pairs, the B operand of the P.V products.
template <int N>
struct Probs {
  uint32_t w[N / 2];
  float prev;
  __device__ __forceinline__ void set(int e, float p) {
    if (e & 1) w[e / 2] = pack_bf16(prev, p);
    else prev = p;
  }
  __device__ __forceinline__ bf16x8 operand(int h = 0) const {
    return __builtin_bit_cast(bf16x8, u32x4{w[4 * h], w[4 * h + 1], w[4 * h + 2], w[4 * h + 3]});
  }
};

template <int RTW, int BS, int NW>
__global__ void __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) attn_bf16(AttnArgs a) {
  constexpr int D = 128;
  constexpr int kRing = NW == 4 ? 4 : 8;
  static_assert(BS == 16 || BS == 32, "unsupported block size");
  __shared__ uint4 smem[kRing][kStageChunks];
  __shared__ __align__(16) int tab[kUnitBlocks];
  __shared__ int next_unit;
  // Persistent workgroup: it takes the next unit of its compute unit's list
  // (shared with the other workgroup resident there) until the list is done.
  const int tid = threadIdx.x;
  const int list = static_cast<int>(blockIdx.x) % a.n_lists;
  const int list0 = load_int_uniform(a.wg_off + list), list_len = load_int_uniform(a.wg_off + list + 1) - list0;
  // Thread 0 takes each unit before the workgroup needs it: the first here,
  // each next one at the end of the current unit, before its partial results
  // are stored, so neither the atomic's round trip nor the stores' sit
  // between two units. A barrier without a memory fence publishes the take.
  if (tid == 0) next_unit = atomicAdd(a.cursors + list * kCursorStride, 1);
  for (;;) {
  barrier_lds();
  const int taken = __builtin_amdgcn_readfirstlane(next_unit);
  // told that a list's end is rare, the compiler lays a unit's code out in a row (16 sessions with 16 drafts over
  // 16,383 tokens 254.2 -> 252.1 us a step)
  if (__builtin_expect(taken < 0 || taken >= list_len, 0)) break;
  const WaveDesc w = load_wave_desc(a.waves + list0 + taken);
  const UnitStart u = unit_start<BS>(a, w);
  const int tok_hi = u.tok_hi, tb0 = u.tb0, nstage = u.nstage;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  // Row tiles go to waves by `cw`, the wave index rotated by two in the
  // second workgroup of a compute unit (workgroups b and b + n_lists share
  // one): wave w of both shares SIMD w, and with 5-7 tiles (two for some
  // waves, one for others) the rotation pairs each wave holding two tiles
  // with one holding one.
  const int cw = NW == 4 ? (wave + 2 * (static_cast<int>(blockIdx.x) / a.n_lists)) & 3 : wave;
  const int lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const uint16_t* __restrict__ qg = static_cast<const uint16_t*>(a.q);
  const int ntiles = (w.nrows + 15) >> 4;

  // Row descriptors of this wave's tiles, loaded together with the unit's
  // block table (below); the query rows they name are loaded once the table
  // is staged, and complete behind the ring's first loads.
  RowDesc rdesc[RTW];
  bool own[RTW], has_row[RTW];
#pragma unroll
  for (int j = 0; j < RTW; ++j) {
    const int tile = cw + NW * j;
    own[j] = tile < ntiles;
    const int i = tile * 16 + r16;
    has_row[j] = own[j] && i < w.nrows;
    rdesc[j] = a.rows[u.it.row_off + w.row0 + (has_row[j] ? i : 0)];  // padding lanes: the unit's first row, unused
  }
  stage_table<BS, 64 * NW>(a, u, tid, tab);

  // Query operands and row horizons of this wave's tiles. A padding lane
  // (past the slice's rows) computes on the unit's first row with no causal
  // limit and is never stored; loading it like the others keeps the query
  // loads free of branches, whose merges would wait for them here.
  bf16x8 qop[RTW][4];
  int hz[RTW];
#pragma unroll
  for (int j = 0; j < RTW; ++j) {
    hz[j] = has_row[j] ? rdesc[j].horizon + u.it.grow : INT_MAX;
    const uint4* qp = reinterpret_cast<const uint4*>(qg + static_cast<size_t>(rdesc[j].qidx) * D);
#pragma unroll
    for (int s = 0; s < 4; ++s) qop[j][s] = as_bf16x8(qp[4 * s + g]);
  }
  int hmin = INT_MAX;
#pragma unroll
  for (int j = 0; j < RTW; ++j) hmin = min(hmin, hz[j]);
  hmin = __builtin_amdgcn_readfirstlane(wave_min_int(hmin));
  int nown = 0;  // tiles this wave owns: the first `nown` of its RTW slots
#pragma unroll
  for (int j = 0; j < RTW; ++j) nown += own[j] ? 1 : 0;

  float m[RTW], l[RTW];
  f32x4 o[RTW][8];
#pragma unroll
  for (int j = 0; j < RTW; ++j) {
    m[j] = kNegInf;
    l[j] = 0.0f;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) o[j][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  StageLoader<BS, NW, false> ld;
  ld.init(a, u, wave, lane, tab);
  barrier_lds();  // the table is in LDS; the query loads may still be in flight

  // Per-lane LDS byte addresses of the MFMA operands inside ring slot 0:
  //   K operand (half hh, k-step s): token t = 8*(r16/4) + 4*hh + r16%4,
  //     chunk t*16 + ((4s + g) ^ k_swz(t)). The second half's token is the
  //     first half's plus 4 with the same swizzle, so its addresses are the
  //     first half's plus 1024 bytes.
  //   V operand (channel tile dt): the chunk of channel 16*dt + r16, tokens
  //     8g .. 8g + 7: a per-lane base plus a fixed stride per dt.
  uint32_t kaddr[4];
  const uint32_t smem_base = lds_addr(&smem[0][0]);
  {
    const int t = 8 * (r16 >> 2) + (r16 & 3);
#pragma unroll
    for (int s = 0; s < 4; ++s) kaddr[s] = smem_base + 16u * (t * 16 + ((4 * s + g) ^ k_swz<false>(t)));
  }
  const uint32_t vaddr = smem_base + 16u * (BS == 16 ? 512 + 256 * (g >> 1) + 2 * r16 + (g & 1)
                                                     : 512 + 4 * r16 + (g ^ v_swz<32, false>(r16)));
  const float c = a.scale_log2, masked = masked_score(c);
  auto read_k = [&](u32x4 (&kr)[8], int st) __attribute__((always_inline)) {
    const uint32_t soff = static_cast<uint32_t>(st % kRing) * (kStageChunks * 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) kr[i] = lds_read_b128(kaddr[i] + soff);
#pragma unroll
    for (int i = 0; i < 4; ++i) kr[4 + i] = lds_read_b128<1024>(kaddr[i] + soff);
  };
  auto read_v = [&](u32x4 (&vr)[8], int st) __attribute__((always_inline)) {
    const uint32_t va = vaddr + static_cast<uint32_t>(st % kRing) * (kStageChunks * 16);
    constexpr int kDt = BS == 16 ? 512 : 1024;  // bytes between channel tiles
    vr[0] = lds_read_b128<0 * kDt>(va);
    vr[1] = lds_read_b128<1 * kDt>(va);
    vr[2] = lds_read_b128<2 * kDt>(va);
    vr[3] = lds_read_b128<3 * kDt>(va);
    vr[4] = lds_read_b128<4 * kDt>(va);
    vr[5] = lds_read_b128<5 * kDt>(va);
    vr[6] = lds_read_b128<6 * kDt>(va);
    vr[7] = lds_read_b128<7 * kDt>(va);
  };
  // Stages with positions outside the range or past a row's horizon (first
  // and last stages of a unit, causal rows): all but [inner_lo, inner_lo +
  // inner_n).
  const int inner_lo = tb0 < w.tok_lo ? 1 : 0;
  const int inner_n = max(0, (min(tok_hi, hmin < INT_MAX ? hmin + 1 : INT_MAX) - tb0) / kTileTokens - inner_lo);
  // One stage for NT owned tiles. Two workgroups per compute unit: the other
  // workgroup's waves fill the matrix cores; all scores first, then all
  // softmaxes, then the P.V products.
  auto stage = [&](auto nt_c, int st) __attribute__((always_inline)) {
    constexpr int NT = decltype(nt_c)::value;
    const int tb = tb0 + st * kTileTokens;
    const bool edge = static_cast<uint32_t>(st - inner_lo) >= static_cast<uint32_t>(inner_n);
    u32x4 kr[8], vr[8];
    read_k(kr, st);
    lds_wait<0>(kr);
    f32x4 sc[NT][2];
#pragma unroll
    for (int j = 0; j < NT; ++j) sc[j][0] = sc[j][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          sc[j][hh] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[4 * hh + s]),
                                                               qop[j][s], sc[j][hh], 0, 0, 0);
    read_v(vr, st);
    Probs<8> pop[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      float sv[8], ps = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) sv[e] = sc[j][e >> 2][e & 3];
      if (edge) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int tk = tb + 8 * g + e;
          if (tk < w.tok_lo || tk >= tok_hi || tk > hz[j]) sv[e] = masked;
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float pv = exp2_fast(__builtin_fmaf(sv[e], c, -m[j]));
        ps += pv;
        pop[j].set(e, pv);
      }
      if (__ballot(!(ps <= kRescaleSum)) != 0) rescale<16>(sv, c, m[j], l[j], o[j], ps, pop[j]);
      l[j] += ps;
    }
    lds_wait<0>(vr);
    // Positions past the range may hold anything: zero their V (0 * NaN
    // would poison the accumulator).
    if (tb + kTileTokens > tok_hi) {
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) {
        const uint4 z = zero_past(make_uint4(vr[dt][0], vr[dt][1], vr[dt][2], vr[dt][3]), tb + 8 * g, tok_hi);
        vr[dt] = u32x4{z.x, z.y, z.z, z.w};
      }
    }
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
      for (int j = 0; j < NT; ++j)
        o[j][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vr[dt]), pop[j].operand(),
                                                           o[j][dt], 0, 0, 0);
  };

  // Prologue: the first kAhead = kRing - 2 stages in flight. The query rows,
  // loaded before them, complete first (vector loads complete in order):
  // this wait leaves only the prologue's loads in flight, and no wait for the
  // query rows lands inside the loop.
  constexpr int kAhead = kRing - kPer;
#pragma unroll
  for (int st = 0; st < kAhead; ++st) {
    if (st < nstage) {
      uint32_t ent = ld.entry(st);
      tab_wait(ent);
      ld.issue(ent, smem[st]);
    }
  }
  wait_stage<16 / NW>(min(kAhead, nstage));

  // The ring loop, specialised on the number of tiles this wave owns so that
  // no branch on it sits inside the loop. Every wave runs the same barriers.
  auto run = [&](auto nt_c) __attribute__((always_inline)) {
    constexpr int NT = decltype(nt_c)::value;
    // Every kPer stages: wait for this wave's loads of the next kPer stages
    // (the stages issued after them, at most kAhead - kPer, may stay in
    // flight), one barrier that makes them visible to all waves and frees
    // the slots of the previous kPer stages, and the loads of kPer more
    // stages into those slots. The table entries of the stages a barrier
    // issues are read one barrier ahead: the operand waits of the compute in
    // between cover their latency.
    uint32_t ent[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) ent[q] = ld.entry(kAhead + q);
    for (int st = 0; st < nstage; st += kPer) {
      wait_stage<16 / NW>(max(0, min(kAhead - kPer, nstage - kPer - st)));
      barrier_nofence();
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        tab_wait(ent[q]);  // also past the end: the register is read into again below
        if (st + kAhead + q < nstage) ld.issue(ent[q], smem[(st + kAhead + q) % kRing]);
      }
#pragma unroll
      for (int q = 0; q < kPer; ++q) ent[q] = ld.entry(st + kRing + q);
      if constexpr (NT > 0) {
        stage(nt_c, st);
        if (st + 1 < nstage) stage(nt_c, st + 1);
      }
    }
    wait_vmcnt<0>();
    // Table entries read one barrier ahead may still be in flight: wait for
    // them with their registers as operands, so that no later value is placed
    // in those registers before the reads have written them (the reads are
    // inline assembly, invisible to the compiler's wait tracking).
    tab_wait_all(ent);
    // Every wave has read this unit's take (the ring loop's barriers follow
    // it): take the next unit now.
    int nxt = 0;
    if (tid == 0) nxt = atomicAdd(a.cursors + list * kCursorStride, 1);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      float lt = l[j] + __shfl_xor(l[j], 16);
      lt += __shfl_xor(lt, 32);
      const int i = (cw + NW * j) * 16 + r16;
      if (i < w.nrows) {
        const size_t pr = static_cast<size_t>(a.part_slot[w.partial + i]);
        if (g == 0) {
          a.part_ml[2 * pr] = m[j];
          a.part_ml[2 * pr + 1] = lt;
        }
        // bf16, in register order: the lane's 32 channels 16*dt + 4*g + i
        // (dt = 0..7, i = 0..3) at row positions 32*g + 4*dt + i, four
        // 16-byte stores.
        u32x4* dst = reinterpret_cast<u32x4*>(static_cast<__bf16*>(a.part_o) + pr * D + 32 * g);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          bf16x8 h;
#pragma unroll
          for (int e = 0; e < 8; ++e) h[e] = static_cast<__bf16>(o[j][2 * q + (e >> 2)][e & 3]);
          dst[q] = __builtin_bit_cast(u32x4, h);
        }
      }
    }
    if (tid == 0) next_unit = nxt;
  };
  if (RTW >= 2 && nown == 2) run(std::integral_constant<int, (RTW >= 2 ? 2 : 1)>{});
  else if (nown == 1) run(std::integral_constant<int, 1>{});
  else run(std::integral_constant<int, 0>{});
  // The next take's barrier is reached by every wave only after its last
  // reads of this unit's ring slots, table and next_unit.
  }
  argmax_tail<64 * NW>(a, tid, next_unit);
}

// --------------------------------------------------------------------------
// The wide kernel: one workgroup of 8 waves per compute unit, one 32-row tile
// per wave (waves w and w + 4 share a SIMD). The matrix cores bound a stage
// at 512 cycles per tile (16 32x32x16 products of 32 cycles), as long as the
// SIMD's two instruction streams keep them fed: a product of this shape is
// one issue for the work of two 16x16x32 ones and runs long enough for its
// share of the softmax to issue beside it.
//
// Per stage (r32 = lane % 32, g = lane / 32):
//   S^T = K Q^T: A-row r32 is tile token 16*(r32/16) + 8*(r32/4%2) +
//   4*(r32/8%2) + r32%4, so the lane receives scores of query row r32 for
//   tokens 16h + 8g + j (element 8h + j); the contraction slot of channel d is
//   (k-step d/16, lane group d/8%2, element d%8) on both operands.
//   O^T += V^T P^T: A = V^T (channel 32*ct + r32, tokens 16h + 8g .. + 7),
//   B = the lane's own probabilities 8h .. 8h + 7; the accumulator holds query
//   row r32 at channels 32*ct + 8*b + 4*g + q (element 4b + q).
//
// Stages run through a software pipeline: beside the softmax of stage s, the
// P.V products of stage s - 1 and the scores of stage s + 1 are issued, one
// product and 3-4 vector instructions at a time. Stage s reads the K of stage
// s + 1 (kr is free: the scores of stage s are taken) and its own V behind the
// P.V products of stage s - 1, one read beside each product: eight reads in a
// burst held every wave for several hundred cycles. All have arrived when the
// stage ends, so no LDS read is in flight across the loop's back edge (a value
// that crossed it while its read is in flight could be copied before it
// arrives).
// Even stages publish the next two, and the loads into the slots this frees
// are spread over the products up to the next publish.
//
// Measured on batches that the plan sends here (64 query heads on 8 KV heads, us,
// in turn), against the narrow kernel with 8 waves: 32 sessions of 32,000 tokens,
// 24 drafts 1,020 against 1,059, a 30-row probe prefill 1,087 against 1,156 (see
// kWideStages in plan.cpp). Against the loop before both (16-row tiles whose
// operands were read in bursts, a 64-bit address per lane): 8 sessions of 32,000
// tokens, 28 drafts 278 against 328, the prefill 287 against 340.
// The chip runs these steps at its power limit and lowers the clock as the cycles
// get denser: when the K = 50 verify batch ran here its cycles fell from 1.22 to
// 0.99 million per launch, but the clock from 2.19 to 1.97 GHz.
// The stage's variants for the ends of a unit do not fit 256 registers beside the
// loop's: the compiler spills 45 of them (120 bytes of scratch per lane), outside
// the loop of FAST pairs.
// --------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <int BS>
__global__ void __launch_bounds__(512, 1) attn_bf16_wide(AttnArgs a) {
  constexpr int D = 128;
  constexpr int NW = 8;
  constexpr int kRing = 8;
  constexpr int kAhead = kRing - kPer;  // stages loaded ahead of a pair's first
  constexpr int kLoads = 16 / NW;
  static_assert(BS == 16 || BS == 32, "unsupported block size");
  __shared__ __align__(256) uint4 smem[kRing][kStageChunks];
  __shared__ __align__(16) int tab[kUnitBlocks];
  __shared__ int next_unit;
  const int tid = threadIdx.x;
  const int list = static_cast<int>(blockIdx.x) % a.n_lists;
  const int list0 = load_int_uniform(a.wg_off + list), list_len = load_int_uniform(a.wg_off + list + 1) - list0;
  // Thread 0 takes each unit before the workgroup needs it (see attn_bf16).
  if (tid == 0) next_unit = atomicAdd(a.cursors + list * kCursorStride, 1);
  for (;;) {
  barrier_lds();
  const int taken = __builtin_amdgcn_readfirstlane(next_unit);
  if (taken < 0 || taken >= list_len) break;
  const WaveDesc w = load_wave_desc(a.waves + list0 + taken);
  const UnitStart u = unit_start<BS>(a, w);
  const int tok_hi = u.tok_hi, tb0 = u.tb0, nstage = u.nstage;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, r32 = lane & 31, g = lane >> 5;
  const int row = wave * 32 + r32;  // of the unit's slice
  const bool owns = wave * 32 < w.nrows;
  const RowDesc rdesc = a.rows[u.it.row_off + w.row0 + (row < w.nrows ? row : 0)];  // padding lanes: the unit's first row
  stage_table<BS, 64 * NW>(a, u, tid, tab);
  const int hz = row < w.nrows ? rdesc.horizon + u.it.grow : INT_MAX;
  bf16x8 qop[8];
  {
    const uint4* qp = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.q) +
                                                     static_cast<size_t>(rdesc.qidx) * D);
#pragma unroll
    for (int s = 0; s < 8; ++s) qop[s] = as_bf16x8(qp[2 * s + g]);
  }
  const int hmin = __builtin_amdgcn_readfirstlane(wave_min_int(hz));

  float m = kNegInf, l = 0.0f;
  f32x16 o[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[ct][e] = 0.0f;

  StageLoader<BS, NW, true> ld;
  ld.init(a, u, wave, lane, tab);
  barrier_lds();  // the table is in LDS; the query loads may still be in flight

  // Per-lane LDS byte addresses of the operands inside ring slot 0: K (k-step
  // s): chunk t*16 + ((2s + g) ^ k_swz(t)) of the lane's token t, s + 4 the
  // address of s with bit 7 inverted; V (channel tile ct, token half h): a base
  // per lane (32-token blocks: per half, as the swizzle mixes the halves) plus
  // fixed strides.
  const uint32_t smem_base = lds_addr(&smem[0][0]);
  uint32_t kaddr[4], vaddr[2];
  {
    const int t = 16 * (r32 >> 4) + 8 * ((r32 >> 2) & 1) + 4 * ((r32 >> 3) & 1) + (r32 & 3);
#pragma unroll
    for (int s = 0; s < 4; ++s) kaddr[s] = smem_base + 16u * (t * 16 + ((2 * s + g) ^ k_swz<true>(t)));
#pragma unroll
    for (int h = 0; h < 2; ++h)
      vaddr[h] = smem_base + 16u * (BS == 16 ? 512 + 256 * h + 2 * r32 + (g ^ v_swz<16, true>(r32))
                                             : 512 + 4 * r32 + ((2 * h + g) ^ v_swz<32, true>(r32)));
  }
  const float c = a.scale_log2, masked = masked_score(c);
  auto slot_off = [&](int st) __attribute__((always_inline)) {
    return static_cast<uint32_t>(st % kRing) * (kStageChunks * 16);
  };
  auto read_k = [&](u32x4 (&kr)[8], int s, uint32_t soff) __attribute__((always_inline)) {
    kr[s] = lds_read_b128(s < 4 ? kaddr[s] + soff : (kaddr[s - 4] + soff) ^ 128u);
  };
  auto read_v = [&](u32x4 (&vr)[8], int i, uint32_t soff) __attribute__((always_inline)) {  // vr[4h + ct]
    constexpr int kCt = BS == 16 ? 1024 : 2048;  // bytes between channel tiles; 16-token blocks: h 4 KB apart
    const uint32_t va = vaddr[BS == 16 ? 0 : i >> 2] + soff;
    const int step = BS == 16 ? i : i & 3;
    vr[i] = step == 0   ? lds_read_b128<0 * kCt>(va)
            : step == 1 ? lds_read_b128<1 * kCt>(va)
            : step == 2 ? lds_read_b128<2 * kCt>(va)
            : step == 3 ? lds_read_b128<3 * kCt>(va)
            : step == 4 ? lds_read_b128<4 * kCt>(va)
            : step == 5 ? lds_read_b128<5 * kCt>(va)
            : step == 6 ? lds_read_b128<6 * kCt>(va)
                        : lds_read_b128<7 * kCt>(va);
  };
  // Stages with positions outside the range or past a row's horizon: all but
  // [inner_lo, inner_lo + inner_n).
  const int inner_lo = tb0 < w.tok_lo ? 1 : 0;
  const int inner_n = max(0, (min(tok_hi, hmin < INT_MAX ? hmin + 1 : INT_MAX) - tb0) / kTileTokens - inner_lo);

  struct State {
    f32x16 sc;      // scores of the stage
    Probs<16> pop;  // probabilities of the stage before
    u32x4 vr[8];    // V of the stage before
  };
  auto score_product = [&](f32x16& sc, int s, const u32x4 (&kr)[8]) __attribute__((always_inline)) {
    f32x16 acc;
    if (s == 0) {
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
    } else {
      acc = sc;
    }
    sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kr[s]), qop[s], acc, 0, 0, 0);
  };
  auto pv_product = [&](int i, const State& x) __attribute__((always_inline)) {
    o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x.vr[i]), x.pop.operand(i >> 2),
                                                       o[i & 3], 0, 0, 0);
  };
  // The pair of stages a publish makes room for, loaded until the next one;
  // the table entries of the pair after it are read one publish ahead.
  const char* src[kPer] = {nullptr, nullptr};
  int st_load = 0;
  uint32_t ent[kPer];
  auto load = [&](auto fast_c, int i) __attribute__((always_inline)) {
    if (decltype(fast_c)::value || st_load + i / kLoads < nstage)
      ld.load(src[i / kLoads], smem[(st_load + i / kLoads) % kRing], i % kLoads);
  };
  // One stage. FAST: no position to mask, every load inside the unit, the
  // steady number of loads in flight. FIRST: no stage before it; LAST: none
  // after it; PUBLISH: stages st + 1 and st + 2 become readable (this wave's
  // loads of them have landed, and the barrier makes every wave's loads
  // visible), stages up to st - 1 are no longer read. LOAD: first of the two
  // loads issued here.
  auto stage = [&](auto owns_c, auto fast_c, auto first_c, auto last_c, auto publish_c, auto load_c, int st, State& x,
                   u32x4 (&kr)[8]) __attribute__((always_inline)) {
    constexpr bool OWNS = decltype(owns_c)::value, FAST = decltype(fast_c)::value, FIRST = decltype(first_c)::value;
    constexpr bool LAST = decltype(last_c)::value, PUBLISH = decltype(publish_c)::value;
    constexpr int LOAD = decltype(load_c)::value;
    if constexpr (PUBLISH) {
      if constexpr (FAST) wait_vmcnt<3 * kLoads>();
      else wait_stage<kLoads>(max(0, min(3, nstage - 3 - st)));
      barrier_nofence();
      st_load = st + kAhead;
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        tab_wait(ent[q]);
        src[q] = ld.base(ent[q]);
      }
#pragma unroll
      for (int q = 0; q < kPer; ++q) ent[q] = ld.entry(st_load + kPer + q);
      // Near a unit's ends registers are short: no read may be in flight
      // where the compiler could spill its register.
      if constexpr (!FAST) tab_wait_all(ent);
    }
    if constexpr (!OWNS) {
      if constexpr (LOAD >= 0) {
        load(fast_c, LOAD);
        load(fast_c, LOAD + 1);
      }
    } else {
      // The softmax in 16 slots of one product each: slots 0-7 the P.V of the
      // stage before, 8-15 the scores of the stage after. The steps of an
      // element (scale, exponential, sum, conversion) follow each other one
      // or more slots apart so that none waits for the last.
      float sv[16], ex[16], pv[16], ps = 0.0f;
      Probs<16> pop;
#pragma unroll
      for (int e = 0; e < 16; ++e) sv[e] = x.sc[e];
      if (!FAST && static_cast<uint32_t>(st - inner_lo) >= static_cast<uint32_t>(inner_n)) {
        // the visible positions, counted from the lane's first
        const int at = tb0 + st * kTileTokens + 8 * g, lo = w.tok_lo - at, hi = min(tok_hi - 1, hz) - at;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int pos = 16 * (e >> 3) + (e & 7);
          sv[e] = pos < lo || pos > hi ? masked : sv[e];
        }
      }
      const float nm = -m;
      const uint32_t k_off = slot_off(st + 1), v_off = slot_off(st);
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        if (!FIRST && t < 8) pv_product(t, x);
        if (!LAST && t >= 8) {
          // K operand s = t - 8, read in slot s: wait for all LDS reads but
          // those issued after it, K s + 1 .. 7 and V max(0, s - 4) ..
          // min(7, s + 3).
          constexpr int kAfter[8] = {11, 11, 11, 11, 11, 9, 7, 5};
          lds_wait_one(kr[t - 8], kAfter[t - 8]);
          score_product(x.sc, t - 8, kr);
        }
        if (!LAST && t < 8) read_k(kr, t, k_off);
        if (t >= 4 && t < 12) read_v(x.vr, t - 4, v_off);
        if (LOAD >= 0 && t % 8 == 4) load(fast_c, LOAD + t / 8);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          if (t == 3 * e / 4) ex[e] = __builtin_fmaf(sv[e], c, nm);
          if (t == 3 * e / 4 + 1) pv[e] = exp2_fast(ex[e]);
          if (t == 3 * e / 4 + 3) ps += pv[e];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if (t == 3 * (2 * i + 1) / 4 + 3) {
            pop.w[i] = pack_bf16(pv[2 * i], pv[2 * i + 1]);
            asm volatile("" : "+v"(pop.w[i]));  // here, not behind the branch below
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (__builtin_expect(__ballot(!(ps <= kRescaleSum)) != 0, 0)) rescale<32>(sv, c, m, l, o, ps, pop);
      l += ps;
      x.pop = pop;
      lds_wait<0>(x.vr);
      if constexpr (LAST) {
        // Positions past the range may hold anything: zero their V (0 * NaN
        // would poison the accumulator).
        const int tb = tb0 + st * kTileTokens;
        if (tb + kTileTokens > tok_hi) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const uint4 z = zero_past(make_uint4(x.vr[i][0], x.vr[i][1], x.vr[i][2], x.vr[i][3]),
                                      tb + 16 * (i >> 2) + 8 * g, tok_hi);
            x.vr[i] = u32x4{z.x, z.y, z.z, z.w};
          }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) pv_product(i, x);
      }
    }
  };

  // Prologue: the ring's first stages in flight. The compiler waits for every
  // load in flight where the queries are first used: four stages are issued
  // before that point and two behind it.
  auto prologue = [&](auto lo_c, auto hi_c) __attribute__((always_inline)) {
    constexpr int LO = decltype(lo_c)::value, N = decltype(hi_c)::value - LO;
    uint32_t e0[N];
#pragma unroll
    for (int i = 0; i < N; ++i) e0[i] = ld.entry(LO + i);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      tab_wait(e0[i]);
      if (LO + i < nstage) ld.issue(e0[i], smem[LO + i]);
    }
  };
  prologue(std::integral_constant<int, 0>{}, std::integral_constant<int, 4>{});
#pragma unroll
  for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(qop[s]));
  prologue(std::integral_constant<int, 4>{}, std::integral_constant<int, kAhead>{});

  // Every wave runs the same barriers, whether it owns a tile or not.
  auto run = [&](auto owns_c) __attribute__((always_inline)) {
    constexpr bool OWNS = decltype(owns_c)::value;
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    constexpr std::integral_constant<int, -1> none{};
    constexpr std::integral_constant<int, 0> load0{};
    constexpr std::integral_constant<int, 2> load2{};
#pragma unroll
    for (int q = 0; q < kPer; ++q) ent[q] = ld.entry(kAhead + q);
    tab_wait_all(ent);
    State x;
    u32x4 kr[8];
    wait_stage<kLoads>(min(kAhead, nstage) - 1);
    barrier_nofence();  // stage 0 is readable
    if constexpr (OWNS) {
#pragma unroll
      for (int s = 0; s < 8; ++s) read_k(kr, s, 0);
      lds_wait<0>(kr);
#pragma unroll
      for (int s = 0; s < 8; ++s) score_product(x.sc, s, kr);
    }
    if (nstage == 1) {
      stage(owns_c, no, yes, yes, no, none, 0, x, kr);
    } else {
      stage(owns_c, no, yes, no, yes, load0, 0, x, kr);
      int st = 0;  // the last stage done
      auto pair = [&](auto fast_c) __attribute__((always_inline)) {
        stage(owns_c, fast_c, no, no, no, load2, st + 1, x, kr);
        stage(owns_c, fast_c, no, no, yes, load0, st + 2, x, kr);
        st += 2;
      };
      // The bulk of a unit runs pairs without branches for its ends.
      const int fast_end = min(inner_lo + inner_n - 2, nstage - kRing);
      while (st < fast_end) pair(yes);
      while (st + 3 < nstage) pair(no);
      // One or two stages are left, all loaded: the last publish, in stage st,
      // made room for stages st + 6 and st + 7.
      if (st + 2 < nstage) {
        stage(owns_c, no, no, no, no, none, st + 1, x, kr);
        ++st;
      }
      stage(owns_c, no, no, yes, no, none, st + 1, x, kr);
    }
    wait_vmcnt<0>();
    tab_wait_all(ent);  // read ahead, maybe still in flight (see attn_bf16)
    // Every wave has read this unit's take: take the next unit now.
    int nxt = 0;
    if (tid == 0) nxt = atomicAdd(a.cursors + list * kCursorStride, 1);
    if constexpr (OWNS) {
      const float lt = l + __shfl_xor(l, 32);
      if (row < w.nrows) {
        const size_t pr = static_cast<size_t>(a.part_slot[w.partial + row]);
        if (g == 0) {
          a.part_ml[2 * pr] = m;
          a.part_ml[2 * pr + 1] = lt;
        }
        // The row layout of attn_bf16 (channel 16*dt + 4*g' + q at position
        // 32*g' + 4*dt + q): element 4b + q of channel tile ct is channel
        // 32*ct + 8*b + 4*g + q, so g' = 2*(b % 2) + g and dt = 2*ct + b / 2;
        // the elements of even and of odd b are 32 positions in a row each.
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          u32x4* dst = reinterpret_cast<u32x4*>(static_cast<__bf16*>(a.part_o) + pr * D + 32 * (2 * b + g));
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) {
            const f32x16& v = o[ct];
            dst[ct] = u32x4{pack_bf16(v[4 * b], v[4 * b + 1]), pack_bf16(v[4 * b + 2], v[4 * b + 3]),
                            pack_bf16(v[4 * b + 8], v[4 * b + 9]), pack_bf16(v[4 * b + 10], v[4 * b + 11])};
          }
        }
      }
    }
    if (tid == 0) next_unit = nxt;
  };
  if (owns) run(std::true_type{});
  else run(std::false_type{});
  }
  argmax_tail<64 * NW>(a, tid, next_unit);
}

// --------------------------------------------------------------------------
// fp32 partial attention (full-precision v_mfma_f32_16x16x4_f32).
//   Scores: half hh of the tile has A-row r16 = token tb + 16*hh + r16, and the
//   contraction slot of channel d is (k-step d/4, lane group d%4); the lane
//   receives query row r16 for tokens tb + 16*hh + 4g + i.
//   P.V: one MFMA per (hh, i) over the 4 tokens tb + 16*hh + 4g' + i
//   (g' = 0..3): A = V^T (channel 16*dt + r16, the lane's token), B = the
//   lane's own probability. Accumulator layout as in the bf16 kernel.
// --------------------------------------------------------------------------
template <int RT, int D, int BS>
__global__ void __launch_bounds__(64) attn_f32(AttnArgs a) {
  static_assert(D % 16 == 0 && (BS == 16 || BS == 32 || BS == 64), "unsupported shape");
  constexpr int KS = D / 4;
  constexpr int DT = D / 16;
  if (static_cast<int>(blockIdx.x) >= a.grid) {  // a verify step's argmax, beside the attention
    verify_argmax_unit<64>(a.acc, blockIdx.x - a.grid);
    return;
  }
  const WaveDesc w = a.waves[blockIdx.x];
  if (w.item < 0) return;
  const ItemDesc it = a.items[w.item];
  const int lane = threadIdx.x, r16 = lane & 15, g = lane >> 4;
  const float* __restrict__ qg = static_cast<const float*>(a.q);
  const float* __restrict__ kc = static_cast<const float*>(a.k_cache);
  const float* __restrict__ vc = static_cast<const float*>(a.v_cache);
  const int32_t* __restrict__ table = a.tables + it.table_off;
  const int grow = it.grow;  // tokens appended since the plan (see the bf16 kernel)
  const int tok_hi = w.tok_hi == it.hi ? w.tok_hi + grow : w.tok_hi;
  const int nb = grow != 0 ? (it.hi + grow + BS - 1) / BS : it.n_blocks;
  const size_t head = static_cast<size_t>(it.kv_head);
  const size_t hkv = static_cast<size_t>(a.hkv);
  const int ntiles = (w.nrows + 15) >> 4;

  float qop[RT][KS];
  int hz[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int i = t * 16 + r16;
    if (i < w.nrows) {
      const RowDesc rd = a.rows[it.row_off + w.row0 + i];
      hz[t] = rd.horizon + grow;
      const float* qp = qg + static_cast<size_t>(rd.qidx) * D;
#pragma unroll
      for (int s = 0; s < KS; ++s) qop[t][s] = qp[4 * s + g];
    } else {
      hz[t] = INT_MAX;
#pragma unroll
      for (int s = 0; s < KS; ++s) qop[t][s] = 0.0f;
    }
  }
  int hmin = INT_MAX;
#pragma unroll
  for (int t = 0; t < RT; ++t) hmin = min(hmin, hz[t]);
  hmin = wave_min_int(hmin);

  float m[RT], l[RT];
  f32x4 o[RT][DT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    m[t] = kNegInf;
    l[t] = 0.0f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[t][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  auto blk = [&](int tb, int j) {
    int bi = tb / BS + j;
    bi = bi < nb ? bi : nb - 1;
    return static_cast<size_t>(table[bi]);
  };

  const float c = a.scale_log2;
  for (int tb = w.tok_lo & ~(kTileTokens - 1); tb < tok_hi; tb += kTileTokens) {
    const size_t b0 = blk(tb, 0);
    const size_t b1 = BS == 16 ? blk(tb, 1) : b0;
    float kop[2][KS];
    f32x4 vop[2][DT];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const size_t b = (BS == 16 && hh == 1) ? b1 : b0;
      const int offk = (tb + 16 * hh + r16) % BS;
      const float* kp = kc + ((b * hkv + head) * BS + offk) * D;
#pragma unroll
      for (int s = 0; s < KS; ++s) kop[hh][s] = kp[4 * s + g];
      const int offv = (tb + 16 * hh + 4 * g) % BS;
      const float* vp = vc + (b * hkv + head) * (static_cast<size_t>(D) * BS) + offv;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        f32x4 v = *reinterpret_cast<const f32x4*>(vp + static_cast<size_t>(16 * dt + r16) * BS);
        if (tb + kTileTokens > tok_hi) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (tb + 16 * hh + 4 * g + i >= tok_hi) v[i] = 0.0f;
        }
        vop[hh][dt] = v;
      }
    }
    const bool edge = tb < w.tok_lo || tb + kTileTokens > tok_hi || tb + kTileTokens - 1 > hmin;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      if (t < ntiles) {
        f32x4 sc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
          for (int s = 0; s < KS; ++s)
            sc[hh] = __builtin_amdgcn_mfma_f32_16x16x4f32(kop[hh][s], qop[t][s], sc[hh], 0, 0, 0);
        float sv[8];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
          for (int i = 0; i < 4; ++i) sv[4 * hh + i] = sc[hh][i] * c;
        if (edge) {
#pragma unroll
          for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int tk = tb + 16 * hh + 4 * g + i;
              if (tk < w.tok_lo || tk >= tok_hi || tk > hz[t]) sv[4 * hh + i] = kNegInf;
            }
        }
        const float alpha = softmax_step(sv, m[t], l[t]);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          o[t][dt] *= alpha;
#pragma unroll
          for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              o[t][dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(vop[hh][dt][i], sv[4 * hh + i], o[t][dt], 0, 0, 0);
        }
      }
    }
  }

#pragma unroll
  for (int t = 0; t < RT; ++t) {
    if (t < ntiles) {
      float lt = l[t] + __shfl_xor(l[t], 16);
      lt += __shfl_xor(lt, 32);
      const int i = t * 16 + r16;
      if (i < w.nrows) {
        const size_t pr = static_cast<size_t>(a.part_slot[w.partial + i]);
        if (g == 0) {
          a.part_ml[2 * pr] = m[t];
          a.part_ml[2 * pr + 1] = lt;
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          *reinterpret_cast<f32x4*>(static_cast<float*>(a.part_o) + pr * D + 16 * dt + 4 * g) = o[t][dt];
      }
    }
  }
}

// --------------------------------------------------------------------------
// Log-sum-exp merge: one wave per output (query row x query head).
//   M = max m_i, L = sum 2^(m_i - M) l_i, O = sum 2^(m_i - M) o_i / L,
//   lse = (M + log2 L) ln 2. Partials with nothing visible (m = -inf, l = 0)
//   add nothing.
// Partials go in batches of 4 (outputs with at most 4) or 8. An output's
// partials are consecutive rows; lane i loads the (m, l) pair of partial i
// and every lane its channels of all the batch's rows, in one round trip.
// The batch maximum and the weighted sum of l are DPP reductions over lanes
// 0-7; unused slots repeat a valid row with weight 0. Batches after the
// first rescale the running sums to the new maximum.
// --------------------------------------------------------------------------
// Partial rows are in the input dtype: fp32 rows in channel order, bf16 rows
// (D = 128) in the bf16 attention writer's register order, channel
// 16*dt + 4*g + i at position 32*g + 4*dt + i. Lane `lane` reads positions
// PER*lane .. PER*lane + PER - 1 of every partial row (one coalesced pass
// over the row) and merges the channels stored there: channel PER*lane + e
// (fp32), or, for bf16, the pair merge_channel() + e (g = lane / 16,
// dt = lane / 2 mod 8, i = 2 * (lane mod 2) and i + 1).
template <int D, typename PT>
__device__ __forceinline__ int merge_channel(int lane) {
  if constexpr (std::is_same<PT, float>::value) {
    return lane * (D / 64);
  } else {
    static_assert(D == 128, "bf16 partial rows are 128 channels");
    return 16 * ((lane >> 1) & 7) + 4 * (lane >> 4) + 2 * (lane & 1);
  }
}

template <int D, typename PT>
__device__ __forceinline__ void load_partial(const AttnArgs& a, size_t row, int lane, float (&po)[D / 64]) {
  constexpr int PER = D / 64;
  if constexpr (std::is_same<PT, float>::value) {
    const float* src = static_cast<const float*>(a.part_o) + row * D + lane * PER;
#pragma unroll
    for (int e = 0; e < PER; ++e) po[e] = src[e];
  } else {
    const uint32_t w = reinterpret_cast<const uint32_t*>(static_cast<const __bf16*>(a.part_o) + row * D)[lane];
    po[0] = __uint_as_float(w << 16);
    po[1] = __uint_as_float(w & 0xFFFF0000u);
  }
}

// One batch of at most B partials (entries c0 .. c0 + k - 1 of the output's
// list), folded into the running (max, sum, accumulator).
template <int B, int D, typename PT>
__device__ __forceinline__ void merge_batch(const AttnArgs& a, int c0, int k, bool first, int lane, float& run_max,
                                            float& mu, float& sum, float (&acc)[D / 64]) {
  constexpr int PER = D / 64;
  // the output's partials are consecutive: rows c0 .. c0 + k - 1
  const float2 ml = reinterpret_cast<const float2*>(a.part_ml)[c0 + min(lane, k - 1)];
  float po[B][PER];
#pragma unroll
  for (int i = 0; i < B; ++i) load_partial<D, PT>(a, static_cast<size_t>(c0 + min(i, k - 1)), lane, po[i]);
  const bool live = lane < k;
  const float pm = live ? ml.x : kNegInf;
  const float pl = live ? ml.y : 0.0f;
  const float bm = lanes8_max(pm);  // lanes k.. hold -inf
  const float new_max = fmaxf(run_max, bm);
  const float new_mu = new_max == kNegInf ? 0.0f : new_max;
  if (!first) {
    const float alpha = exp2_fast(mu - new_mu);
    sum *= alpha;
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] *= alpha;
  }
  run_max = new_max;
  mu = new_mu;
  const float w = exp2_fast(pm - mu);  // lane i: weight of partial i, 0 for unused slots (pm = -inf)
  sum += lanes8_sum(w * pl);
#pragma unroll
  for (int i = 0; i < B; ++i) {
    const float wgt = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), i));
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] += wgt * po[i][e];
  }
}

template <int D, typename OutT>
__global__ void __launch_bounds__(256) merge_kernel(AttnArgs a) {
  constexpr int PER = D / 64;
  // The attention launch is done with its cursors: return them to zero for
  // the workspace's next call.
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < a.n_cursors; i += 256) a.cursors[i * kCursorStride] = 0;
  const int merge_blocks = (a.n_out + 3) / 4;
  if (static_cast<int>(blockIdx.x) >= merge_blocks) {
    // fused accept: one verify thread per wave
    const int sv = (blockIdx.x - merge_blocks) * 4 + (threadIdx.x >> 6);
    if (sv < a.acc.n_verify) accept_unit(a.acc, sv);
    return;
  }
  const int o = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (o >= a.n_out) return;
  const int beg = a.merge_off[o], end = a.merge_off[o + 1];
  float acc[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) acc[e] = 0.0f;
  float mu = 0.0f, sum = 0.0f, run_max = kNegInf;
  if (end - beg <= 4) {
    merge_batch<4, D, OutT>(a, beg, end - beg, true, lane, run_max, mu, sum, acc);
  } else {
    for (int c0 = beg; c0 < end; c0 += 8)
      merge_batch<8, D, OutT>(a, c0, min(8, end - c0), c0 == beg, lane, run_max, mu, sum, acc);
  }
  const float inv = sum > 0.0f ? 1.0f / sum : 0.0f;
  OutT* out = static_cast<OutT*>(a.out) + static_cast<size_t>(o) * D + merge_channel<D, OutT>(lane);
#pragma unroll
  for (int e = 0; e < PER; ++e) out[e] = static_cast<OutT>(acc[e] * inv);
  if (lane == 0 && a.lse != nullptr)
    a.lse[o] = sum > 0.0f ? (mu + __log2f(sum)) * kLn2 : kNegInf;
}

__global__ void __launch_bounds__(256) counter_reset_kernel(int32_t* counters, int32_t n) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) counters[i] = 0;
}

// --------------------------------------------------------------------------
// Dispatch tables.
// --------------------------------------------------------------------------
typedef void (*AttnKernel)(AttnArgs);

template <int BS, int NW>
AttnKernel pick_bf16(int row_tiles) {
  switch ((row_tiles + NW - 1) / NW) {
    case 1: return attn_bf16<1, BS, NW>;
    case 2: return attn_bf16<2, BS, NW>;
    default: return nullptr;
  }
}

template <int D, int BS>
AttnKernel pick_f32(int rt) {
  switch (rt) {
    case 1: return attn_f32<1, D, BS>;
    case 2: return attn_f32<2, D, BS>;
    case 3: return attn_f32<3, D, BS>;
    case 4: return attn_f32<4, D, BS>;
    default: return nullptr;
  }
}

// Exactly the shapes attention_supported (dispatch_rules.cpp) accepts.
AttnKernel pick_attention(int32_t dtype, int32_t d, int32_t bs, int32_t rt, int32_t waves, bool wide) {
  if (dtype == 1 && d == 128 && (waves == 4 || waves == 8)) {
    if (waves == 8 && wide && rt <= 16) return bs == 16 ? attn_bf16_wide<16> : bs == 32 ? attn_bf16_wide<32> : nullptr;
    if (bs == 16) return waves == 4 ? pick_bf16<16, 4>(rt) : pick_bf16<16, 8>(rt);
    if (bs == 32) return waves == 4 ? pick_bf16<32, 4>(rt) : pick_bf16<32, 8>(rt);
  }
  if (dtype == 0) {
    if (d == 64 && bs == 16) return pick_f32<64, 16>(rt);
    if (d == 64 && bs == 32) return pick_f32<64, 32>(rt);
    if (d == 128 && bs == 16) return pick_f32<128, 16>(rt);
    if (d == 128 && bs == 32) return pick_f32<128, 32>(rt);
  }
  return nullptr;
}

}  // namespace

hipError_t launch_attn_partial(const AttnArgs& a, hipStream_t stream) {
  AttnKernel k = pick_attention(a.dtype, a.head_dim, a.block_size, a.row_tiles, a.wg_waves, a.wide);
  if (k == nullptr) return hipErrorInvalidValue;
  const int threads = a.dtype == 1 ? 64 * a.wg_waves : 64;
  const int grid = a.dtype == 1 ? a.grid : a.grid + a.tail_units;
  if (grid > 0) hipLaunchKernelGGL(k, dim3(grid), dim3(threads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_counter_reset(int32_t* counters, int32_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const int blocks = n / 256 + 1 < 64 ? n / 256 + 1 : 64;
  hipLaunchKernelGGL(counter_reset_kernel, dim3(blocks), dim3(256), 0, stream, counters, n);
  return hipGetLastError();
}

hipError_t launch_merge(const AttnArgs& a, hipStream_t stream) {
  int blocks = (a.n_out + 3) / 4 + (a.acc.n_verify + 3) / 4;
  if (blocks == 0 && a.n_cursors == 0) return hipSuccess;
  if (blocks == 0) blocks = 1;  // only the cursors to clear
  if (a.dtype == 1 && a.head_dim == 128)
    hipLaunchKernelGGL((merge_kernel<128, __bf16>), dim3(blocks), dim3(256), 0, stream, a);
  else if (a.dtype == 0 && a.head_dim == 128)
    hipLaunchKernelGGL((merge_kernel<128, float>), dim3(blocks), dim3(256), 0, stream, a);
  else if (a.dtype == 0 && a.head_dim == 64)
    hipLaunchKernelGGL((merge_kernel<64, float>), dim3(blocks), dim3(256), 0, stream, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace spork
