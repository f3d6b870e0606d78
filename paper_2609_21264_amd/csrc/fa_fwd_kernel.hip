// Fused attention forward for gfx950 (MI355X): one kernel computes, per (batch, query heads, block of
// query rows), O = softmax(scale * Q K^T) V with the online softmax of the paper's per-tile algorithm
// (Alg. 1, Sec. 2.1): key/value rows are streamed in tiles, each query row keeps a reference maximum
// and a running sum, and the unnormalised output accumulator is rescaled when the reference moves.
// Scores and probabilities live only in registers; K and V tiles are staged in LDS.
//
// Mapping onto CDNA4:
//  * A workgroup has NWAVES = 4 wavefronts (one per SIMD) sharing one key/value head; each wave owns
//    32*QB = 64 query rows of one query head: 256 rows of one head, or 128 rows of 2 heads or 64 rows
//    of 4 heads of the same GQA group when the group size allows (long instance, one workgroup per CU,
//    two at d = 64; the short instance has 32-row waves and two workgroups per CU, the key-halves
//    instance two sets of two 32-row waves that split every key tile between them, with two or three
//    workgroups per CU, and the key-quarters instance four waves that share 32 rows).
//  * Scores are computed transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16: the K tile (LDS)
//    is the A operand and the wave's Q rows (AGPRs, loaded once) are the B operand. In the 32x32
//    accumulator a lane then holds ONE query row (column = lane % 32) and 16 keys, so row
//    reductions are in-lane plus one exchange between the two lane halves (v_permlane32_swap).
//  * The A-operand rows of K are loaded in a permuted key order (bits 2 and 3 of the row index
//    swapped), which makes each 8-register group of the accumulator hold 8 consecutive keys. After
//    rounding to bf16, those registers are already the B operand of the second product
//    O^T += V^T P^T, so P never moves between lanes or through LDS.
//  * V^T is the A operand of that product and needs keys contiguous per lane. V tiles stay
//    row-major in LDS and are read with ds_read_b64_tr_b16: within each 16-lane group the
//    instruction gathers a 4 (keys) x 16 (dims) block and hands lane i the 4 keys of dim i.
//  * Three-stage software pipeline: step j runs the score MFMAs of key tile j+1, the exponentials
//    of tile j and the P V MFMAs of tile j-1. The three are independent inside a step, so the
//    softmax arithmetic is spread evenly between the MFMAs and one wave per SIMD keeps the matrix
//    unit fed while it issues VALU work (VALU work from the same wave overlaps a running MFMA).
//  * K/V tiles move HBM -> LDS with buffer loads that write LDS directly (no VGPR staging, no LDS
//    write instructions), in two rings: K tiles (2 slots by default, step j loads K(j+2)) and V
//    tiles (4 slots, step j loads V(j+2)). One wait on the wave's own loads plus one barrier per step
//    publishes the tiles of the step and frees the slots of the previous one. Rows past Sk load as
//    zeros (buffer range check), so partial tiles need no special path.
//  * 16-byte LDS chunks are XOR-swizzled per row (K: by the reading lane's key slot; V: by the key
//    mod 4) so that the lanes the LDS serves in one cycle hit 16 different bank slots. The swizzle
//    is produced by choosing each lane's source offset, since the load writes LDS lane-linearly.
//  * The output accumulators O and the Q operand live in AGPRs for the whole kernel where a SIMD holds
//    one wave (VGPRs otherwise); scores, probabilities and LDS fragments use VGPRs.
//  * Causal masking skips key tiles above the diagonal entirely and applies the element mask only on
//    diagonal and tail tiles.
//  * Workgroup order: heaviest query blocks first when causal, and the workgroups that share a
//    key/value head at one query block are dispatched consecutively onto the same XCD (workgroup IDs
//    are assigned to the 8 XCDs round-robin), so their K/V tiles are served from one L2.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "fa_device.h"
#include "fa_internal.h"

namespace fa {
namespace {

constexpr float kLn2 = 0.69314718055994530942f;
// A tile's exponentials are accepted when every lane's sum of them is at most 2^8: then no
// probability exceeds 2^8 relative to the reference maximum.
constexpr float kOverflowSum = 256.0f;

// Layout of the output tile staged in LDS for coalesced stores: row R of a wave's tile (DV bf16,
// 16-byte chunks) keeps logical chunk c at chunk c ^ o_swizzle(R), with the chunk's two 8-byte
// halves exchanged when o_half(R) = 1. The accumulator layout writes 8 bytes per lane for 32 rows at
// once and the coalesced read takes 8 bytes per lane across consecutive rows; with this layout both
// touch 32 different 8-byte bank slots per cycle.
template <int DV>
__device__ __forceinline__ int o_swizzle(int r) { return DV >= 128 ? (r & 15) : ((r >> 1) & 7); }
template <int DV>
__device__ __forceinline__ int o_half(int r) { return DV >= 128 ? ((r ^ (r >> 4)) & 1) : (((r >> 1) ^ (r >> 4)) & 1); }

// The P V product is issued through inline asm so that its accumulators O stay in AGPRs for the
// whole kernel (the score product uses the builtin; its accumulators are VGPRs). The compiler does
// not model hazards of inline asm, so:
//  * mfma_out starts with s_nop 1: its P operand may have just been written by VALU, which needs
//    2 wait states before an MFMA reads it (mfma_out_settled omits them where P is old);
//  * agpr_fence() separates asm MFMA writes of O from compiler-generated accesses (initialisation,
//    rescale, epilogue) in both directions: 18 wait states cover the MFMA write-to-read distance,
//    and the operand tie keeps the order;
//  * consecutive MFMAs accumulating into exactly the same registers need no wait states.
// AG selects where O and Q live: AGPRs (one wave per SIMD, where the VGPRs alone cannot hold the
// step's scores, probabilities and fragments next to them) or VGPRs (two waves per SIMD: the
// compiler splits a wave's 256 registers evenly between the two files as soon as any AGPR is used,
// which would leave 128 VGPRs for the step; with no AGPR all 256 are VGPRs).
template <bool AG>
__device__ __forceinline__ void mfma_out(f32x16& acc, const bf16x8& v, const bf16x8& pt) {
  if constexpr (AG)
    asm("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(v), "v"(pt));
  else
    asm("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(v), "v"(pt));
}
// Same without the leading wait states, for operands no VALU instruction has written recently: in
// the pipelined step, P was packed a whole step earlier and V comes from LDS.
template <bool AG>
__device__ __forceinline__ void mfma_out_settled(f32x16& acc, const bf16x8& v, const bf16x8& pt) {
  if constexpr (AG)
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(v), "v"(pt));
  else
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(v), "v"(pt));
}
template <bool AG>
__device__ __forceinline__ void agpr_fence(f32x16& acc) {
  if constexpr (AG)
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 3" : "+a"(acc));
  else
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 3" : "+v"(acc));
}
// 16 bytes of Q straight into its register tuple (only read as an MFMA operand, so it never needs a
// copy). The load is not waited for here: the caller waits on vmcnt and then passes the value
// through q_ready(), which keeps every read of it after that wait.
template <bool AG>
__device__ __forceinline__ void load_q(bf16x8& r, const void* ptr) {
  if constexpr (AG)
    asm volatile("global_load_dwordx4 %0, %1, off" : "=a"(r) : "v"(ptr) : "memory");
  else
    asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(r) : "v"(ptr) : "memory");
}
template <bool AG>
__device__ __forceinline__ void q_ready(bf16x8& r) {
  if constexpr (AG)
    asm volatile("" : "+a"(r));
  else
    asm volatile("" : "+v"(r));
}

// Slot of a tile in a ring of N slots of STEP bytes. A ring of 2 or 4 slots takes the low bits of the
// tile index. For 3 slots the remainder would cost a multiply-high chain in front of each step's first
// LDS reads, so the offset is carried from tile to tile instead (next()): one add, compare and select,
// in inline assembly so that they stay scalar: the loads' LDS base (M0) must be a scalar, and a select
// that also feeds vector addresses is selected as a vector instruction. Measured (interleaved, one
// box): H4 777 x 3001 d128 28.5 -> 26.7 us, one head S16384 d128 153.9 -> 145.2 us, B2 28/4 777 x 5001
// 119.5 -> 114.3 us; carrying the power-of-two rings too cost B8 H12 S512 d64 2.5 %, so they are not.
template <int STEP, int N>
struct Ring {
  static constexpr bool kCarried = (N & (N - 1)) != 0;
  int off;  // carried offset
  __device__ __forceinline__ explicit Ring(int tile) : off(tile % N * STEP) {}
  __device__ __forceinline__ void next() {
    if constexpr (kCarried)
      asm("s_add_u32 %0, %0, %1\n\ts_cmp_eq_u32 %0, %2\n\ts_cselect_b32 %0, 0, %0"
          : "+s"(off)
          : "i"(STEP), "i"(STEP * N)
          : "scc");
  }
  // Offset of tile `t`, which is the tile the carried offset stands at.
  __device__ __forceinline__ int at(int t) const {
    if constexpr (kCarried) return off;
    return (int)((unsigned)t % N) * STEP;
  }
};

// Compile-time configuration of one kernel instance: head dimensions, key-tile width, waves per
// workgroup, 32-row query blocks per wave, causal masking, split mode, workgroups sharing a CU (OCC),
// K and V fragments read ahead from LDS (KPF, VPF), K and V ring slots in LDS (NKR, NVR), and the
// parts each key tile is split into between the waves (KSPLIT).
template <int DQK_, int DV_, int BN_, int NWAVES_, int QB_, bool CAUSAL_, bool SPLIT_, int OCC_, int KPF_, int VPF_,
          int NKR_, int NVR_, int KSPLIT_ = 1>
struct Cfg {
  static constexpr int DQK = DQK_, DV = DV_, BN = BN_, NWAVES = NWAVES_, QB = QB_;
  // KSPLIT = 2: the waves form two sets of NWAVES / 2 (RWAVES) that own the same query rows; set k
  // takes the k-th 32-key half of every key tile (WBN keys per wave and tile), and the two partial
  // results of each row are merged in LDS at the end.
  static constexpr int KSPLIT = KSPLIT_, RWAVES = NWAVES / KSPLIT_, WBN = BN_ / KSPLIT_;
  static constexpr int KPF = KPF_, VPF = VPF_;
  static constexpr int OCC = OCC_;  // workgroups sharing a CU
  static constexpr bool CAUSAL = CAUSAL_;
  // SPLIT: each workgroup takes one of n_split contiguous parts of its query block's key tiles and
  // writes a partial result (O normalised by its own row sum, fp32, and its LSE) for a merge pass.
  static constexpr bool SPLIT = SPLIT_;
  static constexpr bool CHUNKED = QB > 1;  // long instance: key/value heads in chunks (launch_cfg)
  static constexpr int NT = NWAVES * 64;
  // Waves per SIMD the registers are budgeted for: the workgroup's own (4 SIMDs per CU) times the
  // workgroups that share a CU (OCC_).
  static constexpr int WPE = (NWAVES > 4 ? NWAVES / 4 : 1) * OCC_;
  static constexpr int BM = RWAVES * 32 * QB;  // query rows per workgroup holding one query head
  static constexpr int KCH = DQK / 8;          // 16-byte chunks per K-tile row
  static constexpr int VCH = DV / 8;           // 16-byte chunks per V-tile row
  static constexpr int K_BYTES = BN * DQK * 2;
  static constexpr int V_BYTES = BN * DV * 2;
  // Ring slots. Step j loads K(j + KA) into the slot of K(j) and V(j + VA) into the slot of V(j-2):
  // both were last read in step j-1, which every wave has finished at the barrier of step j.
  static constexpr int NKR = NKR_, NVR = NVR_;
  static constexpr int KA = NKR, VA = NVR - 2;  // how far ahead step j loads K and V tiles
  static constexpr int RING_BYTES = NKR * K_BYTES + NVR * V_BYTES;
  // The rings' LDS also stages the output tile (STAGE_BYTES) and, behind it, the exchange of the key
  // parts' results (XCH_BYTES: per lane of every row chunk, O of all parts but one and every part's
  // reference maximum and row sum); with small key tiles these are the larger.
  static constexpr int STAGE_BYTES = RWAVES * 32 * QB * DV * 2;
  static constexpr int XCH_BYTES =
      KSPLIT > 1 ? RWAVES * ((KSPLIT - 1) * (DV / 2) + KSPLIT * 2) * QB * 64 * 4 : 0;
  static constexpr int LDS_BYTES =
      RING_BYTES > STAGE_BYTES + XCH_BYTES ? RING_BYTES : STAGE_BYTES + XCH_BYTES;
  // Direct-to-LDS loads per wave per tile (each moves 64 lanes x 16 bytes).
  static constexpr int K_LOADS = BN * KCH / 64 / NWAVES;
  static constexpr int V_LOADS = BN * VCH / 64 / NWAVES;
  static_assert(DQK % 32 == 0 && DV % 64 == 0, "head dims: d_qk multiple of 32, d_v multiple of 64");
  static_assert(WBN % 32 == 0, "every wave takes whole 32-key blocks of a tile");
  static_assert((BN * KCH) % (64 * NWAVES) == 0 && (BN * VCH) % (64 * NWAVES) == 0, "tile split over waves");
  // KA - 1 <= VA <= KA: V(j-1) is issued before K(j+1) (so one counted wait covers both), and the
  // prologue's groups j = -KA .. -1 hold every tile's first load.
  static_assert(NKR >= 2 && NKR + 1 <= NVR && NVR <= NKR + 2, "ring sizes");
  static_assert(V_LOADS + KA * (K_LOADS + V_LOADS) < 64 && VA * (K_LOADS + V_LOADS) < 64, "vmcnt range");
  static_assert(LDS_BYTES * OCC_ <= 163840, "LDS budget of the workgroups sharing a CU");
  static_assert(KSPLIT == 1 || (!SPLIT && NWAVES % KSPLIT == 0), "key parts: equal wave sets, not split mode");
};

// Division by a divisor that is fixed for the launch, as a multiply-high and two shifts (Granlund and
// Montgomery, "Division by invariant integers using multiplication", PLDI 1994, the algorithm for
// unsigned 32-bit operands): with l = ceil(log2 d) and m = floor(2^32 (2^l - d) / d) + 1, every 32-bit
// n has n / d = (t + ((n - t) >> min(l, 1))) >> max(l - 1, 0), t = mulhi(m, n). The host computes m and
// the two shifts (6 bits: min(l, 1) | max(l - 1, 0) << 1); the kernel's work decomposition then needs
// no division sequence (a runtime division by a value the compiler cannot see is ~25 instructions).
struct FastDiv {
  uint32_t m, sh;
};
FastDiv make_fastdiv(uint32_t d) {
  uint32_t l = 0;
  while ((uint64_t{1} << l) < d) ++l;
  const uint64_t m = ((uint64_t{1} << 32) * ((uint64_t{1} << l) - d)) / d + 1;
  return {static_cast<uint32_t>(m), (l < 1 ? l : 1u) | ((l > 0 ? l - 1 : 0u) << 1)};
}
__device__ __forceinline__ uint32_t fast_div(uint32_t n, uint32_t m, uint32_t sh) {
  const uint32_t t = __umulhi(m, n);
  return (t + ((n - t) >> (sh & 1u))) >> (sh >> 1);
}

// What the work decomposition needs, all uniform over the launch: workgroups per query block of one
// key/value head (`group`: the GQA group size over the query heads a workgroup packs), key/value heads,
// batch, query blocks per head, the items in whole XCD spans (below), and the fast divisions by
// `group`, the key/value heads and the batch (their shifts packed 6 bits apart in bits 0-17; bits
// 18-19 hold log2 of the query heads packed per workgroup).
struct WorkMap {
  int group, hkv, batch, n_qtiles, full;
  uint32_t m_group, m_hkv, m_batch, shifts;
};

// Map a hardware workgroup index to (batch, key/value head, member, query block); the member selects
// which of the key/value head's query heads the workgroup takes. Workgroup t runs on XCD t % 8.
// Logical work items are ordered by chunk of key/value heads (head_chunk heads each, the first
// head_chunked of the batch's heads in whole chunks; the short and key-parts instances have one chunk),
// then heaviest query block first (causal), then batch, key/value head and member; each group of `group`
// consecutive items (the workgroups of one key/value head at one query block) is placed on one XCD, and
// groups go to XCDs round-robin (`full` = the items in whole spans of 8 groups; the rest keep their order).
// FAST divides through
// the multiply-high constants, else with the compiler's division sequence (the long instance: there
// the faster prologue measured no gain in time, and on the 128K workload it shifted the relative
// start times of the workgroups that stream one K/V head through an XCD's L2 enough to double the L2
// misses; the mapping is the same either way).
template <bool FAST>
__device__ __forceinline__ void decode_workgroup(uint32_t t, const WorkMap& w, int head_chunk, int head_chunked,
                                                 bool causal, int& b, int& kvh, int& member, int& qtile) {
  if constexpr (FAST) {
    const uint32_t G = w.group, sg = w.shifts & 63u, sh = (w.shifts >> 6) & 63u, sb = (w.shifts >> 12) & 63u;
    uint32_t L = t;
    if (t < (uint32_t)w.full) {
      const uint32_t xcd = t % kNumXcd, slot = t / kNumXcd, sq = fast_div(slot, w.m_group, sg);
      L = (sq * kNumXcd + xcd) * G + (slot - sq * G);
    }
    const uint32_t r = fast_div(L, w.m_group, sg);
    member = (int)(L - r * G);
    const uint32_t r2 = fast_div(r, w.m_hkv, sh);
    kvh = (int)(r - r2 * (uint32_t)w.hkv);
    const uint32_t qt = fast_div(r2, w.m_batch, sb);
    b = (int)(r2 - qt * (uint32_t)w.batch);
    qtile = causal ? w.n_qtiles - 1 - (int)qt : (int)qt;
  } else {
    const int G = w.group;
    int L = (int)t;
    if (L < w.full) {
      const int xcd = L % kNumXcd, slot = L / kNumXcd;
      L = ((slot / G) * kNumXcd + xcd) * G + slot % G;
    }
    member = L % G;
    const int r = L / G;
    // The span of key/value heads this item belongs to: a whole chunk, or the heads after them.
    const int chunked = head_chunked * w.n_qtiles;
    int first = 0, heads = head_chunk, rr = r;
    if (r < chunked) {
      first = r / (head_chunk * w.n_qtiles) * head_chunk;
      rr -= first * w.n_qtiles;
    } else {
      first = head_chunked;
      heads = w.hkv * w.batch - head_chunked;
      rr -= chunked;
    }
    const int qt = rr / heads, hd = first + rr % heads;
    kvh = hd % w.hkv;
    b = hd / w.hkv;
    qtile = causal ? w.n_qtiles - 1 - qt : qt;
  }
}

// Per-wave state and the math of the pipelined step.
//
// Reference maximum (the lazy form of Alg. 1's running maximum): the first tile sets m_run to the
// exact row maximum. Afterwards the per-element maximum is not computed: each lane's sum of its
// tile exponentials bounds every one of them, so when all lane sums stay <= 2^8 no probability
// exceeds 2^8 and the tile is final. Otherwise (a new maximum well above the reference; rare) the
// tile is redone from its exact row maximum, with O and l rescaled by 2^(m_old - m_new) (rebase).
// O / l is invariant under the choice of reference, and l >= 1 since the reference is always a
// score that has been seen.
template <class C>
struct Attn {
  static constexpr int DQK = C::DQK, DV = C::DV, BN = C::WBN, QB = C::QB;  // BN: this wave's keys of a tile
  static constexpr int KS = DQK / 16;  // k-steps of the score product
  static constexpr int KB = BN / 32;   // 32-key blocks per tile
  static constexpr int DB = DV / 32;   // 32-dim blocks of the output
  static constexpr int PS = BN / 16;   // k-steps of the P V product (16-key chunks)

  typedef f32x16 Scores[KB][QB];    // S^T of one tile, raw (unscaled)
  typedef uint32_t Probs[KB][QB][8];  // P of one tile as packed bf16 pairs

  static constexpr int NMS = KS * KB * QB;  // score MFMAs per tile
  static constexpr int NMP = PS * DB * QB;  // P V MFMAs per tile
  static constexpr int NSL = NMS + NMP;     // MFMA slots per step
  static constexpr bool AG = C::WPE == 1;   // O and Q in AGPRs
  static constexpr int NEP = KB * QB * 8;   // exponential pairs per lane per tile
  static constexpr int NVF = PS * DB;       // V fragments per tile
  static constexpr int KPF = C::KPF;        // K fragments read ahead
  static constexpr int VPF = C::VPF;        // V fragments read ahead

  int i32, h, qw, diag, sk;
  const uint16_t* kg;  // this workgroup's K head in global memory (rebase only)
  float cs;            // scale * log2(e), signed
  float mask_val;      // a score that cs maps to -inf
  int v_key, v_t, v_half;
  bf16x8 qf[QB][KS];
  f32x16 oacc[DB][QB];
  float m_run[QB], l_run[QB];

  // Slot order of a step: the P V MFMAs of tile j-1 first (chunk c of P, 16 keys, in slots
  // [c * E0, (c + 1) * E0)), then the score MFMAs of tile j+1 (32-key-block-major, so that the score
  // accumulators of block kb of the new tile are written only after the exponentials of block kb of
  // the current one, and the two score tiles overlap in registers only partly).
  static constexpr int E0 = NMP / PS;
  static constexpr bool slot_is_score(int sl) { return sl >= NMP; }

  __device__ __forceinline__ u32x4 kfrag(const unsigned char* sK, int ks, int kb) const {
    const int row = kb * 32 + perm32(i32);
    return *reinterpret_cast<const u32x4*>(sK + row * (DQK * 2) + (((ks * 2 + h) ^ k_lane_swizzle<DQK>(i32)) << 4));
  }
  // A operand V^T[dims db*32 + 0..31][keys 16*ps + 0..15]: lane (group G, slot j) points the
  // transpose read at key 16*ps + 8*(G/2) + j/4 (then +4), dims db*32 + 16*(G%2) + 4*(j%4).
  __device__ __forceinline__ bf16x8 vfrag(const unsigned char* sV, int ps, int db) const {
    const unsigned char* base = sV + (ps * 16 + v_key) * (DV * 2) + (((db * 4) ^ v_t) << 4) + v_half;
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(base));
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(base + 4 * DV * 2));
    return bit_cast<bf16x8>(__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }

  // Score MFMA number i of a tile in 32-key-block-major order (kb, ks, qb); K fragments (sequence
  // f = kb*KS + ks) are read KPF ahead.
  __device__ __forceinline__ void score_mfma(Scores& s, u32x4 (&kf)[KB * KS], const unsigned char* sK, int i) {
    const int kb = i / (KS * QB), ks = (i / QB) % KS, qb = i % QB, f = kb * KS + ks;
    if (qb == 0 && f + KPF < KB * KS) kf[f + KPF] = kfrag(sK, (f + KPF) % KS, (f + KPF) / KS);
    s[kb][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bit_cast<bf16x8>(kf[f]), qf[qb][ks],
                                                        ks == 0 ? f32x16{} : s[kb][qb], 0, 0, 0);
  }
  __device__ __forceinline__ void scores(Scores& s, const unsigned char* sK) {
    u32x4 kf[KB * KS];
#pragma unroll
    for (int f = 0; f < KPF && f < KB * KS; ++f) kf[f] = kfrag(sK, f % KS, f / KS);
#pragma unroll
    for (int i = 0; i < NMS; ++i) score_mfma(s, kf, sK, i);
  }

  // Masked keys of tile n0 (key > i + diag, or key >= Sk) get mask_val. The select is a bit
  // select on the sign of (lim - key offset): a compare per element would need a scalar register
  // pair per mask, and the scheduler hoists all 64 of them.
  __device__ __forceinline__ void mask_tile(Scores& s, int n0) const {
    const uint32_t mv = __float_as_uint(mask_val);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const int row = qw + qb * 32 + i32;
      const int last_key = C::CAUSAL ? min(row + diag, sk - 1) : sk - 1;
      const int lim = last_key - n0 - 8 * h;  // key offset kb*32 + 16*(r/8) + r%8 is masked iff > lim
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const uint32_t m = (uint32_t)((lim - (kb * 32 + 16 * (r >> 3) + (r & 7))) >> 31);  // all ones if masked
          s[kb][qb][r] = __uint_as_float((__float_as_uint(s[kb][qb][r]) & ~m) | (mv & m));
        }
    }
  }

  // Exact maximum of cs * score over the row (both lane halves), -inf if every key is masked.
  __device__ __forceinline__ float row_max(const Scores& s, int qb) const {
    float m = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) m = fmaxf(m, s[kb][qb][r] * cs);
    return half_swap_max(m);
  }

  // Element schedule of the step: the NEL = 2 * NEP exponentials of a tile are spread
  // one by one over the NSL MFMA slots (element e in slot e * NSL / NEL), each as one fma and one
  // exp2 right after the slot's MFMA; the two adds and the pack of pair u follow in the slot after
  // the one of its second element. At d = 128 a slot then carries 3 and 6 full-rate-equivalent VALU
  // instructions in turn, within what a 32-cycle MFMA absorbs. A pair's pack writes P chunk c only
  // after the P V MFMAs of chunk c (slots [c * E0, (c + 1) * E0)) for every c >= 1, so the old and new
  // P share registers there; chunk 0 is written earlier and takes registers of its own.
  static constexpr int NEL = 2 * NEP;
  static constexpr int elem_begin(int sl) { return (sl * NEL + NSL - 1) / NSL; }
  static constexpr int elem_end(int sl) { return ((sl + 1) * NEL + NSL - 1) / NSL; }
  static constexpr bool packs_follow_pv() {
    for (int u = 0; u < NEP; ++u) {
      int sl = 0;
      while (elem_end(sl) <= 2 * u + 1) ++sl;  // slot of element 2u+1
      const int c = u / (QB * 4);             // P chunk (16 keys) of pair u
      if (c >= 1 && sl + 1 < (c + 1) * E0) return false;
    }
    return true;
  }
  static_assert(packs_follow_pv(), "a pack would overwrite P of a chunk before its P V MFMAs");
  static constexpr bool at_most_two_elems_per_slot() {
    for (int sl = 0; sl < NSL; ++sl)
      if (elem_end(sl) - elem_begin(sl) > 2) return false;
    return true;
  }

  // Element e of a tile: p = 2^(cs * s - m_ref).
  __device__ __forceinline__ float exp_elem(int e, const Scores& cur, const float (&mref)[QB]) const {
    const int u = e >> 1, qb = u % QB, rp = (u / QB) % 8, kb = u / (QB * 8);
    float x = __builtin_amdgcn_exp2f(fmaf(cur[kb][qb][2 * rp + (e & 1)], cs, -mref[qb]));
    asm volatile("" : "+v"(x));
    return x;
  }
  // Pair u: the lane's row sum and the bf16 pair. The first pair of each row block starts the sum.
  __device__ __forceinline__ void pack_pair(int u, float e0, float e1, Probs& pk, float (&rs)[QB]) const {
    const int qb = u % QB, rp = (u / QB) % 8, kb = u / (QB * 8);
    if (u < QB)
      rs[qb] = e0 + e1;
    else
      rs[qb] += e0 + e1;
    pk[kb][qb][rp] = pack_bf16x2(e0, e1);
    asm volatile("" : "+v"(pk[kb][qb][rp]));
  }

  // P V MFMA number p of a tile (order ps, db, qb), V fragments read VPF ahead. `settled`: P was
  // written long before (in the step: one step earlier), so no wait states are needed.
  __device__ __forceinline__ void pv_mfma(int p, const Probs& pk, bf16x8 (&vf)[NVF], const unsigned char* sV,
                                          bool settled = false) {
    const int t = p / QB, qb = p % QB, ps = t / DB, db = t % DB;
    if (qb == 0 && t + VPF < NVF) vf[t + VPF] = vfrag(sV, (t + VPF) / DB, (t + VPF) % DB);
    const int kb = ps >> 1, base = (ps & 1) * 4;
    const u32x4 w = {pk[kb][qb][base], pk[kb][qb][base + 1], pk[kb][qb][base + 2], pk[kb][qb][base + 3]};
    if (settled)
      mfma_out_settled<AG>(oacc[db][qb], vf[t], bit_cast<bf16x8>(w));
    else
      mfma_out<AG>(oacc[db][qb], vf[t], bit_cast<bf16x8>(w));
  }

  // All P V MFMAs of one tile (the last tile, after the loop).
  __device__ __forceinline__ void pv_tile(const Probs& pk, const unsigned char* sV) {
    bf16x8 vf[NVF];
#pragma unroll
    for (int t = 0; t < VPF && t < NVF; ++t) vf[t] = vfrag(sV, t / DB, t % DB);
#pragma unroll
    for (int pi = 0; pi < NMP; ++pi) pv_mfma(pi, pk, vf, sV);
  }

  // Redo a tile's exponentials from its exact row maximum; O and l follow the new reference. The
  // tile's scores are recomputed from K in global memory (rows clamped to Sk-1, masked anyway): by
  // the end of the step the raw scores are gone and the tile's LDS slot holds a later tile.
  __device__ __forceinline__ void rebase(Probs& pk, float (&rs)[QB], int n0, bool masked) {
    Scores cur;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const int row = min(n0 + kb * 32 + perm32(i32), sk - 1);
      const uint16_t* krow = kg + (size_t)row * DQK + 8 * h;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const u32x4 a = *reinterpret_cast<const u32x4*>(krow + 16 * ks);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
          cur[kb][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bit_cast<bf16x8>(a), qf[qb][ks],
                                                                ks == 0 ? f32x16{} : cur[kb][qb], 0, 0, 0);
      }
    }
    if (masked) mask_tile(cur, n0);
    float mref[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const float m_new = fmaxf(m_run[qb], row_max(cur, qb));
      const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run[qb] - m_new);
      m_run[qb] = m_new;
      l_run[qb] *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        agpr_fence<AG>(oacc[db][qb]);
        oacc[db][qb] *= alpha;
        agpr_fence<AG>(oacc[db][qb]);
      }
      mref[qb] = m_new == -INFINITY ? 0.f : m_new;
    }
#pragma unroll
    for (int u = 0; u < NEP; ++u) {
      const float e0 = exp_elem(2 * u, cur, mref), e1 = exp_elem(2 * u + 1, cur, mref);
      pack_pair(u, e0, e1, pk, rs);
    }
  }

  // One pipeline step: P V of tile j-1 (pk_old, V slot sVo), exponentials of tile j (cur, key n0,
  // into pk_new) and scores of tile j+1 (K slot sKn, into nxt).
  // `issue(k)` starts load k (0 <= k < LOADS) of the tiles this step prefetches; the loads are spread
  // one every NSL / LOADS slots, between MFMAs (a burst of them would stall the wave).
  template <class Issue>
  __device__ __forceinline__ void step(Scores& cur, Scores& nxt, Probs& pk_new, const Probs& pk_old,
                                       const unsigned char* sKn, const unsigned char* sVo, bool masked, int n0,
                                       Issue&& issue) {
    if (masked) mask_tile(cur, n0);
    float mref[QB], rs[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      mref[qb] = m_run[qb] == -INFINITY ? 0.f : m_run[qb];
      rs[qb] = 0.f;
    }
    // V fragments first: the step's first MFMAs are P V's, so with one wave per SIMD every LDS read in
    // front of them is latency the wave waits out (one head S16384 d64 112.4 -> 107.4 us, GPT-2 S2048
    // 15.9 -> 15.6 us against K first; level where other waves fill the wait).
    bf16x8 vf[NVF];
#pragma unroll
    for (int t = 0; t < VPF && t < NVF; ++t) vf[t] = vfrag(sVo, t / DB, t % DB);
    __builtin_amdgcn_sched_barrier(0);
    u32x4 kf[KB * KS];
#pragma unroll
    for (int f = 0; f < KPF && f < KB * KS; ++f) kf[f] = kfrag(sKn, f % KS, f / KS);
    static_assert(at_most_two_elems_per_slot(), "ev holds the elements of two slots");
    float ev[4];  // exponentials in flight, element e in ev[e % 4]
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int sl = 0; sl < NSL; ++sl) {
      {
        constexpr int NLD = C::K_LOADS + C::V_LOADS, SP = NSL / NLD;
        static_assert(SP >= 1, "more loads than slots");
        if (sl % SP == SP / 2 && sl / SP < NLD) issue(sl / SP);
      }
      if (slot_is_score(sl))
        score_mfma(nxt, kf, sKn, sl - NMP);
      else
        pv_mfma(sl, pk_old, vf, sVo, true);
      __builtin_amdgcn_sched_barrier(0);  // the slot's MFMA is issued before its VALU work
      if (sl > 0) {
#pragma unroll
        for (int e = elem_begin(sl - 1); e < elem_end(sl - 1); ++e)
          if (e & 1) pack_pair(e >> 1, ev[(e - 1) % 4], ev[e % 4], pk_new, rs);
      }
#pragma unroll
      for (int e = elem_begin(sl); e < elem_end(sl); ++e) ev[e % 4] = exp_elem(e, cur, mref);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int e = elem_begin(NSL - 1); e < elem_end(NSL - 1); ++e)
      if (e & 1) pack_pair(e >> 1, ev[(e - 1) % 4], ev[e % 4], pk_new, rs);
    bool over = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) over = over || !(rs[qb] <= kOverflowSum);
    if (__builtin_amdgcn_ballot_w64(over) != 0) rebase(pk_new, rs, n0, masked);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) l_run[qb] += rs[qb];
  }
};

// The kernel body, shared by the two entry kernels below.
template <class C>
__device__ __forceinline__ void fa_fwd_body(FwdParams p, const WorkMap wm) {
  using A = Attn<C>;
  constexpr int DQK = C::DQK, DV = C::DV, BN = C::BN, QB = C::QB;

  __shared__ __attribute__((aligned(1024))) unsigned char smem[C::LDS_BYTES];
  auto kswz = [](int row) { return k_swizzle<DQK>(row); };
  auto vswz = [](int row) { return v_swizzle<DV>(row); };

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  A st;
  st.i32 = lane & 31;
  st.h = lane >> 5;
  // Lane constants of the V transpose read: group G = lane/16, slot j = lane%16.
  st.v_key = 8 * (lane >> 5) + ((lane & 15) >> 2);                             // key in the 16-key step
  st.v_t = (2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ v_swizzle<DV>(st.v_key);  // low chunk bits, swizzled
  st.v_half = (lane & 1) * 8;                                                  // byte offset in the chunk
  st.sk = p.sk;

  // Split mode: workgroup t takes part t / n_wg of work item t % n_wg.
  const int split = C::SPLIT ? (int)(blockIdx.x / p.n_wg) : 0;
  int b, g, member, qtile;
  decode_workgroup<!C::CHUNKED>(C::SPLIT ? blockIdx.x % (uint32_t)p.n_wg : blockIdx.x, wm, p.head_chunk,
                                p.head_chunked, C::CAUSAL, b, g, member, qtile);
  // Query heads packed per workgroup (HW = 1, 2 or 4, the largest that divides the GQA group size):
  // the waves split into HW heads of the same key/value head, each taking NWAVES / HW consecutive
  // 32*QB-row chunks of the block's rows, so that all heads of the workgroup share every K/V tile
  // and, when HW = NWAVES, every wave visits the same key tiles (no wave idles through the tiles of
  // a causal diagonal that its rows do not see).
  // With key parts (KSPLIT = 2 or 4) the same applies within each wave set: wave w belongs to set
  // w / RWAVES, which takes keys [kpart, kpart + WBN) of every tile, and to row chunk w % RWAVES.
  const int hw_log = (int)((wm.shifts >> 18) & 3u);
  const int kset = C::KSPLIT > 1 ? wave / C::RWAVES : 0, rwave = C::KSPLIT > 1 ? wave % C::RWAVES : wave;
  const int kpart = kset * C::WBN;                       // first key of this wave's part of a tile
  const int rw = C::RWAVES >> hw_log;                    // row chunks per head
  const int bmr = rw * 32 * QB;                          // query rows of the block
  const int hq = g * p.group + (member << hw_log) + rwave / rw;
  const uint16_t* __restrict__ qh = p.q + (size_t)(b * p.hq + hq) * p.sq * DQK;

  const int q0 = qtile * bmr;
  st.qw = q0 + (rwave % rw) * 32 * QB;  // first query row of this wave
  st.diag = p.sk - p.sq;        // key j is visible to query i iff j <= i + diag

  // Key tiles this workgroup visits, and how many leading ones need no mask for any of its rows.
  int kv_end = p.sk;
  int n_plain = p.sk / BN;
  if (C::CAUSAL) {
    const int last_row = min(q0 + bmr, p.sq) - 1;
    kv_end = max(0, min(p.sk, last_row + st.diag + 1));
    n_plain = min(n_plain, max(0, q0 + st.diag + 1) / BN);
  }
  // Key tiles [t0, t0 + nt) of the query block: all of them, or one contiguous part in split mode.
  int t0 = 0, nt = (kv_end + BN - 1) / BN;
  if (C::SPLIT) {
    const int per = (nt + p.n_split - 1) / p.n_split;
    t0 = min(nt, split * per);
    nt = min(nt, t0 + per) - t0;
  }
  const int kb0 = t0 * BN;                     // first key of the range
  n_plain = min(max(n_plain - t0, 0), nt);     // leading tiles of the range that need no mask
  const int kv_lim = min(kv_end, kb0 + nt * BN);  // keys loaded; past it the tile loads read zeros

  // Q rows of this wave as B operands of the score product, resident in AGPRs: lane (i32, h) holds
  // row qw+32*qb+i32, dims 16*ks + 8*h .. +7. Rows past Sq read row Sq-1 instead; their outputs are
  // never stored. Issued first, waited for together with the first K tile below.
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int row = min(st.qw + qb * 32 + st.i32, p.sq - 1);
#pragma unroll
    for (int ks = 0; ks < A::KS; ++ks) load_q<A::AG>(st.qf[qb][ks], qh + (size_t)row * DQK + ks * 16 + st.h * 8);
  }
  // What comes from the argument block (not preloaded) is used only from here on, but for the chunks of
  // heads in decode_workgroup (long instance: see the entry kernels).
  const uint16_t* __restrict__ kh = p.k + (size_t)(b * p.hkv + g) * p.sk * DQK;
  const uint16_t* __restrict__ vh = p.v + (size_t)(b * p.hkv + g) * p.sk * DV;
  st.kg = kh;
  st.cs = p.cs;
  st.mask_val = p.cs < 0.f ? INFINITY : -INFINITY;

  // Rings: step j loads K(j+KA) and V(j+VA) (the group of step j); the prologue loads the groups of
  // j = -KA .. -1 (with the defaults KA = VA = 2: K0, V0, K1, V1 in this order), each group's V tile
  // only from V0 on. Every group is issued in full: a tile at or past the last one loads
  // zeros into a slot nobody reads any more, so the number of loads issued after any given one is a
  // constant and every wait below is a fixed count.
  TileLoader<C::NWAVES, BN, C::KCH> kload;
  TileLoader<C::NWAVES, BN, C::VCH> vload;
  kload.init(kh, kv_lim, wave, lane, kswz);
  vload.init(vh, kv_lim, wave, lane, vswz);
  // (tile indices are never negative: unsigned remainders, a mask for the power-of-two ring sizes)
  auto kslot = [&](int t) { return smem + ((unsigned)t % C::NKR) * C::K_BYTES; };
  auto vslot = [&](int t) { return smem + C::NKR * C::K_BYTES + ((unsigned)t % C::NVR) * C::V_BYTES; };
  // This wave's keys of K tile t (rows kpart .. kpart + WBN - 1 of the slot). The K and V swizzles
  // repeat every 32 rows, so a part starting at row 32 reads like a tile of its own.
  auto kmine = [&](int t) { return kslot(t) + kpart * (DQK * 2); };
#pragma unroll
  for (int g = -C::KA; g < 0; ++g) {
    // P of "tile -1" is zero, and so must its V be, or an infinity or a NaN there would reach every row: zeros
    // into the slot before V0's, which the loads reach in step 1. Issued before K1, whose wait covers them.
    // They cost 0-0.2 us a workgroup (128-head calls of 23 rows at d_qk = 192 9.7 -> 9.9 us, one head S256 and
    // the prefills of 8K and 128K tokens level); zeros stored by the threads 0.3 us in the key quarters, and a
    // first step compiled without its P V 2 % of 14/2 S32768 d64 and 1.8 % of 32/8 S131072.
    if (g == 1 - C::KA) vload.issue_zeros(vslot(C::NVR - 1), wave);
    kload.issue(kb0 + (g + C::KA) * BN, kslot(g + C::KA), wave);
    if (g + C::VA >= 0) vload.issue(kb0 + (g + C::VA) * BN, vslot(g + C::VA), wave);
  }
  // Q and K0 must have landed: issued after K0 are V0 when VA = KA, the zeros, then the groups of j =
  // -KA+1 .. -1 (K and V each, since VA >= KA - 1).
  wait_vmcnt<C::V_LOADS + (C::VA == C::KA ? C::V_LOADS : 0) + (C::KA - 1) * (C::K_LOADS + C::V_LOADS)>();
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int ks = 0; ks < A::KS; ++ks) q_ready<A::AG>(st.qf[qb][ks]);

#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    st.m_run[qb] = -INFINITY;
    st.l_run[qb] = 0.f;
#pragma unroll
    for (int db = 0; db < A::DB; ++db) {
      st.oacc[db][qb] = f32x16{};
      agpr_fence<A::AG>(st.oacc[db][qb]);
    }
  }

  typename A::Scores sA, sB;
  typename A::Probs pA, pB;
  if (nt > 0) {
    // Tile 0: scores, mask, exact row maxima.
    compiler_fence();
    __builtin_amdgcn_s_barrier();
    compiler_fence();
    st.scores(sA, kmine(0));
    if (n_plain == 0) st.mask_tile(sA, kb0 + kpart);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) st.m_run[qb] = st.row_max(sA, qb);
#pragma unroll
    for (int kb = 0; kb < A::KB; ++kb)
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int r = 0; r < 8; ++r) pB[kb][qb][r] = 0u;
  }
  // Before step j: K(j+1) and V(j-1) must have landed. K(j+1) belongs to the group of step j+1-KA;
  // this wave's loads issued after it are that group's V tile and the KA-2 groups after it (with
  // the defaults only V(j+1)); V(j-1), from the group of step j+1-NVR, came before it.
  // The barrier then publishes every wave's part and guarantees that all waves are done with step
  // j-1, whose slots (K(j), V(j-2)) the loads of step j overwrite.
  // The steps run in order j = 0, 1, ..., so the buffers of the tiles a step loads are the previous
  // step's moved on by one tile (they start one tile before those of step 0).
  int krem, vrem;
  u32x4 gk = kload.rsrc_walk(kb0 + (C::KA - 1) * BN, krem), gv = vload.rsrc_walk(kb0 + (C::VA - 1) * BN, vrem);
  uint32_t gkl = 0, gvl = 0;
  // The rings at the start of step j: K(j+KA) overwrites the slot of K(j) and V(j+VA) that of V(j-2);
  // moved on by one tile they stand at K(j+1) and V(j-1), which the step reads.
  unsigned char* const vring = smem + C::NKR * C::K_BYTES;
  Ring<C::K_BYTES, C::NKR> kring(0);
  Ring<C::V_BYTES, C::NVR> vpos(C::NVR - 2);
  auto kread = [&](int t) { return smem + kring.at(t) + kpart * (DQK * 2); };
  auto vread = [&](int t) { return vring + vpos.at(t) + kpart * (DV * 2); };
  // What step 0 reads in V(-1)'s place. It is the slot vread(-1) would find; named, the compiler's code for the
  // loop measured 0.3 % slower than without the zeros, through vread 0.9 % (GQA 14/2 S32768 d64 causal).
  unsigned char* const vzero = vslot(C::NVR - 1) + kpart * (DV * 2);
  auto sync_step = [&](int j) {
    wait_vmcnt<C::V_LOADS + (C::KA - 2) * (C::K_LOADS + C::V_LOADS)>();
    compiler_fence();
    __builtin_amdgcn_s_barrier();
    compiler_fence();
    kload.advance(gk, krem);
    gkl = kload.lds(smem + kring.at(j + C::KA), wave);
    vload.advance(gv, vrem);
    gvl = vload.lds(vring + vpos.at(j + C::VA), wave);
    if constexpr (decltype(kring)::kCarried) gkl = __builtin_amdgcn_readfirstlane(gkl);
    if constexpr (decltype(vpos)::kCarried) gvl = __builtin_amdgcn_readfirstlane(gvl);
    kring.next();
    vpos.next();
  };
  auto issue = [&](int k) {
    if (k < C::K_LOADS)
      kload.issue_one(gk, gkl, k);
    else
      vload.issue_one(gv, gvl, k - C::K_LOADS);
  };
  // Steps in pairs so that the two score tiles and the two P tiles swap roles without copies. A step
  // masks its current tile from tile n_plain on; tile 0 was masked above when n_plain = 0, and masking
  // it again in step 0 changes nothing (masked scores already hold mask_val), so the test needs no
  // j > 0 term (one scalar compare per step instead of two compares and the mask logic).
  int j = 0;
  for (; j + 1 < nt; j += 2) {
    sync_step(j);
    st.step(sA, sB, pA, pB, kread(j + 1), j > 0 ? vread(j - 1) : vzero, j >= n_plain,
            kb0 + j * BN + kpart, issue);
    sync_step(j + 1);
    st.step(sB, sA, pB, pA, kread(j + 2), vread(j), j + 1 >= n_plain, kb0 + (j + 1) * BN + kpart, issue);
  }
  if (j < nt) {
    sync_step(j);
    st.step(sA, sB, pA, pB, kread(j + 1), j > 0 ? vread(j - 1) : vzero, j >= n_plain,
            kb0 + j * BN + kpart, issue);
  }
  if (nt > 0) {
    // P V of the last tile, on a selected copy of P: two calls would leave O in different
    // registers and the copies that merge them could read MFMA results before they are written.
    // (The select is a bit mask: a ternary on the elements would be folded into a select of the
    // two arrays' addresses, which forces both into scratch memory.) V(nt-1) belongs to the load
    // group of step nt-1-VA; the VA groups after it may still be in flight.
    wait_vmcnt<C::VA * (C::K_LOADS + C::V_LOADS)>();
    compiler_fence();
    __builtin_amdgcn_s_barrier();
    compiler_fence();
    typename A::Probs pl;
    const uint32_t take_a = (nt & 1) ? 0xffffffffu : 0u;
#pragma unroll
    for (int kb = 0; kb < A::KB; ++kb)
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int r = 0; r < 8; ++r) pl[kb][qb][r] = (pA[kb][qb][r] & take_a) | (pB[kb][qb][r] & ~take_a);
    vpos.next();
    st.pv_tile(pl, vread(nt - 1));
  }

  // No load may still be writing this workgroup's LDS when it exits (the prologue issues loads even
  // when there is no key tile to visit), and the output tile is staged in the ring slots below: every
  // wave's loads must have landed and every wave must be done with the last V tile.
  wait_vmcnt<0>();
  compiler_fence();
  __builtin_amdgcn_s_barrier();
  compiler_fence();

  if constexpr (C::KSPLIT > 1) {
    // Merge of the key parts (the combination step of Alg. 2 inside the workgroup). The waves with the
    // same rows, one per set, hold the same rows and dims in the same registers. Each set finishes a
    // share of them: the accumulators of a wave are NCH chunks of 4 registers, set t owns chunks
    // [t * CPS, (t + 1) * CPS), and every wave hands the chunks it does not own, with its reference
    // maxima and lane row sums, to their owners through LDS, lane by lane. With m the maximum of the
    // parts' references m_k: O = sum O_k 2^(m_k - m), likewise l, added in the order of the parts; a part
    // that saw no visible key (m_k = -inf, O = 0, l = 0) gets weight 0. The output tile is staged like
    // below, and each set stores its share of its rows. The exchange area lies past the staging tiles.
    // (One set merging everything while the others exit took 0.1-0.4 us more per workgroup.)
    constexpr int KP = C::KSPLIT, NCH = A::DB * QB * 4, CPS = NCH / KP;
    static_assert(NCH % KP == 0, "accumulator chunks split over the sets");
    constexpr int WSTR = (KP - 1) * NCH * 256 + KP * 2 * QB * 64;  // exchanged floats per row chunk
    static_assert(C::STAGE_BYTES + C::RWAVES * WSTR * 4 <= C::LDS_BYTES, "exchange area fits the LDS");
    float* const xo = reinterpret_cast<float*>(smem + C::STAGE_BYTES) + rwave * WSTR;
    float* const xml = xo + (KP - 1) * NCH * 256;
    // Chunk c of its owner t, as handed over by part k != t.
    auto xchunk = [&](int t, int k, int c) {
      return reinterpret_cast<f32x4*>(xo + (((t * (KP - 1) + (k < t ? k : k - 1)) * CPS + c % CPS) * 64 + lane) * 4);
    };
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int db = 0; db < A::DB; ++db) agpr_fence<A::AG>(st.oacc[db][qb]);
#pragma unroll
    for (int t = 0; t < KP; ++t)
      if (kset != t)
#pragma unroll
        for (int c = t * CPS; c < (t + 1) * CPS; ++c) {
          const f32x16& o = st.oacc[(c / 4) % A::DB][c / (4 * A::DB)];
          const int g4 = c % 4;
          *xchunk(t, kset, c) = f32x4{o[4 * g4], o[4 * g4 + 1], o[4 * g4 + 2], o[4 * g4 + 3]};
        }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      xml[(kset * 2 * QB + qb) * 64 + lane] = st.m_run[qb];
      xml[(kset * 2 * QB + QB + qb) * 64 + lane] = st.l_run[qb];
    }
    __syncthreads();  // with the wait for this wave's LDS writes
    constexpr int RB = DV * 2, WROWS = 32 * QB;
    unsigned char* const tile = smem + rwave * WROWS * RB;
    const int osw = o_swizzle<DV>(st.i32) << 4, ohalf = (st.h ^ o_half<DV>(st.i32)) << 3;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      float w[KP], l = 0.f, m = -INFINITY;
#pragma unroll
      for (int k = 0; k < KP; ++k) {
        w[k] = xml[(k * 2 * QB + qb) * 64 + lane];
        m = fmaxf(m, w[k]);
      }
#pragma unroll
      for (int k = 0; k < KP; ++k) {
        w[k] = w[k] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(w[k] - m);
        l += xml[(k * 2 * QB + QB + qb) * 64 + lane] * w[k];
      }
      const float l_tot = half_swap_sum(l);
      const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
      unsigned char* const srow = tile + (qb * 32 + st.i32) * RB + ohalf;
#pragma unroll
      for (int t = 0; t < KP; ++t)
        if (kset == t)
#pragma unroll
          for (int c = t * CPS; c < (t + 1) * CPS; ++c) {
            if (c / (4 * A::DB) != qb) continue;
            const f32x16& own = st.oacc[(c / 4) % A::DB][qb];
            f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < KP; ++k) {
              const int g4 = c % 4;
              const f32x4 ok = k == t ? f32x4{own[4 * g4], own[4 * g4 + 1], own[4 * g4 + 2], own[4 * g4 + 3]}
                                      : *xchunk(t, k, c);
#pragma unroll
              for (int e = 0; e < 4; ++e) o[e] = k == 0 ? ok[e] * w[k] : o[e] + ok[e] * w[k];
            }
            *reinterpret_cast<uint2*>(srow + (((c % (4 * A::DB)) << 4) ^ osw)) =
                make_uint2(pack_bf16x2(o[0] * inv, o[1] * inv), pack_bf16x2(o[2] * inv, o[3] * inv));
          }
      const int row = st.qw + qb * 32 + st.i32;
      if (p.lse != nullptr && kset == 0 && st.h == 0 && row < p.sq)
        p.lse[(size_t)(b * p.hq + hq) * p.sq + row] = l_tot > 0.f ? (m + log2f(l_tot)) * kLn2 : -INFINITY;
    }
    __syncthreads();
    constexpr int CPR = RB / 16, RPI = 64 / CPR, NIT = WROWS / RPI / KP;
    static_assert(NIT >= 1, "rows split over the sets");
    uint16_t* const ohead = p.o + (size_t)(b * p.hq + hq) * p.sq * DV;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int r = (kset * NIT + it) * RPI + lane / CPR, c = lane % CPR, row = st.qw + r;
      const unsigned char* chunk = tile + r * RB + ((c ^ o_swizzle<DV>(r)) << 4);
      const int hl = o_half<DV>(r) << 3;
      const uint2 x = *reinterpret_cast<const uint2*>(chunk + hl);
      const uint2 y = *reinterpret_cast<const uint2*>(chunk + (hl ^ 8));
      if (row < p.sq) *reinterpret_cast<u32x4*>(ohead + (size_t)row * DV + c * 8) = u32x4{x.x, x.y, y.x, y.y};
    }
    return;
  }

  // ---- epilogue: O = acc / l, LSE = ln 2 * (m + log2 l) ---------------------------------------
  if constexpr (C::SPLIT) {
    // Partial result of this part of the key range, for the merge pass: O normalised by this part's
    // row sum (fp32, 16 bytes per lane and block) and this part's LSE; an empty part gives O = 0 and
    // LSE = -inf, which the merge weighs with 0.
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int db = 0; db < A::DB; ++db) agpr_fence<A::AG>(st.oacc[db][qb]);
    const size_t head_rows = ((size_t)split * p.batch * p.hq + (size_t)b * p.hq + hq) * p.sq;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const float l_tot = half_swap_sum(st.l_run[qb]);
      const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
      const int row = st.qw + qb * 32 + st.i32;
      if (row < p.sq) {
        float* orow = p.o_part + (head_rows + row) * DV;
#pragma unroll
        for (int db = 0; db < A::DB; ++db)
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4)
            *reinterpret_cast<f32x4*>(orow + db * 32 + 8 * g4 + 4 * st.h) =
                f32x4{st.oacc[db][qb][4 * g4] * inv, st.oacc[db][qb][4 * g4 + 1] * inv,
                      st.oacc[db][qb][4 * g4 + 2] * inv, st.oacc[db][qb][4 * g4 + 3] * inv};
        if (st.h == 0) p.lse_part[head_rows + row] = l_tot > 0.f ? (st.m_run[qb] + log2f(l_tot)) * kLn2 : -INFINITY;
      }
    }
  } else {
    // O goes through LDS so that each store instruction writes whole rows (1 KiB contiguous); stored
    // straight from the accumulator layout, every instruction would touch 32 rows 16 bytes at a time.
    constexpr int RB = DV * 2;           // bytes per output row
    constexpr int WROWS = 32 * QB;       // rows per wave
    static_assert(C::RWAVES * WROWS * RB <= C::LDS_BYTES, "output staging fits in the ring slots");
    unsigned char* stage = smem + wave * WROWS * RB;
  #pragma unroll
    for (int qb = 0; qb < QB; ++qb)
  #pragma unroll
      for (int db = 0; db < A::DB; ++db) agpr_fence<A::AG>(st.oacc[db][qb]);
    {
      const int osw = o_swizzle<DV>(st.i32) << 4;             // qb * 32 leaves the low 5 row bits alone
      const int ohalf = (st.h ^ o_half<DV>(st.i32)) << 3;
  #pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const float l_tot = half_swap_sum(st.l_run[qb]);
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        unsigned char* srow = stage + (qb * 32 + st.i32) * RB + ohalf;
  #pragma unroll
        for (int db = 0; db < A::DB; ++db)
  #pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) {
            const int c = 4 * db + g4;  // 16-byte chunk: dims 8c .. 8c+7, this lane's half 4h .. 4h+3
            const uint32_t w0 = pack_bf16x2(st.oacc[db][qb][4 * g4] * inv, st.oacc[db][qb][4 * g4 + 1] * inv);
            const uint32_t w1 = pack_bf16x2(st.oacc[db][qb][4 * g4 + 2] * inv, st.oacc[db][qb][4 * g4 + 3] * inv);
            *reinterpret_cast<uint2*>(srow + ((c << 4) ^ osw)) = make_uint2(w0, w1);
          }
        const int row = st.qw + qb * 32 + st.i32;
        if (p.lse != nullptr && st.h == 0 && row < p.sq)
          p.lse[(size_t)(b * p.hq + hq) * p.sq + row] =
              l_tot > 0.f ? (st.m_run[qb] + log2f(l_tot)) * kLn2 : -INFINITY;
      }
    }
    // Each wave reads back only its own rows, so no barrier: LDS serves one wave's accesses in order.
    {
      constexpr int CPR = RB / 16;        // 16-byte chunks per row
      constexpr int RPI = 64 / CPR;       // rows per store instruction
      const int c = lane % CPR;
      uint16_t* ohead = p.o + (size_t)(b * p.hq + hq) * p.sq * DV;
      // All reads first, pinned before the stores as a group: the compiler would otherwise sink each
      // read into its store's row guard and wait out an LDS round trip per store.
      constexpr int NIT = WROWS / RPI;
      u32x4 ov[NIT];
  #pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int r = it * RPI + lane / CPR;
        const unsigned char* chunk = stage + r * RB + ((c ^ o_swizzle<DV>(r)) << 4);
        const int hl = o_half<DV>(r) << 3;
        const uint2 x = *reinterpret_cast<const uint2*>(chunk + hl);
        const uint2 y = *reinterpret_cast<const uint2*>(chunk + (hl ^ 8));
        ov[it] = u32x4{x.x, x.y, y.x, y.y};
      }
  #pragma unroll
      for (int it = 0; it < NIT; ++it) asm volatile("" : "+v"(ov[it]));
  #pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int row = st.qw + it * RPI + lane / CPR;
        if (row < p.sq) *reinterpret_cast<u32x4*>(ohead + (size_t)row * DV + c * 8) = ov[it];
      }
    }
  }
}

// Entry kernels. The instances with one workgroup per CU (long at d = 128 and 192, key quarters at d = 128)
// read everything from the argument block. Those with several workgroups per CU, whose workgroups are
// mostly short chains on which the first loads' latency is felt, take the values their prologue needs first
// as leading scalar arguments, which the command processor preloads into SGPRs before the first instruction
// (kernel-argument preloading, enabled at build time for the first 14 SGPRs of a kernel's leading
// scalar arguments), and issue their Q loads before they read the argument block. Preloading is kept
// off the long instance at d = 128: it slows the launch of each wave, and on the 128K
// workload the spread-out starts of the workgroups that stream one K/V head through an XCD's L2
// doubled the L2 misses, at no gain in time. At d = 64 the long instance takes it for having two workgroups
// per CU, though its work order reads the chunks of heads from the argument block before the Q loads:
// preloaded or not measured level (26 shapes of 1 025 to 4 000 blocks, 0.98-1.01x, mean 1.00x).
template <class C>
__global__ __attribute__((amdgpu_flat_work_group_size(C::NT, C::NT), amdgpu_waves_per_eu(C::WPE, C::WPE)))
void fa_fwd_kernel(FwdParams p) {
  fa_fwd_body<C>(p, WorkMap{p.group >> ((p.shifts >> 18) & 3u), p.hkv, p.batch, p.n_qtiles, p.full, p.m_group, p.m_hkv,
                            p.m_batch, p.shifts});
}
template <class C>
__global__ __attribute__((amdgpu_flat_work_group_size(C::NT, C::NT), amdgpu_waves_per_eu(C::WPE, C::WPE)))
void fa_fwd_kernel_preload(const uint16_t* a_q, int a_sq, int a_sk, int a_hq, int a_batch, int a_hkv, int a_group,
                           int a_nqt, int a_full, uint32_t a_mg, uint32_t a_mh, uint32_t a_mb, uint32_t a_shifts,
                           FwdParams p) {
  p.q = a_q;
  p.sq = a_sq;
  p.sk = a_sk;
  p.hq = a_hq;
  p.batch = a_batch;
  p.hkv = a_hkv;
  p.group = a_group;
  p.n_qtiles = a_nqt;
  fa_fwd_body<C>(p, WorkMap{a_group >> ((a_shifts >> 18) & 3u), a_hkv, a_batch, a_nqt, a_full, a_mg, a_mh, a_mb,
                            a_shifts});
}

// The instances. Long: 4 waves x 64 query rows (256 row-heads per workgroup), one workgroup per CU,
// one wave per SIMD (at d = 64 two, in 32-key tiles: Instance<64, 64> below); the register budget of a wave (O 128 + Q 64 AGPRs at d = 128, two score tiles
// and P in VGPRs) is what fixes 64 query rows per wave. K tiles are loaded two ahead: a third K slot
// measured 2-3 % slower on the 8K, 4K-d192 and 128K prefill shapes (one box, interleaved).
// Short: 4 waves x 32 query rows (128 row-heads per workgroup), two workgroups per CU (two waves per SIMD,
// 256 registers each, O and Q in VGPRs), shallower fragment prefetch at d = 128 so that the step fits
// the registers without spilling, and a V ring of 3 slots at d = 128 (so that two rings fit one CU's
// LDS) and 4 at d = 64 (V tiles loaded two steps ahead; 3-8 % faster than 3 slots on the d = 64
// shapes it runs, while a deeper K ring measured slower). It
// runs problems with few query blocks (short sequences, few heads), where 256-row blocks leave CUs
// idle and each block's serial chain of steps sets the time: on the paper's S = 512 and 2048 GPT-2
// and BERT shapes and the 128K single-head workload it measured 1.2-1.4x faster than the long
// instance, and slower once the long instance's grid fills the GPU. Split mode runs it by a rule of its
// own (split_short). At d_qk = 192 two waves per SIMD
// do not fit, so those problems always run the long instance.
#ifndef FA_BN
#define FA_BN 64
#endif
#ifndef FA_NWAVES
#define FA_NWAVES 4
#endif
#ifndef FA_QB
#define FA_QB 2
#endif
#ifndef FA_KPF
#define FA_KPF 2
#endif
#ifndef FA_VPF
#define FA_VPF 6
#endif
#ifndef FA_NKR
#define FA_NKR 2
#endif
#ifndef FA_NVR
#define FA_NVR 4
#endif

template <int DQK, int DV, bool CAUSAL, bool SPLIT = false>
struct Instance {
  using C = Cfg<DQK, DV, FA_BN, FA_NWAVES, FA_QB, CAUSAL, SPLIT, 1, FA_KPF, FA_VPF, FA_NKR, FA_NVR>;
};
// The long instance at d = 64: the same 256-row blocks in 32-key tiles, two workgroups per CU. At d = 64
// every MFMA comes with 9 full-rate-equivalent VALU instructions of softmax (36 cycles against its own
// 32), which one wave per SIMD serialises behind it (measured 49 cycles a slot against 44 with two
// waves). A wave's 64 rows with 32 keys need O 64, Q 32, two score tiles 64 and P 32 registers, so two
// waves per SIMD fit (218 VGPRs, no AGPR) and every K and V fragment still feeds two MFMAs. Measured
// against 64-key tiles with one wave per SIMD (interleaved, one box): GQA 14/2 S32768 causal 1892 ->
// 1782 us, H16 S32768 causal 2103 -> 1978, B8 H12 S4096 412 -> 380, B8 H16 S3000 causal 192 -> 167. A
// third K slot cost 5 %, reading K fragments 1 ahead 1.5 %, key halves on 64-key tiles 2-6 %. Split mode
// keeps the 64-key tiles: its grids of about one workgroup per CU measured 0.74-1.08x with these.
template <bool CAUSAL>
struct Instance<64, 64, CAUSAL, false> {
  using C = Cfg<64, 64, 32, 4, 2, CAUSAL, false, 2, 2, 4, 2, 4>;
};
template <int DQK, int DV, bool CAUSAL, bool SPLIT = false>
struct ShortInstance {
  using C = Cfg<DQK, DV, 64, 4, 1, CAUSAL, SPLIT, 2, DQK >= 128 ? 1 : 2, DQK >= 128 ? 2 : 6, 2, DQK >= 128 ? 3 : 4>;
};
// The short instance at d = 64 with 128-key tiles, for keys of at least kWideTileKeys: a step then
// carries 32 MFMAs per wave instead of 16, over which the per-step waits, barrier, load issue and
// addressing are spread (250 VGPRs; the 16 KiB tiles allow a V ring of 3 slots, 80 KiB per
// workgroup). Measured against the 64-key tiles (one box, interleaved): 1.5-6 % faster from 1 536
// keys on (BERT-Base and -Large S2048 1.05-1.06x, GPT-2 Small S8192 and S16384 1.02-1.03x), level at
// 1 024, 1.5 % slower at 512 keys (workload 2), where the four steps of a block leave too little to
// overlap with the pipeline's fill and drain.
template <int DQK, int DV, bool CAUSAL>
struct ShortWideInstance {
  using C = Cfg<DQK, DV, 128, 4, 1, CAUSAL, false, 2, 2, 6, 2, 3>;
};
constexpr int kWideTileKeys = 1024;
// Key halves: 4 waves as two sets of 2 x 32 query rows (64 row-heads per workgroup), each set taking
// one 32-key half of every tile; three workgroups per CU at d = 64 (three waves per SIMD, 132 VGPRs,
// 48 KiB of LDS each), two at d = 128 (208 VGPRs, 80 KiB). It runs problems whose grid of long-
// instance blocks is small enough that each workgroup's chain of steps sets the time: the chain
// keeps its number of steps but each step carries half the work per wave. V fragments are read 4
// ahead at d = 64 and 2 at d = 128, the best of 2-8 measured (one box, interleaved).
template <int DQK, int DV, bool CAUSAL>
struct HalfInstance {
  using C = Cfg<DQK, DV, 64, 4, 1, CAUSAL, false, DQK >= 128 ? 2 : 3, 2, DQK >= 128 ? 2 : 4, 2, DQK >= 128 ? 3 : 4, 2>;
};

// Key quarters: the 4 waves share 32 query rows and each takes one 32-key quarter of every 128-key tile
// (the merge takes the four parts' results). Half the steps of the key halves at the same work per wave
// and step, but every workgroup reads each K/V tile for 32 rows only, so it is for grids that leave CUs
// idle, where nothing but the length of a chain counts: there a step takes 350-600 ns whatever it
// computes (waits, barrier, LDS and MFMA latency with one wave per SIMD). Two workgroups per CU at
// d = 64 (80 KiB of LDS), one at d = 128 (160 KiB).
template <int DQK, int DV, bool CAUSAL>
struct QuarterInstance {
  using C = Cfg<DQK, DV, 128, 4, 1, CAUSAL, false, DQK >= 128 ? 1 : 2, 2, DQK >= 128 ? 2 : 4, 2, 3, 4>;
};

constexpr int64_t kCus = 256;  // compute units of MI355X

// Whether a problem of the key-halves instance runs the quarters: its 32-row workgroups are at most one
// per CU. Measured against the halves (interleaved, one box): d = 64 one head S256 5.15 -> 4.62 us, H12
// S512 causal 6.48 -> 5.37, H8 S1024 9.1 -> 6.8, 16/2 100 x 16384 97 -> 57; d = 128 H8 S1024 12.3 -> 10.6,
// 4 heads 333 x 999 12.1 -> 9.8, 16/2 100 x 16384 142 -> 83; at 320 workgroups 0.68-0.95x at d = 128
// and level at d = 64. Twice as many where the causal triangle makes the second half of the grid short
// (at least half as many rows as keys): d = 64 H16 S1024 9.3 -> 7.6, H4 S4096 26.3 -> 19.4 (at 640 0.85x
// at S1024); d = 128 from 2048 keys on, H8 S2048 level, H4 S4096 35.4 -> 30.4, one head S16384 145 -> 98
// (512 workgroups at S1024 0.83x). Up to 64 keys at d = 64 (0.92x) and 256 at d = 128 (0.85-1.00x) the
// four-way merge costs more than the one or two steps saved.
bool key_quarters(const FwdParams& p, int d_qk, bool causal) {
  const int64_t wgs = (int64_t)p.batch * p.hq * ((p.sq + 31) / 32);
  const bool triangle = causal && (int64_t)p.sq * 2 >= p.sk;
  if (d_qk == 64) return p.sk > 64 && wgs <= (triangle ? 2 * kCus : kCus);
  return p.sk > 256 && wgs <= (triangle && p.sk >= 2048 ? 2 * kCus : kCus);
}

// Largest grid of long-instance blocks (256 row-heads) that runs the short instance instead. At
// d = 128 the CU count of MI355X, where the long instance would leave CUs idle. At d = 64 the line comes
// from the long instance's earlier form with one wave per SIMD (short 5-17 % faster at 384-768 blocks, level
// at 1024-1152). Against its present form (32-key tiles, two waves per SIMD; 110 random shapes, causal and
// not, interleaved) the short instance takes 0.51-0.99 of the long one's time up to 512 blocks (five shapes
// 1.02-1.08). From there it is a matter of padding: 0.52-0.97 up to 1024 where the long blocks pad over 1.05
// times the short ones' rows, else 0.86-1.07 up to 704 blocks and 0.88-1.21 from 768 on (13 of 20 shapes
// above 1.01; 16 heads B5 3031 x 3031 207 us against 188), and above 1024 likewise 0.53-1.11 and 0.78-1.15.
// So a count of blocks fits neither side alone; 1024 lies where equal padding has mostly turned.
constexpr int64_t kShortMaxBlocks64 = 1024, kShortMaxBlocks128 = 256;
// Largest grid of such blocks that runs the key-halves instance, by head dimension and masking.
// Causal problems have a longest chain of steps (the last query block's) that halving each step's
// work per wave shortens; problems without a mask gain only while the grid leaves SIMDs idle. At
// d = 128 causal grids of 256 blocks measured 0.96-1.06x against the short instance (the paper's
// Llama S = 2048 shapes on the slow side), so they stay with it. Measured again with the merge by all wave
// sets (88 random shapes around the four lines): below them the short instance takes 1.0-1.3 times the
// halves' time, but for short sequences at the line itself (0.76-0.95: 24/12 heads B8 165 x 165), above them
// 0.84-1.06 (0.86-1.25 at d = 64).
constexpr int64_t kHalfMaxCausal64 = 320, kHalfMaxFull64 = 64, kHalfMaxCausal128 = 192, kHalfMaxFull128 = 128;

enum class Kind { kLong, kShort, kShortWide, kHalf, kQuarter };

// By the grid alone: kHalf stands for both key-parts instances and kShort for both tile widths.
Kind pick_instance(const FwdParams& p, int d_qk, int d_v, bool causal) {
  if (!((d_qk == 64 && d_v == 64) || (d_qk == 128 && d_v == 128))) return Kind::kLong;
  const int bm = Instance<64, 64, false>::C::BM;
  const int64_t blocks = (int64_t)p.batch * p.hq * ((p.sq + bm - 1) / bm);
  const int64_t half_max = d_qk == 64 ? (causal ? kHalfMaxCausal64 : kHalfMaxFull64)
                                      : (causal ? kHalfMaxCausal128 : kHalfMaxFull128);
  if (blocks <= half_max) return Kind::kHalf;
  return blocks <= (d_qk == 64 ? kShortMaxBlocks64 : kShortMaxBlocks128) ? Kind::kShort : Kind::kLong;
}

// log2 of the query heads a workgroup of `nwaves` waves packs: 4, 2 or 1 heads, the largest that
// divides the GQA group size (and the wave count).
int packed_heads_log2(int group, int nwaves) {
  if (group % 4 == 0 && nwaves % 4 == 0) return 2;
  if (group % 2 == 0 && nwaves % 2 == 0) return 1;
  return 0;
}

// Workgroups and padded query rows per head of an instance whose workgroups hold `rowheads` row-heads in
// `rwaves` waves with rows of their own (launch_cfg's decomposition).
struct Grid {
  int64_t wgs, rows;
};
Grid grid_of(const FwdParams& p, int rowheads, int rwaves) {
  const int hw_log = packed_heads_log2(p.group, rwaves);
  const int64_t rows = rowheads >> hw_log, blocks = (p.sq + rows - 1) / rows;
  return {(int64_t)p.batch * p.hkv * (p.group >> hw_log) * blocks, blocks * rows};
}

// pick_instance, except where the keys are more than twice the query rows (a chunk of a prompt against its
// cache). Such a grid is flat, its chains are about equally long with or without the mask, so what a causal
// triangle gains from small blocks (a shorter longest chain) is not there, and blocks with more rows read
// each K/V fragment for more of them. That pays only where the larger blocks still fill the chip and pad no
// more rows, so the rule counts the workgroups and padded rows that each instance would launch (the blocks
// of pick_instance count neither a GQA group's packing nor padding). Measured over 530 random shapes of 160
// to 256 blocks at d = 128 and 201 to 320 at d = 64, each in every instance (us, interleaved, one box):
//  * d = 128, the short instance's grid exceeds a workgroup per CU: from the halves (causal, up to 192
//    blocks) to the short instance, unless it pads over a seventh more rows: 8/8 8 x 537 x 3786 0.84x the
//    time, 16/16 4 x 550 x 17276 0.73x, 15/5 4 x 706 x 2486 0.93x; at 1.2 times the rows 32/32 3 x 299 x
//    2260 1.27x. At or below a workgroup per CU it leaves CUs idle: 32/8 5 x 61 x 12957 1.17x.
//  * d = 128, on to the long instance where that pads at most an eighth more rows again and the grid is
//    flat enough (no mask, or six times as many keys): 20 heads 2000 x 20000 483 -> 402, 32/8 1500 x 9000
//    208 -> 194, 16/16 16 x 229 x 3760 196 -> 120, without a mask 16 heads 2560 x 8000 179 -> 161. With more
//    padding it is slower (28/4 2 x 777 x 5001, 1024 rows for 896: 118.5 against 114.5 in the short
//    instance, 64/16 3 x 154 x 5481 1.20x), with fewer keys per row too (64/8 770 x 3013 1.05x), and with
//    idle CUs most of all (B4 64/8 1 x 3454, a grid of 64: 1.29x, 35/5 5 x 1 x 358: 2.3x). Grids without a
//    mask are flat with fewer keys as well (9 heads 5000 x 5000 123 against 112 in the long instance, 24
//    heads 2048 x 2048 55.5 against 51.9); they stay with the grid's choice.
//  * d = 64 (causal, halves): to the short instance where its grid takes one and a half to two workgroups
//    per CU and it pads at most a tenth more rows, a fifth from seven quarters per CU on: 16 heads 4000 x
//    16000 268 -> 246, 12 heads 2 x 2500 x 10000 170 -> 151, 9/9 4 x 1363 x 31199 0.71x, 5/5 32 x 303 x
//    11131 (1.2 times the rows, 480 workgroups) 0.66x; at 1.11 times the rows in 400 workgroups 16/16 5 x
//    528 x 6548 1.09x, at 4/3 1.10-1.21x, grids of 257 to 384 1.00-1.13x, above 512 0.84-1.11x. Of
//    at most a workgroup per CU: where the halves need more than that (16/2 16 x 73 x 22765 0.80x, 56/8 4 x
//    76 x 1996 0.95x), or K and V are too large to be read twice as often (above 80 MiB: 32/8 8 x 51 x 27897
//    0.75x, 8/8 32 x 42 x 6307 0.85x; below, 32/8 8 x 48 x 588 1.13x). Problems of the key quarters stay
//    there (the short instance 1.3-1.9x).
constexpr int64_t kFlatMin128 = 160, kFlatMin64 = 201;  // blocks
Kind pick_launch(const FwdParams& p, int d_qk, int d_v, bool causal) {
  const Kind kind = pick_instance(p, d_qk, d_v, causal);
  if (kind == Kind::kLong || p.sk <= (int64_t)p.sq * 2) return kind;
  const int64_t blocks = (int64_t)p.batch * p.hq * ((p.sq + 255) / 256);
  if (blocks < (d_qk == 128 ? kFlatMin128 : kFlatMin64)) return kind;
  const Grid lng = grid_of(p, 256, 4), sht = grid_of(p, 128, 4), hlf = grid_of(p, 64, 2);
  if (d_qk == 128) {
    if (sht.wgs <= kCus || (kind == Kind::kHalf && 7 * sht.rows > 8 * hlf.rows)) return kind;
    const bool flat = !causal || p.sk >= (int64_t)p.sq * 6;
    return flat && 8 * lng.rows <= 9 * sht.rows ? Kind::kLong : Kind::kShort;
  }
  if (kind != Kind::kHalf || key_quarters(p, d_qk, causal)) return kind;
  const bool short_fits = 10 * sht.rows <= (4 * sht.wgs >= 7 * kCus ? 12 : 11) * hlf.rows;
  if (sht.wgs <= kCus) {
    const bool large_kv = 2.0 * p.batch * p.hkv * p.sk * (d_qk + d_v) > 80.0 * (1 << 20);
    return (short_fits && hlf.wgs > kCus) || large_kv ? Kind::kShort : kind;
  }
  return short_fits && 2 * sht.wgs > 3 * kCus && sht.wgs <= 2 * kCus ? Kind::kShort : kind;
}

template <class C>
hipError_t launch_cfg(FwdParams p, hipStream_t stream) {
  const int hw_log = packed_heads_log2(p.group, C::RWAVES);
  const int gi = p.group >> hw_log;  // workgroups per key/value head and query block
  const int bmr = (C::RWAVES >> hw_log) * 32 * C::QB;
  p.n_qtiles = (p.sq + bmr - 1) / bmr;
  p.n_wg = p.batch * p.hkv * gi * p.n_qtiles;
  const int span = kNumXcd * gi;
  p.full = (p.n_wg / span) * span;
  const FastDiv fg = make_fastdiv(gi), fh = make_fastdiv(p.hkv), fb = make_fastdiv(p.batch);
  p.m_group = fg.m;
  p.m_hkv = fh.m;
  p.m_batch = fb.m;
  p.shifts = fg.sh | fh.sh << 6 | fb.sh << 12 | (uint32_t)hw_log << 18;
  // Large grids run their key/value heads in chunks, one after the other, the query blocks of a chunk
  // heaviest first: the workgroups of an XCD then share a few heads' K and V through its L2 and the
  // Infinity Cache instead of streaming every head at once. A chunk is the fewest heads, a multiple of
  // the XCD count (so that a head stays on one XCD), that give every workgroup slot of an XCD two items
  // when causal, one otherwise; the last chunk takes the rest, at least a whole chunk's heads, so that
  // the light blocks of several heads still fill the end of the grid. Measured (interleaved, one box):
  // H128 S4096 192/128 causal 647 -> 615 us (chunks of 32 heads; 16: 629, 8: 644), without a mask
  // 1181 -> 1060, B4 H32 S4096 d128 causal 525 -> 510, without 923 -> 875, B16 H32 S512 91.7 -> 88.1.
  // (The smaller chunks' times hold their smaller last chunk too, whose heads then fill less of the end.)
  // Fewer than four chunks stay in one: H16 S32768 d64 causal measured 1.4 % slower in two.
  p.head_chunk = p.batch * p.hkv;
  p.head_chunked = 0;
  if constexpr (C::CHUNKED && !C::SPLIT) {
    const int64_t heads = (int64_t)p.batch * p.hkv, items = (int64_t)gi * p.n_qtiles;
    const int64_t want = (int64_t)(C::CAUSAL ? 2 : 1) * C::OCC * kCusPerXcd;
    const int64_t chunk = kNumXcd * ((want + items - 1) / items);
    if (heads >= 4 * chunk) {
      p.head_chunk = (int)chunk;
      p.head_chunked = (int)((heads - chunk) / chunk * chunk);
    }
  }
  const dim3 grid(p.n_wg * (C::SPLIT ? p.n_split : 1));
  if constexpr (C::OCC > 1) {
    void* args[] = {&p.q,        &p.sq,   &p.sk,      &p.hq,    &p.batch,   &p.hkv,    &p.group,
                    &p.n_qtiles, &p.full, &p.m_group, &p.m_hkv, &p.m_batch, &p.shifts, &p};
    return hipLaunchKernel(reinterpret_cast<const void*>(&fa_fwd_kernel_preload<C>), grid, dim3(C::NT), args, 0,
                           stream);
  } else {
    void* args[] = {&p};
    return hipLaunchKernel(reinterpret_cast<const void*>(&fa_fwd_kernel<C>), grid, dim3(C::NT), args, 0, stream);
  }
}

// Whether a split-mode problem runs the short instance: its blocks of 128 row-heads pad the query rows to
// fewer than the long instance's 256, or the long instance's grid leaves CUs idle. Split mode has few query
// rows, so most of a block can be padding. Measured, long against short (interleaved, one box, d = 128
// causal): 28/4 heads 100 x 20001 (padded to 256 rows against 128) 79.9 -> 57.5 us, 16/16 100 x 32768 83.3
// -> 67.0, 16/16 300 x 16384 (512 against 384) 86.6 -> 75.3, 32/8 16 x 32768 (64 against 32 rows of four
// heads) 49.3 -> 40.3, 32/8 64 x 32768 (equal, long grid of 128) 58.0 -> 53.4; d = 64 12/12 90 x 8192 18.6
// -> 14.5. With equal padding on a full grid the long instance reads each fragment for twice the rows:
// 32/8 100 x 32768 75.3 against 78.8, 8/1 500 x 131072 253 against 274.
bool split_short(const FwdParams& p) {
  const Grid lng = grid_of(p, 256, 4), sht = grid_of(p, 128, 4);
  if (sht.wgs * p.n_split > INT32_MAX) return false;
  return sht.rows < lng.rows || lng.wgs * p.n_split < kCus;
}

// The instance a launch runs (every kind, and split mode's own choice).
Kind launch_kind(const FwdParams& p, int d_qk, int d_v, bool causal, bool split) {
  if (split) return d_qk != 192 && split_short(p) ? Kind::kShort : Kind::kLong;
  const Kind kind = pick_launch(p, d_qk, d_v, causal);
  if (kind == Kind::kHalf && key_quarters(p, d_qk, causal)) return Kind::kQuarter;
  if (kind == Kind::kShort && d_qk == 64 && p.sk >= kWideTileKeys) return Kind::kShortWide;
  return kind;
}

template <int DQK, int DV, bool CAUSAL, bool SPLIT>
hipError_t launch_instance(FwdParams p, Kind kind, hipStream_t stream) {
  if constexpr (!SPLIT && DQK != 192) {
    if (kind == Kind::kQuarter) return launch_cfg<typename QuarterInstance<DQK, DV, CAUSAL>::C>(p, stream);
    if (kind == Kind::kHalf) return launch_cfg<typename HalfInstance<DQK, DV, CAUSAL>::C>(p, stream);
  }
  if constexpr (!SPLIT && DQK == 64) {
    if (kind == Kind::kShortWide) return launch_cfg<typename ShortWideInstance<DQK, DV, CAUSAL>::C>(p, stream);
  }
  if constexpr (DQK != 192) {
    if (kind == Kind::kShort) return launch_cfg<typename ShortInstance<DQK, DV, CAUSAL, SPLIT>::C>(p, stream);
  }
  return launch_cfg<typename Instance<DQK, DV, CAUSAL, SPLIT>::C>(p, stream);
}

template <bool SPLIT>
hipError_t launch_dims(FwdParams p, int d_qk, int d_v, bool causal, hipStream_t stream) {
  const Kind sh = launch_kind(p, d_qk, d_v, causal, SPLIT);
  if (d_qk == 64 && d_v == 64)
    return causal ? launch_instance<64, 64, true, SPLIT>(p, sh, stream)
                  : launch_instance<64, 64, false, SPLIT>(p, sh, stream);
  if (d_qk == 128 && d_v == 128)
    return causal ? launch_instance<128, 128, true, SPLIT>(p, sh, stream)
                  : launch_instance<128, 128, false, SPLIT>(p, sh, stream);
  if (d_qk == 192 && d_v == 128)
    return causal ? launch_instance<192, 128, true, SPLIT>(p, sh, stream)
                  : launch_instance<192, 128, false, SPLIT>(p, sh, stream);
  return hipErrorInvalidValue;
}

// Merge of the n_split partial results of every query row (log-sum-exp combination): with
// M = max_s LSE_s, w_s = exp(LSE_s - M), O = sum_s w_s O_s / sum_s w_s and LSE = M + ln(sum_s w_s).
// A row whose parts are all empty (LSE_s = -inf) gets O = 0 and LSE = -inf. A row is handled by
// DV / 4 * pg threads: thread (g, q) takes output dims 4q .. 4q+3 of the parts s = g (mod pg), so the
// loads of a row are independent and in flight together; the pg partial maxima, weighted sums and
// weight sums are combined through LDS. pg is the smallest power of two >= n_split, at most
// 256 / (DV / 4); a workgroup of 256 threads takes 256 / (DV / 4 * pg) rows. Reads fp32, writes bf16
// (round to nearest even) and the fp32 LSE.
template <int DV>
__global__ __launch_bounds__(256) void fa_merge_kernel(MergeParams p, int pg) {
  constexpr int TD = DV / 4;     // threads per part group (one per 4 output dims)
  constexpr int NG = 256 / TD;   // part groups per workgroup
  __shared__ float s_m[NG], s_den[NG];
  __shared__ f32x4 s_acc[NG][TD];
  const int q = threadIdx.x % TD, gw = threadIdx.x / TD;  // group within the workgroup
  const int g = gw % pg;                                  // part group within the row
  const int64_t row = (int64_t)blockIdx.x * (NG / pg) + gw / pg;
  const bool live = row < p.rows;
  const int g0 = gw - g;                                  // first group of this row
  float m = -INFINITY;
  if (live)
    for (int sp = g; sp < p.n_split; sp += pg) m = fmaxf(m, p.lse_part[sp * p.rows + row]);
  if (q == 0) s_m[gw] = m;
  __syncthreads();
  float M = -INFINITY;
  for (int k = 0; k < pg; ++k) M = fmaxf(M, s_m[g0 + k]);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float den = 0.f;
  if (live && M != -INFINITY) {
    for (int sp = g; sp < p.n_split; sp += pg) {
      const float w = expf(p.lse_part[sp * p.rows + row] - M);
      den += w;
      acc += w * *reinterpret_cast<const f32x4*>(p.o_part + (sp * p.rows + row) * DV + 4 * q);
    }
  }
  s_acc[gw][q] = acc;
  if (q == 0) s_den[gw] = den;
  __syncthreads();
  if (live && g == 0) {
    float dsum = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < pg; ++k) {
      dsum += s_den[g0 + k];
      o += s_acc[g0 + k][q];
    }
    o *= dsum > 0.f ? 1.f / dsum : 0.f;
    f32x2 lo = {o.x, o.y}, hi = {o.z, o.w};
    *reinterpret_cast<uint2*>(p.o + row * DV + 4 * q) =
        make_uint2(bit_cast<uint32_t>(__builtin_convertvector(lo, bf16x2)),
                   bit_cast<uint32_t>(__builtin_convertvector(hi, bf16x2)));
    if (q == 0 && p.lse != nullptr) p.lse[row] = dsum > 0.f ? M + logf(dsum) : -INFINITY;
  }
}

}  // namespace

int block_rows(int d_qk, int d_v, bool causal) {
  (void)causal;
  if (d_qk == 64 && d_v == 64) return Instance<64, 64, false>::C::BM;
  if (d_qk == 128 && d_v == 128) return Instance<128, 128, false>::C::BM;
  if (d_qk == 192 && d_v == 128) return Instance<192, 128, false>::C::BM;
  return 0;
}

int instance_rows(int batch, int hq, int sq, int d_qk, int d_v, bool causal) {
  const int bm = block_rows(d_qk, d_v, causal);
  if (bm == 0 || batch < 0 || hq < 0 || sq < 0) return 0;
  FwdParams p{};
  p.batch = batch;
  p.hq = hq;
  p.sq = sq;
  switch (pick_instance(p, d_qk, d_v, causal)) {
    case Kind::kHalf:
      return HalfInstance<64, 64, false>::C::BM;
    case Kind::kShort:
      return ShortInstance<64, 64, false>::C::BM;
    default:
      return bm;
  }
}

int launch_instance_id(int batch, int hq, int hkv, int sq, int sk, int d_qk, int d_v, bool causal, int n_split) {
  if (block_rows(d_qk, d_v, causal) == 0 || batch <= 0 || hq <= 0 || hkv <= 0 || hq % hkv != 0 || sq <= 0 || sk < 0 ||
      n_split < 0)
    return 0;
  FwdParams p{};
  p.batch = batch;
  p.hq = hq;
  p.hkv = hkv;
  p.group = hq / hkv;
  p.sq = sq;
  p.sk = sk;
  p.n_split = n_split;
  switch (launch_kind(p, d_qk, d_v, causal, n_split > 0)) {
    case Kind::kQuarter:
      return 1;
    case Kind::kHalf:
      return 2;
    case Kind::kShort:
      return 3;
    case Kind::kShortWide:
      return 4;
    default:
      return 5;
  }
}

int64_t forward_workgroups(int batch, int hq, int hkv, int sq) {
  // the long instance's grid (the other instances of the fused forward run at most 2 048 workgroups; split
  // mode's short one checks its own)
  using C = Instance<64, 64, false>::C;
  const int group = hq / hkv, hw_log = packed_heads_log2(group, C::RWAVES);
  const int64_t bmr = (C::NWAVES >> hw_log) * 32 * C::QB;
  return (int64_t)batch * hkv * (group >> hw_log) * ((sq + bmr - 1) / bmr);
}

hipError_t launch_forward(FwdParams p, int d_qk, int d_v, bool causal, hipStream_t stream) {
  return launch_dims<false>(p, d_qk, d_v, causal, stream);
}

hipError_t launch_merge(MergeParams m, int d_v, hipStream_t stream) {
  const int groups = 256 / (d_v / 4);
  int pg = 1;
  while (pg < m.n_split && pg < groups) pg *= 2;
  const int64_t rows_per_wg = groups / pg;
  const dim3 grid((unsigned)((m.rows + rows_per_wg - 1) / rows_per_wg));
  void* args[] = {&m, &pg};
  const void* k = d_v == 64 ? reinterpret_cast<const void*>(&fa_merge_kernel<64>)
                            : reinterpret_cast<const void*>(&fa_merge_kernel<128>);
  return hipLaunchKernel(k, grid, dim3(256), args, 0, stream);
}

hipError_t launch_forward_split(FwdParams p, int d_qk, int d_v, bool causal, hipStream_t stream) {
  const hipError_t e = launch_dims<true>(p, d_qk, d_v, causal, stream);
  if (e != hipSuccess) return e;
  MergeParams m;
  m.o_part = p.o_part;
  m.lse_part = p.lse_part;
  m.o = p.o;
  m.lse = p.lse;
  m.rows = (int64_t)p.batch * p.hq * p.sq;
  m.n_split = p.n_split;
  return launch_merge(m, d_v, stream);
}

}  // namespace fa
