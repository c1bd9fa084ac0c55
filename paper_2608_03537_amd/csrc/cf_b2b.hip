// Back-to-back attention kernel for gfx950 (Sec. IV, Eq. 2 with F = scaled
// softmax: P = softmax(scale Q K^T), O = P V) with the intermediate P kept in
// registers.
//
// Register hand-off between the two products.  The first product is computed
// in the transposed form S^T = K Q^T, so in each 32x32 accumulator block a
// lane holds one query row m and 16 of its key columns: rows
// 8*(i/4) + 4*g + i%4 of the block for element i, g = lane/32.  The second
// product (O^T = V^T P^T) consumes P^T as its B operand, where lane group g
// supplies 8 values of the contraction index per MFMA step; step s takes
// accumulator elements 8s .. 8s+7 of the lane, so P never leaves the
// registers of the wave that produced it (the register-resident S_tile of
// Sec. IV-A).  The k order inside a step is free as long as both operands use
// the same one: step s of block b is DEFINED to use
//     n1(s, g, j) = 32 b + 16 s + 8 (j/4) + 4 g + j%4,   j = 0..7,
// and the V operand is read from LDS as two 8-byte pieces per lane in that
// same order.
//
// Each wave owns 32 complete query rows, so the softmax statistics need only
// the lane pair (l, l^32) — no cross-wave or cross-workgroup exchange.
#include <algorithm>

#include "cf_gemm_tile.h"
#include "comfuse.h"

namespace cf {

// Accumulator elements 8s .. 8s+7 of a block, as 8 packed bf16.
__device__ __forceinline__ u32x4_t pack_step(const f32x16_t& v, int s) {
  return u32x4_t{pack_bf16x2(v[8 * s + 0], v[8 * s + 1]), pack_bf16x2(v[8 * s + 2], v[8 * s + 3]),
                 pack_bf16x2(v[8 * s + 4], v[8 * s + 5]), pack_bf16x2(v[8 * s + 6], v[8 * s + 7])};
}

// Transposing 8-byte LDS read (ds_read_b64_tr_b16) at LDS byte address
// addr + OFF, written as inline assembly.  The compiler builtin carries no
// memory operand, so the compiler's wait insertion assumes it may read bytes
// that an outstanding direct-to-LDS load is still writing and puts a wait for
// every such load (vmcnt(0)) in front of it.  The caller knows the stage it
// reads is not the one being loaded; it waits for the result itself
// (lgkm_wait), since the compiler does not know this instruction loads.
template <int OFF>
__device__ __forceinline__ u32x2_t ds_read_tr_b64(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset field");
  u32x2_t v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(OFF));
  return v;
}
// 16-byte LDS read at byte address addr + OFF as inline assembly, for the
// same reason (K rows sit in a stage that direct loads also write); the
// caller waits for the result.
template <int OFF>
__device__ __forceinline__ u32x4_t ds_read_b128_at(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset field");
  u32x4_t v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(OFF));
  return v;
}
// Wait until at most N LDS operations of this wave are outstanding; v is tied
// to the wait so that its uses cannot move above it.  The count is exact only
// while no scalar memory load is in flight (they share the counter and return
// out of order): the kernel's loop issues none, and each step begins with a
// full wait (lds_sync).
template <int N>
__device__ __forceinline__ void lgkm_wait(u32x4_t& v) {
  asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(v) : "i"(N));
}
// Calls f(std::integral_constant<int, I>) for I = B .. E-1 in order.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

__device__ __forceinline__ float lane_pair_sum(float v) { return v + __shfl_xor(v, 32); }
__device__ __forceinline__ float lane_pair_max(float v) { return fmaxf(v, __shfl_xor(v, 32)); }

// ===========================================================================
// Attention: O = softmax(scale * Q K^T) V per (batch*head), online softmax.
// 4 waves x 32 queries = 128 queries per workgroup; key/value blocks of 64.
// Q fragments stay in registers for the whole sweep.  Per block j:
//   S^T = K Q^T (K rows from LDS); lane-local row max / sum over its 32
//   values + the lane pair; P = exp2(S*scale*log2e - m); O = O*corr + P V
//   with P fed from registers and V^T rows from LDS.
// Two workgroups share a CU (at most 256 VGPRs per wave), so each SIMD runs
// two waves of different workgroups, which no barrier holds in step: one
// wave's softmax overlaps the other's MFMAs (the PingPong of Sec. III-C across
// waves rather than inside one).
// The running maximum is raised lazily: O and the row sum are rescaled only
// when a block's maximum exceeds the one in use by more than 2^8, so
// exp2(s - m) <= 256 and the common case skips the rescale; the final O / l
// uses the same maximum throughout, so the result is unchanged.
// K and V blocks arrive by wave-wide direct loads, both key-major; the
// second product reads V^T fragments with transposing LDS reads.
//
// Key groups.  QG waves own 32 queries each; KS groups of QG waves share the
// same queries and take the key blocks in turn (block j belongs to group
// j % KS), each group with a ring of its own, and their (maximum, sum, O)
// merge through LDS at the end.  With KS = 1 and QG = 4 a CU needs two
// workgroups to give every SIMD two waves and to keep enough bytes in flight;
// few queries (a decoding step, short batches) do not make that many, and
// each workgroup's key loop is then a serial chain.  See attention_form.
//
// Split keys.  With few workgroups even so, gridDim.z of them share a query
// block, each with a contiguous part of the key blocks; each publishes its partial
// (m, l, O) in the workspace and the last to finish merges them in order.
// ===========================================================================
template <int D, int QG_, int KS_, int BK_>
struct AttnShape {
  static constexpr int QG = QG_, KS = KS_;
  static constexpr int NW = QG * KS, NT = 64 * NW;
  static constexpr int TM = 32 * QG, TN = BK_;
  static constexpr int NH = TN / 32;              // 32-key halves of a block
  static constexpr int KB = TN * D * 2;           // K block bytes (TN rows of D*2 bytes)
  static constexpr int VB = TN * D * 2;           // V block bytes (TN rows of D*2 bytes)
  static constexpr int STAGE = KB + VB;
  static constexpr int LDS_RING = KS * 2 * STAGE;
  static constexpr int OROW = D * 4 + 16;         // merge: one query's fp32 O
  static constexpr int LDS_OUT = KS == 1 ? TM * (D * 2 + 8) : NW * 32 * (OROW + 8) + 16;
  static constexpr int LDS = LDS_RING > LDS_OUT ? LDS_RING : LDS_OUT;
  static constexpr int DK = D / 16;               // MFMA k steps over d
  static constexpr int BD = D / 32;               // output blocks over d
  static constexpr int KROW = D * 2;              // bytes per K row
  static constexpr int KCH = KROW / 16;           // 16-byte chunks per K row
  static constexpr int NSA = NH * DK;             // MFMAs of one S^T block
  static constexpr int NSB = 2 * NH * BD;         // MFMAs of one P V block
  using Out = TileShape<bf16_t, 1, BD, 4, 1, 128, 0>;
  static_assert(D % 32 == 0 && D <= 128 && TN % 32 == 0, "head dim, key block");
  static_assert(KS > 1 || QG == 4, "the staged store of one key group covers 128 rows");
  static_assert(LDS <= 160 * 1024 && 2 * STAGE <= 65536, "LDS budget, ds offset field");
};

// Softmax state of one block for one lane (query row lane % 32).
struct SoftmaxStep {
  float bmax, corr;
  bool need;
  u32x4_t P[2][2];   // bf16 P^T fragments: [32-key half][MFMA step]
};

template <int D, int QG, int KS, int BK>
__global__ __launch_bounds__(64 * QG * KS, 2) void b2b_attention_kernel(B2BParams p) {
  using A = AttnShape<D, QG, KS, BK>;
  __shared__ __attribute__((aligned(16))) char smem[A::LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform
  const int lr = lane & 31, lg = lane >> 5;
  const int wq = KS == 1 ? wave : wave % QG, grp = KS == 1 ? 0 : wave / QG;   // query rows, key group
  // XCD-aware order: workgroups go round-robin over the 8 XCDs by linear id,
  // so linear id L runs on XCD L % 8.  Give each XCD a contiguous range of
  // (head, query block) pairs: the query blocks of one head then share that
  // XCD's L2 copy of the head's K and V instead of fetching it on all eight.
  const int nq = gridDim.x, T = gridDim.x * gridDim.y;
  const int L = blockIdx.x + nq * blockIdx.y;
  const int g = (T & 7) == 0 ? (L & 7) * (T >> 3) + (L >> 3) : L;
  const int bz = g / nq;
  const int m0 = (g % nq) * A::TM;
  const int Lk = p.N1;
  const bf16_t* Q = p.X + (int64_t)bz * p.sx;
  const bf16_t* Kp = p.W1 + (int64_t)bz * p.sw1;
  const bf16_t* Vp = p.W2 + (int64_t)bz * p.sw2;
  const float sl2 = p.mid_scale * 1.4426950408889634f;   // scale * log2(e), > 0
  const int NBall = (Lk + A::TN - 1) / A::TN;
  // key blocks [jb, je) of this workgroup
  const int jb = KS == 1 ? 0 : (int)((int64_t)NBall * blockIdx.z / gridDim.z);
  const int NB = KS == 1 ? NBall : (int)((int64_t)NBall * (blockIdx.z + 1) / gridDim.z);
  constexpr float kLazy = 8.0f;                           // rescale threshold (log2 units)

  // Q fragments (B operand of S^T = K Q^T): row m, 8 d per lane per step.
  const int m = m0 + wq * 32 + lr;
  const int mc = min(m, p.M - 1);
  u32x4_t qf[A::DK];
#pragma unroll
  for (int ks = 0; ks < A::DK; ++ks) qf[ks] = gload16(Q + (int64_t)mc * p.ldx + ks * 16 + lg * 8);

  // K block rows: swizzled 16-byte chunks inside D*2-byte rows (D/8 chunks;
  // the XOR uses only chunk bits that exist).  Rows past Lk are clamped and
  // masked out of P in the last block.
  // 256-byte rows (d = 128) all start on bank 0, so 16 consecutive rows need
  // 16 distinct chunk positions: XOR with (row & 15).  128-byte rows (d = 64)
  // pair up within 256 bytes: XOR with ((row >> 1) & 7).
  auto kswz = [](int row) { return A::KCH == 16 ? (row & 15) : ((row >> 1) & 7); };
  auto koff = [&](int row, int c) { return row * A::KROW + ((c ^ kswz(row)) << 4); };
  // V rows in LDS as they are in memory (key-major, D*2 bytes), 16-byte chunk
  // c of key row k at position c ^ vswz(k).  The second product reads V^T
  // fragments with transposing LDS reads (see vfrag), and this swizzle keeps
  // each 32-lane half of such a read on distinct banks.
  auto vswz = [](int k) { return A::KCH == 16 ? 4 * (k & 3) : 4 * ((k >> 1) & 1); };
  constexpr int LPR = A::KCH;                   // lanes per row in one wave-wide load
  constexpr int RPI = 64 / LPR;                 // rows per instruction
  // Wave-wide direct loads of key block j (K, or V when v_t is true) into a
  // ring stage of this wave's group.  Load ins of a wave covers rows in * RPI
  // .. + RPI - 1, in = wq + QG ins.  The V swizzle depends on the row only
  // through bits that lane / LPR sets, the K swizzle (row & 15 for d = 128,
  // (row >> 1) & 7 for d = 64) also through in % 4 or in % 2, which takes NP
  // values over a wave's loads: the lane's byte offset inside its rows is one
  // of NP fixed ones and the rest is wave-uniform.  Rows past Lk (the last
  // block only) are clamped, and masked out of P.
  constexpr int NP = A::KCH == 16 ? (QG >= 4 ? 1 : 4 / QG) : (QG >= 2 ? 1 : 2);
  uint32_t kl_off[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i)
    kl_off[i] = (uint32_t)((lane / LPR) * p.ldw1 * 2 + (((lane % LPR) ^ kswz((wq + QG * i) * RPI + lane / LPR)) << 4));
  const uint32_t vl_off = (uint32_t)((lane / LPR) * p.ldw2 * 2 + (((lane % LPR) ^ vswz(lane / LPR)) << 4));
  constexpr int NINS = A::TN / RPI / QG;   // direct loads per wave for one K or V block
  char* const ring = smem + grp * 2 * A::STAGE;
  // Load ins of this wave for key block j (K, or V when v_t is true) into a
  // ring stage; `full` (block j lies inside Lk) selects the wave-uniform form.
  auto issue_one = [&](int j, auto stage_t, auto v_t, int ins, bool full) {
    constexpr bool VS = decltype(v_t)::value;
    char* dst = ring + decltype(stage_t)::value * A::STAGE + (VS ? A::KB : 0);
    const bf16_t* src = VS ? Vp : Kp;
    const int64_t ld = VS ? p.ldw2 : p.ldw1;
    const int in = wq + QG * ins;
    if (full) {
      const char* base = reinterpret_cast<const char*>(src + (int64_t)(j * A::TN + in * RPI) * ld);
      dma16(base + (VS ? vl_off : kl_off[ins % NP]), dst + in * 1024);
    } else {
      const int row = in * RPI + lane / LPR;
      const int c = (lane % LPR) ^ (VS ? vswz(row) : kswz(row));
      const int key = min(j * A::TN + row, Lk - 1);
      dma16(reinterpret_cast<const char*>(src + (int64_t)key * ld) + c * 16, dst + in * 1024);
    }
  };
  auto issue_kv = [&](int j, auto stage_t) {
    const bool full = (j + 1) * A::TN <= Lk;
#pragma unroll
    for (int ins = 0; ins < NINS; ++ins) issue_one(j, stage_t, std::false_type{}, ins, full);
#pragma unroll
    for (int ins = 0; ins < NINS; ++ins) issue_one(j, stage_t, std::true_type{}, ins, full);
  };
  auto lds_sync = [] {   // this wave's LDS accesses are done, then a workgroup barrier
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14));
    lds_barrier();
  };

  // LDS byte address of K-fragment reads for d step ks (lane row lr of a
  // 32-key half; the half and the stage are compile-time offsets).  The
  // swizzle of row 32 h + lr equals that of row lr.
  uint32_t kbase[A::DK];
  // LDS byte address of the V^T fragment reads of output block b, less the
  // stage and key offsets (compile-time constants at each read).  In a group
  // of 16 lanes, lane r names 4 consecutive d (offset 4 (r % 4)) of key
  // k0 + r / 4, where k0 = 32 bl + 16 s + 4 lg is a multiple of 4, so the V
  // swizzle of that key depends on r only.
  uint32_t vbase[A::BD];
  {
    const int r = lane & 15;
    const int dcol = (lane & 16) + 4 * (r & 3);
    const int krow = 4 * lg + (r >> 2);
    const uint32_t s0 =
        (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)smem) + grp * 2 * A::STAGE;
#pragma unroll
    for (int ks = 0; ks < A::DK; ++ks) kbase[ks] = s0 + koff(lr, 2 * ks + lg);
#pragma unroll
    for (int b = 0; b < A::BD; ++b)
      vbase[b] = s0 + krow * A::KROW + ((((32 * b + dcol) >> 3) ^ vswz(krow)) << 4) + 8 * (r & 1);
  }

  f32x16_t Oa[A::BD];
#pragma unroll
  for (int b = 0; b < A::BD; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) Oa[b][i] = 0.0f;
  float m_used = -INFINITY;
  // This lane's part of the row sum l of P (its 32 of each block's keys),
  // summed from the same bf16 P as the numerator by dot products with
  // (1, 1); the lane pair's parts are added at the end.
  float lsum = 0.0f;

  // One MFMA of an S^T block: 32-key half b, d step ks.
  auto mma_s = [&](f32x16_t (&S)[A::NH], int b, int ks, u32x4_t kf) {
    const f32x16_t zero = {};
    S[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, kf),
                                                   __builtin_bit_cast(bf16x8_t, qf[ks]), ks == 0 ? zero : S[b],
                                                   0, 0, 0);
  };
  // Softmax of block j (S is this lane's 16 NH scores, raw).
  auto softmax_all = [&](f32x16_t (&S)[A::NH], int j, SoftmaxStep& st, auto mask_t) {
    constexpr bool MASK = decltype(mask_t)::value;
    float t = -INFINITY;   // block maximum of the raw scores (scale > 0)
#pragma unroll
    for (int e = 0; e < 16 * A::NH; ++e) t = fmaxf(t, S[e >> 4][e & 15]);
    st.bmax = lane_pair_max(t) * sl2;
    const float mnew = fmaxf(m_used, st.bmax);
    st.need = mnew > m_used + kLazy;
    const float m_eff = st.need ? mnew : m_used;
    // exactly 1 when the maximum in use stays (also at -infinity, with key groups)
    st.corr = KS > 1 && !st.need ? 1.0f : __builtin_amdgcn_exp2f(m_used - m_eff);
    m_used = m_eff;
    // P = exp2(s * scale * log2e - m).  A key group whose scores so far are
    // all -infinity keeps the maximum -infinity; its P are 0.
    const float nm = KS > 1 && m_used == -INFINITY ? 0.0f : -m_used;
#pragma unroll
    for (int e = 0; e < 16 * A::NH; ++e) {
      float pv = __builtin_amdgcn_exp2f(fmaf(S[e >> 4][e & 15], sl2, nm));
      if constexpr (MASK) {
        const int key = j * A::TN + (e >> 4) * 32 + acc_row(e & 15, lane);
        pv = key < Lk ? pv : 0.0f;
      }
      S[e >> 4][e & 15] = pv;
    }
#pragma unroll
    for (int h = 0; h < A::NH; ++h) {
      st.P[h][0] = pack_step(S[h], 0);
      st.P[h][1] = pack_step(S[h], 1);
    }
  };
  auto rescale = [&](const SoftmaxStep& st) {
    if (__any(st.need)) {
#pragma unroll
      for (int b = 0; b < A::BD; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) Oa[b][i] *= st.corr;
      lsum *= st.corr;
    }
  };
  // O^T += V^T P^T for block j (V^T fragments two MFMAs ahead).  Fragment
  // (b, s, bl) gives lane (lr, lg) V[k0 + 0..3][32 b + lr] and
  // V[k0 + 8 + 0..3][32 b + lr], k0 = 32 bl + 16 s + 4 lg: the permuted k order
  // of pack_step.  Each half comes from one ds_read_b64_tr_b16: in a group of
  // 16 lanes, lane r names 4 consecutive d of key k0 + r / 4 (d offset
  // 4 (r % 4)), and lane i receives the 4 keys of d offset i.
  auto pv_block = [&](auto stage_t, const SoftmaxStep& st) {
    constexpr int VT = decltype(stage_t)::value * A::STAGE + A::KB;   // this stage's V rows
    auto vfrag = [&](auto i_t) {   // i = (bl * 2 + s) * BD + b
      constexpr int i = decltype(i_t)::value;
      constexpr int b = i % A::BD, s = (i / A::BD) & 1, bl = i / (2 * A::BD);
      constexpr int off = VT + (32 * bl + 16 * s) * A::KROW;
      const u32x2_t lo = ds_read_tr_b64<off>(vbase[b]);
      const u32x2_t hi = ds_read_tr_b64<off + 8 * A::KROW>(vbase[b]);
      return u32x4_t{lo[0], lo[1], hi[0], hi[1]};
    };
    u32x4_t vf[3];
    vf[0] = vfrag(std::integral_constant<int, 0>{});
    vf[1] = vfrag(std::integral_constant<int, 1>{});
    static_for<0, A::NSB>([&](auto i_t) {
      constexpr int i = decltype(i_t)::value;
      constexpr int b = i % A::BD, s = (i / A::BD) & 1, bl = i / (2 * A::BD);
      // Two reads per fragment and no other LDS operation in between, so
      // fragment i is complete once at most fragment i + 1's two reads are
      // outstanding.  Fragment i + 2 is read after MFMA i, into the registers
      // MFMA i - 1 read.
      lgkm_wait<(i + 1 < A::NSB ? 2 : 0)>(vf[i % 3]);
      Mma<bf16_t>::run(Oa[b], vf[i % 3], st.P[bl][s]);
      if constexpr (i + 2 < A::NSB) vf[(i + 2) % 3] = vfrag(std::integral_constant<int, i + 2>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const bf16x2_t one2 = __builtin_bit_cast(bf16x2_t, 0x3F803F80u);   // bf16 (1.0, 1.0)
    // Each packed pair goes through a 32-bit value of its own: with the
    // vector element written inside the call, the compiler passed the
    // fragment's first register for all four pairs.
#pragma unroll
    for (int q = 0; q < 2 * A::NH; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t x = st.P[q >> 1][q & 1][e];
        lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, x), one2, lsum, false);
      }
  };
  // S^T of block j from its K rows in LDS: one 16-byte read per MFMA, KLA
  // reads ahead; MFMA i takes half i % NH and d step i / NH, so the halves'
  // accumulation chains alternate.  No other LDS operation is issued
  // in between, so read i is complete once at most the KLA - 1 later ones
  // are outstanding.
  auto s_block = [&](f32x16_t (&S)[A::NH], auto stage_t, auto&& after_mma) {
    constexpr int KST = decltype(stage_t)::value * A::STAGE;
    constexpr int KLA = 4;
    auto kread = [&](auto i_t) {
      constexpr int i = decltype(i_t)::value;
      constexpr int h = i % A::NH, ks = i / A::NH;
      return ds_read_b128_at<KST + h * 32 * A::KROW>(kbase[ks]);
    };
    u32x4_t kf[KLA];
    static_for<0, KLA>([&](auto i_t) { kf[decltype(i_t)::value] = kread(i_t); });
    static_for<0, A::NSA>([&](auto i_t) {
      constexpr int i = decltype(i_t)::value;
      constexpr int rest = A::NSA - 1 - i;
      lgkm_wait<(rest < KLA - 1 ? rest : KLA - 1)>(kf[i % KLA]);
      mma_s(S, i % A::NH, i / A::NH, kf[i % KLA]);
      if constexpr (i + KLA < A::NSA) kf[(i + KLA) % KLA] = kread(std::integral_constant<int, i + KLA>{});
      after_mma(i_t);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  f32x16_t S[A::NH];
  SoftmaxStep st;
  // Prologue: K and V of the group's first block on their way into LDS stage 0.
  using S0_ = std::integral_constant<int, 0>;
  using S1_ = std::integral_constant<int, 1>;
  if (KS == 1 || jb + grp < NB) issue_kv(jb + grp, S0_{});
  // Step j: K(j) and V(j) are in the step's stage once every wave has passed
  // the barrier, and every wave is then done with the group's previous block,
  // so the other stage takes the group's next block (direct loads).  Then
  // S^T(j), softmax, rescale and the P V of block j.  With KS = 1 two
  // workgroups share a CU, so while one wave of a SIMD runs the softmax the
  // other (from the other workgroup) can issue MFMAs.  The loop runs two
  // steps per trip so that the stage, and with it every LDS offset, is a
  // compile-time constant.
  // The next block's loads go between the MFMAs of S^T(j): a wave's load issue
  // waits while the CU's load path takes earlier loads, and MFMAs already
  // issued keep the matrix core busy meanwhile (eight loads in a row at the
  // barrier cost a quarter of the step).
  constexpr int SPC = A::NSA / (2 * NINS) > 0 ? A::NSA / (2 * NINS) : 1;   // MFMAs per load
  constexpr int LPM = 2 * NINS > A::NSA ? 2 * NINS / A::NSA : 1;          // loads per MFMA
  auto step = [&](int j, auto stage_t, auto next_t) {
    wait_vmcnt<0>();
    lds_sync();
    if (KS > 1 && j >= NB) return;   // this group has no block in the last step
    // Loads q of the next block (K for q < NINS, then V), spread over the MFMAs.
    auto loads = [&](auto full_t) {
      using FT = decltype(full_t);
      return [&](auto i_t) {
        constexpr int i = decltype(i_t)::value;
        static_for<0, LPM>([&](auto l_t) {
          constexpr int q = i / SPC * LPM + decltype(l_t)::value;
          if constexpr (i % SPC == SPC - 1 && q < 2 * NINS) {
            constexpr bool VS = q >= NINS;
            issue_one(j + KS, next_t, std::integral_constant<bool, VS>{}, VS ? q - NINS : q, FT::value);
          }
        });
      };
    };
    // The three cases are separate code paths so that the common one (the
    // next block lies inside Lk) keeps its wave-uniform addressing.
    if (j + KS < NB && (j + KS + 1) * A::TN <= Lk) s_block(S, stage_t, loads(std::true_type{}));
    else if (j + KS < NB) s_block(S, stage_t, loads(std::false_type{}));
    else s_block(S, stage_t, [](auto) {});
    if (KS == 1 ? j + 1 < NB : (j + 1) * A::TN <= Lk) softmax_all(S, j, st, std::false_type{});
    else softmax_all(S, j, st, std::true_type{});
    rescale(st);
    pv_block(stage_t, st);
  };
  // Every group runs the same number of steps (the barriers are the workgroup's).
  for (int j = jb; j < NB; j += 2 * KS) {
    step(j + grp, S0_{}, S1_{});
    if (j + KS < NB) step(j + KS + grp, S1_{}, S0_{});
  }

  __syncthreads();
  if constexpr (KS == 1) {
    const float inv = 1.0f / lane_pair_sum(lsum);
#pragma unroll
    for (int b = 0; b < A::BD; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) Oa[b][i] *= inv;
    store_tile_staged<typename A::Out>(reinterpret_cast<f32x16_t(&)[1][A::BD]>(Oa), p.O + (int64_t)bz * p.so, p.ldo, 0, p.M, D, m0, 0, smem, tid, lane,
                                       wave, 0);
  } else {
    // Every wave leaves its O (fp32, one padded row per query) and (m, l) in
    // LDS; then thread t takes 8 consecutive d of one query and adds the
    // groups in order, each scaled to the common maximum.
    const float l = lane_pair_sum(lsum);
    char* const orow = smem + (wave * 32 + lr) * A::OROW;
#pragma unroll
    for (int b = 0; b < A::BD; ++b)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4)
        *reinterpret_cast<f32x4_t*>(orow + (32 * b + 8 * g4 + 4 * lg) * 4) =
            f32x4_t{Oa[b][4 * g4], Oa[b][4 * g4 + 1], Oa[b][4 * g4 + 2], Oa[b][4 * g4 + 3]};
    float* const ml = reinterpret_cast<float*>(smem + A::NW * 32 * A::OROW);   // [wave][query][2]
    int* const flag = reinterpret_cast<int*>(smem + A::NW * 32 * (A::OROW + 8));
    if (lg == 0) {
      ml[(wave * 32 + lr) * 2] = m_used;
      ml[(wave * 32 + lr) * 2 + 1] = l;
    }
    __syncthreads();
    constexpr int TPR = D / 8;                      // threads per query
    constexpr int QPI = A::NT / TPR;                // queries per iteration
    const int nz = gridDim.z, rows = min(A::TM, p.M - m0);
    const int d0 = tid % TPR * 8;
    uint16_t* const O = p.O + (int64_t)bz * p.so;
    auto store8 = [&](int r, const float (&o)[8], float s) {
      const u32x4_t w = {pack_bf16x2(o[0] * s, o[1] * s), pack_bf16x2(o[2] * s, o[3] * s),
                         pack_bf16x2(o[4] * s, o[5] * s), pack_bf16x2(o[6] * s, o[7] * s)};
      __builtin_nontemporal_store(w, reinterpret_cast<u32x4_t*>(O + (int64_t)(m0 + r) * p.ldo + d0));
    };
    // Partials of the query block (split keys): [z][row][D] O, then [z][row][2]
    // (m, l), in the block's own region; device-coherent accesses, since the
    // workgroups of a block need not share an XCD.
    constexpr int kSc1 = 16;
    float* const part = p.ws_part + (int64_t)g * nz * A::TM * (D + 2);
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(part, 0, nz * A::TM * (D + 2) * 4, 0x00020000);
    const int ml_off = nz * A::TM * D * 4;
    for (int r = tid / TPR; r < rows; r += QPI) {
      float mg[KS], M = -INFINITY, L = 0.0f, o[8] = {};
#pragma unroll
      for (int q = 0; q < KS; ++q) M = fmaxf(M, mg[q] = ml[((q * QG + r / 32) * 32 + r % 32) * 2]);
#pragma unroll
      for (int q = 0; q < KS; ++q) {
        const int w = (q * QG + r / 32) * 32 + r % 32;
        const float f = mg[q] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mg[q] - M);
        L = fmaf(f, ml[w * 2 + 1], L);
        const float* src = reinterpret_cast<const float*>(smem + w * A::OROW) + d0;
        const f32x4_t a = *reinterpret_cast<const f32x4_t*>(src), b = *reinterpret_cast<const f32x4_t*>(src + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o[e] = fmaf(f, a[e], o[e]);
          o[4 + e] = fmaf(f, b[e], o[4 + e]);
        }
      }
      if (nz == 1) {
        store8(r, o, 1.0f / L);
      } else {
        const int at = (blockIdx.z * A::TM + r) * D * 4 + d0 * 4;
        const f32x4_t a = {o[0], o[1], o[2], o[3]}, b = {o[4], o[5], o[6], o[7]};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, a), rsrc, at, 0, kSc1);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, b), rsrc, at + 16, 0, kSc1);
        if (d0 == 0) {
          const u32x2_t v = {__float_as_uint(M), __float_as_uint(L)};
          __builtin_amdgcn_raw_buffer_store_b64(v, rsrc, ml_off + (blockIdx.z * A::TM + r) * 8, 0, kSc1);
        }
      }
    }
    if (nz == 1) return;
    // Count the arrival; the last workgroup of the block merges (a counter goes
    // back to 0, ready for the next call).
    wait_vmcnt<0>();          // this wave's partial stores have completed
    __syncthreads();          // ... and every wave's
    if (tid == 0) {
      const unsigned old = __hip_atomic_fetch_add(p.ws_count + g, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int last = old == (unsigned)(nz - 1);
      if (last) __hip_atomic_store(p.ws_count + g, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      *flag = last;
    }
    __syncthreads();
    if (!*flag) return;
    for (int r = tid / TPR; r < rows; r += QPI) {
      float M = -INFINITY, L = 0.0f, o[8] = {};
      // parts in order, rescaled to the running maximum, four loaded at a time
      for (int z0 = 0; z0 < nz; z0 += 4) {
        u32x4_t a[4], b[4];
        u32x2_t v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int z = min(z0 + q, nz - 1), at = (z * A::TM + r) * D * 4 + d0 * 4;
          a[q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, 0, kSc1);
          b[q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at + 16, 0, kSc1);
          v[q] = __builtin_amdgcn_raw_buffer_load_b64(rsrc, ml_off + (z * A::TM + r) * 8, 0, kSc1);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (z0 + q >= nz) break;
          const float mz = __uint_as_float(v[q][0]), mn = fmaxf(M, mz);
          const float fo = M == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(M - mn);
          const float fz = mz == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mz - mn);
          M = mn;
          L = fmaf(fz, __uint_as_float(v[q][1]), fo * L);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            o[e] = fmaf(fz, __uint_as_float(a[q][e]), fo * o[e]);
            o[4 + e] = fmaf(fz, __uint_as_float(b[q][e]), fo * o[4 + e]);
          }
        }
      }
      store8(r, o, 1.0f / L);
    }
  }
}

// ---------------------------------------------------------------------------
bool b2b_attention_supported(int d) { return d == 64 || d == 128; }

template <int D, int QG, int KS, int BK>
static hipError_t launch_attention(const B2BParams& p, int nz, hipStream_t st) {
  using A = AttnShape<D, QG, KS, BK>;
  const dim3 grid((unsigned)((p.M + A::TM - 1) / A::TM), (unsigned)p.batch, (unsigned)nz), block(A::NT);
  hipLaunchKernelGGL((b2b_attention_kernel<D, QG, KS, BK>), grid, block, 0, st, p);
  return hipGetLastError();
}

// The workgroup form (query waves QG, 0 for two workgroups per CU with QG = 4
// and one key group) and the number nz of workgroups that split a query
// block's keys.  One workgroup of a several-group form fills a CU (128 KB of
// rings, two waves per SIMD), so the form with the fewest queries per
// workgroup that fits one generation of 256 CUs is taken, and the two-per-CU
// form beyond.  Measured (us, heads x queries x keys x d; QG 1 / 2 / 4 / two
// per CU): 8 x 345 x 345 x 64 5.7 / 6.5 / 7.8 / 8.3; 16 x 1000 x 1000 x 128
// 24.4 / 16.4 / 19.6 / 22.5; 24 x 1000 x 1000 x 64 22.7 / 18.5 / 14.7 / 17.5;
// 32 x 2048 x 2048 x 128 152 / 95 / 73 / 71.  Queries that fit one or two waves
// take that form however many heads there are (256 x 1 x 4095 x 128 91 us, two
// per CU 99).  Keys are split while workgroups are fewer than CUs and every
// wave keeps two key blocks, at most eight ways (the last workgroup's merge
// grows with them): 16 x 1 x 4095 x 128 34.5 us unsplit, 14.5 / 13.6 / 16.6 in
// 4 / 8 / 16; 128 x 1 x 4095 x 128 65 and 50 in 2.
AttentionForm attention_form(int64_t M, int64_t batch, int64_t Lk, int d) {
  constexpr int64_t kCUs = 256;
  auto wgs = [&](int qg) { return (M + 32 * qg - 1) / (32 * qg) * batch; };
  AttentionForm f{0, 1};
  if (M <= 32 || wgs(1) <= kCUs) f.qg = 1;
  else if (M <= 64 || wgs(2) <= kCUs) f.qg = 2;
  else if (wgs(4) <= kCUs) f.qg = 4;
  // Few keys: the merge costs more than the groups save.  Kernel us, this form / two per
  // CU: QG 4, 36 x 722 x 192 x 64 7.1 / 6.7, x 256 7.5 / 7.6; 128 x 185 x 192 x 128 10.1 / 9.0, x 256
  // 10.5 / 10.4; QG 2, 16 x 800 x 128 x 64 5.6 / 5.6, x 192 6.0 / 6.4, 16 x 800 x 128 x 128 7.5 / 7.2,
  // x 192 8.3 / 8.4; QG 1, 8 x 300 x 64 x 64 5.2 / 4.6, 16 x 300 x 96 x 64 5.1 / 5.3, x 64 x 128 5.6 / 6.0.
  if (Lk <= (f.qg == 4 ? 192 : f.qg == 2 ? 128 : d == 64 ? 64 : 0)) return AttentionForm{0, 1};
  if (f.qg == 1) {
    const int64_t per_wave = (Lk + 31) / 32 / (d == 128 ? 4 : 8);   // key blocks of one wave, unsplit
    f.nz = (int)std::max<int64_t>(1, std::min<int64_t>({kCUs / wgs(1), per_wave / 2, 8}));
  }
  return f;
}

hipError_t launch_b2b_attention(const B2BParams& p, hipStream_t st) {
  const int qg = attention_form(p.M, p.batch, p.N1, p.K).qg;
  if (p.K == 128) {
    if (qg == 1) return launch_attention<128, 1, 4, 32>(p, p.cn, st);
    if (qg == 2) return launch_attention<128, 2, 4, 32>(p, 1, st);
    if (qg == 4) return launch_attention<128, 4, 2, 64>(p, 1, st);
    return launch_attention<128, 4, 1, 64>(p, 1, st);
  }
  if (p.K == 64) {
    if (qg == 1) return launch_attention<64, 1, 8, 32>(p, p.cn, st);
    if (qg == 2) return launch_attention<64, 2, 4, 64>(p, 1, st);
    if (qg == 4) return launch_attention<64, 4, 2, 64>(p, 1, st);
    return launch_attention<64, 4, 1, 64>(p, 1, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace cf
