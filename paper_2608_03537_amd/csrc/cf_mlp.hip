// Back-to-back MLP for gfx950 (Sec. IV, Eq. 2 with F = ReLU(. + b1);
// Sec. IV-A): O = ReLU(X W1 + b1) W2 + b2, optionally ReLU(O) -- the DLRM
// bottom-MLP pattern of Table 2 (1024 -> 512 -> 128).
//
// Work split (the cross-workgroup dataflow of Sec. IV-A).  The hidden
// dimension N1 is split into chunks of 256 units; the cn = N1 / 256
// workgroups of a 128-row block each own one chunk c:
//   ML1   P_c^T = W1_c^T X^T on the direct-to-LDS ring of the GEMM kernels
//         (the accumulators start from b1, so they hold P_c + b1_c);
//   Epi1  S_c = ReLU(.) packed to bf16 in registers;
//   ML2   O_c = S_c W2_c, the partial second product over the chunk, with
//         the W2^T chunk staged in LDS;
//   Epi2  O = sum_c O_c + b2 (the partial-sum identity of Sec. IV-A), summed
//         at commit: each workgroup publishes O_c, the last one of its row
//         block to arrive adds the partials in the fixed order c = 0, 1, ...
//         and stores O.  No workgroup waits for another, so no co-residency
//         is needed, and the result does not depend on the arrival order.
//
// Register hand-off.  The rows of each 32-row block of W1_c^T are loaded with
// bits 2 and 3 of the row index swapped (perm23), so accumulator elements
// 8s .. 8s+7 of lane half g hold hidden units 16s + 8g + 0..7 of the block.
// Packed to bf16 they are the B operand of one MFMA step of the second
// product O^T = W2^T S^T, whose A operand is then one contiguous 16-byte piece
// of a W2^T row (k order inside an MFMA step is free as long as both operands
// use the same one).
//
// Commit visibility.  Partials are written with agent-scope stores, the
// writer waits for their completion before its arrival add (agent scope), and
// the last arriver reads them with agent-scope loads issued after its add
// returned: every access involved is device-coherent, so no cache flush is
// needed.  The arrival counter of a row block goes back to 0 at the end of
// the call (the last arriver resets it), so a zero-filled counter area stays
// valid for every later call.
//
// This is the split form (b2b_mlp_kernel).  b2b_mlp_whole_kernel runs the chunks of
// a row block in turn, b2b_mlp_wide_kernel all 512 hidden units at once, and
// b2b_mlp_few_kernel works on 32-row blocks; launch_b2b_mlp chooses.
#include "cf_gemm_tile.h"
#include "comfuse.h"

namespace cf {

using MlpS = TileShape<bf16_t, 2, 4, 2, 2, 128, 3>;   // 128 rows x 256 hidden units, 4 waves (2 x 2)
static_assert(MlpS::TM == kMlpRows && MlpS::TN == kMlpHidden, "MLP tile");

template <int N2>
struct MlpLayout {
  static constexpr int NB2 = N2 / 32;                 // output column blocks
  static constexpr int W2_ROWB = kMlpHidden * 2;      // bytes of one W2^T chunk row
  static constexpr int W2_BYTES = N2 * W2_ROWB;       // W2^T chunk in LDS
  static constexpr int OFF_RED = W2_BYTES;            // partial sums of the wn = 1 waves
  static constexpr int RED_WAVE = 64 * N2 * 4;        // one wave's 64 rows x N2 fp32
  static constexpr int W2_LOADS = W2_BYTES / 1024;    // wave-wide 1 KB loads
  static constexpr int PT_ROWB = N2 * 4;              // row-major fp32 partial tile (over the W2 chunk)
  static constexpr int OFF_FLAG = OFF_RED + 2 * RED_WAVE;   // "this workgroup commits" flag
  static_assert(OFF_FLAG + 16 <= MlpS::SMEM_V2, "flag in LDS");
  static_assert(kMlpRows * PT_ROWB <= OFF_RED, "partial tile fits the W2 region");
  static_assert(OFF_RED + 2 * RED_WAVE <= MlpS::SMEM_V2, "LDS budget");
  static_assert(W2_LOADS % MlpS::NW == 0, "W2 loads per wave");
};

// Commit of a TM x N2 row-major tile by column quads: quad(j) gives thread t the
// quad (t + NT j) % QPR of row (t + NT j) / QPR, so every wave-wide access
// covers whole rows.  cn workgroups (c of them) share the rows; the partials
// go through memory with device-coherent 16-byte accesses (sc1): the
// workgroups of a row block need not share an XCD, and the reader reads only
// after the writer's stores completed (arrival count).
template <int TM, int NT, int N2, typename Quad>
__device__ __forceinline__ void mlp_commit(const B2BParams& p, Quad&& quad, int bz, int rbs, int rb,
                                           int cn, int c, int m0, int& flag) {
  constexpr int QPR = N2 / 4;                          // column quads per row
  constexpr int QUADS = TM * QPR / NT;                 // quads per thread
  static_assert(NT % QPR == 0, "a thread's column quad is the same in every step");
  constexpr int kSc1 = 16;                             // cache policy: device-coherent
  const int tid = threadIdx.x, q4 = tid % QPR;
  float* part = p.ws_part + (int64_t)bz * cn * p.M * N2;
  const int rows = min(TM, p.M - m0);
  // Buffer resource over chunk k's partial rows [m0, m0 + rows): raw 32-bit
  // data; accesses past its end are dropped (stores) or read as 0 (loads).
  auto part_rsrc = [&](int k) {
    return __builtin_amdgcn_make_buffer_rsrc(part + ((int64_t)k * p.M + m0) * N2, 0, rows * N2 * 4, 0x00020000);
  };
  if (cn > 1) {
    // publish O_c, then count this workgroup's arrival
    const auto mine = part_rsrc(c);
#pragma unroll 8
    for (int j = 0; j < QUADS; ++j) {
      const int r = (tid + j * NT) / QPR;
      if (r < rows)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, quad(j)), mine, (r * QPR + q4) * 16, 0, kSc1);
    }
    wait_vmcnt<0>();          // this wave's partial stores have completed
    __syncthreads();          // ... and every wave's
    if (tid == 0) {
      unsigned* cnt = p.ws_count + (int64_t)bz * rbs + rb;
      const unsigned old = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int last = old == (unsigned)(cn - 1);
      if (last) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
      flag = last;
    }
    __syncthreads();
    if (!flag) return;        // the last workgroup of the row block commits
  }

  // O = O_0 + O_1 + ... (chunk order, whichever workgroup finished last; its
  // own partial comes from its tile, equal to what it stored) + b2, output
  // ReLU, bf16 rows.  A thread's column quad is the same in every step, so b2 is
  // read once; another chunk's partials are loaded for all steps before any is
  // used, so their latencies overlap.
  uint16_t* O = p.O + (int64_t)bz * p.so;
  f32x4_t bb = {0.0f, 0.0f, 0.0f, 0.0f};
  if (p.b2) bb = *reinterpret_cast<const f32x4_t*>(p.b2 + 4 * q4);
  f32x4_t t[QUADS];
#pragma unroll
  for (int j = 0; j < QUADS; ++j) t[j] = quad(j);
  if (cn > 1) {
    f32x4_t acc2[QUADS];
    for (int k = 0; k < cn; ++k) {
      if (k == c) {
#pragma unroll
        for (int j = 0; j < QUADS; ++j) acc2[j] = k == 0 ? t[j] : acc2[j] + t[j];
        continue;
      }
      const auto src = part_rsrc(k);
      u32x4_t w[QUADS];
#pragma unroll
      for (int j = 0; j < QUADS; ++j) {
        const int r = min((tid + j * NT) / QPR, rows - 1);
        w[j] = __builtin_amdgcn_raw_buffer_load_b128(src, (r * QPR + q4) * 16, 0, kSc1);
      }
#pragma unroll
      for (int j = 0; j < QUADS; ++j) {
        const f32x4_t v = __builtin_bit_cast(f32x4_t, w[j]);
        acc2[j] = k == 0 ? v : acc2[j] + v;
      }
    }
#pragma unroll
    for (int j = 0; j < QUADS; ++j) t[j] = acc2[j];
  }
#pragma unroll
  for (int j = 0; j < QUADS; ++j) {
    const int m = m0 + (tid + j * NT) / QPR;
    if (m >= p.M) continue;
    f32x4_t y = t[j];
    if (p.b2) y += bb;
    if (p.out_relu)
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = fmaxf(y[e], 0.0f);
    const u32x2_t o2 = {pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
    __builtin_nontemporal_store(o2, reinterpret_cast<u32x2_t*>(O + (int64_t)m * p.ldo + 4 * q4));
  }
}

template <int N2>
__global__ __launch_bounds__(MlpS::NT, 1) __attribute__((amdgpu_waves_per_eu(1, 1)))
void b2b_mlp_kernel(B2BParams p) {
  using S = MlpS;
  using L = MlpLayout<N2>;
  constexpr int NB2 = L::NB2;
  // One LDS array only: a second __shared__ object makes the compiler wait
  // for every outstanding direct-to-LDS load before each LDS read of the main
  // loop (it can no longer tell the loads' targets apart).
  __shared__ __attribute__((aligned(16))) char smem[S::SMEM_V2];
  int& last_flag = *reinterpret_cast<int*>(smem + L::OFF_FLAG);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / S::WN, wn = wave % S::WN;
  const int lr = lane & 31, lg = lane >> 5;
  const int cn = p.cn;
  // XCD-aware order: linear id L runs on XCD L % 8.  In full groups of 8 row
  // blocks, the cn workgroups of row block 8 i + x are L = 8 (cn i + c) + x:
  // they share XCD x and run at about the same time, so the row block's X
  // comes from HBM into that XCD's L2 once for all its chunks.  The rows past
  // the last full group go in plain order.
  int c, rb;
  {
    const int L = blockIdx.x, full = (int)(gridDim.x / cn) / 8 * 8 * cn;
    if (L < full) {
      c = (L >> 3) % cn;
      rb = (L >> 3) / cn * 8 + (L & 7);
    } else {
      c = (L - full) % cn;
      rb = full / cn + (L - full) / cn;
    }
  }
  const int m0 = rb * S::TM, h0 = c * kMlpHidden;
  const int bz = blockIdx.y;
  const bf16_t* X = p.X + (int64_t)bz * p.sx;
  const bf16_t* W1 = p.W1 + (int64_t)bz * p.sw1;
  const bf16_t* W2 = p.W2 + (int64_t)bz * p.sw2;

  // ---- ML1 (+ b1): P_c^T on the ring, hidden rows in perm23 order
  GemmRowsParams g{};
  g.batch = 1;
  g.M = p.M;
  g.N = p.N1;
  g.K = p.K;
  g.X = X;
  g.ldx = p.ldx;
  g.W = W1;
  g.ldw = p.ldw1;
  g.w_nk = 1;
  g.epi.alpha = 1.0f;
  g.epi.bias = p.b1;
  f32x16_t acc[S::BM][S::BN];
  mainloop_v2<S, false, true>(acc, X, W1, g, m0, h0, 0, smem, lane, wave, wm, wn, p.b1 != nullptr);

  // ---- W2^T chunk (N2 rows x 256 hidden) to LDS; 16-byte chunk q of row r
  // at position q ^ (r & 15), so the 16 rows a 16-lane group reads spread over
  // all banks.  The ring is free after the main loop's final barrier.
#pragma unroll
  for (int j = 0; j < L::W2_LOADS / S::NW; ++j) {
    const int ld = wave + j * S::NW;                  // one load = two W2^T rows
    const int r = 2 * ld + (lane >> 5);
    const int q = (lane & 31) ^ (r & 15);
    dma16(W2 + (int64_t)r * p.ldw2 + h0 + q * 8, smem + ld * 1024);
  }

  // ---- Epi1: S = ReLU(P + b1), packed bf16, the B operands of ML2
  u32x4_t sf[S::BM][S::BN][2];
#pragma unroll
  for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
    for (int bn = 0; bn < S::BN; ++bn)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int w = 0; w < 4; ++w)
          sf[bm][bn][s][w] = pack_bf16x2(fmaxf(acc[bm][bn][8 * s + 2 * w], 0.0f),
                                         fmaxf(acc[bm][bn][8 * s + 2 * w + 1], 0.0f));
  wait_vmcnt<0>();
  __syncthreads();

  // ---- ML2: O_c partial over this wave's 128 hidden units (wave column wn)
  f32x16_t o[S::BM][NB2];
#pragma unroll
  for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
    for (int b2 = 0; b2 < NB2; ++b2)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[bm][b2][i] = 0.0f;
#pragma unroll
  for (int bn = 0; bn < S::BN; ++bn)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int q = (wn * S::WTN + bn * 32 + 16 * s + 8 * lg) / 8;
      u32x4_t a[NB2];
#pragma unroll
      for (int b2 = 0; b2 < NB2; ++b2) {
        const int r = b2 * 32 + lr;
        a[b2] = lds_read16(smem + r * L::W2_ROWB + ((q ^ (r & 15)) << 4));
      }
#pragma unroll
      for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
        for (int b2 = 0; b2 < NB2; ++b2) Mma<bf16_t>::run(o[bm][b2], a[b2], sf[bm][bn][s]);
    }

  // ---- the two wave columns of a row group add their halves (wn = 0 keeps the sum)
  char* red = smem + L::OFF_RED + wm * L::RED_WAVE;
  auto red_at = [&](int bm, int b2, int gq) { return red + (((bm * NB2 + b2) * 4 + gq) * 64 + lane) * 16; };
  if (wn == 1) {
#pragma unroll
    for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
      for (int b2 = 0; b2 < NB2; ++b2)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq)
          *reinterpret_cast<f32x4_t*>(red_at(bm, b2, gq)) =
              f32x4_t{o[bm][b2][4 * gq], o[bm][b2][4 * gq + 1], o[bm][b2][4 * gq + 2], o[bm][b2][4 * gq + 3]};
  }
  __syncthreads();
  if (wn == 0) {
#pragma unroll
    for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
      for (int b2 = 0; b2 < NB2; ++b2)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          const f32x4_t v = *reinterpret_cast<const f32x4_t*>(red_at(bm, b2, gq));
#pragma unroll
          for (int e = 0; e < 4; ++e) o[bm][b2][4 * gq + e] += v[e];
        }
  }

  // ---- the workgroup's partial O_c (128 rows x N2 fp32) to LDS, row-major
  // with 16-byte chunk q of row r at position q ^ (r & 31) (the W2 chunk
  // region is free: every wave passed the barrier above after its last read).
  // Accumulator element 4 gq + e of block (bm, b2): row wm 64 + bm 32 + lr,
  // column b2 32 + 8 gq + 4 lg + e.
  auto pt_at = [&](int r, int q) { return smem + r * L::PT_ROWB + ((q ^ (r & 31)) << 4); };
  if (wn == 0) {
#pragma unroll
    for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
      for (int b2 = 0; b2 < NB2; ++b2)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq)
          *reinterpret_cast<f32x4_t*>(pt_at(wm * S::WTM + bm * 32 + lr, b2 * 8 + 2 * gq + lg)) =
              f32x4_t{o[bm][b2][4 * gq], o[bm][b2][4 * gq + 1], o[bm][b2][4 * gq + 2], o[bm][b2][4 * gq + 3]};
  }
  __syncthreads();

  // ---- Epi2 over the row-major tile
  constexpr int QPR = N2 / 4;
  mlp_commit<S::TM, S::NT, N2>(
      p, [&](int j) { return *reinterpret_cast<const f32x4_t*>(pt_at((tid + j * S::NT) / QPR, tid % QPR)); }, bz,
      gridDim.x / cn, rb, cn, c, m0, last_flag);
}

// Whole-row-block form: one workgroup per 128-row block runs the N1 / 256
// chunks in turn and accumulates the partial second products O_c in
// registers, in chunk order, so nothing goes through memory.  For the second
// product a wave takes its 64 rows and half of the N2 output columns over all
// 256 hidden units of the chunk: its own S half from registers, its wave-
// column partner's half from LDS.  So each output element has one owner (no
// reduction across waves), and a wave keeps 64 accumulator registers live
// across the next chunk's first product.  It needs as many row blocks as
// the split form has workgroups to fill the chip; the host takes it when the
// row blocks alone fill every CU.
template <int N2>
__global__ __launch_bounds__(MlpS::NT, 1) __attribute__((amdgpu_waves_per_eu(1, 1)))
void b2b_mlp_whole_kernel(B2BParams p) {
  using S = MlpS;
  using L = MlpLayout<N2>;
  constexpr int NB2 = L::NB2, HB2 = NB2 / 2;        // output blocks: all, per wave column
  constexpr int OFF_XS = L::W2_BYTES;               // S exchange: [wave 4][bm][bn][s][lane 64][16 B]
  constexpr int XS_WAVE = S::BM * S::BN * 2 * 1024;
  static_assert(OFF_XS + 4 * XS_WAVE <= S::SMEM_V2 && S::TM * L::PT_ROWB <= S::SMEM_V2, "LDS budget");
  __shared__ __attribute__((aligned(16))) char smem[S::SMEM_V2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / S::WN, wn = wave % S::WN;
  const int lr = lane & 31, lg = lane >> 5;
  const int rb = blockIdx.x, m0 = rb * S::TM;
  const int bz = blockIdx.y;
  const bf16_t* X = p.X + (int64_t)bz * p.sx;
  const bf16_t* W1 = p.W1 + (int64_t)bz * p.sw1;
  const bf16_t* W2 = p.W2 + (int64_t)bz * p.sw2;
  GemmRowsParams g{};
  g.batch = 1;
  g.M = p.M;
  g.N = p.N1;
  g.K = p.K;
  g.X = X;
  g.ldx = p.ldx;
  g.W = W1;
  g.ldw = p.ldw1;
  g.w_nk = 1;
  g.epi.alpha = 1.0f;
  g.epi.bias = p.b1;

  // O^T blocks (bm, h): rows wm 64 + bm 32 + lr, output columns (wn HB2 + h) 32 + ...
  f32x16_t o[S::BM][HB2];
#pragma unroll
  for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
    for (int h = 0; h < HB2; ++h)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[bm][h][i] = 0.0f;
  char* xs_own = smem + OFF_XS + wave * XS_WAVE + lane * 16;
  const char* xs_par = smem + OFF_XS + (wm * S::WN + (1 - wn)) * XS_WAVE + lane * 16;
  const int cn = p.N1 / kMlpHidden;
  for (int c = 0; c < cn; ++c) {
    const int h0 = c * kMlpHidden;
    // ML1 (+ b1) of chunk c.  Its ring prologue writes LDS at once: the
    // barrier that ends the previous chunk keeps it behind every wave's
    // reads of that chunk's W2^T and S exchange.  The row offset is opaque
    // to the compiler here, so the ring's X addresses are formed per chunk
    // instead of being hoisted and kept live (spilled) across the loop.
    int m0c = m0;
    asm volatile("" : "+s"(m0c));
    f32x16_t acc[S::BM][S::BN];
    mainloop_v2<S, false, true>(acc, X, W1, g, m0c, h0, 0, smem, lane, wave, wm, wn, p.b1 != nullptr);
    // W2^T chunk to LDS (layout as in the split form)
#pragma unroll
    for (int j = 0; j < L::W2_LOADS / S::NW; ++j) {
      const int ld = wave + j * S::NW;
      const int r = 2 * ld + (lane >> 5);
      const int q = (lane & 31) ^ (r & 15);
      dma16(W2 + (int64_t)r * p.ldw2 + h0 + q * 8, smem + ld * 1024);
    }
    // Epi1: S = ReLU(P + b1), packed bf16 (hidden units wn 128 + bn 32 +
    // 16 s + 8 lg + 0..7 of the chunk), and to the partner through LDS
    u32x4_t sf[S::BM][S::BN][2];
#pragma unroll
    for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
      for (int bn = 0; bn < S::BN; ++bn)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
          for (int w = 0; w < 4; ++w)
            sf[bm][bn][s][w] = pack_bf16x2(fmaxf(acc[bm][bn][8 * s + 2 * w], 0.0f),
                                           fmaxf(acc[bm][bn][8 * s + 2 * w + 1], 0.0f));
          lds_write16(xs_own + ((bm * S::BN + bn) * 2 + s) * 1024, sf[bm][bn][s]);
        }
    wait_vmcnt<0>();
    __syncthreads();
    // ML2: O += S_c W2_c over all 256 hidden units of the chunk, half e of
    // them (e = wn: own registers, else the partner's LDS copy)
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int bn = 0; bn < S::BN; ++bn)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const int q = (e * S::WTN + bn * 32 + 16 * s + 8 * lg) / 8;
          u32x4_t a[HB2], b[S::BM];
#pragma unroll
          for (int h = 0; h < HB2; ++h) {
            const int r = (wn * HB2 + h) * 32 + lr;
            a[h] = lds_read16(smem + r * L::W2_ROWB + ((q ^ (r & 15)) << 4));
          }
#pragma unroll
          for (int bm = 0; bm < S::BM; ++bm)
            b[bm] = e == wn ? sf[bm][bn][s] : lds_read16(xs_par + ((bm * S::BN + bn) * 2 + s) * 1024);
#pragma unroll
          for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
            for (int h = 0; h < HB2; ++h) Mma<bf16_t>::run(o[bm][h], a[h], b[bm]);
        }
    __syncthreads();   // every wave is done with the W2^T chunk and the S exchange
  }

  // O to LDS, row-major fp32 with 16-byte chunk q of row r at position
  // q ^ (r & 31); element 4 gq + e of block (bm, h): row wm 64 + bm 32 + lr,
  // column (wn HB2 + h) 32 + 8 gq + 4 lg + e.
  auto pt_at = [&](int r, int q) { return smem + r * L::PT_ROWB + ((q ^ (r & 31)) << 4); };
#pragma unroll
  for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
    for (int h = 0; h < HB2; ++h)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq)
        *reinterpret_cast<f32x4_t*>(pt_at(wm * S::WTM + bm * 32 + lr, (wn * HB2 + h) * 8 + 2 * gq + lg)) =
            f32x4_t{o[bm][h][4 * gq], o[bm][h][4 * gq + 1], o[bm][h][4 * gq + 2], o[bm][h][4 * gq + 3]};
  __syncthreads();
  // O + b2 (ReLU) as bf16 rows: thread t takes column quad t % QPR of rows
  // (t + 256 j) / QPR, so every wave-wide store covers two whole rows.
  constexpr int QPR = N2 / 4;
  constexpr int QUADS = S::TM * QPR / S::NT;
  static_assert(S::NT % QPR == 0, "a thread's column quad is the same in every step");
  const int q4 = tid % QPR;
  uint16_t* O = p.O + (int64_t)bz * p.so;
  f32x4_t bb = {0.0f, 0.0f, 0.0f, 0.0f};
  if (p.b2) bb = *reinterpret_cast<const f32x4_t*>(p.b2 + 4 * q4);
#pragma unroll
  for (int j = 0; j < QUADS; ++j) {
    const int r = (tid + j * S::NT) / QPR, m = m0 + r;
    if (m >= p.M) continue;
    f32x4_t y = *reinterpret_cast<const f32x4_t*>(pt_at(r, q4));
    if (p.b2) y += bb;
    if (p.out_relu)
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = fmaxf(y[e], 0.0f);
    const u32x2_t o2 = {pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
    __builtin_nontemporal_store(o2, reinterpret_cast<u32x2_t*>(O + (int64_t)m * p.ldo + 4 * q4));
  }
}

// Wide form of the whole-row-block kernel, for N1 = 512: all hidden units at
// once.  The chunked form above streams X once per 256 units, and its 128 x 256
// product is bound by the CU's load path (48 KB a 64-deep k step at about 32 bytes
// a clock, 0.96 us a step however the waves are arranged); 128 x 512 streams 80 KB
// for twice the products, about 1.3 us a step.  (With more hidden units O would
// have to stay in registers through the next 512: 64 spilled registers, 137 us
// against the chunked form's 108 at 65536 x 512 x 1024.)
//
// ML1 (128 rows x 512 hidden units) runs on eight waves in two groups one section
// apart, as the 256 x 256 GEMM tile: a wave alternates a read section (LDS
// fragments) with an MFMA section (8 MFMAs, the loads between them), and waves w
// and w + 4, which share a SIMD, are in opposite sections.  A k step has five 16 KB
// pieces: X (128 rows) and W0..W3 (128 hidden rows each); wave (wm, wn) owns rows
// 64 wm .. +63 and hidden units 32 wn .. +31 of every W piece.  Phase i multiplies X by
// Wi; the read sections of phases 0..3 read X; W1; W2; W3 and the next step's W0.
// LDS holds nine pieces in a ring, in the order W0 X W1 W2 W3 of each step: a
// piece's space takes the ninth piece after it one phase after its read, about
// six phases before that piece is read.  The four quarters of the first half of
// the W2^T chunk follow the last step through the ring as pieces of a further step.
//
// Waits (two loads a piece and wave, issued in ring order): at the end of the
// read section of phase 0 the pieces younger than W1(k) are W2(k) W3(k) W0(k+1) X(k+1)
// W1(k+1); phase 1, younger than W2(k): W3(k) .. W1(k+1) W2(k+1) W3(k+1); phase 2, younger
// than W0(k+1): X(k+1) .. W0(k+2); phase 3, younger than X(k+1): W1(k+1) .. X(k+2).
//
// ML2: wave (wm, wn) takes rows 64 wm .. +63 and output columns 32 wn .. +31, over the
// two halves of the 512 hidden units in turn; S = ReLU(P + b1) goes through LDS in
// fragment order.  Each output element has one owner.
namespace {
constexpr int kWPiece = 16384, kWSlots = 9;

// Fragments of two 32-row blocks (4 KB apart), of one, and of two at different places.
__device__ __forceinline__ void read_one(u32x4_t (&w)[4], const uint32_t (&a)[4]) {
  asm volatile(
      "ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3])
      : "memory");
}
__device__ __forceinline__ void read_two(u32x4_t (&u)[4], u32x4_t (&w)[4], const uint32_t (&a)[4],
                                         const uint32_t (&b)[4]) {
  asm volatile(
      "ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
      "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(u[0]), "=&v"(u[1]), "=&v"(u[2]), "=&v"(u[3]), "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3])
      : "memory");
}
}  // namespace

template <int N2>
__global__ __launch_bounds__(512, 1) __attribute__((amdgpu_waves_per_eu(2, 2)))
void b2b_mlp_wide_kernel(B2BParams p) {
  static_assert(N2 == 128, "four wave columns of 32 outputs");
  constexpr int W2_ROWB = kMlpHidden * 2;           // bytes of one row of a W2^T half (256 hidden units)
  constexpr int PT_ROWB = N2 * 4 + 16;              // staged fp32 output row
  constexpr int LDS = kWSlots * kWPiece;
  static_assert(kMlpRows * PT_ROWB <= LDS && N2 * W2_ROWB == 4 * kWPiece, "LDS budget");
  __shared__ __attribute__((aligned(16))) char smem[LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;          // waves 0..3: wm 0, waves 4..7: wm 1
  const int lr = lane & 31, lg = lane >> 5;
  const int m0 = blockIdx.x * kMlpRows, bz = blockIdx.y;
  const char* X = reinterpret_cast<const char*>(p.X + (int64_t)bz * p.sx + (int64_t)m0 * p.ldx);
  const char* W1 = reinterpret_cast<const char*>(p.W1 + (int64_t)bz * p.sw1);
  const char* W2 = reinterpret_cast<const char*>(p.W2 + (int64_t)bz * p.sw2);
  const int KT = p.K / 64;

  // Load j (of two) of this wave for an X or W piece: rows 8 (2 wave + j) .. +7 of
  // 128 bytes, the 16-byte chunk ch of row r at position ch ^ ((r >> 1) & 7)
  // (conflict-free fragment reads).  The W1^T rows of every 32-row block are
  // taken in perm23 order.  A W2^T quarter holds 32 output rows of 512 bytes, chunk
  // q of row r at position q ^ (r & 15); a load fills two rows.
  uint32_t xo[2], wo[2], vo[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int ld = 2 * wave + j, row = 8 * ld + (lane >> 3), ch = (lane & 7) ^ ((row >> 1) & 7);
    xo[j] = (uint32_t)(min(row, p.M - 1 - m0) * (int)p.ldx * 2 + ch * 16);
    wo[j] = (uint32_t)(((row & ~31) | perm23(row & 31)) * (int)p.ldw1 * 2 + ch * 16);
    const int r = 2 * ld + (lane >> 5);
    vo[j] = (uint32_t)(r * (int)p.ldw2 * 2 + ((lane & 31) ^ (r & 15)) * 16);
  }
  // Ring position of piece i of step st (0 W0, 1 X, 2..4 W1..W3), rotated so that
  // the pieces of step KT start at slot 0.
  const int rot = (kWSlots - 5 * KT % kWSlots) % kWSlots;
  auto at = [&](int st, int i) { return (5 * st + i + rot) % kWSlots * kWPiece; };
  const uint32_t s0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)smem);
  uint32_t xa[4], wa[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int ch = ((2 * ks + lg) ^ ((lr >> 1) & 7)) << 4;
    xa[ks] = s0 + (wm * 64 + lr) * 128 + ch;
    wa[ks] = s0 + (wn * 32 + lr) * 128 + ch;
  }
  const int64_t wpiece = (int64_t)128 * p.ldw1 * 2, vq = (int64_t)32 * p.ldw2 * 2;

  // P + b1: the accumulators start from b1 (element 4 g + q of lane half lg holds
  // hidden unit 16 (g / 2) + 8 lg + 4 (g % 2) + q of the wave's 32)
  f32x16_t acc[2][4];   // [32-row block][W piece]
#pragma unroll
  for (int h = 0; h < 4; ++h)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = h * 128 + wn * 32 + 16 * (g >> 1) + 8 * lg + 4 * (g & 1);
      const f32x4_t b = p.b1 ? *reinterpret_cast<const f32x4_t*>(p.b1 + n) : f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[0][h][4 * g + q] = acc[1][h][4 * g + q] = b[q];
    }
  __builtin_amdgcn_sched_barrier(0);
  auto load_x = [&](int st, int j) {
    dma16(X + (int64_t)st * 128 + xo[j], smem + at(st, 1) + (2 * wave + j) * 1024);
  };
  auto load_w = [&](int st, int h, int j) {
    dma16(W1 + h * wpiece + (int64_t)st * 128 + wo[j], smem + at(st, h == 0 ? 0 : h + 1) + (2 * wave + j) * 1024);
  };
  // Quarter q of the W2^T half at hidden offset `off` (bytes) into slot q.
  auto load_v = [&](int off, int q, int j) {
    dma16(W2 + off + q * vq + vo[j], smem + q * kWPiece + (2 * wave + j) * 1024);
  };
  u32x4_t xf[2][4], w[2][4];
  auto mma = [&](auto piece_t, auto&& load) {
    constexpr int H = decltype(piece_t)::value;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int bm = 0; bm < 2; ++bm) {
        Mma<bf16_t>::run(acc[bm][H], w[H & 1][ks], xf[bm][ks]);
        if (bm == 1) {
          __builtin_amdgcn_sched_barrier(0);
          load(ks);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  using P2 = std::integral_constant<int, 2>;
  using P3 = std::integral_constant<int, 3>;
  // Step k, LEFT steps after it (2: at least two).
  auto step = [&](int k, auto left_t) {
    constexpr int LEFT = decltype(left_t)::value;
    uint32_t a[4], b[4];
    auto addr = [&](uint32_t (&d)[4], const uint32_t (&base)[4], int off) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) d[ks] = base[ks] + (uint32_t)off;
    };
    addr(a, xa, at(k, 1));
    read_blocks(xf, a);
    wait_vmcnt<10>();
    lds_barrier();
    mma(P0{}, [&](int i) {
      if (LEFT >= 1) load_w(k + 1, i < 2 ? 2 : 3, i & 1);
      else if (i < 2) load_v(0, 3, i);
    });
    addr(a, wa, at(k, 2));
    read_one(w[1], a);
    wait_vmcnt<(LEFT >= 1 ? 12 : 10)>();
    lds_barrier();
    mma(P1{}, [&](int i) {
      if (i >= 2) return;
      if (LEFT >= 2) load_w(k + 2, 0, i);
      else if (LEFT == 1) load_v(0, 0, i);
    });
    addr(a, wa, at(k, 3));
    read_one(w[0], a);
    wait_vmcnt<(LEFT >= 1 ? 10 : 8)>();
    lds_barrier();
    mma(P2{}, [&](int i) {
      if (i >= 2) return;
      if (LEFT >= 2) load_x(k + 2, i);
      else if (LEFT == 1) load_v(0, 1, i);
    });
    addr(a, wa, at(k, 4));
    if constexpr (LEFT >= 1) {
      addr(b, wa, at(k + 1, 0));
      read_two(w[1], w[0], a, b);
      wait_vmcnt<10>();
    } else {
      read_one(w[1], a);
    }
    lds_barrier();
    mma(P3{}, [&](int i) {
      if (i >= 2) return;
      if (LEFT >= 2) load_w(k + 2, 1, i);
      else if (LEFT == 1) load_v(0, 2, i);
    });
  };
  // The first eight pieces, in ring order.
#pragma unroll
  for (int j = 0; j < 2; ++j) load_w(0, 0, j);
#pragma unroll
  for (int j = 0; j < 2; ++j) load_x(0, j);
#pragma unroll
  for (int h = 1; h < 4; ++h)
#pragma unroll
    for (int j = 0; j < 2; ++j) load_w(0, h, j);
#pragma unroll
  for (int j = 0; j < 2; ++j) load_w(1, 0, j);
#pragma unroll
  for (int j = 0; j < 2; ++j) load_x(1, j);
#pragma unroll
  for (int j = 0; j < 2; ++j) load_w(1, 1, j);
  wait_vmcnt<14>();
  lds_barrier();
  {
    const uint32_t a[4] = {wa[0] + (uint32_t)at(0, 0), wa[1] + (uint32_t)at(0, 0), wa[2] + (uint32_t)at(0, 0),
                           wa[3] + (uint32_t)at(0, 0)};
    read_one(w[0], a);
  }
  wait_vmcnt<12>();
  lds_barrier();
  if (wave >= 4) lds_barrier();   // one section behind
  int k = 0;
  for (; k < KT - 2; ++k) step(k, std::integral_constant<int, 2>{});
  step(k, std::integral_constant<int, 1>{});
  step(k + 1, std::integral_constant<int, 0>{});
  if (wave < 4) lds_barrier();
  wait_vmcnt<0>();                // the W2^T quarters
  __syncthreads();

  // ML2 over half hf of the hidden units: S = ReLU(P + b1) as bf16 fragments in
  // slots 4..7, [wm][32-row block][k step of 16 hidden units][lane][16 B]; W2^T rows
  // 32 wn .. +31 are quarter wn.
  f32x16_t o[2];
#pragma unroll
  for (int bm = 0; bm < 2; ++bm)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[bm][i] = 0.0f;
  char* const xs = smem + (4 + 2 * wm) * kWPiece + lane * 16;
  const char* const w2l = smem + wn * kWPiece + lr * W2_ROWB;
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    if (hf == 1) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < 2; ++j) load_v(512, q, j);
    }
#pragma unroll
    for (int bm = 0; bm < 2; ++bm)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const f32x16_t& v = acc[bm][2 * hf + h];
          u32x4_t f;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            f[e] = pack_bf16x2(fmaxf(v[8 * s + 2 * e], 0.0f), fmaxf(v[8 * s + 2 * e + 1], 0.0f));
          lds_write16(xs + (bm * 16 + h * 8 + wn * 2 + s) * 1024, f);
        }
    wait_vmcnt<0>();
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
      const u32x4_t a = lds_read16(w2l + (((2 * ks + lg) ^ (lr & 15)) << 4));
#pragma unroll
      for (int bm = 0; bm < 2; ++bm) Mma<bf16_t>::run(o[bm], a, lds_read16(xs + (bm * 16 + ks) * 1024));
    }
    __syncthreads();   // every wave is done with the W2^T half and the S exchange
  }

  // O to LDS (fp32 rows), then + b2 (ReLU) as bf16: thread t takes 8 columns of
  // row t / 16 + 32 j, so every wave-wide store covers four whole rows.
#pragma unroll
  for (int bm = 0; bm < 2; ++bm)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4_t*>(smem + (wm * 64 + bm * 32 + lr) * PT_ROWB + (wn * 32 + 8 * g + 4 * lg) * 4) =
          f32x4_t{o[bm][4 * g], o[bm][4 * g + 1], o[bm][4 * g + 2], o[bm][4 * g + 3]};
  const int n = (tid & 15) * 8;
  uint16_t* O = p.O + (int64_t)bz * p.so;
  float bb[8] = {};
  if (p.b2) {
    load4<float>(p.b2 + n, reinterpret_cast<float(&)[4]>(bb[0]));
    load4<float>(p.b2 + n + 4, reinterpret_cast<float(&)[4]>(bb[4]));
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = (tid >> 4) + 32 * j, m = m0 + r;
    if (m >= p.M) continue;
    const float* src = reinterpret_cast<const float*>(smem + r * PT_ROWB) + n;
    float y[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      y[q] = src[q];
      if (p.b2) y[q] += bb[q];
      if (p.out_relu) y[q] = fmaxf(y[q], 0.0f);
    }
    const u32x4_t v = {pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]),
                       pack_bf16x2(y[6], y[7])};
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t*>(O + (int64_t)m * p.ldo + n));
  }
}

// ---------------------------------------------------------------------------
// Few rows.  On 128-row blocks a batch of a few thousand rows leaves most CUs
// without a workgroup, and the ring's barriers make each k step wait for the
// slowest of its loads.  Here a workgroup owns 32 rows and 256 UPW hidden units;
// its four waves take units of 64 hidden (wave w: w, w + 4) and run both products for them
// on their own.  The rows of X (at most 1024 wide) stay in LDS, the only thing the
// waves share; the weights stream through a ring of S stages per wave, each stage
// 64 rows x 128 bytes (whole lines): K / 64 stages of W1^T, then two of W2^T (64
// output rows, the unit's 64 hidden each).  No barrier between the arrival of X and
// the sum of the waves' O tiles (in wave order, through LDS).  What bounds it is the CU's
// load path: 512 K + 64 KB of weights per 256 hidden units (1 KB per about 32 cycles).
// The register hand-off of S is the 128-row kernels'.
// ---------------------------------------------------------------------------
constexpr int kMlpRowsLds = 160 * 1024;
template <int UPW, int S>
struct MlpFew {
  static constexpr int TM = 32, NW = 4, NT = 64 * NW, N2 = 128;
  static constexpr int STAGE = 64 * 128, RING = S * STAGE, OFF_X = NW * RING;
  static constexpr int MAX_K = (kMlpRowsLds - OFF_X) / (TM * 2);
  static constexpr int PITCH = N2 * 4 + 16, TILE = TM * PITCH;   // one wave's O tile
  static_assert(NW * TILE + 16 <= OFF_X, "O tiles and the flag over the rings");
};

template <int UPW, int S>
__global__ __launch_bounds__(256, 1) __attribute__((amdgpu_waves_per_eu(1, 1)))
void b2b_mlp_few_kernel(B2BParams p) {
  using F = MlpFew<UPW, S>;
  __shared__ __attribute__((aligned(16))) char smem[kMlpRowsLds];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lg = lane >> 5;
  const int cn = p.cn, c = blockIdx.x % cn, rb = blockIdx.x / cn;
  const int bz = blockIdx.y, m0 = rb * F::TM;
  const int KT = p.K / 64, SPU = KT + 2, n_st = UPW * SPU;
  const int h0 = c * 256 * UPW + 64 * wave;       // the wave's unit u: hidden h0 + 256 u .. + 63
  const char* W1 = reinterpret_cast<const char*>(p.W1 + (int64_t)bz * p.sw1 + (int64_t)h0 * p.ldw1);
  const char* W2 = reinterpret_cast<const char*>(p.W2 + (int64_t)bz * p.sw2 + h0);

  // b1 in accumulator order: elements 8 s .. 8 s + 7 of block bn hold hidden
  // units 32 bn + 16 s + 8 lg + 0..7 of the unit.
  f32x4_t b1v[UPW][8] = {};
  if (p.b1) {
#pragma unroll
    for (int u = 0; u < UPW; ++u)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        b1v[u][i] = *reinterpret_cast<const f32x4_t*>(p.b1 + h0 + 256 * u + 32 * (i >> 2) + 16 * ((i >> 1) & 1) +
                                                      8 * lg + 4 * (i & 1));
  }

  // A wave-wide load fills 8 rows of 128 bytes: row r, 16-byte chunk c at position
  // c ^ ((r >> 1) & 7) (conflict-free fragment reads).  X: 64-wide k blocks of 32
  // rows (4 KB), the wave loads rows 8 wave .. + 7 of each.
  const int r8 = lane >> 3, ch = (lane & 7) ^ (lane >> 4);
  {
    const char* xg = reinterpret_cast<const char*>(p.X + (int64_t)bz * p.sx +
                                                   (int64_t)min(m0 + 8 * wave + r8, p.M - 1) * p.ldx) +
                     (ch ^ ((wave & 1) << 2)) * 16;
    char* dst = smem + F::OFF_X + wave * 1024;
    for (int kb = 0; kb < KT; ++kb) dma16(xg + 128 * kb, dst + 4096 * kb);
  }
  // Load j (rows 8 j .. + 7) of a stage.  W1^T: the rows of each 32-row block are
  // taken with bits 2 and 3 of the row swapped, so load j starts at row
  // 16 (j / 2) + 4 (j % 2) and the lane's bit 2 counts 8; W2^T: row 8 j.
  char* const ring = smem + wave * F::RING;
  const uint32_t ring0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)ring);
  const int64_t p1 = 2 * p.ldw1, p2 = 2 * p.ldw2;
  const uint32_t l1 = (uint32_t)(((r8 & 3) | ((r8 & 4) << 1)) * p1), l2 = (uint32_t)(r8 * p2);
  struct Src {
    const char* base;
    int64_t d16, dodd;
    uint32_t l;
  };
  int nu = 0, nq = 0, issued = 0;                 // the next stage to load
  auto next = [&]() __attribute__((always_inline)) {
    const bool first = nq < KT;
    const int64_t pitch = first ? p1 : p2;
    Src s{first ? W1 + 256 * nu * p1 + 128 * nq : W2 + 64 * (nq - KT) * p2 + 512 * nu, 16 * pitch,
          (first ? 4 : 8) * pitch, first ? l1 : l2};
    ++issued;
    if (++nq == SPU) nq = 0, ++nu;
    return s;
  };
  auto load = [&](const Src& s, int slot, int j) __attribute__((always_inline)) {
    dma16(s.base + (j >> 1) * s.d16 + (j & 1) * s.dodd + (s.l + (uint32_t)(ch ^ ((j & 1) << 2)) * 16),
          ring + slot * F::STAGE + j * 1024);
  };
#pragma unroll
  for (int st = 0; st < S; ++st) {                // n_st >= S: K >= 128
    const Src s = next();
#pragma unroll
    for (int j = 0; j < 8; ++j) load(s, st, j);
  }
  wait_vmcnt<8 * S>();
  lds_barrier();                                  // X is in LDS

  f32x16_t O[4], P[2];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) O[b][i] = 0.0f;
  const int sw = (lr >> 1) & 7;
  const uint32_t x0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)smem) + F::OFF_X;
  uint32_t fa[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) fa[ks] = lr * 128 + (((2 * ks + lg) ^ sw) << 4);
  u32x4_t f[2][4], x[1][4];
  int st = 0, slot = 0;
  // Fragments of the oldest stage; its slot then takes stage st + S, whose loads
  // go between the MFMAs.
  auto open = [&]() __attribute__((always_inline)) {
    const int after = n_st - 1 - st;              // at most S - 1 stages are in flight behind st
    if (after >= S - 1) wait_vmcnt<8 * (S - 1)>();
    else if (after == 2) wait_vmcnt<16>();
    else if (after == 1) wait_vmcnt<8>();
    else wait_vmcnt<0>();
    uint32_t a[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) a[ks] = ring0 + slot * F::STAGE + fa[ks];
    read_blocks(f, a);
  };
  auto products = [&](f32x16_t& d0, f32x16_t& d1, const u32x4_t (&b)[4]) __attribute__((always_inline)) {
    const bool more = issued < n_st;
    Src s{};
    if (more) s = next();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      Mma<bf16_t>::run(i & 1 ? d1 : d0, f[i & 1][i >> 1], b[i >> 1]);
      __builtin_amdgcn_sched_barrier(0);
      if (more) load(s, slot, i);
      __builtin_amdgcn_sched_barrier(0);
    }
    ++st;
    if (++slot == S) slot = 0;
  };
#pragma unroll
  for (int u = 0; u < UPW; ++u) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) P[i >> 2][4 * (i & 3) + e] = b1v[u][i][e];
#pragma unroll 1
    for (int kb = 0; kb < KT; ++kb) {             // P^T += W1^T X^T
      open();
      uint32_t a[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) a[ks] = x0 + kb * 4096 + fa[ks];
      read_blocks(x, a);
      products(P[0], P[1], x[0]);
    }
    u32x4_t sf[4];                                // S = ReLU(P): k step 2 bn + s of the second product
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        sf[i][e] = pack_bf16x2(fmaxf(P[i >> 1][8 * (i & 1) + 2 * e], 0.0f), fmaxf(P[i >> 1][8 * (i & 1) + 2 * e + 1], 0.0f));
#pragma unroll
    for (int h = 0; h < 2; ++h) {                 // O^T += W2^T S^T, output rows 64 h .. + 63
      open();
      products(O[2 * h], O[2 * h + 1], sf);
    }
  }

  __syncthreads();   // every wave is done with its ring
  {
    char* dst = smem + wave * F::TILE + lr * F::PITCH + 16 * lg;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4_t*>(dst + (32 * b + 8 * g) * 4) =
            f32x4_t{O[b][4 * g], O[b][4 * g + 1], O[b][4 * g + 2], O[b][4 * g + 3]};
  }
  __syncthreads();
  f32x4_t t[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const char* src = smem + ((tid >> 5) + 8 * j) * F::PITCH + (tid & 31) * 16;
    t[j] = *reinterpret_cast<const f32x4_t*>(src);
#pragma unroll
    for (int w = 1; w < F::NW; ++w) t[j] += *reinterpret_cast<const f32x4_t*>(src + w * F::TILE);
  }
  mlp_commit<F::TM, F::NT, F::N2>(p, [&](int j) { return t[j]; }, bz, gridDim.x / cn, rb, cn, c, m0,
                                  *reinterpret_cast<int*>(smem + F::NW * F::TILE));
}

bool b2b_mlp_supported(int K, int N1, int N2) {
  return N2 == 128 && N1 % kMlpHidden == 0 && N1 > 0 && K % 64 == 0 && K / 64 >= MlpS::STAGES - 1;
}

hipError_t launch_b2b_mlp(const B2BParams& p, hipStream_t st) {
  if (!b2b_mlp_supported(p.K, p.N1, p.N2) || (p.cn != 1 && p.cn != p.N1 / kMlpHidden)) return hipErrorInvalidValue;
  // 32-row workgroups of 256 hidden units while they fit one generation of 256 CUs
  // (each streams its share of the weights), of 512 while those do; K limited by X in
  // LDS.  Without the split's workspace a row block is one workgroup.  Measured (us,
  // this form / 128-row forms, K x N1): 1 row 256 x 256 5.6 / 10.5, 1024 x 512 12.3 / 20.1;
  // 1000 rows 512 x 512 10.6 / 18.7; 4000 rows 1024 x 512 16.7 / 24.3; with two units a wave:
  // 8000 rows 256 x 512 9.7 / 17.5, 1024 x 512 22.0 / 25.3, 4000 rows 1024 x 1024 24.5 / 26.6.  A
  // second generation (or a third unit a wave) costs more than the 128-row forms.
  const int cn_all = p.N1 / kMlpHidden;
  const int64_t few_rbs = (p.M + 31) / 32;
  const bool single = p.K <= 1024 && (cn_all == 1 || p.cn > 1) && few_rbs * p.batch * cn_all <= 256;
  const bool pairs = p.K <= 1024 && cn_all % 2 == 0 && (cn_all == 2 || p.cn > 1) && few_rbs * p.batch * cn_all <= 512;
  if (single || pairs) {
    B2BParams q = p;
    q.cn = single ? cn_all : cn_all / 2;
    const dim3 grid((unsigned)(few_rbs * q.cn), (unsigned)q.batch), block(256);
    if (single) {
      if (q.K <= 512) hipLaunchKernelGGL((b2b_mlp_few_kernel<1, 4>), grid, block, 0, st, q);
      else hipLaunchKernelGGL((b2b_mlp_few_kernel<1, 3>), grid, block, 0, st, q);
    } else {
      if (q.K <= 512) hipLaunchKernelGGL((b2b_mlp_few_kernel<2, 4>), grid, block, 0, st, q);
      else hipLaunchKernelGGL((b2b_mlp_few_kernel<2, 3>), grid, block, 0, st, q);
    }
    return hipGetLastError();
  }
  const unsigned rbs = (unsigned)((p.M + kMlpRows - 1) / kMlpRows);
  // N1 = 512: the wide form for every whole row block, and also where the chunks
  // would be split but K is short: a workgroup then has little to stream, and the
  // split form's commit costs more than the idle CUs.  Measured at N1 = 512 (us,
  // wide / split): 16384 x 256 15.1 / 20.2, 16384 x 512 19.8 / 23.0, 16384 x 1024 29.3 / 29.7;
  // against the chunked whole form: 65536 x 1024 77.8 / 92 on one box (90.6 / 101 on another),
  // 65536 x 256 33.7 / 45.7.
  const bool wide = p.N1 == 512 && (p.cn == 1 || p.K <= 512);
  const dim3 grid(rbs * (unsigned)(wide ? 1 : p.cn), (unsigned)p.batch), block(MlpS::NT);
  if (wide) hipLaunchKernelGGL((b2b_mlp_wide_kernel<128>), grid, dim3(512), 0, st, p);
  else if (p.cn == 1) hipLaunchKernelGGL((b2b_mlp_whole_kernel<128>), grid, block, 0, st, p);
  else hipLaunchKernelGGL((b2b_mlp_kernel<128>), grid, block, 0, st, p);
  return hipGetLastError();
}

}  // namespace cf
