// GEMM (+ row subgraph) on small tiles, for products with few rows.
//
// With 128-row tiles a short batch gives a handful of workgroups, and each of
// them streams its operands through one CU's load path (about 75 GB/s) while
// most CUs idle: 333 x 768 x 3072 ran on 18 workgroups.  Here a tile is 32 or 64
// rows by 32 or 64 columns, so the same product has 132.
//
// Split K inside the workgroup.  A tile this small has too little work per k
// step for waves to share, so each of the four waves computes the whole tile
// over every fourth 128-byte k stage, with a ring of S stages of its own in
// LDS: no barrier in the main loop, and S stages per wave (128 or 144 KB per
// workgroup) in flight to cover the memory latency.  The four partial tiles are
// added through LDS in wave order.
//
// Pairs.  Row clusters of more than 8 peers take half the stages (48 or 64 KB), so
// that two workgroups fit a CU and the peers of overlapping calls, which wait for
// each other, all find a place.  The stage's next contents are on their way while
// its MFMAs run, so little is lost: post-norm 333 x 768 x 3072 14.7 us (deep ring
// 13.7), 333 x 768 x 768 8.8 (9.1), fp32 128 x 768 x 768 13.3 (14.5).
//
// Rows.  For the epilogue a row belongs to 256 / TM neighbouring lanes, so row
// reductions are lane exchanges and every global access is a row segment.  The
// row statistics of a tile are completed by the row-cluster exchange (the cn
// workgroups of a row block share an XCD and exchange tagged records through
// its L2; see cluster_exchange for the protocol, which this kernel follows: one
// add to the group's round counter per tile, records that carry the round,
// bounded waits, the sticky error word; only the add goes out in front of the main
// loop here, whose first wait then covers it).  A record's position here is peer x TM
// + row within the slot's area; positions of different slots never meet, so any
// record in a slot's area carries a round of that slot whatever tile wrote it.
//
// K need not fill whole stages: chunks past K are loaded from clamped addresses
// and replaced by zeros in the fragments of the last stage.
#include "cf_gemm_tile.h"

namespace cf {

namespace {

template <typename T_, int BM_, int BN_, bool KN_, bool PAIR_>
struct Small {
  using T = T_;
  static constexpr int BM = BM_, BN = BN_, NW = 4, NT = 256;
  static constexpr bool KN = KN_;                  // W stored K x N (bf16)
  static constexpr int TM = 32 * BM, TN = 32 * BN;
  static constexpr int EPC = 16 / (int)sizeof(T);  // elements per 16-byte chunk
  static constexpr int TK = 8 * EPC;               // k per 128-byte stage
  static constexpr int STAGE = (TM + TN) * 128;
  static constexpr int PX = TM / 8, PW = TN / 8;   // wave-wide loads per stage
  static constexpr bool PAIR = PAIR_;              // two workgroups fit a CU
  static constexpr int S = PAIR ? (BM + BN == 2 ? 2 : 1) : BM + BN == 2 ? 4 : BM + BN == 3 ? 3 : 2;
  static constexpr int RING = S * STAGE;           // one wave's ring
  static constexpr int PITCH = TN * 4 + 16;        // row of a partial tile
  static constexpr int TPR = NT / TM;              // lanes per row
  static constexpr int CPT = TN / TPR;             // columns per lane
  static constexpr int G = CPT < 8 ? CPT : 8, NG = CPT / G;   // consecutive columns, groups of them
  static constexpr int TAG = NW * (RING > TM * PITCH ? RING : TM * PITCH);   // rings, partial tiles; then the round tag
  static constexpr int LDS = TAG + 16;
  static_assert(LDS <= (PAIR ? 80 : 160) * 1024, "LDS budget");
  static_assert(!KN || sizeof(T) == 2, "K x N: bf16");
  static_assert((PX + PW) * S < 64, "vmcnt range");
  static_assert(TM <= kRecRows, "records of kClusterPeers peers");
};

// The K x N form: fragments of one 32-column block by transposing reads, k
// rows of ROWB bytes; a0 and a1 address the k rows 0..3 and 4..7 of the lane's
// first chunk (k step 0), the steps are 16 rows apart.
template <int ROWB>
__device__ __forceinline__ void read_block_kn(u32x4_t (&w)[4], uint32_t a0, uint32_t a1) {
  u32x2_t v[8];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %9\n\t"
      "ds_read_b64_tr_b16 %2, %8 offset:%10\n\tds_read_b64_tr_b16 %3, %9 offset:%10\n\t"
      "ds_read_b64_tr_b16 %4, %8 offset:%11\n\tds_read_b64_tr_b16 %5, %9 offset:%11\n\t"
      "ds_read_b64_tr_b16 %6, %8 offset:%12\n\tds_read_b64_tr_b16 %7, %9 offset:%12\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
      : "v"(a0), "v"(a1), "i"(16 * ROWB), "i"(32 * ROWB), "i"(48 * ROWB)
      : "memory");
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) w[ks] = u32x4_t{v[2 * ks][0], v[2 * ks][1], v[2 * ks + 1][0], v[2 * ks + 1][1]};
}

// Publishes (a, b) of the lane's row (b unless MAX) and reads the peers'
// records, peer tq + TPR j by lane tq of the row, until all carry `tag`.
template <class S, int NV, int PP>
__device__ __forceinline__ void small_exchange(const GemmRowsParams& p, int stage, int slot, int c, unsigned tag, float a,
                                               float b, int row, int tq, float (&ra)[PP], float (&rb)[PP],
                                               bool (&has)[PP]) {
  unsigned long long* rec = reinterpret_cast<unsigned long long*>(p.ws_part) + stage * kRecStageWords +
                            (tag & 1u) * kRecSetWords + (size_t)slot * kRecPeers * kRecRows * 2;
  if (tq == 0) {
    unsigned long long* w = rec + (c * S::TM + row) * 2;
    __hip_atomic_store(w, rec_word(a, tag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (NV > 1) __hip_atomic_store(w + 1, rec_word(b, tag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
#pragma unroll
  for (int j = 0; j < PP; ++j) has[j] = tq + S::TPR * j < p.cn;
  for (int spins = 0;; ++spins) {
    const unsigned err = __hip_atomic_load(p.ws_err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long w[PP][NV];
    bool ok = true;
#pragma unroll
    for (int j = 0; j < PP; ++j) {
      const int peer = has[j] ? tq + S::TPR * j : c;
      const unsigned long long* r = rec + (peer * S::TM + row) * 2;
#pragma unroll
      for (int v = 0; v < NV; ++v) w[j][v] = __builtin_nontemporal_load(r + v);
    }
#pragma unroll
    for (int j = 0; j < PP; ++j) {
#pragma unroll
      for (int v = 0; v < NV; ++v) ok = ok && (unsigned)(w[j][v] >> 32) == tag;
      ra[j] = __uint_as_float((unsigned)w[j][0]);
      rb[j] = __uint_as_float((unsigned)w[j][NV - 1]);
    }
    if (__all(ok)) break;
    if (__builtin_amdgcn_readfirstlane(err) != 0u) break;   // an earlier wait failed: give up now
    if (spins >= p.spin_limit) {
      __hip_atomic_store(p.ws_err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      break;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

}  // namespace

template <class S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(S::PAIR ? 2 : 1, S::PAIR ? 2 : 1)))
void gemm_small_kernel(GemmRowsParams p) {
  using T = typename S::T;
  __shared__ __attribute__((aligned(16))) char smem[S::LDS];
  unsigned* const tag_lds = reinterpret_cast<unsigned*>(smem + S::TAG);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lg = lane >> 5;
  const int bz = blockIdx.y;
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
  const bool cluster = p.mode == ROWS_CLUSTER;
  const T* X = reinterpret_cast<const T*>(p.X) + (int64_t)bz * p.sx;
  const T* W = reinterpret_cast<const T*>(p.W) + (int64_t)bz * p.sw;
  const RowEpi& e = p.epi;
  const int M = p.M, N = p.N, K = p.K;
  const int KT = (K + S::TK - 1) / S::TK, KC = K / S::EPC;   // stages, 16-byte chunks per row
  const int n_st = (KT - wave + S::NW - 1) / S::NW;          // this wave's stages: wave, wave + 4, ...
  char* const ring = smem + wave * S::RING;
  const uint32_t ring0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)ring);

  for (int it = 0;; ++it) {
    // Tile.  Row clusters: row block rb on XCD rb % 8, its cn peers side by side
    // there (as the 128-row tiles).  Otherwise each XCD takes a contiguous range
    // of the tiles, column tile by column tile: the row blocks of one share an
    // XCD, which then fetches that part of W once.  (Whole column tiles per XCD
    // gave four of the XCDs two rounds at 1100 x 768 x 768: 12.1 us; here 7.7.)
    int rb, c;
    if (cluster) {
      rb = (it * p.slots + local / p.cn) * 8 + xcd;
      c = local % p.cn;
      if (rb >= p.num_rb) break;
    } else {
      const int tiles = p.num_rb * p.cn, q = tiles >> 3;
      const int t = xcd * q + min(xcd, tiles & 7) + local;
      if (it > 0) break;
      rb = t % p.num_rb;
      c = t / p.num_rb;
    }
    const int slot = local / p.cn * 8 + xcd;
    const int m0 = rb * S::TM, n0 = c * S::TN;
    unsigned long long round_old = 0;
    if (cluster && p.cn > 1) round_old = round_begin(p, slot, lane, wave);

    // Loads of a stage: 8 rows x 128 bytes each, chunk ch of row r at position
    // ch ^ ((r >> 1) & 7) (conflict-free fragment reads).  K x N: 64 k rows of
    // TN columns; with 128-byte rows the two 64-byte blocks of row k are swapped
    // where bit 1 of k is set, so that the four k rows of a transposing read lie
    // on distinct banks.
    uint32_t xo[S::PX], wo[S::PW];
#pragma unroll
    for (int j = 0; j < S::PX; ++j)
      xo[j] = (uint32_t)min(8 * j + (lane >> 3), M - 1 - m0) * (uint32_t)(p.ldx * sizeof(T));
    const int ch0 = (lane & 7) ^ (lane >> 4);                  // chunk of the lane, even loads (odd: ^ 4)
    constexpr int LPK = S::TN / 8;                             // K x N: lanes per k row
    const int kr = lane / LPK, kp = lane % LPK;
#pragma unroll
    for (int j = 0; j < S::PW; ++j) {
      if constexpr (S::KN) {
        const int k = j * (64 / LPK) + kr, q = S::BN == 2 ? kp ^ (((k >> 1) & 1) << 2) : kp;
        wo[j] = (uint32_t)min(8 * q, N - 8 - n0) * 2u;
      } else {
        wo[j] = (uint32_t)min(8 * j + (lane >> 3), N - 1 - n0) * (uint32_t)(p.ldw * sizeof(T));
      }
    }
    const char* xg = reinterpret_cast<const char*>(X + (int64_t)m0 * p.ldx);
    const char* wg = reinterpret_cast<const char*>(W) + (S::KN ? (int64_t)n0 : (int64_t)n0 * p.ldw) * (int)sizeof(T);
    // Load j of stage st into ring slot sl.
    auto load = [&](int st, int sl, int j) {
      char* dst = ring + sl * S::STAGE + j * 1024;
      if (j < S::PX) {
        dma16(xg + xo[j] + (uint32_t)min(st * 8 + (ch0 ^ ((j & 1) << 2)), KC - 1) * 16u, dst);
      } else if constexpr (S::KN) {
        const int k = min(st * S::TK + (j - S::PX) * (64 / LPK) + kr, K - 1);
        dma16(wg + (int64_t)k * p.ldw * 2 + wo[j - S::PX], dst);
      } else {
        dma16(wg + wo[j - S::PX] + (uint32_t)min(st * 8 + (ch0 ^ ((j & 1) << 2)), KC - 1) * 16u, dst);
      }
    };
    static_assert(S::PX % 2 == 0, "W loads keep the parity of their row group");
#pragma unroll
    for (int i = 0; i < S::S; ++i)
      if (i < n_st)
#pragma unroll
        for (int j = 0; j < S::PX + S::PW; ++j) load(wave + i * S::NW, i, j);

    // Epilogue operands of the lane's row segment, on their way under the main loop.
    const int row = tid / S::TPR, tq = tid % S::TPR, m = m0 + row;
    const bool mv = m < M;
    auto col = [&](int g) { return n0 + g * (S::TPR * S::G) + tq * S::G; };

    f32x16_t acc[S::BM][S::BN];
#pragma unroll
    for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
      for (int bn = 0; bn < S::BN; ++bn)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[bm][bn][i] = 0.0f;
    const int sw = (lr >> 1) & 7;
    int sl = 0;
#pragma unroll 1
    for (int i = 0; i < n_st; ++i) {
      constexpr int P = S::PX + S::PW;
      // stage i has landed: at most the stages after it are outstanding
      const int after = min(S::S - 1, n_st - 1 - i);
      if (after >= 3) wait_vmcnt<3 * P < 64 ? 3 * P : 63>();
      else if (after == 2) wait_vmcnt<2 * P>();
      else if (after == 1) wait_vmcnt<P>();
      else wait_vmcnt<0>();
      const int st = wave + i * S::NW;
      u32x4_t xf[S::BM][4], wf[S::BN][4];
      uint32_t a[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) a[ks] = ring0 + sl * S::STAGE + lr * 128 + (((2 * ks + lg) ^ sw) << 4);
      read_blocks(xf, a);
      if constexpr (S::KN) {
        constexpr int ROWB = S::TN * 2;
        const int r = lane & 15, k = 8 * lg + (r >> 2);   // and k + 4: bit 1 of k is that of r >> 2
#pragma unroll
        for (int bn = 0; bn < S::BN; ++bn) {
          const int nb = (bn * 32 + (lane & 16) + 4 * (r & 3)) * 2;
          const uint32_t w0 = ring0 + sl * S::STAGE + S::TM * 128 + k * ROWB +
                              (S::BN == 2 ? nb ^ (((r >> 3) & 1) << 6) : nb);
          read_block_kn<ROWB>(wf[bn], w0, w0 + 4 * ROWB);
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) a[ks] += S::TM * 128;
        read_blocks(wf, a);
      }
      if (K % S::TK != 0 && st == KT - 1) {   // chunks past K contribute nothing
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          if (st * 8 + 2 * ks + lg >= KC) {
#pragma unroll
            for (int b = 0; b < S::BM; ++b) xf[b][ks] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
            for (int b = 0; b < S::BN; ++b) wf[b][ks] = u32x4_t{0u, 0u, 0u, 0u};
          }
      }
      // The stage's fragments are in registers, so its slot takes stage i + S;
      // the loads go between the MFMAs.
      const bool more = i + S::S < n_st;
      constexpr int NM = 4 * S::BM * S::BN, LPM = (P + NM - 1) / NM;
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        const int ks = q / (S::BM * S::BN), b = q % (S::BM * S::BN);
        Mma<T>::run(acc[b / S::BN][b % S::BN], wf[b % S::BN][ks], xf[b / S::BN][ks]);
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
#pragma unroll
          for (int l = 0; l < LPM; ++l)
            if (q * LPM + l < P) load(st + S::S * S::NW, sl, q * LPM + l);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      sl = sl + 1 == S::S ? 0 : sl + 1;
    }

    // Residual and bias of the row segment (issued before the tile's sums meet).
    float rs[S::NG][S::G], bs[S::NG][S::G];
#pragma unroll
    for (int g = 0; g < S::NG; ++g)
#pragma unroll
      for (int q = 0; q < S::G; q += 4) {
        const int n = min(col(g) + q, N - 4);
        float t[4] = {0.0f, 0.0f, 0.0f, 0.0f}, u[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (e.R && mv) load4_once<T>(reinterpret_cast<const T*>(e.R) + (int64_t)bz * e.sr + (int64_t)m * e.ldr + n, t);
        if (e.bias) load4<float>(e.bias + n, u);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          rs[g][q + i] = t[i];
          bs[g][q + i] = u[i];
        }
      }
    if (tid == 0) *tag_lds = round_tag(round_old);
    __syncthreads();   // every wave is done with its ring
    {
      char* part = smem + wave * S::TM * S::PITCH;
#pragma unroll
      for (int bm = 0; bm < S::BM; ++bm)
#pragma unroll
        for (int bn = 0; bn < S::BN; ++bn)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            *reinterpret_cast<f32x4_t*>(part + (bm * 32 + lr) * S::PITCH + (bn * 32 + 8 * g + 4 * lg) * 4) =
                f32x4_t{acc[bm][bn][4 * g], acc[bm][bn][4 * g + 1], acc[bm][bn][4 * g + 2], acc[bm][bn][4 * g + 3]};
    }
    __syncthreads();
    const unsigned tag = __builtin_amdgcn_readfirstlane(*tag_lds);

    // ---- stage 1: x = alpha * acc + bias + R; only given terms are added
    float x[S::NG][S::G];
    bool val[S::NG];
#pragma unroll
    for (int g = 0; g < S::NG; ++g) {
      val[g] = col(g) < N;
#pragma unroll
      for (int q = 0; q < S::G; q += 4) {
        const char* src = smem + row * S::PITCH + (g * (S::TPR * S::G) + tq * S::G + q) * 4;
        f32x4_t s = *reinterpret_cast<const f32x4_t*>(src);
#pragma unroll
        for (int w = 1; w < S::NW; ++w) s += *reinterpret_cast<const f32x4_t*>(src + w * S::TM * S::PITCH);
#pragma unroll
        for (int i = 0; i < 4; ++i) x[g][q + i] = s[i];
      }
    }
    auto each = [&](auto f) {
#pragma unroll
      for (int g = 0; g < S::NG; ++g)
#pragma unroll
        for (int q = 0; q < S::G; ++q) f(x[g][q], g, q);
    };
    if (e.alpha != 1.0f) each([&](float& v, int, int) { v *= e.alpha; });
    if (e.bias) each([&](float& v, int g, int q) { v += bs[g][q]; });
    if (e.R) each([&](float& v, int g, int q) { v += rs[g][q]; });

    constexpr int PP = kClusterPeers / S::TPR;   // peers one lane reads
    const bool peers = cluster && p.cn > 1;
    const float invN = 1.0f / (float)N;
    int stage = 0;
    float ra[PP], rbv[PP];
    bool has[PP];

    // ---- stage 2: row statistics, normalisation.  Columns past N (a ragged
    // last tile, never in a cluster) take no part.
    if (e.norm == NORM_LAYER) {
      float t = 0.0f;
      each([&](float& v, int g, int) { t += val[g] ? v : 0.0f; });
      const float nt = (float)min(S::TN, N - n0);
      float mean = row_sum<S::TPR>(t) / nt, d2 = 0.0f;
      each([&](float& v, int g, int) {
        const float d = v - mean;
        d2 = val[g] ? fmaf(d, d, d2) : d2;
      });
      float m2 = row_sum<S::TPR>(d2);
      if (peers) {
        // k-way form of the pairwise update of Chan, Golub and LeVeque over cn
        // tiles of TN columns: mean = sum mean_c / cn, M2 = sum (M2_c + TN (mean_c - mean)^2)
        small_exchange<S, 2, PP>(p, stage++, slot, c, tag, mean, m2, row, tq, ra, rbv, has);
        t = 0.0f;
#pragma unroll
        for (int j = 0; j < PP; ++j) t += has[j] ? ra[j] : 0.0f;
        mean = row_sum<S::TPR>(t) / (float)p.cn;
        t = 0.0f;
#pragma unroll
        for (int j = 0; j < PP; ++j) {
          const float d = ra[j] - mean;
          t += has[j] ? fmaf((float)S::TN * d, d, rbv[j]) : 0.0f;
        }
        m2 = row_sum<S::TPR>(t);
      }
      const float rstd = rsqrtf(m2 * invN + e.eps);
      each([&](float& v, int, int) { v = (v - mean) * rstd; });
    } else if (e.norm == NORM_RMS) {
      float t = 0.0f;
      each([&](float& v, int g, int) { t = val[g] ? fmaf(v, v, t) : t; });
      t = row_sum<S::TPR>(t);
      if (peers) {
        small_exchange<S, 1, PP>(p, stage++, slot, c, tag, t, t, row, tq, ra, rbv, has);
        t = 0.0f;
#pragma unroll
        for (int j = 0; j < PP; ++j) t += has[j] ? ra[j] : 0.0f;
        t = row_sum<S::TPR>(t);
      }
      const float rstd = rsqrtf(t * invN + e.eps);
      each([&](float& v, int, int) { v *= rstd; });
    }
    if (e.norm != NORM_NONE && (e.gamma || e.beta)) {
#pragma unroll
      for (int g = 0; g < S::NG; ++g)
#pragma unroll
        for (int q = 0; q < S::G; q += 4) {
          const int n = min(col(g) + q, N - 4);
          float ga[4] = {1.0f, 1.0f, 1.0f, 1.0f}, be[4] = {0.0f, 0.0f, 0.0f, 0.0f};
          if (e.gamma) load4<float>(e.gamma + n, ga);
          if (e.beta) load4<float>(e.beta + n, be);
#pragma unroll
          for (int i = 0; i < 4; ++i) x[g][q + i] = fmaf(x[g][q + i], ga[i], be[i]);
        }
    }

    // ---- stage 3: activation, softmax, store
    switch (e.act) {
      case ACT_GELU: each([](float& v, int, int) { v = gelu_erf(v); }); break;
      case ACT_GELU_TANH: each([](float& v, int, int) { v = gelu_tanh(v); }); break;
      case ACT_RELU: each([](float& v, int, int) { v = v > 0.0f ? v : 0.0f; }); break;
      case ACT_SOFTCAP: {
        const float cap = e.softcap, inv = 1.0f / cap;
        each([=](float& v, int, int) { v = cap * tanh_exp(v * inv); });
        break;
      }
      default: break;
    }
    if (e.softmax) {
      float mx = -INFINITY;
      each([&](float& v, int g, int) { mx = val[g] ? fmaxf(mx, v) : mx; });
      mx = fmaxf(row_max<S::TPR>(mx), kLowestF32);
      const float nl = softmax_shift(mx);
      float t = 0.0f;
      each([&](float& v, int g, int) {
        v = val[g] ? __builtin_amdgcn_exp2f(fmaf(v, 1.4426950408889634f, nl)) : 0.0f;
        t += v;
      });
      float sm = row_sum<S::TPR>(t), f = 1.0f;
      if (peers) {   // (max, sum) pairs, the sums rescaled to the common maximum
        small_exchange<S, 2, PP>(p, stage++, slot, c, tag, mx, sm, row, tq, ra, rbv, has);
        float mg = -INFINITY;
#pragma unroll
        for (int j = 0; j < PP; ++j) mg = has[j] ? fmaxf(mg, ra[j]) : mg;
        mg = row_max<S::TPR>(mg);
        t = 0.0f;
#pragma unroll
        for (int j = 0; j < PP; ++j)
          t += has[j] ? rbv[j] * __builtin_amdgcn_exp2f((ra[j] - mg) * 1.4426950408889634f) : 0.0f;
        sm = row_sum<S::TPR>(t);
        f = __builtin_amdgcn_exp2f((mx - mg) * 1.4426950408889634f);
      }
      f = f / sm;
      each([&](float& v, int, int) { v *= f; });
    }
    if (e.Y && mv) {
      char* Y = reinterpret_cast<char*>(e.Y) + (int64_t)bz * e.sy * (e.y_f32 ? 4 : 2);
#pragma unroll
      for (int g = 0; g < S::NG; ++g) {
        if (!val[g]) continue;
        const int64_t off = (int64_t)m * e.ldy + col(g);
        if constexpr (S::G == 8) {
          if (!e.y_f32) {
            const u32x4_t o = {pack_bf16x2(x[g][0], x[g][1]), pack_bf16x2(x[g][2], x[g][3]),
                               pack_bf16x2(x[g][4], x[g][5]), pack_bf16x2(x[g][6], x[g][7])};
            __builtin_nontemporal_store(o, reinterpret_cast<u32x4_t*>(reinterpret_cast<bf16_t*>(Y) + off));
            continue;
          }
        }
#pragma unroll
        for (int q = 0; q < S::G; q += 4) {
          const float o[4] = {x[g][q], x[g][q + 1], x[g][q + 2], x[g][q + 3]};
          store4(Y, off + q, e.y_f32, o);
        }
      }
    }

    // ---- stage 4: row amax -> scale -> E4M3 codes
    if (e.quant) {
      float a = 0.0f;
      each([&](float& v, int g, int) { a = val[g] ? fmaxf(a, fabsf(v)) : a; });
      a = row_max<S::TPR>(a);
      if (peers) {
        small_exchange<S, 1, PP>(p, stage, slot, c, tag, a, a, row, tq, ra, rbv, has);
        a = 0.0f;
#pragma unroll
        for (int j = 0; j < PP; ++j) a = has[j] ? fmaxf(a, ra[j]) : a;
        a = row_max<S::TPR>(a);
      }
      const float sc = a / e.qmax;
      if (mv && c == 0 && tq == 0 && e.s_out) e.s_out[m] = sc;
      if (mv && e.q_out) {
        const bool nz = sc > 0.0f;   // a zero row (s = 0) gives codes 0
        const float sd = nz ? sc : 1.0f, inv = nz ? 1.0f / sc : 1.0f;
#pragma unroll
        for (int g = 0; g < S::NG; ++g) {
          if (!val[g]) continue;
#pragma unroll
          for (int q = 0; q < S::G; q += 4) {
            const uint32_t w = e4m3x4(div_rn(x[g][q], sd, inv), div_rn(x[g][q + 1], sd, inv),
                                      div_rn(x[g][q + 2], sd, inv), div_rn(x[g][q + 3], sd, inv));
            *reinterpret_cast<uint32_t*>(e.q_out + (int64_t)m * e.ldq + col(g) + q) = nz ? w : 0u;
          }
        }
      }
    }
    __syncthreads();   // the tile's sums and tag are read; the ring may be filled again
  }
}

template <class S>
static GemmKernel small_entry() {
  const void* f = reinterpret_cast<const void*>(&gemm_small_kernel<S>);
  return GemmKernel{S::TM, S::TN, std::is_same<typename S::T, float>::value ? 1 : 0, S::KN ? 2 : 1, 3, S::NT, 1, S::PAIR ? 1 : 0, f, f};
}

const GemmKernel* gemm_kernels_small(int* n) {
  static const GemmKernel table[] = {
      small_entry<Small<bf16_t, 1, 1, false, false>>(), small_entry<Small<bf16_t, 1, 2, false, false>>(),
      small_entry<Small<bf16_t, 2, 2, false, false>>(), small_entry<Small<bf16_t, 1, 1, true, false>>(),
      small_entry<Small<bf16_t, 1, 2, true, false>>(),  small_entry<Small<bf16_t, 2, 2, true, false>>(),
      small_entry<Small<float, 1, 1, false, false>>(),  small_entry<Small<float, 1, 2, false, false>>(),
      small_entry<Small<float, 2, 2, false, false>>(),
      small_entry<Small<bf16_t, 1, 1, false, true>>(),  small_entry<Small<bf16_t, 1, 2, false, true>>(),
      small_entry<Small<bf16_t, 2, 2, false, true>>(),  small_entry<Small<bf16_t, 1, 1, true, true>>(),
      small_entry<Small<bf16_t, 1, 2, true, true>>(),   small_entry<Small<bf16_t, 2, 2, true, true>>(),
      small_entry<Small<float, 1, 1, false, true>>(),   small_entry<Small<float, 1, 2, false, true>>(),
      small_entry<Small<float, 2, 2, false, true>>(),
  };
  *n = (int)(sizeof(table) / sizeof(table[0]));
  return table;
}

}  // namespace cf
