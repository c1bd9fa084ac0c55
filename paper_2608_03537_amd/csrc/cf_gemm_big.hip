// Plain GEMM on 256 x 256 tiles for large bf16 products: C = alpha X W + bias.
//
// One workgroup of eight waves per tile, two waves per SIMD.  The wave tile is
// 128 x 64 (128 accumulator registers), so a 64-deep k step streams 64 KB of
// operands for 4.2 MMAC, half the bytes per MAC of the 128 x 256 tile, whose
// loop runs at the L2-to-LDS rate.
//
// Half tiles.  A k step consists of four 16 KB pieces: X0, X1 (rows 0..127 and
// 128..255 of the tile, 64 k each) and W0, W1 (columns 0..127, 128..255).  LDS
// holds two steps (2 x 64 KB).  A wave owns rows 64 wm .. +63 of both X halves
// and columns 32 wn .. +31 of both W halves; one phase multiplies one X half by
// one W half (8 MFMAs of 32 x 32 x 16 per wave), four phases make a step:
//     even steps   X0 W0,  X0 W1,  X1 W1,  X1 W0
//     odd steps    X0 W1,  X0 W0,  X1 W0,  X1 W1
// so that each phase needs one new piece: X0, the second W half, X1, and the
// first W half of the next step (read into the registers that the last phase
// no longer uses).  A piece's LDS space is free for the step after next as soon
// as every wave has read it, which is one phase after its read; pieces are
// loaded in the order in which they are read, one per phase, seven phases
// ahead (up to 112 KB in flight).
//
// Ping-pong.  Every wave alternates a read section (the LDS reads of the phase's
// piece, and the waits) with an MFMA section (8 MFMAs, 256 cycles of the SIMD's
// matrix core, and two direct-to-LDS loads of 1 KB between them: in the read
// section the loads held up the LDS reads behind them), a barrier after each.
// Waves 4..7 run one section behind waves 0..3, and waves w and w + 4 share a
// SIMD, so one of the two always issues MFMAs while the other reads.
//
// Waits.  In phase p (counted over all steps) a wave reads piece p + 1 (piece 0
// is read before the loop) and then, with its MFMAs, issues piece p + 8.  Before
// the barrier that ends its read section it waits for its own share of piece
// p + 2, which leaves at most the pieces p + 3 .. p + 7 (two loads each)
// outstanding.  Waves 4..7 do the same one section later, still before the
// barrier in front of the read section in which waves 0..3 read that piece.  A piece read in phase p has
// been read by all waves (each waits for its LDS reads before its barrier) two
// sections later, when waves 0..3 start the read section of phase p + 1, and
// its space is overwritten from there on.
#include "cf_gemm_tile.h"

namespace cf {

namespace {

constexpr int kBigT = 256;                       // tile rows and columns
constexpr int kBigHalf = 16384;                  // bytes of one half-tile piece
constexpr int kBigStep = 4 * kBigHalf;           // X0, X1, W0, W1
constexpr int kBigPitch4 = kBigT * 4 + 16;       // staged output row, fp32
constexpr int kBigPitch2 = kBigT * 2 + 8;        // staged output row, bf16
constexpr int kBigLds = 128 * kBigPitch4 > 2 * kBigStep ? 128 * kBigPitch4 : 2 * kBigStep;
constexpr int kBigGroup = 8;                     // row blocks per group of the tile order

// Eight 16-byte LDS reads (one X half of a wave: k steps 0..3 of row blocks 0
// and 1, 4 KB apart) and the wait for them.  Inline assembly because the
// compiler would wait for every outstanding direct-to-LDS load in front of
// LDS reads it cannot tell apart from the loads' targets; the wait sits in the
// same block, so the outputs are complete when it ends.
template <int OFF>
__device__ __forceinline__ void read_x_half(u32x4_t (&x)[2][4], const uint32_t (&a)[4]) {
  asm volatile(
      "ds_read_b128 %0, %8 offset:%12\n\t"
      "ds_read_b128 %1, %9 offset:%12\n\t"
      "ds_read_b128 %2, %10 offset:%12\n\t"
      "ds_read_b128 %3, %11 offset:%12\n\t"
      "ds_read_b128 %4, %8 offset:%13\n\t"
      "ds_read_b128 %5, %9 offset:%13\n\t"
      "ds_read_b128 %6, %10 offset:%13\n\t"
      "ds_read_b128 %7, %11 offset:%13\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[0][2]), "=&v"(x[0][3]), "=&v"(x[1][0]), "=&v"(x[1][1]),
        "=&v"(x[1][2]), "=&v"(x[1][3])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "i"(OFF), "i"(OFF + 4096)
      : "memory");
}
// One W half of a wave (32 columns): four 16-byte reads, or for W stored K x N
// eight transposing 8-byte reads (k rows 4 apart are 1 KB apart, k steps 4 KB).
template <int OFF>
__device__ __forceinline__ void read_w_half_nk(u32x4_t (&w)[4], const uint32_t (&a)[4]) {
  asm volatile(
      "ds_read_b128 %0, %4 offset:%8\n\t"
      "ds_read_b128 %1, %5 offset:%8\n\t"
      "ds_read_b128 %2, %6 offset:%8\n\t"
      "ds_read_b128 %3, %7 offset:%8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "i"(OFF)
      : "memory");
}
template <int OFF>
__device__ __forceinline__ void read_w_half_kn(u32x4_t (&w)[4], uint32_t a) {
  u32x2_t v[8];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8 offset:%9\n\t"
      "ds_read_b64_tr_b16 %1, %8 offset:%10\n\t"
      "ds_read_b64_tr_b16 %2, %8 offset:%11\n\t"
      "ds_read_b64_tr_b16 %3, %8 offset:%12\n\t"
      "ds_read_b64_tr_b16 %4, %8 offset:%13\n\t"
      "ds_read_b64_tr_b16 %5, %8 offset:%14\n\t"
      "ds_read_b64_tr_b16 %6, %8 offset:%15\n\t"
      "ds_read_b64_tr_b16 %7, %8 offset:%16\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
      : "v"(a), "i"(OFF), "i"(OFF + 1024), "i"(OFF + 4096), "i"(OFF + 5120), "i"(OFF + 8192), "i"(OFF + 9216),
        "i"(OFF + 12288), "i"(OFF + 13312)
      : "memory");
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) w[ks] = u32x4_t{v[2 * ks][0], v[2 * ks][1], v[2 * ks + 1][0], v[2 * ks + 1][1]};
}

// Rows 0..127 or 128..255 of the tile through LDS to coalesced 16-byte stores.
template <int ESZ>
__device__ __forceinline__ void store_half(const f32x16_t (&x)[2][2], char* Y, int64_t ldy, int rows, int cols,
                                           char* smem, int tid, int lane, int wm, int wn) {
  constexpr int PITCH = ESZ == 4 ? kBigPitch4 : kBigPitch2;
  const int lr = lane & 31, lg = lane >> 5;
#pragma unroll
  for (int bm = 0; bm < 2; ++bm)
#pragma unroll
    for (int nh = 0; nh < 2; ++nh)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        char* dst = smem + (wm * 64 + bm * 32 + lr) * PITCH + (nh * 128 + wn * 32 + 8 * g + 4 * lg) * ESZ;
        const f32x16_t& v = x[bm][nh];
        if constexpr (ESZ == 4) {
          *reinterpret_cast<f32x4_t*>(dst) = f32x4_t{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
        } else {
          *reinterpret_cast<u32x2_t*>(dst) =
              u32x2_t{pack_bf16x2(v[4 * g], v[4 * g + 1]), pack_bf16x2(v[4 * g + 2], v[4 * g + 3])};
        }
      }
  __syncthreads();
  constexpr int CPR = kBigT * ESZ / 16, EPC = 16 / ESZ, ITER = 128 * CPR / 512, BATCH = 8;
  static_assert(ITER % BATCH == 0, "store batches");
  const int64_t ldyb = ldy * ESZ;
  const bool full = rows >= 128 && cols >= kBigT;
#pragma unroll 1
  for (int j0 = 0; j0 < ITER; j0 += BATCH) {
    u32x4_t v[BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const int id = tid + (j0 + j) * 512;
      v[j] = *reinterpret_cast<const u32x4_t*>(smem + (id / CPR) * PITCH + (id % CPR) * 16);
    }
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const int id = tid + (j0 + j) * 512, r = id / CPR, cc = id % CPR;
      if (full || (r < rows && cc * EPC < cols))
        __builtin_nontemporal_store(v[j], reinterpret_cast<u32x4_t*>(Y + r * ldyb + cc * 16));
    }
  }
  __syncthreads();
}

}  // namespace

template <bool KN>
__global__ __launch_bounds__(512, 1) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_big_kernel(GemmRowsParams p) {
  __shared__ __attribute__((aligned(16))) char smem[kBigLds];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;          // waves 0..3: wm 0, waves 4..7: wm 1
  const int lr = lane & 31, lg = lane >> 5;
  const int bz = blockIdx.y;

  // Tile order.  Workgroup b runs on XCD b % 8; XCD x takes a contiguous range
  // of the grouped order (groups of 8 row blocks by every column tile, column
  // by column), so the 32 tiles it runs at once share 8 row blocks of X and 4
  // column tiles of W in its L2.
  int rb, c;
  {
    const int T = p.num_rb * p.cn, b = blockIdx.x, x = b & 7, q = T >> 3, r = T & 7;
    const int t = x * q + min(x, r) + (b >> 3);
    const int span = kBigGroup * p.cn;
    const int g0 = t / span * kBigGroup, gsz = min(p.num_rb - g0, kBigGroup), w = t % span;
    rb = g0 + w % gsz;
    c = w / gsz;
  }
  const int m0 = rb * kBigT, n0 = c * kBigT;
  const bf16_t* X = reinterpret_cast<const bf16_t*>(p.X) + (int64_t)bz * p.sx;
  const bf16_t* W = reinterpret_cast<const bf16_t*>(p.W) + (int64_t)bz * p.sw;

  // Direct-to-LDS loads: piece rows are 128 bytes (64 k), a wave-wide load
  // fills 8 of them, load 2 wave + j of a piece rows 8 (2 wave + j) .. +7.  The
  // 16-byte chunk ch of row r sits at chunk position ch ^ ((r >> 1) & 7), which
  // makes the fragment reads (one chunk column of 16 consecutive rows per 16
  // lanes) conflict-free.  W stored K x N: the piece holds 64 k rows of 256
  // bytes as they lie in memory, the 64-byte blocks of row k XOR-swizzled by
  // (k & 3); a load fills 4 rows.  Rows past M and columns past N are clamped
  // (they only feed outputs that are not stored).  Offsets within the tile
  // stay below 2^31 (row pitches are below 2^23 bytes).
  uint32_t xo[2][2], wo[2][2];   // [half][load]
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int row = 8 * (2 * wave + j) + (lane >> 3);
      const int ch = (lane & 7) ^ ((row >> 1) & 7);
      const int m = min(h * 128 + row, p.M - 1 - m0);
      xo[h][j] = (uint32_t)(m * (int)p.ldx * 2 + ch * 16);
      if constexpr (KN) {
        const int k = 4 * (2 * wave + j) + (lane >> 4);
        const int n = min(h * 128 + 8 * ((lane & 15) ^ ((lane >> 4) << 2)), p.N - 8 - n0);
        wo[h][j] = (uint32_t)(k * (int)p.ldw * 2 + n * 2);
      } else {
        const int n = min(h * 128 + row, p.N - 1 - n0);
        wo[h][j] = (uint32_t)(n * (int)p.ldw * 2 + ch * 16);
      }
    }
  const char* xg = reinterpret_cast<const char*>(X + (int64_t)m0 * p.ldx);
  const char* wg = reinterpret_cast<const char*>(W) + (KN ? (int64_t)n0 : (int64_t)n0 * p.ldw) * 2;
  const int64_t wstep = KN ? 128 * p.ldw : 128;     // bytes of W per k step
  char* const lds_w = smem + wave * 2048;
  // Piece h of X or W of step st.
  auto load_x = [&](int st, auto buf_t, auto h_t, int j) {
    constexpr int B = decltype(buf_t)::value, H = decltype(h_t)::value;
    dma16(xg + (int64_t)st * 128 + xo[H][j], lds_w + B * kBigStep + H * kBigHalf + j * 1024);
  };
  auto load_w = [&](int st, auto buf_t, auto h_t, int j) {
    constexpr int B = decltype(buf_t)::value, H = decltype(h_t)::value;
    dma16(wg + st * wstep + wo[H][j], lds_w + B * kBigStep + (2 + H) * kBigHalf + j * 1024);
  };

  // LDS addresses of the fragment reads (less the buffer and half offsets).
  const uint32_t s0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)smem);
  uint32_t xa[4], wa[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int ch = ((2 * ks + lg) ^ ((lr >> 1) & 7)) << 4;
    xa[ks] = s0 + (wm * 64 + lr) * 128 + ch;
    wa[ks] = s0 + 2 * kBigHalf + (wn * 32 + lr) * 128 + ch;
  }
  if constexpr (KN) {
    const int r = lane & 15;
    wa[0] = s0 + 2 * kBigHalf + (8 * lg + (r >> 2)) * 256 +
            (((wn * 32 + (lane & 16) + 4 * (r & 3)) * 2) ^ ((r >> 2) << 6));
  }

  f32x16_t acc[2][2][2];   // [X half][32-row block][W half]
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i >> 2][(i >> 1) & 1][i & 1][e] = 0.0f;
  u32x4_t xf[2][4], wf[2][4];
  const int KT = p.K / 64;

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  auto rd_x = [&](auto buf_t, auto h_t) {
    constexpr int B = decltype(buf_t)::value, H = decltype(h_t)::value;
    if constexpr (B == 0) {
      read_x_half<H * kBigHalf>(xf, xa);
    } else {   // the second buffer lies past the 16-bit offset field
      const uint32_t a[4] = {xa[0] + kBigStep, xa[1] + kBigStep, xa[2] + kBigStep, xa[3] + kBigStep};
      read_x_half<H * kBigHalf>(xf, a);
    }
  };
  auto rd_w = [&](auto buf_t, auto h_t) {
    constexpr int B = decltype(buf_t)::value, H = decltype(h_t)::value;
    const uint32_t a[4] = {wa[0] + B * kBigStep, wa[1] + B * kBigStep, wa[2] + B * kBigStep, wa[3] + B * kBigStep};
    if constexpr (KN) read_w_half_kn<H * kBigHalf>(wf[H], a[0]);
    else read_w_half_nk<H * kBigHalf>(wf[H], a);
  };
  // The MFMA section; load(j) issues the phase's two loads behind the second
  // and the fourth MFMA.
  auto mma = [&](auto xh_t, auto wh_t, auto&& load) {
    constexpr int XH = decltype(xh_t)::value, WH = decltype(wh_t)::value;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int bm = 0; bm < 2; ++bm) {
        Mma<bf16_t>::run(acc[XH][bm][WH], wf[WH][ks], xf[bm][ks]);
        if (bm == 1 && ks < 2) {
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
  // Step k of parity PAR (buffer PAR).  F: the W half of its first phase, G:
  // the other.  The last two steps issue no loads, so fewer may be outstanding
  // after their waits: `left` steps follow step k, at least two when STEADY.
  auto step = [&](int k, auto par_t, auto steady_t) {
    constexpr bool STEADY = decltype(steady_t)::value;
    using P = decltype(par_t);
    using Q = std::integral_constant<int, 1 - P::value>;
    using F = P;
    using G = Q;
    const int left = STEADY ? 2 : KT - 1 - k;
    // end of the read section of phase ph
    auto close = [&](auto ph_t) {
      constexpr int PH = decltype(ph_t)::value;
      if (left >= 2) wait_vmcnt<10>();
      else if (left == 1) wait_vmcnt<2 * (5 - PH)>();
      else wait_vmcnt<(PH == 0 ? 2 : 0)>();
      lds_barrier();
    };
    const bool more = left >= 2;
    rd_x(P{}, I0{});
    close(I0{});
    mma(I0{}, F{}, [&](int j) { if (more) load_w(k + 2, P{}, F{}, j); });
    rd_w(P{}, G{});
    close(I1{});
    mma(I0{}, G{}, [&](int j) { if (more) load_x(k + 2, P{}, I0{}, j); });
    rd_x(P{}, I1{});
    close(std::integral_constant<int, 2>{});
    mma(I1{}, G{}, [&](int j) { if (more) load_w(k + 2, P{}, G{}, j); });
    rd_w(Q{}, G{});   // the next step starts with the other half (after the last step: unused values)
    close(std::integral_constant<int, 3>{});
    mma(I1{}, F{}, [&](int j) { if (more) load_x(k + 2, P{}, I1{}, j); });
  };

  // Pieces of steps 0 and 1, in reading order.
#pragma unroll
  for (int j = 0; j < 2; ++j) load_w(0, I0{}, I0{}, j);
#pragma unroll
  for (int j = 0; j < 2; ++j) load_x(0, I0{}, I0{}, j);
#pragma unroll
  for (int j = 0; j < 2; ++j) load_w(0, I0{}, I1{}, j);
#pragma unroll
  for (int j = 0; j < 2; ++j) load_x(0, I0{}, I1{}, j);
#pragma unroll
  for (int j = 0; j < 2; ++j) load_w(1, I1{}, I1{}, j);
#pragma unroll
  for (int j = 0; j < 2; ++j) load_x(1, I1{}, I0{}, j);
#pragma unroll
  for (int j = 0; j < 2; ++j) load_w(1, I1{}, I0{}, j);
#pragma unroll
  for (int j = 0; j < 2; ++j) load_x(1, I1{}, I1{}, j);
  wait_vmcnt<14>();
  lds_barrier();
  rd_w(I0{}, I0{});
  wait_vmcnt<12>();
  lds_barrier();
  if (wave >= 4) lds_barrier();   // one section behind
  int k = 0;
  for (; k + 3 < KT; k += 2) {
    step(k, I0{}, std::true_type{});
    step(k + 1, I1{}, std::true_type{});
  }
#pragma unroll 1
  for (;; k += 2) {
    step(k, I0{}, std::false_type{});
    if (k + 1 >= KT) break;
    step(k + 1, I1{}, std::false_type{});
    if (k + 2 >= KT) break;
  }
  if (wave < 4) lds_barrier();
  __syncthreads();

  // C = alpha acc + bias; only a given bias is added (x + 0 would turn -0 into +0).
  const RowEpi& e = p.epi;
  if (e.alpha != 1.0f) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i >> 2][(i >> 1) & 1][i & 1][v] *= e.alpha;
  }
  if (e.bias) {
#pragma unroll
    for (int nh = 0; nh < 2; ++nh)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int n = min(n0 + nh * 128 + wn * 32 + 8 * g + 4 * lg, p.N - 4);   // columns past N are not stored
        const f32x4_t b = *reinterpret_cast<const f32x4_t*>(e.bias + n);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[i >> 1][i & 1][nh][4 * g + q] += b[q];
      }
  }
  const int esz = e.y_f32 ? 4 : 2;
  char* Y = reinterpret_cast<char*>(e.Y) + ((int64_t)bz * e.sy + (int64_t)m0 * e.ldy + n0) * esz;
#pragma unroll
  for (int mh = 0; mh < 2; ++mh) {
    char* Yh = Y + (int64_t)mh * 128 * e.ldy * esz;
    const int rows = p.M - m0 - mh * 128, cols = p.N - n0;
    if (e.y_f32) store_half<4>(acc[mh], Yh, e.ldy, rows, cols, smem, tid, lane, wm, wn);
    else store_half<2>(acc[mh], Yh, e.ldy, rows, cols, smem, tid, lane, wm, wn);
  }
}

static const GemmKernel kTable[] = {
    {kBigT, kBigT, 0, 1, 0, 512, 3, 0, reinterpret_cast<const void*>(&gemm_big_kernel<false>),
     reinterpret_cast<const void*>(&gemm_big_kernel<false>)},
    {kBigT, kBigT, 0, 2, 0, 512, 3, 0, reinterpret_cast<const void*>(&gemm_big_kernel<true>),
     reinterpret_cast<const void*>(&gemm_big_kernel<true>)},
};

const GemmKernel* gemm_kernels_big(int* n) {
  *n = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace cf
