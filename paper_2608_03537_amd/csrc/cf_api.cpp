// C ABI of libcomfuse: argument validation, path planning, workspace sizing
// and kernel dispatch.  Every check runs before the first launch, so an
// invalid call enqueues nothing; no exception leaves this file.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <utility>

#include "comfuse.h"
#include "cf_internal.h"

using namespace cf;

// Split-MLP arrival counters: a fixed region at the start of the workspace,
// one word per (batch entry, row block); the partials start after it.
static constexpr size_t kMlpCounterBytes = size_t(1) << 20;
static constexpr int64_t kMlpMaxRowBlocks = int64_t(kMlpCounterBytes / 4);

static_assert(kWsHeaderBytes == CF_WS_HEADER_BYTES, "row-cluster workspace header size in the header file");
static_assert(kMlpCounterBytes == CF_B2B_WS_HEADER_BYTES, "split-MLP counter region size in the header file");

namespace {

thread_local std::string g_last_error;

cf_status fail(cf_status s, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
cf_status fail(cf_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return s;
}

size_t dsize(cf_dtype t) { return t == CF_F32 ? 4 : t == CF_BF16 ? 2 : 1; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

constexpr int64_t kMaxRowPitch = int64_t(1) << 23;   // bytes per row; 256 rows stay below 2^31

cf_status check_matrix(const char* name, const void* p, int64_t rows, int64_t cols, int64_t ld,
                       cf_dtype t, bool required) {
  if (!p) {
    // An empty matrix (rows == 0) may come with a NULL pointer.
    if (required && rows > 0) return fail(CF_ERR_NULL, "%s is NULL", name);
    return CF_OK;
  }
  if (rows > 0 && ld < cols) return fail(CF_ERR_LD, "%s: leading dimension %lld < %lld", name, (long long)ld,
                                         (long long)cols);
  if (!aligned16(p)) return fail(CF_ERR_ALIGN, "%s is not 16-byte aligned", name);
  if ((ld * (int64_t)dsize(t)) % 16 != 0)
    return fail(CF_ERR_ALIGN, "%s: leading dimension %lld is not a multiple of 16 bytes", name, (long long)ld);
  // Kernels address a tile's rows with 32-bit byte offsets.
  if (ld * (int64_t)dsize(t) >= kMaxRowPitch)
    return fail(CF_ERR_LD, "%s: leading dimension %lld is %lld bytes or more", name, (long long)ld,
                (long long)kMaxRowPitch);
  return CF_OK;
}

cf_status check_vec(const char* name, const float* p) {
  if (p && !aligned16(p)) return fail(CF_ERR_ALIGN, "%s is not 16-byte aligned", name);
  return CF_OK;
}

cf_status hip_status(hipError_t e, const char* what) {
  if (e == hipSuccess) return CF_OK;
  return fail(CF_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

// ---------------------------------------------------------------------------
// Planning of the GEMM + row-subgraph launch.
// ---------------------------------------------------------------------------
enum Path { PATH_AUTO = 0, PATH_WHOLE_ROW = 1, PATH_CLUSTER = 2, PATH_SPLIT = 3 };

constexpr int kWholeRowMaxN = 768;
// An incomplete group of peers holds its places while it waits, and one call has at
// most one such group on an XCD.  Up to N = 1024 the automatic choice leaves room to
// complete one of kOverlap calls on as many streams (the hardware queues that HIP
// uses by default): an XCD's 32 CUs do for groups of up to kAutoClusterPeers
// workgroups with a CU each, twice as many places for groups of up to
// kClusterMaxPeers small tiles that fit a CU in pairs (pick_small).  Wider rows have
// up to 16 peers with a CU each, of which one of two calls always completes.  (Small
// tiles with one peer per CU of the XCD were faster for a single stream, 32 x 2048 x
// 2048 13.3 us against 16.7, and two such calls could starve each other.)
constexpr int kClusterMaxPeers = kClusterPeers;
constexpr int kAutoClusterPeers = 8;
constexpr int kOverlap = 4;

struct Plan {
  int kidx = -1, mode = ROWS_LOCAL, cn = 1, num_rb = 0, slots = 0, tm = 0, tn = 0;
  size_t ws = 0;
  size_t off_part = 0, off_x = 0;
  bool optional = false;   // the workspace may be left out: the plan is then whole rows
};

constexpr int kAssumedCUs = 256;   // MI355X; used only to rank tile widths

// Every non-empty workspace starts with the fixed header (error word, round
// counters and exchange records; only the cluster path writes it), which is
// all the cluster path needs.  The split path keeps part[M][cn] float2 and
// x[M][N] after it.
// The allocation-free entry point never runs the cluster path and keeps no
// header (header = false): its split buffers start at the scratch base.
void size_workspace(Plan& pl, int64_t M, int64_t N, bool header) {
  if (pl.mode == ROWS_CLUSTER) {
    pl.off_part = kWsCounterBytes;
    pl.ws = kWsHeaderBytes;
  } else if (pl.mode == ROWS_SPLIT) {
    pl.off_part = header ? kWsHeaderBytes : 0;
    // a plain product (256 x 256 and small tiles) leaves no partial statistics
    pl.off_x = pl.off_part + (gemm_kernel(pl.kidx).epi == 2 ? round_up((size_t)M * pl.cn * 8, 256) : 0);
    pl.ws = pl.off_x + round_up((size_t)M * N * 4, 256);
  } else {
    pl.ws = 0;
  }
}

// Picks the 128-row tile width: the one whose workgroups, laid out in waves
// of one workgroup per CU, give the least work per CU (rounds x width).
// `divides` restricts to widths that split N exactly into <= max_cn peers.
int pick_tile(int64_t M, int64_t N, int64_t K, int in_f32, int loop, int epi, bool divides, int max_cn) {
  int best = -1;
  double best_cost = 1e300;
  for (int tn : {256, 192, 128}) {
    const int idx = find_gemm_kernel(in_f32, 128, tn, loop, epi);
    if (idx < 0) continue;
    // the direct-to-LDS ring is filled with stages-1 stages before the first MFMA
    if (loop >= 1 && K / (in_f32 ? 32 : 64) < gemm_kernel(idx).stages - 1) continue;
    const int64_t cn = (N + tn - 1) / tn;
    if (divides && (N % tn != 0 || cn > max_cn)) continue;
    const int64_t wgs = ((M + 127) / 128) * cn;
    const double cost = (double)((wgs + kAssumedCUs - 1) / kAssumedCUs) * tn - 1e-3 * tn;
    if (cost < best_cost) { best_cost = cost; best = idx; }
  }
  return best;
}

// The 256 x 256 tile where it beats `idx` (a 128-row tile).  Both are priced in
// rounds of one workgroup per CU; a round costs its k steps plus its start and
// store.  Measured with every CU busy (us): 128 x 256 tiles 0.9 a 64-deep step
// and 4 a round, 128 x 192 0.77, 128 x 128 0.55; 256 x 256 tiles 1.4 and 12.
// Products on either side of the line: 4096 x 4096 x 1024 34 us against 39,
// 16384 x 768 x 3072 72 against 80, 8192 x 2048 x 2048 57 against 67; but 8192 x
// 1024 x 1024 27 against 21 and 2048 x 4096 x 4096 77 against 63 (half the CUs idle).
int pick_big(int idx, int64_t M, int64_t N, int64_t K, int in_f32, int loop, int64_t batch) {
  if (in_f32 || loop < 1) return idx;
  const int big = find_gemm_kernel(0, 256, 256, loop, 0);
  if (big < 0 || K / 64 < gemm_kernel(big).stages - 1) return idx;
  auto rounds = [&](int64_t tm, int64_t tn) {
    const int64_t wgs = (M + tm - 1) / tm * ((N + tn - 1) / tn) * batch;
    return (double)((wgs + kAssumedCUs - 1) / kAssumedCUs);
  };
  const double kt = (double)(K / 64);
  const int tn = gemm_kernel(idx).tn;
  const double step = tn == 256 ? 0.9 : tn == 192 ? 0.77 : 0.55;
  return rounds(256, 256) * (1.4 * kt + 12.0) < rounds(128, tn) * (step * kt + 4.0) ? big : idx;
}

// Estimated time (us) of `wgs` workgroups of a kernel in `rounds` rounds, up to
// what all kernels have in common; used to choose between 128-row tiles, 64 x
// 128 row clusters and small tiles.  A round costs its 64-deep k steps (the
// small tiles' grow with the number of CUs that stream at once) and its start
// and epilogue; a row cluster's first round starts under the launch.  Fitted to
// post-norms and plain products of 1 to 4096 rows, N 512 to 4096, K 512 to 4096.
double plan_cost(const GemmKernel& t, int64_t rounds, int64_t wgs, int64_t K, bool cluster) {
  const double kt = (double)((K + 63) / 64), busy = std::min(1.0, (double)wgs / kAssumedCUs);
  double step, start;
  if (t.epi == 3) {   // small tiles: operand stream, or fp32 MFMAs (0.42 TFLOP/s a CU)
    step = t.tm == 64 ? 0.13 + 0.07 * busy : t.tn == 64 ? 0.115 + 0.065 * busy : 0.10 + 0.09 * busy;
    if (t.pair) step += 0.03;   // 1 and 333 x 768 x 3072 13.1 and 14.7 us, with the deep ring 11.1 and 13.7
    if (t.in_f32) step = std::max(2.0 * step, 2.0 * t.tm * t.tn * 64 / 0.42e6);
    start = cluster ? (t.tm == 64 ? 8.0 : 6.0) : t.in_f32 ? 5.0 : t.tm == 64 ? 4.0 : 3.0;
  } else if (t.tm == 64) {
    step = 0.31;
    start = 6.0;
  } else {            // the register-staged loop takes longer than the ring
    step = (t.in_f32 ? 4.4 : 0.4) * t.tn / 128 * (t.loop != 0 ? 1.0 : t.in_f32 ? 1.2 : 2.0);
    start = cluster ? 8.0 : 6.0;
  }
  const double c = (double)rounds * (step * kt + start);
  if (cluster) return c - 4.0;
  // several rounds of small tiles were measured up to 15 % over the estimate
  return t.epi == 3 && rounds > 1 ? 1.15 * c : c;
}
// Rounds of row blocks of cn peers: the groups resident on the 8 XCDs of 32 CUs.
int64_t cluster_rounds(int64_t rb, int64_t cn) {
  const int64_t groups = 8 * std::max<int64_t>(1, std::min<int64_t>(kMaxSlots / 8, kAssumedCUs / 8 / cn));
  return (rb + groups - 1) / groups;
}
// The same for whole rows (32 x TN tiles, one workgroup each): the tile's
// operand stream (75 GB/s a CU) or its fp32 MFMAs.  Measured against 32 x 32 row
// clusters: 128 x 256 x 256 7.3 / 6.6 us, fp32 15.2 / 7.9; 512 rows 7.7 / 7.1, fp32 15.6 / 8.4.
double cost_whole(const GemmKernel& t, int64_t M, int64_t K) {
  const int64_t wgs = (M + 31) / 32;
  double step = (32.0 + t.tn) * (t.in_f32 ? 256 : 128) / 75e3;
  if (t.in_f32) step = std::max(step, 2.0 * 32 * t.tn * 64 / 0.6e6);
  if (t.loop == 0) step *= t.in_f32 ? 2.5 : 3.5;   // the register-staged loop: 512 x 320 x 784 35 us, fp32 97
  return (double)((wgs + kAssumedCUs - 1) / kAssumedCUs) * (step * (double)((K + 63) / 64) + (t.in_f32 ? 3.0 : 0.8));
}
double cost_128(int idx, int64_t M, int64_t N, int64_t K, int64_t batch, bool cluster) {
  const GemmKernel& t = gemm_kernel(idx);
  const int64_t rb = (M + t.tm - 1) / t.tm, cn = (N + t.tn - 1) / t.tn, wgs = rb * cn * batch;
  const int64_t rounds = cluster ? cluster_rounds(rb, cn) : (wgs + kAssumedCUs - 1) / kAssumedCUs;
  return plan_cost(t, rounds, wgs, K, cluster);
}

// The kernel of least cost among the small tiles (32 x 32, 32 x 64, 64 x 64) and,
// for row clusters on the direct-to-LDS ring (loop 1, 2), the 64 x 128 tile, if
// that is below `limit`; else -1.  cluster: column tiles must divide N into at
// most kClusterMaxPeers peers, whose row blocks run in rounds of the groups
// resident on an XCD (32 CUs); small tiles of more than kAutoClusterPeers peers take
// the shorter ring.  Measured post-norms (us; 32 x 64 / 64 x 64 / 64 x
// 128 / 128 x 128): 333 x 768 x 3072 14.1 / 17.8 / - / 26.9; 1024 x 1024 x 1024
// 17.4 / 13.6 / 12.1 / 15.8; 2048 x 1024 x 1024 30 / 22.9 / 13.2 / 16.2; 1536 x
// 768 x 3072 36 / 32.7 / 21.1 / 27.0; two rounds of 64 x 128 lose (3072 x 1024 x
// 1024 23.0 / 17.2); fp32 128 x 768 x 768 15.2 / 21.9 / - / 57.7.  Plain products
// with their row pass: 16 x 4096 x 4096 17.9 / 20.9 against 35.6, 256 rows 30.1 /
// 23.1 against 41.4, 1024 rows 106 / 69 against 49.
int pick_small(int64_t M, int64_t N, int64_t K, int in_f32, bool w_nk, int loop, int64_t batch, bool cluster,
               double limit) {
  int best = -1;
  struct { int tm, tn, loop, epi; } const tiles[] = {
      {32, 32, w_nk ? 1 : 2, 3}, {32, 64, w_nk ? 1 : 2, 3}, {64, 64, w_nk ? 1 : 2, 3}, {64, 128, loop, 1}};
  for (const auto& t : tiles) {
    if (t.epi == 1 && (!cluster || loop < 1)) continue;
    const int64_t rb = (M + t.tm - 1) / t.tm, cn = (N + t.tn - 1) / t.tn;
    const int idx = find_gemm_kernel(in_f32, t.tm, t.tn, t.loop, t.epi,
                                     t.epi == 3 && cluster && cn > kAutoClusterPeers);
    if (idx < 0 || (t.epi == 1 && K / 64 < gemm_kernel(idx).stages - 1)) continue;
    const int64_t wgs = rb * cn * batch;
    int64_t rounds = (wgs + kAssumedCUs - 1) / kAssumedCUs;
    if (cluster) {
      if (N % t.tn != 0 || cn > kClusterMaxPeers) continue;
      rounds = cluster_rounds(rb, cn);
    }
    const double c = plan_cost(gemm_kernel(idx), rounds, wgs, K, cluster);
    if (c < limit) { limit = c; best = idx; }
  }
  return best;
}

// Chooses kernel and row path for a GEMM (+ row subgraph).  `epi` selects the
// epilogue: 0 = plain (alpha, bias, store), 1 = row subgraph.  `need_rows` is
// true when the subgraph has a row reduction (then rows must be completed
// across tiles); without one any tiling is valid.  few_rows = false leaves out
// the tiles for few rows and the row clusters of an optional workspace.
cf_status plan_rows(int64_t M, int64_t N, int64_t K, int in_f32, bool w_nk, int path, int epi, bool need_rows,
                    Plan& pl, bool allow_cluster = true, int64_t batch = 1, bool few_rows = true) {
  pl = Plan();
  if (!allow_cluster && need_rows) {
    if (path == PATH_CLUSTER)
      return fail(CF_ERR_UNSUPPORTED, "the allocation-free entry point has no row-cluster path");
    if (path == PATH_AUTO) path = N <= kWholeRowMaxN ? PATH_WHOLE_ROW : PATH_SPLIT;
  }
  const int tk = in_f32 ? 32 : 64;                     // k per 128-byte stage
  // Direct-to-LDS ring when K fills whole stages: W stored N x K (loop 1), or
  // bf16 W stored K x N with N a multiple of 8 (loop 2, transposing reads).
  const int loop = K % tk != 0 ? 0 : w_nk ? 1 : (!in_f32 && N % 8 == 0) ? 2 : 0;
  // 128-row tile of the direct-to-LDS ring, or of the register-staged loop
  auto tile_128 = [&](int ep, bool divides, int max_cn) {
    const int idx = pick_tile(M, N, K, in_f32, loop, ep, divides, max_cn);
    return idx >= 0 ? idx : pick_tile(M, N, K, in_f32, 0, ep, divides, max_cn);
  };
  if (!need_rows) {
    pl.kidx = tile_128(epi, false, 0);
    pl.mode = ROWS_LOCAL;
    if (pl.kidx >= 0) {
      const int small = pick_small(M, N, K, in_f32, w_nk, loop, batch, false,
                                   cost_128(pl.kidx, M, N, K, batch, false));
      if (small >= 0) pl.kidx = small;
      else if (epi == 0) pl.kidx = pick_big(pl.kidx, M, N, K, in_f32, loop, batch);
    }
  } else {
    const bool automatic = path == PATH_AUTO;
    if (automatic) {
      // Row clusters when N splits into <= kAutoClusterPeers tiles; whole rows
      // instead when N is narrow and they give more workgroups (small M);
      // else split-N.  Every tile's exchange waits for the slowest of its
      // peers, and with 16 peers that wait costs more than split-N's fp32
      // round trip of x, so wide rows go to split-N unless a caller asks
      // for the cluster path.
      path = PATH_SPLIT;
      const int ck = tile_128(1, true, kAutoClusterPeers);
      if (ck >= 0) {
        path = PATH_CLUSTER;
        const GemmKernel& t = gemm_kernel(ck);
        const int64_t cluster_wgs = ((M + t.tm - 1) / t.tm) * ((N + t.tn - 1) / t.tn);
        if (N <= kWholeRowMaxN && (M + 31) / 32 > cluster_wgs) path = PATH_WHOLE_ROW;
      } else if (N <= kWholeRowMaxN) {
        path = PATH_WHOLE_ROW;
      }
    }
    if (path == PATH_WHOLE_ROW) {
      if (N > kWholeRowMaxN)
        return fail(CF_ERR_UNSUPPORTED, "whole-row path needs N <= %d (N = %lld)", kWholeRowMaxN, (long long)N);
      for (int tn : {128, 256, 384, 512, 768})
        if (tn >= N) {
          // the direct-to-LDS ring where compiled and K fills its prologue
          const int v2 = loop >= 1 ? find_gemm_kernel(in_f32, 32, tn, loop, 1) : -1;
          if (v2 >= 0 && K / tk >= gemm_kernel(v2).stages - 1) pl.kidx = v2;
          else pl.kidx = find_gemm_kernel(in_f32, 32, tn, 0, 1);
          break;
        }
      pl.mode = ROWS_LOCAL;
    } else if (path == PATH_CLUSTER) {
      pl.kidx = tile_128(1, true, kClusterMaxPeers);
      if (pl.kidx < 0)
        return fail(CF_ERR_UNSUPPORTED, "cluster path: no tile width divides N = %lld into <= %d peers",
                    (long long)N, kClusterMaxPeers);
      pl.mode = ROWS_CLUSTER;
    } else if (path == PATH_SPLIT) {
      pl.kidx = tile_128(2, false, 0);
      pl.mode = ROWS_SPLIT;
    } else {
      return fail(CF_ERR_UNSUPPORTED, "unknown path %d", path);
    }
    // Whole rows of the register-staged loop up to 384 wide keep several workgroups
    // on a CU, so beyond one generation they stay: 14764 x 256 x 992 40 us, row clusters
    // 55; 14764 x 384 x 496 33 / 38; 20000 x 128 x 1488 43 / 55 (6000 x 256 x 992 37 / 28).
    const bool several = pl.kidx >= 0 && gemm_kernel(pl.kidx).loop == 0 && gemm_kernel(pl.kidx).tn <= 384 &&
                         M > 32 * kAssumedCUs;
    // Fewer rows than fill the chip with 128-row tiles: 64 x 128 or small tiles,
    // as a row cluster or (row pass and second launch: about 4 us) small ones as
    // the plain product of the split path.  Not under an explicit path.  Where the
    // choice so far takes no workspace, the cluster's is optional.
    if (!automatic || !few_rows) {
    } else if (pl.kidx >= 0 && pl.mode == ROWS_LOCAL && !several) {
      // Whole rows of 32 x TN on few CUs, or wide ones in many rounds: row
      // clusters if the caller gives a workspace and they are clearly faster.
      const double now = 0.85 * cost_whole(gemm_kernel(pl.kidx), M, K);
      const int ck = tile_128(1, true, kAutoClusterPeers);
      const double c128 = ck >= 0 ? cost_128(ck, M, N, K, 1, true) : now;
      int sc = pick_small(M, N, K, in_f32, w_nk, loop, 1, true, std::min(now, c128));
      if (sc < 0 && c128 < now) sc = ck;
      if (sc >= 0) {
        pl.kidx = sc;
        pl.mode = ROWS_CLUSTER;
        pl.optional = true;
      }
    } else if (pl.kidx >= 0 && pl.mode != ROWS_LOCAL) {
      const double now = cost_128(pl.kidx, M, N, K, 1, pl.mode == ROWS_CLUSTER);
      const int sc = !allow_cluster ? -1 : pick_small(M, N, K, in_f32, w_nk, loop, 1, true,
                                                      pl.mode == ROWS_SPLIT ? now + 4.0 : now);
      const int sp = sc < 0 && pl.mode == ROWS_SPLIT ? pick_small(M, N, K, in_f32, w_nk, loop, 1, false, now) : -1;
      if (sc >= 0) {
        pl.kidx = sc;
        pl.mode = ROWS_CLUSTER;
      } else if (sp >= 0) {
        pl.kidx = sp;
      }
    }
    if (pl.kidx >= 0 && pl.mode == ROWS_SPLIT && gemm_kernel(pl.kidx).epi == 2)
      pl.kidx = pick_big(pl.kidx, M, N, K, in_f32, loop, 1);
  }
  if (pl.kidx < 0) return fail(CF_ERR_UNSUPPORTED, "no compiled tile for this shape");
  const GemmKernel& t = gemm_kernel(pl.kidx);
  pl.tm = t.tm;
  pl.tn = t.tn;
  pl.cn = (int)((N + t.tn - 1) / t.tn);
  pl.num_rb = (int)((M + t.tm - 1) / t.tm);
  pl.slots = (pl.num_rb + 7) / 8;
  // the finish pass reads a row's partials one per lane of a 64-lane wave
  if (pl.mode == ROWS_SPLIT && t.epi == 2 && pl.cn > 64)
    return fail(CF_ERR_UNSUPPORTED, "split path: %d tiles per row exceed 64", pl.cn);
  if (pl.mode == ROWS_CLUSTER && (pl.tm > kRecRows || pl.cn > kClusterPeers))
    return fail(CF_ERR_UNSUPPORTED, "cluster path: tile of %d rows x %d peers exceeds the exchange records",
                pl.tm, pl.cn);
  size_workspace(pl, M, N, allow_cluster);
  return CF_OK;
}

// Row clusters: every peer group must be resident at once, so the persistent
// grid is capped (queries the device, hence only right before a launch).
// Groups of small tiles also leave the places of kOverlap - 1 other incomplete groups.
cf_status cap_slots(Plan& pl) {
  if (pl.mode != ROWS_CLUSTER) return CF_OK;
  const int places = resident_wgs(pl.kidx) / 8, slots = places / pl.cn;
  if (slots < 1 || (gemm_kernel(pl.kidx).pair && places <= kOverlap * (pl.cn - 1)))
    return fail(CF_ERR_UNSUPPORTED, "cluster path: %d peers do not fit the device", pl.cn);
  pl.slots = std::min(pl.slots, std::min(slots, kMaxSlots / 8));
  return CF_OK;
}

void bind_workspace(const Plan& pl, void* ws, GemmRowsParams& p) {
  char* b = reinterpret_cast<char*>(ws);
  if (pl.mode == ROWS_CLUSTER) {
    p.ws_err = reinterpret_cast<unsigned*>(b);
    p.ws_arrive = reinterpret_cast<unsigned long long*>(b + 256);
    static_assert(kWsCounterBytes % 256 == 0, "records alignment");
    p.ws_part = reinterpret_cast<float*>(b + pl.off_part);
    p.spin_limit = kSpinLimitDefault;
    p.leader = pl.cn >= kLeaderFollowerPeers;
  } else if (pl.mode == ROWS_SPLIT) {
    p.ws_part = reinterpret_cast<float*>(b + pl.off_part);
    p.ws_x = reinterpret_cast<float*>(b + pl.off_x);
  }
}

// Runs a planned GEMM + row subgraph (and the finish pass of the split path).
cf_status run_rows(const Plan& pl, GemmRowsParams p, void* ws, hipStream_t st) {
  p.mode = pl.mode;
  p.cn = pl.cn;
  p.num_rb = pl.num_rb;
  p.slots = pl.slots;
  bind_workspace(pl, ws, p);
  if (pl.mode == ROWS_SPLIT) {
    RowEpi full = p.epi;
    RowKernelParams f{};
    f.M = p.M;
    f.N = p.N;
    f.P = p.ws_x;
    f.ldp = p.N;
    f.p_f32 = 1;
    f.epi = full;
    if (gemm_kernel(pl.kidx).epi != 2) {
      // The plain product in fp32; the row pass runs every stage (it reads the
      // residual and takes the statistics of the rows it holds).
      f.rows_per_batch = p.M;
      p.epi = RowEpi{};
      p.epi.alpha = 1.0f;
      p.epi.Y = p.ws_x;
      p.epi.ldy = p.N;
      p.epi.y_f32 = 1;
      cf_status s = hip_status(launch_gemm_rows(p, pl.kidx, st), "GEMM launch");
      return s != CF_OK ? s : hip_status(launch_row_kernel(f, st), "row pass launch");
    }
    // The GEMM runs stage 1 only and publishes x and partial statistics (the
    // norm stays: it chooses how stage 1 adds a staged residual).
    p.epi.act = ACT_NONE;
    p.epi.softmax = 0;
    p.epi.Y = nullptr;
    p.epi.quant = 0;
    cf_status s = hip_status(launch_gemm_rows(p, pl.kidx, st), "GEMM launch");
    if (s != CF_OK) return s;
    f.finish = 1;
    f.cn = pl.cn;
    f.tn = pl.tn;
    f.part = p.ws_part;
    f.epi.alpha = 1.0f;
    f.epi.bias = nullptr;
    f.epi.R = nullptr;
    return hip_status(launch_row_kernel(f, st), "finish launch");
  }
  return hip_status(launch_gemm_rows(p, pl.kidx, st), "GEMM launch");
}

// ---------------------------------------------------------------------------
// Node lists -> RowEpi (the fixed stage grammar).
// ---------------------------------------------------------------------------
cf_status parse_nodes(const cf_node* nodes, int n, int64_t M, int64_t N, cf_dtype in, RowEpi& e,
                      bool allow_softmax, int* softmax, float* softmax_scale) {
  e = RowEpi{};
  e.alpha = 1.0f;
  e.qmax = 448.0f;
  if (softmax) *softmax = 0;
  if (!nodes || n <= 0) return fail(CF_ERR_NULL, "empty node list");
  if (n == 1 && nodes[0].kind == CF_N_SOFTMAX) {
    if (!allow_softmax) return fail(CF_ERR_UNSUPPORTED, "SOFTMAX is available in cf_rowop only");
    const cf_node& d = nodes[0];
    if (d.dtype != CF_F32 && d.dtype != CF_BF16) return fail(CF_ERR_DTYPE, "SOFTMAX output dtype");
    cf_status s = check_matrix("SOFTMAX out", d.out, M, N, d.ld, d.dtype, true);
    if (s != CF_OK) return s;
    e.Y = d.out;
    e.ldy = d.ld;
    e.y_f32 = d.dtype == CF_F32;
    *softmax = 1;
    *softmax_scale = d.f0;
    return CF_OK;
  }
  // Grammar position of each kind; positions must strictly increase.
  auto rank = [](cf_node_kind k) -> int {
    switch (k) {
      case CF_N_SCALE: return 0;
      case CF_N_BIAS: return 1;
      case CF_N_RESIDUAL: return 2;
      case CF_N_LAYERNORM: case CF_N_RMSNORM: return 3;
      case CF_N_GELU: case CF_N_GELU_TANH: case CF_N_RELU: case CF_N_SOFTCAP: return 4;
      case CF_N_SOFTMAX: return 5;
      case CF_N_STORE: return 6;
      case CF_N_ROWAMAX_QUANT: return 7;
      default: return -1;
    }
  };
  int last = -1;
  for (int i = 0; i < n; ++i) {
    const cf_node& d = nodes[i];
    const int r = rank(d.kind);
    if (r < 0) return fail(CF_ERR_UNSUPPORTED, "node %d: kind %d is not in the fused vocabulary", i, (int)d.kind);
    if (r <= last)
      return fail(CF_ERR_UNSUPPORTED,
                  "node %d: kind %d out of order (grammar: SCALE BIAS RESIDUAL NORM ACT SOFTMAX STORE QUANT)", i,
                  (int)d.kind);
    last = r;
    cf_status s = CF_OK;
    switch (d.kind) {
      case CF_N_SCALE: e.alpha = d.f0; break;
      case CF_N_BIAS:
        if (!d.v0) return fail(CF_ERR_NULL, "BIAS vector is NULL");
        if ((s = check_vec("BIAS", d.v0)) != CF_OK) return s;
        e.bias = d.v0;
        break;
      case CF_N_RESIDUAL:
        if (d.dtype != CF_F32 && d.dtype != CF_BF16) return fail(CF_ERR_DTYPE, "RESIDUAL dtype must be F32 or BF16");
        if (!allow_softmax && d.dtype != in)
          return fail(CF_ERR_DTYPE, "RESIDUAL dtype must equal the GEMM input dtype");
        if ((s = check_matrix("RESIDUAL", d.in, M, N, d.ld, d.dtype, true)) != CF_OK) return s;
        e.R = d.in;
        e.ldr = d.ld;
        e.r_f32 = d.dtype == CF_F32;
        break;
      case CF_N_LAYERNORM: case CF_N_RMSNORM:
        if ((s = check_vec("gamma", d.v0)) != CF_OK || (s = check_vec("beta", d.v1)) != CF_OK) return s;
        if (!(d.f0 >= 0.0f)) return fail(CF_ERR_SHAPE, "eps must be >= 0");
        e.norm = d.kind == CF_N_LAYERNORM ? NORM_LAYER : NORM_RMS;
        e.gamma = d.v0;
        e.beta = d.kind == CF_N_LAYERNORM ? d.v1 : nullptr;
        e.eps = d.f0;
        break;
      case CF_N_GELU: e.act = ACT_GELU; break;
      case CF_N_GELU_TANH: e.act = ACT_GELU_TANH; break;
      case CF_N_RELU: e.act = ACT_RELU; break;
      case CF_N_SOFTCAP:
        if (!(d.f0 > 0.0f) || !std::isfinite(d.f0)) return fail(CF_ERR_SHAPE, "SOFTCAP cap must be finite and > 0");
        e.act = ACT_SOFTCAP;
        e.softcap = d.f0;
        break;
      case CF_N_SOFTMAX:
        if (e.norm != NORM_NONE) return fail(CF_ERR_UNSUPPORTED, "SOFTMAX after a NORM is not in the fused vocabulary");
        e.softmax = 1;
        break;
      case CF_N_STORE:
        if (d.dtype != CF_F32 && d.dtype != CF_BF16) return fail(CF_ERR_DTYPE, "STORE dtype must be F32 or BF16");
        if ((s = check_matrix("STORE", d.out, M, N, d.ld, d.dtype, true)) != CF_OK) return s;
        e.Y = d.out;
        e.ldy = d.ld;
        e.y_f32 = d.dtype == CF_F32;
        break;
      case CF_N_ROWAMAX_QUANT:
        if (!d.out) return fail(CF_ERR_NULL, "ROWAMAX_QUANT scale output is NULL");
        if (!(d.f0 > 0.0f)) return fail(CF_ERR_SHAPE, "ROWAMAX_QUANT qmax must be > 0");
        if (d.out2) {
          if (!aligned16(d.out2) || d.ld % 16 != 0)
            return fail(CF_ERR_ALIGN, "ROWAMAX_QUANT codes: 16-byte alignment and ld %% 16 == 0 required");
          if (M > 0 && d.ld < N) return fail(CF_ERR_LD, "ROWAMAX_QUANT codes: ld < N");
        }
        e.quant = 1;
        e.qmax = d.f0;
        e.s_out = reinterpret_cast<float*>(d.out);
        e.q_out = reinterpret_cast<uint8_t*>(d.out2);
        e.ldq = d.ld;
        break;
      default: break;
    }
  }
  if (!e.Y && !e.quant) return fail(CF_ERR_UNSUPPORTED, "node list has no output (STORE or ROWAMAX_QUANT)");
  return CF_OK;
}

cf_status check_gemm_shape(int64_t M, int64_t N, int64_t K) {
  if (M < 0 || N <= 0 || K <= 0) return fail(CF_ERR_SHAPE, "need M >= 0, N > 0, K > 0");
  if (N % 32 != 0) return fail(CF_ERR_SHAPE, "N = %lld must be a multiple of 32", (long long)N);
  if (K % 16 != 0) return fail(CF_ERR_SHAPE, "K = %lld must be a multiple of 16", (long long)K);
  if (N > 8192) return fail(CF_ERR_SHAPE, "N = %lld exceeds 8192", (long long)N);
  if (M > (int64_t)1 << 30 || K > (int64_t)1 << 30) return fail(CF_ERR_SHAPE, "size exceeds 2^30");
  return CF_OK;
}

bool outputs_alias(const void* out, std::initializer_list<const void*> ins) {
  if (!out) return false;
  for (const void* p : ins)
    if (p && p == out) return true;
  return false;
}

// Shared body of cf_gemm_postnorm / cf_gemm_subgraph.
// scratch = true: ws is the library's own allocation-free scratch (no
// header, no cluster path; a plan needing more than ws_bytes is refused).
cf_status rows_common(int64_t M, int64_t N, int64_t K, cf_dtype in, const void* X, int64_t ldx,
                      const void* W, int64_t ldw, cf_layout wl, const RowEpi& epi, int path,
                      void* ws, size_t ws_bytes, void* stream, bool size_only, size_t* ws_out,
                      bool scratch = false) {
  cf_status s = check_gemm_shape(M, N, K);
  if (s != CF_OK) return s;
  if (in != CF_F32 && in != CF_BF16) return fail(CF_ERR_DTYPE, "input dtype must be F32 or BF16");
  if (wl != CF_LAYOUT_KN && wl != CF_LAYOUT_NK) return fail(CF_ERR_UNSUPPORTED, "unknown weight layout");
  if ((s = check_matrix("X", X, M, K, ldx, in, true)) != CF_OK) return s;
  if ((s = check_matrix("W", W, 1, wl == CF_LAYOUT_NK ? K : N, ldw, in, true)) != CF_OK) return s;
  const bool need_rows = epi.norm != NORM_NONE || epi.quant || epi.softmax;
  // The plain epilogue only applies alpha and bias; anything else runs the
  // row-subgraph epilogue.
  const int epi_kind = (need_rows || epi.R || epi.act != ACT_NONE) ? 1 : 0;
  Plan pl;
  // Validation and sizing never touch the device; residency is queried only
  // right before a launch.
  if ((s = plan_rows(M, N, K, in == CF_F32, wl == CF_LAYOUT_NK, path, epi_kind, need_rows, pl, !scratch)) != CF_OK)
    return s;
  if (size_only) {
    *ws_out = pl.ws + (pl.optional ? CF_WS_OPTIONAL_BYTES - CF_WS_HEADER_BYTES : 0);
    return CF_OK;
  }
  const bool use_optional = ws && ws_bytes >= pl.ws && aligned16(ws);
  if (pl.optional && !use_optional &&
      (s = plan_rows(M, N, K, in == CF_F32, wl == CF_LAYOUT_NK, path, epi_kind, need_rows, pl, !scratch, 1,
                     false)) != CF_OK)
    return s;
  for (const void* out : {(const void*)epi.Y, (const void*)epi.s_out, (const void*)epi.q_out})
    if (outputs_alias(out, {X, W, epi.R, (const void*)epi.bias, (const void*)epi.gamma, (const void*)epi.beta}))
      return fail(CF_ERR_ALIAS, "an output aliases an input");
  if (M == 0) return CF_OK;   // nothing to compute: no workspace needed
  if (scratch && pl.ws > ws_bytes)
    return fail(CF_ERR_WORKSPACE, "this shape needs %zu bytes of scratch; the allocation-free entry point holds %zu",
                pl.ws, ws_bytes);
  if (pl.ws > 0) {
    if (!ws) return fail(CF_ERR_WORKSPACE, "workspace of %zu bytes required", pl.ws);
    if (ws_bytes < pl.ws) return fail(CF_ERR_WORKSPACE, "workspace %zu < %zu bytes", ws_bytes, pl.ws);
    if (!aligned16(ws)) return fail(CF_ERR_ALIGN, "workspace is not 16-byte aligned");
  }
  if ((s = cap_slots(pl)) != CF_OK) {
    // Too few co-resident workgroups for the peers of an automatic choice: the
    // plan without it, where the workspace holds that.
    Plan base;
    if (path != PATH_AUTO ||
        plan_rows(M, N, K, in == CF_F32, wl == CF_LAYOUT_NK, path, epi_kind, need_rows, base, !scratch, 1, false) !=
            CF_OK ||
        base.ws > (ws ? ws_bytes : 0) || cap_slots(base) != CF_OK)
      return s;
    pl = base;
  }
  GemmRowsParams p{};
  p.batch = 1;
  p.M = (int)M;
  p.N = (int)N;
  p.K = (int)K;
  p.X = X;
  p.ldx = ldx;
  p.W = W;
  p.ldw = ldw;
  p.w_nk = wl == CF_LAYOUT_NK;
  p.epi = epi;
  return run_rows(pl, p, ws, reinterpret_cast<hipStream_t>(stream));
}

cf_status postnorm_epi(const cf_postnorm_args* a, RowEpi& e) {
  if (!a) return fail(CF_ERR_NULL, "args is NULL");
  if (a->struct_size != sizeof(cf_postnorm_args))
    return fail(CF_ERR_STRUCT, "struct_size %zu != %zu", a->struct_size, sizeof(cf_postnorm_args));
  if (a->in_dtype != CF_F32 && a->in_dtype != CF_BF16) return fail(CF_ERR_DTYPE, "in_dtype must be F32 or BF16");
  if (a->out_dtype != CF_F32 && a->out_dtype != CF_BF16) return fail(CF_ERR_DTYPE, "out_dtype must be F32 or BF16");
  if (a->in_dtype == CF_F32 && a->out_dtype != CF_F32) return fail(CF_ERR_DTYPE, "F32 input needs F32 output");
  if (!(a->eps >= 0.0f)) return fail(CF_ERR_SHAPE, "eps must be >= 0");
  cf_status s;
  if ((s = check_matrix("Y", a->Y, a->M, a->N, a->ldy, a->out_dtype, true)) != CF_OK) return s;
  if ((s = check_matrix("R", a->R, a->M, a->N, a->ldr, a->in_dtype, false)) != CF_OK) return s;
  if ((s = check_vec("bias", a->bias)) != CF_OK || (s = check_vec("gamma", a->gamma)) != CF_OK ||
      (s = check_vec("beta", a->beta)) != CF_OK)
    return s;
  e = RowEpi{};
  e.alpha = a->alpha;
  e.bias = a->bias;
  e.R = a->R;
  e.ldr = a->ldr;
  e.r_f32 = a->in_dtype == CF_F32;
  e.norm = NORM_LAYER;
  e.gamma = a->gamma;
  e.beta = a->beta;
  e.eps = a->eps;
  e.Y = a->Y;
  e.ldy = a->ldy;
  e.y_f32 = a->out_dtype == CF_F32;
  e.qmax = 448.0f;
  return CF_OK;
}

cf_status subgraph_epi(const cf_subgraph_args* a, RowEpi& e) {
  if (!a) return fail(CF_ERR_NULL, "args is NULL");
  if (a->struct_size != sizeof(cf_subgraph_args))
    return fail(CF_ERR_STRUCT, "struct_size %zu != %zu", a->struct_size, sizeof(cf_subgraph_args));
  if (a->in_dtype != CF_F32 && a->in_dtype != CF_BF16) return fail(CF_ERR_DTYPE, "in_dtype must be F32 or BF16");
  return parse_nodes(a->nodes, a->n_nodes, a->M, a->N, a->in_dtype, e, false, nullptr, nullptr);
}

}  // namespace

namespace cf {
// cf_gemm_subgraph through a given scratch buffer (the allocation-free entry
// point's device array): validation as cf_gemm_subgraph, then a plan without
// the row-cluster path whose buffers must fit in scratch_bytes.
// validate_only: check the arguments and that the plan fits scratch_bytes,
// touch nothing on the device; *empty tells whether the call is a no-op.
cf_status gemm_subgraph_scratch(const cf_subgraph_args* a, void* scratch, size_t scratch_bytes, void* hip_stream,
                                bool validate_only, bool* empty) {
  try {
    RowEpi e;
    cf_status s = subgraph_epi(a, e);
    if (s != CF_OK) return s;
    if (validate_only) {
      size_t need = 0;
      if ((s = rows_common(a->M, a->N, a->K, a->in_dtype, a->X, a->ldx, a->W, a->ldw, a->w_layout, e, a->path,
                           nullptr, 0, nullptr, true, &need, true)) != CF_OK)
        return s;
      if (need > scratch_bytes)
        return fail(CF_ERR_WORKSPACE,
                    "this shape needs %zu bytes of scratch; the allocation-free entry point holds %zu", need,
                    scratch_bytes);
      if (empty) *empty = a->M == 0;
      return CF_OK;
    }
    return rows_common(a->M, a->N, a->K, a->in_dtype, a->X, a->ldx, a->W, a->ldw, a->w_layout, e, a->path,
                       scratch, scratch_bytes, hip_stream, false, nullptr, true);
  } catch (...) {
    return fail(CF_ERR_HIP, "internal error");
  }
}

cf_status record_error(cf_status s, const char* what) { return fail(s, "%s", what); }
}  // namespace cf

extern "C" {

int cf_version(void) { return CF_VERSION; }

const char* cf_last_error(void) { return g_last_error.c_str(); }

const char* cf_status_string(cf_status s) {
  switch (s) {
    case CF_OK: return "CF_OK";
    case CF_ERR_NULL: return "CF_ERR_NULL: a required pointer is NULL";
    case CF_ERR_SHAPE: return "CF_ERR_SHAPE: invalid size";
    case CF_ERR_LD: return "CF_ERR_LD: leading dimension too small";
    case CF_ERR_ALIGN: return "CF_ERR_ALIGN: misaligned pointer or leading dimension";
    case CF_ERR_DTYPE: return "CF_ERR_DTYPE: unsupported dtype";
    case CF_ERR_WORKSPACE: return "CF_ERR_WORKSPACE: workspace missing or too small";
    case CF_ERR_UNSUPPORTED: return "CF_ERR_UNSUPPORTED: outside the compiled vocabulary";
    case CF_ERR_ALIAS: return "CF_ERR_ALIAS: an output aliases an input";
    case CF_ERR_HIP: return "CF_ERR_HIP: HIP runtime error";
    case CF_ERR_STRUCT: return "CF_ERR_STRUCT: struct_size mismatch";
    case CF_ERR_PEER_TIMEOUT: return "CF_ERR_PEER_TIMEOUT: a wait for peer workgroups gave up";
  }
  return "unknown cf_status";
}

size_t cf_gemm_postnorm_workspace(const cf_postnorm_args* a) {
  try {
    RowEpi e;
    if (postnorm_epi(a, e) != CF_OK) return 0;
    size_t ws = 0;
    if (rows_common(a->M, a->N, a->K, a->in_dtype, a->X, a->ldx, a->W, a->ldw, a->w_layout, e, a->path,
                    nullptr, 0, nullptr, true, &ws) != CF_OK)
      return 0;
    return ws;
  } catch (...) {
    return 0;
  }
}

cf_status cf_gemm_postnorm(const cf_postnorm_args* a, void* workspace, size_t ws_bytes, void* hip_stream) {
  try {
    RowEpi e;
    cf_status s = postnorm_epi(a, e);
    if (s != CF_OK) return s;
    return rows_common(a->M, a->N, a->K, a->in_dtype, a->X, a->ldx, a->W, a->ldw, a->w_layout, e, a->path,
                       workspace, ws_bytes, hip_stream, false, nullptr);
  } catch (...) {
    return fail(CF_ERR_HIP, "internal error");
  }
}

size_t cf_gemm_subgraph_workspace(const cf_subgraph_args* a) {
  try {
    RowEpi e;
    if (subgraph_epi(a, e) != CF_OK) return 0;
    size_t ws = 0;
    if (rows_common(a->M, a->N, a->K, a->in_dtype, a->X, a->ldx, a->W, a->ldw, a->w_layout, e, a->path,
                    nullptr, 0, nullptr, true, &ws) != CF_OK)
      return 0;
    return ws;
  } catch (...) {
    return 0;
  }
}

cf_status cf_gemm_subgraph(const cf_subgraph_args* a, void* workspace, size_t ws_bytes, void* hip_stream) {
  try {
    RowEpi e;
    cf_status s = subgraph_epi(a, e);
    if (s != CF_OK) return s;
    return rows_common(a->M, a->N, a->K, a->in_dtype, a->X, a->ldx, a->W, a->ldw, a->w_layout, e, a->path,
                       workspace, ws_bytes, hip_stream, false, nullptr);
  } catch (...) {
    return fail(CF_ERR_HIP, "internal error");
  }
}

cf_status cf_gemm(int64_t batch, int64_t M, int64_t N, int64_t K, cf_dtype in, cf_dtype out, const void* A,
                  int64_t lda, int64_t sa, const void* B, int64_t ldb, int64_t sb, cf_layout b_layout,
                  const float* bias, float alpha, void* C, int64_t ldc, int64_t sc, void* hip_stream) {
  try {
    cf_status s = check_gemm_shape(M, N, K);
    if (s != CF_OK) return s;
    if (batch < 0 || batch > 65535) return fail(CF_ERR_SHAPE, "batch must be in [0, 65535]");
    if (in != CF_F32 && in != CF_BF16) return fail(CF_ERR_DTYPE, "input dtype must be F32 or BF16");
    if (out != CF_F32 && out != CF_BF16) return fail(CF_ERR_DTYPE, "output dtype must be F32 or BF16");
    if (b_layout != CF_LAYOUT_KN && b_layout != CF_LAYOUT_NK) return fail(CF_ERR_UNSUPPORTED, "unknown layout");
    if ((s = check_matrix("A", A, M, K, lda, in, true)) != CF_OK) return s;
    if ((s = check_matrix("B", B, 1, b_layout == CF_LAYOUT_NK ? K : N, ldb, in, true)) != CF_OK) return s;
    if ((s = check_matrix("C", C, M, N, ldc, out, true)) != CF_OK) return s;
    if ((s = check_vec("bias", bias)) != CF_OK) return s;
    if (batch > 1 && (sa % 8 != 0 || sb % 8 != 0 || sc % 8 != 0 || sa < 0 || sb < 0 || sc < 0))
      return fail(CF_ERR_ALIGN, "batch strides must be non-negative multiples of 8 elements");
    if (outputs_alias(C, {A, B, (const void*)bias})) return fail(CF_ERR_ALIAS, "C aliases an input");
    if (M == 0 || batch == 0) return CF_OK;
    Plan pl;
    if ((s = plan_rows(M, N, K, in == CF_F32, b_layout == CF_LAYOUT_NK, PATH_AUTO, 0, false, pl, true, batch)) !=
        CF_OK)
      return s;
    GemmRowsParams p{};
    p.batch = (int)batch;
    p.M = (int)M;
    p.N = (int)N;
    p.K = (int)K;
    p.X = A;
    p.ldx = lda;
    p.sx = sa;
    p.W = B;
    p.ldw = ldb;
    p.sw = sb;
    p.w_nk = b_layout == CF_LAYOUT_NK;
    p.epi.alpha = alpha;
    p.epi.bias = bias;
    p.epi.Y = C;
    p.epi.ldy = ldc;
    p.epi.sy = sc;
    p.epi.y_f32 = out == CF_F32;
    p.epi.qmax = 448.0f;
    return run_rows(pl, p, nullptr, reinterpret_cast<hipStream_t>(hip_stream));
  } catch (...) {
    return fail(CF_ERR_HIP, "internal error");
  }
}

cf_status cf_rowop(int64_t batch, int64_t M, int64_t N, cf_dtype in, const void* P, int64_t ldp, int64_t sp,
                   const cf_node* nodes, int n_nodes, void* hip_stream) {
  try {
    if (M < 0 || N <= 0 || N % 4 != 0 || N > 8192) return fail(CF_ERR_SHAPE, "need M >= 0, 0 < N <= 8192, N %% 4 == 0");
    if (batch < 0 || batch > 65535) return fail(CF_ERR_SHAPE, "batch must be in [0, 65535]");
    if (batch * M > ((int64_t)1 << 31) - 1) return fail(CF_ERR_SHAPE, "batch * M exceeds 2^31 - 1 rows");
    if (in != CF_F32 && in != CF_BF16) return fail(CF_ERR_DTYPE, "input dtype must be F32 or BF16");
    cf_status s = check_matrix("P", P, batch > 0 ? M : 0, N, ldp, in, true);
    if (s != CF_OK) return s;
    if (batch > 1 && (sp < 0 || (sp * (int64_t)dsize(in)) % 16 != 0))
      return fail(CF_ERR_ALIGN, "batch stride of P must be a non-negative multiple of 16 bytes");
    const int64_t rows = batch * M;   // node matrices and s hold batch * M consecutive rows
    RowKernelParams r{};
    if ((s = parse_nodes(nodes, n_nodes, rows, N, in, r.epi, true, &r.softmax, &r.softmax_scale)) != CF_OK) return s;
    for (const void* out : {(const void*)r.epi.Y, (const void*)r.epi.s_out, (const void*)r.epi.q_out})
      if (outputs_alias(out, {P, r.epi.R, (const void*)r.epi.bias}))
        return fail(CF_ERR_ALIAS, "an output aliases an input");
    if (rows == 0) return CF_OK;
    r.M = (int)rows;
    r.N = (int)N;
    r.P = P;
    r.ldp = ldp;
    r.rows_per_batch = (int)M;
    r.sp = batch > 1 ? sp : 0;
    r.p_f32 = in == CF_F32;
    return hip_status(launch_row_kernel(r, reinterpret_cast<hipStream_t>(hip_stream)), "row kernel launch");
  } catch (...) {
    return fail(CF_ERR_HIP, "internal error");
  }
}

cf_status cf_workspace_check(void* workspace, size_t ws_bytes, void* hip_stream) {
  try {
    if (!workspace) return CF_OK;   // no workspace: no cluster exchange ran
    if (ws_bytes < sizeof(unsigned)) return fail(CF_ERR_WORKSPACE, "workspace smaller than its error word");
    if (!aligned16(workspace)) return fail(CF_ERR_ALIGN, "workspace is not 16-byte aligned");
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    cf_status s = hip_status(hipStreamSynchronize(st), "stream synchronize");
    if (s != CF_OK) return s;
    unsigned err = 0;
    if ((s = hip_status(hipMemcpy(&err, workspace, sizeof(err), hipMemcpyDeviceToHost), "read error word")) != CF_OK)
      return s;
    if (err == 0) return CF_OK;
    const unsigned zero = 0;
    if ((s = hip_status(hipMemcpy(workspace, &zero, sizeof(zero), hipMemcpyHostToDevice), "clear error word")) != CF_OK)
      return s;
    return fail(CF_ERR_PEER_TIMEOUT,
                "a row-cluster wait for peer workgroups exceeded its bound; results written through this "
                "workspace since the last check are invalid (the word is now cleared)");
  } catch (...) {
    return fail(CF_ERR_HIP, "internal error");
  }
}

// Whether the MLP's hidden chunks may be split over workgroups (their partial
// products meeting in the workspace): the grid of 128-row blocks and chunks
// fits one generation of a 256-CU device.  The launch then chooses between the
// split form, 32-row workgroups and the wide form; otherwise one workgroup per
// row block runs all chunks and no workspace is needed.  Measured with the
// chunked whole form, 160-255 row blocks at K = 1024, N1 = 512: whole 42-53 us, split
// 51-62.  The rule depends on the arguments only.
static constexpr int64_t kMlpSplitMaxWorkgroups = 256;
static bool mlp_split(const cf_b2b_args* a) {
  return a->N1 > kMlpHidden &&
         a->batch * ((a->M + kMlpRows - 1) / kMlpRows) * (a->N1 / kMlpHidden) <= kMlpSplitMaxWorkgroups;
}

// Workspace of the split MLP: the fixed counter region (words [batch][row
// blocks] at its start), then fp32 partials [batch][cn][M][N2].  The counter
// region does not depend on the shape, so partials of one call never land
// where a later call of another shape expects zeroed counters.  Other B2B
// forms need none.
static size_t mlp_workspace(const cf_b2b_args* a) {
  if (!a || a->struct_size != sizeof(cf_b2b_args) || a->mid != CF_MID_RELU_BIAS || a->M <= 0 || a->batch <= 0 ||
      !mlp_split(a))
    return 0;
  const int64_t cn = a->N1 / kMlpHidden;
  return kMlpCounterBytes + (size_t)(a->batch * cn * a->M * a->N2 * 4);
}
static_assert(kMlpSplitMaxWorkgroups <= kMlpMaxRowBlocks, "split MLP counters");

// Workspace of attention with split keys: the counter region, then for every
// (batch entry, 32-query block) and part 32 rows of fp32 O and (max, sum).
static size_t attention_workspace(const cf_b2b_args* a) {
  if (!a || a->struct_size != sizeof(cf_b2b_args) || a->mid != CF_MID_SOFTMAX || a->M <= 0 || a->batch <= 0 ||
      a->N1 <= 0 || a->K != a->N2 || !b2b_attention_supported((int)std::min<int64_t>(a->K, 1 << 30)))
    return 0;
  const AttentionForm f = attention_form(a->M, a->batch, a->N1, (int)a->K);
  if (f.nz < 2) return 0;
  return kMlpCounterBytes + (size_t)((a->M + 31) / 32 * a->batch * f.nz) * 32 * (size_t)(a->K + 2) * 4;
}

size_t cf_b2bgemm_workspace(const cf_b2b_args* a) {
  try {
    return mlp_workspace(a) + attention_workspace(a);
  } catch (...) {
    return 0;
  }
}

cf_status cf_b2bgemm(const cf_b2b_args* a, void* workspace, size_t ws_bytes, void* hip_stream) {
  try {
    if (!a) return fail(CF_ERR_NULL, "args is NULL");
    if (a->struct_size != sizeof(cf_b2b_args))
      return fail(CF_ERR_STRUCT, "struct_size %zu != %zu", a->struct_size, sizeof(cf_b2b_args));
    if (a->dtype != CF_BF16) return fail(CF_ERR_DTYPE, "cf_b2bgemm computes in bf16 only");
    if (a->batch < 0 || a->batch > 65535 || a->M < 0 || a->K <= 0 || a->N1 <= 0 || a->N2 <= 0)
      return fail(CF_ERR_SHAPE, "need 0 <= batch <= 65535, M >= 0, K, N1, N2 > 0");
    if (a->M > (int64_t)1 << 30 || a->N1 > (int64_t)1 << 30) return fail(CF_ERR_SHAPE, "size exceeds 2^30");
    const bool ffn = a->mid == CF_MID_GELU_BIAS, mlp = a->mid == CF_MID_RELU_BIAS;
    if (!ffn && !mlp && a->mid != CF_MID_SOFTMAX) return fail(CF_ERR_UNSUPPORTED, "unknown mid op");
    if (a->out != CF_OUT_STORE && a->out != CF_OUT_BIAS_RESIDUAL_LN && a->out != CF_OUT_BIAS_RELU)
      return fail(CF_ERR_UNSUPPORTED, "unknown out op");
    if (a->out == CF_OUT_BIAS_RELU && !mlp) return fail(CF_ERR_UNSUPPORTED, "the output ReLU belongs to the MLP form");
    cf_status s;
    if (mlp) {
      if (a->w1_layout != CF_LAYOUT_NK || a->w2_layout != CF_LAYOUT_NK)
        return fail(CF_ERR_UNSUPPORTED, "MLP weights must be stored N x K (W1^T: N1 x K, W2^T: N2 x N1)");
      if (!b2b_mlp_supported((int)std::min<int64_t>(a->K, 1 << 30), (int)a->N1, (int)a->N2))
        return fail(CF_ERR_UNSUPPORTED, "MLP needs N2 = 128, N1 a multiple of %d, K a multiple of 64 and >= 128 "
                    "(K = %lld, N1 = %lld, N2 = %lld)", kMlpHidden, (long long)a->K, (long long)a->N1, (long long)a->N2);
      if (a->out == CF_OUT_BIAS_RESIDUAL_LN || a->R || a->gamma || a->beta)
        return fail(CF_ERR_UNSUPPORTED, "the MLP form stores O + b2 or ReLU(O + b2) only");
      if ((s = check_vec("b1", a->b1)) != CF_OK) return s;
      if (a->M > 0 && a->batch > 0) {
        const size_t need = mlp_workspace(a);
        if (need > 0) {
          if (!workspace) return fail(CF_ERR_WORKSPACE, "workspace of %zu bytes required (N1 split over workgroups)", need);
          if (ws_bytes < need) return fail(CF_ERR_WORKSPACE, "workspace %zu < %zu bytes", ws_bytes, need);
          if (!aligned16(workspace)) return fail(CF_ERR_ALIGN, "workspace is not 16-byte aligned");
        }
      }
    } else if (ffn) {
      if (a->w1_layout != CF_LAYOUT_NK || a->w2_layout != CF_LAYOUT_NK)
        return fail(CF_ERR_UNSUPPORTED, "FFN weights must be stored N x K (W1^T: N1 x K, W2^T: N2 x N1)");
      if (a->K != a->N2) return fail(CF_ERR_UNSUPPORTED, "FFN needs K == N2 = d (K = %lld, N2 = %lld)", (long long)a->K, (long long)a->N2);
      if (!b2b_ffn_supported((int)a->N1, (int)a->N2))
        return fail(CF_ERR_UNSUPPORTED, "FFN (N1, N2) = (%lld, %lld) not compiled", (long long)a->N1,
                    (long long)a->N2);
      if ((s = check_vec("b1", a->b1)) != CF_OK) return s;
    } else {
      if (a->w1_layout != CF_LAYOUT_NK || a->w2_layout != CF_LAYOUT_KN)
        return fail(CF_ERR_UNSUPPORTED, "attention: keys stored Lk x d (NK), values Lk x d (KN)");
      if (a->K != a->N2 || !b2b_attention_supported((int)a->K))
        return fail(CF_ERR_UNSUPPORTED, "attention head dim %lld not compiled (64, 128)", (long long)a->K);
      if (a->out != CF_OUT_STORE || a->b2 || a->R || a->b1)
        return fail(CF_ERR_UNSUPPORTED, "attention supports the plain store of O only");
      if (!std::isfinite(a->mid_scale) || !(a->mid_scale > 0.0f))
        return fail(CF_ERR_SHAPE, "mid_scale must be finite and > 0");
    }
    const bool empty = a->M == 0 || a->batch == 0;
    const int64_t w1_rows = a->N1, w1_cols = a->K;
    const int64_t w2_rows = (ffn || mlp) ? a->N2 : a->N1, w2_cols = (ffn || mlp) ? a->N1 : a->N2;
    if ((s = check_matrix("X", a->X, empty ? 0 : a->M, a->K, a->ldx, CF_BF16, true)) != CF_OK) return s;
    if ((s = check_matrix("W1", a->W1, empty ? 0 : w1_rows, w1_cols, a->ldw1, CF_BF16, true)) != CF_OK) return s;
    if ((s = check_matrix("W2", a->W2, empty ? 0 : w2_rows, w2_cols, a->ldw2, CF_BF16, true)) != CF_OK) return s;
    if ((s = check_matrix("O", a->O, empty ? 0 : a->M, a->N2, a->ldo, CF_BF16, true)) != CF_OK) return s;
    if ((s = check_matrix("R", a->R, empty ? 0 : a->M, a->N2, a->ldr, CF_BF16, false)) != CF_OK) return s;
    if ((s = check_vec("b2", a->b2)) != CF_OK || (s = check_vec("gamma", a->gamma)) != CF_OK ||
        (s = check_vec("beta", a->beta)) != CF_OK)
      return s;
    if (a->batch > 1)
      for (int64_t st : {a->sx, a->sw1, a->sw2, a->so, a->R ? a->sr : (int64_t)0})
        if (st < 0 || st % 8 != 0) return fail(CF_ERR_ALIGN, "batch strides must be non-negative multiples of 8");
    if (outputs_alias(a->O, {a->X, a->W1, a->W2, a->R})) return fail(CF_ERR_ALIAS, "O aliases an input");
    if (!(a->eps >= 0.0f)) return fail(CF_ERR_SHAPE, "eps must be >= 0");
    if (empty) return CF_OK;
    B2BParams p{};
    p.batch = (int)a->batch;
    p.M = (int)a->M;
    p.K = (int)a->K;
    p.N1 = (int)a->N1;
    p.N2 = (int)a->N2;
    p.X = reinterpret_cast<const uint16_t*>(a->X);
    p.ldx = a->ldx;
    p.sx = a->sx;
    p.W1 = reinterpret_cast<const uint16_t*>(a->W1);
    p.ldw1 = a->ldw1;
    p.sw1 = a->sw1;
    p.b1 = a->b1;
    p.mid_scale = a->mid_scale;
    p.W2 = reinterpret_cast<const uint16_t*>(a->W2);
    p.ldw2 = a->ldw2;
    p.sw2 = a->sw2;
    p.out_ln = a->out == CF_OUT_BIAS_RESIDUAL_LN;
    p.b2 = a->b2;
    p.R = reinterpret_cast<const uint16_t*>(a->R);
    p.ldr = a->ldr;
    p.sr = a->sr;
    p.gamma = a->gamma;
    p.beta = a->beta;
    p.eps = a->eps;
    p.O = reinterpret_cast<uint16_t*>(a->O);
    p.ldo = a->ldo;
    p.so = a->so;
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    if (mlp) {
      p.out_relu = a->out == CF_OUT_BIAS_RELU;
      p.cn = mlp_split(a) ? (int)(a->N1 / kMlpHidden) : 1;
      if (p.cn > 1) {
        char* b = reinterpret_cast<char*>(workspace);
        p.ws_count = reinterpret_cast<unsigned*>(b);
        p.ws_part = reinterpret_cast<float*>(b + kMlpCounterBytes);
      }
      return hip_status(launch_b2b_mlp(p, st), "B2B MLP launch");
    }
    if (!ffn) {
      // Without a workspace that holds the parts, a query block's keys stay in
      // one workgroup.
      const size_t need = attention_workspace(a);
      p.cn = 1;
      if (need > 0 && workspace && ws_bytes >= need && aligned16(workspace)) {
        char* b = reinterpret_cast<char*>(workspace);
        p.cn = attention_form(a->M, a->batch, a->N1, (int)a->K).nz;
        p.ws_count = reinterpret_cast<unsigned*>(b);
        p.ws_part = reinterpret_cast<float*>(b + kMlpCounterBytes);
      }
    }
    return hip_status(ffn ? launch_b2b_ffn(p, st) : launch_b2b_attention(p, st), "B2B launch");
  } catch (...) {
    return fail(CF_ERR_HIP, "internal error");
  }
}

}  // extern "C"
